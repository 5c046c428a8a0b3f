"""The matrix-core kernel of the few-query calls at the sizes where its tiling can go wrong, against the fp64 oracle.

Tolerance: with fp32 outputs of unit-variance V rows the error of the sums is about 2^-23 times a few units, and of the
weights 2^-23 (fp32 rows, fp16 as two or three terms, bf16 as three); 1e-5 is some ten times what that adds up to over the rows
attended here, and a thousand times less than one wrong row of the largest span would show."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from test_gpu_multi_append import run_case as run_append
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _dev(a, device):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device)


def _run(cfg, per_seq, q_len, device, q_pos="end", poison=None, **kw):
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists(per_seq, ctx)
    _, K, V = draw_qkv(cfg, ctx, device=device, seed=7 + q_len)
    q = draw_queries(cfg, q_len, device=device)
    pos = (ctx - q_len).astype(np.int32) if isinstance(q_pos, str) else q_pos
    if poison is not None:
        poison(K, V)
    code, _, _, tok = span.span_validate(sp.offsets, sp.starts, sp.ends, sp.ctx_lens)
    assert code == 0
    kw.setdefault("tokens_per_seq", tok)
    launched = kw.pop("launched", None)
    call = span.prepare_span_decode_attn_multi(q, K, V, _dev(sp.offsets, device), _dev(sp.starts, device), _dev(sp.ends, device),
                                               None if pos is None else _dev(pos, device), np.float32(cfg.scale),
                                               max_tokens=int(tok.max()), **kw)
    if launched is not None:
        launched.update(span.span_launch_query(call.desc))
    out = call()
    torch.cuda.synchronize()
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos,
                                 np.float32(cfg.scale), dtype=cfg.dtype)
    return out.cpu().numpy().astype(np.float64), ref


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [3, 16, 17, 32, 33, 64])
def test_tile_and_group_edges(dtype, D, q_len, gpu_device):
    """Token counts around the groups of 16; rows per wave around the tiles of 16 and 32 rows; the long sequences in slices
    of up to 261 rows (whole ones: test_large_slices).  Many pairs: a workgroup serves all tokens."""
    cfg = DecodeConfig(96, "matrix-edges", 10, 13, D, 2500, 2500, dtype, TOL)
    L = cfg.max_len
    spans = [1, 15, 16, 17, 61, 64, 65, 129, 700, 2347]
    per_seq = [[(5, 5 + n - q_len // 2), (L - q_len, L - q_len + q_len // 2)] if n > q_len else [(L - n, L)] for n in spans]
    got, ref = _run(cfg, per_seq, q_len, gpu_device)
    err = float(np.abs(got - ref).max())
    print(f"[parity] matrix edges {dtype} D={D} q_len={q_len}: {err:.3e}", flush=True)
    assert np.isfinite(got).all() and err <= TOL


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [20, 48, 64])
def test_query_blocks_share_a_slice(dtype, D, q_len, gpu_device):
    """Few pairs: several workgroups per slice, each for its own tokens, with one ticket counter per pair; repeated on
    one workspace (the counters must come back to zero), with and without the token counts."""
    cfg = DecodeConfig(97, "matrix-blocks", 2, 3, D, 1500, 1500, dtype, TOL)
    per_seq = [[(0, 700), (800, 1500)], [(3, 40), (100, 411), (1490, 1500)]]
    for kw in (dict(), dict(tokens_per_seq=None)):
        got, ref = _run(cfg, per_seq, q_len, gpu_device, **kw)
        assert np.isfinite(got).all() and float(np.abs(got - ref).max()) <= TOL
    ctx = np.full(2, 1500, np.int32)
    sp = SpanBatch.from_lists(per_seq, ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends)]
    call = span.prepare_span_decode_attn_multi(q, K, V, *lists, None, np.float32(cfg.scale), max_tokens=1400,
                                               tokens_per_seq=sp.tokens_per_seq())
    first = call().clone()
    for _ in range(20):
        call.out.fill_(float("nan"))
        assert torch.equal(call(), first)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
def test_non_finite_rows_reach_only_the_tokens_that_see_them(dtype, D, gpu_device):
    """V rows of +-Inf and NaN that tokens from the 20th on see: earlier tokens equal the oracle, later ones get exactly
    the oracle's infinities and NaNs (no 0 * Inf, and no Inf turned NaN by the terms of a 16-bit weight)."""
    cfg = DecodeConfig(98, "matrix-inf", 2, 4, D, 600, 600, dtype, TOL)
    q_pos = np.array([500, 520], np.int32)

    def poison(K, V):
        for b in range(2):
            p = int(q_pos[b])
            V[b, :, p + 20, ::2] = float("inf")
            V[b, :, p + 25, 1::4] = float("-inf")
            V[b, :, p + 25, 3::4] = float("nan")
            V[b, :, p + 30, ::4] = float("-inf")      # meets +inf: NaN

    got, ref = _run(cfg, [[(0, 100), (400, 600)], [(450, 600)]], 40, gpu_device, q_pos=q_pos, poison=poison)
    assert np.isfinite(ref[:, :20]).all() and np.isinf(ref).any() and np.isnan(ref).any()
    ok = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), ok) and float(np.abs(got[ok] - ref[ok]).max()) <= TOL
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("scale", [-0.2, 0.0])
def test_negative_and_zero_scales(dtype, scale, gpu_device):
    """The scale's sign goes into q and its size into the weight's exponent: both ends of that, with hidden rows."""
    cfg = DecodeConfig(99, "matrix-scale", 3, 4, 128, 400, 400, dtype, TOL)
    ctx = np.full(3, 400, np.int32)
    sp = SpanBatch.from_lists([[(0, 50), (300, 400)], [(390, 400)], [(7, 200)]], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, 6, device=gpu_device)
    pos = np.array([394, 393, 150], np.int32)
    got = span.span_decode_attn_multi(q, K, V, *(_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)), np.float32(scale),
                                      max_tokens=193, tokens_per_seq=sp.tokens_per_seq())
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos,
                                 np.float32(scale), dtype=dtype)
    assert float(np.abs(got.cpu().numpy().astype(np.float64) - ref).max()) <= TOL


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [2, 3, 16, 20, 40])
def test_light_rows_behind_heavy_rows_of_zeros(dtype, D, q_len, gpu_device):
    """Every 50th row outweighs the others by 2^19 .. 2^21 and holds zeros in V, so the output is the light rows' sum alone
    and shows the accuracy of their weights.  Bound on the relative 2-norm: an exponent of up to 21 carries two fp32
    roundings (of the score's scale and of the product), 21 ln 2 * 2 * 2^-24 = 1.7e-6; the step of an fp16 weight is 2^-39
    of the heaviest, half of it over 2^-20 is 1e-6 a row and independent from row to row; sums and exp2 a few 1e-7."""
    L = 1500
    cfg = DecodeConfig(105, "matrix-light-rows", 2, 3, D, L, L, dtype, TOL)
    ctx = np.full(cfg.batch, L, np.int32)
    sp = SpanBatch.from_lists([[(0, L)], [(0, 400), (410, L)]], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = torch.zeros_like(draw_queries(cfg, q_len, device=gpu_device))
    q[..., 0] = 16.0
    per_unit = 16.0 * cfg.scale / np.log(2.0)                    # powers of two per unit of K[..., 0]
    light = np.random.default_rng(D + q_len).uniform(-21, -19, size=K.shape[:3]) / per_unit
    K[..., 0] = _dev(light.astype(np.float32), gpu_device).to(K.dtype)
    K[:, :, 7::50, 0] = 0
    V[:, :, 7::50] = 0
    pos = (ctx - q_len).astype(np.int32)
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos,
                                 np.float32(cfg.scale), dtype=dtype)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    for kw in (dict(tokens_per_seq=sp.tokens_per_seq()), dict(num_splits=1)):
        got = span.span_decode_attn_multi(q, K, V, *lists, np.float32(cfg.scale), max_tokens=L, **kw).cpu().numpy().astype(np.float64)
        rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
        print(f"[parity] light rows {dtype} D={D} q_len={q_len} {sorted(kw)}: relative 2-norm {rel:.2e}", flush=True)
        assert rel <= 4e-6


@pytest.mark.parametrize("dtype,D", [("f32", 128), ("f16", 64), ("bf16", 128)])
@pytest.mark.parametrize("q_len", [3, 16, 64])
@pytest.mark.parametrize("counts", [True, False])
def test_any_workspace_from_the_least_on(dtype, D, q_len, counts, gpu_device):
    """The least that any burst of the shape needs (slots of queries_per_pass token states for the partition that
    span_plan_query reports) is enough for all of them; nothing past the given size is written."""
    cfg = DecodeConfig(106, "matrix-workspace", 4, 6, D, 1800, 1800, dtype, TOL)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(0, 900), (1000, 1800)], [(3, 400)], [(100, 1411), (1490, 1800)], [(0, 130)]], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    pos = (ctx - q_len).astype(np.int32)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    kw = dict(max_tokens=1700, tokens_per_seq=sp.tokens_per_seq() if counts else None)
    plan = span.span_plan_query(span.prepare_span_decode_attn_multi(q, K, V, *lists, np.float32(cfg.scale), **kw).desc)
    states = plan["workgroups"] * plan["queries_per_pass"]
    least = 256 + (states * 8 + 255) // 256 * 256 + states * D * 4
    assert plan["max_splits"] > 1 and least <= plan["workspace_bytes"]
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos,
                                 np.float32(cfg.scale), dtype=dtype)
    for size in sorted({least, (least + plan["workspace_bytes"]) // 2, plan["workspace_bytes"]}):
        buffer = torch.full((plan["workspace_bytes"] + 4096,), 0x5a, dtype=torch.uint8, device=gpu_device)
        buffer[:256] = 0                                                   # the ticket counters
        call = span.prepare_span_decode_attn_multi(q, K, V, *lists, np.float32(cfg.scale), workspace=buffer[:size], **kw)
        for _ in range(3):
            call.out.fill_(float("nan"))
            assert float(np.abs(call().cpu().numpy().astype(np.float64) - ref).max()) <= TOL
        assert bool((buffer[size:] == 0x5a).all()) and not bool(buffer[:256].any())
    call.desc.workspace_bytes = least - 1
    with pytest.raises(span.SpanAttnError):
        call()


@pytest.mark.parametrize("dtype,D,q_len", [("bf16", 128, 32), ("f16", 64, 9), ("f32", 128, 8)])
def test_a_row_that_is_not_finite_costs_about_one_more_pass(dtype, D, q_len, gpu_device):
    """The pass is taken again with the row apart, not every row of the slice singly (which took 6 to 17 times the clean
    call).  Bound: two passes, the second without loads ahead, and a few microseconds for the row: 4 times and 20 us."""
    cfg = DecodeConfig(107, "matrix-inf-time", 16, 16, D, 700, 700, dtype, TOL)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(0, 700)]] * cfg.batch, ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, (ctx - q_len).astype(np.int32))]
    call = span.prepare_span_decode_attn_multi(q, K, V, *lists, np.float32(cfg.scale), max_tokens=700, tokens_per_seq=sp.tokens_per_seq())

    def microseconds():
        for _ in range(5):
            call()
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                call()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3 / 20)
        return min(times)

    clean = microseconds()
    V[:, :, 699] = float("inf")
    poisoned = microseconds()
    print(f"[time] {dtype} D={D} q_len={q_len}: {clean:.1f} us clean, {poisoned:.1f} us with a row of Inf", flush=True)
    assert poisoned <= 4 * clean + 20


@pytest.mark.parametrize("dtype,D,q_len", [("f16", 128, 2), ("bf16", 64, 9), ("f32", 128, 20)])
def test_limits_far_below_and_beyond_the_cache(dtype, D, q_len, gpu_device):
    """Any int32 is a limit: the smallest ones show a token nothing (zero rows), the largest everything."""
    cfg = DecodeConfig(110, "matrix-limits", 5, 3, D, 200, 200, dtype, TOL)
    q_pos = np.array([-2**31, -2**31 + 70, -q_len, 1 - q_len, 2**31 - 1], np.int32)
    got, ref = _run(cfg, [[(0, 90), (95, 200)]] * 5, q_len, gpu_device, q_pos=q_pos)
    assert float(np.abs(got - ref).max()) <= TOL
    assert not got[:3].any() and got[3, -1].any() and got[4].any(axis=-1).all()


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [5, 20, 40])
def test_large_slices(dtype, D, q_len, gpu_device):
    """One slice per sequence (num_splits = 1) for 16, 32 and 64 tokens a workgroup: rows in quarters up to 383 positions a
    slice, from 384 on tiles dealt to the waves in turn, and beyond 2048 (512 a wave) more than one position window."""
    cfg = DecodeConfig(111, "matrix-large-slices", 6, 3, D, 4200, 4200, dtype, TOL)
    L = cfg.max_len
    for spans in ([353, 361, 367, 368, 17, 1], [383, 384, 385, 2047, 2048, 2049], [2060, 2081, 2112, 3000, 4099, 4195]):
        per_seq = [[(3, 3 + n // 3), (L - (n - n // 3), L)] if n > 2 else [(L - n, L)] for n in spans]
        launched = {}
        got, ref = _run(cfg, per_seq, q_len, gpu_device, num_splits=1, tokens_per_seq=None, launched=launched)
        assert launched["max_splits"] == 1 and launched["launches"] == 1 and max(spans) <= launched["slice_tokens"] < max(spans) + 16
        assert (launched["slice_tokens"] >= 384) == (max(spans) >= 384)
        assert launched["query_blocks"] == (2 if (q_len, D, dtype) == (40, 128, "f32") else 1)
        assert np.isfinite(got).all() and float(np.abs(got - ref).max()) <= TOL


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [17, 32, 40, 64])
def test_many_tokens_a_workgroup_with_rows_that_are_not_finite(dtype, D, q_len, gpu_device):
    """130 pairs: a workgroup serves 32 or 64 tokens.  +-Inf and NaN in V at the 10th token's row and later ones."""
    cfg = DecodeConfig(112, "matrix-inf-groups", 10, 13, D, 500, 500, dtype, TOL)
    q_pos = (400 + 3 * np.arange(10)).astype(np.int32)

    def poison(K, V):
        for b in range(10):
            p = int(q_pos[b]) + q_len
            V[b, :, p - 7, ::2] = float("inf")
            V[b, :, p - 5, 1::4] = float("-inf")
            V[b, :, p - 5, 3::4] = float("nan")
            V[b, :, p - 3, ::4] = float("-inf")       # meets +inf: NaN

    launched = {}
    got, ref = _run(cfg, [[(0, 100 + b), (350, 500)] for b in range(10)], q_len, gpu_device, q_pos=q_pos, poison=poison, launched=launched)
    assert launched["query_blocks"] == (2 if (dtype, D) == ("f32", 128) and q_len > 32 else 1)
    assert np.isfinite(ref[:, :q_len - 7]).all() and np.isinf(ref).any() and np.isnan(ref).any()
    ok = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), ok) and float(np.abs(got[ok] - ref[ok]).max()) <= TOL
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [17, 32, 64])
def test_many_tokens_a_workgroup_append_their_rows(dtype, D, q_len, gpu_device):
    """130 pairs, as above, in the append form: outputs against the oracle on the updated cache, the cache bit for bit."""
    cfg = DecodeConfig(113, "matrix-append-groups", 10, 13, D, 600, 600, dtype, TOL)
    pos = (300 + 17 * np.arange(10)).astype(np.int32)
    sp = SpanBatch.from_lists([[(0, 11), (40 + 3 * b, 150 + 7 * b), (int(pos[b]) - 20, int(pos[b]) + q_len)] for b in range(10)], pos + q_len)
    run_append(cfg, sp, pos, q_len, gpu_device, what=f"130 pairs {dtype} D={D} q_len={q_len}")


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f16", 64), ("bf16", 128)])
@pytest.mark.parametrize("q_len", [3, 16, 20])
def test_whole_sequences_dealt_by_length(dtype, D, q_len, gpu_device):
    """20 sequences x 32 heads, 301 .. 453 positions, are not sliced, more than one turn of 256 workgroups, and the longest
    is 20 % over the mean: the table that deals them longest first, each to the CUs that have the least (tests/host_order.cpp)."""
    cfg = DecodeConfig(114, "matrix-dealt", 20, 32, D, 512, 512, dtype, TOL)
    lengths = np.random.default_rng(5).permutation(301 + 8 * np.arange(20))
    launched = {}
    got, ref = _run(cfg, [[(0, int(n) - 100), (412, 512)] for n in lengths], q_len, gpu_device, launched=launched)
    assert launched["max_splits"] == 1 and launched["workgroups"] == 640 and launched["slice_tokens"] == 453
    assert np.isfinite(got).all() and float(np.abs(got - ref).max()) <= TOL
