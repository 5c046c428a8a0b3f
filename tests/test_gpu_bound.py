"""Calls planned from a bound alone: the kernel shares every sequence's positions between its slices.  Sequences that attend far less than
the bound, one position or none, the appended row in any slice; span, dense, append, two and nine tokens; against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["span", "append", "dense", "dense_append", "two", "nine"])
@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f16", 128), ("bf16", 64)])
@pytest.mark.parametrize("batch,heads", [(1, 5), (11, 8), (70, 5)])
def test_shares_of_a_bound(form, dtype, D, batch, heads, gpu_device):
    """Tolerance 1e-5: fp32 sums of unit-variance rows (ten times what they add up to)."""
    L = 1700
    cfg = DecodeConfig(92, "bound", batch, heads, D, L, L, dtype, 1e-5)
    rng = np.random.default_rng(batch)
    ctx = np.array([(1700, 1, 63, 64, 65, 129, 1025, 500, 1600, 200, 2)[b % 11] for b in range(batch)], np.int32)
    if "dense" not in form and batch > 1:
        ctx[:] = np.maximum(ctx, 12)
    q, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=19)
    per_seq = [[(0, max(1, int(n) // 3))] + ([(int(n) - int(n) // 3, int(n))] if n >= 3 else []) for n in ctx]
    sp = SpanBatch.from_lists(per_seq, ctx)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    lists, scale = [dev(a) for a in (sp.offsets, sp.starts, sp.ends)], np.float32(cfg.scale)
    bound = dict(max_tokens=L if "dense" in form else int(sp.tokens_per_seq().max()))
    pos = np.array([rng.integers(0, n) for n in ctx], np.int32)
    k_new, v_new = (torch.randn((batch, heads, D), device=gpu_device).to(K.dtype) for _ in range(2))
    if form == "span":
        out = span.span_decode_attn(q, K, V, *lists, None, scale, **bound)
    elif form == "append":
        out = span.span_decode_attn_append(q, k_new, v_new, K, V, dev(pos), *lists, scale, **bound)
    elif form == "dense":
        out = span.dense_decode_attn(q, K, V, dev(ctx), scale, **bound)
    elif form == "dense_append":
        out = span.dense_decode_attn_append(q, k_new, v_new, K, V, dev(pos), dev(ctx), scale, **bound)
    else:
        tokens = 2 if form == "two" else 9
        q = draw_queries(cfg, tokens, device=gpu_device)
        first = (ctx - tokens).astype(np.int32)
        out = span.span_decode_attn_multi(q, K, V, *lists, dev(first), scale, **bound)
    torch.cuda.synchronize()
    raw = [to_host_raw(x) for x in (q, K, V)]
    if "dense" in form:
        ref = oracle.dense_attn(*raw, ctx, scale, dtype=dtype)
    elif form in ("span", "append"):
        ref = oracle.span_attn(*raw, sp.offsets, sp.starts, sp.ends, scale, dtype=dtype)
    else:
        ref = oracle.span_attn_multi(*raw, sp.offsets, sp.starts, sp.ends, first, scale, dtype=dtype)
    err = float(np.abs(out.cpu().numpy().astype(np.float64) - ref).max())
    print(f"[parity] bound {form} {dtype} D={D} batch={batch}: {err:.3e}", flush=True)
    assert err <= cfg.tol


@pytest.mark.parametrize("given", ["coarse", "between", "full"])
def test_the_workspace_of_the_coarse_cut_is_enough(given, gpu_device):
    """A bound's finer cut wants a larger workspace; one that holds the coarse cut is
    taken as before, and nothing past its size is written.  Tolerance as above."""
    cfg = DecodeConfig(93, "bound-workspace", 9, 16, 64, 4000, 4000, "f32", 1e-5)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    q, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=23)
    sp = SpanBatch.from_lists([[(5, 5 + 90 * (b + 1)), (3000, 3007 + 100 * b)] for b in range(cfg.batch)], ctx)
    lists = [torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device) for a in (sp.offsets, sp.starts, sp.ends)]
    kw = dict(max_tokens=cfg.max_len)
    full = span.span_plan_query(span.prepare_span_decode_attn(q, K, V, *lists, None, np.float32(cfg.scale), **kw).desc)
    states = 3 * cfg.batch * cfg.heads                      # (three slices a sequence)
    coarse = 768 + (states * 8 + 255) // 256 * 256 + states * cfg.head_dim * 4
    size = {"coarse": coarse, "between": full["workspace_bytes"] - 256, "full": full["workspace_bytes"]}[given]
    assert full["max_splits"] == 8 and coarse < size or given == "coarse"
    buffer = torch.full((full["workspace_bytes"] + 4096,), 0x5a, dtype=torch.uint8, device=gpu_device)
    buffer[:768] = 0                                        # the ticket counters
    call = span.prepare_span_decode_attn(q, K, V, *lists, None, np.float32(cfg.scale), workspace=buffer[:size], **kw)
    assert span.span_launch_query(call.desc)["max_splits"] == (8 if given == "full" else 3)
    ref = oracle.span_attn(*(to_host_raw(x) for x in (q, K, V)), sp.offsets, sp.starts, sp.ends, np.float32(cfg.scale), dtype="f32")
    for _ in range(3):
        call.out.fill_(float("nan"))
        assert float(np.abs(call().cpu().numpy().astype(np.float64) - ref).max()) <= cfg.tol
    assert bool((buffer[size:] == 0x5a).all()) and not bool(buffer[:768].any())
    call.desc.workspace_bytes = coarse - 1
    with pytest.raises(span.SpanAttnError):
        call()
