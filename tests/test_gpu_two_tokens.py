"""Two tokens of 16-bit rows on the vector units (more than 32768 (batch, head) x head_dim columns; fewer run on the matrix
cores): slicing, limits, rows that only the second token sees, the append form and the hand-over, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2404_09336_amd as span
from test_gpu_multi import _dev, _poison, check, oracle_multi, run_multi
from test_gpu_multi_append import run_case as run_append
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries

pytestmark = pytest.mark.gpu
SHAPES = [(128, 33), (64, 52)]   # (head_dim, heads) of 10 sequences: 42240 and 33280 columns


def _case(dtype, D, heads, device, seed=0):
    cfg = DecodeConfig(115, "two-tokens", 10, heads, D, 900, 900, dtype, 1e-5)
    ctx = np.full(10, 900, np.int32)
    rng = np.random.default_rng(40 + D + seed)
    sp = SpanBatch.from_lists([[(0, 17), (60 + 11 * b, 150 + 60 * b), (900 - int(rng.integers(20, 90)), 900)] for b in range(10)], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=device)
    return cfg, sp, draw_queries(cfg, 2, device=device), K, V


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D,heads", SHAPES)
def test_slicings_and_hidden_rows(dtype, D, heads, gpu_device):
    """Level, uniform and forced slicings; the limits inside the last interval, inside the middle one and near the end, with
    NaN in K and +-Inf in V past them."""
    cfg, sp, q, K, V = _case(dtype, D, heads, gpu_device)
    q_pos = np.array([885, 100, 888, 70, 889, 230, 300, 885, 150, 886], np.int32)
    for b in range(10):
        lo, hi = sp.offsets[b], sp.offsets[b + 1]
        _poison(K, V, b, [p for s, e in zip(sp.starts[lo:hi], sp.ends[lo:hi]) for p in range(s, e) if p > q_pos[b] + 1], gpu_device)
    ref = oracle_multi(cfg, sp, q, K, V, q_pos)
    assert np.isfinite(ref).all()
    for kw in (dict(), dict(tokens_per_seq=None), dict(num_splits=2, tokens_per_seq=None), dict(num_splits=5, tokens_per_seq=None)):
        check(run_multi(cfg, sp, q, K, V, q_pos, gpu_device, **kw), ref, cfg.tol, f"two tokens {dtype} D={D} {kw}")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D,heads", SHAPES)
def test_a_row_only_the_second_token_sees(dtype, D, heads, gpu_device):
    cfg, sp, q, K, V = _case(dtype, D, heads, gpu_device, seed=1)
    q_pos = np.full(10, 890, np.int32)
    V[:, :, 891] = float("inf")
    ref = oracle_multi(cfg, sp, q, K, V, q_pos)
    for kw in (dict(tokens_per_seq=sp.tokens_per_seq()), dict(num_splits=3)):
        got = span.span_decode_attn_multi(q, K, V, *(_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, q_pos)),
                                          np.float32(cfg.scale), max_tokens=int(sp.tokens_per_seq().max()), **kw)
        got = got.cpu().numpy().astype(np.float64)
        check(got[:, 0], ref[:, 0], cfg.tol, f"band row {dtype} D={D} {sorted(kw)}")
        assert not np.isfinite(ref[:, 1]).any() and not np.isfinite(got[:, 1]).any()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D,heads", SHAPES)
def test_append(dtype, D, heads, gpu_device):
    cfg = DecodeConfig(116, "two-tokens-append", 10, heads, D, 700, 700, dtype, 1e-5)
    pos = (300 + 30 * np.arange(10)).astype(np.int32)
    sp = SpanBatch.from_lists([[(0, 11), (40 + 3 * b, 150 + 7 * b), (int(pos[b]) - 20, int(pos[b]) + 2)] for b in range(10)], pos + 2)
    run_append(cfg, sp, pos, 2, gpu_device, what=f"two tokens {dtype} D={D}")
    run_append(cfg, sp, pos, 2, gpu_device, seed=3, what=f"two tokens {dtype} D={D}, 3 slices", num_splits=3)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D,heads", SHAPES)
def test_sliced_calls_are_bit_reproducible(dtype, D, heads, gpu_device):
    """One workspace, 1024 calls back to back: a stale state in the hand-over would show as a differing output."""
    cfg, sp, q, K, V = _case(dtype, D, heads, gpu_device)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends)]
    call = span.prepare_span_decode_attn_multi(q, K, V, *lists, None, np.float32(cfg.scale), max_tokens=int(sp.tokens_per_seq().max()), num_splits=3)
    plan = span.span_launch_query(call.desc)
    assert plan["max_splits"] == 3 and not plan["matrix_cores"]
    want = call().clone()
    check(want.cpu().numpy().astype(np.float64), oracle_multi(cfg, sp, q, K, V, None), cfg.tol, f"two tokens {dtype} D={D}, 3 slices")
    for _ in range(16):
        for _ in range(64):
            call()
        assert torch.equal(call.out, want)
        call.out.fill_(float("nan"))
