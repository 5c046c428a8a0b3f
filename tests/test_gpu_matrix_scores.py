"""Scores of any size through the few-query and the append calls, against the fp64 oracle.

One component of q and K is not zero, so a score is one product and which rows share the maximum is exact; the scaled
scores (in powers of two of e) run from 2^20 to 2^34, and to 2^114 where the type holds them.  Rows below the maximum are
2^10 and more below it: weight 0.  So the answer is the mean of the V rows that share the maximum, with an error of a few
fp32 roundings of values up to 4.5 (2^-23 * 4.5 * 3 = 1.6e-6)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu
TOL = 2e-6
SCALE = np.float32(1013.7)


def _dev(a, device):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device)


def _draw(cfg, ctx, q_len, device):
    """Keys of 128 levels in [1024, 2048) and queries of either sign and 2^0 .. 2^94 (fp16: 2^14), all in component 0."""
    rng = np.random.default_rng(1000 + cfg.head_dim + q_len)
    _, K, V = draw_qkv(cfg, ctx, device=device)
    q = torch.zeros_like(draw_queries(cfg, q_len, device=device))
    K[..., 1:] = 0
    K[..., 0] = _dev(1024 * (1 + rng.integers(0, 128, size=K.shape[:3]) / 128.0), device).to(K.dtype)
    exponents = rng.integers(0, 15 if cfg.dtype == "f16" else 95, size=q.shape[:3])
    exponents[::2] = np.minimum(exponents[::2], 14)   # (every type: the band in which a rounded reference goes wrong)
    q[..., 0] = _dev(rng.choice([-1, 1], size=exponents.shape) * rng.uniform(1, 2, size=exponents.shape) * 2.0 ** exponents, device).to(q.dtype)
    return q, K, V


def _check(got, ref, what):
    bad = ~(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= TOL)
    print(f"[parity] large scores {what}: {bad.any(axis=-1).sum()} of {bad[..., 0].size} outputs wrong", flush=True)
    assert not bad.any()


def _multi(cfg, per_seq, q_len, device):
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists(per_seq, ctx)
    q, K, V = _draw(cfg, ctx, q_len, device)
    tok, pos = sp.tokens_per_seq(), (ctx - q_len).astype(np.int32)
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, SCALE, dtype=cfg.dtype)
    lists = [_dev(a, device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    for kw in (dict(tokens_per_seq=tok), dict(num_splits=1), dict(num_splits=5)):
        got = span.span_decode_attn_multi(q, K, V, *lists, SCALE, max_tokens=int(tok.max()), **kw)
        _check(got, ref, f"{cfg.dtype} D={cfg.head_dim} q_len={q_len} {sorted(kw)}")


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [2, 3, 16, 40])
def test_large_scores_of_both_signs(dtype, D, q_len, gpu_device):
    cfg = DecodeConfig(102, "matrix-large-scores", 2, 5, D, 700, 700, dtype, TOL)
    _multi(cfg, [[(3, 40), (100, 700)], [(0, 300), (310, 333)]], q_len, gpu_device)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
def test_large_scores_of_two_tokens_on_the_vector_units(dtype, D, gpu_device):
    """Two tokens of 16-bit rows and more than 32768 columns: the row that only the second token sees is merged by itself."""
    cfg = DecodeConfig(103, "vector-large-scores", 10, 64, D, 150, 150, dtype, TOL)
    _multi(cfg, [[(3, 40), (50 + b, 150)] for b in range(10)], 2, gpu_device)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dense", [False, True])
def test_large_scores_of_the_appended_row(dtype, D, dense, gpu_device):
    """One token: the appended row, merged by itself, shares the largest score with cached rows or is the largest alone."""
    cfg = DecodeConfig(104, "append-large-scores", 6, 9, D, 400, 400, dtype, TOL)
    ctx = np.arange(300, 306).astype(np.int32)
    q, K, V = _draw(cfg, ctx, 1, gpu_device)
    q, pos = q[:, 0].contiguous(), (ctx - 1).astype(np.int32)
    at = [torch.arange(6, device=gpu_device), slice(None), _dev(pos, gpu_device).long()]
    k_new, v_new = K[at[0], :, at[2]].clone(), V[at[0], :, at[2]].clone()
    k_new[:, :, 0] = torch.where(q[:, :, 0] > 0, 1024 * (1 + 127 / 128), 1024.0).to(K.dtype)  # the largest score there is
    k_new[::3, :, 0] *= torch.where(q[::3, :, 0] > 0, 2.0, 0.5).to(K.dtype)                     # beyond every cached one
    K[at[0], :, at[2]], V[at[0], :, at[2]] = k_new, v_new
    if dense:
        ref = oracle.dense_attn(to_host_raw(q), to_host_raw(K), to_host_raw(V), ctx, SCALE, dtype=dtype)
    else:
        sp = SpanBatch.from_lists([[(0, 100), (150, int(n))] for n in ctx], ctx)
        ref = oracle.span_attn(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, SCALE, dtype=dtype)
    for splits in (1, 3):
        if dense:
            got = span.dense_decode_attn_append(q, k_new, v_new, K, V, _dev(pos, gpu_device), _dev(ctx, gpu_device), SCALE, num_splits=splits)
        else:
            got = span.span_decode_attn_append(q, k_new, v_new, K, V, _dev(pos, gpu_device), _dev(sp.offsets, gpu_device),
                                               _dev(sp.starts, gpu_device), _dev(sp.ends, gpu_device), SCALE, num_splits=splits)
        _check(got, ref, f"append {dtype} D={D} dense={dense} splits={splits}")


def _random_multi(cfg, q_len, q_size, k_size, scale, device):
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(3, 40), (100, 300)], [(0, 300)], [(290, 300)]], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=device)
    q = draw_queries(cfg, q_len, device=device)
    K *= k_size
    q *= q_size
    pos = (ctx - q_len).astype(np.int32)
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, scale, dtype=cfg.dtype)
    lists = [_dev(a, device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    got = span.span_decode_attn_multi(q, K, V, *lists, scale, max_tokens=300, tokens_per_seq=sp.tokens_per_seq())
    return got.cpu().numpy().astype(np.float64), ref


@pytest.mark.parametrize("dtype,size", [("f32", 1e18), ("bf16", 1e18), ("f16", 1e3)])
@pytest.mark.parametrize("q_len", [2, 6])
def test_scale_zero_weighs_all_rows_alike_whatever_their_scores(dtype, size, q_len, gpu_device):
    """Scores of 10^37 (fp16: 10^7) and scale 0: the mean of the V rows each token sees, as with scores of 1."""
    cfg = DecodeConfig(108, "matrix-scale-0", 3, 4, 64, 300, 300, dtype, TOL)
    got, ref = _random_multi(cfg, q_len, size, size, np.float32(0), gpu_device)
    assert float(np.abs(got - ref).max()) <= TOL


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("scale", [1.2e-38, -1.2e-38])
@pytest.mark.parametrize("q_len", [2, 6, 20])
def test_fp32_scores_beyond_the_range_before_they_are_scaled(D, scale, q_len, gpu_device):
    """fp32 q.K of 10^39 under a scale that brings it back to some tens: the scale's size goes into q ahead of the product.
    Scores up to 200 with a sum's rounding of a few 2^-24: weights to 200 * 4 * 2^-24 = 5e-5, outputs (|V| <= 4.5) to 2e-4."""
    cfg = DecodeConfig(109, "matrix-tiny-scale", 3, 4, D, 300, 300, "f32", TOL)
    got, ref = _random_multi(cfg, q_len, 2e18, 1e20, np.float32(scale), gpu_device)
    assert np.isfinite(got).all() and float(np.abs(got - ref).max()) <= 2e-4
