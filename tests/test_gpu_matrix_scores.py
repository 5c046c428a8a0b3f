"""Scores of any size through the few-query calls, against the fp64 oracle.

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


def _dev(a, device):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [2, 3, 16, 40])
def test_large_scores_of_both_signs(dtype, D, q_len, gpu_device):
    cfg = DecodeConfig(102, "matrix-large-scores", 2, 5, D, 700, 700, dtype, TOL)
    rng = np.random.default_rng(1000 + D + q_len)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(3, 40), (100, 700)], [(0, 300), (310, 333)]], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = torch.zeros_like(draw_queries(cfg, q_len, device=gpu_device))
    K[..., 1:] = 0
    K[..., 0] = _dev(1024 * (1 + rng.integers(0, 128, size=(cfg.batch, cfg.heads, cfg.max_len)) / 128.0), gpu_device).to(K.dtype)
    exponents = rng.integers(0, 15 if dtype == "f16" else 95, size=(cfg.batch, q_len, cfg.heads))
    exponents[0] = np.minimum(exponents[0], 14)   # (every type: the band in which a rounded reference goes wrong)
    q[..., 0] = _dev(rng.choice([-1, 1], size=exponents.shape) * rng.uniform(1, 2, size=exponents.shape) * 2.0 ** exponents, gpu_device).to(q.dtype)
    tok, scale, pos = sp.tokens_per_seq(), np.float32(1013.7), (ctx - q_len).astype(np.int32)
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, scale, dtype=dtype)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    for kw in (dict(tokens_per_seq=tok), dict(num_splits=1), dict(num_splits=5)):
        got = span.span_decode_attn_multi(q, K, V, *lists, scale, max_tokens=int(tok.max()), **kw)
        got = got.cpu().numpy().astype(np.float64)
        bad = ~(np.abs(got - ref) <= TOL)
        print(f"[parity] large scores {dtype} D={D} q_len={q_len} {sorted(kw)}: {bad.any(axis=-1).sum()} of {bad[..., 0].size} "
              f"outputs wrong", flush=True)
        assert not bad.any()
