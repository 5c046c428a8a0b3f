"""Attended K rows that are not finite: NaN reaches the output whichever way a sequence is cut, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu
TOL = 1e-5  # as in test_gpu_matrix: ten times what the sums' rounding adds up to here


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f16", 128)])
@pytest.mark.parametrize("form", ["span", "dense", "two tokens", "five tokens"])
@pytest.mark.parametrize("num_splits", [1, 5, 40])
def test_scores_that_are_not_finite_reach_the_output(dtype, D, form, num_splits, gpu_device):
    """One attended K row of a sequence holds NaN, one of another overflows the score of the first token to +Inf, one of a third to -Inf (no weight).
    520 positions in one slice, in five, and in 33, which is more than the merge's threads take at once; 300 pairs of 128 and fp32 rows keep two tokens off
    the matrix cores."""
    cfg = DecodeConfig(161, "scores", 5, 60, D, 520, 520, dtype, TOL)
    n = {"two tokens": 2, "five tokens": 5}.get(form, 1)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(0, 520)]] * cfg.batch, ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, n, device=gpu_device)
    inf = torch.full_like(q[:, 0], float("inf"))
    overflow = torch.where(q[:, 0] >= 0, inf, -inf)  # [batch, heads, D]
    K[0, :, 203] = float("nan")
    K[1, :, 7] = overflow[1]
    K[2, :, 519] = -overflow[2]
    K[3, ::2, 300] = float("nan")                    # some heads only
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    kw = dict(max_tokens=520, num_splits=num_splits)
    scale, raw = np.float32(cfg.scale), [to_host_raw(x) for x in (q, K, V)]
    if form == "dense":
        got = span.dense_decode_attn(q[:, 0].contiguous(), K, V, dev(ctx), scale, **kw)[:, None]
    elif form == "span":
        got = span.span_decode_attn(q[:, 0].contiguous(), K, V, *(dev(a) for a in (sp.offsets, sp.starts, sp.ends)), None, scale, **kw)[:, None]
    else:
        call = span.prepare_span_decode_attn_multi(q, K, V, *(dev(a) for a in (sp.offsets, sp.starts, sp.ends)), None, scale, **kw)
        assert span.span_launch_query(call.desc)["matrix_cores"] is (n == 5)
        got = call()
    got = got.cpu().numpy().astype(np.float64)
    ref = oracle.span_attn_multi(*raw, sp.offsets, sp.starts, sp.ends, None, scale, dtype=dtype)
    bad = np.isnan(ref)
    assert bad[0].all() and bad[1, 0].all() and not bad[2, 0].any() and bad[3, :, ::2].all() and not bad[3, :, 1::2].any() and not bad[4].any()
    assert np.array_equal(np.isnan(got), bad) and float(np.abs(got - ref)[~bad].max()) <= TOL
