"""Launches of few workgroups keep twice the rows in flight per wave: slices around one and two such batches, the append form with the new
row in any batch, dense and span form, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, to_host_raw

pytestmark = pytest.mark.gpu
L = 700


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("f16", 64), ("f16", 128), ("bf16", 128)])
@pytest.mark.parametrize("n", [1, 15, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300])
@pytest.mark.parametrize("form", ["span", "dense", "append", "lists"])
def test_slices_around_the_batches(dtype, D, n, form, gpu_device):
    """Tolerance 1e-5: fp32 sums of unit-variance rows (ten times what they add up to)."""
    cfg = DecodeConfig(93, "wide", 2, 3, D, L, L, dtype, 1e-5)
    ctx = np.full(2, n, np.int32)
    q, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=17 + n)
    sp = SpanBatch.from_lists([[(0, n)], [(0, max(1, n // 2))]], ctx)
    tok = ctx.astype(np.int64) if form == "dense" else sp.tokens_per_seq()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    lists, scale = [dev(a) for a in (sp.offsets, sp.starts, sp.ends)], np.float32(cfg.scale)
    kw = dict(max_tokens=n, tokens_per_seq=tok)
    if form == "dense":
        out = span.dense_decode_attn(q, K, V, dev(ctx), scale, **kw)
        ref = oracle.dense_attn(to_host_raw(q), to_host_raw(K), to_host_raw(V), ctx, scale, dtype=dtype)
    else:
        if form == "append":
            pos = np.array([n - 1, n // 4], np.int32)
            k_new, v_new = (torch.randn((2, 3, D), device=gpu_device).to(K.dtype) for _ in range(2))
            out = span.span_decode_attn_append(q, k_new, v_new, K, V, dev(pos), *lists, scale, **kw)
        else:
            if form == "lists":
                kw["host_spans"] = (sp.offsets, sp.starts, sp.ends)
            else:
                kw["num_splits"] = 1
            out = span.span_decode_attn(q, K, V, *lists, None, scale, **kw)
        torch.cuda.synchronize()
        ref = oracle.span_attn(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, scale, dtype=dtype)
    err = float(np.abs(out.cpu().numpy().astype(np.float64) - ref).max())
    assert err <= cfg.tol
