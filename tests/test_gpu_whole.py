"""Sequences around the lengths up to which they stay in one slice, and batches of one workgroup per CU, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu
TOL = 1e-5  # as in test_gpu_matrix: ten times what the sums' rounding adds up to here


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("f16", 64), ("f16", 128), ("bf16", 128)])
@pytest.mark.parametrize("q_len", [1, 2, 5, 40])
@pytest.mark.parametrize("lengths", [[128, 129, 64, 65], [160, 161, 192, 193], [256, 257, 255, 1], [512, 513, 400, 30]])
@pytest.mark.parametrize("plan", ["tokens", "bound"])
def test_lengths_around_the_lines(dtype, D, q_len, lengths, plan, gpu_device):
    cfg = DecodeConfig(141, "whole", 4, 3, D, 600, 600, dtype, TOL)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    cut = [n // 3 for n in lengths]
    sp = SpanBatch.from_lists([[(0, c), (c + 7, n + 7)] if c else [(0, n)] for n, c in zip(lengths, cut)], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    pos = (ctx - q_len).astype(np.int32)
    kw = dict(max_tokens=max(lengths), tokens_per_seq=sp.tokens_per_seq() if plan == "tokens" else None)
    lists = [dev(a) for a in (sp.offsets, sp.starts, sp.ends)]
    if q_len == 1:
        got = span.span_decode_attn(q[:, 0].contiguous(), K, V, *lists, None, np.float32(cfg.scale), **kw)[:, None]
    else:
        got = span.span_decode_attn_multi(q, K, V, *lists, dev(pos), np.float32(cfg.scale), **kw)
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale), dtype=dtype)
    assert float(np.abs(got.cpu().numpy().astype(np.float64) - ref).max()) <= TOL


@pytest.mark.parametrize("dtype,D,q_len,batch,positions,slices", [
    ("f16", 128, 1, 8, 768, 1), ("f16", 128, 1, 8, 769, 2), ("bf16", 64, 1, 8, 384, 1), ("bf16", 64, 1, 8, 385, 2), ("f32", 64, 1, 11, 700, 1),  # level batches
    ("f16", 128, 16, 8, 512, 1), ("f16", 128, 16, 8, 513, 2), ("f32", 64, 4, 8, 300, 1), ("f16", 128, 4, 3, 512, 3), ("f16", 128, 4, 7, 512, 1),  # a few tokens: one workgroup per CU
])
def test_batches_of_one_workgroup_per_cu(dtype, D, q_len, batch, positions, slices, gpu_device):
    """32 heads, the rules' lines: lengths a little unequal, as far as a level batch may be, and cut as the rules say."""
    cfg = DecodeConfig(142, "per-cu", batch, 32, D, 800, 800, dtype, TOL)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    lengths = [positions - 3 * (b % 3) for b in range(batch)]
    sp = SpanBatch.from_lists([[(1, n // 4), (n // 4 + 20, n + 21)] for n in lengths], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    lists, pos = [dev(a) for a in (sp.offsets, sp.starts, sp.ends)], (ctx - q_len).astype(np.int32)
    kw = dict(max_tokens=positions, tokens_per_seq=sp.tokens_per_seq())
    if q_len == 1:
        call = span.prepare_span_decode_attn(q[:, 0].contiguous(), K, V, *lists, None, np.float32(cfg.scale), **kw)
    else:
        call = span.prepare_span_decode_attn_multi(q, K, V, *lists, dev(pos), np.float32(cfg.scale), **kw)
    assert span.span_launch_query(call.desc)["max_splits"] == slices
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale), dtype=dtype)
    got = call().cpu().numpy().astype(np.float64).reshape(ref.shape)
    assert float(np.abs(got - ref).max()) <= TOL
