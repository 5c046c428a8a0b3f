"""Ticket counters of few (batch, head) pairs, which spread over their 256 bytes of the workspace, and the merge of many slices."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu
TOL = 2e-3


def _dev(a, device):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device)


@pytest.mark.parametrize("pairs", [1, 3, 12, 21, 32, 33, 64, 65])
@pytest.mark.parametrize("q_len", [1, 2, 20])
def test_counters_stay_in_their_part_and_come_back_to_zero(pairs, q_len, gpu_device):
    """Only the counters' bytes are zeroed: the rest of the workspace holds NaN, and neither that nor a counter outside matters.  Nine slices of 144 positions,
    of which the last two are empty."""
    cfg = DecodeConfig(131, "tickets", 1, pairs, 64, 1300, 1300, "f16", TOL)
    ctx = np.full(1, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(0, 500), (610, 1110)]], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    pos = (ctx - q_len).astype(np.int32)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    kw = dict(max_tokens=1290, num_splits=9)
    need = span.span_plan_query(span.prepare_span_decode_attn_multi(q, K, V, *lists, np.float32(cfg.scale), **kw).desc)["workspace_bytes"]
    counters = (4 * pairs + 255) // 256 * 256
    buffer = torch.full((need + 256,), 0xff, dtype=torch.uint8, device=gpu_device)
    buffer[:counters] = 0
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale), dtype="f16")
    call = span.prepare_span_decode_attn_multi(q, K, V, *lists, np.float32(cfg.scale), workspace=buffer[:need], **kw)
    for _ in range(4):
        call.out.fill_(float("nan"))
        assert float(np.abs(call().cpu().numpy().astype(np.float64) - ref).max()) <= TOL
    assert not bool(buffer[:counters].any()) and bool((buffer[need:] == 0xff).all())


@pytest.mark.parametrize("dtype,D,q_len", [("f32", 64, 3), ("bf16", 64, 20), ("f16", 64, 64), ("f16", 128, 2), ("f32", 128, 16), ("f16", 128, 31), ("bf16", 128, 64)])
@pytest.mark.parametrize("slices", [4, 5, 7, 8, 9, 17])
def test_one_long_sequence_among_short_ones(dtype, D, q_len, slices, gpu_device):
    """Enough pairs for workgroups that serve all tokens, and all slices of one sequence: around four and eight of them, where the merge changes its step, and
    more.  Planned from the bound as well, where the short sequences' later slices are empty.  What is not zeroed holds NaN.  Tolerance as in test_gpu_matrix."""
    positions = 128 * slices - 40
    cfg = DecodeConfig(132, "long-among-short", 16, 8, D, positions + 64, positions + 64, dtype, 1e-5)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(0, positions)]] + [[(5 * b, 5 * b + 20)] for b in range(1, 16)], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    pos = np.full(cfg.batch, positions, np.int32)
    lists = [_dev(a, gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale), dtype=dtype)
    for counts in (sp.tokens_per_seq(), None):
        call = span.prepare_span_decode_attn_multi(q, K, V, *lists, np.float32(cfg.scale), max_tokens=positions, tokens_per_seq=counts)
        launched = span.span_launch_query(call.desc)["max_splits"]
        assert launched == slices if counts is not None else 2 <= launched <= 4
        buffer = torch.full((call.desc.workspace_bytes,), 0xff, dtype=torch.uint8, device=gpu_device)
        buffer[:512] = 0  # the counters of 128 pairs
        call.desc.workspace = buffer.data_ptr()
        call.out.fill_(float("nan"))
        assert float(np.abs(call().cpu().numpy().astype(np.float64) - ref).max()) <= 1e-5
