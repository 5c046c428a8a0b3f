"""A workspace sized once, for the longest call of a shape, and calls planned for fewer positions (host arithmetic)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from paper_2404_09336_amd import binding
from workloads import DecodeConfig, SpanBatch, draw_qkv, to_host_raw


def _desc(batch, heads, D, dtype, positions, counts, intervals=10, size=None):
    given = {} if size is None else dict(workspace_ptr=4096, workspace_bytes=size)
    return binding.make_desc(batch, heads, D, 8000, dtype, intervals, positions, 0, tokens_per_seq=counts, **given)


def _used(batch, heads, D, desc):
    """Bytes that the launch lays out: counters, (m, l) pairs, states."""
    states = binding.span_launch_query(desc)["partial_states"]
    return 0 if states == 0 else (4 * batch * heads + 255) // 256 * 256 + (8 * states + 255) // 256 * 256 + 4 * D * states


@pytest.mark.parametrize("batch,heads,upwards", [(1, 32, 513), (2, 8, 2049), (2, 32, 513)])
@pytest.mark.parametrize("plan", ["counts", "bound", "dense"])
def test_half_size_slices_of_shorter_calls_give_way(batch, heads, upwards, plan):
    """fp32 rows of 128 of one token ask for up to twice the bytes where half-size slices have room, and run without them in what a longer call asks for."""
    desc = lambda n, size=None: _desc(batch, heads, 128, 0, n, np.full(batch, n, np.int64) if plan == "counts" else None, 0 if plan == "dense" else 10, size)  # noqa: E731
    gave_way = 0
    for longest in range(upwards, upwards + 1500, 128):
        size = binding.span_workspace_bytes(desc(longest))
        for n in range(40, longest, 61):
            assert _used(batch, heads, 128, desc(n, size)) <= size, (longest, n)
            gave_way += binding.span_workspace_bytes(desc(n)) > size
    assert gave_way > 0


def test_half_size_slices_where_the_workspace_holds_them():
    desc = lambda size: _desc(1, 32, 128, 0, 1000, np.full(1, 1000, np.int64), size=size)  # noqa: E731
    asked = binding.span_workspace_bytes(_desc(1, 32, 128, 0, 1000, np.full(1, 1000, np.int64)))
    assert [binding.span_launch_query(desc(size))["max_splits"] for size in (asked, asked - 1, 133376)] == [16, 8, 8]


@pytest.mark.parametrize("batch,heads,D,dtype,longest", [(8, 32, 128, 1, 768), (8, 32, 64, 2, 384), (23, 12, 128, 0, 700), (15, 32, 128, 2, 600)])
def test_unequal_lengths_where_level_ones_ask_for_nothing(batch, heads, D, dtype, longest):
    """256 to 511 pairs: a level batch is not sliced, and no shorter one has to be."""
    assert binding.span_workspace_bytes(_desc(batch, heads, D, dtype, longest, np.full(batch, longest, np.int64))) == 0
    ragged = np.linspace(longest // 4, longest, batch).astype(np.int64)
    assert binding.span_workspace_bytes(_desc(batch, heads, D, dtype, longest, ragged)) > 0
    for counts in (ragged, None):
        assert binding.span_launch_query(_desc(batch, heads, D, dtype, longest, counts, size=0))["max_splits"] == 1


@pytest.mark.parametrize("batch,dtype,D,longest,shortest", [(30, 2, 64, 307, 240), (11, 0, 128, 508, 200)])
def test_lengths_around_what_stays_whole(batch, dtype, D, longest, shortest):
    """Short sequences left whole make room for finer slices of the others: what the longest call asks for holds a coarser cut of unequal lengths."""
    gave_way = 0
    for counts_known in (True, False):
        size = binding.span_workspace_bytes(_desc(batch, 8, D, dtype, longest, np.full(batch, longest, np.int64) if counts_known else None))
        for seed in range(100):
            counts = np.random.default_rng(seed).integers(shortest, longest * 9 // 10, batch)
            assert _used(batch, 8, D, _desc(batch, 8, D, dtype, longest, counts, size=size)) <= size, seed
            gave_way += binding.span_workspace_bytes(_desc(batch, 8, D, dtype, longest, counts)) > size
    assert gave_way > 0


@pytest.mark.parametrize("batch,heads,D,dtype,longest,n", [(3, 5, 64, 1, 3013, 2061), (6, 2, 128, 0, 3498, 2591)])
def test_shorter_few_query_calls(batch, heads, D, dtype, longest, n):
    """Three tokens: what the plan for fewer positions must bring at least is in what a longer level call asks for, though that launches fewer slices."""
    desc = lambda n: binding.make_desc(batch, heads, D, 8000, dtype, 10, n, 0, tokens_per_seq=np.full(batch, n, np.int64), q_len=3)  # noqa: E731
    plan = binding.span_plan_query(desc(n))
    states = plan["workgroups"] * plan["queries_per_pass"]
    assert plan["max_splits"] > 1 and 256 + (8 * states + 255) // 256 * 256 + 4 * D * states <= binding.span_workspace_bytes(desc(longest))


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,dtype,lengths,size", [(1, 32, "f32", [1000], 150016), (8, 32, "f16", [700, 100, 650, 3, 512, 256, 257, 700], 0)])
def test_outputs_in_a_smaller_workspace(batch, heads, dtype, lengths, size, gpu_device):
    """Half-size slices that give way, and unequal sequences left whole: the oracle's outputs, and nothing written past the given bytes.  Tolerance as in
    test_gpu_matrix."""
    cfg = DecodeConfig(162, "reuse", batch, heads, 128, 1100, 1100, dtype, 1e-5)
    ctx = np.full(batch, cfg.max_len, np.int32)
    sp = SpanBatch.from_lists([[(0, n // 2), (n // 2 + 9, n + 9)] if n > 1 else [(0, n)] for n in lengths], ctx)
    q, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    call = span.prepare_span_decode_attn(q, K, V, *(dev(a) for a in (sp.offsets, sp.starts, sp.ends)), None, np.float32(cfg.scale),
                                         max_tokens=max(lengths), tokens_per_seq=np.asarray(lengths, np.int64))
    assert call.desc.workspace_bytes > size
    buffer = torch.full((size + 4096,), 0xff, dtype=torch.uint8, device=gpu_device)
    buffer[:min(size, 256)] = 0
    call.desc.workspace, call.desc.workspace_bytes = buffer.data_ptr(), size
    ref = oracle.span_attn(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, np.float32(cfg.scale), dtype=dtype)
    for _ in range(2):
        call.out.fill_(float("nan"))
        assert float(np.abs(call().cpu().numpy().astype(np.float64) - ref).max()) <= cfg.tol
    assert bool((buffer[size:] == 0xff).all())
