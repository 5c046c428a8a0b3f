"""Few-query calls whose interval lists lie off the place the kernel fetches them from ahead of their range, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu
TOL = 1e-5  # as in test_gpu_matrix: ten times what the sums' rounding adds up to here


# Intervals per sequence: all even; lists of 63, 64 and 65 in one and in several sequences; one sequence with nearly all of them (the others' lists are
# outside the window of 64 around the mean, before or after it); none at all in some; means around 64.
COUNTS = [[1], [63], [64], [65], [3, 3, 3, 3], [40, 24], [60, 1, 1, 2], [1, 2, 1, 61], [100, 1, 1, 1], [1, 1, 1, 100], [0, 0, 5, 90], [80, 0, 0, 1],
          [64, 64, 64], [64, 65, 64], [63, 64, 64], [1] * 70 + [60], [60] + [1] * 70]


@pytest.mark.parametrize("counts", COUNTS, ids=lambda c: "-".join(map(str, c[:4])) + f"x{len(c)}")
@pytest.mark.parametrize("spare", [0, 37])
@pytest.mark.parametrize("dtype,q_len", [("f16", 5), ("f32", 9)])
def test_lists_around_the_window(counts, spare, dtype, q_len, gpu_device):
    cfg = DecodeConfig(151, "window", len(counts), 2, 64, 512, 512, dtype, TOL)
    rng = np.random.default_rng(sum(counts) + len(counts))
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    lists = []
    for n in counts:
        cuts = np.sort(rng.choice(500, 2 * n, replace=False))
        lists.append([(int(a), int(b)) for a, b in zip(cuts[::2], cuts[1::2])])
    sp = SpanBatch.from_lists(lists, ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device)
    q = draw_queries(cfg, q_len, device=gpu_device)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    junk = rng.integers(-2**31, 2**31, (2, spare)).astype(np.int32)  # entries of the lists that no sequence owns
    starts, ends = (np.concatenate([a, j]) for a, j in zip((sp.starts, sp.ends), junk))
    pos = (ctx - q_len).astype(np.int32)
    got = span.span_decode_attn_multi(q, K, V, dev(sp.offsets), dev(starts), dev(ends), dev(pos), np.float32(cfg.scale),
                                      max_tokens=max(1, int(sp.tokens_per_seq().max())))
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale), dtype=dtype)
    assert float(np.abs(got.cpu().numpy().astype(np.float64) - ref).max()) <= TOL
