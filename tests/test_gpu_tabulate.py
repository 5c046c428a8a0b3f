"""The rows' positions where marks of several intervals meet: intervals of one token between the rows of a wave, empty and reversed
intervals (which count as none), long ones across the windows of 64 rows, up to 64 in a list; small slices and large ones,
whose rows are dealt to the waves in units.  A wrong position shows as a wrong row: against the fp64 oracle on the cleaned lists."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu
L = 3000


def _lists(rng, dirty):
    """(list as given, list that counts) of sequences with 1 .. 64 intervals."""
    given, counted = [], []
    for lengths in ([1], [1] * 64, [1, 2, 3] * 20, [700] + [1] * 40 + [900, 1, 1, 64, 63, 65], [5] * 10 + [1500] + [1] * 30, [2] * 33 + [128, 256, 129],
                    [64] * 12, [300, 1, 1, 1, 300, 1, 1, 400]):
        at, mine, clean = 0, [], []
        for n in lengths:
            at += int(rng.integers(0, 3))
            if dirty and rng.random() < 0.4 and len(mine) + 2 + len(lengths) - len(clean) <= 64:
                mine.append((at, at - int(rng.integers(0, 4))))  # no position: empty or reversed
            mine.append((at, at + n))
            clean.append((at, at + n))
            at += n
        given.append(mine)
        counted.append(clean)
    return given, counted


@pytest.mark.parametrize("dirty", [False, True])
@pytest.mark.parametrize("dtype,D,q_len,splits", [("f16", 128, 1, 0), ("f16", 128, 1, 1), ("f32", 64, 1, 3), ("f32", 128, 1, 1), ("bf16", 64, 1, 1),
                                                  ("f32", 128, 2, 1), ("f16", 128, 9, 1), ("bf16", 64, 5, 1), ("f32", 64, 17, 2)])
def test_positions_of_meeting_intervals(dirty, dtype, D, q_len, splits, gpu_device):
    """Tolerance 1e-5: fp32 sums of unit-variance rows (ten times what they add up to; one wrong row of the longest span shows as 1e-3)."""
    given, counted = _lists(np.random.default_rng(7), dirty)
    cfg = DecodeConfig(94, "tabulate", len(given), 3, D, L, L, dtype, 1e-5)
    ctx = np.full(cfg.batch, L, np.int32)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=13)
    q = draw_queries(cfg, q_len, device=gpu_device)
    sp, ref_sp = SpanBatch.from_lists(given, ctx), SpanBatch.from_lists(counted, ctx)
    assert np.diff(sp.offsets).max() <= 64
    tok = ref_sp.tokens_per_seq()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)  # noqa: E731
    kw = dict(max_tokens=int(tok.max()), num_splits=splits)
    if splits == 0:
        kw["tokens_per_seq"] = tok
    out = span.span_decode_attn_multi(q, K, V, dev(sp.offsets), dev(sp.starts), dev(sp.ends), None, np.float32(cfg.scale), **kw)
    torch.cuda.synchronize()
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), ref_sp.offsets, ref_sp.starts, ref_sp.ends, None,
                                 np.float32(cfg.scale), dtype=cfg.dtype)
    err = float(np.abs(out.cpu().numpy().astype(np.float64) - ref).max())
    print(f"[parity] tabulate {dtype} D={D} q_len={q_len} splits={splits} dirty={dirty}: {err:.3e}", flush=True)
    assert err <= cfg.tol
