"""The walk over a sequence's interval list at the sizes where its chunks of 64 and the table of chunk counts (256 chunks)
begin and end, one-token and few-query calls, against the fp64 oracle.  Tolerance: fp32 sums over at most 25k rows of unit
variance, 1e-5 (a single wrong row of the longest list moves an output by about 1e-4)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [2, 63, 64, 65, 128, 129, 1000, 16384, 16449])
@pytest.mark.parametrize("how", ["counts", "bound", "splits"])
def test_list_lengths_around_the_chunks(count, how, gpu_device):
    L = 3 * count + 40
    cfg = DecodeConfig(101, "intervals", 2, 3, 64, L, L, "f32", 1e-5)
    rng = np.random.default_rng(count)
    lens = rng.integers(1, 3, size=count)
    starts = np.concatenate(([0], np.cumsum(lens + 1)[:-1])) + rng.integers(0, 2)
    a = [(int(s), int(s + n)) for s, n in zip(starts, lens)]
    sp = SpanBatch.from_lists([a, [(1, 2), (5, 30)]], np.full(2, L, np.int32))
    tok = sp.tokens_per_seq()
    q1, K, V = draw_qkv(cfg, sp.ctx_lens, device=gpu_device)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).to(gpu_device) for x in (sp.offsets, sp.starts, sp.ends)]
    kw = {"counts": dict(tokens_per_seq=tok), "bound": dict(), "splits": dict(num_splits=5)}[how]
    scale = np.float32(cfg.scale)
    raw = [to_host_raw(x) for x in (K, V)]
    got = span.span_decode_attn(q1, K, V, *dev, None, scale, max_tokens=int(tok.max()), **kw)
    ref = oracle.span_attn(to_host_raw(q1), *raw, sp.offsets, sp.starts, sp.ends, scale, dtype="f32")
    assert float(np.abs(got.cpu().numpy() - ref).max()) <= 1e-5
    q = draw_queries(cfg, 3, device=gpu_device)
    got = span.span_decode_attn_multi(q, K, V, *dev, None, scale, max_tokens=int(tok.max()), **kw)
    ref = oracle.span_attn_multi(to_host_raw(q), *raw, sp.offsets, sp.starts, sp.ends, None, scale, dtype="f32")
    assert float(np.abs(got.cpu().numpy() - ref).max()) <= 1e-5
