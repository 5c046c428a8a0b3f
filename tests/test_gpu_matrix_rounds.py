"""17 to 32 tokens of 16-bit rows of 128: one group of 16 rows a tile up to 512 workgroups, two in larger launches.  Sequences around
the tiles of 16 and 32 rows per wave on both sides of the line, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("q_len", [17, 32])
@pytest.mark.parametrize("batch,heads", [(32, 16), (27, 19)])  # 512 and 513 workgroups
def test_both_tiles(dtype, q_len, batch, heads, gpu_device):
    """Tolerance as in test_gpu_matrix.py: 1e-5, ten times what the fp32 sums of unit-variance rows add up to."""
    L = 240
    cfg = DecodeConfig(91, "rounds", batch, heads, 128, L, L, dtype, 1e-5)
    ctx = np.full(batch, L, np.int32)
    lengths = [(33, 63, 64, 65, 127, 128, 129, 200, 239)[b % 9] for b in range(batch)]
    sp = SpanBatch.from_lists([[(0, n - 32), (L - 32, L)] if n > 32 else [(L - n, L)] for n in lengths], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=23)
    q = draw_queries(cfg, q_len, device=gpu_device)
    pos = (ctx - q_len).astype(np.int32)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    call = span.prepare_span_decode_attn_multi(q, K, V, *dev, np.float32(cfg.scale), tokens_per_seq=sp.tokens_per_seq(), max_tokens=max(lengths))
    assert span.span_launch_query(call.desc)["workgroups"] == batch * heads
    out = call()
    torch.cuda.synchronize()
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale),
                                 dtype=dtype)
    err = float(np.abs(out.cpu().numpy().astype(np.float64) - ref).max())
    print(f"[parity] tiles {dtype} q_len={q_len} {batch}x{heads}: {err:.3e}", flush=True)
    assert err <= cfg.tol
