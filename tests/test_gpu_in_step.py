"""Two workgroups of 16 tokens that share a slice's rows: slices long enough to be kept in step and shorter ones, whole windows of rows and a
remainder, with a causal limit, in the append form, and with rows that are not finite, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["plain", "table", "append", "wild"])
@pytest.mark.parametrize("dtype,batch,heads,rows", [("f32", 1, 8, 13000), ("f32", 2, 8, 3000), ("bf16", 1, 8, 30011), ("f16", 2, 8, 15000)])
def test_shared_slices(dtype, batch, heads, rows, form, gpu_device):
    """Tolerance as in test_gpu_matrix.py: 1e-5, ten times what the fp32 sums of unit-variance rows add up to."""
    q_len, L = 20, rows + 100
    cfg = DecodeConfig(99, "in-step", batch, heads, 128, L, L, dtype, 1e-5)
    ctx = np.full(batch, L, np.int32)
    counts = [rows - (rows // 3 if form == "table" and b else 0) for b in range(batch)]
    sp = SpanBatch.from_lists([[(3, 3 + n // 2), (L - (n - n // 2), L)] for n in counts], ctx)
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=41)
    if form == "wild":
        V[:, :, 50] = float("inf")
    q = draw_queries(cfg, q_len, device=gpu_device)
    pos = (ctx - q_len).astype(np.int32)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
    kw = dict(tokens_per_seq=sp.tokens_per_seq(), max_tokens=max(counts))
    if form == "append":
        k_new, v_new = (torch.randn(q.shape, device=gpu_device).to(K.dtype) for _ in range(2))
        call = span.prepare_span_decode_attn_multi_append(q, k_new, v_new, K, V, dev[3], *dev[:3], np.float32(cfg.scale), **kw)
    else:
        call = span.prepare_span_decode_attn_multi(q, K, V, *dev, np.float32(cfg.scale), **kw)
    launch = span.span_launch_query(call.desc)
    assert launch["query_blocks"] == 2 and launch["workgroups"] <= 512 and launch["workgroups"] % 16 == 0
    assert (2 * 128 * (4 if dtype == "f32" else 2) * launch["slice_tokens"] >= 400000) == (rows != 3000)
    out = call()
    torch.cuda.synchronize()
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale), dtype=dtype)
    got = out.cpu().numpy().astype(np.float64)
    ok = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), ok) and (ok.all() or form == "wild")
    err = float(np.abs(got[ok] - ref[ok]).max()) if ok.any() else 0.0
    print(f"[parity] in step {form} {dtype} {batch}x{heads} rows={rows}: {err:.3e}", flush=True)
    assert err <= cfg.tol
