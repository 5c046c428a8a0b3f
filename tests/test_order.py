"""The order in which whole sequences of unequal length go out: host arithmetic under AddressSanitizer + UBSan with plain g++, and on the
GPU against the fp64 oracle and bit for bit against the same sequences in another order."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from workloads import DecodeConfig, SpanBatch, draw_qkv, draw_queries, to_host_raw

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_unequal_sequences_go_out_level(tmp_path):
    exe = tmp_path / "host_order"
    csrc = os.path.join(ROOT, "paper_2404_09336_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-static-libasan", "-static-libubsan", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
           os.path.join(ROOT, "tests", "host_order.cpp"), os.path.join(csrc, "span_host.cpp"), "-o", str(exe)]
    subprocess.run(cmd, check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    sys.stdout.write(res.stdout[-2000:])
    assert res.returncode == 0 and "host_order: ok" in res.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,D,heads,batch,q_len", [("f32", 128, 16, 36, 48), ("f32", 128, 12, 36, 33),  # two query blocks
                                                       ("f16", 64, 200, 6, 5), ("bf16", 128, 300, 4, 20),    # heads that fill a turn
                                                       ("f16", 128, 8, 60, 59), ("f32", 64, 12, 41, 33),     # dealt, less than two turns
                                                       ("f16", 128, 8, 60, 1), ("f32", 64, 5, 90, 2)])       # dealt, on the vector units
def test_order_of_whole_sequences(dtype, D, heads, batch, q_len, gpu_device):
    """Tolerance as in test_gpu_matrix.py: fp32 sums of unit-variance rows, 1e-5 is ten times what they add up to."""
    L = 200
    cfg = DecodeConfig(96, "order", batch, heads, D, L, L, dtype, 1e-5)
    ctx = np.full(batch, L, np.int32)
    tokens = [60 + 37 * i % 131 for i in range(batch)]
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=31)
    q = draw_queries(cfg, q_len, device=gpu_device)
    pos = (ctx - q_len).astype(np.int32)

    def run(order):
        sp = SpanBatch.from_lists([[(1, 1 + tokens[i] // 3), (L - (tokens[i] - tokens[i] // 3), L)] for i in order], ctx)
        dev = [torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
        at = torch.as_tensor(list(order), device=gpu_device)
        out = span.span_decode_attn_multi(q[at].contiguous(), K[at].contiguous(), V[at].contiguous(), *dev, np.float32(cfg.scale),
                                          tokens_per_seq=sp.tokens_per_seq(), max_tokens=max(tokens))
        back = torch.empty_like(out)
        back[at] = out
        torch.cuda.synchronize()
        return back, sp

    a, sp = run(range(batch))
    b, _ = run(range(batch - 1, -1, -1))
    assert torch.equal(a, b)
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale),
                                 dtype=dtype)
    err = float(np.abs(a.cpu().numpy().astype(np.float64) - ref).max())
    print(f"[parity] order {dtype} D={D} {batch}x{heads} q_len={q_len}: {err:.3e}", flush=True)
    assert err <= cfg.tol
