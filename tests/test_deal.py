"""The order in which a launch's slices go out: host arithmetic under AddressSanitizer + UBSan with plain g++, and on the GPU calls
whose slices are dealt, against the fp64 oracle and bit for bit against the same sequences in another order."""
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


def test_a_dealt_table_names_every_slice_once(tmp_path):
    exe = tmp_path / "host_deal"
    csrc = os.path.join(ROOT, "paper_2404_09336_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-static-libasan", "-static-libubsan", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
           os.path.join(ROOT, "tests", "host_deal.cpp"), os.path.join(csrc, "span_host.cpp"), "-o", str(exe)]
    subprocess.run(cmd, check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    sys.stdout.write(res.stdout[-2000:])
    assert res.returncode == 0 and "host_deal: ok" in res.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("lists", [False, True])
@pytest.mark.parametrize("dtype,D,q_len", [("f16", 128, 1), ("f32", 64, 1), ("f32", 128, 2), ("bf16", 128, 16), ("f16", 64, 9)])
@pytest.mark.parametrize("tokens", [[500, 500, 720, 720] * 2,                                # two slices each: the table is the deal's
                                    [60, 130, 900, 880, 300, 20, 700, 700, 410, 1],          # slices of all sizes, three turns
                                    [200 + 31 * (i % 7) for i in range(30)]])                # many sequences, few slices each
def test_dealt_calls(tokens, dtype, D, q_len, lists, gpu_device):
    """Tolerance as in test_gpu_matrix.py: fp32 sums of unit-variance rows, 1e-5 is ten times what they add up to."""
    cfg = DecodeConfig(95, "deal", len(tokens), 32, D, 1000, 1000, dtype, 1e-5)
    ctx = np.full(cfg.batch, cfg.max_len, np.int32)
    per_seq = [[(3, 3 + n // 2), (1000 - (n - n // 2), 1000)] if n > 1 else [(999, 1000)] for n in tokens]
    _, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=11)
    q = draw_queries(cfg, q_len, device=gpu_device)
    pos = (ctx - q_len).astype(np.int32)

    def run(order):
        sp = SpanBatch.from_lists([per_seq[i] for i in order], ctx)
        tok = np.array([tokens[i] for i in order])
        dev = [torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device) for a in (sp.offsets, sp.starts, sp.ends, pos)]
        at = torch.as_tensor(list(order), device=gpu_device)
        kw = dict(tokens_per_seq=tok, max_tokens=int(tok.max()))
        if lists:
            kw["host_spans"] = (sp.offsets, sp.starts, sp.ends)
        out = span.span_decode_attn_multi(q[at].contiguous(), K[at].contiguous(), V[at].contiguous(), *dev, np.float32(cfg.scale), **kw)
        back = torch.empty_like(out)
        back[at] = out
        torch.cuda.synchronize()
        return back, sp

    a, sp = run(range(cfg.batch))
    b, _ = run(range(cfg.batch - 1, -1, -1))
    assert torch.equal(a, b)
    ref = oracle.span_attn_multi(to_host_raw(q), to_host_raw(K), to_host_raw(V), sp.offsets, sp.starts, sp.ends, pos, np.float32(cfg.scale),
                                 dtype=cfg.dtype)
    err = float(np.abs(a.cpu().numpy().astype(np.float64) - ref).max())
    print(f"[parity] dealt {dtype} D={D} q_len={q_len} lists={lists}: {err:.3e}", flush=True)
    assert err <= cfg.tol


def test_the_finer_cut_of_a_bound_needs_its_workspace():
    """What the coarser cut asks for is enough: 9 x 16 pairs, 4000 positions at most, three slices where eight are wanted."""
    from paper_2404_09336_amd import binding
    desc = lambda size: binding.make_desc(9, 16, 64, 4000, 0, 10, 4000, 0, workspace_ptr=4096, workspace_bytes=size)  # noqa: E731
    full = span.span_plan_query(binding.make_desc(9, 16, 64, 4000, 0, 10, 4000, 0))
    assert full["max_splits"] == 8
    states = 3 * 9 * 16
    coarse = 768 + (states * 8 + 255) // 256 * 256 + states * 64 * 4
    splits = [span.span_launch_query(desc(size))["max_splits"] for size in (coarse, full["workspace_bytes"] - 1, full["workspace_bytes"])]
    assert splits == [3, 3, 8]
