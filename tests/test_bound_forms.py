"""One-token calls planned from a bound alone: what the queries say is what each form launches."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09336_amd as span
from paper_2404_09336_amd import binding
from workloads import DecodeConfig, draw_qkv, to_host_raw


@pytest.mark.parametrize("counts", [False, True])
def test_the_queries_tell_the_forms_apart(counts):
    """9 x 16 pairs, 4000 positions at most: eight slices of a span call, three of a dense one.  With counts the forms are planned alike."""
    tok = np.full(9, 700, np.int64) if counts else None
    desc = lambda intervals: binding.make_desc(9, 16, 64, 4000, 0, intervals, 4000, 0, tokens_per_seq=tok)  # noqa: E731
    plans = {n: (span.span_plan_query(desc(n)), span.span_launch_query(desc(n)), binding.span_workspace_bytes(desc(n))) for n in (0, 10)}
    if counts:
        assert plans[0] == plans[10]
        return
    for intervals, splits in ((0, 3), (10, 8)):
        plan, launch, need = plans[intervals]
        states = splits * 9 * 16
        assert plan["max_splits"] == launch["max_splits"] == splits and plan["workgroups"] == launch["workgroups"] == states
        assert need == plan["workspace_bytes"] == 768 + (states * 8 + 255) // 256 * 256 + states * 64 * 4


@pytest.mark.gpu
def test_a_dense_call_writes_what_its_query_says(gpu_device):
    """The workspace that the query asks for is used, and nothing past it.  Tolerance 1e-5: fp32 sums of unit-variance rows (ten times what they add up to)."""
    cfg = DecodeConfig(97, "dense-bound", 9, 16, 64, 4000, 4000, "f32", 1e-5)
    ctx = np.array([4000, 1, 300, 129, 2500, 64, 1200, 3999, 1335], np.int32)
    q, K, V = draw_qkv(cfg, ctx, device=gpu_device, seed=29)
    need = binding.span_workspace_bytes(binding.make_desc(9, 16, 64, 4000, 0, 0, 4000, 0))
    buffer = torch.full((2 * need,), 0x5a, dtype=torch.uint8, device=gpu_device)
    buffer[:768] = 0                                        # the ticket counters
    call = span.prepare_dense_decode_attn(q, K, V, torch.from_numpy(ctx).to(gpu_device), np.float32(cfg.scale), max_tokens=4000, workspace=buffer[:need])
    ref = oracle.dense_attn(to_host_raw(q), to_host_raw(K), to_host_raw(V), ctx, np.float32(cfg.scale), dtype="f32")
    for _ in range(2):
        call.out.fill_(float("nan"))
        assert float(np.abs(call().cpu().numpy().astype(np.float64) - ref).max()) <= cfg.tol
    assert bool((buffer[need:] == 0x5a).all()) and not bool(buffer[:768].any()) and not bool((buffer[768:need] == 0x5a).all())
