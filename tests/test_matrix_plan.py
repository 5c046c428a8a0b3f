"""The launch plan of the few-query calls (host arithmetic), under AddressSanitizer + UBSan with plain g++."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2404_09336_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_matrix_plan_covers_every_position_and_fits_the_workspace(tmp_path):
    exe = tmp_path / "host_matrix_plan"
    csrc = os.path.join(ROOT, "paper_2404_09336_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-static-libasan", "-static-libubsan", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
           os.path.join(ROOT, "tests", "host_matrix_plan.cpp"), os.path.join(csrc, "span_host.cpp"), "-o", str(exe)]
    subprocess.run(cmd, check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    sys.stdout.write(res.stdout[-2000:])
    assert res.returncode == 0 and "host_matrix_plan: ok" in res.stdout


@pytest.mark.parametrize("batch,positions,q_len", [(1, 120, 16), (4, 100, 8), (4, 128, 64), (32, 700, 16)])
def test_calls_that_are_not_sliced_ask_for_no_workspace(batch, positions, q_len):
    tok = np.full(batch, positions)
    assert binding.span_workspace_bytes(binding.make_desc(batch, 32, 128, 1000, 1, 10, positions, 0, tokens_per_seq=tok, q_len=q_len)) == 0


@pytest.mark.parametrize("batch,heads,D,dtype,positions,q_len,want", [
    (1, 4, 128, 1, [16], 64, dict(workgroups=16, query_blocks=4, max_splits=1, partial_states=0)),       # tokens shared out
    (4, 32, 128, 1, [800] * 4, 8, dict(workgroups=512, query_blocks=1, max_splits=4, partial_states=4096)),
    (8, 32, 128, 1, [600] * 8, 2, dict(workgroups=512, query_blocks=1, max_splits=2, partial_states=1024)),
    (64, 32, 128, 1, [155] * 64, 16, dict(workgroups=2048, query_blocks=1, max_splits=1, partial_states=0)),
    (30, 32, 128, 0, [500] * 30, 64, dict(workgroups=1920, query_blocks=2, max_splits=1, partial_states=0)),
    (64, 32, 128, 1, [155] * 64, 2, dict(matrix_cores=False, workgroups=2048, max_splits=1, partial_states=0)),
    (1, 32, 128, 1, [8000], 1, dict(matrix_cores=False, workgroups=512, max_splits=16, partial_states=512)),
])
def test_launch_query_tells_what_the_call_runs(batch, heads, D, dtype, positions, q_len, want):
    """Against the launch rules by hand: 512 workgroups wanted, slices of 128 positions at least, 16 tokens per group."""
    tok = np.array(positions)
    off = np.arange(batch + 1, dtype=np.int32)
    d = binding.make_desc(batch, heads, D, 8192, dtype, batch, int(tok.max()), 0, tokens_per_seq=tok, q_len=q_len,
                          host_spans=(off, np.zeros(batch, np.int32), tok.astype(np.int32)))
    got = binding.span_launch_query(d)
    assert {k: got[k] for k in want} == want and got["launches"] == 1 and got["tokens"] == q_len
    assert got["max_splits"] * got["slice_tokens"] >= tok.max()
    if got["matrix_cores"]:
        assert not binding.span_plan_query(d)["runs_in_arguments"]


def test_launch_query_of_a_fixed_number_of_slices():
    """num_splits stands: as many tokens a launch as a slot holds states (16 for 16-bit rows of 128, else 4)."""
    for D, dtype, per in ((128, 1, 16), (64, 1, 4), (128, 0, 4)):
        got = binding.span_launch_query(binding.make_desc(2, 8, D, 1000, dtype, 10, 1000, 5, q_len=20))
        assert (got["launches"], got["tokens"], got["max_splits"]) == (-(-20 // per), per, 5)
        assert got["workgroups"] == 2 * 8 * 5 and got["partial_states"] == 2 * 8 * 5 * 20


@pytest.mark.parametrize("batch,heads,D,dtype,q_len,fit", [
    (4, 12, 128, 0, 4, 512), (2, 5, 128, 0, 16, 512), (24, 5, 128, 1, 46, 512), (3, 12, 64, 0, 60, 1024), (7, 5, 64, 1, 30, 1024),
    (5, 12, 128, 1, 9, 1024),
])
def test_slices_run_at_once(batch, heads, D, dtype, q_len, fit):
    """Heads that do not divide 512: no few workgroups more than run at once (two per CU for these instances, three or four for others)."""
    tok = np.linspace(300, 5000, batch).astype(np.int64)
    for kw in (dict(tokens_per_seq=tok), dict()):
        got = binding.span_launch_query(binding.make_desc(batch, heads, D, 5000, dtype, 10, 5000, 0, q_len=q_len, **kw))
        assert 0 < got["workgroups"] <= fit, (kw, got)


@pytest.mark.parametrize("q_len,dtype,D,batch,heads,positions,slices", [
    # one or two tokens: up to two batches of rows a wave in one slice, few pairs or many
    (1, 1, 128, 1, 8, 256, 1), (1, 1, 128, 1, 8, 257, 3), (1, 2, 64, 5, 32, 256, 1), (1, 0, 64, 2, 12, 256, 1), (1, 0, 128, 1, 8, 128, 1),
    (2, 1, 64, 2, 32, 256, 1), (2, 0, 64, 2, 32, 160, 1), (2, 0, 64, 2, 32, 161, 2),
    # fp32 rows of 128: slices of 64 where there is room for them
    (1, 0, 128, 1, 8, 129, 3), (1, 0, 128, 1, 32, 640, 10), (1, 0, 128, 4, 32, 640, 4),
    # level batches of one workgroup per CU
    (1, 1, 128, 8, 32, 768, 1), (1, 1, 128, 8, 32, 769, 2), (1, 1, 64, 8, 32, 384, 1), (1, 1, 64, 8, 32, 385, 2), (1, 1, 128, 7, 32, 700, 2),
    # a few tokens: whole up to three or four tiles, then one workgroup per CU at most
    (4, 1, 128, 3, 32, 256, 1), (16, 2, 64, 5, 32, 256, 1), (4, 0, 64, 2, 32, 192, 1), (4, 0, 64, 2, 32, 193, 2), (4, 0, 128, 2, 32, 129, 2),
    (16, 1, 128, 8, 32, 512, 1), (16, 1, 128, 8, 32, 513, 2), (4, 1, 128, 3, 32, 512, 2), (4, 1, 128, 3, 32, 800, 5),
])
def test_where_sequences_are_cut(q_len, dtype, D, batch, heads, positions, slices):
    """The rules for short sequences and for one workgroup per CU, at their lines; the workspace follows."""
    tok = np.full(batch, positions, np.int64)
    d = binding.make_desc(batch, heads, D, positions, dtype, batch, positions, 0, tokens_per_seq=tok, q_len=q_len)
    assert binding.span_launch_query(d)["max_splits"] == slices
    if q_len < 3:
        assert (binding.span_workspace_bytes(d) == 0) == (slices == 1)
