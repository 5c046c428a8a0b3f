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
