"""The launch plan of the few-query calls (host arithmetic), under AddressSanitizer + UBSan with plain g++."""
import os
import subprocess
import sys

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
