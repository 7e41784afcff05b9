"""Host replay of the network kernels' reads of a tile's rows (csrc/net_index.h,
the functions the kernels call), with the tile heights, thread counts and input
widths the kernels are built for and every row count of a 64-patch row tile."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2008_11520_amd", "csrc")


def test_row_reads_in_bounds(tmp_path):
    exe = str(tmp_path / "net_rows_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "net_rows_check.cpp"),
                           "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr
