"""Workgroups that a CU runs at once (csrc/ldpc_internal.h) against what an
MI355X was seen to run: a kernel of workgroups that wait 20 us, 256 k of them,
takes 20 us up to the k listed here."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SEEN = {  # wavefronts per SIMD: workgroups per CU for 1 to 16 wavefronts
    8: [32, 16, 10, 8, 5, 5, 4, 4, 3, 2, 2, 2, 2, 2, 2, 2],
    7: [28, 14, 9, 7, 5, 4, 3, 3, 2, 2, 2, 2, 1, 1, 1, 1],
    6: [24, 12, 8, 6, 4, 3, 3, 3, 2, 2, 2, 2, 1, 1, 1, 1],
    4: [16, 8, 5, 4, 2, 2, 2, 2, 1, 1, 1, 1, 1, 1, 1, 1],
}


def test_workgroups_per_cu(tmp_path):
    out = str(tmp_path / "occupancy_check")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2507_10424_amd", "csrc"),
           os.path.join(ROOT, "tests", "native", "occupancy_check.cpp"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        pytest.fail(res.stderr[-2000:])
    got = subprocess.run([out, *map(str, SEEN)], capture_output=True, text=True, check=True).stdout.splitlines()
    for line, (per_simd, want) in zip(got, SEEN.items()):
        assert [int(x) for x in line.split()] == want, per_simd
