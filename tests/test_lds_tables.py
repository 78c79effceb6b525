"""Host logic of the LDS-resident decoder's tables (csrc/lds_tables.hip),
checked on the CPU by a small C++ driver compiled with that source."""
import os
import subprocess

import numpy as np
import pytest

from paper_2507_10424_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_10424_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("lds") / "lds_tables_check")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-I", CSRC, os.path.join(ROOT, "tests", "native", "lds_tables_check.cpp"),
           os.path.join(CSRC, "lds_tables.hip"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        pytest.fail(res.stderr[-2000:])
    return out


def run(checker, H):
    lines = [f"{H.shape[0]} {H.shape[1]}"]
    for i in range(H.shape[0]):
        c = np.nonzero(H[i])[0]
        lines.append(" ".join([str(len(c))] + [str(x) for x in c]))
    res = subprocess.run([checker], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout.strip()


def codes():
    yield "paper shape", wl.regular_ldpc(8176, 1022, 4, 32, seed=2)
    yield "regular", wl.regular_ldpc(4096, 2048, 3, 6, seed=9)
    for seed, (n, m, dv, most) in enumerate([(65, 30, (1, 2, 3), 16), (500, 230, (0, 1, 2, 9), 32),
                                             (3000, 1400, (2, 3, 3, 4, 6), 16), (1000, 64, (1, 2, 3), 31)]):
        yield f"irregular {seed}", wl.random_irregular_code(n, m, seed=seed, dv_choices=dv, max_row_degree=most)
    H = wl.random_irregular_code(300, 100, seed=5, dv_choices=(1, 2, 3))
    H[::7] = 0  # rows of degree 0
    yield "empty rows", H


@pytest.mark.parametrize("name,H", list(codes()), ids=lambda v: v if isinstance(v, str) else "")
def test_tables(checker, name, H):
    out = run(checker, H).split()
    assert out[0] == "ok"
    # lanes on the busiest bank of a 32-lane gather: 3.5 for random slots, 1 at best
    assert float(out[1]) <= 3.0


def test_out_of_range_graphs_are_refused(checker):
    H = np.zeros((2, 40), np.uint8)
    H[0, :33] = 1  # a row of 33 edges
    H[1, :2] = 1
    assert run(checker, H) == "refused"
    H = np.zeros((1, 16385), np.uint8)  # more bits than 1,024 threads hold
    H[0, :4] = 1
    assert run(checker, H) == "refused"
