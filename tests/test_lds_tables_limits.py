"""What building the LDS-resident decoder's tables may cost the host
(csrc/lds_tables.hip): no memory beyond the graph's own size for one long
column, and no search where a frame's state cannot fit."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_10424_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("lds") / "lds_limits_check")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-I", CSRC, os.path.join(ROOT, "tests", "native", "lds_limits_check.cpp"),
           os.path.join(CSRC, "lds_tables.hip"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        pytest.fail(res.stderr[-2000:])
    return out


def run(checker, *args):
    res = subprocess.run([checker, *map(str, args)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout.split()


def test_one_long_column_takes_little_memory(checker):
    # 28,000 edges; the bins of the row and bit pass, the tables and lists are all below 10 MB, where bins for the
    # longest column at every slot would take 224
    assert float(run(checker, "column", 14000, 8000)[0]) < 20.0


def test_state_beyond_the_lds_is_refused_at_once(checker):
    built, limited = run(checker, "limit", 160 * 1024)  # 80,002 words of state
    assert (built, limited) == ("1", "0")
    assert run(checker, "limit", 4 * (16000 + 64000 + 2))[1] == "1"
    assert run(checker, "limit", 4 * (16000 + 64000 + 2) - 1)[1] == "0"
