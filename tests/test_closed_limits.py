"""The closed-form conflict tests up to the limits of their 32-bit form, on the
CPU under the undefined-behaviour sanitizer: against joined accesses where these
are few, else the 32-bit forms against the 64-bit one."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("closed") / "closed_limits")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fsanitize=undefined",
                           "-fno-sanitize-recover=undefined", "-o", exe,
                           os.path.join(HERE, "closed_limits.cpp")])
    return exe


@pytest.mark.parametrize("seed", [21, 22, 23])
def test_up_to_the_limits(program, seed):
    r = subprocess.run([program, str(seed), "60000"], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, timeout=100)
    text = r.stdout.decode()
    assert r.returncode == 0, text
    n = [int(w) for w in text.replace(",", "").split() if w.isdigit()]
    # comparisons, conflicts, wrong, joined, few terms, near the span
    assert n[2] == 0 and n[0] > 100000 and min(n[1], n[3], n[4], n[5]) > 5000, text
