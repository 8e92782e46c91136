"""The closed-form conflict tests (csrc/closed.h) against the definition, on
the CPU: random pairs of access points over every kind of array size, stride,
guard and block condition, in 32-bit and 64-bit arithmetic, under the
undefined-behaviour sanitizer."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("closed") / "closed_pairs")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fsanitize=undefined",
                           "-fno-sanitize-recover=undefined", "-o", exe,
                           os.path.join(HERE, "closed_pairs.cpp")])
    return exe


@pytest.mark.parametrize("seed", [11, 12, 13])
def test_pairs_against_enumeration(program, seed):
    r = subprocess.run([program, str(seed), "15000"], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, timeout=100)
    text = r.stdout.decode()
    assert r.returncode == 0, text
    assert "0 wrong" in text and int(text.split()[0]) > 50000
