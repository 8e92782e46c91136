"""The plan's rules for how conflicts are decided, on the CPU: the lines are
drawn by the work that a kernel's pair tests are bounded by."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2011_08373_amd import build, synth

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "plan_facts.so")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip",
                           "--cuda-host-only", "-std=c++17", "-O1", "-shared", "-fPIC",
                           "-o", so, os.path.join(HERE, "plan_facts.cpp"),
                           os.path.join(build.CSRC, "librepair.cpp")])
    lib = C.CDLL(so)
    lib.plan_records.restype = lib.call_records.restype = C.c_longlong
    return lib


@pytest.fixture(scope="module")
def arg():
    import torch  # noqa: F401  (its HIP runtime is the one the library is to use)
    from paper_2011_08373_amd import librepair
    return librepair.KernelArg


def _one_array(P, T, B, step, apart):
    """P accesses of one array that never conflict: reads of even words and
    writes of odd ones, step apart per thread, their block strides differing
    by apart."""
    pts = [dict(kind=0, is_write=i & 1, a=step, b=apart * (i & 1), c=i & 1) for i in range(P)]
    return synth.make_kernel(B, T, [(1 << 20, 1)], [(1, 0)], pts, [])


@pytest.mark.parametrize("km,packed", [
    (_one_array(16, 64, 1, 2, 0), 1),
    (_one_array(31, 64, 1, 2, 0), 1),          # 496 pairs, one test each
    (_one_array(32, 64, 1, 2, 0), 0),          # 528
    (_one_array(22, 64, 4, 2, 0), 1),          # two views of 253 pairs
    (_one_array(23, 64, 4, 2, 0), 0),
    (_one_array(16, 64, 64, 2, 2), 0),         # few pairs, each meeting up to 127 values
    (_one_array(128, 256, 256, 128, 2), 0),
    (_one_array(0, 1, 1, 2, 0), 1),
], ids=lambda v: "%dx%dx%d" % (v.n_points, v.threads, v.blocks) if hasattr(v, "blocks") else str(v))
def test_packed_by_tests(plan, arg, km, packed):
    # one workgroup tests a packed kernel's pairs: few points are not enough
    # where each pair's test walks many values
    ka = arg(km)
    assert plan.plan_packed(ka.ref) == packed


def test_small_kernels_are_packed(plan, arg):
    for seed in range(20):
        ka = arg(synth.generate("plain-small", seed=seed))
        assert plan.plan_packed(ka.ref) == 1


def _steps(P, T, words, steps, gap):
    """P writes of T threads of one block, gap words apart, thread steps in turn."""
    pts = [dict(kind=0, is_write=1, a=steps(i), b=0, c=gap * i % (1 << 31)) for i in range(P)]
    return synth.make_kernel(1, T, [(words, 0)], [(1, 0)], pts, [])


@pytest.mark.parametrize("km,records", [
    (_steps(2800, 32, 1 << 17, lambda i: 1, 32), False),
    (_steps(2800, 32, 0xFFFFFFF0, lambda i: 1, 32), False),
    (_steps(2800, 32, 0xFFFFFFF0, lambda i: (1, 2, 4, -1)[i % 4], 128), False),
    # unrelated steps: twenty-odd steps of Euclid's algorithm a pair
    (_steps(2800, 32, 0xFFFFFFF1, lambda i: 1 + 7919 * i, 2654435761), True),
    (_steps(3900, 1024, 0xFFFFFFF1, lambda i: 1 + 397 * i, 2654435761), True),
    (_steps(500, 32, 0xFFFFFFF1, lambda i: 1 + 7919 * i, 2654435761), False),
    (_steps(3000, 32, (1 << 27) - 39, lambda i: 1 + 1399 * i, 2654435761), True),
], ids=["one", "one-64-bit", "related", "unrelated", "unrelated-wide", "few", "unrelated-32-bit"])
def test_steps_that_share_no_divisor(plan, arg, km, records):
    ka = arg(km)
    assert (plan.plan_records(ka.ref) > 0) == records


def _walks(words, steps, strides):
    """28 accesses of 100 threads and 40 blocks: pairs of different block strides
    are gone through block by block."""
    pts = [dict(kind=0, is_write=i & 1, a=steps[i % len(steps)], b=strides[i % len(strides)],
                c=1000 * i) for i in range(28)]
    return synth.make_kernel(40, 100, [(words, 1)], [(1, 0)], pts, [])


UNRELATED = (171417, -254275, 309673)


@pytest.mark.parametrize("km,records", [
    (_walks((1 << 30) - 35, (1007, 2003, 3001), UNRELATED), False),
    (_walks(0xFFFFFFF1, (1007, 2003, 3001), UNRELATED), True),
    (_walks(0xFFFFFFF1, (1,), (0, 100)), False),
], ids=["32-bit", "unrelated-64-bit", "related-64-bit"])
def test_chains_of_64_bit_divisions(plan, arg, km, records):
    # one lane's chain of tests, each several 64-bit divisions where the steps
    # share no divisor
    ka = arg(km)
    assert (plan.plan_records(ka.ref) > 0) == records


def _two_arrays(steps):
    """24 accesses each of a global array whose pairs meet too many values for any
    bound, and of a shared one of the given thread steps; 71 threads, 100 blocks."""
    far = [104729 * (2 * q + 1) for q in range(8)]
    pts = []
    for i in range(24):
        pts.append(dict(kind=0, is_write=i & 1, array=0, a=far[i % 8],
                        b=(188366, -458584, 157627)[i % 3], c=37 * i))
        pts.append(dict(kind=0, is_write=i & 1, array=1, a=steps[i % len(steps)], b=71, c=41 * i))
    return synth.make_kernel(100, 71, [(1 << 20, 1), (1 << 20, 0)], [(1, 0)], pts, [])


@pytest.mark.parametrize("steps,arrays", [((1, 2), 1), ([104729 * (2 * q + 1) for q in range(8)], 2)],
                         ids=["short", "long"])
def test_beside_a_log(plan, arg, steps, arrays):
    # where the launches of a log are made anyway, chains of tests beside it are
    # worth no more than the records they save
    ka = arg(_two_arrays(steps))
    assert plan.plan_records(ka.ref) == 24 * 71 * 100 * (1 + arrays)


def test_one_allowance_per_call(plan, arg):
    # what the closed form may cost beyond the records stands for the launches
    # of a log, which a batch makes once
    from paper_2011_08373_amd import librepair as L
    one = _steps(2800, 32, 1 << 17, lambda i: 1, 32)          # 3.9M pairs
    small = synth.generate("plain-small", seed=1)

    def records(kms):
        b = L.BatchArg(kms)
        over = C.c_double(0)
        n = plan.call_records(b.ptrs, b.n, C.byref(over))
        return n, over.value

    n, over = records([one])
    assert n == 0 and 3.5e6 < over < 4e6
    assert records([one] * 10 + [small] * 50)[0] == 0
    assert records([one] * 11 + [small] * 50) == (11 * 2800 * 32, 11 * over)
    # arrays of less cost first
    half = _steps(1400, 32, 1 << 17, lambda i: 1, 32)
    assert records([one] * 10 + [half] * 8)[0] == 10 * 2800 * 32
    big = [synth.generate_batch(n=128, mode="planted", seed=s) for s in (3, 4)]
    assert [records(kms)[0] for kms in big] == [0, 0]         # ordinary batches
