"""Kernels on both sides of the plan's lines (how conflicts are decided and by
which kernel) against the oracle: alone, together in a batch, and served."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_08373_amd import synth
from test_gpu_parity import L, _first_from_pairs, same_repair  # noqa: F401  (L is a fixture)
from test_plan_rules import UNRELATED, _one_array, _steps, _two_arrays, _walks

pytestmark = pytest.mark.gpu


def _with_barriers(km, every):
    """km with a slot's barrier after every so many points, and some of its
    accesses moved onto the others' words."""
    pts, slots = [], []
    for i, p in enumerate(km.points):
        d = {k: int(p[k]) for k in ("kind", "is_write", "array", "guard", "slot", "a", "b", "c")}
        if i % 5 == 3:
            d["c"] += 1
        pts.append(d)
        if i % every == every - 1 and len(slots) < 6:
            pts.append(dict(kind=1, slot=len(slots)))
            slots.append((len(slots) % 2, 0, 1 + len(slots)))
    return synth.make_kernel(km.blocks, km.threads, [(1 << 20, 1)], [(1, 0)], pts, slots)


def _edge_kernels():
    kms = []
    for P, T, B, step, apart in ((16, 64, 1, 2, 0), (31, 64, 1, 2, 0), (32, 64, 1, 2, 0),
                                 (22, 33, 4, 2, 0), (23, 33, 4, 2, 0), (16, 64, 64, 2, 2),
                                 (100, 33, 40, 128, 2), (128, 64, 3, 2, 64), (130, 64, 3, 2, 64)):
        km = _one_array(P, T, B, step, apart)
        kms += [km, _with_barriers(km, max(3, P // 6))]
    return kms


def test_packed_and_not(L):  # noqa: F811
    kms = _edge_kernels()
    for q, km in enumerate(kms):
        for kw in (dict(), dict(policy=1), dict(policy=1, solver=1)):
            g, o = L.repair(km, **kw), O.repair(km, **kw)
            assert same_repair(g, o), (q, kw, g, o)
        assert L.clauses(km, 0) == O.clauses(km, 0), q
    for order in (kms, kms[::-1], kms[1::2] + [synth.generate("plain-small", seed=4)] + kms[::2]):
        st, res = L.repair_batch(order)
        assert st == 0
        for km, r in zip(order, res):
            o = O.repair(km)
            assert all(r[k] == o[k] for k in ("status", "assign", "weight", "rounds", "n_clauses"))
    srv = L.Server(arena_bytes=4 << 30, max_resident=8)
    for q, km in enumerate(kms):
        assert srv.submit(km, q) == 0
    got = {}
    while len(got) < len(kms):
        srv.step()
        got.update((job, r) for job, r, _ in srv.poll())
    for q, km in enumerate(kms):
        o = O.repair(km)
        assert all(got[q][k] == o[k] for k in ("status", "assign", "weight", "rounds")), q


def test_long_walks_are_spread(L):  # noqa: F811
    # 8,256 pairs, each meeting 256 values: by the rows of the chip in both
    # calls, not by one workgroup in one of them (50 times the other's time)
    km = _one_array(128, 256, 256, 2, 2)
    times = []
    for call in (L.first_partners, L.repair):
        ms = []
        for _ in range(4):
            call(km)
            assert L.last_stats()["records"] == 0
            ms.append(L.last_stats()["ms_total"])
        times.append(min(ms))
    assert times[1] < 8 * times[0], times


@pytest.mark.parametrize("P,words,records", [
    (500, 0xFFFFFFF1, False), (2800, 0xFFFFFFF1, True), (700, (1 << 27) - 39, False),
    (700, (1 << 20) - 3, True),          # (a pair's range is 16 times the array)
    (3000, (1 << 20) - 3, True)])
def test_steps_that_share_no_divisor(L, P, words, records):  # noqa: F811
    km = _steps(P, 32, words, lambda i: 1 + 7919 * i, 2654435761)
    st, first, div = L.first_partners(km, 0)
    assert (L.last_stats()["records"] > 0) == records
    o = O.check(km, 0)
    assert st == 0 and div == o[2]
    assert (first.astype("uint64") == _first_from_pairs(o[1], km.n_points)).all()


def test_one_allowance_per_call(L):  # noqa: F811
    # each of the large ones in closed form alone, all of them by records
    # together, the small ones in closed form beside them
    kms = [_steps(2800, 32, (1 << 17) - q, lambda i: 1, 32 + (q == 3)) for q in range(11)]
    kms[2:2] = [synth.generate("plain-small", mode="planted", seed=s) for s in range(10)]
    assert L.repair(kms[0])["status"] == 0 and L.last_stats()["records"] == 0
    want = [O.repair(km) for km in kms]
    st, res = L.repair_batch(kms)
    assert st == 0 and L.last_stats()["records"] == 11 * 2800 * 32
    srv = L.Server(arena_bytes=4 << 30, max_resident=32)
    for q, km in enumerate(kms):
        assert srv.submit(km, q) == 0
    got = {}
    while len(got) < len(kms):
        srv.step()
        got.update((job, r) for job, r, _ in srv.poll())
    for q, o in enumerate(want):
        for r in (res[q], got[q]):
            assert all(r[k] == o[k] for k in ("status", "assign", "weight", "rounds", "n_clauses")), q


def test_no_sort_where_there_is_no_log(L):  # noqa: F811
    # what the statistics say of a call whose conflicts are all in closed form,
    # and of the same one by records, with every phase timed
    km = synth.generate("plain-large", mode="planted")
    old = L.set_tuning(L.TUNE_TIMING, 2), L.set_tuning(L.TUNE_RACE_ROUTE, 0)
    try:
        r0 = L.repair(km)
        s = L.last_stats()
        assert s["records"] == s["sort_launches"] == s["conf_launches"] == 0
        assert s["ms_gen"] == s["ms_sort"] == s["ms_sort_kernels"] == s["ms_sort_pass_max"] == 0
        assert s["ms_upload"] > 0 and s["ms_j0"] > 0 and s["ms_total"] > 0
        L.set_tuning(L.TUNE_RACE_ROUTE, 1)
        r1 = L.repair(km)
        s = L.last_stats()
        assert s["records"] > 0 and s["sort_launches"] == s["sort_passes"] > 0
        assert s["ms_gen"] > 0 and s["ms_sort"] > 0 and s["ms_sort_kernels"] > 0
        assert same_repair(r0, r1)
    finally:
        L.set_tuning(L.TUNE_TIMING, old[0])
        L.set_tuning(L.TUNE_RACE_ROUTE, old[1])


def _large_words(seed):
    """Points whose steps come up to the largest spans of 32-bit arithmetic, on
    arrays of up to 2^30 words; a third of them on words that others touch."""
    rng = np.random.default_rng(seed)
    T = int(round(2 ** rng.uniform(3, 10)))
    B = int(rng.integers(1, 9))
    W = int(round(2 ** rng.uniform(16, 30)))
    most = min((2**28 - 1) // (T - 1), W // 2)
    steps = [1, most, most - 1] + [max(1, int(most ** u)) for u in rng.random(3)]
    strides = [0, min(T, W // 2)] + [int(min(W // 2, 2**27 // max(1, B - 1)) ** u) for u in rng.random(2)]
    pts = []
    for i in range(60):
        if i % 12 == 11:
            pts.append(dict(kind=1, slot=i // 12))
            continue
        a, b = int(rng.choice(steps)) * int(rng.choice([1, -1])), int(rng.choice(strides))
        c = int(rng.integers(0, min(W, 2**31)))
        if i % 3 == 0:
            c = (int(rng.choice(steps)) * int(rng.integers(0, T))) % W
        pts.append(dict(kind=0, is_write=int(rng.random() < 0.6), a=a, b=b, c=c))
    slots = [(s % 2, 0, 1) for s in range(5)]
    return synth.make_kernel(B, T, [(W, 1)], [(1, 0)], pts, slots)


def test_large_words(L):  # noqa: F811
    closed = 0
    for seed in range(100):
        km = _large_words(seed)
        for x in (0, 5):
            g = L.check(km, x)[:4]
            closed += L.last_stats()["records"] == 0
            assert g == O.check(km, x), (seed, x)
        st, first, _ = L.first_partners(km, 0)
        assert (first.astype("uint64") == _first_from_pairs(O.check(km, 0)[1], km.n_points)).all()
        assert same_repair(L.repair(km), O.repair(km)), seed
    assert closed >= 80


@pytest.mark.parametrize("words", [(1 << 30) - 35, 0xFFFFFFF1])
def test_chains_of_64_bit_divisions(L, words):  # noqa: F811
    # in closed form in 32 bits, by records in 64
    km = _walks(words, (1007, 2003, 3001), UNRELATED)
    for q in range(1, 28, 2):
        km.points["c"][q] = km.points["c"][q - 1] + (q % 3)
    o = O.check(km, 0)
    assert L.check(km, 0)[:4] == o
    assert (L.last_stats()["records"] == 0) == (words < 2**30)
    assert same_repair(L.repair(km), O.repair(km))


@pytest.mark.parametrize("steps,arrays", [((1, 2), 1), ([104729 * (2 * q + 1) for q in range(8)], 2)],
                         ids=["short", "long"])
def test_beside_a_log(L, steps, arrays):  # noqa: F811
    # one array on the records, the other in closed form or beside it; alone and
    # in a batch, where one such kernel decides for all
    km = _two_arrays(steps)
    o = O.check(km, 0)
    assert L.check(km, 0)[:4] == o
    assert L.last_stats()["records"] == 24 * 71 * 100 * (1 + arrays)
    assert same_repair(L.repair(km), O.repair(km))
    kms = [synth.generate("plain-small", mode="planted", seed=s) for s in range(4)] + [km]
    st, res = L.repair_batch(kms + kms[::-1])
    assert st == 0
    for k, r in zip(kms + kms[::-1], res):
        want = O.repair(k)
        assert all(r[q] == want[q] for q in ("status", "assign", "weight", "rounds", "n_clauses"))
