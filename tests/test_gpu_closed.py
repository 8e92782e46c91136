"""First partners in closed form against the oracle and against the access
records, on the GPU: edges of the sizes and strides the closed form takes,
kernels whose arrays go both ways, and the repository's full-size parity with
every conflict decided from the records (RP_TUNE_RACE_ROUTE 1)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_08373_amd import synth
import bruteforce as BF
import test_gpu_full_size as full
import test_gpu_parity as parity
from test_gpu_parity import L, _first_from_pairs, same_repair  # noqa: F401  (L is a fixture)

pytestmark = pytest.mark.gpu


@pytest.fixture()
def records(L):  # noqa: F811
    old = L.set_tuning(L.TUNE_RACE_ROUTE, 1)
    yield
    L.set_tuning(L.TUNE_RACE_ROUTE, old)


def _random_kernel(rng, B, T, words, strides, P=70, glob=True, conds=True):
    pts = []
    for i in range(P):
        if rng.random() < 0.15:
            pts.append(dict(kind=2))
            continue
        pts.append(dict(kind=0, is_write=int(rng.random() < 0.4), array=int(rng.integers(0, 2)),
                        guard=int(rng.integers(0, 5)), a=int(rng.choice(strides[0])),
                        b=int(rng.choice(strides[1])), c=int(rng.integers(-9, 10))))
    guards = [(1, 0), (1, 0), (2, 1), (3, 2), (T + 1, T)]       # the last runs on no thread
    bg = [(1, 0), (2, 1), (3, 0), (1, 0), (1, 0)] if conds else None
    return synth.make_kernel(B, T, [(words, 1 if glob else 0), (words + 1, 1)], guards, pts, [],
                             block_guards=bg)


SHAPES = [
    # blocks, threads, words, thread strides, block strides
    (1, 1, 1, (0, 1), (0, 1)),
    (1, 64, 128, (1, 2, -1), (0,)),                    # 64, 65: one chunk of lanes and one more
    (3, 65, 64, (0, 1, -2, 64), (0, 65)),              # every address wraps
    (7, 33, 4096, (1, 3, -5), (33, 99)),
    (64, 31, 2039, (1, -1, 7), (0, 31, 62)),           # an odd array size
    (5, 40, 0xFFFFFFF0, (1, -1, 2**31 - 1, -2**31), (0, 40, -2**31)),   # 64-bit arithmetic
    (300, 20, 1 << 14, (1, 2), tuple(range(1, 40, 3))),  # more block strides than the rule lists
]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s[:3]) for s in SHAPES])
def test_first_partners_edges(L, shape):  # noqa: F811
    B, T, words, sa, sb = shape
    for seed in range(3):
        rng = np.random.default_rng(1000 * seed + T)
        km = _random_kernel(rng, B, T, words, (sa, sb), glob=seed != 1, conds=seed != 2)
        st, got, div = L.first_partners(km, 0)
        o = O.check(km, 0)
        assert st == 0 and div == o[2]
        assert (got.astype(np.uint64) == _first_from_pairs(o[1], km.n_points)).all(), seed


def _both_ways_kernel(seed):
    # the first array has more distinct block strides than the rule bounds, on
    # many blocks: its accesses get records; the second is closed
    rng = np.random.default_rng(seed)
    pts = []
    for i in range(36):
        if i % 3 == 2:
            pts.append(dict(kind=1, slot=i // 3))
        elif i % 3 == 0:
            pts.append(dict(kind=0, is_write=int(rng.random() < 0.5), array=0, a=1,
                            b=int(8 + 5 * i), c=int(rng.integers(-2, 3))))
        else:
            pts.append(dict(kind=0, is_write=int(rng.random() < 0.5), array=1,
                            a=int(rng.choice([1, -1, 2])), b=8, c=int(rng.integers(-2, 3))))
    slots = [(int(rng.integers(0, 2)), 0, int(rng.integers(1, 4))) for _ in range(12)]
    return synth.make_kernel(1500, 8, [(1 << 20, 1), (1 << 15, 1)], [(1, 0)], pts, slots)


def test_both_ways_in_one_kernel(L):  # noqa: F811
    for seed in range(3):
        km = _both_ways_kernel(seed)
        st, got, div = L.first_partners(km, 0)
        n = L.last_stats()["records"]
        assert n == 2 * 12 * km.blocks * km.threads          # both views of one array only
        assert (got.astype(np.uint64) == _first_from_pairs(O.check(km, 0)[1], km.n_points)).all()
        assert same_repair(L.repair(km), O.repair(km)), seed
    kms = [_both_ways_kernel(7), BF.tiny_kernel(np.random.default_rng(3)), _both_ways_kernel(8)]
    st, res = L.repair_batch(kms)
    assert st == 0
    for km, r in zip(kms, res):
        o = O.repair(km)
        assert all(r[k] == o[k] for k in ("status", "assign", "weight", "rounds", "n_clauses"))


def test_routes_agree_on_the_large_kernels(L):  # noqa: F811
    for name, mode in (("plain-large", "literal"), ("plain-large", "planted")):
        km = synth.generate(name, mode=mode)
        a = L.first_partners(km, 0)
        assert L.last_stats()["records"] == 0                         # no record was generated
        old = L.set_tuning(L.TUNE_RACE_ROUTE, 1)
        try:
            b = L.first_partners(km, 0)
            assert L.last_stats()["records"] > 0
        finally:
            L.set_tuning(L.TUNE_RACE_ROUTE, old)
        assert a[0] == b[0] == 0 and (a[1] == b[1]).all()


# the suites of the sort and of the first-partner scan, on the records
def test_records_scan_variants(L, records):  # noqa: F811
    for name in ("literal", "planted"):
        parity.test_scan_variants_full_size(L, "plain_large_" + name, name)
    parity.test_ragged_tiles(L)
    parity.test_edge_empty_and_degenerate(L)
    parity.test_block_conditions(L)


def test_records_sort_knobs(L, records):  # noqa: F811
    parity.test_pass_shapes_full_size(L)


def test_records_batched(L, records):  # noqa: F811
    full.test_batched_full_size(L, full._expected("batched"), "planted")
    parity.test_batch_many_kernels(L)
    parity.test_server_continuous_batching(L)


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s[:3]) for s in SHAPES])
def test_check_edges(L, shape):  # noqa: F811
    # every racing pair under random assignments, with barriers in between:
    # rows that end inside a 64-point word and rows that span several
    B, T, words, sa, sb = shape
    rng = np.random.default_rng(T)
    for P in (63, 64, 65, 130):
        km = _random_kernel(rng, B, T, words, (sa, sb), P=P)
        km.slots = np.zeros(3, synth.SLOT_DT)
        km.slots["level"], km.slots["weight"] = (0, 1, 0), 1
        for s, at in enumerate((P // 4, P // 2, P - 2)):
            km.points[at] = (1, 0, 0, 0, s, 0, 0, 0)
        for x in (0, 1, 2, 7):
            assert L.check(km, x)[:4] == O.check(km, x), (P, x)


def test_check_both_ways(L):  # noqa: F811
    for seed in range(2):
        km = _both_ways_kernel(seed)
        for x in (0, 0x155):
            assert L.check(km, x)[:4] == O.check(km, x), (seed, x)
            assert L.last_stats()["records"] > 0


def test_check_no_points(L):  # noqa: F811
    km = synth.make_kernel(2, 4, [(8, 1)], [(1, 0)], [], [])
    assert L.check(km, 0)[:4] == O.check(km, 0) and L.check(km, 0)[1] == []


@pytest.mark.parametrize("P", [1, 2, 63, 64, 65, 127, 128, 129, 200])
def test_packed_rows(L, P):  # noqa: F811
    # around the sizes where a job's rows are packed into the rounds kernel:
    # repairs alone, in a batch with larger kernels, and through the server
    kms = []
    for seed, (B, T, words, sa, sb) in enumerate(SHAPES[:5]):
        rng = np.random.default_rng(31 * P + seed)
        km = _random_kernel(rng, B, T, words, (sa, sb), P=P, glob=seed % 2 == 0, conds=seed > 2)
        n = min(4, P // 8)
        km.slots = np.zeros(n, synth.SLOT_DT)
        km.slots["level"], km.slots["weight"] = [q % 2 for q in range(n)], 1
        for s in range(n):
            km.points[(s + 1) * P // (n + 1)] = (1, 0, 0, 0, s, 0, 0, 0)
        kms.append(km)
        for kw in (dict(), dict(policy=1), dict(policy=1, solver=1)):
            g, o = L.repair(km, **kw), O.repair(km, **kw)
            assert same_repair(g, o), (seed, kw, g, o)
        for x in (0, 1):
            assert L.clauses(km, x) == O.clauses(km, x), (seed, x)
    kms.append(synth.generate("plain-small", seed=P))
    st, res = L.repair_batch(kms + [_random_kernel(np.random.default_rng(P), 2, 40, 64,
                                                   ((1, 2), (0, 40)), P=300)])
    assert st == 0
    for km, r in zip(kms, res):
        o = O.repair(km)
        assert all(r[k] == o[k] for k in ("status", "assign", "weight", "rounds", "n_clauses"))


def test_points_that_never_execute(L):  # noqa: F811
    # an array whose accesses run on no thread has no records on either route
    pts = [dict(kind=0, is_write=1, array=0, guard=1, a=1), dict(kind=1, slot=0),
           dict(kind=0, is_write=1, array=0, guard=1, a=1)]
    km = synth.make_kernel(2, 4, [(8, 1)], [(1, 0), (9, 8)], pts, [(0, 0, 1)])
    for route in (0, 1):
        old = L.set_tuning(L.TUNE_RACE_ROUTE, route)
        try:
            assert L.check(km, 0)[:4] == O.check(km, 0)
            assert same_repair(L.repair(km), O.repair(km))
            assert L.clauses(km, 0) == O.clauses(km, 0)
        finally:
            L.set_tuning(L.TUNE_RACE_ROUTE, old)


@pytest.mark.parametrize("P", [1, 7, 8, 9, 63, 64, 65, 129, 1030])
def test_pair_list_sizes(L, P):  # noqa: F811
    # full words, empty words and rows, a last group of rows that is not full
    for writes in (1.0, 0.02):
        rng = np.random.default_rng(P)
        pts = [dict(kind=0, is_write=int(rng.random() < writes), array=int(rng.random() < 0.1), a=0,
                    b=int(rng.integers(0, 2)), c=0) for _ in range(P)]
        km = synth.make_kernel(2, 3, [(4, 1), (4, 0)], [(1, 0)], pts, [])
        assert L.check(km, 0)[:4] == O.check(km, 0), writes
