"""Solve against the oracle where its routes change: clause sets of
contiguous runs (one path over the slots) and nearly so, equal and unequal
weights, widths around the enumeration limit and the 64-slot limit, more
clauses than fit LDS, and the greedy strategy on such constraint sets."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_08373_amd import synth
from test_gpu_parity import L, same_repair  # noqa: F401  (L is a fixture)

pytestmark = pytest.mark.gpu


def _runs(rng, S, n, longest, stray=0, neg=0):
    cl = []
    for _ in range(n):
        lo = int(rng.integers(0, S))
        hi = min(S - 1, lo + int(rng.integers(0, longest)))
        cl.append((((1 << (hi + 1)) - 1) & ~((1 << lo) - 1), 0))
    for _ in range(stray):          # slots apart: not a run
        cl.append(((1 << int(rng.integers(0, S))) | (1 << int(rng.integers(0, S))) |
                   (1 << int(rng.integers(0, S))), 0))
    for _ in range(neg):
        p, q = int(rng.integers(0, S)), int(rng.integers(0, S))
        cl.append(((1 << p) if p != q else 0, 1 << q))
    return cl


def _best_runs(cl, w, S):
    """(status, assign, weight) over positive runs of neighbouring slots: the
    cheapest ascending choice of slots that skips no whole run, keys as one
    integer (weight, count, mask)."""
    key = [(int(w[s]) << 71) + (1 << 64) + (1 << s) for s in range(S)]
    runs = [((p & -p).bit_length() - 1, p.bit_length() - 1) for p, _ in cl]
    best = []
    for s in range(S + 1):          # S: past the last slot
        need = max([lo for lo, hi in runs if hi < s], default=-1)
        best.append(min(([0] if need < 0 else []) + best[max(need, 0):s]) + (key[s] if s < S else 0))
    x = best[S] & ((1 << 64) - 1)
    return 0, x, sum(int(w[s]) for s in range(S) if (x >> s) & 1)


@pytest.mark.parametrize("S", [1, 2, 6, 7, 19, 20, 21, 22, 40, 63, 64])
def test_runs(L, S):  # noqa: F811
    for seed in range(12):
        rng = np.random.default_rng(100 * S + seed)
        wmax = (1, 2, 10, 2**31)[seed % 4]
        few = S <= 22            # the oracle's search is slow on wide sets
        stray, neg = ((0, 0, 1, 3)[seed % 4], seed % 3) if few else (0, 0)
        cl = _runs(rng, S, int(rng.integers(0, 3 * S + 2)), 2 + seed % 5, stray, neg)
        w = rng.integers(1, wmax + 1, size=S).tolist()
        g = L.min_barriers(cl, w, S)
        o = O.min_barriers(cl, w, S) if few else _best_runs(cl, w, S)
        if few and not stray and not neg:
            assert o == _best_runs(cl, w, S)
        assert g[0] == o[0] and (g[0] != 0 or g == o), (S, seed, cl, w, g, o)


@pytest.mark.parametrize("n", [1535, 1536, 1537, 5000])
def test_many_clauses(L, n):  # noqa: F811
    # (no clause of one slot, which would leave nothing to choose, up to the
    # 1,536 clauses of a component; past that every third slot is forced, and
    # the clauses still open are fewer)
    for seed, S in ((0, 12), (1, 30), (2, 64)):
        rng = np.random.default_rng(n + seed)
        cl = []
        while len(cl) < n:
            cl += [c for c in _runs(rng, S, n, 5, stray=n if seed == 0 else 0) if c[0] & (c[0] - 1)]
        cl = [cl[q] for q in rng.permutation(len(cl))[:n]]
        if n > 1536:
            cl = [(1 << s, 0) for s in range(0, S, 3)] + cl[(S + 2) // 3:]
        w = rng.integers(1, 9, size=S).tolist()
        o = O.min_barriers(cl, w, S) if seed == 0 else _best_runs(cl, w, S)
        assert L.min_barriers(cl, w, S) == o, (n, seed)


def test_greedy_and_exact_on_ragged_kernels(L):  # noqa: F811
    # weights that tie and that do not, both strategies, both policies
    cfg = synth.config("batched")
    for seed in range(12):
        rng = np.random.default_rng(5_000 + seed)
        c = dict(cfg)
        c.update(blocks=int(rng.integers(1, 4)), threads=int(rng.integers(33, 130)),
                 P=int(rng.integers(64, 300)), S=int(rng.integers(8, 40)), S_grid=3,
                 weight_mode=("baseline", "paper")[seed % 2])
        km = synth.planted_kernel(c, rng)
        for policy in (0, 1):
            o = O.repair(km, policy=policy)
            assert same_repair(L.repair(km, policy=policy), o), (seed, policy)
            g = L.repair(km, policy=policy, solver=1)
            assert (g["status"], g["assign"], g["weight"]) == (o["status"], o["assign"], o["weight"])


def _races(S, groups, between, wmax, seed):
    """groups of races with between random slots each, on words of their own;
    below three, one word written twice by either thread in turn instead."""
    rng = np.random.default_rng(seed)
    pts = [dict(kind=1, slot=s) for s in range(S)]

    def write(thread, word):
        return dict(kind=0, is_write=1, array=0, guard=1 + thread, a=0, b=0, c=word)

    for g in range(groups):
        gap = [dict(kind=1, slot=int(s)) for s in rng.choice(S, between, replace=False)]
        if between < 3:
            pts += [write(g % 2, 0), write(g % 2, 0)] + gap
        else:
            pts += [write(0, g)] + gap + [write(1, g)]
    slots = [(0, 0, int(w)) for w in rng.integers(max(1, wmax // 2), wmax + 1, size=S)]
    return synth.make_kernel(1, 2, [(groups, 0)], [(1, 0), (2, 0), (2, 1)], pts, slots)


# phi past the 128 clauses of a wave in the middle of the rounds, more racing
# rows than the rounds keep near (1,408), and weights around what is compared
# in 32 bits (2^24 for the greedy picks, a total of 2^25 for the path)
@pytest.mark.parametrize("S,groups,between,wmax", [
    (14, 300, 3, 3), (15, 400, 3, 3), (20, 1000, 2, 1), (30, 60, 3, 2**24 - 1), (30, 60, 3, 2**24),
    (30, 60, 3, 2**32 - 1)])
def test_long_one_trace_rounds(L, S, groups, between, wmax):  # noqa: F811
    km = _races(S, groups, between, wmax, S + groups)
    o = O.repair(km, policy=1, solver=1)
    g = L.repair(km, policy=1, solver=1)
    assert same_repair(g, o), (g, o)


@pytest.mark.parametrize("total", [2**25 - 2, 2**25 - 1, 2**25])
def test_path_weights(L, total):  # noqa: F811
    for S in (21, 64):
        rng = np.random.default_rng(S)
        cl = _runs(rng, S, 2 * S, 6)
        w = [total // S] * (S - 1) + [total - total // S * (S - 1)]
        assert L.min_barriers(cl, w, S) == _best_runs(cl, w, S)
