"""The node budget of the exact search (RP_TUNE_SOLVER_NODES): constraint sets
that are no runs of neighbouring slots and stay wider than the enumeration, so
that the branch and bound itself spends it."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_08373_amd import synth
from test_gpu_parity import L, chain_kernel, same_repair  # noqa: F401  (L is a fixture)
from test_gpu_solve import _races

pytestmark = pytest.mark.gpu


@pytest.fixture()
def budget(L):  # noqa: F811
    old = L.set_tuning(L.TUNE_SOLVER_NODES, 28)
    yield lambda v: L.set_tuning(L.TUNE_SOLVER_NODES, v)
    L.set_tuning(L.TUNE_SOLVER_NODES, old)


def _apart(S, n, seed, neg=0):
    """n clauses of three slots anywhere, equal weights."""
    rng = np.random.default_rng(seed)
    cl = [(sum(1 << int(s) for s in rng.choice(S, 3, replace=False)), 0) for _ in range(n)]
    for _ in range(neg):
        p, q = rng.choice(S, 2, replace=False)
        cl.append((0, 1 << int(p) | 1 << int(q)))
    return cl, [1] * S


# up to 128 clauses are reduced by the waves, more by the workgroup first
@pytest.mark.parametrize("S,n,neg", [(30, 60, 0), (30, 60, 5), (28, 128, 0), (28, 129, 0),
                                     (26, 400, 4)])
def test_search_spends_its_budget(L, budget, S, n, neg):  # noqa: F811
    for seed in range(3):
        cl, w = _apart(S, n, 10 * n + seed, neg)
        for log2 in (4, 5):
            budget(log2)
            assert L.min_barriers(cl, w, S)[0] == L.ERR_SEARCH, (seed, log2)
        budget(28)
        assert L.min_barriers(cl, w, S) == O.min_barriers(cl, w, S), seed


def test_budget_leaves_what_is_not_searched(L, budget):  # noqa: F811
    # enumerated components, and paths of no more slots than the budget has nodes
    budget(4)
    cl, w = _apart(20, 100, 7)
    assert L.min_barriers(cl, w, 20) == O.min_barriers(cl, w, 20)
    assert same_repair(L.repair(chain_kernel(20)), O.repair(chain_kernel(20)))
    budget(5)
    assert same_repair(L.repair(chain_kernel(24)), O.repair(chain_kernel(24)))


@pytest.mark.parametrize("solver", [0, 1])
def test_search_in_one_job_of_a_batch(L, budget, solver):  # noqa: F811
    # the job whose search spends the budget, in the middle of its rounds, reads
    # RP_ERR_SEARCH, alone, in a batch and served; the others end as they do
    hard = _races(30, 60, 3, 3, 90)
    kms = [synth.generate("plain-small", mode="planted", seed=s) for s in range(5)]
    kms.insert(2, hard)
    budget(4)
    g = L.repair(hard, solver=solver)
    assert g["status"] == g["ret"] == L.ERR_SEARCH
    st, res = L.repair_batch(kms, solver=solver)
    srv = L.Server(arena_bytes=1 << 30, max_resident=8, solver=solver)
    for q, km in enumerate(kms):
        assert srv.submit(km, q) == 0
    got = {}
    while len(got) < len(kms):
        srv.step()
        got.update((job, r) for job, r, _ in srv.poll())
    assert st == 0
    for q, km in enumerate(kms):
        o = O.repair(km, solver=solver)
        for r in (res[q], got[q]):
            if q == 2:
                assert r["status"] == L.ERR_SEARCH
            else:
                assert all(r[k] == o[k] for k in ("status", "assign", "weight", "rounds", "n_clauses"))
    budget(28)
    assert same_repair(L.repair(hard, solver=solver), O.repair(hard, solver=solver))
