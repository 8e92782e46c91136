"""The record log (generation, radix sort, scans) against the oracle where the
plan would decide everything in closed form: RP_TUNE_RACE_ROUTE 1, and every call
is held to have made a log and sorted it."""
import pytest

import test_gpu_full_size as full
import test_gpu_parity as parity
from test_gpu_parity import L  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


class Logged:
    """The binding, noting the records and sort passes of each call."""

    def __init__(self, L):
        self._l = L
        self.calls = []

    def __getattr__(self, name):
        f = getattr(self._l, name)
        if name not in ("check", "first_partners", "clauses", "repair"):
            return f

        def call(*a, **kw):
            r = f(*a, **kw)
            s = self._l.last_stats()
            self.calls.append((s["records"], s["sort_launches"]))
            return r
        return call

    def __setattr__(self, name, v):
        if name in ("_l", "calls"):
            object.__setattr__(self, name, v)
        else:
            setattr(self._l, name, v)


@pytest.fixture()
def logged(L):  # noqa: F811
    old = L.set_tuning(L.TUNE_RACE_ROUTE, 1)
    yield Logged(L)
    L.set_tuning(L.TUNE_RACE_ROUTE, old)


def _all_sorted(logged, passes=1):
    assert logged.calls and all(r > 0 and n >= passes for r, n in logged.calls), logged.calls[:5]


def test_sort_knobs(logged):
    parity.test_sort_knobs_full_size(logged)
    _all_sorted(logged, 2)
    assert len(logged.calls) == 320


@pytest.mark.parametrize("pipe,fields", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_first_partners(logged, pipe, fields):
    parity.test_first_partners(logged, pipe, fields)
    # (some of the tiny kernels have no access that runs)
    assert sum(r > 0 for r, _ in logged.calls) > 0.8 * len(logged.calls)


@pytest.mark.parametrize("name,mode", [("plain_large_literal", "literal"),
                                       ("plain_large_planted", "planted")])
def test_plain_large(logged, name, mode):
    parity.test_plain_large_full_size(logged, name, mode)
    _all_sorted(logged, 2)


def test_max_points(logged):
    full.test_max_points(logged)
    _all_sorted(logged)


@pytest.mark.parametrize("mode", ["literal", "planted"])
def test_stress(logged, mode):
    # about 2G records: record offsets past 32 bits, 16K chunks
    full.test_stress_full_size(logged, mode)
    _all_sorted(logged, 3)
    assert max(r for r, _ in logged.calls) > 10**9
