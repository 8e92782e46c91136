"""The work that a user of librepair has it do, as cases to time.

A case is a dict of plain values: which entry point it calls and the sizes of
the kernel models it passes.  Models come from the seeded generator that the
tests and the benchmark use (``paper_2011_08373_amd.synth``); every call goes
through the public Python binding or, where the caller wants plain buffers
back, the C ABI itself.  All results are whole numbers.

Calls: ``check`` (Verify under an assignment: every racing pair), ``first``
(the first racing partner of every point), ``clauses`` (GenerateClause),
``solve`` (one minimum-weight query), ``repair`` and ``noalloc`` (the repair
loop), ``batch`` (many kernels in one call), ``programs`` (structured programs
instrumented beforehand, repaired in one call) and ``serve`` (jobs submitted
together to a continuous-batching server and stepped to their verdicts).
"""
import ctypes as C

import numpy as np

from paper_2011_08373_amd import librepair as L
from paper_2011_08373_amd import synth


def _model(call, name, blocks, threads, points, slots, words, shared, glob, access, write, guard,
           unroll, mode, **more):
    d = dict(call=call, blocks=blocks, threads=threads, points=points, slots=slots, words=words,
             shared=shared, glob=glob, access=access, write=write, guard=guard, unroll=unroll,
             mode=mode, stride=256, conds=False, policy=0, solver=0)
    if name:
        d["name"] = name
    d.update(more)
    return d


def _small(call, name, **more):
    """The small plain configuration: one block, one shared array."""
    d = dict(blocks=1, threads=64, points=16, slots=4, words=128, shared=1, glob=0, access=1.0,
             write=0.4, guard=0.0, unroll=1, mode="planted", stride=0)
    d.update(more)
    return _model(call, name, **d)


def _large(call, name, **more):
    """The large plain configuration."""
    d = dict(blocks=256, threads=256, points=512, slots=32, words=1 << 20, shared=2, glob=2,
             access=1.0, write=0.3, guard=0.10, unroll=8, mode="planted")
    d.update(more)
    return _model(call, name, **d)


def _stress(call, name, **more):
    """The stress configuration: about two billion accesses."""
    d = dict(blocks=4096, threads=1024, points=1024, slots=64, words=1 << 24, shared=4, glob=4,
             access=0.5, write=0.25, guard=0.15, unroll=16, mode="planted")
    d.update(more)
    return _model(call, name, **d)


def listed():
    return [
        # one Verify call on a kernel of the size of the paper's listings: an
        # editor or a test run asking about one assignment, latency only
        _small("check", "check small", mode="literal"),
        # the repair loop on such a kernel
        _small("repair", "repair small"),
        # the loop for callers that cannot allocate: a few ragged blocks, an
        # odd array size, branches on the block id
        _model("noalloc", "noalloc ragged", 5, 65, 40, 8, 4099, 1, 1, 1.0, 0.3, 0.3, 3, "planted",
               stride=65, conds=True),
        # GenerateClause alone on a medium kernel with ragged blocks
        _model("clauses", "clauses ragged", 41, 200, 200, 24, 10007, 1, 2, 1.0, 0.3, 0.2, 4,
               "planted", stride=200),
        # one Solve query over a wide constraint set (the search takes from
        # under a millisecond to about 0.1 s at this width; wider random
        # sets reach seconds)
        dict(name="solve 56", call="solve", slots=56, clauses=300),
        # Verify's full list of racing pairs on an ordinary large kernel
        _large("check", "check large", mode="literal"),
        # the paper's own strategy on it (greedy hitting set, one trace per
        # Verify call): many rounds
        _large("repair", "repair large", policy=1, solver=1),
        # the race check of one assignment on the largest kernel
        _stress("first", "first stress", mode="literal"),
        # the repair of the largest kernel
        _stress("repair", "repair stress"),
        # many kernels of uneven size in one call
        dict(name="batch mixed", call="batch", kernels=128, policy=0, solver=0),
        # a suite of small structured programs in one call
        dict(name="batch programs", call="programs", kernels=512, policy=0, solver=0),
        # a burst of jobs served with continuous batching
        dict(name="serve burst", call="serve", kernels=48, policy=0, solver=0),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    call = rng.choice(["check", "first", "clauses", "repair", "repair", "noalloc", "solve", "batch",
                       "programs", "serve"])
    if call == "solve":
        return dict(call=call, slots=rng.randint(21, 56), clauses=_log(rng, 20, 300))
    if call == "batch":
        return dict(call=call, kernels=_log(rng, 3, 128), policy=rng.choice([0, 0, 1]),
                    solver=rng.choice([0, 1]))
    if call == "programs":
        return dict(call=call, kernels=_log(rng, 10, 512), policy=rng.choice([0, 1]),
                    solver=rng.choice([0, 1]))
    if call == "serve":
        return dict(call=call, kernels=_log(rng, 3, 48), policy=0, solver=rng.choice([0, 1]))
    small = call == "noalloc"
    threads = _log(rng, 33, 256 if small else 1024)
    blocks = _log(rng, 1, 8 if small else 2048)
    points = _log(rng, 16, 100 if small else 1000)
    # at most half of the largest listed kernel's accesses
    blocks = max(1, min(blocks, (1 << 30) // (threads * points)))
    slots = max(2, min(64, int(points * rng.uniform(0.05, 0.25))))
    words = 2 * threads * blocks + rng.randint(0, 1 << 16)
    if rng.random() < 0.5:
        words = 1 << (words - 1).bit_length()
    return _model(call, None, blocks, threads, points, slots, words, rng.randint(1, 4),
                  rng.randint(0, 4), rng.choice([0.5, 1.0]), rng.choice([0.25, 0.3, 0.4]),
                  rng.choice([0.0, 0.1, 0.3]), rng.choice([1, 4, 8]),
                  "literal" if call in ("check", "first") else "planted",
                  stride=threads, conds=rng.random() < 0.3,
                  policy=rng.choice([0, 0, 1]) if call in ("repair", "noalloc") else 0,
                  solver=rng.choice([0, 1]) if call in ("repair", "noalloc") else 0)


def _kernel(c, rng):
    cfg = dict(blocks=c["blocks"], threads=c["threads"],
               arrays=[(c["words"], synth.SHARED)] * c["shared"] +
                      [(c["words"], synth.GLOBAL)] * c["glob"],
               P=c["points"], S=c["slots"], S_grid=c["slots"] // 4 if c["glob"] else 0,
               write_frac=c["write"], a_set=(1, 2) if c["blocks"] == 1 else (-1, 0, 1, 2),
               b_set=(0, c["stride"]), c_rng=(-2, 2), guard_frac=c["guard"],
               loop_frac=0.10 if c["unroll"] > 1 else 0.0, unroll=c["unroll"],
               access_frac=c["access"], pre_frac=0.25, weight_mode="baseline")
    km = (synth.literal_kernel if c["mode"] == "literal" else synth.planted_kernel)(cfg, rng)
    return synth.with_block_conditions(km, rng) if c["conds"] else km


def _options(c):
    return dict(policy=c["policy"], solver=c["solver"])


def prepare(case, seed):
    c = case
    rng = np.random.default_rng(seed)
    s = dict(case=c, ws=L.Workspace())
    if c["call"] == "solve":
        # what GenerateClause hands to Solve: runs of neighbouring slots, and
        # a few slots that diverge
        S = c["slots"]
        cl = []
        for _ in range(c["clauses"]):
            lo = int(rng.integers(0, S - 1))
            hi = int(rng.integers(lo + 1, min(S, lo + 6)))
            cl.append((((1 << (hi + 1)) - 1) & ~((1 << lo) - 1), 0))
        cl += [(0, 1 << int(v)) for v in rng.choice(S, size=2, replace=False)]
        s["clauses"], s["weights"] = cl, rng.integers(1, 11, size=S).tolist()
        s["ws"].get(int(L.lib().rp_solve_workspace_bytes(len(cl))))
    elif c["call"] in ("batch", "programs"):
        if c["call"] == "batch":
            kms = synth.generate_batch(n=c["kernels"], mode="planted", seed=seed)
        else:
            got = [L.instrument(p) for p in synth.generate_programs(c["kernels"], seed=seed)]
            kms = [k for st, k in got if st == L.OK]
        s["batch"] = L.BatchArg(kms)
        s["ws"].get(s["batch"].need())
    elif c["call"] == "serve":
        kms = synth.generate_batch(n=c["kernels"], mode="planted", seed=seed)
        s["jobs"] = [L.KernelArg(k) for k in kms]
        s["server"] = L.Server(arena_bytes=16 << 30, max_resident=64, **_options(c))
    else:
        km = _kernel(c, rng)
        s["km"] = ka = L.KernelArg(km)
        op = dict(check=L.OP_CHECK, first=L.OP_FIRST, clauses=L.OP_CLAUSES).get(c["call"], L.OP_REPAIR)
        P = s["P"] = km.n_points
        if c["call"] != "noalloc":
            s["ws"].get(ka.need(op))
        # an assignment under test: a quarter of the slots enabled
        s["x"] = sum(1 << q for q in range(km.n_slots) if rng.random() < 0.25)
        if c["call"] == "check":
            s["pairs"] = np.zeros(max(1, P * (P + 1)), L.PAIR_DT)
        elif c["call"] == "first":
            s["table"] = np.zeros((2, max(1, P)), np.uint32)
        elif c["call"] == "clauses":
            s["out"] = np.zeros((4 * P + 256, 2), np.uint64)
    return s


def _whole(values):
    return np.array(values, np.uint64).view(np.int64)


def _path(r, n=256):
    """The verified assignments in order, in a buffer of fixed size."""
    t = r["trajectory"][:n]
    return _whole(t + [0] * (n - len(t)))


def _result(r):
    return [r["status"] & 0xFFFFFFFF, r["rounds"], r["n_clauses"], r["assign"], r["weight"],
            r["added"], r["removed"]]


def run(state):
    s, c = state, state["case"]
    call = c["call"]
    if call == "repair":
        r = L.repair(s["km"], ws=s["ws"], **_options(c))
        return [_whole(_result(r)), _path(r)]
    if call == "noalloc":
        r = L.repair_noalloc(s["km"], **_options(c))
        return [_whole(_result(r)), _path(r)]
    if call in ("batch", "programs"):
        st, res = L.repair_batch(s["batch"], ws=s["ws"], **_options(c))
        return [st, _whole([_result(r) for r in res])]
    if call == "serve":
        srv, jobs = s["server"], s["jobs"]
        for n, k in enumerate(jobs):
            srv.submit(k, n)
        got = {}
        while len(got) < len(jobs):
            srv.step()
            for job, r, _ in srv.poll():
                got[job] = r
        return _whole([_result(got[n]) for n in range(len(jobs))])
    if call == "solve":
        st, x, w = L.min_barriers(s["clauses"], s["weights"], c["slots"], ws=s["ws"])
        return _whole([st, x, w])
    # the C ABI with the caller's own buffers
    t = s["ws"].t
    ws, size, stream = C.c_void_p(t.data_ptr()), t.numel(), L._stream()
    n, div, nrec = C.c_uint64(0), C.c_uint64(0), C.c_uint64(0)
    if call == "check":
        st = L.lib().rp_check(s["km"].ref, C.c_uint64(s["x"]), s["pairs"].ctypes.data, len(s["pairs"]),
                              C.byref(n), C.byref(div), C.byref(nrec), ws, size, stream)
        return [_whole([st & 0xFFFFFFFF, n.value, div.value, nrec.value]),
                s["pairs"].view(np.uint8)]
    if call == "first":
        st = L.lib().rp_first_partners(s["km"].ref, C.c_uint64(s["x"]), s["table"].ctypes.data,
                                       C.byref(div), ws, size, stream)
        return [_whole([st & 0xFFFFFFFF, div.value]), s["table"].view(np.int32)]
    st = L.lib().rp_clauses(s["km"].ref, C.c_uint64(s["x"]), s["out"].ctypes.data, len(s["out"]),
                            C.byref(n), ws, size, stream)
    return [_whole([st & 0xFFFFFFFF, n.value]), s["out"].view(np.int64)]


def work(case):
    """The descriptors in (8 bytes an array or guard, 20 a point, 8 a slot)
    and the results out; what an entry point computes between them has no
    fixed number of operations."""
    c = case
    result = 56
    if c["call"] == "solve":
        return dict(bytes=16 * c["clauses"] + 4 * c["slots"] + 24, flops=0)
    if c["call"] == "programs":
        return dict(bytes=c["kernels"] * (41 * 20 + 17 * 8 + result), flops=0)
    if c["call"] in ("batch", "serve"):
        return dict(bytes=c["kernels"] * (520 * 20 + 21 * 8 + result), flops=0)
    byts = 8 * (c["shared"] + c["glob"]) + 20 * c["points"] + 8 * c["slots"] + result
    if c["call"] == "check":
        byts += 6 * c["points"] * c["points"] // 8
    elif c["call"] == "first":
        byts += 8 * c["points"]
    elif c["call"] == "clauses":
        byts += 16 * c["slots"]
    return dict(bytes=byts, flops=0)


def exact(case, seed):
    """Every output is a whole number, which has to come out the same."""
    return None
