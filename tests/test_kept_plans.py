"""The plan a thread keeps from its last call is used only for the very same lengths
and options: workspace sizes and work lists asked for in a mixed order on one thread
equal those asked for on threads of their own, which keep nothing (runs on the CPU).
The work list queries serve the kept plan, as the calls do."""
import ctypes
import threading

import numpy as np

import paper_2606_16824_amd as cwlib


def _sizes(q):
    kind, lp, ls, hkv, g, d, p, dt, tune = q
    for key, value in tune.items():
        cwlib.set_tuning(key, value)
    try:
        if kind == "extend":
            return cwlib.extend_workspace_bytes(lp, ls, hkv, g, d, p)
        if kind == "decode":
            return cwlib.decode_workspace_bytes(lp, hkv, g, d, p, dt)
        return cwlib.step_workspace_bytes(lp, ls, hkv, g, d, p, dt)
    finally:
        cwlib.set_tuning(0, 0)
        cwlib.set_tuning(1, 0)
        cwlib.set_tuning(3, 1)
        cwlib.set_tuning(5, 125)


def test_kept_plan_only_for_the_same_call():
    base = ("step", [5000, 70, 0, 16000], [1, 64, 300, 1], 8, 4, 128, 16, "bf16", {})
    queries = [base]
    for i, other in ((1, [5000, 70, 0, 16001]), (2, [1, 64, 301, 1]), (3, 4), (4, 8), (5, 64), (6, 64), (7, "fp8"),
                     (8, {0: 3}), (8, {1: 64}), (8, {5: 300}), (8, {3: 0}), (0, "extend"), (0, "decode")):
        q = list(base)
        q[i] = other
        queries.append(tuple(q))
    # one sequence fewer or more, and two lists that only differ in where they are cut
    queries += [("extend", [100, 200], [50, 60], 2, 4, 64, 16, "bf16", {}), ("extend", [100], [200], 2, 4, 64, 16, "bf16", {}),
                ("decode", [100, 200, 50, 60], None, 2, 4, 64, 16, "bf16", {})]
    fresh = {}

    def ask(i):
        fresh[i] = _sizes(queries[i])

    for i in range(len(queries)):
        t = threading.Thread(target=ask, args=(i,))
        t.start()
        t.join()
    assert len(set(fresh.values())) > 5
    rng = np.random.default_rng(0)
    for i in list(range(len(queries))) * 2 + rng.integers(0, len(queries), 200).tolist():
        assert _sizes(queries[i]) == fresh[i], queries[i]


def test_lengths_changed_in_place():
    """The caller's array may be reused with other lengths: the plan follows its values."""
    lp, ls = np.array([4000, 9000], np.int32), np.array([700, 1], np.int32)
    first = cwlib.step_workspace_bytes(lp, ls, 8, 4, 128, 16, "bf16")
    lp[0] = 60000
    other = cwlib.step_workspace_bytes(lp, ls, 8, 4, 128, 16, "bf16")
    lp[0] = 4000
    assert cwlib.step_workspace_bytes(lp, ls, 8, 4, 128, 16, "bf16") == first != other


def test_tuning_changed_while_planning():
    """A plan is kept under the tuning it was made with, also when another thread changes
    the tuning while it is being made: asked for again under the first tuning, the size is
    that of the first tuning."""
    rng = np.random.default_rng(139)
    lp = rng.integers(1000, 60000, 600).astype(np.int32)
    ls = np.where(np.arange(600) % 2 == 0, 1, rng.integers(2, 900, 600)).astype(np.int32)
    ask = lambda n: cwlib.step_workspace_bytes(lp[:n], ls[:n], 2, 4, 128, 16, "bf16")
    sizes = {}

    def fresh(n):
        sizes[n] = ask(n)

    for n in range(60, 64):
        t = threading.Thread(target=fresh, args=(n,))
        t.start()
        t.join()
    stop = threading.Event()

    def flip():
        while not stop.is_set():
            cwlib.set_tuning(0, 7)
            cwlib.set_tuning(0, 0)

    try:
        for i in range(400):
            n = 60 + i % 4
            stop.clear()
            t = threading.Thread(target=flip)
            t.start()
            ask(n)
            stop.set()
            t.join()
            assert ask(n) == sizes[n], (i, n)
    finally:
        stop.set()
        cwlib.set_tuning(0, 0)


def _on_own_thread(f):
    got = []
    t = threading.Thread(target=lambda: got.append(f()))
    t.start()
    t.join()
    return got[0]


def _same(a, b):
    return all(x.shape == y.shape and np.array_equal(x, y) for x, y in zip(a, b))


def test_other_plans_of_the_same_size():
    """Calls whose plans take the same bytes but hold other work (lengths permuted, moved
    between sequences or changed within a key tile): each gets its own work list."""
    exts = [([5000, 9000, 300], [400, 70, 900]), ([9000, 5000, 300], [400, 70, 900]), ([5000, 9000, 300], [70, 400, 900]),
            ([5001, 9000, 300], [400, 70, 900]), ([5000, 9000, 300], [399, 71, 900])]
    ask = [(lambda lp=lp, ls=ls: (cwlib.plan_items(lp, ls, 4, 8, 128, 16),)) for lp, ls in exts]
    size = lambda lp, ls: cwlib.extend_workspace_bytes(lp, ls, 4, 8, 128, 16)
    assert len({size(lp, ls) for lp, ls in exts}) < len(exts)
    decs = [[5000, 9000, 300], [9000, 5000, 300], [5000, 300, 9000], [5001, 9000, 300], [4999, 9001, 300]]
    ask += [(lambda lp=lp: cwlib.decode_plan(lp, 4, 8, 128, 16)) for lp in decs]
    assert len({cwlib.decode_workspace_bytes(lp, 4, 8, 128, 16) for lp in decs}) < len(decs)
    fresh = [_on_own_thread(f) for f in ask]
    n = len(exts)
    for group in (fresh[:n], fresh[n:]):
        assert not any(_same(a, b) for i, a in enumerate(group) for b in group[:i])
    rng = np.random.default_rng(149)
    for i in rng.integers(0, len(ask), 200).tolist():
        assert _same(ask[i](), fresh[i]), i


class _MallInfo(ctypes.Structure):
    _fields_ = [(n, ctypes.c_size_t) for n in ("arena", "ordblks", "smblks", "hblks", "hblkhd", "usmblks", "fsmblks",
                                               "uordblks", "fordblks", "keepcost")]


def test_nothing_stays_of_a_large_plan():
    """A plan above 1 MB is not kept, and neither are the lengths it was compared by."""
    libc = ctypes.CDLL(None)
    libc.mallinfo2.restype = _MallInfo

    def in_use():
        m = libc.mallinfo2()
        return m.uordblks + m.hblkhd

    lp, ls = np.full(1 << 20, 5, np.int32), np.zeros(1 << 20, np.int32)
    ls[0] = 3
    cwlib.extend_workspace_bytes(lp[:4], ls[:4], 1, 4, 64, 16)
    before = in_use()
    assert cwlib.extend_workspace_bytes(lp, ls, 1, 4, 64, 16) > 1 << 24
    assert in_use() - before < 1 << 20
