"""Work counters of persistent launches are never shared by launches that can
overlap: launches of several threads on hipStreamPerThread, several executables
of one captured graph, replays of the plan's step graph on several streams.
729 targets (a periodic lattice of 9^3 sub-grids), where AUTO is persistent and
the launches take long enough to overlap. The expected outputs are those of the
ordinary launches, bit for bit (the schedules share one split of the work; the
kernels are compared with the oracle in the other files)."""
import ctypes
import os
import sys
import threading

import pytest

sys.path.insert(0, os.path.dirname(__file__))
import synthetic  # noqa: E402

pytestmark = pytest.mark.gpu

N = 729 * 512
PER_THREAD = 2  # the handle hipStreamPerThread


@pytest.fixture(scope="module")
def ot():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08058_amd as mod
    return mod


def _nan(k):
    import torch
    return torch.full((k, N), float("nan"), dtype=torch.float64, device="cuda")


def _hip(ot, name, *args):
    rc = getattr(ot._lib, name)(*args)
    assert rc == 0, (name, rc)


class _Case:
    """A fresh plan, inputs, and what ordinary launches write."""

    def __init__(self, ot):
        import torch
        b = synthetic.apply_missing(synthetic.lattice_batch(9), 0.2, synthetic._rng(61))
        self.plan = ot.Plan.from_batch(b)
        self.M, self.X = synthetic.device_lattice_store(9, 61)
        self.w = torch.randn((20, N), dtype=torch.float64, device="cuda",
                             generator=torch.Generator("cuda").manual_seed(62))
        self.ref = self.outputs()
        self.run(self.ref, 1, None)
        torch.cuda.synchronize()

    @staticmethod
    def outputs():
        return {"L": _nan(20), "Ls": _nan(20), "Cs": _nan(24), "gM": _nan(20), "gX": _nan(3)}

    def run(self, o, sched, stream):
        self.plan.multipole_batched(self.M, self.X, o["L"], sched=sched, stream=stream)
        self.plan.multipole_batched_save(self.M, self.X, o["Ls"], o["Cs"], sched=sched, stream=stream)
        self.plan.multipole_backward_saved(self.M, self.X, self.w, o["Cs"], o["gM"], o["gX"], sched=sched, stream=stream)

    def check(self, o, what):
        import torch
        for k, v in o.items():
            assert torch.equal(v, self.ref[k]), (what, k)


@pytest.mark.parametrize("sched", [0, 0x11, 0x31])
def test_threads_on_the_per_thread_stream(ot, sched):
    """Three threads launch one plan on hipStreamPerThread at the same time;
    later launches on that handle are whole as well."""
    import torch
    c = _Case(ot)
    outs = [[c.outputs() for _ in range(2)] for _ in range(3)]
    torch.cuda.synchronize()
    start = threading.Barrier(3)
    errors = []

    def work(mine):
        try:
            torch.cuda.set_device(0)
            start.wait()
            for o in mine:
                c.run(o, sched, PER_THREAD)
            _hip(ot, "hipStreamSynchronize", ctypes.c_void_p(PER_THREAD))
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(m,)) for m in outs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i, mine in enumerate(outs):
        for o in mine:
            c.check(o, "thread %d" % i)
    o = c.outputs()
    c.run(o, sched, PER_THREAD)
    torch.cuda.synchronize()
    c.check(o, "after the threads")


@pytest.mark.parametrize("sched", [0, 0x11, 0x31])
def test_two_executables_of_one_captured_graph(ot, sched):
    """The forward recorded into one graph, instantiated twice, the two replayed
    on two streams at the same time, with eager launches on a third."""
    import torch
    c = _Case(ot)
    L, E = _nan(20), _nan(20)
    s = [ctypes.c_void_p() for _ in range(3)]
    for h in s:
        _hip(ot, "hipStreamCreateWithFlags", ctypes.byref(h), 1)
    graph, ex = ctypes.c_void_p(), [ctypes.c_void_p(), ctypes.c_void_p()]
    torch.cuda.synchronize()
    _hip(ot, "hipStreamBeginCapture", s[0], 1)
    c.plan.multipole_batched(c.M, c.X, L, sched=sched, stream=s[0].value)
    _hip(ot, "hipStreamEndCapture", s[0], ctypes.byref(graph))
    for e in ex:
        _hip(ot, "hipGraphInstantiate", ctypes.byref(e), graph, None, None, ctypes.c_size_t(0))
    for rep in range(3):
        L.fill_(float("nan"))
        E.fill_(float("nan"))
        torch.cuda.synchronize()
        for e, h in zip(ex, s):
            _hip(ot, "hipGraphLaunch", e, h)
        c.plan.multipole_batched(c.M, c.X, E, sched=sched, stream=s[2].value)
        torch.cuda.synchronize()
        assert torch.equal(L, c.ref["L"]) and torch.equal(E, c.ref["L"]), rep
    # each executable alone, after they ran side by side
    for e in ex:
        L.fill_(float("nan"))
        torch.cuda.synchronize()
        _hip(ot, "hipGraphLaunch", e, s[0])
        torch.cuda.synchronize()
        assert torch.equal(L, c.ref["L"])
    for e in ex:
        _hip(ot, "hipGraphExecDestroy", e)
    _hip(ot, "hipGraphDestroy", graph)
    for h in s:
        _hip(ot, "hipStreamDestroy", h)


@pytest.mark.parametrize("sched", [0, 0x11, 0x31])
def test_step_graph_replays_on_two_streams(ot, sched):
    """The plan's step graph replayed on two streams without waiting between,
    then once more after it was captured anew."""
    import torch
    c = _Case(ot)
    o = c.outputs()
    s = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(2):
        c.plan.step_graph_create_saved(c.M, c.X, o["Ls"], o["Cs"], c.w, o["gM"], o["gX"], sched, sched)
        for times in (1, 4):
            for v in o.values():
                v.fill_(float("nan"))
            torch.cuda.synchronize()
            for k in range(times):
                c.plan.step_graph_launch(s[k % 2])
            torch.cuda.synchronize()
            for k in ("Ls", "Cs", "gM", "gX"):
                assert torch.equal(o[k], c.ref[k]), (rep, times, k)


@pytest.mark.parametrize("sched", [0, 0x11, 0x31])
def test_two_streams_in_flight(ot, sched):
    """Every pass of one plan on two streams at once, twice on each."""
    import torch
    c = _Case(ot)
    outs = [c.outputs() for _ in range(4)]
    s = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        c.run(o, sched, s[i % 2])
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        c.check(o, "launch %d" % i)


@pytest.mark.parametrize("sched", [0x11, 0x31])
def test_three_launch_step_graph_beside_eager_launches(ot, sched):
    """The three-launch step in the plan's graph, replayed while eager launches
    of the same plan run on another stream; each replay against eager results."""
    import torch
    c = _Case(ot)
    L, gM, gX, R = _nan(20), _nan(20), _nan(3), _nan(3)
    c.plan.multipole_backward(c.M, c.X, c.w, gM, R, sched=0x0101)
    c.plan.step_graph_create(c.M, c.X, L, c.w, gM, gX, sched, sched | sched << 8)
    s = [torch.cuda.Stream(), torch.cuda.Stream()]
    o = c.outputs()
    for rep in range(3):
        for t in (L, gM, gX, *o.values()):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        c.plan.step_graph_launch(s[0])
        c.run(o, sched, s[1])
        torch.cuda.synchronize()
        assert torch.equal(L, c.ref["L"]) and torch.equal(gM, c.ref["gM"]) and torch.equal(gX, R), rep
        c.check(o, ("eager", rep))


@pytest.mark.parametrize("sched", [0, 0x11, 0x31])
def test_full_truncation_in_a_callers_graph(ot, sched):
    """The full truncation's passes recorded into a caller's graph, replayed
    three times beside eager ones (729 and 512 targets: AUTO is persistent for
    its saved sums at both, for its forward at 729)."""
    import torch
    for n in (9, 8):
        b = synthetic.apply_missing(synthetic.lattice_batch(n), 0.2, synthetic._rng(63))
        plan = ot.Plan.from_batch(b)
        M, X = synthetic.device_lattice_store(n, 63)
        w = torch.ones((20, n ** 3 * 512), dtype=torch.float64, device="cuda")
        nan = lambda: [torch.full((k, n ** 3 * 512), float("nan"), dtype=torch.float64, device="cuda")  # noqa: E731
                       for k in (20, 20, 24, 20, 3, 20, 3)]

        def run(o, sc, stream):
            plan.multipole_batched_full(M, X, o[0], sched=sc, stream=stream)
            plan.multipole_batched_save(M, X, o[1], o[2], sched=sc, stream=stream, full=True)
            plan.multipole_backward_saved(M, X, w, o[2], o[3], o[4], sched=sc, stream=stream, full=True)
            plan.multipole_backward_full(M, X, w, o[5], o[6], sched=sc | sc << 8, stream=stream)

        ref, o, e = nan(), nan(), nan()
        run(ref, 1, None)
        s = [torch.cuda.Stream(), torch.cuda.Stream()]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s[0]):
            run(o, sched, s[0])
        for rep in range(3):
            for t in o + e:
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            with torch.cuda.stream(s[0]):
                g.replay()
            run(e, sched, s[1])
            torch.cuda.synchronize()
            for a, x, r in zip(o, e, ref):
                assert torch.equal(a, r) and torch.equal(x, r), (n, rep)
            junk = torch.randn(1 << 20, device="cuda").sum()  # eager work between replays
            del junk


def _plan(ot, n, k=None, periodic=True):
    """The first k sub-grids of a lattice of n^3, all of them targets."""
    import numpy as np
    import torch
    k = k or n ** 3
    full = synthetic.lattice_batch(n, periodic=periodic)
    to = np.full(n ** 3 + 1, -1, np.int32)
    to[:k] = np.arange(k)
    b = {"S": k, "T": k, "tgt": np.arange(k, dtype=np.int32), "nbr": to[full["nbr"][:k]],
         "shift": full["shift"][:k] if periodic else None, "period": full["period"]}
    M, X = synthetic.device_lattice_store(n, 71)
    M, X = M[:, :k * 512].contiguous(), X[:, :k * 512].contiguous()
    out = {c: torch.full((r, k * 512), float("nan"), dtype=torch.float64, device="cuda")
           for c, r in (("L", 20), ("Cs", 24), ("gM", 20), ("gX", 3))}
    w = torch.ones((20, k * 512), dtype=torch.float64, device="cuda")
    return ot.Plan.from_batch(b), M, X, w, out


def test_tuned_auto_on_more_streams_than_counters(ot):
    """A tuned plan's AUTO launches on 70 streams are never refused, whatever
    the tuner chose, and leave the explicit launches their 64 streams."""
    import torch
    c = _Case(ot)
    o = c.outputs()
    ex = ot.Executor(70, 0)
    streams = [ex.stream(i) for i in range(70)]
    # (the tuners' own launches name their schedules, on the last stream)
    f, b = c.plan.autotune_saved(c.M, c.X, o["Ls"], o["Cs"], c.w, o["gM"], o["gX"], stream=streams[-1])
    c.plan.autotune(c.M, c.X, o["L"], stream=streams[-1])
    for i, s in enumerate(streams):
        for v in o.values():
            v.fill_(float("nan"))
        torch.cuda.synchronize()
        c.run(o, 0, s)
        torch.cuda.synchronize()
        c.check(o, ("stream", i, hex(f), hex(b)))
    for s in streams[-64:]:
        c.run(o, 0x11, s)
        torch.cuda.synchronize()
        c.check(o, "explicit")
    with pytest.raises(ot.OtFmmError):
        c.plan.multipole_batched(c.M, c.X, o["L"], sched=0x11, stream=streams[0])
    ex.close()


@pytest.mark.parametrize("n,k", [(2, 8), (3, 27), (6, 130), (6, 150)])
def test_launches_without_counters_are_not_limited_by_them(ot, n, k):
    """Few targets, 8 wavefronts a plane, a rest: an explicit persistent
    schedule takes no counters there, so a 65th stream is as good as any."""
    import torch
    plan, M, X, w, o = _plan(ot, n, k, periodic=n > 2)
    ref = torch.empty_like(o["L"])
    plan.multipole_batched(M, X, ref, sched=1)
    ex = ot.Executor(66, 0)
    torch.cuda.synchronize()
    for i in range(66):
        o["L"].fill_(float("nan"))
        torch.cuda.synchronize()
        plan.multipole_batched(M, X, o["L"], sched=0x11, stream=ex.stream(i))
        torch.cuda.synchronize()
        assert torch.equal(o["L"], ref), i
    ex.close()


@pytest.mark.parametrize("n,k,flags", [(2, 8, {0}), (3, 27, {0, 0x20}), (6, 130, {0}),
                                       (5, 120, {0, 0x10, 0x20, 0x30})])
def test_tuners_choose_among_schedules_that_differ(ot, n, k, flags):
    """Where a flag makes no difference the tuners do not keep it."""
    plan, M, X, w, o = _plan(ot, n, k, periodic=n > 2)
    f, b = plan.autotune(M, X, o["L"], w, o["gM"], o["gX"])
    fs, bs = plan.autotune_saved(M, X, o["L"], o["Cs"], w, o["gM"], o["gX"])
    for s in (f, b & 0xff, b >> 8, fs, bs):
        assert s & 0xf in (1, 3) and s & 0x30 in flags, hex(s)
