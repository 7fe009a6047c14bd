"""The splits of the batched passes over the chip: a work-group per target
cells (few targets), eight, four or two wavefronts a target plane, a launch of
their own for the targets past whole rounds, ordinary and persistent launches, at the target counts where the choice changes; and the
work counters of persistent launches (left at zero by every launch, two pools
per plan). Oracle and criterion as in test_gpu_parity.py (1e-12 per sub-grid
and output order)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
import oracle  # noqa: E402
import synthetic  # noqa: E402
from parity import assert_parity  # noqa: E402
from saved_sums import check_saved  # noqa: E402

pytestmark = pytest.mark.gpu

SUB3 = 512
TOL = 1e-12


@pytest.fixture(scope="module")
def ot():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08058_amd as mod
    return mod


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.float64)).cuda()


def _host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _nan(*shape):
    import torch
    return torch.full(shape, float("nan"), dtype=torch.float64, device="cuda")


def _subset(k, seed):
    """A store of k sub-grids drawn from a 4^3 to 6^3 lattice (periodic), all of
    them targets; neighbours outside the draw are missing."""
    rng = synthetic._rng(seed)
    side = 4 if k <= 64 else 5 if k <= 125 else 6
    M, X = synthetic.store_field(side, rng, 2.0, 3.0, 0.6, sep=6.0)
    full = synthetic.lattice_batch(side)
    ids = np.sort(rng.permutation(side ** 3)[:k])
    to = np.full(side ** 3 + 1, -1, np.int32)
    to[ids] = np.arange(k)
    cols = (ids[:, None] * SUB3 + np.arange(SUB3)).reshape(-1)
    batch = {"S": k, "T": k, "tgt": np.arange(k, dtype=np.int32), "nbr": to[full["nbr"][ids]],
             "shift": full["shift"][ids], "period": full["period"]}
    return batch, np.ascontiguousarray(M[:, cols]), np.ascontiguousarray(X[:, cols])


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("k", [1, 2, 20, 21, 24, 25, 33, 64, 96, 97, 130, 160])
def test_every_split_matches_the_oracle(ot, k, full):
    batch, M, X = _subset(k, 400 + k)
    w = synthetic.weights(k, 500 + k)
    sel = np.unique(np.array([0, k // 2, k - 1], np.int32))
    plan = ot.Plan.from_batch(batch)
    Md, Xd, wd = _dev(M), _dev(X), _dev(w)
    n = k * SUB3
    pick = lambda t: _host(t).reshape(t.shape[0], k, SUB3)[:, sel].reshape(t.shape[0], -1)  # noqa: E731
    ref, A = oracle.batched_forward(batch, M, X, tsel=sel, want_abs=True, full=full)
    L, Ls, Cs, gM, gX = _nan(20, n), _nan(20, n), _nan(24, n), _nan(20, n), _nan(3, n)
    (plan.multipole_batched_full if full else plan.multipole_batched)(Md, Xd, L)
    assert_parity(pick(L), ref, TOL, what="k=%d L" % k, A=A)
    plan.multipole_batched_save(Md, Xd, Ls, Cs, full=full)
    assert_parity(pick(Ls), ref, TOL, what="k=%d saved L" % k, A=A)
    check_saved(pick(Cs), batch, M, X, "k=%d Cs" % k, tsel=sel, full=full)
    gM_ref, gX_ref = oracle.batched_backward(batch, M, X, w, ssel=sel, full=full)
    plan.multipole_backward_saved(Md, Xd, wd, Cs, gM, gX, full=full)
    assert_parity(pick(gM), gM_ref, TOL, what="k=%d gM" % k)
    assert_parity(pick(gX), gX_ref, TOL, what="k=%d gX" % k)
    gM2, gX2 = _nan(20, n), _nan(3, n)
    (plan.multipole_backward_full if full else plan.multipole_backward)(Md, Xd, wd, gM2, gX2)
    assert np.array_equal(_host(gM2), _host(gM))
    assert_parity(pick(gX2), gX_ref, TOL, what="k=%d three-launch gX" % k)


def test_subset_of_targets_with_a_rest(ot):
    """150 of 216 sub-grids are targets, in no order: a rest of 22 targets and,
    in the source role, of 24 sub-grids."""
    batch, M, X = _subset(216, 616)
    k = 150
    tgt = synthetic._rng(617).permutation(216)[:k].astype(np.int32)
    batch.update(T=k, tgt=tgt, nbr=np.ascontiguousarray(batch["nbr"][tgt]),
                 shift=np.ascontiguousarray(batch["shift"][tgt]))
    w = synthetic.weights(k, 618)
    plan = ot.Plan.from_batch(batch)
    Md, Xd, wd = _dev(M), _dev(X), _dev(w)
    L, Cs = _nan(20, k * SUB3), _nan(24, k * SUB3)
    gM, gX = _nan(20, 216 * SUB3), _nan(3, 216 * SUB3)
    plan.multipole_batched_save(Md, Xd, L, Cs)
    plan.multipole_backward_saved(Md, Xd, wd, Cs, gM, gX)
    sel = np.array([0, 127, 128, 149], np.int32)
    pick = lambda t, n, i: _host(t).reshape(t.shape[0], n, SUB3)[:, i].reshape(t.shape[0], -1)  # noqa: E731
    ref, A = oracle.batched_forward(batch, M, X, tsel=sel, want_abs=True)
    assert_parity(pick(L, k, sel), ref, TOL, what="L", A=A)
    check_saved(pick(Cs, k, sel), batch, M, X, "Cs", tsel=sel)
    ssel = np.array([0, 191, 192, 215], np.int32)
    gM_ref, gX_ref = oracle.batched_backward(batch, M, X, w, ssel=ssel)
    assert_parity(pick(gM, 216, ssel), gM_ref, TOL, what="gM")
    assert_parity(pick(gX, 216, ssel), gX_ref, TOL, what="gX")


def _lattice(ot, n, missing=0.2, seed=41):
    """A large lattice of cheap inputs (values do not matter for equality)."""
    import torch
    b = synthetic.apply_missing(synthetic.lattice_batch(n), missing, synthetic._rng(seed))
    M, X = synthetic.device_lattice_store(n, seed)
    return b, ot.Plan.from_batch(b), M, X, torch


def test_launch_forms_agree_bitwise(ot):
    """Ordinary, persistent, XCD-aware and AUTO launches of the same passes,
    each twice in a row (a persistent launch finds its counters at zero)."""
    b, plan, M, X, torch = _lattice(ot, 9)  # 729 targets: AUTO is persistent
    N = b["T"] * SUB3
    w = torch.randn((20, N), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    ref = None
    for sched in (1, 3, 0x11, 0x21, 0x31, 0):
        for rep in range(2):
            L, Ls, Cs, gM, gX = _nan(20, N), _nan(20, N), _nan(24, N), _nan(20, N), _nan(3, N)
            plan.multipole_batched(M, X, L, sched=sched)
            plan.multipole_batched_save(M, X, Ls, Cs, sched=sched)
            plan.multipole_backward_saved(M, X, w, Cs, gM, gX, sched=sched)
            torch.cuda.synchronize()
            if ref is None:
                ref = (L, Ls, Cs, gM, gX)
            for a, r in zip((L, Ls, Cs, gM, gX), ref):
                assert torch.equal(a, r), (sched, rep)


@pytest.mark.parametrize("n", [6, 8])
def test_launch_forms_agree_with_a_rest(ot, n):
    """216 targets: 192 in whole rounds, 24 in a launch of their own, the same
    ones whatever the schedule's order. 512: AUTO is persistent for the saved
    sums only."""
    b, plan, M, X, torch = _lattice(ot, n)
    N = b["T"] * SUB3
    ref = None
    for sched in (1, 0x11, 0x21, 0x31, 0):
        L, Ls, Cs = _nan(20, N), _nan(20, N), _nan(24, N)
        plan.multipole_batched(M, X, L, sched=sched)
        plan.multipole_batched_save(M, X, Ls, Cs, sched=sched)
        torch.cuda.synchronize()
        ref = ref or (L, Ls, Cs)
        assert all(torch.equal(a, r) for a, r in zip((L, Ls, Cs), ref)), sched


def test_auto_on_more_streams_than_counters(ot):
    """AUTO launches on 70 streams of one plan: those past the counters run as
    ordinary launches, and explicit persistent launches keep their own 64."""
    b, plan, M, X, torch = _lattice(ot, 9)
    N = b["T"] * SUB3
    ref = _nan(20, N)
    plan.multipole_batched(M, X, ref, sched=1)
    ex = ot.Executor(70, 0)
    streams = [ex.stream(i) for i in range(70)]
    torch.cuda.synchronize()
    L = _nan(20, N)
    torch.cuda.synchronize()
    for i, s in enumerate(streams):
        if i >= 60:
            L.fill_(float("nan"))
        torch.cuda.synchronize()
        plan.multipole_batched(M, X, L, stream=s)
        torch.cuda.synchronize()
        if i >= 60:
            assert torch.equal(L, ref), i
    for s in streams[:64]:
        plan.multipole_batched(M, X, L, sched=0x11, stream=s)
        torch.cuda.synchronize()
    with pytest.raises(ot.OtFmmError):
        plan.multipole_batched(M, X, L, sched=0x11, stream=streams[64])
    assert torch.equal(L, ref)
    ex.close()
