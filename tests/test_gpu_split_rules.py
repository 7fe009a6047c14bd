"""The rules that choose how a batched pass is split over the chip, at the
counts where they change: few targets by their pairs, and both sides of a rest
that goes in a launch of its own, for each pass. Oracle and
criterion as in test_gpu_parity.py (1e-12 per sub-grid and output order)."""
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


def _pick(t, n, sel):
    return _host(t).reshape(t.shape[0], n, SUB3)[:, sel].reshape(t.shape[0], -1)


@pytest.fixture(scope="module")
def field():
    return synthetic.store_field(4, synthetic._rng(801), 2.0, 3.0, 0.6, sep=6.0)


@pytest.mark.parametrize("k,missing", [(12, 0), (13, 0), (16, 0), (17, 0), (19, 0), (20, 0), (20, 9), (20, 16)])
def test_few_targets_by_their_pairs(ot, field, k, missing):
    """k targets of a periodic 4^3 store, all their neighbours there (12, 16 and
    19 targets' pairs are the limits of the passes) or the last `missing`."""
    M, X = field
    full = synthetic.lattice_batch(4)
    nbr = full["nbr"][:k].copy()
    if missing:
        nbr[:, -missing:] = -1
        nbr[:, 13] = full["nbr"][:k, 13]
    batch = {"S": 64, "T": k, "tgt": full["tgt"][:k], "nbr": nbr, "shift": full["shift"][:k], "period": full["period"]}
    w = synthetic.weights(k, 802)
    plan = ot.Plan.from_batch(batch)
    Md, Xd, wd = _dev(M), _dev(X), _dev(w)
    sel, ssel = np.array([0, k - 1], np.int32), np.array([0, 21], np.int32)
    n = k * SUB3
    dref, dA = oracle.batched_forward_amc(batch, M, X, tsel=sel, want_abs=True)
    for fl in (False, True):
        ref, A = oracle.batched_forward(batch, M, X, tsel=sel, want_abs=True, full=fl)
        L, Ls, Cs = _nan(20, n), _nan(20, n), _nan(24, n)
        (plan.multipole_batched_full if fl else plan.multipole_batched)(Md, Xd, L)
        assert_parity(_pick(L, k, sel), ref, TOL, what="L", A=A)
        plan.multipole_batched_save(Md, Xd, Ls, Cs, full=fl)
        assert_parity(_pick(Ls, k, sel), ref, TOL, what="saved L", A=A)
        check_saved(_pick(Cs, k, sel), batch, M, X, "Cs", tsel=sel, full=fl)
        gM_ref, gX_ref = oracle.batched_backward(batch, M, X, w, ssel=ssel, full=fl)
        gM, gX, gM2, gX2 = _nan(20, 64 * SUB3), _nan(3, 64 * SUB3), _nan(20, 64 * SUB3), _nan(3, 64 * SUB3)
        plan.multipole_backward_saved(Md, Xd, wd, Cs, gM, gX, full=fl)
        (plan.multipole_backward_full if fl else plan.multipole_backward)(Md, Xd, wd, gM2, gX2)
        assert np.array_equal(_host(gM), _host(gM2))
        assert_parity(_pick(gM, 64, ssel), gM_ref, TOL, what="gM")
        assert_parity(_pick(gX, 64, ssel), gX_ref, TOL, what="gX")
        assert_parity(_pick(gX2, 64, ssel), gX_ref, TOL, what="three-launch gX")
        if not fl:
            Lc, dF = _nan(20, n), _nan(3, n)
            plan.multipole_batched_amc(Md, Xd, Lc, dF)
            assert np.array_equal(_host(Lc), _host(Ls))
            assert_parity(_pick(dF, k, sel), dref, TOL, what="dF", A=dA)


def test_the_forward_without_a_plan_keeps_to_the_plans_split(ot, field):
    """20 targets with and without missing neighbours: the call whose table is on
    the device gives the plan's bits."""
    import torch
    M, X = field
    full = synthetic.lattice_batch(4)
    Md, Xd = _dev(M), _dev(X)
    for k in (16, 20, 21):
        for frac in (0.0, 0.5):
            nbr = full["nbr"][:k].copy()
            drop = synthetic._rng(803).random(nbr.shape) < frac
            drop[:, 13] = False
            nbr[drop] = -1
            batch = {"S": 64, "T": k, "tgt": full["tgt"][:k], "nbr": nbr, "shift": full["shift"][:k],
                     "period": full["period"]}
            L, R = _nan(20, k * SUB3), _nan(20, k * SUB3)
            ot.Plan.from_batch(batch).multipole_batched(Md, Xd, L)
            d = {q: torch.from_numpy(np.ascontiguousarray(batch[q])).cuda() for q in ("tgt", "nbr", "shift")}
            ot.ot_fmm_multipole_batched_noalloc(64, k, d["tgt"], d["nbr"], d["shift"], batch["period"], Md, Xd, R)
            assert np.array_equal(_host(L), _host(R)), (k, frac)


@pytest.mark.parametrize("k", [21, 96, 97, 130, 150, 216])
def test_both_sides_of_a_rest(ot, k):
    """k of a periodic 6^3 lattice's sub-grids: the first and the last target of
    whole rounds (64 targets) and of what is past them, every pass."""
    rng = synthetic._rng(810 + k)
    M, X = synthetic.store_field(6, rng, 2.0, 3.0, 0.6, sep=6.0)
    full = synthetic.lattice_batch(6)
    ids = np.sort(rng.permutation(216)[:k])
    to = np.full(217, -1, np.int32)
    to[ids] = np.arange(k)
    cols = (ids[:, None] * SUB3 + np.arange(SUB3)).reshape(-1)
    M, X = np.ascontiguousarray(M[:, cols]), np.ascontiguousarray(X[:, cols])
    batch = {"S": k, "T": k, "tgt": np.arange(k, dtype=np.int32), "nbr": to[full["nbr"][ids]],
             "shift": full["shift"][ids], "period": full["period"]}
    w = synthetic.weights(k, 811)
    plan = ot.Plan.from_batch(batch)
    Md, Xd, wd = _dev(M), _dev(X), _dev(w)
    main = k - k % 64
    sel = np.unique(np.array([0, max(main - 1, 0), main % k, k - 1], np.int32))
    n = k * SUB3
    for fl in (False, True):
        ref, A = oracle.batched_forward(batch, M, X, tsel=sel, want_abs=True, full=fl)
        L, Ls, Cs = _nan(20, n), _nan(20, n), _nan(24, n)
        (plan.multipole_batched_full if fl else plan.multipole_batched)(Md, Xd, L)
        assert_parity(_pick(L, k, sel), ref, TOL, what="L", A=A)
        plan.multipole_batched_save(Md, Xd, Ls, Cs, full=fl)
        assert_parity(_pick(Ls, k, sel), ref, TOL, what="saved L", A=A)
        check_saved(_pick(Cs, k, sel), batch, M, X, "Cs", tsel=sel, full=fl)
        gM_ref, gX_ref = oracle.batched_backward(batch, M, X, w, ssel=sel, full=fl)
        gM, gX, gM2, gX2 = _nan(20, n), _nan(3, n), _nan(20, n), _nan(3, n)
        plan.multipole_backward_saved(Md, Xd, wd, Cs, gM, gX, full=fl)
        (plan.multipole_backward_full if fl else plan.multipole_backward)(Md, Xd, wd, gM2, gX2)
        assert np.array_equal(_host(gM), _host(gM2))
        assert_parity(_pick(gM, k, sel), gM_ref, TOL, what="gM")
        assert_parity(_pick(gX, k, sel), gX_ref, TOL, what="gX")
        assert_parity(_pick(gX2, k, sel), gX_ref, TOL, what="three-launch gX")
        if not fl:
            dref, dA = oracle.batched_forward_amc(batch, M, X, tsel=sel, want_abs=True)
            Lc, dF = _nan(20, n), _nan(3, n)
            plan.multipole_batched_amc(Md, Xd, Lc, dF)
            assert np.array_equal(_host(Lc), _host(Ls))
            assert_parity(_pick(dF, k, sel), dref, TOL, what="dF", A=dA)
