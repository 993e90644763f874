"""Passes that only larger volumes take, at the smallest volumes that take them: the four-voxel passes of FP32 volumes
past 131 072 voxels for every echo count, with their early loads from 2^21 voxels on; columns that the plan pads to a
multiple of 4; runs of one to four planes in the tile passes; and fm_solve_noalloc with padded columns and where only
the caller's columns fit its array.  Bars as in the tests of the smaller volumes: F64 1e-6 Hz, MIX 0.05 Hz RMS (with the
cost trace to 1e-4 where it is compared); calls that do not iterate, the bits of the same plan in natural order, whose
arrays are not padded (the water-fat start 1e-9: its CG sums in another order); the adjoint 1e-3 in MIX."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu

CUDA = "cuda:0"


def volume(shape, necho, niter, seed, wf=False):
    if wf:
        vol = synth.waterfat_volume(shape, 2, 1.2e-3 + 1e-3 * np.arange(necho), 2.0 ** -4, niter, synth.SEED_BASE + seed, 150.0,
                                    40.0)
    else:
        te = 1.0e-3 * np.arange(necho) * (2.2 if necho <= 3 else 1.1)
        vol = synth.fieldmap_volume(shape, 2, te, 0.2, niter, synth.SEED_BASE + seed, 3, 100.0, False, 25.0, mask="full")
    vol.mask = (np.random.default_rng(seed).uniform(size=shape) < 0.85).astype(np.uint8)
    return vol


def solve(vol, prec, diag=False):
    """(map, trace) on the streaming schedule."""
    y, s, m = fmap.to_device(vol, CUDA)
    prm = fmap.params_for(vol, precision=prec, ordering=fmap.REDBLACK, precond=fmap.DIAG if diag else fmap.IC0)
    with fmap.Plan(prm) as plan:
        plan.set_schedule(fmap.SCHED_STREAM)
        f = plan.solve(y, s, m).cpu().numpy()
        plan.status()
        return f, plan.trace()


def check(vol, f, prec, tr=None, diag=False):
    msk = vol.mask.astype(bool)
    ref = O.run_volume(vol, ordering=O.REDBLACK, precond=O.DIAG if diag else O.IC0)
    d = np.abs(f - ref["f"])[msk]
    print(vol.shape, vol.necho, "max %.2e rms %.2e Hz" % (d.max(), np.sqrt(np.mean(d ** 2))), flush=True)
    assert np.all(f[~msk] == 0)
    assert d.max() < 1e-6 if prec == fmap.F64 else np.sqrt(np.mean(d ** 2)) < 0.05
    if tr is not None:
        np.testing.assert_allclose(tr[:, 0], ref["trace"][:, O.TR["cost"]], rtol=1e-4)


@pytest.mark.parametrize("diag", [False, True], ids=["ic0", "diag"])
@pytest.mark.parametrize("necho", [2, 3, 4, 5, 6])
def test_four_voxel_passes(necho, diag):
    vol = volume((64, 65, 36), necho, 8, 1800 + necho)
    f, tr = solve(vol, fmap.MIX, diag)
    check(vol, f, fmap.MIX, tr, diag)


@pytest.mark.parametrize("necho", [2, 3, 4])
def test_early_loads(necho):
    """2^21 voxels, the first with two fours or more per thread, and a ragged volume past them."""
    for shape in ((128, 128, 128), (130, 129, 132)):
        vol = volume(shape, necho, 2, 1810 + necho)
        f, tr = solve(vol, fmap.MIX)
        check(vol, f, fmap.MIX, tr)


# 33 -> 36 (odd) and 34 -> 36, 18 -> 20 (even; six echoes and the diagonal preconditioner are never resident)
@pytest.mark.parametrize("shape,wf,diag", [((75, 60, 33), False, False), ((75, 60, 33), False, True), ((70, 60, 34), False, True),
                                           ((64, 64, 34), True, False), ((90, 85, 18), True, False)],
                         ids=["33", "33-diag", "34-diag", "34-six-echoes", "18-six-echoes"])
def test_columns_padded_to_a_multiple_of_four(shape, wf, diag):
    vol = volume(shape, 6 if wf else 3, 6, 1820 + shape[2], wf)
    msk = vol.mask.astype(bool)
    rng = np.random.default_rng(5)
    f0 = rng.uniform(-40, 40, shape) * msk
    curv, g = np.abs(rng.standard_normal(shape)) * 0.1 * msk, rng.standard_normal(shape) * msk
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(CUDA)  # noqa: E731
    y, s, m = fmap.to_device(vol, CUDA)
    pc, po = (fmap.DIAG, O.DIAG) if diag else (fmap.IC0, O.IC0)
    out = {}
    for order, precond in ((fmap.NATURAL, fmap.IC0), (fmap.REDBLACK, pc)):
        with fmap.Plan(fmap.params_for(vol, precision=fmap.MIX, ordering=order, precond=precond)) as plan:
            plan.setup(y, s, m)
            out[order] = [t.cpu().numpy() for t in [plan.init()] + list(plan.eval(dev(f0))) + [plan.components(dev(f0))]]
            assert plan.mask_count() == int(msk.sum())
            if order == fmap.NATURAL:
                continue
            piv, p = (t.cpu().numpy() for t in plan.precondition(dev(curv), dev(g)))
            assert plan.schedule() == fmap.SCHED_STREAM
            f = plan.solve(y, s, m).cpu().numpy()
            plan.status()
            check(vol, f, fmap.MIX, diag=diag)
            if not wf:  # (a water-fat map far from its minimum need not have a positive definite Hessian)
                fa = plan.iterate(150).cpu().numpy()
                adj = plan.adjoint(dev(g), want_v=True, rtol=1e-6)
    for a, b in zip(out[fmap.NATURAL], out[fmap.REDBLACK]):
        if wf:
            np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9)
        else:
            np.testing.assert_array_equal(a, b)
    if not diag:
        pb = O.problem_for(vol, ordering=O.REDBLACK, precond=po)
        rp = O.factor(pb, vol.mask, curv.astype(np.float32).astype(np.float64))
        ref = O.apply(pb, vol.mask, rp, g)
        np.testing.assert_allclose(piv, rp, rtol=1e-12, atol=0)
        assert np.abs(p - ref).max() <= 1e-5 * np.abs(ref).max()
    if not wf:
        v, db, dz, _ = O.adjoint(O.problem_for(vol, O.REDBLACK, po), O.combine(vol.y, vol.sens), vol.mask, fa, g, maxit=2000,
                                 rtol=1e-12)
        rel = lambda a, b: np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b))  # noqa: E731
        assert rel(adj["v"].cpu().numpy(), v) < 1e-3 and abs(adj["dbeta"] - db) <= 1e-3 * abs(db)
        assert rel(adj["dy"].cpu().numpy(), O.zhat_to_y_grad(dz, vol.sens, vol.ncoil)) < 1e-3


# Strips of ty columns (256 pairs of a plane) x planes, 256 of them to a run of one plane, at most four:
# 4 planes and a last run of 1; 2; 3 and a last run of 2; 4 with strips of 8, 8 and 1 columns and a last run of 2; 1
RUNS = [((1037, 3, 2), 4), ((530, 5, 2), 4), ((800, 4, 6), 4), ((350, 17, 64), 2), ((255, 6, 4), 4)]


@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("shape,niter", RUNS, ids=["x".join(map(str, r[0])) for r in RUNS])
def test_runs_of_planes(shape, niter, prec):
    vol = volume(shape, 3, niter, 1830 + shape[0])
    pr = fmap.F64 if prec == "f64" else fmap.MIX
    f, _ = solve(vol, pr)
    check(vol, f, pr)


def noalloc(vol, prec):
    y, s, m = fmap.to_device(vol, CUDA)
    prm = fmap.params_for(vol, precision=prec, ordering=fmap.REDBLACK)
    out = torch.full(vol.shape, 7.0, dtype=torch.float64, device=CUDA)
    status = torch.full((1,), -1, dtype=torch.int32, device=CUDA)
    fmap.solve_noalloc(prm, y, s, m, out=out, status=status)
    assert int(status.item()) == 0
    return out.cpu().numpy()


@pytest.mark.parametrize("shape", [(75, 60, 33), (60, 66, 34)], ids=["33", "34"])
def test_noalloc_with_padded_columns(shape):
    """The streamed plan's map, bit for bit."""
    vol = volume(shape, 3, 6, 1840 + shape[2])
    np.testing.assert_array_equal(noalloc(vol, fmap.MIX), solve(vol, fmap.MIX)[0])


def test_noalloc_where_only_the_callers_columns_fit():
    """6x4695x9 F64 with 4 echoes takes 48.0 MB of the 50.3 MB array as it is, 53 MB with columns of 10."""
    vol = volume((6, 4695, 9), 4, 4, 1850)
    check(vol, noalloc(vol, fmap.F64), fmap.F64)
