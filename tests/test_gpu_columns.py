"""Columns of odd or other lengths that the plan's own arrays pad (red-black IC(0), the diagonal preconditioner): every
entry point that takes or returns volumes, with a hole-ridden mask that touches the last voxel of columns.  The calls
that do not iterate run the same arithmetic per voxel as a natural-order plan, whose arrays are not padded, so their
results are the same bits; the solve is compared with the oracle (bars: F64 1e-6 Hz as for the other orders, MIX 0.05 Hz
RMS)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu

CUDA = "cuda:0"
PREC = {"f64": fmap.F64, "mix": fmap.MIX}


def volume(nz, wf):
    shape = (11, 13, nz)
    if wf:
        vol = synth.waterfat_volume(shape, 3, 1.2e-3 + 1e-3 * np.arange(6), 2.0 ** -4, 8, synth.SEED_BASE + 61, 150.0, 40.0)
    else:
        vol = synth.fieldmap_volume(shape, 3, [0.0, 1.0e-3, 3.0e-3], 0.1, 8, synth.SEED_BASE + 62, 3, 120.0, False, 25.0)
    vol.mask = (np.random.default_rng(nz).uniform(size=shape) < 0.85).astype(np.uint8)
    return vol


# 15: up to 16; 9: up to 10; 33: MIX up to 36, F64 up to 34; 18: MIX up to 20 (six echoes: never resident)
@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("nz,wf", [(15, False), (9, False), (33, False), (18, True), (33, True)])
def test_every_call_on_padded_columns(nz, wf, prec):
    vol = volume(nz, wf)
    msk = vol.mask.astype(bool)
    rng = np.random.default_rng(5)
    f0 = rng.uniform(-40, 40, vol.shape) * msk
    curv = np.abs(rng.standard_normal(vol.shape)) * 0.1
    g = rng.standard_normal(vol.shape) * msk
    y, s, m = fmap.to_device(vol, CUDA)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(CUDA)  # noqa: E731
    out = {}
    for order in (fmap.NATURAL, fmap.REDBLACK):
        with fmap.Plan(fmap.params_for(vol, precision=PREC[prec], ordering=order)) as plan:
            plan.setup(y, s, m)
            calls = [plan.init()] + list(plan.eval(dev(f0))) + [plan.components(dev(f0))]
            out[order] = [t.cpu().numpy() for t in calls]
            assert plan.mask_count() == int(msk.sum())
            if order == fmap.REDBLACK:
                piv, p = (t.cpu().numpy() for t in plan.precondition(dev(curv * msk), dev(g)))
    for a, b in zip(out[fmap.NATURAL], out[fmap.REDBLACK]):
        if wf:  # the start's CG sums its partials in another order
            np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9)
        else:
            np.testing.assert_array_equal(a, b)
    pb = O.problem_for(vol, ordering=O.REDBLACK)
    cm = (curv * msk).astype(np.float32).astype(np.float64) if prec == "mix" else curv * msk
    rp = O.factor(pb, vol.mask, cm)
    np.testing.assert_allclose(piv, rp, rtol=1e-12, atol=0)
    ref = O.apply(pb, vol.mask, rp, g)
    assert np.abs(p - ref).max() <= (1e-11 if prec == "f64" else 1e-5) * np.abs(ref).max()


@pytest.mark.parametrize("precond", ["ic0", "diag"])
@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("nz,wf", [(15, False), (9, False), (33, False), (18, True), (257, False)])
def test_solve_and_adjoint_on_padded_columns(nz, wf, prec, precond):
    vol = volume(nz, wf)
    msk = vol.mask.astype(bool)
    f0 = np.random.default_rng(6).uniform(-40, 40, vol.shape) * msk
    y, s, m = fmap.to_device(vol, CUDA)
    pc, po = (fmap.IC0, O.IC0) if precond == "ic0" else (fmap.DIAG, O.DIAG)
    with fmap.Plan(fmap.params_for(vol, precision=PREC[prec], ordering=fmap.REDBLACK, precond=pc)) as plan:
        for start in (None, f0):
            f = plan.solve(y, s, m, f0=None if start is None else torch.from_numpy(start).to(CUDA)).cpu().numpy()
            plan.status()
            ref = O.run_volume(vol, ordering=O.REDBLACK, precond=po, f0=start)
            err = np.abs(f - ref["f"])[msk]
            print(nz, wf, prec, precond, "max %.2e rms %.2e" % (err.max(), np.sqrt(np.mean(err ** 2))), flush=True)
            assert np.all(f[~msk] == 0)
            assert err.max() < 1e-6 if prec == "f64" else np.sqrt(np.mean(err ** 2)) < 0.05
        f = plan.iterate(150).cpu().numpy()
        dldf = np.random.default_rng(7).standard_normal(vol.shape) * msk
        if wf or nz == 257:
            return  # a start far from a minimum of a non-convex cost: the Hessian need not be positive definite
        adj = plan.adjoint(torch.from_numpy(dldf).to(CUDA), want_v=True, rtol=1e-12 if prec == "f64" else 1e-6)
    v, db, dz, _ = O.adjoint(O.problem_for(vol, O.REDBLACK), O.combine(vol.y, vol.sens), vol.mask, f, dldf, maxit=2000,
                             rtol=1e-12)
    bar = 1e-7 if prec == "f64" else 1e-3
    rel = lambda a, b: np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b))  # noqa: E731
    assert rel(adj["v"].cpu().numpy(), v) < bar and abs(adj["dbeta"] - db) <= bar * abs(db)
    assert rel(adj["dy"].cpu().numpy(), O.zhat_to_y_grad(dz, vol.sens, vol.ncoil)) < bar
