"""Natural-order and block red-black IC(0) sweeps where their packing can go wrong: columns shorter and longer
than a group of steps, grids below, at and past the 8x8-column tile, masks, and NaN inputs of any payload."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 1, 300), (8, 8, 1), (9, 7, 2), (7, 9, 17), (16, 17, 33), (24, 8, 64), (8, 40, 5), (65, 3, 20),
          (33, 34, 50)]
ORDERS = {"natural": (fmap.NATURAL, O.NATURAL), "blockrb": (fmap.BLOCKRB, O.BLOCKRB)}


def problem(shape, frac, seed):
    rng = np.random.default_rng(seed)
    mask = (rng.uniform(size=shape) < frac).astype(np.uint8)
    mask.flat[0] = 1
    return rng.uniform(0.01, 0.2, shape) * mask, rng.normal(size=shape) * mask, mask


def plan_for(shape, mask, prec, order):
    prm = fmap.make_params(shape, 1, [0.0, 2e-3, 5e-3], 0.1, niter=1, precision=prec, ordering=order)
    plan = fmap.Plan(prm)
    plan.setup(torch.ones((1, 3) + shape, dtype=torch.complex64, device="cuda"), None, torch.from_numpy(mask).cuda())
    return plan


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pivots_and_solve_match_oracle(shape, prec, order):
    """Pivots to 1e-12 and p to 1e-11 of its largest value in FP64; in MIX p carries the FP32 rounding of
    g, x and p (2^-24 each, growth below 1e-5 for these diagonally dominant factors)."""
    for frac in (1.0, 0.6):
        curv, g, mask = problem(shape, frac, 41)
        vol = synth.Volume(y=np.ones((1, 3) + shape, np.complex64), sens=None, te=np.array([0.0, 2e-3, 5e-3]), mask=mask,
                           f_true=np.zeros(shape), beta=0.1, niter=1)
        with plan_for(shape, mask, fmap.F64 if prec == "f64" else fmap.MIX, ORDERS[order][0]) as plan:
            piv, p = (t.cpu().numpy() for t in plan.precondition(torch.from_numpy(curv).cuda(), torch.from_numpy(g).cuda()))
        pb = O.problem_for(vol, ordering=ORDERS[order][1])
        cref = curv if prec == "f64" else curv.astype(np.float32).astype(np.float64)
        ref_piv = O.factor(pb, mask, cref)
        ref_p = O.apply(pb, mask, ref_piv, g)
        np.testing.assert_allclose(piv, ref_piv, rtol=1e-12, atol=0)
        assert np.abs(p - ref_p).max() <= (1e-11 if prec == "f64" else 1e-5) * np.abs(ref_p).max()


@pytest.mark.parametrize("prec", ["f64", "mix"])
def test_nan_of_any_payload_passes_between_tiles(prec):
    """A NaN in g, here the one with every bit set, spreads to p like any other and stalls no tile."""
    shape = (24, 24, 20)
    curv, g, mask = problem(shape, 1.0, 42)
    g.view(np.uint64)[12, 12, 10] = 0xFFFFFFFFFFFFFFFF
    with plan_for(shape, mask, fmap.F64 if prec == "f64" else fmap.MIX, fmap.NATURAL) as plan:
        _, p = plan.precondition(torch.from_numpy(curv).cuda(), torch.from_numpy(g).cuda())
        plan.status()
    p = p.cpu().numpy()
    assert np.isnan(p[12, 12, 10]) and np.isnan(p[23, 23, 19]) and np.isnan(p[0, 0, 0])


@pytest.mark.parametrize("level", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_ict_factor_and_solve_match_oracle(shape, level):
    """IC_t in tiles sheared along x: the factor and its drop set as the oracle's (same arithmetic, quotients
    correctly rounded up to an ulp: 1e-12), p to 1e-11 of its largest value."""
    for frac in (1.0, 0.6):
        curv, g, mask = problem(shape, frac, 43)
        prm = fmap.make_params(shape, 1, [0.0, 2e-3, 5e-3], 0.1, niter=1, precision=fmap.F64, precond=fmap.ICT,
                               ict_factor=1e-2, ict_level=level)
        pb = O.Problem(shape, [0.0, 2e-3, 5e-3], O.gamma_fieldmap(3), 0.1, precond=O.ICT, ict_factor=1e-2, ict_level=level)
        Lref = O.ict_factor(pb, mask, curv)
        pref = O.ict_apply(pb, mask, Lref, g)
        with fmap.Plan(prm) as plan:
            plan.setup(torch.ones((1, 3) + shape, dtype=torch.complex64, device="cuda"), None, torch.from_numpy(mask).cuda())
            piv, p = (t.cpu().numpy() for t in plan.precondition(torch.from_numpy(curv).cuda(), torch.from_numpy(g).cuda()))
            L = plan.factor().cpu().numpy()
        assert np.array_equal(L == 0, Lref == 0)
        np.testing.assert_allclose(L, Lref, rtol=1e-12, atol=0)
        np.testing.assert_allclose(piv, Lref[0] ** 2, rtol=1e-12, atol=0)
        assert np.abs(p - pref).max() <= 1e-11 * np.abs(pref).max()
