"""NaN and infinities in the preconditioner step stay in their part of the mask: the sweeps that keep lanes without a
voxel in step (natural and block red-black IC(0), IC_t of levels 0 and 1) select such lanes' values, they never multiply
them by zero.  Level 2, one launch per level, is held to the same.  Bars as for the finite sweeps: p to 1e-11 (F64) or
1e-5 (MIX, FP32 rounding of g, x and p) of its largest value."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap

pytestmark = pytest.mark.gpu

TE = [0.0, 2e-3, 5e-3]
SHAPE = (20, 19, 18)
KINDS = ["natural", "blockrb", "ict0", "ict1", "ict2"]
PREC = {"f64": fmap.F64, "mix": fmap.MIX}


def step(kind, prec, mask, curv, g, ict_factor=1e-2):
    """(p, factor or None) of the GPU, with the status checked."""
    kw = dict(precision=PREC[prec], ordering=fmap.BLOCKRB if kind == "blockrb" else fmap.NATURAL)
    if kind.startswith("ict"):
        kw.update(precond=fmap.ICT, ict_factor=ict_factor, ict_level=int(kind[3]))
    with fmap.Plan(fmap.make_params(mask.shape, 1, TE, 0.1, niter=1, **kw)) as plan:
        plan.setup(torch.ones((1, 3) + mask.shape, dtype=torch.complex64, device="cuda"), None,
                   torch.from_numpy(mask).cuda())
        _, p = plan.precondition(torch.from_numpy(curv).cuda(), torch.from_numpy(g).cuda())
        L = plan.factor().cpu().numpy() if kind.startswith("ict") else None
        plan.status()
    return p.cpu().numpy(), L


def oracle_step(kind, prec, mask, curv, g, ict_factor=1e-2):
    with np.errstate(over="ignore"):
        c = curv.astype(np.float32).astype(np.float64) if prec == "mix" else curv
    if kind.startswith("ict"):
        pb = O.Problem(mask.shape, TE, O.gamma_fieldmap(3), 0.1, precond=O.ICT, ict_factor=ict_factor, ict_level=int(kind[3]))
        L = O.ict_factor(pb, mask, c)
        return O.ict_apply(pb, mask, L, g), L
    pb = O.Problem(mask.shape, TE, O.gamma_fieldmap(3), 0.1, ordering=O.BLOCKRB if kind == "blockrb" else O.NATURAL)
    return O.apply(pb, mask, O.factor(pb, mask, c), g), None


def inputs(mask, seed):
    rng = np.random.default_rng(seed)
    return rng.uniform(0.01, 0.2, mask.shape) * mask, rng.normal(size=mask.shape) * mask


@pytest.mark.parametrize("value", [np.nan, np.inf], ids=["nan", "inf"])
@pytest.mark.parametrize("axis", [0, 1, 2], ids="xyz")
@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("kind", KINDS)
def test_two_parts_of_the_mask(kind, prec, axis, value):
    """A slab outside the mask between two parts, as thick as the pattern's reach needs (level 2 has entries two voxels
    away); either part stays the oracle's when the other has a value that is not finite."""
    mask = np.ones(SHAPE, np.uint8)
    mask[np.random.default_rng(3).uniform(size=SHAPE) < 0.1] = 0
    cut = 10
    np.moveaxis(mask, axis, 0)[cut:cut + (2 if kind == "ict2" else 1)] = 0
    curv, g = inputs(mask, 51)
    ref, _ = oracle_step(kind, prec, mask, curv, g)
    part = np.zeros(SHAPE, bool)
    np.moveaxis(part, axis, 0)[:cut] = True
    for bad in (part, ~part):
        gb = g.copy()
        where = np.argwhere(bad & (mask != 0))
        gb[tuple(where[len(where) // 2])] = value
        p, _ = step(kind, prec, mask, curv, gb)
        print(kind, prec, "xyz"[axis], value, flush=True)
        assert not np.isfinite(p[bad]).all()
        assert np.all(p[mask == 0] == 0)
        assert np.abs(p - ref)[~bad].max() <= (1e-11 if prec == "f64" else 1e-5) * np.abs(ref).max()


@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("kind", KINDS)
def test_infinite_gradient_of_a_lone_voxel(kind, prec):
    """p of a voxel without neighbours is g / H: infinite where g is."""
    mask = np.zeros((9, 10, 11), np.uint8)
    mask[4, 5, 6] = mask[8, 9, 10] = 1
    curv, g = inputs(mask, 52)
    ref, _ = oracle_step(kind, prec, mask, curv, g)
    g[4, 5, 6] = -np.inf
    p, _ = step(kind, prec, mask, curv, g)
    assert p[4, 5, 6] == -np.inf and np.count_nonzero(p) == 2
    assert abs(p[8, 9, 10] - ref[8, 9, 10]) <= (1e-11 if prec == "f64" else 1e-5) * abs(ref[8, 9, 10])


@pytest.mark.parametrize("ict_factor", [0.0, 1e-2])
@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("kind", KINDS)
def test_infinite_curvature(kind, prec, ict_factor):
    """A voxel of infinite curvature (in MIX 1e50 is one) has p = 0 and the factor sqrt(inf); nothing else is touched."""
    mask = np.ones(SHAPE, np.uint8)
    curv, g = inputs(mask, 53)
    curv[7, 9, 8] = np.inf if prec == "f64" else 1e50
    p, L = step(kind, prec, mask, curv, g, ict_factor)
    ref, Lref = oracle_step(kind, prec, mask, curv, g, ict_factor)
    assert p[7, 9, 8] == 0
    assert np.abs(p - ref).max() <= (1e-11 if prec == "f64" else 1e-5) * np.abs(ref).max()
    if L is not None:
        assert np.array_equal(L == 0, Lref == 0)
        np.testing.assert_allclose(L, Lref, rtol=1e-12, atol=0)
