"""Single slices whose packed sweep rows would take more than 4 GiB (per tile of 8x8 columns 48.8 kB in natural order F64,
40.6 kB MIX; 36.9 and 30.7 kB in block red-black order; 93.2 and 216 kB for IC_t of levels 0 and 1): the plan takes no
such rows and sweeps by levels.  Bars: device memory of the plan at most the arrays that every order has (145 B a voxel
in F64 with 3 echoes, 82 in MIX; 72 more for IC_t level 1, 48 for level 0) and a tenth; pivots and p as for the packed
sweeps (1e-12, and 1e-11 or 1e-5 of the largest p); solves 1e-6 Hz; the adjoint after three CG iterations 1e-7."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu

TE = [0.0, 1.0e-3, 3.0e-3]
CASES = [("natural", "f64", (2401, 2399, 1), 145), ("natural", "mix", (2609, 2603, 1), 82),
         ("blockrb", "f64", (2741, 2743, 1), 145), ("blockrb", "mix", (3001, 3003, 1), 82),
         ("ict0", "f64", (1761, 1759, 1), 193), ("ict1", "f64", (1151, 1153, 1), 217)]


def plan_kw(kind, prec):
    kw = dict(precision=fmap.F64 if prec == "f64" else fmap.MIX, ordering=fmap.BLOCKRB if kind == "blockrb" else fmap.NATURAL)
    if kind.startswith("ict"):
        kw.update(precond=fmap.ICT, ict_factor=1e-2, ict_level=int(kind[3]))
    return kw


@pytest.mark.parametrize("kind,prec,shape,bytes_per_voxel", CASES, ids=lambda v: str(v))
def test_precondition_of_a_large_slice(kind, prec, shape, bytes_per_voxel):
    rng = np.random.default_rng(61)
    mask = (rng.uniform(size=shape) < 0.9).astype(np.uint8)
    curv, g = rng.uniform(0.01, 0.2, shape) * mask, rng.normal(size=shape) * mask
    prm = fmap.make_params(shape, 1, TE, 0.1, niter=1, **plan_kw(kind, prec))
    y = torch.ones((1, 3) + shape, dtype=torch.complex64, device="cuda")
    m = torch.from_numpy(mask).cuda()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with fmap.Plan(prm) as plan:
        used = (free - torch.cuda.mem_get_info()[0]) / mask.size
        print(kind, prec, shape, "%.0f B a voxel" % used, flush=True)
        plan.setup(y, None, m)
        piv, p = (t.cpu().numpy() for t in plan.precondition(torch.from_numpy(curv).cuda(), torch.from_numpy(g).cuda()))
        plan.status()
    c = curv if prec == "f64" else curv.astype(np.float32).astype(np.float64)
    if kind.startswith("ict"):
        pb = O.Problem(shape, TE, O.gamma_fieldmap(3), 0.1, precond=O.ICT, ict_factor=1e-2, ict_level=int(kind[3]))
        L = O.ict_factor(pb, mask, c)
        ref_piv, ref = L[0] ** 2, O.ict_apply(pb, mask, L, g)
    else:
        pb = O.Problem(shape, TE, O.gamma_fieldmap(3), 0.1, ordering=O.BLOCKRB if kind == "blockrb" else O.NATURAL)
        ref_piv = O.factor(pb, mask, c)
        ref = O.apply(pb, mask, ref_piv, g)
    np.testing.assert_allclose(piv, ref_piv, rtol=1e-12, atol=0)
    assert np.abs(p - ref).max() <= (1e-11 if prec == "f64" else 1e-5) * np.abs(ref).max()
    assert np.all(p[mask == 0] == 0)
    assert used < 1.1 * bytes_per_voxel


@pytest.mark.parametrize("kind,shape", [("natural", (2401, 2399, 1)), ("blockrb", (2741, 2743, 1)), ("ict1", (1151, 1153, 1))],
                         ids=["natural", "blockrb", "ict1"])
def test_solve_and_adjoint_of_a_large_slice(kind, shape):
    rng = np.random.default_rng(62)
    X, Y = np.meshgrid(np.linspace(-1, 1, shape[0]), np.linspace(-1, 1, shape[1]), indexing="ij")
    f_true = (40 * np.sin(3 * X) * np.cos(2 * Y))[:, :, None]
    yy = np.stack([np.exp(2j * np.pi * f_true * t) for t in TE])[None] + 0.02 * rng.standard_normal((1, 3) + shape)
    mask = (rng.uniform(size=shape) < 0.9).astype(np.uint8)
    vol = synth.Volume(y=yy.astype(np.complex64), sens=None, te=np.array(TE), mask=mask, f_true=f_true, beta=0.1, niter=2)
    dldf = rng.standard_normal(shape) * mask
    ict = kind == "ict1"
    y, s, m = fmap.to_device(vol)
    with fmap.Plan(fmap.params_for(vol, **plan_kw(kind, "f64"))) as plan:
        f = plan.solve(y, s, m).cpu().numpy()
        plan.status()
        if not ict:
            adj = plan.adjoint(torch.from_numpy(dldf).cuda(), want_dy=False, want_v=True, maxit=3, rtol=0.0)
            f3 = plan.iterate(1)  # the chain goes on after the adjoint
            plan.status()
            assert torch.isfinite(f3).all()
    od = O.BLOCKRB if kind == "blockrb" else O.NATURAL
    ref = O.run_volume(vol, ordering=od, precond=O.ICT if ict else O.IC0, ict_factor=1e-2, ict_level=1)
    print(kind, "max %.2e Hz" % np.abs(f - ref["f"]).max(), flush=True)
    assert np.abs(f - ref["f"]).max() < 1e-6
    if not ict:
        v, _, _, _ = O.adjoint(O.problem_for(vol, O.NATURAL), O.combine(vol.y, vol.sens), mask, f, dldf, maxit=3, rtol=0.0)
        assert np.linalg.norm(adj["v"].cpu().numpy() - v) < 1e-7 * np.linalg.norm(v)
