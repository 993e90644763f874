"""The adjoint's CG in voxel pairs (red-black IC(0), even columns) and its four-voxel update, on columns of 2, 12 and
14 voxels with holes in the mask, against the oracle's adjoint at the GPU's map.  Bars: both CGs to 1e-12 in F64
(1e-7), FP32 vectors and CG to 1e-6 in MIX (1e-3)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("shape", [(9, 7, 2), (17, 9, 12), (8, 15, 14)], ids=lambda s: "x".join(map(str, s)))
def test_adjoint_matches_oracle(shape, prec):
    vol = synth.fieldmap_volume(shape, 2, [0.0, 1.0e-3, 3.0e-3], 0.1, 300, 913, 3, 120.0, False, 25.0)
    rng = np.random.default_rng(31)
    vol.mask = (rng.uniform(size=shape) < 0.85).astype(np.uint8)
    dldf = rng.standard_normal(shape) * vol.mask
    y, s, m = fmap.to_device(vol)
    f64 = prec == "f64"
    with fmap.Plan(fmap.params_for(vol, precision=fmap.F64 if f64 else fmap.MIX, ordering=fmap.REDBLACK)) as plan:
        f = plan.solve(y, s, m).cpu().numpy()
        out = plan.adjoint(torch.from_numpy(dldf).cuda(), want_v=True, rtol=1e-12 if f64 else 1e-6)
    v, db, dz, its = O.adjoint(O.problem_for(vol, O.REDBLACK), O.combine(vol.y, vol.sens), vol.mask, f, dldf, maxit=2000,
                               rtol=1e-12)
    bar = 1e-7 if f64 else 1e-3
    rel = lambda a, b: np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b))  # noqa: E731
    assert rel(out["v"].cpu().numpy(), v) < bar
    assert abs(out["dbeta"] - db) <= bar * abs(db)
    assert rel(out["dy"].cpu().numpy(), O.zhat_to_y_grad(dz, vol.sens, vol.ncoil)) < bar
    if f64:
        assert abs(out["iters"] - its) <= 1
