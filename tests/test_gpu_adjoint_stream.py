"""The adjoint's first call on a plan, on a stream of its own: the workspace is cleared on that stream, whatever the
default stream still has to do.  Bars as for the other adjoints: both CGs to 1e-12 in F64 (1e-7), FP32 vectors and CG
to 1e-6 in MIX (1e-3)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("order", ["blockrb", "natural", "redblack"])
def test_first_adjoint_on_a_side_stream(order, prec):
    shape = (25, 26, 19)
    vol = synth.fieldmap_volume(shape, 2, [0.0, 1.0e-3, 3.0e-3], 0.1, 200, 917, 3, 120.0, False, 25.0)
    rng = np.random.default_rng(33)
    vol.mask = (rng.uniform(size=shape) < 0.9).astype(np.uint8)
    dldf = rng.standard_normal(shape) * vol.mask
    y, s, m = fmap.to_device(vol)
    g = torch.from_numpy(dldf).cuda()
    work = torch.randn(4096, 4096, device="cuda")
    f64 = prec == "f64"
    od = {"blockrb": fmap.BLOCKRB, "natural": fmap.NATURAL, "redblack": fmap.REDBLACK}[order]
    side = torch.cuda.Stream()
    with fmap.Plan(fmap.params_for(vol, precision=fmap.F64 if f64 else fmap.MIX, ordering=od)) as plan:
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            f = plan.solve(y, s, m)
        side.synchronize()
        for _ in range(20):  # the default stream is busy while the workspace is cleared and used
            work = work @ work
            work /= work.abs().max()
        with torch.cuda.stream(side):
            out = plan.adjoint(g, want_v=True, rtol=1e-12 if f64 else 1e-6)
        torch.cuda.synchronize()
    v, db, dz, _ = O.adjoint(O.problem_for(vol, O.NATURAL), O.combine(vol.y, vol.sens), vol.mask, f.cpu().numpy(), dldf,
                             maxit=2000, rtol=1e-12)
    bar = 1e-7 if f64 else 1e-3
    rel = lambda a, b: np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b))  # noqa: E731
    assert rel(out["v"].cpu().numpy(), v) < bar
    assert abs(out["dbeta"] - db) <= bar * abs(db)
    assert rel(out["dy"].cpu().numpy(), O.zhat_to_y_grad(dz, vol.sens, vol.ncoil)) < bar
