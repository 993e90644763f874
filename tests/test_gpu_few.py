"""A thread per voxel and runs of one to three planes: volumes around the largest that take a voxel per thread
(262 144 in F64, 131 072 in MIX), around the tile runs' steps, and of a few voxels, on the streaming schedule against
the oracle (bars as in the tile tests: F64 1e-6 Hz, MIX 0.05 Hz RMS)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu

# the last with a thread per voxel and the first without: 64x64x64, 64x65x64 (F64), 64x64x32, 64x33x64 (MIX);
# 20x30x40 and 60x30x40: one and two planes a run; 2x3x2: less than a wavefront
CASES = [((64, 64, 64), 3), ((64, 65, 64), 3), ((64, 64, 32), 3), ((64, 33, 64), 3), ((20, 30, 40), 6), ((60, 30, 40), 6),
         ((2, 3, 2), 8)]


@pytest.mark.parametrize("order", ["redblack", "diag", "natural"])
@pytest.mark.parametrize("prec", ["f64", "mix"])
@pytest.mark.parametrize("shape,niter", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_small_volumes_match_oracle(shape, niter, prec, order):
    vol = synth.fieldmap_volume(shape, 2, [0.0, 1.5e-3, 4.0e-3], 0.2, niter, synth.SEED_BASE + 1400 + sum(shape), 3, 120.0,
                                False, 25.0, mask="full")
    vol.mask = (np.random.default_rng(sum(shape)).uniform(size=shape) < 0.85).astype(np.uint8)
    msk = vol.mask.astype(bool)
    od, pc = (O.NATURAL, O.IC0) if order == "natural" else (O.REDBLACK, O.DIAG if order == "diag" else O.IC0)
    y, s, m = fmap.to_device(vol, "cuda:0")
    with fmap.Plan(fmap.params_for(vol, precision=fmap.F64 if prec == "f64" else fmap.MIX, ordering=od, precond=pc)) as plan:
        plan.set_schedule(fmap.SCHED_STREAM)
        f = plan.solve(y, s, m).cpu().numpy()
        plan.status()
    d = np.abs(f - O.run_volume(vol, ordering=od, precond=pc)["f"])[msk]
    print(shape, prec, order, "max %.2e Hz" % d.max(), flush=True)
    assert np.all(f[~msk] == 0)
    assert d.max() < 1e-6 if prec == "f64" else np.sqrt(np.mean(d ** 2)) < 0.05
