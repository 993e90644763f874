"""The water-fat sweep's value per voxel (the start with no smoothing iterations) against the oracle's direct
evaluation: each echo count with a recurrence of its own and one without, coarse and fine sweeps, voxels without
signal (every value costs 0: the first is taken)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsweep", [2, 3, 100, 257])
@pytest.mark.parametrize("necho", [3, 4, 5, 6, 7])
def test_sweep_value_is_the_direct_evaluations(necho, nsweep):
    te = [1.2e-3 + 0.9e-3 * k for k in range(necho)]
    vol = synth.waterfat_volume((9, 10, 11), 2, te, 0.1, 1, 77 + necho, 200.0, 25.0)
    y = vol.y.copy()
    y[:, :, 2:4, 3:6] = 0.0
    prm = fmap.make_params(vol.shape, 2, te, 0.1, 1, model=fmap.WATERFAT, fat_hz=vol.fat_hz, fat_amp=vol.fat_amp,
                           nsweep=nsweep, pwls_iters=0, precision=fmap.F64, ordering=fmap.REDBLACK)
    with fmap.Plan(prm) as plan:
        plan.setup(torch.from_numpy(y).cuda(), torch.from_numpy(vol.sens).cuda(), torch.from_numpy(vol.mask).cuda())
        f = plan.init().cpu().numpy()
    pb = O.Problem(vol.shape, te, O.gamma_waterfat(te, vol.fat_hz, vol.fat_amp), 0.1)
    ref = O.init_waterfat_sweep(pb, O.combine(y, vol.sens), vol.mask, vol.fat_hz[int(np.argmax(vol.fat_amp))], nsweep)
    np.testing.assert_allclose(f, ref, rtol=0, atol=1e-9)
