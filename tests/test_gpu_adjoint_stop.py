"""The adjoint stops at convergence: orders whose preconditioner is a sweep run no chunk of CG iterations past the one
that converged, the others none past the first.  A call that converges in its first chunk of 8 takes as long with 1000
iterations allowed as with 8, which is one chunk; a second chunk of sweeps would double it (bar 1.4), one of passes
that do nothing adds two fifths on a tiny volume (bar 1.2)."""
import time

import numpy as np
import pytest
import torch

from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu


def times(shape, order, precond, prec):
    """(seconds with 8 iterations allowed, with 1000, iterations of each) of an adjoint that converges at once."""
    vol = synth.fieldmap_volume(shape, 1, [0.0, 1.0e-3, 3.0e-3], 0.1, 40, 919, 3, 120.0, False, 25.0, mask="full")
    y, s, m = fmap.to_device(vol)
    g = torch.from_numpy(np.random.default_rng(35).standard_normal(shape)).cuda()
    with fmap.Plan(fmap.params_for(vol, precision=prec, ordering=order, precond=precond)) as plan:
        plan.solve(y, s, m)

        def fastest(maxit):
            best, its = 1e9, 0
            for _ in range(20):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                its = plan.adjoint(g, want_dy=False, maxit=maxit, rtol=0.5)["iters"]
                best = min(best, time.perf_counter() - t0)
            return best, its

        fastest(8)
        one, its1 = fastest(8)
        many, its2 = fastest(1000)
    print(shape, order, "%.3f ms, %.3f ms, %d iterations" % (1e3 * one, 1e3 * many, its1), flush=True)
    return one, many, its1, its2


@pytest.mark.parametrize("order", ["natural", "blockrb"])
def test_no_sweeps_after_convergence(order):
    one, many, its1, its2 = times((96, 96, 48), fmap.NATURAL if order == "natural" else fmap.BLOCKRB, fmap.IC0, fmap.MIX)
    assert its1 == its2 < 8
    assert many < 1.4 * one


@pytest.mark.parametrize("precond", ["ic0", "diag"])
@pytest.mark.parametrize("prec", ["f64", "mix"])
def test_no_second_chunk_on_a_tiny_volume(prec, precond):
    one, many, its1, its2 = times((3, 3, 4), fmap.REDBLACK, fmap.IC0 if precond == "ic0" else fmap.DIAG,
                                  fmap.F64 if prec == "f64" else fmap.MIX)
    assert its1 == its2 < 8
    assert many < 1.2 * one
