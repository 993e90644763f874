"""Lines of the rules that choose passes by size.  The thread-per-voxel rule in FP64 (65 536 voxels for second order and for the diagonal preconditioner
with up to 4 echoes, 196 608 for the rest): the last volume below and the first above each, on the streaming schedule
against the oracle (1e-6 Hz; where its factor breaks down, the same status), and past the line no more time a voxel
than a larger volume takes (the second-order diagonal, where a thread per voxel cost a fifth at 245 760 voxels).  And the columns that are padded:
in FP64 with a thread per voxel from 65 536 voxels on, and for the diagonal in FP32 above 2^20, only by a fifteenth; a
volume that its padding takes past the line has several voxels a thread (FP32 bar: 0.05 Hz RMS)."""
import time

import numpy as np
import pytest
import torch

import oracle as O
from paper_2005_08661_amd import fmap, synth

pytestmark = pytest.mark.gpu

CASES = [("diag", 3, (64, 32, 32)), ("diag", 3, (65, 32, 32)), ("diag", 6, (65, 32, 32)), ("order2-diag", 3, (64, 32, 32)),
         ("order2-diag", 3, (65, 32, 32)), ("order2-ic0", 3, (64, 32, 32)), ("order2-ic0", 3, (65, 32, 32)),
         ("redblack", 3, (64, 64, 48)), ("redblack", 3, (64, 65, 48)), ("blockrb", 3, (64, 64, 48)), ("blockrb", 6, (64, 65, 48)),
         ("diag", 6, (64, 64, 48)), ("diag", 6, (64, 65, 48))]


def setting(kind, necho, shape, niter):
    vol = synth.fieldmap_volume(shape, 2, 1.1e-3 * np.arange(necho), 0.2, niter, synth.SEED_BASE + 1900 + sum(shape), 3, 100.0,
                                False, 25.0, mask="full")
    vol.mask = (np.random.default_rng(sum(shape)).uniform(size=shape) < 0.85).astype(np.uint8)
    vol.reg_order = 2 if kind.startswith("order2") else 1
    order = {"order2-ic0": fmap.COLOR3, "order2-diag": fmap.NATURAL, "blockrb": fmap.BLOCKRB}.get(kind, fmap.REDBLACK)
    return vol, dict(ordering=order, precond=fmap.DIAG if kind.endswith("diag") else fmap.IC0)


@pytest.mark.parametrize("kind,necho,shape", CASES, ids=lambda v: str(v))
def test_either_side_matches_oracle(kind, necho, shape):
    vol, kw = setting(kind, necho, shape, 4)
    y, s, m = fmap.to_device(vol, "cuda:0")
    with fmap.Plan(fmap.params_for(vol, precision=fmap.F64, **kw)) as plan:
        f = plan.solve(y, s, m).cpu().numpy()
        try:
            ref = O.run_volume(vol, **kw)  # (the oracle's constants are the same)
        except O.OracleError as e:  # a non-positive pivot (65x32x32 with IC(0) of second order)
            assert "error 5" in str(e)
            with pytest.raises(fmap.FmapError, match="error 5"):
                plan.status()
            return
        plan.status()
    assert np.all(f[vol.mask == 0] == 0)
    assert np.abs(f - ref["f"]).max() < 1e-6


# F64: 9 and 13 not padded, 15 -> 16; below 65 536 voxels 9 -> 10; past 196 608 by their padding 145x145x9, 105x106x17
# and 88x88x25.  MIX diagonal: 25 not padded above 2^20 voxels, 30 -> 32; below, 25 -> 28
COLUMNS = [("redblack", "f64", (105, 105, 9)), ("redblack", "f64", (85, 84, 13)), ("redblack", "f64", (81, 82, 15)),
           ("redblack", "f64", (85, 85, 9)), ("redblack", "f64", (145, 145, 9)), ("redblack", "f64", (105, 106, 17)),
           ("redblack", "f64", (88, 88, 25)), ("diag", "mix", (210, 210, 25)), ("diag", "mix", (190, 190, 30)),
           ("diag", "mix", (100, 99, 25))]


@pytest.mark.parametrize("kind,prec,shape", COLUMNS, ids=lambda v: str(v))
def test_columns_either_side_match_oracle(kind, prec, shape):
    vol, kw = setting(kind, 3, shape, 3)
    y, s, m = fmap.to_device(vol, "cuda:0")
    with fmap.Plan(fmap.params_for(vol, precision=fmap.F64 if prec == "f64" else fmap.MIX, **kw)) as plan:
        f = plan.solve(y, s, m).cpu().numpy()
        plan.status()
    d = np.abs(f - O.run_volume(vol, **kw)["f"])[vol.mask != 0]
    assert np.all(f[vol.mask == 0] == 0)
    assert d.max() < 1e-6 if prec == "f64" else np.sqrt(np.mean(d ** 2)) < 0.05


def test_no_more_time_a_voxel_than_a_larger_volume():
    took = []
    for shape in ((64, 64, 60), (64, 65, 64)):
        vol, kw = setting("order2-diag", 3, shape, 40)
        y, s, m = fmap.to_device(vol, "cuda:0")
        with fmap.Plan(fmap.params_for(vol, precision=fmap.F64, **kw)) as plan:
            out = plan.solve(y, s, m)
            best = 1e9
            for _ in range(8):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                plan.solve(y, s, m, out=out)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t0)
            took.append(best)
    print("%.3f ms, %.3f ms" % (1e3 * took[0], 1e3 * took[1]), flush=True)
    assert took[0] / took[1] < (64 * 64 * 60) / (64 * 65 * 64)
