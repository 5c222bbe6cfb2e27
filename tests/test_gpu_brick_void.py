"""Tiles of cells without home particles: a box that fills the lower part of its
height, whose last tiles are empty and hold the end of the particle arrays
(65,536 records of 32 bytes: an allocation that ends there exactly), against the
gather and the row-tile kernels."""
import numpy as np
import pytest

import initconf
from gpu_common import floored_err, lib_params
from test_gpu_brick import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path,other", [(0, {"path": 1}), (3, {"path": 3, "tile_cells": 4})])
@pytest.mark.parametrize("precision", [0, 1])
def test_slab_with_a_void_at_the_end(torch_cuda, path, other, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case slab path={path} precision={precision}", flush=True)
    n, fill = 65536, 0.84
    s = initconf.fcc_system(n, rho=1.2, seed=21, temperature=0.5, jitter=0.05)
    x = s["x"].copy()
    x[:, 2] *= fill
    out = []
    for kw in ({"path": path}, other):
        sysm = System(lib_params(precision=precision, dt=0.001, **kw), [n], [s["L"]])
        sysm.set_state(x, s["v"], s["type"])
        if path == 0:  # the forms that each path tries
            assert (len(sysm.autotune(reps=1)["tried"]) == 2) == (kw["path"] == 0)
        nc = sysm.replica_info(0)["nc"]
        sysm.forces()
        F = sysm.get_forces().cpu().numpy().astype(np.float64)
        cs, _ = sysm.get_cells(0)
        assert cs[(nc - 2) * nc * nc] == n  # the top two layers are empty
        sysm.step(6)
        xs, vs, img = (a.cpu().numpy() for a in sysm.get_state())
        out.append((F, xs + img * s["L"], vs))
        sysm.close()
    assert floored_err(out[0][0], out[1][0]) <= (2e-12 if precision == 0 else 2e-5)
    # six steps of 0.001 on forces that differ by at most e: dv <= 6 dt e and
    # dx <= 6 dt dv, twice that for the answer of the forces; 1e-13 for the
    # rounding of six position updates
    fmax = float(np.max(np.abs(out[1][0])))
    e = (2e-12 if precision == 0 else 2e-5) * fmax
    assert np.max(np.abs(out[0][2] - out[1][2])) <= 0.012 * e
    assert np.max(np.abs(out[0][1] - out[1][1])) <= 0.012 * 0.006 * e + 1e-13
