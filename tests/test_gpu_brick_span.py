"""A list capacity with which the rows of one tile would lie more than 4 GiB
apart, beyond what the force kernel addresses: the same bits as with the default
capacity, and the same list."""
import numpy as np
import pytest

import initconf
from gpu_common import lib_params
from test_gpu_brick import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
def test_rows_of_a_tile_far_apart(torch_cuda, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case far rows precision={precision}", flush=True)
    n = 6000
    s = initconf.fcc_system(n, seed=3, temperature=1.0)
    # six cells a side, tiles of two: rows of a tile's two layers are 42
    # cells of 27.8 particles apart, four blocks of 256 rows and more
    cap = 2400000
    assert 4 * 256 * (cap // 8) * 16 > 2 ** 32
    out = []
    for kw in ({}, {"max_neighbors": cap}):
        sysm = System(lib_params(precision=precision, **kw), [n], [s["L"]])
        sysm.set_state(s["x"], s["v"], s["type"])
        sysm.forces()
        F = sysm.get_forces().cpu().numpy()
        sysm.step(5)
        count, ids = sysm.get_neighbors(0, cap=160)
        out.append([F, count, ids] + [a.cpu().numpy() for a in sysm.get_state()])
        assert sysm.replica_info(0)["nc"] == 6
        sysm.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
