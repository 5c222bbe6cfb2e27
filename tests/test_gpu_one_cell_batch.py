"""Batches of one-cell boxes on both sides of the list build's block limit
(8,192 blocks, 64 to a tile of 256 particles): every replica gives the bits of a
context of its own, with the replicas rebuilding on different steps."""
import numpy as np
import pytest

import initconf
from gpu_common import lib_params
from test_gpu_brick import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrep,precision", [(64, 0), (65, 1), (200, 0), (200, 1)])
def test_replicas_alone_and_in_a_batch(torch_cuda, nrep, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case one-cell batch nrep={nrep} precision={precision}", flush=True)
    sizes = [500 - k % 7 for k in range(nrep)]  # two tiles each
    temps = [0.5 + 0.02 * (k % 61) for k in range(nrep)]
    systems = initconf.batched_systems(sizes, temps, seed=71)
    x, v, t, n, L = initconf.concat_replicas(systems)
    big = System(lib_params(precision=precision), n, L)
    assert big.replica_info(0)["nc"] == 1
    big.set_state(x, v, t)
    big.step(30, T0=temps)
    gx, gv, gimg = (a.cpu().numpy() for a in big.get_state())
    ob = big.observables()
    big.close()
    for r in (0, 1, nrep // 2, nrep - 1):
        sy = systems[r]
        one = System(lib_params(precision=precision), [sy["n"]], [sy["L"]])
        one.set_state(sy["x"], sy["v"], sy["type"])
        one.step(30, T0=[temps[r]])
        sl = slice(sum(sizes[:r]), sum(sizes[:r + 1]))
        for a, b in zip((gx, gv, gimg), one.get_state()):
            assert np.array_equal(a[sl], b.cpu().numpy()), r
        assert one.observables()[0] == ob[r]
        one.close()
