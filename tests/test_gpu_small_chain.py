"""The one-launch rebuild chain of a one-replica context against the general
launches, bit for bit, where its split changes: one cell and one block, the
sizes where a thread takes another block of particles, a last block that is
nearly empty, list-free steps (the chain's records are committed by another
kernel) and particles that cross the box faces between builds."""
import numpy as np
import pytest

import initconf
from gpu_common import lib_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,path,precision", [
    (220, 0, 0), (257, 1, 0), (500, 0, 1), (4096, 0, 0), (4097, 1, 1), (4097, 3, 0),
    (8193, 0, 1), (10976, 3, 1), (12289, 1, 0), (16384, 0, 0), (16384, 2, 1),
])
def test_chain_in_one_launch_matches_general(n, path, precision):
    from paper_1105_5613_amd import System
    print(f"case chain n={n} path={path} precision={precision}", flush=True)
    s = initconf.fcc_system(n, seed=n % 97, temperature=2.0)
    out = []
    for small_box in (0, 1):
        sysm = System(lib_params(precision=precision, path=path, small_box=small_box), [n],
                      [s["L"]])
        sysm.set_state(s["x"] + 0.49 * s["L"], s["v"], s["type"])
        log = sysm.step(40, T0=[2.0], log_every=5)
        x, v, img = (a.cpu().numpy() for a in sysm.get_state())
        sysm.build_cells()
        cs, order = sysm.get_cells(0)
        out.append([x, v, img, cs, order] + [log[k] for k in sorted(log)])
        rebuilds = sysm.observables()[0]["n_rebuild"]
        sysm.close()
    assert rebuilds >= 4
    for a, b in zip(*out):
        assert np.array_equal(a, b)
