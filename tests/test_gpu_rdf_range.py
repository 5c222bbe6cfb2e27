"""g(r) over ranges of several cells: pair counts equal the oracle's bit for
bit where md_rdf changes its search -- one, two and three cells to each side,
the largest number of cells a box of 5, 6, 7 or 8 cells per side allows, the
fall back to all pairs beyond it, boxes cut into parts of cells and not, one
and 8,192 bins, and states stepped since the last list build."""
import numpy as np
import pytest

import initconf
import oracle
from gpu_common import lib_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return torch


def counts(g, n, L, rmax, nbins):
    dr = rmax / nbins
    r0 = np.arange(nbins) * dr
    shell = 4.0 / 3.0 * np.pi * ((r0 + dr) ** 3 - r0 ** 3)
    return np.round(g * n * n * shell / (2.0 * L ** 3)).astype(np.int64)


@pytest.mark.parametrize("n,steps", [(3375, 0), (4000, 25), (6500, 12), (10500, 25),
                                     (16000, 7)])
def test_rdf_range_matches_oracle(torch_cuda, n, steps):
    from paper_1105_5613_amd import System
    s = initconf.fcc_system(n, seed=n % 89, temperature=2.0)
    sysm = System(lib_params(), [n], [s["L"]])
    sysm.set_state(s["x"], s["v"], s["type"])
    if steps:
        sysm.step(steps)
    else:
        sysm.build_cells()
    nc = sysm.replica_info(0)["nc"]
    side = s["L"] / nc
    x = sysm.get_state()[0].cpu().numpy()
    for h in range(1, (nc - 1) // 2 + 2):
        edge = h * side - 0.3
        for rmax, nbins in ((edge * (1.0 - 1e-11), 400), (min(edge + 0.05, 0.5 * s["L"]), 8192),
                            (edge * 0.93, 1)):
            if rmax > 0.5 * s["L"]:
                continue
            print(f"case rdf n={n} nc={nc} h={h} rmax={rmax:.6f} nbins={nbins}", flush=True)
            g = sysm.rdf(0, rmax, nbins)
            go = oracle.rdf(x, s["L"], rmax, nbins)
            assert np.array_equal(counts(g, n, s["L"], rmax, nbins),
                                  counts(go, n, s["L"], rmax, nbins))
    sysm.close()


def test_rdf_bin_edges(torch_cuda):
    """Distances on bin edges, at zero and at rmax: a perfect lattice puts
    whole shells on edges of bins that divide its spacing."""
    from paper_1105_5613_amd import System
    m = 16
    L = 16.0
    ax = np.arange(m, dtype=np.float64)
    x = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    x[1] = x[0]  # two particles at one place: r = 0
    n = len(x)
    sysm = System(lib_params(), [n], [L])
    sysm.set_state(x, np.zeros_like(x), np.zeros(n, np.int32))
    sysm.build_cells()
    for rmax, nbins in ((2.0, 8), (4.0, 4), (4.0, 400), (5.0, 5), (3.0, 7)):
        print(f"case rdf lattice rmax={rmax} nbins={nbins}", flush=True)
        g = sysm.rdf(0, rmax, nbins)
        go = oracle.rdf(x, L, rmax, nbins)
        assert np.array_equal(counts(g, n, L, rmax, nbins), counts(go, n, L, rmax, nbins))
    sysm.close()
