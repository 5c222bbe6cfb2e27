"""The list-free search where several waves share a crowded cell's particles:
forces, energy and virial against the oracle, the same bits alone and beside
replicas whose tiles hold more waves, and fused, split and in graphs."""
import numpy as np
import pytest

import initconf
import oracle
from gpu_common import floored_err, lib_params, oracle_cells_lists, pair_abs_sums
from test_gpu_brick import TABLES, make, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


# particles per cell: 33 to 64 (two groups of homes), 65 (three); tiles of four,
# two and one cell; a box whose last tiles are smaller
@pytest.mark.parametrize("n,rho,table", [
    (4200, 1.2, "mixture"), (11500, 1.5, "mixture"), (7000, 1.9, "one"), (9000, 2.1, "three"),
    (16000, 2.4, "mixture"), (4000, 2.6, "uneven"), (12500, 2.95, "mixture")])
@pytest.mark.parametrize("precision", [0, 1])
def test_crowded_cells(torch_cuda, n, rho, table, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case crowded n={n} rho={rho} {table} precision={precision}", flush=True)
    eps, sig, rc, mass = TABLES[table]
    s = initconf.fcc_system(n, rho=rho, seed=n % 83, temperature=1.0, jitter=0.12 / rho)
    nt = len(eps)
    types = s["type"] if nt == 2 else \
        np.random.default_rng(n).integers(0, nt, n).astype(np.int32)
    sysm = System(make(TABLES[table], precision, path=3), [n], [s["L"]])
    sysm.set_state(s["x"], s["v"], types)
    sysm.forces()
    F, ob = sysm.get_forces().cpu().numpy(), sysm.observables()[0]
    sysm.close()
    p = oracle.make_params(eps, sig, rc, mass, skin=0.3)
    xw, cs, order, count, ids, nc = oracle_cells_lists(p, s["x"], types, s["L"])
    print(f"  {n / nc ** 3:.1f} per cell", flush=True)
    Fo, peo, wo = oracle.forces_list(p, xw, types, s["L"], count, ids)
    assert floored_err(F, Fo) <= (1e-12 if precision == 0 else 1e-5)
    cpe, cw = pair_abs_sums(eps, sig, rc, types, xw, s["L"], count, ids)
    rel = 1e-12 if precision == 0 else 1e-6
    assert abs(ob["pe"] - peo) <= 2 * rel * cpe and abs(ob["virial"] - wo) <= 2 * rel * cw


@pytest.mark.parametrize("precision", [0, 1])
def test_alone_and_in_a_batch(torch_cuda, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case crowded batch precision={precision}", flush=True)
    sizes, rhos = [4000, 20000, 9000, 3000], [2.4, 1.2, 1.7, 0.4]
    reps = [initconf.fcc_system(n, rho=r, seed=41, temperature=1.0, jitter=0.05)
            for n, r in zip(sizes, rhos)]

    def run(which, **kw):
        sysm = System(lib_params(precision=precision, path=3, dt=0.001, **kw),
                      [sizes[r] for r in which], [reps[r]["L"] for r in which])
        sysm.set_state(*(np.concatenate([reps[r][k] for r in which]) for k in ("x", "v", "type")))
        log = sysm.step(12, log_every=3)
        out = [a.cpu().numpy() for a in sysm.get_state()] + [sysm.get_forces().cpu().numpy()]
        sysm.close()
        return out, log
    big, blog = run([0, 1, 2, 3])
    for r in range(4):
        sl = slice(sum(sizes[:r]), sum(sizes[:r + 1]))
        for kw in ({}, {"split_kick": 1}, {"graph_steps": 3}):
            one, log = run([r], **kw)
            for a, b in zip(big, one):
                assert np.array_equal(a[sl], b), (r, kw)
            for k in log:
                assert np.array_equal(blog[k][:, r], log[k][:, 0]), (r, kw, k)
