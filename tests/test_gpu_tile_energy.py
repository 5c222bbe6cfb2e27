"""Energies of the launches on tiles of cells, which form them from what the pair
force has formed: both potentials and truncations, one to four species, two and
four lanes per particle, lists and the list-free search, against the oracle.

Bounds: the sum of the magnitudes of the terms of V* = 4 e ((s/r)^12 - (s/r)^6)
- V(rc) - (r - rc) V'(rc) times 12 roundings of a pair's arithmetic (FP32 2^-24
in the mixed form; in FP64 the summation, 1e-12), and the same for W = r f(r)."""
import numpy as np
import pytest

import initconf
import oracle
from gpu_common import oracle_cells_lists
from test_gpu_brick import TABLES, make, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def magnitudes(table, soft, shift_only, types, x, L, count, ids):
    eps, sig, rc = (np.asarray(a, dtype=np.float64) for a in table[:3])
    n, cap = ids.shape
    i, j = np.repeat(np.arange(n), cap), ids.reshape(-1)
    m = (np.arange(cap)[None, :] < count[:, None]).reshape(-1)
    i, j = i[m], j[m]
    d = x[i] - x[j]
    d -= L * np.rint(d / L)
    r = np.linalg.norm(d, axis=1)
    a, b = types[i], types[j]
    e, s, c = eps[a, b], sig[a, b], rc[a, b]
    q = 0.0 if soft else 1.0

    def terms(y):
        s6 = (s / y) ** 6
        return 4.0 * e * s6 * s6, 4.0 * e * s6 * q
    p12, p6 = terms(r)
    c12, c6 = terms(c)
    fs = 0.0 if shift_only else np.abs((12.0 * c12 - 6.0 * c6) / c)
    on = r < c
    v = p12 + p6 + np.abs(c12 - c6) + np.abs(r - c) * fs
    w = 12.0 * p12 + 6.0 * p6 + r * fs
    return 0.5 * float(v[on].sum()), 0.5 * float(w[on].sum())


@pytest.mark.parametrize("n,table", [(5000, "mixture"), (4321, "one"), (4321, "three"),
                                     (4321, "uneven"), (70000, "mixture"), (70000, "wide")])
@pytest.mark.parametrize("potential,trunc", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("path", [0, 3])
def test_energy_and_virial(torch_cuda, n, table, potential, trunc, precision, path):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case energy n={n} {table} pot={potential} trunc={trunc} prec={precision} path={path}",
          flush=True)
    eps, sig, rc, mass = TABLES[table]
    s = initconf.fcc_system(n, seed=n % 83, temperature=1.0, jitter=0.12)
    nt = len(eps)
    types = s["type"] if nt == 2 else \
        np.random.default_rng(n).integers(0, nt, n).astype(np.int32)
    sysm = System(make(TABLES[table], precision, potential=potential, trunc=trunc, path=path),
                  [n], [s["L"]])
    sysm.set_state(s["x"], s["v"], types)
    sysm.forces()
    ob = sysm.observables()[0]
    if path == 0:
        assert len(sysm.autotune(reps=1)["tried"]) == 2  # on the tiles
        assert sysm.observables()[0]["pe"] == ob["pe"]   # whatever the lanes
    sysm.close()
    p = oracle.make_params(eps, sig, rc, mass, skin=0.3, potential=potential, trunc=trunc)
    xw, cs, order, count, ids, nc = oracle_cells_lists(p, s["x"], types, s["L"])
    _, pe, w = oracle.forces_list(p, xw, types, s["L"], count, ids)
    av, aw = magnitudes(TABLES[table], potential == 1, trunc == 1, types, xw, s["L"], count, ids)
    rel = 1e-12 if precision == 0 else 12 * 2.0 ** -24
    assert abs(ob["pe"] - pe) <= rel * av, (ob["pe"], pe, av)
    assert abs(ob["virial"] - w) <= rel * aw, (ob["virial"], w, aw)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("log_every", [1, 2, 5])
def test_logged_steps_fused_split_and_interrupted(torch_cuda, precision, log_every):  # noqa: F811
    """Steps that form energies between steps that do not: the same state and
    log with the kick fused or not, in graphs, and where a list outgrows its
    capacity during the run (the interrupted step is finished as it was queued)."""
    from paper_1105_5613_amd import System
    print(f"case logged steps precision={precision} log_every={log_every}", flush=True)
    # a warming crystal at half the usual density of lists: rows grow in the run
    s = initconf.fcc_system(6000, rho=1.0, seed=5, temperature=6.0, jitter=0.01)
    outs, caps = [], []
    for kw in ({"max_neighbors": 200}, {"max_neighbors": 200, "split_kick": 1},
               {"max_neighbors": 200, "graph_steps": 10}, {"max_neighbors": 93}):
        sysm = System(make(TABLES["mixture"], precision, dt=0.005, **kw), [s["n"]], [s["L"]])
        sysm.set_state(s["x"], s["v"], s["type"])
        sysm.forces()
        caps.append([sysm.replica_info(0)["max_neighbors"]])
        log = sysm.step(40, log_every=log_every)
        caps[-1].append(sysm.replica_info(0)["max_neighbors"])
        if kw.get("max_neighbors") == 93 or "graph_steps" in kw:
            log.pop("n_rebuild")
        outs.append(([a.cpu().numpy() for a in sysm.get_state()] +
                     [sysm.get_forces().cpu().numpy()], log))
        sysm.close()
    assert caps[3][1] > caps[3][0] and caps[0][0] == caps[0][1]
    for state, log in outs[1:]:
        for a, b in zip(state, outs[0][0]):
            assert np.array_equal(a, b)
        for k in log:
            assert np.array_equal(log[k], outs[0][1][k]), k
