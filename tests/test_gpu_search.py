"""The list-free path on tiles of cells, which path = 3 takes unless a row tile
is asked for (tile_cells): forces, energy and virial against the oracle where
the search changes form -- cells of 2 to 65 particles (bricks of one and of
several cells, one and several groups of homes and passes over the candidates),
one to four species, the two-species constants and the table -- and against the
row-tile kernel: fused steps, a box that condenses beyond the LDS slots, and the
refusal of two particles at one position."""
import numpy as np
import pytest

import initconf
import oracle
from gpu_common import floored_err, lib_params, oracle_cells_lists, pair_abs_sums
from test_gpu_brick import TABLES, converging_box, make, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rho,table,precision,trunc", [
    (1000, 1.2, "mixture", 0, 0), (1000, 1.2, "mixture", 1, 0), (1100, 1.2, "three", 0, 0),
    (1729, 1.2, "mixture", 0, 0), (2100, 1.2, "one", 0, 0), (2100, 1.2, "one", 1, 0),
    (4321, 1.2, "uneven", 0, 0), (4321, 1.2, "uneven", 1, 0), (5000, 1.2, "four", 0, 0),
    (5000, 1.2, "four", 1, 0), (6900, 1.2, "wide", 0, 0), (9000, 1.2, "mixture", 1, 1),
    (20000, 1.2, "mixture", 0, 1), (9000, 0.1, "mixture", 0, 0), (9000, 0.1, "four", 1, 0),
    (9000, 0.4, "three", 0, 0), (9000, 0.75, "mixture", 1, 0), (9000, 1.6, "mixture", 0, 0),
    (9000, 1.6, "four", 0, 0), (9000, 2.6, "mixture", 1, 0), (12000, 2.6, "mixture", 0, 0),
    (12000, 4.0, "mixture", 0, 0),  # too dense for the tiles: row tiles
])
def test_search_matches_oracle(torch_cuda, n, rho, table, precision, trunc):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case search n={n} rho={rho} table={table} precision={precision}", flush=True)
    eps, sig, rc, mass = TABLES[table]
    s = initconf.fcc_system(n, rho=rho, seed=n % 83, temperature=1.0, jitter=0.12 * min(1.0, 1 / rho))
    nt = len(eps)
    types = s["type"] if nt == 2 else \
        np.random.default_rng(n).integers(0, nt, n).astype(np.int32)
    sysm = System(make(TABLES[table], precision, trunc=trunc, path=3), [n], [s["L"]])
    sysm.set_state(s["x"], s["v"], types)
    sysm.forces()
    F = sysm.get_forces().cpu().numpy()
    ob = sysm.observables()[0]
    sysm.close()
    p = oracle.make_params(eps, sig, rc, mass, skin=0.3, trunc=trunc)
    xw, cs, order, count, ids, nc = oracle_cells_lists(p, s["x"], types, s["L"])
    Fo, peo, wo = oracle.forces_list(p, xw, types, s["L"], count, ids)
    e = floored_err(F, Fo)
    assert e <= (1e-12 if precision == 0 else 1e-5), e
    cpe, cw = pair_abs_sums(eps, sig, rc, types, xw, s["L"], count, ids)
    rel = 1e-12 if precision == 0 else 1e-6
    assert abs(ob["pe"] - peo) <= 2 * rel * cpe and abs(ob["virial"] - wo) <= 2 * rel * cw


@pytest.mark.parametrize("precision", [0, 1])
def test_search_alone_and_in_a_batch(torch_cuda, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case search batch precision={precision}", flush=True)
    sizes, temps = [1000, 40000, 4000], [0.7, 1.5, 2.0]
    systems = initconf.batched_systems(sizes, temps, seed=62)
    x, v, t, n, L = initconf.concat_replicas(systems)
    big = System(lib_params(precision=precision, path=3), n, L)
    big.set_state(x, v, t)
    log = big.step(18, T0=temps, log_every=3)
    gx, gv, gimg = (a.cpu().numpy() for a in big.get_state())
    big.close()
    for r, sy in enumerate(systems):
        one = System(lib_params(precision=precision, path=3), [sy["n"]], [sy["L"]])
        one.set_state(sy["x"], sy["v"], sy["type"])
        lo = one.step(18, T0=[temps[r]], log_every=3)
        ox, ov, oimg = (a.cpu().numpy() for a in one.get_state())
        one.close()
        sl = slice(sum(sizes[:r]), sum(sizes[:r + 1]))
        assert np.array_equal(gx[sl], ox) and np.array_equal(gv[sl], ov), r
        assert np.array_equal(gimg[sl], oimg), r
        for k in lo:
            assert np.array_equal(log[k][:, r], lo[k][:, 0]), (r, k)


@pytest.mark.parametrize("precision", [0, 1])
def test_search_fused_split_and_graph_steps(torch_cuda, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case search fused vs split vs graphs precision={precision}", flush=True)
    s = initconf.fcc_system(30000, seed=9, temperature=2.0)
    outs = []
    for kw in ({}, {"split_kick": 1}, {"graph_steps": 4}):
        sysm = System(lib_params(precision=precision, path=3, **kw), [s["n"]], [s["L"]])
        sysm.set_state(s["x"], s["v"], s["type"])
        log = sysm.step(14, log_every=4)
        outs.append([a.cpu().numpy() for a in sysm.get_state()] +
                    [sysm.get_forces().cpu().numpy()] + [log[k] for k in sorted(log)])
        sysm.close()
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", [0, 1])
def test_condensing_box_goes_on_with_row_tiles(torch_cuda, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case search condensing box precision={precision}", flush=True)
    s, v = converging_box()
    out = []
    for tc in (0, 4):
        sysm = System(lib_params(precision=precision, path=3, tile_cells=tc, dt=0.002), [s["n"]],
                      [s["L"]])
        sysm.set_state(s["x"], v, s["type"])
        log = sysm.step(240, log_every=8)
        x, vv, img = (a.cpu().numpy() for a in sysm.get_state())
        out.append((x + img * s["L"], vv, sysm.observables()[0]["n_rebuild"], log["step"]))
        sysm.close()
    # as between the brick and the gather lists of the same box
    tx, tv = (1e-9, 1e-7) if precision == 0 else (2e-3, 2e-1)
    assert np.max(np.abs(out[0][0] - out[1][0])) < tx
    assert np.max(np.abs(out[0][1] - out[1][1])) < tv
    assert out[0][2] == out[1][2] and np.array_equal(out[0][3], out[1][3])


@pytest.mark.parametrize("precision", [0, 1])
def test_two_particles_at_one_position_are_refused(torch_cuda, precision):  # noqa: F811
    from paper_1105_5613_amd import MDError, System
    print(f"case search r = 0 precision={precision}", flush=True)
    s = initconf.fcc_system(6000, seed=12)
    x = s["x"].copy()
    x[10] = x[4000]
    codes = []
    for tc in (0, 4):
        sysm = System(lib_params(precision=precision, path=3, tile_cells=tc), [s["n"]], [s["L"]])
        sysm.set_state(x, s["v"], s["type"])
        with pytest.raises(MDError) as ex:
            sysm.forces()
            sysm.observables()  # waits for the launch and reads its error state
        codes.append(ex.value.code)
        sysm.close()
    assert codes[0] == codes[1]
