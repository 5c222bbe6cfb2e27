"""The brick path, which a context with default path settings takes in boxes of
three and more cells per side: its list build and force kernel against the
oracle and the gather path where they change form -- cells of 27 to 60
particles (the tile shapes, both LDS layouts, one or two groups of homes per
brick, one or several passes over the candidates), few bricks and many, the
two-species constants and the table of up to four species, pairs at the same
position, and boxes that condense beyond the LDS slots and go on with gather
lists."""
import numpy as np
import pytest

import initconf
import oracle
from gpu_common import floored_err, lib_params, oracle_cells_lists, canonical, pair_abs_sums

pytestmark = pytest.mark.gpu

TABLES = {
    "mixture": initconf.mixture_tables(),
    "one": ([[1.0]], [[1.0]], [[2.5]], [1.0]),
    "wide": ([[1.0, 1.5], [1.5, 0.5]], [[1.0, 0.7], [0.7, 0.4]], [[2.5, 1.75], [1.75, 1.0]],
             [1.0, 0.5]),
    # no base species gives every constant of this table by one exact FMA
    "uneven": ([[1.0, 0.0031], [0.0031, 0.9]], [[1.0, 0.9], [0.9, 0.8]],
               [[2.5, 2.25], [2.25, 2.0]], [1.0, 1.0]),
    "three": ([[1.0, 1.2, 0.8], [1.2, 0.6, 1.0], [0.8, 1.0, 0.9]],
              [[1.0, 0.9, 0.8], [0.9, 0.85, 0.75], [0.8, 0.75, 0.7]],
              [[2.5, 2.25, 2.0], [2.25, 2.125, 1.875], [2.0, 1.875, 1.75]], [1.0, 0.9, 0.8]),
    "four": ([[1.0, 1.1, 0.9, 0.7], [1.1, 0.8, 1.0, 0.6], [0.9, 1.0, 0.5, 0.9],
              [0.7, 0.6, 0.9, 1.2]],
             [[1.0, 0.9, 0.8, 0.95], [0.9, 0.85, 0.75, 0.9], [0.8, 0.75, 0.7, 0.8],
              [0.95, 0.9, 0.8, 0.9]],
             [[2.5, 2.25, 2.0, 2.4], [2.25, 2.1, 1.9, 2.2], [2.0, 1.9, 1.7, 2.0],
              [2.4, 2.2, 2.0, 2.2]], [1.0, 0.9, 0.8, 1.1]),
}


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return torch


def make(tables, precision=0, **kw):
    from paper_1105_5613_amd import make_params
    eps, sig, rc, mass = tables
    return make_params(eps, sig, rc, mass, skin=kw.pop("skin", 0.3), precision=precision, **kw)


@pytest.mark.parametrize("n,table,precision,trunc", [
    (1000, "mixture", 0, 0), (1000, "mixture", 1, 0), (1100, "three", 0, 0),
    (1729, "mixture", 0, 0), (2100, "one", 0, 0), (2100, "one", 1, 0),
    (4321, "uneven", 0, 0), (4321, "uneven", 1, 0), (5000, "four", 0, 0), (5000, "four", 1, 0),
    (6900, "wide", 0, 0), (9000, "mixture", 1, 1), (13500, "three", 1, 0),
    (20000, "mixture", 0, 1), (20000, "mixture", 1, 0), (47000, "mixture", 0, 0),
    (47000, "wide", 1, 0),
])
def test_brick_matches_oracle(torch_cuda, n, table, precision, trunc):
    from paper_1105_5613_amd import System
    print(f"case brick n={n} table={table} precision={precision} trunc={trunc}", flush=True)
    eps, sig, rc, mass = TABLES[table]
    s = initconf.fcc_system(n, seed=n % 83, temperature=1.0, jitter=0.12)
    nt = len(eps)
    types = s["type"] if nt == 2 else \
        np.random.default_rng(n).integers(0, nt, n).astype(np.int32)
    sysm = System(make(TABLES[table], precision, trunc=trunc), [n], [s["L"]])
    sysm.set_state(s["x"], s["v"], types)
    sysm.forces()
    p = oracle.make_params(eps, sig, rc, mass, skin=0.3, trunc=trunc)
    xw, cs, order, count, ids, nc = oracle_cells_lists(p, s["x"], types, s["L"])
    assert sysm.replica_info(0)["nc"] == nc >= 3
    gcount, gids = sysm.get_neighbors(0, cap=ids.shape[1])
    assert np.array_equal(gcount, count)
    assert np.array_equal(canonical(gcount, gids), canonical(count, ids))
    F = sysm.get_forces().cpu().numpy()
    Fo, peo, wo = oracle.forces_list(p, xw, types, s["L"], count, ids)
    e = floored_err(F, Fo)
    assert e <= (1e-12 if precision == 0 else 1e-5), e
    cpe, cw = pair_abs_sums(eps, sig, rc, types, xw, s["L"], count, ids)
    ob = sysm.observables()[0]
    rel = 1e-12 if precision == 0 else 1e-6
    # the sums of magnitudes are those of the shifted force; the plain shift's
    # pair terms are of the same size
    assert abs(ob["pe"] - peo) <= 2 * rel * cpe and abs(ob["virial"] - wo) <= 2 * rel * cw
    assert len(sysm.autotune(reps=1)["tried"]) == 2  # the brick path's variants
    sysm.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_small_replica_alone_and_in_a_large_batch(torch_cuda, precision):
    """Alone: four lanes per particle, the cooperative list build, several
    blocks per tile; beside 210,000 particles: two lanes, one wave per brick,
    one block per tile.  The same bits, energies included."""
    from paper_1105_5613_amd import System
    print(f"case small replica in a batch precision={precision}", flush=True)
    sizes, temps = [1000, 210000, 4000, 13500], [0.7, 1.5, 2.0, 1.0]
    systems = initconf.batched_systems(sizes, temps, seed=61)
    x, v, t, n, L = initconf.concat_replicas(systems)
    big = System(lib_params(precision=precision), n, L)
    big.set_state(x, v, t)
    log = big.step(18, T0=temps, log_every=3)
    gx, gv, gimg = (a.cpu().numpy() for a in big.get_state())
    F = big.get_forces().cpu().numpy()
    big.close()
    for r in (0, 2, 3):
        sy = systems[r]
        one = System(lib_params(precision=precision), [sy["n"]], [sy["L"]])
        one.set_state(sy["x"], sy["v"], sy["type"])
        lo = one.step(18, T0=[temps[r]], log_every=3)
        ox, ov, oimg = (a.cpu().numpy() for a in one.get_state())
        sl = slice(sum(sizes[:r]), sum(sizes[:r + 1]))
        assert np.array_equal(gx[sl], ox) and np.array_equal(gv[sl], ov), r
        assert np.array_equal(gimg[sl], oimg), r
        assert np.array_equal(F[sl], one.get_forces().cpu().numpy()), r
        for k in lo:
            assert np.array_equal(log[k][:, r], lo[k][:, 0]), (r, k)
        one.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_fused_and_split_steps(torch_cuda, precision):
    from paper_1105_5613_amd import System
    print(f"case brick fused vs split precision={precision}", flush=True)
    s = initconf.fcc_system(215000, seed=9, temperature=2.0)
    outs = []
    for split in (0, 1):
        sysm = System(lib_params(precision=precision, split_kick=split), [s["n"]], [s["L"]])
        sysm.set_state(s["x"], s["v"], s["type"])
        log = sysm.step(14, log_every=4)
        outs.append([a.cpu().numpy() for a in sysm.get_state()] +
                    [sysm.get_forces().cpu().numpy()] + [log[k] for k in sorted(log)])
        sysm.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", [0, 1])
def test_pairs_at_one_position_are_skipped(torch_cuda, precision):
    from paper_1105_5613_amd import System
    print(f"case r = 0 precision={precision}", flush=True)
    s = initconf.fcc_system(6000, seed=12)
    x = s["x"].copy()
    for a, b in ((10, 4000), (11, 12), (700, 5999)):
        x[a] = x[b]
    out = []
    for path in (0, 1):
        sysm = System(lib_params(precision=precision, path=path), [s["n"]], [s["L"]])
        sysm.set_state(x, s["v"], s["type"])
        sysm.forces()
        out.append((sysm.get_forces().cpu().numpy().astype(np.float64), sysm.observables()[0]))
        sysm.close()
    assert np.isfinite(out[0][0]).all()
    assert floored_err(out[0][0], out[1][0]) <= (2e-12 if precision == 0 else 2e-5)
    rel = 1e-12 if precision == 0 else 2e-6
    assert out[0][1]["pe"] == pytest.approx(out[1][1]["pe"], rel=rel)


def converging_box():
    """A box at 0.8 whose velocity field piles the particles up around a plane."""
    n = 30000
    s = initconf.fcc_system(n, rho=0.8, seed=14, temperature=0.5)
    v = s["v"].copy()
    v[:, 0] += 9.0 * np.sin(2.0 * np.pi * s["x"][:, 0] / s["L"])
    return s, v


@pytest.mark.parametrize("precision", [0, 1])
def test_condensing_box_goes_on_with_gather_lists(torch_cuda, precision):
    from paper_1105_5613_amd import System
    print(f"case condensing box precision={precision}", flush=True)
    s, v = converging_box()
    steps, logs, out = 80, [], []
    for path in (0, 1):
        sysm = System(lib_params(precision=precision, path=path, dt=0.002), [s["n"]], [s["L"]])
        sysm.set_state(s["x"], v, s["type"])
        if path == 0:
            assert len(sysm.autotune(reps=1)["tried"]) == 2  # starts on the brick path
        logs.append([sysm.step(steps, log_every=8) for _ in range(3)])
        x, vv, img = (a.cpu().numpy() for a in sysm.get_state())
        out.append((x + img * s["L"], vv, sysm.observables()[0]["n_rebuild"]))
        if path == 0:
            assert len(sysm.autotune(reps=1)["tried"]) > 2, "never left the brick path"
        sysm.close()
    # round-off (mixed: FP32 force error) over 240 steps; the piled-up region
    # is hot, with differences growing several hundredfold
    tx, tv = (1e-9, 1e-7) if precision == 0 else (2e-3, 2e-1)
    assert np.max(np.abs(out[0][0] - out[1][0])) < tx
    assert np.max(np.abs(out[0][1] - out[1][1])) < tv
    assert out[0][2] == out[1][2]
    assert np.array_equal(np.concatenate([a["step"] for a in logs[0]]),
                          np.concatenate([a["step"] for a in logs[1]]))


@pytest.mark.parametrize("precision", [0, 1])
def test_crowded_first_build(torch_cuda, precision):
    """Mean density within the path's range, one half of the box twice as dense."""
    from paper_1105_5613_amd import System
    print(f"case crowded first build precision={precision}", flush=True)
    n = 16000
    s = initconf.fcc_system(n, rho=0.7, seed=15, temperature=0.5)
    x = s["x"].copy()
    x[:, 0] *= 0.55
    F, cnt = [], []
    for path in (0, 1):
        sysm = System(lib_params(precision=precision, path=path), [n], [s["L"]])
        sysm.set_state(x, s["v"], s["type"])
        sysm.forces()
        F.append(sysm.get_forces().cpu().numpy().astype(np.float64))
        cnt.append(sysm.get_neighbors(0, cap=4))
        sysm.close()
    assert np.array_equal(cnt[0][0], cnt[1][0])
    assert np.array_equal(F[0], F[1])  # the same kernels after the switch
