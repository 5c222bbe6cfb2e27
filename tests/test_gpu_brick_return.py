"""Contexts that left the tiles of cells because a box condensed: the next state
starts on the tiles again, and the other replicas of the context go on with
their own trajectories."""
import numpy as np
import pytest

import initconf
from gpu_common import lib_params
from test_gpu_brick import converging_box, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def evaluate(sysm, s, x, **step):
    """Forces of a new state and a short run from it."""
    sysm.set_state(x, s["v"], s["type"])
    sysm.forces()
    out = [sysm.get_forces().cpu().numpy()]
    log = sysm.step(9, log_every=3, **step)
    if sysm.params.max_neighbors == 64:
        log.pop("n_rebuild")
    return out + [a.cpu().numpy() for a in sysm.get_state()] + [log[k] for k in sorted(log)]


# rows of up to 150 entries: 200 do, 64 grow (the state that grows them counts
# that build, a later one does not)
@pytest.mark.parametrize("precision,kw", [
    (0, {"max_neighbors": 200}), (1, {"max_neighbors": 200}),
    (1, {"max_neighbors": 200, "graph_steps": 3}), (0, {"max_neighbors": 64}), (0, {"path": 3}),
    (1, {"path": 3, "graph_steps": 3})])
@pytest.mark.parametrize("T0", [None, 0.5])
def test_next_state_starts_on_the_tiles(torch_cuda, precision, kw, T0):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case return precision={precision} kw={kw} T0={T0}", flush=True)
    s = initconf.fcc_system(16000, rho=0.7, seed=15, temperature=0.5)
    crowded = s["x"].copy()
    crowded[:, 0] *= 0.55
    p = dict(precision=precision, dt=0.001, **kw)
    want = []
    for x in (s["x"], crowded):
        one = System(lib_params(**p), [s["n"]], [s["L"]])
        want.append(evaluate(one, s, x, T0=T0))
        if kw.get("path", 0) == 0:
            assert (len(one.autotune(reps=1)["tried"]) == 2) == (x is s["x"])
        one.close()
    sysm = System(lib_params(**p), [s["n"]], [s["L"]], allocator="torch")
    for k in (1, 0, 1, 1, 0, 0):
        got = evaluate(sysm, s, (s["x"], crowded)[k], T0=T0)
        for a, b in zip(got, want[k]):
            assert np.array_equal(a, b), k
    sysm.close()
    assert sysm.allocator.bytes_held() == 0


def test_variant_comes_back(torch_cuda):  # noqa: F811
    """The lanes per particle that md_autotune chose on the tiles."""
    from paper_1105_5613_amd import System
    print("case variant", flush=True)
    s = initconf.fcc_system(16000, rho=0.7, seed=15, temperature=0.5)
    crowded = s["x"].copy()
    crowded[:, 0] *= 0.55
    builds = []
    for path in (1, 0):
        sysm = System(lib_params(max_neighbors=200, path=path), [s["n"]], [s["L"]])
        evaluate(sysm, s, crowded)
        builds.append(sysm.observables()[0]["n_rebuild"])
        if path == 1:
            sysm.close()
    assert builds[0] == builds[1]  # the build that did not fit is not one
    assert len(sysm.autotune(reps=1)["tried"]) > 2
    want = evaluate(sysm, s, s["x"])
    assert len(sysm.autotune(reps=1)["tried"]) == 2
    got = evaluate(sysm, s, s["x"])  # results do not depend on the lanes
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
    sysm.close()


@pytest.mark.parametrize("path,graphs,thermo", [(0, 0, False), (0, 4, True), (3, 0, False),
                                                (3, 4, True)])
def test_other_replicas_of_the_context(torch_cuda, path, graphs, thermo):  # noqa: F811
    """One replica condenses; the two others, which never would, change kernels
    with it: their trajectories stay those of contexts of their own to
    round-off, with at most the one list build more."""
    from paper_1105_5613_amd import System
    print(f"case replicas path={path} graphs={graphs} thermo={thermo}", flush=True)
    s, v = converging_box()
    # (cells of 26 to 27 particles: the LDS layout that the middle box outgrows)
    sizes, calm = [3340, s["n"], 13500], [0, 2]
    reps = [initconf.fcc_system(n, rho=1.2, seed=31 + k, temperature=1.0)
            for k, n in enumerate(sizes)]
    reps[1] = dict(s, v=v)
    T = [1.0, float(np.sum(v * v)) / (3 * s["n"] - 3), 1.0]
    p = dict(path=path, graph_steps=graphs, dt=0.002)

    def run(which):
        sysm = System(lib_params(**p), [sizes[r] for r in which], [reps[r]["L"] for r in which])
        sysm.set_state(np.concatenate([reps[r]["x"] for r in which]),
                       np.concatenate([reps[r]["v"] for r in which]),
                       np.concatenate([reps[r]["type"] for r in which]))
        for _ in range(30):
            sysm.step(8, T0=[T[r] for r in which] if thermo else None)
        x, vs, img = (a.cpu().numpy() for a in sysm.get_state())
        L = np.repeat([reps[r]["L"] for r in which], [sizes[r] for r in which])
        ob = sysm.observables()
        left = len(sysm.autotune(reps=1)["tried"]) > 2
        sysm.close()
        return x + img * L[:, None], vs, ob, left
    xb, vb, ob, left = run([0, 1, 2])
    assert path == 3 or left, "never left the tiles"
    for r in calm:
        x1, v1, o1, left1 = run([r])
        assert not left1
        sl = slice(sum(sizes[:r]), sum(sizes[:r + 1]))
        # 240 steps of 0.002 at T = 1: rounding of the force sums (1e-15) grows
        # less than a thousandfold in half a time unit
        assert np.max(np.abs(xb[sl] - x1)) < 1e-10 and np.max(np.abs(vb[sl] - v1)) < 1e-9
        assert ob[r]["step"] == o1[0]["step"] == 240
        assert 0 <= ob[r]["n_rebuild"] - o1[0]["n_rebuild"] <= 1


@pytest.mark.parametrize("graphs,thermo", [(0, False), (4, False), (4, True)])
def test_list_free_box_is_on_row_tiles(torch_cuda, graphs, thermo):  # noqa: F811
    """The condensed box of the list-free path: its forces are the row-tile
    kernel's, bit for bit, while those of its first state were not."""
    from paper_1105_5613_amd import System
    print(f"case list-free switch graphs={graphs} thermo={thermo}", flush=True)
    s, v = converging_box()
    T0 = float(np.sum(v * v)) / (3 * s["n"] - 3) if thermo else None

    def rows(x):
        sysm = System(lib_params(path=3, tile_cells=4, dt=0.002), [s["n"]], [s["L"]])
        sysm.set_state(x, v, s["type"])
        sysm.forces()
        F = sysm.get_forces().cpu().numpy()
        sysm.close()
        return F

    sysm = System(lib_params(path=3, graph_steps=graphs, dt=0.002), [s["n"]], [s["L"]])
    for _ in range(2):  # the second time after a switch
        sysm.set_state(s["x"], v, s["type"])
        sysm.forces()
        assert not np.array_equal(sysm.get_forces().cpu().numpy(), rows(s["x"]))
        sysm.step(240, T0=T0)
        x = sysm.get_state()[0].cpu().numpy()
        sysm.build_cells()
        sysm.forces()
        assert np.array_equal(sysm.get_forces().cpu().numpy(), rows(x))
    sysm.close()
