"""The autotuner's bookkeeping on the CPU, with contexts that only count calls:
what a candidate runs is what is returned, and what a cached choice answers."""
import json
import time

import pytest

import initconf
from paper_1105_5613_amd import make_params, md, tune


@pytest.fixture
def contexts(monkeypatch):
    import torch
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda *a: "card")
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    made = []

    class Context:
        # seconds per step: gather slower than AUTO, staged slowest
        cost = {md.MD_PATH_AUTO: 1e-4, md.MD_PATH_GATHER: 3e-4, md.MD_PATH_STAGED: 6e-4}

        def __init__(self, params, n, L):
            self.params, self.calls = params, []
            made.append(self)

        def set_state(self, x, v, types):
            pass

        def step(self, nsteps, T0=None):
            self.calls.append("step")
            time.sleep(nsteps * self.cost[self.params.path])

        def autotune(self, reps=5):
            self.calls.append("autotune")
            return {"tpp": 8, "unroll": 1, "force_ms": 1.0, "tried": []}

        def profile(self, every):
            self.calls.append("profile")

        def profile_read(self):
            return {"force_launches": 5, "force_ms": 2.5}

        def close(self):
            pass
    monkeypatch.setattr(md, "System", Context)
    return made


def params(**kw):
    eps, sig, rc, mass = initconf.mixture_tables()
    return make_params(eps, sig, rc, mass, skin=0.3, dt=0.005, **kw)


ALL = (md.MD_PATH_AUTO, md.MD_PATH_GATHER, md.MD_PATH_STAGED)


def run(p, cache, n=4000, rho=1.2, **kw):
    L = (n / rho) ** (1.0 / 3.0)
    return tune.autotune(p, n, L, None, None, None, steps=10, warmup=2, cache_path=cache, **kw)


def test_auto_is_timed_as_it_is_returned(contexts, tmp_path):
    p, rep = run(params(), str(tmp_path / "c.json"), paths=ALL)
    assert (p.path, p.tpp, p.unroll) == (md.MD_PATH_AUTO, 0, 0)
    auto = [c for c in contexts if c.params.path == md.MD_PATH_AUTO]
    assert len(auto) == 1 and "autotune" not in auto[0].calls
    assert auto[0].calls.index("profile") > 1  # not while it is timed
    for c in contexts:
        assert ("autotune" in c.calls) == (c.params.path != md.MD_PATH_AUTO)
    by = {t["choice"]["path"]: t for t in rep["trials"]}
    assert by[md.MD_PATH_AUTO]["force_ms"] == pytest.approx(0.5)
    assert by[md.MD_PATH_GATHER]["choice"]["tpp"] == 8


def test_cached_choice_answers_its_own_question(contexts, tmp_path):
    cache = str(tmp_path / "c.json")
    p, rep = run(params(), cache)
    assert p.path == md.MD_PATH_GATHER and not rep["cached"]
    assert run(params(), cache)[1]["cached"]
    # the same skin is not asked for: the tuned one is part of the result
    assert run(params(), cache, skins=(0.3, 0.4))[1]["cached"]
    # other candidates, potential, precision, density, cells per row tile
    p, rep = run(params(), cache, paths=ALL)
    assert p.path == md.MD_PATH_AUTO and not rep["cached"]
    assert run(params(), cache, paths=ALL[::-1])[1]["cached"]
    assert not run(params(potential=1), cache)[1]["cached"]
    assert not run(params(precision=1), cache)[1]["cached"]
    assert not run(params(), cache, rho=0.6)[1]["cached"]
    assert not run(params(), cache, tile_cells=(2, 4))[1]["cached"]


def test_older_cache_entries_are_left_alone(contexts, tmp_path):
    cache = tmp_path / "c.json"
    old = {"card|n4096|r1|p0|rc2.5000": {"choice": {"path": 1, "skin": 0.3, "tpp": 1, "unroll": 4},
                                        "rate": 1.0}}
    cache.write_text(json.dumps(old))
    p, rep = run(params(), str(cache), paths=ALL)
    assert not rep["cached"] and p.path == md.MD_PATH_AUTO
    kept = json.loads(cache.read_text())
    assert set(old) < set(kept) and len(kept) == 2
