"""Autotuner for choices that need a fresh context: kernel path, list skin, staged
tile length (cells per row tile).  Each candidate runs a short trial from the
caller's state in its own context (the caller's context is never touched).  The
fastest candidate wins.

Paths: gather and staged by default; pass MD_PATH_AUTO among the paths to try
what a context with default settings runs, tiles of cells in most
Lennard-Jones boxes and the fastest there.  On the gather and staged paths
md_autotune picks the force-kernel variant (lanes per particle, unroll) inside
the trial, and the choice names it; a variant named on MD_PATH_AUTO would be a
gather one, so that candidate runs, and is returned, with tpp = unroll = 0.

The skin only trades list length against rebuild frequency: the forces are
those of every pair within the cutoff whatever the skin, so tuning it changes
speed, not results.

Results are cached in a JSON file keyed by device name, particle-count
bucket, replica-count bucket, density, precision, potential and largest cutoff,
and by the paths and tile lengths that were tried; the skin is part of the
result.
"""
from __future__ import annotations

import json
import math
import os
import time

from . import md

DEFAULT_CACHE = os.path.join(os.environ.get("XDG_CACHE_HOME", os.path.expanduser("~/.cache")),
                             "paper_1105_5613_amd", "tune.json")


_FORMAT = 2  # of the cache: what a key tells apart and what a choice means


def _key(params: md.Params, ntot: int, nrep: int, volume: float, paths, tile_cells) -> str:
    import torch
    dev = torch.cuda.get_device_name(torch.cuda.current_device())
    rcmax = max(params.rc[a * md.MAXT + b] for a in range(params.ntypes)
                for b in range(params.ntypes))
    nb = 2 ** int(round(math.log2(max(ntot, 1))))
    rb = 2 ** int(round(math.log2(max(nrep, 1))))
    tried = ",".join(str(int(t)) for t in sorted(set(paths)))
    if md.MD_PATH_STAGED in paths:
        tried += "/" + ",".join(str(int(t)) for t in sorted(set(tile_cells)))
    return (f"v{_FORMAT}|{dev}|n{nb}|r{rb}|rho{ntot / volume:.1f}|p{params.precision}"
            f"|pot{params.potential}|rc{rcmax:.4f}|{tried}")


def _with(params: md.Params, **kw) -> md.Params:
    p = md.Params.from_buffer_copy(params)
    for k, v in kw.items():
        setattr(p, k, v)
    return p


def _min_cells(L, params: md.Params, skin: float) -> int:
    rcmax = max(params.rc[a * md.MAXT + b] for a in range(params.ntypes)
                for b in range(params.ntypes))
    return min(int(math.floor(l / (rcmax + skin))) for l in L)


def autotune(params: md.Params, n, L, x, v, types, *, T0=None, steps: int = 60,
             warmup: int = 20, skins=None, paths=(md.MD_PATH_GATHER, md.MD_PATH_STAGED),
             tile_cells=(0,), cache_path: str | None = DEFAULT_CACHE,
             use_cache: bool = True):
    """Return (tuned Params, report).  n, L: per-replica sizes and box sides;
    x, v, types: the state to trial on (device or host arrays)."""
    import torch
    n = [int(t) for t in (n if hasattr(n, "__len__") else [n])]
    L = [float(t) for t in (L if hasattr(L, "__len__") else [L])]
    key = _key(params, sum(n), len(n), sum(l ** 3 for l in L), paths, tile_cells)
    if use_cache and cache_path and os.path.exists(cache_path):
        with open(cache_path) as f:
            cached = json.load(f).get(key)
        if cached:
            return _with(params, **cached["choice"]), {"cached": True, **cached}
    skins = [params.skin] if skins is None else list(skins)
    cands = []
    for skin in skins:
        for path in paths:
            if path == md.MD_PATH_STAGED:
                if _min_cells(L, params, skin) < 3:
                    continue
                for tc in tile_cells:
                    cands.append(dict(path=path, skin=float(skin), tile_cells=int(tc)))
            elif path == md.MD_PATH_AUTO:
                cands.append(dict(path=path, skin=float(skin), tpp=0, unroll=0))
            else:
                cands.append(dict(path=path, skin=float(skin)))
    trials = []
    for cand in cands:
        p = _with(params, **cand)
        try:
            s = md.System(p, n, L)
        except md.MDError:
            continue
        s.set_state(x, v, types)
        s.step(warmup, T0=T0)
        t = {} if cand["path"] == md.MD_PATH_AUTO else s.autotune(reps=3)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        s.step(steps, T0=T0)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        if not t:  # after the trial: profiled steps are launched one by one
            s.profile(1)
            s.step(min(steps, 5), T0=T0)
            pr = s.profile_read()
            t = {"force_ms": pr["force_ms"] / max(pr["force_launches"], 1)}
        s.close()
        choice = dict({k: t[k] for k in ("tpp", "unroll") if k in t}, **cand)
        trials.append({"choice": choice, "rate": sum(n) * steps / wall,
                       "force_ms": t["force_ms"]})
    if not trials:
        return params, {"cached": False, "trials": []}
    best = max(trials, key=lambda r: r["rate"])
    report = {"cached": False, "choice": best["choice"], "rate": best["rate"], "trials": trials}
    if cache_path:
        os.makedirs(os.path.dirname(cache_path), exist_ok=True)
        data = {}
        if os.path.exists(cache_path):
            with open(cache_path) as f:
                data = json.load(f)
        data[key] = {"choice": best["choice"], "rate": best["rate"]}
        with open(cache_path, "w") as f:
            json.dump(data, f, indent=1)
    return _with(params, **best["choice"]), report
