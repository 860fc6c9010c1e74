"""Autotuner of the library's tuning knobs (chunk size and cutoff-slot groups
of the per-centre work items of the forward, cell-list bin size,
persistent grid size, work items per centre of the adjoint).

Candidates are timed with the HIP events the library records around its
own launches on the current stream (neighbour build + forward, optionally
the adjoint) in two interleaved rounds, the faster round counting; a
candidate displaces the best so far only when it is more than 1% faster
(the first candidate is the default: differences within run-to-run noise
keep it), the choice is set on the plan and cached in
a JSON file keyed by the device, the precision, the probe shape (l_max,
sigmas, species, largest primitive count per element) and log2 buckets of
the atom count and of the mean list length.
GMP_AUTOTUNE=0 disables the search (cached or default values are used);
GMP_TUNE_CACHE sets the cache path.
"""
from __future__ import annotations

import json
import math
import os
import time
from typing import Dict, Iterable, Optional

import torch

from . import gmp as _g

DEFAULT_CANDIDATES = [
    dict(chunk_pairs=c, bin_divisor=b, blocks_per_cu=0, adj_items=0)
    for c in (0, 512, 1024, 2048, 4096) for b in (2, 3, 4)
] + [dict(chunk_pairs=2048, bin_divisor=2, blocks_per_cu=k, adj_items=0) for k in (1, 2)]

# a whole forward + backward step: the forward's chunking and slot groups
# and the cell-list bins crossed with the adjoint's items per centre
STEP_CANDIDATES = [
    dict(chunk_pairs=c, bin_divisor=b, blocks_per_cu=0, adj_items=a, sigma_groups=1)
    for c in (2048, 0) for b in (2, 3) for a in (0, 2)
] + [dict(chunk_pairs=c, bin_divisor=b, blocks_per_cu=0, adj_items=0, sigma_groups=2) for c, b in ((2048, 2), (0, 3))]

_DEFAULT = dict(chunk_pairs=2048, bin_divisor=2, blocks_per_cu=0, adj_items=0, sigma_groups=1)
_MARGIN = 0.01  # a later candidate must be this much faster than the best so far
_ROUNDS = 2     # timing rounds per candidate


def _full(cand: Dict) -> Dict:
    """A candidate with every knob set (unnamed knobs at their defaults)."""
    return dict(_DEFAULT, **cand)


def _cache_path():
    return os.environ.get("GMP_TUNE_CACHE", os.path.join(os.path.expanduser("~"), ".cache", "gmp_tune.json"))


def _bucket(x: float) -> int:
    return int(math.floor(math.log2(max(1.0, x))))


def tuning_key(plan, batch, nb, backward: bool = True) -> str:
    """Device, precision, l_max, sigma count, species count, largest
    primitive count per element, log2 buckets of the atom count and of the
    mean neighbour-list length, and whether the adjoint is part of the
    timed step."""
    dev = torch.cuda.get_device_name(batch.species.device)
    avg = nb.n_pairs / max(1, batch.n_atoms)
    kmax = int(max(int(b) - int(a) for a, b in zip(plan._poff[:-1], plan._poff[1:])))
    return (f"{dev}|{plan.precision}|L{int(max(plan.orders))}|S{plan.n_slots}|E{plan.n_elements}|K{kmax}"
            f"|N{_bucket(batch.n_atoms)}|avg{_bucket(avg)}|{'step' if backward else 'fwd'}")


def _load(path):
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def choose(tried, margin: float = None) -> int:
    """Index of the chosen candidate among [{"ms": ...}, ...] in search
    order: a candidate displaces the best so far only when it is faster by
    more than `margin` (default 1%), so the first (the default tuning) keeps
    its place against differences within run-to-run noise."""
    margin = _MARGIN if margin is None else margin
    best = None
    for i, t in enumerate(tried):
        if best is None or t["ms"] < (1.0 - margin) * tried[best]["ms"]:
            best = i
    return best


def _time_config(plan, batch, ws, G, reps: int, backward: bool) -> float:
    nb = _g.build_neighbors(plan, batch, ws)
    for _ in range(2):  # warm: grows the workspace, fills occupancy caches
        nb = _g.build_neighbors(plan, batch, ws, out=nb)
        F, mu = _g.features(plan, batch, nb, ws)
        if backward:
            _g.features_backward(plan, batch, nb, ws, mu, F, G)
    torch.cuda.synchronize()
    with _g.profile() as pr:
        for _ in range(reps):
            nb = _g.build_neighbors(plan, batch, ws, out=nb)
            F, mu = _g.features(plan, batch, nb, ws)
            if backward:
                _g.features_backward(plan, batch, nb, ws, mu, F, G)
        torch.cuda.synchronize()
    return sum(v[1] for v in pr.result.values()) / reps


def autotune(plan, batch, ws, candidates: Optional[Iterable[Dict]] = None, backward: bool = True,
             reps: int = 3, cache_path: Optional[str] = None, force: bool = False, streams: bool = False) -> Dict:
    """Pick and set the fastest tuning for this plan and batch shape.
    Returns {"tuning": ..., "ms": ..., "key": ..., "cached": bool, "tried": [...]},
    and with backward "concurrent_reverse": False, whatever the cache holds:
    captured steps keep their reverse search on one stream, and streams=True
    (which timed them on two) is refused as CapturedStep refuses it."""
    if streams and backward and batch.n_points == 0:
        _g.refuse_concurrent_reverse()
    # reference points keep no reverse index
    one_stream = dict(concurrent_reverse=False) if backward and batch.n_points == 0 else {}
    path = cache_path or _cache_path()
    nb = _g.build_neighbors(plan, batch, ws)
    key = tuning_key(plan, batch, nb, backward)
    cache = _load(path)
    if not force and key in cache:
        plan.set_tuning(**_full(cache[key]["tuning"]))
        return {**cache[key], **one_stream, "key": key, "cached": True}
    if os.environ.get("GMP_AUTOTUNE", "1") == "0":
        return dict(tuning=plan.get_tuning(), ms=None, key=key, cached=False, tried=[])
    G = torch.ones((batch.n_centres, plan.n_features), dtype=plan.dtype, device=batch.species.device)
    t0 = time.time()
    cands = [_full(c) for c in (candidates or DEFAULT_CANDIDATES)]
    times = [[] for _ in cands]
    for _ in range(_ROUNDS):  # interleaved rounds; a candidate's faster round counts
        for c, cand in enumerate(cands):
            plan.set_tuning(**cand)
            times[c].append(_time_config(plan, batch, ws, G, reps, backward))
    tried = [dict(tuning=cand, ms=min(t)) for cand, t in zip(cands, times)]
    b = choose(tried)
    best = (tried[b]["tuning"], tried[b]["ms"])
    plan.set_tuning(**best[0])
    entry = dict(tuning=best[0], ms=best[1], **one_stream)
    entry["search_s"] = time.time() - t0
    cache[key] = entry
    try:
        os.makedirs(os.path.dirname(path), exist_ok=True)
        tmp = path + ".tmp%d" % os.getpid()
        with open(tmp, "w") as f:
            json.dump(cache, f, indent=1, sort_keys=True)
        os.replace(tmp, path)
    except OSError:
        pass
    return dict(entry, key=key, cached=False, tried=tried)
