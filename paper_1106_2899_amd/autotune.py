"""Autotuner for the chain-to-wavefront mapping of the step kernel.

Chains are bucketed by length into the classes (2..8], (8..16], (16..32],
(32..64], (64..128].  For every class present in an ensemble the tuner times
each supported mapping (W lanes per chain, B beads per lane, W*B >= the
longest chain of the class) on a probe ensemble made of a sample of that
class's chains in their elements, sampled at the ensemble's own stress
interval, using the library's kernel timing mode (HIP events around the
step-kernel launches).  Given the ensemble's velocity-gradient table, every
element of a probe runs under its own kappa, so that the timing includes the
flow terms the workload executes.

A mapping set for one class changes how all chains run: chains with their
default mappings may be packed side by side, and the classes' kernels run side
by side.  Where a class has a faster mapping than its default, the whole
ensemble (of 2^18 chains or fewer, else such a sample of it) is therefore timed
with the faster mappings and with the defaults, and the faster of the two is
applied.

Trajectories do not depend on the mapping but for one thing: in FP32 under
flow, where chains of several elements share a wavefront, a bead in some 10^6
may differ by a rounding (see ssp_set_mapping).
"""
from __future__ import annotations

import json
import os
from dataclasses import dataclass, field
from typing import Dict, List, Optional, Tuple

import numpy as np

CLASSES = [(2, 8), (9, 16), (17, 32), (33, 64), (65, 128)]
MAPPINGS = [(8, 1), (16, 1), (32, 1), (64, 1), (16, 2), (32, 2), (64, 2)]
# A mapping other than the default (the first of MAPPINGS that fits) has to be
# this much faster: of two mappings that differ by less the probes name now the
# one, now the other.
KEEP_DEFAULT = 1.05
# Probes of a class that has more than so many wave tasks hold more, too: below, the
# step runs another kernel (the low-latency form).
PROBE_WAVE_TASKS = 2048
WHOLE_CHAINS = 1 << 18  # most chains of the whole-ensemble probe
CACHE_VERSION = 2


def candidates(n_max: int) -> List[Tuple[int, int]]:
    return [(w, b) for (w, b) in MAPPINGS if w * b >= n_max]


@dataclass
class TuneResult:
    choices: Dict[Tuple[int, int], Tuple[int, int]] = field(default_factory=dict)
    timings: Dict[Tuple[int, int], Dict[Tuple[int, int], float]] = field(default_factory=dict)  # ns per bead-step

    def to_json(self) -> str:
        return json.dumps({
            "choices": {f"{lo}-{hi}": list(m) for (lo, hi), m in self.choices.items()},
            "timings_ns_per_bead_step": {f"{lo}-{hi}": {f"{w}x{b}": t for (w, b), t in d.items()}
                                         for (lo, hi), d in self.timings.items()},
        })


def _time_mappings(lengths: np.ndarray, elements: np.ndarray, mappings, precision: str, steps: int, seed: int, kappa,
                   device, sample_every: int) -> float:
    """ns per bead-step of chains of `lengths` in the elements `elements` (sorted)
    with `mappings` [(n_lo, n_hi, W, B)] set; kappa: None (at rest) or one row of 9
    for each of the ensemble's elements."""
    import torch

    from .ensemble import Ensemble

    present, first = np.unique(elements, return_index=True)
    off = np.append(first, len(lengths))
    e = Ensemble(lengths, n_elements=len(present), element_offsets=off, precision=precision, seed=seed, corr_levels=0,
                 use_graph=False, sample_every=sample_every, max_steps_per_launch=steps, device=device)
    try:
        k = None if kappa is None else torch.as_tensor(np.ascontiguousarray(kappa[present]), device=e.device)
        for m in mappings:
            e.set_mapping(*m)
        e.init()
        e.step(steps, k)  # warm-up launch
        e.set_kernel_timing(True)
        e.step(steps, k)
        e.step(steps, k)
        ms, launches, bead_steps = e.kernel_time()
        return ms * 1e6 / bead_steps
    finally:
        e.close()


def tune(ensemble, kappa=None, *, steps: int = 200, probe_chains: int = 16384, seed: int = 12345,
         cache: Optional[str] = None, apply: bool = True) -> TuneResult:
    """Times every candidate mapping per length class of `ensemble` and applies
    the fastest, unless the ensemble as a whole is faster with the defaults.
    kappa: the ensemble's velocity gradients [E][9] (or [E][3][3]; None: at
    rest), so that probes run the workload's flow terms.  `cache`: optional JSON
    file of previous choices that is reused when present, for ensembles of the
    same precision, flow or rest, and numbers of chains (by powers of two) in
    the classes and of elements."""
    res = TuneResult()
    cached = {}
    if cache and os.path.exists(cache):
        with open(cache) as f:
            cached = json.load(f)
    kap = None
    if kappa is not None:
        k = np.asarray(kappa.detach().cpu() if hasattr(kappa, "detach") else kappa, dtype=np.float64)
        k = k.reshape(-1, 9)
        if k.shape[0] == 1:
            k = np.repeat(k, ensemble.n_elements, axis=0)
        if np.any(k != 0.0):
            kap = k
    N = ensemble.N
    elem = np.repeat(np.arange(ensemble.n_elements), np.diff(np.asarray(ensemble.element_offsets, dtype=np.int64)))
    rng = np.random.default_rng(seed)
    args = (ensemble.precision, steps, seed, kap, ensemble.device, ensemble.sample_every)

    def sample(idx, most):
        return idx if idx.size <= most else np.sort(rng.choice(idx, size=most, replace=False))

    classes = {}  # (lo, hi): chains, the class's range of lengths, its default mapping
    for lo, hi in CLASSES:
        idx = np.nonzero((N >= lo) & (N <= hi))[0]
        if idx.size:
            n_lo, n_hi = int(N[idx].min()), int(N[idx].max())
            classes[lo, hi] = (idx, n_lo, n_hi, candidates(n_hi)[0])
    shape = "-".join(str(int(np.log2(classes[c][0].size))) if c in classes else "x" for c in CLASSES)
    prefix = (f"v{CACHE_VERSION}:{ensemble.precision}{'' if kap is None else ':flow'}:{shape}"
              f":E{int(np.log2(ensemble.n_elements))}")
    keys = {(lo, hi): f"{prefix}:{lo}-{hi}" for lo, hi in classes}
    if all(k in cached for k in keys.values()):
        res.choices = {c: tuple(cached[k]) for c, k in keys.items()}
    else:
        for c, (idx, n_lo, n_hi, default) in classes.items():
            per_wave = 64 // default[0]
            most = probe_chains
            if most >= PROBE_WAVE_TASKS * per_wave:  # (a caller's smaller probe stays as it is)
                most = max(most, 2 * PROBE_WAVE_TASKS * per_wave)
            pick = sample(idx, most)
            times = {m: _time_mappings(N[pick], elem[pick], [(n_lo, n_hi, *m)], *args) for m in candidates(n_hi)}
            res.timings[c] = times
            best = min(times, key=times.get)
            res.choices[c] = default if times[default] <= KEEP_DEFAULT * times[best] else best
            probed_whole = pick.size == N.size
        if not probed_whole and any(res.choices[c] != v[3] for c, v in classes.items()):
            pick = sample(np.arange(N.size), WHOLE_CHAINS)
            chosen = [(v[1], v[2], *res.choices[c]) for c, v in classes.items()]
            t_default = _time_mappings(N[pick], elem[pick], [], *args)
            t_chosen = _time_mappings(N[pick], elem[pick], chosen, *args)
            if t_default <= t_chosen:
                res.choices = {c: v[3] for c, v in classes.items()}
        cached.update({keys[c]: list(m) for c, m in res.choices.items()})
    if apply:
        for c, (idx, n_lo, n_hi, default) in classes.items():
            ensemble.set_mapping(n_lo, n_hi, *res.choices[c])
    if cache:
        with open(cache, "w") as f:
            json.dump(cached, f, indent=1)
    return res
