"""Autotuner for the strided qubit groups of the tile passes.

A subgraph with n > 13 qubits is simulated in group 0 (qubits 0..10 and the
top qubit, which acts on the stored half-state as the complement; 4096-
amplitude tiles of two mirrored blocks) plus strided groups of at most 8 of
the qubits 11..n-2, one HBM pass per group and layer. How the n - 12 strided
qubits are split decides each pass's register layout chain, how many register
bits are real qubits and how long the contiguous rows of a strided tile are
(2^(12 - size) amplitudes). Every split gives the same state; the tuner times the
candidate splits (fewest groups, every ordered composition of n - 12 into
parts of at most 8) on a batch of random graphs with n qubits, one optimiser
evaluation (forward pass + adjoint sweep) or one forward evaluation per
repetition, and keeps the fastest.

The library takes wider tiles for some subgraphs of a size and 4096-amplitude ones
for others (dense gradients), and a split named for the size keeps them all on
4096-amplitude tiles. So each size is timed on dense graphs (density 0.15 or, where
that leaves the weight sum at 1.5 n or below, a little above it), for the split of
4096-amplitude tiles, and on sparse ones (at most 1.5 n edges) with that split named
and without. Where the library's own choice is the faster of the two, or is not timed
by this kind of evaluation (gradients of 26 qubits have 4096-amplitude tiles, their
forward evaluations wide ones), the table holds no named split ("split": null), and the
tuned one applies to 4096-amplitude tiles alone ("split_4096_tiles"). The table is
saved as JSON and applied with `apply()` before batches are created.

Run: python -m paper_2603_26232_amd.autotune --n 21 22 ... --out FILE
"""
from __future__ import annotations

import argparse
import itertools
import json
import os

import numpy as np
import torch

from . import synth, _abi
from .batch import QaoaBatch

DEFAULT_TABLE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tuning_gfx950.json")


def candidates(n: int, max_parts: int = 3):
    """Ordered compositions of n - 12 into the fewest parts of size 1..8."""
    R = n - 12
    if n <= 13:  # whole-state kernel, no strided groups
        return []
    parts = -(-R // 8)
    if parts > max_parts:
        return []
    out = []
    for comp in itertools.product(range(1, 9), repeat=parts):
        if sum(comp) == R:
            out.append(list(comp))
    return out


def default_split(n: int):
    R = n - 12
    G1 = -(-R // 8)
    return [R // G1 + (1 if g < R % G1 else 0) for g in range(G1)]


def _graphs(n, B, dense, seed):
    edges = []
    for b in range(B):
        g = synth.erdos_renyi(n, 0.15, seed + b)
        limit = 3 * n // 2
        if dense and g.num_edges <= limit:
            g = synth.erdos_renyi(n, 0.2, seed + b)
        m = max(limit + 1, g.num_edges) if dense else limit
        pick = np.sort(np.random.default_rng(seed + b).permutation(g.num_edges)[:m])
        edges.append((g.u[pick], g.v[pick], g.w[pick]))
        assert (g.w[pick].sum() > limit) == dense
    return edges


def time_split(n, split, p=3, gradient=True, amps=1 << 24, reps=5, seed=0, dense=False):
    """Device milliseconds per evaluation and per 2^20 amplitudes (the least of
    three times `reps` evaluations)."""
    B = max(1, amps >> n)
    gamma, beta = synth.uniform_angles(seed + 999, p, batch=B)
    _abi.qaoa_tune_group_split(n, split)
    try:
        bt = QaoaBatch([n] * B, _graphs(n, B, dense, seed), max_p=p, max_k=8, gradient=gradient)
    finally:
        _abi.qaoa_tune_group_split(n, None)
    g = torch.as_tensor(gamma, device="cuda")
    b = torch.as_tensor(beta, device="cuda")

    def once():
        if gradient:
            bt.expectation_grad(g, b)
        else:
            bt.apply_layers(g, b)
            bt.expectation()

    once()
    torch.cuda.synchronize()
    ms = []
    for _ in range(3):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(reps):
            once()
        ev[1].record()
        torch.cuda.synchronize()
        ms.append(ev[0].elapsed_time(ev[1]) / reps)
    bt.close()
    return min(ms), min(ms) / (B * (1 << n) / (1 << 20))


def tune(ns, p=3, gradient=True, log=print):
    reset(ns)
    table = {}
    for n in ns:
        cands = candidates(n)
        if len(cands) <= 1:
            continue

        def timed(sp, dense):
            ms, per = time_split(n, sp, p=p, gradient=gradient, dense=dense)
            kind = "dense" if dense else "sparse"
            log(f"autotune: n={n} split {sp}, {kind}: {ms:.3f} ms per evaluation ({per:.4f} ms per 2^20 amplitudes)")
            return {"split": sp, "graphs": kind, "ms_per_mamp": per}

        res = sorted((timed(sp, True) for sp in cands), key=lambda r: r["ms_per_mamp"])
        best = res[0]
        dflt = next(r for r in res if r["split"] == default_split(n))
        named, own = timed(best["split"], False), timed(None, False)
        wide = n in (21, 22, 23, 24, 25, 26, 29, 30)  # of some evaluations
        keep = not wide or (own["ms_per_mamp"] > named["ms_per_mamp"] and not (gradient and n == 26))
        table[str(n)] = {"split": best["split"] if keep else None, "split_4096_tiles": best["split"],
                         "ms_per_mamp": (named if keep else own)["ms_per_mamp"],
                         "ms_per_mamp_4096_tiles": best["ms_per_mamp"], "default_split": dflt["split"],
                         "default_ms_per_mamp": dflt["ms_per_mamp"], "all": res + [named, own]}
        log(f"autotune: n={n}: 4096-amplitude tiles {best['split']} ({best['ms_per_mamp']:.4f}), default {dflt['split']} "
            f"({dflt['ms_per_mamp']:.4f}); sparse {named['ms_per_mamp']:.4f}, library's choice {own['ms_per_mamp']:.4f}")
    return table


def apply(path: str = DEFAULT_TABLE) -> dict:
    """Load a tuning table and set it in the library; returns {n: named split}
    (None: the library's choice of tiles)."""
    if not os.path.exists(path):
        return {}
    with open(path) as f:
        data = json.load(f)
    out = {}
    for n, e in data.get("entries", {}).items():
        _abi.qaoa_tune_group_split(int(n), e["split"])
        _abi.qaoa_tune_narrow_split(int(n), e.get("split_4096_tiles"))
        out[int(n)] = e["split"]
    return out


def reset(ns=range(14, 31)):
    for n in ns:
        _abi.qaoa_tune_group_split(n, None)
        _abi.qaoa_tune_narrow_split(n, None)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--n", type=int, nargs="+", default=list(range(21, 31)))
    ap.add_argument("--p", type=int, default=3)
    ap.add_argument("--forward-only", action="store_true")
    ap.add_argument("--out", default=DEFAULT_TABLE)
    args = ap.parse_args()
    log = lambda *a: print(*a, flush=True)
    table = tune(args.n, p=args.p, gradient=not args.forward_only, log=log)
    dev = torch.cuda.get_device_properties(0)
    with open(args.out, "w") as f:
        json.dump({"device": dev.name, "arch": getattr(dev, "gcnArchName", ""), "p": args.p,
                   "gradient": not args.forward_only, "entries": table}, f, indent=1)
    log(f"autotune: wrote {args.out}")


if __name__ == "__main__":
    main()
