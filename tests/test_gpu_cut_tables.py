"""Cut tables: with every beta zero the state is exp(-i gamma C(z)), so with
gamma = 2 pi / (weight sum + 1) each amplitude's phase names its C(z) among all
possible values (spaced at least 3e-3 rad; the FP32 phase is good to 1e-6). One
layer reads group 0's table, a second layer the last group's. Sizes: fewer
entries than a lane holds, part of a tile, whole tiles, every last group of a few
splits, wide tiles, several tiles and several subgraphs per workgroup, both entry
widths up to the largest weight sum, repeated edges, against the oracle's table."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu


def _graph(n, seed, kind):
    p = {"sparse": 1.5 / n, "dense": 0.6}.get(kind, 0.3)
    g = synth.erdos_renyi(n, p, seed)
    u, v = np.asarray(g.u, np.int32), np.asarray(g.v, np.int32)
    w = np.ones(len(u), np.int32)
    if kind == "heavy" and len(u):  # the largest weight sum, 2047, with a repeated edge the other way round
        u, v = np.append(u, v[0]).astype(np.int32), np.append(v, u[0]).astype(np.int32)
        rng = np.random.default_rng(seed)
        w = np.maximum(1, (rng.dirichlet(np.ones(len(u))) * 1500).astype(np.int32))
        w[-1] += 2047 - w.sum()
    elif kind == "dense":
        w = synth.random_weights(len(u), seed, 1, 9)
    return u, v, np.asarray(w, np.int32)


@pytest.mark.parametrize("kind", ["sparse", "dense", "heavy"])
@pytest.mark.parametrize("sizes", [[1, 2, 3, 4, 5, 6], [11, 12, 13, 14, 15], [13] * 40 + [14] * 3, [16, 17, 18, 19, 20],
                                   [21, 21, 22], [23, 24, 24]])
def test_tables_name_every_cut_value(sizes, kind):
    edges = [_graph(n, 100 * n + b, kind) for b, n in enumerate(sizes)]
    bt = QaoaBatch(sizes, edges, max_p=2, max_k=1)
    sums = np.array([int(w.sum()) + 1 for _, _, w in edges], np.float64)
    for layer in (0, 1):
        gamma, beta = np.zeros((len(sizes), 2)), np.zeros((len(sizes), 2))
        gamma[:, layer] = 2 * np.pi / sums
        bt.apply_layers(gamma, beta)
        for b, n in enumerate(sizes):
            if b > 6 and b % 7:
                continue
            psi = bt.reduced_state(b)
            C = torch.as_tensor(oracle.cut_table(n, *edges[b])[:psi.numel()].astype(np.float64), device="cuda")
            got = torch.remainder(torch.round(-torch.angle(psi.to(torch.complex128)) / gamma[b, layer]), sums[b])
            assert torch.equal(got, C), (n, b, layer)
