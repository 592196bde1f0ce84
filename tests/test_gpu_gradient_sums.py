"""Gradient sums with terms that cancel: dE/dgamma and dE/dbeta each against the
FP64 oracle on its own scale (test_gpu_sim.py's relative tolerance), so that the
smaller of the two does not hide behind the larger. Weighted edges: whole states of at
most 13 qubits near the weight limit, wide tiles (21..23 qubits) at the largest weight
sum they take gradients of."""
import numpy as np
import pytest

import oracle
from paper_2603_26232_amd import synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu

G_TOL = 1e-4


def _check(sizes, edges, gamma, beta, **kw):
    bt = QaoaBatch(sizes, edges, max_p=gamma.shape[1], max_k=1, gradient=True, **kw)
    _, dg, db = (t.cpu().numpy() for t in bt.expectation_grad(gamma, beta))
    for b, n in enumerate(sizes):
        _, g_ref, b_ref = oracle.gradient(n, oracle.cut_table(n, *edges[b]), gamma[b], beta[b])
        for got, ref in ((dg[b], g_ref), (db[b], b_ref)):
            assert np.abs(got - ref).max() <= G_TOL * max(1.0, np.abs(ref).max()), (n, got, ref)
    bt.close()


@pytest.mark.parametrize("p,total,steps", [(2, 1900, 100.0), (4, 250, 10.0), (3, 40, 1.0)])
def test_whole_states(p, total, steps):
    sizes, edges = list(range(2, 14)), []
    for n in sizes:
        g = synth.erdos_renyi(n, 0.6, 90 + n)
        w = synth.random_weights(g.num_edges, 95 + n, 1, 9)
        edges.append((g.u, g.v, np.maximum(1, w * total // max(1, int(w.sum()))).astype(np.int32)))
    gamma, beta = synth.uniform_angles(300 + p, p, batch=len(sizes))
    _check(sizes, edges, gamma / steps, beta)


@pytest.mark.parametrize("memory", ["checkpoints", "inplace"])
@pytest.mark.parametrize("n,B,p", [(21, 2, 2), (22, 1, 3), (23, 1, 4)])
def test_wide_tiles(n, B, p, memory):
    edges = []
    for b in range(B):
        g = synth.erdos_renyi(n, 0.5, 70 + n + b)
        pick = np.random.default_rng(n + b).choice(g.num_edges, n // 4, replace=False)
        w = np.full(pick.size, (3 * n // 2) // pick.size, np.int32)  # weight sum <= 1.5 n
        edges.append((g.u[pick], g.v[pick], w))
    gamma, beta = synth.uniform_angles(310 + p, p, batch=B)
    _check([n] * B, edges, gamma, beta, gradient_memory=memory)
