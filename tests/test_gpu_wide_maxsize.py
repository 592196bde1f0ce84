"""Wide tiles at the largest sizes with rotations (29 and 30 qubits: three groups, strided
ones of 8 and 7 or 8, offsets up to 4 GiB), where the FP64 oracle cannot hold the state:

* p = 1 against the closed form of test_gpu_maxsize.py and its derivatives, forward
  alone and with the adjoint sweep;
* p = 2 with gamma = (g, 0), where the two mixers merge: <C>, dE/dgamma_1 and both
  dE/dbeta are those of p = 1 at beta_1 + beta_2; with gamma = (0, g) the first layer
  does nothing to |+>, so <C>, dE/dgamma_2 and dE/dbeta_2 are those of p = 1 at beta_2 and
  dE/dbeta_1 is 0;
* p = 3 at generic angles against the same circuit on 4096-amplitude tiles.

And the tuned 4096-amplitude split of 24 qubits, named, against the oracle. Which tiles a
batch takes shows in its checkpoints."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import _abi, autotune, synth
from paper_2603_26232_amd.batch import QaoaBatch
from paper_2603_26232_amd.partition import batch_arrays
from test_gpu_maxsize import _norm, _p1_closed_form

E_TOL, G_TOL = 1e-5, 1e-4


def _graph(n):
    if n % 2 == 0:
        g = synth.random_regular3(n, 5)
        return g.u, g.v, g.w
    g = synth.erdos_renyi(n, 0.15, 29)
    pick = np.sort(np.random.default_rng(n).permutation(g.num_edges)[:3 * n // 2])
    return g.u[pick], g.v[pick], g.w[pick]


def _groups(n, edges, split=None):
    nq, off, u, v, w = batch_arrays([n], [edges])
    try:
        _abi.qaoa_tune_group_split(n, split)
        size = lambda p: _abi.qaoa_workspace_bytes(1, nq, off, w, p, 1, 0x1 | 0x80)
        return 1 + (size(3) - size(2)) // (8 << (n - 1))
    finally:
        _abi.qaoa_tune_group_split(n, None)


def _batch(n, edges, split=None, **kw):
    try:
        _abi.qaoa_tune_group_split(n, split)
        return QaoaBatch([n], [edges], max_k=1, **kw)
    finally:
        _abi.qaoa_tune_group_split(n, None)


def _p1(n, u, v, g, b, h=1e-5):
    f = lambda x, y: _p1_closed_form(u, v, n, x, y)
    return f(g, b), (f(g + h, b) - f(g - h, b)) / (2 * h), (f(g, b + h) - f(g, b - h)) / (2 * h)


def test_which_tiles():
    for n in (29, 30):
        assert _groups(n, _graph(n)) == 3 and _groups(n, _graph(n), autotune.default_split(n)) == 4
    g = synth.erdos_renyi(24, 0.15, 2424)
    assert _groups(24, (g.u, g.v, g.w)) == 3  # 47 edges, more than 36
    assert _groups(24, (g.u[:36], g.v[:36], g.w[:36])) == 2


@pytest.mark.gpu
@pytest.mark.parametrize("n,split", [(29, None), (30, None), (30, [6, 6, 6])])
def test_forward_p1(n, split):
    u, v, w = _graph(n)
    g, b = 0.61, 0.37
    bt = _batch(n, (u, v, w), split, max_p=1)
    for beta in (b, b + np.pi / 2):  # (the second flips: |sin| > |cos|)
        bt.apply_layers(np.array([[g]]), np.array([[beta]]))
        ref = _p1_closed_form(u, v, n, g, beta)
        assert abs(float(bt.expectation()[0]) - ref) <= E_TOL * max(1.0, abs(ref))
        assert abs(_norm(bt) - 1.0) <= 1e-5
    bt.close()


def _grad(bt, gamma, beta):
    return [np.atleast_1d(t.cpu().numpy().reshape(-1)) for t in bt.expectation_grad(np.array([gamma]), np.array([beta]))]


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,memory", [(29, "checkpoints"), (30, "checkpoints"), (30, "inplace")])
def test_gradient(n, memory):
    u, v, w = _graph(n)
    m = len(u)
    tol = G_TOL * m  # (each edge's term is of order 1)
    bt = _batch(n, (u, v, w), max_p=2, gradient=True, gradient_memory=memory)
    g, b1, b2 = 0.61, 0.22, 1.13
    E, dg, db = _grad(bt, [g], [b1])
    ref = _p1(n, u, v, g, b1)
    assert abs(E[0] - ref[0]) <= E_TOL * m and abs(dg[0] - ref[1]) <= tol and abs(db[0] - ref[2]) <= tol
    E, dg, db = _grad(bt, [g, 0.0], [b1, b2])
    ref = _p1(n, u, v, g, b1 + b2)
    assert abs(E[0] - ref[0]) <= E_TOL * m and abs(dg[0] - ref[1]) <= tol
    assert np.abs(db - ref[2]).max() <= tol
    E, dg, db = _grad(bt, [0.0, g], [b1, b2])
    ref = _p1(n, u, v, g, b2)
    assert abs(E[0] - ref[0]) <= E_TOL * m and abs(dg[1] - ref[1]) <= tol
    assert abs(db[1] - ref[2]) <= tol and abs(db[0]) <= tol
    bt.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("n", [29, 30])
def test_gradient_p3_on_both_tiles(n):
    u, v, w = _graph(n)
    gamma, beta = synth.uniform_angles(93, 3, batch=1)
    out = []
    for split in (None, autotune.default_split(n)):
        bt = _batch(n, (u, v, w), split, max_p=3, gradient=True, gradient_memory="inplace")
        out.append(_grad(bt, gamma[0], beta[0]))
        bt.close()
        del bt
        torch.cuda.empty_cache()
    (E, dg, db), (En, dgn, dbn) = out
    # each of the two within the bounds of its exact values
    assert abs(E[0] - En[0]) <= 2 * E_TOL * len(u)
    assert np.abs(dg - dgn).max() <= 2 * G_TOL * len(u) and np.abs(db - dbn).max() <= 2 * G_TOL * len(u)


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("edges,split", [(47, [4, 8]), (36, [4, 8]), (36, None)])
def test_gradient_of_24_qubits(edges, split):
    n, p = 24, 3
    g = synth.erdos_renyi(n, 0.15, 2424)
    e = (g.u[:edges], g.v[:edges], g.w[:edges])
    assert _groups(n, e, split) == (3 if split else 2)
    gamma, beta = synth.uniform_angles(2425, p, batch=1)
    bt = _batch(n, e, split, max_p=p, gradient=True)
    E, dg, db = _grad(bt, gamma[0], beta[0])
    e_ref, g_ref, b_ref = oracle.gradient(n, oracle.cut_table(n, *e), gamma[0], beta[0])
    assert abs(E[0] - e_ref) <= E_TOL * max(1.0, abs(e_ref))
    assert np.abs(dg - g_ref).max() <= G_TOL * max(1.0, np.abs(g_ref).max())
    assert np.abs(db - b_ref).max() <= G_TOL * max(1.0, np.abs(b_ref).max())
    bt.close()
