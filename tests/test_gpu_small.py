"""The whole-state kernel (n <= 13) at every size it has a layout for, against
the FP64 oracle with the tolerances of test_gpu_sim.py: states, <C>, gradients,
phase tables of all layers at once and one layer at a time (more than 4096
entries), angles that flip, and its in-kernel optimiser against separate
gradient and Adam calls, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import _abi, synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu

AMP_TOL, E_TOL, G_TOL = 1e-5, 1e-5, 1e-4


def _edges(n, seed, heavy):
    if n < 2:
        return (np.zeros(0, np.int32),) * 3
    g = synth.erdos_renyi(n, 0.5, seed)
    w = synth.random_weights(g.num_edges, seed + 9, 1, 9)
    if heavy:  # weight sum near the limit: 2-byte cut tables, long phase tables
        w = (w * (1900 // max(1, w.sum()))).astype(np.int32)
    return g.u, g.v, w


@pytest.mark.parametrize("p,heavy", [(1, False), (2, False), (5, False), (4, True)])
def test_every_size(p, heavy):
    sizes = list(range(1, 14))
    edges = [_edges(n, 30 + n, heavy) for n in sizes]
    gamma, beta = synth.uniform_angles(40 + p, p, batch=len(sizes))
    gamma = gamma / 100.0 if heavy else gamma  # small steps of the phase where C(z) is large
    bt = QaoaBatch(sizes, edges, max_p=p, max_k=4, gradient=True)
    bt.apply_layers(gamma, beta)
    E = bt.expectation().cpu().numpy()
    states = [bt.state(b).cpu().numpy() for b in range(len(sizes))]
    Eg, dg, db = (t.cpu().numpy() for t in bt.expectation_grad(gamma, beta))
    for b, n in enumerate(sizes):
        C = oracle.cut_table(n, *edges[b])
        ref = oracle.qaoa_state(n, C, gamma[b], beta[b])
        assert np.abs(states[b] - ref).max() <= AMP_TOL, n
        e_ref, g_ref, b_ref = oracle.gradient(n, C, gamma[b], beta[b])
        scale = max(1.0, float(np.abs(np.concatenate([g_ref, b_ref])).max()))
        for e in (E[b], Eg[b]):
            assert abs(e - e_ref) <= E_TOL * max(1.0, abs(e_ref)), n
        assert np.abs(dg[b] - g_ref).max() <= G_TOL * scale, n
        assert np.abs(db[b] - b_ref).max() <= G_TOL * scale, n
    bt.close()


@pytest.mark.parametrize("sizes,heavy,iters,start", [(list(range(1, 14)), False, 5, 0), ([13, 10], True, 3, 2),
                                                     ([9, 14, 12], False, 70, 0)])
def test_optimiser_in_the_kernel_matches_separate_calls(sizes, heavy, iters, start):
    """70 steps pass one block of bias corrections; a batch with a tiled
    subgraph takes its steps beside the kernel's; the step count may start
    above zero."""
    p, B = 3, len(sizes)
    edges = [_edges(n, 60 + n, heavy and n < 14) for n in sizes]
    gamma, beta = synth.uniform_angles(70, p, batch=B)
    bt = QaoaBatch(sizes, edges, max_p=p, max_k=4, gradient=True)
    th0 = torch.as_tensor(np.concatenate([gamma.reshape(-1), beta.reshape(-1)]), device="cuda")
    out = []
    for fused in (True, False):
        th, m, v = th0.clone(), torch.zeros_like(th0), torch.zeros_like(th0)
        st = torch.full((1,), start, dtype=torch.int32, device="cuda")
        E, g = torch.zeros(B, dtype=torch.float64, device="cuda"), torch.zeros_like(th0)
        if fused:
            _abi.qaoa_optimize(bt.handle, p, iters, th.data_ptr(), m.data_ptr(), v.data_ptr(), st.data_ptr(), 0.05,
                               0.9, 0.999, 1e-8, E.data_ptr(), 0)
            left = bt.expectation()  # <C> of the last step's starting angles
            assert torch.equal(left, E)
        else:
            P = B * p
            for _ in range(iters):
                _abi.qaoa_expectation_grad(bt.handle, p, th.data_ptr(), th.data_ptr() + 8 * P, E.data_ptr(),
                                           g.data_ptr(), g.data_ptr() + 8 * P, 0)
                _abi.qaoa_adam_step(2 * P, th.data_ptr(), g.data_ptr(), m.data_ptr(), v.data_ptr(), st.data_ptr(),
                                    0.05, 0.9, 0.999, 1e-8, 1, 0)
        out.append((th, m, v, st, E))
    torch.cuda.synchronize()
    for a, b in zip(*out):
        assert torch.equal(a, b)
    bt.close()
