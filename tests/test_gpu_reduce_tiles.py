"""The reductions of the tiles' sums over one, several and many rounds of a workgroup's
threads (up to 256 tiles, up to 2048, more; 4096-amplitude and wide tiles): optimiser
steps, whose kernel reduces by itself, against separate gradient and Adam calls, bit for
bit, and the gradient against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import _abi, synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu

E_TOL, G_TOL = 1e-5, 1e-4


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,edges,check", [(21, 60, True), (22, 60, True), (24, 70, False), (25, 80, False), (25, 30, False),
                                           (24, 30, True), (21, 20, True), (14, 30, True)])
def test_rounds(n, edges, check):
    p = 2
    g = synth.erdos_renyi(n, 0.5, 3 * n)
    e = (g.u[:edges], g.v[:edges], g.w[:edges])
    gamma, beta = synth.uniform_angles(40 + n, p, batch=1)
    bt = QaoaBatch([n], [e], max_p=p, max_k=1, gradient=True)
    if check:
        E, dg, db = (t.cpu().numpy()[0] for t in bt.expectation_grad(gamma, beta))
        e_ref, g_ref, b_ref = oracle.gradient(n, oracle.cut_table(n, *e), gamma[0], beta[0])
        assert abs(E - e_ref) <= E_TOL * max(1.0, abs(e_ref))
        for got, ref in ((dg, g_ref), (db, b_ref)):
            assert np.abs(got - ref).max() <= G_TOL * max(1.0, np.abs(ref).max())
    th0 = torch.as_tensor(np.concatenate([gamma.reshape(-1), beta.reshape(-1)]), device="cuda")
    out = []
    for fused in (True, False):
        th, m, v, grad = th0.clone(), torch.zeros_like(th0), torch.zeros_like(th0), torch.zeros_like(th0)
        st = torch.zeros(1, dtype=torch.int32, device="cuda")
        E = torch.zeros(1, dtype=torch.float64, device="cuda")
        if fused:
            _abi.qaoa_optimize(bt.handle, p, 2, th.data_ptr(), m.data_ptr(), v.data_ptr(), st.data_ptr(), 0.05, 0.9,
                               0.999, 1e-8, E.data_ptr(), 0)
        for _ in range(0 if fused else 2):
            _abi.qaoa_expectation_grad(bt.handle, p, th.data_ptr(), th.data_ptr() + 8 * p, E.data_ptr(),
                                       grad.data_ptr(), grad.data_ptr() + 8 * p, 0)
            _abi.qaoa_adam_step(2 * p, th.data_ptr(), grad.data_ptr(), m.data_ptr(), v.data_ptr(), st.data_ptr(),
                                0.05, 0.9, 0.999, 1e-8, 1, 0)
        out.append((th, m, v, st, E))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    bt.close()
