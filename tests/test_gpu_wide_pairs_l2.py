"""26-qubit states (pairs of wide tiles) against the FP64 oracle in the L2 norm, all
amplitudes: one state, with and without flips, two states beside another size, both
cut-table widths (the largest difference of single amplitudes, whose size is 1e-4, would
not show a wrong part of the state)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import synth
from test_gpu_wide import AMP_TOL, E_TOL, L2_TOL, _batch, _edges

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("sizes,p,heavy", [([26], 2, True), ([26, 22, 26], 1, False)])
def test_states(sizes, p, heavy):
    edges = [_edges(n, 1, 90 + 3 * i, heavy=heavy)[0] for i, n in enumerate(sizes)]
    gamma, beta = synth.uniform_angles(810 + p, p, batch=len(sizes))
    bt = _batch(sizes, edges, max_p=p, max_k=1)
    bt.apply_layers(gamma, beta)
    E = bt.expectation().cpu().numpy()
    for b, n in enumerate(sizes):
        C = oracle.cut_table(n, *edges[b])
        ref = oracle.qaoa_state(n, C, gamma[b], beta[b])
        e_ref = oracle.expectation(n, ref, C)
        assert abs(E[b] - e_ref) <= E_TOL * max(1.0, abs(e_ref))
        half = torch.as_tensor(ref[:1 << (n - 1)] * np.sqrt(2.0), device="cuda")
        err = (bt.reduced_state(b).to(torch.complex128) - half).abs()
        assert float(err.max()) <= np.sqrt(2) * AMP_TOL and float((err ** 2).sum()) ** 0.5 <= L2_TOL
        del ref, half, err
    bt.close()
