"""Gradients of one layer: subgraphs of at most 13 qubits run their optimiser steps
in the one-layer kernel (against separate gradient and Adam calls, bit for bit; its
gradients meet the oracle in test_gpu_small.py), larger ones keep the
4096-amplitude tiles."""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd import _abi, autotune, synth
from paper_2603_26232_amd.batch import QaoaBatch
from paper_2603_26232_amd.partition import batch_arrays
from test_gpu_small import _edges


@pytest.mark.gpu
@pytest.mark.parametrize("sizes,heavy,iters,start", [(list(range(1, 14)), False, 5, 0), ([13, 10], True, 3, 2),
                                                     ([9, 14, 12], False, 4, 0)])
def test_steps_in_the_kernel_match_separate_calls(sizes, heavy, iters, start):
    B = len(sizes)
    edges = [_edges(n, 60 + n, heavy and n < 14) for n in sizes]
    gamma, beta = synth.uniform_angles(71, 1, batch=B)
    bt = QaoaBatch(sizes, edges, max_p=1, max_k=4, gradient=True)
    th0 = torch.as_tensor(np.concatenate([np.ravel(gamma), np.ravel(beta)]), device="cuda")
    out = []
    for fused in (True, False):
        th, m, v = th0.clone(), torch.zeros_like(th0), torch.zeros_like(th0)
        st = torch.full((1,), start, dtype=torch.int32, device="cuda")
        E, g = torch.zeros(B, dtype=torch.float64, device="cuda"), torch.zeros_like(th0)
        if fused:
            _abi.qaoa_optimize(bt.handle, 1, iters, th.data_ptr(), m.data_ptr(), v.data_ptr(), st.data_ptr(), 0.05,
                               0.9, 0.999, 1e-8, E.data_ptr(), 0)
            assert torch.equal(bt.expectation(), E)  # <C> of the last step's starting angles
        else:
            for _ in range(iters):
                _abi.qaoa_expectation_grad(bt.handle, 1, th.data_ptr(), th.data_ptr() + 8 * B, E.data_ptr(),
                                           g.data_ptr(), g.data_ptr() + 8 * B, 0)
                _abi.qaoa_adam_step(2 * B, th.data_ptr(), g.data_ptr(), m.data_ptr(), v.data_ptr(), st.data_ptr(),
                                    0.05, 0.9, 0.999, 1e-8, 1, 0)
        out.append((th, m, v, st, E))
    torch.cuda.synchronize()
    for a, b in zip(*out):
        assert torch.equal(a, b)
    bt.close()


def test_larger_subgraphs_keep_the_narrow_tiles():
    g = synth.erdos_renyi(24, 0.06, 3)
    arrays = batch_arrays([24], [(g.u, g.v, g.w)])

    def size(p, split=None):
        _abi.qaoa_tune_group_split(24, split)
        try:
            return _abi.qaoa_workspace_bytes(1, arrays[0], arrays[1], arrays[4], p, 1, 0x1 | 0x80)
        finally:
            _abi.qaoa_tune_group_split(24, None)

    narrow = autotune.default_split(24)
    assert size(1) == size(1, narrow)
    assert size(2) < size(2, narrow)  # wide: a checkpoint fewer per layer
