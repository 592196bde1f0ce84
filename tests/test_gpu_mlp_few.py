"""The predictor on few samples (a workgroup each) and on many (several a workgroup):
the same outputs bit for bit on both sides of the line, and gradients against the FP64
oracle on both sides of the line of the errors going back (test_gpu_mlp_sizes.py's
check)."""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd import _abi
from test_gpu_mlp_sizes import test_forward_and_gradient as _check

pytestmark = pytest.mark.gpu


def _forward(P, X, H, out):
    B, n = X.shape
    Y = torch.full((B, out), np.nan, device="cuda")
    A = torch.full((B, 2 * H), np.nan, device="cuda")
    _abi.qaoa_mlp_forward(B, n, H, out, P.data_ptr(), X.data_ptr(), Y.data_ptr(), A.data_ptr(), 0)
    return Y, A


@pytest.mark.parametrize("n,H,out,line", [(18, 128, 6, 256), (64, 256, 64, 256), (3, 65, 7, 256), (64, 64, 3, 1024),
                                          (1, 1, 64, 4096), (33, 31, 2, 3072), (5, 24, 2, 4096)])
def test_forward_on_both_sides_of_the_line(n, H, out, line):
    g = torch.Generator(device="cuda").manual_seed(n + H)
    P = torch.randn(_abi.qaoa_mlp_num_params(n, H, out), dtype=torch.float64, device="cuda", generator=g) / 8
    X = torch.randn(line + 1, n, device="cuda", generator=g)
    many = _forward(P, X, H, out)
    for B in (1, line):
        few = _forward(P, X[:B].contiguous(), H, out)
        for a, b in zip(few, many):
            assert torch.equal(a, b[:B]), B


@pytest.mark.parametrize("B,n,H,out", [(512, 9, 65, 5), (513, 9, 65, 5), (513, 64, 256, 64), (2048, 4, 33, 2),
                                       (2049, 4, 33, 2), (2, 64, 1, 64)])
def test_gradient_on_both_sides_of_the_line(B, n, H, out):
    _check(B, n, H, out)
