"""The predictor's kernels at the edges of their tiles (units above and below a
power of two, one and two chunks of weights, partial groups of samples, tiles of
4 x 8 weight gradients), against the FP64 oracle with the tolerances of
test_gpu_mlp.py; Adam on one workgroup's worth of parameters and on more."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import _abi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,in_dim,H,out", [(1, 1, 1, 1), (5, 7, 33, 3), (33, 64, 129, 64), (9, 3, 256, 1),
                                            (70, 64, 31, 5), (64, 18, 128, 6), (200, 33, 200, 17)])
def test_forward_and_gradient(B, in_dim, H, out):
    rng = np.random.default_rng(B + H)
    npar = _abi.qaoa_mlp_num_params(in_dim, H, out)
    P = rng.normal(0, 1.0 / np.sqrt(max(in_dim, H)), npar)
    X = rng.normal(0, 1, (B, in_dim)).astype(np.float32)
    T = rng.normal(0, 1, (B, out)).astype(np.float32)
    d = {k: torch.as_tensor(v, device="cuda") for k, v in dict(P=P, X=X, T=T).items()}
    Y = torch.full((B, out), np.nan, dtype=torch.float32, device="cuda")
    A = torch.full((B, 2 * H), np.nan, dtype=torch.float32, device="cuda")
    sb = _abi.qaoa_mlp_scratch_bytes(B, in_dim, H, out)
    S = torch.full((sb,), 255, dtype=torch.uint8, device="cuda")
    G = torch.full((npar,), np.nan, dtype=torch.float64, device="cuda")
    L = torch.empty(1, dtype=torch.float64, device="cuda")
    p = lambda t: int(t.data_ptr())
    _abi.qaoa_mlp_forward(B, in_dim, H, out, p(d["P"]), p(d["X"]), p(Y), p(A), 0)
    _abi.qaoa_mlp_backward(B, in_dim, H, out, p(d["P"]), p(d["X"]), p(Y), p(A), p(d["T"]), p(S), sb, p(G), p(L), 0)
    torch.cuda.synchronize()
    Y_ref = oracle.mlp_forward(P, X.astype(np.float64), H, out)
    loss, G_ref = oracle.mlp_loss_grad(P, X.astype(np.float64), T.astype(np.float64), H)
    assert np.max(np.abs(Y.cpu().numpy() - Y_ref) / np.maximum(1, np.abs(Y_ref))) <= 1e-4
    assert abs(float(L[0]) - loss) <= 1e-5 * max(1.0, loss)
    assert np.max(np.abs(G.cpu().numpy() - G_ref)) <= 1e-4 * max(1.0, float(np.abs(G_ref).max()))
    assert not torch.isnan(A).any()


@pytest.mark.parametrize("n", [1, 255, 256, 257, 5000])
def test_adam_step_counts(n):
    rng = np.random.default_rng(n)
    th, m, v = rng.normal(size=n), np.zeros(n), np.zeros(n)
    d = [torch.as_tensor(x.copy(), device="cuda") for x in (th, m, v)]
    step = torch.zeros(1, dtype=torch.int32, device="cuda")
    for t in range(1, 4):
        g = rng.normal(size=n)
        dg = torch.as_tensor(g, device="cuda")
        _abi.qaoa_adam_step(n, d[0].data_ptr(), dg.data_ptr(), d[1].data_ptr(), d[2].data_ptr(), step.data_ptr(), 0.01,
                            0.9, 0.999, 1e-8, 0, 0)
        oracle.adam_update(th, g, m, v, t, 0.01, maximise=False)
    assert int(step[0]) == 3
    assert np.max(np.abs(d[0].cpu().numpy() - th)) <= 1e-12
