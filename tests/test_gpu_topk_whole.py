"""Top-k where a run of tiles holds whole subgraphs (many small ones, with and without
larger ones beside them) and where the k-th probability is shared by about as many
strings as are ranked directly (256), against test_gpu_topk_runs.py's sort."""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd.batch import QaoaBatch, idx_to_uint32
from test_gpu_topk_runs import _expected, _path

pytestmark = pytest.mark.gpu


def _run(sizes, xs, k):
    bt = QaoaBatch(sizes, [_path(n) for n in sizes], max_p=1, max_k=k)
    one = np.full((len(sizes), 1), 0.3)
    bt.apply_layers(one, one)
    for b, x in enumerate(xs):
        bt.reduced_state(b).copy_(torch.as_tensor(x.astype(np.complex64), device="cuda"))
    idx, prob = bt.topk(k)
    idx, prob = idx_to_uint32(idx).astype(np.int64), prob.cpu().numpy()
    for b, n in enumerate(sizes):
        z, p = _expected(n, xs[b], k, False)
        kk = len(z)
        assert np.array_equal(idx[b][:kk], z) and np.array_equal(prob[b][:kk], p), (b, n)
        assert np.all(idx[b][kk:] == 0xFFFFFFFF) and np.all(prob[b][kk:] == -1.0), (b, n)
    bt.close()


@pytest.mark.parametrize("n", [11, 13, 15, 20])
@pytest.mark.parametrize("same", [63, 255, 256, 257, 500])
@pytest.mark.parametrize("k,above", [(64, 10), (64, 63), (16, 0), (1, 0)])
def test_strings_that_share_the_kth_probability(n, same, k, above):
    rng = np.random.default_rng(n + same + k)
    x = (0.1 * rng.random(1 << (n - 1))).astype(np.float32)
    at = rng.choice(x.size, same + above, replace=False)
    x[at[:same]] = 0.5
    x[at[same:]] = (0.5 + 0.5 * rng.random(above)).astype(np.float32)
    _run([n], [x], k)


@pytest.mark.parametrize("sizes,k", [([4] * 2100, 8), ([3, 5] * 1100 + [15], 6), ([14] + [6] * 2500 + [16, 2], 16)])
def test_many_small_subgraphs(sizes, k):
    rng = np.random.default_rng(len(sizes))
    _run(sizes, [rng.random(1 << (n - 1), dtype=np.float32) for n in sizes], k)
