"""Top-k over runs of tiles: states written into the workspace so that the
threshold and the buffer meet their edges (probabilities ascending through the
state, descending, random, all equal, mostly zero), subgraphs that begin and end
inside runs, canonical and raw, against a sort of the same FP32 probabilities."""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd.batch import QaoaBatch, idx_to_uint32

pytestmark = pytest.mark.gpu


def _path(n):  # no free vertex: every tie group is a single string (raw: a complement pair)
    u = np.arange(n - 1, dtype=np.int32)
    return u, (u + 1).astype(np.int32), np.ones(n - 1, np.int32)


def _amplitudes(kind, size, seed):
    rng = np.random.default_rng(seed)
    if kind == "random":
        x = rng.random(size, dtype=np.float32)
    elif kind in ("ascending", "descending"):
        x = (np.arange(size, dtype=np.float64) / size).astype(np.float32)
        x = x if kind == "ascending" else x[::-1].copy()
    elif kind == "equal":
        x = np.full(size, 0.25, np.float32)
    else:
        x = np.zeros(size, np.float32)
        x[rng.integers(0, size, 5)] = 1e-3
    return x


def _expected(n, x, k, raw):
    """Strings by (probability descending, z ascending); raw: a complement
    pair's strings follow each other in rank order, so only pairs are compared."""
    p = np.float32(0.5) * (x * x)
    z = np.arange(x.size, dtype=np.int64)
    full = (1 << n) - 1
    if not raw:
        z = np.where(z & 1, z ^ full, z)  # the member with bit 0 clear
    kk = min(k, p.size)
    cand = np.argpartition(-p, kk - 1)[:kk]
    cand = np.nonzero(p >= p[cand].min())[0]  # with the ties at the boundary
    order = np.lexsort((z[cand], -p[cand].astype(np.float64)))[:kk]
    return z[cand][order], p[cand][order]


@pytest.mark.parametrize("sizes,k,raw", [([14, 25, 9, 20], 16, False), ([25, 13], 64, False), ([24, 25, 3], 7, True),
                                         ([12], 64, True), ([13], 64, False), ([1, 2, 5], 8, False)])
def test_runs_of_tiles(sizes, k, raw):
    bt = QaoaBatch(sizes, [_path(n) for n in sizes], max_p=1, max_k=k, raw_topk=raw)
    one = np.full((len(sizes), 1), 0.3)
    bt.apply_layers(one, one)
    for kind in ("random", "ascending", "descending", "equal", "sparse"):
        xs = [_amplitudes(kind, 1 << (n - 1), 7 + b) for b, n in enumerate(sizes)]
        for b, x in enumerate(xs):
            bt.reduced_state(b).copy_(torch.as_tensor(x.astype(np.complex64), device="cuda"))
        idx, prob = bt.topk(k)
        idx, prob = idx_to_uint32(idx).astype(np.int64), prob.cpu().numpy()
        for b, n in enumerate(sizes):
            full = (1 << n) - 1
            if raw and n > 1:  # groups of two: string and complement
                pairs = k // 2
                z, p = _expected(n, xs[b], pairs, True)
                kk = len(z)
                assert np.array_equal(np.minimum(idx[b][0:2 * kk:2], idx[b][1:2 * kk:2]), z), (kind, n)
                assert np.array_equal(idx[b][0:2 * kk:2] ^ full, idx[b][1:2 * kk:2]), (kind, n)
                assert np.array_equal(prob[b][0:2 * kk:2], p), (kind, n)
            else:
                z, p = _expected(n, xs[b], k, False)
                kk = len(z)
                assert np.array_equal(idx[b][:kk], z) and np.array_equal(prob[b][:kk], p), (kind, n)
                assert np.all(idx[b][kk:] == 0xFFFFFFFF) and np.all(prob[b][kk:] == -1.0), (kind, n)
    bt.close()
