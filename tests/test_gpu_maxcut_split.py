"""maxcut_eval over its groups of assignments (1, 2, 4, 8 to a workgroup, with a
remainder), split edges, vertices beyond those held in LDS, extreme and negative
weights, and out-of-range ids in every form, against the same sum in int64 (exact)."""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd.solve import maxcut_eval

pytestmark = pytest.mark.gpu


def _case(nV, nE, A, seed):
    rng = np.random.default_rng(seed)
    u, v = (rng.integers(0, nV, nE).astype(np.int32) for _ in range(2))
    w = rng.integers(-2 ** 31, 2 ** 31, nE).astype(np.int32)
    x = rng.integers(0, 2 ** 32, (A, (nV + 31) // 32), dtype=np.uint32)
    return u, v, w, x


def _run(u, v, w, x, nV):
    dev = tuple(torch.as_tensor(a, device="cuda") for a in (u, v, w))
    return maxcut_eval(dev, nV, torch.as_tensor(x.view(np.int32), device="cuda")).cpu().numpy()


def _expected(u, v, w, x):
    out = np.empty(len(x), np.int64)
    for a, row in enumerate(x):
        bit = lambda t: (row[t >> 5] >> (t & 31).astype(np.uint32)) & 1
        out[a] = w.astype(np.int64)[bit(u) != bit(v)].sum()
    return out


@pytest.mark.parametrize("nV,nE,A", [(1, 0, 1), (33, 5, 511), (65, 100, 513), (1000, 4097, 1025), (300, 5000, 2050), (300, 1000, 2049), (77, 4095, 1030),
                                     (2000, 16383, 1), (2000, 16384, 1), (2000, 70001, 3), (61440, 40000, 2),
                                     (61441, 40000, 130)])
def test_groups_and_splits(nV, nE, A):
    u, v, w, x = _case(nV, nE, A, nV + nE + A)
    assert np.array_equal(_run(u, v, w, x, nV), _expected(u, v, w, x))


@pytest.mark.parametrize("nV,nE,A,at,bad", [(100, 20, 3, 19, -1), (100, 70001, 3, 70000, 100), (100, 70001, 300, 0, 2 ** 31 - 1),
                                            (70000, 40000, 1, 20000, -2 ** 31), (100, 40, 2050, 7, 128)])
def test_an_id_out_of_range_flags_every_result(nV, nE, A, at, bad):
    u, v, w, x = _case(nV, nE, A, 5)
    v[at] = bad
    assert np.all(_run(u, v, w, x, nV) == -1)
