"""maxcut_eval where assignments are laid out in LDS and where they are looked up in
their packed words, on both sides of the line: vertices to a workgroup's edges (1/2, and
1/4 with 1024 threads and one or two assignments), one or two assignments a workgroup in
the words, split edges, ids out of range. Exact, against the sums in int64 of
test_gpu_maxcut_split.py."""
import numpy as np
import pytest

from test_gpu_maxcut_split import _case, _expected, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nV,nE,A", [(8000, 3999, 2050), (8000, 4000, 2050), (8001, 4000, 2050),    # 256 threads, eight
                                     (10000, 4999, 2049), (10000, 5000, 2049), (20000, 9999, 1030),  # 1024 threads, eight, four
                                     (20000, 4999, 513), (20000, 5000, 513), (20001, 5000, 3),       # two and one
                                     (131072, 5000, 520), (131073, 5000, 520), (61440, 15359, 1),
                                     (100000, 40000, 1), (61000, 40000, 200), (1, 1, 1), (500000, 4097, 2)])
def test_both_sides_of_the_line(nV, nE, A):
    u, v, w, x = _case(nV, nE, A, 3 * nV + nE + A)
    assert np.array_equal(_run(u, v, w, x, nV), _expected(u, v, w, x))


@pytest.mark.parametrize("nV,nE,A,at,bad", [(20000, 100, 300, 99, -1), (50000, 5000, 600, 0, 50000),
                                            (100000, 40000, 2, 39999, 2 ** 31 - 1)])
def test_an_id_out_of_range(nV, nE, A, at, bad):
    u, v, w, x = _case(nV, nE, A, 6)
    u[at] = bad
    assert np.all(_run(u, v, w, x, nV) == -1)
