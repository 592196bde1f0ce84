"""26-qubit states: the strided group's forward passes on pairs of wide tiles
(middle passes, a last pass with and without flips, both cut-table widths, one and
several states, other sizes beside them) against the same circuits on 4096-amplitude
tiles, each of which is within AMP_TOL of the oracle in the tests of the two."""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd import synth
from test_gpu_wide import AMP_TOL, E_TOL, _batch, _edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,p,heavy", [([26], 1, False), ([26], 2, True), ([26, 22, 26], 3, False),
                                           ([26, 14, 9], 4, True)])
def test_pairs(sizes, p, heavy):
    edges = [_edges(n, 1, 90 + 3 * i, heavy=heavy)[0] for i, n in enumerate(sizes)]
    gamma, beta = synth.uniform_angles(800 + p, p, batch=len(sizes))
    both = []
    for narrow in (False, True):
        bt = _batch(sizes, edges, narrow=narrow, max_p=p, max_k=1)
        bt.apply_layers(gamma, beta)
        both.append((bt, bt.expectation().cpu().numpy()))
    (wide, Ew), (tiles, En) = both
    for b in range(len(sizes)):
        x, y = wide.reduced_state(b), tiles.reduced_state(b)
        assert float((x - y).abs().max()) <= 2 * np.sqrt(2) * AMP_TOL  # (stored states are scaled by sqrt 2)
        assert abs(Ew[b] - En[b]) <= 2 * E_TOL * max(1.0, abs(En[b]))
    wide.close()
    tiles.close()
