"""Phase tables of the whole-state kernel: one entry per cut value, or their parts
where a table has more than two entries per thread (64 threads up to 10 qubits, 256 for
11 and 12, 512 for 13) or the layers' tables more than 4096 entries, at the edges of
both, against the FP64 oracle with the tolerances of test_gpu_sim.py (gradients on the
scale of each kind); a short table's results do not depend on a long one beside it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu

AMP_TOL, E_TOL, G_TOL = 1e-5, 1e-5, 1e-4


def _edges(n, total, seed):
    """A graph whose weights add up to `total`."""
    g = synth.erdos_renyi(n, 0.5, seed) if n > 2 else synth.erdos_renyi(n, 1.0, seed)
    m = g.num_edges
    w = np.full(m, total // m, np.int32)
    w[:total % m] += 1
    return g.u, g.v, w


def _check(sizes, edges, p, steps):
    gamma, beta = synth.uniform_angles(50 + p, p, batch=len(sizes))
    gamma = gamma / steps
    bt = QaoaBatch(sizes, edges, max_p=p, max_k=1, gradient=True)
    bt.apply_layers(gamma, beta)
    E = bt.expectation().cpu().numpy()
    states = [bt.state(b).cpu().numpy() for b in range(len(sizes))]
    Eg, dg, db = (t.cpu().numpy() for t in bt.expectation_grad(gamma, beta))
    for b, n in enumerate(sizes):
        C = oracle.cut_table(n, *edges[b])
        assert np.abs(states[b] - oracle.qaoa_state(n, C, gamma[b], beta[b])).max() <= AMP_TOL, n
        e_ref, g_ref, b_ref = oracle.gradient(n, C, gamma[b], beta[b])
        for e in (E[b], Eg[b]):
            assert abs(e - e_ref) <= E_TOL * max(1.0, abs(e_ref)), n
        assert np.abs(dg[b] - g_ref).max() <= G_TOL * max(1.0, np.abs(g_ref).max()), n
        assert np.abs(db[b] - b_ref).max() <= G_TOL * max(1.0, np.abs(b_ref).max()), n
    bt.close()


# entries per layer (weight sum + 1) up to / above two per thread
@pytest.mark.parametrize("sizes,entries", [([2, 5, 8, 9, 10], 128), ([2, 5, 8, 9, 10], 129), ([11, 12], 512),
                                           ([11, 12], 513), ([13], 1024), ([13], 1025), ([3, 7, 10, 12, 13], 2048),
                                           ([6, 10], 160), ([4, 10], 161)])
def test_entries_per_thread(sizes, entries):
    _check(sizes, [_edges(n, entries - 1, 70 + n) for n in sizes], 2, 100.0 if entries > 500 else 10.0)


# all layers' tables up to / above 4096 entries
@pytest.mark.parametrize("sizes,p,entries", [([10, 4], 32, 128), ([11, 12], 16, 256), ([11, 12], 16, 257),
                                             ([13], 8, 512), ([13], 8, 513), ([13, 9], 32, 129), ([12, 7], 32, 2048)])
def test_entries_of_all_layers(sizes, p, entries):
    _check(sizes, [_edges(n, entries - 1, 80 + n) for n in sizes], p, 100.0)


@pytest.mark.parametrize("n", [6, 10, 12, 13])
def test_a_short_table_beside_a_long_one(n):
    p = 3
    gamma, beta = synth.uniform_angles(61, p, batch=2)
    short, long = _edges(n, 60, 91), _edges(n, 2047, 92)

    def run(edges, rows):
        bt = QaoaBatch([n] * len(edges), edges, max_p=p, max_k=1, gradient=True)
        bt.apply_layers(gamma[rows], beta[rows])
        out = [torch.view_as_real(bt.reduced_state(0)).clone()]
        out += [t[0].clone() for t in bt.expectation_grad(gamma[rows], beta[rows])]
        bt.close()
        return out

    for a, b in zip(run([short], [0]), run([short, long], [0, 1])):
        assert torch.equal(a, b)
