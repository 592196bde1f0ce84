"""Subgraphs of different group sizes in one launch per pass: a subgraph's state,
expectation and gradient are bit for bit those it has alone in a batch, whatever
shapes it shares the launches with (groups of 1..4, of 5..8 qubits, of both,
two and three groups, both gradient memories, one stream and several). (The
automatic gradient memory depends on the whole batch, so the largest name one.)"""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd import synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu


def _graph(n, seed):
    g = synth.erdos_renyi(n, 0.5, seed)
    return g.u, g.v, synth.random_weights(g.num_edges, seed, 1, 9)


def _run(sizes, edges, gamma, beta, **kw):
    bt = QaoaBatch(sizes, edges, max_p=3, max_k=1, gradient=True, **kw)
    bt.apply_layers(gamma, beta)
    states = [bt.reduced_state(b).clone() for b in range(len(sizes))]
    E = bt.expectation().clone()
    return states, [E] + list(bt.expectation_grad(gamma, beta))


@pytest.mark.parametrize("sizes,kw", [([14, 16, 15], {}), ([17, 20, 19], {}), ([20, 14, 17, 16, 18], {}),
                                      ([18, 14, 20], dict(gradient_memory="inplace")),
                                      ([16, 9, 17], dict(concurrent_classes=True)), ([22, 21, 23], dict(gradient_memory="checkpoints"))])
def test_a_subgraph_does_not_depend_on_the_others(sizes, kw):
    edges = [_graph(n, 50 + b) for b, n in enumerate(sizes)]
    gamma, beta = synth.uniform_angles(8, 3, batch=len(sizes))
    gamma, beta = np.asarray(gamma).reshape(len(sizes), 3), np.asarray(beta).reshape(len(sizes), 3)
    states, sums = _run(sizes, edges, gamma, beta, **kw)
    for b, n in enumerate(sizes):
        alone, own = _run([n], [edges[b]], gamma[b:b + 1], beta[b:b + 1], **kw)
        assert torch.equal(torch.view_as_real(states[b]), torch.view_as_real(alone[0])), n
        for x, y in zip(sums, own):
            assert torch.equal(x[b].reshape(-1), y.reshape(-1)), n
