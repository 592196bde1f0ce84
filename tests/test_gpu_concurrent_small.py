"""Concurrent classes: qaoa_optimize runs the small subgraphs' steps beside the tiled
ones, forked and joined once. The dependences show in the captured graph: the
small-subgraph kernel waits for nothing and only the step count's advance waits for it;
with a single class of tiled subgraphs the rest is one chain. Results are those of the
serial order, bit for bit, run directly and replayed with other work in between."""
import ctypes as ct
import os

import numpy as np
import pytest
import torch

from paper_2603_26232_amd import _abi, synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu


def _graph_edges(raw):
    """Nodes and (from, to) pairs of a hipGraph_t."""
    path = os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so")
    hip = ct.CDLL(path if os.path.exists(path) else "libamdhip64.so")
    g, n = ct.c_void_p(raw), ct.c_size_t(0)
    assert hip.hipGraphGetNodes(g, None, ct.byref(n)) == 0
    nodes = (ct.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(g, nodes, ct.byref(n)) == 0
    m = ct.c_size_t(0)
    assert hip.hipGraphGetEdges(g, None, None, ct.byref(m)) == 0
    a, b = (ct.c_void_p * m.value)(), (ct.c_void_p * m.value)()
    assert hip.hipGraphGetEdges(g, a, b, ct.byref(m)) == 0
    return list(nodes), list(zip(a, b))


class _Run:
    def __init__(self, sizes, iters, concurrent):
        self.p, self.B, self.iters = 3, len(sizes), iters
        edges = []
        for i, n in enumerate(sizes):
            g = synth.erdos_renyi(n, 0.4, 20 + i)
            edges.append((g.u, g.v, synth.random_weights(g.num_edges, 7 + i, 1, 9)))
        self.bt = QaoaBatch(sizes, edges, max_p=self.p, max_k=1, gradient=True, concurrent_classes=concurrent)
        gamma, beta = synth.uniform_angles(33, self.p, batch=self.B)
        self.start = torch.as_tensor(np.concatenate([gamma.reshape(-1), beta.reshape(-1)]), device="cuda")
        self.th, self.m, self.v = (torch.zeros_like(self.start) for _ in range(3))
        self.step = torch.zeros(1, dtype=torch.int32, device="cuda")
        self.E = torch.zeros(self.B, dtype=torch.float64, device="cuda")
        self.reset()

    def reset(self):
        self.th.copy_(self.start)
        for t in (self.m, self.v, self.step, self.E):
            t.zero_()

    def go(self):
        s = int(torch.cuda.current_stream().cuda_stream)
        _abi.qaoa_optimize(self.bt.handle, self.p, self.iters, self.th.data_ptr(), self.m.data_ptr(),
                           self.v.data_ptr(), self.step.data_ptr(), 0.05, 0.9, 0.999, 1e-8, self.E.data_ptr(), s)

    def results(self):
        torch.cuda.synchronize()
        return [t.clone() for t in (self.th, self.m, self.v, self.step, self.E, self.bt.expectation())]


# tiled subgraphs: one class; two and three group counts (other side streams in use)
@pytest.mark.parametrize("sizes", [[16, 9, 13, 5], [20, 22, 12, 7, 14], [24, 14, 22, 13]])
def test_small_subgraphs_run_beside_the_classes(sizes):
    serial, run = _Run(sizes, 4, False), _Run(sizes, 4, True)
    serial.go()
    ref = serial.results()
    run.go()
    for a, b in zip(ref, run.results()):
        assert torch.equal(a, b)
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        run.go()
    nodes, edges = _graph_edges(g.raw_cuda_graph())
    into, out = {n: [] for n in nodes}, {n: [] for n in nodes}
    for a, b in edges:
        out[a].append(b)
        into[b].append(a)
    roots = [n for n in nodes if not into[n]]
    last = [n for n in nodes if not out[n]]
    assert len(last) == 1  # the step count
    apart = [n for n in roots if out[n] == last]
    assert len(roots) == 2 and len(apart) == 1, (len(roots), len(apart))
    if max(sizes) == 16:  # one class: no forks within the steps
        assert all(len(into[n]) <= 1 for n in nodes if n != last[0])
        assert all(len(out[n]) <= 1 for n in nodes)
    for _ in range(3):
        run.reset()
        g.replay()
        torch.ones(1 << 20, device="cuda").sum()
        for a, b in zip(ref, run.results()):
            assert torch.equal(a, b)
    del g
    serial.bt.close()
    run.bt.close()
