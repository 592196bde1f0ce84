"""Wide tiles (2^14 amplitudes): every strided group size they are used with
(7..12 qubits), both cut-table widths, layers of both parities and angles that
flip (|sin beta| > |cos beta|), against the FP64 oracle with the tolerances of
test_gpu_sim.py; the same batches on 4096-amplitude tiles (forced by naming a
group split) are the general path."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_26232_amd import _abi, autotune, synth
from paper_2603_26232_amd.batch import QaoaBatch, idx_to_uint32

AMP_TOL, L2_TOL, E_TOL, G_TOL = 1e-5, 1e-5, 1e-5, 1e-4


def _edges(n, B, seed, heavy=False, sparse=False):
    out = []
    for b in range(B):
        g = synth.erdos_renyi(n, 0.5 if heavy else 0.06, seed + b)
        keep = slice(0, (3 * n) // 2) if sparse else slice(None)
        w = synth.random_weights(g.num_edges, seed + 40 + b, 3, 9) if heavy else g.w
        out.append((g.u[keep], g.v[keep], w[keep]))
    return out


def _batch(sizes, edges, narrow=False, **kw):
    tiled = [n for n in set(sizes) if n > 13]
    try:
        if narrow:
            for n in tiled:
                _abi.qaoa_tune_group_split(n, autotune.default_split(n))
        return QaoaBatch(sizes, edges, **kw)
    finally:
        for n in tiled:
            _abi.qaoa_tune_group_split(n, None)


def test_rule_for_wide_tiles():
    """The choice shows in the checkpoint slots, p (G - 1) states: two groups
    on wide tiles, three on the others (21..26 qubits)."""
    from paper_2603_26232_amd.partition import batch_arrays

    def slots(n, B, edges, flags=0x1 | 0x80):
        nq, off, u, v, w = batch_arrays([n] * B, edges)
        size = lambda p: _abi.qaoa_workspace_bytes(B, nq, off, w, p, 1, flags)
        return (size(3) - size(2)) // (B * 8 << (n - 1))

    for n, B, sparse, groups in [(20, 4, True, 2), (21, 1, True, 3), (21, 2, True, 2), (24, 1, True, 2),
                                 (25, 1, True, 2), (26, 2, True, 3), (27, 1, True, 3), (29, 1, True, 3),
                                 (24, 1, False, 3)]:
        assert slots(n, B, _edges(n, B, 5, heavy=not sparse, sparse=sparse)) == groups - 1, (n, B, sparse)
    # a named split keeps the 4096-amplitude tiles
    _abi.qaoa_tune_group_split(24, [6, 6])
    try:
        assert slots(24, 1, _edges(24, 1, 5, sparse=True)) == 2
    finally:
        _abi.qaoa_tune_group_split(24, None)


@pytest.mark.gpu
@pytest.mark.parametrize("sizes,p,heavy", [([21, 21], 1, False), ([21, 21, 14, 9], 2, True), ([22], 3, True),
                                           ([23, 22], 4, False), ([24], 2, True), ([25], 1, False),
                                           ([26, 26], 2, False)])
def test_states(sizes, p, heavy):
    edges = [_edges(n, 1, 60 + 7 * i, heavy=heavy)[0] for i, n in enumerate(sizes)]
    gamma, beta = synth.uniform_angles(500 + p, p, batch=len(sizes))
    assert len(sizes) < 2 or p == 1 or (np.abs(np.sin(beta)) > np.abs(np.cos(beta))).any()
    bt = _batch(sizes, edges, max_p=p, max_k=8)
    bt.apply_layers(gamma, beta)
    E = bt.expectation().cpu().numpy()
    idx, prob = bt.topk(8)
    narrow = _batch(sizes, edges, narrow=True, max_p=p, max_k=8)
    narrow.apply_layers(gamma, beta)
    for b in range(len(sizes) if max(sizes) < 26 else 1):
        u, v, w = edges[b]
        C = oracle.cut_table(sizes[b], u, v, w)
        ref = oracle.qaoa_state(sizes[b], C, gamma[b], beta[b])
        got = bt.state(b).cpu().numpy()
        err = np.abs(got - ref)
        assert err.max() <= AMP_TOL and np.sqrt((err ** 2).sum()) <= L2_TOL
        e_ref = oracle.expectation(sizes[b], ref, C)
        assert abs(E[b] - e_ref) <= E_TOL * max(1.0, abs(e_ref))
        # the two tile widths differ by rounding alone: twice the oracle bound
        assert np.abs(got - narrow.state(b).cpu().numpy()).max() <= 2 * AMP_TOL
        pr = np.abs(ref) ** 2
        assert np.all(np.abs(pr[idx_to_uint32(idx[b])] - prob[b].cpu().numpy()) <= 4 * AMP_TOL)
    bt.close()
    narrow.close()


@pytest.mark.gpu
@pytest.mark.parametrize("memory", ["checkpoints", "inplace"])
@pytest.mark.parametrize("sizes,p", [([21, 21], 1), ([22, 12], 2), ([23], 3), ([24], 1), ([25], 2)])
def test_gradient(sizes, p, memory):
    edges = [_edges(n, 1, 80 + 5 * i, sparse=True)[0] for i, n in enumerate(sizes)]
    gamma, beta = synth.uniform_angles(700 + p, p, batch=len(sizes))
    bt = _batch(sizes, edges, max_p=max(p, 2), max_k=4, gradient=True, gradient_memory=memory)  # (one layer: no wide tiles)
    E, dg, db = (t.cpu().numpy() for t in bt.expectation_grad(gamma, beta))
    again = [t.cpu().numpy() for t in bt.expectation_grad(gamma, beta)]
    assert np.array_equal(E, again[0]) and np.array_equal(dg, again[1]) and np.array_equal(db, again[2])
    for b, n in enumerate(sizes):
        u, v, w = edges[b]
        e_ref, g_ref, b_ref = oracle.gradient(n, oracle.cut_table(n, u, v, w), gamma[b], beta[b])
        scale = max(1.0, float(np.abs(np.concatenate([g_ref, b_ref])).max()))
        assert abs(E[b] - e_ref) <= E_TOL * max(1.0, abs(e_ref))
        assert np.abs(dg[b] - g_ref).max() <= G_TOL * scale
        assert np.abs(db[b] - b_ref).max() <= G_TOL * scale
    bt.close()


@pytest.mark.gpu
def test_gradient_29_qubits_matches_the_p1_closed_form():
    """Three wide groups (8 and 7 strided qubits) with single backward passes:
    on a ring of m unit edges without triangles, p = 1, every edge has
    <C_uv> = 1/2 + (1/4) sin 4b sin g (2 cos g) (Wang et al., PRA 97, 022304);
    the other vertices are free."""
    n, m = 29, 10
    u = np.arange(m, dtype=np.int32)
    v = ((u + 1) % m).astype(np.int32)
    g, b = 0.7, 0.3
    bt = QaoaBatch([n], [(u, v, np.ones(m, np.int32))], max_p=2, max_k=1, gradient=True)
    E, dg, db = (float(t.reshape(-1)[0]) for t in bt.expectation_grad(np.array([[g]]), np.array([[b]])))
    s4, c4 = np.sin(4 * b), np.cos(4 * b)
    assert abs(E - m * (0.5 + 0.5 * s4 * np.sin(g) * np.cos(g))) <= E_TOL * m
    assert abs(dg - m * 0.5 * s4 * np.cos(2 * g)) <= G_TOL * m
    assert abs(db - m * 2.0 * c4 * np.sin(g) * np.cos(g)) <= G_TOL * m
    bt.close()
