"""A tuning table's splits reach the subgraphs that run on 4096-amplitude tiles without
taking the wide tiles from the others: with the package's table applied, dense
gradients, matrix-core batches and a lone 21-qubit subgraph give the bits of the tuned
split, named, and sparse gradients and forward batches those of wide tiles."""
import numpy as np
import pytest
import torch

from paper_2603_26232_amd import _abi, autotune, synth
from paper_2603_26232_amd.batch import QaoaBatch
from paper_2603_26232_amd.partition import batch_arrays


def _edges(n, dense):
    g = synth.erdos_renyi(n, 0.4, 17 * n)
    m = 2 * n if dense else n
    pick = np.sort(np.random.default_rng(n).permutation(g.num_edges)[:m])
    return g.u[pick], g.v[pick], g.w[pick]


def _slots(n, dense, flags=0x1 | 0x80):
    """Checkpoints a layer: groups less one."""
    nq, off, u, v, w = batch_arrays([n], [_edges(n, dense)])
    size = lambda p: _abi.qaoa_workspace_bytes(1, nq, off, w, p, 1, flags)
    return (size(3) - size(2)) // (8 << (n - 1))


def test_a_narrow_split_leaves_the_choice_of_tiles():
    try:
        for n, split in ((22, [7, 3]), (24, [4, 8]), (30, [5, 6, 7])):
            wide, narrow = _slots(n, False), _slots(n, True)
            assert wide < narrow
            _abi.qaoa_tune_narrow_split(n, split)
            assert (_slots(n, False), _slots(n, True)) == (wide, narrow)
        for n, sizes, status in [(26, [7, 8], 1), (13, [1], 2), (31, [8, 8, 3], 2), (26, [9, 5], 2)]:
            with pytest.raises(_abi.QaoaError) as ei:
                _abi.qaoa_tune_narrow_split(n, sizes)
            assert ei.value.status == status
    finally:
        autotune.reset()


def test_the_tables_entries():
    """What an entry says was measured: its figures are those of timings it lists."""
    import json
    with open(autotune.DEFAULT_TABLE) as f:
        entries = json.load(f)["entries"]
    for n, e in entries.items():
        of = lambda kind: {tuple(r["split"] or ()): r["ms_per_mamp"] for r in e["all"] if r["graphs"] == kind}
        dense, sparse = of("dense"), of("sparse")
        assert sorted(map(list, dense)) == sorted(autotune.candidates(int(n)))
        assert e["ms_per_mamp_4096_tiles"] == dense[tuple(e["split_4096_tiles"])] == min(dense.values())
        assert e["default_ms_per_mamp"] == dense[tuple(autotune.default_split(int(n)))]
        assert e["ms_per_mamp"] == sparse[tuple(e["split"] or ())]
        if e["split"] is None and n != "26":
            assert sparse[()] <= sparse[tuple(e["split_4096_tiles"])]


def _outputs(n, dense, forward, mixer="valu"):
    gamma, beta = synth.uniform_angles(5, 2, batch=1)
    bt = QaoaBatch([n], [_edges(n, dense)], max_p=2, max_k=1, gradient=not forward, mixer=mixer)
    if forward:
        bt.apply_layers(gamma, beta)
        out = [torch.view_as_real(bt.reduced_state(0)).clone()]
    else:
        out = [t.clone() for t in bt.expectation_grad(gamma, beta)]
    bt.close()
    return out


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.gpu
@pytest.mark.parametrize("n,dense,forward,mixer", [(22, True, False, "valu"), (24, True, False, "valu"),
                                                   (21, False, False, "valu"), (22, True, True, "mfma_f32"),
                                                   (22, False, False, "valu"), (24, True, True, "valu")])
def test_the_table_applies_to_narrow_tiles_alone(n, dense, forward, mixer):
    own = _outputs(n, dense, forward, mixer)
    with_table, named = None, None
    try:
        autotune.apply(autotune.DEFAULT_TABLE)
        with_table = _outputs(n, dense, forward, mixer)
        autotune.reset()
        import json
        with open(autotune.DEFAULT_TABLE) as f:
            split = json.load(f)["entries"][str(n)]["split_4096_tiles"]
        assert split != autotune.default_split(n)
        _abi.qaoa_tune_group_split(n, split)
        named = _outputs(n, dense, forward, mixer)
    finally:
        autotune.reset()
    narrow = n == 21 or (dense and not forward) or mixer != "valu"
    assert _same(with_table, named) == narrow
    assert _same(with_table, own) == (not narrow)
