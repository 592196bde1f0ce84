"""The work that a user of this framework has it do, as cases that can be timed:
forward evaluations, gradients, angle optimisation, top-k, merge, cut
evaluation, predictor training and whole solves, each through the package's
public entry points, from one 12-qubit subgraph to a 30-qubit state.

Energies, gradients and angles come out of the library in FP64 containers, but
they are sums over complex64 amplitudes; `run` hands them on in float32, the
precision they carry (as the predictor's training set does with the angles).
The predictor's own parameters and gradients stay FP64. `exact` computes every
floating output in 64 bits with plain torch.

Where a case returns top-k strings its graphs are connected and weighted, so
that no two strings have equal probabilities by a symmetry of the graph: the
order of such strings is defined by no result of the method.
"""
import math

import numpy as np
import torch

from paper_2603_26232_amd import _abi, synth
from paper_2603_26232_amd.batch import QaoaBatch
from paper_2603_26232_amd.learned import DEFAULT_MODEL, AnglePredictor, LearnedStart
from paper_2603_26232_amd.partition import bucket_edges, partition_chain
from paper_2603_26232_amd.solve import SolveConfig, Solver, cold_start, maxcut_eval, merge_beam

DEV = "cuda"
MAX_WEIGHT_SUM = 2047  # of one subgraph (the library's limit)


def listed():
    return [
        # one 12-vertex graph, the parity size: the smallest call, all latency
        dict(name="eval_12", kind="eval", B=1, lo=12, hi=12, p=2, edge=0.5, weighted=True, k=8, mixer="valu"),
        # the ensemble of 26-qubit 3-regular graphs of the precision sweep, four at a time
        dict(name="eval_26", kind="eval", B=4, lo=26, hi=26, p=4, edge=3.0, weighted=False, k=0, mixer="valu"),
        # the largest single state the library takes
        dict(name="eval_30", kind="eval", B=1, lo=30, hi=30, p=2, edge=3.0, weighted=False, k=0, mixer="valu"),
        # one gradient of a dense weighted 24-vertex graph: 2-byte cut tables, one state at a time
        dict(name="grad_24", kind="grad", B=1, lo=24, hi=24, p=3, edge=0.5, weighted=True, memory="auto"),
        # angle optimisation of a graph cut into subgraphs of at most 13 vertices, the whole-state kernel's range
        dict(name="opt_small", kind="opt", nV=360, lo=9, hi=13, p=3, edge=0.3, iters=20, concurrent=False),
        # angle optimisation of 400 vertices in subgraphs of 20, sparse: the states fit the last-level cache
        dict(name="opt_400", kind="opt", nV=400, lo=20, hi=20, p=3, edge=0.05, iters=10, concurrent=False),
        # two optimiser steps of the 2000-vertex graph in ragged subgraphs of 14..26 vertices
        dict(name="opt_2000", kind="opt", nV=2000, lo=14, hi=26, p=3, edge=0.01, iters=2, concurrent=True),
        # candidate extraction from evaluated states of 20..26 qubits
        dict(name="topk_26", kind="topk", B=4, lo=20, hi=26, p=2, edge=0.4, k=16, raw=False),
        # the beam merge of a 2000-vertex solve
        dict(name="merge_2000", kind="merge", nV=2000, lo=14, hi=26, edge=0.01, K=16, W=4096),
        # cut values of a pool of assignments of a 2000-vertex graph
        dict(name="cut_2000", kind="cut", nV=2000, edge=0.01, weighted=False, A=1024),
        # one training step of the angle predictor on the warm-start set (10 graphs, 87 subgraphs each)
        dict(name="mlp_870", kind="mlp", batch=870, inputs=18, hidden=128, out=6),
        # a whole solve of a small dense weighted graph: rebuild, optimise, top-k, merge, cut value
        dict(name="solve_90", kind="solve", nV=90, lo=14, hi=16, p=3, edge=0.5, iters=10, k=8, beam=256,
             learned=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "grad", "grad", "opt", "opt", "topk", "merge", "cut", "mlp", "solve"])
    if kind in ("eval", "grad"):
        # total stored amplitudes between one small state and a quarter of the largest case
        hi = rng.randint(3, 27 if kind == "eval" else 26)
        lo = max(2, hi - rng.choice([0, 1, 3, 6]))
        B = _log_int(rng, 1, max(1, min(64, 2 ** (28 - hi))))
        c = dict(kind=kind, B=B, lo=lo, hi=hi, p=rng.randint(1, 6 if hi < 24 else 4),
                 edge=round(rng.uniform(0.1, 0.8), 3), weighted=rng.random() < 0.5)
        if kind == "eval":
            c.update(k=0, mixer=rng.choice(["valu", "valu", "valu", "mfma_f32", "mfma_bf16x4"]))
        else:
            c.update(memory=rng.choice(["auto", "auto", "checkpoints", "inplace"]))
        return c
    if kind == "opt":
        hi = rng.randint(4, 24)
        lo = max(3, hi - rng.randint(0, 8))
        nV = hi + _log_int(rng, 4, 400 if hi <= 22 else 150)
        return dict(kind=kind, nV=nV, lo=lo, hi=hi, p=rng.randint(1, 4), edge=round(rng.uniform(0.02, 0.5), 3),
                    iters=rng.randint(1, 6 if hi > 20 else 12), concurrent=rng.random() < 0.5)
    if kind == "topk":
        hi = rng.randint(10, 26)
        return dict(kind=kind, B=rng.randint(1, 6 if hi < 25 else 3), lo=max(10, hi - rng.randint(0, 6)), hi=hi,
                    p=rng.randint(1, 3), edge=round(rng.uniform(0.35, 0.6), 3), k=_log_int(rng, 1, 24),
                    raw=rng.random() < 0.2)
    if kind == "merge":
        hi = rng.randint(4, 26)
        return dict(kind=kind, nV=_log_int(rng, 30, 4000), lo=max(3, hi - rng.randint(0, 12)), hi=hi,
                    edge=round(math.exp(rng.uniform(math.log(0.003), math.log(0.1))), 4), K=_log_int(rng, 1, 64),
                    W=_log_int(rng, 1, 8192))
    if kind == "cut":
        return dict(kind=kind, nV=_log_int(rng, 30, 16000),
                    edge=round(math.exp(rng.uniform(math.log(0.001), math.log(0.05))), 4),
                    weighted=rng.random() < 0.5, A=_log_int(rng, 1, 4096))
    if kind == "mlp":
        return dict(kind=kind, batch=_log_int(rng, 8, 4000), inputs=rng.randint(4, 64),
                    hidden=_log_int(rng, 16, 256), out=2 * rng.randint(1, 6))
    hi = rng.randint(14, 18)
    return dict(kind="solve", nV=hi + rng.randint(20, 90), lo=max(12, hi - rng.randint(0, 3)), hi=hi, p=3,
                edge=round(rng.uniform(0.4, 0.6), 3), iters=rng.randint(1, 10), k=rng.randint(2, 8),
                beam=_log_int(rng, 16, 1024), learned=rng.random() < 0.4)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _pairs(nV, edge, rng):
    """Distinct vertex pairs u < v, edge * nV (nV - 1) / 2 of them, sorted."""
    total = nV * (nV - 1) // 2
    m = min(total, max(1, int(round(edge * total))))
    if total <= 1 << 20:
        iu, iv = np.triu_indices(nV, 1)
        sel = np.sort(rng.choice(total, m, replace=False))
        return iu[sel], iv[sel]
    key = np.zeros(0, np.int64)
    while key.size < m:
        a, b = rng.integers(0, nV, 2 * m), rng.integers(0, nV, 2 * m)
        key = np.unique(np.concatenate([key, (np.minimum(a, b) * nV + np.maximum(a, b))[a != b]]))
    key = np.sort(rng.choice(key, m, replace=False))
    return key // nV, key % nV


def _subgraph(n, edge, weighted, connected, rng):
    """Local edge list: 3-regular for edge = 3, else G(n, m); a path through
    all vertices is added where connected."""
    if edge == 3.0:
        g = synth.random_regular3(n, int(rng.integers(1 << 30)))
        u, v = g.u, g.v
    else:
        u, v = _pairs(n, edge, rng)
    if connected:
        perm = rng.permutation(n)
        a, b = np.concatenate([u, perm[:-1]]), np.concatenate([v, perm[1:]])
        key = np.unique(np.minimum(a, b) * n + np.maximum(a, b))
        u, v = key // n, key % n
    hi = min(9, max(1, MAX_WEIGHT_SUM // max(1, len(u))))
    w = rng.integers(1, hi + 1, len(u)) if weighted else np.ones(len(u))
    return u.astype(np.int32), v.astype(np.int32), w.astype(np.int32)


def _batch_inputs(case, seed):
    rng = np.random.default_rng([seed, 1])
    sizes = synth.ragged_sizes(1, case["lo"], case["hi"], case["B"])  # the same for every seed
    sizes[0] = case["hi"]
    strings = case["kind"] == "topk" or case.get("k", 0) > 0
    edges = [_subgraph(int(n), case["edge"], case.get("weighted", True), strings, rng) for n in sizes]
    gamma = rng.uniform(0.0, math.pi, (case["B"], case["p"]))
    beta = rng.uniform(0.0, math.pi, (case["B"], case["p"]))
    return [int(n) for n in sizes], edges, gamma, beta


def _graph(case, seed):
    """A whole graph and its chain partition."""
    rng = np.random.default_rng([seed, 2])
    nV = case["nV"]
    u, v = _pairs(nV, case["edge"], rng)
    w = None
    if case["kind"] == "solve":
        u, v = np.concatenate([u, np.arange(nV - 1)]), np.concatenate([v, np.arange(1, nV)])
        key = np.unique(u * nV + v)  # with the path 0, 1, 2, ...: every range is connected
        u, v = key // nV, key % nV
        w = rng.integers(1, 10, len(u))
    sizes = synth.ragged_sizes(1, case["lo"], case["hi"], nV)  # the same for every seed
    return synth.Graph(nV, u, v, w), partition_chain(nV, sizes)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("eval", "grad", "topk"):
        sizes, edges, gamma, beta = _batch_inputs(case, seed)
        bt = QaoaBatch(sizes, edges, max_p=case["p"], max_k=max(1, case.get("k", 0)), gradient=kind == "grad",
                       raw_topk=case.get("raw", False), mixer=case.get("mixer", "valu"),
                       gradient_memory=case.get("memory", "auto"))
        st = dict(case=case, batch=bt, gamma=torch.as_tensor(gamma, device=DEV),
                  beta=torch.as_tensor(beta, device=DEV))
        if kind == "topk":
            bt.apply_layers(st["gamma"], st["beta"])
        return st
    if kind in ("opt", "solve"):
        g, part = _graph(case, seed)
        opt = kind == "opt"
        cfg = SolveConfig(p=case["p"], iters=case["iters"], k=16 if opt else case["k"],
                          beam=64 if opt else case["beam"])
        S = Solver(g, part, cfg, skip_edgeless=True, concurrent_classes=case.get("concurrent", False))
        st = dict(case=case, solver=S, start=cold_start(cfg.p, S.B))
        if case.get("learned"):
            st["learned"] = LearnedStart(S, AnglePredictor.from_file(DEFAULT_MODEL))
        return st
    if kind == "merge":
        g, part = _graph(case, seed)
        rng = np.random.default_rng([seed, 3])
        K = case["K"]
        cand = np.full((part.M, K), 0xFFFFFFFF, dtype=np.uint32)
        for i, n in enumerate(part.size):
            pool = 1 << (int(n) - 1)
            pick = rng.choice(pool, min(K, pool), replace=False)
            cand[i, :len(pick)] = 2 * pick
        return dict(case=case, graph=g, part=part, cand=torch.as_tensor(cand.view(np.int32), device=DEV))
    if kind == "cut":
        rng = np.random.default_rng([seed, 4])
        u, v = _pairs(case["nV"], case["edge"], rng)
        w = rng.integers(1, 10, len(u)) if case["weighted"] else np.ones(len(u))
        dev = tuple(torch.as_tensor(np.asarray(x, np.int32), device=DEV) for x in (u, v, w))
        gen = torch.Generator(device=DEV).manual_seed(seed)
        nw = (case["nV"] + 31) // 32
        x = torch.randint(-2 ** 31, 2 ** 31, (case["A"], nw), generator=gen, device=DEV).to(torch.int32)
        return dict(case=case, edges=dev, assign=x)
    X, T, params = _mlp_inputs(case, seed)
    dims = (case["inputs"], case["hidden"], case["out"])
    st = dict(case=case, x=torch.as_tensor(X, device=DEV), t=torch.as_tensor(T, device=DEV),
              params=torch.as_tensor(params, device=DEV))
    st["y"] = torch.empty((case["batch"], case["out"]), dtype=torch.float32, device=DEV)
    st["act"] = torch.empty((case["batch"], 2 * case["hidden"]), dtype=torch.float32, device=DEV)
    st["grad"], st["m"], st["v"] = (torch.zeros_like(st["params"]) for _ in range(3))
    st["step"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    st["loss"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    st["scratch"] = torch.empty(_abi.qaoa_mlp_scratch_bytes(case["batch"], *dims), dtype=torch.uint8, device=DEV)
    return st


def _mlp_inputs(case, seed):
    """Standardised features and targets, He-initialised parameters."""
    rng = np.random.default_rng([seed, 5])
    i, h, o = case["inputs"], case["hidden"], case["out"]
    X = rng.normal(size=(case["batch"], i)).astype(np.float32)
    T = rng.normal(size=(case["batch"], o)).astype(np.float32)
    parts = []
    for a, b in ((i, h), (h, h), (h, o)):
        parts += [rng.normal(0.0, math.sqrt(2.0 / a), a * b), rng.normal(0.0, 0.1, b)]
    return X, T, np.concatenate(parts)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "eval":
        bt = st["batch"]
        bt.apply_layers(st["gamma"], st["beta"])
        out = {"E": bt.expectation().float()}
        if case["k"]:
            out["strings"], out["prob"] = bt.topk(case["k"])
        if case["hi"] > 13 and case["B"] <= 4:
            out["states"] = [bt.reduced_state(b) for b in range(case["B"])]
        return out
    if kind == "grad":
        E, dg, db = st["batch"].expectation_grad(st["gamma"], st["beta"])
        return {"E": E.float(), "dgamma": dg.float(), "dbeta": db.float()}
    if kind == "topk":
        idx, prob = st["batch"].topk(case["k"])
        return {"strings": idx, "prob": prob}
    if kind == "opt":
        S = st["solver"]
        S.set_angles(*st["start"])
        S.optimise(case["iters"])
        return {"theta": S.theta.float(), "E": S.E.float()}
    if kind == "solve":
        S = st["solver"]
        S.rebuild()
        if case["learned"]:
            S.run_learned(st["learned"], case["iters"])
        else:
            S.run()
        return {"cut": S.eval_cut, "assignment": S.best, "strings": S.idx, "prob": S.prob,
                "theta": S.theta.float(), "E": S.E.float()}
    if kind == "merge":
        best, cut, _ = merge_beam(st["graph"], st["part"], st["cand"], case["K"], case["W"])
        return {"assignment": best, "cut": cut}
    if kind == "cut":
        return {"cut": maxcut_eval(st["edges"], case["nV"], st["assign"])}
    b, dims = case["batch"], (case["inputs"], case["hidden"], case["out"])
    s = int(torch.cuda.current_stream().cuda_stream)
    ptr = {k: t.data_ptr() for k, t in st.items() if isinstance(t, torch.Tensor)}
    _abi.qaoa_mlp_forward(b, *dims, ptr["params"], ptr["x"], ptr["y"], ptr["act"], s)
    _abi.qaoa_mlp_backward(b, *dims, ptr["params"], ptr["x"], ptr["y"], ptr["act"], ptr["t"], ptr["scratch"],
                           st["scratch"].numel(), ptr["grad"], ptr["loss"], s)
    _abi.qaoa_adam_step(st["params"].numel(), ptr["params"], ptr["grad"], ptr["m"], ptr["v"], ptr["step"], 1e-3,
                        0.9, 0.999, 1e-8, 0, s)
    return {k: st[k] for k in ("y", "act", "grad", "loss", "params")}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _sizes(case):
    """Mean subgraph sizes."""
    if case["kind"] in ("eval", "grad", "topk"):
        mid = (case["lo"] + case["hi"]) / 2
        return [case["hi"]] + [mid] * (case["B"] - 1)
    mid = (case["lo"] + case["hi"]) / 2
    return [mid] * max(1, round((case["nV"] - 1) / max(1.0, mid - 1)))


def _amps(sizes, lo, hi):
    """Mean stored amplitudes of a subgraph with lo..hi qubits, times their number."""
    mean = sum(2.0 ** (n - 1) for n in range(lo, hi + 1)) / (hi - lo + 1)
    return mean * (len(sizes) - 1) + 2.0 ** (hi - 1)


def work(case):
    kind = case["kind"]
    if kind in ("eval", "grad", "topk", "opt"):
        s = _sizes(case)
        amps, n = _amps(s, case["lo"], case["hi"]), case["hi"]
        if kind == "topk":
            return {"bytes": 8.0 * amps, "flops": 3.0 * amps}
        # a rotation is two fused multiply-adds per stored amplitude and qubit, a phase six operations;
        # a gradient rotates three times as much and takes an inner product (two more) per qubit and layer
        flops = case["p"] * amps * (4.0 * n + 6.0)
        if kind == "eval":
            return {"bytes": 9.0 * amps, "flops": flops + (3.0 * amps if case["k"] else 0.0)}
        grad = 3.0 * flops + case["p"] * amps * 4.0 * (n + 1)
        if kind == "grad":
            return {"bytes": 9.0 * amps, "flops": grad}
        # edgeless subgraphs are not simulated
        share = 1.0 - (1.0 - case["edge"]) ** (n * (n - 1) / 2)
        return {"bytes": 9.0 * amps * share, "flops": grad * case["iters"] * share}
    if kind == "solve":
        s = _sizes(case)
        amps, n = _amps(s, case["lo"], case["hi"]), case["hi"]
        flops = case["p"] * amps * (4.0 * n + 6.0)
        return {"bytes": 17.0 * amps, "flops": flops * (3.7 * case["iters"] + 1.0)}
    nE = case.get("edge", 0.0) * case.get("nV", 0) * (case.get("nV", 0) - 1) / 2
    if kind == "merge":
        levels = len(_sizes(case))
        n = (case["lo"] + case["hi"]) / 2
        # per level: every path's row read and written once, every child's score
        return {"bytes": levels * case["W"] * case["nV"] / 8.0 + 12.0 * nE,
                "flops": case["W"] * (nE + levels * case["K"] * n)}
    if kind == "cut":
        return {"bytes": 12.0 * nE + case["A"] * (case["nV"] / 8.0 + 8.0), "flops": 2.0 * case["A"] * nE}
    i, h, o, b = case["inputs"], case["hidden"], case["out"], case["batch"]
    npar = h * (i + 1) + h * (h + 1) + o * (h + 1)
    return {"bytes": 4.0 * b * (i + 2 * o + 2 * h) + 8.0 * 8 * npar, "flops": 6.0 * b * npar}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _cut_table(n, edges):
    C = torch.zeros(1 << n, dtype=torch.int16, device=DEV)
    for u, v, w in zip(*(e.tolist() for e in edges)):
        a, b = max(u, v), min(u, v)
        x = C.view(1 << (n - 1 - a), 2, 1 << (a - 1 - b), 2, 1 << b)
        x[:, 0, :, 1] += w
        x[:, 1, :, 0] += w
    return C


def _mix(psi, n, beta):
    """prod_j e^{-i beta X_j}, at most five qubits at a time: the top ones by
    a dense product, the index then turned by as many bits."""
    one = torch.tensor([[math.cos(beta), -1j * math.sin(beta)], [-1j * math.sin(beta), math.cos(beta)]],
                       dtype=torch.complex128, device=DEV)
    left = n
    while left:
        k = min(5, left)
        M = torch.ones((1, 1), dtype=torch.complex128, device=DEV)
        for _ in range(k):
            M = torch.kron(M, one)
        psi = (M @ psi.view(1 << k, -1)).t().contiguous().view(-1)
        left -= k
    return psi


def _phase(C, gamma):
    t = -gamma * torch.arange(MAX_WEIGHT_SUM + 1, dtype=torch.float64, device=DEV)
    return torch.polar(torch.ones_like(t), t).index_select(0, C.to(torch.int32))


def _forward(n, C, gamma, beta):
    psi = torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.complex128, device=DEV)
    for g, b in zip(gamma, beta):
        psi = _mix(psi * _phase(C, g), n, b)
    return psi


def _energy(psi, C):
    return float(sum((x.real.square() + x.imag.square()).mul_(c).sum() for x, c in zip(psi.chunk(8), C.chunk(8))))


def _top_probabilities(psi, k, raw):
    """The k largest probabilities of the strings with bit 0 clear (raw: of all), -1 where there are fewer."""
    pi = psi.abs().square()
    pi = pi if raw else pi[::2]
    top = torch.topk(pi, min(k, pi.numel())).values
    return torch.cat([top, top.new_full((k - top.numel(),), -1.0)])


def _gradient(n, C, gamma, beta):
    """<C>, dE/dgamma and dE/dbeta by the adjoint sweep."""
    psi = _forward(n, C, gamma, beta)
    E = _energy(psi, C)
    lam = psi * C
    p = len(gamma)
    dg, db = np.zeros(p), np.zeros(p)
    for l in range(p - 1, -1, -1):
        x = torch.zeros_like(psi)
        for j in range(n):
            x += psi.view(-1, 2, 1 << j).flip(1).view(-1)
        db[l] = 2.0 * float(torch.vdot(lam, x).imag)
        psi, lam = _mix(psi, n, -beta[l]), _mix(lam, n, -beta[l])
        dg[l] = 2.0 * float(torch.vdot(lam, psi * C).imag)
        ph = _phase(C, -gamma[l])
        psi, lam = psi * ph, lam * ph
    return E, dg, db


def _optimise(subs, iters, lr, gamma, beta):
    """Adam ascent; <C> is that of the last step's starting angles."""
    B, p = gamma.shape
    E = np.zeros(B)
    for b, (n, edges) in enumerate(subs):
        if len(edges[0]) == 0:
            continue  # no gradient
        C = _cut_table(n, edges)
        th, m, v = np.concatenate([gamma[b], beta[b]]), np.zeros(2 * p), np.zeros(2 * p)
        for t in range(1, iters + 1):
            E[b], dg, db = _gradient(n, C, th[:p], th[p:])
            g = np.concatenate([dg, db])
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            th = th + lr * (m / (1 - 0.9 ** t)) / (np.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
        gamma[b], beta[b] = th[:p], th[p:]
    return gamma, beta, E


def exact(case, seed):
    kind = case["kind"]
    if kind in ("eval", "grad", "topk"):
        sizes, edges, gamma, beta = _batch_inputs(case, seed)
        tabs = ((n, _cut_table(n, e), g, b) for n, e, g, b in zip(sizes, edges, gamma, beta))
        if kind == "grad":
            r = [_gradient(*t) for t in tabs]
            return {"E": np.array([x[0] for x in r]), "dgamma": np.stack([x[1] for x in r]),
                    "dbeta": np.stack([x[2] for x in r])}
        out, E, prob, states = {}, [], [], []
        keep = kind == "eval" and case["hi"] > 13 and case["B"] <= 4
        for n, C, g, b in tabs:
            psi = _forward(n, C, g, b)
            E.append(_energy(psi, C))
            if case["k"]:
                prob.append(_top_probabilities(psi, case["k"], case.get("raw", False)))
            if keep:
                states.append(psi[:1 << (n - 1)] * math.sqrt(2.0))
            del psi
        if kind == "eval":
            out["E"] = np.array(E)
        if case["k"]:
            out.update(strings=None, prob=torch.stack(prob))
        if keep:
            out["states"] = states
        return out
    if kind == "opt":
        g, part = _graph(case, seed)
        subs = [(int(n), e) for n, e in zip(part.size, bucket_edges(part, g.u, g.v, g.w)[0])]
        live = sum(2.0 ** n for n, e in subs if len(e[0]))
        if case["iters"] * (live + 2.0 ** 22 * len(subs)) > 2.0 ** 32:
            return None
        G, B, E = _optimise(subs, case["iters"], 0.05, *(np.array(x) for x in cold_start(case["p"], part.M)))
        return {"theta": np.concatenate([G.reshape(-1), B.reshape(-1)]), "E": E}
    if kind != "mlp":
        return None  # whole numbers, or a solve that ends in them
    X, T, P = (torch.as_tensor(x, device=DEV).double() for x in _mlp_inputs(case, seed))
    i, h, o = case["inputs"], case["hidden"], case["out"]
    at, w = 0, []
    for a, b in ((i, h), (h, h), (h, o)):
        w += [P[at:at + a * b].view(b, a), P[at + a * b:at + a * b + b]]
        at += a * b + b
    h1 = torch.relu(X @ w[0].t() + w[1])
    h2 = torch.relu(h1 @ w[2].t() + w[3])
    y = h2 @ w[4].t() + w[5]
    d3 = 2.0 * (y - T) / y.numel()
    d2 = (d3 @ w[4]) * (h2 > 0)
    d1 = (d2 @ w[2]) * (h1 > 0)
    grad = torch.cat([t.reshape(-1) for t in (d1.t() @ X, d1.sum(0), d2.t() @ h1, d2.sum(0), d3.t() @ h2, d3.sum(0))])
    params = P - 1e-3 * grad / (grad.abs() + 1e-8)  # the first Adam step
    return {"y": y, "act": torch.cat([h1, h2], 1), "grad": grad, "loss": (y - T).square().mean().view(1),
            "params": params}
