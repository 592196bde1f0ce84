"""States on wide tiles keep their norm however the rotation's tangent rounds.

e^{-i beta X} runs as f (I - i t X) with t = tan(beta) rounded to FP32. With the
exact f = cos(beta) each of the n p rotations changes the norm squared by
2 t dt / (1 + t^2), dt the rounding of t, always in the same direction; with the f of
the rounded t by nothing. What is left per layer is the rounding of what is common to
all amplitudes, FP32 all of them: the factors of the two groups (f^14, f^(n-14), once
in the middle pass and, in the first and last pass, alone) and their product, at most
five roundings of 2^-24 of the norm squared (half an ulp each, twice in the square). The
amplitudes' own roundings are independent and average out over 2^20 of them."""
import numpy as np
import pytest

from paper_2603_26232_amd import synth
from paper_2603_26232_amd.batch import QaoaBatch

pytestmark = pytest.mark.gpu

P = 8


def _tangents():
    """Angles of both modes, |tan| and |cot| below 1, whose FP32 rounding moves the norm most, up and down."""
    b = np.linspace(0.55, 0.78, 20001)
    t = np.tan(b)
    move = (np.float32(t).astype(np.float64) - t) * 2 * t / (1 + t * t)
    return {"up": b[move.argmax()], "down": b[move.argmin()]}, float(np.abs(move).max())


@pytest.mark.parametrize("n", [21, 24, 26])
@pytest.mark.parametrize("which", ["up", "down"])
@pytest.mark.parametrize("flip", [False, True])
def test_norm(n, which, flip):
    betas, move = _tangents()
    tol = 5 * P * 2.0 ** -24
    assert n * P * move > 1.5 * tol  # the rounding of t would show
    beta = betas[which] + (np.pi / 2 if flip else 0.0)  # (flip: cot instead of tan)
    B = 2 if n == 21 else 1
    edges = []
    for b in range(B):
        g = synth.erdos_renyi(n, 0.1, 3 * n + b)
        edges.append((g.u, g.v, g.w))
    bt = QaoaBatch([n] * B, edges, max_p=P, max_k=1)
    gamma = np.random.default_rng(n).uniform(0.2, 3.0, (B, P))
    bt.apply_layers(gamma, np.full((B, P), beta))
    for b in range(B):
        s = bt.reduced_state(b)
        norm = float((s.real.double() ** 2).sum() + (s.imag.double() ** 2).sum())
        assert abs(norm - 1.0) <= tol, (n, norm - 1.0)
    bt.close()
