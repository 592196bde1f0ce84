"""Adam steps of one workgroup of 1024 threads and of several, at the edges, against
the FP64 oracle (test_gpu_mlp_sizes.py's check)."""
import pytest

from test_gpu_mlp_sizes import test_adam_step_counts as _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [258, 1023, 1024, 1025])
def test_adam(n):
    _check(n)
