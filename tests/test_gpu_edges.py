"""GPU: sizes at which a kernel changes the way it works (edges of tiles, of register-
resident runs, of the ranges of a launch rule), through the C ABI against the fp64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_progress import say as _say              # noqa: E402
from test_gpu_parity import _select_case          # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [63, 64, 65, 1023, 1025, 16383, 16384, 16385, 17408])
def test_select_around_the_register_resident_size(S):
    """Up to 16384 candidates are read once and kept in registers, 1024 candidates are one per
    thread; whole and partial batches of sixteen groups take different loops."""
    _say(f"select sizes S={S}")
    rng = np.random.default_rng(S)
    a = np.exp(rng.standard_normal((2, S)) * 2).astype(np.float32)
    b = (np.round(rng.random((2, S)) ** 4 * 64) / 64).astype(np.float32)      # ties and exact zeros
    for alpha in (0.3, 0.95, 0.9999):
        _select_case(a, b, alpha, alpha)
