"""CUR selection where the last columns are few (up to 32 past a multiple of 64 go with the
projection's tile before) and around that rule."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_cur import _select_and_check, _x

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [
    (700, 31), (700, 33), (1000, 65), (1000, 80), (1001, 81), (1000, 96), (1000, 97), (129, 128), (900, 144),
    (1500, 160), (1500, 161), (900, 193), (1300, 224), (127, 82),
])
def test_cur_last_columns(n, d):
    """Leverages and the selected rows against the oracle (within the reference test's bound)."""
    X = _x(n, d, 7 * d + n)
    draws = np.random.default_rng(d).standard_exponential(n)
    orc = oracle.Oracle()
    _select_and_check(orc, X, n // 5, draws, "sampled")
    _select_and_check(orc, X, n // 5, None, "top leverage")
