"""The Cholesky factor of K_MM over the whole range of its diagonal, subnormal pivots included."""
import numpy as np
import pytest

from tests.gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,low,high", [(1, -520, -520), (20, -530, -512), (70, -535, 0), (130, -515, 500), (200, -537, 500)])
def test_cholesky_of_scaled_points(M, low, high):
    """Descriptors of M / 2 independent pairs of points (one of a pair along a unit vector, the other
    with a part across) of lengths 2^low .. 2^high, zeta = 1, no jitter: K_MM holds exact
    numbers, in 2 x 2 blocks 4^k [[1, 1], [1, 5]], whose factor is 2^k [[1, 1], [0, 2]], exact."""
    import torch

    from paper_2207_03803_amd import gap

    pairs = (M + 1) // 2
    k = np.round(np.linspace(low, high, pairs)).astype(int)
    XM = np.zeros((M, 2 * pairs))
    expect = np.zeros((M, M))
    for i in range(pairs):
        s = 2.0 ** int(k[i])
        XM[2 * i, 2 * i] = s
        expect[2 * i, 2 * i] = s
        if 2 * i + 1 < M:
            XM[2 * i + 1, 2 * i:2 * i + 2] = s, 2 * s
            expect[2 * i, 2 * i + 1], expect[2 * i + 1, 2 * i + 1] = s, 2 * s
    X = np.zeros((2, 2 * pairs))
    X[:, 0] = 1.0
    h = gap.Handle(gap.params(2 * pairs, 1, 1.0, 0.0))
    h.alloc_workspace(2, 2, M)
    keep = [to_dev(X), to_dev(np.arange(3)), to_dev(XM), to_dev(np.ones(2))]
    h.build_knm(keep[0], keep[1], keep[2], keep[3])
    assert h.sync()[0] == gap.GAP_OK
    A, _ = h.A_view()
    U = A[:M, 2:2 + M].T.cpu().numpy()
    h.close()
    assert np.array_equal(np.triu(U), expect)
    torch.cuda.synchronize()
