"""The panels' reflectors over the whole range of condition numbers: the Cholesky QR passes solve
with explicit inverses of 16 x 16 blocks, which is safe only while the passes before have done
their part."""
import numpy as np
import pytest

from tests.gpu_helpers import GpuFit, U

pytestmark = pytest.mark.gpu


def _reflectors(X, sigma, seed):
    """[X / sigma; I] from one-atom configurations against unit sparse points, and the Q and R that
    its fit leaves (None where it is refused as rank deficient)."""
    from paper_2207_03803_amd import gap

    N, M = X.shape
    y = np.random.default_rng(seed).standard_normal(N) * sigma
    g = GpuFit(X, np.arange(N + 1), np.eye(M), np.full(N, sigma), y, 1, jitter=0.0)
    g.build()
    A = np.vstack(g.A_top_and_lower())
    try:
        _, info = g.solve()
    except gap.GapError as e:
        assert e.status == gap.GAP_ERANK
        return A, None, None
    assert info.device_status == 0
    m = N + M
    F = g.h.A_view()[0][:M, :m].T.cpu().numpy()
    tau = g.h.tau_view().cpu().numpy()
    g.h.close()
    Q = np.eye(m, M)
    for j in reversed(range(M)):
        v = np.concatenate([[1.0], F[j + 1:, j]])
        Q[j:] -= tau[j] * np.outer(v, v @ Q[j:])
    return A, Q, np.triu(F[:M])


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("kappa", [1.0, 1e4, 1e7, 1e8, 1e10, 1e12, 1e14])
@pytest.mark.parametrize("N,M", [(300, 20), (500, 64), (3000, 64), (700, 130)])
def test_reflectors_of_ill_conditioned_matrices(N, M, kappa, graded):
    """[X / sigma; I] with singular values of X from 1 to 1 / kappa (graded: or columns of such
    lengths), from one-atom configurations against unit sparse points. Householder QR forms a
    Q with ||Q^T Q - I||_F <= m n u and A + dA = Q R with ||dA||_F <= m n u ||A||_F up to a
    small factor (Higham 2002, Theorem 19.4; 4 here): the reconstruction has to as well, whatever kappa.
    A panel of w columns may be refused (GAP_ERANK) only where the shifted first pass cannot bring it
    within reach of the second: its factor is ||P|| sqrt(11 (m w + w (w + 1)) u) at least, and what the
    pass leaves has kappa sqrt(11 (m w + w (w + 1)) u), which Cholesky QR takes up to about u^-1/2 / 8."""
    rng = np.random.default_rng(M + N)
    s = np.geomspace(1.0, 1.0 / kappa, M)
    X = np.linalg.qr(rng.standard_normal((N, M)))[0] * s
    if not graded:
        X = X @ np.linalg.qr(rng.standard_normal((M, M)))[0].T
    sigma = 0.1 / kappa
    A, Q, R = _reflectors(X, sigma, N)
    m, w = N + M, min(M, 64)
    if Q is None:
        assert kappa * np.sqrt(11 * (m * w + w * (w + 1))) * U > 1 / 8
        return
    orth = np.linalg.norm(Q.T @ Q - np.eye(M))
    back = np.linalg.norm(A - Q @ R) / np.linalg.norm(A)
    print(f"N {N} M {M} kappa {kappa:.0e} graded {graded}: orthogonality {orth / U:.1f} u, backward error {back / U:.1f} u",
          flush=True)
    assert orth <= 4 * m * M * U and back <= 4 * m * M * U


@pytest.mark.parametrize("M,c", [(16, 0.6), (16, 0.9), (20, 0.8), (32, 0.3), (32, 0.6)])
def test_reflectors_of_kahan_matrices(M, c):
    """Q K for Kahan's K = diag(s^i) (I - c strictly upper ones), s^2 + c^2 = 1, whose ill-conditioning
    no column scaling takes away (condition 6e4 to 6e9 here): column by column, M rounded steps leave
    about sqrt(M) u of the column; 2 sqrt(M) u."""
    s = np.sqrt(1 - c * c)
    K = np.diag(s ** np.arange(M)) @ (np.eye(M) - c * np.triu(np.ones((M, M)), 1))
    rng = np.random.default_rng(M)
    X = np.linalg.qr(rng.standard_normal((400, M)))[0] @ K
    A, Q, R = _reflectors(X, np.linalg.svd(K, compute_uv=False)[-1] / 10, 1)
    err = (np.linalg.norm(A - Q @ R, axis=0) / np.linalg.norm(A, axis=0)).max()
    print(f"M {M} c {c}: {err / U:.1f} u", flush=True)
    assert err <= 2 * np.sqrt(M) * U
