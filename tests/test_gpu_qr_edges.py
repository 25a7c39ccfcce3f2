"""The QR at the edges of its panels' row splits (64 or 128 rows per workgroup, one or two
levels of sums) and of its tiles: R^T R against A^T A, and the coefficients."""
import numpy as np
import pytest

from paper_2207_03803_amd import synth
from tests.gpu_helpers import GpuFit, U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("rows,M", [
    (2, 1), (64, 16), (65, 17), (128, 63), (129, 64),
    (1023, 64), (1024, 65), (1025, 64),     # 64 rows per workgroup up to 1,024, then 128
    (2048, 130), (2049, 129),               # 16 workgroups of 128 rows, then two levels of sums
    (2176 + 64, 127), (16384, 64), (16385, 66),
])
def test_qr_at_the_edges_of_its_splits(rows, M, precision):
    """||R^T R - A^T A||_F <= 4 m n u ||A||_F^2: the factor of A + dA with ||dA||_F at most
    m n u ||A||_F (Householder QR) and both products in FP64.  c: that of the least-squares problem in 64 bits,
    within 32 u (kappa + kappa^2 ||r|| / (||A|| ||c||)), at most 1e-8 where refined."""
    N = rows - M
    inp = synth.make_fit_inputs(n_configs=N, atoms=(1, 3), d=16, M=M, seed=rows + M)
    rng = np.random.default_rng(rows)
    y = inp.sigma * rng.standard_normal(N)
    g = GpuFit(inp.X, inp.offsets, inp.XM, inp.sigma, y, 2, jitter=1.0, precision=precision, max_refine_iters=60)
    g.build()
    top, low = g.A_top_and_lower()
    A = np.vstack([top, low])
    b = np.concatenate([y / inp.sigma, np.zeros(M)])
    c, info = g.solve()
    assert info.device_status == 0
    ref, *_ = np.linalg.lstsq(A, b, rcond=None)
    sv = np.linalg.svd(A, compute_uv=False)
    kappa = sv[0] / sv[-1]
    bound = 32 * U * (kappa + kappa ** 2 * np.linalg.norm(b - A @ ref) / (sv[0] * np.linalg.norm(ref)))
    err = np.linalg.norm(c - ref) / np.linalg.norm(ref)
    print(f"rows {rows} M {M} precision {precision}: kappa {kappa:.1e}, c {err:.1e} (bound {bound:.1e})", flush=True)
    assert err <= (bound if precision == 0 else max(bound, 1e-8))
    if precision == 0:
        Av, _ = g.h.A_view()
        R = np.triu(Av[:M, :M].T.cpu().numpy())
        assert np.linalg.norm(R.T @ R - A.T @ A) <= 4 * rows * M * U * np.linalg.norm(A) ** 2
