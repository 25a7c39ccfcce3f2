"""Derivative rows at the edges of their column blocks and of an observation's runs of
positions, through both ways of forming them, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import U, to_dev

pytestmark = pytest.mark.gpu

# positions per observation: none, the short loops' steps, one wave's batch, long observations
LENGTHS = [0, 1, 3, 4, 8, 13, 16, 17, 63, 64, 65, 0, 130, 257, 600, 2]


@pytest.mark.parametrize("d,M,zeta,spare", [
    (5, 1, 1, 0), (16, 33, 2, 0), (33, 100, 3, 0), (64, 300, 2, 0),
    (16, 33, 2, 2000), (33, 100, 3, 2000),    # more gradient rows than positions: the position tiles
])
def test_derivative_rows_of_uneven_observations(d, M, zeta, spare):
    """Error bound: two dot products of d terms, the power and a sum over the positions, every
    operation rounded once on each side: 2 ((zeta + 1) (d + 2) + positions) u of the sum of the
    absolute terms."""
    import torch

    from paper_2207_03803_amd import gap

    rng = np.random.default_rng(100 * d + M)
    counts = np.array([9, 30, 1, 24])
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(offsets[-1])
    X = np.abs(rng.standard_normal((n, d)))
    X /= np.sqrt((X * X).sum(axis=1))[:, None]
    XM = X[rng.integers(0, n, M)] if M < 64 else np.abs(rng.standard_normal((M, d))) / np.sqrt(d)
    n_pos = sum(LENGTHS)
    n_grad = n_pos + spare if spare else n_pos // 2
    x_grad = rng.standard_normal((n_grad, d)) * 0.1
    grad_atom = rng.integers(0, n, n_grad)
    obs_offsets = np.concatenate([[0], np.cumsum(LENGTHS)]).astype(np.int64)
    pos_grad = rng.integers(0, n_grad, n_pos)
    pos_weight = rng.standard_normal(n_pos)
    sigma = rng.uniform(0.5, 2.0, len(counts) + len(LENGTHS))
    h = gap.Handle(gap.params(d, zeta, 0.9, 1.0))
    h.alloc_workspace_obs(len(counts), n, len(LENGTHS), n_pos, M)
    obs = dict(x_grad=to_dev(x_grad), grad_atom=to_dev(grad_atom), obs_offsets=to_dev(obs_offsets),
               pos_grad=to_dev(pos_grad), pos_weight=to_dev(pos_weight))
    inputs = [to_dev(X), to_dev(offsets), to_dev(XM), to_dev(sigma)]
    h.build_knm_obs(inputs[0], inputs[1], obs, inputs[2], inputs[3])
    torch.cuda.synchronize()
    assert h.sync()[0] == gap.GAP_OK
    A, lay = h.A_view()
    NE, NO = len(counts), len(LENGTHS)
    got = A[:M, NE:NE + NO].T.cpu().numpy() * sigma[NE:, None]
    orc = oracle.Oracle()
    args = (grad_atom.astype(np.int64), obs_offsets, pos_grad.astype(np.int64))
    expect = orc.kdm(X, x_grad, *args, pos_weight, XM, zeta, 0.9)
    scale = orc.kdm(X, np.abs(x_grad), *args, np.abs(pos_weight), XM, zeta, 0.9)
    bound = 2 * ((zeta + 1) * (d + 2) + max(LENGTHS)) * U * scale
    assert np.all(np.abs(got - expect) <= bound)
    assert np.all(got[np.array(LENGTHS) == 0] == 0.0)
    h.close()
