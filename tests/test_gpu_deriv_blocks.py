"""Derivative rows at every width of their column blocks (32, 64, 96, 128 and 256 columns), chosen by the
sparse points and by the room there is, with ragged last blocks, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import U, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,M,n_obs,n_grad", [
    # by the sparse points: 96 columns for M of 49 .. 64, ragged
    (16, 49, 60, 700), (7, 60, 60, 700), (16, 64, 60, 700),
    # by the room, several blocks with M = 200: 96 + 96 + 8 columns, 3 x 64 + 8, 6 x 32 + 8, position tiles
    (6, 200, 2000, 95_000), (5, 200, 2000, 120_000), (5, 200, 2000, 200_000), (4, 200, 2000, 400_000),
])
def test_derivative_rows_in_blocks_of_every_width(d, M, n_obs, n_grad):
    """Error bound: two dot products of d terms, the power and a sum over the positions, every
    operation rounded once on each side: 2 ((zeta + 1) (d + 2) + positions) u of the sum of the
    absolute terms."""
    import torch

    from paper_2207_03803_amd import gap

    zeta = 3
    rng = np.random.default_rng(n_grad + M)
    counts = np.array([9, 30, 1, 24])
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(offsets[-1])
    X = np.abs(rng.standard_normal((n, d)))
    X /= np.sqrt((X * X).sum(axis=1))[:, None]
    XM = np.abs(rng.standard_normal((M, d))) / np.sqrt(d)
    # uneven observations over at least as many positions as there are gradient rows
    lengths = rng.integers(0, 2 * (n_grad // n_obs) + 2, n_obs)
    lengths[[0, n_obs // 2]] = 0, 700
    lengths[-1] += max(0, n_grad + 5 - int(lengths.sum()))
    n_pos = int(lengths.sum())
    x_grad = rng.standard_normal((n_grad, d)) * 0.1
    grad_atom = rng.integers(0, n, n_grad)
    obs_offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    pos_grad = rng.integers(0, n_grad, n_pos)
    pos_weight = rng.standard_normal(n_pos)
    sigma = rng.uniform(0.5, 2.0, len(counts) + n_obs)
    h = gap.Handle(gap.params(d, zeta, 0.9, 1.0))
    h.alloc_workspace_obs(len(counts), n, n_obs, n_pos, M)
    obs = dict(x_grad=to_dev(x_grad), grad_atom=to_dev(grad_atom), obs_offsets=to_dev(obs_offsets),
               pos_grad=to_dev(pos_grad), pos_weight=to_dev(pos_weight))
    inputs = [to_dev(X), to_dev(offsets), to_dev(XM), to_dev(sigma)]
    h.build_knm_obs(inputs[0], inputs[1], obs, inputs[2], inputs[3])
    torch.cuda.synchronize()
    assert h.sync()[0] == gap.GAP_OK
    A, _ = h.A_view()
    NE = len(counts)
    got = A[:M, NE:NE + n_obs].T.cpu().numpy() * sigma[NE:, None]
    orc = oracle.Oracle()
    args = (grad_atom.astype(np.int64), obs_offsets, pos_grad.astype(np.int64))
    expect = orc.kdm(X, x_grad, *args, pos_weight, XM, zeta, 0.9)
    scale = orc.kdm(X, np.abs(x_grad), *args, np.abs(pos_weight), XM, zeta, 0.9)
    bound = 2 * ((zeta + 1) * (d + 2) + lengths[:, None]) * U * scale
    assert np.all(np.abs(got - expect) <= bound)
    assert np.all(got[lengths == 0] == 0.0)
    h.close()
