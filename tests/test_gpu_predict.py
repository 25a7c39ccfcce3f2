"""Predictions at the edges of their tiles, and the K_NM at ragged descriptor lengths,
against the CPU oracle through the C ABI."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import U, log, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orc_m():
    return oracle.Oracle()


def _rows(n, d, rng):
    x = np.abs(rng.standard_normal((n, d)))
    return x / np.sqrt((x * x).sum(axis=1))[:, None]


def _predict(X, offsets, XM, c, zeta):
    import torch

    from paper_2207_03803_amd import gap

    h = gap.Handle(gap.params(X.shape[1], zeta))
    xm = to_dev(XM)
    h.set_model(xm)
    out = torch.empty(len(offsets) - 1, dtype=torch.float64, device="cuda")
    h.predict(to_dev(X), to_dev(offsets), to_dev(c), out)
    torch.cuda.synchronize()
    h.close()
    return out.cpu().numpy()


CASES = [
    # counts per configuration, d, M
    ([1], 8, 1),
    ([63], 7, 64),
    ([64], 33, 65),
    ([65, 0, 127], 16, 63),
    ([300], 64, 130),                       # one configuration over several tiles
    ([0, 255, 1, 0], 65, 257),              # empty first and last configurations
    ([256, 257, 1], 130, 40),
    ([37] * 333, 20, 300),
    ([40] * 1700, 9, 1100),                 # 256-atom tiles
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_predict_tile_edges(orc_m, case):
    """Error bound: a dot product of d terms, the power, and sums over the sparse points and
    the atoms, each term of each sum rounded once: (d + zeta + M + atoms) u of the sum of the
    absolute terms, for both sides."""
    counts, d, M = CASES[case]
    rng = np.random.default_rng(40 + case)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    X, XM, c = _rows(int(offsets[-1]), d, rng), _rows(M, d, rng), rng.standard_normal(M)
    got = _predict(X, offsets, XM, c, 3)
    expect = orc_m.predict(X, offsets, XM, c, 3)
    scale = orc_m.predict(X, offsets, XM, np.abs(c), 3)
    bound = 2 * (3 * (d + 3) + M + max(counts)) * U * scale
    log(f"  predict {len(counts)} configurations, d={d}, M={M}: max err / bound "
        f"{np.max(np.abs(got - expect) / np.maximum(bound, 1e-300)):.2e}")
    assert np.all(np.abs(got - expect) <= bound)


def test_predict_without_a_slot_is_bitwise_the_same():
    """A request with more pieces than a pool slot holds computes its tiles in the summing
    kernel: empty configurations appended to a small request force it, and leave the
    other energies unchanged to the bit."""
    rng = np.random.default_rng(5)
    counts = rng.integers(0, 90, size=400)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(offsets[-1])
    X, XM, c = _rows(n, 24, rng), _rows(60, 24, rng), rng.standard_normal(60)
    few = _predict(X, offsets, XM, c, 2)
    many = _predict(X, np.concatenate([offsets, np.full(140_000, n, dtype=np.int64)]), XM, c, 2)
    assert np.array_equal(few, many[:400])
    assert np.all(many[400:] == 0.0)


def test_good_groups_keep_their_energies_beside_malformed_offsets():
    """Swapped offsets make their own group of configurations NaN; groups far from it give
    the energies of the well-formed request, bit for bit."""
    rng = np.random.default_rng(6)
    counts = rng.integers(8, 65, size=600)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    X, XM, c = _rows(int(offsets[-1]), 40, rng), _rows(64, 40, rng), rng.standard_normal(64)
    good = _predict(X, offsets, XM, c, 2)
    bad_offsets = offsets.copy()
    bad_offsets[[300, 301]] = bad_offsets[[301, 300]]
    got = _predict(X, bad_offsets, XM, c, 2)
    assert np.isnan(got[300])
    assert np.array_equal(got[:280], good[:280]) and np.array_equal(got[330:], good[330:])


@pytest.mark.parametrize("d,M", [(1, 1), (7, 63), (8, 64), (9, 65), (15, 20), (17, 130), (130, 64), (131, 33)])
def test_knm_ragged_descriptor_lengths(orc_m, d, M):
    """K_NM / sigma elementwise at descriptor lengths around the k slices, even (direct
    loads) and odd (rows not 16-byte aligned): all terms positive, so the relative error is
    at most (zeta (d + 2) + atoms + 2) u on each side."""
    import torch

    from paper_2207_03803_amd import gap

    rng = np.random.default_rng(d)
    counts = np.array([1, 64, 0, 3, 256, 200, 300, 17])
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    X, XM = _rows(int(offsets[-1]), d, rng), _rows(M, d, rng)
    sigma = rng.uniform(0.5, 2.0, len(counts))
    zeta = 2
    for bn in (0, 32):
        h = gap.Handle(gap.params(d, zeta, 1.0, 1.0))
        h.set_tuning(knm_bn=bn)
        h.alloc_workspace(len(counts), X.shape[0], M)
        h.build_knm(to_dev(X), to_dev(offsets), to_dev(XM), to_dev(sigma))
        torch.cuda.synchronize()
        A, _ = h.A_view()
        got = A[:M, :len(counts)].T.cpu().numpy()
        expect = orc_m.knm(X, offsets, XM, zeta) / sigma[:, None]
        bound = 2 * (zeta * (d + 2) + 300 + 2) * U
        assert np.all(np.abs(got - expect) <= bound * np.abs(expect))
        h.close()
