"""A configuration's predicted energy does not depend, to the bit, on the request it is
part of: neither on the other configurations nor on its place among them."""
import numpy as np
import pytest

from tests.gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


class Model:
    def __init__(self, d, M, zeta, seed):
        import torch

        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.d, self.zeta = d, zeta
        self.XM = self.rows(M)
        self.c = torch.randn(M, dtype=torch.float64, device="cuda", generator=self.gen)

    def rows(self, n):
        import torch

        x = torch.rand((n, self.d), dtype=torch.float64, device="cuda", generator=self.gen)
        return x / torch.sqrt((x * x).sum(dim=1, keepdim=True))

    def predict(self, X, offsets, c=None, XM=None):
        import torch

        from paper_2207_03803_amd import gap

        out = torch.full((len(offsets) - 1,), float("nan"), dtype=torch.float64, device="cuda")
        h = gap.Handle(gap.params(self.d, self.zeta))
        h.set_model(self.XM if XM is None else XM)
        h.predict(X, to_dev(np.asarray(offsets, dtype=np.int64)), self.c if c is None else c, out)
        torch.cuda.synchronize()
        h.close()
        return out


# descriptor length, sparse points, configurations, one very large configuration's atoms
@pytest.mark.parametrize("d,M,N,large", [
    (24, 700, 333, 0),          # a column tile per workgroup
    (17, 1300, 4500, 0),        # large requests: whole groups of column tiles
    (33, 260, 900, 5000),       # a configuration over many atom tiles
    (8, 30, 2000, 300),         # one column tile
])
def test_energies_do_not_depend_on_the_request(d, M, N, large):
    m = Model(d, M, 3, 7 * d + M)
    rng = np.random.default_rng(N)
    counts = rng.integers(0, 65, N)
    if large:
        counts[N // 3] = large
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    X = m.rows(int(offsets[-1]))
    whole = m.predict(X, offsets)
    parts = [(0, 1), (N // 3, N // 3 + 1), (N - 1, N), (5, 6), (3, 40), (N // 4, N // 2), (1, N), (0, N - 1), (100, 165)]
    for lo, hi in parts:
        a, b = offsets[lo], offsets[hi]
        got = m.predict(X[a:b].clone(), offsets[lo:hi + 1] - a)
        assert bool((got == whole[lo:hi]).all()), (lo, hi)


def test_requests_of_several_ranges_of_atoms():
    """More atoms than one claim of the pool holds: configurations that lie across the ranges'
    ends are carried on.  Against FP64 torch: a product of d terms, the power, M and the
    atoms, (3 (d + 2) + M + atoms) u of the (positive) sum on each side."""
    import torch

    from tests.gpu_helpers import U

    d, M, N = 4, 60, 80_000
    m = Model(d, M, 3, 5)
    m.c.abs_()
    rng = np.random.default_rng(3)
    counts = rng.integers(0, 80, N)
    counts[rng.integers(0, N, 40)] = 9000
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(offsets[-1])
    assert n > 2_621_440
    X = m.rows(n)
    whole = m.predict(X, offsets)
    cuts = np.searchsorted(offsets, np.linspace(0, n, 5).astype(np.int64))
    for lo, hi in [(int(a), int(b)) for a, b in zip(cuts[:-1], cuts[1:])] + [(N // 2 - 900, N // 2 + 900)]:
        hi = min(hi, N)
        a, b = offsets[lo], offsets[hi]
        got = m.predict(X[a:b].clone(), offsets[lo:hi + 1] - a)
        assert bool((got == whole[lo:hi]).all()), (lo, hi)
    e = ((X @ m.XM.T) ** 3) @ m.c
    expect = torch.zeros(N, dtype=torch.float64, device="cuda")
    expect.index_add_(0, to_dev(np.repeat(np.arange(N), counts)), e)
    assert bool(((whole - expect).abs() <= 2 * (3 * (d + 2) + M + 9000) * U * expect).all())


def test_a_request_without_room_in_the_pool():
    """So many sparse points that not even one tile of atoms has room: the summing kernel forms
    the energies itself, with the same sums (one more sparse point of weight zero than the
    largest model that still has room)."""
    import torch

    M, d = 2_621_441, 2
    m = Model(d, M, 2, 9)
    m.c[-1] = 0.0
    counts = np.array([40, 0, 1, 300, 77, 9])
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    X = m.rows(int(offsets[-1]))
    without = m.predict(X, offsets)
    room = m.predict(X, offsets, c=m.c[:-1].clone(), XM=m.XM[:-1].clone())
    assert bool((without == room).all())
    expect = torch.stack([((X[a:b] @ m.XM.T) ** 2 @ m.c).sum() for a, b in zip(offsets[:-1], offsets[1:])])
    assert torch.allclose(room, expect, rtol=0, atol=1e-10 * float(m.c.abs().sum()) * 300)
