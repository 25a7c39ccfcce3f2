"""The K_NM's tile plan at the edges of its chunks (128, 256 or 512 configurations, by the size
of the K_NM) and of a tile's segments, against torch in FP64."""
import numpy as np
import pytest

from tests.gpu_helpers import GpuFit, U, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,kind,M,d", [
    (1, "mixed", 3, 8), (127, "mixed", 40, 8), (128, "mixed", 40, 8), (129, "mixed", 40, 8), (385, "mixed", 40, 8),
    (700, "ones", 70, 5), (600, "empty", 33, 16), (260, "large", 33, 16), (513, "same", 65, 7),
    (255, "mixed", 4096, 1400), (513, "mixed", 4096, 600), (1025, "mixed", 2048, 600),    # chunks of 256
    (511, "mixed", 4096, 2100), (1025, "mixed", 4096, 1100),                              # chunks of 512
])
def test_plan_covers_every_configuration(N, kind, M, d):
    """Rows against (X XM^T)^2 summed per configuration: every term positive, each dot product
    of d terms and each sum rounded once per operation on both sides: 2 (2 d + atoms + 4) u."""
    import torch

    rng = np.random.default_rng(N + M)
    if kind == "mixed":
        counts = rng.integers(1, 72, N)
        counts[rng.integers(0, N, N // 8)] = 256
    elif kind == "ones":
        counts = np.ones(N, dtype=np.int64)
    elif kind == "empty":
        counts = rng.integers(0, 3, N)
    elif kind == "large":
        counts = rng.integers(200, 300, N)
    else:
        counts = np.full(N, 37)
    counts = np.maximum(counts, 1) if kind == "mixed" else counts
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(offsets[-1])
    gen = torch.Generator(device="cuda").manual_seed(N)
    X = torch.rand(n, d, dtype=torch.float64, device="cuda", generator=gen) / d ** 0.5
    XM = torch.rand(M, d, dtype=torch.float64, device="cuda", generator=gen) / d ** 0.5
    g = GpuFit(X, offsets, XM, np.ones(N), np.zeros(N), 2, jitter=1.0)
    g.build()
    assert g.h.sync()[0] == 0
    A, _ = g.h.A_view()
    expect = torch.zeros(N, M, dtype=torch.float64, device="cuda")
    expect.index_add_(0, to_dev(np.repeat(np.arange(N), counts)), (X @ XM.T) ** 2)
    err = (A[:M, :N].T - expect).abs()
    assert bool((err <= 2 * (2 * d + int(max(counts)) + 4) * U * expect).all())
    g.h.close()
