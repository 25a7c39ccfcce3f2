"""gap_workspace_bytes as a caller uses it who allocates once for the largest problem."""
import random

import pytest

from paper_2207_03803_amd import gap


@pytest.mark.parametrize("n_configs,M,d", [(10_000, 1_000, 400), (40_000, 500, 400), (3_000, 100, 64), (1, 4_000, 256)])
def test_workspace_never_shrinks_with_more_atoms(n_configs, M, d):
    """Around the sizes where the K_NM's tile plan goes over to longer chunks (2 n_atoms M d =
    8.2e10 and 2.8e11 operations) and far from them."""
    p = gap.params(d, 2)
    sizes = sorted({int(f * e / (2 * M * d)) + k for e in (8.2e10, 2.8e11) for f in (0.5, 1.0, 2.0) for k in (-1, 0, 1, 2)})
    bytes_ = [gap.workspace_bytes(p, n_configs, a, M) for a in sizes]
    assert bytes_ == sorted(bytes_), list(zip(sizes, bytes_))


def test_workspace_never_shrinks_with_the_problem():
    rng = random.Random(2)
    for _ in range(4000):
        p = gap.params(rng.choice([37, 64, 128, 256, 400]), 2, precision=rng.choice([gap.GAP_FP64, gap.GAP_MIXED_FP32]),
                       flags=rng.choice([0, gap.GAP_FLAG_KNM_INT8]))
        small = [rng.randint(1, 40_000), rng.randint(1, 2_000_000), rng.randint(1, 3_000)]
        obs = [rng.randint(1, 20_000), rng.randint(1, 900_000)]
        for i in range(5):
            more = small + obs
            more[i] += rng.choice([1, 100, more[i]])
            if i < 3:
                assert gap.workspace_bytes(p, *small) <= gap.workspace_bytes(p, *more[:3]), (small, more)
            assert (gap.lib().gap_workspace_bytes_obs(p, small[0], small[1], *obs, small[2])
                    <= gap.lib().gap_workspace_bytes_obs(p, more[0], more[1], more[3], more[4], more[2])), (small, obs, more)
