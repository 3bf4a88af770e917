"""Device-resident waves: children ranked by counting or by a sort, and those the full list drops at once."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_tree import _compare_all, _trees, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# N = 512 with K = 2 sorts (hundreds of children before the list is full); N = 1 fills its list with the first child
@pytest.mark.parametrize("N,K", [(1, 4), (2, 1), (9, 8), (64, 8), (100, 8), (129, 8), (512, 2)])
@pytest.mark.parametrize("T,sampler,theta", [(0.0, "sequential", 0.0), (1.0, "gumbel", 0.0), (0.7, "sequential", 0.01)])
def test_trees_against_oracle(torch, N, K, T, sampler, theta):  # noqa: F811
    dr = synth.make_drafter(1500, 12, 32, R=3, dtype="bf16", u_sigma=3.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.3,
                            seed=5, u_scale=2.0)
    anchors, thetas = np.array([3, 4, 5], np.int32), np.array([theta, theta / 2, 0.0], np.float32)
    _, tree = _trees(dr, anchors, thetas, N, K, T, 11, sampler=sampler)
    assert int(tree.n.max()) == min(N, 12 if K == 1 else N)
    _compare_all(dr, tree, anchors, thetas, N, K, T, 11, tag=f"wave ranks N={N} K={K} T={T}", sampler=sampler,
                 min_share=0.2)
