"""ts_build_tree of chains (K = 1) on the device's waves: the plan of the bound on their parents, which a price undercuts."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_tree import _compare_all, _trees, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# requests: one, a workgroup's 64 parents and one more, 512 (two parent blocks per wave) and some more; prices that
# stop none, some or most of them on the way
@pytest.mark.parametrize("R,V,dtype", [(1, 5000, "bf16"), (64, 5000, "bf16"), (65, 5003, "bf16"), (512, 2000, "bf16"),
                                       (530, 2003, "bf16"), (520, 2000, "f32")])
@pytest.mark.parametrize("T,sampler", [(0.0, "sequential"), (0.7, "sequential"), (1.0, "gumbel")])
def test_chains(torch, R, V, dtype, T, sampler):  # noqa: F811
    # f32's tolerance of 1e-5 needs logits that are not sharp: log p-hat moves by 0.67 (1 - p-hat) / (1 - q0) times an
    # error of log q0, and log q0 of a logit near 30 carries 2e-6 (q0 = 0.99: 1e-5 a node)
    dr = synth.make_drafter(V, 4, 32, R=R, dtype=dtype, u_sigma=3.0 if dtype == "bf16" else 1.5, planted=None,
                            zipf=(6.0, 1.1), ew_sigma=0.3 if dtype == "bf16" else 0.1, seed=R,
                            u_scale=2.0 if dtype == "bf16" else 1.0)
    anchors, _, _ = synth.make_controls(R, V, 0.0, seed=5)
    thetas = np.tile(np.array([0.0, 0.02, 0.2, 0.6], np.float32), R)[:R]
    _, tree = _trees(dr, anchors, thetas, 4, 1, T, 11, sampler=sampler)
    some = sorted(set(range(0, R, max(1, R // 16))) | {R - 1})
    _compare_all(dr, tree, anchors, thetas, 4, 1, T, 11, requests=some, tag=f"chains R={R} V={V} T={T}", sampler=sampler,
                 min_share=0.5)
    if R > 1:
        assert len(set(tree.n.tolist())) > 1
