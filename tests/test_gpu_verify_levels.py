"""ts_verify_level_counts: the levels of walks whose paths are known."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_tree import _trees, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# sigma: how far the target is from the draft (walks that end at the root, in the middle of the tree, at a leaf);
# rows: every node's logits in the first launch, or one node's a launch
@pytest.mark.parametrize("sigma", [0.02, 0.5, 4.0])
@pytest.mark.parametrize("rows", ["all", "few"])
@pytest.mark.parametrize("mode", ["auto", "staged"])
def test_levels_of_one_walk(torch, sigma, rows, mode):  # noqa: F811
    """One request: a level for each node with children that the walk stands at, one at least."""
    from paper_2609_22098_amd import binding
    V, N, K, T = 2001, 12, 2, 0.9
    dr = synth.make_drafter(V, 12, 32, R=1, dtype="bf16", u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1,
                            seed=3, u_scale=2.0)
    seen = set()
    for seed in range(16):
        dd, tree = _trees(dr, np.array([seed], np.int32), np.zeros(1, np.float32), N, K, T, seed)
        x = synth.make_target_rows(dr, 0, tree.depth[0, :int(tree.n[0]) + 1], sigma, seed=seed)[1]
        tgt = torch.zeros((1, N + 1, V), dtype=torch.bfloat16, device="cuda")
        tgt[0, :x.shape[0]] = torch.from_numpy(x).to(torch.bfloat16)
        ws = binding.torch_empty_bytes(binding.verify_workspace_size(dd, N + 1 if rows == "all" else 1, T))
        before = binding.verify_level_counts()
        binding.verify_set_mode(mode)
        try:
            path, plen, _ = binding.verify(dd, tree, tgt, T, seed, workspace=ws)
        finally:
            binding.verify_set_mode("auto")
        fused, fallbacks, staged = (a - b for a, b in zip(binding.verify_level_counts(), before))
        with_kids = set(tree.parent[0, 1:int(tree.n[0]) + 1].tolist())
        visited = [0] + path[0, :plen[0]].tolist()
        want = max(1, sum(v in with_kids for v in visited))
        if mode == "auto":
            assert (fused, fallbacks, staged) == (want, 0, 0), (seed, visited)
        else:  # a leaf's bonus takes a round of its own
            assert (fused, fallbacks, staged) == (0, 0, len(visited)), (seed, visited)
        seen.add((len(visited), visited[-1] in with_kids))
    assert len(seen) > 1 or sigma > 1, seen
