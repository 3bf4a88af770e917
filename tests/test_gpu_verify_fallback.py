"""ts_verify at T > 0 when waits between the workgroups of a round's launch run out: the way back to the per-stage
launches, from walks that had not begun, were under way or were already reported."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_tree import _trees, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# polls of a wait: none at all, and few enough that some waits of a walk run out and some do not (the workgroups of
# an item reach each exchange within a few polls of one another, the later ones last)
@pytest.mark.parametrize("limit", [0, 1, 2, 3, 4, 6, 8, 12])
@pytest.mark.parametrize("rows", ["all", "few"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_walks_after_a_wait_ran_out(torch, limit, rows, dtype):  # noqa: F811
    """Deep walks over 3001 tokens (3 workgroups an item): the same as the per-stage launches', for 12 seeds.
    rows: the workspace holds the logits of every node, or of one node per request (a round per level: a walk is
    then often complete when the wait of another of its workgroups runs out)."""
    from paper_2609_22098_amd import binding
    R, V, N, K, T = 6, 3001, 40, 2, 0.9
    dr = synth.make_drafter(V, 12, 32, R=R, dtype=dtype, u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1,
                            seed=3, u_scale=2.0)
    anchors, _, _ = synth.make_controls(R, V, 0.0, seed=5)
    dd, tree = _trees(dr, anchors, np.zeros(R, np.float32), N, K, T, 21)
    tgt = torch.zeros((R, N + 1, V), dtype=dd.U.dtype, device="cuda")
    for q in range(R):
        x = synth.make_target_rows(dr, q, tree.depth[q, :int(tree.n[q]) + 1], 0.05, seed=2)[1]
        tgt[q, :x.shape[0]] = torch.from_numpy(x).to(tgt.dtype)
    ws = binding.torch_empty_bytes(binding.verify_workspace_size(dd, N + 1 if rows == "all" else 1, T))
    hook = binding.lib().ts_internal_verify_wait_limit
    deepest = 0
    for seed in range(12):
        binding.verify_set_mode("staged")
        try:
            want = binding.verify(dd, tree, tgt, T, seed, workspace=ws)
        finally:
            binding.verify_set_mode("auto")
        before = binding.verify_level_counts()
        hook(limit)
        try:
            got = binding.verify(dd, tree, tgt, T, seed, workspace=ws)
        finally:
            hook(-1)
        fused, fallbacks, staged = (a - b for a, b in zip(binding.verify_level_counts(), before))
        for a, b, what in zip(got, want, ("path", "length", "bonus")):
            assert np.array_equal(a, b), (what, seed, a, b)
        assert staged == 0 and fused >= fallbacks
        if limit == 0:
            assert fused == fallbacks >= 1
        deepest = max(deepest, int(max(want[1])))
    assert deepest >= 4
