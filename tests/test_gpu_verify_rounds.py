"""ts_verify at T > 0: which nodes a round's launch takes up, and how their items reach it."""
import ctypes

import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_tree import _trees, _verify_compare, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# R requests of N nodes over V tokens: so many that the roots' logits are recomputed before the trees are indexed; all
# nodes in the first round, their items beside the rows (a few) and in a copy of their own; rows that the first round
# leaves out by the draft's estimate
@pytest.mark.parametrize("R,N,V,K", [(40, 64, 48000, 3), (20, 64, 96001, 3), (30, 24, 3000, 2), (60, 40, 500, 2),
                                     (8, 60, 40000, 2), (3, 1, 5000, 1)])
@pytest.mark.parametrize("surv", ["draft", "none", "low", "null"])
def test_rounds(torch, R, N, V, K, surv):  # noqa: F811
    """The same walks as through the per-stage launches, whatever the tree says of its nodes' survival: the draft's
    estimate, nothing (NaN, or no array at all), or that no walk gets past its root."""
    from paper_2609_22098_amd import binding
    T = 0.9
    dr = synth.make_drafter(V, 6, 32, R=R, dtype="bf16", u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1,
                            seed=R, u_scale=2.0)
    anchors, _, _ = synth.make_controls(R, V, 0.0, seed=5)
    dd, tree = _trees(dr, anchors, np.zeros(R, np.float32), N, K, T, 21)
    cap = N + 1
    at = np.minimum(tree.depth, 5) + 6 * np.arange(R)[:, None]
    rows = dd.U.view(-1, V)[torch.from_numpy(at.astype(np.int64)).cuda()]
    gen = torch.Generator(device="cuda").manual_seed(2)
    tgt = rows + (0.2 * torch.randn((R, cap, V), generator=gen, device="cuda")).to(torch.bfloat16)
    ws = binding.torch_empty_bytes(binding.verify_workspace_size(dd, cap, T))
    if surv in ("none", "low"):
        tree.log_surv[:, 1:] = np.nan if surv == "none" else -80.0
    if surv == "null":
        st = tree.struct()
        assert tree.struct() is st
        st.log_surv = ctypes.c_void_p(None)
    got = {}
    for mode in ("staged", "auto"):
        binding.verify_set_mode(mode)
        try:
            got[mode] = [binding.verify(dd, tree, tgt, T, seed, workspace=ws) for seed in range(4)]
        finally:
            binding.verify_set_mode("auto")
    for a, b in zip(got["auto"], got["staged"]):
        for x, y, what in zip(a, b, ("path", "length", "bonus")):
            assert np.array_equal(x, y), (what, x, y)
    if N > 1:
        assert max(int(a[1].max()) for a in got["auto"]) >= 2


def test_large_trees_against_oracle(torch):  # noqa: F811
    """Roots first: 3 requests of 100 nodes over 300007 tokens."""
    R, V, N, K, T = 3, 300007, 100, 3, 0.8
    dr = synth.make_drafter(V, 4, 32, R=R, dtype="bf16", u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1, seed=4,
                            u_scale=2.0)
    anchors, _, _ = synth.make_controls(R, V, 0.0, seed=5)
    dd, tree = _trees(dr, anchors, np.zeros(R, np.float32), N, K, T, 21)
    assert int(tree.n.sum()) // 4 * V * 6 > 112 << 20
    tgt32 = {q: synth.make_target_rows(dr, q, tree.depth[q, :int(tree.n[q]) + 1], 0.3, seed=2)[1] for q in range(R)}
    _verify_compare(dd, dr, tree, tgt32, list(range(R)), T, 33, tag="verify large trees", expect="fused", min_whole=0.6)
