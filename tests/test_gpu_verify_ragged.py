"""ts_verify at T > 0 over vocabularies whose rows start at any element."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_tree import _trees, _verify_compare, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# V: rows cut inside a quad (1 to 3 tokens past it), below one 64-token step, one token past a step and past a
# workgroup's sweep of 1024; 5 requests x 3 depths of odd rows leave U an odd number of elements
@pytest.mark.parametrize("V,r", [(41, 32), (1025, 64), (4098, 32), (9999, 128)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode", ["auto", "staged"])
def test_rows_at_any_element(torch, V, r, dtype, mode):  # noqa: F811
    """Every walk against the oracle's: the logit recompute (whole and cut steps), the rows' quads in one launch
    per level and per stage."""
    R, N, K, T = 5, 12, 3, 0.8
    dr = synth.make_drafter(V, 3, min(r, 64) if dtype == "f32" else r, R=R, dtype=dtype, u_sigma=2.0, planted=None,
                            zipf=(6.0, 1.1), ew_sigma=0.3, seed=V, u_scale=1.5)
    anchors, _, _ = synth.make_controls(R, V, 0.0, seed=5)
    dd, tree = _trees(dr, anchors, np.full(R, 0.001, np.float32), N, K, T, 21)
    tgt32 = {q: synth.make_target_rows(dr, q, tree.depth[q, :int(tree.n[q]) + 1], 1.0, seed=2)[1] for q in range(R)}
    _verify_compare(dd, dr, tree, tgt32, list(range(R)), T, 33, tag=f"verify ragged {dtype} V={V} {mode}", mode=mode,
                    expect="fused" if mode == "auto" else "staged")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_workspaces_of_every_accepted_size(torch, dtype):  # noqa: F811
    """Deep walks (the target follows the draft closely): with the whole workspace a launch goes from node to node
    by itself, with less it comes back to the host more often; the walks are the same, and the oracle's."""
    from paper_2609_22098_amd import binding
    R, V, N, K, T = 6, 3001, 40, 2, 0.9
    dr = synth.make_drafter(V, 12, 32, R=R, dtype=dtype, u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1,
                            seed=3, u_scale=2.0)
    anchors, _, _ = synth.make_controls(R, V, 0.0, seed=5)
    dd, tree = _trees(dr, anchors, np.zeros(R, np.float32), N, K, T, 21)
    tgt32 = {q: synth.make_target_rows(dr, q, tree.depth[q, :int(tree.n[q]) + 1], 0.05, seed=2)[1] for q in range(R)}
    _verify_compare(dd, dr, tree, tgt32, list(range(R)), T, 33, tag=f"verify deep {dtype}", expect="fused")
    tgt = torch.zeros((R, N + 1, V), dtype=dd.U.dtype, device="cuda")
    for q, x in tgt32.items():
        tgt[q, :x.shape[0]] = torch.from_numpy(x).to(tgt.dtype)
    size = binding.verify_workspace_size(dd, N + 1, T)
    want = binding.verify(dd, tree, tgt, T, 33, workspace=binding.torch_empty_bytes(size))
    assert max(want[1]) >= 4, want[1]  # walks of several levels
    least = R * V * 4  # the logits of one node per request alone
    refused = 0
    for n in np.geomspace(least, size, 24).astype(int):
        try:
            got = binding.verify(dd, tree, tgt, T, 33, workspace=binding.torch_empty_bytes(int(n)))
        except binding.TreeSparkError as e:
            assert e.code == binding.TS_ENOSPACE
            refused += 1
            continue
        for a, b, what in zip(got, want, ("path", "length", "bonus")):
            assert np.array_equal(a, b), (what, n)
    assert 0 < refused < 24
