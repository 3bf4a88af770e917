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
