"""ts_expand_noalloc at the largest frontiers its scratch holds over vocabularies that are no multiple of 8."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_zz_no_alloc import FIELDS, _outputs

pytestmark = pytest.mark.gpu


# the block table of sequential draws takes nearly all of the array; what is left holds few chunks per parent
@pytest.mark.parametrize("V,P", [(65537, 7040), (100003, 4608), (151937, 3072)])
def test_largest_frontiers(V, P):
    import torch
    from paper_2609_22098_amd import binding
    R, D, K, T = 8, 4, 2, 0.7
    dr = synth.make_drafter(V, D, 32, R=R, dtype="bf16", u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.05, seed=V)
    dd = binding.drafter_from_host(dr)
    fr = synth.make_frontier(dr, per_depth=P // (R * D), seed=2)
    assert len(fr["token"]) == P
    parents = binding.parents_to_device(fr["token"], fr["depth"], fr["request"], fr["log_surv"], fr["path"])
    got = binding.expand_noalloc(dd, parents, P, K, T, 5, _outputs(torch, P, K), sampler="sequential")
    want = binding.expand(dd, parents, P, K, T, 5, sampler="sequential")
    torch.cuda.synchronize()
    assert int(got["diag"].sum()) == 0
    # other chunks, the same logits and block masses: whole numbers and what comes from the block masses (lse of
    # z / T) are equal; a sum of z over other chunks differs by a few units in the last place of a logit near 10
    for name in FIELDS:
        a, b = got[name].cpu().numpy(), want[name].cpu().numpy()
        if a.dtype == np.int32 or name in ("lseT", "child_log_qT"):
            assert np.array_equal(a, b), name
        else:
            assert np.abs(a - b).max() <= 16 * 2.0**-23 * 16, name
