"""ts_expand's merge with all waves of a workgroup on one parent (few parents), and the edge to one wave each."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_expand import _expand_and_compare, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# either side of the largest cooperative frontier; both operand types; V a multiple of 4 and odd
@pytest.mark.parametrize("P,dtype,r,V,K", [(1, "bf16", 64, 3001, 8), (255, "bf16", 256, 3000, 16),
                                           (256, "f32", 64, 2003, 4), (257, "f32", 16, 2000, 8),
                                           (512, "bf16", 32, 3000, 8)])
@pytest.mark.parametrize("T,sampler", [(0.0, "sequential"), (1.0, "gumbel"), (0.6, "gumbel")])
def test_frontier_sizes(torch, P, dtype, r, V, K, T, sampler):  # noqa: F811
    dr = synth.make_drafter(V, 16, r, R=8, dtype=dtype, u_sigma=1.5, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1,
                            seed=P)
    fr = {k: v[:P] for k, v in synth.make_frontier(dr, per_depth=5, seed=3).items()}
    assert len(fr["token"]) == P
    _expand_and_compare(torch, dr, fr, K, T, seed=7, sample=range(0, P, max(1, P // 24)),
                        tag=f"coop merge P={P} {dtype} r={r} T={T}", sampler=sampler)


@pytest.mark.parametrize("K", [1, 8, 16])
def test_equal_logits(torch, K):  # noqa: F811
    """Every logit equal: whole chunks are rescanned by all waves, and the smallest K token ids win."""
    from paper_2609_22098_amd import binding
    V, P = 5003, 9
    U = torch.zeros((1, 16, V), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((V, 32), dtype=torch.bfloat16, device="cuda")
    dd = binding.DeviceDrafter(U, W, W.clone())
    z = np.zeros(P, np.int32)
    parents = binding.parents_to_device(z, np.arange(P, dtype=np.int32), z, np.zeros(P, np.float32),
                                        np.zeros(P, np.uint64))
    out = binding.expand(dd, parents, P, K, 0.0, 1)
    torch.cuda.synchronize()
    assert torch.equal(out["child_token"].cpu(), torch.arange(K, dtype=torch.int32).expand(P, K))
    assert int(out["diag"].abs().sum()) == 0
