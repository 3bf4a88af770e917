"""ts_expand where the parent groups do not divide the workgroups that fit: chunk counts rounded down to the XCDs."""
import pytest

from paper_2609_22098_amd import synth
from test_gpu_expand import _expand_and_compare, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# 3 groups (8 waves of two blocks, or 4 of them), 5 and 7 groups of 64 parents; V whole and ragged
@pytest.mark.parametrize("P,V", [(320, 60000), (400, 60001), (600, 60000)])
@pytest.mark.parametrize("T,sampler", [(0.0, "sequential"), (0.7, "sequential"), (0.7, "gumbel")])
def test_groups(torch, P, V, T, sampler):  # noqa: F811
    dr = synth.make_drafter(V, 4, 64, R=4, dtype="bf16", u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.05,
                            seed=P)
    fr = {k: v[:P] for k, v in synth.make_frontier(dr, per_depth=38, seed=3).items()}
    assert len(fr["token"]) == P
    _expand_and_compare(torch, dr, fr, 8, T, seed=7, sample=range(0, P, P // 10), tag=f"groups P={P} V={V} T={T}",
                        sampler=sampler)
