"""ts_expand with sequential draws for few parents: the fewest chunks of the longest length."""
import pytest

from paper_2609_22098_amd import synth
from test_gpu_expand import _expand_and_compare, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# V: units of 256 tokens: 257 (one more than the most chunks, which stay), 385 (193 chunks of two), 511 (256), 577 (193 of
# three), an odd vocabulary of 594; one parent, a block and a workgroup of them, one more; f32 keeps the most chunks
@pytest.mark.parametrize("V,dtype", [(65792, "bf16"), (98560, "bf16"), (130816, "bf16"), (147712, "bf16"), (151937, "bf16"), (66000, "f32")])
@pytest.mark.parametrize("P", [1, 16, 64, 65])
@pytest.mark.parametrize("T", [0.7, 1.0])
def test_few_parents(torch, V, dtype, P, T):  # noqa: F811
    dr = synth.make_drafter(V, 13, 32, R=1, dtype=dtype, u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.05, seed=P)
    fr = {k: v[:P] for k, v in synth.make_frontier(dr, per_depth=5, seed=3).items()}
    assert len(fr["token"]) == P
    _expand_and_compare(torch, dr, fr, 8, T, seed=7, sample=range(0, P, max(1, P // 4)), tag=f"few parents P={P} V={V} T={T}",
                        sampler="sequential")
