"""ts_expand with vocabularies of one step: a chunk that has no second tile to load."""
import pytest

from paper_2609_22098_amd import synth
from test_gpu_expand import _expand_and_compare, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# one step whole, without its last runs, and of odd rows; two steps beside it.  600 parents take two blocks per wave; the
# last of each frontier read the last row of U, behind which a second tile would lie
@pytest.mark.parametrize("V", [64, 40, 57, 72])
@pytest.mark.parametrize("r", [64, 256])
@pytest.mark.parametrize("P", [16, 600])
@pytest.mark.parametrize("T,sampler", [(0.0, "gumbel"), (0.7, "gumbel"), (1.0, "gumbel"), (0.7, "sequential")])
def test_one_step(torch, V, r, P, T, sampler):  # noqa: F811
    R, D = (1, 4) if P == 16 else (10, 4)
    dr = synth.make_drafter(V, D, r, R=R, dtype="bf16", u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.05, seed=V + r)
    fr = synth.make_frontier(dr, per_depth=P // (R * D), seed=3)
    assert len(fr["token"]) == P and fr["depth"][-1] == D - 1 and fr["request"][-1] == R - 1
    _expand_and_compare(torch, dr, fr, 4, T, seed=7, sample=[*range(0, P, max(1, P // 8)), P - 1],
                        tag=f"one step V={V} r={r} P={P} T={T} {sampler}", sampler=sampler)
