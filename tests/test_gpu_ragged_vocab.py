"""ts_expand over bf16 vocabularies that are no multiple of 8 tokens (rows of U at any 2-byte address)."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_expand import _expand_and_compare, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# V: under one 16-token run, a run's edges, one step's edges, a chunk's, several chunks and segments.  3 x 5 rows
# of odd length leave the array an odd number of elements, whose last one no whole word holds.
@pytest.mark.parametrize("V,r", [(5, 32), (17, 64), (63, 32), (65, 64), (257, 128), (1023, 256), (4099, 32),
                                 (8190, 64), (12287, 64)])
@pytest.mark.parametrize("T,sampler", [(0.0, "sequential"), (0.7, "sequential"), (1.0, "sequential"),
                                       (1.0, "gumbel"), (0.6, "gumbel")])
def test_rows_at_any_address(torch, V, r, T, sampler):  # noqa: F811
    """37 parents (one block of 16 per wave), each row's last token among its largest."""
    dr = synth.make_drafter(V, 5, r, R=3, dtype="bf16", u_sigma=1.0, planted=None, zipf=None, ew_sigma=0.2, seed=V)
    last = synth.f32_to_bf16_bits(np.full((3, 5), 3.0, np.float32))
    dr.U[:, :, V - 1], dr.U32[:, :, V - 1] = last, 3.0
    fr = {k: v[:37] for k, v in synth.make_frontier(dr, per_depth=3, seed=2).items()}
    fr["depth"][36], fr["request"][36], fr["path"][36] = 4, 2, 0  # the array's last row
    _expand_and_compare(torch, dr, fr, min(6, V), T, seed=3, tag=f"odd vocab V={V} r={r} T={T} {sampler}",
                        sampler=sampler)


@pytest.mark.parametrize("V", [5003, 5004])
@pytest.mark.parametrize("T,sampler", [(0.0, "sequential"), (0.7, "sequential"), (1.0, "sequential"), (0.7, "gumbel"),
                                       (1.0, "gumbel")])
def test_wide_frontier(torch, V, T, sampler):  # noqa: F811
    """560 parents (two blocks per wave), 64 of them against the oracle."""
    dr = synth.make_drafter(V, 16, 64, R=7, dtype="bf16", u_sigma=1.5, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1,
                            seed=V)
    fr = synth.make_frontier(dr, per_depth=5, seed=3)
    _expand_and_compare(torch, dr, fr, 8, T, seed=5, sample=range(0, 560, 9), tag=f"odd vocab wide V={V} T={T}",
                        sampler=sampler)
