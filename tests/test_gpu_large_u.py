"""bf16 drafters whose U is 2 GiB or more, past the 31-bit offsets of the LDS-staged kernels: the streaming pass and the
verification's logit recompute through the register kernel."""
import numpy as np
import pytest

from paper_2609_22098_amd import synth
from test_gpu_expand import _expand_and_compare, torch  # noqa: F401
from test_gpu_tree import _trees

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def flat(torch):  # noqa: F811
    buf = torch.empty((1 << 30) + (1 << 17), dtype=torch.bfloat16, device="cuda")
    yield buf
    del buf
    torch.cuda.empty_cache()


def _widened(flat, dd):
    """The drafter with requests added until U takes 2 GiB (theirs hold whatever the buffer does)."""
    from paper_2609_22098_amd import binding
    n = dd.D * dd.V
    R = -(-(1 << 30) // n)
    U = flat[:R * n].view(R, dd.D, dd.V)
    U[:dd.R].copy_(dd.U)
    assert U.numel() * 2 >= 1 << 31
    return binding.DeviceDrafter(U, dd.E, dd.W2)


# V: whole 16-byte rows with a cut last step, and rows at any address; P: one block of 16 parents per wave, and two
@pytest.mark.parametrize("V,r", [(1032, 32), (1025, 64), (2056, 128), (1999, 256)])
@pytest.mark.parametrize("P", [37, 528])
@pytest.mark.parametrize("T,sampler", [(0.0, "sequential"), (0.7, "sequential"), (1.0, "sequential"), (0.6, "gumbel"),
                                       (1.0, "gumbel")])
def test_expand(torch, flat, monkeypatch, V, r, P, T, sampler):  # noqa: F811
    from paper_2609_22098_amd import binding
    small = binding.drafter_from_host
    monkeypatch.setattr(binding, "drafter_from_host", lambda dr: _widened(flat, small(dr)))
    dr = synth.make_drafter(V, 16, r, R=3, dtype="bf16", u_sigma=1.5, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1, seed=V)
    fr = {k: v[:P] for k, v in synth.make_frontier(dr, per_depth=11, seed=2).items()}
    assert len(fr["token"]) == P
    _expand_and_compare(torch, dr, fr, 6, T, seed=3, sample=range(0, P, max(1, P // 24)),
                        tag=f"large U V={V} r={r} P={P} T={T} {sampler}", sampler=sampler)


def test_expand_last_request(torch, flat):  # noqa: F811
    """Rows at the end of U, past 2^31 bytes: the same children as of equal rows at its start (T = 0)."""
    from paper_2609_22098_amd import binding
    V = 1025
    dr = synth.make_drafter(V, 16, 64, R=3, dtype="bf16", u_sigma=1.5, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1, seed=1)
    dd = _widened(flat, binding.drafter_from_host(dr))
    dd.U[dd.R - 1].copy_(dd.U[1])
    fr = synth.make_frontier(dr, per_depth=3, seed=2)
    outs = []
    for req in (1, dd.R - 1):
        n = 48
        par = binding.parents_to_device(fr["token"][:n], fr["depth"][:n], np.full(n, req, np.int32), fr["log_surv"][:n],
                                        fr["path"][:n])
        outs.append(binding.expand(dd, par, n, 8, 0.0, 1))
    torch.cuda.synchronize()
    for k, v in outs[0].items():
        if not k.startswith("_"):
            assert np.array_equal(v.cpu().numpy(), outs[1][k].cpu().numpy(), equal_nan=True), k


@pytest.mark.parametrize("V,r", [(1032, 64), (1025, 32), (1999, 256)])
def test_verify(torch, flat, V, r):  # noqa: F811
    """The walks of the first requests equal those of the drafter of these requests alone, whose logits the LDS-staged
    kernel recomputes (the logits are the same bit for bit)."""
    from paper_2609_22098_amd import binding
    R, N, K, T = 6, 12, 3, 0.8
    dr = synth.make_drafter(V, 16, r, R=R, dtype="bf16", u_sigma=2.0, planted=None, zipf=(6.0, 1.1), ew_sigma=0.1, seed=V,
                            u_scale=1.5)
    anchors, _, _ = synth.make_controls(R, V, 0.0, seed=5)
    dd, tree = _trees(dr, anchors, np.full(R, 0.001, np.float32), N, K, T, 21)
    big = _widened(flat, dd)
    wide = binding.HostTree.empty(big.R, N + 1)  # the other requests: a root alone
    for f in ("n", "token", "parent", "depth", "rank", "path"):
        getattr(wide, f)[:R] = getattr(tree, f)
    tgt = torch.zeros((big.R, N + 1, V), dtype=torch.bfloat16, device="cuda")
    for q in range(R):
        x = synth.make_target_rows(dr, q, tree.depth[q, :int(tree.n[q]) + 1], 0.3, seed=2)[1]
        tgt[q, :x.shape[0]] = torch.from_numpy(x).to(torch.bfloat16)
    binding.verify_set_mode("staged")
    try:
        for seed in range(3):
            want = binding.verify(dd, tree, tgt[:R].contiguous(), T, seed)
            got = binding.verify(big, wide, tgt, T, seed)
            for a, b, what in zip(got, want, ("path", "length", "bonus")):
                assert np.array_equal(a[:R], b), (what, seed)
            assert not got[1][R:].any()
    finally:
        binding.verify_set_mode("auto")
    assert int(want[1].max()) >= 1
