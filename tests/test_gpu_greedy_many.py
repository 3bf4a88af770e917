"""Greedy verification of many short rows: all of them in one round, or gathered level by level, against a plain walk."""
import numpy as np
import pytest

from test_gpu_greedy_rows import _deep_trees, _walk

pytestmark = pytest.mark.gpu


# either side of the bytes up to which all rows are listed (144 MiB), full trees and roots alone among them
@pytest.mark.parametrize("V,R,cap,dtype", [(64, 700, 34, "bf16"), (1, 300, 5, "f32"), (8192, 260, 34, "bf16"),
                                           (8192, 290, 34, "bf16"), (4096, 300, 34, "f32")])
def test_many_rows(V, R, cap, dtype):
    import torch
    from paper_2609_22098_amd import binding
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(V + R)
    tgt = torch.randint(-40, 41, (R, cap, V), generator=gen, device="cuda").to(dt) / 8  # exact, with ties
    target = tgt.float().cpu().numpy()
    tree = _deep_trees(target, cap, V)
    tree.n[::7] = 0
    z = torch.zeros((V, 32 if dtype == "bf16" else 16), dtype=dt, device="cuda")
    dd = binding.DeviceDrafter(torch.zeros((R, 16, V), dtype=dt, device="cuda"), z, z.clone())
    path, plen, bonus = binding.verify(dd, tree, tgt, 0.0, 1)
    for q in range(R):
        want, b = _walk(tree, target, q)
        assert list(path[q, :plen[q]]) == want and int(bonus[q]) == b, q
