"""Greedy verification: the split argmax of target rows and the walk's rounds, against a plain walk."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _deep_trees(target, cap, seed):
    """Trees whose first child of every node is the target's argmax at it, down to a random depth (so walks
    go deep), with a second child elsewhere.  target [R][cap][V] float32 numpy."""
    from paper_2609_22098_amd import binding
    R, _, V = target.shape
    rng = np.random.default_rng(seed)
    tree = binding.HostTree.empty(R, cap)
    tree.token[:], tree.parent[:] = -1, -1
    for q in range(R):
        tree.token[q, 0] = rng.integers(0, V)
        stop = int(rng.integers(0, 17))
        n, cur, depth = 0, 0, 0
        while n + 2 < cap and depth < 16:
            best = int(np.argmax(target[q, cur]))
            first = best if depth < stop else (best + 1) % V
            for rank, tok in ((1, first), (2, (best + 2) % V)):
                n += 1
                tree.token[q, n], tree.parent[q, n] = tok, cur
                tree.depth[q, n], tree.rank[q, n] = depth + 1, rank
                tree.path[q, n] = int(tree.path[q, cur]) | ((rank - 1) << (4 * depth))
            cur, depth = n - 1, depth + 1
        tree.n[q] = n
    return tree


def _walk(tree, target, q):
    cur, path = 0, []
    while True:
        g = int(np.argmax(target[q, cur]))
        kids = [i for i in range(1, int(tree.n[q]) + 1) if tree.parent[q, i] == cur and tree.token[q, i] == g]
        if not kids or len(path) >= 16:
            return path, g
        path.append(kids[0])
        cur = kids[0]


# V: below one 16-byte group, odd sizes, one sweep of 2048 bf16 tokens and one past it, many pieces; the last
# case's trees (56 x 33 rows of 64 KB: 121 MB) do not fit one round's rows
@pytest.mark.parametrize("V,R,cap,dtype,shift", [
    (7, 3, 8, "bf16", 0), (33, 2, 9, "f32", 1), (2048, 3, 12, "bf16", 3), (2049, 3, 12, "bf16", 0),
    (50001, 2, 34, "bf16", 1), (50001, 2, 34, "f32", 0), (32768, 5, 40, "bf16", 0), (16384, 56, 33, "f32", 2)])
def test_greedy_walk_over_split_rows(V, R, cap, dtype, shift):
    """Accepted paths and bonus tokens equal a plain argmax walk's, for rows that start anywhere (shift elements
    past an aligned address), with ties (values on a coarse grid) and rows of -inf but for one token."""
    import torch
    from paper_2609_22098_amd import binding
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(V + R)
    x = torch.randint(-40, 41, (R, cap, V), generator=gen).float() / 8  # exact in bf16, many ties
    x[0, 0] = -float("inf")
    x[0, 0, V - 1] = 0.5
    target = x.numpy()
    tree = _deep_trees(target, cap, V)
    flat = torch.zeros(R * cap * V + 8, dtype=dt, device="cuda")
    tgt = flat[shift:shift + R * cap * V].view(R, cap, V)
    tgt.copy_(x)
    z = torch.zeros((V, 32 if dtype == "bf16" else 16), dtype=dt, device="cuda")
    dd = binding.DeviceDrafter(torch.zeros((R, 16, V), dtype=dt, device="cuda"), z, z.clone())
    path, plen, bonus = binding.verify(dd, tree, tgt, 0.0, 1)
    for q in range(R):
        want, b = _walk(tree, target, q)
        assert list(path[q, :plen[q]]) == want and int(bonus[q]) == b, q
