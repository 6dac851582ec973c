"""GPU tests of the radix sort behind the octree build and the KD grid: sizes
about its tiles and chunks of tiles, digit widths from one bit to eight."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _morton(pos, depth):
    q = (pos.astype(np.float64) * 2 ** depth).astype(np.int64)
    code = np.zeros(len(pos), np.int64)
    for b in range(depth):
        for a in range(3):
            code |= ((q[:, a] >> b) & 1) << (3 * b + a)
    return code


# 3072 / 4096 items per tile with / without payload, 32 tiles per chunk;
# split_count 0: every occupied cell of the finest level is a leaf, so depth 0
# .. 6 gives 1 to 18 bits of leaf ids (one to three passes)
@pytest.mark.parametrize("n", [1, 2, 63, 513, 3071, 3072, 3073, 4096, 4097, 98304, 98305, 131073, 1000003])
@pytest.mark.parametrize("depth", [0, 1, 3, 6])
def test_octree_sort_stable(ctx, npg, n, depth):
    rng = np.random.default_rng(n + depth)
    pos = rng.random((n, 3), dtype=np.float32) ** 2  # crowded towards the corner: runs of equal leaves
    pos[pos >= 1] = 0.5
    dirs, w = rng.random((n, 3), dtype=np.float32), rng.integers(0, 2 ** 32, n, dtype=np.uint32)
    code = _morton(pos, depth)
    leaves, leaf = np.unique(code, return_inverse=True)
    perm = np.argsort(leaf, kind="stable")
    off = np.concatenate([[0], np.cumsum(np.bincount(leaf, minlength=len(leaves)))])
    p = torch.from_numpy(pos).to(DEV)
    h = npg.build_hierarchy(ctx, p, 0, depth)
    assert h["n_leaves"] == len(leaves)
    assert np.array_equal(h["leaf_of"].cpu().numpy(), leaf)
    assert np.array_equal(h["perm"].cpu().numpy(), perm)
    assert np.array_equal(h["leaf_off"].cpu().numpy(), off)
    s = npg.build_hierarchy_sorted(ctx, p, torch.from_numpy(dirs).to(DEV),
                                   torch.from_numpy(w.view(np.int32)).to(DEV), 0, depth)
    assert np.array_equal(s["perm"].cpu().numpy(), perm)
    assert np.array_equal(s["dirs"].cpu().numpy(), dirs[perm])
    assert np.array_equal(s["w"].cpu().numpy().view(np.uint32), w[perm])
    assert npg.sync_status(ctx) == 0
