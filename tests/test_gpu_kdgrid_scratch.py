"""GPU tests of the memory npg_build_kdgrid takes: the copies in voxel order lie
where the sort was, and are left out where even that does not fit."""
import numpy as np
import pytest
import torch

from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MB, GB = 1 << 20, 1 << 30


def _inputs(n, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    p = torch.rand(n, 3, generator=g, device=DEV)
    v = torch.randn(n, 3, generator=g, device=DEV)
    return p, v / v.norm(dim=1, keepdim=True)


# six sort arrays (key, sorted key, the sort's four), the partition's two and
# the order: nine words a photon, and under one in bitmaps and digit counts
@pytest.mark.parametrize("normals", [False, True])
def test_scratch_of_a_build(npg, normals):
    n, L = 4000000, 10000
    p, v = _inputs(n, 1)
    c = npg.Context(0)
    held = c.memory_usage()[0]
    prm = npg.kdgrid_params(20, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), 1e9, 2.0, 2)
    npg.build_kdgrid(c, prm, p, v if normals else None, max_leaves=L)
    assert c.memory_usage()[0] - held <= 9.3 * 4 * n + 160 * L + MB
    c.close()


def test_no_room_for_the_order(npg):
    """With room for the build and not for the order, levels gather from the
    caller's arrays: the same grid, and the scratch without the order."""
    n, L = 100000000, 100000
    p, v = _inputs(n, 2)
    prm = npg.kdgrid_params(20, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), 5000.0, 2.0, 3)  # voxels of 12,500 split twice
    out = [{"perm": torch.zeros(n, dtype=torch.int32, device=DEV),
            "leaf_off": torch.zeros(L + 1, dtype=torch.int32, device=DEV),
            "cell_root": torch.empty(8000, dtype=torch.int32, device=DEV),
            "nodes": torch.zeros(2 * L, 2, dtype=torch.int32, device=DEV)} for _ in range(2)]
    a, b = npg.Context(0), npg.Context(0)
    held = a.memory_usage()[0]
    ga = npg.build_kdgrid(a, prm, p, v, max_leaves=L, out=out[0])
    used = a.memory_usage()[0] - held
    assert used > 9 * 4 * n
    a.close()
    torch.cuda.empty_cache()
    # all memory but what the build takes without the order (4 bytes a photon) and half of that
    hold = [torch.empty(torch.cuda.mem_get_info()[0] - used - 2 * GB, dtype=torch.uint8, device=DEV)]
    try:
        while True:
            hold.append(torch.empty(32 * MB, dtype=torch.uint8, device=DEV))
    except torch.OutOfMemoryError:
        pass
    del hold[-((used - 2 * n) // (32 * MB)):]
    torch.cuda.empty_cache()
    held = b.memory_usage()[0]
    for _ in range(2):  # the second build does not try again
        gb = npg.build_kdgrid(b, prm, p, v, max_leaves=L, out=out[1])
        assert b.memory_usage()[0] - held < used - 3 * n
    del hold
    torch.cuda.empty_cache()
    assert ga["n_leaves"] == gb["n_leaves"] > 8000 and ga["n_nodes"] == gb["n_nodes"]
    k, m = ga["n_leaves"], ga["n_nodes"]
    assert torch.equal(out[0]["perm"], out[1]["perm"]) and torch.equal(out[0]["cell_root"], out[1]["cell_root"])
    assert torch.equal(out[0]["leaf_off"][:k + 1], out[1]["leaf_off"][:k + 1])
    assert torch.equal(out[0]["nodes"][:m], out[1]["nodes"][:m])
    b.close()
