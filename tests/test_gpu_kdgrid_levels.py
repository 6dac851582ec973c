"""GPU tests of npg_build_kdgrid's level kernels at the sizes where they change:
nodes of one and two registers per lane, of one wavefront and of a workgroup
(64, 128, 512, 2048 and 8192 photons, and one more), levels of more than 1024
nodes, trees of depth 1 (photons read where they lie) and deeper (in voxel
order), and the capacity check at the roots and at a level.  Leaves, photon
order, nodes and locations are integers: all exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import kdgrid as kg
from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def tf(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


def _check(ctx, npg, p, nrm, valid, res, T, Vt, D, slack):
    lo, hi = (0.0, -0.25, 0.0), (1.0, 1.0, 1.5)
    ref = kg.build(p, nrm, valid, res, lo, hi, T, Vt, D)
    prm = npg.kdgrid_params(res, lo, hi, T, Vt, D)
    args = (tf(p), None if nrm is None else tf(nrm), None if valid is None else torch.from_numpy(valid).to(DEV))
    g = npg.build_kdgrid(ctx, prm, *args, max_leaves=max(1, ref.n_leaves + slack))
    off = g["leaf_off"].cpu().numpy().view(np.uint32)
    assert g["n_leaves"] == ref.n_leaves and g["n_nodes"] == ref.n_nodes()
    assert np.array_equal(off, ref.leaf_off())
    assert np.array_equal(g["perm"][:int(off[-1])].cpu().numpy().view(np.uint32), ref.perm())
    assert np.array_equal(np.sort(g["perm"].cpu().numpy()), np.arange(len(p)))  # those of invalid voxels follow
    q = np.concatenate([p, np.random.default_rng(5).random((500, 3)).astype(np.float32) * 1.5 - 0.25])
    assert np.array_equal(npg.locate(ctx, prm, g, tf(q)).cpu().numpy().view(np.uint32), kg.locate(ref, q))
    assert npg.sync_status(ctx) == 0
    return prm, args, ref


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 512, 513, 2047, 2048, 2049, 8192, 8193, 20001])
@pytest.mark.parametrize("D,use_nrm,T", [(1, True, 1e9), (2, True, 1e9), (3, False, 1.0), (16, True, 600.0)])
def test_one_voxel(ctx, npg, n, D, use_nrm, T):
    rng = np.random.default_rng(1000 * D + n)
    p = rng.random((n, 3)).astype(np.float32)
    p[: n // 4, 2] = np.float32(0.375)  # equal keys on the longest axis
    nrm = synth.unit_vectors(rng, n).astype(np.float32) if use_nrm else None
    _check(ctx, npg, p, nrm, None, 1, T, 0.3, D, 0)


@pytest.mark.parametrize("res,n,T,D", [(12, 40000, 9.0, 6), (16, 9000, 1.0, 8), (5, 60000, 300.0, 2)])
def test_many_nodes(ctx, npg, res, n, T, D):
    rng = np.random.default_rng(res)
    p = rng.random((n, 3)).astype(np.float32)
    p[: n // 2] = (0.31 + 0.05 * rng.standard_normal((n // 2, 3))).clip(0, 0.99)  # a few crowded voxels
    nrm = synth.surface_normals(res, p, n_creases=6, crease_radius=0.3, freq=3.0)
    valid = (rng.random(res ** 3) < 0.8).astype(np.uint8)
    prm, args, ref = _check(ctx, npg, p, nrm, valid, res, T, 0.3, D, 3)
    roots = len(ref.roots)
    for cap in (ref.n_leaves - 1, (roots + ref.n_leaves) // 2, roots, roots - 1):  # one leaf, a level, the roots
        with pytest.raises(npg.NpgError) as e:
            npg.build_kdgrid(ctx, prm, *args, max_leaves=cap)
        assert e.value.code == npg.E_CAPACITY
    _check(ctx, npg, p, nrm, valid, res, T, 0.3, D, 0)  # the context is as good as before


def test_budget(ctx, npg):
    """A context with a budget builds without the copies in voxel order, and
    gives the same grid as one without."""
    rng = np.random.default_rng(9)
    n, res, L = 300000, 9, 20000
    p = rng.random((n, 3)).astype(np.float32)
    nrm = synth.unit_vectors(rng, n).astype(np.float32)
    prm = npg.kdgrid_params(res, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), 100.0, 0.3, 4)  # at most 16 leaves a voxel
    small = npg.Context(0, 24 << 20)  # four arrays of n words, the sort's and the levels'; the copies are 8.4 MB more
    a = npg.build_kdgrid(ctx, prm, tf(p), tf(nrm), max_leaves=L)
    b = npg.build_kdgrid(small, prm, tf(p), tf(nrm), max_leaves=L)
    assert a["n_leaves"] == b["n_leaves"] and a["n_nodes"] == b["n_nodes"]
    for k in ("perm", "leaf_off", "cell_root", "nodes"):
        assert torch.equal(a[k], b[k]), k
    small.close()
