"""GPU tests of the rule that cuts large leaves into slices: which batches pay for
the zeroing pass that cut leaves need, and exact sums at the rule's edges."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _photons(seed, counts):
    rng = synth.rng_for(seed)
    n = int(sum(counts))
    dirs = synth.to_f32_dirs(synth.unit_vectors(rng, n))
    w = rng.integers(0, 2 ** 32, n, dtype=np.uint64).astype(np.uint32)
    return dirs, w, np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int32 if a.dtype == np.uint32 else a.dtype)).to(DEV)


def _launches(ctx, call):
    """Launches of a call: the nodes of the graph it is captured into."""
    call()  # attributes are set and modules loaded outside the capture
    torch.cuda.synchronize()
    hip, s = ctx.lib, torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    with torch.cuda.stream(s):
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 2) == 0  # relaxed
        call()
        assert hip.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


# a batch in which only leaves of more than 8192 photons would be cut takes one
# launch: 192 leaves of 64x64 maps are the last that may be cut, 48 of 128x128
@pytest.mark.parametrize("L,H,W,launches", [(200, 64, 64, 1), (193, 64, 64, 1), (192, 64, 64, 2), (49, 128, 128, 1),
                                            (48, 128, 128, 2), (513, 16, 16, 1), (512, 16, 16, 2)])
def test_zeroing_pass(ctx, npg, L, H, W, launches):
    dirs, w, off = _photons(L, [30] * L)
    d, ww, o = _dev(dirs), _dev(w), _dev(off)
    e = torch.empty((L, H, W), dtype=torch.int64, device=DEV)
    assert _launches(ctx, lambda: npg.splat_histograms(ctx, d, ww, o, H, W, energy=e, want_count=False)) == launches


# photons about two and three slices (of 2048, or L H W / 192 where that is more)
# and about n^2 units (L H W / 1152) for n = 4 and 9; large maps with several bands;
# accumulated onto the first result
@pytest.mark.parametrize("L,H,W", [(60, 64, 64), (16, 128, 128), (3, 256, 256), (400, 16, 16)])
@pytest.mark.parametrize("count", [False, True])
def test_uneven_leaves_exact(ctx, npg, orc, L, H, W, count):
    q = L * H * W // (768 if count else 1152)  # unit
    two = 2 * max(2048, 6 * q)
    edges = [0, 1, two - 1, two, two * 3 // 2 - 1, two * 3 // 2, 16 * q - 1, 16 * q, 81 * q - 1, 81 * q, 60000]
    counts = [min(edges[i], 200000) if i < len(edges) else 5 for i in range(L)]
    dirs, w, off = _photons(L + H, counts)
    rc, e_ref, c_ref = orc.splat(dirs, w, off, H, W)
    assert rc == 0
    e = torch.full((L, H, W), -1, dtype=torch.int64, device=DEV)
    c = torch.full((L, H, W), -1, dtype=torch.int32, device=DEV) if count else None
    for acc in (False, True):
        npg.splat_histograms(ctx, _dev(dirs), _dev(w), _dev(off), H, W, energy=e, count=c, want_count=count,
                             accumulate=acc)
    assert npg.sync_status(ctx) == 0
    assert np.array_equal(e.cpu().numpy().view(np.uint64), 2 * e_ref)
    assert not count or np.array_equal(c.cpu().numpy().view(np.uint32), 2 * c_ref)


def test_fused_cuts_as_before(ctx, npg):
    """300 leaves, two of them large: the fused call cuts, the splat alone does not; the same tables."""
    L = 300
    counts = [90000 if k in (7, 211) else 200 + k for k in range(L)]
    dirs, w, off = _photons(5, counts)
    d, ww, o = _dev(dirs), _dev(w), _dev(off)
    m = npg.Model(ctx, synth.unet_model(3))
    e, _ = npg.splat_histograms(ctx, d, ww, o, 64, 64, want_count=False)
    ref = npg.build_cdf(ctx, npg.reconstruct_density(ctx, m, e, "bf16"))
    t = npg.reconstruct_fused(ctx, m, d, ww, o, 64, 64, "bf16")
    assert npg.sync_status(ctx) == 0
    for k in ("pdf", "marg", "cond", "total"):
        assert torch.equal(getattr(t, k), getattr(ref, k)), k
    m.free()
