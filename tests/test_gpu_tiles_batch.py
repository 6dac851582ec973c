"""GPU tests of the convolution tiles at batch size: enough leaves that no tile is
made smaller for want of workgroups, so that the widths a batch takes (up to 512
pixels, 64 channels) are compared with each other and with a few leaves' small
tiles, bit for bit, in the FP32 mode and in the extended 8/16-bit form (ELU,
residual links, stored means) as well; and networks whose deepest level has one
row."""
import numpy as np
import pytest
import torch

from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _i64(e):
    return torch.from_numpy(e.view(np.int64)).to(DEV)


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).to(DEV)


def _photons(seed, counts):
    rng = synth.rng_for(seed)
    mu = synth.unit_vectors(rng, 2 * len(counts)).reshape(-1, 2, 3)
    d = np.concatenate([synth.two_lobe_mixture(rng, c, mu[i, 0], mu[i, 1]) for i, c in enumerate(counts)])
    return d, synth.photon_weights(rng, len(d)), np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32)


def _same_bits(ctx, run, ref, opts):
    """run() gives ref under every option value, each set back to its default."""
    for name, vals, back in opts:
        try:
            for v in vals:
                ctx.set_option(name, v)
                assert torch.equal(run(), ref), (name, v)
        finally:
            ctx.set_option(name, back)


# 260 leaves of 64x64: full tiles on the two upper levels, 32x32 1030 leaves: on
# three; 16x16 maps of 1030 leaves hold several leaves in a tile
@pytest.mark.parametrize("H,L,levels", [(64, 261, (16, 32, 64, 128)), (32, 1031, (16, 32, 64)), (16, 1031, (16, 64)),
                                        (128, 67, (32, 64))])
def test_fp32_tiles_equal_bits(ctx, npg, orc, H, L, levels):
    counts = [4000, 300, 9000, 2500, 20]
    d, w, off = _photons(H, counts)
    rc, e, _ = orc.splat(d, w, off, H, H)
    assert rc == 0
    model = synth.unet_model(H + 1, levels, random_bias=True)
    m = npg.Model(ctx, model)
    few = _i64(e)
    many = few.repeat(L // 5 + 1, 1, 1)[:L].contiguous()
    run = lambda: npg.reconstruct_density(ctx, m, many, "fp32")
    ref = run()
    _same_bits(ctx, run, ref, (("tile_cap", (1, 2, 8), 4), ("pool_outputs", (0,), 1), ("fuse_first", (0,), 1),
                               ("chunk_leaves", (7,), 0)))
    one = npg.reconstruct_density(ctx, m, few, "fp32")
    assert torch.equal(ref[:5], one) and torch.equal(ref[L // 5 * 5 - 5:L // 5 * 5], one)
    assert npg.sync_status(ctx) == 0
    rc, s_ref = orc.net_forward(model, orc.normalize_input(e))
    assert rc == 0
    rel = np.abs(one.cpu().numpy() - s_ref) / s_ref
    assert rel[s_ref >= 1e-6 * s_ref.reshape(5, -1).max(1)[:, None, None]].max() < 1e-5
    m.free()


# 301 leaves of 64x128: every level's tiles at their widest (32x64 x 32 channels,
# 16x32 x 64)
@pytest.mark.parametrize("paper", [True, False])
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_five_channels_equal_bits(ctx, npg, orc, paper, prec):
    H, W, L = 64, 128, 301
    counts = [16384, 12000, 20000]
    d, w, off = _photons(17, counts)
    half = np.concatenate([np.arange(off[i], off[i] + counts[i] // 2) for i in range(3)]).astype(np.int64)
    rc, e, c = orc.splat(d, w, off, H, W)
    rc2, ep, cp = orc.splat(d[half], w[half], (off // 2).astype(np.uint32), H, W)
    assert rc == 0 and rc2 == 0
    model = synth.paper_unet_model(18, (16, 32, 64), random_bias=True) if paper else \
        synth.unet5_model(18, (16, 32, 64), random_bias=True)
    m = npg.Model(ctx, model)
    few = (_i64(e), _i32(c), _i64(ep), _i32(cp))
    many = [t.repeat(L // 3 + 1, 1, 1)[:L].contiguous() for t in few]
    run = lambda: npg.reconstruct_density5(ctx, m, *many, prec)
    ref = run()
    _same_bits(ctx, run, ref, (("tile_cap", (1, 2, 8), 4), ("pool_outputs", (0,), 1), ("chunk_leaves", (7,), 0)))
    npg.autotune(ctx, m, H, W, prec, probe_leaves=L)  # probed on tiles of every width
    assert torch.equal(run(), ref)
    one = npg.reconstruct_density5(ctx, m, *few, prec)
    assert torch.equal(ref[:3], one) and torch.equal(ref[297:300], one)
    assert npg.sync_status(ctx) == 0
    rc, s_ref = orc.net_forward5(model, orc.input5(e, ep, c, cp))
    assert rc == 0
    s = one.cpu().numpy().astype(np.float64)
    if prec == "fp32":
        big = s_ref >= 1e-6 * s_ref.reshape(3, -1).max(1)[:, None, None]
        assert (np.abs(s - s_ref) / np.maximum(s_ref, 1e-300))[big].max() < 1e-5
    else:  # the bar of the smaller five-channel tests
        pn, qn = (x / x.reshape(3, -1).sum(1)[:, None, None] for x in (s, s_ref))
        assert np.abs(pn - qn).reshape(3, -1).sum(1).max() < 5e-2
    m.free()


# deepest levels of one row: 1x4, 1x1 and 1x16
@pytest.mark.parametrize("prec", ["bf16", "fp8", "fp32"])
@pytest.mark.parametrize("levels,H,W", [((16, 32, 64), 4, 16), ((16, 16, 32), 4, 4), ((16, 32, 32), 4, 64)])
def test_one_row_levels(ctx, npg, orc, prec, levels, H, W):
    rng = synth.rng_for(H + W)
    e = (rng.random((9, H, W)) ** 8 * 1e7).astype(np.uint64) + 1
    model = synth.unet_model(W, levels, random_bias=True)
    m = npg.Model(ctx, model)
    if prec == "fp8":
        m.calibrate_fp8(_i64(e))
    ref = npg.reconstruct_density(ctx, m, _i64(e), prec)
    _same_bits(ctx, lambda: npg.reconstruct_density(ctx, m, _i64(e), prec), ref,
               (("tile_cap", (1, 2, 8), 4), ("pool_outputs", (0,), 1), ("chunk_leaves", (2,), 0)))
    assert npg.sync_status(ctx) == 0
    rc, s_ref = orc.net_forward(model, orc.normalize_input(e))
    assert rc == 0
    s = ref.cpu().numpy().astype(np.float64)
    l1 = np.abs(s - s_ref).reshape(9, -1).sum(1) / s_ref.reshape(9, -1).sum(1)
    # the bars of the other tile tests on such maps; 1e-5 a bin in the FP32 mode
    assert l1.max() < {"bf16": 0.1, "fp8": 0.6, "fp32": 1e-5}[prec], l1
    m.free()
