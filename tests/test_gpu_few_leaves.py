"""GPU tests of the forms that batches of few leaves take: a leaf's photons
shared by several workgroups, and the one-channel last layer of a CNN."""
import numpy as np
import pytest
import torch

from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _photons(seed, counts):
    rng = synth.rng_for(seed)
    n = int(sum(counts))
    dirs = synth.to_f32_dirs(synth.unit_vectors(rng, n)) if n else np.zeros((0, 3), np.float32)
    w = rng.integers(0, 2 ** 32, n, dtype=np.uint64).astype(np.uint32)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32)
    return dirs, w, off


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).to(DEV)


# counts about the slice size (2048) and its multiples; 512 leaf bands are the
# last batch cut into slices; 256x256 maps have four bands
@pytest.mark.parametrize("counts,H,W", [([0, 1, 2047, 2048, 4095, 4096, 4097, 200001], 32, 32),
                                        ([70000], 4, 8), ([131073], 128, 128), ([50000, 3, 9000], 256, 256),
                                        ([4100] * 512, 16, 16), ([4100] * 513, 16, 16)])
def test_splat_slices_exact(ctx, npg, orc, counts, H, W):
    dirs, w, off = _photons(len(counts) * H, counts)
    perm = np.random.default_rng(1).permutation(len(w)).astype(np.uint32)
    rc, e_ref, c_ref = orc.splat(dirs, w, off, H, W, perm=perm)
    assert rc == 0
    d, ww, o, p = torch.from_numpy(dirs).to(DEV), _i32(w), _i32(off), _i32(perm)
    e = torch.full((len(counts), H, W), -1, dtype=torch.int64, device=DEV)
    c = torch.full((len(counts), H, W), -1, dtype=torch.int32, device=DEV)
    npg.splat_histograms(ctx, d, ww, o, H, W, perm=p, energy=e, count=c)
    assert npg.sync_status(ctx) == 0
    assert np.array_equal(e.cpu().numpy().view(np.uint64), e_ref)
    assert np.array_equal(c.cpu().numpy().view(np.uint32), c_ref)
    npg.splat_histograms(ctx, d, ww, o, H, W, perm=p, energy=e, count=c, accumulate=True)
    npg.splat_histograms(ctx, d, ww, o, H, W, perm=p, energy=e, want_count=False, accumulate=True)
    assert npg.sync_status(ctx) == 0
    assert np.array_equal(e.cpu().numpy().view(np.uint64), e_ref * np.uint64(3))
    assert np.array_equal(c.cpu().numpy().view(np.uint32), c_ref * np.uint32(2))


# maps narrower and wider than the 8x8 tile, one to three 16-channel chunks;
# two layers leave the 1-channel layer's input stored
@pytest.mark.parametrize("H,W,L,channels", [(4, 64, 2, (1, 16, 1)), (64, 4, 1, (1, 16, 1)), (16, 16, 3, (1, 48, 1)),
                                            (8, 8, 5, (1, 32, 1)), (32, 64, 2, (1, 16, 16, 1))])
def test_last_layer_one_channel(ctx, npg, orc, H, W, L, channels):
    model = synth.cnn_model(H + W, channels=channels, random_bias=True)
    dirs, w, off = _photons(H * W + L, [700 * (k + 1) for k in range(L)])
    rc, e, _ = orc.splat(dirs, w, off, H, W)
    assert rc == 0
    rc, s_ref = orc.net_forward(model, orc.normalize_input(e))
    assert rc == 0
    m = npg.Model(ctx, model)
    s = npg.reconstruct_density(ctx, m, torch.from_numpy(e.view(np.int64)).to(DEV), "fp32").cpu().numpy()
    assert npg.sync_status(ctx) == 0
    # binary64 sums on both sides: the float32 output's rounding, twice
    assert np.max(np.abs(s - s_ref) / s_ref) < 2.0 ** -22
    m.free()


# rows of 1 to 64 lanes, one, four and eight pieces per thread, the last map
# held in registers (32,768 bins) and the first past it; rows past 256 columns
@pytest.mark.parametrize("H,W", [(4, 4), (4, 8), (16, 16), (64, 4), (8, 128), (32, 32), (32, 64), (64, 64), (128, 32),
                                 (128, 128), (256, 128), (128, 256), (256, 256), (8, 512), (1024, 4)])
def test_cdf_tables_every_form(ctx, npg, orc, H, W):
    s = synth.random_density(H * 7 + W, 5, H, W, zero_frac=0.3)
    s[1, H // 2] = 0.0  # a row without mass
    s[2] = 0.0
    s[2, H - 1, W - 1] = 1e-30  # all mass in the last bin
    s[3] = np.float32(3e38)  # a sum past the float32 range
    s[4, :, 0] = 1e-45  # float32's lowest value beside ordinary ones
    pdf, marg, cond, tot = orc.build_cdf(s)[1:5]
    t = npg.build_cdf(ctx, torch.from_numpy(s).to(DEV))
    assert npg.sync_status(ctx) == 0
    # one float32 rounding of binary64 values within a few roundings of each other
    for got, ref in ((t.pdf, pdf), (t.marg, marg), (t.cond, cond)):
        assert np.max(np.abs(got.cpu().numpy() - ref) / np.maximum(ref, 1e-30)) < 2.0 ** -22
    assert np.max(np.abs(t.total.cpu().numpy() - tot) / tot) < 1e-13
    m, c = t.marg.cpu().numpy(), t.cond.cpu().numpy()
    assert np.all(np.diff(m, axis=1) >= 0) and np.all(np.diff(c, axis=2) >= 0)
    assert np.all(m[:, 0] == 0) and np.all(m[:, -1] == 1) and np.all(c[..., 0] == 0) and np.all(c[..., -1] == 1)
    # unaligned caller buffers give the same tables; a bad leaf only its own
    def odd(x, fill):
        b = torch.full((x.numel() + 1,), fill, dtype=x.dtype, device=DEV)
        return b[1:].view(x.shape)
    o = npg.CdfTables(odd(t.pdf, 7.0), odd(t.marg, 7.0), odd(t.cond, 7.0), t.total.clone())
    s2 = odd(t.pdf, 0.0)
    s2.copy_(torch.from_numpy(s))
    npg.build_cdf(ctx, s2, out=o)
    assert npg.sync_status(ctx) == 0
    assert torch.equal(o.pdf, t.pdf) and torch.equal(o.marg, t.marg) and torch.equal(o.cond, t.cond)
    for k, v in ((0, float("nan")), (2, -1.0), (4, float("inf"))):
        s2[k, H - 1, W - 1] = v
    npg.build_cdf(ctx, s2, out=o)
    assert npg.sync_status(ctx) == npg.E_RANGE
    for k in range(5):
        if k in (0, 2, 4):
            assert torch.isnan(o.pdf[k]).all() and torch.isnan(o.cond[k]).all() and torch.isnan(o.marg[k]).all()
            assert o.total[k] == 0
        else:
            assert torch.equal(o.pdf[k], t.pdf[k]) and torch.equal(o.cond[k], t.cond[k])
