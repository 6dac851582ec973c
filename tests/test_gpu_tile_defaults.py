"""GPU test of the tile defaults: option tile_cap set to its default gives the
default tiles again."""
import pytest
import torch

from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _flops(npg, c, m, e, prec):
    c.conv_flops(reset=True)
    npg.reconstruct_density(c, m, e, prec)
    assert npg.sync_status(c) == 0
    return c.conv_flops(reset=True)


# enough leaves for 512-pixel tiles (64 x 4096 pixels = 512 of them); the first
# layer's operations on the tiles' halo tell their size
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
def test_default_restored(npg, prec):
    c = npg.Context(0)
    m = npg.Model(c, synth.unet_model(3))
    e = torch.from_numpy(synth.rng_for(8).integers(0, 1 << 20, (64, 64, 64))).to(DEV)
    if prec == "fp8":
        m.calibrate_fp8(e)
    fresh = _flops(npg, c, m, e, prec)
    seen = set()
    for cap in (1, 2, 8):
        c.set_option("tile_cap", cap)
        seen.add(_flops(npg, c, m, e, prec))
        c.set_option("tile_cap", 4)
        assert _flops(npg, c, m, e, prec) == fresh, cap
    assert len(seen) > 1  # the operations do tell
    m.free()
    c.close()
