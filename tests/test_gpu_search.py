"""GPU tests of the table searches behind npg_sample_dirs and npg_sample_mis:
rows at and above the shortest that the wavefront search takes, tables at
every 4-byte offset from a 64-byte boundary, densities so peaked that the
interpolated windows miss and bisection finishes, uniforms on, just below and
just above table entries, and calls whose last wavefront is ragged.  The bins
are integers and the pdf is the table's entry: both exact."""
import numpy as np
import pytest
import torch

from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _at(a, shift):
    """A device copy of `a` that starts `shift` floats into an allocation."""
    buf = torch.zeros(a.size + 64, dtype=torch.float32, device=DEV)
    t = buf[shift:shift + a.size].view(a.shape)
    t.copy_(torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)))
    return t


def _row(t, u):
    return int(np.searchsorted(t, u, side="right")) - 1


@pytest.mark.parametrize("L,H,W,shift,n", [
    (3, 8, 16, 0, 1000), (3, 16, 32, 1, 1000), (3, 32, 16, 2, 700), (5, 32, 64, 3, 4097), (2, 64, 128, 7, 4095),
    (2, 128, 32, 13, 1), (2, 256, 256, 15, 5000), (1, 512, 1024, 5, 5000),
    (70, 128, 128, 3, (1 << 18) + 5), (9, 512, 512, 6, 1 << 18),  # long rows, many queries, tables above 4 MiB
])
def test_search(ctx, npg, orc, L, H, W, shift, n):
    rng = np.random.default_rng(L * H + W)
    s = np.exp(rng.normal(0, 4, (L, H, W)))  # a few bins hold most of the mass
    s[0] = 1e-12
    s[0, H // 3, W - 1] = 1.0  # all of it in one bin
    rc, pdf, marg, cond, _ = orc.build_cdf(s)
    assert rc == 0
    pdf, marg, cond = (np.asarray(a, dtype=np.float32) for a in (pdf, marg, cond))
    leaf = rng.integers(0, L, n)
    u = synth.uniforms(rng, (n, 2)).astype(np.float32)
    below1 = np.nextafter(np.float32(1), np.float32(0))
    for k in range(n):  # entries and their neighbours
        if k % 4 == 3:
            continue
        i = rng.integers(0, H)
        e = np.float32([marg[leaf[k], i], 0])
        e[1] = cond[leaf[k], _row(marg[leaf[k]], min(e[0], below1)), rng.integers(0, W)]
        u[k] = np.clip(e if k % 4 == 0 else np.nextafter(e, np.float32(0 if k % 4 == 1 else 2)), 0, below1)
    want = np.empty(n, np.int64)
    for k in range(n):
        i = min(_row(marg[leaf[k]], u[k, 0]), H - 1)
        want[k] = i * W + min(_row(cond[leaf[k], i], u[k, 1]), W - 1)
    tabs = npg.CdfTables(_at(pdf, 0), _at(marg, shift), _at(cond, (3 * shift + 1) % 16), None)
    lf = torch.from_numpy(leaf.astype(np.int32)).to(DEV)
    d, p, b = npg.sample_dirs(ctx, tabs, lf, torch.from_numpy(u).to(DEV))
    assert npg.sync_status(ctx) == 0
    assert np.array_equal(b.cpu().numpy(), want)
    assert np.array_equal(p.cpu().numpy(), pdf.reshape(L, -1)[leaf, want])
    # the guided branch of the mixture takes the same bins: with alpha 0.2 and
    # a normal whose lobe is zero on the sampled side, pdf = (1 - a) g
    a = np.full(L, 0.2, np.float32)
    dn = d.cpu().numpy()
    u3 = np.concatenate([np.where(np.arange(n) % 3 == 0, 0.1, 0.7)[:, None], u], 1).astype(np.float32)
    d3, p3, st = npg.sample_mis(ctx, tabs, _at(a, 0), lf, torch.from_numpy(-dn).to(DEV), torch.from_numpy(u3).to(DEV))
    assert npg.sync_status(ctx) == 0
    g = u3[:, 0] >= 0.2
    assert np.array_equal(st.cpu().numpy() == 0, g)
    assert np.array_equal(d3.cpu().numpy()[g], dn[g])
    one = np.float32(1) - a[0]
    assert np.array_equal(p3.cpu().numpy()[g], one * pdf.reshape(L, -1)[leaf, want][g])
