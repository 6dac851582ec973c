"""GPU tests of the mixture sample's choice between the wavefront and the
lane-by-lane search on rows above 64 bins: query counts at and below 900 thousand,
tables on either side of 6 and 16 MiB.  Both searches give the bin that bisection
gives, so a guided sample's direction and pdf are those of npg_sample_dirs on the
same uniforms, and its bin is numpy's: all exact."""
import numpy as np
import pytest
import torch

from paper_2010_01775_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("L,H,W,n", [
    (1, 1024, 1024, 1 << 18), (5, 512, 512, 899999), (6, 512, 512, 899999), (6, 512, 512, 900000),
    (96, 128, 128, (1 << 18) + 7), (252, 128, 128, 900063), (255, 128, 128, 900001), (4, 1024, 1024, 1 << 20),
])
def test_mis_search(ctx, npg, orc, L, H, W, n):
    rng = np.random.default_rng(L + W)
    rc, pdf, marg, cond, _ = orc.build_cdf(np.exp(rng.normal(0, 3, (L, H, W))))
    assert rc == 0
    pdf, marg, cond = (np.ascontiguousarray(a, dtype=np.float32) for a in (pdf, marg, cond))
    leaf = np.sort(rng.integers(0, L, n))
    u = synth.uniforms(rng, (n, 2)).astype(np.float32)
    row = np.empty(n, np.int64)
    ends = np.searchsorted(leaf, np.arange(L + 1))
    for k in range(L):
        q = slice(ends[k], ends[k + 1])
        row[q] = np.minimum(np.searchsorted(marg[k], u[q, 0], side="right") - 1, H - 1)
    order = np.argsort(leaf * H + row, kind="stable")
    ends = np.searchsorted((leaf * H + row)[order], np.arange(L * H + 1))
    col = np.empty(n, np.int64)
    for k in np.flatnonzero(np.diff(ends)):
        q = order[ends[k]:ends[k + 1]]
        col[q] = np.minimum(np.searchsorted(cond[k // H, k % H], u[q, 1], side="right") - 1, W - 1)
    mix = rng.permutation(n)  # neighbouring queries ask different leaves
    leaf, u, want = leaf[mix], u[mix], (row * W + col)[mix]

    tabs = npg.CdfTables(*(torch.from_numpy(t).to(DEV) for t in (pdf, marg, cond)), None)
    lf, ud = torch.from_numpy(leaf.astype(np.int32)).to(DEV), torch.from_numpy(u).to(DEV)
    d, p, b = npg.sample_dirs(ctx, tabs, lf, ud)
    assert npg.sync_status(ctx) == 0
    assert np.array_equal(b.cpu().numpy(), want)
    # alpha 0.25, and a normal whose lobe is zero on the sampled side: pdf = 0.75 g
    first = torch.from_numpy(np.where(np.arange(n) % 3 == 0, 0.1, 0.7).astype(np.float32)).to(DEV)
    d3, p3, st = npg.sample_mis(ctx, tabs, torch.full((L,), 0.25, device=DEV), lf, -d,
                                torch.cat([first[:, None], ud], 1))
    assert npg.sync_status(ctx) == 0
    g = first >= 0.25
    assert torch.equal(st == 0, g)
    assert torch.equal(d3[g], d[g])
    assert torch.equal(p3[g], 0.75 * p[g])
    assert torch.equal(p.cpu(), torch.from_numpy(pdf.reshape(L, -1)[leaf, want]))
