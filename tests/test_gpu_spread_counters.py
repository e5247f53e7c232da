"""Counters of the planes' bins spread over cache lines with skewed rows, at the edges of the rule
and of the rows of 256, where a row of tiles holds a divisor or a multiple of 256 bins: plans keep
every row once, in its bin, and grid and predict as the FP64 oracle."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from gpu_util import rel_max
from oracle import cref
from oracle import wproj_ref as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stable", [False, True])
@pytest.mark.parametrize("n,n_w,images", [
    (256, 15, 1), (256, 16, 1),   # 3840 and 4096 counters
    (256, 17, 1),
    (512, 32, 1),                 # 1024 bins in a row of tiles
    (250, 33, 2), (1040, 9, 1),
    (1024, 64, 1), (1024, 65, 1),  # 2^18 counters, and more
])
def test_spread_counters(n, n_w, images, stable):
    nvis = 30011
    params = dict(n=n, cell_rad=0.02 / n, n_wplanes=n_w, w_max=50.0, support=5, oversample=2, kernel_image_size=32,
                  precision="f64", n_images=images, algorithm="tiled", stable_bins=stable)
    plan = R.Plan(params)
    tabs = R.kernel_tables(plan)
    rng = np.random.default_rng(n + n_w)
    # half of the rows in a column of tiles
    cells = n / 2 + rng.standard_normal((nvis, 2)) * np.where(rng.random((nvis, 1)) < 0.5, [[2.0, n / 6]], n / 6)
    uvw = np.concatenate([(cells - n / 2) / 0.02, rng.uniform(-55, 55, (nvis, 1))], axis=1)
    vis = rng.standard_normal(nvis) + 1j * rng.standard_normal(nvis)
    wt = rng.uniform(0.25, 2.0, nvis)
    wt[rng.random(nvis) < 0.02] = 0.0
    offs = [0, nvis // 3, nvis] if images == 2 else None
    u, v, w = (torch.as_tensor(a).cuda() for a in (uvw, vis, wt))
    k = W.make_kernels(params)
    p = W.Plan(k, u, w, image_offsets=None if offs is None else torch.as_tensor(offs).cuda())
    got = p.rows().cpu().numpy().view(np.uint32)
    geo = R.snap(plan, uvw, wt)["valid"]
    kept = got[got != 0xFFFFFFFF]
    assert np.array_equal(np.sort(kept), np.flatnonzero(geo))
    G, swr, _ = cref.grid(plan, tabs, uvw, vis, wt, offs, nthreads=8)
    g = k.new_grid()
    p.grid(v, g)
    assert rel_max(g.cpu().numpy(), G) < 1e-12
    out = torch.empty_like(v)
    p.degrid(torch.as_tensor(G).cuda(), out)
    pred = np.where(geo, cref.degrid(plan, tabs, uvw, G, offs, nthreads=8), 0.0)
    assert rel_max(out.cpu().numpy(), pred) < 1e-12
    p.free()
    k.free()
