"""Binning with up to 256 counters a bin (few tiles, many planes), at the edges of the rules on
counters and rows, and with the planes kept where they allow few counters: grid, weight sums and
counters, and predictions, against the FP64 oracle."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from gpu_util import CDT, rel_max, run_grid
from oracle import cref
from oracle import wproj_ref as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg", [False, True])
@pytest.mark.parametrize("n,tile,n_w,images,nvis", [
    (64, 32, 257, 1, 30000),      # 4 tiles, 256 counters each
    (64, 32, 255, 1, 30000),      # 1020 planes' bins: kept
    (256, 64, 64, 1, 100000),     # 16 tiles, 64 counters each
    (256, 16, 64, 1, 131071),     # 4096 counters for fewer than 16 rows a counter of 8192
    (256, 16, 64, 1, 131073),
    (256, 16, 65, 1, 600000),     # 16384 counters
    (120, 32, 40, 3, 200000),     # 48 tiles of three images
])
def test_many_counters(n, tile, n_w, images, nvis, agg):
    params = dict(n=n, cell_rad=0.02 / n, n_wplanes=n_w, w_max=50.0, support=4, oversample=4, kernel_image_size=32,
                  precision="f64", n_images=images, algorithm="tiled", tile=tile, bin_aggregate=agg)
    plan = R.Plan(params)
    tabs = R.kernel_tables(plan)
    rng = np.random.default_rng(nvis + n_w)
    # most rows in the middle tiles, in runs of three equal ones; some leave the grid
    cells = n / 2 + rng.standard_normal((nvis, 2)) * np.where(rng.random((nvis, 1)) < 0.7, 3.0, n / 5)
    uvw = np.concatenate([(cells - n / 2) / 0.02, rng.uniform(-55, 55, (nvis, 1))], axis=1)
    uvw = np.repeat(uvw, 3, axis=0)[:nvis]
    vis = rng.standard_normal(nvis) + 1j * rng.standard_normal(nvis)
    wt = rng.uniform(0.25, 2.0, nvis)
    wt[rng.random(nvis) < 0.02] = 0.0
    offs = [0, nvis // 3, nvis // 3, nvis] if images == 3 else None
    G, sw, cnt, host = run_grid(params, uvw, vis, wt, offs)
    Gr, swr, cr = cref.grid(plan, tabs, *host, offs, nthreads=8)
    assert cnt.tolist() == cr.tolist()
    assert np.allclose(sw, swr, rtol=1e-12, atol=0)
    # a cell's sum of up to nvis taps rounds like a random walk, 800 times 1e-16
    assert rel_max(G, Gr) < 1e-12
    k = W.make_kernels(params)
    M = torch.as_tensor(rng.standard_normal((images, n, n)) + 1j * rng.standard_normal((images, n, n)))
    out = torch.full((nvis,), 7.0, dtype=CDT["f64"], device="cuda")
    W.degrid(k, torch.as_tensor(uvw).cuda(), M.cuda(), out, image_offsets=None if offs is None else torch.as_tensor(offs).cuda())
    assert rel_max(out.cpu().numpy(), cref.degrid(plan, tabs, uvw, M.numpy(), offs, nthreads=8)) < 1e-12
    k.free()
