"""Gridding and degridding with one work queue (large sub-kernels, many rows a work item) and with
16 (many small items), directly and through a plan, against the FP64 oracle."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from gpu_util import CDT, RDT, rel_max
from oracle import cref
from oracle import wproj_ref as R

pytestmark = pytest.mark.gpu

# FP32: an item's partial sums over up to 2048 records round like a random walk, 45 times 6e-8,
# and predictions sum up to 400 taps, 20 times 6e-8: below 2e-5 of the peak.  FP16 taps carry 5e-4.
TOL = {"f64": 1e-12, "f32": 2e-5, "f32_f16table": 1e-3}


@pytest.mark.parametrize("prec,S,n,images,tile", [
    ("f64", 16, 256, 1, 16),            # one queue in gridder and degridder
    ("f64", 12, 256, 1, 32),            # one in the degridder
    ("f32", 16, 320, 1, 32),
    ("f32_f16table", 20, 256, 1, 16),   # general gridder
    ("f64", 13, 128, 300, 16),          # 16 queues: many small items
    ("f32", 16, 128, 300, 16),
])
def test_queues_of_many_rows(prec, S, n, images, tile):
    nvis = (1 << 20) + 77
    params = dict(n=n, cell_rad=0.02 / n, n_wplanes=3, w_max=50.0, support=S, oversample=4, kernel_image_size=64,
                  precision=prec, n_images=images, algorithm="tiled", tile=tile)
    plan = R.Plan(params)
    tabs = R.kernel_tables(plan)
    rng = np.random.default_rng(S + images)
    # dense in the middle, a few rows off the grid
    cells = n / 2 + rng.standard_normal((nvis, 2)) * n / 8
    uvw = np.concatenate([(cells - n / 2) / 0.02, rng.uniform(-50, 50, (nvis, 1))], axis=1)
    off = np.sort(rng.integers(0, nvis + 1, images - 1))
    off = np.concatenate([[0], off, [nvis]]) if images > 1 else None
    k = W.make_kernels(params)
    vis = torch.as_tensor(rng.standard_normal(nvis) + 1j * rng.standard_normal(nvis)).to(CDT[prec])
    wt = torch.as_tensor(rng.uniform(0.5, 1.5, nvis)).to(RDT[prec])
    u, v, w = torch.as_tensor(uvw).cuda(), vis.cuda(), wt.cuda()
    o = None if off is None else torch.as_tensor(off).cuda()
    ref = cref.grid(plan, tabs, uvw, vis.to(torch.complex128).numpy(), wt.double().numpy(), off, nthreads=8)[0]
    g = k.new_grid()
    W.grid(k, u, v, w, g, image_offsets=o)
    assert rel_max(g.to(torch.complex128).cpu().numpy(), ref) < TOL[prec]
    M = (rng.standard_normal(ref.shape) + 1j * rng.standard_normal(ref.shape))
    model = torch.as_tensor(M).to(CDT[prec])
    pred = cref.degrid(plan, tabs, uvw, model.to(torch.complex128).numpy(), off, nthreads=8)
    out = torch.full((nvis,), 7.0, dtype=CDT[prec], device="cuda")
    W.degrid(k, u, model.cuda(), out, image_offsets=o)
    assert rel_max(out.to(torch.complex128).cpu().numpy(), pred) < TOL[prec]
    p = W.Plan(k, u, w, image_offsets=o)
    for _ in range(2):
        g.zero_()
        p.grid(v, g)
        assert rel_max(g.to(torch.complex128).cpu().numpy(), ref) < TOL[prec]
        out.fill_(7.0)
        p.degrid(model.cuda(), out)
        assert rel_max(out.to(torch.complex128).cpu().numpy(), pred) < TOL[prec]
    p.free()
    k.free()
