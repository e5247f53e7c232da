"""Per-plane supports in one, two and four passes of 64 taps and beyond, alone and mixed
inside a batch of records, gridded directly and through a plan, against the FP64 oracle."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from oracle import wproj_ref as R

from gpu_util import oracle_grid, rel_max, run_grid

pytestmark = pytest.mark.gpu

# FP32 sums of up to 200 weighted taps: 200 roundings of 6e-8 stay below 2e-5 of the peak;
# FP16 taps carry 5e-4 each.
TOL = {"f64": 1e-12, "f32": 2e-5, "f32_f16table": 1e-3}


@pytest.mark.parametrize("supports", [[8, 1, 5, 8, 2], [9, 11, 9, 10, 11], [12, 16, 13, 14, 15], [17, 24, 32, 20, 18],
                                      [7, 9, 8, 16, 4], [11, 12, 3, 8, 9], [16, 17, 8, 1, 32]])
@pytest.mark.parametrize("prec", list(TOL))
@pytest.mark.parametrize("tile", [16, 32])
def test_mixed_supports(supports, prec, tile):
    n = 256
    params = dict(n=n, cell_rad=5e-5, n_wplanes=5, w_max=200.0, support_per_plane=supports, support=max(supports),
                  oversample=4, kernel_image_size=64, precision=prec, n_images=1, algorithm="tiled", tile=tile,
                  chunk=256)
    rng = np.random.default_rng(sum(supports))
    fov = n * params["cell_rad"]
    uvw = []
    for i, c in enumerate((1, 15, 16, 17, 31, 32, 33, 64, 65, 200)):
        cell = 24 + 20 * i + rng.uniform(0, 4, (c, 2))
        # planes one after the other, in runs of 1 .. c rows, and at random
        w = rng.integers(-2, 3, c) * 100.0 if i % 2 else np.sort(rng.integers(-2, 3, c) * 100.0)
        uvw.append(np.concatenate([(cell - n / 2) / fov, w[:, None]], axis=1))
    uvw = np.concatenate(uvw)
    vis = rng.standard_normal(len(uvw)) + 1j * rng.standard_normal(len(uvw))
    wt = rng.uniform(0.25, 2.0, len(uvw))
    G, sw, cnt, host = run_grid(params, uvw, vis, wt)
    (Gr, swr, cr), _, _ = oracle_grid(params, host)
    assert cnt.tolist() == cr.tolist()
    assert rel_max(G, Gr) < TOL[prec]
    k = W.make_kernels(params)
    plan = W.Plan(k, torch.as_tensor(host[0]).cuda(), torch.as_tensor(host[2]).to(k.real).cuda())
    g = k.new_grid()
    plan.grid(torch.as_tensor(host[1]).to(k.cplx).cuda(), g)
    assert rel_max(g.to(torch.complex128).cpu().numpy(), Gr) < TOL[prec]
    plan.free()
    k.free()
