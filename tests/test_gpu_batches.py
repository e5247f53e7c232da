"""The gridder's record batches: work items that end inside a batch or a group of records,
gridded directly and through a plan, against the FP64 oracle; and a visibility that is not
finite, which reaches the cells of its own footprint only."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from oracle import wproj_ref as R

from gpu_util import oracle_grid, rel_max, run_grid

pytestmark = pytest.mark.gpu

# FP32 sums of up to 65 weighted taps: 65 roundings of 6e-8 stay below 1e-5 of the peak;
# FP16 taps carry 5e-4 each.
TOL = {"f64": 1e-12, "f32": 1e-5, "f32_f16table": 1e-3}
COUNTS = (1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65)


def _params(S, prec):
    return dict(n=512, cell_rad=5e-5, n_wplanes=5, w_max=200.0, support=S, oversample=8, kernel_image_size=64,
                precision=prec, n_images=1, algorithm="tiled", tile=32, chunk=256)


def _rows(params, seed):
    """COUNTS[i] rows in tile i of a diagonal of 32-cell tiles."""
    rng = np.random.default_rng(seed)
    fov = params["n"] * params["cell_rad"]
    uvw = []
    for i, c in enumerate(COUNTS):
        cell = 32 * (i + 1) + rng.uniform(0, 32, (c, 2))
        uvw.append(np.concatenate([(cell - params["n"] / 2) / fov, rng.uniform(-200, 200, (c, 1))], axis=1))
    uvw = np.concatenate(uvw)
    vis = rng.standard_normal(len(uvw)) + 1j * rng.standard_normal(len(uvw))
    return uvw, vis, rng.uniform(0.25, 2.0, len(uvw))


@pytest.mark.parametrize("S", [3, 7, 8, 9, 12, 16])
@pytest.mark.parametrize("prec", list(TOL))
def test_item_lengths(S, prec):
    params = _params(S, prec)
    uvw, vis, wt = _rows(params, S)
    G, sw, cnt, host = run_grid(params, uvw, vis, wt)
    (Gr, swr, cr), _, _ = oracle_grid(params, host)
    assert rel_max(G, Gr) < TOL[prec]
    assert cnt.tolist() == cr.tolist() and abs(sw[0] - swr[0]) < 1e-9 * swr[0]
    k = W.make_kernels(params)
    plan = W.Plan(k, torch.as_tensor(host[0]).cuda(), torch.as_tensor(host[2]).to(k.real).cuda())
    g = k.new_grid()
    plan.grid(torch.as_tensor(host[1]).to(k.cplx).cuda(), g)
    assert rel_max(g.to(torch.complex128).cpu().numpy(), Gr) < TOL[prec]
    plan.free()
    k.free()


@pytest.mark.parametrize("S", [7, 8, 9])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_not_finite_visibility_stays_in_its_footprint(S, prec):
    params = _params(S, prec)
    uvw, vis, wt = _rows(params, 100 + S)
    vis = np.asarray(vis)
    bad = [len(vis) - 1, len(vis) - 40]  # the last record of the last item among them
    vis[bad[0]] = np.inf
    vis[bad[1]] = np.nan
    G = run_grid(params, uvw, vis, wt)[0][0]
    p = R.snap(R.Plan(params), uvw, wt)
    hit = np.zeros(G.shape, dtype=bool)
    for j in bad:
        hit[p["y0"][j]:p["y0"][j] + S, p["x0"][j]:p["x0"][j] + S] = True
    assert np.array_equal(~np.isfinite(G), hit)
