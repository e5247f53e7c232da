"""Single degridding calls with supports above 8, on both sides of the rules for short work items
(rows per tile) and for bins that keep the planes (counters a bin, copies a CU holds), untuned and tuned,
with exactly the workspace that the library asks for, against the FP64 oracle."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from gpu_util import CDT, RDT, rel_max
from oracle import cref
from oracle import wproj_ref as R

pytestmark = pytest.mark.gpu

# sums of up to 289 taps: 289 roundings of 6e-8 stay below 2e-5 of the peak; FP16 taps carry 5e-4
TOL = {"f64": 1e-12, "f32": 2e-5, "f32_f16table": 1e-3}


def _rows(n, nvis, seed):
    """Half of the rows in one tile; some footprints leave the grid."""
    rng = np.random.default_rng(seed)
    cells = n / 2 + rng.standard_normal((nvis, 2)) * np.where(rng.random((nvis, 1)) < 0.5, 2.0, n / 6)
    return np.concatenate([(cells - n / 2) / 0.02, rng.uniform(-90, 90, (nvis, 1))], axis=1), rng


def _check(params, nvis, tuned=False):
    n, prec = params["n"], params["precision"]
    plan = R.Plan(params)
    tabs = R.kernel_tables(plan)
    uvw, rng = _rows(n, nvis, nvis + params["support"])
    k = W.make_kernels(params)
    u = torch.as_tensor(uvw).cuda()
    ws = torch.empty(k.workspace_size(nvis), dtype=torch.uint8, device="cuda")
    if tuned:
        vis = torch.ones(nvis, dtype=CDT[prec], device="cuda")
        W.autotune(k, u, vis, torch.ones(nvis, dtype=RDT[prec], device="cuda"), workspace=ws)
    M = rng.standard_normal((plan.n_grids, n, n)) + 1j * rng.standard_normal((plan.n_grids, n, n))
    model = torch.as_tensor(M).to(CDT[prec])
    off = None if plan.n_images == 1 else np.sort(rng.integers(11, nvis - 11, plan.n_images + 1))
    ref = cref.degrid(plan, tabs, uvw, model.to(torch.complex128).numpy(), off, nthreads=8)
    out = torch.full((nvis,), 7.0, dtype=CDT[prec], device="cuda")
    W.degrid(k, u, model.cuda(), out, image_offsets=None if off is None else torch.as_tensor(off).cuda(), workspace=ws)
    got = out.to(torch.complex128).cpu().numpy()
    assert np.all(got[ref == 0] == 0)
    assert rel_max(got, ref) < TOL[prec]
    k.free()


# 96 cells: 36 tiles of 16, 9 of 32; 128 rows a tile are 4608 and 1152 rows
@pytest.mark.parametrize("nvis,tile", [(1, 16), (255, 32), (1151, 32), (1152, 32), (4607, 16), (4608, 16),
                                       (65537, 16), (200000, 32)])
@pytest.mark.parametrize("prec,S", [("f32", 9), ("f64", 16), ("f32_f16table", 10), ("f32", 17)])
def test_short_items(prec, S, nvis, tile):
    _check(dict(n=96, cell_rad=0.02 / 96, n_wplanes=3, w_max=80.0, support=S, oversample=8, kernel_image_size=32,
                precision=prec, n_images=1, algorithm="tiled", tile=tile), nvis)


# the planes are kept with 1, 2, .. 256 counters a bin (36 tiles of 16: 16 rows a counter and at most
# 65536), from 2^19 rows or 128 a tile on; one copy a CU (FP64 tiles of 64)
@pytest.mark.parametrize("nvis,planes,prec,S,tile", [
    (524287, 68, "f32", 12, 16), (524288, 68, "f32", 12, 16), (524288, 2, "f32", 9, 16), (600000, 7, "f32", 10, 32),
    (524288, 1, "f32", 9, 16), (4608, 4, "f64", 12, 16), (4608, 5, "f64", 12, 16), (30000, 2, "f64", 9, 32),
    (524287, 20, "f64", 9, 64), (524288, 20, "f64", 9, 64), (524288, 20, "f32", 9, 64),
])
def test_planes_kept(nvis, planes, prec, S, tile):
    _check(dict(n=96, cell_rad=0.02 / 96, n_wplanes=planes, w_max=80.0, support=S, oversample=8, kernel_image_size=32,
                precision=prec, n_images=1, algorithm="tiled", tile=tile), nvis)


@pytest.mark.parametrize("images,w_mode,layers", [(3, "linear", 1), (1, "fold", 1), (1, "fold_sqrt", 1), (1, "stack", 3)])
def test_planes_kept_modes(images, w_mode, layers):
    _check(dict(n=96, cell_rad=0.02 / 96, n_wplanes=6, w_max=80.0, support=13, oversample=8, kernel_image_size=32,
                precision="f64", n_images=images, algorithm="tiled", tile=16, w_mode=w_mode, n_wlayers=layers), 60000)


@pytest.mark.parametrize("prec,S,nvis,planes", [("f64", 9, 60000, 3), ("f32", 12, 524288, 9), ("f32", 17, 524288, 2)])
def test_planes_kept_aggregated(prec, S, nvis, planes):
    _check(dict(n=96, cell_rad=0.02 / 96, n_wplanes=planes, w_max=80.0, support=S, oversample=8, kernel_image_size=32,
                precision=prec, n_images=1, algorithm="tiled", tile=16, bin_aggregate=1), nvis)


@pytest.mark.parametrize("prec,S", [("f32", 9), ("f64", 13)])
def test_tuned(prec, S):
    _check(dict(n=128, cell_rad=0.02 / 128, n_wplanes=5, w_max=80.0, support=S, oversample=8, kernel_image_size=32,
                precision=prec, n_images=1, algorithm="tiled"), 300000, tuned=True)
