"""The workspace need: no larger than what programs were told before work queues and spread counters
were laid out (the sizes below), and a call writes nothing beyond it."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from gpu_util import CDT, RDT, rel_max
from oracle import cref
from oracle import wproj_ref as R

pytestmark = pytest.mark.gpu

SIZES = [  # parameters, bytes for 1, 777 and 20000 rows
    (dict(n=32, n_wplanes=9, support=5), (84992, 106496, 1347584)),
    (dict(n=48, n_wplanes=2, support=7), (89600, 111104, 1393920)),
    (dict(n=250, n_wplanes=33, support=8, n_images=3), (1512448, 3511808, 4130304)),
    (dict(n=300, n_wplanes=23, support=9, tile=32), (724992, 1774592, 2441472)),
    (dict(n=128, n_wplanes=4, support=16, tile=64, precision="f32_f16table"), (111104, 535552, 1769216)),
    (dict(n=96, n_wplanes=5, support=4, w_mode="stack", n_wlayers=3), (82944, 499456, 1720064)),
    (dict(n=100, n_wplanes=8, support=5, stable_bins=True), (88320, 233216, 1789696)),
    (dict(n=64, n_wplanes=257, support=4, tile=32), (84992, 114432, 1326848)),
    (dict(n=64, n_wplanes=16, support=24), (132352, 244480, 1922304)),
]
TOL = {"f32": 2e-5, "f32_f16table": 1e-3}


@pytest.mark.parametrize("extra,sizes", SIZES)
def test_workspace_need(extra, sizes):
    params = dict(cell_rad=1e-5, w_max=50.0, oversample=4, kernel_image_size=64, precision="f32", n_images=1,
                  algorithm="tiled")
    params.update(extra)
    prec, n, ni = params["precision"], params["n"], params["n_images"]
    plan = R.Plan(params)
    tabs = R.kernel_tables(plan)
    k = W.make_kernels(params)
    for i, nvis in enumerate((1, 777, 20000)):
        need = k.workspace_size(nvis)
        assert need <= sizes[i]
        rng = np.random.default_rng(nvis)
        cells = n / 2 + rng.standard_normal((nvis, 2)) * n / 8
        uvw = np.concatenate([(cells - n / 2) / (n * 1e-5), rng.uniform(-50, 50, (nvis, 1))], axis=1)
        vis = torch.as_tensor(rng.standard_normal(nvis) + 1j * rng.standard_normal(nvis)).to(CDT[prec])
        wt = torch.as_tensor(rng.uniform(0.5, 1.5, nvis)).to(RDT[prec])
        off = np.array([0, nvis // 3, nvis // 2, nvis]) if ni == 3 else None
        o = None if off is None else torch.as_tensor(off).cuda()
        buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        g = k.new_grid()
        sw = torch.zeros(ni, dtype=torch.float64, device="cuda")
        u = torch.as_tensor(uvw).cuda()
        W.grid(k, u, vis.cuda(), wt.cuda(), g, image_offsets=o, weight_sum=sw, workspace=buf[:need])
        ref, swr, _ = cref.grid(plan, tabs, uvw, vis.to(torch.complex128).numpy(), wt.double().numpy(), off)
        assert rel_max(g.to(torch.complex128).cpu().numpy(), ref) < TOL[prec]
        assert np.allclose(sw.cpu().numpy(), swr, rtol=1e-12, atol=0)
        out = torch.empty_like(vis).cuda()
        model = torch.as_tensor(ref).to(CDT[prec])
        W.degrid(k, u, model.cuda(), out, image_offsets=o, workspace=buf[:need])
        pred = cref.degrid(plan, tabs, uvw, model.to(torch.complex128).numpy(), off)
        assert rel_max(out.to(torch.complex128).cpu().numpy(), pred) < TOL[prec]
        assert bool((buf[need:] == 0xA5).all())
    k.free()
