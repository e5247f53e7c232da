"""A tuned handle is no slower on calls of few rows than an untuned one of the same tile: neither
tuned on them nor tuned on many rows and then called with few.  (Work items of 1024 records and
more, the tuner's fixed lengths, take the gridder three times as long here, so the tests allow
half as much again.)"""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from oracle import wproj_ref as R

from gpu_util import rel_max

pytestmark = pytest.mark.gpu


def _rows(nvis, n):
    rng = np.random.default_rng(nvis)
    cells = n / 2 + rng.standard_normal((nvis, 2)) * 3.0  # a few busy tiles
    uvw = np.concatenate([(cells - n / 2) / 0.02, rng.uniform(-50, 50, (nvis, 1))], axis=1)
    vis = rng.standard_normal(nvis) + 1j * rng.standard_normal(nvis)
    return torch.as_tensor(uvw).cuda(), torch.as_tensor(vis).cuda(), torch.ones(nvis, dtype=torch.float64).cuda()


def _grid_us(k, rows):
    g, ws = k.new_grid(), k.workspace(len(rows[0]))
    best = 1e9
    for i in range(30):
        g.zero_()
        k.profile(True)
        W.grid(k, *rows, g, workspace=ws)
        best = min(best, 1e3 * k.profile_read()["grid"][0])
        k.profile(False)
    return best, g.cpu().numpy()


@pytest.mark.parametrize("tuned_on", [20000, 1100000])
def test_tuned_few_rows(tuned_on):
    n = 252
    params = dict(n=n, cell_rad=0.02 / n, n_wplanes=8, w_max=50.0, support=7, oversample=8, kernel_image_size=32,
                  precision="f64", n_images=1, algorithm="tiled")
    few = _rows(20000, n)
    k = W.make_kernels(params)
    tile, chunk = W.autotune(k, *_rows(tuned_on, n))
    assert tile in (16, 32, 64) and chunk in (1024, 2048, 4096, 8192, 16384)
    tuned, g = _grid_us(k, few)
    plain = W.make_kernels({**params, "tile": tile})
    untuned, _ = _grid_us(plain, few)
    assert tuned <= 1.5 * untuned
    plan = R.Plan(params)
    ref = R.grid(plan, R.kernel_tables(plan), *(t.cpu().numpy() for t in few))[0]
    assert rel_max(g, ref) < 1e-12
    k.free()
    plain.free()


def test_tuned_stable_bins_reproduce():
    """A stable handle's length stays what it was tuned to: two handles of one shape agree bit for bit."""
    n = 244
    params = dict(n=n, cell_rad=0.02 / n, n_wplanes=8, w_max=50.0, support=7, oversample=8, kernel_image_size=32,
                  precision="f32", n_images=1, algorithm="tiled", stable_bins=True)
    u, v, w = _rows(20000, n)
    rows = u, v.to(torch.complex64), w.float()
    out = []
    for _ in range(2):
        k = W.make_kernels(params)
        W.autotune(k, *rows)
        for _ in range(2):
            g = k.new_grid()
            W.grid(k, *rows, g)
            out.append(g.cpu().numpy())
        k.free()
    assert all(np.array_equal(out[0], o) for o in out[1:])
