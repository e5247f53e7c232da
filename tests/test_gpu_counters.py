"""Counters of a single call's bins: several per tile, chosen by the key pass's block and
spread over memory.  Row counts around the key pass's blocks, grids of few and of many
tiles and plane counts that leave room for one, some or all of the counters, one or two
images, against the FP64 oracle.  FP32 sums of at most a few thousand weighted taps per cell
stay within 1e-5 of the peak."""

import numpy as np
import pytest

from gpu_util import oracle_grid, run_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agg", [False, True])
@pytest.mark.parametrize("n,tile,n_w", [(32, 32, 9), (48, 16, 2), (250, 16, 33), (1040, 16, 9)])
@pytest.mark.parametrize("images", [1, 2])
def test_counters(n, tile, n_w, images, agg):
    params = dict(n=n, cell_rad=1e-4, n_wplanes=n_w, w_max=50.0, support=5, oversample=8, kernel_image_size=32,
                  precision="f32", n_images=images, algorithm="tiled", tile=tile, chunk=256, bin_aggregate=agg)
    for nvis in (1, 511, 512, 513, 2047, 2048, 2049, 9000):
        rng = np.random.default_rng(nvis)
        fov = n * params["cell_rad"]
        # half of the rows in the middle tile, runs of three equal rows
        uv = rng.uniform(-0.5, 0.5, (nvis, 2)) * n / fov
        uv[::2] *= 0.02
        uv = np.repeat(uv, 3, axis=0)[:nvis]
        uvw = np.concatenate([uv, rng.uniform(-50, 50, (nvis, 1))], axis=1)
        vis = rng.standard_normal(nvis) + 1j * rng.standard_normal(nvis)
        wt = rng.uniform(0.25, 2.0, nvis)
        offs = [0, nvis // 3, nvis] if images == 2 else None
        G, sw, cnt, host = run_grid(params, uvw, vis, wt, offs)
        (Gr, swr, cr), _, _ = oracle_grid(params, host, offs)
        assert cnt.tolist() == cr.tolist()
        assert np.allclose(sw, swr, rtol=1e-12, atol=0)
        assert np.abs(G - Gr).max() <= 1e-5 * max(np.abs(Gr).max(), 1e-30)
