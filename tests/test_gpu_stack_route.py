"""Few small w-stacking layers go through rocFFT (transforms, then a correction pass), enough
pixels through the library's own transforms (no correction pass), and both give the oracle's
image.  Tolerance: rounding of a transform over up to 2^20 values, 2e-6 of its peak in FP32 and
1e-14 in FP64, a layer's errors adding at most linearly."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from gpu_util import CDT, RDT
from oracle import wproj_ref as R

pytestmark = pytest.mark.gpu
TOL = {"f32": 2e-6, "f64": 1e-14}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,images,layers,own", [(128, 1, 3, False), (128, 48, 2, True), (256, 2, 4, False),
                                                 (256, 11, 1, False), (256, 12, 1, True), (512, 2, 2, False),
                                                 (512, 3, 3, True), (1024, 1, 2, True)])
def test_stack_transform_route(n, images, layers, own, prec, monkeypatch):
    params = dict(n=n, cell_rad=0.5 / n, n_wplanes=3, w_max=20.0, support=5, oversample=8, kernel_image_size=32,
                  precision=prec, n_images=images, w_mode="stack", n_wlayers=layers)
    plan = R.Plan(params)
    k = W.make_kernels(params)
    kap = k.export(W._lib.EXPORT_KAPPA).view(torch.float64).cpu().numpy()
    monkeypatch.setattr(R, "kappa", lambda plan: kap)
    rng = np.random.default_rng(n + layers)
    shape = (images * layers, n, n)
    G = torch.as_tensor(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to(CDT[prec])
    img = torch.empty((images, n, n), dtype=RDT[prec], device="cuda")
    k.profile(True)
    W.image(k, W.GRID_TO_IMAGE_RAW, G.cuda(), img)
    phases = k.profile_read()
    assert phases["correct"][1] == (0 if own else 1)
    exact = G.to(torch.complex128).numpy()
    peak = sum(np.abs(R.centred_idft(exact[l::layers])).max() for l in range(layers))
    err = np.abs(img.double().cpu().numpy() - R.grid_to_image(plan, exact, None))
    assert np.all(err <= (TOL[prec] + 1e-13) * peak * np.outer(kap, kap)[None])
    k.free()
