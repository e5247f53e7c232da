"""Image transforms at every side the library transforms itself (powers of two from 128 to
4096) and at neighbours that go through rocFFT, in each direction, with and without
w-stacking, against the FP64 oracle (FP32 image -> grid and image -> layers are rocFFT's).  Rounding errors of a transform over 2^22 .. 2^24 values
are a few eps of the transform's RMS, below 2e-6 of its peak in FP32 and 1e-14 in FP64; the
grid correction multiplies value and error alike."""

import numpy as np
import pytest
import torch

import paper_1905_03213_amd as W
from gpu_util import CDT, RDT, rel_max
from oracle import wproj_ref as R

pytestmark = pytest.mark.gpu
TOL = {"f32": 2e-6, "f64": 1e-14}


def _own_kappa(k, monkeypatch):
    """The handle's correction factors, also for the oracle: they are tested by themselves, and
    their rounding is far above FP64's in the transform."""
    kap = k.export(W._lib.EXPORT_KAPPA).view(torch.float64).cpu().numpy()
    monkeypatch.setattr(R, "kappa", lambda plan: kap)
    return kap


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,images", [(64, 2), (128, 1), (128, 3), (192, 2), (256, 2), (512, 2), (1024, 2),
                                      (2048, 1), (4096, 1)])
def test_image_transforms(n, images, prec, monkeypatch):
    params = dict(n=n, cell_rad=0.5 / n, n_wplanes=3, w_max=20.0, support=5, oversample=8, kernel_image_size=32,
                  precision=prec, n_images=images)
    plan = R.Plan(params)
    k = W.make_kernels(params)
    kap = _own_kappa(k, monkeypatch)
    kk = np.outer(kap, kap)[None]
    rng = np.random.default_rng(n + images)
    G = torch.as_tensor(rng.standard_normal((images, n, n)) + 1j * rng.standard_normal((images, n, n))).to(CDT[prec])
    exact = G.to(torch.complex128).numpy()
    sw = np.linspace(0.5, 90.0, images)
    sw[0] = 0.0 if images > 1 else 7.0
    img = torch.full((images * n * n + 1,), 7.0, dtype=RDT[prec], device="cuda")[1:].view(images, n, n)
    peak = np.abs(R.centred_idft(exact).real).max()
    for weights in (sw, None):
        g = G.cuda()
        W.image(k, W.GRID_TO_IMAGE if weights is not None else W.GRID_TO_IMAGE_RAW, g, img,
                None if weights is None else torch.as_tensor(weights).cuda())
        got = img.double().cpu().numpy()
        if weights is not None:  # no weight: an image of zeros
            assert images == 1 or not got[0].any()
            got = got * weights[:, None, None]
        ref = R.grid_to_image(plan, exact, None)
        first = 1 if weights is not None and images > 1 else 0
        assert np.all(np.abs(got - ref)[first:] <= TOL[prec] * peak * kk)
    I = torch.as_tensor(rng.standard_normal((images, n, n))).to(RDT[prec])
    img.copy_(I)
    g = torch.empty((images, n, n), dtype=CDT[prec], device="cuda")
    W.image(k, W.IMAGE_TO_GRID, g, img)
    assert rel_max(g.to(torch.complex128).cpu().numpy(), R.image_to_grid(plan, I.double().numpy())) <= TOL[prec]
    k.free()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,images,layers", [(64, 1, 3), (128, 2, 1), (256, 1, 7), (512, 2, 3), (1024, 1, 2),
                                             (2048, 1, 2), (4096, 1, 2)])
def test_stack_transforms(n, images, layers, prec, monkeypatch):
    params = dict(n=n, cell_rad=0.5 / n, n_wplanes=3, w_max=20.0, support=5, oversample=8, kernel_image_size=32,
                  precision=prec, n_images=images, w_mode="stack", n_wlayers=layers)
    plan = R.Plan(params)
    k = W.make_kernels(params)
    kap = _own_kappa(k, monkeypatch)
    rng = np.random.default_rng(n + layers)
    shape = (images * layers, n, n)
    G = torch.as_tensor(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).to(CDT[prec])
    img = torch.empty((images, n, n), dtype=RDT[prec], device="cuda")
    g = G.cuda()
    W.image(k, W.GRID_TO_IMAGE_RAW, g, img)
    exact = G.to(torch.complex128).numpy()
    # the layers' errors add at most linearly; the phases are good to 1e-14 of a turn's radian
    peak = sum(np.abs(R.centred_idft(exact[l::layers])).max() for l in range(layers))
    err = np.abs(img.double().cpu().numpy() - R.grid_to_image(plan, exact, None))
    assert np.all(err <= (TOL[prec] + 1e-13) * peak * np.outer(kap, kap)[None])
    I = torch.as_tensor(rng.standard_normal((images, n, n))).to(RDT[prec])
    W.image(k, W.IMAGE_TO_GRID, g, I.cuda())
    assert rel_max(g.to(torch.complex128).cpu().numpy(), R.image_to_grid(plan, I.double().numpy())) <= TOL[prec] + 1e-13
    k.free()
