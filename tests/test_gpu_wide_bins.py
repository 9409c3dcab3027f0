"""TOF weights at the ends of a bin's support, where they are smallest: never
below zero (the count kernels' fixed-point sheets hold nonnegative shares, and a
bin without background must not get a negative mean), against the FP64 oracle.

2D views along y whose outermost rows lie a hundredth of a table interval inside
the support of the middle bin, for bins of 2 to 250 sigma; few bins have counts,
so that the outermost cells receive nothing but such samples.

Tolerance: the gradient's part that depends on the image to 1e-5 of the norm of
its summands (as for the other geometries of the zero-count-aware path).
"""

import numpy as np
import pytest
import torch

from oracle import recon
from synth import configs

pytestmark = pytest.mark.gpu

SIGMA, NSIGMA, ROWS = 2.0, 3.0, 21
TABLE = 1536  # intervals of the count kernels' table over half the support


def _config(ratio, nsigma=NSIGMA, inside=0.01):
    width = ratio * SIGMA
    support = 0.5 * width + nsigma * SIGMA
    row = support * (1.0 - inside / TABLE) / ((ROWS - 1) // 2)  # the outermost rows' distance, in rows
    return configs.get("mini_2d", nx=9, ny=ROWS, vx=row, vy=row, n_views=4, n_rad=7, rad_spacing=row,
                       half_length=2.0 * support, n_tof=3, tof_bin=width, tof_sigma=SIGMA, tof_nsigma=nsigma,
                       n_subsets=1)


@pytest.mark.parametrize("ratio", [2.0, 12.0, 40.0, 250.0])
def test_counts_gradient_at_the_ends_of_the_support(ratio):
    import paper_2506_04976_amd as pm
    cfg = _config(ratio)
    dev = torch.device("cuda:0")
    geom = pm.Geometry(cfg)
    shape = (cfg["n_views"], cfg["n_rad"], 1, cfg["n_tof"])
    y = np.zeros(shape, np.uint8)
    y[0, ::2, 0, 1] = 3  # view 0 runs along y
    r = np.full(shape, 0.5, np.float32)
    mult = np.ones(shape[:3], np.float32)
    x_np = np.random.default_rng(3).uniform(0.5, 1.5, (1, cfg["ny"], cfg["nx"])).astype(np.float32)

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a).ravel()).to(dev)

    x, counts = t(x_np), pm.Counts(geom, t(y), t(r), t(mult))
    got = torch.full((geom.n_vox,), float("nan"), device=dev)
    pm.pet_subset_grad_counts(geom, counts, 0, x, None, got)
    prob = recon.Problem(cfg, y, r, mult, beta=1.0, gamma=2.0, eps=1.0)
    xo = x_np.astype(np.float64)
    want = -prob.back(prob.a[0] * prob.y[0] / prob.ybar(xo, 0), 0)
    err = np.linalg.norm(got.cpu().double().numpy() - want.ravel()) / np.linalg.norm(want)
    print(f"\n[wide bins] {ratio} sigma: error {err:.2e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("nsigma", [2.5, 4.0, 5.0])
@pytest.mark.parametrize("ratio", [2.0, 12.0])
def test_dense_weights_at_the_ends_of_the_support(ratio, nsigma):
    # an image (a sinogram) that only such samples meet: no bin's mean (no voxel) below zero
    import paper_2506_04976_amd as pm
    lowest = 0.0
    for inside in (*np.linspace(5e-4, 5e-3, 40), 0.02, 0.1, 0.3, 1.0, 3.0):
        cfg = _config(ratio, nsigma, inside)
        geom = pm.Geometry(cfg)
        x = torch.zeros((1, cfg["ny"], cfg["nx"]), device="cuda:0")
        x[0, 0] = x[0, -1] = 1.0
        out = torch.full((geom.n_bins,), float("nan"), device="cuda:0")
        pm.pet_fwd(geom, -1, x.flatten(), None, None, out)
        sino = torch.zeros((geom.n_bins // 3, 3), device="cuda:0")
        sino[:, 1] = 1.0
        img = torch.full((geom.n_vox,), float("nan"), device="cuda:0")
        pm.pet_back(geom, -1, sino.flatten(), None, img)
        assert bool(torch.isfinite(out).all() and torch.isfinite(img).all())
        lowest = min(lowest, float(out.min()), float(img.min()))
    print(f"\n[wide bins] {ratio} sigma, truncated at {nsigma}: lowest {lowest:.2e}", flush=True)
    assert lowest == 0.0
