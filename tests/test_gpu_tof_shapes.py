"""TOF adjoints over the shapes between which the line kernels choose their form,
against the FP64 oracle: axes of 1 to 131 slices (16 to 80 voxels a pass, one pass
or more, a last pass nearly empty), launches of few lines (a line's blocks of rows
dealt to several waves) and of more than the chip holds (small workgroups), one to
several units of planes, one block of bins and two.

Tolerance: as for the other forms of these kernels, backprojections of nonnegative
sinograms to a relative L2 error of 1e-5, gradients and EM ratios (an OSEM update
against its oracle) to 1e-5 of the norm of their summands' magnitudes.
"""

import numpy as np
import pytest
import torch

from oracle import recon
from synth import configs

pytestmark = pytest.mark.gpu

AXES = {1: (3, 1), 5: (3, 2), 16: (7, 1), 17: (9, 3), 32: (16, 2), 33: (12, 5), 48: (20, 1), 49: (9, 3), 64: (13, 2),
        65: (9, 1), 80: (12, 2), 81: (11, 2), 97: (11, 1), 131: (40, 2)}
LINES = {"few": dict(n_views=6, n_crystals=12, n_rad=7), "many": dict(n_views=45, n_crystals=90, n_rad=15)}


@pytest.mark.parametrize("lines", LINES)
@pytest.mark.parametrize("bins", [5, 19])
@pytest.mark.parametrize("nz", AXES)
def test_adjoints(nz, bins, lines):
    import paper_2506_04976_amd as pm
    rings, diff = AXES[nz]
    print(f"\n[tof shapes] {nz} slices, {bins} bins, {lines} lines", flush=True)
    cfg = configs.get("mini_tof", nx=14, ny=18, nz=nz, vz=2.0, n_rings=rings, ring_pitch=2.0 * max(1.0, nz / rings),
                      max_ring_diff=diff, n_tof=bins, tof_bin=110.0 / bins, tof_sigma=70.0 / bins, n_subsets=1,
                      **LINES[lines])
    geom, dev = pm.Geometry(cfg), torch.device("cuda:0")
    rng = np.random.default_rng(nz)
    lors = (cfg["n_views"], cfg["n_rad"], configs.n_planes(cfg))
    x = rng.uniform(0.2, 1.0, (nz, cfg["ny"], cfg["nx"])).astype(np.float32)
    mult = rng.uniform(0.5, 1.0, lors).astype(np.float32)
    add = rng.uniform(0.5, 1.0, lors + (bins,)).astype(np.float32)
    y = rng.poisson(9.0, lors + (bins,)).astype(np.uint8)

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a).ravel()).to(dev)

    prob = recon.Problem(cfg, y, add, mult, beta=1.0, gamma=2.0, eps=1.0)
    xo = x.astype(np.float64)
    out = torch.full((geom.n_vox,), float("nan"), device=dev)
    pm.pet_back(geom, 0, t(add), t(mult), out)
    ref = prob.back(prob.a[0] * prob.r[0], 0).ravel()
    assert np.linalg.norm(out.cpu().double().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
    pm.pet_subset_grad(geom, 0, t(x), t(y), t(add), t(mult), out)
    yb = prob.ybar(xo, 0)
    scale = np.linalg.norm(prob.back(prob.a[0] * (1 + prob.y[0] / yb), 0))
    assert np.linalg.norm(out.cpu().double().numpy() - prob.data_grad(xo, 0).ravel()) <= 1e-5 * scale
    xe = t(x)
    pm.pet_osem_epoch(geom, xe, t(y), t(add), t(mult), [0])
    want = recon.osem_epoch(prob, xo, [0])
    got = xe.cpu().double().numpy().reshape(xo.shape)
    assert np.linalg.norm(got - want) <= 2e-5 * np.linalg.norm(want)
