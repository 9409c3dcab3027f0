"""Adjoints with rings closer than the voxels, where more than two planes of a
segment reach a voxel, against the FP64 oracle: ring pitch over voxel size on both
sides of the lines between the forms of the gather (1 and 2/3), segments of one
to three planes, images shorter and longer than the rings, without TOF and with it.

Tolerance: backprojections of nonnegative sinograms to a relative L2 error of 1e-5,
gradients to 1e-5 of the norm of the sum of their summands' magnitudes (positions
are 32-bit numbers of at most a few dozen cells).
"""

import numpy as np
import pytest
import torch

from oracle import recon
from synth import configs

pytestmark = pytest.mark.gpu

KAPPAS = [2.0, 1.0, 0.999, 0.85, 0.7, 0.667, 0.666, 0.6, 0.5, 0.3, 0.11]
SIZES = {"short_segments": (9, 5, 4), "longer_than_the_rings": (21, 8, 3), "shorter_than_the_rings": (4, 23, 6)}


@pytest.mark.parametrize("name", ["mini_nontof", "mini_tof"])
@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("kappa", KAPPAS)
def test_adjoints(kappa, size, name):
    import paper_2506_04976_amd as pm
    nz, rings, diff = SIZES[size]
    cfg = configs.get(name, nz=nz, vz=4.0, n_rings=rings, ring_pitch=4.0 * kappa, max_ring_diff=diff, n_views=8,
                      n_crystals=16, n_rad=9, n_subsets=2)
    print(f"\n[close rings] {name} {size} kappa {kappa}", flush=True)
    geom, dev = pm.Geometry(cfg), torch.device("cuda:0")
    rng = np.random.default_rng(11)
    lors = (cfg["n_views"], cfg["n_rad"], configs.n_planes(cfg))
    x = rng.uniform(0.2, 1.0, (nz, cfg["ny"], cfg["nx"])).astype(np.float32)
    mult = rng.uniform(0.5, 1.0, lors).astype(np.float32)
    add = rng.uniform(0.5, 1.0, lors + (cfg["n_tof"],)).astype(np.float32)
    sino = rng.uniform(0.0, 2.0, lors + (cfg["n_tof"],)).astype(np.float32)
    y = rng.poisson(9.0, lors + (cfg["n_tof"],)).astype(np.uint8)

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a).ravel()).to(dev)

    prob = recon.Problem(cfg, y, add, mult, beta=1.0, gamma=2.0, eps=1.0)
    out = torch.full((geom.n_vox,), float("nan"), device=dev)
    views = configs.subset_views(cfg, 1)

    def off(ref, scale=None):
        d = np.linalg.norm(out.cpu().double().numpy() - ref.ravel())
        return d / (np.linalg.norm(ref) if scale is None else scale)

    pm.pet_back(geom, 1, t(sino), t(mult), out)
    assert off(prob.back(prob.a[1] * sino[views].reshape(prob.y[1].shape), 1)) <= 1e-5
    pm.pet_back(geom, 1, None, t(mult), out)
    assert off(prob.back(prob.a[1] * np.ones_like(prob.y[1]), 1)) <= 1e-5
    pm.pet_subset_grad(geom, 1, t(x), t(y), t(add), t(mult), out)
    yb = prob.ybar(x.astype(np.float64), 1)
    scale = np.linalg.norm(prob.back(prob.a[1] * (1 + prob.y[1] / yb), 1))
    assert off(prob.data_grad(x.astype(np.float64), 1), scale) <= 1e-5


@pytest.mark.parametrize("name", ["mini_nontof", "mini_tof"])
@pytest.mark.parametrize("kappa", [1.0 / 3.0, 0.75, 1.0, 1.5, 2.0, 3.0, 5.0])
def test_unseen_voxels(kappa, name):
    # Rings centred on the image, with voxels a whole number of voxels away from
    # the planes: a voxel that no LOR sees has a sensitivity of exactly zero (an
    # OSEM step divides by it), and weakly seen ones the same shares in the
    # sensitivity and in what is divided by it.
    import paper_2506_04976_amd as pm
    nz = 15
    rings = max(2, int(nz / kappa))
    cfg = configs.get(name, nz=nz, vz=2.0, n_rings=rings, ring_pitch=2.0 * kappa, max_ring_diff=min(3, rings - 1),
                      nx=14, ny=18, n_views=12, n_crystals=24, n_rad=15, n_subsets=2)
    print(f"\n[unseen voxels] {name} kappa {kappa:.3f}", flush=True)
    geom, dev = pm.Geometry(cfg), torch.device("cuda:0")
    rng = np.random.default_rng(3)
    lors = (cfg["n_views"], cfg["n_rad"], configs.n_planes(cfg))
    x = rng.uniform(0.2, 1.0, (nz, cfg["ny"], cfg["nx"])).astype(np.float32)
    mult = rng.uniform(0.5, 1.0, lors).astype(np.float32)
    add = rng.uniform(0.5, 1.0, lors + (cfg["n_tof"],)).astype(np.float32)
    y = rng.poisson(3.0, lors + (cfg["n_tof"],)).astype(np.uint8)

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a).ravel()).to(dev)

    prob = recon.Problem(cfg, y, add, mult, beta=1.0, gamma=2.0, eps=1.0)
    sens = torch.full((geom.n_vox,), float("nan"), device=dev)
    for i in range(2):
        pm.pet_back(geom, i, None, t(mult), sens)
        # (beyond what FP64 itself makes of an exact zero)
        ref = prob.sens_subset(i).ravel()
        np.testing.assert_array_equal(sens.cpu().numpy() > 0, ref > 1e-12 * ref.max())
    want = recon.osem_epoch(prob, x.astype(np.float64), [0, 1]).ravel()
    dense, sparse = t(x), t(x)
    pm.pet_osem_epoch(geom, dense, t(y), t(add), t(mult), [0, 1])
    pm.pet_osem_epoch_counts(geom, pm.Counts(geom, t(y), t(add), t(mult)), sparse, t(mult), [0, 1])
    for got in (dense, sparse):  # (images after an epoch, as in the other tests of this path)
        assert np.linalg.norm(got.cpu().double().numpy() - want) <= 1e-4 * np.linalg.norm(want)


@pytest.mark.parametrize("rings,diff", [(1, 0), (3, 0), (12, 7), (64, 63)])
def test_sensitivity_at_the_ends_of_the_bins(rings, diff):
    # bins that end inside the image: the sum of their weights differs from row to
    # row and between the ring differences (blocks of 64 rows with 64 of them)
    import paper_2506_04976_amd as pm
    cfg = configs.get("mini_tof", nx=70, ny=66, vx=2.0, vy=2.0, nz=6, vz=3.0, n_rings=rings, ring_pitch=18.0 / rings,
                      max_ring_diff=diff, n_views=9, n_crystals=18, n_rad=5, radius=150.0, n_tof=5, tof_bin=24.0,
                      tof_sigma=11.0, n_subsets=1)
    print(f"\n[ends of the bins] {rings} rings, differences to {diff}", flush=True)
    geom, dev = pm.Geometry(cfg), torch.device("cuda:0")
    lors = (cfg["n_views"], cfg["n_rad"], configs.n_planes(cfg))
    mult = np.random.default_rng(2).uniform(0.5, 1.0, lors).astype(np.float32)
    blank = np.zeros(lors + (cfg["n_tof"],), np.uint8)
    prob = recon.Problem(cfg, blank, blank, mult, beta=1.0, gamma=2.0, eps=1.0)
    out = torch.full((geom.n_vox,), float("nan"), device=dev)
    pm.pet_back(geom, 0, None, torch.from_numpy(mult.ravel()).to(dev), out)
    ref = prob.sens_subset(0).ravel()
    assert np.linalg.norm(out.cpu().double().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
