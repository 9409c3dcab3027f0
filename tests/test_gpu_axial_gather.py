"""The axial gather of the adjoint (cells of a line's sheet collecting the shares
of its planes) at the edges of its forms, against the FP64 oracle:

* rings as far apart as the voxels, twice as far, a little closer (more than two
  planes may reach a voxel) and far closer;
* more planes than the LDS holds at once (chunks), and segments of more than
  1024 planes (in parts);
* a single ring, a single slice, one plane fewer or more than a wave;
* factors that are not finite: they reach the voxels of their LOR and no others.

Tolerance: backprojections of nonnegative sinograms and forward projections of
nonnegative images to a relative L2 error of 1e-5, gradients to 1e-5 of the norm
of the sum of their summands' magnitudes (positions are 32-bit numbers of up to
400 cells, so a share is off by at most 3e-5, with either sign, and each voxel
sums dozens of them).
"""

import numpy as np
import pytest
import torch

from oracle import poisson, projector, recon
from synth import configs, data

pytestmark = pytest.mark.gpu

SMALL = dict(n_views=6, n_crystals=12, n_rad=5, n_subsets=2)
GEOMETRIES = {
    "rings_at_voxels": dict(SMALL, nz=9, vz=4.1, n_rings=9, ring_pitch=4.1, max_ring_diff=4),
    "rings_at_two_voxels": dict(SMALL, nz=17, vz=2.0, n_rings=8, ring_pitch=4.0, max_ring_diff=7),
    "rings_a_little_closer": dict(SMALL, nz=9, vz=4.0, n_rings=11, ring_pitch=3.9, max_ring_diff=5),
    "rings_far_closer": dict(SMALL, nz=5, vz=8.0, n_rings=33, ring_pitch=1.2, max_ring_diff=8),
    "one_ring": dict(SMALL, nz=5, vz=3.0, n_rings=1, ring_pitch=4.0, max_ring_diff=0),
    "one_slice": dict(SMALL, nz=1, vz=6.0, n_rings=3, ring_pitch=6.5, max_ring_diff=2),
    "planes_63": dict(SMALL, nz=70, vz=2.0, n_rings=63, ring_pitch=2.1, max_ring_diff=0),
    "planes_65": dict(SMALL, nz=70, vz=2.0, n_rings=65, ring_pitch=2.1, max_ring_diff=0),
    "chunks": dict(SMALL, nx=6, ny=7, nz=400, vz=1.0, n_rings=390, ring_pitch=1.01, max_ring_diff=20),
    "parts_and_chunks": dict(SMALL, nx=8, ny=6, nz=12, vz=4.0, n_rings=1100, ring_pitch=48.0 / 1100, max_ring_diff=6),
}


class Setup:
    def __init__(self, name):
        import paper_2506_04976_amd as pm
        self.pm = pm
        self.cfg = configs.get("mini_nontof", **GEOMETRIES[name])
        cfg = self.cfg
        self.dev = torch.device("cuda:0")
        self.geom = pm.Geometry(cfg)
        rng = np.random.default_rng(5)
        lors = (cfg["n_views"], cfg["n_rad"], configs.n_planes(cfg))
        self.shape = (cfg["nz"], cfg["ny"], cfg["nx"])
        self.x = rng.uniform(0.2, 1.0, self.shape).astype(np.float32)
        self.mult = rng.uniform(0.5, 1.0, lors).astype(np.float32)
        self.add = rng.uniform(0.5, 1.0, lors + (1,)).astype(np.float32)
        self.sino = rng.uniform(0.0, 2.0, lors + (1,)).astype(np.float32)
        self.y = rng.poisson(20.0, lors + (1,)).astype(np.uint8)

    def t(self, a):
        return torch.from_numpy(np.ascontiguousarray(a).ravel()).to(self.dev)


@pytest.fixture(scope="module", params=GEOMETRIES)
def setup(request):
    print(f"\n[gather case {request.param}]", flush=True)
    return Setup(request.param)


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64).ravel() - b.ravel()) / np.linalg.norm(b))


def test_projections(setup):
    s, pm, cfg = setup, setup.pm, setup.cfg
    for subset in (-1, 1):
        views = list(range(cfg["n_views"])) if subset < 0 else configs.subset_views(cfg, subset)
        p1, p2 = projector.view_lors(cfg, views)
        back = torch.full((s.geom.n_vox,), float("nan"), device=s.dev)
        pm.pet_back(s.geom, subset, s.t(s.sino), s.t(s.mult), back)
        weighted = (s.sino[..., 0] * s.mult.astype(np.float64))[views].reshape(-1, 1)
        assert _rel(back.cpu().numpy(), projector.back(cfg, weighted, p1, p2)) <= 1e-5
        sens = torch.full((s.geom.n_vox,), float("nan"), device=s.dev)
        pm.pet_back(s.geom, subset, None, s.t(s.mult), sens)
        assert _rel(sens.cpu().numpy(), projector.back(cfg, s.mult[views].astype(np.float64).reshape(-1, 1), p1, p2)) <= 1e-5
        out = torch.zeros(s.geom.n_bins, device=s.dev)
        pm.pet_fwd(s.geom, subset, s.t(s.x), s.t(s.mult), None, out)
        got = out.cpu().numpy().reshape(s.sino.shape)[views]
        ref = projector.fwd(cfg, s.x, p1, p2).reshape(got.shape) * s.mult[views][..., None]
        assert _rel(got, ref) <= 1e-5


def test_gradient(setup):
    s, pm, cfg = setup, setup.pm, setup.cfg
    prob = recon.Problem(cfg, s.y, s.add, s.mult, beta=1e-3, gamma=2.0, eps=1e-3)
    grad = torch.full((s.geom.n_vox,), float("nan"), device=s.dev)
    kl = torch.zeros(1, dtype=torch.float64, device=s.dev)
    pm.pet_subset_grad(s.geom, 0, s.t(s.x), s.t(s.y), s.t(s.add), s.t(s.mult), grad, kl)
    xo = s.x.astype(np.float64)
    yb = prob.ybar(xo, 0)
    scale = np.linalg.norm(prob.back(prob.a[0] * (1 + prob.y[0] / yb), 0))
    assert np.linalg.norm(grad.cpu().double().numpy() - prob.data_grad(xo, 0).ravel()) <= 1e-5 * scale


@pytest.mark.parametrize("name", ["mini_nontof", "mini_tof"])
def test_factors_not_finite(name):
    # one infinite bin: exactly the voxels with a weight in its LOR are not finite
    import paper_2506_04976_amd as pm
    cfg = configs.get(name)
    geom = pm.Geometry(cfg)
    dev = torch.device("cuda:0")
    shape = (cfg["n_views"], cfg["n_rad"], configs.n_planes(cfg), cfg["n_tof"])
    view, rad, plane, tof = 4, 7, 11, cfg["n_tof"] // 2
    unit = np.zeros(shape)
    unit[view, rad, plane, tof] = 1.0
    p1, p2 = projector.view_lors(cfg, [view])
    reach = projector.back(cfg, unit[[view]].reshape(-1, cfg["n_tof"]), p1, p2).ravel() > 0
    for bad in (np.inf, np.nan):
        sino = np.ones(shape, np.float32)
        sino[view, rad, plane, tof] = bad
        out = torch.empty(geom.n_vox, device=dev)
        pm.pet_back(geom, -1, torch.from_numpy(sino.ravel()).to(dev), None, out)
        np.testing.assert_array_equal(~np.isfinite(out.cpu().numpy()), reach)


def test_likelihood_and_gradient_without_it(setup):
    # the likelihood is added up over chunks and partial rounds of planes, each
    # LOR once; the gradient does not depend on whether it is asked for
    pm = setup.pm
    prob = recon.Problem(setup.cfg, setup.y, setup.add, setup.mult, beta=1.0, gamma=2.0, eps=1.0)
    x = setup.t(setup.x)
    args = (setup.geom, 1, x, setup.t(setup.y), setup.t(setup.add), setup.t(setup.mult))
    with_kl, without = (torch.full_like(x, float("nan")) for _ in range(2))
    kl = torch.full((1,), float("nan"), dtype=torch.float64, device=setup.dev)
    pm.pet_subset_grad(*args, with_kl, kl)
    pm.pet_subset_grad(*args, without)
    yb = prob.ybar(setup.x.astype(np.float64), 1)
    assert float(kl) == pytest.approx(float(np.sum(poisson.kl(yb, prob.y[1]))), rel=1e-5)
    ref = prob.data_grad(setup.x.astype(np.float64), 1).ravel()
    scale = np.linalg.norm(prob.back(prob.a[1] * (1 + prob.y[1] / yb), 1))
    for g in (with_kl, without):
        assert np.linalg.norm(g.cpu().double().numpy() - ref) / scale <= 1e-5
