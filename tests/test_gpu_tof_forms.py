"""The TOF line kernels at the edges of their forms, against the FP64 oracle:

* one block of bins and two, full and not (1 bin is not TOF; 2, 5, 13, 16, 17,
  25, 31, 32 bins);
* 48 and 80 voxels along z per pass of the adjoint, and several passes;
* units of 1 to 64 planes: tiles of 16 just full and just not, pairs of segments
  of 64 planes together and of a little more;
* rings closer than the voxels (more than two planes may reach a voxel);
* lines of more rows than the waves of a workgroup hold at once;
* more units than the LDS holds at once;
* TOF bins that reach only a part of each line;
* lines that miss the image; every type of counts.

Tolerance as in the other parity tests: 1e-5 of the norm of the sum of the
summands' magnitudes (a bin's weight is off by less than 1e-7 of the largest one
from its table, positions are 32-bit numbers of up to 400 cells).
"""

import numpy as np
import pytest
import torch

from oracle import poisson, projector, recon
from synth import configs

pytestmark = pytest.mark.gpu

BASE = dict(n_views=14, n_crystals=28, n_rad=9, n_subsets=2, nx=16, ny=15)
GEOMETRIES = {
    "bins_2": dict(BASE, nz=5, n_rings=4, max_ring_diff=1, n_tof=2, tof_bin=40.0),
    "bins_13_planes_15": dict(BASE, nz=48, vz=2.0, n_rings=15, ring_pitch=6.0, max_ring_diff=4, n_tof=13, tof_bin=9.0),
    "bins_16_planes_16": dict(BASE, nz=49, vz=2.0, n_rings=16, ring_pitch=6.0, max_ring_diff=2, n_tof=16, tof_bin=8.0),
    "bins_17_planes_17": dict(BASE, nz=30, vz=2.5, n_rings=17, ring_pitch=4.0, max_ring_diff=16, n_tof=17, tof_bin=7.0),
    "bins_25_pairs_of_62": dict(BASE, nz=80, vz=1.9, n_rings=32, ring_pitch=4.5, max_ring_diff=2, n_tof=25, tof_bin=6.0),
    "bins_31_pairs_of_64": dict(BASE, nz=81, vz=2.0, n_rings=33, ring_pitch=4.8, max_ring_diff=2, n_tof=31, tof_bin=5.0),
    "bins_32_groups_of_units": dict(BASE, nx=30, ny=29, vx=2.0, vy=2.0, nz=33, vz=1.4, n_rings=32, ring_pitch=1.5,
                                    max_ring_diff=31, n_tof=32, tof_bin=5.0),
    "planes_33_47_48": dict(BASE, nx=28, ny=27, vx=2.2, vy=2.1, nz=97, vz=1.0, n_rings=48, ring_pitch=2.0,
                             max_ring_diff=15, n_tof=13, tof_bin=12.0),
    "planes_63_64": dict(BASE, nz=20, vz=3.2, n_rings=64, ring_pitch=1.0, max_ring_diff=1, n_tof=5),
    "one_ring_one_slice": dict(BASE, nz=1, vz=5.0, n_rings=1, ring_pitch=5.0, max_ring_diff=0, n_tof=5),
    "one_ring_close_slices": dict(BASE, nz=7, vz=9.0, n_rings=6, ring_pitch=5.0, max_ring_diff=2, n_tof=16, tof_bin=8.0),
    "rows_129": dict(BASE, nx=129, ny=131, vx=0.7, vy=0.68, nz=5, vz=3.0, n_rings=4, ring_pitch=3.5, max_ring_diff=3,
                     n_tof=13, tof_bin=10.0),
    "rows_160_of_few_bins": dict(BASE, nx=160, ny=157, vx=0.6, vy=0.6, nz=4, vz=3.0, n_rings=5, ring_pitch=3.1,
                                 max_ring_diff=4, n_tof=3, tof_bin=6.0, tof_sigma=2.0),
    "narrow_bins": dict(BASE, nx=24, ny=21, nz=9, n_rings=8, max_ring_diff=3, n_tof=4, tof_bin=5.0, tof_sigma=2.5),
    "far_lines": dict(BASE, nx=6, ny=5, n_crystals=42, n_views=21, n_rad=35, n_subsets=4, nz=9, n_rings=8,
                      max_ring_diff=3, n_tof=5),
}


for g in GEOMETRIES.values():
    if "tof_bin" in g:  # (at most eight bins may overlap at one point)
        g.setdefault("tof_sigma", 0.9 * g["tof_bin"])


class Setup:
    def __init__(self, name):
        import paper_2506_04976_amd as pm
        self.pm = pm
        self.cfg = configs.get("mini_tof", **GEOMETRIES[name])
        cfg = self.cfg
        self.dev = torch.device("cuda:0")
        self.geom = pm.Geometry(cfg)
        rng = np.random.default_rng(7)
        lors = (cfg["n_views"], cfg["n_rad"], configs.n_planes(cfg))
        bins = lors + (cfg["n_tof"],)
        self.x = rng.uniform(0.2, 1.0, (cfg["nz"], cfg["ny"], cfg["nx"])).astype(np.float32)
        self.v = rng.uniform(-1.0, 1.0, self.x.shape).astype(np.float32)
        self.mult = rng.uniform(0.5, 1.0, lors).astype(np.float32)
        self.add = rng.uniform(0.5, 1.0, bins).astype(np.float32)
        self.sino = rng.uniform(0.0, 2.0, bins).astype(np.float32)
        dtype = (np.uint8, np.uint16, np.float32)[list(GEOMETRIES).index(name) % 3]
        self.y = rng.poisson(1.5, bins).astype(dtype)
        self.prob = recon.Problem(cfg, self.y, self.add, self.mult, beta=1e-3, gamma=2.0, eps=1e-3)

    def t(self, a):
        return torch.from_numpy(np.ascontiguousarray(a).ravel()).to(self.dev)

    def image(self):
        return torch.full((self.geom.n_vox,), float("nan"), device=self.dev)


@pytest.fixture(scope="module", params=GEOMETRIES)
def setup(request):
    print(f"\n[TOF case {request.param}]", flush=True)
    return Setup(request.param)


def _off(got, ref, scale=None):
    d = np.asarray(got.cpu(), np.float64).ravel() - np.asarray(ref, np.float64).ravel()
    return float(np.linalg.norm(d) / np.linalg.norm(ref if scale is None else scale))


def test_projections(setup):
    s, pm, cfg = setup, setup.pm, setup.cfg
    for subset in (-1, 1):
        views = list(range(cfg["n_views"])) if subset < 0 else configs.subset_views(cfg, subset)
        p1, p2 = projector.view_lors(cfg, views)
        w = s.mult[views].astype(np.float64).reshape(-1, 1)
        back = s.image()
        pm.pet_back(s.geom, subset, s.t(s.sino), s.t(s.mult), back)
        assert _off(back, projector.back(cfg, s.sino[views].reshape(len(w), -1) * w, p1, p2)) <= 1e-5
        sens = s.image()
        pm.pet_back(s.geom, subset, None, s.t(s.mult), sens)
        assert _off(sens, projector.back(cfg, np.repeat(w, cfg["n_tof"], 1), p1, p2)) <= 1e-5
        out = torch.zeros(s.geom.n_bins, device=s.dev)
        pm.pet_fwd(s.geom, subset, s.t(s.x), s.t(s.mult), s.t(s.add), out)
        got = out.view(cfg["n_views"], -1)[views]
        assert _off(got, projector.fwd(cfg, s.x, p1, p2) * w + s.add[views].reshape(len(w), -1)) <= 1e-5


def test_gradient_and_curvature(setup):
    s, pm, prob = setup, setup.pm, setup.prob
    xo = s.x.astype(np.float64)
    x, y, add, mult = s.t(s.x), s.t(s.y), s.t(s.add), s.t(s.mult)
    yb = prob.ybar(xo, 0)
    ref, scale = prob.data_grad(xo, 0), prob.back(prob.a[0] * (1 + prob.y[0] / yb), 0)
    kl = torch.zeros(1, dtype=torch.float64, device=s.dev)
    for wanted in (None, kl):
        grad = s.image()
        pm.pet_subset_grad(s.geom, 0, x, y, add, mult, grad, wanted)
        assert _off(grad, ref, scale) <= 1e-5
    assert float(kl) == pytest.approx(float(np.sum(poisson.kl(yb, prob.y[0]))), rel=1e-5)
    hv, work = s.image(), torch.empty(s.geom.n_bins, device=s.dev)
    pm.pet_subset_hvp(s.geom, 0, x, s.t(s.v), y, add, mult, work, hv)
    curve = prob.a[0] * prob.y[0] / yb ** 2
    ref = prob.back(curve * prob.a[0] * prob.fwd(s.v.astype(np.float64), 0), 0)
    scale = prob.back(curve * prob.a[0] * prob.fwd(np.abs(s.v.astype(np.float64)), 0), 0)
    assert _off(hv, ref, scale) <= 1e-5


def test_objective(setup):
    s, pm = setup, setup.pm
    out = torch.zeros(1, dtype=torch.float64, device=s.dev)
    w27 = pm.rdp_weights27(s.cfg["vx"], s.cfg["vy"], s.cfg["vz"])
    pm.pet_objective(s.geom, s.t(s.x), s.t(s.y), s.t(s.add), s.t(s.mult), None, w27, 1e-3, 2.0, 1e-3, out)
    assert float(out) == pytest.approx(float(s.prob.objective(s.x.astype(np.float64))), rel=1e-5)


@pytest.mark.parametrize("names", [("bins_2", "bins_25_pairs_of_62"), ("bins_17_planes_17", "bins_2"),
                                   ("bins_16_planes_16", "bins_13_planes_15"), ("planes_63_64", "bins_2"),
                                   ("one_ring_close_slices", "bins_17_planes_17")])
def test_batch_of_two_forms(names):
    # a batch runs all its members in one form of the kernels
    runs = []
    for _ in range(2):
        members = []
        for s in (Setup(name) for name in names):
            sens = s.image()
            s.pm.pet_back(s.geom, -1, None, s.t(s.mult), sens)
            st = s.pm.SvrgStateBuffers(s.geom, s.t(s.y), s.t(s.add), s.t(s.mult), sens, beta=1e-3, gamma=2.0, eps=1e-3,
                                       alpha=1.0, delta=1e-3)
            members.append((s.geom, st, s.t(s.x)))
        runs.append(members)
    for geom, st, x in runs[0]:
        s.pm.pet_svrg_epoch(geom, st, x, [0, 1], [0.5, 0.5], [True, False])
    b = s.pm.Batch(runs[1])
    b.epochs([[0, 1]] * 2, [[0.5, 0.5]] * 2, [[True, False]] * 2, use_graph=False)
    torch.cuda.synchronize()
    for (_, _, one), (_, _, many) in zip(*runs):
        assert _off(many, one.cpu().numpy()) <= 1e-5
    b.close()
