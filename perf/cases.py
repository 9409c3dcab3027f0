"""Workloads by which the library's speed is judged: what a reconstruction program
asks of it, through the Python entry points, from the smallest 2D subset
gradient to a whole epoch of the 3D TOF reconstruction.

Inputs are synthetic: an ellipsoid phantom (a shell, an interior and one hot
sphere, sized by the field of view), its exact line integrals (with TOF: the
integrals of the bin-integrated Gaussian), attenuation factors, a 20% background
and Poisson counts, all drawn on the GPU from the seed.  ``exact`` evaluates the
same quantities in FP64 with plain torch operations from the definitions (Joseph
line integrals, KL data term, relative difference prior, SAGA).
"""

import math
import random

import numpy as np
import torch

import paper_2506_04976_amd as pm

MU_WATER = 0.0096  # 1/mm
FWHM = 1.0 / (2.0 * math.sqrt(2.0 * math.log(2.0)))
PITCH = 71 * 2.03 / 64  # 64 rings over the 71-slice image

# ---- the geometries of the repository's workloads ---------------------------
PARALLEL = dict(kind="parallel2d", nx=64, ny=64, nz=1, vx=4.0, vy=4.0, vz=4.0, n_views=60, n_rad=91,
                rad_spacing=4.0, half_length=500.0, n_tof=1, n_subsets=6, counts=1e5)
SMALL = dict(kind="cylinder", nx=96, ny=96, nz=32, vx=128 * 2.086 / 96, vy=128 * 2.086 / 96, vz=4.5, radius=328.0,
             n_views=120, n_rad=180, n_rings=32, ring_pitch=4.5, max_ring_diff=4, n_tof=1, n_subsets=8, counts=5e6)
BRAIN = dict(kind="cylinder", nx=128, ny=128, nz=71, vx=2.086, vy=2.086, vz=2.03, radius=328.0, n_views=252,
             n_rad=344, n_rings=64, ring_pitch=PITCH, max_ring_diff=20, n_tof=1, n_subsets=25, counts=1e7)
TOF13 = dict(n_tof=13, tof_bin=40.0, tof_sigma=60.0 * FWHM, tof_nsigma=3.0)
BRAIN_TOF = dict(BRAIN, counts=3e7, **TOF13)
SMALL_TOF = dict(SMALL, **TOF13)
# 17-ring simulation geometry: 25 TOF bins, 4 mm image-space resolution model
SIM_TOF = dict(kind="cylinder", nx=161, ny=161, nz=33, vx=2.5, vy=2.5, vz=2.5, radius=300.0, n_views=216, n_rad=353,
               n_rings=17, ring_pitch=80.0 / 17, max_ring_diff=16, n_tof=25, tof_bin=24.0,
               tof_sigma=0.390 * 299.792458 / 2 * FWHM, tof_nsigma=3.0, psf_fwhm=4.0, n_subsets=27, counts=1e7)

_ALL_VIEWS = -1


def listed():
    return [
        # one subset gradient of a 2D slice: a few microseconds of work per
        # kernel, so launches and their gaps are the time
        dict(PARALLEL, name="grad_2d", op="grad", subset=2, y="u16"),
        # the prior's gradient, Hessian diagonal and value, as a line search,
        # a MAP solver and the preconditioner ask for them
        dict(BRAIN, name="rdp_brain", op="rdp"),
        # the reverse mode's data-term product (unrolled reconstruction)
        dict(SMALL, name="hvp_small", op="hvp", subset=3, y="u8"),
        # a user's own projections: every view forward, all TOF bins
        dict(SMALL_TOF, name="fwd_small_tof", op="fwd", subset=_ALL_VIEWS),
        # and one subset of a sinogram back
        dict(BRAIN, name="back_brain", op="back", subset=7),
        # the dense subset gradients of the three 3D geometries, with the
        # objective where a program monitors it
        dict(BRAIN, name="grad_brain", op="grad", subset=1, y="u16", kl=True),
        dict(BRAIN_TOF, name="grad_brain_tof", op="grad", subset=4, y="u8"),
        dict(SIM_TOF, name="grad_sim_tof", op="grad", subset=11, y="f32"),
        # the zero-count-aware subset gradient, the inner step of the epochs
        dict(BRAIN_TOF, name="counts_brain_tof", op="counts", subset=9, y="u8"),
        # the sensitivity image, once per reconstruction
        dict(BRAIN_TOF, name="sens_brain_tof", op="sens", subset=_ALL_VIEWS),
        # whole calls: a first SAGA epoch of the small geometry (table fill and
        # 7 steps), and a first SVRG epoch of the 3D TOF reconstruction
        # (preconditioner, snapshot pass over 25 subsets, 24 steps)
        dict(SMALL, name="saga_small", op="saga", y="u8"),
        dict(BRAIN_TOF, name="svrg_brain_tof", op="svrg", y="u8"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _planes(case):
    """(r1, r2) of every plane, segments 0, -1, +1, ..."""
    if case["kind"] == "parallel2d":
        return [(0, 0)]
    nr = case["n_rings"]
    out = [(r, r) for r in range(nr)]
    for k in range(1, case["max_ring_diff"] + 1):
        out += [(r, r - k) for r in range(k, nr)]
        out += [(r, r + k) for r in range(nr - k)]
    return out


def draw(rng):
    """One more case: any entry point above on an image of 20 to 161 voxels
    across and 4 to 72 slices, non-TOF or with 5 to 25 TOF bins."""
    op = rng.choice(["grad", "grad", "grad", "counts", "counts", "fwd", "back", "sens", "hvp", "rdp", "saga"])
    if op == "grad" and rng.random() < 0.25:
        n = _log_int(rng, 20, 160)
        views = rng.randint(12, 120)
        return dict(PARALLEL, op=op, nx=n, ny=max(8, n - rng.randint(0, 9)), vx=rng.uniform(2.0, 4.0),
                    vy=rng.uniform(2.0, 4.0), n_views=views, n_rad=rng.randint(n, 2 * n),
                    rad_spacing=rng.uniform(2.0, 4.0), n_subsets=rng.randint(2, 12), subset=1,
                    y=rng.choice(["u8", "u16", "f32"]), kl=rng.random() < 0.5, counts=math.exp(rng.uniform(9, 13)))
    nx = _log_int(rng, 20, 161)
    ny = max(16, nx - rng.randint(0, 13))
    nz = min(_log_int(rng, 4, 72), 9600 // max(nx, ny) - 4)
    vx, vz = rng.uniform(2.0, 4.0), rng.uniform(2.0, 4.5)
    if max(nx, ny) * vx > 400:
        vx = 400.0 / max(nx, ny)
    half = 0.5 * math.hypot((nx + 4) * vx, (ny + 4) * vx)
    rings = max(2, min(64, int(nz * rng.uniform(0.5, 1.25))))
    views = _log_int(rng, 24, 252)
    case = dict(kind="cylinder", op=op, nx=nx, ny=ny, nz=nz, vx=vx, vy=vx * rng.uniform(0.95, 1.05), vz=vz,
                radius=max(90.0, 1.12 * half * rng.uniform(1.0, 1.5)), n_views=views,
                n_rad=max(3, int(2 * views * rng.uniform(0.4, 0.7))), n_rings=rings, ring_pitch=nz * vz / rings,
                max_ring_diff=rng.randint(0, max(1, rings // 3)), n_tof=1, n_subsets=rng.randint(2, min(25, views // 4)),
                counts=math.exp(rng.uniform(math.log(1e5), math.log(2e7))), y=rng.choice(["u8", "u8", "u16", "f32"]))
    if op == "sens" or (op not in ("rdp", "saga") and rng.random() < 0.5):
        nt = rng.randint(5, 25)
        tof_bin = 1.6 * case["radius"] / nt
        case.update(n_tof=nt, tof_bin=tof_bin, tof_sigma=tof_bin * rng.uniform(0.4, 0.72), tof_nsigma=3.0)
        if rng.random() < 0.3:
            case.update(psf_fwhm=rng.uniform(1.2, 2.0) * vx)
    case["subset"] = rng.randrange(case["n_subsets"])
    if op == "grad":
        case["kl"] = rng.random() < 0.5
    return case


# ---- geometry of the LORs (FP64) --------------------------------------------
def _views(case):
    n, s = case["n_subsets"], case.get("subset", _ALL_VIEWS)
    return list(range(case["n_views"])) if s < 0 else list(range(s, case["n_views"], n))


def _radial(case):
    """Signed distance s and half length h of the radial lines."""
    k = np.arange(case["n_rad"]) - 0.5 * (case["n_rad"] - 1)
    if case["kind"] == "parallel2d":
        s = k * case["rad_spacing"]
        return s, np.full_like(s, case["half_length"])
    s = case["radius"] * np.sin(math.pi * k / (2 * case["n_views"]))
    return s, np.sqrt(case["radius"] ** 2 - s * s)


def _axial(case):
    """z of both ends of every plane's LORs."""
    if case["kind"] == "parallel2d":
        return np.zeros(1), np.zeros(1)
    r = np.array(_planes(case), np.float64)
    z = (r - 0.5 * (case["n_rings"] - 1)) * case["ring_pitch"]
    return z[:, 0].copy(), z[:, 1].copy()


def _sizes(case):
    n_p = len(_planes(case))
    lors = case["n_views"] * case["n_rad"] * n_p
    return n_p, lors, lors * case["n_tof"], case["nx"] * case["ny"] * case["nz"]


def _cfg(case):
    cfg = {k: v for k, v in case.items() if k not in ("name", "op", "subset", "y", "kl", "counts")}
    if case["kind"] == "cylinder":
        cfg["n_crystals"] = 2 * case["n_views"]
    return cfg


# ---- synthetic inputs -------------------------------------------------------
def _shapes(case):
    """Ellipsoids (cx, cy, cz, ax, ay, az, increment)."""
    wx, wy = case["nx"] * case["vx"], case["ny"] * case["vy"]
    wz = case["nz"] * case["vz"] if case["kind"] == "cylinder" else 1e6
    return [(0.0, 0.0, 0.0, 0.337 * wx, 0.281 * wy, 0.486 * wz, 4.0),
            (0.0, 0.0, 0.0, 0.300 * wx, 0.243 * wy, 0.417 * wz, -3.0),
            (0.13 * wx, 0.05 * wy, 0.0, 0.03 * wx, 0.03 * wx, 0.03 * wx if wz < 1e6 else wz, 2.0)]


def _phantom(case, dev):
    ax = [(torch.arange(case[n], device=dev, dtype=torch.float64) - 0.5 * (case[n] - 1)) * case[v]
          for n, v in (("nz", "vz"), ("ny", "vy"), ("nx", "vx"))]
    z, y, x = torch.meshgrid(*ax, indexing="ij")
    out = torch.zeros_like(x)
    for cx, cy, cz, a, b, c, inc in _shapes(case):
        out += inc * (((x - cx) / a) ** 2 + ((y - cy) / b) ** 2 + ((z - cz) / c) ** 2 <= 1.0)
    return out


def _chords(case, view, dev):
    """Per shape: entry and exit (mm from the LOR centre) on the LORs of a view, [R, P]."""
    f32 = dict(dtype=torch.float32, device=dev)
    s, h = (torch.tensor(v, **f32)[:, None] for v in _radial(case))
    z1, z2 = (torch.tensor(v, **f32)[None, :] for v in _axial(case))
    phi = math.pi * view / case["n_views"]
    cx0, cy0, cz0 = s * math.cos(phi), s * math.sin(phi), 0.5 * (z1 + z2)
    half = torch.sqrt(h * h + 0.25 * (z2 - z1) ** 2)
    dx, dy, dz = -h * math.sin(phi) / half, h * math.cos(phi) / half, 0.5 * (z2 - z1) / half
    out = []
    for cx, cy, cz, a, b, c, inc in _shapes(case):
        px, py, pz = (cx0 - cx) / a, (cy0 - cy) / b, (cz0 - cz) / c
        ux, uy, uz = dx / a, dy / b, dz / c
        qa = ux * ux + uy * uy + uz * uz
        qb = px * ux + py * uy + pz * uz
        disc = torch.clamp(qb * qb - qa * (px * px + py * py + pz * pz - 1.0), min=0.0).sqrt() / qa
        mid = -qb / qa
        out.append((mid - disc, mid + disc, inc))
    return out


def _tof_integrals(case, chords, dev):
    """Line integrals of the phantom in every TOF bin, [R, P, T]."""
    nt, w, sg = case["n_tof"], case["tof_bin"], math.sqrt(2.0) * case["tof_sigma"]
    edge = (torch.arange(nt + 1, device=dev, dtype=torch.float32) - 0.5 * nt) * w

    def cum(t):  # integral of erf((edge - t') / sg), up to a constant
        u = (edge - t[..., None]) / sg
        return u.mul(torch.erf(u)).add_(torch.exp(-u * u), alpha=1.0 / math.sqrt(math.pi))

    tot = None
    for t0, t1, inc in chords:
        d = (cum(t0) - cum(t1)).mul_(0.5 * sg * inc)
        tot = d if tot is None else tot.add_(d)
    return (tot[..., 1:] - tot[..., :-1]).clamp_(min=0.0)


_Y_TYPES = {"u8": (torch.uint8, 255), "u16": (torch.int16, 32767), "f32": (torch.float32, 1e30)}


def _inputs(case, seed, data=True, sino=False):
    """Image x, and what the op's data need: mult (LORs), add and y (bins), on the
    views of the case's subset (the other views stay 0: a call on a subset
    reads its own views only)."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * (seed + 1))
    n_p, n_lor, n_bin, n_vox = _sizes(case)
    nv, nr, nt = case["n_views"], case["n_rad"], case["n_tof"]
    # activity scale from the counts, over a few views
    some = range(0, nv, max(1, nv // 4))
    tot = 0.0
    for v in some:
        ch = _chords(case, v, dev)
        att = torch.exp(-MU_WATER * (ch[0][1] - ch[0][0]))
        tot += float((att * sum(inc * (t1 - t0) for t0, t1, inc in ch)).sum(dtype=torch.float64))
    scale = case["counts"] / (tot * nv / len(some))
    out = dict(scale=scale)
    noise = torch.rand(n_vox, generator=gen, device=dev)
    x = _phantom(case, dev).flatten().float()
    out["x"] = (scale * (x * (0.7 + 0.6 * noise) + 0.02 * (1.0 + noise))).contiguous()
    if not data:
        return out
    s = torch.tensor(_radial(case)[0], dtype=torch.float32, device=dev)
    prof = torch.exp(-0.5 * (s / (0.25 * case["nx"] * case["vx"])) ** 2) + 0.01
    bg = prof * (0.25 * case["counts"] / (nv * n_p * nt * float(prof.sum())))
    mult = torch.zeros(n_lor, dtype=torch.float32, device=dev)
    want_y = case["op"] in ("grad", "counts", "hvp", "saga", "svrg")
    add = torch.zeros(n_bin, dtype=torch.float32, device=dev) if want_y or case["op"] == "fwd" else None
    y = torch.zeros(n_bin, dtype=_Y_TYPES[case["y"]][0], device=dev) if want_y else None
    m3 = mult.view(nv, nr, n_p)
    for v in _views(case):
        ch = _chords(case, v, dev)
        m3[v] = torch.exp(-MU_WATER * (ch[0][1] - ch[0][0])) * (0.9 + 0.2 * torch.rand((nr, n_p), generator=gen, device=dev))
        if add is not None:
            add.view(nv, nr, n_p, nt)[v] = bg[:, None, None]
        if want_y:
            if nt > 1:
                p = _tof_integrals(case, ch, dev)
            else:
                p = sum(inc * (t1 - t0) for t0, t1, inc in ch)[..., None].clamp(min=0.0)
            mean = p.mul_(scale).mul_(m3[v][..., None]).add_(bg[:, None, None])
            y.view(nv, nr, n_p, nt)[v] = torch.poisson(mean, generator=gen).clamp_(max=_Y_TYPES[case["y"]][1]).to(y.dtype)
    out.update(mult=mult, add=add, y=y)
    if sino:
        out["sino"] = torch.zeros(n_bin, dtype=torch.float32, device=dev)
        s4 = out["sino"].view(nv, nr, n_p, nt)
        for v in _views(case):
            s4[v] = torch.randn((nr, n_p, nt), generator=gen, device=dev)
    if case["op"] == "hvp":
        out["v"] = scale * torch.randn(n_vox, generator=gen, device=dev)
    return out


def _beta(case):
    return 4.0 * 2e-4 * case["counts"] / 3e7


def _order(case, seed):
    order = list(range(case["n_subsets"]))
    random.Random(seed).shuffle(order)
    return order


def prepare(case, seed):
    op = case["op"]
    geom = pm.Geometry(_cfg(case))
    d = _inputs(case, seed, data=op != "rdp", sino=op == "back")
    dev = d["x"].device
    st = dict(case=case, geom=geom, subset=case.get("subset", _ALL_VIEWS), **d)
    f32 = dict(dtype=torch.float32, device=dev)
    if op in ("grad", "back", "sens", "counts", "hvp", "rdp"):
        st["out"] = torch.zeros(geom.n_vox, **f32)
    if op == "grad":
        st["kl"] = torch.zeros(1, dtype=torch.float64, device=dev) if case.get("kl") else None
    elif op == "fwd":
        st["out"] = torch.zeros(geom.n_bins, **f32)
    elif op == "hvp":
        st["ybar"] = torch.zeros(geom.n_bins, **f32)
    elif op == "rdp":
        st["hess"] = torch.zeros(geom.n_vox, **f32)
        st["value"] = torch.zeros(1, dtype=torch.float64, device=dev)
        st["w27"] = pm.rdp_weights27(case["vx"], case["vy"], case["vz"])
        st["eps"] = 1e-3 * float(d["x"].max())
    if op in ("counts", "saga", "svrg"):
        st["counts"] = pm.Counts(geom, d["y"], d["add"], d["mult"])
    if op in ("saga", "svrg"):
        sens = torch.zeros(geom.n_vox, **f32)
        pm.pet_back(geom, -1, None, d["mult"], sens)
        eps = 1e-3 * float(d["x"].max())
        st["svrg"] = pm.SvrgStateBuffers(geom, d["y"], d["add"], d["mult"], sens, beta=_beta(case), gamma=2.0, eps=eps,
                                         alpha=1.0, delta=eps, counts=st["counts"])
        st["xk"] = torch.empty_like(d["x"])
        n = case["n_subsets"]
        st["order"] = _order(case, seed)
        st["tau"] = [1.0 / (1.0 + 0.02 * j / n) for j in range(n)]
        st["update"] = [j == 0 for j in range(n)]
    return st


def run(state):
    op, g = state["case"]["op"], state["geom"]
    if op == "grad":
        pm.pet_subset_grad(g, state["subset"], state["x"], state["y"], state["add"], state["mult"], state["out"],
                           state["kl"])
        return (state["out"], state["kl"]) if state["kl"] is not None else state["out"]
    if op == "counts":
        return pm.pet_subset_grad_counts(g, state["counts"], state["subset"], state["x"], None, state["out"])
    if op == "fwd":
        return pm.pet_fwd(g, state["subset"], state["x"], state["mult"], state["add"], state["out"])
    if op == "back":
        return pm.pet_back(g, state["subset"], state["sino"], state["mult"], state["out"])
    if op == "sens":
        return pm.pet_back(g, state["subset"], None, state["mult"], state["out"])
    if op == "hvp":
        return pm.pet_subset_hvp(g, state["subset"], state["x"], state["v"], state["y"], state["add"], state["mult"],
                                 state["ybar"], state["out"])
    if op == "rdp":
        pm.pet_rdp_grad_hessdiag(g, state["x"], None, state["w27"], _beta(state["case"]), 2.0, state["eps"],
                                 state["out"], state["hess"], state["value"])
        return state["out"], state["hess"], state["value"]
    # an epoch from its starting image
    st, x = state["svrg"], state["xk"]
    x.copy_(state["x"])
    st.c.k = 0
    epoch = pm.pet_saga_epoch if op == "saga" else pm.pet_svrg_epoch
    epoch(g, st, x, state["order"], state["tau"], state["update"])
    return x, st.ghat_i, st.ghat, st.D


def work(case):
    """Bytes: each input read once, each output written once (of the subset's
    views).  Operations: per Joseph sample one axial interpolation (3) each way,
    with TOF a multiply-add per overlapping bin each way; per voxel and
    neighbour of the prior 12."""
    op = case["op"]
    n_p, n_lor, n_bin, n_vox = _sizes(case)
    views = _views(case)
    nt = case["n_tof"]
    lor = len(views) * case["n_rad"] * n_p
    s, h = _radial(case)
    rows = 0.0
    wx, wy = case["nx"] * case["vx"], case["ny"] * case["vy"]
    some = views[::max(1, len(views) // 8)]
    for v in some:
        c, t = abs(math.cos(math.pi * v / case["n_views"])), abs(math.sin(math.pi * v / case["n_views"]))
        along, across, n, vox = (wy, wx, case["ny"], case["vy"]) if c >= t else (wx, wy, case["nx"], case["vx"])
        big, small = max(c, t), min(c, t)
        m = (np.arange(n) - 0.5 * (n - 1)) * vox
        rows += float((np.abs(s[:, None] - small * m[None, :]) <= big * (0.5 * across)).sum())
    samples = rows * len(views) / len(some) * n_p
    over = 1.0 if nt == 1 else min(nt, (case["tof_bin"] + 2 * case["tof_nsigma"] * case["tof_sigma"]) / case["tof_bin"])
    way = 3.0 + (2.0 * over if nt > 1 else 0.0)  # operations of a sample, one way
    img = 4.0 * n_vox
    ysize = {"u8": 1, "u16": 2, "f32": 4}.get(case.get("y"), 0)
    n_neigh = 26 if case["nz"] > 1 else 8
    rdp = 12.0 * n_neigh * n_vox
    if op == "rdp":
        return {"bytes": 3 * img, "flops": rdp}
    if op == "grad":
        return {"bytes": lor * nt * (ysize + 4.0) + 4.0 * lor + 2 * img, "flops": 2 * way * samples}
    if op == "fwd":
        return {"bytes": lor * nt * 8.0 + 4.0 * lor + img, "flops": way * samples}
    if op == "back":
        return {"bytes": lor * nt * 4.0 + 4.0 * lor + img, "flops": way * samples}
    if op == "sens":
        return {"bytes": 4.0 * lor + img, "flops": 3.0 * samples}
    if op == "hvp":
        return {"bytes": lor * nt * (ysize + 4.0) + 4.0 * lor + 3 * img, "flops": 3 * way * samples}
    # bins with counts: 16 bytes each (index, y, add, mult); their samples lie
    # in one bin's window
    prompts = min(1.25 * case["counts"] * len(views) / case["n_views"], 0.5 * lor * nt)
    per_bin = samples / lor * (over / nt if nt > 1 else 1.0)
    if op == "counts":
        return {"bytes": 16.0 * prompts + 2 * img, "flops": 2 * (3.0 + (2.0 if nt > 1 else 0.0)) * per_bin * prompts}
    passes = 2 * case["n_subsets"] - 1
    each = dict(case, op="counts", subset=0)
    w = work(each)
    return {"bytes": passes * w["bytes"] + case["n_subsets"] * 6 * img, "flops": passes * w["flops"] + case["n_subsets"] * rdp}


# ---- FP64 evaluation with plain torch ---------------------------------------
def _view_tables(case, view, dev):
    """Principal axis and the Joseph sample positions of one view: lambda and the
    transaxial coordinate of every (radial, row), the step length's factor."""
    n = (case["nx"], case["ny"])
    vox = (case["vx"], case["vy"])
    org = tuple(-0.5 * (a - 1) * b for a, b in zip(n, vox))
    s, h = _radial(case)
    phi = math.pi * view / case["n_views"]
    c, t = math.cos(phi), math.sin(phi)
    p = (s * c + h * t, s * t - h * c)
    u = (-2 * h * t, 2 * h * c)
    rx, ry = abs(t) / vox[0], abs(c) / vox[1]
    m = 1 if ry > rx * (1 + 1e-9) else 0
    a = 1 - m
    i = np.arange(n[m])
    lam = (org[m] + i[None, :] * vox[m] - p[m][:, None]) / u[m][:, None]
    xa = (p[a][:, None] + lam * u[a][:, None] - org[a]) / vox[a]
    f64 = dict(dtype=torch.float64, device=dev)
    return dict(m=m, na=n[a], lam=torch.tensor(lam, **f64), xa=torch.tensor(xa, **f64),
                step=torch.tensor(vox[m] / np.abs(u[m]), **f64), lt2=torch.tensor(4 * h * h, **f64))


def _segments(case):
    z1, z2 = _axial(case)
    org = -0.5 * (case["nz"] - 1) * case["vz"]
    zb, zs = (z1 - org) / case["vz"], (z2 - z1) / case["vz"]
    dz = z2 - z1
    out, p0 = [], 0
    for p in range(1, len(z1) + 1):
        if p == len(z1) or dz[p] != dz[p0]:
            out.append((p0, p, zb[p0:p], zs[p0], dz[p0]))
            p0 = p
    return out


def _tof_weights(case, t):
    """Weights of the bins at signed distances t: [..., T]."""
    nt, w, sg, ns = case["n_tof"], case["tof_bin"], case["tof_sigma"], case["tof_nsigma"]
    edge = (torch.arange(nt + 1, device=t.device, dtype=t.dtype) - 0.5 * nt) * w
    e = torch.erf(((edge - t[..., None]) / (math.sqrt(2.0) * sg)).clamp(-ns / math.sqrt(2.0), ns / math.sqrt(2.0)))
    return 0.5 * (e[..., 1:] - e[..., :-1])


def _walk(case, view, img, q_of, back):
    """One view: forward integrals of img (nz, ny, nx; None: not wanted) handed to
    q_of(p0, p1, integrals [R, np, T]) segment by segment; what it returns
    (back: [R, np, T], None: nothing) goes back into an (nz, ny, nx) image."""
    dev = torch.device("cuda:0")
    tab = _view_tables(case, view, dev)
    nr, n = tab["lam"].shape
    nz, na, tof = case["nz"], tab["na"], case["n_tof"] > 1
    jf = torch.floor(tab["xa"])
    f = (tab["xa"] - jf)[..., None]
    j = (jf.long() + 2).clamp(0, na + 2)
    inside = ((jf >= -2) & (jf <= na))[..., None]
    rows = torch.arange(n, device=dev)[None, :].expand(nr, n)
    if img is not None:
        t = img.permute(2, 1, 0) if tab["m"] == 0 else img.permute(1, 2, 0)  # [principal][other][z]
        t = torch.nn.functional.pad(t, (2, 2, 2, 2))
        sheet = (t[rows, j] * (1 - f) + t[rows, (j + 1).clamp(max=na + 3)] * f) * inside
        sheet = sheet.contiguous()
    z_out = torch.zeros((nr, n, nz + 4), dtype=torch.float64, device=dev) if back else None
    for p0, p1, zb, zs, dz in _segments(case):
        length = torch.sqrt(tab["lt2"] + dz * dz)
        ell = (tab["step"] * length)[:, None, None]
        u = torch.tensor(zb, dtype=torch.float64, device=dev) + (tab["lam"] * zs)[..., None]
        k = torch.floor(u)
        fz = u - k
        ok = (k >= -2) & (k <= nz)
        k = (k.long() + 2).clamp(0, nz + 2)
        w = _tof_weights(case, (tab["lam"] - 0.5) * length[:, None]) if tof else None  # [R, N, T]
        vals = None
        if img is not None:
            v = (sheet.gather(2, k) * (1 - fz) + sheet.gather(2, k + 1) * fz) * ok
            if tof:
                vals = torch.matmul(v.transpose(1, 2).contiguous(), w) * ell
            else:
                vals = v.sum(1)[..., None] * ell
        q = q_of(p0, p1, vals)
        if back:
            q = q * ell
            if tof:
                q = torch.matmul(w, q.transpose(1, 2).contiguous())  # [R, N, np]
            else:
                q = q[..., 0][:, None, :].expand(nr, n, p1 - p0)
            q = q * ok
            z_out.scatter_add_(2, k, q * (1 - fz))
            z_out.scatter_add_(2, k + 1, q * fz)
    if not back:
        return None
    t = torch.zeros((n, na + 4, nz), dtype=torch.float64, device=dev)
    zi = z_out[..., 2:nz + 2] * inside
    t.index_put_((rows, j), zi * (1 - f), accumulate=True)
    t.index_put_((rows, (j + 1).clamp(max=na + 3)), zi * f, accumulate=True)
    t = t[:, 2:na + 2]
    return t.permute(2, 1, 0) if tab["m"] == 0 else t.permute(2, 0, 1)


def _psf(case, img):
    fw = case.get("psf_fwhm", 0.0)
    if not fw:
        return img
    axes = [("vx", 2), ("vy", 1)] + ([("vz", 0)] if case["nz"] > 1 else [])
    for vox, ax in axes:
        sg = fw * FWHM / case[vox]
        r = int(4.0 * sg + 0.5)
        w = np.exp(-0.5 * (np.arange(-r, r + 1) / sg) ** 2)
        w /= w.sum()
        n = img.shape[ax]
        out = torch.zeros_like(img)
        for d in range(-r, r + 1):
            if abs(d) < n:
                lo, hi = max(0, -d), min(n, n - d)
                out.narrow(ax, lo, hi - lo).add_(img.narrow(ax, lo + d, hi - lo), alpha=float(w[d + r]))
        img = out
    return img


def _image(case, flat):
    return flat.double().view(case["nz"], case["ny"], case["nx"])


def _bins(case, d, key, view, p0, p1):
    n_p = len(_planes(case))
    return d[key].view(case["n_views"], case["n_rad"], n_p, -1)[view, :, p0:p1].double()


def _data_grad(case, d, img, views, counts_only=False):
    """P^T [mult (1 - y / ybar)] (counts_only: P^T [-mult y / ybar]) and the KL sum."""
    gx = _psf(case, img)
    grad = torch.zeros_like(img)
    kl = torch.zeros(1, dtype=torch.float64, device=img.device)
    for v in views:
        def q_of(p0, p1, fwd):
            m, y = _bins(case, d, "mult", v, p0, p1), _bins(case, d, "y", v, p0, p1)
            yb = m * fwd + _bins(case, d, "add", v, p0, p1)
            kl.add_((yb - y + torch.xlogy(y, y / yb)).sum())
            return m * ((0.0 if counts_only else 1.0) - y / yb)
        grad += _walk(case, v, gx, q_of, True)
    return _psf(case, grad), kl


def _rdp(case, img, beta, gamma, eps, want_hess=True):
    g, h = torch.zeros_like(img), torch.zeros_like(img)
    val = torch.zeros(1, dtype=torch.float64, device=img.device)
    nz, ny, nx = img.shape
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if not (dz or dy or dx):
                    continue
                # (the library takes its weights as 32-bit numbers)
                w = float(np.float32(case["vx"] / math.sqrt((dz * case["vz"]) ** 2 + (dy * case["vy"]) ** 2 + (dx * case["vx"]) ** 2)))
                me, ne = [], []
                for off, n in ((dz, nz), (dy, ny), (dx, nx)):
                    me.append(slice(max(0, -off), min(n, n - off)))
                    ne.append(slice(max(0, off), min(n, n + off)))
                if any(s.stop <= s.start for s in me):
                    continue
                xi, xj = img[tuple(me)], img[tuple(ne)]
                df = xi - xj
                phi = xi + xj + gamma * df.abs() + eps
                g[tuple(me)] += w * df * (2 * phi - df - gamma * df.abs()) / phi ** 2
                if want_hess:
                    h[tuple(me)] += 2 * w * (2 * xj + eps) ** 2 / phi ** 3
                val += 0.5 * w * (df * df / phi).sum()
    return beta * g, beta * h, beta * val


def _f32(v):
    return float(np.float32(v))


def exact(case, seed):
    op = case["op"]
    if op == "svrg":
        return None  # 49 subset gradients of the largest workload
    if op == "sens" and work(case)["flops"] > 8e10:
        return None
    d = _inputs(case, seed, data=op != "rdp", sino=op == "back")
    img = _image(case, d["x"])
    views = _views(case)
    if op == "rdp":
        eps = _f32(1e-3 * float(d["x"].max()))
        g, h, v = _rdp(case, img, _f32(_beta(case)), 2.0, eps)
        return g.flatten(), h.flatten(), v
    if op == "grad":
        g, kl = _data_grad(case, d, img, views)
        return (g.flatten(), kl) if case.get("kl") else g.flatten()
    if op == "counts":
        return _data_grad(case, d, img, views, True)[0].flatten()
    if op == "fwd":
        n_p, _, n_bin, _ = _sizes(case)
        out = torch.zeros((case["n_views"], case["n_rad"], n_p, case["n_tof"]), dtype=torch.float64, device=img.device)
        gx = _psf(case, img)
        for v in views:
            def q_of(p0, p1, fwd):
                out[v, :, p0:p1] = _bins(case, d, "mult", v, p0, p1) * fwd + _bins(case, d, "add", v, p0, p1)
            _walk(case, v, gx, q_of, False)
        return out.flatten()
    if op in ("back", "sens"):
        out = torch.zeros_like(img)
        for v in views:
            def q_of(p0, p1, fwd):
                m = _bins(case, d, "mult", v, p0, p1)
                return m * _bins(case, d, "sino", v, p0, p1) if op == "back" else m.expand(-1, -1, case["n_tof"])
            out += _walk(case, v, None, q_of, True)
        return _psf(case, out).flatten()
    if op == "hvp":
        out = torch.zeros_like(img)
        gx, gv = _psf(case, img), _psf(case, _image(case, d["v"]))
        for v in views:
            ybar = {}

            def first(p0, p1, fwd):
                ybar[p0] = _bins(case, d, "mult", v, p0, p1) * fwd + _bins(case, d, "add", v, p0, p1)

            def second(p0, p1, fwd):
                m = _bins(case, d, "mult", v, p0, p1)
                return m * m * _bins(case, d, "y", v, p0, p1) / ybar[p0] ** 2 * fwd
            _walk(case, v, gx, first, False)
            out += _walk(case, v, gv, second, True)
        return _psf(case, out).flatten()
    return _exact_saga(case, seed, d, img)


def _exact_saga(case, seed, d, x):
    """First SAGA epoch with the table of h_i + (beta / n) grad S, where h_i is
    the part of a subset's data gradient that depends on the image."""
    n = case["n_subsets"]
    beta, eps = _f32(_beta(case)), _f32(1e-3 * float(d["x"].max()))
    sens = torch.zeros_like(x)
    for v in range(case["n_views"]):
        sens += _walk(case, v, None, lambda p0, p1, fwd: _bins(case, d, "mult", v, p0, p1).expand(-1, -1, case["n_tof"]), True)

    def h_of(i, img):
        return _data_grad(case, d, img, range(i, case["n_views"], n), True)[0]

    sens = _psf(case, sens)
    bg, bh, _ = _rdp(case, x, beta, 2.0, eps)
    table = [h_of(i, x) + bg / n for i in range(n)]
    total = sens + sum(table)
    den = sens + bh * (x + eps)
    prec = torch.where(den != 0, (x + eps) / den, torch.zeros_like(den))
    for j, i in enumerate(_order(case, seed)):
        if j == 0:
            est = total
        else:
            ji = h_of(i, x) + _rdp(case, x, beta, 2.0, eps, False)[0] / n
            est = n * (ji - table[i]) + total
            total = total + ji - table[i]
            table[i] = ji
        x = torch.clamp(x - _f32(1.0 / (1.0 + 0.02 * j / n)) * prec * est, min=0.0)
    return x.flatten(), torch.stack([t.flatten() for t in table]), total.flatten(), prec.flatten()
