// Host-side geometry (FP64) for the gfx950 PET library: LOR endpoints from the
// scanner description, per-line Joseph sampling parameters, per-plane axial
// parameters, TOF interval table and TOF weight table, plus the scratch arena.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

#include "pet_internal.h"

using namespace pet;

namespace {

struct Plane {
    int r1, r2, seg;
};

std::vector<Plane> make_planes(const pet_geom_desc &d) {
    std::vector<Plane> out;
    if (d.kind == PET_SCANNER_PARALLEL2D) {
        out.push_back({0, 0, 0});
        return out;
    }
    std::vector<int> segs{0};
    for (int k = 1; k <= d.max_ring_diff; ++k) {
        segs.push_back(-k);
        segs.push_back(k);
    }
    for (size_t si = 0; si < segs.size(); ++si) {
        int dd = segs[si];
        for (int r1 = std::max(0, -dd); r1 < std::min(d.n_rings, d.n_rings - dd); ++r1)
            out.push_back({r1, r1 + dd, (int)si});
    }
    return out;
}

pet_status validate(const pet_geom_desc &d) {
    if (d.kind != PET_SCANNER_PARALLEL2D && d.kind != PET_SCANNER_CYLINDER)
        return fail(PET_E_ARG, "pet_geom_create: unknown scanner kind");
    if (d.nx < 1 || d.ny < 1 || d.nz < 1 || !(d.vx > 0) || !(d.vy > 0) || !(d.vz > 0))
        return fail(PET_E_ARG, "pet_geom_create: image sizes and voxel sizes must be positive");
    if (d.nz > 400) return fail(PET_E_ARG, "pet_geom_create: at most 400 axial voxels");
    if ((int64_t)d.nx * d.ny * d.nz >= ((int64_t)1 << 31)) return fail(PET_E_ARG, "pet_geom_create: too many voxels");
    if (d.nx > 32000 || d.ny > 32000 || d.nz > 32000)
        return fail(PET_E_ARG, "pet_geom_create: image dimension too large");
    if (d.n_views < 1 || d.n_rad < 1) return fail(PET_E_ARG, "pet_geom_create: n_views and n_rad must be >= 1");
    if (d.n_subsets < 1 || d.n_subsets > d.n_views)
        return fail(PET_E_ARG, "pet_geom_create: need 1 <= n_subsets <= n_views");
    if (d.n_tof < 1 || d.n_tof > NT_MAX) return fail(PET_E_ARG, "pet_geom_create: n_tof must be in [1, 32]");
    if (d.n_tof > 1 && (!(d.tof_bin_mm > 0) || !(d.tof_sigma_mm > 0) || !(d.tof_nsigma > 0)))
        return fail(PET_E_ARG, "pet_geom_create: TOF needs tof_bin_mm, tof_sigma_mm, tof_nsigma > 0");
    if (d.kind == PET_SCANNER_CYLINDER) {
        if (!(d.radius_mm > 0) || d.n_crystals != 2 * d.n_views || d.n_rings < 1 || !(d.ring_pitch_mm > 0) ||
            d.max_ring_diff < 0 || d.max_ring_diff >= d.n_rings)
            return fail(PET_E_ARG, "pet_geom_create: inconsistent cylinder description "
                                   "(need radius > 0, n_crystals = 2 n_views, 0 <= max_ring_diff < n_rings)");
        if (d.n_rad > d.n_crystals) return fail(PET_E_ARG, "pet_geom_create: n_rad > n_crystals");
    } else {
        if (d.nz != 1) return fail(PET_E_ARG, "pet_geom_create: 2D parallel-beam geometry needs nz = 1");
        if (!(d.rad_spacing_mm > 0) || !(d.half_length_mm > 0))
            return fail(PET_E_ARG, "pet_geom_create: parallel-beam needs rad_spacing_mm, half_length_mm > 0");
    }
    if (!(d.psf_fwhm_mm >= 0) || !std::isfinite(d.psf_fwhm_mm))
        return fail(PET_E_ARG, "pet_geom_create: psf_fwhm_mm must be finite and >= 0");
    return PET_OK;
}

// Separable Gaussian of the resolution model, one axis: sigma in voxels,
// radius floor(4 sigma + 1/2), weights normalised to sum 1 over -r..r.
bool make_psf_axis(double sigma_vox, int axis, PsfAxis &k) {
    const int r = (int)(4.0 * sigma_vox + 0.5);
    if (r > PSF_RMAX) return false;
    double w[PSF_RMAX + 1], sum = 0.0;
    for (int i = 0; i <= r; ++i) {
        w[i] = std::exp(-0.5 * (double)i * i / (sigma_vox * sigma_vox));
        sum += i == 0 ? w[i] : 2.0 * w[i];
    }
    k.r = r;
    k.axis = axis;
    for (int i = 0; i <= PSF_RMAX; ++i) k.w[i] = i <= r ? (float)(w[i] / sum) : 0.f;
    return true;
}

// Positions of the voxels in rings, shifted by one, for the axial gather
// (line_sheets.h): z / kappa + ring0 + 1 in 32 bits.
//
// A voxel exactly one voxel away from a direct plane (ring difference 0, at the same
// place in every row) does not see it, but its weight, 1 - kappa times their
// distance in rings, may come out as 1e-7.  Its position is then moved by as many
// units in the last place, few, as make the form's weight zero or less.  (With
// rings three voxels apart the slices between them got a sensitivity of 1e-7, and
// an OSEM image was off by its own size.)
std::vector<float> gather_positions(int nz, int n_rings, double kappa_d, double ring0, int form) {
    const float kappa = (float)kappa_d;
    // weight of ring r at shifted position t, as the form computes it
    auto weight = [&](float t, int r) {
        if (form == 2) {
            const int c = r + 1 - (int)std::floor(t);  // ring below (0) or above (1) the voxel
            const float f = t - std::floor(t);
            return c == 0 ? std::fmaf(-kappa, f, 1.f) : c == 1 ? std::fmaf(kappa, f, 1.f - kappa) : 0.f;
        }
        if (form == 3) {
            const float u = t + GATHER_THREE, f = u - std::floor(u);
            const int c = r + 2 - (int)std::floor(u);  // ring below (-1), at (0) or above (1) the nearest
            return c == 0    ? std::fmaf(-kappa, std::fabs(f - 0.5f), 1.f)
                   : c == -1 ? std::fmaf(-kappa, f, std::fmaf(-0.5f, kappa, 1.f))
                   : c == 1  ? std::fmaf(kappa, f, std::fmaf(-1.5f, kappa, 1.f))
                             : 0.f;
        }
        return std::fmaf(-kappa, std::fabs(t - (float)(r + 1)), 1.f);
    };
    std::vector<float> rho(nz);
    for (int z = 0; z < nz; ++z) {
        const float t0 = (float)(z / kappa_d + (ring0 + 1.0));
        std::vector<int> missed;  // rings exactly one voxel away
        for (int r = 0; r < n_rings; ++r)
            if (std::fabs(std::fabs((r - ring0) * kappa_d - z) - 1.0) < 1e-9) missed.push_back(r);
        rho[z] = t0;
        for (int step = 0; step <= 32 && !missed.empty(); ++step) {
            const float t = t0 + (float)((step & 1 ? 1 : -1) * ((step + 1) / 2)) * (std::nextafter(std::fabs(t0), 1e30f) - std::fabs(t0));
            if (std::all_of(missed.begin(), missed.end(), [&](int r) { return weight(t, r) <= 0.f; })) {
                rho[z] = t;
                break;
            }
        }
    }
    return rho;
}

}  // namespace

extern "C" pet_status pet_geom_create(const pet_geom_desc *desc, pet_geom *out) {
    if (!desc || !out) return fail(PET_E_ARG, "pet_geom_create: null argument");
    const pet_geom_desc &d = *desc;
    pet_status st = validate(d);
    if (st != PET_OK) return st;

    pet_geom_s *g = new (std::nothrow) pet_geom_s();
    if (!g) return fail(PET_E_OOM, "pet_geom_create: host allocation failed");
    g->d = d;
    if (d.psf_fwhm_mm > 0) {
        const double sig = d.psf_fwhm_mm / (2.0 * std::sqrt(2.0 * std::log(2.0)));
        const double vox[3] = {d.vx, d.vy, d.vz};
        g->psf_passes = d.nz > 1 ? 3 : 2;
        for (int a = 0; a < g->psf_passes; ++a)
            if (!make_psf_axis(sig / vox[a], a, g->psf[a])) {
                delete g;
                return fail(PET_E_ARG, "pet_geom_create: resolution kernel wider than 16 voxels");
            }
    }
    if (hipGetDevice(&g->device) != hipSuccess) {
        delete g;
        return fail(PET_E_HIP, "pet_geom_create: no HIP device");
    }
    std::vector<Plane> planes = make_planes(d);
    g->n_planes = (int)planes.size();
    g->n_vox = (int64_t)d.nx * d.ny * d.nz;
    for (auto &p : planes) g->seg_of_plane.push_back(p.seg);

    const int N[3] = {d.nx, d.ny, d.nz};
    const double V[3] = {d.vx, d.vy, d.vz};
    double O[3];
    for (int a = 0; a < 3; ++a) O[a] = -0.5 * (N[a] - 1) * V[a];

    // axial table
    std::vector<double> z1(planes.size()), z2(planes.size());
    double max_dz = 0.0;
    for (size_t p = 0; p < planes.size(); ++p) {
        if (d.kind == PET_SCANNER_CYLINDER) {
            z1[p] = (planes[p].r1 - 0.5 * (d.n_rings - 1)) * d.ring_pitch_mm;
            z2[p] = (planes[p].r2 - 0.5 * (d.n_rings - 1)) * d.ring_pitch_mm;
        } else {
            z1[p] = z2[p] = 0.0;
        }
        max_dz = std::max(max_dz, std::fabs(z2[p] - z1[p]));
    }
    std::vector<PlaneP> hplanes(planes.size());
    for (size_t p = 0; p < planes.size(); ++p) {
        hplanes[p].zb = (float)((z1[p] - O[2]) / V[2]);
        hplanes[p].zs = (float)((z2[p] - z1[p]) / V[2]);
        hplanes[p].dz2 = (float)((z2[p] - z1[p]) * (z2[p] - z1[p]));
        hplanes[p].q = 0;
    }

    // line table
    const int nl = d.n_views * d.n_rad;
    std::vector<LineP> hlines(nl);
    int rows_max = 0;
    for (int v = 0; v < d.n_views; ++v) {
        double phi = M_PI * v / d.n_views;
        double nx_ = std::cos(phi), ny_ = std::sin(phi), tx = -std::sin(phi), ty = std::cos(phi);
        for (int k = 0; k < d.n_rad; ++k) {
            double s, h;
            if (d.kind == PET_SCANNER_CYLINDER) {
                s = d.radius_mm * std::sin(M_PI * (k - 0.5 * (d.n_rad - 1)) / d.n_crystals);
                h = std::sqrt(d.radius_mm * d.radius_mm - s * s);
            } else {
                s = (k - 0.5 * (d.n_rad - 1)) * d.rad_spacing_mm;
                h = d.half_length_mm;
            }
            double p1[2] = {s * nx_ - h * tx, s * ny_ - h * ty};
            double u[2] = {2 * h * tx, 2 * h * ty};
            double rx = std::fabs(u[0]) / V[0], ry = std::fabs(u[1]) / V[1];
            int m = (ry > rx * (1.0 + 1e-9)) ? 1 : 0;
            double best = std::max(rx, ry);
            if (max_dz / V[2] > best * (1.0 + 1e-9)) {
                delete g;
                return fail(PET_E_ARG, "pet_geom_create: some LOR has z as principal axis (unsupported)");
            }
            int a = 1 - m;
            LineP L{};
            double lam0 = (O[m] - p1[m]) / u[m];
            double dlam = V[m] / u[m];
            double xa0 = (p1[a] + lam0 * u[a] - O[a]) / V[a];
            double dxa = dlam * u[a] / V[a];
            double lo_c, hi_c;
            if (dxa == 0.0) {
                bool in = xa0 >= -1.5 && xa0 <= N[a] + 0.5;
                lo_c = in ? 0 : 1;
                hi_c = in ? N[m] - 1 : 0;
            } else {
                double ia = (-1.5 - xa0) / dxa, ib = (N[a] + 0.5 - xa0) / dxa;
                lo_c = std::ceil(std::min(ia, ib));
                hi_c = std::floor(std::max(ia, ib));
            }
            // clamp in floating point before converting (near-axis-aligned lines
            // that miss the grid give bounds far outside the int range)
            lo_c = std::max(0.0, lo_c);
            hi_c = std::min((double)N[m] - 1, hi_c);
            int i_lo = 1, i_hi = 0;
            if (lo_c <= hi_c) {
                i_lo = (int)lo_c;
                i_hi = (int)hi_c;
                double l_a = lam0 + i_lo * dlam, l_b = lam0 + i_hi * dlam;
                if (std::min(l_a, l_b) < 0.0 || std::max(l_a, l_b) > 1.0) {
                    delete g;
                    return fail(PET_E_ARG, "pet_geom_create: LOR endpoints lie inside the padded image box");
                }
                rows_max = std::max(rows_max, i_hi - i_lo + 1);
            }
            L.lam0 = (float)lam0;
            L.dlam = (float)dlam;
            L.xa0 = (float)xa0;
            L.dxa = (float)dxa;
            L.vm_um = (float)(V[m] / std::fabs(u[m]));
            L.lt2 = (float)(u[0] * u[0] + u[1] * u[1]);
            L.i_lo = (int16_t)i_lo;
            L.i_hi = (int16_t)i_hi;
            L.axis = m;
            hlines[(size_t)v * d.n_rad + k] = L;
        }
    }

    // subsets: views v = i (mod n)
    g->subset_views.resize(d.n_subsets);
    for (int v = 0; v < d.n_views; ++v) g->subset_views[v % d.n_subsets].push_back(v);
    g->max_views = (int)g->subset_views[0].size();
    g->views_stride = d.n_views;
    std::vector<int> hviews((size_t)(d.n_subsets + 1) * d.n_views, 0);
    for (int i = 0; i < d.n_subsets; ++i)
        for (size_t j = 0; j < g->subset_views[i].size(); ++j) hviews[(size_t)i * d.n_views + j] = g->subset_views[i][j];
    for (int v = 0; v < d.n_views; ++v) hviews[(size_t)d.n_subsets * d.n_views + v] = v;
    // line launches: the lines of each subset (then of all views),
    // longest first (a line's work grows with its rows), so that the last
    // workgroups of a launch run short lines
    std::vector<int> horder;
    horder.reserve(2 * (size_t)d.n_views * d.n_rad);
    for (int row = 0; row <= d.n_subsets; ++row) {
        g->order_off.push_back((int64_t)horder.size());
        const size_t start = horder.size();
        const int nvr = row < d.n_subsets ? (int)g->subset_views[row].size() : d.n_views;
        for (int j = 0; j < nvr; ++j)
            for (int k = 0; k < d.n_rad; ++k) horder.push_back(hviews[(size_t)row * d.n_views + j] * d.n_rad + k);
        auto rows_of = [&](int l) { return std::max(0, hlines[l].i_hi - hlines[l].i_lo + 1); };
        std::stable_sort(horder.begin() + start, horder.end(), [&](int p, int q) { return rows_of(p) > rows_of(q); });
    }

    // TOF tables
    TofTable &T = g->tof;
    T.n_tof = d.n_tof;
    if (d.n_tof > 1) {
        double cut = 0.5 * d.tof_bin_mm + d.tof_nsigma * d.tof_sigma_mm;  // support of a bin's weight
        std::vector<double> tb(d.n_tof), edges;
        for (int b = 0; b < d.n_tof; ++b) {
            tb[b] = (b - 0.5 * (d.n_tof - 1)) * d.tof_bin_mm;
            T.tb[b] = (float)tb[b];
            edges.push_back(tb[b] - cut);
            edges.push_back(tb[b] + cut);
        }
        std::sort(edges.begin(), edges.end());
        std::vector<double> ue;
        for (double e : edges)
            if (ue.empty() || e - ue.back() > 1e-9 * (1.0 + std::fabs(e))) ue.push_back(e);
        T.n_int = (int)ue.size() - 1;
        for (size_t e = 0; e < ue.size(); ++e) T.edge[e] = (float)ue[e];
        for (int s = 0; s < T.n_int; ++s) {
            double mid = 0.5 * (ue[s] + ue[s + 1]);
            int bf = -1, bl = -1;
            for (int b = 0; b < d.n_tof; ++b)
                if (std::fabs(mid - tb[b]) <= cut) {
                    if (bf < 0) bf = b;
                    bl = b;
                }
            if (bf < 0) {
                bf = 0;
                bl = -1;
            }
            T.bf[s] = bf;
            T.na[s] = bl - bf + 1;
            if (T.na[s] > 8) {
                delete g;
                return fail(PET_E_ARG, "pet_geom_create: more than 8 TOF bins overlap at one point");
            }
        }
        T.half_bin = (float)(0.5 * d.tof_bin_mm);
        T.inv_sqrt2_sigma = (float)(1.0 / (std::sqrt(2.0) * d.tof_sigma_mm));
        T.erf_clamp = (float)(d.tof_nsigma / std::sqrt(2.0));
    } else {
        T.n_int = 0;
    }

    // segments (contiguous plane ranges of equal ring difference)
    std::vector<SegP> gsegs;
    for (size_t p = 0; p < planes.size(); ++p) {
        if (gsegs.empty() || planes[p].seg != planes[p - 1].seg) gsegs.push_back({(int)p, 0, hplanes[p].dz2, 0});
        gsegs.back().np++;
    }
    // Axial gather of the adjoint: segments in parts of at most GATHER_PLANES
    // planes, in chunks whose factors fit the LDS beside the image sheet.  The
    // cap holds every plane of any scanner here (2204 planes take 9 KB); it
    // never exceeds what the two FP64 sheets' worth of LDS checked below leaves.
    if (d.kind == PET_SCANNER_CYLINDER) {
        g->kappa = d.ring_pitch_mm / d.vz;
        g->ring0 = -(-0.5 * (d.n_rings - 1) * d.ring_pitch_mm - O[2]) / d.ring_pitch_mm;
    }
    std::vector<GatherSeg> hgather;
    std::vector<GatherChunk> hchunks;
    {
        const size_t sheet_f = ((size_t)rows_max * (d.nz + 2 * PADZ) + 3) & ~(size_t)3;
        const int cap = (int)std::max<size_t>(2 * sheet_f, 12288);
        struct Part {
            int p0, np, k, off;  // first plane, planes, ring difference, ranks before the first
        };
        std::vector<Part> part;
        auto flush = [&]() {
            if (part.empty()) return;
            GatherChunk c{};
            c.s0 = (int)hgather.size();
            c.p0 = part.front().p0;
            c.p1 = part.back().p0 + part.back().np;
            int at = GATHER_ZEROS;  // (before the first part and after each)
            std::vector<int> qb(part.size());
            for (size_t i = 0; i < part.size(); ++i) {
                for (int j = 0; j < part[i].np; ++j) hplanes[part[i].p0 + j].q = at + j;
                qb[i] = at - 1 - part[i].off;
                at += part[i].np + GATHER_ZEROS;
            }
            c.n_q = at;
            for (int neg = 0; neg < 2; ++neg) {
                if (neg) c.s_neg = (int)hgather.size();
                for (size_t i = 0; i < part.size(); ++i) {
                    if ((part[i].k < 0) != (neg == 1)) continue;
                    hgather.push_back({(float)std::abs(part[i].k), (float)part[i].off,
                                       (float)(part[i].off + part[i].np + 1), qb[i]});
                }
            }
            c.s1 = (int)hgather.size();
            hchunks.push_back(c);
            g->q_floats = std::max(g->q_floats, (at + 3) & ~3);
            part.clear();
        };
        int used = GATHER_ZEROS;
        for (const SegP &sg : gsegs)
            for (int off = 0; off < sg.np; off += GATHER_PLANES) {
                const int np = std::min(GATHER_PLANES, sg.np - off);
                if (used + np + GATHER_ZEROS > cap) {
                    flush();
                    used = GATHER_ZEROS;
                }
                part.push_back({sg.p0 + off, np, planes[sg.p0].r2 - planes[sg.p0].r1, off});
                used += np + GATHER_ZEROS;
            }
        flush();
    }
    g->n_gchunk = (int)hchunks.size();
    g->gather_planes = gather_form((float)g->kappa);
    for (const SegP &sg : gsegs)
        if (sg.np > GATHER_PLANES) g->gather_planes = GATHER_SOME;
    const std::vector<float> hrho = gather_positions(d.nz, d.kind == PET_SCANNER_CYLINDER ? d.n_rings : 1, g->kappa, g->ring0, g->gather_planes);
    g->rows_max = rows_max;
    // non-TOF: one thread per plane, in as many waves as the planes need (up to
    // 16; more resident waves hide the LDS latency of the sample loop)
    g->nt_threads = std::min(NT_BLOCK, std::max(64, (g->n_planes + 63) / 64 * 64));
    if (d.n_tof > 1) {
        for (const SegP &sg : gsegs)
            if (sg.np > 64) {
                delete g;
                return fail(PET_E_ARG, "pet_geom_create: TOF needs at most 64 planes per segment (one wave)");
            }
        g->tof_ws = 1;
        for (int s = 0; s < T.n_int; ++s) g->tof_ws = std::max(g->tof_ws, T.na[s]);
    }

    // Largest image served: three sheets of floats in LDS and, with TOF, one wave's
    // tables (the TOF walk; the other line kernels need less).
    int rz = d.nz + 2 * PADZ;
    size_t sheet = ((size_t)rows_max * rz + 3) & ~(size_t)3;
    int max_lds = 0;
    if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, g->device) != hipSuccess) max_lds = 0;
    if (max_lds <= 0) max_lds = 64 * 1024;
    g->max_lds = (size_t)max_lds;
    size_t need = 3 * sheet * sizeof(float);
    const size_t walk_wave = d.n_tof > 1 ? walk_wave_floats(rows_max, g->tof_ws, T.n_int) * sizeof(float) : 0;
    need += walk_wave;
    if (need > (size_t)max_lds) {
        delete g;
        return fail(PET_E_ARG, "pet_geom_create: image too large for the LDS sheets of the line kernels (" +
                                   std::to_string(need) + " > " + std::to_string(max_lds) + " bytes)");
    }

    // TOF line kernels: units, LDS split, table of the halved clamped erf
    std::vector<TofUnit> hunits;
    std::vector<float4> hetab;
    std::vector<int> hwalk;
    if (d.n_tof > 1) {
        auto ring_d = [&](const SegP &sg) { return planes[sg.p0].r2 - planes[sg.p0].r1; };
        int max_np = 0;
        for (const SegP &sg : gsegs) {
            const int k = std::abs(ring_d(sg)), neg = ring_d(sg) < 0;
            if (!hunits.empty()) {
                // segments -k and +k are adjacent in the plane order; they have
                // the same oblique length, so a pair that fits 64 lanes is one
                // unit (its weights are formed once)
                TofUnit &m = hunits.back();
                if (k > 0 && m.n1 == m.np && (int)m.k == k && m.p0 + m.np == sg.p0 && m.np + sg.np <= 64) {
                    m.np = (uint8_t)(m.np + sg.np);
                    max_np = std::max(max_np, (int)m.np);
                    continue;
                }
            }
            hunits.push_back({sg.p0, (uint8_t)sg.np, (uint8_t)sg.np, (uint8_t)neg, 0, sg.dz2, (float)k});
            max_np = std::max(max_np, sg.np);
        }
        g->n_units = (int)hunits.size();
        // TOF walk: as many waves as its LDS holds (up to 16: they wait on LDS
        // latency); wave w takes entries w, w + W, w + 2W, ... of the order.  The two
        // halves -k and +k of a pair of single segments have the same oblique length
        // and so the same weight table, and go to consecutive rounds of one wave, which
        // then fills the table once (both carry the same squared axial extent).  The
        // other units keep their relative order.
        const int ns = g->n_units;
        const int W = std::max(1, std::min({ns, MAX_WAVES, (int)(((size_t)max_lds - 3 * sheet * sizeof(float)) / walk_wave)}));
        g->walk_waves = W;
        std::vector<std::vector<int>> lists(W);
        std::vector<int> cap(W), rest;
        for (int w = 0; w < W; ++w) cap[w] = ns / W + (w < ns % W ? 1 : 0);
        for (int i = 0, w = 0; i < ns; ++i) {
            const TofUnit &u = hunits[i];
            if (!(W > 1 && i + 1 < ns && u.k > 0.f && u.n1 == u.np && hunits[i + 1].n1 == hunits[i + 1].np && hunits[i + 1].k == u.k)) {
                rest.push_back(i);
                continue;
            }
            hunits[i + 1].dz2 = u.dz2;
            int tries = 0;
            while (tries < W && (int)lists[w].size() + 2 > cap[w]) {
                w = (w + 1) % W;
                ++tries;
            }
            std::vector<int> &to = tries < W ? lists[w] : rest;
            to.push_back(i);
            to.push_back(i + 1);
            if (tries < W) w = (w + 1) % W;
            ++i;
        }
        hwalk.resize(ns);
        for (int r = 0, next = 0; r <= ns / W; ++r)  // (the rest fills the free places in order)
            for (int w = 0; w < W; ++w)
                if (r < cap[w]) hwalk[r * W + w] = r < (int)lists[w].size() ? lists[w][r] : rest[next++];
        g->bins_blk = d.n_tof <= 16 ? d.n_tof : (d.n_tof + 1) / 2;
        g->unit_floats = (max_np + 15) / 16 * 16 * d.n_tof;
        // E(x) = erf(x) on [-c, c], c the kernel's truncation (erf is constant in
        // 32 bits past 4.2): cubics between nodes at most 1/32 apart, from the
        // values and slopes there (error at most h^4 / 384 times the fourth
        // derivative, below 1e-8)
        const double c = std::min(d.tof_nsigma / std::sqrt(2.0), 4.2);
        const int N = 32 * (int)std::ceil(2.0 * c);
        g->n_etab = N;
        g->e_scale = N / (2.0 * c) / (std::sqrt(2.0) * d.tof_sigma_mm);
        const double h = 2.0 * c / N;
        for (int k = 0; k <= N; ++k) {
            const double x0 = -c + k * h, x1 = x0 + h;
            const double e0 = 0.5 * std::erf(x0), e1 = 0.5 * std::erf(x1);
            const double s0 = h * std::exp(-x0 * x0) / std::sqrt(M_PI), s1 = h * std::exp(-x1 * x1) / std::sqrt(M_PI);
            if (k == N)
                hetab.push_back(make_float4((float)e0, 0.f, 0.f, 0.f));
            else
                hetab.push_back(make_float4((float)e0, (float)s0, (float)(3.0 * (e1 - e0) - 2.0 * s0 - s1),
                                            (float)(s0 + s1 - 2.0 * (e1 - e0))));
        }
        // (the filled rows where they take at most half of the LDS)
        g->x_stride = tof_x_stride(rz);
        if (sizeof(float) * (size_t)tof_x_floats(rows_max, g->x_stride) > (size_t)max_lds / 2) g->x_stride = rz;
        // Units whose factors are in LDS together: as many as let two workgroups
        // share a CU if that is four or more, else as many as fit (with room for
        // a batch's sixteen waves); then evenly over the rounds.  (One workgroup
        // per CU with all units at once: 1276 us against 863 for a subset gradient
        // of 128 x 128 x 71 voxels and 13 bins, 915 against 601 with 161 x 161 x 33
        // and 25: its waves wait for each other at the ends of the phases.)
        const size_t unit = sizeof(float) * (size_t)g->unit_floats, stage = sizeof(float) * TOF_STAGE_FLOATS;
        // A backprojection has no image sheet and takes more units at once: 558 -> 540
        // us with 13 bins, 390 -> 366 with 25.
        auto units_for = [&](bool x) {
            const size_t fixed = (x ? sizeof(float) * (size_t)tof_x_floats(rows_max, g->x_stride) : 0) +
                                 sizeof(float4) * (size_t)(N + 1 + 2 * g->n_units);
            auto fit = [&](size_t lds, size_t waves) {
                const size_t used = fixed + waves * stage + 512;
                return lds > used ? (int)((lds - used) / unit) : 0;
            };
            const int most = fit((size_t)max_lds, MAX_WAVES);
            int q = fit(CU_LDS_BYTES / 2, TOF_BLOCK / 64);
            if (q < std::min(4, g->n_units)) q = most;
            q = std::max(1, std::min({q, most, g->n_units}));
            const int rounds = (g->n_units + q - 1) / q;
            return (g->n_units + rounds - 1) / rounds;
        };
        g->q_units = units_for(true);
        g->q_units_back = units_for(false);
    }

    // device allocations
    auto alloc = [&](void **p, size_t bytes) { return hipMalloc(p, bytes == 0 ? 16 : bytes) == hipSuccess; };
    g->t0_elems = (size_t)d.nx * (d.ny + 2 * PADA) * rz;
    g->t1_elems = (size_t)d.ny * (d.nx + 2 * PADA) * rz;
    if (std::max(g->t0_elems, g->t1_elems) >= (size_t)INT32_MAX) {
        delete g;
        return fail(PET_E_ARG, "pet_geom_create: image too large for the 32-bit offsets of the line kernels");
    }
    // line-kernel partials (2 per line) or two per image block (BB dots)
    g->n_partial = std::max<size_t>(2 * (size_t)nl, 2 * (size_t)((g->n_vox + IMG_BLOCK - 1) / IMG_BLOCK)) + 64;
    bool ok = alloc((void **)&g->lines, sizeof(LineP) * nl) && alloc((void **)&g->planes, sizeof(PlaneP) * planes.size()) &&
              alloc((void **)&g->units, sizeof(TofUnit) * hunits.size()) &&
              alloc((void **)&g->etab, sizeof(float4) * hetab.size()) &&
              alloc((void **)&g->walk_order, sizeof(int) * hwalk.size()) &&
              alloc((void **)&g->gsegs, sizeof(SegP) * gsegs.size()) &&
              alloc((void **)&g->gather, sizeof(GatherSeg) * hgather.size()) &&
              alloc((void **)&g->gchunk, sizeof(GatherChunk) * hchunks.size()) &&
              alloc((void **)&g->rho, sizeof(float) * hrho.size()) &&
              alloc((void **)&g->views_dev, sizeof(int) * hviews.size()) &&
              alloc((void **)&g->line_order, sizeof(int) * horder.size()) &&
              alloc((void **)&g->T0, sizeof(float) * g->t0_elems) && alloc((void **)&g->T1, sizeof(float) * g->t1_elems) &&
              alloc((void **)&g->G0, sizeof(float) * g->t0_elems) && alloc((void **)&g->G1, sizeof(float) * g->t1_elems) &&
              alloc((void **)&g->g, sizeof(float) * g->n_vox) && alloc((void **)&g->xtmp, sizeof(float) * g->n_vox) &&
              alloc((void **)&g->grad, sizeof(float) * g->n_vox) && alloc((void **)&g->hess, sizeof(float) * g->n_vox) &&
              alloc((void **)&g->num, sizeof(float) * g->n_vox) && alloc((void **)&g->sensi, sizeof(float) * g->n_vox) &&
              alloc((void **)&g->partial, sizeof(double) * g->n_partial) && alloc((void **)&g->dscratch, sizeof(double) * 16) &&
              alloc((void **)&g->check_counts, sizeof(unsigned) * CHECK_SLOTS) &&
              alloc((void **)&g->fscratch, sizeof(float) * 16);
    if (ok && g->psf_passes)
        ok = alloc((void **)&g->psf_a, sizeof(float) * g->n_vox) && alloc((void **)&g->psf_b, sizeof(float) * g->n_vox);
    if (!ok) {
        pet_geom_destroy(g);
        return fail(PET_E_OOM, "pet_geom_create: device allocation failed");
    }
    hipError_t e = hipMemcpy(g->lines, hlines.data(), sizeof(LineP) * nl, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(g->planes, hplanes.data(), sizeof(PlaneP) * planes.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess && !hunits.empty())
        e = hipMemcpy(g->units, hunits.data(), sizeof(TofUnit) * hunits.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess && !hwalk.empty())
        e = hipMemcpy(g->walk_order, hwalk.data(), sizeof(int) * hwalk.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess && !hetab.empty())
        e = hipMemcpy(g->etab, hetab.data(), sizeof(float4) * hetab.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(g->gsegs, gsegs.data(), sizeof(SegP) * gsegs.size(), hipMemcpyHostToDevice);
    g->n_gseg = (int)gsegs.size();
    if (e == hipSuccess) e = hipMemcpy(g->gather, hgather.data(), sizeof(GatherSeg) * hgather.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(g->rho, hrho.data(), sizeof(float) * hrho.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(g->gchunk, hchunks.data(), sizeof(GatherChunk) * hchunks.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(g->views_dev, hviews.data(), sizeof(int) * hviews.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(g->line_order, horder.data(), sizeof(int) * horder.size(), hipMemcpyHostToDevice);
    // TOF weight table (FP64 nodes): W at NW_TAB + 1 nodes over |d| <= D = bin/2 + nsig sigma
    if (e == hipSuccess && d.n_tof > 1) {
        const double h = 0.5 * d.tof_bin_mm, sig = d.tof_sigma_mm, cl = d.tof_nsigma / std::sqrt(2.0);
        const double D = h + d.tof_nsigma * sig;
        g->wD = (float)D;
        auto E = [&](double u) { return std::erf(std::min(std::max(u / (std::sqrt(2.0) * sig), -cl), cl)); };
        std::vector<double> W(NW_TAB + 1);
        for (int k = 0; k <= NW_TAB; ++k) {
            const double dd = -D + 2.0 * D * k / NW_TAB;
            W[k] = k == 0 || k == NW_TAB ? 0.0 : 0.5 * (E(h - dd) - E(-h - dd));
        }
        std::vector<float2> tab(NW_TAB);
        for (int k = 0; k < NW_TAB; ++k) tab[k] = make_float2((float)W[k], (float)(W[k + 1] - W[k]));
        e = hipMalloc(&g->wtab, sizeof(float2) * NW_TAB);
        if (e == hipSuccess) e = hipMemcpy(g->wtab, tab.data(), sizeof(float2) * NW_TAB, hipMemcpyHostToDevice);
        // W on [0, D] as a line per interval, moved so that its largest errors above
        // and below are equal (half those of the chord), but nowhere below zero: the
        // kernels add its products to sheets that hold nonnegative numbers
        std::vector<float2> ctab(CNT_TAB);
        auto w_at = [&](double dd) { return dd >= D ? 0.0 : 0.5 * (E(h - dd) - E(-h - dd)); };
        for (int k = 0; k < CNT_TAB; ++k) {
            const double w0 = w_at(D * k / CNT_TAB), w1 = w_at(D * (k + 1) / CNT_TAB);
            double lo = 0.0, hi = 0.0;
            for (int i = 1; i < 16; ++i) {
                const double off = w_at(D * (k + i / 16.0) / CNT_TAB) - (w0 + (w1 - w0) * i / 16.0);
                lo = std::min(lo, off);
                hi = std::max(hi, off);
            }
            const double move = std::max(0.5 * (lo + hi), -std::min(w0, w1));
            ctab[k] = make_float2((float)(w0 + move), (float)(w1 - w0));
        }
        if (e == hipSuccess) e = hipMalloc(&g->ctab, sizeof(float2) * CNT_TAB);
        if (e == hipSuccess) e = hipMemcpy(g->ctab, ctab.data(), sizeof(float2) * CNT_TAB, hipMemcpyHostToDevice);
    }
    // padded sheet borders must be zero once; interiors are rewritten per use
    if (e == hipSuccess) e = hipMemset(g->T0, 0, sizeof(float) * g->t0_elems);
    if (e == hipSuccess) e = hipMemset(g->T1, 0, sizeof(float) * g->t1_elems);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        pet_geom_destroy(g);
        return hip_check(e, "pet_geom_create");
    }
    // set-up of the allocation-free entry point on this device (its scratch
    // array's address; a failure is reported by that entry point itself)
    void *scratch_addr = nullptr;
    (void)noalloc_scratch(g->device, &scratch_addr);
    *out = g;
    return PET_OK;
}

extern "C" pet_status pet_geom_destroy(pet_geom g) {
    if (!g) return PET_OK;
    (void)hipDeviceSynchronize();  // best effort: destruction goes on whatever it returns
    for (auto &v : g->prof_events)
        for (auto &e : v) g->prof_pool.push_back(e);
    for (auto &e : g->prof_pool) {
        (void)hipEventDestroy(e.first);
        (void)hipEventDestroy(e.second);
    }
    void *ptrs[] = {g->lines, g->planes, g->units, g->etab, g->walk_order, g->views_dev, g->line_order, g->T0, g->T1, g->G0, g->G1, g->g, g->xtmp,
                    g->grad, g->hess, g->num, g->sensi, g->partial, g->dscratch, g->fscratch, g->psf_a, g->psf_b,
                    g->check_counts, g->wtab, g->ctab, g->gsegs, g->gather, g->gchunk, g->rho};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    delete g;
    return PET_OK;
}

extern "C" pet_status pet_geom_info(pet_geom g, int subset, int64_t *n_bins, int64_t *n_lors, int64_t *n_vox) {
    if (!g) return fail(PET_E_ARG, "pet_geom_info: null handle");
    if (subset < -1 || subset >= g->d.n_subsets) return fail(PET_E_ARG, "pet_geom_info: subset out of range");
    int64_t nv = subset < 0 ? g->d.n_views : (int64_t)g->subset_views[subset].size();
    int64_t lors = nv * g->d.n_rad * g->n_planes;
    if (n_lors) *n_lors = lors;
    if (n_bins) *n_bins = lors * g->d.n_tof;
    if (n_vox) *n_vox = g->n_vox;
    return PET_OK;
}
