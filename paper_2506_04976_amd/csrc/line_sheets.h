// Device helpers shared by the line kernels (proj.hip, counts.hip): the
// z range of a LOR's samples, the per-line LDS sheets (transaxial
// interpolation of the image in, gradient sheet out) and block sums.
#pragma once

#include "pet_internal.h"

namespace pet {

// A table entry that no kernel writes, by scalar loads (its address is uniform).
template <typename T>
__device__ __forceinline__ const T &scalar_ref(const T &t) {
    return *(const T *)(const T __attribute__((address_space(4))) *)(uintptr_t)&t;
}

namespace {

// Sample range [is, ie] of a LOR restricted to samples whose z coordinate can
// touch the grid (xi_z in [-1.5, nz + 0.5]).
template <bool FAST = false>
__device__ __forceinline__ void z_clip(const LineP &L, const PlaneP &P, int nz, int &is, int &ie) {
    is = L.i_lo;
    ie = L.i_hi;
    if (P.zs != 0.f) {
        // FAST: reciprocals instead of divisions, for callers that clamp the
        // axial position themselves (the range is then only a work bound)
        const float rzs = FAST ? __builtin_amdgcn_rcpf(P.zs) : 0.f, rdl = FAST ? __builtin_amdgcn_rcpf(L.dlam) : 0.f;
        float la = FAST ? (-1.5f - P.zb) * rzs : (-1.5f - P.zb) / P.zs;
        float lb = FAST ? ((float)nz + 0.5f - P.zb) * rzs : ((float)nz + 0.5f - P.zb) / P.zs;
        float ia = FAST ? (fminf(la, lb) - L.lam0) * rdl : (fminf(la, lb) - L.lam0) / L.dlam;
        float ib = FAST ? (fmaxf(la, lb) - L.lam0) * rdl : (fmaxf(la, lb) - L.lam0) / L.dlam;
        float lo = ceilf(fminf(ia, ib)), hi = floorf(fmaxf(ia, ib));
        if (lo > (float)is) is = lo > (float)ie ? ie + 1 : (int)lo;
        if (hi < (float)ie) ie = hi < (float)is ? is - 1 : (int)hi;
    } else if (P.zb < -1.5f || P.zb > (float)nz + 0.5f) {
        ie = is - 1;
    }
}

__device__ __forceinline__ float load_y(const void *y, int dt, int64_t idx) {
    if (dt == PET_Y_U8) return (float)((const uint8_t *)y)[idx];
    if (dt == PET_Y_U16) return (float)((const uint16_t *)y)[idx];
    return ((const float *)y)[idx];
}

// Poisson deviance term d(ybar, y) of the KL data fidelity, FP64.
__device__ __forceinline__ double kl_term(float ybar, float yv) {
    double s = ybar, t = yv;
    if (t > 0.0) return s - t + t * log(t / s);
    return s;
}

// Number of samples of [is, ie] (in increasing-t order) with t < e.
__device__ __forceinline__ int cut_count(float e, float len, float lam0, float dlam, int is, int ie) {
    float lam_e = e / len + 0.5f;
    float r = (lam_e - lam0) / dlam;
    int nq = ie - is + 1;
    int c;
    if (dlam > 0.f) {
        float cr = ceilf(r);
        c = cr < (float)is ? 0 : (cr > (float)(ie + 1) ? nq : (int)cr - is);
    } else {
        float fr = floorf(r);
        c = fr >= (float)ie ? 0 : (fr < (float)(is - 1) ? nq : ie - (int)fr);
    }
    return c;
}

// Sheet cells (row r, padded axial position zp) are dealt to the threads of
// a workgroup by column: thread t keeps zp = t mod rz and takes rows
// t / rz, t / rz + R, ... with R = blockDim / rz (the threads past R rz idle).
// No division per cell; needs rz <= blockDim (else one cell per thread and
// pass, with a division each).
struct SheetWalk {
    int r0, zp, R;
    bool on;
};

__device__ __forceinline__ SheetWalk sheet_walk(int rz, int tid) {
    SheetWalk w;
    w.R = (int)blockDim.x / rz;
    w.r0 = tid / rz;
    w.zp = tid - w.r0 * rz;
    w.on = w.r0 < w.R;
    return w;
}

// Row i of a line: the transposed image row it interpolates, at the
// transaxial position xa = i dxa + xa0 (cell jf, fraction f).  Offsets are
// 32-bit: a transposed image holds fewer than 2^31 floats (pet_geom_create).
struct SheetRow {
    int base;  // offset of (i, jf + PADA, 0) in the transposed image
    float f;
};

__device__ __forceinline__ SheetRow sheet_row(const LineP &L, int i, int other_stride, int rz) {
    SheetRow s;
    const float xa = fmaf((float)i, L.dxa, L.xa0);
    const float jf = floorf(xa);
    s.f = xa - jf;
    s.base = i * other_stride + ((int)jf + PADA) * rz;
    return s;
}

// Image sheet X of a line (transaxial interpolation of the transposed image),
// xs floats between its rows, by the whole workgroup (thread tid).
// The loads of SHEET_UNROLL rows per thread are issued before any of them is
// used, so that a workgroup waits for memory a few times per line rather than
// once per element it builds.
constexpr int SHEET_UNROLL = 8;

__device__ __forceinline__ void build_sheet(const ProjArgs &a, const LineP &L, int nrow, float *X, int xs, int tid) {
    const int rz = a.rz;
    const float *T = L.axis ? a.T1 : a.T0;
    const int other_stride = ((L.axis ? a.nx : a.ny) + 2 * PADA) * rz;
    if (rz > (int)blockDim.x) {
        for (int e = tid; e < nrow * rz; e += blockDim.x) {
            const int r = e / rz;
            const int zp = e - r * rz;
            const SheetRow sr = sheet_row(L, L.i_lo + r, other_stride, rz);
            const float *src = T + sr.base + zp;
            X[r * xs + zp] = fmaf(sr.f, src[rz] - src[0], src[0]);
        }
        return;
    }
    const SheetWalk w = sheet_walk(rz, tid);
    if (!w.on) return;
    for (int rb = w.r0; rb < nrow; rb += SHEET_UNROLL * w.R) {
        float t0[SHEET_UNROLL], t1[SHEET_UNROLL], f[SHEET_UNROLL];
#pragma unroll
        for (int u = 0; u < SHEET_UNROLL; ++u) {
            const int r = rb + u * w.R;
            t0[u] = t1[u] = f[u] = 0.f;
            if (r < nrow) {
                const SheetRow sr = sheet_row(L, L.i_lo + r, other_stride, rz);
                f[u] = sr.f;
                const float *src = T + sr.base + w.zp;
                t0[u] = src[0];
                t1[u] = src[rz];
            }
        }
#pragma unroll
        for (int u = 0; u < SHEET_UNROLL; ++u) {
            const int r = rb + u * w.R;
            if (r < nrow) X[r * xs + w.zp] = fmaf(f[u], t1[u] - t0[u], t0[u]);
        }
    }
}

// One sheet cell's value spread over the two transaxial neighbours.
__device__ __forceinline__ void spread_cell(float *Gout, const SheetRow &sr, int zp, int rz, float val) {
    const float a1 = val * sr.f;
    atomicAdd(&Gout[sr.base + zp], val - a1);
    atomicAdd(&Gout[sr.base + zp + rz], a1);
}

// Uniform loads of the gather's segment list through the scalar cache (a
// pointer to constant memory: the kernels that read the list never write it).
typedef const GatherSeg __attribute__((address_space(4))) *GatherSegList;

// Shares of the planes around one voxel's shifted position t in a segment whose
// factors lie at Qs + G.qb (see GatherSeg; whole segments only, lo = 0).  Two
// planes at most while the rings are no closer than the voxels (kappa >= 1):
// their weights need no comparison, a plane that is too far gets the clamped
// weight 0.
__device__ __forceinline__ float gather_two(const float *Qs, const GatherSeg &G, float t, float kappa) {
    const float tc = __builtin_amdgcn_fmed3f(t, 0.f, G.hi);
    const float f = __builtin_amdgcn_fractf(tc);
    const float *q = Qs + G.qb + (int)tc;
    const float w0 = __builtin_amdgcn_fmed3f(fmaf(-kappa, f, 1.f), 0.f, 1.f);
    const float w1 = __builtin_amdgcn_fmed3f(fmaf(kappa, f, 1.f - kappa), 0.f, 1.f);
    return fmaf(w1, q[1], w0 * q[0]);
}

// Three planes, the nearest and its neighbours, while a share reaches no further
// than 3/2 rings (2/3 <= kappa; the nearest plane's weight is positive up to
// kappa = 2).  t is shifted by GATHER_THREE more than in the other forms, so that
// its truncation is the nearest plane.
__device__ __forceinline__ float gather_three(const float *Qs, const GatherSeg &G, float t, float kappa) {
    const float tc = __builtin_amdgcn_fmed3f(t, 0.5f, G.hi + 2.5f);
    const float f = __builtin_amdgcn_fractf(tc);
    const float *q = Qs + (G.qb - 2) + (int)tc;
    const float w0 = __builtin_amdgcn_fmed3f(fmaf(-kappa, f, fmaf(-0.5f, kappa, 1.f)), 0.f, 1.f);
    const float w1 = fmaf(-kappa, fabsf(f - 0.5f), 1.f);
    const float w2 = __builtin_amdgcn_fmed3f(fmaf(kappa, f, fmaf(-1.5f, kappa, 1.f)), 0.f, 1.f);
    return fmaf(w2, q[2], fmaf(w1, q[1], w0 * q[0]));
}

// Any kappa: a window of as many planes as a share can reach (the whole segment if
// that is shorter), weights clamped at 0.  The window has the same length in every
// lane, so that the loop does not diverge and its LDS reads are in flight together;
// four planes' shares are added in 32 bits, the sums in 64.
__device__ __forceinline__ double gather_some(const float *Qs, const GatherSeg &G, float t, float kappa) {
    const float h = 1.f / kappa, n = fminf(ceilf(2.f * h), G.hi - G.lo - 1.f);
    const float first = __builtin_amdgcn_fmed3f(ceilf(t - h), G.lo + 1.f, G.hi - n);
    const float *q = Qs + G.qb + (int)first;
    auto share = [&](float d, float v, float s) {
        return fmaf(__builtin_amdgcn_fmed3f(fmaf(-kappa, fabsf(d), 1.f), 0.f, 1.f), v, s);
    };
    float d = t - first;
    double s = 0.0;
    int k = (int)n;
    for (; k >= 4; k -= 4, d -= 4.f, q += 4) {
        const float q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
        s += (double)share(d - 3.f, q3, share(d - 2.f, q2, share(d - 1.f, q1, share(d, q0, 0.f))));
    }
    for (; k > 0; --k, d -= 1.f, ++q) s += (double)share(d, *q, 0.f);
    return s;
}

// Factors that are not finite: planes of weight 0 are left out.
__device__ __forceinline__ double gather_many(const float *Qs, const GatherSeg &G, float t, float kappa) {
    const float h = 1.f / kappa;
    // (clamped to the planes before the conversion; the margin covers the rounding of
    // t, a whole plane on both sides would double the planes of kappa just below 1)
    const float lo = fminf(fmaxf(ceilf(t - h - 1e-3f), G.lo + 1.f), G.hi);
    const float hi = fmaxf(fminf(floorf(t + h + 1e-3f), G.hi - 1.f), G.lo);
    double s = 0.0;
    for (int p = (int)lo; p <= (int)hi; ++p) {
        const float w = fmaf(-kappa, fabsf(t - (float)p), 1.f);
        if (w > 0.f) s += (double)(w * Qs[G.qb + p]);
    }
    return s;
}

// PLANES: 2, 3, GATHER_SOME or GATHER_MANY (the forms above in their order).
template <int PLANES>
__device__ __forceinline__ auto gather_planes(const float *Qs, const GatherSeg &G, float t, float kappa) {
    if constexpr (PLANES == 2)
        return gather_two(Qs, G, t, kappa);
    else if constexpr (PLANES == 3)
        return gather_three(Qs, G, t, kappa);
    else if constexpr (PLANES == GATHER_SOME)
        return gather_some(Qs, G, t, kappa);
    else
        return gather_many(Qs, G, t, kappa);
}

// Shifted position of voxel z before the segment's part, in the form's shift.
template <int PLANES>
__device__ __forceinline__ float gather_rho(const ProjArgs &a, int z) {
    return a.rho[min(z, a.nz - 1)] + (PLANES == 3 ? GATHER_THREE : 0.f);
}

// Backprojection of one chunk of planes of a non-TOF line from their factors
// (mult y / ybar ell and the like) in LDS: each thread owns cells (row i, voxel
// z) of the line's sheet, sums the shares that land on them over the segments in
// FP64 and spreads the sum over the two transaxial neighbours.  No sheet, no LDS
// atomics.
//
// Bound by VALU issue: 13 instructions per cell and segment (position, clamp,
// fraction and cell, two weights, two products, FP64 conversion and add) against one
// two-word LDS read; 17 with three planes.  A scatter instead adds two shares per
// sample with FP64 LDS atomics into a sheet of doubles, which took 77 KB and left
// one workgroup per CU: backprojection of a 10-view subset of the 128x128x71,
// 2204-plane geometry 397 us (now 142), its fused gradient 603 (299), the TOF
// sensitivity over all 252 views 7.6 ms (3.2).  The forms' lines: with kappa just
// below 1, the loop of gather_many takes 65.7 us for a gradient of 96 x 96 x 32
// voxels at kappa 0.9, three fixed planes 51.6, the scatter 76; at kappa 0.6 and 0.2
// the loop takes 71 and 121, the scatter 87 and 191.
//
// fold (a TOF geometry's mult alone): every sample carries the sum of its TOF
// bins' weights, a function of the row and the ring difference.  Where every
// row of a wave lies far enough inside the bins for all segments, that sum is
// one constant; elsewhere it comes from the rows' table in LDS (line_nt_body).
//
// Cells whose sum is no larger than `least` stay zero.  In a sensitivity that is the
// rounding of one share of the line's largest factor, which a cell may get that its
// planes miss by nothing (a voxel exactly one voxel away from them): its zeros are then
// exact, as an OSEM step takes them to be.  (With rings three voxels apart
// the slices between them got a sensitivity of 1e-7, and the image was off by its own
// size.)
//
// Rows [r0, r1) of the line.
template <int PLANES, bool FOLD, typename Fold>
__device__ __forceinline__ void gather_cells(const ProjArgs &a, const LineP &L, int r0, int r1, const float *Qs,
                                             const GatherChunk &ch, int64_t g_off, const Fold &fold, float least, int tid) {
    const int nz = a.nz, rz = a.rz;
    float *Gout = (L.axis ? a.G1 : a.G0) + g_off;
    const int other_stride = ((L.axis ? a.nx : a.ny) + 2 * PADA) * rz;
    const GatherSegList segs = (GatherSegList)(uintptr_t)a.gather;
    const float kappa = a.kappa;
    const int dr = (int)blockDim.x / nz, dz = (int)blockDim.x - dr * nz;
    int r = tid / nz, z = tid - r * nz;
    r += r0;
    while (r < r1) {
        const float lam = fmaf((float)(L.i_lo + r), L.dlam, L.lam0);
        const float rho = gather_rho<PLANES>(a, z);
        double acc = 0.0;
        auto run = [&](int s0, int s1, float slope, auto each) {
            constexpr int UNROLL = PLANES == 2 || PLANES == 3 ? 4 : 1;
#pragma unroll UNROLL
            for (int s = s0; s < s1; ++s) {
                const GatherSeg G = {segs[s].k, segs[s].lo, segs[s].hi, segs[s].qb};
                const float t = fmaf(-slope, G.k, rho);
                acc += (double)each(gather_planes<PLANES>(Qs, G, t, kappa), G.k);
            }
        };
        auto both = [&](auto each) {
            run(ch.s0, ch.s_neg, lam, each);
            run(ch.s_neg, ch.s1, 1.f - lam, each);
        };
        float drop = least;
        if (FOLD && !__all(fold.constant(lam))) {
            const float *w = fold.table + (r - r0) * fold.n_k;
            both([&](auto v, float k) { return v * w[(int)k]; });
            drop *= w[0];  // (the largest)
        } else {
            both([](auto v, float) { return v; });
            if (FOLD) acc *= (double)fold.inside();
        }
        const float val = (float)acc;
        if (!(fabsf(val) <= drop)) spread_cell(Gout, sheet_row(L, L.i_lo + r, other_stride, rz), z + PADZ, rz, val);
        r += dr;
        z += dz;
        if (z >= nz) {
            z -= nz;
            ++r;
        }
    }
}

// Block sums of two doubles into partial[blockIdx.x] (and, for the work counts,
// partial[gridDim.x + blockIdx.x]).
__device__ __forceinline__ void block_sums(double v0, double v1, double *partial, bool two,
                                           int tid = threadIdx.x) {
    __shared__ double red[2][MAX_WAVES];
    for (int off = 32; off > 0; off >>= 1) {
        v0 += __shfl_down(v0, off, 64);
        v1 += __shfl_down(v1, off, 64);
    }
    const int nw = blockDim.x >> 6;
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = v0;
        red[1][tid >> 6] = v1;
    }
    __syncthreads();
    if (tid == 0) {
        double s0 = 0.0, s1 = 0.0;
        for (int w = 0; w < nw; ++w) {
            s0 += red[0][w];
            s1 += red[1][w];
        }
        partial[blockIdx.x] = s0;
        if (two) partial[gridDim.x + blockIdx.x] = s1;
    }
}

}  // namespace
}  // namespace pet
