// Joseph projector kernels for gfx950 (forward, adjoint, fused subset gradient,
// EM ratio, non-TOF likelihood, work counts), line-driven with LDS sheets.
//
// Separability used here: every LOR of a transaxial line (view, radial) has the
// same principal axis m, the same sample positions lambda(i) along m and the
// same transaxial interpolation coordinate; only z (and the step length via
// |u|) depends on the ring pair.  A workgroup therefore owns one line:
//   1. it interpolates the image once along the transaxial axis into an LDS
//      "sheet" X[i][z] (rows i along m, z padded), reading a z-contiguous
//      transposed copy of the image so the loads are coalesced;
//   2. threads take the planes (ring pairs) of the line and walk the samples
//      with one linear interpolation in z from LDS per sample;
//   3. the adjoint gathers the cells of the sheet from the planes and spreads
//      them over the two transaxial neighbours with global atomics into a
//      z-contiguous transposed gradient image.
// TOF: all planes of one ring-difference segment share |u|, hence the signed
// distance t(i) of every sample and its TOF weights, so that the sums over rows
// and over bins are small matrix products (see line_tof_body).
// The arithmetic is Joseph's: sample value = bilinear interpolation of the
// image in the two non-principal axes, line integral = step length * sum.
#include "line_sheets.h"

#include <algorithm>
#include <climits>

namespace pet {
namespace {

template <int V>
struct Int {
    static constexpr int value = V;
};

// The lane index, opaque: what follows from it is formed where it is used and not
// kept in registers across the other phases (which need all 128 of them).
__device__ __forceinline__ int lane_here() {
    int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane));
    return lane;
}

// ---------------------------------------------------------------------------
// Non-TOF: threads over planes (dense), one line per workgroup.
// Sum over all TOF bins of the weights of a sample at signed distance t from
// the LOR centre.  The bins [t_b - w/2, t_b + w/2] tile [lo, hi] = [t_first -
// w/2, t_last + w/2] without gaps, so the sum of 1/2 [E(t_b + w/2 - t) -
// E(t_b - w/2 - t)] telescopes to 1/2 [E(hi - t) - E(lo - t)]; where both
// ends are clamped (t at least nsig sigma inside [lo, hi]) it is erf(c).
struct LineFold {
    float lo, hi, inv_s, c, full;
    float lt2, pitch2, t_in, len_max;
    const float *table = nullptr;  // weights of the rows of a block, n_k each
    int n_k;

    __device__ __forceinline__ LineFold(const ProjArgs &a, const LineP &L) {
        const TofTable &T = a.tof;
        lo = T.tb[0] - T.half_bin;
        hi = T.tb[T.n_tof - 1] + T.half_bin;
        inv_s = T.inv_sqrt2_sigma;
        c = T.erf_clamp;
        full = a.fold_full;
        lt2 = L.lt2;
        pitch2 = a.pitch2;
        // (|t| up to which both ends are clamped, and the longest |u| of the line)
        t_in = a.fold_in;
        len_max = sqrtf(fmaf(a.k_max * a.k_max, pitch2, lt2)) * (1.f + 1e-5f);
        n_k = (int)a.k_max + 1;
    }
    // the samples of the row lie where the sum is `inside` in every segment
    __device__ __forceinline__ bool constant(float lam) const { return fabsf(lam - 0.5f) * len_max <= t_in; }
    __device__ __forceinline__ float inside() const { return full; }
    __device__ __forceinline__ float weight(float lam, float k) const {
        const float t = (lam - 0.5f) * __builtin_amdgcn_sqrtf(fmaf(k * k, pitch2, lt2));
        const float e1 = (hi - t) * inv_s, e0 = (lo - t) * inv_s;
        if (e1 >= c && e0 <= -c) return full;
        return 0.5f * (erff(fminf(fmaxf(e1, -c), c)) - erff(fminf(fmaxf(e0, -c), c)));
    }
};

// One transaxial line of a non-TOF geometry, by the whole workgroup; returns
// this thread's FP64 partial (KL or sample count).
//
// Forward: one thread per plane walks the samples of its LOR through the image
// sheet X.  Adjoint: the planes' factors go to LDS (9 KB for 2204 planes) and
// the cells of the sheet gather them (gather_cells).
template <int MODE>
__device__ __forceinline__ double line_nt_body(const ProjArgs &a, int line, float *smem, int tid, int64_t g_off = 0) {
    constexpr bool NEED_X = MODE != M_BACK && MODE != M_COUNT;
    constexpr bool NEED_Z = MODE == M_BACK || MODE == M_GRAD || MODE == M_EM || MODE == M_HVP;
    __shared__ int s_special;      // some factor is not finite
    __shared__ unsigned s_most;    // the largest finite one (a sensitivity's)
    const LineP L = scalar_ref(a.lines[line]);
    const int nrow = L.i_hi - L.i_lo + 1;
    const int rz = a.rz;
    const int sheet = (a.rows_max * rz + 3) & ~3;
    float *X = smem;
    float *Qs = smem + (NEED_X ? sheet : 0);
    // (a line that misses the image has no adjoint; its forward values and
    // likelihood terms stay)
    if (nrow <= 0 && (MODE == M_BACK || MODE == M_HVP || ((MODE == M_GRAD || MODE == M_EM) && !a.partial))) return 0.0;
    if (NEED_X && nrow > 0) build_sheet(a, L, nrow, X, rz, tid);

    double kl = 0.0;
    const int nb = blockDim.x;
    // Folded TOF weights per row and ring difference, in blocks of rows (one block
    // unless the ring differences are many); none where all rows lie inside the bins.
    // Evaluated per share, two error functions each, they cost a sensitivity of 97 x
    // 88 x 27 voxels, 19 bins and 231 planes 33.8 us (scatter, once per sample: 23.8;
    // this table: 19.2).
    LineFold F(a, L);
    float *fold_table = Qs + a.q_floats;
    int fold_rows = INT_MAX;
    auto fill_fold = [&](int r0) {
        if (fold_rows == INT_MAX) return;
        for (int e = tid; e < min(fold_rows, nrow - r0) * F.n_k; e += nb) {
            const int r = e / F.n_k;
            fold_table[e] = F.weight(fmaf((float)(L.i_lo + r0 + r), L.dlam, L.lam0), (float)(e - r * F.n_k));
        }
    };
    if (MODE == M_BACK && a.tof_fold) {
        if (!F.constant(fmaf((float)L.i_lo, L.dlam, L.lam0)) || !F.constant(fmaf((float)L.i_hi, L.dlam, L.lam0)))
            fold_rows = FOLD_FLOATS / F.n_k;  // (uniform)
        fill_fold(0);
    }
    for (int ic = 0; ic < (MODE == M_COUNT ? 1 : a.n_gchunk); ++ic) {
        GatherChunk ch{0, 0, 0, 0, a.n_planes, 0};
        if (MODE != M_COUNT) ch = a.gchunk[ic];
        if (NEED_Z) {
            // (the zeros around the segments; the previous chunk's cells are done)
            if (ic > 0) __syncthreads();
            for (int k = tid; k < ch.n_q; k += nb) Qs[k] = 0.f;
            if (tid == 0) s_special = s_most = 0;
        }
        if (NEED_Z || (NEED_X && ic == 0)) __syncthreads();

        // planes in rounds of blockDim threads; the planes of the line's last,
        // partial round take c threads each (c a power of two: the threads of a
        // plane are lanes of one wave), which split its rows and add their forward
        // sums by shuffles (chunks of planes do not change which planes those are,
        // nor so their sums)
        const int full = NEED_X ? a.n_planes / nb * nb : a.n_planes;
        const int rem = a.n_planes - full;
        int lg_c = 0;
        while (rem > 0 && lg_c < 6 && (rem << (lg_c + 1)) <= nb) ++lg_c;
        float most = 0.f;
        for (int base = ch.p0, end; base < ch.p1; base = end) {
            const int lg = base >= full ? lg_c : 0, cc = 1 << lg;
            end = min(base >= full ? ch.p1 : min(ch.p1, full), base + (nb >> lg));
            const int cs = tid & (cc - 1);
            const bool act = base + (tid >> lg) < end;
            const int p = act ? base + (tid >> lg) : base;
            const PlaneP P = a.planes[p];
            const int64_t lor = (int64_t)line * a.n_planes + p;
            const float len = sqrtf(L.lt2 + P.dz2);
            const float ell = L.vm_um * len;
            int is = 0, ie = -1;
            if ((NEED_X || MODE == M_COUNT) && act && nrow > 0) z_clip(L, P, a.nz, is, ie);
            if constexpr (MODE == M_COUNT) {
                if (cs == 0 && ie >= is) kl += (double)(ie - is + 1);
                continue;
            }
            float s = 0.f;
            if (NEED_X) {
                // padded axial cell of sample i: u = zA i + zB = z + PADZ, clamped
                // to [0, nz + 2] (the clamp only guards the LDS bounds; z-clipped
                // samples lie inside), where truncation is the floor; two samples
                // per iteration, their LDS reads in flight together, added one after
                // the other (the likelihood's FP64 sum shows the order)
                const float zA = P.zs * L.dlam, zB = fmaf(L.lam0, P.zs, P.zb) + (float)PADZ;
                const float umax = (float)(a.nz + PADZ);
                const float fc = (float)cc, fie = (float)ie;
                const int step = cc * rz;
                const float *xr = X + (is + cs - L.i_lo) * rz;
                float fi = (float)(is + cs);
                for (; fi + fc <= fie; fi += 2.f * fc, xr += 2 * step) {
                    const float u0 = __builtin_amdgcn_fmed3f(fmaf(fi, zA, zB), 0.f, umax);
                    const float u1 = __builtin_amdgcn_fmed3f(fmaf(fi + fc, zA, zB), 0.f, umax);
                    const int j0 = (int)u0, j1 = (int)u1;
                    const float a0 = xr[j0], b0 = xr[j0 + 1], a1 = xr[step + j1], b1 = xr[step + j1 + 1];
                    s += fmaf(__builtin_amdgcn_fractf(u0), b0 - a0, a0);
                    s += fmaf(__builtin_amdgcn_fractf(u1), b1 - a1, a1);
                }
                if (fi <= fie) {
                    const float u = __builtin_amdgcn_fmed3f(fmaf(fi, zA, zB), 0.f, umax);
                    const int j = (int)u;
                    const float x0 = xr[j], x1 = xr[j + 1];
                    s += fmaf(__builtin_amdgcn_fractf(u), x1 - x0, x0);
                }
                for (int o = 1; o < cc; o <<= 1) s += __shfl_xor(s, o, 64);
            }
            if (!act || cs != 0) continue;
            const float m = a.mult ? a.mult[lor] : 1.f;
            float Q = 0.f;
            if constexpr (MODE == M_BACK) {
                Q = (a.sino ? a.sino[lor] : 1.f) * m * ell;
            } else if constexpr (MODE == M_HVP) {
                // data-term Hessian: mult^2 y / ybar^2 (P v), then back
                const float yv = load_y(a.y, a.y_dtype, lor);
                const float yb = a.ybar[lor];
                Q = yv != 0.f ? m * m * yv / (yb * yb) * (s * ell) * ell : 0.f;
            } else {
                const float ybar = fmaf(m, s * ell, a.add ? a.add[lor] : 0.f);
                if constexpr (MODE == M_FWD) {
                    a.out[lor] = ybar;
                } else {
                    const float yv = load_y(a.y, a.y_dtype, lor);
                    if (a.partial) kl += kl_term(ybar, yv);
                    // a bin without counts has d(s, 0) = s: derivative 1 and EM ratio 0,
                    // also where ybar = 0 (no 0 * inf)
                    if constexpr (MODE == M_GRAD) Q = m * (yv != 0.f ? 1.f - yv / ybar : 1.f) * ell;
                    if constexpr (MODE == M_EM) Q = yv != 0.f ? m * (yv / ybar) * ell : 0.f;
                }
            }
            if (NEED_Z) {
                Qs[P.q] = Q;
                if (!(fabsf(Q) < INFINITY)) s_special = 1;
                if (MODE == M_BACK) most = fabsf(Q) < INFINITY ? fmaxf(most, fabsf(Q)) : most;
            }
        }
        if (!NEED_Z) continue;
        if (MODE == M_BACK && !a.sino) {
            for (int o = 32; o; o >>= 1) most = fmaxf(most, __shfl_xor(most, o, 64));
            if ((tid & 63) == 0) atomicMax(&s_most, __float_as_uint(most));
        }
        __syncthreads();
        if (nrow <= 0) continue;
        const int form = s_special ? GATHER_MANY : a.gather_planes;  // (uniform)
        const float least = MODE == M_BACK && !a.sino ? a.least_weight * __uint_as_float(s_most) : 0.f;
        auto cells = [&](auto fold, int r0, int r1) {
            constexpr bool FOLD = fold.value != 0;
            if (form == 2)
                gather_cells<2, FOLD>(a, L, r0, r1, Qs, ch, g_off, F, least, tid);
            else if (form == 3)
                gather_cells<3, FOLD>(a, L, r0, r1, Qs, ch, g_off, F, least, tid);
            else if (form == GATHER_SOME)
                gather_cells<GATHER_SOME, FOLD>(a, L, r0, r1, Qs, ch, g_off, F, least, tid);
            else
                gather_cells<GATHER_MANY, FOLD>(a, L, r0, r1, Qs, ch, g_off, F, least, tid);
        };
        if (MODE == M_BACK && a.tof_fold) {
            F.table = fold_table;
            for (int r0 = 0; r0 < nrow; r0 = fold_rows < nrow - r0 ? r0 + fold_rows : nrow) {
                if (r0 > 0 || (ic > 0 && fold_rows < nrow)) {
                    __syncthreads();
                    fill_fold(r0);
                    __syncthreads();
                }
                cells(Int<MODE == M_BACK>(), r0, fold_rows < nrow - r0 ? r0 + fold_rows : nrow);
            }
        } else {
            cells(Int<0>(), 0, nrow);
        }
    }
    return kl;
}

// (Eight waves per SIMD, for the scalar registers: left alone the compiler takes
// 106 of them, which lets seven waves onto a SIMD and so one workgroup of 1024 on
// a CU; with 78 there are two, and one walks while the other waits: a 3D subset
// gradient of 128 x 128 x 71 voxels and 2204 planes 387 -> 304 us, its sensitivity
// over all views 3785 -> 3380 us.)
template <int MODE>
__global__ void __launch_bounds__(NT_BLOCK, 8) k_line_nt(ProjArgs a) {
    extern __shared__ float4 smem4[];
    // one line per workgroup, the launch's lines longest first
    const double kl = line_nt_body<MODE>(a, a.order[blockIdx.x], reinterpret_cast<float *>(smem4), threadIdx.x);
    if (MODE != M_FWD && MODE != M_BACK && a.partial) block_sums(kl, kl, a.partial, MODE == M_COUNT);
}

// ---------------------------------------------------------------------------
// TOF: matrix products over the TOF weights.
//
// All planes of one ring difference share |u|, hence the signed distance t of
// every row and its TOF weights W[row][bin].  So, per unit (a segment, or a pair
// -k, +k of at most 64 planes together),
//     forward   A[bin][plane] = sum_row W[bin][row] V[row][plane],
//     adjoint   Q[row][plane] = sum_bin W[row][bin] F[bin][plane],
// with V the axially interpolated samples and F the factors mult (1 - y / ybar)
// ell (and the like): both run on the f32 matrix instruction 16x16x4.
//
//  * Forward: one wave takes a unit; a step covers 4 rows x 64 planes (four
//    samples per lane) and multiplies them by the weights of the 4 rows x 16
//    bins (one weight per lane) into one 16 x 16 tile per 16 planes.
//  * The factors of q_units units go to LDS, [16-plane tile][bin][plane].
//  * Adjoint: one wave takes 16 rows.  Per unit it forms the 16 rows x 64 planes
//    of Q (only the groups of four bins that reach those rows), passes them
//    through its own LDS rows, four at a time, and its lanes (4 rows x 16
//    voxels) gather the axial shares of their cells (gather_two), in FP64
//    registers over all units.  No LDS atomics, no sheet of doubles.
//
// The weight of bin b at t is 1/2 [E(hi_b - t) - E(lo_b - t)], E the clamped erf,
// from a table of cubics in LDS: off by less than 1e-8 in exact arithmetic (see
// pet_geom_create) and by about 6e-8 a weight in 32 bits, plus the rounding of the
// table position times the slope there.  The forward adds the position up in parts
// (TofPos); the adjoint forms it in one multiply-add.
//
// What bounds it: vector instructions (61% of the cycles of a subset gradient of
// 128 x 128 x 71 voxels, 2204 planes and 13 bins; 12 per gathered cell and unit,
// 6 to 8 per sample), then the matrix cores (18% of its 755 us) and the data's
// loads.  A wave per segment with FP64 LDS adds per sample took 1016 us for it;
// 934 -> 496 us with 161 x 161 x 33 voxels and 25 bins, and a forward projection
// of 96 x 96 x 32 voxels 694 -> 225 us.
//
// Lane layouts of the 16x16x4 instruction: A[m][k] in lane 16 k + m, B[k][n] in
// lane 16 k + n, D[m][n] in register m mod 4 of lane 16 (m / 4) + n.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const TofUnit __attribute__((address_space(4))) *TofUnitList;

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float cubic_at(const float4 &c, float f) {
    return fmaf(fmaf(fmaf(c.w, f, c.z), f, c.y), f, c.x);
}

// 1/2 E at table position pos (clamped to the table: E is constant outside).
__device__ __forceinline__ float half_erf_at(const float4 *tab, float pos, float last) {
    const float p = __builtin_amdgcn_fmed3f(pos, 0.f, last);
    const float f = __builtin_amdgcn_fractf(p);
    return cubic_at(tab[(int)p], f);
}

// Table position of the lower edge of bin b at row j of a line (rows counted
// from i_lo) in a unit: pA j + pB + b dpos; the step length of its samples.
struct TofPos {
    float pA, pB, ell;
    // the same in parts that the forward adds up without loss: pA = a_hi + a_lo,
    // and the table's middle (lower edge of bin 0) lies at row j0 - b0 / pA
    float a_hi, a_lo, b0, j0, pad;
};
static_assert(sizeof(TofPos) == 32, "two 16-byte LDS reads");

// Forward tiles of one unit: NPB tiles of 16 planes, MB blocks of bins.  Lanes
// past the unit's planes have zA = zB = 0 (they read the zero padding); rows
// past the line's are zeros in X.  The next step's weights are looked up while
// this step's samples are under way.
template <int MB, int NPB, int TILES>
__device__ __forceinline__ void tof_fwd_rows(const ProjArgs &a, const float4 *tab, const float *X, int j_lo, int j_hi,
                                             int i_lo, int lane, const TofPos &tp, const float (&zA)[TILES],
                                             const float (&zB)[TILES], f32x4 (&D)[MB][TILES]) {
    const int xs = a.x_stride;
    const float umax = (float)(a.nz + PADZ), last = (float)a.n_etab;
    const int jr = lane >> 4;
    const bool full = a.bins_blk == 16;
    float pos[MB], w[MB];
    // p = pA rel + pos, rel the row counted from one near the bin's lower edge: p is
    // rounded on the scale of the table, not on that of the line
    float rel[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const float b = (float)(mb * a.bins_blk + (lane & 15));
        const float jb = rintf(__builtin_amdgcn_fmed3f(-b * a.dpos * __builtin_amdgcn_rcpf(tp.pA), -4095.f, 4095.f));
        pos[mb] = fmaf(jb, tp.a_hi, b * a.dpos_hi) + fmaf(jb, tp.a_lo, fmaf(b, a.dpos_lo, tp.b0)) + a.e_mid;
        rel[mb] = (float)(j_lo + jr) - tp.j0 - jb;
    }
    auto weights = [&]() {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const float p = fmaf(rel[mb], tp.pA, pos[mb]);
            rel[mb] += 4.f;
            const float lo = half_erf_at(tab, p, last);
            // the upper edge is the next lane's lower one (16 bins: the last
            // lane has no next one)
            float hi = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, lo),
                                                                              0x101 /* row_shl:1 */, 0xf, 0xf, true));
            if (full) hi = half_erf_at(tab, p + a.dpos, last);
            w[mb] = fmaxf(hi - lo, 0.f);  // (the table's rounding: -3e-8 where E is flat)
        }
    };
    const float *xr = X + (j_lo + jr) * xs;
    float fi = (float)(i_lo + j_lo + jr);
    weights();
    for (int j = j_lo; j <= j_hi; j += 4) {
        float x0[NPB], x1[NPB], f[NPB], wj[MB];
#pragma unroll
        for (int pb = 0; pb < NPB; ++pb) {
            const float u = __builtin_amdgcn_fmed3f(fmaf(fi, zA[pb], zB[pb]), 0.f, umax);
            const int c = (int)u;
            f[pb] = __builtin_amdgcn_fractf(u);
            x0[pb] = xr[c];
            x1[pb] = xr[c + 1];
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) wj[mb] = w[mb];
        weights();
#pragma unroll
        for (int pb = 0; pb < NPB; ++pb) {
            const float v = fmaf(f[pb], x1[pb] - x0[pb], x0[pb]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) D[mb][pb] = mfma16(wj[mb], v, D[mb][pb]);
        }
        xr += 4 * xs;
        fi += 4.f;
    }
}

// Weight of bin b at row j.
__device__ __forceinline__ float tof_weight(const ProjArgs &a, const float4 *tab, const TofPos &tp, float fj, int b) {
    const float p = fmaf((float)b, a.dpos, fmaf(fj, tp.pA, tp.pB)), last = (float)a.n_etab;
    return fmaxf(half_erf_at(tab, p + a.dpos, last) - half_erf_at(tab, p, last), 0.f);
}

// The forward sum of one bin of one LOR without the products of zero weights
// (an image that is not finite must not reach the bins beyond it).
__device__ __forceinline__ float tof_fwd_guarded(const ProjArgs &a, const float4 *tab, const float *X, const LineP &L,
                                                 int nrow, const TofPos &tp, const PlaneP &P, int b) {
    const float zA = P.zs * L.dlam, zB = fmaf(L.lam0, P.zs, P.zb) + (float)PADZ;
    const float umax = (float)(a.nz + PADZ);
    float s = 0.f;
#pragma unroll 1
    for (int j = 0; j < nrow; ++j) {
        const float w = tof_weight(a, tab, tp, (float)j, b);
        if (!(w > 0.f)) continue;
        const float u = __builtin_amdgcn_fmed3f(fmaf((float)(L.i_lo + j), zA, zB), 0.f, umax);
        const int c = (int)u;
        const float f = __builtin_amdgcn_fractf(u);
        const float x0 = X[j * a.x_stride + c], x1 = X[j * a.x_stride + c + 1];
        s = fmaf(w, f > 0.f ? fmaf(f, x1 - x0, x0) : x0, s);
    }
    return s;
}

// A factor that is not finite, spread by itself: the matrix products would take
// it to the rows and planes where its weight is 0.
__device__ __forceinline__ void tof_back_special(const ProjArgs &a, const LineP &L, const float4 *tab, int nrow,
                                                 const TofPos &tp, const PlaneP &P, int b, float Q, int64_t g_off) {
    const float zA = P.zs * L.dlam, zB = fmaf(L.lam0, P.zs, P.zb) + (float)PADZ;
    float *Gout = (L.axis ? a.G1 : a.G0) + g_off;
    const int other_stride = ((L.axis ? a.nx : a.ny) + 2 * PADA) * a.rz;
#pragma unroll 1
    for (int j = 0; j < nrow; ++j) {
        const float w = tof_weight(a, tab, tp, (float)j, b);
        const float u = fmaf((float)(L.i_lo + j), zA, zB);
        if (!(w > 0.f) || !(u > (float)PADZ - 1.f && u < (float)(a.nz + PADZ))) continue;
        const int c = (int)u;
        const float f = __builtin_amdgcn_fractf(u);
        const SheetRow sr = sheet_row(L, L.i_lo + j, other_stride, a.rz);
        if (f < 1.f && c >= PADZ) spread_cell(Gout, sr, c, a.rz, Q * (w * (1.f - f)));
        if (f > 0.f && c + 1 < a.nz + PADZ) spread_cell(Gout, sr, c + 1, a.rz, Q * (w * f));
    }
}

// Four consecutive bins of which the first n exist, in one load where all do
// (the arrays need no more than their elements' alignment).
__device__ __forceinline__ void load_bins(const float *p, int n, float (&v)[4]) {
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    if (n >= 4) {
        const f4 q = *reinterpret_cast<const f4 *>(p);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = q[r];
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r) v[r] = r < n ? p[r] : 0.f;
        v[3] = 0.f;
    }
}

__device__ __forceinline__ void store_bins(float *p, int n, const float (&v)[4]) {
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    if (n >= 4) {
        *reinterpret_cast<f4 *>(p) = f4{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
            if (r < n) p[r] = v[r];
    }
}

__device__ __forceinline__ void load_counts(const void *y, int dt, int64_t base, int n, float (&v)[4]) {
    if (dt == PET_Y_U8) {
        typedef uint32_t u4 __attribute__((aligned(1)));
        const uint8_t *p = (const uint8_t *)y + base;
        uint32_t q = 0;
        if (n >= 4) {
            q = *reinterpret_cast<const u4 *>(p);
        } else {
#pragma unroll
            for (int r = 0; r < 3; ++r) q |= r < n ? (uint32_t)p[r] << (8 * r) : 0u;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (float)((q >> (8 * r)) & 0xffu);
    } else if (dt == PET_Y_U16) {
        const uint16_t *p = (const uint16_t *)y + base;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = r < n ? (float)p[r] : 0.f;
    } else {
        load_bins((const float *)y + base, n, v);
    }
}

// LDS of a wave of the adjoint: 4 rows of a unit's planes (at most 64, with the
// zeros around its two segments), 16 banks apart.
constexpr int STAGE_COLS = 80, STAGE_ROWS = 4;
static_assert(64 + 3 * GATHER_ZEROS <= STAGE_COLS, "a unit's planes and the zeros around its segments");
static_assert(TOF_STAGE_FLOATS == STAGE_COLS * STAGE_ROWS, "LDS layout of the TOF line kernels");
// Voxels along z of one pass of the adjoint: at most STAGE_ZB groups of 16.
constexpr int STAGE_ZB = 5;
static_assert(16 * STAGE_ZB <= STAGE_COLS, "the finished cells leave through the staged rows");
constexpr unsigned CUS = 256;
// Lines of a launch up to which a CU has two workgroups at most.
constexpr unsigned FEW_LINES = 2 * CUS;
// Groups of four bins whose weights a wave of the adjoint keeps for a pair of
// segments of the same length.
constexpr int KEEP_KK = 3;

// Order of LDS accesses within a wave: its LDS instructions are carried out in
// order, so only the compiler has to keep them so.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// What the adjoint of one block of 16 rows works on: the units [u0, u1) whose
// factors are in LDS, the wave's staged rows, the tables, the block and the groups
// of four bins [kk0, kk0 + nkk) that reach its rows.
struct TofBack {
    const float *Fs;
    float *stage;
    const TofPos *utab;
    const float4 *tab;
    int u0, u1, rb, kk0, nkk;
};

// Adjoint of one block of 16 rows over units [u0, u1): adds to the lane's cells
// acc[h][zb] (row 4 (lane / 16) + h, voxel z0 + 16 zb + lane mod 16).  Per unit
// the 16 rows x 64 planes of Q (one matrix product per 16 planes and group of
// bins), which pass through the wave's four LDS rows; the products of the next
// unit are under way while the last rows of this one are gathered.
template <int NZB, int PLANES>
__device__ __forceinline__ void tof_back_rows(const ProjArgs &a, const LineP &L, const TofBack &k, int z0,
                                              double (&acc)[4][NZB]) {
    const TofUnitList units = (TofUnitList)(uintptr_t)a.units;
    const int nt = a.tof.n_tof;
    float rho[NZB];
#pragma unroll
    for (int zb = 0; zb < NZB; ++zb) {
        rho[zb] = gather_rho<PLANES>(a, z0 + 16 * zb + (lane_here() & 15));
        __builtin_amdgcn_sched_barrier(0);  // (one by one: registers)
    }
    const float last = (float)a.n_etab, kappa = a.kappa;
    float w[KEEP_KK], w_dz2 = -1.f;
#pragma unroll
    for (int q = 0; q < KEEP_KK; ++q) w[q] = 0.f;

    // Tiles of unit u: 16 T planes, K groups of bins from the kc-th on.  Bins past
    // the last one and planes past the unit's last tile read other factors (the
    // LDS past the units holds finite numbers too): weight 0, or columns that
    // nothing uses.
    f32x4 D[4];
    auto groups = [&](auto tiles, auto count, auto first, int u, int kc, bool fresh) {
        constexpr int T = tiles.value, K = count.value;
        const int lane = lane_here();
        const float *F = k.Fs + (u - k.u0) * a.unit_floats + 64 * (k.kk0 + kc) + lane;
        float fv[T][K];
#pragma unroll
        for (int pb = 0; pb < T; ++pb) {
            const float *Fb = F + pb * nt * 16;
#pragma unroll
            for (int q = 0; q < K; ++q) fv[pb][q] = Fb[64 * q];
        }
        if (fresh) {
            const TofPos tp = k.utab[u];
            const int b = 4 * (k.kk0 + kc) + (lane >> 4);  // this lane's bin of the first group
            const float p = fmaf((float)b, a.dpos, fmaf((float)(16 * k.rb + (lane & 15)), tp.pA, tp.pB));
            float f[2 * K];
            float4 c[2 * K];
            // (the table reads together)
#pragma unroll
            for (int q = 0; q < 2 * K; ++q) {
                const float pq = __builtin_amdgcn_fmed3f(fmaf((float)(4 * (q / 2) + q % 2), a.dpos, p), 0.f, last);
                f[q] = __builtin_amdgcn_fractf(pq);
                c[q] = k.tab[(int)pq];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < K; ++q) {
                const float lo = cubic_at(c[2 * q], f[2 * q]), hi = cubic_at(c[2 * q + 1], f[2 * q + 1]);
                w[q] = b + 4 * q < nt ? fmaxf(hi - lo, 0.f) : 0.f;
            }
        }
#pragma unroll
        for (int q = 0; q < K; ++q)
#pragma unroll
            for (int pb = 0; pb < T; ++pb)
                D[pb] = mfma16(w[q], fv[pb][q], first.value && q == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : D[pb]);
    };
    auto products = [&](int u) {
        const float dz2 = units[u].dz2;
        const int np = units[u].np;
        // (segments -k and +k are neighbours: the same length, the same weights)
        const bool fresh = dz2 != w_dz2;
        w_dz2 = dz2;
        auto all = [&](auto tiles) {
            groups(tiles, Int<2>(), Int<1>(), u, 0, true);
            for (int kc = 2; kc < k.nkk; kc += 2) groups(tiles, Int<2>(), Int<0>(), u, kc, true);
            w_dz2 = -1.f;
        };
        if (np <= 32)
            all(Int<2>());
        else if (k.nkk == 2)
            groups(Int<4>(), Int<2>(), Int<1>(), u, 0, fresh);
        else if (k.nkk == 3)
            groups(Int<4>(), Int<3>(), Int<1>(), u, 0, fresh);
        else
            all(Int<4>());
    };

    if ((lane_here() & 15) < GATHER_ZEROS) k.stage[(lane_here() >> 4) * STAGE_COLS + (lane_here() & 15)] = 0.f;
    products(k.u0);
    for (int u = k.u0; u < k.u1; ++u) {
        const int np = units[u].np, n1 = units[u].n1, neg = units[u].neg;
        const float rd = units[u].k;
        const int npb = (np + 15) >> 4;
        const int lane = lane_here(), pl = lane & 15, g = lane >> 4;
        float *srow = k.stage + g * STAGE_COLS;
        // in the gather, this lane's rows are 4 g + h of the block
        const float row0 = (float)(L.i_lo + 16 * k.rb + 4 * g);
        // the columns of this lane's planes (opaque: formed once per unit)
        float *col[4];
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
            int c = g * STAGE_COLS + 16 * pb + pl + (n1 == np || 16 * pb + pl < n1 ? 1 : 2) * GATHER_ZEROS;
            asm volatile("" : "+v"(c));
            col[pb] = k.stage + c;
        }
        wave_lds_order();
        // The zeros between and after the segments (those before stay; the planes that
        // fill up the last tile are zeros too, three of them are enough after a single
        // segment).
        if ((n1 < np || 16 * npb < np + GATHER_ZEROS) && (pl & 3) < GATHER_ZEROS && pl < 8)
            srow[(pl < 4 ? n1 + GATHER_ZEROS : np + 2 * GATHER_ZEROS) + (pl & 3)] = 0.f;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            wave_lds_order();
#pragma unroll
            for (int pb = 0; pb < 4; ++pb)
                if (pb < npb) *col[pb] = D[pb][h];
            wave_lds_order();
            __builtin_amdgcn_sched_barrier(0);
            if (h == 3 && u + 1 < k.u1) products(u + 1);
            __builtin_amdgcn_sched_barrier(0);
            // (as gather_cells: the sensitivity and what is divided by it have the same shares)
            const float lam = fmaf(row0 + (float)h, L.dlam, L.lam0);
            auto segment = [&](const GatherSeg &G, float slope) {
                decltype(gather_planes<PLANES>(srow, G, 0.f, kappa)) v[NZB];
#pragma unroll
                for (int zb = 0; zb < NZB; ++zb)
                    v[zb] = gather_planes<PLANES>(srow, G, fmaf(-slope, G.k, rho[zb]), kappa);
#pragma unroll
                for (int zb = 0; zb < NZB; ++zb) acc[h][zb] += (double)v[zb];
            };
            segment({rd, 0.f, (float)(n1 + 1), GATHER_ZEROS - 1}, neg ? 1.f - lam : lam);
            if (n1 < np) segment({rd, 0.f, (float)(np - n1 + 1), n1 + 2 * GATHER_ZEROS - 1}, lam);
        }
    }
}

// A line that misses the image: forward values from the additive terms alone, in
// memory order; it has no adjoint.
__device__ __forceinline__ void tof_line_outside(const ProjArgs &a, int line, int tid) {
    const int nt = a.tof.n_tof, n = a.n_planes * nt, nb = blockDim.x;
    const int64_t lor0 = (int64_t)line * a.n_planes, base = lor0 * nt;
    for (int e0 = tid; e0 < n; e0 += 4 * nb) {
        float m[4], v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + q * nb;
            m[q] = v[q] = 0.f;
            if (e >= n) continue;
            m[q] = a.mult ? a.mult[lor0 + e / nt] : 1.f;
            if (a.add) v[q] = a.add[base + e];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + q * nb;
            if (e < n) a.out[base + e] = fmaf(m[q], 0.f, v[q]);
        }
    }
}

// What the adjoint spreads of a bin: m its factor, s its projection, v the
// additive term (M_HVP: the mean data, M_BACK: the data), y its counts.  em: the EM
// ratio instead of the gradient's factor.
template <int MODE>
__device__ __forceinline__ float tof_factor(bool em, float m, float s, float v, float y, float ell) {
    if constexpr (MODE == M_BACK) return v * m * ell;
    // data-term Hessian: mult^2 y / ybar^2 (P v), then back
    if constexpr (MODE == M_HVP) return y != 0.f ? m * m * y / (v * v) * s * ell : 0.f;
    // a bin without counts: derivative 1, EM ratio 0
    const float ri = __builtin_amdgcn_rcpf(fmaf(m, s, v)), one = em ? 0.f : 1.f;
    return m * (y != 0.f ? fmaf(em ? y : -y, ri, one) : one) * ell;
}

// A value that is the same in all lanes, in a scalar register.
__device__ __forceinline__ float uniform(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// One transaxial line of a TOF geometry by the whole workgroup (the likelihood has
// kernels of its own, walk.hip).  MB blocks of 16 bins; the adjoint takes 16 NZB
// voxels along z at a time and gathers with the form PLANES; the forward takes
// TILES tiles of 16 planes at a time (16 registers of sums with four tiles or two
// blocks of bins).
template <int MODE, int MB, int NZB, int PLANES, int TILES>
__device__ __forceinline__ void line_tof_body(const ProjArgs &a, int line, float *smem, int wave, int64_t g_off = 0) {
    constexpr bool NEED_X = MODE != M_BACK;
    constexpr bool NEED_Z = MODE == M_BACK || MODE == M_GRAD || MODE == M_HVP;
    const int nw = blockDim.x >> 6;
    const LineP L = scalar_ref(a.lines[line]);
    const int nrow = L.i_hi - L.i_lo + 1;
    const int rz = a.rz, nt = a.tof.n_tof;
    if (nrow <= 0) {  // (uniform)
        if (MODE == M_FWD) tof_line_outside(a, line, 64 * wave + lane_here());
        return;
    }
    const int tid = 64 * wave + lane_here();
    // LDS: X | factors of q_units units | per wave: rows of Q | units' table
    // positions | table of E
    float *X = smem;
    float *Fs = smem + (NEED_X ? tof_x_floats(a.rows_max, a.x_stride) : 0);
    const int n_slots = NEED_Z ? a.q_units : 0;
    float *stage = Fs + n_slots * a.unit_floats + wave * TOF_STAGE_FLOATS;
    TofPos *utab = reinterpret_cast<TofPos *>(Fs + n_slots * a.unit_floats + (NEED_Z ? nw * TOF_STAGE_FLOATS : 0));
    float4 *tab = reinterpret_cast<float4 *>(utab + a.n_units);
    const float lam_s = fmaf((float)L.i_lo, L.dlam, L.lam0) - 0.5f;
    const TofUnitList units = (TofUnitList)(uintptr_t)a.units;
    for (int k = tid; k <= a.n_etab; k += blockDim.x) tab[k] = a.etab[k];
    for (int k = tid; k < a.n_units; k += blockDim.x) {
        const float len = sqrtf(L.lt2 + a.units[k].dz2);
        const double len_d = sqrt((double)L.lt2 + a.units[k].dz2), da = -L.dlam * len_d * a.e_scale;
        const double db = ((double)a.tof.tb[0] - a.tof.half_bin - ((double)L.i_lo * L.dlam + L.lam0 - 0.5) * len_d) * a.e_scale;
        const double j0 = rint(fmin(fmax(-db / da, -1e6), 1e6));
        const float a_hi = high_part((float)da);
        utab[k] = {(float)da, (float)(db + a.e_mid),
                   L.vm_um * len, a_hi, (float)(da - a_hi), (float)fma(j0, da, db), (float)j0, 0.f};
    }
    if (NEED_Z)  // (read past the units' bins and planes: finite numbers)
        for (int k = tid; k < n_slots * a.unit_floats + nw * TOF_STAGE_FLOATS; k += blockDim.x) Fs[k] = 0.f;
    if (NEED_X) {
        build_sheet(a, L, nrow, X, a.x_stride, tid);
        // (the forward walks four rows at a time)
        for (int e = nrow * a.x_stride + tid; e < ((nrow + 3) & ~3) * a.x_stride; e += blockDim.x) X[e] = 0.f;
    }
    __syncthreads();

    // rows [j_lo, j_hi] that some bin reaches (|t| grows with the length, so the
    // shortest LOR bounds it; one row of margin)
    const float reach = uniform(a.tof.tb[nt - 1] + a.tof.half_bin + a.tof.erf_clamp / a.tof.inv_sqrt2_sigma);
    const float len0 = uniform(sqrtf(L.lt2)), len1 = uniform(sqrtf(fmaf(a.k_max * a.k_max, a.pitch2, L.lt2)));
    int j_lo = 0, j_hi = nrow - 1;
    if (NEED_X) {
        const float h = reach / len0, r0 = (-h - lam_s) / L.dlam, r1 = (h - lam_s) / L.dlam;
        const float lo = fmaxf(floorf(fminf(r0, r1)) - 1.f, 0.f), hi = fminf(ceilf(fmaxf(r0, r1)) + 1.f, (float)(nrow - 1));
        if (lo <= hi) {
            j_lo = __builtin_amdgcn_readfirstlane((int)lo) & ~3;  // (steps of four end inside X)
            j_hi = __builtin_amdgcn_readfirstlane((int)hi);
        } else {
            j_hi = -1;
        }
    }

    // A line of few blocks of rows deals each block to several waves, which take shares
    // of the units and spread their cells by themselves: gradient of 161 x 161 x 33
    // voxels, 25 bins, 17 units 589 -> 546 us, of 128 x 128 x 71, 13 bins, 41 units
    // 874 -> 795.  Shares of one unit cost more in the spreading than they gain
    // (backprojection of 96 x 96 x 5 voxels, three units, 38.5 -> 42.5 us) unless the
    // lines leave the chip idle, as do those of a group of units where the cells leave
    // per group.
    const int nblk = NEED_Z ? (nrow + 15) >> 4 : 0;
    int lg_parts = 0, part = 0, rb0 = wave;
    if (NEED_Z && a.nz <= 16 * NZB) {
        const int least = gridDim.x > FEW_LINES ? 2 : 1;  // units of a share
        while ((nblk << (lg_parts + 1)) <= nw && min(a.q_units, a.n_units) >> (lg_parts + 1) >= least) ++lg_parts;
        while (rb0 >= nblk && part + 1 < 1 << lg_parts) {
            rb0 -= nblk;
            ++part;
        }
    }
    const int nzc = (a.nz + 16 * NZB - 1) / (16 * NZB);
    // a wave's cells stay in its registers over the groups of units if it has
    // one block of rows and one pass along z; else they are spread per group
    const bool keep = nblk <= nw && nzc == 1;
    double acc[4][NZB];
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int zb = 0; zb < NZB; ++zb) acc[h][zb] = 0.0;

    for (int u0 = 0; u0 < a.n_units; u0 += a.q_units) {
        const int u1 = NEED_Z ? min(u0 + a.q_units, a.n_units) : a.n_units;
        // ---- forward projection and factors, one unit per wave ----
        for (int u = u0 + wave; u < u1; u += nw) {
            const int lane = lane_here(), pl = lane & 15, g = lane >> 4;
            const int p0 = units[u].p0, np = units[u].np;
            const int npb = (np + 15) >> 4;
            const TofPos tp = utab[u];
            // Bin b of plane idx in LDS: F[(idx / 16 nt + b) 16 + idx mod 16] (the
            // tiles are filled up with zero planes), in memory base + idx nt + b.
            float *F = Fs + (u - u0) * a.unit_floats;
            const int64_t lor0 = (int64_t)line * a.n_planes + p0, base = lor0 * nt;
            auto slow = [&](int i0, int i1, auto each) {  // the bins of planes [i0, i1), one per lane and round
#pragma unroll 1
                for (int e = i0 * nt + lane_here(); e < i1 * nt; e += 64) {
                    const int idx = (e * a.inv_nt) >> 16, b = e - idx * nt;  // (e < 64 n_tof <= 2048)
                    each(e, idx, b, F + ((idx >> 4) * nt + b) * 16 + (idx & 15));
                }
            };
            bool bad = false;  // a factor that is not finite
            // (TILES tiles of 16 planes at a time)
            for (int t0 = 0; t0 < (TILES == 4 ? 1 : npb); t0 += TILES) {
                const int nt0 = min(TILES, npb - t0);
                f32x4 D[MB][TILES];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int pb = 0; pb < TILES; ++pb) D[mb][pb] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (NEED_X) {
                    float zA[TILES], zB[TILES];
#pragma unroll
                    for (int pb = 0; pb < TILES; ++pb) {
                        const int idx = 16 * (t0 + pb) + pl;
                        const PlaneP P = a.planes[p0 + min(idx, np - 1)];
                        zA[pb] = idx < np ? P.zs * L.dlam : 0.f;
                        zB[pb] = idx < np ? (float)fma((double)L.lam0, P.zs, P.zb + (double)PADZ) : 0.f;
                    }
                    auto rows = [&](auto tiles) {
                        tof_fwd_rows<MB, tiles.value, TILES>(a, tab, X, j_lo, j_hi, L.i_lo, lane, tp, zA, zB, D);
                    };
                    if (nt0 == 1)
                        rows(Int<1>());
                    else if (nt0 == 2 || TILES == 2)
                        rows(Int<2>());
                    else if (nt0 == 3)
                        rows(Int<(TILES > 2 ? 3 : 2)>());
                    else
                        rows(Int<TILES>());
                }
                // (this lane's bins of plane idx = 16 (t0 + pb) + pl: mb bins_blk + 4 g + r)
                const int i0 = 16 * t0, i1 = min(np, 16 * (t0 + nt0));
                bool special = false;
                if (MODE == M_FWD) {
                    float top = 0.f;  // (NaN and inf stay)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int pb = 0; pb < TILES; ++pb)
#pragma unroll
                            for (int r = 0; r < 4; ++r) top += fabsf(D[mb][pb][r]);
                    special = __any(!(top < INFINITY));
                }
                if (MODE == M_FWD && special) {
                    // (without the products of zero weights)
                    slow(i0, i1, [&](int e, int idx, int b, float *) {
                        const float sum = tof_fwd_guarded(a, tab, X, L, nrow, tp, a.planes[p0 + idx], b);
                        a.out[base + e] = fmaf(a.mult ? a.mult[lor0 + idx] : 1.f, sum * tp.ell, a.add ? a.add[base + e] : 0.f);
                    });
                    continue;
                }
                float top = 0.f;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int b0 = mb * a.bins_blk + 4 * g;
                    const int nb = min(a.bins_blk - 4 * g, nt - b0);  // this lane's bins of the block (at most 4 used)
                    // (two tiles' loads in flight together)
#pragma unroll
                    for (int ph = 0; ph < TILES; ph += 2) {
                        if (ph < nt0) {
                            float v[TILES][4], yv[TILES][4], m[TILES];
#pragma unroll
                            for (int pb = ph; pb < ph + 2; ++pb) {
                                const int idx = 16 * (t0 + pb) + pl;
                                const bool has = idx < np;
                                const int n = has ? nb : 0;
                                const int off = idx * nt + b0;
                                m[pb] = 0.f;
#pragma unroll
                                for (int r = 0; r < 4; ++r) v[pb][r] = yv[pb][r] = 0.f;
                                if (n <= 0) continue;
                                m[pb] = a.mult ? a.mult[lor0 + idx] : 1.f;
                                if constexpr (MODE == M_BACK) {
#pragma unroll
                                    for (int r = 0; r < 4; ++r) v[pb][r] = 1.f;
                                    if (a.sino) load_bins(a.sino + base + off, n, v[pb]);
                                } else if constexpr (MODE == M_HVP) {
                                    load_bins(a.ybar + base + off, n, v[pb]);
                                } else {
                                    if (a.add) load_bins(a.add + base + off, n, v[pb]);
                                }
                                if constexpr (MODE != M_BACK && MODE != M_FWD)
                                    load_counts(a.y, a.y_dtype, base + off, n, yv[pb]);
                            }
#pragma unroll
                            for (int pb = ph; pb < ph + 2; ++pb) {
                                const int idx = 16 * (t0 + pb) + pl;
                                const bool has = idx < np;
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    if (r >= nb || pb >= nt0) continue;
                                    const float s = D[mb][pb][r] * tp.ell;
                                    float Q = 0.f;
                                    if constexpr (MODE == M_FWD) v[pb][r] = fmaf(m[pb], s, v[pb][r]);
                                    if constexpr (NEED_Z)
                                        Q = tof_factor<MODE>(a.em, m[pb], s, v[pb][r], yv[pb][r], tp.ell);
                                    if (NEED_Z) {
                                        if (!has) Q = 0.f;
                                        top += fabsf(Q);
                                        F[((t0 + pb) * nt + b0 + r) * 16 + pl] = Q;
                                    }
                                }
                                if constexpr (MODE == M_FWD)
                                    if (has) store_bins(a.out + base + idx * nt + b0, nb, v[pb]);
                            }
                        }
                    }
                }
                bad |= !(top < INFINITY);
            }
            if (NEED_Z && __any(bad)) {
                // (the products also take a bin's sum from rows, and its factor to
                // rows and planes, where the weight is 0)
                wave_lds_order();
                slow(0, np, [&](int e, int idx, int b, float *f) {
                    float Q = *f;
                    if (fabsf(Q) < INFINITY) return;
                    if (NEED_X) {
                        const float s = tof_fwd_guarded(a, tab, X, L, nrow, tp, a.planes[p0 + idx], b) * tp.ell;
                        const float v = MODE == M_HVP ? a.ybar[base + e] : a.add ? a.add[base + e] : 0.f;
                        Q = tof_factor<MODE>(a.em, a.mult ? a.mult[lor0 + idx] : 1.f, s, v, load_y(a.y, a.y_dtype, base + e), tp.ell);
                    }
                    if (fabsf(Q) < INFINITY) {
                        *f = Q;
                        return;
                    }
                    tof_back_special(a, L, tab, nrow, tp, a.planes[p0 + idx], b, Q, g_off);
                    *f = 0.f;
                });
            }
        }
        if (!NEED_Z) break;
        __syncthreads();

        // ---- adjoint, one block of 16 rows per wave ----
        for (int iz = 0; iz < nzc; ++iz) {
            const int z0 = 16 * NZB * iz;
            for (int rb = rb0; rb < nblk; rb += nw) {
                const int ua = u0 + ((u1 - u0) * part >> lg_parts), ub = u0 + ((u1 - u0) * (part + 1) >> lg_parts);
                if (!keep) {
#pragma unroll
                    for (int h = 0; h < 4; ++h)
#pragma unroll
                        for (int zb = 0; zb < NZB; ++zb) acc[h][zb] = 0.0;
                }
                // the groups of four bins that reach these rows at some length
                const float la = fmaf((float)(16 * rb), L.dlam, lam_s);
                const float lb = fmaf((float)min(16 * rb + 15, nrow - 1), L.dlam, lam_s);
                const float l0 = fminf(la, lb), l1 = fmaxf(la, lb);
                const float t0 = l0 * (l0 < 0.f ? len1 : len0), t1 = l1 * (l1 < 0.f ? len0 : len1);
                const float rbw = 0.5f / a.tof.half_bin, sup = reach - a.tof.tb[nt - 1];
                const int b0 = (int)fmaxf(floorf((t0 - sup - a.tof.tb[0]) * rbw - 0.01f), 0.f);
                const int b1 = (int)fmaxf(fminf(ceilf((t1 + sup - a.tof.tb[0]) * rbw + 0.01f), (float)(nt - 1)), -1.f);
                const int kk0 = __builtin_amdgcn_readfirstlane(b0) >> 2;
                const int nkk = (__builtin_amdgcn_readfirstlane(b1) >> 2) + 1 - kk0;
                if (nkk > 0 && ua < ub) {
                    const TofBack k = {Fs + (ua - u0) * a.unit_floats, stage, utab, tab, ua, ub, rb, kk0, nkk};
                    tof_back_rows<NZB, PLANES>(a, L, k, z0, acc);
                }
                if (!keep || u1 == a.n_units) {
                    // the cells to the global sheet, through the staged rows so that
                    // consecutive lanes add to consecutive voxels
                    const int ln = lane_here();
                    float *Gout = (L.axis ? a.G1 : a.G0) + g_off;
                    const int other_stride = ((L.axis ? a.nx : a.ny) + 2 * PADA) * rz;
                    const int nz = min(16 * NZB, a.nz - z0);
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        wave_lds_order();
                        float *sc = stage + (ln >> 4) * STAGE_COLS + (ln & 15);
#pragma unroll
                        for (int zb = 0; zb < NZB; ++zb) sc[16 * zb] = (float)acc[h][zb];
                        wave_lds_order();
                        for (int sr = 0; sr < STAGE_ROWS; ++sr) {
                            const int j = 16 * rb + 4 * sr + h;
                            if (j >= nrow) break;
                            const SheetRow row = sheet_row(L, L.i_lo + j, other_stride, rz);
                            for (int z = ln; z < nz; z += 64) {
                                const float val = stage[sr * STAGE_COLS + z];
                                if (val != 0.f) spread_cell(Gout, row, z0 + z + PADZ, rz, val);
                            }
                        }
                    }
                }
            }
        }
        if (u1 < a.n_units) __syncthreads();
    }
}

// One line per workgroup, in the order a.order (longest first).
template <int MODE, int MB, int NZB, int PLANES>
__global__ void __launch_bounds__(TOF_BLOCK, MODE == M_FWD && MB == 1 ? 8 : 4) k_line_tof(ProjArgs a) {
    extern __shared__ float4 smem4[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    line_tof_body<MODE, MB, NZB, PLANES, MB == 1 ? 4 : 2>(a, a.order[blockIdx.x], reinterpret_cast<float *>(smem4), wave);
}

// Work counts of a TOF line: samples, and sample-bin pairs within the bins'
// supports (intervals between the support edges), one plane per thread.
__global__ void __launch_bounds__(NT_BLOCK) k_count_tof(ProjArgs a) {
    const LineP L = a.lines[a.order[blockIdx.x]];
    const int nrow = L.i_hi - L.i_lo + 1;
    double samples = 0.0, pairs = 0.0;
    for (int p = threadIdx.x; nrow > 0 && p < a.n_planes; p += blockDim.x) {
        const PlaneP P = a.planes[p];
        const float len = sqrtf(L.lt2 + P.dz2);
        int is, ie;
        z_clip<true>(L, P, a.nz, is, ie);
        if (ie < is) continue;
        // this plane's samples in t order
        const int qlo = L.dlam > 0.f ? is - L.i_lo : L.i_hi - ie;
        const int qhi = L.dlam > 0.f ? ie - L.i_lo : L.i_hi - is;
        samples += (double)(ie - is + 1);
        for (int s = 0; s < a.tof.n_int; ++s) {
            const int na = a.tof.na[s];
            if (na <= 0) continue;
            const int c0 = max(cut_count(a.tof.edge[s], len, L.lam0, L.dlam, L.i_lo, L.i_hi), qlo);
            const int c1 = min(cut_count(a.tof.edge[s + 1], len, L.lam0, L.dlam, L.i_lo, L.i_hi), qhi + 1);
            if (c1 > c0) pairs += (double)na * (c1 - c0);
        }
    }
    block_sums(samples, pairs, a.partial, true);
}

// The form of the TOF kernels that serves a geometry:
//  * one or two blocks of 16 bins (a second, empty one would cost as many weights
//    and products as the first);
//  * 16 to 80 voxels along z per pass of the adjoint, so that passes and cells past
//    the axis, gathered for nothing, cost least (each pass forms the products of all
//    units, worth 1.3 groups of 16 voxels): gradient of 33 slices and 25 bins, 690 us
//    in passes of 80, 601 of 48; of 16 slices and 13 bins, 78 of 48, 68 of 16;
//  * two or three planes of a segment per voxel, or any number (see line_sheets.h).
template <typename F>
void tof_form(int n_tof, int nz, int planes, F &&f) {
    auto bins = [&](auto nzb, auto pl) { n_tof <= 16 ? f(Int<1>(), nzb, pl) : f(Int<2>(), nzb, pl); };
    const int groups = (nz + 15) / 16;
    auto slices = [&](auto pl) {
        auto cost = [&](int n) { return (groups + n - 1) / n * (10 * n + 13); };
        int best = 1;
        for (int n = 2; n <= STAGE_ZB; ++n)
            if (cost(n) < cost(best)) best = n;
        switch (best) {
            case 1: bins(Int<1>(), pl); break;
            case 2: bins(Int<2>(), pl); break;
            case 3: bins(Int<3>(), pl); break;
            case 4: bins(Int<4>(), pl); break;
            default: bins(Int<STAGE_ZB>(), pl);
        }
    };
    if (planes == 2)
        slices(Int<2>());
    else if (planes == 3)
        slices(Int<3>());
    else
        groups == 1 ? bins(Int<1>(), Int<GATHER_SOME>()) : bins(Int<3>(), Int<GATHER_SOME>());
}

// Persistent subset-gradient kernel over a batch: the work items of one step
// are the transaxial lines of every active member (all lines at a snapshot,
// each into the gradient-sheet slot of its view's subset; else the lines of
// the step's subset into slot 0), concatenated in `order`.  Workgroups take
// items from a global counter (zeroed by the step's prep kernel) until none
// is left.  MB, NZB, PLANES: the TOF form that serves every member (see tof_form;
// each form of the line body also serves fewer bins, shorter axes, fewer planes).
template <int MB, int NZB, int PLANES>
__global__ void __launch_bounds__(64 * MAX_WAVES) k_line_batched(const BMember *__restrict__ mem,
                                                                     const int *__restrict__ order, int n_mem,
                                                                     int step, int *__restrict__ counter) {
    extern __shared__ float4 smem4[];
    float *smem = reinterpret_cast<float *>(smem4);
    __shared__ int s_cum[BATCH_MAX + 1];
    __shared__ int s_item;
    if (threadIdx.x == 0) {
        int c = 0;
        for (int q = 0; q < n_mem; ++q) {
            s_cum[q] = c;
            const BMember &m = mem[order[q]];
            const BStep st = m.steps[step];
            if (st.flags & B_ACTIVE) c += ((st.flags & B_SNAP) ? m.n_views : m.sub_nviews[st.subset]) * m.pa.n_rad;
        }
        s_cum[n_mem] = c;
    }
    __syncthreads();
    const int total = __builtin_amdgcn_readfirstlane(s_cum[n_mem]);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (;;) {
        if (wave == 0 && lane_here() == 0) s_item = atomicAdd(counter, 1);
        __syncthreads();
        // (scalar, and so the member's arguments)
        const int item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= total) break;
        int q = 0;
        while (__builtin_amdgcn_readfirstlane(s_cum[q + 1]) <= item) ++q;
        const BMember &m = mem[order[q]];
        const ProjArgs &pa = scalar_ref(m.pa);
        const BStep st = m.steps[step];
        const int local = item - __builtin_amdgcn_readfirstlane(s_cum[q]);
        const int n_rad = pa.n_rad;
        const int jv = local / n_rad;
        const int k = local - jv * n_rad;
        const bool snap = (st.flags & B_SNAP) != 0;
        const int view = __builtin_amdgcn_readfirstlane(snap ? jv : m.views[st.subset * m.views_stride + jv]);
        const int64_t g_off = snap ? (int64_t)(jv % m.n_sub) * m.g_slot : 0;
        if (m.is_tof) {
            line_tof_body<M_GRAD, MB, NZB, PLANES, MB == 1 ? 4 : 2>(pa, view * n_rad + k, smem, wave, g_off);
        } else {
            line_nt_body<M_GRAD>(pa, view * n_rad + k, smem, 64 * wave + lane_here(), g_off);
        }
        __syncthreads();
    }
}

// LDS of the non-TOF line kernel: the image sheet (modes that project), the planes'
// factors (modes that backproject) and the folded TOF weights of a block of rows.
template <int MODE>
size_t nt_lds(const pet_geom_s *g) {
    if (MODE == M_COUNT) return 0;
    const size_t sheet = ((size_t)g->rows_max * (g->d.nz + 2 * PADZ) + 3) & ~(size_t)3;
    const bool x = MODE != M_BACK, q = MODE == M_BACK || MODE == M_GRAD || MODE == M_EM || MODE == M_HVP;
    return sizeof(float) * ((x ? sheet : 0) + (q ? (size_t)g->q_floats : 0) +
                            (MODE == M_BACK && g->d.n_tof > 1 ? (size_t)FOLD_FLOATS : 0));
}

// Threads of a non-TOF line.  With a forward projection as many as planes (the sums'
// order depends on it); a backprojection's work are the cells of the line's sheet:
// eight per thread (two planes at most) where the lines fill the chip, two where they
// leave it idle.  (Sensitivity of 96 x 96 x 32 voxels and 32 planes 45 us with 64
// threads, 36 with 448; of 97 x 88 x 27 and 231 planes, 350 lines, 22 with 384, 19
// with 1024; backprojection of 128 x 128 x 48 and 1037 planes 106 us with 1024, 102
// with 512.)
template <int MODE>
int nt_threads(const pet_geom_s *g, unsigned lines) {
    if (MODE != M_BACK) return g->nt_threads;
    const bool few = lines <= FEW_LINES;
    const int work = std::max(g->rows_max * g->d.nz / (few ? 2 : 8), g->n_planes / 2);
    return std::max(64, std::min((work + 63) / 64 * 64, few ? NT_BLOCK : NT_BLOCK / 2));
}

template <int MODE, int MB, int NZB, int PLANES>
hipError_t launch_tof(const pet_geom_s *g, dim3 grid, ProjArgs a, hipStream_t s) {
    const bool x = MODE != M_BACK, z = MODE != M_FWD;
    if (MODE == M_BACK) a.q_units = g->q_units_back;
    // Without an adjoint a wave has nothing but units to do: no more waves than units
    // (four at least, for the image sheet), and more workgroups on a CU instead: five
    // units, all views, 96 x 96 x 32, 255 -> 225 us with 64 registers.  Fewer waves for
    // even rounds of many units are slower (41 on 7 waves 367 us against 347 on 8; 17
    // on 6: 173 against 162): less is in flight.
    // With an adjoint: fewer waves, and more workgroups on a CU, so that one workgroup's
    // phases overlap the others', where the lines fill the chip with them and the LDS
    // takes three workgroups of four waves (four with more units than eight waves take
    // at once).  Four waves from three lines per CU: gradients (backprojections) of
    // 96 x 96 x 32 voxels and five units 101 -> 90 (72 -> 61) us, of 96 x 96 x 5 and
    // three units 51 -> 36 (39 -> 28), 784 lines of 13 units 52 -> 42; but 576 lines 44
    // -> 56, 85 lines 23 -> 28, and 29 units with room for three workgroups 98 -> 119.
    // Where units and blocks of rows are four at most there is nothing for more waves, so
    // from FEW_LINES on: 735 lines, 58 x 52 x 7 voxels, three units 27 -> 21, four 34 -> 24.
    // Two waves for one or two units, from six lines per CU: 1896 lines of one unit 61
    // -> 42 (four: 49), 10191 of two 308 -> 220 (228); three units 565 -> 482 (405).
    // Units in several groups are slower so (29, backprojection, 276 -> 303).
    int waves = TOF_BLOCK / 64;
    if (!z)
        waves = std::min(waves, std::max(4, g->n_units));
    else if (grid.x >= (g->n_units <= 4 && g->rows_max <= 64 ? FEW_LINES : 3 * CUS) && a.q_units >= g->n_units &&
             tof_lds_bytes(g, x, a.q_units, 4) <= CU_LDS_BYTES / (g->n_units > waves ? 4 : 3))
        waves = g->n_units <= 2 && grid.x >= 6 * CUS ? 2 : 4;
    const size_t lds = tof_lds_bytes(g, x, z ? a.q_units : 0, z ? waves : 0);
    static size_t granted = 64 * 1024;
    if (lds > granted) {
        hipError_t e = hipFuncSetAttribute((const void *)k_line_tof<MODE, MB, NZB, PLANES>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e == hipSuccess) granted = lds;
        (void)hipGetLastError();
    }
    hipLaunchKernelGGL((k_line_tof<MODE, MB, NZB, PLANES>), grid, dim3(64 * waves), lds, s, a);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const pet_geom_s *g, dim3 grid, const ProjArgs &a, hipStream_t s) {
    if (g->d.n_tof == 1) {
        hipLaunchKernelGGL((k_line_nt<MODE>), grid, dim3(nt_threads<MODE>(g, grid.x)), nt_lds<MODE>(g), s, a);
        return hipGetLastError();
    }
    if constexpr (MODE == M_COUNT) {
        hipLaunchKernelGGL(k_count_tof, grid, dim3(g->nt_threads), 0, s, a);
        return hipGetLastError();
    } else if constexpr (MODE == M_OBJ) {
        return launch_tof_walk(g, M_OBJ, grid, a, s);
    } else if constexpr (MODE == M_EM) {
        ProjArgs em = a;
        em.em = 1;
        return launch_mode<M_GRAD>(g, grid, em, s);
    } else {
        if (MODE == M_GRAD && a.partial) return launch_tof_walk(g, M_GRAD, grid, a, s);
        hipError_t e = hipSuccess;
        tof_form(a.tof.n_tof, a.nz, a.gather_planes, [&](auto mb, auto nzb, auto planes) {
            // (without an adjoint the last two make no difference, without a forward the first)
            if constexpr (MODE == M_FWD)
                e = launch_tof<MODE, mb.value, STAGE_ZB, 2>(g, grid, a, s);
            else
                e = launch_tof<MODE, MODE == M_BACK ? 2 : mb.value, nzb.value, planes.value>(g, grid, a, s);
        });
        return e;
    }
}

// Raise the dynamic-LDS limit of the non-TOF line kernels to what this geometry
// needs (checked against the device limit at creation).  Only needed above the
// default; a failure here is reported by the launch itself.
void set_lds_attr(size_t need) {
    static size_t granted = 64 * 1024;
    if (need <= granted) return;
    const void *fns[] = {(const void *)k_line_nt<M_FWD>,  (const void *)k_line_nt<M_BACK>,
                         (const void *)k_line_nt<M_GRAD>, (const void *)k_line_nt<M_EM>,
                         (const void *)k_line_nt<M_OBJ>,  (const void *)k_line_nt<M_HVP>};
    hipError_t e = hipSuccess;
    for (const void *f : fns)
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)need);
    if (e == hipSuccess) granted = need;
    (void)hipGetLastError();
}

// TOF backprojection of mult alone (the sensitivity P^T mult, no sinogram):
// with the bins' weights summed per sample, the non-TOF kernel does it, one
// share per LOR and cell instead of one per TOF bin.
hipError_t launch_back_fold(const pet_geom_s *g, dim3 grid, const ProjArgs &a0, hipStream_t s) {
    ProjArgs a = a0;
    a.tof_fold = 1;
    hipLaunchKernelGGL((k_line_nt<M_BACK>), grid, dim3(nt_threads<M_BACK>(g, grid.x)), nt_lds<M_BACK>(g), s, a);
    return hipGetLastError();
}

hipError_t launch_line_kernel_impl(const pet_geom_s *g, int mode, dim3 grid, const ProjArgs &a, hipStream_t s) {
    set_lds_attr(std::max(nt_lds<M_GRAD>(g), nt_lds<M_BACK>(g)));
    switch (mode) {
        case M_FWD: return launch_mode<M_FWD>(g, grid, a, s);
        case M_BACK:
            if (g->d.n_tof > 1 && !a.sino) return launch_back_fold(g, grid, a, s);
            return launch_mode<M_BACK>(g, grid, a, s);
        case M_GRAD: return launch_mode<M_GRAD>(g, grid, a, s);
        case M_EM: return launch_mode<M_EM>(g, grid, a, s);
        case M_OBJ: return launch_mode<M_OBJ>(g, grid, a, s);
        case M_COUNT: return launch_mode<M_COUNT>(g, grid, a, s);
        case M_HVP: return launch_mode<M_HVP>(g, grid, a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// (The batched kernel comes in passes of 48 and 80 voxels only.)
template <typename F>
static void batch_form(const BatchForm &f, F &&launch) {
    tof_form(f.n_tof, f.nz, f.planes, [&](auto mb, auto nzb, auto planes) {
        launch(mb, Int<(nzb.value <= 3 ? 3 : STAGE_ZB)>(), planes);
    });
}

hipError_t prime_line_batched(const BatchForm &f, size_t lds) {
    hipError_t e = hipSuccess;
    batch_form(f, [&](auto mb, auto nzb, auto planes) {
        static size_t granted = 64 * 1024;
        if (lds <= granted) return;
        e = hipFuncSetAttribute((const void *)k_line_batched<mb.value, nzb.value, planes.value>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e == hipSuccess) granted = lds;
    });
    return e;
}

hipError_t launch_line_batched(const BatchForm &f, const BMember *mem, const int *order, int n_mem, int step,
                               int *counter, int blocks, int waves, size_t lds, hipStream_t s) {
    batch_form(f, [&](auto mb, auto nzb, auto planes) {
        hipLaunchKernelGGL((k_line_batched<mb.value, nzb.value, planes.value>), dim3(blocks), dim3(64 * waves), lds, s, mem,
                           order, n_mem, step, counter);
    });
    return hipGetLastError();
}

int n_line_blocks(const pet_geom_s *g, int subset) {
    const int nv = subset < 0 ? g->d.n_views : (int)g->subset_views[subset].size();
    return nv * g->d.n_rad;
}

hipError_t launch_line_kernel(pet_geom_s *g, int mode, int subset, const ProjArgs &a, hipStream_t s) {
    dim3 grid(n_line_blocks(g, subset));
    if (grid.x == 0) return hipSuccess;
    if (!g->profiling) return launch_line_kernel_impl(g, mode, grid, a, s);
    std::pair<hipEvent_t, hipEvent_t> ev;
    if (!g->prof_pool.empty()) {
        ev = g->prof_pool.back();
        g->prof_pool.pop_back();
    } else {
        hipError_t e = hipEventCreate(&ev.first);
        if (e == hipSuccess) e = hipEventCreate(&ev.second);
        if (e != hipSuccess) return e;
    }
    hipError_t e = hipEventRecord(ev.first, s);
    if (e == hipSuccess) e = launch_line_kernel_impl(g, mode, grid, a, s);
    if (e == hipSuccess) e = hipEventRecord(ev.second, s);
    g->prof_events[mode].push_back(ev);
    return e;
}

}  // namespace pet
