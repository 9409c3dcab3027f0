// TOF line kernels with the Poisson likelihood (objective; fused subset gradient
// where its likelihood is wanted): the samples of every LOR walked one after the
// other.
//
// The likelihood is an FP64 output, a sum over 32-bit means, and shows their
// roundings: with the matrix products of line_tof_body (proj.hip), as exact as
// this walk, it moves by up to 3e-8 on small data.  The gradient without the
// likelihood, projections and Hessian products take the matrix form, which is
// 1.3 to 3.9 times as fast.
//
// All planes of one ring-difference segment share |u|, hence the signed distance
// t(i) of every sample and its TOF weights.  One wave takes one unit (a segment, or
// a pair -k, +k of at most 64 planes), one plane per lane, fills a table with the
// weights of the line's samples (increasing-t order) once, and the lanes read it by
// broadcast.  Per wave the LDS holds, for the unit being processed:
//   cuts[s]  (s = 0 .. n_int)   first sample (t order) at or beyond edge s;
//   w4[q], w1[q]                the TOF weights of the bins active at sample q
//                               (first four in a float4, the rest after).
// Samples q are numbered in increasing t along the LOR; the sample index,
// lambda and the sheet row follow from q and are the same for all lanes.
//
// Bound by the latency of its LDS reads and FP64 LDS atomics: a subset gradient of
// 128 x 128 x 71 voxels, 2204 planes and 13 bins 1.38 ms, 0.8 ms of it the
// likelihood's part.
#include "line_sheets.h"

#include <algorithm>
#include <climits>

namespace pet {
namespace {

constexpr int NT_BLK = 16;  // TOF bins a lane holds in registers at once

// The nt values src[base .. base + nt) of one LOR (one block of at most
// NT_BLK TOF bins), all loads issued before the first use (zero above nt).
template <typename T>
__device__ __forceinline__ void load_row(const T *src, int64_t base, int nt, float (&v)[NT_BLK]) {
#pragma unroll
    for (int b = 0; b < NT_BLK; ++b) v[b] = b < nt ? (float)src[base + b] : 0.f;
}
__device__ __forceinline__ void load_y_row(const void *y, int dt, int64_t base, int nt, float (&v)[NT_BLK]) {
    if (dt == PET_Y_U8)
        load_row((const uint8_t *)y, base, nt, v);
    else if (dt == PET_Y_U16)
        load_row((const uint16_t *)y, base, nt, v);
    else
        load_row((const float *)y, base, nt, v);
}

// erf of u / (sqrt2 sigma) with the argument clamped to the truncation window.
__device__ __forceinline__ float clamped_erf(float u, float inv_s, float c) {
    return erff(fminf(fmaxf(u * inv_s, -c), c));
}

// Order of a wave's LDS accesses across its lanes.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Per-wave TOF weight table of one LOR (one unit of the line): lane s
// computes the cut cuts[s] (rows before interval s in t order) and returns it;
// each row q of a non-empty interval gets the weights of its na bins.
__device__ __forceinline__ int fill_table(const ProjArgs &a, const LineP &L, float len, int *cuts, float *w4,
                                          float *w1) {
    const int lane = threadIdx.x & 63;
    const int nq = L.i_hi - L.i_lo + 1;
    const int e1 = a.ws > 4 ? a.ws - 4 : 0;
    int *sid = reinterpret_cast<int *>(w4);  // interval of row q, parked in w4[q].x
    int cut = 0;
    if (lane <= a.tof.n_int) {
        cut = cut_count(a.tof.edge[lane], len, L.lam0, L.dlam, L.i_lo, L.i_hi);
        cuts[lane] = cut;
    }
    for (int q = lane; q < nq; q += 64) sid[4 * q] = -1;
    wave_fence();
    // lane s marks the rows of interval s
    if (lane < a.tof.n_int && a.tof.na[lane] > 0) {
        const int hi = cuts[lane + 1];
        for (int q = cut; q < hi; ++q) sid[4 * q] = lane;
    }
    wave_fence();
    const float inv_s = a.tof.inv_sqrt2_sigma, c = a.tof.erf_clamp, h = a.tof.half_bin;
    for (int q = lane; q < nq; q += 64) {
        const int s = sid[4 * q];
        if (s < 0) continue;
        const int na = a.tof.na[s];
        const int i = L.dlam > 0.f ? L.i_lo + q : L.i_hi - q;
        const float lam = fmaf((float)i, L.dlam, L.lam0);
        const float t = (lam - 0.5f) * len;
        // weights of bins bf .. bf + na - 1 from shared bin edges
        const float t0 = a.tof.tb[a.tof.bf[s]] - h - t;
        float e_prev = clamped_erf(t0, inv_s, c);
        float w[WS_MAX];
        for (int j = 0; j < WS_MAX; ++j) w[j] = 0.f;
        for (int j = 0; j < na; ++j) {
            const float e_next = clamped_erf(t0 + (float)(j + 1) * (2.f * h), inv_s, c);
            w[j] = 0.5f * (e_next - e_prev);
            e_prev = e_next;
        }
        reinterpret_cast<float4 *>(w4)[q] = make_float4(w[0], w[1], w[2], w[3]);
        for (int j = 0; j < e1; ++j) w1[q * e1 + j] = w[4 + j];
    }
    wave_fence();
    return cut;
}

// Sample loops of one TOF interval: n rows walked in t order from row pointer
// xr / zr (row of the first sample), principal-plane index fi stepping by dfi and
// row stride drz.  The weights of a row are the same for every lane that walks it
// (broadcast LDS reads when the whole wave does).
//
// Axial positions are taken in padded-row cells, u = zA i + zB = z + PADZ: a sample
// at axial position z interpolates cells floor(u) and floor(u) + 1 of its sheet
// row.  u is clamped to [0, nz + 2], where the truncating conversion is the floor
// and v_fract the fraction.
template <int NA>
__device__ __forceinline__ void read_wq(const float *wq, const float *w1q, float (&w)[NA]) {
    const float4 v = *reinterpret_cast<const float4 *>(wq);
    if (NA > 0) w[0] = v.x;
    if (NA > 1) w[1] = v.y;
    if (NA > 2) w[2] = v.z;
    if (NA > 3) w[3] = v.w;
#pragma unroll
    for (int j = 4; j < NA; ++j) w[j] = w1q[j - 4];
}

// Forward: no lane predicate.  A sample outside the z-valid range
// [-1.5, nz + 0.5] (u outside [0.5, nz + 2.5]) interpolates between two cells
// of the zero padding and adds exactly zero, as does a lane without a plane
// (zA = 0, zB = 0).
template <int NA>
__device__ __forceinline__ void tof_fwd_run(float zA, float zB, float umax, const float *xr, int drz, float fi,
                                            float dfi, const float *wq, const float *w1q, int e1, int n, float *win) {
#pragma unroll 2
    for (; n > 0; --n) {
        float w[NA];
        read_wq<NA>(wq, w1q, w);
        const float u = __builtin_amdgcn_fmed3f(fmaf(fi, zA, zB), 0.f, umax);
        const int j = (int)u;
        const float f = __builtin_amdgcn_fractf(u);
        const float x0 = xr[j], x1 = xr[j + 1];
        const float v = fmaf(f, x1 - x0, x0);
#pragma unroll
        for (int b = 0; b < NA; ++b) win[b] = fmaf(v, w[b], win[b]);
        xr += drz;
        fi += dfi;
        wq += 4;
        w1q += e1;
    }
}

// Adjoint: a lane adds its samples k = q - qlo in [0, span] only.
template <int NA>
__device__ __forceinline__ void tof_back_run(float zA, float zB, float umax, double *zr, int drz, float fi, float dfi,
                                             const float *wq, const float *w1q, int e1, int n, int k, unsigned span,
                                             const float *win) {
#pragma unroll 2
    for (; n > 0; --n) {
        float w[NA];
        read_wq<NA>(wq, w1q, w);
        float Q = 0.f;
#pragma unroll
        for (int b = 0; b < NA; ++b) Q = fmaf(win[b], w[b], Q);
        if ((unsigned)k <= span) {
            // (the clamp only guards the LDS bounds; valid samples lie inside)
            const float u = __builtin_amdgcn_fmed3f(fmaf(fi, zA, zB), 0.f, umax);
            const int j = (int)u;
            const float a1 = Q * __builtin_amdgcn_fractf(u);
            atomicAdd(&zr[j], (double)(Q - a1));
            atomicAdd(&zr[j + 1], (double)a1);
        }
        zr += drz;
        fi += dfi;
        wq += 4;
        w1q += e1;
        ++k;
    }
}

// Bin window <-> the per-bin accumulators of one block of NT_BLK bins.  The
// window's first bin relative to the block, REL (from -(WS_MAX - 1) to
// NT_BLK - 1), is a template argument so that every register index is static:
// indexing a register array by a run-time value compiles to indexed register
// moves, which the compiler may execute speculatively for indices the source
// guards out and which then write registers past the array.
template <int REL>
__device__ __forceinline__ void add_window(float (&acc)[NT_BLK], const float (&win)[WS_MAX], int na) {
#pragma unroll
    for (int j = 0; j < WS_MAX; ++j)
        if (REL + j >= 0 && REL + j < NT_BLK && j < na) acc[REL + j] += win[j];
}

template <int REL>
__device__ __forceinline__ void get_window(const float (&acc)[NT_BLK], float (&win)[WS_MAX], int na) {
#pragma unroll
    for (int j = 0; j < WS_MAX; ++j) win[j] = (REL + j >= 0 && REL + j < NT_BLK && j < na) ? acc[REL + j] : 0.f;
}

static_assert(NT_BLK == 16 && WS_MAX == 8, "the window switch below covers first bins -7 .. 15 of a block");
#define PET_REL_SWITCH(FN, ...)                \
    switch (rel) {                             \
        case -7: FN<-7>(__VA_ARGS__); break;   \
        case -6: FN<-6>(__VA_ARGS__); break;   \
        case -5: FN<-5>(__VA_ARGS__); break;   \
        case -4: FN<-4>(__VA_ARGS__); break;   \
        case -3: FN<-3>(__VA_ARGS__); break;   \
        case -2: FN<-2>(__VA_ARGS__); break;   \
        case -1: FN<-1>(__VA_ARGS__); break;   \
        case 0: FN<0>(__VA_ARGS__); break;     \
        case 1: FN<1>(__VA_ARGS__); break;     \
        case 2: FN<2>(__VA_ARGS__); break;     \
        case 3: FN<3>(__VA_ARGS__); break;     \
        case 4: FN<4>(__VA_ARGS__); break;     \
        case 5: FN<5>(__VA_ARGS__); break;     \
        case 6: FN<6>(__VA_ARGS__); break;     \
        case 7: FN<7>(__VA_ARGS__); break;     \
        case 8: FN<8>(__VA_ARGS__); break;     \
        case 9: FN<9>(__VA_ARGS__); break;     \
        case 10: FN<10>(__VA_ARGS__); break;   \
        case 11: FN<11>(__VA_ARGS__); break;   \
        case 12: FN<12>(__VA_ARGS__); break;   \
        case 13: FN<13>(__VA_ARGS__); break;   \
        case 14: FN<14>(__VA_ARGS__); break;   \
        default: FN<15>(__VA_ARGS__); break;   \
    }

#define PET_NA_SWITCH(FN, ...)              \
    switch (na) {                           \
        case 1: FN<1>(__VA_ARGS__); break;  \
        case 2: FN<2>(__VA_ARGS__); break;  \
        case 3: FN<3>(__VA_ARGS__); break;  \
        case 4: FN<4>(__VA_ARGS__); break;  \
        case 5: FN<5>(__VA_ARGS__); break;  \
        case 6: FN<6>(__VA_ARGS__); break;  \
        case 7: FN<7>(__VA_ARGS__); break;  \
        default: FN<8>(__VA_ARGS__); break; \
    }

// Live intervals of a unit as a bit mask (bit s: interval s).  With the rows split
// over C chunks, chunk k takes the k-th set bit (-1 if there are fewer), and the
// wave then drops the lowest C.
__device__ __forceinline__ int kth_interval(uint64_t mk, int k) {
    for (int i = 0; i < k && mk; ++i) mk &= mk - 1;
    return mk ? (int)__builtin_ctzll(mk) : -1;
}
__device__ __forceinline__ uint64_t drop_intervals(uint64_t mk, int c) {
    for (int i = 0; i < c && mk; ++i) mk &= mk - 1;
    return mk;
}

// FP64 gradient sheet of a line, spread over the two transaxial neighbours.
__device__ __forceinline__ void scatter_sheet(const ProjArgs &a, const LineP &L, int nrow, const double *Z) {
    const int rz = a.rz;
    float *Gout = L.axis ? a.G1 : a.G0;
    const int other_stride = ((L.axis ? a.nx : a.ny) + 2 * PADA) * rz;
    if (rz <= (int)blockDim.x) {
        const SheetWalk w = sheet_walk(rz, threadIdx.x);
        if (!w.on) return;
        for (int r = w.r0; r < nrow; r += w.R) {
            const float val = (float)Z[r * rz + w.zp];
            if (val == 0.f) continue;
            spread_cell(Gout, sheet_row(L, L.i_lo + r, other_stride, rz), w.zp, rz, val);
        }
    } else {
        for (int e = threadIdx.x; e < nrow * rz; e += blockDim.x) {
            const float val = (float)Z[e];
            if (val == 0.f) continue;
            const int r = e / rz;
            spread_cell(Gout, sheet_row(L, L.i_lo + r, other_stride, rz), e - r * rz, rz, val);
        }
    }
}

// One line per workgroup, in the order a.order (longest first).  MODE M_GRAD: the
// gradient sheets receive P^T [mult (1 - y / ybar)]; M_OBJ: none.  Both write the
// workgroup's FP64 likelihood to a.partial.
template <int MODE>
__global__ void __launch_bounds__(64 * MAX_WAVES) k_tof_walk(ProjArgs a) {
    constexpr bool NEED_Z = MODE == M_GRAD;
    extern __shared__ float4 smem4[];
    float *smem = reinterpret_cast<float *>(smem4);
    const int lane = threadIdx.x & 63;
    // wave index and wave count are wave-uniform: the unit loop below runs
    // under scalar control flow
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = blockDim.x >> 6;
    const int line = a.order[blockIdx.x];
    const LineP L = a.lines[line];
    const int nrow = L.i_hi - L.i_lo + 1;
    const int rz = a.rz;
    const int nt = a.tof.n_tof;
    // LDS: X sheet (float) | Z sheet (double) | per wave: w4 [rows][4], w1 [rows][e1], cuts
    const int sheet = (a.rows_max * rz + 3) & ~3;
    const int ws = a.ws;  // widest bin window of any interval
    const int e1 = ws > 4 ? ws - 4 : 0;
    float *X = smem;
    double *Z = reinterpret_cast<double *>(smem + sheet);
    float *w4 = smem + (NEED_Z ? 3 : 1) * sheet + wave * walk_wave_floats(a.rows_max, ws, a.tof.n_int);
    float *w1 = w4 + 4 * a.rows_max;
    int *cuts = (int *)(w1 + a.rows_max * e1);
    if (nrow > 0) {
        build_sheet(a, L, nrow, X, rz, threadIdx.x);
        if (NEED_Z)
            for (int e = threadIdx.x; e < nrow * rz; e += blockDim.x) Z[e] = 0.0;
    }
    __syncthreads();

    double kl = 0.0;
    // lane s holds the bin count and first bin of interval s
    const int na_l = lane < a.tof.n_int ? a.tof.na[lane] : 0;
    const int bf_l = lane < a.tof.n_int ? a.tof.bf[lane] : 0;

    // the unit order puts units of the same length in consecutive rounds of a wave,
    // which then fills the table once
    float table_dz2 = -1.f;
    for (int sg = wave; sg < a.n_units; sg += nwaves) {
        const TofUnit S = a.units[a.walk_order[sg]];
        // lanes: plane pl of the unit and chunk ch; a unit of at most 32 planes
        // splits its live intervals over C = 64 / np_pad chunks (np_pad the planes
        // rounded up to a power of two)
        int lg = 0;
        while ((1 << lg) < S.np) ++lg;
        lg = __builtin_amdgcn_readfirstlane(lg);
        const int np_pad = 1 << lg, C = 64 >> lg;
        const bool has = (lane & (np_pad - 1)) < S.np;
        const int p = S.p0 + (has ? (lane & (np_pad - 1)) : 0);
        const PlaneP P = a.planes[p];
        const int64_t lor = (int64_t)line * a.n_planes + p;
        const float len = sqrtf(L.lt2 + S.dz2);
        const float ell = L.vm_um * len;
        int is = 0, ie = -1;
        if (nrow > 0 && has) z_clip<true>(L, P, a.nz, is, ie);
        // this lane's samples in t order: q in [qlo, qhi]
        const int qlo = L.dlam > 0.f ? is - L.i_lo : L.i_hi - ie;
        const int qhi = L.dlam > 0.f ? ie - L.i_lo : L.i_hi - is;

        int cut = 0;
        if (S.dz2 != table_dz2) {
            cut = nrow > 0 ? fill_table(a, L, len, cuts, w4, w1) : 0;
            table_dz2 = S.dz2;
        } else if (nrow > 0 && lane <= a.tof.n_int) {
            cut = cuts[lane];  // kept in the table by the fill
        }
        // padded axial cell of row i: u = zA * i + zB (z + PADZ)
        const float zA = P.zs * L.dlam, zB = fmaf(L.lam0, P.zs, P.zb) + (float)PADZ;
        const float zAf = has ? zA : 0.f, zBf = has ? zB : 0.f, umax = (float)(a.nz + PADZ);
        const int drz = L.dlam > 0.f ? rz : -rz;
        const float dfi = L.dlam > 0.f ? 1.f : -1.f;
        // back-projection predicate: k = q - qlo_b in [0, span]; a lane with
        // no samples gets a base far below every row
        const unsigned span = qlo <= qhi ? (unsigned)(qhi - qlo) : 0u;
        const int qlo_b = qlo <= qhi ? qlo : -(1 << 30);
        const int cut_next = __shfl_down(cut, 1, 64);
        // intervals with bins whose rows meet some lane's sample range
        int qa = qlo <= qhi ? qlo : INT_MAX, qb = qlo <= qhi ? qhi : -1;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            qa = min(qa, __shfl_xor(qa, o, 64));
            qb = max(qb, __shfl_xor(qb, o, 64));
        }
        const bool meets = nrow > 0 && na_l > 0 && max(cut, qa) < min(cut_next, qb + 1);
        const float m = has ? (a.mult ? a.mult[lor] : 1.f) : 0.f;
        const int64_t base = lor * nt;

        // TOF bins in blocks of NT_BLK held in registers (one block unless
        // the geometry has more bins); an interval whose bins straddle two
        // blocks is walked once per block
        for (int b0 = 0; b0 < nt; b0 += NT_BLK) {
            const int nb = min(NT_BLK, nt - b0);
            const uint64_t live_mask = __ballot(meets && bf_l < b0 + NT_BLK && bf_l + na_l > b0);
            float acc[NT_BLK];
#pragma unroll
            for (int b = 0; b < NT_BLK; ++b) acc[b] = 0.f;

            // ---- forward projection ----
            if (C == 1) {
                // every lane walks the same rows of one interval at a time: a scalar loop
                for (uint64_t mk = live_mask; mk; mk &= mk - 1) {
                    const int s = __builtin_amdgcn_readfirstlane(__builtin_ctzll(mk));
                    const int na = __builtin_amdgcn_readlane(na_l, s);
                    const int c0 = __builtin_amdgcn_readlane(cut, s);
                    const int c1 = __builtin_amdgcn_readlane(cut_next, s);
                    const int rel = __builtin_amdgcn_readlane(bf_l, s) - b0;
                    float win[WS_MAX];
#pragma unroll
                    for (int j = 0; j < WS_MAX; ++j) win[j] = 0.f;
                    const int i0 = L.dlam > 0.f ? L.i_lo + c0 : L.i_hi - c0;
                    const float *xr0 = X + (i0 - L.i_lo) * rz;
                    PET_NA_SWITCH(tof_fwd_run, zAf, zBf, umax, xr0, drz, (float)i0, dfi, w4 + 4 * c0, w1 + c0 * e1,
                                  e1, c1 - c0, win)
                    PET_REL_SWITCH(add_window, acc, win, na)
                }
            } else {
                // chunk k = lane >> lg takes all rows of the k-th of the next C live
                // intervals, with the geometry's widest window (the weights past an
                // interval's own bins are zero)
                for (uint64_t mk = live_mask; mk; mk = drop_intervals(mk, C)) {
                    const int s = kth_interval(mk, lane >> lg);
                    const int sc = s < 0 ? 0 : s;
                    // every lane shuffles (a lane-permute reads zero from a lane that
                    // is switched off), then selects
                    const int c0 = __shfl(cut, sc, 64), c1 = __shfl(cut_next, sc, 64);
                    const int nas = __shfl(na_l, sc, 64), bfs = __shfl(bf_l, sc, 64);
                    const int rel = s < 0 ? 0 : bfs - b0;
                    const int nl = s < 0 ? 0 : c1 - c0;
                    float win[WS_MAX];
#pragma unroll
                    for (int j = 0; j < WS_MAX; ++j) win[j] = 0.f;
                    const int i0 = L.dlam > 0.f ? L.i_lo + c0 : L.i_hi - c0;
                    const float *xr0 = X + (i0 - L.i_lo) * rz;
                    {
                        const int na = ws;
                        PET_NA_SWITCH(tof_fwd_run, zAf, zBf, umax, xr0, drz, (float)i0, dfi, w4 + 4 * c0,
                                      w1 + c0 * e1, e1, nl, win)
                    }
                    {
                        const int na = s < 0 ? 0 : nas;
                        PET_REL_SWITCH(add_window, acc, win, na)
                    }
                }
            }
            // the chunks of a plane hold partial sums over their intervals
            for (int o = np_pad; o < 64; o <<= 1) {
#pragma unroll
                for (int b = 0; b < NT_BLK; ++b) acc[b] += __shfl_xor(acc[b], o, 64);
            }

            // ---- likelihood and factors ----
            if (has) {
                const int64_t bb = base + b0;
                float ad[NT_BLK], yv[NT_BLK];
#pragma unroll
                for (int b = 0; b < NT_BLK; ++b) ad[b] = 0.f;
                if (a.add) load_row(a.add, bb, nb, ad);
                load_y_row(a.y, a.y_dtype, bb, nb, yv);
#pragma unroll
                for (int b = 0; b < NT_BLK; ++b) {
                    if (b >= nb) continue;
                    const float ybar = fmaf(m, acc[b] * ell, ad[b]);
                    if (lane < np_pad) kl += kl_term(ybar, yv[b]);
                    // a bin without counts: derivative 1
                    if (NEED_Z)
                        acc[b] = m * (yv[b] != 0.f ? fmaf(-yv[b], __builtin_amdgcn_rcpf(ybar), 1.f) : 1.f) * ell;
                }
            }

            // ---- adjoint into the LDS gradient sheet ----
            if (NEED_Z) {
                if (C == 1) {
                    for (uint64_t mk = live_mask; mk; mk &= mk - 1) {
                        const int s = __builtin_amdgcn_readfirstlane(__builtin_ctzll(mk));
                        const int na = __builtin_amdgcn_readlane(na_l, s);
                        const int c0 = __builtin_amdgcn_readlane(cut, s);
                        const int c1 = __builtin_amdgcn_readlane(cut_next, s);
                        const int rel = __builtin_amdgcn_readlane(bf_l, s) - b0;
                        float win[WS_MAX];
                        PET_REL_SWITCH(get_window, acc, win, na)
                        const int i0 = L.dlam > 0.f ? L.i_lo + c0 : L.i_hi - c0;
                        double *zr0 = Z + (i0 - L.i_lo) * rz;
                        PET_NA_SWITCH(tof_back_run, zA, zB, umax, zr0, drz, (float)i0, dfi, w4 + 4 * c0,
                                      w1 + c0 * e1, e1, c1 - c0, c0 - qlo_b, span, win)
                    }
                } else {
                    // the intervals split over the chunks as in the forward pass
                    for (uint64_t mk = live_mask; mk; mk = drop_intervals(mk, C)) {
                        const int s = kth_interval(mk, lane >> lg);
                        const int sc = s < 0 ? 0 : s;
                        const int c0 = __shfl(cut, sc, 64), c1 = __shfl(cut_next, sc, 64);
                        const int nas = __shfl(na_l, sc, 64), bfs = __shfl(bf_l, sc, 64);
                        const int rel = s < 0 ? 0 : bfs - b0;
                        const int nl = s < 0 ? 0 : c1 - c0;
                        float win[WS_MAX];
                        {
                            const int na = s < 0 ? 0 : nas;
                            PET_REL_SWITCH(get_window, acc, win, na)
                        }
                        const int i0 = L.dlam > 0.f ? L.i_lo + c0 : L.i_hi - c0;
                        double *zr0 = Z + (i0 - L.i_lo) * rz;
                        {
                            const int na = ws;
                            PET_NA_SWITCH(tof_back_run, zA, zB, umax, zr0, drz, (float)i0, dfi, w4 + 4 * c0,
                                          w1 + c0 * e1, e1, nl, c0 - qlo_b, span, win)
                        }
                    }
                }
            }
        }
        // the next unit may overwrite this wave's table
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
    if (NEED_Z && nrow > 0) {
        __syncthreads();
        scatter_sheet(a, L, nrow, Z);
    }
    block_sums(kl, kl, a.partial, false);
}

template <int MODE>
hipError_t launch_walk(const pet_geom_s *g, dim3 grid, const ProjArgs &a, hipStream_t s) {
    const size_t lds = walk_lds_bytes(g, MODE == M_GRAD);
    static size_t granted = 64 * 1024;
    if (lds > granted) {
        hipError_t e = hipFuncSetAttribute((const void *)k_tof_walk<MODE>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
        if (e == hipSuccess) granted = lds;
        (void)hipGetLastError();
    }
    hipLaunchKernelGGL((k_tof_walk<MODE>), grid, dim3(64 * g->walk_waves), lds, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_tof_walk(const pet_geom_s *g, int mode, dim3 grid, const ProjArgs &a, hipStream_t s) {
    return mode == M_GRAD ? launch_walk<M_GRAD>(g, grid, a, s) : launch_walk<M_OBJ>(g, grid, a, s);
}

}  // namespace pet
