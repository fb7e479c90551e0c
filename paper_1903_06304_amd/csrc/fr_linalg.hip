// Element-block-Jacobi preconditioner and Krylov building blocks for gfx950.
//
//  - block assembly: the true diagonal block inv_dtau Gamma + c_time M - dR_e/dq_e (paper Eq.
//    unsteady_pre_discretized_3) from the linearisation packs, entry by entry (fr_assembly.hip), or
//    column by column with seeded tangents where a seed reaches beyond its element's faces
//  - block inversion (fr_invert.hip): the explicit inverse is stored in FP64, FP32 or BF16
//    (round to nearest even), column-major so the apply reads it coalesced
//  - block apply z_e = P_e^-1 r_e: memory-bound GEMV, FP64 accumulation
//  - Krylov reductions: two-stage, fixed-order (deterministic) dot products
#include "fr_internal.hpp"

#include <hip/hip_bf16.h>

namespace {

constexpr int RED_THREADS = 256;
static_assert(MAXV <= RED_THREADS, "the coefficient staging takes one thread per Krylov vector");
constexpr int MAX_GRID = 8192;    // workgroups of the chunk-walking kernels

// case of tile t of a group (binary search over the group's tile prefix); uniform
__device__ __forceinline__ int tile_member(const GroupArgs& ga, int t) {
    int lo = 0, hi = ga.nmem - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ga.pfx[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// z_e = Ainv_e r_e for the elements of one group; state layout [4][E][Np] per case, block row/col
// index v*Np + s.  The columns make four sums, part q those of the columns 4 u + q in ascending order,
// added in order.  Four parts of an element's threads take one each: a load of the element's threads
// covers four columns, consecutive in memory (a column alone is 72 to 800 bytes, no whole lines), and a
// thread's chain of loads is a quarter as long, which is the whole time where the elements do not fill
// the chip.  A thread holds R consecutive rows, one load of 16 bytes (8 in BF16) each column; FP64
// accumulation.
//
// Bound by the read of the blocks.  STREAM: with loads that leave no line in the last-level cache
// (stream_blocks).  One application, us, against one sum and part to an element with ordinary loads:
//     elements         256            2,048          65,536
//     p = 2 BF16   3.6 (4.7)      4.0 (4.8)       30.7 (33.4)
//     p = 3 BF16   3.5 (5.3)      4.6 (6.6)        108 (117)
//     p = 3 FP32   3.4 (5.0)      5.7 (7.4)        195 (220)
//     p = 3 FP64   3.3 (4.5)     11.5 (11.5)       347 (388)
//     p = 4 FP64   4.7 (5.6)     24.8 (24.6)       891 (995; 5.9 TB/s of blocks, a plain read 6.1)
// FULL: FP64 blocks that do fill the chip (apply_as), one row a thread and loads of 8 bytes; at
// p = 4 in one part, whose threads keep the four sums.  us, against two rows and four parts:
//     p = 3   8,192 plain 40.1 (41.3)   65,536 streamed 348 (359)    1,024 plain 6.1 (5.1)
//     p = 4   3,000 plain 34.7 (36.4)   4,096 streamed 54.0 (52.0)   512 plain 7.9 (7.4)
template <class Tin, int R> struct RowPack;
template <> struct RowPack<double, 1> {
    typedef double V;
    __device__ static void expand(V v, double* x) { x[0] = v; }
};
template <> struct RowPack<double, 2> {
    typedef double V __attribute__((ext_vector_type(2)));
    __device__ static void expand(V v, double* x) { x[0] = v.x; x[1] = v.y; }
};
template <> struct RowPack<float, 4> {
    typedef float V __attribute__((ext_vector_type(4)));
    __device__ static void expand(V v, double* x) { x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }
};
template <> struct RowPack<uint16_t, 4> {
    typedef unsigned V __attribute__((ext_vector_type(2)));
    __device__ static void expand(V v, double* x) {
        x[0] = (double)__uint_as_float(v.x << 16);
        x[1] = (double)__uint_as_float(v.x & 0xffff0000u);
        x[2] = (double)__uint_as_float(v.y << 16);
        x[3] = (double)__uint_as_float(v.y & 0xffff0000u);
    }
};

// a workgroup: one element, or as many as 256 threads hold where an element's are fewer than a wave
// or fill their last one badly (p <= 2; FP32 at p = 1 half of them: 32,768 elements 7.5 us, 8.1 with 256)
template <class Tin, int NB, bool FULL = false>
struct ApplyShape {
    static constexpr int R = FULL ? 1 : sizeof(Tin) == 8 ? 2 : 4, SUMS = 4, PARTS = FULL && NB == 100 ? 1 : 4;
    static constexpr int TPE = NB / R, TPT = TPE * PARTS, HOLD = NB == 16 && sizeof(Tin) == 4 ? 128 : 256;
    static constexpr int EPB = NB <= 36 || PARTS == 1 ? HOLD / TPT : 1, threads = EPB * TPT;
    static_assert(NB % R == 0 && NB % SUMS == 0 && threads <= 256, "whole packs, whole quarters");
};

// z_e = D_e^-1 r_e for every element, or, for the Gauss-Seidel sweeps, for the elements of
// one colour only (tiles over that colour, ga.csel): z_e = D_e^-1 (r_e - b_e) (b may be null),
// or z_e -= D_e^-1 r_e (sub).
template <class Tin, int NB, bool STREAM, bool FULL>
__global__ void __launch_bounds__(256)
k_block_apply(GroupArgs ga, const Tin* __restrict__ inv, const double* __restrict__ r, const double* __restrict__ b,
              double* __restrict__ z, int sub, const int* __restrict__ flags, int flag, int cl) {
    using SH = ApplyShape<Tin, NB, FULL>;
    constexpr int Np = NB / 4, R = SH::R, TPE = SH::TPE, EPB = SH::EPB, S = SH::SUMS, Q = NB / S;
    constexpr int PARTS = SH::PARTS, M = S / PARTS;   // M: sums of a thread, those of q = part + PARTS j
    using P = RowPack<Tin, R>;
    __shared__ double rs[EPB][NB + 1];
    __shared__ double sh[EPB][S][NB];
    const int t = blockIdx.x;
    if (t >= ga.ntiles) return;
    const int lo = tile_member(ga, t);
    const int cid = ga.ids[lo];
    if (flags && flags[cid * GI_STRIDE + flag]) return;
    const CaseDev& cd = ga.cases[cid];
    const int el = threadIdx.x / SH::TPT, part = threadIdx.x / TPE % PARTS, r0 = (threadIdx.x % TPE) * R;
    // one colour of the Gauss-Seidel sweeps (ga.csel set): the tiles run over the member's
    // elements of that colour, taken from its colour-sorted element list.  slot: the
    // element's block in the stored inverse (its position in that list in the colour layout)
    int slot = (t - ga.pfx[lo]) * EPB + el;
    bool act = slot < cd.E;
    if (ga.csel) {
        act = slot < ga.csel[2 * lo + 1];
        slot += ga.csel[2 * lo];
    }
    int e = slot;
    if (ga.csel || cl) e = act ? cd.g.corder[slot] : 0;
    if (!cl) slot = e;
    const size_t EN = (size_t)cd.E * Np;
    auto gid = [&](int row) { return cd.off + (row / Np) * EN + (size_t)e * Np + (row % Np); };
    // a row to each part, as far as there are
    static_assert(R <= PARTS, "a part stages and writes one row");
    const bool has_row = act && part < R;
    if (has_row) {
        const size_t g = gid(r0 + part);
        rs[el][r0 + part] = b ? r[g] - b[g] : r[g];
    }
    __syncthreads();
    const Tin* A = inv + cd.boff + (size_t)slot * NB * NB + r0;
    double acc[M][R];
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
        for (int k = 0; k < R; ++k) acc[j][k] = 0.0;
    // a thread's columns in batches whose loads are all issued before any is used
    constexpr int NBAT = (Q * M + 15) / 16, U = (Q + NBAT - 1) / NBAT;
    if (act) {
#pragma unroll
        for (int u0 = 0; u0 < Q; u0 += U) {
            typename P::V raw[U][M];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < M; ++j)
                    if (u0 + u < Q) {
                        const auto* x =
                            reinterpret_cast<const typename P::V*>(A + (size_t)(S * (u0 + u) + part + PARTS * j) * NB);
                        raw[u][j] = STREAM ? __builtin_nontemporal_load(x) : *x;
                    }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < M; ++j)
                    if (u0 + u < Q) {
                        double x[R];
                        P::expand(raw[u][j], x);
                        const double rc = rs[el][S * (u0 + u) + part + PARTS * j];
#pragma unroll
                        for (int k = 0; k < R; ++k) acc[j][k] += x[k] * rc;
                    }
        }
    }
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
        for (int k = 0; k < R; ++k) sh[el][part + PARTS * j][r0 + k] = acc[j][k];
    __syncthreads();
    if (!has_row) return;
    const int row = r0 + part;
    const double v = ((sh[el][0][row] + sh[el][1][row]) + sh[el][2][row]) + sh[el][3][row];
    const size_t g = gid(row);
    if (sub) z[g] -= v;
    else z[g] = v;
}

// ------------------------------------------------------------------ segmented Krylov reductions
// The solver vectors are concatenations of per-case segments; the reductions run over items, ranges
// of entries of one case (Item).  First stage: one partial per item and output; second stage: per
// case, a fixed-order sum over its items (deterministic).  The padding after a case's entries
// belongs to no item: it is neither read nor written, so a non-finite value there (a scaling by a
// non-finite coefficient once produced some) cannot reach a dot product of a later solve.
struct RedArgs {
    const CaseDev* cases;
    const Item* items;
    int nitems;
    const int* flags;        // per-case skip flags or NULL
    int flag;
};

// where a workgroup finds the dot products of the previous launch
struct DotRef {
    const double* part;      // [MAXV][nditem]
    int nditem;
    const int* first;        // first dot item of each case
};

__device__ __forceinline__ bool case_skipped(const RedArgs& ra, int c) {
    return ra.flags && ra.flags[c * GI_STRIDE + ra.flag];
}
__device__ __forceinline__ size_t case_size(const RedArgs& ra, int c) {
    return (size_t)4 * ra.cases[c].E * ra.cases[c].Np;
}

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Sums of eight values over the wave: in three steps each lane hands half of its values to its
// partner and keeps the other half, in three more the last value is summed over eight lanes: 10
// exchanges instead of 48.  The sum of value wave_sum8_index(lane) is returned on the lanes with
// lane % 8 == 0.
__device__ __forceinline__ int wave_sum8_index(int lane) { return ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1); }
__device__ __forceinline__ double wave_sum8(const double* a, int lane) {
    double b[4], c[2];
    const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = (h5 ? a[i + 4] : a[i]) + __shfl_xor(h5 ? a[i] : a[i + 4], 32, 64);
#pragma unroll
    for (int i = 0; i < 2; ++i) c[i] = (h4 ? b[i + 2] : b[i]) + __shfl_xor(h4 ? b[i] : b[i + 2], 16, 64);
    double d = (h3 ? c[1] : c[0]) + __shfl_xor(h3 ? c[0] : c[1], 8, 64);
    d += __shfl_xor(d, 4, 64);
    d += __shfl_xor(d, 2, 64);
    d += __shfl_xor(d, 1, 64);
    return d;
}

// An entry of the basis.  STREAM: with a load that leaves no line in the last-level cache (streamed()).
template <bool STREAM> __device__ __forceinline__ double basis_entry(const double* p) {
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}

// Dot products V_i . w for i in [DB*blockIdx.y, DB*blockIdx.y + DB) ∩ [0, nv) into
// partial[i][item], plus |w|^2 into npart[item] when it is not null (y-block 0 only; mass_only:
// over the first E Np entries of the case).  DB = 8 vectors per pass (16 measured slower: fewer
// workgroups, heavier reduction).
constexpr int DB = 8;
template <bool STREAM>
__global__ void __launch_bounds__(RED_THREADS) k_dots8(RedArgs ra, const double* __restrict__ V, size_t ldv, int nv,
                                                       const double* __restrict__ w, int mass_only,
                                                       double* __restrict__ partial, double* __restrict__ npart) {
    __shared__ double red[RED_THREADS / 64][DB + 1];
    const int i0 = blockIdx.y * DB;
    const int cnt = nv - i0 < DB ? nv - i0 : DB;
    const bool nrm = npart && blockIdx.y == 0;
    const double* Vc = V + (size_t)i0 * ldv;
    const int lane = threadIdx.x % 64, wid = threadIdx.x / 64;
    for (int it = blockIdx.x; it < ra.nitems; it += gridDim.x) {
        const Item im = ra.items[it];
        if (case_skipped(ra, im.c)) continue;
        const size_t end = im.start + im.len;
        size_t lim = end;
        if (mass_only) {
            const CaseDev& cd = ra.cases[im.c];
            const size_t m = cd.off + (size_t)cd.E * cd.Np;
            lim = m < lim ? m : lim;
        }
        double acc[DB];
#pragma unroll
        for (int i = 0; i < DB; ++i) acc[i] = 0.0;
        double nacc = 0.0;
        for (size_t t = im.start + threadIdx.x; t < end; t += RED_THREADS) {
            const double wt = w[t];
            if (cnt > 0) {
                // all rows loaded before any is used (rows past cnt - 1 reload row cnt - 1, unused)
                double x[DB];
#pragma unroll
                for (int i = 0; i < DB; ++i) x[i] = basis_entry<STREAM>(Vc + (size_t)(i < cnt ? i : cnt - 1) * ldv + t);
#pragma unroll
                for (int i = 0; i < DB; ++i)
                    if (i < cnt) acc[i] += x[i] * wt;
            }
            if (nrm && t < lim) nacc += wt * wt;
        }
        __syncthreads();   // red[] of the previous item consumed
        if (cnt > 0) {
            const double v = wave_sum8(acc, lane);
            if (lane % 8 == 0) red[wid][wave_sum8_index(lane)] = v;
        }
        if (nrm) {
            const double v = wave_sum(nacc);
            if (lane == 0) red[wid][DB] = v;
        }
        __syncthreads();
        const int k = threadIdx.x;
        if (k < cnt || (k == DB && nrm)) {
            double v = 0.0;
            for (int q = 0; q < RED_THREADS / 64; ++q) v += red[q][k];
            if (k < DB) partial[(size_t)(i0 + k) * ra.nitems + it] = v;
            else npart[it] = v;
        }
    }
}

// Coefficients of the update that follows a dots launch, per workgroup: cf[i] = h_i s_i with
// h_i = s_i (s_j) (v_i . w); the workgroup of the case's first item stores the h_i.  The dot
// products of a small case (at most SMALL_ITEMS partials each, one round of loads) are summed
// here, those of a larger one were by k_final.  Returns the factor of w.
__device__ __forceinline__ double update_coefs(const RedArgs& ra, const DotRef& dr, const GsRef& g, int c, int nv,
                                               bool owner, double* cf) {
    double* gs = g.gs + (size_t)c * g.stride;
    const double sj = g.first ? gs[g.sc + g.j] : 1.0;
    const int i = threadIdx.x;
    if (i < nv) {
        double d;
        if (is_small(case_size(ra, c))) {
            const int i0 = dr.first[c], n = dr.first[c + 1] - i0;
            const double* p = dr.part + (size_t)i * dr.nditem + i0;
            double x[SMALL_ITEMS];
#pragma unroll
            for (int k = 0; k < SMALL_ITEMS; ++k) x[k] = p[k < n ? k : 0];
            d = 0.0;
#pragma unroll
            for (int k = 0; k < SMALL_ITEMS; ++k)
                if (k < n) d += x[k];
        } else {
            d = gs[g.dt + i];
        }
        const double si = gs[g.sc + i], h = d * si * sj;
        cf[i] = h * si;
        if (owner) gs[g.h + i] = h;
    }
    return sj;
}

// sum_{i0 <= i < i1} cf[i] V_i(t): 16 basis entries loaded before any is used
__device__ __forceinline__ double basis_sum(const double* __restrict__ V, size_t ldv, const double* cf, int i0, int i1,
                                            size_t t) {
    double s = 0.0;
    for (int i = i0; i < i1; i += 16) {
        double x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = V[(size_t)(i + u < i1 ? i + u : i1 - 1) * ldv + t];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (i + u < i1) s += cf[i + u] * x[u];
    }
    return s;
}

// The entries of a small case's update item (64 at most), one per lane, with the vectors shared
// out over the workgroup's waves: every wave's part of sum_i cf[i] V_i, added on wave 0 (valid
// there).  A wave walks a quarter of a serial chain of loads that is the whole cost at these sizes.
__device__ __forceinline__ double split_sum(const double* __restrict__ V, size_t ldv, const double* cf, int nv,
                                            size_t t, bool live, double (*sh)[64]) {
    constexpr int W = RED_THREADS / 64;
    const int lane = threadIdx.x % 64, wid = threadIdx.x / 64, q = (nv + W - 1) / W;
    const int i0 = wid * q < nv ? wid * q : nv, i1 = i0 + q < nv ? i0 + q : nv;
    sh[wid][lane] = live ? basis_sum(V, ldv, cf, i0, i1, t) : 0.0;
    __syncthreads();
    double s = 0.0;
    if (wid == 0)
        for (int k = 0; k < W; ++k) s += sh[k][lane];
    return s;
}

// s_j w, rounded: the kernels that must agree bit for bit may not fuse it into the subtraction that
// follows in one of them and not in the other
__device__ __forceinline__ double scaled(double sj, double w) {
#pragma clang fp contract(off)
    return sj * w;
}

// w_out = (s_j) w_in - sum_{i < nv} h_i s_i V_i, and the partial |w_out|^2 of each item when
// npart is not null
template <bool STREAM>
__global__ void __launch_bounds__(RED_THREADS) k_update(RedArgs ra, DotRef dr, GsRef g, const double* __restrict__ V,
                                                        size_t ldv, int nv, const double* w_in, double* w_out,
                                                        double* __restrict__ npart, int rev) {
    __shared__ double cf[MAXV];
    __shared__ double red[RED_THREADS / 64];
    __shared__ double sh[RED_THREADS / 64][64];
    const int lane = threadIdx.x % 64, wid = threadIdx.x / 64;
    for (int ci = blockIdx.x; ci < ra.nitems; ci += gridDim.x) {
        const int it = rev ? ra.nitems - 1 - ci : ci;   // items last to first (partials by item)
        const Item im = ra.items[it];
        if (case_skipped(ra, im.c)) continue;
        const size_t end = im.start + im.len;
        __syncthreads();   // cf[] / red[] of the previous item consumed
        const double sj = update_coefs(ra, dr, g, im.c, nv, im.start == ra.cases[im.c].off, cf);
        __syncthreads();
        double nacc = 0.0;
        if (npart && is_small(case_size(ra, im.c))) {
            const size_t t = im.start + lane;
            const double s = split_sum(V, ldv, cf, nv, t, t < end, sh);
            if (wid != 0) continue;   // (the next item's first barrier is met by every wave)
            if (t < end) {
                const double wt = sj * w_in[t] - s;
                w_out[t] = wt;
                nacc = wt * wt;
            }
            nacc = wave_sum(nacc);
            if (lane == 0) npart[it] = nacc;
            continue;
        }
        for (size_t t = im.start + threadIdx.x; t < end; t += RED_THREADS) {
            double wt = scaled(sj, w_in[t]);
            int i = 0;
            // 16 basis entries loaded before any is used, summed in the groups of four below
            for (; i + 16 <= nv; i += 16) {
                double x[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) x[u] = basis_entry<STREAM>(V + (size_t)(i + u) * ldv + t);
#pragma unroll
                for (int u = 0; u < 16; u += 4)
                    wt -= cf[i + u] * x[u] + cf[i + u + 1] * x[u + 1] + cf[i + u + 2] * x[u + 2] + cf[i + u + 3] * x[u + 3];
            }
            for (; i + 4 <= nv; i += 4) {
                double x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = basis_entry<STREAM>(V + (size_t)(i + u) * ldv + t);
                wt -= cf[i] * x[0] + cf[i + 1] * x[1] + cf[i + 2] * x[2] + cf[i + 3] * x[3];
            }
            for (; i < nv; ++i) wt -= cf[i] * basis_entry<STREAM>(V + (size_t)i * ldv + t);
            w_out[t] = wt;
            nacc += wt * wt;
        }
        if (!npart) continue;
        nacc = wave_sum(nacc);
        if (lane == 0) red[wid] = nacc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double v = 0.0;
            for (int q = 0; q < RED_THREADS / 64; ++q) v += red[q];
            npart[it] = v;
        }
    }
}

// The re-orthogonalising pass of classical Gram-Schmidt applied twice, in one read of the basis:
// w_out as k_update and the partial dots V_k . w_out, k < nv, of each dot item (as k_dots8 on
// w_out), from the basis entries already loaded for the update.  The update's grouping and the
// reductions' order are those of the two kernels, so the results are theirs bit for bit.  NV bounds
// nv.
template <int NV, bool STREAM>
__global__ void __launch_bounds__(RED_THREADS) k_update_dots(RedArgs ra, DotRef dr, GsRef g,
                                                             const double* __restrict__ V, size_t ldv, int nv,
                                                             const double* w_in, double* w_out,
                                                             double* __restrict__ partial, int rev) {
    __shared__ double cf[NV];
    __shared__ double red[RED_THREADS / 64][NV];
    const int lane = threadIdx.x % 64, wid = threadIdx.x / 64;
    for (int ci = blockIdx.x; ci < ra.nitems; ci += gridDim.x) {
        const int it = rev ? ra.nitems - 1 - ci : ci;   // items last to first (partials by item)
        const Item im = ra.items[it];
        if (case_skipped(ra, im.c)) continue;
        const size_t end = im.start + im.len;
        __syncthreads();   // cf[] / red[] of the previous item consumed
        const double sj = update_coefs(ra, dr, g, im.c, nv, im.start == ra.cases[im.c].off, cf);
        if ((int)threadIdx.x >= nv && (int)threadIdx.x < NV) cf[threadIdx.x] = 0.0;
        __syncthreads();
        double acc[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[k] = 0.0;
        for (size_t t = im.start + threadIdx.x; t < end; t += RED_THREADS) {
            // all rows loaded before any is used (rows past nv - 1 reload row nv - 1, unused)
            double x[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) x[k] = basis_entry<STREAM>(V + (size_t)(k < nv ? k : nv - 1) * ldv + t);
            double wt = scaled(sj, w_in[t]);
            const int n4 = nv & ~3;
#pragma unroll
            for (int k = 0; k < NV; k += 4)
                if (k < n4) wt -= cf[k] * x[k] + cf[k + 1] * x[k + 1] + cf[k + 2] * x[k + 2] + cf[k + 3] * x[k + 3];
#pragma unroll
            for (int k = 0; k < NV; ++k)
                if (k >= n4 && k < nv) wt -= cf[k] * x[k];
            w_out[t] = wt;
#pragma unroll
            for (int k = 0; k < NV; ++k)
                if (k < nv) acc[k] += x[k] * wt;
        }
#pragma unroll
        for (int k = 0; k < NV; k += 8) {
            if (k >= nv) continue;
            const double v = wave_sum8(acc + k, lane);
            if (lane % 8 == 0) red[wid][k + wave_sum8_index(lane)] = v;
        }
        __syncthreads();
        const int k = threadIdx.x;
        if (k < nv) {
            double v = 0.0;
            for (int q = 0; q < RED_THREADS / 64; ++q) v += red[q][k];
            partial[(size_t)k * ra.nitems + it] = v;
        }
    }
}

// out = sum_{i < cyc_c} y_c[i] V_i
__global__ void __launch_bounds__(RED_THREADS) k_combine(RedArgs ra, const double* __restrict__ V, size_t ldv,
                                                         const double* gs, int stride, int yfield,
                                                         double* __restrict__ out) {
    __shared__ double y[MAXV];
    __shared__ double sh[RED_THREADS / 64][64];
    const int lane = threadIdx.x % 64, wid = threadIdx.x / 64;
    for (int it = blockIdx.x; it < ra.nitems; it += gridDim.x) {
        const Item im = ra.items[it];
        if (case_skipped(ra, im.c)) continue;
        const int nv = ra.flags[im.c * GI_STRIDE + GI_CYC];
        const size_t end = im.start + im.len;
        __syncthreads();
        if ((int)threadIdx.x < nv) y[threadIdx.x] = gs[(size_t)im.c * stride + yfield + threadIdx.x];
        __syncthreads();
        if (is_small(case_size(ra, im.c))) {
            const size_t t = im.start + lane;
            const double s = split_sum(V, ldv, y, nv, t, t < end, sh);
            if (wid == 0 && t < end) out[t] = s;
            continue;
        }
        for (size_t t = im.start + threadIdx.x; t < end; t += RED_THREADS) out[t] = basis_sum(V, ldv, y, 0, nv, t);
    }
}

// dt_c[i] = sum over the dot items of case c of part[i][item], for the cases that are not small;
// grid (ncase, nv)
__device__ __forceinline__ double items_sum(const double* __restrict__ p, int i0, int i1, double* red) {
    double v = 0.0;
    for (int b = i0 + threadIdx.x; b < i1; b += 256) v += p[b];
    v = wave_sum(v);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}
__global__ void __launch_bounds__(256) k_final(RedArgs ra, DotRef dr, GsRef g) {
    __shared__ double red[4];
    const int c = blockIdx.x, i = blockIdx.y;
    if (case_skipped(ra, c) || is_small(case_size(ra, c))) return;
    const double v = items_sum(dr.part + (size_t)i * dr.nditem, dr.first[c], dr.first[c + 1], red);
    if (threadIdx.x == 0) g.gs[(size_t)c * g.stride + g.dt + i] = v;
}
// out_c = sum over the items of case c of npart[item]
__global__ void __launch_bounds__(256) k_final_norm(RedArgs ra, const double* __restrict__ npart,
                                                    const int* __restrict__ first, double* __restrict__ out,
                                                    int ostride) {
    __shared__ double red[4];
    const int c = blockIdx.x;
    if (case_skipped(ra, c)) return;
    const double v = items_sum(npart, first[c], first[c + 1], red);
    if (threadIdx.x == 0) out[(size_t)c * ostride] = v;
}

// ------------------------------------------------------------------ pointwise physics per case
// The points of every case, 256 to a workgroup: chunk ch, part sub of it.  Point t of case c covers
// entries v * E Np + t, v = 0..3, so the chunks past the first variable's have none.
struct ChunkArgs {
    const CaseDev* cases;
    const int* chunk_case;   // [nchunks]
    int nchunks;
    const int* flags;        // per-case skip flags or NULL
    int flag;
};
#define FR_POINT_LOOP(ca, ...)                                                                  \
    for (long long w_ = blockIdx.x; w_ < (long long)(ca).nchunks * (CHUNK / 256); w_ += gridDim.x) { \
        const int ch = (int)(w_ / (CHUNK / 256)), sub = (int)(w_ % (CHUNK / 256));               \
        const int c = (ca).chunk_case[ch];                                                       \
        if ((ca).flags && (ca).flags[c * GI_STRIDE + (ca).flag]) continue;                       \
        const CaseDev& cd = (ca).cases[c];                                                       \
        const size_t EN = (size_t)cd.E * cd.Np;                                                  \
        const size_t t = (size_t)ch * CHUNK - cd.off + (size_t)sub * 256 + threadIdx.x;          \
        if (t < EN) {                                                                            \
            const size_t base = cd.off + t;                                                      \
            __VA_ARGS__                                                                          \
        }                                                                                        \
    }

// q^c of the state
__global__ void k_cons(ChunkArgs ca, const double* __restrict__ q, double* __restrict__ Qc) {
    FR_POINT_LOOP(ca, {
        double qs[4], qc[4];
        for (int v = 0; v < 4; ++v) qs[v] = q[base + v * EN];
        fr_cons(cd.pc, qs, qc);
        for (int v = 0; v < 4; ++v) Qc[base + v * EN] = qc[v];
    })
}

// b = R - (a0 q^c(q) + a1 Q^n + a2 Q^{n-1}) / dt with the case's BDF coefficients
__global__ void k_bdf_rhs(ChunkArgs ca, const CaseStep* __restrict__ st, const double* __restrict__ q,
                          const double* __restrict__ Qn, const double* __restrict__ Qnm1, const double* __restrict__ R,
                          double* __restrict__ b) {
    FR_POINT_LOOP(ca, {
        const CaseStep& cs = st[c];
        double qs[4], qc[4];
        for (int v = 0; v < 4; ++v) qs[v] = q[base + v * EN];
        fr_cons(cd.pc, qs, qc);
        for (int v = 0; v < 4; ++v) {
            double acc = cs.a0 * qc[v] + cs.a1 * Qn[base + v * EN];
            if (cs.has_nm1) acc += cs.a2 * Qnm1[base + v * EN];
            b[base + v * EN] = R[base + v * EN] - acc * cs.inv_dt;
        }
    })
}

// q^c in place for the cases with a q^{n-1}
__global__ void k_cons_nm1(ChunkArgs ca, const CaseStep* __restrict__ st, double* __restrict__ buf) {
    FR_POINT_LOOP(ca, {
        if (st[c].has_nm1) {
            double qs[4], qc[4];
            for (int v = 0; v < 4; ++v) qs[v] = buf[base + v * EN];
            fr_cons(cd.pc, qs, qc);
            for (int v = 0; v < 4; ++v) buf[base + v * EN] = qc[v];
        }
    })
}

ChunkArgs chunk_args(const Solver& sv, const int* flags, int flag) {
    return ChunkArgs{sv.d_cases, sv.d_chunk_case, sv.nchunks, flags, flag};
}

unsigned point_grid(const Solver& sv) {
    const long long g = (long long)sv.nchunks * (CHUNK / 256);
    return (unsigned)(g < MAX_GRID ? g : MAX_GRID);
}

RedArgs dot_args(const Solver& sv, const int* flags, int flag) {
    return RedArgs{sv.d_cases, sv.d_ditem, sv.nditem, flags, flag};
}
RedArgs upd_args(const Solver& sv, const int* flags, int flag) {
    return RedArgs{sv.d_cases, sv.d_uitem, sv.nuitem, flags, flag};
}
unsigned item_grid(int nitems) { return (unsigned)(nitems < MAX_GRID ? nitems : MAX_GRID); }

// the tiles of a group at a tile width; color >= 0: the tiles over the members' elements of
// that colour (pfx null when a table is missing)
GroupArgs group_args(const Solver& sv, const Group& gr, int epb, int color = -1) {
    GroupArgs ga;
    ga.cases = sv.d_cases;
    ga.ids = gr.d_ids;
    ga.pfx = gr.tile_pfx(epb);
    ga.nmem = (int)gr.ids.size();
    ga.ntiles = gr.ntiles(epb);
    ga.xcd = 0;
    if (color >= 0) {
        const Group::ColorTiles* ct = gr.color_tiles(epb, color);
        ga.pfx = ct ? ct->d_pfx : nullptr;
        ga.ntiles = ct ? ct->ntiles : 0;
        ga.csel = ct ? ct->d_csel : nullptr;
    }
    return ga;
}

}  // namespace

// ----------------------------------------------------------------------------- launchers
fr_status launch_block_assembly(Solver& sv, const double* q, const KArgs& base, hipStream_t s) {
    PhaseRange range("lmfr: block assembly (enqueue)");
    if (!base.fpack || !base.spack) { fr_set_error("block assembly without packs"); return FR_EINVAL; }
    KArgs a = base;
    a.q = q; a.v = nullptr; a.out = sv.d_blk; a.out2 = nullptr;
    for (const Group& gr : sv.groups) {
        if (direct_assembly(gr)) {
            FR_TRY(launch_direct_assembly(sv, gr, a, s));
            continue;
        }
        // meshes with boundary faces or self-neighbours: the seeded columns of every element's block
        FR_TRY(launch_fused(sv, gr, MODE_LINBLK, a, gr.tune[MODE_LINBLK], s));
    }
    return FR_OK;
}

// explicit inverse of every element block (fr_invert.hip)
static fr_status invert_all(Solver& sv, int prec, const int* flags, hipStream_t s) {
    for (const Group& gr : sv.groups) {
        GroupArgs ga = group_args(sv, gr, 1);
        if (!ga.pfx) { fr_set_error("tile prefix missing"); return FR_EINVAL; }
        FR_TRY(launch_block_invert_group(sv, gr.p, ga, prec, flags, s));
    }
    return FR_OK;
}

fr_status launch_block_invert(Solver& sv, int prec, const int* flags, hipStream_t s) {
    PhaseRange range("lmfr: block inversion (enqueue)");
    if (prec < FR_FP64 || prec > FR_BF16) { fr_set_error("unknown precision"); return FR_EINVAL; }
    // the Gauss-Seidel sweeps apply one colour at a time: colour-sorted blocks keep each
    // colour's reads contiguous (every other block of the element order reads at about half
    // the bandwidth)
    sv.inv_colour = sv.precond != 0;
    FR_TRY(invert_all(sv, prec, flags, s));
    sv.inv_prec = prec;
    return FR_OK;
}

// orders whose FP64 blocks have a form for launches that fill the chip
constexpr bool full_order(int nb) { return nb >= 64; }

// tile widths (elements per workgroup) of the block apply
template <int NB> static std::vector<int> apply_widths() {
    return {ApplyShape<double, NB>::EPB, ApplyShape<float, NB>::EPB, ApplyShape<uint16_t, NB>::EPB,
            ApplyShape<double, NB, full_order(NB)>::EPB};
}
std::vector<int> block_apply_widths(int p) {
    switch (p) {
        case 1: return apply_widths<16>();
        case 2: return apply_widths<36>();
        case 3: return apply_widths<64>();
    }
    return apply_widths<100>();
}

// size of the last-level cache
constexpr size_t LLC_BYTES = (size_t)256 << 20;
// Blocks and Krylov basis are each read once or twice an iteration; together beyond the cache they
// only evict each other and the smaller vectors and packs, so the blocks are then streamed.  m: restart
// length of the solve the apply belongs to (0: none, no basis).  Whole
// BDF2 steps, ms, streamed (plain): p = 3 FP32, blocks and basis 268 + 260 MB 19.2 (20.5); BF16
// 134 + 260 MB 16.6 (16.9); FP32 151 + 146 MB 13.0 (13.1); p = 4 FP64 328 + 101 MB 18.9 (20.8); and
// below the line 184 + 57 MB 13.7 (13.1), 134 + 65 MB 9.8 (9.7).
static bool stream_blocks(const Solver& sv, size_t entry, int m) {
    const size_t basis = m > 0 ? (size_t)(m + 1) * sv.Ntot * sizeof(double) : 0;
    return sv.Btot * entry + basis > LLC_BYTES;
}

struct ApplyArgs {
    const double* r;
    const double* b;
    double* z;
    int color;
    int sub;
    int m;
    const int* flags;
    int flag;
};

template <class Tin, int NB, bool FULL>
static fr_status apply_form(const Solver& sv, const GroupArgs& ga, bool stream, const ApplyArgs& x, hipStream_t s) {
    if (!ga.pfx) { fr_set_error("tile prefix missing"); return FR_EINVAL; }
    if (ga.ntiles == 0) return FR_OK;
    auto kernel = stream ? k_block_apply<Tin, NB, true, FULL> : k_block_apply<Tin, NB, false, FULL>;
    hipLaunchKernelGGL(kernel, dim3(ga.ntiles), dim3(ApplyShape<Tin, NB, FULL>::threads), 0, s, ga,
                       (const Tin*)sv.d_inv, x.r, x.b, x.z, x.sub, x.flags, x.flag, sv.inv_colour ? 1 : 0);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

template <class Tin, int NB>
static fr_status apply_as(const Solver& sv, const Group& gr, const ApplyArgs& x, hipStream_t s) {
    const bool stream = stream_blocks(sv, sizeof(Tin), x.m);
    const GroupArgs ga = group_args(sv, gr, ApplyShape<Tin, NB>::EPB, x.color);
    if constexpr (sizeof(Tin) == 8 && full_order(NB)) {
        // from about eight elements a compute unit on (a tile of the other form holds one); at p = 4
        // streamed loads want the wider ones (times at the kernel)
        static_assert(ApplyShape<Tin, NB>::EPB == 1, "tiles count elements");
        if (ga.ntiles >= 2048 && !(NB == 100 && stream))
            return apply_form<Tin, NB, true>(sv, group_args(sv, gr, ApplyShape<Tin, NB, true>::EPB, x.color), stream, x, s);
    }
    return apply_form<Tin, NB, false>(sv, ga, stream, x, s);
}

template <class Tin>
static fr_status apply_p(const Solver& sv, const Group& gr, const ApplyArgs& x, hipStream_t s) {
    switch (gr.p) {
        case 1: return apply_as<Tin, 16>(sv, gr, x, s);
        case 2: return apply_as<Tin, 36>(sv, gr, x, s);
        case 3: return apply_as<Tin, 64>(sv, gr, x, s);
        case 4: return apply_as<Tin, 100>(sv, gr, x, s);
    }
    fr_set_error("order outside 1..4");
    return FR_EUNSUPPORTED;
}

fr_status launch_block_apply(const Solver& sv, const double* r, const double* b, double* z, int color, bool sub,
                             int m, const int* flags, int flag, hipStream_t s, int only) {
    const ApplyArgs x{r, b, z, color, sub ? 1 : 0, m, flags, flag};
    for (const Group& gr : sv.groups) {
        if (only >= 0 && &gr != &sv.groups[only]) continue;
        switch (sv.inv_prec) {
            case FR_FP64: FR_TRY(apply_p<double>(sv, gr, x, s)); break;
            case FR_FP32: FR_TRY(apply_p<float>(sv, gr, x, s)); break;
            case FR_BF16: FR_TRY(apply_p<uint16_t>(sv, gr, x, s)); break;
            default: fr_set_error("preconditioner not factored"); return FR_EINVAL;
        }
    }
    return FR_OK;
}

// Symmetric block Gauss-Seidel over the elements in colour order, P = (D + L) D^-1 (D + U)
// with L / U the couplings of the Newton operator A to elements of lower / higher colour
// (elements of one colour never share a face, so A restricted to a colour is D):
//   forward   z_k = D_k^-1 (r_k - [A z_{<k}]_k),   k = 0 .. K-1
//   backward  z_k -= D_k^-1 [A z_{>k}]_k,          k = K-2 .. 0
// where z_{<k} (z_{>k}) is z on the colours below (above) k and zero elsewhere.  Costs
// 2 (K - 1) operator applications and about 1.5 block-apply passes per application.
// Forward block Gauss-Seidel (option value 2), P = D + L, is the forward sweep alone:
// K - 1 operator applications over one colour each and one block-apply pass.
fr_status precond_apply(Solver& sv, const double* r, double* z, const KArgs& op, int m, const int* flags, int flag,
                        hipStream_t s, int only) {
    if (sv.precond == 0) return launch_block_apply(sv, r, nullptr, z, -1, false, m, flags, flag, s, only);
    FR_TRY(dalloc(&sv.d_gst, sv.Ntot));
    const int K = sv.ncolors;
    KArgs a = op;
    a.v = z;
    a.out = sv.d_gst;
    a.flags = flags;
    a.flag = flag;
    // each coupling pass computes the rows of the colour that its block apply updates, from z
    // on the elements of lower colours (forward sweep) or of higher colours (backward sweep)
    for (int k = 0; k < K; ++k) {
        if (k > 0) {
            a.csweep = 1 + k;
            a.cbelow = 1;
            FR_TRY(solver_fused(sv, MODE_LIN, a, s, only));
        }
        FR_TRY(launch_block_apply(sv, r, k > 0 ? sv.d_gst : nullptr, z, k, false, m, flags, flag, s, only));
    }
    for (int k = K - 2; k >= 0 && sv.precond == 1; --k) {
        a.csweep = 1 + k;
        a.cbelow = 0;
        FR_TRY(solver_fused(sv, MODE_LIN, a, s, only));
        FR_TRY(launch_block_apply(sv, sv.d_gst, nullptr, z, k, true, m, flags, flag, s, only));
    }
    return FR_OK;
}

static fr_status too_many(int nv) {
    if (nv <= MAXV - 1) return FR_OK;
    fr_set_error("too many Krylov vectors");
    return FR_EINVAL;
}

// second stage of the dots of partial set `set`, where a case needs one
static fr_status final_dots(const Solver& sv, int nv, const GsRef& g, int set, const int* flags, int flag,
                            hipStream_t s) {
    if (sv.all_small) return FR_OK;
    const DotRef dr{part_dots(sv, set), sv.nditem, sv.d_dfirst};
    hipLaunchKernelGGL(k_final, dim3(sv.n, nv), dim3(256), 0, s, dot_args(sv, flags, flag), dr, g);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

// a launch's basis vectors exceed the cache: nothing of them is left for the next launch, and loads
// that leave no line spare what the cache holds of the blocks, packs and other vectors.  BDF2 steps of
// 256 x 256 elements, 30 Krylov vectors: p = 4 FP64 237.0 -> 232.5 ms, p = 3 BF16 39.6 -> 38.5 ms; below
// the line a batch of 12 cases, 46.0 ms plain, 46.5 streamed.
static bool streamed(int nv, size_t ldv) { return nv * ldv * sizeof(double) > LLC_BYTES; }

fr_status la_dots(const Solver& sv, const double* V, size_t ldv, int nv, const double* w, const GsRef& g, int set,
                  const int* flags, int flag, hipStream_t s) {
    FR_TRY(too_many(nv));
    hipLaunchKernelGGL(streamed(nv, ldv) ? k_dots8<true> : k_dots8<false>, dim3(item_grid(sv.nditem), (nv + DB - 1) / DB), dim3(RED_THREADS), 0, s,
                       dot_args(sv, flags, flag), V, ldv, nv, w, 0, part_dots(sv, set), (double*)nullptr);
    FR_HIP(hipGetLastError());
    return final_dots(sv, nv, g, set, flags, flag, s);
}

fr_status la_update(const Solver& sv, const double* V, size_t ldv, int nv, const double* w_in, double* w_out,
                    bool want_norm, const GsRef& g, int set, const int* flags, int flag, hipStream_t s, bool rev) {
    FR_TRY(too_many(nv));
    const DotRef dr{part_dots(sv, set), sv.nditem, sv.d_dfirst};
    hipLaunchKernelGGL(streamed(nv, ldv) ? k_update<true> : k_update<false>, dim3(item_grid(sv.nuitem)), dim3(RED_THREADS), 0, s, upd_args(sv, flags, flag), dr, g,
                       V, ldv, nv, w_in, w_out, want_norm ? part_norm(sv) : nullptr, rev ? 1 : 0);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

fr_status la_update_dots(const Solver& sv, const double* V, size_t ldv, int nv, const double* w_in, double* w_out,
                         const GsRef& g, int set, const int* flags, int flag, hipStream_t s, bool rev) {
    if (nv > 32) { fr_set_error("update with dots: at most 32 vectors"); return FR_EINVAL; }
    const DotRef dr{part_dots(sv, set), sv.nditem, sv.d_dfirst};
    const RedArgs ra = dot_args(sv, flags, flag);
    const dim3 grid(item_grid(sv.nditem)), block(RED_THREADS);
    double* out = part_dots(sv, 1 - set);
    const bool st = streamed(nv, ldv);
    if (nv <= 8)
        hipLaunchKernelGGL((st ? k_update_dots<8, true> : k_update_dots<8, false>), grid, block, 0, s, ra, dr, g, V, ldv, nv, w_in, w_out, out, rev ? 1 : 0);
    else if (nv <= 16)
        hipLaunchKernelGGL((st ? k_update_dots<16, true> : k_update_dots<16, false>), grid, block, 0, s, ra, dr, g, V, ldv, nv, w_in, w_out, out, rev ? 1 : 0);
    else
        hipLaunchKernelGGL((st ? k_update_dots<32, true> : k_update_dots<32, false>), grid, block, 0, s, ra, dr, g, V, ldv, nv, w_in, w_out, out, rev ? 1 : 0);
    FR_HIP(hipGetLastError());
    return final_dots(sv, nv, g, 1 - set, flags, flag, s);
}

fr_status la_combine(const Solver& sv, const double* V, size_t ldv, const double* gs, int stride, int yfield,
                     double* out, const int* flags, int flag, hipStream_t s) {
    hipLaunchKernelGGL(k_combine, dim3(item_grid(sv.nuitem)), dim3(RED_THREADS), 0, s, upd_args(sv, flags, flag), V,
                       ldv, gs, stride, yfield, out);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

fr_status la_norm(const Solver& sv, const double* w, bool mass_only, double* out, int ostride, const int* flags,
                  int flag, hipStream_t s) {
    const RedArgs ra = dot_args(sv, flags, flag);
    hipLaunchKernelGGL(k_dots8<false>, dim3(item_grid(sv.nditem)), dim3(RED_THREADS), 0, s, ra, w, (size_t)0, 0, w,
                       mass_only ? 1 : 0, part_dots(sv, 0), part_norm(sv));
    FR_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_final_norm, dim3(sv.n), dim3(256), 0, s, ra, part_norm(sv), sv.d_dfirst, out, ostride);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

fr_status launch_cons(const Solver& sv, const double* q, double* Qc, const int* flags, hipStream_t s) {
    hipLaunchKernelGGL(k_cons, dim3(point_grid(sv)), dim3(256), 0, s, chunk_args(sv, flags, GI_NDONE), q, Qc);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

fr_status launch_bdf_rhs(const Solver& sv, const double* q, const double* Qn, const double* Qnm1, const double* R,
                         double* b, const int* flags, hipStream_t s) {
    hipLaunchKernelGGL(k_bdf_rhs, dim3(point_grid(sv)), dim3(256), 0, s, chunk_args(sv, flags, GI_NDONE), sv.d_step, q,
                       Qn, Qnm1, R, b);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

fr_status launch_cons_nm1(const Solver& sv, double* buf, hipStream_t s) {
    hipLaunchKernelGGL(k_cons_nm1, dim3(point_grid(sv)), dim3(256), 0, s, chunk_args(sv, nullptr, 0), sv.d_step, buf);
    FR_HIP(hipGetLastError());
    return FR_OK;
}
