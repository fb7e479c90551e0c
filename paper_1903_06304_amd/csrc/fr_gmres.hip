// Restarted, right-preconditioned FP64 GMRES(m) and the BDF2 dual-time Newton loop for
// every case of a solver at once, with the small dense state of each case (Hessenberg
// matrix, Givens rotations, least-squares right-hand side, counters) on the device.
//
// One restart cycle is a fixed sequence of launches over all cases:
//   cycle init (per case: idle test, g = beta e1, s_0 = 1 / beta) |
//   m x [ z = P^-1 v_j ; w = A z ; classical Gram-Schmidt (2 streaming passes over the basis, or
//         4 when re-orthogonalised: option "gram_schmidt" = 2), its result is v_{j+1} ;
//         Givens update of column j and of g, convergence test, s_{j+1} = 1 / h_{j+1,j} ] |
//   y = H^-1 g ; x += P^-1 (V y) ; r = b - A x (into v_0) ; beta = |r|
// The basis is stored unnormalised, V_i = s_i v_i with the scale s_i in the case's state: the
// operator is linear, so the scales enter the dot products' and the update's coefficients, and no
// pass over the vectors normalises one (k_scale_case took 9.7 us of a 0.50 ms iteration at p = 3 on
// 256 x 256 elements, and one launch of seven at every size).
// Per-case flags decide which cases a launch touches: a case whose Arnoldi process has
// stopped (|g_{j+1}| <= tol |b|, breakdown, iteration cap) is skipped by the rest of the
// cycle's Arnoldi launches; a case that did not start the cycle is skipped by its update
// too.  The sequence is captured into hipGraphs once and replayed: the Arnoldi steps in segments,
// then the cycle's end.  The host keeps one segment queued behind the one that runs and
// stops launching them when a segment that has ended reports every case stopped; it synchronises
// once per cycle to read one "needs another cycle" flag per case.  The Newton loop (paper Sec. 3.2)
// keeps per-case convergence on the device as well and synchronises once per Newton iteration.
#include <cmath>
#include <cstring>

#include "fr_internal.hpp"

namespace {

// layout of one case's GMRES state (doubles) for restart length m
struct GsLayout {
    int m, H, CS, SN, G, Y, H1, H2, DT, SC, NRM, BN, BETA, total;   // H: column by column, m + 1 rows each
    __host__ __device__ explicit GsLayout(int m_) : m(m_) {
        H = 0;
        CS = H + (m + 1) * m;
        SN = CS + m;
        G = SN + m;
        Y = G + m + 1;
        H1 = Y + m;
        H2 = H1 + MAXV;
        DT = H2 + MAXV;
        SC = DT + MAXV;
        NRM = SC + m + 1;
        BN = NRM + 1;
        BETA = BN + 1;
        total = ((BETA + 1 + 7) / 8) * 8;
    }
};

struct Ctl {
    double* gs;
    int gs_stride;
    int* gi;
    CaseStep* step;   // written only by the Newton check (SER)
    double* sum;
    int n;
};

__device__ __forceinline__ int case_index() { return blockIdx.x * blockDim.x + threadIdx.x; }

// start of a solve: counters and flags of the solve
__global__ void k_gm_start(Ctl k, int maxit) {
    const int c = case_index();
    if (c >= k.n) return;
    int* gi = k.gi + c * GI_STRIDE;
    gi[GI_TOTAL] = 0;
    gi[GI_CYC] = 0;
    gi[GI_MAXIT] = maxit;
    gi[GI_DONE] = 1;
    gi[GI_IDLE] = 1;
}

// beta = bn = |b|
__global__ void k_gm_norm0(Ctl k, int m) {
    const int c = case_index();
    if (c >= k.n) return;
    if (k.gi[c * GI_STRIDE + GI_NDONE]) return;
    const GsLayout L(m);
    double* gs = k.gs + (size_t)c * k.gs_stride;
    const double b = sqrt(gs[L.NRM]);
    gs[L.BN] = b;
    gs[L.BETA] = b;
}

// the case's test for another cycle (also used by the host through the summary)
__device__ __forceinline__ bool wants_cycle(const int* gi, double beta, double bn, double tol) {
    return !gi[GI_NDONE] && isfinite(beta) && beta > 0.0 && beta > tol * bn && gi[GI_TOTAL] < gi[GI_MAXIT];
}

// per case: does it take part in this cycle?  g = beta e1, scale of V_0
__global__ void k_cycle_init(Ctl k, int m) {
    const int c = case_index();
    if (c >= k.n) return;
    const GsLayout L(m);
    double* gs = k.gs + (size_t)c * k.gs_stride;
    int* gi = k.gi + c * GI_STRIDE;
    const double beta = gs[L.BETA], bn = gs[L.BN];
    const bool run = wants_cycle(gi, beta, bn, k.step[c].tol_res);
    gi[GI_IDLE] = run ? 0 : 1;
    gi[GI_DONE] = run ? 0 : 1;
    gi[GI_CYC] = 0;
    if (!run) return;
    for (int i = 0; i <= m; ++i) gs[L.G + i] = 0.0;
    gs[L.G] = beta;
    gs[L.SC] = 1.0 / beta;
}

// One workgroup of 256 threads per case: the second stage of |v_{j+1}|^2 (the update pass's item
// partials), then column j of H: the Gram-Schmidt coefficients h_0..h_j (one or two passes summed)
// through the previous rotations, the new rotation, g and the convergence test.  The rotations are a
// serial chain on thread 0; its operands are staged in LDS by all threads, so that the chain waits
// for one round of loads and not for one every eight rows.
__global__ void __launch_bounds__(256) k_norm_givens(Ctl k, const int* __restrict__ ufirst,
                                                     const double* __restrict__ npart, int j, int m, int passes) {
    __shared__ double red[4];
    __shared__ double h[MAXV + 8], cs[MAXV + 8], sn[MAXV + 8];
    const int c = blockIdx.x, tid = threadIdx.x;
    int* gi = k.gi + c * GI_STRIDE;
    if (gi[GI_DONE]) return;   // uniform per workgroup
    const GsLayout L(m);
    double* gs = k.gs + (size_t)c * k.gs_stride;
    if (tid <= j) {
        h[tid] = passes == 2 ? gs[L.H1 + tid] + gs[L.H2 + tid] : gs[L.H1 + tid];
        cs[tid] = gs[L.CS + tid];   // (row j is not used)
        sn[tid] = gs[L.SN + tid];
    }
    double v = 0.0;
    for (int b = ufirst[c] + tid; b < ufirst[c + 1]; b += 256) v += npart[b];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (tid % 64 == 0) red[tid / 64] = v;
    __syncthreads();
    if (tid == 0) {
        const double hn = sqrt(red[0] + red[1] + red[2] + red[3]);
        // rows 0..j-1: the running row-i entry a and the next row's h through rotation i
        double a = h[0];
        for (int i0 = 0; i0 < j; i0 += 8) {
            double h8[8], c8[8], s8[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) { h8[t] = h[i0 + t + 1]; c8[t] = cs[i0 + t]; s8[t] = sn[i0 + t]; }
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                if (i0 + t < j) {
                    h[i0 + t] = c8[t] * a + s8[t] * h8[t];
                    a = -s8[t] * a + c8[t] * h8[t];
                }
            }
        }
        const double den = sqrt(a * a + hn * hn);
        const double cj = den == 0.0 ? 1.0 : a / den, sj = den == 0.0 ? 0.0 : hn / den;
        h[j] = cj * a + sj * hn;
        gs[L.CS + j] = cj;
        gs[L.SN + j] = sj;
        const double gj = gs[L.G + j], gn = -sj * gj;
        gs[L.G + j + 1] = gn;
        gs[L.G + j] = cj * gj;
        gi[GI_CYC] = j + 1;
        const int total = gi[GI_TOTAL] + 1;
        gi[GI_TOTAL] = total;
        gs[L.SC + j + 1] = hn > 0.0 ? 1.0 / hn : 0.0;
        const bool conv = fabs(gn) <= k.step[c].tol_res * gs[L.BN];
        if (conv || !(hn > 0.0) || !isfinite(hn) || total >= gi[GI_MAXIT] || j == m - 1) gi[GI_DONE] = 1;
    }
    __syncthreads();
    if (tid <= j) gs[L.H + (size_t)j * (m + 1) + tid] = h[tid];
}

// y = H^-1 g on the iterations of this cycle, times the scales of the basis vectors: one workgroup
// per case, thread q holding row q.  Column by column from the last, each column's loads issued one
// step ahead (one thread walking the rows took 205 us at m = 150).
__global__ void __launch_bounds__(256) k_backsub(Ctl k, int m) {
    __shared__ double ys[MAXV];
    const int c = blockIdx.x, q = threadIdx.x;
    const int* gi = k.gi + c * GI_STRIDE;
    if (gi[GI_IDLE]) return;   // uniform per workgroup
    const GsLayout L(m);
    double* gs = k.gs + (size_t)c * k.gs_stride;
    const int jd = gi[GI_CYC];
    const double* H = gs + L.H;
    double g = q < jd ? gs[L.G + q] : 0.0;
    double hn = q < jd ? H[(size_t)(jd - 1) * (m + 1) + q] : 0.0;
    for (int i = jd - 1; i >= 0; --i) {
        const double hi = hn;
        if (i > 0 && q < i) hn = H[(size_t)(i - 1) * (m + 1) + q];
        if (q == i) ys[i] = g / hi;
        __syncthreads();
        if (q < i) g -= hi * ys[i];
    }
    if (q < m) gs[L.Y + q] = q < jd ? ys[q] * gs[L.SC + q] : 0.0;
}

// beta = |r| after the update; a non-finite beta retires the case; summary for the host
__global__ void k_cycle_end(Ctl k, int m) {
    const int c = case_index();
    if (c >= k.n) return;
    const GsLayout L(m);
    double* gs = k.gs + (size_t)c * k.gs_stride;
    int* gi = k.gi + c * GI_STRIDE;
    if (!gi[GI_IDLE]) {
        const double beta = sqrt(gs[L.NRM]);
        gs[L.BETA] = beta;
        if (!isfinite(beta)) { gi[GI_STATUS] = 1; gi[GI_NDONE] = 1; }
    }
    double* s = k.sum + (size_t)c * SUM_STRIDE;
    s[S_BN] = gs[L.BN];
    s[S_BETA] = gs[L.BETA];
    s[S_TOTAL] = gi[GI_TOTAL];
    s[S_MORE] = (!gi[GI_IDLE] && gi[GI_CYC] > 0 && wants_cycle(gi, gs[L.BETA], gs[L.BN], k.step[c].tol_res)) ? 1.0 : 0.0;
}

// GMRES iterations of this Newton step into the case's total
__global__ void k_gm_finish(Ctl k) {
    const int c = case_index();
    if (c >= k.n) return;
    k.sum[(size_t)c * SUM_STRIDE + S_GMRES] += k.gi[c * GI_STRIDE + GI_TOTAL];
}

// ---- chunk-walking vector kernels (every chunk belongs to one case)
struct Vec {
    const int* chunk_case;
    int nchunks;
    const int* gi;
    int flag;   // skip flag
};

// 1024 entries to a workgroup pass
static_assert(CHUNK % 1024 == 0, "a pass of the vector kernels lies in one chunk");
#define FR_CHUNKS(vc, ...)                                                                                \
    for (long long w_ = blockIdx.x; w_ < (long long)(vc).nchunks * (CHUNK / 1024); w_ += gridDim.x) {      \
        const int c = (vc).chunk_case[w_ / (CHUNK / 1024)];                                                \
        if ((vc).gi[c * GI_STRIDE + (vc).flag]) continue;                                                  \
        for (size_t t = (size_t)w_ * 1024 + threadIdx.x; t < (size_t)(w_ + 1) * 1024; t += blockDim.x) {   \
            __VA_ARGS__                                                                                    \
        }                                                                                                  \
    }

__global__ void k_add(Vec vc, const double* __restrict__ z, double* __restrict__ x) { FR_CHUNKS(vc, x[t] += z[t];) }
__global__ void k_sub(Vec vc, const double* __restrict__ b, const double* __restrict__ w, double* __restrict__ r) {
    FR_CHUNKS(vc, r[t] = b[t] - w[t];)
}
__global__ void k_fill(Vec vc, double v, double* __restrict__ x) { FR_CHUNKS(vc, x[t] = v;) }
__global__ void k_copy(Vec vc, const double* __restrict__ a, double* __restrict__ b) { FR_CHUNKS(vc, b[t] = a[t];) }

unsigned vgrid(const Solver& sv) {
    const long long g = (long long)sv.nchunks * (CHUNK / 1024);
    return (unsigned)(g < 8192 ? g : 8192);
}
unsigned cgrid(const Solver& sv) { return (unsigned)((sv.n + 63) / 64); }

Ctl ctl(const Solver& sv) { return Ctl{sv.d_gs, sv.gs_stride, sv.d_gi, sv.d_step, sv.d_sum, sv.n}; }
Vec vec(const Solver& sv, int flag) { return Vec{sv.d_chunk_case, sv.nchunks, sv.d_gi, flag}; }

double* wv(const Solver& sv, int i) { return sv.d_w + (size_t)i * sv.Ntot; }

// Newton operator at the iterate whose linearisation packs the Newton loop has written
KArgs bdf_args(const Solver& sv, const double* q) {
    KArgs a{};
    a.q = q; a.cstep = sv.d_step; a.flags = sv.d_gi;
    a.fpack = sv.d_fpack; a.spack = sv.d_spack;
    return a;
}

fr_status bdf_op(const Solver& sv, const double* q, const double* v, double* Av, int flag, hipStream_t s, int only = -1) {
    KArgs a = bdf_args(sv, q);
    a.v = v; a.out = Av; a.flag = flag;
    return solver_fused(sv, MODE_LIN, a, s, only);
}

// Whether the groups' launches of an Arnoldi step go to parallel branches of its graph.  A fork and
// join of the graph costs about 20 us a step; side by side the kernels of ten launches and more, each
// too small for the chip, save more than that.  BDF2 steps of batches, ms, in branches (one after the
// other): 5 groups, Jacobi 42.0 (45.2), 6 groups 31.6 (35.7); symmetric Gauss-Seidel, 4 groups 27.5
// (33.7), 6 groups 49.1 (63.1); forward sweeps, 4 groups of cases up to 96 x 96 18.0 (19.5) and 27.8
// (32.5), up to 32 x 32 16.2 (17.8) and 16.6 (16.4); not taken: 3 groups, forward sweeps 16.8 (14.8), 4
// groups, Jacobi 29.9 (28.1), 5 groups of 8 x 8 cases 28.4 (27.4).
bool in_branches(const Solver& sv) {
    const int ng = (int)sv.groups.size(), K = sv.ncolors;
    const int each = sv.precond == 0 ? 2 : sv.precond == 1 ? 4 * K - 2 : 2 * K;
    return ng >= 4 && ng * each >= 10 && sv.Ntot > ((size_t)1 << 16);
}

// w = A P^-1 v.  The groups of a batch have no part of z or w in common (nor of the sweeps' scratch).
fr_status operate(Solver& sv, int m, const double* q, const double* v, double* z, double* w, hipStream_t s) {
    const int ng = (int)sv.groups.size();
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (in_branches(sv)) FR_HIP(hipStreamIsCapturing(s, &cap));
    if (cap != hipStreamCaptureStatusActive) {
        FR_TRY(precond_apply(sv, v, z, bdf_args(sv, q), m, sv.d_gi, GI_DONE, s));
        return bdf_op(sv, q, z, w, GI_DONE, s);
    }
    const int nside = ng - 1 < SIDE_STREAMS ? ng - 1 : SIDE_STREAMS;
    FR_HIP(hipEventRecord(sv.ev_fork, s));
    for (int k = 0; k < nside; ++k) FR_HIP(hipStreamWaitEvent(sv.side[k], sv.ev_fork, 0));
    for (int i = 0; i < ng; ++i) {
        const int k = i % (nside + 1);
        hipStream_t t = k < nside ? sv.side[k] : s;
        FR_TRY(precond_apply(sv, v, z, bdf_args(sv, q), m, sv.d_gi, GI_DONE, t, i));
        FR_TRY(bdf_op(sv, q, z, w, GI_DONE, t, i));
    }
    for (int k = 0; k < nside; ++k) {
        FR_HIP(hipEventRecord(sv.ev_join[k], sv.side[k]));
        FR_HIP(hipStreamWaitEvent(s, sv.ev_join[k], 0));
    }
    return FR_OK;
}

// the launches of one cycle (enqueued eagerly or under capture): an Arnoldi step
fr_status enqueue_arnoldi(Solver& sv, int m, int j, hipStream_t s) {
    const size_t N = sv.Ntot;
    const GsLayout L(m);
    const double* q = sv.d_q;
    double* w = wv(sv, WW);
    double* z = wv(sv, WZ);
    double* V = sv.d_V;
    double* vj = V + (size_t)j * N;
    double* vn = vj + N;
    FR_TRY(operate(sv, m, q, vj, z, w, s));
    // classical Gram-Schmidt: h = V^T w, w -= V h (and once more when re-orthogonalising); each pass
    // over the basis walks its items the other way from the pass before it
    const GsRef g1{sv.d_gs, sv.gs_stride, L.DT, L.SC, L.H1, j, 1};
    FR_TRY(la_dots(sv, V, N, j + 1, w, g1, 0, sv.d_gi, GI_DONE, s));
    if (sv.gs_passes == 2) {
        const GsRef g2{sv.d_gs, sv.gs_stride, L.DT, L.SC, L.H2, j, 0};
        if (sv.fuse_gs && j + 1 <= 32) {
            FR_TRY(la_update_dots(sv, V, N, j + 1, w, vn, g1, 0, sv.d_gi, GI_DONE, s, true));
        } else {
            FR_TRY(la_update(sv, V, N, j + 1, w, vn, false, g1, 0, sv.d_gi, GI_DONE, s, true));
            FR_TRY(la_dots(sv, V, N, j + 1, vn, g2, 1, sv.d_gi, GI_DONE, s));
        }
        FR_TRY(la_update(sv, V, N, j + 1, vn, vn, true, g2, 1, sv.d_gi, GI_DONE, s, !sv.fuse_gs));
    } else {
        FR_TRY(la_update(sv, V, N, j + 1, w, vn, true, g1, 0, sv.d_gi, GI_DONE, s, true));
    }
    // |v_{j+1}|^2's second stage and the Givens update in one launch
    hipLaunchKernelGGL(k_norm_givens, dim3(sv.n), dim3(256), 0, s, ctl(sv), sv.d_ufirst, part_norm(sv), j, m,
                       sv.gs_passes);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

// Arnoldi steps per segment.  The steps after the last case has stopped skip every case, but their
// launches cost 2 to 3 us each (with m = 150 on 16 x 16 elements 410 of 750 launched steps did
// nothing); a graph launch costs about 15 us.  6 measured best of 4, 6 and 10: 16 x 16 steady
// GMRES(150) 24.1 -> 20.1 ms a pass, 256 x 256 p = 3 46.8 -> 46.3 ms a step, 128 x 128 deforming
// 25.0 -> 24.5 ms.  Small cases (about 20 us a step) with a short restart have little to skip and
// keep the whole cycle, with its end, in one graph: 8 x 8 p = 2, m = 20: 1.83 ms a step against 1.91.
int segment_len(const Solver& sv, int m) { return sv.all_small && m <= 40 ? m : 6; }
int nsegments(const Solver& sv, int m) { return (m + segment_len(sv, m) - 1) / segment_len(sv, m); }

// whether some case's Arnoldi process goes on after a segment, to pinned host memory
__global__ void k_segment_end(Ctl k, int* __restrict__ more) {
    const int lane = threadIdx.x;   // one wave
    bool any = false;
    for (int c = lane; c < k.n; c += 64) any = any || !k.gi[c * GI_STRIDE + GI_DONE];
    const bool r = __any(any);
    if (lane == 0) *more = r ? 1 : 0;
}

// segment i of the cycle (with the cycle's start in the first)
fr_status enqueue_segment(Solver& sv, int m, int i, hipStream_t s) {
    if (i == 0) {
        hipLaunchKernelGGL(k_cycle_init, dim3(cgrid(sv)), dim3(64), 0, s, ctl(sv), m);
        FR_HIP(hipGetLastError());
    }
    const int len = segment_len(sv, m), j1 = (i + 1) * len < m ? (i + 1) * len : m;
    for (int j = i * len; j < j1; ++j) FR_TRY(enqueue_arnoldi(sv, m, j, s));
    if (j1 < m) {
        hipLaunchKernelGGL(k_segment_end, dim3(1), dim3(64), 0, s, ctl(sv), sv.h_seg + i);
        FR_HIP(hipGetLastError());
    }
    return FR_OK;
}

fr_status enqueue_end(Solver& sv, int m, hipStream_t s) {
    const size_t N = sv.Ntot;
    const GsLayout L(m);
    const double* q = sv.d_q;
    const double* b = wv(sv, WB);
    double* x = wv(sv, WDQ);
    double* w = wv(sv, WW);
    double* z = wv(sv, WZ);
    double* r = sv.d_V;   // the residual is the next cycle's v_0
    const Ctl k = ctl(sv);
    hipLaunchKernelGGL(k_backsub, dim3(sv.n), dim3(256), 0, s, k, m);
    FR_HIP(hipGetLastError());
    FR_TRY(la_combine(sv, sv.d_V, N, sv.d_gs, sv.gs_stride, L.Y, w, sv.d_gi, GI_IDLE, s));
    FR_TRY(precond_apply(sv, w, z, bdf_args(sv, q), m, sv.d_gi, GI_IDLE, s));
    hipLaunchKernelGGL(k_add, dim3(vgrid(sv)), dim3(256), 0, s, vec(sv, GI_IDLE), z, x);
    FR_HIP(hipGetLastError());
    FR_TRY(bdf_op(sv, q, x, w, GI_IDLE, s));
    hipLaunchKernelGGL(k_sub, dim3(vgrid(sv)), dim3(256), 0, s, vec(sv, GI_IDLE), b, w, r);
    FR_HIP(hipGetLastError());
    FR_TRY(la_norm(sv, r, false, sv.d_gs + L.NRM, sv.gs_stride, sv.d_gi, GI_IDLE, s));
    hipLaunchKernelGGL(k_cycle_end, dim3(cgrid(sv)), dim3(64), 0, s, k, m);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

// capture `enqueue` into an executable graph
template <class F>
fr_status capture(hipStream_t s, F&& enqueue, void** out) {
    hipGraph_t gr;
    FR_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    const fr_status cst = enqueue();
    const hipError_t ee = hipStreamEndCapture(s, &gr);
    if (cst != FR_OK) { if (ee == hipSuccess) (void)hipGraphDestroy(gr); return cst; }
    FR_HIP(ee);
    hipGraphExec_t ex;
    const hipError_t ie = hipGraphInstantiate(&ex, gr, nullptr, nullptr, 0);
    (void)hipGraphDestroy(gr);
    FR_HIP(ie);
    *out = ex;
    return FR_OK;
}

// launches i of a cycle of nseg segments: the segments, then the end (with a single segment, all at once)
fr_status enqueue_part(Solver& sv, int m, int i, hipStream_t s) {
    const int nseg = nsegments(sv, m);
    if (i < nseg) FR_TRY(enqueue_segment(sv, m, i, s));
    return i >= nseg || nseg == 1 ? enqueue_end(sv, m, s) : FR_OK;
}
int nparts(const Solver& sv, int m) { return nsegments(sv, m) == 1 ? 1 : nsegments(sv, m) + 1; }

// One restart cycle.  Running one segment ahead keeps the GPU busy while the host learns how the
// last one ended.
fr_status run_cycle(Solver& sv, int m, bool graph, hipStream_t s) {
    const int last = nparts(sv, m) - 1;
    auto launch = [&](int i) -> fr_status {
        if (!graph) return enqueue_part(sv, m, i, s);
        FR_HIP(hipGraphLaunch((hipGraphExec_t)sv.graph_exec[i], s));
        return FR_OK;
    };
    for (int i = 0; i < last; ++i) {
        FR_TRY(launch(i));
        if (i + 1 < last) FR_HIP(hipEventRecord(sv.ev_seg[i & 1], s));
        if (i == 0) continue;
        FR_HIP(hipEventSynchronize(sv.ev_seg[(i - 1) & 1]));
        if (!*(volatile int*)(sv.h_seg + i - 1)) break;
    }
    return launch(last);
}

// ---- Newton-level kernels
__global__ void k_step_init(Ctl k) {
    const int c = case_index();
    if (c >= k.n) return;
    int* gi = k.gi + c * GI_STRIDE;
    for (int f = 0; f < GI_STRIDE; ++f) gi[f] = 0;
    double* s = k.sum + (size_t)c * SUM_STRIDE;
    for (int f = 0; f < SUM_STRIDE; ++f) s[f] = 0.0;
}

// per case: Newton test on the mass-row norm of b (in the NRM slot).  With SER (steady
// solves, paper Eq. SER) the pseudo-time step of this iteration follows from the previous
// one and the residual ratio Res_{m-1}/Res_m, clipped to [dtau_min, dtau_max].
__global__ void k_newton_check(Ctl k, int m, int it) {
    const int c = case_index();
    if (c >= k.n) return;
    int* gi = k.gi + c * GI_STRIDE;
    double* s = k.sum + (size_t)c * SUM_STRIDE;
    if (gi[GI_NDONE]) return;
    const GsLayout L(m);
    const double rr = sqrt(k.gs[(size_t)c * k.gs_stride + L.NRM]);
    if (it == 0) s[S_RES0] = rr;
    s[S_RES] = rr;
    s[S_NEWTON] = it;
    CaseStep& st = k.step[c];
    if (st.ser && st.reject_growth > 0.0 && it > 0 && !st.retry && !(rr <= st.reject_growth * st.res_prev)) {
        // step rejection (not in the paper; off unless requested): the step just taken is undone
        // by k_reject_restore and retried from the same state with a ten times smaller dtau;
        // the case sits out the rest of this iteration and recomputes its residual in the next
        st.dtau *= 0.1;
        st.idt = 1.0 / st.dtau;
        st.retry = 1;
        s[S_DTAU] = st.dtau;
        s[S_REJ] += 1.0;
        gi[GI_REJECT] = 1;
        gi[GI_NDONE] = 1;
        return;
    }
    if (!isfinite(rr)) { gi[GI_STATUS] = 1; gi[GI_NDONE] = 1; return; }
    if (rr <= st.tol_abs || rr <= st.tol_pseudo * s[S_RES0]) { gi[GI_CONV] = 1; gi[GI_NDONE] = 1; return; }
    if (it >= st.max_newton) { gi[GI_STATUS] = 2; gi[GI_NDONE] = 1; return; }
    if (st.ser) {
        if (it > 0 && !st.retry) {
            const double d = st.dtau * pow(st.res_prev / rr, st.r_ser);
            st.dtau = fmax(st.dtau_min, fmin(st.dtau_max, d));
            st.idt = 1.0 / st.dtau;
        }
        st.retry = 0;
        st.res_prev = rr;
        s[S_DTAU] = st.dtau;
    }
}

// q -= dq for the cases whose step k_newton_check undid
__global__ void k_reject_restore(Vec vc, const double* __restrict__ dq, double* __restrict__ q) {
    for (long long w = blockIdx.x; w < (long long)vc.nchunks * (CHUNK / 1024); w += gridDim.x) {
        const int c = vc.chunk_case[w / (CHUNK / 1024)];
        if (!vc.gi[c * GI_STRIDE + GI_REJECT]) continue;
        for (size_t t = (size_t)w * 1024 + threadIdx.x; t < (size_t)(w + 1) * 1024; t += blockDim.x) q[t] -= dq[t];
    }
}

// a case whose step was undone takes part again, from its restored state
__global__ void k_retry(Ctl k) {
    const int c = case_index();
    if (c >= k.n) return;
    int* gi = k.gi + c * GI_STRIDE;
    if (gi[GI_REJECT]) { gi[GI_REJECT] = 0; gi[GI_NDONE] = 0; }
}

// a singular block (status 3) takes its case out of the iteration; flags to the summary
__global__ void k_after_factor(Ctl k) {
    const int c = case_index();
    if (c >= k.n) return;
    int* gi = k.gi + c * GI_STRIDE;
    if (gi[GI_STATUS] == 3) gi[GI_NDONE] = 1;
}

__global__ void k_publish(Ctl k) {
    const int c = case_index();
    if (c >= k.n) return;
    const int* gi = k.gi + c * GI_STRIDE;
    double* s = k.sum + (size_t)c * SUM_STRIDE;
    s[S_NDONE] = gi[GI_NDONE] && !gi[GI_REJECT];
    s[S_CONV] = gi[GI_CONV];
    s[S_STATUS] = gi[GI_STATUS];
}

__global__ void k_axpy_case(Vec vc, const double* __restrict__ dq, double* __restrict__ q) {
    FR_CHUNKS(vc, q[t] += dq[t];)
}

}  // namespace

size_t gmres_state_doubles(int m) { return (size_t)GsLayout(m).total; }

void gmres_release(Solver& sv) {
    for (void* g : sv.graph_exec) (void)hipGraphExecDestroy((hipGraphExec_t)g);
    sv.graph_exec.clear();
}

// GMRES on every case still in the Newton iteration: A dq = b with b = WB, dq = WDQ
fr_status gmres_device(Solver& sv, int m, int prec, int max_it, hipStream_t s) {
    PhaseRange range("lmfr: GMRES solve");
    const GsLayout L(m);
    const Ctl k = ctl(sv);
    hipLaunchKernelGGL(k_gm_start, dim3(cgrid(sv)), dim3(64), 0, s, k, max_it);
    FR_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_fill, dim3(vgrid(sv)), dim3(256), 0, s, vec(sv, GI_NDONE), 0.0, wv(sv, WDQ));
    FR_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_copy, dim3(vgrid(sv)), dim3(256), 0, s, vec(sv, GI_NDONE), wv(sv, WB), sv.d_V);
    FR_HIP(hipGetLastError());
    FR_TRY(la_norm(sv, wv(sv, WB), false, sv.d_gs + L.NRM, sv.gs_stride, sv.d_gi, GI_NDONE, s));
    hipLaunchKernelGGL(k_gm_norm0, dim3(cgrid(sv)), dim3(64), 0, s, k, m);
    FR_HIP(hipGetLastError());

    if (sv.precond != 0) {   // the sweeps' work vector exists before any capture
        FR_TRY(dalloc(&sv.d_gst, sv.Ntot));
    }
    const bool graph = sv.use_graph;
    // the operator kernel of a group depends on whether its elements are all affine
    std::vector<char> aff(sv.groups.size());
    for (size_t g = 0; g < sv.groups.size(); ++g) {
        bool all = true;
        for (int id : sv.groups[g].ids) all = all && sv.cs[id]->all_affine;
        aff[g] = all ? 1 : 0;
    }
    if (graph && (sv.graph_exec.empty() || sv.graph_m != m || sv.graph_prec != prec || sv.graph_passes != sv.gs_passes ||
                  sv.graph_precond != sv.precond || sv.graph_cl != (int)sv.inv_colour || sv.graph_aff != aff)) {
        gmres_release(sv);
        // capture one cycle (all buffers are solver-owned; tolerances, time coefficients and
        // caps are read on the device, so the graphs depend on m, the block precision and
        // layout, the Gram-Schmidt passes and the preconditioner only)
        for (int i = 0; i < nparts(sv, m); ++i) {
            void* ex = nullptr;
            const fr_status st = capture(s, [&] { return enqueue_part(sv, m, i, s); }, &ex);
            if (st != FR_OK) { gmres_release(sv); return st; }
            sv.graph_exec.push_back(ex);
        }
        sv.graph_m = m;
        sv.graph_prec = prec;
        sv.graph_passes = sv.gs_passes;
        sv.graph_precond = sv.precond;
        sv.graph_cl = (int)sv.inv_colour;
        sv.graph_aff = aff;
    }
    double* hs = sv.h_pin;
    for (;;) {
        FR_TRY(run_cycle(sv, m, graph, s));
        FR_HIP(hipMemcpyAsync(hs, sv.d_sum, (size_t)sv.n * SUM_STRIDE * sizeof(double), hipMemcpyDeviceToHost, s));
        FR_HIP(hipStreamSynchronize(s));
        bool more = false;
        for (int c = 0; c < sv.n; ++c) more |= hs[(size_t)c * SUM_STRIDE + S_MORE] != 0.0;
        if (!more) break;
    }
    hipLaunchKernelGGL(k_gm_finish, dim3(cgrid(sv)), dim3(64), 0, s, k);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

// The BDF2 (BDF1 for cases without q^{n-1}) dual-time Newton iteration of every case,
// paper Sec. 3.2, Eq. (unsteady_pre_discretized_3): the iterate and Q^n, Q^{n-1} are in
// the solver's vectors (WQN, WQNM1 hold the states on entry; converted here).
fr_status solver_newton(Solver& sv, const fr_step_opts* o, hipStream_t s) {
    PhaseRange range("lmfr: BDF2 step (Newton loop)");
    const Ctl k = ctl(sv);
    const GsLayout L(o->krylov);
    hipLaunchKernelGGL(k_step_init, dim3(cgrid(sv)), dim3(64), 0, s, k);
    FR_HIP(hipGetLastError());
    FR_TRY(launch_cons(sv, sv.d_q, wv(sv, WQN), sv.d_gi, s));
    FR_TRY(launch_cons_nm1(sv, wv(sv, WQNM1), s));
    double* hs = sv.h_pin;
    for (int it = 0;; ++it) {
        PhaseRange it_range("lmfr: Newton iteration");
        if (sv.reject_on) {
            hipLaunchKernelGGL(k_retry, dim3(cgrid(sv)), dim3(64), 0, s, k);
            FR_HIP(hipGetLastError());
        }
        // R at the iterate, and the linearisation packs the GMRES operator reads
        KArgs a{};
        a.q = sv.d_q; a.out = wv(sv, WR); a.flags = sv.d_gi; a.flag = GI_NDONE;
        a.fpack = sv.d_fpack; a.spack = sv.d_spack;
        FR_TRY(solver_fused(sv, MODE_PREP, a, s));
        FR_TRY(launch_bdf_rhs(sv, sv.d_q, wv(sv, WQN), wv(sv, WQNM1), wv(sv, WR), wv(sv, WB), sv.d_gi, s));
        FR_TRY(la_norm(sv, wv(sv, WB), true, sv.d_gs + L.NRM, sv.gs_stride, sv.d_gi, GI_NDONE, s));
        hipLaunchKernelGGL(k_newton_check, dim3(cgrid(sv)), dim3(64), 0, s, k, o->krylov, it);
        FR_HIP(hipGetLastError());
        if (sv.reject_on) {
            hipLaunchKernelGGL(k_reject_restore, dim3(vgrid(sv)), dim3(256), 0, s, vec(sv, GI_NDONE), wv(sv, WDQ),
                               sv.d_q);
            FR_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(k_publish, dim3(cgrid(sv)), dim3(64), 0, s, k);
        FR_HIP(hipGetLastError());
        FR_HIP(hipMemcpyAsync(hs, sv.d_sum, (size_t)sv.n * SUM_STRIDE * sizeof(double), hipMemcpyDeviceToHost, s));
        FR_HIP(hipStreamSynchronize(s));
        bool any = false;
        for (int c = 0; c < sv.n; ++c) any |= hs[(size_t)c * SUM_STRIDE + S_NDONE] == 0.0;
        if (!any) break;
        if (it % o->jac_lag == 0) {
            PhaseRange refresh_range("lmfr: preconditioner refresh (enqueue)");
            KArgs b{};
            b.cstep = sv.d_step; b.flags = sv.d_gi; b.flag = GI_NDONE;
            b.fpack = sv.d_fpack; b.spack = sv.d_spack;   // written by this iteration's residual pass
            FR_TRY(launch_block_assembly(sv, sv.d_q, b, s));
            if (sv.keep_blocks) {
                FR_HIP(hipMemcpyAsync(sv.d_blk_keep, sv.d_blk, sv.Btot * sizeof(double), hipMemcpyDeviceToDevice, s));
            }
            FR_TRY(launch_block_invert(sv, o->prec, sv.d_gi, s));
            hipLaunchKernelGGL(k_after_factor, dim3(cgrid(sv)), dim3(64), 0, s, k);
            FR_HIP(hipGetLastError());
        }
        FR_TRY(gmres_device(sv, o->krylov, o->prec, o->max_lin_it, s));
        hipLaunchKernelGGL(k_axpy_case, dim3(vgrid(sv)), dim3(256), 0, s, vec(sv, GI_NDONE), wv(sv, WDQ), sv.d_q);
        FR_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_publish, dim3(cgrid(sv)), dim3(64), 0, s, k);
    FR_HIP(hipGetLastError());
    FR_HIP(hipMemcpyAsync(hs, sv.d_sum, (size_t)sv.n * SUM_STRIDE * sizeof(double), hipMemcpyDeviceToHost, s));
    FR_HIP(hipStreamSynchronize(s));
    return FR_OK;
}
