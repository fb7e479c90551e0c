// Explicit inverse of every element block (the element-block-Jacobi preconditioner of the
// paper's Sec. 4 set-up): in-place Gauss-Jordan elimination with partial pivoting, the whole
// block in registers.
//
// A group of TR x CT threads holds an element, RPT x CPT entries each (Map): one wave up to
// 64 x 64 (more for a few blocks), four for 100 x 100.  Thread (tr, tc) holds the rows 2 tr + 2 TR i, + 1 (pairs, so that
// loads and LDS reads are 16 bytes wide and consecutive) and the columns tc + CT b.  Step k, with
// the column of step k at register column 0:
//   1. its owners put the column into LDS; every wave reads it, one or two rows a lane, and takes
//      the unused row with the largest |a(r, k)| as pivot row p: one DPP maximum over integer keys,
//      the leading bits of |a| above 127 - row (two entries that agree to 2^-13 count as a tie,
//      which goes to the lower row);
//   2. the owners of row p put it into LDS, and everyone applies a(r, c) -= a(r, k) a(p, c) / a(p, k).
// Row p and column k of the in-place inverse come out of the same update: the row is zeroed in
// its owners and its multiplier is 1 / a(p, k), the column is zeroed and its entry of the row is 1.
// Register columns move down by one once the CT columns of register 0 have been pivots: the last
// of these steps writes each result one register lower, so the loop is one small body with
// constant register numbers.  Rows stay where they are; at the end the block holds the inverse
// with rows and columns permuted by the pivot order, inverse(pos(r), piv(k)) = a(r, k), pos the
// step at which row r was the pivot, and goes out through LDS, CT whole columns at a time.
//
// Arithmetic type TC: FP64 for an FP64 inverse; FP32 for an FP32 or BF16 inverse, the FP64 block
// rounded to FP32 on load and the FP32 result rounded to nearest even for BF16.
//
// What bounds it: instruction issue.  FP64 matrix instructions share the vector pipe and reach
// 1.27 times its rate, while a panel form needs the block in LDS (80 KB at p = 4: two workgroups a
// compute unit) and leaves three waves of four idle through its panels.  65,536 blocks, against
// panels of 16 columns in LDS with the trailing update on the matrix cores, ms:
//     nb            16           36           64           100
//     FP64     0.12 (0.45)  0.59 (1.93)  2.28 (3.41)  7.94 (20.1)
//     FP32     0.09 (0.27)  0.40 (1.12)  1.12 (1.63)  4.73 (8.34)
#include "fr_internal.hpp"
#include <type_traits>

namespace {

template <class TO, class TC> __device__ __forceinline__ TO store_as(TC x);
template <> __device__ __forceinline__ double store_as<double, double>(double x) { return x; }
template <> __device__ __forceinline__ float store_as<float, float>(float x) { return x; }
template <> __device__ __forceinline__ uint16_t store_as<uint16_t, float>(float x) {
    const uint32_t u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);   // inf / nan
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);           // round to nearest even
}

// one lane's value, read into scalar registers
__device__ __forceinline__ double lane_value(double x, int lane) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ float lane_value(float x, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
// maximum over the wave by DPP: within rows of 16 lanes, then across the rows; lane 63 holds it
template <int CTRL> __device__ __forceinline__ unsigned umax_dpp(unsigned x) {
    const unsigned y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
    return x > y ? x : y;
}
__device__ __forceinline__ unsigned wave_umax(unsigned x) {
    x = umax_dpp<0x111>(x);   // row_shr 1, 2, 4, 8
    x = umax_dpp<0x112>(x);
    x = umax_dpp<0x114>(x);
    x = umax_dpp<0x118>(x);
    x = umax_dpp<0x142>(x);   // row_bcast 15, 31
    x = umax_dpp<0x143>(x);
    return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}

__device__ __forceinline__ int case_of_tile(const GroupArgs& ga, int t) {
    int lo = 0, hi = ga.nmem - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ga.pfx[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// threads and entries of one element: TR x CT threads in NW waves, RPT x CPT entries each.  One
// wave needs no barrier and shares a step's fixed work over most entries; 100 x 100 takes four for
// its registers (two waves of 4 x 20 entries: 8.3 ms for 7.9 at FP64, 6.2 for 4.7 at FP32), 64 x 64
// two or four where the blocks are too few to fill the chip (waves_64).  The arithmetic on an entry
// is the same in all.
template <int NB, int NW> struct Map;
template <> struct Map<16, 1> { static constexpr int TR = 8, CT = 8, OCC = 8; };
template <> struct Map<36, 1> { static constexpr int TR = 9, CT = 6, OCC = 4; };
template <> struct Map<64, 1> { static constexpr int TR = 8, CT = 8, OCC = 2; };
template <> struct Map<64, 2> { static constexpr int TR = 16, CT = 8, OCC = 4; };
template <> struct Map<64, 4> { static constexpr int TR = 16, CT = 16, OCC = 4; };
template <> struct Map<100, 4> { static constexpr int TR = 25, CT = 10, OCC = 3; };

// what the LDS traffic of an element needs between its threads: a barrier, or only order within
// its one wave
template <int NW> __device__ __forceinline__ void group_sync() {
    if constexpr (NW > 1) __syncthreads();
    else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// pivot key of entry x in the given row: 0 for a NaN, else at least 1
__device__ __forceinline__ unsigned pivot_key(unsigned hi, unsigned inf, int row) {
    hi &= 0x7fffffffu;
    return hi > inf ? 0u : (hi & ~127u) | (unsigned)(127 - row);
}
__device__ __forceinline__ unsigned pivot_key(double x, int row) {
    return pivot_key((unsigned)(__double_as_longlong(x) >> 32), 0x7ff00000u, row);
}
__device__ __forceinline__ unsigned pivot_key(float x, int row) { return pivot_key(__float_as_uint(x), 0x7f800000u, row); }

template <int NB, int NW, class TC, class TO>
__global__ void __launch_bounds__(64 * NW, (Map<NB, NW>::OCC))
k_block_invert(GroupArgs ga, const double* __restrict__ blk, TO* __restrict__ inv, int* __restrict__ gi,
               const int* __restrict__ flags, int cl) {
    using M = Map<NB, NW>;
    constexpr int TR = M::TR, CT = M::CT, RPT = NB / TR, CPT = NB / CT, NTH = 64 * NW;
    // The reciprocal pivot multiplies the pivot row (ROW) or the column.  The row's products round to
    // errors 3 to 7% smaller in the mean of |B X - 1|, those of the elimination in panels at one panel;
    // the larger blocks are below their panels' errors with the column too (0.3 to 0.95 times), which
    // is a multiplication less in six to ten
    constexpr bool ROW = NB <= 36;
    static_assert(RPT * TR == NB && CPT * CT == NB && RPT % 2 == 0 && CPT % 2 == 0, "whole pairs");
    static_assert(NB <= 127 && TR * CT <= NTH, "row numbers in 7 bits");
    typedef TC V2 __attribute__((ext_vector_type(2)));
    __shared__ V2 s_col[NB / 2], s_row[NB / 2];
    __shared__ TC s_out[CT * NB];
    __shared__ uint8_t s_piv[NB], s_pos[NB];   // pivot row of each step, step of each pivot row
    const int tid = threadIdx.x, lane = tid & 63;
    const int t = blockIdx.x;
    if (t >= ga.ntiles) return;                                   // uniform per workgroup
    const int lo = case_of_tile(ga, t);
    const int cid = ga.ids[lo];
    if (flags && flags[cid * GI_STRIDE + GI_NDONE]) return;       // uniform per workgroup
    const CaseDev& cd = ga.cases[cid];
    // slot of the stored inverse; its element is the same index, or the slot's entry of the
    // colour-sorted element list in the colour layout
    const int slot = t - ga.pfx[lo];
    const int e = cl ? cd.g.corder[slot] : slot;
    const double* src = blk + cd.boff + (size_t)e * NB * NB;

    // idle threads (TR CT < NTH) read as thread 0 does and own nothing
    const bool act = tid < TR * CT;
    const int tr = act ? tid % TR : 0, tc = act ? tid / TR : 0;
    const int own_r = act ? tr : -1, own_c = act ? tc : -1;
    TC A[RPT][CPT];
#pragma unroll
    for (int b = 0; b < CPT; ++b)
#pragma unroll
        for (int i = 0; i < RPT / 2; ++i) {
            const double2 x = *(const double2*)(src + (tc + CT * b) * NB + 2 * tr + 2 * TR * i);
            A[2 * i][b] = (TC)x.x;
            A[2 * i + 1][b] = (TC)x.y;
        }
    // rows whose entries this lane looks at in a pivot search
    bool u0 = lane >= NB, u1 = lane + 64 >= NB, bad = false;

    // the owners' register column 0 into LDS, and zero there
    auto put_column = [&](int jc) {
        if (own_c == jc) {
#pragma unroll
            for (int i = 0; i < RPT / 2; ++i) {
                s_col[tr + TR * i] = V2{A[2 * i][0], A[2 * i + 1][0]};
                A[2 * i][0] = TC(0);
                A[2 * i + 1][0] = TC(0);
            }
        }
    };
    // one elimination step, SHIFT: results one register column lower
    auto step = [&](auto shift, int k, int jc) {
        constexpr int SH = decltype(shift)::value;
        put_column(jc);
        group_sync<NW>();
        const TC* col = (const TC*)s_col;
        const TC x0 = col[NB > 64 ? lane : (lane < NB ? lane : 0)];
        const TC x1 = NB > 64 ? col[lane + 64 < NB ? lane + 64 : 0] : TC(0);
        V2 f[RPT / 2];
#pragma unroll
        for (int i = 0; i < RPT / 2; ++i) f[i] = s_col[tr + TR * i];
        unsigned key = u0 ? 0u : pivot_key(x0, lane);
        if (NB > 64) {
            const unsigned key1 = u1 ? 0u : pivot_key(x1, lane + 64);
            key = key > key1 ? key : key1;
        }
        key = wave_umax(key);
        // no usable pivot: the block is singular, or not finite in TC (an infinity or a NaN anywhere
        // spreads over the unused rows of its column, or is itself the largest there); the steps run
        // on, with row 0 where there is none, so that the loop stays straight-line code, and the
        // block is discarded
        const int p = key ? 127 - (int)(key & 127u) : 0;
        TC pv = lane_value(x0, p & 63);
        if (NB > 64) pv = p < 64 ? pv : lane_value(x1, p & 63);
        bad = bad || !key || !(fabs(pv) > TC(0) && fabs(pv) < TC(INFINITY));
        u0 = u0 || lane == p;
        u1 = u1 || lane + 64 == p;
        const int pq = (p >> 1) % TR, pa = 2 * ((p >> 1) / TR) + (p & 1);
#pragma unroll
        for (int a = 0; a < RPT; ++a)
            if (a == pa) {   // uniform
                if (own_r == pq) {
#pragma unroll
                    for (int i = 0; i < CPT / 2; ++i) {
                        s_row[tc * (CPT / 2) + i] = V2{i == 0 && tc == jc ? TC(1) : A[a][2 * i], A[a][2 * i + 1]};
                        A[a][2 * i] = TC(0);
                        A[a][2 * i + 1] = TC(0);
                    }
                }
            }
        if (tid == 0) {
            s_piv[k] = (uint8_t)p;
            s_pos[p] = (uint8_t)k;
        }
        const TC ip = TC(1) / pv;
        TC g[RPT];
#pragma unroll
        for (int a = 0; a < RPT; ++a) {
            const bool own = own_r == pq && a == pa;
            if (ROW) g[a] = own ? TC(1) : -f[a / 2][a % 2];
            else g[a] = own ? ip : -f[a / 2][a % 2] * ip;
        }
        group_sync<NW>();
        V2 y[CPT / 2];
#pragma unroll
        for (int i = 0; i < CPT / 2; ++i) {
            y[i] = s_row[tc * (CPT / 2) + i];
            if (ROW) y[i] *= ip;
        }
        TC c0[RPT];
#pragma unroll
        for (int b = 0; b < CPT; ++b)
#pragma unroll
            for (int a = 0; a < RPT; ++a) {
                const TC x = fma(g[a], y[b / 2][b % 2], A[a][b]);
                if (SH == 0) A[a][b] = x;
                else if (b == 0) c0[a] = x;
                else A[a][b - 1] = x;
            }
        if (SH) {
#pragma unroll
            for (int a = 0; a < RPT; ++a) A[a][CPT - 1] = c0[a];
        }
    };
#pragma unroll 1
    for (int kb = 0; kb < NB; kb += CT) {
#pragma unroll 1
        for (int jc = 0; jc < CT - 1; ++jc) step(std::integral_constant<int, 0>{}, kb + jc, jc);
        step(std::integral_constant<int, 1>{}, kb + CT - 1, CT - 1);
    }
    if (bad) {                                                    // uniform per workgroup
        if (tid == 0) gi[cid * GI_STRIDE + GI_STATUS] = 3;   // plain vector store
        return;
    }
    group_sync<NW>();
    int pos[RPT];
#pragma unroll
    for (int a = 0; a < RPT; ++a) pos[a] = s_pos[2 * tr + 2 * TR * (a / 2) + a % 2];
    // inverse(pos(r), piv(k)) = a(r, k), written column-major: the columns tc + CT b of one b at a
    // time, consecutive threads on consecutive rows
    TO* dst = inv + cd.boff + (size_t)slot * NB * NB;
#pragma unroll
    for (int b = 0; b < CPT; ++b) {
        if (act) {
#pragma unroll
            for (int a = 0; a < RPT; ++a) s_out[tc * NB + pos[a]] = A[a][b];
        }
        group_sync<NW>();
        for (int idx = tid; idx < CT * NB / 2; idx += NTH) {
            const int c = idx / (NB / 2), r = 2 * (idx % (NB / 2));
            TO* w = dst + s_piv[c + CT * b] * NB + r;
            typedef TO W2 __attribute__((ext_vector_type(2)));
            *(W2*)w = W2{store_as<TO, TC>(s_out[c * NB + r]), store_as<TO, TC>(s_out[c * NB + r + 1])};
        }
        group_sync<NW>();
    }
}

template <int NB, int NW, class TC, class TO>
fr_status launch_nb(Solver& sv, const GroupArgs& ga, const int* flags, hipStream_t s) {
    hipLaunchKernelGGL((k_block_invert<NB, NW, TC, TO>), dim3(ga.ntiles), dim3(64 * NW), 0, s, ga, sv.d_blk,
                       (TO*)sv.d_inv, sv.d_gi, flags, sv.inv_colour ? 1 : 0);
    FR_HIP(hipGetLastError());
    return FR_OK;
}

// Waves of a 64 x 64 block.  A few blocks take the latency of their 64 steps, which more waves shorten
// until the chip holds more than it can run of them.  us, one / two / four waves (panels in LDS, above):
//     blocks       64               256              512              1,024            2,048
//     FP64  49.8 39.9 38.2   51.2 42.0 40.7   58.3 53.8 50.6   76.6 60.2 67.2   85.6 88.4 104
//           (41.0)           (42.4)           (49.2)           (70.5)           (126)
//     FP32  44.7 35.9 33.3   45.6 37.0 34.9   49.5 44.0 40.1   59.4 48.5 53.2   73.8 65.9 78.5
//           (32.5)           (33.4)           (38.5)           (49.9)           (71.6)
template <class TC> int waves_64(int blocks) {
    return blocks <= 512 ? 4 : blocks <= (sizeof(TC) == 8 ? 1024 : 2048) ? 2 : 1;
}

template <class TC, class TO>
fr_status launch_p(Solver& sv, int p, const GroupArgs& ga, const int* flags, hipStream_t s) {
    switch (p) {
        case 1: return launch_nb<16, 1, TC, TO>(sv, ga, flags, s);
        case 2: return launch_nb<36, 1, TC, TO>(sv, ga, flags, s);
        case 3:
            switch (waves_64<TC>(ga.ntiles)) {
                case 4: return launch_nb<64, 4, TC, TO>(sv, ga, flags, s);
                case 2: return launch_nb<64, 2, TC, TO>(sv, ga, flags, s);
            }
            return launch_nb<64, 1, TC, TO>(sv, ga, flags, s);
        case 4: return launch_nb<100, 4, TC, TO>(sv, ga, flags, s);
    }
    fr_set_error("order outside 1..4");
    return FR_EUNSUPPORTED;
}

}  // namespace

fr_status launch_block_invert_group(Solver& sv, int p, const GroupArgs& ga, int prec, const int* flags,
                                    hipStream_t s) {
    if (ga.ntiles == 0) return FR_OK;
    switch (prec) {
        case FR_FP64: return launch_p<double, double>(sv, p, ga, flags, s);
        case FR_FP32: return launch_p<float, float>(sv, p, ga, flags, s);
        case FR_BF16: return launch_p<float, uint16_t>(sv, p, ga, flags, s);
    }
    fr_set_error("unknown precision");
    return FR_EINVAL;
}
