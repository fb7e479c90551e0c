// The diagonal blocks P_e = inv_dtau Gamma + c_time M - dR_e/dq_e of the Newton operator, written
// down entry by entry from the linearisation packs.
//
// The tangent kernels form a column of a block by sending its unit seed through every stage of the
// residual; almost all of what they add up is zero.  A seed at solution point (a, b) has traces at
// four flux points only, and gradients on its row j = b and its column i = a of points only.  With
// 1-D operators along the rows and columns, the entry for the output point (i, j) is a sum of
// products of point (or flux-point) Jacobians with 1-D weights:
//   every (a, b): the cross derivatives of the viscous terms, one source point on the row of (i, j),
//                 (a, j), one on its column, (i, b), and one flux point on each of its four faces;
//   b = j:        the sources along the row: derivative along xi twice, the inviscid Jacobian at
//                 (a, j), the traces at the two flux points of the row;
//   a = i:        the same along the column;
//   both:         the time terms.
// The stress is linear in the gradient, so a viscous source is seven numbers (visc7: rows of momentum
// and energy, columns u, v, T), from two weights of the fluxes (wf, wg) and two of the gradient.
// Jacobians are computed once per element into LDS (point: f, g and, on moving meshes, q^c; flux
// point: the common flux with respect to the own trace), the weights once per element or lane.
// About 4,000 FP64 instructions per wave and element group at p = 3 in place of 64 columns of 650:
// the blocks of 256 x 256 affine elements take 1.18 ms at p = 3 (3.91 before; writing them alone 0.46).
//
// Work mapping: a workgroup of n waves holds EPB elements, NT lanes each, the same in every wave; wave
// a writes the columns of the seeds (a, b), b = 0..n-1, so that LDS (about 13 KB an element at p = 3)
// feeds n waves and small meshes use n times the waves.  Lanes run along the output points: the 16
// entries of a point pair are stored as 16 contiguous runs of Np doubles.
//
// Not for meshes with boundary faces or with an element that neighbours itself (their seeds reach
// the state beyond a face): those keep the tangent kernel, column by column.
#include "fr_fused.hpp"

namespace {
using namespace fused;

// -(wf f_visc + wg g_visc) of a unit seed in u, v or T whose gradient is (Gx, Gy), added to x:
// rows x-momentum, y-momentum, energy; columns u, v, T: x = (1u, 1v, 2u, 2v, 3u, 3v, 3T).  u, v: the
// velocity at the source.
__device__ __forceinline__ void visc7(const PhysConst& pc, double wf, double wg, double Gx, double Gy, double u,
                                      double v, double* x) {
    const double a = wf * Gx, b = wg * Gy, c = wf * Gy, d = wg * Gx, mu = pc.mu_re;
    const double x1u = -mu * ((4.0 / 3.0) * a + b), x1v = -mu * (d - (2.0 / 3.0) * c);
    const double x2u = -mu * (c - (2.0 / 3.0) * d), x2v = -mu * (a + (4.0 / 3.0) * b);
    x[0] += x1u; x[1] += x1v; x[2] += x2u; x[3] += x2v;
    x[4] += u * x1u + v * x2u;
    x[5] += u * x1v + v * x2v;
    x[6] -= pc.kc_re * (a + b);
}
// the seven numbers into the 4 x 4 entries [row * 4 + column]
__device__ __forceinline__ void add7(const double* x, double* m) {
    m[5] += x[0]; m[6] += x[1]; m[9] += x[2]; m[10] += x[3]; m[13] += x[4]; m[14] += x[5]; m[15] += x[6];
}

// A value the compiler takes as new: the value parts of the dual numbers do not depend on the seed,
// and hoisted out of the loop over the seeds they hold some 200 registers.
__device__ __forceinline__ double fresh(double x) {
    asm volatile("" : "+v"(x));
    return x;
}
__device__ __forceinline__ int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

template <int P, bool VISC, bool MOV>
__global__ void __launch_bounds__(64 * (P + 1), 2) k_assemble(GroupArgs ga, KArgs a, OpTab op) {
    using D = Dual<1>;
    constexpr int n = P + 1, Np = n * n, NF = 4 * n, NT = Sz<P>::NT, EPB = Shape<P, 64>::EPB, nb = 4 * Np;
    constexpr int NM = MOV ? 7 : 5, NJ = MOV ? 48 : 32, SP = EPB * Np, SF = EPB * NF;
    __shared__ double s_m[NM * SP];      // xi_x, xi_y, eta_x, eta_y, 1/|J| (, v_g . grad xi, v_g . grad eta)
    __shared__ double s_J[NJ * SP];      // Jacobians of f, g (, q^c) with respect to q, row * 4 + column
    __shared__ double s_up[2 * SP];      // velocity
    __shared__ double s_gr[VISC ? 2 * n * SP : 1];   // corrected gradient at a point from each seed of its row
    __shared__ double s_gc[VISC ? 2 * n * SP : 1];   // ... of its column
    __shared__ double s_S[3 * SF];       // element-oriented S, S . v_g
    __shared__ double s_N[16 * SF];      // scaled common flux with respect to the own trace
    __shared__ double s_uc[2 * SF];      // common velocity
    __shared__ double s_u[VISC ? 2 * n * SF : 1];    // half the own gradient trace from each seed of the flux point's line
    __shared__ double s_D[n * n], s_lam[2][n], s_gam[2][n];

    const int wv = threadIdx.x / 64, lane = threadIdx.x % 64, el = lane / NT, lt = lane % NT;
    for (int t = threadIdx.x; t < n * n; t += 64 * n) s_D[t] = op.D[t];
    if (threadIdx.x < n) {
        s_lam[0][threadIdx.x] = op.lamL[threadIdx.x]; s_lam[1][threadIdx.x] = op.lamR[threadIdx.x];
        s_gam[0][threadIdx.x] = op.gamL[threadIdx.x]; s_gam[1][threadIdx.x] = op.gamR[threadIdx.x];
    }
    const int tile = blockIdx.x;
    if (tile >= ga.ntiles) return;                                               // uniform per workgroup
    const int lo = find_member(ga, tile);
    const int cid = sld(ga.ids + lo);
    if (a.flags && rfl(a.flags[cid * GI_STRIDE + a.flag])) return;               // uniform per workgroup
    const CaseDev cd = load_case(ga.cases + cid);
    const PhysConst& pc = cd.pc;
    const Geo g = cd.g;
    const int E = cd.E;
    const int e = (tile - sld(ga.pfx + lo)) * EPB + el;
    const bool act = el < EPB && e < E;
    const bool isS = act && lt < Np, isF = act && lt < NF;
    const unsigned EN = (unsigned)E * Np, FE = (unsigned)E * NF;
    const double* fpk = a.fpack + cd.fpoff;
    const double* spk = a.spack + cd.spoff;
    const int i = lt % n, j = lt / n;
    const int eb = el * Np, ef = el * NF;          // the element's part of a point / flux-point field
    auto mk = [](double v, double d) { D r; r.v = v; r.d[0] = d; return r; };

    // ---- Jacobians: the four columns shared out over the waves
    LaneGeo lg;
    double qv[4] = {0.0, 0.0, 0.0, 1.0};
    if (isS) {
        const unsigned id = (unsigned)e * Np + lt;
        lg.xix = ldo(g.sp + G_XIX * EN, id); lg.xiy = ldo(g.sp + G_XIY * EN, id);
        lg.etx = ldo(g.sp + G_ETX * EN, id); lg.ety = ldo(g.sp + G_ETY * EN, id);
        lg.ij = ldo(g.sp + G_IJ * EN, id);
        lg.ug = MOV ? ldo(g.sp + G_UG * EN, id) : 0.0;
        lg.vg = MOV ? ldo(g.sp + G_VG * EN, id) : 0.0;
        double tau[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) qv[vv] = ldo(spk + (size_t)vv * EN, id);
        if (VISC) {
#pragma unroll
            for (int c = 0; c < 3; ++c) tau[c] = ldo(spk + (size_t)(4 + c) * EN, id);
        }
        if (wv == 0) {
            s_m[0 * SP + eb + lt] = lg.xix; s_m[1 * SP + eb + lt] = lg.xiy;
            s_m[2 * SP + eb + lt] = lg.etx; s_m[3 * SP + eb + lt] = lg.ety;
            s_m[4 * SP + eb + lt] = lg.ij;
            if constexpr (MOV) {
                s_m[5 * SP + eb + lt] = lg.ug * lg.xix + lg.vg * lg.xiy;
                s_m[6 * SP + eb + lt] = lg.ug * lg.etx + lg.vg * lg.ety;
            }
            s_up[eb + lt] = qv[1];
            s_up[SP + eb + lt] = qv[2];
        }
#pragma unroll 1
        for (int w = wv; w < 4; w += n) {
            D qs[4], fl[4], gl[4], qc[4];
#pragma unroll
            for (int vv = 0; vv < 4; ++vv) qs[vv] = mk(fresh(qv[vv]), vv == w ? 1.0 : 0.0);
            fr_point_flux<D, false>(pc, qs, nullptr, nullptr, nullptr, fl, gl, qc);
            double ft[4], gt[4];
#pragma unroll
            for (int vv = 0; vv < 4; ++vv) { ft[vv] = fl[vv].d[0]; gt[vv] = gl[vv].d[0]; }
            if (VISC) {
                // the work of the stresses
                ft[3] -= qs[1].d[0] * tau[0] + qs[2].d[0] * tau[2];
                gt[3] -= qs[1].d[0] * tau[2] + qs[2].d[0] * tau[1];
            }
#pragma unroll
            for (int vv = 0; vv < 4; ++vv) {
                s_J[(vv * 4 + w) * SP + eb + lt] = ft[vv];
                s_J[(16 + vv * 4 + w) * SP + eb + lt] = gt[vv];
                if constexpr (MOV) s_J[(32 + vv * 4 + w) * SP + eb + lt] = qc[vv].d[0];
            }
        }
    }
    if (isF) {
        const unsigned sid = (unsigned)e * NF + lt;
        const double nx = ldo(g.fp + F_NX * FE, sid), ny = ldo(g.fp + F_NY * FE, sid), sc = ldo(g.fp + F_SC * FE, sid);
        const double cc = VISC ? ldo(g.fp + F_CC * FE, sid) : 0.0;
        const double fug = MOV ? ldo(g.fp + F_UG * FE, sid) : 0.0, fvg = MOV ? ldo(g.fp + F_VG * FE, sid) : 0.0;
        double qm[4], qp[4];
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) {
            qm[vv] = ldo(fpk + (size_t)vv * FE, sid);
            qp[vv] = ldo(fpk + (size_t)(4 + vv) * FE, sid);
        }
        const double tnx = VISC ? ldo(fpk + (size_t)8 * FE, sid) : 0.0, tny = VISC ? ldo(fpk + (size_t)9 * FE, sid) : 0.0;
        const double qcu = 0.5 * (qm[1] + qp[1]), qcv = 0.5 * (qm[2] + qp[2]);
        if (wv == 0) {
            s_S[0 * SF + ef + lt] = sc * nx;
            s_S[1 * SF + ef + lt] = sc * ny;
            s_S[2 * SF + ef + lt] = MOV ? sc * (fug * nx + fvg * ny) : 0.0;
            s_uc[ef + lt] = qcu;
            s_uc[SF + ef + lt] = qcv;
        }
#pragma unroll 1
        for (int w = wv; w < 4; w += n) {
            D dm[4], dp[4], fn[4], dq[4];
#pragma unroll
            for (int vv = 0; vv < 4; ++vv) {
                dm[vv] = mk(fresh(qm[vv]), vv == w ? 1.0 : 0.0);
                dp[vv] = mk(fresh(qp[vv]), 0.0);
            }
            fr_common_inviscid<D>(pc, dm, dp, nx, ny, fug, fvg, fn, dq);
            double ft[4] = {0.0, 0.0, 0.0, 0.0};
            if (VISC) {
                const double gs[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
                double dqt[4], dqh[3];
#pragma unroll
                for (int vv = 0; vv < 4; ++vv) dqt[vv] = -dm[vv].d[0];
                fr_common_viscous_tan(pc, dqt, qcu, qcv, 0.5 * dm[1].d[0], 0.5 * dm[2].d[0], tnx, tny, gs, nx, ny, cc, ft,
                                      dqh);
            }
#pragma unroll
            for (int vv = 0; vv < 4; ++vv) s_N[(vv * 4 + w) * SF + ef + lt] = sc * (fn[vv].d[0] + ft[vv]);
        }
    }
    __syncthreads();
    // ---- gradient weights, four tasks over the waves.  Corrected gradient: the chain rule plus the
    // lift of half the jump; trace gradient: of the uncorrected one
#pragma unroll 1
    for (int task = wv; VISC && task < 4; task += n) {
        if (task < 2 && isS) {
            const bool row = task == 0;
            const int d = row ? i : j;                               // position along the seeds' line
            const int f0 = row ? j : 2 * n + i, f1 = f0 + n;         // the line's two flux points
            const double mx = row ? lg.xix : lg.etx, my = row ? lg.xiy : lg.ety;
            const double l0 = 0.5 * lg.ij * s_gam[0][d], l1 = 0.5 * lg.ij * s_gam[1][d];
            const double S0x = s_S[ef + f0], S1x = s_S[ef + f1], S0y = s_S[SF + ef + f0], S1y = s_S[SF + ef + f1];
            double* dst = row ? s_gr : s_gc;
#pragma unroll
            for (int s = 0; s < n; ++s) {
                const double Ds = s_D[d * n + s], c0 = l0 * s_lam[0][s], c1 = l1 * s_lam[1][s];
                dst[s * SP + eb + lt] = mx * Ds - (c0 * S0x + c1 * S1x);
                dst[(n + s) * SP + eb + lt] = my * Ds - (c0 * S0y + c1 * S1y);
            }
        }
        if (task >= 2 && isF) {
            const int f = lt / n, k = lt % n, c = (f < 2 ? 0 : 2) + task - 2;   // metric of the line's direction
            for (int s = 0; s < n; ++s) {
                double acc = 0.0;
#pragma unroll
                for (int m = 0; m < n; ++m)
                    acc += s_lam[f & 1][m] * s_m[c * SP + eb + line_pt(n, f, k, m)] * s_D[m * n + s];
                s_u[((task - 2) * n + s) * SF + ef + lt] = 0.5 * acc;
            }
        }
    }
    __syncthreads();
    if (!isS) return;   // (no barrier follows)
    double ct = a.c_time, idt = a.inv_dtau;
    if (a.cstep) { ct = rfl(a.cstep[cid].ct); idt = rfl(a.cstep[cid].idt); }
    // ---- weights of the lane's own output point (i, j)
    const double h0 = lg.ij * s_gam[0][i], h1 = lg.ij * s_gam[1][i], h2 = lg.ij * s_gam[0][j], h3 = lg.ij * s_gam[1][j];
    const int fp0 = ef + j, fp1 = ef + n + j, fp2 = ef + 2 * n + i, fp3 = ef + 3 * n + i;
    const double S0x = s_S[fp0], S1x = s_S[fp1], S0y = s_S[SF + fp0], S1y = s_S[SF + fp1];
    const double S2x = s_S[fp2], S3x = s_S[fp3], S2y = s_S[SF + fp2], S3y = s_S[SF + fp3];
    // inv_dtau Gamma + c_time M at the point
    double tA, tT, tr, th;
    {
        const double iT = rcp(qv[3]), rho = qv[0] * pc.inv_Rg * iT;
        const double Ur2 = fr_ur2<double>(pc, qv[1] - lg.ug, qv[2] - lg.vg, pc.gRg * qv[3]);
        tA = idt * (rcp(Ur2) + pc.inv_Cp * iT) + ct * (pc.inv_Rg * iT);
        tT = -(idt + ct) * rho * iT;
        tr = (idt + ct) * rho;
        th = pc.Cp * qv[3] + 0.5 * (qv[1] * qv[1] + qv[2] * qv[2]);
    }
    // ---- the seeds (sa, b) of this wave.  The weights of the row source (sa, j):
    double* out = a.out + cd.boff + (size_t)e * nb * nb + lt;
    const int sa = wv;
    const double Da = s_D[i * n + sa], c0 = h0 * s_lam[0][sa], c1 = h1 * s_lam[1][sa];
    const double wf_ = lg.xix * Da - (c0 * S0x + c1 * S1x), wg_ = lg.xiy * Da - (c0 * S0y + c1 * S1y);
    const int rs_ = eb + sa + n * j, f01 = ef + j, f23 = ef + 2 * n + i;
#pragma unroll 1
    for (int b = 0; b < n; ++b) {
        const double Db = s_D[j * n + b], l2 = s_lam[0][b], l3 = s_lam[1][b], c2 = h2 * l2, c3 = h3 * l3;
        const int cs = eb + i + n * b;   // the column source (i, b) and its weights
        const double vf = lg.etx * Db - (c2 * S2x + c3 * S3x), vg = lg.ety * Db - (c2 * S2y + c3 * S3y);
        double m[16], x[7];
        // (as new in every round: what depends on them and not on b, LDS reads above all, is not worth
        // the registers that hold it)
        const int rs = fresh(rs_), fp0 = fresh(f01), fp1 = fp0 + n, fp2 = fresh(f23), fp3 = fp2 + n;
        const double wf = fresh(wf_), wg = fresh(wg_), p0 = fresh(h0), p1 = fresh(h1), p2 = fresh(h2), p3 = fresh(h3);
#pragma unroll
        for (int t = 0; t < 16; ++t) m[t] = 0.0;
        if constexpr (VISC) {
            const double l0 = s_lam[0][sa], l1 = s_lam[1][sa];
            const double ex = 0.5 * s_m[2 * SP + rs], ey = 0.5 * s_m[3 * SP + rs];
            const double gx = 0.5 * s_m[0 * SP + cs], gy = 0.5 * s_m[1 * SP + cs];
#pragma unroll
            for (int t = 0; t < 7; ++t) x[t] = 0.0;
            visc7(pc, p0 * S0x, p0 * S0y, (l0 * Db) * ex, (l0 * Db) * ey, s_uc[fp0], s_uc[SF + fp0], x);
            visc7(pc, p1 * S1x, p1 * S1y, (l1 * Db) * ex, (l1 * Db) * ey, s_uc[fp1], s_uc[SF + fp1], x);
            __builtin_amdgcn_sched_barrier(0);
            visc7(pc, p2 * S2x, p2 * S2y, (l2 * Da) * gx, (l2 * Da) * gy, s_uc[fp2], s_uc[SF + fp2], x);
            visc7(pc, p3 * S3x, p3 * S3y, (l3 * Da) * gx, (l3 * Da) * gy, s_uc[fp3], s_uc[SF + fp3], x);
            __builtin_amdgcn_sched_barrier(0);
            visc7(pc, wf, wg, s_gc[b * SP + rs], s_gc[(n + b) * SP + rs], s_up[rs], s_up[SP + rs], x);
            visc7(pc, vf, vg, s_gr[sa * SP + cs], s_gr[(n + sa) * SP + cs], s_up[cs], s_up[SP + cs], x);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (b == j) {   // the sources along the row
            const double wq = MOV ? c0 * s_S[2 * SF + fp0] + c1 * s_S[2 * SF + fp1] - s_m[(MOV ? 5 : 0) * SP + eb + lt] * Da : 0.0;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                if (t % 4 == 0) __builtin_amdgcn_sched_barrier(0);   // (not all 64 reads at once)
                double c = wf * s_J[t * SP + rs] + wg * s_J[(16 + t) * SP + rs];
                if (MOV) c += wq * s_J[(MOV ? 32 + t : 0) * SP + rs];
                m[t] += c + c0 * s_N[t * SF + fp0] + c1 * s_N[t * SF + fp1];
            }
            if constexpr (VISC) {
#pragma unroll 1
                for (int k = 0; k < n; ++k) {
                    const int src = eb + k + n * j;
                    const double Dk = s_D[i * n + k], d0 = p0 * s_lam[0][k], d1 = p1 * s_lam[1][k];
                    visc7(pc, lg.xix * Dk - (d0 * S0x + d1 * S1x), lg.xiy * Dk - (d0 * S0y + d1 * S1y),
                          s_gr[sa * SP + src], s_gr[(n + sa) * SP + src], s_up[src], s_up[SP + src], x);
                }
                visc7(pc, p0 * S0x, p0 * S0y, s_u[sa * SF + fp0], s_u[(n + sa) * SF + fp0], s_uc[fp0], s_uc[SF + fp0], x);
                visc7(pc, p1 * S1x, p1 * S1y, s_u[sa * SF + fp1], s_u[(n + sa) * SF + fp1], s_uc[fp1], s_uc[SF + fp1], x);
            }
        }
        if (sa == i) {   // the sources along the column
            const double wq = MOV ? c2 * s_S[2 * SF + fp2] + c3 * s_S[2 * SF + fp3] - s_m[(MOV ? 6 : 0) * SP + eb + lt] * Db : 0.0;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                if (t % 4 == 0) __builtin_amdgcn_sched_barrier(0);   // (not all 64 reads at once)
                double c = vf * s_J[t * SP + cs] + vg * s_J[(16 + t) * SP + cs];
                if (MOV) c += wq * s_J[(MOV ? 32 + t : 0) * SP + cs];
                m[t] += c + c2 * s_N[t * SF + fp2] + c3 * s_N[t * SF + fp3];
            }
            if constexpr (VISC) {
#pragma unroll 1
                for (int k = 0; k < n; ++k) {
                    const int src = eb + i + n * k;
                    const double Dk = s_D[j * n + k], d2 = p2 * s_lam[0][k], d3 = p3 * s_lam[1][k];
                    visc7(pc, lg.etx * Dk - (d2 * S2x + d3 * S3x), lg.ety * Dk - (d2 * S2y + d3 * S3y),
                          s_gc[b * SP + src], s_gc[(n + b) * SP + src], s_up[src], s_up[SP + src], x);
                }
                visc7(pc, p2 * S2x, p2 * S2y, s_u[b * SF + fp2], s_u[(n + b) * SF + fp2], s_uc[fp2], s_uc[SF + fp2], x);
                visc7(pc, p3 * S3x, p3 * S3y, s_u[b * SF + fp3], s_u[(n + b) * SF + fp3], s_uc[fp3], s_uc[SF + fp3], x);
            }
            if (b == j) {   // time terms
                const double u = s_up[eb + lt], v = s_up[SP + eb + lt];
                m[0] += tA;                 m[3] += tT;
                m[4] += u * tA; m[5] += tr; m[7] += u * tT;
                m[8] += v * tA; m[10] += tr; m[11] += v * tT;
                m[12] += th * tA - (idt + ct); m[13] += tr * u; m[14] += tr * v; m[15] += th * tT + tr * pc.Cp;
            }
        }
        if constexpr (VISC) add7(x, m);
        const int col = sa + n * b;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
#pragma unroll
            for (int vv = 0; vv < 4; ++vv) out[(size_t)(w * Np + col) * nb + vv * Np] = m[vv * 4 + w];
        }
    }
}

template <int P>
fr_status assemble_p(const Solver& sv, const Group& gr, const KArgs& a, hipStream_t s) {
    GroupArgs ga;
    ga.cases = sv.d_cases;
    ga.ids = gr.d_ids;
    ga.pfx = gr.tile_pfx(Shape<P, 64>::EPB);
    ga.nmem = (int)gr.ids.size();
    ga.ntiles = gr.ntiles(Shape<P, 64>::EPB);
    ga.xcd = 0;
    if (!ga.pfx) { fr_set_error("tile prefix missing"); return FR_EINVAL; }
    if (ga.ntiles == 0) return FR_OK;
    const OpTab& op = sv.cs[gr.ids[0]]->op;
    const dim3 grid(ga.ntiles), block(64 * (P + 1));
    if (gr.visc) {
        if (gr.mov) hipLaunchKernelGGL((k_assemble<P, true, true>), grid, block, 0, s, ga, a, op);
        else hipLaunchKernelGGL((k_assemble<P, true, false>), grid, block, 0, s, ga, a, op);
    } else {
        if (gr.mov) hipLaunchKernelGGL((k_assemble<P, false, true>), grid, block, 0, s, ga, a, op);
        else hipLaunchKernelGGL((k_assemble<P, false, false>), grid, block, 0, s, ga, a, op);
    }
    FR_HIP(hipGetLastError());
    return FR_OK;
}

}  // namespace

fr_status launch_direct_assembly(const Solver& sv, const Group& gr, const KArgs& a, hipStream_t s) {
    if (!a.fpack || !a.spack || !a.out) { fr_set_error("block assembly without packs"); return FR_EINVAL; }
    switch (gr.p) {
        case 1: return assemble_p<1>(sv, gr, a, s);
        case 2: return assemble_p<2>(sv, gr, a, s);
        case 3: return assemble_p<3>(sv, gr, a, s);
        case 4: return assemble_p<4>(sv, gr, a, s);
    }
    fr_set_error("order outside 1..4");
    return FR_EUNSUPPORTED;
}
