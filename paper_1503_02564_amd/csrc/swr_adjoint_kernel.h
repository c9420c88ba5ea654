// swr_adjoint_kernel.h -- discrete adjoint of the subdomain Crank-Nicolson
// scheme, solved through the same Schwarz decomposition (static real potential,
// Robin and S0^2), in the row form of the sweep (swr_rows.h).  Included by the
// translation units that instantiate it for one row count each.
//
// Forward (eq. CNS_L with P1): A v_n = c M u_{n-1}, u_n = 2 v_n - u_{n-1},
// A = c M - S + M_V complex symmetric.  For a real objective J(u_nt) with
// upstream gradient gbar = dJ/dRe + i dJ/dIm, write P_n for the conjugate of
// the gradient with respect to u_n.  The chain rule gives
//   P_nt = conj(gbar);  A Q_n = P_n;  P_{n-1} = 2 c M Q_n - P_n;
//   dJ/dV_i = -2 Re sum_n Q_n^T (dM_V/dV_i) v_n,   dJ/du0 = conj(P_0).
// With w = P this is the forward recursion written on dual vectors
// (A x = w_prev, w_new = 2 c M x - w_prev): the same subdomain matrices, the
// same transmission and so the same interface operator L; only the data
// differ.  Subdomain k carries the local part w_k of the assembled dual vector
// (a node shared by two subdomains is split half/half; the split only changes
// the iterates, not the converged result); the S0^2 history starts from
// v_0 = 0 on both sides of every interface.  Matrix and w are held over
// i kappa as in the sweep, so that w_new = 2 stencil(x) - w.
//
// Without gradient a launch is the dual sweep (d of the adjoint interface
// problem).  With gradient it walks the 64-step segments of the adjoint time
// m = nt - n + 1 in order; for each it first replays the forward steps from a
// checkpoint of u (stored by the forward final sweep every 64 steps counted
// back from nt), with the boundary sums (S0^2 history less flux) that sweep
// stored, keeping the forward v_n of the segment in a per-task buffer; then it
// advances the adjoint over the segment, consuming v_n in reverse.  With
// r_i = sum over time of Re Q_i v_i and c_i of Re (Q_i v_{i+1} + Q_{i+1} v_i),
//   dJ/dV_i = -h/6 ((r_{i-1} + 3 r_i + c_{i-1}) + (3 r_i + r_{i+1} + c_i)),
// one bracket per element at the node, so a step adds six multiply-adds a node.
//
// Bound: FP64 issue of two solves a step (replay and adjoint), and beside it
// the segment buffer's write and read, 16 bytes a node each.  In the 64-lane
// form (one wave per task, history of both sweeps summed anew in every segment,
// 18 complex products a node for dJ/dV) the two launches for 16 potentials on
// 256 x 64 cells over 2000 steps took 26.2 ms; now 8.5 ms in 16 launches and 1.9 ms for
// the old history parts.
#pragma once
#include "swr_sweep_rows_kernel.h"

namespace swr {

template <int P, int RW, bool LDSF, int NW, int TR>
__device__ inline void adj_body(const AdjArgs& a, int first, int count, cd* smem) {
    constexpr int T = 16 * RW, SLOTS = 4 / RW;
    constexpr bool WRAP = P == 1;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = NW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : 0;
    const int t = lane % T;
    const int slot0 = wv * SLOTS, mine = slot0 + lane / T;
    // LDS as in rows_body: [beta window][per wave: v left, v right, sums left, sums right][record]
    double* sb = reinterpret_cast<double*>(smem);
    cd* lg = smem + kRowsBetaLds / 2 + wv * kRowsWaveLds;
    cd* sfac = smem + kRowsBetaLds / 2 + NW * kRowsWaveLds;
    const int nt = a.nt;
    if (TR == TR_S02) {
        const int nbeta = max(nt, kWave) + kWave + 1;
        for (int i = threadIdx.x; i < kRowsBetaLds; i += NW * kWave) sb[i] = i < nbeta ? a.beta[i] : 0.0;
    }
    if (LDSF) {
        const cd* src = a.fac + (size_t)a.tasks[first].f * a.fstride;
        for (int i = threadIdx.x; i < rows_fields(P, RW) * T; i += NW * kWave) sfac[i] = src[i];
    }
    __syncthreads();
    if (NW > 1 && slot0 >= count) return;             // no later workgroup barrier
    const bool live = mine < count;                   // else: repeats the last task, writes nothing
    const int tix = first + min(mine, count - 1);
    const Task task = a.tasks[tix];
    const int k = task.k, b = task.b;
    const int n = a.J[k] + 1, o = a.off[k];
    const bool lif = k > 0, rif = k < a.N - 1;
    const int tl = P > 1 ? T - 1 : n - 1;             // lane of node n - 1 (slot P - 1)
    int s;
    bool dup;
    rows_place<P, RW>(n, t, s, dup);
    const cd zero = mk(0, 0);
    const bool t0 = t == 0, tL = t == tl;
    const int jr = P > 1 ? T - 1 - t : (tl - t) & (T - 1);   // output step of my right sum

    RowsFac<P, RW, LDSF> F;
    F.lds = sfac + t;
    F.load(a.fac + (size_t)task.f * a.fstride + t);

    const double ik = 1.0 / a.kappa;
    cd* const stp = a.state ? a.state + (size_t)tix * 2 * a.pstride * kWave + t : nullptr;
    cd w[P];
    double sp[P], sc[P];                              // sums r_i and c_i of my slots
    if (a.m_begin == 0) {
        // conj(gbar) / (i kappa), split half/half at interface nodes
        const cd* gb = a.gbar + (size_t)b * a.nx + o;
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int i = s + q;
            cd v = zero;
            if (i < n) v = gb[i];
            if ((i == 0 && lif) || (i == n - 1 && rif)) v = 0.5 * v;
            w[q] = mk(-v.y * ik, -v.x * ik);
            sp[q] = sc[q] = 0.0;
        }
    } else {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            w[q] = stp[q * T];
            const cd x = stp[(P + q) * T];
            sp[q] = x.x;
            sc[q] = x.y;
        }
    }
    const double w0 = t0 ? 2.0 : 4.0;
    const double wL = (tL || (P == 1 && t0)) ? 2.0 : 4.0;
    const cd cc = TR == TR_S02 ? a.c2 : mk(1, 0);
    const cd cs = mk(cc.y * ik, -cc.x * ik);
    const cd ic = TR == TR_S02 ? inv(a.c2) : mk(1, 0);
    double bl = 0.0, br = 0.0;                        // beta of my lag in the two running sums
    if (TR == TR_S02) {
        bl = a.beta[t + 1];
        br = a.beta[jr + 1];
    }
    const bool ml = lif && t0, mr = rif && tL;
    cd* lgl = lg + (lane - t);
    cd* const Ha = TR == TR_S02 ? a.hist + (size_t)tix * 2 * (nt + 1) : nullptr;
    if (TR == TR_S02 && a.m_begin == 0 && live && t0) { Ha[0] = zero; Ha[nt + 1] = zero; }
    cd* const seg = a.grad ? a.seg + (size_t)tix * kWave * a.pstride * kWave + t : nullptr;

    for (int m0 = a.m_begin; m0 < a.m_end; m0 += kWave) {
        const int ns = min(kWave, a.m_end - m0);      // steps of the segment
        if (a.grad) {
            // ---- replay forward steps nsf+1 .. nsf+ns from the checkpoint ----
            const int jj = m0 / kWave + 1;
            const int nsf = max(0, nt - kWave * jj);
            const cd* ck = a.ckpt + ((size_t)tix * (a.Jc + 1) + jj) * a.pstride * kWave;   // by node
            const cd* bs = a.bsum + (size_t)tix * 2 * nt + nsf;
            cd u[P];
#pragma unroll
            for (int q = 0; q < P; ++q) {
                u[q] = zero;
                if (s + q < n) u[q] = ck[s + q];
            }
            for (int i0 = 0; i0 < ns; i0 += T) {
                const int nb = min(T, ns - i0);
                cd accA = zero, accB = zero;
                if (lif && t < nb) accA = bs[i0 + t];
                if (rif && jr < nb) accB = bs[nt + i0 + jr];
                cd* sg = seg + (size_t)i0 * P * T;
                for (int i = 0; i < nb; ++i, sg += P * T) {
                    const cd uL = rows_up1<RW>(u[P - 1], t);
                    const cd uR = rows_dn1<RW>(rows_front<P>(u, dup), t);
                    auto stencil = [&](int q) { return rows_stencil<P>(u, uL, uR, w0, wL, q); };
                    cd dF = stencil(0), dS = P > 1 ? stencil(P - 1) : zero;
                    if (ml) dF = madd_x(dF, cs, accA);
                    if (P == 1) dS = dF;
                    if (mr) dS = madd_x(dS, cs, accB);
                    cd x[P];
                    rows_solve(F, dF, dS, stencil, t, dup, x);
#pragma unroll
                    for (int q = 0; q < P; ++q) {
                        u[q] = mk(2.0 * x[q].x - u[q].x, 2.0 * x[q].y - u[q].y);
                        if (live) sg[q * T] = x[q];
                    }
                    accA = rows_roll_dn<RW>(accA);
                    accB = rows_roll_up<RW, WRAP>(accB);
                }
            }
        }
        // ---- adjoint steps m0+1 .. m0+ns; v of the last replayed step first ----
        cd v[P];
        if (a.grad) {
#pragma unroll
            for (int q = 0; q < P; ++q) v[q] = seg[((size_t)(ns - 1) * P + q) * T];
        }
        for (int n0 = m0; n0 < m0 + ns; n0 += T) {
            const int nb = min(T, m0 + ns - n0);
            const size_t gi = ((size_t)b * a.ns + 2 * k) * nt + n0;
            const bool okl = t < nb, okr = jr < nb;
            cd accA = zero, accB = zero;
            if (TR == TR_S02) {
                __threadfence_block();
                rows_far<RW>(a.hist, a.beta, nt, a.far_old != nullptr, first + slot0, count - slot0, n0, sb, lg);
                rows_fence();
                accA = lg[lane];
                accB = lg[kWave + lane - t + jr];
                rows_fence();
                const int C = n0 - n0 % kFarSuper;
                if (a.far_old && C > 0) {
                    const cd* fo = a.far_old + (size_t)tix * 2 * kFarSuper + (n0 - C);
                    accA = accA + fo[t];
                    accB = accB + fo[kFarSuper + jr];
                }
            }
            if (a.g_in) {
                cd l = zero, rr = zero;
                if (lif && okl) l = a.g_in[gi - nt + t];
                if (rif && okr) rr = a.g_in[gi + jr];
                accA = accA - ic * l;
                accB = accB - ic * rr;
            }
            for (int i = 0; i < nb; ++i) {
                cd dF = w[0], dS = w[P - 1];
                if (ml) {
                    dF = madd_x(dF, cs, accA);
                    lgl[2 * kWave + i] = accA;
                }
                if (P == 1) dS = dF;
                if (mr) {
                    dS = madd_x(dS, cs, accB);
                    lgl[3 * kWave + i] = accB;
                }
                cd x[P];
                rows_solve(F, dF, dS, [&](int q) { return w[q]; }, t, dup, x);
                const cd xL = rows_up1<RW>(x[P - 1], t);
                const cd xR = rows_dn1<RW>(rows_front<P>(x, dup), t);
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    const cd m = rows_stencil<P>(x, xL, xR, w0, wL, q);
                    w[q] = mk(2.0 * m.x - w[q].x, 2.0 * m.y - w[q].y);
                }
                if (a.grad) {
                    const cd vR = rows_dn1<RW>(rows_front<P>(v, dup), t);
#pragma unroll
                    for (int q = 0; q < P; ++q) {
                        const cd xn = sel_c(q == P - 1, xR, x[q == P - 1 ? 0 : q + 1]);
                        const cd vn = sel_c(q == P - 1, vR, v[q == P - 1 ? 0 : q + 1]);
                        sp[q] = fma(x[q].x, v[q].x, fma(-x[q].y, v[q].y, sp[q]));
                        sc[q] = fma(x[q].x, vn.x, fma(-x[q].y, vn.y, sc[q]));
                        sc[q] = fma(xn.x, v[q].x, fma(-xn.y, v[q].y, sc[q]));
                    }
                    // the next step's v, read while that step is solved
                    const int is = ns - 2 - (n0 - m0 + i);
                    if (is >= 0) {
#pragma unroll
                        for (int q = 0; q < P; ++q) v[q] = seg[((size_t)is * P + q) * T];
                    }
                }
                if (t0) lgl[i] = x[0];
                if (tL) lgl[kWave + i] = x[P - 1];
                accA = rows_roll_dn<RW>(accA);
                accB = rows_roll_up<RW, WRAP>(accB);
                if (TR == TR_S02) {
                    const cd va = rows_first<RW>(x[0]), vb = rows_last<RW, P>(x[P - 1], tl);
                    accA = mk(fma(bl, va.x, accA.x), fma(bl, va.y, accA.y));
                    accB = mk(fma(br, vb.x, accB.x), fma(br, vb.y, accB.y));
                }
            }
            // the block's outputs, as in rows_body
            rows_fence();
            const cd va = lg[lane], vb = lg[kWave + lane], sa = lg[2 * kWave + lane], se = lg[3 * kWave + lane];
            rows_fence();
            if (okl && live) {
                if (TR == TR_S02) {
                    Ha[n0 + 1 + t] = va;
                    Ha[nt + 1 + n0 + 1 + t] = vb;
                }
                auto put = [&](cd sum, cd y, size_t in, size_t out) {
                    cd l = zero;
                    if (a.g_in) l = a.g_in[in];
                    a.g_out[out] = TR == TR_S02 ? 2.0 * madd(cc * sum, a.sigma, y) + l : 2.0 * (a.sigma * y) - l;
                };
                if (lif && a.g_out) put(sa, va, gi - nt + t, gi - 2 * (size_t)nt + t);
                if (rif && a.g_out) put(se, vb, gi + t, gi + nt + t);
            }
        }
    }

    if (a.m_end < nt) {
        if (stp && live) {
#pragma unroll
            for (int q = 0; q < P; ++q) {
                stp[q * T] = w[q];
                stp[(P + q) * T] = mk(sp[q], sc[q]);
            }
        }
    } else if (a.grad) {
        double* dV = a.dV + (size_t)b * a.nx + o;
        cd* du = a.du0 + (size_t)b * a.nx + o;
        const double spL = rows_up1<RW>(mk(sp[P - 1], 0), t).x, scL = rows_up1<RW>(mk(sc[P - 1], 0), t).x;
        const double spF = sel_c(P > 1 && dup, mk(sp[P > 1 ? 1 : 0], 0), mk(sp[0], 0)).x;
        const double spR = rows_dn1<RW>(mk(spF, 0), t).x;
        const size_t en = ((size_t)b * a.N + k) * 2;
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int i = s + q;
            const double pm = q == 0 ? spL : sp[q == 0 ? 0 : q - 1], cm = q == 0 ? scL : sc[q == 0 ? 0 : q - 1];
            const double pp = q == P - 1 ? spR : sp[q == P - 1 ? 0 : q + 1];
            double g = 0.0;
            if (i > 0) g += pm + 3.0 * sp[q] + cm;
            if (i < n - 1) g += 3.0 * sp[q] + pp + sc[q];
            g *= -a.h / 6.0;
            const cd wq = a.kappa * mul_i(w[q]);
            if (!live || i >= n || (q == 0 && dup)) continue;
            if (i > 0 && i < n - 1) {
                dV[i] = g;
                du[i] = conjc(wq);
            } else {
                const int e = i == 0 ? 0 : 1;
                a.gends[en + e] = g;
                a.wends[en + e] = wq;
            }
        }
    }
}

template <int P, int PHI, int RW, bool LDSF, int NW, int TR>
__device__ inline void adj_pick(const AdjArgs& a, int first, int count, int p, cd* smem) {
    if (p == P) adj_body<P, RW, LDSF, NW, TR>(a, first, count, smem);
    else if constexpr (P < PHI) adj_pick<P + 1, PHI, RW, LDSF, NW, TR>(a, first, count, p, smem);
}

// widths PLO .. PHI of one row count; NW waves per workgroup
template <int RW, int PLO, int PHI, bool LDSF, int NW, int WPE, int TR>
__global__ __launch_bounds__(NW * kWave, WPE) void adjoint_rows_kernel(AdjArgs a) {
    extern __shared__ cd smem[];
    const int4 it = a.items[blockIdx.x];              // first task, tasks, P
    adj_pick<PLO, PHI, RW, LDSF, NW, TR>(a, it.x, it.y, it.z, smem);
}

template <int RW, int PLO, int PHI, bool LDSF, int NW, int WPE>
hipError_t launch_adj(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    if (trans == TR_S02) adjoint_rows_kernel<RW, PLO, PHI, LDSF, NW, WPE, TR_S02><<<nitems, NW * kWave, lds, st>>>(a);
    else adjoint_rows_kernel<RW, PLO, PHI, LDSF, NW, WPE, TR_ROBIN><<<nitems, NW * kWave, lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
