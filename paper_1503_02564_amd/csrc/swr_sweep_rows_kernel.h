// swr_sweep_rows_kernel.h -- subdomain sweep of a static potential with Robin
// or S0^2 transmission, RW rows of 16 lanes per task (swr_rows.h).  Included by
// the translation units that instantiate it for one row count each.
//
// Every width (nodes per lane) of a task list runs in one launch: the
// workgroup's item names its tasks and its P, and the kernel branches to that
// width's code.  (One launch per width, as before, ran the widths of an
// uneven decomposition one after the other on a stream.)
//
// Time runs in blocks of T = 16 RW steps, lane t of a task carrying output
// step t of the block.  S0^2 history of the block's outputs, sum over q <= n of
// beta_{n-q} v_q:
//   * terms up to the block start n0: one product on the matrix cores per
//     block (v_mfma_f64_16x16x4_f64), A the Toeplitz block of beta, B the
//     boundary values.  The 16 columns are (16-step part of the block, task,
//     end, re / im): part s takes the sources q + 16 s for its outputs j + 16 s,
//     so all parts share A.  Sources older than the 256-step super-chunk come
//     summed from far_old_kernel.
//   * terms inside the block: after every step the running sums move one lane
//     towards the end they are for (lane 0: left, lane T - 1: right) and add
//     beta_{lag} times the new boundary value, lag fixed per lane.
// The boundary terms of a step are then formed by the two end lanes alone.
// The incoming flux is folded into the running sum (Robin: it is all of it).
//
// Bound: FP64 issue.  Per step and wave about 26 instructions per node slot
// (P) plus 130 to 190 that do not depend on P; a wave carries 4 / RW tasks, so
// batches take fewer rows per task (rule in swr_rows_plan.h).  Against one wave per
// task with a 64-lane reduction and one launch per width (before): 32 problems on
// 500 uneven subdomains over 2000 steps 103.5 -> 75 ms per solve (67 with the
// interface products' later forms), gradient of 16 potentials on 256 x 64 cells 148
// -> 111 ms, one problem on 64 x 256 cells 3.59 -> 3.1 ms, one Robin iteration on 4
// x 100 cells over 500 steps 0.367 -> 0.275 ms.
#pragma once
#include <type_traits>

#include "swr_rows.h"

namespace swr {

constexpr int kRowsBetaLds = 324;       // beta_0 .. of the in-super-chunk products
constexpr int kRowsWaveLds = 4 * kWave; // complex values per wave: logs of v and of the running sums

// LDS of a workgroup: [beta window][logs of each wave][record]
inline size_t rows_lds_bytes(const RowsKind& k, int pmax) {
    return sizeof(cd) * (kRowsBetaLds / 2 + (size_t)k.waves * kRowsWaveLds +
                         (k.lds ? (size_t)rows_fields(pmax, k.RW) * 16 * k.RW : 0));
}

typedef double rows_f64x4 __attribute__((ext_vector_type(4)));

__device__ inline void rows_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// History terms q <= n0 of a block's outputs (without the part older than the
// super-chunk when split) -> ex[end][lane], lane = task slot * T + output.
template <int RW>
__device__ inline void rows_far(const cd* hist, const double* beta, int nt, bool split, int task0, int ntask,
                                int n0, const double* sb, cd* ex) {
    constexpr int SLOTS = 4 / RW, T = 16 * RW, U = 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int r = lane & 15, kq = lane >> 4;
    const int part = r & 1, e = (r >> 1) & 1, sc = r >> 2;
    const int sl = sc % SLOTS, sh = sc / SLOTS;      // task slot, 16-step part of the block
    const int C = n0 - n0 % kFarSuper;
    const int q_lo = split && C > 0 ? C - kWave : 0;
    const int qs = q_lo - 16 * (RW - 1);
    const double* hb = reinterpret_cast<const double*>(
                           hist + ((size_t)(task0 + min(sl, ntask - 1)) * 2 + e) * (nt + 1)) + part;
    const int qb = 16 * sh + kq;                     // my source of group qg: qg + qb
    const int ab = n0 + 1 + r - kq;                  // my beta index of group qg: ab - qg
    const int ng = (n0 - qs) / 4 + 1;
    rows_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    // groups that meet a source outside [q_lo, n0]: the first H and those from g1
    // on, their reads issued first; the ones between come in fours, without tests
    // and at constant offsets (with them the loop took 20 instructions a group: one
    // sweep of 32 problems on 500 uneven subdomains, 512 steps, 6.5 -> 5.8 ms)
    constexpr int H = 4 * (RW - 1);
    const int g0 = min(H, ng), g1 = max((n0 - 16 * (RW - 1) - qs) / 4, g0);
    double vh[H + 1], vt[H + 1];
    auto edge = [&](int g) {
        const int q = qs + 4 * g + qb;
        double v = 0.0;
        if (q >= q_lo && q <= n0) v = hb[2 * q];
        return v;
    };
#pragma unroll
    for (int u = 0; u < H; ++u) vh[u] = edge(u);
#pragma unroll
    for (int u = 0; u <= H; ++u) vt[u] = edge(g1 + u);
    auto sum = [&](const double* wt) {
        auto add = [&](int g, double v) {
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wt[max(ab - qs - 4 * g, 0)], v, acc, 0, 0, 0);
        };
        double an[U], bn[U];
        const double* hp = hb + 2 * (qs + 4 * g0 + qb);
        const double* wp = wt + (ab - qs - 4 * (g0 + U - 1));
        auto fetch = [&]() {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                bn[u] = hp[8 * u];
                an[u] = wp[4 * (U - 1 - u)];
            }
            hp += 8 * U;
            wp -= 4 * U;
        };
        if (g0 < g1) fetch();
#pragma unroll
        for (int u = 0; u < H; ++u) add(u, vh[u]);
        for (int g = g0; g < g1; g += U) {
            double ac[U], bc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) { ac[u] = an[u]; bc[u] = bn[u]; }
            if (g + U < g1) fetch();
#pragma unroll
            for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ac[u], bc[u], acc, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u <= H; ++u) add(g1 + u, vt[u]);
    };
    // (one pointer to either would make the reads of the beta window flat ones)
    if (split) sum(sb);
    else sum(beta);
    double* o = reinterpret_cast<double*>(ex + e * kWave + sl * T + 16 * sh) + part;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[2 * (kq + 4 * k)] = acc[k];
}

// The tasks first .. first + count - 1 (at most SLOTS per wave of the
// workgroup), all of P nodes per lane; with LDSF all of one factor record.
template <int P, int RW, bool LDSF, int NW, int TR, int VK = VK_STATIC>
__device__ inline void rows_body(const SweepArgs& a, int first, int count, cd* smem) {
    static_assert(VK == VK_STATIC || (RW == 4 && !LDSF && NW == 1), "V(t,x), |u|^2: one task per wave");
    constexpr int T = 16 * RW, SLOTS = 4 / RW;
    constexpr bool WRAP = P == 1;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = NW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : 0;
    const int t = lane % T;
    const int slot0 = wv * SLOTS, mine = slot0 + lane / T;
    // LDS: [beta window][per wave: v left, v right, sums left, sums right][record]
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
    const int fl = live ? (task.flags & a.flags_and) | a.flags_or : (task.flags & a.flags_and) & T_DATA_U0;
    const int n = a.J[k] + 1, o = a.off[k];
    const bool lif = k > 0, rif = k < a.N - 1;
    const int tl = P > 1 ? T - 1 : n - 1;             // lane of node n - 1 (slot P - 1)
    int s;
    bool dup;
    rows_place<P, RW>(n, t, s, dup);
    const cd zero = mk(0, 0);
    const bool t0 = t == 0, tL = t == tl;
    const int jr = P > 1 ? T - 1 - t : (tl - t) & (T - 1);   // output step of my right sum
    const int special = a.flags_or & (T_CKPT | T_OUT_SNAP | T_OUT_TRACE);

    RowsFac<P, RW, LDSF> F;
    F.lds = sfac + t;
    if (VK != VK_TIME) F.load(a.fac + (size_t)task.f * a.fstride + t);

    const int nbeg = a.n_begin, nend = a.n_end;
    const bool begins = nbeg == 0, last = nend == nt;
    cd* stp = a.state ? a.state + (size_t)tix * 2 * a.pstride * kWave + t : nullptr;
    cd u[P], vlast[P];                                // vlast: v_n, where |u|^2's inner iteration starts
    if (begins) {
        const cd* u0 = a.u0 + (size_t)b * a.nx + o;
#pragma unroll
        for (int q = 0; q < P; ++q) {
            u[q] = zero;
            if ((fl & T_DATA_U0) && s + q < n) u[q] = u0[s + q];
        }
    } else {
#pragma unroll
        for (int q = 0; q < P; ++q) u[q] = stp[q * T];
    }
    int nl_worst = 0, nl_fail = 0;
    if (VK == VK_CUBIC) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            vlast[q] = u[q];
            if (!begins) vlast[q] = stp[(a.pstride + q) * kWave];
        }
    }
    // node weights of the mass stencil: 4, and 2 at the two end nodes
    const double w0 = t0 ? 2.0 : 4.0;
    const double wL = (tL || (P == 1 && t0)) ? 2.0 : 4.0;
    // boundary terms over i kappa: c2 (S0^2) or 1 (Robin) times the running sum
    const double ik = 1.0 / a.kappa;
    const cd cc = TR == TR_S02 ? a.c2 : mk(1, 0);
    const cd cs = mk(cc.y * ik, -cc.x * ik);
    const cd ic = TR == TR_S02 ? inv(a.c2) : mk(1, 0);
    double bl = 0.0, br = 0.0;                        // beta of my lag in the two running sums
    if (TR == TR_S02) {
        bl = a.beta[t + 1];
        br = a.beta[jr + 1];
    }

    cd* const Ha = a.hist ? a.hist + (size_t)tix * 2 * (nt + 1) : nullptr;
    // Stores of u at chosen steps.  Their addresses are formed from task
    // indices the compiler cannot follow, or it would compute them once and
    // hold them (50 registers) through the step loop.
    auto put_u = [&](int nstep) {
        int x = tix, kk = k, bb = b;
        asm volatile("" : "+v"(x), "+v"(kk), "+v"(bb));
        if ((fl & T_CKPT) && ((nt - nstep) & (kWave - 1)) == 0 && nstep < nt) {
            cd* ck = a.ckpt + ((size_t)x * (a.Jc + 1) + (nt - nstep) / kWave) * a.pstride * kWave;
#pragma unroll
            for (int q = 0; q < P; ++q)
                if (s + q < n && !(q == 0 && dup)) ck[s + q] = u[q];
        }
        if ((fl & T_OUT_SNAP) && nstep % a.snap_stride == 0) {
            const int j = nstep / a.snap_stride;
            cd* sp = a.snaps + ((size_t)bb * a.nsnap + j) * a.nx + o;
#pragma unroll
            for (int q = 0; q < P; ++q)
                if (s + q > 0 && s + q < n - 1 && !(q == 0 && dup)) sp[s + q] = u[q];
            cd* se = a.snap_ends + (((size_t)bb * a.nsnap + j) * a.N + kk) * 2;
            if (t0) se[0] = u[0];
            if (tL) se[1] = u[P - 1];
        }
        if (fl & T_OUT_TRACE) {
            cd* tr = a.trace + (size_t)(bb * a.N + kk) * 2 * (nt + 1) + nstep;
            if (t0) tr[0] = u[0];
            if (tL) tr[nt + 1] = u[P - 1];
        }
    };
    // steps up to and including the next one at which put_u has work
    auto until = [&](int nstep) {
        int m = kWave;
        if (special & T_CKPT) m = min(m, (nt - nstep - 1) % kWave + 1);
        if (special & T_OUT_SNAP) m = min(m, a.snap_stride - nstep % a.snap_stride);
        return (special & T_OUT_TRACE) ? 1 : m;
    };
    if (begins) {
        if (TR == TR_S02 && live) {
            // v_0 of the history
            if (t0) Ha[0] = u[0];
            if (tL) Ha[nt + 1] = u[P - 1];
        }
        if (special) {
            if (fl & T_CKPT) {
                // u_0 closes the checkpoints, whatever nt is
                cd* ck = a.ckpt + ((size_t)tix * (a.Jc + 1) + a.Jc) * a.pstride * kWave;
#pragma unroll
                for (int q = 0; q < P; ++q)
                    if (s + q < n && !(q == 0 && dup)) ck[s + q] = u[q];
            }
            put_u(0);
        }
    }
    double maxd = 0.0;

    for (int n0 = nbeg; n0 < nend; n0 += T) {
        const int nb = min(T, nend - n0);
        const size_t gi = ((size_t)b * a.ns + 2 * k) * nt + n0;   // slot 2k; l_k is the slot before
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
        {
            cd l = zero, rr = zero;
            if (lif && okl) {
                if (fl & T_FLUX_G) l = a.g_in[gi - nt + t];
                if ((fl & T_IMP_L) && n0 + t == 0) l = mk(1, 0);
            }
            if (rif && okr) {
                if (fl & T_FLUX_G) rr = a.g_in[gi + jr];
                if ((fl & T_IMP_R) && n0 + jr == 0) rr = mk(1, 0);
            }
            accA = accA - ic * l;
            accB = accB - ic * rr;
        }
        const bool ml = lif && t0, mr = rif && tL;
        cd* lgl = lg + (lane - t);

        for (int i = 0; i < nb;) {
          const int ie = special ? min(nb, i + until(n0 + i)) : nb;
          for (; i < ie; ++i) {
            if constexpr (VK == VK_TIME) {
                __syncthreads();                      // this step's record is in LDS (time_helper)
                F.load(sfac + ((n0 + i - nbeg) & 1) * (rows_fields(P, RW) * T) + t);
            }
            const cd uL = rows_up1<RW>(u[P - 1], t);
            const cd uR = rows_dn1<RW>(rows_front<P>(u, dup), t);
            auto stencil = [&](int q) { return rows_stencil<P>(u, uL, uR, w0, wL, q); };
            cd dF = stencil(0), dS = P > 1 ? stencil(P - 1) : zero;
            if (ml) {
                dF = madd_x(dF, cs, accA);
                lgl[2 * kWave + i] = accA;
            }
            if (P == 1) dS = dF;
            if (mr) {
                dS = madd_x(dS, cs, accB);
                lgl[3 * kWave + i] = accB;
            }
            cd y[P];
            if constexpr (VK == VK_CUBIC) {
                // inner fixed point of eq. AvMNL from zeta^0 = v_{n-1}:
                // (cM - S - sigma E) zeta^{s+1} = rhs - M_{|zeta^s|^2} zeta^s, over
                // i kappa; the generalised mass (nodal weight |zeta|^2, the element
                // matrix of M_W) is h / 12 times ((f_{i-1} + f_i) zeta_{i-1} +
                // (f_{i-1} + 6 f_i + f_{i+1}) zeta_i + (f_i + f_{i+1}) zeta_{i+1}),
                // 3 f_i at an end node
                cd d[P];
#pragma unroll
                for (int q = 0; q < P; ++q) d[q] = stencil(q);
                d[0] = dF;
                d[P - 1] = dS;
                const double gk = a.h / 12.0 * ik, tol2 = a.nl_tol * a.nl_tol;
                int it = 1;
                bool conv = false;
                for (; it <= a.nl_maxit; ++it) {
                    const cd zL = rows_up1<RW>(vlast[P - 1], t);
                    const cd zR = rows_dn1<RW>(rows_front<P>(vlast, dup), t);
                    auto rhs = [&](int q) {
                        const cd zm = sel_c(q == 0, zL, vlast[q == 0 ? 0 : q - 1]);
                        const cd zp = sel_c(q == P - 1, zR, vlast[q == P - 1 ? 0 : q + 1]);
                        const double w = q == P - 1 ? wL : (q == 0 ? w0 : 4.0);
                        const double fm = abs2(zm), fi = abs2(vlast[q]), fp = abs2(zp);
                        const double c0 = fma(1.5 * w, fi, fm + fp), cm = fm + fi, cp = fi + fp;
                        const double sx = fma(cm, zm.x, fma(c0, vlast[q].x, cp * zp.x));
                        const double sy = fma(cm, zm.y, fma(c0, vlast[q].y, cp * zp.y));
                        return mk(fma(-gk, sy, d[q].x), fma(gk, sx, d[q].y));
                    };
                    rows_solve(F, rhs(0), P > 1 ? rhs(P - 1) : rhs(0), rhs, t, dup, y);
                    double dm = 0.0, zm2 = 0.0;
#pragma unroll
                    for (int q = 0; q < P; ++q) {
                        dm = fmax(dm, abs2(y[q] - vlast[q]));
                        zm2 = fmax(zm2, abs2(vlast[q]));
                        vlast[q] = y[q];
                    }
                    // max |x - z| <= tol max(1, max |z|) on the squares; the maxima are the
                    // same bits on every lane
                    const bool done = wave_max(dm) <= tol2 * fmax(1.0, wave_max(zm2));
                    if (__builtin_amdgcn_readfirstlane(done)) { conv = true; break; }
                }
                if (!conv) nl_fail = 1;
                nl_worst = max(nl_worst, conv ? it : a.nl_maxit);
            } else {
                rows_solve(F, dF, dS, stencil, t, dup, y);
            }
            const cd X = y[P - 1];
#pragma unroll
            for (int q = 0; q < P; ++q) u[q] = mk(2.0 * y[q].x - u[q].x, 2.0 * y[q].y - u[q].y);
            if (t0) lgl[i] = y[0];
            if (tL) lgl[kWave + i] = X;
            accA = rows_roll_dn<RW>(accA);
            accB = rows_roll_up<RW, WRAP>(accB);
            if (TR == TR_S02) {
                const cd va = rows_first<RW>(y[0]), vb = rows_last<RW, P>(X, tl);
                accA = mk(fma(bl, va.x, accA.x), fma(bl, va.y, accA.y));
                accB = mk(fma(br, vb.x, accB.x), fma(br, vb.y, accB.y));
            }
          }
          if (special) put_u(n0 + i);
        }
        // the block's outputs, lane t the step n0 + 1 + t:
        // rho = -flux + 2 (sigma v + h) with h - flux = cc * (logged sum); Robin: h = 0
        rows_fence();
        const cd va = lg[lane], vb = lg[kWave + lane], sa = lg[2 * kWave + lane], sc = lg[3 * kWave + lane];
        rows_fence();
        if (okl && live) {
            if (fl & T_CKPT) {
                cd* bs = a.bsum + (size_t)tix * 2 * nt + n0 + t;
                if (lif) bs[0] = sa;
                if (rif) bs[nt] = sc;
            }
            if (TR == TR_S02) {
                Ha[n0 + 1 + t] = va;
                Ha[nt + 1 + n0 + 1 + t] = vb;
            }
            auto flux = [&](bool on, size_t at, int imp) {
                cd l = zero;
                if (on && (fl & T_FLUX_G)) l = a.g_in[at];
                if ((fl & imp) && n0 + t == 0) l = mk(1, 0);
                return l;
            };
            auto put = [&](cd sum, cd v, cd l, cd* out, const cd* old) {
                const cd rho = TR == TR_S02 ? 2.0 * madd(cc * sum, a.sigma, v) + l : 2.0 * (a.sigma * v) - l;
                *out = rho;
                if (old) maxd = fmax(maxd, sqrt(abs2(rho - *old)));
            };
            const bool md = (fl & T_MAXDIFF) != 0;
            if (fl & T_OUT_G) {
                // left end -> slot 2k - 2, right end -> slot 2k + 1
                const size_t ol = gi - 2 * (size_t)nt + t, orr = gi + nt + t;
                if (lif) put(sa, va, flux(true, gi - nt + t, T_IMP_L), a.g_out + ol, md ? a.g_in + ol : nullptr);
                if (rif) put(sc, vb, flux(true, gi + t, T_IMP_R), a.g_out + orr, md ? a.g_in + orr : nullptr);
            } else if (fl & T_OUT_COLS) {
                cd* c = a.cols + ((size_t)task.f * 4 + ((fl & T_IMP_L) ? 0 : 1)) * nt + n0 + t;
                if (lif) put(sa, va, flux(false, 0, T_IMP_L), c, nullptr);
                if (rif) put(sc, vb, flux(false, 0, T_IMP_R), c + 2 * (size_t)nt, nullptr);
            }
        }
    }

    if (!last && stp && live) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            stp[q * T] = u[q];
            if (VK == VK_CUBIC) stp[(a.pstride + q) * kWave] = vlast[q];
        }
    }
    if ((fl & T_OUT_UT) && last) {
        cd* uT = a.uT + (size_t)b * a.nx + o;
#pragma unroll
        for (int q = 0; q < P; ++q)
            if (s + q > 0 && s + q < n - 1 && !(q == 0 && dup)) uT[s + q] = u[q];
        cd* en = a.ends + ((size_t)b * a.N + k) * 2;
        if (t0) en[0] = u[0];
        if (tL) en[1] = u[P - 1];
    }
    if (a.flags_or & T_MAXDIFF) {
        maxd = wave_max(maxd);
        if (lane == 0 && maxd > 0.0)
            atomicMax(a.maxdiff, (unsigned long long)__double_as_longlong(maxd));
    }
    if (VK == VK_CUBIC && lane == 0 && a.nl_stats) {
        atomicMax(&a.nl_stats[0], nl_worst);
        if (nl_fail) atomicMax(&a.nl_stats[1], 1);
    }
}

template <int P, int PHI, int RW, int PLDS, int NW, int TR>
__device__ inline void rows_pick(const SweepArgs& a, int first, int count, int p, cd* smem) {
    if (p == P) rows_body<P, RW, (P >= PLDS), NW, TR>(a, first, count, smem);
    else if constexpr (P < PHI) rows_pick<P + 1, PHI, RW, PLDS, NW, TR>(a, first, count, p, smem);
}

// widths PLO .. PHI, those from PLDS on with their records in LDS; NW waves
// per workgroup
template <int RW, int PLO, int PHI, int PLDS, int NW, int WPE, int TR>
__global__ __launch_bounds__(NW * kWave, WPE) void sweep_rows_kernel(SweepArgs a) {
    extern __shared__ cd smem[];
    const int4 it = a.items[blockIdx.x];              // first task, tasks, P
    rows_pick<PLO, PHI, RW, PLDS, NW, TR>(a, it.x, it.y, it.z, smem);
}

}  // namespace swr
