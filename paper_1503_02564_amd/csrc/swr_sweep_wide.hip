// swr_sweep_wide.hip -- subdomains of more than 64 * 8 nodes, static potential,
// Robin and S0^2: a task is swept by a workgroup of NW waves, four rows of 16
// lanes each (swr_rows.h with T = 64 NW lanes; up to 12 nodes per lane, so up
// to 6144 nodes).  Longer subdomains and the other potentials run the
// streaming sweep (swr_sweep_long.hip).
//
// Why: the streaming sweep walks such a subdomain on one wave and moves every
// per-node array through memory three times a step, 97 us a step at 4201 nodes,
// nearly all of it waiting.  Here u and the intermediate stay in registers, the
// interior coefficients in registers and LDS (what does not fit is read from L2
// every step, each once), and eight waves share the work.
//
// Coupling of the waves.  A wave solves its 64 separators with zero values
// beyond its two ends (row reduction and row coupling as in swr_rows.h), giving
// y.  With E_w, S_w the separator values of lanes 63 and 0 of wave w and F_w the
// interior response y of its first node,
//   X = y + PW E_{w-1} + QW S_{w+1} + RW F_{w+1}
// (RW: response to the part of lane 63's right-hand side that the next wave
// holds).  The waves exchange (y at lane 63, y at lane 0, F) through LDS, one
// barrier a step, and each forms its E_{w-1} and S_{w+1} as two dot products
// with the 3 NW exchanged values, one weight per lane.  The neighbours' u at the
// wave's borders are carried as copies (they follow from the same values) and
// renewed at every block start.
//
// Bound: FP64 issue of NW / 4 waves per SIMD, about 26 P + 250 instructions a
// step and wave.  Measured on 100 subdomains of 4200 cells, 300 steps (100 + 300
// tasks, 8 waves and 9 nodes per lane each): 59.4 -> 5.2 ms per solve,
// its two sweeps 29 -> 2.1 ms each on average.
#include <type_traits>

#include "swr_sweep_rows_kernel.h"

namespace swr {

constexpr int kWideTail = rows_tail(4) + 4;      // + PW, QW, RW, dot-product weight
__host__ __device__ constexpr int wide_fields(int P) { return 4 * (P - 1) + kWideTail; }

// ---------------------------------------------------------------------------
// Factorisation: one workgroup per record, as rows_factor_body with the waves
// coupled.  No cancellation (row sums carried beside the couplings).
// ---------------------------------------------------------------------------
template <int P, int NW>
__device__ inline void wide_factor_body(const FactorArgs& a, int f, cd* sh) {
    constexpr int T = 64 * NW, PI = P - 1;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave, t = threadIdx.x;
    const int k = f % a.N, v = f / a.N;
    const int n = a.J[k] + 1, o = a.off[k];
    const bool lif = k > 0, rif = k < a.N - 1;
    const double kap = a.h / (3.0 * a.dt);
    const double p1 = 1.0 / (a.h * kap), q1 = a.h / (12.0 * kap), ik = 1.0 / kap;
    const cd sig = mk(a.sigma.y * ik, -a.sigma.x * ik);
    const int r0 = n - T * (P - 1);
    const bool dup = t >= r0;
    const int s = t * P - max(0, t - r0 + 1);
    const double* V = a.V ? a.V + (size_t)v * a.nx + o : nullptr;
    auto W = [&](int i) { return (V && i >= 0 && i < n) ? V[i] : 0.0; };
    const cd zero = mk(0, 0), one = mk(1, 0);
    auto row = [&](int i, cd& cl, cd& cr, cd& ex) {
        cl = cr = ex = zero;
        const double wm = W(i - 1), wi = W(i), wp = W(i + 1);
        if (i > 0) {
            cl = mk(-1.0, p1 + q1 * (wm + wi));
            ex = ex + mk(3.0, -q1 * (4.0 * wi + 2.0 * wm));
        }
        if (i < n - 1) {
            cr = mk(-1.0, p1 + q1 * (wi + wp));
            ex = ex + mk(3.0, -q1 * (4.0 * wi + 2.0 * wp));
        }
        if (i == 0 && lif) ex = ex - sig;
        if (i == n - 1 && rif) ex = ex - sig;
    };
    cd* rec = a.fac + (size_t)f * a.fstride + t;
    cd m[PI], al[PI], ga[PI], de[PI];
    cd mp = zero, wa = zero, wd = zero;
    bool started = false;
#pragma unroll
    for (int q = 0; q < PI; ++q) {
        cd cl, cr, ex;
        row(s + q, cl, cr, ex);
        const bool real = !(q == 0 && dup);
        wa = sel_c(started, mp * wa, cl);
        wd = sel_c(started, madd(ex, mp, wd), ex);
        const cd iv = sel_c(real, inv((cr + wa) + wd), zero);
        m[q] = cr * iv;
        al[q] = iv * wa;
        de[q] = iv * wd;
        started = started || real;
        mp = m[q];
        rec[(4 * q) * T] = iv;
        rec[(4 * q + 1) * T] = -m[q];
    }
    ga[PI - 1] = m[PI - 1];
#pragma unroll
    for (int q = P - 3; q >= 0; --q) {
        al[q] = madd(al[q], m[q], al[q + 1]);
        de[q] = madd(de[q], m[q], de[q + 1]);
        ga[q] = m[q] * ga[q + 1];
    }
    if (dup) {
        al[0] = one;
        ga[0] = zero;
        de[0] = zero;
    }
#pragma unroll
    for (int q = 0; q < PI; ++q) {
        rec[(4 * q + 2) * T] = al[q];
        rec[(4 * q + 3) * T] = ga[q];
    }
    cd cl, cr, ex;
    row(s + P - 1, cl, cr, ex);
    const cd gF = sel_c(dup, ga[1], ga[0]), dF = sel_c(dup, de[1], de[0]);
    // the next wave's first lane -> my lane 63
    cd* shF = sh;                                 // [NW][2]
    if (lane == 0) {
        shF[2 * wv] = gF;
        shF[2 * wv + 1] = dF;
    }
    __syncthreads();
    cd gR = rows_dn1<4>(gF, lane), dR = rows_dn1<4>(dF, lane);
    if (lane == kWave - 1 && wv < NW - 1) {
        gR = shF[2 * (wv + 1)];
        dR = shF[2 * (wv + 1) + 1];
    }
    cd At = cl * al[PI - 1], Ct = cr * gR, Et = madd(madd(ex, cl, de[PI - 1]), cr, dR);
    const bool rf = (lane & 15) == 0, rl = (lane & 15) == 15;
    // spikes of the rows' borders, the row sums, and lane 63's response to the
    // next wave's F (right-hand side + cr F)
    cd ps = sel_c(rf, At, zero), qs = sel_c(rl, Ct, zero), ds = Et;
    cd fs = sel_c(lane == kWave - 1 && wv < NW - 1, cr, zero);
    if (rf) { Et = Et + At; At = zero; }
    if (rl) { Et = Et + Ct; Ct = zero; }
    cd* tail = rec + 4 * (P - 1) * T;
    tail[0] = -cl;
    tail[T] = -cr;
    auto level = [&](auto lc) {
        constexpr int L = decltype(lc)::value;
        constexpr int UP = 0x110 + (1 << L), DN = 0x100 + (1 << L);
        const cd iB = inv((Et + At) + Ct);
        const cd k1 = At * dpp_c<UP>(iB), k2 = Ct * dpp_c<DN>(iB);
        const cd Am = dpp_c<UP>(At), Cp = dpp_c<DN>(Ct);
        auto fold = [&](cd x) { return madd(madd(x, k1, dpp_c<UP>(x)), k2, dpp_c<DN>(x)); };
        Et = fold(Et);
        ps = fold(ps);
        qs = fold(qs);
        ds = fold(ds);
        fs = fold(fs);
        At = k1 * Am;
        Ct = k2 * Cp;
        tail[(2 + L) * T] = -k1;
        tail[(2 + kRowLevels + L) * T] = -k2;
    };
    level(std::integral_constant<int, 0>{});
    level(std::integral_constant<int, 1>{});
    level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{});
    const cd iB = inv((Et + At) + Ct);
    ps = ps * iB;
    qs = qs * iB;
    ds = ds * iB;
    fs = fs * iB;
    tail[(2 + 2 * kRowLevels) * T] = iB;
    auto at = [&](cd x, int l) { return mk(__shfl(x.x, l), __shfl(x.y, l)); };
    // the rows of the wave: unknowns e_0, s_1, e_1, s_2, e_2, s_3 as in
    // rows_factor_body; lane j solves right-hand side j: 0 .. 5 the unit vectors
    // over B, 6 E_{w-1}, 7 S_{w+1}, 8 F_{w+1}, 9 the row sums
    cd O[6][6], xs[6], x[6];
    const int j = lane % 10;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int r = (i + 1) / 2;
        const int l = (i & 1) ? 16 * r : 16 * r + 15;
        const cd p = at(ps, l), q = at(qs, l), ib = at(iB, l), d = at(ds, l), g = at(fs, l);
#pragma unroll
        for (int c = 0; c < 6; ++c) O[i][c] = zero;
        xs[i] = d;
        if (r > 0) O[i][2 * (r - 1)] = p;
        else xs[i] = xs[i] + p;
        if (r < 3) O[i][2 * r + 1] = q;
        else xs[i] = xs[i] + q;
        x[i] = sel_c(i == j, ib, zero);
        if (r == 0) x[i] = sel_c(j == 6, p, x[i]);
        if (r == 3) x[i] = sel_c(j == 7, q, sel_c(j == 8, g, x[i]));
        x[i] = sel_c(j == 9, d, x[i]);
    }
    cd ip[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        cd p = xs[c];
#pragma unroll
        for (int d = c + 1; d < 6; ++d) p = p + O[c][d];
        ip[c] = inv(p);
#pragma unroll
        for (int i = c + 1; i < 6; ++i) {
            const cd w = O[i][c] * ip[c];
#pragma unroll
            for (int d = c + 1; d < 6; ++d)
                if (d != i) O[i][d] = madd(O[i][d], w, O[c][d]);
            xs[i] = madd(xs[i], w, xs[c]);
            x[i] = madd(x[i], w, x[c]);
        }
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
#pragma unroll
        for (int d = i + 1; d < 6; ++d) x[i] = madd(x[i], O[i][d], x[d]);
        x[i] = x[i] * ip[i];
    }
    const int r = lane >> 4;
    // my lane's value for right-hand side jj beyond its own row
    auto coupled = [&](int jj) {
        cd e[3], sn[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            e[q] = at(x[2 * q], jj);
            sn[q] = at(x[2 * q + 1], jj);
        }
        cd wj = zero;
        if (r > 0) wj = ps * sel_c(r == 1, e[0], sel_c(r == 2, e[1], e[2]));
        if (r < 3) wj = madd(wj, qs, sel_c(r == 0, sn[0], sel_c(r == 1, sn[1], sn[2])));
        return wj;
    };
#pragma unroll
    for (int jj = 0; jj < 6; ++jj) tail[(3 + 2 * kRowLevels + jj) * T] = coupled(jj);
    cd PW = coupled(6), QW = coupled(7), FW = coupled(8), DW = coupled(9) + ds;
    if (r == 0) PW = PW + ps;
    if (r == 3) { QW = QW + qs; FW = FW + fs; }
    const int tb = rows_tail(4);
    tail[tb * T] = PW;
    tail[(tb + 1) * T] = QW;
    tail[(tb + 2) * T] = FW;
    // The waves: unknowns E_w (2 w), S_w (2 w + 1) of
    //   X = y + P E_{w-1} + Q S_{w+1} + R F_{w+1}, row sums D;
    // right-hand sides 3 w + (0: y of E_w, 1: y of S_w, 2: F_w)
    constexpr int U = 2 * NW, NR = 3 * NW;
    cd* sO = sh + 2 * NW;                         // [U][U] minus the off-diagonal entries
    cd* sx = sO + U * U;                          // [U] row sums
    cd* sr = sx + U;                              // [U][NR]
    for (int i = t; i < U * U + U + U * NR; i += T) sO[i] = zero;
    __syncthreads();
    if (lane == kWave - 1 || lane == 0) {
        const int i = 2 * wv + (lane == 0 ? 1 : 0);
        if (wv > 0) sO[i * U + 2 * (wv - 1)] = PW;
        if (wv < NW - 1) {
            sO[i * U + 2 * (wv + 1) + 1] = QW;
            sr[i * NR + 3 * (wv + 1) + 2] = FW;
        }
        sx[i] = DW;
        sr[i * NR + 3 * wv + (lane == 0 ? 1 : 0)] = one;
    }
    __syncthreads();
    for (int c = 0; c < U; ++c) {
        // pivot = row sum plus the couplings to the unknowns still there
        cd p = sx[c];
        for (int d = c + 1; d < U; ++d) p = p + sO[c * U + d];
        const cd ipc = inv(p);
        __syncthreads();
        for (int e = t; e < (U - 1 - c) * (U + 1 + NR); e += T) {
            const int i = c + 1 + e / (U + 1 + NR), d = e % (U + 1 + NR);
            const cd w = sO[i * U + c] * ipc;
            if (d < U) {
                if (d > c && d != i) sO[i * U + d] = madd(sO[i * U + d], w, sO[c * U + d]);
            } else if (d == U) {
                sx[i] = madd(sx[i], w, sx[c]);
            } else {
                const int h = d - U - 1;
                sr[i * NR + h] = madd(sr[i * NR + h], w, sr[c * NR + h]);
            }
        }
        // (the pivot's reciprocal waits in its own, unused diagonal entry)
        if (t == 0) sO[c * U + c] = ipc;
        __syncthreads();
    }
    if (t < NR) {
        for (int i = U - 1; i >= 0; --i) {
            cd xv = sr[i * NR + t];
            for (int d = i + 1; d < U; ++d) xv = madd(xv, sO[i * U + d], sr[d * NR + t]);
            sr[i * NR + t] = xv * sO[i * U + i];
        }
    }
    __syncthreads();
    // lanes 0 .. NR - 1: weights of E_{w-1}; lanes 32 ..: of S_{w+1}
    cd wt = zero;
    const int h = lane & 31;
    if (h < NR) {
        if (lane < 32 && wv > 0) wt = sr[(2 * (wv - 1)) * NR + h];
        if (lane >= 32 && wv < NW - 1) wt = sr[(2 * (wv + 1) + 1) * NR + h];
    }
    tail[(tb + 3) * T] = wt;
}

template <int P, int PHI, int NW>
__device__ inline void wide_factor_pick(const FactorArgs& a, int f, int p, cd* sh) {
    if (p == P) wide_factor_body<P, NW>(a, f, sh);
    else if constexpr (P < PHI) wide_factor_pick<P + 1, PHI, NW>(a, f, p, sh);
}

template <int NW, int PLO, int PHI>
__global__ __launch_bounds__(NW * kWave) void wide_factor_kernel(FactorArgs a) {
    __shared__ cd sh[2 * NW + 2 * NW * 2 * NW + 2 * NW + 2 * NW * 3 * NW];
    const int f = blockIdx.x;
    const int key = a.Pk[f % a.N];                    // P + 32 NW of the subdomain (0: another form)
    if (key / 32 != NW) return;
    wide_factor_pick<PLO, PHI, NW>(a, f, key % 32, sh);
}

// ---------------------------------------------------------------------------
// The sweep
// ---------------------------------------------------------------------------
// LDS of a workgroup: exchanged values [2][3 NW], logs of the two end waves,
// then interior fields
__host__ __device__ constexpr int wide_fixed(int NW) { return 2 * 3 * NW + 2 * kRowsWaveLds; }
// interior fields held in LDS: as many as 160 KiB take
__host__ __device__ constexpr int wide_lds_fields(int P, int NW) {
    const int room = (160 * 1024 / 16 - wide_fixed(NW)) / (64 * NW), want = 3 * (P - 1);
    return room < want ? room : want;
}

// Interior coefficients: cp in registers (a step reads them twice), then inv,
// al, ga in LDS as far as they fit, the rest in memory
template <int P, int NW>
struct WideFac {
    static constexpr int T = 64 * NW, NL = wide_lds_fields(P, NW);
    static constexpr bool CPR = P <= 9;          // cp in registers
    cd c[CPR ? P - 1 : 1];
    cd tl[kWideTail];
    const cd* lds;
    const cd* mem;
    __device__ void load(const cd* rec) {
        mem = rec;
        if (CPR) {
#pragma unroll
            for (int q = 0; q < P - 1; ++q) c[q] = rec[(4 * q + 1) * T];
        }
#pragma unroll
        for (int i = 0; i < kWideTail; ++i) tl[i] = rec[(4 * (P - 1) + i) * T];
    }
    // field j (0 inv, 1 al, 2 ga) of slot q: place j (P - 1) + q
    static __device__ constexpr int rec_field(int pl) {
        return 4 * (pl % (P - 1)) + (pl / (P - 1) == 0 ? 0 : pl / (P - 1) + 1);
    }
    __device__ cd get(int pl) const { return pl < NL ? lds[pl * T] : mem[rec_field(pl) * T]; }
    __device__ cd inv(int q) const { return get(q); }
    __device__ cd al(int q) const { return get(P - 1 + q); }
    __device__ cd ga(int q) const { return get(2 * (P - 1) + q); }
    __device__ cd cp(int q) const { return CPR ? c[CPR ? q : 0] : mem[(4 * q + 1) * T]; }
    __device__ cd k1(int l) const { return tl[2 + l]; }
    __device__ cd k2(int l) const { return tl[2 + kRowLevels + l]; }
    __device__ cd invB() const { return tl[2 + 2 * kRowLevels]; }
    __device__ cd W(int j) const { return tl[3 + 2 * kRowLevels + j]; }
};

// sum over the 32 lanes of each half of the wave, on every lane of the half
__device__ inline double half_sum(double v) {
    v += dpp_shift<0x128>(v);                     // row_ror:8
    v += dpp_shift<0x124>(v);
    v += dpp_shift<0x122>(v);
    v += dpp_shift<0x121>(v);
    const RowPair p = swap16(v);
    return p.first + p.second;
}

template <int P, int NW, int TR>
__device__ inline void wide_body(const SweepArgs& a, int tix, cd* smem) {
    constexpr int T = 64 * NW, kAhead = 2;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int t = threadIdx.x;
    const bool wfirst = wv == 0, wlast = wv == NW - 1;
    cd* bx = smem;                                // [2][3 NW]
    cd* lg = smem + 2 * 3 * NW + (wlast ? kRowsWaveLds : 0);
    cd* sfac = smem + wide_fixed(NW);
    const int nt = a.nt;
    const Task task = a.tasks[tix];
    const int k = task.k, b = task.b;
    const int fl = (task.flags & a.flags_and) | a.flags_or;
    const int n = a.J[k] + 1, o = a.off[k];
    const bool lif = k > 0, rif = k < a.N - 1;
    const int r0 = n - T * (P - 1);
    const bool dup = t >= r0;
    const int s = t * P - max(0, t - r0 + 1);
    const cd zero = mk(0, 0);
    const bool t0 = t == 0, tL = t == T - 1, l0 = lane == 0, l63 = lane == kWave - 1;
    const int special = a.flags_or & (T_OUT_SNAP | T_OUT_TRACE);

    const cd* rec = a.fac + (size_t)task.f * a.fstride;
    for (int i = t; i < WideFac<P, NW>::NL * T; i += T) {
        const int pl = i / T;
        sfac[i] = rec[(4 * (pl % (P - 1)) + (pl / (P - 1) == 0 ? 0 : pl / (P - 1) + 1)) * T + i % T];
    }
    WideFac<P, NW> F;
    F.lds = sfac + t;
    F.load(rec + t);
    // the next wave's first node: its responses to my lane 63 and to S_{w+1}
    cd alF = zero, gaF = zero;
    if (!wlast) {
        const int q = (t - lane) + kWave >= r0 ? 1 : 0;
        const cd* rn = rec + (t - lane) + kWave;
        alF = rn[(4 * q + 2) * T];
        gaF = rn[(4 * q + 3) * T];
    }

    cd u[P];
    const cd* u0 = a.u0 + (size_t)b * a.nx + o;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        u[q] = zero;
        if (fl & T_DATA_U0) u[q] = u0[s + q];
    }
    const double w0 = t0 ? 2.0 : 4.0, wL = tL ? 2.0 : 4.0;
    const double ik = 1.0 / a.kappa;
    const cd cc = TR == TR_S02 ? a.c2 : mk(1, 0);
    const cd cs = mk(cc.y * ik, -cc.x * ik);
    const cd ic = TR == TR_S02 ? inv(a.c2) : mk(1, 0);
    const int jr = kWave - 1 - lane;
    // beta of my lag in the running sum: the first wave's moves to lane 0, the
    // last one's to lane 63
    double bw = 0.0;
    if (TR == TR_S02) bw = a.beta[(wfirst ? lane : jr) + 1];
    cd* const Ha = a.hist ? a.hist + (size_t)tix * 2 * (nt + 1) : nullptr;
    if (TR == TR_S02) {
        if (t0) Ha[0] = u[0];
        if (tL) Ha[nt + 1] = u[P - 1];
    }
    auto put_u = [&](int nstep) {
        int x = k, bb = b;
        asm volatile("" : "+v"(x), "+v"(bb));
        if ((fl & T_OUT_SNAP) && nstep % a.snap_stride == 0) {
            const int j = nstep / a.snap_stride;
            cd* sp = a.snaps + ((size_t)bb * a.nsnap + j) * a.nx + o;
#pragma unroll
            for (int q = 0; q < P; ++q)
                if (s + q > 0 && s + q < n - 1 && !(q == 0 && dup)) sp[s + q] = u[q];
            cd* se = a.snap_ends + (((size_t)bb * a.nsnap + j) * a.N + x) * 2;
            if (t0) se[0] = u[0];
            if (tL) se[1] = u[P - 1];
        }
        if (fl & T_OUT_TRACE) {
            cd* tr = a.trace + (size_t)(bb * a.N + x) * 2 * (nt + 1) + nstep;
            if (t0) tr[0] = u[0];
            if (tL) tr[nt + 1] = u[P - 1];
        }
    };
    auto until = [&](int nstep) {
        int m = kWave;
        if (special & T_OUT_SNAP) m = min(m, a.snap_stride - nstep % a.snap_stride);
        return (special & T_OUT_TRACE) ? 1 : m;
    };
    if (special) put_u(0);
    double maxd = 0.0;
    int par = 0;
    cd uLc = zero, uRc = zero;                    // u of the nodes beside the wave

    for (int n0 = 0; n0 < nt; n0 += kWave) {
        const int nb = min(kWave, nt - n0);
        const size_t gi = ((size_t)b * a.ns + 2 * k) * nt + n0;
        const bool ok = lane < nb, okr = jr < nb;
        // the border copies, from their owners
        {
            const cd fr = rows_front<P>(u, dup);
            __syncthreads();
            if (l63) bx[3 * wv] = u[P - 1];
            if (l0) bx[3 * wv + 1] = fr;
            __syncthreads();
            if (!wfirst) uLc = bx[3 * (wv - 1)];
            if (!wlast) uRc = bx[3 * (wv + 1) + 1];
            __syncthreads();
        }
        cd acc = zero;                            // first wave: left end; last wave: right end
        if (wfirst || wlast) {
            const int jo = wfirst ? lane : jr;
            if (TR == TR_S02) {
                __threadfence_block();
                rows_far<4>(a.hist, a.beta, nt, false, tix, 1, n0, nullptr, lg);
                rows_fence();
                acc = lg[(wfirst ? 0 : kWave) + jo];
                rows_fence();
            }
            cd l = zero;
            if (wfirst ? lif && ok : rif && okr) {
                if (fl & T_FLUX_G) l = a.g_in[(wfirst ? gi - nt : gi) + jo];
                if ((fl & (wfirst ? T_IMP_L : T_IMP_R)) && n0 + jo == 0) l = mk(1, 0);
            }
            acc = acc - ic * l;
        }
        const bool me = wfirst ? (lif && l0) : (wlast && rif && l63);

        for (int i = 0; i < nb;) {
          const int ie = special ? min(nb, i + until(n0 + i)) : nb;
          for (; i < ie; ++i) {
            asm volatile("" ::: "memory");        // read the coefficients anew
            const cd uL = sel_c(l0, uLc, rows_up1<4>(u[P - 1], lane));
            const cd uR = sel_c(l63, uRc, rows_dn1<4>(rows_front<P>(u, dup), lane));
            auto stencil = [&](int q) {
                const cd up = sel_c(q == 0, uL, u[q == 0 ? 0 : q - 1]);
                const cd un = sel_c(q == P - 1, uR, u[q == P - 1 ? 0 : q + 1]);
                const double w = q == P - 1 ? wL : (q == 0 ? w0 : 4.0);
                return mk(fma(w, u[q].x, up.x) + un.x, fma(w, u[q].y, up.y) + un.y);
            };
            cd dF = stencil(0), dS = stencil(P - 1);
            if (me) {
                const cd h = cmul_x(cs, acc);
                if (wfirst) dF = dF + h;
                else dS = dS + h;
                lg[2 * kWave + i] = acc;
            }
            cd y[P];
            {
                cd iv[P], cb[P];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) iv[q] = F.inv(q);
                cd w = dF;
#pragma unroll
                for (int q = 0; q < P - 1; ++q) {
                    if (q + kAhead < P - 1) iv[q + kAhead] = F.inv(q + kAhead);
                    __builtin_amdgcn_sched_barrier(0);
                    cb[q] = F.cp(q);
                    if (q > 0) w = msub_x(stencil(q), cb[q - 1], w);
                    y[q] = cmul_x(w, iv[q]);
                }
#pragma unroll
                for (int q = P - 3; q >= 0; --q) y[q] = msub_x(y[q], F.cp(q), y[q + 1]);
            }
            const cd yF = sel_c(dup, y[1], y[0]);
            const cd yR = rows_dn1<4>(yF, lane);  // (lane 63: the next wave's is in RW F)
            cd D = msub_x(msub_x(dS, F.tl[0], y[P - 2]), F.tl[1], yR);
            rows_level<0>(D, F.k1(0), F.k2(0));
            rows_level<1>(D, F.k1(1), F.k2(1));
            rows_level<2>(D, F.k1(2), F.k2(2));
            rows_level<3>(D, F.k1(3), F.k2(3));
            cd S = cmul_x(F.W(0), rdlane(D, 15)), S2 = cmul_x(F.W(1), rdlane(D, 16));
#pragma unroll
            for (int r = 1; r < 3; ++r) {
                S = madd_x(S, F.W(2 * r), rdlane(D, 16 * r + 15));
                S2 = madd_x(S2, F.W(2 * r + 1), rdlane(D, 16 * r + 16));
            }
            cd X = madd_x(S + S2, D, F.invB());
            // the waves
            cd* be = bx + par * 3 * NW;
            par ^= 1;
            if (l63) be[3 * wv] = X;
            if (l0) {
                be[3 * wv + 1] = X;
                be[3 * wv + 2] = yF;
            }
            __syncthreads();
            const int h = lane & 31;
            cd bj = zero;
            if (h < 3 * NW) bj = be[h];
            cd yFn = zero;
            if (!wlast) yFn = be[3 * (wv + 1) + 2];
            const cd pr = cmul_x(F.tl[rows_tail(4) + 3], bj);
            const cd hs = mk(half_sum(pr.x), half_sum(pr.y));
            const cd XL = rdlane(hs, 0), XR = rdlane(hs, 32);
            cd C = cmul_x(F.tl[rows_tail(4)], XL);
            C = madd_x(C, F.tl[rows_tail(4) + 1], XR);
            C = madd_x(C, F.tl[rows_tail(4) + 2], yFn);
            X = X + C;
            const cd Xm = sel_c(l0, XL, rows_up1<4>(X, lane));
            {
                cd al[P], ga[P];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) { al[q] = F.al(q); ga[q] = F.ga(q); }
#pragma unroll
                for (int q = 0; q < P - 1; ++q) {
                    if (q + kAhead < P - 1) { al[q + kAhead] = F.al(q + kAhead); ga[q + kAhead] = F.ga(q + kAhead); }
                    __builtin_amdgcn_sched_barrier(0);
                    y[q] = madd_x(madd_x(y[q], al[q], Xm), ga[q], X);
                }
            }
            y[P - 1] = X;
            uLc = mk(2.0 * XL.x - uLc.x, 2.0 * XL.y - uLc.y);
            {
                const cd xf = madd_x(madd_x(yFn, alF, rdlane(X, kWave - 1)), gaF, XR);
                uRc = mk(2.0 * xf.x - uRc.x, 2.0 * xf.y - uRc.y);
            }
#pragma unroll
            for (int q = 0; q < P; ++q) u[q] = mk(2.0 * y[q].x - u[q].x, 2.0 * y[q].y - u[q].y);
            if (wfirst || wlast) {
                // my end's boundary value, and the running sum one lane on
                const cd ve = wfirst ? rdlane(y[0], 0) : rdlane(X, kWave - 1);
                if (l0) lg[i] = ve;
                acc = wfirst ? rows_roll_dn<4>(acc) : rows_roll_up<4, false>(acc);
                if (TR == TR_S02) acc = mk(fma(bw, ve.x, acc.x), fma(bw, ve.y, acc.y));
            }
          }
          if (special) put_u(n0 + i);
        }
        if (wfirst || wlast) {
            rows_fence();
            const cd v = lg[lane], sm = lg[2 * kWave + lane];
            rows_fence();
            if (ok) {
                if (TR == TR_S02) Ha[(wfirst ? 0 : nt + 1) + n0 + 1 + lane] = v;
                const bool on = wfirst ? lif : rif;
                cd* out = nullptr;
                const cd* old = nullptr;
                if (on && (fl & T_OUT_G)) {
                    const size_t ol = (wfirst ? gi - 2 * (size_t)nt : gi + nt) + lane;
                    out = a.g_out + ol;
                    if (fl & T_MAXDIFF) old = a.g_in + ol;
                } else if (on && (fl & T_OUT_COLS)) {
                    out = a.cols + ((size_t)task.f * 4 + ((fl & T_IMP_L) ? 0 : 1) + (wfirst ? 0 : 2)) * nt + n0 + lane;
                }
                if (out) {
                    cd l = zero;
                    if (fl & T_FLUX_G) l = a.g_in[(wfirst ? gi - nt : gi) + lane];
                    if ((fl & (wfirst ? T_IMP_L : T_IMP_R)) && n0 + lane == 0) l = mk(1, 0);
                    const cd rho = TR == TR_S02 ? 2.0 * madd(cc * sm, a.sigma, v) + l : 2.0 * (a.sigma * v) - l;
                    *out = rho;
                    if (old) maxd = fmax(maxd, sqrt(abs2(rho - *old)));
                }
            }
        }
    }

    if (fl & T_OUT_UT) {
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
}

template <int NW, int P, int TR>
__global__ __launch_bounds__(NW * kWave) void sweep_wide_kernel(SweepArgs a) {
    extern __shared__ cd smem[];
    wide_body<P, NW, TR>(a, a.task0 + blockIdx.x, smem);
}

hipError_t launch_wide_factor(const FactorArgs& a, int NW, hipStream_t st) {
    if (NW == 2) wide_factor_kernel<2, 5, 9><<<a.nf, 2 * kWave, 0, st>>>(a);
    else if (NW == 4) wide_factor_kernel<4, 5, 9><<<a.nf, 4 * kWave, 0, st>>>(a);
    else if (NW == 8) wide_factor_kernel<8, 5, 12><<<a.nf, 8 * kWave, 0, st>>>(a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int NW, int P>
static hipError_t launch_wide_p(const SweepArgs& a, int trans, hipStream_t st) {
    const size_t lds = sizeof(cd) * (wide_fixed(NW) + (size_t)wide_lds_fields(P, NW) * 64 * NW);
    if (trans == TR_S02) sweep_wide_kernel<NW, P, TR_S02><<<a.ntasks, NW * kWave, lds, st>>>(a);
    else sweep_wide_kernel<NW, P, TR_ROBIN><<<a.ntasks, NW * kWave, lds, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_sweep_wide(const SweepArgs& a, int trans, int NW, int P, hipStream_t st) {
    if (a.ntasks == 0) return hipSuccess;
    if (!a.fac || (trans != TR_S02 && trans != TR_ROBIN) || a.far_old) return hipErrorInvalidValue;
    if (trans == TR_S02 && (!a.hist || !a.beta)) return hipErrorInvalidValue;
    // one launch over the whole window (no chunked launches, no checkpoints)
    if (a.n_begin != 0 || a.n_end != a.nt) return hipErrorInvalidValue;
    switch (32 * NW + P) {
#define CASE(W, Q) case 32 * W + Q: return launch_wide_p<W, Q>(a, trans, st);
        CASE(2, 5) CASE(2, 6) CASE(2, 7) CASE(2, 8) CASE(2, 9)
        CASE(4, 5) CASE(4, 6) CASE(4, 7) CASE(4, 8) CASE(4, 9)
        CASE(8, 5) CASE(8, 6) CASE(8, 7) CASE(8, 8) CASE(8, 9) CASE(8, 10) CASE(8, 11) CASE(8, 12)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace swr
