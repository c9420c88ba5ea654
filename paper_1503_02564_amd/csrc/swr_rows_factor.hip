// swr_rows_factor.hip -- assembly and factorisation of the subdomain matrices
// for the row form of the static sweep (swr_rows.h): one wave per (potential,
// subdomain) record, every task slot of the wave computing the same record.
//
// On a fine mesh (dt / h^2 >> 1) the matrix is nearly a discrete Laplacian: the
// couplings are of size 3 dt / h^2 and what a step depends on, mass and
// potential, is the small sum of a row.  Pivots formed by subtraction keep that
// sum only to 3 dt / h^2 units in the last place, an error that is the same
// every step (at dt / h^2 = 1e5 about 1e-12 of u a step).  So the sums ("excess")
// are carried beside the couplings and every pivot is formed as excess plus
// couplings, which have one sign: no cancellation in the chunk elimination, in
// the reduction levels or in the coupling of the rows.  In an emulation over
// random meshes at dt / h^2 = 5e4 .. 3e5 the error of a step from the factors fell
// from 6e-13 to below 1e-14.
//
// Runs once per solve.  What bounds it is the chain of P - 1 pivots and four
// reduction levels with one complex reciprocal each, a few microseconds; the
// records of a row count are built by one launch.
#include <type_traits>

#include "swr_rows.h"

namespace swr {

template <int P, int RW>
__device__ inline void rows_factor_body(const FactorArgs& a, int f) {
    constexpr int T = 16 * RW, PI = P > 1 ? P - 1 : 1;
    const int lane = threadIdx.x, t = lane % T;
    const int k = f % a.N, v = f / a.N;
    const int n = a.J[k] + 1, o = a.off[k];
    const bool lif = k > 0, rif = k < a.N - 1;
    const double kap = a.h / (3.0 * a.dt);
    // rows over i kappa: (x + i y) / (i kappa) = (y - i x) / kappa
    const double p1 = 1.0 / (a.h * kap), q1 = a.h / (12.0 * kap), ik = 1.0 / kap;
    const cd sig = mk(a.sigma.y * ik, -a.sigma.x * ik);
    int s;
    bool dup;
    rows_place<P, RW>(n, t, s, dup);
    const double* V = a.V ? a.V + (size_t)v * a.nx + o : nullptr;
    // (V(t,x): the mean of the step's two rows, eq. CNS_L)
    auto W = [&](int i) {
        if (!V || i < 0 || i >= n) return 0.0;
        return a.steps ? 0.5 * (V[a.nx + i] + V[i]) : V[i];
    };
    const cd zero = mk(0, 0), one = mk(1, 0);
    // node i: minus its couplings to i - 1 and i + 1, and the sum of its row
    auto row = [&](int i, cd& cl, cd& cr, cd& ex) {
        cl = cr = ex = zero;
        if (i >= n) { ex = one; return; }             // no node (P = 1)
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
    // m_q = -cp_q; al, ga: response to the separators; de = 1 - al - ga, the
    // response to the row sums
    cd m[PI], al[PI], ga[PI], de[PI];
    cd mp = zero, wa = zero, wd = zero;
    bool started = false;                             // a real row has been met
#pragma unroll
    for (int q = 0; q < P - 1; ++q) {
        cd cl, cr, ex;
        row(s + q, cl, cr, ex);
        const bool real = !(q == 0 && dup);           // (a copy's fields are zero)
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
    if (P > 1) {
        ga[PI - 1] = m[PI - 1];
#pragma unroll
        for (int q = P - 3; q >= 0; --q) {
            al[q] = madd(al[q], m[q], al[q + 1]);
            de[q] = madd(de[q], m[q], de[q + 1]);
            ga[q] = m[q] * ga[q + 1];
        }
        if (dup) {
            al[0] = one;                              // the copy: x = X_{t-1}
            ga[0] = zero;
            de[0] = zero;
        }
#pragma unroll
        for (int q = 0; q < P - 1; ++q) {
            rec[(4 * q + 2) * T] = al[q];
            rec[(4 * q + 3) * T] = ga[q];
        }
    }
    cd cl, cr, ex;
    row(s + P - 1, cl, cr, ex);
    // responses of this lane's last interior node and of its first real node
    // (the left neighbour's row); without interior nodes, the separators
    cd aL = one, dL = zero, gF = one, dF = zero;
    if (P > 1) {
        aL = al[PI - 1];
        dL = de[PI - 1];
        gF = sel_c(dup, sel_c(P > 2, ga[P > 2 ? 1 : 0], one), ga[0]);
        dF = sel_c(dup, sel_c(P > 2, de[P > 2 ? 1 : 0], zero), de[0]);
    }
    const cd gR = rows_dn1<RW>(gF, t), dR = rows_dn1<RW>(dF, t);
    // reduced rows -At X_{t-1} + B X_t - Ct X_{t+1} with sum Et, B = Et + At + Ct
    cd At = cl * aL, Ct = cr * gR, Et = madd(madd(ex, cl, dL), cr, dR);
    // a row of 16 lanes for itself: the couplings across its borders become
    // two right-hand sides (spikes), the sums a third
    const bool rf = (t & 15) == 0, rl = (t & 15) == 15;
    cd ps = sel_c(rf, At, zero), qs = sel_c(rl, Ct, zero), ds = Et;
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
        At = k1 * Am;
        Ct = k2 * Cp;
        tail[(2 + L) * T] = -k1;
        tail[(2 + kRowLevels + L) * T] = -k2;
    };
    level(std::integral_constant<int, 0>{});
    level(std::integral_constant<int, 1>{});
    level(std::integral_constant<int, 2>{});
    level(std::integral_constant<int, 3>{});
    cd iB = inv((Et + At) + Ct);
    ps = ps * iB;
    qs = qs * iB;
    ds = ds * iB;
    if (P == 1 && t >= n) iB = zero;                  // no node: zero
    tail[(2 + 2 * kRowLevels) * T] = iB;
    // y = D / B is a row's solution with zero across its borders, X = y + ps
    // X_{row start - 1} + qs X_{row end + 1}, and ps + qs + ds = 1
    auto at = [&](cd x, int l) { return mk(__shfl(x.x, l), __shfl(x.y, l)); };
    if (RW == 2) {
        const int b = lane - t;
        const cd q15 = at(qs, b + 15), d15 = at(ds, b + 15), p16 = at(ps, b + 16), d16 = at(ds, b + 16);
        const cd i15 = at(iB, b + 15), i16 = at(iB, b + 16);
        const cd g = inv(madd(d16, p16, d15));        // 1 - p16 q15
        // row 0: qs X_16, X_16 = g (y16 + p16 y15); row 1: ps X_15
        const cd own = sel_c(t < 16, qs * (g * (p16 * i15)), ps * (g * (q15 * i16)));
        const cd oth = sel_c(t < 16, qs * (g * i16), ps * (g * i15));
        tail[(3 + 2 * kRowLevels) * T] = own;
        tail[(4 + 2 * kRowLevels) * T] = oth;
    }
    if (RW == 4) {
        // unknowns e_0, s_1, e_1, s_2, e_2, s_3 (e_r = X at lane 16 r + 15, s_r
        // at 16 r): x - ps e_{r-1} - qs s_{r+1} = y.  Lane j solves for y = the
        // j-th unit vector (j < 6), scaled by 1 / B of that lane.  O: minus the
        // off-diagonal entries, xs: row sums.
        cd O[6][6], xs[6], x[6];
        const int j = lane % 6;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int r = (i + 1) / 2;                // row of lanes of unknown i
            const int l = (i & 1) ? 16 * r : 16 * r + 15;
            const cd p = at(ps, l), q = at(qs, l), ib = at(iB, l);
#pragma unroll
            for (int c = 0; c < 6; ++c) O[i][c] = zero;
            if (r > 0) O[i][2 * (r - 1)] = p;
            if (r < 3) O[i][2 * r + 1] = q;
            xs[i] = at(ds, l);
            x[i] = sel_c(i == j, ib, zero);
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
        // weights of my lane: ps e_{r-1} + qs s_{r+1} for every unit vector
        const int r = t >> 4;
#pragma unroll
        for (int jj = 0; jj < 6; ++jj) {
            cd e[3], sn[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                e[q] = at(x[2 * q], jj);
                sn[q] = at(x[2 * q + 1], jj);
            }
            cd wj = zero;
            if (r > 0) wj = ps * sel_c(r == 1, e[0], sel_c(r == 2, e[1], e[2]));
            if (r < 3) wj = madd(wj, qs, sel_c(r == 0, sn[0], sel_c(r == 1, sn[1], sn[2])));
            if (P == 1 && t >= n) wj = zero;
            tail[(3 + 2 * kRowLevels + jj) * T] = wj;
        }
    }
}

// records of the subdomains with this row count and PLO <= P <= PHI
template <int P, int PHI, int RW>
__device__ inline void rows_factor_pick(const FactorArgs& a, int f, int p) {
    if (p == P) rows_factor_body<P, RW>(a, f);
    else if constexpr (P < PHI) rows_factor_pick<P + 1, PHI, RW>(a, f, p);
}

template <int RW, int PLO, int PHI>
__global__ __launch_bounds__(64) void rows_factor_kernel(FactorArgs a) {
    const int f = blockIdx.x;
    const int pr = a.Pk[f % a.N];                     // P + 32 RW of the subdomain (0: another form)
    if (pr / 32 != RW) return;
    rows_factor_pick<PLO, PHI, RW>(a, f, pr % 32);
}

hipError_t launch_rows_factor(const FactorArgs& a, int RW, int pmax, hipStream_t st) {
    if (RW == 4 && pmax <= kMaxP) rows_factor_kernel<4, 1, 8><<<a.nf, 64, 0, st>>>(a);
    else if (RW == 2 && pmax <= kRowsMaxP) rows_factor_kernel<2, 5, 16><<<a.nf, 64, 0, st>>>(a);
    else if (RW == 1 && pmax <= 14) rows_factor_kernel<1, 1, 14><<<a.nf, 64, 0, st>>>(a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace swr
