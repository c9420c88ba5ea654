// swr_rows.h -- row form of the subdomain solver (static potential, Robin and
// S0^2): a task is swept by RW rows of 16 lanes, so a wave carries 4 / RW
// tasks.  Lane moves, factor records and the right-hand-side solve; shared by
// the sweep (swr_sweep_rows_kernel.h) and the factorisation (swr_rows_factor.hip).
//
// Scaling.  The subdomain matrix A = c M - S + M_W - sigma E is divided by
// i kappa (kappa = h / (3 dt), c M = i kappa tridiag(1, 4, 1)): the right-hand
// side is then the plain stencil sum u_{i-1} + 4 u_i + u_{i+1} (2 u at an end
// node), two real instructions per component and node.
//
// Nodes.  T = 16 RW lanes own the n nodes in order, P or P - 1 each with P =
// ceil(n / T).  With n = T (P - 1) + r, lanes t < r own P nodes, the others P - 1
// and their slot 0 holds a copy of the node to the left (the left lane's
// separator): its row is x = X_{t-1}.  So slot q of lane t is node s_t + q with
// s_t = t P - max(0, t - r) (the copy included), every lane's separator is slot
// P - 1, node 0 is slot 0 of lane 0 and node n - 1 is slot P - 1 of lane T - 1:
// no masks in the stencil, and the end values sit in fixed registers.  With
// fewer nodes than lanes (P = 1) lane t owns node t, lanes past n hold zeros.
//
// Solve.  Chunk interiors are eliminated against the separators as in
// swr_lane.h (A is complex symmetric, so the multiplier of row q is the c' of
// row q - 1).  The T separators are reduced by cyclic reduction inside each
// row of 16 lanes only (distances 1, 2, 4, 8: DPP row shifts, no LDS and no
// select); the rows are then coupled through the values on either side of
// their borders: X = D / B + sum_j W_j D_j with D_j the reduced right-hand
// sides of the 2 (RW - 1) border lanes and W precomputed.  The reduction over
// all 64 lanes that this replaces took six levels, three of them through
// ds_bpermute and two through lane swaps.
#pragma once
#include "swr_lane.h"

namespace swr {

// by value: a conditional of two lvalues would put both in scratch memory
__device__ inline cd sel_c(bool c, cd x, cd y) { return mk(c ? x.x : y.x, c ? x.y : y.y); }

template <int CTRL>
__device__ inline cd dpp_c(cd v) { return mk(dpp_shift<CTRL>(v.x), dpp_shift<CTRL>(v.y)); }

// value of lane t - 1 / t + 1 of the same task, zero where there is none
template <int RW>
__device__ inline cd rows_up1(cd v, int t) {
    if (RW == 1) return dpp_c<0x111>(v);              // row_shr:1
    const cd r = dpp_c<0x138>(v);                     // wave_shr:1
    if (RW == 2) return sel_c(t == 0, mk(0, 0), r);        // (the wave's other task)
    return r;
}
template <int RW>
__device__ inline cd rows_dn1(cd v, int t) {
    if (RW == 1) return dpp_c<0x101>(v);              // row_shl:1
    const cd r = dpp_c<0x130>(v);                     // wave_shl:1
    if (RW == 2) return sel_c(t == 16 * RW - 1, mk(0, 0), r);
    return r;
}

// the same moves for the running history sums, whose lanes without a source
// are not read: lane t <- t + 1, and lane t <- t - 1 (wrapping when WRAP)
template <int RW>
__device__ inline cd rows_roll_dn(cd v) { return RW == 1 ? dpp_c<0x101>(v) : dpp_c<0x130>(v); }
template <int RW, bool WRAP>
__device__ inline cd rows_roll_up(cd v) {
    if (RW == 1) return dpp_c<WRAP ? 0x121 : 0x111>(v);   // row_ror:1 / row_shr:1
    return dpp_c<WRAP ? 0x13C : 0x138>(v);                // wave_ror:1 / wave_shr:1
}

__device__ inline cd swap16_first(cd v) { return mk(swap16(v.x).first, swap16(v.y).first); }
__device__ inline cd swap16_second(cd v) { return mk(swap16(v.x).second, swap16(v.y).second); }

// lane 0's value on every lane of the task, and lane tl's (tl = T - 1 unless
// P = 1)
template <int RW>
__device__ inline cd rows_first(cd v) {
    if (RW == 4) return rdlane(v, 0);
    const cd r = dpp_c<0x150>(v);                     // row_newbcast:0
    return RW == 1 ? r : swap16_first(r);
}
template <int RW, int P>
__device__ inline cd rows_last(cd v, int tl) {
    if (RW == 4) return rdlane(v, tl);
    if (RW == 1 && P == 1) {
        const int src = (lane_id() & ~15) + tl;
        return mk(__shfl(v.x, src), __shfl(v.y, src));
    }
    const cd r = dpp_c<0x15F>(v);                     // row_newbcast:15
    return RW == 1 ? r : swap16_second(r);
}

// (the two small terms are summed before they meet D: one rounding at its size
// where four chained multiply-adds have four)
template <int L>
__device__ inline void rows_level(cd& D, cd k1, cd k2) {
    const cd Dm = dpp_c<0x110 + (1 << L)>(D), Dp = dpp_c<0x100 + (1 << L)>(D);
    D = D - madd_x(cmul_x(k1, Dm), k2, Dp);
}

// What a lane keeps of its record in registers: all of it, or with LDSF as
// many fields as the register file has room for beside u and y -- the cp first
// (a step reads them twice), then the tail -- the rest read from the
// workgroup's LDS copy
template <int P, int RW, bool LDSF>
struct RowsFac {
    static constexpr int T = 16 * RW;
    static constexpr int NT = rows_tail(RW), NI = 4 * (P - 1);
    static constexpr int ROOM = LDSF ? (kRowsRegs - 8 * P) / 4 : NI + NT;
    // fields by place: cp_0 .., tail, inv_0 .., al_0 .., ga_0 ..
    static constexpr int NR = ROOM < 1 ? 1 : (ROOM > NI + NT ? NI + NT : ROOM);
    static constexpr int place(int q, int j) {      // field j (inv, cp, al, ga) of slot q
        return j == 1 ? q : NT + (j == 0 ? 1 : j) * (P - 1) + q;
    }
    static constexpr int tplace(int i) { return P - 1 + i; }
    cd in[NR];
    const cd* lds;

    // rec: the record at this lane, fields T apart
    __device__ void load(const cd* rec) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < P - 1; ++q)
                if (place(q, j) < NR) in[place(q, j)] = rec[(4 * q + j) * T];
#pragma unroll
        for (int i = 0; i < NT; ++i)
            if (tplace(i) < NR) in[tplace(i)] = rec[(NI + i) * T];
    }
    __device__ cd get(int pl, int f) const { return pl < NR ? in[pl < NR ? pl : 0] : lds[f * T]; }
    __device__ cd inv(int q) const { return get(place(q, 0), 4 * q); }
    __device__ cd cp(int q) const { return get(place(q, 1), 4 * q + 1); }
    __device__ cd al(int q) const { return get(place(q, 2), 4 * q + 2); }
    __device__ cd ga(int q) const { return get(place(q, 3), 4 * q + 3); }
    __device__ cd tail(int i) const { return get(tplace(i), NI + i); }
    __device__ cd ae() const { return tail(0); }
    __device__ cd ce() const { return tail(1); }
    __device__ cd k1(int l) const { return tail(2 + l); }
    __device__ cd k2(int l) const { return tail(2 + kRowLevels + l); }
    __device__ cd invB() const { return tail(2 + 2 * kRowLevels); }
    __device__ cd W(int j) const { return tail(3 + 2 * kRowLevels + j); }
};

// Reduced system of the separators: X from its right-hand side D
template <int P, int RW, bool LDSF>
__device__ inline cd rows_reduce(const RowsFac<P, RW, LDSF>& F, cd D, int t) {
    rows_level<0>(D, F.k1(0), F.k2(0));
    rows_level<1>(D, F.k1(1), F.k2(1));
    rows_level<2>(D, F.k1(2), F.k2(2));
    rows_level<3>(D, F.k1(3), F.k2(3));
    if (RW == 1) return cmul_x(D, F.invB());
    // the border terms first, D / B last: one rounding fewer in X
    cd S;
    if (RW == 2) {
        // z: the border value on this row's side, zo: the one across
        const cd b0 = dpp_c<0x150>(D), b15 = dpp_c<0x15F>(D);
        const cd z = sel_c(t < 16, b15, b0);
        const cd s1 = swap16_first(z), s2 = swap16_second(z);
        const cd zo = sel_c(t < 16, s2, s1);
        S = madd_x(cmul_x(F.W(0), z), F.W(1), zo);
    } else {
        S = cmul_x(F.W(0), rdlane(D, 15));
        cd S2 = cmul_x(F.W(1), rdlane(D, 16));
#pragma unroll
        for (int r = 1; r < 3; ++r) {
            S = madd_x(S, F.W(2 * r), rdlane(D, 16 * r + 15));
            S2 = madd_x(S2, F.W(2 * r + 1), rdlane(D, 16 * r + 16));
        }
        S = S + S2;
    }
    return madd_x(S, D, F.invB());
}

// first real slot of a lane (dup: its slot 0 is a copy), for the left
// neighbour's separator row
template <int P>
__device__ inline cd rows_front(const cd (&v)[P], bool dup) {
    if (P < 2) return v[0];
    return sel_c(dup, v[P < 2 ? 0 : 1], v[0]);
}

// the mass stencil u_{i-1} + 4 u_i + u_{i+1} of slot q (2 u at an end node:
// weights w0, wL of slots 0 and P - 1); uL, uR: the neighbouring lanes' nodes
template <int P>
__device__ inline cd rows_stencil(const cd (&u)[P], cd uL, cd uR, double w0, double wL, int q) {
    const cd up = sel_c(q == 0, uL, u[q == 0 ? 0 : q - 1]);
    const cd un = sel_c(q == P - 1, uR, u[q == P - 1 ? 0 : q + 1]);
    const double w = q == P - 1 ? wL : (q == 0 ? w0 : 4.0);
    return mk(fma(w, u[q].x, up.x) + un.x, fma(w, u[q].y, up.y) + un.y);
}

// One step's solve A x = d: dF and dS the right-hand sides of slots 0 and
// P - 1 with the boundary terms in, rhs(q) those between; y the solution
template <int P, int RW, bool LDSF, class RHS>
__device__ __forceinline__ void rows_solve(const RowsFac<P, RW, LDSF>& F, cd dF, cd dS, RHS rhs, int t,
                                           bool dup, cd (&y)[P]) {
    const cd zero = mk(0, 0);
    // interior fields in LDS are read anew every step (the compiler would
    // otherwise keep them in registers across the loop)
    if (LDSF) asm volatile("" ::: "memory");
    // chunk interior: w_q = d_q - cp_{q-1} w_{q-1}, y_q = inv_q w_q - cp_q y_{q+1}.
    // From LDS the coefficients are read kAhead slots before their use,
    // held there by the scheduling barriers: read at their use, each of
    // the 2 P reads waited for LDS (2600 of about 6000 cycles a step at P = 12).
    constexpr int kAhead = P >= 14 ? 2 : 3;
    if constexpr (P > 1 && !LDSF) {
        cd w = dF;
        y[0] = cmul_x(w, F.inv(0));
#pragma unroll
        for (int q = 1; q < P - 1; ++q) {
            w = msub_x(rhs(q), F.cp(q - 1), w);
            y[q] = cmul_x(w, F.inv(q));
        }
#pragma unroll
        for (int q = P - 3; q >= 0; --q) y[q] = msub_x(y[q], F.cp(q), y[q + 1]);
    }
    if constexpr (P > 1 && LDSF) {
        cd iv[P], cp[P];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) { iv[q] = F.inv(q); cp[q] = F.cp(q); }
        cd w = dF;
#pragma unroll
        for (int q = 0; q < P - 1; ++q) {
            if (q + kAhead < P - 1) { iv[q + kAhead] = F.inv(q + kAhead); cp[q + kAhead] = F.cp(q + kAhead); }
            __builtin_amdgcn_sched_barrier(0);
            if (q > 0) w = msub_x(rhs(q), cp[q - 1], w);
            y[q] = cmul_x(w, iv[q]);
        }
        cd cb[P];
#pragma unroll
        for (int q = P - 3; q > P - 3 - 2 * kAhead; --q) cb[q] = F.cp(q);
#pragma unroll
        for (int q = P - 3; q >= 0; --q) {
            if (q - 2 * kAhead >= 0) cb[q - 2 * kAhead] = F.cp(q - 2 * kAhead);
            __builtin_amdgcn_sched_barrier(0);
            y[q] = msub_x(y[q], cb[q], y[q + 1]);
        }
    }
    cd D = dS;
    if (P > 1) {
        // first real node's value for the left neighbour (a copy's y is zero)
        cd yF = y[0];
        if (P == 2) yF = sel_c(dup, zero, yF);
        if (P > 2) yF = sel_c(dup, y[P > 2 ? 1 : 0], yF);
        const cd yR = rows_dn1<RW>(yF, t);
        D = msub_x(msub_x(D, F.ae(), y[P > 1 ? P - 2 : 0]), F.ce(), yR);
    }
    const cd X = rows_reduce(F, D, t);
    if constexpr (P > 1) {
        cd al[P], ga[P];
        if (LDSF) {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) { al[q] = F.al(q); ga[q] = F.ga(q); }
            __builtin_amdgcn_sched_barrier(0);
        }
        const cd Xm = rows_up1<RW>(X, t);
#pragma unroll
        for (int q = 0; q < P - 1; ++q) {
            if (LDSF) {
                if (q + kAhead < P - 1) { al[q + kAhead] = F.al(q + kAhead); ga[q + kAhead] = F.ga(q + kAhead); }
                __builtin_amdgcn_sched_barrier(0);
                y[q] = madd_x(madd_x(y[q], al[q], Xm), ga[q], X);
            } else {
                y[q] = madd_x(madd_x(y[q], F.al(q), Xm), F.ga(q), X);
            }
        }
    }
    y[P - 1] = X;
}

// node of slot 0, and whether that slot is a copy of the node to the left
template <int P, int RW>
__device__ inline void rows_place(int n, int t, int& s, bool& dup) {
    constexpr int T = 16 * RW;
    const int r = n - T * (P - 1);
    dup = P > 1 && t >= r;
    s = t * P - (P > 1 ? max(0, t - r + 1) : 0);
}

}  // namespace swr
