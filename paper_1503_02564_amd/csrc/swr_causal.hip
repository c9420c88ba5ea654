// swr_causal.hip -- exact causal solve of the interface problem
// (I - L) g = d for a time-independent potential (Besse & Xing,
// arXiv 1503.02564, Secs. 3-4).
//
// Every block of L is lower triangular in time (Props. 3-4), so with C_m the
// matrix of the m-th Toeplitz coefficients of all blocks, time step n reads
//     (I - C_0) g_n = d_n + sum_{s<n} C_{n-s} g_s.
// Per time step the unknowns of interface j (between subdomains j and j+1)
// are p_j = (r_j, l_{j+1}) (slots 2j, 2j+1).  Row r_j is subdomain j+1's left
// output, row l_{j+1} subdomain j's right output, so (I - C_0) is block
// tridiagonal with 2x2 blocks
//     D_j = [[1, -x1_{j+1}], [-x4_j, 1]],  U_j = [[-x2_{j+1}, 0], [0, 0]],
//     L_j = [[0, 0], [0, -x3_j]]
// (x_p^{k} the lag-0 entry of X^{k,p}).  Up to 64 interfaces it is reduced by
// block parallel cyclic reduction on one wave, above by block elimination as
// two prefix sums over a workgroup; the multipliers are computed once.  Both
// are stable when the system is block diagonally dominant
// (max_j ||D_j^{-1}|| (||L_j|| + ||U_j||) < 1), which setup checks.
//
// Time is processed in super-blocks of 256 steps (absolute windows) and,
// inside them, in blocks of kTb steps (above 64 interfaces 2 to 8).  The contribution of every earlier
// super-block to the outputs being solved is formed by one block-Toeplitz
// product on the matrix cores (launch_ltt).  `causal_far_kernel` adds to d that product and
// the contribution of the earlier blocks of the current super-block (a short
// rectangle, one workgroup per subdomain and problem; for a batch of
// problems with one potential `causal_far_mfma_kernel`, one
// wave per subdomain and eight problems on the matrix cores);
// `causal_near_kernel` then
// marches through the block on one workgroup per problem: wave 0 runs the
// per-step PCR solve and adds the lag-1 and lag-2 history, while the other
// waves gather the lags >= 3 of the step two ahead, from the block's g kept in
// LDS and the lag coefficients kept in registers.  `causal_march_kernel` does
// the same above 64 interfaces.
//
// These kernels and the history products run at raised wave priority: beside the
// sweeps of the other streams they are the chain everything waits for (100
// subdomains x 32 problems, 768 steps 4.53 -> 4.27 ms, 200 x 16 4.62 -> 4.42).
#include <algorithm>
#include <type_traits>

#include "swr_common.h"

namespace swr {

constexpr int kTb = kNearTb;                  // near block (time steps)
constexpr int kNearClasses = 4;                            // gather threads per subdomain
constexpr int kNearLags = kTb / kNearClasses;              // lags per thread: c+3, c+3+C, ...
constexpr int kNearGroup = 4;                              // lags whose loads are issued together
// gather threads: kNearClasses per subdomain, N <= kWave + 1 subdomains
constexpr int kNearGather = (kNearClasses * (kWave + 1) + kWave - 1) / kWave * kWave;
constexpr int kNearThreads = kWave + kNearGather;
constexpr int kNearCols = kNearSlots + 2;                  // slot q in column q + 1; 0 and ns + 1 stay zero
static_assert(kTb % (kNearClasses * kNearGroup) == 0, "near block: whole lag groups");
// per-potential record of the one-wave form: PCR multipliers and inverse
// diagonals [kPcrRec][64], then the near kernel's lag coefficients packed by
// thread: gather [kNearLags][4][kNearGather] (lags >= 3), solver [2][4][64]
// (lags 1, 2), zero where the coupling does not exist
constexpr size_t kNearPackG = (size_t)kNearLags * 4 * kNearGather;
constexpr size_t kFastRec = (size_t)kPcrRec * kWave + kNearPackG + 2 * 4 * kWave;
size_t causal_fast_rec() { return kFastRec; }

struct C2x2 { cd a, b, c, d; };   // [[a, b], [c, d]]

__device__ inline C2x2 m2(cd a, cd b, cd c, cd d) { C2x2 r; r.a = a; r.b = b; r.c = c; r.d = d; return r; }
__device__ inline C2x2 operator*(const C2x2& x, const C2x2& y) {
    return m2(madd(x.a * y.a, x.b, y.c), madd(x.a * y.b, x.b, y.d),
              madd(x.c * y.a, x.d, y.c), madd(x.c * y.b, x.d, y.d));
}
__device__ inline C2x2 operator-(const C2x2& x, const C2x2& y) {
    return m2(x.a - y.a, x.b - y.b, x.c - y.c, x.d - y.d);
}
__device__ inline C2x2 neg(const C2x2& x) { return m2(-x.a, -x.b, -x.c, -x.d); }
__device__ inline C2x2 inv2(const C2x2& x) {
    const cd idet = inv(x.a * x.d - x.b * x.c);
    return m2(x.d * idet, -(x.b * idet), -(x.c * idet), x.a * idet);
}
__device__ inline double norm_inf(const C2x2& x) {
    return fmax(sqrt(abs2(x.a)) + sqrt(abs2(x.b)), sqrt(abs2(x.c)) + sqrt(abs2(x.d)));
}
__device__ inline C2x2 shfl_up_m(const C2x2& x, int d, const C2x2& fill) {
    return m2(shfl_up_c(x.a, d, fill.a), shfl_up_c(x.b, d, fill.b), shfl_up_c(x.c, d, fill.c),
              shfl_up_c(x.d, d, fill.d));
}
__device__ inline C2x2 shfl_dn_m(const C2x2& x, int d, const C2x2& fill) {
    return m2(shfl_dn_c(x.a, d, fill.a), shfl_dn_c(x.b, d, fill.b), shfl_dn_c(x.c, d, fill.c),
              shfl_dn_c(x.d, d, fill.d));
}

// Block PCR multipliers of (I - C_0), one wave per potential, lane j =
// interface j (N - 1 <= 64 interfaces).  Record per lane: for each level
// K1 (4), K2 (4), then D^{-1} (4).  eta[v] = block dominance measure.
__global__ __launch_bounds__(64) void causal_pcr_setup_kernel(int N, int nt, const cd* cols, cd* pcr,
                                                              double* eta) {
    const int v = blockIdx.x, j = threadIdx.x;
    const int ni = N - 1;
    const cd* base = cols + (size_t)v * N * 4 * nt;
    auto col0 = [&](int k, int p) { return base[((size_t)k * 4 + p) * nt]; };
    const cd zero = mk(0, 0), one = mk(1, 0);
    const C2x2 I = m2(one, zero, zero, one), Z = m2(zero, zero, zero, zero);
    C2x2 D = I, Lm = Z, U = Z;
    if (j < ni) {
        const cd x1 = col0(j + 1, 0);
        const cd x2 = (j + 1 <= N - 2) ? col0(j + 1, 1) : zero;
        const cd x3 = (j >= 1) ? col0(j, 2) : zero;
        const cd x4 = col0(j, 3);
        D = m2(one, -x1, -x4, one);
        U = m2(-x2, zero, zero, zero);
        Lm = m2(zero, zero, zero, -x3);
    }
    cd* rec = pcr + (size_t)v * kFastRec + j;
    // per level: the coupling measure and the inverse diagonal block of the
    // current system, then one reduction.  Runs once per solve: keep the
    // loop rolled (the unrolled chain of 2x2 products is slow to compile).
#pragma unroll 1
    for (int l = 0; l <= kPcrLevels; ++l) {
        double e = norm_inf(inv2(D)) * (norm_inf(Lm) + norm_inf(U));
        e = wave_max(e);
        if (j == 0) eta[(size_t)v * (kPcrLevels + 1) + l] = e;
        const C2x2 Di = inv2(D);
        cd* r = rec + (size_t)(kPcrLevels * 8 + 4 * l) * kWave;
        r[0 * kWave] = Di.a; r[1 * kWave] = Di.b; r[2 * kWave] = Di.c; r[3 * kWave] = Di.d;
        if (l == kPcrLevels) break;
        const int d = 1 << l;
        const C2x2 Dm = shfl_up_m(D, d, I), Lmm = shfl_up_m(Lm, d, Z), Um = shfl_up_m(U, d, Z);
        const C2x2 Dp = shfl_dn_m(D, d, I), Lp = shfl_dn_m(Lm, d, Z), Up = shfl_dn_m(U, d, Z);
        const C2x2 K1 = (j - d >= 0) ? Lm * inv2(Dm) : Z;
        const C2x2 K2 = (j + d < kWave) ? U * inv2(Dp) : Z;
        const C2x2 Dn = D - K1 * Um - K2 * Lp;
        const C2x2 Ln = neg(K1 * Lmm), Un = neg(K2 * Up);
        D = Dn;
        Lm = Ln;
        U = Un;
        cd* q = rec + (size_t)l * 8 * kWave;
        q[0 * kWave] = K1.a; q[1 * kWave] = K1.b; q[2 * kWave] = K1.c; q[3 * kWave] = K1.d;
        q[4 * kWave] = K2.a; q[5 * kWave] = K2.b; q[6 * kWave] = K2.c; q[7 * kWave] = K2.d;
    }
}

__device__ inline void slot_src(int o, int N, int& k, int& pl, int& pr, int& sl, int& sr) {
    if ((o & 1) == 0) { k = o / 2 + 1; pl = 0; pr = 1; }
    else { k = (o - 1) / 2; pl = 2; pr = 3; }
    sl = (k >= 1) ? 2 * k - 1 : -1;
    sr = (k <= N - 2) ? 2 * k : -1;
}

struct FarArgs {
    int N, nt, ns, per_problem;
    int n0, nb;
    const cd* cols;    // [nv][N][4][nt]
    const cd* d;       // [B][ns][nt]
    const cd* g;       // [B][ns][nt]
    cd* out;           // d + contribution of steps s < n0: [B][ns][kTb], or [B][TB][ns] (far_out)
    const cd* facc;    // [nseg][B][ns][kCausalSuper]: contributions of the finished
                       // super-blocks to steps s_from .. s_from + kCausalSuper - 1
    int nseg;          // partials they come in (facc null when 0)
    int s_from;        // this kernel sums steps s_from <= s < n0
    int B;             // problems
};

// where output step i of slot o goes: by slot for the near march of blocks of
// kTb steps, by step for the general march, whose threads read it by interface
template <int TB>
__device__ inline size_t far_out(int b, int ns, int o, int i) {
    return TB == kTb ? ((size_t)b * ns + o) * TB + i : ((size_t)b * TB + i) * ns + o;
}

// One workgroup of NW waves per (subdomain k, problem).  Subdomain k feeds the
// output slots 2k - 2 (if k >= 1) and 2k + 1 (if k <= N - 2) from the same two
// source rows, g of slots 2k - 1 and 2k.  The source rows over [s_from, n0) and
// the coefficient rows over the lags they meet are staged in LDS.  A lane takes R
// consecutive output steps of one slot and a share of the sources, four at a
// time: each coefficient read serves R products (the next source meets the same
// coefficients one step on).  The shares are summed over lanes, then waves.  out = d + the finished
// super-blocks' partials + that contribution.  Which sources a share has, the
// order of terms in it and the order in which the shares are added depend on TB,
// NW and the range only.
//
// Bound: the round of memory latency of the staging and the launch.  Before (one
// output per lane, 1024 threads for two problems, two workgroups per compute
// unit and so four rounds of staging) and now, per launch: 16 potentials on 256
// subdomains, blocks of 8, beside the sweeps 41 -> 27.5 us; one problem on 64
// subdomains, blocks of 32: 7.5 -> 6.5 us.  One wave each from kFarWaves pairs on,
// where one wave per SIMD is there; with fewer, four waves shorten the chain (128
// subdomains, blocks of 8: 4.1 us).
// sum over the lanes of a wave that are equal modulo G, on the first G lanes
template <int G>
__device__ inline double far_lanes(double v) {
    if (G <= 2) v += dpp_shift<0x122>(v);              // row_ror:2
    if (G <= 4) v += dpp_shift<0x124>(v);
    if (G <= 8) v += dpp_shift<0x128>(v);
    const RowPair r = swap16(v);
    v = r.first + r.second;
    const RowPair h = swap32(v);
    return h.first + h.second;
}

template <int TB, int NW>
__global__ __launch_bounds__(NW * kWave) void causal_far_kernel(FarArgs f) {
    __builtin_amdgcn_s_setprio(2);
    constexpr int NT = NW * kWave, R = TB < 4 ? TB : 4, GROUPS = 2 * TB / R, SPLITS = NT / GROUPS;
    constexpr int kWin = kCausalSuper + TB, kPad = 4;   // coefficient rows: kPad zeros first
    constexpr int OUT = 2 * TB;
    __shared__ cd sx[2][kCausalSuper + kPad];           // zeros from len on
    __shared__ cd sc[4][kPad + kWin];
    static_assert(NW * OUT <= 4 * (kPad + kWin) && GROUPS <= 16 && GROUPS > 1, "shares: lanes, then waves");
    const int k = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
    const bool hasl = k >= 1, hasr = k <= f.N - 2;      // source rows 2k - 1, 2k
    const int len = f.n0 - f.s_from;                    // < kCausalSuper
    const cd zero = mk(0, 0);
    // rows of coefficients: p = 0, 1: slot 2k - 2 with the left, right source;
    // p = 2, 3: slot 2k + 1
    const int v = f.per_problem ? b : 0;
    const cd* cr = f.cols + (size_t)(v * f.N + k) * 4 * f.nt;
    const cd* xr = f.g + ((size_t)b * f.ns + 2 * k - 1) * f.nt + f.s_from;
    // every load is in flight before the first is stored
    constexpr int kCt = (kWin + NT - 1) / NT, kXt = (kCausalSuper + NT - 1) / NT;
    cd c[4][kCt], x[2][kXt];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const bool ok = (p == 0 || p == 2 ? hasl : hasr) && (p < 2 ? hasl : hasr);
#pragma unroll
        for (int m = 0; m < kCt; ++m) {
            const int e = t + m * NT;
            c[p][m] = zero;
            if (ok && e < len + TB && e < f.nt) c[p][m] = cr[(size_t)p * f.nt + e];
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int m = 0; m < kXt; ++m) {
            const int e = t + m * NT;
            x[q][m] = zero;
            if ((q == 0 ? hasl : hasr) && e < len) x[q][m] = xr[(size_t)q * f.nt + e];
        }
    // outputs: lane o (< OUT) of the last step
    const int oh = t / TB, oi = t % TB, on = f.n0 + oi;
    const int oslot = oh == 0 ? 2 * k - 2 : 2 * k + 1;
    const bool out_ok = t < OUT && (oh == 0 ? hasl : hasr) && oi < f.nb;
    cd r = zero;
    if (out_ok) {
        r = f.d[((size_t)b * f.ns + oslot) * f.nt + on];
        const size_t seg_stride = (size_t)f.B * f.ns * kCausalSuper;
        const cd* fp = f.facc + ((size_t)b * f.ns + oslot) * kCausalSuper + (on - f.s_from);
        for (int q = 0; q < f.nseg; ++q) r = r + fp[q * seg_stride];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (t < kPad) sc[p][t] = zero;
#pragma unroll
        for (int m = 0; m < kCt; ++m) {
            const int e = t + m * NT;
            if (e < kWin) sc[p][kPad + e] = c[p][m];
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (t < kPad) sx[q][kCausalSuper + t] = zero;
#pragma unroll
        for (int m = 0; m < kXt; ++m) {
            const int e = t + m * NT;
            if (e < kCausalSuper) sx[q][e] = x[q][m];
        }
    }
    __syncthreads();
    const int grp = t % GROUPS, sp = t / GROUPS;
    const int h = grp / (TB / R), i0 = grp % (TB / R) * R;
    const int per = (len + 4 * SPLITS - 1) / (4 * SPLITS) * 4;
    const int e_lo = sp * per, e_hi = min(len, e_lo + per);
    cd acc[R];
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] = zero;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        // output i0 + q meets source e at lag len + i0 + q - e
        const cd* cw = sc[2 * h + side] + kPad + len + i0;
        const cd* xw = sx[side];
        cd w[R + 3];                                    // lags of outputs 0 .. R - 1 and sources e .. e + 3
#pragma unroll
        for (int q = 0; q < R - 1; ++q) w[q + 4] = e_lo < e_hi ? cw[q + 1 - e_lo] : zero;
        for (int e = e_lo; e < e_hi; e += 4) {
            cd xs[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[3 - j] = cw[-e - j];
                xs[j] = xw[e + j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int q = 0; q < R; ++q) acc[q] = madd(acc[q], w[3 + q - j], xs[j]);
#pragma unroll
            for (int q = R - 2; q >= 0; --q) w[q + 4] = w[q];
        }
    }
    // the wave's shares: lanes of a group are GROUPS apart
#pragma unroll
    for (int q = 0; q < R; ++q) {
        acc[q].x = far_lanes<GROUPS>(acc[q].x);
        acc[q].y = far_lanes<GROUPS>(acc[q].y);
    }
    __syncthreads();
    cd* part = &sc[0][0];                               // [wave][output]
    if (t % kWave < GROUPS) {
#pragma unroll
        for (int q = 0; q < R; ++q) part[t / kWave * OUT + h * TB + i0 + q] = acc[q];
    }
    __syncthreads();
    if (out_ok) {
        cd y = part[t];
#pragma unroll
        for (int q = 1; q < NW; ++q) y = y + part[q * OUT + t];
        f.out[far_out<TB>(b, f.ns, oslot, oi)] = r + y;
    }
}

// Matrix-core form of the same sums for a large batch with one potential
// (batch_form; TB = 8 or 32).  One wave per (subdomain k, 8 problems): the
// rows of the product are the block's TB outputs of the two slots subdomain
// k feeds (slot 2k - 2, then slot 2k + 1: 2 TB rows in 16-row blocks), the
// columns the 8 problems' real and imaginary parts, and K runs over the
// sources s in [s_from, n0) of the left row (g of slot 2k - 1), then of the
// right row (slot 2k), four per instruction.  Two accumulators per row block
// collect Re C [Re x | Im x] and Im C [Re x | Im x]; neighbouring lanes
// combine them (Re y = Re C Re x - Im C Im x, Im y = Re C Im x + Im C Re x).
// At N = 500, B = 32 a launch has 2000 waves where the form above has
// 128000, so it finds room quickly beside the sweeps that run concurrently
// on the other streams.  Per output: d, the finished super-blocks' partials,
// then the product (sources ascending in fours, left row before right).
typedef double fd4 __attribute__((ext_vector_type(4)));
static __device__ inline fd4 far_mfma(double a, double b, fd4 c) {
    // lane l supplies A[l%16][l/16] and B[l/16][l%16]; accumulator register
    // q of lane l is D[l/16 + 4q][l%16]
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
static __device__ inline double far_swap_pair(double v) {   // the value of lane l ^ 1
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __builtin_amdgcn_mov_dpp(t.x, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
    t.y = __builtin_amdgcn_mov_dpp(t.y, 0xB1, 0xf, 0xf, false);
    return *reinterpret_cast<double*>(&t);
}
constexpr int kFarMfmaB = 8;    // problems per wave of the matrix-core form
constexpr size_t kFarWaves = 1024;

template <int TB>
__global__ __launch_bounds__(64) void causal_far_mfma_kernel(FarArgs f) {
    __builtin_amdgcn_s_setprio(2);
    static_assert((2 * TB) % 16 == 0, "whole 16-row blocks");
    constexpr int RB = 2 * TB / 16;
    const int k = blockIdx.x, b0 = blockIdx.y * kFarMfmaB;
    const int lane = threadIdx.x, r = lane & 15, kq = lane >> 4;
    const bool hasl = k >= 1, hasr = k <= f.N - 2;       // source rows 2k - 1, 2k
    const cd* crow = f.cols + (size_t)k * 4 * f.nt;       // coefficient rows p = 0..3
    // B operand column r: problem b0 + r / 2, real (r even) or imaginary part
    const int bcol = b0 + (r >> 1), part = r & 1;
    const bool col_ok = bcol < f.B;
    fd4 d1[RB], d2[RB];
#pragma unroll
    for (int I = 0; I < RB; ++I) {
        d1[I] = fd4{0.0, 0.0, 0.0, 0.0};
        d2[I] = fd4{0.0, 0.0, 0.0, 0.0};
    }
    // operands of U k-steps are loaded one group ahead of the instructions
    // that use them (k-steps past the range load zeros)
    constexpr int U = RB == 1 ? 4 : 2;
    const int nblk = (f.n0 - f.s_from + 3) / 4;
    for (int side = 0; side < 2; ++side) {
        if (side == 0 ? !hasl : !hasr) continue;          // uniform over the wave
        const double* gs = reinterpret_cast<const double*>(
                               f.g + ((size_t)(col_ok ? bcol : 0) * f.ns + 2 * k - 1 + side) * f.nt) + part;
        double bv[2][U];
        cd av[2][U][RB];
        auto fetch = [&](int buf, int j0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = f.s_from + 4 * (j0 + u) + kq;
                const bool s_ok = s < f.n0;
                bv[buf][u] = (col_ok && s_ok) ? gs[2 * (size_t)s] : 0.0;
#pragma unroll
                for (int I = 0; I < RB; ++I) {
                    // A row r of block I: output R = 16 I + r, slot h = R / TB,
                    // step i = R % TB
                    const int R = 16 * I + r, h = R / TB, lag = f.n0 + R % TB - s;
                    const bool a_ok = s_ok && (h == 0 ? hasl : hasr) && lag < f.nt;
                    av[buf][u][I] = a_ok ? crow[(size_t)(2 * h + side) * f.nt + lag] : mk(0, 0);
                }
            }
        };
        auto apply = [&](int buf) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int I = 0; I < RB; ++I) {
                    d1[I] = far_mfma(av[buf][u][I].x, bv[buf][u], d1[I]);
                    d2[I] = far_mfma(av[buf][u][I].y, bv[buf][u], d2[I]);
                }
            }
        };
        fetch(0, 0);
        for (int j0 = 0; j0 < nblk; j0 += 2 * U) {
            fetch(1, j0 + U);
            apply(0);
            if (j0 + U >= nblk) break;
            fetch(0, j0 + 2 * U);
            apply(1);
        }
    }
    const size_t seg_stride = (size_t)f.B * f.ns * kCausalSuper;
#pragma unroll
    for (int I = 0; I < RB; ++I) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double other = far_swap_pair(d2[I][q]);
            const double v = part ? d1[I][q] + other : d1[I][q] - other;
            const int R = 16 * I + kq + 4 * q, h = R / TB, i = R % TB;
            if (col_ok && (h == 0 ? hasl : hasr) && i < f.nb) {
                const int o = h == 0 ? 2 * k - 2 : 2 * k + 1, n = f.n0 + i;
                const size_t row = (size_t)bcol * f.ns + o;
                double acc = reinterpret_cast<const double*>(f.d + row * f.nt + n)[part];
                for (int q2 = 0; q2 < f.nseg; ++q2)
                    acc += reinterpret_cast<const double*>(f.facc + q2 * seg_stride + row * kCausalSuper +
                                                           (n - f.s_from))[part];
                reinterpret_cast<double*>(f.out + far_out<TB>(bcol, f.ns, o, i))[part] = acc + v;
            }
        }
    }
}

struct NearArgs {
    int N, nt, ns, per_problem;
    int n0, nb;
    const cd* cols;
    const cd* pcr;     // [nv][kFastRec]
    int levels;        // PCR levels run per step (the rest of the coupling is negligible)
    const cd* base;    // [B][ns][kTb]: d + far part
    cd* g;             // [B][ns][nt]
};


// neighbour values for the lag-1/lag-2 history: lane j - 1 / j + 1 (zero outside)
__device__ inline cd lane_up1(cd v) { return shfl_up1z(v); }
__device__ inline cd lane_dn1(cd v) { return shfl_dn1z(v); }

// sum over the four lanes of a quad (DPP quad permutations); every lane of
// the quad gets the same bits
template <int CTRL>
__device__ inline double quad_move(double v) {
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __builtin_amdgcn_update_dpp(0, t.x, CTRL, 0xf, 0xf, false);
    t.y = __builtin_amdgcn_update_dpp(0, t.y, CTRL, 0xf, 0xf, false);
    return *reinterpret_cast<double*>(&t);
}
__device__ inline cd quad_sum(cd v) {
    v = mk(v.x + quad_move<0xB1>(v.x), v.y + quad_move<0xB1>(v.y));   // lanes (1,0,3,2)
    return mk(v.x + quad_move<0x4E>(v.x), v.y + quad_move<0x4E>(v.y)); // lanes (2,3,0,1)
}

// One workgroup per problem.  Wave 0 solves the per-step block system; lane
// j owns interface j, i.e. slots 2j (r_j) and 2j+1 (l_{j+1}), and adds the
// lag-1 and lag-2 history itself from the solutions of the two previous
// steps it keeps in registers (slot 2j reads x1 of lane j and x0 of lane j+1
// through X^{j+1,1}, X^{j+1,2}; slot 2j+1 reads x1 of lane j-1 and x0 of lane
// j through X^{j,3}, X^{j,4}).  The other waves gather lags >= 3 of the step
// two ahead from the block's g kept in LDS, so a step costs one barrier and
// the solver never waits for LDS written in the same step.  They work per
// subdomain k: its two outgoing traces (slots 2k-1, 2k) enter exactly the
// slots 2k-2 (through X^{k,1}, X^{k,2}) and 2k+1 (through X^{k,3}, X^{k,4}),
// so each pair of LDS values read serves two slots; kNearClasses threads
// split the lags of one subdomain and sum through DPP.  Lags are taken in
// groups whose LDS loads are issued together: a source before the block or
// outside the interface range reads the zero row / zero columns of `gh`,
// which adds exact zeros.  Row s + 1 of `gh` holds, in turn, the base of step
// s (staged at the start), its full right-hand side (written by the gather
// two steps before) and its solution (written by the solver at step s).
__global__ __launch_bounds__(kNearThreads) void causal_near_kernel(NearArgs a) {
    __builtin_amdgcn_s_setprio(2);
    __shared__ cd gh[kTb + 1][kNearCols];
    __shared__ cd spcr[kPcrLevels * 8 + 4][kWave];
    const int b = blockIdx.x, v = a.per_problem ? b : 0;
    const int tid = threadIdx.x;
    const int ns = a.ns, nt = a.nt, n0 = a.n0, nb = a.nb;
    const int ni = a.N - 1;
    const cd zero = mk(0, 0);
    cd* gb = a.g + (size_t)b * ns * nt;
    const cd* bb = a.base + (size_t)b * ns * kTb;
    const cd* prec = a.pcr + (size_t)v * kFastRec;
    const cd* pk = prec + (size_t)kPcrRec * kWave;   // packed lag coefficients

    // gather role: subdomain k, lag class c (lags c+3, c+3+C, c+3+2C, ...).
    // wa*: slot 2k-2 from slots 2k-1, 2k; wb*: slot 2k+1 from the same pair.
    const int gt = tid - kWave;
    const int k = gt / kNearClasses, c = gt % kNearClasses;
    const bool gather = tid >= kWave && k < a.N;
    // a gather wave with no subdomain at all skips the sums (it would add
    // zeros and hold its SIMD)
    const bool gwave = tid >= kWave && ((tid & ~(kWave - 1)) - kWave) / kNearClasses < a.N;
    const bool has_a = gather && k >= 1, has_b = gather && k <= a.N - 2;
    const int kk = gather ? k : 0;
    // (coalesced reads of the table packed once per solve)
    cd wa0[kNearLags], wa1[kNearLags], wb0[kNearLags], wb1[kNearLags];
#pragma unroll
    for (int m = 0; m < kNearLags; ++m) { wa0[m] = zero; wa1[m] = zero; wb0[m] = zero; wb1[m] = zero; }
    if (tid >= kWave) {
#pragma unroll
        for (int m = 0; m < kNearLags; ++m) {
            const cd* q = pk + (size_t)m * 4 * kNearGather + gt;
            wa0[m] = q[0];
            wa1[m] = q[kNearGather];
            wb0[m] = q[2 * kNearGather];
            wb1[m] = q[3 * kNearGather];
        }
    }
    // solver role: lag-1 and lag-2 coefficients of my two slots
    const int j = tid;
    cd a0[2] = {zero, zero}, a1[2] = {zero, zero}, a2[2] = {zero, zero}, a3[2] = {zero, zero};
    if (tid < kWave) {
        const cd* q = pk + kNearPackG + j;
#pragma unroll
        for (int l = 0; l < 2; ++l) {
            a0[l] = q[(l * 4 + 0) * kWave];
            a1[l] = q[(l * 4 + 1) * kWave];
            a2[l] = q[(l * 4 + 2) * kWave];
            a3[l] = q[(l * 4 + 3) * kWave];
        }
    }
    // base (d + far part) of every step of the block -> its row of gh; then
    // the multipliers of the levels run and the matching inverse diagonal ->
    // LDS.  The lag coefficients above and the base are in flight together,
    // so the set-up waits for one round of memory latency (two when PCR
    // levels run).
    const int lev = a.levels;
    {
        constexpr int kIt = (kNearSlots * kTb + kNearThreads - 1) / kNearThreads;
        const int lim = ns * nb;
        // q = e / nb as (e * ceil(2^32 / nb)) >> 32: exact for e < 2^32 / kTb
        const unsigned long long rnb = (0x100000000ull + nb - 1) / nb;
        cd t[kIt];
#pragma unroll
        for (int u = 0; u < kIt; ++u) {
            const int e = tid + u * kNearThreads;
            const int q = (int)(((unsigned long long)e * rnb) >> 32), s = e - q * nb;
            t[u] = zero;
            if (e < lim) t[u] = bb[(size_t)q * kTb + s];
        }
#pragma unroll
        for (int u = 0; u < kIt; ++u) {
            const int e = tid + u * kNearThreads;
            const int q = (int)(((unsigned long long)e * rnb) >> 32), s = e - q * nb;
            if (e < lim) gh[s + 1][q + 1] = t[u];
        }
    }
    {
        constexpr int kIt = (kPcrLevels * 8 * kWave + kNearThreads - 1) / kNearThreads;
        const int lim = lev * 8 * kWave;
        cd t[kIt];
        cd di = zero;
#pragma unroll
        for (int u = 0; u < kIt; ++u) {
            const int e = tid + u * kNearThreads;
            t[u] = zero;
            if (e < lim) t[u] = prec[e];
        }
        if (tid < 4 * kWave) di = prec[(size_t)(kPcrLevels * 8 + 4 * lev) * kWave + tid];
#pragma unroll
        for (int u = 0; u < kIt; ++u) {
            const int e = tid + u * kNearThreads;
            if (e < lim) (&spcr[0][0])[e] = t[u];
        }
        if (tid < 4 * kWave) (&spcr[kPcrLevels * 8][0])[tid] = di;
    }
    // zero row (steps before the block) and zero columns (no such slot)
    for (int e = tid; e < kNearCols; e += kNearThreads) gh[0][e] = zero;
    for (int e = tid; e < kTb; e += kNearThreads) {
        gh[e + 1][0] = zero;
        gh[e + 1][ns + 1] = zero;
    }
    cd x0 = zero, x1 = zero, y0 = zero, y1 = zero;   // solutions of steps i-1 and i-2
    __syncthreads();
    // every load of the set-up has landed: the step loop then waits on no
    // memory counter, so its stores never hold a step
    __builtin_amdgcn_s_waitcnt(0);
    // lag-1 and lag-2 part of the next step's right-hand side, formed from
    // the solver's own registers before the step's barrier
    cd h0 = zero, h1 = zero;
    // neighbour values of the previous step's solution (lane j+1's x0, lane
    // j-1's x1): this step's lag-2 neighbours, shuffled once
    cd x0p = zero, x1m = zero;

    for (int i = 0; i < nb; ++i) {
        if (tid < kWave) {
            // right-hand side: base + lags >= 3 (gathered; steps 0 and 1 have
            // none in the block) + lags 1, 2 (h); lags reaching before the
            // block are in base
            cd p0 = zero, p1 = zero;
            if (j < ni) { p0 = gh[i + 1][2 * j + 1] + h0; p1 = gh[i + 1][2 * j + 2] + h1; }
#pragma unroll
            for (int l = 0; l < kPcrLevels; ++l) {
                if (l >= lev) break;                    // uniform over the workgroup
                // the multipliers are zero on lanes without a partner
                const int d = 1 << l;
                const cd q0m = shfl_up_raw(p0, d), q1m = shfl_up_raw(p1, d);
                const cd q0p = shfl_dn_raw(p0, d), q1p = shfl_dn_raw(p1, d);
                const cd* K = &spcr[l * 8][j];
                const cd k1a = K[0 * kWave], k1b = K[1 * kWave], k1c = K[2 * kWave], k1d = K[3 * kWave];
                const cd k2a = K[4 * kWave], k2b = K[5 * kWave], k2c = K[6 * kWave], k2d = K[7 * kWave];
                p0 = msub(msub(msub(msub(p0, k1a, q0m), k1b, q1m), k2a, q0p), k2b, q1p);
                p1 = msub(msub(msub(msub(p1, k1c, q0m), k1d, q1m), k2c, q0p), k2d, q1p);
            }
            const cd* Di = &spcr[kPcrLevels * 8][j];
            y0 = x0;
            y1 = x1;
            x0 = madd(Di[0] * p0, Di[1 * kWave], p1);
            x1 = madd(Di[2 * kWave] * p0, Di[3 * kWave], p1);
            if (j >= ni) { x0 = zero; x1 = zero; }
            if (j < ni) {
                gh[i + 1][2 * j + 1] = x0;
                gh[i + 1][2 * j + 2] = x1;
                gb[(size_t)(2 * j) * nt + n0 + i] = x0;
                gb[(size_t)(2 * j + 1) * nt + n0 + i] = x1;
            }
            // lags 1 (this step) and 2 (the step before) for step i+1
            const cd y0p = x0p, y1m = x1m;
            x0p = lane_dn1(x0);
            x1m = lane_up1(x1);
            h0 = madd(a1[0] * x0p, a0[0], x1);
            h1 = madd(a3[0] * x0, a2[0], x1m);
            if (i >= 1) {
                h0 = madd(madd(h0, a0[1], y1), a1[1], y0p);
                h1 = madd(madd(h1, a2[1], y1m), a3[1], y0);
            }
        } else if (gwave && i + 2 < nb) {
            // lags >= 3 of step i+2, from in-block steps up to i-1: lag
            // c+3+C*m reads row i - c - C*m (step i+2-lag), row 0 if earlier
            cd pa = zero, pb = zero;
#pragma unroll
            for (int g0 = 0; g0 < kNearLags; g0 += kNearGroup) {
                // first lag of the group: 3 + C*g0 <= i + 2 for some class
                if (i >= 1 + kNearClasses * g0) {
                    cd xl[kNearGroup], xr[kNearGroup];
#pragma unroll
                    for (int u = 0; u < kNearGroup; ++u) {
                        const int r = max(i - c - kNearClasses * (g0 + u), 0);
                        xl[u] = gh[r][2 * kk];
                        xr[u] = gh[r][2 * kk + 1];
                    }
#pragma unroll
                    for (int u = 0; u < kNearGroup; ++u) {
                        pa = madd(madd(pa, wa0[g0 + u], xl[u]), wa1[g0 + u], xr[u]);
                        pb = madd(madd(pb, wb0[g0 + u], xl[u]), wb1[g0 + u], xr[u]);
                    }
                }
            }
            pa = quad_sum(pa);
            pb = quad_sum(pb);
            if (c == 0 && has_a) gh[i + 3][2 * k - 1] = gh[i + 3][2 * k - 1] + pa;   // slot 2k-2
            if (c == 1 && has_b) gh[i + 3][2 * k + 2] = gh[i + 3][2 * k + 2] + pb;   // slot 2k+1
        }
        __syncthreads();
    }
}

// The near kernel's lag coefficients of one potential, packed by thread so
// that every launch reads them with coalesced loads: gather thread gt
// (subdomain k = gt / C, class c) gets, for lag c+3+C*m, X^{k,1..4} (those of
// slot 2k-2 from slots 2k-1, 2k and of slot 2k+1 from the same pair); solver
// lane j gets the lag-1 and lag-2 values of its two slots.  Zero where the
// slot or the source does not exist, or the lag is past nt or the near block.
__global__ __launch_bounds__(kNearGather) void causal_near_pack_kernel(int N, int nt, const cd* cols,
                                                                       cd* pcr) {
    const int v = blockIdx.x, gt = threadIdx.x;
    const cd zero = mk(0, 0);
    const cd* cbase = cols + (size_t)v * N * 4 * nt;
    cd* pk = pcr + (size_t)v * kFastRec + (size_t)kPcrRec * kWave;
    const int k = gt / kNearClasses, c = gt % kNearClasses;
    const bool gather = k < N;
    const bool has_a = gather && k >= 1, has_b = gather && k <= N - 2;
    const cd* cb = cbase + (size_t)(gather ? k : 0) * 4 * nt;
    for (int m = 0; m < kNearLags; ++m) {
        const int lag = c + 3 + kNearClasses * m;
        cd w0 = zero, w1 = zero, w2 = zero, w3 = zero;
        if (lag < nt && lag < kTb) {
            if (has_a) {
                w0 = cb[lag];
                if (k <= N - 2) w1 = cb[(size_t)nt + lag];
            }
            if (has_b) {
                if (k >= 1) w2 = cb[(size_t)2 * nt + lag];
                w3 = cb[(size_t)3 * nt + lag];
            }
        }
        cd* q = pk + (size_t)m * 4 * kNearGather + gt;
        q[0] = w0;
        q[kNearGather] = w1;
        q[2 * kNearGather] = w2;
        q[3 * kNearGather] = w3;
    }
    if (gt < kWave) {
        const int j = gt, ni = N - 1;
        cd* q = pk + kNearPackG + j;
        for (int l = 0; l < 2; ++l) {
            const int lag = l + 1;
            cd x0 = zero, x1 = zero, x2 = zero, x3 = zero;
            if (j < ni && lag < nt) {
                x0 = cbase[((size_t)(j + 1) * 4 + 0) * nt + lag];                        // x1_j
                if (j + 1 <= N - 2) x1 = cbase[((size_t)(j + 1) * 4 + 1) * nt + lag];   // x0_{j+1}
                if (j >= 1) x2 = cbase[((size_t)j * 4 + 2) * nt + lag];                  // x1_{j-1}
                x3 = cbase[((size_t)j * 4 + 3) * nt + lag];                              // x0_j
            }
            q[(l * 4 + 0) * kWave] = x0;
            q[(l * 4 + 1) * kWave] = x1;
            q[(l * 4 + 2) * kWave] = x2;
            q[(l * 4 + 3) * kWave] = x3;
        }
    }
}

hipError_t launch_causal_pcr_setup(int N, int nt, int nv, const cd* cols, cd* pcr, double* eta,
                                   hipStream_t st) {
    if (N > kWave + 1) return hipErrorInvalidValue;
    causal_pcr_setup_kernel<<<nv, 64, 0, st>>>(N, nt, cols, pcr, eta);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    causal_near_pack_kernel<<<nv, kNearGather, 0, st>>>(N, nt, cols, pcr);
    return hipGetLastError();
}

template <int TB>
static hipError_t launch_causal_far(int N, int nt, int ns, int B, int per_problem, int n0, int nb,
                                    const cd* cols, const cd* d, const cd* g, cd* out,
                                    const cd* facc, int nseg, int s_from, hipStream_t st) {
    // the staged rows hold less than one super-block of sources
    if (n0 - s_from < 0 || n0 - s_from >= kCausalSuper) return hipErrorInvalidValue;
    if (ns != 2 * (N - 1)) return hipErrorInvalidValue;
    FarArgs f{N, nt, ns, per_problem, n0, nb, cols, d, g, out, facc,
              facc ? nseg : 0, s_from, B};
    if constexpr (TB == 8 || TB == 32) {
        if (batch_form(N, B, per_problem)) {
            causal_far_mfma_kernel<TB><<<dim3(N, (B + kFarMfmaB - 1) / kFarMfmaB), 64, 0, st>>>(f);
            return hipGetLastError();
        }
    }
    if ((size_t)N * B >= kFarWaves) causal_far_kernel<TB, 1><<<dim3(N, B), kWave, 0, st>>>(f);
    else causal_far_kernel<TB, 4><<<dim3(N, B), 4 * kWave, 0, st>>>(f);
    return hipGetLastError();
}

hipError_t launch_causal_near(int N, int nt, int ns, int B, int per_problem, int n0, int nb,
                              const cd* cols, const cd* pcr, int levels, const cd* base, cd* g,
                              hipStream_t st) {
    if (ns > kNearSlots || N - 1 > kWave || levels < 0 || levels > kPcrLevels)
        return hipErrorInvalidValue;
    NearArgs a{N, nt, ns, per_problem, n0, nb, cols, pcr, levels, base, g};
    causal_near_kernel<<<B, kNearThreads, 0, st>>>(a);
    return hipGetLastError();
}

// the whole forward substitution: far part then near march, block by block
hipError_t launch_causal_fast(int N, int nt, int ns, int B, int per_problem, const cd* cols,
                              const cd* pcr, int levels, const cd* d, cd* base, cd* g, int n_lo,
                              int n_hi, const cd* facc, int nseg, int s_from, hipStream_t st) {
    if (n_lo % kTb != 0 || n_lo < 0 || n_hi > nt || s_from < 0 || s_from > n_lo)
        return hipErrorInvalidValue;
    for (int n0 = n_lo; n0 < n_hi; n0 += kTb) {
        const int nb = min(kTb, n_hi - n0);
        hipError_t e = launch_causal_far<kTb>(N, nt, ns, B, per_problem, n0, nb, cols, d, g, base,
                                              facc, nseg, s_from, st);
        if (e != hipSuccess) return e;
        e = launch_causal_near(N, nt, ns, B, per_problem, n0, nb, cols, pcr, levels, base, g, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// General path: up to kGenMaxIf interfaces.
//
// With L_j and U_j of one entry each, block elimination of (I - C_0) from the
// left keeps one new number per interface.  Write r_j, l_j (= l_{j+1} above) for
// the unknowns of interface j, x1, x2 for the lag-0 entries of subdomain j + 1
// and x3, x4 for those of subdomain j:
//     r_j = b_j + x1 l_j + x2 r_{j+1},   l_j = c_j + x4 r_j + x3 l_{j-1}.
// Then l_j = A_j r_j + s_j with
//     A_j = x4 + x3 w_{j-1} A_{j-1} x2_{j-1},   w_j = 1 / (1 - A_j x1),
//     z_j = (c_j + A_j b_j) + alpha_j z_{j-1},  alpha_j = x3 w_{j-1},  s_j = z_j - A_j b_j,
//     r_j = w_j b_j + w_j x1 s_j + beta_j r_{j+1},   beta_j = w_j x2.
// (Block LU; stable where the block system is diagonally dominant, which the
// set-up checks.)  Both recurrences are prefix sums with fixed multipliers:
// they run by doubling of the distance, two doublings per exchange, until the
// product of the multipliers over the distance is at most 2^-60 everywhere.
// ---------------------------------------------------------------------------

// Set-up, one workgroup per potential, thread j = interface j: record
// [kMarchRows][ni] (A, w, w x1; per round of the prefix sums the multipliers
// over 1, 2, 3 distances, left then right; the lag coefficients 1 .. 7 of
// X^{j+1,1}, X^{j+1,2}, X^{j,3}, X^{j,4}); eta[v]: block dominance, then the
// largest multiplier over 1, 2, 4, .. interfaces.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void causal_march_setup_kernel(int N, int nt, const cd* cols, cd* rec,
                                                                    double* eta) {
    __shared__ cd sh[THREADS];
    __shared__ double se[THREADS / kWave];
    const int v = blockIdx.x, j = threadIdx.x;
    const int ni = N - 1;
    const bool act = j < ni;
    const cd* base = cols + (size_t)v * N * 4 * nt;
    const cd zero = mk(0, 0), one = mk(1, 0);
    cd x1 = zero, x2 = zero, x3 = zero, x4 = zero;
    if (act) {
        x1 = base[((size_t)(j + 1) * 4 + 0) * nt];
        if (j + 1 <= N - 2) x2 = base[((size_t)(j + 1) * 4 + 1) * nt];
        if (j >= 1) x3 = base[((size_t)j * 4 + 2) * nt];
        x4 = base[((size_t)j * 4 + 3) * nt];
    }
    auto block_max = [&](double e) {
        e = wave_max(e);
        if ((j & (kWave - 1)) == 0) se[j / kWave] = e;
        __syncthreads();
        double m = 0;
        for (int w = 0; w < THREADS / kWave; ++w) m = fmax(m, se[w]);
        __syncthreads();
        return m;
    };
    // value of thread j + d (zero outside)
    auto shifted = [&](cd x, int d) {
        sh[j] = x;
        __syncthreads();
        cd r = zero;
        if (j + d >= 0 && j + d < THREADS) r = sh[j + d];
        __syncthreads();
        return r;
    };
    double* ev = eta + (size_t)v * (kGenLevelsMax + 1);
    {
        const double e = act ? norm_inf(inv2(m2(one, -x1, -x4, one))) * (sqrt(abs2(x3)) + sqrt(abs2(x2))) : 0.0;
        // (fmax drops a NaN: it must reach the host)
        const int bad = __syncthreads_or(!(e < 1e300));
        const double m = block_max(e);
        if (j == 0) ev[0] = bad ? nan("") : m;
    }
    // A_j: all j at once, repeated until nothing changes (after m rounds the
    // first m are final; the recurrence contracts by |alpha beta| a round)
    cd A = x4;
    for (int it = 0; it < ni; ++it) {
        const cd w = inv(one - A * x1);
        const cd An = x4 + x3 * shifted((w * A) * x2, -1);
        const bool ch = An.x != A.x || An.y != A.y;
        A = An;
        if (!__syncthreads_or(ch)) break;
    }
    const cd w = inv(one - A * x1);
    cd al = x3 * shifted(w, -1), be = w * x2;
    cd* q = rec + (size_t)v * kMarchRows * ni + j;
    if (act) {
        q[0] = A;
        q[ni] = w;
        q[(size_t)2 * ni] = w * x1;
    }
#pragma unroll 1
    for (int r = 0; r < kMarchRounds; ++r) {
        const int d = 1 << (2 * r);
        const cd al2 = al * shifted(al, -d), al3 = al2 * shifted(al, -2 * d);
        const cd be2 = be * shifted(be, d), be3 = be2 * shifted(be, 2 * d);
        if (act) {
            cd* f = q + (size_t)(3 + 6 * r) * ni;
            f[0] = al; f[ni] = al2; f[(size_t)2 * ni] = al3;
            f[(size_t)3 * ni] = be; f[(size_t)4 * ni] = be2; f[(size_t)5 * ni] = be3;
        }
        const double m1 = block_max(sqrt(fmax(abs2(al), abs2(be))));
        const double m2_ = block_max(sqrt(fmax(abs2(al2), abs2(be2))));
        if (j == 0) { ev[1 + 2 * r] = m1; ev[2 + 2 * r] = m2_; }
        al = al2 * shifted(al2, -2 * d);
        be = be2 * shifted(be2, 2 * d);
    }
    if (act) {
        for (int m = 0; m < kMarchTb - 1; ++m) {
            const int lag = m + 1;
            cd c0 = zero, c1 = zero, c2 = zero, c3 = zero;
            if (lag < nt) {
                c0 = base[((size_t)(j + 1) * 4 + 0) * nt + lag];
                if (j + 1 <= N - 2) c1 = base[((size_t)(j + 1) * 4 + 1) * nt + lag];
                if (j >= 1) c2 = base[((size_t)j * 4 + 2) * nt + lag];
                c3 = base[((size_t)j * 4 + 3) * nt + lag];
            }
            cd* f = q + (size_t)(kMarchLag0 + 4 * m) * ni;
            f[0] = c0; f[ni] = c1; f[(size_t)2 * ni] = c2; f[(size_t)3 * ni] = c3;
        }
    }
}

struct MarchArgs {
    int ni, nt, ns, per_problem;
    int n0, nb;
    int levels;        // doublings of the prefix sums
    int inner, halo;   // interfaces per workgroup and on either side of them
    const cd* rec;     // [nv][kMarchRows][ni]
    const cd* base;    // [B][TB][ns]: d + far part
    cd* g;             // [B][ns][nt]
};

// One block of TB steps.  A workgroup marches a window of THREADS interfaces,
// thread by interface: the `inner` ones it answers for and up to `halo` on
// either side, which it computes as well.  What a step's solution at an
// interface depends on reaches 2^levels - 1 interfaces within the step and one
// more through the lags, so with halo = TB 2^levels the inner values are those
// of the whole system, bit for bit, and no workgroup waits for another.  With
// the whole system in one window there is no halo.
//
// The right-hand sides of the block's steps sit in registers; a solved step
// adds its share to all later ones (coefficients of the lags in registers).  A
// step's exchanges go through LDS, one barrier each: the rounds of the two
// prefix sums (multipliers of the first R in registers, the others in LDS or,
// LDSC = false, read from memory) and the solution.
//
// Bound: the chain of exchanges (about 200 cycles each) and FP64 issue of one
// to two waves per SIMD; the waves run at raised priority beside the sweeps.
// Against block PCR on one workgroup (8 multipliers per interface and level
// read from memory in every step, blocks of 8 steps to 512 interfaces and of 2
// above, coefficients gathered with a stride at every launch), per block:
// 255 interfaces, 16 potentials, 2 doublings 31.3 -> 11.6 us; 127 interfaces, 1
// doubling 14.6 -> 7.2 us; 499 interfaces, 32 problems, 3 doublings 56 -> 21 us;
// 999 interfaces, 5 doublings 26.8 us for 2 steps -> 18.2 us for 4, the solve on
// 1000 subdomains over 500 steps 10.7 -> 4.6 ms.
template <int THREADS, int TB, int R, bool LDSC>
__global__ __launch_bounds__(THREADS) void causal_march_kernel(MarchArgs a) {
    extern __shared__ cd smem[];
    constexpr int ROW = THREADS + 2;                   // entries tid + 1; both ends zero
    cd* zb = smem;                                     // [2][ROW] prefix sums
    cd* xb = smem + 2 * ROW;                           // [2][2][ROW] solution, by step parity
    cd* sc = smem + 6 * ROW;                           // [rounds - R][6][THREADS]
    __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, b = blockIdx.y, ni = a.ni, nb = a.nb;
    const int i_lo = blockIdx.x * a.inner, i_hi = min(ni, i_lo + a.inner);
    const int j = max(i_lo - a.halo, 0) + tid;
    const bool act = j < ni, mine = j >= i_lo && j < i_hi;
    const cd zero = mk(0, 0);
    const cd* rec = a.rec + (size_t)(a.per_problem ? b : 0) * kMarchRows * ni + (act ? j : 0);
    const int rounds = (a.levels + 1) / 2;
    const bool odd = a.levels & 1;                     // the last round doubles once

    auto get = [&](int row) {
        cd x = zero;
        if (act) x = rec[(size_t)row * ni];
        return x;
    };
    cd p[TB], l[TB];                                   // right-hand sides of slots 2j, 2j + 1
    {
        const cd* bb = a.base + (size_t)b * TB * a.ns + 2 * (act ? j : 0);
#pragma unroll
        for (int i = 0; i < TB; ++i) {
            p[i] = l[i] = zero;
            if (act && i < nb) {
                p[i] = bb[(size_t)i * a.ns];
                l[i] = bb[(size_t)i * a.ns + 1];
            }
        }
    }
    const cd A = get(0), W = get(1), O = get(2);
    cd f[R > 0 ? R : 1][6];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            f[r][q] = zero;
            if (r < rounds) f[r][q] = get(3 + 6 * r + q);
        }
    cd c0[TB - 1], c1[TB - 1], c2[TB - 1], c3[TB - 1];
#pragma unroll
    for (int m = 0; m < TB - 1; ++m) {
        c0[m] = get(kMarchLag0 + 4 * m);
        c1[m] = get(kMarchLag0 + 4 * m + 1);
        c2[m] = get(kMarchLag0 + 4 * m + 2);
        c3[m] = get(kMarchLag0 + 4 * m + 3);
    }
    if (LDSC) {
        for (int r = R; r < rounds; ++r)
#pragma unroll
            for (int q = 0; q < 6; ++q) sc[((r - R) * 6 + q) * THREADS + tid] = get(3 + 6 * r + q);
    }
    if (tid < 12) smem[(tid >> 1) * ROW + (tid & 1) * (ROW - 1)] = zero;

    // one prefix sum: dir = -1 from the left (multipliers 0 .. 2), +1 from the
    // right (3 .. 5); s takes the same additions as z
    int par = 0;
    auto scan = [&](cd& z, cd& s, auto right) __attribute__((always_inline)) {
        constexpr bool RIGHT = decltype(right)::value;
        auto one_round = [&](int r, cd m1, cd m2, cd m3) __attribute__((always_inline)) {
            const int d = 1 << (2 * r);
            cd* buf = zb + par * ROW + tid + 1;
            par ^= 1;
            *buf = z;
            __syncthreads();
            auto at = [&](int k) {
                const int o = RIGHT ? min(k * d, THREADS - tid) : max(-k * d, -1 - tid);
                return buf[o];
            };
            cd e = m1 * at(1);
            if (!(odd && r == rounds - 1)) e = madd(madd(e, m2, at(2)), m3, at(3));
            z = z + e;
            s = s + e;
        };
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r < rounds) one_round(r, f[r][RIGHT ? 3 : 0], f[r][RIGHT ? 4 : 1], f[r][RIGHT ? 5 : 2]);
        for (int r = R; r < rounds; ++r) {
            cd m[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int k = q + (RIGHT ? 3 : 0);
                if (LDSC) m[q] = sc[((r - R) * 6 + k) * THREADS + tid];
                else m[q] = get(3 + 6 * r + k);
            }
            one_round(r, m[0], m[1], m[2]);
        }
    };
    cd* gp = a.g + ((size_t)b * a.ns + 2 * (mine ? j : 0)) * a.nt + a.n0;
#pragma unroll
    for (int i = 0; i < TB; ++i) {
        if (i < nb) {
            cd z = madd(l[i], A, p[i]), s = l[i];
            scan(z, s, std::false_type{});
            cd r = madd(W * p[i], O, s), dummy = zero;
            scan(r, dummy, std::true_type{});
            const cd x = madd(s, A, r);
            if (mine) {
                gp[i] = r;
                gp[(size_t)a.nt + i] = x;
            }
            if (i + 1 < TB && i + 1 < nb) {
                cd* rb = xb + (i & 1) * 2 * ROW + tid + 1;
                cd* lb = rb + ROW;
                *rb = r;
                *lb = x;
                __syncthreads();
                const cd rn = rb[1], xp = lb[-1];
#pragma unroll
                for (int m = 0; m < TB - 1 - i; ++m) {
                    p[i + 1 + m] = madd(madd(p[i + 1 + m], c0[m], x), c1[m], rn);
                    l[i + 1 + m] = madd(madd(l[i + 1 + m], c2[m], xp), c3[m], r);
                }
            }
        }
    }
}

// How a system is marched.  Up to 256 interfaces, one workgroup of one wave per
// SIMD takes the whole of it; up to 512, two.  Above, windows of 512 with halos
// of at most 128, i.e. blocks of 8 steps for up to 4 doublings and of 4 for 5
// (the halves that the halos cost are other CUs' time); with more doublings
// the halos would leave nothing, and one workgroup of 1024 threads, with
// registers for two steps, takes the system.  More than 6 doublings' multipliers
// do not fit in LDS beside blocks of 8 steps.
struct MarchPlan { int threads, tb, inner, halo; };
static MarchPlan march_plan(int ni, int levels) {
    if (ni <= 256) return {256, 8, ni, 0};
    if (ni <= 512) return {512, levels <= 6 ? 8 : 4, ni, 0};
    if (levels <= 5) {
        const int tb = levels <= 4 ? 8 : 4, halo = tb << levels;
        return {512, tb, 512 - 2 * halo, halo};
    }
    return {1024, 2, ni, 0};
}
int march_tb(int N, int levels) { return march_plan(N - 1, levels).tb; }

hipError_t launch_causal_march_setup(int N, int nt, int nv, const cd* cols, cd* rec, double* eta,
                                     hipStream_t st) {
    if (N < 2 || N - 1 > kGenMaxIf) return hipErrorInvalidValue;
    if (N - 1 <= 256) causal_march_setup_kernel<256><<<nv, 256, 0, st>>>(N, nt, cols, rec, eta);
    else if (N - 1 <= 512) causal_march_setup_kernel<512><<<nv, 512, 0, st>>>(N, nt, cols, rec, eta);
    else causal_march_setup_kernel<1024><<<nv, 1024, 0, st>>>(N, nt, cols, rec, eta);
    return hipGetLastError();
}

template <int THREADS, int TB, int R, bool LDSC>
static hipError_t launch_march(const MarchArgs& a, int B, hipStream_t st) {
    const int rounds = (a.levels + 1) / 2, more = LDSC ? std::max(0, rounds - R) : 0;
    const size_t lds = sizeof(cd) * (6 * (size_t)(THREADS + 2) + (size_t)more * 6 * THREADS);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    // (the halos may reach past the window's threads only where nothing is left)
    const int wins = (a.ni + a.inner - 1) / a.inner;
    if (wins > 1 && a.inner + 2 * a.halo > THREADS) return hipErrorInvalidValue;
    if (wins == 1 && a.ni > THREADS) return hipErrorInvalidValue;
    causal_march_kernel<THREADS, TB, R, LDSC><<<dim3(wins, B), THREADS, lds, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_causal_gen(int N, int nt, int ns, int B, int per_problem, const cd* cols, const cd* rec,
                             int levels, const cd* d, cd* base, cd* g, int n_lo, int n_hi, const cd* facc,
                             int nseg, int s_from, hipStream_t st) {
    if (N < 2 || N - 1 > kGenMaxIf || ns != 2 * (N - 1) || levels < 0 || levels > kGenLevelsMax)
        return hipErrorInvalidValue;
    const MarchPlan pl = march_plan(N - 1, levels);
    const int tb = pl.tb;
    if (n_lo % tb != 0 || n_lo < 0 || n_hi > nt || s_from < 0 || s_from > n_lo)
        return hipErrorInvalidValue;
    for (int n0 = n_lo; n0 < n_hi; n0 += tb) {
        const int nb = min(tb, n_hi - n0);
        auto far = tb == 8 ? launch_causal_far<8> : tb == 4 ? launch_causal_far<4> : launch_causal_far<2>;
        hipError_t e = far(N, nt, ns, B, per_problem, n0, nb, cols, d, g, base, facc, nseg, s_from, st);
        if (e != hipSuccess) return e;
        MarchArgs m{N - 1, nt, ns, per_problem, n0, nb, levels, pl.inner, pl.halo, rec, base, g};
        if (pl.threads == 256) e = launch_march<256, 8, 1, true>(m, B, st);
        else if (pl.threads == 512 && tb == 8) e = launch_march<512, 8, 1, true>(m, B, st);
        else if (pl.threads == 512) e = launch_march<512, 4, 3, true>(m, B, st);
        else e = launch_march<1024, 2, 1, false>(m, B, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace swr
