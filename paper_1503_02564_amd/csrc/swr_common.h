// swr_common.h -- types and wave-level helpers shared by the SWR kernels.
//
// All arithmetic is FP64 complex, interleaved (re, im) -- the layout of
// std::complex<double> / torch.complex128.  One wavefront is 64 lanes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swr {

constexpr int kWave = 64;

struct __align__(16) cd {
    double x, y;
};

__host__ __device__ inline cd mk(double x, double y) { cd r; r.x = x; r.y = y; return r; }
__host__ __device__ inline cd operator+(cd a, cd b) { return mk(a.x + b.x, a.y + b.y); }
__host__ __device__ inline cd operator-(cd a, cd b) { return mk(a.x - b.x, a.y - b.y); }
__host__ __device__ inline cd operator-(cd a) { return mk(-a.x, -a.y); }
__host__ __device__ inline cd operator*(cd a, cd b) { return mk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__host__ __device__ inline cd operator*(double s, cd a) { return mk(s * a.x, s * a.y); }
__host__ __device__ inline cd conjc(cd a) { return mk(a.x, -a.y); }
__host__ __device__ inline double abs2(cd a) { return a.x * a.x + a.y * a.y; }
// 1/z as conj(z)/|z|^2 (reciprocal-multiply; only used outside the time loop)
__host__ __device__ inline cd inv(cd a) { double s = 1.0 / abs2(a); return mk(a.x * s, -a.y * s); }
// i*a
__host__ __device__ inline cd mul_i(cd a) { return mk(-a.y, a.x); }
// a - b*c (one complex multiply-subtract)
__host__ __device__ inline cd msub(cd a, cd b, cd c) {
    return mk(a.x - b.x * c.x + b.y * c.y, a.y - b.x * c.y - b.y * c.x);
}
// a + b*c
__host__ __device__ inline cd madd(cd a, cd b, cd c) {
    return mk(a.x + b.x * c.x - b.y * c.y, a.y + b.x * c.y + b.y * c.x);
}

__device__ inline int lane_id() { return __lane_id(); }

__device__ inline double rdlane(double v, int l) {
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __builtin_amdgcn_readlane(t.x, l);
    t.y = __builtin_amdgcn_readlane(t.y, l);
    return *reinterpret_cast<double*>(&t);
}
__device__ inline cd rdlane(cd v, int l) { return mk(rdlane(v.x, l), rdlane(v.y, l)); }

// whole-wave shift of one double by one lane through DPP (CTRL 0x138: lane
// i reads lane i - 1; 0x130: lane i reads lane i + 1); the lane without a
// source reads 0 (bound_ctrl: no old value to materialise)
template <int CTRL>
__device__ inline double dpp_shift(double v) {
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __builtin_amdgcn_mov_dpp(t.x, CTRL, 0xf, 0xf, true);
    t.y = __builtin_amdgcn_mov_dpp(t.y, CTRL, 0xf, 0xf, true);
    return *reinterpret_cast<double*>(&t);
}

// Row moves of one double through the gfx950 lane swaps (rows = 16 lanes).
// With both operands equal to x, v_permlane16_swap returns
//   first  = (x.row0, x.row0, x.row2, x.row2)   second = (x.row1, x.row1, x.row3, x.row3)
// and v_permlane32_swap returns
//   first  = (x.row0, x.row1, x.row0, x.row1)   second = (x.row2, x.row3, x.row2, x.row3).
struct RowPair { double first, second; };
__device__ inline RowPair swap16(double v) {
    int2 t = *reinterpret_cast<int2*>(&v);
    const auto lo = __builtin_amdgcn_permlane16_swap(t.x, t.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(t.y, t.y, false, false);
    int2 f = make_int2(lo[0], hi[0]), s = make_int2(lo[1], hi[1]);
    return RowPair{*reinterpret_cast<double*>(&f), *reinterpret_cast<double*>(&s)};
}
__device__ inline RowPair swap32(double v) {
    int2 t = *reinterpret_cast<int2*>(&v);
    const auto lo = __builtin_amdgcn_permlane32_swap(t.x, t.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(t.y, t.y, false, false);
    int2 f = make_int2(lo[0], hi[0]), s = make_int2(lo[1], hi[1]);
    return RowPair{*reinterpret_cast<double*>(&f), *reinterpret_cast<double*>(&s)};
}
// value of lane - 16 (rows 1..3) and of lane + 16 (rows 0..2)
__device__ inline double up16(double v) {
    const RowPair a = swap16(v);
    const double r2 = swap32(a.second).first;          // row 2 <- row 1
    const int row = lane_id() >> 4;
    return row == 2 ? r2 : a.first;                    // rows 1, 3 <- rows 0, 2
}
__device__ inline double dn16(double v) {
    const RowPair a = swap16(v);
    const double r1 = swap32(a.first).second;          // row 1 <- row 2
    const int row = lane_id() >> 4;
    return row == 1 ? r1 : a.second;                   // rows 0, 2 <- rows 1, 3
}

// value of lane (lane - d); lanes below d receive `fill`.  Distance 1 is a
// DPP wave shift, distances 16 and 32 are lane swaps (no LDS round trip),
// other distances a permute.  All run on every lane of the wave.
__device__ inline cd shfl_up_c(cd v, int d, cd fill) {
    if (d == 1) {
        const cd r = mk(dpp_shift<0x138>(v.x), dpp_shift<0x138>(v.y));
        return lane_id() == 0 ? fill : r;
    }
    if (d == 32) {
        const cd r = mk(swap32(v.x).first, swap32(v.y).first);
        return lane_id() < 32 ? fill : r;
    }
    if (d == 16) {
        const cd r = mk(up16(v.x), up16(v.y));
        return lane_id() < 16 ? fill : r;
    }
    int src = lane_id() - d;
    cd r = mk(__shfl(v.x, src < 0 ? 0 : src), __shfl(v.y, src < 0 ? 0 : src));
    return src < 0 ? fill : r;
}
// value of lane (lane + d); lanes with lane + d >= 64 receive `fill`
__device__ inline cd shfl_dn_c(cd v, int d, cd fill) {
    if (d == 1) {
        const cd r = mk(dpp_shift<0x130>(v.x), dpp_shift<0x130>(v.y));
        return lane_id() == kWave - 1 ? fill : r;
    }
    if (d == 32) {
        const cd r = mk(swap32(v.x).second, swap32(v.y).second);
        return lane_id() >= 32 ? fill : r;
    }
    if (d == 16) {
        const cd r = mk(dn16(v.x), dn16(v.y));
        return lane_id() >= kWave - 16 ? fill : r;
    }
    int src = lane_id() + d;
    cd r = mk(__shfl(v.x, src > 63 ? 63 : src), __shfl(v.y, src > 63 ? 63 : src));
    return src > 63 ? fill : r;
}

// Value of lane - 1 / lane + 1 with zero where there is none: the DPP shift
// already reads zero there, so no select is needed
__device__ inline cd shfl_up1z(cd v) { return mk(dpp_shift<0x138>(v.x), dpp_shift<0x138>(v.y)); }
__device__ inline cd shfl_dn1z(cd v) { return mk(dpp_shift<0x130>(v.x), dpp_shift<0x130>(v.y)); }

// The same moves without the fill: lanes with no source get some other
// lane's (finite) value.  For reductions whose multiplier is exactly zero on
// those lanes (the PCR levels), the product is zero and the select is saved.
__device__ inline cd shfl_up_raw(cd v, int d) {
    if (d == 1) return mk(dpp_shift<0x138>(v.x), dpp_shift<0x138>(v.y));
    if (d == 32) return mk(swap32(v.x).first, swap32(v.y).first);
    if (d == 16) return mk(up16(v.x), up16(v.y));
    const int src = (lane_id() - d) & (kWave - 1);
    return mk(__shfl(v.x, src), __shfl(v.y, src));
}
__device__ inline cd shfl_dn_raw(cd v, int d) {
    if (d == 1) return mk(dpp_shift<0x130>(v.x), dpp_shift<0x130>(v.y));
    if (d == 32) return mk(swap32(v.x).second, swap32(v.y).second);
    if (d == 16) return mk(dn16(v.x), dn16(v.y));
    const int src = (lane_id() + d) & (kWave - 1);
    return mk(__shfl(v.x, src), __shfl(v.y, src));
}

// Sum and maximum over the wave, on every lane: rotations inside rows of 16
// lanes, then the lane swaps between rows -- no LDS round trips (as
// butterflies of __shfl_xor the six steps took about 1000 cycles of latency).
// Every lane of the result has the same bits.
__device__ inline double wave_max(double v) {
    v = fmax(v, dpp_shift<0x128>(v));             // row_ror:8
    v = fmax(v, dpp_shift<0x124>(v));
    v = fmax(v, dpp_shift<0x122>(v));
    v = fmax(v, dpp_shift<0x121>(v));
    const RowPair r = swap16(v);
    v = fmax(r.first, r.second);
    const RowPair h = swap32(v);
    return fmax(h.first, h.second);
}
__device__ inline double wave_sum(double v) {
    v += dpp_shift<0x128>(v);
    v += dpp_shift<0x124>(v);
    v += dpp_shift<0x122>(v);
    v += dpp_shift<0x121>(v);
    const RowPair r = swap16(v);
    v = r.first + r.second;
    const RowPair h = swap32(v);
    return h.first + h.second;
}

// ---------------------------------------------------------------------------
// Problem-wide constants handed to every kernel.
// ---------------------------------------------------------------------------
// kernel forms of the transmission operator: Robin, S0^2, the general
// convolution form that carries S0^3, S0^4, S1^2 and S1^4 (EndCoef), and the
// Pade strategy's auxiliary-function form (S2^{2,m}, S2^{4,m})
enum Trans { TR_ROBIN = 0, TR_S02 = 1, TR_GEN = 2, TR_PADE = 3 };
// Pade strategy: at most two auxiliary functions of each end per lane
constexpr int kPadeMax = 2 * 64;

// Coefficients of the higher-order transmission operators at one interface
// end for a time-independent potential (Sec. 2.2).  With x_s = e^{-i calW_s}
// v_s the stored boundary history (calW_s = (s - 1/2) omega, calW_0 = 0;
// omega = W dt for the gauge strategy, 0 for the potential strategy):
//   Sbar v_n = sig v_n + e^{i calW_n} [ cp E_n + cm O_n + a G_n ]
//   E_n / O_n = sum over s < n with n-s even / odd of beta_{n-s} x_s
//   G_n = 2 sum_{s<n} x_s
// where cp = c2 + d, cm = c2 - d, d = -e^{i pi/4} sqrt(dt/2) W/2 (S0^3, S0^4;
// alpha_k = +-beta_k splits the alpha sum by parity), a = -i (dn W/4)(dt/2)
// (S0^4, S1^4), sig = c2 + d + a.  The part that crosses the interface drops
// the a terms: sig_s = c2 + d.
// Pade strategy (c = 2i/dt, W and dn W at the end node):
//   sig_s = -i sum_{s=0}^m a_s + i sum_{s=1}^m a_s d_s / (c + W + d_s),
//   sig = sig_s + (dn W/4) / (c + W) at order 4 (else sig_s),
//   cp = 1/(c + W), omega = W, pad = dn W.
struct EndCoef {
    cd sig, sig_s, cp, cm, a;
    double omega, pad;
};
enum VKind { VK_STATIC = 0, VK_TIME = 1, VK_CUBIC = 2 };

// Task flags: one sweep of one subdomain of one problem.
enum TaskFlags {
    T_DATA_U0   = 1 << 0,   // initial data from u0 (else zero data, zero v_0 history)
    T_FLUX_G    = 1 << 1,   // incoming fluxes l_k, r_k from g_in slots
    T_IMP_L     = 1 << 2,   // l_{k,1} = 1, everything else 0
    T_IMP_R     = 1 << 3,   // r_{k,1} = 1
    T_OUT_G     = 1 << 4,   // outgoing fluxes -> g_out slots
    T_OUT_COLS  = 1 << 5,   // outgoing fluxes -> first-column store
    T_OUT_UT    = 1 << 6,   // u(T) -> uT (interior nodes) + ends
    T_OUT_TRACE = 1 << 7,   // u_n at the two end nodes -> trace store
    T_MAXDIFF   = 1 << 8,   // fold max |g_out - g_in| over written slots
    T_CKPT      = 1 << 9,   // store u at steps nt - 64 j (and u_0) for the adjoint
    T_OUT_SNAP  = 1 << 10,  // u at steps 0, s, 2s, ... -> snapshot store
};

struct Task {
    int k;      // subdomain
    int b;      // problem (batch member)
    int f;      // factor set (potential index)
    int flags;
};

// Layout of the per-lane factor record of one subdomain (see factor kernel).
// For a chunk of up to P nodes per lane: P-1 interior nodes with
// {inv, ainv, cp, alpha, gamma}, then {a_sep, c_sep}, then PCR {k1[6], k2[6]},
// then 1/B of the decoupled reduced equation.
constexpr int kPcrLevels = 6;
__host__ __device__ constexpr int fac_fields(int P) { return 5 * (P - 1) + 2 + 2 * kPcrLevels + 1; }
constexpr int kMaxP = 8;
// subdomains of more than 64 * kMaxP nodes run the long-chunk sweep
// (swr_sweep_long.hip) with up to this many nodes per lane
constexpr int kLongMaxQ = 8192;
// default schedule: the S0^2 helper wave up to this many tasks per launch (every
// wave then has a SIMD of its own); the static causal solve pipelined in
// chunks of this many steps (32 problems on 500 uneven subdomains, 2000 steps:
// 66.5 ms per solve, staged 79.5; chunks of 128 steps 81.4, 192 79.7, 320 76.0,
// 384 73.4, 512 69.4, 1024 73.0: chunks that straddle the 256-step super-blocks
// split their launches, longer ones overlap less)
constexpr int kHelpMaxTasks = 512;
constexpr int kPipeChunk = 256;
// V(t,x) with Robin or S0^2: up to this many (problem, subdomain) tasks the
// sweeps read each step's factor record from memory (swr_sweep_rows_time.hip),
// above they refactor in every step.  A workgroup of the former fills a compute
// unit, so from 256 tasks on it runs in two rounds, and the latter's chain is the
// same up to 1024.  One sweep of 256 steps with all records built for it, against
// refactoring: 128 x 256 cells 0.57 / 1.09 ms, 256 x 256 0.99 / 1.10, 320 x 256
// 1.37 / 1.13, 256 x 500 1.42 / 1.40 (a solve builds them once for 10 to 40 sweeps).
constexpr int kTimeRecordTasks = 240;
// ... and the memory of the records (at most a quarter of what is free, given
// back when another buffer of the context needs it); longer windows are factored
// piece by piece, anew for every sweep.  128 x 256 cells over 4000 steps, 17 GB
// of records, a solve of 16 iterations: 326 ms in pieces, 483 refactoring, 239 with
// all of them held (a bound that a context shares the card under, not the fastest).
constexpr size_t kTimeRecordBytes = (size_t)4 << 30;
// sweeps of V(t,x) and |u|^2 in the row form sum their S0^2 history in one
// piece up to this many steps: 64 cycles of matrix instructions per 4 past
// steps and block of 64 outputs, which passes the cost of the split (a product
// and a launch per 256 steps, about 30 us) near 1000 past steps
constexpr int kUnsplitSteps = 2048;
// static sweeps with the higher-order or Pade operators: all chunk widths of a
// list of at most this many tasks run in one launch, one wave per SIMD (24 uneven
// subdomains of three widths, 1000 steps: 5.3 -> 2.2 ms a solve); longer
// lists take a launch per width, whose narrow widths run more waves per SIMD
constexpr int kAnyMaxTasks = 1024;
// schedule parameters of launch forms that no longer exist; still validated,
// saved and reported (bounds and defaults)
constexpr int kPairFrom = kMaxP + 1;
constexpr int kGroupMax = 8;
constexpr int kGroupDefault = 4;

// Row form of the static sweep (swr_rows.h): the kernels, by rows per task,
// whether interior coefficients are read from LDS, waves per workgroup, and
// the widest instantiation
struct RowsKind { int RW; bool lds; int waves, pmax; };
constexpr int kRowsKinds = 5;
constexpr RowsKind kRowsKind[kRowsKinds] = {{4, false, 1, 8}, {1, false, 1, 8}, {1, true, 2, 14},
                                              {2, false, 1, 8}, {2, true, 2, 16}};
constexpr int kRowLevels = 4;      // cyclic reduction levels inside a row of 16 lanes
constexpr int kRowsMaxP = 16;      // nodes per lane of the widest instantiation (RW 1 and 2)

__host__ __device__ constexpr int rows_borders(int RW) { return 2 * (RW - 1); }
// fields of the record after the 4 (P - 1) interior ones: a_sep, c_sep, the
// reduction's multipliers, 1 / B, the border weights
__host__ __device__ constexpr int rows_tail(int RW) { return 2 + 2 * kRowLevels + 1 + rows_borders(RW); }
__host__ __device__ constexpr int rows_fields(int P, int RW) { return 4 * (P - 1) + rows_tail(RW); }
// wide form: complex entries of a record
constexpr int kWideMaxP = 12;
__host__ __device__ constexpr size_t wide_record(int P, int NW) {
    return (size_t)(4 * (P - 1) + rows_tail(4) + 4) * 64 * NW;
}
constexpr int kRowsRegs = 138;       // registers for u, y and the record when it is partly in LDS
constexpr int kRowsLdsP = 9;         // widths from this on keep them in LDS
// Tasks of a context (build sweeps and final sweep together, which overlap)
// from which fewer rows per task pay.  Measured on solves of 32 to 256 subdomains
// over 512 steps, S0^2 (ms per solve, fewer rows against four):
//   up to 128 nodes, one row:   101 nodes, 2016 tasks 1.65 / 1.60, 4032 1.90 / 2.25, 4158 2.34 / 2.62
//   up to 256 nodes, two rows:  201 nodes, 2110 tasks 2.25 / 2.09, 4158 2.56 / 2.87, 8254 3.28 / 4.54
//   above, two rows from LDS:   351 nodes, 2110 tasks 2.69 / 2.17, 4158 3.10 / 3.07, 8254 3.95 / 4.96
//   up to 224 nodes, one row from LDS against two in registers: 201 nodes,
//   8254 tasks 3.67 / 3.43, 16510 6.53 / 6.81, 33022 11.0 / 11.6 (251 nodes:
//   16.5 / 14.9, so not there: 16 slots per lane spill)
// The lines are drawn for solves.  A list that runs alone (swr_apply_R, the
// classical iteration) has about half of those tasks; just above the lines, and
// with one potential per problem on uneven widths well above them, it loses what
// the solve gains (S0^2, sweep of 500 and solve of 400 steps, fewer rows / four):
//   one row:  101 nodes, 860 tasks of 3438 0.43 / 0.31 and 1.93 / 2.27 ms; 41 to 121
//             nodes, 1200 of 2998 0.49 / 0.53 and 1.94 / 2.20; 65 nodes, 2000 of 7998 0.40 / 0.58
//   two rows: 131 to 251 nodes, 1030 of 4118 0.53 / 0.59; 301 nodes from LDS, 2560 of
//             5246 0.88 / 0.98 and 2.34 / 2.71; 301 to 501 nodes, 2400 of 4998 1.15 / 1.07
//   both, 41 to 241 nodes, a potential per problem (sweep of 400 steps): 1600 of 6384
//             0.98 / 0.59 and 2.58 / 3.28; 3000 of 11940 1.04 / 0.89 and 3.41 / 4.78
// LDS forms want records shared by four tasks or more (one potential, batch >= 4).
constexpr size_t kRowsFill1 = 2560;
constexpr size_t kRowsFill1Lds = 12288;
constexpr size_t kRowsFill2 = 3072;
constexpr size_t kRowsFill2Lds = 4608;

// S0^2: the time window is cut into super-chunks of this many steps for the
// far history (the part of a block's far sum older than its super-chunk is
// one batched Toeplitz product on the matrix cores per super-chunk; a
// multiple of 256).  256 steps bound the terms that a sweep's block sums itself
// by 320, the length of its beta window in LDS; 512 steps were no faster (146.6
// against 146.1 ms, with the 64-lane sweeps that summed them lane by lane)
constexpr int kFarSuper = 256;

struct SweepArgs {
    int N, nt, B, nx, ns;        // ns = 2N-2 interface slots
    int ntasks;
    int P;                       // nodes-per-lane bound the factors were built for
    double kappa;                // h / (3 dt):  c M = i kappa * tridiag(1,4,1)
    cd sigma;                    // implicit transmission coefficient
    cd c2;                       // S0^2 history prefactor e^{-i pi/4} sqrt(2/dt)
    const int* J;                // [N] cells per subdomain
    const int* off;              // [N] first global node
    const Task* tasks;
    const cd* fac;               // [nf][fac_fields(P)][64]
    const double* beta;          // [nt + 65]
    const cd* u0;                // [B][nx]
    const cd* g_in;              // [B][ns][nt]
    cd* g_out;                   // [B][ns][nt]
    cd* cols;                    // [nf/N ... ] first columns [nv][N][4][nt]
    cd* hist;                    // [ntasks][2][nt+1] boundary v_n history
    cd* uT;                      // [B][nx]
    cd* ends;                    // [B][N][2] u(T) at the two end nodes
    cd* trace;                   // [B][N][2][nt+1] u_n at the two end nodes
    unsigned long long* maxdiff; // max |g_out - g_in| as ordered bits
    double h;                    // mesh size
    const double* Vt;            // [nt+1][nx] time-dependent potential
    int nl_maxit;                // |u|^2 inner fixed point: cap and tolerance
    double nl_tol;
    int* nl_stats;               // [0] largest inner count, [1] nonconvergence flag
    int flags_and, flags_or;     // per-launch override of the task flags
    cd* ckpt;                    // [ntasks][Jc+1][P][64] checkpoints of u
    int Jc;                      // ceil(nt / 64)
    cd* bsum;                    // [ntasks][2][nt] with the checkpoints: running sums (history less
                                 // flux) of every step's two boundary terms, for the replay
    int task0;                   // this launch runs tasks task0 .. task0 + ntasks - 1
    int n_begin, n_end;          // steps n_begin+1 .. n_end of this launch (n_begin % 64 == 0)
    cd* state;                   // [ntasks][2][P][64] u_n and v_n carried between launches
    const EndCoef* endc;         // TR_GEN: [nf][2] end coefficients (left, right)
    int help_max;                // S0^2: launches of at most this many tasks use the helper wave
    int pstride;                 // chunk-width stride of the per-task state and checkpoint
                                 // records (the context's largest width; a launch's own P may
                                 // be smaller: subdomains are grouped by width)
    size_t fstride;              // complex entries per subdomain factor record
    cd* snaps;                   // [B][nsnap][nx] u at steps 0, snap_stride, ... (interior nodes)
    cd* snap_ends;               // [B][nsnap][N][2] the same at the two end nodes
    int snap_stride, nsnap;
    int tr;                      // swr_transmission code (time-dependent end coefficients)
    // Pade strategy
    double dt;
    const cd* pade;              // [2][m+1]: a_0..a_m, then d_0..d_m (d_0 unused)
    int pade_m, pade_order;      // auxiliary functions per end; 2 or 4
    cd* pstate;                  // [ntasks][6][64] auxiliary functions carried between launches
                                 // (phi of the left end: slots 0, 1; right end: 2, 3; psi: 4, 5)
    // long-chunk sweep (subdomains of more than 64 * kMaxP nodes)
    int lq;                      // nodes per lane of this launch
    cd* lfac;                    // [nf][fac_fields(lq max)][64] factor records (static, |u|^2)
    size_t lfstride;             // complex entries per long factor record
    cd* lwork;                   // [ntasks][3 Q (+ fac_fields(Q) for V(t,x))][64] per-task arrays
    // S0^2 split at super-chunks: [list tasks][2][kFarSuper] the old part of
    // the far sums of the launch's super-chunk (null: the far sums run from
    // q = 0; the launch then need not end at a super-chunk boundary)
    const cd* far_old;
    // row form of the static sweep: one entry per workgroup, (first task, tasks, nodes per lane, -)
    const int4* items;
    const cd* rfac;              // row-form and wide-form records and their strides
    size_t rstride;
    const cd* tfac;              // V(t,x): row-form records [step - tfac_begin][N][rstride]
    int tfac_begin;
    const cd* wfac;
    size_t wstride;
};

// far_old_kernel: for the super-chunk starting at step C (> 0), every task
// t < ntasks of a list, both ends e and outputs j < kFarSuper (step C+1+j <=
// nt): out[t][e][j] = sum_{q <= C-65} beta_{C+1+j-q} x_q, x the task's
// boundary history hist[t][e][.] ([ntasks][2][nt+1]).
struct FarOldArgs {
    const cd* hist;
    const double* beta;          // [nt + 65]
    cd* out;
    int ntasks, nt, C;
};

struct FactorArgs {
    int N, nx, nf, P;
    double h, dt;
    cd sigma;                    // Robin / S0^2: implicit coefficient at both ends
    int tr;                      // swr_transmission code; 2..7 fill endc
    cd c2;                       // e^{-i pi/4} sqrt(2/dt)
    EndCoef* endc;               // [nf][2] output for the higher-order operators
    const int* Pk;               // [N] chunk width of each subdomain (this launch builds width P)
    size_t fstride;              // complex entries per subdomain factor record
    const int* J;
    const int* off;
    const double* V;             // [nv][nx] static potential (nullptr = 0)
    bool steps;                  // row form: V is rows of V(t,x), record v from their mean over step v
    cd* fac;
    const cd* pade;              // Pade strategy: [2][m+1] coefficients a, d
    int pade_m;
};

struct LttArgs {
    int N, nt, ns, B;
    int per_problem;       // cols indexed by problem (1) or shared (0)
    const cd* cols;        // [nv][N][4][nt]
    const cd* x;           // [B][ns][nt]
    cd* y;                 // output, see y_ld / n_lo
    const cd* base;        // y = base + sign * L x  (base may be x itself or null)
    double sign;
    int n_lo, n_hi;        // output time window
    int s_lo, s_hi;        // only inputs s_lo <= s < s_hi contribute (and s <= n)
    int y_ld;              // leading dimension of y / base per (b, slot)
    int s_seg;             // > 0: split the inputs into segments of s_seg steps, segment z
                           // writing its own partial at y + z * y_seg_stride (base ignored)
    size_t y_seg_stride;
};

// In-block forward substitution of the causal interface solve.
struct CausalArgs {
    int N, nt, ns, B, per_problem;
    int n0, nb;
    const cd* cols;
    const cd* Minv;    // [nv][ns][ns]  (I - C_0)^{-1}
    const cd* d;       // [B][ns][nt]
    const cd* far;     // [B][ns][kCausalTb]
    cd* g;             // [B][ns][nt]
};
constexpr int kCausalTb = 64;
constexpr int kRedBlocks = 240;   // partial-sum blocks per problem
constexpr int kRedThreads = 256;

// launchers (swr_sweep.hip)
hipError_t launch_factor(const FactorArgs& a, hipStream_t st);
hipError_t launch_sweep(const SweepArgs& a, int trans, int vk, hipStream_t st, bool plain = false);
hipError_t launch_sweep_static(const SweepArgs& a, int trans, hipStream_t st);
hipError_t launch_sweep_static_pade(const SweepArgs& a, hipStream_t st);
// subdomains of more than 64 * kMaxP nodes (swr_sweep_long.hip): a.lq nodes per lane
hipError_t launch_sweep_long(const SweepArgs& a, int trans, int vk, hipStream_t st);
hipError_t launch_factor_long(const FactorArgs& a, int Q, hipStream_t st);
hipError_t launch_sweep_time(const SweepArgs& a, int trans, hipStream_t st);
hipError_t launch_sweep_any(const SweepArgs& a, int trans, hipStream_t st);
hipError_t launch_sweep_cubic_hi(const SweepArgs& a, int trans, hipStream_t st);
// static potential, Robin or S0^2 (swr_sweep_rows*.hip): the workgroups a.items[0 .. nitems - 1] of
// one kind, records a.fac with stride a.fstride; pmax: their widest
hipError_t launch_sweep_rows(const SweepArgs& a, int kind, int trans, int vk, int nitems, int pmax,
                             hipStream_t st);
// row-form records of the subdomains with RW rows (a.Pk: P + 32 RW per subdomain)
hipError_t launch_rows_factor(const FactorArgs& a, int RW, int pmax, hipStream_t st);
// static potential, Robin or S0^2, subdomains of more than 64 * kMaxP nodes
// (swr_sweep_wide.hip): NW waves per task, P nodes per lane; records a.fac with
// stride a.fstride (a.Pk of the factorisation: P + 32 NW per subdomain)
hipError_t launch_sweep_wide(const SweepArgs& a, int trans, int NW, int P, hipStream_t st);
hipError_t launch_wide_factor(const FactorArgs& a, int NW, hipStream_t st);
// the old part of the S0^2 far sums of one super-chunk (swr_sweep.hip)
hipError_t launch_far_old(const FarOldArgs& a, hipStream_t st);
hipError_t launch_finalize_ut(int N, int nx, int B, const int* off, const cd* ends, cd* uT,
                              hipStream_t st);
// the same for every snapshot: ends [B][S][N][2] -> snaps [B][S][nx]
hipError_t launch_finalize_snaps(int N, int nx, int B, int S, const int* off, const cd* ends,
                                 cd* snaps, hipStream_t st);
hipError_t launch_beta(int n, double* beta, hipStream_t st);
// launchers (swr_iface.hip)
// Batches of at least eight problems with one potential: from this many
// (problem, subdomain) pairs on, the interface products take eight problems as the
// columns of a matrix instruction (no zero operands, eight times fewer waves);
// below, the one-problem forms, which fill the GPU.  768 steps, 100 cells each,
// one-problem / batched: 32 subdomains x 8 problems 1.90 / 2.61 ms, 64 x 32 3.16 /
// 3.78, 300 x 8 4.78 / 4.98, 100 x 32 4.57 / 4.53, 300 x 16 6.81 / 6.27 ms.
constexpr size_t kBatchFrom = 3072;
inline bool batch_form(int N, int B, bool per_problem) {
    return B >= 8 && !per_problem && (size_t)N * B >= kBatchFrom;
}
hipError_t launch_ltt(const LttArgs& a, hipStream_t st);
int ltt_seg_blocks(int N, int B, bool per_problem, int nblk);
// BiCGStab's scalars of one problem, and the stages of an iteration (bicg_kernel)
struct BicgState {
    cd rho, rho_new, alpha, omega;
    double bn, rel;              // |rhs|; relative residual of the last iteration
    int act, half, bad;          // still iterating; |s| already small; a norm was not finite
};
enum { kBicgInit, kBicgBeta, kBicgAlpha, kBicgHalf, kBicgOmega, kBicgEnd };
hipError_t launch_bicg(int stage, const cd* u, const cd* w, long M, int B, double* partial, BicgState* st,
                       cd* coef, double tol, hipStream_t stream);
hipError_t launch_lincomb(const cd* x0, const cd* x1, const cd* x2, const cd* coef, cd* z, long M,
                          int B, hipStream_t st);
hipError_t launch_multidot(const cd* basis, int nv, const cd* w, long M, int B, double* partial,
                           cd* out, int out_ld, int accumulate, hipStream_t st);
hipError_t launch_multiaxpy(const cd* basis, int nv, const cd* coef, int coef_ld, double sign,
                            cd* w, long M, int B, hipStream_t st);
hipError_t launch_norm(const cd* w, long M, int B, double* partial, double* nrm, hipStream_t st);
hipError_t launch_scale(const cd* src, const double* den, cd* dst, long M, int B, const int* active,
                        hipStream_t st);
hipError_t launch_givens(int j, int m, int B, const cd* hproj, const double* hnext, cd* H, cd* cs,
                         cd* sn, cd* e, const double* bnorm, double* resid, int* active,
                         hipStream_t st);
hipError_t launch_gmres_solve(int jj, int m, int B, const cd* H, const cd* e, cd* y,
                              const int* active, hipStream_t st);
hipError_t launch_gmres_init(int m, int B, const double* beta, cd* e, int* active,
                             const double* bnorm, double tol, double* resid, hipStream_t st);
hipError_t launch_c0_inverse(int N, int ns, int nt, int nv, const cd* cols, cd* work, cd* Minv,
                             int* piv_ok, hipStream_t st);
hipError_t launch_causal_block(const CausalArgs& a, hipStream_t st);
// launchers (swr_causal.hip): block-PCR causal solve for N - 1 <= 64
// interfaces and ns <= kNearSlots slots
constexpr int kNearTb = 32;
constexpr int kNearSlots = 128;
// PCR record per lane: multipliers of every level, then the inverse of the
// reduced diagonal block after 0 .. kPcrLevels levels
constexpr int kPcrRec = kPcrLevels * 8 + (kPcrLevels + 1) * 4;
// remaining coupling below which further PCR levels cannot change an FP64
// result: ||D_l^{-1}|| (||L_l|| + ||U_l||) <= 2^-60 (unit roundoff is 2^-53)
constexpr double kPcrNegligible = 8.673617379884035e-19;
// eta: [nv][levels + 1] coupling measure of the system before each level
// per-potential record size (complex values) of the one-wave causal form:
// PCR multipliers plus the near kernel's packed lag coefficients
size_t causal_fast_rec();
hipError_t launch_causal_pcr_setup(int N, int nt, int nv, const cd* cols, cd* pcr, double* eta,
                                   hipStream_t st);
hipError_t launch_causal_fast(int N, int nt, int ns, int B, int per_problem, const cd* cols,
                              const cd* pcr, int levels, const cd* d, cd* base, cd* g, int n_lo,
                              int n_hi, const cd* facc, int nseg, int s_from, hipStream_t st);
// general causal solve for up to kGenMaxIf interfaces (causal_march_kernel)
constexpr int kCausalSuper = 256;    // causal solve super-block (time steps)
constexpr int kGenMaxIf = 1024;
constexpr int kGenLevelsMax = 10;    // doublings that reach kGenMaxIf interfaces
constexpr int kMarchTb = 8;          // longest near block
constexpr int kMarchRounds = kGenLevelsMax / 2;
// record per interface: A, w, w x1; multipliers of the rounds; lag coefficients
constexpr int kMarchLag0 = 3 + 6 * kMarchRounds;
constexpr int kMarchRows = kMarchLag0 + 4 * (kMarchTb - 1);
int march_tb(int N, int levels);     // steps per near block
// eta: [nv][kGenLevelsMax + 1] block dominance, then the largest multiplier
// over 2^l interfaces, l = 0 ..
hipError_t launch_causal_march_setup(int N, int nt, int nv, const cd* cols, cd* rec, double* eta,
                                     hipStream_t st);
hipError_t launch_causal_gen(int N, int nt, int ns, int B, int per_problem, const cd* cols,
                             const cd* pcr, int levels, const cd* d, cd* base, cd* g, int n_lo,
                             int n_hi, const cd* facc, int nseg, int s_from, hipStream_t st);
struct AdjArgs {
    int N, nt, B, nx, ns, Jc;
    int pstride;                 // record stride of checkpoints, segments and state, as SweepArgs
    size_t fstride;
    double kappa, h;
    cd sigma, c2;
    const int* J;
    const int* off;
    const Task* tasks;
    const int4* items;           // workgroups, as SweepArgs
    const cd* fac;               // row-form records
    const double* beta;
    const cd* gbar;          // [B][nx]
    const cd* g_in;          // adjoint fluxes [B][ns][nt] (null: zero)
    cd* g_out;               // outgoing adjoint fluxes
    cd* hist;                // adjoint boundary history [ntasks][2][nt+1]
    const cd* far_old;       // as SweepArgs
    cd* state;               // [ntasks][2][P][64] w and the gradient sums carried between launches
    int m_begin, m_end;      // adjoint steps of this launch (m_begin % 64 == 0)
    int grad;                // replay the forward and accumulate dJ/dV
    const cd* ckpt;          // [ntasks][Jc+1][P][64]
    const cd* bsum;          // [ntasks][2][nt] the forward's boundary sums
    cd* seg;                 // [ntasks][64][P][64] forward v of one block
    double* dV;              // [B][nx] (nodes interior to a subdomain)
    cd* du0;                 // [B][nx] (nodes interior to a subdomain)
    double* gends;           // [B][N][2] dJ/dV partial sums at the end nodes
    cd* wends;               // [B][N][2] w at the end nodes
};
hipError_t launch_adjoint(const AdjArgs& a, int kind, int trans, int nitems, int pmax, hipStream_t st);
hipError_t launch_finalize_grad(int N, int nx, int B, const int* off, const double* gends,
                                const cd* wends, double* dV, cd* du0, hipStream_t st);
hipError_t launch_maxabs(const cd* x, long M, int B, double* partial, double* out, hipStream_t st);
hipError_t launch_axpby(const cd* x, double a, const cd* y, double b, cd* z, long n, hipStream_t st);

}  // namespace swr
