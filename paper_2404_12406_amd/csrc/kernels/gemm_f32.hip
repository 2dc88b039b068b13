// fp32 implicit-GEMM kernel for gfx950: the three contractions of a layer
// that is linear in input and weight (Sec. 2.2.1 of the paper) on fp32 NHWC
// activations and KRSC filters.  The GEMM views and the stride-phase split
// of the input gradient are those of igemm.hip.
//
// Bound: the fp32 matrix cores (v_mfma_f32_32x32x2_f32, 64 FLOP per clock and
// SIMD, 157 TFLOP/s on the chip).  At that rate a 128 x 128 x 32 step takes
// 2 us on a CU and reads 32 KB, so the operand path has an order of magnitude
// to spare, and the kernel spends it on generality:
//  * operands go from memory straight into LDS (buffer_load ... lds), 16
//    bytes a lane when every row is whole aligned vectors (V = 4), else 4
//    bytes a lane (V = 1: any channel count, no padded copies).  Padding,
//    ragged tails and missing taps read zeros through the descriptor's range.
//  * the fp32 MFMA and the vector ALU do not overlap (over the main loop, cycles
//    = 64 per MFMA + 4 per vector instruction, counted on 8192^3), so a step's
//    addresses are kept to a few instructions.  Where a step lies in one tap
//    (UT: the reduction's channels a multiple of 32, at most 32 taps; every
//    Linear with K % 32 == 0) each load's lane offset is fixed, the step's part
//    is a scalar, and a tap costs a bit test.  Other reductions decompose k
//    into (tap, channel) once per lane and step, by multiplication (FastDiv).
//  * BK = 32, two LDS stages: the loads of step k + 1 fly during the MFMAs of
//    step k; one barrier a step.
//  * an operand contiguous along k lies as [row][32 k], 16-byte chunks swizzled
//    by row, and a lane reads the four k of one chunk at once; an operand
//    contiguous along m/n lies as [k][m], and a lane reads its TM (TN)
//    adjacent columns of one k at once.  Both feed MFMA step (j, q) with
//    k = 8 j + 4 (lane / 32) + q.
//  * wave tiles of up to 64 x 64 in four waves; each lane ends with TN
//    adjacent output columns and stores them as one vector.
// Tile and split of the reduction are chosen by plan() below.
//
// Measured against the 16x16x4 kernel of igemm.hip that it replaces (us a
// contraction, forward / input gradient / weight gradient, warm: after some 30
// passes; the first dozen after idling run at a lower clock, 10 to 17% slower):
//   4096 x 1024 x 4096        320 / 457 / 424  ->  260 / 265 / 267 (130 TFLOP/s)
//   3x3 64 -> 64, 32 x 56^2   191 / 215 / 275  ->   76 /  79 /  79
//   3x3 256 -> 256, 32 x 14^2 218 / 300 / 120  ->   85 /  88 /  78
//   7x7/2 3 -> 64, 16 x 224^2 126 / 2068 / 202 ->   75 / 664 /  87
//   512 x 768 x 768            73 /  87 /  22  ->   20 /  20 /  18
#include <algorithm>
#include <cmath>

#include "common.h"
#include "lds_dma.h"
#include "limits.h"
#include "../device.h"

namespace ms {

// convolutions of few channels (few_f32.hip)
namespace few {
double fwd_us(const ConvGeom &g, const void *x);
double dgrad_us(const ConvGeom &g, const void *dy);
bool wgrad_applies(const ConvGeom &g);
int conv_fwd(const ConvGeom &g, const void *x, const void *w, const void *bias, void *y, hipStream_t st);
int conv_dgrad(const ConvGeom &g, const void *dy, const void *w, const void *bias, void *dx, hipStream_t st);
int wgrad_parts(const ConvGeom &g, const void *dy, const void *x, float *part, int64_t stride, int n, hipStream_t st);
}  // namespace few

namespace f32g {

using g2::dma16s;
using g2::dma4s;
using g2::kOOB;

enum Mode { kFwd = 0, kDgrad = 1, kWgrad = 2 };

constexpr int BK = 32;    // reduction step: a 128-byte row
// Steps an accumulator runs before it is added up (even).  The weight
// gradient's is shorter: its long sums were split into chains of 64 pixels and
// more before, and its error is to be no larger.
template <int MODE> constexpr int flush_steps() { return MODE == kWgrad ? 4 : 8; }

// Division of n < 2^31 by a fixed d >= 1: q = (umulhi(n, m) + n) >> s, the
// round-up reciprocal of Granlund and Montgomery, Division by Invariant Integers
// using Multiplication (1994).
struct FastDiv {
    uint32_t m, s, d;
};
FastDiv fastdiv(uint32_t d) {
    FastDiv f{0, 0, std::max<uint32_t>(d, 1)};
    while ((1ull << f.s) < f.d) ++f.s;
    f.m = (uint32_t)((((1ull << f.s) - f.d) << 32) / f.d + 1);
    return f;
}
__device__ __forceinline__ uint32_t quot(uint32_t n, const FastDiv &f) { return (__umulhi(n, f.m) + n) >> f.s; }

struct Args {
    const float *a, *b, *bias;
    float *c;        // output, or split partials (splits > 1)
    ConvGeom g;
    int M, N, K;     // GEMM extents (DGRAD: bounds over the stride phases)
    int ntm, ntn;
    int splits, k_split;
    int64_t part_stride;   // floats between the partials of two splits
    uint32_t a_bytes, b_bytes;
    FastDiv dch;     // channels of the reduction: C (FWD), K (DGRAD); WGRAD: C of the columns
    FastDiv ds;      // S
    FastDiv dpq, dq; // P * Q and Q
};

struct Phase {
    int fh, fw, h0, w0, Hp, Wp, Rp, Sp, dh, dw;
};

__device__ __forceinline__ Phase make_phase(const ConvGeom &g, int z) {
    Phase f;
    f.fh = z / g.sw;
    f.fw = z % g.sw;
    f.h0 = ((f.fh - g.ph) % g.sh + g.sh) % g.sh;
    f.w0 = ((f.fw - g.pw) % g.sw + g.sw) % g.sw;
    f.Hp = f.h0 < g.H ? (g.H - f.h0 + g.sh - 1) / g.sh : 0;
    f.Wp = f.w0 < g.W ? (g.W - f.w0 + g.sw - 1) / g.sw : 0;
    f.Rp = f.fh < g.R ? (g.R - f.fh + g.sh - 1) / g.sh : 0;
    f.Sp = f.fw < g.S ? (g.S - f.fw + g.sw - 1) / g.sw : 0;
    f.dh = (f.h0 + g.ph - f.fh) / g.sh;
    f.dw = (f.w0 + g.pw - f.fw) / g.sw;
    return f;
}

// Exact quotient of two numbers below 2^16 through the reciprocal m =
// ceil(2^32 / d) (n * d < 2^32).
__device__ __forceinline__ int small_quot(int n, uint32_t m, int d) { return d == 1 ? n : (int)__umulhi((uint32_t)n, m); }

template <int N> struct Const { static constexpr int value = N; };

// Floats T adjacent in LDS, read at once.
template <int T> struct Run { float e[T]; };

// One operand tile of R rows (or columns) x BK in LDS.
template <int R, int V, bool KC>
struct Tile {
    static constexpr int BYTES = R * BK * 4;
    static constexpr int INS = BYTES / (V * 256);   // load instructions of one wave each
    static constexpr int NI = INS / 4;              // per wave
    static_assert(NI >= 1 && NI * 4 == INS, "load split");
    // KC: 16-byte chunk c of row r lies at slot c ^ key(r): the 16 rows that
    // one pass of a 16-byte read serves fall on 16 different bank groups
    static __device__ __forceinline__ int key(int row) { return (row >> 1) & 7; }
    // MC: the two half-waves read k-rows 4 apart, which share their banks;
    // rows of 64 and more columns move every second group of four rows by
    // 32 columns, rows of 32 trade places with their neighbour
    static __device__ __forceinline__ int shift(int k) { return V == 4 && R >= 64 ? ((k >> 2) & 1) * 32 : 0; }
    static __device__ __forceinline__ int place(int k) { return V == 4 && R == 32 ? k ^ ((k >> 2) & 1) : k; }
};

template <int MODE, int BM, int BN, int WR, int WC, int V, int OCC, bool UT>
__global__ __launch_bounds__(256, OCC) void gemm_kernel(const Args P) {
    constexpr bool A_KC = MODE != kWgrad, B_KC = MODE == kFwd;
    using TA = Tile<BM, V, A_KC>;
    using TB = Tile<BN, V, B_KC>;
    constexpr int NIA = TA::NI, NIB = TB::NI;
    constexpr int WM = BM / WR, WN = BN / WC, TM = WM / 32, TN = WN / 32;
    static_assert(!UT || V == 4, "tap steps read whole vectors");
    static_assert(WR * WC == 4 && TM >= 1 && TN >= 1 && TM <= 2 && TN <= 2, "wave tile");
    __shared__ __attribute__((aligned(1024))) char smem[2 * (TA::BYTES + TB::BYTES)];

    const ConvGeom &g = P.g;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm0 = (wave / WC) * WM, wn0 = (wave % WC) * WN;

    int M = P.M, Kg = P.K, ntm = P.ntm;
    const int N = P.N;
    const int zsplit = (int)blockIdx.z % P.splits, zphase = (int)blockIdx.z / P.splits;
    Phase f{};
    if constexpr (MODE == kDgrad) {
        f = make_phase(g, zphase);
        M = g.N * f.Hp * f.Wp;
        Kg = f.Rp * f.Sp * g.K;
        ntm = (M + BM - 1) / BM;
    }
    int k_begin = 0, k_end = Kg;
    if (P.splits > 1) {
        k_begin = min(Kg, zsplit * P.k_split);
        k_end = min(Kg, k_begin + P.k_split);
    }
    // XCD-aware tile order, 8 row tiles sharing each column sweep
    int tm, tn;
    {
        const int lt = xcd_remap((int)blockIdx.x, P.ntm * P.ntn);
        const int GM = 8, per = GM * P.ntn;
        const int gid = lt / per, first = gid * GM;
        const int gsz = min(P.ntm - first, GM);
        const int r = lt - gid * per;
        tm = first + r % gsz;
        tn = r / gsz;
    }
    if (tm >= ntm) return;   // a stride phase smaller than the bound; nothing in flight
    const int m0 = tm * BM, n0 = tn * BN;
    const int nk = k_end > k_begin ? (k_end - k_begin + BK - 1) / BK : 0;

    // UT: the A descriptor starts a_shift elements early, so that the offset of
    // a row's first tap, which may lie in the padding, is not negative; only
    // taps inside the image are read
    int a_shift = 0;
    if constexpr (UT && MODE == kFwd) a_shift = (g.ph * g.W + g.pw) * g.C;
    if constexpr (UT && MODE == kDgrad) a_shift = max(0, ((f.Rp - 1 - f.dh) * g.Q + f.Sp - 1 - f.dw) * g.K);
    const __amdgpu_buffer_rsrc_t ra = g2::rsrc(P.a - a_shift, P.a_bytes + (uint32_t)a_shift * 4u);
    const __amdgpu_buffer_rsrc_t rb = g2::rsrc(P.b, P.b_bytes);

    // ---------------------------------------------- what each lane loads
    // Instruction i of this wave is number wave + 4 i of the tile.  KC: it
    // covers 2 V rows, its lane's chunk (V = 4) or word (V = 1) of the row;
    // NVK variants of the lane's k over i (V = 1: the key alternates).
    constexpr int NVK = V == 4 ? 1 : 2;
    constexpr int LPR = BK / V;                     // lanes per KC row
    auto kc_row = [&](int i) { return (wave + 4 * i) * (64 / LPR) + lane / LPR; };
    auto kc_k = [&](int v) {                        // k within the step, variant v
        const int w = (lane % LPR) * V;             // word within the LDS row
        return ((w / 4) ^ TA::key(kc_row(v))) * 4 + w % 4;
    };
    // A_KC: pixel (y, x) of row i at tap (0, 0) and its element offset; UT: byte
    // offset at the tap that lies first in memory, and the taps inside the image
    int a_base[A_KC ? NIA : 1], a_y[A_KC && !UT ? NIA : 1], a_x[A_KC && !UT ? NIA : 1];
    uint32_t a_mask[UT && A_KC ? NIA : 1];
    int b_base[B_KC ? NIB : 1];
    if constexpr (A_KC) {
        const unsigned HH = MODE == kFwd ? g.H : g.P, WW = MODE == kFwd ? g.W : g.Q;
#pragma unroll
        for (int i = 0; i < NIA; ++i) {
            const int m = m0 + kc_row(i);
            const int mm = m < M ? m : 0;
            int y, x, base;
            if constexpr (MODE == kFwd) {
                const int n = (int)quot(mm, P.dpq), pq = mm - n * (int)P.dpq.d;
                const int p = (int)quot(pq, P.dq), q = pq - p * (int)P.dq.d;
                y = p * g.sh - g.ph;
                x = q * g.sw - g.pw;
                base = ((n * g.H + y) * g.W + x) * g.C;
            } else {
                const int HW = f.Hp * f.Wp;
                const int n = HW > 0 ? mm / HW : 0, ij = mm - n * HW;
                const int i2 = f.Wp > 0 ? ij / f.Wp : 0, j2 = ij - i2 * f.Wp;
                y = i2 + f.dh;
                x = j2 + f.dw;
                base = ((n * g.P + y) * g.Q + x) * g.K;
            }
            if constexpr (UT) {
                constexpr int SG = MODE == kFwd ? 1 : -1;
                const int nr = MODE == kFwd ? g.R : f.Rp, ns = MODE == kFwd ? g.S : f.Sp;
                if (MODE == kDgrad) base -= ((f.Rp - 1) * g.Q + f.Sp - 1) * g.K;
                a_base[i] = (base + a_shift + kc_k(0)) * 4;
                uint32_t mask = 0;
                if (m < M) {
                    for (int t = 0, r = 0, sx = 0; t < nr * ns; ++t) {
                        if ((unsigned)(y + SG * r) < HH && (unsigned)(x + SG * sx) < WW) mask |= 1u << t;
                        if (++sx == ns) {
                            sx = 0;
                            ++r;
                        }
                    }
                }
                a_mask[i] = mask;
            } else {
                a_base[i] = base;
                a_y[i] = m < M ? y : INT32_MIN / 2;   // never inside
                a_x[i] = x;
            }
        }
    }
    if constexpr (B_KC) {
        // LDS row 32 j + l of a wave's columns holds column l TN + j: a lane's
        // TN results are then adjacent
#pragma unroll
        for (int i = 0; i < NIB; ++i) {
            const int row = kc_row(i), w0 = row / WN * WN, r = row - w0;
            const int n = n0 + w0 + (r % 32) * TN + r / 32;
            if constexpr (UT) b_base[i] = n < N ? (n * Kg + kc_k(0)) * 4 : (int)kOOB;
            else b_base[i] = n < N ? n * Kg : -1;
        }
    }
    // MC: instruction covers 64 V / R k-rows (or part of one); the lane's column
    // is the same for every instruction of the tile
    auto mc_k = [&](int i, int R) { return ((wave + 4 * i) * 64 + lane) * V / R; };
    auto mc_col = [&](int R) { return (wave * 64 + lane) * V % R; };
    int a_col = 0, b_col = 0;
    if constexpr (!A_KC) a_col = m0 + (mc_col(BM) ^ TA::shift(TA::place(mc_k(0, BM))));
    if constexpr (!B_KC) b_col = n0 + (mc_col(BN) ^ TB::shift(TB::place(mc_k(0, BN))));
    // WGRAD: (tap, channel) of the lane's B columns
    int w_r = 0, w_s = 0, w_off = 0;
    const bool a_ok = a_col < M, b_ok = b_col < N;
    if constexpr (MODE == kWgrad) {
        const int nn = b_ok ? b_col : 0;
        const int rs = (int)quot(nn, P.dch), c = nn - rs * (int)P.dch.d;
        w_r = (int)quot(rs, P.ds);
        w_s = rs - w_r * (int)P.ds.d;
        w_off = (w_r * g.W + w_s) * g.C + c;
    }
    const uint32_t sp_m = MODE == kDgrad && f.Sp > 1 ? 0xFFFFFFFFu / (uint32_t)f.Sp + 1u : 0u;

    // UT: tap cursor of the step being loaded (uniform), advanced in order
    int u_t = 0, u_r = 0, u_s = 0, u_c0 = 0;
    if constexpr (UT && MODE != kWgrad) {
        u_t = (int)quot(k_begin, P.dch);
        u_c0 = k_begin - u_t * (int)P.dch.d;
        const int ns = MODE == kFwd ? g.S : max(f.Sp, 1);
        u_r = u_t / ns;
        u_s = u_t - u_r * ns;
    }
    auto u_next = [&]() {
        u_c0 += BK;
        if (u_c0 == (int)P.dch.d) {
            u_c0 = 0;
            ++u_t;
            if (++u_s == (MODE == kFwd ? g.S : f.Sp)) {
                u_s = 0;
                ++u_r;
            }
        }
    };

    // One step's loads, in parts: part `part` of `parts` (part < 0: all of
    // them).  Loads past the reduction read zeros, or (UT) bytes of the operand
    // that no one uses.
    int dy[NVK], dx[NVK], del[NVK], kb[NVK];
    bool in[NVK];
    auto prep = [&](int k0) __attribute__((always_inline)) {
        if constexpr (A_KC && !UT) {
#pragma unroll
            for (int v = 0; v < NVK; ++v) {
                const int kk = k0 + kc_k(v);
                in[v] = kk < k_end;
                kb[v] = kk;
                const int t = (int)quot(kk, P.dch), ch = kk - t * (int)P.dch.d;
                if constexpr (MODE == kFwd) {
                    const int r = (int)quot(t, P.ds), s = t - r * (int)P.ds.d;
                    dy[v] = r;
                    dx[v] = s;
                    del[v] = (r * g.W + s) * g.C + ch;
                } else {
                    const int r = small_quot(t, sp_m, f.Sp), s = t - r * f.Sp;
                    dy[v] = -r;
                    dx[v] = -s;
                    del[v] = ch - (r * g.Q + s) * g.K;
                }
            }
        }
    };
    auto issue = [&](int stage, int k0, int part, int parts) __attribute__((always_inline)) {
        char *sA = smem + stage * (TA::BYTES + TB::BYTES), *sB = sA + TA::BYTES;
        auto put = [&](__amdgpu_buffer_rsrc_t r, char *dst, uint32_t off, uint32_t soff) {
            if constexpr (V == 4) dma16s(r, dst, off, soff);
            else dma4s(r, dst, off, soff);
        };
        auto mine = [&](int i) { return part < 0 || i * parts / (NIA + NIB) == part; };
        const bool live = k0 < k_end;
        // uniform parts of the UT offsets (zero past the end: in bounds)
        uint32_t a_so = 0, b_so = 0, bit = 0;
        if constexpr (UT && MODE != kWgrad) {
            if (live) {
                bit = 1u << (u_t & 31);
                if constexpr (MODE == kFwd) {
                    a_so = (uint32_t)((u_r * g.W + u_s) * g.C + u_c0) * 4u;
                    b_so = (uint32_t)k0 * 4u;
                } else {
                    a_so = (uint32_t)(((f.Rp - 1 - u_r) * g.Q + f.Sp - 1 - u_s) * g.K + u_c0) * 4u;
                    b_so = (uint32_t)(((u_c0 * g.R + f.fh + u_r * g.sh) * g.S + f.fw + u_s * g.sw) * g.C) * 4u;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NIA; ++i) {
            if (!mine(i)) continue;
            uint32_t off;
            if constexpr (A_KC && UT) {
                off = (a_mask[i] & bit) ? (uint32_t)a_base[i] : kOOB;
            } else if constexpr (A_KC) {
                const unsigned HH = MODE == kFwd ? g.H : g.P, WW = MODE == kFwd ? g.W : g.Q;
                const int v = i % NVK;
                const bool ok = in[v] && (unsigned)(a_y[i] + dy[v]) < HH && (unsigned)(a_x[i] + dx[v]) < WW;
                off = ok ? (uint32_t)(a_base[i] + del[v]) * 4u : kOOB;
            } else {
                const int k = TA::place(mc_k(i, BM));
                off = a_ok && k0 + k < k_end ? ((uint32_t)k * (uint32_t)g.K + (uint32_t)a_col) * 4u : kOOB;
                a_so = live ? (uint32_t)k0 * (uint32_t)g.K * 4u : 0u;
            }
            put(ra, sA + (wave + 4 * i) * (V * 256), off, a_so);
        }
#pragma unroll
        for (int i = 0; i < NIB; ++i) {
            if (!mine(NIA + i)) continue;
            uint32_t off;
            if constexpr (B_KC && UT) {
                off = (uint32_t)b_base[i];
            } else if constexpr (B_KC) {
                const int v = i % NVK;
                off = in[v] && b_base[i] >= 0 ? (uint32_t)(b_base[i] + kb[v]) * 4u : kOOB;
            } else if constexpr (MODE == kDgrad && UT) {
                const int k = TB::place(mc_k(i, BN));
                off = b_ok ? (uint32_t)(k * g.R * g.S * g.C + b_col) * 4u : kOOB;
            } else if constexpr (MODE == kWgrad && UT) {   // unit geometry: pixel rows of C floats
                const int k = TB::place(mc_k(i, BN));
                off = b_ok && k0 + k < k_end ? ((uint32_t)k * (uint32_t)g.C + (uint32_t)b_col) * 4u : kOOB;
                b_so = live ? (uint32_t)k0 * (uint32_t)g.C * 4u : 0u;
            } else {
                const int k = TB::place(mc_k(i, BN)), kk = k0 + k;
                bool ok = kk < k_end && b_ok;
                if constexpr (MODE == kDgrad) {
                    const int t = (int)quot(kk, P.dch), ch = kk - t * (int)P.dch.d;
                    const int tr = small_quot(t, sp_m, f.Sp), ts = t - tr * f.Sp;
                    off = (uint32_t)(((ch * g.R + f.fh + tr * g.sh) * g.S + f.fw + ts * g.sw) * g.C + b_col);
                } else {
                    const int n = (int)quot(kk, P.dpq), pq = kk - n * (int)P.dpq.d;
                    const int p = (int)quot(pq, P.dq), q = pq - p * (int)P.dq.d;
                    const int ih = p * g.sh - g.ph, iw = q * g.sw - g.pw;
                    ok = ok && (unsigned)(ih + w_r) < (unsigned)g.H && (unsigned)(iw + w_s) < (unsigned)g.W;
                    off = (uint32_t)(((n * g.H + ih) * g.W + iw) * g.C + w_off);
                }
                off = ok ? off * 4u : kOOB;
            }
            put(rb, sB + (wave + 4 * i) * (V * 256), off, b_so);
        }
    };

    // acc runs over kFlush steps, then is added to sum: the rounding errors of
    // a K-long sum grow like sqrt(256 + K / 256) instead of sqrt(K).  Against 64
    // bits, forward, input and weight gradient of 4096 x 1024 x 4096: 2.9e-7,
    // 3.0e-7 and 2.3e-7; the three together 5.7e-7 as one chain, 2.9e-7 so.
    constexpr int kFlush = flush_steps<MODE>();
    floatx16 acc[TM][TN], sum[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = sum[i][j][v] = 0.f;

    const int l32 = lane & 31, half = lane >> 5;
    // LDS offsets of the fragments, without the stage's and the unrolled parts
    int a_frag[A_KC ? BK / 8 : 1], b_frag[B_KC ? BK / 8 : 1];
    if constexpr (A_KC) {
#pragma unroll
        for (int j = 0; j < BK / 8; ++j) a_frag[j] = (wm0 + l32) * (BK * 4) + (((2 * j + half) ^ TA::key(l32)) << 4);
    }
    if constexpr (B_KC) {
#pragma unroll
        for (int j = 0; j < BK / 8; ++j) b_frag[j] = (wn0 + l32) * (BK * 4) + (((2 * j + half) ^ TB::key(l32)) << 4);
    }
    auto step = [&](auto stage_c, int kt) __attribute__((always_inline)) {
        constexpr int ST = decltype(stage_c)::value;
        g2::wait_vmcnt<0>();
        g2::wait_lgkm0();         // this wave has read the other stage: the refills below are not
                                  // tracked, so nothing else keeps them behind its reads
        g2::block_sync<true>();   // step kt has landed for every wave; the other stage is free
        const int k1 = k_begin + (kt + 1) * BK;
        if constexpr (UT && MODE != kWgrad) u_next();
        prep(k1);
        const char *sA = smem + ST * (TA::BYTES + TB::BYTES), *sB = sA + TA::BYTES;
#pragma unroll
        for (int j = 0; j < BK / 8; ++j) {
            float fa[TM][4], fb[TN][4];
            if constexpr (A_KC) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    *reinterpret_cast<floatx4 *>(fa[i]) =
                        *reinterpret_cast<const floatx4 *>(sA + a_frag[j] + i * 32 * (BK * 4));
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int k = 8 * j + 4 * half + q;
                    const int col = (wm0 + l32 * TM) ^ TA::shift(4 * half);
                    const Run<TM> r = *reinterpret_cast<const Run<TM> *>(sA + (TA::place(k) * BM + col) * 4);
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[i][q] = r.e[i];
                }
            }
            if constexpr (B_KC) {
#pragma unroll
                for (int i = 0; i < TN; ++i)
                    *reinterpret_cast<floatx4 *>(fb[i]) =
                        *reinterpret_cast<const floatx4 *>(sB + b_frag[j] + i * 32 * (BK * 4));
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int k = 8 * j + 4 * half + q;
                    const int col = (wn0 + l32 * TN) ^ TB::shift(4 * half);
                    const Run<TN> r = *reinterpret_cast<const Run<TN> *>(sB + (TB::place(k) * BN + col) * 4);
#pragma unroll
                    for (int i = 0; i < TN; ++i) fb[i][q] = r.e[i];
                }
            }
            if (j < 2) issue(ST ^ 1, k1, j, 2);   // early in the step: they have the rest of it to land
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int n = 0; n < TN; ++n)
                        acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][q], fb[n][q], acc[i][n], 0, 0, 0);
        }
    };
    prep(k_begin);
    if (nk > 0) issue(0, k_begin, -1, 1);
    for (int kt = 0; kt < nk; kt += 2) {
        step(Const<0>{}, kt);
        if (kt + 1 < nk) step(Const<1>{}, kt + 1);
        if (kt % kFlush == kFlush - 2) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int n = 0; n < TN; ++n)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        sum[i][n][v] += acc[i][n][v];
                        acc[i][n][v] = 0.f;
                    }
        }
    }
    g2::wait_vmcnt<0>();   // the last refill (zeros) writes this block's LDS
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int n = 0; n < TN; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][n][v] += sum[i][n][v];

    // ---------------------------------------------- epilogue
    // acc[i][j][v]: row rr = 8 (v / 4) + 4 half + v % 4 of the wave's tile i
    // (A along k: row 32 i + rr; else rr TM + i), column l32 TN + j.
    const int n = n0 + wn0 + l32 * TN;
    float bv[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bv[j] = MODE != kWgrad && P.bias && n + j < N ? P.bias[n + j] : 0.f;
    float *out = P.c + (P.splits > 1 ? (size_t)zsplit * P.part_stride : 0);
    // pairs of columns as one store when every row starts even
    const bool pair = TN == 2 && (N & 1) == 0 && (reinterpret_cast<uintptr_t>(out) & 7u) == 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rr = 8 * (v / 4) + 4 * half + v % 4;
            const int m = m0 + wm0 + (A_KC ? 32 * i + rr : rr * TM + i);
            if (m >= M || n >= N) continue;
            size_t row = (size_t)m;
            if constexpr (MODE == kDgrad) {
                if (g.sh != 1 || g.sw != 1) {
                    const int HW = f.Hp * f.Wp;
                    const int im = m / HW, ij = m - im * HW, i2 = ij / f.Wp, j2 = ij - i2 * f.Wp;
                    row = ((size_t)im * g.H + f.h0 + i2 * g.sh) * g.W + f.w0 + j2 * g.sw;
                }
            }
            float *dst = out + row * N + n;
            if constexpr (TN == 2) {
                typedef float floatx2 __attribute__((ext_vector_type(2)));
                if (pair) {
                    *reinterpret_cast<floatx2 *>(dst) = floatx2{acc[i][0][v] + bv[0], acc[i][1][v] + bv[1]};
                } else {
                    dst[0] = acc[i][0][v] + bv[0];
                    if (n + 1 < N) dst[1] = acc[i][1][v] + bv[1];
                }
            } else {
                dst[0] = acc[i][0][v] + bv[0];
            }
        }
}

// out[i] = bias[i % ncol] + sum_z part[z * stride + i], in a fixed order.  A
// block owns 256 / G float4 columns; its G thread groups take every G-th
// split, eight loads in flight, and meet in LDS.
template <int G>
__global__ __launch_bounds__(256) void reduce_kernel(const float *__restrict__ part, int splits, int64_t n4,
                                                     int64_t stride4, const float *__restrict__ bias, int ncol,
                                                     int64_t n, float *__restrict__ out) {
    constexpr int COLS = 256 / G;
    __shared__ floatx4 red[G][COLS];
    const int col = threadIdx.x % COLS, grp = threadIdx.x / COLS;
    const int64_t i = (int64_t)blockIdx.x * COLS + col;
    const floatx4 *p = reinterpret_cast<const floatx4 *>(part);
    floatx4 s = {0.f, 0.f, 0.f, 0.f};
    if (i < n4) {
        for (int z = grp; z < splits; z += 8 * G) {
            floatx4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (z + u * G < splits) v[u] = p[(int64_t)(z + u * G) * stride4 + i];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    }
    if constexpr (G > 1) {
        red[grp][col] = s;
        __syncthreads();
        if (grp != 0) return;
        for (int q = 1; q < G; ++q) s += red[q][col];
    }
    if (i >= n4) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t k = i * 4 + e;
        if (k < n) out[k] = s[e] + (bias ? bias[k % ncol] : 0.f);
    }
}

// ------------------------------------------------------------------ host
namespace {

struct TileInfo {
    int bm, bn, per_cu;
    double eff;   // share of the fp32 MFMA rate when CUs are full
};
// 128 x 128 first; 32-wide columns for few output channels, 32-wide rows
// for a weight gradient of few.  The shares, and est_us() with its splits, against
// measurement (us measured / estimated, every tile forced; * the planner's choice):
//                                128x128     128x64      64x64       128x32      32x128
//   512 x 768 x 768, forward     24.4/22.7  *19.3/17.8   17.6/18.3   18.3/18.7
//   2048 x 1024 x 1024, dx       51.8/51.8  *45.0/41.8   40.9/45.0   44.5/47.8
//   3x3 64 -> 64, 32 x 56^2       174/169    92.7/92.4  *80.7/89.5   87.6/95.1
//     weight gradient             152/140     150/135   *82.6/82.6    140/156     104/89.7
//   3x3 256 -> 256, 32 x 14^2    86.5/91.0  *85.9/83.9   78.6/91.2   83.5/97.2
//     weight gradient           *77.5/76.4   74.3/78.6   81.7/84.3   74.2/89.2   90.6/89.2
//   3x3 512 -> 512, 32 x 7^2     84.0/91.0   89.2/89.5  *70.6/84.1   88.3/103
//   3x3 32 -> 32, 16 x 64^2      50.7/47.7   29.8/27.9   28.4/29.9  *19.6/19.1
//     weight gradient            69.4/63.4   58.2/53.1   35.0/34.8   53.0/58.7  *29.1/27.7
// Over 30 such passes the choice is within 5% of the fastest tile, but for five
// where 64 x 64, whose share is 10% low on whole reduction steps, was 6 to 13%
// faster.
constexpr TileInfo kTiles[] = {{128, 128, 2, 0.85}, {128, 64, 3, 0.82}, {64, 64, 4, 0.75}, {128, 32, 4, 0.70}, {32, 128, 4, 0.70}};
constexpr int kNumTiles = 5;
constexpr int kCUs = 256;
constexpr double kFlopsPerUs = 0.60e6;   // one CU's fp32 MFMA rate, per us
constexpr int64_t kPartialCap = int64_t(16) << 20;

struct Plan {
    int tile, splits, k_split;
    double us;   // estimated
};

// Estimated time of z GEMMs of M x N x K in us: the busiest CU's blocks, each
// a chain of BK steps bound by the MFMAs or (alone on its CU) by the load
// round trip, plus the partials' traffic and the reduction's launch.
double est_us(const TileInfo &t, int64_t M, int64_t N, int64_t K, int z, int splits) {
    const int64_t blocks = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * z * splits;
    const int64_t per = (blocks + kCUs - 1) / kCUs;   // blocks of the busiest CU
    const int64_t steps = (K + splits - 1) / splits / BK + 1;
    const double mfma = 2.0 * t.bm * t.bn * BK / (kFlopsPerUs * t.eff);
    const double conc = (double)std::min<int64_t>(per, t.per_cu);
    const double step = std::max(mfma, 1.0 / conc);
    double us = (double)per * (steps * step + 1.5 / conc) + 3.0;
    const double out = 4.0 * (double)M * N * z;
    us += out * splits / 4.0e6;
    if (splits > 1) us += 4.0 + out * splits / 4.0e6;
    return us;
}

// floats between the partials of two splits: whole vectors
int64_t part_stride(int64_t elems) { return (elems + 3) / 4 * 4; }

// `cap_bytes`: what the partials, part_stride(out_elems) apart, may take
Plan plan(int mode, int64_t M, int64_t N, int64_t K, int z, int64_t out_elems, int64_t cap_bytes) {
    Plan best{0, 1, 0, 1e300};
    for (int ti = 0; ti < kNumTiles; ++ti) {
        const TileInfo &t = kTiles[ti];
        if (t.bm == 32 && mode != kWgrad) continue;   // rows are pixels there: never few
        const int64_t most = std::max<int64_t>(1, std::min<int64_t>(K / (4 * BK), cap_bytes / std::max<int64_t>(1, 4 * part_stride(out_elems))));
        for (int64_t sp = 1; sp <= std::min<int64_t>(most, 1024); sp += sp < 16 ? 1 : sp / 8) {
            const double us = est_us(t, M, N, K, z, (int)sp);
            if (us < best.us * 0.999) {
                best.us = us;
                best.tile = ti;
                best.splits = (int)sp;
            }
        }
    }
    const int64_t per = ((K + best.splits - 1) / best.splits + BK - 1) / BK * BK;
    best.k_split = (int)std::min<int64_t>(std::max<int64_t>(per, BK), INT32_MAX / 2);
    best.splits = (int)std::max<int64_t>(1, (K + best.k_split - 1) / best.k_split);
    return best;
}

bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
size_t part_bytes(const Plan &p, int64_t elems) {
    return p.splits > 1 ? (size_t)p.splits * part_stride(elems) * sizeof(float) : 0;
}

int64_t x_elems(const ConvGeom &g) { return (int64_t)g.N * g.H * g.W * g.C; }
int64_t y_elems(const ConvGeom &g) { return (int64_t)g.N * g.P * g.Q * g.K; }
int64_t w_elems(const ConvGeom &g) { return (int64_t)g.K * g.R * g.S * g.C; }
// 32-bit byte offsets of 4-byte elements; k and tap indexes below 2^31 / 2^16
bool fits(int64_t elems) { return elems * 4 <= (int64_t)(kOOB)-16; }
bool geom_ok(const ConvGeom &g) {
    return fits(x_elems(g)) && fits(y_elems(g)) && fits(w_elems(g)) && (int64_t)g.R * g.S <= 65535;
}

Plan fwd_plan(const ConvGeom &g) {
    return plan(kFwd, (int64_t)g.N * g.P * g.Q, g.K, (int64_t)g.R * g.S * g.C, 1, y_elems(g), kPartialCap);
}
Plan dgrad_plan(const ConvGeom &g) {
    const int64_t Hb = (g.H + g.sh - 1) / g.sh, Wb = (g.W + g.sw - 1) / g.sw;
    const int64_t Kb = (int64_t)((g.R + g.sh - 1) / g.sh) * ((g.S + g.sw - 1) / g.sw) * g.K;
    return plan(kDgrad, g.N * Hb * Wb, g.C, Kb, g.sh * g.sw, x_elems(g), kPartialCap);
}
Plan wgrad_plan(const ConvGeom &g, int64_t cap_bytes) {
    return plan(kWgrad, g.K, (int64_t)g.R * g.S * g.C, (int64_t)g.N * g.P * g.Q, 1, w_elems(g), cap_bytes);
}

template <int MODE, int BM, int BN, int WR, int WC, int V, int OCC, bool UT>
int go(const Args &a, dim3 grid, hipStream_t st) {
    const unsigned pk = MODE == kFwd ? kProfFwd : MODE == kDgrad ? kProfDgrad : kProfWgrad;
    prof_mark(pk, st, true);
    hipLaunchKernelGGL((gemm_kernel<MODE, BM, BN, WR, WC, V, OCC, UT>), grid, dim3(256), 0, st, a);
    const int err = (int)hipGetLastError();
    prof_mark(pk, st, false);
    return err;
}

template <int MODE, int V, bool UT>
int go_tile(int tile, const Args &a, dim3 grid, hipStream_t st) {
    switch (tile) {
    case 0:
        if constexpr (V == 4) return go<MODE, 128, 128, 2, 2, V, 2, UT>(a, grid, st);
        return (int)hipErrorInvalidValue;
    case 1: return go<MODE, 128, 64, 2, 2, V, V == 4 ? 3 : 2, UT>(a, grid, st);
    case 2: return go<MODE, 64, 64, 2, 2, V, V == 4 ? 4 : 3, UT>(a, grid, st);
    case 3: return go<MODE, 128, 32, 4, 1, V, V == 4 ? 4 : 3, UT>(a, grid, st);
    default:
        if constexpr (MODE == kWgrad) return go<MODE, 32, 128, 1, 4, V, V == 4 ? 4 : 3, UT>(a, grid, st);
        return (int)hipErrorInvalidValue;
    }
}

int reduce(const float *part, int splits, int64_t n, const float *bias, int ncol, float *out, hipStream_t st) {
    const int64_t n4 = (n + 3) / 4, s4 = part_stride(n) / 4;
    // thread groups per column: more while blocks are few and splits many
    const int G = n4 >= 65536 || splits < 8 ? 1 : n4 >= 8192 || splits < 64 ? 4 : 32;
    const dim3 grid((unsigned)((n4 + 256 / G - 1) / (256 / G)));
    if (G == 1) hipLaunchKernelGGL(reduce_kernel<1>, grid, dim3(256), 0, st, part, splits, n4, s4, bias, ncol, n, out);
    else if (G == 4) hipLaunchKernelGGL(reduce_kernel<4>, grid, dim3(256), 0, st, part, splits, n4, s4, bias, ncol, n, out);
    else hipLaunchKernelGGL(reduce_kernel<32>, grid, dim3(256), 0, st, part, splits, n4, s4, bias, ncol, n, out);
    return (int)hipGetLastError();
}

// Steps of one tap each with fixed lane offsets (see the kernel): the
// reduction's channels whole steps and at most 32 taps (of a stride phase);
// for the weight gradient, pixels in memory order (1 x 1, stride 1, no pad).
// The shifted A descriptor stays below the out-of-range offset.
template <int MODE>
bool tap_steps(const ConvGeom &g) {
    if (MODE == kWgrad) return g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
    if (MODE == kFwd) return g.C % BK == 0 && g.R * g.S <= 32 && fits(x_elems(g) + ((int64_t)g.ph * g.W + g.pw) * g.C);
    const int64_t Rb = (g.R + g.sh - 1) / g.sh, Sb = (g.S + g.sw - 1) / g.sw;
    return g.K % BK == 0 && Rb * Sb <= 32 && fits(y_elems(g) + (Rb * g.Q + Sb) * g.K);
}

template <int MODE>
int run(const Plan &p, bool vec, Args &a, int z, int64_t out_elems, const float *bias, float *out, void *ws, hipStream_t st) {
    // 4-byte loads keep a row's pixel per load in registers: no 128 x 128 tile
    const int tile = p.tile == 0 && !vec ? 1 : p.tile;
    const TileInfo &t = kTiles[tile];
    a.ntm = (a.M + t.bm - 1) / t.bm;
    a.ntn = (a.N + t.bn - 1) / t.bn;
    a.splits = p.splits;
    a.k_split = p.k_split;
    a.part_stride = part_stride(out_elems);
    a.c = p.splits > 1 ? static_cast<float *>(ws) : out;
    a.bias = p.splits > 1 ? nullptr : bias;
    a.a_bytes = (uint32_t)(MODE == kFwd ? x_elems(a.g) * 4 : y_elems(a.g) * 4);
    a.b_bytes = (uint32_t)(MODE == kWgrad ? x_elems(a.g) * 4 : w_elems(a.g) * 4);
    a.dch = fastdiv(MODE == kDgrad ? a.g.K : a.g.C);
    a.ds = fastdiv(a.g.S);
    a.dpq = fastdiv(a.g.P * a.g.Q);
    a.dq = fastdiv(a.g.Q);
    const dim3 grid((unsigned)(a.ntm * a.ntn), 1, (unsigned)(z * p.splits));
    const int err = !vec ? go_tile<MODE, 1, false>(tile, a, grid, st)
                    : tap_steps<MODE>(a.g) ? go_tile<MODE, 4, true>(tile, a, grid, st)
                                           : go_tile<MODE, 4, false>(tile, a, grid, st);
    if (err || p.splits <= 1) return err;
    return reduce(static_cast<const float *>(ws), p.splits, out_elems, bias, a.N, out, st);
}

}  // namespace

// Partial rows of the few-channel weight gradient, two blocks a CU; 0: the GEMM
// takes it.
static int few_rows(const ConvGeom &g, size_t cap) {
    const int64_t rows = std::min<int64_t>(512, (int64_t)cap / (part_stride(w_elems(g)) * 4));
    return rows >= 64 && few::wgrad_applies(g) ? (int)rows : 0;
}

// Workspace in bytes (split partials).  A forward or input gradient that is
// given no workspace runs unsplit.
size_t fwd_workspace(const ConvGeom &g) { return geom_ok(g) ? part_bytes(fwd_plan(g), y_elems(g)) : 0; }
size_t dgrad_workspace(const ConvGeom &g) { return geom_ok(g) ? part_bytes(dgrad_plan(g), x_elems(g)) : 0; }

// Each returns -1 when an operand is too large for 32-bit byte offsets (the
// general kernel takes it), else a hipError_t.
int conv_fwd(const ConvGeom &g, const void *x, const void *w, const void *bias, void *y, void *ws, hipStream_t st) {
    if (!geom_ok(g)) return -1;
    Args a{};
    a.a = (const float *)x; a.b = (const float *)w; a.g = g;
    a.M = g.N * g.P * g.Q; a.N = g.K; a.K = g.R * g.S * g.C;
    if (a.M == 0 || a.N == 0) return 0;
    Plan p = fwd_plan(g);
    if (few::fwd_us(g, x) < p.us) return few::conv_fwd(g, x, w, bias, y, st);
    if (p.splits > 1 && (!ws || !al16(ws))) p.splits = 1;
    return run<kFwd>(p, g.C % 4 == 0 && al16(x) && al16(w), a, 1, y_elems(g), (const float *)bias, (float *)y, ws, st);
}

int conv_dgrad(const ConvGeom &g, const void *dy, const void *w, const void *bias, void *dx, void *ws, hipStream_t st) {
    if (!geom_ok(g)) return -1;
    Args a{};
    a.a = (const float *)dy; a.b = (const float *)w; a.g = g;
    const int Hb = (g.H + g.sh - 1) / g.sh, Wb = (g.W + g.sw - 1) / g.sw;
    a.M = g.N * Hb * Wb; a.N = g.C;
    a.K = ((g.R + g.sh - 1) / g.sh) * ((g.S + g.sw - 1) / g.sw) * g.K;
    if (a.M == 0 || a.N == 0) return 0;
    Plan p = dgrad_plan(g);
    if (few::dgrad_us(g, dy) < p.us) return few::conv_dgrad(g, dy, w, bias, dx, st);
    if (p.splits > 1 && (!ws || !al16(ws))) p.splits = 1;
    return run<kDgrad>(p, g.K % 4 == 0 && g.C % 4 == 0 && al16(dy) && al16(w), a, g.sh * g.sw, x_elems(g),
                       (const float *)bias, (float *)dx, ws, st);
}

// `cap`: the bytes of workspace the caller sized for the partials
int conv_wgrad(const ConvGeom &g, const void *dy, const void *x, void *dw, void *ws, size_t cap, hipStream_t st) {
    if (!geom_ok(g)) return -1;
    Args a{};
    a.a = (const float *)dy; a.b = (const float *)x; a.g = g;
    a.M = g.K; a.N = g.R * g.S * g.C; a.K = g.N * g.P * g.Q;
    if (a.M == 0 || a.N == 0) return 0;
    const int rows = few_rows(g, cap);
    if (rows && ws && al16(ws)) {
        const int err = few::wgrad_parts(g, dy, x, static_cast<float *>(ws), part_stride(w_elems(g)), rows, st);
        return err ? err : reduce(static_cast<const float *>(ws), rows, w_elems(g), nullptr, 1, (float *)dw, st);
    }
    const Plan p = wgrad_plan(g, (int64_t)cap);
    if (p.splits > 1 && (!ws || !al16(ws))) return (int)hipErrorInvalidValue;
    return run<kWgrad>(p, g.K % 4 == 0 && g.C % 4 == 0 && al16(dy) && al16(x), a, 1, w_elems(g), nullptr, (float *)dw, ws, st);
}

// What a pass (0 forward, 1 input gradient, 2 weight gradient) lays out: out =
// {splits, bytes of their partials, blocks along grid z, whether the few-channel
// kernels take it}; -1: it is not taken.
int plan_info(int pass, const ConvGeom &g, size_t cap, int64_t out[4]) {
    if (!geom_ok(g)) return -1;
    const int z = pass == kDgrad ? g.sh * g.sw : 1;
    const int64_t elems = pass == kFwd ? y_elems(g) : pass == kDgrad ? x_elems(g) : w_elems(g);
    const Plan p = pass == kFwd ? fwd_plan(g) : pass == kDgrad ? dgrad_plan(g) : wgrad_plan(g, (int64_t)cap);
    out[0] = p.splits;
    out[1] = (int64_t)part_bytes(p, elems);
    out[2] = (int64_t)z * p.splits;
    out[3] = 0;
    const int rows = pass == kWgrad && elems > 0 ? few_rows(g, cap) : 0;
    const double us = pass == kFwd ? few::fwd_us(g, nullptr) : pass == kDgrad ? few::dgrad_us(g, nullptr) : HUGE_VAL;
    if (rows || us < p.us) {
        out[0] = std::max(rows, 1);
        out[1] = rows * part_stride(elems) * 4;
        out[2] = z;
        out[3] = 1;
    }
    return 0;
}

}  // namespace f32g
}  // namespace ms
