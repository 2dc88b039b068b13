// fp32 convolutions with few output channels (the forward of a layer with at
// most 16 filters, the input gradient of one with at most 16 input channels)
// and the weight gradient of a 3 x 3 layer with at most 16 of each, on
// v_mfma_f32_4x4x1_16b_f32: sixteen independent 4 x 4 outer products at the
// full fp32 matrix rate.  A GEMM tile 32 columns wide wastes 4x of its work on
// 8 channels; here the unit is 4.
//
// Forward and input gradient.  A block computes a tile of output pixels; its
// input neighbourhood, 4 (or all of 1 to 3) channels at a time, comes into
// LDS once by LDS-DMA.  A lane is an output pixel column of kPx rows.  Its
// pixels' channels are the second operand, as they lie; four output channels'
// weights are the first, the same for all sixteen blocks; the lane ends with
// four adjacent output channels of its own pixels and stores 16 bytes.  With
// RT > 0 taps along the height (unit vertical step) each input row of the strip
// is read once for all of them.
//
// Weight gradient.  A wave owns 16 adjacent pixels of one row after another;
// lane (pixel b, channel j) holds channel j of x and of dy, and each
// instruction adds sixteen pixels' 4 x 4 products of four filters and four
// input channels at one tap.  The sixteen sums meet at the end.
//
// The 4x4x1 instruction issues every 16 cycles, not the 8 it occupies the matrix
// core (timed without loads: 75 us for 9216 a SIMD), so 8 x 8 channels are bound
// by it (62 us) next to HBM (54 us at the rate of a large copy).
//
// Measured, us (kernel, warm; forward / input gradient / weight gradient),
// against the GEMM tiles of gemm_f32.hip:
//   3x3 8 -> 8, 64 x 256^2         310 / 375 / 428  ->  79 /  83 / 103
//   3x3 16 -> 16, 32 x 128^2        63 /  72 / 113  ->  43 /  45 /  57
//   7x7/2 3 -> 64, 16 x 224^2, dx        663        ->      129
#include <algorithm>
#include <cmath>

#include "common.h"
#include "lds_dma.h"
#include "limits.h"
#include "../device.h"

namespace ms {
namespace few {

using g2::kOOB;

constexpr int kPx = 4;               // output rows per lane
constexpr int kFlush = 256;          // products an accumulator runs over
constexpr int kBufBytes = 20 << 10;  // an input buffer at most
constexpr int kCUs = 256;
// Lanes of a launch, and pixels of a weight gradient, below which the GEMM is left
// alone: it splits its reduction over CUs that these kernels leave idle.  3x3, us,
// GEMM / here:
//   lanes        8192         16384        32768        65536
//   8 -> 8       7.4 / 8.6    9.8 / 9.0    14.8 / 9.6   25.4 / 11.1
//   3 -> 16      7.8 / 8.5    10.0 / 9.4   15.5 / 11.3  25.2 / 15.2
// (with three input channels or one tap they win by up to a third at any size).
// Above it the estimates decide (fwd_us(), and the GEMM's est_us()).  The weight
// gradient, with its sums' reduction:
//   pixels       32768        65536        131072       262144
//   4 -> 4       11.0 / 9.6   15.0 / 9.6   20.1 / 10.4  31.4 / 10.9
//   8 -> 8       12.6 / 13.7  16.8 / 14.8  23.0 / 15.8  36.8 / 17.2
//   16 -> 16     16.7 / 21.3  23.2 / 23.9  36.2 / 27.3  62.9 / 38.4
constexpr int64_t kMinUnits = 16384, kMinPixels = 65536;

struct Args {
    const float *in, *w, *bias;
    float *out;
    uint32_t in_bytes, out_bytes;
    ConvGeom g;
    int cin, cout;       // reduction and output channels
    int ih, iw;          // input extent
    int tw, rows;        // a tile: tw columns, `rows` strips of kPx rows
    int wfloats, bfloats;   // LDS: the weights, then two buffers
};

// One stride phase of the input gradient, or the forward: output pixel (i, j)
// of an oh x ow grid reads input (i * si + dh + t, j * sj + dw + s) for tap
// (t, s) of tr x ts, and is element ((n * OH + h0 + i * sh) * OW + w0 + j * sw).
struct View {
    int oh, ow, si, sj, dh, dw, tr, ts;
    int OH, OW, h0, w0, sh, sw;
    int fh, fw;          // input gradient: first filter tap of the phase
};

template <bool DG>
__host__ __device__ __forceinline__ View view_of(const ConvGeom &g, int z) {
    View v;
    if (!DG) {
        v.oh = v.OH = g.P;
        v.ow = v.OW = g.Q;
        v.si = g.sh;
        v.sj = g.sw;
        v.dh = -g.ph;
        v.dw = -g.pw;
        v.tr = g.R;
        v.ts = g.S;
        v.h0 = v.w0 = v.fh = v.fw = 0;
        v.sh = v.sw = 1;
        return v;
    }
    v.fh = z / g.sw;
    v.fw = z % g.sw;
    v.h0 = ((v.fh - g.ph) % g.sh + g.sh) % g.sh;
    v.w0 = ((v.fw - g.pw) % g.sw + g.sw) % g.sw;
    v.oh = v.h0 < g.H ? (g.H - v.h0 + g.sh - 1) / g.sh : 0;
    v.ow = v.w0 < g.W ? (g.W - v.w0 + g.sw - 1) / g.sw : 0;
    v.tr = v.fh < g.R ? (g.R - v.fh + g.sh - 1) / g.sh : 0;
    v.ts = v.fw < g.S ? (g.S - v.fw + g.sw - 1) / g.sw : 0;
    // dy row i + delta - tap, taps counted from the last: t = tr - 1 - tap
    v.dh = (v.h0 + g.ph - v.fh) / g.sh - (v.tr - 1);
    v.dw = (v.w0 + g.pw - v.fw) / g.sw - (v.ts - 1);
    v.si = v.sj = 1;
    v.OH = g.H;
    v.OW = g.W;
    v.sh = g.sh;
    v.sw = g.sw;
    return v;
}

template <int N> struct Const { static constexpr int value = N; };
template <int CV> struct Vec { float e[CV]; };

// CV channels of the reduction per chunk (4, or all 1 to 3), KG groups of four
// output channels, RT taps along the height held in registers (0: any number,
// or a vertical step above 1).
//
// A block walks a range of tiles; (tile, chunk) steps alternate between two
// LDS buffers, so one step's loads fly during the products of the step before.
// A tile's stores have a fixed count and stay in flight past the next step's
// wait.
//
// LONG: sums of more than kFlush products.  An accumulator that has run over
// kFlush of them is added to a second one and starts again, as in gemm_f32.hip: a
// sum's rounding error grows with its longest chain (2304 equal products that a
// large partial sum always rounds down: 3.4e-5 of the sum as one chain, at most
// 8.4e-6 so).
template <bool DG, int CV, int KG, int RT, bool LONG>
__global__ __launch_bounds__(256) void conv_kernel(const Args P) {
    // weights [tap][c / CV][kg][4 output channels][4], the last index CV used;
    // then two input buffers [row][column][CV]
    extern __shared__ __attribute__((aligned(1024))) float lds[];
    const ConvGeom &g = P.g;
    const View v = view_of<DG>(g, (int)blockIdx.y);
    const int tiles_w = (v.ow + P.tw - 1) / P.tw, tiles_h = (v.oh + P.rows * kPx - 1) / (P.rows * kPx);
    const int64_t tiles = (int64_t)g.N * tiles_h * tiles_w;
    const int64_t blk = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const int t0 = (int)(tiles * blk / gridDim.x), t1 = (int)(tiles * (blk + 1) / gridDim.x);
    if (t0 >= t1) return;   // uniform, nothing in flight

    const int cvn = P.cin / CV, taps = v.tr * v.ts;
    for (int i = threadIdx.x; i < taps * cvn * KG * 16; i += 256) {
        const int e = i & 3, o = (i >> 2) & 3, r0 = i >> 4;
        const int kg = r0 % KG, r1 = r0 / KG, cv = r1 % cvn, tap = r1 / cvn;
        const int t = tap / v.ts, s = tap - t * v.ts, ch = cv * CV + e, oc = kg * 4 + o;
        float x = 0.f;
        if (e < CV && oc < P.cout) {
            if constexpr (DG) {
                const int r = v.fh + (v.tr - 1 - t) * g.sh, q = v.fw + (v.ts - 1 - s) * g.sw;
                x = P.w[((size_t)(ch * g.R + r) * g.S + q) * g.C + oc];
            } else {
                x = P.w[((size_t)(oc * g.R + t) * g.S + s) * g.C + ch];
            }
        }
        lds[i] = x;
    }

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *const xl = lds + P.wfloats;
    const __amdgpu_buffer_rsrc_t rin = g2::rsrc(P.in, P.in_bytes);
    const __amdgpu_buffer_rsrc_t rout = g2::rsrc(P.out, P.out_bytes);
    // a tile's neighbourhood: hr rows of hc columns
    const int hr = (P.rows * kPx - 1) * v.si + v.tr, hc = (P.tw - 1) * v.sj + v.ts;
    constexpr int U = CV == 4 ? 4 : 1;          // floats per DMA lane
    const int per_row = hc * CV / U, units = hr * per_row;
    // reciprocal of per_row (0 when it is 1 or 0): exact for units, per_row < 2^14
    const uint32_t inv_row = per_row > 1 ? 0xFFFFFFFFu / (uint32_t)per_row + 1u : 0u;
    auto issue = [&](int buf, int tile, int cv) __attribute__((always_inline)) {
        const int tx = tile % tiles_w, t2 = tile / tiles_w, ty = t2 % tiles_h, n = t2 / tiles_h;
        const int y0 = ty * P.rows * kPx * v.si + v.dh, x0 = tx * P.tw * v.sj + v.dw;
        float *dst = xl + buf * P.bfloats;
        for (int b = wave * 64; b < units; b += 256) {
            const int e = b + lane;
            const int r = per_row > 1 ? (int)__umulhi((uint32_t)e, inv_row) : e, f = (e - r * per_row) * U;
            const int x = f / CV, c = f - x * CV;
            const int y = y0 + r, xx = x0 + x;
            const bool in = e < units && (unsigned)y < (unsigned)P.ih && (unsigned)xx < (unsigned)P.iw;
            const uint32_t off = in ? (uint32_t)(((n * P.ih + y) * P.iw + xx) * P.cin + cv * CV + c) * 4u : kOOB;
            if constexpr (CV == 4) g2::dma16<true>(rin, reinterpret_cast<char *>(dst + b * U), off);
            else g2::dma4s(rin, reinterpret_cast<char *>(dst + b * U), off, 0);
        }
    };

    // this lane's column and strip of a tile; lanes past them stay, each
    // supplies its block's weights
    const int col = (int)threadIdx.x % P.tw, strip = (int)threadIdx.x / P.tw;
    const int xoff = strip < P.rows ? (strip * kPx * v.si * hc + col * v.sj) * CV : 0;
    const float *wlane = lds + (threadIdx.x & 3) * 4;   // this lane's output channel of each group
    floatx4 bias[KG];
#pragma unroll
    for (int k = 0; k < KG; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[k][e] = P.bias && k * 4 + e < P.cout ? P.bias[k * 4 + e] : 0.f;
    // whole output vectors: one 16-byte store per pixel and group, masked lanes
    // sent past the output
    const bool vec = (P.cout & 3) == 0 && (reinterpret_cast<uintptr_t>(P.out) & 15u) == 0;

    floatx4 acc[kPx][KG], sum[LONG ? kPx : 1][LONG ? KG : 1];
    // the pixels' products of one tap, every accumulator once before any twice
    // (a chain on one accumulator waits for the result each time)
    auto fma = [&](const Vec<CV> *x, const floatx4 (&a)[KG]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < CV; ++e)
#pragma unroll
            for (int px = 0; px < kPx; ++px)
#pragma unroll
                for (int k = 0; k < KG; ++k)
                    acc[px][k] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k][e], x[px].e[e], acc[px][k], 0, 0, 0);
    };
    auto weights = [&](int tap, int cv, floatx4 (&a)[KG]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < KG; ++k) a[k] = *reinterpret_cast<const floatx4 *>(wlane + ((tap * cvn + cv) * KG + k) * 16);
    };

    // after a column of filter taps: products since the last flush
    int run = 0;
    const int column = v.tr * CV;
    auto flush = [&]() __attribute__((always_inline)) {
        if constexpr (LONG) {
            run += column;
            if (run + column <= kFlush) return;
            run = 0;
#pragma unroll
            for (int px = 0; px < kPx; ++px)
#pragma unroll
                for (int k = 0; k < KG; ++k) {
                    sum[px][k] += acc[px][k];
                    acc[px][k] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
        }
    };

    int buf = 0, ltile = t0, lcv = 0;   // the step being loaded
    issue(0, t0, 0);
    for (int tile = t0; tile < t1; ++tile) {
#pragma unroll
        for (int px = 0; px < kPx; ++px)
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                acc[px][k] = floatx4{0.f, 0.f, 0.f, 0.f};
                if constexpr (LONG) sum[px][k] = acc[px][k];
            }
        run = 0;
        for (int cv = 0; cv < cvn; ++cv) {
            // this step's loads have landed (the stores of the tile before are
            // newer than they); the first wait covers the weights too
            if (cv == 0 && tile > t0 && vec) g2::wait_vmcnt<kPx * KG>();
            else g2::wait_vmcnt<0>();
            g2::wait_lgkm0();
            g2::block_sync<true>();
            if (++lcv == cvn) {
                lcv = 0;
                ++ltile;
            }
            if (ltile < t1) issue(buf ^ 1, ltile, lcv);
            const float *xlane = xl + buf * P.bfloats + xoff;
            buf ^= 1;
            auto pixel = [&](int row, int s) __attribute__((always_inline)) {   // row and column from the lane's first
                Vec<CV> x;
                const float *p = xlane + (row * hc + s) * CV;
                if constexpr (CV == 4) {
                    const floatx4 u = *reinterpret_cast<const floatx4 *>(p);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x.e[e] = u[e];
                } else {
#pragma unroll
                    for (int e = 0; e < CV; ++e) x.e[e] = p[e];
                }
                return x;
            };
            for (int s = 0; s < v.ts; ++s) {
                if constexpr (RT > 0) {
                    constexpr int NR = kPx + RT - 1;
                    Vec<CV> in[NR];
#pragma unroll
                    for (int i = 0; i < NR; ++i) in[i] = pixel(i, s);
#pragma unroll
                    for (int t = 0; t < RT; ++t) {
                        floatx4 a[KG];
                        weights(t * v.ts + s, cv, a);
                        fma(in + t, a);
                    }
                } else {
                    for (int t = 0; t < v.tr; ++t) {
                        Vec<CV> in[kPx];
#pragma unroll
                        for (int px = 0; px < kPx; ++px) in[px] = pixel(px * v.si + t, s);
                        floatx4 a[KG];
                        weights(t * v.ts + s, cv, a);
                        fma(in, a);
                    }
                }
                flush();
            }
        }
        const int tx = tile % tiles_w, t2 = tile / tiles_w, ty = t2 % tiles_h, n = t2 / tiles_h;
        const int j = tx * P.tw + col, i0 = (ty * P.rows + strip) * kPx;
        const bool live = strip < P.rows && j < v.ow;
#pragma unroll
        for (int px = 0; px < kPx; ++px) {
            const bool ok = live && i0 + px < v.oh;
            const uint32_t off = (uint32_t)(((n * v.OH + v.h0 + (i0 + px) * v.sh) * v.OW + v.w0 + j * v.sw) * P.cout) * 4u;
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                floatx4 r = acc[px][k];
                if constexpr (LONG) r += sum[px][k];
                r += bias[k];
                u32x4 u;
#pragma unroll
                for (int e = 0; e < 4; ++e) u[e] = __float_as_uint(r[e]);
                if (vec) {
                    const uint32_t o = ok && k * 4 < P.cout ? off + k * 16u : kOOB;
                    __builtin_amdgcn_raw_buffer_store_b128(u, rout, (int)o, 0, 0);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t o = ok && k * 4 + e < P.cout ? off + k * 16u + e * 4u : kOOB;
                        __builtin_amdgcn_raw_buffer_store_b32(u[e], rout, (int)o, 0, 0);
                    }
                }
            }
        }
    }
}

// ------------------------------------------------------------ weight gradient
struct WArgs {
    const float *dy, *x;
    float *part;         // a row of K * 9 * C sums per block of grid x
    int64_t stride;      // floats between rows
    uint32_t dy_bytes, x_bytes;
    ConvGeom g;
};

// Rows prefetched together: their loads fly during the products of the batch
// before (36 a row for 8 x 8 channels).  Four rows spilled.
constexpr int kRows = 3;

// 3 x 3, stride 1.  Grid x: ranges of (image, 16-pixel strip, row) steps; grid
// y: blocks of 4 KG filters x 4 CG input channels.
template <int KG, int CG>
__global__ __launch_bounds__(256, 2) void wgrad_kernel(const WArgs P) {
    __shared__ float red[16][KG * 4 * 9 * CG * 4];
    const ConvGeom &g = P.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ncg = (g.C + 4 * CG - 1) / (4 * CG);
    const int k0 = ((int)blockIdx.y / ncg) * 4 * KG, c0 = ((int)blockIdx.y % ncg) * 4 * CG;
    const int pb = lane >> 2, ch = lane & 3;
    const __amdgpu_buffer_rsrc_t rd = g2::rsrc(P.dy, P.dy_bytes), rx = g2::rsrc(P.x, P.x_bytes);
    const int strips = (g.Q + 15) / 16;
    const int64_t steps = (int64_t)g.N * strips * g.P, waves = (int64_t)gridDim.x * 4;
    const int64_t w = (int64_t)xcd_remap((int)blockIdx.x, (int)gridDim.x) * 4 + wave;
    int64_t t = steps * w / waves;
    const int64_t t1 = steps * (w + 1) / waves;

    floatx4 acc[KG][3][3][CG];
#pragma unroll
    for (int k = 0; k < KG; ++k)
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int c = 0; c < CG; ++c) acc[k][r][s][c] = floatx4{0.f, 0.f, 0.f, 0.f};

    while (t < t1) {   // one strip's rows [p, p1)
        const int64_t sidx = t / g.P;
        int p = (int)(t - sidx * g.P);
        const int p1 = (int)min((int64_t)g.P, p + (t1 - t));
        const int n = (int)(sidx / strips), q = (int)(sidx % strips) * 16 + pb;
        t += p1 - p;
        // per-lane byte offsets of row 0 (x: per shift), and whether they are read at all
        uint32_t xo[3][CG], dyo[KG];
        bool xin[3][CG], din[KG];
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                const int xx = q - g.pw + s, cc = c0 + 4 * c + ch;
                xin[s][c] = q < g.Q && (unsigned)xx < (unsigned)g.W && cc < g.C;
                xo[s][c] = (uint32_t)((n * g.H * g.W + xx) * g.C + cc) * 4u;
            }
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const int kk = k0 + 4 * k + ch;
            din[k] = q < g.Q && kk < g.K;
            dyo[k] = (uint32_t)((n * g.P * g.Q + q) * g.K + kk) * 4u;
        }
        const uint32_t xrow = (uint32_t)(g.W * g.C) * 4u, drow = (uint32_t)(g.Q * g.K) * 4u;
        auto load_x = [&](int y, float (&v)[3][CG]) __attribute__((always_inline)) {
            const bool in = (unsigned)y < (unsigned)g.H;
            const uint32_t ro = (uint32_t)y * xrow;
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int c = 0; c < CG; ++c) {
                    const uint32_t off = in && xin[s][c] ? xo[s][c] + ro : kOOB;
                    v[s][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)off, 0, 0));
                }
        };
        auto load_dy = [&](int y, float (&v)[KG]) __attribute__((always_inline)) {
            const bool in = y < p1;
            const uint32_t ro = (uint32_t)y * drow;
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                const uint32_t off = in && din[k] ? dyo[k] + ro : kOOB;
                v[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rd, (int)off, 0, 0));
            }
        };
        // x rows p - ph ..: two carried, then kRows per batch, in two buffers that
        // trade places (a copy would wait for the loads)
        float xc[2][3][CG], xa[kRows][3][CG], da[kRows][KG], xb[kRows][3][CG], db[kRows][KG];
        auto load_batch = [&](int y, float (&xv)[kRows][3][CG], float (&dv)[kRows][KG]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                load_x(y < p1 ? y - g.ph + 2 + i : -1, xv[i]);
                load_dy(y + i, dv[i]);
            }
        };
        auto add_batch = [&](const float (&xv)[kRows][3][CG], const float (&dv)[kRows][KG]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                // no product of a row past the end: its zero dy would turn an
                // infinity of x, which the next range reads, into a NaN
                if (i > 0 && p + i >= p1) break;
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int s = 0; s < 3; ++s)
#pragma unroll
                        for (int c = 0; c < CG; ++c) {
                            const float x = i + r < 2 ? xc[i + r][s][c] : xv[i + r - 2][s][c];
#pragma unroll
                            for (int k = 0; k < KG; ++k)
                                acc[k][r][s][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(dv[i][k], x, acc[k][r][s][c], 0, 0, 0);
                        }
            }
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int c = 0; c < CG; ++c) {
                    xc[0][s][c] = xv[kRows - 2][s][c];
                    xc[1][s][c] = xv[kRows - 1][s][c];
                }
            p += kRows;
        };
        load_x(p - g.ph, xc[0]);
        load_x(p - g.ph + 1, xc[1]);
        load_batch(p, xa, da);
        while (p < p1) {
            load_batch(p + kRows, xb, db);
            add_batch(xa, da);
            if (p >= p1) break;
            load_batch(p + kRows, xa, da);
            add_batch(xb, db);
        }
    }

    // The sixteen pixel classes: four lanes apart within each row of 16 lanes by
    // rotations, then the block's sixteen rows in LDS, in a fixed order.
    auto ror = [](float x, auto n) __attribute__((always_inline)) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + decltype(n)::value, 0xf, 0xf, true));
    };
    const int row = wave * 4 + (lane >> 4);
#pragma unroll
    for (int k = 0; k < KG; ++k)
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int c = 0; c < CG; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float a = acc[k][r][s][c][i];
                        a += ror(a, Const<4>{});
                        a += ror(a, Const<8>{});
                        if ((lane & 15) < 4) red[row][(((k * 4 + i) * 3 + r) * 3 + s) * CG * 4 + c * 4 + ch] = a;
                    }
    __syncthreads();
    float *part = P.part + (size_t)blockIdx.x * P.stride;
    for (int i = threadIdx.x; i < KG * 4 * 9 * CG * 4; i += 256) {
        const int c = i % (CG * 4), rs = i / (CG * 4) % 9, k = i / (CG * 4) / 9;
        float a = 0.f;
#pragma unroll
        for (int w4 = 0; w4 < 16; ++w4) a += red[w4][i];
        if (k0 + k < g.K && c0 + c < g.C) part[((size_t)(k0 + k) * 9 + rs) * g.C + c0 + c] = a;
    }
}

// ------------------------------------------------------------------ host
namespace {

// groups of four output channels a launch computes (three run as four)
int groups(int cout) { return cout <= 4 ? 1 : cout <= 8 ? 2 : 4; }

bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// A launch's tiles: the width split into the fewest column tiles of at most 64,
// then as many strips of kPx rows as 256 lanes, the output and kBufBytes hold, fewer while the tiles would leave CUs without a block.
struct Tiling {
    int cv, tw, rows;
    double us;      // estimated time of the launch
    int64_t products;   // of a sum, at most
    int64_t tiles, wfloats, bfloats;   // tiles of a phase (bound); floats of weights and of a buffer
    bool rt3;
    int64_t lds_bytes() const { return (wfloats + 2 * bfloats) * 4; }
};

template <bool DG>
bool tiling(const ConvGeom &g, Tiling *out) {
    const int cin = DG ? g.K : g.C, cout = DG ? g.C : g.K;
    if (cout < 1 || cout > 16 || cin < 1 || (cin % 4 != 0 && cin > 3)) return false;
    Tiling t;
    t.cv = cin % 4 == 0 ? 4 : cin;
    const int oh = DG ? (g.H + g.sh - 1) / g.sh : g.P, ow = DG ? (g.W + g.sw - 1) / g.sw : g.Q;
    const int tr = DG ? (g.R + g.sh - 1) / g.sh : g.R, ts = DG ? (g.S + g.sw - 1) / g.sw : g.S;
    const int si = DG ? 1 : g.sh, sj = DG ? 1 : g.sw, phases = DG ? g.sh * g.sw : 1;
    if (oh < 1 || ow < 1 || tr > 16 || ts > 16 || si > 4 || sj > 4 || phases > 65535) return false;
    t.rt3 = g.sh == 1 && g.R == 3;
    t.products = (int64_t)tr * ts * cin;
    t.wfloats = ((int64_t)tr * ts * (cin / t.cv) * groups(cout) * 16 + 255) / 256 * 256;
    const int tiles_w = (ow + 63) / 64;
    t.tw = (ow + tiles_w - 1) / tiles_w;
    const int strips = (oh + kPx - 1) / kPx;
    const int64_t hc = (int64_t)(t.tw - 1) * sj + ts;
    auto buf_bytes = [&](int rows) { return (((int64_t)(rows * kPx - 1) * si + tr) * hc * t.cv * 4 + 1023) / 1024 * 1024; };
    t.rows = std::min(256 / t.tw, strips);
    while (t.rows > 1 && buf_bytes(t.rows) > kBufBytes) --t.rows;
    while (t.rows > 1 && (int64_t)g.N * phases * tiles_w * ((strips + t.rows - 1) / t.rows) < kCUs) --t.rows;
    t.tiles = (int64_t)g.N * tiles_w * ((strips + t.rows - 1) / t.rows);
    t.bfloats = buf_bytes(t.rows) / 4;
    if (buf_bytes(t.rows) > kBufBytes || t.lds_bytes() > 64 << 10 || t.tiles * 256 > UINT32_MAX) return false;
    const int64_t pixels = (int64_t)g.N * oh * ow * phases;
    if ((int64_t)g.N * strips * ow * phases < kMinUnits) return false;
    // The launch in us.  A tile takes its 4x4x1 products at 16 clocks each on
    // every wave, whichever of its lanes have work (two thirds of that with tiles
    // enough for several blocks a CU), or its loads: 16-byte pieces of pixels 4 C
    // bytes apart, 700 a us and CU out of the caches, 260 where the input is past
    // them and every chunk of channels fetches its lines again; pieces that share
    // lines come cheaper.  Over a tile's chunks 0.3 us of latency each; over the
    // launch, the bytes.  Over some 300 launches measured (1x1, 3x3 and 7x7, 2 to
    // 256 channels, images of 1 to 224 pixels a side, both ways) the smaller of
    // this estimate and the GEMM's names the faster kernel to within 10%, but for
    // 1x1 on 14 x 14 with 16 channels (29 us here, 24 there).  A Linear, images of
    // one pixel, is never it: 16384 x 768 -> 10 takes 4500 us here, 18 there.
    const int cvn = cin / t.cv, kg = groups(cout);
    const double rounds = (double)((t.tiles * phases + kCUs - 1) / kCUs);
    const double products = tr * ts * (double)cin * kPx * kg * 16 / 2400 * (rounds > 3 ? 0.7 : 1.0);
    const double bytes_in = 4.0 * g.N * (DG ? (double)g.P * g.Q : (double)g.H * g.W) * cin;
    const double loads = (double)((t.rows * kPx - 1) * si + tr) * hc * cvn / (bytes_in > 96e6 ? 260 : 700) * std::min(1.0, cin / 16.0);
    t.us = 4 + 0.3 * cvn + std::max(rounds * std::max(products, loads), (bytes_in + 4.0 * pixels * cout) / 4.5e6);
    *out = t;
    return true;
}

template <bool DG, int CV, int KG>
int go_rt(const Args &a, const Tiling &t, dim3 grid, hipStream_t st) {
    const unsigned pk = DG ? kProfDgrad : kProfFwd;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), (size_t)t.lds_bytes(), st, a); };
    prof_mark(pk, st, true);
    if (t.rt3) t.products > kFlush ? go(conv_kernel<DG, CV, KG, 3, true>) : go(conv_kernel<DG, CV, KG, 3, false>);
    else t.products > kFlush ? go(conv_kernel<DG, CV, KG, 0, true>) : go(conv_kernel<DG, CV, KG, 0, false>);
    const int err = (int)hipGetLastError();
    prof_mark(pk, st, false);
    return err;
}

template <bool DG, int CV>
int go_kg(const Args &a, const Tiling &t, dim3 grid, hipStream_t st) {
    switch (groups(a.cout)) {
    case 1: return go_rt<DG, CV, 1>(a, t, grid, st);
    case 2: return go_rt<DG, CV, 2>(a, t, grid, st);
    default: return go_rt<DG, CV, 4>(a, t, grid, st);
    }
}

template <bool DG>
int run(const ConvGeom &g, const void *in, const void *w, const void *bias, void *out, hipStream_t st) {
    Tiling t;
    if (!tiling<DG>(g, &t)) return (int)hipErrorInvalidValue;
    Args a{};
    a.in = (const float *)in; a.w = (const float *)w; a.bias = (const float *)bias; a.out = (float *)out; a.g = g;
    a.cin = DG ? g.K : g.C;
    a.cout = DG ? g.C : g.K;
    a.ih = DG ? g.P : g.H;
    a.iw = DG ? g.Q : g.W;
    a.in_bytes = (uint32_t)((int64_t)g.N * a.ih * a.iw * a.cin * 4);
    a.out_bytes = (uint32_t)((int64_t)g.N * (DG ? g.H : g.P) * (DG ? g.W : g.Q) * a.cout * 4);
    a.tw = t.tw; a.rows = t.rows;
    a.wfloats = (int)t.wfloats;
    a.bfloats = (int)t.bfloats;
    // two tiles a block once there are 16 a CU: 84 against 92 us on 4096 tiles;
    // on 1024 it costs (47.5 against 42.9 us), and longer ranges cost on both
    const int64_t phases = DG ? g.sh * g.sw : 1, per = t.tiles * phases >= 16 * kCUs ? 2 : 1;
    const dim3 grid((unsigned)((t.tiles + per - 1) / per), (unsigned)phases);
    switch (t.cv) {
    case 1: return go_kg<DG, 1>(a, t, grid, st);
    case 2: return go_kg<DG, 2>(a, t, grid, st);
    case 3: return go_kg<DG, 3>(a, t, grid, st);
    default: return go_kg<DG, 4>(a, t, grid, st);
    }
}

}  // namespace

// Estimated us of the forward / input gradient of g (whose tensors the caller has
// found to fit 32-bit byte offsets); infinite where the kernels do not take it.
double fwd_us(const ConvGeom &g, const void *x) {
    Tiling t;
    return (g.C % 4 != 0 || al16(x)) && tiling<false>(g, &t) ? t.us : HUGE_VAL;
}
double dgrad_us(const ConvGeom &g, const void *dy) {
    Tiling t;
    return (g.K % 4 != 0 || al16(dy)) && tiling<true>(g, &t) ? t.us : HUGE_VAL;
}
// Whether the kernel takes the weight gradient.  Lanes past a row's end work for
// nothing, and the more the more groups of channels there are, so the share of a
// strip's 16 columns that are pixels is bounded below.  About 400,000 pixels, us,
// GEMM / here:
//   image     4 x 4          7 x 7         10 x 10       14 x 14
//   4 -> 4    42.9 / 30.8    42.5 / 19.0   42.6 / 15.4   42.3 / 12.2   (2 x 2: 29.4 / 45.6)
//   8 -> 8    49.6 / 55.4    49.7 / 32.9   50.1 / 25.9   50.1 / 19.6
//   16 -> 16  92.6 / 237     91.1 / 129    90.0 / 83.2   90.8 / 60.7
bool wgrad_applies(const ConvGeom &g) {
    if (g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1 || g.C < 1 || g.C > 16 || g.K < 1 || g.K > 16) return false;
    const int blocks = (g.K > 8 ? 2 : 1) * (g.C > 8 ? 2 : 1);
    const int groups = (g.K > 4 ? 2 : 1) * (g.C > 4 ? 2 : 1) * blocks;   // 1, 2, 4, 8 or 16
    const double share = g.Q / (16.0 * ((g.Q + 15) / 16));
    return share >= 0.2 + 0.1 * std::log2(groups) && (int64_t)g.N * g.P * g.Q >= kMinPixels * (groups > 4 ? 2 : 1);
}

int conv_fwd(const ConvGeom &g, const void *x, const void *w, const void *bias, void *y, hipStream_t st) {
    return run<false>(g, x, w, bias, y, st);
}
int conv_dgrad(const ConvGeom &g, const void *dy, const void *w, const void *bias, void *dx, hipStream_t st) {
    return run<true>(g, dy, w, bias, dx, st);
}

// n partial rows of K * 9 * C sums, `stride` floats apart, into `part`.
int wgrad_parts(const ConvGeom &g, const void *dy, const void *x, float *part, int64_t stride, int n, hipStream_t st) {
    WArgs a{};
    a.dy = (const float *)dy; a.x = (const float *)x; a.part = part; a.stride = stride; a.g = g;
    a.dy_bytes = (uint32_t)((int64_t)g.N * g.P * g.Q * g.K * 4);
    a.x_bytes = (uint32_t)((int64_t)g.N * g.H * g.W * g.C * 4);
    const int kg = g.K > 4 ? 2 : 1, cg = g.C > 4 ? 2 : 1;
    const dim3 grid((unsigned)n, (unsigned)(((g.K + 4 * kg - 1) / (4 * kg)) * ((g.C + 4 * cg - 1) / (4 * cg))));
    prof_mark(kProfWgrad, st, true);
    if (kg == 1 && cg == 1) hipLaunchKernelGGL((wgrad_kernel<1, 1>), grid, dim3(256), 0, st, a);
    else if (kg == 1) hipLaunchKernelGGL((wgrad_kernel<1, 2>), grid, dim3(256), 0, st, a);
    else if (cg == 1) hipLaunchKernelGGL((wgrad_kernel<2, 1>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((wgrad_kernel<2, 2>), grid, dim3(256), 0, st, a);
    const int err = (int)hipGetLastError();
    prof_mark(kProfWgrad, st, false);
    return err;
}

}  // namespace few
}  // namespace ms
