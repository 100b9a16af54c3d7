#include "sfc_kernels.hpp"

#include <algorithm>

#include "launch.hpp"
#include "sfc_device.hpp"

namespace canvas {
namespace sfc {

namespace {

using f4 = __attribute__((ext_vector_type(4))) float;
using f4u = __attribute__((ext_vector_type(4), aligned(4))) float;  // in memory, at any element

constexpr int kThreads = 256;
constexpr int kLinearKc = 32;   // channels per chunk without a window
constexpr int kMaxLds = 64 * 1024;

// Forward and data gradient.  A workgroup owns 16*WM outputs of one group and TP = 16*NT*(4/WM) consecutive pixels of the
// batch, a wavefront 16 outputs and 16*NT pixels; the contraction runs over chunks of KC channels with all their taps.  With the small tiles
// that fill the chip at these sizes it is bound by the latency of its steps: the matrix pipes (v_mfma_f32_16x16x4_f32: 32
// cycles for 2048 flops, 157 TFLOP/s on the chip) are busy a third of the time, three wavefronts per SIMD wait for data in
// a third of their cycles and for their turn to issue in two fifths (SQ counters at the size below).  The operand tile in LDS holds image rows with a
// zero margin, so a tap is a constant LDS offset and the Unfold costs no memory traffic and no mask; the next chunk's
// is loaded into registers while this one is multiplied.  The weights go from the caches straight to registers, where
// a lane finds its channel's taps side by side (36 bytes for 3 x 3, 16 for four channels without a window): staged
// through LDS they cost more vector instructions than the rest of the loop.
// Sums: the products of one or two taps (without a window: of 16 channels) are chained in the matrix unit, these parts
// are added per four channels, these to the result: the rounding errors of the chains stay below those of one sum per
// tap over all channels, whatever the number of channels (measured against fp64 over 16-128 channels: y 0.8-1.3e-7,
// dx 0.8-1.3e-7; one thread per element and one chain: 2.0-6.0e-7 and 0.9-2.1e-7).
// N=32, C=64, 28x28, 3x3 (1.85 GFLOP): 39 us forward, 35 us data gradient, 48-52 TFLOP/s; one thread per output element
// and a materialised Unfold took 563 + 29 us and 400 + 40 us.  All 16 outputs x 64 pixels of a wavefront on the same
// outputs (each weight loaded by four wavefronts) 58 and 38 us: a lane's 36 bytes lie a row apart, and the tag lookups
// of the first-level cache were the limit.
template <int WM, int NT, int TVT, bool WIN, int NP, int KC, bool TR>
__global__ __launch_bounds__(kThreads) void k_fwd(Params Q) {
    extern __shared__ float lds[];
    float* Bs = lds;  // [KC][CS]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, quad = lane >> 4;
    constexpr int TP = 16 * NT * (4 / WM);
    const int wm = wave % WM, wn = wave / WM;
    unsigned b = tile_of_block();
    if (b >= (unsigned)Q.tiles) return;
    const int mtile = (int)(b % (unsigned)Q.mtiles);
    b /= (unsigned)Q.mtiles;
    const int g = (int)(b % (unsigned)Q.G);
    const int64_t m0 = (int64_t)(b / (unsigned)Q.G) * TP;
    const int64_t n0 = m0 / Q.P;
    const int p0 = (int)(m0 - n0 * Q.P);
    const int h0 = WIN ? quotient(p0, Q.W, Q.mW) : 0;
    const int o0 = (mtile * WM + wm) * 16;
    const int64_t P = Q.P;

    // this thread's positions of the operand tile, in channel 0 of the group (a position of the margin reads the first
    // element instead and drops it)
    constexpr int kBRegs = WIN ? NP * KC : KC * TP / kThreads;
    constexpr int kChStep = kThreads / TP;  // without a window: channels one pass of the workgroup covers
    const float* src = Q.src + (int64_t)g * Q.R * P;
    const float* from[NP];
    bool inside[NP];
    const int c0 = WIN ? 0 : tid / TP, j0 = WIN ? tid : tid & (TP - 1);
    if (WIN) {
#pragma unroll
        for (int i = 0; i < NP; i++) {
            const int j = tid + i * kThreads;
            const int64_t at = j < Q.S ? window_source(Q, n0, h0, j) : -1;
            inside[i] = at >= 0;
            from[i] = src + (at >= 0 ? at : 0);
        }
    } else {
        const int p = p0 + j0, dn = image_of(Q, p);
        inside[0] = m0 + j0 < Q.M;
        from[0] = src + (inside[0] ? (n0 + dn) * Q.G * Q.R * P + (p - dn * Q.P) : 0);
    }
    // the pixels this lane multiplies
    int lofs[NT];
    int64_t dofs[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) {
        const int j = (wn * NT + t) * 16 + col;
        const bool in = m0 + j < Q.M;
        const int p = in ? p0 + j : p0;
        const int dn = image_of(Q, p), pp = p - dn * Q.P;
        if (WIN) {
            const int h = quotient(pp, Q.W, Q.mW);
            lofs[t] = (dn * Q.HP + h - h0) * Q.Wp + (pp - h * Q.W);
        } else {
            lofs[t] = in ? j : 0;
        }
        dofs[t] = in ? (n0 + dn) * Q.G * Q.Og * P + pp : -1;
    }

    float breg[kBRegs];
    auto load_b = [&](int r0) {
        if (WIN) {
#pragma unroll
            for (int c = 0; c < KC; c++) {
                const int64_t ch = min(r0 + c, Q.R - 1) * P;
#pragma unroll
                for (int i = 0; i < NP; i++) breg[c * NP + i] = from[i][ch];
            }
        } else {
#pragma unroll
            for (int c = 0; c < kBRegs; c++) breg[c] = from[0][min(r0 + c0 + c * kChStep, Q.R - 1) * P];
        }
    };
    auto store_b = [&](int r0) {  // (channels past the last are zero: they meet zero weights)
        if (WIN) {
#pragma unroll
            for (int i = 0; i < NP; i++) {
                const int j = tid + i * kThreads;
                if (j < Q.S) {
#pragma unroll
                    for (int c = 0; c < KC; c++) Bs[c * Q.CS + j] = inside[i] && r0 + c < Q.R ? breg[c * NP + i] : 0.f;
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < kBRegs; c++) {
                const int ch = c0 + c * kChStep;
                Bs[ch * Q.CS + j0] = inside[0] && r0 + ch < Q.R ? breg[c] : 0.f;
            }
        }
    };
    // this lane's weights: output `col` of the wavefront's 16 (the last one again past the end: not stored)
    const int tv = TVT ? TVT : Q.TV;
    const int64_t wch = TR ? (int64_t)Q.Og * tv : (TVT ? TVT : tv);  // elements between two channels
    const float* wrow = Q.w + (int64_t)g * Q.Og * Q.K + min(o0 + col, Q.Og - 1) * (int64_t)(TR ? tv : Q.K);
    constexpr int NA = TVT == 9 ? 9 : (TVT == 1 ? 4 : 1);  // weights of a step loaded ahead: nine taps of a channel, or four channels
    // 3 x 3: the taps of channel ch + quad.  No window: channels ch + 4*quad ... + 3.  Channels past the last are zero.
    auto load_w = [&](int ch, float (&a)[NA]) {
        if (TVT == 9) {
            const int c = ch + quad;
            const float* from = wrow + min(c, Q.R - 1) * wch;
#pragma unroll
            for (int t = 0; t < NA; t++) a[TR ? NA - 1 - t : t] = from[t];  // (transposed: the window read backwards)
            if (ch + 4 > Q.R)
#pragma unroll
                for (int t = 0; t < NA; t++) a[t] = c < Q.R ? a[t] : 0.f;
        } else if (TVT == 1) {
            const int c = ch + quad * 4;
            if (ch + 16 <= Q.R) {
#pragma unroll
                for (int t = 0; t < NA; t++) a[t] = wrow[(c + t) * wch];
            } else {
#pragma unroll
                for (int t = 0; t < NA; t++) {
                    a[t] = wrow[min(c + t, Q.R - 1) * wch];
                    a[t] = c + t < Q.R ? a[t] : 0.f;
                }
            }
        }
    };

    f4 acc[NT], sum[NT], part[NT];
    const f4 zero{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; t++) acc[t] = zero;
    // one matrix step (four products per output and pixel), the first of a part from zero
    auto mul = [&](bool first, float av, const float* b) {
        float bv[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) bv[t] = b[lofs[t]];
#pragma unroll
        for (int t = 0; t < NT; t++) part[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[t], first ? zero : part[t], 0, 0, 0);
    };
    auto add = [&](f4 (&to)[NT], const f4 (&v)[NT], bool first) {
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int r = 0; r < 4; r++) to[t][r] = first ? v[t][r] : to[t][r] + v[t][r];
    };

    constexpr int kStepCh = TVT == 1 ? 16 : 4, kSteps = KC / kStepCh;  // channels per step, steps per chunk
    float wreg[2][NA];
    load_w(0, wreg[0]);
    load_b(0);
    for (int r0 = 0; r0 < Q.R; r0 += KC) {
        store_b(r0);
        __syncthreads();
        const int steps = (min(KC, Q.R - r0) + kStepCh - 1) / kStepCh;
#pragma unroll
        for (int s = 0; s < kSteps; s++) {
            if (s >= steps) break;
            const float (&w)[NA] = wreg[kSteps == 1 ? 0 : s & 1];
            const int ch = r0 + s * kStepCh;
            if (kSteps > 1) load_w(min(ch + kStepCh, Q.R - 1), wreg[(s + 1) & 1]);  // (an even number of steps: a chunk begins with the first set)
            if (s == 0 && r0 + KC < Q.R) load_b(r0 + KC);
            if (TVT == 1) {
                const float* b = Bs + (s * 16 + quad * 4) * Q.CS;
#pragma unroll
                for (int t = 0; t < 4; t++) mul(t == 0, w[t < NA ? t : 0], b + t * Q.CS);
                add(acc, part, false);
            } else if (TVT == 9) {
                const float* b = Bs + (s * 4 + quad) * Q.CS;
#pragma unroll
                for (int tap = 0; tap < 9; tap++) {
                    mul(tap % 2 == 0, w[tap < NA ? tap : 0], b + tap / 3 * Q.Wp + tap % 3);
                    if (tap % 2 == 1 || tap == 8) add(sum, part, tap == 1);
                }
                add(acc, sum, false);
            } else {
                const float* b = Bs + (s * 4 + quad) * Q.CS;
                const int c = ch + quad;
                const float* from = wrow + min(c, Q.R - 1) * wch;
                for (int kh = 0; kh < Q.KH; kh++) {
                    float row[7];
#pragma unroll
                    for (int kw = 0; kw < 7; kw++) {
                        const int tap = kh * Q.KW + min(kw, Q.KW - 1);
                        row[kw] = from[TR ? tv - 1 - tap : tap];
                        row[kw] = c < Q.R ? row[kw] : 0.f;
                    }
#pragma unroll
                    for (int kw = 0; kw < 7; kw++) {
                        if (kw >= Q.KW) break;
                        mul(true, row[kw], b + kh * Q.Wp + kw);
                        add(sum, part, kh + kw == 0);
                    }
                }
                add(acc, sum, false);
            }
        }
        if (kSteps == 1 && r0 + KC < Q.R) load_w(r0 + KC, wreg[0]);
        __syncthreads();
    }
    // lane: pixel `col` of its 16, outputs 4*quad .. 4*quad + 3
    const int o = o0 + quad * 4, left = Q.Og - o;
#pragma unroll
    for (int t = 0; t < NT; t++) {
        if (dofs[t] < 0) continue;
        float* d = Q.dst + dofs[t] + ((int64_t)g * Q.Og + o) * P;
        float old[4] = {0.f, 0.f, 0.f, 0.f};
        if (Q.acc) {
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (r < left) old[r] = d[r * P];
        }
#pragma unroll
        for (int r = 0; r < 4; r++)
            if (r < left) d[r * P] = Q.acc ? old[r] + acc[t][r] : acc[t][r];
    }
}

constexpr int kNarrowPix = 4 * kThreads;  // pixels per step of the narrow weight gradient
constexpr int kPix = 64;        // pixels per step of the weight gradient
constexpr int kDyStride = 68;   // 4 mod 64: the 16 outputs x 4 pixels of an operand read lie in 64 banks

// Weight gradient: contraction over pixels.  A workgroup owns 16*MT*WM outputs x 16*NT*(4/WM) contraction indices of one
// group and one slice of the batch's pixels; 64 pixels of dy and of the channels behind those indices (image rows with a
// zero margin, as above) go through LDS.  A lane's column is one (channel, tap): its LDS base; the pixel's place in the
// tile comes from a table.  No padding beyond the tile's edges whatever R, Og and the window are.  Bound like k_fwd: the
// matrix pipes are busy a quarter of the time, two wavefronts per SIMD.
// Sums: chains of eight pixels in the matrix unit, added as a tree over the 64 pixels of a step, the steps in a row.
// N=32, C=64, 28x28, 3x3: 46 us (40 TFLOP/s) and 4 us for the sum of the slices; one workgroup per weight took 1259 us.
template <int MT, int NT, int WM, bool WIN>
__global__ __launch_bounds__(kThreads) void k_wgrad(Params Q) {
    constexpr int WN = 4 / WM, BM = 16 * MT * WM, BN = 16 * NT * WN;
    extern __shared__ float lds[];
    int64_t* sofs = reinterpret_cast<int64_t*>(lds);   // [2][S]: source of each position, -1 = zero; this step's and the next
    int* pofs = reinterpret_cast<int*>(sofs + 2 * Q.S);  // [kPix]: place of each pixel in the tile
    float* Dy = reinterpret_cast<float*>(pofs + kPix);  // [BM][kDyStride]
    float* Xs = Dy + BM * kDyStride;                   // [nch][CS]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, quad = lane >> 4;
    const int wm = wave % WM, wn = wave / WM;
    unsigned b = tile_of_block();
    if (b >= (unsigned)Q.tiles) return;
    const int mtile = (int)(b % (unsigned)Q.mtiles);
    b /= (unsigned)Q.mtiles;
    const int ktile = (int)(b % (unsigned)Q.ktiles);
    b /= (unsigned)Q.ktiles;
    const int g = (int)(b % (unsigned)Q.G);
    const int slice = (int)(b / (unsigned)Q.G);
    const int o0 = mtile * BM, k0 = ktile * BN;
    const int r0 = k0 / Q.TV, nch = min(Q.nch, Q.R - r0);
    const int64_t first = slice * Q.per_slice, last = min(Q.M, first + Q.per_slice);

    int kbase[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) {
        const int k = min(k0 + (wn * NT + t) * 16 + col, Q.K - 1);  // (columns past the last are not stored)
        const int r = k / Q.TV, tap = k - r * Q.TV, kh = tap / Q.KW;
        kbase[t] = (r - r0) * Q.CS + kh * Q.Wp + (tap - kh * Q.KW);
    }
    f4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
        for (int t = 0; t < NT; t++) acc[i][t] = f4{0.f, 0.f, 0.f, 0.f};

    const int rows = min(BM, Q.Og - o0);
    const float* xs = Q.src + ((int64_t)g * Q.R + r0) * Q.P;
    const float* ds = Q.dy + ((int64_t)g * Q.Og + o0) * Q.P;
    auto table = [&](int64_t n0, int p0, int count, int64_t* to) {
        const int h0 = WIN ? quotient(p0, Q.W, Q.mW) : 0;
        for (int j = tid; j < Q.S; j += kThreads) {
            if (WIN) {
                to[j] = window_source(Q, n0, h0, j);
            } else {
                const int p = p0 + j, dn = image_of(Q, p);
                to[j] = j < count ? (n0 + dn) * Q.G * Q.R * (int64_t)Q.P + (p - dn * Q.P) : -1;
            }
        }
    };
    // What a thread loads of a step in one go: dy of one pixel for BM/4 outputs, and the first kAhead of its x elements (a
    // wavefront takes every fourth channel, 64 positions at a time: pass k covers channel c = wave + 4*(k / npos)).
    // (Kept in flight across the multiplication of the step before, they cost a wavefront of occupancy and gained nothing.)
    constexpr int kRows = BM * kPix / kThreads, kAhead = 16;
    const int npos = (Q.S + 63) / 64, passes = (nch + 3 - __builtin_amdgcn_readfirstlane(wave)) / 4 * npos;
    float dreg[kRows], xreg[kAhead];
    auto load_dy = [&](int64_t n0, int p0, int count) {
        const int p = p0 + lane, dn = image_of(Q, p);
        const bool in = lane < count;
        const float* from = ds + (in ? (n0 + dn) * Q.G * Q.Og * (int64_t)Q.P + (p - dn * Q.P) : 0);
#pragma unroll
        for (int i = 0; i < kRows; i++) {
            const int m = i * 4 + wave;
            dreg[i] = from[min(m, rows - 1) * (int64_t)Q.P];
            dreg[i] = in && m < rows ? dreg[i] : 0.f;
        }
    };
    auto load_x = [&](int first_pass, const int64_t* table) {
        int c = __builtin_amdgcn_readfirstlane(wave) + first_pass / npos * 4, j = first_pass % npos;
#pragma unroll
        for (int i = 0; i < kAhead; i++) {
            const int64_t o = table[min(j * 64 + lane, Q.S - 1)];
            xreg[i] = xs[(o < 0 ? 0 : o) + (int64_t)min(c, nch - 1) * Q.P];
            xreg[i] = o < 0 ? 0.f : xreg[i];
            if (++j == npos) {
                j = 0;
                c += 4;
            }
        }
    };
    auto store_x = [&](int first_pass) {
        int c = __builtin_amdgcn_readfirstlane(wave) + first_pass / npos * 4, j = first_pass % npos;
#pragma unroll
        for (int i = 0; i < kAhead; i++) {
            if (first_pass + i < passes && j * 64 + lane < Q.S) Xs[c * Q.CS + j * 64 + lane] = xreg[i];
            if (++j == npos) {
                j = 0;
                c += 4;
            }
        }
    };
    int cur = 0;
    int64_t n0 = first / Q.P;
    int p0 = (int)(first - n0 * Q.P), count = (int)min((int64_t)kPix, last - first);
    table(n0, p0, count, sofs);
    __syncthreads();
    for (int64_t m0 = first; m0 < last; m0 += kPix, cur ^= 1) {
        load_dy(n0, p0, count);
        load_x(0, sofs + cur * Q.S);
        if (tid < kPix) {
            const int h0 = WIN ? quotient(p0, Q.W, Q.mW) : 0;
            const int p = tid < count ? p0 + tid : p0;
            const int dn = image_of(Q, p), pp = p - dn * Q.P, h = WIN ? quotient(pp, Q.W, Q.mW) : 0;
            pofs[tid] = WIN ? (dn * Q.HP + h - h0) * Q.Wp + (pp - h * Q.W) : (tid < count ? tid : 0);
        }
#pragma unroll
        for (int i = 0; i < kRows; i++) Dy[(i * 4 + wave) * kDyStride + lane] = dreg[i];
        store_x(0);
        for (int p = kAhead; p < passes; p += kAhead) {
            load_x(p, sofs + cur * Q.S);
            store_x(p);
        }
        const bool whole = count == kPix, more = m0 + kPix < last;
        const int here = count;
        if (more) {
            const int p = p0 + kPix, dn = image_of(Q, p);
            n0 += dn;
            p0 = p - dn * Q.P;
            count = (int)min((int64_t)kPix, last - m0 - kPix);
            table(n0, p0, count, sofs + (cur ^ 1) * Q.S);
        }
        __syncthreads();
        const float* a0 = Dy + (wm * 16 * MT + col) * kDyStride + quad;
        float av[MT][kPix / 4];
        int po[kPix / 4];
#pragma unroll
        for (int i = 0; i < MT; i++)
#pragma unroll
            for (int s = 0; s < kPix / 4; s++) av[i][s] = a0[i * 16 * kDyStride + s * 4];
#pragma unroll
        for (int s = 0; s < kPix / 4; s++) po[s] = pofs[s * 4 + quad];
#pragma unroll
        for (int t = 0; t < NT; t++) {
            f4 part[kPix / 8][MT];
#pragma unroll
            for (int s = 0; s < kPix / 4; s++) {
                float bv = Xs[kbase[t] + po[s]];
                if (!whole) bv = s * 4 + quad < here ? bv : 0.f;  // (a pixel past the slice meets dy = 0, and its x must not be an infinity)
#pragma unroll
                for (int i = 0; i < MT; i++)
                    part[s / 2][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][s], bv, s % 2 ? part[s / 2][i] : f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                // each finished part joins its neighbours as in a binary counter
#pragma unroll
                for (int w = 1; w < kPix / 8; w *= 2)
                    if (s % 2 == 1 && (s / 2) % (2 * w) == 2 * w - 1)
#pragma unroll
                        for (int i = 0; i < MT; i++)
#pragma unroll
                            for (int r = 0; r < 4; r++) part[s / 2 - (2 * w - 1)][i][r] += part[s / 2 - (w - 1)][i][r];
            }
#pragma unroll
            for (int i = 0; i < MT; i++)
#pragma unroll
                for (int r = 0; r < 4; r++) acc[i][t][r] += part[0][i][r];
            __builtin_amdgcn_sched_barrier(0);  // (the next column's parts would need another set of registers)
        }
        __syncthreads();
    }
    float* dw = Q.partial + (int64_t)slice * Q.G * Q.Og * Q.K + (int64_t)g * Q.Og * Q.K;
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
        for (int t = 0; t < NT; t++) {
            const int k = k0 + (wn * NT + t) * 16 + col;
            const int o = o0 + (wm * MT + i) * 16 + quad * 4;
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (k < Q.K && o + r < Q.Og) dw[(int64_t)(o + r) * Q.K + k] = acc[i][t][r];
        }
}

// Few rows and outputs per group (a depthwise or nearly depthwise contraction): a matrix tile would consist of padding, 16
// outputs and 4 to 32 channels of which one to four are there.  One thread per V pixels of a group and OT outputs on the
// vector unit, numbered through [N, G, P], so that a wavefront reads and writes whole lines also of planes smaller than
// itself; a window's taps are loads of their own, mostly from the first-level cache.  Bound by memory without a window, by
// the loads of the taps with one.
// Sums: chains of a window row's taps (without a window: of four channels), these parts added per channel, these to the result.
// N=64, 56x56, 64 channels, one per group: 17 us without a window (6.2 TB/s, x partly in the last-level cache), 102 us with
// 3 x 3, 275 us with 5 x 5; k_fwd takes 328, 415 and 970 us there.  Errors against fp64 are those of k_fwd or smaller
// (1 x 1 2.5-5.7e-8, 3 x 3 5.0-6.4e-8 against 5.5-6.9e-8).
template <int OT, int V, int TVT, bool TR>
__global__ __launch_bounds__(kThreads) void k_fwd_narrow(Params Q) {
    unsigned b = tile_of_block();
    if (b >= (unsigned)Q.tiles) return;
    const int o0 = (int)(b % (unsigned)Q.mtiles) * OT;
    const int64_t base = (int64_t)(b / (unsigned)Q.mtiles) * (kThreads * V);  // V divides P: a thread's pixels lie in one plane
    const int64_t P = Q.P, ng0 = base / P;
    int p = (int)(base - ng0 * P) + (int)threadIdx.x * V;
    const int dn = Q.P >= kThreads * V ? (p >= Q.P ? 1 : 0) : quotient(p, Q.P, Q.mP);
    p -= dn * Q.P;
    const int64_t ng = ng0 + dn;
    if (ng >= Q.N * Q.G) return;
    const int g = (int)(((uint32_t)(ng0 % Q.G) + (uint32_t)dn) % (uint32_t)Q.G);
    const float* src = Q.src + ng * Q.R * P;
    const int tv = TVT ? TVT : Q.TV;
    // element (output o0 + o, row r, tap t) of the weights; an output past the last reads the last one's and is not stored
    const float* w = Q.w + (int64_t)g * Q.Og * Q.K;
    int64_t wo[OT];
#pragma unroll
    for (int o = 0; o < OT; o++) wo[o] = (int64_t)min(o0 + o, Q.Og - 1) * (TR ? tv : Q.K);
    const int64_t wr = TR ? (int64_t)Q.Og * tv : tv;
    float acc[OT][V];
#pragma unroll
    for (int o = 0; o < OT; o++)
#pragma unroll
        for (int v = 0; v < V; v++) acc[o][v] = 0.f;
    if (TVT == 1) {
        for (int r0 = 0; r0 < Q.R; r0 += 4) {
            float part[OT][V];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int r = r0 + k;
                if (k > 0 && r >= Q.R) break;
                float x[V];
                if (V == 4) {
                    const f4u d = *reinterpret_cast<const f4u*>(src + r * P + p);
#pragma unroll
                    for (int v = 0; v < V; v++) x[v] = d[v];
                } else {
                    x[0] = src[r * P + p];
                }
#pragma unroll
                for (int o = 0; o < OT; o++) {
                    const float a = w[wo[o] + r * wr];
#pragma unroll
                    for (int v = 0; v < V; v++) part[o][v] = k == 0 ? a * x[v] : fmaf(a, x[v], part[o][v]);
                }
            }
#pragma unroll
            for (int o = 0; o < OT; o++)
#pragma unroll
                for (int v = 0; v < V; v++) acc[o][v] += part[o][v];
        }
    } else {
        int h[V], c[V];
#pragma unroll
        for (int v = 0; v < V; v++) {
            h[v] = quotient(p + v, Q.W, Q.mW);
            c[v] = p + v - h[v] * Q.W;
        }
        constexpr int KW = TVT == 9 ? 3 : 7;
        const int kh_n = TVT == 9 ? 3 : Q.KH, kw_n = TVT == 9 ? 3 : Q.KW;
        for (int r = 0; r < Q.R; r++) {
            float sum[OT][V];
#pragma unroll TVT == 9 ? 3 : 1
            for (int kh = 0; kh < kh_n; kh++) {
                float x[KW][V], part[OT][V];
#pragma unroll
                for (int kw = 0; kw < KW; kw++) {
                    if (kw >= kw_n) break;
#pragma unroll
                    for (int v = 0; v < V; v++) {
                        const int hh = h[v] + kh - kh_n / 2, cc = c[v] + kw - kw_n / 2;
                        const bool in = (unsigned)hh < (unsigned)Q.H && (unsigned)cc < (unsigned)Q.W;
                        x[kw][v] = src[r * P + (in ? hh * Q.W + cc : p)];
                        x[kw][v] = in ? x[kw][v] : 0.f;
                    }
                }
#pragma unroll
                for (int o = 0; o < OT; o++) {
#pragma unroll
                    for (int kw = 0; kw < KW; kw++) {
                        if (kw >= kw_n) break;
                        const int tap = kh * kw_n + kw;
                        const float a = w[wo[o] + r * wr + (TR ? tv - 1 - tap : tap)];  // (transposed: the window read backwards)
#pragma unroll
                        for (int v = 0; v < V; v++) part[o][v] = kw == 0 ? a * x[kw][v] : fmaf(a, x[kw][v], part[o][v]);
                    }
#pragma unroll
                    for (int v = 0; v < V; v++) sum[o][v] = kh == 0 ? part[o][v] : sum[o][v] + part[o][v];
                }
            }
#pragma unroll
            for (int o = 0; o < OT; o++)
#pragma unroll
                for (int v = 0; v < V; v++) acc[o][v] += sum[o][v];
        }
    }
    float* dst = Q.dst + (ng * Q.Og + o0) * P + p;
#pragma unroll
    for (int o = 0; o < OT; o++) {
        if (o0 + o >= Q.Og) break;
        float* d = dst + o * P;
        if (Q.acc) {
            asm volatile("");  // (keeps the compiler from reading dst also where nothing is added: +51 MB at the size above)
#pragma unroll
            for (int v = 0; v < V; v++) acc[o][v] += d[v];
        }
        if (V == 4) {
            f4u out;
#pragma unroll
            for (int v = 0; v < V; v++) out[v] = acc[o][v];
            *reinterpret_cast<f4u*>(d) = out;
        } else {
            *d = acc[o][0];
        }
    }
}

// Weight gradient of such a contraction.  A workgroup owns OT outputs and one row of a group, with all taps of a 3 x 3
// window or one window row of another, and a slice of the batch's pixels; a thread takes every 256th pixel.
// Sums: chains of four pixels, these per thread, the threads as a tree.
// The same tensors: 21, 45 and 158 us; k_wgrad takes 1070, 1285 and 1371 us.  Errors as k_wgrad's (1.0-1.2e-7).
template <int OT, int TVT>
__global__ __launch_bounds__(kThreads) void k_wgrad_narrow(Params Q) {
    constexpr int NT = TVT == 1 ? 1 : (TVT == 9 ? 9 : 7), U = 4;
    __shared__ float red[kThreads / 64][OT * NT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned b = tile_of_block();
    if (b >= (unsigned)Q.tiles) return;
    const int o0 = (int)(b % (unsigned)Q.mtiles) * OT;
    b /= (unsigned)Q.mtiles;
    const int kt = (int)(b % (unsigned)Q.ktiles);
    b /= (unsigned)Q.ktiles;
    const int g = (int)(b % (unsigned)Q.G);
    const int slice = (int)(b / (unsigned)Q.G);
    const int r = TVT ? kt : kt / Q.KH, kh0 = TVT ? 0 : kt - r * Q.KH;
    const int64_t P = Q.P, first = slice * Q.per_slice, last = min(Q.M, first + Q.per_slice);
    // every 256th pixel: the image and the place in it advance by a fixed step and a carry
    const int step_n = kThreads / Q.P, step_p = kThreads - step_n * Q.P;
    const int64_t m_first = first + tid;
    int64_t n = m_first / P;
    int p = (int)(m_first - n * P);
    const float* xs = Q.src + ((int64_t)g * Q.R + r) * P;
    const float* ds = Q.dy + ((int64_t)g * Q.Og + o0) * P;
    const int64_t xn = (int64_t)Q.G * Q.R * P, dn = (int64_t)Q.G * Q.Og * P;
    float acc[OT][NT];
#pragma unroll
    for (int o = 0; o < OT; o++)
#pragma unroll
        for (int t = 0; t < NT; t++) acc[o][t] = 0.f;
    for (int64_t m = m_first; m < last; m += U * kThreads) {
        float x[U][NT], dy[U][OT];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const bool in = m + u * kThreads < last;
            const float* xp = xs + (in ? n * xn : 0);  // (a pixel past the slice reads the first image and counts as zero)
            const int q = in ? p : 0;
#pragma unroll
            for (int o = 0; o < OT; o++) {
                dy[u][o] = ds[(in ? n * dn : 0) + min(o, Q.Og - 1 - o0) * P + q];
                dy[u][o] = in ? dy[u][o] : 0.f;
            }
            if (TVT == 1) {
                x[u][0] = xp[q];
                x[u][0] = in ? x[u][0] : 0.f;
            } else {
                const int h = quotient(q, Q.W, Q.mW), c = q - h * Q.W;
#pragma unroll
                for (int t = 0; t < NT; t++) {
                    x[u][t] = 0.f;
                    if (TVT != 9 && t >= Q.KW) continue;
                    const int hh = h + (TVT == 9 ? t / 3 - 1 : kh0 - Q.KH / 2), cc = c + (TVT == 9 ? t % 3 - 1 : t - Q.KW / 2);
                    const bool inside = in && (unsigned)hh < (unsigned)Q.H && (unsigned)cc < (unsigned)Q.W;
                    x[u][t] = xp[inside ? hh * Q.W + cc : q];
                    x[u][t] = inside ? x[u][t] : 0.f;
                }
            }
            n += step_n;
            p += step_p;
            if (p >= Q.P) {
                p -= Q.P;
                n++;
            }
        }
#pragma unroll
        for (int o = 0; o < OT; o++)
#pragma unroll
            for (int t = 0; t < NT; t++) {
                float part = dy[0][o] * x[0][t];
#pragma unroll
                for (int u = 1; u < U; u++) part = fmaf(dy[u][o], x[u][t], part);
                acc[o][t] += part;
            }
    }
#pragma unroll
    for (int o = 0; o < OT; o++)
#pragma unroll
        for (int t = 0; t < NT; t++) {
            float v = acc[o][t];
#pragma unroll
            for (int d = 32; d >= 1; d /= 2) v += __shfl_xor(v, d);
            if (lane == 0) red[wave][o * NT + t] = v;
        }
    __syncthreads();
    const int taps = TVT ? TVT : Q.KW;
    if (tid < OT * NT) {
        const int o = tid / NT, t = tid - o * NT;
        if (o0 + o < Q.Og && t < taps)
            Q.partial[(int64_t)slice * Q.G * Q.Og * Q.K + ((int64_t)g * Q.Og + o0 + o) * Q.K + (int64_t)r * Q.TV + kh0 * Q.KW + t] =
                (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
    }
}

// Positions a tile of `pixels` consecutive pixels of the batch covers at most, margin included: the image rows it
// touches, KH - 1 rows for each change of image, and the window's own KH - 1.
int window_positions(const Params& p, int pixels) {
    const int rows = (pixels - 1 + p.W - 1) / p.W + 1;
    const int changes = (rows - 1 + p.H - 1) / p.H;
    return (rows + (changes + 1) * (p.KH - 1)) * p.Wp;
}

int up(int v, int mod, int rem) { return v + (rem - v % mod + mod) % mod; }

constexpr int kMaxWindowPositions = 1024;  // what a workgroup's threads keep the offsets of (4 each)

size_t fwd_lds(const Params& p) { return 4 * (size_t)(p.TV == 1 ? kLinearKc : (p.wide ? 4 : 8)) * p.CS; }

size_t wgrad_lds(const Params& p) {
    return 4 * ((size_t)kPix + 4 * (size_t)p.S + (size_t)16 * p.mt * p.wm * kDyStride + (size_t)p.nch * p.CS);
}

}  // namespace

bool window_supported(int KH, int KW, int H, int W) {
    if (KH > 7 || KW > 7 || KH * KW < 2 || W > kMaxWindowPositions) return false;
    Params p = shape(1, 1, 1, KH, KW, 1, H, W);
    p.S = window_positions(p, kPix);
    p.CS = up(p.S, 2, 1);
    if (p.S > kMaxWindowPositions) return false;
    if ((int64_t)p.P * W >= (int64_t)1 << 32 || (int64_t)(H + 2 * kMaxWindowPositions) * p.HP >= (int64_t)1 << 32) return false;  // quotient()
    for (p.wm = 1; p.wm <= 2; p.wm++) {  // the weight gradient's smallest tiles: 32 x 64 and 64 x 32, any number of channels
        p.mt = 2;
        p.nch = (16 * (4 / p.wm) + p.TV - 2) / p.TV + 1;
        if (wgrad_lds(p) > (size_t)kMaxLds) return false;
    }
    return true;
}

// Where the vector unit is faster than padded matrix tiles (both measured at N=32, 28x28, about 64 channels, 1-16 rows and
// outputs per group; us matrix / narrow).  Without a window up to eight rows, since each costs a load: R=8, Og=1 9.0 / 4.2,
// Og=16 8.6 / 5.5; R=16 5.8 / 4.4 at one output, but transposed 6.3 / 6.6 at four.  3 x 3: R=1, Og=8 12.3 / 9.2, Og=16
// 8.0 / 9.2; R=2, Og=4 20.0 / 13.8, Og=6 13.5 / 13.9; R=3 20.9 / 21.7.  Other windows (5 x 5): R=1, Og=4 37.8 / 27.1, Og=6
// 25.4 / 27.4; R=2, Og=2 63.9 / 72.6.  A window on few pixels is a chain of loads on an empty chip: 8 images of 15x15 in four
// groups, 5 x 5 6.4 / 7.3, 50 176 pixels and groups 5.4 / 5.0.
constexpr int64_t kNarrowWindowPixels = 32768;

static int narrow_forward(const Params& p) {
    if (p.TV == 1) return p.R <= 8 ? p.Og <= 16 : p.R <= 16 && p.Og <= 2;
    if (p.M * p.G < kNarrowWindowPixels) return 0;
    if (p.KH == 3 && p.KW == 3) return p.R == 1 ? p.Og <= 8 : p.R == 2 && p.Og <= 4;
    return p.R == 1 && p.Og <= 4;
}

// The same for the weight gradient, whose cost is that of its R * Og products per pixel and tap.  Without a window: R=8, Og=8
// 28.9 / 14.4 (N=64, 56x56: 147 / 41), R=64, Og=1 21.1 / 14.9, 16 x 16 20.2 / 18.8.  3 x 3: 4 x 4 50.2 / 31.0, R=4, Og=6
// 34.4 / 34.6, R=16, Og=1 29.4 / 14.8.  5 x 5: R=1, Og=8 32.3 / 28.0, R=2, Og=6 36.6 / 39.6.  Few pixels, 3 x 3: 12 544
// 10.9 / 14.8, 50 176 14.8 / 5.2.
static int narrow_wgrad(const Params& p) {
    const int64_t products = (int64_t)p.R * p.Og;
    if (p.TV == 1) return products <= 64;
    if (p.M * p.G < kNarrowWindowPixels) return 0;
    return products <= (p.KH == 3 && p.KW == 3 ? 16 : 8);
}

Params shape(int64_t N, int G, int R, int KH, int KW, int Og, int H, int W) {
    Params p;
    p.N = N;
    p.G = G;
    p.R = R;
    p.KH = KH;
    p.KW = KW;
    p.TV = KH * KW;
    p.K = R * p.TV;
    p.Og = Og;
    p.H = H;
    p.W = W;
    p.P = H * W;
    p.M = N * p.P;
    p.HP = H + KH - 1;
    p.Wp = W + KW - 1;
    auto magic = [](uint32_t d) { return (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
    p.mP = magic(p.P);
    p.mW = magic(W);
    p.mHP = magic(p.HP);
    p.mWp = magic(p.Wp);
    return p;
}

Params data_gradient_of(const Params& f) {
    Params p = shape(f.N, f.G, f.Og, f.KH, f.KW, f.R, f.H, f.W);
    p.transposed = 1;
    return p;
}

// Where the bf16 matrix units are faster, the cutting of the weights included (fp32 units / here, us; 4.2 for the launch that
// cuts the weights of both directions).  3 x 3, forward + data gradient: 64 channels 32x28x28 38.6 + 36.4 / 21.0 + 21.2, 8x40x40
// 22.4 + 22.1 / 15.0 + 15.2, 1x28x28 15.8 + 16.0 / 12.4 + 12.4; 96 channels 8x40x40 52.0 + 49.5 / 30.7 + 30.7; 128 channels
// 32x14x14 40.8 + 39.7 / 21.4 + 21.4; eight groups of 32 32x14x14 22.8 + 21.0 / 14.2 + 14.2, of 64 16x7x7 16.7 + 17.4 / 13.4 + 13.4
// (6.0 for the weights); 32 channels 32x28x28 13.9 + 13.0 / 10.6 + 10.7; but 48 channels 32x14x14 (98 workgroups) 12.7 + 13.0 /
// 11.1 + 11.2.  Without a window: 128 channels 32x28x28 24.8 + 23.5 / 18.4 + 18.2, 512 channels 32x14x14 69.6 + 68.3 / 41.1 + 41.0;
// but 64 channels 32x28x28 9.2 + 8.9 / 8.1 + 8.2, 512 channels 16x7x7 (104 workgroups) 19.1 + 18.2 / 17.7 + 16.8.  Not below 32
// channels or outputs, where part of a tile is padding: 3 x 3, the weights included, 24 channels 32x28x28 21.8 / 24.7, 5x14x14 15.9 / 22.6, 16
// channels 32x28x28 13.7 / 18.8, eight groups of 16 44.6 / 58.0, of 24 16x14x14 21.6 / 23.9; 24 -> 64 channels 32x28x28 39.7 / 32.6 would gain.
static bool split_forward(Params& p) {
    const bool win = p.KH == 3 && p.KW == 3;
    if (!win && p.TV != 1) return false;
    Params q = p;
    q.split = 1;
    q.wm = p.Og > 32 ? 2 : 1;
    const int pixels = 32 * (4 / q.wm);
    q.mtiles = (q.Og + 32 * q.wm - 1) / (32 * q.wm);
    q.tiles = (q.M + pixels - 1) / pixels * q.G * q.mtiles;
    if (win ? p.Og < 32 || p.R < 32 || (p.R < 64 && q.tiles < 192) : p.Og <= 32 || p.R < 128 || q.tiles < 384) return false;
    q.S = win ? window_positions(q, pixels) : pixels;
    if (q.S > 512) return false;  // (four items of the operand tile per thread)
    // 32-bit byte offsets within the images of a tile and within a group's weights, and 3 GB of cut weights
    const int64_t images = (pixels + q.P - 1) / q.P + 1;
    if (images * q.G * q.R * q.P >= (int64_t)1 << 29 || (int64_t)q.Og * q.K >= (int64_t)1 << 29) return false;
    if ((int64_t)q.G * q.mtiles * q.wm * ((q.R + 15) / 16) * q.TV * 64 >= (int64_t)1 << 26) return false;
    p = q;
    return true;
}

void prepare_forward(Params& p, bool may_split) {
    const bool win = p.TV > 1;
    p.narrow = narrow_forward(p);
    if (p.narrow) {
        p.ot = p.Og > 2 ? 4 : p.Og;
        p.vec = p.P % 4 == 0 ? 4 : 1;
        p.mtiles = (p.Og + p.ot - 1) / p.ot;
        p.tiles = (p.M * p.G + kThreads * p.vec - 1) / (kThreads * p.vec) * p.mtiles;
        return;
    }
    if (may_split && split_forward(p)) return;
    // Up to four wavefronts side by side over the outputs: a weight then reaches the workgroup once, a staged pixel
    // serves up to 64 outputs.  Half the pixels where the launch would otherwise have less than two workgroups per
    // compute unit.
    p.wm = p.Og > 32 ? 4 : (p.Og > 16 ? 2 : 1);
    p.nt = p.wm == 1 ? 2 : 4;
    p.mtiles = (p.Og + 16 * p.wm - 1) / (16 * p.wm);
    auto pixels = [&]() { return 16 * p.nt * (4 / p.wm); };
    auto tiles = [&]() { return (p.M + pixels() - 1) / pixels() * p.G * p.mtiles; };
    if (tiles() < 2 * 256) p.nt /= 2;
    p.wide = 0;
    if (win) {
        if (window_positions(p, pixels()) > 2 * kThreads && pixels() > 64) p.nt /= 2;
        if (window_positions(p, pixels()) > 2 * kThreads) {
            p.wide = 1;
            p.nt = p.wm;  // (64 pixels)
        }
        p.S = window_positions(p, pixels());
        p.CS = up(p.S, 64, 16);  // the four channels of an operand read in different banks
    } else {
        p.S = pixels();
        p.CS = up(p.S, 16, 4);  // the same for channels four apart
    }
    p.tiles = tiles();
}

// Slices of whole steps, for about `workgroups` of them.
static void split(Params& p, int workgroups, int step, int64_t max_partial_bytes) {
    const int64_t tiles = (int64_t)p.ktiles * p.mtiles * p.G * (p.split ? p.KH : 1);
    const int64_t places = p.split ? p.N * p.HP * p.Wp : p.M;
    const int64_t steps = (places + step - 1) / step;
    const int64_t bytes = (int64_t)p.G * p.Og * p.K * 4;
    int64_t slices = std::max<int64_t>(1, workgroups / tiles);
    if (p.split && steps <= 4) slices = 1;  // (a step takes 1.2 us, the launch that sums two slices 4.1)
    slices = std::min(slices, steps);
    slices = std::min(slices, std::max<int64_t>(1, max_partial_bytes / std::max<int64_t>(1, bytes)));
    p.per_slice = (steps + slices - 1) / slices * step;
    p.slices = (int)((places + p.per_slice - 1) / p.per_slice);
    p.tiles = p.slices * tiles;
}

// Weight gradient on the bf16 matrix units, behind a 3 x 3 window where a tile of 32 x 32 is filled (fp32 units / here, us): 64
// channels 32x28x28 46.5 / 28.0, 1x28x28 10.3 / 7.9, 32x7x7 11.2 / 9.0; 128 channels 32x14x14 45.4 / 30.5, 16x56x20 95 / 62;
// eight groups of 32 32x14x14 43.6 / 21.5, of 64 16x7x7 22.0 / 15.2; 48 channels 6x23x17 11.4 / 8.7; 32 channels 32x28x28
// 22.7 / 14.7, 4x28x28 7.7 / 7.5; 64 channels 1x8x8 9.8 / 9.7.  Below 32 channels it is a tile of padding in part: 16 channels 32x28x28
// 11.2 / 12.4, eight groups of 16 42.4 / 52.6, though 24 channels 18.6 / 13.1.
static bool split_wgrad(Params& p, int64_t max_partial_bytes) {
    if (p.KH != 3 || p.KW != 3 || p.Og < 32 || p.R < 32) return false;
    Params q = p;
    q.split = 1;
    q.wm = q.Og > 32 ? 2 : 1;
    q.mtiles = (q.Og + 32 * q.wm - 1) / (32 * q.wm);
    q.ktiles = (q.R + 31) / 32;
    q.HP = q.H + 1;
    q.Wp = q.W + 1;
    q.mWp = (uint32_t)((((uint64_t)1 << 32) + q.Wp - 1) / q.Wp);
    // 32-bit byte offsets within the tensors, exact quotients
    if (q.N * q.G * std::max(q.R, q.Og) * (int64_t)q.P >= (int64_t)1 << 30 || (int64_t)q.HP * q.Wp * q.Wp >= (int64_t)1 << 31 || q.N * q.HP * q.Wp >= (int64_t)1 << 31)
        return false;
    split(q, 2 * 256, kPix, max_partial_bytes);
    p = q;
    return true;
}

void prepare_wgrad(Params& p, int64_t max_partial_bytes) {
    const bool win = p.TV > 1;
    p.narrow = narrow_wgrad(p);
    if (p.narrow) {
        p.ot = p.Og > 2 ? 4 : p.Og;
        p.mtiles = (p.Og + p.ot - 1) / p.ot;
        p.ktiles = p.R * (p.TV == 1 || (p.KH == 3 && p.KW == 3) ? 1 : p.KH);
        split(p, 4096, kNarrowPix, max_partial_bytes);
        return;
    }
    if (split_wgrad(p, max_partial_bytes)) return;
    p.S = win ? window_positions(p, kPix) : kPix;
    p.CS = win ? up(p.S, 2, 1) : up(p.S, 64, 4);
    // outputs: one or two 16-tiles per wavefront, one or two wavefronts across them
    p.mt = p.Og > 16 ? 2 : 1;
    p.wm = p.Og > 32 ? 2 : 1;
    const int wn = 4 / p.wm;
    // contraction indices: the widest tile that does not add padding, as far as LDS holds the channels behind it
    int best = 1;
    int64_t least = INT64_MAX;
    for (int nt = 4; nt >= 1; nt--) {
        p.nt = nt;
        const int bn = 16 * nt * wn;
        p.nch = std::min(p.R, win ? (bn + p.TV - 2) / p.TV + 1 : bn);
        if (wgrad_lds(p) > (size_t)kMaxLds && nt > 1) continue;
        const int64_t cols = (int64_t)(p.K + bn - 1) / bn * bn;
        if (cols < least) {
            least = cols;
            best = nt;
        }
    }
    p.nt = best;
    const int bn = 16 * p.nt * wn, bm = 16 * p.mt * p.wm;
    p.nch = std::min(p.R, win ? (bn + p.TV - 2) / p.TV + 1 : bn);
    p.ktiles = (p.K + bn - 1) / bn;
    p.mtiles = (p.Og + bm - 1) / bm;
    split(p, 2 * 256, kPix, max_partial_bytes);  // (one round: two workgroups of the wide tiles fit a compute unit)
}

// A launch has fewer than 2^32 threads along x: one output per group and 128 pixels per workgroup reach that at 2^31
// elements, 8 GB.  Longer grids get more than one row.
static dim3 grid_of(int64_t tiles) {
    constexpr int64_t kMaxX = ((int64_t)1 << 32) / kThreads - 8;
    const int64_t rows = std::max<int64_t>(1, (tiles + kMaxX - 1) / kMaxX);
    const int64_t per_row = (tiles + rows - 1) / rows;
    return dim3((unsigned)((per_row + 7) / 8 * 8), (unsigned)rows);
}

void forward(const Params& p, hipStream_t s) {
    const dim3 grid = grid_of(p.tiles), block(kThreads);
    if (p.narrow) {
#define CANVAS_SFC_T(OT, V, TVT)                                                                                       \
    do {                                                                                                               \
        if (p.transposed) CANVAS_LAUNCH((k_fwd_narrow<OT, V, TVT, true>), grid, block, 0, s, p);                       \
        else CANVAS_LAUNCH((k_fwd_narrow<OT, V, TVT, false>), grid, block, 0, s, p);                                   \
    } while (0)
#define CANVAS_SFC(OT, V)                                               \
    do {                                                                \
        if (p.TV == 1) CANVAS_SFC_T(OT, V, 1);                          \
        else if (p.KH == 3 && p.KW == 3) CANVAS_SFC_T(OT, V, 9);        \
        else CANVAS_SFC_T(OT, V, 0);                                    \
    } while (0)
        switch (p.ot * 10 + p.vec) {
        case 11: CANVAS_SFC(1, 1); break;
        case 14: CANVAS_SFC(1, 4); break;
        case 21: CANVAS_SFC(2, 1); break;
        case 24: CANVAS_SFC(2, 4); break;
        case 41: CANVAS_SFC(4, 1); break;
        default: CANVAS_SFC(4, 4); break;
        }
#undef CANVAS_SFC
#undef CANVAS_SFC_T
        return;
    }
    if (p.split) {
        forward_split(p, grid, s);
        return;
    }
    const size_t lds = fwd_lds(p);
#define CANVAS_SFC_T(WM, NT, TVT, WIN, NP, KC)                                                                          \
    do {                                                                                                               \
        if (p.transposed) CANVAS_LAUNCH((k_fwd<WM, NT, TVT, WIN, NP, KC, true>), grid, block, lds, s, p);              \
        else CANVAS_LAUNCH((k_fwd<WM, NT, TVT, WIN, NP, KC, false>), grid, block, lds, s, p);                          \
    } while (0)
#define CANVAS_SFC(WM, NT)                                                                                             \
    do {                                                                                                               \
        if (p.TV == 1) CANVAS_SFC_T(WM, NT, 1, false, 1, kLinearKc);                                                   \
        else if (p.wide && p.KH == 3 && p.KW == 3) CANVAS_SFC_T(WM, WM, 9, true, 4, 4);                                \
        else if (p.wide) CANVAS_SFC_T(WM, WM, 0, true, 4, 4);                                                          \
        else if (p.KH == 3 && p.KW == 3) CANVAS_SFC_T(WM, NT, 9, true, 2, 8);                                          \
        else CANVAS_SFC_T(WM, NT, 0, true, 2, 8);                                                                      \
    } while (0)
    switch (p.wm * 10 + p.nt) {
    case 11: CANVAS_SFC(1, 1); break;
    case 12: CANVAS_SFC(1, 2); break;
    case 22: CANVAS_SFC(2, 2); break;
    case 24: CANVAS_SFC(2, 4); break;
    case 42: CANVAS_SFC(4, 2); break;
    default: CANVAS_SFC(4, 4); break;
    }
#undef CANVAS_SFC
#undef CANVAS_SFC_T
}

void wgrad_partial(const Params& p, hipStream_t s) {
    const dim3 grid = grid_of(p.tiles), block(kThreads);
    if (p.narrow) {
#define CANVAS_SFC(OT)                                                                                       \
    do {                                                                                                     \
        if (p.TV == 1) CANVAS_LAUNCH((k_wgrad_narrow<OT, 1>), grid, block, 0, s, p);                         \
        else if (p.KH == 3 && p.KW == 3) CANVAS_LAUNCH((k_wgrad_narrow<OT, 9>), grid, block, 0, s, p);       \
        else CANVAS_LAUNCH((k_wgrad_narrow<OT, 0>), grid, block, 0, s, p);                                   \
    } while (0)
        switch (p.ot) {
        case 1: CANVAS_SFC(1); break;
        case 2: CANVAS_SFC(2); break;
        default: CANVAS_SFC(4); break;
        }
#undef CANVAS_SFC
        return;
    }
    if (p.split) {
        wgrad_split(p, grid, s);
        return;
    }
    const size_t lds = wgrad_lds(p);
#define CANVAS_SFC(MT, NT, WM)                                                           \
    do {                                                                                 \
        if (p.TV == 1) CANVAS_LAUNCH((k_wgrad<MT, NT, WM, false>), grid, block, lds, s, p); \
        else CANVAS_LAUNCH((k_wgrad<MT, NT, WM, true>), grid, block, lds, s, p);         \
    } while (0)
#define CANVAS_SFC_NT(MT, WM)                    \
    switch (p.nt) {                              \
    case 1: CANVAS_SFC(MT, 1, WM); break;        \
    case 2: CANVAS_SFC(MT, 2, WM); break;        \
    case 3: CANVAS_SFC(MT, 3, WM); break;        \
    default: CANVAS_SFC(MT, 4, WM); break;       \
    }
    if (p.wm == 2) CANVAS_SFC_NT(2, 2)
    else if (p.mt == 2) CANVAS_SFC_NT(2, 1)
    else CANVAS_SFC_NT(1, 1)
#undef CANVAS_SFC_NT
#undef CANVAS_SFC
}

}  // namespace sfc
}  // namespace canvas
