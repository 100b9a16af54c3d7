// Fused kernels for the pattern
//     x -> Shift (one offset per FC group) -> grouped FC -> unary -> (+ x) -> y
// on bf16 NCHW tensors: shift-convolution plus residual, the shape of the best kernel the paper
// reports for ResNet-34 (Section 8, kernel-level analysis) built from the Shift, Group,
// Fully-connected, element-wise and Broadcast primitives of Section 5.
//
// The pattern is bound by HBM traffic (8 flop per byte), so the kernels touch x, y (forward) and
// x, dy, dx (backward) once in HBM and keep everything else in registers (plus, in backward, one
// wave-private LDS tile used as a transposer):
//  * one wavefront owns a tile of 16*KC input channels x 128 pixels of one image and one FC group;
//  * every lane loads 16 bytes (8 consecutive pixels of one channel), so a load instruction covers
//    four channel rows x 256 contiguous bytes;
//  * the FC is a 16x16x16 bf16 MFMA with pixels as the N (or M) dimension.  A lane needs four
//    channels of ONE pixel per MFMA operand but holds eight pixels of four channels; eight MFMAs,
//    one per pixel offset q, take their operands from the q-th halves of the loaded registers
//    (two byte-permutes each), so no cross-lane transpose is needed;
//  * the spatial shift is an address offset of the load plus a zero mask at image borders.  All
//    tensor accesses are buffer loads/stores with the tensor size as the hardware bound, so a shifted
//    16-byte access that leaves the tensor at its two ends returns zeros instead of faulting;
//  * backward recomputes the FC output instead of saving it.  dX = W^T dz contracts over channels like
//    the forward FC; dW = dz x^T contracts over pixels, so x and dz go once through LDS to reach the
//    register distribution that contraction needs (a second pass over global memory for it, even one
//    served by L2, costs a full memory round trip per tile and was measurably slower);
//  * each wavefront writes one dW partial; a second small kernel sums them in a fixed order: no atomics;
//  * throughput is set by the bytes a SIMD keeps in flight to HBM (latency under load is several
//    microseconds), so every load of a tile is issued before any arithmetic and registers are kept
//    below 128 (4 wavefronts per SIMD).
#include "sgfc_kernels.hpp"

#include <hip/hip_runtime.h>

#include "device_util.hpp"
#include "launch.hpp"
#include "tile_util.hpp"

namespace canvas {
namespace sgfc {

namespace {

using namespace canvas::tile;

constexpr int kTilePx = 128;  // pixels per wavefront tile
constexpr int kWaves = 4;     // wavefronts per workgroup
constexpr int kActNone = -1;  // ACT template value: no unary node; otherwise a UnaryKind

// True (wave-uniform) when a tile's shifted accesses, planes starting at elements [first, last] x [p0+off, p0+off+136), leave the tensor.
__device__ __forceinline__ bool tile_near_ends(int first, int last, int p0, int off, int total_elems) {
    return first + p0 + off < 0 || last + p0 + off + kTilePx + 8 > total_elems;
}
// Elements a tensor of N images spans: `stride` apart, `planes` planes of Pn each (the last image ends with its own planes).
__device__ __forceinline__ int extent(int N, int stride, int planes, int Pn) { return (N - 1) * stride + planes * Pn; }

// Validity of the 128 pixels of a tile under a shift: bit i is 1 when tile pixel i exists (p < P) and
// its source pixel (h+dh, w+dw) lies inside the image.  magic = ceil(2^32 / W) gives h = p / W exactly.
struct TileMask {
    uint64_t lo, hi;  // pixels 0..63, 64..127
};
__device__ __forceinline__ TileMask tile_mask(int p0, int lane, const Params& P, int dh, int dw) {
    TileMask m;
    int pa = p0 + lane, pb = p0 + 64 + lane;
    int ha = (int)__umulhi((uint32_t)pa, P.magicW), wa = pa - ha * P.W;
    int hb = (int)__umulhi((uint32_t)pb, P.magicW), wb = pb - hb * P.W;
    bool va = pa < P.P && (unsigned)(ha + dh) < (unsigned)P.H && (unsigned)(wa + dw) < (unsigned)P.W;
    bool vb = pb < P.P && (unsigned)(hb + dh) < (unsigned)P.H && (unsigned)(wb + dw) < (unsigned)P.W;
    m.lo = __ballot(va);
    m.hi = __ballot(vb);
    return m;
}
// The 8 validity bits of unit u (pixels 8u..8u+7 of the tile): byte u of the 128-bit mask, picked with
// byte permutes (a dynamically indexed array would be spilled to LDS).
__device__ __forceinline__ uint32_t unit_bits(const TileMask& m, int u) {
    const uint32_t sel = 0x0c0c0c00u | (uint32_t)(u & 7);
    const uint32_t a = __builtin_amdgcn_perm((uint32_t)(m.lo >> 32), (uint32_t)m.lo, sel);
    const uint32_t b = __builtin_amdgcn_perm((uint32_t)(m.hi >> 32), (uint32_t)m.hi, sel);
    return (u & 8) ? b : a;
}


template <int ACT>
__device__ __forceinline__ float act_apply(const Params& P, float z) {
    if (ACT == kActNone) return z;
    return unary_apply(ACT, z, P.ulo, P.uhi);
}
// dz = dy * act'(z)
template <int ACT>
__device__ __forceinline__ float act_dz(const Params& P, float z, float dy) {
    if (ACT == kActNone) return dy;
    if (ACT == 0) return z > 0.f ? dy : 0.f;
    return dy * unary_grad(ACT, z, P.ulo, P.uhi);
}

// Planes that are no multiple of eight pixels (RAG): a plane's last unit is `left` < 8 pixels of its own, then the next plane's.
// Those are cleared where a sum over pixels would take them in and never stored, rows begin at any element, and an unshifted
// access too can cross the tensor's end.  (The lowering by units, which such planes used to take: a step of N=6, 64 channels, 20x41 72.7 us, here
// 19.6; N=64, 27x29 235, here 19.5; 64 => 128 channels N=5, 21x11 289, here 19.8.)
template <bool RAG>
__device__ __forceinline__ void store_unit(rsrc_t r, int off, const u32x4& v, int left) {
    if (!RAG) {
        bstore16_nt(r, off, v);
    } else if (left >= 8) {
        bstore16(r, off, v);  // (unaligned: kept in the cache until its lines are whole)
    } else {
#pragma unroll
        for (int q = 0; q < 8; q++)
            if (q < left) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(v[q >> 1] >> (16 * (q & 1))), r, off + 2 * q, 0, 0);
    }
}
__device__ __forceinline__ u32x4 own_pixels(int left) { return mask_of(left >= 8 ? 0xffu : (left > 0 ? (1u << left) - 1u : 0u)); }

// ------------------------------------------------------------------------------------------ forward
template <int KC, int MO, int ACT, bool RES, bool RAG>
__global__ __launch_bounds__(64 * kWaves) void k_fwd(Params P) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk = blockIdx.x * kWaves + wave;
    if (chunk >= P.chunks) return;
    const int g = blockIdx.y, n = blockIdx.z;
    const int r = lane >> 4, s = lane & 15;
    constexpr int CG = 16 * KC, OG = 16 * MO;
    const int Cout = P.G * OG;
    const int p0 = chunk * kTilePx, p = p0 + 8 * s;
    const int dh = P.dh[g], dw = P.dw[g], off = dh * P.W + dw;
    const int xelems = extent(P.N, P.xs, P.C, P.P), yelems = extent(P.N, P.ys, Cout, P.P);
    const rsrc_t rx = make_rsrc(P.x, xelems * 2);
    const rsrc_t ry = make_rsrc(P.y, yelems * 2);
    const TileMask tm = tile_mask(p0, lane, P, dh, dw);
    const bool live = p < P.P;
    const uint32_t bits = live ? unit_bits(tm, s) : 0u;
    const u32x4 msk = mask_of(bits);
    const int xg = (n * P.xs + g * CG * P.P) * 2;  // byte offset of the group's first input plane

    // weights: A operand, lane holds W[g][mo*16 + s][kc*16 + 4r .. +3]
    short4_t wa[MO][KC];
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int kc = 0; kc < KC; kc++) __builtin_memcpy(&wa[mo][kc], P.w + ((g * OG + mo * 16 + s) * CG + kc * 16 + 4 * r), 8);

    u32x4 xs[KC][4];
#pragma unroll
    for (int kc = 0; kc < KC; kc++)
#pragma unroll
        for (int j = 0; j < 4; j++) xs[kc][j] = bload16(rx, live ? xg + ((kc * 16 + 4 * r + j) * P.P + p + off) * 2 : kOob);
    if (tile_near_ends(xg / 2, xg / 2 + (CG - 1) * P.P, p0, off, xelems)) {
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int j = 0; j < 4; j++)
                reload_if_partial(xs[kc][j], rx, live ? xg + ((kc * 16 + 4 * r + j) * P.P + p + off) * 2 : kOob, xelems * 2);
    }
    u32x4 xr[MO][4];
    if (RES) {
        const int xo = (n * P.xs + g * OG * P.P) * 2;
#pragma unroll
        for (int mo = 0; mo < MO; mo++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                xr[mo][j] = bload16_nt(rx, live ? xo + ((mo * 16 + 4 * r + j) * P.P + p) * 2 : kOob);
                pin(xr[mo][j]);
            }
        if (RAG && tile_near_ends(xo / 2, xo / 2 + (OG - 1) * P.P, p0, 0, xelems)) {
#pragma unroll
            for (int mo = 0; mo < MO; mo++)
#pragma unroll
                for (int j = 0; j < 4; j++) reload_if_partial(xr[mo][j], rx, live ? xo + ((mo * 16 + 4 * r + j) * P.P + p) * 2 : kOob, xelems * 2);
        }
    }

    float4_t acc[MO][8];
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int q = 0; q < 8; q++) acc[mo][q] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < KC; kc++) {
#pragma unroll
        for (int j = 0; j < 4; j++) xs[kc][j] = xs[kc][j] & msk;
        short4_t b[8];
        gather_all(xs[kc], b);
#pragma unroll
        for (int q = 0; q < 8; q++)
#pragma unroll
            for (int mo = 0; mo < MO; mo++) acc[mo][q] = mfma16(wa[mo][kc], b[q], acc[mo][q]);  // (a group contracts 16 channels: K = 16 is the whole depth)
    }
    const int yo = (n * P.ys + g * OG * P.P) * 2;
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; q++) v[q] = act_apply<ACT>(P, acc[mo][q][j]);
            if (RES) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    v[2 * k] += lo_f32(xr[mo][j][k]);
                    v[2 * k + 1] += hi_f32(xr[mo][j][k]);
                }
            }
            u32x4 out;
#pragma unroll
            for (int k = 0; k < 4; k++) out[k] = pack_bf16(v[2 * k], v[2 * k + 1]);
            store_unit<RAG>(ry, live ? yo + ((mo * 16 + 4 * r + j) * P.P + p) * 2 : kOob, out, P.P - p);
        }
}

// ----------------------------------------------------------------------------------------- backward
// dx[i,p] = (residual ? dy[i,p] : 0) + sum_o W[o,i] dz[o,p-d],  dz = dy * act'(z),  z[o,p-d] = sum_i W[o,i] x[i,p]
// dW[o,i] = sum_{n,p} dz[o,p-d] x[i,p]
//
// Registers hold the tile as: lane (r = lane/16, s = lane%16) -> channels 4r+j (j = 0..3) of the 8-pixel
// unit s.  That suits z = W x and dX = W^T dz (contractions over channels).  dW contracts over pixels and
// needs channel s with runs of consecutive pixels per lane instead; x and dz are passed through a
// wave-private LDS tile ([16 channels][128 pixels], rows padded to 272 bytes) to change distribution.
constexpr int kLdsRow = 17;  // u32x4 per LDS row: 16 units + 1 pad

// Whether dz enters dX and dW as two bf16 parts, dz = hi + lo, 16 bits of it.  Behind relu, abs or nothing it is +-dy or zero and one
// part holds all of it; behind gelu and clipped exp (ACT 2, 3) one part is off by 2^-9, which dW then is too (1.7e-3 in norm, with
// two parts 2.5e-6).  The instances for ragged planes take two, which is what the lowering by units gives there; those for
// planes of whole units one, as they always have.
template <int ACT, bool RAG>
constexpr bool kTwoParts = RAG && (ACT == 2 || ACT == 3);
template <int KC, int MO, int ACT, bool RES, bool RAG>
__device__ __forceinline__ void bwd_tile(const Params& P, rsrc_t rx, rsrc_t rdy, rsrc_t rdx, u32x4* lds_x, u32x4* lds_dz, int n, int g,
                                         int p0, int lane, const short4_t (&wa)[MO][KC], const short4_t (&wt)[KC][MO],
                                         float4_t (&dwacc)[MO][KC]) {
    const int r = lane >> 4, s = lane & 15;
    constexpr int CG = 16 * KC, OG = 16 * MO;
    constexpr bool TWO = kTwoParts<ACT, RAG>;
    u32x4* const lds_low = lds_dz + MO * 16 * kLdsRow;
    const int dh = P.dh[g], dw = P.dw[g], off = dh * P.W + dw;
    const int Cout = P.G * OG;
    const int pA = p0 + 8 * s;
    const bool liveA = pA < P.P;
    const int xg = (n * P.xs + g * CG * P.P) * 2;
    const int dyg = (n * P.ys + g * OG * P.P) * 2;
    // dy is read at p - d: validity of the shifted source uses (-dh, -dw)
    const TileMask tm = tile_mask(p0, lane, P, -dh, -dw);
    const u32x4 msk = mask_of(liveA ? unit_bits(tm, s) : 0u);

    u32x4 xa[KC][4], dya[MO][4], dyu[KC][4];
#pragma unroll
    for (int kc = 0; kc < KC; kc++)
#pragma unroll
        for (int j = 0; j < 4; j++) xa[kc][j] = bload16_nt(rx, liveA ? xg + ((kc * 16 + 4 * r + j) * P.P + pA) * 2 : kOob);
    const int xelems = extent(P.N, P.xs, P.C, P.P);
    if (RAG && tile_near_ends(xg / 2, xg / 2 + (CG - 1) * P.P, p0, 0, xelems)) {
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int j = 0; j < 4; j++) reload_if_partial(xa[kc][j], rx, liveA ? xg + ((kc * 16 + 4 * r + j) * P.P + pA) * 2 : kOob, xelems * 2);
    }
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int j = 0; j < 4; j++) dya[mo][j] = bload16(rdy, liveA ? dyg + ((mo * 16 + 4 * r + j) * P.P + pA - off) * 2 : kOob);
    if (tile_near_ends(dyg / 2, dyg / 2 + (OG - 1) * P.P, p0, -off, extent(P.N, P.ys, Cout, P.P))) {
        const int dyelems = extent(P.N, P.ys, Cout, P.P);
#pragma unroll
        for (int mo = 0; mo < MO; mo++)
#pragma unroll
            for (int j = 0; j < 4; j++)
                reload_if_partial(dya[mo][j], rdy, liveA ? dyg + ((mo * 16 + 4 * r + j) * P.P + pA - off) * 2 : kOob, dyelems * 2);
    }
    auto reload_residual = [&](int kc, u32x4 (&v)[4]) {
        const int dyelems = extent(P.N, P.ys, Cout, P.P);
        if (RAG && tile_near_ends(dyg / 2, dyg / 2 + (OG - 1) * P.P, p0, 0, dyelems)) {
#pragma unroll
            for (int j = 0; j < 4; j++) reload_if_partial(v[j], rdy, liveA ? dyg + ((kc * 16 + 4 * r + j) * P.P + pA) * 2 : kOob, dyelems * 2);
        }
    };
    // (the unshifted dy of the residual: with one 16-channel block per group it is fetched with everything else; with
    // more the registers are short, and each block's rows are fetched just ahead of its dx)
    if (RES && KC == 1) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            dyu[0][j] = bload16_nt(rdy, liveA ? dyg + ((4 * r + j) * P.P + pA) * 2 : kOob);
            pin(dyu[0][j]);
        }
        reload_residual(0, dyu[0]);
    }
    if (RAG) {
        const u32x4 own = own_pixels(P.P - pA);
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int j = 0; j < 4; j++) xa[kc][j] = xa[kc][j] & own;
    }
    // x -> LDS rows (channel 4r+j, unit s) and -> MFMA operands
    short4_t xq[KC][8];
#pragma unroll
    for (int kc = 0; kc < KC; kc++) {
#pragma unroll
        for (int j = 0; j < 4; j++) lds_x[(kc * 16 + 4 * r + j) * kLdsRow + s] = xa[kc][j];
        gather_all(xa[kc], xq[kc]);
    }

    short4_t dzq[MO][8];
#pragma unroll
    for (int mo = 0; mo < MO; mo++) {
#pragma unroll
        for (int j = 0; j < 4; j++) dya[mo][j] = dya[mo][j] & msk;
        u32x4 dzrow[4], dzlow[4];  // dz of channel 4r+j over the unit's 8 pixels, for the LDS tile
        // steps of QS pixel offsets keep the live accumulators at 4 * QS registers (16; 8 where a group has more than
        // one 16-channel block and the tile's registers are short)
        constexpr int QS = KC > 1 ? 2 : 4;
#pragma unroll
        for (int h = 0; h < 8 / QS; h++) {
            float4_t z[QS];
#pragma unroll
            for (int q = 0; q < QS; q++) {
                z[q] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < KC; kc++) z[q] = mfma16(wa[mo][kc], xq[kc][QS * h + q], z[q]);
            }
            float d[QS][4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
#pragma unroll
                for (int q = 0; q < QS; q += 2) {
                    const uint32_t w = dya[mo][j][(QS * h + q) / 2];
                    d[q][j] = act_dz<ACT>(P, z[q][j], lo_f32(w));
                    d[q + 1][j] = act_dz<ACT>(P, z[q + 1][j], hi_f32(w));
                    const uint32_t hi = pack_bf16(d[q][j], d[q + 1][j]);
                    dzrow[j][(QS * h + q) / 2] = hi;
                    if (TWO) dzlow[j][(QS * h + q) / 2] = pack_bf16(d[q][j] - lo_f32(hi), d[q + 1][j] - hi_f32(hi));
                }
            }
#pragma unroll
            for (int q = 0; q < QS; q++) dzq[mo][QS * h + q] = pack4(d[q][0], d[q][1], d[q][2], d[q][3]);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            lds_dz[(mo * 16 + 4 * r + j) * kLdsRow + s] = dzrow[j];
            if (TWO) lds_low[(mo * 16 + 4 * r + j) * kLdsRow + s] = dzlow[j];
        }
    }
#pragma unroll
    for (int kc = 0; kc < KC; kc++) {
        if (RES && KC > 1) {
            asm volatile("" ::: "memory");  // (not earlier: the registers are needed until here)
#pragma unroll
            for (int j = 0; j < 4; j++) dyu[kc][j] = bload16_nt(rdy, liveA ? dyg + ((kc * 16 + 4 * r + j) * P.P + pA) * 2 : kOob);
            reload_residual(kc, dyu[kc]);
        }
        float4_t dxs[8];
#pragma unroll
        for (int q = 0; q < 8; q++) {
            dxs[q] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int mo = 0; mo < MO; mo++) dxs[q] = mfma16(wt[kc][mo], dzq[mo][q], dxs[q]);
        }
        if (TWO) {  // (the lane's own rows, from LDS: there are no registers to keep them in)
#pragma unroll
            for (int mo = 0; mo < MO; mo++) {
                u32x4 v[4];
                short4_t low[8];
#pragma unroll
                for (int j = 0; j < 4; j++) v[j] = lds_low[(mo * 16 + 4 * r + j) * kLdsRow + s];
                gather_all(v, low);
#pragma unroll
                for (int q = 0; q < 8; q++) dxs[q] = mfma16(wt[kc][mo], low[q], dxs[q]);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; q++) v[q] = dxs[q][j];
            if (RES) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    v[2 * k] += lo_f32(dyu[kc][j][k]);
                    v[2 * k + 1] += hi_f32(dyu[kc][j][k]);
                }
            }
            u32x4 out;
#pragma unroll
            for (int k = 0; k < 4; k++) out[k] = pack_bf16(v[2 * k], v[2 * k + 1]);
            store_unit<RAG>(rdx, liveA ? xg + ((kc * 16 + 4 * r + j) * P.P + pA) * 2 : kOob, out, P.P - pA);
        }
    }
    // dW += dz x^T over the tile's pixels: lane reads channel s, unit 4m+r (8 consecutive pixels) of both tiles;
    // MFMA k-slot 4r+jj <-> pixel 8(4m+r) + 4*half + jj for both operands.  Lanes of dead units hold zeros.
#pragma unroll
    for (int m = 0; m < 4; m++)
#pragma unroll
        for (int mo = 0; mo < MO; mo++) {
            const u32x4 dzb = lds_dz[(mo * 16 + s) * kLdsRow + 4 * m + r];
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
                const u32x4 xb = lds_x[(kc * 16 + s) * kLdsRow + 4 * m + r];
                dwacc[mo][kc] = mfma32(as_short4(dzb[0], dzb[1]), as_short4(dzb[2], dzb[3]), as_short4(xb[0], xb[1]), as_short4(xb[2], xb[3]), dwacc[mo][kc]);
                if (TWO) {
                    const u32x4 lowb = lds_low[(mo * 16 + s) * kLdsRow + 4 * m + r];
                    dwacc[mo][kc] = mfma32(as_short4(lowb[0], lowb[1]), as_short4(lowb[2], lowb[3]), as_short4(xb[0], xb[1]), as_short4(xb[2], xb[3]), dwacc[mo][kc]);
                }
            }
        }
}

template <int KC, int MO, int ACT, bool RES, bool RAG>
__device__ __forceinline__ void bwd_body(const Params& P) {
    __shared__ u32x4 lds[kWaves][(KC + (kTwoParts<ACT, RAG> ? 2 : 1) * MO) * 16 * kLdsRow];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane >> 4, s = lane & 15;
    constexpr int CG = 16 * KC, OG = 16 * MO;
    const int g = blockIdx.y;
    const int wg = blockIdx.x;
    const int Cout = P.G * OG;
    const rsrc_t rx = make_rsrc(P.x, extent(P.N, P.xs, P.C, P.P) * 2);
    const rsrc_t rdx = make_rsrc(P.dx, extent(P.N, P.xs, P.C, P.P) * 2);
    const rsrc_t rdy = make_rsrc(P.dy, extent(P.N, P.ys, Cout, P.P) * 2);
    u32x4* lds_x = lds[wave];
    u32x4* lds_dz = lds[wave] + KC * 16 * kLdsRow;

    short4_t wa[MO][KC];  // W[o = mo*16+s][i = kc*16+4r..+3]
    short4_t wt[KC][MO];  // W[o = mo*16+4r+j][i = kc*16+s], j = 0..3
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int kc = 0; kc < KC; kc++) {
            __builtin_memcpy(&wa[mo][kc], P.w + ((g * OG + mo * 16 + s) * CG + kc * 16 + 4 * r), 8);
#pragma unroll
            for (int j = 0; j < 4; j++) wt[kc][mo][j] = (short)P.w[(g * OG + mo * 16 + 4 * r + j) * CG + kc * 16 + s];
        }
    float4_t dwacc[MO][KC];
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int kc = 0; kc < KC; kc++) dwacc[mo][kc] = float4_t{0.f, 0.f, 0.f, 0.f};

    const int tiles_per_group = P.N * P.chunks;
    for (int it = 0; it < P.tiles_per_wave; it++) {
        const int t = (wg * kWaves + wave) * P.tiles_per_wave + it;
        if (t >= tiles_per_group) break;
        const int n = P.chunks == 1 ? t : (int)__umulhi((uint32_t)t, P.magicChunks), chunk = t - n * P.chunks;  // magic overflows for 1
        bwd_tile<KC, MO, ACT, RES, RAG>(P, rx, rdy, rdx, lds_x, lds_dz, n, g, chunk * kTilePx, lane, wa, wt, dwacc);
    }
    // the workgroup's four wavefronts are summed in a fixed order through LDS: one partial per workgroup;
    // the reduction kernel then sums the partials in a fixed order
    __syncthreads();
    float* red = reinterpret_cast<float*>(&lds[0][0]);
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int j = 0; j < 4; j++) red[wave * (OG * CG) + (mo * 16 + 4 * r + j) * CG + kc * 16 + s] = dwacc[mo][kc][j];
    __syncthreads();
    float* part = P.partial + ((long long)g * P.wgs_per_group + wg) * (OG * CG);
    for (int e = threadIdx.x; e < OG * CG; e += 64 * kWaves) {
        float sum = red[e];
#pragma unroll
        for (int wv = 1; wv < kWaves; wv++) sum += red[wv * (OG * CG) + e];
        part[e] = sum;
    }
}

// Cheap activations fit 128 registers (4 wavefronts per SIMD); gelu, clipped exp and planes with a ragged end need more.
template <int KC, int MO, int ACT, bool RES>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_bwd(Params P) {
    bwd_body<KC, MO, ACT, RES, false>(P);
}
template <int KC, int MO, int ACT, bool RES, bool RAG>
__global__ __launch_bounds__(64 * kWaves) void k_bwd_wide(Params P) {
    bwd_body<KC, MO, ACT, RES, RAG>(P);
}
// Groups of 32 channels: two wavefronts per SIMD is what the tile's registers allow, one its LDS with the low parts of dz.
template <int KC, int MO, int ACT, bool RES, bool RAG>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(kTwoParts<ACT, RAG> ? 1 : 2, 2))) void k_bwd_two(Params P) {
    bwd_body<KC, MO, ACT, RES, RAG>(P);
}

// ----------------------------------------------------------------------- m instances on one tile (blocks)
// Expand: every instance reads the same x, instance j reads and writes slice j of y and dy, dx is the instances' sum.
// Reduce: instance j reads and writes slice j of x and dx, y is the sum, every instance reads the same dy.  Bound by
// memory, like the kernels above: a wavefront walks over the instances of ONE tile, so the shared tensor crosses the bus
// once and not m times, and the sum is taken in fp32 in instance order in registers and rounded once; the instances as
// launches of their own wrote m rounded parts and added them in one more launch.  The loads of instance j + 1 are issued
// as soon as the registers of instance j's are free.  N=64, 56x56, a step, launches
// of their own / here: 64 => 128 channels 84.6 / 46.8 us, 128 => 64 85.4 / 50.5, 64 => 256 159 / 82.6, 256 => 64 165 / 82.1.

// dW accumulators of the instances live in LDS between tiles (m of them in registers would have to be indexed by a
// constant); rows of the transposers are not padded but swizzled (unit ^ row), which leaves room for two instances'
// accumulators at four workgroups per compute unit.
constexpr int kDead = -0x7fffffff - 1;  // plus any offset inside a tensor: still outside
// Wavefronts per SIMD that the registers of the backward kernel leave room for (expand with relu and residual: 173 registers;
// held to three wavefronts it spills four and takes 28.1 instead of 26.3 us, 64 => 128).
constexpr int multi_waves(int act, bool res, bool expand, bool rag) { return act == 2 || rag || (res && expand) ? 2 : 3; }
constexpr int tiles_multi(int act, bool rag) { return rag && (act == 2 || act == 3) ? 3 : 2; }  // x, dz, its low parts
constexpr int lds_pieces_multi(int KC, int m, int tiles) { return kWaves * (tiles * KC * 16 * 16 + m * KC * KC * 64); }
__device__ __forceinline__ int swz(int row, int unit) { return row * 16 + (unit ^ (row & 15)); }

template <int KC, int ACT, bool RES, bool EXPAND, bool RAG>
__global__ __launch_bounds__(64 * kWaves) void k_fwd_multi(Params P, Instances I) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk = blockIdx.x * kWaves + wave;
    if (chunk >= P.chunks) return;
    const int g = blockIdx.y, n = blockIdx.z;
    const int r = lane >> 4, s = lane & 15;
    constexpr int CG = 16 * KC;
    const int p0 = chunk * kTilePx, p = p0 + 8 * s;
    const int dh = P.dh[g], dw = P.dw[g], off = dh * P.W + dw;
    const int xelems = P.N * P.xs;
    const rsrc_t rx = make_rsrc(P.x, xelems * 2);
    const rsrc_t ry = make_rsrc(P.y, P.N * P.ys * 2);
    const TileMask tm = tile_mask(p0, lane, P, dh, dw);
    const bool live = p < P.P;
    const u32x4 msk = mask_of(live ? unit_bits(tm, s) : 0u);
    const int xg = (n * P.xs + g * CG * P.P) * 2, yg = (n * P.ys + g * CG * P.P) * 2;
    // (a lane without pixels starts beyond every tensor and stays there: one offset per tensor, rows are added to it)
    const int px = live ? (4 * r * P.P + p) * 2 : kDead, pxs = live ? px + off * 2 : kDead;

    short4_t wa[KC][KC];
    u32x4 xs[KC][4], xr[KC][4];
    short4_t b[KC][8];
    auto load_w = [&](int j) {
#pragma unroll
        for (int mo = 0; mo < KC; mo++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++) __builtin_memcpy(&wa[mo][kc], I.w[j] + ((g * CG + mo * 16 + s) * CG + kc * 16 + 4 * r), 8);
    };
    auto load_x = [&](int j) {
        const int xj = xg + j * I.slice * 2;
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int k = 0; k < 4; k++) xs[kc][k] = bload16(rx, pxs + (xj + (kc * 16 + k) * P.P * 2));
        if (tile_near_ends(xj / 2, xj / 2 + (CG - 1) * P.P, p0, off, xelems)) {
#pragma unroll
            for (int kc = 0; kc < KC; kc++)
#pragma unroll
                for (int k = 0; k < 4; k++)
                    reload_if_partial(xs[kc][k], rx, pxs + (xj + (kc * 16 + k) * P.P * 2), xelems * 2);
        }
    };
    auto load_res = [&](int j) {
        const int xj = xg + j * I.slice * 2;
#pragma unroll
        for (int mo = 0; mo < KC; mo++)
#pragma unroll
            for (int k = 0; k < 4; k++) {
                xr[mo][k] = bload16_nt(rx, px + (xj + (mo * 16 + k) * P.P * 2));
                pin(xr[mo][k]);
            }
        if (RAG && tile_near_ends(xj / 2, xj / 2 + (CG - 1) * P.P, p0, 0, xelems)) {
#pragma unroll
            for (int mo = 0; mo < KC; mo++)
#pragma unroll
                for (int k = 0; k < 4; k++) reload_if_partial(xr[mo][k], rx, px + (xj + (mo * 16 + k) * P.P * 2), xelems * 2);
        }
    };
    auto gather_x = [&]() {
#pragma unroll
        for (int kc = 0; kc < KC; kc++) {
#pragma unroll
            for (int k = 0; k < 4; k++) xs[kc][k] = xs[kc][k] & msk;
            gather_all(xs[kc], b[kc]);
        }
    };
    load_w(0);
    load_x(0);
    if (RES && EXPAND) load_res(0);
    float4_t sum[EXPAND ? 1 : KC][8];
    if (!EXPAND) {
#pragma unroll
        for (int mo = 0; mo < KC; mo++)
#pragma unroll
            for (int q = 0; q < 8; q++) sum[EXPAND ? 0 : mo][q] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    if (EXPAND) gather_x();
    for (int j = 0; j < I.m; j++) {
        if (!EXPAND) {
            gather_x();
            if (RES) load_res(j);  // (nearly all of it has just come as the shifted x)
        }
        float4_t acc[KC][8];
#pragma unroll
        for (int mo = 0; mo < KC; mo++)
#pragma unroll
            for (int q = 0; q < 8; q++) {
                acc[mo][q] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < KC; kc++) acc[mo][q] = mfma16(wa[mo][kc], b[kc][q], acc[mo][q]);
            }
        if (j + 1 < I.m) {
            load_w(j + 1);
            if (!EXPAND) load_x(j + 1);
        }
#pragma unroll
        for (int mo = 0; mo < KC; mo++)
#pragma unroll
            for (int k = 0; k < 4; k++) {
                float v[8];
#pragma unroll
                for (int q = 0; q < 8; q++) v[q] = act_apply<ACT>(P, acc[mo][q][k]);
                if (RES) {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        v[2 * e] += lo_f32(xr[mo][k][e]);
                        v[2 * e + 1] += hi_f32(xr[mo][k][e]);
                    }
                }
                if (!EXPAND) {
#pragma unroll
                    for (int q = 0; q < 8; q++) v[q] = sum[EXPAND ? 0 : mo][q][k] += v[q];
                }
                if (EXPAND || j + 1 == I.m) {
                    u32x4 out;
#pragma unroll
                    for (int e = 0; e < 4; e++) out[e] = pack_bf16(v[2 * e], v[2 * e + 1]);
                    store_unit<RAG>(ry, px + (yg + ((EXPAND ? j * I.slice : 0) + (mo * 16 + k) * P.P) * 2), out, P.P - p);
                }
            }
    }
}

template <int KC, int ACT, bool RES, bool EXPAND, bool RAG>
__device__ __forceinline__ void bwd_multi_body(const Params& P, const Instances& I, u32x4* lds) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane >> 4, s = lane & 15;
    constexpr int CG = 16 * KC;
    const int g = blockIdx.y, wg = blockIdx.x;
    const int dh = P.dh[g], dw = P.dw[g], off = dh * P.W + dw;
    const int dyelems = P.N * P.ys;
    const rsrc_t rx = make_rsrc(P.x, P.N * P.xs * 2);
    const rsrc_t rdx = make_rsrc(P.dx, P.N * P.xs * 2);
    const rsrc_t rdy = make_rsrc(P.dy, dyelems * 2);
    // LDS of the wavefront: x rows | dz rows (| their low parts) | dW accumulators of the instances
    constexpr bool TWO = kTwoParts<ACT, RAG>;
    constexpr int TILES = tiles_multi(ACT, RAG);
    u32x4* const lds_x = lds + wave * (TILES * KC * 16 * 16);
    u32x4* const lds_dz = lds_x + KC * 16 * 16;
    u32x4* const lds_low = lds_dz + KC * 16 * 16;
    u32x4* const lds_dw = lds + kWaves * (TILES * KC * 16 * 16) + wave * (I.m * KC * KC * 64);
    for (int j = 0; j < I.m * KC * KC; j++) lds_dw[j * 64 + lane] = u32x4{0u, 0u, 0u, 0u};

    short4_t wa[KC][KC];  // W[o = mo*16+s][i = kc*16+4r..+3]
    short4_t wt[KC][KC];  // W[o = mo*16+4r+j][i = kc*16+s], j = 0..3
    auto load_w = [&](int j) {
        const uint16_t* w = I.w[j];
#pragma unroll
        for (int mo = 0; mo < KC; mo++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
                __builtin_memcpy(&wa[mo][kc], w + ((g * CG + mo * 16 + s) * CG + kc * 16 + 4 * r), 8);
#pragma unroll
                for (int k = 0; k < 4; k++) wt[kc][mo][k] = (short)w[(g * CG + mo * 16 + 4 * r + k) * CG + kc * 16 + s];
            }
    };
    const int tiles_per_group = P.N * P.chunks;
    for (int it = 0; it < P.tiles_per_wave; it++) {
        const int t = (wg * kWaves + wave) * P.tiles_per_wave + it;
        if (t >= tiles_per_group) break;
        const int n = P.chunks == 1 ? t : (int)__umulhi((uint32_t)t, P.magicChunks), chunk = t - n * P.chunks;
        const int p0 = chunk * kTilePx, pA = p0 + 8 * s;
        const bool liveA = pA < P.P;
        const int xg = (n * P.xs + g * CG * P.P) * 2, dyg = (n * P.ys + g * CG * P.P) * 2;
        const TileMask tm = tile_mask(p0, lane, P, -dh, -dw);
        const u32x4 msk = mask_of(liveA ? unit_bits(tm, s) : 0u);
        const int px = liveA ? (4 * r * P.P + pA) * 2 : kDead, pxs = liveA ? px - off * 2 : kDead;
        u32x4 xa[KC][4], dya[KC][4], dyu[KC][4];
        short4_t xq[KC][8];
        auto load_x = [&](int j) {
            const int xj = xg + j * I.slice * 2;
#pragma unroll
            for (int kc = 0; kc < KC; kc++)
#pragma unroll
                for (int k = 0; k < 4; k++) xa[kc][k] = bload16_nt(rx, px + (xj + (kc * 16 + k) * P.P * 2));
            const int xelems = P.N * P.xs;
            if (RAG && tile_near_ends(xj / 2, xj / 2 + (CG - 1) * P.P, p0, 0, xelems)) {
#pragma unroll
                for (int kc = 0; kc < KC; kc++)
#pragma unroll
                    for (int k = 0; k < 4; k++) reload_if_partial(xa[kc][k], rx, px + (xj + (kc * 16 + k) * P.P * 2), xelems * 2);
            }
        };
        auto load_dy = [&](int j) {
            const int dyj = dyg + j * I.slice * 2;
#pragma unroll
            for (int mo = 0; mo < KC; mo++)
#pragma unroll
                for (int k = 0; k < 4; k++) dya[mo][k] = bload16(rdy, pxs + (dyj + (mo * 16 + k) * P.P * 2));
            if (tile_near_ends(dyj / 2, dyj / 2 + (CG - 1) * P.P, p0, -off, dyelems)) {
#pragma unroll
                for (int mo = 0; mo < KC; mo++)
#pragma unroll
                    for (int k = 0; k < 4; k++)
                        reload_if_partial(dya[mo][k], rdy, pxs + (dyj + (mo * 16 + k) * P.P * 2), dyelems * 2);
            }
        };
        auto load_res = [&](int j) {
            const int dyj = dyg + j * I.slice * 2;
#pragma unroll
            for (int kc = 0; kc < KC; kc++)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    dyu[kc][k] = bload16_nt(rdy, px + (dyj + (kc * 16 + k) * P.P * 2));
                    pin(dyu[kc][k]);
                }
            if (RAG && tile_near_ends(dyj / 2, dyj / 2 + (CG - 1) * P.P, p0, 0, dyelems)) {
#pragma unroll
                for (int kc = 0; kc < KC; kc++)
#pragma unroll
                    for (int k = 0; k < 4; k++) reload_if_partial(dyu[kc][k], rdy, px + (dyj + (kc * 16 + k) * P.P * 2), dyelems * 2);
            }
        };
        auto mask_dy = [&]() {
#pragma unroll
            for (int mo = 0; mo < KC; mo++)
#pragma unroll
                for (int k = 0; k < 4; k++) dya[mo][k] = dya[mo][k] & msk;
        };
        auto take_x = [&]() {  // x -> LDS rows (channel 4r+k, unit s) and -> MFMA operands
            if (RAG) {
                const u32x4 own = own_pixels(P.P - pA);
#pragma unroll
                for (int kc = 0; kc < KC; kc++)
#pragma unroll
                    for (int k = 0; k < 4; k++) xa[kc][k] = xa[kc][k] & own;
            }
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
#pragma unroll
                for (int k = 0; k < 4; k++) lds_x[swz(kc * 16 + 4 * r + k, s)] = xa[kc][k];
                gather_all(xa[kc], xq[kc]);
            }
        };
        load_w(0);
        load_x(0);
        load_dy(0);
        if (RES && !EXPAND) load_res(0);
        float4_t dxs[KC][8];
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int q = 0; q < 8; q++) dxs[kc][q] = float4_t{0.f, 0.f, 0.f, 0.f};
        if (EXPAND) take_x();
        else mask_dy();
        for (int j = 0; j < I.m; j++) {
            if (EXPAND) mask_dy();
            else {
                take_x();
                if (j + 1 < I.m) load_x(j + 1);
            }
            short4_t dzq[KC][8];
#pragma unroll
            for (int mo = 0; mo < KC; mo++) {
                u32x4 dzrow[4], dzlow[4];
                constexpr int QS = 2;
#pragma unroll
                for (int h = 0; h < 8 / QS; h++) {
                    float4_t z[QS];
#pragma unroll
                    for (int q = 0; q < QS; q++) {
                        z[q] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int kc = 0; kc < KC; kc++) z[q] = mfma16(wa[mo][kc], xq[kc][QS * h + q], z[q]);
                    }
                    float d[QS][4];
#pragma unroll
                    for (int k = 0; k < 4; k++) {
#pragma unroll
                        for (int q = 0; q < QS; q += 2) {
                            const uint32_t w = dya[mo][k][(QS * h + q) / 2];
                            d[q][k] = act_dz<ACT>(P, z[q][k], lo_f32(w));
                            d[q + 1][k] = act_dz<ACT>(P, z[q + 1][k], hi_f32(w));
                            const uint32_t hi = pack_bf16(d[q][k], d[q + 1][k]);
                            dzrow[k][(QS * h + q) / 2] = hi;
                            if (TWO) dzlow[k][(QS * h + q) / 2] = pack_bf16(d[q][k] - lo_f32(hi), d[q + 1][k] - hi_f32(hi));
                        }
                    }
#pragma unroll
                    for (int q = 0; q < QS; q++) dzq[mo][QS * h + q] = pack4(d[q][0], d[q][1], d[q][2], d[q][3]);
                    __builtin_amdgcn_sched_barrier(0);  // (the steps one after the other: side by side their registers do not fit)
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    lds_dz[swz(mo * 16 + 4 * r + k, s)] = dzrow[k];
                    if (TWO) lds_low[swz(mo * 16 + 4 * r + k, s)] = dzlow[k];
                }
            }
            // (the unshifted dy only now: nearly all of it has just come as the shifted one, and its registers were needed above)
            if (EXPAND && RES) load_res(j);
            if (EXPAND && j + 1 < I.m) load_dy(j + 1);
#pragma unroll
            for (int kc = 0; kc < KC; kc++) {
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    if (!EXPAND) dxs[kc][q] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int mo = 0; mo < KC; mo++) dxs[kc][q] = mfma16(wt[kc][mo], dzq[mo][q], dxs[kc][q]);
                }
                if (TWO) {
#pragma unroll
                    for (int mo = 0; mo < KC; mo++) {
                        u32x4 v[4];
                        short4_t low[8];
#pragma unroll
                        for (int k = 0; k < 4; k++) v[k] = lds_low[swz(mo * 16 + 4 * r + k, s)];
                        gather_all(v, low);
#pragma unroll
                        for (int q = 0; q < 8; q++) dxs[kc][q] = mfma16(wt[kc][mo], low[q], dxs[kc][q]);
                    }
                }
                if (RES) {
#pragma unroll
                    for (int k = 0; k < 4; k++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            dxs[kc][2 * e][k] += lo_f32(dyu[kc][k][e]);
                            dxs[kc][2 * e + 1][k] += hi_f32(dyu[kc][k][e]);
                        }
                }
            }
            if (j + 1 < I.m) load_w(j + 1);
            if (!EXPAND || j + 1 == I.m) {
#pragma unroll
                for (int kc = 0; kc < KC; kc++)
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        u32x4 out;
#pragma unroll
                        for (int e = 0; e < 4; e++) out[e] = pack_bf16(dxs[kc][2 * e][k], dxs[kc][2 * e + 1][k]);
                        store_unit<RAG>(rdx, px + (xg + ((EXPAND ? 0 : j * I.slice) + (kc * 16 + k) * P.P) * 2), out, P.P - pA);
                    }
            }
            // dW_j += dz x^T over the tile's pixels (the operand layout of bwd_tile)
#pragma unroll
            for (int mo = 0; mo < KC; mo++)
#pragma unroll
                for (int kc = 0; kc < KC; kc++) {
                    u32x4* const at = lds_dw + ((j * KC + mo) * KC + kc) * 64 + lane;
                    const u32x4 held = *at;
                    float4_t a;
                    __builtin_memcpy(&a, &held, 16);
#pragma unroll
                    for (int m4 = 0; m4 < 4; m4++)
                        a = mfma32(lds_dz[swz(mo * 16 + s, 4 * m4 + r)], lds_x[swz(kc * 16 + s, 4 * m4 + r)], a);
                    if (TWO) {
#pragma unroll
                        for (int m4 = 0; m4 < 4; m4++)
                            a = mfma32(lds_low[swz(mo * 16 + s, 4 * m4 + r)], lds_x[swz(kc * 16 + s, 4 * m4 + r)], a);
                    }
                    u32x4 put;
                    __builtin_memcpy(&put, &a, 16);
                    *at = put;
                }
        }
    }
    // the four wavefronts' accumulators are summed in a fixed order: one partial per workgroup and instance
    __syncthreads();
    const float* acc = reinterpret_cast<const float*>(lds + kWaves * (TILES * KC * 16 * 16));
    const int per_wave = I.m * KC * KC * 256;
    for (int e = threadIdx.x; e < per_wave; e += 64 * kWaves) {
        float sum = acc[e];
#pragma unroll
        for (int wv = 1; wv < kWaves; wv++) sum += acc[wv * per_wave + e];
        // e = (((j * KC + mo) * KC + kc) * 64 + lane) * 4 + k: output mo*16 + 4*(lane/16) + k, input kc*16 + lane%16
        const int k = e & 3, l = (e >> 2) & 63, b = e >> 8;
        const int kc = b % KC, mo = (b / KC) % KC, j = b / (KC * KC);
        float* part = P.partial + j * I.part_stride + ((long long)g * P.wgs_per_group + wg) * (CG * CG);
        part[(mo * 16 + 4 * (l >> 4) + k) * CG + kc * 16 + (l & 15)] = sum;
    }
}

template <int KC, int ACT, bool RES, bool EXPAND, bool RAG>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(multi_waves(ACT, RES, EXPAND, RAG), multi_waves(ACT, RES, EXPAND, RAG)))) void k_bwd_multi(Params P, Instances I) {
    extern __shared__ __align__(16) u32x4 lds_multi[];
    bwd_multi_body<KC, ACT, RES, EXPAND, RAG>(P, I, lds_multi);
}

// dW[g][e] = sum over the group's partials in a fixed order (grid.z: the instances of a block).  Bound by the launch itself: a
// workgroup takes 32 elements (one 128-byte line of every partial; OG * CG is a multiple of 256) and its 1024 threads 128
// partials at a time, 16 bytes each, up to four loads in flight; eight lanes of a wavefront are added by lane exchanges, the
// sixteen wavefronts through LDS with one barrier.  4 x 200 partials of 256 elements take 4.2-4.5 us, two instances' 4.2; with
// eight elements per workgroup and a tree of seven barriers it was 4.2-4.6 (the step 0.1 us longer).
__device__ __forceinline__ void dw_reduce_body(const float* __restrict__ partial, float* __restrict__ dw, int n_partials, int elems) {
    __shared__ float4_t red[16][8];
    const int g = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 7, row = wave * 8 + (lane >> 3);
    const float* src = partial + (long long)g * n_partials * elems + blockIdx.x * 32 + col * 4;
    float4_t sum = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = row; k0 < n_partials; k0 += 512) {
        float4_t v[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int k = k0 + 128 * i;
            v[i] = float4_t{0.f, 0.f, 0.f, 0.f};
            if (k < n_partials) __builtin_memcpy(&v[i], src + (long long)k * elems, 16);
        }
        sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
        sum[e] += __shfl_xor(sum[e], 8);
        sum[e] += __shfl_xor(sum[e], 16);
        sum[e] += __shfl_xor(sum[e], 32);
    }
    if (lane < 8) red[wave][lane] = sum;
    __syncthreads();
    if (threadIdx.x < 32) {
        float total = 0.f;
#pragma unroll
        for (int w = 0; w < 16; w++) total += reinterpret_cast<const float*>(red[w])[threadIdx.x];
        dw[(long long)g * elems + blockIdx.x * 32 + threadIdx.x] = total;
    }
}
__global__ __launch_bounds__(1024) void k_dw_reduce(const float* __restrict__ partial, float* __restrict__ dw, int n_partials, int elems) {
    dw_reduce_body(partial, dw, n_partials, elems);
}
__global__ __launch_bounds__(1024) void k_dw_reduce_multi(const float* __restrict__ partial, Instances I, int n_partials, int elems) {
    dw_reduce_body(partial + blockIdx.z * I.part_stride, I.dw[blockIdx.z], n_partials, elems);
}

}  // namespace

bool supported(int KC, int MO) { return KC == MO && (KC == 1 || KC == 2); }

template <int ACT, bool RES>
static void launch_fwd(const Params& P, int W, hipStream_t s) {
    const dim3 grid((unsigned)((P.chunks + kWaves - 1) / kWaves), (unsigned)P.G, (unsigned)P.N), block(64 * kWaves);
    if (!P.total_tiles) return;
    if (P.P % 8) {
        if (W == 2) CANVAS_LAUNCH((k_fwd<2, 2, ACT, RES, true>), grid, block, 0, s, P);
        else CANVAS_LAUNCH((k_fwd<1, 1, ACT, RES, true>), grid, block, 0, s, P);
    } else if (W == 2) CANVAS_LAUNCH((k_fwd<2, 2, ACT, RES, false>), grid, block, 0, s, P);
    else CANVAS_LAUNCH((k_fwd<1, 1, ACT, RES, false>), grid, block, 0, s, P);
}
// Planes that the backward instances for ragged planes take: ragged ones, and narrow ones for the two parts of dz.
template <int ACT>
static bool ragged_bwd(const Params& P) { return P.P % 8 || (P.W < 8 && kTwoParts<ACT, true>); }
template <int ACT, bool RES>
static void launch_bwd(const Params& P, int W, hipStream_t s) {
    const dim3 grid((unsigned)P.wgs_per_group, (unsigned)P.G), block(64 * kWaves);
    if (!P.total_tiles) return;
    if (ragged_bwd<ACT>(P)) {
        if (W == 2) CANVAS_LAUNCH((k_bwd_two<2, 2, ACT, RES, true>), grid, block, 0, s, P);
        else CANVAS_LAUNCH((k_bwd_wide<1, 1, ACT, RES, true>), grid, block, 0, s, P);
    } else if (W == 2) CANVAS_LAUNCH((k_bwd_two<2, 2, ACT, RES, false>), grid, block, 0, s, P);
    else if (ACT == 2 || ACT == 3) CANVAS_LAUNCH((k_bwd_wide<1, 1, ACT, RES, false>), grid, block, 0, s, P);
    else CANVAS_LAUNCH((k_bwd<1, 1, ACT, RES>), grid, block, 0, s, P);
}

#define SGFC_DISPATCH(fn)                                                        \
    switch (P.act) {                                                             \
    case kActNone: P.residual ? fn<kActNone, true>(P, KC, s) : fn<kActNone, false>(P, KC, s); break; \
    case 0: P.residual ? fn<0, true>(P, KC, s) : fn<0, false>(P, KC, s); break;          \
    case 1: P.residual ? fn<1, true>(P, KC, s) : fn<1, false>(P, KC, s); break;          \
    case 2: P.residual ? fn<2, true>(P, KC, s) : fn<2, false>(P, KC, s); break;          \
    default: P.residual ? fn<3, true>(P, KC, s) : fn<3, false>(P, KC, s); break;         \
    }

void forward(const Params& P, int KC, int MO, hipStream_t s) {
    (void)MO;
    SGFC_DISPATCH(launch_fwd)
}

void backward(const Params& P, int KC, int MO, hipStream_t s) {
    (void)MO;
    SGFC_DISPATCH(launch_bwd)
}

template <int ACT, bool RES, bool RAG>
static void launch_fwd_of(const Params& P, const Instances& I, bool expand, hipStream_t s) {
    const dim3 grid((unsigned)((P.chunks + kWaves - 1) / kWaves), (unsigned)P.G, (unsigned)P.N);
    if (!P.total_tiles) return;
    if (expand) CANVAS_LAUNCH((k_fwd_multi<1, ACT, RES, true, RAG>), grid, dim3(64 * kWaves), 0, s, P, I);
    else CANVAS_LAUNCH((k_fwd_multi<1, ACT, RES, false, RAG>), grid, dim3(64 * kWaves), 0, s, P, I);
}
template <int ACT, bool RES, bool RAG>
static void launch_bwd_of(const Params& P, const Instances& I, bool expand, hipStream_t s) {
    const dim3 grid((unsigned)P.wgs_per_group, (unsigned)P.G);
    if (!P.total_tiles) return;
    const size_t lds = (size_t)lds_pieces_multi(1, I.m, tiles_multi(ACT, RAG)) * 16;
    if constexpr (kTwoParts<ACT, RAG>) {  // (80 KB for eight instances)
        constexpr int most = lds_pieces_multi(1, kMaxInstances, tiles_multi(ACT, RAG)) * 16;
        static std::atomic<uint64_t> asked[2];
        if (expand) allow_lds(asked[0], (const void*)k_bwd_multi<1, ACT, RES, true, RAG>, most);
        else allow_lds(asked[1], (const void*)k_bwd_multi<1, ACT, RES, false, RAG>, most);
    }
    if (expand) CANVAS_LAUNCH((k_bwd_multi<1, ACT, RES, true, RAG>), grid, dim3(64 * kWaves), lds, s, P, I);
    else CANVAS_LAUNCH((k_bwd_multi<1, ACT, RES, false, RAG>), grid, dim3(64 * kWaves), lds, s, P, I);
}

template <int ACT, bool RES>
static void launch_fwd_multi(const Params& P, const Instances& I, bool expand, hipStream_t s) {
    P.P % 8 ? launch_fwd_of<ACT, RES, true>(P, I, expand, s) : launch_fwd_of<ACT, RES, false>(P, I, expand, s);
}
template <int ACT, bool RES>
static void launch_bwd_multi(const Params& P, const Instances& I, bool expand, hipStream_t s) {
    ragged_bwd<ACT>(P) ? launch_bwd_of<ACT, RES, true>(P, I, expand, s) : launch_bwd_of<ACT, RES, false>(P, I, expand, s);
}

#define SGFC_DISPATCH_MULTI(fn)                                                  \
    switch (P.act) {                                                             \
    case kActNone: P.residual ? fn<kActNone, true>(P, I, expand, s) : fn<kActNone, false>(P, I, expand, s); break; \
    case 0: P.residual ? fn<0, true>(P, I, expand, s) : fn<0, false>(P, I, expand, s); break;          \
    case 1: P.residual ? fn<1, true>(P, I, expand, s) : fn<1, false>(P, I, expand, s); break;          \
    case 2: P.residual ? fn<2, true>(P, I, expand, s) : fn<2, false>(P, I, expand, s); break;          \
    default: P.residual ? fn<3, true>(P, I, expand, s) : fn<3, false>(P, I, expand, s); break;         \
    }

void forward_multi(const Params& P, const Instances& I, bool expand, hipStream_t s) { SGFC_DISPATCH_MULTI(launch_fwd_multi) }
void backward_multi(const Params& P, const Instances& I, bool expand, hipStream_t s) { SGFC_DISPATCH_MULTI(launch_bwd_multi) }

void dw_reduce(const float* partial, float* dw, int G, int n_partials, int elems, hipStream_t s) {
    CANVAS_LAUNCH(k_dw_reduce, dim3((unsigned)(elems / 32), (unsigned)G), dim3(1024), 0, s, partial, dw, n_partials, elems);
}
void dw_reduce_multi(const float* partial, const Instances& I, int G, int n_partials, int elems, hipStream_t s) {
    CANVAS_LAUNCH(k_dw_reduce_multi, dim3((unsigned)(elems / 32), (unsigned)G, (unsigned)I.m), dim3(1024), 0, s, partial, I, n_partials, elems);
}

}  // namespace sgfc
}  // namespace canvas
