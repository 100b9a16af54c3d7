// v = x (*|+) shift(act(z)) and its adjoint, one thread per 8 consecutive pixels of one channel
// (16-byte bf16 accesses).  The shift is an address offset plus a zero mask applied AFTER the
// activation (Shift zero-fills its own output, whatever act(0) is).  Memory-bound: forward reads x, z
// and writes v; backward reads dv, x, z and writes dz and dx1, each element once.
#include "ufc_kernels.hpp"

#include <type_traits>

#include "launch.hpp"
#include "ufc_device.hpp"

namespace canvas {
namespace ufc {

namespace {

struct Unit {
    int plane, p, dh, dw, nvalid;
    bool live;
};
__device__ __forceinline__ Unit decode(const MidParams& P) {
    Unit u;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long total = (long long)P.N * P.C * P.upi;
    u.live = idx < total;
    const uint32_t i = u.live ? (uint32_t)idx : 0u;
    int nc = (int)div_magic(i, P.magicUpi), unit = (int)i - nc * P.upi;
    if (unit < 0) {  // (the multiplier is exact below 2^32 / upi and one too high at most beyond)
        unit += P.upi;
        nc--;
    }
    u.p = unit * 8;
    u.plane = nc * P.P;
    const int c = nc % P.C;
    u.dh = u.dw = 0;
    for (int k = 0; k < P.nslices; k++)
        if (c >= P.c0[k] && c < P.c1[k]) {
            u.dh = P.dh[k];
            u.dw = P.dw[k];
        }
    u.nvalid = min(8, P.P - u.p);
    return u;
}

template <int ACT, int BIN>
__global__ __launch_bounds__(256) void k_mid_fwd(MidParams P) {
    const Unit u = decode(P);
    if (!u.live) return;
    const int bytes = P.N * P.C * P.P * 2;
    const rsrc_t rx = make_rsrc(P.x, bytes), rz = make_rsrc(P.z, bytes), rv = make_rsrc(P.v, bytes);
    const int off = u.dh * P.W + u.dw;
    const uint32_t bits = shift_bits(P, u.p, u.dh, u.dw);
    float x[8], z[8], v[8];
    unpack8(load8(rx, u.plane + u.p, bytes), x);
    unpack8(load8(rz, u.plane + u.p + off, bytes), z);
#pragma unroll
    for (int q = 0; q < 8; q++) {
        float t = act_apply<ACT>(z[q]);
        t = ((bits >> q) & 1u) ? t : 0.f;
        v[q] = BIN ? x[q] * t : x[q] + t;
    }
    store8(rv, P.v, u.plane + u.p, v, u.nvalid);
}

// The adjoint, written from the side of p:
//     dx1(p) = dv(p) * t(p)    with t(p) = act(z(p + d)), zero where p + d leaves the image;  dv(p) for a sum
//     dz(p + d) = act'(z(p + d)) * dv(p) * x(p)
// Everything then needs dv and x at p and z at p + d, each once, and act at one point; dz is stored at p + d (an unaligned
// 16-byte store, as planes that are no multiple of 8 pixels have anyway).  p -> p + d is a bijection of the plane's flat
// pixel indices except at its two ends: targets outside the plane are dropped, and the thread that owns a pixel without a
// source writes its zero.  A target that lies in the plane but in another image row receives zero.
// (Gathered from the side of dz, a shifted channel read dv and z at two points each and evaluated act twice per pixel.
// With half of the channels shifted, gelu and product: N=128 C=64 56x56 53.7 -> 43.7 us = 5.9 TB/s, C=256 14x14 17.2 -> 14.9,
// C=512 7x7 11.9 -> 9.4.  As the end of the data gradient that produces dv, without dv in memory, it was slower: 71 us
// against 44 + 23 at C=64, 36 against 15 + 14 at C=256; the tile's registers leave two or three wavefronts per SIMD.)
template <int ACT, int BIN>
__global__ __launch_bounds__(256) void k_mid_bwd(MidParams P) {
    const Unit u = decode(P);
    if (!u.live) return;
    const int bytes = P.N * P.C * P.P * 2;
    const rsrc_t rx = make_rsrc(P.x, bytes), rz = make_rsrc(P.z, bytes), rdv = make_rsrc(P.dv, bytes);
    const rsrc_t rdz = make_rsrc(P.dz, bytes), rdx = make_rsrc(P.dx1, bytes);
    // a shift by the image's size or more: no pixel has a target
    const bool none = u.dh >= P.H || u.dh <= -P.H || u.dw >= P.W || u.dw <= -P.W;
    const int off = none ? P.P : u.dh * P.W + u.dw;
    const int q0 = u.p + off, e = u.plane + u.p;
    float dv[8], z[8], x[8], dx1[8], dz[8];
    unpack8(load8(rdv, e, bytes), dv);
    unpack8(load8(rz, q0 < P.P && q0 + 7 >= 0 ? e + off : kOob / 2, bytes), z);
    if (BIN) unpack8(load8(rx, e, bytes), x);
    const uint32_t bits = none ? 0u : ((u.dh | u.dw) != 0 ? shift_bits(P, u.p, u.dh, u.dw) : 0xffu);
#pragma unroll
    for (int q = 0; q < 8; q++) {
        float t, d;
        act_both<ACT>(z[q], t, d);
        const bool in = (bits >> q) & 1u;
        dx1[q] = BIN ? dv[q] * (in ? t : 0.f) : dv[q];
        dz[q] = (in ? (BIN ? dv[q] * x[q] : dv[q]) : 0.f) * d;
    }
    store8(rdx, P.dx1, e, dx1, u.nvalid);
    if (u.nvalid == 8 && q0 >= 0 && q0 + 8 <= P.P) {
        store8(rdz, P.dz, e + off, dz, 8, off == 0);  // (unaligned stores leave partial lines: kept in the cache until whole)
    } else {
#pragma unroll
        for (int q = 0; q < 8; q++)
            if (q < u.nvalid && (unsigned)(q0 + q) < (unsigned)P.P) P.dz[e + off + q] = (uint16_t)(pack_bf16(dz[q], 0.f) & 0xffffu);
    }
    if (off != 0 && (u.p - off < 0 || u.p + u.nvalid - 1 - off >= P.P)) {
        for (int q = 0; q < u.nvalid; q++)
            if ((unsigned)(u.p + q - off) >= (unsigned)P.P) {
                float t, d;
                act_both<ACT>(__uint_as_float((uint32_t)P.z[e + q] << 16), t, d);
                P.dz[e + q] = (uint16_t)(pack_bf16(0.f * d, 0.f) & 0xffffu);
            }
    }
}

// The activation's adjoint as the chain programs have it: relu selects (an infinite or overflowing gradient does not pass where the input is not positive).
template <int ACT>
__device__ __forceinline__ float through_act(float x, float d, float g) {
    if constexpr (ACT == 0) return x > 0.f ? g : 0.f;
    else return d * g;
}

// The adjoint of y = x (*|+) shift(act(x)), where x is both operands (MidParams: x, dv = dy, dx1 = dx):
//     dx(p) = dv(p) t(p) + act'(x(p)) dv(p - d) x(p - d),  t(p) = act(x(p + d)), either term zero where its other pixel leaves the image
// (for a sum dv(p) + act'(x(p)) dv(p - d)).  Reads of x and dv at three pixels, two of them unaligned and served by the caches; bound by
// the vector unit (two evaluations of the activation).  As programs of the fused-chain kernels, gelu, half of the channels shifted,
// product, 128x64 planes of 56x56: backward 121.6 us, now 36.7 (4.2 TB/s of what it must move).
template <int ACT, int BIN>
__global__ __launch_bounds__(256) void k_self_bwd(MidParams P) {
    const Unit u = decode(P);
    if (!u.live) return;
    const int bytes = P.N * P.C * P.P * 2;
    const rsrc_t rx = make_rsrc(P.x, bytes), rdv = make_rsrc(P.dv, bytes), rdx = make_rsrc(P.dx1, bytes);
    const bool none = u.dh >= P.H || u.dh <= -P.H || u.dw >= P.W || u.dw <= -P.W;
    const int off = none ? 0 : u.dh * P.W + u.dw, e = u.plane + u.p;
    float x[8], dv[8], dx[8];
    unpack8(load8(rx, e, bytes), x);
    unpack8(load8(rdv, e, bytes), dv);
    if (!none && (u.dh | u.dw) == 0) {
#pragma unroll
        for (int q = 0; q < 8; q++) {
            float t, d;
            act_both<ACT>(x[q], t, d);
            const float through = through_act<ACT>(x[q], d, BIN ? dv[q] * x[q] : dv[q]);
            dx[q] = BIN ? dv[q] * t + through : dv[q] + through;
        }
    } else {
        float xf[8], xs[8], dvs[8];  // x at p + d, x and dv at p - d
        if (BIN) unpack8(load8(rx, e + off, bytes), xf);
        if (BIN) unpack8(load8(rx, e - off, bytes), xs);
        unpack8(load8(rdv, e - off, bytes), dvs);
        const uint32_t to = none ? 0u : shift_bits(P, u.p, u.dh, u.dw), from = none ? 0u : shift_bits(P, u.p, -u.dh, -u.dw);
#pragma unroll
        for (int q = 0; q < 8; q++) {
            float t = 0.f, d, unused;
            if (BIN) t = act_apply<ACT>(xf[q]);
            act_both<ACT>(x[q], unused, d);
            const float a = BIN ? dv[q] * ((to >> q) & 1u ? t : 0.f) : dv[q];
            const float b = (from >> q) & 1u ? through_act<ACT>(x[q], d, BIN ? dvs[q] * xs[q] : dvs[q]) : 0.f;
            dx[q] = a + b;
        }
    }
    store8(rdx, P.dx1, e, dx, u.nvalid);
}

template <typename F>
void by_act(int act, F f) {
    switch (act) {
    case 0: f(std::integral_constant<int, 0>()); break;
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    default: f(std::integral_constant<int, -1>()); break;
    }
}

}  // namespace

void mid_forward(const MidParams& P, hipStream_t s) {
    const long long total = (long long)P.N * P.C * P.upi;
    if (total <= 0) return;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    if (P.bin) by_act(P.act, [&](auto a) { CANVAS_LAUNCH((k_mid_fwd<decltype(a)::value, 1>), grid, block, 0, s, P); });
    else by_act(P.act, [&](auto a) { CANVAS_LAUNCH((k_mid_fwd<decltype(a)::value, 0>), grid, block, 0, s, P); });
}

void mid_backward(const MidParams& P, hipStream_t s) {
    const long long total = (long long)P.N * P.C * P.upi;
    if (total <= 0) return;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    if (P.bin) by_act(P.act, [&](auto a) { CANVAS_LAUNCH((k_mid_bwd<decltype(a)::value, 1>), grid, block, 0, s, P); });
    else by_act(P.act, [&](auto a) { CANVAS_LAUNCH((k_mid_bwd<decltype(a)::value, 0>), grid, block, 0, s, P); });
}

void self_backward(const MidParams& P, hipStream_t s) {
    const long long total = (long long)P.N * P.C * P.upi;
    if (total <= 0) return;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    if (P.bin) by_act(P.act, [&](auto a) { CANVAS_LAUNCH((k_self_bwd<decltype(a)::value, 1>), grid, block, 0, s, P); });
    else by_act(P.act, [&](auto a) { CANVAS_LAUNCH((k_self_bwd<decltype(a)::value, 0>), grid, block, 0, s, P); });
}

}  // namespace ufc
}  // namespace canvas
