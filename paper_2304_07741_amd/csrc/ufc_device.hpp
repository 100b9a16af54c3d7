// The element-wise middle of a sampled kernel, v = x (*|+) shift(act(z)), and its adjoint, for 8 consecutive pixels of one channel: shared by the
// launches of its own (ufc_kernels.hip) and by the FC kernels that go on with it (gfc_staged_kernel.hpp).
#pragma once
#include <type_traits>

#include "device_util.hpp"
#include "tile_util.hpp"
#include "ufc_kernels.hpp"

namespace canvas {
namespace ufc {

namespace {

using namespace canvas::tile;

__device__ __forceinline__ uint32_t div_magic(uint32_t x, uint32_t magic) { return magic ? __umulhi(x, magic) : x; }

// bits [lo, hi), 0 <= lo, hi <= 8
__device__ __forceinline__ uint32_t run_of_bits(int lo, int hi) { return hi > lo ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u; }
// bit q: pixel p+q exists and its source (h+dh, w+dw) is inside the image
__device__ __forceinline__ uint32_t shift_bits(const MidParams& P, int p, int dh, int dw) {
    int h = (int)div_magic((uint32_t)p, P.magicW), c = p - h * P.W;
    if (c < 0) {  // (the multiplier is exact below 2^32 / W and one too high at most beyond)
        c += P.W;
        h--;
    }
    if (P.W >= 8) {  // a run of pixels in each of at most two image rows
        const int n1 = min(8, P.W - c);  // pixels [0, n1) lie in row h
        uint32_t bits = 0;
        if ((unsigned)(h + dh) < (unsigned)P.H) bits = run_of_bits(max(0, -(c + dw)), min(n1, P.W - c - dw));
        if ((unsigned)(h + 1 + dh) < (unsigned)P.H) bits |= run_of_bits(max(n1, n1 - dw), min(8, n1 + P.W - dw));
        return P.P - p < 8 ? bits & ((1u << (P.P - p)) - 1u) : bits;
    }
    uint32_t bits = 0;
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const bool v = p + q < P.P && (unsigned)(h + dh) < (unsigned)P.H && (unsigned)(c + dw) < (unsigned)P.W;
        bits |= (v ? 1u : 0u) << q;
        if (++c == P.W) { c = 0; h++; }
    }
    return bits;
}

__device__ __forceinline__ void unpack8(const u32x4& v, float (&f)[8]) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
        f[2 * k] = lo_f32(v[k]);
        f[2 * k + 1] = hi_f32(v[k]);
    }
}

__device__ __forceinline__ u32x4 load8(rsrc_t r, int e, int bytes) {
    u32x4 v = bload16(r, e * 2);
    reload_if_partial(v, r, e * 2, bytes);
    return v;
}

__device__ __forceinline__ void store8(rsrc_t r, uint16_t* base, int e, const float (&f)[8], int nvalid, bool nt = true) {
    if (nvalid == 8) {
        u32x4 out;
#pragma unroll
        for (int k = 0; k < 4; k++) out[k] = pack_bf16(f[2 * k], f[2 * k + 1]);
        if (nt) bstore16_nt(r, e * 2, out);
        else bstore16(r, e * 2, out);
    } else {
#pragma unroll
        for (int q = 0; q < 8; q++)
            if (q < nvalid) base[e + q] = (uint16_t)(pack_bf16(f[q], 0.f) & 0xffffu);
    }
}

// Normal CDF and density at z.  erfc by the rational-times-Gaussian approximation of Abramowitz and Stegun,
// formula 7.1.26 (absolute error of erf below 1.5e-7, far below the bf16 rounding of every tensor these
// kernels write); the Gaussian is shared with the density, so gelu and its derivative at one point cost one
// exponential and one reciprocal.  (The fp32 per-node kernels use erff.)
__device__ __forceinline__ void normal_parts(float z, float& cdf, float& pdf) {
    const float t = __builtin_amdgcn_rcpf(1.f + 0.3275911f * 0.70710678f * fabsf(z));
    const float e = __expf(-0.5f * z * z);
    const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
    const float tail = 0.5f * poly * e;  // 0.5 * erfc(|z| / sqrt 2)
    cdf = z >= 0.f ? 1.f - tail : tail;
    pdf = 0.39894228f * e;
}

// ACT: -1 none, else UnaryKind (relu 0, abs 1, gelu 2, sin 4)
template <int ACT>
__device__ __forceinline__ float act_apply(float z) {
    if constexpr (ACT == 2) {
        float cdf, pdf;
        normal_parts(z, cdf, pdf);
        return z * cdf;
    } else if constexpr (ACT < 0) {
        return z;
    } else {
        return unary_apply(ACT, z, 0.f, 0.f);
    }
}

// act(z) and act'(z)
template <int ACT>
__device__ __forceinline__ void act_both(float z, float& t, float& d) {
    if constexpr (ACT == 2) {
        float cdf, pdf;
        normal_parts(z, cdf, pdf);
        t = z * cdf;
        d = cdf + z * pdf;
    } else {
        t = act_apply<ACT>(z);
        if constexpr (ACT < 0) d = 1.f;
        else d = unary_grad(ACT, z, 0.f, 0.f);
    }
}

// ---- in the registers of a kernel that has just computed z or dv (activation and blend by uniform branches)
struct UnitAt {
    int e = 0, p = 0, nvalid = 0;  // first element in the tensors, its pixel in the plane, pixels that exist (0: none)
};
struct Near {
    int dh = 0, dw = 0, off = 0;  // shift of the channel; the flat distance from p to its source, the plane's size where no pixel has one
    bool none = false;
};
struct Read {
    u32x4 x, z;
};
__device__ __forceinline__ Near shift_of(const MidParams& P, int c) {
    Near n;
#pragma unroll
    for (int k = 0; k < kMaxSlices; k++) {  // (constant indices: the parameters stay where the kernel received them)
        if (k >= P.nslices) break;
        const bool in = c >= P.c0[k] && c < P.c1[k];
        n.dh = in ? P.dh[k] : n.dh;
        n.dw = in ? P.dw[k] : n.dw;
    }
    n.none = n.dh >= P.H || n.dh <= -P.H || n.dw >= P.W || n.dw <= -P.W;
    n.off = n.none ? P.P : n.dh * P.W + n.dw;
    return n;
}
// Eight elements of plane pixels q .. q + 7, element e; what lies outside the plane is not used.
__device__ __forceinline__ u32x4 read8(const MidParams& P, const uint16_t* t, int e, int q, bool wanted) {
    const int bytes = P.N * P.C * P.P * 2;
    const rsrc_t r = make_rsrc(t, bytes);
    const int o = wanted && q < P.P && q + 7 >= 0 ? e * 2 : kOob;
    u32x4 v = bload16(r, o);
    reload_if_partial(v, r, o, bytes);
    return v;
}
// KIND 1, forward: x where z's pixels go.  2, adjoint: x at p, z at p + off.
template <int KIND>
__device__ __forceinline__ void mid_read(const MidParams& P, const UnitAt& u, const Near& s, Read& r) {
    if (KIND == 1) {
        r.x = read8(P, P.x, u.e - s.off, u.p - s.off, u.nvalid > 0);
    } else {
        if (P.bin) r.x = read8(P, P.x, u.e, u.p, u.nvalid > 0);
        r.z = read8(P, P.z, u.e + s.off, u.p + s.off, u.nvalid > 0);
    }
}
// act(z) and act'(z) for a uniform kind: none, relu, abs or gelu (takes_middle in gfc_staged_mid_kernels.hip: the sine's code would be there once per unit)
__device__ __forceinline__ void act_uniform(int act, const float (&z)[8], float (&t)[8], float (&d)[8]) {
    if (act == 2) {
#pragma unroll
        for (int q = 0; q < 8; q++) act_both<2>(z[q], t[q], d[q]);
    } else {
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const float sign = z[q] > 0.f ? 1.f : (z[q] < 0.f && act == 1 ? -1.f : 0.f);
            t[q] = act < 0 ? z[q] : (act == 0 ? __builtin_fmaxf(z[q], 0.f) : fabsf(z[q]));
            d[q] = act < 0 ? 1.f : sign;
        }
    }
}
// Eight results to pixels q .. q + 7 of the plane of element e (= pixel q), of which `nvalid` exist and those outside the plane are dropped.
__device__ __forceinline__ void write8(const MidParams& P, uint16_t* t, int e, int q, const float (&f)[8], int nvalid) {
    if (nvalid == 8 && q >= 0 && q + 8 <= P.P) {
        u32x4 out;
#pragma unroll
        for (int k = 0; k < 4; k++) out[k] = pack_bf16(f[2 * k], f[2 * k + 1]);
        bstore16(make_rsrc(t, P.N * P.C * P.P * 2), e * 2, out);
    } else {
#pragma unroll
        for (int k = 0; k < 8; k++)
            if (k < nvalid && (unsigned)(q + k) < (unsigned)P.P) t[e + k] = (uint16_t)(pack_bf16(f[k], 0.f) & 0xffffu);
    }
}

// v from the side of z (z8: its eight values as stored): v(p - d) = x(p - d) (*|+) act(z(p)).  p -> p - off is a bijection of the
// plane's flat pixel indices except at its two ends (see the adjoint in ufc_kernels.hip): targets outside the plane are dropped, and a pixel whose flat source is
// outside it is written by its own thread; a target in another image row than its source takes the zero that the shift fills in.
__device__ __forceinline__ void mid_forward_unit(const MidParams& P, const UnitAt& u, const Near& s, const Read& r, const u32x4& z8) {
    float x[8], z[8], v[8];
    unpack8(r.x, x);
    unpack8(z8, z);
    const uint32_t bits = s.none ? 0u : ((s.dh | s.dw) != 0 ? shift_bits(P, u.p, -s.dh, -s.dw) : 0xffu);
    float t[8], d[8];
    act_uniform(P.act, z, t, d);
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const float tq = (bits >> q) & 1u ? t[q] : 0.f;
        v[q] = P.bin ? x[q] * tq : x[q] + tq;
    }
    write8(P, P.v, u.e - s.off, u.p - s.off, v, u.nvalid);
    if (s.off != 0 && (u.p + s.off < 0 || u.p + u.nvalid - 1 + s.off >= P.P)) {
        for (int q = 0; q < u.nvalid; q++)
            if ((unsigned)(u.p + q + s.off) >= (unsigned)P.P) {
                const float xq = __uint_as_float((uint32_t)P.x[u.e + q] << 16);
                P.v[u.e + q] = (uint16_t)(pack_bf16(P.bin ? xq * 0.f : xq, 0.f) & 0xffffu);
            }
    }
}

// The adjoint, as k_mid_bwd in ufc_kernels.hip: dx1(p) = dv(p) t(p), dz(p + d) = act'(z(p + d)) dv(p) x(p).
__device__ __forceinline__ void mid_backward_unit(const MidParams& P, const UnitAt& u, const Near& s, const Read& r, const float (&dv)[8]) {
    float z[8], x[8], dx1[8], dz[8];
    unpack8(r.z, z);
    unpack8(r.x, x);
    const uint32_t bits = s.none ? 0u : ((s.dh | s.dw) != 0 ? shift_bits(P, u.p, s.dh, s.dw) : 0xffu);
    float t[8], d[8];
    act_uniform(P.act, z, t, d);
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const bool in = (bits >> q) & 1u;
        dx1[q] = P.bin ? dv[q] * (in ? t[q] : 0.f) : dv[q];
        dz[q] = (in ? (P.bin ? dv[q] * x[q] : dv[q]) : 0.f) * d[q];
    }
    write8(P, P.dx1, u.e, u.p, dx1, u.nvalid);
    write8(P, P.dz, u.e + s.off, u.p + s.off, dz, u.nvalid);
    if (s.off != 0 && (u.p - s.off < 0 || u.p + u.nvalid - 1 - s.off >= P.P)) {
        // (a zero, or 0 * act'(z) where that is no number)
        for (int q = 0; q < u.nvalid; q++)
            if ((unsigned)(u.p + q - s.off) >= (unsigned)P.P) {
                const float zq = __uint_as_float((uint32_t)P.z[u.e + q] << 16);
                float t, d = P.act < 0 ? 1.f : (zq > 0.f ? 1.f : (zq < 0.f && P.act == 1 ? -1.f : 0.f));
                if (P.act == 2) act_both<2>(zq, t, d);
                P.dz[u.e + q] = (uint16_t)(pack_bf16(0.f * d, 0.f) & 0xffffu);
            }
    }
}

}  // namespace

}  // namespace ufc
}  // namespace canvas
