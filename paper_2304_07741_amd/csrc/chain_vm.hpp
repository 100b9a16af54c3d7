// Per-thread execution of the fused-chain instruction set (see chain_isa.hpp).  A thread owns V consecutive pixels of
// one image plane; a value is T x V floats (lane t * V + v = tap t of pixel v), so one interpreted instruction works
// on 8 to 25 elements and every tensor access is one vector access of V elements.  Everything here is per-pixel
// arithmetic on the thread's own state; the one instruction that moves data between threads (OP_XADD) is driven by the
// kernel around two helpers of this file.  Primitive definitions: Canvas paper, Section 5; subgradient choices:
// relu'(0) = 0, sign(0) = 0, clipped exp flat outside the open interval, first maximum of a max fold, ties of
// min / max to the LHS.
//
// The file compiles for the device (raw buffer accesses) and for the host (checked scalar accesses), so that the
// interpreter can be run on the CPU, workgroup by workgroup, against the same programs.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

#include "chain_isa.hpp"

#if defined(__HIP_DEVICE_COMPILE__)
#include "tile_util.hpp"
#endif

#if defined(__HIPCC__)
#define CHAIN_HD __host__ __device__ __forceinline__
#else
#define CHAIN_HD inline
#endif

namespace canvas {
namespace chain {

template <int TM, int V, int U>
struct State {
    float A[U * TM * V];
};

// 16-byte pieces of a register R[r] (lanes floats, rounded up); piece q of register r of thread i is at float
// ((r * pieces + q) * threads + i) * 4 of the register area, so that a wavefront's access is one contiguous run.
constexpr int reg_pieces(int lanes) { return (lanes + 3) / 4; }

// What a thread knows about its pixels.  p0 is the plane index of its first pixel (a multiple of V; threads of the
// halo may lie before the plane or behind it: active == false); only `own` threads store.
struct Thread {
    int ptid = 0, n = 0, p0 = 0, row0 = 0, col0 = 0;
    bool active = false, own = false;
};

// Geometry in uniform registers.
struct Geo {
    int H = 0, W = 0, C = 0, HW = 0, N = 0;
    int npx = 0;  // pixels a slice of the workgroup computes = pix_threads * V
    bool whole_rows = false;  // W is a multiple of V: the V pixels of a thread never straddle two image rows
    // HW is no multiple of V: planes begin at any element, and the last thread of a plane has pixels behind it, which it computes
    // on what the next plane holds there and never stores (nothing but a store or a hand-over leaves a pixel's own lanes)
    bool ragged = false;
};

// Each case of the dispatch begins with an empty volatile asm statement: the cases are small, and without it the
// compiler executes the arithmetic of ALL of them for every instruction and selects the result.
#if defined(__HIP_DEVICE_COMPILE__)
#define CHAIN_CASE asm volatile("")
#else
#define CHAIN_CASE ((void)0)
#endif

// The program is interpreted from LDS, whose loads land in vector registers: the compiler cannot know that every
// lane read the same word.  vm_u() tells it (one v_readfirstlane), so that instruction fields, tensor descriptors and
// geometry live in scalar registers and the dispatch on them is a scalar branch.
#if defined(__HIP_DEVICE_COMPILE__)
CHAIN_HD int vm_u(int v) { return __builtin_amdgcn_readfirstlane(v); }
#else
CHAIN_HD int vm_u(int v) { return v; }
#endif
// A uniform value that the compiler knows nothing about: a branch on it stays where it is (a loop is not copied for each of its outcomes).
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ int vm_opaque(int v) {
    v = vm_u(v);
    asm volatile("" : "+s"(v));
    return v;
}
#endif
#if !defined(__HIP_DEVICE_COMPILE__)
inline int vm_opaque(int v) { return v; }
#endif
// A 16-byte instruction, made uniform.
CHAIN_HD Instr vm_fetch(const Instr& src) {
    uint32_t w[4];
    memcpy(w, &src, 16);
    for (int k = 0; k < 4; k++) w[k] = (uint32_t)vm_u((int)w[k]);
    Instr I;
    memcpy(&I, w, 16);
    return I;
}
#if defined(__HIPCC__)
// The same for an instruction that has already been read as four dwords.
__device__ __forceinline__ Instr vm_uniform(const uint4& raw) {
    uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
    for (int k = 0; k < 4; k++) w[k] = (uint32_t)vm_u((int)w[k]);
    Instr I;
    memcpy(&I, w, 16);
    return I;
}
#endif
CHAIN_HD Geo vm_geo(const Program& pg) {
    Geo g;
    g.H = vm_u(pg.H);
    g.W = vm_u(pg.W);
    g.C = vm_u(pg.C);
    g.N = vm_u(pg.N);
    g.HW = g.H * g.W;
    g.npx = vm_u(pg.pix_threads) * vm_u(pg.vec);
    g.whole_rows = g.W % vm_u(pg.vec) == 0;
    return g;
}

CHAIN_HD float vm_bf16_to_f32(uint16_t h) {
    uint32_t u = (uint32_t)h << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}
CHAIN_HD float vm_bits_to_f32(uint32_t u) {
    float f;
    memcpy(&f, &u, 4);
    return f;
}
CHAIN_HD uint32_t vm_f32_to_bits(float f) {
    uint32_t u;
    memcpy(&u, &f, 4);
    return u;
}

CHAIN_HD uint16_t vm_f32_to_bf16(float f) {  // round to nearest even; NaN stays NaN
    uint32_t u = vm_f32_to_bits(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------------------------------- tensors
// A tensor of the program in uniform registers.  Element indices are 32-bit (the planner only admits tensors below
// 2^31 bytes) and may lie outside the tensor (a shifted access at the first or last image): such elements read as
// zero on the device and as NaN on the host, and are masked by the caller either way.
struct Tensor {
#if defined(__HIP_DEVICE_COMPILE__)
    tile::rsrc_t rs;
#else
    void* ptr = nullptr;
#endif
    int bytes = 0;
    int T = 1;
    int bf16 = 0;
};

CHAIN_HD Tensor vm_tensor(const Program& pg, const Geo& g, int a) {
    uint32_t w[4];
    memcpy(w, &pg.ext[a], 16);
    for (int k = 0; k < 4; k++) w[k] = (uint32_t)vm_u((int)w[k]);
    Tensor t;
    t.T = (int)w[2];
    t.bf16 = (int)w[3];
    t.bytes = g.N * g.C * t.T * g.HW * (t.bf16 ? 2 : 4);
    void* p = (void*)(((uint64_t)w[1] << 32) | w[0]);
#if defined(__HIP_DEVICE_COMPILE__)
    t.rs = tile::make_rsrc(p, t.bytes);
#else
    t.ptr = p;
#endif
    return t;
}

#if defined(__HIP_DEVICE_COMPILE__)
typedef uint32_t vm_u32x2 __attribute__((ext_vector_type(2)));

// V elements that begin at element `elem`.  ALIGNED: elem is a multiple of V (so is every tensor's size), the access
// is wholly inside or wholly outside the tensor and no piece of it needs a second look.
template <int V, bool ALIGNED>
__device__ __forceinline__ void vm_load(const Tensor& e, int elem, float* out) {
    if (e.bf16) {
        const int o = elem * 2;
        if (V % 8 == 0) {
#pragma unroll
            for (int q = 0; q < V / 8; q++) {
                tile::u32x4 d = tile::bload16(e.rs, o + 16 * q);
                if (!ALIGNED && tile::straddles_an_end(o + 16 * q, 16, e.bytes)) {
                    // (rare: a shifted vector across the very start or end of the tensor; the empty asm keeps the
                    // compiler from computing the element addresses of this branch ahead of it, for every access)
                    int o2 = o + 16 * q;
                    asm volatile("" : "+v"(o2));
#pragma unroll
                    for (int k = 0; k < 4; k++) d[k] = tile::elem_b16(e.rs, o2 + 4 * k, e.bytes) | (tile::elem_b16(e.rs, o2 + 4 * k + 2, e.bytes) << 16);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    out[8 * q + 2 * k] = tile::lo_f32(d[k]);
                    out[8 * q + 2 * k + 1] = tile::hi_f32(d[k]);
                }
            }
        } else if (V == 4) {
            vm_u32x2 d = __builtin_amdgcn_raw_buffer_load_b64(e.rs, o, 0, 0);
            if (!ALIGNED && tile::straddles_an_end(o, 8, e.bytes)) {
#pragma unroll
                for (int k = 0; k < 2; k++) d[k] = tile::elem_b16(e.rs, o + 4 * k, e.bytes) | (tile::elem_b16(e.rs, o + 4 * k + 2, e.bytes) << 16);
            }
#pragma unroll
            for (int k = 0; k < 2; k++) {
                out[2 * k] = tile::lo_f32(d[k]);
                out[2 * k + 1] = tile::hi_f32(d[k]);
            }
        } else if (V == 2) {
            uint32_t d = __builtin_amdgcn_raw_buffer_load_b32(e.rs, o, 0, 0);
            if (!ALIGNED) tile::reload_pair_if_partial(d, e.rs, o, e.bytes);
            out[0] = tile::lo_f32(d);
            out[1] = tile::hi_f32(d);
        } else {
#pragma unroll
            for (int v = 0; v < V; v++) out[v] = tile::lo_f32(tile::elem_b16(e.rs, o + 2 * v, e.bytes));
        }
    } else {
        const int o = elem * 4;
        if (V % 4 == 0) {
#pragma unroll
            for (int q = 0; q < V / 4; q++) {
                tile::u32x4 d = tile::bload16(e.rs, o + 16 * q);
                if (!ALIGNED && tile::straddles_an_end(o + 16 * q, 16, e.bytes)) {
                    int o2 = o + 16 * q;
                    asm volatile("" : "+v"(o2));
#pragma unroll
                    for (int k = 0; k < 4; k++) d[k] = tile::elem_b32(e.rs, o2 + 4 * k, e.bytes);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) out[4 * q + k] = __uint_as_float(d[k]);
            }
        } else {
#pragma unroll
            for (int v = 0; v < V; v++) out[v] = __uint_as_float(tile::elem_b32(e.rs, o + 4 * v, e.bytes));
        }
    }
}

// `left` (V in all, a multiple of V, unless planes are ragged) elements to element `elem`: only owned pixels are stored.
template <int V>
__device__ __forceinline__ void vm_store(const Tensor& e, int elem, const float* in, bool add, bool ragged, int left) {
    if (ragged && left < V) {
#pragma unroll
        for (int v = 0; v < V; v++)
            if (v < left) {
                if (e.bf16) {
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(tile::pack_bf16(in[v], 0.f) & 0xffffu), e.rs, (elem + v) * 2, 0, 0);
                } else {
                    const float old = add ? __uint_as_float(tile::elem_b32(e.rs, (elem + v) * 4, e.bytes)) : 0.f;
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(add ? old + in[v] : in[v]), e.rs, (elem + v) * 4, 0, 0);
                }
            }
        return;
    }
    if (e.bf16) {
        const int o = elem * 2;
        if (V % 8 == 0) {
#pragma unroll
            for (int q = 0; q < V / 8; q++) {
                tile::u32x4 d;
#pragma unroll
                for (int k = 0; k < 4; k++) d[k] = tile::pack_bf16(in[8 * q + 2 * k], in[8 * q + 2 * k + 1]);
                if (ragged) tile::bstore16(e.rs, o + 16 * q, d);  // (unaligned: kept in the cache until its lines are whole)
                else tile::bstore16_nt(e.rs, o + 16 * q, d);
            }
        } else if (V == 4) {
            vm_u32x2 d;
#pragma unroll
            for (int k = 0; k < 2; k++) d[k] = tile::pack_bf16(in[2 * k], in[2 * k + 1]);
            __builtin_amdgcn_raw_buffer_store_b64(d, e.rs, o, 0, 0);
        } else if (V == 2) {
            __builtin_amdgcn_raw_buffer_store_b32(tile::pack_bf16(in[0], in[1]), e.rs, o, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(tile::pack_bf16(in[0], 0.f) & 0xffffu), e.rs, o, 0, 0);
        }
    } else {
        const int o = elem * 4;
        float v[V];
        if (add) {
            vm_load<V, true>(e, elem, v);
#pragma unroll
            for (int k = 0; k < V; k++) v[k] += in[k];
        } else {
#pragma unroll
            for (int k = 0; k < V; k++) v[k] = in[k];
        }
        if (V % 4 == 0) {
#pragma unroll
            for (int q = 0; q < V / 4; q++) {
                tile::u32x4 d;
#pragma unroll
                for (int k = 0; k < 4; k++) d[k] = __float_as_uint(v[4 * q + k]);
                if (ragged) tile::bstore16(e.rs, o + 16 * q, d);
                else tile::bstore16_nt(e.rs, o + 16 * q, d);
            }
        } else {
#pragma unroll
            for (int k = 0; k < V; k++) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[k]), e.rs, o + 4 * k, 0, 0);
        }
    }
}
#else
// Host: element by element, checked.  An element outside the tensor reads as NaN, so that a missing mask shows in
// the results; a store outside the tensor is a bug of the planner and aborts.
#include <cstdio>
#include <cstdlib>
template <int V, bool ALIGNED>
inline void vm_load(const Tensor& e, int elem, float* out) {
    const int64_t n = e.bytes / (e.bf16 ? 2 : 4);
    if (ALIGNED && elem % V != 0) {
        std::fprintf(stderr, "chain vm: an aligned load of %d elements at %d\n", V, elem);
        std::abort();
    }
    for (int v = 0; v < V; v++) {
        const int64_t i = (int64_t)elem + v;
        if (i < 0 || i >= n) out[v] = NAN;
        else out[v] = e.bf16 ? vm_bf16_to_f32(((const uint16_t*)e.ptr)[i]) : ((const float*)e.ptr)[i];
    }
}
template <int V>
inline void vm_store(const Tensor& e, int elem, const float* in, bool add, bool ragged, int left) {
    const int64_t n = e.bytes / (e.bf16 ? 2 : 4);
    if (!ragged || left > V) left = V;
    if (elem < 0 || (int64_t)elem + left > n || (!ragged && elem % V)) {
        std::fprintf(stderr, "chain vm: store of %d elements at %d outside a tensor of %lld\n", V, elem, (long long)n);
        std::abort();
    }
    for (int v = 0; v < left; v++) {
        if (e.bf16) ((uint16_t*)e.ptr)[elem + v] = vm_f32_to_bf16(in[v]);
        else if (add) ((float*)e.ptr)[elem + v] += in[v];
        else ((float*)e.ptr)[elem + v] = in[v];
    }
}
#endif

// ---------------------------------------------------------------------------------------------------- arithmetic
// The element-wise functions, one per kind: the dispatch on the kind happens once per instruction, outside the loops
// over the lanes (a switch inside the loop costs a scalar branch tree per element).
CHAIN_HD float vm_gelu(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752f)); }
CHAIN_HD float vm_gelu_grad(float x) { return 0.5f * (1.f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x); }
CHAIN_HD float vm_sign(float x) { return x > 0.f ? 1.f : (x < 0.f ? -1.f : 0.f); }
// Normal CDF and density for programs of bf16 DAGs (Program::fast_math): erfc by the rational-times-Gaussian
// approximation of Abramowitz and Stegun, formula 7.1.26 (absolute error of erf below 1.5e-7, five orders below the
// tolerance of a bf16 DAG); the Gaussian is shared with the density, so gelu or its derivative costs one exponential
// and one division.  fp32 DAGs keep erff.  Exponential and reciprocal of such programs are the hardware's (base-2
// exponential of x * log2 e: relative error about 1e-7 * (1 + |x|), results below 2^-126 are 0; reciprocal to one unit
// in the last place): a fifth of the instructions of expf and of a division.
#if defined(__HIP_DEVICE_COMPILE__)
CHAIN_HD float vm_exp_fast(float x) { return __expf(x); }
CHAIN_HD float vm_rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }
#else
CHAIN_HD float vm_exp_fast(float x) { return expf(x); }
CHAIN_HD float vm_rcp_fast(float x) { return 1.f / x; }
#endif
CHAIN_HD void vm_normal_parts(float z, float& cdf, float& pdf) {
    const float t = vm_rcp_fast(1.f + 0.3275911f * 0.70710678f * fabsf(z));
    const float e = vm_exp_fast(-0.5f * z * z);
    const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
    const float tail = 0.5f * poly * e;  // 0.5 * erfc(|z| / sqrt 2)
    cdf = z >= 0.f ? 1.f - tail : tail;
    pdf = 0.39894228f * e;
}
CHAIN_HD float vm_gelu_fast(float x) {
    float cdf, pdf;
    vm_normal_parts(x, cdf, pdf);
    return x * cdf;
}
CHAIN_HD float vm_gelu_grad_fast(float x) {
    float cdf, pdf;
    vm_normal_parts(x, cdf, pdf);
    return cdf + x * pdf;
}

// x / n as a product with the reciprocal and one correction step from the remainder: the quotient to within one unit in the last
// place, a fifth of the instructions of a division per pixel (infinities and NaN come out as a division gives them).
CHAIN_HD float vm_over(float x, float n) {
#if defined(__HIP_DEVICE_COMPILE__)
    const float r = 1.f / n, q = x * r;
    return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-n, q, x), r, q), n, x);
#else
    return x / n;
#endif
}

// Sum of the offsets of a position for channel c: terms [b >> 8, (b >> 8) + (b & 255)) that cover c.
CHAIN_HD void vm_offset(const Program& pg, uint16_t b, int c, int& dh, int& dw) {
    dh = 0;
    dw = 0;
    const int first = b >> 8, cnt = b & 255;
    for (int k = 0; k < cnt; k++) {
        uint32_t w[2];
        memcpy(w, &pg.term[first + k], 8);
        const int off = vm_u((int)w[0]), rng = vm_u((int)w[1]);  // (dh, dw) and (c0, c1) as packed halves
        if (c >= (rng & 0xffff) && c < (int)((uint32_t)rng >> 16)) {
            dh += (int16_t)(off & 0xffff);
            dw += (int16_t)((uint32_t)off >> 16);
        }
    }
}

// Row and column of tap t of a KH x KW window (t is a compile-time constant after unrolling, KW is uniform: the
// windows the planner admits are 1, 3 or 5 wide).
CHAIN_HD void vm_tap(int t, int KH, int KW, int& oh, int& ow) {
    const int kh = KW == 3 ? t / 3 : (KW == 5 ? t / 5 : t);
    oh = kh - KH / 2;
    ow = t - kh * KW - KW / 2;
}

// Lanes of a value: channel u < U of the trip, tap t < T (T is uniform: 1, or the taps of a window), pixel v < V.
// The body sees e = (u * TM + t) * V + v and l = t * V + v.
#define CHAIN_EACH(T, e, l, ...)                                                          \
    do {                                                                                  \
        if (TM == 1 || (T) == 1) {                                                        \
            _Pragma("unroll") for (int u_ = 0; u_ < U; u_++) {                            \
                _Pragma("unroll") for (int l = 0; l < V; l++) {                           \
                    const int e = u_ * TM * V + l;                                        \
                    __VA_ARGS__                                                           \
                }                                                                         \
            }                                                                             \
        } else {                                                                          \
            _Pragma("unroll") for (int u_ = 0; u_ < U; u_++) {                            \
                _Pragma("unroll") for (int t_ = 0; t_ < TM; t_++) if (t_ < (T)) {         \
                    _Pragma("unroll") for (int v_ = 0; v_ < V; v_++) {                    \
                        const int l = t_ * V + v_;                                        \
                        const int e = u_ * TM * V + l;                                    \
                        __VA_ARGS__                                                       \
                    }                                                                     \
                }                                                                         \
            }                                                                             \
        }                                                                                 \
    } while (0)

// Register r (uniform) of all U channels <-> X: lanes [0, T * V) of every channel.  Rm: piece 0 of register 0 of this
// thread; rstride: floats between pieces (threads * 4); a register is its U * TM * V lanes in pieces of four.
template <int TM, int V, int U>
CHAIN_HD void vm_reg_read(const float* Rm, int rstride, int r, int T, float* X) {
    constexpr int L = U * TM * V, Q = reg_pieces(L);
    const float* src = Rm + r * Q * rstride;
#pragma unroll
    for (int q = 0; q < Q; q++) {
        bool needed = false;
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (q * 4 + k < L && (q * 4 + k) % (TM * V) < T * V) needed = true;
        if (needed) {
            float w[4];
            memcpy(w, src + q * rstride, 16);
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (q * 4 + k < L) X[q * 4 + k] = w[k];
        }
    }
}
// A += X * R[r], a piece at a time (a second array of lanes would cost the instances with taps wavefronts or scratch)
template <int TM, int V, int U>
CHAIN_HD void vm_reg_madd(const float* Rm, int rstride, int r, int T, const float* X, float* A) {
    constexpr int L = U * TM * V, Q = reg_pieces(L);
    const float* src = Rm + r * Q * rstride;
#pragma unroll
    for (int q = 0; q < Q; q++) {
        float w[4];
        memcpy(w, src + q * rstride, 16);
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (q * 4 + k < L && (q * 4 + k) % (TM * V) < T * V) A[q * 4 + k] += X[q * 4 + k] * w[k];
        asm volatile("" ::: "memory");
    }
}
template <int TM, int V, int U>
CHAIN_HD void vm_reg_write(float* Rm, int rstride, int r, int T, const float* X) {
    constexpr int L = U * TM * V, Q = reg_pieces(L);
    float* dst = Rm + r * Q * rstride;
#pragma unroll
    for (int q = 0; q < Q; q++) {
        bool needed = false;
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (q * 4 + k < L && (q * 4 + k) % (TM * V) < T * V) needed = true;
        if (needed) {
            float w[4];
#pragma unroll
            for (int k = 0; k < 4; k++) w[k] = q * 4 + k < L ? X[q * 4 + k] : 0.f;
            memcpy(dst + q * rstride, w, 16);
        }
    }
}

// Which of the thread's V pixels see the image at offset (oh, ow): bit v of the result.  The thread's pixels are a run
// of at most two image rows (V <= W), so the valid ones are at most two runs of bits: no per-pixel arithmetic.
CHAIN_HD uint32_t vm_bits(int lo, int hi) {  // bits [lo, hi), 0 <= lo, hi <= 32
    const uint32_t upto_hi = hi >= 32 ? 0xffffffffu : ((1u << hi) - 1u);
    return hi > lo ? (upto_hi & ~((1u << lo) - 1u)) : 0u;
}
// x where bit v of m is set, else +0 (two bit operations instead of a compare and a select).
CHAIN_HD float vm_keep(float x, uint32_t m, int v) { return vm_bits_to_f32(vm_f32_to_bits(x) & (0u - ((m >> v) & 1u))); }
template <int V>
CHAIN_HD uint32_t vm_valid(const Geo& g, const Thread& th, int oh, int ow) {
    if (V == 1) return th.active && (unsigned)(th.row0 + oh) < (unsigned)g.H && (unsigned)(th.col0 + ow) < (unsigned)g.W ? 1u : 0u;
    if (!th.active) return 0;
    if (g.whole_rows) {
        // all V pixels lie in row0 (col0 is a multiple of V): the row is inside or not as a whole, and columns fall off only
        // at the row's first pixels (to the left) or last pixels (to the right)
        if ((unsigned)(th.row0 + oh) >= (unsigned)g.H) return 0;
        const int first = -(th.col0 + ow), behind = g.W - th.col0 - ow;
        return vm_bits(first > 0 ? first : 0, behind < V ? behind : V);
    }
    const int n1 = g.W - th.col0 < V ? g.W - th.col0 : V;  // pixels [0, n1) lie in row0, [n1, V) in row0 + 1
    const int first = -(th.col0 + ow), behind = g.W - th.col0 - ow;  // pixel v of row0 has column v - first; valid for first <= v < behind
    uint32_t m = 0;
    if ((unsigned)(th.row0 + oh) < (unsigned)g.H) m |= vm_bits(first > 0 ? first : 0, behind < n1 ? behind : n1);
    if (n1 < V && (unsigned)(th.row0 + 1 + oh) < (unsigned)g.H) {
        // pixel v of row0 + 1 has column v - n1, displaced v - n1 + ow = v - behind + ... : valid for behind <= v < behind + W
        const int lo2 = behind > n1 ? behind : n1, hi2 = behind + g.W < V ? behind + g.W : V;
        m |= vm_bits(lo2, hi2);
    }
    return m;
}

// out[v] = tensor(plane, pixel p0 + v displaced by (oh, ow)), 0 outside the image.  Without displacement nothing is
// masked: what a thread outside the plane reads (zeros, or pixels of another plane) is never stored nor handed over.
template <int V>
CHAIN_HD void vm_load_at(const Tensor& e, const Geo& g, const Thread& th, int plane, int oh, int ow, float* out) {
    if (oh == 0 && ow == 0) {
        if (g.ragged) vm_load<V, false>(e, plane * g.HW + th.p0, out);
        else vm_load<V, true>(e, plane * g.HW + th.p0, out);
    } else {
        float raw[V];
        vm_load<V, false>(e, plane * g.HW + th.p0 + oh * g.W + ow, raw);
        const uint32_t m = vm_valid<V>(g, th, oh, ow);
#pragma unroll
        for (int v = 0; v < V; v++) out[v] = vm_keep(raw[v], m, v);
    }
}

#if defined(__HIP_DEVICE_COMPILE__)
// One pixel per thread and a constant window: byte offset of tap (i, j) = offset of its row, or beyond every tensor where the row is
// outside the image, plus its column's; outside columns are sent to kOob.  Five row tests and five column tests for 25 taps,
// two instructions a tap.  (With a test per tap, a branch and the tensor's descriptor fetched again for each, a 5x5 window was
// 700 vector and 450 scalar instructions: under a product and an avg fold, 16x96 planes of 32x32, 82 us forward and 202 backward; now
// 69 and 156.)
template <int KHC, int KWC, int ES, typename F>
__device__ __forceinline__ void vm_window_offsets(const Geo& g, const Thread& th, int chan, int dh, int dw, F each) {
    uint32_t row[KHC];
    int col[KWC];
    bool in[KWC];
#pragma unroll
    for (int i = 0; i < KHC; i++) {
        const int r = th.row0 + dh + i - KHC / 2;
        row[i] = (int)((unsigned)r < (unsigned)g.H) & (int)th.active ? (uint32_t)((chan * g.HW + r * g.W) * ES) : 0x80000000u;
    }
#pragma unroll
    for (int j = 0; j < KWC; j++) {
        const int c = th.col0 + dw + j - KWC / 2;
        in[j] = (unsigned)c < (unsigned)g.W;
        col[j] = c * ES;
    }
#pragma unroll
    for (int i = 0; i < KHC; i++)
#pragma unroll
        for (int j = 0; j < KWC; j++) {
            int off = in[j] ? (int)(row[i] + (uint32_t)col[j]) : tile::kOob;
            asm volatile("" : "+v"(off));  // (an offset in a register of its own, no immediate)
            each(i * KWC + j, off);
        }
}

// The T = KH * KW taps of a window of a bf16 tensor, displaced by (dh, dw), for the thread's V pixels of plane `chan`:
// out[t * V + v], 0 outside the image.  All loads are issued before the first is looked at: one round trip to memory
// for the T taps, not T (tap by tap, each load was followed by its own wait: the fix-up of an access that straddles an
// end of the tensor may overwrite what was loaded).  KHC x KWC: the window as constants (tap geometry folds, the taps
// of a window row share the row test and the taps of a window column the column mask), or 0 x 0 for the window (KH, KW).
template <int TM, int V, int KHC, int KWC>
__device__ __forceinline__ void vm_ld_window_bf16(const Tensor& e, const Geo& g, const Thread& th, int chan, int dh, int dw, int KH, int KW, int T,
                                                  float* out) {
    if constexpr (V == 1 && KHC > 0) {
        uint32_t raw[KHC * KWC];
        vm_window_offsets<KHC, KWC, 2>(g, th, chan, dh, dw, [&](int t, int off) { raw[t] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(e.rs, off, 0, 0); });
#pragma unroll
        for (int t = 0; t < KHC * KWC; t++) out[t] = tile::lo_f32(raw[t]);
        return;
    }
    constexpr int D = V == 1 ? 1 : V / 2;
    if (KHC > 0) {
        KH = KHC;
        KW = KWC;
        T = KHC * KWC;
    }
    uint32_t raw[TM][D];
    int off[TM];
    // Threads that never cross an image row: a tap's row is inside the image or not as a whole (outside, the load is
    // sent to the offset that reads zeros), and its columns fall off at the row's ends only.
    const bool by_rows = g.whole_rows;
    const int centre_off = (chan * g.HW + th.p0) * 2;
#pragma unroll
    for (int t = 0; t < TM; t++)
        if (t < T) {
            int oh, ow;
            vm_tap(t, KH, KW, oh, ow);
            off[t] = centre_off + ((dh + oh) * g.W + dw + ow) * 2;
            if (V == 1) {  // (one element: inside the image or not)
                const bool inside = th.active && (unsigned)(th.row0 + dh + oh) < (unsigned)g.H && (unsigned)(th.col0 + dw + ow) < (unsigned)g.W;
                off[t] = inside ? off[t] : tile::kOob;
            } else if (by_rows) {
                const bool row_inside = th.active && (unsigned)(th.row0 + dh + oh) < (unsigned)g.H;
                off[t] = row_inside ? off[t] : tile::kOob;
            }
            // (each tap's offset in a register of its own: a negative base register plus the tap's distance as the
            // instruction's immediate offset is not what the bounds check expects)
            asm volatile("" : "+v"(off[t]));
            if (V == 4) {
                const vm_u32x2 d = __builtin_amdgcn_raw_buffer_load_b64(e.rs, off[t], 0, 0);
                raw[t][0] = d[0];
                raw[t][D - 1] = d[1];
            } else if (V == 2) {
                raw[t][0] = __builtin_amdgcn_raw_buffer_load_b32(e.rs, off[t], 0, 0);
            } else {
                raw[t][0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(e.rs, off[t], 0, 0);
            }
        }
    if (V == 1) {
#pragma unroll
        for (int t = 0; t < TM; t++)
            if (t < T) out[t] = tile::lo_f32(raw[t][0]);
        return;
    }
    // An access may straddle an end of the tensor only when the window of this thread reaches across that end: one
    // test for all taps (false for nearly every thread), then tap by tap.
    const int reach = (((KH >> 1) + (dh < 0 ? -dh : dh)) * g.W + (KW >> 1) + (dw < 0 ? -dw : dw)) * 2;
    if (centre_off - reach < 0 || centre_off + reach + 2 * V > e.bytes) {
#pragma unroll
        for (int t = 0; t < TM; t++)
            if (t < T && tile::straddles_an_end(off[t], 2 * V, e.bytes)) {
#pragma unroll
                for (int k = 0; k < D; k++)
                    raw[t][k] = tile::elem_b16(e.rs, off[t] + 4 * k, e.bytes) | (tile::elem_b16(e.rs, off[t] + 4 * k + 2, e.bytes) << 16);
            }
    }
    if (by_rows) {
        // pixel v of a tap in window column j is inside for first <= v < behind: a mask over the packed pairs, then the
        // pairs are taken apart
        constexpr int NM = KWC > 0 ? KWC : 1;
        uint32_t cm[NM][D];
#pragma unroll
        for (int t = 0; t < TM; t++)
            if (t < T) {
                int oh, ow;
                vm_tap(t, KH, KW, oh, ow);
                const int j = KWC > 0 ? ow + KWC / 2 : 0;
                if (KWC == 0 || t < KWC) {  // (first window row: the masks of its columns serve the rows below)
                    const int first = -(th.col0 + dw + ow), behind = g.W - th.col0 - dw - ow;
                    const uint32_t m = vm_bits(first > 0 ? first : 0, behind < V ? behind : V);
#pragma unroll
                    for (int k = 0; k < D; k++) {
                        const uint32_t lo = (uint32_t)((int32_t)(m << (31 - 2 * k)) >> 31), hi = (uint32_t)((int32_t)(m << (30 - 2 * k)) >> 31);
                        cm[j][k] = (lo & 0xffffu) | (hi & 0xffff0000u);
                    }
                }
#pragma unroll
                for (int k = 0; k < D; k++) {
                    const uint32_t kept = raw[t][k] & cm[j][k];
                    out[t * V + 2 * k] = tile::lo_f32(kept);
                    out[t * V + 2 * k + 1] = tile::hi_f32(kept);
                }
            }
    } else {
#pragma unroll
        for (int t = 0; t < TM; t++)
            if (t < T) {
                int oh, ow;
                vm_tap(t, KH, KW, oh, ow);
                const bool centre = dh + oh == 0 && dw + ow == 0;  // (uniform; without displacement nothing is masked)
                const uint32_t m = centre ? 0xffffffffu : vm_valid<V>(g, th, dh + oh, dw + ow);
#pragma unroll
                for (int k = 0; k < D; k++) {
                    out[t * V + 2 * k] = vm_keep(tile::lo_f32(raw[t][k]), m, 2 * k);
                    out[t * V + 2 * k + 1] = vm_keep(tile::hi_f32(raw[t][k]), m, 2 * k + 1);
                }
            }
    }
}

// The same for an fp32 tensor (one between two units of a lowering): again all loads of the window before the first is
// looked at (forward of a 5x5 window under a product and an avg fold, 16x96 planes of 32x32: 104 -> 69 us).
template <int TM, int V, int KHC, int KWC>
__device__ __forceinline__ void vm_ld_window_f32(const Tensor& e, const Geo& g, const Thread& th, int chan, int dh, int dw, int KH, int KW, int T,
                                                 float* out) {
    if constexpr (V == 1 && KHC > 0) {
        vm_window_offsets<KHC, KWC, 4>(g, th, chan, dh, dw, [&](int t, int off) { out[t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(e.rs, off, 0, 0)); });
        return;
    }
    if (KHC > 0) {
        KH = KHC;
        KW = KWC;
        T = KHC * KWC;
    }
    int off[TM];
    const bool by_rows = g.whole_rows;
    const int centre_off = (chan * g.HW + th.p0) * 4;
#pragma unroll
    for (int t = 0; t < TM; t++)
        if (t < T) {
            int oh, ow;
            vm_tap(t, KH, KW, oh, ow);
            off[t] = centre_off + ((dh + oh) * g.W + dw + ow) * 4;
            const bool row_inside = th.active && (unsigned)(th.row0 + dh + oh) < (unsigned)g.H;
            if (V == 1) off[t] = row_inside && (unsigned)(th.col0 + dw + ow) < (unsigned)g.W ? off[t] : tile::kOob;
            else if (by_rows) off[t] = row_inside ? off[t] : tile::kOob;
            asm volatile("" : "+v"(off[t]));  // (see vm_ld_window_bf16)
            if (V == 4) {
                const tile::u32x4 d = tile::bload16(e.rs, off[t]);
#pragma unroll
                for (int k = 0; k < V; k++) out[t * V + k] = __uint_as_float(d[k]);
            } else if (V == 2) {
                const vm_u32x2 d = __builtin_amdgcn_raw_buffer_load_b64(e.rs, off[t], 0, 0);
#pragma unroll
                for (int k = 0; k < V; k++) out[t * V + k] = __uint_as_float(d[k]);
            } else {
                out[t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(e.rs, off[t], 0, 0));
            }
        }
    if (V == 1) return;
    const int reach = (((KH >> 1) + (dh < 0 ? -dh : dh)) * g.W + (KW >> 1) + (dw < 0 ? -dw : dw)) * 4;
    if (centre_off - reach < 0 || centre_off + reach + 4 * V > e.bytes) {
#pragma unroll
        for (int t = 0; t < TM; t++)
            if (t < T && tile::straddles_an_end(off[t], 4 * V, e.bytes)) {
#pragma unroll
                for (int k = 0; k < V; k++) out[t * V + k] = __uint_as_float(tile::elem_b32(e.rs, off[t] + 4 * k, e.bytes));
            }
    }
    uint32_t cm[KWC > 0 ? KWC : 1];  // valid pixels of a window column (the same for every row, if rows are inside as a whole)
#pragma unroll
    for (int t = 0; t < TM; t++)
        if (t < T) {
            int oh, ow;
            vm_tap(t, KH, KW, oh, ow);
            const int j = KWC > 0 ? ow + KWC / 2 : 0;
            if (by_rows) {
                if (KWC == 0 || t < KWC) {
                    const int first = -(th.col0 + dw + ow), behind = g.W - th.col0 - dw - ow;
                    cm[j] = vm_bits(first > 0 ? first : 0, behind < V ? behind : V);
                }
            } else {
                cm[j] = dh + oh == 0 && dw + ow == 0 ? 0xffffffffu : vm_valid<V>(g, th, dh + oh, dw + ow);
            }
#pragma unroll
            for (int k = 0; k < V; k++) out[t * V + k] = vm_keep(out[t * V + k], cm[j], k);
        }
}
#endif

// What an instruction needs besides its own fields.
struct Env {
    int c = 0;        // first channel of the trip; channel u of the thread is c + u
    int h = 0;        // channels of the trip that exist (0 .. U)
    bool pro = false; // the prologue of a pass (once per workgroup item, not per channel)
    bool fast = false; // Program::fast_math
    bool f32_windows = true;  // window loads of fp32 tensors by vm_ld_window_f32, not by the general loads; without taps: OP_LDFOLD
    int np = 0;       // persistent floats per pixel and channel
    int pstride = 0;  // floats between consecutive persistent floats of a thread (the workgroup's size)
    int rstride = 0;  // floats between consecutive register pieces of a thread
};

// The loads of OP_LD / OP_BINLD: lanes [0, T) of every channel of the trip into dst.
template <int TM, int V, int U>
CHAIN_HD void vm_ld(const Program& pg, const Geo& g, const Instr& I, const Env& ev, const Thread& th, float* dst, int T) {
    constexpr int TV = TM * V;
    const Tensor e = vm_tensor(pg, g, I.a);
#pragma unroll
    for (int u = 0; u < U; u++)
        if (u < ev.h) {
            int dh, dw;
            vm_offset(pg, I.b, ev.c + u, dh, dw);
            const int chan = (th.n * g.C + ev.c + u) * e.T;  // first plane of (image, channel): uniform
            if (I.kind & kWin) {
                const int KH = I.r >> 4, KW = I.r & 15;
#if defined(__HIP_DEVICE_COMPILE__)
                if ((V == 4 || V == 2 || V == 1) && e.bf16) {
                    // (the common windows with their sizes as constants: tap geometry folds, taps of one window row share
                    // the row test and taps of one window column the column masks)
                    float* out = dst + u * TV;
                    if (TM >= 9 && KH == 3 && KW == 3 && T == 9) vm_ld_window_bf16<TM, V, (TM >= 9 ? 3 : 0), (TM >= 9 ? 3 : 0)>(e, g, th, chan, dh, dw, 3, 3, 9, out);
                    else if (TM >= 25 && KH == 5 && KW == 5 && T == 25) vm_ld_window_bf16<TM, V, (TM >= 25 ? 5 : 0), (TM >= 25 ? 5 : 0)>(e, g, th, chan, dh, dw, 5, 5, 25, out);
                    else vm_ld_window_bf16<TM, V, 0, 0>(e, g, th, chan, dh, dw, KH, KW, T, out);
                    continue;
                }
                if ((V == 4 || V == 2 || V == 1) && ev.f32_windows) {
                    float* out = dst + u * TV;
                    if (TM >= 9 && KH == 3 && KW == 3 && T == 9) vm_ld_window_f32<TM, V, (TM >= 9 ? 3 : 0), (TM >= 9 ? 3 : 0)>(e, g, th, chan, dh, dw, 3, 3, 9, out);
                    else if (TM >= 25 && KH == 5 && KW == 5 && T == 25) vm_ld_window_f32<TM, V, (TM >= 25 ? 5 : 0), (TM >= 25 ? 5 : 0)>(e, g, th, chan, dh, dw, 5, 5, 25, out);
                    else vm_ld_window_f32<TM, V, 0, 0>(e, g, th, chan, dh, dw, KH, KW, T, out);
                    continue;
                }
#endif
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) {
                        int oh, ow;
                        vm_tap(t, KH, KW, oh, ow);
                        vm_load_at<V>(e, g, th, chan, dh + oh, dw + ow, dst + u * TV + t * V);
                    }
            } else {
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) {
                        const int te = (I.kind & kExtTaps) ? (t < e.T ? t : t % e.T) : 0;
                        vm_load_at<V>(e, g, th, chan + te, dh, dw, dst + u * TV + t * V);
                    }
            }
        }
}

// A = blend(X, A) (x_lhs) or blend(A, X), lanes [0, T) of every channel.  min and max return the same value whichever
// side is the LHS; the sides matter for sub only.
template <int TM, int V, int U>
CHAIN_HD void vm_blend_lanes(int kind, bool x_lhs, const float* X, float* A, int T) {
    switch (kind) {
    case 0: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = X[e] + A[e];); break;
    case 1: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = X[e] * A[e];); break;
    case 2:
        CHAIN_CASE;
        if (x_lhs) CHAIN_EACH(T, e, l, A[e] = X[e] - A[e];);
        else CHAIN_EACH(T, e, l, A[e] = A[e] - X[e];);
        break;
    case 3: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = X[e] <= A[e] ? X[e] : A[e];); break;
    default: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = X[e] >= A[e] ? X[e] : A[e];); break;
    }
}

// A row of a window as a thread of V pixels (4 or 8, of one image row) sees it: its pixels and two more on either side, 0 outside the
// image.  The main access is aligned and lies inside the tensor or is sent outside as a whole; so does each pair beside it.
// BF16: the tensor's type, as a constant: with a branch on it between the loads and their use the compiler waits for each load where it stands.
template <int V, bool BF16>
struct RowRaw {
    uint32_t d[BF16 ? V / 2 + 2 : V + 4];  // bf16: pairs; fp32: pixels
};
#if defined(__HIP_DEVICE_COMPILE__)
template <int V, bool BF16>
__device__ __forceinline__ void vm_row_issue(const Tensor& e, const Geo& g, const Thread& th, int chan, int row, RowRaw<V, BF16>& raw) {
    constexpr int es = BF16 ? 2 : 4;
    const bool ok = (int)th.active & (int)((unsigned)row < (unsigned)g.H);
    const int o = (chan * g.HW + row * g.W + th.col0) * es;
    int left = (int)ok & (int)(th.col0 > 0) ? o - 2 * es : tile::kOob, main = ok ? o : tile::kOob, right = (int)ok & (int)(th.col0 + V < g.W) ? o + V * es : tile::kOob;
    asm volatile("" : "+v"(left), "+v"(main), "+v"(right));
    if constexpr (BF16) {
        raw.d[0] = __builtin_amdgcn_raw_buffer_load_b32(e.rs, left, 0, 0);
        if constexpr (V == 8) {
            const tile::u32x4 m = tile::bload16(e.rs, main);
#pragma unroll
            for (int k = 0; k < 4; k++) raw.d[1 + k] = m[k];
        } else {
            const vm_u32x2 m = __builtin_amdgcn_raw_buffer_load_b64(e.rs, main, 0, 0);
            raw.d[1] = m[0];
            raw.d[2] = m[1];
        }
        raw.d[1 + V / 2] = __builtin_amdgcn_raw_buffer_load_b32(e.rs, right, 0, 0);
    } else {
        const vm_u32x2 l = __builtin_amdgcn_raw_buffer_load_b64(e.rs, left, 0, 0);
        raw.d[0] = l[0];
        raw.d[1] = l[1];
#pragma unroll
        for (int q = 0; q < V / 4; q++) {
            int p = main == tile::kOob ? tile::kOob : main + 16 * q;
            asm volatile("" : "+v"(p));
            const tile::u32x4 m = tile::bload16(e.rs, p);
#pragma unroll
            for (int k = 0; k < 4; k++) raw.d[2 + 4 * q + k] = m[k];
        }
        const vm_u32x2 r = __builtin_amdgcn_raw_buffer_load_b64(e.rs, right, 0, 0);
        raw.d[V + 2] = r[0];
        raw.d[V + 3] = r[1];
    }
}
#else
template <int V, bool BF16>
inline void vm_row_issue(const Tensor& e, const Geo& g, const Thread& th, int chan, int row, RowRaw<V, BF16>& raw) {
    for (int k = 0; k < V + 4; k++) {
        const int col = th.col0 + k - 2;
        const bool ok = th.active && (unsigned)row < (unsigned)g.H && (unsigned)col < (unsigned)g.W;
        const int64_t i = (int64_t)chan * g.HW + row * g.W + col;
        if (BF16) {
            const uint32_t h = ok ? ((const uint16_t*)e.ptr)[i] : 0;
            raw.d[k / 2] = k & 1 ? raw.d[k / 2] | h << 16 : h;
        } else {
            raw.d[k] = ok ? ((const uint32_t*)e.ptr)[i] : 0;
        }
    }
}
#endif
template <int V, bool BF16>
CHAIN_HD void vm_row_floats(const RowRaw<V, BF16>& raw, float* x) {
#pragma unroll
    for (int k = 0; k < V + 4; k++) {
        if (BF16) x[k] = vm_bits_to_f32(k & 1 ? raw.d[k / 2] & 0xffff0000u : raw.d[k / 2] << 16);
        else x[k] = vm_bits_to_f32(raw.d[BF16 ? 0 : k]);
    }
}

// One of the planner's streamable unaries (no clipped exp) on L lanes.
template <int L>
CHAIN_HD void vm_unary_lanes(int kind, bool fast, float* x) {
    switch (kind) {
    case 0:
        CHAIN_CASE;
#pragma unroll
        for (int e = 0; e < L; e++) x[e] = fmaxf(x[e], 0.f);
        break;
    case 1:
        CHAIN_CASE;
#pragma unroll
        for (int e = 0; e < L; e++) x[e] = fabsf(x[e]);
        break;
    case 2:
        CHAIN_CASE;
        if (fast) {
#pragma unroll
            for (int e = 0; e < L; e++) x[e] = vm_gelu_fast(x[e]);
        } else {
            for (int e = 0; e < L; e++) x[e] = vm_gelu(x[e]);
        }
        break;
    default:
        CHAIN_CASE;
#pragma unroll
        for (int e = 0; e < L; e++) x[e] = -x[e];
        break;
    }
}

// A row of an OP_LDFOLD: its KW taps, blended, join the fold.  x, y: the row of the tap's tensor and of the other operand (a second window's row, or
// the pixel's own value in y[2 ..]).  Sums begin at -0, which changes no first term.
template <int V, int KW, bool SECOND>
CHAIN_HD void vm_fold_row(const Instr& I, bool first, const float* x, const float* y, float* acc) {
    const int blend = I.kind & kLfBlend ? I.kind >> kLfBlendShift & 7 : 7;
#define CHAIN_TAPS(JOIN)                                                                       \
    _Pragma("unroll") for (int j = 0; j < KW; j++) {                                           \
        _Pragma("unroll") for (int v = 0; v < V; v++) {                                        \
            const float a = x[v + 2 + j - KW / 2], b = y[SECOND ? v + 2 + j - KW / 2 : v + 2]; \
            (void)b;                                                                           \
            JOIN;                                                                              \
        }                                                                                      \
    }
    if (vm_opaque((I.kind & 3) == 2)) {
        const int kind = vm_opaque(blend);
        CHAIN_TAPS({
            const float t = kind == 0 ? a + b : (kind == 1 ? a * b : (kind == 2 ? a - b : (kind == 3 ? b - a : a)));
            acc[v] = (first && j == 0) || t > acc[v] ? t : acc[v];
        })
        return;
    }
    switch (vm_opaque(blend)) {
    case 0: CHAIN_CASE; CHAIN_TAPS(acc[v] += a + b) break;
    case 1: CHAIN_CASE; CHAIN_TAPS(acc[v] += a * b) break;
    case 2: CHAIN_CASE; CHAIN_TAPS(acc[v] += a - b) break;
    case 3: CHAIN_CASE; CHAIN_TAPS(acc[v] += b - a) break;
    default: CHAIN_CASE; CHAIN_TAPS(acc[v] += a) break;
    }
#undef CHAIN_TAPS
}

// OP_LDFOLD for one channel: A (its V lanes) becomes the fold.  Row by row, the next row's loads in flight; a row is loaded and
// taken apart once for all its taps.  Taps are added in their order, as OP_FOLD adds them.
template <int V, bool BF16, bool SECOND, bool BF16_2>
CHAIN_HD void vm_ldfold(const Geo& g, const Instr& I, const Env& ev, const Thread& th, const Tensor& e, const Tensor& e2, int c, float* A) {
    const int KH = I.r >> 4, KW = I.r & 15;
    const int before = (int)I.f0;
    const int chan = th.n * g.C + c, row0 = th.row0 - KH / 2;
    float acc[V], x[V + 4], y[V + 4];
#pragma unroll
    for (int v = 0; v < V; v++) {
        acc[v] = -0.f;
        y[v + 2] = A[v];
    }
    RowRaw<V, BF16> n1;
    RowRaw<V, BF16_2> n2;
    vm_row_issue<V, BF16>(e, g, th, chan, row0, n1);
    if (SECOND) vm_row_issue<V, BF16_2>(e2, g, th, chan, row0, n2);
#pragma unroll 1
    for (int i = 0; i < KH; i++) {
        const RowRaw<V, BF16> r1 = n1;
        const RowRaw<V, BF16_2> r2 = n2;
        // (past the last row: row H, outside the image)
        vm_row_issue<V, BF16>(e, g, th, chan, i + 1 < KH ? row0 + i + 1 : g.H, n1);
        if (SECOND) vm_row_issue<V, BF16_2>(e2, g, th, chan, i + 1 < KH ? row0 + i + 1 : g.H, n2);
        vm_row_floats<V, BF16>(r1, x);
        if (vm_opaque(before) >= 0) vm_unary_lanes<V + 4>(before, ev.fast, x);
        if (SECOND) vm_row_floats<V, BF16_2>(r2, y);
        if (vm_opaque(KW) == 3) vm_fold_row<V, 3, SECOND>(I, i == 0, x, y, acc);
        else vm_fold_row<V, 5, SECOND>(I, i == 0, x, y, acc);
    }
    const bool avg = (I.kind & 3) == 1;
#pragma unroll
    for (int v = 0; v < V; v++) A[v] = avg ? vm_over(acc[v], (float)I.T) : acc[v];
}

// Every instruction except OP_XADD.  Pm: this thread's persistent floats.  A float that lives across the channel loop
// (softmax statistics, the sums of a softmax's adjoint: written by the prologue and the OP_SMC instructions) exists once,
// float k of pixel v at Pm[(k * V + v) * pstride]; an accumulator of one channel (OP_PSET in a body, OP_PADD, OP_PLD,
// OP_XADD) once per channel u of the trip, at Pm[((u * np + k) * V + v) * pstride].  Rm: its registers (vm_reg_read).
// TC: the lanes of the instruction as a constant (the loops over the taps then carry no test per tap), or 0 for I.T.
template <int TM, int V, int U, int TC>
CHAIN_HD void vm_exec_lanes(const Program& pg, const Geo& g, const Instr& I, const Env& ev, const Thread& th, State<TM, V, U>& st, float* Pm, float* Rm) {
    float* A = st.A;
    const int T = TC > 0 ? TC : I.T;
    const int pstride = ev.pstride, rstride = ev.rstride;
    constexpr int TV = TM * V;
    float X[U * TV];
    switch (I.op) {
    case OP_LD:
        CHAIN_CASE;
        vm_ld<TM, V, U>(pg, g, I, ev, th, A, T);
        break;
    case OP_BINLD: {
        CHAIN_CASE;
        const bool sc = I.kind & kBinLdLoadedScalar;
        vm_ld<TM, V, U>(pg, g, I, ev, th, X, sc ? 1 : T);
        if (TM > 1 && sc) CHAIN_EACH(T, e, l, X[e] = X[e - l + l % V];);
        vm_blend_lanes<TM, V, U>((I.kind >> kBinLdKindShift) & 7, (I.kind & kBinLdLoadedIsLhs) != 0, X, A, T);
        break;
    }
    case OP_MASK: {
        CHAIN_CASE;
#pragma unroll
        for (int u = 0; u < U; u++)
            if (u < ev.h) {
                int dh, dw;
                vm_offset(pg, I.b, ev.c + u, dh, dw);
                if (I.kind & kWin) {
                    const int KH = I.r >> 4, KW = I.r & 15;
#pragma unroll
                    for (int t = 0; t < TM; t++)
                        if (t < T) {
                            int oh, ow;
                            vm_tap(t, KH, KW, oh, ow);
                            const uint32_t m = vm_valid<V>(g, th, dh + oh, dw + ow);
#pragma unroll
                            for (int v = 0; v < V; v++) A[u * TV + t * V + v] = vm_keep(A[u * TV + t * V + v], m, v);
                        }
                } else {
                    const uint32_t m = vm_valid<V>(g, th, dh, dw);
#pragma unroll
                    for (int t = 0; t < TM; t++)
                        if (t < T) {
#pragma unroll
                            for (int v = 0; v < V; v++) A[u * TV + t * V + v] = vm_keep(A[u * TV + t * V + v], m, v);
                        }
                }
            }
        break;
    }
    case OP_UN:
        switch (I.kind) {
        case 0: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = fmaxf(A[e], 0.f);); break;
        case 1: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = fabsf(A[e]);); break;
        case 2:
            CHAIN_CASE;
            if (ev.fast) CHAIN_EACH(T, e, l, A[e] = vm_gelu_fast(A[e]););
            else CHAIN_EACH(T, e, l, A[e] = vm_gelu(A[e]););
            break;
        case 4: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = sinf(A[e]);); break;
        case kUnNeg: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = -A[e];); break;
        default:
            CHAIN_CASE;
            if (ev.fast) CHAIN_EACH(T, e, l, A[e] = vm_exp_fast(fminf(fmaxf(A[e], I.f0), I.f1)););
            else CHAIN_EACH(T, e, l, A[e] = expf(fminf(fmaxf(A[e], I.f0), I.f1)););
            break;
        }
        break;
    case OP_MOVR:
        CHAIN_CASE;
        vm_reg_write<TM, V, U>(Rm, rstride, I.r, T, A);
        break;
    case OP_MOVA:
        CHAIN_CASE;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, T, A);
        break;
    case OP_BIN: {
        CHAIN_CASE;
        const int kind = I.kind & 7;
        const bool reg_lhs = I.kind & kBinRegIsLhs, reg_sc = I.kind & kBinRegScalar, acc_sc = I.kind & kBinAccScalar;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, reg_sc ? 1 : T, X);
        if (TM > 1 && reg_sc) CHAIN_EACH(T, e, l, X[e] = X[e - l + l % V];);
        if (TM > 1 && acc_sc) CHAIN_EACH(T, e, l, A[e] = A[e - l + l % V];);
        vm_blend_lanes<TM, V, U>(kind, reg_lhs, X, A, T);
        break;
    }
    case OP_FOLD: {
        CHAIN_CASE;
#pragma unroll
        for (int u = 0; u < U; u++) {
            float* Au = A + u * TV;
            if (I.kind == 2) {
#pragma unroll
                for (int t = 1; t < TM; t++)
                    if (t < T) {
#pragma unroll
                        for (int v = 0; v < V; v++) Au[v] = Au[t * V + v] > Au[v] ? Au[t * V + v] : Au[v];
                    }
            } else {
#pragma unroll
                for (int t = 1; t < TM; t++)
                    if (t < T) {
#pragma unroll
                        for (int v = 0; v < V; v++) Au[v] += Au[t * V + v];
                    }
                if (I.kind == 1) {
#pragma unroll
                    for (int v = 0; v < V; v++) Au[v] = vm_over(Au[v], (float)T);
                }
            }
        }
        break;
    }
    case OP_SMT: {
        CHAIN_CASE;
#pragma unroll
        for (int u = 0; u < U; u++) {
            float* Au = A + u * TV;
#pragma unroll
            for (int v = 0; v < V; v++) {
                float m = Au[v];
#pragma unroll
                for (int t = 1; t < TM; t++)
                    if (t < T) m = fmaxf(m, Au[t * V + v]);
                float z = 0.f;
                if (ev.fast) {
#pragma unroll
                    for (int t = 0; t < TM; t++)
                        if (t < T) {
                            Au[t * V + v] = vm_exp_fast(Au[t * V + v] - m);
                            z += Au[t * V + v];
                        }
                    const float rz = vm_rcp_fast(z);
#pragma unroll
                    for (int t = 0; t < TM; t++)
                        if (t < T) Au[t * V + v] = Au[t * V + v] * rz;
                    continue;
                }
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) {
                        Au[t * V + v] = expf(Au[t * V + v] - m);
                        z += Au[t * V + v];
                    }
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) Au[t * V + v] = Au[t * V + v] / z;
            }
        }
        break;
    }
    case OP_ST: {
        CHAIN_CASE;
        if (!th.own) break;
        const Tensor e = vm_tensor(pg, g, I.a);
#pragma unroll
        for (int u = 0; u < U; u++)
            if (u < ev.h) {
                const int chan = (th.n * g.C + ev.c + u) * e.T;
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) vm_store<V>(e, (chan + t) * g.HW + th.p0, A + u * TV + t * V, (I.kind & kStAdd) != 0, g.ragged, g.HW - th.p0);
            }
        break;
    }
    case OP_UNBX:
        CHAIN_CASE;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, T, X);
        switch (I.kind) {
        case 0: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = A[e] > 0.f ? X[e] : 0.f;); break;
        case 1: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = X[e] * vm_sign(A[e]);); break;
        case 2:
            CHAIN_CASE;
            if (ev.fast) CHAIN_EACH(T, e, l, A[e] = X[e] * vm_gelu_grad_fast(A[e]););
            else CHAIN_EACH(T, e, l, A[e] = X[e] * vm_gelu_grad(A[e]););
            break;
        case 4: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = X[e] * cosf(A[e]);); break;
        case kUnNeg: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = -X[e];); break;
        default:
            CHAIN_CASE;
            if (ev.fast) CHAIN_EACH(T, e, l, A[e] = (A[e] > I.f0 && A[e] < I.f1) ? X[e] * vm_exp_fast(A[e]) : 0.f;);
            else CHAIN_EACH(T, e, l, A[e] = (A[e] > I.f0 && A[e] < I.f1) ? X[e] * expf(A[e]) : 0.f;);
            break;
        }
        break;
    case OP_BING: {
        CHAIN_CASE;
        const int kind = I.kind & 7;
        const bool rhs_side = I.kind & kBingRhsSide, l_sc = I.kind & kBingLhsScalar, r_sc = I.kind & kBingRhsScalar;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, l_sc ? 1 : T, X);
        if (TM > 1 && l_sc) CHAIN_EACH(T, e, l, X[e] = X[e - l + l % V];);
        if (TM > 1 && r_sc) CHAIN_EACH(T, e, l, A[e] = A[e - l + l % V];);
        // X: the LHS value, A: the RHS value; the result is d blend / d side (a tie of min / max belongs to the LHS)
        switch (kind) {
        case 0: CHAIN_CASE; CHAIN_EACH(T, e, l, A[e] = 1.f;); break;
        case 1:
            CHAIN_CASE;
            if (!rhs_side) break;  // d (l * r) / d l = r, which A holds
            CHAIN_EACH(T, e, l, A[e] = X[e];);
            break;
        case 2:
            CHAIN_CASE;
            if (rhs_side) CHAIN_EACH(T, e, l, A[e] = -1.f;);
            else CHAIN_EACH(T, e, l, A[e] = 1.f;);
            break;
        case 3:
            CHAIN_CASE;
            if (rhs_side) CHAIN_EACH(T, e, l, A[e] = X[e] <= A[e] ? 0.f : 1.f;);
            else CHAIN_EACH(T, e, l, A[e] = X[e] <= A[e] ? 1.f : 0.f;);
            break;
        default:
            CHAIN_CASE;
            if (rhs_side) CHAIN_EACH(T, e, l, A[e] = X[e] >= A[e] ? 0.f : 1.f;);
            else CHAIN_EACH(T, e, l, A[e] = X[e] >= A[e] ? 1.f : 0.f;);
            break;
        }
        break;
    }
    case OP_MADD:
        if constexpr (TM > 1) {
            CHAIN_CASE;
            vm_reg_read<TM, V, U>(Rm, rstride, I.r, T, X);
            vm_reg_madd<TM, V, U>(Rm, rstride, I.a, T, X, A);
        }
        break;
    case OP_SMTBX:
        CHAIN_CASE;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, T, X);
#pragma unroll
        for (int u = 0; u < U; u++) {
            float* Au = A + u * TV;
            const float* Xu = X + u * TV;
#pragma unroll
            for (int v = 0; v < V; v++) {
                float dot = 0.f;
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) dot += Xu[t * V + v] * Au[t * V + v];
                if (I.kind) {
#pragma unroll
                    for (int t = 0; t < TM; t++)
                        if (t < T) Au[t * V + v] = Xu[t * V + v] * (Au[t * V + v] - dot);
                } else {
#pragma unroll
                    for (int t = 0; t < TM; t++)
                        if (t < T) Au[t * V + v] = Au[t * V + v] * (Xu[t * V + v] - dot);
                }
            }
        }
        break;
    case OP_FOLDBX:
        CHAIN_CASE;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, 1, X);
        if (I.kind == 2) {
#pragma unroll
            for (int u = 0; u < U; u++) {
                float* Au = A + u * TV;
#pragma unroll
                for (int v = 0; v < V; v++) {
                    const float gr = X[u * TV + v];
                    int best = 0;
                    float m = Au[v];
#pragma unroll
                    for (int t = 1; t < TM; t++)
                        if (t < T && Au[t * V + v] > m) {
                            m = Au[t * V + v];
                            best = t;
                        }
#pragma unroll
                    for (int t = 0; t < TM; t++)
                        if (t < T) Au[t * V + v] = t == best ? gr : 0.f;
                }
            }
        } else {
            if (I.kind == 1) {
#pragma unroll
                for (int u = 0; u < U; u++)
#pragma unroll
                    for (int v = 0; v < V; v++) X[u * TV + v] = X[u * TV + v] / (TM == 1 && I.f0 > 0.f ? I.f0 : (float)T);
            }
            CHAIN_EACH(T, e, l, A[e] = X[e - l + l % V];);
        }
        break;
    case OP_PSET:
        CHAIN_CASE;
        if (ev.pro) {
#pragma unroll
            for (int t = 0; t < TM; t++)
                if (t < T) {
#pragma unroll
                    for (int v = 0; v < V; v++) Pm[((I.a + t) * V + v) * pstride] = I.f0;
                }
        } else {
            CHAIN_EACH(T, e, l, Pm[(((e - l) / TV * ev.np + I.a) * V + l) * pstride] = I.f0;);
        }
        break;
    case OP_PADD: {
        CHAIN_CASE;
        const int Tb = I.b;
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int t = 0; t < TM; t++)
                if (t < T) {
                    const int tp = t < Tb ? t : t % Tb;
#pragma unroll
                    for (int v = 0; v < V; v++) Pm[((u * ev.np + I.a + tp) * V + v) * pstride] += A[u * TV + t * V + v];
                }
        break;
    }
    case OP_PLD:
        CHAIN_CASE;
        CHAIN_EACH(T, e, l, A[e] = Pm[(((e - l) / TV * ev.np + I.a) * V + l) * pstride];);
        break;
    case OP_SMCSTAT:
        CHAIN_CASE;
        if (ev.fast) {
            // the channels of the trip join the running maximum and sum together: one update of the pair per pixel and
            // trip, U + 1 exponentials for U channels, no branch on the data
#pragma unroll
            for (int t = 0; t < TM; t++)
                if (t < T) {
#pragma unroll
                    for (int v = 0; v < V; v++) {
                        float& m = Pm[((I.a + t) * V + v) * pstride];
                        float& z = Pm[((I.a + T + t) * V + v) * pstride];
                        const float before = m;
                        float top = before;
#pragma unroll
                        for (int u = 0; u < U; u++)
                            if (u < ev.h) top = fmaxf(top, A[u * TV + t * V + v]);
                        float sum = z * vm_exp_fast(before - top);  // (before = -inf at the first channel: 0 * 0)
#pragma unroll
                        for (int u = 0; u < U; u++)
                            if (u < ev.h) sum += vm_exp_fast(A[u * TV + t * V + v] - top);
                        m = top;
                        z = sum;
                    }
                }
            break;
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (u < ev.h) {
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) {
#pragma unroll
                        for (int v = 0; v < V; v++) {
                            float& m = Pm[((I.a + t) * V + v) * pstride];
                            float& z = Pm[((I.a + T + t) * V + v) * pstride];
                            const float val = A[u * TV + t * V + v];
                            if (val > m) {
                                z = z * expf(m - val) + 1.f;  // (m = -inf at the first channel: z = 0 * 0 + 1)
                                m = val;
                            } else {
                                z += expf(val - m);
                            }
                        }
                    }
            }
        break;
    case OP_SMCAPPLY:
        CHAIN_CASE;
        if (ev.fast) CHAIN_EACH(T, e, l, A[e] = vm_exp_fast(A[e] - Pm[(I.a * V + l) * pstride]) * vm_rcp_fast(Pm[((I.a + T) * V + l) * pstride]););
        else CHAIN_EACH(T, e, l, A[e] = expf(A[e] - Pm[(I.a * V + l) * pstride]) / Pm[((I.a + T) * V + l) * pstride];);
        break;
    case OP_SMCDOT:
        CHAIN_CASE;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, T, X);
#pragma unroll
        for (int u = 0; u < U; u++)
            if (u < ev.h) {
#pragma unroll
                for (int t = 0; t < TM; t++)
                    if (t < T) {
#pragma unroll
                        for (int v = 0; v < V; v++) Pm[((I.a + t) * V + v) * pstride] += A[u * TV + t * V + v] * X[u * TV + t * V + v];
                    }
            }
        break;
    case OP_SMCBX:
        CHAIN_CASE;
        vm_reg_read<TM, V, U>(Rm, rstride, I.r, T, X);
        CHAIN_EACH(T, e, l, A[e] = A[e] * (X[e] - Pm[(I.a * V + l) * pstride]););
        break;
    case OP_LDFOLD:
        if constexpr (TM == 1 && (V == 4 || V == 8)) {
            if (!ev.f32_windows) break;
            CHAIN_CASE;
            const Tensor e = vm_tensor(pg, g, I.a);
            const Tensor e2 = vm_tensor(pg, g, (I.kind & kLfSecond) ? I.b : I.a);
            // (one copy of the code for all channels of the trip: as many copies as channels spilled scalar registers)
#pragma unroll 1
            for (int u = 0; u < ev.h; u++) {
                float a[V];
#pragma unroll
                for (int v = 0; v < V; v++) {
                    a[v] = A[v];
#pragma unroll
                    for (int w = 1; w < U; w++) a[v] = u == w ? A[w * V + v] : a[v];
                }
                const int c = ev.c + u;
                switch (vm_opaque((e.bf16 ? 1 : 0) | ((I.kind & kLfSecond) ? (e2.bf16 ? 6 : 2) : 0))) {
                case 0: vm_ldfold<V, false, false, false>(g, I, ev, th, e, e2, c, a); break;
                case 1: vm_ldfold<V, true, false, false>(g, I, ev, th, e, e2, c, a); break;
                case 2: vm_ldfold<V, false, true, false>(g, I, ev, th, e, e2, c, a); break;
                case 3: vm_ldfold<V, true, true, false>(g, I, ev, th, e, e2, c, a); break;
                case 6: vm_ldfold<V, false, true, true>(g, I, ev, th, e, e2, c, a); break;
                default: vm_ldfold<V, true, true, true>(g, I, ev, th, e, e2, c, a); break;
                }
#pragma unroll
                for (int w = 0; w < U; w++)
#pragma unroll
                    for (int v = 0; v < V; v++) A[w * V + v] = u == w ? a[v] : A[w * V + v];
            }
        }
        break;
    default: break;
    }
}

// An instruction over all TM lanes of the instance (the common case of a program with taps) runs the copy of the
// dispatch whose tap loops are straight-line code, in the one-pixel instances as well: with one channel per trip the second
// copy fits them (9 lanes: 99 registers, four wavefronts per SIMD; 25 lanes: 201, two, as geometry_for() counts).
template <int TM, int V, int U>
CHAIN_HD void vm_exec(const Program& pg, const Geo& g, const Instr& I, const Env& ev, const Thread& th, State<TM, V, U>& st, float* Pm, float* Rm) {
    constexpr int TC = TM > 1 ? TM : 0;
    if (TC > 0 && I.T == TM) vm_exec_lanes<TM, V, U, TC>(pg, g, I, ev, th, st, Pm, Rm);
    else vm_exec_lanes<TM, V, U, 0>(pg, g, I, ev, th, st, Pm, Rm);
}

// OP_XADD of channel u, first half: the thread's lanes go to the hand-over buffer of its slice (lane t of local pixel q
// at buf[t * npx + q]).
template <int TM, int V>
CHAIN_HD void vm_xadd_write(const Geo& g, const Instr& I, const Thread& th, const float* Au, float* buf) {
#pragma unroll
    for (int t = 0; t < TM; t++)
        if (t < I.T) {
#pragma unroll
            for (int v = 0; v < V; v++) buf[t * g.npx + th.ptid * V + v] = Au[t * V + v];
        }
}

// The gather of OP_XADD for one pixel per thread and a window over a tensor without taps: the sum of the lanes whose
// window reached this pixel.  Only pixels the workgroup owns need it, and the halo holds every source of theirs, so a
// source is tested against the image alone: once per window row, once per window column.  All reads are issued before
// the first is added.  KHC x KWC: the window as constants, or 0 x 0 for the window (KH, KW).  (Backward of a 5x5 window
// under a product and an avg fold, 16x96 planes of 32x32: 515 us with the general gather below and a test per tap in every
// instruction, 369 us.)
template <int TM, int KHC, int KWC>
CHAIN_HD float vm_xadd_window(const Geo& g, int KH, int KW, int T, int dh, int dw, const Thread& th, const float* buf) {
    if (KHC > 0) {
        KH = KHC;
        KW = KWC;
        T = KHC * KWC;
    }
    float got[TM];
    const int base = th.ptid - (dh * g.W + dw);
#pragma unroll
    for (int t = 0; t < TM; t++)
        if (t < T) {
            int oh, ow;
            vm_tap(t, KH, KW, oh, ow);
            const bool ok = th.own && (unsigned)(th.row0 - dh - oh) < (unsigned)g.H && (unsigned)(th.col0 - dw - ow) < (unsigned)g.W;
            const float x = buf[t * g.npx + (ok ? base - (oh * g.W + ow) : th.ptid)];
            got[t] = ok ? x : 0.f;
        }
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < TM; t++)
        if (t < T) sum += got[t];
    return sum;
}

// The same for a 3x3 window and V pixels per thread: summed in registers (the general gather below adds every tap to P, in LDS, each behind the last: backward
// of unfold 3x3 -> softmax -> product -> gelu -> sum, 16x96 planes of 32x32, 109 us, now 97).
template <int TM, int V>
CHAIN_HD void vm_xadd_window3(const Geo& g, int dh, int dw, const Thread& th, const float* buf, float (&sum)[V]) {
#pragma unroll
    for (int v = 0; v < V; v++) sum[v] = 0.f;
#pragma unroll
    for (int t = 0; t < 9; t++) {
        int oh, ow;
        vm_tap(t, 3, 3, oh, ow);
        oh += dh;
        ow += dw;
        const uint32_t m = th.own ? vm_valid<V>(g, th, -oh, -ow) : 0u;
        const int at = th.ptid * V - (oh * g.W + ow);
#pragma unroll
        for (int v = 0; v < V; v++) {
            const bool ok = (m >> v) & 1u;
            const float x = buf[t * g.npx + (ok ? at + v : th.ptid * V)];
            sum[v] += ok ? x : 0.f;
        }
    }
}

// OP_XADD of channel u, second half (after a barrier): P[a (+ t)] of every pixel of the thread collects lane t of the
// pixel whose load at offset (dh, dw) [+ window tap t] read it, if that pixel is inside the image and inside the pixels
// the slice computes (the planner sizes the halo so that an owned pixel never misses one).  Fixed order: deterministic.
// Pu: the persistent floats of this thread and channel.
template <int TM, int V>
CHAIN_HD void vm_xadd_gather(const Geo& g, const Instr& I, int dh, int dw, const Thread& th, const float* buf, float* Pu, int pstride) {
    if (V == 1 && TM > 1 && (I.kind & kWin) && !(I.kind & kExtTaps)) {
        const int KH = I.r >> 4, KW = I.r & 15, T = I.T;
        float sum;
        if (TM >= 9 && KH == 3 && KW == 3 && T == 9) sum = vm_xadd_window<TM, (TM >= 9 ? 3 : 0), (TM >= 9 ? 3 : 0)>(g, 3, 3, 9, dh, dw, th, buf);
        else if (TM >= 25 && KH == 5 && KW == 5 && T == 25) sum = vm_xadd_window<TM, (TM >= 25 ? 5 : 0), (TM >= 25 ? 5 : 0)>(g, 5, 5, 25, dh, dw, th, buf);
        else sum = vm_xadd_window<TM, 0, 0>(g, KH, KW, T, dh, dw, th, buf);
        if (th.own) Pu[I.a * pstride] += sum;
        return;
    }
    if constexpr (V == 2 && TM >= 9) {
        if ((I.kind & kWin) && !(I.kind & kExtTaps) && I.r == 0x33 && I.T == 9) {
            float sum[V];
            vm_xadd_window3<TM, V>(g, dh, dw, th, buf, sum);
#pragma unroll
            for (int v = 0; v < V; v++)
                if (th.own) Pu[(I.a * V + v) * pstride] += sum[v];
            return;
        }
    }
#pragma unroll
    for (int t = 0; t < TM; t++)
        if (t < I.T) {
            int oh = dh, ow = dw;
            if (I.kind & kWin) {
                int th_, tw_;
                vm_tap(t, I.r >> 4, I.r & 15, th_, tw_);
                oh += th_;
                ow += tw_;
            }
            // the source of pixel (r, c) is pixel (r - oh, c - ow)
            const uint32_t m = vm_valid<V>(g, th, -oh, -ow);
            const int slot = I.a + ((I.kind & kExtTaps) ? t : 0);
#pragma unroll
            for (int v = 0; v < V; v++) {
                const int src = th.ptid * V + v - (oh * g.W + ow);
                if (((m >> v) & 1u) && src >= 0 && src < g.npx) Pu[(slot * V + v) * pstride] += buf[t * g.npx + src];
            }
        }
}

// Combination of the slices' partial results of lane e (= t * V + v) of a Red (see chain_isa.hpp) for the pixels of
// thread `ptid`: float k of slice s is at Pbase[(k * V + v) * pstride + s * pix_threads + ptid].  kind 0 returns the
// total maximum and sum.
template <int V>
CHAIN_HD void vm_combine(const Red& R, int e, int S, int PT, const float* Pbase, int pstride, int ptid, float& v0, float& v1) {
    const float* p0 = Pbase + (R.slot * V + e) * pstride + ptid;
    if (R.kind == 0) {
        const float* p1 = Pbase + ((R.slot + R.T) * V + e) * pstride + ptid;
        float m = -INFINITY;
        for (int s = 0; s < S; s++) m = fmaxf(m, p0[s * PT]);
        float z = 0.f;
        for (int s = 0; s < S; s++) {
            const float zs = p1[s * PT];
            if (zs > 0.f) z += zs * expf(p0[s * PT] - m);  // (a slice without channels has no sum and no maximum)
        }
        v0 = m;
        v1 = z;
    } else {
        float d = 0.f;
        for (int s = 0; s < S; s++) d += p0[s * PT];
        v0 = d;
        v1 = 0.f;
    }
}

}  // namespace chain
}  // namespace canvas
