// Softmax over channels: a workgroup takes the pixels of one wavefront and all channels, which its wavefronts share; a thread keeps its
// channels' values in registers, so every tensor is read once, and the wavefronts exchange maximum and sum (backward: then the
// sum of gradient x result) through LDS.  Bound by memory for large tensors, by three dependent steps (loads, exchange, stores) for small ones.
// As interpreted programs of the fused-chain kernels, us: 16x96 planes of 32x32 forward 18-21, backward 28-38 (here 5.6-6.3 and 6.6-11.5); 128x64 of 56x56
// forward + backward 246 (78), 32x256 of 14x14 104 (18), 64x128 of 27x29 187 (40).
#include "smc_kernels.hpp"

#include <algorithm>
#include <cstddef>

#include "launch.hpp"
#include "tile_util.hpp"
#include "ufc_device.hpp"

namespace canvas {
namespace smc {

namespace {

using namespace canvas::tile;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int V, bool F32>
__device__ __forceinline__ void load(const void* p, int64_t e, float (&v)[V]) {
    if constexpr (F32) {
        const float* q = (const float*)p + e;
        if constexpr (V == 4) {
            const float4_t x = *(const float4_t*)q;
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] = x[k];
        } else if constexpr (V == 2) {
            const float2_t x = *(const float2_t*)q;
            v[0] = x[0];
            v[1] = x[1];
        } else {
            v[0] = *q;
        }
    } else {
        const uint16_t* q = (const uint16_t*)p + e;
        if constexpr (V == 4) {
            const u32x2 x = *(const u32x2*)q;
#pragma unroll
            for (int k = 0; k < 2; k++) {
                v[2 * k] = lo_f32(x[k]);
                v[2 * k + 1] = hi_f32(x[k]);
            }
        } else if constexpr (V == 2) {
            const uint32_t x = *(const uint32_t*)q;
            v[0] = lo_f32(x);
            v[1] = hi_f32(x);
        } else {
            v[0] = lo_f32(*q);
        }
    }
}
template <int V, bool F32>
__device__ __forceinline__ void store(void* p, int64_t e, float (&v)[V], bool acc) {
    if constexpr (F32) {
        float* q = (float*)p + e;
        if (acc) {
            float old[V];
            load<V, true>(p, e, old);
#pragma unroll
            for (int k = 0; k < V; k++) v[k] += old[k];
        }
        if constexpr (V == 4) *(float4_t*)q = float4_t{v[0], v[1], v[2], v[3]};
        else if constexpr (V == 2) *(float2_t*)q = float2_t{v[0], v[1]};
        else *q = v[0];
    } else {
        uint16_t* q = (uint16_t*)p + e;
        if constexpr (V == 4) *(u32x2*)q = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        else if constexpr (V == 2) *(uint32_t*)q = pack_bf16(v[0], v[1]);
        else *q = (uint16_t)(pack_bf16(v[0], 0.f) & 0xffffu);
    }
}

// act(x) and, where wanted, act'(x), for a uniform kind
template <bool GRAD>
__device__ __forceinline__ float unary(int kind, bool fast, float x, float& d) {
    if (kind == 2) {
        if (fast) {
            float cdf, pdf;
            ufc::normal_parts(x, cdf, pdf);
            if (GRAD) d = cdf + x * pdf;
            return x * cdf;
        }
        if (GRAD) d = unary_grad(2, x, 0.f, 0.f);
        return unary_apply(2, x, 0.f, 0.f);
    }
    if (GRAD) d = x > 0.f ? 1.f : (x < 0.f && kind == 1 ? -1.f : 0.f);
    return kind == 0 ? __builtin_fmaxf(x, 0.f) : fabsf(x);
}

template <int V, int CPT, bool XF, bool GF, bool OF, bool BWD>
__global__ __launch_bounds__(1024) void k_softmax_c(Params P) {
    extern __shared__ __align__(16) float lds[];  // [slices][2][64 * V], backward: [slices][64 * V] more
    const int lane = threadIdx.x & 63, S = P.slices;
    const int slice = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = blockIdx.x / P.tiles, tile = blockIdx.x - n * P.tiles;
    const int p = (tile * 64 + lane) * V;
    const bool in = p < P.P;  // (V divides the plane)
    const int c0 = slice * CPT, nc = min(CPT, P.C - c0);  // (one channel at least)
    const int64_t base = ((int64_t)n * P.C + c0) * P.P + (in ? p : 0);
    float x[CPT][V], g[BWD ? CPT : 1][V];
#pragma unroll
    for (int k = 0; k < CPT; k++) load<V, XF>(P.x, base + (int64_t)min(k, nc - 1) * P.P, x[k]);  // (past the last channel: the last one again)
    if constexpr (BWD) {
#pragma unroll
        for (int k = 0; k < CPT; k++) load<V, GF>(P.dy, base + (int64_t)min(k, nc - 1) * P.P, g[k]);
    }
#pragma unroll 1
    for (int i = 0; i < P.n_before; i++) {
        const int kind = P.before[i];
        float unused;
#pragma unroll
        for (int k = 0; k < CPT; k++)
#pragma unroll
            for (int v = 0; v < V; v++) x[k][v] = unary<false>(kind, P.fast, x[k][v], unused);
    }
    // maximum and sum of this thread's channels, then of all
    float m[V], z[V];
#pragma unroll
    for (int v = 0; v < V; v++) {
        m[v] = -INFINITY;
        z[v] = 0.f;
    }
#pragma unroll
    for (int k = 0; k < CPT; k++)
        if (k < nc) {
#pragma unroll
            for (int v = 0; v < V; v++) m[v] = fmaxf(m[v], x[k][v]);
        }
    float base_m[V];  // (channels that are all -inf have no sum)
#pragma unroll
    for (int v = 0; v < V; v++) base_m[v] = m[v] == -INFINITY ? 0.f : m[v];
#pragma unroll
    for (int k = 0; k < CPT; k++)
        if (k < nc) {
#pragma unroll
            for (int v = 0; v < V; v++) {
                const float d = x[k][v] - base_m[v];
                x[k][v] = P.fast ? __expf(d) : expf(d);
                z[v] += x[k][v];
            }
        }
    float* const pm = lds + slice * 128 * V + lane;
#pragma unroll
    for (int v = 0; v < V; v++) {
        pm[v * 64] = m[v];
        pm[(V + v) * 64] = z[v];
    }
    __syncthreads();
    float scale[V];
#pragma unroll
    for (int v = 0; v < V; v++) {
        float top = -INFINITY;
        for (int s = 0; s < S; s++) top = fmaxf(top, lds[s * 128 * V + v * 64 + lane]);
        float sum = 0.f;
        for (int s = 0; s < S; s++) {
            const float d = lds[s * 128 * V + v * 64 + lane] - top;
            sum += lds[s * 128 * V + (V + v) * 64 + lane] * (P.fast ? __expf(d) : expf(d));
        }
        const float d = m[v] - top, e = P.fast ? __expf(d) : expf(d);
        scale[v] = P.fast ? e * __builtin_amdgcn_rcpf(sum) : e / sum;
    }
#pragma unroll
    for (int k = 0; k < CPT; k++)
#pragma unroll
        for (int v = 0; v < V; v++) x[k][v] = k < nc ? x[k][v] * scale[v] : 0.f;
    if constexpr (BWD) {
        float dot[V];
#pragma unroll
        for (int v = 0; v < V; v++) dot[v] = 0.f;
#pragma unroll
        for (int k = 0; k < CPT; k++)
            if (k < nc) {
#pragma unroll
                for (int v = 0; v < V; v++) dot[v] += x[k][v] * g[k][v];
            }
        float* const pd = lds + S * 128 * V;
#pragma unroll
        for (int v = 0; v < V; v++) pd[(slice * V + v) * 64 + lane] = dot[v];
        __syncthreads();
#pragma unroll
        for (int v = 0; v < V; v++) {
            dot[v] = 0.f;
            for (int s = 0; s < S; s++) dot[v] += pd[(s * V + v) * 64 + lane];
        }
#pragma unroll
        for (int k = 0; k < CPT; k++)
            if (k < nc) {
#pragma unroll
                for (int v = 0; v < V; v++) x[k][v] = x[k][v] * (g[k][v] - dot[v]);
            }
        if (P.n_before > 0) {  // (x once more: from the caches)
#pragma unroll
            for (int k = 0; k < CPT; k++) load<V, XF>(P.x, base + (int64_t)min(k, nc - 1) * P.P, g[k]);
#pragma unroll 1
            for (int i = 0; i < P.n_before; i++) {
                const int kind = P.before[i];
#pragma unroll
                for (int k = 0; k < CPT; k++)
#pragma unroll
                    for (int v = 0; v < V; v++) {
                        float d;
                        g[k][v] = unary<true>(kind, P.fast, g[k][v], d);
                        x[k][v] = kind == 0 && d == 0.f ? 0.f : x[k][v] * d;  // (relu selects, whatever the gradient)
                    }
            }
        }
    }
    if (!in) return;
#pragma unroll
    for (int k = 0; k < CPT; k++)
        if (k < nc) store<V, OF>(P.out, base + (int64_t)k * P.P, x[k], BWD && P.acc);
}

template <bool XF, bool GF, bool OF, bool BWD>
void launch(const Params& P, hipStream_t s) {
    const dim3 grid((unsigned)((int64_t)P.N * P.tiles)), block((unsigned)(64 * P.slices));
    const size_t lds = (size_t)P.slices * 64 * P.vec * (BWD ? 3 : 2) * sizeof(float);
    if (P.cpt == 8) {
        if (P.vec == 4) CANVAS_LAUNCH((k_softmax_c<4, 8, XF, GF, OF, BWD>), grid, block, lds, s, P);
        else if (P.vec == 2) CANVAS_LAUNCH((k_softmax_c<2, 8, XF, GF, OF, BWD>), grid, block, lds, s, P);
        else CANVAS_LAUNCH((k_softmax_c<1, 8, XF, GF, OF, BWD>), grid, block, lds, s, P);
    } else {
        if (P.vec == 2) CANVAS_LAUNCH((k_softmax_c<2, 16, XF, GF, OF, BWD>), grid, block, lds, s, P);
        else CANVAS_LAUNCH((k_softmax_c<1, 16, XF, GF, OF, BWD>), grid, block, lds, s, P);
    }
}

}  // namespace

bool plan(Params& P, int N, int C, int pixels) {
    if (C > 256 || (int64_t)N * ((pixels + 63) / 64) >= ((int64_t)1 << 31)) return false;
    P.N = N;
    P.C = C;
    P.P = pixels;
    P.cpt = C <= 128 ? 8 : 16;
    P.slices = (C + P.cpt - 1) / P.cpt;
    // as many pixels per thread as leave two workgroups per compute unit
    for (P.vec = P.cpt == 8 ? 4 : 2; P.vec > 1; P.vec /= 2)
        if (pixels % P.vec == 0 && (int64_t)N * ((pixels + 64 * P.vec - 1) / (64 * P.vec)) >= 512) break;
    P.tiles = (pixels + 64 * P.vec - 1) / (64 * P.vec);
    return true;
}

void forward(const Params& P, hipStream_t s) {
    if (P.x_f32) {
        if (P.out_f32) launch<true, false, true, false>(P, s);
        else launch<true, false, false, false>(P, s);
    } else {
        if (P.out_f32) launch<false, false, true, false>(P, s);
        else launch<false, false, false, false>(P, s);
    }
}

void backward(const Params& P, hipStream_t s) {
    if (P.x_f32) {
        if (P.dy_f32) {
            if (P.out_f32) launch<true, true, true, true>(P, s);
            else launch<true, true, false, true>(P, s);
        } else {
            if (P.out_f32) launch<true, false, true, true>(P, s);
            else launch<true, false, false, true>(P, s);
        }
    } else {
        if (P.dy_f32) {
            if (P.out_f32) launch<false, true, true, true>(P, s);
            else launch<false, true, false, true>(P, s);
        } else {
            if (P.out_f32) launch<false, false, true, true>(P, s);
            else launch<false, false, false, true>(P, s);
        }
    }
}

}  // namespace smc
}  // namespace canvas
