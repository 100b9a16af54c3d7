// The fp32 contraction on the bf16 matrix instructions, without loss: every operand is cut into three bf16 parts that hold all
// of its 24 bits, x = h + m + l, and a product is the six parts' products down to 2^-24 of it,
//     x * w = hh' + (hm' + mh' + mm' + hl' + lh') + [ml' + lm' + ll' < 2^-24, dropped],
// each exact in the matrix unit.  v_mfma_f32_32x32x16_bf16 does 16 times the work of the fp32 instruction, six of them 2.7
// times.
#include <algorithm>

#include "launch.hpp"
#include "sfc_device.hpp"
#include "tile_util.hpp"

namespace canvas {
namespace sfc {

namespace {

using tile::bf16x8_t;
using tile::u32x4;
using f16v = __attribute__((ext_vector_type(16))) float;

constexpr int kThreads = 256;
constexpr int kNotMfma = 0x3f6;  // what may move across a scheduling barrier: anything but matrix instructions

__device__ __forceinline__ f16v mfma(const u32x4& a, const u32x4& b, f16v c) {
    bf16x8_t av, bv;
    __builtin_memcpy(&av, &a, 16);
    __builtin_memcpy(&bv, &b, 16);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, c, 0, 0, 0);
}

// Eight floats -> their three bf16 parts.  A value that is infinite, NaN or rounds to an infinity makes the second part NaN:
// every result that it reaches is NaN then, and is computed again in fp32.
__device__ __forceinline__ void split8(const float (&v)[8], u32x4& h, u32x4& m, u32x4& l) {
#pragma unroll
    for (int k = 0; k < 4; k++) {
        h[k] = tile::pack_bf16(v[2 * k], v[2 * k + 1]);
        const float r0 = v[2 * k] - tile::lo_f32(h[k]), r1 = v[2 * k + 1] - tile::hi_f32(h[k]);
        m[k] = tile::pack_bf16(r0, r1);
        l[k] = tile::pack_bf16(r0 - tile::lo_f32(m[k]), r1 - tile::hi_f32(m[k]));
    }
}

// Forward and data gradient.  A workgroup owns 32*WM outputs of one group and 32*(4/WM) consecutive pixels of the batch, a
// wavefront 32 x 32 of them; a step is one matrix instruction's depth, 16 channels of one tap, a chunk of the operand tile 16
// channels with their nine taps, or 64 channels without a window.  The weights come cut and in the order of the matrix
// operands from k_split_weights, once per step of training: cut by every workgroup again they cost as many vector
// instructions as the rest of the kernel, and their LDS tile left room for two workgroups per compute unit (30 us at the
// size below).  A wavefront reads the three kilobytes of a step straight from the caches, AHEAD steps ahead.  The operand
// tile is read as eight channels per thread into registers while the chunk before is multiplied, cut and put into the other
// of two LDS buffers, [part][half][position] with image rows and a zero margin as in k_fwd, so that a tap is an LDS offset.
// Sums: the leading products of a chunk are chained in the matrix unit, the chunks added in fp32; the small products have a
// chain of their own over all chunks, which joins at the end.
// Bound by the latency of its chunks: in a wavefront the loads of a chunk's operand tile come back in order with those of the
// weights, so that every chunk takes the round trip of its tile (0.18 us a step where six matrix instructions take 0.08), with
// one and a half wavefronts per SIMD at the size below.  N=32, C=64, 28x28, 3x3 (1.85 GFLOP): 21 us, 88 TFLOP/s (k_fwd 38.6);
// 32 x 512 channels of 14x14 without a window: 41 us, 80 TFLOP/s (69).  Errors against fp64 below k_fwd's: 3x3, 64 / 128 channels
// 7.9 / 8.8e-8 (1.04 / 1.27e-7), without a window 5.0 / 5.7e-8 (8.5 / 9.3e-8).
template <int WM, int TVT, int NPI>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_fwd_split(Params Q) {
    constexpr bool WIN = TVT > 1;
    constexpr int NS = WIN ? TVT : 4, CH = WIN ? 16 : 64, AHEAD = !WIN ? 3 : (NPI == 2 ? 4 : 2);
    constexpr int TP = 32 * (4 / WM);
    extern __shared__ u32x4 lds_split[];  // [2][3][2][XH], without a window [2][3][4][2][TP]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
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
    const int o0 = (mtile * WM + wm) * 32;
    const int64_t P = Q.P;
    constexpr int XPART = NPI * kThreads, XH = WIN ? XPART / 2 : TP;  // LDS strides of the parts and halves
    const int S = WIN ? Q.S : TP;

    // where this thread's items of the operand tile (half of the 16 channels, position) come from; byte offsets from uniform
    // addresses, so that a load costs no vector arithmetic (the host checks that they fit 32 bits)
    const float* const src = Q.src + (n0 * Q.G + g) * Q.R * P;
    uint32_t xat[NPI];
    int xch[NPI];  // first channel of the item in the chunk; -1: in the margin
#pragma unroll
    for (int i = 0; i < NPI; i++) {
        const int id = tid + i * kThreads;
        int64_t at;
        int ch;
        if (WIN) {
            const int hf = id >= XH ? 1 : 0, j = id - hf * XH;
            at = j < S ? window_source(Q, n0, h0, j) : -1;
            if (at >= 0) at -= n0 * Q.G * Q.R * P;
            ch = hf * 8;
        } else {
            const int j = id % TP, p = p0 + j, dn = image_of(Q, p);
            at = m0 + j < Q.M ? dn * Q.G * Q.R * P + (p - dn * Q.P) : -1;
            ch = id / TP * 8;
        }
        xch[i] = at >= 0 ? ch : -1;
        xat[i] = at >= 0 ? (uint32_t)(at + ch * P) * 4u : 0u;
    }
    float xreg[NPI][8];
    auto at = [](const float* base, uint32_t bytes) { return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + bytes); };
    auto load = [&](int r0) {
        if (r0 + CH <= Q.R) {
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const float* const xk = src + (r0 + k) * P;
#pragma unroll
                for (int i = 0; i < NPI; i++) xreg[i][k] = at(xk, xat[i]);
            }
        } else {  // (the last channel again past the end; an item's channels count from its own first)
            int left = Q.R - 1 - r0;
            asm volatile("" : "+s"(left));  // (keeps these addresses out of the registers of the main loop)
#pragma unroll
            for (int i = 0; i < NPI; i++)
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const int c = max(xch[i], 0);
                    xreg[i][k] = at(src + r0 * P, xat[i] + (uint32_t)((min(c + k, left) - c) * Q.P) * 4u);
                }
        }
    };
    auto store = [&](int r0, u32x4* to) {  // (channels past the last and the margin are zero)
        const bool ragged = r0 + CH > Q.R;
#pragma unroll
        for (int i = 0; i < NPI; i++) {
            const int id = tid + i * kThreads;  // (the items are numbered as they lie in LDS)
            if (ragged)
#pragma unroll
                for (int k = 0; k < 8; k++) xreg[i][k] = r0 + xch[i] + k < Q.R ? xreg[i][k] : 0.f;
#pragma unroll
            for (int k = 0; k < 8; k++) xreg[i][k] = xch[i] >= 0 ? xreg[i][k] : 0.f;
            u32x4 h, m, l;
            split8(xreg[i], h, m, l);
            to[id] = h;
            to[XPART + id] = m;
            to[2 * XPART + id] = l;
        }
    };
    // the pixel this lane multiplies
    const int j = wn * 32 + col, p = m0 + j < Q.M ? p0 + j : p0;
    const int dn = image_of(Q, p), pp = p - dn * Q.P, hh = WIN ? quotient(pp, Q.W, Q.mW) : 0;
    const int lofs = half * XH + (WIN ? (dn * Q.HP + hh - h0) * Q.Wp + (pp - hh * Q.W) : j);

    // this lane's part of the weights of a step: three pieces, the steps in a row
    const int nsteps = (Q.R + 15) / 16 * TVT;
    const char* const wp = reinterpret_cast<const char*>(Q.wsplit) + (int64_t)((g * Q.mtiles + mtile) * WM + wm) * nsteps * 3072;
    u32x4 a[NS][3];
    auto load_w = [&](int step, u32x4 (&to)[3]) {
        const char* const from = wp + min(step, nsteps - 1) * 3072;
#pragma unroll
        for (int k = 0; k < 3; k++) to[k] = *reinterpret_cast<const u32x4*>(from + k * 1024 + (uint32_t)lane * 16u);
    };
#pragma unroll
    for (int d = 0; d < AHEAD; d++) load_w(d, a[d]);
    f16v total, lead, small[2];
#pragma unroll
    for (int r = 0; r < 16; r++) total[r] = small[0][r] = small[1][r] = 0.f;
    load(0);
    store(0, lds_split);
    u32x4* cur = lds_split;
    u32x4* next = lds_split + 3 * XPART;
    int step = 0;
    for (int r0 = 0; r0 < Q.R; r0 += CH) {
        __syncthreads();  // (this chunk is written, and the other buffer has been read)
        if (r0 + CH < Q.R) load(r0 + CH);
#pragma unroll
        for (int r = 0; r < 16; r++) lead[r] = 0.f;
        u32x4 xb[2][3];  // the pixels of this step and of the next
        auto load_x = [&](int s, u32x4 (&to)[3]) {
            const u32x4* const x = cur + lofs + (WIN ? s / 3 * Q.Wp + s % 3 : s * 2 * TP);
#pragma unroll
            for (int k = 0; k < 3; k++) to[k] = x[k * XPART];
        };
        load_x(0, xb[0]);
#pragma unroll
        for (int s = 0; s < NS; s++) {
            if (!WIN && step >= nsteps) break;
            load_w(step + AHEAD, a[(s + AHEAD) % NS]);
            if (s + 1 < NS) load_x(s + 1, xb[(s + 1) & 1]);
            const u32x4 (&w)[3] = a[s];
            const u32x4 (&x)[3] = xb[s & 1];
            // (in this order: a product that continues the chain of the one before it would wait for it)
            const int c = s & 1;
            __builtin_amdgcn_sched_barrier(0);
            small[c] = mfma(w[2], x[0], small[c]);
            __builtin_amdgcn_sched_barrier(kNotMfma);
            small[1 - c] = mfma(w[1], x[0], small[1 - c]);
            __builtin_amdgcn_sched_barrier(kNotMfma);
            lead = mfma(w[0], x[0], lead);
            __builtin_amdgcn_sched_barrier(kNotMfma);
            small[c] = mfma(w[1], x[1], small[c]);
            __builtin_amdgcn_sched_barrier(kNotMfma);
            small[1 - c] = mfma(w[0], x[1], small[1 - c]);
            __builtin_amdgcn_sched_barrier(kNotMfma);
            small[c] = mfma(w[0], x[2], small[c]);
            __builtin_amdgcn_sched_barrier(0);
            step++;
        }
#pragma unroll
        for (int r = 0; r < 16; r++) total[r] += lead[r];
        if (r0 + CH < Q.R) store(r0 + CH, next);
        u32x4* const t = cur;
        cur = next;
        next = t;
    }
    // lane: pixel `col` of the wavefront's 32, outputs r % 4 + 8 * (r / 4) + 4 * half
    const int ob = o0 + 4 * half;
    const bool tr = Q.transposed;
    const float* const wbase = Q.w + (int64_t)g * Q.Og * Q.K;
    const int64_t wch = tr ? (int64_t)Q.Og * TVT : TVT;
    if (m0 + j >= Q.M) return;
    float* const d = Q.dst + ((n0 + dn) * Q.G + g) * Q.Og * P + ob * P + pp;
    float old[16];
    unsigned again = 0;
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int o = r % 4 + 8 * (r / 4);
        total[r] += small[0][r] + small[1][r];
        old[r] = 0.f;
        if (ob + o < Q.Og) {
            if (!(fabsf(total[r]) <= 3.4e38f)) again |= 1u << r;
            if (Q.acc) old[r] = d[o * P];
        }
    }
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int o = r % 4 + 8 * (r / 4);
        if (ob + o < Q.Og && !(again >> r & 1u)) d[o * P] = Q.acc ? old[r] + total[r] : total[r];
    }
    // results that an infinity, a NaN or a value beyond the range of bf16 reached: once more, in fp32
    while (again) {
        const int r = __ffs(again) - 1, o = r % 4 + 8 * (r / 4);
        again &= again - 1u;
        const float* const w = wbase + (tr ? (int64_t)(ob + o) * TVT : (int64_t)(ob + o) * Q.K);
        const float* const xs = src + dn * Q.G * Q.R * P;
        float sum = 0.f;
        for (int c = 0; c < Q.R; c++)
            for (int k = 0; k < TVT; k++) {
                const int y = hh + k / 3 - 1, x = pp - hh * Q.W + k % 3 - 1;
                if (WIN && ((unsigned)y >= (unsigned)Q.H || (unsigned)x >= (unsigned)Q.W)) continue;
                sum = fmaf(w[c * wch + (tr ? TVT - 1 - k : k)], xs[c * P + (WIN ? y * Q.W + x : pp)], sum);
            }
        d[o * P] = Q.acc ? d[o * P] + sum : sum;
    }
}

// The weights of a contraction in the order in which k_fwd_split reads them: [group][32 outputs][step][part][lane], a lane's
// output lane % 32 and its eight channels from 8 * (lane / 32) of the step's sixteen; zero past the last output and channel.
__global__ __launch_bounds__(kThreads) void k_split_weights(SplitJobs jobs) {
    const SplitJob& J = jobs.j[blockIdx.y];
    const int id = blockIdx.x * kThreads + threadIdx.x, lane = id & 63;
    if (id >= J.items) return;
    const int steps = (J.R + 15) / 16 * J.TV;
    int t = id >> 6;
    const int step = t % steps;
    t /= steps;
    const int mt = t % J.mt32, g = t / J.mt32;
    const int tap = step % J.TV, c = step / J.TV * 16 + (lane >> 5) * 8, o = mt * 32 + (lane & 31);
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int cc = min(c + k, J.R - 1), oc = min(o, J.Og - 1);
        v[k] = J.w[J.transposed ? (((int64_t)g * J.R + cc) * J.Og + oc) * J.TV + (J.TV - 1 - tap) : (((int64_t)g * J.Og + oc) * J.R + cc) * J.TV + tap];
        v[k] = o < J.Og && c + k < J.R ? v[k] : 0.f;
    }
    u32x4 h, m, l;
    split8(v, h, m, l);
    u32x4* const out = reinterpret_cast<u32x4*>(J.out) + (int64_t)(id >> 6) * 192 + lane;
    out[0] = h;
    out[64] = m;
    out[128] = l;
}

template <int WM, int TVT, int NPI>
void launch_one(const Params& p, dim3 grid, hipStream_t s) {
    static const hipError_t lds_ok = hipFuncSetAttribute((const void*)k_fwd_split<WM, TVT, NPI>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxSplitLds);
    (void)lds_ok;
    CANVAS_LAUNCH((k_fwd_split<WM, TVT, NPI>), grid, dim3(kThreads), split_lds(p), s, p);
}

}  // namespace

// Items of the operand tile per thread: eight channels of a position each, two per position, without a window eight.
static int split_items(const Params& p) { return p.TV == 1 ? 4 / p.wm : (p.S + 127) / 128; }

size_t split_lds(const Params& p) { return (size_t)16 * 2 * 3 * kThreads * std::max(2, split_items(p)); }

SplitJob split_job(const Params& p) {
    SplitJob j;
    j.G = p.G;
    j.R = p.R;
    j.Og = p.Og;
    j.TV = p.TV;
    j.transposed = p.transposed;
    j.mt32 = p.mtiles * p.wm;
    j.items = p.G * j.mt32 * ((p.R + 15) / 16) * p.TV * 64;
    return j;
}

void split_weights(const SplitJobs& jobs, hipStream_t s) {
    int most = 0;
    for (int k = 0; k < jobs.n; k++) most = std::max(most, jobs.j[k].items);
    CANVAS_LAUNCH(k_split_weights, dim3((unsigned)((most + kThreads - 1) / kThreads), (unsigned)jobs.n), dim3(kThreads), 0, s, jobs);
}

void forward_split(const Params& p, dim3 grid, hipStream_t s) {
    const int items = split_items(p);
    if (p.TV == 1) {
        launch_one<2, 1, 2>(p, grid, s);
    } else if (p.wm == 2) {
        if (items <= 2) launch_one<2, 9, 2>(p, grid, s);
        else if (items == 3) launch_one<2, 9, 3>(p, grid, s);
        else launch_one<2, 9, 4>(p, grid, s);
    } else {
        if (items <= 2) launch_one<1, 9, 2>(p, grid, s);
        else if (items == 3) launch_one<1, 9, 3>(p, grid, s);
        else launch_one<1, 9, 4>(p, grid, s);
    }
}

}  // namespace sfc
}  // namespace canvas
