// The fp32 contraction on the bf16 matrix instructions, without loss: every operand is cut into three bf16 parts that hold all
// of its 24 bits, x = h + m + l, and a product is the six parts' products down to 2^-24 of it,
//     x * w = hh' + (hm' + mh' + mm' + hl' + lh') + [ml' + lm' + ll' < 2^-24, dropped],
// each exact in the matrix unit.  v_mfma_f32_32x32x16_bf16 does 16 times the work of the fp32 instruction, six of them 2.7
// times.  The operands are cut times 2^24, the sums taken times 2^-48: the smallest fp32 subnormal's last bit then is 2^-125, a
// normal bf16 value, so that no part of any operand is lost.  (As they are, operands below 2^-110 lose their third part and then
// their second: 3e-5 of the result at 1e-36.)  What lies above, operands of 2^104 and results of 2^80 and more, becomes an
// infinity, and such results are computed again in fp32.
#include <algorithm>
#include <type_traits>

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

// The fp32 instruction with the same tile, for what the parts cannot hold: 32 x 32 results, two of the contraction's elements (lane / 32)
__device__ __forceinline__ f16v mfma_f32(float a, float b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;

// Eight floats (times kUp) -> their three bf16 parts.  A value that is infinite, NaN or rounds to an infinity makes the second part NaN:
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
            for (int k = 0; k < 8; k++) xreg[i][k] = xch[i] >= 0 ? xreg[i][k] * kUp : 0.f;
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
    const bool live = m0 + j < Q.M;
    unsigned again = 0;
#pragma unroll
    for (int r = 0; r < 16; r++) {
        total[r] = (total[r] + (small[0][r] + small[1][r])) * kDown;
        if (live && ob + r % 4 + 8 * (r / 4) < Q.Og && !(fabsf(total[r]) <= 3.4e38f)) again |= 1u << r;
    }
    // Results that an infinity, a NaN or a value beyond the scaled parts' range reached: once more, in fp32.  All of the wavefront's tile
    // on the fp32 units, whatever the values are: operands straight from memory, the margin's zeros among them.  (Forward + data
    // gradient at the size above 42 us, 166 where all of x, w and dy is NaN.)
    if (__builtin_expect(__ballot(again != 0) != 0, 0)) {
        f16v exact;
#pragma unroll
        for (int r = 0; r < 16; r++) exact[r] = 0.f;
        const bool tr = Q.transposed;
        const int o = min(o0 + col, Q.Og - 1);
        const float* const wo = Q.w + (int64_t)g * Q.Og * Q.K + (tr ? (int64_t)o * TVT : (int64_t)o * Q.K);
        const int64_t wch = tr ? (int64_t)Q.Og * TVT : TVT;
        const float* const xs = src + (int64_t)dn * Q.G * Q.R * P;
        const int ww = pp - hh * Q.W;
        int from[TVT];  // of the taps in a channel's plane, -1: in the margin
#pragma unroll
        for (int k = 0; k < TVT; k++) {
            const int y = hh + k / 3 - 1, x = ww + k % 3 - 1;
            from[k] = !WIN ? pp : ((unsigned)y < (unsigned)Q.H && (unsigned)x < (unsigned)Q.W ? y * Q.W + x : -1);
        }
        constexpr int PAIRS = WIN ? 1 : 8;  // of channels whose loads are in flight together
        for (int c0 = 0; c0 < Q.R; c0 += 2 * PAIRS) {
            float wk[PAIRS][TVT], xk[PAIRS][TVT];
#pragma unroll
            for (int u = 0; u < PAIRS; u++) {
                const int c = c0 + 2 * u + half, cc = min(c, Q.R - 1);
#pragma unroll
                for (int k = 0; k < TVT; k++) {
                    wk[u][k] = wo[cc * wch + (tr ? TVT - 1 - k : k)];
                    xk[u][k] = xs[cc * P + max(from[k], 0)];
                    if (c >= Q.R) wk[u][k] = 0.f;
                    if (c >= Q.R || from[k] < 0) xk[u][k] = 0.f;
                }
            }
            f16v part;  // (short chains, added in fp32: the matrix unit cuts off what its sums cannot hold)
#pragma unroll
            for (int r = 0; r < 16; r++) part[r] = 0.f;
#pragma unroll
            for (int u = 0; u < PAIRS; u++)
#pragma unroll
                for (int k = 0; k < TVT; k++) part = mfma_f32(wk[u][k], xk[u][k], part);
#pragma unroll
            for (int r = 0; r < 16; r++) exact[r] += part[r];
        }
#pragma unroll
        for (int r = 0; r < 16; r++) total[r] = again >> r & 1u ? exact[r] : total[r];
    }
    if (!live) return;
    float* const d = Q.dst + ((n0 + dn) * Q.G + g) * Q.Og * P + ob * P + pp;
    float old[16];
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int o = r % 4 + 8 * (r / 4);
        old[r] = Q.acc && ob + o < Q.Og ? d[o * P] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int o = r % 4 + 8 * (r / 4);
        if (ob + o < Q.Og) d[o * P] = Q.acc ? old[r] + total[r] : total[r];
    }
}

constexpr int kXRow = 36;  // dwords of a channel's row of the operand tile: 34 pairs of positions, 16-byte pieces in different banks

// Weight gradient behind a 3 x 3 window, with the same parts and products.  A workgroup owns 32*WM outputs x 32 channels x the
// three taps of one window row and one slice of the batch's positions; a wavefront 32 outputs x 32 channels x three taps of
// every (4/WM)th part of a step, the depth of a matrix instruction being sixteen positions.  Positions are those of the image
// with one zero column behind each row and one zero row behind each image, so that a tap is a constant distance and needs no
// mask: dy is zero in the margin, x too.  64 positions of dy and 68 of x, from two before the window row's first, go cut into
// LDS, [part][row][position], where a lane finds eight positions of its output or channel in one 16-byte read; the taps to the
// left and right are the same dwords moved by one position.
// Sums: per step the five small products first, then the leading ones, in one chain; the steps in a row in fp32, the
// wavefronts' sums at the end.  The matrix unit cuts off what its sums cannot hold, always downwards: over the thousands of steps
// of a batch that adds up (3.6e-7 of the result at 32 channels, 32x28x28), so every other step multiplies -dy.  Where a result is not finite, its workgroup sums its slice again on the fp32 units (28 us at the
// size below, 100 where everything is NaN).
// Bound by the vector instructions that cut and stage the operands, about 510 per wavefront and step (half of a wavefront's life at
// two per SIMD; its 36 matrix instructions a quarter).  N=32, C=64, 28x28: 28 us (66 TFLOP/s), k_wgrad 46.5; 128 channels 32x14x14
// 30.5 / 45.4, 384 in eight groups 51 / 73.  Errors against fp64: 1.04e-7 and 9.1e-8, k_wgrad's 1.15 and 1.02e-7.
template <int WM>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad_split(Params Q) {
    constexpr int WS = 4 / WM, NS = 4 / WS;               // wavefronts that share a tile's steps, matrix steps of each
    constexpr int AR = 32 * WM;                           // rows of dy
    constexpr int APART = AR * 32, XPART = 32 * kXRow;    // dwords of a part
    constexpr int BUF = 3 * (APART + XPART);
    extern __shared__ u32x4 lds_split[];  // [2][BUF] dwords
    __shared__ int redo;
    uint32_t* const lds = reinterpret_cast<uint32_t*>(lds_split);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int wm = wave % WM, ws = wave / WM;
    unsigned b = tile_of_block();
    if (b >= (unsigned)Q.tiles) return;
    const int kh = (int)(b % 3u);  // (neighbours in the launch: they read the same rows, and write the same lines)
    b /= 3u;
    const int mtile = (int)(b % (unsigned)Q.mtiles);
    b /= (unsigned)Q.mtiles;
    const int ctile = (int)(b % (unsigned)Q.ktiles);
    b /= (unsigned)Q.ktiles;
    const int g = (int)(b % (unsigned)Q.G);
    const int slice = (int)(b / (unsigned)Q.G);
    const int o0 = mtile * AR, r0 = ctile * 32;
    const int rows = min(AR, Q.Og - o0), chans = min(32, Q.R - r0);
    const int HPW = Q.HP * Q.Wp;
    const int64_t end = Q.N * HPW;
    const int64_t first = slice * Q.per_slice, last = min(end, first + Q.per_slice);

    const float* const ds = Q.dy + ((int64_t)g * Q.Og + o0) * Q.P;
    const float* const xs = Q.src + ((int64_t)g * Q.R + r0) * Q.P;
    // Two neighbouring positions: image and place in it of the first; what they hold comes from an element offset or is zero.
    struct Pair {
        int n, rem;
    };
    auto place = [&](int64_t q) {
        Pair at;
        if (q < 0) {  // (before the first image)
            at.n = -1;
            at.rem = (int)q + HPW;  // (a row and two positions at most, and an image has two rows of two)
        } else {
            at.n = (int)(q / HPW);
            at.rem = (int)(q - (int64_t)at.n * HPW);
        }
        return at;
    };
    auto advance = [&](Pair& at) {
        at.rem += 64;
        while (at.rem >= HPW) {
            at.rem -= HPW;
            at.n++;
        }
    };
    auto offsets = [&](const Pair& at, int rowlen, uint32_t (&off)[2], bool (&in)[2]) {
        int n = at.n, h = quotient(at.rem, Q.Wp, Q.mWp), w = at.rem - h * Q.Wp;
#pragma unroll
        for (int e = 0; e < 2; e++) {
            in[e] = (unsigned)n < (unsigned)Q.N && h < Q.H && w < Q.W;
            off[e] = in[e] ? (uint32_t)(n * rowlen + h * Q.W + w) : 0u;
            if (++w == Q.Wp) {
                w = 0;
                if (++h == Q.HP) {
                    h = 0;
                    n++;
                }
            }
        }
    };
    const int pair = tid & 31, rr = tid >> 5;  // this thread's positions of the step and its first row (of every eighth)
    const int64_t xfirst = first + (int64_t)(kh - 1) * Q.Wp - 2;
    Pair da = place(first + 2 * pair), xa = place(xfirst + 2 * pair), xe = place(xfirst + 64 + 2 * (tid & 1));
    const int dlen = Q.G * Q.Og * Q.P, xlen = Q.G * Q.R * Q.P;
    constexpr int DN = AR / 8;
    float dreg[DN][2], xreg[4][2], ereg[2];
    bool din[2], xin[2], ein[2];
    // `n` pairs of every eighth row from this thread's first on; byte offsets from uniform addresses where the tile is whole
    auto at = [](const float* base, uint32_t elem) { return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + elem * 4u); };
    auto load_rows = [&](const float* from, const uint32_t (&off)[2], int have, auto& to, auto count) {
        constexpr int n = decltype(count)::value;
        if (have == n * 8) {
            const uint32_t ro = (uint32_t)(rr * Q.P);
#pragma unroll
            for (int i = 0; i < n; i++)
#pragma unroll
                for (int e = 0; e < 2; e++) to[i][e] = at(from + (int64_t)i * 8 * Q.P, off[e] + ro);
        } else {
#pragma unroll
            for (int i = 0; i < n; i++)
#pragma unroll
                for (int e = 0; e < 2; e++) to[i][e] = at(from, off[e] + (uint32_t)(min(i * 8 + rr, have - 1) * Q.P));
        }
    };
    auto load = [&]() {
        uint32_t off[2];
        offsets(da, dlen, off, din);
        load_rows(ds, off, rows, dreg, std::integral_constant<int, DN>());
        advance(da);
        offsets(xa, xlen, off, xin);
        load_rows(xs, off, chans, xreg, std::integral_constant<int, 4>());
        advance(xa);
        if (wave == 0) {  // the last two pairs of the 32 rows
            offsets(xe, xlen, off, ein);
#pragma unroll
            for (int e = 0; e < 2; e++) ereg[e] = at(xs, off[e] + (uint32_t)(min(tid >> 1, chans - 1) * Q.P));
            advance(xe);
        }
    };
    auto put = [&](uint32_t* to, int part, const float (&v)[2]) {
        const uint32_t h = tile::pack_bf16(v[0], v[1]);
        const float m0 = v[0] - tile::lo_f32(h), m1 = v[1] - tile::hi_f32(h);
        const uint32_t m = tile::pack_bf16(m0, m1);
        to[0] = h;
        to[part] = m;
        to[2 * part] = tile::pack_bf16(m0 - tile::lo_f32(m), m1 - tile::hi_f32(m));
    };
    auto store = [&](uint32_t* to, float dy_factor) {  // (zero in the margin and past the last row)
#pragma unroll
        for (int i = 0; i < DN; i++) {  // (the 16-byte pieces of a row change places with its number: reads of 32 rows in different banks)
            const int row = i * 8 + rr;
            float v[2];
#pragma unroll
            for (int e = 0; e < 2; e++) v[e] = din[e] && row < rows ? dreg[i][e] * dy_factor : 0.f;
            put(to + row * 32 + (((pair >> 2) ^ (row & 7)) << 2) + (pair & 3), APART, v);
        }
        uint32_t* const x = to + 3 * APART;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int row = i * 8 + rr;
            float v[2];
#pragma unroll
            for (int e = 0; e < 2; e++) v[e] = xin[e] && row < chans ? xreg[i][e] * kUp : 0.f;
            put(x + row * kXRow + pair, XPART, v);
        }
        if (wave == 0) {
            float v[2];
#pragma unroll
            for (int e = 0; e < 2; e++) v[e] = ein[e] && (tid >> 1) < chans ? ereg[e] * kUp : 0.f;
            put(x + (tid >> 1) * kXRow + 32 + (tid & 1), XPART, v);
        }
    };
    f16v total[3];
#pragma unroll
    for (int t = 0; t < 3; t++)
#pragma unroll
        for (int r = 0; r < 16; r++) total[t][r] = 0.f;
    uint32_t *cur = lds, *next = lds + BUF;
    // (sign of dy in the step that begins at q)
    auto sign_of = [](int64_t q) { return (q >> 6) & 1 ? -1.f : 1.f; };
    if (tid == 0) redo = 0;  // (read after the barriers of the steps)
    load();
    store(cur, sign_of(first) * kUp);
    for (int64_t q = first; q < last; q += 64) {
        __syncthreads();  // (this step is written, and the other buffer has been read)
        const bool more = q + 64 < last;
        if (more) load();
        f16v sum[3];
#pragma unroll
        for (int t = 0; t < 3; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) sum[t][r] = 0.f;
        u32x4 lead_a[NS], lead_b[NS][3];
#pragma unroll
        for (int s = 0; s < NS; s++) {
            const int piece = (ws * NS + s) * 2 + half;  // this lane's eight positions
            const int arow = wm * 32 + col;
            u32x4 a[3], x[3][3];
#pragma unroll
            for (int k = 0; k < 3; k++) {
                a[k] = *reinterpret_cast<const u32x4*>(cur + k * APART + arow * 32 + ((piece ^ (arow & 7)) << 2));
                const uint32_t* const from = cur + 3 * APART + k * XPART + col * kXRow + piece * 4;
                const u32x4 lo = *reinterpret_cast<const u32x4*>(from);
                const uint2 hi = *reinterpret_cast<const uint2*>(from + 4);
                const uint32_t d[6] = {lo[0], lo[1], lo[2], lo[3], hi.x, hi.y};
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    x[0][k][v] = __builtin_amdgcn_alignbit(d[v + 1], d[v], 16);
                    x[1][k][v] = d[v + 1];
                    x[2][k][v] = __builtin_amdgcn_alignbit(d[v + 2], d[v + 1], 16);
                }
            }
#pragma unroll
            for (int t = 0; t < 3; t++) sum[t] = mfma(a[2], x[t][0], sum[t]);
#pragma unroll
            for (int t = 0; t < 3; t++) sum[t] = mfma(a[0], x[t][2], sum[t]);
#pragma unroll
            for (int t = 0; t < 3; t++) sum[t] = mfma(a[1], x[t][1], sum[t]);
#pragma unroll
            for (int t = 0; t < 3; t++) sum[t] = mfma(a[1], x[t][0], sum[t]);
#pragma unroll
            for (int t = 0; t < 3; t++) sum[t] = mfma(a[0], x[t][1], sum[t]);
            lead_a[s] = a[0];
#pragma unroll
            for (int t = 0; t < 3; t++) lead_b[s][t] = x[t][0];
        }
#pragma unroll
        for (int s = 0; s < NS; s++)
#pragma unroll
            for (int t = 0; t < 3; t++) sum[t] = mfma(lead_a[s], lead_b[s][t], sum[t]);
#pragma unroll
        for (int t = 0; t < 3; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) total[t][r] = fmaf(sum[t][r], sign_of(q), total[t][r]);
        if (more) store(next, sign_of(q + 64) * kUp);
        uint32_t* const t = cur;
        cur = next;
        next = t;
    }
    // the sums of the wavefronts that shared the tile
    float* const share = reinterpret_cast<float*>(lds_split);  // [WS - 1][WM][3 * 16][64]
    auto sum_up = [&](f16v (&part)[3]) {
        __syncthreads();
        if (ws > 0) {
#pragma unroll
            for (int t = 0; t < 3; t++)
#pragma unroll
                for (int r = 0; r < 16; r++) share[(((ws - 1) * WM + wm) * 48 + t * 16 + r) * 64 + lane] = part[t][r];
        }
        __syncthreads();
        if (ws > 0) return;
#pragma unroll
        for (int k = 0; k < WS - 1; k++)
#pragma unroll
            for (int t = 0; t < 3; t++)
#pragma unroll
                for (int r = 0; r < 16; r++) part[t][r] += share[((k * WM + wm) * 48 + t * 16 + r) * 64 + lane];
    };
    sum_up(total);
    // lane: channel `col`, outputs r % 4 + 8 * (r / 4) + 4 * half
    const int ob = wm * 32 + 4 * half;
    float* const dw = Q.partial + (((int64_t)slice * Q.G + g) * Q.Og + o0) * Q.K + (int64_t)(r0 + col) * 9 + kh * 3;
    uint64_t again = 0;
    if (ws == 0 && col < chans) {
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int o = ob + r % 4 + 8 * (r / 4);
            if (o >= rows) continue;
#pragma unroll
            for (int t = 0; t < 3; t++) {
                total[t][r] *= kDown;
                dw[(int64_t)o * Q.K + t] = total[t][r];
                if (!(fabsf(total[t][r]) <= 3.4e38f)) again |= (uint64_t)1 << (r * 3 + t);
            }
        }
    }
    if (__ballot(again != 0) != 0 && lane == 0) redo = 1;
    __syncthreads();
    // Once more in fp32, as in k_fwd_split; the wavefronts take eight positions in turn.
    if (!redo) return;
    f16v exact[3];
#pragma unroll
    for (int t = 0; t < 3; t++)
#pragma unroll
        for (int r = 0; r < 16; r++) exact[t][r] = 0.f;
    const float* const dr = ds + (int64_t)min(wm * 32 + col, rows - 1) * Q.P;
    const float* const xr = xs + (int64_t)min(col, chans - 1) * Q.P;
    constexpr int STEP = 8;
    Pair pos = place(first + ws * STEP + half);
    for (int64_t q = first + ws * STEP; q < last; q += WS * STEP) {
        float a[STEP / 2], x[STEP / 2][3];
#pragma unroll
        for (int u = 0; u < STEP / 2; u++) {
            while (pos.rem >= HPW) {
                pos.rem -= HPW;
                pos.n++;
            }
            const int h = quotient(pos.rem, Q.Wp, Q.mWp), w = pos.rem - h * Q.Wp, y = h + kh - 1;
            const bool in = q + 2 * u + half < last && pos.n < Q.N && h < Q.H && w < Q.W;  // (else there is no such pixel of dy)
            a[u] = dr[in ? (int64_t)pos.n * dlen + h * Q.W + w : 0];
            if (!in) a[u] = 0.f;
#pragma unroll
            for (int t = 0; t < 3; t++) {
                const bool xin = in && (unsigned)y < (unsigned)Q.H && (unsigned)(w + t - 1) < (unsigned)Q.W;
                x[u][t] = xr[xin ? (int64_t)pos.n * xlen + y * Q.W + w + t - 1 : 0];
                if (!xin) x[u][t] = 0.f;
            }
            pos.rem += 2;
        }
        f16v part[3];
#pragma unroll
        for (int t = 0; t < 3; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) part[t][r] = 0.f;
#pragma unroll
        for (int u = 0; u < STEP / 2; u++)
#pragma unroll
            for (int t = 0; t < 3; t++) part[t] = mfma_f32(a[u], x[u][t], part[t]);
#pragma unroll
        for (int t = 0; t < 3; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) exact[t][r] += part[t][r];
        pos.rem += (WS - 1) * STEP;
    }
    sum_up(exact);
#pragma unroll
    for (int r = 0; r < 16; r++)
#pragma unroll
        for (int t = 0; t < 3; t++)
            if (again >> (r * 3 + t) & 1u) dw[(int64_t)(ob + r % 4 + 8 * (r / 4)) * Q.K + t] = exact[t][r];
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
        v[k] = o < J.Og && c + k < J.R ? v[k] * kUp : 0.f;
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
    static std::atomic<uint64_t> asked;
    allow_lds(asked, (const void*)k_fwd_split<WM, TVT, NPI>, kMaxSplitLds);
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

static size_t wgrad_split_lds(const Params& p) { return (size_t)4 * 2 * 3 * (32 * p.wm * 32 + 32 * kXRow); }

void wgrad_split(const Params& p, dim3 grid, hipStream_t s) {
    const dim3 block(kThreads);
    const size_t lds = wgrad_split_lds(p);
    if (p.wm == 2) {
        static std::atomic<uint64_t> asked;
        allow_lds(asked, (const void*)k_wgrad_split<2>, kMaxSplitLds);
        CANVAS_LAUNCH((k_wgrad_split<2>), grid, block, lds, s, p);
    } else {
        CANVAS_LAUNCH((k_wgrad_split<1>), grid, block, lds, s, p);
    }
}

}  // namespace sfc
}  // namespace canvas
