// Weight gradient of a grouped FC behind a 3x3 window on bf16 MFMA (Canvas paper, Section 5: Fully-connected, Group, Unfold), by image rows
// staged through LDS.
//
// dW[o][k][tap] = sum over the pixels of dy[o] and of src[k] displaced by the tap: the contraction runs over the pixels, which both tensors
// keep contiguous, so an MFMA operand is eight consecutive pixels of a channel, and what has to be made is the displacement.  A step
// brings some rows of both tensors to LDS, each image row padded with zeros to whole units of eight pixels, and src three times: displaced
// by one pixel to either side, and not at all.  A tap is then a copy and a distance in units: every operand is one aligned 16-byte
// read, and there are no masks behind the staging.  (The tap-major kernel gives every wavefront 16 x 32 pixels of its own and makes each tap from
// registers, with masks, byte shifts and lane exchanges, and reads src once per window row.)
// At 128x256x14x14 a launch is 10 us of one workgroup per compute unit: four steps of about 1.5 us (LDS, 40 % of the cycles; vector instructions
// 15 %, MFMA 15 %), the first loads and the partial.  The loads of two steps are in flight, and two steps are in LDS: one barrier per step.
#include "gfc_wgrad_kernels.hpp"

#include <algorithm>

#include "launch.hpp"
#include "magic.hpp"
#include "tile_util.hpp"

namespace canvas {
namespace gfcwg {

namespace {

using namespace canvas::tile;

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int MT = 2;                   // a workgroup's tile: 16 MT outputs x 16 MT rows x 9 taps
constexpr int KS = kWaves / (2 * MT);   // wavefronts that share a tile and split its contraction steps

constexpr int items_for(int U) { return 2 / U; }  // image rows of either tensor per thread and step

extern __shared__ __align__(16) unsigned char lds[];

template <int U>
__global__ __launch_bounds__(kThreads, 2) void k_wgrad_taps(Params P) {
    constexpr int NI = items_for(U), D = 4 * U;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane >> 4, s = lane & 15;
    const int nk = wave % MT, th = wave / MT & 1, kq = wave / (2 * MT);  // row tile; taps 0-4 or 5-8; share of the contraction steps
    const int ot = P.Omp / (16 * MT), kt = P.Rp / (16 * MT), tiles = P.Gm * ot * kt;
    const int seq = (int)xcd_sequence();
    const int slice = (int)div_magic((uint32_t)seq, P.magicTiles), t2 = seq - slice * tiles;
    const int gmi = (int)div_magic((uint32_t)t2, P.magicGroup), t3 = t2 - gmi * (ot * kt);
    const int oi = (int)div_magic((uint32_t)t3, P.magicKt), o0 = oi * 16 * MT, k0 = (t3 - oi * kt) * 16 * MT;
    const int gcount = min(P.gm, P.G - gmi * P.gm);
    const int Rm = gcount * P.R, Om = gcount * P.Og;
    const int src_img = P.G * P.R * P.P, dy_img = P.G * P.Og * P.P;
    const rsrc_t rs = make_rsrc(P.src, P.N * src_img * 2), rdy = make_rsrc(P.dy, P.N * dy_img * 2);
    const int begin = slice * P.per_slice, end = min(P.steps, begin + P.per_slice);
    const int copy = 16 * MT * P.xu * 16;  // bytes of a copy of src

    // this thread's image rows: first element in image 0 (of a tile from row 0), image, row, place in LDS
    int xe[NI], xj[NI], xh[NI], xat[NI], de[NI], dj[NI], dh[NI], dat[NI];
#pragma unroll
    for (int i = 0; i < NI; i++) {
        const int it = tid + i * kThreads;
        int c = (int)div_magic((uint32_t)it, P.magicRx), y = it - c * P.rx;
        xj[i] = P.J > 1 ? (int)div_magic((uint32_t)y, P.magicH) : 0;
        xh[i] = P.J > 1 ? y - xj[i] * P.H : y - 1;
        xat[i] = c < 16 * MT ? (c * P.xu + (P.J > 1 ? xj[i] * (P.H + 1) + 1 + xh[i] : y) * U) * 16 : -1;
        if (c >= 16 * MT || k0 + c >= Rm) xj[i] = P.N;
        xe[i] = (gmi * P.gm * P.R + k0 + c) * P.P + xj[i] * src_img + xh[i] * P.W;
        c = (int)div_magic((uint32_t)it, P.magicRd);
        y = it - c * P.rd;
        dj[i] = P.J > 1 ? (int)div_magic((uint32_t)y, P.magicH) : 0;
        dh[i] = P.J > 1 ? y - dj[i] * P.H : y;
        dat[i] = c < 16 * MT ? 3 * copy + (c * P.du + (P.J > 1 ? dj[i] * (P.H + 1) + dh[i] : y) * U) * 16 : -1;
        if (c >= 16 * MT || o0 + c >= Om) dj[i] = P.N;
        de[i] = (gmi * P.gm * P.Og + o0 + c) * P.P + dj[i] * dy_img + dh[i] * P.W;
    }

    // The last unit of a row is loaded so that it ends with the row and moved down when it is used: past the tensor's end there is
    // nothing to read.  Rows of less than a unit begin before themselves then, except the tensor's first.
    const int over = 8 * U - P.W;  // pixels of the last unit that do not exist
    struct Rows {
        u32x4 x[NI][U], d[NI][U];
        int xm[NI], dm[NI];  // by how many pixels the last unit moves
    };
    auto issue = [&](int step, Rows& v) {
        const int g = P.J > 1 ? step : (int)div_magic((uint32_t)step, P.magicRowTiles);
        const int n0 = g * P.J, h0 = P.J > 1 ? 0 : (step - g * P.row_tiles) * P.TH;
        const bool live = step < end;
#pragma unroll
        for (int i = 0; i < NI; i++) {
            const bool okx = live & (n0 + xj[i] < P.N) & ((unsigned)(h0 + xh[i]) < (unsigned)P.H);
            const int ex = n0 * src_img + h0 * P.W + xe[i];
            v.xm[i] = U == 1 && ex < over ? 0 : over;
            const bool okd = live & (n0 + dj[i] < P.N) & (h0 + dh[i] < P.H);
            const int ed = n0 * dy_img + h0 * P.W + de[i];
            v.dm[i] = U == 1 && ed < over ? 0 : over;
            int ax[U], ad[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                ax[u] = okx ? (ex + 8 * u - (u == U - 1 ? v.xm[i] : 0)) * 2 : kOob;
                ad[u] = okd ? (ed + 8 * u - (u == U - 1 ? v.dm[i] : 0)) * 2 : kOob;
                asm volatile("" : "+v"(ax[u]), "+v"(ad[u]));  // (selects, not loads under a branch)
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                v.x[i][u] = bload16(rs, ax[u]);
                v.d[i][u] = bload16(rdy, ad[u]);
            }
        }
    };
    u32x4 keep;  // the pixels of a row's last unit that exist
#pragma unroll
    for (int k = 0; k < 4; k++) keep[k] = (2 * k < 8 - over ? 0xffffu : 0u) | (2 * k + 1 < 8 - over ? 0xffff0000u : 0u);
    auto write = [&](Rows& v, int buf) {
#pragma unroll
        for (int i = 0; i < NI; i++) {
            if (over) {
                v.x[i][U - 1] = drop_first(v.x[i][U - 1], v.xm[i]) & keep;
                v.d[i][U - 1] = drop_first(v.d[i][U - 1], v.dm[i]) & keep;
            }
            if (xat[i] >= 0) {
                uint32_t d[D + 2];  // [zeros | the row | zeros]
                d[0] = d[D + 1] = 0;
#pragma unroll
                for (int k = 0; k < D; k++) d[k + 1] = v.x[i][k / 4][k % 4];
#pragma unroll
                for (int u = 0; u < U; u++) {
                    u32x4 left, right;  // pixel p of the copies is pixel p - 1 or p + 1 of the row
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        left[k] = __builtin_amdgcn_alignbit(d[4 * u + k + 1], d[4 * u + k], 16);
                        right[k] = __builtin_amdgcn_alignbit(d[4 * u + k + 2], d[4 * u + k + 1], 16);
                    }
                    if (u == U - 1) left = left & keep;
                    unsigned char* to = lds + buf + xat[i] + u * 16;
                    *reinterpret_cast<u32x4*>(to) = left;
                    *reinterpret_cast<u32x4*>(to + copy) = v.x[i][u];
                    *reinterpret_cast<u32x4*>(to + 2 * copy) = right;
                }
            }
            if (dat[i] >= 0) {
#pragma unroll
                for (int u = 0; u < U; u++) *reinterpret_cast<u32x4*>(lds + buf + dat[i] + u * 16) = v.d[i][u];
            }
        }
    };

    float4_t acc[MT][5];
#pragma unroll
    for (int mo = 0; mo < MT; mo++)
#pragma unroll
        for (int i = 0; i < 5; i++) acc[mo][i] = float4_t{0.f, 0.f, 0.f, 0.f};
    int tap[5];  // offsets of this wavefront's taps (taps 0-4, or 5-8 and none)
#pragma unroll
    for (int i = 0; i < 5; i++) {
        const int t = min(th * 5 + i, 8);
        tap[i] = t % 3 * copy + t / 3 * U * 16;
    }
    const unsigned char* const a0 = lds + 3 * copy + (s * P.du + r) * 16;
    const unsigned char* const b0 = lds + ((nk * 16 + s) * P.xu + r) * 16;
    auto contract = [&](int buf) {
#pragma unroll 2
        for (int ks = kq; ks < P.ksteps; ks += KS) {
            u32x4 a[MT], b[5];
#pragma unroll
            for (int mo = 0; mo < MT; mo++) a[mo] = *reinterpret_cast<const u32x4*>(a0 + buf + mo * 16 * P.du * 16 + ks * 64);
#pragma unroll
            for (int i = 0; i < 5; i++) b[i] = *reinterpret_cast<const u32x4*>(b0 + buf + tap[i] + ks * 64);
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int mo = 0; mo < MT; mo++) acc[mo][i] = mfma32(a[mo], b[i], acc[mo][i]);
            if (th == 0) {
#pragma unroll
                for (int mo = 0; mo < MT; mo++) acc[mo][4] = mfma32(a[mo], b[4], acc[mo][4]);
            }
        }
    };

    Rows v[2];
    issue(begin, v[0]);
    issue(begin + 1, v[1]);
    // (what lies between and behind the rows stays zero)
    for (int o = tid * 16; o < 2 * P.lds_bytes; o += kThreads * 16) *reinterpret_cast<u32x4*>(lds + o) = u32x4{0, 0, 0, 0};
    lds_barrier();
    for (int c = begin; c < end; c += 2) {
#pragma unroll
        for (int f = 0; f < 2; f++) {
            const int buf = f * P.lds_bytes;
            write(v[f], buf);
            issue(c + f + 2, v[f]);
            lds_barrier();  // (the buffer written next is the one that all wavefronts have read before this)
            if (c + f < end) contract(buf);
        }
    }

    // sum of the KS shares in order, then the partial
    lds_barrier();
    float* const red = reinterpret_cast<float*>(lds) + ((wave % (2 * MT)) * MT * 20 * 64 + lane);
    if (kq > 0) {
#pragma unroll
        for (int mo = 0; mo < MT; mo++)
#pragma unroll
            for (int i = 0; i < 5; i++)
#pragma unroll
                for (int j = 0; j < 4; j++) red[(kq - 1) * 2 * MT * MT * 20 * 64 + ((mo * 5 + i) * 4 + j) * 64] = acc[mo][i][j];
    }
    lds_barrier();
    if (kq > 0) return;
    float* part = P.partial + (long long)slice * P.Gm * P.Omp * 9 * P.Rp;
#pragma unroll
    for (int mo = 0; mo < MT; mo++)
#pragma unroll
        for (int i = 0; i < 5; i++) {
            const int t = th * 5 + i;
            if (t >= 9) continue;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                float x = acc[mo][i][j];
#pragma unroll
                for (int q = 1; q < KS; q++) x += red[(q - 1) * 2 * MT * MT * 20 * 64 + ((mo * 5 + i) * 4 + j) * 64];
                const int o = o0 + mo * 16 + 4 * r + j;
                part[((long long)(gmi * P.Omp + o) * 9 + t) * P.Rp + k0 + nk * 16 + s] = x;
            }
        }
}

constexpr int kMaxLds = 78 * 1024;  // of a step: two of them in flight, of the 160 KB of a compute unit

template <int U>
void launch(const Params& P, hipStream_t s) {
    static std::atomic<uint64_t> asked;
    allow_lds(asked, (const void*)k_wgrad_taps<U>, 2 * kMaxLds);
    const dim3 grid((unsigned)(P.slices * P.Gm * (P.Omp / (16 * MT)) * (P.Rp / (16 * MT))));
    CANVAS_LAUNCH((k_wgrad_taps<U>), grid, dim3(kThreads), (size_t)P.lds_bytes * 2, s, P);
}

}  // namespace

// Which weight gradients.  Against the tap-major kernels (8 groups), us there / here: 128x256x14x14 18.9 / 13.2, 128x512x7x7 21.9 / 16.4,
// 32x512x14x14 16.1 / 13.2, 64x512x8x8 14.1 / 11.2, 100x256x7x9 13.4 / 11.5, 30x192x16x16 10.1 / 8.8.  They stay for rows of three units and more
// (64x256x28x28 22.0 / 25.2, 32x256x20x20 11.4 / 11.3), for tiles of 16 x 16 (128x128x28x28 18.2 / 21.2, 64x128x7x7 6.6 / 8.3), where much of
// the rows is padding (128x512x5x6 12.3 / 14.4) and for a few steps (8x512x7x7 8.1 / 9.4, 4x256x14x14 7.3 / 7.2).
bool plan(Params& P, const gfctm::Params& T) {
    if (T.KH != 3 || T.KW != 3 || T.W > 16 || T.Rp % (16 * MT) || T.Omp % (16 * MT)) return false;
    P.N = T.N;
    P.H = T.H;
    P.W = T.W;
    P.P = T.P;
    P.G = T.G;
    P.R = T.R;
    P.Og = T.Og;
    P.gm = T.gm;
    P.Gm = T.Gm;
    P.Rp = T.Rp;
    P.Omp = T.Omp;
    P.U = (P.W + 7) / 8;
    const int ch = 16 * MT, most_rows = kThreads * items_for(P.U) / ch;  // image rows per channel that the threads can load
    auto size = [&](int rows_x, int rows_d) {
        P.ksteps = (rows_d * P.U + 3) / 4;
        P.xu = (std::max(rows_x * P.U, 4 * P.ksteps + 2 * P.U)) | 1;
        P.du = (4 * P.ksteps) | 1;
        const int sum = (KS - 1) * 2 * MT * MT * 20 * 64 * 4;
        P.lds_bytes = std::max((3 * P.xu + P.du) * ch * 16, sum);
        return P.lds_bytes <= kMaxLds;
    };
    bool ok = false;
    for (int J = std::min(P.N, most_rows / P.H); J >= 2 && !ok; J--) {
        P.J = J;
        P.TH = P.H;
        P.rx = P.rd = J * P.H;
        ok = size(J * (P.H + 1) + 1, J * (P.H + 1) - 1);
    }
    for (int t = 1; t <= P.H && !ok; t++) {
        P.J = 1;
        P.TH = (P.H + t - 1) / t;
        P.rx = P.TH + 2;
        P.rd = P.TH;
        ok = P.rx <= most_rows && size(P.rx, P.rd);
    }
    if (!ok) return false;
    P.row_tiles = (P.H + P.TH - 1) / P.TH;
    const int64_t steps = P.J > 1 ? (P.N + P.J - 1) / P.J : (int64_t)P.N * P.row_tiles;
    const int64_t tiles = (int64_t)P.Gm * (P.Omp / ch) * (P.Rp / ch), packed = gfctm::packed_elems(T);
    const double used = P.J > 1 ? (double)P.P / ((P.H + 1) * 8 * P.U) : (double)P.W / (8 * P.U);  // of the pixels that are contracted
    if (steps < 8 || used < 0.65) return false;
    // one workgroup per compute unit; at most 10 MB of partials (6 MB: 17.5 us instead of 13.2 at 128x256x14x14, 21.8 instead of 16.4 at
    // 128x512x7x7; the sum of the partials took 1 us less)
    int64_t slices = std::max<int64_t>(1, std::min<int64_t>(steps, (256 + tiles - 1) / tiles));
    slices = std::max<int64_t>(1, std::min<int64_t>(slices, ((int64_t)10 << 20) / (packed * 4)));
    P.magicTiles = magic_u32((uint32_t)tiles);  // (all quotients are exact: indices times divisors stay below 2^32)
    P.magicGroup = magic_u32((uint32_t)((P.Omp / ch) * (P.Rp / ch)));
    P.magicKt = magic_u32((uint32_t)(P.Rp / ch));
    P.magicRx = magic_u32((uint32_t)P.rx);
    P.magicRd = magic_u32((uint32_t)P.rd);
    P.magicH = magic_u32((uint32_t)P.H);
    P.magicRowTiles = magic_u32((uint32_t)P.row_tiles);
    P.steps = (int)steps;
    P.per_slice = (int)((steps + slices - 1) / slices);
    P.slices = (int)((steps + P.per_slice - 1) / P.per_slice);
    return true;
}

void wgrad_partial(const Params& P, hipStream_t s) {
    if (P.U == 1) launch<1>(P, s);
    else launch<2>(P, s);
}

}  // namespace gfcwg
}  // namespace canvas
