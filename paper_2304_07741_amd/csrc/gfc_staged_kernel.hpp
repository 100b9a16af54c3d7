// Grouped FC (forward, data gradient) on bf16 MFMA with the source tile of a workgroup staged through LDS: the kernels for 3x3 windows and
// for contractions without one over bf16 tensors (Canvas paper, Section 5: Fully-connected, Group, Unfold).
//
// What bounds these launches: at 14x14 and 7x7 pixels they are one round of workgroups, whose time is the number of instructions
// that a wavefront issues from its first load to its last store -- at four wavefronts per SIMD the vector unit is busy throughout,
// although the MFMAs are 1-2 us of it -- and, for weights, the shape of their loads.  Hence
//   * the source is transposed once, on its way into LDS ([pixel][row], a row of zeros around every image and a zero pixel between
//     image rows): a tap of the window is then a constant added to an LDS address, one 16-byte read is an MFMA operand, and no
//     mask is left (the tap-major kernels gather every operand from four registers and mask the taps; 1200 -> 700 vector
//     instructions per wavefront at 128x256x14x14);
//   * the weights are packed in the order in which the wavefronts read them (1 KB contiguous per load; in the tap-major layout
//     a load touches 16 lines, and the same kernel took 15.2 instead of 11.0 us);
//   * the pixels are the rows of the MFMA result, dealt out so that a lane ends up with 8 consecutive pixels of one output.
#pragma once
#include "gfc_staged_kernels.hpp"
#include "launch.hpp"
#include "tile_util.hpp"
#include "ufc_device.hpp"

namespace canvas {
namespace gfcst {

namespace {

using namespace canvas::tile;

constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kGuard = 8;   // LDS slots on either side of the tile that pieces beyond it may write
constexpr int kMaxBatch = 4;  // source pieces (4 rows x 8 pixels) per thread
constexpr int kAhead = 4;   // contraction steps whose weights are in flight

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

extern __shared__ __align__(16) unsigned char lds_src[];

// TP: taps per step of 32 contraction indices: 0 without a window (a step is 32 rows), 1 (a step is 32 rows of one tap), 2 (16 rows
// of two taps).  NW: weight steps in flight; where it is all of them (NW >= steps) they are loaded once.
// MID: the element-wise middle v = x (*|+) shift(act(z)) of a sampled kernel follows in the registers (ufc_device.hpp): 1 its forward, with
// the result as z, 2 its adjoint, with the result as dv (which then never goes to memory).  A lane's results are the 8 pixels of a unit, which
// is what a thread of the launches of ufc_kernels.hip works on.
struct None {};
template <int KW, int MO, int NP, int WO, int TP, int NW, int NB, bool SM = false, int MID = 0>
__global__ __launch_bounds__(kThreads, 2) void k_fc(Params P, std::conditional_t<MID != 0, ufc::MidParams, None> M) {
    constexpr int HW = KW / 2, TV = KW * KW;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wo = wave % WO, wp = wave / WO;
    const int r = lane >> 4, s = lane & 15;
    const int seq = (int)xcd_sequence();
    const Place at_tile = place_of(P, seq);
    const int gmi = at_tile.gmi, tile = at_tile.tile, og = at_tile.og;
    const int gcount = min(P.gm, P.G - gmi * P.gm);
    const int Rm = gcount * P.R, Om = gcount * P.Og;
    const int rows_img = P.G * P.R, outs_img = P.G * P.Og;
    const int grow0 = gmi * P.gm * P.R, gout0 = gmi * P.gm * P.Og;
    const int src_bytes = P.N * rows_img * P.P * 2;
    const rsrc_t rs = make_rsrc(P.src, src_bytes);
    const int pitch = P.pitch, P2 = P.P * 2;
    const int WS = P.W + HW;  // slots of an image row
    const int total_units = P.N * P.upi;
    // the tile of a window: rows [h0, h0 + TH) of images [n0, n0 + J); the pixels of an image begin at `first` in LDS
    const int tg = KW > 1 ? (int)div_magic((uint32_t)tile, P.magicRowTiles) : 0;
    const int h0 = KW > 1 ? (tile - tg * P.row_tiles) * P.TH : 0, n0 = tg * P.J;
    const int first = KW > 1 && P.J == 1 ? (h0 - HW) * P.W : 0;
    const int skip = KW > 1 && P.J > 1 ? HW * P.W : 0;  // (several images: the rows around them are not loaded, but cleared)

    // ---- source pieces of this thread, 4 rows x 8 pixels each: neighbouring lanes take 4 units, then row quads, units, row chunks
    u32x4 v[NB][4];
    int at[NB], col[NB];
    const bool crosses = (P.P & 7) && gmi == P.Gm - 1 && tile >= P.last_tile;  // (uniform) an access may cross the tensor's end
#pragma unroll
    for (int b = 0; b < NB; b++) {
        at[b] = -1;
        const int i = tid + b * kThreads;
        const int u = (i & 3) | (((i >> (2 + P.qshift)) & ((1 << P.ushift) - 1)) << 2);
        const int quad = ((i >> 2) & ((1 << P.qshift) - 1)) | ((i >> (2 + P.qshift + P.ushift)) << P.qshift);
        int n, q;
        bool in;
        if constexpr (KW == 1) {
            const int U = tile * P.units_in + u;
            n = (int)div_magic((uint32_t)U, P.magicUpi);
            q = (U - n * P.upi) * 8;
            if (quad < P.quads) at[b] = u * 8 * pitch + quad * 8;
            in = U < total_units;
        } else {
            const int j = u >> P.ishift, uu = u & ((1 << P.ishift) - 1);
            n = n0 + j;
            q = ((first >> 3) + uu) * 8;
            in = n < P.N && q >= 0 && q < P.P;
            const int rel = q - first + skip;  // -7 at least
            const int h = rel < 0 ? -1 : (int)div_magic((uint32_t)rel, P.magicW);
            col[b] = rel - h * P.W;
            if (quad < P.quads && uu < P.units_img && j < P.J && rel < (P.TH + 2 * HW) * P.W)
                at[b] = (kGuard + HW + j * P.SI + h * WS + col[b]) * pitch + quad * 8;
        }
        const int e = ((n * rows_img + grow0 + quad * 4) * P.P + q) * 2;
        in = in && at[b] >= 0;
        int o[4];
#pragma unroll
        for (int j = 0; j < 4; j++) o[j] = in && quad * 4 + j < Rm ? e + j * P2 : kOob;
        if (crosses) {  // such a piece is loaded so that it ends with the tensor, and moved down below
#pragma unroll
            for (int j = 0; j < 4; j++) o[j] = min(o[j], src_bytes - 16);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) v[b][j] = bload16(rs, o[j]);
        if (crosses) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int gone = in && quad * 4 + j < Rm ? (e + j * P2 - o[j]) >> 1 : 0;  // elements before the piece, 0 .. 7
                u32x4& x = v[b][j];
                if (gone & 4) x = u32x4{x[2], x[3], 0, 0};
                if (gone & 2) x = u32x4{x[1], x[2], x[3], 0};
                if (gone & 1) x = u32x4{(x[0] >> 16) | (x[1] << 16), (x[1] >> 16) | (x[2] << 16), (x[2] >> 16) | (x[3] << 16), x[3] >> 16};
            }
        }
        if (KW > 1 && (P.P & 7)) {  // pixels behind the plane are zeros
            const int left = P.P - q;
            if (left < 8) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t m = (2 * k < left ? 0xffffu : 0u) | (2 * k + 1 < left ? 0xffff0000u : 0u);
#pragma unroll
                    for (int j = 0; j < 4; j++) v[b][j][k] &= m;
                }
            }
        }
    }

    // ---- weights of the first steps
    const int steps = P.steps;
    const rsrc_t rw = make_rsrc(P.wp, P.Gm * P.Omp * steps * 64);
    const int o_first = (og * WO + wo) * 16 * MO;
    const int wbase = lane * 16;
    u32x4 w[NW][MO];
    auto load_w = [&](int ks, int f) {
#pragma unroll
        for (int mo = 0; mo < MO; mo++)  // (past the last output: the last ones' weights, whose results are not stored)
            w[f][mo] = __builtin_amdgcn_raw_buffer_load_b128(rw, wbase, ((gmi * P.Omp + min(o_first + mo * 16, P.Omp - 16)) * steps + ks * 16) * 64, 0);
    };
#pragma unroll
    for (int f = 0; f < NW; f++)
        if (f < steps) load_w(f, f);

    // ---- zeros between the image rows, and around the images where their margins are not loaded
    if constexpr (KW > 1) {
        if (P.J > 1) {
            for (int o = tid * 16; o < P.lds_bytes; o += kThreads * 16) *reinterpret_cast<u32x4*>(lds_src + o) = u32x4{0, 0, 0, 0};
            __syncthreads();
        } else if (tid <= P.TH + 2 * HW) {
#pragma unroll
            for (int k = 0; k < HW; k++)
                for (int o = 0; o < pitch; o += 16) *reinterpret_cast<u32x4*>(lds_src + (kGuard + tid * WS + k) * pitch + o) = u32x4{0, 0, 0, 0};
        }
    }
#pragma unroll
    for (int b = 0; b < NB; b++) {
        if (at[b] < 0) continue;
        unsigned char* to = lds_src + at[b];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint32_t sel = (k & 1) ? 0x07060302u : 0x05040100u;
            u32x2 o;
            o[0] = __builtin_amdgcn_perm(v[b][1][k >> 1], v[b][0][k >> 1], sel);
            o[1] = __builtin_amdgcn_perm(v[b][3][k >> 1], v[b][2][k >> 1], sel);
            *reinterpret_cast<u32x2*>(to) = o;
            to += pitch;
            if (KW > 1 && ++col[b] == P.W) {
                col[b] = 0;
                to += HW * pitch;
            }
        }
    }

    // ---- the pixels of this wavefront: pairs of MFMA tiles = 4 units of 8 pixels.  Rows m = 4 a + e of tile t are pixels
    // 4 (t ^ swap(a)) + e of unit a: a lane's results of the two tiles are the 8 pixels of one unit, and the 16 pixels that a
    // tile reads fall into different banks
    auto swap_of = [](int a) { return (a ^ (a >> 1)) & 1; };
    int ab[2 * NP];
#pragma unroll
    for (int k = 0; k < NP; k++) {
        const int x = (wp * NP + k) * 4 + (s >> 2);
        int j = KW > 1 && P.J > 1 ? (int)div_magic((uint32_t)x, P.magicUnits) : 0;
        const int pu = KW > 1 ? (x - j * P.units_out) * 8 : 0;
        if (KW > 1 && j >= P.J) j = 0;
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const int e = 4 * (t ^ swap_of(s >> 2)) + (s & 3);
            if constexpr (KW == 1) {
                ab[2 * k + t] = (x * 8 + e) * pitch + r * 16;
            } else {
                int px = pu + e;
                if (px >= P.TH * P.W) px = 0;
                const int h = (int)div_magic((uint32_t)px, P.magicW);
                ab[2 * k + t] = (kGuard + HW + j * P.SI + (h + HW) * WS + px - h * P.W) * pitch + (TP == 2 ? r & 1 : r) * 16;
            }
        }
    }
    float4_t acc[MO][2 * NP];
#pragma unroll
    for (int mo = 0; mo < MO; mo++)
#pragma unroll
        for (int t = 0; t < 2 * NP; t++) acc[mo][t] = float4_t{0.f, 0.f, 0.f, 0.f};

    // ---- where the results go: the 8 pixels of unit r of each pair, output s of each tile
    const int dst_bytes = P.N * outs_img * P2;
    const rsrc_t rd = make_rsrc(P.dst, P.dst_f32 ? dst_bytes * 2 : dst_bytes), rad = make_rsrc(P.addend, dst_bytes);
    int de[NP], left[NP], px0[NP];
#pragma unroll
    for (int k = 0; k < NP; k++) {
        const int x = (wp * NP + k) * 4 + r;
        int n, p;
        if constexpr (KW == 1) {
            const int U = tile * P.units_in + x;
            n = (int)div_magic((uint32_t)U, P.magicUpi);
            p = (U - n * P.upi) * 8;
            left[k] = U < total_units ? P.P - p : 0;
        } else {
            const int j = P.J > 1 ? (int)div_magic((uint32_t)x, P.magicUnits) : 0, pu = (x - j * P.units_out) * 8;
            n = n0 + j;
            p = h0 * P.W + pu;
            left[k] = j < P.J && n < P.N ? min(P.TH, P.H - h0) * P.W - pu : 0;
        }
        px0[k] = p;
        de[k] = ((n * outs_img + gout0 + o_first + s) * P.P + p) * 2;
    }
    // (what the middle reads: ahead of the contraction where the registers have room for it)
    constexpr bool kEarly = NP * MO <= 4;
    ufc::Near near[MID ? MO : 1];
    ufc::Read read[MID ? (kEarly ? NP : 1) : 1][MID ? MO : 1];
    auto unit_of = [&](int k, int mo) {
        ufc::UnitAt u;
        u.e = (de[k] + mo * 16 * P2) >> 1;
        u.p = px0[k];
        u.nvalid = o_first + mo * 16 + s < Om ? max(0, min(left[k], 8)) : 0;
        return u;
    };
    if constexpr (MID != 0) {
#pragma unroll
        for (int mo = 0; mo < MO; mo++) near[mo] = ufc::shift_of(M, gout0 + min(o_first + mo * 16 + s, Om - 1));
        if constexpr (kEarly) {
#pragma unroll
            for (int k = 0; k < NP; k++)
#pragma unroll
                for (int mo = 0; mo < MO; mo++) ufc::mid_read<MID>(M, unit_of(k, mo), near[mo], read[k][mo]);
        }
    }
    u32x4 ad[MID ? 1 : NP][MO];
    if (!MID && P.addend) {
#pragma unroll
        for (int k = 0; k < NP; k++)
#pragma unroll
            for (int mo = 0; mo < MO; mo++) ad[MID ? 0 : k][mo] = bload16(rad, o_first + mo * 16 + s < Om && left[k] >= 8 ? de[k] + mo * 16 * P2 : kOob);
    }
    __syncthreads();

    // ---- contraction
    auto step = [&](int f, const int (&off)[2 * NP]) {
        u32x4 a[2 * NP];
#pragma unroll
        for (int t = 0; t < 2 * NP; t++) a[t] = *reinterpret_cast<const u32x4*>(lds_src + off[t]);
#pragma unroll
        for (int t = 0; t < 2 * NP; t++)
#pragma unroll
            for (int mo = 0; mo < MO; mo++) acc[mo][t] = mfma32(a[t], w[f][mo], acc[mo][t]);
    };
    if constexpr (TP == 2) {
        static_assert(NW == (TV + 1) / 2, "all taps' weights");
#pragma unroll
        for (int f = 0; f < NW; f++) {
            constexpr int last = TV - 1;
            const int ta = 2 * f, tb = 2 * f + 1 > last ? last : 2 * f + 1;
            const int oa = ((ta / KW - HW) * WS + ta % KW - HW) * pitch, ob = ((tb / KW - HW) * WS + tb % KW - HW) * pitch;
            const int o = r < 2 ? oa : ob;
            int off[2 * NP];
#pragma unroll
            for (int t = 0; t < 2 * NP; t++) off[t] = 2 * f + 1 > last && r >= 2 ? kGuard * pitch : ab[t] + o;  // (slot kGuard holds zeros)
            step(f, off);
        }
    } else {
        int so = KW > 1 ? -(HW * WS + HW) * pitch : 0, kw = 0, c = 0;  // offset of the step's tap and rows
        for (int k0 = 0; k0 < steps; k0 += NW) {
#pragma unroll
            for (int f = 0; f < NW; f++) {
                if (k0 + f < steps) {
                    int off[2 * NP];
#pragma unroll
                    for (int t = 0; t < 2 * NP; t++) off[t] = ab[t] + so;
                    step(f, off);
                    if (k0 + f + NW < steps) load_w(k0 + f + NW, f);
                    so += 64;
                    if (KW > 1 && ++c == P.chunks) {
                        c = 0;
                        so += pitch - P.chunks * 64;
                        if (++kw == KW) {
                            kw = 0;
                            so += (WS - KW) * pitch;
                        }
                    }
                }
            }
        }
    }

    // ---- results
    if constexpr (SM) {  // the outputs of a pixel are the 16 lanes of a row: maximum and sum by lane exchanges
        static_assert(MO == 1 && WO == 1 && KW == 1, "softmax: one tile of outputs, no window");
#pragma unroll
        for (int t = 0; t < 2 * NP; t++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                float m = s < Om ? acc[0][t][q] : -INFINITY;
#pragma unroll
                for (int d = 1; d < 16; d *= 2) m = fmaxf(m, __shfl_xor(m, d));
                const float x = s < Om ? expf(acc[0][t][q] - m) : 0.f;
                float sum = x;
#pragma unroll
                for (int d = 1; d < 16; d *= 2) sum += __shfl_xor(sum, d);
                acc[0][t][q] = x * (1.f / sum);
            }
    }
    const bool sw = swap_of(r);
#pragma unroll
    for (int k = 0; k < NP; k++) {
        if constexpr (MID != 0 && !kEarly) {
#pragma unroll
            for (int mo = 0; mo < MO; mo++) ufc::mid_read<MID>(M, unit_of(k, mo), near[mo], read[0][mo]);
        }
        if constexpr (MID == 2) {
#pragma unroll
            for (int mo = 0; mo < MO; mo++) {
                const float4_t lo = sw ? acc[mo][2 * k + 1] : acc[mo][2 * k], hi = sw ? acc[mo][2 * k] : acc[mo][2 * k + 1];
                const float dv[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                ufc::mid_backward_unit(M, unit_of(k, mo), near[mo], read[kEarly ? k : 0][mo], dv);
            }
            continue;
        }
#pragma unroll
        for (int mo = 0; mo < MO; mo++) {
            if (left[k] <= 0 || o_first + mo * 16 + s >= Om) continue;
            const int e = de[k] + mo * 16 * P2;
            if (!MID && P.dst_f32) {
                const float4_t lo = sw ? acc[mo][2 * k + 1] : acc[mo][2 * k], hi = sw ? acc[mo][2 * k] : acc[mo][2 * k + 1];
                u32x4 a, b;
                __builtin_memcpy(&a, &lo, 16);
                __builtin_memcpy(&b, &hi, 16);
                if (left[k] >= 8) {
                    bstore16(rd, e * 2, a);
                    bstore16(rd, e * 2 + 16, b);
                } else {
#pragma unroll
                    for (int q = 0; q < 7; q++)
                        if (q < left[k]) __builtin_amdgcn_raw_buffer_store_b32(q < 4 ? a[q] : b[q - 4], rd, e * 2 + 4 * q, 0, 0);
                }
                continue;
            }
            u32x4 d;
            if (!MID && P.addend && left[k] >= 8) {
                const float4_t lo = sw ? acc[mo][2 * k + 1] : acc[mo][2 * k], hi = sw ? acc[mo][2 * k] : acc[mo][2 * k + 1];
                const u32x4& x = ad[MID ? 0 : k][mo];
                d[0] = pack_bf16(lo[0] + lo_f32(x[0]), lo[1] + hi_f32(x[0]));
                d[1] = pack_bf16(lo[2] + lo_f32(x[1]), lo[3] + hi_f32(x[1]));
                d[2] = pack_bf16(hi[0] + lo_f32(x[2]), hi[1] + hi_f32(x[2]));
                d[3] = pack_bf16(hi[2] + lo_f32(x[3]), hi[3] + hi_f32(x[3]));
            } else if (!MID && P.addend) {
                const float4_t lo = sw ? acc[mo][2 * k + 1] : acc[mo][2 * k], hi = sw ? acc[mo][2 * k] : acc[mo][2 * k + 1];
                const float x8[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                float y8[8];
#pragma unroll
                for (int q = 0; q < 8; q++) y8[q] = x8[q] + lo_f32(__builtin_amdgcn_raw_buffer_load_b16(rad, q < left[k] ? e + 2 * q : kOob, 0, 0));
#pragma unroll
                for (int q = 0; q < 4; q++) d[q] = pack_bf16(y8[2 * q], y8[2 * q + 1]);
            } else {
                const float4_t &t0 = acc[mo][2 * k], &t1 = acc[mo][2 * k + 1];
                const uint32_t a0 = pack_bf16(t0[0], t0[1]), a1 = pack_bf16(t0[2], t0[3]), b0 = pack_bf16(t1[0], t1[1]), b1 = pack_bf16(t1[2], t1[3]);
                d = u32x4{sw ? b0 : a0, sw ? b1 : a1, sw ? a0 : b0, sw ? a1 : b1};
            }
            if constexpr (MID == 1) ufc::mid_forward_unit(M, unit_of(k, mo), near[mo], read[kEarly ? k : 0][mo], d);
            if (left[k] >= 8) {
                bstore16(rd, e, d);
            } else {
                int o = e;
                uint32_t x0 = d[0], x1 = d[1];
                if (left[k] & 4) {
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{x0, x1}, rd, o, 0, 0);
                    o += 8;
                    x0 = d[2];
                    x1 = d[3];
                }
                if (left[k] & 2) {
                    __builtin_amdgcn_raw_buffer_store_b32(x0, rd, o, 0, 0);
                    o += 4;
                    x0 = x1;
                }
                if (left[k] & 1) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(x0 & 0xffffu), rd, o, 0, 0);
            }
        }
    }
}

// (The instances are those that plan comes to, as tests/host/staged_plans.cpp checks.)
template <int KW, int MO, int NP, int WO, int TP, int NW, int MID, bool SM = false, class M>
void launch_nb(const Params& P, const M& m, hipStream_t s) {
    const dim3 grid((unsigned)(P.tiles * P.ogroups * P.Gm)), block(kThreads);
    if (P.batches == 1) {
        CANVAS_LAUNCH((k_fc<KW, MO, NP, WO, TP, NW, 1, SM, MID>), grid, block, (size_t)P.lds_bytes, s, P, m);
    } else if (P.batches == 2) {
        CANVAS_LAUNCH((k_fc<KW, MO, NP, WO, TP, NW, 2, SM, MID>), grid, block, (size_t)P.lds_bytes, s, P, m);
    } else if constexpr (KW > 1 || WO > 1) {
        CANVAS_LAUNCH((k_fc<KW, MO, NP, WO, TP, NW, kMaxBatch, SM, MID>), grid, block, (size_t)P.lds_bytes, s, P, m);
    }
}

template <int KW, int MO, int NP, int WO, int MID, class M>
void launch(const Params& P, const M& m, hipStream_t s) {
    if constexpr (KW == 1) {
        if constexpr (MO == 1 && WO == 1 && MID == 0) {
            if (P.softmax) {
                launch_nb<1, 1, NP, 1, 0, kAhead, 0, true>(P, m, s);
                return;
            }
        }
        launch_nb<1, MO, NP, WO, 0, kAhead, MID>(P, m, s);
    } else {
        if (P.Rp == 16) launch_nb<KW, MO, NP, WO, 2, (KW * KW + 1) / 2, MID>(P, m, s);
        else if (P.Rp == 32) launch_nb<KW, MO, NP, WO, 1, KW * KW, MID>(P, m, s);
        else launch_nb<KW, MO, NP, WO, 1, kAhead, MID>(P, m, s);
    }
}

template <int KW, int MO, int WO, int MID, class M>
void launch_np(const Params& P, const M& m, hipStream_t s) {
    if (P.np == 4) {
        if constexpr (KW == 3 && MO == 2 && WO == 1) launch<KW, MO, 4, WO, MID>(P, m, s);
    } else if (P.np == 2) {
        launch<KW, MO, 2, WO, MID>(P, m, s);
    } else {
        launch<KW, MO, 1, WO, MID>(P, m, s);
    }
}

}  // namespace

}  // namespace gfcst
}  // namespace canvas
