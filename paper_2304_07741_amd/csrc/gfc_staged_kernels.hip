// Grouped FC on bf16 MFMA with the source tile staged through LDS (gfc_staged_kernel.hpp): the plan and the launches without a middle.
#include "gfc_staged_kernel.hpp"

#include <algorithm>

namespace canvas {
namespace gfcst {

static int log2_up(int x) {
    int l = 0;
    while ((1 << l) < x) l++;
    return l;
}

bool plan_as(Params& P, int KW, int mo, int wo, int np) {
    const int HW = KW / 2;
    P.mo = mo;
    P.wo = wo;
    P.np = np;
    P.KW = KW;
    P.upi = (P.P + 7) / 8;
    if (KW > 1 && P.W < 7) return false;
    if (KW > 1 && P.Rp > 16) P.Rp = (P.Rp + 31) / 32 * 32;  // (a step is 32 rows of one tap)
    const int Kr = KW == 1 ? (P.Rp + 31) / 32 * 32 : P.Rp;  // rows of a pixel in LDS
    P.pitch = Kr * 2 + 16;
    P.quads = Kr / 4;
    P.qshift = Kr == 16 ? 2 : 3;
    P.chunks = Kr / 32;
    P.steps = (KW * KW * P.Rp + 31) / 32;
    const int Om = P.gm * P.Og;
    P.ogroups = (Om + 16 * mo * wo - 1) / (16 * mo * wo);
    const int units = 4 * np * (kWaves / wo);
    if (KW == 1) {
        P.units_in = units;
        P.ushift = log2_up(units / 4);
        P.tiles = (P.N * P.upi + units - 1) / units;
        P.lds_bytes = units * 8 * P.pitch;
        P.last_tile = P.tiles - 1;
    } else {
        // whole images while several fit, else as many rows as fit, spread evenly over the image
        const int per_img = (P.P + 7) / 8;
        if (per_img * 2 <= units && P.N > 1) {
            P.J = std::min(P.N, units / per_img);
            P.TH = P.H;
            P.units_img = per_img;
        } else {
            P.J = 1;
            const int most = std::min(P.H, units * 8 / P.W);
            if (most < 1) return false;
            P.row_tiles = (P.H + most - 1) / most;
            P.TH = (P.H + P.row_tiles - 1) / P.row_tiles;
            for (int t = P.TH; t <= most; t++)  // (whole units where that costs no row tile more)
                if (t * P.W % 8 == 0) {
                    P.TH = t;
                    break;
                }
            P.units_img = ((P.TH + 2 * HW) * P.W + 14) / 8;
        }
        P.row_tiles = (P.H + P.TH - 1) / P.TH;
        P.ishift = P.J > 1 ? log2_up(P.units_img) : 30;
        P.ushift = std::max(0, log2_up(P.J > 1 ? P.J << P.ishift : P.units_img) - 2);
        P.units_out = per_img;
        P.SI = (P.TH + HW) * (P.W + HW);
        P.tiles = (P.N + P.J - 1) / P.J * P.row_tiles;
        P.lds_bytes = (2 * kGuard + P.J * P.SI + HW * (P.W + HW) + HW) * P.pitch;
        P.last_tile = P.tiles - P.row_tiles;
    }
    if (P.lds_bytes > 64 * 1024) return false;
    const int items = (P.quads + (1 << P.qshift) - 1) >> P.qshift << (P.qshift + P.ushift + 2);
    P.batches = (items + kThreads - 1) / kThreads;
    if (P.batches > kMaxBatch) return false;
    P.magicOgroups = magic_u32((uint32_t)P.ogroups);
    P.magicTiles = magic_u32((uint32_t)P.tiles);
    P.magicUpi = magic_u32((uint32_t)P.upi);
    P.magicW = magic_u32((uint32_t)P.W);
    P.magicRowTiles = magic_u32((uint32_t)P.row_tiles);
    P.magicUnits = magic_u32((uint32_t)P.units_out);
    return true;
}

// Which contractions, and which tile.  A workgroup's life is a chain (load, transpose, contract, store) in which most instructions are
// the same for 32 and for 128 pixels, so a launch wants as many pixels per workgroup as leave about one and a half workgroups
// per compute unit.  Measured against the tap-major kernels on 450 shapes of 1-128 images, 16-512 channels, planes of 7x7 to 56x56,
// us there / here: window of 3x3, 8 groups: 128x256x14x14 14.6 / 11.4 (data gradient 19.3 / 12.3), 128x512x7x7 12.8 / 9.2 (13.8 / 10.4),
// 128x64x56x56 26.4 / 22.0 (29.9 / 25.2), 20x80x27x29 7.1 / 5.1 (9.7 / 5.3), 1x256x14x14 6.5 / 4.0, 32x64x28x28 in one group 9.2 / 6.5; without
// a window: 128x256x14x14 12.4 / 10.1, 128x512x7x7 12.2 / 10.2, 128x64x56x56 19.5 / 18.0, 20x80x27x29 5.6 / 4.5, 1x256x14x14 5.0 / 3.5.
// Where the tap-major kernels stay: few rows for few outputs without a window (16 rows for 16 outputs, 9x56x56: 3.7 / 5.0; 40 for 40,
// 105x40x40: 8.0 / 8.5; 192 for 9, 127x14x14: 4.8 / 5.3; 144 for 18, 3x19x46: 5.0 / 5.4), outputs that fill their tiles badly in large launches (264 outputs in 384,
// 55x28x28: 18.7 / 19.9; windows of 80 outputs in 128, 127x33x15: 22.5 / 24.6), several rounds of workgroups with 17 to 32
// rows per group (79x192x28x28 21.9 / 24.3) or 40 rows in 64 (108x320x20x20 40.8 / 45.3), 5x5 windows, rows shorter than 7 pixels.
bool plan(Params& P, const gfctm::Params& T, bool dst_f32, bool adds, bool softmax) {
    const int KW = T.KW;
    if (KW > 3 || (dst_f32 && adds) || (softmax && !(dst_f32 && gfctm::softmax_fusable(T)))) return false;
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
    P.Omp = (T.gm * T.Og + 15) / 16 * 16;
    P.dst_f32 = dst_f32 ? 1 : 0;
    P.softmax = softmax ? 1 : 0;
    if ((int64_t)P.N * P.G * P.R * P.P * 2 < 16) return false;
    const int Om = P.gm * P.Og;
    auto wgs = [&] { return (int64_t)P.tiles * P.ogroups * P.Gm; };
    if (KW == 1) {
        if ((P.Rp <= 64 && Om <= 32) || (P.Rp <= 48 && Om <= 64) || (Om > 16 && Om <= 32)) return false;
        // outputs of a workgroup: 256, 128 or 64, whichever computes the fewest that do not exist (each group of them reads the source again)
        int mo = 1, best = 1 << 30;
        const int wo = Om <= 16 ? 1 : 4;
        for (int m = 4; m >= 1 && wo == 4; m /= 2) {
            const int og = (Om + 64 * m - 1) / (64 * m), cost = og * (64 * m + 32);
            if (cost < best) {
                best = cost;
                mo = m;
            }
        }
        for (;; mo /= 2) {
            if (plan_as(P, KW, mo, wo, 2) && wgs() >= 384) break;
            if (!plan_as(P, KW, mo, wo, 1)) return false;
            if (wgs() >= 256 || mo == 1) break;
        }
        return wo == 1 ? P.batches <= 2 : wgs() <= 512 || 10 * Om >= 7 * P.ogroups * 64 * P.mo;
    }
    const int wo = Om <= 32 ? 1 : 2;
    if (Om > 64 && 10 * ((Om + 63) / 64 * 64) > 14 * Om) return false;
    for (int mo = Om <= 16 ? 1 : 2;; mo /= 2) {
        // workgroups x what one costs with 1, 2, 4 pairs of pixel tiles per wavefront; four only where all workgroups are resident at
        // once (their registers leave two wavefronts per SIMD: 128x256x14x14, 512 workgroups, 12.5 / 12.2 / 11.6 with 1 / 2 / 4;
        // 79x192x28x28, 1264, 22.7 / 23.0 / 24.2; 59x40x56x56 in one group, 826, 23.1 / 19.6 / 22.9)
        int best_np = 0;
        double best = 1e30;
        for (int np = 1; np <= (mo == 2 && wo == 1 ? 4 : 2); np *= 2) {
            if (!plan_as(P, KW, mo, wo, np) || (np == 4 && wgs() > 768)) continue;
            const double each = mo == 1 ? 1.6 + np : (np == 4 ? 4.55 : 0.3 + np), cost = (double)std::max<int64_t>(wgs(), 384) * each;
            if (cost < best) {
                best = cost;
                best_np = np;
            }
        }
        if (!best_np || !plan_as(P, KW, mo, wo, best_np)) return false;
        if (mo == 2 && best > 2500 && (wo == 1 || (2 * P.R * P.Og < P.Rp * P.ogroups * 64 && best > 4000))) return false;
        if (wgs() >= 256 || mo == 1 || wo == 2) return true;
    }
}

void forward(const Params& P, hipStream_t s) {
    const None m;
    if (P.KW == 1) {
        if (P.wo == 4) {
            if (P.mo == 1) launch_np<1, 1, 4, 0>(P, m, s);
            else if (P.mo == 2) launch_np<1, 2, 4, 0>(P, m, s);
            else launch_np<1, 4, 4, 0>(P, m, s);
        } else {
            launch_np<1, 1, 1, 0>(P, m, s);
        }
    } else {
        if (P.wo == 2) launch_np<3, 2, 2, 0>(P, m, s);
        else if (P.mo == 1) launch_np<3, 1, 1, 0>(P, m, s);
        else launch_np<3, 2, 1, 0>(P, m, s);
    }
}

}  // namespace gfcst
}  // namespace canvas
