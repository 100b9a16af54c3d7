// Decodes every workgroup number of plans of the staged FC kernels, and the units, rows and slices behind it, with the arithmetic of the kernels, and
// compares with plain division; and whether each plan has its kernel instance.  Prints the number of plans looked at and, per wrong quotient, the shape.
#include <algorithm>
#include <cstdio>
#include <random>

#include "../../paper_2304_07741_amd/csrc/gfc_staged_kernels.hpp"
#include "../../paper_2304_07741_amd/csrc/gfc_wgrad_kernels.hpp"

using namespace canvas;

static int plans = 0, slices = 0, largest = 0, wrong = 0;

static bool quotients(int last, int d, uint32_t magic) {  // of 0 .. last: wrong first, if at all, just below a multiple
    for (int64_t x = d - 1; x <= last; x += d)
        if ((int)div_magic((uint32_t)x, magic) != x / d) return false;
    return (int)div_magic((uint32_t)last, magic) == last / d;
}

// Whether there is a kernel instance of this tile (gfc_staged_kernel.hpp: launch_np, launch_nb).
static bool has_instance(const gfcst::Params& P) {
    if (P.batches < 1 || P.batches > 4 || (P.np != 1 && P.np != 2 && P.np != 4)) return false;
    if (P.np == 4 && !(P.KW == 3 && P.mo == 2 && P.wo == 1)) return false;
    if (P.KW == 1) return P.wo == 4 ? (P.mo == 1 || P.mo == 2 || P.mo == 4) : P.wo == 1 && P.mo == 1 && P.batches <= 2;
    return P.KW == 3 && ((P.wo == 2 && P.mo == 2) || (P.wo == 1 && (P.mo == 1 || P.mo == 2)));
}

static void look(int N, int G, int R, int K, int Og, int H, int W, bool f32) {
    if (!gfctm::supported(N, G, R, K, K, Og, H, W)) return;
    const gfctm::Params T = gfctm::shape(N, G, R, K, K, Og, H, W);
    bool ok = true;
    gfcst::Params P;
    if (gfcst::plan(P, T, f32, false, false)) {
        plans++;
        largest = std::max(largest, P.tiles);
        ok = has_instance(P);
        const int total = P.tiles * P.ogroups * P.Gm;
        for (int seq = 0; seq < total && ok; seq++) {
            const gfcst::Place at = gfcst::place_of(P, seq);
            const int t2 = seq / P.ogroups;
            ok = at.og == seq - t2 * P.ogroups && at.gmi == t2 / P.tiles && at.tile == t2 - at.gmi * P.tiles;
        }
        if (K == 1) ok = ok && quotients(P.N * P.upi - 1, P.upi, P.magicUpi);
        else
            ok = ok && quotients(P.tiles - 1, P.row_tiles, P.magicRowTiles) && quotients((P.TH + 2) * P.W + 7, P.W, P.magicW) &&
                 (P.J == 1 || quotients(16 * P.np, P.units_out, P.magicUnits));
    }
    gfcwg::Params S;
    if (K == 3 && gfcwg::plan(S, T)) {
        slices++;
        const int ot = S.Omp / 32, kt = S.Rp / 32, tiles = S.Gm * ot * kt;
        ok = ok && quotients(S.slices * tiles - 1, tiles, S.magicTiles) && quotients(tiles - 1, ot * kt, S.magicGroup) && quotients(ot * kt - 1, kt, S.magicKt);
        ok = ok && quotients(1023, S.rx, S.magicRx) && quotients(1023, S.rd, S.magicRd) && quotients(1023, S.H, S.magicH);
        ok = ok && (S.J > 1 || quotients(S.steps - 1, S.row_tiles, S.magicRowTiles));
    }
    if (!ok && wrong++ < 20) std::printf("wrong: N=%d groups=%d rows=%d window=%d outputs=%d plane=%dx%d f32=%d\n", N, G, R, K, Og, H, W, f32);
}

int main() {
    for (int N : {1405, 1404, 2000, 2364, 2500, 2674}) {
        look(N, 1, 64, 1, 64, 56, 56, false);
        look(N, 8, 8, 3, 8, 56, 56, false);
        look(N, 8, 8, 3, 8, 56, 56, true);
    }
    look(200, 1, 64, 1, 64, 160, 160, false);
    look(4170, 1, 96, 1, 96, 32, 32, false);
    look(4789, 1, 16, 3, 16, 56, 56, false);
    std::mt19937 rng(7);
    auto pick = [&](double lo, double hi) { return (int)std::lround(std::exp(std::uniform_real_distribution<double>(std::log(lo), std::log(hi))(rng))); };
    for (int i = 0; i < 4000; i++) {  // up to the largest tensors that the kernels take
        const int K = rng() % 2 ? 1 : 3, G = rng() % 2 ? 1 : 8, R = pick(1, 96), Og = pick(1, 96), H = pick(4, 200), W = pick(4, i % 3 ? 200 : 16);
        const int64_t most = ((int64_t)1 << 29) / ((int64_t)G * std::max(R, Og) * H * W);
        if (most < 1) continue;
        look(i % 4 ? (int)std::min<int64_t>(most, 1 << 20) : pick(1, (double)most), G, R, K, Og, H, W, i % 8 == 7);
    }
    for (int i = 0; i < 20000; i++) {  // ordinary sizes
        const int K = rng() % 2 ? 1 : 3, G = 1 << rng() % 5, R = pick(1, 700), Og = pick(1, 700), H = pick(1, 60), W = pick(4, 60);
        look(pick(1, 130), G, R, K, Og, H, W, i % 8 == 7);
    }
    std::printf("plans %d, weight gradients %d, most pixel tiles %d, wrong %d\n", plans, slices, largest, wrong);
    return wrong != 0;
}
