// Plans of the weight gradient of bf16 FCs without a window, for every count of channels up to 640 and several batches: prints what a tile covers
// beside the weights where that is no reason for it, and workgroups beyond the compute units.
#include <cstdio>

#include "../../paper_2304_07741_amd/csrc/gfc_kernels.hpp"

using namespace canvas;

int main() {
    int plans = 0, wrong = 0;
    for (int C = 64; C <= 640; C += 4)
        for (int side : {7, 14, 20, 28, 40, 56})
            for (int N : {1, 5, 16, 24, 50, 128}) {
                gfc::Params P = gfc::shape(N, 1, C, 1, 1, C, side, side);
                P.src_f32 = P.dy_f32 = 0;
                gfc::prepare_wgrad(P);
                plans++;
                const long steps = P.chunks32, tiles = (long)P.otiles * P.ktiles, small = (long)((C + 63) / 64) * ((C + 63) / 64);
                bool ok = P.wtile == 4 && P.otiles * 32 * P.wo >= C && P.ktiles * 64 >= C && (long)P.slices * P.per_slice >= steps;
                if (P.wo == 4) ok = ok && (tiles * 192 < small * 128 || steps >= 420);  // rows read per step: fewer than with 64 x 64 tiles
                if (tiles <= 256) ok = ok && (tiles * P.slices <= 256 || P.per_slice <= 4);
                if (!ok && wrong++ < 20) std::printf("wrong: C=%d N=%d plane=%d tile=%dx64 slices=%d per_slice=%d steps=%ld\n", C, N, side, 32 * P.wo, P.slices, P.per_slice, steps);
            }
    std::printf("plans %d wrong %d\n", plans, wrong);
    return wrong != 0;
}
