// Weight gradient of a bf16 FC behind a 3x3 window on image rows of at most 16 pixels (gfc_wgrad_kernels.hip).  It shares the geometry (merged
// groups, padded rows) and the layout of the partials with the tap-major kernels (gfc_tm_kernels.hpp).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "gfc_tm_kernels.hpp"

namespace canvas {
namespace gfcwg {

struct Params {
    const uint16_t* src = nullptr;  // [N, G, R, P] bf16
    const uint16_t* dy = nullptr;   // [N, G*Og, P] bf16
    float* partial = nullptr;       // [slices][Gm][Omp][9][Rp] fp32
    int N = 0, H = 0, W = 0, P = 0;
    int G = 0, R = 0, Og = 0, gm = 1, Gm = 0, Rp = 0, Omp = 0;
    int U = 1;                      // 8-pixel units of an image row, 1 or 2
    int J = 1, TH = 1, row_tiles = 1;  // a step: TH rows of J images (J > 1: whole images)
    int rx = 0, rd = 0;             // image rows of src and of dy that a step loads per channel
    int xu = 0, du = 0;             // units per channel in LDS, of src and of dy (odd: 16 channels fall into different banks)
    int ksteps = 0;                 // contraction steps of 32 pixels per step
    int steps = 0, per_slice = 0, slices = 0;
    int lds_bytes = 0;              // of one step; two are in LDS
    uint32_t magicTiles = 0, magicGroup = 0, magicKt = 0, magicRx = 0, magicRd = 0, magicH = 0, magicRowTiles = 0;
};

// Whether the weight gradient of T runs here; sets everything but the pointers.
bool plan(Params& P, const gfctm::Params& T);
void wgrad_partial(const Params& P, hipStream_t s);

}  // namespace gfcwg
}  // namespace canvas
