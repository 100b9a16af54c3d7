// Grouped FC through LDS (gfc_staged_kernel.hpp): bf16 source, 3x3 window or none, for the shapes where it is faster than the
// tap-major kernels (gfc_tm_kernels.hpp), whose geometry (merged groups, padded rows) it shares.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "gfc_tm_kernels.hpp"
#include "magic.hpp"
#include "ufc_kernels.hpp"

namespace canvas {
namespace gfcst {

struct Params {
    const uint16_t* src = nullptr;     // [N, G, R, P] bf16
    const uint16_t* wp = nullptr;      // weights packed by a job of wprep_kernels.hpp, kind 2: [Gm][Omp / 16][steps][64 lanes][8]
    void* dst = nullptr;               // [N, G*Og, P] bf16, or fp32 (no addend then)
    const uint16_t* addend = nullptr;  // optional tensor of dst's shape added before rounding
    int N = 0, H = 0, W = 0, P = 0, upi = 0;
    int G = 0, R = 0, Og = 0, gm = 1, Gm = 0, Rp = 0, Omp = 0;
    int mo = 1, wo = 1, np = 1;        // 16 * mo outputs and np pairs of 16-pixel tiles per wavefront, wo wavefronts side by side over the outputs
    int tiles = 1, ogroups = 1, last_tile = 0;  // pixel tiles of the batch, workgroups over the outputs of a merged group
    int pitch = 0, lds_bytes = 0;      // bytes of a pixel in LDS, of the tile
    int KW = 1, batches = 1;           // window; source pieces per thread
    int dst_f32 = 0, softmax = 0;
    int steps = 0, chunks = 0;         // steps of 32 contraction indices; of one tap
    int units_in = 1, quads = 0, qshift = 2, ushift = 0, ishift = 0;  // 8-pixel units per tile (no window), 4-row quads; how threads are dealt out to them
    int TH = 1, J = 1, row_tiles = 1;  // windows: rows of a tile, images of a tile
    int SI = 0, units_img = 1, units_out = 1;         // slots and loaded units per image
    uint32_t magicOgroups = 0, magicTiles = 0, magicUpi = 0, magicW = 0, magicRowTiles = 0, magicUnits = 0;
};

// What workgroup number `seq` works on: outputs fastest, then pixel tiles, then merged groups.  (Pixel tiles and workgroups are not limited by
// gfctm::supported as units, image rows and pixels of a plane are: from 2^16 tiles on their products pass 2^32.)
struct Place {
    int gmi, tile, og;
};
__host__ __device__ inline Place place_of(const Params& P, int seq) {
    Place at;
    const int t2 = div_magic(seq, P.ogroups, P.magicOgroups, at.og);
    at.gmi = div_magic(t2, P.tiles, P.magicTiles, at.tile);
    return at;
}

// Whether the contraction of T (a source in bf16) runs here, and with which tile; sets everything but the pointers.
bool plan(Params& P, const gfctm::Params& T, bool dst_f32, bool adds, bool softmax);
inline int64_t packed_elems(const Params& P) { return (int64_t)P.Gm * P.Omp * P.steps * 32; }
void forward(const Params& P, hipStream_t s);
// Whether a planned launch has a form that goes on with the middle v = x (*|+) shift(act(z)) of a sampled kernel: with its forward (the result
// is z, stored as ever, and v follows), or with its adjoint (the result is dv, which is not stored; dx1 and dz follow); act as in
// MidParams.
bool takes_middle(const Params& P, bool adjoint, int act);
void forward_with_middle(const Params& P, const ufc::MidParams& M, hipStream_t s);  // M: x, v
void dgrad_with_middle(const Params& P, const ufc::MidParams& M, hipStream_t s);    // M: x, z, dz, dx1
bool plan_as(Params& P, int KW, int mo, int wo, int np);  // the tile `mo, wo, np`, or false where it does not fit

}  // namespace gfcst
}  // namespace canvas
