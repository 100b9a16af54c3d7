// Sums of weight-gradient partials, several FCs per launch: every workgroup of a weight-gradient kernel writes one
// partial, and the fixed-order sums over the partials of all FCs of a DAG run as ONE launch at the end of
// the backward pass (each alone is a launch of a few microseconds on well under a megabyte).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace canvas {
namespace wreduce {

struct Job {
    const float* partial = nullptr;  // [slices][count] fp32
    float* dw = nullptr;             // [G][Og][R][TV] fp32, overwritten
    int slices = 0;
    int kind = 0;                    // 0: partials in the order of dw; 1: tap-major packed [Gm][Omp][TV][Rp] (gfc_tm_kernels.hpp)
    unsigned count = 0;              // elements per partial
    int segs = 1;                    // segments of partials per element (1 ... 16), combined through LDS in order
    int vec = 1;                     // consecutive elements per thread (4 where the partials' elements are 16-byte aligned: count % 4 == 0)
    unsigned blocks = 0;             // workgroups of 256 threads = vec * 256 / segs elements each
    int G = 0, R = 0, Og = 0, TV = 1, gm = 1, Omp = 0, Rp = 0;  // kind 1 only
    uint32_t magicRp = 0, magicTV = 0, magicOmp = 0, magicOg = 0, magicR = 0;    // exact division by them, or 0: divided by
};

constexpr int kMaxJobs = 8;
struct Jobs {
    Job j[kMaxJobs];
    int n = 0;
};

// Fills segs, vec, blocks and the multipliers from the rest.
void plan(Job& job);

void run(const Jobs& jobs, hipStream_t s);

}  // namespace wreduce
}  // namespace canvas
