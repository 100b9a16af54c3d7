// Softmax over the channels of a tensor without taps, behind up to two unaries (Canvas paper, Section 5), forward and backward, each tensor in bf16 or fp32.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace canvas {
namespace smc {

struct Params {
    const void* x = nullptr;   // [N, C, P]
    const void* dy = nullptr;  // backward: gradient of the result
    void* out = nullptr;       // the result, or dx
    int x_f32 = 0, dy_f32 = 0, out_f32 = 0;
    int acc = 0;               // backward, fp32 dx: added to what is there
    int n_before = 0, before[2] = {0, 0};  // unaries of x before the softmax, in their order: relu 0, abs 1 or gelu 2
    int fast = 0;              // exponential and reciprocal by the hardware's instructions (micro-DAGs in bf16)
    int N = 0, C = 0, P = 0;
    int vec = 1, cpt = 8, slices = 1, tiles = 1;  // pixels and channels per thread, wavefronts that share the channels, pixel tiles of a plane
};

bool plan(Params& P, int N, int C, int pixels);  // whether the kernels take it
void forward(const Params& P, hipStream_t s);
void backward(const Params& P, hipStream_t s);

}  // namespace smc
}  // namespace canvas
