// Grouped fully-connected contraction on fp32 row tensors, on the fp32 matrix instructions, with an optional implicit
// Unfold of the operand (im2col never materialised).  Section 5 of the Canvas paper: Fully-connected, Group, Unfold.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace canvas {
namespace sfc {

// A row tensor is [N, G, R, P], P = H*W pixels per row.  With a window KH x KW every row is seen TV = KH*KW times,
// shifted by the tap offset (kh - KH/2, kw - KW/2; windows are odd) and zero outside the image; the contraction index is
// k = row*TV + tap, K = R*TV.
struct Params {
    const float* src = nullptr;  // row tensor
    const float* w = nullptr;    // [G][Og][R][TV]; transposed: [G][R][Og][TV], taps flipped
    float* dst = nullptr;        // forward: [N, G*Og, P]
    const float* dy = nullptr;   // weight gradient: [N, G*Og, P]
    float* partial = nullptr;    // weight gradient: [slices][G*Og*K] (one slice: dw itself)
    int64_t N = 0, M = 0;        // images, pixels of the batch (N * P)
    int G = 0, R = 0, Og = 0, KH = 1, KW = 1, TV = 1, K = 0, H = 0, W = 0, P = 0;
    int transposed = 0, acc = 0;  // acc: dst += result
    // a window's operand tile in LDS: image rows with the window's margin, Wp columns each; HP rows per image
    int HP = 0, Wp = 0, S = 0, CS = 0;  // positions per channel, LDS stride of a channel
    uint32_t mP = 0, mW = 0, mHP = 0, mWp = 0;  // 2^32 / d, rounded up
    // forward tile: 16*wm outputs x 16*nt*(4/wm) pixels; weight gradient: 16*mt*wm outputs x 16*nt*(4/wm) contraction indices
    int wm = 1, mt = 1, nt = 1, wide = 0;  // wide: an operand tile of more than 512 positions
    int ktiles = 1, mtiles = 1, nch = 0, slices = 1;
    // narrow: few rows and outputs per group, one thread per pixel on the vector unit; ot outputs, vec pixels per thread
    int narrow = 0, ot = 1, vec = 1;
    int64_t per_slice = 0;                             // pixels per slice; split: positions
    int64_t tiles = 0;                                 // workgroups with work
    // operands cut into three bf16 parts; forward: 32*wm outputs x 32*(4/wm) pixels; weight gradient: 32*wm outputs x 32 rows x
    // one window row, with HP = H + 1 and Wp = W + 1.  (At the end, where the kernels that do not read them load nothing more for them:
    // k_fwd over 5x24 planes of 14x14 8.0 us, 8.25 with them further up)
    const void* wsplit = nullptr;  // the weights as k_split_weights leaves them
    int split = 0;
};

// Whether the window KH x KW on images of H x W is taken implicitly (its operand tile has to fit LDS).
bool window_supported(int KH, int KW, int H, int W);

// Geometry of a contraction whose operand has R rows per group seen through a KH x KW window (1 x 1: any "image").
Params shape(int64_t N, int G, int R, int KH, int KW, int Og, int H, int W);
// The data gradient of a contraction: rows and outputs swapped, transposed weights, the window read backwards.
Params data_gradient_of(const Params& fwd);
// may_split: whether the caller keeps the split weights (split_job) that the plan then asks for.
void prepare_forward(Params& p, bool may_split = false);
// Splits the pixels over slices, at most max_partial_bytes of partials (0: one slice, written straight to dw).
void prepare_wgrad(Params& p, int64_t max_partial_bytes);

// The kernels of sfc_split_kernels.hip: forward and weight gradient with Params::split, and the LDS forward takes (at most kMaxSplitLds).
constexpr int kMaxSplitLds = 128 * 1024;
void forward_split(const Params& p, dim3 grid, hipStream_t s);
void wgrad_split(const Params& p, dim3 grid, hipStream_t s);
size_t split_lds(const Params& p);

// The weights that a split contraction reads (Params::wsplit): 48 * items bytes at `out`, from w as Params::w.
struct SplitJob {
    const float* w = nullptr;
    void* out = nullptr;
    int G = 0, R = 0, Og = 0, TV = 1, transposed = 0, mt32 = 0, items = 0;
};
constexpr int kMaxSplitJobs = 8;
struct SplitJobs {
    SplitJob j[kMaxSplitJobs];
    int n = 0;
};
SplitJob split_job(const Params& p);
void split_weights(const SplitJobs& jobs, hipStream_t s);

// dst[n, g*Og+o, p] (+)= sum_k w[g][o][k] * src_row(n, g, k)[p + off(k)]
void forward(const Params& p, hipStream_t s);
// partial[slice][g][o][k] = sum over the slice's (n, p) of dy[n, g*Og+o, p] * src_row(n, g, k)[p + off(k)]
void wgrad_partial(const Params& p, hipStream_t s);

}  // namespace sfc
}  // namespace canvas
