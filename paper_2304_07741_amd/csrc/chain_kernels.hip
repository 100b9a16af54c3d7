// Fused-chain kernels: one workgroup = one image x one tile of the image plane (plus a halo in backward programs) x one
// range of channels; one thread = V consecutive pixels; the program (chain_isa.hpp) arrives in the kernel arguments and
// is interpreted with workgroup-uniform control flow.  A tensor access is one vector access of V elements per thread,
// coalesced along the plane (the innermost dims of NCHW); stencil offsets are address offsets of those accesses;
// reductions over taps stay in registers; the statistics of a softmax over channels and the gradient hand-over of
// shifted loads live in LDS.
#include "chain_kernel.hpp"

namespace canvas {
namespace chain {

void run(const Program& pg, hipStream_t stream) {
    const int v = pg.vec;
    if (pg.H * pg.W % v != 0) {
        run_ragged(pg, stream);
        return;
    }
    if (pg.tm <= 1 && streams_windows(pg)) {
        run_streamed(pg, stream);
    } else if (pg.tm <= 1) {
        if (v == 16) launch<1, 16, false>(pg, stream);
        else if (v == 8) launch<1, 8, false>(pg, stream);
        else if (v == 4) launch<1, 4, false>(pg, stream);
        else if (v == 2) launch<1, 2, false>(pg, stream);
        else launch<1, 1, false>(pg, stream);
    } else {
        run_taps(pg, stream);
    }
}

}  // namespace chain
}  // namespace canvas
