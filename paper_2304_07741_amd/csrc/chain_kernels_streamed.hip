// The instances of the fused-chain kernel for programs without taps that fold windows as they load them (OP_LDFOLD).
#include "chain_kernel.hpp"

namespace canvas {
namespace chain {

void run_streamed(const Program& pg, hipStream_t stream) {
    const int v = pg.vec;  // (divides the rows)
    if (v == 8) launch<1, 8>(pg, stream);
    else launch<1, 4>(pg, stream);
}

}  // namespace chain
}  // namespace canvas
