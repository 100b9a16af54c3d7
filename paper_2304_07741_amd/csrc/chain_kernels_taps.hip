// The instances of the fused-chain kernel for programs with taps.
#include "chain_kernel.hpp"

namespace canvas {
namespace chain {

void run_taps(const Program& pg, hipStream_t stream) {
    const int v = pg.vec;
    if (pg.tm <= 9) {
        if (v == 4) launch<9, 4>(pg, stream);
        else if (v == 2 && f32_windows(pg)) launch<9, 2>(pg, stream);
        else if (v == 2) launch<9, 2, false>(pg, stream);
        else launch<9, 1>(pg, stream);
    } else {
        launch<25, 1>(pg, stream);
    }
}

}  // namespace chain
}  // namespace canvas
