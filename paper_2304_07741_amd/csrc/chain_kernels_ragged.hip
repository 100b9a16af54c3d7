// The instances of the fused-chain kernel for planes that are no multiple of the pixels of a thread.
#include "chain_kernel.hpp"

namespace canvas {
namespace chain {

void run_ragged(const Program& pg, hipStream_t stream) {
    const int v = pg.vec;
    if (pg.tm <= 1) {
        if (v == 16) launch<1, 16, false, true>(pg, stream);
        else if (v == 8) launch<1, 8, false, true>(pg, stream);
        else if (v == 4) launch<1, 4, false, true>(pg, stream);
        else launch<1, 2, false, true>(pg, stream);
    } else if (v == 4) {
        launch<9, 4, true, true>(pg, stream);
    } else if (f32_windows(pg)) {
        launch<9, 2, true, true>(pg, stream);
    } else {
        launch<9, 2, false, true>(pg, stream);
    }
}

}  // namespace chain
}  // namespace canvas
