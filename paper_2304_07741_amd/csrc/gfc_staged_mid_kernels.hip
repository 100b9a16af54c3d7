// The launches of gfc_staged_kernel.hpp that go on with the element-wise middle of a sampled kernel.
#include "gfc_staged_kernel.hpp"

namespace canvas {
namespace gfcst {

bool takes_middle(const Params& P, bool adjoint, int act) {
    if (P.dst_f32 || P.softmax || act == 4 || P.np > 2) return false;  // (large tiles: too many units per wavefront)
    return adjoint ? P.KW == 1 && P.wo == 4 : P.KW == 3;
}

template <int KW, int MO, int WO, int MID>
static void launch_small(const Params& P, const ufc::MidParams& M, hipStream_t s) {
    if (P.np == 2) launch<KW, MO, 2, WO, MID>(P, M, s);
    else launch<KW, MO, 1, WO, MID>(P, M, s);
}

void forward_with_middle(const Params& P, const ufc::MidParams& M, hipStream_t s) {
    if (P.wo == 2) launch_small<3, 2, 2, 1>(P, M, s);
    else if (P.mo == 1) launch_small<3, 1, 1, 1>(P, M, s);
    else launch_small<3, 2, 1, 1>(P, M, s);
}

void dgrad_with_middle(const Params& P, const ufc::MidParams& M, hipStream_t s) {
    if (P.mo == 1) launch_small<1, 1, 4, 2>(P, M, s);
    else if (P.mo == 2) launch_small<1, 2, 4, 2>(P, M, s);
    else launch_small<1, 4, 4, 2>(P, M, s);
}

}  // namespace gfcst
}  // namespace canvas
