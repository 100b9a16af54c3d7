// Lowering by units, for every legal DAG.  The DAG is cut at its FC nodes; the runs of memory-bound primitives
// between them are grown, one node at a time in topological order, into fused chains (chain_plan.hpp: one forward
// and one backward kernel per chain, nothing inside a chain is materialised, an Unfold is never written out); a
// node joins the chain of one of its operands as long as the grown chain still compiles (a stencil above a
// reduction, a blend across channel counts, too many taps, registers, instructions or LDS end a chain).  What no
// chain takes (folds over space or channels, joint softmax, grouped blends ...) is one kernel per node, and so is
// everything when fusion is switched off.  FC nodes run on the bf16 MFMA kernels (bf16 dtype) or the fp32 ones.
// Tensors that cross a unit boundary live in the workspace as fp32 [N, C, T, H, W] together with their gradients;
// x, y, dy and dx are read and written in place, in their own type, wherever the unit at that end can do so.
#include "lowering.hpp"
#include "../../include/canvas_dag.h"
#include "chain_kernels.hpp"
#include "chain_plan.hpp"
#include "fc_emit.hpp"
#include "gfc_kernels.hpp"
#include "gfc_tm_kernels.hpp"
#include "ref_kernels.hpp"
#include "sfc_kernels.hpp"
#include "smc_kernels.hpp"
#include "ufc_kernels.hpp"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <stdexcept>

namespace canvas {

namespace {

constexpr int64_t kMaxSfcPartialBytes = 16 << 20;

std::string sfc_name(const char* what, const sfc::Params& q) { return std::string(what) + (q.TV > 1 ? "_unfold" : "") + (q.narrow ? "_narrow" : ""); }

struct Layout {
    std::vector<int64_t> val, grad, wf;  // byte offsets into the workspace; -1 = not in the workspace
    std::vector<int64_t> wt, part;       // per fc (bf16 path): transposed weights, weight-gradient partials
    uint64_t total = 0;
};

const char* op_name(Op op) {
    switch (op) {
    case Op::Unfold: return "unfold";
    case Op::Shift: return "shift";
    case Op::Fc: return "fc";
    case Op::Unary: return "unary";
    case Op::Binary: return "binary";
    case Op::Softmax: return "softmax";
    case Op::Fold: return "fold";
    case Op::Group: return "group";
    default: return "input";
    }
}

}  // namespace

namespace {

struct Unit {
    bool chain = false;
    std::vector<int> nodes;       // ascending
    chain::UnitPlan plan;         // chain units
};

// A program ready to launch: the pointers of its external tensors are resolved per call.
struct Binding {
    int node = -1;
    chain::ExtRole role = chain::kValueIn;
    int where = 0;   // 0 = workspace offset `off` (fp32), 1 = x, 2 = y, 3 = dy, 4 = dx (the caller's tensors, in the DAG's dtype)
    int64_t off = 0;
};

void run_program(const chain::Program& pg0, const std::vector<Binding>& bind, bool bf16, const RunArgs& a) {
    chain::Program pg = pg0;
    pg.fast_math = bf16 ? 1 : 0;
    for (size_t i = 0; i < bind.size(); i++) {
        const Binding& b = bind[i];
        switch (b.where) {
        case 0: pg.ext[i].ptr = a.ws + b.off; pg.ext[i].bf16 = 0; break;
        case 1: pg.ext[i].ptr = const_cast<void*>(a.x); pg.ext[i].bf16 = bf16; break;
        case 2: pg.ext[i].ptr = a.y; pg.ext[i].bf16 = bf16; break;
        case 3: pg.ext[i].ptr = const_cast<void*>(a.dy); pg.ext[i].bf16 = bf16; break;
        default: pg.ext[i].ptr = a.dx; pg.ext[i].bf16 = bf16; break;
        }
    }
    chain::run(pg, a.stream);
}

// A tensor of a unit as its kernel finds it.
const void* bound(const Binding& b, const RunArgs& a) {
    switch (b.where) {
    case 0: return a.ws + b.off;
    case 1: return a.x;
    case 2: return a.y;
    case 3: return a.dy;
    default: return a.dx;
    }
}

// Whether the unit is a softmax over channels, behind up to two unaries of its input, and nothing else, which has kernels of its own.
bool softmax_of_channels(const Dag& dag, const Unit& U, smc::Params& P) {
    const int n = (int)U.nodes.size();
    if (n > 3 || U.plan.inputs.size() != 1 || U.plan.outputs != std::vector<int>{U.nodes.back()}) return false;
    for (int i = 0; i < n; i++) {  // (a path: each node reads the one before it)
        const Node& nd = dag.nodes[U.nodes[i]];
        if (nd.a != (i ? U.nodes[i - 1] : U.plan.inputs[0]) || nd.T != 1) return false;
        if (i == n - 1) return nd.op == Op::Softmax && nd.kind == kAxisC && dag.nodes[nd.a].T == 1 && smc::plan(P, dag.N, nd.C, dag.H * dag.W);
        if (nd.op != Op::Unary || (nd.kind != kRelu && nd.kind != kAbs && nd.kind != kGelu)) return false;
        P.before[P.n_before++] = nd.kind;
    }
    return false;
}

// Whether the unit is y = x (*|+) shift(act(x)) of one tensor and nothing else: an activation and shifts of disjoint channel slices in any order
// (an activation that keeps zeros commutes with what shifts fill in), blended with the tensor itself.  Kernels of their own take it where
// it goes from x to y in bf16: 3-4 operations per pixel and tensor access against the dispatch, the LDS registers and the general masks of
// the interpreted programs (128x64 planes of 56x56, forward + backward, us: gelu, half shifted, product 48.7 + 121.6 / 26.3 + 36.7; shifts, relu, sum
// 124.6 / 48.4).
bool self_blend(const Dag& dag, const Unit& U, ufc::MidParams& M) {
    if (U.plan.inputs.size() != 1 || U.plan.outputs.size() != 1 || U.nodes.size() < 2) return false;
    const int in = U.plan.inputs[0], out = U.plan.outputs[0];
    const Node& b = dag.nodes[out];
    if (out != U.nodes.back() || b.op != Op::Binary || (b.kind != kAdd && b.kind != kMul) || b.T != 1 || dag.nodes[in].T != 1) return false;
    const int other = b.a == in ? b.b : (b.b == in ? b.a : -1);
    if (other < 0 || other == in) return false;
    const int C = dag.nodes[in].C, H = dag.H, W = dag.W;
    const int64_t P = (int64_t)H * W, upi = (P + 7) / 8;
    if (dag.N * (int64_t)C * P * 2 >= ((int64_t)1 << 31) || dag.N * (int64_t)C * upi >= ((int64_t)1 << 31)) return false;
    std::vector<bool> shifted(C, false);
    size_t seen = 1;
    for (int k = other; k != in; k = dag.nodes[k].a, seen++) {
        const Node& nd = dag.nodes[k];
        if (std::find(U.nodes.begin(), U.nodes.end(), k) == U.nodes.end() || nd.T != 1) return false;
        if (nd.op == Op::Unary) {
            if (M.act >= 0 || (nd.kind != kRelu && nd.kind != kAbs && nd.kind != kGelu)) return false;
            M.act = nd.kind;
        } else if (nd.op == Op::Shift) {
            if ((nd.dh == 0 && nd.dw == 0) || nd.c1 <= nd.c0) continue;
            if (M.nslices == ufc::kMaxSlices) return false;
            for (int c = nd.c0; c < nd.c1; c++) {
                if (shifted[c]) return false;
                shifted[c] = true;
            }
            M.c0[M.nslices] = nd.c0;
            M.c1[M.nslices] = nd.c1;
            M.dh[M.nslices] = nd.dh;
            M.dw[M.nslices] = nd.dw;
            M.nslices++;
        } else {
            return false;
        }
    }
    if (seen != U.nodes.size()) return false;
    M.bin = b.kind == kMul ? 1 : 0;
    M.N = dag.N;
    M.C = C;
    M.H = H;
    M.W = W;
    M.P = (int)P;
    M.upi = (int)upi;
    M.magicW = gfc::magic_u32(W);
    M.magicUpi = gfc::magic_u32((uint32_t)upi);
    return true;
}

}  // namespace

// Costs of chains by their plain programs, with whole planes and with halos; negative where there is none (the searches ask for some chains
// several times).
typedef std::map<std::vector<int>, std::pair<double, double>> ChainCosts;

// The lowering whose search over the chains goes by the costs with halos or by the others; nullptr where it comes to the chains of `unlike`.
static std::unique_ptr<Lowering> lower_by(const Dag& dag, bool bf16, bool fuse_chains, bool inference, bool halos, ChainCosts& costs, const Lowering* unlike) {
    auto low = std::make_unique<Lowering>();
    const int n = (int)dag.nodes.size();
    const int P = dag.P();
    const int64_t N = dag.N;
    Layout lay;
    lay.val.assign(n, -1);
    lay.grad.assign(n, -1);
    lay.wf.assign(dag.n_weights, -1);
    uint64_t off = 0;
    auto take = [&](int64_t numel) {
        uint64_t o = off;
        off += align_up((uint64_t)numel * 4);
        return (int64_t)o;
    };
    // FC nodes read an Unfold operand implicitly: an Unfold whose every consumer is such an FC is never materialised
    // (no value, no gradient, no launch).  The bf16 kernels take windows up to 7 x 7, the fp32 ones those whose rows
    // fit their operand tile.
    auto bytes_ok = [&](int64_t numel) { return numel * 4 < ((int64_t)1 << 31); };
    bool mfma = bf16 && dag.W >= 4 && (int64_t)dag.N * dag.P() < ((int64_t)1 << 28);
    for (int k = 1; k < n && mfma; k++) {
        const Node& f = dag.nodes[k];
        if (!f.live || f.op != Op::Fc) continue;
        const Node& A = dag.nodes[f.a];
        const int srcn = A.op == Op::Unfold ? A.a : f.a;  // the larger of the two possible operands is f.a
        mfma = bytes_ok(dag.numel(f.a)) && bytes_ok(dag.numel(srcn)) && bytes_ok(dag.numel(k)) &&
               bytes_ok((int64_t)f.out * (A.C / f.groups) * A.T);
    }
    std::vector<bool> virt(n, false);
    if (mfma || !bf16) {
        for (int k = 1; k < n; k++) {
            const Node& u = dag.nodes[k];
            if (!u.live || u.op != Op::Unfold || u.kh > 7 || u.kw > 7) continue;
            if (!bf16 && !sfc::window_supported(u.kh, u.kw, dag.H, dag.W)) continue;
            bool only_fc = true;
            for (int j = k + 1; j < n; j++) {
                const Node& c = dag.nodes[j];
                if (!c.live) continue;
                if ((c.a == k || c.b == k) && c.op != Op::Fc) only_fc = false;
            }
            virt[k] = only_fc && dag.out != k;
        }
    }
    // which fc nodes use the bf16 MFMA kernels (32-bit buffer offsets must cover their tensors; a 1 x 1 image has no
    // 8-pixel units: the fp32 kernels take it)
    std::vector<bool> fc_mfma(n, false);
    for (int k = 1; k < n; k++)
        if (dag.nodes[k].live && dag.nodes[k].op == Op::Fc) fc_mfma[k] = mfma && !dag.nodes[k].pooled;

    // ---------------------------------------------------------------- units
    std::vector<std::vector<int>> consumers(n);
    for (int k = 1; k < n; k++) {
        const Node& nd = dag.nodes[k];
        if (!nd.live) continue;
        consumers[nd.a].push_back(k);
        if (nd.b >= 0 && nd.b != nd.a) consumers[nd.b].push_back(k);
    }
    std::vector<Unit> units;
    std::vector<int> unit_of(n, -1);
    auto outputs_of = [&](const std::vector<int>& nodes) {
        std::vector<bool> in(n, false), outp(n, false);
        for (int k : nodes) in[k] = true;
        for (int k : nodes) {
            if (k == dag.out) outp[k] = true;
            for (int c : consumers[k])
                if (!in[c]) outp[k] = true;
        }
        return outp;
    };
    const bool log = std::getenv("CANVAS_LOG") != nullptr;
    std::string why;
    auto chain_cost = [&](const std::vector<int>& nodes) {
        auto it = costs.find(nodes);
        if (it == costs.end()) {
            chain::UnitPlan plan;
            const bool compiles = chain::compile_unit(dag, nodes, outputs_of(nodes), false, plan, why);
            it = costs.insert({nodes, compiles ? std::make_pair(plan.cost, plan.halo_cost) : std::make_pair(-1.0, -1.0)}).first;
        }
        return halos ? it->second.second : it->second.first;
    };
    for (int k = 1; k < n; k++) {
        const Node& nd = dag.nodes[k];
        if (!nd.live || virt[k]) continue;
        bool placed = false;
        if (fuse_chains && chain::chain_candidate(dag, k)) {
            // the chains of the operands, latest first; joining chain u needs every operand inside u or produced before u runs
            std::vector<int> cands;
            for (int o : {nd.b, nd.a})
                if (o > 0 && unit_of[o] >= 0 && units[unit_of[o]].chain && std::find(cands.begin(), cands.end(), unit_of[o]) == cands.end())
                    cands.push_back(unit_of[o]);
            std::sort(cands.rbegin(), cands.rend());
            for (int u : cands) {
                bool ok = true;
                for (int o : {nd.a, nd.b})
                    if (o > 0 && !virt[o] && unit_of[o] != u && unit_of[o] > u) ok = false;
                if (!ok) continue;
                std::vector<int> grown = units[u].nodes;
                grown.push_back(k);
                if (chain_cost(grown) >= 0) {
                    units[u].nodes = grown;
                    unit_of[k] = u;
                    placed = true;
                    break;
                }
                if (log) std::fprintf(stderr, "canvas: node %d does not join chain %d: %s\n", k, u, why.c_str());
            }
            if (!placed) {
                std::vector<int> alone{k};
                if (chain_cost(alone) >= 0) {
                    Unit U;
                    U.chain = true;
                    U.nodes = alone;
                    units.push_back(U);
                    unit_of[k] = (int)units.size() - 1;
                    placed = true;
                } else if (log) {
                    std::fprintf(stderr, "canvas: node %d takes a kernel of its own: %s\n", k, why.c_str());
                }
            }
        }
        if (!placed) {
            Unit U;
            U.nodes = {k};
            units.push_back(U);
            unit_of[k] = (int)units.size() - 1;
        }
    }
    // Full recomputation makes a long chain dearer than its parts (every unary's adjoint evaluates its operand again,
    // every softmax over channels adds passes).  A grown chain is therefore cut in two, at the place that pays most,
    // while the halves together cost less than four fifths of the whole, and the halves are looked at again.  A cut
    // materialises what crosses it: across a tensor with taps (an unfolded tensor, which a chain otherwise never
    // writes) it is only made when the halves cost less than two fifths of the whole, which in practice means a
    // softmax over channels of an unfolded tensor, whose passes each recompute the whole window.
    for (size_t u = 0; u < units.size(); u++) {
        if (!units[u].chain || units[u].nodes.size() < 2) continue;
        const std::vector<int> nodes = units[u].nodes;
        const double whole = chain_cost(nodes);
        double best = whole;
        size_t cut = 0;
        for (size_t i = 1; i < nodes.size(); i++) {
            const std::vector<int> A(nodes.begin(), nodes.begin() + i), Bn(nodes.begin() + i, nodes.end());
            bool taps = false;
            for (int k : Bn)
                for (int o : {dag.nodes[k].a, dag.nodes[k].b})
                    if (o > 0 && std::find(A.begin(), A.end(), o) != A.end() && dag.nodes[o].T != 1) taps = true;
            const double ca = chain_cost(A), cb = ca < 0 ? -1 : chain_cost(Bn);
            if (cb < 0) continue;
            const double apart = (ca + cb) / (taps ? 0.4 : 0.8);  // (as if the whole had to be that much dearer)
            if (apart < best) {
                best = apart;
                cut = i;
            }
        }
        if (cut == 0) continue;
        if (log) std::fprintf(stderr, "canvas: chain %zu cut after %zu of %zu nodes: weighted cost %.0f apart, %.0f whole\n", u, cut, nodes.size(), best, whole);
        Unit B;
        B.chain = true;
        B.nodes.assign(nodes.begin() + cut, nodes.end());
        units[u].nodes.assign(nodes.begin(), nodes.begin() + cut);
        units.insert(units.begin() + u + 1, B);
        for (size_t v = 0; v < units.size(); v++)
            for (int k : units[v].nodes) unit_of[k] = (int)v;
        u--;  // (the first half again, then the second)
    }
    for (const Unit& U : units)
        if (U.chain) low->chains.push_back(U.nodes);
    if (unlike && unlike->chains == low->chains) return nullptr;
    // a unit was last compiled when it last grew, against the consumers known then; later nodes may have joined
    // other units, which never removes an output, but a later joiner of THIS unit may have: compile the final sets
    for (Unit& U : units)
        if (U.chain) {
            if (!chain::compile_unit(dag, U.nodes, outputs_of(U.nodes), true, U.plan, why)) throw std::runtime_error("chain unit no longer compiles: " + why);
            low->chain_units++;
            low->chain_nodes += (int)U.nodes.size();
            if (log) {
                std::string ids;
                for (int k : U.nodes) ids += " " + std::to_string(k);
                std::fprintf(stderr, "canvas: chain of %zu nodes [%s ] cost fwd %.1f bwd %.1f\n%s%s", U.nodes.size(), ids.c_str(),
                             chain::program_cost(U.plan.fwd), chain::program_cost(U.plan.bwd), chain::dump(U.plan.fwd).c_str(), chain::dump(U.plan.bwd).c_str());
            }
        }
    // materialised nodes: everything outside a chain, and the stored nodes of a chain
    std::vector<bool> mat(n, false);
    for (const Unit& U : units) {
        if (!U.chain) mat[U.nodes[0]] = true;
        else
            for (int o : U.plan.outputs) mat[o] = true;
    }
    // who can use the caller's tensors in place: chains, and FC nodes whose kernels have the caller's type
    auto fc_in_place = [&](int k) { return dag.nodes[k].op == Op::Fc && (fc_mfma[k] || !bf16); };
    auto in_place = [&](int k) { return k > 0 && unit_of[k] >= 0 && (units[unit_of[k]].chain || fc_in_place(k)); };
    // x: read in place by such units (FC nodes also through a virtual Unfold); a widened copy only for the others
    bool need_x32 = dag.out == 0;
    for (int c : consumers[0]) {
        if (virt[c]) continue;  // (its consumers are FC nodes that read x)
        if (!in_place(c)) need_x32 = true;
    }
    // y and dy: in place when the output node is produced by such a unit and nothing else reads it
    const bool y_direct = in_place(dag.out) && consumers[dag.out].empty();
    // dx: in place when exactly one unit writes the gradient of x and it can
    int x_writers = 0;
    bool x_writer_ok = true;
    {
        std::vector<int> seen;
        for (int c : consumers[0]) {
            if (virt[c]) {
                for (int f : consumers[c]) x_writers++, x_writer_ok = x_writer_ok && fc_in_place(f);
                continue;
            }
            const int u = unit_of[c];
            if (units[u].chain) {
                if (std::find(seen.begin(), seen.end(), u) != seen.end()) continue;
                seen.push_back(u);
            }
            x_writers++;
            x_writer_ok = x_writer_ok && in_place(c);
        }
    }
    const bool dx_direct = x_writers == 1 && x_writer_ok;
    for (int k = 0; k < n; k++) {
        if (!dag.nodes[k].live || virt[k]) continue;
        if (k == 0) {
            if (bf16 && need_x32) lay.val[0] = take(dag.numel(0));
            if (!dx_direct) lay.grad[0] = take(dag.numel(0));
            continue;
        }
        if (!mat[k]) continue;
        if (k == dag.out && y_direct) continue;  // value in y, gradient in dy
        lay.val[k] = take(dag.numel(k));
        lay.grad[k] = take(dag.numel(k));
    }
    std::vector<int64_t> wnumel(dag.n_weights);
    for (int i = 0; i < dag.n_weights; i++) {
        const Node& f = dag.nodes[dag.weight_node[i]];
        const Node& A = dag.nodes[f.a];
        wnumel[i] = (int64_t)f.out * (A.C / f.groups) * A.T;
    }
    // MFMA contraction parameters of fc node k (forward orientation); src pointer filled at run time
    auto fc_params = [&](int k) {
        const Node& f = dag.nodes[k];
        const bool v = virt[f.a];
        const Node& U = dag.nodes[f.a];
        const int srcn = v ? U.a : f.a;
        const Node& S = dag.nodes[srcn];
        gfc::Params Q = gfc::shape(dag.N, f.groups, (S.C / f.groups) * S.T, v ? U.kh : 1, v ? U.kw : 1, f.out / f.groups, dag.H, dag.W);
        return Q;
    };
    auto fc_src = [&](int k) { return virt[dag.nodes[k].a] ? dag.nodes[dag.nodes[k].a].a : dag.nodes[k].a; };

    // geometry of the weight-gradient launch of MFMA fc node k (operand types decide its tile shape)
    auto wgrad_params = [&](int k) {
        gfc::Params Q = fc_params(k);
        Q.src_f32 = fc_src(k) == 0 ? 0 : 1;
        Q.dy_f32 = (k == dag.out && y_direct) ? 0 : 1;
        gfc::prepare_wgrad(Q);
        return Q;
    };
    // the same for fc nodes on the fp32 kernels
    auto sfc_params = [&](int k) {
        const Node& f = dag.nodes[k];
        const bool v = virt[f.a];
        const Node& U = dag.nodes[f.a];
        const int srcn = fc_src(k);
        const Node& S = dag.nodes[srcn];
        return sfc::shape(dag.N, f.groups, (S.C / f.groups) * S.T, v ? U.kh : 1, v ? U.kw : 1, f.out / f.groups, dag.Hk(srcn), dag.Wk(srcn));
    };
    // Contractions whose operand is the caller's bf16 tensor take the tap-major kernels: forward where the FC reads x, the data
    // gradient where it reads dy (generic / tap-major kernels, us, forward + data gradient: 3x3, 2x48
    // planes of 40x40 36.0 + 40.6 / 8.3 + 8.2, 7x32 of 14x14 21.7 + 22.5 / 7 + 7, 32x128 of 14x14 93.6 + 94.9 / 10.8 + 10.7).  Not the
    // weight gradient: those kernels multiply what lies behind a plane's last pixel by zero, so that an infinity there spreads.
    // An fp32 tensor between units is cut into bf16 pairs first, hi = bf16(x) and lo = bf16(x - hi), and contracted as twice the rows
    // against the same weights: the values and products are those of the generic kernels, which cut every element again for every
    // output tile.  Where the contraction is long (us, generic kernels / cutting, packing the weights and contracting): 3x3, 96 -> 96
    // channels (K = 864) 16x96 planes of 32x32 91 / 32, 4x96 of 22x17 95 / 21, 96 -> 8 16x96 of 32x32 73 / 22; without a window, tensors of
    // nine taps (K = 864) 4x96 planes of 22x17 70 / 27, 16x96 of 32x32 (14 M elements) 64 / 46, of 25 taps (K = 2400) 4x96 of 22x17 201 / 55.
    // Not where what is cut without a window is longer: 39 M elements are 315 MB to move, and the whole contraction of two groups
    // of 96 outputs takes 90.
    enum { kTmFwd = 1, kTmData = 2, kTmFwdPairs = 4 };
    constexpr int kLongContraction = 512;
    constexpr int64_t kLongPairs = (int64_t)16 << 20;
    std::vector<int> tm(dag.n_weights, 0);
    uint64_t plain_bytes = 0, tm_bytes = 0;  // weight copies and partials without and with them
    uint64_t packed_bytes = 0;               // of the latter, what emit_fc and the cutting take when their launches are written
    for (int i = 0; i < dag.n_weights; i++) {
        const int k = dag.weight_node[i];
        if (!dag.nodes[k].live) continue;
        if (!fc_mfma[k]) {
            const uint64_t widened = bf16 ? align_up((uint64_t)wnumel[i] * 4) : 0;
            plain_bytes += widened;
            tm_bytes += widened;
            continue;
        }
        const bool from_x = fc_src(k) == 0, from_dy = k == dag.out && y_direct;
        const gfc::Params Q = fc_params(k), Wg = wgrad_params(k);
        const uint64_t wt = align_up((uint64_t)wnumel[i] * 2), part = align_up((uint64_t)gfc::wgrad_partials(Wg) * wnumel[i] * 4);
        plain_bytes += wt + part;
        // (groups that share a tile meet each other's infinities as 0 * inf: those keep the generic kernels)
        auto covers = [&](int R, int Og) {
            return gfctm::supported(Q.N, Q.G, R, Q.KH, Q.KW, Og, Q.H, Q.W) && gfctm::shape(Q.N, Q.G, R, Q.KH, Q.KW, Og, Q.H, Q.W).gm == 1;
        };
        // (forward without a window only where the weights are read as they are: packing them is one more launch)
        const bool as_they_are = Q.TV == 1 && Q.R % 16 == 0 && covers(Q.R, Q.Og) && gfctm::shape(Q.N, Q.G, Q.R, 1, 1, Q.Og, Q.H, Q.W).Omp == Q.Og;
        if (from_x && covers(Q.R, Q.Og) && (Q.TV > 1 || as_they_are)) {
            tm[i] |= kTmFwd;
            if (!as_they_are) packed_bytes += align_up(fc_packed_bytes(dag, Q.G, Q.R, Q.KH, Q.KW, Q.Og));
        }
        if (from_dy && covers(Q.Og, Q.R)) {
            tm[i] |= kTmData;
            packed_bytes += align_up(fc_packed_bytes(dag, Q.G, Q.Og, Q.KH, Q.KW, Q.R));
        }
        if (!from_x && Q.K >= kLongContraction && (Q.TV > 1 || dag.numel(fc_src(k)) <= kLongPairs) && covers(2 * Q.R, Q.Og)) {
            tm[i] |= kTmFwd | kTmFwdPairs;
            packed_bytes += align_up(fc_packed_bytes(dag, Q.G, 2 * Q.R, Q.KH, Q.KW, Q.Og)) + align_up((uint64_t)dag.numel(fc_src(k)) * 4);
        }
        tm_bytes += part;
        if (!(tm[i] & kTmData)) tm_bytes += wt;
    }
    // (a plan that fits the library's static workspace keeps fitting it)
    if (off + plain_bytes <= CANVAS_STATIC_WORKSPACE_BYTES && off + tm_bytes + packed_bytes > CANVAS_STATIC_WORKSPACE_BYTES) {
        tm.assign(dag.n_weights, 0);
        packed_bytes = 0;
    }
    const TakeFn take_bytes = [&off](uint64_t bytes) {
        const uint64_t o = off;
        off += align_up(bytes);
        return (int64_t)o;
    };
    // Packed weights and pairs get their place now: what follows shares out the rest of the static workspace.
    uint64_t packed_at = off;
    off += packed_bytes;
    const uint64_t packed_end = off;
    const TakeFn take_packed = [&packed_at, packed_end](uint64_t bytes) {
        const uint64_t o = packed_at;
        packed_at += align_up(bytes);
        if (packed_at > packed_end) throw std::runtime_error("internal: packed weights without a place");
        return (int64_t)o;
    };
    lay.wt.assign(dag.n_weights, -1);
    lay.part.assign(dag.n_weights, -1);
    std::vector<sfc::Params> sgrad(dag.n_weights);  // weight gradients of the fp32 fc nodes
    int sfc_count = 0;
    for (int i = 0; i < dag.n_weights; i++) {
        const int k = dag.weight_node[i];
        const Node& f = dag.nodes[k];
        if (!f.live) continue;
        if (!fc_mfma[k]) {
            if (bf16) lay.wf[i] = take(wnumel[i]);
            sfc_count++;
            continue;
        }
        if (!(tm[i] & kTmData)) lay.wt[i] = take_bytes((uint64_t)wnumel[i] * 2);
        const gfc::Params Q = wgrad_params(k);
        const int64_t slices = gfc::wgrad_partials(Q);
        lay.part[i] = take_bytes((uint64_t)slices * wnumel[i] * 4);
    }
    // fp32 contractions on the bf16 matrix units read their weights cut into parts, forward and transposed, from the workspace;
    // a plan that fits the library's static workspace without them keeps to the fp32 units if it would not with them.
    std::vector<sfc::Params> sfwd(dag.n_weights), sdata(dag.n_weights);
    std::vector<std::pair<int, int64_t>> wsplit[2];  // (weight, offset) of the split weights, forward and transposed
    for (int i = 0; i < dag.n_weights; i++) {
        const int k = dag.weight_node[i];
        if (!dag.nodes[k].live || fc_mfma[k]) continue;
        sfwd[i] = sfc_params(k);
        sdata[i] = sfc::data_gradient_of(sfwd[i]);
        // (both directions or neither: one launch cuts the weights for both, and costs what one direction gains at the least)
        sfc::prepare_forward(sfwd[i], !bf16);
        sfc::prepare_forward(sdata[i], !bf16);
        uint64_t bytes[2] = {0, 0};
        const bool both = sfwd[i].split && sdata[i].split;
        const int directions = inference ? 1 : 2;  // (the transposed weights: for the backward pass alone)
        if (both)
            for (int d = 0; d < directions; d++) bytes[d] = align_up((uint64_t)48 * sfc::split_job(d ? sdata[i] : sfwd[i]).items);
        if (!both || (off <= CANVAS_STATIC_WORKSPACE_BYTES && off + bytes[0] + bytes[1] > CANVAS_STATIC_WORKSPACE_BYTES)) {
            sfwd[i] = sfc_params(k);
            sdata[i] = sfc::data_gradient_of(sfwd[i]);
            sfc::prepare_forward(sfwd[i]);
            sfc::prepare_forward(sdata[i]);
            continue;
        }
        for (int d = 0; d < directions; d++) {
            wsplit[d].push_back({i, (int64_t)off});
            off += bytes[d];
        }
    }
    auto split_at = [&](int d, int widx) {
        for (const auto& s : wsplit[d])
            if (s.first == widx) return s.second;
        return (int64_t)-1;
    };
    // Partials of the fp32 weight gradients: at most 16 MB each, and never so much that a plan which fits the library's
    // static workspace without them no longer does (one slice writes dw itself and needs none).
    const int64_t room = off < CANVAS_STATIC_WORKSPACE_BYTES ? (int64_t)(CANVAS_STATIC_WORKSPACE_BYTES - off) / std::max(1, sfc_count) - 256 : kMaxSfcPartialBytes;
    for (int i = 0; i < dag.n_weights; i++) {
        const int k = dag.weight_node[i];
        if (!dag.nodes[k].live || fc_mfma[k]) continue;
        sgrad[i] = sfc_params(k);
        sfc::prepare_wgrad(sgrad[i], std::min(room, kMaxSfcPartialBytes));
        if (sgrad[i].slices > 1) lay.part[i] = take(wnumel[i] * sgrad[i].slices);
    }
    low->ws_bytes = std::max<uint64_t>(off, 256);  // (a caller always hands over a workspace, also to a plan that needs none)
    // An fp32 FC that is the whole DAG reads x and writes y, reads dy and writes dx in one launch each.  A call that passes
    // overlapping buffers for them (in place, say) writes to this end of the workspace first and copies.
    auto fc_alone = [&](int k) { return !bf16 && k == dag.out && y_direct && fc_src(k) == 0; };
    int64_t stage = -1;
    if (dag.out > 0 && dag.nodes[dag.out].op == Op::Fc && fc_alone(dag.out)) {
        const int64_t nx = dag.numel(0) * 4, ny = dag.numel(dag.out) * 4, nw = wnumel[dag.nodes[dag.out].widx] * 4;
        const int widx = dag.nodes[dag.out].widx;
        stage = (int64_t)low->ws_bytes;
        low->stage_bytes = align_up((uint64_t)std::max(nx, ny));
        low->ws_bytes += low->stage_bytes;
        low->fwd_staged = [=](const RunArgs& a) { return overlap(a.y, ny, a.x, nx) || overlap(a.y, ny, a.w[widx], nw); };
    }
    const double esz = bf16 ? 2.0 : 4.0;

    // pointer resolvers
    auto val = [lay](const RunArgs& a, int k) -> const float* {
        return lay.val[k] >= 0 ? (const float*)(a.ws + lay.val[k]) : (const float*)a.x;
    };
    auto valw = [lay](const RunArgs& a, int k) -> float* { return (float*)(a.ws + lay.val[k]); };
    auto grad = [lay](const RunArgs& a, int k) -> float* { return (float*)(a.ws + lay.grad[k]); };
    auto wptr = [lay, bf16](const RunArgs& a, int i) -> const float* {
        return bf16 ? (const float*)(a.ws + lay.wf[i]) : (const float*)a.w[i];
    };

    // ---------------------------------------------------------------- forward
    if (bf16) {
        int64_t ne = dag.numel(0);
        if (lay.val[0] >= 0) low->fwd.push_back({"widen_x", ne * 6.0, 0, [=](const RunArgs& a) { ref::widen_bf16(a.x, valw(a, 0), ne, a.stream); }});
        for (int i = 0; i < dag.n_weights; i++) {
            if (lay.wf[i] < 0) continue;  // MFMA fc nodes read the bf16 weights as they are
            int64_t nw = wnumel[i];
            int64_t o = lay.wf[i];
            low->fwd.push_back({"widen_w", nw * 6.0, 0, [=](const RunArgs& a) { ref::widen_bf16(a.w[i], (float*)(a.ws + o), nw, a.stream); }, true});
        }
    }
    // the split weights of forward and backward, several per launch (backward runs on the weights and the workspace of the
    // preceding forward)
    {
        std::vector<std::pair<sfc::SplitJob, std::pair<int, int64_t>>> all;
        for (int d = 0; d < 2; d++)
            for (const auto& s : wsplit[d]) all.push_back({sfc::split_job(d ? sdata[s.first] : sfwd[s.first]), s});
        for (size_t first = 0; first < all.size(); first += sfc::kMaxSplitJobs) {
            const auto part = std::vector<std::pair<sfc::SplitJob, std::pair<int, int64_t>>>(
                all.begin() + first, all.begin() + std::min(all.size(), first + (size_t)sfc::kMaxSplitJobs));
            double bytes = 0;
            for (const auto& j : part) bytes += 48.0 * j.first.items + 4.0 * wnumel[j.second.first];
            low->fwd.push_back({"weight_prep", bytes, 0, [part](const RunArgs& a) {
                                    sfc::SplitJobs J;
                                    for (const auto& j : part) {
                                        sfc::SplitJob& d = J.j[J.n++];
                                        d = j.first;
                                        d.w = (const float*)a.w[j.second.first];
                                        d.out = a.ws + j.second.second;
                                    }
                                    sfc::split_weights(J, a.stream);
                                }, true});
        }
    }
    // where an external tensor of a chain program lives
    auto bind = [&](const std::vector<chain::ExtRef>& ext) {
        std::vector<Binding> b(ext.size());
        for (size_t i = 0; i < ext.size(); i++) {
            const int e = ext[i].node;
            b[i].node = e;
            b[i].role = ext[i].role;
            switch (ext[i].role) {
            case chain::kValueIn:
                if (e == 0) b[i].where = 1;
                else b[i].off = lay.val[e];
                break;
            case chain::kValueOut:
                if (e == dag.out && y_direct) b[i].where = 2;
                else b[i].off = lay.val[e];
                break;
            case chain::kGradIn:
                if (e == dag.out && y_direct) b[i].where = 3;
                else b[i].off = lay.grad[e];
                break;
            case chain::kGradOut:
                if (e == 0 && dx_direct) b[i].where = 4;
                else b[i].off = lay.grad[e];
                break;
            }
            if (b[i].where == 0 && b[i].off < 0) throw std::runtime_error("chain: an external tensor without a buffer");
        }
        return b;
    };
    auto ext_bytes = [&](const std::vector<Binding>& b) {
        double t = 0;
        for (const Binding& e : b) t += (e.where == 0 ? 4.0 : esz) * dag.numel(e.node);
        return t;
    };
    auto bind_of = [](const std::vector<Binding>& b, chain::ExtRole role) {
        for (const Binding& e : b)
            if (e.role == role) return e;
        throw std::runtime_error("chain: a tensor of the unit is missing");
    };
    auto self_direct = [&](const Unit& U, ufc::MidParams& M) {
        return bf16 && y_direct && dx_direct && U.plan.inputs == std::vector<int>{0} && U.plan.outputs == std::vector<int>{dag.out} && self_blend(dag, U, M);
    };
    for (size_t ui = 0; ui < units.size(); ui++) {
        const Unit& U = units[ui];
        if (U.chain) {
            const chain::Program pg = U.plan.fwd;
            const std::vector<Binding> b = bind(U.plan.fwd_ext);
            smc::Params S;
            if (softmax_of_channels(dag, U, S)) {
                if (log) std::fprintf(stderr, "canvas: chain of node %d: the kernels of a softmax over channels\n", U.nodes[0]);
                low->est_us += ext_bytes(b) / 3e6;
                const Binding bx = bind_of(b, chain::kValueIn), by = bind_of(b, chain::kValueOut);
                low->fwd.push_back({"chain_fwd", ext_bytes(b), 0, [=](const RunArgs& a) {
                                        smc::Params Q = S;
                                        Q.x = bound(bx, a);
                                        Q.out = const_cast<void*>(bound(by, a));
                                        Q.x_f32 = !bf16 || bx.where == 0;
                                        Q.out_f32 = !bf16 || by.where == 0;
                                        Q.fast = bf16;
                                        smc::forward(Q, a.stream);
                                    }});
                continue;
            }
            ufc::MidParams M;
            if (self_direct(U, M)) {
                if (log) std::fprintf(stderr, "canvas: chain of node %d: the kernels of a tensor blended with itself\n", U.nodes[0]);
                low->est_us += ext_bytes(b) / 3e6;
                low->fwd.push_back({"chain_fwd", ext_bytes(b), 0, [=](const RunArgs& a) {
                                        ufc::MidParams Q = M;
                                        Q.x = Q.z = (const uint16_t*)a.x;
                                        Q.v = (uint16_t*)a.y;
                                        ufc::mid_forward(Q, a.stream);
                                    }});
                continue;
            }
            low->est_us += chain::launch_us(pg);
            low->fwd.push_back({"chain_fwd", ext_bytes(b), 0, [=](const RunArgs& a) { run_program(pg, b, bf16, a); }});
            continue;
        }
        const int k = U.nodes[0];
        const Node nd = dag.nodes[k];
        const Node A = dag.nodes[nd.a];
        Launch L;
        L.name = std::string("node_") + op_name(nd.op) + "_fwd";
        L.bytes = 4.0 * (dag.numel(nd.a) + dag.numel(k));
        switch (nd.op) {
        case Op::Unfold:
            L.run = [=](const RunArgs& a) { ref::unfold_fwd(val(a, nd.a), valw(a, k), N * A.C, A.T, nd.kh, nd.kw, dag.H, dag.W, a.stream); };
            break;
        case Op::Shift:
            L.run = [=](const RunArgs& a) {
                ref::shift(val(a, nd.a), valw(a, k), N, nd.C, nd.T, dag.H, dag.W, nd.dh, nd.dw, nd.c0, nd.c1, 0, a.stream);
            };
            break;
        case Op::Fc: {
            const int K = (A.C / nd.groups) * A.T;
            L.flops = 2.0 * N * dag.Pk(k) * nd.out * K;
            if (fc_mfma[k]) {
                gfc::Params Q = fc_params(k);
                const int srcn = fc_src(k);
                const bool src_x = srcn == 0;  // the caller's bf16 input is read directly
                const bool to_y = k == dag.out && y_direct;  // the output node: written as bf16 where the caller wants it
                if (tm[nd.widx] & kTmFwd) {
                    const int64_t pairs = tm[nd.widx] & kTmFwdPairs ? take_packed((uint64_t)dag.numel(srcn) * 4) : -1;
                    if (pairs >= 0) {
                        const int64_t ne = dag.numel(srcn), block = (int64_t)Q.R * Q.P;
                        low->fwd.push_back({"gfc_split", 8.0 * ne, 0, [=](const RunArgs& a) { ref::split_bf16(val(a, srcn), a.ws + pairs, ne, block, a.stream); }});
                    }
                    emit_fc(*low, false, dag, take_packed, Q.TV > 1 ? "gfc_fwd_unfold" : "gfc_fwd", Q.G, Q.R, Q.KH, Q.KW, Q.Og, false, nd.widx,
                            FcOperand{[=](const RunArgs& a) { return pairs >= 0 ? (const void*)(a.ws + pairs) : a.x; }, false, pairs >= 0},
                            [=](const RunArgs& a) { return to_y ? (const void*)a.y : (const void*)valw(a, k); }, false,
                            (pairs >= 0 ? 4.0 : 2.0) * dag.numel(srcn) + (to_y ? 2.0 : 4.0) * dag.numel(k) + 2.0 * wnumel[nd.widx], L.flops, !to_y, false, pairs < 0 && Q.TV == 1);
                    continue;
                }
                Q.src_f32 = src_x ? 0 : 1;
                Q.dst_f32 = to_y ? 0 : 1;
                gfc::prepare_forward(Q);
                L.name = Q.TV > 1 ? "gfc_fwd_unfold" : "gfc_fwd";
                L.bytes = (src_x ? 2.0 : 4.0) * dag.numel(srcn) + (to_y ? 2.0 : 4.0) * dag.numel(k) + 2.0 * wnumel[nd.widx];
                const int widx = nd.widx;
                L.run = [=](const RunArgs& a) {
                    gfc::Params R = Q;
                    R.src = src_x ? a.x : (const void*)val(a, srcn);
                    R.w = (const uint16_t*)a.w[widx];
                    R.dst = to_y ? a.y : (void*)valw(a, k);
                    gfc::forward(R, a.stream);
                };
                break;
            }
            const int srcn = fc_src(k), widx = nd.widx;
            const sfc::Params Q = sfwd[widx];
            const int64_t woff = split_at(0, widx);
            const bool to_y = k == dag.out && y_direct;
            const int64_t ny = dag.numel(k);
            const auto overlaps = stage >= 0 ? low->fwd_staged : [](const RunArgs&) { return false; };
            L.name = sfc_name("sfc_fwd", Q);
            L.bytes = 4.0 * (dag.numel(srcn) + dag.numel(k) + wnumel[widx]);
            L.run = [=](const RunArgs& a) {
                sfc::Params R = Q;
                R.src = val(a, srcn);
                R.w = wptr(a, widx);
                R.wsplit = a.ws + woff;
                R.dst = to_y ? (float*)a.y : valw(a, k);
                const bool staged = overlaps(a);
                if (staged) R.dst = (float*)(a.ws + stage);
                sfc::forward(R, a.stream);
                if (staged) ref::copy_f32(R.dst, (float*)a.y, ny, a.stream);
            };
            break;
        }
        case Op::Unary: {
            int64_t ne = dag.numel(k);
            L.run = [=](const RunArgs& a) { ref::unary_fwd(val(a, nd.a), valw(a, k), ne, nd.kind, nd.lo, nd.hi, a.stream); };
            break;
        }
        case Op::Binary: {
            const Node B = dag.nodes[nd.b];
            L.bytes = 4.0 * (dag.numel(nd.a) + dag.numel(nd.b) + dag.numel(k));
            const int Pn = dag.Pk(k), PL = dag.Pk(nd.a);
            // a common Group dim: (image, group) pairs are independent, each blends [CL/G, TL] onto [CR/G, TR]
            const int Gb = nd.bgroups;
            // lhs=pixels: the [H*W, 1, 1, 1] LHS is a one-channel full-size tensor to the kernel
            const int CLk = nd.lhs_pixels ? 1 : A.C / Gb, TLk = nd.lhs_pixels ? 1 : A.T, PLk = nd.lhs_pixels ? Pn : PL;
            // an LHS that has folded away one spatial dim the result still has is replicated along it
            const int lost = A.pooled & ~nd.pooled, Wd = dag.Wk(k);
            const int rep = nd.lhs_pixels || lost == 3 || lost == 0 ? 0 : lost;
            L.run = [=](const RunArgs& a) {
                ref::binary_fwd(val(a, nd.a), val(a, nd.b), valw(a, k), N * Gb, CLk, TLk, B.C / Gb, B.T, Pn, PLk, rep, Wd, nd.kind, a.stream);
            };
            break;
        }
        case Op::Group: {  // (live only as the output: a copy of the viewed tensor)
            int64_t ne = dag.numel(k);
            L.run = [=](const RunArgs& a) { ref::copy_f32(val(a, nd.a), valw(a, k), ne, a.stream); };
            break;
        }
        case Op::Softmax:
            {
                const int Pn = dag.Pk(k);
                if (nd.kind >= kAxisH) {  // rows of every (image, channel, tap) plane: along W or the whole plane contiguous, along H strided by W
                    const int Hn = dag.Hk(k), Wn = dag.Wk(k);
                    const int len = nd.kind == kAxisH ? Hn : (nd.kind == kAxisW ? Wn : Hn * Wn), inner = nd.kind == kAxisH ? Wn : 1;
                    const int64_t rows = (int64_t)N * nd.C * nd.T * Pn / len;
                    L.run = [=](const RunArgs& a) { ref::softmax_rows_fwd(val(a, nd.a), valw(a, k), rows, len, inner, a.stream); };
                    break;
                }
                L.run = [=](const RunArgs& a) { ref::softmax_fwd(val(a, nd.a), valw(a, k), N, nd.C, nd.T, Pn, nd.kind == kAxisCT ? 2 : (nd.kind == kAxisC ? 1 : 0), a.stream); };
            }
            break;
        case Op::Fold:
            if (nd.axis_c) {
                const int64_t TP = (int64_t)A.T * dag.Pk(nd.a);
                const int Cg = A.C / nd.groups;
                L.name = "node_cfold_fwd";
                L.run = [=](const RunArgs& a) { ref::cfold_fwd(val(a, nd.a), valw(a, k), N * nd.groups, Cg, TP, nd.kind, a.stream); };
            } else if (nd.axis_hw == 1) {
                // over H alone: the H rows of a plane are "channels" of Wi elements each to the channel-fold kernel
                const int Hi = dag.Hk(nd.a), Wi = dag.Wk(nd.a);
                L.name = "node_hfold_fwd";
                L.run = [=](const RunArgs& a) { ref::cfold_fwd(val(a, nd.a), valw(a, k), N * A.C * A.T, Hi, Wi, nd.kind, a.stream); };
            } else if (nd.axis_hw) {
                // over W alone: every image row is a plane of Wi pixels; over both: every (channel, tap) plane
                const int Hi = dag.Hk(nd.a), Wi = dag.Wk(nd.a);
                const int64_t rows = N * A.C * A.T * (nd.axis_hw == 2 ? Hi : 1);
                const int len = nd.axis_hw == 2 ? Wi : Hi * Wi;
                L.name = "node_pool_fwd";
                L.run = [=](const RunArgs& a) { ref::pool_fwd(val(a, nd.a), valw(a, k), rows, len, nd.kind, a.stream); };
            } else {
                const int Pn = dag.Pk(k);
                L.run = [=](const RunArgs& a) { ref::fold_fwd(val(a, nd.a), valw(a, k), N * A.C, A.T, Pn, nd.kind, a.stream); };
            }
            break;
        default: break;
        }
        low->fwd.push_back(std::move(L));
    }
    if (!y_direct) {
        int64_t ne = dag.numel(dag.out);
        int o = dag.out;
        if (bf16) low->fwd.push_back({"narrow_y", ne * 6.0, 0, [=](const RunArgs& a) { ref::narrow_bf16(val(a, o), a.y, ne, a.stream); }});
        else low->fwd.push_back({"copy_y", ne * 8.0, 0, [=](const RunArgs& a) { ref::copy_f32(val(a, o), (float*)a.y, ne, a.stream); }});
    }

    // --------------------------------------------------------------- backward
    std::vector<bool> written(n, false);
    if (!y_direct) {
        int64_t ne = dag.numel(dag.out);
        int o = dag.out;
        if (bf16) low->bwd.push_back({"widen_dy", ne * 6.0, 0, [=](const RunArgs& a) { ref::widen_bf16(a.dy, grad(a, o), ne, a.stream); }});
        else low->bwd.push_back({"copy_dy", ne * 8.0, 0, [=](const RunArgs& a) { ref::copy_f32((const float*)a.dy, grad(a, o), ne, a.stream); }});
        written[o] = true;
    }
    for (int ui = (int)units.size() - 1; ui >= 0; ui--) {
        const Unit& U = units[ui];
        if (U.chain) {
            chain::Program pg = U.plan.bwd;
            const std::vector<Binding> b = bind(U.plan.bwd_ext);
            bool adds = false;
            for (size_t i = 0; i < b.size(); i++)
                if (b[i].role == chain::kGradOut) {
                    adds = written[b[i].node];
                    // the first writer of a gradient overwrites, later ones add (fp32 buffers only)
                    if (written[b[i].node]) pg.ins[U.plan.bwd_ext[i].store_instr].kind |= chain::kStAdd;
                    written[b[i].node] = true;
                }
            smc::Params S;
            if (softmax_of_channels(dag, U, S)) {
                if (!inference) low->est_us += ext_bytes(b) / 3e6;
                const Binding bx = bind_of(b, chain::kValueIn), bg = bind_of(b, chain::kGradIn), bd = bind_of(b, chain::kGradOut);
                low->bwd.push_back({"chain_bwd", ext_bytes(b), 0, [=](const RunArgs& a) {
                                        smc::Params Q = S;
                                        Q.x = bound(bx, a);
                                        Q.dy = bound(bg, a);
                                        Q.out = const_cast<void*>(bound(bd, a));
                                        Q.x_f32 = !bf16 || bx.where == 0;
                                        Q.dy_f32 = !bf16 || bg.where == 0;
                                        Q.out_f32 = !bf16 || bd.where == 0;
                                        Q.acc = adds;
                                        Q.fast = bf16;
                                        smc::backward(Q, a.stream);
                                    }});
                continue;
            }
            ufc::MidParams M;
            if (self_direct(U, M)) {
                if (!inference) low->est_us += ext_bytes(b) / 3e6;
                low->bwd.push_back({"chain_bwd", ext_bytes(b), 0, [=](const RunArgs& a) {
                                        ufc::MidParams Q = M;
                                        Q.x = (const uint16_t*)a.x;
                                        Q.dv = (const uint16_t*)a.dy;
                                        Q.dx1 = (uint16_t*)a.dx;
                                        ufc::self_backward(Q, a.stream);
                                    }});
                continue;
            }
            if (!inference) low->est_us += chain::launch_us(pg);
            low->bwd.push_back({"chain_bwd", ext_bytes(b), 0, [=](const RunArgs& a) { run_program(pg, b, bf16, a); }});
            continue;
        }
        const int k = U.nodes[0];
        const Node nd = dag.nodes[k];
        const Node A = dag.nodes[nd.a];
        if (nd.op == Op::Fc && fc_mfma[k]) {
            const int srcn = fc_src(k), widx = nd.widx;
            const bool src_x = srcn == 0;
            const bool from_dy = k == dag.out && y_direct;   // the output node: its gradient is the caller's dy
            const bool to_dx = src_x && dx_direct;           // the only writer of dx: written in place, in bf16
            const int acc_s = written[srcn] ? 1 : 0;
            const double flops = 2.0 * N * P * nd.out * (double)(wnumel[widx] / nd.out);
            // weight gradient: partial sums over slices of the (image, pixel) range, then a fixed-order sum
            const gfc::Params Q = wgrad_params(k);
            const int64_t nw = wnumel[widx];
            const int64_t poff = lay.part[widx];
            const int slices = gfc::wgrad_partials(Q);
            low->bwd.push_back({Q.TV > 1 ? "gfc_wgrad_unfold" : "gfc_wgrad", (src_x ? 2.0 : 4.0) * dag.numel(srcn) + 4.0 * dag.numel(k) + 4.0 * slices * nw, flops,
                                [=](const RunArgs& a) {
                                    gfc::Params R = Q;
                                    R.src = src_x ? a.x : (const void*)val(a, srcn);
                                    R.dy = from_dy ? a.dy : (const void*)grad(a, k);
                                    R.partial = (float*)(a.ws + poff);
                                    gfc::wgrad_partial(R, a.stream);
                                }});
            ReduceJob rj;  // (one launch at the end of the backward pass sums the partials of every FC)
            rj.job.slices = slices;
            rj.job.kind = 0;
            rj.job.count = (unsigned)nw;
            wreduce::plan(rj.job);
            rj.widx = widx;
            rj.off = poff;
            rj.bytes = 4.0 * (slices + 1) * nw;
            low->rjobs.push_back(rj);
            // data gradient: the same contraction on dy with transposed, tap-flipped weights; it writes the
            // gradient of the FC's source tensor directly (the Unfold adjoint is part of it)
            gfc::Params D = gfc::data_gradient_of(Q);
            const int Rrows = Q.R, Og = Q.Og;
            D.src_f32 = from_dy ? 0 : 1;
            D.dst_f32 = to_dx ? 0 : 1;
            D.acc = to_dx ? 0 : acc_s;
            const int G = nd.groups, TV = D.TV;
            const double dgrad_bytes = (from_dy ? 2.0 : 4.0) * dag.numel(k) + (to_dx ? 2.0 : 4.0 * (1 + acc_s)) * dag.numel(srcn) + 2.0 * nw;
            if (tm[widx] & kTmData) {  // (the output's gradient is the first of the backward pass: there is nothing to add to yet)
                if (D.acc) throw std::runtime_error("internal: a gradient before the output's");
                emit_fc(*low, true, dag, take_packed, TV > 1 ? "gfc_dgrad_unfold" : "gfc_dgrad", G, Og, Q.KH, Q.KW, Rrows, true, widx,
                        FcOperand{[](const RunArgs& a) { return a.dy; }, false},
                        [=](const RunArgs& a) { return to_dx ? (const void*)a.dx : (const void*)grad(a, srcn); }, false, dgrad_bytes, flops, !to_dx);
                const WeightJob job = low->wjobs.back();  // (packed in the backward pass, where they are needed)
                low->wjobs.pop_back();
                low->bwd.insert(low->bwd.end() - 1, {"gfc_transpose_w", job.bytes, 0, [=](const RunArgs& a) {
                                                         wprep::Jobs J;
                                                         J.n = 1;
                                                         J.j[0] = job.job;
                                                         J.j[0].w = (const uint16_t*)a.w[widx];
                                                         J.j[0].out = (uint16_t*)(a.ws + job.off);
                                                         wprep::run(J, a.stream);
                                                     }});
                written[srcn] = true;
                continue;
            }
            const int64_t toff = lay.wt[widx];
            low->bwd.push_back({"gfc_transpose_w", 4.0 * nw, 0, [=](const RunArgs& a) {
                                    gfc::transpose_weights((const uint16_t*)a.w[widx], (uint16_t*)(a.ws + toff), G, Og, Rrows, TV, a.stream);
                                }});
            low->bwd.push_back({TV > 1 ? "gfc_dgrad_unfold" : "gfc_dgrad", dgrad_bytes, flops,
                                [=](const RunArgs& a) {
                                    gfc::Params R = D;
                                    R.src = from_dy ? a.dy : (const void*)grad(a, k);
                                    R.w = (const uint16_t*)(a.ws + toff);
                                    R.dst = to_dx ? a.dx : (void*)grad(a, srcn);
                                    gfc::forward(R, a.stream);
                                }});
            written[srcn] = true;
            continue;
        }
        if (nd.op == Op::Fc) {
            const int srcn = fc_src(k), widx = nd.widx;
            const bool from_dy = k == dag.out && y_direct, to_dx = srcn == 0 && dx_direct;
            const int acc_s = !to_dx && written[srcn] ? 1 : 0;
            const int64_t nw = wnumel[widx], poff = lay.part[widx];
            const double flops = 2.0 * N * dag.Pk(k) * (double)nw;
            const sfc::Params Q = sgrad[widx];
            low->bwd.push_back({sfc_name("sfc_wgrad", Q), 4.0 * (dag.numel(srcn) + dag.numel(k) + (double)Q.slices * nw), flops,
                                [=](const RunArgs& a) {
                                    sfc::Params R = Q;
                                    R.src = val(a, srcn);
                                    R.dy = from_dy ? (const float*)a.dy : grad(a, k);
                                    R.partial = poff >= 0 ? (float*)(a.ws + poff) : (float*)a.dw[widx];
                                    sfc::wgrad_partial(R, a.stream);
                                }});
            if (poff >= 0) {
                ReduceJob rj;
                rj.job.slices = Q.slices;
                rj.job.kind = 0;
                rj.job.count = (unsigned)nw;
                wreduce::plan(rj.job);
                rj.widx = widx;
                rj.off = poff;
                rj.bytes = 4.0 * (Q.slices + 1) * nw;
                low->rjobs.push_back(rj);
            }
            sfc::Params D = sdata[widx];
            D.acc = acc_s;
            const int64_t woff = split_at(1, widx);
            const int64_t nx = dag.numel(0), ny = dag.numel(k);
            low->bwd.push_back({sfc_name("sfc_dgrad", D), 4.0 * (dag.numel(k) + dag.numel(srcn) * (1 + acc_s) + nw), flops,
                                [=](const RunArgs& a) {
                                    sfc::Params R = D;
                                    R.src = from_dy ? (const float*)a.dy : grad(a, k);
                                    R.w = wptr(a, widx);
                                    R.wsplit = a.ws + woff;
                                    R.dst = to_dx ? (float*)a.dx : grad(a, srcn);
                                    const bool staged = stage >= 0 && (overlap(a.dx, nx * 4, a.dy, ny * 4) || overlap(a.dx, nx * 4, a.w[widx], nw * 4));
                                    if (staged) R.dst = (float*)(a.ws + stage);
                                    sfc::forward(R, a.stream);
                                    if (staged) ref::copy_f32(R.dst, (float*)a.dx, nx, a.stream);
                                }});
            written[srcn] = true;
            continue;
        }
        const int acc = written[nd.a] ? 1 : 0;
        Launch L;
        L.name = std::string("node_") + op_name(nd.op) + "_bwd";
        L.bytes = 4.0 * (dag.numel(nd.a) * (1 + acc) + dag.numel(k));
        switch (nd.op) {
        case Op::Unfold:
            L.run = [=](const RunArgs& a) { ref::unfold_bwd(grad(a, k), grad(a, nd.a), N * A.C, A.T, nd.kh, nd.kw, dag.H, dag.W, acc, a.stream); };
            break;
        case Op::Shift:
            L.run = [=](const RunArgs& a) {
                ref::shift(grad(a, k), grad(a, nd.a), N, nd.C, nd.T, dag.H, dag.W, -nd.dh, -nd.dw, nd.c0, nd.c1, acc, a.stream);
            };
            break;
        case Op::Unary: {
            int64_t ne = dag.numel(k);
            L.bytes += 4.0 * ne;
            L.run = [=](const RunArgs& a) { ref::unary_bwd(val(a, nd.a), grad(a, k), grad(a, nd.a), ne, nd.kind, nd.lo, nd.hi, acc, a.stream); };
            break;
        }
        case Op::Binary: {
            const Node B = dag.nodes[nd.b];
            // LHS first, then RHS (which may be the same tensor and then accumulates)
            L.name = "node_binary_bwd_lhs";
            L.bytes = 4.0 * (dag.numel(nd.a) * (1 + acc) + dag.numel(k) * (nd.kind == kAdd || nd.kind == kSub ? 1 : 2));
            const int Pn = dag.Pk(k), PL = dag.Pk(nd.a), Gb = nd.bgroups;
            const int CLk = nd.lhs_pixels ? 1 : A.C / Gb, TLk = nd.lhs_pixels ? 1 : A.T, PLk = nd.lhs_pixels ? Pn : PL;
            const int lost = A.pooled & ~nd.pooled, Wd = dag.Wk(k);
            const int rep = nd.lhs_pixels || lost == 3 || lost == 0 ? 0 : lost;
            L.run = [=](const RunArgs& a) {
                ref::binary_bwd_lhs(val(a, nd.a), val(a, nd.b), grad(a, k), grad(a, nd.a), N * Gb, CLk, TLk, B.C / Gb, B.T, Pn, PLk, rep, Wd, nd.kind, acc, a.stream);
            };
            low->bwd.push_back(std::move(L));
            written[nd.a] = true;
            const int acc_r = written[nd.b] ? 1 : 0;
            Launch R;
            R.name = "node_binary_bwd_rhs";
            R.bytes = 4.0 * (dag.numel(nd.b) * (1 + acc_r) + dag.numel(k) + (nd.kind == kAdd || nd.kind == kSub ? 0 : dag.numel(nd.a)));
            R.run = [=](const RunArgs& a) {
                ref::binary_bwd_rhs(val(a, nd.a), val(a, nd.b), grad(a, k), grad(a, nd.b), N * Gb, CLk, TLk, B.C / Gb, B.T, Pn, PLk, rep, Wd, nd.kind, acc_r, a.stream);
            };
            low->bwd.push_back(std::move(R));
            written[nd.b] = true;
            continue;
        }
        case Op::Group: {  // a shift by nothing: copies, or adds to, the gradient of the viewed tensor
            const int Pn = dag.Pk(k);
            L.run = [=](const RunArgs& a) { ref::shift(grad(a, k), grad(a, nd.a), N, nd.C, nd.T, 1, Pn, 0, 0, 0, 0, acc, a.stream); };
            break;
        }
        case Op::Softmax:
            L.bytes += 4.0 * dag.numel(k);
            {
                const int Pn = dag.Pk(k);
                if (nd.kind >= kAxisH) {
                    const int Hn = dag.Hk(k), Wn = dag.Wk(k);
                    const int len = nd.kind == kAxisH ? Hn : (nd.kind == kAxisW ? Wn : Hn * Wn), inner = nd.kind == kAxisH ? Wn : 1;
                    const int64_t rows = (int64_t)N * nd.C * nd.T * Pn / len;
                    L.run = [=](const RunArgs& a) { ref::softmax_rows_bwd(val(a, k), grad(a, k), grad(a, nd.a), rows, len, inner, acc, a.stream); };
                    break;
                }
                L.run = [=](const RunArgs& a) { ref::softmax_bwd(val(a, k), grad(a, k), grad(a, nd.a), N, nd.C, nd.T, Pn, nd.kind == kAxisCT ? 2 : (nd.kind == kAxisC ? 1 : 0), acc, a.stream); };
            }
            break;
        case Op::Fold:
            L.bytes += 4.0 * dag.numel(nd.a);
            if (nd.axis_c) {
                const int64_t TP = (int64_t)A.T * dag.Pk(nd.a);
                const int Cg = A.C / nd.groups;
                L.name = "node_cfold_bwd";
                L.run = [=](const RunArgs& a) { ref::cfold_bwd(val(a, nd.a), grad(a, k), grad(a, nd.a), N * nd.groups, Cg, TP, nd.kind, acc, a.stream); };
            } else if (nd.axis_hw == 1) {
                const int Hi = dag.Hk(nd.a), Wi = dag.Wk(nd.a);
                L.name = "node_hfold_bwd";
                L.run = [=](const RunArgs& a) { ref::cfold_bwd(val(a, nd.a), grad(a, k), grad(a, nd.a), N * A.C * A.T, Hi, Wi, nd.kind, acc, a.stream); };
            } else if (nd.axis_hw) {
                const int Hi = dag.Hk(nd.a), Wi = dag.Wk(nd.a);
                const int64_t rows = N * A.C * A.T * (nd.axis_hw == 2 ? Hi : 1);
                const int len = nd.axis_hw == 2 ? Wi : Hi * Wi;
                L.name = "node_pool_bwd";
                L.run = [=](const RunArgs& a) { ref::pool_bwd(val(a, nd.a), grad(a, k), grad(a, nd.a), rows, len, nd.kind, acc, a.stream); };
            } else {
                const int Pn = dag.Pk(k);
                L.run = [=](const RunArgs& a) { ref::fold_bwd(val(a, nd.a), grad(a, k), grad(a, nd.a), N * A.C, A.T, Pn, nd.kind, acc, a.stream); };
            }
            break;
        default: break;
        }
        low->bwd.push_back(std::move(L));
        written[nd.a] = true;
    }
    for (int i = 0; i < dag.n_weights; i++) {
        if (dag.nodes[dag.weight_node[i]].live) continue;
        int64_t nw = wnumel[i];  // an fc the output does not depend on has a zero weight gradient
        low->bwd.push_back({"zero_dw", nw * 4.0, 0, [=](const RunArgs& a) { ref::fill_f32((float*)a.dw[i], 0.f, nw, a.stream); }});
    }
    if (!dx_direct) {
        int64_t ne = dag.numel(0);
        if (bf16) low->bwd.push_back({"narrow_dx", ne * 6.0, 0, [=](const RunArgs& a) { ref::narrow_bf16(grad(a, 0), a.dx, ne, a.stream); }});
        else low->bwd.push_back({"copy_dx", ne * 8.0, 0, [=](const RunArgs& a) { ref::copy_f32(grad(a, 0), (float*)a.dx, ne, a.stream); }});
    }
    (void)esz;
    low->est_us += 5.0 * (double)(low->fwd.size() + (inference ? 0 : low->bwd.size()));  // (about what an empty launch and the gap behind it take)
    return low;
}

// Planes that a workgroup holds whole need no halo, which makes every part of a chain cheaper, but not alike: the search then cuts some chains that it
// keeps whole by the costs with halos, and keeps some that it cuts.  Neither is always the better one, so both are written where they
// differ, and the estimated times of their launches decide: the one with whole planes where it is 5 % shorter.  (760 plans of 46 random
// micro-DAGs that differ, time over that of the better one, geometric mean: by halos 1.044, by whole planes 1.305, by this
// rule 1.003.  16x96 planes of 27x15, |x|, product with a 5x5 window, avg: 213 / 239 us; 7x96 of 19x25, softmax, relu, max over 5x5, product: 212 / 143.)
// Except that a plan which fits the library's static workspace either way fits it.
std::unique_ptr<Lowering> lower_per_node(const Dag& dag, bool bf16, bool fuse_chains, bool inference) {
    ChainCosts costs;
    std::unique_ptr<Lowering> a = lower_by(dag, bf16, fuse_chains, inference, true, costs, nullptr);
    if (!fuse_chains) return a;
    std::unique_ptr<Lowering> b = lower_by(dag, bf16, fuse_chains, inference, false, costs, a.get());
    if (!b) return a;
    auto fits = [](const Lowering& l) { return l.ws_bytes - l.stage_bytes <= CANVAS_STATIC_WORKSPACE_BYTES; };
    if (fits(*a) != fits(*b)) return fits(*a) ? std::move(a) : std::move(b);
    return b->est_us * 1.05 < a->est_us ? std::move(b) : std::move(a);
}

}  // namespace canvas
