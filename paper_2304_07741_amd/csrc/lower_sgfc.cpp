// Pattern match and lowering for  x -> Shift* -> grouped FC -> unary{0..2} -> (binary add with x) -> output.
#include <algorithm>
#include <cstdlib>
#include <vector>

#include "lowering.hpp"
#include "sgfc_kernels.hpp"

namespace canvas {

std::unique_ptr<Lowering> lower_sgfc(const Dag& dag, bool bf16) {
    if (!bf16) return nullptr;
    const int n = (int)dag.nodes.size();
    for (int k = 0; k < n; k++)
        if (!dag.nodes[k].live || dag.nodes[k].pooled) return nullptr;  // (no tensor with folded spatial dims in this pattern)
    int k = 1, prev = 0;
    // shifts
    std::vector<int> sdh(dag.nodes[0].C, 0), sdw(dag.nodes[0].C, 0);
    std::vector<bool> shifted(dag.nodes[0].C, false);
    while (k < n && dag.nodes[k].op == Op::Shift) {
        const Node& s = dag.nodes[k];
        if (s.a != prev || s.T != 1) return nullptr;
        if (s.dh != 0 || s.dw != 0)
            for (int c = s.c0; c < s.c1; c++) {
                if (shifted[c]) return nullptr;  // two shifts with zero fill do not compose into one
                shifted[c] = true;
                sdh[c] = s.dh;
                sdw[c] = s.dw;
            }
        prev = k++;
    }
    if (k >= n || dag.nodes[k].op != Op::Fc || dag.nodes[k].a != prev) return nullptr;
    const Node fc = dag.nodes[k];
    const int C = dag.nodes[0].C, G = fc.groups, CG = C / G, OG = fc.out / G;
    if (dag.nodes[fc.a].T != 1 || CG % 16 || OG % 16 || !sgfc::supported(CG / 16, OG / 16) || G > sgfc::kMaxGroups) return nullptr;
    prev = k++;
    sgfc::Params P;
    if (k < n && dag.nodes[k].op == Op::Unary) {
        const Node& u = dag.nodes[k];
        if (u.a != prev || u.kind > kExpClip) return nullptr;  // the kernels are instantiated for relu, abs, gelu, expclip
        P.act = u.kind;
        P.ulo = u.lo;
        P.uhi = u.hi;
        prev = k++;
    }
    if (k < n && dag.nodes[k].op == Op::Binary) {
        const Node& b = dag.nodes[k];
        bool with_input = (b.a == 0 && b.b == prev) || (b.a == prev && b.b == 0);
        if (!with_input || b.kind != kAdd || fc.out != C) return nullptr;
        P.residual = 1;
        prev = k++;
    }
    if (k != n || dag.out != prev) return nullptr;
    // every FC group must see one shift
    for (int g = 0; g < G; g++) {
        for (int c = g * CG; c < (g + 1) * CG; c++)
            if (sdh[c] != sdh[g * CG] || sdw[c] != sdw[g * CG]) return nullptr;
        P.dh[g] = sdh[g * CG];
        P.dw[g] = sdw[g * CG];
    }
    const int Pn = dag.P();
    if (dag.W < 2 || (int64_t)Pn * dag.W >= ((int64_t)1 << 31)) return nullptr;
    // tensors are addressed with 32-bit byte offsets through buffer descriptors
    if ((int64_t)dag.N * std::max(C, fc.out) * Pn * 2 >= ((int64_t)1 << 31) || dag.N > 65535) return nullptr;
    if ((int64_t)dag.N * ((Pn + 127) / 128) * ((Pn + 127) / 128) >= ((int64_t)1 << 31)) return nullptr;
    // the input may only feed the first node of the chain and the residual
    for (int j = 2; j < n; j++) {
        const Node& nd = dag.nodes[j];
        bool is_res = P.residual && j == n - 1;
        if (!is_res && (nd.a == 0 || nd.b == 0)) return nullptr;
    }

    P.N = dag.N;
    P.C = C;
    P.H = dag.H;
    P.W = dag.W;
    P.P = Pn;
    P.G = G;
    P.magicW = (uint32_t)((((uint64_t)1 << 32) + dag.W - 1) / dag.W);
    P.chunks = (Pn + 127) / 128;
    P.magicChunks = (uint32_t)((((uint64_t)1 << 32) + P.chunks - 1) / P.chunks);
    P.total_tiles = (long long)dag.N * G * P.chunks;
    // Tiles per wavefront of the backward kernels: two share a wavefront's weights and its partial, but come one after the other.
    // Backward with one / two, us, by the tiles of the launch, 56x56: 64 channels 2000 6.7 / 8.0, 4100 10.7 / 12.9, 5100 13.8 / 14.6,
    // 5600 15.3 / 14.6, 6400 16.7 / 16.8, 7200 17.7 / 17.6, 8200 19.3 / 20.6; 128 channels 2000 10.5 / 12.8, 5100 25.4 / 26.9, 6400 30.3 / 32.4,
    // 8200 38.2 / 38.6; blocks 64 => 128 2000 9.0 / 12.5, 3100 14.7 / 15.0, 5100 20.9 / 23.2, 6400 26.1 / 26.1, 128 => 64 2000 9.8 / 12.6, 5100 19.9 / 19.7,
    // 6400 24.3 / 26.5; 55x55 4900 18.8 / 20.2, 6144 20.0 / 22.7.  One is faster or level by less than 5 % up to the line; beyond it
    // the kernel alone would take one as well, within 6 % (on ragged planes 20), but a partial per workgroup then is 1 KB for every four tiles of a
    // group, which two tiles halve: at most 1.6 MB below the line (6.3 with groups of 32), and above it what the reduction reads and the workspace holds grow with the
    // batch (4096x64 planes of 56x56: 52 MB with two, within the 64 MB of the static workspace).
    int tpw = P.total_tiles > 6144 ? 2 : 1;
    if (const char* e = std::getenv("CANVAS_SGFC_TPW")) tpw = std::max(1, std::atoi(e));
    P.tiles_per_wave = tpw;
    const int tiles_per_group = dag.N * P.chunks;
    P.wgs_per_group = (tiles_per_group + 4 * tpw - 1) / (4 * tpw);

    auto low = std::make_unique<Lowering>();
    low->fused = Pn % 8 == 0 && dag.W >= 8;  // (what the query has always reported; `family` says it for every plane)
    low->family = CANVAS_FAMILY_SHIFT_FC;
    low->strided_io = true;
    const int elems = OG * CG;
    low->ws_bytes = align_up((uint64_t)G * P.wgs_per_group * elems * 4);
    const int KC = CG / 16, MO = OG / 16;
    const int widx = fc.widx;
    const int xs_dense = C * Pn, ys_dense = fc.out * Pn;
    const double act = 2.0 * dag.numel(0), wb = 2.0 * G * elems;
    const double flops = 2.0 * dag.N * Pn * fc.out * CG;
    low->fwd.push_back({"sgfc_fwd", act + 2.0 * dag.numel(dag.out) + wb, flops, [=](const RunArgs& a) {
                            sgfc::Params Q = P;
                            Q.xs = a.x_stride ? (int)a.x_stride : xs_dense;
                            Q.ys = a.y_stride ? (int)a.y_stride : ys_dense;
                            Q.x = (const uint16_t*)a.x;
                            Q.w = (const uint16_t*)a.w[widx];
                            Q.y = (uint16_t*)a.y;
                            sgfc::forward(Q, KC, MO, a.stream);
                        }});
    low->bwd.push_back({"sgfc_bwd", 2.0 * act + 2.0 * dag.numel(dag.out) + wb + 4.0 * G * P.wgs_per_group * elems, 3.0 * flops,
                        [=](const RunArgs& a) {
                            sgfc::Params Q = P;
                            Q.xs = a.x_stride ? (int)a.x_stride : xs_dense;
                            Q.ys = a.y_stride ? (int)a.y_stride : ys_dense;
                            Q.x = (const uint16_t*)a.x;
                            Q.w = (const uint16_t*)a.w[widx];
                            Q.dy = (const uint16_t*)a.dy;
                            Q.dx = (uint16_t*)a.dx;
                            Q.partial = (float*)a.ws;
                            sgfc::backward(Q, KC, MO, a.stream);
                        }});
    const int wpg = P.wgs_per_group;
    low->bwd.push_back({"sgfc_dw_reduce", 4.0 * G * elems * (wpg + 1), 0, [=](const RunArgs& a) {
                            sgfc::dw_reduce((const float*)a.ws, (float*)a.dw[widx], G, wpg, elems, a.stream);
                        }});
    // Blocks: the instances of one tile in one wavefront.  Groups of 16 channels and an output as wide as the input; up to
    // eight instances, whose dW accumulators (4 KB of LDS each per workgroup) leave two workgroups a compute unit.  One
    // instance's workspace holds its partials and nothing else, so the instances' partials lie a workspace apart.
    if (KC == 1 && MO == 1 && fc.out == C) {
        low->max_instances = sgfc::kMaxInstances;
        auto fill = [=](const BlockArgs& b, sgfc::Params& Q, sgfc::Instances& I) {
            Q = P;
            I.m = b.m;
            I.slice = xs_dense;
            I.part_stride = (long long)(b.ws_stride / 4);
            Q.xs = b.expand ? xs_dense : b.m * xs_dense;
            Q.ys = b.expand ? b.m * ys_dense : ys_dense;
            Q.x = (const uint16_t*)b.args.x;
            Q.y = (uint16_t*)b.args.y;
            Q.dy = (const uint16_t*)b.args.dy;
            Q.dx = (uint16_t*)b.args.dx;
            Q.partial = (float*)b.args.ws;
            for (int j = 0; j < b.m; j++) {
                I.w[j] = (const uint16_t*)b.args.w[j];
                if (b.args.dw) I.dw[j] = (float*)b.args.dw[j];
            }
        };
        low->block_fwd = [=](const BlockArgs& b) {
            sgfc::Params Q;
            sgfc::Instances I;
            fill(b, Q, I);
            sgfc::forward_multi(Q, I, b.expand, b.args.stream);
        };
        low->block_bwd = [=](const BlockArgs& b) {
            sgfc::Params Q;
            sgfc::Instances I;
            fill(b, Q, I);
            sgfc::backward_multi(Q, I, b.expand, b.args.stream);
            sgfc::dw_reduce_multi(Q.partial, I, G, wpg, elems, b.args.stream);
        };
    }
    return low;
}

}  // namespace canvas
