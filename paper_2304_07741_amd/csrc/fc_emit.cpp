#include "fc_emit.hpp"

#include "gfc_kernels.hpp"
#include "gfc_staged_kernels.hpp"
#include "gfc_tm_kernels.hpp"
#include "gfc_wgrad_kernels.hpp"

namespace canvas {

// Room for the weights of the contraction T (R rows per group of the FC's own) in the layout of the staged kernels (S) or of the tap-major ones, and
// the job that fills it; returns the offset.
static int64_t pack_weights(Lowering& low, const TakeFn& take, const gfctm::Params& T, const gfcst::Params* S, int R, bool transposed, int widx) {
    const int64_t elems = S ? gfcst::packed_elems(*S) : gfctm::packed_elems(T);
    WeightJob j;
    j.job.kind = S ? 2 : 0;
    j.job.steps = S ? S->steps : 0;
    j.job.G = T.G;
    j.job.R = T.R;
    j.job.Rw = R;
    j.job.Og = T.Og;
    j.job.TV = T.TV;
    j.job.gm = T.gm;
    j.job.Gm = T.Gm;
    j.job.Rp = S ? S->Rp : T.Rp;
    j.job.Omp = S ? S->Omp : T.Omp;
    j.job.transposed = transposed ? 1 : 0;
    j.job.total = elems;
    j.widx = widx;
    j.off = take((uint64_t)elems * 2);
    j.bytes = 2.0 * T.G * T.Og * R * T.TV + 2.0 * elems;
    low.wjobs.push_back(j);
    return j.off;
}

void emit_fc(Lowering& low, bool backward, const Dag& dag, const TakeFn& take, const std::string& name, int G, int R, int kh, int kw, int Og,
             bool transposed, int widx, FcOperand src, PtrFn dst, bool addend_is_dst, double bytes, double flops, bool dst_f32, bool softmax, bool weights_as_they_are) {
    std::vector<Launch>& list = backward ? low.bwd : low.fwd;
    const int64_t nw = (int64_t)G * Og * R * kh * kw;
    const int rows = src.pairs ? 2 * R : R;
    if (!src.f32 && gfctm::supported(dag.N, G, rows, kh, kw, Og, dag.H, dag.W)) {
        const gfctm::Params T = gfctm::shape(dag.N, G, rows, kh, kw, Og, dag.H, dag.W);
        gfcst::Params S;
        const bool staged = !weights_as_they_are && gfcst::plan(S, T, dst_f32, addend_is_dst, softmax);
        const bool identity = !src.pairs && !transposed && gfctm::reads_weights_as_they_are(T) && !staged;
        const int64_t opk = identity ? -1 : pack_weights(low, take, T, staged ? &S : nullptr, R, transposed, widx);
        if (staged) {
            list.push_back({name, bytes, flops, [=](const RunArgs& a) {
                                gfcst::Params Q = S;
                                Q.src = (const uint16_t*)src.ptr(a);
                                Q.wp = (const uint16_t*)(a.ws + opk);
                                Q.dst = const_cast<void*>(dst(a));
                                Q.addend = addend_is_dst ? (const uint16_t*)dst(a) : nullptr;  // each lane reads the elements it then overwrites
                                gfcst::forward(Q, a.stream);
                            }});
            return;
        }
        list.push_back({name, bytes, flops, [=](const RunArgs& a) {
                            gfctm::Params Q = T;
                            Q.src = (const uint16_t*)src.ptr(a);
                            Q.wp = identity ? (const uint16_t*)a.w[widx] : (const uint16_t*)(a.ws + opk);
                            Q.dst = const_cast<void*>(dst(a));
                            Q.dst_f32 = dst_f32 ? 1 : 0;
                            Q.softmax = softmax ? 1 : 0;
                            Q.addend = addend_is_dst ? (const uint16_t*)dst(a) : nullptr;  // each lane reads the elements it then overwrites
                            gfctm::forward(Q, a.stream);
                        }});
        return;
    }
    gfc::Params F = gfc::shape(dag.N, G, R, kh, kw, Og, dag.H, dag.W);
    F.src_f32 = src.f32 ? 1 : 0;
    F.dst_f32 = dst_f32 ? 1 : 0;
    gfc::prepare_forward(F);
    const int64_t owt = transposed ? take((uint64_t)nw * 2) : -1;
    if (transposed) {  // (R, Og) are the swapped dims: the FC's own weights are [G][R][Og][taps]
        WeightJob j;
        j.job.kind = 1;
        j.job.G = G;
        j.job.Og = R;  // (the job reads [G][its Og][its R][TV]: the FC's own output and row counts)
        j.job.R = Og;
        j.job.TV = kh * kw;
        j.job.total = nw;
        j.widx = widx;
        j.off = owt;
        j.bytes = 4.0 * nw;
        low.wjobs.push_back(j);
    }
    list.push_back({name, bytes, flops, [=](const RunArgs& a) {
                        gfc::Params Q = F;
                        Q.src = src.ptr(a);
                        Q.w = transposed ? (const uint16_t*)(a.ws + owt) : (const uint16_t*)a.w[widx];
                        Q.dst = const_cast<void*>(dst(a));
                        Q.addend = addend_is_dst ? (const uint16_t*)dst(a) : nullptr;
                        gfc::forward(Q, a.stream);
                    }});
}

bool emit_fc_with_middle(Lowering& low, bool adjoint, const Dag& dag, const TakeFn& take, const std::string& name, int G, int R, int kh, int kw, int Og,
                         int widx, PtrFn src, PtrFn dst, double bytes, double flops, int act,
                         const std::function<ufc::MidParams(const RunArgs&)>& middle) {
    if (!gfctm::supported(dag.N, G, R, kh, kw, Og, dag.H, dag.W)) return false;
    const gfctm::Params T = gfctm::shape(dag.N, G, R, kh, kw, Og, dag.H, dag.W);
    gfcst::Params S;
    if (!gfcst::plan(S, T, false, false, false) || !gfcst::takes_middle(S, adjoint, act)) return false;
    const int64_t opk = pack_weights(low, take, T, &S, R, adjoint, widx);
    (adjoint ? low.bwd : low.fwd).push_back({name, bytes, flops, [=](const RunArgs& a) {
                                                 gfcst::Params Q = S;
                                                 Q.src = (const uint16_t*)src(a);
                                                 Q.wp = (const uint16_t*)(a.ws + opk);
                                                 if (adjoint) {
                                                     gfcst::dgrad_with_middle(Q, middle(a), a.stream);
                                                     return;
                                                 }
                                                 Q.dst = const_cast<void*>(dst(a));
                                                 gfcst::forward_with_middle(Q, middle(a), a.stream);
                                             }});
    return true;
}

uint64_t fc_packed_bytes(const Dag& dag, int G, int rows, int kh, int kw, int Og) {
    const gfctm::Params T = gfctm::shape(dag.N, G, rows, kh, kw, Og, dag.H, dag.W);
    gfcst::Params S;
    return 2 * (uint64_t)(gfcst::plan(S, T, false, false, false) ? gfcst::packed_elems(S) : gfctm::packed_elems(T));
}

bool fc_softmax_fusable(const Dag& dag, int G, int R, int kh, int kw, int Og, const FcOperand& src) {
    return !src.f32 && gfctm::supported(dag.N, G, R, kh, kw, Og, dag.H, dag.W) &&
           gfctm::softmax_fusable(gfctm::shape(dag.N, G, R, kh, kw, Og, dag.H, dag.W));
}

void emit_wgrad(Lowering& low, const Dag& dag, const TakeFn& take, const std::string& name, int G, int R, int kh, int kw, int Og,
                int widx, FcOperand src, FcOperand dy, double operand_bytes, double flops) {
    std::vector<Launch>& list = low.bwd;
    const int64_t nw = (int64_t)G * Og * R * kh * kw;
    if (kh * kw > 1 && !src.f32 && !dy.f32 && gfctm::supported(dag.N, G, R, kh, kw, Og, dag.H, dag.W)) {
        gfctm::Params T = gfctm::shape(dag.N, G, R, kh, kw, Og, dag.H, dag.W);
        gfcwg::Params S;
        const bool by_taps = gfcwg::plan(S, T);
        if (!by_taps) gfctm::prepare_wgrad(T);
        const int ts = by_taps ? S.slices : gfctm::wgrad_slices(T);
        const int64_t pk = gfctm::packed_elems(T);
        const int64_t opt = take((uint64_t)ts * pk * 4);
        auto bind = [=](auto Q, const RunArgs& a) {
            Q.src = (const uint16_t*)src.ptr(a);
            Q.dy = (const uint16_t*)dy.ptr(a);
            Q.partial = (float*)(a.ws + opt);
            return Q;
        };
        list.push_back({name, operand_bytes + 4.0 * ts * pk, flops, [=](const RunArgs& a) {
                            if (by_taps) gfcwg::wgrad_partial(bind(S, a), a.stream);
                            else gfctm::wgrad_partial(bind(T, a), a.stream);
                        }});
        ReduceJob rj;
        rj.job.slices = ts;
        rj.job.kind = 1;
        rj.job.count = (unsigned)pk;
        rj.job.G = T.G; rj.job.R = T.R; rj.job.Og = T.Og; rj.job.TV = T.TV;
        rj.job.gm = T.gm; rj.job.Omp = T.Omp; rj.job.Rp = T.Rp;
        wreduce::plan(rj.job);
        rj.widx = widx;
        rj.off = opt;
        rj.bytes = 4.0 * ts * pk + 4.0 * nw;
        low.rjobs.push_back(rj);
        return;
    }
    gfc::Params W = gfc::shape(dag.N, G, R, kh, kw, Og, dag.H, dag.W);
    W.src_f32 = src.f32 ? 1 : 0;
    W.dy_f32 = dy.f32 ? 1 : 0;
    gfc::prepare_wgrad(W);
    const int slices = gfc::wgrad_partials(W);
    const int64_t op = take((uint64_t)slices * nw * 4);
    list.push_back({name, operand_bytes + 4.0 * slices * nw, flops, [=](const RunArgs& a) {
                        gfc::Params Q = W;
                        Q.src = src.ptr(a);
                        Q.dy = dy.ptr(a);
                        Q.partial = (float*)(a.ws + op);
                        gfc::wgrad_partial(Q, a.stream);
                    }});
    ReduceJob rj;
    rj.job.slices = slices;
    rj.job.kind = 0;
    rj.job.count = (unsigned)nw;
    wreduce::plan(rj.job);
    rj.widx = widx;
    rj.off = op;
    rj.bytes = 4.0 * (slices + 1) * nw;
    low.rjobs.push_back(rj);
}

}  // namespace canvas
