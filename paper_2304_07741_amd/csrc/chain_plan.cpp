// Planner of the fused-chain kernels (host only).
//
// The unit's nodes are first expanded into an instance graph: an instance is "the value of node k as seen through a
// position context", the context being the stencil offsets (Shift terms, at most one Unfold window) collected on the
// way down from a consumer.  A Shift or Unfold node itself only adds to the context of its operand and masks what
// falls outside the image; the loads at the leaves carry the total offset.  Reductions (Fold, Softmax) are only
// legal in the empty context: a stencil above a reduction would need the reduction's result at other pixels.
// Code is then emitted by demand-driven recursion, with full recomputation instead of saved values: forward
// emit_eval(instance), backward emit_grad(instance) = sum over its users of their local adjoint applied to
// emit_grad(user).  A Softmax over channels splits a program into passes over the channel range (statistics first;
// in the backward program also the sum of gradient x output that its adjoint needs).
#include "chain_plan.hpp"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <memory>
#include <set>
#include <sstream>
#include <tuple>

#include "chain_kernels.hpp"

namespace canvas {
namespace chain {

namespace {

struct Fail {
    std::string why;
};

struct Ctx {
    std::vector<Term> terms;
    bool win = false;
    int kh = 1, kw = 1;
    bool empty() const { return terms.empty() && !win; }
    std::string key() const {
        std::ostringstream os;
        for (const Term& t : terms) os << t.dh << ',' << t.dw << ',' << t.c0 << ',' << t.c1 << ';';
        if (win) os << 'w' << kh << 'x' << kw;
        return os.str();
    }
    // how far (in pixels of the flattened plane) a read through this context can lie from the reading pixel
    int64_t reach_px(int W) const {
        int64_t r = win ? (int64_t)(kh / 2) * W + kw / 2 : 0;
        for (const Term& t : terms) r += (int64_t)std::abs((int)t.dh) * W + std::abs((int)t.dw);
        return r;
    }
};

enum InstKind { kExt, kIdent, kStencil, kUnaryI, kBinaryI, kSmT, kSmC, kFoldI, kBoxAdj };

struct Inst {
    int node = -1, ctx = 0, lanes = 1;
    InstKind kind = kExt;
    int opnd[2] = {-1, -1};
    std::vector<std::pair<int, int>> users;  // (instance, operand slot)
    int aux = -1;                            // kBoxAdj: the context of the window (see Graph::add_box_adjoints)
    int level = 0;                           // softmax-over-channels instances at or below this one (longest chain)
    int down = -1;                           // such instances above it (memo)
};

// Estimated cost of an instruction per pixel and channel, in units of one cheap lane operation.
double instr_weight(const Instr& I) {
    double w = 1;
    switch (I.op) {
    case OP_LD:
    case OP_BINLD:
    case OP_ST: w = 4; break;
    case OP_XADD: w = 6; break;
    case OP_LDFOLD: w = 4; break;
    case OP_UN:
    case OP_UNBX: w = (I.kind == 0 || I.kind == 1 || I.kind == kUnNeg) ? 1 : 6; break;
    case OP_SMT:
    case OP_SMTBX:
    case OP_SMCSTAT:
    case OP_SMCAPPLY: w = 6; break;
    default: break;
    }
    return w * I.T;
}

class Graph {
   public:
    Graph(const Dag& d, const std::vector<bool>& in_unit, const std::vector<bool>& is_output)
        : dag(d), in_unit_(in_unit), is_output_(is_output) {
        ctxs.push_back(Ctx());
        ctx_ids[""] = 0;
    }

    int ctx_id(const Ctx& c) {
        const std::string k = c.key();
        auto it = ctx_ids.find(k);
        if (it != ctx_ids.end()) return it->second;
        ctxs.push_back(c);
        return ctx_ids[k] = (int)ctxs.size() - 1;
    }

    int natural_lanes(int node, int ctx) const { return ctxs[ctx].win ? ctxs[ctx].kh * ctxs[ctx].kw : dag.nodes[node].T; }

    // the instance of `node` in context `ctx`; want > 0: an external tensor with fewer taps is read with lane t -> tap t % T
    int build(int node, int ctx, int want = 0) {
        const Node& nd = dag.nodes[node];
        if (ctxs[ctx].win && nd.T != 1) throw Fail{"a window over a tensor that has taps"};
        int lanes = natural_lanes(node, ctx);
        const bool external = !in_unit_[node];
        if (external && want > lanes && lanes > 1) {
            if (want % lanes) throw Fail{"tap counts of a blend do not divide"};
            lanes = want;
        }
        const auto key = std::make_tuple(node, ctx, lanes);
        auto it = memo.find(key);
        if (it != memo.end()) return it->second;
        Inst I;
        I.node = node;
        I.ctx = ctx;
        I.lanes = lanes;
        if (external) {
            I.kind = kExt;
            return add(key, I);
        }
        const bool reduction = nd.op == Op::Softmax || nd.op == Op::Fold;
        if (reduction && !ctxs[ctx].empty()) throw Fail{"a stencil above a reduction"};
        switch (nd.op) {
        case Op::Unfold: {
            if (ctxs[ctx].win) throw Fail{"nested windows"};
            Ctx c2 = ctxs[ctx];
            c2.win = true;
            c2.kh = nd.kh;
            c2.kw = nd.kw;
            I.kind = kStencil;
            I.opnd[0] = build(nd.a, ctx_id(c2));
            break;
        }
        case Op::Shift: {
            if ((nd.dh == 0 && nd.dw == 0) || nd.c0 >= nd.c1) {
                I.kind = kIdent;
                I.opnd[0] = build(nd.a, ctx);
            } else {
                Ctx c2 = ctxs[ctx];
                Term t;
                t.dh = (int16_t)nd.dh;
                t.dw = (int16_t)nd.dw;
                t.c0 = (uint16_t)nd.c0;
                t.c1 = (uint16_t)nd.c1;
                c2.terms.push_back(t);
                I.kind = kStencil;
                I.opnd[0] = build(nd.a, ctx_id(c2));
            }
            break;
        }
        case Op::Unary:
            I.kind = kUnaryI;
            I.opnd[0] = build(nd.a, ctx);
            break;
        case Op::Softmax:
            I.kind = nd.kind == kAxisC ? kSmC : kSmT;
            I.opnd[0] = build(nd.a, ctx);
            break;
        case Op::Fold:
            I.kind = kFoldI;
            I.opnd[0] = build(nd.a, ctx);
            break;
        case Op::Binary: {
            I.kind = kBinaryI;
            I.opnd[1] = build(nd.b, ctx);
            const int tr = insts[I.opnd[1]].lanes;
            if (tr != lanes) throw Fail{"blend: RHS lanes"};
            I.opnd[0] = build(nd.a, ctx, tr);
            const int tl = insts[I.opnd[0]].lanes;
            if (tl != 1 && tl != tr) throw Fail{"blend: an LHS inside the unit with fewer taps than the RHS"};
            break;
        }
        default: throw Fail{"not a chain primitive"};
        }
        return add(key, I);
    }

    int add(const std::tuple<int, int, int>& key, Inst I) {
        int lvl = 0;
        for (int s = 0; s < 2; s++)
            if (I.opnd[s] >= 0) lvl = std::max(lvl, insts[I.opnd[s]].level);
        I.level = lvl + (I.kind == kSmC ? 1 : 0);
        insts.push_back(I);
        const int id = (int)insts.size() - 1;
        for (int s = 0; s < 2; s++)
            if (I.opnd[s] >= 0) insts[I.opnd[s]].users.push_back({id, s});
        memo[key] = id;
        return id;
    }

    // Unfold followed at once by a sum / avg Fold that is an output of the unit and feeds nothing inside it is a linear
    // operator on the unfolded tensor's source (a box filter); its adjoint is the same filter applied to the incoming
    // gradient (the window is symmetric), which the pixel reads itself: a window load of dy and a fold, no hand-over of
    // T lanes to the neighbours.  Where EVERY Unfold of the unit is of that kind, each gets a pseudo user of its source's
    // own-pixel instance that stands for this adjoint in the backward program, and the leaves read through windows drop
    // out of it.  Returns whether that is so.
    bool add_box_adjoints() {
        std::vector<std::pair<int, int>> pairs;  // (unfold instance, fold instance)
        for (size_t i = 0; i < insts.size(); i++) {
            const Inst& U = insts[i];
            if (U.kind != kStencil || dag.nodes[U.node].op != Op::Unfold) continue;
            if (U.users.size() != 1 || is_output_[U.node]) return false;  // (a reader outside the unit has a gradient of its own to send through the window)
            const Inst& F = insts[U.users[0].first];
            const Node& fn = dag.nodes[F.node];
            if (F.kind != kFoldI || (fn.kind != kSum && fn.kind != kAvg) || !F.users.empty() || !is_output_[F.node] || F.ctx != 0 || U.ctx != 0)
                return false;
            pairs.push_back({(int)i, U.users[0].first});
        }
        if (pairs.empty()) return false;
        for (const auto& pr : pairs) {
            const int win_ctx = insts[insts[pr.first].opnd[0]].ctx;
            const int src = build(dag.nodes[insts[pr.first].node].a, insts[pr.first].ctx);
            if (insts[src].lanes != 1) throw Fail{"internal: the source of an unfold with taps"};
            Inst B;
            B.node = insts[pr.second].node;
            B.ctx = insts[pr.first].ctx;
            B.lanes = 1;
            B.kind = kBoxAdj;
            B.opnd[0] = src;
            B.aux = win_ctx;
            add(std::make_tuple(-1 - B.node, B.ctx, 1), B);
        }
        return true;
    }

    // softmax-over-channels instances on the longest way from instance i up to an output (i itself not counted)
    int down(int i) {
        if (insts[i].down >= 0) return insts[i].down;
        int d = 0;
        for (auto& u : insts[i].users) d = std::max(d, down(u.first) + (insts[u.first].kind == kSmC ? 1 : 0));
        return insts[i].down = d;
    }

    const Dag& dag;
    int root_ctx = 0;  // the context the unit's outputs are built in (not the empty one for a displaced unit)
    std::vector<Ctx> ctxs;
    std::map<std::string, int> ctx_ids;
    std::vector<Inst> insts;
    std::map<std::tuple<int, int, int>, int> memo;
    std::vector<bool> in_unit_, is_output_;
};

class Emitter {
   public:
    Emitter(Graph& g, int tm) : G(&g), NR(regs_for(tm)), used(regs_for(tm), false) { pg.tm = tm; }

    // Instructions may come from several instance graphs (the unit as it is, and the unit displaced by a stencil's
    // offsets: see compile_unit); `gidx` tells their instances apart in the tables below.
    void use(Graph& g, int idx) {
        G = &g;
        gidx = idx;
    }
    int gkey(int v) const { return gidx * (1 << 20) + v; }

    void emit(const Instr& I) {
        if (I.op == OP_MOVA && I.r == a_reg && I.T <= a_lanes) return;  // (A was just written there, or read from there)
        if (pg.n_instr >= kMaxInstr) throw Fail{"too many instructions"};
        pg.ins[pg.n_instr++] = I;
        weight += instr_weight(I);
        if (I.op == OP_MOVR || I.op == OP_MOVA) {
            a_reg = I.r;
            a_lanes = I.T;
        } else if (I.op != OP_ST && I.op != OP_PSET && I.op != OP_PADD && I.op != OP_XADD && I.op != OP_SMCSTAT && I.op != OP_SMCDOT) {
            a_reg = -1;
        }
    }
    int alloc() {
        for (int r = 0; r < NR; r++)
            if (!used[r]) {
                used[r] = true;
                pg.n_regs = std::max(pg.n_regs, r + 1);
                return r;
            }
        throw Fail{"out of registers"};
    }
    void release(int r) { used[r] = false; }
    int persist(int n) {
        const int a = pg.n_persist;
        pg.n_persist += n;
        return a;
    }
    int ext_slot(int node, ExtRole role) {
        for (size_t i = 0; i < ext.size(); i++)
            if (ext[i].node == node && ext[i].role == role) return (int)i;
        if ((int)ext.size() >= kMaxExt) throw Fail{"too many external tensors"};
        ExtRef e;
        e.node = node;
        e.role = role;
        ext.push_back(e);
        pg.ext[ext.size() - 1].T = G->dag.nodes[node].T;
        pg.n_ext = (int)ext.size();
        return (int)ext.size() - 1;
    }
    uint16_t terms(int ctx) {
        auto it = term_of.find(gkey(ctx));
        if (it != term_of.end()) return it->second;
        const Ctx& c = G->ctxs[ctx];
        if (pg.n_terms + (int)c.terms.size() > kMaxTerms) throw Fail{"too many stencil offsets"};
        const int first = pg.n_terms;
        for (const Term& t : c.terms) pg.term[pg.n_terms++] = t;
        return term_of[gkey(ctx)] = (uint16_t)((first << 8) | (int)c.terms.size());
    }
    Instr positional(Opcode op, int ctx, int lanes) {
        Instr I;
        I.op = op;
        I.T = (uint8_t)lanes;
        I.b = terms(ctx);
        const Ctx& c = G->ctxs[ctx];
        if (c.win) {
            I.kind |= kWin;
            I.r = (uint8_t)((c.kh << 4) | c.kw);
        }
        return I;
    }
    // OP_BINLD: A (lanes) blended with the external instance i, read in place (its own lanes: `lanes`, or 1 replicated)
    Instr load_and_blend(int i, int lanes, int blend, bool loaded_is_lhs) {
        const Inst& L = G->insts[i];
        Instr I = positional(OP_BINLD, L.ctx, lanes);
        I.a = (uint16_t)ext_slot(L.node, kValueIn);
        if (G->dag.nodes[L.node].T > 1) I.kind |= kExtTaps;
        I.kind |= (uint8_t)(blend << kBinLdKindShift);
        if (loaded_is_lhs) I.kind |= kBinLdLoadedIsLhs;
        if (L.lanes == 1 && lanes > 1) I.kind |= kBinLdLoadedScalar;
        return I;
    }
    static Instr simple(Opcode op, int T, int r = 0, int kind = 0, int a = 0) {
        Instr I;
        I.op = op;
        I.T = (uint8_t)T;
        I.r = (uint8_t)r;
        I.kind = (uint8_t)kind;
        I.a = (uint16_t)a;
        return I;
    }

    // ---------------------------------------------------------------- values kept for another use
    // A value (key 2 * instance) or a gradient (key 2 * instance + 1) that `keep` names is stored in a register the
    // first time a pass body computes it and fetched from there afterwards.  `stats` records, per key, how often it was
    // computed and what one computation cost: what the choice of `keep` is made from.
    struct Stat {
        int computed = 0, lanes = 1;
        double cost = 0;
    };
    void cached(int key0, int lanes, void (Emitter::*raw)(int), int i) {
        const int key = gkey(key0);
        auto it = held.find(key);
        if (it != held.end()) {
            emit(simple(OP_MOVA, lanes, it->second));
            return;
        }
        const double before = weight;
        (this->*raw)(i);
        Stat& st = stats[key];
        st.computed++;
        st.lanes = lanes;
        st.cost = std::max(st.cost, weight - before);
        if (keep.count(key)) {
            const int r = alloc();
            emit(simple(OP_MOVR, lanes, r));
            held[key] = r;
        }
    }
    void forget_graph(int idx) {  // (what a displaced copy kept is of no use to the next one)
        for (auto it = held.begin(); it != held.end();) {
            if (it->first / (1 << 20) == idx) {
                release(it->second);
                it = held.erase(it);
            } else {
                ++it;
            }
        }
    }
    void forget() {  // (a register's content does not outlive the body it was written in)
        for (auto& kv : held) release(kv.second);
        held.clear();
    }
    // an instance whose value is another one's (a stencil that has nothing to mask)
    int same_value(int i) const {
        while (G->insts[i].kind == kIdent || (G->insts[i].kind == kStencil && zero_outside(G->insts[i].opnd[0]))) i = G->insts[i].opnd[0];
        return i;
    }
    void eval(int i) {
        i = same_value(i);
        cached(2 * i, G->insts[i].lanes, &Emitter::eval_raw, i);
    }
    void grad(int i) { cached(2 * i + 1, G->insts[i].lanes, &Emitter::grad_raw, i); }
    // The register that holds the value (grad_key = 0) or the gradient (1) of instance i already, or -1.
    int kept(int i, int grad_key) const {
        if (!grad_key) i = same_value(i);
        auto it = held.find(gkey(2 * i + grad_key));
        return it == held.end() ? -1 : it->second;
    }
    // The same value in a register, wherever it has to come from; `mine` says that the caller releases it.
    int to_reg(int i, int grad_key, bool& mine) {
        mine = false;
        int r = kept(i, grad_key);
        if (r >= 0) return r;
        if (grad_key) grad(i);
        else eval(i);
        r = kept(i, grad_key);
        if (r >= 0) return r;
        mine = true;
        r = alloc();
        emit(simple(OP_MOVR, G->insts[i].lanes, r));
        return r;
    }
    // Whether instance i is zero by itself wherever its position lies outside the image: what it loads is, and what
    // is done to it keeps zeros (every position below it is its own: no further stencil in between).
    bool zero_outside(int i) const {
        const Inst& I = G->insts[i];
        const Node& nd = G->dag.nodes[I.node];
        switch (I.kind) {
        case kExt: return true;
        case kIdent: return zero_outside(I.opnd[0]);
        case kUnaryI: return nd.kind != kExpClip && zero_outside(I.opnd[0]);
        case kBinaryI: return zero_outside(I.opnd[0]) && zero_outside(I.opnd[1]);
        default: return false;
        }
    }
    // Whether every tensor instance i is made of is read at i's own position: the gradient of a position outside the
    // image then ends at a read that no pixel receives.
    bool own_position(int i) const {
        const Inst& I = G->insts[i];
        switch (I.kind) {
        case kExt: return true;
        case kIdent:
        case kUnaryI: return own_position(I.opnd[0]);
        case kBinaryI: return own_position(I.opnd[0]) && own_position(I.opnd[1]);
        default: return false;
        }
    }

    // ---------------------------------------------------------------- forward values
    void eval_raw(int i) {
        const Inst& I = G->insts[i];
        const Node& nd = G->dag.nodes[I.node];
        switch (I.kind) {
        case kExt: {
            Instr ld = positional(OP_LD, I.ctx, I.lanes);
            ld.a = (uint16_t)ext_slot(I.node, kValueIn);
            if (nd.T > 1) ld.kind |= kExtTaps;
            emit(ld);
            break;
        }
        case kIdent: eval(I.opnd[0]); break;
        case kStencil: {
            eval(I.opnd[0]);
            const Inst& S = G->insts[I.opnd[0]];
            if (!zero_outside(I.opnd[0])) emit(positional(OP_MASK, S.ctx, I.lanes));  // (a load checks its own position)
            break;
        }
        case kUnaryI: {
            eval(I.opnd[0]);
            Instr u = simple(OP_UN, I.lanes, 0, nd.kind);
            u.f0 = nd.lo;
            u.f1 = nd.hi;
            emit(u);
            break;
        }
        case kBinaryI: {
            const int tl = G->insts[I.opnd[0]].lanes;
            if (G->insts[I.opnd[0]].kind == kExt) {  // the LHS comes straight from memory
                eval(I.opnd[1]);
                emit(load_and_blend(I.opnd[0], I.lanes, nd.kind, true));
                break;
            }
            if (G->insts[I.opnd[1]].kind == kExt && tl == I.lanes) {  // the RHS does
                eval(I.opnd[0]);
                emit(load_and_blend(I.opnd[1], I.lanes, nd.kind, false));
                break;
            }
            const bool lhs_scalar = tl == 1 && I.lanes > 1;
            bool mine;
            if (kept(I.opnd[0], 0) < 0) {  // (an RHS in a register is taken from there, also when computing the LHS put it there)
                eval(I.opnd[0]);
                const int rr = kept(I.opnd[1], 0);
                if (rr >= 0) {
                    emit(simple(OP_BIN, I.lanes, rr, nd.kind | (lhs_scalar ? kBinAccScalar : 0)));
                    break;
                }
                int r = kept(I.opnd[0], 0);
                mine = r < 0;
                if (mine) emit(simple(OP_MOVR, tl, r = alloc()));
                eval(I.opnd[1]);
                emit(simple(OP_BIN, I.lanes, r, nd.kind | kBinRegIsLhs | (lhs_scalar ? kBinRegScalar : 0)));
                if (mine) release(r);
                break;
            }
            const int r = to_reg(I.opnd[0], 0, mine);
            eval(I.opnd[1]);
            emit(simple(OP_BIN, I.lanes, r, nd.kind | kBinRegIsLhs | (lhs_scalar ? kBinRegScalar : 0)));
            if (mine) release(r);
            break;
        }
        case kSmT:
            eval(I.opnd[0]);
            emit(simple(OP_SMT, I.lanes));
            break;
        case kSmC:
            eval(I.opnd[0]);
            emit(simple(OP_SMCAPPLY, I.lanes, 0, 0, stat_slot(i)));
            break;
        case kFoldI:
            eval(I.opnd[0]);
            emit(simple(OP_FOLD, G->insts[I.opnd[0]].lanes, 0, nd.kind));
            break;
        case kBoxAdj: throw Fail{"internal: the value of a box adjoint"};
        }
    }

    int stat_slot(int i) {
        auto it = stat_slots.find(i);
        if (it != stat_slots.end()) return it->second;
        return stat_slots[i] = persist(2 * G->insts[i].lanes);
    }
    int dot_slot(int i) {
        auto it = dot_slots.find(i);
        if (it != dot_slots.end()) return it->second;
        return dot_slots[i] = persist(G->insts[i].lanes);
    }

    // ---------------------------------------------------------------- gradients
    // leaves d loss / d instance i in A (lanes of i)
    void grad_raw(int i) {
        const Inst& I = G->insts[i];
        bool first = true;
        int held = -1;
        auto begin_term = [&]() {
            if (!first) {
                held = alloc();
                emit(simple(OP_MOVR, I.lanes, held));
            }
        };
        auto end_term = [&]() {
            if (!first) {
                emit(simple(OP_BIN, I.lanes, held, kAdd | kBinRegIsLhs));
                release(held);
            }
            first = false;
        };
        if (I.kind != kExt && I.ctx == G->root_ctx && G->is_output_[I.node] && I.lanes == G->dag.nodes[I.node].T) {
            begin_term();
            Instr ld = positional(OP_LD, G->root_ctx, I.lanes);  // (a displaced unit reads the incoming gradient displaced)
            ld.a = (uint16_t)ext_slot(I.node, kGradIn);
            if (I.lanes > 1) ld.kind |= kExtTaps;
            emit(ld);
            end_term();
        }
        for (const auto& u : I.users) {
            begin_term();
            contribution(u.first, u.second, i);
            end_term();
        }
        if (first) throw Fail{"internal: an instance without users"};
    }

    // d loss / d (operand `slot` of user instance u), which is instance i
    void contribution(int u, int slot, int i) {
        const Inst& U = G->insts[u];
        const Inst& I = G->insts[i];
        const Node& un = G->dag.nodes[U.node];
        if (U.kind == kBoxAdj) {  // the box filter's adjoint: the same filter over the incoming gradient of the fold's output
            const Ctx& wc = G->ctxs[U.aux];
            Instr ld = positional(OP_LD, U.aux, wc.kh * wc.kw);
            ld.a = (uint16_t)ext_slot(U.node, kGradIn);
            emit(ld);
            emit(simple(OP_FOLD, wc.kh * wc.kw, 0, un.kind));
            return;
        }
        // (registers and A: a gradient or value that a register keeps is used there, not copied to another one)
        bool mine = false;
        switch (U.kind) {
        case kIdent: grad(u); break;
        case kStencil:
            grad(u);
            if (!own_position(i)) emit(positional(OP_MASK, I.ctx, U.lanes));
            break;
        case kUnaryI: {
            const int r = to_reg(u, 1, mine);
            eval(un.kind == kRelu && kept(u, 0) >= 0 ? u : i);  // (relu: its result is positive where its argument is)
            Instr b = simple(OP_UNBX, U.lanes, r, un.kind);
            b.f0 = un.lo;
            b.f1 = un.hi;
            emit(b);
            if (mine) release(r);
            break;
        }
        case kBinaryI: {
            const int other = U.opnd[1 - slot];
            const int tl = G->insts[U.opnd[0]].lanes;
            const bool lhs_scalar = tl == 1 && U.lanes > 1;
            if (un.kind == kAdd || (un.kind == kSub && slot == 0)) {
                grad(u);
            } else if (un.kind == kSub) {
                grad(u);
                emit(simple(OP_UN, U.lanes, 0, kUnNeg));
            } else if (un.kind == kMul && kept(other, 0) < 0 && G->insts[other].kind == kExt) {
                // the gradient in A times the other operand, which comes straight from memory
                grad(u);
                emit(load_and_blend(other, U.lanes, kMul, false));
            } else if (un.kind == kMul) {
                // the other operand is a scalar when it is the 1-lane LHS
                const bool scalar = slot == 1 && lhs_scalar;
                if (kept(u, 1) < 0) grad(u);
                const int ro = kept(other, 0), rg = kept(u, 1);
                if (ro >= 0) {
                    if (rg >= 0) emit(simple(OP_MOVA, U.lanes, rg));
                    emit(simple(OP_BIN, U.lanes, ro, kMul | (scalar ? kBinRegScalar : 0)));
                } else {
                    const int r = rg >= 0 ? rg : alloc();
                    if (rg < 0) emit(simple(OP_MOVR, U.lanes, r));
                    eval(other);
                    emit(simple(OP_BIN, U.lanes, r, kMul | (scalar ? kBinAccScalar : 0)));
                    if (rg < 0) release(r);
                }
            } else {  // min / max: the indicator needs both operands
                bool mine_l;
                const int rg = to_reg(u, 1, mine);
                const int rl = to_reg(U.opnd[0], 0, mine_l);
                eval(U.opnd[1]);
                emit(simple(OP_BING, U.lanes, rl, un.kind | (slot == 1 ? kBingRhsSide : 0) | (lhs_scalar ? kBingLhsScalar : 0)));
                emit(simple(OP_BIN, U.lanes, rg, kMul));
                if (mine_l) release(rl);
                if (mine) release(rg);
            }
            if (slot == 0 && lhs_scalar) emit(simple(OP_FOLD, U.lanes, 0, kSum));  // the replicated LHS collects all lanes
            break;
        }
        case kSmT: {
            int r = kept(u, 1);
            if (r < 0) {
                grad(u);
                if (kept(u, 0) >= 0) {  // (evaluated on the way: the gradient stays in A)
                    emit(simple(OP_SMTBX, U.lanes, kept(u, 0), 1));
                    break;
                }
                r = kept(u, 1);
                if (r < 0) {
                    mine = true;
                    r = alloc();
                    emit(simple(OP_MOVR, U.lanes, r));
                }
            }
            eval(u);
            emit(simple(OP_SMTBX, U.lanes, r));
            if (mine) release(r);
            break;
        }
        case kSmC: {
            const int r = to_reg(u, 1, mine);
            eval(u);
            emit(simple(OP_SMCBX, U.lanes, r, 0, dot_slot(u)));
            if (mine) release(r);
            break;
        }
        case kFoldI: {
            const int r = to_reg(u, 1, mine);
            if (un.kind == kMax) eval(i);
            emit(simple(OP_FOLDBX, I.lanes, r, un.kind));
            if (mine) release(r);
            break;
        }
        case kBoxAdj: break;  // (handled above)
        case kExt: throw Fail{"internal: an external tensor as a user"};
        }
    }

    // ---------------------------------------------------------------- gradients through a window, fetched by the source pixel
    // The gradient of a tensor read through a window is, for its pixel p, the sum over the taps t of what lane t of the
    // consumer at p - offset(t) hands back.  Where that depends on nothing but the consumer's own values (lanes equal) and on
    // the source pixel's, p evaluates it itself: whatever the consumer reads at its own position is read through the window
    // (which is symmetric: the lanes come in the opposite order, for all of them alike), whatever it reads through the window
    // is p's own.  Lanes and positions change places; a value that the consumer computes from all of its taps (a fold's
    // result, a softmax over the taps, the first maximum) cannot be had this way and the leaf keeps its hand-over (Fail).
    // mlanes: lanes of instance i in that view; meval: its value; mgrad: its gradient, mlanes(i) lanes.  The factor 1/T of
    // an avg fold on the way is applied where the lanes are added (`avg`; everything in between is linear).
    // A consumer outside the image does not exist: its gradient is loaded as 0 and adds nothing, but times p's own value, if that is
    // infinite or NaN, it would; then (mproduct) the lanes are masked before they are added.
    int mwin = -1;  // the window's context
    bool mproduct = false;
    int mtaps() const { return G->ctxs[mwin].kh * G->ctxs[mwin].kw; }
    int mlanes(int i) const {
        const Inst& I = G->insts[i];
        if (I.ctx != 0 && I.ctx != mwin) throw Fail{"mirror: another position"};
        switch (I.kind) {
        case kExt:
            if (G->dag.nodes[I.node].T != 1) throw Fail{"mirror: a tensor with taps"};
            return I.ctx == mwin ? 1 : mtaps();
        case kIdent:
        case kUnaryI: return mlanes(I.opnd[0]);
        case kStencil:
            if (G->dag.nodes[I.node].op != Op::Unfold || G->insts[I.opnd[0]].ctx != mwin) throw Fail{"mirror: a shift"};
            return mlanes(I.opnd[0]);
        case kBinaryI: return std::max(mlanes(I.opnd[0]), mlanes(I.opnd[1]));
        default: throw Fail{"mirror: a value of all taps"};
        }
    }
    int mctx(int i) const { return G->insts[i].ctx == mwin ? 0 : mwin; }  // (of a leaf)
    // A (lanes) blended with the leaf i in its place: OP_BINLD as load_and_blend
    void mblend(int i, int lanes, int blend, bool loaded_is_lhs) {
        Instr I = positional(OP_BINLD, mctx(i), lanes);
        I.a = (uint16_t)ext_slot(G->insts[i].node, kValueIn);
        I.kind |= (uint8_t)(blend << kBinLdKindShift);
        if (loaded_is_lhs) I.kind |= kBinLdLoadedIsLhs;
        if (mlanes(i) == 1 && lanes > 1) {
            I.kind = (uint8_t)((I.kind & ~kWin) | kBinLdLoadedScalar);
            I.r = 0;
        }
        emit(I);
    }
    void meval(int i) {
        const Inst& I = G->insts[i];
        const Node& nd = G->dag.nodes[I.node];
        const int lanes = mlanes(i);
        switch (I.kind) {
        case kExt: {
            Instr ld = positional(OP_LD, mctx(i), lanes);
            ld.a = (uint16_t)ext_slot(I.node, kValueIn);
            emit(ld);
            break;
        }
        case kUnaryI: {
            meval(I.opnd[0]);
            Instr u = simple(OP_UN, lanes, 0, nd.kind);
            u.f0 = nd.lo;
            u.f1 = nd.hi;
            emit(u);
            break;
        }
        case kBinaryI: {
            const int a = I.opnd[0], b = I.opnd[1];
            if (G->insts[a].kind == kExt && mlanes(b) == lanes) {
                meval(b);
                mblend(a, lanes, nd.kind, true);
                break;
            }
            if (G->insts[b].kind == kExt && mlanes(a) == lanes) {
                meval(a);
                mblend(b, lanes, nd.kind, false);
                break;
            }
            meval(a);
            const int r = alloc();
            emit(simple(OP_MOVR, mlanes(a), r));
            meval(b);
            emit(simple(OP_BIN, lanes, r, nd.kind | kBinRegIsLhs | (mlanes(a) < lanes ? kBinRegScalar : 0) | (mlanes(b) < lanes ? kBinAccScalar : 0)));
            release(r);
            break;
        }
        default: meval(I.opnd[0]);  // (a view: the values outside the image belong to pixels that do not exist)
        }
    }
    void mgrad(int i, bool& avg) {
        const Inst& I = G->insts[i];
        const int lanes = mlanes(i);
        bool first = true;
        int sum = -1;
        auto begin_term = [&]() {
            if (!first) emit(simple(OP_MOVR, lanes, sum = alloc()));
        };
        auto end_term = [&](bool a) {
            if (!first) {
                if (a != avg) throw Fail{"mirror: terms with and without the factor of an avg fold"};
                emit(simple(OP_BIN, lanes, sum, kAdd | kBinRegIsLhs));
                release(sum);
            }
            avg = a;
            first = false;
        };
        if (I.kind != kExt && I.ctx == 0 && G->is_output_[I.node] && I.lanes == G->dag.nodes[I.node].T) {
            if (I.lanes != 1) throw Fail{"mirror: an output with taps"};
            begin_term();
            Instr ld = positional(OP_LD, mwin, mtaps());
            ld.a = (uint16_t)ext_slot(I.node, kGradIn);
            emit(ld);
            end_term(false);
        }
        for (const auto& u : I.users) {
            begin_term();
            bool a = false;
            mcontribution(u.first, u.second, i, a);
            end_term(a);
        }
        if (first) throw Fail{"internal: an instance without users"};
    }
    // lanes of the user's gradient in this view (a fold's result is a value of the consumer: one per tap of the window)
    int mglanes(int u) const {
        if (G->insts[u].kind == kFoldI && G->insts[u].ctx == 0) return mtaps();
        return mlanes(u);
    }
    void mgrad_of_user(int u, bool& avg) {
        const Inst& U = G->insts[u];
        if (U.kind != kFoldI) {
            mgrad(u, avg);
            return;
        }
        if (U.ctx != 0 || G->dag.nodes[U.node].kind == kMax || G->insts[U.opnd[0]].lanes != mtaps()) throw Fail{"mirror: a fold of other lanes"};
        // the fold's own gradient: only the one that comes from memory (a consumer of its result inside the unit would go on here)
        if (!U.users.empty() || !G->is_output_[U.node]) throw Fail{"mirror: a fold whose result is used inside the unit"};
        Instr ld = positional(OP_LD, mwin, mtaps());
        ld.a = (uint16_t)ext_slot(U.node, kGradIn);
        emit(ld);
        avg = G->dag.nodes[U.node].kind == kAvg;
    }
    void mcontribution(int u, int slot, int i, bool& avg) {
        const Inst& U = G->insts[u];
        const Node& un = G->dag.nodes[U.node];
        const int lanes = mglanes(u), mine = mlanes(i);
        switch (U.kind) {
        case kIdent:
        case kStencil:
        case kFoldI: mgrad_of_user(u, avg); break;
        case kUnaryI: {
            mgrad(u, avg);
            const int r = alloc();
            emit(simple(OP_MOVR, lanes, r));
            meval(i);
            Instr b = simple(OP_UNBX, lanes, r, un.kind);
            b.f0 = un.lo;
            b.f1 = un.hi;
            emit(b);
            release(r);
            mproduct |= lanes > 1;
            break;
        }
        case kBinaryI: {
            const int other = U.opnd[1 - slot];
            mgrad(u, avg);
            if (un.kind == kAdd || (un.kind == kSub && slot == 0)) break;
            if (un.kind == kSub) {
                emit(simple(OP_UN, lanes, 0, kUnNeg));
                break;
            }
            if (un.kind == kMul && G->insts[other].kind == kExt) {
                mblend(other, lanes, kMul, false);
                mproduct |= lanes > 1 && mlanes(other) == 1;  // (else the consumer's own, which is loaded as 0 as well)
                break;
            }
            mproduct |= lanes > 1;
            const int rg = alloc();
            emit(simple(OP_MOVR, lanes, rg));
            if (un.kind == kMul) {
                meval(other);
                emit(simple(OP_BIN, lanes, rg, kMul | (mlanes(other) < lanes ? kBinAccScalar : 0)));
            } else {
                const int ll = mlanes(U.opnd[0]), lr = mlanes(U.opnd[1]);
                meval(U.opnd[0]);
                const int rl = alloc();
                emit(simple(OP_MOVR, ll, rl));
                meval(U.opnd[1]);
                emit(simple(OP_BING, lanes, rl, un.kind | (slot == 1 ? kBingRhsSide : 0) | (ll < lanes ? kBingLhsScalar : 0) | (lr < lanes ? kBingRhsScalar : 0)));
                emit(simple(OP_BIN, lanes, rg, kMul));
                release(rl);
            }
            release(rg);
            break;
        }
        default: throw Fail{"mirror: a gradient of all taps"};
        }
        if (mine < lanes) {
            if (mproduct) emit(positional(OP_MASK, mwin, lanes));
            mproduct = false;
            emit(simple(OP_FOLD, lanes, 0, avg ? kAvg : kSum));
            avg = false;
        }
    }
    // the whole of it: d loss / d (the tensor leaf i reads through its window), one lane, in A
    void mirror(int i) {
        mwin = G->insts[i].ctx;
        const Ctx& c = G->ctxs[mwin];
        if (!c.terms.empty() || mlanes(i) != 1) throw Fail{"mirror: a window behind a shift"};
        bool avg = false;
        mproduct = false;
        mgrad(i, avg);
        if (avg) throw Fail{"mirror: lanes that were never added"};
    }

    void begin_pass() {
        a_reg = -1;
        if (pg.n_pass >= kMaxPass) throw Fail{"too many passes"};
        pg.pass[pg.n_pass].pro_begin = (uint16_t)pg.n_instr;
        pg.pass[pg.n_pass].red_begin = pg.pass[pg.n_pass].red_end = (uint16_t)pg.n_red;
    }
    // a quantity of the current pass that runs across the channel loop (the slices of a workgroup combine it at the end)
    void reduce(int slot, int T, int kind) {
        if (pg.n_red >= kMaxRed) throw Fail{"too many reductions across channels"};
        Red r;
        r.slot = (uint16_t)slot;
        r.T = (uint8_t)T;
        r.kind = (uint8_t)kind;
        pg.red[pg.n_red++] = r;
        pg.pass[pg.n_pass].red_end = (uint16_t)pg.n_red;
    }
    void begin_body() {
        a_reg = -1;
        pg.pass[pg.n_pass].pro_end = pg.pass[pg.n_pass].body_begin = (uint16_t)pg.n_instr;
    }
    void end_pass() {
        pg.pass[pg.n_pass++].body_end = (uint16_t)pg.n_instr;
        if (!one_trip) forget();
    }

    // the passes that collect the statistics of every softmax over channels, lowest first
    void stat_passes(const std::vector<int>& smc) {
        int top = 0;
        for (int i : smc) top = std::max(top, G->insts[i].level);
        for (int lvl = 1; lvl <= top; lvl++) {
            begin_pass();
            for (int i : smc)
                if (G->insts[i].level == lvl) {
                    Instr m = simple(OP_PSET, G->insts[i].lanes, 0, 0, stat_slot(i));
                    m.f0 = -INFINITY;
                    emit(m);
                    emit(simple(OP_PSET, G->insts[i].lanes, 0, 0, stat_slot(i) + G->insts[i].lanes));
                    reduce(stat_slot(i), G->insts[i].lanes, 0);
                }
            begin_body();
            for (int i : smc)
                if (G->insts[i].level == lvl) {
                    eval(G->insts[i].opnd[0]);
                    emit(simple(OP_SMCSTAT, G->insts[i].lanes, 0, 0, stat_slot(i)));
                }
            end_pass();
        }
    }

    Graph* G;
    int gidx = 0;
    // The threads make one trip through every body (the workgroup has a thread for every channel): what one pass kept is
    // there in the next, for the same channels.  A value or gradient that a pass computes rests on statistics that are
    // complete by then, so it is the same in every later pass.
    bool one_trip = false;
    Program pg;
    std::vector<ExtRef> ext;
    int NR;
    std::vector<bool> used;
    std::map<int, uint16_t> term_of;
    std::map<int, int> stat_slots, dot_slots;
    std::set<int> keep;
    std::map<int, int> held;
    std::map<int, Stat> stats;
    double weight = 0;                // of the instructions so far
    int a_reg = -1, a_lanes = 0;      // the register whose lanes A equals at this point of the program (-1: none)
    std::map<int, int64_t> reach_of;  // per OP_XADD instruction: how far (in pixels) its sources can lie
};

int ceil_div(int a, int b) { return (a + b - 1) / b; }

double workgroups_per_cu(const Program& pg) {
    // (the instances with 9 lanes x 4 pixels and with 25 lanes hold more than 128 vector registers: two wavefronts per
    // SIMD, not four)
    const double resident_threads = (pg.tm > 9 || (pg.tm > 1 && pg.vec >= 4)) ? 512.0 : 1024.0;
    return std::max(1.0, std::min(resident_threads / pg.threads, std::floor(160.0 * 1024.0 / (double)(lds_bytes(pg) + 4352))));
}
// How many times over the launch fills the chip.
double rounds_of(const Program& pg) { return (double)pg.N * pg.tiles * pg.chunks / (256.0 * workgroups_per_cu(pg)); }

// Workgroup shape for the pixels per thread already set and `pt` threads per slice (at most `cap`): tile and halo (`own`
// threads of the tile store, HT more on either side), channel range and slices.
// Returns the estimated cost of the launch (arbitrary units, see set_geometry) or a negative number when it does not fit.
double geometry_for(Program& pg, const Dag& dag, int C, bool all_channels, bool one_trip, int PP, int HT, int cap, int own, int pt, int trips) {
    pg.pix_threads = pt;
    pg.own_threads = own;
    pg.halo_threads = HT;
    pg.tiles = ceil_div(PP, own);
    // channel slices: the loads of different channels are independent, so threads are worth more than trips
    const int max_slices = std::max(1, cap / pt);
    if (all_channels) {
        pg.chunk = C;
        pg.chunks = 1;
        pg.slices = std::min(max_slices, std::min(ceil_div(C, pg.unroll), 16));
    } else {
        const int S = std::max(1, std::min(std::min(max_slices, 4), ceil_div(C, pg.unroll)));
        const int chunks = ceil_div(C, S * pg.unroll * trips);
        pg.chunk = ceil_div(C, chunks);
        pg.chunks = ceil_div(C, pg.chunk);
        pg.slices = std::min(S, ceil_div(pg.chunk, pg.unroll));
    }
    if (one_trip && pg.slices * pg.unroll < pg.chunk) return -1;
    pg.threads = pg.slices * pg.pix_threads;
    if (lds_bytes(pg) > kMaxLdsBytes || (int64_t)dag.N * pg.tiles * pg.chunks >= ((int64_t)1 << 31)) return -1;
    // cost: trips of a thread x what a trip costs (a fixed part for fetching and dispatching the instructions, worth
    // about eight pixels of arithmetic, plus per channel the pixels and about four pixels' worth for its narrow memory
    // accesses) x how many times over the launch fills the chip (256 compute units, about 1024 resident threads each)
    const double trips_per_thread = (double)ceil_div(pg.chunk, pg.slices * pg.unroll);
    // (whole rounds: a round that a few left-over workgroups make takes as long as a full one)
    const double rounds = std::max(1.0, std::ceil(rounds_of(pg) - 0.05));
    // (a work item also costs its set-up: the thread's position, the pass headers; worth about 6 of these units)
    return (6.0 + trips_per_thread * (8.0 + (pg.vec + 4.0) * pg.unroll)) * rounds;
}

// Pixels per thread, threads per slice and trips per thread: whatever the estimate likes best.
// whole_planes: a tile that holds a plane whole has no halo.  Returns the estimate.
double set_geometry(Program& pg, const Dag& dag, int C, int64_t reach_px, bool all_channels, bool one_trip, bool whole_planes = true) {
    pg.N = dag.N;
    pg.C = C;
    pg.H = dag.H;
    pg.W = dag.W;
    pg.xadd_lanes = 0;
    for (int i = 0; i < pg.n_instr; i++)
        if (pg.ins[i].op == OP_XADD) pg.xadd_lanes = std::max<int>(pg.xadd_lanes, pg.ins[i].T);
    if (pg.tm == 1 || pg.xadd_lanes == 0 || (int64_t)pg.n_regs * reg_pieces_of(pg.tm, 1) * 4 < pg.xadd_lanes) pg.xadd_alias = 0;
    const int HW = dag.H * dag.W;
    // (a program that makes one trip keeps its registers' LDS: floats that no channel has for itself exist once.  The other
    // programs' workgroups were weighed with a copy per channel of the trip, and the estimate errs without them: softmax over
    // channels, 128x64 planes of 56x56 backward 177 us with the workgroup it chooses so, 250 otherwise.)
    // Except where the launch then still has a compute unit for every workgroup: more slices of the channels are all that
    // helps there (two softmaxes over 192 channels, 7 planes of 16x28, backward: 280 us with three slices, 153 with eight).
    bool one_copy = all_channels;
    for (int p = 0; p < pg.n_pass; p++)
        for (int i = pg.pass[p].body_begin; i < pg.pass[p].body_end; i++)
            if (pg.ins[i].op == OP_PSET || pg.ins[i].op == OP_PADD || pg.ins[i].op == OP_PLD || pg.ins[i].op == OP_XADD) one_copy = false;
    const bool streams = streams_windows(pg);  // (threads of one image row each)
    Program best_shape = pg;
    double best_cost = -1;
    auto look = [&](bool one_copy, int widest, int narrowest, int64_t most_workgroups) {
        for (int V = widest; V >= narrowest; V /= 2) {
            // (planes that V does not divide have a last thread with fewer pixels: gate, 64x120 planes of 27x23, 40 + 101 us with one
            // pixel per thread, 18 + 37 with sixteen.  Not where four divide them: 64x64 planes of 14x14 8.9 + 19.3 with four, 9.6 + 18.8
            // with eight.  Nor where a workgroup holds all channels: there the estimate errs, one program over 9x96 planes of 23x17
            // took 126 us with two pixels, 38 with one)
            if (dag.W < V || (streams && dag.W % V != 0) || (HW % V != 0 && (all_channels || HW % 4 == 0))) continue;
            pg.vec = V;
            pg.unroll = unroll_for(pg.tm, V);
            pg.persist_copies = one_copy ? 1 : pg.unroll;
            const int PP = ceil_div(HW, V);                          // pixel threads of a plane
            const int64_t HT = (reach_px + V - 1) / V;               // halo, in pixel threads
            const int per_thread = std::max<int>(1, (int)lds_bytes_per_thread(pg));
            const int cap = (int)(std::min<int64_t>(max_threads_for(pg.tm), (int64_t)kMaxLdsBytes / per_thread) / 64 * 64);
            for (int pt = 64; pt <= cap; pt += 64) {
                int own = pt - 2 * (int)HT, ht = (int)HT;
                const int one_tile = PP + (whole_planes ? 0 : 2 * (int)HT);
                if (pt >= one_tile) {  // the whole plane in one tile: nothing comes from beside it
                    if (ceil_div(one_tile, 64) * 64 != pt) break;  // (counted once, at its own size)
                    own = PP;
                    if (whole_planes) ht = 0;
                } else if (own <= 0) {
                    continue;
                } else {
                    own = ceil_div(PP, ceil_div(PP, own));  // tiles evened out over the plane
                }
                for (int trips = 1; trips <= (all_channels ? 1 : 8); trips *= 2) {
                    const double cost = geometry_for(pg, dag, C, all_channels, one_trip, PP, ht, cap, own, pt, trips);
                    if (cost >= 0 && (int64_t)dag.N * pg.tiles * pg.chunks <= most_workgroups && (best_cost < 0 || cost < best_cost * 0.999)) {  // (ties: the wider vector, the smaller workgroup, fewer trips)
                        best_cost = cost;
                        best_shape = pg;
                    }
                    if (pg.chunks == 1) break;  // (more trips give the same shape)
                }
            }
        }
    };
    look(one_trip && one_copy, streams ? kMaxStreamVec : max_vec_for(pg.tm), streams ? kMinStreamVec : 1, INT64_MAX);
    if (!one_trip && one_copy && best_cost >= 0) look(true, best_shape.vec, best_shape.vec, 256);
    if (best_cost < 0) throw Fail{"tile, halo and persistent state do not fit one workgroup"};
    pg = best_shape;
    return best_cost;
}

}  // namespace

// A sum with a product of two registers, of all taps: one instruction, and a register less while it runs (OP_COUNT: gone).  With the softmax's
// gradient left in the accumulator (kSmT above) the program below takes three registers instead of four, which lets a workgroup hold
// a plane of 32x32 whole, two pixels per thread and no halo: 192 -> 109 us (97 with the gather of two pixels in registers).
void add_products(Program& pg) {
    for (int p = 0; p < pg.n_pass; p++)
        for (int i = pg.pass[p].body_begin; i + 3 < pg.pass[p].body_end; i++) {
            const Instr &keep = pg.ins[i], &get = pg.ins[i + 1], &mul = pg.ins[i + 2], &add = pg.ins[i + 3];
            if (keep.op != OP_MOVR || get.op != OP_MOVA || mul.op != OP_BIN || add.op != OP_BIN) continue;
            if (keep.T < 2 || get.T != keep.T || mul.T != keep.T || add.T != keep.T || add.r != keep.r || get.r == keep.r || mul.r == keep.r) continue;
            if ((mul.kind & ~kBinRegIsLhs) != kMul || (add.kind & ~kBinRegIsLhs) != kAdd) continue;
            bool read_on = false;  // (what was kept must not be needed again)
            for (int j = i + 4; j < pg.pass[p].body_end; j++) {
                const Instr& I = pg.ins[j];
                if (I.r == keep.r && I.op == OP_MOVR) break;
                if (I.r == keep.r && I.op != OP_LD && I.op != OP_ST) read_on = true;
                if (I.op == OP_MADD && I.a == keep.r) read_on = true;
            }
            if (read_on) continue;
            Instr m = get;
            m.op = OP_MADD;
            m.kind = 0;
            m.a = mul.r;
            pg.ins[i].op = pg.ins[i + 1].op = pg.ins[i + 2].op = OP_COUNT;
            pg.ins[i + 3] = m;
        }
}

// Fewer registers for a finished program: stores that nothing reads go, the others get the lowest register that is free where they stand (a
// register is as many bytes of LDS per thread as the instance has lanes, and LDS decides how many wavefronts a compute unit holds);
// where no register holds anything during a hand-over, its buffer takes their place.  Backward of unfold 3x3 -> softmax -> product ->
// gelu -> sum, 16x96 planes of 32x32: 280 -> 196 bytes per thread, 239 -> 192 us (97 with add_products).
// Not for programs that keep registers from pass to pass: those are left as they are.
void compact_registers(Emitter& E) {
    Program& pg = E.pg;
    auto reads = [](const Instr& I) {
        return I.op == OP_MADD || I.op == OP_MOVA || I.op == OP_BIN || I.op == OP_UNBX || I.op == OP_BING || I.op == OP_SMTBX || I.op == OP_FOLDBX || I.op == OP_SMCDOT || I.op == OP_SMCBX;
    };
    for (int p = 0; p < pg.n_pass; p++) {
        std::set<int> defined;
        for (int i = pg.pass[p].pro_begin; i < pg.pass[p].body_end; i++) {
            const Instr& I = pg.ins[i];
            if (reads(I) && !defined.count(I.r)) return;  // (a value from elsewhere)
            if (I.op != OP_MOVR) continue;
            if (i < pg.pass[p].body_begin) return;        // (a prologue's value holds for every channel of the body)
            defined.insert(I.r);
        }
    }
    if (pg.tm > 1) add_products(pg);
    std::vector<int> last_use(pg.n_instr, -1);  // of a store's value
    for (int p = 0; p < pg.n_pass; p++) {
        std::map<int, int> def;
        for (int i = pg.pass[p].body_begin; i < pg.pass[p].body_end; i++) {
            const Instr& I = pg.ins[i];
            if (reads(I)) last_use[def.at(I.r)] = i;
            if (I.op == OP_MADD) last_use[def.at(I.a)] = i;
            if (I.op == OP_MOVR) def[I.r] = i;
        }
    }
    std::vector<int> where(pg.n_instr, -1);
    std::map<int, int64_t> reach;
    int n = 0, n_regs = 0;
    bool alias = true;
    for (int p = 0; p < pg.n_pass; p++) {
        Pass& P = pg.pass[p];
        const int pro = P.pro_begin, body = P.body_begin, end = P.body_end;
        P.pro_begin = (uint16_t)n;
        std::map<int, int> color, until;  // of the value that a register holds; by color: its last use
        for (int i = pro; i < end; i++) {
            if (i == body) P.pro_end = P.body_begin = (uint16_t)n;
            Instr I = pg.ins[i];
            if (I.op == OP_COUNT) continue;
            if (I.op == OP_MOVR) {
                if (last_use[i] < 0) continue;
                int c = 0;
                while (until.count(c) && until[c] > i) c++;
                color[I.r] = c;
                until[c] = last_use[i];
                n_regs = std::max(n_regs, c + 1);
                I.r = (uint8_t)c;
            } else if (reads(I)) {
                I.r = (uint8_t)color[I.r];
                if (I.op == OP_MADD) I.a = (uint16_t)color[I.a];
            } else if (I.op == OP_XADD) {
                for (const auto& u : until)
                    if (u.second > i) alias = false;
                reach[n] = E.reach_of[i];
            }
            where[i] = n;
            pg.ins[n++] = I;
        }
        if (body == end) P.pro_end = P.body_begin = (uint16_t)n;
        P.body_end = (uint16_t)n;
    }
    pg.n_instr = n;
    pg.n_regs = n_regs;
    pg.xadd_alias = alias ? 1 : 0;
    E.reach_of = reach;
    for (ExtRef& r : E.ext)
        if (r.store_instr >= 0) r.store_instr = where[r.store_instr];
}

// Windows whose taps are folded right away (an elementwise function of a window's tap, of the pixel's own values and of a second window's tap,
// under sum, avg or max): OP_LD ... OP_FOLD becomes one OP_LDFOLD.  Done only where no instruction over taps is left: the program then
// runs on the instances without taps, with up to 16 pixels per thread instead of one or two.
// The lanes of A and of the registers are followed symbolically; what computes lanes is not emitted, what computes one lane is.
class Streamer {
   public:
    explicit Streamer(const Program& p) : in_(p), out_(p) {}
    bool run(std::vector<ExtRef>& refs) {
        bool any = false;
        std::vector<int> where(in_.n_instr, -1);
        out_.n_instr = 0;
        for (int p = 0; p < in_.n_pass; p++) {
            const Pass& P = in_.pass[p];
            Pass& Q = out_.pass[p];
            Q.pro_begin = (uint16_t)out_.n_instr;
            for (int i = P.pro_begin; i < P.pro_end; i++) {
                if (in_.ins[i].T > 1) return false;
                where[i] = push(in_.ins[i]);
            }
            Q.pro_end = Q.body_begin = (uint16_t)out_.n_instr;
            a_ = Value();
            for (int i = P.body_begin; i < P.body_end; i++) {
                if (!step(in_.ins[i], any)) return false;
                where[i] = out_.n_instr - 1;
            }
            Q.body_end = (uint16_t)out_.n_instr;
        }
        if (!any) return false;
        out_.tm = 1;
        out_.n_regs = 0;
        for (int i = 0; i < out_.n_instr; i++) {
            const Opcode op = (Opcode)out_.ins[i].op;
            if (op == OP_MOVR || op == OP_MOVA || op == OP_BIN || op == OP_UNBX || op == OP_BING || op == OP_FOLDBX || op == OP_SMCDOT || op == OP_SMCBX || op == OP_SMTBX)
                out_.n_regs = std::max(out_.n_regs, out_.ins[i].r + 1);
        }
        for (ExtRef& r : refs)
            if (r.store_instr >= 0) r.store_instr = where[r.store_instr];
        return true;
    }
    const Program& result() const { return out_; }

   private:
    struct Value {
        enum Kind { kOne, kWin, kSpread, kBlend } kind = kOne;  // one lane (or nothing), a window, a register's lane in every tap, a blend
        Instr win, win2;           // the window loads
        int before = -1;           // unary of the window's taps
        int blend = -1;
        bool tap_is_lhs = true, second = false;
        // the other operand, or what is spread: a register's lane (`version` of it), or a lane loaded from a tensor
        int reg = -1, version = 0, divisor = 0;
        bool from_ext = false;
        Instr load;
        int T = 1;
    };
    int push(const Instr& I) {
        out_.ins[out_.n_instr] = I;
        return out_.n_instr++;
    }
    static int as_unary(const Instr& I) { return I.kind == 0 || I.kind == 1 || I.kind == 2 || I.kind == kUnNeg ? I.kind : -1; }
    bool blend_with(Value& a, int kind, bool tap_is_lhs) {
        if (a.kind != Value::kWin || a.blend >= 0 || (kind != kAdd && kind != kMul && kind != kSub)) return false;
        a.kind = Value::kBlend;
        a.blend = kind;
        a.tap_is_lhs = tap_is_lhs;
        return true;
    }
    bool step(const Instr& I, bool& any) {
        switch (I.op) {
        case OP_LD:
            if (I.T == 1) break;
            if (!(I.kind & kWin) || (I.kind & kExtTaps) || in_.ext[I.a].T != 1 || (I.b & 255) || ((I.r & 15) != 3 && (I.r & 15) != 5)) return false;
            a_ = Value();
            a_.kind = Value::kWin;
            a_.win = I;
            a_.T = I.T;
            return true;
        case OP_UN: {
            if (a_.kind == Value::kOne) break;
            const int u = as_unary(I);
            if (u < 0 || I.T != a_.T) return false;
            if (a_.kind == Value::kWin && a_.before < 0) a_.before = u;
            else return false;
            return true;
        }
        case OP_MOVR:
            if (a_.kind == Value::kOne) {
                version_[I.r]++;
                r_[I.r] = Value();
                if (I.T != 1) return false;
                break;
            }
            if (I.T != a_.T) return false;
            r_[I.r] = a_;  // (nothing is written: a lane that the register held stays there)
            return true;
        case OP_MOVA:
            a_ = r_[I.r];
            if (a_.kind != Value::kOne) return I.T == a_.T;
            if (I.T != 1) return false;
            break;
        case OP_BIN: {
            const bool reg_lhs = I.kind & kBinRegIsLhs, reg_one = I.kind & kBinRegScalar, acc_one = I.kind & kBinAccScalar;
            const Value& r = r_[I.r];
            if (I.T == 1) {
                if (a_.kind != Value::kOne || r.kind != Value::kOne) return false;
                break;
            }
            if (acc_one) return false;
            if (reg_one || r.kind == Value::kSpread) {  // lanes with one lane of a register
                if (a_.T != I.T || !blend_with(a_, I.kind & 7, !reg_lhs)) return false;
                if (reg_one) {
                    if (r.kind != Value::kOne) return false;
                    a_.reg = I.r;
                    a_.version = version_[I.r];
                } else {
                    if (r.from_ext || r.T != I.T) return false;
                    a_.reg = r.reg;
                    a_.version = r.version;
                    a_.divisor = r.divisor;
                }
                return true;
            }
            if (r.kind == Value::kWin && r.before < 0 && r.win.r == a_.win.r && r.T == I.T && a_.T == I.T) {  // two windows
                if (!blend_with(a_, I.kind & 7, !reg_lhs)) return false;
                a_.second = true;
                a_.win2 = r.win;
                return true;
            }
            return false;
        }
        case OP_BINLD: {
            if (I.T == 1) {
                if (a_.kind != Value::kOne) return false;
                break;
            }
            const bool loaded_lhs = I.kind & kBinLdLoadedIsLhs;
            if (a_.T != I.T || !blend_with(a_, I.kind >> kBinLdKindShift & 7, !loaded_lhs)) return false;
            Instr L;
            L.op = OP_LD;
            L.kind = I.kind & (kWin | kExtTaps);
            L.a = I.a;
            L.b = I.b;
            L.r = I.r;
            L.T = 1;
            if (I.kind & kBinLdLoadedScalar) {
                if (L.kind) return false;
                a_.from_ext = true;
                a_.load = L;
                return true;
            }
            if (L.kind != kWin || in_.ext[I.a].T != 1 || I.r != a_.win.r || (I.b & 255)) return false;
            L.T = I.T;
            a_.second = true;
            a_.win2 = L;
            return true;
        }
        case OP_FOLDBX: {  // a register's lane spread over the taps
            const Value& r = r_[I.r];
            if (r.kind != Value::kOne || I.kind == 2 || I.T == 1) return false;
            a_ = Value();
            a_.kind = Value::kSpread;
            a_.reg = I.r;
            a_.version = version_[I.r];
            a_.divisor = I.kind == 1 ? I.T : 0;
            a_.T = I.T;
            return true;
        }
        case OP_FOLD: {
            if (I.T == 1 || I.T != a_.T || (a_.kind != Value::kWin && a_.kind != Value::kBlend)) return false;
            if (a_.from_ext) push(a_.load);
            else if (a_.reg >= 0) {
                if (version_[a_.reg] != a_.version) return false;  // (overwritten in between)
                Instr m;
                m.op = a_.divisor ? OP_FOLDBX : OP_MOVA;
                m.T = 1;
                m.r = (uint8_t)a_.reg;
                m.kind = a_.divisor ? 1 : 0;
                m.f0 = (float)a_.divisor;
                push(m);
            }
            Instr f;
            f.op = OP_LDFOLD;
            f.T = I.T;
            f.a = a_.win.a;
            f.r = a_.win.r;
            f.kind = (uint8_t)(I.kind & 3);
            if (a_.blend >= 0) f.kind |= (uint8_t)(kLfBlend | ((a_.blend == kSub && !a_.tap_is_lhs ? 3 : a_.blend) << kLfBlendShift));
            if (a_.second) {
                f.kind |= kLfSecond;
                f.b = a_.win2.a;
            }
            f.f0 = (float)a_.before;
            push(f);
            any = true;
            a_ = Value();
            return true;
        }
        default:
            if (I.T != 1 || a_.kind != Value::kOne || I.op == OP_XADD) return false;
            if ((I.op == OP_UNBX || I.op == OP_BING || I.op == OP_SMCDOT || I.op == OP_SMCBX) && r_[I.r].kind != Value::kOne) return false;
            break;
        }
        if (out_.n_instr >= kMaxInstr) return false;
        push(I);
        if (I.op == OP_LD) a_ = Value();
        return true;
    }
    const Program& in_;
    Program out_;
    Value a_;
    std::map<int, Value> r_;
    std::map<int, int> version_;
};

bool chain_candidate(const Dag& dag, int k) {
    const Node& nd = dag.nodes[k];
    if (k == 0 || !nd.live || nd.pooled || nd.T > 25 || nd.C > 65535) return false;
    const Node& A = dag.nodes[nd.a];
    if (A.pooled || A.T > 25) return false;
    switch (nd.op) {
    case Op::Unfold: return A.T == 1 && nd.kh * nd.kw <= 25 && (nd.kw == 1 || nd.kw == 3 || nd.kw == 5);
    case Op::Shift: return std::abs(nd.dh) < 32768 && std::abs(nd.dw) < 32768;
    case Op::Unary: return true;
    case Op::Binary: {
        const Node& B = dag.nodes[nd.b];
        return nd.bgroups == 1 && !nd.lhs_pixels && !B.pooled && A.C == B.C && B.T <= 25 && B.T % A.T == 0;
    }
    // (a softmax over the channels of a tensor with taps stays a kernel of its own on the materialised tensor: each of
    // its passes over the channel range would evaluate the whole window again, and backward hands T lanes over per channel
    // and pass; measured on the 200 random DAGs such chains took 1.2-2.5 ms where the kernels per node take 0.1-0.4 ms)
    case Op::Softmax: return (nd.kind == kAxisC && nd.T == 1) || nd.kind == kAxisT;
    case Op::Fold: return !nd.axis_hw && !nd.axis_c;
    default: return false;
    }
}

bool compile_unit(const Dag& dag, const std::vector<int>& nodes, const std::vector<bool>& is_output, bool variants, UnitPlan& out, std::string& why) {
    try {
        if (nodes.empty()) throw Fail{"empty unit"};
        std::vector<bool> in_unit(dag.nodes.size(), false);
        for (int k : nodes) in_unit[k] = true;
        const int C = dag.nodes[nodes[0]].C;
        for (int k : nodes)
            if (dag.nodes[k].C != C) throw Fail{"channel counts differ inside the unit"};
        Graph G(dag, in_unit, is_output);
        out = UnitPlan();
        out.nodes = nodes;
        std::vector<int> out_inst;
        for (int k : nodes)
            if (is_output[k]) {
                out.outputs.push_back(k);
                out_inst.push_back(G.build(k, 0));
            }
        if (out.outputs.empty()) throw Fail{"unit without an output"};
        const bool box = G.add_box_adjoints();  // (backward only: the forward program never evaluates what this adds)
        int lanes = 1;
        std::vector<int> smc, leaves;
        for (size_t i = 0; i < G.insts.size(); i++) {
            lanes = std::max(lanes, G.insts[i].lanes);
            if (G.insts[i].kind == kSmC) smc.push_back((int)i);
            if (G.insts[i].kind == kExt) {
                if (!(box && G.ctxs[G.insts[i].ctx].win)) leaves.push_back((int)i);  // (a box adjoint replaces the way through its window)
                if (std::find(out.inputs.begin(), out.inputs.end(), G.insts[i].node) == out.inputs.end()) out.inputs.push_back(G.insts[i].node);
            }
        }
        std::sort(out.inputs.begin(), out.inputs.end());
        for (int e : out.inputs)
            if (dag.nodes[e].C != C) throw Fail{"an external tensor with another channel count"};
        auto fits32 = [&](int k) { return (int64_t)dag.N * C * std::max(dag.nodes[k].T, 1) * dag.H * dag.W * 4 < ((int64_t)1 << 31); };
        for (int k : nodes)
            if (!fits32(k)) throw Fail{"a tensor beyond 32-bit byte offsets"};
        for (int k : out.inputs)
            if (!fits32(k)) throw Fail{"a tensor beyond 32-bit byte offsets"};
        if (lanes > 25) throw Fail{"more than 25 taps"};
        const int tm = lanes <= 1 ? 1 : (lanes <= 9 ? 9 : 25);

        // ------------------------------------------------------------ displaced units
        // The gradient of a leaf that reads an external tensor through Shift offsets belongs to another pixel.  Where the
        // unit has no reduction, the pixel fetches it itself: the whole unit is instantiated once more, displaced by
        // the negated offsets (every load of it, the incoming gradient included, moves with it), and the gradient of
        // the same leaf in that copy, masked where the displaced pixel leaves the image, is what this pixel's tensor
        // element receives.  No hand-over between threads, no halo, no barrier; windows keep the hand-over (OP_XADD),
        // one displaced copy per tap would cost more than it saves.
        struct Pull {
            std::unique_ptr<Graph> g;
            int leaf = -1, mask_ctx = -1;
        };
        std::map<int, Pull> pulls;  // by leaf instance of the unit's own graph
        for (int i : leaves) {
            const Ctx& c = G.ctxs[G.insts[i].ctx];
            if (c.empty() || c.win) continue;
            try {
                Pull P;
                P.g.reset(new Graph(dag, in_unit, is_output));
                Ctx d;
                for (const Term& t : c.terms) {
                    Term n = t;
                    n.dh = (int16_t)-t.dh;
                    n.dw = (int16_t)-t.dw;
                    d.terms.push_back(n);
                }
                P.g->root_ctx = P.g->ctx_id(d);
                P.mask_ctx = P.g->root_ctx;
                for (int k : out.outputs) P.g->build(k, P.g->root_ctx);
                Ctx full = d;  // the same leaf in the displaced copy: the displacement, then the leaf's own offsets
                for (const Term& t : c.terms) full.terms.push_back(t);
                const int want_ctx = P.g->ctx_id(full);
                for (size_t j = 0; j < P.g->insts.size(); j++)
                    if (P.g->insts[j].kind == kExt && P.g->insts[j].node == G.insts[i].node && P.g->insts[j].ctx == want_ctx &&
                        P.g->insts[j].lanes == G.insts[i].lanes)
                        P.leaf = (int)j;
                if (P.leaf >= 0) pulls[i] = std::move(P);
            } catch (const Fail&) {
            }
        }
        // ------------------------------------------------------------ the two programs
        auto emit_fwd = [&](Emitter& E) {
            E.stat_passes(smc);
            E.begin_pass();
            E.begin_body();
            for (size_t o = 0; o < out.outputs.size(); o++) {
                E.eval(out_inst[o]);
                Instr st = Emitter::simple(OP_ST, dag.nodes[out.outputs[o]].T, 0, 0, E.ext_slot(out.outputs[o], kValueOut));
                E.ext[st.a].store_instr = E.pg.n_instr;
                E.emit(st);
            }
            E.end_pass();
        };
        // Leaves read through a window whose gradient the source pixel fetches (Emitter::mirror), found by trying.
        std::set<int> mirrored;
        for (int i : leaves) {
            if (!variants || !G.ctxs[G.insts[i].ctx].win) continue;
            try {
                Emitter trial(G, tm);
                trial.mirror(i);
                mirrored.insert(i);
            } catch (const Fail&) {
            }
        }
        bool use_mirrors = false;
        auto emit_bwd = [&](Emitter& E) {
            E.stat_passes(smc);
            int deepest = 0;
            for (int i : smc) deepest = std::max(deepest, G.down(i));
            for (int d = 0; d <= deepest && !smc.empty(); d++) {  // the sums of gradient x output, outermost softmax first
                E.begin_pass();
                for (int i : smc)
                    if (G.down(i) == d) {
                        E.emit(Emitter::simple(OP_PSET, G.insts[i].lanes, 0, 0, E.dot_slot(i)));
                        E.reduce(E.dot_slot(i), G.insts[i].lanes, 1);
                    }
                E.begin_body();
                for (int i : smc)
                    if (G.down(i) == d) {
                        bool mine;
                        const int r = E.to_reg(i, 1, mine);
                        E.eval(i);
                        E.emit(Emitter::simple(OP_SMCDOT, G.insts[i].lanes, r, 0, E.dot_slot(i)));
                        if (mine) E.release(r);
                    }
                E.end_pass();
            }
            E.begin_pass();
            E.begin_body();
            for (int e : out.inputs) {
                std::vector<int> mine;
                for (int i : leaves)
                    if (G.insts[i].node == e) mine.push_back(i);
                const int Te = dag.nodes[e].T;
                const int slot = E.ext_slot(e, kGradOut);
                const bool direct = mine.size() == 1 && G.insts[mine[0]].ctx == 0 && G.insts[mine[0]].lanes == Te;
                // no hand-over among the leaves: their contributions are summed in a register instead of LDS floats
                bool local = !direct;
                for (int i : mine)
                    if (!(use_mirrors && mirrored.count(i)) && (G.insts[i].lanes != Te || (G.insts[i].ctx != 0 && !pulls.count(i)))) local = false;
                int acc = -1, racc = -1;
                if (!direct && !local) {
                    acc = E.persist(Te);
                    E.emit(Emitter::simple(OP_PSET, Te, 0, 0, acc));
                }
                bool first_term = true;
                auto add_term = [&](int lanes) {  // A holds one more contribution
                    if (local) {
                        if (!first_term) {
                            E.emit(Emitter::simple(OP_BIN, Te, racc, kAdd | kBinRegIsLhs));
                            E.release(racc);
                            racc = -1;
                        }
                        first_term = false;
                        return;
                    }
                    Instr p = Emitter::simple(OP_PADD, lanes, 0, 0, acc);
                    p.b = (uint16_t)Te;
                    E.emit(p);
                };
                for (size_t mi = 0; mi < mine.size(); mi++) {
                    const int i = mine[mi];
                    const Inst& L = G.insts[i];
                    if (local && !first_term) {  // (the sum so far waits in a register while the next term is computed)
                        racc = E.alloc();
                        E.emit(Emitter::simple(OP_MOVR, Te, racc));
                    }
                    if (use_mirrors && mirrored.count(i)) {
                        E.mirror(i);
                        add_term(1);
                        continue;
                    }
                    auto pl = pulls.find(i);
                    if (pl != pulls.end()) {  // fetched from the displaced copy of the unit
                        int idx = 1;
                        for (auto it = pulls.begin(); it != pl; ++it) idx++;
                        E.use(*pl->second.g, idx);
                        E.grad(pl->second.leaf);
                        E.emit(E.positional(OP_MASK, pl->second.mask_ctx, L.lanes));
                        E.forget_graph(idx);
                        E.use(G, 0);
                        add_term(L.lanes);
                        continue;
                    }
                    E.grad(i);
                    if (direct) break;
                    if (L.ctx == 0) {
                        add_term(L.lanes);
                    } else {
                        if (!G.ctxs[L.ctx].win && L.lanes != Te) throw Fail{"a shifted read of an external tensor with replicated taps"};
                        Instr x = E.positional(OP_XADD, L.ctx, L.lanes);
                        x.a = (uint16_t)acc;
                        if (Te > 1) x.kind |= kExtTaps;
                        E.reach_of[E.pg.n_instr] = G.ctxs[L.ctx].reach_px(dag.W);
                        E.emit(x);
                    }
                }
                if (!direct && !local) E.emit(Emitter::simple(OP_PLD, Te, 0, 0, acc));
                Instr st = Emitter::simple(OP_ST, Te, 0, 0, slot);
                E.ext[slot].store_instr = E.pg.n_instr;
                E.emit(st);
            }
            E.end_pass();
        };
        // A program is emitted with full recomputation first; then, greedily, the value or gradient whose repeated
        // computation costs the most is kept in a register, as long as that makes the program cheaper and the registers
        // last.  Returns the emitter of the cheapest program that could be emitted.
        auto shortest = [&](const std::function<void(Emitter&)>& emit_program, bool one_trip, int most_kept) {
            std::set<int> keep;
            auto best = std::make_shared<Emitter>(G, tm);
            best->one_trip = one_trip;
            emit_program(*best);  // (throws when even the plain program does not fit)
            for (int round = 0; round < most_kept; round++) {
                int pick = -1;
                double gain = 0;
                for (const auto& kv : best->stats) {
                    const double g = (kv.second.computed - 1) * (kv.second.cost - kv.second.lanes) - kv.second.lanes;  // (fetched instead; - the store)
                    if (!keep.count(kv.first) && g > gain) {
                        gain = g;
                        pick = kv.first;
                    }
                }
                if (pick < 0) break;
                keep.insert(pick);
                try {
                    auto E = std::make_shared<Emitter>(G, tm);
                    E->keep = keep;
                    E->one_trip = one_trip;
                    emit_program(*E);
                    if (E->weight >= best->weight) break;
                    best = E;
                } catch (const Fail&) {
                    break;
                }
            }
            return best;
        };
        // The variants of a program: backward also with the gradients of windows fetched by the source pixel, if that is
        // cheaper by instructions x halo (bit 1; a 5x5 window under a product and an avg fold, 16x96 planes of 32x32: 368 -> 200 us); with softmaxes over channels also with values kept across the passes
        // (bit 0), where the workgroup that suits the plain program has a thread for every channel anyway: 16x96 planes of
        // 32x32 forward + backward 19.9 + 38.7 -> 16.9 + 26.5 us; a workgroup chosen for it lost more than the passes gained
        // (128x64 planes of 56x56 backward 177 -> 252 us, 128x40 of 28x28 48.5 -> 75.4).  Where a chain is cut goes by the plain
        // programs.  Adds the plain program's cost to out.cost and, with a halo around whole planes too, to out.halo_cost.
        auto best_of = [&](const std::function<void(Emitter&)>& emit_program, bool backward, Program& pg, std::vector<ExtRef>& refs) {
            struct Shape {
                double estimate = 0;
                int vec = 0;
                bool suits(const Shape& plain) const { return estimate <= plain.estimate * 1.001 && vec == plain.vec; }
            };
            double best = -1;
            Shape packed, emitted;  // the workgroup of the best program; the one before its registers were packed
            for (int v = 0; v < 4; v++) {
                const bool one_trip = v & 1, mirrors = v & 2;
                if ((one_trip && (!variants || smc.empty())) || (mirrors && (!backward || mirrored.empty()))) continue;
                use_mirrors = mirrors;
                // (fewer kept values where their registers leave no room for the threads that one trip takes)
                for (int most_kept = regs_for(tm); most_kept >= (one_trip ? 1 : regs_for(tm)); most_kept--) {
                    try {
                        auto E = shortest(emit_program, one_trip, most_kept);
                        most_kept = std::min(most_kept, (int)E->keep.size());
                        int64_t halo = 0;
                        for (int i = 0; i < E->pg.n_instr; i++)  // (the reach of the hand-overs of the program that was chosen)
                            if (E->pg.ins[i].op == OP_XADD) halo = std::max(halo, E->reach_of[i]);
                        Program unpacked = E->pg;
                        if (!one_trip && variants) compact_registers(*E);
                        Shape shape, before;
                        shape.estimate = set_geometry(E->pg, dag, C, halo, !smc.empty(), one_trip);
                        shape.vec = E->pg.vec;
                        if (!one_trip && variants && !smc.empty()) {
                            try {
                                before.estimate = set_geometry(unpacked, dag, C, halo, true, false);
                                before.vec = unpacked.vec;
                            } catch (const Fail&) {
                            }
                        }
                        const double cost = program_cost(E->pg);
                        if (v == 0) {
                            out.cost += cost;
                            double halo_cost = cost;
                            if (!variants && halo > 0) {
                                try {
                                    set_geometry(unpacked, dag, C, halo, !smc.empty(), false, false);
                                    halo_cost = program_cost(unpacked);
                                } catch (const Fail&) {
                                    halo_cost = -1;
                                }
                            }
                            out.halo_cost = halo_cost < 0 || out.halo_cost < 0 ? -1 : out.halo_cost + halo_cost;
                        }
                        // (packed registers can leave room for a workgroup that suits the plain program better; where kept values suit the one before,
                        // the estimates of the launches decide: two softmaxes over 96 channels, 16 planes of 16x16, forward + backward 159 us with packed
                        // registers, 109 with kept values)
                        if (v == 0 || (cost < best && (!one_trip || shape.suits(packed) || (shape.suits(emitted) && launch_us(E->pg) < launch_us(pg))))) {
                            best = cost;
                            packed = shape;
                            emitted = before;
                            pg = E->pg;
                            refs = E->ext;
                        }
                        break;
                    } catch (const Fail&) {
                        if (v == 0) throw;
                    }
                }
            }
        };
        best_of(emit_fwd, false, out.fwd, out.fwd_ext);
        best_of(emit_bwd, true, out.bwd, out.bwd_ext);
        // (Pays off from a plane of 32 threads and 3.6 M taps on, with four pixels per thread from 7.2 M on: the channels of a trip go one after
        // the other here.  3x3 box, forward + backward, us with all lanes / streamed: 128x64 planes of 56x56 327 / 163, 16x96 of 32x32 33 / 17, 8x64 of
        // 56x56 32 / 17, 128x64 of 28x28 90 / 74, 16x64 of 28x28 20.8 / 20.3, 8x32 of 28x28 14.8 / 19.9, 128x128 of 8x8 26 / 40, 16x64 of 16x16 15.2 / 15.7; 5x5 under a product
        // and an avg fold, 16x96 of 32x32, forward 69 / 13, backward 159 / 20.)
        auto stream = [&](Program& pg, std::vector<ExtRef>& refs) {
            std::vector<ExtRef> r = refs;
            Streamer S(pg);
            if (!S.run(r)) return;
            try {
                Program q = S.result();
                set_geometry(q, dag, C, 0, !smc.empty(), false);
                const int64_t taps = (int64_t)dag.N * C * dag.H * dag.W * tm;
                if (dag.H * dag.W < 32 * q.vec || taps < (q.vec < kMaxStreamVec ? 7200000 : 3600000)) return;
                pg = q;
                refs = r;
            } catch (const Fail&) {
            }
        };
        if (variants && tm > 1) {
            stream(out.fwd, out.fwd_ext);
            stream(out.bwd, out.bwd_ext);
        }
        return true;
    } catch (const Fail& f) {
        why = f.why;
        return false;
    }
}

double launch_us(const Program& pg) {
    double weight = 0, instructions = 0;
    for (int p = 0; p < pg.n_pass; p++)
        for (int i = pg.pass[p].body_begin; i < pg.pass[p].body_end; i++) {
            weight += instr_weight(pg.ins[i]);
            instructions++;
        }
    const double trips = (double)ceil_div(pg.chunk, pg.slices * pg.unroll), rounds = rounds_of(pg);
    // threads that share a compute unit's vector units, of about 1024
    const double resident = pg.threads / 1024.0 * (rounds >= 1 ? workgroups_per_cu(pg) : std::min(1024.0 / pg.threads, (double)pg.N * pg.tiles * pg.chunks / 256.0));
    return std::max(1.0, std::ceil(rounds - 0.05)) * trips * (0.75 * instructions + 0.025 * weight * pg.unroll * (pg.vec * resident + 0.5));
}

double program_cost(const Program& pg) {
    double sum = 0;
    for (int p = 0; p < pg.n_pass; p++)
        for (int i = pg.pass[p].body_begin; i < pg.pass[p].body_end; i++) sum += instr_weight(pg.ins[i]);
    // pixels computed per pixel owned (the halo), and the serial walk over the channels where the workgroup's shape leaves
    // a thread more than 16 trips (a program that keeps all channels in one workgroup and has no LDS left for slices)
    const double halo = (double)pg.pix_threads / std::max(1, pg.own_threads + (pg.halo_threads > 0 ? 0 : pg.pix_threads - pg.own_threads));
    const double trips = std::ceil((double)pg.chunk / std::max(1, pg.slices * pg.unroll));
    return sum * halo * std::max(1.0, trips / 16.0);
}

std::string dump(const Program& pg) {
    static const char* names[] = {"LD", "MASK", "UN", "MOVR", "MOVA", "BIN", "FOLD", "SMT", "ST", "UNBX", "BING", "SMTBX", "FOLDBX",
                                  "PSET", "PADD", "PLD", "SMCSTAT", "SMCAPPLY", "SMCDOT", "SMCBX", "XADD", "BINLD", "LDFOLD", "MADD"};
    std::ostringstream os;
    os << "program: C=" << pg.C << " HxW=" << pg.H << "x" << pg.W << " vec=" << pg.vec << " own=" << pg.own_threads << " halo=" << pg.halo_threads
       << " unroll=" << pg.unroll << " tiles=" << pg.tiles << " chunk=" << pg.chunk << " slices=" << pg.slices << " threads=" << pg.threads << " persist=" << pg.n_persist
       << " lanes=" << pg.tm << "\n";
    for (int p = 0; p < pg.n_pass; p++) {
        os << " pass " << p << "\n";
        for (int i = pg.pass[p].pro_begin; i < pg.pass[p].body_end; i++) {
            const Instr& I = pg.ins[i];
            os << (i < pg.pass[p].pro_end ? "  pro  " : "  body ") << i << ": " << (I.op < OP_COUNT ? names[I.op] : "?") << " T=" << (int)I.T
               << " kind=" << (int)I.kind << " r=" << (int)I.r << " a=" << I.a << " b=" << I.b << " f0=" << I.f0 << "\n";
        }
    }
    return os.str();
}

}  // namespace chain
}  // namespace canvas
