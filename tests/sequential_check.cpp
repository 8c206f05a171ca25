// sequential_check.cpp -- compile_sequential (gp_eval_sequential.h) on the CPU:
// every word it stores lies within its program's room in the instruction
// stream, and the stream, run by a plain interpreter of gp_eval_code.h's
// instructions, gives the value of the prefix list evaluated directly.
//
//   sequential_check chains     long runs of user calls on a deep stack
//   sequential_check random N   N random programs with random definitions
//   sequential_check malformed N   N lists that are no programs: their words
//                               stay in their room too, and their streams end
// Prints the number of programs checked, or the first fault and exit status 1.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "gp_eval_sequential.h"

using namespace gp;
using Words = std::vector<uint32_t>;

static uint32_t node(uint32_t op, uint32_t arg = 0) { return GP_NODE(op, arg); }

// Any fixed float functions will do: both sides call these.
static float un(uint32_t fn, float x) {
    switch (fn) {
    case 0: return -x;
    case 1: return std::fabs(x) > 0.001f ? 0.3f + 0.1f * x : 0.0f;
    case 2: return std::sqrt(std::fabs(x));
    case 6: return std::fabs(x);
    default: return 0.5f * x + 0.01f * static_cast<float>(fn);
    }
}
static float bi(uint32_t fn, float a, float b) {
    switch (fn) {
    case 0: return a + b;
    case 1: return a - b;
    case 2: return a * b;
    case 3: return std::fabs(b) > 0.001f ? a / b : 1.0f;
    case 4: return std::max(a, b);
    case 5: return std::min(a, b);
    default: return a - 0.25f * b;
    }
}

struct Shadow {
    uint32_t e[kCompileDepth] = {};
    float v[kCompileDepth] = {};
    uint32_t& entry(int i) { return e[i]; }
    float& value(int i) { return v[i]; }
};

struct Check {
    Words prog;
    std::vector<float> consts;
    UserDefs ud{};
    int loss = -1;
    std::vector<float> X = {0.7f, -1.3f, 0.2f};
    float y = 0.4f;

    int mul() const {
        int m = 1;
        for (int u = 0; u < kUserFns; ++u) m = std::max(m, ud.len[u]);
        return m;
    }
    int64_t room() const {
        return 2 * (static_cast<int64_t>(prog.size()) * mul() + (loss >= 0 ? 1 + ud.len[kUserFns / 2 + loss] : 0));
    }
    void define(uint32_t op, const Words& def, const std::vector<float>& c) {
        const int u = static_cast<int>(op - GP_OP_USER1);
        ud.len[u] = static_cast<int>(def.size());
        std::copy(def.begin(), def.end(), ud.nodes[u]);
        std::copy(c.begin(), c.end(), ud.consts[u]);
    }

    // ---- the prefix list itself ----
    float walk(const uint32_t* w, int n, const float* c, const float* vars) const {
        std::vector<float> st;
        for (int i = n - 1; i >= 0; --i) {
            const uint32_t op = GP_NODE_OP(w[i]), arg = GP_NODE_ARG(w[i]);
            if (op == GP_OP_VAR) st.push_back(vars[arg]);
            else if (op == GP_OP_CONST) st.push_back(c[arg]);
            else {
                const float a = st.back();
                float b = 0.0f;
                if (arity(op) == 2) b = st[st.size() - 2];
                st.resize(st.size() - static_cast<size_t>(arity(op)));
                if (is_user_op(op)) {
                    const int u = static_cast<int>(op - GP_OP_USER1);
                    const float args[2] = {a, b};
                    st.push_back(walk(ud.nodes[u], ud.len[u], ud.consts[u], args));
                } else {
                    st.push_back(arity(op) == 1 ? un(unary_index(op), a) : bi(binary_index(op), a, b));
                }
            }
        }
        return st.back();
    }
    float direct() const {
        const float v = walk(prog.data(), static_cast<int>(prog.size()), consts.data(), X.data());
        if (loss < 0) return v;
        const int u = kUserFns / 2 + loss;
        const float args[2] = {v, y};
        return walk(ud.nodes[u], ud.len[u], ud.consts[u], args);
    }

    // ---- the stream ----
    struct Out {
        std::vector<uint32_t> h, p;
        int64_t room = 0, worst = -1;
        void put(int64_t q, uint32_t handler, uint32_t pay) {
            worst = std::max(worst, q);
            if (q < 0 || q >= room) return;
            h[static_cast<size_t>(q)] = handler;
            p[static_cast<size_t>(q)] = pay;
        }
        void payload(int64_t q, uint32_t pay) {
            worst = std::max(worst, q);
            if (q >= 0 && q < room) p[static_cast<size_t>(q)] = pay;
        }
    };
    float run(const Out& o, uint32_t head, const Emit& em, bool* fine) const {
        float t = y, m = 0.0f;
        std::vector<float> slot(kRegSlots, 0.0f), lds(kEvalLdsUser, 0.0f);
        int32_t next = head & kHdrFetch ? static_cast<int32_t>(head & kHdrFeature) : -1;
        const EvalOps& ops = em.ops;
        auto src = [&](uint32_t q, uint32_t pay) {
            if (q == 0) {
                float v;
                std::memcpy(&v, &pay, 4);
                return v;
            }
            if (!em.mem) return X[q - 1];
            if (next < 0) *fine = false;
            const float v = X[static_cast<size_t>(std::max(next, 0))];
            next = static_cast<int32_t>(pay);
            return v;
        };
        auto op = [&](uint32_t f, float tv, float x, bool fold) {   // top (op) slot, or source (op) top
            const float a = fold ? x : tv, b = fold ? tv : x;
            switch (f) {
            case kBAdd: return bi(0, a, b);
            case kBSub: return bi(1, a, b);
            case kBSubRev: return bi(1, b, a);
            case kBMul: return bi(2, a, b);
            case kBDiv: return bi(3, a, b);
            case kBDivRev: return bi(3, b, a);
            case kBMax: return bi(4, a, b);
            case kBMin: return bi(5, a, b);
            case kBAtan2: return bi(6, a, b);
            default: return bi(6, b, a);
            }
        };
        const uint32_t n = ops.n_src;
        for (int64_t q = 0; q < o.room; ++q) {
            if (o.h[static_cast<size_t>(q)] % kOpBytes) {
                *fine = false;
                return t;
            }
            const uint32_t id = o.h[static_cast<size_t>(q)] / kOpBytes, pay = o.p[static_cast<size_t>(q)];
            if ((q % 64 == 63) != (id == kOpReload)) *fine = false;
            const size_t at = pay / static_cast<uint32_t>(em.R * 256);
            if (id == kOpEnd) return t;
            if (id == kOpReload) continue;
            if (id == kOpLoadY) {
                if (q != 0) *fine = false;
            } else if (id == kOpSaveL || id == kOpLoadTopL || id == kOpLoadL) {
                if (at >= lds.size()) {
                    *fine = false;
                    return t;
                }
                if (id == kOpSaveL) lds[at] = t;
                else (id == kOpLoadTopL ? t : m) = lds[at];
            } else if (id < kOpSave) t = un(id - kOpUnary, t);
            else if (id < kOpLoadS) slot[id - kOpSave] = t;
            else if (id < kOpSet) t = slot[id - kOpLoadS];
            else if (id < ops.push) t = src(id - kOpSet, pay);
            else if (id < ops.fold) {
                slot[(id - ops.push) / n] = t;
                t = src((id - ops.push) % n, pay);
            } else if (id < ops.bin) t = op((id - ops.fold) / n, t, src((id - ops.fold) % n, pay), true);
            else {
                const uint32_t s = (id - ops.bin) % (kRegSlots + 1);
                t = op((id - ops.bin) / (kRegSlots + 1), t, s < kRegSlots ? slot[s] : m, false);
            }
        }
        *fine = false;      // no end
        return t;
    }

    // Compiles and runs the program for every kind of feature source (a
    // malformed one: compiles, and looks for the end).
    bool check(const char* what, bool malformed = false) {
        for (int freg : {0, 2, 8})
            for (int R : {1, 4}) {
                if (freg == 2 && X.size() > 2) continue;
                const Emit em{eval_ops(freg), R, freg == 0};
                Out o;
                o.room = room();
                o.h.assign(static_cast<size_t>(o.room), 0xdeadbeefu);
                o.p.assign(static_cast<size_t>(o.room), 0u);
                uint32_t head = 0;
                Shadow sh;
                compile_sequential(prog.data(), consts.data(), static_cast<int32_t>(prog.size()), o, room(), &head, em, ud, loss,
                                   sh, un, bi);
                if (o.worst >= o.room) {
                    std::printf("%s: %zu nodes, word pair %lld stored, room for %lld\n", what, prog.size(),
                                static_cast<long long>(o.worst), static_cast<long long>(o.room));
                    return false;
                }
                if (malformed) {
                    if (std::find(o.h.begin(), o.h.end(), kOpEnd * kOpBytes) == o.h.end()) {
                        std::printf("%s: %zu nodes, no end\n", what, prog.size());
                        return false;
                    }
                    for (size_t q = 0; o.h[q] != kOpEnd * kOpBytes; ++q)
                        if (o.h[q] % kOpBytes || o.h[q] / kOpBytes >= em.ops.bin + 10u * (kRegSlots + 1)) {
                            std::printf("%s: %zu nodes, word %zu is no handler\n", what, prog.size(), q);
                            return false;
                        }
                    continue;
                }
                bool fine = true;
                const float got = run(o, head, em, &fine), want = direct();
                if (!fine || (std::memcmp(&got, &want, 4) != 0 && !(std::isnan(got) && std::isnan(want)))) {
                    std::printf("%s: %zu nodes, freg %d: %a instead of %a%s\n", what, prog.size(), freg, got, want,
                                fine ? "" : " (malformed stream)");
                    return false;
                }
            }
        return true;
    }
};

// A random valid prefix list of about n nodes whose right-to-left scan holds at
// most `peak` values; terminals 0 .. nv-1 and the constants.
static Words random_list(std::mt19937& g, int n, int peak, int nv, int nc, const std::vector<uint32_t>& un_ops,
                         const std::vector<uint32_t>& bi_ops, double deep) {
    auto pick = [&](int k) { return static_cast<uint32_t>(std::uniform_int_distribution<int>(0, k - 1)(g)); };
    auto chance = [&](double p) { return std::uniform_real_distribution<double>(0, 1)(g) < p; };
    Words r;      // right to left
    int h = 0;
    while (static_cast<int>(r.size()) < n || h != 1) {
        const bool closing = static_cast<int>(r.size()) >= n;
        if (h == 0 || (!closing && h < peak && chance(deep)))
            r.push_back(nc && chance(0.3) ? node(GP_OP_CONST, pick(nc)) : node(GP_OP_VAR, pick(nv))), ++h;
        else if (h >= 2 && (closing || chance(0.6))) r.push_back(node(bi_ops[pick(static_cast<int>(bi_ops.size()))])), --h;
        else r.push_back(node(un_ops[pick(static_cast<int>(un_ops.size()))]));
    }
    std::reverse(r.begin(), r.end());
    return r;
}

// `calls` calls of a one-argument function (or two-argument ones on the chain
// and a feature) on a stack already `depth` deep.
static Words chain(uint32_t op, int calls, int depth) {
    Words w(static_cast<size_t>(depth), node(GP_OP_SUB));
    for (int i = 0; i < calls; ++i) {
        w.push_back(node(op));
        if (arity(op) == 2) w.push_back(node(GP_OP_VAR, 1));
    }
    w.push_back(node(GP_OP_VAR, 0));
    w.insert(w.end(), static_cast<size_t>(depth), node(GP_OP_VAR, 1));
    return w;
}

static int chains() {
    const uint32_t u1 = GP_OP_USER1, u2 = GP_OP_USER2, A = node(GP_OP_VAR, 0), B = node(GP_OP_VAR, 1),
                   C = node(GP_OP_CONST, 0), add = node(GP_OP_ADD), mul = node(GP_OP_MUL), sub = node(GP_OP_SUB);
    struct Def {
        uint32_t op;
        Words w;
    };
    std::vector<Def> defs = {{u1, {A}}, {u1, {add, A, C}}, {u1, {add, A, A}}, {u1, {sub, C, A}}, {u1, {node(GP_OP_SQRT), A}},
                             {u1, {add, mul, A, A, sub, A, C}}, {u1, {C}}, {u2, {A}}, {u2, {B}}, {u2, {add, A, B}},
                             {u2, {sub, B, A}}, {u2, {add, mul, A, B, sub, B, A}}, {u2, {node(GP_OP_SQRT), B}}};
    Words nested;       // right-nested: every first operand a terminal
    for (int i = 0; i < 15; ++i) {
        nested.push_back(sub);
        nested.push_back(i & 1 ? A : C);
    }
    nested.push_back(A);
    defs.push_back({u1, nested});
    // and the densest of many: as few terminals that are first operands as the stack allows
    std::mt19937 g(11);
    const std::vector<uint32_t> un_ops = {GP_OP_NEG, GP_OP_SQRT}, bi_ops = {GP_OP_ADD, GP_OP_SUB, GP_OP_DIV};
    for (int i = 0; i < 120; ++i) {
        Words d;
        const uint32_t op = i & 1 ? u1 : u2;
        do d = random_list(g, 1 + static_cast<int>(g() % 31), 1 + static_cast<int>(g() % GP_USER_MAX_STACK), op == u1 ? 1 : 2, 1, un_ops, bi_ops, 0.9);
        while (d.size() > GP_USER_MAX_NODES);
        defs.push_back({op, d});
    }
    int n = 0;
    for (const Def& d : defs)
        for (int calls : {1, 100, 2000})
            for (int depth : {0, 11, 12, 18})
                for (int loss : {-1, 0}) {
                    Check c;
                    c.X = {0.7f, -1.3f};
                    c.consts = {0.5f};
                    c.define(d.op, d.w, {0.25f});
                    if (loss >= 0) {
                        if (d.op == u2) continue;
                        c.define(u2, {mul, sub, A, B, sub, A, B}, {});
                        c.loss = 0;
                    }
                    c.prog = chain(d.op, calls, depth);
                    if (!c.check("chain")) return 1;
                    ++n;
                }
    std::printf("%d programs\n", n);
    return 0;
}

static int random_programs(int n) {
    std::mt19937 g(7);
    const std::vector<uint32_t> un_ops = {GP_OP_NEG, GP_OP_LOG, GP_OP_SQRT, GP_OP_SIN, GP_OP_ABS, GP_OP_SQ, GP_OP_CBRT};
    const std::vector<uint32_t> bi_ops = {GP_OP_ADD, GP_OP_SUB, GP_OP_MUL, GP_OP_DIV, GP_OP_MAX, GP_OP_MIN, GP_OP_ATAN2};
    for (int i = 0; i < n; ++i) {
        Check c;
        if (i & 1) c.X.resize(2);
        for (int k = 0; k < 6; ++k) c.consts.push_back(std::uniform_real_distribution<float>(-1, 1)(g));
        std::vector<uint32_t> us = un_ops, bs = bi_ops;
        for (uint32_t op : {24u, 25u, 28u, 29u}) {
            if (g() % 4 == 0) continue;
            Words d;
            do d = random_list(g, 1 + static_cast<int>(g() % 28), 1 + static_cast<int>(g() % GP_USER_MAX_STACK), op < 28 ? 1 : 2, 3, un_ops, bi_ops, 0.5);
            while (d.size() > GP_USER_MAX_NODES);
            c.define(op, d, {0.3f, -0.7f, 1.1f});
            for (int k = 0; k < 4; ++k) (op < 28 ? us : bs).push_back(op);
        }
        if (c.ud.len[kUserFns / 2] > 0 && g() % 3 == 0) c.loss = 0;
        c.prog = random_list(g, 1 + static_cast<int>(g() % (i % 16 ? 60 : 3000)), 1 + static_cast<int>(g() % GP_MAX_STACK),
                             static_cast<int>(c.X.size()), 6, us, bs, 0.3 + 0.6 * (g() % 8) / 7.0);
        if (!c.check("random")) return 1;
    }
    std::printf("%d programs\n", n);
    return 0;
}

// Words no population may hold: too few operands, too many, unknown functions,
// features out of range.
static int malformed_programs(int n) {
    std::mt19937 g(13);
    {
        Check c;                 // no nodes, no room: nothing stored
        Check::Out o;
        o.room = 0;
        uint32_t head = 1u;
        compile_sequential(c.prog.data(), c.consts.data(), 0, o, 0, &head, Emit{eval_ops(0), 1, 1}, c.ud, -1, Shadow{}, un, bi);
        if (o.worst >= 0 || head != 0u) {
            std::printf("empty: a word stored\n");
            return 1;
        }
    }
    for (int i = 0; i < n; ++i) {
        Check c;
        c.X.resize(2);
        c.consts.assign(256, 0.5f);
        c.define(GP_OP_USER1, {node(GP_OP_ADD), node(GP_OP_VAR, 0), node(GP_OP_CONST, 0)}, {0.25f});
        const int L = 1 + static_cast<int>(g() % (i % 8 ? 40 : 3000));
        const int kind = i % 4;
        for (int k = 0; k < L; ++k) {
            if (kind == 0) c.prog.push_back(node(GP_OP_VAR, g() % 2));
            else if (kind == 1) c.prog.push_back(node(GP_OP_ADD));
            else c.prog.push_back(node(g() % (kind == 2 ? GP_OP_LIMIT : 256u), g() % 256));
        }
        if (!c.check("malformed", true)) return 1;
    }
    std::printf("%d programs\n", n);
    return 0;
}

int main(int argc, char** argv) {
    if (argc > 2 && !std::strcmp(argv[1], "malformed")) return malformed_programs(std::atoi(argv[2]));
    if (argc > 1 && !std::strcmp(argv[1], "chains")) return chains();
    return random_programs(argc > 2 ? std::atoi(argv[2]) : 2000);
}
