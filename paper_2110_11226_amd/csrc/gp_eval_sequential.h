// gp_eval_sequential.h -- one program to the evaluation kernel's instruction
// stream (gp_eval_code.h) in the prefix list's own right-to-left order: for
// programs with user functions or a user loss, and for those too long or too
// deep for the wavefront-parallel compiler.  Host- and device-compilable, so
// that a check on the CPU runs the very same code.
#pragma once

#include <cstdint>

#include "gp_eval_code.h"
#include "gp_internal.h"

namespace gp {

constexpr int kEvalSlots = GP_MAX_STACK - 1;   // entries below the top
constexpr int kEvalLds = kEvalSlots - kRegSlots;
// with user functions or a user loss: the target below the program, and a
// definition's own GP_USER_MAX_STACK values above its arguments
constexpr int kEvalSlotsUser = GP_MAX_STACK + GP_USER_MAX_STACK;
constexpr int kEvalLdsUser = kEvalSlotsUser - kRegSlots;
constexpr int kCompileDepth = kEvalSlotsUser + 1;   // entries the compiler tracks
// A program's header word: bit 31, it has more than one block of 64
// instructions; bit 30, it reads features from memory, the first of which is
// the one in the low bits (kOpReload and the fetch chain of gp_eval_code.h).
constexpr uint32_t kHdrBlocks = 1u << 31, kHdrFetch = 1u << 30, kHdrFeature = (1u << 24) - 1u;

// Word pair of instruction q: every 64th is a kOpReload.
GP_HD int64_t code_pos(int64_t q) { return q + q / 63; }

// How the operations of a program map to handlers for one configuration of
// the evaluation kernel.
struct Emit {
    EvalOps ops;
    int32_t R;
    int32_t mem;        // features come from memory
    GP_HD uint32_t handler(uint32_t id) const { return id * kOpBytes; }
    // (the bound only keeps a malformed program within the table)
    GP_HD uint32_t source(bool is_c, uint32_t arg) const {
        return is_c ? 0u : (mem ? 1u : (arg + 1u < ops.n_src ? arg + 1u : ops.n_src - 1u));
    }
    GP_HD uint32_t set(uint32_t src) const { return handler(kOpSet + src); }
    GP_HD uint32_t push(uint32_t slot, uint32_t src) const { return handler(ops.push + slot * ops.n_src + src); }
    GP_HD uint32_t fold(uint32_t op, uint32_t src) const { return handler(ops.fold + op * ops.n_src + src); }
    GP_HD uint32_t bin(uint32_t op, uint32_t slot) const {
        return handler(ops.bin + op * (kRegSlots + 1) + slot);
    }
    GP_HD uint32_t lds(uint32_t slot) const { return (slot - kRegSlots) * static_cast<uint32_t>(R * 64 * 4); }
};

// The interpreter's operation for binary function index fn (ADD, SUB, MUL,
// DIV, MAX, MIN, ATAN2) with its operands as given, or exchanged.
GP_HD uint32_t bin_op(uint32_t fn, bool rev) {
    switch (fn) {
    case 0: return kBAdd;
    case 1: return rev ? kBSubRev : kBSub;
    case 2: return kBMul;
    case 3: return rev ? kBDivRev : kBDiv;
    case 4: return kBMax;
    case 5: return kBMin;
    default: return rev ? kBAtan2Rev : kBAtan2;
    }
}

GP_HD uint32_t float_bits(float v) {
    uint32_t u;
    __builtin_memcpy(&u, &v, sizeof u);
    return u;
}

// One program by one lane.  out.put(position, handler, payload) stores a word
// pair, out.payload(position, payload) changes its second word; unary(fn, x)
// and binary(fn, a, b) are the float32 functions of constant subtrees;
// sh.entry(e) (an unsigned word) and sh.value(e) (a float) are kCompileDepth
// entries of the caller's.  `room` is the program's in word pairs.
//
// Room: two word pairs per node, of the program (times the longest definition's
// nodes) and of the loss's definition.  A node takes at most two instructions,
// and only from kRegSlots entries on (one instruction and a transfer to or from
// LDS): a terminal that is pushed, or a binary function whose operands are both
// on the stack.  A terminal that is the first operand of a binary function takes
// at most two together with it, and a function of one argument one.  Follow
// first operands from a binary function down to one of those: each such walk
// spares an instruction, and no walk is longer than the entries from kRegSlots
// on (or, within a definition, its 32 nodes), so that at least one instruction
// in 63 is spared.  Those make room for the reload after every 63rd, and the
// nodes of the first kRegSlots entries for the end.  A definition of one node
// takes one instruction at most, as it need not keep its arguments.  (Only a
// malformed program, which callers are not to pass, could take more: its stream
// ends where its room does.)
template <typename Out, typename Shadow, typename Unary, typename Binary>
GP_HD void compile_sequential(const uint32_t* pn, const float* pc, int32_t L, Out& out, int64_t room, uint32_t* hdr,
                              const Emit& em, const UserDefs& ud, int32_t loss_fn, Shadow sh, Unary&& unary,
                              Binary&& binary) {
    int h = 0;                                // entries on the stack
    int64_t k = 0;                            // instructions emitted
    // those there is room for, with an end after them
    const int64_t limit = (room - 1) - (room - 1) / 64 - (room % 64 == 0 ? 1 : 0);
    int64_t last_fetch = -1;                  // the latest feature fetch (its payload names the next)
    uint32_t head = 0u;
    auto clampe = [](int e) { return e < 0 ? 0 : e < kCompileDepth ? e : kCompileDepth - 1; };
    auto emit = [&](uint32_t handler, uint32_t payload) {
        out.put(code_pos(k), handler, payload);
        ++k;
    };
    // an instruction whose handler consumes the fetched feature arg
    auto fetch = [&](uint32_t handler, uint32_t arg) {
        if (last_fetch >= 0) out.payload(code_pos(last_fetch), arg);
        else head |= kHdrFetch | (arg & kHdrFeature);
        last_fetch = k;
        emit(handler, 0xffffffffu);
    };
    // a terminal as entry e
    auto push = [&](int e, bool is_c, uint32_t arg, float v) {
        const uint32_t src = em.source(is_c, arg);
        uint32_t handler;
        if (e < 1) {
            handler = em.set(src);
        } else if (e - 1 < kRegSlots) {
            handler = em.push(static_cast<uint32_t>(e - 1), src);
        } else {
            emit(em.handler(kOpSaveL), em.lds(static_cast<uint32_t>(e - 1)));
            handler = em.set(src);
        }
        if (is_c) emit(handler, float_bits(v));
        else if (em.mem) fetch(handler, arg);
        else emit(handler, 0u);
    };
    // the top takes the value in entry src, below it
    auto load_s = [&](int src) {
        const uint32_t s = static_cast<uint32_t>(clampe(src));
        if (s < static_cast<uint32_t>(kRegSlots)) emit(em.handler(kOpLoadS + s), 0u);
        else emit(em.handler(kOpLoadTopL), em.lds(s));
    };
    // a copy of entry src as entry e
    auto push_s = [&](int e, int src) {
        if (e >= 1) {
            if (e - 1 < kRegSlots) emit(em.handler(kOpSave + static_cast<uint32_t>(e - 1)), 0u);
            else emit(em.handler(kOpSaveL), em.lds(static_cast<uint32_t>(e - 1)));
        }
        if (src != e - 1) load_s(src);        // (else the entry just covered)
    };
    // top (op) the entry in slot s, or with `rev` the operands exchanged
    auto bin_slot = [&](uint32_t fn, bool rev, int s) {
        uint32_t slot = static_cast<uint32_t>(clampe(s));
        if (slot >= static_cast<uint32_t>(kRegSlots)) {
            emit(em.handler(kOpLoadL), em.lds(slot));
            slot = kRegSlots;
        }
        emit(em.bin(bin_op(fn, rev), slot), 0u);
    };
    // The item source: the program right to left; while a user function is
    // expanded, its definition right to left.  (i: next program position;
    // uf: the function being expanded or -1, di its next position, call_h
    // the stack height when it began, call_ar its arity.)
    int32_t i = L - 1;
    int uf = -1, di = 0, call_h = 0, call_ar = 0;
    bool loss_pending = loss_fn >= 0;
    if (loss_pending) {
        // entry 0: the target, under the program's value
        emit(em.handler(kOpLoadY), 0u);
        sh.entry(0) = 0u;
        h = 1;
    }
    // end of an expansion: the value, in the top's registers, replaces the
    // arguments as the deepest one's entry
    auto finish = [&]() {
        const int base = clampe(call_h - call_ar);
        sh.entry(base) &= 0x7fffffffu;              // (that argument's start)
        h = base + 1;
        uf = -1;
    };
    auto call = [&](int u, int ar) {
        uf = u;
        di = ud.len[u] - 1;
        call_h = h;
        call_ar = ar;
        if (di != 0) return;
        // a definition of one node: an argument or a constant
        const uint32_t w = ud.nodes[u][0], arg = w >> 8;
        if ((w & 0xffu) == GP_OP_CONST) emit(em.set(em.source(true, 0u)), float_bits(ud.consts[u][arg & (GP_USER_MAX_CONSTS - 1)]));
        else if (arg > 0u) load_s(call_h - 1 - static_cast<int>(arg));     // (argument 0 is the top)
        finish();
    };
    for (;;) {
        if (k >= limit && (i >= 0 || uf >= 0 || loss_pending)) break;    // (an item takes two at most: the end's place may be lost)
        uint32_t w;
        bool in_def;
        if (uf >= 0) {
            if (di < 0) {
                finish();
                continue;
            }
            w = ud.nodes[uf][di];
            in_def = true;
        } else {
            if (i < 0) {
                if (!loss_pending) break;
                loss_pending = false;
                call(kUserFns / 2 + loss_fn, 2);   // the two-argument user functions follow the one-argument ones
                continue;
            }
            w = pn[i];
            in_def = false;
        }
        const uint32_t op = w & 0xffu;
        const uint32_t arg = w >> 8;
        if (!in_def && is_user_op(op)) {
            call(static_cast<int>(op - GP_OP_USER1), arity(op));
            --i;
            continue;
        }
        // position and the item before it in the same source (a terminal
        // fuses only with a built-in binary function of its own source)
        const int32_t pos = in_def ? di : i;
        const int32_t last = in_def ? ud.len[uf] - 1 : L - 1;
        const uint32_t prev = pos >= 1 ? ((in_def ? ud.nodes[uf][pos - 1] : pn[pos - 1]) & 0xffu) : 0u;
        const float cval = op == GP_OP_CONST ? (in_def ? ud.consts[uf][arg & (GP_USER_MAX_CONSTS - 1)] : pc[arg])
                                             : 0.0f;
        auto advance = [&](int n) {
            if (in_def) di -= n;
            else i -= n;
        };
        const int ar = arity(op);
        const int top = clampe(h - 1);
        if (in_def && op == GP_OP_VAR) {
            // argument `arg` of the function: entry call_h - 1 - arg
            const int src = call_h - 1 - static_cast<int>(arg);
            if (pos >= 1 && pos != last && is_builtin_binary(prev)) {
                // first operand of the binary function before it; the top is the second
                bin_slot(binary_index(prev), true, src);
                sh.entry(top) &= 0x7fffffffu;
                di -= 2;
            } else {
                const int e = clampe(h);
                sh.entry(e) = static_cast<uint32_t>(k);
                push_s(e, src);
                ++h;
                --di;
            }
            continue;
        }
        if (ar == 1) {
            if (h >= 1 && (sh.entry(top) >> 31)) {
                // a unary function of a constant: its push (the last
                // instruction) takes the value
                sh.value(top) = unary(unary_index(op), sh.value(top));
                if (k >= 1) out.payload(code_pos(k - 1), float_bits(sh.value(top)));
            } else {
                emit(em.handler(kOpUnary + unary_index(op)), 0u);
            }
            advance(1);
            continue;
        }
        if (ar == 0) {
            const bool is_c = op == GP_OP_CONST;
            if (pos >= 1 && pos != last && is_builtin_binary(prev) && h >= 1) {
                // first operand of the binary function before it; the top is the second
                const uint32_t fn = binary_index(prev);
                const uint32_t e2 = sh.entry(top);
                if (is_c && (e2 >> 31)) {
                    const float v = binary(fn, cval, sh.value(top));
                    k = static_cast<int64_t>(e2 & 0x7fffffffu);   // drop the operand's instructions
                    push(top, true, 0u, v);
                    sh.value(top) = v;
                } else {
                    const uint32_t handler = em.fold(bin_op(fn, false), em.source(is_c, arg));
                    if (is_c) emit(handler, float_bits(cval));
                    else if (em.mem) fetch(handler, arg);
                    else emit(handler, 0u);
                    sh.entry(top) = e2 & 0x7fffffffu;
                }
                advance(2);
                continue;
            }
            const int e = clampe(h);
            sh.entry(e) = static_cast<uint32_t>(k) | (is_c ? 1u << 31 : 0u);
            sh.value(e) = cval;
            push(e, is_c, arg, cval);
            ++h;
            advance(1);
            continue;
        }
        // binary, operands not fused: the first is the top (entry h-1), the
        // second the entry below it (slot h-2)
        const int e1 = clampe(h - 1), e2 = clampe(h - 2);
        const uint32_t first = sh.entry(e1), second = sh.entry(e2);
        const uint32_t fn = binary_index(op);
        if ((first >> 31) && (second >> 31)) {
            const float v = binary(fn, sh.value(e1), sh.value(e2));
            k = static_cast<int64_t>(second & 0x7fffffffu);
            push(e2, true, 0u, v);
            sh.value(e2) = v;
        } else {
            bin_slot(fn, false, e2);
            sh.entry(e2) = second & 0x7fffffffu;
        }
        h = h > 0 ? h - 1 : 0;
        advance(1);
    }
    if (room < 1) {                           // (no nodes)
        *hdr = 0u;
        return;
    }
    const int64_t end = k <= limit ? code_pos(k) : room - 1;
    out.put(end, em.handler(kOpEnd), 0u);
    for (int64_t b = 63; b < end; b += 64) out.put(b, em.handler(kOpReload), 0u);
    if (end >= 64) head |= kHdrBlocks;
    *hdr = head;
}

}  // namespace gp
