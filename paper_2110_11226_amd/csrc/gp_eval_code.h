// Generated by gen_eval_asm.py; do not edit.  The instruction stream that
// the compile kernels write and the evaluation kernel's interpreter runs.
//
// An instruction is two words: the byte offset of its handler in the
// interpreter's table, and a payload (a constant's bits; the index of the next
// feature to fetch from memory, or -1; the byte offset of a stack slot in LDS).
// Programs run in execution order; the value on top of the stack lives in its
// own registers and entry e below it (from the bottom) in slot e.  The 64th
// word pair of every 64 is kOpReload unless the program has ended.
#pragma once

#include <cstdint>

constexpr int kRegSlots = 11;        // slots held in registers; deeper ones live in LDS
constexpr uint32_t kOpBytes = 64;    // bytes per handler
enum : uint32_t {
    kOpEnd = 0,
    kOpReload = 1,       // the next 64 instructions
    kOpLoadY = 2,        // top = the row's target (first instruction only: the caller put it there)
    kOpSaveL = 3,        // LDS slot = top
    kOpLoadTopL = 4,     // top = LDS slot
    kOpLoadL = 5,        // operand register = LDS slot (for a kOpBin of slot kRegSlots)
    kOpUnary = 6,        // + unary index: top = f(top)
    kOpSave = 20,        // + slot: slot = top
    kOpLoadS = 31,       // + slot: top = slot
    kOpSet = 42,         // + source: top = source
};
// Sources: 0 a constant; 1 + f feature f in registers, or 1 the feature fetched
// from memory (FREG = 0).  kPush + slot * n_src + source: slot = top, top = source.
// kFold + op * n_src + source: top = source (op) top; kBin + op * (kRegSlots + 1) + slot:
// top = top (op) slot; the reversed forms exchange the operands.
struct EvalOps {
    uint32_t n_src, push, fold, bin;
};
constexpr uint32_t eval_n_src(int freg) { return 1u + static_cast<uint32_t>(freg > 0 ? freg : 1); }
constexpr EvalOps eval_ops(int freg) {
    const uint32_t n = eval_n_src(freg), push = kOpSet + n, fold = push + kRegSlots * n;
    return EvalOps{n, push, fold, fold + 10u * n};
}
enum : uint32_t {
    kBAdd = 0,
    kBSub = 1,
    kBSubRev = 2,
    kBMul = 3,
    kBDiv = 4,
    kBDivRev = 5,
    kBMax = 6,
    kBMin = 7,
    kBAtan2 = 8,
    kBAtan2Rev = 9,
};
// What the interpreter leaves to its caller: 1 + unary index (top = f(top)), or one of
// these on the top t and the operand register m.
enum : uint32_t {
    kExitEnd = 0,
    kExitAtan2TM = 34,   // atan2(t, m)
    kExitAtan2MT = 35,   // atan2(m, t)
};

// The adjoint kernel's instructions, after the table above (FREG = 0).  t is the
// top (in the reverse part the adjoint), m the operand register, u a third.
// kAPutT/M/U + entry: tape entry = t / m / u; kAGMul + entry: t *= entry; kAMMul +
// entry: m = t * entry.  Entries from kTapeRegs on use the ...L forms (LDS, the
// payload a byte offset), from kTapeRegs + kTapeLds on the ...G forms (memory).
// kALoadM / kASaveM + slot: m = slot / slot = m.  kASetMC, kASetMF: m = constant, fetched
// feature.  kAMovMT m = t, kANegMT m = -t, kAMovUT u = t.  kADInvM/T: u = protected
// reciprocal of m / t; kADNegT/M: u = -t u u / -m u u; kADSqrt: u = d sqrt (u the input,
// t the root); kASinD, kACosD: t = f(t), u = f'(t).  kACAdd + slot: the constant's adjoint
// += m over the rows that count; kACAddX: the same by the caller (payload: slot).
// kAUnX + unary index - that of tan: t = f(t), u = f'(t) by the caller; kABinX + kind: by the caller,
// t = f of t and m, u = its derivative by t, m = by m (kinds: max and min with t, then
// with m as the first operand, atan2(t, m), atan2(m, t)).
constexpr int kTapeRegs = 26, kTapeLds = 16, kAccRegs = 8;
constexpr uint32_t kAUnFirst = 5;
enum : uint32_t {
    kAPutT = 206,
    kAPutM = 232,
    kAPutU = 258,
    kAGMul = 284,
    kAMMul = 310,
    kAPutTL = 336,
    kAPutML = 337,
    kAPutUL = 338,
    kAGMulL = 339,
    kAMMulL = 340,
    kAPutTG = 341,
    kAPutMG = 342,
    kAPutUG = 343,
    kAGMulG = 344,
    kAMMulG = 345,
    kALoadM = 346,
    kASaveM = 357,
    kASetMC = 368,
    kASetMF = 369,
    kAMovMT = 370,
    kANegMT = 371,
    kAMovUT = 372,
    kADInvM = 373,
    kADInvT = 374,
    kADNegT = 375,
    kADNegM = 376,
    kADSqrt = 377,
    kASinD = 378,
    kACosD = 379,
    kACAddX = 380,
    kACAdd = 381,
    kAUnX = 389,
    kABinX = 398,
    kAdjointOps = 404,
    kExitAdjUnary = 64,
    kExitAdjBinary = 96,
    kExitCAdd = 112,
};
