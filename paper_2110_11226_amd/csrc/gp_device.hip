// gp_device.hip -- gfx950 kernels and the device entry points of the C ABI.
//
// Hot path (Sec. III-C3 of "Accelerating Genetic Programming using GPUs"):
// every program of the population is evaluated on every dataset row by a
// right-to-left stack scan of its prefix list (Sec. III-A), each row's loss
// against the target is formed in registers, and the losses are summed per
// program.  The paper launches one thread per (program, row) and materialises
// the (rows x programs) prediction matrix before two library reductions; here
//   1. k_compile_streams rewrites each prefix list once per call into the
//      instructions of an assembly interpreter (the stack-schedule pre-pass):
//      of a binary function's operands the one that needs more stack entries
//      comes first, a terminal is fused with the function it is an operand of,
//      and a constant's value travels inside its instruction;
//   2. one persistent launch of k_eval walks (row chunk, program) work items,
//      a wavefront's first by its position and the others from a counter per
//      XCD; the 64 lanes of a wavefront run the same program on 64 different
//      rows, and each lane carries R rows, so that an instruction's fetch and
//      jump are scalar work shared by 64 R rows; the row loss is formed in
//      registers and only one float64 partial per (program, chunk) leaves the
//      kernel;
//   3. k_finalize merges the partials in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <tuple>
#include <string>
#include <type_traits>
#include <vector>

#include "gp_crmath.h"
#include "gp_eval_asm.h"
#include "gp_eval_code.h"
#include "gp_eval_sequential.h"
#include "gp_internal.h"

using namespace gp;

namespace {

constexpr int kWave = 64;
constexpr int kBlock = 256;                  // 4 independent wavefronts per block
constexpr int kSpill = GP_MAX_STACK - 1;     // stack entries below the cached top

// ---------------------------------------------------------------------------
// Views passed to kernels by value.
// ---------------------------------------------------------------------------
struct PopView {
    const uint32_t* nodes;
    const int64_t* prog_off;
    const float* consts;
    const int64_t* const_off;
    const int32_t* len;
    int32_t P;
};

struct DataView {
    const float* X;
    int64_t ld;
    int32_t F;
    int64_t N;
    const float* y;
    const float* w;
};

// Compiled programs: program p's instructions are code[prog_off[p] ..
// prog_off[p] + clen[p]) (clen[p] <= len[p]), in execution order.
struct CodeView {
    const uint4* code;     // the adjoint's format (k_compile)
    const int32_t* clen;
    const uint4* ecode;    // the evaluation kernel's format (gp_eval_code.h, two instructions per
    const uint32_t* ehdr;  // uint4): program p from ecode[prog_off[p] * ex_mul + p * ex_add], its header
    int32_t ex_mul;        // room per node (1, or the longest user definition)
    int32_t ex_add;        // room per program for a user loss
};

// Work decomposition: rows are split into n_chunks chunks of `chunk` rows
// (a multiple of the 64*R rows one wavefront covers per tile).  Work item
// it = chunk_index * P + k covers program order[k] on that chunk; programs are
// ordered longest first so each chunk's long programs start early.
// The work counters: one per XCD queue, 64 bytes apart, in a 1 KiB block
// whose word kFlagWord serves the backward pass's user-function check.
constexpr int kQueues = 8;
constexpr int kQueueStride = 16;
constexpr size_t kCounterBytes = 1024;
constexpr int kFlagWord = 128;
// two more such blocks, in scratch that grows, hold the adjoint kernels', and
// in word kLongWord the number of programs of more than kParNodes nodes, which
// come first in the order
constexpr int kCounterSet = kCounterBytes / sizeof(uint32_t);
constexpr int kCounterSets = 3;
constexpr int kLongWord = 129;

struct Sched {
    int64_t chunk;
    int32_t n_chunks;
    int64_t n_items;
    const int32_t* order;
    uint32_t* counter;
    int32_t batch;     // work items per claim
    int32_t lds_slots; // stack slots per row in LDS (kEvalLds or kEvalLdsUser)
    int32_t blocks;    // the launch's blocks, and wavefronts per block
    int32_t wpb;
};

// ---------------------------------------------------------------------------
// Instruction format (word x; word y):
//   bits 0-1  class: kPush (push a terminal), kFold (terminal fused with the
//             binary function whose first operand it is; the current top is
//             the second operand), kBin (binary: top op next-below), kUn
//   bits 2-5  function: binary ADD..DIV, MAX..ATAN2 as 0..6; unary NEG..TAN,
//             ABS..CBRT as 0..13
//   bit 6     the terminal is a constant (value in y) rather than a feature
//   bit 7     "active": the subtree this instruction completes holds a
//             constant (only such instructions carry derivatives back)
//   bits 8-31 feature index, or the constant's slot
//   y         a constant's float bits; for an inactive instruction, the
//             index of the first instruction of the subtree it completes
//   z         up to 8 unary functions applied, in order, to the result of
//             the instruction (4 bits each from the lowest: unary function
//             index + 1; 0 ends the chain), so that a unary function costs no
//             dispatch of its own
//   w         (active instructions, in the adjoint's compile only) bits
//             0..25: index + 1 of the next active instruction its reverse
//             walk visits (0: none); bits 26..31: the subtrees without a
//             constant it skips before that one
// ---------------------------------------------------------------------------
enum : uint32_t { kPush = 0, kFold = 1, kBin = 2, kUn = 3 };
constexpr uint32_t kConstBit = 64u;
constexpr uint32_t kActive = 128u;
constexpr uint32_t kNextBits = 26u;
constexpr uint32_t kNextMask = (1u << kNextBits) - 1u;
constexpr int64_t kMaxAdjointLen = int64_t{1} << 25;   // program length the reverse links can address

GP_HD uint32_t enc(uint32_t cls, uint32_t fn, uint32_t is_const, uint32_t arg) {
    return cls | (fn << 2) | (is_const << 6) | (arg << 8);
}

// ---------------------------------------------------------------------------
// Register-resident arrays.  The compiler keeps a small local array in
// VGPRs, indexed by a wave-uniform value through M0-relative addressing,
// only when each array is a separate plain local; the R per-row copies are
// therefore spelled out one by one.
// ---------------------------------------------------------------------------
#define GP_ARRAYS(name, n) float name##0[n], name##1[n], name##2[n], name##3[n]
#define GP_PUT(name, idx, v)                         \
    do {                                             \
        name##0[idx] = v[0];                         \
        if constexpr (R > 1) name##1[idx] = v[1];    \
        if constexpr (R > 2) name##2[idx] = v[2];    \
        if constexpr (R > 3) name##3[idx] = v[3];    \
    } while (0)
#define GP_GET(name, idx, v)                         \
    do {                                             \
        v[0] = name##0[idx];                         \
        if constexpr (R > 1) v[1] = name##1[idx];    \
        if constexpr (R > 2) v[2] = name##2[idx];    \
        if constexpr (R > 3) v[3] = name##3[idx];    \
    } while (0)

// Uniform loads of read-only data through the scalar data cache: the pointer
// is cast to the constant address space so the compiler issues s_load.
template <typename T>
__device__ __forceinline__ T ldu(const T* p) {
    return *(const __attribute__((address_space(4))) T*)p;
}

// A wavefront's claims of work items, `batch` consecutive items each.  One
// queue per XCD: queue x holds the chunks c with c % kQueues == x, chunk-major,
// each chunk's programs in LPT order (longest first), so that a chunk's rows
// are read into one L2 while every program walks them.  With fewer chunks than
// queues, queue x holds every eighth program instead, of every chunk: the rows
// are few then, and all claims on one counter, at some 15 ns each, bound the
// launch (20,000 programs of up to 40 nodes on 200 rows: the call 491 us with
// one counter, 209 with eight; 1,000 programs on 1,000 rows: 128 and 63).
// Blocks are dealt to the XCDs in turn, so a block starts on queue blockIdx.x %
// kQueues.
// Every wavefront's first claim is its own by position, and the counters
// count only the claims after those: a job of at most one claim per wavefront
// touches no counter (with every claim an atomic, 4,096 rows x 256 programs
// spent 150 of its 180 us on 70 thousand of them, most from wavefronts finding
// all eight queues dry one after the other).  A wavefront whose queue has run
// dry reads all the counters at once to find one that has not.
struct Claims {
    uint32_t* counter;
    uint32_t P, n_chunks, batch, blocks, wpb;
    uint32_t per;                      // places of one chunk in a queue (the last may be none, see program)
    uint32_t index;                    // this wavefront among its queue's
    int q0, q;
    bool first;
    __device__ Claims(const Sched& s, uint32_t programs, uint32_t wid)
        : counter(s.counter), P(programs), n_chunks(static_cast<uint32_t>(s.n_chunks)),
          batch(static_cast<uint32_t>(s.batch)), blocks(static_cast<uint32_t>(s.blocks)),
          wpb(static_cast<uint32_t>(s.wpb)), per(striped() ? (P + kQueues - 1) / kQueues : P), index(blockIdx.x / kQueues * static_cast<uint32_t>(s.wpb) + wid), q0(static_cast<int>(blockIdx.x % kQueues)), q(q0),
          first(true) {}
    __device__ bool striped() const { return n_chunks < static_cast<uint32_t>(kQueues); }
    // where place k of chunk cq of queue x lies: its chunk, and its program, which
    // may be P, none, or above.  (As many places in every queue, so that the
    // division by their number has its reciprocal once: one for each queue cost
    // 300 programs on 50,021 rows 1.3 us of 276.)
    __device__ int32_t chunk(uint32_t cq, int x) const {
        return static_cast<int32_t>(striped() ? cq : cq * kQueues + static_cast<uint32_t>(x));
    }
    __device__ uint32_t program(uint32_t k, int x) const {
        return striped() ? k * kQueues + static_cast<uint32_t>(x) : k;
    }
    // (items stay below 2^31: n_items is at most 2^30)
    __device__ uint32_t items(uint32_t x) const {
        return striped() ? (x < P ? n_chunks * per : 0u) : (n_chunks - x + kQueues - 1) / kQueues * P;
    }
    // items covered by the first claims of queue x's wavefronts
    __device__ uint32_t given(uint32_t x) const {
        return (blocks - x + kQueues - 1) / kQueues * wpb * batch;
    }
    // The next claim: queue *qx, items [*it0, *it1).  False once all are dry.
    __device__ bool next(int lane, int* qx, uint32_t* it0, uint32_t* it1) {
        if (first) {
            first = false;
            const uint32_t n = items(static_cast<uint32_t>(q)), i = index * batch;
            if (i < n) {
                *qx = q;
                *it0 = i;
                *it1 = min(i + batch, n);
                return true;
            }
        }
        for (;;) {
            const uint32_t n = items(static_cast<uint32_t>(q)), g = given(static_cast<uint32_t>(q));
            if (g < n) {
                uint32_t c = 0;
                if (lane == 0) c = atomicAdd(counter + q * kQueueStride, batch);
                const uint32_t i = g + static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(c)));
                if (i < n) {
                    *qx = q;
                    *it0 = i;
                    *it1 = min(i + batch, n);
                    return true;
                }
            }
            // dry: the next queue, from q0 on, that still has items
            // (formed from the lane here: hoisted, it would hold registers
            // throughout the caller's loops)
            bool left = false;
            int ln = lane;
            asm volatile("" : "+v"(ln));
            if (ln < kQueues) {
                const uint32_t x = static_cast<uint32_t>((q0 + ln) % kQueues);
                const uint32_t nx = items(x), gx = given(x);
                left = gx < nx && gx + __hip_atomic_load(counter + x * kQueueStride, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT) < nx;
            }
            const uint64_t m = __ballot(left);
            if (m == 0) return false;
            q = (q0 + __builtin_ctzll(m)) % kQueues;
        }
    }
};

// A wave-uniform value the compiler cannot see is one.
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}

// Orders a wavefront's own LDS writes before its later LDS reads (its LDS
// operations complete in order; this only keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The adjoint kernel's stack slots: slots below kStackRegs live in VGPRs, slots
// from kStackRegs on in a per-wavefront memory area; register slot kStackRegs is
// a sink for the speculative writes of those deeper slots.  Slot 0 is never
// read, so a full stack of GP_MAX_STACK values uses slots 1 .. GP_MAX_STACK-1.
constexpr int kStackRegs = 15;
constexpr int kStackLds = GP_MAX_STACK - kStackRegs;

// Tables of the correctly rounded sin, cos and log (gp_crmath.h): staged in
// LDS by the evaluation and adjoint kernels, read from global memory
// elsewhere.
struct MathTabs {
    const crm::SinCosEntry* sc;
    const crm::LogEntry* lg;
};
__device__ __forceinline__ MathTabs global_tabs() { return MathTabs{crm::kSinCosTab, crm::kLogTab}; }

// The kernel-resident copies (one per block, filled before its first use).
struct MathTabsLds {
    crm::LogEntry lg[256];       // (at offset 0: its entries' address is the index alone)
    crm::SinCosEntry sc[256];    // (at 4 KB: the offset is the read's immediate)
};
__device__ __forceinline__ MathTabs stage_tabs(MathTabsLds& lds) {
    for (int i = threadIdx.x; i < 256; i += blockDim.x) lds.sc[i] = crm::kSinCosTab[i];
    for (int i = threadIdx.x; i < 256; i += blockDim.x) lds.lg[i] = crm::kLogTab[i];
    __syncthreads();
    return MathTabs{lds.sc, lds.lg};
}

// Protected operators (reading of Sec. III-C3's function set: the gplearn
// convention).  Comparisons are written so that NaN takes the protected arm.
__device__ __forceinline__ float op_div(float a, float b) {
    return fabsf(b) > GP_PROTECT_EPS ? a / b : 1.0f;
}
__device__ __forceinline__ float op_log(float a, const MathTabs& mt, const crm::LogK& K) {
    // (evaluated on every lane, the protected ones included, so that the
    // protection is a select rather than a branch)
    const float l = crm::log_cr(fabsf(a), mt.lg, K);
    return fabsf(a) > GP_PROTECT_EPS ? l : 0.0f;
}

// sqrt|a|, correctly rounded: in double from the hardware reciprocal square
// root y (relative error below 2^-22): s = d y, e = 1 - s y, and
// sqrt d = s (1 - e)^(-1/2) = s + s e (1/2 + 3/8 e + O(e^2)), where the e^3
// left out is below 2^-61 and the rounding of s enters e, so that the result
// is within 2^-52.  A float's square root lies at least 2^-51 (relative)
// from every float rounding boundary (a - m^2 is a nonzero multiple of the
// least bit of m^2 for a midpoint m), so the double result rounds to float
// as the exact one does.  Zeros and infinity are passed through (the
// steps would give NaN there); NaN stays NaN.
__device__ __forceinline__ float op_sqrt(float a) {
    const double d = static_cast<double>(fabsf(a));
    const double y = __builtin_amdgcn_rsq(d);
    const double s0 = d * y;
    const double e = fma(-s0, y, 1.0);
    const double s = fma(s0 * e, fma(e, crm::kreg(0.375), 0.5), s0);
    // class mask: +0 (bit 6) or +inf (bit 9)
    return __builtin_amdgcn_class(d, 0x240) ? fabsf(a) : static_cast<float>(s);
}
__device__ __forceinline__ float op_inv(float a) {
    return fabsf(a) > GP_PROTECT_EPS ? 1.0f / a : 0.0f;
}

// t = sin t (is_cos false) or cos t on the R rows of a lane: the common
// path on every row, then one branch, rarely taken, for the rows with
// |t| >= 2^24, inf or NaN
template <int R>
__device__ __forceinline__ void sincos_rows(bool is_cos, float (&t)[R], const MathTabs& mt) {
    const crm::SinCosK K = crm::sincos_k(is_cos);   // (once for the R rows)
    float f[R];
    bool rare = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        f[j] = crm::sincos_common(t[j], mt.sc, K);
        rare |= crm::sincos_rare_input(t[j]);
    }
    if (rare) {
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (crm::sincos_rare_input(t[j])) f[j] = crm::sincos_rare(t[j], is_cos, mt.sc, K);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) t[j] = f[j];
}

// a = a (op) b for the wider binary functions (MAX, MIN, ATAN2 as 4..6)
template <int R>
__device__ __forceinline__ void apply_binary_wide(uint32_t fn, float (&a)[R], const float (&b)[R]) {
    // max / min ignore a NaN operand; on equal operands the sign bits are
    // combined so that -0 orders below +0 whatever order fmaxf takes them in
    if (fn == 4) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float m = fmaxf(a[j], b[j]);
            a[j] = a[j] == b[j] ? __int_as_float(__float_as_int(a[j]) & __float_as_int(b[j])) : m;
        }
    } else if (fn == 5) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float m = fminf(a[j], b[j]);
            a[j] = a[j] == b[j] ? __int_as_float(__float_as_int(a[j]) | __float_as_int(b[j])) : m;
        }
    } else {
#pragma unroll
        for (int j = 0; j < R; ++j) a[j] = atan2f(a[j], b[j]);
    }
}

// t = f(t) for the wider unary functions (ABS..CBRT as 6..13)
template <int R>
__device__ __forceinline__ void apply_unary_wide(uint32_t fn, float (&t)[R]) {
    switch (fn) {
    case 6:
#pragma unroll
        for (int j = 0; j < R; ++j) t[j] = fabsf(t[j]);
        break;
    case 7:
#pragma unroll
        for (int j = 0; j < R; ++j) t[j] = expf(t[j]);
        break;
    case 8:
#pragma unroll
        for (int j = 0; j < R; ++j) t[j] = op_inv(t[j]);
        break;
    case 9:
#pragma unroll
        for (int j = 0; j < R; ++j) t[j] = t[j] * t[j];
        break;
    case 10:
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float q = t[j] * t[j];
            t[j] = q * t[j];
        }
        break;
    case 11:
#pragma unroll
        for (int j = 0; j < R; ++j) t[j] = tanhf(t[j]);
        break;
    case 12:
#pragma unroll
        for (int j = 0; j < R; ++j) t[j] = atanf(t[j]);
        break;
    default:
#pragma unroll
        for (int j = 0; j < R; ++j) t[j] = cbrtf(t[j]);
        break;
    }
}

// a = a (op) b for the binary function index fn (ADD, SUB, MUL, DIV first,
// then the wider set)
template <int R>
__device__ __forceinline__ void apply_binary(uint32_t fn, float (&a)[R], const float (&b)[R]) {
    if (fn >= 4) {
        apply_binary_wide<R>(fn, a, b);
    } else if (fn < 2) {
        if (fn == 0) {
#pragma unroll
            for (int j = 0; j < R; ++j) a[j] = a[j] + b[j];
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) a[j] = a[j] - b[j];
        }
    } else {
        if (fn == 2) {
#pragma unroll
            for (int j = 0; j < R; ++j) a[j] = a[j] * b[j];
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) a[j] = op_div(a[j], b[j]);
        }
    }
}

// t = f(t) for the unary function index fn (NEG, LOG, SQRT, SIN, COS, TAN
// first, then the wider set)
template <int R>
__device__ __forceinline__ void apply_unary(uint32_t fn, float (&t)[R], const MathTabs& mt) {
    if (fn >= 6) {
        apply_unary_wide<R>(fn, t);
    } else if (fn < 3) {
        if (fn == 0) {
#pragma unroll
            for (int j = 0; j < R; ++j) t[j] = -t[j];
        } else if (fn == 1) {
            const crm::LogK K = crm::log_k();   // (once for the R rows)
#pragma unroll
            for (int j = 0; j < R; ++j) t[j] = op_log(t[j], mt, K);
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) t[j] = op_sqrt(t[j]);
        }
    } else {
        if (fn == 3) {
            sincos_rows<R>(false, t, mt);
        } else if (fn == 4) {
            sincos_rows<R>(true, t, mt);
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) t[j] = tanf(t[j]);
        }
    }
}

// ---------------------------------------------------------------------------
// The evaluation order: programs by length, longest first, and the work
// counters reset.  One block of THREADS: a counting sort over min(len,
// kBins-1).  Block 0 of the compilers below does it while the others compile;
// a launch of its own took 4.6 us of every call.
// ---------------------------------------------------------------------------
constexpr int kBins = 1024;
struct OrderLds {
    int32_t start[kBins];
    int32_t wtot[kBlock / kWave];
};
struct OrderArgs {
    const int32_t* len;
    int32_t P;
    int32_t* order;
    uint32_t* counter;     // `sets` sets of queues' counters: one, or kCounterSets
    int32_t sets;
};
// the longest program of the wavefront-parallel compilers and of k_adjoint
constexpr int kParNodes = 1024;
// 16-byte units of the adjoint's code per node, two instructions of k_adjoint's
// each.  A program of n nodes takes at most 6 n instructions, the reloads and
// both ends 6.1 n (quotients of roots of constants: 10 a quotient of two
// subtrees, 8 a root of a constant; no other nodes take more for their number).
constexpr int64_t kAdjCodePerNode = 4;

template <int THREADS>
__device__ __forceinline__ void order_programs(const OrderArgs& oa, OrderLds& sh) {
    constexpr int kPer = kBins / THREADS, kE = 8;     // bins per thread; lengths in flight per thread
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid >> 6;
    const int32_t* __restrict__ len = oa.len;
    const int32_t P = oa.P;
    for (int b = tid; b < kBins; b += THREADS) sh.start[b] = 0;
    for (int q = tid; q < oa.sets * kQueues; q += THREADS)
        oa.counter[(q / kQueues) * kCounterSet + (q % kQueues) * kQueueStride] = 0u;
    __syncthreads();
    // key: 0 above kParNodes, else kBins-1 - min(len, kBins-2), so that longer
    // programs come first
    auto walk = [&](auto visit) {
        for (int64_t p0 = tid; p0 < P; p0 += THREADS * kE) {
            int32_t key[kE];
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                const int64_t p = p0 + e * THREADS;
                const int32_t n = p < P ? len[p] : 0;
                key[e] = p >= P ? -1 : n > kParNodes ? 0 : kBins - 1 - min(max(n, 0), kBins - 2);
            }
#pragma unroll
            for (int e = 0; e < kE; ++e)
                if (key[e] >= 0) visit(static_cast<int32_t>(p0 + e * THREADS), key[e]);
        }
    };
    walk([&](int32_t, int32_t key) { atomicAdd(&sh.start[key], 1); });
    __syncthreads();
    int32_t c[kPer], sum = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        c[e] = sh.start[tid * kPer + e];
        sum += c[e];
    }
    int32_t v = sum;
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t o = __shfl_up(v, d, kWave);
        if (lane >= d) v += o;
    }
    if (lane == kWave - 1) sh.wtot[wid] = v;
    __syncthreads();
    int32_t at = v - sum;
    for (int q = 0; q < THREADS / kWave; ++q) at += q < wid ? sh.wtot[q] : 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        sh.start[tid * kPer + e] = at;
        at += c[e];
    }
    __syncthreads();
    if (tid > 0 && tid < oa.sets) oa.counter[tid * kCounterSet + kLongWord] = static_cast<uint32_t>(sh.start[1]);
    __syncthreads();
    walk([&](int32_t p, int32_t key) { oa.order[atomicAdd(&sh.start[key], 1)] = p; });
}

// ---------------------------------------------------------------------------
// k_compile: the instructions of k_adjoint_long, one lane per program of more
// than kParNodes nodes.  Scans the prefix list right to left (the evaluation
// order of Sec. III-A) and emits instructions in that order.  A terminal at
// position i is the first operand of the function at i-1 exactly when that
// function is binary (its first operand starts right after it), so such pairs
// become one kFold instruction; a unary function is chained onto the
// instruction before it.  A shadow stack (in LDS, one column per lane) tracks,
// for each value on the evaluation stack, the first instruction of the subtree
// that produced it and whether that subtree holds a constant.
// ---------------------------------------------------------------------------
constexpr uint32_t kShStartMask = 0x3fffffffu;   // shadow entry: start | active << 31

__global__ __launch_bounds__(kBlock) void k_compile(PopView pop, uint4* __restrict__ code, int32_t* __restrict__ clen) {
    __shared__ uint32_t shadow[GP_MAX_STACK][kBlock];
    const int32_t p = static_cast<int32_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (p >= pop.P || pop.len[p] <= kParNodes) return;
    const int64_t off = pop.prog_off[p];
    const int32_t L = pop.len[p];
    const uint32_t* pn = pop.nodes + off;
    const float* pc = pop.consts + pop.const_off[p];
    uint4* out = code + off * kAdjCodePerNode;
    uint32_t* sh = &shadow[0][threadIdx.x];   // entry h at sh[h * kBlock]
    int h = 0;                                // shadow stack height
    int32_t k = 0;                            // instructions emitted
    uint4 pend = make_uint4(0u, 0u, 0u, 0u);  // the last instruction, still open for a unary chain
    int chain = -1;                           // unary functions chained on it (-1: none pending)
    for (int32_t i = L - 1; i >= 0; --i) {
        const uint32_t w = pn[i];
        const uint32_t op = w & 0xffu;
        const uint32_t arg = w >> 8;          // feature index, or constant slot
        const int top_i = min(max(h - 1, 0), GP_MAX_STACK - 1);
        const int ar = arity(op);
        if (ar == 1 && chain >= 0 && chain < 8) {
            // a unary function applied to the pending instruction's result:
            // same subtree start and activity as its operand
            pend.z |= (unary_index(op) + 1u) << (4 * chain);
            ++chain;
            continue;
        }
        uint32_t x, start, active, y;
        if (op <= GP_OP_CONST) {
            const uint32_t is_c = op == GP_OP_CONST ? 1u : 0u;
            const uint32_t prev = i >= 1 ? (pn[i - 1] & 0xffu) : 0u;
            if (i >= 1 && i != L - 1 && arity(prev) == 2) {
                const uint32_t top = sh[top_i * kBlock];    // the second operand
                start = top & kShStartMask;
                x = enc(kFold, binary_index(prev), is_c, arg);
                active = is_c | (top >> 31);
                --h;
                --i;
            } else {
                x = enc(kPush, 0, is_c, arg);
                start = static_cast<uint32_t>(k);
                active = is_c;
            }
            y = is_c ? __float_as_uint(pc[arg]) : start;
        } else if (ar == 2) {
            const int i1 = min(max(h - 1, 0), GP_MAX_STACK - 1), i2 = min(max(h - 2, 0), GP_MAX_STACK - 1);
            const uint32_t first = sh[i1 * kBlock];      // top: the first operand
            const uint32_t second = sh[i2 * kBlock];     // evaluated before it
            start = second & kShStartMask;
            h -= 2;
            x = enc(kBin, binary_index(op), 0, 0);
            active = (first >> 31) | (second >> 31);
            y = start;
        } else {
            // a unary function with a full chain before it: its own instruction
            const uint32_t top = sh[top_i * kBlock];
            x = enc(kUn, unary_index(op), 0, 0);
            start = top & kShStartMask;
            active = top >> 31;
            --h;
            y = start;
        }
        if (chain >= 0) out[k - 1] = pend;
        pend = make_uint4(x | (active ? kActive : 0u), y, 0u, 0u);
        chain = 0;
        // (valid programs keep 1 <= h <= GP_MAX_STACK; the clamps only keep an
        // invalid one inside this array)
        h = max(h, 0);
        sh[min(h, GP_MAX_STACK - 1) * kBlock] = start | (active << 31);
        ++h;
        ++k;
    }
    if (chain >= 0) out[k - 1] = pend;
    clen[p] = k;
    // the reverse walk, from the last instruction down: an inactive instruction
    // stands for its whole subtree (skipped, one stack entry); each active one
    // is linked to the next active one and counts the skips between them.
    // (Indices stay below 2^26 for programs the adjoint accepts; skips never
    // exceed the stack depth, below 2^6.)
    int32_t last = -1;
    uint32_t skips = 0u;
    for (int32_t q = k - 1; q >= 0;) {
        const uint4 ins = out[q];
        if (!(ins.x & kActive)) {
            ++skips;
            q = min(static_cast<int32_t>(ins.y), q) - 1;   // (the clamp only guards a malformed program)
            continue;
        }
        if (last >= 0) out[last].w = (static_cast<uint32_t>(q + 1) & kNextMask) | (min(skips, 63u) << kNextBits);
        last = q;
        skips = 0u;
        --q;
    }
    if (last >= 0) out[last].w = 0u;
}

// ---------------------------------------------------------------------------
// The evaluation kernel's instruction stream: gp_eval_code.h.  A terminal that
// is an operand of a binary function is fused with it, a subtree of constants
// only is replaced by its value (formed here, once, by the same float32
// functions the kernel applies per row), and every other node is one
// instruction.
//
// A binary function's operands are evaluated in the order that needs fewer
// stack entries (the one that needs more of them first), whichever comes first
// in the prefix list: the same operations on the same operands, so the same
// value, but a random program of 200 nodes needs at most 5 entries instead of
// up to 20.
//
// A user function (Sec. V: custom function sets) is expanded in place: its
// arguments are evaluated as usual, its definition's argument references
// become copies of the argument entries, and once the definition has left its
// value on top, the arguments below it are simply forgotten (the next push
// overwrites their slots).  A user loss (GP_METRIC_USER_i) is the same
// expansion around the whole program: kOpLoadY pushes the row's target first,
// and the loss function's definition runs on (output, target) last.
// These stacks reach past the program's own GP_MAX_STACK, into LDS slots
// kEvalLds .. kEvalLdsUser-1, which launches that may meet them provide.
// ---------------------------------------------------------------------------
// instructions the evaluation kernel may fetch past a program's end (whole
// blocks of 64), in 16-byte units
constexpr int64_t kCodePad = 32;


// A wavefront's program in the parallel path, one entry per node, at most
// kParNodes (13 KB: twelve wavefronts per CU).
constexpr int kSeqLanes = 60;     // programs side by side: their entries take no more LDS than that
struct ParNodes {
    float val[kParNodes];        // value of a constant subtree; later, an instruction's feature
    uint16_t sec[kParNodes];     // second operand of a binary function
    uint16_t cnt[kParNodes];     // instructions of the subtree
    uint16_t start[kParNodes];   // its first instruction
    uint8_t op[kParNodes];
    uint8_t ent[kParNodes];      // stack entries the subtree needs; kLeaf, kConst
    uint8_t lev[kParNodes];      // entries below it when it is evaluated
};
constexpr uint8_t kEntMask = 31, kLeaf = 64, kConst = 128;

// compile_eval_program: one wavefront per program.
//   1. From the right, blocks of 64 nodes: the stack height after each node of
//      the right-to-left scan (a suffix sum of 1 - arity).  A binary function's
//      first operand is the node after it; its second is the nearest node to
//      its right with its own height (the entry below its first operand came
//      about there), found among the block's nodes by one ballot per height
//      and beyond it from the leftmost node so far of each height, which lane
//      `height` holds.
//   2. From the leaves up, each block's nodes as their operands are done: the
//      entries and instructions each subtree takes, and constant subtrees'
//      values.
//   3. From the root down: each evaluated subtree's first instruction and the
//      entries below it.
//   4. Every node writes its instruction.
// A lane per program, scanning it node by node (as before), took 64 to 500 us:
// every step waited for memory, and 64 programs took each other's branches,
// the functions of constant subtrees among them.  A wavefront per program
// takes about as many steps as the program is deep.
//
// Programs with user functions or a user loss, and those too long or too deep,
// are left to compile_sequential, a lane each.  While user functions are
// defined, a wavefront takes a group of programs, compiles those it can one
// after the other and then the rest side by side (20,000 programs of up to 40
// nodes with user functions on 1,000 rows: 733 us with one of 64 lanes at work
// for each, 413 in groups of seven; 4,096 of up to 120 on 4,096 rows 754 and
// 570).
struct SeqShadow {              // one lane's column
    uint32_t* e;
    float* v;
    __device__ uint32_t& entry(int i) { return e[i * kSeqLanes]; }
    __device__ float& value(int i) { return v[i * kSeqLanes]; }
};
union EvalCompileLds {
    ParNodes nodes;
    struct {
        uint32_t e[kCompileDepth][kSeqLanes];
        float v[kCompileDepth][kSeqLanes];
    } seq;
};
static_assert(sizeof(EvalCompileLds) == sizeof(ParNodes), "twelve wavefronts per CU");
// Callers are not to pass programs that gp_validate_population refuses.  One all
// the same has no operands where the parallel compilers look for them: they
// leave it alone, so that what they write stays within its room.  h: the height
// of the right-to-left scan after the node.
__device__ __forceinline__ bool malformed(int arity, int h) { return arity < 0 || h < 1 || h > GP_MAX_STACK; }

// Where compile_sequential puts its word pairs.
struct CodeOut {
    uint2* at;
    __device__ void put(int64_t q, uint32_t handler, uint32_t payload) { at[q] = make_uint2(handler, payload); }
    __device__ void payload(int64_t q, uint32_t payload) { at[q].y = payload; }
};
struct EvalCompile {
    uint4* code;
    uint32_t* hdr;
    UserDefs ud;
    int32_t loss_fn, ex_mul, ex_add;
    Emit em;
    int32_t group;       // programs per wavefront, at most kSeqLanes
};

__device__ __forceinline__ uint2* eval_code(const PopView& pop, const EvalCompile& ec, int32_t p) {
    return reinterpret_cast<uint2*>(ec.code + pop.prog_off[p] * ec.ex_mul + static_cast<int64_t>(p) * ec.ex_add);
}

// The programs p0 + l, l < group, of which compile_eval_program's return marked
// bit l.
__device__ __forceinline__ void compile_eval_rest(const PopView& pop, const EvalCompile& ec, EvalCompileLds& sh,
                                                  int32_t p0, uint64_t rest, int lane) {
    if (!((rest >> lane) & 1ull)) return;
    const int32_t p = p0 + lane;
    CodeOut out{eval_code(pop, ec, p)};
    compile_sequential(
        pop.nodes + pop.prog_off[p], pop.consts + pop.const_off[p], pop.len[p], out,
        2 * (static_cast<int64_t>(pop.len[p]) * ec.ex_mul + ec.ex_add), ec.hdr + p, ec.em, ec.ud, ec.loss_fn,
        SeqShadow{&sh.seq.e[0][lane], &sh.seq.v[0][lane]},
        [](uint32_t fn, float x) __attribute__((always_inline)) {
            float t[1] = {x};
            apply_unary<1>(fn, t, global_tabs());
            return t[0];
        },
        [](uint32_t fn, float a, float b) __attribute__((always_inline)) {
            float t[1] = {a};
            const float u[1] = {b};
            apply_binary<1>(fn, t, u);
            return t[0];
        });
}

// True if the program is left to compile_sequential.
__device__ __forceinline__ bool compile_eval_program(const PopView& pop, const EvalCompile& ec, ParNodes& nd, int32_t p,
                                                     int lane) {
    uint32_t* __restrict__ hdr = ec.hdr;
    const Emit& em = ec.em;
    const int64_t off = pop.prog_off[p];
    const int32_t L = pop.len[p];
    const uint32_t* pn = pop.nodes + off;
    const float* pc = pop.consts + pop.const_off[p];
    uint2* out = eval_code(pop, ec, p);
    if (ec.loss_fn >= 0 || L > kParNodes) return true;
    const int nb = (L + kWave - 1) / kWave;
    // ---- 1. heights and second operands ----
    int carry = 0;                 // height to the right of the block
    int lastpos = 0;               // lane h: the leftmost node so far of height h
    uint64_t rest = 0;             // lanes that met a user function, or a height no valid program has
    for (int b = nb - 1; b >= 0; --b) {
        const int i = b * kWave + lane;
        const bool valid = i < L;
        const uint32_t op = valid ? (pn[i] & 0xffu) : 0u;
        const int ar = arity(op);
        int hs = valid ? 1 - ar : 0;
        for (int d = 1; d < kWave; d <<= 1) {
            const int o = __shfl_down(hs, d, kWave);
            if (lane + d < kWave) hs += o;
        }
        rest |= __ballot(valid && (is_user_op(op) || malformed(ar, hs + carry)));
        const int H = min(max(hs + carry, 0), 31);
        uint64_t same = 0, mine = 0;
        for (int hv = 1; hv <= GP_MAX_STACK; ++hv) {
            const uint64_t m = __ballot(valid && H == hv);
            if (H == hv) same = m;
            if (lane == hv) mine = m;
        }
        const uint64_t right = lane < 63 ? same >> (lane + 1) : 0;
        const int beyond = __shfl(lastpos, H, kWave);
        const int sec = right ? i + 1 + __builtin_ctzll(right) : beyond;
        if (mine) lastpos = b * kWave + __builtin_ctzll(mine);
        carry = __builtin_amdgcn_readfirstlane(hs + carry);
        if (valid) {
            nd.op[i] = static_cast<uint8_t>(op);
            nd.sec[i] = static_cast<uint16_t>(min(max(sec, 0), L - 1));   // (a malformed program's may lie anywhere)
            nd.start[i] = 0xffffu;
        }
    }
    if (rest || carry != 1) return true;
    wave_lds_sync();
    // ---- 2. entries, instructions, constants ----
    // (a round reads both operands' words at once and chooses: read as they
    // were needed, one after the other, they cost a round three latencies)
    uint64_t folds = 0;            // blocks with a function of constants
    for (int b = nb - 1; b >= 0; --b) {
        const int i = b * kWave + lane;
        const bool valid = i < L;
        const uint32_t op = valid ? nd.op[i] : 0u;
        const int ar = arity(op);
        const int c1 = min(i + 1, L - 1), c2 = valid && ar == 2 ? nd.sec[i] : c1;
        // an operand outside the block is done
        const uint64_t need = (ar >= 1 && c1 < (b + 1) * kWave ? 1ull << (c1 & 63) : 0ull) |
                              (ar == 2 && c2 < (b + 1) * kWave ? 1ull << (c2 & 63) : 0ull);
        bool done = !valid || ar == 0, fold = false;
        if (valid && ar == 0) {
            nd.ent[i] = static_cast<uint8_t>(1 | (op == GP_OP_CONST ? kConst : kLeaf));
            nd.cnt[i] = 1;
            nd.val[i] = op == GP_OP_CONST ? pc[pn[i] >> 8] : 0.0f;
        }
        wave_lds_sync();
        for (int round = 0; round <= kWave; ++round) {
            const uint64_t ready = __ballot(done);
            if (ready == ~0ull) break;
            const uint32_t e1 = nd.ent[c1], e2 = nd.ent[c2], n1 = nd.cnt[c1], n2 = nd.cnt[c2];
            if (!done && (need & ~ready) == 0) {
                const bool two = ar == 2, t1 = e1 & (kLeaf | kConst), t2 = e2 & (kLeaf | kConst);
                const uint32_t m1 = e1 & kEntMask, m2 = e2 & kEntMask;
                fold = (e1 & kConst) && (!two || (e2 & kConst));
                uint32_t ent = two ? (t1 ? m2 : t2 ? m1 : m1 == m2 ? m1 + 1u : max(m1, m2)) : max(m1, 1u);
                uint32_t cnt = 1u + (two ? (t1 ? n2 : t2 ? n1 : n1 + n2) : n1);
                ent = fold ? 1u | kConst : ent;
                cnt = fold ? 1u : cnt;
                nd.ent[i] = static_cast<uint8_t>(ent);
                nd.cnt[i] = static_cast<uint16_t>(cnt);
                done = true;
            }
            wave_lds_sync();
        }
        if (__ballot(fold)) folds |= 1ull << b;
    }
    // the values of constant subtrees, by themselves: among the rounds above,
    // each with such a node would wait for the functions
    for (; folds; folds &= ~(1ull << (63 - __builtin_clzll(folds)))) {
        const int b = 63 - __builtin_clzll(folds);
        const int i = b * kWave + lane, ii = min(i, L - 1);
        const uint32_t op = nd.op[ii];
        const int ar = arity(op);
        const int c1 = min(i + 1, L - 1), c2 = ar == 2 ? nd.sec[ii] : c1;
        const uint64_t need = (c1 < (b + 1) * kWave ? 1ull << (c1 & 63) : 0ull) |
                              (c2 < (b + 1) * kWave ? 1ull << (c2 & 63) : 0ull);
        bool todo = i < L && ar >= 1 && (nd.ent[ii] & kConst);
        for (int round = 0; round <= kWave; ++round) {
            const uint64_t left = __ballot(todo);
            if (left == 0ull) break;
            if (todo && (need & left) == 0) {
                float v[1] = {nd.val[c1]};
                const float second[1] = {nd.val[c2]};
                if (ar == 1) apply_unary<1>(unary_index(op), v, global_tabs());
                else apply_binary<1>(binary_index(op), v, second);
                nd.val[i] = v[0];
                todo = false;
            }
            wave_lds_sync();
        }
    }
    if ((nd.ent[0] & kEntMask) > kRegSlots + 1) return true;
    // ---- 3. and 4. places and instructions ----
    const int total = nd.cnt[0];
    if (lane == 0) {
        nd.start[0] = 0;
        nd.lev[0] = 0;
    }
    wave_lds_sync();
    for (int b = 0; b < nb; ++b) {
        const int i = b * kWave + lane;
        const bool valid = i < L;
        const uint32_t op = valid ? nd.op[i] : 0u;
        const int ar = arity(op);
        const int c1 = min(i + 1, L - 1), c2 = valid && ar == 2 ? nd.sec[i] : c1;
        const uint32_t ea = nd.ent[c1], eb = nd.ent[c2];
        const bool ta = ea & (kLeaf | kConst), tb = eb & (kLeaf | kConst);
        const bool is_c = valid && (nd.ent[min(i, L - 1)] & kConst);
        bool done = !valid;
        uint32_t start = 0xffffu, lev = 0;
        // a node whose place is known gives its evaluated operands theirs; a
        // round without a new one ends the block (the others belong to
        // constant subtrees or are fused)
        for (int round = 0; round <= kWave; ++round) {
            bool fresh = false;
            if (!done) {
                start = nd.start[i];
                if (start != 0xffffu) {
                    lev = nd.lev[i];
                    done = fresh = true;
                    if (ar == 1 && !is_c) {
                        nd.start[c1] = static_cast<uint16_t>(start);
                        nd.lev[c1] = static_cast<uint8_t>(lev);
                    } else if (ar == 2 && !is_c) {
                        // the operand evaluated first, and (if neither is a
                        // terminal) the one evaluated above it
                        const bool a_first = ta ? false : (tb ? true : (ea & kEntMask) > (eb & kEntMask));
                        const int f = a_first ? c1 : c2, s = a_first ? c2 : c1;
                        nd.lev[f] = static_cast<uint8_t>(lev);
                        nd.start[f] = static_cast<uint16_t>(start);
                        if (!ta && !tb) {
                            nd.lev[s] = static_cast<uint8_t>(lev + 1);
                            nd.start[s] = static_cast<uint16_t>(start + nd.cnt[f]);
                        }
                    }
                }
            }
            wave_lds_sync();
            if (__ballot(fresh) == 0) break;
        }
    }
    // features by instruction (-1: none) replace the constants' values, which
    // each lane reads before any is overwritten
    for (int b = 0; b < nb; ++b) {
        const int i = b * kWave + lane;
        const bool valid = i < L;
        const int ii = min(i, L - 1);
        const uint32_t start = valid ? nd.start[ii] : 0xffffu;
        if (start == 0xffffu) continue;
        const uint32_t op = nd.op[ii], lev = nd.lev[ii], me = nd.ent[ii];
        const int ar = arity(op);
        const int64_t pos = code_pos(start + nd.cnt[ii] - 1);
        uint32_t handler, payload = 0u;
        if (me & (kLeaf | kConst)) {
            const bool is_c = me & kConst;
            const uint32_t arg = is_c ? 0u : pn[ii] >> 8;
            const uint32_t src = em.source(is_c, arg);
            handler = lev == 0 ? em.set(src) : em.push(lev - 1, src);
            payload = is_c ? __float_as_uint(nd.val[ii]) : arg;
        } else if (ar == 1) {
            handler = em.handler(kOpUnary + unary_index(op));
        } else {
            const int c1 = ii + 1, c2 = nd.sec[ii];
            const uint32_t ea = nd.ent[c1], eb = nd.ent[c2];
            const bool ta = ea & (kLeaf | kConst), tb = eb & (kLeaf | kConst);
            const uint32_t fn = binary_index(op);
            if (ta || tb) {
                // terminal (op) top, or top (op) terminal
                const int c = ta ? c1 : c2;
                const bool is_c = (ta ? ea : eb) & kConst;
                const uint32_t arg = is_c ? 0u : pn[c] >> 8;
                handler = em.fold(bin_op(fn, !ta), em.source(is_c, arg));
                payload = is_c ? __float_as_uint(nd.val[c]) : arg;
            } else {
                // the second operand evaluated first, the first on top of it; or exchanged
                const bool a_first = (ea & kEntMask) > (eb & kEntMask);
                handler = em.bin(bin_op(fn, a_first), lev);
            }
        }
        out[pos] = make_uint2(handler, payload);
    }
    const int64_t end = code_pos(total);
    if (lane == 0) out[end] = make_uint2(em.handler(kOpEnd), 0u);
    for (int64_t r = 63 + 64 * static_cast<int64_t>(lane); r < end; r += 64 * kWave)
        out[r] = make_uint2(em.handler(kOpReload), 0u);
    uint32_t head = end >= 64 ? kHdrBlocks : 0u;
    if (em.mem) {
        // the fetch chain: each instruction that consumes a feature names the
        // next one's, found from the last instruction back
        wave_lds_sync();
        uint32_t* feat = reinterpret_cast<uint32_t*>(nd.val);
        for (int q = lane; q < total; q += kWave) feat[q] = 0xffffffffu;
        wave_lds_sync();
        for (int b = 0; b < nb; ++b) {
            const int i = b * kWave + lane;
            if (i >= L || nd.start[i] == 0xffffu) continue;
            const uint32_t op = nd.op[i], me = nd.ent[i];
            const int q = nd.start[i] + nd.cnt[i] - 1;
            if (me & kLeaf) {
                feat[q] = pn[i] >> 8;
            } else if (!(me & kConst) && arity(op) == 2) {
                const int c1 = i + 1, c2 = nd.sec[i];
                const uint32_t ea = nd.ent[c1], eb = nd.ent[c2];
                if (ea & kLeaf) feat[q] = pn[c1] >> 8;
                else if (!(ea & kConst) && (eb & kLeaf)) feat[q] = pn[c2] >> 8;
            }
        }
        wave_lds_sync();
        uint32_t next = 0xffffffffu;
        for (int q0 = (total - 1) & ~63; q0 >= 0; q0 -= kWave) {
            const int q = q0 + lane;
            const uint32_t f = q < total ? feat[q] : 0xffffffffu;
            const uint64_t m = __ballot(f != 0xffffffffu);
            const uint64_t right = lane < 63 ? m >> (lane + 1) : 0;
            const uint32_t fr = __shfl(f, right ? lane + 1 + __builtin_ctzll(right) : lane, kWave);
            if (f != 0xffffffffu) out[code_pos(q)].y = right ? fr : next;
            if (m) next = __shfl(f, __builtin_ctzll(m), kWave);
        }
        if (next != 0xffffffffu) head |= kHdrFetch | (next & kHdrFeature);
    }
    if (lane == 0) hdr[p] = head;
    return false;
}

// ---------------------------------------------------------------------------
// compile_adjoint_program: one wavefront per program of at most kParNodes nodes, as
// compile_eval_program: the forward instructions of the adjoint kernel (every
// constant stays, active operations record their partial derivatives), kOpEnd,
// the reverse instructions, kOpEnd.
// ---------------------------------------------------------------------------
// Forward and reverse instructions, tape entries, feature fetches: one word,
// read and written at once.
struct __align__(8) AdjCounts {
    uint16_t f, r, t, x;
};
struct AdjNodes {
    uint16_t sec[kParNodes];      // second operand of a binary function
    AdjCounts cnt[kParNodes];     // of the subtree
    AdjCounts start[kParNodes];   // where they begin (f = 0xffff: not known)
    uint8_t op[kParNodes], ent[kParNodes], lev[kParNodes];
    uint32_t feat[kParNodes / 2 + 1];   // the features in the order they are fetched
};
constexpr int kAdjCompileWaves = 2;
constexpr uint8_t kActiveEnt = 32;      // ent bit: the subtree holds a constant

// What a binary function does with its operands: which is fused (kOpFold...)
// or evaluated first, and in which order the function takes them.
struct BinShape {
    bool fold;      // one operand is a terminal, fused; else both are evaluated
    bool a_first;   // the first operand is the one evaluated first (fold: the one evaluated)
};
__device__ __forceinline__ BinShape bin_shape(uint32_t ea, uint32_t eb) {
    const bool ta = ea & kLeaf, tb = eb & kLeaf;
    return BinShape{ta || tb, ta ? false : (tb ? true : (ea & kEntMask) > (eb & kEntMask))};
}

// The instructions of one node itself, given to fw (forward) and rv (reverse):
// called to count them and again to write them, so the two agree.  For a
// function of one argument or a fold, E is the evaluated operand and T the
// fused terminal; else F is evaluated first (its value in slot `lev`), S on
// top of it.  Tape entry e of the node is tape(e).
template <typename Fw, typename Rv>
__device__ __forceinline__ void adjoint_ops(uint32_t op, bool act, uint32_t lev, bool leaf_const, uint32_t slot_c,
                                            float cval, uint32_t ea, uint32_t eb, const Emit& em, Fw&& fw, Rv&& rv) {
    auto id = [](uint32_t i) { return i * kOpBytes; };
    const int ar = arity(op);
    enum { kPlain = 0, kFetch = 1, kTape = 2 };      // what a payload names
    auto cadd = [&](uint32_t slot) __attribute__((always_inline)) {
        if (slot < static_cast<uint32_t>(kAccRegs)) rv(id(kACAdd + slot), 0u, kPlain);
        else rv(id(kACAddX), slot, kPlain);
    };
    if (ar == 0) {
        const uint32_t src = em.source(op == GP_OP_CONST, 0u);
        fw(lev == 0 ? em.set(src) : em.push(lev - 1, src), __float_as_uint(cval), op == GP_OP_CONST ? kPlain : kFetch);
        if (op == GP_OP_CONST) {
            rv(id(kAMovMT), 0u, kPlain);
            cadd(slot_c);
        }
        return;
    }
    if (ar == 1) {
        const uint32_t u = unary_index(op);
        if (!act) {
            fw(id(kOpUnary + u), 0u, kPlain);
        } else if (u == 0) {
            fw(id(kOpUnary + u), 0u, kPlain);
            rv(id(kOpUnary + u), 0u, kPlain);
        } else {
            if (u == 1) {
                fw(id(kADInvT), 0u, kPlain);
                fw(id(kAPutU), 0u, kTape);
                fw(id(kOpUnary + u), 0u, kPlain);
            } else if (u == 2) {
                fw(id(kAMovUT), 0u, kPlain);
                fw(id(kOpUnary + u), 0u, kPlain);
                fw(id(kADSqrt), 0u, kPlain);
                fw(id(kAPutU), 0u, kTape);
            } else {
                fw(id(u == 3 ? kASinD : u == 4 ? kACosD : kAUnX + u - kAUnFirst), 0u, kPlain);
                fw(id(kAPutU), 0u, kTape);
            }
            rv(id(kAGMul), 0u, kTape);
        }
        return;
    }
    const BinShape sh = bin_shape(ea, eb);
    const uint32_t fn = binary_index(op);
    if (sh.fold) {
        const bool t_is_a = !sh.a_first;
        const bool tc = leaf_const, e_act = (t_is_a ? eb : ea) & kActiveEnt;
        const uint32_t src = em.source(tc, 0u), cb = __float_as_uint(cval);
        if (!act || fn < 2 || (fn == 2 && tc)) {
            if (act && fn == 2) fw(id(kAPutT), 0u, kTape);
            fw(em.fold(bin_op(fn, !t_is_a), src), cb, tc ? kPlain : kFetch);
            if (!act) return;
            if (fn < 2) {
                // T - E carries -g to E; E - T carries -g to T
                if (tc) {
                    rv(id(fn == 1 && !t_is_a ? kANegMT : kAMovMT), 0u, kPlain);
                    cadd(slot_c);
                }
                if (e_act && fn == 1 && t_is_a) rv(id(kOpUnary + 0), 0u, kPlain);
            } else {
                rv(id(kAMMul), 0u, kTape);
                cadd(slot_c);
                if (e_act) rv(em.fold(kBMul, 0u), cb, kPlain);
            }
            return;
        }
        // the terminal as the operand register; entry 0 belongs to E (if
        // active), the next to T
        const uint32_t et = e_act ? 1u : 0u;
        fw(id(tc ? kASetMC : kASetMF), cb, tc ? kPlain : kFetch);
        if (fn == 2) {
            fw(id(kAPutM), 0u, kTape);
            fw(em.bin(kBMul, kRegSlots), 0u, kPlain);
        } else if (fn == 3) {
            fw(id(t_is_a ? kADInvT : kADInvM), 0u, kPlain);
            if (t_is_a) {
                if (tc) fw(id(kAPutU), et, kTape);
                if (e_act) {
                    fw(id(kADNegM), 0u, kPlain);
                    fw(id(kAPutU), 0u, kTape);
                }
            } else {
                if (e_act) fw(id(kAPutU), 0u, kTape);
                if (tc) {
                    fw(id(kADNegT), 0u, kPlain);
                    fw(id(kAPutU), et, kTape);
                }
            }
            fw(em.bin(t_is_a ? kBDivRev : kBDiv, kRegSlots), 0u, kPlain);
        } else {
            const uint32_t kind = fn == 4 ? (t_is_a ? 1u : 0u) : fn == 5 ? (t_is_a ? 3u : 2u) : (t_is_a ? 5u : 4u);
            fw(id(kABinX + kind), 0u, kPlain);
            if (e_act) fw(id(kAPutU), 0u, kTape);
            if (tc) fw(id(kAPutM), et, kTape);
        }
        if (tc) {
            rv(id(kAMMul), et, kTape);
            cadd(slot_c);
        }
        if (e_act) rv(id(kAGMul), 0u, kTape);
        return;
    }
    // both evaluated: S on top, F in slot lev; s_is_a: S is the function's first operand
    const bool s_is_a = !sh.a_first;
    const bool s_act = (s_is_a ? ea : eb) & kActiveEnt, f_act = (s_is_a ? eb : ea) & kActiveEnt;
    const uint32_t plain = em.bin(bin_op(fn, !s_is_a), lev);
    if (!act) {
        fw(plain, 0u, kPlain);
        return;
    }
    if (fn < 2) {
        fw(plain, 0u, kPlain);
        const bool s_neg = fn == 1 && !s_is_a, f_neg = fn == 1 && s_is_a;
        if (s_act && f_act) {
            if (f_neg) {
                rv(id(kANegMT), 0u, kPlain);
                rv(id(kASaveM + lev), 0u, kPlain);
            } else {
                rv(id(kOpSave + lev), 0u, kPlain);
            }
            if (s_neg) rv(id(kOpUnary + 0), 0u, kPlain);
        } else if (s_act ? s_neg : f_neg) {
            rv(id(kOpUnary + 0), 0u, kPlain);
        }
        return;
    }
    const uint32_t ef = s_act ? 1u : 0u;      // entry 0 belongs to S (if active), the next to F
    if (fn == 2) {
        if (f_act) fw(id(kAPutT), ef, kTape);
        if (s_act) {
            fw(id(kALoadM + lev), 0u, kPlain);
            fw(id(kAPutM), 0u, kTape);
        }
        fw(plain, 0u, kPlain);
    } else if (fn == 3) {
        fw(id(kALoadM + lev), 0u, kPlain);
        if (s_is_a) {                          // t / m
            fw(id(kADInvM), 0u, kPlain);
            if (s_act) fw(id(kAPutU), 0u, kTape);
            if (f_act) {
                fw(id(kADNegT), 0u, kPlain);
                fw(id(kAPutU), ef, kTape);
            }
        } else {                               // m / t
            fw(id(kADInvT), 0u, kPlain);
            if (f_act) fw(id(kAPutU), ef, kTape);
            if (s_act) {
                fw(id(kADNegM), 0u, kPlain);
                fw(id(kAPutU), 0u, kTape);
            }
        }
        fw(plain, 0u, kPlain);
    } else {
        fw(id(kALoadM + lev), 0u, kPlain);
        const uint32_t kind = fn == 4 ? (s_is_a ? 0u : 1u) : fn == 5 ? (s_is_a ? 2u : 3u) : (s_is_a ? 4u : 5u);
        fw(id(kABinX + kind), 0u, kPlain);
        if (s_act) fw(id(kAPutU), 0u, kTape);
        if (f_act) fw(id(kAPutM), ef, kTape);
    }
    if (s_act && f_act) {
        rv(id(kAMMul), ef, kTape);
        rv(id(kASaveM + lev), 0u, kPlain);
        rv(id(kAGMul), 0u, kTape);
    } else {
        rv(id(kAGMul), 0u, kTape);
    }
}

// A tape instruction's register form and entry as the form its tier takes.
__device__ __forceinline__ uint2 tape_ins(uint32_t handler, uint32_t e, int32_t R) {
    if (e < static_cast<uint32_t>(kTapeRegs)) return make_uint2(handler + e * kOpBytes, 0u);
    const uint32_t kind = (handler / kOpBytes - kAPutT) / kTapeRegs;     // PutT, PutM, PutU, GMul, MMul
    const uint32_t bytes = static_cast<uint32_t>(R * kWave * 4);
    if (e < static_cast<uint32_t>(kTapeRegs + kTapeLds))
        return make_uint2((kAPutTL + kind) * kOpBytes, (e - kTapeRegs) * bytes);
    return make_uint2((kAPutTG + kind) * kOpBytes, (e - kTapeRegs - kTapeLds) * bytes);
}

struct AdjCompile {
    uint4* code;
    uint32_t* hdr;
    Emit em;
    double* gextra;      // sums of constants beyond kGradLds (cleared here)
};

__device__ __forceinline__ void compile_adjoint_program(const PopView& pop, const AdjCompile& ac, AdjNodes& nd,
                                                        int32_t p, int lane) {
    uint4* __restrict__ code = ac.code;
    uint32_t* __restrict__ hdr = ac.hdr;
    const Emit& em = ac.em;
    const int64_t cend = pop.const_off[p + 1];
    for (int64_t i = pop.const_off[p] + lane; i < cend; i += kWave) ac.gextra[i] = 0.0;
    const int64_t off = pop.prog_off[p];
    const int32_t L = pop.len[p];
    if (L > kParNodes) return;         // (k_compile's)
    const uint32_t* pn = pop.nodes + off;
    const float* pc = pop.consts + pop.const_off[p];
    uint2* out = reinterpret_cast<uint2*>(code + off * kAdjCodePerNode);
    const int nb = (L + kWave - 1) / kWave;
    // ---- heights and second operands (as compile_eval_program) ----
    int carry = 0, lastpos = 0;
    uint64_t bad = 0;
    for (int b = nb - 1; b >= 0; --b) {
        const int i = b * kWave + lane;
        const bool valid = i < L;
        const uint32_t op = valid ? (pn[i] & 0xffu) : 0u;
        const int ar = arity(op);
        int hs = valid ? 1 - ar : 0;
        for (int d = 1; d < kWave; d <<= 1) {
            const int o = __shfl_down(hs, d, kWave);
            if (lane + d < kWave) hs += o;
        }
        bad |= __ballot(valid && malformed(ar, hs + carry));
        const int H = min(max(hs + carry, 0), 31);
        uint64_t same = 0, mine = 0;
        for (int hv = 1; hv <= GP_MAX_STACK; ++hv) {
            const uint64_t m = __ballot(valid && H == hv);
            if (H == hv) same = m;
            if (lane == hv) mine = m;
        }
        const uint64_t right = lane < 63 ? same >> (lane + 1) : 0;
        const int beyond = __shfl(lastpos, H, kWave);
        const int sec = right ? i + 1 + __builtin_ctzll(right) : beyond;
        if (mine) lastpos = b * kWave + __builtin_ctzll(mine);
        carry = __builtin_amdgcn_readfirstlane(hs + carry);
        if (valid) {
            nd.op[i] = static_cast<uint8_t>(op);
            nd.sec[i] = static_cast<uint16_t>(min(max(sec, 0), L - 1));
            nd.start[i].f = 0xffffu;
        }
    }
    if (bad || carry != 1) {       // nothing to do for a malformed program
        if (lane < 2 && L > 0) out[lane] = make_uint2(em.handler(kOpEnd), 0u);
        if (lane == 0) hdr[p] = 0u;
        return;
    }
    wave_lds_sync();
    // ---- from the leaves up: entries, activity, counts ----
    for (int b = nb - 1; b >= 0; --b) {
        const int i = b * kWave + lane;
        const bool valid = i < L;
        const uint32_t op = valid ? nd.op[i] : 0u;
        const int ar = arity(op);
        const int c1 = min(i + 1, L - 1), c2 = valid && ar == 2 ? nd.sec[i] : c1;
        const uint32_t o1 = nd.op[c1], o2 = nd.op[c2];
        bool done = !valid;
        const uint64_t need = (ar >= 1 && c1 < (b + 1) * kWave ? 1ull << (c1 & 63) : 0ull) |
                              (ar == 2 && c2 < (b + 1) * kWave ? 1ull << (c2 & 63) : 0ull);
        for (int round = 0; round <= kWave; ++round) {
            const uint64_t ready = __ballot(done);
            if (ready == ~0ull) break;
            // both operands' words at once, then the choice between them
            const uint32_t e1 = nd.ent[c1], e2 = nd.ent[c2];
            const AdjCounts n1 = nd.cnt[c1], n2 = nd.cnt[c2];
            if (!done && (need & ~ready) == 0) {
                const uint32_t ea = ar >= 1 ? e1 : 0u, eb = ar == 2 ? e2 : 0u;
                uint32_t ent = 1u | kLeaf, fc = op != GP_OP_CONST, cn = 0, rn = 0, tn = 0;
                const uint32_t act = ar == 0 ? op == GP_OP_CONST : ((ea | eb) & kActiveEnt) != 0u;
                bool tc = false;
                if (ar == 1) {
                    ent = max(ea & kEntMask, 1u);
                    cn = n1.f;
                    rn = n1.r;
                    tn = n1.t;
                    fc = n1.x;
                } else if (ar == 2) {
                    const BinShape sh = bin_shape(ea, eb);
                    const AdjCounts ne = sh.a_first ? n1 : n2, no = sh.a_first ? n2 : n1;
                    const uint32_t na = ea & kEntMask, nb2 = eb & kEntMask;
                    ent = sh.fold ? (sh.a_first ? na : nb2) : (na == nb2 ? na + 1u : max(na, nb2));
                    tc = sh.fold && (sh.a_first ? o2 : o1) == GP_OP_CONST;
                    cn = ne.f + (sh.fold ? 0u : no.f);
                    rn = ne.r + (sh.fold ? 0u : no.r + ((ea & eb & kActiveEnt) ? 1u : 0u));   // the slot taken back
                    tn = ne.t + (sh.fold ? 0u : no.t);
                    fc = n1.x + n2.x;
                }
                // the tape entries are the highest entry a forward instruction names, plus one
                // (the two counts in one word: as two variables the compiler keeps
                // them in memory, chosen by address)
                uint64_t n64 = static_cast<uint64_t>(rn) << 32 | cn;
                uint32_t te = 0;
                adjoint_ops(op, act, 0u, tc, 0u, 0.0f, ea, eb, em,
                            [&](uint32_t, uint32_t e, int kind) __attribute__((always_inline)) {
                                n64 += 1ull;
                                if (kind == 2) te = max(te, e + 1u);
                            },
                            [&](uint32_t, uint32_t, int) __attribute__((always_inline)) { n64 += 1ull << 32; });
                nd.ent[i] = static_cast<uint8_t>(ent | (act ? kActiveEnt : 0u));
                nd.cnt[i] = AdjCounts{static_cast<uint16_t>(n64), static_cast<uint16_t>(n64 >> 32),
                                      static_cast<uint16_t>(tn + te), static_cast<uint16_t>(fc)};
                done = true;
            }
            wave_lds_sync();
        }
    }
    // ---- from the root down: places ----
    const int total = nd.cnt[0].f, rtotal = nd.cnt[0].r;
    if (lane == 0) {
        nd.start[0] = AdjCounts{0, static_cast<uint16_t>(total + 1), 0, 0};
        nd.lev[0] = 0;
    }
    wave_lds_sync();
    for (int b = 0; b < nb; ++b) {
        const int i = b * kWave + lane;
        const bool valid = i < L;
        const uint32_t op = valid ? nd.op[i] : 0u;
        const int ar = arity(op);
        const int c1 = min(i + 1, L - 1), c2 = valid && ar == 2 ? nd.sec[i] : c1;
        const uint32_t ea = nd.ent[c1], eb = nd.ent[c2];
        // the operand evaluated first (a unary function's only one), and the other
        const BinShape sh = bin_shape(ea, eb);
        const int f = ar == 2 && !sh.a_first ? c2 : c1, q = f == c1 ? c2 : c1;
        const AdjCounts own = nd.cnt[min(i, L - 1)], nf = nd.cnt[f], nq = nd.cnt[q];
        const uint32_t back = (ea & eb & kActiveEnt) ? 1u : 0u;
        bool done = !valid;
        for (int round = 0; round <= kWave; ++round) {
            bool fresh = false;
            if (!done) {
                const AdjCounts at = nd.start[i];
                const uint32_t lev = nd.lev[i];
                if (at.f != 0xffffu) {
                    done = fresh = true;
                    if (ar >= 1) {
                        // the reverse part ends with the operand evaluated first
                        nd.lev[f] = static_cast<uint8_t>(lev);
                        nd.start[f] = AdjCounts{at.f, static_cast<uint16_t>(at.r + own.r - nf.r), at.t, at.x};
                        if (ar == 2 && !sh.fold) {
                            nd.lev[q] = static_cast<uint8_t>(lev + 1);
                            nd.start[q] = AdjCounts{static_cast<uint16_t>(at.f + nf.f),
                                                    static_cast<uint16_t>(at.r + own.r - nf.r - back - nq.r),
                                                    static_cast<uint16_t>(at.t + nf.t), static_cast<uint16_t>(at.x + nf.x)};
                        }
                    }
                }
            }
            wave_lds_sync();
            if (__ballot(fresh) == 0) break;
        }
    }
    // ---- the features in the order of their fetches ----
    for (int b = 0; b < nb; ++b) {
        const int i = b * kWave + lane;
        if (i >= L || nd.start[i].f == 0xffffu) continue;
        const uint32_t op = nd.op[i];
        if (op == GP_OP_VAR) {
            nd.feat[nd.start[i].x] = pn[i] >> 8;
        } else if (arity(op) == 2) {
            const int c1 = i + 1, c2 = nd.sec[i];
            const BinShape sh = bin_shape(nd.ent[c1], nd.ent[c2]);
            const int t = sh.a_first ? c2 : c1;
            if (sh.fold && nd.op[t] == GP_OP_VAR) nd.feat[nd.start[i].x + nd.cnt[i].x - 1] = pn[t] >> 8;
        }
    }
    wave_lds_sync();
    const int fetches = nd.cnt[0].x;
    // ---- instructions ----
    for (int b = 0; b < nb; ++b) {
        const int i = b * kWave + lane;
        if (i >= L || nd.start[i].f == 0xffffu) continue;
        const uint32_t op = nd.op[i], me = nd.ent[i], lev = nd.lev[i];
        const int ar = arity(op);
        const int c1 = min(i + 1, L - 1), c2 = ar == 2 ? nd.sec[i] : c1;
        const uint32_t ea = ar >= 1 ? nd.ent[c1] : 0u, eb = ar == 2 ? nd.ent[c2] : 0u;
        uint32_t q = nd.start[i].f;
        uint32_t tape = nd.start[i].t;
        int fetch = nd.start[i].x + nd.cnt[i].x - 1;     // this node's own, if it has one: its subtree's last
        int term = i;
        bool both = false;
        int ce = c1, co = c1;
        if (ar == 1) {
            q += nd.cnt[c1].f;
            tape += nd.cnt[c1].t;
        } else if (ar == 2) {
            const BinShape sh = bin_shape(ea, eb);
            ce = sh.a_first ? c1 : c2;
            co = sh.a_first ? c2 : c1;
            q += nd.cnt[ce].f;
            tape += nd.cnt[ce].t;
            if (sh.fold) {
                term = co;
            } else {
                q += nd.cnt[co].f;
                tape += nd.cnt[co].t;
                both = (ea & eb & kActiveEnt) != 0u;
            }
        }
        const bool is_c = nd.op[term] == GP_OP_CONST;
        const uint32_t slot_c = is_c ? pn[term] >> 8 : 0u;
        const float cval = is_c ? pc[slot_c] : 0.0f;
        // the next forward instruction in the low word, the next reverse one in
        // the high word
        uint64_t at2 = static_cast<uint64_t>(nd.start[i].r) << 32 | q;
        auto put = [&](uint32_t at, uint32_t handler, uint32_t payload, int kind) __attribute__((always_inline)) {
            uint2 ins = make_uint2(handler, payload);
            if (kind == 1) ins.y = fetch + 1 < fetches ? nd.feat[fetch + 1] : 0xffffffffu;
            else if (kind == 2) ins = tape_ins(handler, tape + payload, em.R);
            out[code_pos(at)] = ins;
        };
        adjoint_ops(op, (me & kActiveEnt) != 0u, lev, is_c, slot_c, cval, ea, eb, em,
                    [&](uint32_t h, uint32_t y, int kind) __attribute__((always_inline)) {
                        put(static_cast<uint32_t>(at2), h, y, kind);
                        at2 += 1ull;
                    },
                    [&](uint32_t h, uint32_t y, int kind) __attribute__((always_inline)) {
                        put(static_cast<uint32_t>(at2 >> 32), h, y, kind);
                        at2 += 1ull << 32;
                    });
        // between the two operands' reverse parts: the second's adjoint back on top
        if (both) put(nd.start[i].r + nd.cnt[i].r - nd.cnt[ce].r - 1u, (kOpLoadS + lev) * kOpBytes, 0u, 0);
    }
    const int64_t end = code_pos(total), end2 = code_pos(total + 1 + rtotal);
    if (lane == 0) {
        out[end] = make_uint2(em.handler(kOpEnd), 0u);
        out[end2] = make_uint2(em.handler(kOpEnd), 0u);
        hdr[p] = (end2 >= 64 ? kHdrBlocks : 0u) | (fetches ? kHdrFetch | (nd.feat[0] & kHdrFeature) : 0u);
    }
    for (int64_t x = 63 + 64 * static_cast<int64_t>(lane); x < end2; x += 64 * kWave)
        out[x] = make_uint2(em.handler(kOpReload), 0u);
}

// ---------------------------------------------------------------------------
// k_compile_streams: the evaluation kernel's stream of every program, the
// adjoint's, or both, a wavefront each; block 0 orders the programs.  A
// backward pass that evaluates first has the two compiled side by side (100
// programs of up to 120 nodes: 35 and 53 us one after the other; a refinement
// step of theirs on 10,007 rows 277 us with each compiler and the order in its
// own launch, 232 so; the fitness of 256 programs on 4,096 rows 25.6 and 22.3).  Their
// bound is the depth: each level of a tree is a round of dependent LDS reads.
// With the operands' words read together rather than as they were needed, and
// constant subtrees' functions in rounds of their own: evaluation streams of
// those 100 programs 35 -> 31 us, both streams 53 -> 49, the step 229 -> 220.
// ---------------------------------------------------------------------------
template <bool EVAL, bool ADJOINT>
constexpr int compile_waves() { return ADJOINT ? kAdjCompileWaves : kBlock / kWave; }

template <bool EVAL, bool ADJOINT>
__global__ __launch_bounds__((compile_waves<EVAL, ADJOINT>()) * kWave) void k_compile_streams(PopView pop, OrderArgs oa,
                                                                                        EvalCompile ec,
                                                                                        AdjCompile ac) {
    constexpr int kW = compile_waves<EVAL, ADJOINT>();
    constexpr size_t kLds = std::max(std::max(EVAL ? sizeof(EvalCompileLds) : 0, ADJOINT ? sizeof(AdjNodes) : 0) * kW,
                                     sizeof(OrderLds));
    __shared__ __align__(16) unsigned char lds[kLds];
    if (blockIdx.x == 0) {
        order_programs<kW * kWave>(oa, *reinterpret_cast<OrderLds*>(lds));
        return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = static_cast<int>(uniform(threadIdx.x >> 6));
    const int32_t per = (pop.P + kW - 1) / kW;      // blocks to compile one of the streams
    int32_t b = static_cast<int32_t>(blockIdx.x) - 1;
    // (the adjoint's first: it takes longer)
    if constexpr (ADJOINT) {
        if (b < per) {
            const int32_t p = b * kW + wid;
            if (p < pop.P) compile_adjoint_program(pop, ac, reinterpret_cast<AdjNodes*>(lds)[wid], p, lane);
            return;
        }
        b -= per;
    }
    if constexpr (EVAL) {
        EvalCompileLds& sh = reinterpret_cast<EvalCompileLds*>(lds)[wid];
        const int32_t p0 = (b * kW + wid) * ec.group, n = min(ec.group, pop.P - p0);
        uint64_t rest = 0;
        for (int32_t g = 0; g < n; ++g) {
            if (compile_eval_program(pop, ec, sh.nodes, p0 + g, lane)) rest |= 1ull << g;
            wave_lds_sync();
        }
        if (rest) compile_eval_rest(pop, ec, sh, p0, rest, lane);
    }
}

// ---------------------------------------------------------------------------
// k_find_user: raises flag[0] (which the caller zeroes, k_zero_u32) if any
// of the n nodes is a user function.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_find_user(const uint32_t* __restrict__ nodes, int64_t n,
                                                       uint32_t* __restrict__ flag) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * kBlock)
        if (is_user_op(nodes[i] & 0xffu)) flag[0] = 1u;
}

__global__ void k_zero_u32(uint32_t* __restrict__ p) { p[0] = 0u; }

// ---------------------------------------------------------------------------
// k_ystats: per chunk, float64 sums of the weights and of the shifted target
// (shift = y at the chunk's first row): S0 = sum w, S1 = sum w (y-K),
// S2 = sum w (y-K)^2, K.  One wavefront per chunk.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__global__ __launch_bounds__(kBlock) void k_ystats(DataView d, int64_t chunk, int32_t n_chunks,
                                                    double* __restrict__ ystat) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t c = static_cast<int64_t>(blockIdx.x) * (kBlock / kWave) + (threadIdx.x >> 6);
    if (c >= n_chunks) return;
    const int64_t r0 = c * chunk;
    const int64_t r1 = min(r0 + chunk, d.N);
    const double K = static_cast<double>(d.y[r0]);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int64_t r = r0 + lane; r < r1; r += kWave) {
        const double w = d.w ? static_cast<double>(d.w[r]) : 1.0;
        const double b = static_cast<double>(d.y[r]) - K;
        s0 += w;
        s1 += w * b;
        s2 += w * b * b;
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) {
        ystat[c * 4 + 0] = s0;
        ystat[c * 4 + 1] = s1;
        ystat[c * 4 + 2] = s2;
        ystat[c * 4 + 3] = K;
    }
}

// ---------------------------------------------------------------------------
// The evaluation kernel.
//   MODE 0: write every program output out[p * N + r]   (gp_evaluate)
//   MODE 1: accumulate the metric's float64 row sums per (program, chunk)
//           into part[(p * n_chunks + c) * KK + k]     (gp_fitness)
// R rows per lane; FREG > 0 keeps the tile's F <= FREG feature values in
// registers, FREG == 0 fetches each feature from memory where the program
// uses it, one use ahead.  The program itself runs in the interpreter of
// gp_eval_asm.h.
// ---------------------------------------------------------------------------
template <int METRIC>
struct MetricTraits {
    static constexpr int K = (METRIC == GP_METRIC_PEARSON) ? 3 : 1;   // moments per row
    static constexpr int KK = (METRIC == GP_METRIC_PEARSON) ? 4 : 1;  // doubles per partial
};

#define GP_ROWS(stmt)                  \
    _Pragma("unroll") for (int j = 0; j < R; ++j) { stmt; }

// Element j of an interpreter register group (a vector, or one value).
template <typename V>
__device__ __forceinline__ auto ev_get(const V& v, int j) {
    if constexpr (std::is_arithmetic_v<V>) return v;
    else return v[j];
}
template <typename V, typename T>
__device__ __forceinline__ void ev_set(V& v, int j, T x) {
    if constexpr (std::is_arithmetic_v<V>) v = x;
    else v[j] = x;
}
// The interpreter's constants: scalar register groups c0 and c1, vector ones k0
// and k1, in the generator's order.
__device__ __forceinline__ EvVec<uint32_t, 16> interp_c0() {
    const double c[8] = {crm::kInvPi128, crm::kPi128a, crm::kPi128b, crm::kS5, crm::kC4, crm::kL2, crm::kL3, crm::kL5};
    EvVec<uint32_t, 16> v{};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint64_t u = crm::dbits(c[q]);
        v[2 * q] = static_cast<uint32_t>(u);
        v[2 * q + 1] = static_cast<uint32_t>(u >> 32);
    }
    return v;
}
__device__ __forceinline__ EvVec<uint32_t, 8> interp_c1() {
    const uint64_t ln2 = crm::dbits(crm::kLn2), c375 = crm::dbits(0.375);
    return EvVec<uint32_t, 8>{static_cast<uint32_t>(ln2), static_cast<uint32_t>(ln2 >> 32),
                              static_cast<uint32_t>(c375), static_cast<uint32_t>(c375 >> 32),
                              crm::fbits(GP_PROTECT_EPS), 0x7fffffu, 0x240u, 4u};
}
template <typename I>
__device__ __forceinline__ void interp_vector_constants(I& in) {
    const double k[5] = {crm::kRound, crm::kRoundCos, crm::kS3, crm::kC2, crm::kL4};
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const uint64_t u = crm::dbits(k[q]);
        const float lo = crm::bitsf(static_cast<uint32_t>(u)), hi = crm::bitsf(static_cast<uint32_t>(u >> 32));
        if (q < 4) {
            in.k0[2 * q] = lo;
            in.k0[2 * q + 1] = hi;
        } else {
            in.k1[0] = lo;
            in.k1[1] = hi;
        }
    }
}

// The caller's part of the interpreter: the operation `code` on the top t (and
// the operand m) of R rows.  One test of the code for all rows, then the rows
// one after the other (their functions' registers would cost an occupancy
// step).  With the test inside the rows' loop each row went through it, and
// through another copy of every function: 777 programs over all 21 functions on
// 131,101 weighted rows took 3.51 ms, 2.95 so (max, min and the protected
// inverse, which used to come here too, became handlers with it).
template <int R, typename V>
__device__ __forceinline__ void leave_rows(uint32_t code, V& t, const V& m, const unsigned char* lds) {
    const MathTabsLds& tabs = *reinterpret_cast<const MathTabsLds*>(lds);
    const MathTabs mt{tabs.sc, tabs.lg};
    auto rows = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            float x[1] = {ev_get(t, j)};
            f(x, j);
            ev_set(t, j, x[0]);
            asm volatile("" : "+v"(t));
        }
    };
#define GP_LEAVE_UNARY(FN)                                                                  \
    case 1 + FN: rows([&](float (&x)[1], int) __attribute__((always_inline)) { apply_unary<1>(FN, x, mt); }); break
    switch (code) {
    GP_LEAVE_UNARY(1);
    GP_LEAVE_UNARY(3);
    GP_LEAVE_UNARY(4);
    GP_LEAVE_UNARY(5);
    GP_LEAVE_UNARY(7);
    GP_LEAVE_UNARY(11);
    GP_LEAVE_UNARY(12);
    GP_LEAVE_UNARY(13);
    case kExitAtan2TM:
        rows([&](float (&x)[1], int j) __attribute__((always_inline)) {
            const float y[1] = {ev_get(m, j)};
            apply_binary_wide<1>(6, x, y);
        });
        break;
    default:
        rows([&](float (&x)[1], int j) __attribute__((always_inline)) {
            float y[1] = {ev_get(m, j)};
            apply_binary_wide<1>(6, y, x);
            x[0] = y[0];
        });
        break;
    }
#undef GP_LEAVE_UNARY
}

// LDS: the function tables (at offset 0, where the interpreter expects them),
// then s.lds_slots * R * 64 stack words per wavefront (dynamic, sized at launch:
// kEvalLds slots, or kEvalLdsUser when user functions may be expanded).
// Wavefronts per SIMD asked of the compiler: what the interpreter's own
// registers leave room for.
constexpr int eval_waves(int R, int freg) {
    return R == 1 ? (freg == 8 ? 6 : 7) : R == 2 ? (freg == 8 ? 4 : 5) : (freg == 8 ? 3 : 4);
}

template <int R, int FREG, int MODE, int METRIC>
__global__ __launch_bounds__(kBlock, eval_waves(R, FREG)) void k_eval(PopView pop, CodeView cv, DataView d, Sched s,
                                                  float* __restrict__ out,
                                                  double* __restrict__ part) {
    constexpr int K = MetricTraits<METRIC>::K;
    constexpr int KK = MetricTraits<METRIC>::KK;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t N = d.N;
    const int64_t ld = d.ld;
    const float* __restrict__ X = d.X;
    extern __shared__ __align__(16) unsigned char lds_all[];
    stage_tabs(*reinterpret_cast<MathTabsLds*>(lds_all));

    Interp<R, FREG> in;
    in.c0 = interp_c0();
    in.c1 = interp_c1();
    interp_vector_constants(in);
    const uint32_t wid = uniform(threadIdx.x >> 6);
    in.lds = static_cast<uint32_t>(sizeof(MathTabsLds)) + wid * static_cast<uint32_t>(s.lds_slots * R * kWave * 4);
    if constexpr (FREG == 0) in.ld4 = static_cast<uint64_t>(ld) * 4u;

    const uint32_t P = static_cast<uint32_t>(pop.P);
    Claims claims(s, P, wid);
    int qx;
    uint32_t it0, it1;
    while (claims.next(lane, &qx, &it0, &it1)) {
        it0 = uniform(it0);
        it1 = uniform(it1);
        qx = static_cast<int>(uniform(static_cast<uint32_t>(qx)));
        uint32_t cq = it0 / claims.per, k = it0 - cq * claims.per;
        for (uint32_t it = it0; it < it1; ++it) {
            const int32_t c = claims.chunk(cq, qx);
            const uint32_t place = claims.program(k, qx);
            if (++k == claims.per) {
                k = 0;
                ++cq;
            }
            if (place >= P) continue;
            const int32_t p = ldu(s.order + place);
            const int64_t off = ldu(pop.prog_off + p);
            const uint32_t head = ldu(cv.ehdr + p);
            const uint4* __restrict__ pcode = cv.ecode + off * cv.ex_mul + static_cast<int64_t>(p) * cv.ex_add;
            in.ins = reinterpret_cast<const EvVec<uint32_t, 2>*>(pcode)[lane];
            const int64_t r0 = static_cast<int64_t>(c) * s.chunk;
            const int64_t r1 = min(r0 + s.chunk, N);

            double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0;
            float shift = 0.0f, yshift = 0.0f;     // (scalar registers)
            if constexpr (METRIC == GP_METRIC_PEARSON) yshift = ldu(d.y + r0);
            bool first_tile = true;

            for (int64_t base = r0; base < r1; base += kWave * R) {
                // byte offset of row j * 64 + lane; rows past the chunk's end
                // repeat its last one
                const int left = static_cast<int>(min<int64_t>(r1 - base, kWave * R));
                auto row_off = [left](int ln, int j) {
                    return static_cast<uint32_t>(min(j * kWave + ln, left - 1)) * 4u;
                };
                auto at = [](const float* col, uint32_t o) {
                    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(col) + o);
                };
                if constexpr (FREG > 0) {
#pragma unroll
                    for (int f = 0; f < FREG; ++f)
                        if (f < d.F) {
                            const float* __restrict__ col = X + f * ld + base;
                            GP_ROWS(in.x0[f * R + j] = at(col, row_off(lane, j)));
                        }
                } else {
                    in.xb = reinterpret_cast<uint64_t>(X + base);
                    GP_ROWS(ev_set(in.off, j, row_off(lane, j)));
                    if (head & kHdrFetch) {
                        const float* __restrict__ col = X + static_cast<int64_t>(head & kHdrFeature) * ld + base;
                        GP_ROWS(ev_set(in.p, j, at(col, row_off(lane, j))));
                    }
                }
                if constexpr (METRIC == GP_METRIC_USER_0) GP_ROWS(ev_set(in.t, j, at(d.y + base, row_off(lane, j))));
                const uint64_t blk = reinterpret_cast<uint64_t>(pcode);
                in.blk0 = static_cast<uint32_t>(blk);
                in.blk1 = static_cast<uint32_t>(blk >> 32);
                if ((head & kHdrBlocks) && !first_tile) in.ins = reinterpret_cast<const EvVec<uint32_t, 2>*>(pcode)[lane];
                in.idx = 0;
                uint32_t code;
                while ((code = in.run()) != kExitEnd) leave_rows<R>(code, in.t, in.m, lds_all);
                float t[R];
                GP_ROWS(t[j] = ev_get(in.t, j));
                // (row offsets and targets are formed here again rather than held
                // across the program: their registers would cost an occupancy step)
                int ln = lane;
                asm volatile("" : "+v"(ln));
                bool valid[R];
                GP_ROWS(valid[j] = j * kWave + ln < left);

                if constexpr (MODE == 0) {
                    float* __restrict__ o = out + static_cast<int64_t>(p) * N + base;
#pragma unroll
                    for (int j = 0; j < R; ++j)
                        if (valid[j]) o[j * kWave + ln] = t[j];
                } else {
                    float yv4[R], wv4[R];
                    GP_ROWS(yv4[j] = at(d.y + base, row_off(ln, j)));
                    if (d.w) {
                        GP_ROWS(wv4[j] = at(d.w + base, row_off(ln, j)));
                    } else {
                        GP_ROWS(wv4[j] = 1.0f);
                    }
                    if constexpr (METRIC == GP_METRIC_PEARSON) {
                        if (first_tile) shift = __uint_as_float(uniform(__float_as_uint(t[0])));
                    }
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const float yv = yv4[j];
                        const double wv = static_cast<double>(wv4[j]);
                        if constexpr (METRIC == GP_METRIC_MSE || METRIC == GP_METRIC_RMSE) {
                            const double e = static_cast<double>(t[j]) - static_cast<double>(yv);
                            const double l = e * e;
                            const double term = wv * l;
                            acc0 += valid[j] ? term : 0.0;
                        } else if constexpr (METRIC == GP_METRIC_MAE) {
                            const double e = static_cast<double>(t[j]) - static_cast<double>(yv);
                            const double term = wv * fabs(e);
                            acc0 += valid[j] ? term : 0.0;
                        } else if constexpr (METRIC == GP_METRIC_USER_0) {
                            // a user loss: the stream already ends in the row loss
                            (void)yv;
                            const double term = wv * static_cast<double>(t[j]);
                            acc0 += valid[j] ? term : 0.0;
                        } else if constexpr (METRIC == GP_METRIC_LOGLOSS) {
                            const float z = t[j];
                            const float t1 = fmaxf(z, 0.0f);
                            const float t2 = yv * z;
                            const float t3 = t1 - t2;
                            const float t5 = crm::log1p_exp_neg(fabsf(z), reinterpret_cast<const MathTabsLds*>(lds_all)->lg, crm::log_k());
                            const double term = wv * static_cast<double>(t3 + t5);
                            acc0 += valid[j] ? term : 0.0;
                            asm volatile("" : "+v"(acc0));     // (one row after the other)
                        } else {  // PEARSON: shifted first and second moments
                            const double a = static_cast<double>(t[j]) - static_cast<double>(shift);
                            const double bb = static_cast<double>(yv) - static_cast<double>(yshift);
                            const double wa = wv * a;
                            acc0 += valid[j] ? wa : 0.0;
                            acc1 += valid[j] ? wa * a : 0.0;
                            acc2 += valid[j] ? wa * bb : 0.0;
                        }
                    }
                }
                first_tile = false;
            }
            if constexpr (MODE == 1) {
                acc0 = wave_sum(acc0);
                if constexpr (K > 1) {
                    acc1 = wave_sum(acc1);
                    acc2 = wave_sum(acc2);
                }
                if (lane == 0) {
                    double* dst = part + (static_cast<int64_t>(p) * s.n_chunks + c) * KK;
                    dst[0] = acc0;
                    if constexpr (K > 1) {
                        dst[1] = acc1;
                        dst[2] = acc2;
                        dst[3] = static_cast<double>(shift);
                    }
                }
            }
        }
    }
}
#undef GP_ROWS

// ---------------------------------------------------------------------------
// k_finalize: merge each program's chunk partials in a fixed order (float64)
// and apply the metric.  One wavefront per program.
// ---------------------------------------------------------------------------
struct Moments {  // weighted count, means and centred second moments
    double W, ma, mb, Maa, Mbb, Mab;
};

__device__ __forceinline__ Moments merge(const Moments& x, const Moments& y) {
    // pairwise update (Chan, Golub, LeVeque) for weighted means and
    // co-moments
    if (!(x.W > 0.0)) return y;
    if (!(y.W > 0.0)) return x;
    Moments m;
    m.W = x.W + y.W;
    const double da = y.ma - x.ma, db = y.mb - x.mb;
    const double f = x.W * y.W / m.W;
    m.ma = x.ma + da * (y.W / m.W);
    m.mb = x.mb + db * (y.W / m.W);
    m.Maa = x.Maa + y.Maa + da * da * f;
    m.Mbb = x.Mbb + y.Mbb + db * db * f;
    m.Mab = x.Mab + y.Mab + da * db * f;
    return m;
}

__device__ __forceinline__ Moments shfl_moments(const Moments& m, int src) {
    Moments r;
    r.W = __shfl_xor(m.W, src, kWave);
    r.ma = __shfl_xor(m.ma, src, kWave);
    r.mb = __shfl_xor(m.mb, src, kWave);
    r.Maa = __shfl_xor(m.Maa, src, kWave);
    r.Mbb = __shfl_xor(m.Mbb, src, kWave);
    r.Mab = __shfl_xor(m.Mab, src, kWave);
    return r;
}

// stats (nullable) receives per program: [0] sum of weights W, [1] mean of
// yhat, [2] mean of y, [3] sum w (yhat - mean)^2, [4] sum w (y - mean)^2,
// [5] sum w (yhat - mean)(y - mean), [6] the metric in float64 (Pearson: the
// signed r), [7] unused.
constexpr int kStats = 8;

template <int METRIC>
__global__ __launch_bounds__(kBlock) void k_finalize(const double* __restrict__ part,
                                                      const double* __restrict__ ystat,
                                                      int32_t n_chunks, int32_t P, int64_t N,
                                                      int has_w, float* __restrict__ fitness,
                                                      double* __restrict__ stats) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t p = static_cast<int64_t>(blockIdx.x) * (kBlock / kWave) + (threadIdx.x >> 6);
    if (p >= P) return;
    if constexpr (METRIC == GP_METRIC_PEARSON) {
        Moments m{0, 0, 0, 0, 0, 0};
        for (int c = lane; c < n_chunks; c += kWave) {
            const double* q = part + (p * n_chunks + c) * 4;
            const double* ys = ystat + static_cast<int64_t>(c) * 4;
            Moments x;
            x.W = ys[0];
            const double Sa = q[0], Saa = q[1], Sab = q[2], Ka = q[3];
            const double Sb = ys[1], Sbb = ys[2], Kb = ys[3];
            x.ma = Ka + Sa / x.W;
            x.mb = Kb + Sb / x.W;
            x.Maa = Saa - Sa * (Sa / x.W);
            x.Mbb = Sbb - Sb * (Sb / x.W);
            x.Mab = Sab - Sa * (Sb / x.W);
            m = merge(m, x);
        }
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) m = merge(m, shfl_moments(m, off));
        if (lane == 0) {
            const double va = m.Maa, vb = m.Mbb;
            double r = 0.0;
            if (va > 0.0 && vb > 0.0 && isfinite(va) && isfinite(vb)) r = m.Mab / sqrt(va * vb);
            fitness[p] = static_cast<float>(fabs(r));
            if (stats) {
                double* o = stats + p * kStats;
                o[0] = m.W; o[1] = m.ma; o[2] = m.mb; o[3] = m.Maa; o[4] = m.Mbb; o[5] = m.Mab;
                o[6] = r; o[7] = 0.0;
            }
        }
    } else {
        double s = 0.0, sw = 0.0;
        for (int c = lane; c < n_chunks; c += kWave) {
            s += part[p * n_chunks + c];
            if (has_w) sw += ystat[static_cast<int64_t>(c) * 4];
        }
        s = wave_sum(s);
        sw = has_w ? wave_sum(sw) : static_cast<double>(N);
        if (lane == 0) {
            double v = s / sw;
            if constexpr (METRIC == GP_METRIC_RMSE) v = sqrt(v);
            fitness[p] = static_cast<float>(v);
            if (stats) {
                double* o = stats + p * kStats;
                o[0] = sw; o[1] = o[2] = o[3] = o[4] = o[5] = 0.0; o[6] = v; o[7] = 0.0;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// k_adjoint_long: derivative of every program's fitness with respect to each
// of its constants (not in the paper), by reverse mode over the compiled
// instructions, one wavefront per (row chunk, program) work item; for
// programs of more than kParNodes nodes (k_adjoint takes the rest: its compiler
// holds a program's nodes in LDS).
//
// Per tile of 64*R rows: a forward pass runs the stack machine and records
// on a tape the local derivatives each instruction will need (both partials
// of a product or quotient; the derivative of log, sqrt, sin, cos, tan at
// its input); the seed is d fitness / d yhat of each row; a reverse pass
// walks the instructions back with an adjoint stack that mirrors the value
// stack, multiplying by the taped partials, and at each constant reduces its
// adjoint over the wavefront into a per-program float64 sum.  Only
// instructions whose subtree holds a constant (kActive) record partials, and
// the reverse pass jumps over every subtree without one.  The first
// tape_lds_bytes<R>() of each wavefront's tape live in LDS, the rest (long
// programs) in a per-wavefront global area; the forward values are
// recomputed per tile, never kept.  Local derivatives (reading): add (1,1),
// sub (1,-1), mul (b,a), div (1/b, -a/b^2) if |b| > 0.001 else (0,0),
// log 1/a if |a| > 0.001 else 0, sqrt sign(a)/(2 sqrt|a|) (0 at a = 0),
// sin cos a, cos -sin a, tan 1 + tan^2 a, neg -1.
// ---------------------------------------------------------------------------
constexpr int kGradLds = 16;            // constants per program summed in a fixed order
// Four wavefronts a block share one LDS copy of the function tables (8 KB); they
// work independently of each other.  Per-wavefront tape held in LDS: 12 KB,
// 15 KB at 4 rows per lane (two waves per SIMD there, so eight per CU still
// fit in LDS)
constexpr int kAdjWaves = 4;
template <int R>
constexpr int tape_lds_bytes() { return R == 4 ? 15360 : 12288; }

// tape entries an instruction records (0, 1 or 2)
__device__ __forceinline__ int tape_entries(uint32_t cls, uint32_t fn) {
    if (cls == kPush) return 0;
    if (cls == kUn) return fn == 0 ? 0 : 1;           // neg: the constant -1
    return fn >= 2 ? 2 : 0;                           // mul / div: both partials
}

// floats of a wavefront's global area: value- and adjoint-stack overflow, then
// the tape entries beyond those in LDS
template <int R>
constexpr int64_t adjoint_wave_floats(int64_t tape_entries_max) {
    const int64_t lds_entries = tape_lds_bytes<R>() / (R * kWave * 4);
    const int64_t beyond = tape_entries_max > lds_entries ? tape_entries_max - lds_entries : 0;
    return (2 * kStackLds + beyond) * R * kWave;
}

// t = sin t (is_cos false) or cos t and dv = the derivative at the input, on
// the R rows of a lane.  With theta the table's angle, sin and cos are both
// sin(theta + r) = S cos r + C sin r, whose derivative C cos r - S sin r takes
// two more operations on the same reduction, table entry and polynomials (a
// library cos or sin at the input cost about thirty).
template <int R>
__device__ __forceinline__ void sincos_rows_derivative(bool is_cos, float (&t)[R], float (&dv)[R],
                                                       const MathTabs& mt) {
    const crm::SinCosK K = crm::sincos_k(is_cos);
    float f[R];
    bool rare = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const crm::SinCosArg a = crm::sincos_reduce(static_cast<double>(t[j]), K);
        const crm::SinCosEntry& e = crm::sincos_entry(mt.sc, a.off);
        double sr, cr;
        crm::sincos_poly(a.r, K, &sr, &cr);
        f[j] = static_cast<float>(fma(e.c, sr, e.s * cr));
        dv[j] = static_cast<float>(fma(-e.s, sr, e.c * cr));
        rare |= crm::sincos_rare_input(t[j]);
    }
    if (rare) {
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (crm::sincos_rare_input(t[j])) {
                f[j] = crm::sincos_rare(t[j], is_cos, mt.sc, K);
                const float g = crm::sincos_rare(t[j], !is_cos, mt.sc, K);
                dv[j] = is_cos ? -g : g;
            }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) t[j] = f[j];
}

// derivative of unary function fn (1, 2, 5: log, sqrt, tan; 6..13:
// abs, exp, inv, sq, cube, tanh, atan, cbrt) at input x, whose result is y.
// Reciprocals here (and in the quotient's partials) come from the hardware
// reciprocal, within 1 ulp: a partial's own rounding, well inside the
// derivative tolerance, at a tenth of a correctly rounded division's cost.
// Every argument is normal: |x| > 0.001, 2 sqrt|x| >= 2^-73.5, 1 + x^2 >= 1,
// 3 cbrt(x)^2 >= 2^-99 for nonzero float x.
template <int R>
__device__ __forceinline__ void unary_derivative(uint32_t fn, const float (&x)[R], const float (&y)[R],
                                                 float (&dv)[R]) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
        switch (fn) {
        case 1: dv[j] = fabsf(x[j]) > GP_PROTECT_EPS ? __builtin_amdgcn_rcpf(x[j]) : 0.0f; break;
        case 2: dv[j] = x[j] == 0.0f ? 0.0f : copysignf(__builtin_amdgcn_rcpf(2.0f * y[j]), x[j]); break;
        case 5: dv[j] = 1.0f + y[j] * y[j]; break;
        case 6: dv[j] = x[j] > 0.0f ? 1.0f : (x[j] < 0.0f ? -1.0f : 0.0f); break;
        case 7: dv[j] = y[j]; break;
        case 8: dv[j] = fabsf(x[j]) > GP_PROTECT_EPS ? -y[j] * y[j] : 0.0f; break;
        case 9: dv[j] = 2.0f * x[j]; break;
        case 10: dv[j] = 3.0f * (x[j] * x[j]); break;
        case 11: dv[j] = 1.0f - y[j] * y[j]; break;
        case 12: dv[j] = __builtin_amdgcn_rcpf(1.0f + x[j] * x[j]); break;
        default: dv[j] = y[j] != 0.0f ? __builtin_amdgcn_rcpf(3.0f * (y[j] * y[j])) : 0.0f; break;
        }
    }
}

template <int R, int METRIC>
__global__ __launch_bounds__(kAdjWaves * kWave) void k_adjoint_long(PopView pop, CodeView cv, DataView d, Sched s,
                                                    const double* __restrict__ stats,
                                                    const double* __restrict__ wsum,
                                                    const float* __restrict__ gscale,
                                                    double* __restrict__ part,
                                                    double* __restrict__ gpart,
                                                    double* __restrict__ gextra,
                                                    float* __restrict__ gmem,
                                                    int64_t wave_floats) {
    constexpr int kTapeLds = tape_lds_bytes<R>() / (R * kWave * 4);
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int64_t N = d.N;
    const int64_t ld = d.ld;
    const float* __restrict__ X = d.X;
    __shared__ float ltape_all[kAdjWaves][kTapeLds * R * kWave];
    __shared__ double gw_all[kAdjWaves][kGradLds];
    float* ltape = ltape_all[wid];
    double* gw = gw_all[wid];
    float* __restrict__ wmem = gmem + (static_cast<int64_t>(blockIdx.x) * kAdjWaves + wid) * wave_floats;
    float* __restrict__ ovf = wmem;                                 // value stack beyond registers
    float* __restrict__ aovf = wmem + kStackLds * R * kWave;        // adjoint stack beyond registers
    float* __restrict__ gtape = wmem + 2 * kStackLds * R * kWave;   // tape entries beyond LDS
    const double W = *wsum;
    __shared__ MathTabsLds tabs_lds;
    const MathTabs mt = stage_tabs(tabs_lds);

    // entry e of row slot j: LDS for e < kTapeLds, the global area beyond
    auto tape_put = [&](int e, const float (&v)[R]) {
        if (e < kTapeLds) {
#pragma unroll
            for (int j = 0; j < R; ++j) ltape[(e * R + j) * kWave + lane] = v[j];
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) gtape[((e - kTapeLds) * R + j) * kWave + lane] = v[j];
        }
    };
    auto tape_get = [&](int e, float (&v)[R]) {
        if (e < kTapeLds) {
#pragma unroll
            for (int j = 0; j < R; ++j) v[j] = ltape[(e * R + j) * kWave + lane];
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) v[j] = gtape[((e - kTapeLds) * R + j) * kWave + lane];
        }
    };

    // work items: the evaluation kernel's per-XCD queues, one item per claim
    Claims claims(s, ldu(s.counter + kLongWord), static_cast<uint32_t>(wid));
    int qx;
    uint32_t it, it_end;
    while (claims.next(lane, &qx, &it, &it_end)) {
        it = uniform(it);
        qx = static_cast<int>(uniform(static_cast<uint32_t>(qx)));
        const uint32_t cq = it / claims.per, place = claims.program(it - cq * claims.per, qx);
        if (place >= claims.P) continue;
        const int32_t c = claims.chunk(cq, qx);
        const int32_t p = ldu(s.order + place);
        const int64_t off = ldu(pop.prog_off + p);
        const int32_t CL = ldu(cv.clen + p);
        const int64_t cbase = ldu(pop.const_off + p);
        const int32_t nconst = static_cast<int32_t>(ldu(pop.const_off + p + 1) - cbase);
        const uint4* __restrict__ pcode = cv.code + off * kAdjCodePerNode;
        const int64_t r0 = static_cast<int64_t>(c) * s.chunk;
        const int64_t r1 = min(r0 + s.chunk, N);
        const float gsc = gscale ? ldu(gscale + p) : 1.0f;
        double sm0 = 0.0, sm1 = 0.0, sm2 = 0.0, sm3 = 0.0, sm4 = 0.0, sm5 = 0.0, sm6 = 0.0;
        if (stats) {
            sm0 = stats[p * kStats + 0]; sm1 = stats[p * kStats + 1]; sm2 = stats[p * kStats + 2];
            sm3 = stats[p * kStats + 3]; sm4 = stats[p * kStats + 4]; sm5 = stats[p * kStats + 5];
            sm6 = stats[p * kStats + 6];
        }
        (void)sm0; (void)sm5;
        const int nlds = min(nconst, kGradLds);
        if (lane < nlds) gw[lane] = 0.0;
        wave_lds_sync();
        double lacc = 0.0;
        // a program without constants needs only its loss, and only when asked
        const int64_t r_end = (nconst == 0 && !part) ? r0 : r1;

        for (int64_t base = r0; base < r_end; base += kWave * R) {
            int64_t row[R];
            bool valid[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int64_t r = base + j * kWave + lane;
                valid[j] = r < r1;
                row[j] = valid[j] ? r : r1 - 1;
            }
            // ---------------- forward pass, recording the tape ----------------
            float t[R];
#pragma unroll
            for (int j = 0; j < R; ++j) t[j] = 0.0f;
            GP_ARRAYS(st, kStackRegs + 1);
            int dp = -1;
            int ntape = 0;
            uint4 nxt = pcode[0];
            for (int q = 0; q < CL; ++q) {
                const uint4 cur = nxt;
                nxt = pcode[min(q + 1, CL - 1)];
                const uint32_t w = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(cur.x)));
                const uint32_t cls = w & 3u;
                const uint32_t fn = (w >> 2) & 15u;
                const bool act = (w & kActive) != 0u;
                GP_PUT(st, min(dp + 1, kStackRegs), t);
                float a[R], b[R];
                bool binary = false;
                if (cls == kUn) {
                    float x[R];
#pragma unroll
                    for (int j = 0; j < R; ++j) x[j] = t[j];
                    if (act && (fn == 3 || fn == 4)) {
                        float dv[R];
                        sincos_rows_derivative<R>(fn == 4, t, dv, mt);
                        tape_put(ntape, dv);
                        ++ntape;
                    } else {
                        apply_unary<R>(fn, t, mt);
                        if (fn != 0 && act) {
                            float dv[R];
                            unary_derivative<R>(fn, x, t, dv);
                            tape_put(ntape, dv);
                            ++ntape;
                        }
                    }
                } else if (cls == kBin) {
                    if (dp < kStackRegs) {
                        GP_GET(st, dp, b);
                    } else {
#pragma unroll
                        for (int j = 0; j < R; ++j) b[j] = ovf[((dp - kStackRegs) * R + j) * kWave + lane];
                    }
                    --dp;
#pragma unroll
                    for (int j = 0; j < R; ++j) a[j] = t[j];
                    binary = true;
                } else {
                    float v[R];
                    if (w & kConstBit) {
                        const float cval = __uint_as_float(cur.y);
#pragma unroll
                        for (int j = 0; j < R; ++j) v[j] = cval;
                    } else {
                        const float* __restrict__ col = X + static_cast<int64_t>(w >> 8) * ld;
#pragma unroll
                        for (int j = 0; j < R; ++j) v[j] = col[row[j]];
                    }
                    if (cls == kPush) {
                        ++dp;
                        if (dp >= kStackRegs) {
#pragma unroll
                            for (int j = 0; j < R; ++j) ovf[((dp - kStackRegs) * R + j) * kWave + lane] = t[j];
                        }
#pragma unroll
                        for (int j = 0; j < R; ++j) t[j] = v[j];
                    } else {
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            a[j] = v[j];
                            b[j] = t[j];
                        }
                        binary = true;
                    }
                }
                if (binary) {
                    if (fn >= 2 && act) {   // mul, div, max, min, atan2: both partials
                        float da[R], db[R];
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            if (fn == 2) {
                                da[j] = b[j];
                                db[j] = a[j];
                            } else if (fn == 3) {
                                if (fabsf(b[j]) > GP_PROTECT_EPS) {
                                    const float inv = __builtin_amdgcn_rcpf(b[j]);
                                    da[j] = inv;
                                    db[j] = -a[j] * inv * inv;
                                } else {
                                    da[j] = 0.0f;
                                    db[j] = 0.0f;
                                }
                            } else if (fn == 4 || fn == 5) {
                                // the selected operand (the first on ties) carries it
                                const bool first = (fn == 4 ? a[j] >= b[j] : a[j] <= b[j]) || isnan(b[j]);
                                da[j] = first ? 1.0f : 0.0f;
                                db[j] = first ? 0.0f : 1.0f;
                            } else {
                                const float r2 = a[j] * a[j] + b[j] * b[j];
                                da[j] = r2 > 0.0f ? b[j] / r2 : 0.0f;
                                db[j] = r2 > 0.0f ? -a[j] / r2 : 0.0f;
                            }
                        }
                        tape_put(ntape, da);
                        tape_put(ntape + 1, db);
                        ntape += 2;
                    }
                    apply_binary<R>(fn, a, b);
#pragma unroll
                    for (int j = 0; j < R; ++j) t[j] = a[j];
                }
                // the chained unary functions, each taping its derivative
                for (uint32_t ch = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(cur.z)));
                     ch != 0u; ch >>= 4) {
                    const uint32_t u = (ch & 15u) - 1u;
                    float x[R];
#pragma unroll
                    for (int j = 0; j < R; ++j) x[j] = t[j];
                    if (act && (u == 3 || u == 4)) {
                        float dv[R];
                        sincos_rows_derivative<R>(u == 4, t, dv, mt);
                        tape_put(ntape, dv);
                        ++ntape;
                    } else {
                        apply_unary<R>(u, t, mt);
                        if (u != 0 && act) {
                            float dv[R];
                            unary_derivative<R>(u, x, t, dv);
                            tape_put(ntape, dv);
                            ++ntape;
                        }
                    }
                }
            }

            // ---------------- seeds: d fitness / d yhat per row ----------------
            float g[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const double yh = static_cast<double>(t[j]);
                const double yv = static_cast<double>(d.y[row[j]]);
                const double wv = d.w ? static_cast<double>(d.w[row[j]]) : 1.0;
                double sd;
                if constexpr (METRIC == GP_METRIC_MSE) {
                    const double e = yh - yv;
                    sd = 2.0 * wv * e / W;
                    lacc += valid[j] ? wv * (e * e) : 0.0;
                } else if constexpr (METRIC == GP_METRIC_RMSE) {
                    const double e = yh - yv;
                    sd = sm6 > 0.0 ? (wv * e / W) / sm6 : 0.0;
                } else if constexpr (METRIC == GP_METRIC_MAE) {
                    const double e = yh - yv;
                    sd = wv * (e > 0.0 ? 1.0 : (e < 0.0 ? -1.0 : 0.0)) / W;
                    lacc += valid[j] ? wv * fabs(e) : 0.0;
                } else if constexpr (METRIC == GP_METRIC_LOGLOSS) {
                    const float z = t[j];
                    const float yf = d.y[row[j]];
                    const float t1 = fmaxf(z, 0.0f);
                    const float t2 = yf * z;
                    const float t3 = t1 - t2;
                    const float t5 = crm::log1p_exp_neg(fabsf(z), mt.lg, crm::log_k());
                    lacc += valid[j] ? wv * static_cast<double>(t3 + t5) : 0.0;
                    sd = wv * (1.0 / (1.0 + exp(-yh)) - yv) / W;
                } else {  // PEARSON: d|r|/dyhat
                    const double va = sm3, vb = sm4, rr = sm6;
                    if (va > 0.0 && vb > 0.0 && isfinite(va) && isfinite(vb)) {
                        const double dr = wv * ((yv - sm2) / sqrt(va * vb) - rr * (yh - sm1) / va);
                        sd = rr >= 0.0 ? dr : -dr;
                    } else {
                        sd = 0.0;
                    }
                }
                g[j] = valid[j] ? static_cast<float>(sd) * gsc : 0.0f;
            }

            if (nconst == 0) continue;   // no constant: nothing to carry back
            // ---------------- reverse pass ----------------
            GP_ARRAYS(as, kStackRegs + 1);   // adjoints of the entries below the top
            int ad = dp;                     // mirrors the value stack (dp == 0 here)
            // the walk visits the active instructions through their links (the
            // root, the last instruction, is active: the program holds a
            // constant); the next one is fetched while this one runs
            uint4 cur = pcode[CL - 1];
            for (;;) {
                const uint32_t link = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(cur.w)));
                const int qn = static_cast<int>(link & kNextMask) - 1;
                const uint4 nxt_ins = pcode[max(qn, 0)];
                const uint32_t w = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(cur.x)));
                const uint32_t cls = w & 3u;
                const uint32_t fn = (w >> 2) & 15u;
                // the chained unary functions first, the last one first
                const uint32_t chain = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(cur.z)));
                if (chain != 0u) {
                    const int nch = (32 - __clz(static_cast<int>(chain)) + 3) >> 2;
                    for (int kq = nch - 1; kq >= 0; --kq) {
                        const uint32_t u = ((chain >> (4 * kq)) & 15u) - 1u;
                        if (u == 0u) {
#pragma unroll
                            for (int j = 0; j < R; ++j) g[j] = -g[j];
                        } else {
                            --ntape;
                            float dv[R];
                            tape_get(ntape, dv);
#pragma unroll
                            for (int j = 0; j < R; ++j) g[j] = g[j] * dv[j];
                        }
                    }
                }
                const int ne = tape_entries(cls, fn);
                ntape -= ne;
                float gb[R];   // adjoint handed to the entry below the top (binary only)
#pragma unroll
                for (int j = 0; j < R; ++j) gb[j] = 0.0f;
                float gc[R];   // adjoint of the terminal (push / fold)
#pragma unroll
                for (int j = 0; j < R; ++j) gc[j] = 0.0f;
                if (cls == kUn) {
                    if (ne == 0) {
#pragma unroll
                        for (int j = 0; j < R; ++j) g[j] = -g[j];
                    } else {
                        float dv[R];
                        tape_get(ntape, dv);
#pragma unroll
                        for (int j = 0; j < R; ++j) g[j] = g[j] * dv[j];
                    }
                } else if (cls == kPush) {
#pragma unroll
                    for (int j = 0; j < R; ++j) gc[j] = g[j];
                } else {
                    // binary: operands (a, b); fold: a is the terminal, b the old top
                    float ga[R];
                    if (ne == 0) {
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            ga[j] = g[j];
                            gb[j] = fn == 0 ? g[j] : -g[j];
                        }
                    } else {
                        float da[R], db[R];
                        tape_get(ntape, da);
                        tape_get(ntape + 1, db);
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            ga[j] = g[j] * da[j];
                            gb[j] = g[j] * db[j];
                        }
                    }
                    if (cls == kBin) {
#pragma unroll
                        for (int j = 0; j < R; ++j) g[j] = ga[j];
                    } else {
#pragma unroll
                        for (int j = 0; j < R; ++j) {
                            gc[j] = ga[j];
                            g[j] = gb[j];
                        }
                    }
                }
                // adjoint stack: a binary hands gb to the (restored) entry below
                GP_PUT(as, min(ad + 1, kStackRegs), gb);
                if (cls == kBin) {
                    ++ad;
                    if (ad >= kStackRegs) {
#pragma unroll
                        for (int j = 0; j < R; ++j) aovf[((ad - kStackRegs) * R + j) * kWave + lane] = gb[j];
                    }
                }
                // a constant terminal: its adjoint summed over the wavefront's rows
                if (cls <= kFold && (w & kConstBit)) {
                    const int slot = static_cast<int>(w >> 8);
                    double sum = 0.0;
#pragma unroll
                    for (int j = 0; j < R; ++j) sum += valid[j] ? static_cast<double>(gc[j]) : 0.0;
                    const double tot = wave_sum(sum);
                    if (lane == 0) {
                        if (slot < kGradLds) gw[slot] += tot;
                        else atomicAdd(gextra + cbase + slot, tot);
                    }
                }
                // a push is undone, and so is each skipped subtree (one value on
                // the stack, carrying nothing back): the entry below becomes
                // the top again
                const int undo = (cls == kPush ? 1 : 0) + static_cast<int>(link >> kNextBits);
                if (undo > 0) {
                    ad -= undo;
                    const int top = ad + 1;
                    if (top >= 0) {
                        if (top < kStackRegs) {
                            GP_GET(as, top, g);
                        } else {
#pragma unroll
                            for (int j = 0; j < R; ++j) g[j] = aovf[((top - kStackRegs) * R + j) * kWave + lane];
                        }
                    }
                }
                if (qn < 0) break;
                cur = nxt_ins;
            }
        }
        // ---------------- per-item results ----------------
        wave_lds_sync();
        if (lane < nlds) gpart[(cbase + lane) * s.n_chunks + c] = gw[lane];
        if (part) {
            lacc = wave_sum(lacc);
            if (lane == 0) part[static_cast<int64_t>(p) * s.n_chunks + c] = lacc;
        }
        wave_lds_sync();
    }
}

// ---------------------------------------------------------------------------
// k_adjoint: the same derivative for programs of at most kParNodes nodes, the
// program in the interpreter of gp_eval_asm.h.  Its forward part records each
// active operation's partial derivatives on a tape: kTapeRegs entries in
// vector registers, kTapeLds in LDS, the rest in memory (a program of 200
// nodes over 8 features records 22 on average, 54 at most); its reverse part
// is straight-line instructions over the active operations alone.  Two
// wavefronts per SIMD at four rows per lane, the registers' worth, which is too
// few to hide every wait: the vector pipes are busy 73% of the time and a
// wavefront waits a third of its cycles (the evaluation kernel, with four, 97%
// busy).  1,024 programs of 1 to 200 nodes on 262,144 rows
// of 8 features: 23.9 ms by k_adjoint_long, 8.3 ms here (two rows per lane and
// three wavefronts 9.3 ms, one row and four 12.3 ms; one tile per item to 64
// within 7%); 100 programs of up to 120 nodes on 10,007 weighted rows,
// forward pass, derivative and their preparation: 410 and 277 us.
// ---------------------------------------------------------------------------
template <int R>
constexpr size_t adjoint_lds_wave() { return static_cast<size_t>(kTapeLds) * R * kWave * 4 + kGradLds * sizeof(double); }
// bytes of a wavefront's memory area for at most `entries` tape entries
template <int R>
int64_t adjoint_area(int64_t entries) {
    return std::max<int64_t>(entries - kTapeRegs - kTapeLds, 1) * R * kWave * 4;
}

// The caller's part of the adjoint's instructions (as leave_rows): the
// operation on t (and m), its partials to u (and m).
template <int R, typename V>
__device__ __forceinline__ void leave_rows_adjoint(uint32_t code, V& t, V& m, V& u, const unsigned char* lds) {
    const MathTabsLds& tabs = *reinterpret_cast<const MathTabsLds*>(lds);
    const MathTabs mt{tabs.sc, tabs.lg};
    auto unary = [&](uint32_t fn) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            float x[1] = {ev_get(t, j)}, y[1] = {x[0]}, dv[1];
            if (fn == 3 || fn == 4) {
                sincos_rows_derivative<1>(fn == 4, y, dv, mt);
            } else {
                apply_unary<1>(fn, y, mt);
                unary_derivative<1>(fn, x, y, dv);
            }
            ev_set(t, j, y[0]);
            ev_set(u, j, dv[0]);
            asm volatile("" : "+v"(t), "+v"(u));
        }
    };
    auto binary = [&](uint32_t fn, bool t_first) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float tj = ev_get(t, j), mj = ev_get(m, j);
            float a[1] = {t_first ? tj : mj}, b[1] = {t_first ? mj : tj};
            float da, db;
            if (fn < 6) {
                // the selected operand (the first on ties) carries it
                const bool first = (fn == 4 ? a[0] >= b[0] : a[0] <= b[0]) || isnan(b[0]);
                da = first ? 1.0f : 0.0f;
                db = first ? 0.0f : 1.0f;
            } else {
                const float r2 = a[0] * a[0] + b[0] * b[0];
                da = r2 > 0.0f ? b[0] / r2 : 0.0f;
                db = r2 > 0.0f ? -a[0] / r2 : 0.0f;
            }
            apply_binary_wide<1>(fn, a, b);
            ev_set(t, j, a[0]);
            ev_set(u, j, t_first ? da : db);
            ev_set(m, j, t_first ? db : da);
            asm volatile("" : "+v"(t), "+v"(m), "+v"(u));
        }
    };
    switch (code) {
    case kExitAdjUnary + 3: unary(3); break;
    case kExitAdjUnary + 4: unary(4); break;
    case kExitAdjUnary + 5: unary(5); break;
    case kExitAdjUnary + 6: unary(6); break;
    case kExitAdjUnary + 7: unary(7); break;
    case kExitAdjUnary + 8: unary(8); break;
    case kExitAdjUnary + 9: unary(9); break;
    case kExitAdjUnary + 10: unary(10); break;
    case kExitAdjUnary + 11: unary(11); break;
    case kExitAdjUnary + 12: unary(12); break;
    case kExitAdjUnary + 13: unary(13); break;
    case kExitAdjBinary: binary(4, true); break;
    case kExitAdjBinary + 1: binary(4, false); break;
    case kExitAdjBinary + 2: binary(5, true); break;
    case kExitAdjBinary + 3: binary(5, false); break;
    case kExitAdjBinary + 4: binary(6, true); break;
    default: binary(6, false); break;
    }
}

constexpr int adjoint_waves(int R) { return R == 4 ? 2 : R == 2 ? 3 : 4; }

template <int R, int METRIC>
__global__ __launch_bounds__(kAdjWaves * kWave, adjoint_waves(R)) void k_adjoint(
    PopView pop, CodeView cv, DataView d, Sched s, const double* __restrict__ stats, const double* __restrict__ wsum,
    const float* __restrict__ gscale, double* __restrict__ part, double* __restrict__ gpart,
    double* __restrict__ gextra, unsigned char* __restrict__ area, int64_t area_bytes) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wid = uniform(threadIdx.x >> 6);
    const int64_t N = d.N;
    const int64_t ld = d.ld;
    const float* __restrict__ X = d.X;
    extern __shared__ __align__(16) unsigned char lds_all[];
    // k_adjoint_long's programs, first in the order (read while the tables are)
    const uint32_t n_long = ldu(s.counter + kLongWord);
    stage_tabs(*reinterpret_cast<MathTabsLds*>(lds_all));
    // per wavefront: the sums of constants from kAccRegs on, then the LDS tape
    unsigned char* lds_wave = lds_all + sizeof(MathTabsLds) + wid * adjoint_lds_wave<R>();
    double* gw = reinterpret_cast<double*>(lds_wave);
    InterpAdjoint<R> in;
    in.c0 = interp_c0();
    in.c1 = interp_c1();
    interp_vector_constants(in);
    in.lds = static_cast<uint32_t>(sizeof(MathTabsLds) + wid * adjoint_lds_wave<R>() + kGradLds * sizeof(double));
    in.ld4 = static_cast<uint64_t>(ld) * 4u;
    in.area = reinterpret_cast<uint64_t>(area + (static_cast<int64_t>(blockIdx.x) * kAdjWaves + wid) * area_bytes);
    const double W = *wsum;
    const int32_t* __restrict__ order = s.order + n_long;
    Claims claims(s, static_cast<uint32_t>(pop.P) - n_long, wid);
    int qx;
    uint32_t it, it_end;
    while (claims.next(lane, &qx, &it, &it_end)) {
        it = uniform(it);
        qx = static_cast<int>(uniform(static_cast<uint32_t>(qx)));
        const uint32_t cq = it / claims.per, place = claims.program(it - cq * claims.per, qx);
        if (place >= claims.P) continue;
        const int32_t c = claims.chunk(cq, qx);
        const int32_t p = ldu(order + place);
        const int64_t off = ldu(pop.prog_off + p);
        const uint32_t head = static_cast<uint32_t>(ldu(cv.clen + p));
        const int64_t cbase = ldu(pop.const_off + p);
        const int32_t nconst = static_cast<int32_t>(ldu(pop.const_off + p + 1) - cbase);
        const uint4* __restrict__ pcode = cv.code + off * kAdjCodePerNode;
        in.ins = reinterpret_cast<const EvVec<uint32_t, 2>*>(pcode)[lane];
        const int64_t r0 = static_cast<int64_t>(c) * s.chunk;
        const int64_t r1 = min(r0 + s.chunk, N);
        const float gsc = gscale ? ldu(gscale + p) : 1.0f;
        if (lane < kGradLds) gw[lane] = 0.0;
        wave_lds_sync();
        in.acc = EvVec<float, 2 * kAccRegs>{};
        double lacc = 0.0;
        bool first_tile = true;
        // a program without constants needs only its loss, and only when asked
        const int64_t r_end = (nconst == 0 && !part) ? r0 : r1;
        for (int64_t base = r0; base < r_end; base += kWave * R) {
            const int left = static_cast<int>(min<int64_t>(r1 - base, kWave * R));
            auto row_off = [left](int ln, int j) {
                return static_cast<uint32_t>(min(j * kWave + ln, left - 1)) * 4u;
            };
            auto at = [](const float* col, uint32_t o) {
                return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(col) + o);
            };
            in.xb = reinterpret_cast<uint64_t>(X + base);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                ev_set(in.off, j, row_off(lane, j));
                in.mask[j] = __ballot(j * kWave + lane < left);
            }
            if (head & kHdrFetch) {
                const float* __restrict__ col = X + static_cast<int64_t>(head & kHdrFeature) * ld + base;
#pragma unroll
                for (int j = 0; j < R; ++j) ev_set(in.p, j, at(col, row_off(lane, j)));
            }
            const uint64_t blk = reinterpret_cast<uint64_t>(pcode);
            in.blk0 = static_cast<uint32_t>(blk);
            in.blk1 = static_cast<uint32_t>(blk >> 32);
            if ((head & kHdrBlocks) && !first_tile) in.ins = reinterpret_cast<const EvVec<uint32_t, 2>*>(pcode)[lane];
            first_tile = false;
            in.idx = 0;
            // the forward part, then (with constants) the reverse part: one walk
            // of the caller's instructions serves both
            for (int phase = 0;; ++phase) {
                uint32_t code;
                while ((code = in.run()) != kExitEnd) {
                    if (code == kExitCAdd) {
                        // a constant beyond the register sums
                        double sum = 0.0;
#pragma unroll
                        for (int j = 0; j < R; ++j)
                            sum += j * kWave + lane < left ? static_cast<double>(ev_get(in.m, j)) : 0.0;
                        const double tot = wave_sum(sum);
                        const int slot = static_cast<int>(in.payload);
                        if (lane == 0) {
                            if (slot < kGradLds) gw[slot] += tot;
                            else atomicAdd(gextra + cbase + slot, tot);
                        }
                        continue;
                    }
                    if (code < kExitAdjUnary) leave_rows<R>(code, in.t, in.m, lds_all);
                    else leave_rows_adjoint<R>(code, in.t, in.m, in.u, lds_all);
                }
                if (phase == 1) break;
                // ---------------- seeds: d fitness / d yhat per row ----------------
                int ln = lane;
                asm volatile("" : "+v"(ln));
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const bool valid = j * kWave + ln < left;
                    const float tj = ev_get(in.t, j);
                    const float yf = at(d.y + base, row_off(ln, j));
                    const double yh = static_cast<double>(tj);
                    const double yv = static_cast<double>(yf);
                    const double wv = d.w ? static_cast<double>(at(d.w + base, row_off(ln, j))) : 1.0;
                    double sd;
                    if constexpr (METRIC == GP_METRIC_MSE) {
                        const double e = yh - yv;
                        sd = 2.0 * wv * e / W;
                        lacc += valid ? wv * (e * e) : 0.0;
                    } else if constexpr (METRIC == GP_METRIC_RMSE) {
                        const double sm6 = stats[static_cast<int64_t>(p) * kStats + 6];
                        const double e = yh - yv;
                        sd = sm6 > 0.0 ? (wv * e / W) / sm6 : 0.0;
                    } else if constexpr (METRIC == GP_METRIC_MAE) {
                        const double e = yh - yv;
                        sd = wv * (e > 0.0 ? 1.0 : (e < 0.0 ? -1.0 : 0.0)) / W;
                        lacc += valid ? wv * fabs(e) : 0.0;
                    } else if constexpr (METRIC == GP_METRIC_LOGLOSS) {
                        const float t1 = fmaxf(tj, 0.0f);
                        const float t2 = yf * tj;
                        const float t3 = t1 - t2;
                        const float t5 = crm::log1p_exp_neg(fabsf(tj), reinterpret_cast<const MathTabsLds*>(lds_all)->lg, crm::log_k());
                        lacc += valid ? wv * static_cast<double>(t3 + t5) : 0.0;
                        asm volatile("" : "+v"(lacc));
                        sd = wv * (1.0 / (1.0 + exp(-yh)) - yv) / W;
                    } else {  // PEARSON: d|r|/dyhat
                        const double* sp = stats + static_cast<int64_t>(p) * kStats;
                        const double va = sp[3], vb = sp[4], rr = sp[6];
                        if (va > 0.0 && vb > 0.0 && isfinite(va) && isfinite(vb)) {
                            const double dr = wv * ((yv - sp[2]) / sqrt(va * vb) - rr * (yh - sp[1]) / va);
                            sd = rr >= 0.0 ? dr : -dr;
                        } else {
                            sd = 0.0;
                        }
                    }
                    ev_set(in.t, j, valid ? static_cast<float>(sd) * gsc : 0.0f);
                    asm volatile("" : "+v"(in.t));     // (one row after the other)
                }
                if (nconst == 0) break;   // nothing to carry back
            }
        }
        // ---------------- per-item results ----------------
        const int nlds = min(nconst, kGradLds);
#pragma unroll
        for (int q = 0; q < kAccRegs; ++q)
            if (q < nlds) {
                const uint64_t u = static_cast<uint64_t>(__float_as_uint(in.acc[2 * q])) |
                                   static_cast<uint64_t>(__float_as_uint(in.acc[2 * q + 1])) << 32;
                const double tot = wave_sum(__longlong_as_double(static_cast<long long>(u)));
                if (lane == 0) gw[q] = tot;
            }
        wave_lds_sync();
        if (lane < nlds) gpart[(cbase + lane) * s.n_chunks + c] = gw[lane];
        if (part) {
            lacc = wave_sum(lacc);
            if (lane == 0) part[static_cast<int64_t>(p) * s.n_chunks + c] = lacc;
        }
        wave_lds_sync();
    }
}

// grad[i] = sum over chunks of gpart[i * n_chunks + c] (fixed order) plus
// gextra[i]; one lane per constant.
__global__ __launch_bounds__(kBlock) void k_finalize_grad(const double* __restrict__ gpart,
                                                           const double* __restrict__ gextra,
                                                           const int64_t* __restrict__ const_off,
                                                           int32_t P, int32_t n_chunks,
                                                           float* __restrict__ grad) {
    const int32_t p = static_cast<int32_t>(blockIdx.x) * (kBlock / kWave) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & (kWave - 1);
    if (p >= P) return;
    const int64_t c0 = const_off[p], c1 = const_off[p + 1];
    for (int64_t i = c0 + lane; i < c1; i += kWave) {
        double sum = gextra[i];
        if (i - c0 < kGradLds)
            for (int c = 0; c < n_chunks; ++c) sum += gpart[i * n_chunks + c];
        grad[i] = static_cast<float>(sum);
    }
}

// sum of weights over all rows (float64), from the per-chunk statistics
__global__ __launch_bounds__(kWave) void k_wsum(const double* __restrict__ ystat, int32_t n_chunks,
                                                 int has_w, int64_t N, double* __restrict__ out) {
    double s = 0.0;
    if (has_w)
        for (int c = threadIdx.x; c < n_chunks; c += kWave) s += ystat[static_cast<int64_t>(c) * 4];
    s = wave_sum(s);
    if (threadIdx.x == 0) *out = has_w ? s : static_cast<double>(N);
}

// ---------------------------------------------------------------------------
// k_tournament (Sec. III-C1): 2^lg lanes per tournament, each taking every
// 2^lg-th block of four draws; shuffles then give the tournament's lanes its
// winner: the first drawn of the programs with the best value, where a NaN
// loses to any other value.  A draw is a random read of two words, so the
// kernel is a chain of memory latencies: with one lane per tournament five of
// them, and half a wavefront per CU (8,192 tournaments of 20 among 4,096
// programs, back to back: 8.5 us with one lane each, 4.1 with eight).
// ---------------------------------------------------------------------------
constexpr int64_t kTourLanes = 131072;

__global__ __launch_bounds__(kBlock) void k_tournament(const float* __restrict__ fit,
                                                        const int32_t* __restrict__ len,
                                                        int32_t P, int larger, float c, int32_t k,
                                                        int32_t T, int lg, uint64_t seed, uint32_t gen_value,
                                                        const uint32_t* __restrict__ gen_dev,
                                                        int32_t* __restrict__ winners) {
    const uint32_t lanes = 1u << lg;
    const uint32_t sub = threadIdx.x & (lanes - 1u);
    const int64_t t = static_cast<int64_t>(blockIdx.x) * (kBlock >> lg) + (threadIdx.x >> lg);
    // a captured generation graph reads the generation number from memory
    const uint32_t gen = gen_dev ? *gen_dev : gen_value;
    int32_t best = -1;
    uint32_t best_d = 0;      // its draw
    float best_adj = 0.0f;
    auto beats = [&](float adj, uint32_t d) {
        if (best < 0) return true;
        if (isnan(adj)) return isnan(best_adj) && d < best_d;
        if (isnan(best_adj)) return true;
        if (adj == best_adj) return d < best_d;
        return larger ? adj > best_adj : adj < best_adj;
    };
    const uint32_t draws = static_cast<uint32_t>(k), blocks = (draws - 1u) / 4u + 1u;
    if (t < T) {
        for (uint32_t q = sub; q < blocks; q += lanes) {
            const Philox4 blk = philox4x32_10(q, static_cast<uint32_t>(t), gen, kStreamTournament, seed);
            int32_t idx[4], ln[4];
            float raw[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) idx[e] = static_cast<int32_t>(below(blk.v[e], static_cast<uint32_t>(P)));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ln[e] = len[idx[e]];
                raw[e] = fit[idx[e]];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t d = q * 4u + static_cast<uint32_t>(e);
                const float pen = __fmul_rn(c, static_cast<float>(ln[e]));
                const float adj = larger ? __fsub_rn(raw[e], pen) : __fadd_rn(raw[e], pen);
                if (d < draws && beats(adj, d)) {
                    best = idx[e];
                    best_d = d;
                    best_adj = adj;
                }
            }
        }
    }
    for (uint32_t m = 1; m < lanes; m <<= 1) {
        const int32_t ob = __shfl_xor(best, static_cast<int>(m), kWave);
        const uint32_t od = __shfl_xor(best_d, static_cast<int>(m), kWave);
        const float oa = __shfl_xor(best_adj, static_cast<int>(m), kWave);
        if (ob >= 0 && beats(oa, od)) {
            best = ob;
            best_d = od;
            best_adj = oa;
        }
    }
    if (t < T && sub == 0) winners[t] = best;
}

// ---------------------------------------------------------------------------
// Spearman (Sec. III-C3 ranks each program's outputs with a sort): the outputs
// of a batch of programs become order-preserving 32-bit keys in the first
// pass of a segmented LSD radix sort (four passes of 8 bits: per-tile digit
// counts, a per-segment scan, a stable scatter), each carrying its row's
// target rank (or its row, with weights) through the sort, and one workgroup
// per program walks its sorted keys, giving tied values the mean of their
// ranks, and forms the float64 moments of the (value rank, target rank)
// pairs.
// ---------------------------------------------------------------------------
constexpr int kRsBlock = 256;                  // threads of the count kernel
constexpr int kRsScatterBlock = 512;           // threads of the scatter
constexpr int kRsItems = 16;                   // keys per scatter thread
constexpr int kRsTile = kRsScatterBlock * kRsItems;   // keys per tile
constexpr int kRsRadix = 256;

// float -> uint32 with the same order; -0 and +0 map to one key
__device__ __forceinline__ uint32_t order_key(float v) {
    uint32_t b = __float_as_uint(v == 0.0f ? 0.0f : v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// counts[(seg * 256 + digit) * T + tile] for one pass.  The first pass reads
// the float values themselves (their order-preserving keys are formed here)
// and raises nan[seg] for a NaN.  Eight keys per thread are in flight at a
// time, and eight copies of the counters, a bank apart, keep lanes with one
// digit (an exponent's, in the last pass) out of each other's way: 33.6M keys, the
// first to the last pass, 38, 52, 54 and 81 us with one copy and one key in
// flight, 27, 38, 38 and 39 so (134 MB read: 3.5 TB/s and more).
constexpr int kRsCopies = 8;

template <bool FIRST>
__global__ __launch_bounds__(kRsBlock) void k_rs_count(const uint32_t* __restrict__ keys, int64_t N, int32_t T,
                                                        int shift, uint32_t* __restrict__ counts,
                                                        int32_t* __restrict__ nan_flag) {
    constexpr int kE = 8;
    __shared__ uint32_t hist[kRsCopies][kRsRadix + 1];
    const int32_t tile = blockIdx.x, seg = blockIdx.y;
    uint32_t* mine = hist[threadIdx.x % kRsCopies];
#pragma unroll
    for (int q = 0; q < kRsCopies; ++q) hist[q][threadIdx.x] = 0;
    __syncthreads();
    const uint32_t* __restrict__ in = keys + static_cast<int64_t>(seg) * N + static_cast<int64_t>(tile) * kRsTile;
    const int len = static_cast<int>(min<int64_t>(kRsTile, N - static_cast<int64_t>(tile) * kRsTile));
    bool nan = false;
    for (int k = 0; k < kRsTile / kRsBlock; k += kE) {
        uint32_t key[kE];
#pragma unroll
        for (int e = 0; e < kE; ++e) key[e] = in[min((k + e) * kRsBlock + static_cast<int>(threadIdx.x), len - 1)];
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            if constexpr (FIRST) {
                const float v = __uint_as_float(key[e]);
                nan |= isnan(v);
                key[e] = order_key(v);
            }
            if ((k + e) * kRsBlock + static_cast<int>(threadIdx.x) < len) atomicAdd(&mine[(key[e] >> shift) & 255u], 1u);
        }
    }
    if (FIRST && nan) nan_flag[seg] = 1;
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kRsCopies; ++q) sum += hist[q][threadIdx.x];
    counts[(static_cast<int64_t>(seg) * kRsRadix + threadIdx.x) * T + tile] = sum;
}

// exclusive scan of one segment's 256*T counts, digit-major (in place), in
// chunks of 1,024 consecutive counts (coalesced; four chunks' loads issued
// together): shuffle scans within each wavefront, the wavefronts' totals
// through LDS (double-buffered, so one barrier per chunk), then the carry of
// the earlier chunks.
__global__ __launch_bounds__(1024) void k_rs_scan(uint32_t* __restrict__ counts, int32_t T) {
    constexpr int kW = 1024 / kWave, kE = 4;
    __shared__ uint32_t wtot[2][kW];
    const int64_t n = static_cast<int64_t>(kRsRadix) * T;
    uint32_t* c = counts + static_cast<int64_t>(blockIdx.x) * n;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid >> 6;
    uint32_t carry = 0;
    int par = 0;
    for (int64_t c0 = 0; c0 < n; c0 += 1024 * kE) {
        uint32_t v[kE];
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const int64_t i = c0 + e * 1024 + tid;
            v[e] = i < n ? c[i] : 0u;
        }
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            uint32_t x = v[e];
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t o = __shfl_up(x, d, kWave);
                if (lane >= d) x += o;
            }
            if (lane == kWave - 1) wtot[par][wid] = x;
            __syncthreads();
            uint32_t pre = carry, all = carry;
            for (int q = 0; q < kW; ++q) {
                const uint32_t t = wtot[par][q];
                pre += q < wid ? t : 0u;
                all += t;
            }
            const int64_t i = c0 + e * 1024 + tid;
            if (i < n) c[i] = pre + x - v[e];
            carry = all;
            par ^= 1;
        }
    }
}

// stable scatter of one tile, staged through LDS.  Wavefront w takes the
// tile's keys w*1024 ... w*1024+1023 in index order, 64 a round; within a
// round, lanes holding the same digit find each other by ballots over the
// digit's bits, and the wavefront's running count of that digit (its own row
// of LDS counters, updated by the lowest such lane; a wavefront's LDS
// operations are ordered, so no barrier is needed) gives each key its rank
// among the wavefront's keys of that digit.  One barrier later, each digit's
// counts are turned into exclusive prefixes over the wavefronts, which puts
// every key at its digit-sorted position within the tile in LDS.  The tile
// then goes out run by run: consecutive threads write consecutive addresses
// of each digit's output range.  The tile's count of digit d is the
// difference of adjacent scanned offsets (digit-major over tiles, the last
// one closed by N).  The first pass reads the float values, forms their
// keys, and gives each the value it carries through the sort: its row's
// target rank where rank2_y is given (then the sorted values are the target
// ranks in the program's order), else its row.
template <bool FIRST>
__global__ __launch_bounds__(kRsScatterBlock) void k_rs_scatter(const uint32_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ vin,
                                                          uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                          int64_t N, int32_t T, int shift,
                                                          const uint32_t* __restrict__ offsets,
                                                          const uint32_t* __restrict__ rank2_y) {
    constexpr int kWaves = kRsScatterBlock / kWave;
    constexpr int kDigitWaves = kRsRadix / kWave;     // the wavefronts that keep one digit per thread
    constexpr int kPerWave = kRsTile / kWaves;        // keys per wavefront (kRsItems rounds of 64)
    __shared__ uint32_t base_off[kRsRadix];           // global start of each digit for this tile
    __shared__ uint32_t loc_off[kRsRadix];            // local start of each digit within the tile
    __shared__ uint32_t hist[kWaves][kRsRadix];       // per-wavefront digit counts, then their prefixes
    __shared__ uint32_t wsum[kDigitWaves];
    __shared__ uint32_t skey[kRsTile], sval[kRsTile];
    const int32_t tile = blockIdx.x, seg = blockIdx.y;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid >> 6;
    // threads below kRsRadix keep digit tid's offsets
    const bool digit_thread = tid < kRsRadix;
    uint32_t start = 0, cnt = 0;
    if (digit_thread) {
        const int64_t cidx = (static_cast<int64_t>(seg) * kRsRadix + tid) * T + tile;
        const int64_t nidx = static_cast<int64_t>(kRsRadix) * T;     // offsets per segment
        start = offsets[cidx];
        const int64_t cnext = (static_cast<int64_t>(tid) * T + tile + 1 < nidx) ? cidx + 1 : -1;
        cnt = (cnext >= 0 ? offsets[cnext] : static_cast<uint32_t>(N)) - start;
    }
    const int64_t sbase = static_cast<int64_t>(seg) * N;
    const int64_t t0 = static_cast<int64_t>(tile) * kRsTile;
    const int tile_len = static_cast<int>(min<int64_t>(kRsTile, N - t0));
    // this wavefront's keys, all loads issued before the ranking
    uint32_t pkey[kRsItems], pval[kRsItems];
#pragma unroll
    for (int k = 0; k < kRsItems; ++k) {
        const int64_t i = t0 + wave * kPerWave + k * kWave + lane;
        if constexpr (FIRST) {
            pkey[k] = i < N ? order_key(__uint_as_float(kin[sbase + i])) : 0u;
            pval[k] = i < N ? (rank2_y ? rank2_y[i] : static_cast<uint32_t>(i)) : 0u;
        } else {
            pkey[k] = i < N ? kin[sbase + i] : 0u;
            pval[k] = i < N ? vin[sbase + i] : 0u;
        }
    }
    if (digit_thread) {
        base_off[tid] = start;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) hist[w][tid] = 0;
    }
    // exclusive scan of the tile's digit counts (shuffles within each wave,
    // then the waves' totals)
    uint32_t v = cnt;
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(v, d, kWave);
        if (lane >= d) v += o;
    }
    if (digit_thread && lane == kWave - 1) wsum[wave] = v;
    __syncthreads();
    if (digit_thread) {
        uint32_t pre = 0;
        for (int q = 0; q < wave; ++q) pre += wsum[q];
        loc_off[tid] = pre + v - cnt;
    }
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t prank[kRsItems];
#pragma unroll
    for (int k = 0; k < kRsItems; ++k) {
        const int64_t i = t0 + wave * kPerWave + k * kWave + lane;
        const bool valid = i < N;
        const uint32_t d = (pkey[k] >> shift) & 255u;
        // lanes of this wave holding a valid key with the same digit
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t bal = __ballot((d >> bit) & 1u);
            peers &= ((d >> bit) & 1u) ? bal : ~bal;
        }
        const uint32_t rank_w = static_cast<uint32_t>(__popcll(peers & lt_mask));
        const uint32_t before = hist[wave][d];
        prank[k] = before + rank_w;
        if (valid && rank_w == 0) hist[wave][d] = before + static_cast<uint32_t>(__popcll(peers));
    }
    __syncthreads();
    if (digit_thread) {   // exclusive prefix over the wavefronts of digit tid's counts
        uint32_t acc = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = hist[w][tid];
            hist[w][tid] = acc;
            acc += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRsItems; ++k) {
        const int64_t i = t0 + wave * kPerWave + k * kWave + lane;
        if (i < N) {
            const uint32_t d = (pkey[k] >> shift) & 255u;
            const uint32_t lp = loc_off[d] + hist[wave][d] + prank[k];
            if (lp < static_cast<uint32_t>(kRsTile)) {
                skey[lp] = pkey[k];
                sval[lp] = pval[k];
            }
        }
    }
    __syncthreads();
    // the tile, digit-sorted, to its digits' output ranges
    for (int j = tid; j < tile_len; j += kRsScatterBlock) {
        const uint32_t key = skey[j];
        const uint32_t d = (key >> shift) & 255u;
        const uint32_t pos = base_off[d] + (static_cast<uint32_t>(j) - loc_off[d]);
        if (pos < static_cast<uint64_t>(N)) {
            kout[sbase + pos] = key;
            vout[sbase + pos] = sval[j];
        }
    }
}

// First position in [lo, hi) of the sorted keys whose key is at least x (above:
// above x), hi if there is none; by a whole wavefront, 64 probes at a time.
__device__ __forceinline__ uint32_t run_bound(const uint32_t* __restrict__ k, uint32_t lo, uint32_t hi, uint32_t x,
                                              bool above) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    while (lo < hi) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint64_t at = static_cast<uint64_t>(lo) + static_cast<uint64_t>(lane) * step;
        bool past = true;
        if (at < hi) {
            const uint32_t key = k[at];
            past = above ? key > x : key >= x;
        }
        // the first lane past it: the answer lies after the probe before
        const uint64_t m = __ballot(past);
        const uint32_t f = m ? static_cast<uint32_t>(__builtin_ctzll(m)) : kWave;
        const uint64_t end = static_cast<uint64_t>(lo) + static_cast<uint64_t>(f) * step;
        hi = end < hi ? static_cast<uint32_t>(end) : hi;
        if (step == 1) return hi;
        if (f > 0) lo += (f - 1) * step + 1;
    }
    return hi;
}

// Where a lane's tied run lies, from the ballot S of the run starts among 64
// consecutive positions: the lane of its start (the highest at or below) and
// of the next one.
__device__ __forceinline__ int run_first(uint64_t S, int lane) {
    return 63 - __builtin_clzll(S & (~0ull >> (63 - lane)));
}
__device__ __forceinline__ int run_next(uint64_t S, int lane) { return __builtin_ctzll(S & ~(~0ull >> (63 - lane))); }

// The target's ranks, from its sorted keys: rank2[row] is twice the mean rank
// of the tied run holding the row, an integer.  A wavefront takes 64
// consecutive positions at a time: the runs that lie within them come from one
// ballot, and the first's start and the last's end, where the neighbouring
// keys are equal, from a search of the sorted keys.  Each block leaves its
// weighted sums (w, w b, w b^2) of the centred ranks b = rank - (N+1)/2, which
// every program's correlation shares.  One block that scanned all keys took
// 160 us for 65,536 rows, 4.8 here.
constexpr int kTargetBlocks = 512;

__global__ __launch_bounds__(kBlock) void k_spear_rank_target(const uint32_t* __restrict__ keys,
                                                               const uint32_t* __restrict__ idx, int64_t N,
                                                               const float* __restrict__ w,
                                                               uint32_t* __restrict__ rank2_out,
                                                               double* __restrict__ tsum) {
    constexpr int kW = kBlock / kWave;
    __shared__ double red[3][kW];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = static_cast<int>(uniform(threadIdx.x >> 6));
    const uint32_t n = static_cast<uint32_t>(N);      // below 2^31
    const double mid = 0.5 * (static_cast<double>(N) + 1.0);
    double v[3] = {0.0, 0.0, 0.0};
    for (uint32_t c = (blockIdx.x * kW + wid) * kWave; c < n; c += gridDim.x * (kW * kWave)) {
        const uint32_t i = c + lane, m = min(n - c, static_cast<uint32_t>(kWave));
        const bool in = i < n;
        const uint32_t key = in ? keys[i] : 0u;
        const uint32_t row = in ? idx[i] : 0u;
        uint32_t prev = __shfl_up(key, 1, kWave);
        if (lane == 0) prev = i > 0 ? keys[i - 1] : ~key;
        const uint64_t S = __ballot(in && key != prev);
        uint32_t start = c, end = c + m;       // of the run before the first start, and of the last run
        const uint32_t k0 = uniform(key), kl = static_cast<uint32_t>(__builtin_amdgcn_readlane(key, m - 1));
        if (!(S & 1ull)) start = run_bound(keys, 0, c, k0, false);
        if (c + m < n && keys[c + m] == kl) end = run_bound(keys, c + m, n, kl, true);
        if (S) {
            const int first = __builtin_ctzll(S), last = 63 - __builtin_clzll(S);
            if (lane >= first) start = c + run_first(S, lane);
            if (lane < last) end = c + run_next(S, lane);
        }
        if (in) {
            const uint32_t r2 = start + 1u + end;
            rank2_out[row] = r2;
            const double wv = w ? static_cast<double>(w[row]) : 1.0;
            const double b = 0.5 * static_cast<double>(r2) - mid;
            v[0] += wv;
            v[1] += wv * b;
            v[2] += wv * b * b;
        }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double t = wave_sum(v[q]);
        if (lane == 0) red[q][wid] = t;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double acc = 0.0;
        for (int j = 0; j < kW; ++j) acc += red[threadIdx.x][j];
        tsum[threadIdx.x * kTargetBlocks + blockIdx.x] = acc;
    }
}

// Rank correlation of a batch of programs, one workgroup per program and one
// pass over its sorted keys, each wavefront a range of its own.  The tied run
// holding position i spans [start, end) and twice its mean rank is start + 1 +
// end.  Of 64 consecutive positions a ballot marks the run starts; the run
// still open at their end is carried on: each lane sums its rows' weights and
// weighted target ranks for it, and folds those sums in with the run's mean
// rank where it ends.  A range's first start and last end, where a run crosses
// its edge, come from a search of the sorted keys, so the wavefronts never
// wait for each other (scans over a workgroup's 1,024 positions, a barrier
// each: 204 us for 512 programs on 65,536 rows, 96 here).  With a = rank -
// (N+1)/2 for the program and b likewise for the target, the weighted sums of
// a, a^2 and a b and the target's sums (tsum, by its blocks) give |r|: 0 for a
// constant rank vector, NaN if the outputs or the target held a NaN.
// Unweighted, the sorted values are the target ranks themselves; weighted,
// they are rows, whose target ranks and weights are gathered.
template <bool WEIGHTED>
__global__ __launch_bounds__(1024) void k_spear_corr(const uint32_t* __restrict__ keys,
                                                      const uint32_t* __restrict__ vals, int64_t N,
                                                      const uint32_t* __restrict__ rank2_y,
                                                      const float* __restrict__ w,
                                                      const double* __restrict__ tsum, int32_t target_blocks,
                                                      const int32_t* __restrict__ nan_flag,
                                                      const int32_t* __restrict__ target_nan,
                                                      float* __restrict__ fitness, int32_t prog0) {
    constexpr int kW = 1024 / kWave, kE = 4;
    __shared__ double red[3][kW];
    const int32_t seg = blockIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = static_cast<int>(uniform(threadIdx.x >> 6));
    const uint32_t n = static_cast<uint32_t>(N);      // below 2^31
    const uint32_t* __restrict__ k = keys + static_cast<int64_t>(seg) * N;
    const uint32_t* __restrict__ ix = vals + static_cast<int64_t>(seg) * N;
    const double mid = 0.5 * (static_cast<double>(N) + 1.0);
    double s_a = 0.0, s_aa = 0.0, s_ab = 0.0;
    double o_w = 0.0, o_wb = 0.0;     // this lane's rows of the open run
    auto fold = [&](uint32_t start, uint32_t end) {
        const double a = 0.5 * (static_cast<double>(start) + 1.0 + static_cast<double>(end)) - mid;
        s_a += a * o_w;
        s_aa += a * a * o_w;
        s_ab += a * o_wb;
    };
    // this wavefront's range, whole groups of 64
    const uint32_t groups = (n + kWave - 1) / kWave, per = (groups + kW - 1) / kW * kWave;
    const uint32_t r0 = min(static_cast<uint32_t>(wid) * per, n), r1 = min(r0 + per, n);
    if (r0 < r1) {
        uint32_t last_key = r0 > 0 ? k[r0 - 1] : 0u;      // the key before the group
        uint32_t open = r0;                               // start of the open run
        if (r0 > 0 && k[r0] == last_key) open = run_bound(k, 0, r0, last_key, false);
        for (uint32_t c0 = r0; c0 < r1; c0 += kWave * kE) {
            uint32_t key[kE], ry[kE];
            float wf[kE];
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                const uint32_t i = min(c0 + e * kWave + lane, n - 1);
                key[e] = k[i];
                ry[e] = ix[i];
            }
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                wf[e] = 1.0f;
                if constexpr (WEIGHTED) {
                    wf[e] = w[ry[e]];
                    ry[e] = rank2_y[ry[e]];
                }
            }
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                const uint32_t c = c0 + e * kWave, i = c + lane;
                if (c >= r1) break;
                const bool in = i < r1;
                uint32_t prev = __shfl_up(key[e], 1, kWave);
                if (lane == 0) prev = i > 0 ? last_key : ~key[e];
                const uint64_t S = __ballot(in && key[e] != prev);
                last_key = static_cast<uint32_t>(__builtin_amdgcn_readlane(key[e], kWave - 1));
                const double wv = in ? static_cast<double>(wf[e]) : 0.0;
                const double wb = wv * (0.5 * static_cast<double>(ry[e]) - mid);
                if (S == 0ull) {
                    o_w += wv;
                    o_wb += wb;
                    continue;
                }
                const int first = __builtin_ctzll(S), last = 63 - __builtin_clzll(S);
                if (lane < first) {
                    o_w += wv;
                    o_wb += wb;
                }
                fold(open, c + first);
                o_w = lane >= last ? wv : 0.0;
                o_wb = lane >= last ? wb : 0.0;
                open = c + last;
                if (lane >= first && lane < last) {
                    const double a = 0.5 * (static_cast<double>(c + run_first(S, lane)) + 1.0 + static_cast<double>(c + run_next(S, lane))) - mid;
                    s_a += a * wv;
                    s_aa += a * a * wv;
                    s_ab += a * wb;
                }
            }
        }
        uint32_t end = r1;
        const uint32_t tail = k[r1 - 1];
        if (r1 < n && k[r1] == tail) end = run_bound(k, r1, n, tail, true);
        fold(open, end);
    }
    double v[3] = {s_a, s_aa, s_ab};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double t = wave_sum(v[q]);
        if (lane == 0) red[q][wid] = t;
    }
    __syncthreads();
    if (wid == 0) {
        double tot[3], ts[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            double acc = 0.0;
            for (int j = 0; j < kW; ++j) acc += red[q][j];
            tot[q] = acc;
            double t = 0.0;
            for (int j = lane; j < target_blocks; j += kWave) t += tsum[q * kTargetBlocks + j];
            ts[q] = wave_sum(t);
        }
        if (lane == 0) {
            const double W = ts[0];
            const double va = tot[1] - tot[0] * tot[0] / W;
            const double vb = ts[2] - ts[1] * ts[1] / W;
            const double cab = tot[2] - tot[0] * ts[1] / W;
            const bool constant = k[0] == k[n - 1];    // one run of equal values
            float f;
            if (nan_flag[seg] || *target_nan) f = __builtin_nanf("");
            else if (constant || !(va > 0.0) || !(vb > 0.0) || !isfinite(va) || !isfinite(vb)) f = 0.0f;
            else f = static_cast<float>(fabs(cab / sqrt(va * vb)));
            fitness[prog0 + seg] = f;
        }
    }
}

// k_stamp: one lane records the device's constant-rate clock (kernel timing
// inside a captured graph, where event records are not available).
__global__ __launch_bounds__(kWave) void k_stamp(uint64_t* __restrict__ out) {
    if (threadIdx.x == 0) out[0] = wall_clock64();
}

// ---------------------------------------------------------------------------
// Host side: scratch, launch configuration, entry points.
// ---------------------------------------------------------------------------

struct DeviceScratch {
    void* counter = nullptr;     // the work counters: kCounterSets blocks of 1 KiB
    int32_t* order = nullptr;
    size_t order_cap = 0;
    double* part = nullptr;
    size_t part_cap = 0;         // doubles
    double* ystat = nullptr;
    size_t ystat_cap = 0;        // doubles
    uint4* code = nullptr;       // the adjoint's instruction stream
    size_t code_cap = 0;         // instructions
    int32_t* clen = nullptr;
    size_t clen_cap = 0;
    uint4* ecode = nullptr;      // the evaluation kernel's instruction stream
    size_t ecode_cap = 0;
    uint32_t* ehdr = nullptr;    // its programs' headers
    size_t ehdr_cap = 0;
    double* stats = nullptr;     // per-program statistics (kStats doubles each)
    size_t stats_cap = 0;
    double* gpart = nullptr;     // gradient partials
    size_t gpart_cap = 0;
    double* gextra = nullptr;    // gradient sums of constants beyond kGradLds
    size_t gextra_cap = 0;
    float* tape = nullptr;       // adjoint tape overflow
    size_t tape_cap = 0;
    float* fit_tmp = nullptr;
    size_t fit_tmp_cap = 0;
    // Spearman: sort keys (the first also takes the program outputs) and
    // carried values, double-buffered; digit counts,
    // the target's ranks, NaN flags
    uint32_t* sp_k0 = nullptr;
    size_t sp_k0_cap = 0;
    uint32_t* sp_k1 = nullptr;
    size_t sp_k1_cap = 0;
    uint32_t* sp_v0 = nullptr;
    size_t sp_v0_cap = 0;
    uint32_t* sp_v1 = nullptr;
    size_t sp_v1_cap = 0;
    uint32_t* sp_cnt = nullptr;
    size_t sp_cnt_cap = 0;
    uint32_t* sp_r2y = nullptr;
    size_t sp_r2y_cap = 0;
    int32_t* sp_nan = nullptr;
    size_t sp_nan_cap = 0;
    double* sp_ty = nullptr;     // the target ranks' weighted sums (w, w b, w b^2)
    size_t sp_ty_cap = 0;
    int n_cu = 0;
    int dev = -1;
    std::string arch;
    bool fixed = false;          // carved from preallocated memory: never grown
};

std::mutex g_mu;
std::vector<DeviceScratch> g_dev;   // per-device arena of the plain entry points

// kernel timing (gp_profile_enable / gp_profile_read)
struct ProfRec {
    hipEvent_t a, b;
    int64_t node_rows;
};
bool g_prof_on = false;
std::vector<ProfRec> g_prof_pending;
gp_profile g_prof_acc{0, 0.0, 0};

gp_status grow(void** ptr, size_t* cap, size_t need_elems, size_t elem) {
    if (*cap >= need_elems && *ptr) return GP_OK;
    size_t n = std::max<size_t>(need_elems, 1);
    n = std::max(n, *cap * 2);
    if (*ptr) {
        GP_HIP(hipDeviceSynchronize());
        GP_HIP(hipFree(*ptr));
        *ptr = nullptr;
        *cap = 0;
    }
    hipError_t e = hipMalloc(ptr, n * elem);
    if (e != hipSuccess) {
        *ptr = nullptr;
        return fail(GP_ERR_OUT_OF_MEMORY, std::string("scratch allocation: ") + hipGetErrorString(e));
    }
    *cap = n;
    return GP_OK;
}

gp_status scratch_init(DeviceScratch& s, int dev) {
    if (s.counter) return GP_OK;
    GP_HIP(hipMalloc(&s.counter, kCounterSets * kCounterBytes));
    GP_HIP(hipMemset(s.counter, 0, kCounterSets * kCounterBytes));
    hipDeviceProp_t prop;
    GP_HIP(hipGetDeviceProperties(&prop, dev));
    s.n_cu = prop.multiProcessorCount;
    s.dev = dev;
    s.arch = prop.gcnArchName;
    const size_t colon = s.arch.find(':');
    if (colon != std::string::npos) s.arch.resize(colon);
    return GP_OK;
}

bool scratch_empty(const DeviceScratch& s) {
    return !s.counter && !s.order && !s.part && !s.ystat && !s.code && !s.clen && !s.ecode && !s.ehdr &&
           !s.stats && !s.gpart &&
           !s.gextra && !s.tape && !s.fit_tmp && !s.sp_k0 && !s.sp_k1 && !s.sp_v0 && !s.sp_v1 &&
           !s.sp_cnt && !s.sp_r2y && !s.sp_nan && !s.sp_ty;
}

// Frees every buffer of s (the caller has made its device current and idle).
void scratch_free(DeviceScratch& s) {
    for (void* q : {s.counter, static_cast<void*>(s.order), static_cast<void*>(s.part),
                    static_cast<void*>(s.ystat), static_cast<void*>(s.code), static_cast<void*>(s.clen),
                    static_cast<void*>(s.ecode), static_cast<void*>(s.ehdr),
                    static_cast<void*>(s.stats), static_cast<void*>(s.gpart), static_cast<void*>(s.gextra),
                    static_cast<void*>(s.tape), static_cast<void*>(s.fit_tmp),
                    static_cast<void*>(s.sp_k0), static_cast<void*>(s.sp_k1), static_cast<void*>(s.sp_v0),
                    static_cast<void*>(s.sp_v1), static_cast<void*>(s.sp_cnt),
                    static_cast<void*>(s.sp_r2y), static_cast<void*>(s.sp_nan), static_cast<void*>(s.sp_ty)})
        if (q) (void)hipFree(q);
    s = DeviceScratch{};
}

// The shared arena of the current device.
gp_status arena(DeviceScratch** out) {
    int dev = 0;
    GP_HIP(hipGetDevice(&dev));
    if (static_cast<int>(g_dev.size()) <= dev) g_dev.resize(dev + 1);
    gp_status rc = scratch_init(g_dev[dev], dev);
    if (rc != GP_OK) return rc;
    *out = &g_dev[dev];
    return GP_OK;
}

gp_status check_pop(const gp_population_dev* pop, const char* who) {
    if (!pop) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": population is NULL");
    if (pop->n_programs < 0) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": n_programs < 0");
    if (pop->n_programs > 0 && (!pop->nodes || !pop->prog_off || !pop->const_off || !pop->len))
        return fail(GP_ERR_INVALID_ARG, std::string(who) + ": population pointer is NULL");
    if (pop->n_programs > 0 && pop->total_nodes < pop->n_programs)
        return fail(GP_ERR_INVALID_ARG, std::string(who) + ": total_nodes below n_programs");
    return GP_OK;
}

gp_status check_data(const gp_dataset_dev* d, const char* who, bool need_y) {
    if (!d) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": dataset is NULL");
    if (!d->X || d->n_features < 1)
        return fail(GP_ERR_INVALID_ARG, std::string(who) + ": dataset needs X and n_features >= 1");
    if (d->n_rows < 1) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": n_rows must be >= 1");
    if (d->ld < d->n_rows) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": ld below n_rows");
    if (need_y && !d->y) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": y is NULL");
    return GP_OK;
}

gp_status check_fitness_metric(int metric, const char* who, bool spearman_ok = false) {
    if (gp_metric_larger_is_better(static_cast<gp_metric>(metric)) < 0)
        return fail(GP_ERR_INVALID_ARG, std::string(who) + ": unknown metric");
    if (metric >= GP_METRIC_USER_0 && metric <= GP_METRIC_USER_3 &&
        !((user_defined_mask() >> (GP_OP_USER2 + metric - GP_METRIC_USER_0)) & 1u))
        return fail(GP_ERR_INVALID_ARG, std::string(who) + ": a user loss needs its two-argument user function "
                                                            "(GP_OP_USER2 + i) defined");
    if (metric == GP_METRIC_SPEARMAN && !spearman_ok)
        return fail(GP_ERR_UNSUPPORTED, std::string(who) + ": Spearman has no derivative or launch configuration "
                                                            "(gp_fitness, generations and evolution compute it)");
    return GP_OK;
}

// ---------------------------------------------------------------------------
// Launch configuration of the evaluation kernel: forced > tuned > heuristic.
// ---------------------------------------------------------------------------
struct LaunchCfg {
    int R;        // rows per lane: 1, 2 or 4
    int freg;     // features held in registers: 0, 2 or 8
    int tiles;    // tiles of 64*R rows per chunk
    int wpb;      // wavefronts per block: 1, 2 or 4
};

bool cfg_valid(const LaunchCfg& c) {
    return (c.R == 1 || c.R == 2 || c.R == 4) && (c.freg == 0 || c.freg == 2 || c.freg == 8) && c.tiles >= 1 &&
           c.tiles <= (1 << 20) && (c.wpb == 1 || c.wpb == 2 || c.wpb == 4);
}

bool g_forced = false;
int64_t g_spear_workset = 0;       // Spearman batch working-set limit in bytes (0: automatic)
LaunchCfg g_forced_cfg{4, 0, 1, 4};

// Evaluation kernels differ by metric; each class is tuned on its own.
int kernel_class(int mode, int metric) {
    if (mode == 0) return 0;
    switch (metric) {
    case GP_METRIC_MSE:
    case GP_METRIC_RMSE: return 1;
    case GP_METRIC_MAE: return 2;
    case GP_METRIC_LOGLOSS: return 3;
    case GP_METRIC_PEARSON: return 4;
    default: return 5;   // user losses
    }
}

struct TuneKey {
    std::string arch;
    int n_cu;
    int F;
    int64_t N;
    int32_t P;
    int kclass;
    bool operator<(const TuneKey& o) const {
        return std::tie(arch, n_cu, F, N, P, kclass) < std::tie(o.arch, o.n_cu, o.F, o.N, o.P, o.kclass);
    }
};
struct TuneVal {
    LaunchCfg cfg;
    double ms;
};
std::map<TuneKey, TuneVal> g_tuned;

// doubles per partial sum of a kernel class
int64_t class_doubles(int kclass) { return kclass == 4 ? 4 : 1; }
constexpr int64_t kMostTiles = 64;              // tiles of the heuristic's longest chunk
constexpr int64_t kMostPartials = int64_t{6} << 20;

LaunchCfg heuristic_cfg(int F, int64_t N, int32_t P, int n_cu, int kclass) {
    LaunchCfg c;
    // four rows per lane amortise an instruction's fetch and jump best (1M rows
    // x 1,000 programs: 3.3 ms, 3.9 with two, 5.1 with one), and at 256
    // programs x 4,096 rows too (26 us against 28 and 32); fewer only where
    // the rows do not fill them
    c.R = N > 2 * kWave ? 4 : N > kWave ? 2 : 1;
    c.wpb = 4;
    // features in registers only for F <= 2: eight of them cost a wavefront per
    // SIMD at 4 rows per lane, which fetching them one use ahead does not
    // (equal for the nine-function set, 3.5 ms against 4.0 for all 21)
    c.freg = F <= 2 ? 2 : 0;
    const int64_t tile_rows = static_cast<int64_t>(kWave) * c.R;
    const int64_t n_tiles = (N + tile_rows - 1) / tile_rows;
    // about 10 items per resident wavefront, of at most 16 tiles: longer items
    // leave the last ones alone (1M x 1,000: 3.26 ms at 16 tiles, 3.36 at 32,
    // 3.65 at 64), shorter ones pay each item's claim and start (65,536 rows x
    // 1,024 short programs: 246 us at 8 tiles, 281 at 4, 428 at 2)
    const int64_t target_items = static_cast<int64_t>(n_cu) * 16 * 10;
    int64_t want_chunks = std::max<int64_t>(1, (target_items + P - 1) / std::max<int32_t>(P, 1));
    want_chunks = std::min(want_chunks, n_tiles);
    int64_t tiles = (n_tiles + want_chunks - 1) / want_chunks;
    tiles = std::min<int64_t>(std::max<int64_t>(tiles, 1), 16);
    // the chunks are dealt to the XCDs' queues in turn: of the sizes from half
    // to a quarter more, the one that leaves the least of a last round empty,
    // the nearest of those (65,536 rows x 1,024: 37 chunks 287 us, 32 chunks 246)
    auto waste = [&](int64_t t) {
        const int64_t nc = (n_tiles + t - 1) / t;
        return static_cast<double>((nc + kQueues - 1) / kQueues * kQueues) / static_cast<double>(nc);
    };
    int64_t best = tiles;
    for (int64_t t = std::max<int64_t>(1, tiles / 2); t <= std::min<int64_t>(16, tiles + tiles / 4); ++t)
        if (waste(t) < waste(best) - 0.005 ||
            (waste(t) < waste(best) + 0.005 && std::abs(t - tiles) < std::abs(best - tiles)))
            best = t;
    // beyond 48 MiB of partial sums longer chunks, since scratch and the 2^30
    // bound on the items go by the chunks: a wavefront then has hundreds of items,
    // and longer ones cost next to nothing (16.8M rows x 4,096 programs of up to
    // 60 nodes: 342 ms at 16 tiles, 341 at 43; of up to 200: 1,187 and 1,191; x
    // 1,000, Pearson: 89.0, 89.6, and 91.3 at 64).  With more than eight features
    // only beyond 192 MiB: the chunks that about a thousand programs have in
    // flight together then exceed an L2 (20 features x 1,024 programs: 70.9 ms at
    // 16 tiles, 81.0 at 43; eight features 80.7 and 82.0; 28 x 4,096 265 at both)
    const int64_t doubles = F > 8 ? 4 * kMostPartials : kMostPartials;
    const int64_t most = std::max<int64_t>(1, doubles / (class_doubles(kclass) * std::max<int32_t>(P, 1)));
    best = std::max(best, std::min(kMostTiles, (n_tiles + most - 1) / most));
    c.tiles = static_cast<int>(best);
    return c;
}

LaunchCfg pick_cfg(const DeviceScratch& sc, int F, int64_t N, int32_t P, int kclass, bool* automatic = nullptr) {
    if (g_forced) return g_forced_cfg;
    auto it = g_tuned.find(TuneKey{sc.arch, sc.n_cu, F, N, P, kclass});
    if (it != g_tuned.end()) return it->second.cfg;
    if (automatic) *automatic = true;
    return heuristic_cfg(F, N, P, sc.n_cu, kclass);
}

// How a launch of the evaluation kernel is timed: by the process-wide profile
// (plain entry points), by a pair of events recorded as graph nodes (captured
// generations), or not at all (autotuning, capture without timing).
struct Timing {
    bool profile = false;
    uint64_t* stamp = nullptr;   // device [2]: clock before and after the kernel
    const void** launched = nullptr;   // receives the evaluation kernel launched
};

template <int MODE, int METRIC>
gp_status launch_eval_m(const LaunchCfg& cfg, int n_cu, const PopView& pv, const CodeView& cv,
                        const DataView& dv, const Sched& s, float* out, double* part, hipStream_t st,
                        int64_t node_rows, const Timing& tm) {
    const int block = cfg.wpb * kWave;
    const size_t lds = sizeof(MathTabsLds) + static_cast<size_t>(cfg.wpb) * s.lds_slots * cfg.R * kWave * sizeof(float);
    auto go = [&](auto kernel) -> gp_status {
        int per_cu = 0;
        GP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, lds));
        per_cu = std::max(per_cu, 1);
        // as many as are resident, at most those whose first claims cover the
        // longest queue (by the items alone, a queue with one more than its
        // wavefronts left that one to all of them: one program on 1M rows, a
        // kernel of 34 to 42 us, 9.6 so)
        const int64_t longest = s.n_chunks < kQueues ? s.n_chunks * ((static_cast<int64_t>(pv.P) + kQueues - 1) / kQueues)
                                                     : (static_cast<int64_t>(s.n_chunks) + kQueues - 1) / kQueues * pv.P;
        const int64_t claim = static_cast<int64_t>(cfg.wpb) * s.batch;
        const int64_t blocks = std::max<int64_t>(
            1, std::min<int64_t>(static_cast<int64_t>(per_cu) * n_cu, kQueues * ((longest + claim - 1) / claim)));
        const bool prof = tm.profile && g_prof_on;
        ProfRec rec{nullptr, nullptr, node_rows};
        if (prof) {
            GP_HIP(hipEventCreate(&rec.a));
            GP_HIP(hipEventCreate(&rec.b));
            GP_HIP(hipEventRecord(rec.a, st));
        }
        if (tm.launched) *tm.launched = reinterpret_cast<const void*>(kernel);
        if (tm.stamp) hipLaunchKernelGGL(k_stamp, dim3(1), dim3(kWave), 0, st, tm.stamp);
        Sched sl = s;
        sl.blocks = static_cast<int32_t>(blocks);
        sl.wpb = cfg.wpb;
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(block), lds, st, pv, cv, dv, sl, out,
                           part);
        GP_HIP(hipGetLastError());
        if (tm.stamp) {
            hipLaunchKernelGGL(k_stamp, dim3(1), dim3(kWave), 0, st, tm.stamp + 1);
            GP_HIP(hipGetLastError());
        }
        if (prof) {
            GP_HIP(hipEventRecord(rec.b, st));
            g_prof_pending.push_back(rec);
        }
        return GP_OK;
    };
#define GP_CASE(RR, FF)                                                \
    if (cfg.R == RR && cfg.freg == FF) return go(k_eval<RR, FF, MODE, METRIC>);
    GP_CASE(1, 0) GP_CASE(1, 2) GP_CASE(1, 8)
    GP_CASE(2, 0) GP_CASE(2, 2) GP_CASE(2, 8)
    GP_CASE(4, 0) GP_CASE(4, 2) GP_CASE(4, 8)
#undef GP_CASE
    return fail(GP_ERR_INVALID_ARG, "no kernel for this launch configuration");
}

gp_status launch_eval(int mode, int metric, const LaunchCfg& cfg, int n_cu, const PopView& pv,
                      const CodeView& cv, const DataView& dv, const Sched& s, float* out, double* part,
                      hipStream_t st, int64_t node_rows, const Timing& tm) {
    if (mode == 0)
        return launch_eval_m<0, GP_METRIC_MSE>(cfg, n_cu, pv, cv, dv, s, out, part, st, node_rows, tm);
    switch (metric) {
    case GP_METRIC_MAE:
        return launch_eval_m<1, GP_METRIC_MAE>(cfg, n_cu, pv, cv, dv, s, out, part, st, node_rows, tm);
    case GP_METRIC_MSE:
    case GP_METRIC_RMSE:
        return launch_eval_m<1, GP_METRIC_MSE>(cfg, n_cu, pv, cv, dv, s, out, part, st, node_rows, tm);
    case GP_METRIC_LOGLOSS:
        return launch_eval_m<1, GP_METRIC_LOGLOSS>(cfg, n_cu, pv, cv, dv, s, out, part, st, node_rows, tm);
    case GP_METRIC_PEARSON:
        return launch_eval_m<1, GP_METRIC_PEARSON>(cfg, n_cu, pv, cv, dv, s, out, part, st, node_rows, tm);
    case GP_METRIC_USER_0:
    case GP_METRIC_USER_1:
    case GP_METRIC_USER_2:
    case GP_METRIC_USER_3:
        return launch_eval_m<1, GP_METRIC_USER_0>(cfg, n_cu, pv, cv, dv, s, out, part, st, node_rows, tm);
    default: return fail(GP_ERR_UNSUPPORTED, "metric not supported by the fused fitness kernel");
    }
}

// How the evaluation stream expands user functions (Sec. V): the
// definitions, the loss wrapped around every program (GP_METRIC_USER_i), and
// the room this takes: program p's stream starts at prog_off[p] * mul +
// p * add, and the kernel's LDS holds lds_slots stack slots per row.
struct ExpandPlan {
    UserDefs defs;
    int32_t loss_fn = -1;
    int32_t mul = 1, add = 0;
    int32_t lds_slots = kEvalLds;
};

bool is_user_metric(int metric) { return metric >= GP_METRIC_USER_0 && metric <= GP_METRIC_USER_3; }

ExpandPlan expand_plan(int mode, int metric) {
    ExpandPlan x;
    user_defs(&x.defs);
    const uint32_t mask = user_defined_mask();
    if (mask == 0u) return x;
    for (int u = 0; u < kUserFns; ++u)
        if ((mask >> (GP_OP_USER1 + u)) & 1u) x.mul = std::max(x.mul, x.defs.len[u]);
    if (mode == 1 && is_user_metric(metric)) {
        x.loss_fn = metric - GP_METRIC_USER_0;
        x.add = 1 + x.defs.len[kUserFns / 2 + x.loss_fn];
    }
    x.lds_slots = kEvalLdsUser;
    return x;
}

// Scratch sizes one evaluation needs; grows sc's buffers to them (a fixed
// scratch must already hold them).  Called outside any stream capture (it may
// allocate).  adjoint_per_node: 16-byte units of the adjoint's instruction
// stream per node (0: none).
gp_status reserve(DeviceScratch* sc, int32_t P, int64_t total_nodes, int64_t n_chunks, int mode, int metric,
                  int64_t adjoint_per_node = 0, int32_t ex_mul = 1, int32_t ex_add = 0) {
    auto need = [sc](auto** ptr, size_t* cap, size_t n, size_t elem) -> gp_status {
        if (!sc->fixed) return grow(reinterpret_cast<void**>(ptr), cap, n, elem);
        if (*ptr && *cap >= n) return GP_OK;
        return fail(GP_ERR_BUFFER_TOO_SMALL, "fixed scratch smaller than the evaluation needs");
    };
    gp_status rc = need(&sc->order, &sc->order_cap, P, sizeof(int32_t));
    if (rc != GP_OK) return rc;
    if (adjoint_per_node > 0) {
        rc = need(&sc->code, &sc->code_cap, static_cast<size_t>(total_nodes * adjoint_per_node + kCodePad), sizeof(uint4));
        if (rc != GP_OK) return rc;
        rc = need(&sc->clen, &sc->clen_cap, P, sizeof(int32_t));
        if (rc != GP_OK) return rc;
    }
    // (the evaluation kernel fetches whole blocks of instructions, past a
    // program's end; in a fixed scratch other buffers follow)
    rc = need(&sc->ecode, &sc->ecode_cap,
              static_cast<size_t>(total_nodes) * ex_mul + static_cast<size_t>(P) * ex_add +
                  static_cast<size_t>(sc->fixed ? 1 : kCodePad),
              sizeof(uint4));
    if (rc != GP_OK) return rc;
    rc = need(&sc->ehdr, &sc->ehdr_cap, P, sizeof(uint32_t));
    if (rc != GP_OK) return rc;
    if (mode == 1) {
        const size_t kk = metric == GP_METRIC_PEARSON ? 4 : 1;
        rc = need(&sc->part, &sc->part_cap, static_cast<size_t>(P) * n_chunks * kk, sizeof(double));
        if (rc != GP_OK) return rc;
        rc = need(&sc->ystat, &sc->ystat_cap, static_cast<size_t>(n_chunks) * 4, sizeof(double));
        if (rc != GP_OK) return rc;
    }
    return GP_OK;
}

gp_status chunking(const gp_population_dev* pop, const gp_dataset_dev* data, const LaunchCfg& cfg,
                   int64_t* chunk, int64_t* n_chunks) {
    if (!cfg_valid(cfg)) return fail(GP_ERR_INVALID_ARG, "invalid launch configuration");
    if (cfg.freg > 0 && data->n_features > cfg.freg)
        return fail(GP_ERR_INVALID_ARG, "launch configuration holds fewer feature registers than n_features");
    *chunk = static_cast<int64_t>(cfg.tiles) * kWave * cfg.R;
    *n_chunks = (data->n_rows + *chunk - 1) / *chunk;
    // the 32-bit work counter overshoots n_items by at most one per wavefront
    if (*n_chunks * pop->n_programs > (int64_t{1} << 30))
        return fail(GP_ERR_INVALID_ARG, "too many work items (n_programs * row chunks above 2^30)");
    return GP_OK;
}

// Shared front half of the evaluation paths: configuration, scratch, the
// length ordering and the instruction streams.  `force` (nullable) overrides
// the configuration choice.  The evaluation kernel's stream (constant
// subtrees folded) is compiled unless adjoint_R > 0 asks for the adjoint's
// instead, for k_adjoint at that many rows per lane and, where `longer` says
// that there may be programs of more than kParNodes nodes, for k_adjoint_long;
// `both` compiles the two (a backward pass that runs a forward pass first).
gp_status prepare(DeviceScratch* sc, const gp_population_dev* pop, const gp_dataset_dev* data, int mode,
                  int metric, hipStream_t st, const LaunchCfg* force, PopView* pv, CodeView* cvw, DataView* dv,
                  Sched* sch, LaunchCfg* cfg, int adjoint_R = 0, bool both = false, bool longer = false) {
    const bool adjoint = adjoint_R > 0;
    *pv = PopView{pop->nodes, pop->prog_off, pop->consts, pop->const_off, pop->len, pop->n_programs};
    *dv = DataView{data->X, data->ld, data->n_features, data->n_rows, data->y, data->w};
    *cfg = force ? *force
                 : pick_cfg(*sc, data->n_features, data->n_rows, pop->n_programs, kernel_class(mode, metric));
    int64_t chunk = 0, n_chunks = 0;
    gp_status rc = chunking(pop, data, *cfg, &chunk, &n_chunks);
    if (rc != GP_OK) return rc;
    const ExpandPlan xp = expand_plan(mode, metric);
    rc = reserve(sc, pop->n_programs, pop->total_nodes, n_chunks, mode, metric,
                 adjoint ? kAdjCodePerNode : 0, xp.mul, xp.add);
    if (rc != GP_OK) return rc;
    // items per claim: single ones up to 64 a resident wavefront (16 per CU).
    // A claim costs its queue about 25 ns, but consecutive items are programs of
    // like length, and a wavefront that claims several of the longest holds up
    // the rest (1M rows x 1,000 programs, 62 items a wavefront: 3.26 ms with
    // single claims, 3.9 with seven items each)
    const int64_t n_items = n_chunks * pop->n_programs;
    const int64_t claims = static_cast<int64_t>(sc->n_cu) * 16 * 32;
    const int32_t batch = static_cast<int32_t>(std::min<int64_t>(8, std::max<int64_t>(1, n_items / claims)));
    *sch = Sched{chunk, static_cast<int32_t>(n_chunks), n_items, sc->order, static_cast<uint32_t*>(sc->counter),
                 batch, xp.lds_slots, 0, 0};
    const bool eval = !adjoint || both;
    const OrderArgs oa{pop->len, pop->n_programs, sc->order, static_cast<uint32_t*>(sc->counter), adjoint ? kCounterSets : 1};
    // programs per compiling wavefront: one, or while user functions are
    // defined as many as leave each resident wavefront (12 per CU) one group
    const int64_t resident = static_cast<int64_t>(sc->n_cu) * 12;
    const int32_t group = xp.lds_slots == kEvalLdsUser
                              ? static_cast<int32_t>(std::min<int64_t>(kSeqLanes, std::max<int64_t>(1, (pop->n_programs + resident - 1) / resident)))
                              : 1;
    const EvalCompile ec{sc->ecode, sc->ehdr, xp.defs, xp.loss_fn, xp.mul, xp.add,
                         Emit{eval_ops(cfg->freg), cfg->R, cfg->freg == 0}, group};
    const AdjCompile ac{sc->code, reinterpret_cast<uint32_t*>(sc->clen), Emit{eval_ops(0), adjoint_R, 1}, sc->gextra};
    auto compile = [&](auto kernel, int waves, bool with_eval, bool with_adjoint) {
        const int64_t P = pop->n_programs, per = static_cast<int64_t>(waves) * group;
        const int64_t blocks = 1 + (with_adjoint ? (P + waves - 1) / waves : 0) + (with_eval ? (P + per - 1) / per : 0);
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(waves * kWave), 0, st, *pv, oa, ec, ac);
    };
    if (adjoint && eval) compile(k_compile_streams<true, true>, compile_waves<true, true>(), true, true);
    else if (adjoint) compile(k_compile_streams<false, true>, compile_waves<false, true>(), false, true);
    else compile(k_compile_streams<true, false>, compile_waves<true, false>(), true, false);
    GP_HIP(hipGetLastError());
    if (adjoint && longer) {
        const unsigned blocks = (pop->n_programs + kBlock - 1) / kBlock;
        hipLaunchKernelGGL(k_compile, dim3(blocks), dim3(kBlock), 0, st, *pv, sc->code, sc->clen);
        GP_HIP(hipGetLastError());
    }
    *cvw = CodeView{adjoint ? sc->code : nullptr, adjoint ? sc->clen : nullptr,
                    (!adjoint || both) ? sc->ecode : nullptr, (!adjoint || both) ? sc->ehdr : nullptr, xp.mul,
                    xp.add};
    return GP_OK;
}

// Fitness of every program into `fitness` (device), on scratch sc.
gp_status fitness_impl(DeviceScratch* sc, const gp_population_dev* pop, const gp_dataset_dev* data, int metric,
                       float* fitness, hipStream_t st, const LaunchCfg* force, const Timing& tm) {
    PopView pv;
    CodeView cvw;
    DataView dv;
    Sched sch;
    LaunchCfg cfg;
    gp_status rc = prepare(sc, pop, data, 1, metric, st, force, &pv, &cvw, &dv, &sch, &cfg);
    if (rc != GP_OK) return rc;
    const bool need_ystats = data->w != nullptr || metric == GP_METRIC_PEARSON;
    if (need_ystats) {
        const int blocks = (sch.n_chunks + (kBlock / kWave) - 1) / (kBlock / kWave);
        hipLaunchKernelGGL(k_ystats, dim3(blocks), dim3(kBlock), 0, st, dv, sch.chunk, sch.n_chunks, sc->ystat);
        GP_HIP(hipGetLastError());
    }
    rc = launch_eval(1, metric, cfg, sc->n_cu, pv, cvw, dv, sch, nullptr, sc->part, st,
                     pop->total_nodes * data->n_rows, tm);
    if (rc != GP_OK) return rc;
    const int fblocks = (pop->n_programs + (kBlock / kWave) - 1) / (kBlock / kWave);
    const int has_w = data->w != nullptr;
#define GP_FIN(M)                                                                                  \
    hipLaunchKernelGGL(k_finalize<M>, dim3(fblocks), dim3(kBlock), 0, st, sc->part, sc->ystat,   \
                       sch.n_chunks, pop->n_programs, data->n_rows, has_w, fitness, nullptr)
    switch (metric) {
    case GP_METRIC_MAE: GP_FIN(GP_METRIC_MAE); break;
    case GP_METRIC_USER_0: case GP_METRIC_USER_1: case GP_METRIC_USER_2: case GP_METRIC_USER_3:
        GP_FIN(GP_METRIC_MAE);   // the weighted mean of the row losses
        break;
    case GP_METRIC_MSE: GP_FIN(GP_METRIC_MSE); break;
    case GP_METRIC_RMSE: GP_FIN(GP_METRIC_RMSE); break;
    case GP_METRIC_LOGLOSS: GP_FIN(GP_METRIC_LOGLOSS); break;
    default: GP_FIN(GP_METRIC_PEARSON); break;
    }
#undef GP_FIN
    GP_HIP(hipGetLastError());
    return GP_OK;
}

// ---- fitness without allocation ----
// One static array per device serves every gp_fitness_noalloc call on it.
// In host code `scratch` names a host-side stand-in: the device address comes
// from hipGetSymbolAddress, once per device, and only that address reaches
// kernels.
constexpr size_t kNoAllocBytes = size_t{64} << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocBytes];
constexpr int kNoAllocMaxDevices = 64;
struct NoAllocDevice {
    unsigned char* ptr = nullptr;   // this device's copy of `scratch`
    int n_cu = 0;
    char arch[64] = {};
};
NoAllocDevice g_noalloc[kNoAllocMaxDevices];

size_t align256(size_t n) { return (n + 255) & ~size_t{255}; }

// Bytes of the device's array that one fitness evaluation takes.
size_t noalloc_bytes(int32_t P, int64_t total_nodes, int64_t n_chunks, int metric) {
    const size_t kk = metric == GP_METRIC_PEARSON ? 4 : 1;
    const ExpandPlan xp = expand_plan(1, metric);
    const size_t n_code = static_cast<size_t>(total_nodes) * xp.mul + static_cast<size_t>(P) * xp.add + 1;
    return kCounterBytes + align256(static_cast<size_t>(P) * sizeof(int32_t)) * 2 + align256(n_code * sizeof(uint4)) +
           align256(static_cast<size_t>(P) * static_cast<size_t>(n_chunks) * kk * sizeof(double)) +
           align256(static_cast<size_t>(n_chunks) * 4 * sizeof(double));
}

// Carves the scratch of one fitness evaluation out of the device's array into
// sc (caps exact, fixed: reserve() checks instead of growing).  Fails if the
// evaluation needs more than kNoAllocBytes.
gp_status noalloc_carve(unsigned char* base, DeviceScratch* sc, int32_t P, int64_t total_nodes, int64_t n_chunks,
                        int metric) {
    const size_t kk = metric == GP_METRIC_PEARSON ? 4 : 1;
    const ExpandPlan xp = expand_plan(1, metric);
    const size_t n_code = static_cast<size_t>(total_nodes) * xp.mul + static_cast<size_t>(P) * xp.add + 1;
    const size_t n_part = static_cast<size_t>(P) * static_cast<size_t>(n_chunks) * kk;
    const size_t n_ystat = static_cast<size_t>(n_chunks) * 4;
    const size_t bytes = noalloc_bytes(P, total_nodes, n_chunks, metric);
    if (bytes > kNoAllocBytes)
        return fail(GP_ERR_INVALID_ARG, "gp_fitness_noalloc: this evaluation needs " + std::to_string(bytes) +
                                            " bytes of scratch, above the limit of " +
                                            std::to_string(kNoAllocBytes) + " (use gp_fitness)");
    size_t off = 0;
    auto take = [&](size_t n) {
        unsigned char* q = base + off;
        off += align256(n);
        return q;
    };
    sc->counter = take(kCounterBytes);
    sc->order = reinterpret_cast<int32_t*>(take(static_cast<size_t>(P) * sizeof(int32_t)));
    sc->order_cap = static_cast<size_t>(P);
    sc->ehdr = reinterpret_cast<uint32_t*>(take(static_cast<size_t>(P) * sizeof(uint32_t)));
    sc->ehdr_cap = static_cast<size_t>(P);
    sc->ecode = reinterpret_cast<uint4*>(take(n_code * sizeof(uint4)));
    sc->ecode_cap = n_code;
    // (whole blocks of instructions are fetched, up to 504 bytes past the
    // stream's end: the two buffers after it, at least 256 bytes each, cover that)
    sc->part = reinterpret_cast<double*>(take(n_part * sizeof(double)));
    sc->part_cap = n_part;
    sc->ystat = reinterpret_cast<double*>(take(n_ystat * sizeof(double)));
    sc->ystat_cap = n_ystat;
    sc->fixed = true;
    return GP_OK;
}

gp_status tournament_impl(const float* fitness, const int32_t* len, int32_t P, int larger, float parsimony,
                          int32_t k, int32_t T, uint64_t seed, uint32_t gen, const uint32_t* gen_dev,
                          int32_t* winners, hipStream_t st) {
    if (T == 0) return GP_OK;
    // a lane per block of four draws, up to a wavefront, while T tournaments then
    // take at most two wavefronts per SIMD; beyond that, lanes without a block
    // cost more than the shorter chains give (size 7: T = 32,768, 3.8 us with two
    // lanes, 4.2 with four; T = 131,072, 5.3 with one, 6.5 with four)
    int lg = 0;
    while (lg < 6 && (4 << lg) < k && (static_cast<int64_t>(T) << (lg + 1)) <= kTourLanes) ++lg;
    const int64_t blocks = ((static_cast<int64_t>(T) << lg) + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_tournament, dim3(static_cast<unsigned>(blocks)), dim3(kBlock), 0, st, fitness, len, P, larger,
                       parsimony, k, T, lg, seed, gen, gen_dev, winners);
    GP_HIP(hipGetLastError());
    return GP_OK;
}

__global__ __launch_bounds__(kBlock) void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) p[i] = v;
}

// Sorts the B segments of N float values at src (keys formed in the first
// pass, each carrying its row's target rank, or its row when rank2_y is
// NULL): the sorted keys and values end in k0 / v0, and nan_flag[s] is
// raised for a segment holding a NaN.  src may be k0 itself (the first pass
// writes k1 / v1 only).
gp_status radix_sort_segments(DeviceScratch* sc, const float* src, const uint32_t* rank2_y, int64_t N, int32_t B,
                              int32_t* nan_flag, hipStream_t st) {
    const int32_t T = static_cast<int32_t>((N + kRsTile - 1) / kRsTile);
    const uint32_t* in0 = reinterpret_cast<const uint32_t*>(src);
    hipLaunchKernelGGL(k_rs_count<true>, dim3(T, B), dim3(kRsBlock), 0, st, in0, N, T, 0, sc->sp_cnt, nan_flag);
    GP_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_rs_scan, dim3(B), dim3(1024), 0, st, sc->sp_cnt, T);
    GP_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_rs_scatter<true>, dim3(T, B), dim3(kRsScatterBlock), 0, st, in0, nullptr, sc->sp_k1,
                       sc->sp_v1, N, T, 0, sc->sp_cnt, rank2_y);
    GP_HIP(hipGetLastError());
    uint32_t *kin = sc->sp_k1, *vin = sc->sp_v1, *kout = sc->sp_k0, *vout = sc->sp_v0;
    for (int pass = 1; pass < 4; ++pass) {
        const int shift = 8 * pass;
        hipLaunchKernelGGL(k_rs_count<false>, dim3(T, B), dim3(kRsBlock), 0, st, kin, N, T, shift, sc->sp_cnt,
                           nullptr);
        GP_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_rs_scan, dim3(B), dim3(1024), 0, st, sc->sp_cnt, T);
        GP_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_rs_scatter<false>, dim3(T, B), dim3(kRsScatterBlock), 0, st, kin, vin, kout, vout, N,
                           T, shift, sc->sp_cnt, nullptr);
        GP_HIP(hipGetLastError());
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    return GP_OK;
}

// Spearman fitness (Sec. III-C3): programs in batches of B are evaluated,
// ranked by a sort, and correlated with the target's ranks.
gp_status spearman_impl(DeviceScratch* sc, const gp_population_dev* pop, const gp_dataset_dev* data,
                        float* fitness, hipStream_t st) {
    const int64_t N = data->n_rows;
    const int32_t P = pop->n_programs;
    if (N >= (int64_t{1} << 31)) return fail(GP_ERR_INVALID_ARG, "gp_fitness: Spearman needs n_rows below 2^31");
    const int32_t T = static_cast<int32_t>((N + kRsTile - 1) / kRsTile);
    // working set per program: keys and carried values twice, the outputs
    // sharing the first key buffer (16 bytes per row).  Up to the set limit,
    // else 16 GiB of it and at most half the
    // free memory; a program's fitness does not depend on its batch.  When
    // the programs need several batches, a batch is a whole number of rounds
    // of resident correlation workgroups (one per program).
    int64_t budget = g_spear_workset;
    if (budget <= 0) {
        size_t free_b = 0, total_b = 0;
        GP_HIP(hipMemGetInfo(&free_b, &total_b));
        budget = std::max<int64_t>(std::min<int64_t>(int64_t{16} << 30, static_cast<int64_t>(free_b / 2)),
                                   int64_t{256} << 20);
    }
    int64_t Bmax = std::max<int64_t>(1, budget / (16 * N));
    if (Bmax < P) {
        int per_cu = 0;
        GP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_spear_corr<false>, 1024, 0));
        const int64_t round = static_cast<int64_t>(std::max(per_cu, 1)) * sc->n_cu;
        if (Bmax > round) Bmax = (Bmax / round) * round;
    }
    const int32_t B = static_cast<int32_t>(std::min<int64_t>(P, Bmax));
    const size_t BN = static_cast<size_t>(B) * static_cast<size_t>(N);
    gp_status rc = GP_OK;
    auto need = [&](void** ptr, size_t* cap, size_t n, size_t elem) {
        if (rc == GP_OK) rc = grow(ptr, cap, n, elem);
    };
    need(reinterpret_cast<void**>(&sc->sp_k0), &sc->sp_k0_cap, BN, sizeof(uint32_t));
    need(reinterpret_cast<void**>(&sc->sp_k1), &sc->sp_k1_cap, BN, sizeof(uint32_t));
    need(reinterpret_cast<void**>(&sc->sp_v0), &sc->sp_v0_cap, BN, sizeof(uint32_t));
    need(reinterpret_cast<void**>(&sc->sp_v1), &sc->sp_v1_cap, BN, sizeof(uint32_t));
    need(reinterpret_cast<void**>(&sc->sp_cnt), &sc->sp_cnt_cap, static_cast<size_t>(B) * kRsRadix * T,
         sizeof(uint32_t));
    need(reinterpret_cast<void**>(&sc->sp_r2y), &sc->sp_r2y_cap, static_cast<size_t>(N), sizeof(uint32_t));
    need(reinterpret_cast<void**>(&sc->sp_nan), &sc->sp_nan_cap, static_cast<size_t>(B) + 1, sizeof(int32_t));
    need(reinterpret_cast<void**>(&sc->sp_ty), &sc->sp_ty_cap, 3 * kTargetBlocks, sizeof(double));
    if (rc != GP_OK) return rc;
    auto fill_nan_flags = [&](int32_t* flags, int32_t n) -> gp_status {
        hipLaunchKernelGGL(k_fill_i32, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, flags,
                           static_cast<int64_t>(n), 0);
        GP_HIP(hipGetLastError());
        return GP_OK;
    };
    // the target's ranks (twice the mean rank of each row); a NaN in the
    // target (flag B) makes every program's fitness NaN
    int32_t* target_nan = sc->sp_nan + B;
    if ((rc = fill_nan_flags(target_nan, 1)) != GP_OK) return rc;
    if ((rc = radix_sort_segments(sc, data->y, nullptr, N, 1, target_nan, st)) != GP_OK) return rc;
    const int32_t target_blocks = static_cast<int32_t>(std::min<int64_t>((N + kBlock - 1) / kBlock, kTargetBlocks));
    hipLaunchKernelGGL(k_spear_rank_target, dim3(target_blocks), dim3(kBlock), 0, st, sc->sp_k0, sc->sp_v0, N, data->w,
                       sc->sp_r2y, sc->sp_ty);
    GP_HIP(hipGetLastError());
    for (int32_t p0 = 0; p0 < P; p0 += B) {
        const int32_t b = std::min(B, P - p0);
        gp_population_dev view = *pop;
        view.prog_off = pop->prog_off + p0;
        view.const_off = pop->const_off + p0;
        view.len = pop->len + p0;
        view.n_programs = b;
        PopView pv;
        CodeView cvw;
        DataView dv;
        Sched sch;
        LaunchCfg cfg;
        rc = prepare(sc, &view, data, 0, GP_METRIC_MSE, st, nullptr, &pv, &cvw, &dv, &sch, &cfg);
        if (rc != GP_OK) return rc;
        // the outputs go to the first key buffer, which the sort's first pass
        // reads before anything writes it again
        float* out = reinterpret_cast<float*>(sc->sp_k0);
        rc = launch_eval(0, GP_METRIC_MSE, cfg, sc->n_cu, pv, cvw, dv, sch, out, nullptr, st, 0, Timing{});
        if (rc != GP_OK) return rc;
        if ((rc = fill_nan_flags(sc->sp_nan, b)) != GP_OK) return rc;
        if ((rc = radix_sort_segments(sc, out, data->w ? nullptr : sc->sp_r2y, N, b, sc->sp_nan, st)) != GP_OK)
            return rc;
        if (data->w)
            hipLaunchKernelGGL(k_spear_corr<true>, dim3(b), dim3(1024), 0, st, sc->sp_k0, sc->sp_v0, N, sc->sp_r2y,
                               data->w, sc->sp_ty, target_blocks, sc->sp_nan, target_nan, fitness, p0);
        else
            hipLaunchKernelGGL(k_spear_corr<false>, dim3(b), dim3(1024), 0, st, sc->sp_k0, sc->sp_v0, N, sc->sp_r2y,
                               nullptr, sc->sp_ty, target_blocks, sc->sp_nan, target_nan, fitness, p0);
        GP_HIP(hipGetLastError());
    }
    return GP_OK;
}

// ---------------------------------------------------------------------------
// Autotuner: times candidate configurations of the fitness kernel on a prefix
// of at most kTuneRows rows and keeps the fastest for the full shape.
// ---------------------------------------------------------------------------
constexpr int64_t kTuneRows = int64_t{1} << 20;

gp_status autotune_impl(DeviceScratch* sc, const gp_population_dev* pop, const gp_dataset_dev* data, int metric,
                        int repeats, hipStream_t st, LaunchCfg* best_out, double* best_ms_out) {
    gp_dataset_dev sub = *data;
    sub.n_rows = std::min(data->n_rows, kTuneRows);
    gp_status rc = grow(reinterpret_cast<void**>(&sc->fit_tmp), &sc->fit_tmp_cap,
                        static_cast<size_t>(std::max(pop->n_programs, 1)), sizeof(float));
    if (rc != GP_OK) return rc;
    const LaunchCfg h = heuristic_cfg(data->n_features, data->n_rows, pop->n_programs, sc->n_cu, kernel_class(1, metric));
    std::vector<int> fregs;
    if (data->n_features <= 2) fregs.push_back(2);
    if (data->n_features <= 8) fregs.push_back(8);
    fregs.push_back(0);
    // none beyond the heuristic's longest: the prefix has few items a wavefront
    // and flatters them (4,096 programs: 75.2 ms at 64 tiles and 74.8 at 128 on
    // the prefix, 1,194 and 1,203 on 16.8M rows)
    std::vector<int> tiles;
    for (int t : {h.tiles / 4, h.tiles / 2, h.tiles, h.tiles * 2})
        if (t >= 1 && t <= kMostTiles && std::find(tiles.begin(), tiles.end(), t) == tiles.end()) tiles.push_back(t);
    hipEvent_t a = nullptr, b = nullptr;
    GP_HIP(hipEventCreate(&a));
    GP_HIP(hipEventCreate(&b));
    LaunchCfg best = h;
    double best_ms = -1.0;
    auto trial = [&](const LaunchCfg& c) {
        int64_t chunk = 0, n_chunks = 0;
        if (chunking(pop, data, c, &chunk, &n_chunks) != GP_OK) return;   // does not fit this shape
        double ms_min = -1.0;
        for (int rep = 0; rep <= repeats && rc == GP_OK; ++rep) {
            rc = hipEventRecord(a, st) == hipSuccess ? GP_OK : GP_ERR_DEVICE;
            if (rc == GP_OK) rc = fitness_impl(sc, pop, &sub, metric, sc->fit_tmp, st, &c, Timing{});
            if (rc == GP_OK) rc = hipEventRecord(b, st) == hipSuccess ? GP_OK : GP_ERR_DEVICE;
            if (rc == GP_OK) rc = hipEventSynchronize(b) == hipSuccess ? GP_OK : GP_ERR_DEVICE;
            float ms = 0.0f;
            if (rc == GP_OK) rc = hipEventElapsedTime(&ms, a, b) == hipSuccess ? GP_OK : GP_ERR_DEVICE;
            if (rc == GP_OK && rep > 0 && (ms_min < 0.0 || ms < ms_min)) ms_min = ms;  // rep 0 warms up
        }
        if (rc == GP_OK && ms_min >= 0.0 && (best_ms < 0.0 || ms_min < best_ms)) {
            best_ms = ms_min;
            best = c;
        }
    };
    // stage 1: rows per lane, feature registers, rows per work item (keeping
    // the heuristic's rows per item within a factor of 4), 4 waves per block
    for (int R : {1, 2, 4})
        for (int fr : fregs)
            for (int t : tiles)
                if (rc == GP_OK) trial(LaunchCfg{R, fr, std::max(1, t * 4 / R), 4});
    // stage 2: the block size for the best of stage 1
    const LaunchCfg s1 = best;
    for (int wpb : {1, 2})
        if (rc == GP_OK) trial(LaunchCfg{s1.R, s1.freg, s1.tiles, wpb});
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (rc != GP_OK) return rc == GP_ERR_DEVICE ? fail(GP_ERR_DEVICE, "autotune: a timed launch failed") : rc;
    if (best_ms < 0.0) return fail(GP_ERR_INVALID_ARG, "autotune: no launch configuration fits this shape");
    g_tuned[TuneKey{sc->arch, sc->n_cu, data->n_features, data->n_rows, pop->n_programs, kernel_class(1, metric)}] =
        TuneVal{best, best_ms};
    *best_out = best;
    if (best_ms_out) *best_ms_out = best_ms;
    return GP_OK;
}

// ---------------------------------------------------------------------------
// One generation as a HIP graph.
// ---------------------------------------------------------------------------
size_t align_up(size_t v) { return (v + 255) & ~size_t{255}; }

struct StageLayout {
    size_t gen, len, prog_off, const_off, nodes, consts, bytes;
};

StageLayout stage_layout(int32_t P, int64_t node_cap, int64_t const_cap) {
    StageLayout l;
    l.gen = 0;
    l.len = 256;
    l.prog_off = align_up(l.len + sizeof(int32_t) * static_cast<size_t>(P));
    l.const_off = align_up(l.prog_off + sizeof(int64_t) * (static_cast<size_t>(P) + 1));
    l.nodes = align_up(l.const_off + sizeof(int64_t) * (static_cast<size_t>(P) + 1));
    l.consts = align_up(l.nodes + sizeof(uint32_t) * static_cast<size_t>(node_cap));
    l.bytes = align_up(l.consts + sizeof(float) * static_cast<size_t>(std::max<int64_t>(const_cap, 1)));
    return l;
}

}  // namespace

struct gp_generation_s {
    gp_generation_params prm{};
    gp_dataset_dev data{};
    int dev = 0;
    hipStream_t stream = nullptr;
    DeviceScratch sc;
    StageLayout lay{};
    char* h_stage = nullptr;     // pinned: the population of the next generation
    char* d_stage = nullptr;
    float* d_fit = nullptr;
    int32_t* d_win = nullptr;
    float* h_fit = nullptr;      // pinned outputs
    int32_t* h_win = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    uint64_t* d_stamp = nullptr;  // evaluation-kernel clock stamps (time_kernel)
    uint64_t* h_stamp = nullptr;
    int clock_khz = 0;
    hipEvent_t ev_a = nullptr, ev_b = nullptr;   // event nodes around the evaluation kernel
    bool events = false;
    const void* eval_kernel = nullptr;
    LaunchCfg cfg{4, 0, 1};
    bool captured = false;
    double tuned_ms = -1.0;
    float kernel_ms = -1.0f;    // HIP events if inserted, else the clock stamps
    float clock_ms = -1.0f;     // clock stamps
};

namespace {

gp_population_dev stage_view(const gp_generation_s* g, int64_t total_nodes, int64_t total_consts) {
    gp_population_dev v{};
    v.nodes = reinterpret_cast<const uint32_t*>(g->d_stage + g->lay.nodes);
    v.prog_off = reinterpret_cast<const int64_t*>(g->d_stage + g->lay.prog_off);
    v.consts = reinterpret_cast<const float*>(g->d_stage + g->lay.consts);
    v.const_off = reinterpret_cast<const int64_t*>(g->d_stage + g->lay.const_off);
    v.len = reinterpret_cast<const int32_t*>(g->d_stage + g->lay.len);
    v.n_programs = g->prm.n_programs;
    v.total_nodes = total_nodes;
    v.max_len = 0;
    v.total_consts = total_consts;
    return v;
}

void generation_release(gp_generation_s* g) {
    if (g->stream) (void)hipStreamSynchronize(g->stream);
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    if (g->ev_a) (void)hipEventDestroy(g->ev_a);
    if (g->ev_b) (void)hipEventDestroy(g->ev_b);
    if (g->d_stamp) (void)hipFree(g->d_stamp);
    if (g->h_stamp) (void)hipHostFree(g->h_stamp);
    if (g->h_stage) (void)hipHostFree(g->h_stage);
    if (g->h_fit) (void)hipHostFree(g->h_fit);
    if (g->h_win) (void)hipHostFree(g->h_win);
    if (g->d_stage) (void)hipFree(g->d_stage);
    if (g->d_fit) (void)hipFree(g->d_fit);
    if (g->d_win) (void)hipFree(g->d_win);
    scratch_free(g->sc);
    if (g->stream) (void)hipStreamDestroy(g->stream);
}

// Fitness step of the generation objects: the fused kernels, or for
// Spearman the batched evaluate / rank / correlate pipeline (whose buffers
// must exist before a capture: one eager call grows them).
gp_status graph_fitness(DeviceScratch* sc, const gp_population_dev* view, const gp_dataset_dev* data, int metric,
                        float* fit, hipStream_t st, const LaunchCfg* cfg, const Timing& tm) {
    if (metric == GP_METRIC_SPEARMAN) return spearman_impl(sc, view, data, fit, st);
    return fitness_impl(sc, view, data, metric, fit, st, cfg, tm);
}

// Records the generation into g->stream: population upload, fitness,
// tournament, result download.  Run under capture.
gp_status record_generation(gp_generation_s* g) {
    const gp_generation_params& p = g->prm;
    GP_HIP(hipMemcpyAsync(g->d_stage, g->h_stage, g->lay.bytes, hipMemcpyHostToDevice, g->stream));
    const gp_population_dev view = stage_view(g, p.node_capacity, p.const_capacity);
    Timing tm;
    tm.stamp = g->d_stamp;
    tm.launched = &g->eval_kernel;
    gp_status rc = graph_fitness(&g->sc, &view, &g->data, p.metric, g->d_fit, g->stream, &g->cfg, tm);
    if (rc != GP_OK) return rc;
    rc = tournament_impl(g->d_fit, view.len, p.n_programs, gp_metric_larger_is_better(static_cast<gp_metric>(p.metric)), p.parsimony,
                         p.tournament_size, p.n_tournaments, p.seed, 0,
                         reinterpret_cast<const uint32_t*>(g->d_stage + g->lay.gen), g->d_win, g->stream);
    if (rc != GP_OK) return rc;
    GP_HIP(hipMemcpyAsync(g->h_fit, g->d_fit, sizeof(float) * p.n_programs, hipMemcpyDeviceToHost, g->stream));
    if (p.n_tournaments > 0)
        GP_HIP(hipMemcpyAsync(g->h_win, g->d_win, sizeof(int32_t) * p.n_tournaments, hipMemcpyDeviceToHost,
                              g->stream));
    if (g->d_stamp)
        GP_HIP(hipMemcpyAsync(g->h_stamp, g->d_stamp, 2 * sizeof(uint64_t), hipMemcpyDeviceToHost, g->stream));
    return GP_OK;
}

// Puts event-record nodes right before and right after the evaluation-kernel
// node of a captured graph, so that the graph's launches record ev_a / ev_b
// around that kernel.  Returns false (graph unchanged or not) if HIP refuses;
// the caller then relies on the clock stamps.
bool insert_event_nodes(hipGraph_t graph, const void* func, hipEvent_t ev_a, hipEvent_t ev_b) {
    size_t n = 0;
    if (hipGraphGetNodes(graph, nullptr, &n) != hipSuccess || n == 0) return false;
    std::vector<hipGraphNode_t> nodes(n);
    if (hipGraphGetNodes(graph, nodes.data(), &n) != hipSuccess) return false;
    hipGraphNode_t K = nullptr;
    for (hipGraphNode_t nd : nodes) {
        hipGraphNodeType t;
        if (hipGraphNodeGetType(nd, &t) != hipSuccess || t != hipGraphNodeTypeKernel) continue;
        hipKernelNodeParams kp{};
        if (hipGraphKernelNodeGetParams(nd, &kp) != hipSuccess) continue;
        if (kp.func == func) {
            if (K) return false;   // not unique
            K = nd;
        }
    }
    if (!K) return false;
    size_t nd_in = 0, nd_out = 0;
    if (hipGraphNodeGetDependencies(K, nullptr, &nd_in) != hipSuccess) return false;
    if (hipGraphNodeGetDependentNodes(K, nullptr, &nd_out) != hipSuccess) return false;
    std::vector<hipGraphNode_t> pred(nd_in), succ(nd_out);
    if (nd_in && hipGraphNodeGetDependencies(K, pred.data(), &nd_in) != hipSuccess) return false;
    if (nd_out && hipGraphNodeGetDependentNodes(K, succ.data(), &nd_out) != hipSuccess) return false;
    std::vector<hipGraphNode_t> Ks_in(nd_in, K), Ks_out(nd_out, K);
    hipGraphNode_t A = nullptr, B = nullptr;
    if (nd_in && hipGraphRemoveDependencies(graph, pred.data(), Ks_in.data(), nd_in) != hipSuccess) return false;
    if (hipGraphAddEventRecordNode(&A, graph, pred.data(), nd_in, ev_a) != hipSuccess) return false;
    if (hipGraphAddDependencies(graph, &A, &K, 1) != hipSuccess) return false;
    if (nd_out && hipGraphRemoveDependencies(graph, Ks_out.data(), succ.data(), nd_out) != hipSuccess) return false;
    if (hipGraphAddEventRecordNode(&B, graph, &K, 1, ev_b) != hipSuccess) return false;
    std::vector<hipGraphNode_t> Bs(nd_out, B);
    if (nd_out && hipGraphAddDependencies(graph, Bs.data(), succ.data(), nd_out) != hipSuccess) return false;
    return true;
}

// ---------------------------------------------------------------------------
// The device-resident loop: two alternating populations, a fitness history,
// the generation counter in device memory.
// ---------------------------------------------------------------------------
// History entry *gen - first: the fitness of every program and the
// population's node count (prog_off[P]).
__global__ void k_evo_record(const float* __restrict__ fit, int32_t P, const uint32_t* __restrict__ gen,
                             uint32_t first, int32_t cap, float* __restrict__ hist, int64_t* __restrict__ hist_nodes,
                             const int64_t* __restrict__ prog_off) {
    const uint32_t g = *gen - first;
    if (g >= static_cast<uint32_t>(cap)) return;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < P) hist[static_cast<int64_t>(g) * P + i] = fit[i];
    if (i == 0) hist_nodes[g] = prog_off[P];
}

// End of a generation: keep the mutation status bits, advance the counter.
__global__ void k_evo_step(uint32_t* __restrict__ gen, const int64_t* __restrict__ info,
                           unsigned long long* __restrict__ sticky) {
    if (threadIdx.x == 0) {
        *sticky |= static_cast<unsigned long long>(info[2]);
        *gen += 1u;
    }
}

// Sets the counter and the status word (a fill kernel: no memset node).
__global__ void k_evo_set(uint32_t* __restrict__ gen, uint32_t g, unsigned long long* __restrict__ sticky) {
    if (threadIdx.x == 0) {
        *gen = g;
        *sticky = 0ull;
    }
}

}  // namespace

struct EvoPop {
    uint32_t* nodes = nullptr;
    int64_t* prog_off = nullptr;
    float* consts = nullptr;
    int64_t* const_off = nullptr;
    int32_t* len = nullptr;
};

struct gp_evolution_s {
    gp_evolution_params prm{};
    gp_dataset_dev data{};
    int dev = 0;
    hipStream_t stream = nullptr;
    DeviceScratch sc;
    MutateWork mw;
    EvoPop pop[2];
    int64_t node_cap = 0, const_cap = 0;
    int cur = 0;                         // the current population
    float* d_fit = nullptr;
    int32_t* d_win = nullptr;            // [2P]
    int32_t* d_ops = nullptr;
    int32_t* d_first = nullptr;
    int32_t* d_nt = nullptr;
    int64_t* d_info = nullptr;           // [4]
    uint32_t* d_gen = nullptr;
    unsigned long long* d_sticky = nullptr;
    float* d_hist = nullptr;             // [(max_generations + 1) * P]
    int64_t* d_hist_nodes = nullptr;     // [max_generations + 1]
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    hipEvent_t ev_a = nullptr, ev_b = nullptr;
    bool events = false;
    const void* eval_kernel = nullptr;
    LaunchCfg cfg{4, 0, 1};
    double tuned_ms = -1.0;
    float kernel_ms = -1.0f;
    int64_t generation = 0;              // generations run (host mirror of *d_gen)
    int64_t recorded = 0;                // history entries written
    bool captured = false;
};

namespace {

gp_population_dev evo_view(const gp_evolution_s* e, int which) {
    gp_population_dev v{};
    const EvoPop& q = e->pop[which];
    v.nodes = q.nodes;
    v.prog_off = q.prog_off;
    v.consts = q.consts;
    v.const_off = q.const_off;
    v.len = q.len;
    v.n_programs = e->prm.n_programs;
    v.total_nodes = e->node_cap;
    v.max_len = 0;
    v.total_consts = e->const_cap;
    return v;
}

void evolution_release(gp_evolution_s* e) {
    if (e->stream) (void)hipStreamSynchronize(e->stream);
    for (int k = 0; k < 2; ++k) {
        if (e->exec[k]) (void)hipGraphExecDestroy(e->exec[k]);
        if (e->graph[k]) (void)hipGraphDestroy(e->graph[k]);
        EvoPop& q = e->pop[k];
        for (void* p : {static_cast<void*>(q.nodes), static_cast<void*>(q.prog_off), static_cast<void*>(q.consts),
                        static_cast<void*>(q.const_off), static_cast<void*>(q.len)})
            if (p) (void)hipFree(p);
        q = EvoPop{};
    }
    if (e->ev_a) (void)hipEventDestroy(e->ev_a);
    if (e->ev_b) (void)hipEventDestroy(e->ev_b);
    for (void* p : {static_cast<void*>(e->d_fit), static_cast<void*>(e->d_win), static_cast<void*>(e->d_ops),
                    static_cast<void*>(e->d_first), static_cast<void*>(e->d_nt), static_cast<void*>(e->d_info),
                    static_cast<void*>(e->d_gen), static_cast<void*>(e->d_sticky), static_cast<void*>(e->d_hist),
                    static_cast<void*>(e->d_hist_nodes)})
        if (p) (void)hipFree(p);
    mutate_work_free(&e->mw);
    scratch_free(e->sc);
    if (e->stream) (void)hipStreamDestroy(e->stream);
}

// Fitness of population `which` and its history entry (plain launches or
// under capture).
gp_status evo_evaluate(gp_evolution_s* e, int which, bool timed) {
    const gp_evolution_params& p = e->prm;
    const gp_population_dev v = evo_view(e, which);
    Timing tm;
    if (timed) tm.launched = &e->eval_kernel;
    gp_status rc = graph_fitness(&e->sc, &v, &e->data, p.metric, e->d_fit, e->stream, &e->cfg, tm);
    if (rc != GP_OK) return rc;
    const int32_t P = p.n_programs;
    hipLaunchKernelGGL(k_evo_record, dim3((P + 255) / 256), dim3(256), 0, e->stream, e->d_fit, P, e->d_gen,
                       static_cast<uint32_t>(p.first_generation), p.max_generations + 1, e->d_hist,
                       e->d_hist_nodes, v.prog_off);
    GP_HIP(hipGetLastError());
    return GP_OK;
}

// One generation from population a to population a ^ 1 (recorded under capture).
gp_status record_evolution(gp_evolution_s* e, int a) {
    const gp_evolution_params& p = e->prm;
    const int32_t P = p.n_programs;
    gp_status rc = evo_evaluate(e, a, true);
    if (rc != GP_OK) return rc;
    const gp_population_dev v = evo_view(e, a);
    rc = tournament_impl(e->d_fit, v.len, P, gp_metric_larger_is_better(static_cast<gp_metric>(p.metric)),
                         p.parsimony, p.tournament_size, 2 * P, p.tournament_seed, 0, e->d_gen, e->d_win, e->stream);
    if (rc != GP_OK) return rc;
    rc = plan_launch(p.evolve, P, 0, e->d_gen, e->d_ops, e->d_first, e->d_nt, e->stream);
    if (rc != GP_OK) return rc;
    const EvoPop& b = e->pop[a ^ 1];
    const gp_population_out_dev out{b.nodes, b.prog_off, b.consts, b.const_off, b.len, e->node_cap, e->const_cap};
    rc = mutate_launch(e->mw, p.evolve, p.init, v, e->d_ops, e->d_first, e->d_win, 2 * P, P, 0, e->d_gen, out,
                       e->d_info, e->stream);
    if (rc != GP_OK) return rc;
    hipLaunchKernelGGL(k_evo_step, dim3(1), dim3(64), 0, e->stream, e->d_gen, e->d_info, e->d_sticky);
    GP_HIP(hipGetLastError());
    return GP_OK;
}

gp_status evo_capture(gp_evolution_s* e, int a, bool with_events, bool* got_events) {
    *got_events = false;
    GP_HIP(hipStreamSynchronize(e->stream));
    GP_HIP(hipStreamBeginCapture(e->stream, hipStreamCaptureModeThreadLocal));
    gp_status rc = record_evolution(e, a);
    hipGraph_t graph = nullptr;
    const hipError_t err = hipStreamEndCapture(e->stream, &graph);
    if (rc != GP_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    if (err != hipSuccess) return fail(GP_ERR_DEVICE, std::string("hipStreamEndCapture: ") + hipGetErrorString(err));
    if (with_events) {
        if (!insert_event_nodes(graph, e->eval_kernel, e->ev_a, e->ev_b)) {
            // a half-edited graph is not used: capture again without events
            (void)hipGraphDestroy(graph);
            return evo_capture(e, a, false, got_events);
        }
        *got_events = true;
    }
    e->graph[a] = graph;
    return GP_OK;
}

}  // namespace

extern "C" {

void gp_shutdown(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (size_t d = 0; d < g_dev.size(); ++d) {
        DeviceScratch& s = g_dev[d];
        if (scratch_empty(s)) continue;
        (void)hipSetDevice(static_cast<int>(d));
        (void)hipDeviceSynchronize();
        scratch_free(s);
    }
    (void)hipSetDevice(cur);
}

gp_status gp_get_launch_config(int32_t n_features, int64_t n_rows, int32_t n_programs, gp_metric metric,
                               gp_launch_config* out) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!out || n_features < 1 || n_rows < 1 || n_programs < 0)
        return fail(GP_ERR_INVALID_ARG, "gp_get_launch_config: bad arguments");
    gp_status rc = check_fitness_metric(metric, "gp_get_launch_config");
    if (rc != GP_OK) return rc;
    DeviceScratch* sc = nullptr;
    rc = arena(&sc);
    if (rc != GP_OK) return rc;
    const LaunchCfg c = pick_cfg(*sc, n_features, n_rows, n_programs, kernel_class(1, metric));
    *out = gp_launch_config{c.R, c.freg, c.tiles, c.wpb};
    return GP_OK;
}

gp_status gp_set_launch_config(const gp_launch_config* cfg) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!cfg) {
        g_forced = false;
        return GP_OK;
    }
    const LaunchCfg c{cfg->rows_per_lane, cfg->feature_regs, cfg->tiles_per_chunk, cfg->waves_per_block};
    if (!cfg_valid(c))
        return fail(GP_ERR_INVALID_ARG, "gp_set_launch_config: rows_per_lane in {1,2,4}, feature_regs in {0,2,8}, "
                                        "tiles_per_chunk in [1, 2^20], waves_per_block in {1,2,4}");
    g_forced_cfg = c;
    g_forced = true;
    return GP_OK;
}

gp_status gp_set_spearman_workset(int64_t max_bytes) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (max_bytes < 0) return fail(GP_ERR_INVALID_ARG, "gp_set_spearman_workset: max_bytes must be >= 0");
    g_spear_workset = max_bytes;
    return GP_OK;
}

gp_status gp_autotune(const gp_population_dev* pop, const gp_dataset_dev* data, gp_metric metric,
                      int32_t repeats, gp_launch_config* best, double* best_ms, void* stream) {
    std::lock_guard<std::mutex> lk(g_mu);
    gp_status rc = check_pop(pop, "gp_autotune");
    if (rc != GP_OK) return rc;
    rc = check_data(data, "gp_autotune", true);
    if (rc != GP_OK) return rc;
    rc = check_fitness_metric(metric, "gp_autotune");
    if (rc != GP_OK) return rc;
    if (pop->n_programs < 1) return fail(GP_ERR_INVALID_ARG, "gp_autotune: empty population");
    if (repeats < 1 || repeats > 100) return fail(GP_ERR_INVALID_ARG, "gp_autotune: repeats in [1, 100]");
    DeviceScratch* sc = nullptr;
    rc = arena(&sc);
    if (rc != GP_OK) return rc;
    LaunchCfg c{};
    rc = autotune_impl(sc, pop, data, metric, repeats, static_cast<hipStream_t>(stream), &c, best_ms);
    if (rc != GP_OK) return rc;
    if (best) *best = gp_launch_config{c.R, c.freg, c.tiles, c.wpb};
    return GP_OK;
}

gp_status gp_autotune_save(const char* path) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!path) return fail(GP_ERR_INVALID_ARG, "gp_autotune_save: path is NULL");
    FILE* f = std::fopen(path, "w");
    if (!f) return fail(GP_ERR_INVALID_ARG, std::string("gp_autotune_save: cannot open ") + path);
    for (const auto& kv : g_tuned) {
        const TuneKey& k = kv.first;
        const TuneVal& v = kv.second;
        std::fprintf(f,
                     "{\"arch\": \"%s\", \"n_cu\": %d, \"n_features\": %d, \"n_rows\": %lld, \"n_programs\": %d, "
                     "\"kernel\": %d, \"rows_per_lane\": %d, \"feature_regs\": %d, \"tiles_per_chunk\": %d, "
                     "\"waves_per_block\": %d, \"ms\": %.6f}\n",
                     k.arch.c_str(), k.n_cu, k.F, static_cast<long long>(k.N), k.P, k.kclass, v.cfg.R, v.cfg.freg,
                     v.cfg.tiles, v.cfg.wpb, v.ms);
    }
    const bool ok = std::fclose(f) == 0;
    return ok ? GP_OK : fail(GP_ERR_INVALID_ARG, "gp_autotune_save: write failed");
}

gp_status gp_autotune_load(const char* path) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!path) return fail(GP_ERR_INVALID_ARG, "gp_autotune_load: path is NULL");
    FILE* f = std::fopen(path, "r");
    if (!f) return fail(GP_ERR_INVALID_ARG, std::string("gp_autotune_load: cannot open ") + path);
    std::vector<std::pair<TuneKey, TuneVal>> got;
    char line[1024];
    int lineno = 0;
    bool bad = false;
    while (std::fgets(line, sizeof line, f)) {
        ++lineno;
        if (line[0] == '\n' || line[0] == '\0') continue;
        char arch[64] = {0};
        int n_cu = 0, F = 0, P = 0, kc = 0, R = 0, fr = 0, t = 0, wpb = 0;
        long long N = 0;
        double ms = 0.0;
        const int n = std::sscanf(line,
                                  "{\"arch\": \"%63[^\"]\", \"n_cu\": %d, \"n_features\": %d, \"n_rows\": %lld, "
                                  "\"n_programs\": %d, \"kernel\": %d, \"rows_per_lane\": %d, \"feature_regs\": %d, "
                                  "\"tiles_per_chunk\": %d, \"waves_per_block\": %d, \"ms\": %lf}",
                                  arch, &n_cu, &F, &N, &P, &kc, &R, &fr, &t, &wpb, &ms);
        const LaunchCfg c{R, fr, t, wpb};
        if (n != 11 || !cfg_valid(c) || F < 1 || N < 1 || P < 0 || kc < 0 || kc > 4 ||
            (c.freg > 0 && F > c.freg)) {
            bad = true;
            break;
        }
        got.push_back({TuneKey{arch, n_cu, F, static_cast<int64_t>(N), P, kc}, TuneVal{c, ms}});
    }
    std::fclose(f);
    if (bad)
        return fail(GP_ERR_INVALID_ARG,
                    std::string("gp_autotune_load: malformed entry at line ") + std::to_string(lineno));
    for (auto& kv : got) g_tuned[kv.first] = kv.second;
    return GP_OK;
}

gp_status gp_autotune_clear(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_tuned.clear();
    return GP_OK;
}

gp_status gp_profile_enable(int enable) {
    std::lock_guard<std::mutex> lk(g_mu);
    for (auto& r : g_prof_pending) {
        (void)hipEventSynchronize(r.b);
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
    }
    g_prof_pending.clear();
    g_prof_acc = gp_profile{0, 0.0, 0};
    g_prof_on = enable != 0;
    return GP_OK;
}

gp_status gp_profile_read(gp_profile* out) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!out) return fail(GP_ERR_INVALID_ARG, "gp_profile_read: out is NULL");
    for (auto& r : g_prof_pending) {
        GP_HIP(hipEventSynchronize(r.b));
        float ms = 0.0f;
        GP_HIP(hipEventElapsedTime(&ms, r.a, r.b));
        g_prof_acc.launches += 1;
        g_prof_acc.total_ms += ms;
        g_prof_acc.node_rows += r.node_rows;
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
    }
    g_prof_pending.clear();
    *out = g_prof_acc;
    return GP_OK;
}

gp_status gp_evaluate(const gp_population_dev* pop, const gp_dataset_dev* data, float* out, void* stream) {
    std::lock_guard<std::mutex> lk(g_mu);
    gp_status rc = check_pop(pop, "gp_evaluate");
    if (rc != GP_OK) return rc;
    rc = check_data(data, "gp_evaluate", false);
    if (rc != GP_OK) return rc;
    if (!out) return fail(GP_ERR_INVALID_ARG, "gp_evaluate: out is NULL");
    if (pop->n_programs == 0) return GP_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    DeviceScratch* sc;
    rc = arena(&sc);
    if (rc != GP_OK) return rc;
    PopView pv;
    CodeView cvw;
    DataView dv;
    Sched sch;
    LaunchCfg cfg;
    rc = prepare(sc, pop, data, 0, GP_METRIC_MSE, st, nullptr, &pv, &cvw, &dv, &sch, &cfg);
    if (rc != GP_OK) return rc;
    Timing tm;
    tm.profile = true;
    return launch_eval(0, GP_METRIC_MSE, cfg, sc->n_cu, pv, cvw, dv, sch, out, nullptr, st,
                       pop->total_nodes * data->n_rows, tm);
}

gp_status gp_fitness(const gp_population_dev* pop, const gp_dataset_dev* data, gp_metric metric,
                     float* fitness, void* stream) {
    std::lock_guard<std::mutex> lk(g_mu);
    gp_status rc = check_pop(pop, "gp_fitness");
    if (rc != GP_OK) return rc;
    rc = check_data(data, "gp_fitness", true);
    if (rc != GP_OK) return rc;
    if (!fitness) return fail(GP_ERR_INVALID_ARG, "gp_fitness: fitness is NULL");
    rc = check_fitness_metric(metric, "gp_fitness", true);
    if (rc != GP_OK) return rc;
    if (pop->n_programs == 0) return GP_OK;
    DeviceScratch* sc;
    rc = arena(&sc);
    if (rc != GP_OK) return rc;
    if (metric == GP_METRIC_SPEARMAN)
        return spearman_impl(sc, pop, data, fitness, static_cast<hipStream_t>(stream));
    Timing tm;
    tm.profile = true;
    return fitness_impl(sc, pop, data, metric, fitness, static_cast<hipStream_t>(stream), nullptr, tm);
}

gp_status gp_fitness_noalloc(const gp_population_dev* pop, const gp_dataset_dev* data, gp_metric metric,
                             float* fitness, void* stream) {
    std::lock_guard<std::mutex> lk(g_mu);
    gp_status rc = check_pop(pop, "gp_fitness_noalloc");
    if (rc != GP_OK) return rc;
    rc = check_data(data, "gp_fitness_noalloc", true);
    if (rc != GP_OK) return rc;
    if (!fitness) return fail(GP_ERR_INVALID_ARG, "gp_fitness_noalloc: fitness is NULL");
    rc = check_fitness_metric(metric, "gp_fitness_noalloc");
    if (rc != GP_OK) return rc;
    if (pop->n_programs == 0) return GP_OK;
    int dev = 0;
    GP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNoAllocMaxDevices)
        return fail(GP_ERR_UNSUPPORTED, "gp_fitness_noalloc: device index above the supported 64");
    NoAllocDevice& nd = g_noalloc[dev];
    if (!nd.ptr) {   // first call on this device (which is current)
        void* p = nullptr;
        GP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(GP_ERR_DEVICE, "gp_fitness_noalloc: no device address for the scratch array");
        hipDeviceProp_t prop;
        GP_HIP(hipGetDeviceProperties(&prop, dev));
        nd.n_cu = prop.multiProcessorCount;
        size_t i = 0;
        for (; i + 1 < sizeof nd.arch && prop.gcnArchName[i] && prop.gcnArchName[i] != ':'; ++i)
            nd.arch[i] = prop.gcnArchName[i];
        nd.arch[i] = 0;
        nd.ptr = static_cast<unsigned char*>(p);
    }
    DeviceScratch sc;
    sc.n_cu = nd.n_cu;
    sc.dev = dev;
    sc.arch = nd.arch;
    bool automatic = false;
    LaunchCfg cfg = pick_cfg(sc, data->n_features, data->n_rows, pop->n_programs, kernel_class(1, metric), &automatic);
    int64_t chunk = 0, n_chunks = 0;
    if ((rc = chunking(pop, data, cfg, &chunk, &n_chunks)) != GP_OK) return rc;
    // longer chunks where the partial sums of the heuristic's, beside the
    // instruction streams, do not fit the array
    while (automatic && cfg.tiles < kMostTiles &&
           noalloc_bytes(pop->n_programs, pop->total_nodes, n_chunks, metric) > kNoAllocBytes) {
        cfg.tiles = static_cast<int>(std::min<int64_t>(kMostTiles, 2 * cfg.tiles));
        if ((rc = chunking(pop, data, cfg, &chunk, &n_chunks)) != GP_OK) return rc;
    }
    if ((rc = noalloc_carve(nd.ptr, &sc, pop->n_programs, pop->total_nodes, n_chunks, metric)) != GP_OK)
        return rc;
    return fitness_impl(&sc, pop, data, metric, fitness, static_cast<hipStream_t>(stream), &cfg, Timing{});
}

gp_status gp_tournament(const float* fitness, const int32_t* len, int32_t n_programs, gp_metric metric,
                        float parsimony, int32_t tournament_size, int32_t n_tournaments, uint64_t seed,
                        uint64_t generation, int32_t* winners, void* stream) {
    if (n_programs < 1) return fail(GP_ERR_INVALID_ARG, "gp_tournament: n_programs must be >= 1");
    if (tournament_size < 1) return fail(GP_ERR_INVALID_ARG, "gp_tournament: tournament_size must be >= 1");
    if (n_tournaments < 0) return fail(GP_ERR_INVALID_ARG, "gp_tournament: n_tournaments < 0");
    if (generation > 0xffffffffull) return fail(GP_ERR_INVALID_ARG, "gp_tournament: generation above 2^32-1");
    const int larger = gp_metric_larger_is_better(metric);
    if (larger < 0) return fail(GP_ERR_INVALID_ARG, "gp_tournament: unknown metric");
    if (n_tournaments == 0) return GP_OK;
    if (!fitness || !len || !winners) return fail(GP_ERR_INVALID_ARG, "gp_tournament: NULL pointer");
    return tournament_impl(fitness, len, n_programs, larger, parsimony, tournament_size, n_tournaments, seed,
                           static_cast<uint32_t>(generation), nullptr, winners, static_cast<hipStream_t>(stream));
}

gp_status gp_generation_create(const gp_generation_params* prm, const gp_dataset_dev* data, gp_generation** out) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!prm || !out) return fail(GP_ERR_INVALID_ARG, "gp_generation_create: NULL argument");
    *out = nullptr;
    gp_status rc = check_data(data, "gp_generation_create", true);
    if (rc != GP_OK) return rc;
    rc = check_fitness_metric(prm->metric, "gp_generation_create", true);
    if (rc != GP_OK) return rc;
    if (prm->n_programs < 1 || prm->node_capacity < prm->n_programs || prm->const_capacity < 0 ||
        prm->tournament_size < 1 || prm->n_tournaments < 0 || prm->autotune < 0 || prm->time_kernel < 0)
        return fail(GP_ERR_INVALID_ARG, "gp_generation_create: bad sizes (n_programs >= 1, node_capacity >= "
                                        "n_programs, const_capacity >= 0, tournament_size >= 1, n_tournaments >= 0)");
    if (prm->node_capacity > (int64_t{1} << 32))
        return fail(GP_ERR_INVALID_ARG, "gp_generation_create: node_capacity above 2^32");
    auto* g = new (std::nothrow) gp_generation_s();
    if (!g) return fail(GP_ERR_OUT_OF_MEMORY, "gp_generation_create: out of host memory");
    g->prm = *prm;
    g->data = *data;
    g->lay = stage_layout(prm->n_programs, prm->node_capacity, prm->const_capacity);
    auto bail = [&](gp_status r) {
        generation_release(g);
        delete g;
        return r;
    };
    auto hip = [&](hipError_t e, const char* what) -> gp_status {
        return e == hipSuccess ? GP_OK : fail(GP_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
    };
    if ((rc = hip(hipGetDevice(&g->dev), "hipGetDevice")) != GP_OK) return bail(rc);
    if ((rc = scratch_init(g->sc, g->dev)) != GP_OK) return bail(rc);
    if ((rc = hip(hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking), "hipStreamCreate")) != GP_OK)
        return bail(rc);
    if ((rc = hip(hipHostMalloc(reinterpret_cast<void**>(&g->h_stage), g->lay.bytes, hipHostMallocDefault),
                  "hipHostMalloc")) != GP_OK)
        return bail(rc);
    std::memset(g->h_stage, 0, g->lay.bytes);
    if ((rc = hip(hipHostMalloc(reinterpret_cast<void**>(&g->h_fit), sizeof(float) * prm->n_programs,
                                hipHostMallocDefault), "hipHostMalloc")) != GP_OK)
        return bail(rc);
    if ((rc = hip(hipHostMalloc(reinterpret_cast<void**>(&g->h_win),
                                sizeof(int32_t) * std::max(prm->n_tournaments, 1), hipHostMallocDefault),
                  "hipHostMalloc")) != GP_OK)
        return bail(rc);
    if ((rc = hip(hipMalloc(reinterpret_cast<void**>(&g->d_stage), g->lay.bytes), "hipMalloc")) != GP_OK)
        return bail(rc == GP_ERR_DEVICE ? GP_ERR_OUT_OF_MEMORY : rc);
    if ((rc = hip(hipMalloc(reinterpret_cast<void**>(&g->d_fit), sizeof(float) * prm->n_programs), "hipMalloc")) !=
        GP_OK)
        return bail(rc);
    if ((rc = hip(hipMalloc(reinterpret_cast<void**>(&g->d_win), sizeof(int32_t) * std::max(prm->n_tournaments, 1)),
                  "hipMalloc")) != GP_OK)
        return bail(rc);
    if (prm->time_kernel) {
        if ((rc = hip(hipMalloc(reinterpret_cast<void**>(&g->d_stamp), 2 * sizeof(uint64_t)), "hipMalloc")) != GP_OK)
            return bail(rc);
        if ((rc = hip(hipHostMalloc(reinterpret_cast<void**>(&g->h_stamp), 2 * sizeof(uint64_t),
                                    hipHostMallocDefault), "hipHostMalloc")) != GP_OK)
            return bail(rc);
        if ((rc = hip(hipDeviceGetAttribute(&g->clock_khz, hipDeviceAttributeWallClockRate, g->dev),
                      "hipDeviceGetAttribute")) != GP_OK)
            return bail(rc);
        if (g->clock_khz <= 0) return bail(fail(GP_ERR_DEVICE, "gp_generation_create: no device wall clock rate"));
    }
    *out = g;
    return GP_OK;
}

gp_status gp_generation_run(gp_generation* g, const uint32_t* nodes, const int64_t* prog_off, const float* consts,
                            const int64_t* const_off, const int32_t* len, uint64_t generation, float* fitness_out,
                            int32_t* winners_out) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g || !nodes || !prog_off || !const_off || !len)
        return fail(GP_ERR_INVALID_ARG, "gp_generation_run: NULL argument");
    const gp_generation_params& p = g->prm;
    const int32_t P = p.n_programs;
    if (generation > 0xffffffffull) return fail(GP_ERR_INVALID_ARG, "gp_generation_run: generation above 2^32-1");
    if (prog_off[0] != 0 || const_off[0] != 0)
        return fail(GP_ERR_INVALID_ARG, "gp_generation_run: offsets must start at 0");
    const int64_t total_nodes = prog_off[P];
    const int64_t total_consts = const_off[P];
    if (total_nodes > p.node_capacity || total_consts > p.const_capacity)
        return fail(GP_ERR_BUFFER_TOO_SMALL, "gp_generation_run: population exceeds the capacity given at creation");
    if (total_consts > 0 && !consts) return fail(GP_ERR_INVALID_ARG, "gp_generation_run: consts is NULL");
    for (int32_t q = 0; q < P; ++q)
        if (len[q] != prog_off[q + 1] - prog_off[q] || len[q] < 1 || const_off[q + 1] < const_off[q])
            return fail(GP_ERR_INVALID_ARG, "gp_generation_run: len / offsets are inconsistent at program " +
                                                std::to_string(q));
    // the device code assumes valid programs
    int32_t bad = -1;
    gp_status rc = gp_validate_population(nodes, prog_off, const_off, P, g->data.n_features, nullptr, &bad);
    if (rc != GP_OK) return rc;
    int cur = 0;
    GP_HIP(hipGetDevice(&cur));
    if (cur != g->dev) return fail(GP_ERR_INVALID_ARG, "gp_generation_run: another device is current");
    GP_HIP(hipStreamSynchronize(g->stream));
    // stage the population in pinned memory (one upload per generation)
    const uint32_t gen32 = static_cast<uint32_t>(generation);
    std::memcpy(g->h_stage + g->lay.gen, &gen32, sizeof gen32);
    std::memcpy(g->h_stage + g->lay.len, len, sizeof(int32_t) * P);
    std::memcpy(g->h_stage + g->lay.prog_off, prog_off, sizeof(int64_t) * (P + 1));
    std::memcpy(g->h_stage + g->lay.const_off, const_off, sizeof(int64_t) * (P + 1));
    std::memcpy(g->h_stage + g->lay.nodes, nodes, sizeof(uint32_t) * total_nodes);
    if (total_consts > 0) std::memcpy(g->h_stage + g->lay.consts, consts, sizeof(float) * total_consts);
    if (!g->captured) {
        // configuration: forced, tuned on this first population, or cached/heuristic
        const bool spear = p.metric == GP_METRIC_SPEARMAN;
        g->cfg = pick_cfg(g->sc, g->data.n_features, g->data.n_rows, P, kernel_class(spear ? 0 : 1, p.metric));
        if (p.autotune && !g_forced && !spear) {
            GP_HIP(hipMemcpyAsync(g->d_stage, g->h_stage, g->lay.bytes, hipMemcpyHostToDevice, g->stream));
            const gp_population_dev cur_view = stage_view(g, total_nodes, total_consts);
            rc = autotune_impl(&g->sc, &cur_view, &g->data, p.metric, 2, g->stream, &g->cfg, &g->tuned_ms);
            if (rc != GP_OK) return rc;
        }
        // every buffer the graph touches exists before capture
        int64_t chunk = 0, n_chunks = 0;
        const gp_population_dev cap_view = stage_view(g, p.node_capacity, p.const_capacity);
        rc = chunking(&cap_view, &g->data, g->cfg, &chunk, &n_chunks);
        if (rc != GP_OK) return rc;
        const ExpandPlan xp = expand_plan(1, p.metric);
        rc = reserve(&g->sc, P, p.node_capacity, n_chunks, 1, p.metric, 0, xp.mul, xp.add);
        if (rc != GP_OK) return rc;
        if (spear) {
            // grow the Spearman buffers outside the capture (on this population)
            GP_HIP(hipMemcpyAsync(g->d_stage, g->h_stage, g->lay.bytes, hipMemcpyHostToDevice, g->stream));
            const gp_population_dev cap_full = stage_view(g, p.node_capacity, p.const_capacity);
            rc = spearman_impl(&g->sc, &cap_full, &g->data, g->d_fit, g->stream);
            if (rc != GP_OK) return rc;
        }
        GP_HIP(hipStreamSynchronize(g->stream));
        GP_HIP(hipStreamBeginCapture(g->stream, hipStreamCaptureModeThreadLocal));
        rc = record_generation(g);
        hipGraph_t graph = nullptr;
        const hipError_t e = hipStreamEndCapture(g->stream, &graph);
        if (rc != GP_OK) {
            if (graph) (void)hipGraphDestroy(graph);
            return rc;
        }
        if (e != hipSuccess) return fail(GP_ERR_DEVICE, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
        g->graph = graph;
        if (p.time_kernel) {
            GP_HIP(hipEventCreate(&g->ev_a));
            GP_HIP(hipEventCreate(&g->ev_b));
            g->events = insert_event_nodes(g->graph, g->eval_kernel, g->ev_a, g->ev_b);
            if (!g->events) {
                // a half-edited graph is not used: capture it again, stamps only
                (void)hipGraphDestroy(g->graph);
                g->graph = nullptr;
                GP_HIP(hipStreamBeginCapture(g->stream, hipStreamCaptureModeThreadLocal));
                rc = record_generation(g);
                const hipError_t e2 = hipStreamEndCapture(g->stream, &graph);
                if (rc != GP_OK) {
                    if (graph) (void)hipGraphDestroy(graph);
                    return rc;
                }
                if (e2 != hipSuccess)
                    return fail(GP_ERR_DEVICE, std::string("hipStreamEndCapture: ") + hipGetErrorString(e2));
                g->graph = graph;
            }
        }
        GP_HIP(hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0));
        g->captured = true;
    }
    GP_HIP(hipGraphLaunch(g->exec, g->stream));
    GP_HIP(hipStreamSynchronize(g->stream));
    if (p.time_kernel && p.metric != GP_METRIC_SPEARMAN) {
        g->clock_ms = static_cast<float>(static_cast<double>(g->h_stamp[1] - g->h_stamp[0]) / g->clock_khz);
        g->kernel_ms = g->clock_ms;
        if (g->events) GP_HIP(hipEventElapsedTime(&g->kernel_ms, g->ev_a, g->ev_b));
    }
    if (fitness_out) std::memcpy(fitness_out, g->h_fit, sizeof(float) * P);
    if (winners_out && p.n_tournaments > 0) std::memcpy(winners_out, g->h_win, sizeof(int32_t) * p.n_tournaments);
    return GP_OK;
}

gp_status gp_generation_info(const gp_generation* g, gp_launch_config* cfg, float* kernel_ms, float* clock_ms,
                             int32_t* timed_by_events, double* tuned_ms) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g) return fail(GP_ERR_INVALID_ARG, "gp_generation_info: NULL generation");
    if (cfg) *cfg = gp_launch_config{g->cfg.R, g->cfg.freg, g->cfg.tiles, g->cfg.wpb};
    if (kernel_ms) *kernel_ms = g->kernel_ms;
    if (clock_ms) *clock_ms = g->clock_ms;
    if (timed_by_events) *timed_by_events = g->events ? 1 : 0;
    if (tuned_ms) *tuned_ms = g->tuned_ms;
    return GP_OK;
}

void gp_generation_destroy(gp_generation* g) {
    if (!g) return;
    std::lock_guard<std::mutex> lk(g_mu);
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(g->dev);
    generation_release(g);
    (void)hipSetDevice(cur);
    delete g;
}

gp_status gp_evolution_create(const gp_evolution_params* prm, const gp_dataset_dev* data, const uint32_t* nodes,
                              const int64_t* prog_off, const float* consts, const int64_t* const_off,
                              const int32_t* len, gp_evolution** out) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!prm || !out || !nodes || !prog_off || !const_off || !len)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: NULL argument");
    *out = nullptr;
    gp_status rc = check_data(data, "gp_evolution_create", true);
    if (rc != GP_OK) return rc;
    rc = check_fitness_metric(prm->metric, "gp_evolution_create", true);
    if (rc != GP_OK) return rc;
    const int32_t P = prm->n_programs;
    if (P < 1 || P > (1 << 29) || prm->tournament_size < 1 || prm->max_generations < 1 ||
        prm->max_generations > (1 << 24) || prm->autotune < 0 || prm->time_kernel < 0)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: need 1 <= n_programs <= 2^29, tournament_size >= 1, "
                                        "1 <= max_generations <= 2^24");
    rc = mutate_check(&prm->evolve, &prm->init, P, "gp_evolution_create");
    if (rc != GP_OK) return rc;
    if (prm->first_generation + static_cast<uint64_t>(prm->max_generations) > 0xffffffffull)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: generation numbers above 2^32-1");
    if (prm->init.n_features != data->n_features)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: init.n_features must equal the dataset's");
    if (prog_off[0] != 0 || const_off[0] != 0)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: offsets must start at 0");
    int32_t longest = 1;
    for (int32_t q = 0; q < P; ++q) {
        if (len[q] != prog_off[q + 1] - prog_off[q] || len[q] < 1 || const_off[q + 1] < const_off[q])
            return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: len / offsets are inconsistent at program " +
                                                std::to_string(q));
        longest = std::max(longest, len[q]);
    }
    if (const_off[P] > 0 && !consts) return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: consts is NULL");
    rc = gp_validate_population(nodes, prog_off, const_off, P, data->n_features, nullptr, nullptr);
    if (rc != GP_OK) return rc;
    const int64_t lmax = std::max<int64_t>(prm->evolve.max_len, longest);
    const int64_t cap = static_cast<int64_t>(P) * lmax;
    if (cap > (int64_t{1} << 32))
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_create: n_programs * max length above 2^32 nodes");
    auto* e = new (std::nothrow) gp_evolution_s();
    if (!e) return fail(GP_ERR_OUT_OF_MEMORY, "gp_evolution_create: out of host memory");
    e->prm = *prm;
    e->data = *data;
    e->node_cap = cap;
    e->const_cap = cap;
    auto bail = [&](gp_status r) {
        evolution_release(e);
        delete e;
        return r;
    };
    auto hip = [&](hipError_t err, const char* what) -> gp_status {
        return err == hipSuccess ? GP_OK : fail(GP_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(err));
    };
    auto dmalloc = [&](void** ptr, size_t bytes) -> gp_status {
        return hipMalloc(ptr, std::max<size_t>(bytes, 4)) == hipSuccess
                   ? GP_OK
                   : fail(GP_ERR_OUT_OF_MEMORY, "gp_evolution_create: hipMalloc failed");
    };
    if ((rc = hip(hipGetDevice(&e->dev), "hipGetDevice")) != GP_OK) return bail(rc);
    if ((rc = scratch_init(e->sc, e->dev)) != GP_OK) return bail(rc);
    if ((rc = hip(hipStreamCreateWithFlags(&e->stream, hipStreamNonBlocking), "hipStreamCreate")) != GP_OK)
        return bail(rc);
    for (int k = 0; k < 2; ++k) {
        EvoPop& q = e->pop[k];
        if ((rc = dmalloc(reinterpret_cast<void**>(&q.nodes), sizeof(uint32_t) * cap)) != GP_OK) return bail(rc);
        if ((rc = dmalloc(reinterpret_cast<void**>(&q.consts), sizeof(float) * cap)) != GP_OK) return bail(rc);
        if ((rc = dmalloc(reinterpret_cast<void**>(&q.prog_off), sizeof(int64_t) * (P + 1))) != GP_OK) return bail(rc);
        if ((rc = dmalloc(reinterpret_cast<void**>(&q.const_off), sizeof(int64_t) * (P + 1))) != GP_OK)
            return bail(rc);
        if ((rc = dmalloc(reinterpret_cast<void**>(&q.len), sizeof(int32_t) * P)) != GP_OK) return bail(rc);
    }
    const size_t hist_n = static_cast<size_t>(prm->max_generations + 1);
    if ((rc = dmalloc(reinterpret_cast<void**>(&e->d_fit), sizeof(float) * P)) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_win), sizeof(int32_t) * 2 * P)) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_ops), sizeof(int32_t) * P)) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_first), sizeof(int32_t) * P)) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_nt), sizeof(int32_t))) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_info), sizeof(int64_t) * 4)) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_gen), sizeof(uint32_t))) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_sticky), sizeof(unsigned long long))) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_hist), sizeof(float) * hist_n * P)) != GP_OK ||
        (rc = dmalloc(reinterpret_cast<void**>(&e->d_hist_nodes), sizeof(int64_t) * hist_n)) != GP_OK)
        return bail(rc);
    if ((rc = mutate_work_reserve(&e->mw, P, prm->init)) != GP_OK) return bail(rc);
    // the initial population
    const EvoPop& q0 = e->pop[0];
    if ((rc = hip(hipMemcpy(q0.nodes, nodes, sizeof(uint32_t) * prog_off[P], hipMemcpyHostToDevice), "hipMemcpy")) !=
            GP_OK ||
        (const_off[P] > 0 &&
         (rc = hip(hipMemcpy(q0.consts, consts, sizeof(float) * const_off[P], hipMemcpyHostToDevice), "hipMemcpy")) !=
             GP_OK) ||
        (rc = hip(hipMemcpy(q0.prog_off, prog_off, sizeof(int64_t) * (P + 1), hipMemcpyHostToDevice), "hipMemcpy")) !=
            GP_OK ||
        (rc = hip(hipMemcpy(q0.const_off, const_off, sizeof(int64_t) * (P + 1), hipMemcpyHostToDevice),
                  "hipMemcpy")) != GP_OK ||
        (rc = hip(hipMemcpy(q0.len, len, sizeof(int32_t) * P, hipMemcpyHostToDevice), "hipMemcpy")) != GP_OK)
        return bail(rc);
    hipLaunchKernelGGL(k_evo_set, dim3(1), dim3(64), 0, e->stream, e->d_gen,
                       static_cast<uint32_t>(prm->first_generation), e->d_sticky);
    if ((rc = hip(hipGetLastError(), "k_evo_set")) != GP_OK) return bail(rc);
    if ((rc = hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize")) != GP_OK) return bail(rc);
    *out = e;
    return GP_OK;
}

namespace {
gp_status evo_prepare(gp_evolution_s* e) {
    if (e->captured) return GP_OK;
    const gp_evolution_params& p = e->prm;
    const int32_t P = p.n_programs;
    const bool spear = p.metric == GP_METRIC_SPEARMAN;
    e->cfg = pick_cfg(e->sc, e->data.n_features, e->data.n_rows, P, kernel_class(spear ? 0 : 1, p.metric));
    if (p.autotune && !g_forced && !spear) {
        const gp_population_dev v = evo_view(e, e->cur);
        gp_status rc = autotune_impl(&e->sc, &v, &e->data, p.metric, 2, e->stream, &e->cfg, &e->tuned_ms);
        if (rc != GP_OK) return rc;
    }
    int64_t chunk = 0, n_chunks = 0;
    const gp_population_dev v = evo_view(e, 0);
    gp_status rc = chunking(&v, &e->data, e->cfg, &chunk, &n_chunks);
    if (rc != GP_OK) return rc;
    const ExpandPlan xp = expand_plan(1, p.metric);
    rc = reserve(&e->sc, P, e->node_cap, n_chunks, 1, p.metric, 0, xp.mul, xp.add);
    if (rc != GP_OK) return rc;
    if (spear) {
        // grow the Spearman buffers outside the capture (on the current population)
        const gp_population_dev vc = evo_view(e, e->cur);
        rc = spearman_impl(&e->sc, &vc, &e->data, e->d_fit, e->stream);
        if (rc != GP_OK) return rc;
        GP_HIP(hipStreamSynchronize(e->stream));
    }
    if (p.time_kernel) {
        GP_HIP(hipEventCreate(&e->ev_a));
        GP_HIP(hipEventCreate(&e->ev_b));
    }
    // events count only if both graphs carry them
    bool events = p.time_kernel != 0;
    for (int a = 0; a < 2; ++a) {
        bool got = false;
        rc = evo_capture(e, a, p.time_kernel != 0, &got);
        if (rc != GP_OK) return rc;
        events = events && got;
        GP_HIP(hipGraphInstantiate(&e->exec[a], e->graph[a], nullptr, nullptr, 0));
    }
    e->events = events;
    e->captured = true;
    return GP_OK;
}
}  // namespace

gp_status gp_evolution_run(gp_evolution* e, int32_t n) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!e || n < 0) return fail(GP_ERR_INVALID_ARG, "gp_evolution_run: bad arguments");
    if (e->generation + n > e->prm.max_generations)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_run: beyond max_generations");
    int cur_dev = 0;
    GP_HIP(hipGetDevice(&cur_dev));
    if (cur_dev != e->dev) return fail(GP_ERR_INVALID_ARG, "gp_evolution_run: another device is current");
    gp_status rc = evo_prepare(e);
    if (rc != GP_OK) return rc;
    for (int32_t k = 0; k < n; ++k) {
        GP_HIP(hipGraphLaunch(e->exec[e->cur], e->stream));
        e->cur ^= 1;
    }
    GP_HIP(hipStreamSynchronize(e->stream));
    e->generation += n;
    e->recorded = std::max(e->recorded, e->generation);
    unsigned long long sticky = 0;
    GP_HIP(hipMemcpy(&sticky, e->d_sticky, sizeof sticky, hipMemcpyDeviceToHost));
    if (n > 0 && e->events) GP_HIP(hipEventElapsedTime(&e->kernel_ms, e->ev_a, e->ev_b));
    if (sticky)
        return fail(GP_ERR_DEVICE, "gp_evolution_run: mutation status bits " + std::to_string(sticky) +
                                       " (1 capacity, 2 index out of range)");
    return GP_OK;
}

gp_status gp_evolution_evaluate(gp_evolution* e) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!e) return fail(GP_ERR_INVALID_ARG, "gp_evolution_evaluate: NULL");
    if (e->generation > e->prm.max_generations)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_evaluate: beyond max_generations");
    gp_status rc = evo_prepare(e);
    if (rc != GP_OK) return rc;
    rc = evo_evaluate(e, e->cur, false);
    if (rc != GP_OK) return rc;
    GP_HIP(hipStreamSynchronize(e->stream));
    e->recorded = std::max(e->recorded, e->generation + 1);
    return GP_OK;
}

gp_status gp_evolution_history(const gp_evolution* e, int32_t capacity, int32_t* n_recorded, float* fitness_history,
                               int64_t* nodes_history) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!e || capacity < 0) return fail(GP_ERR_INVALID_ARG, "gp_evolution_history: bad arguments");
    if (n_recorded) *n_recorded = static_cast<int32_t>(e->recorded);
    const int64_t n = std::min<int64_t>(capacity, e->recorded);
    const int64_t P = e->prm.n_programs;
    GP_HIP(hipStreamSynchronize(e->stream));
    if (fitness_history && n > 0)
        GP_HIP(hipMemcpy(fitness_history, e->d_hist, sizeof(float) * n * P, hipMemcpyDeviceToHost));
    if (nodes_history && n > 0)
        GP_HIP(hipMemcpy(nodes_history, e->d_hist_nodes, sizeof(int64_t) * n, hipMemcpyDeviceToHost));
    return GP_OK;
}

gp_status gp_evolution_population(const gp_evolution* e, uint32_t* nodes, int64_t nodes_cap, int64_t* prog_off,
                                  float* consts, int64_t consts_cap, int64_t* const_off, int32_t* len,
                                  int64_t* total_nodes, int64_t* total_consts) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!e || !prog_off || !const_off || !len || !total_nodes || !total_consts)
        return fail(GP_ERR_INVALID_ARG, "gp_evolution_population: NULL argument");
    const int32_t P = e->prm.n_programs;
    const EvoPop& q = e->pop[e->cur];
    GP_HIP(hipStreamSynchronize(e->stream));
    GP_HIP(hipMemcpy(prog_off, q.prog_off, sizeof(int64_t) * (P + 1), hipMemcpyDeviceToHost));
    GP_HIP(hipMemcpy(const_off, q.const_off, sizeof(int64_t) * (P + 1), hipMemcpyDeviceToHost));
    GP_HIP(hipMemcpy(len, q.len, sizeof(int32_t) * P, hipMemcpyDeviceToHost));
    *total_nodes = prog_off[P];
    *total_consts = const_off[P];
    if (*total_nodes > nodes_cap || *total_consts > consts_cap || !nodes || (*total_consts > 0 && !consts))
        return fail(GP_ERR_BUFFER_TOO_SMALL, "gp_evolution_population: a capacity is short");
    GP_HIP(hipMemcpy(nodes, q.nodes, sizeof(uint32_t) * *total_nodes, hipMemcpyDeviceToHost));
    if (*total_consts > 0) GP_HIP(hipMemcpy(consts, q.consts, sizeof(float) * *total_consts, hipMemcpyDeviceToHost));
    return GP_OK;
}

gp_status gp_evolution_info(const gp_evolution* e, gp_launch_config* cfg, float* kernel_ms, int64_t* generation,
                            double* tuned_ms) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!e) return fail(GP_ERR_INVALID_ARG, "gp_evolution_info: NULL");
    if (cfg) *cfg = gp_launch_config{e->cfg.R, e->cfg.freg, e->cfg.tiles, e->cfg.wpb};
    if (kernel_ms) *kernel_ms = e->events ? e->kernel_ms : -1.0f;
    if (generation) *generation = e->generation;
    if (tuned_ms) *tuned_ms = e->tuned_ms;
    return GP_OK;
}

void gp_evolution_destroy(gp_evolution* e) {
    if (!e) return;
    std::lock_guard<std::mutex> lk(g_mu);
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(e->dev);
    evolution_release(e);
    (void)hipSetDevice(cur);
    delete e;
}

gp_status gp_fitness_backward(const gp_population_dev* pop, const gp_dataset_dev* data, gp_metric metric,
                              const float* grad_fitness, float* fitness_out, float* grad_consts,
                              void* stream) {
    std::lock_guard<std::mutex> lk(g_mu);
    gp_status rc = check_pop(pop, "gp_fitness_backward");
    if (rc != GP_OK) return rc;
    rc = check_data(data, "gp_fitness_backward", true);
    if (rc != GP_OK) return rc;
    rc = check_fitness_metric(metric, "gp_fitness_backward");
    if (rc != GP_OK) return rc;
    if (is_user_metric(metric))
        return fail(GP_ERR_UNSUPPORTED, "gp_fitness_backward: user losses have no derivative here");
    if (pop->n_programs == 0) return GP_OK;
    if (pop->total_consts < 0 || (pop->total_consts > 0 && (!grad_consts || !pop->consts)))
        return fail(GP_ERR_INVALID_ARG, "gp_fitness_backward: grad_consts and consts are needed");
    if (pop->max_len < 1)
        return fail(GP_ERR_INVALID_ARG, "gp_fitness_backward: max_len must bound the program lengths");
    if (pop->max_len > kMaxAdjointLen)
        return fail(GP_ERR_INVALID_ARG, "gp_fitness_backward: programs longer than 2^25 nodes are not supported");
    hipStream_t st = static_cast<hipStream_t>(stream);
    DeviceScratch* sc;
    rc = arena(&sc);
    if (rc != GP_OK) return rc;
    if (user_defined_mask() != 0u) {
        // user functions have no derivative here: look for them (this
        // waits for the stream)
        uint32_t* flag = static_cast<uint32_t*>(sc->counter) + kFlagWord;
        hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, st, flag);
        GP_HIP(hipGetLastError());
        const int64_t nb = std::min<int64_t>((pop->total_nodes + kBlock - 1) / kBlock, 4096);
        hipLaunchKernelGGL(k_find_user, dim3(static_cast<unsigned>(std::max<int64_t>(nb, 1))), dim3(kBlock), 0, st,
                           pop->nodes, pop->total_nodes, flag);
        GP_HIP(hipGetLastError());
        uint32_t found = 0u;
        GP_HIP(hipMemcpyAsync(&found, flag, sizeof found, hipMemcpyDeviceToHost, st));
        GP_HIP(hipStreamSynchronize(st));
        if (found)
            return fail(GP_ERR_UNSUPPORTED, "gp_fitness_backward: the population uses user functions, which have "
                                            "no derivative here");
    }
    PopView pv;
    CodeView cvw;
    DataView dv;
    Sched sch;
    LaunchCfg cfg;
    // the adjoint's stream (no constant folding: every constant carries its
    // own derivative); RMSE and Pearson also run the evaluation kernel first
    const bool needs_forward = metric == GP_METRIC_RMSE || metric == GP_METRIC_PEARSON;
    // programs of at most kParNodes nodes: k_adjoint, at the rows per lane of a
    // forced configuration, else of the heuristic (4: the fastest, or within 5%
    // of it, from 300 rows of 20 programs to 1M rows of 100); longer ones, by
    // their real lengths: k_adjoint_long, at a forced configuration's, else the
    // one (2 or 4) that keeps more rows in flight per CU (below).  max_len only
    // says whether there may be any.
    const bool longer = pop->max_len > kParNodes;
    const int RA = g_forced ? g_forced_cfg.R
                            : heuristic_cfg(data->n_features, data->n_rows, pop->n_programs, sc->n_cu, kernel_class(1, metric)).R;
    const int64_t nc = std::max<int64_t>(pop->total_consts, 1);
    rc = grow(reinterpret_cast<void**>(&sc->gextra), &sc->gextra_cap, static_cast<size_t>(nc), sizeof(double));
    if (rc != GP_OK) return rc;
    rc = prepare(sc, pop, data, 1, metric, st, nullptr, &pv, &cvw, &dv, &sch, &cfg, RA, needs_forward,
                 longer);
    if (rc != GP_OK) return rc;
    const int32_t P = pop->n_programs;
    const int64_t tape_max = 2 * static_cast<int64_t>(pop->max_len) + 2;   // tape entries per wavefront
    rc = grow(reinterpret_cast<void**>(&sc->stats), &sc->stats_cap, static_cast<size_t>(P) * kStats + 1,
              sizeof(double));
    if (rc != GP_OK) return rc;
    rc = grow(reinterpret_cast<void**>(&sc->gpart), &sc->gpart_cap, static_cast<size_t>(nc) * sch.n_chunks,
              sizeof(double));
    if (rc != GP_OK) return rc;
    rc = grow(reinterpret_cast<void**>(&sc->fit_tmp), &sc->fit_tmp_cap, static_cast<size_t>(P), sizeof(float));
    if (rc != GP_OK) return rc;
    double* wsum = sc->stats + static_cast<size_t>(P) * kStats;
    const int has_w = data->w != nullptr;
    const int ys_blocks = (sch.n_chunks + (kBlock / kWave) - 1) / (kBlock / kWave);
    hipLaunchKernelGGL(k_ystats, dim3(ys_blocks), dim3(kBlock), 0, st, dv, sch.chunk, sch.n_chunks, sc->ystat);
    GP_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_wsum, dim3(1), dim3(kWave), 0, st, sc->ystat, sch.n_chunks, has_w, data->n_rows, wsum);
    GP_HIP(hipGetLastError());
    const int fblocks = (P + (kBlock / kWave) - 1) / (kBlock / kWave);
    float* fit = fitness_out ? fitness_out : sc->fit_tmp;
    if (needs_forward) {
        rc = launch_eval(1, metric, cfg, sc->n_cu, pv, cvw, dv, sch, nullptr, sc->part, st,
                         pop->total_nodes * data->n_rows, Timing{});
        if (rc != GP_OK) return rc;
        if (metric == GP_METRIC_RMSE)
            hipLaunchKernelGGL(k_finalize<GP_METRIC_RMSE>, dim3(fblocks), dim3(kBlock), 0, st, sc->part, sc->ystat,
                               sch.n_chunks, P, data->n_rows, has_w, fit, sc->stats);
        else
            hipLaunchKernelGGL(k_finalize<GP_METRIC_PEARSON>, dim3(fblocks), dim3(kBlock), 0, st, sc->part,
                               sc->ystat, sch.n_chunks, P, data->n_rows, has_w, fit, sc->stats);
        GP_HIP(hipGetLastError());
    }
    auto occ = [](const void* k) {
        int n = 0;
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, kAdjWaves * kWave, 0);
        return n;
    };
    double* lossp = needs_forward ? nullptr : sc->part;
    // `tape_floats` of the tape area per wavefront; `area` in the unit the
    // kernel takes its size in; counter set `set`
    auto go = [&](auto kernel, int set, size_t lds, int64_t tape_floats, auto* tape, int64_t area) -> gp_status {
        int per_cu = 0;
        GP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kAdjWaves * kWave, lds));
        per_cu = std::max(per_cu, 1);
        int64_t blocks = std::min<int64_t>(static_cast<int64_t>(per_cu) * sc->n_cu,
                                           (sch.n_items + kAdjWaves - 1) / kAdjWaves);
        blocks = std::max<int64_t>(blocks, 1);
        gp_status r2 = grow(reinterpret_cast<void**>(&sc->tape), &sc->tape_cap,
                            static_cast<size_t>(blocks) * kAdjWaves * static_cast<size_t>(tape_floats), sizeof(float));
        if (r2 != GP_OK) return r2;
        Sched sl = sch;
        sl.counter += set * kCounterSet;
        sl.batch = 1;
        sl.blocks = static_cast<int32_t>(blocks);
        sl.wpb = kAdjWaves;
        using Tape = std::remove_pointer_t<decltype(tape)>;
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kAdjWaves * kWave), lds, st, pv, cvw, dv, sl,
                           needs_forward ? sc->stats : nullptr, wsum, grad_fitness, lossp, sc->gpart, sc->gextra,
                           reinterpret_cast<Tape*>(sc->tape), area);
        GP_HIP(hipGetLastError());
        return GP_OK;
    };
    // k_adjoint: tape entries are at most one per unary function and two per
    // binary one, of which there are fewer than half the nodes
    const int64_t entries = std::min<int64_t>(pop->max_len, kParNodes) + 2;
    auto go_short = [&](auto kernel, size_t lds_wave, int64_t bytes) {
        return go(kernel, 1, sizeof(MathTabsLds) + kAdjWaves * lds_wave, bytes / 4, static_cast<unsigned char*>(nullptr), bytes);
    };
    auto go_long = [&](auto kernel, int64_t floats) {
        return go(kernel, 2, size_t{0}, floats, static_cast<float*>(nullptr), floats);
    };
#define GP_ADJ_SHORT(RR) go_short(k_adjoint<RR, M>, adjoint_lds_wave<RR>(), adjoint_area<RR>(entries))
#define GP_ADJ_LONG(RR) go_long(k_adjoint_long<RR, M>, adjoint_wave_floats<RR>(tape_max))
    auto adjoints = [&](auto metric_c) -> gp_status {
        constexpr int M = decltype(metric_c)::value;
        if (longer) {
            const int RL = g_forced ? RA
                           : 4 * occ(reinterpret_cast<const void*>(k_adjoint_long<4, M>)) >
                                   2 * occ(reinterpret_cast<const void*>(k_adjoint_long<2, M>))
                               ? 4
                               : 2;
            const gp_status r2 = RL == 1 ? GP_ADJ_LONG(1) : RL == 2 ? GP_ADJ_LONG(2) : GP_ADJ_LONG(4);
            if (r2 != GP_OK) return r2;
        }
        return RA == 1 ? GP_ADJ_SHORT(1) : RA == 2 ? GP_ADJ_SHORT(2) : GP_ADJ_SHORT(4);
    };
#undef GP_ADJ_LONG
#undef GP_ADJ_SHORT
    switch (metric) {
    case GP_METRIC_MAE: rc = adjoints(std::integral_constant<int, GP_METRIC_MAE>{}); break;
    case GP_METRIC_MSE: rc = adjoints(std::integral_constant<int, GP_METRIC_MSE>{}); break;
    case GP_METRIC_RMSE: rc = adjoints(std::integral_constant<int, GP_METRIC_RMSE>{}); break;
    case GP_METRIC_LOGLOSS: rc = adjoints(std::integral_constant<int, GP_METRIC_LOGLOSS>{}); break;
    default: rc = adjoints(std::integral_constant<int, GP_METRIC_PEARSON>{}); break;
    }
    if (rc != GP_OK) return rc;
    if (!needs_forward && fitness_out) {
        if (metric == GP_METRIC_MAE)
            hipLaunchKernelGGL(k_finalize<GP_METRIC_MAE>, dim3(fblocks), dim3(kBlock), 0, st, sc->part, sc->ystat,
                               sch.n_chunks, P, data->n_rows, has_w, fitness_out, nullptr);
        else if (metric == GP_METRIC_MSE)
            hipLaunchKernelGGL(k_finalize<GP_METRIC_MSE>, dim3(fblocks), dim3(kBlock), 0, st, sc->part, sc->ystat,
                               sch.n_chunks, P, data->n_rows, has_w, fitness_out, nullptr);
        else
            hipLaunchKernelGGL(k_finalize<GP_METRIC_LOGLOSS>, dim3(fblocks), dim3(kBlock), 0, st, sc->part,
                               sc->ystat, sch.n_chunks, P, data->n_rows, has_w, fitness_out, nullptr);
        GP_HIP(hipGetLastError());
    }
    if (pop->total_consts > 0) {
        hipLaunchKernelGGL(k_finalize_grad, dim3(fblocks), dim3(kBlock), 0, st, sc->gpart, sc->gextra,
                           pop->const_off, P, sch.n_chunks, grad_consts);
        GP_HIP(hipGetLastError());
    }
    return GP_OK;
}

}  // extern "C"
