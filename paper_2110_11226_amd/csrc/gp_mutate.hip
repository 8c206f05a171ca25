// gp_mutate.hip -- the genetic operations of a generation on the device, a
// wavefront per offspring (a lane per subtree-mutation donor), with the draws,
// choices and output layout of the host gp_mutate (so the two agree bit for
// bit).
//
// Sec. II-A lists the operations (crossover, subtree, hoist and point
// mutation, reproduction) and Sec. III-C2 gives hoisted crossover; the paper
// applies them on the CPU, which costs a host round trip per generation.
// Here a generation's offspring come from a short pipeline on one stream:
//   k_plan          the operation of every offspring (draw 0 of stream 2)
//                   and where its tournaments start (a block scan);
//   k_donor         every subtree-mutation donor (the initialisation method on
//                   stream 3), each in a place of the largest donor's size;
//   k_child<0>      every offspring's splice, length and constant count;
//   k_scan2         offspring offsets (nodes and constants), totals;
//   k_child<1>      the offspring, constants renumbered in prefix order.
// Every launch has a fixed shape, so a generation can be captured in a graph.
// The generation number may be read from device memory, so one captured
// graph serves every generation.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "gp_internal.h"

namespace gp {
namespace {

constexpr int kMutBlock = 64;     // one wave per block
constexpr int kScanBlock = 1024;
constexpr int kChildBlock = 256;   // four offspring, a wavefront each
constexpr int64_t kSpreadLanes = int64_t{1} << 15;   // lanes of half a wavefront per SIMD
constexpr int kPendMax = 32;      // pending depths of a tree walk (<= max depth + 1)

// Counter-based draws of one offspring: words of Philox4x32-10 with counter
// (block, item, generation, tag), consumed in order (the host's Draws).
struct DevDraws {
    uint64_t seed;
    uint32_t item, gen, tag, n;
    uint32_t w0, w1, w2, w3;
    __device__ DevDraws(uint64_t s, uint32_t i, uint32_t g, uint32_t t)
        : seed(s), item(i), gen(g), tag(t), n(0), w0(0), w1(0), w2(0), w3(0) {}
    __device__ uint32_t next() {
        const uint32_t k = n & 3u;
        if (k == 0u) {
            const Philox4 b = philox4x32_10(n >> 2, item, gen, tag, seed);
            w0 = b.v[0];
            w1 = b.v[1];
            w2 = b.v[2];
            w3 = b.v[3];
        }
        ++n;
        return k == 0u ? w0 : (k == 1u ? w1 : (k == 2u ? w2 : w3));
    }
};

// The initialisation settings the generators and point mutation read, with
// the enabled functions in opcode order (all, unary, binary).
struct InitDev {
    int32_t n_features, method, min_depth, max_depth, min_len, max_len, max_consts;
    int32_t consts_enabled;
    float const_lo, const_hi;
    int32_t n_all, n_un, n_bin;
    uint8_t all[GP_OP_LIMIT], un[GP_OP_LIMIT], bin[GP_OP_LIMIT];
};

struct EvolveDev {
    float th[4];          // float32 running sums of the operation probabilities
    float p_point_replace;
    int32_t max_len;
    uint64_t seed;
};

// A read-only population: program p is nodes[off[p] .. off[p+1]), constants
// consts[coff[p] ..).
struct ProgSet {
    const uint32_t* nodes;
    const int64_t* off;
    const float* consts;
    const int64_t* coff;
    int32_t n;
};

// The donors: offspring i's at i * bound (where it has one).
struct DonorSet {
    const uint32_t* nodes;
    const float* consts;
    const int64_t* len;
    int64_t bound;
};

__device__ __forceinline__ uint32_t resolve_gen(uint32_t gen, const uint32_t* d_gen) {
    return d_gen ? *d_gen : gen;
}

// The function tables, copied to LDS once per block so that a drawn index
// reads them without local-memory indexing.
struct FnLds {
    uint8_t all[GP_OP_LIMIT], un[GP_OP_LIMIT], bin[GP_OP_LIMIT];
};

__device__ __forceinline__ void load_fns(FnLds& f, const InitDev& in) {
    for (int i = threadIdx.x; i < GP_OP_LIMIT; i += blockDim.x) {
        f.all[i] = in.all[i];
        f.un[i] = in.un[i];
        f.bin[i] = in.bin[i];
    }
    __syncthreads();
}

__device__ __forceinline__ bool const_available(const InitDev& in, int used) {
    return in.consts_enabled && (in.max_consts <= 0 || used < in.max_consts);
}

__device__ __forceinline__ float draw_const(const InitDev& in, DevDraws& dr) {
    const float u = unit(dr.next());
    const float span = in.const_hi - in.const_lo;
    const float scaled = span * u;
    return in.const_lo + scaled;
}

// ---------------------------------------------------------------------------
// Program generation by the initialisation method (Sec. II-A), as the host's
// Gen::program, with the nodes to nodes[0..) and the constants, numbered in the
// order they are drawn, to consts[0..) (an offspring numbers its own afresh).
// ---------------------------------------------------------------------------
__device__ void gen_tree(const InitDev& in, const FnLds& f, DevDraws& dr, int target, bool full, int8_t* pend,
                         uint32_t* nodes, float* consts, int64_t* n_nodes) {
    int np = 1;
    pend[0] = 0;
    int used = 0;
    int64_t pos = 0;
    const int nf = in.n_features;
    while (np > 0) {
        const int depth = pend[--np];
        const int n_term = nf + (const_available(in, used) ? 1 : 0);
        int pick;
        bool func;
        if (depth == target) {
            func = false;
            pick = static_cast<int>(below(dr.next(), static_cast<uint32_t>(n_term)));
        } else if (depth == 0 || full) {
            func = true;
            pick = static_cast<int>(below(dr.next(), static_cast<uint32_t>(in.n_all)));
        } else {
            const int nall = in.n_all + n_term;
            pick = static_cast<int>(below(dr.next(), static_cast<uint32_t>(nall)));
            func = pick < in.n_all;
            if (!func) pick -= in.n_all;
        }
        if (func) {
            const uint32_t op = f.all[pick];
            nodes[pos] = GP_NODE(op, 0);
            const int a = arity(op);
            for (int k = 0; k < a && np < kPendMax; ++k) pend[np++] = static_cast<int8_t>(depth + 1);
        } else if (pick < nf) {
            nodes[pos] = GP_NODE(GP_OP_VAR, pick);
        } else {
            nodes[pos] = GP_NODE(GP_OP_CONST, used);
            consts[used] = draw_const(in, dr);
            ++used;
        }
        ++pos;
    }
    *n_nodes = pos;
}

__device__ void gen_exact(const InitDev& in, const FnLds& f, DevDraws& dr, uint32_t* nodes, float* consts,
                          int64_t* n_nodes) {
    uint32_t L = static_cast<uint32_t>(in.min_len) +
                 below(dr.next(), static_cast<uint32_t>(in.max_len - in.min_len + 1));
    const bool no_unary = in.n_un == 0;
    if (no_unary && (L % 2u) == 0u)
        L = (L - 1 >= static_cast<uint32_t>(in.min_len) && L > 1) ? L - 1 : L + 1;
    int h = 0;
    int64_t nc = 0;
    const int nf = in.n_features;
    for (int i = static_cast<int>(L) - 1; i >= 0; --i) {
        const int n_term = nf + (const_available(in, static_cast<int>(nc)) ? 1 : 0);
        bool t_ok = h + 1 <= GP_MAX_STACK && h <= i;
        const bool u_ok = !no_unary && h >= 1 && h - 1 <= i;
        bool b_ok = in.n_bin > 0 && h >= 2 && h - 2 <= i;
        if (no_unary) {
            if (t_ok && ((h + i) & 1)) t_ok = false;
            if (b_ok && ((h - 2 + i) & 1)) b_ok = false;
        }
        const int nt = t_ok ? n_term : 0;
        const int nu = u_ok ? in.n_un : 0;
        const int nb = b_ok ? in.n_bin : 0;
        int pick = static_cast<int>(below(dr.next(), static_cast<uint32_t>(nt + nu + nb)));
        if (pick < nt) {
            if (pick < nf) {
                nodes[i] = GP_NODE(GP_OP_VAR, pick);
            } else {
                nodes[i] = GP_NODE(GP_OP_CONST, static_cast<uint32_t>(nc));
                consts[nc] = draw_const(in, dr);
                ++nc;
            }
            ++h;
        } else if ((pick -= nt) < nu) {
            nodes[i] = GP_NODE(f.un[pick], 0);
        } else {
            nodes[i] = GP_NODE(f.bin[pick - nu], 0);
            --h;
        }
    }
    *n_nodes = L;
}

__device__ void gen_program(const InitDev& in, const FnLds& f, DevDraws& dr, int8_t* pend, uint32_t* nodes,
                            float* consts, int64_t* n_nodes) {
    if (in.method == GP_INIT_EXACT_LEN) {
        gen_exact(in, f, dr, nodes, consts, n_nodes);
        return;
    }
    bool full;
    if (in.method == GP_INIT_RHH) full = !(unit(dr.next()) < 0.5f);
    else full = in.method == GP_INIT_FULL;
    const int depth = in.min_depth +
                      static_cast<int>(below(dr.next(), static_cast<uint32_t>(in.max_depth - in.min_depth + 1)));
    gen_tree(in, f, dr, depth, full, pend, nodes, consts, n_nodes);
}

// ---------------------------------------------------------------------------
// k_plan: one block.  ops[i] from draw 0 of (seed, i, generation, stream 2);
// first[i] = sum over j < i of (2 for crossover, else 1); *n_tournaments =
// the total.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kScanBlock) void k_plan(EvolveDev ev, int32_t n, uint32_t gen, const uint32_t* d_gen,
                                                     int32_t* __restrict__ ops, int32_t* __restrict__ first,
                                                     int32_t* __restrict__ n_tournaments) {
    __shared__ int32_t wsum[kScanBlock / 64];
    __shared__ int32_t carry_s;
    const uint32_t g = resolve_gen(gen, d_gen);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int32_t base = 0; base < n; base += kScanBlock) {
        const int32_t i = base + static_cast<int32_t>(threadIdx.x);
        int32_t t = 0;
        if (i < n) {
            DevDraws dr(ev.seed, static_cast<uint32_t>(i), g, kStreamMutation);
            const float u = unit(dr.next());
            int32_t op = GP_GENOP_REPRODUCTION;
            for (int k = 3; k >= 0; --k)
                if (u < ev.th[k]) op = k;
            ops[i] = op;
            t = op == GP_GENOP_CROSSOVER ? 2 : 1;
        }
        // inclusive scan within the wave, then across the block's waves
        int32_t v = t;
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t o = __shfl_up(v, d, 64);
            if (lane >= d) v += o;
        }
        if (lane == 63) wsum[wid] = v;
        __syncthreads();
        int32_t before = carry_s;
        for (int k = 0; k < wid; ++k) before += wsum[k];
        if (i < n) first[i] = before + v - t;
        __syncthreads();
        if (threadIdx.x == kScanBlock - 1) carry_s = before + v;
        __syncthreads();
    }
    if (threadIdx.x == 0) *n_tournaments = carry_s;
}

// ---------------------------------------------------------------------------
// k_scan2: one block.  out_a[i] = sum of a[j < i] (i = 0..n), likewise b;
// info[0], info[1] = the totals; a total above its capacity sets info[2].
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kScanBlock) void k_scan2(const int64_t* __restrict__ a, const int64_t* __restrict__ b,
                                                      int32_t n, int64_t* __restrict__ out_a,
                                                      int64_t* __restrict__ out_b, int64_t cap_a, int64_t cap_b,
                                                      int64_t* __restrict__ info) {
    __shared__ int64_t wa[kScanBlock / 64], wb[kScanBlock / 64];
    __shared__ int64_t ca, cb;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (threadIdx.x == 0) {
        ca = 0;
        cb = 0;
    }
    __syncthreads();
    for (int32_t base = 0; base < n; base += kScanBlock) {
        const int32_t i = base + static_cast<int32_t>(threadIdx.x);
        const int64_t ta = i < n ? a[i] : 0, tb = i < n ? b[i] : 0;
        int64_t va = ta, vb = tb;
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t oa = __shfl_up(va, d, 64);
            const int64_t ob = __shfl_up(vb, d, 64);
            if (lane >= d) {
                va += oa;
                vb += ob;
            }
        }
        if (lane == 63) {
            wa[wid] = va;
            wb[wid] = vb;
        }
        __syncthreads();
        int64_t pa = ca, pb = cb;
        for (int k = 0; k < wid; ++k) {
            pa += wa[k];
            pb += wb[k];
        }
        if (i < n) {
            out_a[i] = pa + va - ta;
            out_b[i] = pb + vb - tb;
        }
        __syncthreads();
        if (threadIdx.x == kScanBlock - 1) {
            ca = pa + va;
            cb = pb + vb;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out_a[n] = ca;
        out_b[n] = cb;
        if (info) {
            info[0] = ca;
            info[1] = cb;
            if (ca > cap_a || cb > cap_b) info[2] |= 1;
        }
    }
}

// Donors per wavefront: of its 64 lanes, those at multiples of 2^lg have an
// offspring each.  A wavefront's lanes wait for its longest donor and take each
// other's branches, so few of them do work while the offspring alone would not
// fill the chip (spread()): donors of 1,024 offspring, trees of depth 2 to 6,
// 25.6 us with 64 a wavefront, 20.8 with 4; exact lengths up to 120, 59 and 43.
__device__ __forceinline__ int32_t offspring(int lg) {
    const uint32_t at = blockIdx.x * kMutBlock + threadIdx.x;
    return (at & ((1u << lg) - 1u)) == 0u ? static_cast<int32_t>(at >> lg) : INT32_MAX;
}

// ---------------------------------------------------------------------------
// k_donor: one lane per offspring; only subtree-mutation offspring have a
// donor, of at most `bound` nodes.  Clears the pipeline's status words (a
// kernel's store, not a memset, so that a captured graph replays it).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kMutBlock) void k_donor(InitDev in, EvolveDev ev, int32_t n, int lg, uint32_t gen,
                                                     const uint32_t* d_gen, const int32_t* __restrict__ ops,
                                                     int64_t* __restrict__ dlen, uint32_t* __restrict__ dnodes,
                                                     float* __restrict__ dconsts, int64_t bound,
                                                     int64_t* __restrict__ info) {
    __shared__ FnLds f;
    __shared__ int8_t pend[kMutBlock][kPendMax];
    load_fns(f, in);
    if (blockIdx.x == 0 && threadIdx.x < 4) info[threadIdx.x] = 0;
    const int32_t i = offspring(lg);
    if (i >= n || ops[i] != GP_GENOP_SUBTREE) return;
    const uint32_t g = resolve_gen(gen, d_gen);
    DevDraws dr(ev.seed, static_cast<uint32_t>(i), g, kStreamDonor);
    int64_t nn = 0;
    gen_program(in, f, dr, pend[threadIdx.x], dnodes + i * bound, dconsts + i * bound, &nn);
    dlen[i] = nn;
}

// ---------------------------------------------------------------------------
// Splice arithmetic on read-only programs, by a whole wavefront: lane l takes
// every 64th node, and what is summed along the prefix list (1 - arity, the
// constants so far) is counted in the lanes' ballots.  All arguments and
// results are the same in every lane.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return static_cast<int>(threadIdx.x & 63u); }
__device__ __forceinline__ uint64_t lanes_below(int l) { return (uint64_t{1} << l) - 1; }

// One past the last node of the subtree rooted at s (bounded by len).
__device__ __forceinline__ int64_t subtree_end(const uint32_t* w, int64_t len, int64_t s) {
    int open = 1;
    for (int64_t c = s; c < len; c += 64) {
        const int64_t i = c + lane_id();
        const int ar = i < len ? arity(GP_NODE_OP(w[i])) : 1;
        const uint64_t leaf = __ballot(ar == 0), bin = __ballot(ar == 2);
        const uint64_t upto = lanes_below(lane_id()) | (uint64_t{1} << lane_id());
        const int here = open + __popcll(bin & upto) - __popcll(leaf & upto);
        const uint64_t done = __ballot(here == 0);
        if (done) return min(c + __builtin_ctzll(done) + 1, len);
        open += __popcll(bin) - __popcll(leaf);
    }
    return len;
}

// A segment of the right-to-left scan: the height h after w[b-1] .. w[a], and
// hmax, this lane's largest on the way.
__device__ __forceinline__ void scan_heights(const uint32_t* w, int64_t a, int64_t b, int* h, int* hmax) {
    for (int64_t c = b; c > a; c -= 64) {
        const int64_t i = c - 1 - lane_id();
        const int ar = i >= a ? arity(GP_NODE_OP(w[i])) : 1;
        const uint64_t leaf = __ballot(ar == 0), bin = __ballot(ar == 2);
        const uint64_t upto = lanes_below(lane_id()) | (uint64_t{1} << lane_id());
        *hmax = max(*hmax, *h + __popcll(leaf & upto) - __popcll(bin & upto));
        *h += __popcll(leaf) - __popcll(bin);
    }
}

// Peak height of the right-to-left scan of parent[0:s) + donor[ds:de) + parent[e:L).
__device__ __forceinline__ int splice_peak(const uint32_t* pw, int64_t L, int64_t s, int64_t e, const uint32_t* dw,
                                           int64_t ds, int64_t de) {
    int h = 0, hmax = 0;
    scan_heights(pw, e, L, &h, &hmax);
    scan_heights(dw, ds, de, &h, &hmax);
    scan_heights(pw, 0, s, &h, &hmax);
    for (int d = 32; d > 0; d >>= 1) hmax = max(hmax, __shfl_xor(hmax, d, 64));
    return hmax;
}

__device__ __forceinline__ int64_t count_consts(const uint32_t* w, int64_t a, int64_t b) {
    int64_t n = 0;
    for (int64_t c = a; c < b; c += 64) {
        const int64_t i = c + lane_id();
        n += __popcll(__ballot(i < b && GP_NODE_OP(w[i]) == GP_OP_CONST));
    }
    return n;
}

// Copies w[a:b) to out[*pos ..), constants renumbered from *slot (values from cv by
// their old slot).
__device__ __forceinline__ void copy_seg(const uint32_t* w, const float* cv, int64_t a, int64_t b, uint32_t* out,
                                         float* oc, int64_t* pos, uint32_t* slot) {
    for (int64_t c = a; c < b; c += 64) {
        const int64_t i = c + lane_id();
        uint32_t x = i < b ? w[i] : 0u;
        const bool is_const = i < b && GP_NODE_OP(x) == GP_OP_CONST;
        const uint64_t consts = __ballot(is_const);
        if (is_const) {
            const uint32_t q = *slot + static_cast<uint32_t>(__popcll(consts & lanes_below(lane_id())));
            oc[q] = cv[GP_NODE_ARG(x)];
            x = GP_NODE(GP_OP_CONST, q);
        }
        if (i < b) out[*pos + (i - a)] = x;
        *slot += static_cast<uint32_t>(__popcll(consts));
    }
    *pos += max(b - a, int64_t{0});
}

// ---------------------------------------------------------------------------
// k_child<WRITE>: one wavefront per offspring.  WRITE = false draws the splice
// (crossover / subtree: parent cut (s, e) and donor subtree (ds, de) after
// hoisting; hoist: (s, e) and (s2, e2)), stores it in plan[i] and the child's
// length and constant count; WRITE = true writes the child.  Point mutation
// re-draws in both passes.  An index out of range (operation, tournament,
// winner) sets info[2] bit 2 and yields the one-node program x0.
//
// A lane per offspring waited for memory at every node, and for the other
// operations of its wavefront: with trees of depth 2 to 6, the two passes over
// 1,024 offspring took 58 + 55 us, 11 + 12 so; over 65,536, 66 + 70 and 56 + 43.
// ---------------------------------------------------------------------------
template <bool WRITE>
__global__ __launch_bounds__(kChildBlock) void k_child(
    InitDev in, EvolveDev ev, ProgSet par, DonorSet don, int32_t n, uint32_t gen, const uint32_t* d_gen,
    const int32_t* __restrict__ ops, const int32_t* __restrict__ first, const int32_t* __restrict__ winners,
    int32_t n_winners, int4* __restrict__ plan, int64_t* __restrict__ clen, int64_t* __restrict__ cnc,
    const int64_t* __restrict__ coff, const int64_t* __restrict__ ccoff, uint32_t* __restrict__ out_nodes,
    float* __restrict__ out_consts, int32_t* __restrict__ out_len, int64_t nodes_cap, int64_t consts_cap,
    int64_t* __restrict__ info) {
    __shared__ FnLds f;
    load_fns(f, in);
    const int32_t wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int64_t at = static_cast<int64_t>(blockIdx.x) * (kChildBlock / 64) + wave;
    if (at >= n) return;
    const int32_t i = static_cast<int32_t>(at);
    const bool one = lane_id() == 0;      // the lane that writes what the wavefront has once
    if (WRITE) {
        if (coff[n] > nodes_cap || ccoff[n] > consts_cap) return;   // flagged by k_scan2
    }
    const int32_t op = ops[i];
    const int32_t need = op == GP_GENOP_CROSSOVER ? 2 : 1;
    const int32_t t0 = first[i];
    bool bad = op < 0 || op > GP_GENOP_REPRODUCTION || t0 < 0 || static_cast<int64_t>(t0) + need > n_winners;
    int32_t pa = 0, pb = 0;
    if (!bad) {
        pa = winners[t0];
        pb = need == 2 ? winners[t0 + 1] : 0;
        bad = pa < 0 || pa >= par.n || pb < 0 || pb >= par.n;
    }
    auto counts = [&](int64_t len, int64_t consts) {
        if (one) {
            clen[i] = len;
            cnc[i] = consts;
        }
    };
    if (bad) {
        if (!WRITE) {
            if (one) atomicOr(reinterpret_cast<unsigned long long*>(info + 2), 2ull);
            counts(1, 0);
        } else if (one) {
            out_nodes[coff[i]] = GP_NODE(GP_OP_VAR, 0);
            out_len[i] = 1;
        }
        return;
    }
    const uint32_t g = resolve_gen(gen, d_gen);
    DevDraws dr(ev.seed, static_cast<uint32_t>(i), g, kStreamMutation);
    (void)dr.next();   // the operation draw
    const uint32_t* pw = par.nodes + par.off[pa];
    const float* pc = par.consts + par.coff[pa];
    const int64_t L = par.off[pa + 1] - par.off[pa];
    uint32_t* on = out_nodes + (WRITE ? coff[i] : 0);
    float* oc = out_consts + (WRITE ? ccoff[i] : 0);
    int64_t pos = 0;
    uint32_t slot = 0;
    auto written = [&]() {
        if (one) out_len[i] = static_cast<int32_t>(pos);
    };

    if (op == GP_GENOP_CROSSOVER || op == GP_GENOP_SUBTREE) {
        const uint32_t* dw;
        const float* dc;
        int64_t DL;
        if (op == GP_GENOP_CROSSOVER) {
            dw = par.nodes + par.off[pb];
            dc = par.consts + par.coff[pb];
            DL = par.off[pb + 1] - par.off[pb];
        } else {
            dw = don.nodes + i * don.bound;
            dc = don.consts + i * don.bound;
            DL = don.len[i];
        }
        int64_t s, e, ds, de;
        if (!WRITE) {
            s = below(dr.next(), static_cast<uint32_t>(L));
            e = subtree_end(pw, L, s);
            ds = below(dr.next(), static_cast<uint32_t>(DL));
            de = subtree_end(dw, DL, ds);
            for (;;) {
                const int64_t clen_try = L - (e - s) + (de - ds);
                const bool fits = splice_peak(pw, L, s, e, dw, ds, de) <= GP_MAX_STACK && clen_try <= ev.max_len;
                if (fits || de - ds == 1) break;
                ds = ds + 1 + below(dr.next(), static_cast<uint32_t>(de - ds - 1));
                de = subtree_end(dw, DL, ds);
            }
            if (one)
                plan[i] = make_int4(static_cast<int>(s), static_cast<int>(e), static_cast<int>(ds), static_cast<int>(de));
            counts(L - (e - s) + (de - ds), count_consts(pw, 0, s) + count_consts(dw, ds, de) + count_consts(pw, e, L));
        } else {
            const int4 q = plan[i];
            copy_seg(pw, pc, 0, q.x, on, oc, &pos, &slot);
            copy_seg(dw, dc, q.z, q.w, on, oc, &pos, &slot);
            copy_seg(pw, pc, q.y, L, on, oc, &pos, &slot);
            written();
        }
        return;
    }
    if (op == GP_GENOP_HOIST) {
        if (!WRITE) {
            const int64_t s = below(dr.next(), static_cast<uint32_t>(L));
            const int64_t e = subtree_end(pw, L, s);
            const int64_t s2 = s + below(dr.next(), static_cast<uint32_t>(e - s));
            const int64_t e2 = subtree_end(pw, L, s2);
            if (one)
                plan[i] = make_int4(static_cast<int>(s), static_cast<int>(e), static_cast<int>(s2), static_cast<int>(e2));
            counts(L - (e - s) + (e2 - s2), count_consts(pw, 0, s) + count_consts(pw, s2, e2) + count_consts(pw, e, L));
        } else {
            const int4 q = plan[i];
            copy_seg(pw, pc, 0, q.x, on, oc, &pos, &slot);
            copy_seg(pw, pc, q.z, q.w, on, oc, &pos, &slot);
            copy_seg(pw, pc, q.y, L, on, oc, &pos, &slot);
            written();
        }
        return;
    }
    if (op == GP_GENOP_POINT) {
        // node by node (a node's draws depend on those before it), 64 at a time
        // in the lanes' registers; each lane keeps its own node's result
        int n_const = static_cast<int>(count_consts(pw, 0, L));
        const int nf = in.n_features;
        for (int64_t c = 0; c < L; c += 64) {
            const int64_t mine = c + lane_id();
            uint32_t word = mine < L ? pw[mine] : 0u;
            float value = 0.0f;
            if (mine < L && GP_NODE_OP(word) == GP_OP_CONST) value = pc[GP_NODE_ARG(word)];
            const int m = static_cast<int>(min(L - c, int64_t{64}));
            for (int j = 0; j < m; ++j) {
                if (!(unit(dr.next()) < ev.p_point_replace)) continue;
                uint32_t x = __builtin_amdgcn_readlane(word, j);
                float v = 0.0f;
                const uint32_t xop = GP_NODE_OP(x);
                const int ar = arity(xop);
                if (ar > 0) {
                    const int ns = ar == 1 ? in.n_un : in.n_bin;
                    if (ns > 0) {
                        const uint32_t k = below(dr.next(), static_cast<uint32_t>(ns));
                        x = GP_NODE(ar == 1 ? f.un[k] : f.bin[k], 0);
                    }
                } else {
                    const int others = n_const - (xop == GP_OP_CONST ? 1 : 0);
                    const int n_term = nf + (const_available(in, others) ? 1 : 0);
                    const int pick = static_cast<int>(below(dr.next(), static_cast<uint32_t>(n_term)));
                    if (pick < nf) {
                        x = GP_NODE(GP_OP_VAR, pick);
                        n_const = others;
                    } else {
                        x = GP_NODE(GP_OP_CONST, 0);
                        v = draw_const(in, dr);
                        n_const = others + 1;
                    }
                }
                if (lane_id() == j) {
                    word = x;
                    value = v;
                }
            }
            if (WRITE) {
                const bool is_const = mine < L && GP_NODE_OP(word) == GP_OP_CONST;
                const uint64_t consts = __ballot(is_const);
                if (is_const) {
                    const uint32_t q = slot + static_cast<uint32_t>(__popcll(consts & lanes_below(lane_id())));
                    oc[q] = value;
                    word = GP_NODE(GP_OP_CONST, q);
                }
                if (mine < L) on[mine] = word;
                slot += static_cast<uint32_t>(__popcll(consts));
            }
        }
        pos = L;
        if (!WRITE) counts(L, n_const);
        else written();
        return;
    }
    // reproduction
    if (!WRITE) {
        counts(L, count_consts(pw, 0, L));
    } else {
        copy_seg(pw, pc, 0, L, on, oc, &pos, &slot);
        written();
    }
}

// Programs longer than the donor capacity cannot come from these settings:
// the largest donor the initialisation method can produce.
int64_t donor_bound(const gp_init_params& in) {
    if (in.method == GP_INIT_EXACT_LEN) return static_cast<int64_t>(in.max_len) + 1;
    bool has_binary = false;
    for (uint32_t op = GP_OP_ADD; op < GP_OP_LIMIT; ++op)
        has_binary |= arity(op) == 2 && ((in.function_mask >> op) & 1u);
    return has_binary ? (int64_t{1} << (in.max_depth + 1)) - 1 : in.max_depth + 1;
}

// The donors' spread over wavefronts (offspring()): one to a wavefront up to 511
// offspring, all 64 from 16,384 on (there 16 to a wavefront took 35 us against
// 37 for trees, 75 against 64 for exact lengths).
int spread(int64_t n) {
    int lg = 0;
    while (lg < 6 && (n << (lg + 1)) < kSpreadLanes) ++lg;
    return lg;
}

InitDev to_dev(const gp_init_params& p) {
    InitDev d{};
    d.n_features = p.n_features;
    d.method = p.method;
    d.min_depth = p.min_depth;
    d.max_depth = p.max_depth;
    d.min_len = p.min_len;
    d.max_len = p.max_len;
    d.max_consts = p.max_consts;
    d.consts_enabled = !(p.const_lo > p.const_hi);
    d.const_lo = p.const_lo;
    d.const_hi = p.const_hi;
    for (uint32_t op = GP_OP_ADD; op < GP_OP_LIMIT; ++op) {
        if (!(p.function_mask & (1u << op)) || arity(op) < 1) continue;
        d.all[d.n_all++] = static_cast<uint8_t>(op);
        if (arity(op) == 1) d.un[d.n_un++] = static_cast<uint8_t>(op);
        else d.bin[d.n_bin++] = static_cast<uint8_t>(op);
    }
    return d;
}

EvolveDev to_dev(const gp_evolve_params& e) {
    EvolveDev d{};
    d.th[0] = e.p_crossover;
    d.th[1] = d.th[0] + e.p_subtree;
    d.th[2] = d.th[1] + e.p_hoist;
    d.th[3] = d.th[2] + e.p_point;
    d.p_point_replace = e.p_point_replace;
    d.max_len = e.max_len;
    d.seed = e.seed;
    return d;
}

template <typename T>
gp_status grow_buf(T** p, int64_t* cap, int64_t need) {
    if (*cap >= need && *p) return GP_OK;
    if (*p) {
        GP_HIP(hipDeviceSynchronize());
        GP_HIP(hipFree(*p));
        *p = nullptr;
        *cap = 0;
    }
    const int64_t n = std::max<int64_t>(need, 1);
    if (hipMalloc(reinterpret_cast<void**>(p), sizeof(T) * static_cast<size_t>(n)) != hipSuccess) {
        *p = nullptr;
        return fail(GP_ERR_OUT_OF_MEMORY, "device mutation: hipMalloc failed");
    }
    *cap = n;
    return GP_OK;
}

}  // namespace

gp_status mutate_check(const gp_evolve_params* ev, const gp_init_params* in, int32_t n_offspring, const char* who) {
    if (!ev || !in) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": params are NULL");
    const float ps[5] = {ev->p_crossover, ev->p_subtree, ev->p_hoist, ev->p_point, ev->p_point_replace};
    for (float v : ps)
        if (!(v >= 0.0f && v <= 1.0f))
            return fail(GP_ERR_INVALID_ARG, std::string(who) + ": probabilities must lie in [0, 1]");
    const EvolveDev e = to_dev(*ev);
    if (!(e.th[3] <= 1.0f)) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": operation probabilities sum above 1");
    if (ev->max_len < 1) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": max_len must be >= 1");
    if (n_offspring < 0) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": n_offspring < 0");
    if (in->n_features < 1) return fail(GP_ERR_INVALID_ARG, std::string(who) + ": n_features >= 1");
    if (in->function_mask == 0 || (in->function_mask & ~allowed_function_mask()))
        return fail(GP_ERR_INVALID_ARG, std::string(who) + ": function_mask must select functions (bits 2..22, "
                                                           "or 24..31 once defined) only");
    if (in->method == GP_INIT_EXACT_LEN) {
        if (in->min_len < 1 || in->max_len < in->min_len || in->max_len > (1 << 20))
            return fail(GP_ERR_INVALID_ARG, std::string(who) + ": need 1 <= min_len <= max_len <= 2^20");
        if (donor_bound(*in) > 1 && in->max_len > 1) {
            bool has_binary = false;
            for (uint32_t op = GP_OP_ADD; op < GP_OP_LIMIT; ++op)
                has_binary |= arity(op) == 2 && ((in->function_mask >> op) & 1u);
            if (!has_binary)
                return fail(GP_ERR_INVALID_ARG, std::string(who) + ": exact lengths above 1 need a binary function");
        }
    } else if (in->method >= GP_INIT_RHH && in->method <= GP_INIT_GROW) {
        if (in->min_depth < 0 || in->max_depth < in->min_depth || in->max_depth > GP_MAX_STACK - 1)
            return fail(GP_ERR_INVALID_ARG, std::string(who) + ": need 0 <= min_depth <= max_depth <= 19");
    } else {
        return fail(GP_ERR_INVALID_ARG, std::string(who) + ": unknown method");
    }
    return GP_OK;
}

gp_status mutate_work_reserve(MutateWork* w, int32_t n_offspring, const gp_init_params& in) {
    const int64_t n1 = static_cast<int64_t>(n_offspring) + 1;
    const int64_t dcap = std::max<int64_t>(donor_bound(in) * std::max<int32_t>(n_offspring, 1), 1);
    if (dcap > (int64_t{1} << 25))
        return fail(GP_ERR_INVALID_ARG, "device mutation: donors of these initialisation settings could need more "
                                        "than 2^25 nodes; lower max_depth / max_len or mutate on the host");
    gp_status rc;
    if ((rc = grow_buf(&w->dlen, &w->dlen_cap, n1)) != GP_OK) return rc;
    if ((rc = grow_buf(&w->clen, &w->clen_cap, n1)) != GP_OK) return rc;
    if ((rc = grow_buf(&w->cnc, &w->cnc_cap, n1)) != GP_OK) return rc;
    if ((rc = grow_buf(&w->plan, &w->plan_cap, n1)) != GP_OK) return rc;
    if ((rc = grow_buf(&w->dnodes, &w->dnodes_cap, dcap)) != GP_OK) return rc;
    if ((rc = grow_buf(&w->dconsts, &w->dconsts_cap, dcap)) != GP_OK) return rc;
    w->donor_cap = std::min(w->dnodes_cap, w->dconsts_cap);
    return GP_OK;
}

void mutate_work_free(MutateWork* w) {
    for (void* p : {static_cast<void*>(w->dlen), static_cast<void*>(w->clen), static_cast<void*>(w->cnc),
                    static_cast<void*>(w->plan), static_cast<void*>(w->dnodes), static_cast<void*>(w->dconsts)})
        if (p) (void)hipFree(p);
    *w = MutateWork{};
}

gp_status plan_launch(const gp_evolve_params& ev, int32_t n_offspring, uint32_t gen, const uint32_t* d_gen,
                      int32_t* ops, int32_t* first, int32_t* n_tournaments, hipStream_t s) {
    hipLaunchKernelGGL(k_plan, dim3(1), dim3(kScanBlock), 0, s, to_dev(ev), n_offspring, gen, d_gen, ops, first,
                       n_tournaments);
    GP_HIP(hipGetLastError());
    return GP_OK;
}

gp_status mutate_launch(MutateWork& w, const gp_evolve_params& evp, const gp_init_params& inp,
                        const gp_population_dev& par, const int32_t* ops, const int32_t* first, const int32_t* winners,
                        int32_t n_winners, int32_t n_offspring, uint32_t gen, const uint32_t* d_gen,
                        const gp_population_out_dev& out, int64_t* info, hipStream_t s) {
    const InitDev in = to_dev(inp);
    const EvolveDev ev = to_dev(evp);
    const int32_t n = n_offspring;
    const int64_t bound = donor_bound(inp);
    if (bound * n > w.donor_cap) return fail(GP_ERR_BUFFER_TOO_SMALL, "device mutation: the donors' buffers are too small");
    const int lg = spread(n);
    const dim3 grid(static_cast<unsigned>((std::max<int64_t>(static_cast<int64_t>(n) << lg, 1) + kMutBlock - 1) / kMutBlock));
    const dim3 blk(kMutBlock);
    hipLaunchKernelGGL(k_donor, grid, blk, 0, s, in, ev, n, lg, gen, d_gen, ops, w.dlen, w.dnodes, w.dconsts, bound, info);
    GP_HIP(hipGetLastError());
    if (n == 0) {
        hipLaunchKernelGGL(k_scan2, dim3(1), dim3(kScanBlock), 0, s, w.clen, w.cnc, 0, out.prog_off, out.const_off,
                           out.node_capacity, out.const_capacity, info);
        GP_HIP(hipGetLastError());
        return GP_OK;
    }
    const ProgSet p{par.nodes, par.prog_off, par.consts, par.const_off, par.n_programs};
    const DonorSet d{w.dnodes, w.dconsts, w.dlen, bound};
    const dim3 cgrid(static_cast<unsigned>((static_cast<int64_t>(n) + kChildBlock / 64 - 1) / (kChildBlock / 64)));
    const dim3 cblk(kChildBlock);
    hipLaunchKernelGGL(k_child<false>, cgrid, cblk, 0, s, in, ev, p, d, n, gen, d_gen, ops, first, winners, n_winners,
                       w.plan, w.clen, w.cnc, static_cast<const int64_t*>(nullptr),
                       static_cast<const int64_t*>(nullptr), out.nodes, out.consts, out.len, out.node_capacity,
                       out.const_capacity, info);
    GP_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_scan2, dim3(1), dim3(kScanBlock), 0, s, w.clen, w.cnc, n, out.prog_off, out.const_off,
                       out.node_capacity, out.const_capacity, info);
    GP_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_child<true>, cgrid, cblk, 0, s, in, ev, p, d, n, gen, d_gen, ops, first, winners, n_winners,
                       w.plan, w.clen, w.cnc, out.prog_off, out.const_off, out.nodes, out.consts, out.len,
                       out.node_capacity, out.const_capacity, info);
    GP_HIP(hipGetLastError());
    return GP_OK;
}

}  // namespace gp

namespace {
std::mutex g_mut_mu;
std::vector<gp::MutateWork> g_mut_work;   // per device
}  // namespace

extern "C" {

gp_status gp_plan_generation_device(const gp_evolve_params* params, int32_t n_offspring, uint64_t generation,
                                    int32_t* ops, int32_t* first_tournament, int32_t* n_tournaments, void* stream) {
    using namespace gp;
    if (!params) return fail(GP_ERR_INVALID_ARG, "gp_plan_generation_device: params is NULL");
    gp_init_params dummy{};
    dummy.n_features = 1;
    dummy.method = GP_INIT_GROW;
    dummy.function_mask = 1u << GP_OP_ADD;
    gp_status rc = mutate_check(params, &dummy, n_offspring, "gp_plan_generation_device");
    if (rc != GP_OK) return rc;
    if (generation > 0xffffffffull || !n_tournaments || (n_offspring > 0 && (!ops || !first_tournament)))
        return fail(GP_ERR_INVALID_ARG, "gp_plan_generation_device: bad arguments");
    if (static_cast<int64_t>(n_offspring) * 2 > 0x7fffffff)
        return fail(GP_ERR_INVALID_ARG, "gp_plan_generation_device: too many offspring");
    return plan_launch(*params, n_offspring, static_cast<uint32_t>(generation), nullptr, ops, first_tournament,
                       n_tournaments, static_cast<hipStream_t>(stream));
}

gp_status gp_mutate_device(const gp_evolve_params* params, const gp_init_params* init,
                           const gp_population_dev* parents, const int32_t* ops, const int32_t* first_tournament,
                           const int32_t* winners, int32_t n_winners, int32_t n_offspring, uint64_t generation,
                           const gp_population_out_dev* out, int64_t* info, void* stream) {
    using namespace gp;
    gp_status rc = mutate_check(params, init, n_offspring, "gp_mutate_device");
    if (rc != GP_OK) return rc;
    if (!parents || !out || !info || generation > 0xffffffffull || n_winners < 0)
        return fail(GP_ERR_INVALID_ARG, "gp_mutate_device: bad arguments");
    if (parents->n_programs < 1 || !parents->nodes || !parents->prog_off || !parents->const_off ||
        (parents->total_consts > 0 && !parents->consts))
        return fail(GP_ERR_INVALID_ARG, "gp_mutate_device: parents need n_programs >= 1 and their arrays");
    if (!out->prog_off || !out->const_off || out->node_capacity < 0 || out->const_capacity < 0 ||
        (n_offspring > 0 && (!out->len || !ops || !first_tournament || !out->nodes || (n_winners > 0 && !winners))) ||
        (out->const_capacity > 0 && !out->consts))
        return fail(GP_ERR_INVALID_ARG, "gp_mutate_device: output arrays missing");
    std::lock_guard<std::mutex> lk(g_mut_mu);
    int dev = 0;
    GP_HIP(hipGetDevice(&dev));
    if (static_cast<int>(g_mut_work.size()) <= dev) g_mut_work.resize(dev + 1);
    MutateWork& w = g_mut_work[dev];
    rc = mutate_work_reserve(&w, n_offspring, *init);
    if (rc != GP_OK) return rc;
    return mutate_launch(w, *params, *init, *parents, ops, first_tournament, winners, n_winners, n_offspring,
                         static_cast<uint32_t>(generation), nullptr, *out, info, static_cast<hipStream_t>(stream));
}

}  // extern "C"
