// k_dag.hip -- building Handley's population DAG on the GPU.
//
// The paper caches the results of structurally identical subtrees so that
// code shared between individuals is not executed again (Sec. 1, Sec. 3.1),
// generalising the trees to a DAG as in Handley's work (Sec. 2).  The DAG is
// built here by hash-consing, in three steps:
//   1. structure: one wave per tree scans its postfix tokens 64 at a time,
//      validates arities and opcodes, and records each token's children and
//      height (a terminal has height 0);
//   2. hash-consing, level by level in increasing height (one launch each): a token's key is
//      (opcode, payload, classes of its children), whose children all lie on
//      lower, already finished levels.  Keys go into an open-addressing table
//      (linear probing, capacity >= 2 x tokens); equal keys are detected by
//      comparing the full key, never the hash alone.  While the levels run, a
//      token's class is the table slot of its key (a slot never moves, so the
//      keys built from classes stay put); the representative of a key is its
//      smallest token index (atomicMin over every level: with rewrites, one
//      key can occur at several tree heights), and a later pass replaces each
//      class by its representative, so the result does not depend on thread
//      timing;
//   3. compaction: representatives are numbered by an exclusive scan in token
//      order, which is the order of first occurrence in a postfix walk of the
//      trees in population order, so children get smaller ids than parents.
// A small population takes steps 2 and 3 in one workgroup (k_build_small),
// whose barriers cost a microsecond where a launch per pass costs several.
#include <hip/hip_runtime.h>

#include <algorithm>

#include <stddef.h>
#include <stdio.h>
#include <string.h>
#include <vector>

#include "runtime_internal.h"
#include "tree_scan.h"

namespace tgp {

constexpr int kLvlBins = 512;  // tree levels counted in LDS

// What the host reads back.  A build ends with one copy of it and the DAG's
// arrays (small populations), or of it, then of the arrays.
struct BuildStatus {
    unsigned long long first_error;  // (tree << 4) | code, min over trees; ~0 = none
    int64_t first_off, last_off;     // the population's first and last offset
    int32_t max_height;
    int32_t max_var;
    int32_t max_stack;
    int32_t nodes;                   // distinct subtrees
    int32_t cnt[kLvlBins];           // tokens of each height
    int32_t cursor[kLvlBins];        // and how many of them are listed
};
// The head of a DAG's device block, in front of its arrays.
constexpr size_t kBlobHead = (sizeof(BuildStatus) + 255) / 256 * 256;

enum { ERR_NONE = 0, ERR_OP = 1, ERR_PARSE = 2, ERR_RANGE = 3 };

__device__ __forceinline__ void report(BuildStatus *st, int64_t r, int code) {
    atomicMin(&st->first_error, ((unsigned long long)r << 4) | (unsigned long long)code);
}

// 1. Structure scan, one wave per tree (tree_scan.h): every token's children
// and height.  info[r]: the tree's height, stack depth and highest axis
// (reduced by the next launch: an atomic per tree would serialise on a few
// addresses).  1.31 ms with one thread per tree on the 1000 x 3 depth-12
// population, 0.48 ms on 200 trees to depth 10; 0.11 and 0.03 ms with one wave.
constexpr int64_t kStructBlocks = 1 << 20;

__global__ __launch_bounds__(64) void k_structure(const uint2 *tok, const int64_t *off, int64_t R, int64_t T,
                                                  int32_t *kid, int32_t *height, int32_t *stk, int32_t *root_tok,
                                                  int4 *info, BuildStatus *st) {
    __shared__ int2 last[kScanSlots];
    const int lane = threadIdx.x;
    for (int64_t r = blockIdx.x; r < R; r += gridDim.x) {
        const int64_t o0 = off[r], o1 = off[r + 1];
        TreeInfo found{0, 0, -1};
        int err = ERR_NONE;
        if (o0 < 0 || o1 > T || o1 < o0) {
            err = ERR_RANGE;
        } else if (o1 == o0) {
            err = ERR_PARSE;
        } else {
            const int v = tree_scan<true>(tok, o0, o1, lane, last, stk + o0, height, found,
                                          [&](int64_t t, const TreeToken &x) {
                                              kid[3 * t + 0] = x.kid[0];
                                              kid[3 * t + 1] = x.kid[1];
                                              kid[3 * t + 2] = x.kid[2];
                                              height[t] = x.height;
                                          });
            err = v == kTreeOp ? ERR_OP : (v == kTreeParse ? ERR_PARSE : ERR_NONE);
        }
        if (lane == 0) {
            if (err != ERR_NONE) report(st, r, err);
            root_tok[r] = (int32_t)(o1 - 1);
            info[r] = int4{found.height, found.stack, found.max_var, 0};
        }
    }
}

// The status of a build that has not started, with the population's ends.
// The ends go to *host too, if given (pinned memory).
__global__ __launch_bounds__(256) void k_build_init(BuildStatus *st, const int64_t *off, int64_t R,
                                                    BuildStatus *host) {
    for (int i = threadIdx.x; i < kLvlBins; i += blockDim.x) st->cnt[i] = st->cursor[i] = 0;
    if (threadIdx.x == 0) {
        st->first_error = ~0ull;
        st->first_off = off[0];
        st->last_off = off[R];
        if (host) {
            host->first_off = off[0];
            host->last_off = off[R];
        }
        st->max_height = st->max_stack = st->nodes = 0;
        st->max_var = -1;
    }
}

// The tallest tree, deepest stack and highest axis over the trees' info: the
// maxima of trees first, first + step, ... into *st.
__device__ __forceinline__ void tree_max(const int4 *info, int64_t R, int64_t first, int64_t step, BuildStatus *st) {
    int32_t h = 0, sp = 0, v = -1;
    for (int64_t r = first; r < R; r += step) {
        const int4 x = info[r];
        h = max(h, x.x);
        sp = max(sp, x.y);
        v = max(v, x.z);
    }
    for (int o = 32; o > 0; o >>= 1) {
        h = max(h, __shfl_xor(h, o));
        sp = max(sp, __shfl_xor(sp, o));
        v = max(v, __shfl_xor(v, o));
    }
    if ((threadIdx.x & 63) == 0) {
        if (h > 0) atomicMax(&st->max_height, h);
        if (sp > 0) atomicMax(&st->max_stack, sp);
        if (v >= 0) atomicMax(&st->max_var, v);
    }
}

__global__ void k_level_hist(const int32_t *height, int64_t T, int32_t *cnt) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < T) atomicAdd(&cnt[height[t]], 1);
}

__global__ void k_level_scatter(const int32_t *height, int64_t T, int32_t *cursor, int32_t *list) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < T) {
        const int32_t pos = atomicAdd(&cursor[height[t]], 1);
        list[pos] = (int32_t)t;
    }
}

// The same two passes with the counters privatised in LDS (most tokens are
// leaves, so the global forms above serialise on one address).  A block
// takes kLvlPer tokens per thread and touches each global counter once.
// Used when the tallest tree has at most kLvlBins levels; the order of the
// tokens inside a level is not significant.  The count runs before the trees
// are known to be sound, so it leaves out heights outside the bins (a
// malformed tree's are not written).
constexpr int kLvlPer = 16;
constexpr int kMaxBlocks = 4;  // of the count launch, reduce the trees' info as well

__global__ void __launch_bounds__(256) k_level_hist_lds(const int32_t *height, int64_t T, const int4 *info, int64_t R,
                                                        BuildStatus *st) {
    __shared__ int32_t c[kLvlBins];
    for (int i = threadIdx.x; i < kLvlBins; i += blockDim.x) c[i] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * blockDim.x * kLvlPer + threadIdx.x;
    for (int j = 0; j < kLvlPer; ++j) {
        const int64_t t = base + (int64_t)j * blockDim.x;
        const uint32_t h = t < T ? (uint32_t)height[t] : ~0u;
        if (h < kLvlBins) atomicAdd(&c[h], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kLvlBins; i += blockDim.x)
        if (c[i]) atomicAdd(&st->cnt[i], c[i]);
    const int64_t nb = min((int64_t)gridDim.x, (int64_t)kMaxBlocks);
    if (blockIdx.x < nb)
        tree_max(info, R, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nb * blockDim.x, st);
}

// First list entry of every level, into start[0 .. kLvlBins] (256 threads).
__device__ __forceinline__ void level_starts(const int32_t *cnt, int32_t *start, int32_t *tmp) {
    const int tid = threadIdx.x;
    const int32_t a = cnt[2 * tid], b = cnt[2 * tid + 1];
    int32_t s = wave_scan(a + b, tid & 63);
    if ((tid & 63) == 63) tmp[tid >> 6] = s;
    __syncthreads();
    for (int w = 0; w < (tid >> 6); ++w) s += tmp[w];
    start[2 * tid] = s - a - b;
    start[2 * tid + 1] = s - b;
    if (tid == 255) start[kLvlBins] = s;
    __syncthreads();
}

__global__ void __launch_bounds__(256) k_level_scatter_lds(const int32_t *height, int64_t T, BuildStatus *st,
                                                           int32_t *list) {
    static_assert(kLvlBins == 512, "two levels per thread");
    __shared__ int32_t c[kLvlBins], start[kLvlBins + 1], tmp[4];
    level_starts(st->cnt, start, tmp);
    for (int i = threadIdx.x; i < kLvlBins; i += blockDim.x) c[i] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * blockDim.x * kLvlPer + threadIdx.x;
    int32_t h[kLvlPer], r[kLvlPer];
    for (int j = 0; j < kLvlPer; ++j) {
        const int64_t t = base + (int64_t)j * blockDim.x;
        h[j] = t < T ? height[t] : -1;
        r[j] = h[j] >= 0 ? atomicAdd(&c[h[j]], 1) : 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kLvlBins; i += blockDim.x)
        if (c[i]) c[i] = start[i] + atomicAdd(&st->cursor[i], c[i]);
    __syncthreads();
    for (int j = 0; j < kLvlPer; ++j)
        if (h[j] >= 0) list[c[h[j]] + r[j]] = (int32_t)(base + (int64_t)j * blockDim.x);
}

// Key of token t: k0 = opcode | axis << 8 (the axis only for a variable);
// k1 = constant bits or first child's canonical id; k2, k3 = further
// children; unused fields are all-ones.
struct Key {
    uint32_t k0, k1, k2, k3;
};

// Operators whose operands commute bitwise in this library (see
// tgp_ctx_set_hashing).
__device__ __forceinline__ bool commutes(uint32_t op) {
    return op == TGP_ADD || op == TGP_MULT || op == TGP_MIN || op == TGP_MAX || op == TGP_MDIST ||
           op == TGP_LEN || op == TGP_OR || op == TGP_XOR || op == TGP_AND;
}

// (I: the width the children and classes are held at, 16 bits in LDS.)
template <class I>
__device__ __forceinline__ Key key_of(int32_t t, const uint2 *tok, const I *kid, const I *canon, bool commute) {
    const uint2 w = tok[t];
    const uint32_t op = w.x & 0xffu;
    Key k{op, 0xffffffffu, 0xffffffffu, 0xffffffffu};
    if (op == TGP_VAR) {
        k.k0 = op | (w.x & 0xff00u);
    } else if (op == TGP_CONST) {
        k.k1 = w.y;
    } else {
        const int a = arity_of(op);
        k.k1 = (uint32_t)canon[kid[3 * t + 0]];
        if (a > 1) k.k2 = (uint32_t)canon[kid[3 * t + 1]];
        if (a > 2) k.k3 = (uint32_t)canon[kid[3 * t + 2]];
        if (commute && commutes(op) && k.k1 > k.k2) {
            const uint32_t x = k.k1;
            k.k1 = k.k2;
            k.k2 = x;
        }
    }
    return k;
}

__device__ __forceinline__ bool key_eq(const Key &a, const Key &b) {
    return a.k0 == b.k0 && a.k1 == b.k1 && a.k2 == b.k2 && a.k3 == b.k3;
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t key_hash(const Key &k, uint32_t hash_mask_bits) {
    uint64_t h = mix64(((uint64_t)k.k0 << 32) | k.k1);
    h = mix64(h ^ (((uint64_t)k.k2 << 32) | k.k3));
    if (hash_mask_bits) h &= ((1ull << hash_mask_bits) - 1);  // collision stress (tests)
    return h;
}

// Identity rewrites (tgp_ctx_set_rewrite; the algebraic equivalences of Wong
// and Zhang's subtree caching, Sec. 2, and the simplification the paper
// proposes as future work, Sec. 5), restricted to those that hold bit for bit
// under this library's readings (NaN payloads aside) and whose result is a
// node that already exists: the representative token that token t stands for,
// or -1 (as a class, like canon while the levels run).  The rules:
//   neg(neg(x)) -> x; abs(abs(x)) -> abs(x); sign(sign(x)) -> sign(x);
//   step(step(x)) -> step(x); min(x, x) -> x; max(x, x) -> x;
//   if(c, y, y) -> y; sub(x, +0) -> x; add(x, -0), add(-0, x) -> x;
//   mult(x, 1), mult(1, x) -> x; div(x, 1) -> x.
// The children are already canonical (lower levels), so a rule sees through
// earlier rewrites.
template <class I>
__device__ __forceinline__ int32_t rewrite_target(int32_t t, const uint2 *tok, const I *kid, const I *canon,
                                                  const int32_t *table) {
    const uint32_t op = tok[t].x & 0xffu;
    const int a = arity_of(op);
    if (a == 0) return -1;
    // classes (table slots) of the children; any token of a class (its
    // slot's current value) has the class's opcode, payload and children
    const int32_t c0 = canon[kid[3 * t]];
    const int32_t c1 = a > 1 ? canon[kid[3 * t + 1]] : -1;
    const int32_t c2 = a > 2 ? canon[kid[3 * t + 2]] : -1;
    auto op_of = [&](int32_t c) { return tok[table[c]].x & 0xffu; };
    auto is_const = [&](int32_t c, uint32_t bits) { return op_of(c) == TGP_CONST && tok[table[c]].y == bits; };
    switch (op) {
    case TGP_NEG: return op_of(c0) == TGP_NEG ? canon[kid[3 * table[c0]]] : -1;
    case TGP_ABS:
    case TGP_SIGN:
    case TGP_STEP: return op_of(c0) == op ? c0 : -1;
    case TGP_MIN:
    case TGP_MAX: return c0 == c1 ? c0 : -1;
    case TGP_IF: return c1 == c2 ? c1 : -1;
    case TGP_SUB: return is_const(c1, 0x00000000u) ? c0 : -1;
    case TGP_ADD: return is_const(c1, 0x80000000u) ? c0 : (is_const(c0, 0x80000000u) ? c1 : -1);
    case TGP_MULT: return is_const(c1, 0x3f800000u) ? c0 : (is_const(c0, 0x3f800000u) ? c1 : -1);
    case TGP_DIV: return is_const(c1, 0x3f800000u) ? c0 : -1;
    default: return -1;
    }
}

// 2a. Inserts token t (-1: none) into the table; the slot of a key ends up
// holding the smallest token index with that key, and is the token's class.
// A rewritten token is not inserted: its class is the one it stands for.
// Every lane of the wave calls it (the leaves' ballots).
template <class I>
__device__ __forceinline__ void hash_token(int32_t t, const uint2 *tok, const I *kid, I *canon, int32_t *table,
                                           uint64_t mask, uint32_t hash_bits, bool commute, bool rewrite) {
    const bool live = t >= 0;
    const Key k = live ? key_of(t, tok, kid, canon, commute) : Key{0xffffffffu, 0, 0, 0};
    const int32_t target = live && rewrite ? rewrite_target(t, tok, kid, canon, table) : -1;
    // Leaves (x, y, z and common constants) repeat many times within one
    // wave: lanes holding the same leaf key (its first two words) insert once,
    // through the group's lowest lane, with the group's smallest token index.
    // The axes first, then two constants (the distinct constants of a random
    // population would each make a group); four groups a wave at most.
    const uint32_t op = k.k0 & 0xffu;
    const bool leaf = live && (op == TGP_VAR || op == TGP_CONST);
    bool insert = live && target < 0;
    int from = (int)(threadIdx.x & 63u);  // the lane that inserts this lane's key
    const int lane = from;
    int32_t smallest = t;
    uint64_t todo = __ballot(leaf), axes = __ballot(live && op == TGP_VAR), consts = todo & ~axes;
    for (int round = 0; round < 4 && todo; ++round) {
        todo = axes ? axes : consts;
        const int leader = __ffsll((unsigned long long)todo) - 1;
        const uint32_t l0 = __shfl(k.k0, leader), l1 = __shfl(k.k1, leader);
        const uint64_t same = __ballot(leaf && k.k0 == l0 && k.k1 == l1) & todo;
        if (__popcll(same) > 1) {
            int32_t m = ((same >> lane) & 1u) ? t : INT32_MAX;
            for (int d = 32; d > 0; d >>= 1) m = min(m, __shfl_xor(m, d));
            if ((same >> lane) & 1u) {
                from = leader;
                insert = lane == leader;
                smallest = m;
            }
        }
        axes &= ~same;
        consts &= ~same;
        todo = axes | consts;
    }
    uint64_t s = 0;
    if (insert) {
        s = key_hash(k, hash_bits) & mask;
        for (;;) {  // at most half the table is ever taken
            int32_t e = table[s];
            if (e < 0) {
                e = atomicCAS(&table[s], -1, smallest);
                if (e < 0) break;  // claimed an empty slot
            }
            if (key_eq(key_of(e, tok, kid, canon, commute), k)) {
                // A slot's value only decreases and its key never changes, so a
                // token that is not below the value it read (which may be stale,
                // never lower than the current one) cannot lower it.  Skipping
                // those leaves the atomics to the few tokens that can: without
                // this, every leaf x or y of the level updated one address.
                if (smallest < e) atomicMin(&table[s], smallest);
                break;
            }
            s = (s + 1) & mask;
        }
    }
    const int32_t slot = __shfl((int32_t)s, from);
    if (live) canon[t] = (I)(target >= 0 ? target : slot);
}

// One level of tokens.  (The class needs no second look-up: a key's slot
// never moves once it is claimed, and the children's classes are final.)
__global__ __launch_bounds__(256) void k_hash_level(const int32_t *list, int32_t n, const uint2 *tok,
                                                    const int32_t *kid, int32_t *canon, int32_t *table, uint64_t mask,
                                                    uint32_t hash_bits, bool commute, bool rewrite) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    hash_token(i < n ? list[i] : -1, tok, kid, canon, table, mask, hash_bits, commute, rewrite);
}

// Levels h0 .. H - 1, listed from `first` on, by one workgroup with a barrier
// after each (the vector cache is its compute unit's; classes are plain
// stores, and what an atomic did to the table is waited for).  The upper
// levels of a population's trees hold few tokens: a launch each is some 6 us
// for work below 3.  Levels of up to 1024 tokens, one a thread: the build of 500
// bred trees (9.7 k tokens) took 175 us with a launch per level and 156 us with
// this, 300 trees of three axes 190 and 178 us, 200 trees to depth 10 253 and
// 244 us (268 with levels of up to 2048; up to 512 is as 1024).
constexpr int32_t kRestTokens = 1024;
constexpr int kRestThreads = 1024;

__global__ __launch_bounds__(kRestThreads) void k_hash_rest(const int32_t *list, int32_t first, int32_t h0, int32_t H,
                                                            const BuildStatus *st, const uint2 *tok,
                                                            const int32_t *kid, int32_t *canon, int32_t *table,
                                                            uint64_t mask, uint32_t hash_bits, bool commute,
                                                            bool rewrite) {
    __shared__ int32_t cnt[kLvlBins];
    const int tid = threadIdx.x, wave = tid >> 6;
    for (int h = h0 + tid; h < H; h += kRestThreads) cnt[h] = st->cnt[h];
    __syncthreads();
    for (int32_t h = h0; h < H; ++h) {
        const int32_t n = cnt[h];
        for (int32_t i0 = 0; i0 < n; i0 += kRestThreads)  // whole waves take part
            if (i0 + wave * 64 < n)
                hash_token(i0 + tid < n ? list[first + i0 + tid] : -1, tok, kid, canon, table, mask, hash_bits,
                           commute, rewrite);
        first += n;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
}

__global__ void k_fill(int32_t *p, int64_t n, int32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// 2b. After the last level: every class becomes its representative, the
// smallest token index with that key; representatives get their rank within
// the 1024 tokens of the block, and the block its count.
constexpr int kRankTokens = 1024;

__global__ __launch_bounds__(256) void k_rank(int32_t *canon, int64_t T, const int32_t *table, int32_t *pos,
                                              int32_t *block_sum) {
    __shared__ int32_t tmp[4];
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kRankTokens + tid * 4;
    int32_t f[4], sum = 0;
    for (int j = 0; j < 4; ++j) {
        const int64_t t = base + j;
        f[j] = 0;
        if (t < T) {
            const int32_t c = table[canon[t]];
            canon[t] = c;
            f[j] = c == (int32_t)t ? 1 : 0;
        }
        sum += f[j];
    }
    int32_t run = wave_scan(sum, tid & 63);
    if ((tid & 63) == 63) tmp[tid >> 6] = run;
    __syncthreads();
    for (int w = 0; w < (tid >> 6); ++w) run += tmp[w];
    if (tid == 255) block_sum[blockIdx.x] = run;
    run -= sum;
    for (int j = 0; j < 4; ++j) {
        if (base + j < T) pos[base + j] = run;
        run += f[j];
    }
}

// Exclusive scan of the blocks' counts by one block; the total is the number
// of nodes.
__global__ __launch_bounds__(1024) void k_rank_blocks(int32_t *block_sum, int64_t nb, BuildStatus *st) {
    __shared__ int32_t tmp[16];
    const int tid = threadIdx.x;
    int32_t carry = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += 1024) {
        const int32_t v = c0 + tid < nb ? block_sum[c0 + tid] : 0;
        int32_t run = wave_scan(v, tid & 63);
        if ((tid & 63) == 63) tmp[tid >> 6] = run;
        __syncthreads();
        int32_t total = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < (tid >> 6)) run += tmp[w];
            total += tmp[w];
        }
        if (c0 + tid < nb) block_sum[c0 + tid] = carry + run - v;
        carry += total;
        __syncthreads();
    }
    if (tid == 0) st->nodes = carry;
}

// The arrays of a DAG's block (DagDevice), laid out for U nodes.
struct NodeArrays {
    int32_t *op, *value, *kid, *height, *mult, *indeg, *roots;
    __device__ __forceinline__ NodeArrays(int32_t *b, int64_t U)
        : op(b), value(b + U), kid(b + 2 * U), height(b + 5 * U), mult(b + 6 * U), indeg(b + 7 * U), roots(b + 8 * U) {}
};

// Fields of the node that token w stands for.
__device__ __forceinline__ void put_node(const NodeArrays &A, int32_t id, uint2 w, int32_t height) {
    const uint32_t op = w.x & 0xffu;
    A.op[id] = (int32_t)(op == TGP_VAR ? (op | (w.x & 0xff00u)) : op);
    A.value[id] = op == TGP_CONST ? (int32_t)w.y : 0;
    A.height[id] = height;
}

// 3a. Node fields of every representative, the roots, and zeroed counts.
__global__ void k_emit_nodes(const uint2 *tok, const int32_t *canon, const int32_t *pos, const int32_t *block_off,
                             const int32_t *height, int64_t T, const int32_t *root_tok, int64_t R, int32_t *blob,
                             const BuildStatus *st) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // up to max(T, R)
    const int64_t U = st->nodes;
    const NodeArrays A(blob, U);
    auto id_of = [&](int32_t c) { return pos[c] + block_off[c / kRankTokens]; };
    if (t < T && canon[t] == (int32_t)t) put_node(A, id_of((int32_t)t), tok[t], height[t]);
    if (t < U) A.mult[t] = A.indeg[t] = 0;
    if (t < R) A.roots[t] = id_of(canon[root_tok[t]]);
}

// 3b. Children ids, in-degrees and multiplicities.
// Block-level counts: an open-addressing table in LDS of (id, count), filled
// with LDS atomics and flushed to the device counters with one atomic per
// distinct id of the block.  An id that finds no free entry within a few
// probes goes straight to its device counter.
constexpr int kCountSlots = 1024;  // at most 256 + 768 distinct ids per block of 256
struct BlockCounts {
    int32_t id[kCountSlots];
    int32_t n[kCountSlots];
};

__device__ __forceinline__ void block_counts_clear(BlockCounts &c) {
    for (int e = threadIdx.x; e < kCountSlots; e += blockDim.x) {
        c.id[e] = -1;
        c.n[e] = 0;
    }
}

__device__ __forceinline__ void block_counts_add(BlockCounts &c, int32_t *counter, int32_t id, int32_t k) {
    uint32_t h = ((uint32_t)id * 2654435761u) & (kCountSlots - 1);
    for (int probe = 0; probe < 8; ++probe) {
        const int32_t prev = atomicCAS(&c.id[h], -1, id);
        if (prev == -1 || prev == id) {
            atomicAdd(&c.n[h], k);
            return;
        }
        h = (h + 1) & (kCountSlots - 1);
    }
    atomicAdd(&counter[id], k);
}

__device__ __forceinline__ void block_counts_flush(const BlockCounts &c, int32_t *counter) {
    for (int e = threadIdx.x; e < kCountSlots; e += blockDim.x)
        if (c.id[e] >= 0) atomicAdd(&counter[c.id[e]], c.n[e]);
}

// Blocks of four waves: a block of many waves waits for that many free wave
// slots on one compute unit, which it rarely finds while a long evaluation
// kernel runs beside it (DAGs are built on side streams when serving).
constexpr int kEmitBlock = 256;

// (Lanes add to the block's LDS table one by one: equal ids serialise there
// for a cycle each.  Grouping them by ballots first took up to 64 rounds a
// wave, 25 us for the smallest population.)
__global__ __launch_bounds__(kEmitBlock) void k_emit_edges(const int32_t *canon, const int32_t *pos,
                                                           const int32_t *block_off, const int32_t *kid, int64_t T,
                                                           int32_t *blob, const BuildStatus *st) {
    __shared__ BlockCounts cm, ci;
    block_counts_clear(cm);
    block_counts_clear(ci);
    __syncthreads();
    const NodeArrays A(blob, st->nodes);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    auto id_of = [&](int32_t c) { return pos[c] + block_off[c / kRankTokens]; };
    if (t < T) {
        const int32_t c = canon[t];
        const int32_t id = id_of(c);
        block_counts_add(cm, A.mult, id, 1);
        if (c == (int32_t)t) {  // the token that represents node id
            for (int j = 0; j < 3; ++j) {
                const int32_t k = kid[3 * t + j];
                const int32_t kid_id = k < 0 ? -1 : id_of(canon[k]);
                A.kid[3 * (int64_t)id + j] = kid_id;
                if (k >= 0) block_counts_add(ci, A.indeg, kid_id, 1);
            }
        }
    }
    __syncthreads();
    block_counts_flush(cm, A.mult);
    block_counts_flush(ci, A.indeg);
}

// Steps 2 and 3 for a small population, after k_structure, in one workgroup
// of 16 waves: level lists, hash-consing level by level, ranks, emission, all
// separated by workgroup barriers.  What bounds it is the chain of dependent
// reads of each level (list, children, their classes, the table slot, the
// slot's token and its children's classes), so all of these but the tokens
// themselves are in LDS, indexes in 16 bits: 14 bytes a token and 4 a table
// slot, 148 KB of the 160 at the most.  The counts hold every node's tokens
// (low half) and edges (high half, at most three per node).  The head of the
// blob gets the status; nothing else is written when a tree is malformed or
// too tall for the bins.
//
// A population of 50 trees (690 tokens) took 42 launches, copies and fills and
// five waits, 0.30 ms a build; with one workgroup and two waits 0.078 ms, and
// 0.065 ms since the indexes are in LDS (5.0 k tokens: 0.164 and 0.122 ms, 5.2 k
// with image operators 0.136 and 0.092 ms).  The line is the LDS: past 6144
// tokens the table would have to be denser or stay in memory, where at 9.4 k
// tokens one workgroup lost to a launch per level (0.21 and 0.19 ms).
constexpr int64_t kSmallTokens = 6144;
constexpr int kSmallThreads = 1024;

__global__ __launch_bounds__(kSmallThreads) void k_build_small(const uint2 *tok, int32_t T, const int32_t *kid,
                                                               const int32_t *height, const int32_t *root_tok,
                                                               const int4 *info, int32_t R, uint32_t mask,
                                                               uint32_t hash_bits, bool commute, bool rewrite,
                                                               int32_t *blob, const BuildStatus *st) {
    extern __shared__ uint32_t counts[];  // [T]
    int32_t *const table = reinterpret_cast<int32_t *>(counts + T);       // [mask + 1]
    uint16_t *const kids = reinterpret_cast<uint16_t *>(table + mask + 1);  // [3 T], 0xffff for none
    uint16_t *const canon = kids + 3 * T, *const list = canon + T;        // [T] each
    uint16_t *const pos = list;  // once the levels are done
    __shared__ int32_t c[kLvlBins], start[kLvlBins + 1], tmp[16];
    __shared__ int32_t most[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 3) most[tid] = tid < 2 ? 0 : -1;
    for (int i = tid; i < kLvlBins; i += kSmallThreads) c[i] = 0;
    for (uint32_t i = tid; i <= mask; i += kSmallThreads) table[i] = -1;
    for (int i = tid; i < T; i += kSmallThreads) counts[i] = 0;
    for (int i = tid; i < 3 * T; i += kSmallThreads) kids[i] = (uint16_t)kid[i];
    __syncthreads();
    for (int r = tid; r < R; r += kSmallThreads) {
        const int4 x = info[r];
        atomicMax(&most[0], x.x);
        atomicMax(&most[1], x.y);
        atomicMax(&most[2], x.z);
    }
    __syncthreads();
    const int32_t H = most[0] + 1;
    BuildStatus *const head = reinterpret_cast<BuildStatus *>(reinterpret_cast<char *>(blob) - kBlobHead);
    if (tid == 0) {
        head->first_error = st->first_error;
        head->max_height = most[0];
        head->max_stack = most[1];
        head->max_var = most[2];
        head->nodes = 0;
    }
    if (st->first_error != ~0ull || H > kLvlBins) return;  // (the host reports it, or takes the general way)
    for (int t = tid; t < T; t += kSmallThreads) atomicAdd(&c[height[t]], 1);
    __syncthreads();
    if (tid == 0) {
        int32_t run = 0;
        for (int h = 0; h < H; ++h) {
            start[h] = run;
            run += c[h];
        }
        start[H] = run;
        head->cnt[0] = c[0];
    }
    __syncthreads();
    for (int i = tid; i < H; i += kSmallThreads) c[i] = start[i];
    __syncthreads();
    for (int t = tid; t < T; t += kSmallThreads) list[atomicAdd(&c[height[t]], 1)] = (uint16_t)t;
    __syncthreads();
    for (int32_t h = 0; h < H; ++h) {
        const int32_t end = start[h + 1];
        for (int32_t i0 = start[h]; i0 < end; i0 += kSmallThreads)  // whole waves take part
            if (i0 + wave * 64 < end)
                hash_token(i0 + tid < end ? (int32_t)list[i0 + tid] : -1, tok, kids, canon, table, mask, hash_bits,
                           commute, rewrite);
        __syncthreads();
    }
    // representatives and their ids
    int32_t U = 0;
    for (int t0 = 0; t0 < T; t0 += kSmallThreads) {
        const int t = t0 + tid;
        int32_t rep = -1;
        if (t < T) {
            rep = table[canon[t]];
            canon[t] = (uint16_t)rep;
        }
        const uint64_t m = __ballot(rep == t && t < T);
        if (lane == 0) tmp[wave] = (int32_t)__popcll(m);
        __syncthreads();
        int32_t run = U;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) run += tmp[w];
            U += tmp[w];
        }
        if (t < T) pos[t] = (uint16_t)(run + (int32_t)__popcll(m & ((1ull << lane) - 1)));
        __syncthreads();
    }
    const NodeArrays A(blob, U);
    for (int t = tid; t < T; t += kSmallThreads) {
        const int32_t rep = canon[t], id = pos[rep];
        atomicAdd(&counts[id], 1u);
        if (rep != t) continue;
        put_node(A, id, tok[t], height[t]);
        for (int j = 0; j < 3; ++j) {
            const uint32_t k = kids[3 * t + j];
            const int32_t kid_id = k == 0xffffu ? -1 : pos[canon[k]];
            A.kid[3 * id + j] = kid_id;
            if (kid_id >= 0) atomicAdd(&counts[kid_id], 1u << 16);
        }
    }
    for (int r = tid; r < R; r += kSmallThreads) A.roots[r] = pos[canon[root_tok[r]]];
    __syncthreads();
    for (int i = tid; i < U; i += kSmallThreads) {
        A.mult[i] = (int32_t)(counts[i] & 0xffffu);
        A.indeg[i] = (int32_t)(counts[i] >> 16);
    }
    if (tid == 0) head->nodes = U;
}

// Its LDS for T tokens and a table of cap slots.
static size_t small_lds(int64_t T, uint64_t cap) { return (size_t)(14 * T) + 4 * (size_t)cap; }

// The status and, with a blob, its 8 U + R words (U the nodes found) to pinned
// memory at out, laid out as a DAG's block.  What a copy would take is the
// number of words, which the host knows only after a round trip of its own;
// this launch reads it from the status.  The build of 200 trees to depth 10
// took 268 us with copies and 253 us with this, that of 60 individuals of
// three channels with image operators 145 and 136 us.
__global__ __launch_bounds__(256) void k_publish(const BuildStatus *st, const int32_t *blob, int64_t R, int32_t *out) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    const int32_t *head = reinterpret_cast<const int32_t *>(st);
    for (int64_t i = i0; i < (int64_t)(sizeof(BuildStatus) / 4); i += step) out[i] = head[i];
    if (!blob) return;
    out += kBlobHead / 4;
    const int64_t n = 8 * (int64_t)st->nodes + R;
    for (int64_t i = i0; i < n / 4; i += step) reinterpret_cast<int4 *>(out)[i] = reinterpret_cast<const int4 *>(blob)[i];
    if (i0 < n % 4) out[n / 4 * 4 + i0] = blob[n / 4 * 4 + i0];
}

// The largest DAG block that is published whole: the staging is sized for as
// many nodes as tokens (32 bytes each), of which a large population's DAG
// needs a third or less, and beyond this size the second copy's round trip is
// a small part of the build.
constexpr size_t kPublishBytes = 8 << 20;

// A DAG's block is allocated for as many nodes as tokens.  One of this size and
// four times what the nodes need is worth a copy, which costs a published block
// (and a build of 250 us or more) a wait of 15 us.
constexpr size_t kShrinkBytes = 4 << 20;
static size_t pool_bytes(size_t bytes) { return (size_t)1 << DevicePool::class_of(bytes); }

static inline dim3 grid_for(int64_t n, int b = 256) { return dim3((unsigned)((n + b - 1) / b)); }

// A quarter of one block's words for each thread, on at most 256 blocks.
static inline dim3 publish_grid(int64_t T, int64_t R) {
    return dim3((unsigned)std::min<int64_t>(256, (8 * T + R) / 1024 + 1));
}

void dag_device_free(DagDevice *d, DevicePool &pool) {
    pool.release(d->block);
    *d = DagDevice{};
}

#define DCHK(x)                                                                  \
    do {                                                                         \
        hipError_t _e = (x);                                                     \
        if (_e != hipSuccess) {                                                  \
            snprintf(err, errlen, "%s: %s", #x, hipGetErrorString(_e));          \
            res.status = TGP_EHIP;                                               \
            goto done;                                                           \
        }                                                                        \
    } while (0)

uint32_t g_debug_hash_bits = 0;  // set by tests to force hash collisions

DagBuildResult build_dag_device(tgp_ctx ctx, const tgp_token *tok_dev, const int64_t *off_dev, int64_t R, int64_t T,
                                DagDevice *dev, const int32_t **host, char *err, size_t errlen) {
    DagBuildResult res{};
    res.status = TGP_OK;
    res.bad_tree = -1;
    DevicePool &pool = ctx->pool;
    const hipStream_t s = ctx->stream;
    const bool commute = ctx->commute != 0, rewrite = ctx->rewrite != 0;
    const uint2 *tok = reinterpret_cast<const uint2 *>(tok_dev);
    // scratch, in one block: see the offsets below
    char *scratch = nullptr, *old = nullptr;
    BuildStatus *st = nullptr, *hs = nullptr;
    int32_t *kid, *height, *stk, *root_tok, *list, *canon, *pos, *table, *sums, *blob, *cnt = nullptr;
    int4 *info;
    void *stage = nullptr;
    uint64_t cap = 1024;
    size_t at = 0;
    int64_t H = 0, nb = 0;
    bool small = false, publish = false;
    *dev = DagDevice{};
    *host = nullptr;

    // The status first: a device-resident population's size is not known yet.
    DCHK(pool.alloc((void **)&st, sizeof(BuildStatus)));
    if (T < 0) {
        DCHK(ctx_pinned(ctx, kBlobHead, &stage));
        hs = static_cast<BuildStatus *>(stage);
    }
    hipLaunchKernelGGL(k_build_init, dim3(1), dim3(256), 0, s, st, off_dev, R, hs);
    DCHK(hipGetLastError());
    if (T < 0) {
        DCHK(hipStreamSynchronize(s));
        T = hs->last_off;
        if (hs->first_off != 0 || T < 0 || T > 0x7fffffffLL) {
            res.status = TGP_EINVAL;
            snprintf(err, errlen, hs->first_off != 0 ? "offsets[0] must be 0" : "bad token count");
            goto done;
        }
    }
    res.T = T;
    dev->T = T;
    dev->R = R;
    while (cap < (uint64_t)(2 * T)) cap <<= 1;
    nb = (T + kRankTokens - 1) / kRankTokens;
    {
        auto part = [&at](size_t bytes) {
            const size_t o = at;
            at += (bytes + 255) & ~(size_t)255;
            return o;
        };
        const size_t okid = part(sizeof(int32_t) * 3 * T), oheight = part(sizeof(int32_t) * T),
                     ostk = part(sizeof(int32_t) * T), oroot = part(sizeof(int32_t) * R), oinfo = part(sizeof(int4) * R),
                     olist = part(sizeof(int32_t) * T), ocanon = part(sizeof(int32_t) * T),
                     opos = part(sizeof(int32_t) * T), otable = part(sizeof(int32_t) * cap),
                     osums = part(sizeof(int32_t) * nb);
        DCHK(pool.alloc((void **)&scratch, at));
        kid = (int32_t *)(scratch + okid);
        height = (int32_t *)(scratch + oheight);
        stk = (int32_t *)(scratch + ostk);
        root_tok = (int32_t *)(scratch + oroot);
        info = (int4 *)(scratch + oinfo);
        list = (int32_t *)(scratch + olist);
        canon = (int32_t *)(scratch + ocanon);
        pos = (int32_t *)(scratch + opos);
        table = (int32_t *)(scratch + otable);
        sums = (int32_t *)(scratch + osums);
    }
    // The DAG's block, sized for T distinct nodes, with the status in front.
    DCHK(pool.alloc((void **)&dev->block, kBlobHead + DagDevice::blob_bytes(T, R)));
    blob = reinterpret_cast<int32_t *>(dev->block + kBlobHead);
    small = T > 0 && T <= kSmallTokens && R <= kSmallTokens;
    publish = kBlobHead + DagDevice::blob_bytes(T, R) <= kPublishBytes;
    hipLaunchKernelGGL(k_structure, dim3((unsigned)std::min<int64_t>(R, kStructBlocks)), dim3(64), 0, s, tok, off_dev,
                       R, T, kid, height, stk, root_tok, info, st);
    DCHK(hipGetLastError());
    if (small) {
        // one workgroup, whose status and arrays are published together
        hipLaunchKernelGGL(k_build_small, dim3(1), dim3(kSmallThreads), small_lds(T, cap), s, tok, (int32_t)T, kid,
                           height, root_tok, info, (int32_t)R, (uint32_t)(cap - 1), g_debug_hash_bits, commute, rewrite,
                           blob, st);
        DCHK(hipGetLastError());
        DCHK(ctx_pinned(ctx, kBlobHead + DagDevice::blob_bytes(T, R), &stage));
        hipLaunchKernelGGL(k_publish, publish_grid(T, R), dim3(256), 0, s, reinterpret_cast<BuildStatus *>(dev->block),
                           blob, R, static_cast<int32_t *>(stage));
        DCHK(hipGetLastError());
    } else {
        DCHK(ctx_pinned(ctx, kBlobHead, &stage));
        if (T > 0) {
            hipLaunchKernelGGL(k_level_hist_lds, grid_for(T, 256 * kLvlPer), dim3(256), 0, s, height, T, info, R, st);
            hipLaunchKernelGGL(k_publish, dim3(1), dim3(256), 0, s, st, (const int32_t *)nullptr, R,
                               static_cast<int32_t *>(stage));
            hipLaunchKernelGGL(k_fill, dim3((unsigned)std::min<uint64_t>(1024, cap / 1024)), dim3(256), 0, s, table,
                               (int64_t)cap, -1);
        } else {
            hipLaunchKernelGGL(k_publish, dim3(1), dim3(256), 0, s, st, (const int32_t *)nullptr, R,
                               static_cast<int32_t *>(stage));
        }
        DCHK(hipGetLastError());
    }
    DCHK(hipStreamSynchronize(s));
    hs = static_cast<BuildStatus *>(stage);
    if (hs->first_error != ~0ull) {
        const int code = (int)(hs->first_error & 15ull);
        res.bad_tree = (int64_t)(hs->first_error >> 4);
        res.status = code == ERR_OP ? TGP_EOP : (code == ERR_PARSE ? TGP_EPARSE : TGP_EINVAL);
        snprintf(err, errlen, "tree %lld: %s", (long long)res.bad_tree,
                 code == ERR_OP ? "unknown opcode"
                                : (code == ERR_PARSE ? "token range is not exactly one postfix tree"
                                                     : "offsets out of range or decreasing"));
        goto done;
    }
    res.max_height = hs->max_height;
    res.max_stack = hs->max_stack;
    res.max_var = hs->max_var;
    H = res.max_height + 1;
    if (!small || H > kLvlBins) {
        std::vector<int32_t> start(H + 1, 0);
        if (H <= kLvlBins) {
            for (int64_t h = 0; h < H; ++h) start[h + 1] = start[h] + hs->cnt[h];
            hipLaunchKernelGGL(k_level_scatter_lds, grid_for(T, 256 * kLvlPer), dim3(256), 0, s, height, T, st, list);
            DCHK(hipGetLastError());
        } else {
            // very tall trees: counters in global memory, one per level
            std::vector<int32_t> hcnt(H);
            DCHK(pool.alloc((void **)&cnt, sizeof(int32_t) * H));
            hipLaunchKernelGGL(k_fill, grid_for(H), dim3(256), 0, s, cnt, H, 0);
            if (small)
                hipLaunchKernelGGL(k_fill, dim3((unsigned)std::min<uint64_t>(1024, cap / 1024)), dim3(256), 0, s, table,
                                   (int64_t)cap, -1);
            hipLaunchKernelGGL(k_level_hist, grid_for(T), dim3(256), 0, s, height, T, cnt);
            DCHK(hipGetLastError());
            DCHK(hipMemcpyAsync(hcnt.data(), cnt, sizeof(int32_t) * H, hipMemcpyDeviceToHost, s));
            DCHK(hipStreamSynchronize(s));
            for (int64_t h = 0; h < H; ++h) start[h + 1] = start[h] + hcnt[h];
            DCHK(hipMemcpyAsync(cnt, start.data(), sizeof(int32_t) * H, hipMemcpyHostToDevice, s));
            hipLaunchKernelGGL(k_level_scatter, grid_for(T), dim3(256), 0, s, height, T, cnt, list);
            DCHK(hipGetLastError());
        }
        res.tree_internal = T - (start[1] - start[0]);  // a token of height 0 is a terminal
        // a launch for each of the large levels, one for the rest
        int64_t h0 = H;
        if (H <= kLvlBins)
            while (h0 > 0 && start[h0] - start[h0 - 1] <= kRestTokens) --h0;
        for (int64_t h = 0; h < h0; ++h) {
            const int32_t n = start[h + 1] - start[h];
            if (n > 0)
                hipLaunchKernelGGL(k_hash_level, grid_for(n), dim3(256), 0, s, list + start[h], n, tok, kid, canon,
                                   table, (uint64_t)(cap - 1), g_debug_hash_bits, commute, rewrite);
        }
        if (h0 < H)
            hipLaunchKernelGGL(k_hash_rest, dim3(1), dim3(kRestThreads), 0, s, list, start[h0], (int32_t)h0, (int32_t)H,
                               st, tok, kid, canon, table, (uint64_t)(cap - 1), g_debug_hash_bits, commute, rewrite);
        hipLaunchKernelGGL(k_rank, dim3((unsigned)nb), dim3(256), 0, s, canon, T, table, pos, sums);
        hipLaunchKernelGGL(k_rank_blocks, dim3(1), dim3(1024), 0, s, sums, nb, st);
        hipLaunchKernelGGL(k_emit_nodes, grid_for(std::max(T, R)), dim3(256), 0, s, tok, canon, pos, sums, height, T,
                           root_tok, R, blob, st);
        hipLaunchKernelGGL(k_emit_edges, grid_for(T, kEmitBlock), dim3(kEmitBlock), 0, s, canon, pos, sums, kid, T,
                           blob, st);
        DCHK(hipGetLastError());
        DCHK(ctx_pinned(ctx, kBlobHead + (publish ? DagDevice::blob_bytes(T, R) : 0), &stage));
        hipLaunchKernelGGL(k_publish, publish ? publish_grid(T, R) : dim3(1), dim3(256), 0, s, st,
                           publish ? blob : (const int32_t *)nullptr, R, static_cast<int32_t *>(stage));
        DCHK(hipGetLastError());
        DCHK(hipStreamSynchronize(s));
        res.U = static_cast<BuildStatus *>(stage)->nodes;
        const size_t bytes = DagDevice::blob_bytes(res.U, R);
        // The block goes with the DAG for its life: one of its nodes' size takes
        // its place where that saves much.
        const size_t held = pool_bytes(kBlobHead + DagDevice::blob_bytes(T, R));
        char *fit = nullptr;
        if (held >= kShrinkBytes && held >= 4 * pool_bytes(bytes)) {
            DCHK(pool.alloc((void **)&fit, bytes));
            old = dev->block;
            dev->block = fit;
            DCHK(hipMemcpyAsync(fit, blob, bytes, hipMemcpyDeviceToDevice, s));
        }
        if (publish) {
            *host = reinterpret_cast<const int32_t *>(static_cast<char *>(stage) + kBlobHead);
            if (fit) DCHK(hipStreamSynchronize(s));
        } else {
            DCHK(ctx_pinned(ctx, bytes, &stage));
            DCHK(hipMemcpyAsync(stage, blob, bytes, hipMemcpyDeviceToHost, s));
            DCHK(hipStreamSynchronize(s));
            *host = static_cast<const int32_t *>(stage);
        }
        if (fit) blob = reinterpret_cast<int32_t *>(fit);
    } else {
        res.U = hs->nodes;
        res.tree_internal = T - hs->cnt[0];
        *host = reinterpret_cast<const int32_t *>(static_cast<char *>(stage) + kBlobHead);
    }
    dev->U = res.U;
    dev->node_op = blob;
    dev->node_value = reinterpret_cast<float *>(blob + res.U);
    dev->node_kid = blob + 2 * res.U;
    dev->node_height = blob + 5 * res.U;
    dev->mult = blob + 6 * res.U;
    dev->indeg = blob + 7 * res.U;
    dev->roots = blob + 8 * res.U;
done:
    if (res.status != TGP_OK) {
        hipStreamSynchronize(s);  // every kernel that used the scratch has finished
        dag_device_free(dev, pool);
    }
    pool.release(st);
    pool.release(scratch);
    pool.release(cnt);
    pool.release(old);
    return res;
}

}  // namespace tgp
