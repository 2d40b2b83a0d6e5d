// tree_scan.h -- a wave's scan of one postfix tree, 64 tokens at a time.
//
// With D(i) the stack depth after token i (a prefix sum of 1 - arity), token
// i writes stack slot D(i) - 1.  Its last child is token i - 1, each earlier
// child j of its children is the last token before i that wrote slot
// D(i) - 1 + j, and its subtree begins just after the last token before i of
// depth D(i) - 1.  Among the 64 tokens those are found by ballots over their
// distinct depths (about a dozen); before them, in the wave's table of the
// last (token, height) of every slot.  Heights settle by repeated maxima over
// the children, one round per level that the 64 tokens span.
//
// A tree used to be walked by one thread, so a launch took as long as its
// longest tree's serial chain of one LDS round trip per token (3.5k tokens:
// 1.3 ms).
#pragma once

#include <hip/hip_runtime.h>

#include "tgp_internal.h"

namespace tgp {

constexpr int kScanSlots = 256;  // stack slots of the LDS table

enum { kTreeOk = 0, kTreeParse = 1, kTreeOp = 2, kTreeDeep = 3 };

// Inclusive prefix sum over the wave's lanes.
__device__ __forceinline__ int32_t wave_scan(int32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    return v;
}

// Children, height and first token of one token (absent children are -1).
struct TreeToken {
    int32_t kid[3];
    int32_t height;
    int64_t first;
};

// What a scan finds out about a whole tree.
struct TreeInfo {
    int32_t height, stack, max_var;
};

// Scans the tree of tokens [o0, o1) (not empty) with one wave in a workgroup
// of its own; put(t, token) is called once for every token, by the lane that
// holds it.  Slots past the LDS table `last` (kScanSlots entries) are kept in
// deep_slot(slot) with their heights in deep_height(token), both in global
// memory; without them (DEEP false) such a tree ends the scan with kTreeDeep.
// Returns kTreeOk, or the tree's first error in token order.
template <bool DEEP, typename Put>
__device__ __forceinline__ int tree_scan(const uint2 *tok, int64_t o0, int64_t o1, int lane, int2 *last,
                                         int32_t *deep_slot, const int32_t *deep_height, TreeInfo &info, Put &&put) {
    int32_t sp = 0, maxsp = 0, maxvar = -1, h = 0;
    for (int64_t base = o0; base < o1; base += 64) {
        const int64_t t = base + lane;
        const bool live = t < o1;
        const uint2 w = live ? tok[t] : uint2{(uint32_t)TGP_CONST, 0};
        const uint32_t op = w.x & 0xffu;
        const bool bad_op = op >= TGP_NUM_OPS;
        const int a = bad_op || !live ? 0 : arity_of(op);
        const int32_t d = sp + wave_scan(live ? 1 - a : 0, lane);  // depth after the token
        const uint64_t ops = __ballot(live && bad_op), under = __ballot(live && d < 1);
        if (ops | under) return (ops >> (__ffsll((unsigned long long)(ops | under)) - 1)) & 1u ? kTreeOp : kTreeParse;
        if (!DEEP && __ballot(live && d > kScanSlots)) return kTreeDeep;
        // lanes of the same depth, of one more (the slot of child 1 of three)
        // and of one less (the last one before the subtree)
        uint64_t same = 0, above = 0, below = 0, todo = __ballot(live);
        while (todo) {
            const int32_t v = __builtin_amdgcn_readlane(d, __ffsll((unsigned long long)todo) - 1);
            const uint64_t m = __ballot(live && d == v);
            if (d == v) same = m;
            if (d + 1 == v) above = m;
            if (d - 1 == v) below = m;
            todo &= ~m;
        }
        const uint64_t before = (1ull << lane) - 1;
        auto slot_token = [&](int32_t slot, int32_t &height) {
            if (!DEEP || slot < kScanSlots) {
                const int2 e = last[slot];
                height = e.y;
                return e.x;
            }
            const int32_t c = __hip_atomic_load(deep_slot + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            height = __hip_atomic_load(deep_height + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return c;
        };
        int cl[3] = {-1, -1, -1};         // child lanes (-1: before these tokens)
        int32_t ch[3] = {-1, -1, -1};     // heights of the children before these tokens
        TreeToken x{{-1, -1, -1}, 0, o0};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (j >= a) continue;
            if (j == a - 1) cl[j] = lane - 1;
            else if (const uint64_t m = (j == 0 ? same : above) & before) cl[j] = 63 - __clzll((long long)m);
            x.kid[j] = cl[j] >= 0 ? (int32_t)(base + cl[j]) : slot_token(d - 1 + j, ch[j]);
        }
        if (live && d > 1) {
            int32_t unused;
            const uint64_t m = below & before;
            x.first = 1 + (m ? base + 63 - __clzll((long long)m) : (int64_t)slot_token(d - 2, unused));
        }
        h = 0;
        for (;;) {
            int32_t nh = 0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int32_t in = __shfl(h, cl[j] < 0 ? lane : cl[j]);
                if (j < a) nh = max(nh, 1 + (cl[j] < 0 ? ch[j] : in));
            }
            const bool moved = nh != h;
            h = nh;
            if (!__ballot(moved)) break;  // at most 64 rounds: a child is a lower lane
        }
        x.height = h;
        if (live) put(t, x);
        __syncthreads();  // (one wave) the table's reads are done
        if (live && !(same >> lane >> 1)) {  // the last writer of its slot
            if (!DEEP || d <= kScanSlots) last[d - 1] = int2{(int32_t)t, h};
            else deep_slot[d - 1] = (int32_t)t;
        }
        __syncthreads();
        maxsp = max(maxsp, live ? d : 0);
        if (live && op == TGP_VAR) maxvar = max(maxvar, (int32_t)((w.x >> 8) & 0xffu));
        sp = __shfl(d, (int)min((int64_t)63, o1 - 1 - base));
    }
    if (sp != 1) return kTreeParse;
    info.height = __shfl(h, (int)((o1 - 1 - o0) & 63));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        maxsp = max(maxsp, __shfl_xor(maxsp, o));
        maxvar = max(maxvar, __shfl_xor(maxvar, o));
    }
    info.stack = maxsp;
    info.max_var = maxvar;
    return kTreeOk;
}

// Depth from the root of every token of a well-formed tree whose stack depth
// is at most kScanSlots, 64 tokens at a time from the root back: the parent
// of token i is the first token after it of depth D(i) or less, which is of
// depth D(i) - 2 or more (no operator takes more than three operands).
// `next` (kScanSlots + 1 entries) holds the next (token, tree depth) of every
// stack depth.  put(t, depth) as above.
template <typename Put>
__device__ __forceinline__ void tree_depths(const uint2 *tok, int64_t o0, int64_t o1, int lane, int2 *next, Put &&put) {
    __syncthreads();
    for (int i = lane; i <= kScanSlots; i += 64) next[i] = int2{INT32_MAX, 0};
    __syncthreads();
    int32_t top = 1;  // stack depth after the last of these tokens
    for (int64_t end = o1; end > o0; end -= 64) {
        const int64_t base = end - 64, t = base + lane;
        const bool live = t >= o0;
        const int a = live ? arity_of(tok[t].x & 0xffu) : 1;
        // D(i) = top + sum over the later tokens of (arity - 1)
        const int32_t incl = wave_scan(a - 1, lane);
        const int32_t d = top + __builtin_amdgcn_readlane(incl, 63) - incl;
        uint64_t same = 0, le = 0, todo = __ballot(live);
        while (todo) {
            const int32_t v = __builtin_amdgcn_readlane(d, __ffsll((unsigned long long)todo) - 1);
            const uint64_t m = __ballot(live && d == v);
            if (d == v) same = m;
            if (v <= d) le |= m;
            todo &= ~m;
        }
        const uint64_t after = lane == 63 ? 0ull : ~0ull << (lane + 1);
        const int pl = le & after ? __ffsll((unsigned long long)(le & after)) - 1 : -1;
        int32_t pd = -1;  // depth of a parent after these tokens (-1: the root's)
        if (live && pl < 0 && t != o1 - 1) {
            int2 p = next[d];
            const int2 q = next[d - 1], u = next[max(d - 2, 0)];  // (entry 0: none)
            if (q.x < p.x) p = q;
            if (u.x < p.x) p = u;
            pd = p.y;
        }
        int32_t dep = 0;
        for (;;) {
            const int32_t in = __shfl(dep, pl < 0 ? lane : pl);
            const int32_t nd = 1 + (pl < 0 ? pd : in);
            const bool moved = nd != dep;
            dep = nd;
            if (!__ballot(moved)) break;  // at most 64 rounds: a parent is a higher lane
        }
        if (live) put(t, dep);
        __syncthreads();
        if (live && !(same & ((1ull << lane) - 1))) next[d] = int2{(int32_t)t, dep};
        __syncthreads();
        top = __builtin_amdgcn_readlane(d, 0) - 1 + __builtin_amdgcn_readlane(a, 0);
    }
}

}  // namespace tgp
