// forest_dev.hpp -- device functions shared by the tree-growth kernels:
// node creation / classification and wave-level candidate reductions.
#pragma once

#include "dev_common.hpp"
#include "reg_dev.hpp"

namespace boruta {

// Lane-ordered comparison of two candidates of ONE feature: higher Q first,
// then the smaller threshold (the smallest b of an equal-score partition).
// Invalid candidates (nl == 0) lose to everything.
__device__ __forceinline__ bool cand_wins_same_feature(const Cand& a, const Cand& b) {
    if (b.nl == 0) return a.nl != 0 || a.b < b.b;
    if (a.nl == 0) return false;
    if (cand_better(a, b)) return true;
    if (cand_better(b, a)) return false;
    return a.b < b.b;
}

__device__ __forceinline__ Cand shfl_cand(const Cand& c, int src) {
    Cand o;
    o.q = __shfl(c.q, src);
    o.f = __shfl(c.f, src);
    o.b = __shfl(c.b, src);
    o.nl = __shfl(c.nl, src);
    o.nr = __shfl(c.nr, src);
    o.pad = 0;
    o.sl = __shfl(c.sl, src);
    o.sr = __shfl(c.sr, src);
    return o;
}

__device__ __forceinline__ Cand shfl_xor_cand(const Cand& c, int m) {
    return shfl_cand(c, (int)((threadIdx.x & 63) ^ m));
}

// Exact wave-wide best of one feature's candidates (all lanes get it).
__device__ __forceinline__ Cand wave_best_exact(Cand c) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const Cand o = shfl_xor_cand(c, m);
        if (cand_wins_same_feature(o, c)) c = o;
    }
    return c;
}

// Wave-wide scans through DPP row shifts (within rows of 16 lanes) and row
// broadcasts (lane 15 -> next row, lane 31 -> rows 2-3); lanes whose DPP
// source is outside the pattern take the identity.  No LDS traffic.
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

// Maximum over the wave (a max-scan; lane 63 ends with the total), as a
// wave-uniform value, of scores that are -1 or not negative: their bits order
// as signed integers, one instruction per step.
__device__ __forceinline__ float wave_max_f_dpp(float f) {
    int v = __float_as_int(f);
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return __int_as_float(__builtin_amdgcn_readlane(v, 63));
}

// The same for FP64 scores that are -1 or not negative.
__device__ __forceinline__ double dpp_f64(double v, int sel) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    int lo = (int)(uint32_t)b, hi = (int)(uint32_t)(b >> 32);
    switch (sel) {
#define BORUTA_DPP(S, CTRL, ROWS)                                              \
    case S:                                                                    \
        lo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);      \
        hi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);      \
        break;
        BORUTA_DPP(0, 0x111, 0xf)
        BORUTA_DPP(1, 0x112, 0xf)
        BORUTA_DPP(2, 0x114, 0xf)
        BORUTA_DPP(3, 0x118, 0xf)
        BORUTA_DPP(4, 0x142, 0xa)
        BORUTA_DPP(5, 0x143, 0xc)
#undef BORUTA_DPP
    }
    return __builtin_bit_cast(double, (uint64_t)(uint32_t)lo | (uint64_t)(uint32_t)hi << 32);
}
__device__ __forceinline__ double wave_max_f64_dpp(double v) {
#pragma unroll
    for (int s = 0; s < 6; ++s) v = fmax(v, dpp_f64(v, s));
    return __builtin_bit_cast(double, readlane64(__builtin_bit_cast(uint64_t, v), 63));
}

// Minimum over the wave, as a wave-uniform value.
__device__ __forceinline__ uint32_t wave_min_u_dpp(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x112, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x114, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x118, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xa, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Margin of the FP32 ranking.  An FP32 score is within eps of its exact value
// Q: eps = 5u (u = 2^-24) for cand_q32 and (K + 4)u <= 20u for hist_q32
// below.  The exact best then scores at least (1 - 2 eps) * FP32 max, so
// every candidate at or above (1 - 2^-18) * FP32 max (64u > 2 * 20u plus the
// rounding of this product) is re-ranked exactly, and the FP32-ranked choice
// equals the exact one.  Two scores farther apart than this margin are in
// exact order.
__device__ __forceinline__ float fp32_floor(float qmax) { return qmax * (1.0f - 0x1.0p-18f); }

// FP32 score straight from the left class counts of a threshold:
// S_L = sum cl_k^2 and S_R = sum (c_k - cl_k)^2 by FMA chains (K roundings
// each; the counts are exact in FP32 below 2^24), then S_L rcp(N_L) +
// S_R rcp(N_R).  Relative error <= (K + 4)u.  Returns -1 when one side is
// empty.
template <int KMAX>
__device__ __forceinline__ float hist_q32(const uint32_t* cl, const uint32_t* cnode, uint32_t N) {
    float nl = 0.0f, sl = 0.0f, sr = 0.0f;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const float l = (float)cl[k], r = (float)(cnode[k] - cl[k]);
        nl += l;
        sl = fmaf(l, l, sl);
        sr = fmaf(r, r, sr);
    }
    const float nr = (float)N - nl;
    if (nl == 0.0f || nr == 0.0f) return -1.0f;
    return sl * __builtin_amdgcn_rcpf(nl) + sr * __builtin_amdgcn_rcpf(nr);
}

// Packed class counters: a side's class counts as fields of FB bits -- 8 for
// nodes of weight N < 256 (four classes to a 32-bit word), 16 for N < 65536
// (two).  The dot product of bytes or halves (full rate) gives the exact
// integers of a split: for left counts l and node counts c, N_L = sum l,
// S_L = sum l^2 and, from sum c l, S_R = sum (c - l)^2 = S - 2 sum c l + S_L
// (all below 2^32; modulo 2^32 on the way).
struct Side {
    uint32_t nl, sl, sr;
};

__device__ __forceinline__ uint32_t dot4(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_udot4(a, b, c, false);
}
__device__ __forceinline__ uint32_t dot2(uint32_t a, uint32_t b, uint32_t c) {
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_udot2(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b), c,
                                  false);
}
template <int FB>
__device__ __forceinline__ uint32_t dotf(uint32_t a, uint32_t b, uint32_t c) {
    if constexpr (FB == 8)
        return dot4(a, b, c);
    else
        return dot2(a, b, c);
}

// Field k of a packed side.
template <int FB>
__device__ __forceinline__ uint32_t pk_field(const uint32_t* l, int k) {
    constexpr int P = 32 / FB;
    return l[k / P] >> (FB * (k % P)) & ((1u << FB) - 1u);
}

template <int WORDS, int FB>
__device__ __forceinline__ Side side_of(const uint32_t* l, const uint32_t* c, uint32_t S) {
    Side s;
    uint32_t nl = 0, sl = 0, cl = 0;
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        nl = dotf<FB>(l[w], FB == 8 ? 0x01010101u : 0x00010001u, nl);
        sl = dotf<FB>(l[w], l[w], sl);
        cl = dotf<FB>(l[w], c[w], cl);
    }
    s.nl = nl;
    s.sl = sl;
    s.sr = S - 2u * cl + sl;
    return s;
}

// FP32 ranking score (both sides non-empty): relative error within 5u, as
// cand_q32 (the integers convert exactly for N < 256).
__device__ __forceinline__ float side_q32(const Side& s, uint32_t N) {
    return (float)s.sl * __builtin_amdgcn_rcpf((float)s.nl) +
           (float)s.sr * __builtin_amdgcn_rcpf((float)(N - s.nl));
}

// Q as an exact fraction: numerator S_L N_R + S_R N_L (below 2^25 for N < 256,
// 2^49 for N < 65536) over N_L N_R (below 2^14, 2^30); nd = 0: no candidate.
struct Frac {
    uint64_t nn;
    uint32_t nd;
};
__device__ __forceinline__ Frac side_frac(const Side& s, uint32_t N) {
    const uint32_t nr = N - s.nl;
    return Frac{(uint64_t)s.sl * nr + (uint64_t)s.sr * s.nl, s.nl * nr};
}
template <int FB>
__device__ __forceinline__ bool frac_better(const Frac& a, const Frac& b) {
    if constexpr (FB == 8)
        return a.nn * b.nd > b.nn * a.nd;
    else
        return (u128)a.nn * b.nd > (u128)b.nn * a.nd;
}
template <int FB>
__device__ __forceinline__ bool side_better(const Side& a, const Side& b, uint32_t N) {
    return frac_better<FB>(side_frac(a, N), side_frac(b, N));
}

// A histogram item's best threshold: FP32 score (negative: none) and bin.
struct ItemBest {
    float q;
    int b;
};

// Best threshold over the wave's candidates of one feature, NS per lane in
// any order (score q, threshold b, split side; ok: valid).
// With FP32 ranking the candidates within the margin of the wave's maximum are
// compared exactly, and not at all when they are one threshold; with exact
// ranking all are.  Ties keep the smaller threshold; without a candidate the
// score is negative and the bin 0.
template <int FB, int NS>
__device__ __forceinline__ ItemBest pick_threshold(const float* q, const int* b, const Side* sd,
                                                   const bool* ok, uint32_t N, int split_rank) {
    bool fin[NS];
    ItemBest r;
    r.q = -1.0f;
    r.b = 0;
    if (split_rank) {
        float q1 = q[0];
#pragma unroll
        for (int u = 1; u < NS; ++u) q1 = fmaxf(q1, q[u]);
        r.q = wave_max_f_dpp(q1);
        if (r.q < 0.0f) return r;
        const float fl = fp32_floor(r.q);
        bool any = false;
        int bf = 0;
#pragma unroll
        for (int u = NS - 1; u >= 0; --u) {
            fin[u] = q[u] >= fl;
            any |= fin[u];
            bf = fin[u] ? b[u] : bf;
        }
        r.b = __builtin_amdgcn_readlane(bf, (int)__ffsll((unsigned long long)__ballot(any)) - 1);
        bool other = false;
#pragma unroll
        for (int u = 0; u < NS; ++u) other |= fin[u] && b[u] != r.b;
        if (!__ballot(other)) return r;
    } else {
#pragma unroll
        for (int u = 0; u < NS; ++u) fin[u] = ok[u];
    }
    Frac best{0, 0};
    int bb = 0x7FFFFFFF;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        if (fin[u]) {
            const Frac c = side_frac(sd[u], N);
            if (best.nd == 0 || frac_better<FB>(c, best) ||
                (b[u] < bb && !frac_better<FB>(best, c))) {
                best = c;
                bb = b[u];
            }
        }
    }
#pragma unroll 1
    for (int m = 1; m < 64; m <<= 1) {  // seldom run with FP32 ranking: kept small
        Frac o;
        o.nn = __shfl_xor(best.nn, m);
        o.nd = __shfl_xor(best.nd, m);
        const int ob = __shfl_xor(bb, m);
        const bool take = o.nd != 0 && (best.nd == 0 || frac_better<FB>(o, best) ||
                                        (ob < bb && !frac_better<FB>(best, o)));
        if (take) {
            best = o;
            bb = ob;
        }
    }
    // no candidate: bin 0, as callers read the histogram at the bin they get
    const bool any = uniform(best.nd) != 0u;
    r.b = any ? (int)uniform((uint32_t)bb) : 0;
    if (!split_rank) r.q = any ? 1.0f : -1.0f;
    return r;
}

enum : int { kLeaf = 0, kSmall = 1, kLarge = 2 };

// Children of tree level d start at n_roots + 2 * (searched nodes of levels
// 0..d-1): every searched node owns a pair of child slots.
__device__ __forceinline__ uint32_t level_next_base(const ForestDev& F, int level) {
    uint64_t b = F.n_roots;
    for (int e = 0; e < level; ++e) b += 2ull * ((uint64_t)F.ctrs[e].n_small + F.ctrs[e].n_slots);
    return b < F.node_cap ? (uint32_t)b : F.node_cap;  // past the pool: splits flag overflow
}

// Work lists of tree level `level` as counted on the device; empty once a
// capacity overflow has been flagged for the level (the host reports it).
__device__ __forceinline__ uint32_t level_small(const ForestDev& F, int level) {
    const LevelCtr& c = F.ctrs[level];
    return c.overflow ? 0u : min(c.n_small, F.small_cap);
}
__device__ __forceinline__ uint32_t level_slots(const ForestDev& F, int level) {
    const LevelCtr& c = F.ctrs[level];
    return c.overflow ? 0u : min(c.n_slots, F.slot_cap);
}

// The launch-local view of the forest for tree level `level`: appends go to
// the next level's counters.
__device__ __forceinline__ ForestDev level_view(const ForestDev& F, int level) {
    ForestDev L = F;
    L.ctr = F.ctrs + level + 1;
    L.next_base = level_next_base(F, level);
    L.n_small_cur = F.ctrs[level].n_small;
    return L;
}

// Write a new node record -- a leaf until a split search turns it into a
// split -- and return what it needs next: nothing (final leaf: maximum depth,
// fewer than two row records or a single class), the wave path (up to
// small_rows records) or the histogram path.
__device__ inline int write_node(const ForestDev& F, const JobDev& J, uint32_t idx, uint32_t tree,
                                 uint32_t heap, uint32_t seg, uint32_t len, uint32_t n,
                                 uint32_t depth, const uint32_t* counts) {
    uint32_t arg = 0, nonzero = 0;
    for (int k = 0; k < J.K; ++k) {
        F.cls[(size_t)idx * F.kmax + k] = counts[k];
        if (counts[k] > counts[arg]) arg = k;
        nonzero += counts[k] != 0;
    }
    NodeDev nd;
    nd.tree = tree;
    nd.heap = heap;
    nd.seg = seg;
    nd.len = len;
    nd.n = n;
    nd.feat = -1;
    nd.left = 0;
    nd.thr = 0;
    nd.leaf_class = (uint8_t)arg;
    nd.depth = (uint8_t)depth;
    F.nodes[idx] = nd;
    F.ngain[idx] = 0;
    if ((int)depth >= J.D || len < 2 || nonzero <= 1) return kLeaf;
    return (len <= F.small_rows && n < F.small_ncap) ? kSmall : kLarge;
}

// Regression node: weight W and weighted target sum T (kept in the node's
// first two class words); it is a final leaf at the maximum depth or with
// fewer than two row records, else it takes the wave path (up to small_rows
// records) or the histogram path.  A leaf's prediction floor(T / W) is read
// from these fields.
__device__ inline int write_node_reg(const ForestDev& F, const JobDev& J, uint32_t idx,
                                     uint32_t tree, uint32_t heap, uint32_t seg, uint32_t len,
                                     uint32_t W, int64_t T, uint32_t depth) {
    F.cls[(size_t)idx * F.kmax] = (uint32_t)(uint64_t)T;
    F.cls[(size_t)idx * F.kmax + 1] = (uint32_t)((uint64_t)T >> 32);
    NodeDev nd;
    nd.tree = tree;
    nd.heap = heap;
    nd.seg = seg;
    nd.len = len;
    nd.n = W;
    nd.feat = -1;
    nd.left = 0;
    nd.thr = 0;
    nd.leaf_class = 0;
    nd.depth = (uint8_t)depth;
    F.nodes[idx] = nd;
    F.ngain[idx] = 0;
    if ((int)depth >= J.D || len < 2) return kLeaf;
    return len <= F.small_rows ? kSmall : kLarge;
}

// Weighted target sum of a regression node from its class words.
__device__ __forceinline__ int64_t node_tsum(const uint32_t* cls, int kmax, uint32_t idx) {
    return (int64_t)((uint64_t)cls[(size_t)idx * kmax] |
                     ((uint64_t)cls[(size_t)idx * kmax + 1] << 32));
}

// Place node idx in the next level's lists at already reserved positions.
__device__ inline void put_small(const ForestDev& F, uint32_t pos, uint32_t idx) {
    if (pos < F.small_cap)
        F.small_out[pos] = idx;
    else
        atomicOr(&F.ctr->overflow, 1u);
}

__device__ inline void put_large(const ForestDev& F, uint32_t slot, uint32_t idx) {
    if (slot >= F.slot_cap) {
        atomicOr(&F.ctr->overflow, 2u);
        return;
    }
    F.slot_node_out[slot] = idx;
}

// Reserve list positions for up to two new nodes (one atomic per list) and
// place them.
__device__ inline void enqueue_nodes(const ForestDev& F, const JobDev& J, uint32_t idx0,
                                     const int* kinds, int count) {
    uint32_t ns = 0, nl = 0;
    for (int c = 0; c < count; ++c) {
        ns += kinds[c] == kSmall;
        nl += kinds[c] == kLarge;
    }
    uint32_t ps = ns ? atomicAdd(&F.ctr->n_small, ns) : 0u;
    uint32_t pl = nl ? atomicAdd(&F.ctr->n_slots, nl) : 0u;
    for (int c = 0; c < count; ++c) {
        if (kinds[c] == kSmall) put_small(F, ps++, idx0 + c);
        if (kinds[c] == kLarge) put_large(F, pl++, idx0 + c);
    }
}

// Children of the i-th searched node of a level (small nodes first, then
// large-node slots) live at next_base + 2 i: no allocation counter.  A
// searched node that stays a leaf marks its pair unused.
__device__ inline void mark_unused_pair(const ForestDev& F, uint32_t child) {
    if (child + 2 <= F.node_cap) {
        F.nodes[child].tree = 0xFFFFFFFFu;
        F.nodes[child + 1].tree = 0xFFFFFFFFu;
    }
}

// Turn node `id` into a split on (best.f, best.b) and write both children
// at child, child + 1; kinds[] receives what each child needs next.
__device__ inline void split_node(const ForestDev& F, JobDev& J, const TreeDev& tr, uint32_t id,
                                  const NodeDev& nd, const Cand& best, uint32_t nl_rows,
                                  const uint32_t* cl, const uint32_t* cr, uint64_t gain,
                                  uint32_t child, int* kinds) {
    kinds[0] = kinds[1] = kLeaf;
    if (child + 2 > F.node_cap) {
        atomicOr(&F.ctr->overflow, 4u);
        return;  // stays a leaf; the host reports the failure
    }
    F.nodes[id].feat = best.f;
    F.nodes[id].thr = (uint16_t)best.b;
    F.nodes[id].left = child;
    F.ngain[id] = gain;
    if (J.mode == 0)
        atomicAdd((unsigned long long*)&J.G[(size_t)tr.tau * J.pw_cap + best.f],
                  (unsigned long long)gain);
    kinds[0] = write_node(F, J, child, nd.tree, 2 * nd.heap, nd.seg, nl_rows, best.nl,
                          nd.depth + 1u, cl);
    kinds[1] = write_node(F, J, child + 1, nd.tree, 2 * nd.heap + 1, nd.seg + nl_rows,
                          nd.len - nl_rows, best.nr, nd.depth + 1u, cr);
}

// Regression form of split_node: the children's weights and target sums
// come from the winning candidate.
__device__ inline void split_node_reg(const ForestDev& F, JobDev& J, const TreeDev& tr,
                                      uint32_t id, const NodeDev& nd, const Cand& best,
                                      uint32_t nl_rows, uint64_t gain, uint32_t child,
                                      int* kinds) {
    kinds[0] = kinds[1] = kLeaf;
    if (child + 2 > F.node_cap) {
        atomicOr(&F.ctr->overflow, 4u);
        return;
    }
    F.nodes[id].feat = best.f;
    F.nodes[id].thr = (uint16_t)best.b;
    F.nodes[id].left = child;
    F.ngain[id] = gain;
    if (J.mode == 0)
        atomicAdd((unsigned long long*)&J.G[(size_t)tr.tau * J.pw_cap + best.f],
                  (unsigned long long)gain);
    kinds[0] = write_node_reg(F, J, child, nd.tree, 2 * nd.heap, nd.seg, nl_rows, best.nl,
                              reg_tl(best), nd.depth + 1u);
    kinds[1] = write_node_reg(F, J, child + 1, nd.tree, 2 * nd.heap + 1, nd.seg + nl_rows,
                              nd.len - nl_rows, best.nr, reg_tr(best), nd.depth + 1u);
}

}  // namespace boruta
