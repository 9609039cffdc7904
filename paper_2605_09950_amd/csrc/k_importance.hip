// k_importance.hip -- importance scores, hits and decisions (gfx950).
//
//   * TreeImp (Algorithm 2, Sec. 2.1): per tree, each widened column's summed
//     fixed-point Gini decrease G (accumulated at split time) is normalised
//     to floor(2^44 G / sum_f G) and the shares are summed over trees; the
//     mean's 1/T cancels in the final renormalisation.
//   * Permut (Kursa's accuracy drop, Sec. 2; Sec. 2.2): for every tree, OOB
//     row j, column f on the row's path and replica r, the row is re-routed
//     with f's bin taken from OOB row pi(j), pi the keyed permutation of the
//     tree's OOB rows for (t, tree, f, r); the drop in correct predictions is
//     summed per column.  Columns off the path cannot change the prediction,
//     so only path columns are re-routed, from their first node on the path.
//   * KL permutation importance (Algorithm 3, Sec. 2.2; importance mode 2):
//     the forest's class distribution for row r is the sum over trees of
//     floor(2^32 c_k / N) at the leaf r reaches; one keyed row permutation
//     pi per iteration serves every column, whose bin at row r is replaced
//     by the bin at row pi(r); the column scores the sum over rows of
//     KL(P || Q) in bits with 32 fractional bits (a class Q misses while P
//     has it counts one unit).  Again only the columns on a row's path in a
//     tree can move it to another leaf of that tree: per (row, tree) those
//     columns are re-routed and the leaf differences accumulated per
//     (column, row); rows are taken in blocks that bound that buffer.
//   * hits (strictly above the best shadow) and the binomial decision;
//   * Algorithm 1's final ranking: confirmed 1, undecided 2, rejected from 3
//     by descending historical importance (the mean of the feature's finite
//     history entries, summed in iteration order; equal means share a rank).
#include <cstddef>

#include "dev_common.hpp"
#include "reg_dev.hpp"

namespace boruta {

// Per tree: total fixed-point decrease over its columns.
__global__ __launch_bounds__(256) void k_tree_totals(JobDev* jobs, const TreeDev* trees,
                                                     uint64_t* tot) {
    __shared__ unsigned long long s[4];
    const TreeDev tr = trees[blockIdx.x];
    const JobDev& J = jobs[tr.job];
    if (!J.live || J.mode != 0) return;  // finished job, or Permut job of a mixed batch
    const uint64_t* G = J.G + (size_t)tr.tau * J.pw_cap;
    unsigned long long v = 0;
    for (int f = threadIdx.x; f < J.p_w; f += 256) v += G[f];
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) tot[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}

// Per (column, tree): I_f += floor(2^44 G[tree][f] / total of the tree),
// summed with 64-bit integer atomics (exact in any order).  G is cleared
// behind the read, ready for the next iteration.
__global__ __launch_bounds__(256) void k_treeimp(JobDev* jobs, const TreeDev* trees,
                                                 const uint64_t* tot) {
    const uint32_t g = blockIdx.y;
    const TreeDev tr = trees[g];
    JobDev& J = jobs[tr.job];
    const int f = blockIdx.x * 256 + threadIdx.x;
    if (!J.live || J.mode != 0 || f >= J.p_w) return;
    uint64_t* Gp = J.G + (size_t)tr.tau * J.pw_cap + f;
    const uint64_t gv = ldg(Gp);
    if (gv == 0) return;
    *Gp = 0;
    atomicAdd((unsigned long long*)&J.imp[f],
              (unsigned long long)udiv128((u128)gv << 44, (u128)tot[g]));
}

// Prediction of a regression leaf: floor(T / W), T in the node's first two
// class words and W its weighted count.
__device__ __forceinline__ long long leaf_pred(const NodeDev* nodes, const uint32_t* cls, int kmax,
                                               uint32_t node) {
    const int64_t T = (int64_t)((uint64_t)cls[(size_t)node * kmax] |
                                ((uint64_t)cls[(size_t)node * kmax + 1] << 32));
    return (long long)reg_pred(T, nodes[node].n);
}

// floor((y_fix - pred)^2 / 2^s_perm) (|y_fix - pred| < 2^40).
__device__ __forceinline__ long long sq_error_fix(const NodeDev* nodes, const uint32_t* cls,
                                                  int kmax, uint32_t node, long long yfix,
                                                  int s_perm) {
    const long long e = yfix - leaf_pred(nodes, cls, kmax, node);
    const u128 a = (u128)(uint64_t)(e < 0 ? -e : e);
    return (long long)((a * a) >> s_perm);
}

// What a walk needs of a node: one 16-byte load.
struct Hop {
    int32_t feat;       // widened column, negative for a leaf
    uint32_t left;      // left child; the right one is left + 1
    uint32_t thr, leaf; // threshold bin, leaf class
};
__device__ __forceinline__ Hop load_hop(const NodeDev* nodes, uint32_t node) {
    static_assert(sizeof(NodeDev) == 32 && offsetof(NodeDev, n) == 16, "node record layout");
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = ldg(reinterpret_cast<const u32x4*>(nodes + node) + 1);
    return Hop{(int32_t)v[1], v[2], v[3] & 0xFFFFu, v[3] >> 16 & 0xFFu};
}

// A thread's walk from a root, kept in LDS by position (stride 256): column
// and direction, the child not taken, the threshold bin.  A permuted column
// changes the row's prediction only where its new bin turns the other way at
// one of its positions, and then from the child not taken on: positions that
// keep the direction need no walk, and a turned one none of the nodes above.
struct PathLds {
    uint32_t* pf;  // [depth][256] column | went left << 31
    uint32_t* ps;  // [depth][256] the child not taken
    uint8_t* pt;   // [depth][256] threshold bin
};
__host__ __device__ constexpr uint32_t path_lds_words(int max_depth) {
    return (uint32_t)max_depth * 256u * 2u + (uint32_t)max_depth * 64u;
}
__device__ __forceinline__ PathLds path_lds(uint32_t* s, int max_depth) {
    return PathLds{s, s + max_depth * 256, reinterpret_cast<uint8_t*>(s + max_depth * 512)};
}
struct Walked {
    uint32_t leaf, leaf_class;
    int len;
    uint32_t dup;  // positions whose column is on the path before (depth <= 30)
};
__device__ __forceinline__ Walked walk_path(const JobDev& J, const NodeDev* nodes, uint32_t node,
                                            uint32_t row, const PathLds& P, int tid) {
    Walked w{node, 0u, 0, 0u};
    Hop h = load_hop(nodes, node);
    while (h.feat >= 0) {
        const bool left = (uint32_t)ldg(ldg(J.colptr + h.feat) + row) <= h.thr;
        bool dup = false;
        for (int q = 0; q < w.len; ++q)
            dup |= (P.pf[q * 256 + tid] & 0x7FFFFFFFu) == (uint32_t)h.feat;
        w.dup |= (uint32_t)dup << w.len;
        P.pf[w.len * 256 + tid] = (uint32_t)h.feat | (uint32_t)left << 31;
        P.ps[w.len * 256 + tid] = left ? h.left + 1u : h.left;
        P.pt[w.len * 256 + tid] = (uint8_t)h.thr;
        ++w.len;
        w.leaf = left ? h.left : h.left + 1u;
        h = load_hop(nodes, w.leaf);
    }
    w.leaf_class = h.leaf;
    return w;
}
// The child from which the row's walk differs when the column first met at
// position a takes bin sb; 0xFFFFFFFF when it does not (roots are never a child).
__device__ __forceinline__ uint32_t turned_at(const PathLds& P, const Walked& w, int a,
                                              uint32_t sb, int tid) {
    const uint32_t e = P.pf[a * 256 + tid], f = e & 0x7FFFFFFFu;
    if ((sb <= P.pt[a * 256 + tid]) != (bool)(e >> 31)) return P.ps[a * 256 + tid];
    // later positions of the same column
    for (uint32_t m = a < 31 ? w.dup >> (a + 1) << (a + 1) : 0u; m; m &= m - 1u) {
        const int q = __builtin_ctz(m);
        const uint32_t g = P.pf[q * 256 + tid];
        if ((g & 0x7FFFFFFFu) == f && (sb <= P.pt[q * 256 + tid]) != (bool)(g >> 31))
            return P.ps[q * 256 + tid];
    }
    return 0xFFFFFFFFu;
}

// (path column, replica) pairs whose OOB sources are walked together
constexpr int kPermGroup = 8;
// walks a lane advances at a time
constexpr int kPermWalks = 4;

// A k_permut workgroup's paths by position (stride: the workgroup's threads);
// directions are kept in a register.
template <class Col>
struct PermPath {
    uint32_t* ps;  // the child not taken
    Col* pf;       // column
    uint8_t* pt;   // threshold bin
    uint32_t stride;
};
template <class Col>
__host__ __device__ constexpr uint32_t perm_path_bytes(int max_depth, uint32_t threads) {
    return (uint32_t)max_depth * threads * (4u + (uint32_t)sizeof(Col) + 1u);
}

// Permut: one thread per (tree, OOB row).  The row's path is walked once and
// kept in LDS: a permuted column changes the prediction only where its new bin
// turns the other way at one of its positions, and then from the child not
// taken on.  The row's (path column, replica) pairs are taken kPermGroup at a
// time: their source rows pi(j) by cycle walks interleaved in one loop, then
// all their source bins, then -- for the pairs that turn at a node -- the walks
// from there, kPermWalks at a time, a lane starting its next pair's walk as
// soon as one ends.  When the job's widened width is at most lds_cols, the
// drops are summed per column in LDS and each workgroup adds its nonzero sums
// to the importances: once most columns are decided, few remain and per-row
// atomics would all meet on them.  For a regression job a row's score is the
// negated squared error against its leaf's prediction, sq_error_fix above, and
// the per-column sums in LDS are 64-bit.
// Bound: the chains of dependent loads (node, column address, bin) of the walks
// beside the permutations' multiplies, and for a matrix past the last-level
// cache the 128-byte lines of its scattered bins.  So: one tree per XCD at a
// time (consecutive workgroups go to the 8 XCDs in turn), whose nodes and bins
// then stay in that XCD's L2 (100,000 x 2,000, 300 trees of depth 16, five
// replicas: 2.6e9 -> 1.7e9 lines); four walks per lane; 128 rows per workgroup
// and 7 bytes per path position, for 20 waves per compute unit; the positions
// of a row dealt to up to 8 workgroups where the rows alone leave the chip idle
// (each walks the path again).  An iteration's time with one walk per lane, any
// XCD, 256 rows and 9 bytes, and now: 100,000 x 2,000 80.0 -> 54.4 ms; 10,000 x
// 500, 200 trees 455 -> 305 us; 64 jobs up to 5,000 x 2,000 6.2 -> 3.4 ms; 3,000
// x 120, 60 trees 199 -> 133 us.  Rounds of the permutations tabulated in LDS
// for the rows of one node (sorted by path) saved 35% of the multiplies and
// lost the time again in barriers and occupancy.
template <class Col>
__global__ __launch_bounds__(128) void k_permut(JobDev* jobs, const TreeDev* trees, int n_trees,
                                                const NodeDev* nodes, const uint32_t* cls,
                                                int kmax, int max_depth, int slices,
                                                int lds_cols, int lds_words,
                                                unsigned long long* visits) {
    // [kPermGroup][threads]: a group's source rows, then its walks' first nodes;
    // the column drops (lds_words); the paths
    extern __shared__ uint32_t s_perm[];
    const uint32_t S = blockDim.x;
    // grid: x = (chunk, slice) times the 8 XCDs, y = eighths of the trees
    const uint32_t g = blockIdx.y * 8u + blockIdx.x % 8u;
    if (g >= (uint32_t)n_trees) return;
    const uint32_t slice = blockIdx.x / 8u % (uint32_t)slices;
    const uint32_t chunk = blockIdx.x / 8u / (uint32_t)slices;
    const TreeDev tr = trees[g];
    JobDev& J = jobs[tr.job];
    if (!J.live || J.mode != 1) return;  // finished job, or TreeImp job of a mixed batch
    const uint32_t tid = threadIdx.x;
    const uint32_t m = (uint32_t)J.tstat[tr.tau * 4 + 1];
    if (chunk * S >= m) return;
    uint32_t* g_src = s_perm;
    int* s_drop = reinterpret_cast<int*>(g_src + kPermGroup * S);
    long long* s_drop64 = reinterpret_cast<long long*>(s_drop);  // regression jobs
    PermPath<Col> P;
    P.stride = S;
    P.ps = reinterpret_cast<uint32_t*>(s_drop) + lds_words;
    P.pf = reinterpret_cast<Col*>(P.ps + (uint32_t)max_depth * S);
    P.pt = reinterpret_cast<uint8_t*>(P.pf + (uint32_t)max_depth * S);
    const bool reg = J.reg != 0;
    const bool lds = J.p_w <= lds_cols;  // uniform: one tree per workgroup
    if (lds) {
        for (uint32_t c = tid; c < (uint32_t)J.p_w; c += S) {
            if (reg)
                s_drop64[c] = 0;
            else
                s_drop[c] = 0;
        }
    }
    const uint32_t j = chunk * S + tid;
    const bool active = j < m;
    const uint32_t* oob = J.oob + (size_t)tr.tau * J.n;
    const uint32_t row = active ? oob[j] : 0u;
    const uint32_t yv = reg ? 0u : (uint32_t)J.y[row];
    const long long yfv = reg ? (long long)J.yfix[row] : 0ll;
    // the path: its length, its directions from the top bit (1: right), and the
    // positions whose column is on it before (depth <= 30)
    int len = 0;
    uint32_t dir = 0u, dup = 0u;
    bool base_ok = false;
    long long base_err = 0;
    unsigned long long nv = 0;  // node visits (statistics)
    if (active) {
        uint32_t leaf = g;
        Hop h = load_hop(nodes, g);
        while (h.feat >= 0) {
            const uint32_t right = (uint32_t)ldg(ldg(J.colptr + h.feat) + row) > h.thr ? 1u : 0u;
            bool again = false;
            for (int q = 0; q < len; ++q) again |= P.pf[q * S + tid] == (Col)h.feat;
            dup |= (uint32_t)again << len;
            dir |= right << (31 - len);
            P.pf[len * S + tid] = (Col)h.feat;
            P.ps[len * S + tid] = h.left + (right ^ 1u);
            P.pt[len * S + tid] = (uint8_t)h.thr;
            ++len;
            leaf = h.left + right;
            h = load_hop(nodes, leaf);
        }
        if (slice == 0u) nv += (unsigned long long)len + 1u;
        if (reg)
            base_err = sq_error_fix(nodes, cls, kmax, leaf, yfv, J.s_perm);
        else
            base_ok = h.leaf == yv;
    }
    const unsigned long long okm = __ballot(active && base_ok && slice == 0u);
    if ((tid & 63) == 0 && okm) atomicAdd(&J.tstat[tr.tau * 4 + 2], (int)__popcll(okm));
    if (lds) __syncthreads();
    const uint32_t R = (uint32_t)J.R;
    KeyedPerm K = make_perm(J.seed_lo, J.seed_hi, kOobPerm, (uint32_t)J.t, (uint32_t)tr.tau, 0u,
                            0u, (uint64_t)m);
    // whether the column of position a with bin sb sends the row another way:
    // the child from which its walk differs, else 0xFFFFFFFF (roots are never a child)
    auto turned_to = [&](int a, uint32_t sb) -> uint32_t {
        const uint32_t f = P.pf[a * S + tid];
        if ((uint32_t)(sb > P.pt[a * S + tid]) != (dir >> (31 - a) & 1u)) return P.ps[a * S + tid];
        for (uint32_t q = a < 31 ? dup >> (a + 1) << (a + 1) : 0u; q; q &= q - 1u) {
            const int b = __builtin_ctz(q);
            if (P.pf[b * S + tid] == (Col)f &&
                (uint32_t)(sb > P.pt[b * S + tid]) != (dir >> (31 - b) & 1u))
                return P.ps[b * S + tid];
        }
        return 0xFFFFFFFFu;
    };
    auto add_drop = [&](uint32_t f, int drop, long long drop_sq) {
        if (reg) {
            if (drop_sq) {
                if (lds)
                    atomicAdd((unsigned long long*)&s_drop64[f], (unsigned long long)drop_sq);
                else
                    atomicAdd((unsigned long long*)&J.imp[f], (unsigned long long)drop_sq);
            }
        } else if (drop) {
            if (lds)
                atomicAdd(&s_drop[f], drop);
            else
                atomicAdd((unsigned long long*)&J.imp[f], (unsigned long long)(int64_t)drop);
        }
    };
    // scores a group: k pairs, their source positions in g_src, the path
    // positions of their columns in bytes of pos
    auto score = [&](int k, uint64_t pos) {
        // source bins: the rows' loads, then the bins' loads, all in flight
        uint32_t srow[kPermGroup];
        uint64_t sbs = 0;
#pragma unroll
        for (int e = 0; e < kPermGroup; ++e) srow[e] = ldg(oob + (e < k ? g_src[e * S + tid] : 0u));
        uint32_t sb[kPermGroup];
#pragma unroll
        for (int e = 0; e < kPermGroup; ++e) {
            const uint32_t f = P.pf[(uint32_t)(pos >> (8 * e) & 0xFFu) * S + tid];
            sb[e] = ldg(ldg(J.colptr + f) + srow[e]);
        }
        // the pairs that turn, and where their walks go on
        uint32_t turn = 0;
#pragma unroll
        for (int e = 0; e < kPermGroup; ++e) {
            sbs |= (uint64_t)sb[e] << (8 * e);
            if (e < k) {
                const uint32_t at = turned_to((int)(pos >> (8 * e) & 0xFFu), sb[e]);
                g_src[e * S + tid] = at;
                turn |= (uint32_t)(at != 0xFFFFFFFFu) << e;
            }
        }
        // their walks, kPermWalks at a time
        uint32_t f[kPermWalks], node[kPermWalks], sbin[kPermWalks];
        bool on[kPermWalks];
        auto begin = [&](int v) {
            on[v] = turn != 0u;
            const int e = on[v] ? __builtin_ctz(turn) : 0;
            turn &= turn - 1u;
            f[v] = P.pf[(uint32_t)(pos >> (8 * e) & 0xFFu) * S + tid];
            node[v] = on[v] ? g_src[e * S + tid] : g;
            sbin[v] = (uint32_t)(sbs >> (8 * e)) & 0xFFu;
        };
        bool any = false;
#pragma unroll
        for (int v = 0; v < kPermWalks; ++v) {
            begin(v);
            any |= on[v];
        }
        while (any) {
            any = false;
            Hop h[kPermWalks];
            uint32_t b[kPermWalks];
#pragma unroll
            for (int v = 0; v < kPermWalks; ++v) h[v] = load_hop(nodes, node[v]);
#pragma unroll
            for (int v = 0; v < kPermWalks; ++v)
                b[v] = ldg(ldg(J.colptr + (h[v].feat >= 0 ? h[v].feat : 0)) + row);
#pragma unroll
            for (int v = 0; v < kPermWalks; ++v) {
                nv += on[v];
                if (h[v].feat >= 0) {
                    if ((uint32_t)h[v].feat == f[v]) b[v] = sbin[v];
                    if (on[v]) node[v] = b[v] <= h[v].thr ? h[v].left : h[v].left + 1u;
                } else if (on[v]) {
                    if (reg)
                        add_drop(f[v], 0,
                                 sq_error_fix(nodes, cls, kmax, node[v], yfv, J.s_perm) -
                                     base_err);
                    else
                        add_drop(f[v], (int)base_ok - (int)(h[v].leaf == yv), 0);
                    begin(v);
                }
                any |= on[v];
            }
        }
    };
    uint32_t done = dup;  // positions that need no more pairs here
    if (slices > 1)
        for (uint32_t l = 0; l < (uint32_t)len; ++l)
            if (l % (uint32_t)slices != slice) done |= 1u << l;
    uint32_t left = active ? ~done & ((1u << len) - 1u) : 0u;
    uint32_t cr = 0;
    while (left) {
        uint64_t pos = 0;
        int k = 0;
        uint32_t x = j;
        int a = __builtin_ctz(left);
        K.b = P.pf[a * S + tid];
        K.c_hi = cr << 16;
        while (k < kPermGroup && left) {
            if (m > 1u) x = perm_pass(K, x);
            if (m <= 1u || x < m) {
                g_src[k * S + tid] = m <= 1u ? 0u : x;
                pos |= (uint64_t)a << (8 * k);
                ++k;
                if (++cr == R) {
                    cr = 0;
                    left &= left - 1u;
                }
                x = j;
                if (left) {
                    a = __builtin_ctz(left);
                    K.b = P.pf[a * S + tid];
                    K.c_hi = cr << 16;
                }
            }
        }
        score(k, pos);
    }
    if (lds) {
        __syncthreads();
        for (uint32_t c = tid; c < (uint32_t)J.p_w; c += S) {
            const long long v = reg ? s_drop64[c] : (long long)s_drop[c];
            if (v) atomicAdd((unsigned long long*)&J.imp[c], (unsigned long long)v);
        }
    }
    if (visits) {
        for (int q = 1; q < 64; q <<= 1) nv += __shfl_xor(nv, q);
        if ((tid & 63) == 0 && nv)
            atomicAdd(visits + ((blockIdx.x * 8u + (tid >> 6)) & (kAlgWords - 1)), nv);
    }
}

// ---------------------------------------------------------------------------
// KL permutation importance.

// Fixed-point class frequency of a leaf, floor(2^32 c / N), with inv = 1.0 / N:
// the product is within one of the quotient (2^33 2^-52 < 1) and put right by
// its remainder; a 64-bit division takes about four times its instructions.
__device__ __forceinline__ uint64_t leaf_freq(uint32_t c, uint32_t N, double inv) {
    const uint64_t num = (uint64_t)c << 32;
    uint64_t q = (uint64_t)((double)c * 4294967296.0 * inv);
    const int64_t rem = (int64_t)(num - q * N);
    if (rem < 0) --q;
    if (rem >= (int64_t)N) ++q;
    return q;
}

__device__ __forceinline__ uint32_t leaf_weight(const uint32_t* cls, int kmax, uint32_t node,
                                                int K) {
    uint32_t N = 0;
    for (int k = 0; k < K; ++k) N += cls[(size_t)node * kmax + k];
    return N;
}

// 2^32 log2(x), 1 <= x < 2^62: bit length, then 32 digits of the fraction
// from successive squares of the mantissa (62 fractional bits, truncated).
// The digits are those of log2 but for an error below 2^-28 of the last one
// (32 truncated squares), so they are taken from the FP64 logarithm (error below
// 2^-51, that is 2^-19 of the last digit) wherever that is 2^-16 or more from
// a change of the last digit: the loop is left to one value in 32,768.
// k_kl_reduce at 10,000 x 500: 612 -> 212 us.
__device__ __forceinline__ uint64_t lg2_q32(uint64_t x) {
    const int e = 63 - __builtin_clzll(x);
    uint64_t m = x << (62 - e);
    const uint64_t whole = (uint64_t)e << 32;
    if (m == (uint64_t)1 << 62) return whole;
    const double t = log2((double)m * 0x1p-62) * 4294967296.0;
    const double down = floor(t), part = t - down;
    if (part >= 0x1p-16 && part <= 1.0 - 0x1p-16) return whole | (uint32_t)down;
    uint64_t frac = 0;
    for (int i = 0; i < 32; ++i) {
        const uint64_t hi = __umul64hi(m, m), lo = m * m;
        m = (hi << 2) | (lo >> 62);
        const uint64_t top = m >> 63;
        frac = (frac << 1) | top;
        m >>= top;
    }
    return whole | frac;
}

// KL(P || Q) in 2^-32 bits for summed fixed-point frequencies S (P) and
// Sq (Q), Q's missing classes raised to one unit where P has them:
// floor(sum_k S_k (lg S_k - lg Q_k) / sum S) + lg sum Q - lg sum S.
// lgS[k] = lg S_k (where S_k > 0) and lgsum = lg sum S come with P: a row's
// P is shared by every column.
template <int KMAX>
__device__ int64_t kl_q32(const uint64_t* S, const uint64_t* lgS, uint64_t lgsum,
                          const uint64_t* Sq, int K) {
    u128 pos = 0, neg = 0;
    uint64_t sp = 0, sq = 0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        if (k >= K) break;
        const uint64_t q = (Sq[k] == 0 && S[k] != 0) ? 1 : Sq[k];
        sp += S[k];
        sq += q;
        if (S[k]) {
            const uint64_t a = lgS[k], b = q == S[k] ? a : lg2_q32(q);
            if (a >= b)
                pos += (u128)S[k] * (a - b);
            else
                neg += (u128)S[k] * (b - a);
        }
    }
    int64_t first;
    if (pos >= neg) {
        first = (int64_t)udiv128(pos - neg, (u128)sp);
    } else {  // floor of a negative quotient
        const u128 m = neg - pos;
        const uint64_t qt = udiv128(m, (u128)sp);
        first = -(int64_t)qt - (((u128)qt * sp != m) ? 1 : 0);
    }
    return first + (int64_t)(sq == sp ? lgsum : lg2_q32(sq)) - (int64_t)lgsum;
}

// Rows [r0, r0 + rb) of job J, 64 per workgroup, a lane each; the 16 waves deal
// the job's trees among them, four walks in flight per lane (near a root the
// lanes share nodes, and read neighbouring bins of one column).  Writes the
// row's summed leaf frequencies S_k, their lg S_k and lg sum S (S[row][2K + 1]),
// and pi(row).  With a wave per row and a tree per lane 10,000 rows through 200
// trees of depth 12 took 393 us; this takes 151.
template <int KMAX>
__global__ __launch_bounds__(1024) void k_kl_base(JobDev* jobs, int j, const NodeDev* nodes,
                                                  const uint32_t* cls, int kmax, uint32_t tree0,
                                                  uint32_t r0, uint32_t rb, uint64_t* S,
                                                  uint32_t* pi) {
    __shared__ unsigned long long s_acc[KMAX][64];
    const JobDev& J = jobs[j];
    if (!J.live) return;
    const int lane = threadIdx.x & 63, wave = (int)(threadIdx.x >> 6);
    const uint32_t rr = blockIdx.x * 64u + (uint32_t)lane;
    const bool mine = rr < rb && r0 + rr < (uint32_t)J.n;
    const uint32_t row = mine ? r0 + rr : r0;
    const int K = J.K;
    if (wave == 0 && mine) {
        const KeyedPerm P = make_perm(J.seed_lo, J.seed_hi, kFlush, (uint32_t)J.t, 0u, 0u, 0u,
                                      (uint64_t)J.n);
        pi[rr] = perm_apply(P, row);
    }
    if (J.reg) return;  // regression: the loss depends on the change of the prediction only
    for (int i = (int)threadIdx.x; i < KMAX * 64; i += 1024) s_acc[i >> 6][i & 63] = 0ull;
    __syncthreads();
    uint64_t acc[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) acc[k] = 0;
    for (int t0 = wave * 4; t0 < J.T; t0 += 64) {
        uint32_t node[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) node[v] = tree0 + (uint32_t)min(t0 + v, J.T - 1);
        for (bool any = true; any;) {
            any = false;
            Hop h[4];
            uint32_t b[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) h[v] = load_hop(nodes, node[v]);
#pragma unroll
            for (int v = 0; v < 4; ++v) b[v] = ldg(ldg(J.colptr + max(h[v].feat, 0)) + row);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (h[v].feat >= 0) {
                    node[v] = b[v] <= h[v].thr ? h[v].left : h[v].left + 1u;
                    any = true;
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (t0 + v >= J.T) break;
            const uint32_t N = leaf_weight(cls, kmax, node[v], K);
            const double inv = 1.0 / (double)N;
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if (k < K) acc[k] += leaf_freq(cls[(size_t)node[v] * kmax + k], N, inv);
        }
    }
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k < K) atomicAdd(&s_acc[k][lane], (unsigned long long)acc[k]);
    __syncthreads();
    if (!mine) return;
    // the logarithms: one class (or the sum) per wave
    uint64_t* row_out = S + (size_t)rr * (2 * K + 1);
    for (int k = wave; k <= K; k += 16) {
        uint64_t v = 0;
        if (k < K) {
            v = s_acc[k][lane];
            row_out[k] = v;
        } else {
            for (int q = 0; q < K; ++q) v += s_acc[q][lane];
        }
        row_out[K + k] = v ? lg2_q32(v) : 0ull;
    }
}

// One thread per (tree, row of the block), rows fastest so that a wave
// walks one tree for 64 rows (its node and bin loads and its atomics then
// spread over rows, not over trees meeting at one column): the row's path;
// for each column on it whose bin at row pi(row) turns the other way at one of
// the column's positions, the row is re-routed from there, and the leaf adds
// its frequency difference to delta[column][row][k] (64-bit two's complement).
// Bound: the address units, by the scattered loads of the walks (a wave's 480
// load instructions took 1.23 ms at 10,000 x 500, 200 trees; now four walks
// advance at a time, a finished one reads the root, and a leaf's counts are read
// once: 0.80 ms).  Which rows or trees share an XCD makes no difference there.
template <int KMAX>
__global__ __launch_bounds__(256) void k_kl_delta(JobDev* jobs, int j, const NodeDev* nodes,
                                                  const uint32_t* cls, int kmax, uint32_t tree0,
                                                  uint32_t r0, uint32_t rb, const uint32_t* pi,
                                                  unsigned long long* delta, int max_depth) {
    extern __shared__ uint32_t s_path[];  // the paths; [max_depth][256] source bins
    const JobDev& J = jobs[j];
    if (!J.live) return;
    const int tid = threadIdx.x;
    // one tree per XCD at a time (workgroups go to the 8 XCDs in turn)
    const uint32_t T = (uint32_t)J.T, per = (rb + 255u) / 256u;
    const uint32_t idx = blockIdx.x / 8u;
    const uint32_t tau = idx / per * 8u + blockIdx.x % 8u, rr = idx % per * 256u + (uint32_t)tid;
    if (tau >= T || rr >= rb || r0 + rr >= (uint32_t)J.n) return;
    const uint32_t row = r0 + rr, src = pi[rr];
    const int K = J.K;
    const PathLds P = path_lds(s_path, max_depth);
    uint8_t* s_bin = reinterpret_cast<uint8_t*>(s_path + path_lds_words(max_depth));
    const Walked w = walk_path(J, nodes, tree0 + tau, row, P, tid);
    // a leaf's class frequencies, each count read once
    auto freqs = [&](uint32_t node, uint64_t (&q)[KMAX]) {
        uint32_t c[KMAX], N = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) c[k] = ldg(cls + (size_t)node * kmax + min(k, K - 1));
#pragma unroll
        for (int k = 0; k < KMAX; ++k) N += k < K ? c[k] : 0u;
        const double inv = 1.0 / (double)N;
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
            if (k < K) q[k] = leaf_freq(c[k], N, inv);
    };
    uint64_t q0[KMAX];
    if (!J.reg) freqs(w.leaf, q0);
    // the columns' source bins, eight positions' loads in flight
    for (int a0 = 0; a0 < w.len; a0 += 8) {
        uint32_t sb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int a = min(a0 + e, w.len - 1);
            sb[e] = ldg(ldg(J.colptr + (P.pf[a * 256 + tid] & 0x7FFFFFFFu)) + src);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (a0 + e < w.len) s_bin[(a0 + e) * 256 + tid] = (uint8_t)sb[e];
    }
    // Four positions at a time over the wave's rows, the atomics position by
    // position (near the root they hold one column, and those of neighbouring
    // rows share lines; one loop over each lane's own columns took twice the time).
    for (int a0 = 0; a0 < w.len; a0 += 4) {
        uint32_t node[4], leaf[4], f[4], sb[4];
        bool turned[4], on[4];
        bool any = false;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int a = min(a0 + v, w.len - 1);
            sb[v] = s_bin[a * 256 + tid];
            f[v] = P.pf[a * 256 + tid] & 0x7FFFFFFFu;
            const uint32_t at = a0 + v < w.len && !(w.dup >> a & 1u)
                                    ? turned_at(P, w, a, sb[v], tid)
                                    : 0xFFFFFFFFu;
            turned[v] = at != 0xFFFFFFFFu;
            node[v] = turned[v] ? at : tree0 + tau;
            leaf[v] = w.leaf;
            on[v] = turned[v];
            any |= turned[v];
        }
        while (any) {
            any = false;
            Hop h[4];
            uint32_t b[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) h[v] = load_hop(nodes, node[v]);
#pragma unroll
            for (int v = 0; v < 4; ++v) b[v] = ldg(ldg(J.colptr + max(h[v].feat, 0)) + row);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (on[v] && h[v].feat >= 0) {
                    if ((uint32_t)h[v].feat == f[v]) b[v] = sb[v];
                    node[v] = b[v] <= h[v].thr ? h[v].left : h[v].left + 1u;
                    any = true;
                } else if (on[v]) {  // its lane reads the root from here on, as its
                    leaf[v] = node[v];  // neighbours do: one line
                    node[v] = tree0 + tau;
                    on[v] = false;
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (!turned[v] || leaf[v] == w.leaf) continue;
            unsigned long long* d = delta + ((size_t)f[v] * rb + rr) * K;
            if (J.reg) {  // change of the leaf's prediction, in the first slot
                const long long dv =
                    leaf_pred(nodes, cls, kmax, leaf[v]) - leaf_pred(nodes, cls, kmax, w.leaf);
                if (dv) atomicAdd(d, (unsigned long long)dv);
                continue;
            }
            uint64_t q1[KMAX];
            freqs(leaf[v], q1);
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if (k < K && q1[k] != q0[k]) atomicAdd(d + k, (unsigned long long)(q1[k] - q0[k]));
        }
    }
}

// One thread per (column, row of the block): the row's divergence for the
// column from S and S + delta (zero when delta is), delta cleared behind the
// read; one 64-bit atomic per workgroup into the column's importance.
template <int KMAX>
__global__ __launch_bounds__(256) void k_kl_reduce(JobDev* jobs, int j, uint32_t r0, uint32_t rb,
                                                   uint32_t row_groups, const uint64_t* S,
                                                   unsigned long long* delta) {
    __shared__ long long s_sum[4];
    JobDev& J = jobs[j];
    if (!J.live) return;
    const uint32_t f = blockIdx.x / row_groups;
    const uint32_t rr = (blockIdx.x % row_groups) * 256u + threadIdx.x;
    const int K = J.K;
    long long kl = 0;
    if (J.reg && f < (uint32_t)J.p_w && rr < rb && r0 + rr < (uint32_t)J.n) {
        // regression: floor(D^2 / n_trees^2) >> s_kl, D the change of the summed
        // leaf predictions (|D| < 2^56); the 128-bit quotient by 32-bit limbs
        unsigned long long* d = delta + ((size_t)f * rb + rr) * K;
        const long long D = (long long)d[0];
        if (D) {
            const uint64_t a = (uint64_t)(D < 0 ? -D : D), T2 = (uint64_t)J.T * (uint64_t)J.T;
            const u128 num = (u128)a * a;
            u128 q = 0;
            uint64_t rem = 0;
            for (int i = 3; i >= 0; --i) {
                const uint64_t cur = (rem << 32) | (uint32_t)(num >> (32 * i));
                q |= (u128)(cur / T2) << (32 * i);
                rem = cur % T2;
            }
            kl = (long long)(q >> J.s_kl);
            d[0] = 0;
        }
    } else if (f < (uint32_t)J.p_w && rr < rb && r0 + rr < (uint32_t)J.n) {
        unsigned long long* d = delta + ((size_t)f * rb + rr) * K;
        uint64_t base[KMAX], lg[KMAX], q[KMAX];
        const uint64_t* row_in = S + (size_t)rr * (2 * K + 1);
        bool moved = false;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            base[k] = q[k] = lg[k] = 0;
            if (k < K) {
                const uint64_t dv = d[k];
                moved |= dv != 0;
                base[k] = row_in[k];
                q[k] = base[k] + dv;
            }
        }
        if (moved) {
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if (k < K) lg[k] = row_in[K + k];
            kl = kl_q32<KMAX>(base, lg, row_in[2 * K], q, K);
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if (k < K) d[k] = 0;
        }
    }
    for (int m = 1; m < 64; m <<= 1) kl += __shfl_xor(kl, m);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = kl;
    __syncthreads();
    if (threadIdx.x == 0) {
        const long long v = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        if (v) atomicAdd((unsigned long long*)&J.imp[f], (unsigned long long)v);
    }
}

// Selection of the k-th smallest (0-based) of the job's n_sha shadow
// importances by a most-significant-digit radix select over the order-
// preserving unsigned keys (sign bit flipped): eight passes of an 8-bit
// digit histogram in LDS.  All 256 threads call it.
__device__ long long shadow_select(const JobDev& J, int k, unsigned* s_hist, int* s_sel) {
    const int tid = threadIdx.x;
    const int p_cur = J.p_cur, p_w = J.p_w;
    unsigned long long prefix = 0, mask = 0;
    for (int shift = 56; shift >= 0; shift -= 8) {
        s_hist[tid] = 0u;
        __syncthreads();
        for (int c = p_cur + tid; c < p_w; c += 256) {
            const unsigned long long u = (unsigned long long)J.imp[c] ^ (1ull << 63);
            if ((u & mask) == prefix) atomicAdd(&s_hist[(u >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (tid == 0) {
            int d = 0;
            unsigned below = 0;
            while (d < 255 && below + s_hist[d] <= (unsigned)k) below += s_hist[d++];
            s_sel[0] = d;
            s_sel[1] = k - (int)below;
        }
        __syncthreads();
        prefix |= (unsigned long long)s_sel[0] << shift;
        mask |= 0xFFull << shift;
        k = s_sel[1];
        __syncthreads();  // s_sel and s_hist are rewritten by the next pass
    }
    return (long long)(prefix ^ (1ull << 63));
}

// Per job: hits, history row, shadow threshold, decisions, liveness.  The
// hit threshold is the maximum shadow importance (perc = 100) or the
// ceil(perc n_sha / 100)-th smallest one.
__global__ __launch_bounds__(256) void k_hits_decide(JobDev* jobs, int perc) {
    __shared__ long long s_max[4], s_sum[4];
    __shared__ int s_und[4];
    __shared__ unsigned s_hist[256];
    __shared__ int s_sel[2];
    JobDev& J = jobs[blockIdx.x];
    if (!J.live) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = J.t, p_cur = J.p_cur, p_w = J.p_w;
    long long mx = LLONG_MIN, sum = 0;
    for (int c = tid; c < p_w; c += 256) {
        const long long v = J.imp[c];
        if (c >= p_cur) mx = v > mx ? v : mx;
        sum += v;
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const long long o = __shfl_xor(mx, m);
        mx = o > mx ? o : mx;
        sum += __shfl_xor(sum, m);
    }
    if (lane == 0) {
        s_max[wave] = mx;
        s_sum[wave] = sum;
    }
    __syncthreads();
    long long best = s_max[0], total = s_sum[0];
    for (int v = 1; v < 4; ++v) {
        best = s_max[v] > best ? s_max[v] : best;
        total += s_sum[v];
    }
    if (perc < 100) {
        const int rank = (int)(((long long)perc * J.n_sha + 99) / 100);  // 1-based
        best = shadow_select(J, rank - 1, s_hist, s_sel);
    }
    // reported value = ldexp(v / denom, rep_exp): regression scores come back
    // to squared target units (rep_exp is 0 for classification and TreeImp)
    double denom;
    if (J.mode == 0) {
        denom = (double)total;
    } else if (J.mode == 2) {  // mean divergence per row, in bits
        denom = (double)J.n * (J.reg ? 1.0 : 4294967296.0);
    } else {
        long long oob = 0;
        for (int tau = 0; tau < J.T; ++tau) oob += J.tstat[tau * 4 + 1];
        denom = (double)((long long)J.R * oob);
    }
    const int rexp = J.reg ? J.rep_exp : 0;
    double* hrow = J.hist + (size_t)(t - 1) * J.p;
    for (int j = tid; j < J.p; j += 256)
        if (J.state[j] < 0) hrow[j] = __longlong_as_double(0x7FF8000000000000ll);
    for (int c = tid; c < p_cur; c += 256) {
        const int j = J.act[c];
        const long long v = J.imp[c];
        hrow[j] = denom > 0.0 ? ldexp((double)v / denom, rexp) : 0.0;
        if (v > best) J.hits[j] += 1;
    }
    if (tid == 0) J.shadow_max[t - 1] = denom > 0.0 ? ldexp((double)best / denom, rexp) : 0.0;
    __syncthreads();
    int und = 0;
    const int hc = J.h_conf[t], hr = J.h_rej[t];
    for (int j = tid; j < J.p; j += 256) {
        int8_t s = J.state[j];
        if (s == 0) {
            const int h = J.hits[j];
            if (h >= hc)
                s = 1;
            else if (h <= hr)
                s = -1;
            J.state[j] = s;
        }
        und += s == 0;
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) und += __shfl_xor(und, m);
    if (lane == 0) s_und[wave] = und;
    __syncthreads();
    if (tid == 0) {
        const int u = s_und[0] + s_und[1] + s_und[2] + s_und[3];
        J.n_undecided = u;
        J.live = (u > 0 && t < J.max_iter) ? 1 : 0;
    }
}

// Final ranking, step 1: one thread per feature; a rejected feature's mean
// over its finite history entries of iterations [t0, t1).
__global__ __launch_bounds__(256) void k_rank_mean(const int8_t* state, const double* hist,
                                                   int64_t p, int t0, int t1, double* mean) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= p) return;
    double s = 0.0, m = 0.0;
    int c = 0;
    if (state[j] == -1) {
        for (int t = t0; t < t1; ++t) {
            const double v = hist[(size_t)t * p + j];
            if (v != v) continue;  // NaN: not active in iteration t
            s += v;
            ++c;
        }
        m = c ? s / c : 0.0;
    }
    mean[j] = m;
}

// Step 2: one thread per feature; a rejected feature ranks 3 plus the number
// of rejected features with a strictly larger mean.
__global__ __launch_bounds__(256) void k_rank_count(const int8_t* state, const double* mean,
                                                    int64_t p, int32_t* rank) {
    __shared__ double s_m[256];
    __shared__ int8_t s_s[256];
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int8_t sj = j < p ? state[j] : (int8_t)0;
    const double mj = j < p ? mean[j] : 0.0;
    int above = 0;
    for (int64_t g0 = 0; g0 < p; g0 += 256) {
        __syncthreads();
        const int64_t g = g0 + threadIdx.x;
        s_m[threadIdx.x] = g < p ? mean[g] : 0.0;
        s_s[threadIdx.x] = g < p ? state[g] : (int8_t)0;
        __syncthreads();
        const int lim = (int)(p - g0 < 256 ? p - g0 : 256);
        for (int i = 0; i < lim; ++i) above += (s_s[i] == -1 && s_m[i] > mj) ? 1 : 0;
    }
    if (j < p) rank[j] = sj == 1 ? 1 : (sj == 0 ? 2 : 3 + above);
}

// Multi-seed aggregate over the n_jobs runs of one problem (same p): one
// thread per feature; per run the mean of the feature's finite history
// entries (summed in iteration order), then the median over runs (mean of
// the middle pair for an even count) and the lower median of the decisions.
__global__ __launch_bounds__(256) void k_seed_median(const JobDev* jobs,
                                                     const int8_t* const* decisions, int n_jobs,
                                                     int64_t p, double* med, int8_t* dec) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= p) return;
    double v[64];
    int dv[64];
    for (int r = 0; r < n_jobs; ++r) {
        const JobDev& J = jobs[r];
        double s = 0.0;
        int c = 0;
        for (int t = 0; t < J.t; ++t) {
            const double x = J.hist[(size_t)t * p + j];
            if (x != x) continue;  // NaN: rejected before iteration t + 1
            s += x;
            ++c;
        }
        const double m = c ? s / c : 0.0;
        const int d = decisions[r][j];
        int i = r;  // insertion into the sorted prefixes
        while (i > 0 && v[i - 1] > m) {
            v[i] = v[i - 1];
            --i;
        }
        v[i] = m;
        i = r;
        while (i > 0 && dv[i - 1] > d) {
            dv[i] = dv[i - 1];
            --i;
        }
        dv[i] = d;
    }
    med[j] = n_jobs % 2 ? v[n_jobs / 2] : (v[n_jobs / 2 - 1] + v[n_jobs / 2]) / 2.0;
    dec[j] = (int8_t)dv[(n_jobs - 1) / 2];
}

// Rough fix of the features still tentative (an option outside Algorithm 1,
// from Kursa's Boruta): one workgroup per feature.  A tentative feature is
// confirmed when the median of its history entries of iterations [t0, t1)
// exceeds the median of the shadow thresholds of those iterations, else
// rejected; other decisions are copied.  Medians by rank counting in LDS
// (t1 - t0 <= 1000 values); an even count takes the mean of the middle two.
__device__ double lds_median(const double* v, int m, double* s_mid) {
    // the element of rank r (0-based) is v[i] with #{v < v[i]} + #{v[j] ==
    // v[i], j < i} == r: one writer per rank
    const int r0 = (m - 1) / 2, r1 = m / 2;
    for (int i = threadIdx.x; i < m; i += 256) {
        int less = 0, eq_before = 0;
        for (int j = 0; j < m; ++j) {
            less += v[j] < v[i];
            eq_before += j < i && v[j] == v[i];
        }
        const int r = less + eq_before;
        if (r == r0) s_mid[0] = v[i];
        if (r == r1) s_mid[1] = v[i];
    }
    __syncthreads();
    const double med = m % 2 ? s_mid[0] : (s_mid[0] + s_mid[1]) / 2.0;
    __syncthreads();  // s_mid is rewritten by the next call
    return med;
}

__global__ __launch_bounds__(256) void k_rough_fix(const int8_t* state, const double* hist,
                                                   const double* smax, int64_t p, int t0, int t1,
                                                   int8_t* out) {
    __shared__ double s_v[1000];
    __shared__ double s_mid[2];
    const int64_t j = blockIdx.x;
    const int8_t st = state[j];
    if (st != 0) {
        if (threadIdx.x == 0) out[j] = st;
        return;
    }
    const int m = t1 - t0;
    for (int i = threadIdx.x; i < m; i += 256) s_v[i] = smax[t0 + i];
    __syncthreads();
    const double ms = lds_median(s_v, m, s_mid);
    for (int i = threadIdx.x; i < m; i += 256) s_v[i] = hist[(size_t)(t0 + i) * p + j];
    __syncthreads();
    const double mf = lds_median(s_v, m, s_mid);
    if (threadIdx.x == 0) out[j] = mf > ms ? (int8_t)1 : (int8_t)-1;
}

// Capacity flags of an iteration's tree levels, accumulated into the word
// after them, which only the session set-up clears: iterations enqueued back
// to back then report a failure of any one of them.
__global__ void k_ctr_sticky(LevelCtr* c, int n_levels) {
    if (threadIdx.x != 0) return;
    uint32_t o = 0;
    for (int d = 0; d <= n_levels; ++d) o |= c[d].overflow;
    c[n_levels + 1].overflow |= o;
}

void launch_ctr_sticky(LevelCtr* c, int n_levels, hipStream_t st) {
    hipLaunchKernelGGL(k_ctr_sticky, dim3(1), dim3(64), 0, st, c, n_levels);
}

// Streaming copy used to calibrate hardware byte counters.
__global__ void k_copy(uint4* dst, const uint4* src, size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        dst[i] = src[i];
}

void launch_tree_totals(JobDev* jobs, const TreeDev* trees, int n_trees, uint64_t* tot,
                        hipStream_t st) {
    hipLaunchKernelGGL(k_tree_totals, dim3(n_trees), dim3(256), 0, st, jobs, trees, tot);
}

void launch_treeimp(JobDev* jobs, const TreeDev* trees, int n_trees, const uint64_t* tot,
                    int max_pw, hipStream_t st) {
    hipLaunchKernelGGL(k_treeimp, dim3((unsigned)((max_pw + 255) / 256), (unsigned)n_trees),
                       dim3(256), 0, st, jobs, trees, tot);
}

PermutShape permut_shape(int n_trees, int64_t max_n, int max_depth, int max_pw, bool any_reg) {
    PermutShape s;
    // 128 rows per workgroup: 256 take 4.6 instead of 3.5 ms in the 64-job batch
    // (workgroups that few OOB rows leave half empty), 64 take 374 instead of
    // 314 us at 10,000 x 500
    s.threads = 128;
    // per-column drop sums in LDS for jobs of at most 1024 widened columns
    // (64-bit when the batch has a regression job)
    s.lds_cols = max_pw < 1024 ? max_pw : 1024;
    s.lds_words = s.lds_cols * (any_reg ? 2 : 1);
    s.wide = max_pw > 65536;
    s.lds = (s.wide ? perm_path_bytes<uint32_t>(max_depth, s.threads)
                    : perm_path_bytes<uint16_t>(max_depth, s.threads)) +
            (size_t)s.threads * kPermGroup * 4 + (size_t)s.lds_words * 4;
    s.chunks = (int)((max_n + s.threads - 1) / s.threads);
    // workgroups sharing a row's path: doubled while they hold no more threads than
    // the chip a few times over (about 3/8 of a tree's rows are out of bag;
    // 3,000 x 120, 60 trees: 146 us with four, 133 with eight)
    const int64_t oob = max_n * 3 / 8;
    s.slices = 1;
    while (s.slices < 8 && (int64_t)n_trees * oob * s.slices * 2 <= 512 * 1024) s.slices *= 2;
    return s;
}

void launch_permut(JobDev* jobs, const TreeDev* trees, const NodeDev* nodes, const uint32_t* cls,
                   int kmax, int n_trees, int max_depth, const PermutShape& s,
                   unsigned long long* visits, hipStream_t st) {
    const dim3 grid(8u * (unsigned)(s.chunks * s.slices), (unsigned)((n_trees + 7) / 8));
    const dim3 wg(s.threads);
    if (s.wide)
        hipLaunchKernelGGL(k_permut<uint32_t>, grid, wg, s.lds, st, jobs, trees, n_trees, nodes,
                           cls, kmax, max_depth, s.slices, s.lds_cols, s.lds_words, visits);
    else
        hipLaunchKernelGGL(k_permut<uint16_t>, grid, wg, s.lds, st, jobs, trees, n_trees, nodes,
                           cls, kmax, max_depth, s.slices, s.lds_cols, s.lds_words, visits);
}

// The KL importance of job j over rows [r0, r0 + rb): base, deltas, reduce.
void launch_kl_block(JobDev* jobs, int j, const NodeDev* nodes, const uint32_t* cls, int kmax,
                     uint32_t tree0, int T, int p_w_cap, uint32_t r0, uint32_t rb, uint64_t* S,
                     uint32_t* pi, unsigned long long* delta, int max_depth, hipStream_t st) {
    const dim3 b256(256);
    const unsigned g_base = (rb + 63) / 64;
    const dim3 b1024(1024);
    switch (kmax) {
        case 2: hipLaunchKernelGGL(k_kl_base<2>, dim3(g_base), b1024, 0, st, jobs, j, nodes, cls, kmax, tree0, r0, rb, S, pi); break;
        case 3: hipLaunchKernelGGL(k_kl_base<3>, dim3(g_base), b1024, 0, st, jobs, j, nodes, cls, kmax, tree0, r0, rb, S, pi); break;
        case 4: hipLaunchKernelGGL(k_kl_base<4>, dim3(g_base), b1024, 0, st, jobs, j, nodes, cls, kmax, tree0, r0, rb, S, pi); break;
        case 8: hipLaunchKernelGGL(k_kl_base<8>, dim3(g_base), b1024, 0, st, jobs, j, nodes, cls, kmax, tree0, r0, rb, S, pi); break;
        default: hipLaunchKernelGGL(k_kl_base<16>, dim3(g_base), b1024, 0, st, jobs, j, nodes, cls, kmax, tree0, r0, rb, S, pi); break;
    }
    const size_t lds =
        ((size_t)path_lds_words(max_depth) + (size_t)max_depth * 64) * sizeof(uint32_t);
    const unsigned g_delta = (unsigned)((T + 7) / 8 * 8) * ((rb + 255) / 256);
    const auto kl_delta = kmax == 2   ? k_kl_delta<2>
                          : kmax == 3 ? k_kl_delta<3>
                          : kmax == 4 ? k_kl_delta<4>
                          : kmax == 8 ? k_kl_delta<8>
                                      : k_kl_delta<16>;
    hipLaunchKernelGGL(kl_delta, dim3(g_delta), b256, lds, st, jobs, j, nodes, cls, kmax, tree0,
                       r0, rb, pi, delta, max_depth);
    const uint32_t groups = (rb + 255) / 256;
    const unsigned g_red = (unsigned)(groups * (uint64_t)p_w_cap);
    switch (kmax) {
        case 2: hipLaunchKernelGGL(k_kl_reduce<2>, dim3(g_red), b256, 0, st, jobs, j, r0, rb, groups, S, delta); break;
        case 3: hipLaunchKernelGGL(k_kl_reduce<3>, dim3(g_red), b256, 0, st, jobs, j, r0, rb, groups, S, delta); break;
        case 4: hipLaunchKernelGGL(k_kl_reduce<4>, dim3(g_red), b256, 0, st, jobs, j, r0, rb, groups, S, delta); break;
        case 8: hipLaunchKernelGGL(k_kl_reduce<8>, dim3(g_red), b256, 0, st, jobs, j, r0, rb, groups, S, delta); break;
        default: hipLaunchKernelGGL(k_kl_reduce<16>, dim3(g_red), b256, 0, st, jobs, j, r0, rb, groups, S, delta); break;
    }
}

void launch_hits_decide(JobDev* jobs, int n_jobs, int perc, hipStream_t st) {
    hipLaunchKernelGGL(k_hits_decide, dim3(n_jobs), dim3(256), 0, st, jobs, perc);
}

void launch_rough_fix(const int8_t* state, const double* hist, const double* smax, int64_t p,
                      int t0, int t1, int8_t* out, hipStream_t st) {
    hipLaunchKernelGGL(k_rough_fix, dim3((unsigned)p), dim3(256), 0, st, state, hist, smax, p, t0,
                       t1, out);
}

void launch_rank(const int8_t* state, const double* hist, int64_t p, int t0, int t1,
                 double* mean, int32_t* rank, hipStream_t st) {
    const unsigned g = (unsigned)((p + 255) / 256);
    hipLaunchKernelGGL(k_rank_mean, dim3(g), dim3(256), 0, st, state, hist, p, t0, t1, mean);
    hipLaunchKernelGGL(k_rank_count, dim3(g), dim3(256), 0, st, state, mean, p, rank);
}

void launch_seed_median(const JobDev* jobs, const int8_t* const* decisions, int n_jobs, int64_t p,
                        double* med, int8_t* dec, hipStream_t st) {
    hipLaunchKernelGGL(k_seed_median, dim3((unsigned)((p + 255) / 256)), dim3(256), 0, st, jobs,
                       decisions, n_jobs, p, med, dec);
}

void launch_copy(void* dst, const void* src, size_t bytes, hipStream_t st) {
    const size_t n16 = bytes / 16;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    if (blocks == 0) blocks = 1;
    hipLaunchKernelGGL(k_copy, dim3((unsigned)blocks), dim3(256), 0, st, (uint4*)dst,
                       (const uint4*)src, n16);
}

}  // namespace boruta
