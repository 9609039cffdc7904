// k_forest.hip -- random-forest growth kernels (gfx950).
//
// Trees grow level by level, all trees of all live jobs in the same launch:
//   * k_boot_compact  per tree: in-bag row records and OOB rows from the
//                     bootstrap multiplicities, root node;
//   * k_split_small   one wavefront per node with <= small_rows row records:
//                     rows in lanes, left class counts by all pairs up to 16
//                     rows, by an LDS histogram per feature above;
//                     k_split_small_reg the same for regression nodes;
//   * k_draws         one wavefront per large node: its drawn features and
//                     their columns, and the node's slot record;
//   * k_hist_tile     node-major: one wavefront per (large node, fw drawn
//                     features): LDS histograms [feature][bin] of packed class
//                     counts from batched global bin gathers, then a scan per
//                     feature; writes the item's best threshold;
//   * k_col_scan, k_col_scatter, k_hist_col  column-major (deep levels of
//                     large matrices): the level's items bucketed by bin
//                     column, each column staged once per unit in LDS, the
//                     same histogram and scan per item from the staged bins;
//   * k_split_finalize one wavefront per large node: best over the node's
//                     items, then a partition of its rows;
//   * k_lists_count, k_lists_write  the next level's node lists, in parent
//                     order, without atomics;
//   * k_grow          small forests: all levels of a tree in one workgroup.
// The split rule (reading of the Gini forest of Sec. 2.1): maximise
// Q = S_L/N_L + S_R/N_R over drawn features and thresholds "bin <= b",
// exact rational comparison, ties to the earlier draw then the smaller b;
// split only on a strictly positive decrease Q - S/N.
#include <algorithm>
#include <type_traits>

#include "forest_dev.hpp"

namespace boruta {

// ---------------------------------------------------------------------------
// Per tree: compact the in-bag rows (multiplicity > 0, ascending) into row
// records and the out-of-bag rows into a list; create the root node.  The
// multiplicities are cleared behind the read.  A regression root keeps its
// bootstrap weight W and weighted fixed-point target sum T.
__global__ __launch_bounds__(1024) void k_boot_compact(ForestDev F0) {
    __shared__ uint32_t s_win[16], s_wout[16], s_rin[16];
    __shared__ uint32_t s_cls[16];
    __shared__ unsigned long long s_tsum;
    __shared__ uint32_t s_base_in, s_base_out, s_base_rows;
    ForestDev F = F0;
    F.ctr = F0.ctrs;  // the roots form the lists of level 0
    const uint32_t g = blockIdx.x;
    const TreeDev tr = F.trees[g];
    JobDev& J = F.jobs[tr.job];
    if (!J.live) {  // finished job: its tree slots stay empty
        if (threadIdx.x == 0) F.nodes[g].tree = 0xFFFFFFFFu;
        return;
    }
    const uint32_t n = (uint32_t)J.n;
    const bool reg = J.reg != 0;
    uint32_t* w = J.wbuf + (size_t)tr.tau * n;
    uint32_t* recs = J.rec[0] + (size_t)tr.tau * J.rstride;
    uint32_t* oob = J.oob + (size_t)tr.tau * n;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 16) s_cls[tid] = 0;
    if (tid == 0) {
        s_tsum = 0;
        s_base_in = 0;
        s_base_out = 0;
        s_base_rows = 0;
    }
    __syncthreads();
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (uint32_t base = 0; base < n; base += 1024) {
        const uint32_t i = base + tid;
        const uint32_t wi = i < n ? w[i] : 0u;
        if (i < n) w[i] = 0;  // multiplicities start from zero next iteration
        const bool inb = i < n && wi > 0, isoob = i < n && wi == 0;
        const uint32_t yi = inb && !reg ? (uint32_t)J.y[i] : 0u;
        const uint64_t mi = __ballot(inb), mo = __ballot(isoob);
        // records of the row; more than one only for rows drawn over 15 times
        const uint32_t nr = inb ? (wi + kRecWeight - 1u) / kRecWeight : 0u;
        uint32_t wpre = (uint32_t)__popcll(mi & below), wrec = (uint32_t)__popcll(mi);
        if (__ballot(nr > 1u)) {
            const uint32_t incl = wave_incl_sum(nr);
            wpre = incl - nr;
            wrec = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        if (lane == 0) {
            s_win[wave] = wrec;
            s_wout[wave] = __popcll(mo);
            s_rin[wave] = __popcll(mi);
        }
        __syncthreads();
        uint32_t pin = s_base_in, pout = s_base_out;
        for (int v = 0; v < wave; ++v) {
            pin += s_win[v];
            pout += s_wout[v];
        }
        if (inb) {
            uint32_t left = wi;
            for (uint32_t k = 0; k < nr; ++k) {
                const uint32_t w = min(left, kRecWeight);
                recs[pin + wpre + k] = rec_pack(i, w, yi);
                if (reg)
                    J.wy[0][(size_t)tr.tau * J.rstride + pin + wpre + k] =
                        (int64_t)w * ldg(J.yfix + i);
                left -= w;
            }
            atomicAdd(&s_cls[yi], wi);
        }
        if (reg) {  // the root's weighted target sum: one LDS atomic per wave
            long long tv = inb ? (long long)wi * (long long)ldg(J.yfix + i) : 0ll;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) tv += __shfl_xor(tv, m);
            if (lane == 0 && tv) atomicAdd(&s_tsum, (unsigned long long)tv);
        }
        if (isoob) oob[pout + __popcll(mo & below)] = i;
        __syncthreads();
        if (tid == 0) {
            uint32_t ti = 0, to = 0, tr_ = 0;
            for (int v = 0; v < 16; ++v) {
                ti += s_win[v];
                to += s_wout[v];
                tr_ += s_rin[v];
            }
            s_base_in += ti;
            s_base_out += to;
            s_base_rows += tr_;
        }
        __syncthreads();
    }
    if (tid == 0) {
        J.tstat[tr.tau * 4 + 0] = (int32_t)s_base_rows;
        J.tstat[tr.tau * 4 + 1] = (int32_t)s_base_out;
        J.tstat[tr.tau * 4 + 2] = 0;
        uint32_t counts[16], tot = 0;
        for (int k = 0; k < 16; ++k) {
            counts[k] = s_cls[k];
            tot += s_cls[k];
        }
        const int kind = reg ? write_node_reg(F, J, g, g, 1u, 0u, s_base_in, tot,
                                              (int64_t)s_tsum, 0u)
                             : write_node(F, J, g, g, 1u, 0u, s_base_in, tot, 0u, counts);
        enqueue_nodes(F, J, g, &kind, 1);
        F.kinds[g] = (uint8_t)kind;  // k_grow starts from it
    }
}

// ---------------------------------------------------------------------------
// Small nodes: one wavefront per node.  With W = the node's row count rounded
// up to a power of two, the wave is split into 64/W segments of W lanes; a
// segment holds the node's rows (one per lane) and evaluates one drawn
// feature, so 64/W features are scored per pass.  The bins of the next passes
// are gathered while this one computes.  A node of this path weighs less than
// 256 rows, so the class counts on the left of the threshold at a lane's own
// bin are 8-bit fields, four classes to a word (Pk8), from
//   * segments of up to 16 lanes: an all-pairs sum (W lane permutes a pass);
//   * segments of 32 or 64 lanes: a histogram of the packed counters in LDS,
//     one word per bin, summed over the bins by a wave scan and read back at
//     the lane's bin.
// A lane permute costs 6 cycles of the CU's one LDS pipe, so W of them pass
// the histogram's six 16-byte accesses (8 cycles each) between W = 16 and 32.
// Against 64-bit class sums and an exact butterfly per node (traced beside the
// histogram kernels): 64 jobs of 2-5 classes 155 -> 47 ms over six iterations,
// n = 10,000 x 500 of 3 classes 50 -> 35 us a launch, n = 100,000 x 2,000 of 4
// 830 -> 730 us (there the bin gathers bound it).
struct SmallOut {
    int kinds[2];
    uint32_t child;
    uint64_t alg;
};

__device__ __forceinline__ uint32_t readlane_w(uint32_t v, int src) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, src);
}

// LDS of a wave of the small-node kernels: the head -- the permutation round
// table and the node's bins by row (which take the table's place where one
// round of 64 draws serves every node) --, then the rows' counters and two
// packed histograms, or a regression node's rows.
constexpr uint32_t kBinStride = 68;  // bytes per row: 17 words, so that a column's bytes of
                                     // different rows lie in different banks
__host__ __device__ constexpr uint32_t small_lds_words(uint32_t head, int words) {
    return head + (uint32_t)words * (64u + 512u);
}

// A node's bins of one round of draws, read row by row from the row-major copy
// (plans with column-major levels) into LDS: a load covers 64 / F2 rows x F2 draws (F2: the draws rounded up to a
// power of two), so it touches a row's few cache lines once instead of one line
// per lane, and the passes then take their bins from LDS.  myf: lane q holds draw
// q's widened column; row: lane i < len holds the node's row i.
__device__ __forceinline__ void load_bins(const JobDev& J, uint8_t* bins, int myf, uint32_t row,
                                          int len, int nq) {
    const int lane = threadIdx.x & 63;
    int F2 = 1;
    while (F2 < nq) F2 <<= 1;
    const int per = 64 / F2, rr = lane / F2, f = lane & (F2 - 1);
    const uint32_t c = (uint32_t)__shfl(myf, f < nq ? f : 0);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the table's or earlier bins' reads
    for (int r0 = 0; r0 < len; r0 += 8 * per) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int r = min(r0 + u * per + rr, len - 1);
            const uint32_t i = (uint32_t)__shfl((int)row, r);
            v[u] = ldg(J.rowmaj + (size_t)i * J.rm_stride + c);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int r = r0 + u * per + rr;
            if (r < len) bins[r * (int)kBinStride + f] = (uint8_t)v[u];
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// lds: the wave's LDS region of small_lds_words(F.small_head, WORDS) words
// RM: the job keeps a row-major copy of its bins
template <int WORDS, bool RM>
__device__ __forceinline__ void small_node(const ForestDev& F, uint32_t id, const NodeDev& nd,
                                           const TreeDev& tr, JobDev& J, SmallOut& out,
                                           uint32_t* lds) {
    uint16_t* tab = reinterpret_cast<uint16_t*>(lds);
    uint8_t* bins = reinterpret_cast<uint8_t*>(lds + F.bins_off);  // [64][kBinStride]
    uint32_t* scnt = lds + F.small_head;    // [WORDS][64] the rows' counter words
    uint32_t* hist = scnt + WORDS * 64;     // [2][WORDS][256] packed histograms
    const int lane = threadIdx.x & 63;
    const int B = J.B, mtry = J.mtry;
    const size_t tbase = (size_t)tr.tau * J.rstride + nd.seg;
    const uint32_t* rin = J.rec[F.parity] + tbase;
    uint32_t* rout = J.rec[F.parity ^ 1] + tbase;
    const int len = (int)uniform(nd.len);
    int W = 2;
    while (W < len) W <<= 1;
    const int G = 64 / W;                // features per pass
    const int seg = lane / W, i = lane & (W - 1);
    const bool valid = i < len;
    const uint32_t rec = valid ? ldg(rin + i) : 0u;
    const uint32_t row = rec_row(rec), wt = rec_w(rec), yv = rec_y(rec);
    const uint32_t inc = wt << ((yv & 3u) * 8u);  // this lane's row in its counter word
    const uint32_t yw = yv >> 2;                  // that word
    uint32_t cn[WORDS];  // the node's class counts, packed (each below 256)
    uint32_t S = 0;      // their sum of squares
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        cn[w] = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (4 * w + k < J.K) cn[w] |= F.cls[(size_t)id * F.kmax + 4 * w + k] << (8 * k);
        S = dot4(cn[w], cn[w], S);
    }
    const uint32_t N = nd.n;
    const KeyedPerm P = make_perm(J.seed_lo, J.seed_hi, kMtry, (uint32_t)J.t, (uint32_t)tr.tau,
                                  nd.heap, 0u, (uint64_t)J.p_w);
    // the wave tabulates the round functions once, evenly, instead of every
    // lane walking its draw through all rounds (halves of up to 8 bits)
    const bool use_tab = (P.rounds << P.half) <= kDrawTab;
    if (use_tab) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the previous node's lookups
        for (uint32_t e = (uint32_t)lane; e < (P.rounds << P.half); e += 64u)
            tab[e] = (uint16_t)perm_round(P, e >> P.half, e & P.mask);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    // Each lane keeps the best of its own candidates over the passes (they
    // arrive in increasing draw position, so an exact tie keeps the earlier
    // one); one wave-wide selection per node picks the winner.  With FP32
    // ranking, two candidates are compared exactly only when their FP32
    // scores are within the ranking margin of each other and their partitions
    // are not the same one (equal or mirrored counts: an exact tie, which is
    // what most near scores of small nodes are).
    bool has = false;
    float lq = -1.0f;
    int ld = 0, lb = 0;     // draw position and threshold of the lane's best
    uint32_t la[WORDS];     // its left counts
#pragma unroll
    for (int w = 0; w < WORDS; ++w) la[w] = 0;
    const bool fp32 = F.split_rank != 0;
    const int abase = (lane - i) << 2;  // ds_bpermute byte address of the segment's lane 0
    const bool pairs = W <= 16;
    if (pairs) {
        // row j's counter words at scnt[w][j] (lane j holds row j in segment
        // 0; every other lane holds zero): the passes read four rows'
        // counters per LDS broadcast
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the previous node's reads
#pragma unroll
        for (int w = 0; w < WORDS; ++w)
            scnt[w * 64 + lane] = seg == 0 && valid && yw == (uint32_t)w ? inc : 0u;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    const uint8_t* rowbase = J.colbase + row;
    int myf = 0;  // the round's draw of this lane
    for (int q0 = 0; q0 < mtry; q0 += 64) {
        const int nq = min(64, mtry - q0);
        myf =
            lane < nq ? (int)(use_tab ? perm_apply_tab(P, tab, (uint32_t)(q0 + lane))
                                      : perm_apply(P, (uint32_t)(q0 + lane)))
                      : 0;
        // the drawn feature's bins: by row in LDS, or in its column, 256 * myoff
        // bytes from the start of the region
        uint32_t myoff = 0;
        if constexpr (RM)
            load_bins(J, bins, myf, row, len, nq);
        else
            myoff = lane < nq ? (uint32_t)((uint64_t)(ldg(J.colptr + myf) - J.colbase) >> 8) : 0u;
        const int passes = (nq + G - 1) / G;
        // The bin load is unconditional (lanes without a row read row 0, lanes
        // past the drawn features read the first one) so that blocks of loads
        // issue back to back; eval() masks what does not count.
        auto gather = [&](int pass) {
            const int qq = pass * G + seg, qc = qq < nq ? qq : 0;
            if constexpr (RM) return (int)bins[(valid ? i : 0) * (int)kBinStride + qc];
            else return (int)ldg(rowbase + (uint64_t)(uint32_t)__shfl((int)myoff, qc) * 256u);
        };
        auto eval = [&](int pass, int raw) {
            const int qq = pass * G + seg;
            const bool act = valid && qq < nq;
            const int b = act ? raw : 0x7FFF;
            // acc: the segment's rows j with bin <= b
            uint32_t acc[WORDS];
            if (pairs) {
#pragma unroll
                for (int w = 0; w < WORDS; ++w) acc[w] = 0;
                for (int j0 = 0; j0 < len; j0 += 4) {
                    int bj[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        bj[u] = __builtin_amdgcn_ds_bpermute(abase + ((j0 + u) << 2), b);
#pragma unroll
                    for (int w = 0; w < WORDS; ++w) {
                        const uint4 c = *reinterpret_cast<const uint4*>(scnt + w * 64 + j0);
                        acc[w] += bj[0] <= b ? c.x : 0u;
                        acc[w] += bj[1] <= b ? c.y : 0u;
                        acc[w] += bj[2] <= b ? c.z : 0u;
                        acc[w] += bj[3] <= b ? c.w : 0u;
                    }
                }
            } else {
                uint4* h4 = reinterpret_cast<uint4*>(hist);
                const int ng = G;  // 2 or 1 features
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the last pass's reads
#pragma unroll
                for (int u = 0; u < 2 * WORDS; ++u)
                    if (u < ng * WORDS) h4[u * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                if (act) atomicAdd(&hist[(uint32_t)(seg * WORDS) * 256u + yw * 256u + (uint32_t)b], inc);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
                for (int u = 0; u < 2 * WORDS; ++u) {
                    if (u < ng * WORDS) {
                        uint4 v = h4[u * 64 + lane];
                        v.y += v.x;
                        v.z += v.y;
                        v.w += v.z;
                        const uint32_t ex = wave_incl_sum(v.w) - v.w;
                        h4[u * 64 + lane] = make_uint4(v.x + ex, v.y + ex, v.z + ex, v.w + ex);
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
                for (int w = 0; w < WORDS; ++w)
                    acc[w] = hist[(uint32_t)(seg * WORDS + w) * 256u + (act ? (uint32_t)b : 0u)];
            }
            const Side c = side_of<WORDS, 8>(acc, cn, S);
            const bool ok = act && b <= B - 2 && c.nl < N;  // nl >= the lane's own row
            bool better;
            float qc = -1.0f;
            if (fp32) {
                const float qu = side_q32(c, N);  // unconditional: a select, no branch
                qc = ok ? qu : -1.0f;
                bool eq = true, mir = true;  // the same partition, the mirrored one
#pragma unroll
                for (int w = 0; w < WORDS; ++w) {
                    eq = eq && acc[w] == la[w];
                    mir = mir && acc[w] == cn[w] - la[w];
                }
                const bool near = ok && has && qc >= fp32_floor(lq) && lq >= fp32_floor(qc);
                bool exact = false;
                if (__ballot(near && !eq && !mir))
                    exact = !eq && !mir && side_better<8>(c, side_of<WORDS, 8>(la, cn, S), N);
                better = ok && (!has || (near ? exact : qc > lq));
            } else {
                better = ok && (!has || side_better<8>(c, side_of<WORDS, 8>(la, cn, S), N));
            }
            if (better) {
                has = true;
                lq = qc;
                ld = q0 + qq;
                lb = b;
#pragma unroll
                for (int w = 0; w < WORDS; ++w) la[w] = acc[w];
            }
        };
        if constexpr (RM) {
            for (int pass = 0; pass < passes; ++pass) eval(pass, gather(pass));
            continue;
        }
        // bins of kPF passes are in flight while the previous kPF are scored
        constexpr int kPF = 2;
        int bq[kPF];
#pragma unroll
        for (int u = 0; u < kPF; ++u) bq[u] = gather(u);
        for (int pb = 0; pb < passes; pb += kPF) {
            int bn[kPF];
            if (pb + kPF < passes) {
#pragma unroll
                for (int u = 0; u < kPF; ++u) bn[u] = gather(pb + kPF + u);
            }
#pragma unroll
            for (int u = 0; u < kPF; ++u)
                if (pb + u < passes) eval(pb + u, bq[u]);
#pragma unroll
            for (int u = 0; u < kPF; ++u) bq[u] = bn[u];
        }
    }
    out.alg = (uint64_t)len * (uint64_t)(mtry + 6);
    // The winner: with FP32 ranking among the lanes within the margin of the
    // wave's maximum.  When they all hold one partition (or its mirror) they
    // tie exactly, and the earliest draw, then the smallest threshold wins;
    // otherwise they are compared exactly one after the other.
    bool fin = has;
    if (fp32) {
        const float qmax = wave_max_f_dpp(lq);
        fin = has && lq >= fp32_floor(qmax);
    }
    const uint64_t fm = __ballot(fin);
    int win = -1;
    uint32_t ba[WORDS];
    if (fm) {
        win = (int)__ffsll((unsigned long long)fm) - 1;
        bool eq = true, mir = true;
#pragma unroll
        for (int w = 0; w < WORDS; ++w) {
            ba[w] = readlane_w(la[w], win);
            eq = eq && la[w] == ba[w];
            mir = mir && la[w] == cn[w] - ba[w];
        }
        if (!__ballot(fin && !eq && !mir)) {
            const uint32_t dmin = wave_min_u_dpp(fin ? (uint32_t)ld : 0xFFFFFFFFu);
            const uint32_t bmin =
                wave_min_u_dpp(fin && (uint32_t)ld == dmin ? (uint32_t)lb : 0xFFFFFFFFu);
            win = (int)__ffsll((unsigned long long)__ballot(fin && (uint32_t)ld == dmin &&
                                                            (uint32_t)lb == bmin)) - 1;
        } else {
            Side cb = side_of<WORDS, 8>(ba, cn, S);
            for (uint64_t m = fm & (fm - 1); m; m &= m - 1) {
                const int l = (int)__ffsll((unsigned long long)m) - 1;
                uint32_t a[WORDS];
#pragma unroll
                for (int w = 0; w < WORDS; ++w) a[w] = readlane_w(la[w], l);
                const Side c = side_of<WORDS, 8>(a, cn, S);
                const int d0 = __builtin_amdgcn_readlane(ld, win),
                          d1 = __builtin_amdgcn_readlane(ld, l);
                const int b0 = __builtin_amdgcn_readlane(lb, win),
                          b1 = __builtin_amdgcn_readlane(lb, l);
                if (side_better<8>(c, cb, N) ||
                    (!side_better<8>(cb, c, N) && (d1 < d0 || (d1 == d0 && b1 < b0)))) {
                    win = l;
                    cb = c;
                }
            }
        }
#pragma unroll
        for (int w = 0; w < WORDS; ++w) ba[w] = readlane_w(la[w], win);
    }
    Cand best;
    best.nl = 0;
    if (win >= 0) {
        const Side c = side_of<WORDS, 8>(ba, cn, S);
        best.q = __builtin_amdgcn_readlane(ld, win);
        best.b = __builtin_amdgcn_readlane(lb, win);
        best.nl = c.nl;
        best.nr = N - c.nl;
        best.pad = 0;
        best.sl = c.sl;
        best.sr = c.sr;
        const uint32_t q = (uint32_t)best.q;
        if (mtry <= 64)  // one round: the draw is still in its lane
            best.f = __builtin_amdgcn_readlane(myf, best.q);
        else
            best.f = (int)(use_tab ? perm_apply_tab(P, tab, q) : perm_apply(P, q));
    }
    if (best.nl == 0 || !cand_positive(best, S, N)) {  // stays the leaf it was created as
        if (lane == 0) mark_unused_pair(F, out.child);
        return;
    }
    // partition with the lanes of segment 0
    const bool mine = seg == 0 && valid;
    int wb;  // the row's bin in the winning column
    if (RM && mtry <= 64)
        wb = bins[(valid ? i : 0) * (int)kBinStride + best.q];
    else
        wb = (int)ldg(ldg(J.colptr + best.f) + row);
    const bool left = mine && wb <= best.b;
    const uint64_t lm = __ballot(left), vm = __ballot(mine);
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const uint32_t nl_rows = (uint32_t)__popcll(lm);
    if (mine) {
        const uint32_t pos = left ? (uint32_t)__popcll(lm & below)
                                  : nl_rows + (uint32_t)__popcll(vm & ~lm & below);
        rout[pos] = rec;
    }
    if (lane == 0) {
        uint32_t cl[16], cr[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            cl[k] = k < 4 * WORDS ? pk_field<8>(ba, k % (4 * WORDS)) : 0u;
            cr[k] = (k < 4 * WORDS ? pk_field<8>(cn, k % (4 * WORDS)) : 0u) - cl[k];
        }
        split_node(F, J, tr, id, nd, best, nl_rows, cl, cr, cand_gain_fix(best, S, N),
                   out.child, out.kinds);
    }
}

// One wavefront per node (grid-stride over the level's small-node list).
// The small nodes of tree level `level`: all of them (count from the level's
// counters, grid-stride) or, with an explicit count, list entries
// [first, first + count).  WORDS: counter words of the plan's widest job; a
// job of fewer classes takes the narrower form.  RM: the plan's jobs keep
// row-major copies.
template <int WORDS, bool RM>
__device__ __forceinline__ void small_node_of(const ForestDev& F, uint32_t id, const NodeDev& nd,
                                              const TreeDev& tr, JobDev& J, SmallOut& out,
                                              uint32_t* lds) {
    if (WORDS == 1 || J.K <= 4)
        small_node<1, RM>(F, id, nd, tr, J, out, lds);
    else if (WORDS == 2 || J.K <= 8)
        small_node<WORDS == 1 ? 1 : 2, RM>(F, id, nd, tr, J, out, lds);
    else
        small_node<WORDS, RM>(F, id, nd, tr, J, out, lds);
}

template <int WORDS, bool RM>
__global__ __launch_bounds__(256) void k_split_small(ForestDev F0, int level, uint32_t first,
                                                     uint32_t count) {
    const ForestDev F = level_view(F0, level);
    if (count == 0xFFFFFFFFu) {
        first = 0;
        count = level_small(F0, level);
    }
    extern __shared__ uint4 lds_raw[];  // [4][small_lds_words(F.small_head, WORDS)]
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    uint32_t* lds =
        reinterpret_cast<uint32_t*>(lds_raw) + wave * small_lds_words(F.small_head, WORDS);
    unsigned long long alg = 0;  // statistics
    for (uint32_t li = blockIdx.x * 4u + (uint32_t)wave; li < count; li += gridDim.x * 4u) {
        SmallOut o;
        o.kinds[0] = o.kinds[1] = kLeaf;
        o.child = F.next_base + 2u * (first + li);
        o.alg = 0;
        const uint32_t id = uniform(F.small_in[first + li]);
        const NodeDev nd = F.nodes[id];
        const TreeDev tr = F.trees[nd.tree];
        JobDev& J = F.jobs[tr.job];
        if (F.has_reg && J.reg) continue;  // k_split_small_reg
        small_node_of<WORDS, RM>(F, id, nd, tr, J, o, lds);
        // what the children need next; the next level's lists are built from these
        if (lane == 0) F.kinds[first + li] = (uint8_t)(o.kinds[0] | o.kinds[1] << 2);
        alg += o.alg;
    }
    // one atomic per wave for the statistics
    if (F.alg_bytes && lane == 0 && alg)
        atomicAdd((unsigned long long*)&F.alg_bytes[kAlgWords + ((blockIdx.x * 4u + wave) &
                                                                 (kAlgWords - 1))], alg);
}

// Small regression nodes, as small_node: a segment's lanes hold the rows'
// weights and weighted targets as FP64 integers (at most 64 records of weight
// 15 and |y_fix| < 2^38: sums below 2^49, exact), and the left sums of the
// threshold at a lane's own bin come from an all-pairs sum over the segment,
// two fused multiply-adds per row.  Thresholds are ranked by reg_score and
// compared exactly (reg_small_better) within the FP64 margin, except those
// that leave the same or the mirrored sums: an exact tie.
// These nodes took one wavefront and one 256-bin, 64-bit histogram scan per
// drawn feature: of the 3.75 ms of an iteration at n = 10,000, 50 features, 200
// trees of depth 12, the histogram, partition and draw kernels spent 2.7 ms on
// the levels whose nodes have a few dozen rows (at the deepest level 662 us of
// histograms, 165 of partitions and 66 of draws became 221, 15 and 99 beside 182
// for the nodes that stay).
__host__ __device__ constexpr uint32_t small_reg_words(uint32_t head) { return head + 64u * 4u; }

__device__ __forceinline__ void small_node_reg(const ForestDev& F, uint32_t id, const NodeDev& nd,
                                               const TreeDev& tr, JobDev& J, SmallOut& out,
                                               uint32_t* lds) {
    uint16_t* tab = reinterpret_cast<uint16_t*>(lds);
    double2* rows = reinterpret_cast<double2*>(lds + F.small_head);  // [64] (w, w y)
    const int lane = threadIdx.x & 63;
    const int B = J.B, mtry = J.mtry;
    const size_t tbase = (size_t)tr.tau * J.rstride + nd.seg;
    const uint32_t* rin = J.rec[F.parity] + tbase;
    uint32_t* rout = J.rec[F.parity ^ 1] + tbase;
    const int len = (int)uniform(nd.len);
    int W = 2;
    while (W < len) W <<= 1;
    const int G = 64 / W;
    const int seg = lane / W, i = lane & (W - 1);
    const bool valid = i < len;
    const uint32_t rec = valid ? ldg(rin + i) : 0u;
    const int64_t wy = valid ? ldg(J.wy[F.parity] + tbase + i) : 0;
    const uint32_t row = rec_row(rec), wt = rec_w(rec);
    const int64_t Ti = node_tsum(F.cls, F.kmax, id);
    const uint32_t Wi = nd.n;
    const double T = (double)Ti, Wn = (double)Wi;
    const KeyedPerm P = make_perm(J.seed_lo, J.seed_hi, kMtry, (uint32_t)J.t, (uint32_t)tr.tau,
                                  nd.heap, 0u, (uint64_t)J.p_w);
    const bool use_tab = (P.rounds << P.half) <= kDrawTab;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the previous node's reads
    if (use_tab) {
        for (uint32_t e = (uint32_t)lane; e < (P.rounds << P.half); e += 64u)
            tab[e] = (uint16_t)perm_round(P, e >> P.half, e & P.mask);
    }
    {
        const bool mine = seg == 0 && valid;
        rows[lane] = double2{mine ? (double)wt : 0.0, mine ? (double)wy : 0.0};
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    bool has = false;
    double lq = -1.0, lt = 0.0, lw = 0.0;  // the lane's best: score, left sums
    int ld = 0, lb = 0;                    // its draw position and threshold
    const bool rank = F.split_rank != 0;
    const int abase = (lane - i) << 2;
    int myf = 0;  // the round's draw of this lane
    for (int q0 = 0; q0 < mtry; q0 += 64) {
        const int nq = min(64, mtry - q0);
        myf = lane < nq ? (int)(use_tab ? perm_apply_tab(P, tab, (uint32_t)(q0 + lane))
                                      : perm_apply(P, (uint32_t)(q0 + lane)))
                      : 0;
        const uint32_t myoff =
            lane < nq ? (uint32_t)((uint64_t)(ldg(J.colptr + myf) - J.colbase) >> 8) : 0u;
        const int passes = (nq + G - 1) / G;
        auto gather = [&](int pass) {
            const int qq = pass * G + seg;
            const uint32_t off = (uint32_t)__shfl((int)myoff, qq < nq ? qq : 0);
            return (int)ldg(J.colbase + row + (uint64_t)off * 256u);
        };
        int nb = gather(0);
        for (int pass = 0; pass < passes; ++pass) {
            const int qq = pass * G + seg;
            const bool act = valid && qq < nq;
            const int b = act ? nb : 0x7FFF;
            nb = gather(pass + 1 < passes ? pass + 1 : pass);
            double wl = 0.0, tl = 0.0;
            for (int j0 = 0; j0 < len; j0 += 4) {
                int bj[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    bj[u] = __builtin_amdgcn_ds_bpermute(abase + ((j0 + u) << 2), b);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double2 r = rows[j0 + u];  // zero past the node's rows
                    const double m = bj[u] <= b ? 1.0 : 0.0;
                    wl = __builtin_fma(m, r.x, wl);
                    tl = __builtin_fma(m, r.y, tl);
                }
            }
            const bool ok = act && b <= B - 2 && wl < Wn;  // wl holds the lane's own row
            const double qu = reg_score(tl, wl, T, Wn);
            const double qc = ok ? qu : -1.0;
            const bool tie = (tl == lt && wl == lw) || (tl == T - lt && wl == Wn - lw);
            const bool near =
                ok && has && !tie &&
                (!rank || (qc >= fp64_floor(lq) && lq >= fp64_floor(qc)));
            bool better = ok && (!has || (!tie && qc > lq));
            if (__ballot(near)) {
                const bool ex = reg_small_better((int64_t)tl, (uint32_t)wl, (int64_t)lt,
                                                 (uint32_t)lw, Ti, Wi);
                better = near ? ex : better;
            }
            if (better) {
                has = true;
                lq = qc;
                lt = tl;
                lw = wl;
                ld = q0 + qq;
                lb = b;
            }
        }
    }
    out.alg = (uint64_t)len * (uint64_t)(mtry + 6);
    // the winner, as in small_node
    bool fin = has;
    if (rank) {
        const double qmax = wave_max_f64_dpp(lq);
        fin = has && lq >= fp64_floor(qmax);
    }
    const uint64_t fm = __ballot(fin);
    int win = -1;
    if (fm) {
        win = (int)__ffsll((unsigned long long)fm) - 1;
        auto lane_f64 = [&](double v, int l) {
            return __builtin_bit_cast(double, readlane64(__builtin_bit_cast(uint64_t, v), l));
        };
        double bt = lane_f64(lt, win), bw = lane_f64(lw, win);
        const bool tie = (lt == bt && lw == bw) || (lt == T - bt && lw == Wn - bw);
        if (!__ballot(fin && !tie)) {
            const uint32_t dmin = wave_min_u_dpp(fin ? (uint32_t)ld : 0xFFFFFFFFu);
            const uint32_t bmin =
                wave_min_u_dpp(fin && (uint32_t)ld == dmin ? (uint32_t)lb : 0xFFFFFFFFu);
            win = (int)__ffsll((unsigned long long)__ballot(fin && (uint32_t)ld == dmin &&
                                                            (uint32_t)lb == bmin)) - 1;
        } else {
            for (uint64_t m = fm & (fm - 1); m; m &= m - 1) {
                const int l = (int)__ffsll((unsigned long long)m) - 1;
                const double ct = lane_f64(lt, l), cw = lane_f64(lw, l);
                const int d0 = __builtin_amdgcn_readlane(ld, win),
                          d1 = __builtin_amdgcn_readlane(ld, l);
                const int b0 = __builtin_amdgcn_readlane(lb, win),
                          b1 = __builtin_amdgcn_readlane(lb, l);
                const bool up = reg_small_better((int64_t)ct, (uint32_t)cw, (int64_t)bt,
                                                 (uint32_t)bw, Ti, Wi);
                const bool down = reg_small_better((int64_t)bt, (uint32_t)bw, (int64_t)ct,
                                                   (uint32_t)cw, Ti, Wi);
                if (up || (!down && (d1 < d0 || (d1 == d0 && b1 < b0)))) {
                    win = l;
                    bt = ct;
                    bw = cw;
                }
            }
        }
    }
    Cand best;
    best.nl = 0;
    if (win >= 0) {
        const int64_t tl =
            (int64_t)__builtin_bit_cast(double, readlane64(__builtin_bit_cast(uint64_t, lt), win));
        best.nl = (uint32_t)__builtin_bit_cast(
            double, readlane64(__builtin_bit_cast(uint64_t, lw), win));
        best.nr = Wi - best.nl;
        best.q = __builtin_amdgcn_readlane(ld, win);
        best.b = __builtin_amdgcn_readlane(lb, win);
        best.pad = 0;
        best.sl = (uint64_t)tl;
        best.sr = (uint64_t)(Ti - tl);
        if (mtry <= 64)  // one round: the draw is still in its lane
            best.f = __builtin_amdgcn_readlane(myf, best.q);
        else
            best.f = (int)(use_tab ? perm_apply_tab(P, tab, (uint32_t)best.q)
                                   : perm_apply(P, (uint32_t)best.q));
    }
    if (best.nl == 0 || reg_gap(best) == 0) {  // no decrease: stays the leaf it was created as
        if (lane == 0) mark_unused_pair(F, out.child);
        return;
    }
    const bool mine = seg == 0 && valid;
    const uint8_t* col = ldg(J.colptr + best.f);
    const bool left = mine && (int)ldg(col + row) <= best.b;
    const uint64_t lm = __ballot(left), vm = __ballot(mine);
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const uint32_t nl_rows = (uint32_t)__popcll(lm);
    if (mine) {
        const uint32_t pos = left ? (uint32_t)__popcll(lm & below)
                                  : nl_rows + (uint32_t)__popcll(vm & ~lm & below);
        rout[pos] = rec;
        J.wy[F.parity ^ 1][tbase + pos] = wy;
    }
    if (lane == 0)
        split_node_reg(F, J, tr, id, nd, best, nl_rows, reg_gain_fix(best, J.s_gain), out.child,
                       out.kinds);
}

// The regression nodes of a level's small-node list (k_split_small takes the
// others).
__global__ __launch_bounds__(256) void k_split_small_reg(ForestDev F0, int level, uint32_t first,
                                                         uint32_t count) {
    const ForestDev F = level_view(F0, level);
    if (count == 0xFFFFFFFFu) {
        first = 0;
        count = level_small(F0, level);
    }
    extern __shared__ uint4 lds_raw[];  // [4][small_reg_words(F.small_head)]
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    uint32_t* lds = reinterpret_cast<uint32_t*>(lds_raw) + wave * small_reg_words(F.small_head);
    unsigned long long alg = 0;
    for (uint32_t li = blockIdx.x * 4u + (uint32_t)wave; li < count; li += gridDim.x * 4u) {
        SmallOut o;
        o.kinds[0] = o.kinds[1] = kLeaf;
        o.child = F.next_base + 2u * (first + li);
        o.alg = 0;
        const uint32_t id = uniform(F.small_in[first + li]);
        const NodeDev nd = F.nodes[id];
        const TreeDev tr = F.trees[nd.tree];
        JobDev& J = F.jobs[tr.job];
        if (!J.reg) continue;
        small_node_reg(F, id, nd, tr, J, o, lds);
        if (lane == 0) F.kinds[first + li] = (uint8_t)(o.kinds[0] | o.kinds[1] << 2);
        alg += o.alg;
    }
    if (F.alg_bytes && lane == 0 && alg)
        atomicAdd((unsigned long long*)&F.alg_bytes[kAlgWords + ((blockIdx.x * 4u + wave) &
                                                                 (kAlgWords - 1))], alg);
}

// ---------------------------------------------------------------------------
// Best threshold of one feature from its LDS histogram h[KMAX][256] (class
// rows of 256 bins; bins >= B stay zero).  Lane l owns bins 4l .. 4l+3, read
// as one 16-byte word per class (consecutive lanes, consecutive words: no
// bank conflicts); class prefix sums come from a DPP wave scan.
template <int KMAX>
__device__ Cand feature_best(const uint32_t* h, int B, int q, int f, const uint32_t* cnode,
                             uint32_t N, int split_rank) {
    constexpr bool kRegs = KMAX <= 4;  // keep the lane's counts in registers
    const int lane = threadIdx.x & 63;
    const int b0 = lane * 4;
    uint32_t hv[kRegs ? KMAX : 1][4];
    uint32_t excl[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const uint4 v = *reinterpret_cast<const uint4*>(h + k * 256 + b0);
        if constexpr (kRegs) {
            hv[k][0] = v.x;
            hv[k][1] = v.y;
            hv[k][2] = v.z;
            hv[k][3] = v.w;
        }
        const uint32_t a = v.x + v.y + v.z + v.w;
        excl[k] = wave_incl_sum(a) - a;
    }
    auto hval = [&](int k, int u) -> uint32_t {
        if constexpr (kRegs)
            return hv[k][u];
        else
            return h[k * 256 + b0 + u];
    };
    // candidates of this lane, in ascending threshold order
    auto make = [&](int b, const uint32_t* cl) {
        Cand c;
        c.q = q;
        c.f = f;
        c.b = b;
        c.pad = 0;
        uint32_t nl = 0;
        uint64_t sl = 0, sr = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const uint32_t r = cnode[k] - cl[k];
            nl += cl[k];
            sl += (uint64_t)cl[k] * cl[k];
            sr += (uint64_t)r * r;
        }
        c.nl = nl;
        c.nr = N - nl;
        c.sl = sl;
        c.sr = sr;
        return c;
    };
    Cand lb;
    lb.nl = 0;
    lb.b = 0x7FFFFFFF;
    lb.q = q;
    lb.f = f;
    lb.nr = 0;
    lb.pad = 0;
    lb.sl = lb.sr = 0;
    uint32_t cl[KMAX];
    if (!split_rank) {
#pragma unroll
        for (int k = 0; k < KMAX; ++k) cl[k] = excl[k];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = b0 + u;
            uint32_t add = 0;
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                const uint32_t v = hval(k, u);
                cl[k] += v;
                add += v;
            }
            // an empty bin repeats the previous threshold's partition, which the
            // smaller threshold already represents
            if (b > B - 2 || add == 0) continue;
            const Cand c = make(b, cl);
            if (c.nl == 0 || c.nl == N) continue;
            if (lb.nl == 0 || cand_better(c, lb)) lb = c;
        }
        return wave_best_exact(lb);
    }
    // FP32 ranking: the lane's best and second-best FP32 scores; finalists
    // are the lanes whose best is within the margin of the wave maximum.  A
    // finalist lane whose second-best is also within it re-ranks its bins
    // exactly; otherwise its finalist is the best bin alone.
    float q1 = -1.0f, q2 = -1.0f;
    int u1 = 0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) cl[k] = excl[k];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int b = b0 + u;
        uint32_t add = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const uint32_t v = hval(k, u);
            cl[k] += v;
            add += v;
        }
        if (b > B - 2 || add == 0) continue;
        const float qc = hist_q32<KMAX>(cl, cnode, N);
        if (qc < 0.0f) continue;
        if (qc > q1) {
            q2 = q1;
            q1 = qc;
            u1 = u;
        } else if (qc > q2) {
            q2 = qc;
        }
    }
    const float qmax = wave_max_f_dpp(q1);
    if (qmax < 0.0f) return lb;
    const float floor32 = fp32_floor(qmax);
    const bool fin = q1 >= floor32;
    const bool multi = fin && q2 >= floor32;
    if (__ballot(multi)) {
        if (multi) {
#pragma unroll
            for (int k = 0; k < KMAX; ++k) cl[k] = excl[k];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int b = b0 + u;
                uint32_t add = 0;
#pragma unroll
                for (int k = 0; k < KMAX; ++k) {
                    const uint32_t v = hval(k, u);
                    cl[k] += v;
                    add += v;
                }
                if (b > B - 2 || add == 0) continue;
                const float qc = hist_q32<KMAX>(cl, cnode, N);
                if (qc < floor32) continue;  // includes the empty-side -1
                const Cand c = make(b, cl);
                if (lb.nl == 0 || cand_better(c, lb)) lb = c;
            }
        }
    }
    if (fin && !multi) {
        // class counts left of bin b0 + u1
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            uint32_t v = excl[k];
#pragma unroll
            for (int u = 0; u < 4; ++u) v += u <= u1 ? hval(k, u) : 0u;
            cl[k] = v;
        }
        lb = make(b0 + u1, cl);
    }
    const unsigned long long finm = __ballot(lb.nl != 0);
    if (__popcll(finm) == 1) return shfl_cand(lb, (int)__ffsll(finm) - 1);
    return wave_best_exact(lb);
}

// Best threshold of one feature, compacted form (up to 4 classes): as
// feature_best, but the thresholds worth scoring (a non-empty bin below
// B - 1 with rows on both sides) are first packed into a dense list, so a
// node with few distinct bins costs one scoring round instead of four.  The
// list overwrites the feature's histogram h (read first); each entry is
// KMAX words, the bin in the top byte of the first (counts stay below 2^24).
// cl_out receives the winner's left class counts.
template <int KMAX>
__device__ Cand feature_best_compact(uint32_t* h, int B, int q, int f, const uint32_t* cnode,
                                     uint32_t N, int split_rank, uint32_t* cl_out) {
    static_assert(KMAX <= 4, "compact scan keeps four bins per class in registers");
    const int lane = threadIdx.x & 63;
    const int b0 = lane * 4;
    uint32_t hv[KMAX][4], excl[KMAX], a[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const uint4 v = *reinterpret_cast<const uint4*>(h + k * 256 + b0);
        hv[k][0] = v.x;
        hv[k][1] = v.y;
        hv[k][2] = v.z;
        hv[k][3] = v.w;
        a[k] = v.x + v.y + v.z + v.w;
    }
#pragma unroll
    for (int k = 0; k < KMAX; ++k) excl[k] = wave_incl_sum(a[k]) - a[k];
    // the lane's thresholds worth scoring: a non-empty bin below B - 1 with
    // rows on both sides (prefix counts are rebuilt in the writing pass)
    uint32_t okm = 0, cnt = 0;
    {
        uint32_t nl = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) nl += excl[k];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint32_t add = 0;
#pragma unroll
            for (int k = 0; k < KMAX; ++k) add += hv[k][u];
            nl += add;
            const bool ok = b0 + u <= B - 2 && add != 0 && nl != 0 && nl != N;
            okm |= (uint32_t)ok << u;
            cnt += ok;
        }
    }
    const uint32_t incl = wave_incl_sum(cnt);
    const int total = __builtin_amdgcn_readlane((int)incl, 63);
    uint32_t pos = incl - cnt;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // h has been read
    {
        uint32_t cl[KMAX];
#pragma unroll
        for (int k = 0; k < KMAX; ++k) cl[k] = excl[k];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int k = 0; k < KMAX; ++k) cl[k] += hv[k][u];
            if (okm >> u & 1u) {
#pragma unroll
                for (int k = 0; k < KMAX; ++k)
                    h[pos * KMAX + k] = cl[k] | (k == 0 ? (uint32_t)(b0 + u) << 24 : 0u);
                ++pos;
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    auto entry = [&](int e, uint32_t* c) {
#pragma unroll
        for (int k = 0; k < KMAX; ++k) c[k] = h[e * KMAX + k];
        const int b = (int)(c[0] >> 24);
        c[0] &= 0xFFFFFFu;
        return b;
    };
    auto make = [&](int b, const uint32_t* c) {
        Cand x;
        x.q = q;
        x.f = f;
        x.b = b;
        x.pad = 0;
        uint32_t nl = 0;
        uint64_t sl = 0, sr = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const uint32_t r = cnode[k] - c[k];
            nl += c[k];
            sl += (uint64_t)c[k] * c[k];
            sr += (uint64_t)r * r;
        }
        x.nl = nl;
        x.nr = N - nl;
        x.sl = sl;
        x.sr = sr;
        return x;
    };
    Cand lb;
    lb.nl = 0;
    lb.b = 0x7FFFFFFF;
    lb.q = q;
    lb.f = f;
    lb.nr = 0;
    lb.pad = 0;
    lb.sl = lb.sr = 0;
    uint32_t lcl[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) lcl[k] = 0;
    if (!split_rank) {
        // exact: each lane ranks its entries (ascending thresholds: a strictly
        // better score replaces, so ties keep the smaller threshold)
        for (int e = lane; e < total; e += 64) {
            uint32_t c[KMAX];
            const int b = entry(e, c);
            const Cand x = make(b, c);
            if (lb.nl == 0 || cand_better(x, lb)) {
                lb = x;
#pragma unroll
                for (int k = 0; k < KMAX; ++k) lcl[k] = c[k];
            }
        }
    } else {
        float q1 = -1.0f, q2 = -1.0f;
        int e1 = 0;
        for (int e = lane; e < total; e += 64) {
            uint32_t c[KMAX];
            (void)entry(e, c);
            const float qc = hist_q32<KMAX>(c, cnode, N);
            if (qc > q1) {
                q2 = q1;
                q1 = qc;
                e1 = e;
            } else if (qc > q2) {
                q2 = qc;
            }
        }
        const float qmax = wave_max_f_dpp(q1);
        if (qmax < 0.0f) return lb;
        const float floor32 = fp32_floor(qmax);
        const bool fin = q1 >= floor32;
        const bool multi = fin && q2 >= floor32;
        if (__ballot(multi)) {
            if (multi) {
                for (int e = lane; e < total; e += 64) {
                    uint32_t c[KMAX];
                    const int b = entry(e, c);
                    if (hist_q32<KMAX>(c, cnode, N) < floor32) continue;
                    const Cand x = make(b, c);
                    if (lb.nl == 0 || cand_better(x, lb)) {
                        lb = x;
#pragma unroll
                        for (int k = 0; k < KMAX; ++k) lcl[k] = c[k];
                    }
                }
            }
        }
        if (fin && !multi) {
            uint32_t c[KMAX];
            const int b = entry(e1, c);
            lb = make(b, c);
#pragma unroll
            for (int k = 0; k < KMAX; ++k) lcl[k] = c[k];
        }
    }
    const unsigned long long finm = __ballot(lb.nl != 0);
    if (!finm) return lb;
    int src;
    Cand w;
    if (__popcll(finm) == 1) {
        src = (int)__ffsll(finm) - 1;
        w = shfl_cand(lb, src);
    } else {
        w = wave_best_exact(lb);
        const unsigned long long m = __ballot(lb.nl != 0 && lb.b == w.b);
        src = (int)__ffsll(m) - 1;
    }
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        cl_out[k] = (uint32_t)__builtin_amdgcn_readlane((int)lcl[k], src);
    return w;
}

// ---------------------------------------------------------------------------
// Best threshold of one feature from a packed LDS histogram h[WORDS][256]:
// lane l owns bins 4l .. 4l+3, one 16-byte read per word, and a wave scan adds
// up the packed prefix counts.  Two forms:
//   * rows (nodes of at most 128 rows): the prefix counts go back to LDS and
//     every row scores the threshold at its own bin (rows lane and lane + 64,
//     bins b0 and b1): one or two scores per lane, however the rows spread
//     over bins;
//   * bins: every lane scores its four bins where they hold rows.
// The scan is what an item of a small node costs (an unpacked one of four
// classes takes four prefix scans and two passes over the bins): against one
// word per class k_hist_tile went from 82 to 62 us a launch at n = 10,000, 3
// classes, and from 353 to 225 us at 2,000 x 20,000, 2 classes.  l receives the
// packed left counts of the best threshold.
template <int WORDS, int FB, int NS>
__device__ __forceinline__ ItemBest scan_rows(uint32_t* h, uint32_t len, int b0, int b1, int B,
                                              const uint32_t* cn, uint32_t S, uint32_t N,
                                              int split_rank, uint32_t* l) {
    const int lane = threadIdx.x & 63;
    int rb[NS];
    rb[0] = b0;
    if constexpr (NS > 1) rb[1] = b1;
    uint4* h4 = reinterpret_cast<uint4*>(h);
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        uint4 v = h4[w * 64 + lane];
        v.y += v.x;
        v.z += v.y;
        v.w += v.z;
        const uint32_t ex = wave_incl_sum(v.w) - v.w;
        h4[w * 64 + lane] = make_uint4(v.x + ex, v.y + ex, v.z + ex, v.w + ex);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    float q[NS];
    Side sd[NS];
    bool ok[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        uint32_t a[WORDS];
#pragma unroll
        for (int w = 0; w < WORDS; ++w) a[w] = h[w * 256 + rb[u]];
        sd[u] = side_of<WORDS, FB>(a, cn, S);
        // nl >= the row's own weight
        ok[u] = (uint32_t)(lane + 64 * u) < len && rb[u] <= B - 2 && sd[u].nl < N;
        const float qu = side_q32(sd[u], N);  // unconditional: a select, no branch
        q[u] = ok[u] ? qu : -1.0f;
    }
    const ItemBest r = pick_threshold<FB, NS>(q, rb, sd, ok, N, split_rank);
#pragma unroll
    for (int w = 0; w < WORDS; ++w) l[w] = uniform(h[w * 256 + r.b]);
    return r;
}

template <int WORDS, int FB>
__device__ __forceinline__ ItemBest scan_bins(const uint32_t* h, int B, const uint32_t* cn,
                                              uint32_t S, uint32_t N, int split_rank,
                                              uint32_t* l) {
    const int lane = threadIdx.x & 63;
    const uint4* h4 = reinterpret_cast<const uint4*>(h);
    uint32_t p[4][WORDS];
    uint32_t own[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        const uint4 v = h4[w * 64 + lane];
        own[0] |= v.x;
        own[1] |= v.y;
        own[2] |= v.z;
        own[3] |= v.w;
        p[0][w] = v.x;
        p[1][w] = p[0][w] + v.y;
        p[2][w] = p[1][w] + v.z;
        p[3][w] = p[2][w] + v.w;
        const uint32_t ex = wave_incl_sum(p[3][w]) - p[3][w];
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u][w] += ex;
    }
    float q[4];
    int b[4];
    Side sd[4];
    bool ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        b[u] = lane * 4 + u;
        sd[u] = side_of<WORDS, FB>(p[u], cn, S);
        // an empty bin repeats the previous threshold's partition
        ok[u] = own[u] != 0 && b[u] <= B - 2 && sd[u].nl < N;
        const float qu = side_q32(sd[u], N);  // unconditional: a select, no branch
        q[u] = ok[u] ? qu : -1.0f;
    }
    const ItemBest r = pick_threshold<FB, 4>(q, b, sd, ok, N, split_rank);
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        uint32_t v = p[0][w];
#pragma unroll
        for (int u = 1; u < 4; ++u) v = b[u] == r.b ? p[u][w] : v;
        l[w] = readlane_w(v, r.b >> 2);
    }
    return r;
}

// Form of an item's histogram (count_bits): a row of class y and weight w adds
// w << (y & fm) * fb to word y >> fs of its bin; words: what the scan of K
// classes reads.
struct CountForm {
    uint32_t fb, fs, fm, words;
};
template <int KMAX>
__device__ __forceinline__ CountForm count_form(uint32_t N, uint32_t K) {
    const uint32_t fb = count_bits(KMAX, N);
    if (fb == 8u) return CountForm{8u, 2u, 3u, K <= 4u ? 1u : (K <= 8u ? 2u : 4u)};
    if (fb == 16u)
        return CountForm{16u, 1u, 1u, KMAX == 2 ? 1u : (K <= 4u ? 2u : (K <= 8u ? 4u : 8u))};
    return CountForm{0u, 0u, 0u, (uint32_t)KMAX};
}
template <int KMAX>
__device__ __forceinline__ void count_row(uint32_t* h, const CountForm& cf, uint32_t rec,
                                          uint32_t b) {
    const uint32_t y = rec_y(rec), w = rec_w(rec);
    if (KMAX <= 4 && cf.words == 1u)  // uniform
        atomicAdd(&h[b], w << (y * cf.fb));
    else
        atomicAdd(&h[(y >> cf.fs) * 256u + b], w << ((y & cf.fm) * cf.fb));
}

// Words of a histogram and of an item's left counts.
template <int KMAX, bool BIG>
__host__ __device__ constexpr int item_counts() {
    return BIG ? KMAX : pk_words(KMAX);
}

// Field k of left counts l in fb-bit form.
template <int KMAX, bool BIG>
__device__ __forceinline__ uint32_t left_count(const uint32_t* l, uint32_t fb, int k) {
    const uint32_t v16 = pk_field<16>(l, k);
    const uint32_t v8 = KMAX > 2 ? pk_field<8>(l, k) : v16;
    const uint32_t v = fb == 8u ? v8 : v16;
    return BIG && fb == 0u ? l[k] : v;
}

template <int KMAX, int WORDS, int FB>
__device__ __forceinline__ ItemBest scan_packed(uint32_t* h, uint32_t len, int b0, int b1, int B,
                                                const uint32_t* cn, uint32_t N, int split_rank,
                                                uint32_t* l) {
    uint32_t S = 0;
#pragma unroll
    for (int w = 0; w < WORDS; ++w) S = dotf<FB>(cn[w], cn[w], S);
    if ((FB == 8 || KMAX == 2) && len <= 64u)
        return scan_rows<WORDS, FB, 1>(h, len, b0, b1, B, cn, S, N, split_rank, l);
    if ((FB == 8 || KMAX == 2) && len <= 128u)
        return scan_rows<WORDS, FB, 2>(h, len, b0, b1, B, cn, S, N, split_rank, l);
    return scan_bins<WORDS, FB>(h, B, cn, S, N, split_rank, l);
}

// One feature's best threshold from its histogram in form cf: through the
// packed scans, or one word per class above a weight of 65535 (BIG: the plan
// may hold such nodes).  pk: the node's packed class counts, cnode: its plain
// ones; l: the best threshold's left class counts in the node's form.  b0, b1:
// the bins of rows lane and lane + 64 (nodes of at most 128 rows; those of
// 16-bit counts are larger but for odd weights).
template <int KMAX, bool BIG>
__device__ __forceinline__ ItemBest scan_item(uint32_t* h, const CountForm& cf, uint32_t K,
                                              uint32_t len, int b0, int b1, int B,
                                              const uint32_t* pk, const uint32_t* cnode,
                                              uint32_t N, int split_rank, uint32_t* l) {
    if (KMAX > 2 && cf.fb == 8u) {
        if constexpr (KMAX > 2) {
            if (KMAX <= 4 || K <= 4u)
                return scan_packed<KMAX, 1, 8>(h, len, b0, b1, B, pk, N, split_rank, l);
        }
        if constexpr (KMAX > 4) {
            if (KMAX <= 8 || K <= 8u)
                return scan_packed<KMAX, 2, 8>(h, len, b0, b1, B, pk, N, split_rank, l);
        }
        if constexpr (KMAX > 8)
            return scan_packed<KMAX, 4, 8>(h, len, b0, b1, B, pk, N, split_rank, l);
    }
    if (!BIG || cf.fb == 16u) {
        if constexpr (KMAX <= 2) {
            return scan_packed<KMAX, 1, 16>(h, len, b0, b1, B, pk, N, split_rank, l);
        } else {
            if (KMAX <= 4 || K <= 4u)
                return scan_packed<KMAX, 2, 16>(h, len, b0, b1, B, pk, N, split_rank, l);
            if constexpr (KMAX > 4) {
                if (KMAX <= 8 || K <= 8u)
                    return scan_packed<KMAX, 4, 16>(h, len, b0, b1, B, pk, N, split_rank, l);
            }
            if constexpr (KMAX > 8)
                return scan_packed<KMAX, 8, 16>(h, len, b0, b1, B, pk, N, split_rank, l);
        }
    }
    ItemBest r;
    r.q = -1.0f;
    r.b = 0;
    if constexpr (BIG) {
        Cand c;
        if constexpr (KMAX <= 4) {
            c = feature_best_compact<KMAX>(h, B, 0, 0, cnode, N, split_rank, l);
        } else {
            const int lane = threadIdx.x & 63;
            c = feature_best<KMAX>(h, B, 0, 0, cnode, N, split_rank);
            const int bt = c.nl != 0 ? c.b : -1;
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                const uint4 v4 = *reinterpret_cast<const uint4*>(h + k * 256 + lane * 4);
                const int bl = lane * 4;
                const uint32_t a = (bl <= bt ? v4.x : 0u) + (bl + 1 <= bt ? v4.y : 0u) +
                                   (bl + 2 <= bt ? v4.z : 0u) + (bl + 3 <= bt ? v4.w : 0u);
                l[k] = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(a), 63);
            }
        }
        if (c.nl != 0) {
            r.q = cand_q32(c);
            r.b = c.b;
        }
    }
    return r;
}

// Record of a classification item in F.icand, F.item_words words: the FP32
// score of its best threshold (negative: none), the threshold bin | the draw's
// place in the item << 8, and the left class counts in the node's form.
template <int KMAX, bool BIG>
__device__ __forceinline__ void put_item(const ForestDev& F, uint32_t item, const ItemBest& r,
                                         uint32_t draw, const uint32_t* l) {
    constexpr int C = item_counts<KMAX, BIG>();
    const int lane = threadIdx.x & 63;
    uint32_t v = lane == 0 ? __float_as_uint(r.q) : (uint32_t)r.b | draw << 8;
#pragma unroll
    for (int k = 0; k < C; ++k) v = lane == k + 2 ? l[k] : v;
    if (lane < C + 2) F.icand[(size_t)item * (uint32_t)F.item_words + lane] = v;
}

// Exact form of a threshold's left counts l (fb-bit form).
template <int KMAX, bool BIG>
__device__ __forceinline__ Cand cand_of(const uint32_t* l, uint32_t fb, int b,
                                        const uint32_t* cnode, uint32_t N) {
    Cand c;
    c.q = c.f = 0;
    c.pad = 0;
    c.b = b;
    uint32_t nl = 0;
    uint64_t sl = 0, sr = 0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const uint32_t x = left_count<KMAX, BIG>(l, fb, k), r = cnode[k] - x;
        nl += x;
        sl += (uint64_t)x * x;
        sr += (uint64_t)r * r;
    }
    c.nl = nl;
    c.nr = N - nl;
    c.sl = sl;
    c.sr = sr;
    return c;
}

// ---------------------------------------------------------------------------
// Regression items (a job of the float-target regressor).  For each of the
// item's drawn features in turn: an LDS histogram of the bootstrap weights
// W[256] (32-bit) and the weighted fixed-point target sums T[256] (64-bit LDS
// atomics, two's complement) over the node's rows, then the threshold scan.
// Lane l owns bins 4l .. 4l+3; prefix sums over the lanes give each
// threshold's left (W_L, T_L).  Thresholds are ranked by an FP64 score
// g^2 / (W_L W_R) (g = T_L W_R - T_R W_L) and every threshold within the
// ranking margin of the maximum is compared exactly (reg_cmp); with exact
// ranking every valid threshold is.
// In nodes of weight up to 2^15 every target sum is below 2^53: the prefix
// sums and scores stay in FP64 (reg_score); wider nodes (WIDE plans hold them)
// keep 64-bit integers and take the score from the 128-bit gap.
constexpr uint32_t kRegF64Weight = 1u << 15;

template <class T>
__device__ __forceinline__ T dpp_zero_shift(T v, int s) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    int lo = (int)(uint32_t)b, hi = (int)(uint32_t)(b >> 32);
    switch (s) {  // a constant where this is unrolled
#define BORUTA_DPP(S, CTRL, ROWS)                                         \
    case S:                                                               \
        lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROWS, 0xf, false);  \
        hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROWS, 0xf, false);  \
        break;
        BORUTA_DPP(0, 0x111, 0xf)
        BORUTA_DPP(1, 0x112, 0xf)
        BORUTA_DPP(2, 0x114, 0xf)
        BORUTA_DPP(3, 0x118, 0xf)
        BORUTA_DPP(4, 0x142, 0xa)
        BORUTA_DPP(5, 0x143, 0xc)
#undef BORUTA_DPP
    }
    return __builtin_bit_cast(T, (uint64_t)(uint32_t)lo | (uint64_t)(uint32_t)hi << 32);
}
template <class T>
__device__ __forceinline__ T wave_incl_sum64(T v) {
#pragma unroll
    for (int s = 0; s < 6; ++s) v += dpp_zero_shift(v, s);
    return v;
}

// V: the type of the target sums (double or int64_t).
template <class V>
__device__ __forceinline__ Cand reg_feature_best(const uint32_t* hw, const long long* ht, int B,
                                                 int q, int f, uint32_t W, int64_t T,
                                                 int split_rank) {
    const int lane = threadIdx.x & 63;
    const uint4 wv = reinterpret_cast<const uint4*>(hw)[lane];
    const longlong2 ta = reinterpret_cast<const longlong2*>(ht)[2 * lane],
                    tb = reinterpret_cast<const longlong2*>(ht)[2 * lane + 1];
    const uint32_t w4[4] = {wv.x, wv.y, wv.z, wv.w};
    uint32_t wl[4];
    V tl[4];
    wl[0] = wv.x;
    tl[0] = (V)ta.x;
    wl[1] = wl[0] + wv.y;
    tl[1] = tl[0] + (V)ta.y;
    wl[2] = wl[1] + wv.z;
    tl[2] = tl[1] + (V)tb.x;
    wl[3] = wl[2] + wv.w;
    tl[3] = tl[2] + (V)tb.y;
    const uint32_t wex = wave_incl_sum(wl[3]) - wl[3];
    const V tex = wave_incl_sum64(tl[3]) - tl[3];
    Cand c;
    c.q = q;
    c.f = f;
    c.pad = 0;
    double qs[4], q1 = -1.0;
    bool ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        wl[u] += wex;
        tl[u] += tex;
        ok[u] = lane * 4 + u <= B - 2 && w4[u] != 0 && wl[u] != W;
        double s;
        if constexpr (std::is_same<V, double>::value) {
            s = reg_score(tl[u], (double)wl[u], (double)T, (double)W);
        } else {
            c.nl = ok[u] ? wl[u] : 1u;
            c.nr = W - c.nl;
            c.sl = (uint64_t)tl[u];
            c.sr = (uint64_t)(T - tl[u]);
            s = reg_q64(c);
        }
        qs[u] = ok[u] ? s : -1.0;
        q1 = fmax(q1, qs[u]);
    }
    const double qmax = wave_max_f64_dpp(q1);
    c.nl = 0;
    c.nr = 0;
    c.b = 0x7FFFFFFF;
    c.sl = c.sr = 0;
    if (qmax < 0.0) return c;
    const double floor64 = split_rank ? fp64_floor(qmax) : 0.0;
    uint32_t fin = 0;  // the lane's finalists
#pragma unroll
    for (int u = 0; u < 4; ++u) fin |= (uint32_t)(ok[u] && qs[u] >= floor64) << u;
    // candidate of the lane's threshold u
    auto cand = [&](int u, Cand& o) {
        const V t = u == 0 ? tl[0] : (u == 1 ? tl[1] : (u == 2 ? tl[2] : tl[3]));
        const uint32_t w = u == 0 ? wl[0] : (u == 1 ? wl[1] : (u == 2 ? wl[2] : wl[3]));
        o.b = lane * 4 + u;
        o.nl = w;
        o.nr = W - w;
        o.sl = (uint64_t)(int64_t)t;
        o.sr = (uint64_t)(T - (int64_t)t);
    };
    const unsigned long long fm = __ballot(fin != 0);
    Cand best = c;
    if (fin) {  // in ascending threshold order: a strictly better one replaces
        cand(__builtin_ctz(fin), best);
#pragma unroll 1
        for (uint32_t m = fin & (fin - 1u); m; m &= m - 1u) {
            Cand o = c;
            cand(__builtin_ctz(m), o);
            if (reg_cmp(o, best) > 0) best = o;
        }
    }
    if (__popcll(fm) == 1) return shfl_cand(best, (int)__ffsll(fm) - 1);
#pragma unroll 1
    for (int m = 1; m < 64; m <<= 1) {
        const Cand o = shfl_xor_cand(best, m);
        if (o.nl == 0) continue;
        const int s = best.nl == 0 ? 1 : reg_cmp(o, best);
        if (s > 0 || (s == 0 && o.b < best.b)) best = o;
    }
    return best;
}

// One regression item: draws q0 .. q0 + nf - 1 of the node, one after the
// other in the wave's LDS region (256 words of W, then 256 64-bit sums).  The
// rows' weighted targets stream beside their records.
template <int RB, bool WIDE>
__device__ __forceinline__ Cand reg_item(const ForestDev& F, const SlotRec& sr, int q0, int nf,
                                         const int* fq, const uint8_t* const* col,
                                         uint32_t* hist) {
    const int lane = threadIdx.x & 63;
    uint32_t* hw = hist;
    long long* ht = reinterpret_cast<long long*>(hist + 256);
    const int64_t T = (int64_t)((uint64_t)sr.cnode[0] | ((uint64_t)sr.cnode[1] << 32));
    const uint32_t W = sr.n, len = sr.len;
    const int64_t* wy = sr.wy;
    const uint32_t* recs = sr.recs;
    Cand best;
    best.nl = 0;
    for (int v = 0; v < nf; ++v) {
        reinterpret_cast<uint4*>(hw)[lane] = make_uint4(0u, 0u, 0u, 0u);
        reinterpret_cast<uint4*>(ht)[lane] = make_uint4(0u, 0u, 0u, 0u);
        reinterpret_cast<uint4*>(ht)[64 + lane] = make_uint4(0u, 0u, 0u, 0u);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        auto batch = [&](uint32_t i0, auto nb) {
            constexpr int NB = decltype(nb)::value;
            uint32_t r[NB];
            int64_t t[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const uint32_t i = min(i0 + u * 64 + lane, len - 1u);
                r[u] = rec_raw(recs, i, len);
                t[u] = ldg(reinterpret_cast<const int64_t*>(
                    reinterpret_cast<const char*>(wy) + i * 8u));
            }
            uint32_t b[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) b[u] = ldg(col[v] + rec_row(r[u]));
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                if (i0 + u * 64 + lane < len) {
                    atomicAdd(&hw[b[u]], rec_w(r[u]));
                    atomicAdd(reinterpret_cast<unsigned long long*>(&ht[b[u]]),
                              (unsigned long long)t[u]);
                }
            }
        };
        if (len <= 128u)
            batch(0u, std::integral_constant<int, 2>{});
        else
            for (uint32_t i0 = 0; i0 < len; i0 += 64 * RB)
                batch(i0, std::integral_constant<int, RB>{});
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        Cand fb;
        if (WIDE && W > kRegF64Weight)
            fb = reg_feature_best<int64_t>(hw, ht, (int)sr.B, q0 + v, fq[v], W, T, F.split_rank);
        else
            fb = reg_feature_best<double>(hw, ht, (int)sr.B, q0 + v, fq[v], W, T, F.split_rank);
        // draws in order: a strictly better score replaces
        if (fb.nl != 0 && (best.nl == 0 || reg_better(fb, best))) best = fb;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the next draw rewrites
    }
    return best;
}

// Large nodes, phase 0: each node's mtry drawn features (the keyed
// permutation of its heap id, in draw order), their bin columns and the
// node's slot record.  A wavefront serves 64 / S nodes at once, S = the
// plan's draws per node rounded up to a power of two (at most 64): lane l
// takes the draws l mod S, l mod S + S, ... of node l / S, so few draws per
// node do not leave most of the lanes idle.  When the permutation's round
// functions fit the segment's table (rounds << half 16-bit entries, at most
// F.draw_tab: halves of up to 8 bits, at most 2^16 widened columns), the
// node's lane segment first tabulates them in LDS: each lane then evaluates
// a few round functions, uniformly, instead of every round of every
// cycle-walking step of its draws, where the segment waits for its longest
// walk.
__global__ __launch_bounds__(256) void k_draws(ForestDev F, int level) {
    extern __shared__ uint16_t dtab[];  // [256 / S][F.draw_tab]
    const uint32_t count = level_slots(F, level);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t S = F.draw_seg, G = 64u / S;
    const uint32_t sub = lane / S, ql = lane % S;
    const uint32_t w0 = blockIdx.x * 4u + uniform(threadIdx.x >> 6);
    uint16_t* tab = dtab + (size_t)(threadIdx.x / S) * F.draw_tab;
    for (uint32_t base = w0 * G; base < count; base += gridDim.x * 4u * G) {
        const uint32_t slot = base + sub;
        if (slot >= count) continue;
        const uint32_t id = F.slot_node_in[slot];
        const NodeDev nd = F.nodes[id];
        const TreeDev tr = F.trees[nd.tree];
        const JobDev& J = F.jobs[tr.job];
        const KeyedPerm P = make_perm(J.seed_lo, J.seed_hi, kMtry, (uint32_t)J.t,
                                      (uint32_t)tr.tau, nd.heap, 0u, (uint64_t)J.p_w);
        uint32_t* out = F.feat + (size_t)slot * F.mtry_cap;
        const uint8_t** oc = F.fcol + (size_t)slot * F.mtry_cap;
        uint32_t* pos = F.fpos + (size_t)slot * F.mtry_cap;
        const bool use_tab = (P.rounds << P.half) <= F.draw_tab;  // uniform over the segment
        if (use_tab) {
            // the previous node's lookups of this segment are done (program order)
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            for (uint32_t e = ql; e < (P.rounds << P.half); e += S)
                tab[e] = (uint16_t)perm_round(P, e >> P.half, e & P.mask);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
        for (uint32_t q = ql; q < (uint32_t)J.mtry; q += S) {
            const uint32_t f = use_tab ? perm_apply_tab(P, tab, q) : perm_apply(P, q);
            out[q] = f;
            oc[q] = ldg(J.colptr + f);
            // column-major path without k_col_count: the item's place among
            // its column's items
            if (F.col_count == 1) pos[q] = atomicAdd(F.fcnt + J.gbase + f, 1u);
        }
        SlotRec* sr = F.srec + slot;
        for (uint32_t c = ql; c < 16u; c += S)
            sr->cnode[c] = c < (uint32_t)J.K ? F.cls[(size_t)id * F.kmax + c] : 0u;
        const uint32_t fb = count_bits(F.kmax, nd.n), per = fb == 8u ? 4u : 2u;
        for (uint32_t w = ql; w < 8u; w += S) {
            uint32_t v = 0;
            for (uint32_t k = 0; k < per; ++k)
                if (w * per + k < (uint32_t)J.K)
                    v |= F.cls[(size_t)id * F.kmax + w * per + k] << (fb * k);
            sr->pk[w] = J.reg || fb == 0u ? 0u : v;
        }
        if (ql == 0) {
            if (F.col_count && nd.n >= 65536u) {  // too heavy for k_hist_col
                const uint32_t at = atomicAdd(&F.ctrs[level].n_big, 1u);
                if (at < F.big_cap) F.big[at] = slot;
            }
            sr->recs = J.rec[F.parity] + (size_t)tr.tau * J.rstride + nd.seg;
            sr->wy = J.reg ? J.wy[F.parity] + (size_t)tr.tau * J.rstride + nd.seg : nullptr;
            sr->id = id;
            sr->len = nd.len;
            sr->n = nd.n;
            sr->mtry = (uint32_t)J.mtry;
            sr->B = (uint32_t)J.B;
            sr->reg = (uint32_t)J.reg;
            sr->K = (uint32_t)J.K;
        }
    }
}

// Large nodes, phase 1: one wavefront per (node, FW consecutive draws)
// item, with its own LDS histograms, F.hist_words words per bin and draw: the
// class counts packed two or four to a word, or one word per class where the
// plan may hold nodes of weight 65536 and more (2 KB per draw of 3 or 4 classes,
// 1 KB of 2).  The wave gathers the bins of its features at the node's rows,
// adds each row's weight to its class's field with an LDS atomic, scans each
// feature and writes the record of the item's best threshold (put_item).  No
// barriers: the four waves of a workgroup are independent.
// Work of a level for the node-major histogram kernels: node slots [0, n)
// with npi items each.  Workgroup b takes the slots congruent to b mod 8 (the
// grid is a multiple of 8), and its waves walk those slots' items in order,
// so a node's items run side by side in one XCD and share its records
// through that XCD's L2 when the hardware deals workgroups round-robin to the
// 8 XCDs (any mapping gives the same results: every item is visited once).
// With an explicit count, items [first, first + count) are walked directly
// (plain form); kBigItems: the items of the level's F.big slots.
constexpr uint32_t kBigItems = 0xFFFFFFFEu;
struct ItemWalk {
    bool dyn;
    const uint32_t* big;
    uint32_t x, r, R, m_end, first, npi;
    __device__ ItemWalk(const ForestDev& F, int level, uint32_t first_, uint32_t count,
                        uint32_t wave) {
        npi = (uint32_t)F.npi;
        first = first_;
        dyn = count == 0xFFFFFFFFu;
        big = count == kBigItems ? F.big : nullptr;
        x = 0;
        r = blockIdx.x * 4u + wave;
        R = gridDim.x * 4u;
        m_end = big ? min(F.ctrs[level].n_big, F.big_cap) * npi : count;
        if (dyn) {
            const uint32_t n_slots = level_slots(F, level);
            x = blockIdx.x % 8u;
            r = (blockIdx.x / 8u) * 4u + wave;
            R = (gridDim.x / 8u) * 4u;
            m_end = n_slots > x ? (n_slots - x + 7u) / 8u * npi : 0u;
        }
    }
    __device__ uint32_t item(uint32_t cur) const {
        if (big) return big[cur / npi] * npi + cur % npi;
        return dyn ? (8u * (cur / npi) + x) * npi + cur % npi : first + cur;
    }
};

// Regression nodes of the node-major levels: one wavefront per (node, F.fw
// consecutive draws) item, the histograms and scan of reg_item in the wave's
// LDS region (F.fw * F.hist_words * 256 words, at least 768).  Items of
// classification nodes are left to k_hist_tile, which in turn skips these:
// the regression item's registers and code stay out of the classification
// kernel.
template <int RB, bool WIDE>
__global__ __launch_bounds__(256) void k_hist_reg(ForestDev F, int level, uint32_t first,
                                                  uint32_t count) {
    extern __shared__ uint4 lds_raw[];
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    const int fw = F.fw;
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds_raw) +
                     (size_t)wave * max(fw * F.hist_words * 256, 768);
    const ItemWalk wk(F, level, first, count, (uint32_t)wave);
    unsigned long long alg = 0;
    for (uint32_t cur = wk.r; cur < wk.m_end; cur += wk.R) {
        const uint32_t item = wk.item(cur);
        const uint32_t slot = item / wk.npi, j = item % wk.npi;
        const SlotRec& sr = F.srec[slot];
        if (!sr.reg) continue;  // a classification node: k_hist_tile
        const int q0 = (int)j * fw;
        const int mtry = (int)sr.mtry;
        if (q0 >= mtry) continue;  // the job draws fewer features this iteration
        const int nf = min(fw, mtry - q0);
        const uint32_t* drawn = F.feat + (size_t)slot * F.mtry_cap + q0;
        const uint8_t* const* dcol = F.fcol + (size_t)slot * F.mtry_cap + q0;
        int fq[4];
        const uint8_t* col[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            fq[u] = (int)drawn[u < nf ? u : 0];
            col[u] = dcol[u < nf ? u : 0];
        }
        const Cand best = reg_item<RB, WIDE>(F, sr, q0, nf, fq, col, hist);
        if (lane == 0) F.cand[item] = best;
        alg += (unsigned long long)sr.len * (unsigned long long)(nf + (j == 0 ? 6 : 0));
    }
    if (F.alg_bytes && lane == 0 && alg)
        atomicAdd((unsigned long long*)&F.alg_bytes[(blockIdx.x * 4u + wave) & (kAlgWords - 1)],
                  alg);
}

template <int KMAX, int FW, int RB, bool BIG>
__global__ __launch_bounds__(256) void k_hist_tile(ForestDev F, int level, uint32_t first,
                                                   uint32_t count) {
    // RB rows per lane per batch: RB record loads and RB * FW bin gathers in
    // flight (a launch tuning choice; every RB gives the same histograms)
    extern __shared__ uint4 lds_raw[];
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    const uint32_t hw = (uint32_t)F.hist_words;  // LDS words per bin and feature
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds_raw) + (size_t)wave * FW * hw * 256u;
    const ItemWalk wk(F, level, first, count, (uint32_t)wave);
    const uint32_t npi = wk.npi;
    unsigned long long alg = 0;
    for (uint32_t cur = wk.r; cur < wk.m_end; cur += wk.R) {
        const uint32_t item = wk.item(cur);
        const uint32_t slot = item / npi, j = item % npi;
        const SlotRec& sr = F.srec[slot];
        if (sr.reg) continue;  // a regression node: k_hist_reg
        const int q0 = (int)j * FW;
        const int mtry = (int)sr.mtry;
        if (q0 >= mtry) continue;  // the job draws fewer features this iteration
        const int nf = min(FW, mtry - q0);
        const uint8_t* const* dcol = F.fcol + (size_t)slot * F.mtry_cap + q0;
        const uint8_t* col[FW];
#pragma unroll
        for (int u = 0; u < FW; ++u) col[u] = dcol[u < nf ? u : 0];
        const uint32_t N = sr.n, K = sr.K;
        const CountForm cf = count_form<KMAX>(N, K);
#pragma unroll
        for (int v = 0; v < FW; ++v)
            for (uint32_t i = 0; i < cf.words; ++i)
                reinterpret_cast<uint4*>(hist + v * hw * 256u)[i * 64u + lane] =
                    make_uint4(0u, 0u, 0u, 0u);
        const uint32_t* recs = sr.recs;
        const uint32_t len = sr.len;
        int b0[FW], b1[FW];  // bins of rows lane and lane + 64 (nodes of at most 128 rows)
        // One batch of NB rows per lane: all record loads, then all bin
        // gathers, then the counts.  (Loading the next batch's records ahead
        // of this batch's gathers was measured slower here: the other waves
        // of the SIMD hide the latency.)
        auto batch = [&](uint32_t i0, auto nb) {
            constexpr int NB = decltype(nb)::value;
            uint32_t r[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) r[u] = rec_raw(recs, i0 + u * 64 + lane, len);
            uint32_t b[NB][FW];
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int v = 0; v < FW; ++v) b[u][v] = ldg(col[v] + rec_row(r[u]));
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                if (i0 + u * 64 + lane >= len) continue;
#pragma unroll
                for (int v = 0; v < FW; ++v)
                    if (v < nf) count_row<KMAX>(hist + v * hw * 256u, cf, r[u], b[u][v]);
            }
#pragma unroll
            for (int v = 0; v < FW; ++v) {
                b0[v] = (int)b[0][v];
                b1[v] = (int)b[1][v];
            }
        };
        if (len <= 128u)
            batch(0u, std::integral_constant<int, 2>{});
        else
            for (uint32_t i0 = 0; i0 < len; i0 += 64 * RB)
                batch(i0, std::integral_constant<int, RB>{});
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        constexpr int C = item_counts<KMAX, BIG>();
        uint32_t cnode[KMAX], pk[pk_words(KMAX)];
#pragma unroll
        for (int c = 0; c < KMAX; ++c) cnode[c] = sr.cnode[c];
#pragma unroll
        for (int c = 0; c < pk_words(KMAX); ++c) pk[c] = sr.pk[c];
        const int B = (int)sr.B;
        ItemBest best;
        best.q = -1.0f;
        best.b = 0;
        uint32_t bi = 0;
        uint32_t best_l[C];
#pragma unroll
        for (int c = 0; c < C; ++c) best_l[c] = 0;
#pragma unroll
        for (int v = 0; v < FW; ++v) {
            if (v >= nf) break;
            uint32_t l[C];
#pragma unroll
            for (int c = 0; c < C; ++c) l[c] = 0;
            const ItemBest fb = scan_item<KMAX, BIG>(hist + v * hw * 256u, cf, K, len, b0[v],
                                                     b1[v], B, pk, cnode, N, F.split_rank, l);
            if (fb.q < 0.0f) continue;
            // draws in order: a strictly better score replaces
            bool better = best.q < 0.0f;
            if (FW > 1 && !better) {
                if (F.split_rank && (fb.q < fp32_floor(best.q) || best.q < fp32_floor(fb.q)))
                    better = fb.q > best.q;
                else
                    better = cand_better(cand_of<KMAX, BIG>(l, cf.fb, fb.b, cnode, N),
                                         cand_of<KMAX, BIG>(best_l, cf.fb, best.b, cnode, N));
            }
            if (better) {
                best = fb;
                bi = (uint32_t)v;
#pragma unroll
                for (int c = 0; c < C; ++c) best_l[c] = l[c];
            }
        }
        put_item<KMAX, BIG>(F, item, best, bi, best_l);
        alg += (unsigned long long)len * (unsigned long long)(nf + (j == 0 ? 6 : 0));
        // the histogram is rewritten by the wave's next item
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    // one atomic per wave for the statistics
    if (F.alg_bytes && lane == 0 && alg)
        atomicAdd((unsigned long long*)&F.alg_bytes[(blockIdx.x * 4u + wave) & (kAlgWords - 1)],
                  alg);
}

// ---------------------------------------------------------------------------
// Column-major histogram path.  At deep levels the nodes are small and a
// node-major gather pulls one cache line per row and drawn feature from a
// column far larger than the node; here the items (node, draw) of a level are
// bucketed by bin column instead, and each workgroup stages one column in LDS
// once and serves the histograms of a run of that column's items from it.
//
// k_col_scan (one workgroup): exclusive offsets of the per-column item counts
// that k_draws accumulated, the units (runs of at most col_unit items of one
// column), and zero counts for the next level.
__global__ __launch_bounds__(256) void k_col_scan(ForestDev F, int level) {
    __shared__ uint32_t s_i[4], s_u[4];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t G = F.n_gcol, U = F.col_unit;
    const uint32_t C = (G + 255u) / 256u;
    const uint32_t a = min(G, tid * C), b = min(G, a + C);
    uint32_t si = 0, su = 0;
    for (uint32_t g = a; g < b; ++g) {
        const uint32_t c = F.fcnt[g];
        si += c;
        su += (c + U - 1u) / U;
    }
    const uint32_t ii = wave_incl_sum(si), iu = wave_incl_sum(su);
    if (lane == 63) {
        s_i[wave] = ii;
        s_u[wave] = iu;
    }
    __syncthreads();
    uint32_t oi = ii - si, ou = iu - su, tu = 0;
    for (uint32_t v = 0; v < 4; ++v) {
        if (v < wave) {
            oi += s_i[v];
            ou += s_u[v];
        }
        tu += s_u[v];
    }
    for (uint32_t g = a; g < b; ++g) {
        const uint32_t c = F.fcnt[g];
        F.fcnt[g] = 0;
        F.fpos[(size_t)F.slot_cap * F.mtry_cap + g] = oi;  // column offsets follow the places
        const uint32_t gq = F.gcol_q[g];
        for (uint32_t k = 0; k * U < c; ++k) {
            if (ou < F.unit_cap) {
                ColUnit cu;
                cu.begin = oi + k * U;
                cu.end = oi + min(c, (k + 1u) * U);
                cu.gq = gq;
                cu.pad = 0;
                F.units[ou] = cu;
            }
            ++ou;
        }
        oi += c;
    }
    if (tid == 0) {
        if (tu > F.unit_cap) atomicOr(&F.ctrs[level].overflow, 16u);
        F.ctrs[level].n_units = min(tu, F.unit_cap);
    }
}

// k_col_count: the items' places within their columns, counted per workgroup
// in LDS.  Workgroup w takes a contiguous run of the level's node slots,
// ranks each item among the workgroup's items of its column (LDS atomics),
// reserves one run per touched column in the global per-column counts (one
// global atomic per column and workgroup, not one per item), then adds the
// run's start to its items' places.  The places of a column's items are
// unique and dense; their order is immaterial.
__global__ __launch_bounds__(256) void k_col_count(ForestDev F, int level) {
    extern __shared__ uint32_t lcnt[];  // [n_gcol]
    const uint32_t count = level_slots(F, level);
    const uint32_t G = F.n_gcol;
    const uint32_t per = (count + gridDim.x - 1u) / gridDim.x;
    const uint32_t s0 = min(count, blockIdx.x * per), s1 = min(count, s0 + per);
    if (s0 >= s1) return;  // the whole workgroup: no barrier is skipped by part of it
    for (uint32_t g = threadIdx.x; g < G; g += blockDim.x) lcnt[g] = 0u;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, wave = uniform(threadIdx.x >> 6);
    for (uint32_t slot = s0 + wave; slot < s1; slot += 4u) {
        const SlotRec& sr = F.srec[slot];
        const NodeDev nd = F.nodes[uniform(sr.id)];
        const uint32_t gb = F.jobs[F.trees[nd.tree].job].gbase;
        const size_t row = (size_t)slot * F.mtry_cap;
        for (uint32_t q = lane; q < sr.mtry; q += 64u)
            F.fpos[row + q] = atomicAdd(&lcnt[gb + F.feat[row + q]], 1u);
    }
    __syncthreads();
    for (uint32_t g = threadIdx.x; g < G; g += blockDim.x) {
        const uint32_t c = lcnt[g];
        lcnt[g] = c ? atomicAdd(F.fcnt + g, c) : 0u;
    }
    __syncthreads();
    for (uint32_t slot = s0 + wave; slot < s1; slot += 4u) {
        const SlotRec& sr = F.srec[slot];
        const NodeDev nd = F.nodes[uniform(sr.id)];
        const uint32_t gb = F.jobs[F.trees[nd.tree].job].gbase;
        const size_t row = (size_t)slot * F.mtry_cap;
        for (uint32_t q = lane; q < sr.mtry; q += 64u)
            F.fpos[row + q] += lcnt[gb + F.feat[row + q]];
    }
}

// k_col_scatter: one wavefront per large node; each drawn item goes to its
// column's run of the sorted list (order within a run is immaterial: every
// item writes only its own candidate).
__global__ __launch_bounds__(256) void k_col_scatter(ForestDev F, int level) {
    const uint32_t count = level_slots(F, level);
    const int lane = threadIdx.x & 63;
    const uint32_t* off = F.fpos + (size_t)F.slot_cap * F.mtry_cap;
    for (uint32_t slot = blockIdx.x * 4u + uniform(threadIdx.x >> 6); slot < count;
         slot += gridDim.x * 4u) {
        const SlotRec& sr = F.srec[slot];
        const NodeDev nd = F.nodes[uniform(sr.id)];
        const uint32_t gb = F.jobs[F.trees[nd.tree].job].gbase;
        const size_t row = (size_t)slot * F.mtry_cap;
        for (uint32_t q = lane; q < sr.mtry; q += 64) {
            const uint32_t dst = off[gb + F.feat[row + q]] + F.fpos[row + q];
            F.fitems[dst] = (uint32_t)(row + q);
        }
    }
}

// k_hist_col: grid-stride over units.  The workgroup copies the unit's bin
// column into LDS (16-byte loads, the whole column once), then each wave
// takes the unit's items in turn: an LDS class-count histogram from the node's
// row records and the staged bins, the threshold scan, and the item's record
// (item = slot * mtry_cap + draw).  Class counts take 16 bits at most: the items
// of a node of weight 65536 and more (F.big) are left to k_hist_tile, so that
// the histograms take two classes to a word (79 instead of 107 registers, half the
// LDS per wave; 100,000 x 2,000, 3 iterations: 148.4 -> 143.9 ms).
// Bound: the records (4 bytes per row and draw, mostly from the last-level
// cache) at the shallow levels, the vector instructions of the scan at the
// deep ones.  The first two records per lane of the wave's next item are
// loaded while this item is scanned, always and into the same registers: a
// conditional load here is waited for where its paths join.  With 4-byte
// instead of 8-byte records and the prefetch in flight a launch takes 2.42
// instead of 2.69 ms (n = 100,000, 2,000 features, mean of tree levels 5-15).
template <int KMAX>
__global__ __launch_bounds__(1024) void k_hist_col(ForestDev F, int level, uint32_t col_words) {
    constexpr int RB = 8, C = pk_words(KMAX);
    extern __shared__ uint4 lds_raw[];  // the column (col_words 16-byte words), the histograms
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    const uint32_t nw = blockDim.x >> 6;
    uint4* colq = lds_raw;
    const uint8_t* colb = reinterpret_cast<const uint8_t*>(colq);
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds_raw + col_words) + wave * C * 256;
    const LevelCtr& lc = F.ctrs[level];
    const uint32_t n_units = lc.overflow ? 0u : min(lc.n_units, F.unit_cap);
    const uint32_t mc = (uint32_t)F.mtry_cap;
    unsigned long long alg = 0;
    for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
        const ColUnit cu = F.units[u];
        const uint32_t item0 = F.fitems[cu.begin];
        const uint4* src = reinterpret_cast<const uint4*>(F.fcol[item0]);
        const uint32_t K = F.srec[item0 / mc].K;  // a column's items are of one job
        const int B = (int)F.srec[item0 / mc].B;
        for (uint32_t i = threadIdx.x; i < cu.gq; i += blockDim.x) colq[i] = src[i];
        __syncthreads();
        // The wave's items are k0 + t * nw; their node records are loaded
        // one per lane, 64 at a time, and read back with readlane.
        for (uint32_t k0 = cu.begin + (uint32_t)wave; k0 < cu.end; k0 += 64u * nw) {
            const uint32_t kk = k0 + (uint32_t)lane * nw;
            const bool have = kk < cu.end;
            const uint32_t my_item = F.fitems[have ? kk : k0];
            const SlotRec* msr = F.srec + my_item / mc;
            const uint64_t my_recs = reinterpret_cast<uint64_t>(msr->recs);
            const uint32_t my_len = msr->len, my_n = msr->n;
            uint32_t my_pk[C];
#pragma unroll
            for (int c = 0; c < C; ++c) my_pk[c] = msr->pk[c];
            const uint32_t n_here = min(64u, (cu.end - k0 + nw - 1u) / nw);
            auto recs_of = [&](uint32_t t) {
                return reinterpret_cast<const uint32_t*>(readlane64(my_recs, (int)t));
            };
            uint32_t p0, p1;  // records lane and lane + 64 of the next item
            {
                const uint32_t len = readlane_w(my_len, 0);
                p0 = rec_raw(recs_of(0), (uint32_t)lane, len);
                p1 = rec_raw(recs_of(0), (uint32_t)lane + 64u, len);
            }
            for (uint32_t t = 0; t < n_here; ++t) {
                const uint32_t item = readlane_w(my_item, (int)t);
                const uint32_t len = readlane_w(my_len, (int)t), N = readlane_w(my_n, (int)t);
                const CountForm cf = count_form<KMAX>(N, K);
#pragma unroll
                for (int i = 0; i < C; ++i)
                    if ((uint32_t)i < cf.words)
                        reinterpret_cast<uint4*>(hist)[i * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
                const uint32_t* recs = recs_of(t);
                uint32_t rn[RB];  // a larger item's next batch
                if (len > 128u) {
#pragma unroll
                    for (int v = 0; v < RB; ++v) rn[v] = rec_raw(recs, 128u + v * 64 + lane, len);
                }
                const uint32_t r0 = p0, r1 = p1;
                const int b0 = colb[rec_row(r0)], b1 = colb[rec_row(r1)];
                {
                    const uint32_t tn = min(t + 1u, n_here - 1u);
                    const uint32_t nlen = readlane_w(my_len, (int)tn);
                    p0 = rec_raw(recs_of(tn), (uint32_t)lane, nlen);
                    p1 = rec_raw(recs_of(tn), (uint32_t)lane + 64u, nlen);
                }
                if (N >= 65536u) continue;
                if ((uint32_t)lane < len) count_row<KMAX>(hist, cf, r0, (uint32_t)b0);
                if ((uint32_t)lane + 64u < len) count_row<KMAX>(hist, cf, r1, (uint32_t)b1);
                if (len > 128u) {
                    for (uint32_t i0 = 128u;;) {
                        uint32_t r[RB];
#pragma unroll
                        for (int v = 0; v < RB; ++v) r[v] = rn[v];
                        const uint32_t i1 = i0 + 64 * RB;
                        if (i1 < len) {
#pragma unroll
                            for (int v = 0; v < RB; ++v)
                                rn[v] = rec_raw(recs, i1 + v * 64 + lane, len);
                        }
                        // all bins of the batch first, then the counts: one
                        // LDS round trip for the batch, not one per row
                        uint32_t bb[RB];
#pragma unroll
                        for (int v = 0; v < RB; ++v) bb[v] = colb[rec_row(r[v])];
#pragma unroll
                        for (int v = 0; v < RB; ++v)
                            if (i0 + (uint32_t)(v * 64 + lane) < len)
                                count_row<KMAX>(hist, cf, r[v], bb[v]);
                        if (i1 >= len) break;
                        i0 = i1;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                uint32_t pk[C], l[C];
#pragma unroll
                for (int c = 0; c < C; ++c) pk[c] = readlane_w(my_pk[c], (int)t);
#pragma unroll
                for (int c = 0; c < C; ++c) l[c] = 0;
                const ItemBest best = scan_item<KMAX, false>(hist, cf, K, len, b0, b1, B, pk,
                                                             nullptr, N, F.split_rank, l);
                put_item<KMAX, false>(F, item, best, 0u, l);
                if (F.alg_bytes)
                    alg += (unsigned long long)len * (item % mc == 0u ? 7ull : 1ull);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            }
        }
        __syncthreads();  // the column is replaced by the next unit's
    }
    if (F.alg_bytes && lane == 0 && alg)
        atomicAdd((unsigned long long*)&F.alg_bytes[2 * kAlgWords +
                                                    ((blockIdx.x * nw + wave) & (kAlgWords - 1))],
                  alg);
}

// Partition of a split node's first `len` row records in one pass: left rows
// (bin <= b) from the front in row order, right rows from the back in reverse
// row order (no result depends on a node's row order, and each child segment
// stays monotone in row index for the next level's gathers); returns the
// left rows.  len = 0 when neither child is searched again.  Lanes take
// consecutive records (coalesced reads, and writes that a ballot packs), 64 at
// a time, up to 8 such groups in flight; REG: the weighted targets move along.
template <bool REG>
__device__ __forceinline__ uint32_t partition_rows(const ForestDev& F, const JobDev& J,
                                                   const TreeDev& tr, const NodeDev& nd,
                                                   const uint32_t* recs, const int64_t* wy,
                                                   const Cand& best, const uint8_t* col,
                                                   uint32_t len) {
    const uint32_t lane = threadIdx.x & 63u;
    const size_t seg = (size_t)tr.tau * J.rstride + nd.seg;
    uint32_t* rout = J.rec[F.parity ^ 1] + seg;
    int64_t* wout = REG ? J.wy[F.parity ^ 1] + seg : nullptr;
    uint32_t runl = 0, runr = 0;
    auto block = [&](uint32_t blk, auto nb) {
        constexpr int NB = decltype(nb)::value;
        uint32_t r[NB];
        int64_t t[REG ? NB : 1];
#pragma unroll
        for (int u = 0; u < NB; ++u) r[u] = rec_raw(recs, blk + u * 64 + lane, len);
        if constexpr (REG) {
#pragma unroll
            for (int u = 0; u < NB; ++u)
                t[u] = ldg(reinterpret_cast<const int64_t*>(
                    reinterpret_cast<const char*>(wy) + min(blk + u * 64 + lane, len - 1u) * 8u));
        }
        int bb[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) bb[u] = (int)ldg(col + rec_row(r[u]));
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const bool in = blk + u * 64 + lane < len, left = in && bb[u] <= best.b;
            const uint64_t lm = __ballot(left), rm = __ballot(in && !left);
            const uint64_t m = left ? lm : rm;
            const uint32_t before = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const uint32_t at = left ? runl + before : len - 1u - runr - before;
            if (in) {
                rout[at] = r[u];
                if constexpr (REG) wout[at] = t[u];
            }
            runl += (uint32_t)__popcll(lm);
            runr += (uint32_t)__popcll(rm);
        }
    };
    if (len != 0 && len <= 128u)
        block(0u, std::integral_constant<int, 2>{});
    else
        for (uint32_t blk = 0; blk < len; blk += 512u)
            block(blk, std::integral_constant<int, 8>{});
    return runl;
}

// Regression form of the split choice and partition: the node's best
// candidate (exact total order), a split when its gap is nonzero, the rows
// partitioned as for classification when the children are searched next.
__device__ void finalize_reg(const ForestDev& F, JobDev& J, const TreeDev& tr, uint32_t slot,
                             const SlotRec& sr, const NodeDev& nd, Cand c) {
    const int lane = threadIdx.x & 63;
    if (F.split_rank) {
        // FP64 ranking: only the candidates within the margin of the wave's
        // maximum take part in the exact comparison
        const double q = c.nl != 0 ? reg_q64(c) : -1.0;
        double qmax = q;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const double o = __shfl_xor(qmax, m);
            qmax = o > qmax ? o : qmax;
        }
        if (c.nl != 0 && q < fp64_floor(qmax)) c.nl = 0;
        const unsigned long long fin = __ballot(c.nl != 0);
        if (__popcll(fin) == 1) {
            c = shfl_cand(c, (int)__ffsll(fin) - 1);
        } else {
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const Cand o = shfl_xor_cand(c, m);
                if (reg_wins_total(o, c)) c = o;
            }
        }
    } else {
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const Cand o = shfl_xor_cand(c, m);
            if (reg_wins_total(o, c)) c = o;
        }
    }
    const Cand best = c;
    const uint32_t child = F.next_base + 2u * (F.n_small_cur + slot);
    if (best.nl == 0 || reg_gap(best) == 0) {  // no decrease: stays the leaf it was created as
        if (lane == 0) {
            mark_unused_pair(F, child);
            F.kinds[F.n_small_cur + slot] = 0;
        }
        return;
    }
    const bool part = (int)nd.depth + 1 < J.D;
    const uint32_t runl = partition_rows<true>(F, J, tr, nd, sr.recs, sr.wy, best, ldg(J.colptr + best.f), part ? sr.len : 0u);
    if (lane == 0) {
        int kinds[2];
        split_node_reg(F, J, tr, sr.id, nd, best, runl, reg_gain_fix(best, J.s_gain), child,
                       kinds);
        F.kinds[F.n_small_cur + slot] = (uint8_t)(kinds[0] | kinds[1] << 2);
    }
}

// Large nodes, phase 2: one wavefront per node (four per workgroup, no
// barriers).  The node's split is the best of its histogram items' candidates
// (exact score, then draw position, then threshold); a strictly positive
// decrease splits the node and its rows are partitioned in one pass: left
// rows from the front in row order, right rows from the back in reverse row
// order.  No result depends on the order of a node's rows, and each child
// segment stays monotone in row index for the next level's gathers.
// Phase 2 for the regression nodes of a level (k_split_finalize skips them,
// so that the 256-bit arithmetic stays out of the classification kernel).
__global__ __launch_bounds__(256) void k_split_finalize_reg(ForestDev F0, int level,
                                                            uint32_t first, uint32_t count) {
    const ForestDev F = level_view(F0, level);
    if (count == 0xFFFFFFFFu) {
        first = 0;
        count = level_slots(F0, level);
    }
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    for (uint32_t k = blockIdx.x * 4u + (uint32_t)wave; k < count; k += gridDim.x * 4u) {
        const uint32_t slot = first + k;
        const SlotRec& sr = F.srec[slot];
        if (!sr.reg) continue;  // a classification node: k_split_finalize
        const NodeDev nd = F.nodes[sr.id];
        const TreeDev tr = F.trees[nd.tree];
        JobDev& J = F.jobs[tr.job];
        // rank the items' candidates: each lane keeps the best of its items
        const int ni = ((int)sr.mtry + F.fw - 1) / F.fw;
        Cand c;
        c.nl = 0;
        c.q = 0x7FFFFFFF;
        c.b = 0x7FFFFFFF;
        c.f = 0;
        c.nr = 0;
        c.pad = 0;
        c.sl = c.sr = 0;
        for (int t = lane; t < ni; t += 64) {
            const Cand d = F.cand[(size_t)slot * F.npi + t];
            if (d.nl != 0 && (c.nl == 0 || reg_wins_total(d, c))) c = d;
        }
        finalize_reg(F, J, tr, slot, sr, nd, c);
    }
}

template <int KMAX, bool BIG>
__global__ __launch_bounds__(256) void k_split_finalize(ForestDev F0, int level, uint32_t first,
                                                        uint32_t count) {
    const ForestDev F = level_view(F0, level);
    if (count == 0xFFFFFFFFu) {
        first = 0;
        count = level_slots(F0, level);
    }
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    for (uint32_t k = blockIdx.x * 4u + (uint32_t)wave; k < count; k += gridDim.x * 4u) {
        const uint32_t slot = first + k;
        const SlotRec& sr = F.srec[slot];
        if (sr.reg) continue;  // a regression node: k_split_finalize_reg
        const uint32_t id = sr.id;
        const NodeDev nd = F.nodes[id];
        const TreeDev tr = F.trees[nd.tree];
        JobDev& J = F.jobs[tr.job];
        uint32_t cnode[KMAX];
        uint64_t S = 0;
#pragma unroll
        for (int c = 0; c < KMAX; ++c) {
            cnode[c] = sr.cnode[c];
            S += (uint64_t)cnode[c] * cnode[c];
        }
        const uint32_t N = sr.n;
        // The items' records, lanes over items: with FP32 ranking those within
        // the margin of the maximum, else all, are compared exactly in draw
        // order, a strictly better one replacing (so ties keep the earlier
        // draw); one finalist alone is taken as it is.
        const int ni = ((int)sr.mtry + F.fw - 1) / F.fw;
        constexpr int IW = item_counts<KMAX, BIG>() + 2;
        const uint32_t fb = count_bits(KMAX, N);
        const uint32_t* items = F.icand + (size_t)slot * F.npi * IW;
        float fl = 0.0f;
        if (F.split_rank) {
            float q1 = -1.0f;
            for (int t = lane; t < ni; t += 64)
                q1 = fmaxf(q1, __uint_as_float(items[(size_t)t * IW]));
            const float qmax = wave_max_f_dpp(q1);
            fl = qmax < 0.0f ? 2.0f * (float)N : fp32_floor(qmax);  // Q <= N
        }
        Cand best;
        best.nl = 0;
        int bt = -1;
        for (int t0 = 0; t0 < ni; t0 += 64) {
            const float q =
                t0 + lane < ni ? __uint_as_float(items[(size_t)(t0 + lane) * IW]) : -1.0f;
            for (uint64_t m = __ballot(q >= fl); m; m &= m - 1) {
                const int t = t0 + (int)__ffsll((unsigned long long)m) - 1;
                const uint32_t* rec = items + (size_t)t * IW;
                const Cand d = cand_of<KMAX, BIG>(rec + 2, fb, (int)(rec[1] & 0xFFu), cnode, N);
                if (best.nl == 0 || cand_better(d, best)) {
                    best = d;
                    bt = t;
                }
            }
        }
        const uint32_t child = F.next_base + 2u * (F.n_small_cur + slot);
        const bool split = bt >= 0 && cand_positive(best, S, N);
        if (!split) {  // stays the leaf it was created as
            if (lane == 0) {
                mark_unused_pair(F, child);
                F.kinds[F.n_small_cur + slot] = 0;
            }
            continue;
        }
        const uint32_t* rec = items + (size_t)bt * IW;
        best.q = bt * F.fw + (int)(rec[1] >> 8);
        best.f = (int)F.feat[(size_t)slot * F.mtry_cap + best.q];
        uint32_t cl[16], cr[16];
        int nzl = 0, nzr = 0;
#pragma unroll
        for (int c2 = 0; c2 < 16; ++c2) {
            cl[c2] = c2 < KMAX ? left_count<KMAX, BIG>(rec + 2, fb, c2 % KMAX) : 0u;
            cr[c2] = (c2 < KMAX ? cnode[c2] : 0u) - cl[c2];
            nzl += cl[c2] != 0;
            nzr += cr[c2] != 0;
        }
        // Rows are partitioned only for a child that is searched next: below
        // the maximum depth with two or more classes (which implies two or
        // more distinct rows); other children are final leaves.
        const bool part = (int)nd.depth + 1 < J.D && (nzl >= 2 || nzr >= 2);
        const uint32_t runl = partition_rows<false>(F, J, tr, nd, sr.recs, nullptr, best, ldg(J.colptr + best.f), part ? sr.len : 0u);
        if (lane == 0) {
            int kinds[2];
            split_node(F, J, tr, id, nd, best, runl, cl, cr, cand_gain_fix(best, S, N), child,
                       kinds);
            F.kinds[F.n_small_cur + slot] = (uint8_t)(kinds[0] | kinds[1] << 2);
        }
    }
}

// ---------------------------------------------------------------------------
// Whole trees in one launch: one workgroup per tree grows all its levels, with
// workgroup barriers in place of the level kernels' launches.  For jobs of few
// rows, whose level kernels are launch and dependent-load latency (a 500 x 20
// forest of 50 trees of depth 8: 56 launches an iteration, each 3-15 us; 20
// iterations 7.4 ms, 3.7 with this kernel; the engine's rule says where).  The
// level's node lists live in LDS; a wave takes a small node as k_split_small
// does, and a group of g waves a large one: each wave counts and scans its
// share of the drawn features (draw = lane * g + its place in the group), the
// group's first wave picks the best and partitions.  g falls from all waves to
// one as a level's large nodes become as many as the waves.  Trees, child pairs
// and results are those of the level kernels (child pairs are handed out per
// tree and level instead of per level).
struct GrowLds {
    uint32_t cnt[2][2];      // [level parity] small, large nodes of the level
    uint32_t base;           // first child pair of the level
    uint32_t best[16][12];   // a wave's best: score, bin, draw, left counts
};

// Children of a searched node into the next level's lists (one lane).
__device__ __forceinline__ void grow_push(GrowLds& G, uint32_t* next, uint32_t cap, int parity,
                                          const int* kinds, uint32_t child) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        if (kinds[c] == kSmall) next[atomicAdd(&G.cnt[parity][0], 1u)] = child + c;
        if (kinds[c] == kLarge) next[cap - 1u - atomicAdd(&G.cnt[parity][1], 1u)] = child + c;
    }
}

template <int KMAX>
__device__ __forceinline__ void grow_large(const ForestDev& F, JobDev& J, const TreeDev& tr,
                                           GrowLds& G, const uint32_t* list, uint32_t cap,
                                           uint32_t ns, uint32_t nl, uint32_t* next, int nparity,
                                           uint32_t* lds, uint32_t* hist, uint32_t wave,
                                           uint32_t nw) {
    constexpr int C = item_counts<KMAX, false>(), PW = pk_words(KMAX);
    const int lane = threadIdx.x & 63;
    uint16_t* tab = reinterpret_cast<uint16_t*>(lds);
    const int B = J.B, mtry = J.mtry;
    const uint32_t K = (uint32_t)J.K;
    uint32_t g = nw;
    while (g > 1u && (nl * g > nw || g > (uint32_t)mtry)) g >>= 1;
    const uint32_t npr = nw / g, sub = wave % g;
    for (uint32_t i0 = 0; i0 < nl; i0 += npr) {
        const uint32_t i = i0 + wave / g;
        const bool on = i < nl;  // uniform over the wave
        const uint32_t id = uniform(on ? list[cap - 1u - i] : 0u);
        const NodeDev nd = F.nodes[on ? id : 0u];
        const uint32_t N = nd.n, len = uniform(nd.len);
        const uint32_t* recs = J.rec[F.parity] + (size_t)tr.tau * J.rstride + nd.seg;
        const CountForm cf = count_form<KMAX>(N, K);
        uint32_t cnode[KMAX], pk[PW];
        ItemBest best;
        best.q = -1.0f;
        best.b = 0;
        uint32_t draw = 0, bl[C];
#pragma unroll
        for (int c = 0; c < C; ++c) bl[c] = 0;
        if (on) {
#pragma unroll
            for (int c = 0; c < KMAX; ++c)
                cnode[c] = (uint32_t)c < K ? F.cls[(size_t)id * F.kmax + c] : 0u;
#pragma unroll
            for (int w = 0; w < PW; ++w) {
                uint32_t v8 = 0, v16 = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (4 * w + k < KMAX) v8 |= cnode[4 * w + k < KMAX ? 4 * w + k : 0] << (8 * k);
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (2 * w + k < KMAX) v16 |= cnode[2 * w + k < KMAX ? 2 * w + k : 0] << (16 * k);
                pk[w] = cf.fb == 8u ? v8 : v16;
            }
            const KeyedPerm P = make_perm(J.seed_lo, J.seed_hi, kMtry, (uint32_t)J.t,
                                          (uint32_t)tr.tau, nd.heap, 0u, (uint64_t)J.p_w);
            const bool use_tab = (P.rounds << P.half) <= kDrawTab;
            if (use_tab) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // earlier lookups
                for (uint32_t e = (uint32_t)lane; e < (P.rounds << P.half); e += 64u)
                    tab[e] = (uint16_t)perm_round(P, e >> P.half, e & P.mask);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            }
            for (uint32_t q0 = sub; q0 < (uint32_t)mtry; q0 += 64u * g) {
                const uint32_t q = q0 + (uint32_t)lane * g;
                const bool mine = q < (uint32_t)mtry;
                const uint32_t f = use_tab ? perm_apply_tab(P, tab, mine ? q : 0u)
                                           : perm_apply(P, mine ? q : 0u);
                const uint32_t off =
                    (uint32_t)((uint64_t)(ldg(J.colptr + f) - J.colbase) >> 8);
                const uint32_t n_here = min(64u, ((uint32_t)mtry - q0 + g - 1u) / g);
                for (uint32_t t = 0; t < n_here; ++t) {
                    const uint8_t* col =
                        J.colbase + (uint64_t)readlane_w(off, (int)t) * 256u;
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // earlier reads
#pragma unroll
                    for (int w = 0; w < C; ++w)
                        if ((uint32_t)w < cf.words)
                            reinterpret_cast<uint4*>(hist)[w * 64 + lane] =
                                make_uint4(0u, 0u, 0u, 0u);
                    int b0 = 0, b1 = 0;
                    auto batch = [&](uint32_t r0, auto nb) {
                        constexpr int NB = decltype(nb)::value;
                        uint32_t r[NB], b[NB];
#pragma unroll
                        for (int u = 0; u < NB; ++u) r[u] = rec_raw(recs, r0 + u * 64 + lane, len);
#pragma unroll
                        for (int u = 0; u < NB; ++u) b[u] = ldg(col + rec_row(r[u]));
#pragma unroll
                        for (int u = 0; u < NB; ++u)
                            if (r0 + u * 64 + lane < len) count_row<KMAX>(hist, cf, r[u], b[u]);
                        b0 = (int)b[0];
                        b1 = (int)b[1];
                    };
                    if (len <= 128u)
                        batch(0u, std::integral_constant<int, 2>{});
                    else
                        for (uint32_t r0 = 0; r0 < len; r0 += 512u)
                            batch(r0, std::integral_constant<int, 8>{});
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    uint32_t l[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) l[c] = 0;
                    const ItemBest r = scan_item<KMAX, false>(hist, cf, K, len, b0, b1, B, pk,
                                                              cnode, N, F.split_rank, l);
                    // draws in order: a strictly better score replaces
                    bool better = r.q >= 0.0f;
                    if (better && best.q >= 0.0f) {
                        if (F.split_rank &&
                            (r.q < fp32_floor(best.q) || best.q < fp32_floor(r.q)))
                            better = r.q > best.q;
                        else
                            better = cand_better(cand_of<KMAX, false>(l, cf.fb, r.b, cnode, N),
                                                 cand_of<KMAX, false>(bl, cf.fb, best.b, cnode, N));
                    }
                    if (better) {
                        best = r;
                        draw = q0 + t * g;
#pragma unroll
                        for (int c = 0; c < C; ++c) bl[c] = l[c];
                    }
                }
            }
        }
        if (g > 1u) {  // the same for every wave of the workgroup
            if (lane == 0) {
                G.best[wave][0] = __float_as_uint(best.q);
                G.best[wave][1] = (uint32_t)best.b;
                G.best[wave][2] = draw;
#pragma unroll
                for (int c = 0; c < C; ++c) G.best[wave][3 + c] = bl[c];
            }
            __syncthreads();
            if (on && sub == 0u) {
                for (uint32_t o = 1; o < g; ++o) {
                    const uint32_t* e = G.best[wave + o];
                    ItemBest r;
                    r.q = __uint_as_float(uniform(e[0]));
                    r.b = (int)uniform(e[1]);
                    const uint32_t rd = uniform(e[2]);
                    if (r.q < 0.0f) continue;
                    uint32_t l[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) l[c] = uniform(e[3 + c]);
                    bool better = best.q < 0.0f;
                    if (!better) {
                        if (F.split_rank &&
                            (r.q < fp32_floor(best.q) || best.q < fp32_floor(r.q))) {
                            better = r.q > best.q;
                        } else {  // exact; ties to the earlier draw
                            const Cand x = cand_of<KMAX, false>(l, cf.fb, r.b, cnode, N);
                            const Cand y = cand_of<KMAX, false>(bl, cf.fb, best.b, cnode, N);
                            better = cand_better(x, y) || (rd < draw && !cand_better(y, x));
                        }
                    }
                    if (better) {
                        best = r;
                        draw = rd;
#pragma unroll
                        for (int c = 0; c < C; ++c) bl[c] = l[c];
                    }
                }
            }
        }
        if (on && sub == 0u) {
            const uint32_t child = F.next_base + 2u * (ns + i);
            Cand c;
            c.nl = 0;
            uint64_t S = 0;
#pragma unroll
            for (int k = 0; k < KMAX; ++k) S += (uint64_t)cnode[k] * cnode[k];
            if (best.q >= 0.0f) c = cand_of<KMAX, false>(bl, cf.fb, best.b, cnode, N);
            if (c.nl == 0 || !cand_positive(c, S, N)) {  // stays the leaf it was created as
                if (lane == 0) mark_unused_pair(F, child);
            } else {
                const KeyedPerm P = make_perm(J.seed_lo, J.seed_hi, kMtry, (uint32_t)J.t,
                                              (uint32_t)tr.tau, nd.heap, 0u, (uint64_t)J.p_w);
                c.q = (int)draw;
                c.f = (int)((P.rounds << P.half) <= kDrawTab ? perm_apply_tab(P, tab, draw)
                                                             : perm_apply(P, draw));
                uint32_t cl[16], cr[16];
                int nzl = 0, nzr = 0;
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    cl[k] = k < KMAX ? left_count<KMAX, false>(bl, cf.fb, k % KMAX) : 0u;
                    cr[k] = (k < KMAX ? cnode[k % KMAX] : 0u) - cl[k];
                    nzl += cl[k] != 0;
                    nzr += cr[k] != 0;
                }
                const bool part = (int)nd.depth + 1 < J.D && (nzl >= 2 || nzr >= 2);
                const uint32_t runl = partition_rows<false>(F, J, tr, nd, recs, nullptr, c,
                                                            ldg(J.colptr + c.f), part ? len : 0u);
                if (lane == 0) {
                    int kinds[2];
                    split_node(F, J, tr, id, nd, c, runl, cl, cr, cand_gain_fix(c, S, N), child,
                               kinds);
                    grow_push(G, next, cap, nparity, kinds, child);
                }
            }
        }
        if (g > 1u) __syncthreads();  // the waves' bests are rewritten
    }
}

template <int KMAX>
__global__ __launch_bounds__(1024) void k_grow(ForestDev F0, uint32_t cap) {
    constexpr int WORDS = KMAX <= 4 ? 1 : (KMAX <= 8 ? 2 : 4);
    // [waves][small_lds_words(F.small_head, WORDS)], then [2][cap] node lists: small nodes
    // from the front, large ones from the back
    extern __shared__ uint4 lds_raw[];
    __shared__ GrowLds G;
    static_assert(sizeof(GrowLds) <= kGrowStaticLds, "k_grow's share of the LDS");
    const uint32_t g = blockIdx.x;
    const TreeDev tr = F0.trees[g];
    JobDev& J = F0.jobs[tr.job];
    if (!J.live) return;  // the whole workgroup
    const int lane = threadIdx.x & 63;
    const uint32_t wave = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const uint32_t region = small_lds_words(F0.small_head, WORDS);
    uint32_t* lds = reinterpret_cast<uint32_t*>(lds_raw) + wave * region;
    uint32_t* hist = lds + F0.small_head + WORDS * 64;
    uint32_t* lists = reinterpret_cast<uint32_t*>(lds_raw) + nw * region;
    if (threadIdx.x == 0) {
        const int kind = F0.kinds[g];
        G.cnt[0][0] = kind == kSmall;
        G.cnt[0][1] = kind == kLarge;
        lists[kind == kLarge ? cap - 1u : 0u] = g;
    }
    __syncthreads();
    ForestDev F = F0;
    for (int d = 0; d < J.D; ++d) {
        const int p = d & 1;
        const uint32_t ns = G.cnt[p][0], nl = G.cnt[p][1];
        if (ns + nl == 0u) break;
        if (threadIdx.x == 0) {
            G.base = F.n_roots + 2u * atomicAdd(&F.ctrs[0].pairs, ns + nl);
            G.cnt[p ^ 1][0] = G.cnt[p ^ 1][1] = 0;
            if (d > 0) {  // the roots were counted when they were made
                if (ns) atomicAdd(&F.ctrs[d].n_small, ns);
                if (nl) atomicAdd(&F.ctrs[d].n_slots, nl);
            }
        }
        __syncthreads();
        const uint32_t* cur = lists + (size_t)p * cap;
        uint32_t* next = lists + (size_t)(p ^ 1) * cap;
        F.parity = p;
        F.ctr = F.ctrs + d + 1;
        F.next_base = G.base;
        if (nl)
            grow_large<KMAX>(F, J, tr, G, cur, cap, ns, nl, next, p ^ 1, lds, hist, wave, nw);
        for (uint32_t i = wave; i < ns; i += nw) {
            SmallOut o;
            o.kinds[0] = o.kinds[1] = kLeaf;
            o.child = F.next_base + 2u * i;
            o.alg = 0;
            const uint32_t id = uniform(cur[i]);
            const NodeDev nd = F.nodes[id];
            small_node_of<WORDS, false>(F, id, nd, tr, J, o, lds);
            if (lane == 0) grow_push(G, next, cap, p ^ 1, o.kinds, o.child);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Next-level lists, without atomics: searched node i of level d (the small
// nodes first, then the large-node slots) owns the child pair at
// next_base + 2i, and its children's kinds were recorded in kinds[i].  Two
// passes over chunks of kListChunk nodes: count the wave-path and the
// histogram-path children per chunk, then let every chunk add up the counts
// of the chunks before it and write its children to the lists in node order.
constexpr uint32_t kListChunk = 4096;  // 1024 threads x 4 nodes

__device__ __forceinline__ uint32_t level_searched(const ForestDev& F, int level) {
    return level_small(F, level) + level_slots(F, level);
}

// Packed (wave path | histogram path << 16) children of 4 nodes from i0.
__device__ __forceinline__ uint32_t kinds4(const ForestDev& F, uint32_t i0, uint32_t n,
                                           uint32_t* kd) {
    uint32_t c = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        kd[u] = i0 + u < n ? F.kinds[i0 + u] : 0u;
        const uint32_t a = kd[u] & 3u, b = kd[u] >> 2;
        c += (a == (uint32_t)kSmall) + (b == (uint32_t)kSmall) +
             (((a == (uint32_t)kLarge) + (b == (uint32_t)kLarge)) << 16);
    }
    return c;
}

// Sum over the workgroup of 1024 threads (16 waves); all threads get it.
__device__ __forceinline__ unsigned long long block_sum64(unsigned long long v,
                                                          unsigned long long* s_w) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
    if (lane == 0) s_w[wave] = v;
    __syncthreads();
    unsigned long long t = 0;
    for (int w = 0; w < 16; ++w) t += s_w[w];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(1024) void k_lists_count(ForestDev F, int level) {
    __shared__ unsigned long long s_w[16];
    const uint32_t n = level_searched(F, level);
    const uint32_t nchunks = (n + kListChunk - 1) / kListChunk;
    for (uint32_t b = blockIdx.x; b < nchunks; b += gridDim.x) {
        uint32_t kd[4];
        const uint32_t c = kinds4(F, b * kListChunk + threadIdx.x * 4u, n, kd);
        const unsigned long long t =
            block_sum64((unsigned long long)(c & 0xFFFFu) | ((unsigned long long)(c >> 16) << 32),
                        s_w);
        if (threadIdx.x == 0) F.chunk_sums[b] = t;
    }
}

__global__ __launch_bounds__(1024) void k_lists_write(ForestDev F0, int level) {
    __shared__ unsigned long long s_w[16];
    __shared__ uint32_t s_wc[16];
    const ForestDev F = level_view(F0, level);  // appends describe level + 1
    const uint32_t n = level_searched(F0, level);
    const uint32_t nchunks = (n + kListChunk - 1) / kListChunk;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t b = blockIdx.x; b < nchunks; b += gridDim.x) {
        // children of the chunks before this one
        unsigned long long pre = 0;
        for (uint32_t e = threadIdx.x; e < b; e += 1024) pre += F.chunk_sums[e];
        pre = block_sum64(pre, s_w);
        uint32_t kd[4];
        const uint32_t i0 = b * kListChunk + threadIdx.x * 4u;
        const uint32_t c = kinds4(F0, i0, n, kd);
        const uint32_t incl = wave_incl_sum(c);  // per field < 2^16: 4096 nodes, 2 children
        if (lane == 63) s_wc[wave] = incl;
        __syncthreads();
        uint32_t off = incl - c;
        for (int w = 0; w < wave; ++w) off += s_wc[w];
        uint32_t ps = (uint32_t)pre + (off & 0xFFFFu), pl = (uint32_t)(pre >> 32) + (off >> 16);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int ch = 0; ch < 2; ++ch) {
                const uint32_t k = (kd[u] >> (2 * ch)) & 3u;
                const uint32_t node = F.next_base + 2u * (i0 + u) + ch;
                if (k == (uint32_t)kSmall) {
                    if (ps < F.small_cap)
                        F.small_out[ps] = node;
                    else
                        atomicOr(&F.ctr->overflow, 1u);
                    ++ps;
                } else if (k == (uint32_t)kLarge) {
                    if (pl < F.slot_cap)
                        F.slot_node_out[pl] = node;
                    else
                        atomicOr(&F.ctr->overflow, 2u);
                    ++pl;
                }
            }
        }
        if (b == nchunks - 1 && threadIdx.x == 1023) {  // the last node's totals
            F.ctr->n_small = min(ps, F.small_cap);
            F.ctr->n_slots = min(pl, F.slot_cap);
        }
        __syncthreads();  // shared sums are reused by the next chunk
    }
}

// ---------------------------------------------------------------------------
// Host launchers.
void launch_boot_compact(const ForestDev& F, uint32_t n_trees, hipStream_t st) {
    hipLaunchKernelGGL(k_boot_compact, dim3(n_trees), dim3(1024), 0, st, F);
}

// count == 0xFFFFFFFF: the whole level, sized on the device (grid-stride).
void launch_split_small(const ForestDev& F, int level, uint32_t first, uint32_t count,
                        uint32_t grid_wg, hipStream_t st) {
    if (!count) return;
    const dim3 grid(grid_wg);
    if (F.has_reg)
        hipLaunchKernelGGL(k_split_small_reg, grid, dim3(256),
                           (size_t)4 * small_reg_words(F.small_head) * sizeof(uint32_t), st, F, level, first,
                           count);
    if (!F.has_cls) return;
    const int words = F.kmax <= 4 ? 1 : (F.kmax <= 8 ? 2 : 4);
    const size_t lds = (size_t)4 * small_lds_words(F.small_head, words) * sizeof(uint32_t);
#define BORUTA_SMALL(W)                                                                         \
    if (F.rowmaj)                                                                               \
        hipLaunchKernelGGL((k_split_small<W, true>), grid, dim3(256), lds, st, F, level, first, \
                           count);                                                              \
    else                                                                                        \
        hipLaunchKernelGGL((k_split_small<W, false>), grid, dim3(256), lds, st, F, level,       \
                           first, count);
    switch (words) {
        case 1: BORUTA_SMALL(1) break;
        case 2: BORUTA_SMALL(2) break;
        default: BORUTA_SMALL(4) break;
    }
#undef BORUTA_SMALL
}

void launch_lists(const ForestDev& F, int level, uint32_t grid_wg, hipStream_t st) {
    hipLaunchKernelGGL(k_lists_count, dim3(grid_wg), dim3(1024), 0, st, F, level);
    hipLaunchKernelGGL(k_lists_write, dim3(grid_wg), dim3(1024), 0, st, F, level);
}

void launch_draws(const ForestDev& F, int level, uint32_t grid_wg, hipStream_t st) {
    const size_t lds = (size_t)(256u / F.draw_seg) * F.draw_tab * sizeof(uint16_t);
    hipLaunchKernelGGL(k_draws, dim3(grid_wg), dim3(256), lds, st, F, level);
}

template <int KMAX, int FW>
static void launch_tile_rb(const ForestDev& F, int level, uint32_t first, uint32_t count,
                           dim3 grid, size_t lds, int rb, hipStream_t st) {
    // plans that may hold nodes of weight 65536 and more: one class per word
    const bool big = F.hist_words == F.kmax;
#define BORUTA_TILE(RB)                                                                          \
    if (big)                                                                                     \
        hipLaunchKernelGGL((k_hist_tile<KMAX, FW, RB, true>), grid, dim3(256), lds, st, F, level, \
                           first, count);                                                        \
    else                                                                                         \
        hipLaunchKernelGGL((k_hist_tile<KMAX, FW, RB, false>), grid, dim3(256), lds, st, F,      \
                           level, first, count);
    switch (rb) {
        case 4: BORUTA_TILE(4) break;
        case 16: BORUTA_TILE(16) break;
        default: BORUTA_TILE(8) break;
    }
#undef BORUTA_TILE
}

// rb: rows per lane per batch (4, 8 or 16); F.fw draws per item with
// F.fw * F.kmax <= 8 (the engine validates both).  Regression items run in
// k_hist_reg, classification items in k_hist_tile: two launches over the
// same items for a plan holding both kinds of job.
void launch_hist_tile(const ForestDev& F, int level, uint32_t first, uint32_t count,
                      uint32_t grid_wg, int rb, hipStream_t st) {
    if (!count) return;
    // four waves of fw histograms of hist_words words per bin
    const size_t lds = (size_t)4 * F.fw * F.hist_words * 256 * sizeof(uint32_t);
    const dim3 grid(grid_wg);
    if (F.has_reg) {
        const size_t rl = std::max(lds, (size_t)4 * 768 * sizeof(uint32_t));
#define BORUTA_REG(RB)                                                                          \
    if (F.wide_reg)                                                                             \
        hipLaunchKernelGGL((k_hist_reg<RB, true>), grid, dim3(256), rl, st, F, level, first,    \
                           count);                                                              \
    else                                                                                        \
        hipLaunchKernelGGL((k_hist_reg<RB, false>), grid, dim3(256), rl, st, F, level, first,   \
                           count);
        switch (rb) {
            case 4: BORUTA_REG(4) break;
            case 16: BORUTA_REG(16) break;
            default: BORUTA_REG(8) break;
        }
#undef BORUTA_REG
    }
    if (!F.has_cls) return;
    switch (F.kmax * 8 + F.fw) {
        case 2 * 8 + 4: launch_tile_rb<2, 4>(F, level, first, count, grid, lds, rb, st); break;
        case 2 * 8 + 2: launch_tile_rb<2, 2>(F, level, first, count, grid, lds, rb, st); break;
        case 2 * 8 + 1: launch_tile_rb<2, 1>(F, level, first, count, grid, lds, rb, st); break;
        case 3 * 8 + 2: launch_tile_rb<3, 2>(F, level, first, count, grid, lds, rb, st); break;
        case 3 * 8 + 1: launch_tile_rb<3, 1>(F, level, first, count, grid, lds, rb, st); break;
        case 4 * 8 + 2: launch_tile_rb<4, 2>(F, level, first, count, grid, lds, rb, st); break;
        case 4 * 8 + 1: launch_tile_rb<4, 1>(F, level, first, count, grid, lds, rb, st); break;
        case 8 * 8 + 1: launch_tile_rb<8, 1>(F, level, first, count, grid, lds, rb, st); break;
        default: launch_tile_rb<16, 1>(F, level, first, count, grid, lds, rb, st); break;
    }
}

size_t hist_col_lds(int kmax, int waves, uint32_t gq_max) {
    return (size_t)waves * pk_words(kmax) * 256 * sizeof(uint32_t) + (size_t)gq_max * 16;
}

// F.col_count == 2: the places are counted by k_col_count (n_gcol <= kColCountLds)
void launch_col_sort(const ForestDev& F, int level, uint32_t grid_wg, hipStream_t st) {
    if (F.col_count == 2)
        hipLaunchKernelGGL(k_col_count, dim3(kColCountGrid), dim3(256),
                           (size_t)F.n_gcol * sizeof(uint32_t), st, F, level);
    hipLaunchKernelGGL(k_col_scan, dim3(1), dim3(256), 0, st, F, level);
    hipLaunchKernelGGL(k_col_scatter, dim3(grid_wg), dim3(256), 0, st, F, level);
}

// k_grow: dynamic LDS of a workgroup of `waves`, and its launch (after
// prepare_grow allowed that LDS).
size_t grow_lds(int kmax, uint32_t head, int waves, uint32_t cap) {
    const int words = kmax <= 4 ? 1 : (kmax <= 8 ? 2 : 4);
    return ((size_t)waves * small_lds_words(head, words) + 2 * (size_t)cap) * sizeof(uint32_t);
}

static const void* grow_fn(int kmax) {
    switch (kmax) {
        case 2: return reinterpret_cast<const void*>(&k_grow<2>);
        case 3: return reinterpret_cast<const void*>(&k_grow<3>);
        case 4: return reinterpret_cast<const void*>(&k_grow<4>);
        case 8: return reinterpret_cast<const void*>(&k_grow<8>);
        default: return reinterpret_cast<const void*>(&k_grow<16>);
    }
}

hipError_t prepare_grow(int kmax) {
    return hipFuncSetAttribute(grow_fn(kmax), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(kLdsPerWorkgroup - kGrowStaticLds));
}

void launch_grow(const ForestDev& F, uint32_t n_trees, int waves, uint32_t cap, hipStream_t st) {
    ForestDev f = F;
    void* args[] = {&f, &cap};
    // a refused launch is reported by the caller's hipGetLastError
    (void)hipLaunchKernel(grow_fn(F.kmax), dim3(n_trees), dim3(64 * waves), args,
                          grow_lds(F.kmax, F.small_head, waves, cap), st);
}

// Allows the column path's dynamic LDS (above the default per-launch limit)
// for the instantiation of kmax classes.
static const void* hist_col_fn(int kmax) {
    switch (kmax) {
        case 2: return reinterpret_cast<const void*>(&k_hist_col<2>);
        case 3: return reinterpret_cast<const void*>(&k_hist_col<3>);
        case 4: return reinterpret_cast<const void*>(&k_hist_col<4>);
        case 8: return reinterpret_cast<const void*>(&k_hist_col<8>);
        default: return reinterpret_cast<const void*>(&k_hist_col<16>);
    }
}

hipError_t prepare_hist_col(int kmax) {
    return hipFuncSetAttribute(hist_col_fn(kmax), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kLdsPerWorkgroup);
}

void launch_hist_col(const ForestDev& F, int level, uint32_t grid_wg, int waves, uint32_t gq_max,
                     hipStream_t st) {
    const size_t lds = hist_col_lds(F.kmax, waves, gq_max);
    ForestDev f = F;
    void* args[] = {&f, &level, &gq_max};
    // a refused launch is reported by the caller's hipGetLastError
    (void)hipLaunchKernel(hist_col_fn(F.kmax), dim3(grid_wg), dim3(64 * waves), args, lds, st);
    // the level's nodes past its 16-bit counts (plans of 65536 rows and more)
    if (F.big_cap) {
        const uint32_t need = std::max(1u, std::min(F.big_cap * (uint32_t)F.npi / 4u, 2048u));
        launch_hist_tile(F, level, 0, kBigItems, need, 8, st);
    }
}

void launch_split_finalize(const ForestDev& F, int level, uint32_t first, uint32_t count,
                           uint32_t grid_wg, hipStream_t st) {
    if (!count) return;
    const dim3 grid(grid_wg);
    if (F.has_reg)
        hipLaunchKernelGGL(k_split_finalize_reg, grid, dim3(256), 0, st, F, level, first, count);
    if (!F.has_cls) return;
#define BORUTA_FINALIZE(K)                                                                       \
    if (F.hist_words == F.kmax)                                                                  \
        hipLaunchKernelGGL((k_split_finalize<K, true>), grid, dim3(256), 0, st, F, level, first, \
                           count);                                                               \
    else                                                                                         \
        hipLaunchKernelGGL((k_split_finalize<K, false>), grid, dim3(256), 0, st, F, level,       \
                           first, count);
    switch (F.kmax) {
        case 2: BORUTA_FINALIZE(2) break;
        case 3: BORUTA_FINALIZE(3) break;
        case 4: BORUTA_FINALIZE(4) break;
        case 8: BORUTA_FINALIZE(8) break;
        default: BORUTA_FINALIZE(16) break;
    }
#undef BORUTA_FINALIZE
}

}  // namespace boruta
