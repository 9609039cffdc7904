"""The choice among a feature's thresholds (pick_threshold of forest_dev.hpp) on
the CPU: its source is compiled with g++, a thread for each of the wave's 64
lanes, and compared with a loop over all candidates in exact integers.  Whatever
the candidates -- none valid among them: a node whose rows share one bin, or are
all past the last threshold -- the bin that it returns has to be a bin, as its
callers read the histogram there."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2605_09950_amd", "csrc", "forest_dev.hpp")

WAVE = r"""
#include <barrier>
#include <bit>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>
#define __device__
#define __host__
#define __forceinline__ inline
#define ext_vector_type(n) vector_size(2 * n)
using u128 = unsigned __int128;
using std::max;
static std::barrier g_sync(64);
static uint64_t g_lane_value[64];
static thread_local int g_lane;
// every lane's value, and lane `src` of it
template <class T> T lane_of(T v, int src) {
    static_assert(sizeof(T) <= 8);
    uint64_t w = 0;
    __builtin_memcpy(&w, &v, sizeof(T));
    g_lane_value[g_lane] = w;
    g_sync.arrive_and_wait();
    T o;
    __builtin_memcpy(&o, &g_lane_value[src & 63], sizeof(T));
    g_sync.arrive_and_wait();
    return o;
}
template <class T> T __shfl_xor(T v, int m) { return lane_of(v, g_lane ^ m); }
inline uint64_t __ballot(bool p) {
    g_lane_value[g_lane] = p;
    g_sync.arrive_and_wait();
    uint64_t r = 0;
    for (int l = 0; l < 64; ++l) r |= g_lane_value[l] << l;
    g_sync.arrive_and_wait();
    return r;
}
inline int __builtin_amdgcn_readlane(int v, int l) { return lane_of(v, l); }
inline uint32_t uniform(uint32_t v) { return lane_of(v, 0); }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __float_as_int(float f) { return std::bit_cast<int>(f); }
inline float __int_as_float(int i) { return std::bit_cast<float>(i); }
// row_shr:n (0x110 + n), row_bcast:15 (0x142) and row_bcast:31 (0x143)
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int rows, int, bool) {
    const int row = g_lane / 16;
    int src = ctrl == 0x142 ? row * 16 - 1 : ctrl == 0x143 ? 31 : g_lane - (ctrl - 0x110);
    const bool in = (rows >> row & 1) && (ctrl < 0x140 ? src >= row * 16 : row > 0);
    const int o = lane_of(v, in ? src : g_lane);
    return in ? o : old;
}
inline uint32_t __builtin_amdgcn_udot4(uint32_t a, uint32_t b, uint32_t c, bool) {
    for (int k = 0; k < 32; k += 8) c += (a >> k & 255u) * (b >> k & 255u);
    return c;
}
template <class V> uint32_t __builtin_amdgcn_udot2(V a, V b, uint32_t c, bool) {
    return c + (uint32_t)a[0] * b[0] + (uint32_t)a[1] * b[1];
}
inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
"""

CHECK = r"""
// 64 * NS candidates of a node of weight N: thresholds of a histogram of rows over
// `bins` bins, two classes, of which the valid ones (a non-empty bin below B - 1
// with rows on the right) number from none to all
template <int FB, int NS> void check(int rank, int bins, int rows, int B, unsigned seed) {
    std::mt19937 rng(seed);
    std::vector<uint32_t> left(256, 0);  // packed counts per bin, then up to each bin
    std::vector<bool> own(256, false);
    const uint32_t base = bins > 1 ? rng() % 8 : rng() % 256;
    for (int r = 0; r < rows; ++r) {
        const uint32_t b = base + (bins > 1 ? rng() % bins : 0);
        left[b] += 1u << FB * (rng() & 1u);
        own[b] = true;
    }
    for (int b = 1; b < 256; ++b) left[b] += left[b - 1];
    const uint32_t cn = left[255], S = dotf<FB>(cn, cn, 0u), N = (uint32_t)rows;
    int want = -1;
    Frac best{0, 0};
    for (int b = 0; b <= B - 2; ++b) {
        const Side s = side_of<1, FB>(&left[b], &cn, S);
        if (!own[b] || s.nl == N) continue;
        const Frac f = side_frac(s, N);
        if (want < 0 || (u128)f.nn * best.nd > (u128)best.nn * f.nd) want = b, best = f;
    }
    ItemBest got[64];
    std::vector<std::thread> lanes;
    for (int l = 0; l < 64; ++l)
        lanes.emplace_back([&, l] {
            g_lane = l;
            float q[NS];
            int b[NS];
            Side sd[NS];
            bool ok[NS];
            for (int u = 0; u < NS; ++u) {
                // NS = 4: the bins in order; fewer: some of them, any number of times
                b[u] = NS == 4 ? 4 * l + u : (int)((base + (l * NS + u) % (2 * bins)) & 255u);
                sd[u] = side_of<1, FB>(&left[b[u]], &cn, S);
                ok[u] = own[b[u]] && b[u] <= B - 2 && sd[u].nl < N;
                q[u] = ok[u] ? side_q32(sd[u], N) : -1.0f;
            }
            got[l] = pick_threshold<FB, NS>(q, b, sd, ok, N, rank);
        });
    for (auto& t : lanes) t.join();
    for (int l = 0; l < 64; ++l)
        if (got[l].b < 0 || got[l].b > 255 || (want < 0) != (got[l].q < 0.0f) ||
            (want >= 0 && got[l].b != want)) {
            std::printf("FB %d NS %d rank %d bins %d rows %d B %d seed %u lane %d: bin %d score %g, "
                        "expected bin %d\n", FB, NS, rank, bins, rows, B, seed, l, got[l].b,
                        (double)got[l].q, want);
            std::exit(1);
        }
}
template <int FB, int NS> void all(int rank) {
    unsigned seed = 1;
    for (int bins : {1, 2, 3, 30})
        for (int rows : {2, 9, 64, 200}) check<FB, NS>(rank, bins, rows, 256, seed++);
    check<FB, NS>(rank, 3, 40, 2, seed++);  // most rows past the last threshold
    check<FB, NS>(rank, 1, 40, 2, seed++);
}
int main(int, char** a) {
    const int rank = std::atoi(a[1]);
    all<8, 1>(rank), all<8, 2>(rank), all<8, 4>(rank);
    all<16, 1>(rank), all<16, 2>(rank), all<16, 4>(rank);
    return 0;
}
"""


def part(text, first, last):
    i = text.index(first)
    return text[i:text.index(last, i)]


@pytest.mark.parametrize("rank", [0, 1], ids=["exact", "fp32"])
def test_the_chosen_threshold_is_a_bin_and_the_best_one(rank, tmp_path):
    text = open(HEADER).read()
    src = tmp_path / "choice.cpp"
    src.write_text(WAVE + part(text, "__device__ __forceinline__ float wave_max_f_dpp", "// The same") +
                   part(text, "__device__ __forceinline__ float fp32_floor", "\n") + "\n" +
                   part(text, "struct Side {", "enum : int { kLeaf") + CHECK)
    exe = str(tmp_path / "choice")
    subprocess.run(["g++", "-std=c++20", "-O1", "-Wno-unknown-pragmas", "-pthread", str(src), "-o",
                    exe], check=True)
    r = subprocess.run([exe, str(rank)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
