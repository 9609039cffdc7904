"""Where boruta_bin places its buffers (bin_plan of engine.hip, compiled with g++):
the keys, which the kernels read 16 bytes at a time, and the bins on multiples of
256 bytes whatever the table's size, no buffer over another, all within the
allocation."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ENGINE = os.path.join(ROOT, "paper_2605_09950_amd", "csrc", "engine.hip")

CHECK = r"""
int main() {
    for (int64_t n : {1, 2, 255, 257, 8193, 8195, 16385, 100003})
        for (int64_t p : {1, 2, 3, 5, 9, 31}) {
            const BinPlan b = bin_plan(n, p);
            const size_t at[] = {b.X, b.keys, b.bins, b.flags, b.total};
            const size_t len[] = {(size_t)(n * p * 4), (size_t)(p * b.P * 4), (size_t)(p * b.n_pad), 4};
            for (int i = 0; i < 4; ++i)
                if (at[i] % 256 || at[i] + len[i] > at[i + 1]) {
                    std::printf("n %ld p %ld: buffer %d of %zu bytes at %zu, the next at %zu\n",
                                (long)n, (long)p, i, len[i], at[i], at[i + 1]);
                    return 1;
                }
        }
    return 0;
}
"""


def test_the_buffers_are_aligned_and_apart(tmp_path):
    text = open(ENGINE).read()

    def part(first, last):
        i = text.index(first)
        return text[i:text.index(last, i)]

    src = tmp_path / "layout.cpp"
    src.write_text("#include <algorithm>\n#include <cstdint>\n#include <cstdio>\n" +
                   part("int64_t round_up(", "int bit_len") +
                   part("int64_t pow2_at_least(", "int isqrt_i") +
                   part("struct Region {", "struct JobPlan {") + CHECK)
    exe = str(tmp_path / "layout")
    subprocess.run(["g++", "-std=c++17", str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
