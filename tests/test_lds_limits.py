"""The LDS limits of the kernels that take more than 64 KB belong to the process:
preparing a plan sets the same limit whatever its size (the functions that set
them, compiled with g++ around a recording hipFuncSetAttribute), so that a smaller
plan leaves a larger one's session running.  The GPU test steps such a session."""
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2605_09950_amd import binding as B

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2605_09950_amd", "csrc")

HEAD = r"""
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <type_traits>
enum hipError_t { hipSuccess };
enum { hipFuncAttributeMaxDynamicSharedMemorySize, hipDeviceAttributeMaxSharedMemoryPerBlock };
static int g_limit;
hipError_t hipFuncSetAttribute(const void*, int, int v) { return g_limit = v, hipSuccess; }
hipError_t hipGetDevice(int*) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, int, int) { return *v = 160 * 1024, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
static const void* grow_fn(int) { return nullptr; }
static const void* hist_col_fn(int) { return nullptr; }
static void k_boot_draw_lds() {}
"""
MAIN = r"""
template <class F> int limit(F f, size_t lds) {
    if constexpr (std::is_invocable_v<F, int, size_t>) f(3, lds); else f(3);
    return g_limit;
}
int main() {
    const int a[] = {limit(prepare_grow, 120000), limit(prepare_hist_col, 120000)};
    const int b[] = {limit(prepare_grow, 70000), limit(prepare_hist_col, 70000)};
    prepare_boot_draw(30000);
    const int c = g_limit;
    prepare_boot_draw(17000);
    std::printf("%d %d %d after smaller plans %d %d %d\n", a[0], a[1], c, b[0], b[1], g_limit);
    return a[0] == b[0] && a[1] == b[1] && c == g_limit && a[0] >= 120000 && a[1] >= 120000 &&
           c >= 120000 ? 0 : 1;
}
"""


def test_a_smaller_plan_leaves_the_limits(tmp_path):
    forest, prep, common = (open(os.path.join(CSRC, f)).read()
                            for f in ("k_forest.hip", "k_prep.hip", "dev_common.hpp"))

    def function(text, name):
        i = text.index(name + "(")
        i = text.rindex("\n", 0, i) + 1
        return text[i:text.index("\n}\n", i) + 3]

    consts = "\n".join(re.findall(r"^constexpr \w+ k(?:LdsPerWorkgroup|GrowStaticLds|BootLds\w+) = [^;]*;",
                                  common + prep, re.M))
    src = tmp_path / "limits.cpp"
    src.write_text(HEAD + consts + "\n" + function(forest, "prepare_grow") +
                   function(forest, "prepare_hist_col") + function(prep, "prepare_boot_draw") + MAIN)
    exe = str(tmp_path / "limits")
    subprocess.run(["g++", "-std=c++17", str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("tune", [None, dict(col_level=1)], ids=["whole_trees", "column"])
def test_a_session_runs_on_beside_a_smaller_plan(tune):
    rng = np.random.default_rng(77)
    n = 4000 if tune is None else 60000
    X = rng.standard_normal((n, 5)).astype(np.float32)
    y = np.argmax(X[:, :3], axis=1).astype(np.int32)

    def job(m):
        return dict(X=X[:m], y=y[:m], n_classes=3, n_trees=4, max_depth=5, max_iter=4, seed=1)

    kw = dict(graph=False, tune=tune)
    print(f"a session of {n} rows beside one of 200, tune={tune}", flush=True)
    with B.Session([job(n)], **kw) as alone:
        while alone.step():
            pass
        want = alone.result(0)
    with B.Session([job(n)], **kw) as big:
        big.step()
        with B.Session([job(200)], **kw) as small:
            small.step()
            while big.step():
                pass
        got = big.result(0)
    for k in ("decision", "hits", "imp_history", "shadow_max"):
        assert np.array_equal(got[k], want[k], equal_nan=True)
