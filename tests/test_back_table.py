"""The backward contractions' pair table (dstd_back.h), its code compiled for the
CPU. g_table_fill runs with one thread per GPU thread: every thread may read every
entry as soon as the call returns, however late another thread is. grad_triple's
interval index leads g_rows to entries that exist, whatever the caller's is."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_14672_amd", "csrc")

HARNESS = r"""
#include <pthread.h>
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#include <unistd.h>
#define __device__
#define __host__
#define __forceinline__ inline
#define __syncthreads() pthread_barrier_wait(&bar)
struct float2 { float x, y; };
static float2 make_float2(float x, float y) { return float2{x, y}; }
struct Dim { int x; };
static thread_local Dim threadIdx;
static Dim blockDim;
static pthread_barrier_t bar;
struct LifConst { int M; float dt, inv_tv, inv_ti, t0, slope_floor; };
static float kern(const LifConst &, float u) { return 1.f + u; }
using std::min;
@FUNCS@
// the first and last entry that g_rows reads for an interval index
static int rows(int M) {
    const LifConst C{M, 0.25f, 1.f, 2.f, 0.f, 1e-6f};
    for (int q : {-5, -1, 0, 1, M - 1, M, M + 1, M + 2, 3 * M + 7, 1 << 30}) {
        const GradTriple t = grad_triple(C, 0.25f * M + 0.1f, 1.f, q, 1.f);
        const int lo = t.q + M + 3 - (M + 2), hi = t.q + M + 3 - 1;  // rows r = 1 .. M + 2
        if (t.q < -1 || lo < 0 || hi >= g_table_len(M)) return printf("q %d -> %d\n", q, t.q), 1;
        if (t.q != (q < 0 ? -1 : min(q, M))) return printf("q %d -> %d\n", q, t.q), 1;
    }
    return 0;
}
int main(int argc, char **argv) {
    if (argc == 2) return rows(atoi(argv[1]));
    const int M = atoi(argv[1]), n = atoi(argv[2]), late = atoi(argv[3]);
    const LifConst C{M, 0.25f, 1.f, 1.f, 0.f, 1e-6f};
    blockDim.x = n;
    pthread_barrier_init(&bar, nullptr, n);
    std::vector<float2> tab(g_table_len(M), float2{-7.f, -7.f});
    std::vector<int> bad(n, 0);
    std::vector<std::thread> th;
    for (int t = 0; t < n; ++t)
        th.emplace_back([&, t] {
            threadIdx.x = t;
            if (t == late) usleep(200000);
            g_table_fill(C, tab.data());
            for (int k = 0; k < g_table_len(M); ++k) {
                const int d = k - (M + 2);
                const float y = d >= 0 ? 1.f + d * 0.25f : 0.f;
                bad[t] += reinterpret_cast<volatile float &>(tab[k].y) != y;
            }
        });
    for (auto &t : th) t.join();
    int sum = 0;
    for (int b : bad) sum += b;
    printf("%d\n", sum);
    return sum != 0;
}
"""


def _function(src, head):
    i = src.index(head)
    j = src.index("{", i)
    depth = 0
    for k in range(j, len(src)):
        depth += {"{": 1, "}": -1}.get(src[k], 0)
        if depth == 0:
            return src[i:k + 1]
    raise AssertionError(f"{head}: no end")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    src = ""
    for name in ("dstd_internal.h", "dstd_back.h"):
        with open(os.path.join(CSRC, name)) as f:
            src += re.sub(r"//[^\n]*", "", f.read())
    fn = "\n".join(_function(src, h) for h in (
        "struct GradPrep", "__device__ __forceinline__ GradPrep grad_prep",
        "__host__ __device__ __forceinline__ int g_table_len",
        "__device__ __forceinline__ void g_table_fill", "struct GradTriple",
        "__device__ __forceinline__ GradTriple grad_triple"))
    fn = re.sub(r"(struct \w+ {[^}]*})", r"\1;", fn)
    d = tmp_path_factory.mktemp("back_table")
    cpp, out = str(d / "t.cpp"), str(d / "t")
    with open(cpp, "w") as f:
        f.write(HARNESS.replace("@FUNCS@", fn))
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-o", out, cpp], check=True)
    return out


# threads per block x grid lengths: a table of more and of fewer entries than threads
@pytest.mark.parametrize("M,threads,late", [(32, 64, 0), (32, 64, 63), (8, 64, 19), (256, 128, 127)])
def test_table_is_complete_for_every_thread(exe, M, threads, late):
    r = subprocess.run([exe, str(M), str(threads), str(late)], capture_output=True, text=True,
                       timeout=60)
    assert r.returncode == 0, f"{r.stdout.strip()} entries read before they were written"


@pytest.mark.parametrize("M", [1, 8, 256])
def test_interval_index_stays_in_the_table(exe, M):
    r = subprocess.run([exe, str(M)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
