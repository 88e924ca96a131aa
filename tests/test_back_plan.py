"""The dense backward's launch shapes (plan_back in dstd_back.hip), compiled for
the CPU: they fill the chip for small layers and for every number of intervals, fit
the hardware and the workspace, and give one gradient alone the sums of both."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_14672_amd", "csrc")

HARNESS = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#define __device__
#define __host__
#define __forceinline__ inline
struct float2 { float x, y; };
constexpr int kWave = 64;
@CODE@
int main(int argc, char **argv) {
    int64_t v[7];  // B, N_in, N_out, F, M, copied G, which gradients (1 dW, 2 dt_in, 3 both)
    while (scanf("%ld %ld %ld %ld %ld %ld %ld", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6) == 7) {
        const int64_t cap = back_split_cap(v[0], v[1], v[2]), buf = back_buf_cap(v[0], v[1], v[3], v[2]);
        const BackPlan p = plan_back(BackSize{v[0], v[1], v[2], v[3], v[5] != 0, cap, buf},
                                     static_cast<int>(v[4]), v[6] & 1, v[6] & 2);
        printf("%d %d %d %d %d %d %d %d %zu %ld %ld\n", p.nt, p.tj, p.tiles, p.groups, p.waves, p.nsplit,
               p.b_per_split, p.ahead, p.lds, cap, buf);
    }
}
"""
FIELDS = "nt tj tiles groups waves nsplit b_per_split ahead lds cap n_buf".split()


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    def read(name):
        with open(os.path.join(CSRC, name)) as f:
            return f.read()
    back, kern = read("dstd_back.hip"), read("dstd_kernels.h")
    code = re.search(r"struct BackPlan \{.*?\n\};", kern, re.S)[0] + "\n"
    code += re.search(r"struct BackSize \{.*?\n\};", kern, re.S)[0] + "\n"
    code += re.search(r"[^\n]*int g_table_len\(int M\)[^\n]*", read("dstd_back.h"))[0] + "\n"
    code += "\n".join(re.findall(r"^constexpr int kBack(?:WavesMax|Ahead) [^\n]*", back, re.M)) + "\n"
    code += back[back.index("constexpr int kBackLdsDense"):back.index("// ---- end of the launch rules")]
    d = tmp_path_factory.mktemp("back_plan")
    cpp, exe = str(d / "t.cpp"), str(d / "t")
    with open(cpp, "w") as f:
        f.write(HARNESS.replace("@CODE@", code))
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, cpp], check=True)

    def run(shapes):
        text = "\n".join(" ".join(str(int(x)) for x in s) for s in shapes)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        out = [dict(zip(FIELDS, map(int, line.split()))) for line in r.stdout.splitlines()]
        assert len(out) == len(shapes)
        return out
    return run


SIZES = [(B, i, o, F, M) for B in (1, 3, 24, 100, 256, 65535) for i in (1, 17, 400, 6000)
         for o in (1, 64, 65, 128, 129, 1000, 4096) for F in (1, 4) for M in (1, 32, 65, 147, 148, 256)
         if B * i * o < 1 << 31]


def test_plans_fit_hardware_and_workspace(plan):
    shapes = [s + (F > 1, m) for s in SIZES for F in (s[3],) for m in (1, 2, 3)]
    for s, p in zip(shapes, plan(shapes)):
        B, i, o, F, M, mem, mode = s
        assert p["nt"] in (1, 2) and p["tj"] in (8, 16) and 1 <= p["waves"] <= 16, (s, p)
        assert p["tiles"] * p["nt"] * 64 >= o > (p["tiles"] - 1) * p["nt"] * 64, (s, p)
        assert p["groups"] * p["waves"] * p["tj"] >= i, (s, p)
        assert p["nsplit"] * p["b_per_split"] >= B > (p["nsplit"] - 1) * p["b_per_split"], (s, p)
        assert p["lds"] <= 160 * 1024 and p["ahead"] in (1, 2, 4), (s, p)
        assert p["lds"] == 2 * p["ahead"] * (M + 3) * p["nt"] * 256 + (2 * M + 4) * 8, (s, p)
        assert p["nsplit"] <= 65535 and p["tiles"] <= 65535
        if mode & 1:
            assert p["nsplit"] <= p["cap"], (s, p)


def test_one_gradient_alone_keeps_the_order_of_its_sums(plan):
    shapes = [s + (F > 1,) for s in SIZES for F in (s[3],)]
    both = plan([s + (3,) for s in shapes])
    for s, b, w, t in zip(shapes, both, plan([s + (1,) for s in shapes]), plan([s + (2,) for s in shapes])):
        assert w["b_per_split"] == b["b_per_split"], s
        assert t["nt"] == b["nt"] and t["n_buf"] == b["n_buf"], s


@pytest.mark.parametrize("mode", [1, 2, 3])
@pytest.mark.parametrize("B,N_in,N_out,F,M", [
    (24, 400, 120, 1, 64), (32, 256, 128, 1, 64), (8, 784, 100, 1, 16), (64, 100, 50, 1, 32),
    (32, 256, 64, 4, 32), (16, 64, 40, 4, 20)])
def test_small_layers_fill_the_chip(plan, B, N_in, N_out, F, M, mode):
    """At least a wave per CU (50 to 128 waves with one shape for every layer), or a
    quarter of what one sample and eight inputs per wave come to."""
    p, = plan([(B, N_in, N_out, F, M, F > 1, mode)])
    waves = p["groups"] * p["waves"] * p["tiles"] * p["nsplit"]
    pieces = -(-N_in // 8) * -(-N_out // (64 * p["nt"])) * B
    assert waves >= min(256, pieces / 4), (waves, p)


@pytest.mark.parametrize("N_out", [100, 1000])
def test_multispike_splits_do_not_end_at_64_intervals(plan, N_out):
    a, b = plan([(128, 784, N_out, 4, M, 1, 3) for M in (64, 65)])
    assert b["groups"] * b["waves"] * b["nsplit"] * b["tiles"] >= \
        0.9 * a["groups"] * a["waves"] * a["nsplit"] * a["tiles"]
    assert b["n_buf"] >= b["tiles"] - 1
