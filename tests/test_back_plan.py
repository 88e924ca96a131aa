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


CONV_HARNESS = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#define __device__
#define __host__
#define __forceinline__ inline
struct float2 { float x, y; };
constexpr int kWave = 64;
struct ConvGeom { int C_in, C_out, KH, KW, stride, Hp, Wp, Ho, Wo, P, PC; };
@CODE@
int main() {
    long v[11];  // B, C_in, C_out, KH, KW, stride, map, output map, P, M, which gradients
    while (scanf("%ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6,
                 v + 7, v + 8, v + 9, v + 10) == 11) {
        auto n = [&](int k) { return static_cast<int>(v[k]); };
        const ConvGeom g{n(1), n(2), n(3), n(4), n(5), n(6), n(6), n(7), n(7), n(8), n(1) * n(8)};
        const ConvBackPlan p = plan_conv_back(g, v[0], n(9), v[10] & 1, v[10] & 2);
        printf("%d %d %d %d %d %d %d %d %d %d %d %d %zu\n", p.kwt, p.nt, p.tj, p.kg, p.tiles, p.tiles_dt, p.cpt,
               p.n_chunk, p.groups, p.waves, p.nsplit, p.rows_per_split, p.lds);
    }
}
"""
CONV_FIELDS = "kwt nt tj kg tiles tiles_dt cpt n_chunk groups waves nsplit rows_per_split lds".split()


@pytest.fixture(scope="module")
def conv_plan(tmp_path_factory):
    def read(name):
        with open(os.path.join(CSRC, name)) as f:
            return f.read()
    conv, kern = read("dstd_conv.hip"), read("dstd_kernels.h")
    code = re.search(r"struct ConvBackPlan \{.*?\n\};", kern, re.S)[0] + "\n"
    code += re.search(r"[^\n]*int g_table_len\(int M\)[^\n]*", read("dstd_back.h"))[0] + "\n"
    code += re.search(r"constexpr int back_ring\(int kwt\)[^\n]*", conv)[0] + "\n"
    code += "\n".join(re.findall(r"^constexpr int k(?:BackWaves|DwPairs) [^\n]*", conv, re.M)) + "\n"
    code += conv[conv.index("constexpr int kBackLds "):
                 conv.index("// ---- end of the launch rules of conv_back_kernel")]
    d = tmp_path_factory.mktemp("conv_plan")
    cpp, exe = str(d / "t.cpp"), str(d / "t")
    with open(cpp, "w") as f:
        f.write(CONV_HARNESS.replace("@CODE@", code))
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, cpp], check=True)

    def run(shapes):
        text = "\n".join(" ".join(str(int(x)) for x in s) for s in shapes)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        out = [dict(zip(CONV_FIELDS, map(int, line.split()))) for line in r.stdout.splitlines()]
        assert len(out) == len(shapes)
        return out
    return run


def _conv_shapes(mode):
    return [(B, ci, co, k, k, s, hw, (hw - 1) // s + 1, P, M, mode)
            for B in (1, 16, 128) for ci in (1, 8, 9, 100) for co in (16, 64, 65, 512) for k in (1, 3, 7)
            for s in (1, 2) for hw in (4, 28) for P in (1, 4) for M in (1, 32, 100, 150, 256)]


def test_conv_plans_fit_hardware_and_workspace(conv_plan):
    for mode in (1, 2, 3):
        for s, p in zip(_conv_shapes(mode), conv_plan(_conv_shapes(mode))):
            B, ci, co, k, _, st, hw, ho, P, M, _ = s
            assert (p["kwt"], p["nt"], p["tj"]) in ((3, 2, 8), (3, 1, 16), (3, 1, 8), (1, 2, 16), (1, 2, 8),
                                                    (1, 1, 16), (1, 1, 8)), (s, p)
            assert p["kwt"] == 1 or (st == 1 and k > 1), (s, p)
            assert p["tiles"] * p["nt"] * 64 >= co and p["kg"] * p["kwt"] >= k, (s, p)
            assert p["cpt"] * p["tj"] >= ci and p["n_chunk"] == p["cpt"] * k * p["kg"], (s, p)
            assert p["groups"] * p["waves"] >= p["n_chunk"] and 1 <= p["waves"] <= 12, (s, p)
            assert (p["groups"] - 1) * p["waves"] < p["n_chunk"], (s, p)
            assert p["nsplit"] * p["rows_per_split"] >= B * ho > (p["nsplit"] - 1) * p["rows_per_split"], (s, p)
            assert p["lds"] + 1024 <= 160 * 1024 and p["nsplit"] <= 4096, (s, p)
            assert 1 <= p["tiles_dt"] <= p["tiles"]
            entries = k * p["kg"] * p["tiles_dt"]
            assert entries <= max(k * k + 1, k * p["kg"]) or entries * B * hw * hw * ci * P * 4 <= 32 << 20, (s, p)
            if mode & 1 and p["nsplit"] > 1:
                assert p["nsplit"] * k * k * ci * co * 4 <= 64 << 20, (s, p)


def test_one_conv_gradient_alone_keeps_the_order_of_its_sums(conv_plan):
    both = conv_plan(_conv_shapes(3))
    for s, b, w, t in zip(_conv_shapes(3), both, conv_plan(_conv_shapes(1)), conv_plan(_conv_shapes(2))):
        assert w["rows_per_split"] == b["rows_per_split"], s
        assert all(t[f] == b[f] for f in ("kwt", "nt", "kg", "tiles", "tiles_dt")), s


@pytest.mark.parametrize("B,ci,co,k,hw,P,M", [
    (16, 16, 32, 3, 8, 1, 32), (4, 53, 101, 1, 5, 4, 21), (8, 160, 16, 1, 10, 1, 16), (5, 2, 132, 3, 5, 1, 64)])
def test_small_conv_layers_take_every_row(conv_plan, B, ci, co, k, hw, P, M):
    """A split per output row where there are fewer rows than CUs (16 positions or
    more per split had left 1 to 32 blocks)."""
    p, = conv_plan([(B, ci, co, k, k, 1, hw, hw, P, M, 3)])
    assert p["nsplit"] >= min(B * hw, 256) / 2, p
