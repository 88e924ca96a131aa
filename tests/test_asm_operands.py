"""Inline assembly of several instructions: the registers it writes are none that
a later instruction of the same statement still reads as another operand, also
where operands start out equal (the compiler may then share a register unless the
output is marked as written early). The statements are compiled for gfx950 with
every operand equal, and their instructions read back."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_14672_amd import build

CSRC = os.path.join(build.PKG, "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SRC = r"""
#include <hip/hip_runtime.h>
#include "dstd_back.h"
namespace dstd {
constexpr int kCBatch = 8;
@FWD@
template <int NT> __device__ float fma_same(float v) {
    float a[NT], x[NT];
    for (int c = 0; c < NT; ++c) a[c] = x[c] = v;
    fma_bcast<0, 1, NT>(a, v, v, x, x);
    float s = 0.f;
    for (int c = 0; c < NT; ++c) s += a[c];
    return s;
}
template <int NT> __device__ float dot_same(float v) {
    float a[NT], x[NT];
    for (int c = 0; c < NT; ++c) x[c] = v;
    dot_bcast<0, 1, NT>(a, v, v, x, x);
    float s = 0.f;
    for (int c = 0; c < NT; ++c) s += a[c];
    return s;
}
}  // namespace dstd
using namespace dstd;
extern "C" __global__ void k(float *p, const float *q) {
    const int t = threadIdx.x;
    p[t] = fma_same<1>(q[t]);
    p[t + 64] = fma_same<2>(q[t + 64]);
    p[t + 128] = fma_same<4>(q[t + 128]);
    p[t + 192] = dot_same<1>(q[t + 192]);
    p[t + 256] = dot_same<2>(q[t + 256]);
    p[t + 320] = dot_same<4>(q[t + 320]);
    {
        float v = q[t + 384], L = v, R = v;
        sum_entry<3>(L, R, v, v, v);
        p[t + 384] = L - R;
    }
    {
        float v = q[t + 448], L = v, R = v, w[4] = {v, v, v, v};
        sum_entries4(L, R, v, v, w);
        p[t + 448] = L - R;
    }
    {
        float v = q[t + 512], L = v, R = v, w[8] = {v, v, v, v, v, v, v, v};
        sum_entries8(L, R, v, v, w);
        p[t + 512] = L - R;
    }
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_no_operand_shares_a_register_written_before_its_last_read(tmp_path):
    with open(os.path.join(CSRC, "dstd_conv.hip")) as f:
        conv = f.read()
    fwd = conv[conv.index("#define FWD_FMA"):conv.index("#undef FWD_FMA")]
    src, out = tmp_path / "t.hip", tmp_path / "t.s"
    src.write_text(SRC.replace("@FWD@", fwd))
    flags = [x for x in build.HIPCC_FLAGS if x != "-fPIC"]
    subprocess.run([HIPCC] + flags + ["-I", CSRC, "--cuda-device-only", "-S", "-o", str(out), str(src)],
                   check=True, capture_output=True)
    blocks = re.findall(r";;?#ASMSTART\n(.*?);;?#ASMEND", out.read_text(), re.S)
    blocks = [b for b in blocks if "row_newbcast" in b]
    assert len(blocks) == 9
    for b in blocks:
        written = set()
        for d, x, y in re.findall(r"^\s*v_(?:fmac|mul)_f32_dpp (v\d+), (v\d+), (v\d+) ", b, re.M):
            assert x not in written and y not in written, b
            written.add(d)
        assert written
