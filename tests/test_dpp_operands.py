"""Register assignment of the row-broadcast multiply-adds (csrc/dpp.h): no
accumulator shares registers with the row or the multiplier, also where a
caller starts one from either of them.  The instructions of one call run one
after the other, so a shared register would change what the later ones read.
A small kernel is compiled for gfx950 and its assembly is read; no GPU needed.
"""
import os
import re
import subprocess

import pytest

from paper_1110_4874_amd import build

SOURCE = """
#include "dpp.h"
using namespace sht;
template <int N, int C0, int FROM>
__device__ void body(const double *in, double *out) {
    const double rv = in[threadIdx.x], p = in[threadIdx.x + 64];
    double acc[N];
    for (int c = 0; c < N; c++) acc[c] = FROM == 0 ? p : FROM == 1 ? rv : 0.0;
    fmac_row_bcast<N, C0>(acc, FROM == 2 ? 0.0 : rv, FROM == 3 ? 0.0 : p);
    for (int c = 0; c < N; c++) out[c * 64 + threadIdx.x] = acc[c];
}
#define K(N, C0, F) extern "C" __global__ void k_##N##_##C0##_##F(const double *in, double *out) { body<N, C0, F>(in, out); }
#define KS(N, C0) K(N, C0, 0) K(N, C0, 1) K(N, C0, 2) K(N, C0, 3)
KS(2, 0) KS(4, 0) KS(6, 0) KS(8, 0) KS(10, 0) KS(12, 0) KS(16, 0) KS(2, 8) KS(4, 8) KS(6, 8) KS(8, 8)
"""
FMAC = re.compile(r"v_fmac_f64_dpp\s+v\[(\d+):(\d+)\],\s*v\[(\d+):(\d+)\],\s*v\[(\d+):(\d+)\]")


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    """The multiply-adds of every asm block: lists of (dst, rv, p) first registers."""
    d = tmp_path_factory.mktemp("dpp")
    src, out = str(d / "k.hip"), str(d / "k.s")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.check_call([build.HIPCC, *build.HIP_FLAGS, "-O3", "-std=c++17", "-I", build.CSRC, "--cuda-device-only",
                           "-S", src, "-o", out], stderr=subprocess.DEVNULL)
    found, cur = [], None
    for line in open(out):
        if "#APP" in line or "#ASMSTART" in line:
            cur = []
        elif "#NO_APP" in line or "#ASMEND" in line:
            if cur:
                found.append(cur)
            cur = None
        elif cur is not None and (m := FMAC.search(line)):
            cur.append(tuple(int(x) for x in m.groups()[::2]))
    return found


def test_accumulators_have_their_own_registers(blocks):
    assert sum(len(b) for b in blocks) == 4 * (2 + 4 + 6 + 8 + 10 + 12 + 16 + 2 + 4 + 6 + 8)
    for b in blocks:
        dst = [x[0] for x in b]
        assert len(set(dst)) == len(dst), b
        for d, rv, p in b:
            assert rv not in dst and p not in dst, b
