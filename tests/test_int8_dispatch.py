"""Which int8 kernel forward_i8_launch (csrc/int8.hip) takes for a call: the host code by itself, its launches replaced by a line of
text (no GPU needed)."""
import collections
import os
import subprocess

import pytest

from paper_2605_29517_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")

HARNESS = r"""
#include "%(csrc)s/int8_impl.h"
#include <cstdio>
#undef hipLaunchKernelGGL
#define hipGetLastError() hipSuccess // (there is no device)
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) printf("%%s %%u %%u\n", #kernel, dim3(grid).x, dim3(block).x)
#include "%(csrc)s/int8.hip"
#include "%(csrc)s/int8_rows64.hip"
int main()
{
    int n_q, l_q, ragged;
    long b, tokens;
    static int32_t some[4];
    static float scale[4];
    while (scanf("%%d %%d %%ld %%ld %%d", &n_q, &l_q, &b, &tokens, &ragged) == 5)
        if (maxsim::forward_i8_launch((int8_t *)some, scale, n_q, l_q, (int8_t *)some, scale, ragged ? some : nullptr, b, ragged ? 0 : (int)(tokens / b), tokens, scale, b, 256, nullptr) != hipSuccess)
            return 1;
    return 0;
}
"""

Call = collections.namedtuple("Call", "n_q l_q b tokens ragged")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    d = tmp_path_factory.mktemp("int8")
    src = d / "harness.hip"
    src.write_text(HARNESS % {"csrc": B.CSRC})
    exe = d / "harness"
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--cuda-host-only", "-Wl,--unresolved-symbols=ignore-all", str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)

    def run(calls):
        text = "".join(" ".join(str(int(v)) for v in c) + "\n" for c in calls)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(calls)
        return [(line[line.index("fwd_"):line.index("_kernel")], int(line.split()[-1]) // 64) for line in out]  # the kernel, its wavefronts
    return run


# documents of equal length on few CUs' worth of documents: eight wavefronts share each of them, where 64 rows per step are not ahead
@pytest.mark.parametrize("n_q,l_q,b,l_d,want", [
    (1, 32, 149, 634, "i8_split"), (1, 20, 7, 334, "i8_split"), (1, 73, 9, 351, "i8_split"), (1, 32, 253, 939, "i8_split"), (4, 31, 237, 776, "i8_split"), (3, 32, 20, 665, "i8_split"),
    (6, 32, 400, 1030, "i8_split"), (1, 509, 128, 1030, "i8_split"), (1, 32, 149, 255, "i8_split"),
    (9, 18, 1160, 807, "i8_split"), (9, 18, 1290, 807, "i8_rows64"), (3, 145, 3705, 378, "i8_rows64"), (4, 114, 282, 959, "i8_rows64"), (13, 16, 249, 1072, "i8_rows64"),
    (1, 29, 1024, 1030, "i8_rows64"), (1, 224, 1050, 332, "i8_rows64"), (16, 32, 4, 1030, "i8_rows64"), (17, 32, 20, 300, "i8_rows64"), (1, 602, 3, 300, "i8_rows64"), (4, 310, 500, 1000, "i8_rows64"),
    (1, 64, 3000, 1024, "i8_rows64"), (5, 70, 5, 159, "i8_rows64"), (1, 1009, 300, 64, "i8_rows64"), (1, 1024, 40000, 1024, "i8_rows64"), (1, 32, 40000, 300, "i8_doc")])
def test_equal_documents(kernels, n_q, l_q, b, l_d, want):
    (kernel, waves), = kernels([Call(n_q, l_q, b, b * l_d, 0)])
    assert kernel == "fwd_" + want
    assert waves == (2 if l_d < 256 and want == "i8_split" else 8)


def test_ragged_documents_are_not_shared_by_eight(kernels):
    for b, tokens in ((7, 300), (1000, 180), (4095, 1000)):
        for n_q, l_q, want in ((1, 32, ("fwd_i8_split", 2)), (8, 32, ("fwd_i8_split", 4)), (9, 32, ("fwd_i8", 4))):
            assert kernels([Call(n_q, l_q, b, b * tokens, 1)])[0] == want
