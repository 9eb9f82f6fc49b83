"""What the backward's host code (csrc/backward.hip) launches: the code by itself, its launches replaced by a line of text (no GPU
needed)."""
import collections
import os
import subprocess

import pytest

from paper_2605_29517_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")

HARNESS = r"""
#include "%(csrc)s/common.h"
#include <cstdio>
#include <cstring>
#include <tuple>
#undef hipLaunchKernelGGL
#define hipGetLastError() hipSuccess // (there is no device)
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) report(#kernel, grid, __VA_ARGS__)
template <typename P, typename... A> void report(const char *kernel, dim3 grid, const P &p, A... a)
{
    if (strstr(kernel, "ce_"))
        printf("%%s ", strstr(kernel, "small") ? "small" : strstr(kernel, "loss") ? "loss" : "grad");
    if constexpr (sizeof...(A) >= 9) { // bwd_both_kernel
        const auto t = std::make_tuple(a...);
        printf("both %%u %%u %%d\n", grid.x, (unsigned)std::get<6>(t), (int)std::get<7>(t));
    } else if constexpr (sizeof...(A) == 6) { // bwd_dd_kernel
        const auto t = std::make_tuple(a...);
        printf("dD %%u %%d %%d\n", grid.x, std::get<5>(t).n_blocks, p.doc_blocks);
    }
}
#include "%(csrc)s/backward.hip"
int main(int argc, char **)
{
    if (argc > 1) {
        int n, b;
        float x;
        while (scanf("%%d %%d", &n, &b) == 2)
            printf("%%s\n", maxsim::ce_grad_launch(&x, n, b, 1.0f, &x, &x, nullptr) == hipSuccess ? "" : "error");
        return 0;
    }
    int n_q, l_q, ragged, d, dtype;
    long b, tokens;
    static int32_t some[4];
    static float grad[4];
    while (scanf("%%d %%d %%ld %%ld %%d %%d %%d", &n_q, &l_q, &b, &tokens, &ragged, &d, &dtype) == 7)
        if (maxsim::backward_launch(some, n_q, l_q, some, ragged ? some : nullptr, b, ragged ? 0 : (int)(tokens / b), tokens, d, dtype, some, grad, grad, grad, 256, nullptr) != hipSuccess)
            return 1;
    return 0;
}
"""

F32, F16 = 0, 1
Call = collections.namedtuple("Call", "n_q l_q b tokens ragged d dtype", defaults=(128, F16))
Launch = collections.namedtuple("Launch", "kind workgroups n_dq n_part")  # of dD by itself: blocks, blocks per document (0: consecutive rows)


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    d = tmp_path_factory.mktemp("backward")
    src = d / "harness.hip"
    src.write_text(HARNESS % {"csrc": B.CSRC})
    exe = d / "harness"
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--cuda-host-only", "-Wl,--unresolved-symbols=ignore-all", str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)

    def run(calls, *mode):
        text = "".join(" ".join(str(int(v)) for v in c) + "\n" for c in calls)
        out = subprocess.run([str(exe), *mode], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(calls)
        if mode:
            return [line.split() for line in out]
        return [Launch(f[0], *(int(v) for v in f[1:])) for f in (line.split() for line in out)]
    return run


# (queries, tokens, documents, tokens of each, partitions, sets of as many wavefronts in a workgroup)
@pytest.mark.parametrize("n_q,l_q,b,l_d,parts,sets", [(64, 64, 64, 64, 1, 8), (2, 2000, 90, 64, 1, 8), (16, 250, 90, 64, 1, 8), (50, 40, 100, 50, 2, 4), (41, 25, 100, 50, 4, 2), (64, 20, 100, 128, 8, 1),
                                                      (16, 64, 64, 16, 1, 1), (16, 32, 16, 128, 4, 1), (1, 1, 1, 1, 1, 1)])
@pytest.mark.parametrize("ragged", [0, 1])
def test_one_launch_has_no_idle_wavefronts(launches, n_q, l_q, b, l_d, parts, sets, ragged):
    """A wavefront per four query tokens and partition, in workgroups of eight, from a workgroup per CU on; their number is rounded up to a
    multiple of eight."""
    r, = launches([Call(n_q, l_q, b, b * l_d, ragged)])
    assert r.kind == "both" and r.n_part == parts
    assert r.n_dq == -(-n_q * l_q // (32 * sets)) * 8


# Many rows to gather beside many blocks of dD: three launches
@pytest.mark.parametrize("n_q,l_q,b,l_d,d,dtype,kind", [(40, 32, 300, 100, 128, F16, "dD"), (40, 32, 300, 96, 128, F16, "both"), (40, 32, 280, 128, 128, F16, "both"), (40, 32, 300, 200, 256, F16, "dD"),
                                                        (116, 27, 116, 60, 256, F16, "both"), (116, 27, 116, 336, 256, F32, "dD"), (103, 24, 103, 400, 128, F16, "both"), (80, 24, 80, 1024, 128, F16, "both"),
                                                        (64, 64, 64, 64, 512, F32, "both"), (8, 64, 700, 128, 128, F32, "both"), (9, 60, 700, 128, 128, F32, "dD")])
def test_one_launch_by_what_is_gathered(launches, n_q, l_q, b, l_d, d, dtype, kind):
    assert launches([Call(n_q, l_q, b, b * l_d, 0, d, dtype)])[0].kind == kind


# dD by itself: blocks of 32, 64 or 128 rows that end with their document, or of consecutive rows where those by document would need
# one round more; ragged corpora have consecutive rows, as many as the rule by itself says
@pytest.mark.parametrize("n_q,l_q,b,l_d,d,dtype,rows,by_document", [(146, 104, 146, 48, 128, F32, 32, False), (24, 86, 67, 473, 256, F16, 128, False), (105, 86, 151, 52, 128, F32, 32, False),
                                                                    (114, 870, 114, 504, 128, F16, 128, True), (256, 32, 256, 1024, 128, F16, 128, True), (38, 486, 38, 1288, 128, F16, 128, True), (26, 1007, 26, 902, 128, F16, 32, True),
                                                                    (250, 64, 250, 1000, 128, F16, 128, True), (256, 32, 256, 33, 128, F16, 32, True), (64, 1000, 64, 100, 128, F16, 32, True),
                                                                                    (95, 935, 440, 27, 256, F32, 32, True)])
def test_blocks_of_dd(launches, n_q, l_q, b, l_d, d, dtype, rows, by_document):
    n = -(-l_d // rows)
    r, ragged = launches([Call(n_q, l_q, b, b * l_d, 0, d, dtype), Call(n_q, l_q, b, b * l_d, 1, d, dtype)])
    assert (r.kind, *r[2:]) == ("dD", *((b * n, n) if by_document else (-(-b * l_d // rows), 0)))
    assert ragged.n_part == 0 and ragged.n_dq in [-(-b * l_d // x) for x in (32, 64, 128)]


# gradient and loss in one launch, of one workgroup: sixteen rows of up to 256 columns, 64 rows of up to 64
@pytest.mark.parametrize("n,b,one", [(1, 1, True), (16, 256, True), (16, 257, False), (17, 64, True), (17, 65, False), (64, 64, True), (33, 256, False), (64, 256, False), (65, 65, False)])
def test_cross_entropy_in_one_launch(launches, n, b, one):
    assert launches([(n, b)], "ce") == [["small"] if one else ["grad", "loss"]]
