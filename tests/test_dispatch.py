"""Which kernel shape forward_launch (csrc/forward.hip) takes for a call: the host code by itself, its launches replaced by a
line of text (no GPU needed)."""
import collections
import os
import subprocess

import pytest

from paper_2605_29517_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")

HARNESS = r"""
#include "%(csrc)s/forward.hip"
#include <cstdio>
namespace maxsim {
static void print(const char *kind, const FwdParams &p, int nu, int x)
{
    printf("%%s %%d %%d %%d %%d %%d\n", kind, nu, x, p.n_groups, p.qpg, p.n_pass);
}
static hipError_t one(const FwdParams &p, int nu, bool tile, int x) { print(tile ? "tile" : p.n_chunks ? "stream" : "split", p, nu, x); return hipSuccess; }
hipError_t forward_run_f16(const FwdParams &p, int nu, bool, bool tile, int x, int, hipStream_t) { return one(p, nu, tile, x); }
hipError_t forward_run_bf16(const FwdParams &p, int nu, bool, bool tile, int x, int, hipStream_t) { return one(p, nu, tile, x); }
hipError_t forward_run_f32(const FwdParams &p, int nu, bool, bool tile, int x, int, hipStream_t) { return one(p, nu, tile, x); }
hipError_t forward_splitd_launch(FwdParams p, int, int, int, hipStream_t) { print("slabs", p, 0, 0); return hipSuccess; }
hipError_t forward_wide_launch(FwdParams p, int, int, int, hipStream_t) { print("slabs", p, 0, 0); return hipSuccess; }
double forward_splitd_time(FwdParams, int, int, int) { return 1; }
double forward_wide_time(FwdParams, int) { return 1; }
}
int main()
{
    int dtype, d, n_q, l_q, ragged, argmax;
    long b, tokens;
    static int32_t some[1];
    while (scanf("%%d %%d %%d %%d %%ld %%ld %%d %%d", &dtype, &d, &n_q, &l_q, &b, &tokens, &ragged, &argmax) == 8) {
        maxsim::FwdParams p = {};
        p.n_q = n_q;
        p.l_q = l_q;
        p.b = b;
        p.l_d = ragged ? 0 : (int)(tokens / b);
        p.total_tokens = tokens;
        p.offsets = ragged ? some : nullptr;
        p.argmax = argmax ? some : nullptr;
        if (maxsim::forward_launch(p, dtype, d, 256, nullptr) != hipSuccess)
            return 1;
    }
    return 0;
}
"""

Call = collections.namedtuple("Call", "dtype d n_q l_q b tokens ragged argmax")
Route = collections.namedtuple("Route", "kind nu shape n_groups qpg n_pass")
F32, F16, BF16 = 0, 1, 2


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    src = d / "harness.hip"
    src.write_text(HARNESS % {"csrc": B.CSRC})
    exe = d / "harness"
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--cuda-host-only", str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)

    def run(calls):
        text = "".join(" ".join(str(int(v)) for v in c) + "\n" for c in calls)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(calls)
        return [Route(f[0], *(int(v) for v in f[1:])) for f in (line.split() for line in out)]
    return run


def test_groups_are_evened_only_for_three_blocks_per_wavefront(routes):
    """Equal shares cost blocks (a wavefront that holds one block computes all of its own): only where the fullest falls to 24."""
    shapes = [(n_q, l_q) for n_q in list(range(1, 70)) + [100, 180, 200, 256] for l_q in (32, 48, 90, 128, 150, 190, 280, 350, 512)]
    calls = [Call(F16, 128, n_q, l_q, 200, 200 * 350, 0, 1) for n_q, l_q in shapes]
    for c, r in zip(calls, routes(calls)):
        bpq = (c.l_q + 31) // 32
        if r.kind != "tile" or r.shape not in (8, 83) or bpq > 32:
            continue
        most = min(c.n_q, 32 // bpq)
        even = -(-c.n_q // -(-c.n_q // most))
        assert r.n_groups == -(-c.n_q // r.qpg) == -(-c.n_q // most), c
        assert r.qpg == (even if most * bpq > 24 >= even * bpq else most), c
        assert r.shape == (83 if r.qpg * bpq <= 24 else 8), c
