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
#include <cstdlib>
namespace maxsim {
static void print(const char *kind, const FwdParams &p, int nu, int x)
{
    printf("%%s %%d %%d %%d %%d %%d %%d %%d\n", kind, nu, x, p.n_groups, p.qpg, p.n_pass, p.doc_waves, p.docs_per_wg);
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
int main(int argc, char **argv)
{
    const int cus = argc > 1 ? atoi(argv[1]) : 256;
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
        if (maxsim::forward_launch(p, dtype, d, cus, nullptr) != hipSuccess)
            return 1;
    }
    return 0;
}
"""

Call = collections.namedtuple("Call", "dtype d n_q l_q b tokens ragged argmax")
Route = collections.namedtuple("Route", "kind nu shape n_groups qpg n_pass doc_waves docs_per_wg")
F32, F16, BF16 = 0, 1, 2


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    src = d / "harness.hip"
    src.write_text(HARNESS % {"csrc": B.CSRC})
    exe = d / "harness"
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--cuda-host-only", str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)

    def run(calls, cus=256):
        text = "".join(" ".join(str(int(v)) for v in c) + "\n" for c in calls)
        out = subprocess.run([str(exe), str(cus)], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
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


# (documents, tokens of each, ragged, argmax) -> shape, of queries with five to six and with nine to twelve blocks; d = 128
FEW = [(767, 300, 0, 0, 42, 43), (768, 300, 0, 0, 23, 43), (1024, 64, 0, 0, 42, 43), (1024, 65, 0, 0, 23, 43), (1024, 64, 0, 1, 23, 43),
       (1025, 256, 0, 0, 42, 43), (1280, 257, 0, 0, 23, 43), (1280, 96, 0, 1, 42, 43), (1280, 97, 0, 1, 23, 43),
       (1281, 224, 0, 0, 23, 43), (1281, 225, 0, 0, 42, 43), (1536, 640, 0, 1, 42, 43), (1536, 641, 0, 1, 23, 43), (1537, 300, 0, 0, 23, 43),
       (1023, 100, 1, 0, 42, 43), (1024, 128, 1, 0, 23, 43), (1791, 129, 1, 0, 42, 43), (1792, 129, 1, 0, 23, 43), (1535, 129, 1, 1, 42, 43),
       (1536, 129, 1, 1, 23, 43), (300, 96, 0, 0, 42, 82), (512, 97, 0, 0, 42, 43), (513, 160, 0, 1, 42, 82), (768, 161, 0, 0, 23, 43),
       (700, 64, 0, 0, 42, 82), (700, 64, 1, 0, 42, 43), (4096, 100, 0, 1, 23, 43)]


@pytest.mark.parametrize("docs,tokens,ragged,argmax,six,twelve", FEW)
def test_three_blocks_per_wavefront_on_few_documents(routes, docs, tokens, ragged, argmax, six, twelve):
    for blocks, want in (((2, 90), six), ((1, 130) if not argmax else (5, 32), six), ((3, 64), six), ((1, 300) if ragged else (9, 32), twelve), ((2, 192), twelve)):
        n_q, l_q = blocks
        if docs >= 4096 and n_q * ((l_q + 31) // 32) <= 6 and not argmax:
            continue
        call = Call(BF16, 128, n_q, l_q, docs, docs * tokens, ragged, argmax)
        assert routes([call])[0].shape == want, call


# (dtype, d, n_q, l_q, documents, tokens of each, ragged, argmax) -> shape, of queries with 13 to 16 blocks
SIXTEEN = [(F16, 128, 1, 512, 256, 1000, 0, 0, 82), (F16, 128, 1, 512, 257, 1000, 0, 0, 4), (BF16, 128, 1, 400, 384, 512, 0, 0, 4), (BF16, 128, 16, 32, 300, 512, 0, 0, 4),
           (BF16, 128, 1, 400, 385, 512, 0, 0, 82), (BF16, 128, 1, 512, 300, 511, 0, 0, 82), (F16, 128, 1, 512, 300, 1000, 1, 0, 82), (F16, 128, 1, 512, 300, 1000, 0, 1, 82),
           (F16, 64, 1, 512, 300, 1000, 0, 0, 82), (F32, 64, 1, 512, 300, 1000, 0, 0, 82), (F16, 128, 1, 384, 300, 1000, 0, 0, 43)]


@pytest.mark.parametrize("dtype,d,n_q,l_q,docs,tokens,ragged,argmax,want", SIXTEEN)
def test_four_blocks_per_wavefront_on_few_long_documents(routes, dtype, d, n_q, l_q, docs, tokens, ragged, argmax, want):
    call = Call(dtype, d, n_q, l_q, docs, docs * tokens, ragged, argmax)
    assert routes([call])[0].shape == want, call


def test_fp32_and_narrow_rows_keep_three_blocks(routes):
    for dtype, d, l_q, docs, tokens, want in ((F32, 64, 300, 700, 64, 43), (F32, 32, 180, 3000, 300, 42), (F16, 64, 300, 700, 64, 82), (F16, 64, 300, 700, 65, 43),
                                             (F16, 64, 180, 768, 40, 23), (F16, 64, 180, 1500, 500, 23)):
        call = Call(dtype, d, 1, l_q, docs, docs * tokens, 0, 0)
        assert routes([call])[0].shape == want, call


# The same with many column groups, which fill the chip: large ones, whatever the estimate says (queries, tokens, documents, tokens)
@pytest.mark.parametrize("n_q,l_q,b,tokens,ragged,want", [(278, 496, 256, 28, 0, 8), (160, 399, 160, 62, 0, 8), (65, 412, 65, 36, 1, 8), (104, 238, 104, 19, 1, 8), (286, 55, 173, 67, 1, 8), (65, 458, 57, 88, 0, 8), (217, 210, 93, 17, 0, 8),
                                                          (57, 58, 195, 27, 0, 81), (32 * 32, 32, 48, 60, 0, 82), (32 * 32 + 1, 32, 48, 60, 0, 8)])
def test_many_column_groups_with_argmax(routes, n_q, l_q, b, tokens, ragged, want):
    for d in (64, 128):
        r, = routes([Call(BF16, d, n_q, l_q, b, b * tokens, ragged, 1)])
        assert r.kind == "tile" and r.shape == want


# n queries of l_q tokens on as many documents, winners wanted -> kernel and blocks (split) or shape (tile): small batches take a workgroup
# per document and one or two column blocks, then small column groups, large ones the groups that any other corpus takes
@pytest.mark.parametrize("n,l_q,tokens,ragged,want", [(16, 32, 128, 0, ("split", 1)), (16, 64, 500, 0, ("split", 2)), (33, 32, 208, 1, ("split", 1)), (50, 32, 1024, 0, ("tile", 43)),
                                                      (64, 32, 188, 1, ("tile", 81)), (128, 32, 500, 0, ("tile", 8)), (256, 32, 1024, 0, ("tile", 8)), (8, 300, 300, 0, ("tile", 43)),
                                                      (12, 256, 1030, 0, ("tile", 81)), (8, 1030, 300, 0, ("tile", 83))])
def test_few_documents_with_argmax(routes, n, l_q, tokens, ragged, want):
    call = Call(BF16, 128, n, l_q, n, n * tokens, ragged, 1)
    assert (routes([call])[0].kind, routes([call])[0].shape) == want, call
    assert routes([call._replace(dtype=F32, d=64)])[0].kind == routes([call._replace(argmax=0)])[0].kind == "tile"


@pytest.mark.parametrize("cus", [64, 256, 304])
def test_fp32_short_queries(routes, cus):
    """Wavefronts per document and documents per workgroup for fp32 rows of 512 bytes, by documents per CU: what launch_stream builds
    wherever there are no runs of documents."""
    def shape(l_q, b, tokens, ragged=0):
        r, = routes([Call(F32, 128, 1, l_q, b, b * tokens, ragged, 1)], cus)
        assert r.kind == "stream" or r.doc_waves
        assert (r.doc_waves, r.docs_per_wg) in ({(4, 1), (2, 1), (1, 1), (2, 2), (1, 4), (0, 1)} if l_q <= 32 else {(4, 1), (2, 1), (1, 1), (1, 2), (0, 1)})
        return r.doc_waves, r.docs_per_wg
    assert [shape(32, 2 * cus, t) for t in (32, 33, 96, 97)] == [(1, 1), (2, 1), (2, 1), (4, 1)]
    assert [shape(32, b, 128) for b in (2 * cus + 1, 3 * cus, 3 * cus + 1, 4 * cus, 4 * cus + 1, 6 * cus, 6 * cus + 1, 8 * cus, 8 * cus + 1, 10 * cus + 1, 64 * cus, 64 * cus + 1)] == [
        (1, 1), (1, 1), (1, 4), (1, 4), (2, 2), (2, 2), (1, 1), (1, 1), (2, 2), (1, 1), (1, 1), (0, 1)]
    assert [shape(32, 4 * cus + 1, t) for t in (96, 97)] == [(1, 1), (2, 2)]
    assert [shape(32, 4 * cus + 1, t, 1) for t in (160, 161)] == [(1, 1), (2, 2)]
    # two blocks: by themselves, two to a workgroup, in runs
    assert [shape(64, cus, t) for t in (20, 64, 300)] == [(1, 1), (2, 1), (4, 1)]
    assert [shape(64, b, 64) for b in (cus + 1, 2 * cus, 2 * cus + 1, 5 * cus, 5 * cus + 1, 6 * cus, 8 * cus)] == [(1, 2), (1, 2), (1, 1), (1, 1), (1, 2), (1, 2), (0, 1)]
    assert [shape(64, 2 * cus + x, t) for x, t in ((0, 300), (1, 300), (1, 128))] == [(1, 2), (0, 1), (0, 1)]
    assert [routes([Call(F16, 256, 1, 32, b, b * 64, 0, 1)], cus)[0].doc_waves for b in (2 * cus, 64 * cus + 1)] == [2, 0]


# two blocks of fp32: runs of documents where a SIMD's share of tiles is no smaller without them (by an eighth at least)
@pytest.mark.parametrize("b,tokens,ragged,waves", [(1536, 64, 0, 1), (2048, 64, 0, 0), (2200, 64, 0, 1), (1700, 100, 0, 0), (2000, 100, 0, 0), (4000, 40, 0, 0), (2200, 127, 0, 1), (8000, 32, 0, 0),
                                                   (8000, 20, 0, 1), (5000, 33, 0, 1), (5000, 90, 0, 1), (2000, 100, 1, 1), (3000, 60, 1, 1), (3000, 40, 1, 1)])
def test_fp32_two_blocks_in_runs(routes, b, tokens, ragged, waves):
    assert routes([Call(F32, 128, 1, 64, b, b * tokens, ragged, 1)])[0].doc_waves == waves


# without argmax always by themselves, up to 127 tokens
@pytest.mark.parametrize("b,tokens,ragged,waves", [(2048, 64, 0, 1), (2000, 100, 0, 1), (4000, 40, 0, 1), (3098, 34, 0, 1), (5000, 90, 0, 1), (1575, 120, 1, 1), (1575, 128, 0, 0), (64 * 256 + 1, 40, 0, 0)])
def test_fp32_two_blocks_without_argmax(routes, b, tokens, ragged, waves):
    assert routes([Call(F32, 128, 1, 64, b, b * tokens, ragged, 0)])[0].doc_waves == waves


def test_every_shape_is_reached_and_no_other(routes):
    """dispatch_tile and launch_stream instantiate exactly what forward_launch asks for."""
    calls = [Call(dt, row // (4 if dt == F32 else 2), n_q, l_q, b, b * t, ragged, am)
             for dt in (F32, F16) for row in (128, 256, 512) for am in (0, 1) for ragged in (0, 1)
             for n_q in (1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 16, 17, 24, 30, 64)
             for l_q in (1, 32, 33, 65, 97, 130, 190, 250, 300, 512, 600, 1024, 1030, 2100) for b in (1, 200, 768, 1800, 4096, 20000) for t in (20, 100, 300)]
    tile = collections.defaultdict(set)
    stream = collections.defaultdict(set)
    for c, r in zip(calls, routes(calls)):
        if r.kind == "tile":
            tile[c.dtype == F32, r.nu == 16, c.argmax].add(r.shape)
        elif r.kind != "slabs":
            stream[r.nu == 16].add((r.kind, r.shape, r.n_groups))
    for fp32 in (False, True):
        narrow = {82, 42, 83, 43, 4, 8} | (set() if fp32 else {23, 2})
        assert tile[fp32, False, 1] == narrow | {81}
        assert tile[fp32, False, 0] == narrow | {93, 94, 943, 944} | (set() if fp32 else {923, 924})
        assert tile[fp32, True, 0] == tile[fp32, True, 1] == {2, 4}
    assert stream[False] == {(kind, n, 1) for kind in ("split", "stream") for n in (1, 2, 3, 4)}
    assert stream[True] == {("split", 1, 1), ("stream", 1, 1), ("stream", 2, 1), ("stream", 2, 2), ("stream", 2, 4)}
