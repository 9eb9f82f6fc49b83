"""GPU parity of maxsim_forward / maxsim_forward_ragged against the CPU oracle (through the C ABI)."""
import numpy as np
import pytest
import torch

from paper_2605_29517_amd import binding as M
from paper_2605_29517_amd import workloads as W

from parity import RTOL_16, RTOL_F32, forward_parity_ragged, forward_parity_uniform

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_config1_tiny_fp32_with_argmax():
    Q, D = W.tiny_forward()
    worst = forward_parity_uniform(Q.to(DEV), D.to(DEV), M.maxsim_forward, True, RTOL_F32)
    print("config 1 max rel err %.2e" % worst)


# (n_q, l_q, b, l_d): streaming kernel (<= 4 column blocks), every tile-kernel width, ragged tails,
# single-token documents, one document, a query longer than one workgroup's 1024 tokens
SHAPES = [
    (1, 32, 37, 128), (1, 1, 5, 1), (1, 31, 9, 33), (2, 33, 11, 31), (4, 32, 50, 100), (1, 100, 20, 65),
    (3, 17, 1, 300), (8, 32, 40, 64), (5, 40, 13, 97), (16, 32, 70, 200), (2, 256, 9, 130),
    (64, 32, 33, 150), (1, 1024, 6, 260), (3, 700, 5, 95), (1, 1100, 4, 70), (2, 2100, 3, 40),
    # several wavefronts of the streaming kernel sharing a run of documents (2, 3 and 4 groups)
    (12, 32, 45, 130), (3, 64, 21, 77), (4, 96, 17, 140), (7, 50, 30, 33), (6, 1, 9, 5),
    # one long query of 5-16 blocks: tile kernel with one or two blocks per wavefront and a ring of tiles in flight
    (1, 200, 7, 90), (1, 256, 5, 64), (1, 300, 4, 100), (1, 512, 3, 70), (2, 160, 9, 45),
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_uniform_16bit(shape, want_argmax, dtype):
    n_q, l_q, b, l_d = shape
    Q = W.unit_rows((n_q, l_q, 128), dtype, 11 + l_q, DEV)
    D = W.unit_rows((b, l_d, 128), dtype, 12 + l_d, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, RTOL_16)


@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("shape", [(1, 32, 9, 40), (2, 32, 7, 33), (3, 32, 21, 100), (9, 20, 30, 70), (40, 32, 5, 64)])
def test_uniform_fp32(shape, want_argmax):
    n_q, l_q, b, l_d = shape
    Q = W.unit_rows((n_q, l_q, 128), "f32", 21, DEV)
    D = W.unit_rows((b, l_d, 128), "f32", 22, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, RTOL_F32)


# Column blocks that do not fill wavefronts of four: three per wavefront in workgroups of 8 (17-24 blocks), 4 (9-12) and 2
# wavefronts (5 and 6, 16-bit, from 768 documents of three tiles on), two passes of 24 blocks (33-48), even column groups.
# fp32 sums of at most 128 products (relative error about sqrt(128) 2^-24 = 7e-7), with 16-bit argmax maxima cut by 2^-19: 1e-5
# of the score; a query token lost or counted twice among 1536 is 6.5e-4 of it
THREES = [(1, 600, 5, 70), (3, 200, 6, 33), (1, 768, 3, 95), (1, 300, 7, 64), (6, 64, 9, 45), (1, 130, 800, 9), (2, 96, 770, 5),
          (1, 1030, 4, 70), (1, 1536, 3, 40), (5, 256, 6, 50), (7, 130, 4, 61), (2, 90, 770, 70), (5, 31, 771, 65), (1, 190, 769, 66)]


@pytest.mark.parametrize("dtype,d", [("f16", 128), ("bf16", 128), ("f32", 64), ("f16", 64), ("f32", 32)])
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("shape", THREES)
def test_blocks_in_threes(shape, want_argmax, dtype, d):
    n_q, l_q, b, l_d = shape
    Q = W.unit_rows((n_q, l_q, d), dtype, 13 + l_q, DEV)
    D = W.unit_rows((b, l_d, d), dtype, 14 + l_d, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, 1e-5)


def _ragged_case(n_q, l_q, lens, dtype, seed, d=128):
    lens = np.asarray(lens)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp = W.unit_rows((int(lens.sum()), d), dtype, seed, DEV)
    Q = W.unit_rows((n_q, l_q, d), dtype, seed + 1, DEV)
    return Q, Dp, off


# 13 to 16 blocks on a little more documents than CUs, of sixteen tiles and more: four wavefronts with four blocks each (16-bit)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n_q,l_q,l_d", [(1, 400, 512), (4, 128, 513), (16, 32, 545), (13, 20, 530)])
def test_sixteen_blocks_on_few_long_documents(n_q, l_q, l_d, dtype):
    b = torch.cuda.get_device_properties(0).multi_processor_count + 3
    Q = W.unit_rows((n_q, l_q, 128), dtype, 23 + l_q, DEV)
    D = W.unit_rows((b, l_d, 128), dtype, 24 + l_d, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, False, 1e-5)  # (the bound: see THREES)


# The same on ragged corpora with empty documents at both ends and in between; five and six blocks with more than four
# documents per CU, which take two wavefronts with three blocks each (16-bit)
@pytest.mark.parametrize("dtype,d", [("f16", 128), ("bf16", 64), ("f32", 64), ("f32", 32)])
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("n_q,l_q", [(1, 600), (3, 200), (1, 300), (6, 64), (1, 1030), (5, 256), (1, 190), (5, 32), (2, 96)])
def test_blocks_in_threes_ragged(n_q, l_q, want_argmax, dtype, d):
    lens = [0, 0, 1, 31, 32, 33, 0, 64, 0, 0, 70, 97, 2, 300, 0]
    if n_q * ((l_q + 31) // 32) <= 6:
        n = torch.cuda.get_device_properties(0).multi_processor_count * 4
        lens += list(np.random.default_rng(l_q).integers(0, 70, n)) + [0]
    Q, Dp, off = _ragged_case(n_q, l_q, lens, dtype, 17 + l_q, d)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, want_argmax, 1e-5)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("n_q,l_q", [(1, 32), (3, 32), (5, 32), (8, 30), (3, 40), (7, 33), (64, 32), (2, 300)])
def test_ragged_edge_lengths(n_q, l_q, want_argmax, dtype):
    lens = [1, 31, 32, 33, 0, 64, 300, 0, 0, 2, 65, 128, 1, 97]
    Q, Dp, off = _ragged_case(n_q, l_q, lens, dtype, 31)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, want_argmax, RTOL_F32 if dtype == "f32" else RTOL_16)


@pytest.mark.parametrize("n_q", [1, 4, 6, 64])
def test_ragged_colbert_like(n_q):
    Q, Dp, off, _ = W.colbert_rerank(n_q=n_q, n_docs=700, device=DEV)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, n_q == 4, RTOL_16)


def test_leading_and_trailing_empty_documents():
    Q, Dp, off = _ragged_case(2, 32, [0, 0, 5, 0, 40, 0, 0], "f16", 41)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, True, RTOL_16)


def test_duplicate_tokens_keep_first_index():
    """Exact ties: the lowest index wins ("Tied maxima"), also across tiles and lane halves."""
    Q = W.unit_rows((1, 32, 128), "f16", 51, DEV)
    base = W.unit_rows((1, 5, 128), "f16", 52, DEV)
    D = base.repeat(1, 20, 1).contiguous()  # 100 tokens, every token repeated 20 times, period 5
    s, a = M.maxsim_forward(Q, D, want_argmax=True)
    torch.cuda.synchronize()
    assert int(a.max()) < 5
    s1, a1 = M.maxsim_forward(Q, base.contiguous(), want_argmax=True)
    torch.cuda.synchronize()
    assert torch.equal(a, a1) and torch.equal(s, s1)


# Exact ties on the tile kernel: a document of equal rows `period` apart, so that they lie in other quarters (4) and halves (16)
# of a tile, a register on (1: all rows equal, 5, 17), in the same place of a later tile (32) and in the repeated rows past the end.
# fp32 (16x16 results) with two, three and four blocks per wavefront and 512-byte rows, 16-bit (32x32 results) likewise
@pytest.mark.parametrize("dtype,d,n_q,l_q", [("f32", 64, 1, 300), ("f32", 64, 1, 640), ("f32", 64, 1, 1030), ("f32", 32, 3, 100), ("f32", 64, 6, 32),
                                             ("f32", 64, 1, 1024), ("f32", 128, 1, 200), ("f16", 128, 1, 300), ("f16", 128, 1, 640), ("bf16", 128, 1, 1024),
                                             ("f16", 128, 6, 32), ("bf16", 64, 1, 200), ("f16", 256, 1, 200)])
@pytest.mark.parametrize("period", [1, 4, 5, 16, 17, 32])
def test_ties_keep_the_first_row_on_the_tile_kernel(period, dtype, d, n_q, l_q):
    Q = W.unit_rows((n_q, l_q, d), dtype, 53, DEV)
    for l_d in (37, 64, 100):
        base = W.unit_rows((3, min(period, l_d), d), dtype, 54 + l_d, DEV)
        D = base.repeat(1, -(-l_d // period), 1)[:, :l_d].contiguous()
        _, a = M.maxsim_forward(Q, D, want_argmax=True)
        torch.cuda.synchronize()
        s = torch.einsum("qid,bjd->qbij", Q.double().cpu(), base.double().cpu())
        top = s.topk(min(2, base.shape[1]), dim=-1)
        clear = (top.values[..., 0] - top.values[..., -1] > 1e-3) | (base.shape[1] == 1)
        assert clear.float().mean() > 0.9
        assert torch.equal(a.cpu()[clear], top.indices[..., 0][clear].int())


# Similarities that are negative throughout, partly, or shifted per document (token rows of real encoders share a
# mean direction): the argmax fold of the tile kernel orders cells through their bit patterns, which is only right
# among non-negative values, and falls back to compare-and-select while a running maximum is negative.
# (n_q, l_q, b, l_d): tile kernel with 4, 2 and 1 blocks per wavefront; streaming kernel; ragged
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape", [(40, 32, 6, 200), (2, 256, 5, 130), (1, 1024, 3, 100), (1, 200, 4, 90), (2, 32, 9, 70)])
@pytest.mark.parametrize("q_bias,d_bias", [(1.0, -1.0), (0.6, 0.6), (0.4, -0.2)])
def test_argmax_with_negative_and_shifted_similarities(shape, q_bias, d_bias, dtype):
    n_q, l_q, b, l_d = shape
    Q = W.biased_rows((n_q, l_q, 128), dtype, 61, DEV, bias=q_bias)
    D = W.biased_rows((b, l_d, 128), dtype, 62, DEV, bias=d_bias)
    D[b // 2:] = W.biased_rows((b - b // 2, l_d, 128), dtype, 63, DEV, bias=-d_bias)   # half of the documents the other way
    rtol = RTOL_F32 if dtype == "f32" else RTOL_16
    forward_parity_uniform(Q, D.contiguous(), M.maxsim_forward, True, rtol)
    lens = np.array([l_d, 1, 33, 0, l_d // 2, 70])
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp = W.biased_rows((int(lens.sum()), 128), dtype, 64, DEV, bias=d_bias)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, True, rtol)


# Rows that are not unit-norm (the ABI does not ask for it): similarities of 1e-6 and of 1e+6
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("scale", [1e-3, 30.0, 1e3])
@pytest.mark.parametrize("shape", [(40, 32, 6, 200), (1, 32, 20, 100), (3, 300, 4, 70)])
def test_rows_that_are_not_unit_norm(shape, scale, want_argmax, dtype):
    if dtype == "f16" and scale > 100:
        pytest.skip("fp16 cannot hold rows of that magnitude times each other")
    n_q, l_q, b, l_d = shape
    Q = W.biased_rows((n_q, l_q, 128), dtype, 71, DEV, bias=0.3, scale=scale)
    D = W.biased_rows((b, l_d, 128), dtype, 72, DEV, bias=-0.1, scale=scale)
    # the absolute slack for scores that sit at zero scales with the similarities (scale^2)
    forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, RTOL_F32 if dtype == "f32" else RTOL_16,
                           atol_per_token=1e-6 * scale * scale)


def test_argument_errors():
    Q = W.unit_rows((1, 32, 128), "f16", 1, DEV)
    D = W.unit_rows((4, 40, 128), "f16", 2, DEV)
    with pytest.raises(M.MaxSimError):
        M.maxsim_forward(Q.cpu(), D)
    with pytest.raises(M.MaxSimError):
        M.maxsim_forward(Q[..., :100].contiguous(), D[..., :100].contiguous())  # rows of 200 bytes: not a multiple of 64
    L = M.load()
    assert L.maxsim_forward(None, 1, 32, None, 4, 40, 128, 1, None, None, None) == -1


# Other embedding widths (rows of 128, 512 and 1024 bytes): stream and tile kernels, several passes, ragged, argmax
WIDTH_SHAPES = [(1, 32, 9, 40), (3, 17, 5, 100), (8, 32, 12, 65), (2, 200, 6, 130), (1, 1030, 3, 70), (40, 32, 7, 33)]


@pytest.mark.parametrize("dtype,d", [("f16", 64), ("f16", 256), ("f16", 512), ("bf16", 64), ("bf16", 256), ("bf16", 512),
                                     ("f32", 32), ("f32", 64), ("f32", 256)])
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("shape", WIDTH_SHAPES)
def test_uniform_other_widths(shape, want_argmax, dtype, d):
    n_q, l_q, b, l_d = shape
    Q = W.unit_rows((n_q, l_q, d), dtype, 61 + l_q, DEV)
    D = W.unit_rows((b, l_d, d), dtype, 62 + l_d, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, RTOL_F32 if dtype == "f32" else RTOL_16)


@pytest.mark.parametrize("dtype,d", [("f16", 64), ("bf16", 256), ("f16", 512), ("f32", 256)])
@pytest.mark.parametrize("n_q,l_q", [(1, 32), (5, 40), (2, 300)])
def test_ragged_other_widths(n_q, l_q, dtype, d):
    lens = np.asarray([1, 31, 32, 33, 0, 64, 150, 0, 2, 65, 97])
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp = W.unit_rows((int(lens.sum()), d), dtype, 71, DEV)
    Q = W.unit_rows((n_q, l_q, d), dtype, 72, DEV)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, True, RTOL_F32 if dtype == "f32" else RTOL_16)


# Widths without a register-stationary kernel go through the slab-streaming ("split-d") kernel: rows that are any
# multiple of 64 bytes.  Shapes: one block, ragged column tail, more than one group of 16 blocks (several queries),
# a query of more than 16 blocks (two passes), documents shorter and longer than a macro tile of 128 tokens.
SPLITD_SHAPES = [(1, 32, 9, 40), (3, 17, 5, 300), (8, 32, 12, 65), (2, 200, 6, 130), (1, 1030, 3, 70), (40, 32, 7, 33),
                 (3, 600, 4, 257)]
SPLITD_WIDTHS = [("f16", 32), ("f16", 96), ("bf16", 160), ("f16", 384), ("bf16", 768), ("f16", 1024), ("bf16", 2048),
                 ("f32", 48), ("f32", 80), ("f32", 512)]


@pytest.mark.parametrize("dtype,d", SPLITD_WIDTHS)
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("shape", SPLITD_SHAPES)
def test_uniform_split_d(shape, want_argmax, dtype, d):
    n_q, l_q, b, l_d = shape
    Q = W.unit_rows((n_q, l_q, d), dtype, 81 + l_q, DEV)
    D = W.unit_rows((b, l_d, d), dtype, 82 + l_d, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, RTOL_F32 if dtype == "f32" else RTOL_16)


@pytest.mark.parametrize("dtype,d", [("f16", 96), ("bf16", 768), ("f16", 1024), ("f32", 48)])
@pytest.mark.parametrize("n_q,l_q", [(1, 32), (5, 40), (2, 300), (1, 700)])
def test_ragged_split_d(n_q, l_q, dtype, d):
    lens = np.asarray([1, 31, 32, 33, 0, 64, 150, 0, 2, 65, 97, 128, 129, 300])
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp = W.unit_rows((int(lens.sum()), d), dtype, 91, DEV)
    Q = W.unit_rows((n_q, l_q, d), dtype, 92, DEV)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, True, RTOL_F32 if dtype == "f32" else RTOL_16)


# Chunk counts that are no multiple of the 8 XCDs, one and several rounds of workgroups, fewer documents than chunks asked for
@pytest.mark.parametrize("n_q,l_q,b,l_d", [(20, 300, 60, 33), (3, 700, 37, 40), (33, 32, 301, 20), (1, 130, 509, 64), (2, 1100, 11, 70)])
def test_chunk_counts(n_q, l_q, b, l_d):
    Q = W.unit_rows((n_q, l_q, 128), "f16", 66, DEV)
    forward_parity_uniform(Q, W.unit_rows((b, l_d, 128), "f16", 67, DEV), M.maxsim_forward, True, RTOL_16)
    lens = np.random.default_rng(b).integers(0, 2 * l_d, b)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    forward_parity_ragged(Q, W.unit_rows((int(lens.sum()), 128), "f16", 68, DEV), off, M.maxsim_forward_ragged, False, RTOL_16)


# The wide kernel's shapes: by column blocks of a workgroup (1, 2, 4, 6, 8; one query of 9 and of 19 blocks in several
# passes; groups of unequal numbers of queries) and by the documents' length (macro tiles of 64, 128 and 256 rows: one
# row either side of them, a single tile, several); widths of two and several slabs of 128 bytes (one: test_wide_one_slab), with and without a half one.
# fp32 accumulation of at most 384 products and sums of at most 600 maxima: 1e-5 relative to the score
@pytest.mark.parametrize("n_q,l_q", [(1, 30), (2, 32), (3, 40), (3, 60), (1, 256), (5, 50), (1, 270), (1, 600)])
@pytest.mark.parametrize("l_d", [1, 32, 64, 65, 128, 129, 255, 256, 257, 545])
def test_wide_shapes(l_d, n_q, l_q):
    for dtype, d, want_argmax in (("f16", 160, False), ("bf16", 384, True), ("f32", 48, True)):
        Q = W.unit_rows((n_q, l_q, d), dtype, 61 + l_q, DEV)
        D = W.unit_rows((5, l_d, d), dtype, 62 + l_d, DEV)
        forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, 1e-5)


@pytest.mark.parametrize("n_q,l_q", [(1, 20), (2, 130), (1, 300)])
def test_wide_many_documents(n_q, l_q):
    """More documents than workgroups, ragged and uniform: a workgroup goes from one document to the next."""
    n = torch.cuda.get_device_properties(0).multi_processor_count * 2 + 7
    lens = np.random.default_rng(l_q).integers(0, 300, n)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp = W.unit_rows((int(lens.sum()), 96), "f16", 63, DEV)
    Q = W.unit_rows((n_q, l_q, 96), "f16", 64, DEV)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, True, 1e-5)
    forward_parity_uniform(Q, W.unit_rows((n, 70, 96), "f16", 65, DEV), M.maxsim_forward, False, 1e-5)


# Without argmax the wide kernel's results are 16x16: every shape, several ragged documents per workgroup with empty ones among them,
# widths of one and a half, two and four and a half slabs
@pytest.mark.parametrize("dtype,d", [("f16", 96), ("bf16", 128 + 128), ("bf16", 288)])
@pytest.mark.parametrize("longest", [40, 120, 600])
@pytest.mark.parametrize("n_q,l_q", [(1, 16), (2, 33), (3, 60), (8, 31), (1, 257), (1, 600)])
def test_wide_16x16_results(n_q, l_q, longest, dtype, d):
    n = torch.cuda.get_device_properties(0).multi_processor_count + 9
    lens = np.random.default_rng(longest + l_q).integers(0, longest, n)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Q = W.unit_rows((n_q, l_q, d), dtype, 64, DEV)
    forward_parity_ragged(Q, W.unit_rows((int(lens.sum()), d), dtype, 63, DEV), off, M.maxsim_forward_ragged, False, 1e-5)


# fp32 rows of 512 bytes, one or two column blocks: one, two and four wavefronts per document and block, documents of fewer tiles than
# wavefronts, of a single row, empty ones; two queries of one block and one of two
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("n_q,l_q", [(1, 32), (1, 7), (2, 20), (1, 33), (1, 64)])
@pytest.mark.parametrize("b,longest", [(3, 300), (40, 130), (200, 33), (300, 70), (700, 30), (600, 150)])
def test_fp32_short_queries(b, longest, n_q, l_q, want_argmax):
    lens = np.random.default_rng(b + l_q).integers(0, longest + 1, b)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Q = W.unit_rows((n_q, l_q, 128), "f32", 64, DEV)
    forward_parity_ragged(Q, W.unit_rows((int(lens.sum()), 128), "f32", 63, DEV), off, M.maxsim_forward_ragged, want_argmax, RTOL_F32)
    forward_parity_uniform(Q, W.unit_rows((b, longest, 128), "f32", 65, DEV), M.maxsim_forward, want_argmax, RTOL_F32)


# The same with two or four documents to a workgroup, the last of which is not full (three to six documents per CU of 256)
@pytest.mark.parametrize("want_argmax", [False, True])
@pytest.mark.parametrize("n_q,l_q", [(1, 32), (1, 7), (2, 20), (1, 64)])
@pytest.mark.parametrize("b,longest", [(301, 70), (769, 130), (1023, 33), (1027, 130), (1027, 400), (1301, 40)])
def test_fp32_short_queries_documents_to_a_workgroup(b, longest, n_q, l_q, want_argmax):
    test_fp32_short_queries(b, longest, n_q, l_q, want_argmax)


# Many queries on few documents with winners: a workgroup of one, two or four wavefronts per document and one or two column blocks, or
# small column groups of the tile kernel; a last group that is not full, documents of fewer tiles than wavefronts, empty ones
@pytest.mark.parametrize("dtype,d", [("f16", 128), ("bf16", 64)])
@pytest.mark.parametrize("n_q,l_q,b,longest", [(16, 32, 16, 129), (17, 20, 3, 1000), (5, 64, 9, 400), (16, 50, 5, 33), (33, 32, 33, 333), (50, 17, 41, 100), (61, 32, 70, 60),
                                               (23, 40, 90, 200), (9, 300, 8, 200), (7, 250, 13, 500), (90, 24, 80, 277)])
def test_many_queries_on_few_documents(n_q, l_q, b, longest, dtype, d):
    lens = np.random.default_rng(longest + l_q).integers(0, longest + 1, b)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Q = W.unit_rows((n_q, l_q, d), dtype, 64, DEV)
    forward_parity_ragged(Q, W.unit_rows((int(lens.sum()), d), dtype, 63, DEV), off, M.maxsim_forward_ragged, True, RTOL_16)
    forward_parity_uniform(Q, W.unit_rows((b, longest, d), dtype, 65, DEV), M.maxsim_forward, True, RTOL_16)


# Rows of a single slab (d = 32 in 16 bits): one barrier per macro tile, so that with short documents the loads run up to three
# documents ahead and the merge and the sum of one document fall into the next two.  Several documents per workgroup, a few of
# them empty, in the shapes for 1 to 8 column blocks and for every height of the macro tiles
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("longest", [40, 200, 600])
@pytest.mark.parametrize("n_q,l_q", [(1, 20), (2, 30), (2, 40), (3, 60), (7, 32), (8, 32), (1, 300)])
def test_wide_one_slab(n_q, l_q, longest, dtype):
    n = torch.cuda.get_device_properties(0).multi_processor_count * (8 if longest < 100 else 3) + 7
    lens = np.random.default_rng(longest + l_q).integers(0, longest, n)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Q = W.unit_rows((n_q, l_q, 32), dtype, 64, DEV)
    forward_parity_ragged(Q, W.unit_rows((int(lens.sum()), 32), dtype, 63, DEV), off, M.maxsim_forward_ragged, True, 1e-5)
    forward_parity_uniform(Q, W.unit_rows((n, longest // 2 + 1, 32), dtype, 65, DEV), M.maxsim_forward, True, 1e-5)


# Ragged corpora scored by more than 16 queries of one column block take 32-row windows over the packed rows (a window
# may hold the end of one document and the start of the next).  Length mixes: runs of tiny documents (several
# boundaries close together, a document that lies inside one window whole), empty documents at the start, in a row
# and at the end, lengths around the window size, and long documents.
PACK_LENGTHS = {
    "tiny": [1, 1, 1, 2, 1, 3, 1, 1, 5, 1, 1, 1, 40, 1, 1],
    "empties": [0, 0, 7, 0, 33, 0, 0, 0, 31, 1, 0, 64, 0],
    "window": [32, 32, 31, 33, 1, 63, 64, 65, 32, 16, 16, 16, 16],
    "long": [300, 64, 129, 5, 700, 31, 257],
}


@pytest.mark.parametrize("dtype,d", [("f16", 128), ("bf16", 128), ("f16", 64), ("f32", 64), ("f32", 32)])
@pytest.mark.parametrize("n_q,l_q", [(5, 32), (6, 9), (7, 32), (8, 31), (9, 32), (10, 32), (12, 7), (13, 32), (16, 32), (17, 32), (40, 20), (64, 32), (33, 1)])
@pytest.mark.parametrize("mix", sorted(PACK_LENGTHS))
def test_ragged_packed_windows(mix, n_q, l_q, dtype, d):
    lens = np.asarray(PACK_LENGTHS[mix] * 3)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp = W.unit_rows((int(lens.sum()), d), dtype, 101, DEV)
    Q = W.unit_rows((n_q, l_q, d), dtype, 102, DEV)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, False, RTOL_F32 if dtype == "f32" else RTOL_16)


@pytest.mark.parametrize("n_q", [6, 8, 11, 48])
def test_ragged_packed_windows_many_chunks(n_q):
    # enough documents that every workgroup gets its own chunk, with chunk borders inside runs of short documents
    # (workgroups of two, four and eight wavefronts)
    rng = np.random.default_rng(7)
    lens = rng.integers(0, 90, size=6000)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp = W.unit_rows((int(lens.sum()), 128), "f16", 103, DEV)
    Q = W.unit_rows((n_q, 32, 128), "f16", 104, DEV)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, False, RTOL_16)


@pytest.mark.parametrize("dtype,d", [("f16", 128), ("bf16", 64)])
@pytest.mark.parametrize("n_q,l_q", [(5, 32), (8, 32), (11, 32), (14, 3), (17, 32), (64, 20)])
@pytest.mark.parametrize("b,l_d", [(50, 1), (33, 7), (21, 33), (40, 100), (9, 300), (700, 45), (30, 64), (12, 256), (3000, 32)])
def test_uniform_packed_windows(b, l_d, n_q, l_q, dtype, d):
    """Uniform corpora whose documents are not a whole number of 32-row tiles take the packed windows as well, and so
    do corpora of whole tiles at 5-16 queries."""
    Q = W.unit_rows((n_q, l_q, d), dtype, 111, DEV)
    D = W.unit_rows((b, l_d, d), dtype, 112, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, False, RTOL_16)


# Five to sixteen column blocks on a corpus of thousands of documents: the workgroups of two and four wavefronts with
# three (five, six and nine to twelve blocks) or four blocks each (tile kernel: argmax or queries of several blocks; packed
# windows otherwise), uniform and ragged.  1e-5: see THREES
@pytest.mark.parametrize("dtype,d", [("f16", 128), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("n_q,l_q,want_argmax", [(1, 200, False), (1, 256, True), (3, 130, True), (2, 250, False), (7, 32, True),
                                                 (12, 32, True), (6, 32, False), (14, 20, False), (1, 130, False), (1, 190, False), (5, 32, True),
                                                 (2, 96, False), (2, 96, True), (1, 190, True)])
@pytest.mark.parametrize("ragged", [False, True])
def test_mid_block_counts_on_many_documents(ragged, n_q, l_q, want_argmax, dtype, d):
    b = 4500
    rtol = 1e-5
    Q = W.unit_rows((n_q, l_q, d), dtype, 131, DEV)
    if ragged:
        lens = np.random.default_rng(n_q * 1000 + l_q).integers(0, 50, size=b)
        lens[:3] = [0, 33, 1]
        off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
        Dp = W.unit_rows((int(lens.sum()), d), dtype, 132, DEV)
        forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, want_argmax, rtol)
    else:
        D = W.unit_rows((b, 32 if l_q > 100 else 40, d), dtype, 132, DEV)
        forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, rtol)


# Small corpora take a workgroup per document, whose two wavefronts share its tiles: documents of one to five tiles
# (an empty second wavefront, uneven shares, ragged ends), every number of column blocks, more documents than
# workgroups; fp32 accumulation of 128 products and a sum of at most 128 maxima: 1e-5 relative
@pytest.mark.parametrize("dtype,n_q,l_q", [("f16", 1, 32), ("bf16", 2, 30), ("f16", 1, 90), ("bf16", 4, 32), ("f32", 1, 17)])
@pytest.mark.parametrize("want_argmax", [False, True])
def test_a_workgroup_per_document(dtype, n_q, l_q, want_argmax):
    lens = [64, 65, 1, 32, 33, 0, 95, 96, 97, 128, 129, 160, 2, 300] * 2 + [70] * 3
    Q, Dp, off = _ragged_case(n_q, l_q, lens, dtype, 71)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, want_argmax, 1e-5)
    for b, l_d in ((3, 64), (5, 100), (1, 1000)):
        D = W.unit_rows((b, l_d, 128), dtype, 72 + b, DEV)
        forward_parity_uniform(Q, D, M.maxsim_forward, want_argmax, 1e-5)


def test_more_documents_than_workgroups():
    n = torch.cuda.get_device_properties(0).multi_processor_count * 4 + 13
    Q, D = W.unit_rows((2, 32, 128), "f16", 81, DEV), W.unit_rows((n, 66, 128), "f16", 82, DEV)
    forward_parity_uniform(Q, D, M.maxsim_forward, True, 1e-5)


@pytest.mark.parametrize("b", [1, 2, 62, 63, 64, 65, 128, 4094, 4095, 4096, 4160])
def test_runs_of_documents_are_found(b):
    """Where a run of a ragged corpus begins is searched for with 64 probes a step: numbers of documents around the powers of 64."""
    lens = np.random.default_rng(b).integers(0, 4, b)
    lens[b // 2] = 40
    Q, Dp, off = _ragged_case(1, 8, lens, "f16", 91)
    forward_parity_ragged(Q, Dp, off, M.maxsim_forward_ragged, False, 1e-5)


@pytest.mark.parametrize("n_q", [6, 8, 15, 24])
@pytest.mark.parametrize("dtype,d", [("f16", 128), ("bf16", 64)])
def test_corpora_larger_than_the_last_cache(n_q, dtype, d):
    """Above 256 MB the windows of five to 32 queries are read with another hint: the documents at both ends against the oracle,
    all of them against the kernel for four queries (fp32 accumulation of 128 products, sums of 32 maxima: 1e-5 relative)."""
    rows = (256 << 20) // (2 * d) + 5000
    lens = np.random.default_rng(n_q).integers(0, 300, 2 * rows // 290)
    lens = lens[:np.searchsorted(np.cumsum(lens), rows) + 1]
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(DEV)
    Dp, Q = W.unit_rows((int(lens.sum()), d), dtype, 141, DEV), W.unit_rows((n_q, 32, d), dtype, 142, DEV)
    s = M.maxsim_forward_ragged(Q, Dp, off)
    few = torch.cat([M.maxsim_forward_ragged(Q[i:i + 4].contiguous(), Dp, off) for i in range(0, n_q, 4)])
    assert torch.equal(torch.isinf(s), torch.isinf(few))
    assert torch.allclose(s, few, rtol=1e-5)
    for a, b in ((0, 40), (len(lens) - 40, len(lens))):
        part, po = Dp[off[a]:off[b]].contiguous(), (off[a:b + 1] - off[a]).contiguous()
        forward_parity_ragged(Q, part, po, lambda q, dd, o, want_argmax: s[:, a:b], False, 1e-5)
    l_d = 190
    D = Dp[:rows // l_d * l_d].view(-1, l_d, d)
    assert D.numel() * 2 > 256 << 20
    s = M.maxsim_forward(Q, D)
    few = torch.cat([M.maxsim_forward(Q[i:i + 4].contiguous(), D) for i in range(0, n_q, 4)])
    assert torch.allclose(s, few, rtol=1e-5)
