"""Sizes at which the kernels chosen by size change over: edges of tiles and blocks, remainders, the smallest and the
largest of each kernel's range.  The comparisons are those of the tests that are called."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import test_gpu_attend as A
from tests import test_gpu_parity as T
from tests import test_gpu_split as S

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")


@pytest.mark.parametrize("bits,n,kind", [(2, 1, "bf16"), (3, 15, "f32"), (0, 16, "unit"), (4, 17, "bf16unit"), (1, 4095, "f32"),
                                         (2, 4096, "bf16"), (3, 4097, "f32")])
def test_small_batches_at_128(bits, n, kind):
    """Blocks of 16 vectors up to 4096 vectors."""
    T.test_quantize_prod(128, bits, n, kind)
    if bits:
        T.test_quantize_mse(128, bits, n, kind)


@pytest.mark.parametrize("d,bits,n,kind", [(512, 2, 1, "bf16"), (544, 3, 1, "f32"), (4096, 1, 1, "bf16unit"), (1568, 4, 2, "bf16"),
                                          (1024, 1, 13, "f32"), (544, 2, 64, "bf16")])
def test_long_vectors_decided_where_they_are_multiplied(d, bits, n, kind):
    """One vector, four at a time with 8 and with 16 rows per workgroup; row lengths that are no multiple of 256."""
    T.test_quantize_a_handful_of_long_vectors(d, bits, n, kind)
    T.test_quantize_prod_of_a_handful_of_long_vectors(d, bits, n, kind)


@pytest.mark.parametrize("d_hi,bits_lo,prod,n,bf16", [(32, 1, True, 1, True), (64, 2, False, 17, False), (96, 0, True, 4096, True),
                                                      (32, 3, False, 4097, True)])
def test_small_split_batches(d_hi, bits_lo, prod, n, bf16):
    S.test_quantize_split(d_hi, bits_lo, prod, n, bf16)


@pytest.mark.parametrize("vb,vprod,groups,qpg,npg", [(2, False, 1, 4, 511), (4, False, 2, 1, 512), (1, True, 1, 5, 513), (3, False, 1, 16, 1),
                                                     (2, False, 128, 1, 2048), (2, False, 128, 1, 2049)])
def test_attend_chunks(vb, vprod, groups, qpg, npg):
    """Workgroups of 512 keys while those of 2048 would leave half of the chip idle; the last two lie on either side."""
    A.run_attend(128, 2, True, vb, vprod, groups, qpg, npg, True)


@pytest.mark.parametrize("d_hi,vbits_lo,npg", [(64, 2, 512), (96, 1, 513)])
def test_attend_chunks_of_split_values(d_hi, vbits_lo, npg):
    S.test_attend_with_values_in_two_instances(d_hi, vbits_lo, 0, 2, 4, npg)


@pytest.mark.parametrize("d,bits,prod,groups,qpg,npg,topk", [
    (256, 4, True, 1, 1, 1, 1), (384, 1, False, 2, 2, 255, 0), (640, 2, True, 1, 3, 257, 3), (896, 4, False, 1, 4, 1025, 0),
    (3072, 1, True, 1, 5, 513, 10), (1536, 3, True, 3, 7, 63, 0), (4096, 0, True, 1, 8, 130, 2), (512, 2, True, 1, 2, 20000, 5),
])
def test_few_queries_at_multiples_of_128(d, bits, prod, groups, qpg, npg, topk):
    T.test_score_and_topk(d, bits, prod, groups, qpg, npg, topk)


@pytest.mark.parametrize("npg,topk", [(8191, 64), (8192, 1), (8193, 16), (16385, 33), (65, 64)])
def test_topk_segments(npg, topk):
    """Segments of a row, with equal scores on both sides of their edges and scores that are not numbers."""
    p = T.setup(128, 2, False)[0]
    c = T._random_codes(p, 128, 2, False, npg, npg)
    c["norm"][npg // 2:npg // 2 + 40] = 90.0
    c["idx"][npg // 2:npg // 2 + 40] = c["idx"][0]
    c["norm"][max(0, npg - 3):] = 90.0
    T._topk_both_ways(p, T.dev(W.gaussian_queries(3, 128, 5, unit=False)), 1, 3, c, npg, topk)
    c["norm"][5] = float("nan")
    q = T.dev(W.gaussian_queries(3, 128, 5, unit=False))
    scores = torch.zeros((3, npg), device=T.DEV)
    tq.tq_score(p, q, 1, 3, c["idx"], None, None, c["norm"], npg, scores)
    ti = torch.zeros((3, topk), dtype=torch.int32, device=T.DEV)
    tq.tq_score(p, q, 1, 3, c["idx"], None, None, c["norm"], npg, None, topk, ti, None)
    s = scores.cpu().numpy()
    assert np.isnan(s[:, 5]).all() and np.isnan(s).sum() == 3
    s[:, 5] = -np.inf  # never taken: every row has topk others
    assert np.array_equal(ti.cpu().numpy(), np.argsort(-s, axis=1, kind="stable")[:, :topk])


@pytest.mark.parametrize("d,bits,n,prod", [
    (32, 2, 1, True), (64, 3, 257, True), (64, 1, 256, False), (96, 4, 63, True), (160, 0, 129, True), (384, 2, 3001, False),
    (512, 3, 700, True), (640, 1, 65, False), (1024, 4, 255, True), (768, 2, 6000, True), (1536, 1, 9000, False), (544, 3, 4097, True),
])
def test_dequantiser_tiles(d, bits, n, prod):
    """Every tile and depth of buffers; with the matrices' images, and with images built for the call in the workspace."""
    T.test_dequantize(d, bits, n, prod, True)
    p = T.setup(d, bits, prod)[0]
    keep = (p.workspace, p.c.workspace, p.c.workspace_bytes)
    try:
        p.drop_images().reserve(n)
        T.test_dequantize(d, bits, n, prod, False)
        p.workspace, p.c.workspace, p.c.workspace_bytes = None, 0, 0
        T.test_dequantize(d, bits, n, prod, False)
    finally:
        p.workspace, p.c.workspace, p.c.workspace_bytes = keep
        p.build_images()


@pytest.mark.parametrize("d,bits,n,kind", [(512, 2, 65, "f32"), (512, 1, 16384, "bf16"), (256, 3, 16385, "f32"), (768, 4, 129, "unit"),
                                           (1024, 0, 1025, "bf16"), (640, 2, 2600, "f32"), (3072, 1, 66, "f32")])
def test_quantiser_tiles(d, bits, n, kind):
    """The small tiles' four buffers, and either side of the line between the two contractions."""
    T.test_quantize_prod(d, bits, n, kind)
    if bits:
        T.test_quantize_mse(d, bits, n, kind)


@pytest.mark.parametrize("d,bits,prod,nq,n,topk", [
    (128, 4, False, 17, 8191, 10), (128, 4, False, 17, 8192, 10), (128, 3, True, 33, 8193, 1), (256, 2, False, 65, 20000, 16),
    (384, 0, True, 129, 9001, 5), (512, 1, True, 257, 30001, 64), (640, 3, False, 130, 40000, 64), (1536, 4, False, 64, 12000, 2),
    (4096, 1, True, 20, 8200, 3), (128, 1, False, 32, 70001, 10),
])
def test_search_by_candidates(d, bits, prod, nq, n, topk):
    """Top-k alone, by candidates and their exact scores: the same indices and bits as from the score matrix."""
    p = T.setup(d, bits, prod)[0]
    c = T._random_codes(p, d, bits, prod, n, d + n)
    T._topk_both_ways(p, T.dev(W.gaussian_queries(nq, d, 3, unit=False)), 1, nq, c, n, topk)


@pytest.mark.parametrize("d,bits,prod,nq,n,topk", [
    (1152, 1, False, 32, 140033, 10), (128, 2, False, 97, 140033, 3), (256, 3, True, 96, 8321, 64), (384, 4, True, 128, 9999, 16),
    (128, 4, True, 40, 66000, 64), (512, 0, True, 64, 16385, 1), (2048, 2, True, 145, 8192, 7), (3072, 1, False, 129, 10001, 10),
    (256, 2, True, 641, 23041, 5),
])
def test_search_by_candidates_few_queries(d, bits, prod, nq, n, topk):
    """The kernel for few queries: one to four blocks of 32 of them, long codes, numbers of query blocks that do not divide the chip.  (Up to 32
    queries come to it beyond d = 1024 only.)"""
    test_search_by_candidates(d, bits, prod, nq, n, topk)


# more queries than compute units, on either side of the lengths of which four workgroups that rank find room in a compute unit's LDS
@pytest.mark.parametrize("d,bits,prod,n,topk", [(1664, 4, False, 8300, 5), (1792, 4, False, 8300, 5), (768, 3, True, 8300, 64), (896, 3, True, 8300, 64),
                                                (512, 4, False, 16001, 10), (128, 0, True, 20001, 1)])
def test_search_ranks_more_queries_than_compute_units(d, bits, prod, n, topk):
    test_search_by_candidates(d, bits, prod, 259, n, topk)


# workgroups of 32 queries up to five, four, three and two to a compute unit, as codes are long, and of more queries beyond
@pytest.mark.parametrize("d,bits,prod,nq,n,topk", [
    (128, 3, False, 128, 40960, 10), (128, 3, False, 128, 40961, 10), (512, 2, True, 65, 54529, 3), (1024, 1, True, 97, 32768, 5), (1024, 1, True, 97, 32769, 5),
    (1152, 4, False, 96, 32768, 1), (1152, 3, False, 96, 32897, 1), (1536, 4, False, 64, 32768, 10), (1536, 4, False, 64, 32769, 10), (1152, 2, True, 33, 32900, 64),
    (2048, 4, False, 129, 13056, 2), (2048, 4, False, 129, 13185, 2),
])
def test_search_blocks_of_32_queries(d, bits, prod, nq, n, topk):
    test_search_by_candidates(d, bits, prod, nq, n, topk)


def search_flags(p, q, c, d, prod, nq, n, topk):
    """Which queries of a search without a score buffer overflowed their lists, from the words that say so in the workspace: behind the rotated queries
    and the score matrix (topk > 16) that such queries need, where matrix-vector products rotate them."""
    assert topk > 16 and (d == 128 or nq * d <= 65536)
    p.workspace, p.c.workspace, p.c.workspace_bytes = None, 0, 0
    p.reserve_score(1, nq, n, prod, False, topk)
    p.workspace.fill_(85)
    top = torch.zeros((nq, topk), dtype=torch.int32, device=T.DEV), torch.zeros((nq, topk), device=T.DEV)
    tq.tq_score(p, q, 1, nq, c["idx"], c["qjl"], c["gamma"], c["norm"], n, None, topk, *top)
    line = lambda b: (b + 255) // 256 * 256  # noqa: E731
    at = line(nq * d * 4) * (2 if prod else 1) + line(nq * ((n + 3) // 4 * 4) * 4)
    return p.workspace.view(torch.uint8)[at:at + 4 * nq].view(torch.int32).cpu().numpy()


@pytest.mark.parametrize("d,bits,prod,nq,n,topk", [
    (1152, 2, False, 32, 140033, 17), (1152, 3, True, 17, 140033, 64), (1152, 4, False, 21, 140033, 64), (1152, 1, True, 29, 131201, 20),
    (1152, 0, True, 32, 135000, 17), (128, 0, True, 64, 140033, 17), (256, 4, True, 57, 70001, 33), (128, 3, True, 96, 140033, 17), (128, 4, False, 128, 140033, 64),
    (128, 1, False, 200, 30001, 17), (128, 2, True, 500, 140033, 33),
])
def test_search_finds_no_more_candidates_than_it_has_room_for(d, bits, prod, nq, n, topk):
    """Several tiles of codes to a workgroup in every block size of the kernel for few queries and in the one for many; and of random codes no query's
    list overflows, so that the answer is the candidates' and not that of the kernels which look at everything."""
    p = T.setup(d, bits, prod)[0]
    c = T._random_codes(p, d, bits, prod, n, d + n)
    q = T.dev(W.gaussian_queries(nq, d, 3, unit=False))
    T._topk_both_ways(p, q, 1, nq, c, n, topk)
    assert (search_flags(p, q, c, d, prod, nq, n, topk) == 0).all()


@pytest.mark.parametrize("d,nq", [(1152, 20), (128, 70), (128, 200)])
def test_search_says_which_lists_are_too_short(d, nq):
    """Equal scores: every query's list overflows."""
    n = 20000
    p = T.setup(d, 2, False)[0]
    c = T._random_codes(p, d, 2, False, n, 4)
    c["idx"], c["norm"] = c["idx"][:1].repeat(n, 1).contiguous(), torch.ones(n, device=T.DEV)
    assert (search_flags(p, T.dev(W.gaussian_queries(nq, d, 9, unit=False)), c, d, False, nq, n, 17) == 1).all()


@pytest.mark.parametrize("d,bits,prod", [(128, 2, True), (256, 3, False)])
def test_search_by_candidates_with_too_many_of_them(d, bits, prod):
    """Equal scores fill every query's list; rising ones defeat a bar from a sample; vectors of length zero tie at zero."""
    nq, n, topk = 40, 30000, 10
    p = T.setup(d, bits, prod)[0]
    q = T.dev(W.gaussian_queries(nq, d, 9, unit=False))
    c = T._random_codes(p, d, bits, prod, n, 4)
    for name in ("idx", "qjl", "gamma"):
        if c[name] is not None:
            c[name] = c[name][:1].repeat(n, *[1] * (c[name].dim() - 1)).contiguous()
    for norm in (np.ones(n), np.linspace(1.0, 2.0, n), np.where(np.arange(n) % 3 == 0, 1.0, 0.0)):
        c["norm"] = T.dev(norm.astype(np.float32))
        T._topk_both_ways(p, q, 1, nq, c, n, topk)


@pytest.mark.parametrize("d,bits,prod,nq", [(128, 2, True, 100), (256, 4, False, 70), (128, 0, True, 129)])
def test_search_by_candidates_with_infinite_norms(d, bits, prod, nq):
    """Scores that are infinite, or whose bound is, reach every bar: those of the places behind the last query are none."""
    n, topk = 20000, 64
    p = T.setup(d, bits, prod)[0]
    c = T._random_codes(p, d, bits, prod, n, 5)
    c["norm"][7::1013] = float("inf")
    c["norm"][11::517] = -float("inf")
    c["norm"][13::2001] = 3e38
    T._topk_both_ways(p, T.dev(W.gaussian_queries(nq, d, 9, unit=False)), 1, nq, c, n, topk)


@pytest.mark.parametrize("vprod,groups,qpg,npg", [(True, 2, 3, 1), (False, 2, 2, 8193), (True, 1, 1, 32768), (False, 1, 2, 32769)])
def test_attend_joins_of_chunks(vprod, groups, qpg, npg):
    """One chunk, more than sixteen, the 64 that a wavefront's lanes hold, and one more."""
    A.run_attend(128, 2, True, 2, vprod, groups, qpg, npg, True)


@pytest.mark.parametrize("bits,prod,npg", [(0, True, 65), (1, False, 1), (2, True, 2049), (3, True, 511), (4, False, 20500), (4, True, 130)])
def test_masked_sums_at_their_largest(bits, prod, npg):
    """Queries whose rotated coordinates are one large value among zeros, all equal, and of every sign pattern mod 4 (the digit
    scales go by coordinate mod 4); codes without norms."""
    p, Pi, S, c32, _ = T.setup(128, bits, prod)
    rng = np.random.default_rng(npg)
    y = np.zeros((7, 128))
    for k in range(4):
        y[k, 5 + 31 * k] = (-1.0) ** k * 3.0
    y[4] = 1.0
    y[5] = np.where(np.arange(128) % 4 < 2, 1.0, -1.0)
    y[6] = rng.standard_normal(128) * 10.0 ** rng.integers(-6, 7, 128)
    q = (y @ Pi).astype(np.float32)  # Pi q = y
    idx = rng.integers(0, 1 << bits, size=(npg, 128)).astype(np.int32)
    z = rng.integers(0, 2, size=(npg, 128)).astype(bool)
    gamma = rng.uniform(0.05, 0.6, size=npg).astype(np.float32)
    ones = np.ones(npg, dtype=np.float32)
    xt = T.o.dequant_prod(idx, z, gamma, Pi, S, c32, ones) if prod else T.o.dequant_mse(idx, Pi, c32, ones)
    idx_w = T.dev(T.o.pack_planes(idx, bits).view(np.int32)) if bits else None
    qjl_w = T.dev(T.o.pack_signs(z).view(np.int32)) if prod else None
    scores = torch.zeros((7, npg), device=T.DEV)
    p.reserve(npg, 7)
    tq.tq_score(p, T.dev(q), 1, 7, idx_w, qjl_w, T.dev(gamma) if prod else None, None, npg, scores)
    T.P.check_close(scores.cpu().numpy(), T.o.score(q, xt), np.linalg.norm(q.astype(np.float64), axis=1)[:, None] * ones[None, :], "score")
