"""Top-k over rows in which many scores pass for candidates: equal ones, rising ones, infinities and zeros of both signs."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import test_gpu_parity as T

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")


def rows(kind, n):
    """Factors of one code's score, so that they are the scores up to rounding and a common sign."""
    i = np.arange(n)
    rng = np.random.default_rng(n)
    return {"drawn": rng.uniform(1, 2, n), "rising": 1.0 + i / n, "falling": 2.0 - i / n, "equal": np.ones(n),
            "ties at the end": np.where(rng.random(n) < 20 / n, 2.0, 0.0), "zeros": np.where(i % 2 == 0, -0.0, 0.0),
            "steps": 1.0 + i // 1000, "period": 1.0 + (i % 1024 < 40) * i, "infinite": np.where(i % 3 == 0, np.inf, 1.0),
            }[kind].astype(np.float32)


def call(p, q, c, n, topk, nq=2):
    scores = torch.zeros((nq, n), device=T.DEV)
    top = torch.zeros((nq, topk), dtype=torch.int32, device=T.DEV), torch.zeros((nq, topk), device=T.DEV)
    p.reserve_score(1, nq, n, False, True, topk)
    run = lambda: tq.tq_score(p, q, 1, nq, c["idx"], None, None, c["norm"], n, scores, topk, *top)  # noqa: E731
    run()
    return scores, top, run


def both_signs(nq):
    """One query nq // 2 times, then its opposite."""
    q = W.gaussian_queries(1, 128, 5, unit=False)
    return T.dev(np.concatenate([q.repeat(nq // 2, 0), -q.repeat(nq - nq // 2, 0)]))


def case(kind, n):
    p = T.setup(128, 2, False)[0]
    c = T._random_codes(p, 128, 2, False, 1, 3)
    c["idx"] = c["idx"].repeat(n, 1).contiguous()
    c["norm"] = T.dev(rows(kind, n))
    return p, c


@pytest.mark.parametrize("topk", [1, 10, 64])
@pytest.mark.parametrize("nq,n", [(2, 8192), (2, 50001), (2, 300000), (129, 50001)])  # one segment, chunks and their joining, a workgroup's several segments
@pytest.mark.parametrize("kind", ["rising", "falling", "equal", "ties at the end", "zeros", "steps", "period", "infinite"])
def test_many_candidates(kind, nq, n, topk):
    p, c = case(kind, n)
    scores, (ti, tv), _ = call(p, both_signs(nq), c, n, topk, nq)
    s = scores.cpu().numpy()
    for r in (0, nq // 2):
        want = np.argsort(-s[r], kind="stable")[:topk]  # equal scores by lower index
        assert np.array_equal(ti[r].cpu().numpy(), want)
        assert np.array_equal(tv[r].cpu().numpy(), s[r][want])


@pytest.mark.parametrize("nq,n", [(2, 16384), (2, 16385), (128, 16385), (129, 40001),  # two segments; chunks from there; several segments of a workgroup
                                  (2, 16 * 8192), (2, 16 * 8192 + 1), (2, 33 * 8192 - 5)])  # of 64: 1024, 1088 and 2112 pairs to be joined
@pytest.mark.parametrize("topk", [16, 17, 64])  # bars from the maxima of four threads, of one
@pytest.mark.parametrize("kind", ["drawn", "rising", "equal", "period", "infinite"])
def test_chunks_and_bars(kind, nq, n, topk):
    p, c = case(kind, n)
    q = W.gaussian_queries(nq, 128, 5, unit=False)
    scores, (ti, tv), _ = call(p, T.dev(q), c, n, topk, nq)
    s = scores.cpu().numpy()
    for r in range(0, nq, 1 if nq < 10 else 37):
        want = np.argsort(-s[r], kind="stable")[:topk]  # equal scores by lower index
        assert np.array_equal(ti[r].cpu().numpy(), want)
        assert np.array_equal(tv[r].cpu().numpy(), s[r][want])


@pytest.mark.parametrize("nq,n", [(2, 63), (2, 4096), (2, 4097), (2, 8193),  # fewer than k; a segment of 256 threads, of 512, of 1024
                                  (2, 3 * 16384), (2, 3 * 16384 + 1), (513, 20001),  # three segments, chunks from there, more rows than workgroups fit
                                  (65, 65537), (128, 70001)])  # more chunks than compute units: as many of 512 threads, fewer
@pytest.mark.parametrize("topk", [16, 64])  # bars from 64 maxima, from 256
@pytest.mark.parametrize("kind", ["drawn", "falling", "equal", "zeros", "infinite"])
def test_segments_and_threads(kind, nq, n, topk):
    p, c = case(kind, n)
    scores, (ti, tv), _ = call(p, T.dev(W.gaussian_queries(nq, 128, 5, unit=False)), c, n, topk, nq)
    s = scores.cpu().numpy()
    for r in range(0, nq, max(1, nq // 3)):
        want = np.argsort(-s[r], kind="stable")[:topk]
        k = len(want)
        assert np.array_equal(ti[r, :k].cpu().numpy(), want) and (ti[r, k:] == -1).all()
        assert np.array_equal(tv[r, :k].cpu().numpy().view(np.int32), s[r][want].view(np.int32))  # the sign of a zero, too


@pytest.mark.parametrize("nq,n", [(257, 9217), (513, 8193), (513, 200003), (768, 20001),  # more rows than the chip takes of 1024 threads, up to three of 512 each
                                  (769, 8192), (769, 40001), (1024, 8191), (1025, 20001), (1025, 40001),  # a few more, many more; long and short rows
                                  (43, 131072), (64, 131071), (65, 131073), (24, 200001), (100, 41001)])  # chunks of 512 threads, of 1024, two to a compute unit
@pytest.mark.parametrize("topk", [1, 3, 16, 64])  # the largest maximum is the bar, up to eight of them pass
@pytest.mark.parametrize("kind", ["drawn", "rising", "zeros", "infinite"])
def test_rows_that_fill_the_chip(kind, nq, n, topk):
    p, c = case(kind, n)
    scores, (ti, tv), _ = call(p, both_signs(nq), c, n, topk, nq)
    for r in (0, nq // 2 - 1, nq - 1):
        s = scores[r].cpu().numpy()
        want = np.argsort(-s, kind="stable")[:topk]  # equal scores by lower index
        assert np.array_equal(ti[r].cpu().numpy(), want)
        assert np.array_equal(tv[r].cpu().numpy().view(np.int32), s[want].view(np.int32))


@pytest.mark.parametrize("nq", [2, 129])  # a segment per workgroup, seven
@pytest.mark.parametrize("kind", ["rising", "equal", "ties at the end", "steps"])
def test_their_cost_is_bounded(kind, nq):
    """50001 scores per row: within ten times a row of drawn scores (the quadratic ranking of whole segments
    that this guards against takes thousands of times as long)."""
    def us(kind):
        p, c = case(kind, 50001)
        _, _, run = call(p, both_signs(nq), c, 50001, 10, nq)
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        torch.cuda.synchronize()
        best = float("inf")
        for _ in range(5):
            e[0].record()
            run()
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) * 1e3)
        return best

    many, drawn = us(kind), us("drawn")
    print(f"{kind}: {many:.0f} us, drawn {drawn:.0f} us")
    assert many <= 10 * drawn + 20


@pytest.mark.parametrize("d,bits,prod", [(128, 2, True), (256, 3, False), (384, 0, True), (512, 1, True)])
def test_search_with_scalars_of_both_signs(d, bits, prod):
    """Norms and residual norms are lengths, but nothing refuses others: the bounds of a search by candidates hold for them."""
    n, nq, rng = 20000, 40, np.random.default_rng(d)
    p = T.setup(d, bits, prod)[0]
    q = T.dev(W.gaussian_queries(nq, d, 9, unit=False))
    c = T._random_codes(p, d, bits, prod, n, 4)
    for name in ("norm", "gamma"):
        if c[name] is not None:
            c[name] = c[name] * T.dev(rng.choice(np.float32([-1, 1]), size=n))
    T._topk_both_ways(p, q, 1, nq, c, n, 10)


@pytest.mark.parametrize("d,nq", [(128, 256), (128, 257), (2048, 40), (2176, 40)])  # eight wavefronts per query, four; eight; four
@pytest.mark.parametrize("topk", [1, 64])
def test_selection_from_the_candidates(d, nq, topk):
    n = 9000
    p = T.setup(d, 2, True)[0]
    q = T.dev(W.gaussian_queries(nq, d, 9, unit=False))
    T._topk_both_ways(p, q, 1, nq, T._random_codes(p, d, 2, True, n, 4), n, topk)
