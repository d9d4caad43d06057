"""Few queries against many long codes: steps of every width (whole lines, whole rows, what is left), wavefronts that gather the scores of
several blocks, ragged ends, rows of scores that are not aligned.  The sums are exact, so a list gives the same bits in one call and in pieces;
the pieces' kernel is checked against the oracle elsewhere and here on the first codes."""
import numpy as np
import pytest
import torch

from oracle import turboquant_oracle as o
from tests import test_gpu_parity as T

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")


@pytest.mark.parametrize("d,bits,prod,n,nq", [(2048, 0, True, 100037, 3), (1536, 1, True, 60037, 4), (1024, 1, True, 100037, 7), (768, 2, True, 60001, 4),
                                              (1536, 1, False, 100001, 1), (3072, 1, True, 50003, 6), (256, 4, True, 300007, 8), (640, 3, False, 100037, 5)])
def test_one_call_and_pieces(d, bits, prod, n, nq):
    p, Pi, S, c32, _ = T.setup(d, bits, prod)
    g = torch.Generator(device=T.DEV).manual_seed(d + n)

    def words(k):
        return torch.randint(-2**31, 2**31 - 1, (n, k), dtype=torch.int32, device=T.DEV, generator=g)

    idx, qjl = words(p.idx_words) if bits else None, words(p.qjl_words) if prod else None
    gamma = torch.rand(n, device=T.DEV, generator=g) if prod else None
    norm = torch.rand(n, device=T.DEV, generator=g) + 0.5
    q = torch.randn(nq, d, device=T.DEV, generator=g)
    p.reserve(1, nq, 0)
    wide = torch.full((nq, n + 5), 7.0, device=T.DEV)
    tq.tq_score(p, q, 1, nq, idx, qjl, gamma, norm, n, wide[:, :n])
    assert bool((wide[:, n:] == 7).all())
    step = 20000
    part = torch.empty((nq, step), device=T.DEV)
    for a in range(0, n, step):
        b = min(n, a + step)
        cut = [None if t is None else t[a:b] for t in (idx, qjl, gamma, norm)]
        tq.tq_score(p, q, 1, nq, *cut, b - a, part[:, :b - a])
        assert torch.equal(part[:, :b - a], wide[:, a:b])
    k = 64
    planes = o.unpack_planes(idx[:k].cpu().numpy().view(np.uint32), bits, d) if bits else np.zeros((k, d), dtype=np.int32)
    nrm = norm[:k].cpu().numpy()
    if prod:
        xt = o.dequant_prod(planes, o.unpack_signs(qjl[:k].cpu().numpy().view(np.uint32), d), gamma[:k].cpu().numpy(), Pi, S, c32, nrm)
    else:
        xt = o.dequant_mse(planes, Pi, c32, nrm)
    qh = q.cpu().numpy()
    T.P.check_close(wide[:, :k].cpu().numpy(), o.score(qh, xt), np.linalg.norm(qh.astype(np.float64), axis=1)[:, None] * nrm[None], "score")


@pytest.mark.parametrize("d,bits,prod,n,groups,nq", [(256, 2, False, 30011, 1, 20), (512, 1, True, 9001, 3, 9), (768, 3, True, 50003, 1, 32), (256, 4, False, 130, 5, 33),
                                                     (3072, 1, True, 49151, 1, 9), (3072, 1, True, 49152, 1, 9), (384, 2, True, 16001, 1, 61)])
def test_blocks_of_queries(d, bits, prod, n, groups, nq):
    """Several blocks of queries over the same codes, some of them not full, in grids that are no multiple of the XCDs: the bits of one query at a time."""
    p = T.setup(d, bits, prod)[0]
    c = T._random_codes(p, d, bits, prod, groups * n, d + n)
    q = torch.randn(groups * nq, d, device=T.DEV, generator=torch.Generator(device=T.DEV).manual_seed(n))
    p.reserve(1, groups * nq, 0)
    out, one = torch.zeros((groups * nq, n), device=T.DEV), torch.zeros((groups, n), device=T.DEV)
    tq.tq_score(p, q, groups, nq, c["idx"], c["qjl"], c["gamma"], c["norm"], n, out)
    for i in (0, 3, 4, 7, 8, nq - 1):
        tq.tq_score(p, q.view(groups, nq, d)[:, i].contiguous(), groups, 1, c["idx"], c["qjl"], c["gamma"], c["norm"], n, one)
        assert torch.equal(out.view(groups, nq, n)[:, i], one)


def random_words(p, n, seed):
    g = torch.Generator(device=T.DEV).manual_seed(seed)
    words = lambda k: torch.randint(-2**31, 2**31 - 1, (n, k), dtype=torch.int32, device=T.DEV, generator=g)  # noqa: E731
    return words(p.idx_words), words(p.qjl_words), torch.rand(n, device=T.DEV, generator=g), torch.rand(n, device=T.DEV, generator=g) + 0.5


# on either side of where eight queries a pass take the place of four
@pytest.mark.parametrize("d,bits,groups,nq,n", [(3072, 1, 1, 9, 40001), (3072, 1, 1, 5, 390001), (3072, 2, 1, 16, 30001), (3072, 2, 1, 16, 60001), (3072, 3, 1, 8, 20001),
                                                (3072, 3, 1, 8, 40001), (3200, 3, 4, 9, 8001), (3072, 4, 1, 9, 20001), (3072, 4, 1, 11, 30001), (3200, 4, 2, 7, 17001)])
def test_four_or_eight_queries_a_pass(d, bits, groups, nq, n):
    """Digits that fill LDS: the bits of one query at a time."""
    p = T.setup(d, bits, True)[0]
    c = random_words(p, groups * n, n)
    q = torch.randn(groups * nq, d, device=T.DEV, generator=torch.Generator(device=T.DEV).manual_seed(n))
    p.reserve(1, groups * nq, 0)
    out, one = torch.zeros((groups * nq, n), device=T.DEV), torch.zeros((groups, n), device=T.DEV)
    tq.tq_score(p, q, groups, nq, *c, n, out)
    for i in {0, 3, 4, min(8, nq - 1), nq - 1}:
        tq.tq_score(p, q.view(groups, nq, d)[:, i].contiguous(), groups, 1, *c, n, one)
        assert torch.equal(out.view(groups, nq, n)[:, i], one)


@pytest.mark.parametrize("d,bits,nq,most", [(3200, 3, 8, 1.7), (3072, 4, 16, 3.7)])
def test_a_pass_serves_eight_queries_of_a_long_list(d, bits, nq, most):
    """Four queries at a time would take nq / 4 times as long as four queries do."""
    n = 300000
    p = T.setup(d, bits, True)[0]
    c = random_words(p, n, n)
    p.reserve(1, nq, 0)

    def us(k):
        q, out = torch.randn(k, d, device=T.DEV), torch.zeros((k, n), device=T.DEV)
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = float("inf")
        for _ in range(6):
            e[0].record()
            for _ in range(4):
                tq.tq_score(p, q, 1, k, *c, n, out)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) * 250)
        return best

    four, all_of_them = us(4), us(nq)
    print(f"4 queries {four:.0f} us, {nq} {all_of_them:.0f} us")
    assert all_of_them <= most * four
