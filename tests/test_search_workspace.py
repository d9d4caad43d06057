"""A search by more queries than the workspace's blocks hold."""
import ctypes as C

import numpy as np
import pytest

import workloads as W


def plan_bytes(lib, d, bits, nq, n, topk, prod=False):
    from paper_2504_19874_amd import _lib
    c, t = np.linspace(-1, 1, 1 << bits, dtype=np.float32), np.zeros((1 << bits) - 1, dtype=np.float32)
    p = _lib.TqParams()
    p.d, p.bits_mse, p.centroids, p.bounds, p.images = d, bits, c.ctypes.data, t.ctypes.data, 4096
    p.flags = _lib.TQ_FLAG_DEQUANT_IMAGES
    return lib.tq_score_workspace_bytes(C.byref(p), 1, nq, n, int(prod), 0, topk)


@pytest.mark.parametrize("nq,d,n,topk,prod", [(100_000, 1536, 1_000_000, 10, False), (262_140, 128, 1_000_000, 16, True), (2_000, 768, 50_000_000, 10, False)])
def test_large_batches_need_little_more_than_their_rotated_queries(nq, d, n, topk, prod):
    """Beside the rotated queries and the partial lists of the scoring kernel: half a gigabyte of candidate lists and the
    pieces of 16384 queries."""
    from paper_2504_19874_amd import _lib
    rotated = nq * d * 4 * (2 if prod else 1)
    lists = 2 * nq * 4096 * 4 // 8  # at most 512 pairs a query for these numbers of queries
    assert plan_bytes(_lib.load(), d, 4, nq, n, topk, prod) <= rotated + lists + (512 << 20) + 16384 * (d * 4 + 4) + nq * 4 + 4096


@pytest.mark.parametrize("nq,n,d,topk", [(1000, 1_000_000, 1536, 64), (1000, 1_000_000, 3072, 10)])
def test_the_usual_batch_is_one_block(nq, n, d, topk):
    """Twice the queries take about twice the room where all of them are one block."""
    from paper_2504_19874_amd import _lib
    lib = _lib.load()
    assert plan_bytes(lib, d, 4, nq, n, topk) > 1.9 * plan_bytes(lib, d, 4, nq // 2, n, topk)


@pytest.mark.gpu
@pytest.mark.parametrize("d,bits,prod,nq,topk", [(128, 2, True, 11000, 10), (256, 3, False, 17000, 3)])
def test_blocks_of_queries(d, bits, prod, nq, topk):
    """Two blocks of lists (and two passes of the rotation): the same indices and bits as from the score matrix."""
    import torch
    import paper_2504_19874_amd as tq
    from tests import test_gpu_parity as T
    n = 8200
    p = T.setup(d, bits, prod)[0]
    c = T._random_codes(p, d, bits, prod, n, d)
    q = T.dev(np.tile(W.gaussian_queries(1000, d, 3, unit=False), (nq // 1000, 1)) * np.linspace(1, 2, nq, dtype=np.float32)[:, None])
    out = []
    for scores in (torch.zeros((nq, n), device=T.DEV), None):
        top = torch.full((nq, topk), -5, dtype=torch.int32, device=T.DEV), torch.zeros((nq, topk), device=T.DEV)
        p.reserve_score(1, nq, n, prod, scores is not None, topk)
        tq.tq_score(p, q, 1, nq, c["idx"], c["qjl"], c["gamma"], c["norm"], n, scores, topk, *top)
        out.append(top)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
