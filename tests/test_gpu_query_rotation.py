"""Queries into the rotated and the sketch basis, on either side of what matrix-vector products take: 64 of any length, 65536 values, 1024 at d = 128."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import turboquant_oracle as o
from tests import parity as P
from tests import test_gpu_parity as T

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")


def problem(d, bits, nq, seed):
    """A Pi that is orthogonal to 1e-3 only: what is documented as <S q, z> then differs from any S Pi^T (Pi q)."""
    rng = np.random.default_rng(seed)
    Pi = o.rotation_from_gaussian(W.gaussian_matrix(d, 100)) + rng.standard_normal((d, d)) * 1e-3 / np.sqrt(d)
    Pi = Pi.astype(np.float32)
    S = W.sketch_matrix(d, 200)
    c32, t32, _ = o.codebook_fp32(d, bits)
    p = tq.Params(d, bits, torch.from_numpy(Pi), torch.from_numpy(S), c32, t32)
    n = 700
    index = rng.integers(0, 1 << bits, size=(n, d))
    sign = rng.integers(0, 2, size=(n, d))
    gamma, norm = rng.uniform(0.5, 1, n).astype(np.float32), rng.uniform(0.5, 2, n).astype(np.float32)
    codes = (T.dev(o.pack_planes(index, bits).view(np.int32)) if bits else None, T.dev(o.pack_signs(sign > 0).view(np.int32)),
             T.dev(gamma), T.dev(norm))
    q = W.gaussian_queries(nq, d, 3, unit=False).astype(np.float32)
    q64 = q.astype(np.float64)
    want = norm * (q64 @ Pi.T.astype(np.float64) @ np.asarray(c32, dtype=np.float64)[index].T
                   + np.sqrt(np.pi / 2) / d * gamma * (q64 @ S.T.astype(np.float64) @ (2.0 * sign - 1).T))
    return p, q, codes, n, want, np.linalg.norm(q64, axis=1)[:, None] * norm


def run(p, q, codes, n):
    s = torch.zeros((q.shape[0], n), device=T.DEV)
    p.reserve_score(1, q.shape[0], n, True, True)
    tq.tq_score(p, T.dev(q), 1, q.shape[0], *codes, n, s)
    return s


@pytest.mark.parametrize("d,bits,nq", [(256, 0, 64), (256, 0, 65), (768, 1, 300), (160, 2, 129), (1536, 0, 100), (128, 0, 90),
                                       (256, 0, 256), (256, 0, 257), (160, 2, 409), (160, 2, 410), (128, 0, 1024), (128, 0, 1025), (1536, 0, 64), (1536, 1, 65)])
def test_the_sketch_comes_from_s(d, bits, nq):
    p, q, codes, n, want, scale = problem(d, bits, nq, d + nq)
    P.check_close(run(p, q, codes, n).cpu().numpy(), want, scale, "score")


# rows shorter than a wavefront's load, not a multiple of one, of two; blocks of four queries with one to four of them
@pytest.mark.parametrize("d,bits,nq", [(32, 1, 64), (96, 1, 33), (224, 0, 61), (288, 2, 42), (384, 2, 64), (544, 1, 35)])
def test_a_wavefront_per_row(d, bits, nq):
    p, q, codes, n, want, scale = problem(d, bits, nq, d + nq)
    P.check_close(run(p, q, codes, n).cpu().numpy(), want, scale, "score")


@pytest.mark.parametrize("d,bits,few,many", [(128, 1, 70, 1100), (256, 2, 65, 300)])
def test_the_fp32_instructions_for_any_number_above_64(d, bits, few, many):
    """TQ_FLAG_FP32_MFMA: a query's scores do not depend on how many come with it."""
    p, q, codes, n, want, scale = problem(d, bits, many, d)
    try:
        p.fp32_mfma = True
        whole = run(p, q, codes, n)
        assert torch.equal(run(p, q[:few], codes, n), whole[:few])
    finally:
        p.fp32_mfma = False
    P.check_close(whole.cpu().numpy(), want, scale, "score")


@pytest.mark.parametrize("d,bits,nq", [(256, 1, 257), (1024, 0, 130)])
def test_images_change_no_bit(d, bits, nq):
    """The matrices' pieces from the images, or made in a workspace of the size that is asked for without them."""
    p, q, codes, n, want, scale = problem(d, bits, nq, d)
    with_images = run(p, q, codes, n)
    p.workspace, p.c.workspace, p.c.workspace_bytes = None, 0, 0
    without = run(p.drop_images(), q, codes, n)
    assert torch.equal(with_images, without)
    # the least that a call takes: rotated on the fp32 instructions
    p.workspace, p.c.workspace, p.c.workspace_bytes = None, 0, 0
    p.reserve_bytes(2 * q.shape[0] * d * 4 + 2048)
    s = torch.zeros_like(without)
    tq.tq_score(p, T.dev(q), 1, q.shape[0], *codes, n, s)
    P.check_close(s.cpu().numpy(), want, scale, "score")
