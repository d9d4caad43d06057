"""How much of an fp32 vector the quantisers read: with Pi = I and no normalisation the rotated coordinates are the
vector itself, and coordinates a little beside the cell boundaries show the bits that an operand form leaves out."""
import numpy as np
import pytest
import torch

from tests import test_gpu_parity as T
from oracle import turboquant_oracle as o

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")


def check_decisions(d, bits, prod, n, beside):
    """beside(t): fp32 values next to the boundaries t, whose cells the quantiser has to tell apart."""
    c, t, _ = tq.tq_build_codebook(d, bits)
    eye = torch.eye(d)
    p = tq.Params(d, bits, eye, eye if prod else None, c, t).reserve(n)
    rng = np.random.default_rng(d + n)
    x = beside(t[rng.integers(0, t.size, size=(n, d))], rng)
    assert x.dtype == np.float32
    idx = torch.zeros((n, p.idx_words), dtype=torch.int32, device=T.DEV)
    if prod:
        qjl = torch.zeros((n, p.qjl_words), dtype=torch.int32, device=T.DEV)
        gamma = torch.zeros(n, device=T.DEV)
        tq.tq_quantize_prod(p, T.dev(x), idx, qjl, gamma, None)
    else:
        tq.tq_quantize_mse(p, T.dev(x), idx, None)
    got = o.unpack_planes(T.words(idx), bits, d)
    want = np.searchsorted(t, x, side="right")  # on a boundary: the upper cell
    assert np.array_equal(got, want), f"{(got != want).sum()} of {got.size} decisions"


def all_bits(t, rng):
    """The boundary itself and the fp32 value below it: 24 bits."""
    return np.where(rng.random(t.shape) < 0.5, t, np.nextafter(t, np.float32(-1))).astype(np.float32)


@pytest.mark.parametrize("d,bits,prod,n", [(512, 4, False, 64), (1024, 4, False, 64), (1536, 4, False, 61), (3072, 3, False, 16), (4096, 4, False, 1),
                                           (4096, 3, False, 8), (1024, 3, True, 64), (1536, 4, True, 32), (3072, 4, True, 8), (4096, 3, True, 4)])
def test_few_long_vectors_in_fp32(d, bits, prod, n):
    """Up to 64 vectors of 512 coordinates and more, while their blocks of four times d^2 stay within the limit: plain fp32."""
    check_decisions(d, bits, prod, n, all_bits)


@pytest.mark.parametrize("d,bits,n", [(32, 2, 100), (64, 3, 1000), (96, 3, 65), (384, 4, 3000), (416, 4, 129), (64, 3, 16384)])
def test_small_residuals_in_fp32(d, bits, n):
    """Alg. 2 of fp32 vectors whose residual is small: the rotation stays on the fp32 instructions whatever the batch size."""
    check_decisions(d, bits, True, n, all_bits)
