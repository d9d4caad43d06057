"""What the arithmetic on pieces and digits leaves of fp32, against 64-bit sums on the GPU: no further from them than the fp32 matrix
instructions where these served before, and within twice the errors that the header states."""
import math

import numpy as np
import pytest
import torch

from tests import test_gpu_parity as T

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")

D = 128


def unpack(words, bits, d):
    w = words.view(words.shape[0], d // 32, bits, 1)
    b = (w >> torch.arange(32, device=T.DEV, dtype=torch.int32)) & 1
    return (b << torch.arange(bits, device=T.DEV, dtype=torch.int32).view(1, 1, bits, 1)).sum(2).view(words.shape[0], d)


def table(a):
    return torch.tensor(np.asarray(a).reshape(-1), device=T.DEV, dtype=torch.float64)


# ------------------------------------------------------------------ quantisation of few bf16 vectors


def rows(g, kind, n):
    x = torch.randn(n, D, generator=g, device=T.DEV)
    if kind == "outliers":
        x[:, torch.randperm(D, generator=g, device=T.DEV)[:4]] *= 20
    if kind == "centres":
        c = torch.randn(256, D, generator=g, device=T.DEV)
        x = 0.3 * x + c[torch.randint(256, (n,), generator=g, device=T.DEV)]
    return x.to(torch.bfloat16)


def errors(p, x, bits, prod, Pi, W, c, t):
    """Wrong indices and signs, and the summed squares of gamma's and the norm's relative errors."""
    n = x.shape[0]
    idx = torch.zeros((n, max(1, p.idx_words)), dtype=torch.int32, device=T.DEV)
    qjl = torch.zeros((n, p.qjl_words), dtype=torch.int32, device=T.DEV)
    gamma, norm = torch.zeros(n, device=T.DEV), torch.zeros(n, device=T.DEV)
    if prod:
        tq.tq_quantize_prod(p, x, idx, qjl, gamma, norm)
    else:
        tq.tq_quantize_mse(p, x, idx, norm)
    xd = x.double()
    nu = xd.norm(dim=1)
    y = (xd / nu[:, None]) @ Pi.T
    out = [0.0, 0.0, 0.0, float(((norm.double() - nu) / nu).pow(2).sum())]
    got = unpack(idx, bits, D)
    out[0] = float((got != torch.bucketize(y, t, right=True)).sum())
    if prod:
        e = y - c[got.long()]
        size = e.norm(dim=1)
        out[1] = float((unpack(qjl, 1, D) != (e @ W.T >= 0)).sum())
        out[2] = float(((gamma.double() - size) / size).pow(2).sum())
    return np.array(out)


@pytest.mark.parametrize("kind", ["outliers", "normal", "centres"])
@pytest.mark.parametrize("bits,prod,n", [(4, False, 8192), (3, True, 8192), (2, True, 512), (1, True, 4096)])
def test_few_vectors_no_further_off_than_the_fp32_instructions(kind, bits, prod, n):
    """Two fp16 pieces hold 22 bits of an entry of Pi, but a sum meets a quarter of the roundings."""
    p, Pi, S, c32, t32 = T.setup(D, bits, prod)
    Pi = T.dev(Pi).double()
    W = T.dev(S).double() @ Pi.T if prod else None
    g = torch.Generator(device=T.DEV)
    g.manual_seed(bits + n)
    pieces, fp32 = np.zeros(4), np.zeros(4)
    for _ in range((1 << 19) // n):  # 6.7e7 coordinates
        x = rows(g, kind, n)
        try:
            pieces += errors(p, x, bits, prod, Pi, W, table(c32), table(t32))
            p.fp32_mfma = True
            fp32 += errors(p, x, bits, prod, Pi, W, table(c32), table(t32))
        finally:
            p.fp32_mfma = False
    # counts of rare events: two standard deviations of their own number
    assert np.all(pieces[:2] <= fp32[:2] + 2 * np.sqrt(fp32[:2] + 1)), (pieces, fp32)
    assert np.all(pieces[2:] <= 1.02 * fp32[2:]), (pieces, fp32)


# ------------------------------------------------------------------ quantisation below d = 512


@pytest.mark.parametrize("d,bits,n,bf16", [(64, 3, 16385, True), (64, 4, 20001, False), (256, 4, 17003, True), (192, 3, 16400, False), (384, 4, 16385, False),
                                           (384, 3, 40001, True), (256, 2, 16385, False), (256, 4, 200, False), (96, 3, 5, True)])
def test_every_bit_of_pi(d, bits, n, bf16):
    """More than 16384 vectors below d = 512 (and a few at any d) meet all 24 bits of an entry of Pi: of a unit vector that is one entry, here
    on a cell's boundary or the next number below it.  One product and zeros: every sum is exact."""
    rng = np.random.default_rng(d + bits)
    half = np.sort(rng.uniform(0.02, 0.3, 1 << bits - 1).astype(np.float32))
    bounds = np.concatenate([-half[1:][::-1], np.zeros(1, np.float32), half[1:]])
    c = np.concatenate([-half[::-1], half])
    at = rng.choice(bounds[bounds != 0], size=(d, d))
    Pi = np.where(rng.random((d, d)) < 0.5, at, np.nextafter(at, np.float32(-1))).astype(np.float32)
    p = tq.Params(d, bits, torch.from_numpy(Pi), None, c, bounds)
    k = np.arange(n) % d
    x = torch.zeros((n, d), device=T.DEV, dtype=torch.bfloat16 if bf16 else torch.float32)
    x[torch.arange(n), torch.from_numpy(k)] = 1
    idx = torch.zeros((n, p.idx_words), dtype=torch.int32, device=T.DEV)
    p.reserve(n)
    tq.tq_quantize_mse(p, x, idx, None)
    want = torch.from_numpy(np.searchsorted(bounds, Pi, side="right")).to(T.DEV).T[torch.from_numpy(k).to(T.DEV)]
    assert int((unpack(idx, bits, d) != want).sum()) == 0


# ------------------------------------------------------------------ dequantisation of sums of signs


def restore_error(p, d, bits, prod, n, Pi, S, c32):
    """Error in units of a coordinate's root mean square: (root mean square, largest)."""
    g = torch.Generator(device=T.DEV)
    g.manual_seed(n + bits)
    word = lambda k: torch.empty((n, k), dtype=torch.int32, device=T.DEV).random_(-2**31, 2**31 - 1, generator=g)  # noqa: E731
    idx, qjl = word(max(1, p.idx_words)), word(p.qjl_words)
    gamma, norm = 0.2 + 0.3 * torch.rand(n, generator=g, device=T.DEV), 0.5 + torch.rand(n, generator=g, device=T.DEV)
    out = torch.empty((n, d), device=T.DEV)
    p.reserve(n)
    tq.tq_dequantize(p, idx if bits else None, qjl if prod else None, gamma if prod else None, norm, out)
    want = table(c32)[unpack(idx, bits, d).long()] @ Pi if bits else 0.0
    if prod:
        want = want + math.sqrt(math.pi / 2) / d * gamma.double()[:, None] * ((2.0 * unpack(qjl, 1, d) - 1).double() @ S)
    e = (out.double() / norm.double()[:, None] - want) / want.pow(2).mean().sqrt()
    return float(e.pow(2).mean().sqrt()), float(e.abs().max())


# (d, codes): the error that is stated for it, root mean square
STATED = {(128, 8): 0.8e-7, (128, 8192): 0.8e-7, (128, 8193): 1.55e-6, (128, 60000): 1.55e-6, (256, 5000): 1.2e-7, (768, 3000): 1.7e-7,
          (1536, 700): 2.2e-7, (3072, 400): 3.1e-7}


@pytest.mark.parametrize("bits,prod", [(0, True), (1, False), (1, True), (2, False), (2, True)])
@pytest.mark.parametrize("d,n", list(STATED))
def test_signs_against_digits(d, n, bits, prod):
    from paper_2504_19874_amd import _lib
    p, Pi, S, c32, _ = T.setup(d, bits, prod)
    Pi, S = T.dev(Pi).double(), T.dev(S).double() if prod else None
    rms, most = restore_error(p, d, bits, prod, n, Pi, S, c32)
    # errors of a few million coordinates, none of them an outlier: up to about 15 times their root mean square (where a code's
    # kinds of sign add up to a long vector)
    assert rms <= 2 * STATED[d, n] and most <= 30 * STATED[d, n], (rms, most)
    flags = p.c.flags
    try:
        p.c.flags = flags & ~_lib.TQ_FLAG_SIGN_IMAGES  # the kernels of the other tables
        before = restore_error(p, d, bits, prod, n, Pi, S, c32)
        p.c.flags = flags | _lib.TQ_FLAG_FP32_MFMA
        fp32 = restore_error(p, d, bits, prod, n, Pi, S, c32)
    finally:
        p.c.flags = flags
    assert rms <= before[0] and (rms <= fp32[0] or (d == 128 and n > 8192)), (rms, before, fp32)


# ------------------------------------------------------------------ attention read-out of one short chunk


@pytest.mark.parametrize("bits,prod", [(2, False), (4, False), (0, True), (2, True)])
@pytest.mark.parametrize("npg", [1, 100, 256, 512])
def test_one_chunk_no_further_off_than_chunks_that_are_joined(npg, bits, prod):
    """Up to 512 tokens the workgroup that has a query's sums rotates them back itself: chains of 16 products, as in the joining kernel, which
    the same values come to in a call with more groups than the chip has compute units.  Queries of length zero: every weight is 1 / npg
    exactly, and what is left of the error is the sums', the division's and the rotation's."""
    pk = T.setup(D, 2, True)[0]
    pv, Pi, S, c32, _ = T.setup(D, bits, prod)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    part, groups = cus // 4, cus + cus // 4
    n = groups * npg
    g = torch.Generator(device=T.DEV)
    g.manual_seed(npg + bits)
    word = lambda k: torch.empty((n, k), dtype=torch.int32, device=T.DEV).random_(-2**31, 2**31 - 1, generator=g)  # noqa: E731
    scalar = lambda: (0.3 * torch.randn(n, generator=g, device=T.DEV)).exp()  # noqa: E731
    keys = word(pk.idx_words), word(pk.qjl_words), 0.3 * scalar(), scalar()
    idx, qjl, gamma, norm = word(max(1, pv.idx_words)), word(pv.qjl_words), 0.3 * scalar(), scalar()
    values = idx if bits else None, qjl if prod else None, gamma if prod else None, norm
    q, joined, own = (torch.zeros((groups, D), device=T.DEV) for _ in range(3))
    tq.tq_attend(pk, pv, q, groups, 1, keys, values, npg, 0.09, joined)
    for g0 in range(0, groups, part):
        cut = lambda ts: tuple(t if t is None else t[g0 * npg:(g0 + part) * npg] for t in ts)  # noqa: E731
        tq.tq_attend(pk, pv, q[g0:g0 + part], part, 1, cut(keys), cut(values), npg, 0.09, own[g0:g0 + part])
    mean = lambda t: t.view(groups, npg, D).mean(1)  # noqa: E731
    want = mean(norm.double()[:, None] * table(c32)[unpack(idx, bits, D).long()]) @ T.dev(Pi).double() if bits else 0.0
    if prod:
        want = want + math.sqrt(math.pi / 2) / D * mean((norm.double() * gamma.double())[:, None] * (2.0 * unpack(qjl, 1, D) - 1).double()) @ T.dev(S).double()
    error = lambda o: float((((o.double() - want).pow(2).sum(1) / want.pow(2).sum(1)).mean()).sqrt())  # noqa: E731
    mine, theirs = error(own), error(joined)
    print(f"{npg} tokens, {bits} bits{' and signs' if prod else ''}: {mine:.3e}, joined {theirs:.3e}")
    # Values of three planes and more than 256 tokens: eight wavefronts' sums of 64 keys are added one after the other, of 256 keys in a call with
    # many groups, so two here.  (2 + 3 + ... + 8) / 8 - 1 = 3.4 more squared roundings, each 2^-24 / sqrt(3) at most of the sum, 0.72 of that in the
    # root mean square of mantissas from 1 to 2.
    more = 3.4 * (0.72 * 2.0**-24 / math.sqrt(3)) ** 2 if npg > 256 and bits + prod > 2 else 0.0
    # 40960 coordinates: two independent estimates of one error differ by 0.5 %
    assert mine <= 1.02 * math.sqrt(theirs**2 + more), (mine, theirs)
