"""Dequantisation where the centroid table is a sum of signs (none, one bit, two symmetric bits): at d = 128 blocks of 32 codes, four or
five digits of an entry, from the images or made in the workspace, and the tables that have to go elsewhere; at longer d
workgroups of 256 and 512 codes."""
import numpy as np
import pytest
import torch

from oracle import turboquant_oracle as o
from tests import test_gpu_parity as T

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")

D = 128


def make(bits, prod, n, d=D):
    p, Pi, S, c32, _ = T.setup(d, bits, prod)
    rng = np.random.default_rng(100 * n + bits)
    idx = rng.integers(0, 1 << bits, size=(n, d)).astype(np.int32)
    z = rng.integers(0, 2, size=(n, d)).astype(bool)
    gamma = rng.uniform(0.05, 0.6, size=n).astype(np.float32)
    norm = np.exp(rng.normal(0, 1, size=n)).astype(np.float32)
    codes = [T.dev(o.pack_planes(idx, bits).view(np.int32)) if bits else None, T.dev(o.pack_signs(z).view(np.int32)) if prod else None,
             T.dev(gamma) if prod else None]
    return p, codes, (idx, z, gamma, Pi, S, c32), norm


def reference(parts, prod, norm):
    idx, z, gamma, Pi, S, c = parts
    return o.dequant_prod(idx, z, gamma, Pi, S, c, norm) if prod else o.dequant_mse(idx, Pi, c, norm)


def close(got, want, norm, n):
    # Five digits of an entry: the rounding of fp32 sums of 128 terms, below 128 2^-24 of a coordinate's typical size.  Four, above
    # 8192 codes: an entry is off by at most half of its column's largest (0.4 here) / 17301504 * 32, uniformly: of 128 terms of
    # typical size 1 / sqrt(128), 2.5e-6, and no more than 7 times that in a few million coordinates.  Two kinds of sign add.
    scale = (np.ones(n) if norm is None else norm.astype(np.float64))[:, None] / np.sqrt(D)
    assert np.abs((got.astype(np.float64) - want) / scale).max() < (8e-6 if n <= 8192 else 3.5e-5)


@pytest.mark.parametrize("bits,prod,n", [(0, True, 1), (1, False, 31), (1, True, 33), (2, False, 64), (2, True, 511), (2, True, 2049),
                                         (2, True, 8192), (1, True, 8193), (2, False, 16421), (0, True, 16385)])
def test_blocks_and_images(bits, prod, n):
    p, codes, parts, norm = make(bits, prod, n)
    wide = torch.full((n + 1, 132), 7.0, device=T.DEV)  # rows of a larger matrix: what lies around them stays
    tq.tq_dequantize(p, *codes, T.dev(norm), wide[:n, :D])
    got = wide[:n, :D].clone()
    assert bool((wide[:n, D:] == 7).all()) and bool((wide[n] == 7).all())
    close(got.cpu().numpy(), reference(parts, prod, norm), norm, n)
    out = torch.empty((n, D), device=T.DEV)
    tq.tq_dequantize(p, *codes, None, out)
    close(out.cpu().numpy(), reference(parts, prod, None), None, n)
    try:
        p.drop_images().reserve(n)  # the digits made in the call: the same bits
        tq.tq_dequantize(p, *codes, T.dev(norm), out)
        assert torch.equal(out, got)
    finally:
        p.build_images()


@pytest.mark.parametrize("table", [(-0.09, -0.03, 0.04, 0.09), (-0.08, -0.08, 0.08, 0.08), (-0.1, 0.0, 0.0, 0.1), (0.0, 0.0, 0.0, 0.0)])
@pytest.mark.parametrize("n", [100, 8200])
def test_other_tables(table, n):
    """Two bits that are not symmetric, or of one magnitude, or with zeros: whatever kernel takes them."""
    p0, codes, parts, norm = make(2, False, n)
    c = np.array(table, dtype=np.float32)
    p = tq.Params(D, 2, p0.Pi, p0.S, c, (c[1:] + c[:-1]) / 2)
    out = torch.empty((n, D), device=T.DEV)
    tq.tq_dequantize(p, *codes, T.dev(norm), out)
    T.P.check_close(out.cpu().numpy(), reference(parts[:5] + (c,), False, norm), norm.astype(np.float64)[:, None] / np.sqrt(D), "coordinate")


@pytest.mark.parametrize("d,bits,prod,n", [(256, 1, True, 65), (384, 0, True, 300), (640, 2, True, 257), (896, 1, False, 1000), (256, 2, False, 4097),
                                           (512, 2, True, 24577), (1536, 2, True, 130), (384, 1, True, 40001)])
def test_long_codes(d, bits, prod, n):
    p, codes, parts, norm = make(bits, prod, n, d)
    wide = torch.full((n + 1, d + 4), 7.0, device=T.DEV)
    tq.tq_dequantize(p, *codes, T.dev(norm), wide[:n, :d])
    got = wide[:n, :d].clone()
    assert bool((wide[:n, d:] == 7).all()) and bool((wide[n] == 7).all())
    # five digits of every 64 indices and kind of sign are added in turn, each rounding at most 2^-24 of a sum of up to six times its typical size
    scale = norm.astype(np.float64)[:, None] / np.sqrt(d)
    assert np.abs((got.cpu().numpy() - reference(parts, prod, norm)) / scale).max() < 5 * d / 64 * (bits + prod) * 6 * 2.0**-24
    out = torch.empty((n, d), device=T.DEV)
    try:
        p.drop_images().reserve(n)  # the digits made in the call: the same bits
        tq.tq_dequantize(p, *codes, T.dev(norm), out)
        assert torch.equal(out, got)
    finally:
        p.build_images()


# up to 32 codes of a workgroup and up to 64, the last of several, the ends of the range (256 compute units); fewer steps than wavefronts, a remainder of them
@pytest.mark.parametrize("d,bits,prod,n", [(256, 2, False, 1), (256, 2, True, 32), (256, 0, True, 33), (384, 1, True, 31), (384, 2, False, 65), (512, 1, False, 1024), (512, 1, False, 1025),
                                           (640, 1, True, 64), (640, 2, True, 1600), (1152, 2, False, 129), (1536, 2, True, 64), (1024, 1, True, 100), (768, 2, True, 33),
                                           (256, 1, True, 2048), (256, 1, True, 2049), (512, 1, True, 1025), (640, 1, True, 1537), (1536, 2, True, 14), (1536, 2, True, 15), (2048, 1, True, 8)])
def test_few_long_codes(d, bits, prod, n):
    p, codes, parts, norm = make(bits, prod, n, d)
    wide = torch.full((n + 1, d + 4), 7.0, device=T.DEV)
    tq.tq_dequantize(p, *codes, T.dev(norm), wide[:n, :d])
    assert bool((wide[:n, d:] == 7).all()) and bool((wide[n] == 7).all())
    # as above, and the eight wavefronts' sums are added
    scale = norm.astype(np.float64)[:, None] / np.sqrt(d)
    assert np.abs((wide[:n, :d].cpu().numpy() - reference(parts, prod, norm)) / scale).max() < (5 * d / 64 * (bits + prod) + 8) * 6 * 2.0**-24


# matrix-vector products: fewer coordinates than lanes, than threads, not a multiple of either; one, two and four rows per wavefront; full and partial
# blocks of two, four and eight codes; the ends of the range and one beyond
@pytest.mark.parametrize("d,bits,prod,n", [(32, 3, False, 1), (32, 4, True, 3), (64, 3, True, 9), (96, 4, False, 13), (128, 4, False, 512), (128, 3, True, 513), (160, 3, True, 31),
                                           (288, 4, False, 250), (544, 3, True, 66), (1056, 3, False, 61), (1056, 4, True, 186), (2080, 3, True, 5), (2080, 4, False, 47),
                                           (2080, 4, False, 48), (2048, 3, False, 5), (2048, 4, False, 90), (2048, 4, True, 5), (2048, 3, True, 90), (2016, 4, False, 33), (2016, 3, True, 33),
                                           (64, 0, True, 100), (96, 2, True, 200), (1536, 2, True, 9)])
def test_few_codes_of_any_table(d, bits, prod, n):
    p, codes, parts, norm = make(bits, prod, n, d)
    wide = torch.full((n + 1, d + 4), 7.0, device=T.DEV)
    tq.tq_dequantize(p, *codes, T.dev(norm), wide[:n, :d])
    assert bool((wide[:n, d:] == 7).all()) and bool((wide[n] == 7).all())
    T.P.check_close(wide[:n, :d].cpu().numpy(), reference(parts, prod, norm), norm.astype(np.float64)[:, None] / np.sqrt(d), "coordinate")


@pytest.mark.parametrize("d,n", [(128, 100), (128, 8200), (256, 5000)])
def test_images_without_digits(d, n):
    """TQ_FLAG_DEQUANT_IMAGES alone: images that end before the digits (made so here: the buffer is cut there), and the kernels that do without."""
    from paper_2504_19874_amd import _lib
    p, codes, parts, norm = make(2, True, n, d)
    out = torch.empty((n, d), device=T.DEV)
    whole = p.images
    sign_bytes = 2 * ((d // 64) * (d // 32) * 5 * 1536 + 512) if d == 128 else 8 * d * d
    cut = torch.empty(int(tq.tq_images_bytes(d)) + int(_lib.load().tq_dequant_images_bytes(d)) - sign_bytes, dtype=torch.uint8, device=T.DEV)
    cut.copy_(torch.as_strided(whole, (cut.numel(),), (1,)))
    try:
        p.images, p.c.images = cut, cut.data_ptr()
        p.c.flags &= ~_lib.TQ_FLAG_SIGN_IMAGES
        tq.tq_dequantize(p, *codes, T.dev(norm), out)
    finally:
        p.build_images()
    assert p.c.flags & _lib.TQ_FLAG_SIGN_IMAGES
    T.P.check_close(out.cpu().numpy(), reference(parts, True, norm), norm.astype(np.float64)[:, None] / np.sqrt(d), "coordinate")


@pytest.mark.parametrize("bits,prod,n", [(0, True, 5), (1, False, 4097), (2, True, 300), (2, False, 16000), (2, True, 24576), (2, True, 40000), (3, True, 1000)])
def test_workspace_is_left_alone_at_128(bits, prod, n):
    """Two streams may dequantise with one parameter set at d = 128: without images nothing that they share is written."""
    p, codes, parts, norm = make(bits, prod, n)
    out = torch.empty((n, D), device=T.DEV)
    try:
        p.drop_images().reserve(n)
        p.workspace.fill_(0x5a)
        tq.tq_dequantize(p, *codes, T.dev(norm), out)
        assert bool((p.workspace == 0x5a).all())
        keep = p.c.workspace, p.c.workspace_bytes
        p.c.workspace, p.c.workspace_bytes = 0, 0  # nor needed
        again = torch.empty_like(out)
        tq.tq_dequantize(p, *codes, T.dev(norm), again)
        p.c.workspace, p.c.workspace_bytes = keep
        assert torch.equal(out, again)
    finally:
        p.build_images()
    T.P.check_close(out.cpu().numpy(), reference(parts, prod, norm), norm.astype(np.float64)[:, None] / np.sqrt(D), "coordinate")


@pytest.mark.parametrize("d,bits,prod,matrices", [(256, 4, False, 0), (256, 3, True, 0), (256, 2, False, 1), (256, 1, True, 2), (128, 4, False, 0), (128, 2, False, 1),
                                                  (128, 2, True, 2), (320, 2, True, 0)])
def test_digits_only_where_a_call_can_take_them(d, bits, prod, matrices):
    """A parameter set's images hold the digits of the matrices that its own table lets tq_dequantize multiply, and of no others."""
    from paper_2504_19874_amd import _lib
    p = T.setup(d, bits, prod)[0]
    one = (d // 64) * (d // 32) * 5 * 1536 + 512 if d == 128 else 4 * d * d
    most = int(_lib.load().tq_dequant_images_bytes(d)) - (2 * one if d % 128 == 0 else 0)
    assert p.images.untyped_storage().nbytes() == int(tq.tq_images_bytes(d)) + most + matrices * one


def test_images_for_any_table():
    """tq_build_dequant_images fills the whole buffer, whatever the table of the parameter set it is called with: the images are those of
    the matrices, and a set with another table may use them."""
    import ctypes
    from paper_2504_19874_amd import _lib
    lib = _lib.load()
    for d in (128, 256):
        four, codes, parts, norm = make(2, True, 3000, d)
        want, got = torch.empty((3000, d), device=T.DEV), torch.empty((3000, d), device=T.DEV)
        tq.tq_dequantize(four, *codes, T.dev(norm), want)
        other = T.setup(d, 4, True)[0]  # (the same Pi and S)
        size = int(tq.tq_images_bytes(d)) + int(lib.tq_dequant_images_bytes(d))
        whole = torch.zeros(size, dtype=torch.uint8, device=T.DEV)
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert lib.tq_build_images(ctypes.byref(other.c), ctypes.c_void_p(whole.data_ptr()), stream) == 0
        assert lib.tq_build_dequant_images(ctypes.byref(other.c), ctypes.c_void_p(whole.data_ptr()), stream) == 0
        keep = four.c.images
        try:
            four.c.images = whole.data_ptr()
            tq.tq_dequantize(four, *codes, T.dev(norm), got)
        finally:
            four.c.images = keep
        assert torch.equal(got, want)


def run(p, codes, norm, n, d):
    out = torch.empty((n, d), device=T.DEV)
    tq.tq_dequantize(p, *codes, T.dev(norm), out)
    return out.cpu().numpy()


@pytest.mark.parametrize("d,bits,prod,n", [(128, 0, True, 70), (128, 2, True, 300), (128, 1, False, 8200), (128, 2, True, 9000), (256, 1, True, 65), (640, 2, True, 300),
                                           (256, 0, True, 5000)])
@pytest.mark.parametrize("images", [True, False])
def test_factors_that_are_not_finite(d, bits, prod, n, images):
    """A code's own coordinates are not finite then, and nothing else is touched by it."""
    p, codes, parts, norm = make(bits, prod, n, d)
    try:
        if not images:
            p.drop_images().reserve(n)
        want = run(p, codes, norm, n, d)
        bad = np.zeros(n, dtype=bool)
        norm = norm.copy()
        for k, v in enumerate((np.inf, np.nan, -np.inf)):
            norm[7 + 20 * k] = v
            bad[7 + 20 * k] = True
            if prod:
                codes[2][5 + 20 * k] = float(v)
                bad[5 + 20 * k] = True
        got = run(p, codes, norm, n, d)
    finally:
        p.build_images()
    assert np.isfinite(want).all() and not np.isfinite(got[bad]).any()
    assert np.array_equal(got[~bad], want[~bad])


@pytest.mark.parametrize("d,bits,prod,n", [(128, 2, True, 300), (128, 0, True, 40), (128, 1, False, 9000), (256, 2, True, 700), (384, 1, True, 65), (256, 0, True, 100)])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 0.0])
@pytest.mark.parametrize("images", [True, False])
def test_columns_that_are_not_finite_or_zero(d, bits, prod, n, value, images):
    """An entry of Pi or S that is not finite makes that output of every code not finite, and a column of zeros leaves it to the other
    matrix; the other outputs do not change."""
    p0, codes, (idx, z, gamma, Pi, S, c), norm = make(bits, prod, n, d)
    want = run(p0, codes, norm, n, d)
    Pi, S = Pi.copy(), S.copy() if prod else None
    hit = np.zeros(d, dtype=bool)
    for M, cols in ((Pi if bits else None, (3, 70)), (S, (9, 70))):
        if M is not None:
            for k in cols:
                if value == 0.0:
                    M[:, k] = 0.0
                else:
                    M[(5 * k) % d, k] = value
                hit[k] = True
    p = tq.Params(d, bits, torch.from_numpy(Pi), torch.from_numpy(S) if prod else None, p0.centroids, p0.bounds)
    if not images:
        p.drop_images().reserve(n)
    got = run(p, codes, norm, n, d)
    assert np.array_equal(got[:, ~hit], want[:, ~hit])
    if value != 0.0:
        assert not np.isfinite(got[:, hit]).any()
        return
    exact = reference((idx, z, gamma, Pi, S, c), prod, norm)
    assert np.all(got[:, 70] == 0.0)
    close(got[:, hit], exact[:, hit], norm, n)


@pytest.mark.parametrize("bits,prod,n", [(2, True, 70), (1, True, 513), (0, True, 100), (2, False, 400)])
def test_the_longest_stored_vectors(bits, prod, n):
    """d = 3072, where an entry of S is 55 times one of Pi and the sums of the two are joined in units of the one."""
    test_long_codes(3072, bits, prod, n)
