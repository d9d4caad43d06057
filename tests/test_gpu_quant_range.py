"""Residuals of any size at d = 128: rows that are taken as given (no norm) may be far longer than 1, and a caller's table may hold
centroids far from a unit vector's coordinates.  The sketch's operands are 16-bit pieces of the residual; its signs have to be those of the residual all the same."""
import numpy as np
import pytest
import torch

from oracle import turboquant_oracle as o
from tests import parity as P
from tests import test_gpu_parity as T

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")

D = 128


def quantise(p, x, n, normalise):
    k = p.scalars_per_vector
    out = [torch.zeros((n, max(1, p.idx_words)), dtype=torch.int32, device=T.DEV), torch.zeros((n, p.qjl_words), dtype=torch.int32, device=T.DEV),
           torch.zeros(n * k, device=T.DEV), torch.zeros(n * k, device=T.DEV) if normalise else None]
    tq.tq_quantize_prod(p, x, *out)
    return out


def as_input(x, dtype):
    if dtype == "f32":
        return x, T.dev(x)
    bits = T.W.f32_to_bf16_bits(x)
    return o.bf16_bits_to_f64(bits), T.bf16_tensor(bits)


@pytest.mark.parametrize("images", [True, False])
@pytest.mark.parametrize("dtype,bits,n", [("bf16", 2, 40), ("bf16", 0, 1000), ("bf16", 1, 3000), ("bf16", 3, 24600), ("f32", 1, 8200), ("f32", 2, 700)])
def test_rows_taken_as_given(dtype, bits, n, images):
    """Rows from 1 to 10^12 long: the residual passes 1024, where 64 times it leaves the range of fp16, from the second decade on."""
    p, Pi, S, c32, t32 = T.setup(D, bits, True)
    rng = np.random.default_rng(n + bits)
    x = (rng.standard_normal((n, D)) * 10.0 ** rng.uniform(-1, 11, size=(n, 1))).astype(np.float32)
    x[1] = 0.0
    x[2, 1:] = 0.0  # one coordinate only
    x_or, x_dev = as_input(x, dtype)
    try:
        if not images:
            p.drop_images()
        idx, qjl, gamma, _ = quantise(p, x_dev, n, False)
    finally:
        p.build_images()
    y = np.float64(x_or) @ np.float64(Pi).T
    got = o.unpack_planes(T.words(idx)[:, : p.idx_words], bits, D) if bits else np.zeros((n, D), dtype=np.int64)
    e = y - np.asarray(c32, dtype=np.float64).reshape(-1)[got]
    P.check_close(gamma.cpu().numpy(), np.linalg.norm(e, axis=1), 0.0, "gamma", rel=1e-5)
    scale = np.linalg.norm(np.float64(S), axis=1)[None, :] * np.linalg.norm(e, axis=1)[:, None]
    P.check_signs(o.unpack_signs(T.words(qjl), D), e @ (np.float64(S) @ np.float64(Pi).T).T, scale)


@pytest.mark.parametrize("table", [(-3000.0, 3000.0), (-5e4, -0.07, 0.07, 5e4)])
@pytest.mark.parametrize("dtype,n", [("bf16", 40), ("bf16", 24600), ("f32", 8200)])
def test_tables_beyond_the_unit_ball(table, dtype, n):
    c = np.array(table, dtype=np.float32)
    t = (c[1:] + c[:-1]) / 2
    p0, Pi, S, _, _ = T.setup(D, 2, True)
    p = tq.Params(D, int(np.log2(c.size)), p0.Pi, p0.S, c, t)
    x = T.W.unit_gaussian_rows(n, D, 5)
    if c.size == 4:
        x[::2] *= 1e-3
    x_or, x_dev = as_input(x, dtype)
    idx, qjl, gamma, _ = quantise(p, x_dev, n, True)
    y = o.unit_normalise(x_or)[0] @ np.float64(Pi).T
    got = o.unpack_planes(T.words(idx), p.bits_mse, D)
    P.check_indices(got, o.nearest_centroid(y, t), y, t)
    e = y - np.float64(c)[got]
    P.check_close(gamma.cpu().numpy(), np.linalg.norm(e, axis=1), 0.0, "gamma", rel=1e-5)
    scale = np.linalg.norm(np.float64(S), axis=1)[None, :] * np.linalg.norm(e, axis=1)[:, None]
    P.check_signs(o.unpack_signs(T.words(qjl), D), e @ (np.float64(S) @ np.float64(Pi).T).T, scale)


@pytest.mark.parametrize("n", [40, 24600])
def test_two_instances_of_such_a_table(n):
    d_hi, gs = 64, 2
    Pi, S = np.zeros((D, D)), np.zeros((D, D))
    for b in range(2):
        at = slice(64 * b, 64 * b + 64)
        Pi[at, at] = o.rotation_from_gaussian(T.W.gaussian_matrix(64, 70 + b))
        S[at, at] = T.W.sketch_matrix(64, 80 + b)
    Pi, S = Pi.astype(np.float32), S.astype(np.float32)
    lo, hi = np.array([-2500.0, 2500.0], dtype=np.float32), np.array([-2500.0, -0.1, 0.1, 2500.0], dtype=np.float32)
    mid = lambda c: (c[1:] + c[:-1]) / 2  # noqa: E731
    p = tq.Params(D, 1, torch.from_numpy(Pi), torch.from_numpy(S), lo, mid(lo), d_hi=d_hi, bits_mse_hi=2, centroids_hi=hi, bounds_hi=mid(hi))
    x_or, x_dev = as_input(T.W.unit_gaussian_rows(n, D, 6), "bf16")
    idx, qjl, gamma, norm = quantise(p, x_dev, n, True)
    w = T.words(idx)
    for b, (c, bits, words) in enumerate([(hi, 2, w[:, : 2 * gs]), (lo, 1, w[:, 2 * gs:])]):
        at = slice(64 * b, 64 * b + 64)
        y = o.unit_normalise(x_or[:, at])[0] @ np.float64(Pi[at, at]).T
        got = o.unpack_planes(np.ascontiguousarray(words), bits, 64)
        P.check_indices(got, o.nearest_centroid(y, mid(c)), y, mid(c))
        e = y - np.float64(c)[got]
        g = np.linalg.norm(e, axis=1)
        P.check_close(gamma.cpu().numpy().reshape(n, 2)[:, b], g, 0.0, "gamma", rel=1e-5)
        z = o.unpack_signs(np.ascontiguousarray(T.words(qjl)[:, 2 * b: 2 * b + 2]), 64)
        P.check_signs(z, e @ (np.float64(S[at, at]) @ np.float64(Pi[at, at]).T).T, np.linalg.norm(np.float64(S[at, at]), axis=1)[None, :] * g[:, None])
