"""The quantiser on two fp16 pieces per factor (every d other than 128): edges of its three tile sizes, one- and two-step
k-loops, an odd number of k-steps, passes cut by a small workspace, and rows whose magnitudes differ widely."""
import numpy as np
import pytest
import torch

from oracle import turboquant_oracle as o
from tests import parity as P
from tests import test_gpu_parity as T

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")


@pytest.mark.parametrize("d,bits,n,kind", [
    (32, 2, 1, "f32"), (64, 4, 63, "f32"), (96, 3, 65, "bf16"), (160, 1, 257, "unit"), (288, 4, 127, "bf16unit"),
    (384, 2, 4097, "f32"), (512, 4, 3000, "bf16"), (544, 3, 1025, "f32"), (768, 1, 20000, "f32"), (1536, 4, 8193, "unit"),
])
def test_indices(d, bits, n, kind):
    T.test_quantize_mse(d, bits, n, kind)


@pytest.mark.parametrize("d,bits_mse,n,kind", [
    (32, 1, 33, "bf16"), (64, 0, 129, "f32"), (96, 4, 4095, "f32"), (224, 2, 257, "bf16unit"), (320, 3, 1000, "f32"),
    (512, 1, 9000, "bf16"), (768, 2, 5000, "unit"), (1536, 4, 700, "f32"),
])
def test_residual_and_sketch(d, bits_mse, n, kind):
    T.test_quantize_prod(d, bits_mse, n, kind)


@pytest.mark.parametrize("d,bits_mse,n", [(256, 2, 3001), (544, 1, 1300)])
def test_workspace_that_holds_only_a_part(d, bits_mse, n):
    """The same codes whatever the number of passes, and from the kernel that needs none of the pieces' room."""
    p, Pi, S, c32, t32 = T.setup(d, bits_mse, True)
    x_or, x_dev, normalise = T._quant_inputs(n, d, "f32", 3)
    keep = (p.workspace, p.c.workspace, p.c.workspace_bytes)
    try:
        whole = T._run_prod(p, x_dev, n, normalise)
        T._check_prod(p, Pi, S, c32, t32, x_or, normalise, *whole)
        for rows in (600, 0):
            p.workspace, p.c.workspace, p.c.workspace_bytes = None, 0, 0
            p.reserve_bytes(rows * (8 * d + 8 + (d + 63) // 64 * 4) + 8192 if rows else 128 * d * 4 + 512)
            out = [torch.zeros_like(t) for t in whole]
            tq.tq_quantize_prod(p, x_dev, *out)
            T._check_prod(p, Pi, S, c32, t32, x_or, normalise, *out)
            if rows:
                assert all(torch.equal(a, b) for a, b in zip(out, whole))
    finally:
        p.workspace, p.c.workspace, p.c.workspace_bytes = keep


def test_rows_of_any_magnitude():
    """Row scales are powers of two taken from each row's largest value: rows from 1e-15 to 1e15, single spikes, and
    values that vanish beside the row's largest."""
    d, bits_mse, n = 192, 2, 400
    p, Pi, S, c32, t32 = T.setup(d, bits_mse, True)
    rng = np.random.default_rng(8)
    x = rng.standard_normal((n, d)) * np.exp(rng.uniform(np.log(1e-15), np.log(1e15), size=(n, 1)))
    x[::5, 7] *= 1e4
    x[1::5] *= np.exp(rng.uniform(-20, 0, size=x[1::5].shape))
    x = x.astype(np.float32)
    x[3] = 0.0
    out = T._run_prod(p, T.dev(x), n, True)
    T._check_prod(p, Pi, S, c32, t32, x, True, *out)
    y = o.rotate(o.unit_normalise(x, True)[0], Pi)
    P.check_indices(o.unpack_planes(T.words(out[0])[:, : p.idx_words], bits_mse, d), o.nearest_centroid(y, t32), y, t32)
