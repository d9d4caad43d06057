"""bf16 vectors at d = 128 in batches too small for the kernel that keeps its matrices in LDS: blocks of 16 vectors, shared by
up to eight workgroups while they leave compute units idle, two and more per workgroup at the other end."""
import pytest
import torch

from tests import test_gpu_parity as T
from tests import test_gpu_split as S

pytestmark = pytest.mark.gpu

tq = pytest.importorskip("paper_2504_19874_amd")


@pytest.mark.parametrize("bits,n,kind", [(1, 1, "bf16unit"), (2, 512, "bf16"), (3, 513, "bf16"), (4, 1040, "bf16unit"), (0, 2065, "bf16"),
                                         (2, 8193, "bf16unit"), (3, 24576, "bf16"), (1, 24577, "bf16")])
def test_blocks_and_shares(bits, n, kind):
    T.test_quantize_prod(128, bits, n, kind)
    if bits:
        T.test_quantize_mse(128, bits, n, kind)


# matrix-vector products of short vectors: fewer values than lanes, not a multiple of them, blocks of four in part; the ends of the range with and without a
# sketch, one beyond
@pytest.mark.parametrize("d,bits,n,kind", [(32, 3, 1, "f32"), (32, 2, 256, "bf16"), (64, 4, 257, "unit"), (96, 3, 7, "bf16unit"), (160, 1, 65, "f32"), (256, 4, 128, "bf16"),
                                           (256, 2, 129, "f32"), (256, 3, 256, "unit"), (384, 2, 85, "bf16"), (384, 3, 170, "f32"), (768, 1, 64, "unit"), (1536, 2, 52, "f32"), (1536, 2, 53, "bf16"),
                                           (1536, 3, 61, "f32")])
def test_short_vectors(d, bits, n, kind):
    T.test_quantize_prod(d, bits, n, kind)
    T.test_quantize_mse(d, bits, n, kind)


# tiles of 32 vectors: one and several, the last in part, the ends of the range (256 compute units); of long vectors one tile of 64 or two of 32
@pytest.mark.parametrize("d,bits,n,kind", [(512, 2, 65, "f32"), (512, 4, 1024, "bf16"), (512, 1, 1025, "unit"), (1088, 3, 288, "bf16unit"), (1088, 2, 257, "f32"), (2560, 1, 97, "bf16"),
                                           (2080, 2, 96, "f32"), (2080, 1, 56, "bf16"), (2080, 3, 57, "unit"), (2080, 2, 57, "bf16unit"), (2560, 1, 33, "f32")])
def test_tiles_of_32(d, bits, n, kind):
    T.test_quantize_prod(d, bits, n, kind)
    T.test_quantize_mse(d, bits, n, kind)


# d = 128, fp32: as many as go by products, and one more
@pytest.mark.parametrize("bits,n,kind", [(4, 1, "f32"), (1, 63, "unit"), (2, 64, "f32"), (3, 65, "f32"), (4, 256, "unit"), (0, 31, "f32"), (3, 257, "f32")])
def test_fp32_vectors_at_128(bits, n, kind):
    T.test_quantize_prod(128, bits, n, kind)
    T.test_quantize_mse(128, bits, n, kind)


@pytest.mark.parametrize("bits,n,bf16", [(2, 1, False), (1, 64, False), (2, 65, False), (3, 257, False), (0, 33, False), (2, 1, True), (3, 64, True), (1, 257, True)])
def test_workspace_is_left_alone_at_128(bits, n, bf16):
    """Two streams may quantise, or one of them score, with one parameter set at d = 128: nothing that they share is written, or needed."""
    p = T.setup(128, bits, True)[0]
    x = torch.randn(n, 128, generator=torch.Generator().manual_seed(n)).to(torch.bfloat16 if bf16 else torch.float32).to(T.DEV)
    p.reserve(n).workspace.fill_(0x5a)
    keep = p.c.workspace, p.c.workspace_bytes

    def run(prod):
        c = [torch.zeros((n, max(1, p.idx_words)), dtype=torch.int32, device=T.DEV), torch.zeros((n, p.qjl_words), dtype=torch.int32, device=T.DEV),
             torch.zeros(n, device=T.DEV), torch.zeros(n, device=T.DEV)]
        if prod:
            tq.tq_quantize_prod(p, x, *c)
        else:
            tq.tq_quantize_mse(p, x, c[0], c[3])
        return c

    for prod in (False, True):
        want = run(prod)
        assert bool((p.workspace == 0x5a).all())
        try:
            p.c.workspace, p.c.workspace_bytes = 0, 0
            again = run(prod)
        finally:
            p.c.workspace, p.c.workspace_bytes = keep
        assert all(torch.equal(a, b) for a, b in zip(want, again))


# short vectors beyond 16384: the contraction that splits them on the fly
@pytest.mark.parametrize("d,bits,n,kind", [(64, 3, 16385, "bf16"), (64, 3, 32769, "f32"), (64, 4, 20001, "f32"), (192, 3, 16400, "unit"), (256, 4, 17003, "bf16"), (384, 4, 16385, "f32"),
                                           (256, 2, 16385, "f32")])
def test_many_short_vectors(d, bits, n, kind):
    T.test_quantize_mse(d, bits, n, kind)


@pytest.mark.parametrize("d_hi,bits_lo,prod,n", [(64, 1, True, 513), (32, 3, True, 8209), (96, 0, False, 33), (96, 2, False, 24576)])
def test_two_instances(d_hi, bits_lo, prod, n):
    S.test_quantize_split(d_hi, bits_lo, prod, n, True)


@pytest.mark.parametrize("bits,prod,n", [(2, True, 8), (4, False, 100), (3, True, 9000)])
def test_without_images_and_scattered(bits, prod, n):
    """The matrices split in the kernel, and rows written `step` apart: the same bits."""
    p = T.setup(128, bits, prod)[0]
    x = (torch.randn(n, 128, generator=torch.Generator().manual_seed(n)) * 3).to(torch.bfloat16).to(T.DEV)
    x[n // 2] = 0  # a zero row stays zero
    first, step = 5, 3

    def run(scattered):
        rows = first + step * n if scattered else n
        c = [torch.full((rows, p.idx_words), 7, dtype=torch.int32, device=T.DEV), torch.full((rows, p.qjl_words), 7, dtype=torch.int32, device=T.DEV),
             torch.full((rows,), 7.0, device=T.DEV), torch.full((rows,), 7.0, device=T.DEV)]
        if not prod:
            c[1] = c[2] = None
        if scattered:
            tq.tq_append(p, x, *c, first, step)
            at = first + step * torch.arange(n, device=T.DEV)
            others = torch.ones(rows, dtype=torch.bool, device=T.DEV)
            others[at] = False
            assert all(bool((v[others] == 7).all()) for v in c if v is not None)
            return [v[at] for v in c if v is not None]
        if prod:
            tq.tq_quantize_prod(p, x, *c)
        else:
            tq.tq_quantize_mse(p, x, c[0], c[3])
        return [v for v in c if v is not None]

    want = run(False)
    assert float(want[-1][n // 2]) == 0.0
    assert all(torch.equal(a, b) for a, b in zip(want, run(True)))
    try:
        p.drop_images()
        assert all(torch.equal(a, b) for a, b in zip(want, run(False)))
    finally:
        p.build_images()
