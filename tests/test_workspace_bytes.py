"""tq_workspace_bytes against what the quantiser's routes take, on the host: the library's sizes need no GPU."""
import ctypes as C

import pytest

from paper_2504_19874_amd import _lib


@pytest.mark.parametrize("d,n,prod", [(512, 64, True), (4096, 3, True), (4096, 64, False), (1536, 64, True), (128, 1, False)])
def test_few_vectors(d, n, prod):
    """The fp16 contraction's pieces (8 d + 8 bytes and the partial residual norms a vector) are more than the residuals of the matrix-vector
    route (4 d), and only one of the two runs: nothing is asked for beside them but the alignment of five arrays."""
    p = _lib.TqParams()
    p.d, p.bits_mse = d, 2
    p.S = 256 if prod else 0  # (only asked whether it is there)
    p.images = 256
    got = _lib.load().tq_workspace_bytes(C.byref(p), n, 0, 0)
    need = n * (8 * d + 8 + (d + 63) // 64 * 4)
    assert need <= got <= need + 8192


@pytest.mark.parametrize("d,most,prod", [(64, 1024, True), (256, 256, False), (384, 170, True), (768, 85, False), (1536, 64, True), (4096, 64, False)])
def test_no_room_to_split_queries_that_matrix_vector_products_rotate(d, most, prod):
    """Up to 64 queries, and short ones up to 65536 values, need their rotation's result alone; from the next on pieces and two images, too."""
    c, t = (C.c_float * 4)(-1, -0.5, 0.5, 1), (C.c_float * 3)(-0.75, 0, 0.75)
    p = _lib.TqParams()
    p.d, p.bits_mse, p.S = d, 2, 256 if prod else 0
    p.centroids, p.bounds = C.addressof(c), C.addressof(t)
    lib = _lib.load()
    result = lambda nq: nq * d * 4 * (2 if prod else 1)  # noqa: E731
    call = lambda nq: lib.tq_score_workspace_bytes(C.byref(p), 1, nq, 1 << 20, int(prod), 1, 0)  # noqa: E731
    assert call(most) <= result(most) + 2048
    assert call(most + 1) >= result(most + 1) + (most + 1) * d * 4 + (2 if prod else 1) * 4 * d * d
    bound = lambda nq: lib.tq_workspace_bytes(C.byref(p), 0, nq, 0)  # noqa: E731
    assert bound(most + 1) - bound(most) >= (most + 1) * d * 4 + (2 if prod else 1) * 4 * d * d


@pytest.mark.parametrize("rows,n,topk,chunks", [
    (128, 41000, 10, 0), (129, 200000, 10, 0), (128, 40960, 64, 0), (100, 41000, 64, 3),  # one workgroup per row
    (43, 60000, 16, 4), (4, 1000000, 10, 62), (1, 4000000, 64, 64),  # a segment of 1024 threads each; no more pairs than are joined in one go
    (43, 131072, 10, 16), (5, 1000000, 1, 123), (65, 66000, 16, 9),  # of 512 threads, three to a compute unit at most
    (43, 131072, 17, 8), (64, 131072, 10, 8), (86, 131072, 10, 8),  # of 1024 threads, two to a compute unit, or 512 threads in two steps
    (128, 200000, 10, 4), (33, 1000000, 64, 15),  # two workgroups to a compute unit
])
def test_lists_of_a_top_k_over_chunks(rows, n, topk, chunks):
    """As many chunks of a row as are all at work at once on 256 compute units: each has a list of topk pairs."""
    c, t = (C.c_float * 4)(-1, -0.5, 0.5, 1), (C.c_float * 3)(-0.75, 0, 0.75)
    p = _lib.TqParams()
    p.d, p.bits_mse = 128, 2
    p.centroids, p.bounds = C.addressof(c), C.addressof(t)
    call = lambda k: _lib.load().tq_score_workspace_bytes(C.byref(p), rows, 1, n, 0, 1, k)  # noqa: E731
    assert call(topk) - call(0) == 2 * ((rows * chunks * topk * 4 + 255) // 256 * 256)
