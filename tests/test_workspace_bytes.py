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
