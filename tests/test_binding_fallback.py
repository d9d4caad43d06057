"""The binding without its compiled half, which belongs to one Python and one torch build."""
import sys

import pytest
import torch

from paper_2504_19874_amd import _lib, api


@pytest.fixture
def no_call_lib(monkeypatch):
    import paper_2504_19874_amd
    monkeypatch.setitem(sys.modules, "paper_2504_19874_amd._tqcall", None)  # an import of it fails
    monkeypatch.delattr(paper_2504_19874_amd, "_tqcall", raising=False)
    monkeypatch.setattr(_lib, "_call", None)


def test_calls_take_the_checked_path(no_call_lib):
    class P:
        c, d, idx_words, qjl_words, scalars_per_vector = _lib.TqParams(), 128, 8, 4, 1

    x = torch.zeros(4, 128)
    with pytest.warns(RuntimeWarning, match="_tqcall"):
        with pytest.raises(api.TurboQuantError, match="GPU tensor"):
            api.tq_quantize_mse(P, x, torch.zeros(4, 8, dtype=torch.int32), None)
    with pytest.raises(api.TurboQuantError, match="qjl"):
        api.tq_quantize_prod(P, x, torch.zeros(4, 8, dtype=torch.int32), torch.zeros(4, 3, dtype=torch.int32), torch.zeros(4), None)


@pytest.mark.gpu
def test_the_checked_path_gives_the_same(no_call_lib):
    from tests import test_gpu_attend as A
    from tests import test_gpu_kernel_edges as K
    from tests import test_gpu_parity as T
    with pytest.warns(RuntimeWarning, match="_tqcall"):
        T.test_quantize_prod(128, 2, 100, "bf16")
    T.test_quantize_mse(256, 3, 100, "f32")
    K.test_dequantiser_tiles(96, 4, 63, True)
    K.test_few_queries_at_multiples_of_128(640, 2, True, 1, 3, 257, 3)
    A.run_attend(128, 2, True, 2, False, 1, 4, 511, True)
