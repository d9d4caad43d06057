"""bench.py prices a call by the products that the library executes for it; this pins them to the kernels' own numbers."""
import pytest

import bench
import workloads as W


@pytest.mark.parametrize("name,products", [("C1", (3, 3, 0)), ("C2", (2.5, 2.5, 0)), ("C3", (2.5, 2.5, 0)), ("C4", (3, 3, 1)), ("C5", (3, 2, 1))])
def test_piece_products(name, products):
    cfg = W.CONFIGS[name]
    calls = ("quantize", "dequantize", "score")
    got = tuple(bench.piece_products(cfg, c) for c in calls)
    if cfg.d == 128 and cfg.n * cfg.n_groups <= 8192:
        products = (0, 0, 0)  # the fp32 kernels
    assert got == products
    for c, k in zip(calls, got):
        assert ("MFMA" in bench.arithmetic(cfg)[c]) == (k > 0 or c == "score")
        assert ("pieces" in bench.path_dtype(cfg).split("; ")[calls.index(c)]) == (k > 0)


def test_no_call_executes_more_than_the_peak():
    """C4's search at the rate it was once reported with three products: 1.04 of the chip's peak; it executes one."""
    r = bench.call_roofline(W.CONFIGS["C4"], "score", 3.55)
    assert r["executed_frac"] == pytest.approx(r["frac"]) and r["executed_frac"] < 0.4
