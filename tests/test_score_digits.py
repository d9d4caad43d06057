"""The fixed-point arithmetic of few-query scoring at the ends of its range."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_digit_sums_on_the_host(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "score_digits")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host", "score_digits.cpp"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "digits ok" in r.stdout and r.stderr == "", r.stdout + r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("d,bits,prod", [(3072, 1, True), (4096, 1, False), (2048, 4, True), (4096, 2, True)])
def test_flat_rotated_queries(d, bits, prod):
    """A caller who rotates beforehand passes Pi = I; rotated coordinates that are all alike make the largest masked sums:
    within 2^-20 of a coordinate (the query's rounding) and the rounding of the fp32 result of the exact ones."""
    tq = pytest.importorskip("paper_2504_19874_amd")
    c, t, _ = tq.tq_build_codebook(d, bits)
    eye = torch.eye(d)
    p = tq.Params(d, bits, eye, eye if prod else None, c, t)
    n, rng = 96, np.random.default_rng(d + bits)
    index = rng.integers(0, 1 << bits, size=(n, d))
    index[:32] = (1 << bits) - 1
    index[32:64] = 0
    planes = ((index.reshape(n, d // 32, 1, 32) >> np.arange(bits).reshape(1, 1, bits, 1)) & 1).astype(np.uint64)
    idx = (planes << np.arange(32, dtype=np.uint64)).sum(-1).astype(np.uint32).reshape(n, -1)
    sign = rng.integers(0, 2, size=(n, d))
    sign[::3], sign[1::3] = 1, 0
    qjl = (sign.reshape(n, d // 32, 32).astype(np.uint64) << np.arange(32, dtype=np.uint64)).sum(-1).astype(np.uint32)
    q = np.stack([np.full(d, 0.99), np.full(d, -0.99), np.ones(d), rng.choice([-1.0, 0.999], size=d)]).astype(np.float32)
    gamma = np.full(n, 0.5, dtype=np.float32)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()  # noqa: E731
    p.reserve_score(1, 4, n, prod, True)
    got = torch.zeros(4, n, device="cuda")
    tq.tq_score(p, dev(q), 1, 4, dev(idx.view(np.int32)), dev(qjl.view(np.int32)) if prod else None, dev(gamma) if prod else None, None, n, got)
    kg = np.sqrt(np.pi / 2) / d * 0.5
    parts = [np.float64(c)[index]] + ([kg * (2.0 * sign - 1)] if prod else [])
    want = sum(np.float64(q) @ a.T for a in parts)
    # a coordinate is rounded to 2^-20 of the largest one (half a unit); the sums of a score, a dozen roundings of 2^-24 of up to
    # the size, come to less than that again
    size = sum(np.abs(np.float64(q)) @ np.abs(a).T for a in parts)
    assert np.all(np.abs(got.cpu().numpy() - want) <= 2.0**-19 * size), np.max(np.abs(got.cpu().numpy() - want) / size)
