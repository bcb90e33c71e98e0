"""From the compiler's resource report of the last build: no rollout kernel uses
scratch, and the kernels that run all bins in one launch keep two waves per
SIMD by their registers and their LDS areas.
"""
import json
import os

import pytest

from paper_2502_11129_amd import build as B

CU_LDS = 160 * 1024


def _report():
    path = os.path.join(B.BUILD, B.RESOURCES)
    if not os.path.exists(path):
        pytest.skip("no resource report: run build() first")
    with open(path) as f:
        return json.load(f)


def test_no_rollout_kernel_uses_scratch():
    kernels = {n: r for n, r in _report().items() if "14rollout_kernelI" in n or "rollout_multi_kernel" in n}
    assert len(kernels) >= 36
    assert {n: r["ScratchSize [bytes/lane]"] for n, r in kernels.items() if r["ScratchSize [bytes/lane]"]} == {}


def test_the_one_launch_keeps_two_waves_per_simd():
    kernels = [r for n, r in _report().items() if "rollout_multi_kernel" in n]
    assert len(kernels) == 2
    for r in kernels:
        assert r["Occupancy [waves/SIMD]"] >= 2
        assert r["LDS Size [bytes/block]"] * 4 * 2 <= CU_LDS
