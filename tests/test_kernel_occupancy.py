"""Waves per SIMD of the rollout kernels, from the compiler's resource report
of the last build and the size of their LDS areas (160 KB per CU, four SIMDs):
two waves for every plane and self-collision family of 20 DoFs and more with at
most 8 contacts in registers, three for the smaller ones."""
import json
import os
import re

import pytest

from paper_2502_11129_amd import build as B

PAT = re.compile(r"rollout_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb([01])ELb([01])ELb([01])E")
CU_LDS = 160 * 1024


def _expected(nvc, ncr, ball, self_):
    if nvc > 16:
        return 1 if ncr > 8 or (ball and nvc > 24) else 2
    return 2 if ncr > 8 else 3


def test_registers_and_lds_allow_the_waves_per_simd():
    path = os.path.join(B.BUILD, B.RESOURCES)
    if not os.path.exists(path):
        pytest.skip("no resource report: run build() first")
    with open(path) as f:
        rep = json.load(f)
    seen = 0
    for name, r in rep.items():
        m = PAT.search(name)
        if not m:
            continue
        nvc, sb, ncr, ball, self_, tree = (int(x) for x in m.groups())
        if tree:
            continue
        waves = _expected(nvc, ncr, ball, self_)
        assert r["Occupancy [waves/SIMD]"] >= waves, (m.groups(), r)
        assert r["LDS Size [bytes/block]"] * 4 * waves <= CU_LDS, (m.groups(), r)
        seen += 1
    assert seen >= 30
