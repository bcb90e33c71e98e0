"""Features at the edges of the 64-candidate tiles, for chains of depth 20, all
limbs at the core, single hinges, invalid rows and arrays off their natural
alignment: bit for bit the oracle's, nothing written past the last row."""
import numpy as np
import pytest
import torch

from oracle import mlp_oracle as M
from paper_2502_11129_amd import workloads as W
from paper_2502_11129_amd.surrogate import Surrogate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1, 4])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 1000])
def test_features_at_tile_edges(n, shift):
    g = W.random_genotypes(n, key=n)
    for i in range(0, n, 5):                       # chain, star, one hinge
        g.nh[i] = (20, 20, 1)[(i // 5) % 3]
        g.parent[i] = np.arange(20) if (i // 5) % 3 == 0 else 0
        g.face[i], g.axis[i] = np.arange(20) % 4, np.arange(20) % 2
        g.cpg[i] = np.random.default_rng(i).normal(0, 4, (20, 3))
    bad = np.arange(3, n, 17)
    ok = np.setdiff1d(np.arange(n), bad)
    ref = (M.bf16(M.features(g)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    for k, i in enumerate(bad):
        last = int(g.nh[i]) - 1
        if k % 5 == 0:
            g.nh[i] = (0, 21, -1)[(k // 5) % 3]
        elif k % 5 == 1:
            g.parent[i, last] = last + 1
        elif k % 5 == 2:
            g.parent[i, last] = -1
        elif k % 5 == 3:
            g.face[i, last] = 4
        else:
            g.axis[i, last] = -1
    s = Surrogate(max_batch=64)
    gd = s.upload_genotypes(g)
    for name in ("nh", "parent", "face", "axis", "cpg"):  # the arrays `shift` elements into larger ones
        a = gd[name]
        room = torch.zeros(a.numel() + shift, dtype=a.dtype, device="cuda")
        room[shift:] = a.reshape(-1)
        gd[name] = room[shift:]
    X = s.features(gd, n).cpu().view(torch.int16).numpy().view(np.uint16)
    np.testing.assert_array_equal(X[ok], ref[ok])
    assert np.isnan(M_float(X[bad])).all()
    s.close()


def M_float(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32)
