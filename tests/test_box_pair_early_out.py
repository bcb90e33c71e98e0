"""The self-collision kernels skip a candidate pair that boxes_apart finds apart.
The kernel's own functions, compiled for the host in float32 (products and sums
fused or not), on pairs whose gap along a face normal lies around the margin:
what is skipped has no corner of either box inside the other, no edge contact and
no face case, so the skipped tests would have found nothing."""
import ctypes as C
import subprocess

import numpy as np
import pytest

from paper_2502_11129_amd import build as B

SOURCE = """
#include "rollout_kernel.hpp"
using namespace simk;
// per pair: bit 0 skipped, bit 1 a corner inside, bit 2 edge contact, bit 3 face case
extern "C" void pairs(int n, const float* pP, const float* RP, const float* hP, const float* pQ, const float* RQ,
                      const float* hQ, int* out) {
  for (int i = 0; i < n; ++i) {
    m33 A, B;
    for (int k = 0; k < 9; ++k) { A.m[k] = RP[9 * i + k]; B.m[k] = RQ[9 * i + k]; }
    const f3 p = {pP[3 * i], pP[3 * i + 1], pP[3 * i + 2]}, q = {pQ[3 * i], pQ[3 * i + 1], pQ[3 * i + 2]};
    const f3 h = {hP[3 * i], hP[3 * i + 1], hP[3 * i + 2]}, g = {hQ[3 * i], hQ[3 * i + 1], hQ[3 * i + 2]};
    bool inside = false;
    for (int c = 0; c < 8; ++c)
      inside = inside || point_in_box(box_corner(A, p, h, c), q, B, g) || point_in_box(box_corner(B, q, g, c), p, A, h);
    f3 x, nn;
    float depth;
    int face = -1;
    const bool edge = edge_contact(p, A, h, q, B, g, x, nn, depth, face);
    out[i] = boxes_apart(p, A, h, q, B, g) | inside << 1 | edge << 2 | (face >= 0) << 3;
  }
}
"""
F32, F64 = np.float32, np.float64


@pytest.fixture(scope="module", params=["fused", "unfused"])
def pairs(request, tmp_path_factory):
    d = tmp_path_factory.mktemp("pairs")
    (d / "pairs.hip").write_text(SOURCE)
    arch = ["-mfma", "-ffp-contract=on"] if request.param == "fused" else ["-ffp-contract=off"]
    so = d / "pairs.so"
    r = subprocess.run([B.HIPCC, *B.COMMON, *arch, f"--offload-arch={B.ARCH}", "--cuda-host-only", "-shared", "-I", B.CSRC,
                        str(d / "pairs.hip"), "-o", str(so)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    fn = C.CDLL(str(so)).pairs

    def call(*arrays):
        arrays = [np.ascontiguousarray(a, F32) for a in arrays]
        out = np.zeros(len(arrays[0]), np.int32)
        fn(len(out), *(a.ctypes.data_as(C.c_void_p) for a in arrays), out.ctypes.data_as(C.c_void_p))
        return out
    return call


def _rot(rng, n, links):
    """Rotations as a chain of bodies forms them: float32 products of `links` unit quaternions' matrices."""
    R = np.tile(np.eye(3, dtype=F32), (n, 1, 1))
    for _ in range(links):
        q = rng.normal(size=(n, 4))
        w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(F32).T
        E = np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)], -1),
                      np.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)], -1),
                      np.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1)], 1)
        R = R @ E
    return R


@pytest.mark.parametrize("at", [0.0, 3.0, 300.0, 30000.0])
@pytest.mark.parametrize("links", [1, 20])
def test_what_is_skipped_has_no_contact(pairs, at, links):
    rng = np.random.default_rng([41, int(at), links])
    n = 60_000
    hP, hQ = (np.exp(rng.uniform(np.log(0.005), np.log(0.5), (n, 3))).astype(F32) for _ in range(2))
    RP, RQ = _rot(rng, n, links), _rot(rng, n, links)
    pP = (rng.normal(0, 1, (n, 3)) * at).astype(F32)
    # Q at a gap along one of P's face normals, from touching to four margins, and aside along the others
    k = rng.integers(0, 3, n)
    ar = np.arange(n)
    axes = RP.astype(F64).transpose(0, 2, 1)
    u = axes[ar, k]
    reach = hP[ar, k] + (np.abs(np.einsum("ni,nij->nj", u, RQ.astype(F64))) * hQ).sum(1)
    margin = 1e-5 + 2e-6 * np.abs(pP).sum(1) + 1e-5 * reach
    gap = rng.uniform(-1.0, 4.0, n) * margin
    side = axes[ar, (k + 1) % 3] * (rng.uniform(-1, 1, n) * reach)[:, None]
    pQ = (pP - u * (reach + gap)[:, None] * rng.choice([-1, 1], n)[:, None] + side).astype(F32)
    for a, b in (((pP, RP, hP), (pQ, RQ, hQ)), ((pQ, RQ, hQ), (pP, RP, hP))):   # either box first
        got = pairs(*a, *b)
        skipped = got & 1 == 1
        assert 0.3 < skipped.mean() < 0.99
        assert not (got[skipped] >> 1).any()
    assert (got[~skipped] >> 1).any()                    # some of the others touch


def test_not_a_number_is_never_skipped(pairs):
    one = np.ones((1, 3), F32) * 0.1
    R = np.eye(3, dtype=F32)[None]
    for bad in range(3):
        p = np.zeros((1, 3), F32)
        p[0, bad] = np.nan
        assert pairs(p, R, one, one * 50, R, one)[0] & 1 == 0
    assert pairs(one * 0, R, one, one * 50, R, one)[0] & 1 == 1
