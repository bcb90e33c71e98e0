"""The self-collision kernels skip a candidate pair whose boxes are apart along
a face normal by the kernel's margin.  In double precision such a pair has no
corner of either box inside the other and a negative least overlap, so the
skipped tests would have found nothing (random pairs near contact, near the
origin and far from it, the margin formed in float32 as the kernel does)."""
import numpy as np
import pytest


def _rot(rng, n):
    q = rng.normal(size=(n, 4))
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    return np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)], -1),
                     np.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)], -1),
                     np.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1)], 1)


def _overlaps(pP, RP, hP, pQ, RQ, hQ):
    axes = np.concatenate([RP.transpose(0, 2, 1), RQ.transpose(0, 2, 1)], 1)          # [n, 6, 3]
    reach = (np.abs(axes @ RP) * hP[:, None]).sum(-1) + (np.abs(axes @ RQ) * hQ[:, None]).sum(-1)
    return np.abs((axes * (pP - pQ)[:, None]).sum(-1)), reach


@pytest.mark.parametrize("at", [0.0, 3.0, 300.0])
def test_a_pair_that_is_skipped_has_no_contact(at):
    rng = np.random.default_rng([31, int(at)])
    n = 200_000
    f = np.float32
    hP, hQ = (rng.uniform(0.01, 0.15, (n, 3)).astype(f) for _ in range(2))
    RP, RQ = _rot(rng, n).astype(f), _rot(rng, n).astype(f)
    pP = (rng.normal(0, 1, (n, 3)) * at).astype(f)
    pQ = (pP + rng.normal(0, 0.1, (n, 3))).astype(f)
    dist, reach = _overlaps(pP, RP, hP, pQ, RQ, hQ)
    slack = f(1e-5) + f(2e-6) * np.abs(pP).sum(1, dtype=f)
    skip = (dist - reach > slack[:, None] + f(1e-5) * reach).any(1)
    assert 0.2 < skip.mean() < 0.98
    D = [a[skip].astype(np.float64) for a in (pP, RP, hP, pQ, RQ, hQ)]
    dist, reach = _overlaps(*D)
    assert ((reach - dist).min(1) < 0).all()
    signs = np.array([[(c & 1) * 2 - 1, (c >> 1 & 1) * 2 - 1, (c >> 2 & 1) * 2 - 1] for c in range(8)], float)
    for (p, R, h), (q, S, g) in ((D[:3], D[3:]), (D[3:], D[:3])):
        x = p[:, None] + (signs[None] * h[:, None]) @ R.transpose(0, 2, 1)
        local = (x - q[:, None]) @ S
        assert not (np.abs(local) < g[:, None]).all(-1).any()
