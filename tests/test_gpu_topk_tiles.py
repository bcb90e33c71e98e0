"""Top-k at the edges of the one-workgroup selections (4096 and 16 384 scores), of the
8192-score tiles and of 256 tiles, for continuous, tied, equal and special
scores: exactly the indices of a stable sort by descending score, NaN last, in
index order; nothing written past k; the static-scratch entry point alike."""
import numpy as np
import pytest
import torch

from paper_2502_11129_amd import surrogate as SU

pytestmark = pytest.mark.gpu


def _scores(n, kind):
    rng = np.random.default_rng([n, kind])
    if kind == 0:
        return rng.normal(0, 1, n).astype(np.float32)
    if kind == 1:
        x = np.round(rng.normal(0, 1, n), 1).astype(np.float32)
        for v in (np.nan, np.inf, -np.inf, -0.0, -np.finfo(np.float32).max, 1e-45, -1e-45):
            x[rng.integers(0, n, n // 40 + 1)] = v
        return x
    return np.full(n, (np.nan, 0.25, -np.inf)[n % 3], np.float32)


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 4095, 4096, 4097, 16383, 16384, 16385, 24576, 24577, 100003, 2097152, 2097153])
def test_topk_at_tile_edges(n):
    s = SU.Surrogate(max_batch=64)
    for kind in range(3):
        x = _scores(n, kind)
        order = np.lexsort((np.arange(n), np.isnan(x), -np.where(np.isnan(x), -np.inf, x).astype(np.float64)))
        room = torch.zeros(n + 1, device="cuda")     # also off the natural alignment of wide loads
        room[1:] = torch.from_numpy(x).cuda()
        for k in sorted({1, (n + 2) // 3, max(1, n - 1), n}):
            ref = np.sort(order[:k]).astype(np.int32)
            np.testing.assert_array_equal(s.topk(room[1:], k).cpu().numpy(), ref)
            out = torch.full((k + 64,), -7, dtype=torch.int32, device="cuda")
            SU.topk_noalloc(room[1:], k, out=out[:k])
            out = out.cpu().numpy()
            np.testing.assert_array_equal(out[:k], ref)
            assert (out[k:] == -7).all()
    s.close()
