"""The one-launch prediction at the edges of its tiles (16, 32 and 48 rows, at
most 256 tiles of the smaller ones): against the BF16-emulating FP64 oracle
within 1e-2 |ref| + 1e-3 rms(ref) per element, gathered rows equal to the plain
ones, nothing written past the last row, indices outside the rows NaN."""
import numpy as np
import pytest
import torch

from oracle import mlp_oracle as M
from paper_2502_11129_amd import workloads as W
from paper_2502_11129_amd.surrogate import Surrogate

pytestmark = pytest.mark.gpu

N_MAX = 12288 + 300


@pytest.fixture(scope="module")
def net():
    p = W.mlp_init(9)
    s = Surrogate(params=p)
    X = s.features(s.upload_genotypes(W.random_genotypes(N_MAX, key=91)))
    ref, _ = M.forward(X.float().cpu().numpy().astype(np.float64), *M.unflatten(p.astype(np.float64)))
    yield s, X, np.asarray(ref)
    s.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 255, 4095, 4096, 4097, 8192, 8193, 12288, 12289, N_MAX])
def test_predictions_at_tile_edges(net, n):
    s, X, ref = net
    out = torch.full((n + 64,), 7.0, device="cuda")
    y = s.predict(X[:n].contiguous(), out=out[:n]).cpu().numpy().astype(np.float64)
    assert (out[n:] == 7.0).all()
    bar = 1e-2 * np.abs(ref[:n]) + 1e-3 * np.sqrt(np.mean(ref ** 2))
    assert (np.abs(y - ref[:n]) <= bar).all()
    idx = torch.randperm(N_MAX, generator=torch.Generator().manual_seed(n))[:n].to(torch.int32)
    if n > 2:
        idx[n // 2], idx[n - 1] = -1, N_MAX
    yi = s.predict(X, idx=idx.cuda()).cpu()
    ok = (idx >= 0) & (idx < N_MAX)
    assert torch.isnan(yi[~ok]).all()
    full = s.predict(X).cpu()
    assert torch.equal(yi[ok], full[idx[ok].long()])


@pytest.mark.parametrize("n", [16384, 16385, 24576, 24577])
def test_predictions_in_long_tiles(net, n):
    """64- and 96-row tiles: the rows again and again, bit for bit the same."""
    s, X, ref = net
    rep = X.repeat(3, 1)[:n].contiguous()
    out = torch.full((n + 64,), 7.0, device="cuda")
    y = s.predict(rep, out=out[:n])
    assert (out[n:] == 7.0).all()
    assert torch.equal(y, s.predict(X).repeat(3)[:n])


def test_predictions_do_not_depend_on_the_rows_beside():
    """Which form of erf a wave takes depends on the rows of its tile: rows with
    small arguments give the same bits alone and among rows with large ones."""
    s = Surrogate(params=W.mlp_init(9), max_batch=64)
    X = s.features(s.upload_genotypes(W.random_genotypes(3000, key=92)))
    mixed = X.clone()
    mixed[::3] *= 32.0
    mixed[5::48] = float("nan")
    y, ym = s.predict(X), s.predict(mixed)
    same = (mixed == X).all(dim=1)
    assert torch.equal(y[same], ym[same])
    assert torch.isnan(ym[5::48]).all() and torch.isfinite(ym[same]).all()
    large = s.predict(mixed[~same].contiguous())
    assert torch.equal(large.nan_to_num(), ym[~same].nan_to_num())
    s.close()
