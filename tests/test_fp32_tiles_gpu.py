"""GPU tests of the fp32 kernel's 128 x 128 tiles, against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import workloads
from tests.util import compare, to_host_f64, upload

pytestmark = pytest.mark.gpu


# shapes that fill the chip with 128 x 128 tiles: ragged rows and columns (one over a tile, four short), K the smallest, of an
# odd number of tiles of 32, with a ragged last one, and the largest
@pytest.mark.parametrize("M,K,N", [(2048, 192, 4096), (1921, 292, 1924), (2048, 512, 4096), (1023, 1000, 4092), (1020, 4096, 4092)])
def test_tiles(M, K, N):
    import torch
    import paper_2405_05751_amd as rl
    w = workloads.make(M, K, N, "f32", 1e-5, 9400 + M + K, n_check_rows=48, outlier_frac=0.01)
    X, g, W = upload(w)
    pad = 256
    buf = torch.full((pad + M * N + pad,), 99.0, device="cuda")
    Y = buf[pad:pad + M * N].view(M, N)
    rl.rmsnorm_linear(X, g, W, w.eps, Y)
    torch.cuda.synchronize()
    assert rl.rl_last_launch()[:3] == ("f32", 128, 1)
    assert torch.all(buf[:pad] == 99.0) and torch.all(buf[pad + M * N:] == 99.0)
    rows = np.unique(np.concatenate([np.asarray(w.check_rows), [0, 31, 32, 63, 64, 127, 128, M - 2, M - 1]]))
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps, rows=rows)
    got = to_host_f64(Y[torch.from_numpy(rows).cuda()], "f32")
    # the fp32 bar is 1e-5; the first kernel's tests hold it to 2e-6, and so does this one's summation order
    ratio, _ = compare(got, Z, "f32", f"{M}x{K}x{N}")
    assert ratio <= 2e-6, ratio


@pytest.mark.parametrize("M,K,N", [(1921, 292, 1924), (1023, 1000, 4092)])
def test_special_values(M, K, N):
    """Infinities in W keep sign and column, NaN and infinity in X keep to their rows, a zero row gives zeros."""
    import torch
    import paper_2405_05751_amd as rl
    w = workloads.make(M, K, N, "f32", 1e-5, 9450, n_check_rows=8)
    X, g, W = upload(w)
    X[:, K - 1] = torch.where(torch.arange(M, device="cuda") % 2 == 0, 1.0, -1.0)
    clean = rl.rmsnorm_linear(X, g, W, w.eps)
    W[K - 1, 130] = float("inf")
    X[M - 1] = 0.0
    X[127, 3] = float("nan")
    X[128, K - 2] = float("inf")
    Y = rl.rmsnorm_linear(X, g, W, w.eps)
    torch.cuda.synchronize()
    assert rl.rl_last_launch()[:3] == ("f32", 128, 1)
    plain = torch.tensor([r for r in range(M) if r not in (127, 128, M - 1)], device="cuda")
    others = torch.tensor([n for n in range(N) if n != 130], device="cuda")
    assert torch.equal(Y[plain, 130], X[plain, K - 1] * float("inf"))
    assert torch.equal(Y[plain][:, others], clean[plain][:, others])
    assert torch.isnan(Y[127]).all() and torch.isnan(Y[128]).all()
    assert (Y[M - 1, others] == 0).all() and torch.isnan(Y[M - 1, 130])
