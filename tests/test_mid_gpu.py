"""GPU tests of the two-kernel form's 128-row tiles (mid.hip), against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import workloads
from tests.util import compare, compare_gated, to_host_f64, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rl():
    import paper_2405_05751_amd as pkg
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    yield pkg
    pkg.rl_set_variant("auto")
    pkg.rl_set_tuning(0, 0)


def _run(rl, fn, variant, cols, slabs):
    import torch
    rl.rl_set_variant(variant)
    rl.rl_set_tuning(cols, slabs)
    try:
        Y = fn()
        torch.cuda.synchronize()
        return Y, rl.rl_last_launch()
    finally:
        rl.rl_set_variant("auto")
        rl.rl_set_tuning(0, 0)


# one short of a tile, whole, one over, in rows (128) and columns (64 and 128); K under one tile of 64, whole, ragged; fewer K
# tiles than stages; nine tile rows (two panels of eight)
SIZES = [(1, 8, 8), (127, 64, 64), (128, 128, 128), (129, 72, 136), (65, 200, 56), (257, 1000, 640), (130, 4104, 264),
         (1100, 136, 72), (300, 448, 1288)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("cols", [64, 128])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_tiles_and_splits(rl, M, K, N, cols, dtype):
    w = workloads.make(M, K, N, dtype, 1e-5, 9100 + M + K + N, outlier_frac=0.05 if M > 8 else 0.0)
    X, g, W = upload(w)
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps)
    for slabs in (1, 2, 5):
        Y, used = _run(rl, lambda: rl.rmsnorm_linear(X, g, W, w.eps), "tile_pre", cols, slabs)
        assert used[0] == "tile_pre" and used[1] == cols
        compare(to_host_f64(Y, dtype), Z, dtype, f"{M}x{K}x{N} {used}")


@pytest.mark.parametrize("cols", [64, 128])
@pytest.mark.parametrize("M,K,H", [(129, 136, 24), (200, 520, 192), (66, 1000, 320)])
def test_gated(rl, M, K, H, cols):
    w = workloads.make(M, K, 2 * H, "bf16", 1e-5, 9200 + M + K + H)
    X, g, W = upload(w)
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps)
    for slabs in (1, 3):
        Y, used = _run(rl, lambda: rl.rmsnorm_gated_mlp(X, g, W, w.eps), "tile_pre", cols, slabs)
        assert used[1] == cols
        compare_gated(to_host_f64(Y, "bf16"), Z, "bf16", f"gated {M}x{K}x{H} {used}")
        if H % 64 == 0:
            Wi = rl.rl_interleave_gate_up(W)
            Yi, _ = _run(rl, lambda: rl.rmsnorm_gated_mlp_interleaved(X, g, Wi, w.eps), "tile_pre", cols, slabs)
            assert (Yi == Y).all()


@pytest.mark.parametrize("M,K,N,shares,without", [(300, 1024, 10000, False, ("tile_pre",)), (268, 3584, 3512, False, ("skinny",)),
                                                  (1024, 4096, 4096, True, ("tile",))])
def test_automatic_choice(rl, M, K, N, shares, without):
    """The rule takes these.  Without room for X-hat: tiles that form it themselves where the call needs no workspace by
    the query (it shares none with other streams then), else the kernels that run without X-hat."""
    import torch
    w = workloads.make(M, K, N, "bf16", 1e-5, 9300 + M, n_check_rows=40)
    X, g, W = upload(w)
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps, rows=w.check_rows)
    rows = torch.from_numpy(np.asarray(w.check_rows)).cuda()
    Y, used = _run(rl, lambda: rl.rmsnorm_linear(X, g, W, w.eps), "auto", 0, 0)
    assert used[0] == "tile_pre" and used[1] in (64, 128)
    assert (rl.rl_workspace_bytes(M, K, N, X.dtype) > 2 * M * K) == shares
    compare(to_host_f64(Y[rows], "bf16"), Z, "bf16", f"auto {M}x{K}x{N} {used}")
    small = torch.zeros(1280 * 1024 + 4096, dtype=torch.uint8, device="cuda")
    rl.rl_set_workspace(small)
    try:
        Y, used = _run(rl, lambda: rl.rmsnorm_linear(X, g, W, w.eps), "auto", 0, 0)
    finally:
        rl.rl_set_workspace(None)
    assert used[0] in without
    compare(to_host_f64(Y[rows], "bf16"), Z, "bf16", f"no room {M}x{K}x{N} {used}")


@pytest.mark.parametrize("M,K,N,dtype", [(268, 3584, 3512, "bf16"), (140, 4096, 4096, "f16"), (900, 7272, 520, "bf16"), (245, 992, 2496, "f16")])
def test_no_alloc_entry_point(rl, M, K, N, dtype):
    """The same launch and the same bits where X-hat and the partial tiles are larger than the first scratch array."""
    import torch
    w = workloads.make(M, K, N, dtype, 1e-5, 9400 + M, n_check_rows=1)
    X, g, W = upload(w)
    Y = rl.rmsnorm_linear(X, g, W, w.eps)
    used = rl.rl_last_launch()
    assert used[0] == "tile_pre" and used[1] in (64, 128)
    Y2 = torch.full_like(Y, 99.0)
    rl.rmsnorm_linear_noalloc(X, g, W, w.eps, Y2)
    torch.cuda.synchronize()
    assert rl.rl_last_launch() == used
    assert torch.equal(Y, Y2)


@pytest.mark.parametrize("cols", [64, 128])
@pytest.mark.parametrize("M,K,H", [(129, 136, 24), (200, 520, 192), (66, 1000, 320)])
def test_gated_f16(rl, M, K, H, cols):
    w = workloads.make(M, K, 2 * H, "f16", 1e-5, 9200 + M + K + H)
    X, g, W = upload(w)
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps)
    for slabs in (1, 3):
        Y, used = _run(rl, lambda: rl.rmsnorm_gated_mlp(X, g, W, w.eps), "tile_pre", cols, slabs)
        assert used[1] == cols
        compare_gated(to_host_f64(Y, "f16"), Z, "f16", f"gated {M}x{K}x{H} {used}")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("cols,slabs", [(64, 1), (128, 1), (64, 2), (128, 5)])
@pytest.mark.parametrize("M,K,N", [(129, 456, 136), (257, 1000, 648)])
def test_special_values_and_edges(rl, M, K, N, cols, slabs, dtype):
    """An infinity in the last row of W keeps its sign and its column, NaN and infinity in X keep to their rows, a zero row gives
    zeros; nothing outside Y is written; the launch has the slabs that whole K tiles of 64 make of those asked for."""
    import torch
    w = workloads.make(M, K, N, dtype, 1e-5, 9500 + M)
    X, g, W = upload(w)
    X[:, K - 1] = torch.where(torch.arange(M, device="cuda") % 2 == 0, 1.0, -1.0).to(X.dtype)
    W[K - 1, 7] = float("inf")
    X[M - 1] = 0.0
    X[M - 2, 3] = float("nan")
    X[5, K - 2] = float("inf")
    pad = 512
    buf = torch.full((pad + M * N + pad,), 99.0, dtype=X.dtype, device="cuda")
    Y = buf[pad:pad + M * N].view(M, N)
    _, used = _run(rl, lambda: rl.rmsnorm_linear(X, g, W, w.eps, Y), "tile_pre", cols, slabs)
    slab = -(-(-(-K // slabs)) // 64) * 64
    assert used[:3] == ("tile_pre", cols, -(-K // slab))
    assert torch.all(buf[:pad] == 99.0) and torch.all(buf[pad + M * N:] == 99.0)
    plain = [r for r in range(M) if r not in (5, M - 2, M - 1)]
    assert torch.equal(Y[plain, 7].float(), X[plain, K - 1].float() * float("inf"))
    others = [n for n in range(N) if n != 7]
    assert torch.isfinite(Y[plain][:, others]).all()
    assert torch.isnan(Y[5]).all() and torch.isnan(Y[M - 2]).all()
    assert (Y[M - 1, others] == 0).all() and torch.isnan(Y[M - 1, 7])
    W[K - 1, 7] = 0.0
    X[M - 2, 3] = X[5, K - 2] = 1.0                      # (rows that are not compared)
    xs, ws = X.cpu().double(), W.cpu().double()
    Z = (xs * g.cpu().double()) @ ws / torch.sqrt((xs ** 2).mean(1, keepdim=True) + w.eps)
    compare(to_host_f64(Y[plain][:, others], dtype), Z[plain][:, others].numpy(), dtype, f"{M}x{K}x{N} {used}")
