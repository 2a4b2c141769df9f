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
