"""The skinny variant's form for a small W (narrow tiles, all of K in one workgroup): edges of its steps of 32 k, of the waves' rounds
(512 k up to 32 rows, 256 above), of its 16, 32 and 64 columns and of its row blocks, against the fp64 oracle.  Needs an MI355X."""
import numpy as np
import pytest

import oracle
import workloads
from util import compare, compare_gated, to_host_f64, upload

pytestmark = pytest.mark.gpu


# (tests/test_routes.py pins the kernel that each of these launches, which the columns and slabs alone do not tell)
EDGES = [
    (1, 8, 8, 16), (1, 24, 16, 16), (2, 32, 24, 16), (5, 40, 40, 16), (7, 504, 264, 16), (16, 512, 512, 16), (16, 520, 4096, 16),
    (17, 480, 136, 16), (32, 1032, 1000, 16), (33, 248, 72, 16), (48, 256, 1016, 16), (49, 264, 2048, 16), (64, 776, 1048, 16),
    (3, 304, 6472, 32), (16, 544, 5000, 32), (31, 1000, 4968, 32), (57, 768, 6008, 32), (16, 264, 12808, 64), (24, 264, 10248, 64), (64, 264, 12296, 64),
]
BLOCKS = [(65, 8, 8, "bf16"), (65, 264, 136, "f16"), (127, 520, 1016, "bf16"), (128, 512, 512, "f16"), (129, 40, 24, "bf16"),
          (200, 1000, 1016, "bf16"), (320, 256, 2056, "f16"), (512, 264, 520, "bf16"), (66, 1536, 2048, "f16")]
GATED = [(100, 520, 448, "f16"), (300, 264, 1024, "bf16"), (1, 40, 64, "bf16"), (4, 520, 128, "bf16"), (5, 520, 128, "f16"),
         (16, 776, 1024, "bf16"), (32, 264, 2112, "f16"), (33, 512, 576, "bf16"),
         (64, 272, 6400, "f16")]


@pytest.fixture(scope="module")
def rl():
    import torch
    import paper_2405_05751_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pkg.rl_set_variant("auto")
    pkg.rl_set_tuning(0, 0)
    return pkg


def small(rl):
    """Tiles narrower than 128 columns that nobody asked for, unsplit: what the form reports (and the 64-column tiles in one slab too)."""
    used, cols, slabs, _ = rl.rl_last_launch()
    return used == "skinny" and cols in (16, 32, 64) and slabs == 1


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N,columns", EDGES)
def test_edges(rl, M, K, N, columns, dtype):
    import torch
    w = workloads.make(M, K, N, dtype, 1e-5, 9100 + K + N)
    X, g, W = upload(w)
    Y = torch.full((M, N), float("nan"), dtype=X.dtype, device="cuda")
    rl.rmsnorm_linear(X, g, W, w.eps, Y)
    torch.cuda.synchronize()
    if M <= 4 and dtype == "f16":            # (fp32 arithmetic: see test_few_rows_gpu.py)
        assert rl.rl_last_variant() == "gemv"
    else:
        assert small(rl) and rl.rl_last_launch()[1] == columns
        assert rl.rl_workspace_bytes(M, K, N, X.dtype) == 0
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, dtype, w.eps)
    compare(to_host_f64(Y, dtype), Z, dtype, f"{M}x{K}x{N}")
    # the same bits whatever the entry point
    Y2 = torch.full_like(Y, float("nan"))
    assert rl.lib().rmsnorm_linear_noalloc(X.data_ptr(), g.data_ptr(), W.data_ptr(), float(w.eps), Y2.data_ptr(), M, K, N,
                                           {"f16": 0, "bf16": 1}[dtype], torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))


@pytest.mark.parametrize("M,K,N,dtype", BLOCKS)
def test_row_blocks(rl, M, K, N, dtype):
    import torch
    w = workloads.make(M, K, N, dtype, 1e-5, 9400 + M + N)
    X, g, W = upload(w)
    Y = torch.full((M, N), float("nan"), dtype=X.dtype, device="cuda")
    rl.rmsnorm_linear(X, g, W, w.eps, Y)
    torch.cuda.synchronize()
    assert small(rl) and rl.rl_last_launch()[3] == -(-M // 64) * -(-N // rl.rl_last_launch()[1])
    compare(to_host_f64(Y, dtype), oracle.rmsnorm_linear(w.X, w.g, w.W, dtype, w.eps), dtype, f"{M}x{K}x{N}")
    assert rl.rl_workspace_bytes(M, K, N, X.dtype) == 0


@pytest.mark.parametrize("interleaved", [False, True])
@pytest.mark.parametrize("M,K,H,dtype", GATED)
def test_gated(rl, M, K, H, dtype, interleaved):
    import torch
    w = workloads.make(M, K, 2 * H, dtype, 1e-5, 9200 + K + H)
    X, g, W = upload(w)
    if interleaved:
        Y = rl.rmsnorm_gated_mlp_interleaved(X, g, rl.rl_interleave_gate_up(W), w.eps)
    else:
        Y = rl.rmsnorm_gated_mlp(X, g, W, w.eps)
    torch.cuda.synchronize()
    assert small(rl)
    compare_gated(to_host_f64(Y, dtype), oracle.rmsnorm_linear(w.X, w.g, w.W, dtype, w.eps), dtype, f"{M}x{K}x2*{H}")


@pytest.mark.parametrize("M,dtype", [(7, "bf16"), (40, "f16")])
def test_rows_keep_to_themselves(rl, M, dtype):
    """A row of NaN, one of infinities and one of zeros change no other row; the plain product takes the same form."""
    import torch
    w = workloads.make(M, 264, 520, dtype, 1e-5, 9300 + M)
    X, g, W = upload(w)
    Y0 = rl.rmsnorm_linear(X, g, W, w.eps)
    bad = X.clone()
    bad[1, 3], bad[4, 263], bad[M - 1] = float("nan"), float("inf"), 0.0
    Y = rl.rmsnorm_linear(bad, g, W, w.eps)
    torch.cuda.synchronize()
    assert small(rl)
    rest = [m for m in range(M) if m not in (1, 4, M - 1)]
    assert torch.equal(Y[rest].view(torch.int16), Y0[rest].view(torch.int16))
    assert bool(Y[1].isnan().all()) and bool(Y[4].isnan().all()) and bool((Y[M - 1] == 0).all())
    P = rl.matmul(X, W)
    torch.cuda.synchronize()
    assert small(rl)
    Z = to_host_f64(X, dtype) @ to_host_f64(W, dtype)
    compare(to_host_f64(P, dtype), Z, dtype, "plain product")
