"""One to four rows and a small W, where the narrow tiles of the matrix cores stand in for the GEMV kernel: what that one
gives for the ends of a type's range and for infinite weights.  Needs an MI355X."""
import numpy as np
import pytest

import oracle
from util import to_host_f64

pytestmark = pytest.mark.gpu

# (hidden size, columns): one trip of the waves over K and two, whole and ragged tiles
SIZES = [(512, 512), (1000, 1016)]


@pytest.fixture(scope="module")
def rl():
    import torch
    import paper_2405_05751_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pkg.rl_set_variant("auto")
    pkg.rl_set_tuning(0, 0)
    return pkg


def inputs(M, K, N, dtype, seed):
    import torch
    r = torch.Generator().manual_seed(seed)
    X, g = torch.randn(M, K, generator=r), torch.rand(K, generator=r) + 0.5
    W = torch.randn(K, N, generator=r) * K ** -0.5
    return X, g, W


def call(rl, X, g, W, eps, dtype):
    """The library's Y and the one of 64 bits on the same (rounded) inputs."""
    import torch
    t = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    X, g, W = X.to(t), g.to(t), W.to(t)
    Y = rl.rmsnorm_linear(X.cuda(), g.cuda(), W.cuda(), eps)
    torch.cuda.synchronize()
    x, w = X.double().numpy(), W.double().numpy()
    with np.errstate(all="ignore"):
        Z = (x * g.double().numpy()) @ w / np.sqrt((x * x).mean(1, keepdims=True) + eps)
    return to_host_f64(Y, dtype), Z


def close(Y, Z, dtype):
    """Each output is one rounding off (2^-11 or 2^-8 of itself at most), the sums before it are fp32: products of two
    16-bit numbers are exact in them, and K 2^-24 is far below that rounding.  A quarter of it more for them."""
    assert np.isfinite(Y).all()
    err = np.linalg.norm(Y - Z) / np.linalg.norm(Z)
    assert err <= 1.25 * 2.0 ** -{"f16": 11, "bf16": 8}[dtype], err


@pytest.mark.parametrize("K,N", SIZES)
@pytest.mark.parametrize("M", [1, 4])
@pytest.mark.parametrize("x,gain", [(50000.0, 1.5), (2500.0, 30.0), (60000.0, 4.0)])
def test_products_beyond_fp16(rl, M, K, N, x, gain):
    """x g beyond 65504, X, g and Y within it."""
    X, g, W = inputs(M, K, N, "f16", 31 + K)
    X[M - 1, 5], g[5] = x, gain
    close(*call(rl, X, g, W, 1e-5, "f16"), "f16")


@pytest.mark.parametrize("K,N", SIZES)
@pytest.mark.parametrize("M", [1, 4])
@pytest.mark.parametrize("dtype,scale,gain", [("f16", 1e-4, 1.0), ("f16", 1e-5, 1.0), ("f16", 3e-6, 1.0), ("f16", 1e-4, 0.02),
                                              ("bf16", 1e-5, 1.0), ("bf16", 1e-18, 1.0), ("bf16", 1e-18, 1e-18), ("bf16", 1e17, 1.0)])
def test_small_and_large_products(rl, M, K, N, dtype, scale, gain):
    """Products near and below a type's smallest numbers keep the bits that fp32 has for them."""
    X, g, W = inputs(M, K, N, dtype, 37 + K)
    close(*call(rl, X * scale, g * gain, W, 0.0, dtype), dtype)


@pytest.mark.parametrize("K,N", SIZES)
@pytest.mark.parametrize("M", [1, 4])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("gain", ["ones", "any"])
def test_infinite_weights(rl, M, K, N, dtype, gain):
    """One infinity in a column of W, or in g, gives the infinities that it gives in 64 bits; the other columns stay as they are,
    with products of zero of either sign among theirs.  (Gains of one: products that one 16-bit number holds.)"""
    import torch
    X, g, W = inputs(M, K, N, dtype, 41 + K)
    if gain == "ones":
        g[:] = 1.0
    X[:, 9], X[M - 1, 11], g[13] = X[:, 9].abs() + 0.5, -0.0, 0.0
    plain = W.clone()
    W[9, 3], W[K - 1, 17], W[100, N - 1] = float("inf"), float("-inf"), float("inf")
    Y, Z = call(rl, X, g, W, 1e-5, dtype)
    infinite = [3, 17, N - 1]
    assert np.isinf(Z[:, infinite]).all() and np.array_equal(Y[:, infinite], Z[:, infinite])
    rest = [n for n in range(N) if n not in infinite]
    close(Y[:, rest], Z[:, rest], dtype)
    t = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    P = rl.matmul(X.to(t).cuda(), W.to(t).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(to_host_f64(P, dtype)[:, infinite], Z[:, infinite])
    g[9] = float("inf")                      # an infinite product of every column
    Y, Z = call(rl, X, g, plain, 1e-5, dtype)
    assert np.isinf(Z).all() and np.array_equal(Y, Z)


@pytest.mark.parametrize("M,K,N,dtype,want", [(1, 512, 512, "f16", "gemv"), (4, 1000, 1016, "f16", "gemv"), (3, 1024, 1952, "f16", "gemv"),
                                              (15, 2384, 3208, "bf16", "skinny"), (32, 2304, 1344, "f16", "skinny")])
def test_no_room_for_a_split(rl, M, K, N, dtype, want):
    """A lent buffer with no room for partial sums: a small W runs without a split, and with one again afterwards."""
    import torch
    X, g, W = inputs(M, K, N, dtype, 43 + K)
    lent = torch.zeros((1280 << 10) + 1024, dtype=torch.uint8, device="cuda")
    rl.rl_set_workspace(lent)
    try:
        Y, Z = call(rl, X, g, W, 1e-5, dtype)
        used = rl.rl_last_launch()
    finally:
        rl.rl_set_workspace(None)
    assert used[0] == want and used[2] == 1
    close(Y, Z, dtype)
    Y, Z = call(rl, X, g, W, 1e-5, dtype)
    assert rl.rl_last_launch()[2] > 1
    close(Y, Z, dtype)
