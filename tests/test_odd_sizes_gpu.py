"""GPU tests of the 16-bit fused block at sizes that are no multiple of eight (odd.hip), against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import workloads
from tests.util import to_host_f64, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rl():
    import paper_2405_05751_amd as pkg
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _check(Y, Z, dtype, what):
    """One rounding of the output (half an ulp: at most 2^-8 or 2^-11 of the value), and the fp32 sums: a few 1e-6 of
    the row's rms, 2e-5 allowed.  X-hat rounded to 16 bits would show 1e-3 (bf16) or 1.4e-4 (f16) of it."""
    half_ulp = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -11
    rms = np.sqrt((Z ** 2).mean(axis=1, keepdims=True))
    bound = half_ulp * 1.001 * np.abs(Z) + 2e-5 * rms + 2.0 ** -25      # (2^-25: f16 subnormals)
    worst = float((np.abs(Y - Z) / bound).max())
    assert worst <= 1.0, f"{what}: |err| / bound = {worst:.3f}"


SIZES = [
    # tiles of 128 columns: one short, whole, one over; K around runs of 64 and steps of 32
    (1, 64, 127), (2, 63, 129), (3, 65, 255), (5, 127, 130), (4, 128, 257), (16, 31, 100), (7, 33, 1), (3000, 33, 65), (1025, 95, 131),
    (1, 1, 3), (2, 3, 2), (9, 7, 250), (16, 1000, 1001), (1, 4096, 1003), (1, 4095, 1002), (13, 514, 514),
    # row blocks of 16, and of 64; K % 8 == 0 and not; N % 8 == 0 with an odd K
    (17, 512, 1001), (31, 515, 770), (33, 776, 1161), (48, 777, 256), (64, 1032, 363), (65, 1031, 363),
    (129, 264, 1100), (200, 513, 1025), (300, 520, 130), (1100, 72, 301), (140, 65, 1025),
    # splits over K
    (8, 4096, 3001), (24, 2049, 4003), (60, 3000, 500), (70, 2048, 1201),
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_odd_sizes(rl, M, K, N, dtype):
    import torch
    w = workloads.make(M, K, N, dtype, 1e-5, 5000 + M + 3 * K + 7 * N, outlier_frac=0.1 if M > 8 else 0.0)
    X, g, W = upload(w)
    Y = rl.rmsnorm_linear(X, g, W, w.eps)
    torch.cuda.synchronize()
    assert rl.rl_last_launch()[1] == (0 if K <= 96 and M * N <= 1 << 17 else 128)
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps)
    _check(to_host_f64(Y, dtype), Z, dtype, f"{M}x{K}x{N} {dtype}")
    Y2 = torch.empty_like(Y)                             # the workspace the call needs fits every entry point's
    rl.rmsnorm_linear_noalloc(X, g, W, w.eps, Y2)
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2)


@pytest.mark.parametrize("M,K,N", [(3, 515, 131), (20, 520, 131)])
def test_fp16_range(rl, M, K, N):
    """Rows far outside the range in which X (.) g has two fp16 parts without a scale."""
    import torch
    w = workloads.make(M, K, N, "f16", 0.0, 77)
    X, g, W = upload(w)
    for scale in (2.0 ** -20, 2.0 ** 13):                # (powers of two; at 2^-20 most elements are subnormal)
        Xs = (X.float().clamp(-3, 3) * scale).to(torch.float16)
        gs = g * (1 if scale < 1 else 1.25)              # products of up to 3 * 2^13 * 1.9 = 46 000 and over
        Xs[0, 0] = 65504.0 if scale > 1 else Xs[0, 0]
        Y = rl.rmsnorm_linear(Xs, gs, W, 0.0)
        torch.cuda.synchronize()
        Z = oracle.rmsnorm_linear(Xs.cpu().numpy(), gs.cpu().numpy(), w.W, "f16", 0.0)
        _check(to_host_f64(Y, "f16"), Z, "f16", f"scale {scale}")


@pytest.mark.parametrize("what", ["small x, large gain", "large behind small", "first runs zero", "both large", "all small"])
@pytest.mark.parametrize("M,K,N", [(3, 1001, 131), (40, 1024, 131), (70, 2049, 258)])
def test_fp16_uneven_gain(rl, M, K, N, what):
    """Products of very different size, and their largest in another column than the largest x or the largest gain: an
    operand that is rounded, or a product that is cut off, shows above the fp32 sums (see _check)."""
    import torch
    w = workloads.make(M, K, N, "f16", 1e-5, 78 + M)
    x, g = w.X.copy(), w.g.copy()
    if what == "small x, large gain":
        x[:, 5], g[5] = 7.4e-5, 60000.0                  # a product of 4.4
        x[:, K - 1], g[K - 1] = 30000.0, 1e-4            # of 3, but x and g alone bound the row's by 1.8e9
    elif what == "large behind small":
        x[:, :260] *= np.float16(2.0 ** -12)             # (the first run of each wave)
        x[:, K - 3], g[K - 3] = 30000.0, 3000.0
    elif what == "first runs zero":
        x[:, :300] = 0.0
        x[0, 300:] *= np.float16(2.0 ** -12)
        x[1, K - 3] = 30000.0
    elif what == "both large":
        x[:, 70], g[70] = 60000.0, 3000.0
    else:
        x *= np.float16(2.0 ** -16)
    X, G, W = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda(), upload(w)[2]
    Y = rl.rmsnorm_linear(X, G, W, 0.0)
    torch.cuda.synchronize()
    assert rl.rl_last_launch()[1] == 128
    Z = oracle.rmsnorm_linear(x, g, w.W, "f16", 0.0)
    _check(to_host_f64(Y, "f16"), Z, "f16", f"{M}x{K}x{N} {what}")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("K", [264, 261])
def test_special_values(rl, dtype, K):
    """Infinities in W keep their sign, NaN and infinity in X stay in their row, a zero row gives zeros."""
    import torch
    M, N = 5, 243
    w = workloads.make(M, K, N, dtype, 1e-5, 91)
    X, g, W = upload(w)
    X[X == 0] = 1.0
    g[3] = 1.0                                           # a product with nothing left for its second part
    X[1, 3] = 1.0
    W[3, 7] = float("inf")
    W[K - 1, N - 1] = float("-inf")
    X[2, 5] = float("nan")
    X[3] = 0.0
    X[4, 0] = float("inf")
    Y = rl.rmsnorm_linear(X, g, W, w.eps).float().cpu()
    want = lambda n, k, sign: torch.sign(X[0:2, k].float().cpu()) * sign * float("inf")
    assert torch.equal(Y[0:2, 7], want(7, 3, 1.0))
    assert torch.equal(Y[0:2, N - 1], want(N - 1, K - 1, -1.0))
    others = [n for n in range(N) if n not in (7, N - 1)]
    assert torch.isfinite(Y[0:2][:, others]).all()
    assert torch.isnan(Y[2]).all()
    assert (Y[3][others] == 0).all() and torch.isnan(Y[3, 7]) and torch.isnan(Y[3, N - 1])
    assert torch.isnan(Y[4]).all()


def test_no_room_runs_unsplit(rl):
    """With a lent workspace too small for the partial sums of a split the same kernel runs without one."""
    import torch
    w = workloads.make(40, 4001, 65, "bf16", 1e-5, 93)
    X, g, W = upload(w)
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps)
    small = torch.zeros(1280 * 1024 + 4096, dtype=torch.uint8, device="cuda")
    rl.rl_set_workspace(small)
    try:
        Y = rl.rmsnorm_linear(X, g, W, w.eps)
        torch.cuda.synchronize()
        assert rl.rl_last_launch()[1:3] == (128, 1)
    finally:
        rl.rl_set_workspace(None)
    _check(to_host_f64(Y, "bf16"), Z, "bf16", "no room")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,K,N,slabs", [(1, 1, 3, 0), (2, 3, 2, 0), (9, 7, 250, 1), (65, 64, 127, 0), (5, 96, 64, 0), (8, 512, 512, 2), (70, 1032, 264, 4),
                                         (24, 2051, 1001, 8)])
def test_asked_for(rl, M, K, N, slabs, dtype):
    """Asked for by its columns: also at sizes where the automatic choice is another, and in a given number of slabs."""
    import torch
    w = workloads.make(M, K, N, dtype, 1e-5, 5600 + M + K + N)
    X, g, W = upload(w)
    Y = rl.rmsnorm_linear_ex(X, g, W, w.eps, variant="naive", columns=128, slabs=slabs)
    torch.cuda.synchronize()
    used = rl.rl_last_launch()
    assert used[:2] == ("naive", 128) and (slabs == 0 or used[2] == slabs)
    Z = oracle.rmsnorm_linear(w.X, w.g, w.W, w.dtype, w.eps)
    _check(to_host_f64(Y, dtype), Z, dtype, f"{M}x{K}x{N} {dtype} in {slabs} slabs")


def test_w_of_two_gib(rl):
    """W beyond 2^31 bytes: slabs that are addressed one by one.  Columns at the ends of tiles, of the first and the last."""
    import torch
    M, K, N = 3, 8200, 131075
    gen = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16)
    g = torch.rand((K,), generator=gen, device="cuda").add_(0.5).to(torch.bfloat16)
    W = torch.empty((K, N), dtype=torch.bfloat16, device="cuda")
    assert W.numel() * 2 > 1 << 31
    for k in range(0, K, 1025):
        W[k:k + 1025] = torch.randn((min(1025, K - k), N), generator=gen, device="cuda").mul_(K ** -0.5)
    Y = rl.rmsnorm_linear(X, g, W, 1e-5)
    torch.cuda.synchronize()
    used = rl.rl_last_launch()
    assert used[1] == 128 and used[2] > 1
    cols = torch.tensor([0, 1, 126, 127, 128, 129, 255, 256, 65535, 65536, N - 132, N - 131, N - 130, N - 4, N - 3, N - 2, N - 1], device="cuda")
    x = X.double()
    Z = (x * g.double()) @ W[:, cols].double() / torch.sqrt((x ** 2).mean(1, keepdim=True) + 1e-5)
    _check(Y[:, cols].double().cpu().numpy(), Z.cpu().numpy(), "bf16", f"{M}x{K}x{N} {used}")
