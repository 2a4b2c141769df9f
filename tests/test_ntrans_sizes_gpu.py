"""GPU tests of the nTrans kernel at the edges of its forms: rows of one wave and of one workgroup, chunks that two rows share."""
import numpy as np
import pytest

import oracle
from tests.test_ntrans import _make
from tests.util import to_device, to_host_f64

pytestmark = pytest.mark.gpu

# a chunk is 8 (16-bit) or 4 (fp32) elements; a wave's row ends at 256 (16-bit) or 128 chunks (fp32), a workgroup's
# of 256 threads at 1280, of 512 at 2560
SIZES = [1, 3, 7, 8, 9, 15, 63, 255, 257, 510, 513, 1020, 1023, 1025, 1032, 1537, 2041, 2047, 2048, 2049, 3001, 4095, 4100, 5121, 6146,
         8185, 8188, 8192, 8193, 10233, 10240, 10241,
         20473, 20480, 20481]


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("D", SIZES)
def test_row_lengths(D, dtype):
    """Against the fp64 oracle: half an ulp of the output, and fp32 sums (two of D terms, in at most 64 steps per
    thread: 1e-6 of the value is allowed for them and for the roots); nothing outside Y is written."""
    import torch
    import paper_2405_05751_amd as rl
    M = 19
    x, h, a = _make(M, D, dtype, 8300 + D)
    eps = float(np.float32(1e-6))
    n, pad = M * D, 64
    X, H, A = to_device(x, dtype), to_device(h, dtype), to_device(a, dtype)
    buf = torch.full((pad + n + pad,), 99.0, dtype=X.dtype, device="cuda")
    Y = buf[pad:pad + n].view(M, D)
    rl.rl_ntrans(X, H, A, eps, Y)
    torch.cuda.synchronize()
    assert torch.all(buf[:pad] == 99.0) and torch.all(buf[pad + n:] == 99.0)
    want = oracle.ntrans(x, h, a, dtype, eps)
    half_ulp = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 2.0 ** -24}[dtype]
    rms = np.sqrt((want ** 2).mean(axis=1, keepdims=True))
    # u = x + alpha n may cancel: its rounding is relative to its terms, which are a few rms
    bound = half_ulp * 1.001 * np.abs(want) + 1e-6 * np.abs(want) + 2e-6 * rms + 2.0 ** -25
    worst = float((np.abs(to_host_f64(Y, dtype) - want) / bound).max())
    assert worst <= 1.0, f"{M}x{D} {dtype}: |err| / bound = {worst:.3f}"


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("D", [1, 7, 63, 513, 2047, 3001, 10241])
def test_special_values_keep_to_their_row(D, dtype):
    """Rows that share a chunk with one of NaN or infinities, or of the type's largest values, are what they are without."""
    import torch
    import paper_2405_05751_amd as rl
    M = 11
    X, H, A = (to_device(t, dtype) for t in _make(M, D, dtype, 8400 + D))
    clean = rl.rl_ntrans(X, H, A, 1e-6)
    X[2], H[5], X[8], H[8] = float("nan"), float("inf"), float("-inf"), torch.finfo(X.dtype).max
    Y = rl.rl_ntrans(X, H, A, 1e-6)
    torch.cuda.synchronize()
    keep = [0, 1, 3, 4, 6, 7, 9, 10]
    assert torch.equal(Y[keep], clean[keep])
    assert torch.isnan(Y[[2, 5, 8]]).all()
