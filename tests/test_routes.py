"""Which kernels a call launches and what memory it takes for them, without a GPU (see tests/host/routes.py)."""
import pytest

from tests.host import routes


@pytest.mark.parametrize("M,K,N", [(24, 4096, 32003), (24, 4095, 32003), (8, 4095, 3001), (8, 4096, 3001), (300, 513, 130)])
@pytest.mark.parametrize("dt", ["F16", "BF16"])
def test_odd_sizes_under_capture_before_any_other_call(M, K, N, dt):
    """Nothing may be allocated then; the matrix-core kernel runs all the same, unsplit."""
    out = routes.run(f"""
rec.rec_capture(V(7), 1)
print(linear({M}, {K}, {N}, {dt}, 7), rec.rec_mallocs(), names(), last()[2])
""")
    assert out == ["0 0 ['odd_kernel'] 1"]


def test_failed_allocation():
    """Calls that have a form without a workspace run it, and HIP's last error does not stay behind to be taken for theirs;
    the others say what failed."""
    out = routes.run("""
rec.rec_fail_mallocs(100)
print(linear(8, 4096, 3001), names(), last()[2])                 # a split over K gives way to none
print(linear(300, 1024, 10000), names())                         # X-hat in the workspace to row blocks
print(linear(1, 4096, 4096), names(), b"hipMalloc" in lib.rl_last_error())
print(rec.hipGetLastError())
""")
    assert out == ["0 ['odd_kernel'] 1", "0 ['skinny_kernel']", "3 [] True", "0"]


@pytest.mark.parametrize("M,K,N,dt", [(300, 1024, 10000, "F16"), (89, 1280, 12712, "BF16"), (1914, 664, 624, "BF16"), (654, 2392, 4352, "F16")])
def test_mid_size_products_without_a_workspace(M, K, N, dt):
    """Where the 128-row tiles form X-hat themselves a call is one launch, and two streams have nothing in common."""
    out = routes.run(f"""
print(linear({M}, {K}, {N}, {dt}), rec.rec_mallocs(), names(), lib.rl_workspace_bytes({M}, {K}, {N}, {dt}))
""")
    assert out == ["0 0 ['mid_kernel'] 0"]


def test_row_block_sizes_launch_the_same_through_both_entry_points():
    """65 to 1024 rows where row blocks are the alternative: what rmsnorm_linear_noalloc runs, rmsnorm_linear runs."""
    out = routes.run("""
import math, random
r = random.Random(3)
spread = lambda lo, hi: int(math.exp(r.uniform(math.log(lo), math.log(hi))))
ran = 0
for n in range(6000):
    M, K, N, dt = spread(65, 1024), 8 * spread(16, 1024), 8 * spread(16, 2048), r.choice((F16, BF16))
    blocks = (M + 63) // 64
    if blocks * K * N > (1.4e8 if N <= 6144 or blocks == 2 else 0.9e8):
        continue
    st = linear(M, K, N, dt, 0, "rmsnorm_linear_noalloc")
    a = [(l.mangled, l.grid) for l in launches() if l.name.startswith(("skinny", "xhat", "mid", "tile"))]
    if st == 4:                                          # partial sums that the scratch does not hold: refused
        continue
    assert st == 0 and linear(M, K, N, dt) == 0
    b = [(l.mangled, l.grid) for l in launches() if l.name.startswith(("skinny", "xhat", "mid", "tile"))]
    assert a == b, (M, K, N, dt, a, b)
    ran += 1
print(ran > 2000)
""")
    assert out == ["True"]
