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
print(linear(300, 1024, 10000), names())                         # X-hat in the workspace to tiles that form it themselves
print(linear(1, 4096, 4096), names(), b"hipMalloc" in lib.rl_last_error())
print(rec.hipGetLastError())
""")
    assert out == ["0 ['odd_kernel'] 1", "0 ['mid_kernel']", "3 [] True", "0"]


@pytest.mark.parametrize("M,K,N,dt", [(300, 1024, 10000, "F16"), (862, 1544, 2136, "BF16"), (1914, 664, 624, "BF16"), (654, 2392, 4352, "F16")])
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


# calls that could do without a workspace and are faster with one: (call, kernel, which word of its argument is the workspace)
SPARING = {
    "odd sizes, split": ("linear(8, 4095, 3001, BF16, {s})", "odd_kernel", (9, 32, 3), "lib.rl_workspace_bytes(8, 4095, 3001, BF16)"),
    "X-hat": ("linear(300, 1024, 10000, BF16, {s})", "xhat_rows_kernel", (2, 8, 0), "lib.rl_workspace_bytes(300, 1024, 10000, BF16)"),
    "attention, many heads": ("qknorm(8, 40, 4096, 128, BF16, {s})", "qkattn_kernel", (0, 72, 8), "0"),
    "attention, short sequence": ("qknorm(1, 32, 300, 128, BF16, {s})", "qkattn_kernel", (0, 72, 8), "0"),
}


@pytest.mark.parametrize("what", SPARING)
def test_streams_share_nothing(what):
    """Every stream has memory of its own for them, apart from the shared workspace too; without any (under capture, while a
    buffer is lent, too many streams, the handle that means another stream in every thread) the form that needs none runs."""
    call, kernel, (arg, size, word), query = SPARING[what]
    out = routes.run(f"""
rec.rec_watch(b"{kernel}", {arg}, {size})
def place(s):
    st = {call.format(s="s")}
    assert st == 0, lib.rl_last_error()
    got = [l for l in launches() if l.name == "{kernel}"]
    return got[0].words[{word}] if got and got[0].words[{word}] else 0
linear(1, 4096, 4096, BF16, 0)
shared_mallocs, shared_bytes = rec.rec_mallocs(), rec.rec_malloc_bytes()
at = [place(s) for s in (0, 5, 6, 5, 0)]
print(0 in at, at[3] == at[1], at[4] == at[0], len(set(at)) == 3, min(abs(a - b) for a in at for b in at if a != b) >= 4 << 20)
shared = (1 << 40, (1 << 40) + shared_bytes)
print([shared[0] <= a < shared[1] for a in at])
rec.rec_capture(V(5), 1)
print(place(5) != 0, rec.rec_mallocs() - shared_mallocs)
rec.rec_capture(V(5), 0)
print(place(2))
many = [place(100 + i) for i in range(40)]
print(len(set(many)), many[-1], rec.rec_malloc_bytes() - shared_bytes <= 16 * (24 << 20), place(6) == at[2])
lib.rl_set_workspace(V(1 << 43), 1 << 28)
print(place(6), place(7))
print({query})
""")
    assert out[:2] == ["False True True True True", "[False, False, False, False, False]"]
    assert out[2] == "False 3"
    assert out[3] == "0"
    assert out[4] == "14 0 True True"                    # 13 regions were left; the rest goes without
    assert out[5] == "0 0"
    assert out[6] == "0"


def test_default_stream_while_another_is_captured():
    """Whether the default stream is captured cannot be asked then: the calls that could do without a workspace do."""
    out = routes.run("""
rec.rec_capture(V(5), 1)
print(linear(8, 4095, 3001), names(), linear(300, 1024, 10000), names(), qknorm(1, 32, 300, 128), len(names()), rec.hipGetLastError())
""")
    assert out == ["0 ['odd_kernel'] 0 ['mid_kernel'] 0 1 0"]


@pytest.mark.parametrize("call,kernels", [
    ("linear(300, 1024, 10000, BF16, 5)", ["xhat_rows_kernel", "mid_kernel"]),
    ("linear(245, 992, 2496, BF16, 5)", ["xhat_rows_kernel", "mid_kernel", "tile_reduce_kernel"]),
    ("linear(4096, 4096, 4096, BF16, 5)", ["xhat_rows_kernel", "tile_kernel"]),
    ("linear(300, 1024, 10000, BF16, 5, 'rmsnorm_linear_noalloc')", ["xhat_rows_kernel", "mid_kernel"]),
])
def test_two_threads_on_one_stream(call, kernels):
    """The kernels of a call that pass data through a workspace are enqueued together."""
    out = routes.run(f"""
{call}
rec.rec_take()
rec.rec_launch_pause(300)
def work():
    for i in range(30):
        assert {call} == 0
threads = [threading.Thread(target=work) for i in range(3)]
for t in threads: t.start()
for t in threads: t.join()
print(names() == {kernels} * 90)
""")
    assert out == ["True"]


@pytest.mark.parametrize("M,K,N,dt", [(1443343563, 8, 16, "F16"), (1177524770, 24, 32, "F16"), (2056937954, 16, 56, "BF16")])
def test_most_rows(M, K, N, dt):
    """No launch of more threads than a grid may hold (the recorder refuses those, as HIP does)."""
    out = routes.run(f"""
print(linear({M}, {K}, {N}, {dt}), len(launches()) > 0)
""")
    assert out == ["0 True"]


def test_odd_size_kernel_can_be_asked_for():
    """RL_NAIVE with 128 columns: so it is reported, so it runs when it is asked for (aligned and tiny sizes too, in a given number of
    slabs), and a choice of the tuner's that is played back is the launch that was timed."""
    out = routes.run("""
NAIVE = 4
print(linear(24, 4096, 32003), last()[:2])
lib.rl_set_variant(NAIVE)
lib.rl_set_tuning(128, 3)
print(linear(8, 4096, 3000), last()[:3], linear(2, 64, 100), linear(8, 4096, 3001, F32), last()[:2])
lib.rl_set_tuning(128, 17)
print(linear(8, 4096, 3001))
lib.rl_set_tuning(0, 0)
print(linear(8, 4096, 3001), last()[:2])
lib.rl_set_variant(0)
lib.rl_set_tuning(0, 0)
lib.rl_autotune.argtypes = [V, V, V, F, V, L, L, L, I, I, I, V, V]
rec.rec_take()
assert lib.rl_autotune(P[0], P[1], P[2], 1e-5, P[3], 8, 4095, 3001, BF16, 0, 1, None, None) == 0
tried = {l.grid for l in launches() if l.name == "odd_kernel"}
print(sorted(g // 24 for g in tried) == list(range(1, 17)))
v, nt, ks = I(), I(), I()
lib.rl_autotune_get.argtypes = [L, L, L, I, I, V, V, V]
lib.rl_autotune_get(8, 4095, 3001, BF16, 0, *[ctypes.byref(x) for x in (v, nt, ks)])
linear(8, 4095, 3001)
tuned = [(l.name, l.grid) for l in launches()][-1]
lib.rl_autotune_clear()
lib.rl_set_variant(v.value)
lib.rl_set_tuning(nt.value, ks.value)
linear(8, 4095, 3001)
print((v.value, nt.value), tuned[0], tuned == [(l.name, l.grid) for l in launches()][-1])
""")
    assert out == ["0 (4, 128)", "0 (4, 128, 3) 2 0 (4, 0)", "2", "0 (4, 0)", "True", "(4, 128) odd_kernel True"]


def test_widths_of_128_row_tiles():
    """The tuner tries both in 1 to 8 slabs; a call's own options name them; what does not fit is refused."""
    out = routes.run("""
class Opts(ctypes.Structure):
    _fields_ = [("struct_size", Z), ("variant", I), ("columns", I), ("slabs", I), ("waves", I), ("rem_slabs", I), ("workspace", V), ("bytes", Z)]
lib.rl_autotune.argtypes = [V, V, V, F, V, L, L, L, I, I, I, V, V]
lib.rmsnorm_linear_ex.argtypes = [V, V, V, F, V, L, L, L, I, V, V]
assert lib.rl_autotune(P[0], P[1], P[2], 1e-5, P[3], 256, 4096, 1024, BF16, 0, 1, None, None) == 0
print(sorted({(l.grid, "Li64" in l.mangled) for l in launches() if l.name == "mid_kernel"}) ==
      sorted([(32 * s, True) for s in range(1, 9)] + [(16 * s, False) for s in range(1, 9)]))
def ex(columns, slabs, M=256, K=4096, N=1024):
    o = Opts(ctypes.sizeof(Opts), 5, columns, slabs, 0, 0, None, 0)
    return lib.rmsnorm_linear_ex(P[0], P[1], P[2], 1e-5, P[3], M, K, N, BF16, ctypes.byref(o), None)
print(ex(64, 3), last(), ex(128, 0), last(), ex(256, 2), last()[1:3])
print(ex(128, 17), ex(64, 1, 256, 4096, 1 << 22), lib.rl_last_error())
""")
    assert out == ["True", "0 (5, 64, 3, 96) 0 (5, 128, 1, 16) 0 (256, 2)",
                   "2 2 b'128-row tiles: 1 to 16 slabs, K < 2^23, N < 2^22, and a slab of W below 2 GiB'"]


@pytest.mark.parametrize("M,K,N,dt,kernels", [
    (509, 4096, 4160, "BF16", ["xhat_rows_kernel", "mid_kernel"]),                           # 264 row blocks, 256 compute units
    (292, 6536, 3688, "F16", ["xhat_rows_kernel", "mid_kernel", "tile_reduce_kernel"]),      # 256 x 256 tiles would beat the row blocks too
    (1000, 1000, 1000, "BF16", ["mid_kernel"]),
    (509, 4096, 4096, "BF16", ["skinny_kernel"]), (128, 2048, 2048, "BF16", ["skinny_kernel"]),
])
def test_row_blocks_or_128_row_tiles(M, K, N, dt, kernels):
    """Row blocks only where they are not the slower form, through either entry point."""
    out = routes.run(f"""
print(linear({M}, {K}, {N}, {dt}), names())
print(linear({M}, {K}, {N}, {dt}, 0, 'rmsnorm_linear_noalloc'), [n for n in names() if "scratch_clear" not in n])
""")
    assert out == [f"0 {kernels}"] * 2


@pytest.mark.parametrize("M,K,N,kernel", [
    (1, 152, 34028, "f32_kernel"), (1, 4096, 32000, "f32_kernel"), (4, 2048, 20000, "f32_kernel"), (16, 4164, 55336, "f32_kernel"),
    (17, 2612, 46528, "f32_kernel"), (32, 5448, 30728, "f32_kernel"),
    (33, 4392, 37972, "f32_kernel"), (47, 1952, 36224, "f32_kernel"), (33, 224, 23864, "f32_tile_kernel"), (48, 4376, 18748, "f32_tile_kernel"),
    (49, 2388, 23784, "f32_tile_kernel"), (64, 4096, 28672, "f32_tile_kernel"), (65, 68, 20000, "f32_tile_kernel"),
])
def test_fp32_rows_of_one_block(M, K, N, kernel):
    """Tiles of 64 rows only where they are not the slower form: the kernel for row blocks works on 16 rows at a time."""
    out = routes.run(f"""
print(linear({M}, {K}, {N}, F32), names())
""")
    assert out == [f"0 ['{kernel}']"]


SPLIT, UNSPLIT, WIDE = ["xhat_rows_kernel", "mid_kernel", "tile_reduce_kernel"], ["mid_kernel"], ["xhat_rows_kernel", "tile_kernel"]


@pytest.mark.parametrize("fn,M,K,N,dt,kernels", [
    # a workgroup or less to a unit: long K, one row of tiles and several, up to K = 1280 and 2500
    ("rmsnorm_gated_mlp", 109, 2840, 4840, "F16", SPLIT), ("rmsnorm_linear", 104, 3256, 9352, "F16", SPLIT),
    ("rmsnorm_linear", 127, 1528, 5864, "F16", SPLIT), ("rmsnorm_gated_mlp", 887, 3696, 904, "F16", SPLIT), ("rmsnorm_linear", 1036, 2672, 1040, "BF16", SPLIT),
    ("rmsnorm_linear", 862, 1544, 2136, "BF16", UNSPLIT), ("rmsnorm_linear", 7117, 224, 352, "BF16", UNSPLIT),
    # many rows
    ("rmsnorm_linear", 5988, 3808, 192, "F16", UNSPLIT), ("rmsnorm_linear", 4939, 328, 1632, "F16", UNSPLIT), ("rmsnorm_linear", 6126, 448, 832, "F16", UNSPLIT),
    # a full chip of 128-column tiles
    ("rmsnorm_gated_mlp", 3414, 7632, 2584, "F16", WIDE), ("rmsnorm_gated_mlp", 1118, 3400, 3560, "F16", WIDE), ("rmsnorm_linear", 731, 768, 10840, "F16", WIDE),
])
def test_tiles_that_form_x_hat_themselves(fn, M, K, N, dt, kernels):
    """128-row tiles without a first kernel only where that is not slower than a split, or 256 x 256 tiles, with one."""
    out = routes.run(f"""
lib.rmsnorm_gated_mlp.argtypes = [V, V, V, F, V, L, L, L, I, V]
print(linear({M}, {K}, {N}, {dt}, 0, {fn!r}), [n for n in names() if "scratch_clear" not in n])
""")
    assert out == [f"0 {kernels}"]


@pytest.mark.parametrize("fn,M,K,N,dt", [("rmsnorm_linear", 66, 1344, 7776, "F16"), ("rmsnorm_linear", 128, 1712, 6144, "F16"),
                                        ("rmsnorm_gated_mlp", 93, 1464, 3232, "F16")])
def test_tiles_in_place_of_split_row_blocks_without_a_workspace(fn, M, K, N, dt):
    """A split is the faster form here; without a workspace (under capture before any other call) the one that needs none runs."""
    out = routes.run(f"""
lib.rmsnorm_gated_mlp.argtypes = [V, V, V, F, V, L, L, L, I, V]
rec.rec_capture(V(7), 1)
print(linear({M}, {K}, {N}, {dt}, 7, {fn!r}), rec.rec_mallocs(), names())
rec.rec_capture(V(7), 0)
print(linear({M}, {K}, {N}, {dt}, 7, {fn!r}), [n for n in names() if "clear" not in n])
""")
    assert out[0] == "0 0 ['mid_kernel']" and out[1] == f"0 {SPLIT}"


@pytest.mark.parametrize("M,K,N", [(1, 8, 16), (1, 896, 2232), (2, 1024, 1952), (3, 304, 6472), (4, 1000, 1016), (4, 120, 16384)])
def test_one_to_four_rows_of_a_small_w(M, K, N):
    """Narrow tiles where they keep what the GEMV kernel has for a product: in bf16 and for the plain product, not with the norm in fp16."""
    out = routes.run(f"""
lib.rmsnorm_gated_mlp.argtypes = [V, V, V, F, V, L, L, L, I, V]
print(linear({M}, {K}, {N}), names(), linear({M}, {K}, {N}, F16), names(), linear({M}, {K}, {N // 16 * 8}, BF16, 0, "rmsnorm_gated_mlp"), names(),
      linear({M}, {K}, {N // 16 * 8}, F16, 0, "rmsnorm_gated_mlp"), names())
print([(lib.matmul(P[0], P[2], P[3], {M}, {K}, {N}, dt, None), names()) for dt in (F16, BF16)])
""")
    small, gemv = "['small_kernel']", "['gemv_splitk_kernel']"
    assert out == [f"0 {small} 0 {gemv} 0 {small} 0 {gemv}", f"[(0, {small}), (0, {small})]"]


@pytest.mark.parametrize("M,K,N,gated,want", [
    (1, 40, 18432, 0, "gemv_splitk_kernel"), (1, 8, 17152, 1, "gemv_splitk_kernel"), (4, 64, 31248, 0, "gemv_splitk_kernel"),
    (29, 128, 17408, 1, "skinny_kernel"), (55, 32, 17680, 0, "skinny_kernel"), (5, 96, 21504, 1, "skinny_kernel"), (6, 24, 24320, 0, "skinny_kernel"),
    (12, 2432, 2008, 0, "skinny_kernel"), (15, 2384, 3208, 0, "skinny_kernel"), (48, 1328, 8872, 0, "skinny_kernel"), (16, 1488, 4032, 1, "skinny_kernel"),
    (32, 2304, 1344, 0, "skinny_kernel"), (1, 1024, 640, 1, "gemv_splitk_kernel"), (1, 1024, 640, 0, "small_kernel"), (1, 896, 640, 1, "small_kernel"),
    (55, 32, 16384, 0, "small_kernel"), (1, 40, 16384, 0, "small_kernel"), (15, 1168, 6208, 0, "small_kernel"), (22, 2272, 448, 0, "small_kernel")])
def test_small_w_where_narrow_tiles_are_slower(M, K, N, gated, want):
    """More than one round of 64-column tiles, a large W or a long K near the line, one gated row: timed slower in narrow tiles; and sizes beside them."""
    out = routes.run(f"""
print(linear({M}, {K}, {N // 2 if gated else N}, BF16, 0, {"rmsnorm_gated_mlp" if gated else "rmsnorm_linear"!r}), [n for n in names() if "clear" not in n])
""")
    assert out == [f"0 ['{want}']"]


@pytest.mark.parametrize("why", ["capture", "lent", "memory"])
def test_small_w_without_a_workspace(why):
    """Where W is small a call that would be split over K runs unsplit when no workspace is to be had: the GEMV kernel in one slab up to
    four rows (with the norm in fp16 as with one), the narrow tiles near their line.  Other splits are refused."""
    out = routes.run(f"""
import math, random
why = {why!r}
lib.rmsnorm_gated_mlp_interleaved.argtypes = [V, V, V, F, V, L, L, L, I, V]
def none(on):
    if why == "capture": rec.rec_capture(V(7), int(on))
    elif why == "lent": lib.rl_set_workspace(V(1 << 43) if on else None, (1280 << 10) + 16)
    else: rec.rec_fail_mallocs(100000 if on else 0)
def call(M, K, N, dt, fn="rmsnorm_linear"):
    st = linear(M, K, N if fn == "rmsnorm_linear" else N // 2, dt, 7, fn)
    return st, [n for n in names() if "clear" not in n], last()[2]
r = random.Random(8)
spread = lambda lo, hi: int(math.exp(r.uniform(math.log(lo), math.log(hi))))
none(True)
for n in range(600):
    K = 8 * spread(1, 128)
    M, N, dt = r.randint(1, 4), 16 * spread(1, max(1, min(2048, 2000000 // K // 16))), r.choice((F16, BF16))
    fn = r.choice(("rmsnorm_linear", "rmsnorm_gated_mlp"))
    st, ks, slabs = call(M, K, N, dt, fn)
    assert st == 0 and ks in (["gemv_splitk_kernel"], ["small_kernel"], ["skinny_kernel"]) and slabs == 1, (M, K, N, dt, fn, st, ks, slabs)
    assert dt == BF16 or (M == 1 and N >= 10240) or ks == ["gemv_splitk_kernel"], (M, K, N, fn, ks)
for M, K, N, fn in ((15, 2384, 3208, "rmsnorm_linear"), (32, 2304, 1344, "rmsnorm_linear"), (16, 1488, 4032, "rmsnorm_gated_mlp")):
    print(call(M, K, N, BF16, fn)[:2])
print([call(*s)[:2] for s in ((16, 4096, 6144, BF16), (4, 1504, 1000, F16), (1, 4096, 4096, BF16))])
none(False)
print([call(15, 2384, 3208, BF16)[1], call(4, 1000, 1016, F16)[1:]])
""")
    bad = 3 if why == "memory" else 4
    assert out == ["(0, ['small_kernel'])"] * 3 + [f"[({bad}, []), ({bad}, []), ({bad}, [])]", "[['skinny_kernel'], (['gemv_splitk_kernel'], 8)]"]


def test_workspace_query_covers_the_gated_block():
    """What rl_workspace_bytes says of (M, K, N) holds for the plain call and for the gated block with H = N / 2 in both layouts: 0 only
    if none takes partial sums (or X-hat) through the shared workspace, else enough for each to launch what it would with any amount."""
    out = routes.run("""
import math, random
for fn in ("rmsnorm_gated_mlp", "rmsnorm_gated_mlp_interleaved"):
    getattr(lib, fn).argtypes = [V, V, V, F, V, L, L, L, I, V]
r = random.Random(5)
spread = lambda lo, hi: int(math.exp(r.uniform(math.log(lo), math.log(hi))))
def go(fn, M, K, N, dt):
    st = linear(M, K, N if fn == "rmsnorm_linear" else N // 2, dt, 7, fn)
    return st, [(l.mangled, l.grid) for l in launches()]
shapes = [(5, 1984, 2880, BF16), (29, 2224, 1040, F16), (5, 2456, 1504, BF16), (12, 2216, 128, BF16)]
for n in range(1500):
    shapes.append((spread(1, 64) if n % 3 else spread(65, 1024), 8 * spread(8, 1024), 128 * spread(1, 128) if n % 2 else 16 * spread(4, 1024),
                   r.choice((F16, BF16, BF16, F32))))
shared = 0
for M, K, N, dt in shapes:
    need = lib.rl_workspace_bytes(M, K, N, dt)
    for fn in ["rmsnorm_linear", "rmsnorm_gated_mlp"] + ["rmsnorm_gated_mlp_interleaved"] * (N % 128 == 0):
        rec.rec_capture(V(7), 1)                         # no workspace can be had then
        without = go(fn, M, K, N, dt)
        rec.rec_capture(V(7), 0)
        lib.rl_set_workspace(V(1 << 43), 1 << 32)
        any_amount = go(fn, M, K, N, dt)
        assert any_amount[0] == 0
        if need:
            lib.rl_set_workspace(V(1 << 43), need)
            assert go(fn, M, K, N, dt) == any_amount, (fn, M, K, N, dt)
        lib.rl_set_workspace(None, 0)
        assert need or without == any_amount, (fn, M, K, N, dt)
        shared += need != 0
print(shared > 500)
""")
    assert out == ["True"]


@pytest.mark.parametrize("M,K,N", [(16, 264, 12808), (64, 264, 12296), (64, 272, 12800), (8, 512, 512)])
def test_tuner_times_both_kernels_of_the_skinny_variant(M, K, N):
    """The narrow tiles in 64 columns and the 64-column tiles in one slab are different launches of as many workgroups."""
    out = routes.run(f"""
lib.rl_autotune.argtypes = [V, V, V, F, V, L, L, L, I, I, I, V, V]
assert lib.rl_autotune(P[0], P[1], P[2], 1e-5, P[3], {M}, {K}, {N}, BF16, 0, 20, None, None) == 0
tried = [(l.name, l.grid) for l in launches()]           # (a candidate that is dropped has been launched once)
lib.rl_set_variant(2)
lib.rl_set_tuning(64, 1)
assert linear({M}, {K}, {N}) == 0
tiles = launches()[-1]
lib.rl_set_tuning(0, 0)
assert linear({M}, {K}, {N}) == 0
narrow = launches()[-1]
print(tiles.name, narrow.name, *[tried.count((l.name, l.grid)) >= 20 for l in (tiles, narrow)], narrow.grid == tiles.grid)
""")
    assert out == [f"skinny_kernel small_kernel True True {N > 10000}"]


SMALL = r"_ZN5rmsnl12small_kernelINS_4(Bf16|Fp16)ELi(\d+)ELi(\d+)ELb(\d)ELb(\d)E"


def test_kernel_of_every_narrow_tile_test():
    """tests/test_small_gpu.py reads columns and slabs, which 64-column tiles of the other kernel report as well: here its calls by name."""
    import test_small_gpu as t
    out = routes.run(f"""
for fn in ("rmsnorm_gated_mlp", "rmsnorm_gated_mlp_interleaved"):
    getattr(lib, fn).argtypes = [V, V, V, F, V, L, L, L, I, V]
def went():
    l, = launches()
    m = re.match(r"{SMALL}", l.mangled)
    return (m.group(1), *map(int, m.groups()[1:])) if m else l.name
blocks = lambda M: 4 if M > 64 else -(-M // 16)
kinds = ((F16, "Fp16"), (BF16, "Bf16"))
for M, K, N, columns in {t.EDGES}:
    for dt, name in kinds:
        assert linear(M, K, N, dt) == 0
        want = "gemv_splitk_kernel" if M <= 4 and dt == F16 else (name, blocks(M), columns // 16, 1, 0)
        assert went() == want, (M, K, N, dt)
for sizes, fns in (({t.BLOCKS}, ["rmsnorm_linear"]), ({t.GATED}, ["rmsnorm_gated_mlp", "rmsnorm_gated_mlp_interleaved"])):
    for M, K, N, dtype in sizes:
        for fn in fns:
            dt, name = kinds[dtype == "bf16"]
            assert linear(M, K, N, dt, 0, fn) == 0
            w = went()
            assert w[:2] == (name, blocks(M)) and w[3:] == (1, int(len(fns) == 2)), (M, K, N, dt, fn, w)
for M, dt in ((7, BF16), (40, F16)):
    assert linear(M, 264, 520, dt) == 0
    a = went()
    assert lib.matmul(P[0], P[2], P[3], M, 264, 520, dt, None) == 0
    b = went()
    assert (a[1], a[3:]) == (blocks(M), (1, 0)) and (b[1], b[3:]) == (blocks(M), (0, 0))
print("ok")
""")
    assert out == ["ok"]


def test_kernel_of_every_128_column_test():
    """The tests that ask the skinny variant for 128 columns run its own kernel, in all its row counts."""
    import test_gated_gpu as g
    import test_parity_gpu as t
    runs = [(M, 64 * R - 24, 136) for M in (3, 16, 17, 33, 64, 65, 130) for R in t.RUNS]
    out = routes.run(f"""
lib.rl_set_variant(2)
def went(call):
    assert call() == 0
    l = [l for l in launches() if l.name != "clear_counters_kernel"]
    m = re.match(r"_ZN5rmsnl13skinny_kernelINS_4(?:Bf16|Fp16)ELi(\\d)ELb(\\d)ELb(\\d)ELi(\\d)E", l[0].mangled)
    assert len(l) == 1 and m, l[0].mangled
    return tuple(map(int, m.groups()))
seen = set()
lib.rl_set_tuning(128, 0)
for M, K, N in {t.RAGGED + [(16, 1024, 4096), (5, 520, 776), (8, 512, 512), (4, 256, 256), (65, 264, 136), (128, 1032, 520), (200, 4096, 1024), (1024, 520, 264)]}:
    w = went(lambda: linear(M, K, N))
    assert w[:3] == (4 if M > 64 else -(-M // 16), 1, 0) and (w[3] > 0) == (M > 64), (M, K, N, w)
for M, K, H in {g.SHAPES}:
    w = went(lambda: linear(M, K, H, BF16, 0, "rmsnorm_gated_mlp"))
    assert w[:3] == (4 if M > 64 else -(-M // 16), 1, 1), (M, K, H, w)
lib.rl_set_tuning(128, 1)
for M, K, N in {runs}:
    seen.add(went(lambda: linear(M, K, N)))
    seen.add(went(lambda: linear(M, K, N, BF16, 0, "rmsnorm_gated_mlp")))
    seen.add(went(lambda: lib.matmul(P[0], P[2], P[3], M, K, N, BF16, None)))
print(len(seen))
""")
    assert out == ["15"]
