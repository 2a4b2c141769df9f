"""The peaks that bench.py holds a launch against."""
import types

import pytest

import bench


@pytest.mark.parametrize("dtype,launch,peak", [
    ("bf16", ("tile_pre", 256, 8, 1024), 2500.0), ("f16", ("skinny", 128, 1, 224), 2500.0),
    ("f32", ("f32", 64, 1, 2048), 157.3),
    ("f32", ("f32", 128, 1, 512), 2500.0 / 6),           # three bf16 numbers to an fp32 one, six of the nine products
])
def test_peak_of_the_instructions_that_run(dtype, launch, peak):
    res = {"launch": dict(zip(("variant", "columns", "slabs", "workgroups"), launch)), "TFLOPs": 100.0, "variant": launch[0], "us_per_step": 1.0}
    roof = bench.roofline_of("2048x4096x4096", res, types.SimpleNamespace(M=2048, dtype=dtype, flops=1), False)
    assert roof["peak"] == pytest.approx(peak) and roof["frac"] == pytest.approx(100.0 / peak)
