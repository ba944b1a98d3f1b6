"""Kernel names in the bench line (host only): the tuned z kernels are float32's."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402


@pytest.mark.parametrize("nz", [64, 96, 128, 192, 256, 512, 1024])
def test_float64_columns_are_named_by_the_kernel_that_runs(nz):
    assert bench.pass_kernels((8, True, 11), nz, "f64")["z_step"] == "k_z_res"
    assert bench.pass_kernels((8, False, 0), nz, "f64")["z_step"] == "k_z"
    want = {128: "k_z_fast", 192: "k_z_fast", 256: "k_z_wave256", 512: "k_z_wave"}
    assert bench.pass_kernels((8, True, 11), nz, "f32")["z_step"] == want.get(nz, "k_z_res")
