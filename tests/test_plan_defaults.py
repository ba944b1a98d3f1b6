"""Plan lines that hold for every grid of an nz (host only)."""
import os

from paper_2010_00409_amd import tfocus as tf
from synthetic import configs


def test_plan_line_for_every_grid_of_an_nz(tmp_path, monkeypatch):
    for v in ("TFOCUS_ROW_BLOCK", "TFOCUS_GENERIC_KERNELS", "TFOCUS_ZVARIANT", "TFOCUS_YSTRIP"):
        monkeypatch.delenv(v, raising=False)
    plan = tmp_path / "plans.txt"
    plan.write_text("unknown f32 0 0 256 8 1 4 0\n"
                    "unknown f32 256 256 256 256 1 7 0.7\n")
    old = os.environ.get("TFOCUS_PLAN_FILE") or tf.DEFAULT_PLANS
    tf.tf_set_plan_file(str(plan))
    try:
        cube = configs.cube_grid(256, 0.1)
        assert tf.tf_kernel_plan(cube, "f32") == (256, True, 7, 64)          # its own line
        assert tf.tf_kernel_plan(dict(cube, nx=96), "f32") == (8, True, 4, 64)
        assert tf.tf_kernel_plan(dict(cube, nx=96), "f64") == (8, True, 0, 64)
        assert tf.tf_kernel_plan(dict(cube, nz=192), "f32") == (8, True, 0, 64)
    finally:
        tf.tf_set_plan_file(old)
