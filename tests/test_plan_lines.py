"""Lines of the shipped plans that hold for every grid of an nz (host only): only
where the z passes of that length have kernels to choose among."""
from paper_2010_00409_amd import tfocus as tf
from synthetic import configs


def test_lines_by_nz_stand_where_a_variant_differs(monkeypatch):
    for v in ("TFOCUS_ROW_BLOCK", "TFOCUS_GENERIC_KERNELS", "TFOCUS_ZVARIANT", "TFOCUS_YSTRIP"):
        monkeypatch.delenv(v, raising=False)
    lines = [l.split() for l in open(tf.DEFAULT_PLANS) if l.strip() and not l.startswith("#")]
    by_nz = {int(l[4]) for l in lines if l[2] == l[3] == "0"}
    assert by_nz == {128, 192, 256, 512}
    assert tf.tf_kernel_plan(dict(configs.cube_grid(64, 0.1), nx=96), "f32") == (8, True, 0, 64)
