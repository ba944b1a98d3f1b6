"""Steps whose y or z axis is one lane group of the column kernels (up to 64
points), with rows that their strips divide and do not, and row blocks on both
sides of their linear addressing, against the float64 oracle.  Tolerances as
for every other step: float64 1e-12, float32 1e-5 relative L2 per step."""
import numpy as np
import pytest

from oracle import psatd
from paper_2010_00409_amd import tfocus as tf

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx", [8, 32, 56])
@pytest.mark.parametrize("n", [8, 16, 24, 32, 40, 48, 56, 64])
def test_short_axes(n, nx, prec, monkeypatch):
    for ny, nz, block in ((n, 8, "8"), (8, n, "8"), (n, n, "8"), (n, 24, "1"), (n, 16, "2")):
        monkeypatch.setenv("TFOCUS_ROW_BLOCK", block)
        g = dict(nx=nx, ny=ny, nz=nz, dx=0.31, dy=0.27, dz=0.23, x_min=0.0, y_min=0.0, z_min=0.0)
        x = np.random.default_rng(nx + ny + nz).standard_normal((6, nz, ny, nx))
        x = x.astype(np.float64 if prec == "f64" else np.float32)
        with tf.Solver(g, prec) as s:
            s.set_fields(x)
            s.advance(2, 0.57)
            got = np.empty(s.shape, dtype=x.dtype)
            s.get_fields(got)
        E, B = x[:3].astype(np.float64), x[3:].astype(np.float64)
        for _ in range(2):
            E, B = psatd.step_fft(E, B, (0.23, 0.27, 0.31), 0.57)
        ref = np.concatenate([E, B])
        assert np.linalg.norm(got - ref) <= 2 * TOL[prec] * np.linalg.norm(ref), (ny, nz, block)
