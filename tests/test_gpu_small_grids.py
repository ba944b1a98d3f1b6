"""Both sides of the number of columns up to which a y or z length takes the
generic kernels, against the float64 oracle (the grids of the other column tests
lie below it).  Rows that the y strips do not divide, row blocks on both sides of
linear addressing.  Tolerances as for every other step: float64 1e-12, float32
1e-5 relative L2 per step."""
import numpy as np
import pytest

from oracle import psatd
from paper_2010_00409_amd import tfocus as tf

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}


def check(nx, ny, nz, prec):
    g = dict(nx=nx, ny=ny, nz=nz, dx=0.31, dy=0.27, dz=0.23, x_min=0.0, y_min=0.0, z_min=0.0)
    x = np.random.default_rng(nx + ny + nz).standard_normal((6, nz, ny, nx))
    x = x.astype(np.float64 if prec == "f64" else np.float32)
    with tf.Solver(g, prec) as s:
        s.set_fields(x)
        s.advance(1, 0.57)
        got = np.empty(s.shape, dtype=x.dtype)
        s.get_fields(got)
    E, B = psatd.step_fft(x[:3].astype(np.float64), x[3:].astype(np.float64), (0.23, 0.27, 0.31), 0.57)
    ref = np.concatenate([E, B])
    assert np.linalg.norm(got - ref) <= TOL[prec] * np.linalg.norm(ref)


# 168 columns per x row: 48 planes of them are 8064, 56 are 9408
@pytest.mark.parametrize("prec,n,planes", [(p, n, m) for p in ("f64", "f32") for n in (40, 56) for m in (48, 56)]
                         + [(p, n, m) for p, ns in (("f64", (80, 112, 128, 160, 224, 256, 320)), ("f32", (80, 112)))
                            for n in ns for m in (24, 32)]
                         + [("f64", n, m) for n in (384, 448, 512) for m in (48, 56)])
def test_y_lengths_on_both_sides(prec, n, planes):
    check(56, n, planes, prec)


@pytest.mark.parametrize("prec,n,rows", [("f32", n, m) for n in (24, 40, 56) for m in (24, 32)]
                         + [("f64", n, m) for n in (24, 40, 48) for m in (96, 112)]
                         + [("f64", n, m) for n in (80, 112, 128, 160, 224, 256) for m in (48, 56)])
def test_z_lengths_on_both_sides(prec, n, rows):
    check(112 if n in (24, 40, 48, 56) and prec == "f32" else 56, rows, n, prec)


@pytest.mark.parametrize("ny", [96, 112])
def test_z_of_56_points_on_both_sides(ny):
    check(224, ny, 56, "f64")            # 64512 and 75264 columns


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ny,row_block", [(56, 8), (80, 16), (112, 4), (256, 64), (384, 2), (384, 128), (448, 1), (512, 512)])
def test_row_blocks_beyond_the_small_grids(ny, row_block, prec, monkeypatch):
    monkeypatch.setenv("TFOCUS_ROW_BLOCK", str(row_block))
    check(56, ny, 56, prec)
