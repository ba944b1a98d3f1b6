"""The phase factors of float32 steps at the z lengths without a kernel plan of
their own, and at the plans' lengths on rows that their kernels do not divide:
cos and sin of c |k| dt are float64 values rounded once.

The state is E_x = cos(pi z / 2 dz), one mode whose transforms are exact in these
kernels (the values are 0 and +-1, and every twiddle they meet is +-1 or +-i), so
the state after a step shows the factors bit by bit:
E_x(0) = 2 A fl(C sc), |B_y(dz)| = 2 A fl(S sc), A = cells / 2, sc = fl(1 / cells)."""
import numpy as np
import pytest

from paper_2010_00409_amd import tfocus as tf

pytestmark = pytest.mark.gpu

NX, NY = 24, 8                       # 12 mode slots per row
D = 0.31
DTS = [0.37 * (i + 1) for i in range(24)] + [-0.83, 517.3, 2.0e4]


@pytest.mark.parametrize("nx,ny,nz", [(48, 64, 24), (48, 8, 48)]
                         + [(NX, NY, n) for n in (16, 32, 64, 96, 128, 192, 256, 384, 512, 768, 1024)])
def test_factors_are_rounded_float64_values(nx, ny, nz):
    g = dict(nx=nx, ny=ny, nz=nz, dx=D, dy=D, dz=D, x_min=0.0, y_min=0.0, z_min=0.0)
    state = np.zeros((6, nz, ny, nx), dtype=np.float32)
    state[0, 0::4], state[0, 2::4] = 1.0, -1.0
    cells = nx * ny * nz
    a, sc = np.float32(cells // 2), np.float32(1.0 / cells)
    out = np.empty_like(state)
    with tf.Solver(g, "f32") as s:
        for dt in DTS:
            s.set_fields(state, 0.0)
            s.advance(1, dt)
            s.get_fields(out)
            ph = dt * (2.0 * np.pi / (nz * D)) * (nz // 4)
            c, sn = np.float32(np.cos(ph)), np.float32(np.sin(ph))
            assert np.all(out[0, 0] == 2 * (np.float32(c * sc) * a)), dt
            assert np.all(np.abs(out[4, 1]) == 2 * np.abs(np.float32(sn * sc) * a)), dt


def test_a_phase_without_a_fraction_still_conserves_energy():
    nz = 96
    g = dict(nx=NX, ny=NY, nz=nz, dx=D, dy=D, dz=D, x_min=0.0, y_min=0.0, z_min=0.0)
    x = np.random.default_rng(5).standard_normal((6, nz, NY, NX)).astype(np.float32)
    with tf.Solver(g, "f32") as s:
        s.set_fields(x, 0.0)
        s.advance(1, 0.0)                        # removes the longitudinal part of E
        e0 = s.diagnostics()[0]
        s.advance(1, 1.0e18)
        e1 = s.diagnostics()[0]
    # |C + i S| is 1 to a float32 rounding of each; the longitudinal part of B
    # takes C alone, so the energy may only fall
    assert np.isfinite(e1) and e1 <= e0 * (1 + 1e-5)
