"""Steps with a current over the lengths of the z axis that its kernels split
differently (residues of 3, 5, 7 and 8, the generic kernel below them), with
the current read from host memory, from device memory and from a device array
off the 16-byte grid, against the float64 oracle.  Tolerances (relative L2 over
all six components, one step): float64 <= 1e-12, float32 <= 1e-5."""
import numpy as np
import pytest

from oracle import psatd
from paper_2010_00409_amd import tfocus as tf

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}
D = 0.31


def inputs(shape):
    g = dict(nx=shape[2], ny=shape[1], nz=shape[0], dx=D, dy=0.9 * D, dz=1.1 * D, x_min=0.0, y_min=0.0, z_min=0.0)
    rng = np.random.default_rng(shape[0] + shape[1])
    E, B, J = (rng.standard_normal((3,) + shape) for _ in range(3))
    h = (g["dz"], g["dy"], g["dx"])
    _, B = psatd.step_fft(E, B, h, 0.0, project_b_first=True)
    return g, h, E, B, J


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nz", [8, 16, 24, 40, 56, 64, 80, 112, 128, 192, 224, 256, 320, 384, 448, 512, 640, 768, 1024])
def test_current_step_over_z_lengths(nz, prec):
    import torch
    if prec == "f64" and nz > 768:
        pytest.skip("nine float64 columns of more than 768 elements are refused")
    shape = (nz, 8 if nz % 3 else 24, 16 if nz % 5 else 24)
    g, h, E, B, J = inputs(shape)
    dtype = np.float64 if prec == "f64" else np.float32
    state, j = np.concatenate([E, B]).astype(dtype), J.astype(dtype)
    st64, j64 = state.astype(np.float64), j.astype(np.float64)
    ref = np.concatenate(psatd.step_fft_current(st64[:3], st64[3:], j64, h, 0.43))
    flat = torch.from_numpy(np.concatenate([np.zeros(1, dtype), j.ravel()])).cuda()
    sources = dict(host=j, device=torch.from_numpy(j).cuda(), shifted=flat[1:].view(j.shape))
    outs = {}
    for name, src in sources.items():
        with tf.Solver(g, prec) as s:
            s.set_fields(np.ascontiguousarray(state), 0.0)
            s.advance_current(src, 0.43)
            outs[name] = np.empty(s.shape, dtype=dtype)
            s.get_fields(outs[name])
    err = np.linalg.norm((outs["device"].astype(np.float64) - ref).ravel()) / np.linalg.norm(ref.ravel())
    assert err <= TOL[prec]
    assert np.array_equal(outs["host"], outs["device"])
    assert np.array_equal(outs["shifted"], outs["device"])
