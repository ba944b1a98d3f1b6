"""Runs of several steps, whose inner steps join the inverse and the forward x
transform, give the bits of single steps: every x length and both
precisions, through graph replays, for a batch whose instances end at
different steps, and for the allocation-free entry point."""
import numpy as np
import pytest
import torch

from paper_2010_00409_amd import tfocus as tf
from synthetic import configs

pytestmark = pytest.mark.gpu

LENGTHS = [8, 16, 24, 32, 40, 48, 56, 64, 80, 96, 112, 128, 160, 192, 224, 256, 320, 384, 448, 512, 640, 768, 896, 1024]


def grid(nx, ny, nz):
    return dict(nx=nx, ny=ny, nz=nz, dx=0.21, dy=0.23, dz=0.27, x_min=0.0, y_min=0.0, z_min=0.0)


def run(g, prec, x, calls):
    with tf.Solver(g, prec) as s:
        s.set_fields(x)
        for n, dt in calls:
            s.advance(n, dt)
        out = np.empty_like(x)
        s.get_fields(out)
    return out


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx", LENGTHS)
def test_a_run_has_the_bits_of_single_steps(nx, prec):
    g = grid(nx, 8, 24)
    dtype = np.float64 if prec == "f64" else np.float32
    x = np.random.default_rng(nx).standard_normal((6, 24, 8, nx)).astype(dtype)
    one = run(g, prec, x, [(1, 0.31)] * 11)
    assert np.array_equal(run(g, prec, x, [(11, 0.31)]), one)          # a graph of 8 among them
    assert np.array_equal(run(g, prec, x, [(2, 0.31), (9, 0.31)]), one)
    state = torch.from_numpy(x).cuda()
    tf.tf_advance_noalloc(g, prec, state, 11, 0.31, stream=torch.cuda.current_stream())
    got = state.cpu().numpy()
    if prec == "f32":
        assert np.array_equal(got, one)
    else:                                                                # its tables are built on the device
        assert np.linalg.norm(got - one) <= 1e-13 * np.linalg.norm(one)


def test_batch_instances_that_end_at_different_steps():
    ps = [configs.pulse(envelope="cos2", R0=4.0, L=2.0, f_number=0.6, cep=0.1 * i) for i in range(5)]
    g = tf.tf_layer_grid(ps[0], (48, 64, 64), (0.1, 0.1, 0.1))
    win = dict(wx=32, wy=32, wz=32, cx=0.0, cy=0.0, cz=0.0)
    steps = [3, 1, 4, 0, 3]
    dst = torch.empty((5, 6, 32, 32, 32), dtype=torch.float32, device="cuda")
    with tf.Batch([g] * 5, ps, "f32") as b:
        for use_graph in (False, True, True):
            b.run(steps, [1.0] * 5, win, dst, use_graph=use_graph)
            torch.cuda.synchronize()
            for i, (p, n) in enumerate(zip(ps, steps)):
                with tf.Solver(g, "f32") as s:
                    s.set_pulse(p)
                    for _ in range(n):
                        s.advance(1, 1.0)
                    one, full = np.empty((6, 32, 32, 32), np.float32), np.empty(s.shape, np.float32)
                    s.read_focal(win, one)
                    s.get_fields(full)
                assert np.array_equal(dst[i].cpu().numpy(), one)
                assert np.array_equal(b.get_fields(i, np.empty_like(full)), full)
