"""Where tf_advance_current takes its current from: an array that is handed over
as device memory but is none of the solver's device (here pinned and pageable
host memory) is copied first, never read by a kernel in place."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2010_00409_amd import tfocus as tf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_memory_that_is_not_the_devices_is_copied(prec):
    dtype = np.float64 if prec == "f64" else np.float32
    nz, ny, nx = 32, 16, 24
    g = dict(nx=nx, ny=ny, nz=nz, dx=0.31, dy=0.3, dz=0.29, x_min=0.0, y_min=0.0, z_min=0.0)
    rng = np.random.default_rng(3)
    state = rng.standard_normal((6, nz, ny, nx)).astype(dtype)
    j = rng.standard_normal((3, nz, ny, nx)).astype(dtype)
    pinned = torch.from_numpy(j).pin_memory()
    outs = []
    for ptr, dev in ((torch.from_numpy(j).cuda(), None), (pinned.data_ptr(), 1), (j.ctypes.data, 1)):
        with tf.Solver(g, prec) as s:
            s.set_fields(state, 0.0)
            if dev is None:
                s.advance_current(ptr, 0.43)
            else:
                assert tf.load().tf_advance_current(s.h, ctypes.c_void_p(ptr), dev, 0.43) == tf.TF_OK, tf.tf_last_error()
            out = np.empty(s.shape, dtype=dtype)
            s.get_fields(out)
            outs.append(out)
    assert np.array_equal(outs[1], outs[0]) and np.array_equal(outs[2], outs[0])
