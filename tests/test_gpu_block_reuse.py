"""Which device blocks are kept from destroyed solvers: reuse by address, and
their return."""
import pytest
import torch

from paper_2010_00409_amd import tfocus as tf
from synthetic import configs

pytestmark = pytest.mark.gpu

N, D = 128, 1.0 / 8
P = dict(envelope="cos2", R0=6.0, L=2.0, f_number=0.8)
STATE = 6 * N ** 3 * 4               # 50 MB: a block that is kept


def grid(nx=N):
    return tf.tf_layer_grid(configs.pulse(**P), (nx, N, N), (D, D, D))


def room():
    tf.tf_release_memory()
    avail, total = torch.cuda.mem_get_info()
    if avail < 0.6 * total:
        pytest.skip("blocks are kept only while half of the device is free")


def solver_pointer(nx=N):
    with tf.Solver(grid(nx), "f32") as s:
        return s.state_ptr()


def test_a_solver_takes_the_blocks_of_the_one_before_it_until_they_are_released():
    room()
    with tf.Solver(grid(), "f32") as s:
        base = torch.cuda.mem_get_info()[0]
        first = s.state_ptr()
    assert torch.cuda.mem_get_info()[0] - base < STATE               # kept
    with tf.Solver(grid(), "f32") as s:
        second = s.state_ptr()
        with tf.Solver(grid(), "f32") as t:                          # both blocks are in use
            assert t.state_ptr() not in (first, second)
    assert second == first                                           # the older of two of one size
    assert solver_pointer(112) != 0                                  # up to a quarter larger than asked for
    tf.tf_release_memory()
    assert torch.cuda.mem_get_info()[0] - base >= 2 * STATE


def test_a_byte_limit_keeps_nothing(monkeypatch):
    room()
    monkeypatch.setenv("TFOCUS_MAX_DEVICE_BYTES", str(1 << 34))
    with tf.Solver(grid(), "f32"):
        base = torch.cuda.mem_get_info()[0]
    assert torch.cuda.mem_get_info()[0] - base >= 2 * STATE
