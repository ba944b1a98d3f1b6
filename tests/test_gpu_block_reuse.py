"""Which device blocks are kept from destroyed solvers and batches: reuse by
address, across streams and between a solver and a batch, their return, and
graph captures of other threads while objects go."""
import threading

import numpy as np
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


def test_blocks_pass_between_streams_and_between_solvers_and_batches():
    """Work still queued on one stream when its solver goes must not reach into
    the next object, which runs on another stream."""
    room()
    p = configs.pulse(**P)
    win = dict(wx=32, wy=32, wz=32, cx=0.0, cy=0.0, cz=0.0)

    def solver():
        st = torch.cuda.Stream()
        out = np.empty((6, 32, 32, 32), dtype=np.float32)
        with tf.Solver(grid(), "f32", st) as s:
            s.set_pulse(p)
            s.advance(2, 0.5 * P["R0"])
            s.read_focal(win, out)
            s.advance(20, 0.1)                                       # still running when the solver goes
        return out

    def batch():
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            dst = torch.empty((1, 6, 32, 32, 32), dtype=torch.float32, device="cuda")
        with tf.Batch([grid()], [p], "f32", st) as b:
            b.run([2], [0.5 * P["R0"]], win, dst)
            with torch.cuda.stream(st):
                out = dst[0].cpu().numpy()
            b.run([20], [0.1], win, dst)                             # still running when the batch goes
        return out

    want, bad = solver(), []
    assert np.abs(want).max() > 0

    def work():
        for f in (solver, batch, solver, batch):
            try:
                if not np.array_equal(f(), want):
                    bad.append(f.__name__)
            except tf.TfError as e:
                bad.append(str(e))

    ts = [threading.Thread(target=work) for _ in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def test_objects_may_go_while_another_thread_captures():
    room()
    p = configs.pulse(**P)
    win = dict(wx=32, wy=32, wz=32, cx=0.0, cy=0.0, cz=0.0)
    g = tf.tf_layer_grid(p, (64, 64, 64), (D, D, D))
    done, bad, count = threading.Event(), [], [0]

    def captures():
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            dst = torch.empty((1, 6, 32, 32, 32), dtype=torch.float32, device="cuda")
        try:
            for i in range(40):
                with tf.Batch([g], [p], "f32", st) as b:
                    b.run([400 + i % 3], [0.1], win, dst)            # one capture of 1600 launches
        except tf.TfError as e:
            bad.append(str(e))
        done.set()

    def goes():
        st = torch.cuda.Stream()
        while not done.is_set():
            with tf.Solver(grid(), "f32", st):
                count[0] += 1

    ts = [threading.Thread(target=f) for f in (captures, goes)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad and count[0] > 10
