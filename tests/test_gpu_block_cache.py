"""Device blocks kept from destroyed solvers and batches: a reused block must
not show in the results (zero start, same bits), and several threads may
create and destroy objects."""
import threading

import numpy as np
import pytest

from paper_2010_00409_amd import tfocus as tf
from synthetic import configs

pytestmark = pytest.mark.gpu

N, D = 128, 1.0 / 8          # 50 MB of state in float32: above the smallest kept block


def focal_state(n, p):
    g = tf.tf_layer_grid(p, (n, N, N), (D, D, D))
    with tf.Solver(g, "f32") as s:
        zero = np.empty(s.shape, dtype=np.float32)
        s.get_fields(zero)
        s.set_pulse(p)
        s.advance(2, 0.5 * p["R0"])
        out = np.empty(s.shape, dtype=np.float32)
        s.get_fields(out)
    assert not zero.any()
    return out


def test_reused_blocks_start_at_zero_and_keep_the_bits():
    p = configs.pulse(envelope="spectral", R0=6.0, L=4.0, f_number=0.8, bandwidth=0.4)
    first = focal_state(128, p)
    focal_state(112, p)                       # a smaller object in the kept blocks
    assert np.array_equal(focal_state(128, p), first)


def test_threads_create_and_destroy_while_others_compute():
    p = configs.pulse(envelope="cos2", R0=6.0, L=2.0, f_number=0.8)
    want = focal_state(128, p)
    bad = []

    def work():
        for _ in range(3):
            if not np.array_equal(focal_state(128, p), want):
                bad.append(1)

    ts = [threading.Thread(target=work) for _ in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
