"""The init kernel's support bounds along x and its interval polynomials at
their edges, against the float64 oracle.  Tolerance: the float64 init gate of
1e-12 relative L2 (geometry and profile round at a few 1e-16; the longest
window's carrier phase, about 1300 rad, at 1300 x 1.1e-16 = 1.4e-13)."""
import numpy as np
import pytest

from oracle import pulse
from paper_2010_00409_amd import tfocus as tf
from synthetic import configs

pytestmark = pytest.mark.gpu

CASES = {
    # apertures: past 90 degrees, all directions (no bound along x), and an edge wider than the aperture
    "past_half_pi": (dict(envelope="cos2", theta=1.9, eps=0.3, R0=3.0, L=2.0), (24, 64, 64), 0.15, {}),
    "all_directions": (dict(envelope="cos2", theta=3.1, eps=0.3, R0=3.0, L=2.0), (24, 64, 64), 0.15, {}),
    "edge_wider_than_aperture": (dict(envelope="spectral", theta=0.1, eps=0.5, R0=4.0, L=3.0, bandwidth=0.5),
                                 (32, 40, 48), 0.125, {}),
    # many preimages overlap; nodes on the axis and on the support's edges
    "overlapping_preimages": (dict(envelope="spectral", f_number=0.5, R0=6.0, L=2.0, bandwidth=0.6, gdd=0.3, tod=0.2,
                                   ellipticity=0.4, pol_angle=0.3), (24, 80, 80), 0.125, {}),
    "gauss_aperture_replicated": (dict(envelope="gauss", transverse="gauss", f_number=0.6, R0=3.0, L=2.5),
                                  (24, 32, 40), 0.125, dict(replicate_yz=1)),
    # one sample, one interval; and a window too long for the table (direct sum)
    "one_frequency": (dict(envelope="spectral", f_number=0.7, R0=3.0, L=2.0, bandwidth=0.1, nfreq=1), (24, 48, 48), 0.125,
                      {}),
    "window_beyond_the_table": (dict(envelope="spectral", f_number=1.0, R0=110.0, L=200.0, bandwidth=0.3, nfreq=64),
                                (24, 16, 16), 10.0, {}),
}


@pytest.mark.parametrize("name", CASES)
def test_init_support_and_interval_polynomials_match_oracle(name):
    kw, n, d, extra = CASES[name]
    p = configs.pulse(**kw)
    g = dict(pulse.layer_grid(p, n, (d, d, d)), **extra)
    with tf.Solver(g, "f64") as s:
        s.set_pulse(p)
        got = np.empty(s.shape)
        s.get_fields(got)
        # a second, shorter pulse on the kept tables, then the first again
        s.set_pulse(configs.pulse(envelope="spectral", R0=2.0, L=1.0, nfreq=32))
        s.set_pulse(p)
        again = np.empty(s.shape)
        s.get_fields(again)
    E, B = pulse.init_fields(p, g)
    ref = np.concatenate([E, B])
    assert np.linalg.norm(ref) > 0.0
    assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)
    assert np.array_equal(got, again)
