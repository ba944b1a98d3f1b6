"""The surrogate's kernels take several lines, columns and row tiles per wave,
how many depending on the batch.  A sample's arithmetic does not: transforms
and inference of a batch must equal those of its samples taken one by one, bit
for bit (the single samples are held to the oracle elsewhere)."""
import numpy as np
import pytest
import torch

from paper_2010_00409_amd import tfocus as tf

pytestmark = pytest.mark.gpu

WIDTH = 32


def randn(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda")


def zeros(*shape):
    return torch.zeros(shape, dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("batch", [3, 4, 7, 17])
def test_transforms_of_a_batch_equal_those_of_its_samples(batch):
    v, x = randn((batch, 64, 64, 64, WIDTH), 1), randn((batch, 24, 2, 24, 12, WIDTH), 2)
    m, u = zeros(batch, 24, 2, 24, 12, WIDTH), zeros(batch, 64, 64, 64, WIDTH)
    m1, u1 = zeros(1, 24, 2, 24, 12, WIDTH), zeros(1, 64, 64, 64, WIDTH)
    with tf.Surrogate(batch, period=80) as s:
        s.spectral_forward(v, m)
        s.spectral_inverse(x, u)
        for b in range(batch):
            s.spectral_forward(v[b:b + 1], m1)
            s.spectral_inverse(x[b:b + 1], u1)
            assert torch.equal(m1[0], m[b]) and torch.equal(u1[0], u[b]), b


@pytest.mark.parametrize("nbasis, batch, training", [(1, 2, False), (4, 5, False), (4, 18, False), (1, 5, True)])
def test_forward_of_a_batch_equals_that_of_its_samples(nbasis, batch, training):
    rng = np.random.default_rng(batch)
    p = torch.from_numpy(rng.uniform(size=(batch, 8)).astype(np.float32)).cuda()
    w = None if nbasis == 1 else randn((batch, nbasis), 3)
    out, one = zeros(batch, 6, 64, 64, 64), zeros(1, 6, 64, 64, 64)
    with tf.Surrogate(batch, training=training, nbasis=nbasis) as s:
        s.set_params(torch.randn(s.nparams, generator=torch.Generator().manual_seed(4)) * 0.1)
        s.forward(p, out, w)
        for b in range(batch):
            s.forward(p[b:b + 1].contiguous(), one, None if w is None else w[b:b + 1].contiguous())
            assert torch.equal(one[0], out[b]), b
        assert float(out.abs().max()) > 0.0
