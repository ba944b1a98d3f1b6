"""tf_advance_noalloc on a caller's state that is aligned to its elements only,
over x lengths of every kind of block: the bits of the same run on an aligned
state, and nothing written outside it."""
import pytest
import torch

from paper_2010_00409_amd import tfocus as tf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx", [8, 24, 40, 56, 64, 96, 128, 224, 256, 320, 512, 640, 768, 896, 1024])
def test_shifted_state_takes_the_same_steps(nx, prec):
    dtype = torch.float64 if prec == "f64" else torch.float32
    shape = (6, 16, 8, nx)
    g = dict(nx=nx, ny=8, nz=16, dx=0.31, dy=0.27, dz=0.23, x_min=0.0, y_min=0.0, z_min=0.0)
    gen = torch.Generator(device="cuda").manual_seed(nx)
    ref = torch.randn(shape, dtype=dtype, device="cuda", generator=gen)
    n = ref.numel()
    st = torch.cuda.current_stream()
    outs = []
    for shift in range(16 // ref.element_size()):
        buf = torch.full((n + 8,), 7.0, dtype=dtype, device="cuda")
        state = buf[shift:shift + n].view(shape)
        assert state.data_ptr() % 16 == shift * ref.element_size() % 16
        state.copy_(ref)
        tf.tf_advance_noalloc(g, prec, state, 3, 0.43, project_b_first=True, stream=st)
        torch.cuda.synchronize()
        assert bool((buf[:shift] == 7.0).all()) and bool((buf[shift + n:] == 7.0).all())
        outs.append(state.clone())
    assert not torch.equal(outs[0], ref)
    for o in outs[1:]:
        assert torch.equal(o, outs[0])
