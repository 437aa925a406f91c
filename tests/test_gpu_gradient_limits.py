"""The FP64 gradient where the helicity states have no derivative (GPU): both
tops of g g -> t t~ along the beam, reached with cos(theta) = -1 and 1.  There
the states are constants (helicity_states), and the gradient stays finite as it
does in place, where the adjoint differentiates the same constants; f is the
one of the regular branch."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('mt', [173.0, 4.7])
def test_tops_along_the_beam(mt):
    import paper_2106_12631_amd as mg
    e = mg.MEEngine('ggtt', 'fp64', params=dict(mt=mt))
    r = torch.full((2, 8), 0.37, dtype=torch.float64)
    r[0, 0], r[0, 4] = 0.0, 1.0   # t along -z
    r[1, 0], r[1, 4] = 1.0, 0.0   # t~ along -z
    rnd = e.events_rnd(r)
    print('[gpu-test] tops along the beam', mt, flush=True)
    grad, glogw, f = e.adjoint(rnd, 2)
    assert torch.isfinite(e.rnd_events(grad, 2)).all()
    assert torch.isfinite(e.rnd_events(glogw, 2)).all()
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    same, f_same = rnd.clone(), torch.empty_like(f)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert mg.lib().mg_adjoint(e._h, ptr(same), 2, None, ptr(same), None, ptr(f_same), stream) == 0
    assert torch.isfinite(e.rnd_events(same, 2)).all()
    assert ((f - f_same).abs() <= 1e-12 * f_same).all()


@pytest.mark.parametrize('sqrts', [1500.0, 347.0])
def test_two_body_weight_is_constant(sqrts):
    """The weight of two equal masses does not depend on the uniforms: its
    gradient is zero, with no rounding left over however soft the uniforms."""
    import paper_2106_12631_amd as mg
    e = mg.MEEngine('ggtt', 'fp64', params=dict(sqrts=sqrts))
    n = (1 << 18) + 1
    for seed in (3, 4):
        print('[gpu-test] two-body weight', sqrts, seed, flush=True)
        _, glogw, _ = e.adjoint(e.rng(seed, n), n)
        assert (e.rnd_events(glogw, n) == 0.0).all()


@pytest.mark.parametrize('proc', ['ggtt', 'ggttg'])
def test_massless_weight_is_constant(proc):
    """The weight of massless particles is a constant too, also at uniforms that
    make all of them collinear, where the momenta themselves are not defined."""
    import paper_2106_12631_amd as mg
    e = mg.MEEngine(proc, 'fp64', params=dict(mt=0.0, wt=0.0))
    nr = e.layout.nrnd
    r = torch.rand(70, nr, generator=torch.Generator().manual_seed(1), dtype=torch.float64)
    r[::7] = 0.5
    print('[gpu-test] massless weight', proc, flush=True)
    grad, glogw, f = e.adjoint(e.events_rnd(r), 70)
    assert (e.rnd_events(glogw, 70) == 0.0).all()
    assert torch.isfinite(f.cpu()[1:7]).all() and torch.isnan(f.cpu()[::7]).all()
