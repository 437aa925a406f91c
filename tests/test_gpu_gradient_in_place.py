"""mg_adjoint out of place (three kernels, currents shared between helicities)
against in place (one kernel, one helicity after the other) on large samples
(GPU).

Both run RAMBO on the same uniforms and have to reach the same momenta, bit
for bit: events with kappa ~ 1e7 would turn a difference in the last bits into
1e-10 to 1e-9 of the norm of f (the seeds here hold such events).  What remains
is the rounding of the amplitudes on equal momenta, 4e-13 normwise in the
forward kernels of g g -> t t~ g and less for g g -> t t~: 1e-12 for f.  The
derivative adds a factor of the order of the boost's gamma of the events that
dominate the norm, a few tens at most: 2e-11 for the gradient.
"""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('proc', ['ggtt', 'ggttg'])
@pytest.mark.parametrize('sqrts', [1500.0, 1000.0, 400.0])
def test_f_and_gradient_in_place(proc, sqrts):
    import paper_2106_12631_amd as mg
    n = 1 << 18
    e = mg.MEEngine(proc, 'fp64', params=dict(sqrts=sqrts))
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for seed in (3, 5, 6):
        rnd = e.rng(seed, n)
        grad, _, f = e.adjoint(rnd, n, want_logw=False)
        same, f_same = rnd.clone(), torch.empty_like(f)
        assert mg.lib().mg_adjoint(e._h, ptr(same), n, None, ptr(same), None, ptr(f_same),
                                   stream) == 0
        df = float((f - f_same).norm() / f_same.norm())
        dg = float((grad - same).norm() / same.norm())
        print('[gpu-test] gradient in place', proc, sqrts, seed, 'f', df, 'gradient', dg, flush=True)
        assert df <= 1e-12
        assert dg <= 2e-11
