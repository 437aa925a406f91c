"""The FP64 kernels whose currents are shared between helicities (GPU).

Sizes at the edges of the event-to-wave mapping (one event, fewer events
than XCDs, a page and a page plus one; g g -> t t~ g above the size up to
which it spreads helicities over lanes), incoming momenta on the axis and
after a rotation and a boost, every helicity by itself, massless quarks
(half of the helicities exactly zero and filtered out), and the zero-width
flag, against the oracle on the oracle's momenta.

Tolerance: two correct FP64 evaluations of the same momenta differ by the
rounding of the propagator invariants, O(eps kappa) with kappa = s / min
|2 p_i.p_j| (rounding.invariant_condition), and of the sums over diagrams:
1e-12 + 8 eps kappa relative to the helicity sum of the event, for each
helicity as for the sum.

The gradient: sizes at the edges of its events per wave and block, every
optional output left out, the uniforms overwritten by their gradient, slots
past the last event untouched, massless quarks and the weight flag.
Tolerance as in test_gpu_adjoint: normwise 1e-10 + 64 eps gamma^2 against the
oracle's autograd gradient.
"""
import ctypes

import pytest
import torch

from oracle import me as orc
from oracle.params import DEFAULT, TCHANNEL_ZERO_WIDTH, WEIGHT_2PI
from rounding import EPS, boost_gamma, invariant_condition

pytestmark = pytest.mark.gpu

PROCS = ('eemumu', 'ggtt', 'ggttg', 'ggttgg')
SIZES = (1, 7, 64, 65, 129)


@pytest.fixture(scope='module')
def mg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12631_amd as m
    m.lib()
    return m


def bound(p):
    return 1e-12 + 8 * EPS * invariant_condition(p)


def moved(p):
    """Rotated about x and boosted along y: no momentum component vanishes."""
    c, s, ch, sh = 0.8, 0.6, 1.25, 0.75
    E, x, y, z = p.unbind(-1)
    y, z = c * y - s * z, s * y + c * z
    return torch.stack([ch * E + sh * y, x, sh * E + ch * y, z], -1)


def compare(eng, proc, p, prm):
    n = p.shape[0]
    print('[gpu-test] shared', proc, n, prm, flush=True)
    hel = orc.me_per_helicity(proc, p, prm)
    total = hel.sum(0)
    mom = eng.events_mom(p)
    me, evtw = eng.sigmakin(mom, n, wgt=torch.full((n,), 2.0, dtype=torch.float64, device='cuda'))
    assert ((me.cpu() * eng.layout.iden - total).abs() <= bound(p) * total).all()
    assert torch.equal(evtw, 2.0 * me)
    got = eng.sigmakin_hel(mom, n).cpu()
    assert ((got - hel).abs() <= bound(p) * total).all()
    return got


@pytest.mark.parametrize('proc,n', [(p, n) for p in PROCS for n in SIZES]
                         + [('ggtt', 8257), ('ggttg', 2113)])
def test_sizes_and_frames(mg, proc, n):
    eng = mg.MEEngine(proc, 'fp64')
    _, p, _ = orc.sample(proc, 21, 0, n)
    compare(eng, proc, p, DEFAULT)
    # the widths break Lorentz invariance of single helicities only through
    # the helicity axes: each frame is compared with the oracle in that frame
    compare(eng, proc, moved(p), DEFAULT)


@pytest.mark.parametrize('proc', PROCS[1:])
def test_massless_quarks_and_zero_width(mg, proc):
    n = 65
    prm = DEFAULT.with_(mt=0.0, wt=0.0)
    eng = mg.MEEngine(proc, 'fp64', params=dict(mt=0.0, wt=0.0))
    assert eng.layout.nhel_good == eng.layout.nhel // 2
    _, p, _ = orc.sample(proc, 22, 0, n, prm)
    got = compare(eng, proc, p, prm)
    assert int((got != 0).any(1).sum()) == eng.layout.nhel // 2
    prm = DEFAULT.with_(flags=TCHANNEL_ZERO_WIDTH)
    _, p, _ = orc.sample(proc, 23, 0, n, prm)
    compare(mg.MEEngine(proc, 'fp64', params=dict(flags=TCHANNEL_ZERO_WIDTH)), proc, p, prm)


def grad_tolerance(r):
    return 1e-10 + 64 * EPS * boost_gamma(r) ** 2


def normwise(a, b):
    return (a - b).norm(dim=1) / b.norm(dim=1)


@pytest.mark.parametrize('proc', ['ggtt', 'ggttg'])
@pytest.mark.parametrize('n', [1, 3, 4, 5, 17, 63, 65, 257])
def test_gradient_sizes_and_outputs(mg, proc, n):
    print('[gpu-test] shared gradient', proc, n, flush=True)
    eng = mg.MEEngine(proc, 'fp64')
    r, _, _ = orc.sample(proc, 31, 0, n)
    f_orc, g_orc, w_orc = orc.event_weight_and_grad(proc, r)
    rnd = eng.events_rnd(r)
    grad, glogw, f = eng.adjoint(rnd, n)
    assert (normwise(eng.rnd_events(grad, n).cpu(), g_orc) <= grad_tolerance(r)).all()
    assert ((eng.rnd_events(glogw, n).cpu() - w_orc).norm(dim=1)
            <= grad_tolerance(r) * w_orc.norm(dim=1).clamp_min(1.0)).all()
    only, none_w, none_f = eng.adjoint(rnd, n, want_logw=False, want_f=False)
    assert none_w is None and none_f is None
    assert torch.equal(eng.rnd_events(only, n), eng.rnd_events(grad, n))
    # slots past nevt are not written; the gradient may replace the uniforms
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    for out in (torch.full_like(rnd, -7.0), rnd.clone()):
        src = rnd if out[0] == -7.0 else out
        before = out.clone()
        assert mg.lib().mg_adjoint(eng._h, ptr(src), n, None, ptr(out), None, None, stream) == 0
        torch.cuda.synchronize()
        assert (normwise(eng.rnd_events(out, n).cpu(), g_orc) <= grad_tolerance(r)).all()
        lay = eng.layout
        rest = [t.view(-1, lay.nrnd, lay.neppR).permute(0, 2, 1).reshape(-1, lay.nrnd)[n:]
                for t in (out, before)]
        assert torch.equal(*rest)


@pytest.mark.parametrize('proc', ['ggtt', 'ggttg'])
@pytest.mark.parametrize('prm', [dict(mt=0.0, wt=0.0), dict(flags=TCHANNEL_ZERO_WIDTH | WEIGHT_2PI),
                                 dict(sqrts=400.0)])
def test_gradient_parameters(mg, proc, prm):
    print('[gpu-test] shared gradient', proc, prm, flush=True)
    n = 70
    eng = mg.MEEngine(proc, 'fp64', params=prm)
    r, p, _ = orc.sample(proc, 32, 0, n, DEFAULT.with_(**prm))
    _, g_orc, _ = orc.event_weight_and_grad(proc, r, DEFAULT.with_(**prm))
    grad, _, _ = eng.adjoint(eng.events_rnd(r), n)
    # massless quarks: collinear pairs amplify rounding by kappa, twice in a derivative
    tol = grad_tolerance(r) + (8 * EPS * invariant_condition(p) if prm.get('mt') == 0.0 else 0.0)
    assert (normwise(eng.rnd_events(grad, n).cpu(), g_orc) <= tol).all()
