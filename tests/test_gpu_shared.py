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
"""
import sys

import pytest
import torch

from oracle import me as orc
from oracle.params import DEFAULT, TCHANNEL_ZERO_WIDTH
from rounding import EPS, invariant_condition

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


@pytest.mark.parametrize('proc,n', [(p, n) for p in PROCS for n in SIZES] + [('ggttg', 2113)])
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
