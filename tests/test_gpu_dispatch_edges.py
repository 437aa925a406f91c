"""FP64 SIGMAKIN on both sides of the sizes where its kernel changes (GPU).

g g -> t t~ spreads the helicities over lanes up to 8192 events and takes one
event per lane from 8193 on, g g -> t t~ g spreads them up to 2048 and takes
eight lanes an event from 2049 on.  Events in RAMBO's frame, rotated and boosted
along the beam share waves, so both kernels run both of their bodies.  Against
the oracle on the same momenta, with the tolerance of test_gpu_shared: 1e-12 +
8 eps kappa; the weights, which no kernel rounds otherwise, exactly."""
import pytest
import torch

from oracle import me as orc
from rounding import EPS, invariant_condition
from test_gpu_frames import transformed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('proc,n', [('ggtt', 8192), ('ggtt', 8193), ('ggttg', 2048), ('ggttg', 2049)])
def test_both_sides(proc, n):
    import paper_2106_12631_amd as mg
    print('[gpu-test] dispatch edge', proc, n, flush=True)
    _, p, _ = orc.sample(proc, 41, 0, n)
    q, _ = transformed(p, 42)
    want = orc.matrix_element(proc, q)
    e = mg.MEEngine(proc, 'fp64')
    wgt = torch.rand(n, generator=torch.Generator().manual_seed(43), dtype=torch.float64).cuda()
    mom = e.events_mom(q)
    me, evtw = e.sigmakin(mom, n, wgt=wgt)
    assert ((me.cpu() - want).abs() <= (1e-12 + 8 * EPS * invariant_condition(q)) * want).all()
    assert torch.equal(evtw, me * wgt)
    # the same events one by one in their page: no event depends on its neighbours' frames
    alone = torch.cat([e.sigmakin(e.events_mom(q[k:k + 1]), 1).cpu() for k in (0, n // 2, n - 1)])
    assert ((alone - want[[0, n // 2, n - 1]]).abs()
            <= 2 * (1e-12 + 8 * EPS * invariant_condition(q[[0, n // 2, n - 1]])) * alone).all()
