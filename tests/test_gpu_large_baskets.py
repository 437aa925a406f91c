"""Baskets that a kernel with several lanes per event takes in two launches
(GPU): events on both sides of the cut, the last ones and the first, against
the same events in a basket of their own.  Such a basket starts at a page of
the momenta, so the same kernel sees the same events, and the results agree bit
for bit.  The sizes are the real ones, 2^25 events with 64 lanes, 2^27 to 2^29
with 16, 8 and 4."""
import pytest
import torch

pytestmark = pytest.mark.gpu

F64 = torch.float64
PAGE = 64


FILL = 4096   # events ahead of the ones compared: enough for the large launches' kernel


@pytest.fixture(autouse=True)
def memory():
    yield
    torch.cuda.empty_cache()


def parts(n, cut):
    """(first, last + 1) of the ranges of events looked at."""
    return [(0, 300), (cut - 2 * PAGE, cut + PAGE), (cut, n), ((n - 5 * PAGE) // PAGE * PAGE, n)]


def own_pages(buf, row, lo, hi):
    """Pages of the FILL first events and then of lo .. hi-1."""
    return torch.cat([buf[:FILL * row], buf[lo * row:(hi + PAGE - 1) // PAGE * PAGE * row]])


@pytest.mark.parametrize('proc,prec,log2', [('ggttgg', 'fp64', 25), ('ggttgg', 'mixed', 25),
                                            ('ggttgg', 'fp32amp', 25), ('ggttg', 'fp64', 28)])
def test_matrix_elements(proc, prec, log2):
    import paper_2106_12631_amd as mg
    e = mg.MEEngine(proc, prec)
    n = (1 << log2) + 3 * PAGE + 37
    print('[gpu-test] large basket', proc, prec, n, flush=True)
    _, mom, wgt = e.sample(11, n)
    me, evtw = e.sigmakin(mom, n, wgt=wgt)
    row = 4 * e.layout.npar
    for lo, hi in parts(n, 1 << log2):
        w = torch.cat([wgt[:FILL], wgt[lo:hi]])
        me1, evtw1 = e.sigmakin(own_pages(mom, row, lo, hi), FILL + hi - lo, wgt=w)
        assert torch.equal(me[lo:hi], me1[FILL:]) and torch.equal(evtw[lo:hi], evtw1[FILL:])
    if log2 == 25:   # each helicity by itself: 64 values an event
        hel = e.sigmakin_hel(mom, n)
        for lo, hi in parts(n, 1 << log2):
            hel1 = e.sigmakin_hel(own_pages(mom, row, lo, hi), FILL + hi - lo)
            assert torch.equal(hel[:, lo:hi], hel1[:, FILL:])


@pytest.mark.parametrize('proc,log2', [('ggttg', 27), ('ggtt', 29)])
def test_gradient(proc, log2):
    import paper_2106_12631_amd as mg
    e = mg.MEEngine(proc, 'fp64')
    n = (1 << log2) + 3 * PAGE + 37
    print('[gpu-test] large gradient', proc, n, flush=True)
    rnd = e.rng(12, n)
    grad, _, f = e.adjoint(rnd, n, want_logw=False)
    row = e.layout.nrnd
    for lo, hi in parts(n, 1 << log2):
        m = FILL + hi - lo
        grad1, _, f1 = e.adjoint(own_pages(rnd, row, lo, hi), m, want_logw=False)
        assert torch.equal(f[lo:hi], f1[FILL:])
        got = grad[lo * row:(hi + PAGE - 1) // PAGE * PAGE * row]
        assert torch.equal(e.rnd_events(got, hi - lo), e.rnd_events(grad1, m)[FILL:])
