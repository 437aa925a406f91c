"""Event-major uniforms to AoSoA pages and back (GPU): whole pages, ragged
last pages, other types, devices and strides, bit for bit, with 0.5 in the
slots past the last event."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n', [0, 1, 63, 64, 65, 128, 1000])
def test_uniform_pages(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12631_amd as mg
    e = mg.MEEngine('ggttg')
    lay = e.layout
    print('[gpu-test] pages', n, flush=True)
    for dt in (torch.float64, torch.float32):
        r = torch.rand(n, lay.nrnd, dtype=dt)
        npg = (n + lay.neppR - 1) // lay.neppR
        want = torch.full((npg * lay.neppR, lay.nrnd), 0.5, dtype=torch.float64)
        want[:n] = r
        want = want.view(npg, lay.neppR, lay.nrnd).permute(0, 2, 1).reshape(-1)
        for x in (r, r.cuda(), r.cuda().t().contiguous().t()):
            got = e.events_rnd(x)
            assert torch.equal(got.cpu(), want)
            assert torch.equal(e.rnd_events(got, n).cpu(), r.double())
