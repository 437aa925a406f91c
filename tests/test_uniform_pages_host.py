"""MEEngine.events_rnd on CPU tensors: every shape that assigns to an
(events, uniforms) array, at whole and ragged pages, small and large."""
from types import SimpleNamespace

import pytest
import torch

import paper_2106_12631_amd as mg

PAGE = 64


def engine(nrnd):
    lay = SimpleNamespace(nrnd=nrnd, neppR=PAGE)
    return SimpleNamespace(layout=lay, device=torch.device('cpu'),
                           _pages=lambda n, k: (n + k - 1) // k)


def expected(r, nrnd):
    n = r.shape[0]
    npg = (n + PAGE - 1) // PAGE
    buf = torch.full((npg * PAGE, nrnd), 0.5, dtype=torch.float64)
    buf[:n] = r
    return buf.view(npg, PAGE, nrnd).permute(0, 2, 1).reshape(-1)


SHAPES = [(0, 16), (1, 16), (63, 16), (64, 16), (65, 16), (128, 16), (1000, 16),
          (16,),               # the same uniforms for each of 16 events
          (1,), (1, 1, 16), (65, 1), (128, 1),
          (131071, 16), (131072, 16), (131073, 16), (262145, 8)]


@pytest.mark.parametrize('shape', SHAPES, ids=str)
@pytest.mark.parametrize('dtype', [torch.float64, torch.float32])
def test_shapes(shape, dtype):
    nrnd = shape[-1] if shape[-1] > 1 else 16
    r = torch.rand(shape, generator=torch.Generator().manual_seed(3)).to(dtype)
    assert torch.equal(mg.MEEngine.events_rnd(engine(nrnd), r), expected(r, nrnd))
    if r.dim() == 2:
        strided = r.t().contiguous().t()
        assert torch.equal(mg.MEEngine.events_rnd(engine(nrnd), strided), expected(r, nrnd))


@pytest.mark.parametrize('shape', [(64,), (65,), (65, 15), (64, 17), (64, 1, 16), (65, 1, 16), (2, 65, 16)],
                         ids=str)
def test_refused(shape):
    with pytest.raises((RuntimeError, IndexError)):
        mg.MEEngine.events_rnd(engine(16), torch.rand(shape))
