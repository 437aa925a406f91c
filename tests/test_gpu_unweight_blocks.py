"""Unweighting at the edges of its block sizes (GPU): one group of 256 events
per block, four, and sixteen, with the last block holding one event, one whole
group, one group and one event, and all but one; few, half and all events kept.
Exact against the oracle's Philox hit-or-miss."""
import numpy as np
import pytest
import torch

from oracle import integrate as oi

pytestmark = pytest.mark.gpu

SIZES = [(1 << 20) + d for d in (0, 1, 256, 257, 1023)] + [(1 << 22) + d for d in
                                                           (0, 1, 256, 257, 4095)]


@pytest.mark.parametrize('n', SIZES)
def test_unweight_blocks(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2106_12631_amd as mg
    rng = np.random.default_rng(n)
    f = rng.random(n)
    f[n // 3] = np.nan
    f[-1] = 2.0
    d = torch.from_numpy(f).cuda()
    for fmax in (300.0, 1.0, 0.0):
        print('[gpu-test] unweight', n, fmax, flush=True)
        idx = mg.unweight(d, fmax, 17, 3).cpu().numpy()
        assert np.array_equal(idx, oi.unweight(f, fmax, 17, 3))
