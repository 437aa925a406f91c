"""The stream handle of the binding: torch's raw-handle call where this torch
has it, the public one otherwise (CPU), and the same handle from both (GPU)."""
from types import SimpleNamespace

import pytest
import torch

import paper_2106_12631_amd as mg


def test_without_the_raw_call(monkeypatch):
    monkeypatch.setattr(mg, '_raw_stream', None)
    monkeypatch.setattr(torch.cuda, 'current_stream',
                        lambda device: SimpleNamespace(cuda_stream=1000 + device.index))
    assert mg._stream(torch.device('cuda', 3)) == 1003


def test_with_the_raw_call(monkeypatch):
    monkeypatch.setattr(mg, '_raw_stream', lambda index: 2000 + index)
    assert mg._stream(torch.device('cuda', 3)) == 2003


@pytest.mark.gpu
def test_both_give_the_current_stream(monkeypatch):
    dev = torch.device('cuda', torch.cuda.current_device())
    side = torch.cuda.Stream()
    for s in (torch.cuda.default_stream(), side):
        with torch.cuda.stream(s):
            handles = {mg._stream(dev)}
            with monkeypatch.context() as m:
                m.setattr(mg, '_raw_stream', None)
                handles.add(mg._stream(dev))
            assert handles == {s.cuda_stream}
