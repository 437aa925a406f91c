"""The generated FP64 amplitude code of g g -> t t~ g g on the CPU.

The library's FP64 kernels of this process share the currents between
helicities, so that only a build with -DMG_EVENT_PER_LANE_F64 runs this code.
Here it is compiled for the host and compared with the oracle, each helicity,
for beams on the axis (both bodies) and after a boost.

Tolerance: 1e-12 + 8 eps kappa of the event's helicity sum, the rounding of the
propagator invariants and of the sums over diagrams (test_gpu_shared).
"""
import math
import os
import shutil
import subprocess

import pytest
import torch

from oracle import me as orc
from oracle.params import DEFAULT
from rounding import EPS, invariant_condition

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), 'paper_2106_12631_amd', 'csrc')
CLANG = '/opt/rocm/llvm/bin/clang++'


@pytest.fixture(scope='module')
def amplitudes(tmp_path_factory):
    cxx = CLANG if os.path.exists(CLANG) else shutil.which('amdclang++')
    if cxx is None or not os.path.exists(os.path.join(CSRC, 'generated', 'ggttgg.inc')):
        pytest.skip('no HIP host compiler or generated code not written')
    exe = str(tmp_path_factory.mktemp('amplitudes') / 'amplitudes')
    subprocess.check_call([cxx, '-x', 'hip', '--offload-host-only', '-nogpuinc', '-nogpulib',
                           '-std=c++17', '-O0', '-w', '-I', os.path.join(HERE, 'host', 'hip_kernels'),
                           '-I', CSRC, os.path.join(HERE, 'host', 'amplitudes.cpp'), '-o', exe])

    def run(p):
        head = [math.sqrt(4 * math.pi * DEFAULT.alphas), DEFAULT.mt, DEFAULT.wt]
        text = ' '.join(repr(float(x)) for x in head + p.reshape(-1).tolist())
        out = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout
        return torch.tensor([[float(x) for x in line.split()] for line in out.splitlines()],
                            dtype=torch.float64)
    return run


@pytest.mark.parametrize('frame', ['beams on the axis', 'boosted'])
def test_every_helicity_vs_oracle(amplitudes, frame):
    _, p, _ = orc.sample('ggttgg', 24, 0, 5)
    if frame == 'boosted':
        E, x, y, z = p.unbind(-1)
        p = torch.stack([1.25 * E + 0.75 * x, 0.75 * E + 1.25 * x, y, z], -1)
    hel = orc.me_per_helicity('ggttgg', p).T
    got = amplitudes(p)
    assert got.shape == (5, 64 if frame == 'boosted' else 128)
    tol = ((1e-12 + 8 * EPS * invariant_condition(p)) * hel.sum(1))[:, None]
    for body in got.split(64, 1):
        assert ((body - hel).abs() <= tol).all()
