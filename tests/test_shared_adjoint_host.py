"""Reverse-mode routines of the shared-current gradient on the CPU.

tests/host/shared_adj.cpp compiles shared_currents.h and shared_adjoint.h for
the host (clang's HIP mode, tests/host/hip_kernels/hip/hip_runtime.h stands in
for the HIP header) and checks every adjoint routine against fourth-order
central differences of the forward routine it reverses, relative to the size
of the derivatives: h^4 and eps / h leave 1e-9 or less of it.

Along -z and at rest the forward pass takes constant helicity states, so the
adjoint keeps only the roots sqrt(E + P) and sqrt(E - P), which move with E and
with P along the momentum.
"""
import math
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CLANG = '/opt/rocm/llvm/bin/clang++'


def host_report(source, tmp, *defines):
    """The lines that the host build of tests/host/<source> prints."""
    cxx = CLANG if os.path.exists(CLANG) else shutil.which('amdclang++')
    if cxx is None:
        pytest.skip('no HIP host compiler')
    exe = str(tmp / source.replace('.cpp', ''))
    subprocess.check_call([cxx, '-x', 'hip', '--offload-host-only', '-nogpuinc', '-nogpulib',
                           '-std=c++17', '-O1', *defines, '-I', os.path.join(HERE, 'host', 'hip_kernels'),
                           '-I', os.path.join(ROOT, 'paper_2106_12631_amd', 'csrc'),
                           os.path.join(HERE, 'host', source), '-o', exe])
    return subprocess.check_output([exe], text=True).splitlines()


@pytest.fixture(scope='module')
def report(tmp_path_factory):
    return host_report('shared_adj.cpp', tmp_path_factory.mktemp('shared_adj'))


@pytest.mark.parametrize('name', ['QuarkAdjoint(t)', 'QuarkAdjoint(t~)', 'adj_polarisation',
                                  'adj_propagate', 'adj_three_gluon_y', 'adj_slash', 'adj_sdot'])
def test_adjoint_vs_differences(report, name):
    n, worst = next(line.split()[1:] for line in report if line.startswith(name + ' '))
    assert int(n) == 200
    assert float(worst) <= 1e-9


@pytest.mark.parametrize('case', [0, 1, 2], ids=['along -z', 'at rest', 'massless along -z'])
def test_quark_adjoint_at_constant_states(report, case):
    line = next(line for line in report if line.startswith(f'limit {case} '))
    e, x, y, z, want_e, want_z = (float(v) for v in line.split()[2:])
    assert all(math.isfinite(v) for v in (e, x, y, z))
    assert x == 0.0 and y == 0.0
    assert abs(e - want_e) <= 1e-15 and abs(z - want_z) <= 1e-15
