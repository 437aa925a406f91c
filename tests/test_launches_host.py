"""How the library cuts its launches, on the CPU.

A grid holds fewer than 2^32 work-items, so a kernel with several lanes per
event takes a large basket in several launches.  tests/host/launch_record.cpp
stands in for the HIP runtime and records the launches of baskets on both sides
of the cuts: every grid has to stay below the limit, and the launches of a call
have to cover its events once, in order, each from the event where the one
before ended.
"""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIBPATH = os.path.join(ROOT, 'paper_2106_12631_amd', 'libmg5mi.so')
NPAR = {'eemumu': 4, 'ggtt': 4, 'ggttg': 5, 'ggttgg': 6}
PROC = {p: k for k, p in enumerate(NPAR)}
PREC = {'fp64': 0, 'fp32amp': 1, 'mixed': 2, 'mixed_f32mfma': 3}

CHILD = r'''
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
rec.record_kernel.restype = ctypes.c_char_p
rec.record_arg.restype = ctypes.c_uint64
rec.record_grid.restype = rec.record_block.restype = ctypes.c_uint32
vp, i64 = ctypes.c_void_p, ctypes.c_int64
out = []
for call, proc, prec, n in json.loads(sys.argv[3]):
    h = vp()
    assert L.mg_create(proc, prec, None, ctypes.byref(h)) == 0
    rec.record_clear()
    a = [vp(k << 50) for k in range(6)]   # made-up device addresses
    if call == 'sigmakin':
        rc = L.mg_sigmakin(h, a[1], i64(n), a[2], None, None, None)
    elif call == 'hel':
        rc = L.mg_sigmakin_hel(h, a[1], i64(n), a[3], None)
    else:
        rc = L.mg_adjoint(h, a[4], i64(n), None, a[5], None, None, None)
    assert rc == 0
    out.append([[rec.record_kernel(k).decode(), rec.record_grid(k), rec.record_block(k),
                 [rec.record_arg(k, j) for j in range(3)]] for k in range(rec.record_count())])
print(json.dumps(out))
'''


@pytest.fixture(scope='module')
def record(tmp_path_factory):
    cxx = shutil.which('g++')
    if cxx is None or not os.path.exists(LIBPATH):
        pytest.skip('no host C++ compiler or library not built')
    so = str(tmp_path_factory.mktemp('launch') / 'launch_record.so')
    subprocess.check_call([cxx, '-std=c++17', '-O1', '-shared', '-fPIC',
                           os.path.join(HERE, 'host', 'launch_record.cpp'), '-o', so])

    def run(calls):
        r = subprocess.run([sys.executable, '-c', CHILD, so, LIBPATH, json.dumps(calls)],
                           stdout=subprocess.PIPE, text=True, check=True)
        return json.loads(r.stdout)
    return run


def cuts(lanes):
    n = (1 << 31) // lanes
    return [1, n - 1, n, n + 1, 2 * n, 3 * n + 77]


# call, process, precision, name of the kernel, lanes per event, events per block
KERNELS = [
    ('sigmakin', 'ggttgg', 'fp64', 'sigmakin_ggttgg_shared_kernel', 64, 1),
    ('hel', 'ggttgg', 'fp64', 'sigmakin_ggttgg_shared_kernel', 64, 1),
    ('sigmakin', 'ggttg', 'fp64', 'sigmakin_gluon_lanes_kernel', 8, 8),
    ('hel', 'ggttg', 'fp64', 'sigmakin_gluon_lanes_kernel', 8, 8),
    ('sigmakin', 'ggttgg', 'fp32amp', 'sigmakin_hpl_kernel', 64, 1),
    ('hel', 'ggttgg', 'fp32amp', 'sigmakin_hpl_kernel', 64, 1),
    ('sigmakin', 'ggttgg', 'mixed', 'sigmakin_mixed_hpl_kernel', 64, 1),
    ('sigmakin', 'ggttgg', 'mixed_f32mfma', 'sigmakin_mixed_hpl_kernel', 64, 1),
    ('adjoint', 'ggtt', 'fp64', 'momentum_gradient_kernel', 4, 16),
    ('adjoint', 'ggttg', 'fp64', 'momentum_gradient_kernel', 16, 4),
]


@pytest.mark.parametrize('call,proc,prec,kernel,lanes,per_block', KERNELS)
def test_launches_cover_the_events(record, call, proc, prec, kernel, lanes, per_block):
    sizes = cuts(lanes)
    for n, launches in zip(sizes, record([[call, PROC[proc], PREC[prec], n] for n in sizes])):
        for name, grid, block, _ in launches:
            assert 0 < grid * block < 1 << 32, (n, name, grid, block)
        mine = [x for x in launches if kernel in x[0]]
        if n == 1 and not mine:   # a smaller launch's kernel
            continue
        done = 0
        for name, grid, block, (buf, first, _) in mine:
            assert block == 64
            if 'mixed' in name:   # (momenta from the launch's first event on, its events, ...)
                assert first == grid * per_block or first == n - done
                page, rest = divmod(buf - mine[0][3][0], 64 * NPAR[proc] * 4 * 8)
                assert rest == 0
                first = 64 * page
            else:                 # (buffer, first event, ...)
                assert buf == mine[0][3][0]
            assert first == done
            done += grid * per_block
        assert n <= done < n + per_block, (n, done)


@pytest.mark.parametrize('proc', list(NPAR))
@pytest.mark.parametrize('prec', list(PREC))
def test_every_launch_fits_a_grid(record, proc, prec):
    """The largest baskets whose momenta fit 288 GB, in every entry point."""
    n = (288 << 30) // (32 * NPAR[proc]) // 64 * 64 + 5
    calls = ['sigmakin', 'hel'] + ([] if proc == 'ggttgg' else ['adjoint'])
    for launches in record([[c, PROC[proc], PREC[prec], n] for c in calls]):
        assert launches
        for name, grid, block, _ in launches:
            assert 0 < grid * block < 1 << 32, (name, grid, block)
