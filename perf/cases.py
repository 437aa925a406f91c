"""The work a user of this framework has it do, as timed cases.

Kinds of pass:
  iteration   one basket of events from nothing: MEEngine.sample (random
              numbers, phase space) and MEEngine.sigmakin (matrix elements and
              event weights), into buffers the program allocated once;
  me          MEEngine.sigmakin on momenta the program brings itself, here
              partonic events boosted along the beam axis to a lab frame;
  adjoint     MEEngine.adjoint: gradient of the event weight with respect to
              the uniforms, in the library's own page layout;
  weight      MEEngine.event_weight forward and backward through torch
              autograd on event-major uniforms (phase-space adaptation);
  analysis    MEEngine.cross_section and unweight on a large weighted sample.

The values of exact() come from a plain torch evaluation in 64 bits written
below: Philox uniforms, RAMBO, and the colour-decomposed recursion over gluon
subsets, with one tensor axis per helicity.
"""
import itertools
import math

import torch

import paper_2106_12631_amd as mg

NPAR = {'eemumu': 4, 'ggtt': 4, 'ggttg': 5, 'ggttgg': 6}
IDEN = {'eemumu': 4, 'ggtt': 256, 'ggttg': 256, 'ggttgg': 512}
PAGE = 64                     # events per page of the AoSoA buffers
DEV = 'cuda' if torch.cuda.is_available() else 'cpu'
F64, C128 = torch.float64, torch.complex128


def listed():
    return [
        # the benchmark's smallest basket: a few launches, latency
        dict(name='iter_eemumu_16384', kind='iteration', process='eemumu', precision='fp64',
             nevt=16384, sqrts=1500.0),
        # the throughput plateau of the lightest process
        dict(name='iter_eemumu_16M', kind='iteration', process='eemumu', precision='fp64',
             nevt=1 << 24, sqrts=1500.0),
        # an ordinary basket that ends inside a page and a block
        dict(name='iter_ggtt_1000003', kind='iteration', process='ggtt', precision='fp64',
             nevt=1000003, sqrts=1500.0),
        # the benchmark's 2 -> 3 baskets, in both precisions it is quoted in
        dict(name='iter_ggttg_1M', kind='iteration', process='ggttg', precision='fp64',
             nevt=1 << 20, sqrts=1500.0),
        dict(name='iter_ggttg_mixed_1M', kind='iteration', process='ggttg', precision='mixed',
             nevt=1 << 20, sqrts=1500.0),
        # the headline workload, in both precisions
        dict(name='iter_ggttgg_512K', kind='iteration', process='ggttgg', precision='fp64',
             nevt=1 << 19, sqrts=1500.0),
        dict(name='iter_ggttgg_mixed_512K', kind='iteration', process='ggttgg', precision='mixed',
             nevt=1 << 19, sqrts=1500.0),
        # the heaviest process on a small ragged basket (tests, interactive use)
        dict(name='iter_ggttgg_1000', kind='iteration', process='ggttgg', precision='fp64',
             nevt=1000, sqrts=1500.0),
        # reweighting: matrix elements of events in the lab frame
        dict(name='me_ggttgg_lab_65537', kind='me', process='ggttgg', precision='fp64',
             nevt=65537, sqrts=1000.0),
        # the benchmark's gradient workload (with the pT cut that makes it finite)
        dict(name='adjoint_ggttg_256K', kind='adjoint', process='ggttg', precision='fp64',
             nevt=1 << 18, sqrts=1500.0),
        # one training batch of the phase-space adaptation
        dict(name='weight_ggtt_16384', kind='weight', process='ggtt', precision='fp64',
             nevt=1 << 14, sqrts=1500.0),
        # cross section and unweighting of a large weighted sample
        dict(name='analysis_5000011', kind='analysis', process='ggttg', precision='fp64',
             nevt=5000011, sqrts=1500.0),
    ]


# largest basket of each kind and process (none costs more than the headline)
LARGEST = {
    ('iteration', 'eemumu'): 1 << 24, ('iteration', 'ggtt'): 1 << 21,
    ('iteration', 'ggttg'): 1 << 20, ('iteration', 'ggttgg'): 1 << 19,
    ('me', 'ggtt'): 1 << 20, ('me', 'ggttg'): 1 << 20, ('me', 'ggttgg'): 1 << 17,
    ('adjoint', 'ggtt'): 1 << 18, ('adjoint', 'ggttg'): 1 << 18,
    ('weight', 'ggtt'): 1 << 18, ('weight', 'ggttg'): 1 << 17,
    ('analysis', 'ggttg'): 1 << 24,
}


def draw(rng):
    kind = rng.choices(['iteration', 'me', 'adjoint', 'weight', 'analysis'], [8, 2, 2, 2, 1])[0]
    process = rng.choice([p for k, p in LARGEST if k == kind])
    precision = 'fp64'
    if kind == 'iteration' and process != 'eemumu':
        precision = rng.choices(['fp64', 'mixed', 'fp32amp'], [5, 2, 1])[0]
    lo = 4096 if kind == 'analysis' else 64
    nevt = int(math.exp(rng.uniform(math.log(lo), math.log(LARGEST[(kind, process)]))))
    nevt = max(lo, nevt | 1) if rng.random() < 0.6 else max(64, nevt // 64 * 64)
    return dict(kind=kind, process=process, precision=precision, nevt=nevt,
                sqrts=rng.choice([1000.0, 1500.0]))


def pages(nevt):
    return (nevt + PAGE - 1) // PAGE


def uniform_events(case, seed):
    """Event-major uniforms (nevt, nrnd) of the seed."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    r = torch.rand(case['nevt'], 4 * (NPAR[case['process']] - 2), generator=g, device=DEV,
                   dtype=F64)
    return r.clamp_(2.0 ** -53, 1.0 - 2.0 ** -53)


def to_pages(x):
    """(nevt, ...) -> AoSoA pages [page][...][64], slots past nevt filled with
    the first event."""
    n = x.shape[0]
    flat = x.reshape(n, -1)
    pad = pages(n) * PAGE - n
    if pad:
        flat = torch.cat([flat, flat[:1].expand(pad, -1)])
    return flat.view(-1, PAGE, flat.shape[1]).transpose(1, 2).contiguous().view(-1)


def lab_momenta(case, seed):
    """RAMBO events boosted along the beam axis (rapidity of the partonic
    system up to 1.5), those that pass a generator's cuts: every pair of legs
    with |2 p_i.p_j| > (20 GeV)^2."""
    n = case['nevt']
    p, _ = phase_space(uniform_events(dict(case, nevt=n + n // 4 + 64), seed), case)
    d = torch.stack([2 * mdot(p[:, i].T, p[:, j].T)
                     for i, j in itertools.combinations(range(p.shape[1]), 2)])
    p = p[(d.abs().amin(0) > 400.0).nonzero()[:n, 0]]
    g = torch.Generator(device=DEV).manual_seed(seed + 1)
    y = 3.0 * torch.rand(n, generator=g, device=DEV, dtype=F64) - 1.5
    ch, sh = torch.cosh(y)[:, None], torch.sinh(y)[:, None]
    return torch.stack([ch * p[..., 0] + sh * p[..., 3], p[..., 1], p[..., 2],
                        sh * p[..., 0] + ch * p[..., 3]], dim=-1)


def cut_weights(case, seed, r):
    """What reaches the gradient from a loss on cut events: a factor per event,
    zero where the outgoing gluon (or top) has pT below 50 GeV."""
    p, _ = phase_space(r, case)
    pt = torch.hypot(p[:, -1, 1], p[:, -1, 2])
    g = torch.Generator(device=DEV).manual_seed(seed + 2)
    return (pt > 50.0).to(F64) * (0.5 + torch.rand(case['nevt'], generator=g, device=DEV,
                                                   dtype=F64))


def event_weights(case, seed):
    """A heavy-tailed weighted sample, one event in 2^16 not finite."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    f = torch.exp(1.3 * torch.randn(case['nevt'], generator=g, device=DEV, dtype=F64))
    bad = torch.rand(case['nevt'], generator=g, device=DEV) < 2.0 ** -16
    return torch.where(bad, torch.full_like(f, float('nan')), f)


def prepare(case, seed):
    n = case['nevt']
    s = dict(case=case, seed=seed,
             engine=mg.MEEngine(case['process'], case['precision'],
                                params=dict(sqrts=case['sqrts'])))
    new = lambda k: torch.zeros(k, dtype=F64, device='cuda')  # noqa: E731
    if case['kind'] in ('iteration', 'me'):
        s.update(me=new(n), evtw=new(n), wgt=new(n))
        if case['kind'] == 'me':
            s.update(mom=to_pages(lab_momenta(case, seed)))
            s['wgt'].fill_(0.5)
        else:
            s.update(mom=new(pages(n) * NPAR[case['process']] * 4 * PAGE))
    elif case['kind'] == 'adjoint':
        r = uniform_events(case, seed)
        s.update(rnd=to_pages(r), gbar=cut_weights(case, seed, r))
    elif case['kind'] == 'weight':
        r = uniform_events(case, seed)
        s.update(r=r.clone().requires_grad_(True), gbar=cut_weights(case, seed, r))
    else:
        f = event_weights(case, seed)
        s.update(f=f, fmax=float(f[torch.isfinite(f)].max()),
                 kept=torch.zeros(n, dtype=torch.int64, device='cuda'))
    return s


def run(s):
    case, eng, n = s['case'], s['engine'], s['case']['nevt']
    if case['kind'] == 'iteration':
        _, mom, wgt = eng.sample(s['seed'], n, mom=s['mom'], wgt=s['wgt'])
        me, evtw = eng.sigmakin(mom, n, wgt=wgt, me=s['me'], evtw=s['evtw'])
        return dict(mom=mom, wgt=wgt, me=me, evtw=evtw)
    if case['kind'] == 'me':
        me, evtw = eng.sigmakin(s['mom'], n, wgt=s['wgt'], me=s['me'], evtw=s['evtw'])
        return dict(me=me, evtw=evtw)
    if case['kind'] == 'adjoint':
        # the two-body weight is a constant: its gradient is not asked for
        grad, glogw, f = eng.adjoint(s['rnd'], n, gbar=s['gbar'],
                                     want_logw=case['process'] != 'ggtt')
        if n % PAGE:                     # the slots past nevt hold no event
            grad, glogw = (x if x is None else eng.rnd_events(x, n) for x in (grad, glogw))
        return dict(grad=grad, glogw=glogw, f=f)
    if case['kind'] == 'weight':
        f = eng.event_weight(s['r'])
        grad, = torch.autograd.grad(f, s['r'], s['gbar'])
        return dict(f=f.detach(), grad=grad)
    sigma, err, stats = eng.cross_section(s['f'], n)
    idx = mg.unweight(s['f'], s['fmax'], s['seed'])
    s['kept'][:idx.numel()] = idx        # the program's list of unweighted events
    return dict(sigma=sigma, error=err, stats=stats, kept=s['kept'])


# Flops per event that the amplitudes cannot do without: every distinct
# (sub-diagram, helicities of its legs) once, every colour flow's contraction
# per helicity, and the colour sum; the gradient three times that.
ME_FLOPS = {'eemumu': 8e2, 'ggtt': 2.5e3, 'ggttg': 2.4e4, 'ggttgg': 3.6e5}


def work(case):
    n, npar = case['nevt'], NPAR[case['process']]
    if case['kind'] == 'iteration':      # momenta, weights, |M|^2 and w |M|^2 written
        return dict(bytes=8 * n * (4 * npar + 3), flops=n * (ME_FLOPS[case['process']] + 300))
    if case['kind'] == 'me':             # momenta and weights read, two results written
        return dict(bytes=8 * n * (4 * npar + 3), flops=n * ME_FLOPS[case['process']])
    if case['kind'] == 'adjoint':        # uniforms and factors read, three results written
        nr = 4 * (npar - 2)
        return dict(bytes=8 * n * (3 * nr + 2), flops=n * (3 * ME_FLOPS[case['process']] + 2000))
    if case['kind'] == 'weight':
        nr = 4 * (npar - 2)
        return dict(bytes=8 * n * (2 * nr + 2), flops=n * (4 * ME_FLOPS[case['process']] + 2000))
    return dict(bytes=16 * n, flops=60 * n)


# ----------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ----------------------------------------------------------------------------
def philox_uniforms(seed, lo, hi, nrnd):
    """Uniforms (hi - lo, nrnd) of events lo .. hi-1: Philox4x32-10 with key
    (seed) and counter (event, block)."""
    m32 = 0xFFFFFFFF
    ev = torch.arange(lo, hi, dtype=torch.int64, device=DEV)

    def hilo(a, b):
        # 32 x 32 -> 64 bits in two 16-bit halves of a
        p0, p1 = (a & 0xFFFF) * b, (a >> 16) * b
        mid = p1 + (p0 >> 16)
        return (mid >> 16) & m32, ((mid << 16) | (p0 & 0xFFFF)) & m32

    cols = []
    for j in range((nrnd + 1) // 2):
        c = [ev & m32, ev >> 32, torch.full_like(ev, j), torch.zeros_like(ev)]
        k0, k1 = seed & m32, (seed >> 32) & m32
        for r in range(10):
            if r:
                k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
            h0, l0 = hilo(c[0], 0xD2511F53)
            h1, l1 = hilo(c[2], 0xCD9E8D57)
            c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        for lo32, hi32 in ((c[0], c[1]), (c[2], c[3])):
            w = (hi32 << 21) | (lo32 >> 11)
            cols.append((w.to(F64) + 0.5) * 2.0 ** -53)
    return torch.stack(cols[:nrnd], dim=1)


def phase_space(r, case):
    """RAMBO: momenta (n, npar, 4) and weights (n,) of event-major uniforms."""
    npar, rs = NPAR[case['process']], case['sqrts']
    nf = npar - 2
    mt = mg.DEFAULT_PARAMS['mt'] if case['process'] != 'eemumu' else 0.0
    mass = torch.tensor([mt, mt] + [0.0] * (nf - 2), dtype=F64, device=r.device)
    u = r.view(-1, nf, 4)
    c = 2 * u[..., 0] - 1
    st = torch.sqrt(1 - c * c)
    phi = 2 * math.pi * u[..., 1]
    e = -torch.log(u[..., 2] * u[..., 3])
    nh = torch.stack([st * torch.cos(phi), st * torch.sin(phi), c], -1)
    d = nh[:, :, None] - nh[:, None]
    dots = 0.5 * e[:, :, None] * e[:, None] * (d * d).sum(-1)
    M = torch.sqrt(dots.sum((1, 2)))[:, None]
    E = dots.sum(2) / M
    Q = (e[..., None] * nh).sum(1)
    t = (e + E) / (e.sum(1, keepdim=True) + M)
    x = rs / M
    p3 = x[..., None] * (e[..., None] * nh - Q[:, None] * t[..., None])
    E = x * E
    w = (math.pi / 2) ** (nf - 1) * rs ** (2 * (nf - 2)) / (math.factorial(nf - 1)
                                                            * math.factorial(nf - 2))
    w = torch.full_like(E[:, 0], w)
    if mt > 0:
        with torch.no_grad():
            xi = torch.full_like(M, math.sqrt(1 - (2 * mt / rs) ** 2))
            for _ in range(12):
                root = torch.sqrt(mass ** 2 + (xi * E) ** 2)
                xi = xi - (root.sum(1, keepdim=True) - rs) / (xi * E * E / root).sum(1, keepdim=True)
            slope = (xi * E * E / torch.sqrt(mass ** 2 + (xi * E) ** 2)).sum(1, keepdim=True)
        # one more step, whose derivative is that of the implicit function
        xi = xi - (torch.sqrt(mass ** 2 + (xi * E) ** 2).sum(1, keepdim=True) - rs) / slope
        p3 = xi[..., None] * p3
        E = torch.sqrt(mass ** 2 + (xi * E) ** 2)
        k = torch.sqrt((p3 * p3).sum(-1))
        w = w * xi[:, 0] ** (2 * nf - 3) * (k / E).prod(1) * rs / (k * k / E).sum(1)
    beams = torch.zeros(r.shape[0], 2, 4, dtype=F64, device=r.device)
    beams[..., 0] = 0.5 * rs
    beams[:, 0, 3] = 0.5 * rs
    beams[:, 1, 3] = -0.5 * rs
    return torch.cat([beams, torch.cat([E[..., None], p3], -1)], 1), w


def mdot(a, b):
    return a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3]


def blocks(v):
    """The 2 x 2 blocks s.V and sbar.V of V-slash (chiral representation)."""
    a, b = v[1] - 1j * v[2], v[1] + 1j * v[2]
    return (v[0] - v[3], -a, -b, v[0] + v[3]), (v[0] + v[3], a, b, v[0] - v[3])


def row_slash(f, v):
    s, sb = blocks(v)
    return (f[2] * sb[0] + f[3] * sb[2], f[2] * sb[1] + f[3] * sb[3],
            f[0] * s[0] + f[1] * s[2], f[0] * s[1] + f[1] * s[3])


def on_axis(minus, plus, leg, npar):
    """The two helicities on the leg's axis of a tensor with one axis per leg."""
    shape = [1] * npar
    shape[leg] = 2
    return torch.stack([minus, plus]).view(*shape, -1)


def polarisation(p, leg, npar, conj):
    kt = torch.hypot(p[:, 1], p[:, 2])
    K = torch.sqrt(kt * kt + p[:, 3] ** 2)
    safe = torch.where(kt > 0, kt, torch.ones_like(kt))
    cp = torch.where(kt > 0, p[:, 1] / safe, torch.ones_like(kt))
    sp = torch.where(kt > 0, p[:, 2] / safe, torch.zeros_like(kt))
    ct, st = p[:, 3] / K, kt / K
    z = torch.zeros_like(ct)
    e1, e2 = (z, ct * cp, ct * sp, -st), (z, -sp, cp, z)
    sign, r2 = (1.0 if conj else -1.0), math.sqrt(0.5)
    return tuple(on_axis(*(torch.complex(-lam * r2 * a, sign * r2 * b) for lam in (-1, 1)), leg, npar)
                 for a, b in zip(e1, e2))


def spinor(p, m, leg, npar, anti, barred):
    """u or v (anti) spinors, or their Dirac adjoints as rows."""
    P = torch.sqrt((p[:, 1:] ** 2).sum(1))
    pt2 = p[:, 1] ** 2 + p[:, 2] ** 2
    up = P + p[:, 3]
    dn = torch.where(P - p[:, 3] > 0, P - p[:, 3], torch.ones_like(P))
    ppz = torch.where(p[:, 3] >= 0, up, pt2 / dn)
    back = ppz <= 0
    ppz = torch.where(back, torch.ones_like(P), ppz)
    nrm = 1 / torch.sqrt(2 * P * ppz)
    one, zero = torch.ones_like(P), torch.zeros_like(P)
    a = torch.where(back, zero, ppz * nrm)
    xr, xi = torch.where(back, one, p[:, 1] * nrm), torch.where(back, zero, p[:, 2] * nrm)
    chi = {1: (torch.complex(a, zero), torch.complex(xr, xi)),
           -1: (torch.complex(-xr, xi), torch.complex(a, zero))}
    big = torch.sqrt(p[:, 0] + P)
    small = m / big
    both = []
    for lam in (-1, 1):
        c = chi[-lam if anti else lam]
        if anti:
            wl, wr = (big, -small) if lam > 0 else (small, -big)
        else:
            wl, wr = (small, big) if lam > 0 else (big, small)
        w = (wl * c[0], wl * c[1], wr * c[0], wr * c[1])
        both.append(tuple(x.conj() for x in (w[2], w[3], w[0], w[1])) if barred else w)
    return tuple(on_axis(x, y, leg, npar) for x, y in zip(*both))


def add(d, key, v):
    d[key] = tuple(a + b for a, b in zip(d[key], v)) if key in d else v


def subsets(legs):
    for r in range(1, len(legs) + 1):
        yield from itertools.combinations(legs, r)


def couplings():
    q = mg.DEFAULT_PARAMS
    e2 = 4 * math.pi / q['alpha_inv']
    mz2 = q['mZ'] ** 2
    mw2 = mz2 / 2 + math.sqrt(mz2 ** 2 / 4 - math.pi / q['alpha_inv'] * mz2
                              / (math.sqrt(2) * q['gfermi']))
    return q, math.sqrt(4 * math.pi * q['alphas']), math.sqrt(e2), 1 - mw2 / mz2


def leptons(p):
    """i M of e+ e- -> mu+ mu-: photon and Z, axes (2, 2, 2, 2, n)."""
    q, _, e, sw2 = couplings()
    npar = 4
    vb, u = spinor(p[:, 0], 0.0, 0, npar, True, True), spinor(p[:, 1], 0.0, 1, npar, False, False)
    v, ub = spinor(p[:, 2], 0.0, 2, npar, True, False), spinor(p[:, 3], 0.0, 3, npar, False, True)
    K = tuple((p[:, 0] + p[:, 1]).unbind(1))
    s = mdot(K, K)

    def current(f, g, cl, cr):
        a, b, c, d = f[0] * g[2], f[1] * g[3], f[0] * g[3], f[1] * g[2]
        w, x, y, z = f[2] * g[0], f[3] * g[1], f[2] * g[1], f[3] * g[0]
        return (cr * (a + b) + cl * (w + x), cr * (c + d) - cl * (y + z),
                1j * (cr * (d - c) - cl * (z - y)), cr * (a - b) - cl * (w - x))

    pref = e / math.sqrt(sw2 * (1 - sw2))
    zl, zr = -pref * (-0.5 + sw2), -pref * sw2
    je, jm = current(vb, u, e, e), current(ub, v, e, e)
    ze, zm = current(vb, u, zl, zr), current(ub, v, zl, zr)
    den = s - q['mZ'] ** 2 + 1j * q['mZ'] * q['wZ']
    return mdot(je, jm) / s + (mdot(ze, zm) - mdot(K, ze) * mdot(K, zm) / q['mZ'] ** 2) / den


def flows(p, npar):
    """Colour-flow amplitudes of g g -> t t~ + n g: {ordering of the gluon
    legs: tensor with one axis per helicity and one for the events}."""
    q, g, _, _ = couplings()
    gl = [0, 1] + list(range(4, npar))
    J, K = {}, {}
    for l in gl:
        J[(l,)] = {(l,): polarisation(p[:, l], l, npar, l > 1)}
        K[(l,)] = tuple((p[:, l] if l < 2 else -p[:, l]).unbind(1))
    for S in subsets(gl):
        if len(S) < 2:
            continue
        K[S] = tuple(sum(x) for x in zip(*(K[(l,)] for l in S)))
        acc = {}
        rest = S[1:]
        parts = [((S[0],) + c, tuple(x for x in rest if x not in c))
                 for r in range(len(rest)) for c in itertools.combinations(rest, r)]
        for A, B in parts:
            ka, kb = K[A], K[B]
            for (wa, a), (wb, b) in itertools.product(J[A].items(), J[B].items()):
                ab = mdot(a, b)
                qa = mdot(tuple(-(2 * x + y) for x, y in zip(ka, kb)), b)
                qb = mdot(tuple(x + 2 * y for x, y in zip(ka, kb)), a)
                v = tuple(-1j * g * (a[m] * qa + ab * (ka[m] - kb[m]) + b[m] * qb) for m in range(4))
                add(acc, wa + wb, v)
                add(acc, wb + wa, tuple(-x for x in v))
            more = B[1:]
            for B1, B2 in [((B[0],) + c, tuple(x for x in more if x not in c))
                           for r in range(len(more)) for c in itertools.combinations(more, r)]:
                for trio in itertools.product(J[A].items(), J[B1].items(), J[B2].items()):
                    dot = {(i, j): mdot(trio[i][1], trio[j][1]) for i, j in ((0, 1), (0, 2), (1, 2))}
                    for o in itertools.permutations(range(3)):
                        # colour-ordered four-gluon vertex: 2 y (x.z) - x (y.z) - z (x.y)
                        (wx, x), (wy, y), (wz, z) = (trio[k] for k in o)
                        xz, yz, xy = (dot[tuple(sorted(t))] for t in ((o[0], o[2]), (o[1], o[2]),
                                                                     (o[0], o[1])))
                        add(acc, wx + wy + wz,
                            tuple(1j * g * g * (2 * y[m] * xz - x[m] * yz - z[m] * xy)
                                  for m in range(4)))
        prop = -1j / mdot(K[S], K[S])
        J[S] = {w: tuple(prop * c for c in v) for w, v in acc.items()}
    pt = tuple(p[:, 2].unbind(1))
    U = {(): {(): spinor(p[:, 2], q['mt'], 2, npar, False, True)}}
    vb = spinor(p[:, 3], q['mt'], 3, npar, True, False)
    out = {}
    for S in subsets(gl):
        acc = {}
        for T in subsets(S):
            left = tuple(x for x in S if x not in T)
            for (wu, f), (wj, j) in itertools.product(U[left].items(), J[T].items()):
                add(acc, wu + wj, tuple(1j * g * x for x in row_slash(f, j)))
        if len(S) == len(gl):
            return {w: sum(a * b for a, b in zip(r, vb)) for w, r in acc.items()}
        k = tuple(a - b for a, b in zip(pt, K[S]))
        prop = 1j / (mdot(k, k) - q['mt'] ** 2 + 1j * q['mt'] * q['wt'])
        U[S] = {w: tuple(prop * (a + q['mt'] * b) for a, b in zip(row_slash(r, k), r))
                for w, r in acc.items()}
    return out


def colour_matrix(ng):
    """Overlaps of the strings of ng SU(3) generators, orderings in
    itertools.permutations order."""
    lam = torch.zeros(8, 3, 3, dtype=C128)
    for k, (i, j) in zip((0, 3, 5), ((0, 1), (0, 2), (1, 2))):
        lam[k, i, j] = lam[k, j, i] = 1
        lam[k + 1, i, j], lam[k + 1, j, i] = -1j, 1j
    lam[2] = torch.diag(torch.tensor([1, -1, 0], dtype=C128))
    lam[7] = torch.diag(torch.tensor([1, 1, -2], dtype=C128)) / math.sqrt(3)
    T = lam / 2
    s = T
    for _ in range(ng - 1):          # s[a1, ..., ak, i, j]
        s = (s[..., None, :, :, None] * T[:, None]).sum(-2)
    rows = []
    for w in itertools.permutations(range(ng)):
        inv = [w.index(k) for k in range(ng)]
        rows.append(s.permute(*inv, ng, ng + 1).reshape(-1))
    M = torch.stack(rows)
    return (M @ M.conj().T).real


def matrix_elements(p, process):
    npar = NPAR[process]
    if process == 'eemumu':
        a = leptons(p)
        return (a.real ** 2 + a.imag ** 2).sum((0, 1, 2, 3)) / IDEN[process]
    gl = [0, 1] + list(range(4, npar))
    amps = flows(p, npar)
    words = list(itertools.permutations(gl))
    C = colour_matrix(len(gl)).to(p.device)
    total = 0.0
    for i, w in enumerate(words):
        z = sum(float(C[i, j]) * amps[v] for j, v in enumerate(words))
        total = total + (amps[w].real * z.real + amps[w].imag * z.imag)
    return total.sum(tuple(range(npar))) / IDEN[process]


# events worked on together: bounds the memory of the helicity tensors
CHUNK = {'eemumu': 1 << 20, 'ggtt': 1 << 17, 'ggttg': 1 << 15, 'ggttgg': 1 << 13}


def exact(case, seed):
    n, proc = case['nevt'], case['process']
    if case['kind'] == 'analysis':
        f = event_weights(case, seed)
        f = f[torch.isfinite(f)]
        mean, sq = float(f.sum()) / n, float((f * f).sum()) / n
        nf = NPAR[proc] - 2
        scale = 0.3893793721e9 * (2 * math.pi) ** (4 - 3 * nf) / (2 * case['sqrts'] ** 2)
        stats = torch.stack([f.sum(), (f * f).sum(), f.max(), torch.tensor(float(f.numel()), dtype=F64,
                                                                            device=f.device)])
        return dict(sigma=scale * mean, error=scale * math.sqrt((sq - mean * mean) / (n - 1)),
                    stats=stats.cpu(), kept=None)
    step = CHUNK[proc]
    if case['kind'] in ('adjoint', 'weight'):
        r = uniform_events(case, seed)
        gbar = cut_weights(case, seed, r)
        fs, grads, logs = [], [], []
        for lo in range(0, n, step // 4):
            x = r[lo:lo + step // 4].clone().requires_grad_(True)
            p, w = phase_space(x, case)
            f = w * matrix_elements(p, proc)
            fs.append(f.detach())
            grads.append(torch.autograd.grad(f.sum(), x, retain_graph=True)[0])
            if case['kind'] == 'adjoint' and proc != 'ggtt':
                logs.append(torch.autograd.grad(torch.log(w).sum(), x)[0])
        grad = gbar[:, None] * torch.cat(grads)
        if case['kind'] == 'weight':
            return dict(f=torch.cat(fs), grad=grad)
        glogw = torch.cat(logs) if logs else None
        if n % PAGE == 0:
            grad, glogw = (x if x is None else to_pages(x) for x in (grad, glogw))
        return dict(f=torch.cat(fs), grad=grad, glogw=glogw)
    if case['kind'] == 'me':
        p = lab_momenta(case, seed)
        me = torch.cat([matrix_elements(p[lo:lo + step], proc) for lo in range(0, n, step)])
        return dict(me=me, evtw=0.5 * me)
    mes, ws, mom = [], [], torch.zeros(pages(n) * PAGE, 4 * NPAR[proc], dtype=F64, device=DEV)
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        p, w = phase_space(philox_uniforms(seed, lo, hi, 4 * (NPAR[proc] - 2)), case)
        mes.append(matrix_elements(p, proc))
        ws.append(w)
        mom[lo:hi] = p.reshape(hi - lo, -1)
    me, w = torch.cat(mes), torch.cat(ws)
    return dict(mom=to_pages(mom), wgt=w, me=me, evtw=w * me)
