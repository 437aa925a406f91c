// FP64 gradient of |M|^2 with respect to the final-state momenta for
// g g -> t t~ and g g -> t t~ g, with the currents shared between helicities
// (shared_currents.h) in the forward and in the reverse sweep.
//
// Three kernels share the caller's gradient buffer, which holds as many
// numbers per event as RAMBO has uniforms, 4 per final-state particle:
//   1  RAMBO (rambo_grad.hip): final-state momenta into the buffer;
//   2  this one: momenta -> d(sum |M|^2)/dp_i (three-vectors: the energies
//      are on the mass shell) and sum |M|^2 in their place;
//   3  the reverse sweep of RAMBO (rambo_grad.hip): the gradient with
//      respect to the uniforms.
// A lane takes one combination of gluon helicities of an event, with the four
// quark helicities; the lanes of an event are summed by DPP.
//
// g g -> t t~: 4 lanes an event; 2^18 events in 99 us, 16384 in 16 us (one
// event per lane with a helicity loop and 8 dual RAMBO passes: 671 and 167 us).
// g g -> t t~ g: 16 lanes an event, one per helicity of the gluons and the t~,
// since the accumulators of both t~ helicities do not fit the registers (8
// lanes: 1.6 KB of scratch a lane, 3.2 ms).  The U(a) and W(a) depend on one
// gluon's helicity: a lane forms one of each, and their adjoints, summed over
// the lanes of a version through LDS, are taken on by one lane (each lane for
// itself: 1.21 ms).  2^18 events in 0.99 ms, 70 events in 29 us (3.97 and
// 1.05 ms with one event per lane).  Bound: FP64 VALU at one wave per SIMD of
// 512 registers, 6.4e3 instructions a wave, 14 % of them copies to and from
// AGPRs; versions, adjoints of the flows and momenta wait in LDS (35 KB a wave;
// momenta in registers cost 75 reloads from scratch, one after the other), and
// identical forward values are computed again in the reverse sweep rather than
// kept (pin below: without it 2.3 KB of scratch and 6.8 ms).
//
// Adjoints follow helas_adj.h: zb = dL/d(Re z) + i dL/d(Im z).
#pragma once
#include "helas_adj.h"
#include "shared_currents.h"

namespace mg {

// The spinors, vectors and numbers named are fixed here: what went into them
// is computed before, and what is computed from them is not merged with an
// earlier computation of the same, whose result would stay live.
__device__ __forceinline__ void pin_one(c64 (&w)[4]) { opaque4(w); }
__device__ __forceinline__ void pin_one(c64& w) {
  opaque(w.r);
  opaque(w.i);
}
__device__ __forceinline__ void pin_one(double (&k)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) opaque(k[m]);
}
__device__ __forceinline__ void pin_one(double& x) { opaque(x); }
template <class... A>
__device__ __forceinline__ void pin(A&... a) {
  (pin_one(a), ...);
}

// c + conj(a) b, c - conj(a) b
__device__ __forceinline__ c64 cmadd_conj(c64 a, c64 b, c64 c) {
  return {fmadd(a.r, b.r, fmadd(a.i, b.i, c.r)), fmadd(a.r, b.i, fmadd(-a.i, b.r, c.i))};
}
__device__ __forceinline__ c64 cmsub_conj(c64 a, c64 b, c64 c) {
  return {fmadd(-a.r, b.r, fmadd(-a.i, b.i, c.r)), fmadd(-a.r, b.i, fmadd(a.i, b.r, c.i))};
}
__device__ __forceinline__ void clear4(c64 (&w)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = c64{0.0, 0.0};
}

// a = sdot(u, w): ub, wb
__device__ __forceinline__ void adj_sdot(const c64 (&u)[4], const c64 (&w)[4], c64 ab,
                                         c64 (&ub)[4], c64 (&wb)[4]) {
  ub[0] = cmadd_conj(w[1], ab, ub[0]);
  ub[1] = cmsub_conj(w[0], ab, ub[1]);
  ub[2] = cmadd_conj(w[3], ab, ub[2]);
  ub[3] = cmsub_conj(w[2], ab, ub[3]);
  wb[0] = cmsub_conj(u[1], ab, wb[0]);
  wb[1] = cmadd_conj(u[0], ab, wb[1]);
  wb[2] = cmsub_conj(u[3], ab, wb[2]);
  wb[3] = cmadd_conj(u[2], ab, wb[3]);
}

// f = V-slash G: Gb += V-slash^H fb
__device__ __forceinline__ void adj_slash_spinor(const c64 (&V)[4], const c64 (&fb)[4],
                                                 c64 (&Gb)[4]) {
  blk<double> s, sb;
  slash_blocks(V, s, sb);
  Gb[2] = cmadd_conj(s.a, fb[0], cmadd_conj(s.c, fb[1], Gb[2]));
  Gb[3] = cmadd_conj(s.b, fb[0], cmadd_conj(s.d, fb[1], Gb[3]));
  Gb[0] = cmadd_conj(sb.a, fb[2], cmadd_conj(sb.c, fb[3], Gb[0]));
  Gb[1] = cmadd_conj(sb.b, fb[2], cmadd_conj(sb.d, fb[3], Gb[1]));
}
// f = V-slash G: Vb
__device__ __forceinline__ void adj_slash_vector(const c64 (&G)[4], const c64 (&fb)[4],
                                                 c64 (&Vb)[4]) {
  const c64 z{0.0, 0.0};
  const c64 a = cmadd_conj(G[2], fb[0], z), b = cmadd_conj(G[3], fb[1], z),
            c = cmadd_conj(G[0], fb[2], z), d = cmadd_conj(G[1], fb[3], z);
  const c64 e = cmadd_conj(G[3], fb[0], z), f = cmadd_conj(G[2], fb[1], z),
            g = cmadd_conj(G[1], fb[2], z), h = cmadd_conj(G[0], fb[3], z);
  // sV = [[V0 - V3, -V1 + i V2], [-V1 - i V2, V0 + V3]], sbV its spatial reflection
  Vb[0] = Vb[0] + ((a + b) + (c + d));
  Vb[3] = Vb[3] + ((b - a) + (c - d));
  Vb[1] = Vb[1] + ((g + h) - (e + f));
  Vb[2] = Vb[2] + times_i((f - e) + (g - h));
}

// out = d (q-slash + m) f with d = -g / (q^2 - m^2 + i m w): fb (returned) and qb
__device__ __forceinline__ void adj_propagate(const double (&q)[4], double m, double ig, c64 d,
                                              const c64 (&f)[4], const c64 (&ob)[4],
                                              c64 (&fb)[4], double (&qb)[4]) {
  c64 o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) o[k] = conj(d) * ob[k];
  sbK_col(q, o[2], o[3], fb[0], fb[1]);
  sK_col(q, o[0], o[1], fb[2], fb[3]);
#pragma unroll
  for (int k = 0; k < 4; ++k) fb[k] = rmadd(m, o[k], fb[k]);
  adj_kslash_col(f[2], f[3], f[0], f[1], o[0], o[1], o[2], o[3], 1.0, qb);
  // <ob, out> = <fb, f>;  d(d) = (d^2 / g) d(q^2)
  const c64 s = cdot4(fb, f);
  add_msq_grad(q, ig * (d.r * s.r - d.i * s.i), qb);
}

// o = L(x, y): adjoint of y and its momentum (x, kx without derivative)
__device__ __forceinline__ void adj_three_gluon_y(const c64 (&x)[4], const double (&kx)[4],
                                                  const c64 (&y)[4], const double (&ky)[4],
                                                  const c64 (&ob)[4], c64 (&yb)[4],
                                                  double (&kyb)[4]) {
  double qx[4], qy[4], dk[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    qx[m] = -(2.0 * kx[m] + ky[m]);
    qy[m] = kx[m] + 2.0 * ky[m];
    dk[m] = kx[m] - ky[m];
  }
  const c64 cy_ = mdot(qy, x), xy = mdot0(x, y), xo = cdot4(x, ob), yo = cdot4(y, ob);
  c64 dko = dk[0] * ob[0];
#pragma unroll
  for (int m = 1; m < 4; ++m) dko = rmadd(dk[m], ob[m], dko);
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const double g = metric(m);
    yb[m] = cmadd_conj(cy_, ob[m], rmadd(g * qx[m], xo, yb[m]));
    yb[m] = g > 0 ? cmadd_conj(x[m], dko, yb[m]) : cmsub_conj(x[m], dko, yb[m]);
    kyb[m] += g * (2.0 * redot(yo, x[m]) - redot(xo, y[m])) - redot(ob[m], xy);
  }
}

// Helicity states and roots of a quark (helicity_states), and their adjoints
struct QuarkAdjoint {
  double c, x, y, big, small;       // adjoints
  __device__ __forceinline__ QuarkAdjoint() : c(0.0), x(0.0), y(0.0), big(0.0), small(0.0) {}

  // spinor of helicity h (0 / 1) as in quark_spinors, wb its adjoint
  __device__ __forceinline__ void add(const double (&p)[4], double m, bool anti, int h,
                                      const c64 (&wb)[4]) {
    double vc, vx, vy, vbig, vsmall;
    helicity_states<0>(p, m, vc, vx, vy, vbig, vsmall);
    const bool up = (h == 1) != anti;
    const double wp = h ? vbig : vsmall, wm = h ? vsmall : vbig;
    const c64 c0 = up ? c64{vc, 0.0} : c64{-vx, vy}, c1 = up ? c64{vx, vy} : c64{vc, 0.0};
    double wpb, wmb;
    c64 c0b, c1b;
    if (anti) {
      wpb = redot(wb[0], c0) + redot(wb[1], c1);
      wmb = -redot(wb[2], c0) - redot(wb[3], c1);
      c0b = wp * wb[0] - wm * wb[2];
      c1b = wp * wb[1] - wm * wb[3];
    } else {
      wpb = redot(wb[0], conj(c1)) - redot(wb[1], conj(c0));
      wmb = redot(wb[2], conj(c1)) - redot(wb[3], conj(c0));
      c1b = conj(wp * wb[0] + wm * wb[2]);
      c0b = -conj(wp * wb[1] + wm * wb[3]);
    }
    if (h) {
      big += wpb;
      small += wmb;
    } else {
      small += wpb;
      big += wmb;
    }
    c += up ? c0b.r : c1b.r;
    x += up ? c1b.r : -c0b.r;
    y += up ? c1b.i : c0b.i;
  }

  // to the momentum; along -z and at rest the states are constants and P has
  // no derivative (helicity_states, helicity_chi)
  __device__ __forceinline__ void finish(const double (&p)[4], double m, double (&pb)[4]) const {
    double vc, vx, vy, vbig, vsmall;
    helicity_states<0>(p, m, vc, vx, vy, vbig, vsmall);
    const double pt2 = p[1] * p[1] + p[2] * p[2], P2 = pt2 + p[3] * p[3];
    const double iP = P2 > 0.0 ? rsqrt_refined(P2) : 0.0, P = P2 * iP;
    const double ppz = p[3] >= 0.0 ? P + p[3] : pt2 * recip(P - p[3]);
    // (c, x, y) = nrm (P + pz, px, py)
    const double nrm = ppz > 0.0 ? rsqrt_refined(2.0 * P * ppz) : 0.0;
    const double nb = c * ppz + x * p[1] + y * p[2];
    const double Nb = -0.5 * nrm * nrm * nrm * nb;    // N = 2 P (P + pz) = nrm^-2
    const double ppzb = c * nrm + 2.0 * P * Nb;
    const double ibig = recip(vbig);
    const double eb = 0.5 * ibig * (big - small * vsmall * ibig);
    const double Pb = 2.0 * ppz * Nb + eb;
    // d(P + pz) = (px dpx + py dpy + (P + pz) dpz) / P
    pb[0] += eb;
    pb[1] += x * nrm + iP * p[1] * (Pb + ppzb);
    pb[2] += y * nrm + iP * p[2] * (Pb + ppzb);
    pb[3] += iP * (p[3] * Pb + ppz * ppzb);
  }
};

// conjugate polarisation vector of an outgoing gluon: adjoint to its momentum
__device__ __forceinline__ void adj_polarisation(const double (&p)[4], int lam,
                                                 const c64 (&wb)[4], double (&pb)[4]) {
  const double r2 = 0.70710678118654752440;
  const double a = -lam * r2, b = r2;
  const double pt2 = p[1] * p[1] + p[2] * p[2];
  const double iK = rsqrt_refined(pt2 + p[3] * p[3]);
  const bool pt = pt2 > 0.0;
  const double ikt = rsqrt_refined(pt ? pt2 : 1.0);
  const double cph = pt ? p[1] * ikt : 1.0, sph = pt ? p[2] * ikt : 0.0;
  const double cth = p[3] * iK, sth = pt2 * ikt * iK;
  // w = (0, a cth cph - i b sph, a cth sph + i b cph, -a sth)
  const double cthb = a * (cph * wb[1].r + sph * wb[2].r), sthb = -a * wb[3].r;
  const double cphb = a * cth * wb[1].r + b * wb[2].i, sphb = a * cth * wb[2].r - b * wb[1].i;
  const double T = ikt * (sph * cphb - cph * sphb);
  const double S = iK * (sth * cthb - cth * sthb);
  pb[1] += sph * T - cth * S * cph;
  pb[2] -= cph * T + cth * S * sph;
  pb[3] += sth * S;
}

// sum over the L lanes (4 or 16) of an event
template <int L>
__device__ __forceinline__ double lanes_sum(double v) {
  v += dpp_move<0xB1>(v);                   // quad_perm 1 0 3 2
  v += dpp_move<0x4E>(v);                   // quad_perm 2 3 0 1
  if constexpr (L == 16) {
    v += dpp_move<0x141>(v);                // row_half_mirror
    v += dpp_move<0x140>(v);                // row_mirror
  }
  return v;
}

// A helicity's colour flows A (without g): value and adjoint 2 C A of the
// colour sum, both times `scale`
template <class P>
__device__ __forceinline__ double adj_colour(const c64 (&A)[P::NCOL], double scale,
                                             c64 (&Ab)[P::NCOL]) {
  const double s = scale / P::CDEN;
  double v = 0.0;
#pragma unroll
  for (int i = 0; i < P::NCOL; ++i) {
    c64 z{0.0, 0.0};
#pragma unroll
    for (int j = 0; j < P::NCOL; ++j)
      if (P::cnum(i, j)) z = rmadd((double)P::cnum(i, j), A[j], z);
    v += redot(A[i], z);
    Ab[i] = (2.0 * s) * z;
  }
  return s * v;
}

// d(sum |M|^2)/dp of the final-state legs, times nothing else; me: the sum
template <class P>
struct GradGGTT : GGTT<true, ColourSum<P>> {
  static constexpr int LANES = 4, LDS = 1;
  using B = GGTT<true, ColourSum<P>>;
  using B::u; using B::v; using B::d; using B::k0; using B::k1; using B::q; using B::f01; using B::cp;
  __device__ __forceinline__ GradGGTT(const double (&p)[4][4], const Couplings<double>& c)
      : B(p, c) {}

  __device__ __forceinline__ double gradient(const double (&p)[4][4], int g, uint64_t mask, d2*,
                                             double (&pb)[P::NPAR][4]) {
    c64 e[2][4], J[4], ub[2][4];
    polarisation<1>(k0, g & 2 ? 1 : -1, false, e[0]);
    polarisation<-1>(k1, g & 1 ? 1 : -1, false, e[1]);
    three_gluon(e[0], k0, e[1], k1, J);
#pragma unroll
    for (int m = 0; m < 4; ++m) J[m] = -f01 * J[m];
    clear4(ub[0]);
    clear4(ub[1]);
    const double ig = recip(cp.gs);
    QuarkAdjoint qt, qb;
    double me = 0.0;
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      c64 W[2][4], phi[2][4], s[4], R[2][4], Rb[2][4], Wb[4], vb[4], pb_[4];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        slash_col(e[a], v[tb], phi[a]);
        propagate(q[a], cp.mt, d[a], phi[a], W[a]);
      }
      slash_col(J, v[tb], s);
      slash_col(e[0], W[1], R[0]);
      slash_col(e[1], W[0], R[1]);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        R[0][m] = R[0][m] + s[m];
        R[1][m] = R[1][m] - s[m];
      }
      clear4(Rb[0]);
      clear4(Rb[1]);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const c64 z{0.0, 0.0};
        const c64 A[2] = {sdot_add(u[t], R[0], z), sdot_add(u[t], R[1], z)};
        c64 Ab[2];
        const int h = ((g & 3) << 2) | (t << 1) | tb;
        me += adj_colour<P>(A, (mask >> h) & 1 ? cp.gs2 : 0.0, Ab);
        adj_sdot(u[t], R[0], Ab[0], ub[t], Rb[0]);
        adj_sdot(u[t], R[1], Ab[1], ub[t], Rb[1]);
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) s[m] = Rb[0][m] - Rb[1][m];
      clear4(vb);
      adj_slash_spinor(J, s, vb);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        double kb[4] = {0.0, 0.0, 0.0, 0.0};
        clear4(Wb);
        adj_slash_spinor(e[1 - a], Rb[1 - a], Wb);
        adj_propagate(q[a], cp.mt, ig, d[a], phi[a], Wb, pb_, kb);
        adj_slash_spinor(e[a], pb_, vb);
#pragma unroll
        for (int m = 0; m < 4; ++m) pb[3][m] -= kb[m];
      }
      qb.add(p[3], cp.mt, true, tb, vb);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) qt.add(p[2], cp.mt, false, t, ub[t]);
    qt.finish(p[2], cp.mt, pb[2]);
    qb.finish(p[3], cp.mt, pb[3]);
    return me;
  }
};

template <class P>
struct GradGGTTG : GGTTG<true, ColourSum<P>> {
  // LDS in complex numbers: the versions of U and of W, component-major (an
  // event has 12 of each: quark helicity, gluon, gluon helicity), the adjoints
  // of the flows, U's adjoints of the 64 lanes on their way to the sum over the
  // lanes of a version (those of gluon 2 in the place of flows already used),
  // the momenta
  static constexpr int LANES = 16, SU = 0, SW = SU + 192, FLOW = SW + 192, UB = FLOW + 12 * 64,
                       EVENT = UB + 4 * 256, LDS = EVENT + 4 * 6;
  using B = GGTTG<true, ColourSum<P>>;
  using B::u; using B::v; using B::k; using B::cp;
  __device__ __forceinline__ GradGGTTG(const double (&p)[5][4], const Couplings<double>& c)
      : B(p, c) {}

  // what the reverse sweep needs of the polarisation's adjoint
  __device__ __forceinline__ static void pin_eps(c64 (&eb)[4]) {
    pin(eb[1], eb[2], eb[3].r);
  }

  // momentum of leg 2 + l, read again at each use
  __device__ __forceinline__ static void momentum(const d2* lds, int& at, int l, double (&q)[4]) {
    asm volatile("" : "+v"(at));
    lds_get_real(lds + at + 2 * l, q);
  }

  __device__ __forceinline__ double gradient(const double (&p)[5][4], int g, uint64_t mask,
                                             d2* lds, double (&pb)[P::NPAR][4]) {
    const int lane = threadIdx.x;
    int at = EVENT + 6 * (lane / LANES);
#pragma unroll
    for (int l = 0; l < 3; ++l) {  // the same from each lane of the event
      lds[at + 2 * l] = d2{p[l + 2][0], p[l + 2][1]};
      lds[at + 2 * l + 1] = d2{p[l + 2][2], p[l + 2][3]};
    }
    c64 e[3][4], J[3][4], M[2][4];
    const int tb = g & 1, lam2 = g & 2 ? 1 : -1;
    B::gluon_currents(g & 8 ? 1 : -1, g & 4 ? 1 : -1, lam2, e, J, M);
    // U and W depend on one gluon's helicity: each is formed by one lane of the
    // event, that of gluon `own` at the lane's helicity of it and of the quark
    // (two lanes in eight are spare: they repeat gluon 0)
    const int l0 = (g >> 3) & 1, l1 = (g >> 2) & 1, l2 = (g >> 1) & 1;
    const int own = l0 == l1 ? (l1 == l2 ? 0 : 1) : (l0 == l2 ? 2 : 0);
    const bool spare = l0 != l1 && l1 == l2;
    const int ver = 12 * (lane / LANES);
    auto version = [&](int q, int a, int l) { return ver + 2 * (3 * q + a) + l; };
    const int mine = version(tb, own, own == 0 ? l0 : own == 1 ? l1 : l2);
    auto pick = [&](double x0, double x1, double x2) { return own == 0 ? x0 : own == 1 ? x1 : x2; };
    c64 vt[4], ut[4], ea[4];
    double ka[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      vt[m].r = tb ? v[1][m].r : v[0][m].r;
      vt[m].i = tb ? v[1][m].i : v[0][m].i;
      ut[m].r = tb ? u[1][m].r : u[0][m].r;
      ut[m].i = tb ? u[1][m].i : u[0][m].i;
    }
    auto own_gluon = [&]() {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        ea[m].r = pick(e[0][m].r, e[1][m].r, e[2][m].r);
        ea[m].i = pick(e[0][m].i, e[1][m].i, e[2][m].i);
        ka[m] = pick(k[0][m], k[1][m], k[2][m]);
      }
    };
    auto own_factor = [&](const double (&q)[4]) {
      return quark_factor(q, cp.mt, own < 2 ? cp.wtt : cp.wt, cp.gs);
    };
    own_gluon();
    {
      c64 s[4], o[4];
      double q[4], pq[4];
      momentum(lds, at, 0, pq);
      slash_col(ea, ut, s);
      minus4(pq, ka, q);
      propagate(q, cp.mt, own_factor(q), s, o);
      lds_put(lds + SU + mine, 48, o);
      momentum(lds, at, 1, pq);
      slash_col(ea, vt, s);
      minus4(ka, pq, q);
      propagate(q, cp.mt, own_factor(q), s, o);
      lds_put(lds + SW + mine, 48, o);
      pin(ut, ea, ka);
    }
    __syncthreads();
    auto get_U = [&](int t, int a, c64 (&w)[4]) {
      lds_get(lds + SU + version(t, a, a == 0 ? l0 : a == 1 ? l1 : l2), 48, w);
    };
    // adjoints: u, e[2], J[0], J[1] (J[2] and e[0], e[1] have no derivative), M, k[2]
    c64 ub[2][4], eb[4], Jb[2][4], Mb[2][4];
    double k2b[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      clear4(ub[i]);
      clear4(Jb[i]);
      clear4(Mb[i]);
    }
    clear4(eb);
    const double ig = recip(cp.gs);
    QuarkAdjoint qt, qb;
    double me = 0.0;
    const int code = ((g & 12) << 1) | (tb << 1) | ((g >> 1) & 1);
    const c64 z{0.0, 0.0};
    c64 W[3][4];
    // adjoints of the flows: flow k of t helicity t at [64 (2 k + t)]
    d2* flow = lds + FLOW + lane;
    auto flow_adjoint = [&](int t, int k) { return lds_scalar(flow + 64 * (2 * k + t)); };
    {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lds_get(lds + SW + version(tb, a, a == 0 ? l0 : a == 1 ? l1 : l2), 48, W[a]);
        pin(W[a]);
      }
      {
        c64 A[2][6], s[4], r[4];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const int b = a == 0 ? 1 : 0, c = a == 2 ? 1 : 2;
          pin(vt, W[b], W[c]);
          c64 U[2][4];
#pragma unroll
          for (int t = 0; t < 2; ++t) get_U(t, a, U[t]);
          slash_col(J[a], vt, s);
#pragma unroll
          for (int m = 0; m < 4; ++m) r[m] = s[m];
          slash_col_add(e[b], W[c], r);
#pragma unroll
          for (int t = 0; t < 2; ++t) A[t][2 * a] = sdot_add(U[t], r, z);
#pragma unroll
          for (int m = 0; m < 4; ++m) r[m] = -s[m];
          slash_col_add(e[c], W[b], r);
#pragma unroll
          for (int t = 0; t < 2; ++t) A[t][2 * a + 1] = sdot_add(U[t], r, z);
          pin(A[0][2 * a], A[0][2 * a + 1], A[1][2 * a], A[1][2 * a + 1]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const int a = c == 0 ? 1 : 0, b = c == 2 ? 1 : 2;
          pin(W[c], u[0], u[1]);
          slash_col(J[c], W[c], s);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const c64 x = sdot_add(u[t], s, z);
            A[t][2 * a + (b > c)] = A[t][2 * a + (b > c)] + x;
            A[t][2 * b + (a > c)] = A[t][2 * b + (a > c)] - x;
            pin(A[t][2 * a + (b > c)], A[t][2 * b + (a > c)]);
          }
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          pin(vt, u[0], u[1]);
          slash_col(M[m], vt, s);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const c64 y = sdot_add(u[t], s, z);
            const int i = m ? 0 : 2, j = m ? 5 : 4;  // middle 0: (102), (201); middle 1: (012), (210)
            A[t][i] = A[t][i] + y;
            A[t][j] = A[t][j] + y;
            A[t][1] = A[t][1] - y;                   // middle 2
            A[t][3] = A[t][3] - y;
            pin(A[t][i], A[t][j], A[t][1], A[t][3]);
          }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int h = code | (t << 2);
          c64 Ab[6];
          me += adj_colour<P>(A[t], (mask >> h) & 1 ? cp.gs2 : 0.0, Ab);
          pin(Ab[0], Ab[1], Ab[2], Ab[3], Ab[4], Ab[5], me);
#pragma unroll
          for (int k = 0; k < 6; ++k) flow[64 * (2 * k + t)] = d2{Ab[k].r, Ab[k].i};
        }
      }
      // ---- reverse -------------------------------------------------------
      pin(J[0], J[1]);
      pin_eps(e[2]);
      c64 vb[4];
      clear4(vb);
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        pin(vt, u[0], u[1], M[m]);
        c64 s[4], sb[4];
        slash_col(M[m], vt, s);
        clear4(sb);
#pragma unroll
        for (int t = 0; t < 2; ++t)
          adj_sdot(u[t], s, (flow_adjoint(t, m ? 0 : 2) + flow_adjoint(t, m ? 5 : 4)) -
                   (flow_adjoint(t, 1) + flow_adjoint(t, 3)), ub[t],
                   sb);
        adj_slash_spinor(M[m], sb, vb);
        adj_slash_vector(vt, sb, Mb[m]);
        pin(ub[0], ub[1], vb, Mb[m]);
      }
    // M is done with
    {
      double K[4];
      plus4(k[0], k[1], K);
      // M = (g / K3^2) T: T0 = L1 - L3 + Q(1, 0, 2), T1 = -L1 - L2 + Q(0, 1, 2)
      double K3[4];
      plus4(K, k[2], K3);
      pin(K3);
      const double f012 = cp.gs * recip(msq(K3));
      const double s = -ig * f012 * (cdot4(Mb[0], M[0]).r + cdot4(Mb[1], M[1]).r);
      add_msq_grad(K3, s, k2b);
      c64 t0[4], t1[4], o[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        t0[m] = f012 * Mb[0][m];
        t1[m] = f012 * Mb[1][m];
      }
      const c64 d01 = cp.gs * mdot0(e[0], e[1]);
      c64 x = z, y = z;  // adjoints of e1.e2 and e0.e2
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        x = cmadd_conj(e[0][m], 2.0 * t0[m] - t1[m], x);
        y = cmadd_conj(e[1][m], 2.0 * t1[m] - t0[m], y);
      }
      x = cp.gs * x;
      y = cp.gs * y;
#pragma unroll
      for (int m = 1; m < 4; ++m)
        eb[m] = cmsub_conj(d01, t0[m] + t1[m], cmsub_conj(e[1][m], x, cmsub_conj(e[0][m], y, eb[m])));
#pragma unroll
      for (int m = 0; m < 4; ++m) o[m] = t0[m] - t1[m];
      adj_three_gluon_y(J[2], K, e[2], k[2], o, eb, k2b);
      pin(t0, t1, k2b);
      pin_eps(eb);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        t0[m] = -t0[m];
        t1[m] = -t1[m];
      }
      plus4(k[1], k[2], K);
      adj_three_gluon_y(e[0], k[0], J[0], K, t1, Jb[0], k2b);
      plus4(k[0], k[2], K);
      adj_three_gluon_y(e[1], k[1], J[1], K, t0, Jb[1], k2b);
      pin(Jb[0], Jb[1], k2b);
    }
      c64 Wb[3][4];
      clear4(Wb[0]);
      clear4(Wb[1]);
      clear4(Wb[2]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const int a = c == 0 ? 1 : 0, b = c == 2 ? 1 : 2;
        const c64 xb[2] = {flow_adjoint(0, 2 * a + (b > c)) - flow_adjoint(0, 2 * b + (a > c)),
                           flow_adjoint(1, 2 * a + (b > c)) - flow_adjoint(1, 2 * b + (a > c))};
        pin(W[c], u[0], u[1]);
        if (c < 2) pin(J[c]);
        c64 s[4], sb[4];
        slash_col(J[c], W[c], s);
        clear4(sb);
#pragma unroll
        for (int t = 0; t < 2; ++t)
          adj_sdot(u[t], s, xb[t], ub[t], sb);
        adj_slash_spinor(J[c], sb, Wb[c]);
        if (c < 2) adj_slash_vector(W[c], sb, Jb[c]);
        pin(ub[0], ub[1], Wb[c]);
        if (c < 2) pin(Jb[c]);
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int b = a == 0 ? 1 : 0, c = a == 2 ? 1 : 2;
        if (a < 2) pin(J[a]);
        pin_eps(e[2]);
        c64 sb[4], Ub[2][4];
        clear4(sb);
        clear4(Ub[0]);
        clear4(Ub[1]);
#pragma unroll
        for (int o = 0; o < 2; ++o) {  // U(a).r, r = +-J-slash(a) v + e-slash(x) W(y)
          const int x = o ? c : b, y = o ? b : c;
          // read before they are needed: a read stops at the next pin
          c64 U[2][4], r[4], rb[4];
          const c64 Ab[2] = {flow_adjoint(0, 2 * a + o), flow_adjoint(1, 2 * a + o)};
          get_U(0, a, U[0]);
          get_U(1, a, U[1]);
          pin(vt, W[y]);
          slash_col(J[a], vt, r);
          if (o) {
#pragma unroll
            for (int m = 0; m < 4; ++m) r[m] = -r[m];
          }
          slash_col_add(e[x], W[y], r);
          clear4(rb);
          pin(r);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            adj_sdot(U[t], r, Ab[t], Ub[t], rb);
            pin(Ub[t], rb);
          }
          adj_slash_spinor(e[x], rb, Wb[y]);
          if (x == 2) adj_slash_vector(W[y], rb, eb);
#pragma unroll
          for (int m = 0; m < 4; ++m) sb[m] = o ? sb[m] - rb[m] : rb[m];
          pin(Wb[y], sb);
          if (x == 2) pin_eps(eb);
        }
        adj_slash_spinor(J[a], sb, vb);
        if (a < 2) adj_slash_vector(vt, sb, Jb[a]);
        pin(vb);
        if (a < 2) pin(Jb[a]);
        // on to the lanes that sum them
#pragma unroll
        for (int t = 0; t < 2; ++t)
          lds_put(lds + (a < 2 ? UB + 512 * a : FLOW) + 256 * t + lane, 64, Ub[t]);
      }
      __syncthreads();
      // U = d (q-slash + m) e-slash u, q = p(t) - k, of the lane's own version:
      // its adjoint is the sum over the lanes with the same gluon helicity
      const int b1 = own == 2 ? 4 : 2, b2 = own == 0 ? 4 : 8;
      const double last = own == 2 ? 1.0 : 0.0;  // gluon 2: its momentum and polarisation move
      auto own_adjoint = [&](const c64 (&f)[4], const double (&q)[4], const c64 (&ob)[4],
                             c64 (&fb)[4], double (&kb)[4]) {
        c64 s[4];
        slash_col(ea, f, s);
        adj_propagate(q, cp.mt, ig, own_factor(q), s, ob, fb, kb);
        c64 x[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) x[m] = last * fb[m];
        adj_slash_vector(f, x, eb);
      };
      {
        c64 sum[4], fb[4], fu[4];
        double q[4], pq[4], kb[4] = {0.0, 0.0, 0.0, 0.0};
        clear4(sum);
        const d2* from = lds + (own == 0 ? UB : own == 1 ? UB + 512 : FLOW) + 256 * tb;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          c64 x[4];
          lds_get(from + (lane ^ ((j & 1) | (j & 2 ? b1 : 0) | (j & 4 ? b2 : 0))), 64, x);
#pragma unroll
          for (int m = 0; m < 4; ++m) sum[m] = sum[m] + x[m];
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) sum[m] = spare ? c64{0.0, 0.0} : sum[m];
        momentum(lds, at, 0, pq);
        pin(sum, ut, ea, ka);
        minus4(pq, ka, q);
        own_adjoint(ut, q, sum, fb, kb);
        clear4(fu);
        adj_slash_spinor(ea, fb, fu);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          ub[0][m] = rmadd(tb ? 0.0 : 1.0, fu[m], ub[0][m]);
          ub[1][m] = rmadd(tb ? 1.0 : 0.0, fu[m], ub[1][m]);
          pb[2][m] += kb[m];
          k2b[m] = fmadd(-last, kb[m], k2b[m]);
        }
        pin(ub[0], ub[1], pb[2], k2b);
        pin_eps(eb);
      }
      __syncthreads();
#pragma unroll
      for (int a = 0; a < 3; ++a) lds_put(lds + UB + 256 * a + lane, 64, Wb[a]);
      __syncthreads();
      {
        c64 sum[4], fb[4];
        double q[4], pq[4], kb[4] = {0.0, 0.0, 0.0, 0.0};
        clear4(sum);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          c64 x[4];
          lds_get(lds + UB + 256 * own + (lane ^ ((j & 1 ? b1 : 0) | (j & 2 ? b2 : 0))), 64, x);
#pragma unroll
          for (int m = 0; m < 4; ++m) sum[m] = sum[m] + x[m];
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) sum[m] = spare ? c64{0.0, 0.0} : sum[m];
        momentum(lds, at, 1, pq);
        pin(sum, vt, ea, ka);
        minus4(ka, pq, q);
        own_adjoint(vt, q, sum, fb, kb);
        adj_slash_spinor(ea, fb, vb);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          pb[3][m] -= kb[m];
          k2b[m] = fmadd(last, kb[m], k2b[m]);
        }
        pin(vb, pb[3], k2b);
        pin_eps(eb);
      }
    double pt[4], pa[4], pg[4];
    momentum(lds, at, 1, pa);
    pin(pa, vb);
    qb.add(pa, cp.mt, true, tb, vb);
    qb.finish(pa, cp.mt, pb[3]);
    momentum(lds, at, 0, pt);
    pin(pt, ub[0], ub[1], pb[3]);
#pragma unroll
    for (int t = 0; t < 2; ++t) qt.add(pt, cp.mt, false, t, ub[t]);
    qt.finish(pt, cp.mt, pb[2]);
    pin(pb[2]);
#pragma unroll
    for (int c = 0; c < 2; ++c) {  // J[c] = -f[c] L(e[a], e[2]), a = 1 - c
      const int a = 1 - c;
      double K[4];
      c64 o[4];
      plus4(k[a], k[2], K);
      pin(K);
      const double f = cp.gs * recip(msq(K));
      add_msq_grad(K, -ig * f * cdot4(Jb[c], J[c]).r, k2b);
#pragma unroll
      for (int m = 0; m < 4; ++m) o[m] = -f * Jb[c][m];
      adj_three_gluon_y(e[a], k[a], e[2], k[2], o, eb, k2b);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) pb[4][m] -= k2b[m];
    momentum(lds, at, 2, pg);
    adj_polarisation(pg, lam2, eb, pb[4]);
    }
    return me;
  }
};

// buf: in the final-state momenta of each event (slot 4 l + mu of leg l + 2),
// out d(sum |M|^2)/dp as three-vectors (slot 3 l + mu - 1) and the sum (slot
// 3 NF), pages as the uniforms
template <class P, class Event>
__global__ void __launch_bounds__(64)
    momentum_gradient_kernel(double* buf, int64_t first, int64_t nevt, double half, uint64_t mask,
                             Couplings<double> c) {
  constexpr int NP = P::NPAR, NF = NP - 2, NR = 4 * NF, L = Event::LANES;
  __shared__ d2 lds[Event::LDS];
  const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int64_t i = first + j / L;
  if (i >= nevt) return;
  const int g = (int)(j % L);
  double p[NP][4];
#pragma unroll
  for (int l = 0; l < NF; ++l)
#pragma unroll
    for (int m = 0; m < 4; ++m) p[l + 2][m] = buf[aosoa_rnd(i, 4 * l + m, NR)];
  p[0][0] = half;
  p[1][0] = half;
  set_beams(p);
  double pb[NP][4];
#pragma unroll
  for (int l = 0; l < NP; ++l)
#pragma unroll
    for (int m = 0; m < 4; ++m) pb[l][m] = 0.0;
  const double me = lanes_sum<L>(Event(p, c).gradient(p, g, mask, lds, pb));
#pragma unroll
  for (int l = 0; l < NF; ++l) {
    // dE = p.dp / E on the mass shell
    if constexpr (L == 16) {
      int at = Event::EVENT + 6 * (threadIdx.x / L);
      Event::momentum(lds, at, l, p[l + 2]);
    }
    const double e = lanes_sum<L>(pb[l + 2][0]) * recip(p[l + 2][0]);
#pragma unroll
    for (int m = 1; m < 4; ++m) {
      const double s = fmadd(e, p[l + 2][m], lanes_sum<L>(pb[l + 2][m]));
      if (g == 0) buf[aosoa_rnd(i, 3 * l + m - 1, NR)] = s;
    }
  }
  if (g == 0) buf[aosoa_rnd(i, 3 * NF, NR)] = me;
}

// whether the gradient pages of nevt events overlap the uniforms or gbar
inline bool grad_in_place(const double* rnd, const double* gbar, const double* grad, int64_t nevt,
                          int nrnd) {
  const int64_t n = (nevt + NEPPR - 1) / NEPPR * NEPPR * nrnd;
  auto meet = [&](const double* x, int64_t m) {
    return x && (uintptr_t)x < (uintptr_t)(grad + n) && (uintptr_t)grad < (uintptr_t)(x + m);
  };
  return meet(rnd, n) || meet(gbar, nevt);
}

template <class P, class Event>
int shared_gradient_launch(const MeArgs& a, const RamboArgs& ra, const double* rnd, int64_t nevt,
                           const double* gbar, double* grad_rnd, double* grad_logw, double* f,
                           hipStream_t s) {
  constexpr int NF = P::NPAR - 2;
  const int64_t per = 64 / Event::LANES;
  launch_grad_momenta(NF, rnd, nevt, ra, grad_rnd, s);
  for (int64_t i = 0; i < nevt; i += launch_events(Event::LANES)) {
    const int64_t n = std::min(nevt - i, launch_events(Event::LANES));
    momentum_gradient_kernel<P, Event><<<(unsigned)((n + per - 1) / per), 64, 0, s>>>(
        grad_rnd, i, nevt, 0.5 * ra.sqrts, helicity_mask(a.hel), a.c64);
  }
  launch_grad_uniforms(NF, rnd, nevt, ra, a.inv_iden, gbar, grad_rnd, grad_logw, f, s);
  return 0;
}

}  // namespace mg
