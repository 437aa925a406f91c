// g g -> t t~ + gluons with every current shared by the helicities that do
// not distinguish it.
//
// A current of k external legs has 2^k helicity versions, not 2^npar: the
// kernels built on this header compute each version once per event and
// assemble the colour flows of a helicity from them, instead of running all
// the currents of all the diagrams for every helicity.  The diagrams of a
// colour flow are summed inside the currents (Berends-Giele recursion), with
// the Feynman rules, couplings and propagators of helas.h:
//
//   J(a)       polarisation vector of gluon a
//   J(w)       = g/K^2 [ -sum_{w = xy} L(J(x), J(y)) + g sum_{w = xyz} Q(J(x), J(y), J(z)) ]
//   L(x, y)    = x (-(2 kx + ky).y) + (x.y) (kx - ky) + y ((kx + 2 ky).x)
//   Q(x, y, z) = 2 y (x.z) - x (y.z) - z (x.y)
//   U(w)       = -g sum_{w = xy} U(x) J-slash(y) (q-slash + m) / D      t line from the t end
//   W(w)       = -g sum_{w = xy} (q-slash + m) / D J-slash(x) W(y)      and from the t~ end
//
// J(w) with w = (word of gluons) is the coefficient of the string of SU(3)
// generators T^w in the current.  J(ab) = -J(ba); the six orderings of three
// gluons have one value per middle gluon, and the three sum to zero; a
// four-gluon current changes sign under reversal.
//
// Row spinors f of the t side are kept as columns (f1, -f0, f3, -f2), on
// which f V-slash acts as V-slash on a column, so that both ends of the line
// run through the same code.
#pragma once
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace mg {

typedef double d2 __attribute__((ext_vector_type(2)));  // one complex in LDS: 16-byte accesses
typedef cx<double> c64;

// four components of version v of an object whose components are `n` apart
// (component-major: the versions that the lanes of a wave read lie next to
// each other, so a read is free of bank conflicts)
__device__ __forceinline__ void lds_get(const d2* p, int n, c64 (&w)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const d2 t = p[k * n];
    w[k] = c64{t.x, t.y};
  }
}
__device__ __forceinline__ void lds_put(d2* p, int n, const c64 (&w)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) p[k * n] = d2{w[k].r, w[k].i};
}
// polarisation vector: no time component, real z component (ext_vector)
__device__ __forceinline__ void lds_get_eps(const d2* p, c64 (&w)[4]) {
  const d2 a = p[8], b = p[16];
  w[0] = c64{0.0, 0.0};
  w[1] = c64{a.x, a.y};
  w[2] = c64{b.x, b.y};
  w[3] = c64{p[24].x, 0.0};
}
__device__ __forceinline__ c64 lds_scalar(const d2* p) {
  const d2 t = *p;
  return c64{t.x, t.y};
}
__device__ __forceinline__ void lds_get_real(const d2* p, double (&k)[4]) {
  const d2 a = p[0], b = p[1];
  k[0] = a.x;
  k[1] = a.y;
  k[2] = b.x;
  k[3] = b.y;
}

// acc + a.b (Minkowski)
__device__ __forceinline__ c64 mdot_add(const c64 (&a)[4], const c64 (&b)[4], c64 acc) {
  return cmsub(a[3], b[3], cmsub(a[2], b[2], cmsub(a[1], b[1], cmadd(a[0], b[0], acc))));
}
__device__ __forceinline__ c64 mdot0(const c64 (&a)[4], const c64 (&b)[4]) {
  return cmsub(a[3], b[3], cmsub(a[2], b[2], cmsub(a[1], b[1], a[0] * b[0])));
}
// acc + (row spinor kept as column u) times column w
__device__ __forceinline__ c64 sdot_add(const c64 (&u)[4], const c64 (&w)[4], c64 acc) {
  return cmsub(u[3], w[2], cmadd(u[2], w[3], cmsub(u[1], w[0], cmadd(u[0], w[1], acc))));
}
// F gamma^mu G for the row spinor F kept as column u
__device__ __forceinline__ void bilinear(const c64 (&u)[4], const c64 (&G)[4], c64 (&J)[4]) {
  const c64 F[4] = {-u[1], u[0], -u[3], u[2]};
  ffv_bilinear_v<double>(F, G, J);
}
// V-slash acting on a column
__device__ __forceinline__ void slash_col(const c64 (&V)[4], const c64 (&G)[4], c64 (&f)[4]) {
  blk<double> s, sb;
  slash_blocks(V, s, sb);
  mcol(s, G[2], G[3], f[0], f[1]);
  mcol(sb, G[0], G[1], f[2], f[3]);
}
__device__ __forceinline__ void slash_col_add(const c64 (&V)[4], const c64 (&G)[4], c64 (&f)[4]) {
  blk<double> s, sb;
  slash_blocks(V, s, sb);
  f[0] = cmadd(s.a, G[2], cmadd(s.b, G[3], f[0]));
  f[1] = cmadd(s.c, G[2], cmadd(s.d, G[3], f[1]));
  f[2] = cmadd(sb.a, G[0], cmadd(sb.b, G[1], f[2]));
  f[3] = cmadd(sb.c, G[0], cmadd(sb.d, G[1], f[3]));
}
// d (q-slash + m) f
__device__ __forceinline__ void propagate(const double (&q)[4], double m, c64 d, const c64 (&f)[4],
                                          c64 (&out)[4]) {
  c64 y0, y1, y2, y3;
  sK_col(q, f[2], f[3], y0, y1);
  sbK_col(q, f[0], f[1], y2, y3);
  out[0] = d * rmadd(m, f[0], y0);
  out[1] = d * rmadd(m, f[1], y1);
  out[2] = d * rmadd(m, f[2], y2);
  out[3] = d * rmadd(m, f[3], y3);
}
// L(x, y) of the three-gluon vertex
__device__ __forceinline__ void three_gluon(const c64 (&x)[4], const double (&kx)[4],
                                            const c64 (&y)[4], const double (&ky)[4],
                                            c64 (&out)[4]) {
  double qx[4], qy[4], dk[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    qx[m] = -(2.0 * kx[m] + ky[m]);
    qy[m] = kx[m] + 2.0 * ky[m];
    dk[m] = kx[m] - ky[m];
  }
  const c64 cx_ = mdot(qx, y), cy_ = mdot(qy, x), xy = mdot0(x, y);
#pragma unroll
  for (int m = 0; m < 4; ++m) out[m] = rmadd(dk[m], xy, cmadd(y[m], cy_, x[m] * cx_));
}

// Sum over the 64 lanes, in every lane, without LDS: exchanges inside quads
// and rows of 16 by DPP, then of 16- and 32-lane halves.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const unsigned lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xF, 0xF, true);
  const unsigned hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move<0xB1>(v);   // quad_perm 1 0 3 2
  v += dpp_move<0x4E>(v);   // quad_perm 2 3 0 1
  v += dpp_move<0x141>(v);  // row_half_mirror
  v += dpp_move<0x140>(v);  // row_mirror
  unsigned lo, hi;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    lo = (unsigned)b;
    hi = (unsigned)(b >> 32);
    // swap(x, x) returns (x of the lower halves in both, x of the upper ones)
    const auto rl = k ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                      : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto rh = k ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                      : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = __builtin_bit_cast(double, (uint64_t)rl[0] | ((uint64_t)rh[0] << 32)) +
        __builtin_bit_cast(double, (uint64_t)rl[1] | ((uint64_t)rh[1] << 32));
  }
  return v;
}

// 1 / sqrt(x), x > 0: the hardware estimate and two Newton steps (within an
// ulp or two)
__device__ __forceinline__ double rsqrt_refined(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double e = fmadd(-x * y, y, 1.0);
    y = fmadd(0.5 * y, e, y);
  }
  return y;
}

// sqrt(x) from y = rsqrt_refined(x), x > 0: x y corrected by its residual, so
// that it rounds as the square root does (x y alone is off by up to 1.5 ulp).
// rms error of 65536 matrix elements of e+ e- -> mu+ mu- at 1500 GeV against 80
// bits 3.5e-16, and 4.0e-16 with one amplitude per helicity (against 64 bits 5.7e-16
// and 5.5e-16: most of that is the rounding of the 64-bit evaluation, which
// rounds like the latter)
__device__ __forceinline__ double sqrt_refined(double x, double y) {
  const double s = x * y;
  return fmadd(0.5 * y, fmadd(-s, s, x), s);
}

// External wavefunctions of helas.h (ext_vector; ext_u barred, mapped to a
// column; ext_v), in one body for lanes that hold different legs: the roots
// and reciprocals that both kinds need are formed once, from reciprocal
// square roots.
__device__ __forceinline__ void external(const double (&p)[4], double m, int lam, bool gluon,
                                         bool flag, c64 (&w)[4]) {
  const double pt2 = p[1] * p[1] + p[2] * p[2];
  const double P2 = pt2 + p[3] * p[3];
  const double iP = rsqrt_refined(P2);
  const double P = P2 > 0.0 ? sqrt_refined(P2, iP) : 0.0;
  const double epp = p[0] + P;
  const double x = gluon ? (pt2 > 0.0 ? pt2 : 1.0) : epp;
  const double ix = rsqrt_refined(x);
  if (gluon) {  // flag: outgoing
    const double r2 = 0.70710678118654752440;
    const double a = -lam * r2, b = flag ? r2 : -r2;
    const double cph = pt2 > 0.0 ? p[1] * ix : 1.0, sph = pt2 > 0.0 ? p[2] * ix : 0.0;
    const double kt = pt2 * ix;
    const double cth = p[3] * iP;
    w[0] = c64{0.0, 0.0};
    w[1] = c64{a * cth * cph, -b * sph};
    w[2] = c64{a * cth * sph, b * cph};
    w[3] = c64{-a * (kt * iP), 0.0};
  } else {      // flag: the t~
    const double big = sqrt_refined(epp, ix), small = m * ix;  // sqrt(E + P), sqrt(E - P)
    const double ppz = p[3] >= 0.0 ? P + p[3] : pt2 * recip(P - p[3]);
    const bool back = !(ppz > 0.0);
    const double nrm = rsqrt_refined(back ? 1.0 : 2.0 * P * ppz);
    // chi+ = (c, x + i y), chi- = (-x + i y, c); along -z (0, 1), (-1, 0)
    const double c = back ? 0.0 : ppz * nrm;
    const double cx_ = back ? 1.0 : p[1] * nrm, cy_ = back ? 0.0 : p[2] * nrm;
    const bool up = (lam > 0) != flag;  // the t~ has the spinor of the opposite helicity
    const c64 c0 = up ? c64{c, 0.0} : c64{-cx_, cy_}, c1 = up ? c64{cx_, cy_} : c64{c, 0.0};
    const double wp = lam > 0 ? big : small, wm = lam > 0 ? small : big;
    const c64 a0 = wp * c0, a1 = wp * c1, b0 = wm * c0, b1 = wm * c1;
    if (flag) {  // (wp chi, -wm chi)
      w[0] = a0;
      w[1] = a1;
      w[2] = -b0;
      w[3] = -b1;
    } else {     // row (wp chi^+, wm chi^+) as the column (f1, -f0, f3, -f2)
      w[0] = conj(a1);
      w[1] = -conj(a0);
      w[2] = conj(b1);
      w[3] = -conj(b0);
    }
  }
}

// ---------------------------------------------------------------------------
// g g -> t t~ g g: one event per wave
// ---------------------------------------------------------------------------
// Gluons 0..3 = legs 0, 1, 4, 5; colour flows = orderings of the gluons in
// lexicographic order.  With the quark line cut between its second and third
// gluon, the flow (a b c d) is
//   A = g [ U(ab).(c-slash W(d) + J-slash(cd) v) + J(bc).G(a, d)
//         + J(bcd).Y(a) + J(abc).Z(d) + g/K^2 (-P(ab|cd) + g quartic) ]
//   G(a, d) = U(a) gamma W(d)
//   Y(a) = U(a) gamma v + (g/K^2) X(a),  Z(d) = u gamma W(d) - (g/K^2) X(d)
//   B = u gamma v,  X(a) = L(a, B),  P(ab|cd) = L(J(ab), J(cd)).B
// (K the momentum of all four gluons; the three-gluon vertex is
// antisymmetric in its three legs, so L(J(abc), d).B = J(abc).L(d, B)).
//
// The currents are built by the lanes side by side (a lane per current and
// helicity version) and handed on through LDS; then lane h assembles the 24
// flows of helicity h.  Bound: LDS bandwidth (515 accesses of 16 bytes a lane
// at 128 bytes/clock: 4.1e3 of the 4.3e3 clocks per event and CU) close to the
// FP64 VALU (3.3e3 instructions per event; 18.3e3 with one full amplitude per
// lane).  Two waves per SIMD: 232 registers, 18 KB of LDS a wave.  2^19 events
// in 3.71 ms, 141 M events/s (19.05 ms with one full amplitude per lane; 4.40
// before the block-form colour sum, the external wavefunctions from refined
// reciprocal roots and the DPP helicity sum).
namespace ggttgg_shared {

// LDS in units of one complex (16 bytes); versions are bit fields of the
// helicities in the order named, lowest bit first
constexpr int EPS = 0;             // [4][8]   2 g + h
constexpr int QV = EPS + 32;       // [4][4]   2 side + h (side 0: t, 1: t~)
constexpr int KV = QV + 16;        // [32][2]  momenta, see momentum slots below
constexpr int PR = KV + 64;        // [32]     propagator factors of the slots
constexpr int J2 = PR + 32;        // [4][24]  pair * 4 + (a, b)
constexpr int U1 = J2 + 96;        // [4][32]  side * 16 + g * 4 + (quark, g)
constexpr int BB = U1 + 128;       // [4][4]   (t, t~)
constexpr int R = BB + 16;         // reused by the stages
//   stage 1
constexpr int NN = R;              // [4][48]  g/K^2 L(J(ab), J(cd))  pairing * 16 + (0, 1, 2, 3)
constexpr int JB = NN + 192;       // [96]     g^2/K^2 J(ab).B  pair * 16 + (t, t~, a, b)
constexpr int CB = JB + 96;        // [32]     g^2/K^2 c.B     g * 8 + (t, t~, c)
constexpr int JC = CB + 32;        // [96]     J(ab).c   (pair * 2 + which c) * 8 + (a, b, c)
constexpr int CD = JC + 96;        // [24]     c.d       pair * 4 + (c, d)
constexpr int END1 = CD + 24;
//   stage 2
constexpr int J3 = R;              // [4][64]  (missing g * 2 + middle) * 8 + (a, b, c)
constexpr int YZ = J3 + 256;       // [4][64]  side * 32 + g * 8 + (t, t~, g)
constexpr int END2 = YZ + 256;
//   stage 3: G(a, d), four ordered pairs at a time
constexpr int GG = R;              // [4][64]  ordered pair * 16 + (t, t~, a, b), a < b
//   stage 4
constexpr int U2 = R;              // [4][96]  (pair * 2 + order) * 8 + (t, a, b)
constexpr int W2 = U2 + 384;       // [4][96]  (pair * 2 + order) * 8 + (t~, a, b)
constexpr int END4 = W2 + 384;
constexpr int MAX(int a, int b) { return a > b ? a : b; }
constexpr int LDS_UNITS = MAX(MAX(END1, END2), END4);

// momentum slots: incoming momenta of gluon sets, and the momenta q along
// the quark line of its propagators
constexpr int K_ONE = 0;    // + g
constexpr int K_U1 = 4;     // + g
constexpr int K_W1 = 8;     // + g
constexpr int K_THREE = 12; // + g missing
constexpr int K_TWO = 16;   // + pair
constexpr int K_FOUR = 22;
constexpr int K_U2 = 24;    // + pair

// pairs (01) (02) (03) (12) (13) (23)
__host__ __device__ constexpr int pair_of(int a, int b) {
  const int lo = a < b ? a : b, hi = a < b ? b : a;
  return lo == 0 ? hi - 1 : (lo == 1 ? hi + 1 : 5);
}
// the same for a pair index that differs by lane
__device__ __forceinline__ int pair_lo(int p) { return (0x940 >> (2 * p)) & 3; }
__device__ __forceinline__ int pair_hi(int p) { return (0xFB9 >> (2 * p)) & 3; }
// k-th (0, 1, 2) of the gluons other than g
__host__ __device__ constexpr int other3(int g, int k) { return k + (k >= g ? 1 : 0); }
// rank of the ordering (a b c d) in lexicographic order
__host__ __device__ constexpr int flow(int a, int b, int c, int d) {
  return 6 * a + 2 * (b - (b > a)) + (c > d);
}

struct Helicity {  // helicity bits (0 / 1) of a lane
  int t, tb, g[4];
};

// The flows as they are now: what has been added to them is not put off past
// this point (the compiler would otherwise carry the operands along and spill
// them).
__device__ __forceinline__ void settle(c64 (&A)[24]) {
#pragma unroll
  for (int k = 0; k < 24; ++k) {
    opaque(A[k].r);
    opaque(A[k].i);
  }
}

// Colour flows A / g of event i (the same in every lane) for the helicity
// code of the lane; every lane of the wave takes part.
template <class P>
__device__ __forceinline__ void flows(const double* __restrict__ mom, int64_t i,
                                      const Couplings<double>& cp, d2* lds, int lane,
                                      c64 (&A)[24]) {
  // ---- momenta, propagators, external wavefunctions --------------------
  double p[6][4];
  load_event<P>(mom, i, p);
  // lanes 0..7: gluons, 8..11: t and t~, each with both helicities
  const int leg = lane < 4 ? lane >> 1 : (lane < 8 ? 2 + (lane >> 1) : (lane < 10 ? 2 : 3));
  double q[4];
  if (lane < 12) {
#pragma unroll
    for (int m = 0; m < 4; ++m) q[m] = mom[aosoa_mom(i, 0, m, 6) + leg * 4 * NEPPM];
  }
  if (lane < 32) {
    const int g = lane & 3, e = lane & 7;
    const int gm = lane < 12 ? 1 << g : (lane < 16 ? 15 ^ (1 << g) : (0x0FCA6953 >> (4 * e)) & 15);
    const bool top = (lane >= K_U1 && lane < K_W1) || lane >= K_U2;
    const bool atop = lane >= K_W1 && lane < K_THREE;
    const double c0 = gm & 1, c1 = (gm >> 1) & 1, c4 = -((gm >> 2) & 1), c5 = -((gm >> 3) & 1);
    const double ct = top ? -1.0 : 0.0, ctb = atop ? -1.0 : 0.0;
    double K[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
      K[m] = fmadd(c5, p[5][m], fmadd(c4, p[4][m], fmadd(ctb, p[3][m],
             fmadd(ct, p[2][m], fmadd(c1, p[1][m], c0 * p[0][m])))));
    const bool quark = top || atop;
    const double wid = ((gm ^ (gm >> 1)) & 1) ? cp.wtt : cp.wt;
    const double k2 = msq(K);
    const double re = k2 - cp.mt * cp.mt, im = cp.mt * wid;
    const double n = recip(quark ? re * re + im * im : k2);
    // vectors: g / K^2; quarks: -g / (q^2 - m^2 + i m w)
    const c64 pr = quark ? c64{-cp.gs * (re * n), cp.gs * (im * n)} : c64{cp.gs * n, 0.0};
    const double s = top ? -1.0 : 1.0;  // q of the t side runs against K
    lds[KV + 2 * lane] = d2{s * K[0], s * K[1]};
    lds[KV + 2 * lane + 1] = d2{s * K[2], s * K[3]};
    lds[PR + lane] = d2{pr.r, pr.i};
  }
  if (lane < 12) {
    const int lam = (lane & 1) ? 1 : -1;
    c64 w[4];
    external(q, cp.mt, lam, lane < 8, lane < 8 ? leg > 1 : leg == 3, w);
    lds_put(lds + (lane < 8 ? EPS + lane : QV + lane - 8), lane < 8 ? 8 : 4, w);
  }
  __syncthreads();
  // ---- J(ab), U(a) and W(a), B -----------------------------------------
  if (lane < 24) {
    const int pr = lane >> 2, a = pair_lo(pr), b = pair_hi(pr);
    c64 x[4], y[4], o[4];
    double kx[4], ky[4];
    lds_get_eps(lds + EPS + 2 * a + (lane & 1), x);
    lds_get_eps(lds + EPS + 2 * b + ((lane >> 1) & 1), y);
    lds_get_real(lds + KV + 2 * (K_ONE + a), kx);
    lds_get_real(lds + KV + 2 * (K_ONE + b), ky);
    three_gluon(x, kx, y, ky, o);
    const double f = -lds[PR + K_TWO + pr].x;
#pragma unroll
    for (int m = 0; m < 4; ++m) o[m] = f * o[m];
    lds_put(lds + J2 + lane, 24, o);
  }
  if (lane < 32) {
    const int side = lane >> 4, g = (lane >> 2) & 3;
    c64 V[4], f[4], s[4], o[4];
    double q[4];
    lds_get(lds + QV + 2 * side + (lane & 1), 4, s);
    lds_get_eps(lds + EPS + 2 * g + ((lane >> 1) & 1), V);
    const int k = (side ? K_W1 : K_U1) + g;
    lds_get_real(lds + KV + 2 * k, q);
    slash_col(V, s, f);
    propagate(q, cp.mt, lds_scalar(lds + PR + k), f, o);
    lds_put(lds + U1 + lane, 32, o);
  } else if (lane < 36) {
    c64 u[4], v[4], o[4];
    lds_get(lds + QV + (lane & 1), 4, u);
    lds_get(lds + QV + 2 + ((lane >> 1) & 1), 4, v);
    bilinear(u, v, o);
    lds_put(lds + BB + lane - 32, 4, o);
  }
  __syncthreads();

  const Helicity h{(lane >> 3) & 1, (lane >> 2) & 1,
                   {(lane >> 5) & 1, (lane >> 4) & 1, (lane >> 1) & 1, lane & 1}};
  const int htt = h.t | (h.tb << 1);
  const double k4 = lds[PR + K_FOUR].x;  // g / K^2 of all four gluons

  // ---- stage 2: three-gluon currents -----------------------------------
  {
    // J(x m y) of the triple without gluon g, m its smallest or second gluon
    const int g = lane >> 4, mid = (lane >> 3) & 1;
    const int i0 = (g == 0), i1 = 1 + (g <= 1), i2 = 2 + (g <= 2);
    const int h0 = lane & 1, h1 = (lane >> 1) & 1, h2 = (lane >> 2) & 1;
    const int x = mid ? i0 : i1, m = mid ? i1 : i0, hx = mid ? h0 : h1, hm = mid ? h1 : h0;
    c64 ex[4], em[4], ey[4], jxm[4], jmy[4], o1[4], o2[4];
    double kx[4], ky[4], kxm[4], kmy[4];
    lds_get_eps(lds + EPS + 2 * x + hx, ex);
    lds_get_eps(lds + EPS + 2 * m + hm, em);
    lds_get_eps(lds + EPS + 2 * i2 + h2, ey);
    const int p01 = i0 == 0 ? i1 - 1 : 3;               // pair (i0 i1): (01) (02) (12)
    const int pm2 = m == 0 ? i2 - 1 : (m == 1 ? i2 + 1 : 5);
    lds_get(lds + J2 + 4 * p01 + h0 + 2 * h1, 24, jxm);  // J(i0 i1) = -J(x m) when m = i0
    lds_get(lds + J2 + 4 * pm2 + hm + 2 * h2, 24, jmy);
    lds_get_real(lds + KV + 2 * (K_ONE + x), kx);
    lds_get_real(lds + KV + 2 * (K_ONE + i2), ky);
    lds_get_real(lds + KV + 2 * (K_TWO + p01), kxm);
    lds_get_real(lds + KV + 2 * (K_TWO + pm2), kmy);
    three_gluon(jxm, kxm, ey, ky, o1);
    three_gluon(ex, kx, jmy, kmy, o2);
    const double s1 = mid ? -1.0 : 1.0;  // -L(J(xm), y) with the sign of J(xm)
    const c64 xz = cp.gs * mdot0(ex, ey), yz = cp.gs * mdot0(em, ey), xy = cp.gs * mdot0(ex, em);
    const double f = lds[PR + K_THREE + g].x;
    c64 o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      c64 t = rmadd(s1, o1[k], -o2[k]);
      t = cmadd(2.0 * em[k], xz, t);
      t = cmsub(ex[k], yz, t);
      o[k] = f * cmsub(ey[k], xy, t);
    }
    lds_put(lds + J3 + lane, 64, o);
  }
  {
    // Y(g) and Z(g)
    const int side = lane >> 5, g = (lane >> 3) & 3, ht = lane & 1, hb = (lane >> 1) & 1,
              hg = (lane >> 2) & 1;
    c64 u[4], v[4], e[4], B[4], X[4], o[4];
    double kg[4], kb[4];
    // side 0: U(g) gamma v; side 1: u gamma W(g)
    lds_get(lds + (side ? QV + ht : U1 + 4 * g + ht + 2 * hg), side ? 4 : 32, u);
    lds_get(lds + (side ? U1 + 16 + 4 * g + hb + 2 * hg : QV + 2 + hb), side ? 32 : 4, v);
    lds_get_eps(lds + EPS + 2 * g + hg, e);
    lds_get(lds + BB + ht + 2 * hb, 4, B);
    lds_get_real(lds + KV + 2 * (K_ONE + g), kg);
    lds_get_real(lds + KV + 2 * K_FOUR, kb);
#pragma unroll
    for (int m = 0; m < 4; ++m) kb[m] = -kb[m];
    bilinear(u, v, o);
    three_gluon(e, kg, B, kb, X);
    const double s = side ? -k4 : k4;
#pragma unroll
    for (int m = 0; m < 4; ++m) o[m] = rmadd(s, X[m], o[m]);
    lds_put(lds + YZ + lane, 64, o);
  }
  __syncthreads();
  c64 zero{0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 24; ++k) A[k] = zero;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int i0 = other3(g, 0), i1 = other3(g, 1), i2 = other3(g, 2);
    const int v3 = h.g[i0] | (h.g[i1] << 1) | (h.g[i2] << 2);
    c64 y[4], z[4], ym[3], zm[3];
    lds_get(lds + YZ + 8 * g + htt + 4 * h.g[g], 64, y);
    lds_get(lds + YZ + 32 + 8 * g + htt + 4 * h.g[g], 64, z);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      c64 j[4];
      lds_get(lds + J3 + (2 * g + k) * 8 + v3, 64, j);
      ym[k] = mdot0(j, y);
      zm[k] = mdot0(j, z);
    }
    ym[2] = -(ym[0] + ym[1]);
    zm[2] = -(zm[0] + zm[1]);
    // flows (g x m y) and (x m y g), m the k-th gluon of the triple
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int m = other3(g, k), x = other3(g, k == 0 ? 1 : 0), y_ = other3(g, k == 2 ? 1 : 2);
      A[flow(g, x, m, y_)] = A[flow(g, x, m, y_)] + ym[k];
      A[flow(g, y_, m, x)] = A[flow(g, y_, m, x)] + ym[k];
      A[flow(x, m, y_, g)] = A[flow(x, m, y_, g)] + zm[k];
      A[flow(y_, m, x, g)] = A[flow(y_, m, x, g)] + zm[k];
    }
  }
  settle(A);
  __syncthreads();
  // ---- stage 1: diagrams whose quark line carries one four-gluon current,
  // but for those counted in Y and Z
  if (lane < 48) {
    const int k = lane >> 4;  // pairing (01|23) (02|13) (03|12) = pairs (k | 5 - k)
    const int a = pair_lo(k), b = pair_hi(k), c = pair_lo(5 - k), d = pair_hi(5 - k);
    c64 x[4], y[4], o[4];
    double kx[4], ky[4];
    lds_get(lds + J2 + 4 * k + ((lane >> a) & 1) + 2 * ((lane >> b) & 1), 24, x);
    lds_get(lds + J2 + 4 * (5 - k) + ((lane >> c) & 1) + 2 * ((lane >> d) & 1), 24, y);
    lds_get_real(lds + KV + 2 * (K_TWO + k), kx);
    lds_get_real(lds + KV + 2 * (K_TWO + 5 - k), ky);
    three_gluon(x, kx, y, ky, o);
#pragma unroll
    for (int m = 0; m < 4; ++m) o[m] = k4 * o[m];
    lds_put(lds + NN + lane, 48, o);
  }
  // scalar products of the quartic vertices, 64 at a time: J(ab).B of the
  // pairs 0..3; of the pairs 4, 5 and c.B; J(ab).c of the pairs 0..3; of the
  // pairs 4, 5 and c.d
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int l = lane & 31, hi = lane >> 5;
    int xa, xn = 24, ya, yn;
    if (i < 2) {
      const int pr = lane >> 4, xj = J2 + 4 * pr + ((lane >> 2) & 3);
      xa = i == 0 ? xj : (hi ? EPS + 2 * (l >> 3) + ((l >> 2) & 1) : xj + 16);
      if (i == 1) xn = hi ? 8 : 24;
      ya = BB + (lane & 3);
      yn = 4;
    } else {
      const int pr = i == 2 ? lane >> 4 : 4 + (l >> 4), cd = l >> 2;
      const int c = (lane >> 3) & 1 ? pair_hi(5 - pr) : pair_lo(5 - pr);
      xa = J2 + 4 * pr + (lane & 3);
      ya = EPS + 2 * c + ((lane >> 2) & 1);
      yn = 8;
      if (i == 3) {
        xa = hi ? EPS + 2 * pair_lo(cd) + (l & 1) : xa;
        ya = hi ? EPS + 2 * pair_hi(cd) + ((l >> 1) & 1) : ya;
        xn = hi ? 8 : 24;
      }
    }
    c64 x[4], y[4];
    lds_get(lds + xa, xn, x);
    lds_get(lds + ya, yn, y);
    // the products with B carry the factor g^2 / K^2
    const c64 s = (i < 2 ? cp.gs * k4 : 1.0) * mdot0(x, y);
    if (i < 3 || lane < 56) lds[JB + lane + 64 * i] = d2{s.r, s.i};
  }
  __syncthreads();
  {
    c64 B[4], N[3], H[6][3];
    lds_get(lds + BB + htt, 4, B);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      c64 n[4];
      lds_get(lds + NN + 16 * k + (h.g[0] | (h.g[1] << 1) | (h.g[2] << 2) | (h.g[3] << 3)), 48, n);
      N[k] = mdot0(n, B);
    }
    // H[pair][k]: quartic vertices of {J(ab), c, d} and B with J(ab) (k = 0),
    // c (1), d (2) in the middle
#pragma unroll
    for (int pr = 0; pr < 6; ++pr) {
      constexpr int LO[6] = {0, 0, 0, 1, 1, 2}, HI[6] = {1, 2, 3, 2, 3, 3};
      const int a = LO[pr], b = HI[pr], c = LO[5 - pr], d = HI[5 - pr];
      const int hab = h.g[a] | (h.g[b] << 1);
      const c64 q = lds_scalar(lds + JB + 16 * pr + htt + 4 * hab) *
                    lds_scalar(lds + CD + 4 * (5 - pr) + (h.g[c] | (h.g[d] << 1)));
      const c64 rc = lds_scalar(lds + CB + 8 * c + htt + 4 * h.g[c]) *
                     lds_scalar(lds + JC + (2 * pr + 1) * 8 + hab + 4 * h.g[d]);
      const c64 rd = lds_scalar(lds + CB + 8 * d + htt + 4 * h.g[d]) *
                     lds_scalar(lds + JC + (2 * pr) * 8 + hab + 4 * h.g[c]);
      const c64 s = q + rc + rd;
      H[pr][0] = rmsub(-3.0, q, -s);
      H[pr][1] = rmsub(-3.0, rc, -s);
      H[pr][2] = rmsub(-3.0, rd, -s);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int d = a + 1; d < 4; ++d)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (b != a && b != d) {
            const int c = 6 - a - b - d;
            auto sgn = [](int x, int y) { return x < y ? 1.0 : -1.0; };
            // P(ab|cd): pairing of gluon 0, antisymmetric in each pair and in the two
            const int k = pair_of(0, a == 0 ? b : (b == 0 ? a : (c == 0 ? d : c)));
            const double sp = sgn(a, b) * sgn(c, d) * ((a == 0 || b == 0) ? 1.0 : -1.0);
            // middle of V(J(ab), c, d) is c, of V(a, J(bc), d) the current, of V(a, b, J(cd)) b
            const c64 q1 = sgn(a, b) * H[pair_of(a, b)][c < d ? 1 : 2];
            const c64 q2 = sgn(b, c) * H[pair_of(b, c)][0];
            const c64 q3 = sgn(c, d) * H[pair_of(c, d)][b > a ? 2 : 1];
            const c64 e = q1 + q2 + (q3 - sp * N[k]);
            A[flow(a, b, c, d)] = A[flow(a, b, c, d)] + e;
            A[flow(d, c, b, a)] = A[flow(d, c, b, a)] - e;
          }
  }
  settle(A);
  __syncthreads();

  // ---- stage 3: J(bc).G(a, d) ------------------------------------------
#pragma unroll
  for (int i = 0; i < 3; ++i) {  // pairs 2 i and 2 i + 1, both orders
    settle(A);
    __syncthreads();
    {
      const int o = lane >> 4, pr = 2 * i + (o >> 1), v = lane & 15;
      const int a = (o & 1) ? pair_hi(pr) : pair_lo(pr), d = (o & 1) ? pair_lo(pr) : pair_hi(pr);
      const int ha = (o & 1) ? (v >> 3) & 1 : (v >> 2) & 1, hd = (o & 1) ? (v >> 2) & 1 : (v >> 3) & 1;
      c64 u[4], w[4], J[4];
      lds_get(lds + U1 + 4 * a + (v & 1) + 2 * ha, 32, u);
      lds_get(lds + U1 + 16 + 4 * d + ((v >> 1) & 1) + 2 * hd, 32, w);
      bilinear(u, w, J);
      lds_put(lds + GG + lane, 64, J);
    }
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      constexpr int LO[6] = {0, 0, 0, 1, 1, 2}, HI[6] = {1, 2, 3, 2, 3, 3};
      const int pr = 2 * i + (o >> 1);
      const int a = (o & 1) ? HI[pr] : LO[pr], d = (o & 1) ? LO[pr] : HI[pr];
      const int b = LO[5 - pr], c = HI[5 - pr];
      c64 J[4], G[4];
      lds_get(lds + J2 + 4 * (5 - pr) + h.g[b] + 2 * h.g[c], 24, J);
      lds_get(lds + GG + 16 * o + htt + 4 * h.g[LO[pr]] + 8 * h.g[HI[pr]], 64, G);
      const c64 s = mdot0(J, G);
      A[flow(a, b, c, d)] = A[flow(a, b, c, d)] + s;
      A[flow(a, c, b, d)] = A[flow(a, c, b, d)] - s;
    }
  }
  settle(A);
  __syncthreads();
  // ---- stage 4: U(ab).W(cd) --------------------------------------------
  if (lane < 48) {
    const int pr = lane >> 3, a = pair_lo(pr), b = pair_hi(pr);
    const int hq = lane & 1, ha = (lane >> 1) & 1, hb = (lane >> 2) & 1;
    c64 ea[4], eb[4], j[4];
    lds_get_eps(lds + EPS + 2 * a + ha, ea);
    lds_get_eps(lds + EPS + 2 * b + hb, eb);
    lds_get(lds + J2 + 4 * pr + ha + 2 * hb, 24, j);
    {
      c64 s0[4], s1[4], f[4], fab[4], fba[4], o[4];
      double q[4];
      lds_get(lds + QV + hq, 4, s0);
      slash_col(j, s0, f);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        fab[k] = f[k];
        fba[k] = -f[k];
      }
      lds_get(lds + U1 + 4 * a + hq + 2 * ha, 32, s1);
      slash_col_add(eb, s1, fab);
      lds_get(lds + U1 + 4 * b + hq + 2 * hb, 32, s1);
      slash_col_add(ea, s1, fba);
      lds_get_real(lds + KV + 2 * (K_U2 + pr), q);
      const c64 d = lds_scalar(lds + PR + K_U2 + pr);
      propagate(q, cp.mt, d, fab, o);
      lds_put(lds + U2 + 16 * pr + (lane & 7), 96, o);
      propagate(q, cp.mt, d, fba, o);
      lds_put(lds + U2 + 16 * pr + 8 + (lane & 7), 96, o);
    }
    {
      c64 s0[4], s1[4], f[4], o[4];
      lds_get(lds + QV + 2 + hq, 4, s0);
      slash_col(j, s0, f);
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = f[k];
      lds_get(lds + U1 + 16 + 4 * b + hq + 2 * hb, 32, s1);
      slash_col_add(ea, s1, o);  // a-slash W(b) + J-slash(ab) v
      lds_put(lds + W2 + 16 * pr + (lane & 7), 96, o);
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = -f[k];
      lds_get(lds + U1 + 16 + 4 * a + hq + 2 * ha, 32, s1);
      slash_col_add(eb, s1, o);
      lds_put(lds + W2 + 16 * pr + 8 + (lane & 7), 96, o);
    }
  }
  __syncthreads();
#pragma unroll
  for (int pr = 0; pr < 6; ++pr) {
    constexpr int LO[6] = {0, 0, 0, 1, 1, 2}, HI[6] = {1, 2, 3, 2, 3, 3};
    const int a = LO[pr], b = HI[pr], c = LO[5 - pr], d = HI[5 - pr];
    const int vu = h.t | (h.g[a] << 1) | (h.g[b] << 2), vw = h.tb | (h.g[c] << 1) | (h.g[d] << 2);
    c64 u[2][4], w[4];
    lds_get(lds + U2 + 16 * pr + vu, 96, u[0]);
    lds_get(lds + U2 + 16 * pr + 8 + vu, 96, u[1]);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      lds_get(lds + W2 + 16 * (5 - pr) + 8 * o + vw, 96, w);
      const int cc = o ? d : c, dd = o ? c : d;
      A[flow(a, b, cc, dd)] = sdot_add(u[0], w, A[flow(a, b, cc, dd)]);
      A[flow(b, a, cc, dd)] = sdot_add(u[1], w, A[flow(b, a, cc, dd)]);
    }
  }
}

// |M|^2 summed over colours for the helicity code of the lane
template <class P>
__device__ __forceinline__ double hel_value(const double* __restrict__ mom, int64_t i,
                                            const Couplings<double>& c, d2* lds, int lane) {
  c64 A[P::NCOL];
  flows<P>(mom, i, c, lds, lane, A);
  return c.gs2 * P::colour_sum_blocks(A);
}

}  // namespace ggttgg_shared

// One event per wave, lane h assembling helicity h from the shared currents.
// hel_mask: the helicities summed; mehel (or null): each helicity's value.
template <class P>
__global__ void __launch_bounds__(64, 2)
    sigmakin_ggttgg_shared_kernel(const double* __restrict__ mom, int64_t first, int64_t nevt,
                                  double* __restrict__ me, const double* __restrict__ wgt,
                                  double* __restrict__ evtw, double* __restrict__ mehel,
                                  uint64_t hel_mask, Couplings<double> c, double inv_iden) {
  __shared__ d2 lds[ggttgg_shared::LDS_UNITS];
  const int64_t i = first + xcd_event(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x;
  double v = ggttgg_shared::hel_value<P>(mom, i, c, lds, lane);
  if (mehel) mehel[(int64_t)lane * nevt + i] = v;
  v = wave_sum((hel_mask >> lane) & 1 ? v : 0.0);
  if (lane == 0) {
    const double m = v * inv_iden;
    if (me) me[i] = m;
    if (evtw) evtw[i] = m * wgt[i];
  }
}

// ---------------------------------------------------------------------------
// e+ e- -> mu+ mu-, g g -> t t~ and g g -> t t~ g: in one lane's registers
// ---------------------------------------------------------------------------
// e+ e- -> mu+ mu- and g g -> t t~ take one event per lane with all helicities
// unrolled: 2^24 events of the first in 0.46 ms (5.5 TB/s, HBM bound; 1.07 ms
// with one amplitude per helicity), 1000003 events of the second in 52 us
// (340 us; 75 us at one wave per SIMD, without the 36 bytes of scratch that
// two cost).  For g g -> t t~ g that body is 1.6e5 bytes of code and spills
// (2^20 events 1.46 ms); eight lanes per event, one for each helicity of the
// gluons, take 0.95 ms (2.15 ms with one amplitude per helicity; see
// sigmakin_gluon_lanes_kernel).
//
// One object per event holds what no helicity changes (momenta along the
// quark line, propagators, the spinors of both quark helicities); flows_sum
// then takes the gluon helicities and hands the colour-summed |M|^2 of the
// four quark helicities to `emit(t, t~, value)`.  With BEAM the incoming
// gluons run along +z and -z: their polarisation vectors are (0, x, i y, 0)
// with x, y = +-1/sqrt(2), so that slashes and products with them fold to a
// few terms, to a single one where the helicity is known at compile time.

// Helicity states of the direction of p, chi+ = (c, x + i y) and
// chi- = (-x + i y, c), and sqrt(E + P), sqrt(E - P) = m / sqrt(E + P).
// AXIS = +1 / -1: the momentum is along +z / -z, 0: any
template <int AXIS>
__device__ __forceinline__ void helicity_states(const double (&p)[4], double m, double& c,
                                                double& x, double& y, double& big,
                                                double& small) {
  const double pt2 = p[1] * p[1] + p[2] * p[2];
  const double P2 = pt2 + p[3] * p[3];
  const double P = AXIS ? AXIS * p[3] : (P2 > 0.0 ? sqrt_refined(P2, rsqrt_refined(P2)) : 0.0);
  const double epp = p[0] + P, ir = rsqrt_refined(epp);
  big = sqrt_refined(epp, ir);
  small = m * ir;
  if constexpr (AXIS != 0) {
    c = AXIS > 0 ? 1.0 : 0.0;
    x = AXIS > 0 ? 0.0 : 1.0;
    y = 0.0;
  } else {
    const double ppz = p[3] >= 0.0 ? P + p[3] : pt2 * recip(P - p[3]);
    const bool back = !(ppz > 0.0);  // along -z
    const double nrm = rsqrt_refined(back ? 1.0 : 2.0 * P * ppz);
    c = back ? 0.0 : ppz * nrm;
    x = back ? 1.0 : p[1] * nrm;
    y = back ? 0.0 : p[2] * nrm;
  }
}

// ubar (side t, mapped to a column) or v (t~) for both helicities
__device__ __forceinline__ void quark_spinors(const double (&p)[4], double m, bool anti,
                                              c64 (&w)[2][4]) {
  double c, x, y, big, small;
  helicity_states<0>(p, m, c, x, y, big, small);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool up = (h == 1) != anti;
    const double wp = h ? big : small, wm = h ? small : big;
    const c64 c0 = up ? c64{c, 0.0} : c64{-x, y}, c1 = up ? c64{x, y} : c64{c, 0.0};
    if (anti) {
      w[h][0] = wp * c0;
      w[h][1] = wp * c1;
      w[h][2] = -(wm * c0);
      w[h][3] = -(wm * c1);
    } else {
      w[h][0] = wp * conj(c1);
      w[h][1] = -(wp * conj(c0));
      w[h][2] = wm * conj(c1);
      w[h][3] = -(wm * conj(c0));
    }
  }
}

// polarisation vector (ext_vector of helas.h); AXIS = +1 / -1: the momentum
// is along +z / -z, 0: any
template <int AXIS>
__device__ __forceinline__ void polarisation(const double (&p)[4], int lam, bool conjugate,
                                             c64 (&w)[4]) {
  const double r2 = 0.70710678118654752440;
  const double a = -lam * r2, b = conjugate ? r2 : -r2;
  w[0] = c64{0.0, 0.0};
  if constexpr (AXIS != 0) {
    w[1] = c64{AXIS * a, 0.0};
    w[2] = c64{0.0, b};
    w[3] = c64{0.0, 0.0};
  } else {
    const double pt2 = p[1] * p[1] + p[2] * p[2];
    const double iP = rsqrt_refined(pt2 + p[3] * p[3]);
    const bool pt = pt2 > 0.0;
    const double ikt = rsqrt_refined(pt ? pt2 : 1.0);
    const double cph = pt ? p[1] * ikt : 1.0, sph = pt ? p[2] * ikt : 0.0;
    const double cth = p[3] * iP;
    w[1] = c64{a * cth * cph, -b * sph};
    w[2] = c64{a * cth * sph, b * cph};
    w[3] = c64{-a * (pt2 * ikt * iP), 0.0};
  }
}

// -g / (q^2 - m^2 + i m w)
__device__ __forceinline__ c64 quark_factor(const double (&q)[4], double m, double w, double g) {
  const double re = msq(q) - m * m, im = m * w;
  const double n = g * recip(re * re + im * im);
  return c64{-re * n, im * n};
}

// sum and difference of incoming momenta along the quark line
__device__ __forceinline__ void minus4(const double (&a)[4], const double (&b)[4],
                                       double (&o)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) o[m] = a[m] - b[m];
}
__device__ __forceinline__ void plus4(const double (&a)[4], const double (&b)[4],
                                      double (&o)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) o[m] = a[m] + b[m];
}

// Spinors of both helicities as they are now: what follows is computed from
// them in place, not merged across or hoisted out of a helicity loop and kept
// live (and the scheduler keeps the two sides apart).
__device__ __forceinline__ void hold(c64 (&w)[2][4]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) opaque4(w[h]);
  __builtin_amdgcn_sched_barrier(0);
}

template <bool BEAM, class Sum>
struct GGTT {
  c64 u[2][4], v[2][4], d[2];
  double k0[4], k1[4], q[2][4], f01;
  Couplings<double> cp;

  __device__ __forceinline__ GGTT(const double (&p)[4][4], const Couplings<double>& c) : cp(c) {
    quark_spinors(p[2], c.mt, false, u);
    quark_spinors(p[3], c.mt, true, v);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      k0[m] = p[0][m];
      k1[m] = p[1][m];
    }
    double K[4];
    plus4(k0, k1, K);
    f01 = c.gs * recip(msq(K));
    minus4(k0, p[3], q[0]);
    minus4(k1, p[3], q[1]);
#pragma unroll
    for (int a = 0; a < 2; ++a) d[a] = quark_factor(q[a], c.mt, c.wtt, c.gs);
  }

  // flows (01), (10):  A / g = u a-slash W(b) + u J-slash(ab) v
  template <class Emit>
  __device__ __forceinline__ void flows_sum(int lam0, int lam1, Emit emit) {
    c64 e[2][4], J[4];
    hold(v);
    polarisation<BEAM ? 1 : 0>(k0, lam0, false, e[0]);
    polarisation<BEAM ? -1 : 0>(k1, lam1, false, e[1]);
    three_gluon(e[0], k0, e[1], k1, J);
#pragma unroll
    for (int m = 0; m < 4; ++m) J[m] = -f01 * J[m];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      c64 W[2][4], s[4], R[2][4];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        slash_col(e[a], v[tb], s);
        propagate(q[a], cp.mt, d[a], s, W[a]);
      }
      slash_col(J, v[tb], s);
      slash_col(e[0], W[1], R[0]);
      slash_col(e[1], W[0], R[1]);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        R[0][m] = R[0][m] + s[m];
        R[1][m] = R[1][m] - s[m];
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const c64 z{0.0, 0.0};
        const c64 A[2] = {sdot_add(u[t], R[0], z), sdot_add(u[t], R[1], z)};
        emit(t, tb, cp.gs2 * Sum::sum(A));
      }
    }
  }
};

template <bool BEAM, class Sum>
struct GGTTG {
  c64 u[2][4], v[2][4];
  double k[3][4], pt[4], pb[4], f[3], f012;  // f[c]: g / K^2 of the pair without c
  Couplings<double> cp;

  __device__ __forceinline__ GGTTG(const double (&p)[5][4], const Couplings<double>& c) : cp(c) {
    quark_spinors(p[2], c.mt, false, u);
    quark_spinors(p[3], c.mt, true, v);
    double K[4], K3[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      k[0][m] = p[0][m];
      k[1][m] = p[1][m];
      k[2][m] = -p[4][m];
      pt[m] = p[2][m];
      pb[m] = p[3][m];
    }
    plus4(k[0], k[1], K);
    f[2] = c.gs * recip(msq(K));
    plus4(K, k[2], K3);
    f012 = c.gs * recip(msq(K3));
    plus4(k[0], k[2], K);
    f[1] = c.gs * recip(msq(K));
    plus4(k[1], k[2], K);
    f[0] = c.gs * recip(msq(K));
  }

  // polarisation vectors, J[c]: the pair without c, M[m]: J(x m y), m in the middle
  __device__ __forceinline__ void gluon_currents(int lam0, int lam1, int lam2, c64 (&e)[3][4],
                                                 c64 (&J)[3][4], c64 (&M)[2][4]) {
    polarisation<BEAM ? 1 : 0>(k[0], lam0, false, e[0]);
    polarisation<BEAM ? -1 : 0>(k[1], lam1, false, e[1]);
    {
      double p4[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) p4[m] = -k[2][m];
      polarisation<0>(p4, lam2, true, e[2]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int a = c == 0 ? 1 : 0, b = c == 2 ? 1 : 2;
      three_gluon(e[a], k[a], e[b], k[b], J[c]);
#pragma unroll
      for (int m = 0; m < 4; ++m) J[c][m] = -f[c] * J[c][m];
    }
    {
      c64 L1[4], L2[4], L3[4];
      double K[4];
      plus4(k[0], k[1], K);
      three_gluon(J[2], K, e[2], k[2], L1);
      plus4(k[1], k[2], K);
      three_gluon(e[0], k[0], J[0], K, L2);
      plus4(k[0], k[2], K);
      three_gluon(e[1], k[1], J[1], K, L3);
      const c64 d01 = cp.gs * mdot0(e[0], e[1]), d02 = cp.gs * mdot0(e[0], e[2]),
                d12 = cp.gs * mdot0(e[1], e[2]);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        M[0][m] = f012 * cmadd(2.0 * e[0][m], d12,
                               cmsub(e[1][m], d02, cmsub(e[2][m], d01, L1[m] - L3[m])));
        M[1][m] = f012 * cmadd(2.0 * e[1][m], d02,
                               cmsub(e[0][m], d12, cmsub(e[2][m], d01, -(L1[m] + L2[m]))));
      }
    }
  }

  // Gluon whose U and W the lane of gluon helicities (l0 l1 l2) forms, at its
  // own helicity of it: the versions of the three gluons are all covered
  // (two lanes in eight repeat a version of gluon 0)
  __device__ __forceinline__ static int own_gluon(int l0, int l1, int l2) {
    return l0 == l1 ? (l1 == l2 ? 0 : 1) : (l0 == l2 ? 2 : 0);
  }

  // lds: the wave's slots; ev: the event's number in the wave, lane: the lane's.
  // A(abc) / g = U(a).(b-slash W(c) + J-slash(bc) v) + u.(J-slash(ab) W(c) + J-slash(abc) v)
  static constexpr int SU = 0, SW = SU + 4 * 96, SM = SW + 4 * 96, LDS = SM + 8 * 64;
  template <class Emit>
  __device__ __forceinline__ void flows_sum(int l0, int l1, int l2, d2* lds, int ev, int lane,
                                            Emit emit) {
    c64 e[3][4], J[3][4];
    const int ver = 12 * ev;
    auto version = [&](int q, int a) { return ver + 6 * q + 2 * a + (a == 0 ? l0 : a == 1 ? l1 : l2); };
    {
      c64 M[2][4];
      gluon_currents(2 * l0 - 1, 2 * l1 - 1, 2 * l2 - 1, e, J, M);
      lds_put(lds + SM + lane, 64, M[0]);
      lds_put(lds + SM + 256 + lane, 64, M[1]);
      const int own = own_gluon(l0, l1, l2);
      auto pick = [&](double x0, double x1, double x2) { return own == 0 ? x0 : own == 1 ? x1 : x2; };
      const int mine = ver + 2 * own + (own == 0 ? l0 : own == 1 ? l1 : l2);
      const double w = own < 2 ? cp.wtt : cp.wt;
      c64 ea[4], s[4], o[4];
      double ka[4], q[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        ea[m].r = pick(e[0][m].r, e[1][m].r, e[2][m].r);
        ea[m].i = pick(e[0][m].i, e[1][m].i, e[2][m].i);
        ka[m] = pick(k[0][m], k[1][m], k[2][m]);
      }
      minus4(pt, ka, q);
      c64 d = quark_factor(q, cp.mt, w, cp.gs);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        slash_col(ea, u[t], s);
        propagate(q, cp.mt, d, s, o);
        lds_put(lds + SU + mine + 6 * t, 96, o);
      }
      minus4(ka, pb, q);
      d = quark_factor(q, cp.mt, w, cp.gs);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        slash_col(ea, v[t], s);
        propagate(q, cp.mt, d, s, o);
        lds_put(lds + SW + mine + 6 * t, 96, o);
      }
    }
    __syncthreads();
    auto of_antiquark = [&](int tb) {
      __builtin_amdgcn_sched_barrier(0);
      c64 W[3][4], A[2][6], s[4], r[4];
#pragma unroll
      for (int a = 0; a < 3; ++a) lds_get(lds + SW + version(tb, a), 96, W[a]);
      // ordering (a b c): rank 2 a + (b > c)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int b = a == 0 ? 1 : 0, c = a == 2 ? 1 : 2;
        c64 U[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t) lds_get(lds + SU + version(t, a), 96, U[t]);
        slash_col(J[a], v[tb], s);
#pragma unroll
        for (int m = 0; m < 4; ++m) r[m] = s[m];
        slash_col_add(e[b], W[c], r);
#pragma unroll
        for (int t = 0; t < 2; ++t) A[t][2 * a] = sdot_add(U[t], r, c64{0.0, 0.0});
#pragma unroll
        for (int m = 0; m < 4; ++m) r[m] = -s[m];
        slash_col_add(e[c], W[b], r);
#pragma unroll
        for (int t = 0; t < 2; ++t) A[t][2 * a + 1] = sdot_add(U[t], r, c64{0.0, 0.0});
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const int a = c == 0 ? 1 : 0, b = c == 2 ? 1 : 2;
        slash_col(J[c], W[c], s);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const c64 x = sdot_add(u[t], s, c64{0.0, 0.0});
          A[t][2 * a + (b > c)] = A[t][2 * a + (b > c)] + x;
          A[t][2 * b + (a > c)] = A[t][2 * b + (a > c)] - x;
        }
      }
      c64 y[2][2];
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        c64 M[4];
        lds_get(lds + SM + 256 * m + lane, 64, M);
        slash_col(M, v[tb], s);
#pragma unroll
        for (int t = 0; t < 2; ++t) y[t][m] = sdot_add(u[t], s, c64{0.0, 0.0});
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const c64 y2 = -(y[t][0] + y[t][1]);
        A[t][0] = A[t][0] + y[t][1];  // (012)
        A[t][5] = A[t][5] + y[t][1];  // (210)
        A[t][2] = A[t][2] + y[t][0];  // (102)
        A[t][4] = A[t][4] + y[t][0];  // (201)
        A[t][1] = A[t][1] + y2;       // (021)
        A[t][3] = A[t][3] + y2;       // (120)
        emit(t, tb, cp.gs2 * Sum::sum(A[t]));
      }
    };
    of_antiquark(0);
    of_antiquark(1);
  }
};

// e+ e- -> mu+ mu-: massless leptons have one current per chirality and side,
//   j(L) = chi-^+(f) sbar^mu chi-(g),  j(R) = chi+^+(f) s^mu chi+(g)
// (times sqrt(E + P) of both), f the row (e+, mu-), g the column (e-, mu+),
// and four of the 16 helicities; the others vanish identically.
struct LeptonCurrents {
  c64 j[2][4];  // chirality L, R
};
template <int AF, int AG>
__device__ __forceinline__ void lepton_currents(const double (&pf)[4], const double (&pg)[4],
                                                LeptonCurrents& o) {
  double fc, fx, fy, fb, gc, gx, gy, gb, none;
  helicity_states<AF>(pf, 0.0, fc, fx, fy, fb, none);
  helicity_states<AG>(pg, 0.0, gc, gx, gy, gb, none);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const c64 f0 = h ? c64{fc, 0.0} : c64{-fx, -fy}, f1 = h ? c64{fx, -fy} : c64{fc, 0.0};
    const c64 g0 = gb * fb * (h ? c64{gc, 0.0} : c64{-gx, gy}),
              g1 = gb * fb * (h ? c64{gx, gy} : c64{gc, 0.0});
    const c64 a00 = f0 * g0, a11 = f1 * g1, a01 = f0 * g1, a10 = f1 * g0;
    const double s = h ? 1.0 : -1.0;
    o.j[h][0] = a00 + a11;
    o.j[h][1] = s * (a01 + a10);
    o.j[h][2] = s * times_i(a10 - a01);
    o.j[h][3] = s * (a00 - a11);
  }
}

template <class P, bool BEAM, class Take>
__device__ __forceinline__ void eemumu_shared(const double (&p)[4][4], const Couplings<double>& c,
                                              Take take) {
  LeptonCurrents e, mu;
  lepton_currents<BEAM ? 1 : 0, BEAM ? -1 : 0>(p[0], p[1], e);
  lepton_currents<0, 0>(p[3], p[2], mu);
  double K[4];
  plus4(p[0], p[1], K);
  const double k2 = msq(K), re = k2 - c.mz * c.mz, im = c.mz * c.wz;
  const double photon = c.cqed * c.cqed * recip(k2);
  const double n = recip(re * re + im * im);
  const c64 d{re * n, -im * n};
  const double im2 = recip(c.mz * c.mz);
  c64 ke[2], km[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    ke[h] = im2 * mdot(K, e.j[h]);
    km[h] = mdot(K, mu.j[h]);
  }
#pragma unroll
  for (int h = 0; h < 16; ++h) {
    // e+ and e-, mu+ and mu- have opposite helicities; L: the first of each +
    const int a = (h >> 2) == 1 ? 1 : 0, b = (h & 3) == 1 ? 1 : 0;
    double v = 0.0;
    if (((h >> 2) == 1 || (h >> 2) == 2) && ((h & 3) == 1 || (h & 3) == 2)) {
      const double zz = (a ? c.czr : c.czl) * (b ? c.czr : c.czl);
      const c64 s = mdot0(e.j[a], mu.j[b]);
      const c64 A = photon * s + zz * (d * (s - ke[a] * km[b]));
      v = A.r * A.r + A.i * A.i;
    }
    take(h, v);
  }
}

// The colour sum of a process for the objects above
template <class P>
struct ColourSum {
  __device__ static __forceinline__ double sum(const c64 (&A)[P::NCOL]) {
    return P::template colour_sum<double>(A);
  }
};

// One event per lane: |M|^2 summed over the helicities of hel_mask
template <class P, int BS>
__global__ void __launch_bounds__(BS, 2)
    sigmakin_shared_kernel(const double* __restrict__ mom, int64_t nevt, double* __restrict__ me,
                           const double* __restrict__ wgt, double* __restrict__ evtw,
                           double* __restrict__ mehel, uint64_t hel_mask, Couplings<double> c,
                           double inv_iden) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= nevt) return;
  double p[P::NPAR][4];
  load_event<P>(mom, i, p);
  double acc = 0.0;
  auto take = [&](int h, double v) {
    if (mehel) mehel[(int64_t)h * nevt + i] = v;
    acc += (hel_mask >> h) & 1 ? v : 0.0;
  };
  if (__all(beams_on_axis(p))) {
    set_beams(p);
    P::template shared<true>(p, c, take);
  } else {
    P::template shared<false>(p, c, take);
  }
  const double m = acc * inv_iden;
  if (me) me[i] = m;
  if (evtw) evtw[i] = m * wgt[i];
}

// all helicities of one event in a lane
template <class P, bool BEAM, class Take>
__device__ __forceinline__ void ggtt_shared(const double (&p)[4][4], const Couplings<double>& c,
                                            Take take) {
  GGTT<BEAM, ColourSum<P>> ev(p, c);
#pragma unroll
  for (int h = 0; h < 4; ++h)
    ev.flows_sum(h & 2 ? 1 : -1, h & 1 ? 1 : -1,
                 [&](int t, int tb, double v) { take((h << 2) | (t << 1) | tb, v); });
}

// Eight lanes per event, one for each helicity of the three gluons, each with
// the four quark helicities; the sum over the lanes is a DPP butterfly.  The
// U(a) and W(a) depend on one gluon's helicity: an event has 12 versions of
// each, a lane forms four and reads the others from LDS (20 KB a wave, with the
// M of the lane).  Bound: FP64 VALU at one wave per SIMD, 2.7e3 instructions a
// wave, busy 62 % of the time; 2^20 events in 945 us (each lane all of its U and
// W, 3.7e3 instructions: 1023 us; two waves per SIMD of 256 registers: 570 bytes
// of scratch a lane, 1305 us).
template <class P>
__global__ void __launch_bounds__(64)
    sigmakin_gluon_lanes_kernel(const double* __restrict__ mom, int64_t first, int64_t nevt,
                                double* __restrict__ me, const double* __restrict__ wgt,
                                double* __restrict__ evtw, double* __restrict__ mehel,
                                uint64_t hel_mask, Couplings<double> c, double inv_iden) {
  const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int64_t i = first + (j >> 3);
  if (i >= nevt) return;
  const int g = (int)j & 7;
  __shared__ d2 lds[GGTTG<true, ColourSum<P>>::LDS];
  double p[P::NPAR][4];
  load_event<P>(mom, i, p);
  double acc = 0.0;
  const int code = ((g & 6) << 2) | (g & 1);  // gluons 0 and 1: bits 4, 3; gluon 2: bit 0
  auto take = [&](int t, int tb, double v) {
    const int h = code | (t << 2) | (tb << 1);
    if (mehel) mehel[(int64_t)h * nevt + i] = v;
    acc += (hel_mask >> h) & 1 ? v : 0.0;
  };
  const int l0 = g >> 2, l1 = (g >> 1) & 1, l2 = g & 1, ev = threadIdx.x >> 3;
  if (__all(beams_on_axis(p))) {
    set_beams(p);
    GGTTG<true, ColourSum<P>>(p, c).flows_sum(l0, l1, l2, lds, ev, threadIdx.x, take);
  } else {
    GGTTG<false, ColourSum<P>>(p, c).flows_sum(l0, l1, l2, lds, ev, threadIdx.x, take);
  }
  acc += dpp_move<0xB1>(acc);   // quad_perm 1 0 3 2
  acc += dpp_move<0x4E>(acc);   // quad_perm 2 3 0 1
  acc += dpp_move<0x141>(acc);  // row_half_mirror
  if (g == 0) {
    const double m = acc * inv_iden;
    if (me) me[i] = m;
    if (evtw) evtw[i] = m * wgt[i];
  }
}

inline uint64_t helicity_mask(const HelList& l) {
  uint64_t m = 0;
  for (int k = 0; k < l.n; ++k) m |= 1ull << l.code[k];
  return m;
}

template <class P, int BS>
int sigmakin_shared_launch(const MeArgs& a, const double* mom, int64_t nevt, double* me,
                           const double* wgt, double* evtw, double* mehel, hipStream_t s) {
  const unsigned g = (unsigned)((nevt + BS - 1) / BS);
  sigmakin_shared_kernel<P, BS><<<g, BS, 0, s>>>(mom, nevt, me, wgt, evtw, mehel,
                                                 helicity_mask(a.hel), a.c64, a.inv_iden);
  return 0;
}

template <class P>
int sigmakin_ggttgg_shared_launch(const MeArgs& a, const double* mom, int64_t nevt, double* me,
                                  const double* wgt, double* evtw, double* mehel, hipStream_t s) {
  for (int64_t i = 0; i < nevt; i += launch_events(64)) {
    const unsigned g = (unsigned)std::min(nevt - i, launch_events(64));
    sigmakin_ggttgg_shared_kernel<P><<<g, 64, 0, s>>>(mom, i, nevt, me, wgt, evtw, mehel,
                                                      helicity_mask(a.hel), a.c64, a.inv_iden);
  }
  return 0;
}

}  // namespace mg
