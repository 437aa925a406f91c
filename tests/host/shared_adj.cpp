// Reverse-mode routines of the shared-current gradient (shared_adjoint.h)
// against fourth-order central differences of the forward routines they
// reverse (shared_currents.h), compiled for the host by
// test_shared_adjoint_host.py.
//
// For out = f(x) and any output adjoint ob, L(x) = Re<ob, f(x)>; the routine's
// adjoint of x times a random direction must equal the difference quotient of
// L along it.  Prints one line per routine: name, trials, largest relative
// mismatch; then `limit` lines: what the quark adjoint gives along -z and at
// rest, where the helicity states are constants.
#include "shared_adjoint.h"

using namespace mg;

static std::mt19937_64 rng(20261205);
static double U(double a = -1.0, double b = 1.0) {
  return std::uniform_real_distribution<double>(a, b)(rng);
}
static void rvec(c64 (&v)[4]) {
  for (int k = 0; k < 4; ++k) v[k] = c64{U(), U()};
}
static double re4(const c64 (&a)[4], const c64 (&b)[4]) {
  double s = 0;
  for (int k = 0; k < 4; ++k) s += a[k].r * b[k].r + a[k].i * b[k].i;
  return s;
}
static double dot(const double (&a)[4], const double (&b)[4]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + a[3] * b[3];
}
static double slope(const std::function<double(double)>& L, double h) {
  return (8.0 * (L(h) - L(-h)) - (L(2.0 * h) - L(-2.0 * h))) / (12.0 * h);
}
static void along(const double (&p)[4], const double (&d)[4], double t, double (&o)[4]) {
  for (int k = 0; k < 4; ++k) o[k] = p[k] + t * d[k];
}
static void along(const c64 (&p)[4], const c64 (&d)[4], double t, c64 (&o)[4]) {
  for (int k = 0; k < 4; ++k) o[k] = c64{p[k].r + t * d[k].r, p[k].i + t * d[k].i};
}

struct Report {
  const char* name;
  int n = 0;
  double worst = 0;
  // scale: of what cancels in the two sides
  void add(double lhs, double rhs, double scale) {
    ++n;
    worst = std::fmax(worst, std::fabs(lhs - rhs) / scale);
  }
  ~Report() { std::printf("%s %d %.3e\n", name, n, worst); }
};
static const int NTRIAL = 200;

static void momentum(double m, double (&p)[4]) {
  for (int k = 1; k < 4; ++k) p[k] = U(-300.0, 300.0);
  p[0] = std::sqrt(m * m + p[1] * p[1] + p[2] * p[2] + p[3] * p[3]);
}

static void test_quark(bool anti) {
  Report r{anti ? "QuarkAdjoint(t~)" : "QuarkAdjoint(t)"};
  for (int t = 0; t < NTRIAL; ++t) {
    double p[4], d[4], pb[4] = {0, 0, 0, 0};
    momentum(173.0, p);
    for (int k = 0; k < 4; ++k) d[k] = U();
    c64 wb[2][4];
    QuarkAdjoint q;
    for (int h = 0; h < 2; ++h) {
      rvec(wb[h]);
      q.add(p, 173.0, anti, h, wb[h]);
    }
    q.finish(p, 173.0, pb);
    auto L = [&](double x) {
      double s[4];
      c64 w[2][4];
      along(p, d, x, s);
      quark_spinors(s, 173.0, anti, w);
      return re4(wb[0], w[0]) + re4(wb[1], w[1]);
    };
    r.add(slope(L, 1e-2), dot(pb, d), 1e-2);  // d w / d p ~ sqrt(E) / E and larger near the axis
  }
}

static void test_polarisation() {
  Report r{"adj_polarisation"};
  for (int t = 0; t < NTRIAL; ++t) {
    double p[4], d[4], pb[4] = {0, 0, 0, 0};
    momentum(0.0, p);
    for (int k = 0; k < 4; ++k) d[k] = U();
    c64 wb[4];
    rvec(wb);
    const int lam = t & 1 ? 1 : -1;
    adj_polarisation(p, lam, wb, pb);
    auto L = [&](double x) {
      double s[4];
      c64 w[4];
      along(p, d, x, s);
      polarisation<0>(s, lam, true, w);
      return re4(wb, w);
    };
    r.add(slope(L, 1e-3), dot(pb, d), 1e-2);
  }
}

static void test_propagate() {
  Report r{"adj_propagate"};
  for (int t = 0; t < NTRIAL; ++t) {
    const double m = 173.0, w = 1.49, g = 1.21;
    double q[4], dq[4], qb[4] = {0, 0, 0, 0};
    do {
      for (int k = 1; k < 4; ++k) q[k] = U(-300.0, 300.0);
      q[0] = U(-800.0, 800.0);
    } while (std::fabs(msq(q) - m * m) < 2.0e4);
    c64 f[4], df[4], ob[4], fb[4];
    rvec(f); rvec(df); rvec(ob);
    for (int k = 0; k < 4; ++k) dq[k] = U();
    adj_propagate(q, m, 1.0 / g, quark_factor(q, m, w, g), f, ob, fb, qb);
    auto L = [&](double x) {
      double s[4];
      c64 fs[4], o[4];
      along(q, dq, x, s);
      along(f, df, x, fs);
      propagate(s, m, quark_factor(s, m, w, g), fs, o);
      return re4(ob, o);
    };
    r.add(slope(L, 1e-3), dot(qb, dq) + re4(fb, df), 1e-2);
  }
}

static void test_three_gluon() {
  Report r{"adj_three_gluon_y"};
  for (int t = 0; t < NTRIAL; ++t) {
    c64 x[4], y[4], dy[4], ob[4], yb[4];
    double kx[4], ky[4], dk[4], kb[4] = {0, 0, 0, 0};
    rvec(x); rvec(y); rvec(dy); rvec(ob);
    clear4(yb);
    for (int k = 0; k < 4; ++k) {
      kx[k] = U();
      ky[k] = U();
      dk[k] = U();
    }
    adj_three_gluon_y(x, kx, y, ky, ob, yb, kb);
    auto L = [&](double e) {
      double s[4];
      c64 ys[4], o[4];
      along(ky, dk, e, s);
      along(y, dy, e, ys);
      three_gluon(x, kx, ys, s, o);
      return re4(ob, o);
    };
    r.add(slope(L, 1e-3), dot(kb, dk) + re4(yb, dy), 1.0);
  }
}

static void test_slash_and_sdot() {
  Report r{"adj_slash"}, s{"adj_sdot"};
  for (int t = 0; t < NTRIAL; ++t) {
    c64 V[4], G[4], dV[4], dG[4], ob[4], Vb[4], Gb[4];
    rvec(V); rvec(G); rvec(dV); rvec(dG); rvec(ob);
    clear4(Vb);
    clear4(Gb);
    adj_slash_spinor(V, ob, Gb);
    adj_slash_vector(G, ob, Vb);
    auto L = [&](double e) {
      c64 v[4], g[4], o[4];
      along(V, dV, e, v);
      along(G, dG, e, g);
      slash_col(v, g, o);
      return re4(ob, o);
    };
    r.add(slope(L, 1e-3), re4(Vb, dV) + re4(Gb, dG), 1.0);
    const c64 ab = ob[0], z{0.0, 0.0};
    clear4(Vb);
    clear4(Gb);
    adj_sdot(V, G, ab, Vb, Gb);
    auto M = [&](double e) {
      c64 v[4], g[4];
      along(V, dV, e, v);
      along(G, dG, e, g);
      const c64 a = sdot_add(v, g, z);
      return ab.r * a.r + ab.i * a.i;
    };
    s.add(slope(M, 1e-3), re4(Vb, dV) + re4(Gb, dG), 1.0);
  }
}

static void test_limits() {
  const double P[3][4] = {{std::sqrt(173.0 * 173.0 + 400.0 * 400.0), 0.0, 0.0, -400.0},
                          {173.0, 0.0, 0.0, 0.0}, {400.0, 0.0, 0.0, -400.0}};
  const double M[3] = {173.0, 173.0, 0.0};
  for (int c = 0; c < 3; ++c) {
    double p[4], pb[4] = {0, 0, 0, 0};
    for (int k = 0; k < 4; ++k) p[k] = P[c][k];
    QuarkAdjoint q;
    for (int h = 0; h < 2; ++h) {
      c64 wb[4];
      for (int k = 0; k < 4; ++k) wb[k] = c64{0.3 + k, 0.1 * h - k};
      q.add(p, M[c], false, h, wb);
    }
    q.finish(p, M[c], pb);
    // with constant states: w = (sqrt(E + P), sqrt(E - P)) alone moves
    const double v = c == 1 ? 0.0 : p[3] / 400.0, big = std::sqrt(p[0] - p[3]), small = M[c] / big;
    const double eb = 0.5 / big * (q.big - q.small * small / big);
    std::printf("limit %d %.17g %.17g %.17g %.17g %.17g %.17g\n", c, pb[0], pb[1], pb[2], pb[3], eb, v * eb);
  }
}

int main() {
  test_quark(false);
  test_quark(true);
  test_polarisation();
  test_propagate();
  test_three_gluon();
  test_slash_and_sdot();
  test_limits();
  return 0;
}
