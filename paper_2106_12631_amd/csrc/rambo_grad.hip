// First and last kernel of the shared-current gradient (shared_adjoint.h),
// one event per lane: RAMBO into the gradient buffer, and RAMBO's reverse
// sweep from the momentum gradient to the uniforms.
//
// Reverse mode: with L a function of the final-state three-momenta, one sweep
// back through the rescaling, the boost and the uniforms gives all 4 NF
// derivatives (a second one those of log w), where a forward-mode pass is
// needed per uniform: 2^18 g g -> t t~ g events in 43 us for both kernels.  The
// massless |p_i| equals its energy e_i, and the rescaling xi follows the
// implicit-function theorem, as in rambo.h.
#include "common.h"
#include "internal.h"
#include "rambo.h"

namespace mg {

template <int NF>
__global__ void __launch_bounds__(256)
    grad_momenta_kernel(const double* __restrict__ rnd, int64_t nevt, RamboArgs a,
                        double* __restrict__ buf) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nevt) return;
  double r[4 * NF], p[NF + 2][4], w;
#pragma unroll
  for (int k = 0; k < 4 * NF; ++k) r[k] = rnd[aosoa_rnd(i, k, 4 * NF)];
  rambo<NF>(r, a, p, w);
#pragma unroll
  for (int l = 0; l < NF; ++l)
#pragma unroll
    for (int m = 0; m < 4; ++m) buf[aosoa_rnd(i, 4 * l + m, 4 * NF)] = p[l + 2][m];
}

// RAMBO's massless stage, kept for the reverse sweep
template <int NF>
struct Massless {
  double q0[NF], n[NF][3], c[NF], st[NF], cph[NF], sph[NF];
  double Q0, Q[3], M, iM, iQ0M, x, E[NF], t[NF], P[NF][3];  // E: rest-frame energies before scaling

  __device__ __forceinline__ Massless(const double (&r)[4 * NF], double sqrts) {
    const double twopi = 6.283185307179586476925286766559;
    Q0 = 0.0;
    Q[0] = Q[1] = Q[2] = 0.0;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      c[i] = 2.0 * r[4 * i] - 1.0;
      st[i] = sqrt(1.0 - c[i] * c[i]);
      sincos(twopi * r[4 * i + 1], &sph[i], &cph[i]);
      q0[i] = -log(r[4 * i + 2] * r[4 * i + 3]);
      n[i][0] = st[i] * cph[i];
      n[i][1] = st[i] * sph[i];
      n[i][2] = c[i];
      Q0 += q0[i];
#pragma unroll
      for (int m = 0; m < 3; ++m) Q[m] += q0[i] * n[i][m];
    }
    double EM[NF], M2 = 0.0;
#pragma unroll
    for (int i = 0; i < NF; ++i) EM[i] = 0.0;
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int j = i + 1; j < NF; ++j) {
        const double d0 = n[i][0] - n[j][0], d1 = n[i][1] - n[j][1], d2 = n[i][2] - n[j][2];
        const double dij = 0.5 * q0[i] * q0[j] * (d0 * d0 + d1 * d1 + d2 * d2);
        EM[i] += dij;
        EM[j] += dij;
      }
#pragma unroll
    for (int i = 0; i < NF; ++i) M2 += EM[i];
    M = sqrt(M2);
    iM = 1.0 / M;
    iQ0M = 1.0 / (Q0 + M);
    x = sqrts * iM;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      E[i] = EM[i] * iM;
      t[i] = (q0[i] + E[i]) * iQ0M;
#pragma unroll
      for (int m = 0; m < 3; ++m) P[i][m] = x * (q0[i] * n[i][m] - Q[m] * t[i]);
    }
  }

  // adjoints Pb of the massless three-momenta and eb of the energies x E to
  // the uniforms
  __device__ __forceinline__ void reverse(const double (&r)[4 * NF], const double (&Pb)[NF][3],
                                          const double (&eb)[NF], double (&rb)[4 * NF]) const {
    const double twopi = 6.283185307179586476925286766559;
    double q0b[NF], nb[NF][3], Eb[NF], Qb[3] = {0.0, 0.0, 0.0}, xb = 0.0, Q0Mb = 0.0;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      double tb = 0.0;
      q0b[i] = 0.0;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        const double vb = x * Pb[i][m];
        xb += Pb[i][m] * (q0[i] * n[i][m] - Q[m] * t[i]);
        q0b[i] += vb * n[i][m];
        nb[i][m] = vb * q0[i];
        Qb[m] -= vb * t[i];
        tb -= vb * Q[m];
      }
      xb += eb[i] * E[i];
      const double sb = tb * iQ0M;
      q0b[i] += sb;
      Eb[i] = x * eb[i] + sb;
      Q0Mb -= sb * t[i];
    }
    double Mb = Q0Mb - xb * x * iM, EMb[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      EMb[i] = Eb[i] * iM;
      Mb -= EMb[i] * E[i];
    }
    const double M2b = 0.5 * Mb * iM;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      q0b[i] += Q0Mb;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        q0b[i] += Qb[m] * n[i][m];
        nb[i][m] += Qb[m] * q0[i];
      }
    }
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int j = i + 1; j < NF; ++j) {
        const double db = EMb[i] + EMb[j] + 2.0 * M2b;
        const double d[3] = {n[i][0] - n[j][0], n[i][1] - n[j][1], n[i][2] - n[j][2]};
        const double h = 0.5 * db * (d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        q0b[i] += h * q0[j];
        q0b[j] += h * q0[i];
        const double qq = db * q0[i] * q0[j];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          nb[i][m] += qq * d[m];
          nb[j][m] -= qq * d[m];
        }
      }
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const double stb = nb[i][0] * cph[i] + nb[i][1] * sph[i];
      const double phb = st[i] * (nb[i][1] * cph[i] - nb[i][0] * sph[i]);
      const double cb = nb[i][2] - (st[i] > 0.0 ? stb * c[i] / st[i] : 0.0);
      rb[4 * i] = 2.0 * cb;
      rb[4 * i + 1] = twopi * phb;
      rb[4 * i + 2] = -q0b[i] / r[4 * i + 2];
      rb[4 * i + 3] = -q0b[i] / r[4 * i + 3];
    }
  }
};

template <int NF>
__global__ void __launch_bounds__(256)
    grad_uniforms_kernel(const double* __restrict__ rnd, int64_t nevt, RamboArgs a, double inv_iden,
                         const double* __restrict__ gbar, double* grad, double* logw, double* f) {
  constexpr int NR = 4 * NF;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nevt) return;
  double r[NR], kb[NF][3], me;
#pragma unroll
  for (int k = 0; k < NR; ++k) r[k] = rnd[aosoa_rnd(i, k, NR)];
#pragma unroll
  for (int l = 0; l < NF; ++l)
#pragma unroll
    for (int m = 0; m < 3; ++m) kb[l][m] = grad[aosoa_rnd(i, 3 * l + m, NR)];
  me = grad[aosoa_rnd(i, 3 * NF, NR)];
  const Massless<NF> s(r, a.sqrts);
  double e[NF], w = a.w0, Pb[NF][3], eb[NF], zero[NF][3], lb[NF] = {};
#pragma unroll
  for (int l = 0; l < NF; ++l) e[l] = s.x * s.E[l];
  bool ok = true;
  if (a.massive) {
    const double xi = rambo_scale<NF>(e, a, ok);
    double ik0[NF], den2 = 0.0, prod = 1.0, xib = 0.0;
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      ik0[l] = 1.0 / sqrt(a.m2[l] + xi * xi * e[l] * e[l]);
      den2 += e[l] * e[l] * ik0[l];
      prod *= xi * e[l] * ik0[l];
    }
    double xin = 1.0;
#pragma unroll
    for (int k = 0; k < 2 * NF - 3; ++k) xin *= xi;
    const double iden2 = 1.0 / den2;
    w = a.w0 * xin * prod * a.sqrts * iden2 / (xi * xi);
    // k = xi P; d xi = -xi sum(e de / k0) / sum(e^2 / k0)
#pragma unroll
    for (int l = 0; l < NF; ++l)
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        xib += kb[l][m] * s.P[l][m];
        Pb[l][m] = xi * kb[l][m];
      }
    // log w = (2 NF - 5) log xi + sum log(xi e / k0) - log sum(e^2 / k0), k0^2 = m^2 + xi^2 e^2
    double lxi = 2 * NF - 5;
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      const double b2 = xi * xi * e[l] * e[l] * ik0[l] * ik0[l];  // velocity squared
      const double q = e[l] * e[l] * ik0[l] * iden2;
      lxi += 1.0 - b2 + q * b2;
      lb[l] = (1.0 - b2) / e[l] - q * (2.0 - b2) / e[l];
    }
    double emean = 0.0, lmean = 0.0;
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      const double g = e[l] * ik0[l] * iden2;
      eb[l] = -xi * g * xib;
      lb[l] -= g * lxi;
      emean += eb[l] * (1.0 / NF);
      lmean += lb[l] * (1.0 / NF);
    }
    // the energies sum to sqrt(s) whatever the uniforms: what their adjoints
    // have in common drops out, here rather than by cancellation in the sweep
    // (all of it for two equal masses, whose weight is a constant)
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      eb[l] -= emean;
      lb[l] -= lmean;
    }
  } else {
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      eb[l] = 0.0;
#pragma unroll
      for (int m = 0; m < 3; ++m) Pb[l][m] = kb[l][m];
    }
  }
  if (!ok) w = failed_weight();
  double rb[NR], lw[NR];
  s.reverse(r, Pb, eb, rb);
#pragma unroll
  for (int l = 0; l < NF; ++l)
#pragma unroll
    for (int m = 0; m < 3; ++m) zero[l][m] = 0.0;
  if (a.massive) {
    s.reverse(r, zero, lb, lw);
  } else {  // the weight of massless particles is a constant, collinear or not
#pragma unroll
    for (int k = 0; k < NR; ++k) lw[k] = 0.0;
  }
  const double g = gbar ? gbar[i] : 1.0;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    grad[aosoa_rnd(i, k, NR)] = g * (inv_iden * w * (rb[k] + me * lw[k]));
    if (logw) logw[aosoa_rnd(i, k, NR)] = ok ? lw[k] : failed_weight();
  }
  if (f) f[i] = me * inv_iden * w;
}

int launch_grad_momenta(int nf, const double* rnd, int64_t nevt, const RamboArgs& a, double* buf,
                        hipStream_t s) {
  const unsigned g = (unsigned)((nevt + 255) / 256);
  if (nf == 2) grad_momenta_kernel<2><<<g, 256, 0, s>>>(rnd, nevt, a, buf);
  else if (nf == 3) grad_momenta_kernel<3><<<g, 256, 0, s>>>(rnd, nevt, a, buf);
  else return -1;
  return 0;
}

int launch_grad_uniforms(int nf, const double* rnd, int64_t nevt, const RamboArgs& a,
                         double inv_iden, const double* gbar, double* grad, double* logw,
                         double* f, hipStream_t s) {
  const unsigned g = (unsigned)((nevt + 255) / 256);
  if (nf == 2)
    grad_uniforms_kernel<2><<<g, 256, 0, s>>>(rnd, nevt, a, inv_iden, gbar, grad, logw, f);
  else if (nf == 3)
    grad_uniforms_kernel<3><<<g, 256, 0, s>>>(rnd, nevt, a, inv_iden, gbar, grad, logw, f);
  else return -1;
  return 0;
}

}  // namespace mg
