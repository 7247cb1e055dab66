// Device functions of the native-layout Wilson stencils (dslash.hip, hop.hip).
//
// Every hop uses the rank-2 spin projection of (1 +/- gamma_mu) in the chiral basis
// gamma_mu = [[0, A_mu], [A_mu^dag, 0]] (A_x = -i sigma_1, A_y = -i sigma_2,
// A_z = -i sigma_3, A_t = 1):
//   (1 + s gamma_mu) chi = [ h ; s A_mu^dag h ],  h = chi_up + s A_mu chi_down,
// so a hop multiplies two colour vectors by the link instead of four.
#pragma once

#include "qmg_internal.hpp"

namespace qmg {
namespace {

constexpr int kBlock = 256;

// XCD-aware tile index: hardware hands workgroup b to XCD b % 8.
__device__ inline int xcd_tile(int b, int nb) {
  const int q = nb >> 3, rem = nb & 7, x = b & 7, i = b >> 3;
  return x * q + min(x, rem) + i;
}

__device__ inline size_t sp_idx(int rhs, int comp, int site, int V) { return (size_t(rhs) * 12 + comp) * V + site; }
__device__ inline size_t g_idx(int mu, int e, int site, int V) { return (size_t(mu) * 9 + e) * V + site; }

// h = chi_up + s A_mu chi_dn   (2 spin x 3 colour), components index 3*spin + colour
template <int MU, class C>
__device__ inline void project(const cplx<C>* chi, C s, cplx<C>* h) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cplx<C> u0 = chi[c], u1 = chi[3 + c], d0 = chi[6 + c], d1 = chi[9 + c];
    if (MU == 0) {         // A = -i sigma_1: (A d) = (-i d1, -i d0)
      h[c] = u0 + s * times_mi(d1);
      h[3 + c] = u1 + s * times_mi(d0);
    } else if (MU == 1) {  // A = -i sigma_2 = [[0,-1],[1,0]]: (A d) = (-d1, d0)
      h[c] = u0 - s * d1;
      h[3 + c] = u1 + s * d0;
    } else if (MU == 2) {  // A = -i sigma_3 = diag(-i, i)
      h[c] = u0 + s * times_mi(d0);
      h[3 + c] = u1 + s * times_i(d1);
    } else {               // A = 1
      h[c] = u0 + s * d0;
      h[3 + c] = u1 + s * d1;
    }
  }
}

// acc += coef * [ w ; s A_mu^dag w ]
template <int MU, class C>
__device__ inline void reconstruct(cplx<C>* acc, const cplx<C>* w, C s, C coef) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cplx<C> w0 = coef * w[c], w1 = coef * w[3 + c];
    acc[c] += w0;
    acc[3 + c] += w1;
    const C cs = s;
    if (MU == 0) {         // A^dag = i sigma_1: (i w1, i w0)
      acc[6 + c] += cs * times_i(w1);
      acc[9 + c] += cs * times_i(w0);
    } else if (MU == 1) {  // A^dag = [[0,1],[-1,0]]: (w1, -w0)
      acc[6 + c] += cs * w1;
      acc[9 + c] -= cs * w0;
    } else if (MU == 2) {  // A^dag = diag(i, -i)
      acc[6 + c] += cs * times_i(w0);
      acc[9 + c] += cs * times_mi(w1);
    } else {
      acc[6 + c] += cs * w0;
      acc[9 + c] += cs * w1;
    }
  }
}

template <class C, bool ADJ>
__device__ inline void su3_mul(const cplx<C>* u, const cplx<C>* h, cplx<C>* w) {
#pragma unroll
  for (int sp = 0; sp < 2; ++sp) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cplx<C> t = {C(0), C(0)};
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (ADJ) t += cmul_conj(u[3 * b + a], h[3 * sp + b]);
        else t += u[3 * a + b] * h[3 * sp + b];
      }
      w[3 * sp + a] = t;
    }
  }
}

// p0 + p1 + p2 + p3 + d o: the four partial sums of the direction-split stencils and the large diagonal term, which
// comes last (added first, every sum is rounded at its size).  In FP32 in double, rounded once: relative error
// at xi = 1 / 3.5 5.6e-8 / 4.2e-8, plain 5.9e-8 / 4.5e-8, diagonal first 7.1e-8 / 5.8e-8.  16-bit storage rounds the result
// ten thousand times coarser, and the site term of the clover form (d = 1) has roundings of its own.
template <class S>
__device__ inline cplx<ctype<S>> sum_directions(cplx<ctype<S>> p0, cplx<ctype<S>> p1, cplx<ctype<S>> p2,
                                                cplx<ctype<S>> p3, ctype<S> d, cplx<ctype<S>> o) {
  if constexpr (StoreTraits<S>::prec == QMG_F32) {
    auto sum = [&](float a, float b, float c, float e, float f) {
      return float(fma(double(d), double(f), ((double(a) + double(b)) + double(c)) + double(e)));
    };
    return {sum(p0.re, p1.re, p2.re, p3.re, o.re), sum(p0.im, p1.im, p2.im, p3.im, o.im)};
  } else {
    return ((p0 + p1) + p2) + p3 + d * o;
  }
}
// the same with each addition's rounding error, which are summed and added at the end (FP64 canonical, error against
// extended precision at xi = 1 / 3.5: 6.9e-17 / 7.5e-17, plain 7.6e-17 / 7.9e-17, diagonal first 1.06e-16 / 1.05e-16; eight
// hops and the diagonal term one by one 8.0e-17 / 7.9e-17)
__device__ inline double sum_compensated(double p0, double p1, double p2, double p3, double d, double o) {
  double s = p0, e = 0;
  auto add = [&](double x) {
    const double t = s + x, b = t - s;
    e += (s - (t - b)) + (x - b);
    s = t;
  };
  add(p1);
  add(p2);
  add(p3);
  const double t = fma(d, o, s), b = t - s;
  e += (s - (t - b)) + fma(d, o, -b);
  const double r = t + e;
  return isfinite(r) ? r : t;  // an infinite sum has no rounding error: its e is not a number
}

// NE = 6: native links stored as their first two rows ([mu][6][V]); the third row of an SU(3)
// matrix is the complex conjugate of the cross product of the first two
template <class S, int NR, int MU, bool FWD, bool DAG, int NE = 9>
__device__ inline void do_hop(const S* __restrict__ U, const S* __restrict__ in, cplx<ctype<S>> (*acc)[12],
                              int link_site, int nb_site, int rhs0, int V, ctype<S> coef) {
  using C = ctype<S>;
  cplx<C> u[9];
  if constexpr (NE == 9) {
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = ldc(U, g_idx(MU, e, link_site, V));
  } else {
    static_assert(NE == 6, "two-row links");
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = ldc(U, (size_t(MU) * 6 + e) * V + link_site);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
      u[6 + c] = conj(u[c1] * u[3 + c2] - u[c2] * u[3 + c1]);
    }
  }
  // forward hop uses (1 - gamma), backward (1 + gamma); D^dag swaps them
  const C s = (FWD != DAG) ? C(-1) : C(1);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    cplx<C> chi[12], h[6], w[6];
#pragma unroll
    for (int k = 0; k < 12; ++k) chi[k] = ldc(in, sp_idx(rhs0 + r, k, nb_site, V));
    project<MU>(chi, s, h);
    su3_mul<C, !FWD>(u, h, w);
    reconstruct<MU>(acc[r], w, s, coef);
  }
}

// acc[r] += A(x) v[r] for NR right-hand sides, A(x) the site's packed site term: per chirality
// 18 complex entries at A[(alpha * 18 + e) * V + x], e = 0..2 the real diagonal in pairs
// (re: entry 2e, im: entry 2e+1) and e = 3..17 the upper triangle row by row; the lower
// triangle is its conjugate.  Each entry is loaded once for all NR right-hand sides.
template <class S, int NR>
__device__ inline void clover_acc(const S* __restrict__ A, int site, int V, const cplx<ctype<S>> (*v)[12],
                                  cplx<ctype<S>> (*acc)[12]) {
  using C = ctype<S>;
#pragma unroll
  for (int al = 0; al < 2; ++al) {
    const S* b = A + size_t(al) * 18 * V + site;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const cplx<C> d = ldc(b, size_t(e) * V);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        acc[r][6 * al + 2 * e] += d.re * v[r][6 * al + 2 * e];
        acc[r][6 * al + 2 * e + 1] += d.im * v[r][6 * al + 2 * e + 1];
      }
    }
    int e = 3;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int j = i + 1; j < 6; ++j, ++e) {
        const cplx<C> o = ldc(b, size_t(e) * V);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          acc[r][6 * al + i] += o * v[r][6 * al + j];
          acc[r][6 * al + j] += cmul_conj(o, v[r][6 * al + i]);
        }
      }
  }
}

// Rows I0 .. I0+2 of one chirality block of the packed site term (layout of clover_acc)
// applied to that chirality's six spinor components x; compile-time row indices.
template <class S, int I0>
__device__ inline void site_term_rows(const S* __restrict__ b, int V, const cplx<ctype<S>> (&x)[6],
                                      cplx<ctype<S>> (&y)[3]) {
  using C = ctype<S>;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int i = I0 + q;
    const cplx<C> dd = ldc(b, size_t(i >> 1) * V);
    cplx<C> v = ((i & 1) ? dd.im : dd.re) * x[i];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      if (j == i) continue;
      const int lo = i < j ? i : j, hi = i < j ? j : i;
      const cplx<C> o = ldc(b, size_t(3 + lo * (11 - lo) / 2 + (hi - lo - 1)) * V);
      v += (i < j) ? o * x[j] : cmul_conj(o, x[j]);
    }
    y[q] = v;
  }
}

}  // namespace
}  // namespace qmg
