// Two neighbouring sites per thread in FP32 storage: loads, hops and the site term shared by the
// stencils of hop_pair.hip and dslash_pair.hip.
#pragma once

#include "qmg_internal.hpp"

namespace qmg {
namespace {

typedef cplx<float> cf;
struct Two {  // one number of each of the two sites
  cf a, b;
};
// p is uniform over the workgroup, off a byte offset of the thread.  The plane's address is pinned to scalar
// registers: combined with the offsets of the thread, addresses took 64-bit additions and two vector
// registers each
typedef const __attribute__((address_space(1))) char* gptr;
template <class T>
__device__ inline T at_off(const float2* p, unsigned off) {
  gptr g = (gptr)p;
  asm("" : "+s"(g));
  return *reinterpret_cast<const __attribute__((address_space(1))) T*>(g + off);
}
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
__device__ inline Two ld2(const float2* p, unsigned off) {
  const f4v v = at_off<f4v>(p, off);
  return {{v.x, v.y}, {v.z, v.w}};
}
__device__ inline cf ld1(const float2* p, unsigned off) {
  const f2v v = at_off<f2v>(p, off);
  return {v.x, v.y};
}
__device__ inline cf pick(bool c, cf x, cf y) { return {c ? x.re : y.re, c ? x.im : y.im}; }

// acc += coef [ 1 ; s A_mu^dag ] u h(chi), chi the four spins of one colour, u that colour's column
template <int MU>
__device__ inline void add_hop(const cf* chi, const cf* u, float s, float coef, cf* acc) {
  cf h0, h1;
  if (MU == 0) {
    h0 = chi[0] + s * times_mi(chi[3]);
    h1 = chi[1] + s * times_mi(chi[2]);
  } else if (MU == 1) {
    h0 = chi[0] - s * chi[3];
    h1 = chi[1] + s * chi[2];
  } else if (MU == 2) {
    h0 = chi[0] + s * times_mi(chi[2]);
    h1 = chi[1] + s * times_i(chi[3]);
  } else {
    h0 = chi[0] + s * chi[2];
    h1 = chi[1] + s * chi[3];
  }
  h0 = coef * h0;
  h1 = coef * h1;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cf w0 = u[a] * h0, w1 = u[a] * h1;
    acc[a] += w0;
    acc[3 + a] += w1;
    if (MU == 0) {
      acc[6 + a] += s * times_i(w1);
      acc[9 + a] += s * times_i(w0);
    } else if (MU == 1) {
      acc[6 + a] += s * w1;
      acc[9 + a] -= s * w0;
    } else if (MU == 2) {
      acc[6 + a] += s * times_i(w0);
      acc[9 + a] += s * times_mi(w1);
    } else {
      acc[6 + a] += s * w0;
      acc[9 + a] += s * w1;
    }
  }
}

// Sums over hops and colours.  A component of the result has 24 terms, eight hops of three colours; added one
// to another they would be rounded 24 times at up to the size of the whole.  The hops of a colour are summed by
// themselves (t: the space directions, which have one weight, without it, then weight and time hops) and
// the three colours' sums after that (w), so that the error is that of eight whole hops.  FP32 at xi = 1 / 3.5:
// D 6.64e-8 / 5.53e-8 -> 5.99e-8 / 4.42e-8, Schur complement 6.40e-8 / 5.24e-8 -> 6.01e-8 / 4.26e-8 (whole hops, one
// site per thread: 6.00e-8 / 4.43e-8 and 6.01e-8 / 4.28e-8).
// The registers do not hold both sums of two right-hand sides: PARK packs of two numbers of w wait in the LDS, each
// in a slot of its thread (16 bytes per lane), the others are pinned in registers between the colours, or the
// compiler would put off the arithmetic of one colour to the next and keep that colour's loads instead (800 spilled).
constexpr int kPairBlock = 256;
// pack c: numbers k, k + 1 of a site, added after colour b
template <int PARK>
__device__ inline void add_pack(int c, int b, cf t0, cf t1, cf& w0, cf& w1, float4 (*park)[kPairBlock]) {
  if (b) {
    if (c < PARK) {
      const float4 o = park[c][threadIdx.x];
      w0 = {o.x, o.y};
      w1 = {o.z, o.w};
    }
    t0 = w0 + t0;
    t1 = w1 + t1;
  }
  if (c < PARK && b < 2) {
    park[c][threadIdx.x] = {t0.re, t0.im, t1.re, t1.im};
  } else {
    w0 = t0;
    w1 = t1;
    asm volatile("" : "+v"(w0.re), "+v"(w0.im), "+v"(w1.re), "+v"(w1.im));
  }
}
// acc += A v on the pair's sites, A the packed site term (layout of clover_acc)
template <int NR>
__device__ inline void site_term(const float2* A, unsigned off, size_t Vh, const cf (*va)[12], const cf (*vb)[12],
                                 cf (*aa)[12], cf (*ab)[12]) {
#pragma unroll
  for (int al = 0; al < 2; ++al) {
    const float2* p = A + size_t(al) * 18 * Vh;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const Two d = ld2(p + e * Vh, off);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int k = 6 * al + 2 * e;
        aa[r][k] += d.a.re * va[r][k];
        aa[r][k + 1] += d.a.im * va[r][k + 1];
        ab[r][k] += d.b.re * vb[r][k];
        ab[r][k + 1] += d.b.im * vb[r][k + 1];
      }
    }
    int e = 3;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int j = i + 1; j < 6; ++j, ++e) {
        const Two o = ld2(p + e * Vh, off);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          aa[r][6 * al + i] += o.a * va[r][6 * al + j];
          aa[r][6 * al + j] += cmul_conj(o.a, va[r][6 * al + i]);
          ab[r][6 * al + i] += o.b * vb[r][6 * al + j];
          ab[r][6 * al + j] += cmul_conj(o.b, vb[r][6 * al + i]);
        }
      }
  }
}

}  // namespace
}  // namespace qmg
