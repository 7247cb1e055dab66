// D and D^dagger (and the clover forms) on fields in the canonical layouts, gauge [mu][V][3][3] and
// spinor [rhs][V][4][3].
//
// The canonical layouts put a site's numbers side by side, so one thread per site strides by a
// whole site (192 bytes in FP64) from lane to lane: every load of a wavefront touches 64 cache
// lines, and the load pipe, not memory, sets the time.  Here a wavefront reads the spinors (and
// links) of 64 sites in address order, 16 bytes per lane, and hands them out through its own
// part of the LDS.  A workgroup covers 64 consecutive sites; wavefront mu forms the two hops along
// mu, holds its two links in registers over all right-hand sides of the group, the partial spinors
// of the four directions meet in the LDS and wavefront w finishes components 3w .. 3w+2.  Measured against one
// thread per site, FP64: 16^3 x 32 with 1 / 12 right-hand sides 48 -> 39 / 540 -> 321 us; where one thread per site stays
// stands at canon_site.
#include <algorithm>
#include <type_traits>

#include "stencil.hpp"
#include "timing.hpp"

namespace qmg {

namespace {

constexpr int kSites = 64;  // sites per workgroup

// number at byte offset off of a thread from a pointer that is uniform over the workgroup (OFF is
// 64 bits wide on lattices whose fields pass 4 GB)
template <class T, class S, class OFF>
__device__ inline T raw(const S* p, OFF off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + off);
}

// Packs of P numbers (16 bytes where the field's alignment allows it: a load of 8 bytes per lane
// occupies the load pipe as long as one of 16), NP of them per site.  The wavefront reads those of 64
// sites in address order (offsets: byte offsets of packs j * 64 + lane, pack q of site nb at
// nb * NP + q), and land hands them through the LDS to the lane of their site; the stride of NP | 1
// packs (NP + 1 for even NP) keeps the lanes off each other's banks.
template <class S, int P, int NP, class OFF>
__device__ inline void offsets(int nb, int lane, OFF (&off)[NP]) {
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const int e = j * 64 + lane;
    off[j] = OFF(P * sizeof(S)) * (OFF(__shfl(nb, e / NP)) * NP + OFF(e % NP));
  }
}
template <class S, int P, int NP, class OFF>
__device__ inline void issue(const S* p, const OFF (&off)[NP], Pk<S, P> (&t)[NP]) {
#pragma unroll
  for (int j = 0; j < NP; ++j) t[j] = raw<Pk<S, P>>(p, off[j]);
}
template <class S, int P, int NP>
__device__ inline void land(const Pk<S, P> (&t)[NP], void* smem, int lane, cplx<ctype<S>>* v) {
  Pk<S, P>* lds = static_cast<Pk<S, P>*>(smem);
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const int e = j * 64 + lane;
    lds[(e / NP) * (NP | 1) + e % NP] = t[j];
  }
  __builtin_amdgcn_wave_barrier();  // the LDS takes one wavefront's accesses in order
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const Pk<S, P> w = lds[lane * (NP | 1) + q];
#pragma unroll
    for (int i = 0; i < P; ++i) v[P * q + i] = StoreTraits<S>::ld(w.v[i]);
  }
  __builtin_amdgcn_wave_barrier();
}

template <class S, int P, class OFF, int MU, bool DAG>
__device__ inline void hops(const cplx<ctype<S>>* uf, const cplx<ctype<S>>* ub, const S* in, const OFF (&of)[12 / P],
                            const OFF (&ob)[12 / P], void* lds, int lane, ctype<S> cf, ctype<S> cb,
                            cplx<ctype<S>>* acc) {
  using C = ctype<S>;
  const C sf = DAG ? C(1) : C(-1);
  Pk<S, P> tf[12 / P], tb[12 / P];
  cplx<C> chi[12], h[6], w[6];
  issue(in, of, tf);
  if (sizeof(C) == 4) issue(in, ob, tb);  // both in flight; in FP64 there are no registers for that
  land<S>(tf, lds, lane, chi);
  project<MU>(chi, sf, h);
  su3_mul<C, false>(uf, h, w);
  reconstruct<MU>(acc, w, sf, cf);
  if (sizeof(C) == 8) issue(in, ob, tb);
  land<S>(tb, lds, lane, chi);
  project<MU>(chi, -sf, h);
  su3_mul<C, true>(ub, h, w);
  reconstruct<MU>(acc, w, -sf, cb);
}

template <class S, int P, class OFF, bool DAG, bool CLOV>
__global__ __launch_bounds__(256, sizeof(S) == 16 ? 2 : 1) void k_dslash_canon(const S* __restrict__ U, const S* __restrict__ in,
                                                      S* __restrict__ out, DslashArgs a, int ngroup) {
  using C = ctype<S>;
  constexpr int NP = 12 / P;
  constexpr int kSpin = 64 * (NP | 1) * P * int(sizeof(S)), kSum = 12 * 64 * int(sizeof(cplx<C>));
  constexpr int kLink = 64 * 9 * int(sizeof(S));
  constexpr int kWave = std::max(std::max(kSpin, kSum), kLink);
  __shared__ __align__(16) char smem[4][kWave];
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  const int tile = wg / ngroup, grp = wg - tile * ngroup;
  const int r0 = int(long(grp) * a.nrhs / ngroup), r1 = int(long(grp + 1) * a.nrhs / ngroup);
  const int lane = threadIdx.x & 63;
  const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int V = a.V;
  const bool live = tile * kSites + lane < V;
  const int site = live ? tile * kSites + lane : V - 1;  // the last tile's idle lanes repeat a site
  void* lds = smem[mu];
  cplx<C>* mine = reinterpret_cast<cplx<C>*>(smem[mu]);
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  int rem = site;
  const int x = rem % L0; rem /= L0;
  const int y = rem % L1; rem /= L1;
  const int z = rem % L2;
  const int t = rem / L2;
  int c, L, st;
  if (mu == 0) { c = x; L = L0; st = 1; }
  else if (mu == 1) { c = y; L = L1; st = L0; }
  else if (mu == 2) { c = z; L = L2; st = L0 * L1; }
  else { c = t; L = L3; st = L0 * L1 * L2; }
  const int fp = (c + 1 == L) ? site - (L - 1) * st : site + st;
  const int bm = (c == 0) ? site + (L - 1) * st : site - st;
  C cw, diag;
  if constexpr (sizeof(C) == 8) {
    cw = a.cw_d[mu];
    diag = a.diag_d;
  } else {
    cw = a.cw_f[mu];
    diag = a.diag_f;
  }
  C cf = C(-0.5) * cw, cb = cf;
  if (mu == 3 && a.bc_t < 0) {
    if (t == L3 - 1) cf = -cf;
    if (t == 0) cb = -cb;
  }
  cplx<C> uf[9], ub[9];
  {
    OFF o[9], p[9];
    Pk<S, 1> tf[9], tb[9];
    const S* um = U + size_t(mu) * V * 9;
    offsets<S, 1, 9>(site, lane, o);
    offsets<S, 1, 9>(bm, lane, p);
    issue(um, o, tf);
    if (sizeof(C) == 4) issue(um, p, tb);
    land<S>(tf, lds, lane, uf);
    if (sizeof(C) == 8) issue(um, p, tb);
    land<S>(tb, lds, lane, ub);
  }
  OFF of[NP], ob[NP];
  offsets<S, P, NP>(fp, lane, of);
  offsets<S, P, NP>(bm, lane, ob);
  const OFF own = OFF(sizeof(S)) * OFF(site) * 12;
#pragma unroll 1
  for (int r = r0; r < r1; ++r) {
    const S* inr = in + size_t(r) * V * 12;
    S* outr = out + size_t(r) * V * 12;
    cplx<C> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = {C(0), C(0)};
    switch (mu) {  // uniform in the wavefront
      case 0: hops<S, P, OFF, 0, DAG>(uf, ub, inr, of, ob, lds, lane, cf, cb, acc); break;
      case 1: hops<S, P, OFF, 1, DAG>(uf, ub, inr, of, ob, lds, lane, cf, cb, acc); break;
      case 2: hops<S, P, OFF, 2, DAG>(uf, ub, inr, of, ob, lds, lane, cf, cb, acc); break;
      default: hops<S, P, OFF, 3, DAG>(uf, ub, inr, of, ob, lds, lane, cf, cb, acc); break;
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) mine[k * kSites + lane] = acc[k];
    cplx<C> own3[3];  // of this wavefront's components: the site term's, or the spinor's numbers
    if constexpr (CLOV) {
      // rows 3 (mu & 1) .. +2 of chirality mu >> 1
      const int al = mu >> 1;
      cplx<C> xv[6];
#pragma unroll
      for (int j = 0; j < 6; ++j) xv[j] = StoreTraits<S>::ld(raw<S>(inr + 6 * al + j, own));
      const S* b = static_cast<const S*>(a.clov) + size_t(al) * 18 * V + site;
      if (mu & 1) site_term_rows<S, 3>(b, V, xv, own3);
      else site_term_rows<S, 0>(b, V, xv, own3);
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q) own3[q] = StoreTraits<S>::ld(raw<S>(inr + 3 * mu + q, own));
    }
    __syncthreads();
    cplx<C> v[3];
    auto part = [&](int m, int k) { return reinterpret_cast<const cplx<C>*>(smem[m])[k * kSites + lane]; };
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int k = 3 * mu + q;
      const cplx<C> p0 = part(0, k), p1 = part(1, k), p2 = part(2, k), p3 = part(3, k);
      if constexpr (sizeof(C) == 8 && !CLOV)
        v[q] = {sum_compensated(p0.re, p1.re, p2.re, p3.re, diag, own3[q].re),
                sum_compensated(p0.im, p1.im, p2.im, p3.im, diag, own3[q].im)};
      else
        v[q] = sum_directions<S>(p0, p1, p2, p3, CLOV ? C(1) : diag, own3[q]);
    }
    __syncthreads();
    if (live) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
        *reinterpret_cast<S*>(reinterpret_cast<char*>(outr + 3 * mu + q) + own) = StoreTraits<S>::st(v[q]);
    }
  }
}

// One thread per site and right-hand side; the rule stands at canon_site.
template <class S, int MU, bool FWD, bool DAG>
__device__ inline void site_hop(const S* __restrict__ U, const S* __restrict__ in, cplx<ctype<S>>* acc, int link_site,
                                int nb_site, int rhs, int V, ctype<S> coef) {
  using C = ctype<S>;
  cplx<C> u[9], chi[12], h[6], w[6];
  const C s = (FWD != DAG) ? C(-1) : C(1);
#pragma unroll
  for (int e = 0; e < 9; ++e) u[e] = ldc(U, (size_t(MU) * V + link_site) * 9 + e);
#pragma unroll
  for (int k = 0; k < 12; ++k) chi[k] = ldc(in, (size_t(rhs) * V + nb_site) * 12 + k);
  project<MU>(chi, s, h);
  su3_mul<C, !FWD>(u, h, w);
  reconstruct<MU>(acc, w, s, coef);
}

template <class S, bool DAG, bool CLOV>
__global__ __launch_bounds__(256) void k_dslash_canon_site(const S* __restrict__ U, const S* __restrict__ in,
                                                           S* __restrict__ out, DslashArgs a) {
  using C = ctype<S>;
  // the right-hand sides of a tile next to each other on one XCD: they share its links in the L2
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  const int tile = wg / a.nrhs, rhs = wg - tile * a.nrhs;
  const int site = tile * 256 + threadIdx.x;
  const int V = a.V;
  if (site >= V) return;
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  int rem = site;
  const int x = rem % L0; rem /= L0;
  const int y = rem % L1; rem /= L1;
  const int z = rem % L2;
  const int t = rem / L2;
  const int s1 = L0, s2 = L0 * L1, s3 = L0 * L1 * L2;
  const int xp = (x + 1 == L0) ? site - (L0 - 1) : site + 1;
  const int xm = (x == 0) ? site + (L0 - 1) : site - 1;
  const int yp = (y + 1 == L1) ? site - (L1 - 1) * s1 : site + s1;
  const int ym = (y == 0) ? site + (L1 - 1) * s1 : site - s1;
  const int zp = (z + 1 == L2) ? site - (L2 - 1) * s2 : site + s2;
  const int zm = (z == 0) ? site + (L2 - 1) * s2 : site - s2;
  const int tp = (t + 1 == L3) ? site - (L3 - 1) * s3 : site + s3;
  const int tm = (t == 0) ? site + (L3 - 1) * s3 : site - s3;
  C cw[4], diag;
  if constexpr (sizeof(C) == 8) {
    for (int m = 0; m < 4; ++m) cw[m] = a.cw_d[m];
    diag = a.diag_d;
  } else {
    for (int m = 0; m < 4; ++m) cw[m] = a.cw_f[m];
    diag = a.diag_f;
  }
  const C mh = C(-0.5);
  const C bt_f = (a.bc_t < 0 && t == L3 - 1) ? C(-1) : C(1), bt_b = (a.bc_t < 0 && t == 0) ? C(-1) : C(1);
  cplx<C> acc[1][12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[0][k] = {C(0), C(0)};
  site_hop<S, 0, true, DAG>(U, in, acc[0], site, xp, rhs, V, mh * cw[0]);
  site_hop<S, 0, false, DAG>(U, in, acc[0], xm, xm, rhs, V, mh * cw[0]);
  site_hop<S, 1, true, DAG>(U, in, acc[0], site, yp, rhs, V, mh * cw[1]);
  site_hop<S, 1, false, DAG>(U, in, acc[0], ym, ym, rhs, V, mh * cw[1]);
  site_hop<S, 2, true, DAG>(U, in, acc[0], site, zp, rhs, V, mh * cw[2]);
  site_hop<S, 2, false, DAG>(U, in, acc[0], zm, zm, rhs, V, mh * cw[2]);
  site_hop<S, 3, true, DAG>(U, in, acc[0], site, tp, rhs, V, mh * cw[3] * bt_f);
  site_hop<S, 3, false, DAG>(U, in, acc[0], tm, tm, rhs, V, mh * cw[3] * bt_b);
  if constexpr (CLOV) {
    cplx<C> v[1][12];
#pragma unroll
    for (int k = 0; k < 12; ++k) v[0][k] = ldc(in, (size_t(rhs) * V + site) * 12 + k);
    clover_acc<S, 1>(static_cast<const S*>(a.clov), site, V, v, acc);
#pragma unroll
    for (int k = 0; k < 12; ++k) stc(out, (size_t(rhs) * V + site) * 12 + k, acc[0][k]);
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const size_t i = (size_t(rhs) * V + site) * 12 + k;
      cplx<C> v = ldc(in, i);
      stc(out, i, diag * v + acc[0][k]);
    }
  }
}

// Where one thread per site and right-hand side is the faster form, us, that / four directions.  Four directions
// pass everything through the LDS, which costs latency that few waves hide, and keep a tile's links over
// several right-hand sides.  w: sites x right-hand sides.
// FP32: a single right-hand side below 2^19 sites (16^3 x 32 16.4 / 20.6, 24^3 x 48 108 / 99); several for w
// between 2^14 and 3 2^16 (10^3 x 16 with 2 6.8 / 7.4, 8^3 x 16 with 12 11.8 / 15.0, 10^3 x 16 with 12 21.4 / 28.7;
// beyond 6^3 x 8 with 8 6.5 / 5.9, 15 x 17 x 19 x 21 with 2 30.1 / 27.4, 12^3 x 24 with 8 40.0 / 36.3), with the
// site term up to 5 2^16 (12^3 x 24 with 5 32.6 / 34.6, 16^3 x 32 with 2 39.7 / 40.2, with 3 55.4 / 53.3).
// FP16, whose site form needs 89 registers: a single one always (24^3 x 48 39 / 61), several for w between 2^15 and
// 2^22 (12^3 x 24 with 2 8.7 / 11.2, 24^3 x 48 with 3 114 / 129; beyond 24^3 x 48 with 8 318 / 318).  BF16, whose
// site form takes 256: never (16^3 x 32 with 1 16.5 / 16.0, 24^3 x 48 with 2 168 / 105).
// FP64: four directions (16^3 x 32 48 / 38), but the site term spills beside the held links: with it a single one
// from 2^15 sites (12^3 x 24 23.6 / 25.9, 24^3 x 48 371 / 392; 8^3 x 16 15.6 / 9.2), two on 2^17 sites or more (16^3 x 32
// 101 / 107, 24^3 x 48 634 / 630), and several where the site form's workgroups nearly fill up to three rounds of the 256
// CUs (12^3 x 16 with 2, 0.84 rounds, 24.0 / 28.8; 12^3 x 24 with 3, 1.9, 48.9 / 54.0; with 2, 1.3, 42.9 / 40.9; 14^3 x 28
// with 3, 3.5, 94 / 85).
template <class S>
bool canon_site(const DslashArgs& a) {
  const long w = long(a.V) * a.nrhs, one = 1;
  switch (StoreTraits<S>::prec) {
    case QMG_F64: {
      if (!a.clov) return false;
      if (a.nrhs == 1 ? w >= (one << 15) : a.nrhs == 2 && w >= (one << 18)) return true;
      const long tiles = (w + 255) / 256, rounds = (tiles + 255) / 256;
      return rounds <= 3 && tiles >= 256 * rounds - 90;
    }
    case QMG_F32:
      return a.nrhs == 1 ? w < (one << 19) : w > (one << 14) && w < ((a.clov ? 5 : 3) * one << 16);
    case QMG_F16:
      return a.nrhs == 1 || (w > (one << 15) && w < (one << 22));
    default:
      return false;
  }
}

template <class S>
void launch_canon(const S* U, const S* in, S* out, const DslashArgs& a, hipStream_t st) {
  const bool wide = size_t(a.V) * 12 * sizeof(S) >= (size_t(1) << 32);
  const int ntile = (a.V + kSites - 1) / kSites;
  // a group keeps its links over its right-hand sides; small lattices are cut into more groups, up
  // to 2048 workgroups, as even as they go (16^3 x 32, 12 rhs FP64: 316 us with one group, 393 us with two)
  const int most = std::max(1, std::min(a.nrhs, 2048 / ntile)), per = (a.nrhs + most - 1) / most;
  const int ngroup = (a.nrhs + per - 1) / per;
  const dim3 grid(unsigned(ntile) * unsigned(ngroup));
  auto go = [&](auto dag, auto clov) {
    constexpr bool D = decltype(dag)::value, CL = decltype(clov)::value;
    if constexpr (StoreTraits<S>::prec != QMG_BF16 && (sizeof(S) < 16 || CL)) {
      if (canon_site<S>(a)) {
        launch(k_dslash_canon_site<S, D, CL>, dim3(unsigned((a.V + 255) / 256) * unsigned(a.nrhs)), dim3(256), 0, st, U,
               in, out, a);
        return;
      }
    }
    constexpr int P = int(16 / sizeof(S));
    if (wide) launch(k_dslash_canon<S, 1, size_t, D, CL>, grid, dim3(256), 0, st, U, in, out, a, ngroup);
    else if (reinterpret_cast<uintptr_t>(in) & 15)
      launch(k_dslash_canon<S, 1, unsigned, D, CL>, grid, dim3(256), 0, st, U, in, out, a, ngroup);
    else launch(k_dslash_canon<S, P, unsigned, D, CL>, grid, dim3(256), 0, st, U, in, out, a, ngroup);
  };
  using T = std::true_type;
  using F = std::false_type;
  if (a.clov) a.dagger ? go(T{}, T{}) : go(F{}, T{});
  else a.dagger ? go(T{}, F{}) : go(F{}, F{});
  QMG_LAUNCH_CHECK();
}

}  // namespace

void launch_dslash_canonical(qmg_prec prec, const void* U, const void* in, void* out, const DslashArgs& a,
                             hipStream_t st) {
  const double cb = double(prec_bytes(prec));
  const double bytes = double(a.V) * (24.0 * a.nrhs + 36.0 + (a.clov ? 36.0 : 0.0)) * cb;
  const double flops = (a.clov ? 1872.0 : 1368.0) * a.V * a.nrhs;
  TimedLaunch tl(a.clov ? "clover/canonical" : "dslash/canonical", st, bytes, flops);
  auto go = [&](auto tag) {
    using S = decltype(tag);
    launch_canon<S>(static_cast<const S*>(U), static_cast<const S*>(in), static_cast<S*>(out), a, st);
  };
  switch (prec) {
    case QMG_F64: go(double2{}); break;
    case QMG_F32: go(float2{}); break;
    case QMG_BF16: go(cbf16{}); break;
    case QMG_F16: go(chalf{}); break;
  }
}

}  // namespace qmg
