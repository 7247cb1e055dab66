// Wilson-Dirac stencil D and D^dagger (the operator of Eq. (1)), site-parallel.
//
// Every hop uses the rank-2 spin projection of (1 +/- gamma_mu) in the chiral basis
// gamma_mu = [[0, A_mu], [A_mu^dag, 0]] (A_x = -i sigma_1, A_y = -i sigma_2,
// A_z = -i sigma_3, A_t = 1):
//   (1 + s gamma_mu) chi = [ h ; s A_mu^dag h ],  h = chi_up + s A_mu chi_down,
// so a hop multiplies two colour vectors by the link instead of four.  Bandwidth bound:
// per site and right-hand side the algorithm reads the spinor once (24 reals), the four
// forward links once (72 reals, shared across right-hand sides) and writes 24 reals.
//
// With the clover term the site-local part of the operator, (m + 1 + 3/xi) + T(x), is two
// hermitian 6 x 6 blocks per site (T commutes with gamma_5); every form then applies them in
// its epilogue in place of the scalar diagonal term (kernels instantiated with CLOV = true).
//
// Launch: one thread per (site, group of NR right-hand sides), 256 threads per workgroup.
// Workgroups are dispatched round-robin over the 8 XCDs of the MI355X; the tile index is
// remapped so that each XCD walks a contiguous range of sites, keeping the +-t neighbour
// slices of a tile inside that XCD's L2.
#include <string>
#include <type_traits>

#include "stencil.hpp"
#include "timing.hpp"
#include "tune.hpp"

namespace qmg {

namespace {
int g_variant = 0;  // forced native-layout launch variant (0: heuristic or tuned)
}

void set_dslash_variant(int v) { g_variant = v; }

DslashArgs make_dslash_args(const Geom& g, int nrhs, bool dagger, bool canonical) {
  DslashArgs a{};
  a.tchunk = g_variant;
  for (int m = 0; m < 4; ++m) a.L[m] = g.L[m];
  a.V = g.V;
  a.bc_t = g.bc_t;
  a.diag_d = g.diag();
  a.diag_f = float(a.diag_d);
  for (int m = 0; m < 4; ++m) {
    a.cw_d[m] = g.cw(m);
    a.cw_f[m] = float(a.cw_d[m]);
  }
  a.nrhs = nrhs;
  a.dagger = dagger ? 1 : 0;
  a.canonical = canonical ? 1 : 0;
  a.clov = nullptr;
  a.link_ne = 9;
  return a;
}

namespace {

// D (or D^dag) at one site for NR right-hand sides starting at rhs0
template <class S, int NR, bool DAG, bool CLOV = false>
__device__ inline void site_dslash(const S* __restrict__ U, const S* __restrict__ in, S* __restrict__ out,
                                   const DslashArgs& a, int site, int rhs0) {
  using C = ctype<S>;
  const int V = a.V;
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
  const C bt_f = (a.bc_t < 0 && t == L3 - 1) ? C(-1) : C(1);
  const C bt_b = (a.bc_t < 0 && t == 0) ? C(-1) : C(1);

  cplx<C> acc[NR][12];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[r][k] = {C(0), C(0)};

  const C mh = C(-0.5);
  do_hop<S, NR, 0, true, DAG>(U, in, acc, site, xp, rhs0, V, mh * cw[0]);
  do_hop<S, NR, 0, false, DAG>(U, in, acc, xm, xm, rhs0, V, mh * cw[0]);
  do_hop<S, NR, 1, true, DAG>(U, in, acc, site, yp, rhs0, V, mh * cw[1]);
  do_hop<S, NR, 1, false, DAG>(U, in, acc, ym, ym, rhs0, V, mh * cw[1]);
  do_hop<S, NR, 2, true, DAG>(U, in, acc, site, zp, rhs0, V, mh * cw[2]);
  do_hop<S, NR, 2, false, DAG>(U, in, acc, zm, zm, rhs0, V, mh * cw[2]);
  do_hop<S, NR, 3, true, DAG>(U, in, acc, site, tp, rhs0, V, mh * cw[3] * bt_f);
  do_hop<S, NR, 3, false, DAG>(U, in, acc, tm, tm, rhs0, V, mh * cw[3] * bt_b);

  if constexpr (CLOV) {
    cplx<C> v[NR][12];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) v[r][k] = ldc(in, sp_idx(rhs0 + r, k, site, V));
    clover_acc<S, NR>(static_cast<const S*>(a.clov), site, V, v, acc);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) stc(out, sp_idx(rhs0 + r, k, site, V), acc[r][k]);
  } else {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const size_t i = sp_idx(rhs0 + r, k, site, V);
        cplx<C> v = ldc(in, i);
        stc(out, i, diag * v + acc[r][k]);
      }
    }
  }
}

template <class S, int NR, bool DAG, bool CLOV = false>
__global__ __launch_bounds__(kBlock) void k_dslash(const S* __restrict__ U, const S* __restrict__ in,
                                                   S* __restrict__ out, DslashArgs a) {
  // flattened grid over (tile, rhs group) with the rhs groups of a tile adjacent in the
  // XCD-local order, so that they share the tile's links in L2
  const int ng = a.nrhs / NR;
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  const int tile = wg / ng;
  const int site = tile * kBlock + threadIdx.x;
  if (site >= a.V) return;
  site_dslash<S, NR, DAG, CLOV>(U, in, out, a, site, (wg - tile * ng) * NR);
}

// Many lattices in one launch: workgroup (after the XCD remap) w belongs to the lattice whose
// tile range [tile0, tile0 + ntiles * nrhs) holds it; every lattice has its own extents,
// coefficients, gauge field and spinors (native layout).
template <class S, bool DAG>
__global__ __launch_bounds__(kBlock) void k_dslash_batched(const BatchLattice* __restrict__ lat, int n_lat,
                                                           const S* const* __restrict__ U,
                                                           const S* const* __restrict__ in,
                                                           S* const* __restrict__ out) {
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  int lo = 0, hi = n_lat - 1;  // last lattice with tile0 <= wg
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (lat[mid].tile0 <= wg) lo = mid;
    else hi = mid - 1;
  }
  const BatchLattice& b = lat[lo];
  const int local = wg - b.tile0;
  const int ntile = (b.a.V + kBlock - 1) / kBlock;
  const int rhs = local / ntile, tile = local - rhs * ntile;
  const int site = tile * kBlock + threadIdx.x;
  if (site >= b.a.V) return;
  site_dslash<S, 1, DAG>(U[lo], in[lo], out[lo], b.a, site, rhs);
}

// Many lattices in padded layouts (one hierarchy over many small lattices): lattice l's links at
// U + l * 36 Vpad ([4][9][Vpad]) and its nr spinors at in / out + l * nr * 12 Vpad
// ([nr][12][Vpad]); lat[l].a carries the lattice's extents and coefficients with a.V = Vpad (the
// stride).  Grid: nl * nr * ceil(Vpad / 256) workgroups; sites at and beyond the lattice's
// volume are written as zeros, so every output column is zero-padded.
// A thread forms NR right-hand sides of its site (links loaded once for all of them); the
// groups of a tile are adjacent in the schedule.
template <class S, bool DAG, int NR>
__global__ __launch_bounds__(kBlock) void k_dslash_padded(const BatchLattice* __restrict__ lat, const S* __restrict__ U,
                                                          const S* __restrict__ in, S* __restrict__ out, int nr,
                                                          int ntile) {
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  const int ng = nr / NR;
  const int g = wg % ng, tc = wg / ng;
  const int tile = tc % ntile, l = tc / ntile;
  const int rhs0 = g * NR;
  const DslashArgs& a = lat[l].a;
  const int Vpad = a.V;
  const int site = tile * kBlock + threadIdx.x;
  if (site >= Vpad) return;
  const size_t base = size_t(l) * nr * 12 * Vpad;
  if (site >= a.L[0] * a.L[1] * a.L[2] * a.L[3]) {
    for (int r = 0; r < NR; ++r)
      for (int k = 0; k < 12; ++k) stc(out + base, sp_idx(rhs0 + r, k, site, Vpad), cplx<ctype<S>>{0, 0});
    return;
  }
  site_dslash<S, NR, DAG>(U + size_t(l) * 36 * Vpad, in + base, out + base, a, site, rhs0);
}

// Native-layout kernel that walks along t.  Thread (spatial site, t-chunk, group of NR
// right-hand sides) computes the TCH sites t0 .. t0+TCH-1 of its column for NR right-hand
// sides; each link is loaded once for all NR of them.  The spinor of the next slice, loaded
// for the forward t-hop, becomes the own spinor of the next step, and the backward t-hop
// U_t(x, t-1)^dag (1 + gamma_t) psi(x, t-1) is formed from the own spinor and forward t-link
// of the previous step, so t-neighbours and t-links are read once.  Workgroups are 256
// spatial sites of one (t-chunk, rhs group); the rhs groups of a tile are adjacent in the
// XCD-local schedule so that they share its links in L2.  Tiles are 256 consecutive spatial
// sites, or (zfast) 256-site pieces of one xy-plane with z fastest in the schedule, so that
// the tiles holding a site's z-neighbours run next to it.
template <class S, int TCH, int NR, bool DAG, bool CLOV = false>
__global__ __launch_bounds__(kBlock) void k_dslash_t(const S* __restrict__ U, const S* __restrict__ in,
                                                     S* __restrict__ out, DslashArgs a, int ntile_s, int zfast,
                                                     int cmaj) {
  using C = ctype<S>;
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  const int Vs = L0 * L1 * L2, V = a.V;
  const int ng = a.nrhs / NR;
  const int per_chunk = ntile_s * ng;
  int wg;
  if (cmaj) {  // t-chunk major in dispatch order (all XCDs on one chunk), XCD-local tiles within it
    const int ch = blockIdx.x / per_chunk;
    wg = ch * per_chunk + xcd_tile(blockIdx.x - ch * per_chunk, per_chunk);
  } else {
    wg = xcd_tile(blockIdx.x, gridDim.x);
  }
  const int chunk = wg / per_chunk, r0 = wg - chunk * per_chunk;
  const int ts = r0 / ng, g = r0 - ts * ng;
  int xs;  // spatial site
  if (zfast) {
    const int Pxy = L0 * L1;
    const int z = ts % L2, piece = ts / L2;
    const int xy = piece * kBlock + threadIdx.x;
    if (xy >= Pxy) return;
    xs = xy + z * Pxy;
  } else {
    xs = ts * kBlock + threadIdx.x;
    if (xs >= Vs) return;
  }
  const int rhs0 = g * NR;
  const int t0 = chunk * TCH;
  int rem = xs;
  const int x = rem % L0; rem /= L0;
  const int y = rem % L1;
  const int z = rem / L1;
  const int s1 = L0, s2 = L0 * L1;
  const int dxp = (x + 1 == L0) ? -(L0 - 1) : 1, dxm = (x == 0) ? (L0 - 1) : -1;
  const int dyp = (y + 1 == L1) ? -(L1 - 1) * s1 : s1, dym = (y == 0) ? (L1 - 1) * s1 : -s1;
  const int dzp = (z + 1 == L2) ? -(L2 - 1) * s2 : s2, dzm = (z == 0) ? (L2 - 1) * s2 : -s2;
  C cw[4], diag;
  if constexpr (sizeof(C) == 8) {
    for (int m = 0; m < 4; ++m) cw[m] = a.cw_d[m];
    diag = a.diag_d;
  } else {
    for (int m = 0; m < 4; ++m) cw[m] = a.cw_f[m];
    diag = a.diag_f;
  }
  const C mh = C(-0.5);
  const C sf = DAG ? C(1) : C(-1);  // forward projector sign: (1 + sf gamma)
  const C sb = -sf;                  // backward projector sign

  // own spinors of the first site and the backward t-hops carried into them
  cplx<C> psi[NR][12], hb[NR][6];
  {
    const int tm = (t0 == 0) ? L3 - 1 : t0 - 1;
    const int sm = xs + tm * Vs;
    cplx<C> u[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = ldc(U, size_t(3 * 9 + e) * V + sm);
    const int s0 = xs + t0 * Vs;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      cplx<C> chi[12], h[6];
#pragma unroll
      for (int k = 0; k < 12; ++k) chi[k] = ldc(in, sp_idx(rhs0 + r, k, sm, V));
      project<3>(chi, sb, h);
      su3_mul<C, true>(u, h, hb[r]);
#pragma unroll
      for (int k = 0; k < 12; ++k) psi[r][k] = ldc(in, sp_idx(rhs0 + r, k, s0, V));
    }
  }
#pragma unroll 1
  for (int dt = 0; dt < TCH; ++dt) {
    const int t = t0 + dt;
    const int site = xs + t * Vs;
    const int tp = (t + 1 == L3) ? 0 : t + 1;
    const int sp = xs + tp * Vs;
    cplx<C> acc[NR][12];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) acc[r][k] = {C(0), C(0)};
    // the site term first, from the own spinors that are live anyway: each of its entries is
    // loaded once for all NR right-hand sides and nothing more stays live for the epilogue
    if constexpr (CLOV) clover_acc<S, NR>(static_cast<const S*>(a.clov), site, V, psi, acc);
    do_hop<S, NR, 0, true, DAG>(U, in, acc, site, site + dxp, rhs0, V, mh * cw[0]);
    do_hop<S, NR, 0, false, DAG>(U, in, acc, site + dxm, site + dxm, rhs0, V, mh * cw[0]);
    do_hop<S, NR, 1, true, DAG>(U, in, acc, site, site + dyp, rhs0, V, mh * cw[1]);
    do_hop<S, NR, 1, false, DAG>(U, in, acc, site + dym, site + dym, rhs0, V, mh * cw[1]);
    do_hop<S, NR, 2, true, DAG>(U, in, acc, site, site + dzp, rhs0, V, mh * cw[2]);
    do_hop<S, NR, 2, false, DAG>(U, in, acc, site + dzm, site + dzm, rhs0, V, mh * cw[2]);
    // backward t-hop (carried), boundary sign at t = 0
    const C bt_b = (a.bc_t < 0 && t == 0) ? C(-1) : C(1);
    const C bt_f = (a.bc_t < 0 && t == L3 - 1) ? C(-1) : C(1);
    // forward t-hop: this site's t-link and the next spinors
    cplx<C> u[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = ldc(U, size_t(3 * 9 + e) * V + site);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      reconstruct<3>(acc[r], hb[r], sb, mh * cw[3] * bt_b);
      cplx<C> nxt[12], h[6], w[6];
#pragma unroll
      for (int k = 0; k < 12; ++k) nxt[k] = ldc(in, sp_idx(rhs0 + r, k, sp, V));
      project<3>(nxt, sf, h);
      su3_mul<C, false>(u, h, w);
      reconstruct<3>(acc[r], w, sf, mh * cw[3] * bt_f);
      // backward t-hop of the next site from this site's spinor and t-link
      project<3>(psi[r], sb, h);
      su3_mul<C, true>(u, h, hb[r]);
      if constexpr (CLOV) {
#pragma unroll
        for (int k = 0; k < 12; ++k) {
          stc_stream(out, sp_idx(rhs0 + r, k, site, V), acc[r][k]);
          psi[r][k] = nxt[k];
        }
      } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) {
          stc_stream(out, sp_idx(rhs0 + r, k, site, V), diag * psi[r][k] + acc[r][k]);
          psi[r][k] = nxt[k];
        }
      }
    }
  }
}

// Direction-split native kernel: a workgroup covers 64 consecutive sites, wavefront mu forms
// the forward and backward hops along mu for those sites (mu is uniform in the wavefront, so
// there is no divergence), the four partial sums meet in LDS, and wavefront w then writes
// spinor components 3w .. 3w+2 of the 64 sites.  Four times as many threads as the site
// kernel, each with two hops in flight: for lattices too small to fill the GPU with one
// thread per site.
//
// bzt (BZ | BT << 8, or 0): where planes hold whole tiles, the tiles of BZ x BT planes (z, t) are visited
// together (t fastest, then z, then the tiles of a plane), so that the slices a tile's t-hops read are
// read by tiles running close in time.
template <class S, bool DAG, bool CLOV = false>
__global__ __launch_bounds__(kBlock) void k_dslash_dir(const S* __restrict__ U, const S* __restrict__ in,
                                                       S* __restrict__ out, DslashArgs a, int bzt) {
  using C = ctype<S>;
  constexpr int TS = kBlock / 4;  // sites per workgroup
  __shared__ cplx<C> part[4][12][TS];
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  const int ntile = (a.V + TS - 1) / TS;
  int tile = wg % ntile;
  const int rhs = wg / ntile;
  if (bzt) {
    const int BZ = bzt & 0xff, BT = bzt >> 8, tpp = (a.L[0] * a.L[1]) / TS;
    const int h = tile % tpp;
    int r = tile / tpp;
    const int tt = r % BT;
    r /= BT;
    const int zz = r % BZ;
    r /= BZ;
    const int nbz = a.L[2] / BZ;
    tile = h + tpp * ((r % nbz) * BZ + zz + a.L[2] * ((r / nbz) * BT + tt));
  }
  const int lane = threadIdx.x & (TS - 1), mu = threadIdx.x / TS;
  const int site = tile * TS + lane;
  const bool live = site < a.V;
  const int V = a.V;
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  const S* inr = in + size_t(rhs) * 12 * V;
  S* outr = out + size_t(rhs) * 12 * V;
  C cw, diag;
  if constexpr (sizeof(C) == 8) {
    cw = a.cw_d[mu];
    diag = a.diag_d;
  } else {
    cw = a.cw_f[mu];
    diag = a.diag_f;
  }
  const C mh = C(-0.5);
  cplx<C> acc[1][12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[0][k] = {C(0), C(0)};
  if (live) {
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
    C cf = mh * cw, cb = mh * cw;
    if (mu == 3 && a.bc_t < 0) {
      if (t == L3 - 1) cf = -cf;
      if (t == 0) cb = -cb;
    }
    switch (mu) {  // uniform within the wavefront
      case 0:
        do_hop<S, 1, 0, true, DAG>(U, inr, acc, site, fp, 0, V, cf);
        do_hop<S, 1, 0, false, DAG>(U, inr, acc, bm, bm, 0, V, cb);
        break;
      case 1:
        do_hop<S, 1, 1, true, DAG>(U, inr, acc, site, fp, 0, V, cf);
        do_hop<S, 1, 1, false, DAG>(U, inr, acc, bm, bm, 0, V, cb);
        break;
      case 2:
        do_hop<S, 1, 2, true, DAG>(U, inr, acc, site, fp, 0, V, cf);
        do_hop<S, 1, 2, false, DAG>(U, inr, acc, bm, bm, 0, V, cb);
        break;
      default:
        do_hop<S, 1, 3, true, DAG>(U, inr, acc, site, fp, 0, V, cf);
        do_hop<S, 1, 3, false, DAG>(U, inr, acc, bm, bm, 0, V, cb);
        break;
    }
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) part[mu][k][lane] = acc[0][k];
  cplx<C> own[3];  // of components 3 mu .. : the spinor's numbers, or the site term's
  if (live) {
    if constexpr (CLOV) {
      // rows 3 (mu & 1) .. +2 of chirality mu >> 1 (uniform in the wavefront)
      const int al = mu >> 1;
      cplx<C> x[6];
#pragma unroll
      for (int j = 0; j < 6; ++j) x[j] = ldc(inr, size_t(6 * al + j) * V + site);
      const S* b = static_cast<const S*>(a.clov) + size_t(al) * 18 * V + site;
      if (mu & 1) site_term_rows<S, 3>(b, V, x, own);
      else site_term_rows<S, 0>(b, V, x, own);
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q) own[q] = ldc(inr, size_t(3 * mu + q) * V + site);
    }
  }
  __syncthreads();
  if (!live) return;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int k = 3 * mu + q;
    stc(outr, size_t(k) * V + site,
        sum_directions<S>(part[0][k][lane], part[1][k][lane], part[2][k][lane], part[3][k][lane], CLOV ? C(1) : diag,
                          own[q]));
  }
}

template <class S>
void launch_dir(const void* U, const void* in, void* out, const DslashArgs& a, hipStream_t st) {
  dim3 grid(unsigned((a.V + kBlock / 4 - 1) / (kBlock / 4)) * unsigned(a.nrhs));
  // FP64 visits patches of 4 x 4 planes (16^3 x 32, one rhs: 32.6 -> 27.4 us; 8 x 24 x 20 x 30 26.7 -> 25.0; 24^3 x 48 204
  // -> 204), but not on lattices that the L2s hold anyway (8^3 x 16, 12 rhs: 16.8 -> 17.8); the
  // narrower types, whose planes are smaller against the L2, lose by it (BF16 16^3 x 32: 10.0 -> 11.8)
  auto patch = [](int L) { return L % 4 == 0 ? 4 : L % 2 == 0 ? 2 : 1; };
  const bool whole = (a.L[0] * a.L[1]) % (kBlock / 4) == 0;
  const int bzt = whole && sizeof(S) == 16 && a.V >= (1 << 15) ? patch(a.L[2]) | (patch(a.L[3]) << 8) : 0;
  auto go = [&](auto kern) { launch(kern, grid, dim3(kBlock), 0, st, U, in, out, a, bzt); };
  if (a.clov) {
    if (a.dagger) go(k_dslash_dir<S, true, true>);
    else go(k_dslash_dir<S, false, true>);
  } else if (a.dagger) {
    go(k_dslash_dir<S, true>);
  } else {
    go(k_dslash_dir<S, false>);
  }
  QMG_LAUNCH_CHECK();
}

template <class S, int NR>
void launch_t(const void* U, const void* in, void* out, const DslashArgs& a, hipStream_t st) {
  dim3 grid(unsigned((a.V + kBlock - 1) / kBlock) * unsigned(a.nrhs / NR));
  if constexpr (NR == 1) {
    if (a.clov) {
      if (a.dagger)
        launch(k_dslash<S, 1, true, true>, grid, dim3(kBlock), 0, st, U, in, out, a);
      else
        launch(k_dslash<S, 1, false, true>, grid, dim3(kBlock), 0, st, U, in, out, a);
      QMG_LAUNCH_CHECK();
      return;
    }
  }
  if (a.dagger)
    launch(k_dslash<S, NR, true>, grid, dim3(kBlock), 0, st, U, in, out, a);
  else
    launch(k_dslash<S, NR, false>, grid, dim3(kBlock), 0, st, U, in, out, a);
  QMG_LAUNCH_CHECK();
}

template <class S, int TCH, int NR>
void launch_tw(const void* U, const void* in, void* out, const DslashArgs& a, int zfast, hipStream_t st,
               int cmaj = 0) {
  const int Vs = a.L[0] * a.L[1] * a.L[2];
  const int ntile_s = zfast ? ((a.L[0] * a.L[1] + kBlock - 1) / kBlock) * a.L[2] : (Vs + kBlock - 1) / kBlock;
  const int nchunk = a.L[3] / TCH;
  dim3 grid(unsigned(ntile_s * nchunk * (a.nrhs / NR)));
  if constexpr (sizeof(S) >= 8) {  // the site-term forms exist for FP32 and FP64 storage
    if (a.clov) {
      if (a.dagger)
        launch(k_dslash_t<S, TCH, NR, true, true>, grid, dim3(kBlock), 0, st, U, in, out, a, ntile_s, zfast, cmaj);
      else
        launch(k_dslash_t<S, TCH, NR, false, true>, grid, dim3(kBlock), 0, st, U, in, out, a, ntile_s, zfast,
               cmaj);
      QMG_LAUNCH_CHECK();
      return;
    }
  }
  if (a.dagger)
    launch(k_dslash_t<S, TCH, NR, true>, grid, dim3(kBlock), 0, st, U, in, out, a, ntile_s, zfast, cmaj);
  else
    launch(k_dslash_t<S, TCH, NR, false>, grid, dim3(kBlock), 0, st, U, in, out, a, ntile_s, zfast, cmaj);
  QMG_LAUNCH_CHECK();
}

// Multi-RHS t-walking forms, code 1000 * zfast + 100 * NR + TCH (NR = 2 or 3 right-hand sides
// per thread; FP32 storage only: the NR accumulators, own spinors and carried hops take
// 190-250 VGPRs)
inline bool twx_code(int v) {
  const int z = v / 1000, nr = (v % 1000) / 100, tch = v % 100;
  return v > 100 && z <= 1 && (nr == 2 || nr == 3) && (tch == 2 || tch == 4 || tch == 8);
}

template <class S>
void run_twx(int v, const void* U, const void* in, void* out, const DslashArgs& a, hipStream_t st, int cm) {
  if constexpr (sizeof(S) != 8) {
    set_error("dslash launch form %d needs FP32 storage", v);
  } else {
    const int z = v / 1000, nr = (v % 1000) / 100, tch = v % 100;
    auto go = [&](auto nrc) {
      constexpr int NR = decltype(nrc)::value;
      if (tch == 2) launch_tw<S, 2, NR>(U, in, out, a, z, st, cm);
      else if (tch == 4) launch_tw<S, 4, NR>(U, in, out, a, z, st, cm);
      else launch_tw<S, 8, NR>(U, in, out, a, z, st, cm);
    };
    if (nr == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 3>{});
  }
}

// launch codes of the two-sites-per-thread form (dslash_pair.hip) with 1 or 2 right-hand sides per
// thread; chosen by the heuristic or the autotuner
constexpr int kPair1 = 9001, kPair2 = 9002;

template <class S>
void launch_s(const void* U, const void* in, void* out, const DslashArgs& a, hipStream_t st) {
  const bool clov = a.clov != nullptr;
  // algorithmic traffic: spinor in + out (2 x 12 complex per site and rhs) + 4 links per site
  // (+ the site term's 2 x 18 complex entries with the clover term); flops: 1368 per site and
  // rhs for the stencil, 504 more for the two 6 x 6 hermitian blocks
  const double cb = double(sizeof(S));
  const double bytes = double(a.V) * (24.0 * a.nrhs + 36.0 + (clov ? 36.0 : 0.0)) * cb;
  const double flops = (clov ? 1872.0 : 1368.0) * a.V * a.nrhs;
  // Launch variants for the native layout: 1 = one site per thread, 2/4/8 = t-walking with
  // that many sites per thread along t, 16 = direction-split (four threads per site), 32/64 =
  // one site per thread for 2/4 right-hand sides at once (links loaded once for all of them),
  // 1000 z + 100 NR + TCH = t-walking with NR = 2 or 3 right-hand sides per thread (FP32; z:
  // z-fastest tile order); 10000 + a t-walking code: the same in t-chunk-major workgroup order;
  // kPair1 / kPair2 = two sites per thread for 1 or 2 right-hand sides (FP32; not offered as a forced variant).
  // Default: BF16/FP16 storage the direction split.  Else the longest t-chunk that still gives >= 1024
  // workgroups, or the direction split when one thread per site would leave the GPU short of wavefronts;
  // in FP32 for several right-hand sides the multi-RHS t-walk (3 per thread when nrhs is a multiple of 3,
  // else 2), but up to 2^19 sites x rhs the direction split; and over that, where rows are even, fields
  // aligned and sites x rhs between 2^17 and 2^21 (with the clover term for several right-hand sides from
  // 2^17 on), two sites per thread.  With the autotuner enabled every valid variant is timed on first use of
  // (precision, extents, nrhs, adjoint) and the fastest is kept.  With the clover term: forms 1, 16, 2, 4,
  // 8, the multi-RHS t-walks (FP32 and FP64 storage) and the pairs, the direction split alone for
  // BF16/FP16 storage.
  const int Vs = a.L[0] * a.L[1] * a.L[2];
  const long wg1 = long((Vs + kBlock - 1) / kBlock) * a.nrhs;  // workgroups per t-slice
  const int Lt = a.L[3];
  auto run = [&](int v) {
    const int cm = v / 10000;  // 10000 + code: the t-walks in t-chunk-major workgroup order
    v %= 10000;
    const int f = v > 9000 ? 3 : v == 16 ? 0 : (v == 1 || v == 32 || v == 64) ? 1 : 2;
    static const char* const fams[2][4] = {{"dslash/dir", "dslash/site", "dslash/twalk", "dslash/pair"},
                                           {"clover/dir", "clover/site", "clover/twalk", "clover/pair"}};
    // an odd right-hand side behind groups of two is a launch of its own: time both as one
    TimedLaunch tl(fams[clov ? 1 : 0][f], st, bytes, flops, !(v == kPair2 && a.nrhs % 2));
    switch (v) {
      case 8: launch_tw<S, 8, 1>(U, in, out, a, 0, st, cm); break;
      case 4: launch_tw<S, 4, 1>(U, in, out, a, 0, st, cm); break;
      case 2: launch_tw<S, 2, 1>(U, in, out, a, 0, st, cm); break;
      case 16: launch_dir<S>(U, in, out, a, st); break;
      case 32: launch_t<S, 2>(U, in, out, a, st); break;
      case 64: launch_t<S, 4>(U, in, out, a, st); break;
      case kPair1: launch_dslash_pair(U, in, out, a, 1, st); break;
      case kPair2: launch_dslash_pair(U, in, out, a, 2, st); break;
      default:
        if (v > 100) run_twx<S>(v, U, in, out, a, st, cm);
        else launch_t<S, 1>(U, in, out, a, st);
        break;
    }
  };
  const bool pairs = sizeof(S) == 8 && dslash_pair_fits(a, U, in, out);
  auto valid = [&](int v) {
    if (v == kPair1 || v == kPair2) return pairs && a.nrhs >= v - 9000;
    if (v >= 10000) {
      v -= 10000;
      if (v < 2 || v == 16 || v == 32 || v == 64 || v >= 10000) return false;
    }
    if (v == 16) return true;
    if (clov && (sizeof(S) == 4 || v == 32 || v == 64)) return false;
    if (v == 1) return true;
    if (v == 32) return a.nrhs % 2 == 0;
    if (v == 64) return a.nrhs % 4 == 0;
    if (v > 100) {
      const int nr = (v % 1000) / 100, tch = v % 100;
      return sizeof(S) == 8 && twx_code(v) && a.nrhs % nr == 0 && Lt % tch == 0;
    }
    return (v == 2 || v == 4 || v == 8) && Lt % v == 0;
  };
  if (a.tchunk > 0 && valid(a.tchunk)) {
    run(a.tchunk);
    return;
  }
  auto fits = [&](int tch) { return Lt % tch == 0 && wg1 * (Lt / tch) >= 1024; };
  // one thread per site fills 256 CUs x 32 wavefronts only from 2^19 sites x rhs on
  const bool small = long(a.V) * a.nrhs < (1L << 19);
  int choice = fits(8) ? 8 : fits(4) ? 4 : fits(2) ? 2 : small ? 16 : 1;
  // 4-byte storage (BF16/FP16): the one-thread-per-site forms hold every hop's loads in
  // registers (up to 256 VGPRs, one wavefront per SIMD); the direction split needs 64-70
  if (sizeof(S) == 4) choice = 16;
  if (!valid(choice)) choice = 16;
  if (sizeof(S) == 8 && a.nrhs >= 2) {
    // measured at 16^3x32 (8 rhs), 24^3x64 (16) and 32^3x64 (12): 10-20% faster than the
    // one-rhs-per-thread forms; z-fastest tiles only where 256-site pieces tile an xy-plane
    const int nr = a.nrhs % 3 == 0 ? 3 : a.nrhs % 2 == 0 ? 2 : 0;
    const int z = (a.L[0] * a.L[1]) % kBlock == 0 ? 1 : 0;
    const int tch = (nr == 3 && Lt % 8 == 0) ? 8 : Lt % 4 == 0 ? 4 : 2;
    if (nr && valid(1000 * z + 100 * nr + tch)) choice = 1000 * z + 100 * nr + tch;
    // too few sites for that: the direction split (us, direction split / t-walk: Wilson on odd rows, which keep
    // it, 15^3 x 16 with 2 rhs 14.0 / 44.7, 15 x 16^2 x 32 with 2 27 / 45, with 4 49.2 / 49.8, 25 x 24^2 x 18 with 2 58 / 74;
    // clover 12^4 with 4 15.5 / 81, 12 rhs 35 / 107, 16^3 x 32 with 4 72 / 83, with 8 144 / 131)
    if (long(a.V) * a.nrhs <= (1L << 19)) choice = 16;
  }
  // Two sites per thread.  Against them the t-walks carry neighbours from step to step, and win where
  // there are sites enough (Wilson, us, t-walk / pairs: 32^3 x 64 with 1 rhs 261 / 276, 2 rhs 423 / 440;
  // 24^3 x 64 with 8 rhs 616 / 644; 24^3 x 48 with 4 rhs 264 / 261); below, and with the clover term for
  // several right-hand sides everywhere, the pairs' 16-byte loads do (16^3 x 32 with 1 rhs 15.6 / 14.4, 4 rhs
  // 47 / 36, 8 rhs 82 / 76, 12 rhs 127 / 107; 24^3 x 48 with 1 rhs 88 / 72; clover 16^3 x 32 with 4 rhs 83 / 46,
  // 24^3 x 48 with 12 rhs 1068 / 814, 32^3 x 64 with 4 rhs 1196 / 947, 1 rhs 413 / 420).  Below 2^17 sites x rhs half
  // the threads are too few (18 x 5 x 9 x 13, 3 rhs: 9.0 / 10.0).
  const long work = long(a.V) * a.nrhs;
  // One right-hand side, against the direction split, whose workgroups are small: a last round of 512 sites to
  // each of the 256 CUs that is not nearly full costs more than the loads save (rounds, us, direction split /
  // pairs: 16^3 x 36 1.1, 17.0 / 19.9; 18^3 x 32 1.4, 22.3 / 23.7; 20^3 x 28 1.7, 26.0 / 25.0; 16^2 x 32^2 2.0, 31.0 / 27.8;
  // 20^3 x 40 2.4, 35.5 / 37.5), from the fourth round on no longer (24^3 x 32 3.4, 48.7 / 47.6).
  const long ntile = (long(a.V) + 511) / 512, rounds = (ntile + 255) / 256;
  const bool full = a.nrhs > 1 || rounds >= 4 || 20 * ntile >= 17 * 256 * rounds;
  if (pairs && work >= (1L << 17) && full && (work < (1L << 21) || (clov && a.nrhs > 1)))
    choice = a.nrhs > 1 && work >= (1L << 20) ? kPair2 : kPair1;
  // t-walks in t-chunk-major order: every XCD works on the same t-chunk, so the neighbour
  // re-reads that miss an XCD's L2 meet the chunk in the last-level cache (measured at
  // 32^3x64: 4 rhs 824 -> 773 us, 1 and 12 rhs within 2-4%)
  if ((choice == 2 || choice == 4 || choice == 8 || (choice > 100 && choice < 9000)) && valid(10000 + choice))
    choice += 10000;
  if (tune_enabled()) {
    const std::string key = "dslash/" + std::to_string(int(StoreTraits<S>::prec)) + "/" + std::to_string(a.L[0]) +
                            "x" + std::to_string(a.L[1]) + "x" + std::to_string(a.L[2]) + "x" +
                            std::to_string(a.L[3]) + "/" + std::to_string(a.nrhs) + "/" + std::to_string(a.dagger) +
                            (clov ? "/clover" : "");
    const int cached = tune_lookup(key);
    if (cached > 0) {
      if (valid(cached)) choice = cached;  // the pairs' form also asks for aligned fields
    } else {
      int cand[50], n = 0;
      for (int v : {kPair1, kPair2})
        if (valid(v)) cand[n++] = v;
      for (int v : {1, 16, 2, 4, 8, 32, 64, 202, 204, 208, 302, 304, 308, 1202, 1204, 1208, 1302, 1304, 1308})
        for (int c : {0, 10000})
          if ((c == 0 || (v != 1 && v != 16 && v != 32 && v != 64)) && valid(c + v)) cand[n++] = c + v;
      choice = tune_measure(key, cand, n, st, run);
    }
  }
  run(choice);
}

}  // namespace

void launch_dslash_batched(qmg_prec prec, const BatchLattice* lat_dev, int n_lat, int total_tiles,
                           const void* const* U, const void* const* in, void* const* out, bool dagger,
                           double bytes, double flops, hipStream_t st) {
  TimedLaunch tl("dslash/batched", st, bytes, flops);
  auto go = [&](auto tag) {
    using S = decltype(tag);
    if (dagger)
      launch(k_dslash_batched<S, true>, dim3(total_tiles), dim3(kBlock), 0, st, lat_dev, n_lat, U, in, out);
    else
      launch(k_dslash_batched<S, false>, dim3(total_tiles), dim3(kBlock), 0, st, lat_dev, n_lat, U, in, out);
  };
  switch (prec) {
    case QMG_F64: go(double2{}); break;
    case QMG_F32: go(float2{}); break;
    case QMG_BF16: go(cbf16{}); break;
    case QMG_F16: go(chalf{}); break;
  }
  QMG_LAUNCH_CHECK();
}

void launch_dslash_padded(qmg_prec prec, const BatchLattice* lat_dev, int nl, int nr, int Vpad, bool even_rows,
                          const void* U, const void* in, void* out, bool dagger, double bytes, double flops,
                          hipStream_t st) {
  TimedLaunch tl("batch/dslash", st, bytes, flops);
  // FP32 with every row of even length: two sites per thread
  if (prec == QMG_F32 && even_rows) return launch_dslash_pair_padded(lat_dev, nl, nr, Vpad, U, in, out, dagger, st);
  const int ntile = (Vpad + kBlock - 1) / kBlock;
  auto go = [&](auto tag) {
    using S = decltype(tag);
    auto run = [&](auto nrc) {
      constexpr int NR = decltype(nrc)::value;
      const dim3 g(unsigned(ntile) * unsigned(nl) * unsigned(nr / NR));
      if (dagger)
        launch(k_dslash_padded<S, true, NR>, g, dim3(kBlock), 0, st, lat_dev, static_cast<const S*>(U),
               static_cast<const S*>(in), static_cast<S*>(out), nr, ntile);
      else
        launch(k_dslash_padded<S, false, NR>, g, dim3(kBlock), 0, st, lat_dev, static_cast<const S*>(U),
               static_cast<const S*>(in), static_cast<S*>(out), nr, ntile);
    };
    // several right-hand sides per thread in FP32 storage (the setup's test-vector batches)
    if constexpr (sizeof(S) == 8) {
      if (nr % 4 == 0) return run(std::integral_constant<int, 4>{});
      if (nr % 2 == 0) return run(std::integral_constant<int, 2>{});
    }
    run(std::integral_constant<int, 1>{});
  };
  switch (prec) {
    case QMG_F64: go(double2{}); break;
    case QMG_F32: go(float2{}); break;
    case QMG_BF16: go(cbf16{}); break;
    case QMG_F16: go(chalf{}); break;
  }
  QMG_LAUNCH_CHECK();
}

void launch_dslash(qmg_prec prec, const void* U, const void* in, void* out, const DslashArgs& a,
                   hipStream_t st) {
  if (a.canonical) return launch_dslash_canonical(prec, U, in, out, a, st);
  switch (prec) {
    case QMG_F64: launch_s<double2>(U, in, out, a, st); break;
    case QMG_F32: launch_s<float2>(U, in, out, a, st); break;
    case QMG_BF16: launch_s<cbf16>(U, in, out, a, st); break;
    case QMG_F16: launch_s<chalf>(U, in, out, a, st); break;
  }
}

}  // namespace qmg
