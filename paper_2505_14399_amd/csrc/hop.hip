// Even-odd (Schur complement) stencils: the hops between the two parities of a lattice, with the
// site terms of the Schur operator folded into their epilogues.
#include <algorithm>
#include <type_traits>

#include "stencil.hpp"
#include "timing.hpp"

namespace qmg {

namespace {

// ---------------------------------------------------------------------------------------
// Even-odd (Schur complement) forms on half-lattice fields.  Every extent is even; a site of
// parity p = (x + y + z + t) mod 2 has the half-lattice index i = lex / 2, so within a row of
// fixed (y, z, t) the sites of one parity are every other x.  Layouts: spinor [rhs][12][V/2]
// per parity, gauge [parity][mu][9][V/2] (U_mu(x) stored at x's parity), site term and its
// inverse [parity][alpha][18][V/2] in the packed form of clover_acc (nullptr: the scalar
// diagonal term of the Wilson operator).

// out (parity p) = POST( YM(y) + sgn * H in ), H the hopping part of D (of D^dag with DAG),
// in on parity 1 - p.  YM: 0 nothing, 1 y, 2 A_p y.  POST: 0 nothing, 1 A_p^-1.
// Each thread forms NR right-hand sides rhs_base + NR g .. + NR - 1 of its site, so every link
// is loaded once for all NR of them; the NR-groups of a tile are adjacent in the (XCD-aware)
// workgroup order, so the groups of one tile run on one XCD and meet its links in that L2.
template <class S, bool DAG, int YM, int POST, int NE = 9, int NR = 1>
__global__ __launch_bounds__(kBlock) void k_hop_eo(const S* __restrict__ Ue, const S* __restrict__ Uo,
                                                   const S* __restrict__ in, const S* __restrict__ y,
                                                   S* __restrict__ out, const S* __restrict__ Ap,
                                                   const S* __restrict__ Aip, DslashArgs a, int p, float sgn,
                                                   int rhs_base, int ngroup, int bzt) {
  using C = ctype<S>;
  const int Vh = a.V >> 1;
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  int tile = wg / ngroup;
  const int rhs = rhs_base + NR * (wg % ngroup);
  if (bzt) {
    // blocked order over the (z, t) planes: the tiles of a patch of BZ planes x BT slices are
    // adjacent in the schedule (t fastest, then z, then the tiles of a plane), so the slices a
    // site's t-hops read are loaded by tiles running close in time (lexicographic order runs a
    // whole t-slice between them); needs whole tiles per plane, BZ | L2 and BT | L3
    const int BZ = bzt & 0xff, BT = bzt >> 8, tpp = (L0 * L1) / (2 * kBlock);
    const int h = tile % tpp;
    int r = tile / tpp;
    const int tt = r % BT;
    r /= BT;
    const int zz = r % BZ;
    r /= BZ;
    const int nbz = L2 / BZ;
    tile = h + tpp * ((r % nbz) * BZ + zz + L2 * ((r / nbz) * BT + tt));
  }
  const int i = tile * kBlock + threadIdx.x;
  if (i >= Vh) return;
  const int Lxh = L0 >> 1;
  const int xh = i % Lxh;
  int row = i / Lxh;
  const int yy = row % L1;
  row /= L1;
  const int z = row % L2;
  const int t = row / L2;
  const int x = 2 * xh + ((yy + z + t + p) & 1);
  auto cb = [&](int cx, int cy, int cz, int ct) { return (cx + L0 * (cy + L1 * (cz + L2 * ct))) >> 1; };
  const int xp = cb(x + 1 == L0 ? 0 : x + 1, yy, z, t), xm = cb(x == 0 ? L0 - 1 : x - 1, yy, z, t);
  const int yp = cb(x, yy + 1 == L1 ? 0 : yy + 1, z, t), ym = cb(x, yy == 0 ? L1 - 1 : yy - 1, z, t);
  const int zp = cb(x, yy, z + 1 == L2 ? 0 : z + 1, t), zm = cb(x, yy, z == 0 ? L2 - 1 : z - 1, t);
  const int tp = cb(x, yy, z, t + 1 == L3 ? 0 : t + 1), tm = cb(x, yy, z, t == 0 ? L3 - 1 : t - 1);
  const S* Uown = p ? Uo : Ue;  // links leaving this site
  const S* Uoth = p ? Ue : Uo;  // links arriving from the backward neighbours
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
  cplx<C> w[NR][12];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int k = 0; k < 12; ++k) w[r][k] = {C(0), C(0)};
  const C mh = C(-0.5) * C(sgn);
  do_hop<S, NR, 0, true, DAG, NE>(Uown, in, w, i, xp, rhs, Vh, mh * cw[0]);
  do_hop<S, NR, 0, false, DAG, NE>(Uoth, in, w, xm, xm, rhs, Vh, mh * cw[0]);
  do_hop<S, NR, 1, true, DAG, NE>(Uown, in, w, i, yp, rhs, Vh, mh * cw[1]);
  do_hop<S, NR, 1, false, DAG, NE>(Uoth, in, w, ym, ym, rhs, Vh, mh * cw[1]);
  do_hop<S, NR, 2, true, DAG, NE>(Uown, in, w, i, zp, rhs, Vh, mh * cw[2]);
  do_hop<S, NR, 2, false, DAG, NE>(Uoth, in, w, zm, zm, rhs, Vh, mh * cw[2]);
  do_hop<S, NR, 3, true, DAG, NE>(Uown, in, w, i, tp, rhs, Vh, mh * cw[3] * bt_f);
  do_hop<S, NR, 3, false, DAG, NE>(Uoth, in, w, tm, tm, rhs, Vh, mh * cw[3] * bt_b);
  if constexpr (YM == 1) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) w[r][k] += ldc(y, sp_idx(rhs + r, k, i, Vh));
  } else if constexpr (YM == 2) {
    if (Ap) {
      cplx<C> yv[NR][12];
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int k = 0; k < 12; ++k) yv[r][k] = ldc(y, sp_idx(rhs + r, k, i, Vh));
      clover_acc<S, NR>(Ap, i, Vh, yv, w);
    } else {
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int k = 0; k < 12; ++k) w[r][k] += diag * ldc(y, sp_idx(rhs + r, k, i, Vh));
    }
  }
  if constexpr (POST == 1) {
    if (Aip) {
      cplx<C> o[NR][12];
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int k = 0; k < 12; ++k) o[r][k] = {C(0), C(0)};
      clover_acc<S, NR>(Aip, i, Vh, w, o);
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int k = 0; k < 12; ++k) w[r][k] = o[r][k];
    } else {
      const C inv = C(1) / diag;
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int k = 0; k < 12; ++k) w[r][k] = inv * w[r][k];
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int k = 0; k < 12; ++k) stc_stream(out, sp_idx(rhs + r, k, i, Vh), w[r][k]);
}

// Rows I0 .. I0+2 of one chirality of the even-odd epilogue: x holds sgn H in (+ y with YM = 1)
// on the six components of the chirality; YM = 2 adds A_p y, POST = 1 applies A_p^-1
template <class S, int YM, int POST, int I0>
__device__ inline void eo_rows(const S* __restrict__ Ab, const S* __restrict__ Aib, const S* __restrict__ y,
                               size_t ybase, int Vh, ctype<S> diag, cplx<ctype<S>> (&x)[6], cplx<ctype<S>> (&r)[3]) {
  using C = ctype<S>;
  if constexpr (YM == 2) {
    cplx<C> yv[6], ay[3];
#pragma unroll
    for (int j = 0; j < 6; ++j) yv[j] = ldc(y, ybase + size_t(j) * Vh);
    if (Ab) {
      site_term_rows<S, I0>(Ab, Vh, yv, ay);
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q) ay[q] = diag * yv[I0 + q];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) r[q] = x[I0 + q] + ay[q];
  } else if constexpr (POST == 1) {
    if (Aib) {
      site_term_rows<S, I0>(Aib, Vh, x, r);
    } else {
      const C inv = C(1) / diag;
#pragma unroll
      for (int q = 0; q < 3; ++q) r[q] = inv * x[I0 + q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 3; ++q) r[q] = x[I0 + q];
  }
}

// Direction-split form of k_hop_eo for half lattices too small to fill the GPU with one thread
// per site: a workgroup covers 64 half-lattice sites, wavefront mu forms the two hops along mu,
// the partial spinors meet in LDS, and wavefront w then finishes output components
// 3w .. 3w+2 (rows 3 (w & 1) .. +2 of chirality w >> 1) with the epilogue of k_hop_eo.
template <class S, bool DAG, int YM, int POST, int NE = 9>
__global__ __launch_bounds__(kBlock) void k_hop_eo_dir(const S* __restrict__ Ue, const S* __restrict__ Uo,
                                                       const S* __restrict__ in, const S* __restrict__ y,
                                                       S* __restrict__ out, const S* __restrict__ Ap,
                                                       const S* __restrict__ Aip, DslashArgs a, int p, float sgn) {
  using C = ctype<S>;
  constexpr int TS = kBlock / 4;
  __shared__ cplx<C> part[4][12][TS];
  const int Vh = a.V >> 1;
  const int ntile = (Vh + TS - 1) / TS;
  const int wg = xcd_tile(blockIdx.x, gridDim.x);
  const int tile = wg % ntile, rhs = wg / ntile;
  const int lane = threadIdx.x & (TS - 1), mu = threadIdx.x / TS;
  const int i = tile * TS + lane;
  const bool live = i < Vh;
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  C cw, diag;
  if constexpr (sizeof(C) == 8) {
    cw = a.cw_d[mu];
    diag = a.diag_d;
  } else {
    cw = a.cw_f[mu];
    diag = a.diag_f;
  }
  cplx<C> acc[1][12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[0][k] = {C(0), C(0)};
  if (live) {
    const int Lxh = L0 >> 1;
    const int xh = i % Lxh;
    int row = i / Lxh;
    const int yy = row % L1;
    row /= L1;
    const int z = row % L2;
    const int t = row / L2;
    int c[4] = {2 * xh + ((yy + z + t + p) & 1), yy, z, t};
    const int L = a.L[mu];
    const int cmu = c[mu];
    auto cb = [&](int v) {
      int d[4] = {c[0], c[1], c[2], c[3]};
      d[mu] = v;
      return (d[0] + L0 * (d[1] + L1 * (d[2] + L2 * d[3]))) >> 1;
    };
    const int fp = cb(cmu + 1 == L ? 0 : cmu + 1), bm = cb(cmu == 0 ? L - 1 : cmu - 1);
    const C mh = C(-0.5);
    C cf = mh * cw, cbk = mh * cw;
    if (mu == 3 && a.bc_t < 0) {
      if (t == L3 - 1) cf = -cf;
      if (t == 0) cbk = -cbk;
    }
    const S* Uown = p ? Uo : Ue;
    const S* Uoth = p ? Ue : Uo;
    switch (mu) {  // uniform within the wavefront
      case 0:
        do_hop<S, 1, 0, true, DAG, NE>(Uown, in, acc, i, fp, rhs, Vh, cf);
        do_hop<S, 1, 0, false, DAG, NE>(Uoth, in, acc, bm, bm, rhs, Vh, cbk);
        break;
      case 1:
        do_hop<S, 1, 1, true, DAG, NE>(Uown, in, acc, i, fp, rhs, Vh, cf);
        do_hop<S, 1, 1, false, DAG, NE>(Uoth, in, acc, bm, bm, rhs, Vh, cbk);
        break;
      case 2:
        do_hop<S, 1, 2, true, DAG, NE>(Uown, in, acc, i, fp, rhs, Vh, cf);
        do_hop<S, 1, 2, false, DAG, NE>(Uoth, in, acc, bm, bm, rhs, Vh, cbk);
        break;
      default:
        do_hop<S, 1, 3, true, DAG, NE>(Uown, in, acc, i, fp, rhs, Vh, cf);
        do_hop<S, 1, 3, false, DAG, NE>(Uoth, in, acc, bm, bm, rhs, Vh, cbk);
        break;
    }
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) part[mu][k][lane] = acc[0][k];
  __syncthreads();
  if (!live) return;
  const int al = mu >> 1;
  const C sg = C(sgn);
  cplx<C> x6[6], r[3];
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const int k = 6 * al + j;
    cplx<C> h = part[0][k][lane];
#pragma unroll
    for (int m = 1; m < 4; ++m) h += part[m][k][lane];
    x6[j] = sg * h;
    if constexpr (YM == 1) x6[j] += ldc(y, sp_idx(rhs, k, i, Vh));
  }
  const size_t ybase = sp_idx(rhs, 6 * al, i, Vh);
  const S* Ab = Ap ? Ap + size_t(al) * 18 * Vh + i : nullptr;
  const S* Aib = Aip ? Aip + size_t(al) * 18 * Vh + i : nullptr;
  if (mu & 1) eo_rows<S, YM, POST, 3>(Ab, Aib, y, ybase, Vh, diag, x6, r);
  else eo_rows<S, YM, POST, 0>(Ab, Aib, y, ybase, Vh, diag, x6, r);
#pragma unroll
  for (int q = 0; q < 3; ++q) stc(out, sp_idx(rhs, 3 * mu + q, i, Vh), r[q]);
}

// out = M in on one parity's half field, M the packed site term (or its inverse) of that
// parity, or the scalar diag (or 1 / diag) when M is nullptr
template <class S, bool INV>
__global__ __launch_bounds__(kBlock) void k_site_eo(const S* __restrict__ M, const S* __restrict__ in,
                                                    S* __restrict__ out, DslashArgs a) {
  using C = ctype<S>;
  const int Vh = a.V >> 1;
  const int ntile = (Vh + kBlock - 1) / kBlock;
  const int wg = blockIdx.x;
  const int tile = wg % ntile, rhs = wg / ntile;
  const int i = tile * kBlock + threadIdx.x;
  if (i >= Vh) return;
  cplx<C> v[1][12], r[1][12];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    v[0][k] = ldc(in, sp_idx(rhs, k, i, Vh));
    r[0][k] = {C(0), C(0)};
  }
  if (M) {
    clover_acc<S, 1>(M, i, Vh, v, r);
  } else {
    const C d = sizeof(C) == 8 ? C(a.diag_d) : C(a.diag_f);
    const C f = INV ? C(1) / d : d;
#pragma unroll
    for (int k = 0; k < 12; ++k) r[0][k] = f * v[0][k];
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) stc(out, sp_idx(rhs, k, i, Vh), r[0][k]);
}

}  // namespace

// right-hand sides per thread of the even-odd hop for several right-hand sides (links loaded
// once for all of them)
constexpr int kHopNR = 2;
// (z, t) patch of the hop's blocked tile order for two or more right-hand sides (measured at
// 32^3 x 64 FP32, four right-hand sides: 4 x 4 planes 522 us per launch against 543-551 us in
// lexicographic order, the other patches with 4 or 8 slices within 1 %; at one right-hand side
// the blocked orders are slower, 191 against 197-215 us, so it keeps the lexicographic order)
constexpr int kHopBZ = 4, kHopBT = 4;

void launch_hop_eo(qmg_prec prec, const DslashArgs& a, const void* Ue, const void* Uo, int p, const void* in,
                   const void* y, void* out, const void* Ap, const void* Aip, int ym, int post, double sgn,
                   hipStream_t st) {
  const int Vh = a.V / 2;
  // direction split for the clover forms on half lattices too small to fill the GPU with one
  // thread per site (measured FP32, one RHS: clover 23.1 against 25.1 us at 16^3 x 32 and 43.4
  // against 48.7 us at 24^3 x 32; the Wilson forms are faster one site per thread at every size,
  // 12.3 against 21.3 us at 16^3 x 32).  Forced with the launch-variant codes 1 = one site per
  // thread, 16 = direction split.
  // The same holds for BF16/FP16 storage (BF16 at 16^3 x 32: Wilson 8.7 against 17.8 us, clover
  // 21.0 against 18.5 us; the forms tie at 24^3 x 64).  FP32 from 2^18 sites x right-hand sides on goes to two sites per
  // thread instead where rows allow (hop_pair.hip).
  const bool with_site_term = (ym == 2 && Ap) || (post == 1 && Aip);
  // FP32 without a forced variant: two sites per thread where its rule holds
  const bool pair = prec == QMG_F32 && a.tchunk == 0 && hop_pair_fits(a, Ue, Uo, in, y, out, Ap, Aip);
  const bool split =
      a.tchunk == 16 || (a.tchunk != 1 && with_site_term && long(Vh) * a.nrhs < (1L << 19));
  const int per_wg = split ? kBlock / 4 : kBlock;
  const unsigned ntile = unsigned((Vh + per_wg - 1) / per_wg);
  const dim3 grid(ntile * unsigned(a.nrhs));
  // right-hand sides per thread of the one-site-per-thread form: forced with the launch-variant
  // codes 501 .. 504, else HOP_NR (FP32 storage and below) once there are enough of them
  int nr = 1;
  if (pair) {
    // two right-hand sides per thread halve the link loads, but also the waves (16^3 x 32, us, one
    // against two: 4 rhs 60 / 67, 8 rhs 103 / 91; 32^3 x 64: 4 rhs 926 / 813)
    nr = a.nrhs >= 2 && long(a.V) * a.nrhs >= (1L << 20) ? 2 : 1;
  } else if (!split) {
    if (a.tchunk >= 501 && a.tchunk <= 504) nr = a.tchunk - 500;
    else if (prec != QMG_F64 && a.nrhs >= 2) nr = std::min(a.nrhs, kHopNR);
  }
  // tile order of the one-site-per-thread form: blocked over patches of BZ x BT (z, t) planes
  // where whole tiles fill a plane (kHopBZ x kHopBT from two right-hand sides on, or forced
  // with the launch-variant codes 7ZT: BZ = Z, BT = T planes; 700 = lexicographic)
  int bz = a.nrhs >= 2 ? kHopBZ : 0, bt = a.nrhs >= 2 ? kHopBT : 0;
  if (a.tchunk >= 700 && a.tchunk < 800) {
    bz = (a.tchunk / 10) % 10;
    bt = a.tchunk % 10;
  }
  const bool blocked = !split && bz > 0 && bt > 0 && (a.L[0] * a.L[1]) % (2 * kBlock) == 0 && a.L[2] % bz == 0 &&
                       a.L[3] % bt == 0;
  const int bzt = blocked ? bz | (bt << 8) : 0;
  // algorithmic traffic: the other parity's spinors and both parities' links once per site of
  // this parity, y when used, the output, and the packed blocks when used
  const double cb = double(prec_bytes(prec));
  const double bytes = double(Vh) * (a.nrhs * (12.0 + 12.0 + (ym ? 12.0 : 0.0)) + 8.0 * a.link_ne +
                                     ((ym == 2 && Ap) ? 36.0 : 0.0) + ((post && Aip) ? 36.0 : 0.0)) * cb;
  // full groups of nr right-hand sides and a one-per-thread rest are two launches: time the pair
  // as one (events on the stream around both) rather than the first launch alone
  const bool two = nr > 1 && a.nrhs >= nr && a.nrhs % nr != 0;
  TimedLaunch tl("evenodd/hop", st, bytes, 1320.0 * Vh * a.nrhs, !two);
  QMG_CHECK((ym == 0 && post == 1) || (ym == 2 && post == 0) || (ym == 1 && post == 0) || (ym == 1 && post == 1),
            QMG_EINVAL, "even-odd hop form (%d, %d) is not built", ym, post);
  if (pair) {
    launch_hop_pair(a, Ue, Uo, p, in, y, out, Ap, Aip, ym, post, sgn, nr, st);
    QMG_LAUNCH_CHECK();
    return;
  }
  auto go = [&](auto tag) {
    using S = decltype(tag);
    auto run = [&](auto kern) {
      launch(kern, grid, dim3(kBlock), 0, st, static_cast<const S*>(Ue), static_cast<const S*>(Uo),
             static_cast<const S*>(in), static_cast<const S*>(y), static_cast<S*>(out), static_cast<const S*>(Ap),
             static_cast<const S*>(Aip), a, p, float(sgn));
    };
    // one-site-per-thread form: full groups of NR right-hand sides, then the rest one per thread
    auto run_nr = [&](auto k_nr, auto k_1) {
      const int ng = a.nrhs / nr, done = ng * nr;
      auto go1 = [&](auto kern, int base, int groups) {
        launch(kern, dim3(ntile * unsigned(groups)), dim3(kBlock), 0, st, static_cast<const S*>(Ue),
               static_cast<const S*>(Uo), static_cast<const S*>(in), static_cast<const S*>(y), static_cast<S*>(out),
               static_cast<const S*>(Ap), static_cast<const S*>(Aip), a, p, float(sgn), base, groups, bzt);
      };
      if (nr > 1 && ng > 0) go1(k_nr, 0, ng);
      if (nr == 1) go1(k_1, 0, a.nrhs);
      else if (done < a.nrhs) go1(k_1, done, a.nrhs - done);
    };
    const int form = ym * 2 + post;  // forms used by the Schur operator, the source and the reconstruction
    auto pick = [&](auto dag, auto ne) {
      constexpr bool D = decltype(dag)::value;
      constexpr int NE = decltype(ne)::value;
      if (split) {
        if (form == 1) run(k_hop_eo_dir<S, D, 0, 1, NE>);
        else if (form == 4) run(k_hop_eo_dir<S, D, 2, 0, NE>);
        else if (form == 2) run(k_hop_eo_dir<S, D, 1, 0, NE>);
        else run(k_hop_eo_dir<S, D, 1, 1, NE>);
        return;
      }
      auto by_nr = [&](auto ym_c, auto post_c) {
        constexpr int YM = decltype(ym_c)::value, PO = decltype(post_c)::value;
        auto k1 = k_hop_eo<S, D, YM, PO, NE, 1>;
        if (nr == 2) run_nr(k_hop_eo<S, D, YM, PO, NE, 2>, k1);
        else if (nr == 3) run_nr(k_hop_eo<S, D, YM, PO, NE, 3>, k1);
        else if (nr == 4) run_nr(k_hop_eo<S, D, YM, PO, NE, 4>, k1);
        else run_nr(k1, k1);
      };
      using I0 = std::integral_constant<int, 0>;
      using I1 = std::integral_constant<int, 1>;
      using I2 = std::integral_constant<int, 2>;
      if (form == 1) by_nr(I0{}, I1{});
      else if (form == 4) by_nr(I2{}, I0{});
      else if (form == 2) by_nr(I1{}, I0{});
      else by_nr(I1{}, I1{});
    };
    using N9 = std::integral_constant<int, 9>;
    using N6 = std::integral_constant<int, 6>;
    if (a.link_ne == 6) {
      if (a.dagger) pick(std::true_type{}, N6{});
      else pick(std::false_type{}, N6{});
    } else {
      if (a.dagger) pick(std::true_type{}, N9{});
      else pick(std::false_type{}, N9{});
    }
  };
  switch (prec) {
    case QMG_F64: go(double2{}); break;
    case QMG_F32: go(float2{}); break;
    case QMG_BF16: go(cbf16{}); break;
    case QMG_F16: go(chalf{}); break;
  }
  QMG_LAUNCH_CHECK();
}

void launch_site_eo(qmg_prec prec, const DslashArgs& a, const void* M, bool inv, const void* in, void* out,
                    hipStream_t st) {
  const int Vh = a.V / 2;
  const dim3 grid(unsigned((Vh + kBlock - 1) / kBlock) * unsigned(a.nrhs));
  auto go = [&](auto tag) {
    using S = decltype(tag);
    if (inv)
      launch(k_site_eo<S, true>, grid, dim3(kBlock), 0, st, static_cast<const S*>(M), static_cast<const S*>(in),
             static_cast<S*>(out), a);
    else
      launch(k_site_eo<S, false>, grid, dim3(kBlock), 0, st, static_cast<const S*>(M), static_cast<const S*>(in),
             static_cast<S*>(out), a);
  };
  switch (prec) {
    case QMG_F64: go(double2{}); break;
    case QMG_F32: go(float2{}); break;
    case QMG_BF16: go(cbf16{}); break;
    case QMG_F16: go(chalf{}); break;
  }
  QMG_LAUNCH_CHECK();
}

}  // namespace qmg
