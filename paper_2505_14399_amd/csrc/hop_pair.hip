// Even-odd hop in FP32 storage, two neighbouring half-lattice sites per thread.
//
// What bounds it: a wavefront's 8-byte-per-lane load occupies the load pipe about 17 cycles, as long
// as a 16-byte one, so one complex number per lane runs the pipe at half its rate (a standalone
// probe on L2-resident data: 18.8 TB/s with 8 bytes per lane, 36.6 TB/s with 16).  A thread therefore
// takes the sites xh, xh + 1 of a row (one 16-byte load per spinor component and link entry).  In x
// one of the two hops reads the same half-lattice pair, the other that pair moved by one site, of
// which one number is already there and one is loaded by itself.
// Measured on 32^3 x 64, two hops, against one site per thread with the hops outermost: 1 rhs 397 ->
// 347 us, 4 rhs 1057 -> 800 us; 24^3 x 48 with 12 rhs 963 -> 728 us (4 rhs: 3.07 -> 1.48 GB fetched by a hop).
// The colours of the neighbours' spinors are taken one after another over all eight hops
// (each colour's sum by itself, see pair.hpp), so that the planes the workgroups of an XCD read at a time are a third of
// their spinors and fit its 4 MB L2: with the hops outermost nearly every y, z and t neighbour was
// fetched again from beyond the L2.
#include <algorithm>
#include <type_traits>

#include "pair.hpp"
#include "timing.hpp"

namespace qmg {

namespace {

constexpr int kBlock = kPairBlock;

// out (parity p) = POST(YM(y) + sgn H in) as k_hop_eo (hop.hip), NR right-hand sides rhs_base + NR g ..
// of the workgroup's group g.  CLOV: the site term Ap (YM = 2) or Aip (POST = 1) is used, else the scalar one.
// The planes (z, t) are visited in patches of BZ x BT of them (bzt = BZ | BT << 8, divisors of the
// extents), so that the planes that a plane's z and t hops read are visited close in time.
template <bool DAG, int YM, int POST, int NR, bool CLOV>
__global__ __launch_bounds__(kBlock, 2) void k_hop_pair(const float2* __restrict__ Ue, const float2* __restrict__ Uo,
                                                        const float2* __restrict__ in, const float2* __restrict__ y,
                                                        float2* __restrict__ out, const float2* __restrict__ Ap,
                                                        const float2* __restrict__ Aip, DslashArgs a, int p,
                                                        float sgn, int rhs_base, int ngroup, int bzt) {
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  const size_t Vh = size_t(a.V >> 1);
  const int nb = gridDim.x, q8 = nb >> 3, xcd = blockIdx.x & 7;
  const int wg = xcd * q8 + min(xcd, nb & 7) + (blockIdx.x >> 3);  // contiguous tiles per XCD
  const int tile = wg / ngroup, rhs = rhs_base + NR * (wg - tile * ngroup);
  const int g = tile * kBlock + threadIdx.x;
  const int Lxh = L0 >> 1, rp = Lxh >> 1, pp = rp * L1;  // pairs of a row and of a plane
  if (g >= pp * L2 * L3) return;
  int seq = g / pp;
  const int ip = g - seq * pp;
  const int BZ = bzt & 0xff, BT = bzt >> 8;
  const int tt = seq % BT;
  seq /= BT;
  const int zz = seq % BZ;
  seq /= BZ;
  const int nbz = L2 / BZ;
  const int z = (seq % nbz) * BZ + zz, t = (seq / nbz) * BT + tt;
  const int yy = ip / rp, xh = 2 * (ip - yy * rp);
  const bool odd = (yy + z + t + p) & 1;  // x = 2 xh + odd
  // byte offsets of the pair at (xh; cy, cz, ct)
  auto at = [&](int cy, int cz, int ct) { return 8u * unsigned(xh + Lxh * (cy + L1 * (cz + L2 * ct))); };
  const unsigned own = at(yy, z, t);
  const unsigned yp = at(yy + 1 == L1 ? 0 : yy + 1, z, t), ym = at(yy == 0 ? L1 - 1 : yy - 1, z, t);
  const unsigned zp = at(yy, z + 1 == L2 ? 0 : z + 1, t), zm = at(yy, z == 0 ? L2 - 1 : z - 1, t);
  const unsigned tp = at(yy, z, t + 1 == L3 ? 0 : t + 1), tm = at(yy, z, t == 0 ? L3 - 1 : t - 1);
  // the number beyond the pair in x: xh + 2 (x odd, forward) or xh - 1 (x even, backward)
  const unsigned ex = odd ? (xh + 2 == Lxh ? own - 8u * unsigned(xh) : own + 16u)
                          : (xh == 0 ? own + 8u * unsigned(Lxh - 1) : own - 8u);
  const float2* Uown = p ? Uo : Ue;
  const float2* Uoth = p ? Ue : Uo;
  const float mh = -0.5f * sgn;
  const float cs = mh * a.cw_f[0], ct = mh * a.cw_f[3];
  const float ctf = (a.bc_t < 0 && t == L3 - 1) ? -ct : ct, ctb = (a.bc_t < 0 && t == 0) ? -ct : ct;
  constexpr float sf = DAG ? 1.f : -1.f, sb = -sf;
  constexpr int PARK = NR == 2 ? 16 : 6;
  __shared__ float4 park[PARK ? PARK : 1][kPairBlock];
  cf wa[NR][12], wb[NR][12], ta[NR][12], tb[NR][12];
  const float2* inr = in + size_t(rhs) * 12 * Vh;
  auto hop = [&](auto mu, auto fwd, unsigned nbo, float coef, int b) {
    constexpr int MU = decltype(mu)::value;
    constexpr bool F = decltype(fwd)::value;
    const float2* ul = (F ? Uown : Uoth) + size_t(MU) * 9 * Vh;
    const unsigned lo = F ? own : nbo;
    cf ua[3], ub[3];  // column b of U, or of U^dag
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const Two u = ld2(ul + (F ? 3 * c + b : 3 * b + c) * Vh, lo);
      ua[c] = F ? u.a : conj(u.a);
      ub[c] = F ? u.b : conj(u.b);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      cf ca[4], cb[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const Two v = ld2(inr + (r * 12 + 3 * k + b) * Vh, nbo);
        ca[k] = v.a;
        cb[k] = v.b;
      }
      add_hop<MU>(ca, ua, F ? sf : sb, coef, ta[r]);
      add_hop<MU>(cb, ub, F ? sf : sb, coef, tb[r]);
    }
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using T = std::true_type;
  using F = std::false_type;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    {  // both x hops: the pair's own index and the number beyond it
      cf ufa[3], ufb[3], uba[3], ubb[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const Two u = ld2(Uown + (3 * c + b) * Vh, own);
        const Two w = ld2(Uoth + (3 * b + c) * Vh, own);
        const cf m = ld1(Uoth + (3 * b + c) * Vh, odd ? own : ex);
        ufa[c] = u.a;
        ufb[c] = u.b;
        uba[c] = conj(pick(odd, w.a, m));
        ubb[c] = conj(pick(odd, w.b, w.a));
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        cf pa[4], pb[4], ma[4], mb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float2* pl = inr + (r * 12 + 3 * k + b) * Vh;
          const Two v = ld2(pl, own);
          const cf e = ld1(pl, ex);
          pa[k] = mb[k] = pick(odd, v.b, v.a);
          pb[k] = pick(odd, e, v.b);
          ma[k] = pick(odd, v.a, e);
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) ta[r][k] = tb[r][k] = {0.f, 0.f};
        add_hop<0>(pa, ufa, sf, 1.f, ta[r]);
        add_hop<0>(pb, ufb, sf, 1.f, tb[r]);
        add_hop<0>(ma, uba, sb, 1.f, ta[r]);
        add_hop<0>(mb, ubb, sb, 1.f, tb[r]);
      }
    }
    hop(I1{}, T{}, yp, 1.f, b);
    hop(I1{}, F{}, ym, 1.f, b);
    hop(I2{}, T{}, zp, 1.f, b);
    hop(I2{}, F{}, zm, 1.f, b);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) {  // x, y and z have one weight
        ta[r][k] = cs * ta[r][k];
        tb[r][k] = cs * tb[r][k];
      }
    hop(I3{}, T{}, tp, ctf, b);
    hop(I3{}, F{}, tm, ctb, b);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; k += 2) {
        add_pack<PARK>(12 * r + k / 2, b, ta[r][k], ta[r][k + 1], wa[r][k], wa[r][k + 1], park);
        add_pack<PARK>(12 * r + 6 + k / 2, b, tb[r][k], tb[r][k + 1], wb[r][k], wb[r][k + 1], park);
      }
  }
  if constexpr (YM == 1 || (YM == 2 && !CLOV)) {
    const float f = YM == 1 ? 1.f : a.diag_f;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const Two v = ld2(y + (size_t(rhs + r) * 12 + k) * Vh, own);
        wa[r][k] += f * v.a;
        wb[r][k] += f * v.b;
      }
  } else if constexpr (YM == 2) {
    cf va[NR][12], vb[NR][12];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const Two v = ld2(y + (size_t(rhs + r) * 12 + k) * Vh, own);
        va[r][k] = v.a;
        vb[r][k] = v.b;
      }
    site_term<NR>(Ap, own, Vh, va, vb, wa, wb);
  }
  if constexpr (POST == 1 && CLOV) {
    cf oa[NR][12], ob[NR][12];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) oa[r][k] = ob[r][k] = {0.f, 0.f};
    site_term<NR>(Aip, own, Vh, wa, wb, oa, ob);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        wa[r][k] = oa[r][k];
        wb[r][k] = ob[r][k];
      }
  } else if constexpr (POST == 1) {
    const float inv = 1.f / a.diag_f;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        wa[r][k] = inv * wa[r][k];
        wb[r][k] = inv * wb[r][k];
      }
  }
  typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      char* o = reinterpret_cast<char*>(out + (size_t(rhs + r) * 12 + k) * Vh) + own;
      const f4 v = {wa[r][k].re, wa[r][k].im, wb[r][k].re, wb[r][k].im};
      __builtin_nontemporal_store(v, reinterpret_cast<f4*>(o));
    }
}

}  // namespace

// From 2^18 sites x right-hand sides on: below, half as many threads leave the chip short of waves
// (two hops, us, one site per thread against two: 16^3 x 32 with 1 rhs 38 against 55, 2 rhs 50 / 44,
// 4 rhs 72 / 57; 16^3 x 64 with 1 rhs 55 / 51; 24^3 x 48 with 1 rhs 129 / 103; with the site term, whose hops the
// direction split took below 2^20: 16^3 x 32 with 2 rhs 62 / 51, 4 rhs 102 / 62, 24^3 x 48 with 1 rhs 170 / 148)
bool hop_pair_fits(const DslashArgs& a, const void* Ue, const void* Uo, const void* in, const void* y,
                   const void* out, const void* Ap, const void* Aip) {
  uintptr_t bits = 0;
  for (const void* q : {Ue, Uo, in, y, out, Ap, Aip}) bits |= reinterpret_cast<uintptr_t>(q);
  return a.L[0] % 4 == 0 && a.link_ne == 9 && long(a.V) * a.nrhs >= kHopPairSites && (bits & 15) == 0 && size_t(a.V / 2) * 8 < (size_t(1) << 32);
}

void launch_hop_pair(const DslashArgs& a, const void* Ue, const void* Uo, int p, const void* in, const void* y,
                     void* out, const void* Ap, const void* Aip, int ym, int post, double sgn, int nr,
                     hipStream_t st) {
  const bool clov = (ym == 2 && Ap) || (post == 1 && Aip);
  const unsigned ntile = unsigned((a.V / 4 + kBlock - 1) / kBlock);
  auto patch = [](int L) { return L % 8 == 0 ? 8 : L % 4 == 0 ? 4 : L % 2 == 0 ? 2 : 1; };
  const int bzt = patch(a.L[2]) | (patch(a.L[3]) << 8);
  auto go = [&](auto kern, int base, int groups) {
    launch(kern, dim3(ntile * unsigned(groups)), dim3(kBlock), 0, st, static_cast<const float2*>(Ue),
           static_cast<const float2*>(Uo), static_cast<const float2*>(in), static_cast<const float2*>(y),
           static_cast<float2*>(out), static_cast<const float2*>(Ap), static_cast<const float2*>(Aip), a, p,
           float(sgn), base, groups, bzt);
  };
  // full groups of nr right-hand sides, then the rest one at a time
  auto run = [&](auto dag, auto ymc, auto pc, auto cl) {
    constexpr bool D = decltype(dag)::value, CL = decltype(cl)::value;
    constexpr int YM = decltype(ymc)::value, PO = decltype(pc)::value;
    const int ng = nr == 2 ? a.nrhs / 2 : 0, done = 2 * ng;
    if (ng) go(k_hop_pair<D, YM, PO, 2, CL>, 0, ng);
    if (done < a.nrhs) go(k_hop_pair<D, YM, PO, 1, CL>, done, a.nrhs - done);
  };
  auto form = [&](auto dag) {
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using T = std::true_type;
    using F = std::false_type;
    if (ym == 0) clov ? run(dag, I0{}, I1{}, T{}) : run(dag, I0{}, I1{}, F{});
    else if (ym == 2) clov ? run(dag, I2{}, I0{}, T{}) : run(dag, I2{}, I0{}, F{});
    else if (post == 0) run(dag, I1{}, I0{}, F{});
    else clov ? run(dag, I1{}, I1{}, T{}) : run(dag, I1{}, I1{}, F{});
  };
  if (a.dagger) form(std::true_type{});
  else form(std::false_type{});
}

}  // namespace qmg
