// D and D^dagger in FP32 storage on the native layout, two neighbouring sites per thread: 16-byte loads
// and the neighbours' colours one after another over all hops, for the reasons given in hop_pair.hip
// (an 8-byte-per-lane load occupies the load pipe as long as a 16-byte one).  The rule that chooses it
// against the t-walking and direction-split forms stands in dslash.hip with the times of both.
#include <algorithm>
#include <type_traits>

#include "pair.hpp"
#include "timing.hpp"

namespace qmg {

namespace {

constexpr int kBlock = kPairBlock;

__device__ inline void st2(float2* p, unsigned off, cf va, cf vb) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const f4 v = {va.re, va.im, vb.re, vb.im};
  __builtin_nontemporal_store(v, reinterpret_cast<f4*>(reinterpret_cast<char*>(p) + off));
}

// D (D^dag) at the sites x, x + 1 (x even) of row (y, z, t) for NR right-hand sides at in / out; V: stride of a
// component plane (at least the volume)
template <int NR, bool DAG, bool CLOV>
__device__ inline void pair_dslash(const float2* __restrict__ U, const float2* __restrict__ in,
                                   float2* __restrict__ out, const DslashArgs& a, size_t V, int x, int y, int z,
                                   int t) {
  const int L0 = a.L[0], L1 = a.L[1], L2 = a.L[2], L3 = a.L[3];
  auto at = [&](int cy, int cz, int ct) { return 8u * unsigned(x + L0 * (cy + L1 * (cz + L2 * ct))); };
  const unsigned own = at(y, z, t);
  const unsigned yp = at(y + 1 == L1 ? 0 : y + 1, z, t), ym = at(y == 0 ? L1 - 1 : y - 1, z, t);
  const unsigned zp = at(y, z + 1 == L2 ? 0 : z + 1, t), zm = at(y, z == 0 ? L2 - 1 : z - 1, t);
  const unsigned tp = at(y, z, t + 1 == L3 ? 0 : t + 1), tm = at(y, z, t == 0 ? L3 - 1 : t - 1);
  const unsigned xp = x + 2 == L0 ? own - 8u * unsigned(x) : own + 16u;        // the number after the pair
  const unsigned xm = x == 0 ? own + 8u * unsigned(L0 - 1) : own - 8u;         // and the one before it
  const float cs = -0.5f * a.cw_f[0], ct = -0.5f * a.cw_f[3];
  const float ctf = (a.bc_t < 0 && t == L3 - 1) ? -ct : ct, ctb = (a.bc_t < 0 && t == 0) ? -ct : ct;
  constexpr float sf = DAG ? 1.f : -1.f, sb = -sf;
  constexpr int PARK = NR == 2 ? 16 : 0;
  __shared__ float4 park[PARK ? PARK : 1][kPairBlock];
  cf wa[NR][12], wb[NR][12], ta[NR][12], tb[NR][12];
  Two self[12];  // the pair's own numbers, where there are registers for them
  auto hop = [&](auto mu, auto fwd, unsigned nbo, float coef, int b) {
    constexpr int MU = decltype(mu)::value;
    constexpr bool F = decltype(fwd)::value;
    const float2* ul = U + size_t(MU) * 9 * V;
    const unsigned lo = F ? own : nbo;
    cf ua[3], ub[3];  // column b of U, or of U^dag
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const Two u = ld2(ul + (F ? 3 * c + b : 3 * b + c) * V, lo);
      ua[c] = F ? u.a : conj(u.a);
      ub[c] = F ? u.b : conj(u.b);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      cf ca[4], cb[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const Two v = ld2(in + (r * 12 + 3 * k + b) * V, nbo);
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
    {  // both x hops: the pair itself and the numbers on either side of it
      unsigned o = own;  // by another name in each colour: the links here would be kept for the next one
      asm volatile("" : "+v"(o));
      cf ufa[3], ufb[3], uba[3], ubb[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const Two u = ld2(U + (3 * c + b) * V, o);
        ufa[c] = u.a;
        ufb[c] = u.b;
        uba[c] = conj(ld1(U + (3 * b + c) * V, xm));
        ubb[c] = conj(ld1(U + (3 * b + c) * V, o));
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        cf pa[4], pb[4], ma[4], mb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float2* pl = in + (r * 12 + 3 * k + b) * V;
          const Two v = ld2(pl, o);
          if (NR == 1) self[3 * k + b] = v;
          pa[k] = v.b;
          pb[k] = ld1(pl, xp);
          ma[k] = ld1(pl, xm);
          mb[k] = v.a;
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
  if constexpr (CLOV) {
    cf va[NR][12], vb[NR][12];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const Two v = ld2(in + (r * 12 + k) * V, own);
        va[r][k] = v.a;
        vb[r][k] = v.b;
      }
    site_term<NR>(static_cast<const float2*>(a.clov), own, V, va, vb, wa, wb);
  } else {  // the large diagonal term last: added first, every hop would be rounded to its size
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const Two v = NR == 1 ? self[k] : ld2(in + (r * 12 + k) * V, own);
        wa[r][k] += a.diag_f * v.a;
        wb[r][k] += a.diag_f * v.b;
      }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int k = 0; k < 12; ++k) st2(out + (r * 12 + k) * V, own, wa[r][k], wb[r][k]);
}

// contiguous workgroups per XCD (workgroup b runs on XCD b mod 8)
__device__ inline int xcd_wg() {
  const int nb = gridDim.x, q = nb >> 3, x = blockIdx.x & 7;
  return x * q + min(x, nb & 7) + (blockIdx.x >> 3);
}

// One lattice: NR right-hand sides rhs_base + NR g .. of the workgroup's group g; planes (z, t) in patches of
// BZ x BT (bzt = BZ | BT << 8), as in k_hop_pair
template <int NR, bool DAG, bool CLOV>
__global__ __launch_bounds__(kBlock, 2) void k_dslash_pair(const float2* __restrict__ U, const float2* __restrict__ in,
                                                           float2* __restrict__ out, DslashArgs a, int rhs_base,
                                                           int ngroup, int bzt) {
  const int wg = xcd_wg();
  const int tile = wg / ngroup, rhs = rhs_base + NR * (wg - tile * ngroup);
  const int g = tile * kBlock + threadIdx.x;
  const int rp = a.L[0] >> 1, pp = rp * a.L[1];  // pairs of a row and of a plane
  if (g >= pp * a.L[2] * a.L[3]) return;
  int seq = g / pp;
  const int ip = g - seq * pp;
  const int BZ = bzt & 0xff, BT = bzt >> 8;
  const int tt = seq % BT;
  seq /= BT;
  const int zz = seq % BZ;
  seq /= BZ;
  const int nbz = a.L[2] / BZ;
  const int y = ip / rp;
  const size_t V = size_t(a.V), o = size_t(rhs) * 12 * V;
  pair_dslash<NR, DAG, CLOV>(U, in + o, out + o, a, V, 2 * (ip - y * rp), y, (seq % nbz) * BZ + zz,
                             (seq / nbz) * BT + tt);
}

// Many lattices in the padded layouts of k_dslash_padded (dslash.hip): ntile workgroups of 512 sites per
// (lattice, group of NR right-hand sides); numbers beyond a lattice's volume are written as zeros
template <int NR, bool DAG>
__global__ __launch_bounds__(kBlock, 2) void k_dslash_pair_padded(const BatchLattice* __restrict__ lat,
                                                                  const float2* __restrict__ U,
                                                                  const float2* __restrict__ in,
                                                                  float2* __restrict__ out, int nr, int ntile) {
  const int wg = xcd_wg();
  const int ng = nr / NR;
  const int g = wg % ng, tc = wg / ng;
  const int tile = tc % ntile, l = tc / ntile;
  const DslashArgs& a = lat[l].a;
  const int Vpad = a.V;
  const int site = 2 * (tile * kBlock + threadIdx.x);
  if (site >= Vpad) return;
  const size_t o = (size_t(l) * nr + g * NR) * 12 * Vpad;
  if (site >= a.L[0] * a.L[1] * a.L[2] * a.L[3]) {
    for (int k = 0; k < 12 * NR; ++k) st2(out + o + size_t(k) * Vpad, 8u * unsigned(site), {0.f, 0.f}, {0.f, 0.f});
    return;
  }
  int rem = site;
  const int x = rem % a.L[0]; rem /= a.L[0];
  const int y = rem % a.L[1]; rem /= a.L[1];
  pair_dslash<NR, DAG, false>(U + size_t(l) * 36 * Vpad, in + o, out + o, a, size_t(Vpad), x, y, rem % a.L[2],
                              rem / a.L[2]);
}

}  // namespace

bool dslash_pair_fits(const DslashArgs& a, const void* U, const void* in, const void* out) {
  uintptr_t bits = 0;
  for (const void* q : {U, in, out, a.clov}) bits |= reinterpret_cast<uintptr_t>(q);
  return a.L[0] % 2 == 0 && (bits & 15) == 0 && size_t(a.V) * 8 < (size_t(1) << 32);
}

void launch_dslash_pair(const void* U, const void* in, void* out, const DslashArgs& a, int nr, hipStream_t st) {
  const unsigned ntile = unsigned((a.V / 2 + kBlock - 1) / kBlock);
  // patches of 4 x 4 planes (32^3 x 64, 12 rhs: 2256 us; 8 x 8 2368, 2 x 2 2292, 1 x 8 2369)
  auto patch = [](int L) { return L % 4 == 0 ? 4 : L % 2 == 0 ? 2 : 1; };
  const int bzt = patch(a.L[2]) | (patch(a.L[3]) << 8);
  auto go = [&](auto kern, int base, int groups) {
    launch(kern, dim3(ntile * unsigned(groups)), dim3(kBlock), 0, st, static_cast<const float2*>(U),
           static_cast<const float2*>(in), static_cast<float2*>(out), a, base, groups, bzt);
  };
  auto run = [&](auto dag, auto cl) {
    constexpr bool D = decltype(dag)::value, CL = decltype(cl)::value;
    const int ng = nr == 2 ? a.nrhs / 2 : 0, done = 2 * ng;
    if (ng) go(k_dslash_pair<2, D, CL>, 0, ng);
    if (done < a.nrhs) go(k_dslash_pair<1, D, CL>, done, a.nrhs - done);
  };
  using T = std::true_type;
  using F = std::false_type;
  if (a.clov) a.dagger ? run(T{}, T{}) : run(F{}, T{});
  else a.dagger ? run(T{}, F{}) : run(F{}, F{});
  QMG_LAUNCH_CHECK();
}

void launch_dslash_pair_padded(const BatchLattice* lat, int nl, int nr, int Vpad, const void* U, const void* in,
                               void* out, bool dagger, hipStream_t st) {
  const int ntile = (Vpad / 2 + kBlock - 1) / kBlock;
  auto run = [&](auto nrc) {
    constexpr int NR = decltype(nrc)::value;
    const dim3 g(unsigned(ntile) * unsigned(nl) * unsigned(nr / NR));
    auto go = [&](auto kern) {
      launch(kern, g, dim3(kBlock), 0, st, lat, static_cast<const float2*>(U), static_cast<const float2*>(in),
             static_cast<float2*>(out), nr, ntile);
    };
    if (dagger) go(k_dslash_pair_padded<NR, true>);
    else go(k_dslash_pair_padded<NR, false>);
  };
  if (nr % 2 == 0) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, 1>{});
  QMG_LAUNCH_CHECK();
}

}  // namespace qmg
