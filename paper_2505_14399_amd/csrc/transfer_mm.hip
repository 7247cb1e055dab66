// Prolongation and restriction (Eq. (6)) on the matrix cores, on native or canonical fine vectors.
//
// Both are products of the aggregates' P blocks (rows x rank) with a few right-hand sides, bound by
// reading P (4.8 GB at 32^3 x 64, rank 24, FP32), so P is read once for up to 16 right-hand sides.  A
// complex product becomes two real 16 x 16 x 4 matrix instructions: columns 2r and 2r + 1 of the real
// operand are the real and imaginary part of right-hand side r, once as they are (times Re P) and
// once rotated (times Im P).  A lane loads two consecutive rows of a column of P, which feed two
// instructions; sums are in FP32 (FP64) as the vectors' type has it.
// The sites of an aggregate are taken IB = 32 at a time (16 where a block has 16, and to restrict), all
// components of them together: their fine vectors pass through the LDS, so that the canonical layout
// is read and written in whole runs of sites (96 bytes each in FP32) and needs no packed copy.
// Measured at 32^3 x 64, rank 24, FP32, 12 right-hand sides on canonical vectors, against groups of
// four with packed copies: prolong 5.5 -> 1.45 ms (5.0 TB/s of P and vectors), restrict 5.2 -> 1.76 ms.  Where the
// other form is the faster stands at prolong_mm_fits and restrict_mm_fits.
// Relative error against 64 bits at 16^3 x 32: restrict 9.8e-8 -> 8.0e-8, prolong 9.7e-8 -> 7.5e-8.
#include <algorithm>
#include <type_traits>

#include "mfma.hpp"
#include "mg.hpp"
#include "timing.hpp"

namespace qmg {

namespace {

constexpr int kMmSites = 1024;  // largest block

struct MmArgs {
  const int* bsite;
  int nd, N, k, d, V, nrhs, nchunk, cpw;
};

// Workgroup: cpw chunks of IB sites of aggregate j for right-hand sides 8 NT blockIdx.y ..; wavefronts
// 0, 1 form the rows of chirality 0, wavefronts 2, 3 those of chirality 1, in tiles of 32 rows.
template <class S, int KC, int NT, int IB, bool CANON>
__global__ __launch_bounds__(256) void k_prolong_mm(const S* __restrict__ P, const S* __restrict__ vc,
                                                    S* __restrict__ fine, MmArgs a) {
  using C = ctype<S>;
  using M = Mm<C>;
  using V4 = typename M::V4;
  constexpr int T = 6 * IB / 32;
  extern __shared__ __align__(16) unsigned char smem[];
  S* buf = reinterpret_cast<S*>(smem);  // [R][IB][12] canonical, [R][12][IB] native
  __shared__ int sites[IB];
  const int lane = threadIdx.x & 63, li = lane & 15, kk = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), al = w >> 1;
  const int wg = xcd_local(blockIdx.x, gridDim.x);
  const int per = (a.nchunk + a.cpw - 1) / a.cpw;
  const int j = wg / per, ch0 = (wg - j * per) * a.cpw, ch1 = min(a.nchunk, ch0 + a.cpw);
  const int r0 = blockIdx.y * 8 * NT, R = min(8 * NT, a.nrhs - r0);
  const bool im = lane & 1;
  // the coarse coefficients: column n = li of the real operand, rank index 4 c + kk
  C br[KC][NT], bi[KC][NT];
#pragma unroll
  for (int c = 0; c < KC; ++c)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int i = 4 * c + kk, r = nt * 8 + (li >> 1);
      cplx<C> v{C(0), C(0)};
      if (i < a.k && r < R) v = ldc(vc, (size_t(r0 + r) * a.d + j) * 2 * a.k + al * a.k + i);
      br[c][nt] = im ? v.im : v.re;
      bi[c][nt] = im ? v.re : -v.im;
    }
  const S* Pj = P + (size_t(j) * 2 + al) * a.k * a.N;
  for (int ch = ch0; ch < ch1; ++ch) {
    if (threadIdx.x < IB) sites[threadIdx.x] = a.bsite[size_t(j) * a.nd + ch * IB + threadIdx.x];
#pragma unroll
    for (int tq = 0; tq < (T + 1) / 2; ++tq) {
      const int q = 2 * tq + (w & 1);  // tile: rows 32 q + (0 .. 31) of the chunk
      if (q < T) {
        const int lr = 32 * q + 2 * li, s6 = lr / IB, il = lr % IB;
        const size_t row = size_t(s6) * a.nd + ch * IB + il;
        // Re P and Im P, even and odd groups of ranks apart: short chains of roundings
        V4 part[2][NT][4], acc[2][NT];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int g = 0; g < 4; ++g) part[t][nt][g] = V4{C(0), C(0), C(0), C(0)};
        Pk<S, 2> pv[KC];
#pragma unroll
        for (int c = 0; c < KC; ++c) {
          const int i = 4 * c + kk;
          pv[c] = Pk<S, 2>{};
          if (i < a.k) pv[c] = *reinterpret_cast<const Pk<S, 2>*>(Pj + size_t(i) * a.N + row);
        }
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const cplx<C> p = StoreTraits<S>::ld(pv[c].v[t]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              const int g = 2 * (c & 1);
              part[t][nt][g] = M::mul(p.re, br[c][nt], part[t][nt][g]);
              part[t][nt][g + 1] = M::mul(p.im, bi[c][nt], part[t][nt][g + 1]);
            }
          }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[t][nt] = (part[t][nt][0] + part[t][nt][1]) + (part[t][nt][2] + part[t][nt][3]);
        // an even lane holds real parts, the odd one beside it the imaginary parts: the even lane
        // finishes the tile's even rows (t = 0), the odd lane its odd rows
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int r = nt * 8 + (li >> 1);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const C send = im ? acc[0][nt][v] : acc[1][nt][v];
            const C got = dpp_move<0xB1, 0xF>(send);  // quad_perm [1,0,3,2]
            const cplx<C> o = im ? cplx<C>{got, acc[1][nt][v]} : cplx<C>{acc[0][nt][v], got};
            const int lo = 32 * q + 2 * M::row(lane, v) + (im ? 1 : 0), so = lo / IB, io = lo % IB;
            if (r < R)
              buf[CANON ? (r * IB + io) * 12 + 6 * al + so : (r * 12 + 6 * al + so) * IB + io] = StoreTraits<S>::st(o);
          }
        }
      }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < R * 12 * IB; e += 256) {
      const int r = e / (12 * IB), f = e - r * 12 * IB;
      const int comp = CANON ? f % 12 : f / IB, il = CANON ? f / 12 : f % IB;
      fine[fine_idx<CANON>(r0 + r, comp, sites[il], a.V)] = buf[e];
    }
    __syncthreads();
  }
}

// Workgroup: a chirality of aggregate j, right-hand sides 8 NT blockIdx.y ..; each wavefront sums every
// fourth step of 8 rows of a chunk of 16 sites.  A fragment of P holds
// 16 columns, whose rows lie a whole column apart, so P passes through the LDS too (read straight
// into the fragments, loads of 16 segments took 3.2 ms at 32^3 x 64 with 12 right-hand sides).  The next chunk is loaded while the present one is summed.  Chunk sums run in short chains
// (Re P and Im P, even and odd rows apart) and are added up in FP64, so that the result is no further
// from the exact one than a sum over threads.
template <class S, int MT, int NT, bool CANON>
__global__ __launch_bounds__(256) void k_restrict_mm(const S* __restrict__ P, const S* __restrict__ fine,
                                                     S* __restrict__ vc, MmArgs a) {
  using C = ctype<S>;
  using M = Mm<C>;
  using V4 = typename M::V4;
  using P2 = Pk<S, 2>;
  constexpr int IB = 16, ROWS = 6 * IB;
  constexpr int PS = ROWS + 8;  // stride in the LDS (the 8 spread the lanes' banks)
  constexpr int NE = (8 * NT * ROWS + 255) / 256;             // numbers of the vectors per thread
  constexpr int NP = (16 * MT * (ROWS / 2) + 255) / 256;      // row pairs of P per thread
  constexpr int NS = ROWS / 8 / 4;                              // steps of a chunk per wavefront
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, li = lane & 15, kk = lane >> 4;
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ja = xcd_local(blockIdx.x, gridDim.x), j = ja >> 1, al = ja & 1;
  const int r0 = blockIdx.y * 8 * NT, R = min(8 * NT, a.nrhs - r0);
  const bool im = lane & 1;
  S* pbuf = reinterpret_cast<S*>(smem);    // [k] columns of ROWS, stride PS
  S* buf = pbuf + size_t(a.k) * PS;        // [R][ROWS], stride PS
  // the aggregate's sites: looked up in memory inside fetch, a site would hold up the loads behind it
  int* bs = reinterpret_cast<int*>(buf + size_t(min(8 * NT, a.nrhs)) * PS);
  for (int i = threadIdx.x; i < a.nd; i += 256) bs[i] = a.bsite[size_t(j) * a.nd + i];
  __syncthreads();
  const S* Pj = P + size_t(ja) * a.k * a.N;
  S t[NE];
  typedef unsigned Raw __attribute__((ext_vector_type(sizeof(P2) / 4)));  // (an array of packs lands in scratch memory)
  Raw tp[NP];
  auto fetch = [&](int ch) {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int e = u * 256 + threadIdx.x, col = e / (ROWS / 2), lr = 2 * (e - col * (ROWS / 2));
      if (col < a.k)
        tp[u] = *reinterpret_cast<const Raw*>(Pj + size_t(col) * a.N + size_t(lr / IB) * a.nd + ch * IB + lr % IB);
    }
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const int e = u * 256 + threadIdx.x;
      if (e < R * ROWS) {
        const int r = e / ROWS, f = e - r * ROWS;
        const int s6 = CANON ? f % 6 : f / IB, il = CANON ? f / 6 : f % IB;
        t[u] = fine[fine_idx<CANON>(r0 + r, 6 * al + s6, bs[ch * IB + il], a.V)];
      }
    }
  };
  double acc[MT][NT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[m][nt][v] = 0;
  // Columns of P and aggregates lie multiples of 4 KB apart (4^4 blocks), so workgroups on the same
  // chunk would all meet the same L2 and memory channels: each starts at another one
  int ch = j % a.nchunk;
  fetch(ch);
  for (int n = 0; n < a.nchunk; ++n) {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int e = u * 256 + threadIdx.x, col = e / (ROWS / 2), lr = 2 * (e - col * (ROWS / 2));
      if (col < a.k) *reinterpret_cast<Raw*>(pbuf + col * PS + lr) = tp[u];
    }
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const int e = u * 256 + threadIdx.x;
      if (e < R * ROWS) {
        const int r = e / ROWS, f = e - r * ROWS;
        const int s6 = CANON ? f % 6 : f / IB, il = CANON ? f / 6 : f % IB;
        buf[r * PS + s6 * IB + il] = t[u];
      }
    }
    __syncthreads();
    ch = ch + 1 == a.nchunk ? 0 : ch + 1;
    if (n + 1 < a.nchunk) fetch(ch);
    V4 part[4][MT][NT];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) part[q][m][nt] = V4{C(0), C(0), C(0), C(0)};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int lr = 8 * (4 * s + sub) + 2 * kk;
      cplx<C> pv[MT][2];
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        pv[m][0] = pv[m][1] = {C(0), C(0)};
        if (m * 16 + li < a.k) {
          const P2 p = *reinterpret_cast<const P2*>(pbuf + (m * 16 + li) * PS + lr);
          pv[m][0] = StoreTraits<S>::ld(p.v[0]);
          pv[m][1] = StoreTraits<S>::ld(p.v[1]);
        }
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int r = nt * 8 + (li >> 1);
        cplx<C> f[2] = {{C(0), C(0)}, {C(0), C(0)}};
        if (r < R) {
          const P2 q = *reinterpret_cast<const P2*>(buf + r * PS + lr);
          f[0] = StoreTraits<S>::ld(q.v[0]);
          f[1] = StoreTraits<S>::ld(q.v[1]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const cplx<C> x = f[h];
          const C xr = im ? x.im : x.re, xi = im ? -x.re : x.im;
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const cplx<C> p = pv[m][h];
            part[2 * h][m][nt] = M::mul(p.re, xr, part[2 * h][m][nt]);
            part[2 * h + 1][m][nt] = M::mul(p.im, xi, part[2 * h + 1][m][nt]);
          }
        }
      }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          acc[m][nt][v] += double((part[0][m][nt][v] + part[1][m][nt][v]) + (part[2][m][nt][v] + part[3][m][nt][v]));
    __syncthreads();
  }
  // wavefronts 1..3 leave their sums, 0 adds and stores
  double* red = reinterpret_cast<double*>(smem);  // [3][MT][NT][4][64]
  constexpr int RW = MT * NT * 4 * 64;
  if (sub) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(sub - 1) * RW + ((m * NT + nt) * 4 + v) * 64 + lane] = acc[m][nt][v];
  }
  __syncthreads();
  if (sub) return;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double s = acc[m][nt][v];
#pragma unroll
        for (int q = 0; q < 3; ++q) s += red[q * RW + ((m * NT + nt) * 4 + v) * 64 + lane];
        const double other = dpp_move<0xB1, 0xF>(s);  // the imaginary part, for the even lanes
        const int i = m * 16 + M::row(lane, v), r = nt * 8 + (li >> 1);
        if (!im && i < a.k && r < R)
          stc(vc, (size_t(r0 + r) * a.d + j) * 2 * a.k + al * a.k + i, cplx<double>{s, other});
      }
}

template <class F>
void by_prec(qmg_prec p, F&& f) {
  switch (p) {
    case QMG_F64: f(double2{}); break;
    case QMG_F32: f(float2{}); break;
    case QMG_BF16: f(cbf16{}); break;
    case QMG_F16: f(chalf{}); break;
  }
}
template <class F>
void by_layout(int nd, bool canonical, F&& f) {
  using I16 = std::integral_constant<int, 16>;
  using I32 = std::integral_constant<int, 32>;
  if (nd == 16) canonical ? f(I16{}, std::true_type{}) : f(I16{}, std::false_type{});
  else canonical ? f(I32{}, std::true_type{}) : f(I32{}, std::false_type{});
}
template <class F>
void by_nt(int nrhs, F&& f) {
  if (nrhs > 8) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, 1>{});
}

}  // namespace

// Blocks of 16 or a multiple of 32 sites, rank up to 32; from two right-hand sides on.  A single one is
// faster one row pack per thread (transfer.hip): restrict / prolong at 16^3 x 32, rank 24, us, one
// right-hand side FP32 56 / 57 against 77 / 69 here, FP64 119 / 115 against 144 / 123; four FP32
// 112 / 94 against 80 / 70.
static bool mm_shape(const HierarchyDev& h, int nrhs) {
  return nrhs > 1 && (h.blk.nd == 16 || h.blk.nd % 32 == 0) && h.blk.nd <= kMmSites && h.k <= 32;
}

// Native vectors need no packed copy, so up to four right-hand sides, which the row packs too take in one pass over P,
// those are the faster on blocks of 32 sites or more where their threads fill the chip (rank 24, us, row packs /
// here): FP32 from 2^18 sites (32^3 x 64 with 4 rhs 1380 / 1440, 24^3 x 48 with 2 344 / 382, 16^2 x 32^2 with 3 149 / 153;
// 16^3 x 32 with 2 74 / 67), FP64 from 2^15 (24^4 with 4 340 / 370, 16^3 x 32 with 2 127 / 135; 8^3 x 16 10.4 / 9.6), and 16-bit
// storage with two (16^3 x 32 40 / 43, with 4 56 / 50).  Blocks of 16 sites: 12^3 x 24, rank 12, FP32 with 4 25 / 19, BF16 with
// 2 20 / 16, FP64 with 2 28.8 / 29.7, rank 8 22.3 / 20.4.
bool prolong_mm_fits(qmg_prec prec, const HierarchyDev& h, int nrhs, bool canonical) {
  if (!mm_shape(h, nrhs)) return false;
  if (canonical || nrhs > 4) return true;
  if (h.blk.nd == 16) return prec != QMG_F64 || nrhs > 2 || h.k <= 8;
  if (prec == QMG_F64) return h.g.V < (1 << 15);
  return prec == QMG_F32 ? h.g.V < (1 << 18) : nrhs > 2;
}

// In FP64 a workgroup of the few aggregates of a small lattice has more to do here than with groups of four (8^3 x 16,
// rank 24, native, 5 rhs: row packs 52 us, here 56; 4 rhs 54 / 53).
bool restrict_mm_fits(qmg_prec prec, const HierarchyDev& h, int nrhs, bool canonical) {
  return mm_shape(h, nrhs) && (canonical || prec != QMG_F64 || nrhs <= 4 || h.blk.d >= 128);
}

void launch_prolong_mm(qmg_prec prec, const HierarchyDev& h, const void* P, const void* coarse, void* fine, int nrhs,
                       bool canonical, hipStream_t st) {
  MmArgs a{h.bsite.as<int>(), h.blk.nd, h.blk.N, h.k, h.blk.d, h.g.V, nrhs, 0, 1};
  by_prec(prec, [&](auto tag) {
    using S = decltype(tag);
    by_layout(h.blk.nd, canonical, [&](auto ibc, auto canon) {
      constexpr int IB = decltype(ibc)::value;
      constexpr bool CA = decltype(canon)::value;
      a.nchunk = a.nd / IB;
      a.cpw = std::max(1, std::min(a.nchunk, int(long(a.d) * a.nchunk / 2048)));
      by_nt(nrhs, [&](auto ntc) {
        constexpr int NT = decltype(ntc)::value;
        const int G = 8 * NT;
        const size_t lds = size_t(std::min(G, nrhs)) * 12 * IB * sizeof(S);
        const dim3 grid(unsigned(a.d) * unsigned((a.nchunk + a.cpw - 1) / a.cpw), unsigned((nrhs + G - 1) / G));
        auto go = [&](auto kern) {
          if (lds > 64 * 1024)
            QMG_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
          launch(kern, grid, dim3(256), uint32_t(lds), st, static_cast<const S*>(P), static_cast<const S*>(coarse),
                 static_cast<S*>(fine), a);
        };
        if (h.k <= 8) go(k_prolong_mm<S, 2, NT, IB, CA>);
        else if (h.k <= 16) go(k_prolong_mm<S, 4, NT, IB, CA>);
        else if (h.k <= 24) go(k_prolong_mm<S, 6, NT, IB, CA>);
        else go(k_prolong_mm<S, 8, NT, IB, CA>);
      });
    });
  });
  QMG_LAUNCH_CHECK();
}

void launch_restrict_mm(qmg_prec prec, const HierarchyDev& h, const void* P, const void* fine, void* coarse, int nrhs,
                        bool canonical, hipStream_t st) {
  MmArgs a{h.bsite.as<int>(), h.blk.nd, h.blk.N, h.k, h.blk.d, h.g.V, nrhs, 0, 1};
  a.nchunk = a.nd / 16;
  by_prec(prec, [&](auto tag) {
    using S = decltype(tag);
    // 16 right-hand sides a pass only where one pass fills the chip: with fewer than two workgroups a CU, passes of 8
    // run beside each other (FP64, 8^3 x 16, rank 24, 12 rhs: 87.5 us in one pass, in two 55.7; row packs 71)
    by_nt(a.d < 256 ? 8 : nrhs, [&](auto ntc) {
      constexpr int NT = decltype(ntc)::value;
      const int G = 8 * NT;
      auto go = [&](auto kern, int MT) {
        const size_t lds = std::max(size_t(h.k + std::min(G, nrhs)) * 104 * sizeof(S) + size_t(a.nd) * sizeof(int),
                                    size_t(3) * MT * NT * 256 * sizeof(double));
        if (lds > 64 * 1024)
          QMG_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
        launch(kern, dim3(2 * unsigned(a.d), unsigned((nrhs + G - 1) / G)), dim3(256), uint32_t(lds), st,
               static_cast<const S*>(P), static_cast<const S*>(fine), static_cast<S*>(coarse), a);
      };
      auto by_rank = [&](auto canon) {
        constexpr bool CA = decltype(canon)::value;
        if (h.k <= 16) go(k_restrict_mm<S, 1, NT, CA>, 1);
        else go(k_restrict_mm<S, 2, NT, CA>, 2);
      };
      if (canonical) by_rank(std::true_type{});
      else by_rank(std::false_type{});
    });
  });
  QMG_LAUNCH_CHECK();
}

}  // namespace qmg
