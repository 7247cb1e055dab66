// The coarse operator on several right-hand sides, on the matrix cores.
//
// Row j of the coarse stencil is the sum over its nine blocks Y_slot(j) (m x m, column-major) times the
// right-hand sides at v(j + slot): a contraction over 9 m columns, bound by reading Y (1.4 GB at
// 32^3 x 64 with 4^4 aggregates, m = 48, FP32), which is read once for up to 16 right-hand sides.  A
// complex product becomes two real 16 x 16 x 4 matrix instructions: columns 2r and 2r + 1 of the real
// operand are the real and imaginary part of right-hand side r, once as they are (times Re Y) and once
// rotated (times Im Y).  A wavefront takes 16 rows of whole blocks, 16 columns at a time, so that its
// loads of Y are runs of a column, in address order, and none waits for another; the wavefronts'
// partial rows meet in the LDS.  The inputs come straight from memory (L2): at twelve right-hand sides
// they are as many loads as Y, so a lane loads two columns at once.
// Measured against groups of four right-hand sides on the vector units, FP32, rank 24: 32^3 x 64 with twelve
// right-hand sides 942 -> 363 us, eight 632 -> 269 us (5.1 TB/s of Y), 16^3 x 32 with twelve 52 -> 23.5 us;
// relative error against 64 bits 1.42e-7 -> 1.24e-7 and 1.16e-7.
#include <algorithm>
#include <type_traits>

#include "mfma.hpp"
#include "mg.hpp"
#include "timing.hpp"

namespace qmg {

namespace {

// NQ: tiles of 16 rows or columns, NT: groups of 8 right-hand sides.  Row h is aggregate list[h] (or h
// itself); wavefront (w, u) forms row tile u of the slots lo + w, lo + w + W, ... below hi.
template <class S, int NQ, int NT, int W>
__global__ __launch_bounds__(64 * NQ * W, 4) void k_coarse_mm(
    const S* __restrict__ Y, const S* __restrict__ y, const S* __restrict__ a, const S* __restrict__ b,
    S* __restrict__ out, const int* __restrict__ list, const int* __restrict__ nb, int d, int m, int nrhs, int lo,
    int hi, double sgn, const int* __restrict__ skip) {
  using C = ctype<S>;
  using M = Mm<C>;
  using V4 = typename M::V4;
  // chains of sums of a slot: Re Y and Im Y apart and, where the registers have room, even and odd columns
  constexpr int G = sizeof(C) == 8 && NT == 2 ? 2 : 4;
  constexpr int LD = 16 * NQ + 1;
  if (skip && *skip) return;  // device-side early exit of a converged coarse solve
  extern __shared__ __align__(16) unsigned char smem[];
  C* part = reinterpret_cast<C*>(smem);  // [W][8 NT][LD] complex
  const int lane = threadIdx.x & 63, li = lane & 15, kk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), u = wave % NQ, w = wave / NQ;
  const int h = xcd_local(blockIdx.x, gridDim.x), j = list ? list[h] : h;
  const int r0 = blockIdx.y * 8 * NT, R = min(8 * NT, nrhs - r0);
  const int im = li & 1;
  V4 tot[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) tot[nt] = V4{C(0), C(0), C(0), C(0)};
  const int row = min(16 * u + li, m - 1);
  for (int slot = lo + w; slot < hi; slot += W) {
    const int from = slot == 0 ? h : nb[j * 8 + slot - 1];
    const S* in = (slot == 0 ? a : b) + (size_t(r0) * d + from) * m;
    const S* Yb = Y + (size_t(j) * 9 + slot) * m * m;
    V4 acc[NT][G];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int g = 0; g < G; ++g) acc[nt][g] = V4{C(0), C(0), C(0), C(0)};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      // rows past m and right-hand sides past R repeat the last one (their results go nowhere); columns
      // past m, in the last 16 only, count as zero
      cplx<C> ym[4];
      C br[4][NT], bi[4][NT];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int c = 16 * q + 4 * kk + s, col = q == NQ - 1 ? min(c, m - 1) : c;
        ym[s] = ldc(Yb, size_t(col * m + row));
        if (q == NQ - 1 && c >= m) ym[s] = {C(0), C(0)};
      }
      // a lane needs one part of its right-hand side at four columns: of the two lanes of a right-hand
      // side, the even one loads the first two columns, the odd one the others, and they swap
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int c = 16 * q + 4 * kk + 2 * im, col = q == NQ - 1 ? min(c, m - 2) : c;
        S raw[2];
        __builtin_memcpy(raw, in + size_t(min(nt * 8 + (li >> 1), R - 1)) * d * m + col, sizeof raw);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          cplx<C> mine = StoreTraits<S>::ld(raw[e]);
          if (q == NQ - 1 && c >= m) mine = {C(0), C(0)};
          const cplx<C> other = {dpp_move<0xB1, 0xF>(mine.re), dpp_move<0xB1, 0xF>(mine.im)};  // quad_perm [1,0,3,2]
          br[e][nt] = im ? other.im : mine.re;
          bi[e][nt] = im ? other.re : -mine.im;
          br[2 + e][nt] = im ? mine.im : other.re;
          bi[2 + e][nt] = im ? mine.re : -other.im;
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int g = G == 4 ? 2 * (s & 1) : 0;
          acc[nt][g] = M::mul(ym[s].re, br[s][nt], acc[nt][g]);
          acc[nt][g + 1] = M::mul(ym[s].im, bi[s][nt], acc[nt][g + 1]);
        }
    }
    const C sg = slot == 0 ? C(1) : C(sgn);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int g = G / 2; g >= 1; g /= 2)
#pragma unroll
        for (int i = 0; i < g; ++i) acc[nt][i] += acc[nt][i + g];
      tot[nt] += sg * acc[nt][0];
    }
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      part[((w * 8 * NT + nt * 8 + (li >> 1)) * LD + 16 * u + M::row(lane, e)) * 2 + im] = tot[nt][e];
  __syncthreads();
  for (int t = threadIdx.x; t < R * m; t += blockDim.x) {
    const int r = t / m, row = t - r * m;
    cplx<C> s = {C(0), C(0)};
    for (int q = 0; q < W; ++q) {
      const C* p = part + ((q * 8 * NT + r) * LD + row) * 2;
      s += cplx<C>{p[0], p[1]};
    }
    const size_t o = (size_t(r0 + r) * d + h) * m + row;
    if (y) s += ldc(y, o);
    stc(out, o, s);
  }
}

}  // namespace

// From that many rows on, one group of wavefronts forms a row's nine blocks one after the other; with fewer
// the blocks are dealt out over three or five groups, so that the chip is filled.  FP32, rank 24, 8 / 12
// right-hand sides: 512 rows 22.2 / 33.8 us one group, 15.8 / 24.0 us several; 2592 rows (rank 12) 27.4 / 47.5
// against 28.1 / 59.2 us; 8192 rows 270 / 364 against 376 / 604 us.
constexpr int kCoarseMmRows = 2048;

// Where the matrix cores are the faster, us, a thread per two rows and chunk of columns (groups of four right-hand
// sides) / here.  Rows and columns are padded to tiles of 16, so that a fourth tile (ranks above 24) and, up to four
// right-hand sides, ranks between the tiles lose: 2592 rows, three right-hand sides, FP32 rank 24 104 / 95, 22 81 / 89, 20
// 74 / 78, 16 43 / 31, 10 28 / 25; FP64, whose matrix instructions run at the rate of its vector units, rank 24 239 / 186, 20
// 133 / 162, 16 87 / 76, 12 48 / 44 (512 rows: 10.8 / 12.2), 8 32 / 18.  From five on the other form reads Y twice
// (2592 rows, FP32 rank 20 138 / 79, FP64 rank 18 271 / 156), but groups of four on fewer rows than CUs run beside each
// other (64 rows, 8 rhs, FP64 rank 18 8.8 / 12.1, rank 24 13.5 / 12.3, FP32 rank 18 7.3 / 7.9, rank 20 7.8 / 7.8; 32 rows, 12 rhs,
// FP64 rank 24 11.9 / 12.2).
bool coarse_mm_fits(qmg_prec prec, int d, int k, int nrhs) {
  if (nrhs < 3 || k > 32) return false;
  if (k <= 8) return true;
  if (k > 24) return nrhs >= 5;
  const bool f64 = prec == QMG_F64, crowd = long(d) * nrhs >= 1024;
  if (nrhs >= 5) return k <= 16 || crowd || (!f64 && k >= 20) || (k == 24 && d >= 64);
  if (f64) return k == 16 || (k == 24 && d >= 512);
  return k <= 16 || k == 24 || (k >= 20 && d >= 128 && d < 1024);
}

template <class S>
void launch_coarse_mm(const CoarseMm& c, int d, int k, int nrhs, hipStream_t st, const int* skip) {
  const int m = 2 * k, lo = c.a ? 0 : 1, hi = c.b ? 9 : 1;
  auto go = [&](auto nq, auto ntt, auto wt) {
    constexpr int NQ = decltype(nq)::value, NT = decltype(ntt)::value, W = std::min(decltype(wt)::value, 16 / NQ);
    const size_t lds = size_t(W) * 8 * NT * (16 * NQ + 1) * sizeof(cplx<ctype<S>>);
    auto kern = k_coarse_mm<S, NQ, NT, W>;
    if (lds > 64 * 1024)
      QMG_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    launch(kern, dim3(d, (nrhs + 8 * NT - 1) / (8 * NT)), dim3(64 * W * NQ), uint32_t(lds), st,
           static_cast<const S*>(c.Y), static_cast<const S*>(c.y), static_cast<const S*>(c.a),
           static_cast<const S*>(c.b), static_cast<S*>(c.out), c.list, c.nb, d, m, nrhs, lo, hi, c.sgn, skip);
  };
  auto rows = [&](auto ntt, auto wt) {
    if (m <= 16) go(std::integral_constant<int, 1>{}, ntt, wt);
    else if (m <= 32) go(std::integral_constant<int, 2>{}, ntt, wt);
    else if (m <= 48) go(std::integral_constant<int, 3>{}, ntt, wt);
    else go(std::integral_constant<int, 4>{}, ntt, wt);
  };
  using one = std::integral_constant<int, 1>;
  using two = std::integral_constant<int, 2>;
  // 16 right-hand sides a pass, but 8 where a pass of 16 leaves too few workgroups (32 rows, 12 right-hand
  // sides: 8.2 us in passes of 8, 10.5 us in one)
  if (nrhs <= 8 || d < 128) {
    if (d >= kCoarseMmRows) rows(one{}, one{});
    else rows(one{}, std::integral_constant<int, 3>{});
  } else {
    if (d >= kCoarseMmRows) rows(two{}, one{});
    else rows(two{}, std::integral_constant<int, 5>{});
  }
}

template void launch_coarse_mm<double2>(const CoarseMm&, int, int, int, hipStream_t, const int*);
template void launch_coarse_mm<float2>(const CoarseMm&, int, int, int, hipStream_t, const int*);
template void launch_coarse_mm<cbf16>(const CoarseMm&, int, int, int, hipStream_t, const int*);
template void launch_coarse_mm<chalf>(const CoarseMm&, int, int, int, hipStream_t, const int*);

}  // namespace qmg
