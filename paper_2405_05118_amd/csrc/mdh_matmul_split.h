// What the kernels of MatMul on three-slice values share: the evaluation in fp32 of blocks that hold values the split does
// not carry, and the search for elements too small to split exactly (mdh_split.h).  Y[i,k], X[j,k]: YK, XK = stored with
// k contiguous ([row][k], pitch ld), else with the rows contiguous ([k][row]).
#pragma once
#include "mdh_split.h"

namespace mdh {
namespace split {

// four consecutive k of a row; unless all = true, elements at or beyond kend as 0
template <bool KC>
__device__ __forceinline__ f4 four_k(const float* __restrict__ P, int64_t ld, int row, int k, int kend, bool all) {
  if (KC && all) return *(const f4u*)(P + row * ld + k);
  f4 v;
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = all || k + t < kend ? (KC ? P[row * ld + k + t] : P[(k + t) * ld + row]) : 0.f;
  return v;
}

// fp32 evaluation of MB x NB blocks from (m, n) on by one wavefront, for values the split does not carry; 8 KS k at a
// time, the next ones on their way while these are multiplied.  Rows below mlo and columns below nlo are not stored.
template <int MB, int NB, int KS, bool YK, bool XK>
__device__ __forceinline__ void recompute_fp32(const float* __restrict__ Y, const float* __restrict__ X, float* __restrict__ Cout,
                                            int M, int N, int64_t ldy, int64_t ldx, int m, int n, int kbeg, int kend, int mlo = 0,
                                            int nlo = 0) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  if (m >= M || n >= N) return;
  f16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  f4 y[KS][MB], x[KS][NB];
  auto load_ = [&](int k0, bool all) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int i = 0; i < MB; ++i) y[s][i] = four_k<YK>(Y, ldy, min(m + i * 32 + l32, M - 1), k0 + s * 8 + lh * 4, kend, all);
#pragma unroll
      for (int j = 0; j < NB; ++j) x[s][j] = four_k<XK>(X, ldx, min(n + j * 32 + l32, N - 1), k0 + s * 8 + lh * 4, kend, all);
    }
  };
  auto load = [&](int k0) {
    if (k0 + 8 * KS <= kend)
      load_(k0, true);
    else
      load_(k0, false);
  };
  load(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += 8 * KS) {
    f4 yc[KS][MB], xc[KS][NB];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int i = 0; i < MB; ++i) yc[s][i] = y[s][i];
#pragma unroll
      for (int j = 0; j < NB; ++j) xc[s][j] = x[s][j];
    }
    if (k0 + 8 * KS < kend) load(k0 + 8 * KS);
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(yc[s][i][t], xc[s][j][t], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ro = m + i * 32 + 8 * (r / 4) + 4 * lh + (r % 4), co = n + j * 32 + l32;
        if (ro >= mlo && ro < M && co >= nlo && co < N) Cout[(int64_t)ro * N + co] = acc[i][j][r];
      }
}

// does the workgroup's part of an operand, or of its listed rows where they are few, hold an element too small to split
// exactly?  (this thread's share)
template <int ROWS, int NT, bool KC>
__device__ __forceinline__ bool holds_tiny(const float* __restrict__ P, int64_t ld, int r0, int rmax, int kbeg, int kend, const Marks& m) {
  bool t = false;
  const unsigned n = *m.count;
  if (n <= Marks::kFew) {
    for (unsigned i = 0; i < n; ++i) {
      const int r = min(r0 + m.list[i], rmax - 1);
      if (KC)
        t |= tiny_in(P + r * ld + kbeg, kend - kbeg, threadIdx.x, NT);
      else
        for (int k = kbeg + threadIdx.x; k < kend; k += NT) t |= tiny(P[k * ld + r]);
    }
    return t;
  }
  const int rows = min(ROWS, rmax - r0);
  constexpr int W = 16;  // threads per contiguous run
  if (KC) {
    for (int r = threadIdx.x / W; r < rows; r += NT / W) t |= tiny_in(P + (r0 + r) * ld + kbeg, kend - kbeg, threadIdx.x % W, W);
  } else {
    for (int k = kbeg + threadIdx.x / W; k < kend; k += NT / W) t |= tiny_in(P + k * ld + r0, rows, threadIdx.x % W, W);
  }
  return t;
}

}  // namespace split
}  // namespace mdh
