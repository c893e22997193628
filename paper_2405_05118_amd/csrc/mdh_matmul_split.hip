// MatMul / bMatMul / MatMul^T instance of md_hom(*, (++,++,+)) for gfx950 on the bf16 matrix instructions, every
// fp32 value carried as a sum of three bf16 values (mdh_split.h: six products per multiply-add, accuracy of fp32).
//
// De-composition, dims (b,i,j,k):
//   workgroup layer : batch x (M/BM) x (N/BN) x S
//   HBM layer       : K/(BK S) sequential k-tiles, split into their three slices on the way to LDS (double buffered)
//   wavefront layer : (BM/WM) x (BN/WN)
//   LDS layer       : BK/16 sequential k-steps
//   VGPR layer      : (WM/32) x (WN/32) accumulator blocks per wavefront
//   block           : 32 x 32 x 16, six v_mfma_f32_32x32x16_bf16
// LDS layout of an operand: [slice][k / 8][row], 16 bytes (eight k of a row) per entry: the MFMA operand of a
// lane is one ds_read_b128, and 32 lanes read 512 contiguous bytes.  Rows are swizzled inside groups of eight so that
// the writes of a k-contiguous operand (BK/8 lanes per row) spread over the banks too (no bank conflicts counted).
//
// What bounds it.  Large products: power.  4096^3 runs at 1.9 GHz, and leaving single parts of the work out took off
// (256 x 128 tiles, when they took 738 us, before the buffer loads) loads 187, LDS reads 159, the split 110, LDS writes
// 55, and MFMAs alone were 417 us: the parts add up instead of overlapping.  So what counts is bytes and instructions per
// product, and the largest tile wins: 4096^3 256 x 256 588 us, 256 x 128 646, 128 x 128 710, 128 x 64 794, 64 x 64 879
// (fp32 instructions: 1010-1070); where that leaves compute units idle, smaller ones: 2048^3 237, 140, 94, 110, 126
// (145).  The split keeps out of the matrix pipe (mdh_split.h) and is spread evenly over the phases: 4096^3 600 -> 571 us,
// 16 x 1024^3 165 -> 156.  64 x 64 tiles, whose walk is more split than products, lose by it (1021 x 1531 x 777 25.6 ->
// 26.7 us), but k over the wavefronts (mdh_matmul_split_k.hip) is faster there.  The 256 x 256 tile has k-tiles of 16, because two of 32 (192 KB) exceed LDS.  Measured when they were chosen:
// 16x16x32 MFMAs equal at 4096^3 (717 / 726), slower at 1024^3 in 128 x 128 tiles (55.2 / 48.8) -- the smaller one
// leaves room for one vector instruction beside it, the larger for four; 128 x 128 tiles on eight wavefronts of 32 x 64
// rather than four of 64 x 64 (2048^3 99.6 / 107, 4096^3 776 / 819): with one wavefront per SIMD nothing covers its
// waits.  Two or three k-tiles on their way instead of one, and another first k-tile per workgroup for tall operands:
// no difference.
#include "mdh_matmul_split.h"

namespace mdh {
namespace {

using namespace split;

// One operand's k-tile on its way from device memory to LDS.  ROWS rows, NT threads; KC: stored with k contiguous
// ([row][k], row pitch ld), else with the rows contiguous ([k][row], pitch ld).
template <int ROWS, int BK, int NT, bool KC>
struct Operand {
  static constexpr int KP = BK / 8, SWZ = 64 / BK;
  static_assert(ROWS % 64 == 0 && ROWS * KP % NT == 0, "whole wavefronts per group of eight k");
  static constexpr int CH = ROWS * KP / NT;      // chunks of eight k per thread
  static constexpr int PLANE = ROWS * 16;       // bytes of one k / 8
  static constexpr int SLICE = KP * PLANE;
  static constexpr int BYTES = 3 * SLICE;

  float x[CH][8];
  float top[CH];     // largest magnitude of the chunk's row among what this thread has split
  unsigned off[CH];  // byte offset of the thread's chunk from the tile's first element

  // rows beyond the operand's edge repeat its last row: they only reach outputs that are not stored
  __device__ __forceinline__ void init(int64_t ld, int r0, int rmax) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int f = threadIdx.x + c * NT;
      top[c] = 0.f;
      if (KC)
        off[c] = (unsigned)(min(f / KP, rmax - 1 - r0) * ld + f % KP * 8) * 4u;
      else
        off[c] = (unsigned)min(f % ROWS, rmax - 1 - r0) * 4u;
    }
  }
  // P: the operand's element (r0, 0); requests chunk c of the tile whose first k is k0.  Buffer loads: base and
  // row pitch in scalar registers, so that a load takes no vector instruction for its address.
  __device__ __forceinline__ void load(const float* __restrict__ P, int64_t ld, int k0, int c) {
    if (KC) {
      const auto r = rsrc(P + k0);
      const f4 a = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off[c], 0, 0));
      const f4 b = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off[c] + 16, 0, 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) x[c][e] = a[e], x[c][e + 4] = b[e];
    } else {
      const int kc = __builtin_amdgcn_readfirstlane((threadIdx.x + c * NT) / ROWS);
      const auto r = rsrc(P + (k0 + kc * 8) * ld);
      const unsigned pitch = (unsigned)ld * 4u;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        x[c][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off[c], e * pitch, 0));
    }
  }
  // the tile starts `skip` elements of k early: those belong to the tile before it
  __device__ __forceinline__ void mask(int skip, int c) {
    const int f = threadIdx.x + c * NT, k = (KC ? f % KP : f / ROWS) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[c][e] = k + e < skip ? 0.f : x[c][e];
  }
  // the first half of the work on chunk c is its high slice, the second the other two: 24 vector instructions each
  __device__ __forceinline__ void store(char* st, const Split<>& split, int c, bool second) {
    const int f = threadIdx.x + c * NT;
    const int row = KC ? f / KP : f % ROWS, kc = KC ? f % KP : f / ROWS;
    char* p = st + kc * PLANE + (row ^ (SWZ * kc)) * 16;
    if (!second) {
      *(u4*)p = split.template slice<H>(x[c], top[c]);
    } else {
      *(u4*)(p + Mid * SLICE) = split.template slice<Mid>(x[c], top[c]);
      *(u4*)(p + L * SLICE) = split.template slice<L>(x[c], top[c]);
    }
  }
  __device__ __forceinline__ float largest() const {
    float t = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) t = fmaxf(t, finite(top[c]));
    return t;
  }
  // rows: LDS, the largest magnitude of every row (bits of a float), 0 before
  __device__ __forceinline__ void merge(unsigned* rows) const {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int f = threadIdx.x + c * NT;
      atomicMax(rows + (KC ? f / KP : f % ROWS), __float_as_uint(top[c]));
    }
  }
};

// C[i][j] = sum_k Y[i,k] X[j,k]; the accumulator lane holds four consecutive j of one i.
//
// One k-tile is six phases, one per product, of MI * NI MFMAs on different accumulators.  LDS holds two k-tiles:
// while tile t is multiplied, tile t+1 is split and written, tile t+2 is on its way from memory.  All operands of
// tile t are in registers, and all of tile t+1 in LDS, when phase 4 begins: the one barrier of the iteration
// stands there, so that phases 4 and 5 cover the latency of the first LDS reads of tile t+1.
// Order of the products: the smaller ones first (m m', then those with a middle, those with a low slice, h h'), so that
// the slices of a value come together without rounding: a sum of one term is one multiplication, and a product with a
// permutation is exact (h h' second: 0.02 % of the outputs off by an ulp).  XH, XL: the slice of which operand is read
// first -- no difference but for the compiler's schedule (us: 256 x 256 at 4096^3 593 with both of X first, 605 with
// both of Y; 128 x 128 at 1500^3 64 with h of X and l of Y, 66 and 67 otherwise; the other tiles equal within 1 %).
template <int BM, int BN, int BK, int WM, int WN, bool YK, bool XK>
__device__ __forceinline__ void split_tile(const float* __restrict__ Y, const float* __restrict__ X, float* __restrict__ Cout,
                                           int M, int N, int64_t ldy, int64_t ldx, int m0, int n0, int kbeg, int kend, char* lds) {
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  using OY = Operand<BM, BK, NT, YK>;
  using OX = Operand<BN, BK, NT, XK>;
  constexpr int STAGE = OY::BYTES + OX::BYTES, MI = WM / 32, NI = WN / 32;
  constexpr int CH = OY::CH + OX::CH;
  constexpr bool XH = BM == BN && BM > 64, XL = BM != 128 || BN != 128;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave / (BN / WN)) * WM, wn = (wave % (BN / WN)) * WN;
  const int l32 = lane & 31, lh = lane >> 5;
  unsigned* const largest = (unsigned*)(lds + 2 * STAGE);  // magnitude of the values the workgroup has split

  f16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  OY oy;
  OX ox;
  const Split<> split;
  oy.init(ldy, m0, M);
  ox.init(ldx, n0, N);
  if (threadIdx.x == 0) *largest = 0;
  // an MFMA takes 16 k of a k-tile: k / 8 = 2 h + lh
  constexpr int KH = BK / 16;
  int yoff[KH], xoff[KH];
#pragma unroll
  for (int h = 0; h < KH; ++h) {
    const int kc = 2 * h + lh, swz = (l32 ^ (OY::SWZ * kc)) * 16;
    yoff[h] = kc * OY::PLANE + wm * 16 + swz;
    xoff[h] = OY::BYTES + kc * OX::PLANE + wn * 16 + swz;
  }
  const float* const Yt = Y + (YK ? m0 * ldy : m0);
  const float* const Xt = X + (XK ? n0 * ldx : n0);

  // the last tile ends at kend: where the part is no whole number of tiles it starts inside the tile before it,
  // and the elements that tile has already taken are zeroed on the Y side
  const int nk = (kend - kbeg + BK - 1) / BK;
  const int skip = kbeg + nk * BK - kend;
  auto load = [&](int t, int c) {  // beyond the last tile: the last one again, unused
    const int k0 = min(kbeg + min(t, nk - 1) * BK, kend - BK);
    if (c < OY::CH)
      oy.load(Yt, ldy, k0, c);
    else
      ox.load(Xt, ldx, k0, c - OY::CH);
  };
  auto store = [&](char* st, int c, bool second) {
    if (c < OY::CH)
      oy.store(st, split, c, second);
    else
      ox.store(st + OY::BYTES, split, c - OY::CH, second);
  };
  auto mask_last = [&](int t) {
    if (t == nk - 1 && skip) {
#pragma unroll
      for (int c = 0; c < OY::CH; ++c) oy.mask(skip, c);
    }
  };

  u4 y[3][MI][KH], x[3][NI][KH];
  auto read_y = [&](const char* st, int s) {
#pragma unroll
    for (int h = 0; h < KH; ++h)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) y[s][mi][h] = *(const u4*)(st + yoff[h] + s * OY::SLICE + mi * 512);
  };
  auto read_x = [&](const char* st, int s) {
#pragma unroll
    for (int h = 0; h < KH; ++h)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) x[s][ni][h] = *(const u4*)(st + xoff[h] + s * OX::SLICE + ni * 512);
  };
  auto mma = [&](int sy, int sx) {
#pragma unroll
    for (int h = 0; h < KH; ++h)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = mfma(x[sx][ni][h], y[sy][mi][h], acc[mi][ni]);
  };
  // one phase: MFMAs with the LDS reads for the next phase, and a share of the next tile's split, between them
  auto phase = [&](int p, int sy, int sx, bool more, int t) {
    mma(sy, sx);
    constexpr int NM = KH * MI * NI;
    if (more && p < 4) {
#pragma unroll
      for (int h = p * CH / 2; h < (p + 1) * CH / 2; ++h) {
        store(lds + ((t + 1) & 1) * STAGE, h / 2, h % 2);
        if (h % 2) load(t + 2, h / 2);
      }
      constexpr int V = (24 * ((CH + 1) / 2) + NM - 1) / NM;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // tile t is multiplied; more: tile t+1, in registers, is split and its registers requested again
  auto body = [&](int t, auto more_) {
    constexpr bool more = decltype(more_)::value;
    const char* cur = lds + (t & 1) * STAGE;
    if (more) mask_last(t + 1);
    if (XH) read_x(cur, H); else read_y(cur, H);
    phase(0, Mid, Mid, more, t);
    if (XH) read_y(cur, H); else read_x(cur, H);
    phase(1, XH ? Mid : H, XH ? H : Mid, more, t);
    if (XL) read_x(cur, L); else read_y(cur, L);
    phase(2, XH ? H : Mid, XH ? Mid : H, more, t);
    if (XL) read_y(cur, L); else read_x(cur, L);
    phase(3, XL ? H : L, XL ? L : H, more, t);
    if (more) {
      const char* nxt = lds + ((t + 1) & 1) * STAGE;
      __syncthreads();
      read_y(nxt, Mid);
      read_x(nxt, Mid);
    }
    phase(4, XL ? L : H, XL ? H : L, false, t);
    phase(5, H, H, false, t);
  };

#pragma unroll
  for (int c = 0; c < CH; ++c) load(0, c);
  mask_last(0);
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    store(lds, c, false);
    store(lds, c, true);
    load(1, c);
  }
  __syncthreads();
  read_y(lds, Mid);
  read_x(lds, Mid);
  int t = 0;
  for (; t + 1 < nk; ++t) body(t, Yes{});
  body(t, No{});

  const bool whole = m0 + BM <= M && n0 + BN <= N;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    const int row = m0 + wm + mi * 32 + l32;
    float* const p = Cout + (int64_t)row * N + n0 + wn + 4 * lh;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int j = ni * 32 + 8 * g;
        const f4 v = {acc[mi][ni][4 * g], acc[mi][ni][4 * g + 1], acc[mi][ni][4 * g + 2], acc[mi][ni][4 * g + 3]};
        if (whole) {
          *(f4u*)(p + j) = v;
        } else if (row < M) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n0 + wn + 4 * lh + j + r < N) p[j + r] = v[r];
        }
      }
    }
  }

  // Values the split does not carry (mdh_split.h): bit mi * NI + ni of `redo` is a block of this wavefront that holds an
  // output they may have entered.  The outputs are on their way by now: the search takes its time beside the stores, and
  // what is evaluated again is written over them.
  unsigned redo = 0;
  float least = __builtin_huge_valf();
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      float z = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        z = __builtin_fmaf(acc[mi][ni][r], 0.f, z);
        least = fminf(least, fabsf(acc[mi][ni][r]));
      }
      if (__any(!(z == 0.f))) redo |= 1u << (mi * NI + ni);
    }
  const float bound = (float)(kend - kbeg) * kTiny * workgroup_largest(fmaxf(oy.largest(), ox.largest()), largest);
  unsigned long long todo = 0;  // the workgroup's blocks, row by row
  if (__syncthreads_or(redo || least < bound)) {
    unsigned* const rows = (unsigned*)lds;  // the operands' stages are done with
    unsigned* const blocks = rows + BM + BN;
    const Marks ym(blocks + 2, BM), xm(blocks + 2 + Marks::words(BM), BN);
    static_assert((BM + BN + 2 + Marks::words(BM) + Marks::words(BN)) * 4 <= 2 * STAGE, "");
    wait_stores_done();  // (other wavefronts may write some of them again)
    for (int i = threadIdx.x; i < BM + BN + 2 + Marks::words(BM) + Marks::words(BN); i += NT) rows[i] = 0;
    __syncthreads();
    oy.merge(rows);
    ox.merge(rows + BM);
    __syncthreads();
    unsigned small = 0;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      const unsigned cols = nonzero_bits(rows + BM + wn + ni * 32 + 4 * lh);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        unsigned open = 0;  // the block's outputs of this lane
        if (rows[wm + mi * 32 + l32])
#pragma unroll
          for (int r = 0; r < 16; ++r) open |= (unsigned)(fabsf(acc[mi][ni][r]) < bound) << r;
        open &= cols;
        if (!__any(open)) continue;
        small |= 1u << (mi * NI + ni);
        if (open) ym.add(wm + mi * 32 + l32);
        for (; open; open &= open - 1) {
          const int r = __builtin_ctz(open);
          xm.add(wn + ni * 32 + 8 * (r / 4) + 4 * lh + r % 4);
        }
      }
    }
    if (__syncthreads_or(small)) {
      const bool found = holds_tiny<BM, NT, YK>(Y, ldy, m0, M, kbeg, kend, ym) || holds_tiny<BN, NT, XK>(X, ldx, n0, N, kbeg, kend, xm);
      if (__syncthreads_or(found)) redo |= small;
    }
    if (lane < MI * NI && redo >> lane & 1) {
      const int b = (wm / 32 + lane / NI) * (BN / 32) + wn / 32 + lane % NI;
      atomicOr(blocks + b / 32, 1u << b % 32);
    }
    __syncthreads();
    const unsigned lo = __builtin_amdgcn_readfirstlane(blocks[0]), hi = __builtin_amdgcn_readfirstlane(blocks[1]);
    todo = lo | (unsigned long long)hi << 32;
  }

  if (!todo) return;
  // Many blocks: every wavefront takes its own, 64 x 64 at a time, which halves what is loaded.  Few, a row or column
  // of the tile: they are dealt out, so that no wavefront has a whole part of the tile to itself.
  if constexpr (BM * BN / 1024 > 2 * NT / 64) {
    static_assert(MI % 2 == 0 && NI % 2 == 0, "");
    if (__popcll(todo) > 2 * NT / 64) {
      for (int mi = 0; mi < MI; mi += 2)
        for (int ni = 0; ni < NI; ni += 2)
          if (redo >> (mi * NI + ni) & (3u | 3u << NI))
            recompute_fp32<2, 2, 1, YK, XK>(Y, X, Cout, M, N, ldy, ldx, m0 + wm + mi * 32, n0 + wn + ni * 32, kbeg, kend);
      return;
    }
  }
  for (int i = 0; todo; ++i, todo &= todo - 1)
    if (i % (NT / 64) == __builtin_amdgcn_readfirstlane(wave)) {
      const int b = __builtin_ctzll(todo);
      recompute_fp32<1, 1, 4, YK, XK>(Y, X, Cout, M, N, ldy, ldx, m0 + b / (BN / 32) * 32, n0 + b % (BN / 32) * 32, kbeg, kend);
    }
}

// (second launch bound: the wavefronts of a SIMD that LDS has room for, so that the fp32 evaluation, whose registers
// would allow fewer, does not come into it: three workgroups of 64 x 64 tiles.  With A transposed and B plain those take 176
// registers if they may, which leaves two: 64 x 803 x 431 x 216 109 us, 100 with three and four registers spilled in the fp32
// evaluation; 16 x 400 x 700 x 260 30.1 / 28.0)
template <int BM, int BN, int BK, int WM, int WN, bool YK, bool XK>
__global__ __launch_bounds__(((BM / WM) * (BN / WN) * 64), (BM + BN > 128 ? 2 : 3)) void matmul_split_kernel(
    const float* __restrict__ Y, const float* __restrict__ X, float* __restrict__ C, float* __restrict__ ws, int M, int N,
    int K, int tiles_m, int tiles_n, int S, int kchunk, int nbatch, int jmajor) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  // XCD-aware order: workgroup ids are dealt round-robin to the 8 XCDs; each XCD gets a contiguous run (whole
  // batches when there are at least 8), walked in bands of 8 tile rows (jmajor: tile columns) so that the tiles
  // resident on one XCD at a time share few panels of the operands in that XCD's L2.
  int b = xcd_order(blockIdx.x, gridDim.x);
  const int tiles = tiles_m * tiles_n;
  const int batch = b / (tiles * S);
  b -= batch * tiles * S;
  const int s = b / tiles, t = b % tiles;
  constexpr int GM = 8;
  const int fast_n = jmajor ? tiles_n : tiles_m, slow_n = jmajor ? tiles_m : tiles_n;
  const int band = t / (GM * slow_n);
  const int band_w = min(GM, fast_n - band * GM);
  const int in_band = t - band * GM * slow_n;
  const int tf = band * GM + in_band % band_w, tsl = in_band / band_w;
  const int m0 = (jmajor ? tsl : tf) * BM, n0 = (jmajor ? tf : tsl) * BN;
  const int kbeg = s * kchunk, kend = min(K, kbeg + kchunk);
  const int64_t mn = (int64_t)M * N;
  Y += (int64_t)batch * M * K;
  X += (int64_t)batch * K * N;
  float* out = S > 1 ? ws + ((int64_t)s * nbatch + batch) * mn : C + batch * mn;
  const int64_t ldy = YK ? K : M, ldx = XK ? K : N;
  split_tile<BM, BN, BK, WM, WN, YK, XK>(Y, X, out, M, N, ldy, ldx, m0, n0, kbeg, kend, lds);
}

struct Call {
  int64_t batch, M, N, K;
  const float *Y, *X;
  float* C;
  void* ws;
  hipStream_t st;
  int S, jmajor;
};

template <int BM, int BN, int BK, int WM, int WN, bool YK, bool XK>
mdh_status launch_t(const Call& c) {
  constexpr int NT = (BM / WM) * (BN / WN) * 64;
  constexpr int LDS_BYTES = 2 * (BM + BN) * BK * 6 + 16;
  auto kern = matmul_split_kernel<BM, BN, BK, WM, WN, YK, XK>;
  static int64_t lds_allowed[kMaxDevices] = {};
  if (allow_dynamic_lds((const void*)kern, LDS_BYTES, lds_allowed) != MDH_OK) return MDH_ERR_LAUNCH;
  const int64_t tm = cdiv(c.M, BM), tn = cdiv(c.N, BN);
  const int64_t kchunk = cdiv(cdiv(c.K, c.S), BK) * BK;
  if ((c.S - 1) * kchunk >= c.K) return MDH_ERR_TILE_NOT_DIVIDING;  // a part without k
  const int64_t nblocks = tm * tn * c.S * c.batch;
  if (nblocks > 0x7fffffff) return MDH_ERR_SIZE;
  clear_stale_error();
  hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(NT), LDS_BYTES, c.st, c.Y, c.X, c.C, (float*)c.ws, (int)c.M,
                     (int)c.N, (int)c.K, (int)tm, (int)tn, c.S, (int)kchunk, (int)c.batch, c.jmajor);
  mdh_status r = launch_status();
  if (r != MDH_OK || c.S <= 1) return r;
  return launch_combine_sum((const float*)c.ws, c.C, c.batch * c.M * c.N, c.S, c.st);
}

template <int BM, int BN, int BK, int WM, int WN>
mdh_status launch_views(const Call& c, bool yk, bool xk) {
  if (yk) return xk ? launch_t<BM, BN, BK, WM, WN, true, true>(c) : launch_t<BM, BN, BK, WM, WN, true, false>(c);
  return xk ? launch_t<BM, BN, BK, WM, WN, false, true>(c) : launch_t<BM, BN, BK, WM, WN, false, false>(c);
}

}  // namespace

mdh_status launch_matmul_split(const GemmPlan& pl, bool ta, bool tb, bool tc, int64_t batch, int64_t M, int64_t N, int64_t K,
                               const float* A, const float* B, float* C, void* ws, hipStream_t st) {
  if (pl.WK > 1) return launch_matmul_split_k(pl, ta, tb, tc, batch, M, N, K, A, B, C, ws, st);
  // C stored transposed is the product of the transposed operands in the other order
  Call c = {batch, M, N, K, A, B, C, ws, st, pl.S, pl.jmajor};
  bool yk = !ta, xk = tb;
  GemmPlan g = pl;
  if (tc) {
    c = Call{batch, N, M, K, B, A, C, ws, st, pl.S, !pl.jmajor};
    yk = tb;
    xk = !ta;
    g.BM = pl.BN, g.BN = pl.BM, g.WM = pl.WN, g.WN = pl.WM;
  }
#define MDH_MS(bm, bn, bk, wm, wn) \
  if (g.BM == bm && g.BN == bn && g.BK == bk && g.WM == wm && g.WN == wn) return launch_views<bm, bn, bk, wm, wn>(c, yk, xk);
  MDH_MS(256, 256, 16, 64, 128)
  MDH_MS(256, 128, 32, 64, 64)
  MDH_MS(128, 128, 32, 32, 64)
  MDH_MS(128, 64, 32, 64, 32)
  MDH_MS(64, 64, 32, 32, 32)
#undef MDH_MS
  return MDH_ERR_UNSUPPORTED;
}

}  // namespace mdh
