// MatMul / bMatMul / MatMul^T on three-slice values (mdh_split.h) with k over the wavefronts of a workgroup, for outputs
// of about one tile per compute unit.
//
// De-composition, dims (b,i,j,k):
//   workgroup layer : batch x (M/BM) x (N/BN) x S
//   wavefront layer : W parts of k; every wavefront owns the whole tile of its workgroup
//   HBM layer       : chunks of 32 k
//   VGPR layer      : MI x NI x 2 blocks
//   block           : 32 x 32 x 16, six v_mfma_f32_32x32x16_bf16 (eight in tiles of one or two blocks)
// A wavefront loads, splits and multiplies its own k: nothing is shared before the end, where the W partial tiles are
// added up in LDS, so there is no barrier in the walk, and every value of the tile's panels is split once per workgroup,
// in the registers the matrix instructions read.  A k-contiguous operand is turned around in a private piece of LDS
// (rows of 128 bytes, 16-byte pieces swizzled by the row's last three bits: 65536 x 64 x 4096 counts 4.5e6 conflict cycles for
// its 2.3e6 LDS instructions, 4 % of the time); one with contiguous rows is
// loaded as it is multiplied, a lane holding MI or NI neighbouring rows, which the output's index undoes.
//
// What bounds it: instructions issued beside the matrix instructions.  With one in flight a SIMD issues something else
// every 4.6 clocks, so six fit under an MFMA of 32 clocks; the split takes 8 (MI + NI) / (MI NI) of them (2 x 2: 8.0, 2 x
// 3: 6.7, 3 x 3: 5.3).  The kernel that shares the split through LDS (mdh_matmul_split.hip) has fewer with its large tiles
// but needs M N for 256 of them, and on small ones a barrier and two trips through LDS per 32 k: 64 x 64 tiles take
// 0.57 us for that, 0.3 here: 1021 x 1531 x 777 26.0 -> 21.4 us, 1024^3 22.7 -> 17.4, 1500^3 62 -> 45.  Loads are not what
// bounds it (hits in the first level cost the same).
// Measured without gain: the split of the next 16 k between the matrix instructions of these (by the compiler's
// scheduling groups); loads a chunk earlier; 16-byte loads of row-contiguous operands, exchanged between lanes -- with six
// blocks all within the 256 registers that the launch bound leaves them, though LDS (102 KB of partial tiles) holds one
// workgroup of four wavefronts a compute unit, one a SIMD, which could have 512.  Nine blocks have them, and with A transposed
// and B plain still move 30 registers to accumulation registers and back.
#include "mdh_matmul_split.h"

namespace mdh {
namespace {

using namespace split;

// One operand of a wavefront: 32 * BLK rows, 32 k at a time.  KC: stored with k contiguous.
template <int BLK, bool KC>
struct WaveOperand {
  static constexpr int LDS = KC ? 32 * BLK * 128 : 0;  // a chunk, [row][32 k]
  static constexpr int NW = 16 * BLK;
  const float* P;   // first of the operand's rows of the tile
  int64_t left;     // elements from there to the operand's end
  int64_t ld;
  unsigned pitch, off;  // in bytes; off: of this lane
  unsigned w[NW];       // the chunk on its way
  float top[BLK];       // largest magnitude of the lane's rows among what it has split

  // row of block b that lane l (0 to 31) multiplies
  static __device__ __forceinline__ constexpr int row(int b, int l) { return KC ? b * 32 + l : l * BLK + b; }

  __device__ __forceinline__ void init(const float* base, int64_t n, int64_t pitch_elements, int r0) {
    const int lane = threadIdx.x & 63;
    ld = pitch_elements;
    const int64_t o = KC ? r0 * ld : r0;
    P = base + o;
    left = n - o;
    pitch = (unsigned)ld * 4u;
    off = KC ? (lane / 8) * pitch + (lane % 8) * 16 : (lane >> 5) * 8 * pitch + (lane & 31) * BLK * 4;
#pragma unroll
    for (int b = 0; b < BLK; ++b) top[b] = 0.f;
  }
  // KC: requests the 32 k from k0 on; what lies beyond the operand's end reads as 0, what lies beyond a row's end is not
  // used
  __device__ __forceinline__ void load_chunk(int k0) {
    const int64_t bytes = (left - k0) * 4;
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(P + k0), 0, (int)(unsigned)min(bytes, (int64_t)0xffffffff), 0x00027000);
#pragma unroll
    for (int j = 0; j < 4 * BLK; ++j) {
      const u4 v = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(r, off, j * 8 * pitch, 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * j + e] = v[e];
    }
  }
  // rows contiguous: requests the 16 k from k0 on as half h of the chunk
  __device__ __forceinline__ void load_half(int k0, int h) {
    const auto r = rsrc(P + k0 * ld);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      unsigned* const d = w + (h * 8 + e) * BLK;
      if constexpr (BLK == 1) {
        d[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, e * pitch, 0);
      } else if constexpr (BLK == 2) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, e * pitch, 0);
        d[0] = v[0], d[1] = v[1];
      } else {
        const auto v = __builtin_amdgcn_raw_buffer_load_b96(r, off, e * pitch, 0);
        d[0] = v[0], d[1] = v[1], d[2] = v[2];
      }
    }
  }
  // the first `skip` k of the chunk that has arrived (less than 16) as 0
  __device__ __forceinline__ void mask(int skip) {
    const int lane = threadIdx.x & 63, k = KC ? lane % 8 * 4 : lane / 32 * 8;
#pragma unroll
    for (int i = 0; i < (KC ? NW : NW / 2); ++i) w[i] = k + (KC ? i % 4 : i / BLK) < skip ? 0u : w[i];
  }
  // KC: the chunk that has arrived, to LDS
  __device__ __forceinline__ void put(char* lds) const {
    const int lane = threadIdx.x & 63, at = (lane / 8) * 128 + ((lane % 8) ^ (lane / 8)) * 16;
#pragma unroll
    for (int j = 0; j < 4 * BLK; ++j) *(u4*)(lds + at + j * 1024) = u4{w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]};
  }
  // eight k of the lane's row of block b, of half h of the chunk
  __device__ __forceinline__ void get(const char* lds, int h, int b, float (&x)[8]) const {
    if constexpr (KC) {
      const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f4 v = *(const f4*)(lds + row(b, l32) * 128 + ((h * 4 + lh * 2 + q) ^ (l32 & 7)) * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[q * 4 + e] = v[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(w[(h * 8 + e) * BLK + b]);
    }
  }
  __device__ __forceinline__ float largest() const {
    float t = 0.f;
#pragma unroll
    for (int b = 0; b < BLK; ++b) t = fmaxf(t, finite(top[b]));
    return t;
  }
  // rows: LDS, the largest magnitude of every row (bits of a float), 0 before
  __device__ __forceinline__ void merge(unsigned* rows) const {
#pragma unroll
    for (int b = 0; b < BLK; ++b) atomicMax(rows + row(b, threadIdx.x & 31), __float_as_uint(top[b]));
  }
};

template <int MI, int NI, int W, bool YK, bool XK>
struct Lds {
  static constexpr int OPERANDS = W * (WaveOperand<MI, YK>::LDS + WaveOperand<NI, XK>::LDS);
  static constexpr int PITCH = 32 * NI + 4;  // floats between rows of a partial tile
  static constexpr int PARTS = W * 32 * MI * PITCH * 4;
  static constexpr int TOP = OPERANDS > PARTS ? OPERANDS : PARTS;  // a word: largest magnitude the workgroup has split
  static constexpr int BYTES = TOP + 16;
};

// Tiles of one or two blocks stand in for kernels on fp32 instructions, whose sums of few terms are rounded once per term.
// They have registers to spare for a sum of their own for h h', which is exact in 16 bits and rounds once per 16 k where
// products in one accumulator round up to six times, and take eight of the nine products (mdh_split.h; all but l l', below
// 2^-34): with six a single product is off by up to 1.7 x 2^-24 instead of 1.0, and 4 % of them are not the correctly
// rounded ones.  Error against 64 bits, 256 x 256 x 512, n terms of a sum not zero, relative 2-norm in units of 2^-24, fp32
// instructions in LDS tiles / with k over eight wavefronts / these / with six products: n = 1 0.42 / 0.42 / 0.42 / 0.44, 2
// 0.52 / 0.61 / 0.60 / 0.61, 4 0.67 / 0.76 / 0.74 / 0.75, 8 0.90 / 0.92 / 0.88 / 0.88, 32 1.7 / 1.2 / 1.0 / 1.0, dense 6.8 /
// 2.6 / 1.3 / 1.3.  (A pair of sums a wavefront up to the end, h h' and the rest, has 0.43, 0.44, 0.48 for 2, 4, 8 terms but
// takes 6 % more of a call of 5 us.)  The two products more cost 2.4 % over 45 products of 4.6 to 34 us: a step of one block
// 0.128 -> 0.140 us for 32 k, 4 x 203 x 171 x 183 5.2 / 5.2, 288 x 320 x 2880 16.2 / 17.9, 340 x 2912 x 1786 34 / 38.
template <int MI, int NI, int W, bool YK, bool XK>
__global__ __launch_bounds__(W * 64, (MI * NI > 6 ? 1 : 2)) void matmul_split_k_kernel(
    const float* __restrict__ Y, const float* __restrict__ X, float* __restrict__ C, float* __restrict__ ws, int M, int N, int K,
    int tiles_m, int tiles_n, int S, int kchunk, int nbatch, int jmajor) {
  constexpr int BM = 32 * MI, BN = 32 * NI, NT = W * 64;
  constexpr bool OWN = MI * NI <= 2;
  using OY = WaveOperand<MI, YK>;
  using OX = WaveOperand<NI, XK>;
  using LD = Lds<MI, NI, W, YK, XK>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  // XCD-aware order, as in mdh_matmul_split.hip
  int b = xcd_order(blockIdx.x, gridDim.x);
  const int tiles = tiles_m * tiles_n;
  const int batch = b / (tiles * S);
  b -= batch * tiles * S;
  const int sp = b / tiles, t = b % tiles;
  constexpr int GM = 8;
  const int fast_n = jmajor ? tiles_n : tiles_m, slow_n = jmajor ? tiles_m : tiles_n;
  const int band = t / (GM * slow_n);
  const int band_w = min(GM, fast_n - band * GM);
  const int in_band = t - band * GM * slow_n;
  const int tf = band * GM + in_band % band_w, tsl = in_band / band_w;
  const int tm = jmajor ? tsl : tf, tn = jmajor ? tf : tsl;
  // a tile that would stick out is moved inside; the rows and columns it shares with the one before are not stored
  const int m0 = min(tm * BM, M - BM), n0 = min(tn * BN, N - BN);
  const int mskip = tm * BM - m0, nskip = tn * BN - n0;
  const int kbeg = sp * kchunk, kend = min(K, kbeg + kchunk);
  const int64_t mn = (int64_t)M * N, ldy = YK ? K : M, ldx = XK ? K : N;
  Y += (int64_t)batch * M * K;
  X += (int64_t)batch * K * N;
  float* const out = S > 1 ? ws + ((int64_t)sp * nbatch + batch) * mn : C + batch * mn;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  char* const own = lds + wave * (OY::LDS + OX::LDS);
  unsigned* const word = (unsigned*)(lds + LD::TOP);
  if (threadIdx.x == 0) *word = 0;

  // This wavefront's part of k, in steps of 16.  The last one ends with the part of the workgroup: where that is no whole
  // number of steps it starts inside the wavefront before, and the elements that are not its own read as 0.
  const int steps = (kend - kbeg + 15) / 16;
  const int first = steps * wave / W, n = steps * (wave + 1) / W - first;
  const int skip = wave == W - 1 ? steps * 16 - (kend - kbeg) : 0;
  const int kb = kbeg + first * 16 - skip, ke = kb + n * 16;

  f16 acc[MI][NI], sum[OWN ? MI : 1][OWN ? NI : 1];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[i][j][r] = 0.f;
        if (OWN) sum[i][j][r] = 0.f;
      }
  OY oy;
  OX ox;
  // (six blocks on one wavefront a SIMD: 1024^3 in 64 x 96 tiles 21.5 us with v_dot2c, 24.1 without; the others: 96 x 96
  // at 1500^3 45.7 / 44.8, 64 x 64 at 2048^3 105 / 100)
  const Split<MI * NI == 6> split;
  oy.init(Y, (int64_t)M * K, ldy, m0);
  ox.init(X, (int64_t)N * K, ldx, n0);

  auto load = [&](int k0) {  // (beyond the part's last step: that one again, unused)
    if constexpr (YK)
      oy.load_chunk(k0);
    else
      oy.load_half(k0, 0), oy.load_half(min(k0 + 16, ke - 16), 1);
    if constexpr (XK)
      ox.load_chunk(k0);
    else
      ox.load_half(k0, 0), ox.load_half(min(k0 + 16, ke - 16), 1);
  };
  auto step = [&](int h) {
    u4 y[MI][3], x[NI][3];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      float v[8];
      oy.get(own, h, i, v);
      split(v, y[i], oy.top[i]);
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      float v[8];
      ox.get(own + OY::LDS, h, j, v);
      split(v, x[j], ox.top[j]);
    }
    auto mma = [&](int sy, int sx) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = mfma(x[j][sx], y[i][sy], acc[i][j]);
    };
    if constexpr (OWN) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) sum[i][j] = mfma(x[j][H], y[i][H], sum[i][j]);
      mma(Mid, L);
      mma(L, Mid);
    }
    // the smaller products first, as in mdh_matmul_split.hip
    mma(Mid, Mid);
    mma(Mid, H);
    mma(H, Mid);
    mma(H, L);
    mma(L, H);
    if constexpr (!OWN) mma(H, H);
  };
  if (n > 0) {
    load(kb);
    if (skip) {
      oy.mask(skip);
      ox.mask(skip);
    }
    for (int k0 = kb; k0 < ke; k0 += 32) {
      const int next = k0 + 32 < ke ? k0 + 32 : kb;
      if constexpr (YK) {
        oy.put(own);
        oy.load_chunk(next);
      }
      if constexpr (XK) {
        ox.put(own + OY::LDS);
        ox.load_chunk(next);
      }
      step(0);
      if (k0 + 16 < ke) step(1);
      if constexpr (!YK) oy.load_half(next, 0), oy.load_half(min(next + 16, ke - 16), 1);
      if constexpr (!XK) ox.load_half(next, 0), ox.load_half(min(next + 16, ke - 16), 1);
    }
  }
  if constexpr (OWN) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] += sum[i][j];
  }

  // the partial tiles, [wavefront][row][column], and their sum
  __syncthreads();
  float* const parts = (float*)lds;
  {
    float* const p = parts + wave * BM * LD::PITCH;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float* const q = p + OY::row(i, l32) * LD::PITCH;
        if constexpr (XK) {
#pragma unroll
          for (int j = 0; j < NI; ++j)
            *(f4*)(q + j * 32 + 8 * g + 4 * lh) = f4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        } else {
          float v[4 * NI];
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < NI; ++j) v[r * NI + j] = acc[i][j][4 * g + r];
#pragma unroll
          for (int j = 0; j < NI; ++j) *(f4*)(q + (8 * g + 4 * lh) * NI + 4 * j) = f4{v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]};
        }
      }
  }
  const float bound = (float)(kend - kbeg) * kTiny * workgroup_largest(fmaxf(oy.largest(), ox.largest()), word);
  constexpr int QUADS = BM * BN / 4, NQ = (QUADS + NT - 1) / NT;
  f4 c[NQ];
  bool odd = false;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int u = threadIdx.x + i * NT;
    if (QUADS % NT && u >= QUADS) break;
    const float* const p = parts + u / (BN / 4) * LD::PITCH + u % (BN / 4) * 4;
    c[i] = *(const f4*)p;
#pragma unroll
    for (int w = 1; w < W; ++w) c[i] += *(const f4*)(p + w * BM * LD::PITCH);
#pragma unroll
    for (int e = 0; e < 4; ++e) odd |= !(fabsf(c[i][e]) < __builtin_huge_valf()) || fabsf(c[i][e]) < bound;
  }

#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int u = threadIdx.x + i * NT, row = u / (BN / 4), col = u % (BN / 4) * 4;
    if (QUADS % NT && u >= QUADS) break;
    if (row < mskip) continue;
    float* const p = out + (int64_t)(m0 + row) * N + n0 + col;
    if (col >= nskip) {
      *(f4u*)p = c[i];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (col + e >= nskip) p[e] = c[i][e];
    }
  }

  // Values the split does not carry (mdh_split.h): bit of a 32 x 32 block of the tile that holds an output they may have
  // entered.  The outputs are on their way by now: the search takes its time beside the stores, and what is evaluated
  // again is written over them.
  unsigned todo = 0;
  if (__syncthreads_or(odd)) {
    unsigned* const rows = (unsigned*)lds;  // the partial tiles are done with
    unsigned* const blocks = rows + BM + BN;
    const Marks ym(blocks + 2, BM), xm(blocks + 2 + Marks::words(BM), BN);
    constexpr int WORDS = BM + BN + 2 + Marks::words(BM) + Marks::words(BN);
    static_assert(WORDS * 4 <= LD::TOP, "");
    wait_stores_done();  // (other wavefronts may write some of them again)
    for (int i = threadIdx.x; i < WORDS; i += NT) rows[i] = 0;
    __syncthreads();
    oy.merge(rows);
    ox.merge(rows + BM);
    __syncthreads();
    bool small = false;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int u = threadIdx.x + i * NT, row = u / (BN / 4), col = u % (BN / 4) * 4;
      if ((QUADS % NT && u >= QUADS) || row < mskip) continue;
      const unsigned bit = 1u << (row / 32 * NI + col / 32);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (col + e < nskip) continue;
        if (!(fabsf(c[i][e]) < __builtin_huge_valf())) atomicOr(blocks, bit);
        if (fabsf(c[i][e]) < bound && rows[row] && rows[BM + col + e]) {
          small = true;
          atomicOr(blocks + 1, bit);
          ym.add(row);
          xm.add(col + e);
        }
      }
    }
    if (__syncthreads_or(small)) {
      const bool found = holds_tiny<BM, NT, YK>(Y, ldy, m0, M, kbeg, kend, ym) || holds_tiny<BN, NT, XK>(X, ldx, n0, N, kbeg, kend, xm);
      if (__syncthreads_or(found)) todo = blocks[1];
    }
    todo = __builtin_amdgcn_readfirstlane(todo | blocks[0]);
  }
  for (int i = 0; todo; ++i, todo &= todo - 1)
    if (i % W == wave) {
      const int k = __builtin_ctz(todo);
      recompute_fp32<1, 1, 2, YK, XK>(Y, X, out, M, N, ldy, ldx, m0 + k / NI * 32, n0 + k % NI * 32, kbeg, kend, m0 + mskip, n0 + nskip);
    }
}

struct Call {
  int64_t batch, M, N, K;
  const float *Y, *X;
  float* C;
  void* ws;
  hipStream_t st;
  int S, jmajor;
};

template <int MI, int NI, int W, bool YK, bool XK>
mdh_status launch_t(const Call& c) {
  constexpr int BM = 32 * MI, BN = 32 * NI, LDS_BYTES = Lds<MI, NI, W, YK, XK>::BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "");
  if (c.M < BM || c.N < BN || c.K < 32) return MDH_ERR_UNSUPPORTED;
  auto kern = matmul_split_k_kernel<MI, NI, W, YK, XK>;
  static int64_t lds_allowed[kMaxDevices] = {};
  if (allow_dynamic_lds((const void*)kern, LDS_BYTES, lds_allowed) != MDH_OK) return MDH_ERR_LAUNCH;
  const int64_t tm = cdiv(c.M, BM), tn = cdiv(c.N, BN);
  const int64_t kchunk = cdiv(cdiv(c.K, c.S), 32) * 32;
  if ((c.S - 1) * kchunk >= c.K) return MDH_ERR_TILE_NOT_DIVIDING;  // a part without k
  if (c.K - (c.S - 1) * kchunk < 32 && c.S > 1) return MDH_ERR_TILE_NOT_DIVIDING;
  const int64_t nblocks = tm * tn * c.S * c.batch;
  if (nblocks > 0x7fffffff) return MDH_ERR_SIZE;
  clear_stale_error();
  hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(W * 64), LDS_BYTES, c.st, c.Y, c.X, c.C, (float*)c.ws, (int)c.M,
                     (int)c.N, (int)c.K, (int)tm, (int)tn, c.S, (int)kchunk, (int)c.batch, c.jmajor);
  mdh_status r = launch_status();
  if (r != MDH_OK || c.S <= 1) return r;
  return launch_combine_sum((const float*)c.ws, c.C, c.batch * c.M * c.N, c.S, c.st);
}

template <int MI, int NI, int W>
mdh_status launch_views(const Call& c, bool yk, bool xk) {
  if (yk) return xk ? launch_t<MI, NI, W, true, true>(c) : launch_t<MI, NI, W, true, false>(c);
  return xk ? launch_t<MI, NI, W, false, true>(c) : launch_t<MI, NI, W, false, false>(c);
}

}  // namespace

mdh_status launch_matmul_split_k(const GemmPlan& pl, bool ta, bool tb, bool tc, int64_t batch, int64_t M, int64_t N, int64_t K,
                                 const float* A, const float* B, float* C, void* ws, hipStream_t st) {
  // C stored transposed is the product of the transposed operands in the other order
  Call c = {batch, M, N, K, A, B, C, ws, st, pl.S, pl.jmajor};
  bool yk = !ta, xk = tb;
  int mi = pl.BM / 32, ni = pl.BN / 32;
  if (tc) {
    c = Call{batch, N, M, K, B, A, C, ws, st, pl.S, !pl.jmajor};
    yk = tb;
    xk = !ta;
    mi = pl.BN / 32, ni = pl.BM / 32;
  }
#define MDH_SK(i, j, w) \
  if (mi == i && ni == j && pl.WK == w) return launch_views<i, j, w>(c, yk, xk);
  MDH_SK(2, 2, 8)
  MDH_SK(2, 2, 4)
  MDH_SK(2, 3, 4)
  MDH_SK(3, 2, 4)
  MDH_SK(3, 3, 4)
  MDH_SK(1, 2, 8)
  MDH_SK(2, 1, 8)
  MDH_SK(1, 1, 8)
#undef MDH_SK
  return MDH_ERR_UNSUPPORTED;
}

}  // namespace mdh
