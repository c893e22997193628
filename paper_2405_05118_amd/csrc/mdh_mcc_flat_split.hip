// Multi-channel convolution for few input channels (mdh_mcc_flat.hip) on the bf16 matrix instructions, every fp32 value
// carried as three bf16 values (mdh_split.h).
//
// As there, the dimensions s and c of a filter row r are one dimension sc of S*C consecutive values, in the input and in
// the filter.  An operand of v_mfma_f32_32x32x16_bf16 holds eight consecutive k of a row per lane, so sc is walked in
// chunks of eight, ceil(S*C/8) of them a filter row, filled up with zeros in the filter: a 7 x 7 filter on three channels
// takes 11 steps of two chunks (88 instructions of 32 cycles) where the fp32 instructions take 77 of 64.
//
// Precision.  Sums of a filter with many zeros have few terms, and few roundings on the fp32 instructions: one per term
// that is not zero.  Six products a step in one accumulator round six times a step, whatever the terms are.  So the sums
// of h h', which is exact in 16 bits, are kept apart -- a step rounds them at most once, and not if its terms are zeros --
// and the seven other products, below 2^-8 of those, go to sums of their own, which are added at the end (l l', below 2^-34,
// is left out): no more roundings than terms.  Error against 64 bits, relative 2-norm in units of 2^-24, 7 x 7 x 3, n taps of
// 147 not zero, fp32 instructions / these / six products in one accumulator: n = 1 0.42 / 0.42 / 0.60 (largest 1.0 / 1.0 /
// 2.5), 2 0.53 / 0.43 / 0.83, 8 0.90 / 0.48 / 1.65, 24 1.5 / 0.64 / 2.5, 64 2.4 / 0.89 / 3.0.
//
// De-composition, dims (n,p,q,k,c,r,s): a wavefront owns a block of 32 pixels (32/QB rows x QB columns) and NI x 32
// channels at a time; a workgroup of eight wavefronts keeps the filter slice of its NI x 32 channels in LDS, split once,
// and walks its share of the blocks of all images, its wavefronts taking them in turn.  There is no barrier after the
// staging of the filter.  The input goes from memory to registers, two steps ahead -- 32 bytes at any 4-byte boundary, the
// overlap between taps and pixels comes from L1 -- and is split there: 40 vector instructions a step beside 8 NI matrix
// instructions of 32 cycles.  Splitting it once into LDS would need eight consecutive 16-bit values from any 2-byte
// boundary.
// us per call, the kernel on fp32 instructions / this one: 16 x 230 x 230 x 3 -> 64, 7 x 7, stride 2: 45.7 / 41.5 (36 with
// six products); 14 x 178 x 203 x 2 -> 56, 7 x 7: 94 / 60 (51).  Tried with six products: the patch split once into LDS, each
// wavefront its own, one workgroup a compute unit instead of two, 33.9 (then 33.0), the next block's loads ahead of this
// block's stores 35.3; with eight: the split at the start of its own step instead of in the shadow of the one before 43.
#include <type_traits>

#include "mdh_split.h"

namespace mdh {
namespace {

using namespace split;

constexpr int kNT = 512, kWaves = kNT / 64;

struct FlatConv {
  const float *in, *filt;
  float* out;
  int H, W, C, K, R, S, sh, sw, P, Q;
  int qb;         // log2 of the columns of a block
  int tp_n, tq_n; // blocks of an image
  int units;      // blocks of all images
  int G, tk_n;    // workgroups per filter slice, filter slices
  int CH, T;      // chunks of a filter row, steps of two chunks
  int64_t in_elems;
};

__device__ __forceinline__ f4 buf4(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// the largest of a wavefront's 64 values (not negative), in a scalar register; no address register for a shuffle
__device__ __forceinline__ float wave_max(float v) {
  auto other = [&](auto x) { return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), x.value << 10 | 0x1f)); };
  v = fmaxf(v, other(std::integral_constant<int, 1>()));
  v = fmaxf(v, other(std::integral_constant<int, 2>()));
  v = fmaxf(v, other(std::integral_constant<int, 4>()));
  v = fmaxf(v, other(std::integral_constant<int, 8>()));
  v = fmaxf(v, other(std::integral_constant<int, 16>()));
  return fmaxf(__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0)),
               __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32)));
}

// fp32 evaluation of a wavefront's block, for values the split does not carry
template <int NI>
__device__ __forceinline__ void recompute_fp32(const FlatConv& g, const float* __restrict__ x, int kw, int lh, int l32, f16 (&acc)[NI]) {
  const int SC = g.S * g.C, WC = g.W * g.C;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[ni][e] = 0.f;
  for (int r = 0; r < g.R; ++r)
#pragma unroll 4
    for (int s = 0; s < SC; s += 2) {
      const int j = s + lh, at = min(j, SC - 1);
      const float y = j < SC ? x[r * WC + at] : 0.f;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        const int k = kw + ni * 32 + l32;
        const float f = g.filt[((int64_t)min(k, g.K - 1) * g.R + r) * SC + at];
        acc[ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(j < SC && k < g.K ? f : 0.f, y, acc[ni], 0, 0, 0);
      }
    }
}

template <int NI>
__global__ __launch_bounds__(kNT, 4) void mcc_flat_split_kernel(FlatConv g) {
  constexpr int BN = NI * 32;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int chunks = 2 * g.T, slice = chunks * BN * 16;
  unsigned* const ftop = (unsigned*)(lds + 3 * slice);  // largest magnitude of every channel (bits of a float)
  unsigned* const ftiny = ftop + BN;
  const int SC = g.S * g.C, WC = g.W * g.C;
  const int tk = blockIdx.x % g.tk_n, w = blockIdx.x / g.tk_n, k0 = tk * BN;
  // (blocks of 32 channels have half the matrix instructions beside the split of their pixels: 3 x 150 x 100 x 3 -> 30, 7 x 7,
  // stride 2, 8.22 us with v_dot2c, 8.43 without; 64 channels, 8 x 200 x 180 x 4 -> 48, 5 x 5: 38.8 / 37.1)
  const Split<NI == 1> split;

  if (tid <= BN) ftop[tid] = 0;
  __syncthreads();
  // filter slice: entry (chunk, k), 16 bytes of each slice; the k of a chunk are rotated so that the writes of a wavefront,
  // consecutive chunks of one k, meet different banks
#pragma unroll 2
  for (int i = tid; i < chunks * BN; i += kNT) {
    const int k = i / chunks, ch = i - k * chunks, r = ch / g.CH, c = (ch - r * g.CH) * 8;
    const float* const f = g.filt + ((int64_t)min(k0 + k, g.K - 1) * g.R + min(r, g.R - 1)) * SC;
    float x[8];
    bool small = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = f[min(c + e, SC - 1)];
      x[e] = r < g.R && c + e < SC && k0 + k < g.K ? v : 0.f;
      small |= tiny(x[e]);
    }
    u4 v[3];
    float top = 0.f;
    split(x, v, top);
    if (top != 0.f) atomicMax(ftop + k, __float_as_uint(finite(top)));
    if (small) *ftiny = 1;
    char* const p = lds + (ch * BN + (k ^ (ch & 15))) * 16;
#pragma unroll
    for (int s = 0; s < 3; ++s) *(u4*)(p + s * slice) = v[s];
  }
  __syncthreads();
  const float fmost = wave_max(__uint_as_float(ftop[tid % BN]));

  // contiguous shares, and contiguous runs of them per XCD
  const int ws = xcd_order(w, g.G);
  const int u0 = (int)((int64_t)g.units * ws / g.G), u1 = (int)((int64_t)g.units * (ws + 1) / g.G);
  for (int u = u0 + wave; u < u1; u += kWaves) {
    // (the lane's numbers anew for every block: what follows from them would wait in registers through the steps, which have
    // none to spare -- 24 bytes a lane went to memory)
    int lane = tid & 63;
    asm volatile("" : "+v"(lane));
    const int l32 = lane & 31, lh = lane >> 5;
    const int tq = u % g.tq_n, band = u / g.tq_n, tp = band % g.tp_n, n = band / g.tp_n;
    const int p = (tp << (5 - g.qb)) + (l32 >> g.qb), q = (tq << g.qb) + (l32 & ((1 << g.qb) - 1));
    const int64_t first = (int64_t)n * g.H * WC;
    const float* const img = g.in + first;
    const int64_t room = (g.in_elems - first) * 4;  // loads behind the end of the input read as 0
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(img), 0, (int)(unsigned)min(room, (int64_t)0xfffffffc), 0x00027000);
    const int pix = min(p, g.P - 1) * g.sh * WC + min(q, g.Q - 1) * g.sw * g.C;

    f16 acc[NI], low[NI];  // sums of h h'; of the other products
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[ni][e] = low[ni][e] = 0.f;
    float top = 0.f;  // largest magnitude of the lane's share of the window

    // the two chunks of the step that `load` takes, one per half of the wavefront
    int c = 0, at = 0;
    auto load = [&](float (&x)[8]) {
      int at1 = at + 8, c1 = c + 1;
      if (c1 == g.CH) c1 = 0, at1 += WC - g.CH * 8;
      const int off = (pix + (lh ? at1 : at)) * 4;
      const f4 a = buf4(rs, off), b = buf4(rs, off + 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = a[e], x[e + 4] = b[e];
      c = c1 + 1, at = at1 + 8;
      if (c == g.CH) c = 0, at += WC - g.CH * 8;
    };
    auto step = [&](float (&next)[8], const u4 (&y)[3], u4 (&yn)[3], int t, float& top, bool more) {
      const int ch = 2 * t + lh;
      const char* const f = lds + (ch * BN + (l32 ^ (ch & 15))) * 16;
#pragma unroll
      for (int s = L; s >= H; --s) {
        u4 x[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) x[ni] = *(const u4*)(f + s * slice + ni * 512);
#pragma unroll
        for (int sy = L - (s == L); sy >= H + (s == H); --sy)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) low[ni] = mfma(x[ni], y[sy], low[ni]);
        if (s == H)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) acc[ni] = mfma(x[ni], y[H], acc[ni]);
      }
      split(next, yn, top);
      if (more) load(next);
      // (otherwise the next step's magnitudes are taken at the top of this one, and wait for loads just issued)
      __builtin_amdgcn_sched_barrier(0);
    };
    float r0[8], r1[8];
    u4 ya[3], yb[3];
    load(r0);
    load(r1);
    split(r0, ya, top);
    load(r0);
    int t = 0;
    for (; t + 2 < g.T; t += 2) {
      step(r1, ya, yb, t, top, true);
      step(r0, yb, ya, t + 1, top, true);
    }
    float next = top;  // (what the last step splits is not in the windows)
    step(r1, ya, yb, t, next, false);
    if (t + 1 < g.T) {
      top = next;
      step(r0, yb, ya, t + 1, next, false);
    }

#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[ni][e] += low[ni][e];

    // values the split does not carry (mdh_split.h)
    const int kw = k0;
    float z = 0.f, least = __builtin_huge_valf();
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        z = __builtin_fmaf(acc[ni][e], 0.f, z);
        least = fminf(least, fabsf(acc[ni][e]));
      }
    const float bound = (float)(g.R * SC) * kTiny * fmaxf(wave_max(finite(top)), fmost);
    bool fp32 = __any(!(z == 0.f));
    if (!fp32 && __any(least < bound)) {
      // an output too small, of a channel and a window that are not all zeros?
      const float window = fmaxf(top, __shfl_xor(top, 32));
      bool open = false;
      if (window != 0.f && p < g.P && q < g.Q)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            open |= fabsf(acc[ni][e]) < bound && ftop[ni * 32 + 8 * (e / 4) + 4 * lh + e % 4] != 0;
      if (__any(open)) {
        bool found = *ftiny != 0;
        for (int r = lh; r < g.R; r += 2)
          for (int s = 0; s < SC; ++s) found |= tiny(img[pix + r * WC + s]);
        fp32 = __any(found);
      }
    }
    if (fp32) recompute_fp32<NI>(g, img + pix, kw, lh, l32, acc);

    // output view: the lane's pixel, channels 8 (e/4) + 4 lh + e%4 of each 32
    if (p < g.P && q < g.Q) {
      float* const o = g.out + (((int64_t)n * g.P + p) * g.Q + q) * g.K + kw + 4 * lh;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int e = 0; e < 16; e += 4) {
          const int k = ni * 32 + 2 * e;
          if (kw + k + 4 * lh + 3 < g.K) {
            *(f4u*)(o + k) = f4{acc[ni][e], acc[ni][e + 1], acc[ni][e + 2], acc[ni][e + 3]};
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (kw + k + 4 * lh + i < g.K) o[k + i] = acc[ni][e + i];
          }
        }
    }
  }
}

template <int NI>
mdh_status launch_t(FlatConv g, int64_t N, hipStream_t st) {
  constexpr int BN = NI * 32;
  auto kern = mcc_flat_split_kernel<NI>;
  static int64_t lds_allowed[kMaxDevices] = {};
  const int64_t lds = mcc_flat_split_lds_bytes(BN, g.C, g.R, g.S);
  if (lds > 160 * 1024) return MDH_ERR_TILE_RESOURCES;
  if (allow_dynamic_lds((const void*)kern, lds, lds_allowed) != MDH_OK) return MDH_ERR_LAUNCH;
  const int64_t units = N * g.tp_n * g.tq_n;
  if (units > 0x7fffffff - 8 * kWaves) return MDH_ERR_SIZE;
  g.units = (int)units;
  g.tk_n = (int)cdiv(g.K, BN);
  // what the compute units hold at once, shared between the filter slices; no more than there are blocks for
  const int64_t held = 256 * (lds <= 80 * 1024 ? 2 : 1);
  int64_t G = held / g.tk_n;
  if (G > cdiv(units, 4)) G = cdiv(units, 4);
  g.G = (int)(G < 1 ? 1 : G);
  clear_stale_error();
  hipLaunchKernelGGL(kern, dim3((unsigned)(g.G * g.tk_n)), dim3(kNT), (size_t)lds, st, g);
  return launch_status();
}

}  // namespace

// three slices of the filter, its steps filled up to two chunks; the channels' largest magnitudes
int64_t mcc_flat_split_lds_bytes(int BN, int64_t C, int64_t R, int64_t S) {
  return 3 * cdiv(R * cdiv(S * C, 8), 2) * 2 * BN * 16 + 4ll * BN + 16;
}

mdh_status launch_mcc_flat_split(const MccPlan& pl, int64_t N, int64_t H, int64_t W, int64_t C, int64_t K, int64_t R, int64_t S,
                                 int64_t sh, int64_t sw, const float* in, const float* filt, float* out, hipStream_t st) {
  FlatConv g{in, filt, out, (int)H, (int)W, (int)C, (int)K, (int)R, (int)S, (int)sh, (int)sw, (int)((H - R) / sh + 1), (int)((W - S) / sw + 1)};
  g.qb = pl.TQ == 32 ? 5 : pl.TQ == 16 ? 4 : 3;
  g.tp_n = (int)cdiv(g.P, 32 >> g.qb);
  g.tq_n = (int)cdiv(g.Q, 1 << g.qb);
  g.CH = (int)cdiv(S * C, 8);
  g.T = (int)cdiv(R * g.CH, 2);
  g.in_elems = N * H * W * C;
  return pl.BN == 64 ? launch_t<2>(g, N, st) : launch_t<1>(g, N, st);
}

}  // namespace mdh
