// Multi-channel convolution instance of md_hom(*, (++,++,++,++,+,+,+)) for gfx950 on the bf16 matrix instructions,
// every fp32 value carried as a sum of three bf16 values (mdh_split.h: six products per multiply-add, accuracy of
// fp32).  out[n,p,q,k] = sum_{c,r,s} in[n, p*sh + r, q*sw + s, c] * filt[k,r,s,c]    (NHWC, KRSC, NPQK)
//
// De-composition as in mdh_mcc.hip, dims (n,p,q,k,c,r,s): a workgroup owns TP x TQ pixels of one image and BN
// output channels; per chunk of CK channels the input patch is split and staged ONCE for all R*S taps -- so a value
// of the input is split about once per workgroup, not once per product -- and the filter slice of a tap is split and
// staged while the tap before it is multiplied.  Block: 32 pixels x 32 output channels x 16 input channels, six
// v_mfma_f32_32x32x16_bf16.
// LDS: patch [slice][c / 8][pixel] and filter [slice][c / 8][k], 16 bytes (eight channels) per entry, so that an
// MFMA operand of a lane is one ds_read_b128.
#include "mdh_split.h"

namespace mdh {
namespace {

using namespace split;

template <int TP, int TQ, int BN, int CK, int WM, int WN>
struct Cfg {
  static_assert(TQ == 32 || TQ == 16 || TQ == 8, "an MFMA block spans 32 pixels: 32/TQ rows of TQ columns");
  static constexpr int RB = 32 / TQ;  // output rows per block
  static constexpr int MI = WM / 32, NI = WN / 32;
  static_assert(TP % (MI * RB) == 0, "rows of the tile = wavefronts x blocks x rows per block");
  static constexpr int WAVES_M = TP / (MI * RB), WAVES_N = BN / WN;
  static constexpr int NT = WAVES_M * WAVES_N * 64;
  // Wavefronts a SIMD must be able to hold: what LDS has room for.  Without a demand the compiler keeps accumulators in
  // accumulation registers and moves them about, or not, as the rest of the kernel comes out (2 x 17 x 22 x 292 -> 728,
  // 3 x 9, 8 x 16 x 64 tiles 170 / 189 us; 8 x 16 x 128 in chunks of 16 channels 315 / 356).  Tiles of one block a
  // wavefront are ahead without (8 x 118 x 12 x 67 -> 938, 11 x 9: 900 / 1015).
  static constexpr int HELD = MI * NI == 1 ? 1 : CK == 32 && MI * NI == 4 ? 2 : 3;
  static constexpr int KP = CK / 8, KH = CK / 16;
  static constexpr int F_PLANE = BN * 16, F_SLICE = KP * F_PLANE, F_STAGE = 3 * F_SLICE;
  static constexpr int F_CHUNKS = BN * KP;
  static constexpr int F_CH = (F_CHUNKS + NT - 1) / NT;
  // patch planes are padded so that the planes of one pixel start 64 (CK = 16) or 32 bytes apart in the banks
  static constexpr int PAD = CK == 16 ? 4 : 2;
  static_assert((160 * 1024 - 2 * F_STAGE) / (3 * KP * 16) * KP <= 31 * NT, "a bit per pixel of a thread");
  static __host__ __device__ __forceinline__ int plane(int npix) { return ((npix + 7) / 8 * 8 + PAD) * 16; }
};

struct Conv {
  const float *in, *filt;
  float* out;
  int H, W, C, K, R, S, sh, sw, P, Q;
};

// four consecutive channels from c on, those at or beyond cend as 0
__device__ __forceinline__ f4 four_c(const float* __restrict__ p, int c, int cend) {
  if (c + 3 < cend) return *(const f4u*)(p + c);
  f4 v;
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = c + t < cend ? p[c + t] : 0.f;
  return v;
}

// fp32 evaluation of a wavefront's blocks, for values the split does not carry: 16 channels of a tap at a time, the next
// ones on their way while these are multiplied
template <int TP, int TQ, int BN, int CK, int WM, int WN>
__device__ __forceinline__ void recompute_fp32(const Conv& g, float* __restrict__ dst, int n, int p0, int q0, int k0, int cbeg, int cend) {
  using C = Cfg<TP, TQ, BN, CK, WM, WN>;
  constexpr int KS = 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lh = lane >> 5;
  const int pw = p0 + wave / C::WAVES_N * C::MI * C::RB, kw = k0 + wave % C::WAVES_N * WN, q = q0 + l32 % TQ;
  if (pw >= g.P || kw >= g.K) return;
  const float *a[C::MI], *b[C::NI];
#pragma unroll
  for (int mi = 0; mi < C::MI; ++mi)
    a[mi] = g.in + (((int64_t)n * g.H + min(pw + mi * C::RB + l32 / TQ, g.P - 1) * g.sh) * g.W + min(q, g.Q - 1) * g.sw) * g.C + lh * 4;
#pragma unroll
  for (int ni = 0; ni < C::NI; ++ni) b[ni] = g.filt + (int64_t)min(kw + ni * 32 + l32, g.K - 1) * g.R * g.S * g.C + lh * 4;
  f16 acc[C::MI][C::NI];
#pragma unroll
  for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 0.f;
  f4 y[KS][C::MI], x[KS][C::NI];
  int r = 0, s = 0, c = cbeg;  // of the step that `load` takes
  auto load = [&] {
    const int in = (r * g.W + s) * g.C, fl = (r * g.S + s) * g.C;
#pragma unroll
    for (int u = 0; u < KS; ++u) {
#pragma unroll
      for (int mi = 0; mi < C::MI; ++mi) y[u][mi] = four_c(a[mi] + in, c + u * 8, cend - lh * 4);
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni) x[u][ni] = four_c(b[ni] + fl, c + u * 8, cend - lh * 4);
    }
    c += 8 * KS;
    if (c >= cend) {
      c = cbeg;
      if (++s == g.S) s = 0, ++r;
    }
  };
  load();
  for (bool more = true; more;) {
    f4 yc[KS][C::MI], xc[KS][C::NI];
#pragma unroll
    for (int u = 0; u < KS; ++u) {
#pragma unroll
      for (int mi = 0; mi < C::MI; ++mi) yc[u][mi] = y[u][mi];
#pragma unroll
      for (int ni = 0; ni < C::NI; ++ni) xc[u][ni] = x[u][ni];
    }
    more = r < g.R;
    if (more) load();
#pragma unroll
    for (int u = 0; u < KS; ++u)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
          for (int ni = 0; ni < C::NI; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(xc[u][ni][t], yc[u][mi][t], acc[mi][ni], 0, 0, 0);
  }
#pragma unroll
  for (int mi = 0; mi < C::MI; ++mi) {
    const int p = pw + mi * C::RB + l32 / TQ;
    if (p >= g.P || q >= g.Q) continue;
    float* const o = dst + (((int64_t)n * g.P + p) * g.Q + q) * g.K;
#pragma unroll
    for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = kw + ni * 32 + 8 * (e / 4) + 4 * lh + e % 4;
        if (k < g.K) o[k] = acc[mi][ni][e];
      }
  }
}

// does one of `runs` runs of nc channels, run i at p + at(i), hold an element too small to split exactly?  (this thread's
// share)
template <int NT, class At>
__device__ __forceinline__ bool tiny_runs(const float* __restrict__ p, int runs, int nc, At at) {
  bool t = false;
  constexpr int W = 16;  // threads per run
  for (int i = threadIdx.x / W; i < runs; i += NT / W) t |= tiny_in(p + at(i), nc, threadIdx.x % W, W);
  return t;
}

// does the workgroup's part of the input and of the filter -- of the windows and output channels that are listed, where
// they are few -- hold an element too small to split exactly?  (this thread's share)
template <int NT, int TQ>
__device__ __forceinline__ bool holds_tiny(const Conv& g, int n, int p0, int q0, int PH, int PW, int k0, int BN, int cbeg, int cend,
                                           const Marks& pm, const Marks& fm) {
  bool t = false;
  const int nc = cend - cbeg, h0 = p0 * g.sh, w0 = q0 * g.sw, taps = g.R * g.S;
  const int nh = min(PH, g.H - h0), nw = min(PW, g.W - w0);
  const float* const in = g.in + (((int64_t)n * g.H + h0) * g.W + w0) * g.C + cbeg;
  if (*pm.count <= Marks::kFew)
    for (unsigned i = 0; i < *pm.count; ++i) {
      const int first = pm.list[i] / TQ * g.sh * g.W + pm.list[i] % TQ * g.sw;
      t |= tiny_runs<NT>(in, taps, nc, [&](int r) { return (int64_t)(first + r / g.S * g.W + r % g.S) * g.C; });
    }
  else
    t |= tiny_runs<NT>(in, nh * nw, nc, [&](int i) { return (int64_t)(i / nw * g.W + i % nw) * g.C; });
  const float* const f = g.filt + (int64_t)k0 * taps * g.C + cbeg;
  if (*fm.count <= Marks::kFew)
    for (unsigned i = 0; i < *fm.count; ++i)
      t |= tiny_runs<NT>(f + (int64_t)fm.list[i] * taps * g.C, taps, nc, [&](int r) { return (int64_t)r * g.C; });
  else
    t |= tiny_runs<NT>(f, min(BN, g.K - k0) * taps, nc, [&](int i) { return (int64_t)i * g.C; });
  return t;
}

// One tap is six phases, one per product, as a k-tile of the split MatMul: LDS holds the filter slices of two taps,
// the filter of tap t+1 is split while tap t is multiplied, that of tap t+2 is on its way from memory, and the one
// barrier of a tap stands where all its operands are in registers.  The smaller products come first, for the reason
// given there.
template <int TP, int TQ, int BN, int CK, int WM, int WN, bool AHEAD>
__global__ __launch_bounds__((Cfg<TP, TQ, BN, CK, WM, WN>::NT), (AHEAD && CK == 32 && Cfg<TP, TQ, BN, CK, WM, WN>::MI * Cfg<TP, TQ, BN, CK, WM, WN>::NI == 2 ? 2 : Cfg<TP, TQ, BN, CK, WM, WN>::HELD)) void mcc_split_kernel(
    Conv g, float* __restrict__ ws, int tp_n, int tq_n, int tk_n, int n_img, int SC, int cchunk) {
  using F = Cfg<TP, TQ, BN, CK, WM, WN>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  // XCD-aware order: each of the 8 XCDs gets a contiguous run of tiles; inside a run the channel tiles of one
  // pixel patch come first (they share the patch), then q, p, n.
  int b = xcd_order(blockIdx.x, gridDim.x);
  const int tk = b % tk_n, tq = (b / tk_n) % tq_n, tp = (b / (tk_n * tq_n)) % tp_n;
  const int n = (b / (tk_n * tq_n * tp_n)) % n_img;
  const int sc = b / (tk_n * tq_n * tp_n * n_img);  // part of the reduction dimension c
  const int p0 = tp * TP, q0 = tq * TQ, k0 = tk * BN;
  const int cbeg = sc * cchunk, cend = min(g.C, cbeg + cchunk);
  float* const dst = SC > 1 ? ws + (int64_t)sc * n_img * g.P * g.Q * g.K : g.out;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / F::WAVES_N, wn = wave % F::WAVES_N;
  const int l32 = lane & 31, lh = lane >> 5;
  const int PH = (TP - 1) * g.sh + g.R, PW = (TQ - 1) * g.sw + g.S, npix = PH * PW;
  const int pplane = F::plane(npix), pslice = F::KP * pplane;
  char* const patch = lds + 2 * F::F_STAGE;
  unsigned* const largest = (unsigned*)(patch + 3 * pslice);
  if (tid == 0) *largest = 0;

  f16 acc[F::MI][F::NI];
#pragma unroll
  for (int mi = 0; mi < F::MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < F::NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  const Split<> split;
  const int taps = g.R * g.S;
  // filter chunks of this thread: eight channels of one output channel; channels beyond K repeat the last one
  float fx[F::F_CH][8];
  float ftop[F::F_CH], ptop = 0.f;  // largest magnitude split: of the chunk's output channel, of the patch
  unsigned pnz = 0;                 // bit i: this thread's i-th pixel is not all zeros (a patch that fits has less than 32)
  unsigned foff[F::F_CH];
#pragma unroll
  for (int c = 0; c < F::F_CH; ++c) {
    const int f = (tid + c * F::NT) % F::F_CHUNKS;
    ftop[c] = 0.f;
    foff[c] = (unsigned)(min(f / F::KP, g.K - 1 - k0) * (taps * g.C) + f % F::KP * 8) * 4u;
  }
  const float* const fbase = g.filt + (int64_t)k0 * taps * g.C;
  auto load_filter = [&](int tap, int c0, int c) {
    const auto r = rsrc(fbase + tap * g.C + c0);
    const f4 a = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, foff[c], 0, 0));
    const f4 d = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, foff[c] + 16, 0, 0));
#pragma unroll
    for (int e = 0; e < 4; ++e) fx[c][e] = a[e], fx[c][e + 4] = d[e];
  };
  // (a workgroup with more threads than chunks writes some of them twice, the same bytes)
  auto store_filter = [&](char* st, int c) {
    const int f = (tid + c * F::NT) % F::F_CHUNKS;
    const int k = f / F::KP, kc = f % F::KP;
    u4 v[3];
    split(fx[c], v, ftop[c]);
    char* p = st + kc * F::F_PLANE + (k ^ (64 / CK * kc)) * 16;
#pragma unroll
    for (int s = 0; s < 3; ++s) *(u4*)(p + s * F::F_SLICE) = v[s];
  };
  // input patch of the channels from c0 on; the first `skip` of them belong to the chunk before and read as 0
  auto stage_patch = [&](int c0, int skip) {
    unsigned bit = 1;
    for (int f = tid; f < npix * F::KP; f += F::NT, bit <<= 1) {
      const int pix = f / F::KP, kc = f % F::KP;
      const int ph = pix / PW, pw = pix - ph * PW;
      const int hy = min(p0 * g.sh + ph, g.H - 1), wx = min(q0 * g.sw + pw, g.W - 1);
      const float* p = g.in + (((int64_t)n * g.H + hy) * g.W + wx) * g.C + c0 + kc * 8;
      const f4 a = *(const f4u*)p, d = *(const f4u*)(p + 4);
      float x[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = a[e], x[e + 4] = d[e];
      if (skip) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = kc * 8 + e < skip ? 0.f : x[e];
      }
      u4 v[3];
      float top = 0.f;
      split(x, v, top);
      ptop = fmaxf(ptop, finite(top));
      pnz |= top != 0.f ? bit : 0;
#pragma unroll
      for (int s = 0; s < 3; ++s) *(u4*)(patch + s * pslice + kc * pplane + pix * 16) = v[s];
    }
  };

  // Operands of the tap that is multiplied; the high slices of the one before are still in use when those of the next are
  // read, so they have two places.
  struct Regs {
    u4 y[F::MI][F::KH], x[F::NI][F::KH];
  } mid, low, high[2];
  const int pix0 = (wm * F::MI * F::RB + l32 / TQ) * g.sh * PW + l32 % TQ * g.sw;
  const int block_rows = F::RB * g.sh * PW * 16;  // LDS distance between consecutive blocks of a wavefront
  auto read_y = [&](Regs& to, int at, int s) {  // at: the tap's pixel offset
#pragma unroll
    for (int h = 0; h < F::KH; ++h)
#pragma unroll
      for (int mi = 0; mi < F::MI; ++mi)
        to.y[mi][h] = *(const u4*)(patch + s * pslice + (2 * h + lh) * pplane + (pix0 + at) * 16 + mi * block_rows);
  };
  auto read_x = [&](Regs& to, const char* st, int s) {
#pragma unroll
    for (int h = 0; h < F::KH; ++h) {
      const int kc = 2 * h + lh;
      const char* p = st + s * F::F_SLICE + kc * F::F_PLANE + (wn * WN + (l32 ^ (64 / CK * kc))) * 16;
#pragma unroll
      for (int ni = 0; ni < F::NI; ++ni) to.x[ni][h] = *(const u4*)(p + ni * 512);
    }
  };
  auto mma = [&](const Regs& a, const Regs& b) {  // pixels of a, filter of b
#pragma unroll
    for (int h = 0; h < F::KH; ++h)
#pragma unroll
      for (int mi = 0; mi < F::MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < F::NI; ++ni) acc[mi][ni] = mfma(b.x[ni][h], a.y[mi][h], acc[mi][ni]);
  };
  // Phases 0 to 3 are one scheduling region: an MFMA, an LDS read, a share of the next tap's split (out of the matrix pipe:
  // with the reads ahead and the search behind the stores, side by side, 16 x 224 x 224 x 64 -> 128, 7 x 7, 2740 -> 2655 us;
  // 16 x 56 x 56 x 64 -> 64, 3 x 3, 29.3 -> 28.2).
  // AHEAD: the patch is there for all taps, so the pixels of the next one are read from phase 2 on, its filter behind the
  // barrier, and every operand is requested two phases or more before it is multiplied; else one phase.
  constexpr int PM = F::KH * F::MI * F::NI;  // MFMAs of a phase
  auto body = [&](int tap, int at, int at_next, int c0, auto par_, auto more_) {
    constexpr bool more = decltype(more_)::value;
    constexpr int par = decltype(par_)::value ? 1 : 0;
    const char *const cur = lds + (tap & 1) * F::F_STAGE, *const nxt = lds + ((tap + 1) & 1) * F::F_STAGE;
    if (!AHEAD) read_x(high[par], cur, H);
    mma(mid, mid);
    if (!AHEAD) read_y(high[par], at, H);
    mma(mid, high[par]);
    if (!AHEAD) read_x(low, cur, L);
    if (AHEAD && more) read_y(mid, at_next, Mid);
    mma(high[par], mid);
    if (!AHEAD) read_y(low, at, L);
    if (AHEAD && more) read_y(high[par ^ 1], at_next, H);
    mma(high[par], low);
    if (more) {
#pragma unroll
      for (int c = 0; c < F::F_CH; ++c) {
        store_filter(lds + ((tap + 1) & 1) * F::F_STAGE, c);
        load_filter(min(tap + 2, taps - 1), c0, c);
      }
    }
    constexpr int V = (48 * F::F_CH + 4 * PM - 1) / (4 * PM);
#pragma unroll
    for (int i = 0; i < 4 * PM; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (!AHEAD || (more && i >= 2 * PM)) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (more) __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (more) {
      __syncthreads();
      if (!AHEAD) read_y(mid, at_next, Mid);
      read_x(mid, nxt, Mid);
      if (AHEAD) read_x(high[par ^ 1], nxt, H);
      if (AHEAD) read_x(low, nxt, L);
    }
    mma(low, high[par]);
    if (AHEAD && more) read_y(low, at_next, L);
    mma(high[par], high[par]);
    __builtin_amdgcn_sched_barrier(0);
  };

  for (int cc = cbeg; cc < cend; cc += CK) {
    // the last chunk ends with the last channel: where the part is no whole number of chunks it starts inside the
    // chunk before it
    const int c0 = min(cc, cend - CK);
#pragma unroll
    for (int c = 0; c < F::F_CH; ++c) load_filter(0, c0, c);
    if (cc > cbeg) __syncthreads();  // every wavefront is done with the previous patch and filter stages
    stage_patch(c0, cc - c0);
#pragma unroll
    for (int c = 0; c < F::F_CH; ++c) {
      store_filter(lds, c);
      load_filter(min(1, taps - 1), c0, c);
    }
    __syncthreads();
    read_y(mid, 0, Mid);
    read_x(mid, lds, Mid);
    if (AHEAD) {
      read_x(high[0], lds, H);
      read_y(high[0], 0, H);
      read_x(low, lds, L);
      read_y(low, 0, L);
    }
    int r = 0, s = 0, at = 0, tap = 0;
    auto step = [&](auto par) {
      if (++s == g.S) s = 0, ++r;
      const int to = r * PW + s;
      body(tap++, at, to, c0, par, Yes{});
      at = to;
    };
    if constexpr (AHEAD) {
      while (tap + 2 < taps) {
        step(No{});
        step(Yes{});
      }
      if (tap + 1 < taps) {
        step(No{});
        body(tap, at, 0, c0, Yes{}, No{});
      } else {
        body(tap, at, 0, c0, No{}, No{});
      }
    } else {
      while (tap + 1 < taps) step(No{});
      body(tap, at, 0, c0, No{}, No{});
    }
  }

  // output view (n,p,q,k,0,0,0) -> out[n,p,q,k]: a lane holds four consecutive k of one pixel
  const bool whole = p0 + TP <= g.P && q0 + TQ <= g.Q && k0 + BN <= g.K;
#pragma unroll
  for (int mi = 0; mi < F::MI; ++mi) {
    const int p = p0 + (wm * F::MI + mi) * F::RB + l32 / TQ, q = q0 + l32 % TQ, kb = k0 + wn * WN + 4 * lh;
    float* const o = dst + (((int64_t)n * g.P + p) * g.Q + q) * g.K + kb;
#pragma unroll
    for (int ni = 0; ni < F::NI; ++ni)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int j = ni * 32 + 8 * q4;
        const f4 v = {acc[mi][ni][4 * q4], acc[mi][ni][4 * q4 + 1], acc[mi][ni][4 * q4 + 2], acc[mi][ni][4 * q4 + 3]};
        if (whole) {
          *(f4u*)(o + j) = v;
        } else if (p < g.P && q < g.Q) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (kb + j + e < g.K) o[j + e] = v[e];
        }
      }
  }

  // Values the split does not carry (mdh_split.h).  The outputs are on their way by now: the search takes its time beside
  // the stores (before them it was 1.4 us of the 28 of 16 x 56 x 56 x 64 -> 64, 3 x 3).
  float z = 0.f, least = __builtin_huge_valf();
#pragma unroll
  for (int mi = 0; mi < F::MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < F::NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        z = __builtin_fmaf(acc[mi][ni][r], 0.f, z);
        least = fminf(least, fabsf(acc[mi][ni][r]));
      }
  float top = ptop;
#pragma unroll
  for (int c = 0; c < F::F_CH; ++c) top = fmaxf(top, finite(ftop[c]));
  const float bound = (float)(taps * (cend - cbeg)) * kTiny * workgroup_largest(top, largest);
  bool fp32 = __any(!(z == 0.f));
  if (__syncthreads_or(least < bound)) {
    // the operands' stages are done with: the largest magnitude of every output channel (bits of a float), and whether a
    // pixel of the patch is not all zeros
    unsigned* const filters = (unsigned*)lds;
    unsigned* const pixels = filters + BN;
    const Marks pm(pixels + npix, TP * TQ), fm(pixels + npix + Marks::words(TP * TQ), BN);
    static_assert((BN + Marks::words(TP * TQ) + Marks::words(BN)) * 4 <= 2 * F::F_STAGE, "");  // and 4 bytes a pixel in the patch
    for (int i = tid; i < BN + npix + Marks::words(TP * TQ) + Marks::words(BN); i += F::NT) filters[i] = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < F::F_CH; ++c) atomicMax(filters + (tid + c * F::NT) % F::F_CHUNKS / F::KP, __float_as_uint(ftop[c]));
    __syncthreads();
    unsigned small[F::MI][F::NI];  // the block's outputs of this lane
    bool open = false;
#pragma unroll
    for (int ni = 0; ni < F::NI; ++ni) {
      const unsigned live = nonzero_bits(filters + wn * WN + ni * 32 + 4 * lh);
#pragma unroll
      for (int mi = 0; mi < F::MI; ++mi) {
        unsigned bits = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) bits |= (unsigned)(fabsf(acc[mi][ni][r]) < bound) << r;
        const bool stored = p0 + (wm * F::MI + mi) * F::RB + l32 / TQ < g.P && q0 + l32 % TQ < g.Q;
        small[mi][ni] = stored ? bits & live : 0;
        open |= small[mi][ni] != 0;
      }
    }
    if (__syncthreads_or(open)) {
      for (int i = 0; tid + i * F::NT < npix * F::KP; ++i)
        if (pnz >> i & 1) pixels[(tid + i * F::NT) / F::KP] = 1;
      __syncthreads();
      open = false;
#pragma unroll
      for (int mi = 0; mi < F::MI; ++mi) {
        unsigned any = 0, window = 0;
#pragma unroll
        for (int ni = 0; ni < F::NI; ++ni) any |= small[mi][ni];
        if (any)
          for (int r = 0; r < g.R; ++r)
            for (int s = 0; s < g.S; ++s) window |= pixels[pix0 + (mi * F::RB * g.sh + r) * PW + s];
        if (!window) continue;
        open = true;
        pm.add(((wm * F::MI + mi) * F::RB + l32 / TQ) * TQ + l32 % TQ);
#pragma unroll
        for (int ni = 0; ni < F::NI; ++ni)
          for (unsigned bits = small[mi][ni]; bits; bits &= bits - 1) {
            const int r = __builtin_ctz(bits), k = wn * WN + ni * 32 + 8 * (r / 4) + 4 * lh + r % 4;
            if (k0 + k < g.K) fm.add(k);
          }
      }
      open = __any(open);
      if (__syncthreads_or(open)) {
        const bool found = holds_tiny<F::NT, TQ>(g, n, p0, q0, PH, PW, k0, BN, cbeg, cend, pm, fm);
        if (__syncthreads_or(found)) fp32 |= open;
      }
    }
  }
  // (written over what was stored above, by the same lanes; a wavefront's stores to an address stay in order)
  if (fp32) recompute_fp32<TP, TQ, BN, CK, WM, WN>(g, dst, n, p0, q0, k0, cbeg, cend);
}

template <int TP, int TQ, int BN, int CK, int WM, int WN>
mdh_status launch_t(int SC, int64_t N, const Conv& g, void* ws, hipStream_t st) {
  using F = Cfg<TP, TQ, BN, CK, WM, WN>;
  const int npix = ((TP - 1) * g.sh + g.R) * ((TQ - 1) * g.sw + g.S);
  const int64_t lds_bytes = 2ll * F::F_STAGE + 3ll * F::KP * F::plane(npix) + 16;
  if (lds_bytes > 160 * 1024) return MDH_ERR_TILE_RESOURCES;
  // One tap has nothing to read ahead, tiles of 64 x 64 a wavefront have no registers for it, and 64 pixels x 32 channels in
  // chunks of 32 are slower with it (16 x 56 x 56 x 64 -> 64, 3 x 3, 30.6 -> 32.2 us).  The others: 8 x 16 x 16 x 33 -> 90,
  // 5 x 5, 18.3 -> 15.7; 20 x 12 x 12 x 160 -> 100, 7 x 7, 111 -> 95; 32 x 7 x 7 x 200 -> 64, 3 x 3, 17.0 -> 15.0.
  constexpr bool ROOM = F::MI * F::NI == 1 || (F::MI * F::NI == 2 && (CK == 16 || F::NI == 2));
  const bool ahead = ROOM && g.R * g.S > 1;
  auto kern = ahead ? mcc_split_kernel<TP, TQ, BN, CK, WM, WN, ROOM> : mcc_split_kernel<TP, TQ, BN, CK, WM, WN, false>;
  static int64_t lds_allowed[2][kMaxDevices] = {};
  if (allow_dynamic_lds((const void*)kern, lds_bytes, lds_allowed[ahead]) != MDH_OK) return MDH_ERR_LAUNCH;
  const int64_t tp_n = cdiv(g.P, TP), tq_n = cdiv(g.Q, TQ), tk_n = cdiv(g.K, BN);
  if (SC < 1) return MDH_ERR_UNSUPPORTED;
  // Parts of whole steps of 16 channels, also in chunks of 32 (a part's last chunk starts inside the one before; the first needs
  // 32 channels): with whole chunks 66 channels in two parts were 64 and 2, and 1.25 times as far from 64 bits as 48 and 18.
  const int64_t even = cdiv(cdiv(g.C, SC), 16) * 16, cchunk = even > CK ? even : CK;
  if ((SC - 1) * cchunk >= g.C) return MDH_ERR_TILE_NOT_DIVIDING;  // a part without channels
  const int64_t nblocks = N * tp_n * tq_n * tk_n * SC;
  if (nblocks > 0x7fffffff) return MDH_ERR_SIZE;
  clear_stale_error();
  hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(F::NT), (size_t)lds_bytes, st, g, (float*)ws, (int)tp_n, (int)tq_n,
                     (int)tk_n, (int)N, SC, (int)cchunk);
  mdh_status r = launch_status();
  if (r != MDH_OK || SC <= 1) return r;
  return launch_combine_sum((const float*)ws, g.out, N * g.P * g.Q * g.K, SC, st);
}

}  // namespace

mdh_status launch_mcc_split(const MccPlan& pl, int64_t N, int64_t H, int64_t W, int64_t C, int64_t K, int64_t R, int64_t S,
                            int64_t sh, int64_t sw, const float* in, const float* filt, float* out, void* ws, hipStream_t st) {
  const Conv g{in,     filt,   out,    (int)H,  (int)W, (int)C, (int)K, (int)R, (int)S, (int)sh, (int)sw,
               (int)((H - R) / sh + 1), (int)((W - S) / sw + 1)};
#define MDH_CS(tp, tq, bn, ck, wm, wn)                                                        \
  if (pl.TP == tp && pl.TQ == tq && pl.BN == bn && pl.CK == ck && pl.WM == wm && pl.WN == wn) \
    return launch_t<tp, tq, bn, ck, wm, wn>(pl.S, N, g, ws, st);
  MDH_CS(8, 32, 128, 16, 64, 64)
  MDH_CS(4, 32, 128, 16, 64, 64)
  MDH_CS(4, 32, 64, 16, 64, 32)
  MDH_CS(8, 16, 128, 16, 64, 64)
  MDH_CS(8, 16, 64, 16, 64, 32)
  MDH_CS(8, 8, 128, 16, 32, 64)
  MDH_CS(8, 8, 64, 16, 32, 32)
  MDH_CS(8, 32, 128, 32, 64, 64)
  MDH_CS(4, 32, 128, 32, 64, 64)
  MDH_CS(4, 32, 64, 32, 64, 32)
  MDH_CS(8, 16, 128, 32, 64, 64)
  MDH_CS(8, 16, 64, 32, 64, 32)
  MDH_CS(16, 8, 64, 32, 64, 32)
  MDH_CS(8, 8, 128, 32, 32, 64)
  MDH_CS(8, 8, 64, 32, 32, 32)
#undef MDH_CS
  return MDH_ERR_UNSUPPORTED;
}

}  // namespace mdh
