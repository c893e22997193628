// fp32 products on the 16-bit matrix instructions, with the accuracy of fp32.
//
// An fp32 value has 24 significant bits, a bf16 value 8, and both have the same exponents: x = h + m + l with
// h = bf16(x), m = bf16(x - h), l = bf16(x - h - m) is exact (each difference is a float, |m| <= 2^-8 |x|,
// |l| <= 2^-17 |x|) as long as |x| >= 2^-100, whose last bit is well above the smallest normal number.  Of the nine
// products of two such sums the six
//     h h'   h m'   m h'   m m'   h l'   l h'
// are evaluated, each exact in the fp32 accumulation of v_mfma_f32_32x32x16_bf16, the smaller ones first; the three left
// out are below (1 + 2^-10) 2^-24 |x x'| together, the rounding error of ONE fp32 multiply-add.  That instruction cuts
// its sums off instead of rounding them to nearest, so a sum of one term is off by up to 3 x 2^-24 (2.9 met, 0.56 rms;
// fp32 instructions 1.0, 0.43) -- and exact where one factor is a power of two, which has one slice.  Longer sums have
// fewer roundings than a chain of fp32 multiply-adds and come out closer.  Error against 64 bits, 256 x 256 x K, relative
// 2-norm, one v_mfma_f32_32x32x2_f32 per two k against six bf16 instructions per 32 k:
//     U[-1,1]  K = 64: 1.4e-7 / 1.1e-7   256: 2.9e-7 / 2.4e-7   4096: 1.15e-6 / 1.0e-6   25088: 2.8e-6 / 2.7e-6
//     U[0,1]   K = 64: 1.2e-7 / 0.8e-7   256: 2.2e-7 / 1.8e-7   4096: 0.85e-6 / 0.5e-6   25088: 2.4e-6 / 1.6e-6
// (all nine products: the same digits).  Sums with many zeros in one operand have fewer terms than that chain has k, and
// up to six roundings for the steps they spread over: 64 of 147 terms 3.0 x 2^-24 against 2.4 with fp32 instructions, 8 of
// them 1.65 / 0.90 (dense 3.2 / 3.6).  Few-channel MCC, whose filters are like that, keeps h h' in a sum of its own
// and takes eight of the products, as do the tiles of MatMul that stand in for small ones on fp32 instructions.
// Rate of the bare instruction loops on random operands: 154 TFLOP/s in
// fp32, 1850 / 6 = 308 TFLOP/s in six bf16 products (the 16x16x32 form: 2220 / 6).
//
// Two kinds of values need more than that, and get the fp32 instructions (recompute_* in the kernels):
//   - not finite, or an overflow: Inf splits into Inf + NaN.  Every output that such a value enters comes out
//     not finite, so the outputs tell;
//   - |x| < 2^-100: its last slices may be lost to subnormal numbers, up to 2^-126.  That can matter only for an
//     output smaller than K * 2^-100 * (largest |x| of its tile), and only if such an element is there; both are
//     checked, in the output's own row and column.  An output whose row or column is all zeros -- padding, a dead
//     filter -- is small and exact: the largest magnitude of every row, kept as the values are split, tells without
//     reading the operands again.
#pragma once
#include "mdh_internal.h"

namespace mdh {
namespace split {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

enum { H = 0, Mid = 1, L = 2 };  // slices
struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

constexpr float kTiny = 7.88860905e-31f;  // 2^-100

// Two values per register (v_cvt_pk_bf16_f32), unpacked again by a shift and a mask for the subtractions: eight values
// take 48 instructions.  v_dot2c_f32_bf16 (DOT) unpacks and subtracts in one (x += p.lo q.lo + p.hi q.hi with q = (-1, 0)
// or (0, -1): 32 for eight values) but runs in the matrix pipe: beside a 32x32x16 MFMA (32 clocks) two of them take 45,
// four 56 and eight 78, six instructions of the other kinds 35 and eight 41-44 (clocks a slot and wavefront, one and two
// wavefronts a SIMD).
// The constants of the former are hidden from the compiler, which would encode 0x0000bf80 as the inline constant -1.0 --
// in a packed operand that is (0, -1).
template <bool DOT = false>
struct Split {
  unsigned neg_lo = 0x0000bf80u, neg_hi = 0xbf800000u;

  __device__ __forceinline__ Split() {
    if (DOT) asm("" : "+s"(neg_lo), "+s"(neg_hi));
  }

  static __device__ __forceinline__ unsigned pack(float a, float b) {
    const f2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf2));
  }
  // slice s of eight consecutive k of one row; what is left of them takes their place.  H also raises the largest
  // magnitude met so far.  (Level by level: a result of v_dot2c can be read only a few instructions later.)
  template <int s>
  __device__ __forceinline__ u4 slice(float (&x)[8], float& largest) const {
    u4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (s == H) largest = fmaxf(fmaxf(largest, fabsf(x[2 * e])), fabsf(x[2 * e + 1]));
      out[e] = pack(x[2 * e], x[2 * e + 1]);
    }
    if (s < L)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (DOT) {
          const unsigned word = out[e];  // (a cast of the element itself takes the first one's)
          const bf2 p = __builtin_bit_cast(bf2, word);
          x[2 * e] = __builtin_amdgcn_fdot2_f32_bf16(p, __builtin_bit_cast(bf2, neg_lo), x[2 * e], false);
          x[2 * e + 1] = __builtin_amdgcn_fdot2_f32_bf16(p, __builtin_bit_cast(bf2, neg_hi), x[2 * e + 1], false);
        } else {
          x[2 * e] -= __uint_as_float(out[e] << 16);
          x[2 * e + 1] -= __uint_as_float(out[e] & 0xffff0000u);
        }
      }
    return out;
  }
  // all three, 16 bytes each
  __device__ __forceinline__ void operator()(float (&x)[8], u4 (&out)[3], float& largest) const {
    out[H] = slice<H>(x, largest);
    out[Mid] = slice<Mid>(x, largest);
    out[L] = slice<L>(x, largest);
  }
};

__device__ __forceinline__ f16 mfma(u4 a, u4 b, f16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

// is a value of n consecutive ones too small to split exactly?  (a share of the workgroup's threads: part of parts)
__device__ __forceinline__ bool tiny(float v) { return v != 0.f && fabsf(v) < kTiny; }
__device__ __forceinline__ bool tiny_in(const float* __restrict__ p, int n, int part, int parts) {
  bool t = false;
  int i = part * 4;
#pragma unroll 4
  for (; i + 3 < n; i += parts * 4) {
    const f4 v = *(const f4u*)(p + i);
    t |= tiny(v[0]) || tiny(v[1]) || tiny(v[2]) || tiny(v[3]);
  }
  for (int e = i; e < n && e < i + 4; ++e) t |= tiny(p[e]);
  return t;
}

// a row with an infinity has no output that could be too small: what counts is the rows without
__device__ __forceinline__ float finite(float top) { return top < __builtin_huge_valf() ? top : 0.f; }

// The end of a workgroup's tile.  largest: magnitude of the finite values this thread has split; returns that of the
// workgroup's.  `word` is LDS that held 0 since before the last barrier.
__device__ __forceinline__ float workgroup_largest(float largest, unsigned* word) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) largest = fmaxf(largest, __shfl_xor(largest, d));
  if ((threadIdx.x & 63) == 0) atomicMax(word, __float_as_uint(largest));
  __syncthreads();
  return __uint_as_float(*word);
}

// bit r: is the word of an accumulator's output r of this lane not zero?  (rows of a 32 x 32 block, from the lane's on)
__device__ __forceinline__ unsigned nonzero_bits(const unsigned* words) {
  unsigned bits = 0;
#pragma unroll 4
  for (int r = 0; r < 16; ++r) bits |= (unsigned)(words[8 * (r / 4) + r % 4] != 0) << r;
  return bits;
}

// Rows (columns, pixels, output channels) that hold an output the split may not carry, in LDS that was 0: marked by any
// thread, each listed once.  An output depends on its own row and column only, so where few are listed -- a sum that
// came out zero by chance: 16 x 1024^3 random products hold about one -- those are read again, not the operands.
struct Marks {
  static constexpr unsigned kFew = 16;
  unsigned *count, *mark;
  unsigned short* list;
  static __host__ __device__ constexpr int words(int n) { return 1 + n + kFew / 2; }
  __device__ __forceinline__ Marks(unsigned* p, int n) : count(p), mark(p + 1), list((unsigned short*)(p + 1 + n)) {}
  __device__ __forceinline__ void add(int i) const {
    if (mark[i] || atomicExch(mark + i, 1u)) return;
    const unsigned at = atomicAdd(count, 1u);
    if (at < kFew) list[at] = (unsigned short)i;
  }
};

// buffer loads: base in scalar registers, so that a load takes no vector instruction for its address
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const float* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)0xffffffff, 0x00027000);
}

}  // namespace split
}  // namespace mdh
