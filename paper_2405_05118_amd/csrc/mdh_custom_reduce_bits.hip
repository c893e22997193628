// Custom-combine instance md_hom(wght, (++, max_idx)), large products: the records of B as bit maps.
//
// A pair costs the loop over fields (mdh_custom_reduce.hip) three vector instructions per field.  Here 32 pairs share
// them.  A workgroup takes B in chunks of 128 records and keeps in LDS, per field and slot h(value), the 128-bit map of
// the records whose field falls into that slot; one ds_read_b128 then tells a lane, which owns a record of A, all records
// of the chunk that agree with it in that field -- or collide with it, so a map may hold too many records, never too few.
//
// Upper bound of a score, for 32 records at a time: every field has a whole weight q_f in [0, 15], q_f = 0 unless agreeing
// raises the score, sum_f q_f <= 30.  The maps are added up as bits, plane i of the sum holding bit i of 32 records' sums
// u = sum_f q_f [slots agree]: a full adder is two three-input bit operations, and the constant q_f, the same for every
// lane, selects code without the operations its zero bits do not need.
// What u has to reach follows from the 2^nF ways to agree: most[u] = the largest score among those with a sum of at most
// u, so no record with u < t(s) = min { u : most[u] > s } scores more than s.  t comes from the best record so far, the
// comparison u >= t is five more bit operations, and the few records that pass are scored exactly, from the values
// themselves and in the arithmetic of the definition.  The result is that of the definition for any values and weights;
// only the time depends on them.
//
// Best records live in device memory as keys, (score, -index) packed so that a larger key is a better record, and are
// raised with atomicMax: the workgroups that walk other parts of B profit from one another's records.  What the result is
// does not depend on when they see them: a record of an earlier part with an equal score has to pass (t(s - 1)).
//
// Slots that collide throughout or weights that q cannot tell apart would have too many records scored: a wavefront that
// does (`left`) raises a flag and the others stop; the loop over fields, launched behind, starts only if the flag is up.
// us, that loop alone / a call that takes both: weights that wrap around, known before the walk, 2^14 x 2^17 records of 8
// fields 1300 / 1350, 4096 x 2^16 203 / 234; B of eight different records 2^14 x 2^17 953 / 1180, 2^16 x 2^18 6870 / 7810;
// slots that all collide 2^14 x 2^17 957 / 1170, 4096 x 2^16 160 / 377, 2^16 x 2^18 6890 / 7660; in every other eight chunks
// 2^14 x 2^17 954 / 1530.  (32-bit hashes, none equal, stay with the maps: 1290 / 450, 2^16 x 2^18 10030 / 2930.)
//
// Bound by the issue of vector instructions, 320 per 128 x 64 pairs of 8 fields (the loop over fields: 25.6 a pair and
// lane).  us, the loop over fields / this: 2^16 x 2^18 records of 8 fields 6850 / 985; 2^15 x 2^17 of 12 3000 / 520; 2^15 x
// 2^18 of 4 2080 / 346; 2^10 x 2^18 of 8 224 / 83; 2^12 x 2^14 of 8 63 / 51.  Two workgroups of 16 wavefronts a compute unit
// (64 KB of maps) are ahead of one (128 KB, 1024 slots for every field): a wavefront issues every five cycles, a SIMD twice
// as often.
#include <limits.h>

#include "mdh_internal.h"
#include "mdh_prl_bits.h"

namespace mdh {
namespace {

using u4 = __attribute__((ext_vector_type(4))) unsigned;

constexpr int kNT = 1024, kPrepNT = 256, kSeed = 128, kPlanes = 5, kLevels = 1 << kPlanes, kTop = kLevels - 2;
constexpr int kSearchKP = 6;  // weights are searched for up to 12 fields

// Slot of a value: its low bits with the higher ones folded in, so values below the number of slots do not collide.
__device__ __forceinline__ unsigned slot_of(int value, int bits) {
  unsigned v = (unsigned)value;
  v ^= v >> (2 * bits);
  v ^= v >> bits;
  return v & ((1u << bits) - 1);
}

__device__ __forceinline__ unsigned long long key_of(int s, int b) {
  return (unsigned long long)((unsigned)s ^ 0x80000000u) << 32 | ~(unsigned)b;
}

// The weights q, one choice: agreeing in all fields that raise a score makes at most kTop.  Choices differ in scale and
// rounding.
template <int NF>
__device__ __forceinline__ bool choose(const float (&d)[NF], float sum, int choice, int (&q)[NF]) {
  const float scale = sum > 0 ? kTop * (1.f - 0.55f / 64 * (choice & 63)) / sum : 0.f;
  const float up = choice < 64 ? 0.5f : choice < 128 ? 0.3f : choice < 192 ? 0.7f : 0.f;
  int all = 0;
#pragma unroll
  for (int f = 0; f < NF; ++f) all += q[f] = d[f] > 0 ? min(15, (int)(d[f] * scale + up)) : 0;
  return all <= kTop;
}

// Every workgroup looks at the same kSeed records from all over B: their values tell how many slots a field gets (the maps
// of all fields share 64 KB).  The first kSearch workgroups then look for the weights, a choice per wavefront; the others
// find the slots of A and the best of those records, so that the first chunks have few to score.
//
// What a choice costs is the number of records it would have scored, W(p) = w(p) / max(tail(p), 1 / nB)^2 for the time
// pattern p is that of the best record so far and the frequency of sums that reach its t; w(p) from how often each field
// agrees in a sample, the fields taken as independent, tail(p) the frequency of a score as large.  Of 2^18 records of 8
// fields, 6-33 are scored for a record of A (5.6 improve on the best); with the largest scale and plain rounding 12-55.
template <int KP>
__global__ __launch_bounds__(kPrepNT) void prl_bits_prep_kernel(const int* __restrict__ A, const int* __restrict__ B,
                                                                 const int* __restrict__ wp, const int* __restrict__ wm,
                                                                 unsigned long long* __restrict__ keys,
                                                                 unsigned* __restrict__ slots, PrlBitsHead* __restrict__ head,
                                                                 int nA, int nB, int nF) {
  constexpr int NF = 2 * KP, P = KP <= kSearchKP ? 1 << NF : 1, NT = kPrepNT, BINS = NT, WAVES = NT / 64;
  __shared__ int seed[kSeed * NF];
  __shared__ unsigned used[NF];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int seeds = min(kSeed, nB), step = nB / seeds;
  const int a = ((int)blockIdx.x - kSearch) * NT + tid;
  int ar[NF];
  if (blockIdx.x >= kSearch)
#pragma unroll
    for (int f = 0; f < NF; ++f) ar[f] = A[(int64_t)min(a, nA - 1) * nF + min(f, nF - 1)];
  if (tid < NF) used[tid] = 0;
  __syncthreads();
  for (int e = tid; e < seeds * NF; e += NT) {
    const int f = e % NF, v = B[(int64_t)(e / NF) * step * nF + min(f, nF - 1)];
    seed[e] = v;
    atomicOr(&used[f], (unsigned)v);
  }
  __syncthreads();
  PrlSlots sl;
  {
    unsigned u[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) u[f] = __builtin_amdgcn_readfirstlane(used[f]);
    sl = prl_slots<NF>(u, nF);
  }
  if (blockIdx.x >= kSearch) {
    unsigned dw[NF], base = 0;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const unsigned p = f < nF ? (unsigned)wp[min(f, nF - 1)] : 0u, m = f < nF ? (unsigned)wm[min(f, nF - 1)] : 0u;
      dw[f] = p - m;
      base += m;
    }
    int best = INT_MIN, at = 0;
    for (int j = 0; j < seeds; ++j) {
      unsigned sc = base;
#pragma unroll
      for (int f = 0; f < NF; ++f) sc += ar[f] == seed[j * NF + f] ? dw[f] : 0u;
      if ((int)sc > best) best = (int)sc, at = j;
    }
    if (a >= nA) return;
    keys[a] = key_of(best, at * step);
    unsigned h[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) h[f] = f < nF ? (sl.first(f) + slot_of(ar[f], sl.bits(f))) * 16 : 0;
#pragma unroll
    for (int k = 0; k < KP; ++k) slots[(int64_t)a * KP + k] = h[2 * k] | h[2 * k + 1] << 16;
    return;
  }
  if (blockIdx.x == 0 && tid == 0) head->bits = sl.packed;

  float d[NF], sum = 0, least = 0;  // what agreeing adds; the sums of the gains and of the losses
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    d[f] = f < nF ? (float)wp[min(f, nF - 1)] - (float)wm[min(f, nF - 1)] : 0.f;
    sum += fmaxf(d[f], 0.f);
    least += fminf(d[f], 0.f);
  }
  // (scores that may wrap around have no order a sum of weights could follow)
  if (blockIdx.x == 0 && tid == 0) head->stop = !(sum - least < 2147483648.f);
  int q[NF];
  int choice = 192;
  float cost = 0;
  if constexpr (KP <= kSearchKP) {
    // wavefronts that share a choice: with 4096 patterns all four, 77 -> 35 us
    constexpr int SPLIT = P > 1024 ? WAVES : 1, CHOICES = WAVES / SPLIT;
    __shared__ float score[P], often[P], weight[P], bins[BINS], hist[CHOICES][kLevels], best_cost[CHOICES];
    __shared__ int most[CHOICES][kLevels], agree[NF];
    const int mine = wave / SPLIT, first = wave % SPLIT * 64 + lane;
    bins[tid] = 0;
    if (tid < NF) agree[tid] = 0;
    __syncthreads();
    constexpr int SAMPLE = 64;
    int n[NF] = {};
#pragma unroll
    for (int f = 0; f < NF; ++f) ar[f] = (int)slot_of(A[(int64_t)tid * nA / NT * nF + min(f, nF - 1)], sl.bits(f));
    for (int e = tid; e < seeds * NF; e += NT) seed[e] = (int)slot_of(seed[e], sl.bits(e % NF));
    __syncthreads();
    for (int j = 0; j < SAMPLE; ++j) {
      const int* const rb = seed + (j < seeds ? j : 0) * NF;
#pragma unroll
      for (int f = 0; f < NF; ++f) n[f] += ar[f] == rb[f];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
      for (int x = 32; x; x /= 2) n[f] += __shfl_xor(n[f], x);
      if (lane == 0) atomicAdd(&agree[f], n[f]);
    }
    __syncthreads();
    const float range = sum - least;
    const int patterns = 1 << nF;
    for (int p = tid; p < patterns; p += NT) {
      float s = -least, w = 1;
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const float x = (agree[f] + 0.5f) / (NT * SAMPLE + 1);
        if (f < nF) w *= p >> f & 1 ? x : 1 - x, s += p >> f & 1 ? d[f] : 0;
      }
      score[p] = s;
      often[p] = w;
      atomicAdd(&bins[range > 0 ? min(BINS - 1, (int)(s / range * (BINS - 1))) : 0], w);
    }
    __syncthreads();
    for (int x = 1; x < BINS; x *= 2) {
      const float up = tid + x < BINS ? bins[tid + x] : 0;
      __syncthreads();
      bins[tid] += up;
      __syncthreads();
    }
    for (int p = tid; p < patterns; p += NT) {
      const float tail = fmaxf(bins[range > 0 ? min(BINS - 1, (int)(score[p] / range * (BINS - 1))) : 0], 1.f / nB);
      weight[p] = often[p] / (tail * tail);
    }
    if (lane < kLevels) most[mine][lane] = INT_MIN, hist[mine][lane] = 0;
    if (tid < CHOICES) best_cost[tid] = 0;
    __syncthreads();
    choice = blockIdx.x * CHOICES + mine;
    const bool fits = choose<NF>(d, sum, choice, q);
    if (fits)
      for (int p = first; p < patterns; p += 64 * SPLIT) {
        int u = 0;
#pragma unroll
        for (int f = 0; f < NF; ++f) u += p >> f & 1 ? q[f] : 0;
        atomicMax(&most[mine][u], __float_as_int(score[p]));
        atomicAdd(&hist[mine][u], often[p]);
      }
    __syncthreads();
    int m = most[mine][lane % kLevels];
    float h = hist[mine][lane % kLevels];
    __syncthreads();
#pragma unroll
    for (int x = 1; x < kLevels; x *= 2) {
      const int below = __shfl_up(m, x, kLevels);
      const float above = __shfl_down(h, x, kLevels);
      if (lane % kLevels >= x) m = max(m, below);
      if (lane % kLevels + x < kLevels) h += above;
    }
    if (lane < kLevels) most[mine][lane] = m, hist[mine][lane] = h;
    __syncthreads();
    for (int p = first; p < patterns; p += 64 * SPLIT) {
      const int s = __float_as_int(score[p]);
      int t = 0;
#pragma unroll
      for (int x = kLevels / 2; x; x /= 2) t += most[mine][t + x - 1] <= s ? x : 0;
      cost += weight[p] * hist[mine][t];
    }
#pragma unroll
    for (int x = 32; x; x /= 2) cost += __shfl_xor(cost, x);
    if (lane == 0) atomicAdd(&best_cost[mine], fits ? cost : __builtin_huge_valf());
    __syncthreads();
    if (tid) return;
    for (int i = 0; i < CHOICES; ++i)
      if (i == 0 || best_cost[i] < cost) cost = best_cost[i], choice = blockIdx.x * CHOICES + i;
  }
  if (tid == 0) {
    choose<NF>(d, sum, choice, q);
    unsigned long long packed = 0;
#pragma unroll
    for (int f = 0; f < NF; ++f) packed |= (unsigned long long)q[f] << (4 * f);
    head->found[blockIdx.x].q = packed;
    head->found[blockIdx.x].cost = cost;
  }
}

// Adds a constant, the same for every lane, to the sums of the records of the maps e: u += e ? q : 0, in planes of four
// words.  There is code for every q, 256 bytes apart, and it is jumped into; sums that are still small have code that
// leaves out the upper planes.  (A switch has the compiler compare its way to the code, and give every case registers of
// its own, with 20 moves to bring them together: 1310 us at 2^16 x 2^18 records of 8 fields, against 1030 then.)
#define MDH_FOUR(op, ...) op(__VA_ARGS__, 0) op(__VA_ARGS__, 1) op(__VA_ARGS__, 2) op(__VA_ARGS__, 3)
#define MDH_V(x, w) "%[" #x #w "]"
// lowest set bit of q, plane i: carry c
#define MDH_FIRST4(i, w) "v_and_b32 " MDH_V(c, w) ", %[s" #i #w "], " MDH_V(e, w) "\nv_xor_b32 %[s" #i #w "], %[s" #i #w "], " MDH_V(e, w) "\n"
#define MDH_FIRST(i) MDH_FOUR(MDH_FIRST4, i)
#define MDH_ONLY4(i, w) "v_xor_b32 %[s" #i #w "], %[s" #i #w "], " MDH_V(e, w) "\n"
#define MDH_ONLY(i) MDH_FOUR(MDH_ONLY4, i) MDH_DONE
// a set bit, and one that is not: carry x in, y out
#define MDH_ONE4(i, x, y, w)                                                                              \
  "v_bitop3_b32 " MDH_V(y, w) ", %[s" #i #w "], " MDH_V(e, w) ", " MDH_V(x, w) " bitop3:0xe8\n" \
  "v_bitop3_b32 %[s" #i #w "], %[s" #i #w "], " MDH_V(e, w) ", " MDH_V(x, w) " bitop3:0x96\n"
#define MDH_ONE(i, x, y) MDH_FOUR(MDH_ONE4, i, x, y)
#define MDH_NIL4(i, x, y, w) "v_and_b32 " MDH_V(y, w) ", %[s" #i #w "], " MDH_V(x, w) "\nv_xor_b32 %[s" #i #w "], %[s" #i #w "], " MDH_V(x, w) "\n"
#define MDH_NIL(i, x, y) MDH_FOUR(MDH_NIL4, i, x, y)
// the top plane, no carry out
#define MDH_LAST1_4(i, x, w) "v_bitop3_b32 %[s" #i #w "], %[s" #i #w "], " MDH_V(e, w) ", " MDH_V(x, w) " bitop3:0x96\n"
#define MDH_LAST1(i, x) MDH_FOUR(MDH_LAST1_4, i, x) MDH_DONE
#define MDH_LAST0_4(i, x, w) "v_xor_b32 %[s" #i #w "], %[s" #i #w "], " MDH_V(x, w) "\n"
#define MDH_LAST0(i, x) MDH_FOUR(MDH_LAST0_4, i, x) MDH_DONE
#define MDH_DONE "s_branch .Lmdh_end%=\n.p2align 8\n"

// place of the code for q where the sums before it are at most `before`
__device__ __forceinline__ unsigned adder(int q, int before) {
  return before + q < 8 ? q : before + q < 16 ? 8 + q : 24 + q;
}

__device__ __forceinline__ void add_q(u4 (&s)[kPlanes], u4 e, unsigned place) {
  static_assert(kPlanes == 5, "the code is for five planes");
  unsigned c0, c1, c2, c3, d0, d1, d2, d3, at;
  unsigned s00 = s[0][0], s01 = s[0][1], s02 = s[0][2], s03 = s[0][3], s10 = s[1][0], s11 = s[1][1], s12 = s[1][2],
           s13 = s[1][3], s20 = s[2][0], s21 = s[2][1], s22 = s[2][2], s23 = s[2][3], s30 = s[3][0], s31 = s[3][1],
           s32 = s[3][2], s33 = s[3][3], s40 = s[4][0], s41 = s[4][1], s42 = s[4][2], s43 = s[4][3];
  asm("s_getpc_b64 s[30:31]\n"
      ".Lmdh_here%=:\n"
      "s_lshl_b32 %[at], %[place], 8\n"
      "s_add_u32 %[at], %[at], .Lmdh_code%=-.Lmdh_here%=\n"
      "s_add_u32 s30, s30, %[at]\n"
      "s_addc_u32 s31, s31, 0\n"
      "s_setpc_b64 s[30:31]\n"
      ".p2align 8\n"
      ".Lmdh_code%=:\n"
      // sums up to 7: planes 0 to 2
      MDH_DONE
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_LAST0(2, d)
      MDH_FIRST(1) MDH_LAST0(2, c)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_LAST0(2, d)
      MDH_ONLY(2)
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_LAST1(2, d)
      MDH_FIRST(1) MDH_LAST1(2, c)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_LAST1(2, d)
      // up to 15: planes 0 to 3
      MDH_DONE
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_NIL(2, d, c) MDH_LAST0(3, c)
      MDH_FIRST(1) MDH_NIL(2, c, d) MDH_LAST0(3, d)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_NIL(2, d, c) MDH_LAST0(3, c)
      MDH_FIRST(2) MDH_LAST0(3, c)
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_ONE(2, d, c) MDH_LAST0(3, c)
      MDH_FIRST(1) MDH_ONE(2, c, d) MDH_LAST0(3, d)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_ONE(2, d, c) MDH_LAST0(3, c)
      MDH_ONLY(3)
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_NIL(2, d, c) MDH_LAST1(3, c)
      MDH_FIRST(1) MDH_NIL(2, c, d) MDH_LAST1(3, d)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_NIL(2, d, c) MDH_LAST1(3, c)
      MDH_FIRST(2) MDH_LAST1(3, c)
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_ONE(2, d, c) MDH_LAST1(3, c)
      MDH_FIRST(1) MDH_ONE(2, c, d) MDH_LAST1(3, d)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_ONE(2, d, c) MDH_LAST1(3, c)
      // up to 31: all planes
      MDH_DONE
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_NIL(2, d, c) MDH_NIL(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(1) MDH_NIL(2, c, d) MDH_NIL(3, d, c) MDH_LAST0(4, c)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_NIL(2, d, c) MDH_NIL(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(2) MDH_NIL(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_ONE(2, d, c) MDH_NIL(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(1) MDH_ONE(2, c, d) MDH_NIL(3, d, c) MDH_LAST0(4, c)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_ONE(2, d, c) MDH_NIL(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(3) MDH_LAST0(4, c)
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_NIL(2, d, c) MDH_ONE(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(1) MDH_NIL(2, c, d) MDH_ONE(3, d, c) MDH_LAST0(4, c)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_NIL(2, d, c) MDH_ONE(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(2) MDH_ONE(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(0) MDH_NIL(1, c, d) MDH_ONE(2, d, c) MDH_ONE(3, c, d) MDH_LAST0(4, d)
      MDH_FIRST(1) MDH_ONE(2, c, d) MDH_ONE(3, d, c) MDH_LAST0(4, c)
      MDH_FIRST(0) MDH_ONE(1, c, d) MDH_ONE(2, d, c) MDH_ONE(3, c, d) MDH_LAST0(4, d)
      ".Lmdh_end%=:\n"
      : [s00] "+v"(s00), [s01] "+v"(s01), [s02] "+v"(s02), [s03] "+v"(s03), [s10] "+v"(s10), [s11] "+v"(s11),
        [s12] "+v"(s12), [s13] "+v"(s13), [s20] "+v"(s20), [s21] "+v"(s21), [s22] "+v"(s22), [s23] "+v"(s23),
        [s30] "+v"(s30), [s31] "+v"(s31), [s32] "+v"(s32), [s33] "+v"(s33), [s40] "+v"(s40), [s41] "+v"(s41),
        [s42] "+v"(s42), [s43] "+v"(s43), [c0] "=&v"(c0), [c1] "=&v"(c1), [c2] "=&v"(c2), [c3] "=&v"(c3),
        [d0] "=&v"(d0), [d1] "=&v"(d1), [d2] "=&v"(d2), [d3] "=&v"(d3), [at] "=&s"(at)
      : [e0] "v"(e[0]), [e1] "v"(e[1]), [e2] "v"(e[2]), [e3] "v"(e[3]), [place] "s"(place)
      : "s30", "s31", "scc");
  s[0] = u4{s00, s01, s02, s03};
  s[1] = u4{s10, s11, s12, s13};
  s[2] = u4{s20, s21, s22, s23};
  s[3] = u4{s30, s31, s32, s33};
  s[4] = u4{s40, s41, s42, s43};
}

// u >= t, for 32 records
__device__ __forceinline__ unsigned at_least(const u4 (&s)[kPlanes], int w, int t) {
  unsigned g = ~0u;
#pragma unroll
  for (int i = 0; i < kPlanes; ++i) g = __builtin_amdgcn_bitop3_b32(s[i][w], (unsigned)__builtin_amdgcn_sbfe(t, i, 1), g, 0xB2);
  return g;
}

template <int KP>
__global__ __launch_bounds__(kNT, 8) void prl_bits_kernel(const int* __restrict__ A, const int* __restrict__ B,
                                                        const int* __restrict__ wp, const int* __restrict__ wm,
                                                        unsigned long long* keys, const unsigned* __restrict__ slots,
                                                        PrlBitsHead* head, int nA, int nB, int nF, int groups, int sets,
                                                        int chunks) {
  constexpr int NF = 2 * KP, ITEMS = (kPrlChunk * NF + kNT - 1) / kNT;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  int* const rec = (int*)(lds + kPrlMaps);  // the chunk's records
  int* const most = rec + kPrlChunk * nF;
  int* const stop = most + kLevels;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // to be scored: record of A in the workgroup's, above the record of B in its part
  unsigned* const queue = (unsigned*)(stop + 4) + wave * kPrlQueue;
  unsigned char* const tl = (unsigned char*)((unsigned*)(stop + 4) + kNT / 64 * kPrlQueue);  // t of every record of A
  const int group = blockIdx.x % groups, part = blockIdx.x / groups;
  const int a0 = group * sets * kNT;
  const int c_all = (int)(((int64_t)nB + kPrlChunk - 1) / kPrlChunk);
  const int c0 = part * chunks, c1 = min(c0 + chunks, c_all);

  for (int i = tid; i < kPrlMaps / 16; i += kNT) ((u4*)lds)[i] = u4{0, 0, 0, 0};
  if (tid < kLevels) most[tid] = INT_MIN;
  if (tid == 0) *stop = __hip_atomic_load(&head->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int i = 0; i < sets; ++i) tl[i * kNT + tid] = 0;
  static_assert(kSearch == 64, "a lane each");
  float cost = head->found[lane].cost;
  unsigned q_low = (unsigned)head->found[lane].q, q_high = (unsigned)(head->found[lane].q >> 32);
#pragma unroll
  for (int i = 32; i; i /= 2) {
    const float other = __shfl_down(cost, i);
    const unsigned low = __shfl_down(q_low, i), high = __shfl_down(q_high, i);
    if (other < cost) cost = other, q_low = low, q_high = high;
  }
  const unsigned long long q_all = (unsigned long long)__builtin_amdgcn_readfirstlane(q_high) << 32 |
                                   (unsigned)__builtin_amdgcn_readfirstlane(q_low);
  // Scores: what disagreeing everywhere makes, and what agreeing in a field adds (wraps around as the definition does).  The
  // weights are read again for every use, registers for them would be missing elsewhere.  An odd number of fields is
  // followed by one that adds nothing, with the last one's values.  (No branch on the number of fields: with one per field
  // every load was waited for by itself, 4096 x 2^16 records whose slots all collide 710 -> 520 us.)
  auto field = [&](int f) { return f < NF - 1 ? f : nF - 1; };
  unsigned none, adds[NF];
  auto weights = [&] {
    int zero;
    asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
    zero = __builtin_amdgcn_readfirstlane(zero);
    none = 0;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const unsigned m = (unsigned)wm[zero + field(f)], keep = f < NF - 1 || nF == NF ? ~0u : 0u;
      adds[f] = ((unsigned)wp[zero + field(f)] - m) & keep;
      none += m & keep;
    }
  };
  // where the adder's code for each field is, a byte a field
  unsigned long long code[2] = {0, 0};
  for (int f = 0, before = 0; f < nF; ++f) {
    const int q = (int)(q_all >> (4 * f)) & 15;
    code[f / 8] |= (unsigned long long)adder(q, before) << (8 * (f % 8));
    before += q;
  }

  const PrlSlots sl{head->bits};
  // items of a chunk this thread puts into the maps: field and record stay the same from chunk to chunk
  unsigned at[ITEMS], bit[ITEMS], old[ITEMS];
  int width[ITEMS], next[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int e = tid + i * kNT, r = e / nF, f = e - r * nF;
    at[i] = sl.first(f) * 16 + (r >> 5) * 4;
    width[i] = sl.bits(f);
    bit[i] = 1u << (r & 31);
    old[i] = ~0u;
    next[i] = 0;
  }
  auto holds = [&](int c, int i) {
    const int e = tid + i * kNT;
    return e < kPrlChunk * nF && c < c1 && (int64_t)c * kPrlChunk * nF + e < (int64_t)nB * nF;
  };
  auto fetch = [&](int c) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (holds(c, i)) next[i] = B[(int64_t)c * kPrlChunk * nF + tid + i * kNT];
  };
  // The sum that a record from `behind` on has to reach, for the best record of `key`: to score more if that comes before
  // it, as much if not (parts of B are walked at the same time, and the first records compared are from all over B).
  auto reach = [&](unsigned long long key, unsigned behind) {
    int s = (int)((unsigned)(key >> 32) ^ 0x80000000u);
    const bool before = ~(unsigned)key < behind;
    if (!before && s == INT_MIN) return 0;
    s -= before ? 0 : 1;
    int t = 0;
#pragma unroll
    for (int d = kLevels / 2; d; d /= 2) t += most[t + d - 1] <= s ? d : 0;
    return t;
  };
  int queued = 0, left;
  // scores the last `n` records of the queue, one a lane
  auto flush = [&](int n, unsigned behind) {
    __builtin_amdgcn_wave_barrier();
    queued -= n;
    left -= 4;
    if (lane < n) {
      const unsigned e = queue[queued + lane];
      const int ai = (int)(e >> kPrlPartBits), b = c0 * kPrlChunk + (int)(e & ((1u << kPrlPartBits) - 1));
      const int* const ra = A + (int64_t)(a0 + ai) * nF;
      const int* const rb = B + (int64_t)b * nF;
      weights();
      unsigned sc = none;
#pragma unroll
      for (int f = 0; f < NF; ++f) sc += ra[field(f)] == rb[field(f)] ? adds[f] : 0u;
      const unsigned long long k = key_of((int)sc, b);
      const int t = reach(k, behind), before = tl[ai];
      // (two lanes with one record of A: either t holds)
      if (t > before) tl[ai] = (unsigned char)t;
      if (t >= before) atomicMax(keys + a0 + ai, k);
    }
    __builtin_amdgcn_wave_barrier();
  };

  fetch(c0);
  __syncthreads();
  if (*stop) return;
  weights();
  for (int p = tid; p < 1 << nF; p += kNT) {
    unsigned s = none;
    int u = 0;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      s += p >> f & 1 ? adds[f] : 0u;
      u += p >> f & 1 ? (int)(q_all >> (4 * f)) & 15 : 0;
    }
    atomicMax(&most[u], (int)s);
  }
  __syncthreads();
  if (tid < kLevels) {
    int v = most[tid];
#pragma unroll
    for (int d = 1; d < kLevels; d *= 2) {
      const int w = __shfl_up(v, d, kLevels);
      if (tid >= d) v = max(v, w);
    }
    most[tid] = v;
  }

  // sets in which this wavefront has records of A
  const int mine = min(sets, max(0, (int)(((int64_t)nA - a0 - wave * 64 + kNT - 1) / kNT)));
  // An iteration that scores takes about 280 cycles of a wavefront's issue, the loop over fields 27 times as much for the
  // records of a step: so many a step that the rest still pays, a sixth of the loop's time for the whole walk on top (the
  // start, at which little is known), and at least one step whose records all have to be scored.
  left = max(160, 4 * mine * (c1 - c0));
  for (int c = c0; c < c1; ++c) {
    // a bit of a map belongs to one thread: taking the last chunk's out and putting this one's in needs no barrier between
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (old[i] != ~0u) atomicXor((unsigned*)(lds + old[i]), bit[i]);
      old[i] = ~0u;
      if (holds(c, i)) {
        old[i] = at[i] + slot_of(next[i], width[i]) * 16;
        atomicOr((unsigned*)(lds + old[i]), bit[i]);
        rec[tid + i * kNT] = next[i];
      }
    }
    fetch(c + 1);
    __syncthreads();
    const int n = c - c0;
    const unsigned behind = (unsigned)c * kPrlChunk + kPrlChunk;
    const bool look = (n & (n - 1)) == 0 || (n & 15) == 0;
    if (look && tid == 0 && __hip_atomic_load(&head->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) *stop = 1;
    if (look)
      for (int set = 0; set < mine; ++set) {
        const int ai = set * kNT + tid;
        const unsigned long long key = __hip_atomic_load(keys + min(a0 + ai, nA - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        tl[ai] = (unsigned char)max((int)tl[ai], reach(key, behind - kPrlChunk));
      }
    for (int set = 0; set < mine; ++set) {
      const int ai = set * kNT + tid, a = min(a0 + ai, nA - 1);
      const bool real = a0 + ai < nA;
      unsigned d[KP];
#pragma unroll
      for (int k = 0; k < KP; ++k) d[k] = slots[(int64_t)a * KP + k];
      u4 s[kPlanes];
#pragma unroll
      for (int i = 0; i < kPlanes; ++i) s[i] = u4{0, 0, 0, 0};
      unsigned long long q = code[0], q_next = code[1];
      u4 e0 = *(const u4*)(lds + (d[0] & 0xffff)), e1 = *(const u4*)(lds + (d[0] >> 16));
#pragma unroll 1
      for (int k = 1; k <= KP; ++k) {
        const unsigned d0 = d[0];
#pragma unroll
        for (int i = 0; i + 1 < KP; ++i) d[i] = d[i + 1];
        d[KP - 1] = d0;
        add_q(s, e0, (unsigned)q & 255);
        e0 = *(const u4*)(lds + (d[0] & 0xffff));  // (the first pair again after the last)
        add_q(s, e1, (unsigned)(q >> 8) & 255);
        e1 = *(const u4*)(lds + (d[0] >> 16));
        q >>= 16;
        if (KP > 4) q |= q_next << 48, q_next >>= 16;
      }
      left += 24;
      int t = tl[ai];
      unsigned g[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        g[w] = at_least(s, w, t);
        const int held = nB - c * kPrlChunk - w * 32;  // records left from here on
        if (held < 32) g[w] &= held > 0 ? (1u << held) - 1 : 0;
        if (!real) g[w] = 0;
      }
      unsigned long long lanes = __builtin_amdgcn_ballot_w64((g[0] | g[1] | g[2] | g[3]) != 0);
      if (!lanes) continue;
      int here = 0;
      const int most_here = __builtin_popcount(g[0]) + __builtin_popcount(g[1]) + __builtin_popcount(g[2]) + __builtin_popcount(g[3]);
      if (__builtin_popcountll(lanes) <= kPrlQueue - 64 && !__builtin_amdgcn_ballot_w64(most_here > 4)) {
        // a few records of a few lanes: put off until there are enough for all lanes
        do {
          const bool some = (g[0] | g[1] | g[2] | g[3]) != 0;
          if (some) {
            const int w = g[0] ? 0 : g[1] ? 1 : g[2] ? 2 : 3;
            const unsigned x = g[0] ? g[0] : g[1] ? g[1] : g[2] ? g[2] : g[3];
            queue[queued + __builtin_amdgcn_mbcnt_hi((unsigned)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)lanes, 0))] =
                (unsigned)ai << kPrlPartBits | (unsigned)(n * kPrlChunk + w * 32 + __builtin_ctz(x));
#pragma unroll
            for (int i = 0; i < 4; ++i) g[i] = i == w ? x & (x - 1) : g[i];
          }
          queued = __builtin_amdgcn_readfirstlane(queued + __builtin_popcountll(lanes));
          if (queued >= 64) flush(64, behind);
          ++here;
          lanes = __builtin_amdgcn_ballot_w64((g[0] | g[1] | g[2] | g[3]) != 0);
        } while (lanes);
      } else {
        // many, as at the start of a part: each lane scores its next one, and leaves out those that no longer reach t
        weights();
        int ar[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) ar[f] = A[(int64_t)a * nF + field(f)];
        unsigned long long key = __hip_atomic_load(keys + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        t = max(t, reach(key, behind - kPrlChunk));
#pragma unroll 1
        for (int w = 0; w < 4; ++w) {
          unsigned todo = g[0] & at_least(s, 0, t);
          while (__builtin_amdgcn_ballot_w64(todo != 0)) {
            if (todo) {
              const int r = w * 32 + __builtin_ctz(todo);
              todo &= todo - 1;
              unsigned sc = none;
#pragma unroll
              for (int f = 0; f < NF; ++f) sc += ar[f] == rec[r * nF + field(f)] ? adds[f] : 0u;
              const unsigned long long k = key_of((int)sc, c * kPrlChunk + r);
              if (k >= key) {  // (the best record itself: those behind it have to score more)
                key = k;
                t = max(t, reach(key, behind));
                todo &= at_least(s, 0, t);
              }
            }
            ++here;
          }
          // the next 32 records move to the front
#pragma unroll
          for (int i = 0; i < kPlanes; ++i) s[i] = u4{s[i][1], s[i][2], s[i][3], s[i][0]};
          g[0] = g[1], g[1] = g[2], g[2] = g[3];
        }
        if (real) {
          atomicMax(keys + a, key);
          tl[ai] = (unsigned char)t;
        }
      }
      left = __builtin_amdgcn_readfirstlane(left - here);
      if (left < 0) {
        // one store a workgroup: 8192 wavefronts that store to one address take 250 us
        if (lane == 0 && !atomicExch(stop, 1)) __hip_atomic_store(&head->stop, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
    if (look && queued) flush(queued, behind);
    __syncthreads();
    if (*stop) return;
  }
  if (queued) flush(queued, (unsigned)min((int64_t)c1 * kPrlChunk, (int64_t)0x7fffffff));
}

// Output: the keys, or, where the loop over fields ran, its parts folded with max_idx.
__global__ __launch_bounds__(256) void prl_bits_finish_kernel(const unsigned long long* __restrict__ keys,
                                                               const PrlBitsHead* __restrict__ head, const int* __restrict__ ws,
                                                               int* __restrict__ out_s, int* __restrict__ out_i, int nA, int S) {
  const int a = blockIdx.x * 256 + threadIdx.x;
  if (a >= nA) return;
  unsigned long long key = 0;
  if (!head->stop) {
    key = keys[a];
  } else {
    for (int s = 0; s < S; ++s) {
      const int score = ws[(int64_t)s * nA + a], i = ws[(int64_t)(S + s) * nA + a];
      const unsigned long long k = key_of(score, i);
      key = k > key ? k : key;
    }
  }
  out_s[a] = (int)((unsigned)(key >> 32) ^ 0x80000000u);
  out_i[a] = (int)~(unsigned)key;
}

struct Layout {
  unsigned long long* keys;
  unsigned* slots;
  PrlBitsHead* head;
};

// (keys and slots lie before the head)
Layout layout(void* ws, int64_t nA, int S) {
  Layout l;
  l.head = prl_bits_head(ws, nA, S);
  l.keys = (unsigned long long*)(((uintptr_t)ws + 7) & ~(uintptr_t)7);
  l.slots = (unsigned*)(l.keys + nA);
  return l;
}

template <int KP>
mdh_status start(const Layout& l, const PrlBitsGrid& g, int64_t nA, int64_t nB, int nF, const int32_t* A, const int32_t* B,
                 const int32_t* wp, const int32_t* wm, hipStream_t st) {
  auto kern = prl_bits_kernel<KP>;
  static int64_t lds_allowed[kMaxDevices] = {};
  const int64_t lds = prl_bits_lds_bytes(nF, g.sets);
  if (allow_dynamic_lds((const void*)kern, lds, lds_allowed) != MDH_OK) return MDH_ERR_LAUNCH;
  clear_stale_error();
  hipLaunchKernelGGL((prl_bits_prep_kernel<KP>), dim3((unsigned)(kSearch + cdiv(nA, kPrepNT))), dim3(kPrepNT), 0,
                     st, A, B, wp, wm, l.keys, l.slots, l.head, (int)nA, (int)nB, nF);
  hipLaunchKernelGGL(kern, dim3((unsigned)(g.groups * g.parts)), dim3(kNT), (size_t)lds, st, A, B, wp, wm, l.keys,
                     (const unsigned*)l.slots, l.head, (int)nA, (int)nB, nF, g.groups, g.sets, g.chunks);
  return launch_status();
}

}  // namespace

const int* prl_bits_gate(void* ws, int64_t nA, int S) { return &layout(ws, nA, S).head->stop; }

mdh_status launch_prl_bits(int S, int64_t nA, int64_t nB, int nF, const int32_t* A, const int32_t* B, const int32_t* wp,
                           const int32_t* wm, void* ws, hipStream_t st) {
  const PrlBitsGrid g = prl_bits_grid(nA, nB, nF);
  const Layout l = layout(ws, nA, S);
  switch ((nF + 1) / 2) {
#define MDH_KP(n) \
  case n: return start<n>(l, g, nA, nB, nF, A, B, wp, wm, st);
    MDH_KP(1) MDH_KP(2) MDH_KP(3) MDH_KP(4) MDH_KP(5) MDH_KP(6) MDH_KP(7) MDH_KP(8)
#undef MDH_KP
  }
  return MDH_ERR_UNSUPPORTED;
}

mdh_status launch_prl_bits_finish(int S, int64_t nA, void* ws, int32_t* score, int32_t* index, hipStream_t st) {
  const Layout l = layout(ws, nA, S);
  clear_stale_error();
  hipLaunchKernelGGL(prl_bits_finish_kernel, dim3((unsigned)cdiv(nA, 256)), dim3(256), 0, st, l.keys, l.head, (const int*)ws,
                     score, index, (int)nA, S - 1);
  return launch_status();
}

}  // namespace mdh
