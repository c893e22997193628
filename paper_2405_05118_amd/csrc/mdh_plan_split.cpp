// Planner rules shared by MatMul and the batched / transposed MatMul for the kernel that carries every fp32 value
// as three bf16 values (mdh_matmul_split.hip; block 32 x 32 x 16): its tiles, the sizes it takes, and when the
// library's default is one of them.
#include "mdh_internal.h"

namespace mdh {
namespace detail {

static const int kSplitMenu[][5] = {  // BM, BN, BK, WM, WN
    {256, 256, 16, 64, 128}, {256, 128, 32, 64, 64}, {128, 128, 32, 32, 64}, {128, 64, 32, 64, 32}, {64, 64, 32, 32, 32}};
constexpr int kSplitLds = 5;
// k over the wavefronts (mdh_matmul_split_k.hip): BM, BN, wavefronts
static const int kSplitKMenu[][3] = {{64, 64, 8}, {64, 64, 4}, {64, 96, 4}, {96, 64, 4}, {96, 96, 4}, {32, 64, 8}, {64, 32, 8}, {32, 32, 8}};

// C stored transposed runs as the product of the transposed operands in the other order: the tile swaps too
bool split_inst(const GemmPlan& g, bool tc) {
  if (g.WK > 1) {
    for (auto& m : kSplitKMenu)
      if ((tc ? g.BN : g.BM) == m[0] && (tc ? g.BM : g.BN) == m[1] && g.WM == g.BM && g.WN == g.BN &&
          g.WK == m[2] && g.BK == 32)
        return true;
    return false;
  }
  for (auto& m : kSplitMenu)
    if ((tc ? g.BN : g.BM) == m[0] && (tc ? g.BM : g.BN) == m[1] && g.BK == m[2] && (tc ? g.WN : g.WM) == m[3] &&
        (tc ? g.WM : g.WN) == m[4])
      return true;
  return false;
}

int64_t split_lds_bytes(const GemmPlan& g) {
  if (g.WK > 1) {  // partial tiles, or a chunk of both operands (the most any view takes), of every wavefront
    const int64_t parts = (int64_t)g.WK * g.BM * (g.BN + 4) * 4, operands = (int64_t)g.WK * (g.BM + g.BN) * 128;
    return (parts > operands ? parts : operands) + 16;
  }
  return 2ll * (g.BM + g.BN) * g.BK * 6 + 16;
}

// The last k-tile is read whole, ending at the last k, so there must be one; operand addresses are a 32-bit offset
// from the tile's first element.
bool split_sizes(int64_t M, int64_t N, int64_t K) {
  return K >= 32 && K <= (1 << 20) && M <= (1 << 24) && N <= (1 << 24);
}

// Does the table's kernel take these sizes?  With k over the wavefronts a tile that would stick out is moved inside, and a
// part of k holds two steps of 16, so that the last wavefront's can start early.
bool split_fits(int64_t M, int64_t N, int64_t K, const GemmPlan& g) {
  if (!split_sizes(M, N, K)) return false;
  if (g.WK == 1) return true;
  return M >= g.BM && N >= g.BN && (g.S == 1 || K - (g.S - 1) * split_part(K, g) >= 32);
}

int split_tiles(bool tc, GemmPlan* out) {
  int n = 0;
  for (auto& m : kSplitMenu) {
    GemmPlan g{m[0], m[1], m[2], m[3], m[4], 1, 0};
    if (tc) g = GemmPlan{m[1], m[0], m[2], m[4], m[3], 1, 0};
    g.split = 1;
    out[n++] = g;
  }
  for (auto& m : kSplitKMenu) {
    GemmPlan g{m[0], m[1], 32, m[0], m[1], 1, 0};
    if (tc) g = GemmPlan{m[1], m[0], 32, m[1], m[0], 1, 0};
    g.split = 1;
    g.WK = m[2];
    out[n++] = g;
  }
  return n;
}

// Microseconds of 32 k for the workgroups a compute unit holds at once (index: how many, less one); with all compute units
// at work on a large tile the clock gives way, which `full` adds.  Fitted to 570 random products of 2^26 to 7e10
// multiply-adds, 128 to 4096 k, every tile on every one of them: off by 5 % rms with k over the wavefronts, 7 to 10 % with
// the others, and the tile it picks takes 1.2 % longer on average than the fastest (at most 25 %).
struct StepTime {
  double us[3], full;
  int held;
  double first, once;  // what the first, not overlapped loads and the output take in steps; microseconds besides
};
static const StepTime kStep[kSplitTiles] = {
    {{2.96}, 1.12, 1, 4.6, 4.8},  // (256 columns and more: 4 % added, their fit is the poorest)
    {{1.69}, 0.50, 1, 5.8, 3.2},
    {{0.934}, 0.31, 1, 5.1, 3.8},
    {{0.833, 1.300}, 0.117, 2, 3.6, 3.5},
    {{0.575, 0.829, 1.243}, 0.032, 3, 2.8, 3.5},
    {{0.291}, 0.084, 1, 13.6, 2.1},  // k over the wavefronts
    {{0.366, 0.597}, 0.086, 2, 6.7, 2.8},
    {{0.489}, 0.073, 1, 10.1, 2.1},
    {{0.507}, 0.054, 1, 9.6, 2.0},
    {{0.675}, 0.081, 1, 10.1, 2.0},
    {{0.205}, 0.044, 1, 14.8, 2.0},  // (4 % below their times since they take eight products, and left so: the tiles they
    {{0.212}, 0.040, 1, 15.0, 2.0},  // would give way to are further from 64 bits)
    {{0.125, 0.243}, 0.048, 2, 9.3, 3.1}};

// A coarser estimate of the tiles in LDS, which leans towards more parts of k: it has the least number of them.
static const StepTime kStepParts[] = {
    {{3.5}, 0.9, 1, 3, 0}, {{1.95}, 0.45, 1, 3, 0}, {{1.1}, 0.2, 1, 3, 0}, {{0.98, 1.56}, 0, 2, 2, 0}, {{0.57, 0.95, 1.30}, 0, 3, 1, 0}};

static double estimate(const StepTime& t, int64_t tiles, int64_t M, int64_t N, int64_t batch, int64_t K, int S) {
  const int64_t slots = 256 * t.held, work = tiles * S, rest = work % slots;
  const double fill = t.full * (work < 256 ? (double)work / 256 : 1.0);
  double round = (double)(work / slots) * (t.us[t.held - 1] + fill);
  if (rest) round += t.us[cdiv(rest, 256) - 1] + t.full * (double)(rest < 256 ? rest : 256) / 256;
  const double steps = (double)K / (32.0 * S) + t.first;
  return t.once + round * steps + (S > 1 ? 2.0 + (double)(S + 1) * batch * M * N * 4e-6 / 4.0 : 0.0);
}

// The tiles that a search over candidates tries: with k over the wavefronts those whose time is estimated within a quarter
// of the fastest one's.
int split_offered(int64_t batch, int64_t M, int64_t N, int64_t K, bool tc, GemmPlan* out) {
  GemmPlan sp[kSplitTiles];
  double us[kSplitTiles], best = 1e30;
  const int n = split_tiles(tc, sp);
  for (int i = 0; i < n; ++i) {
    us[i] = split_fits(M, N, K, sp[i]) ? estimate(kStep[i], batch * cdiv(M, sp[i].BM) * cdiv(N, sp[i].BN), M, N, batch, K, 1) : 1e30;
    if (us[i] < best) best = us[i];
  }
  int m = 0;
  for (int i = 0; i < n; ++i)
    if (sp[i].WK == 1 || us[i] < 1.25 * best) out[m++] = sp[i];
  return m;
}

// the fastest of the tiles from `first` to before `last` by the estimate `step`, in `least` to S parts of k; < 0: none takes
// these sizes
static double best_tile(const StepTime* step, int first, int last, int64_t batch, int64_t M, int64_t N, int64_t K, bool tc, int least,
                        int S, GemmPlan* g) {
  GemmPlan sp[kSplitTiles];
  split_tiles(tc, sp);
  double best = -1;
  for (int i = first; i < last; ++i)
    for (int s = least; s <= S; s *= 2) {
      sp[i].S = s;
      if ((s - 1) * split_part(K, sp[i]) >= K) break;  // a part without k
      if (!split_fits(M, N, K, sp[i])) continue;
      const int64_t k = step == kStepParts ? cdiv(K, 32 * s) * 32 * s : K;  // (the coarser one counts whole steps)
      const double t = estimate(step[i], batch * cdiv(M, sp[i].BM) * cdiv(N, sp[i].BN), M, N, batch, k, s);
      if (best < 0 || t < best) {
        best = t;
        *g = sp[i];
      }
    }
  return best;
}

// Is the default one of these tiles, and which?  `S` is the number of parts the fp32 rule splits k into: not more
// parts here, so that no call needs more workspace than it does there.
// Against the fp32 kernels, us: 4096^3 566 / 1003; 3000^3 364 / 504; 2048^3 93 / 150; 1021 x 1531 x 777 21.0 / 40.4;
// 65536 x 64 x 4096 258 / 312; 16 x 1024^3 157 / 253; 8 x 200 x 333 x 650 14.6 / 24.4; 1024^3 17.4 / 24.4.  The line:
// below 128 k the first and last tile are most of the walk (4096 x 4096 x 64: 27.9 / 27.0; 16 x 512 x 512 x 64: 10.7
// / 10.5), below 2^26 products a call is its launch (16 x 128^3: 8.1 / 7.8), and less than 48 rows or columns
// leave most of a tile of 64 empty (8192 x 32 x 256: 9.6 / 9.0).  Over 1600 random sizes the split is 5-12 % ahead on
// average from 128 to 224 k and 15-30 % beyond, whatever the number of tiles; 3-4 % of them are 4-25 % behind (167 x 113
// x 1521 x 142, A and B transposed: 155 / 126), with nothing in their sizes to tell them by.
bool split_default(int64_t batch, int64_t M, int64_t N, int64_t K, bool tc, int S, GemmPlan* g) {
  if (!split_sizes(M, N, K) || K < 128 || M < 48 || N < 48 || batch < 1) return false;
  if ((double)batch * M * N * K < (double)(1 << 26)) return false;
  if (best_tile(kStep, 0, kSplitTiles, batch, M, N, K, tc, 1, S, g) < 0) return false;
  // A part is one chain in an accumulator, and twice as long a chain is 1.4 times as far from 64 bits: not fewer parts than
  // the coarser estimate has, though the other one would take fewer for 1 % of tall and narrow outputs and be up to a fifth
  // faster there (us and error in 2^-24, those / these: 25978 x 49 x 1755 56 and 10.7 / 56 and 7.5, 23917 x 54 x 692 24.4 and
  // 6.6 / 28.4 and 4.6, 1844 x 53 x 10969 32.4 and 7.0 / 39.6 and 5.1).  With k over the wavefronts a chain is a quarter or
  // an eighth as long anyway.
  GemmPlan p;
  if (g->WK == 1 && S > 1 && best_tile(kStepParts, 0, kSplitLds, batch, M, N, K, tc, 1, S, &p) >= 0 && p.S > g->S)
    best_tile(kStep, 0, kSplitTiles, batch, M, N, K, tc, p.S, S, g);
  return true;
}

// Small products, which the fp32 rule gives to 64 x 64 tiles in k-tiles of 16 (plan `f`, S parts of k): the same tiles of one
// or two blocks instead (with eight products: see mdh_matmul_split_k.hip for their errors), in one launch, where they are
// estimated at 0.85 of that kernel's time or less -- a line fitted to 230 random batches of 2^19 to 2^26 multiply-adds, off by
// 7 % rms.  Four fifths go there; 170 of them take 0.62 of the time on average, none is slower.  us, replayed from a graph: 2 x
// 68 x 149 x 353, A and B transposed, 11.7 / 5.8; 13 x 108 x 66 x 237 12.9 / 5.2; 4 x 203 x 171 x 183 11.1 / 5.2.
bool split_small_default(int64_t batch, int64_t M, int64_t N, int64_t K, bool tc, const GemmPlan& f, GemmPlan* g) {
  if (f.BM != 64 || f.BN != 64 || f.BK != 16 || batch < 1 || K < 64 || (double)batch * M * N * K > (double)(1 << 26)) return false;
  const double wg = (double)batch * cdiv(M, 64) * cdiv(N, 64) * f.S / 512;
  const double fp32 = 4.15 + (wg > 1 ? wg : 1) * (double)K / f.S * 0.033 + (f.S > 1 ? 1.76 + 0.12 * f.S : 0.0);
  GemmPlan b;
  const double t = best_tile(kStep, kSplitTiles - 3, kSplitTiles, batch, M, N, K, tc, 1, 1, &b);
  if (t < 0 || t > 0.85 * fp32) return false;
  *g = b;
  return true;
}

// Outputs of few tiles, which the fp32 rule gives to its own kernel with k over the wavefronts (plan `f`, small tiles,
// S parts of k): the ones of 32 x 32 to 64 x 32 with a sum of their own for h h' instead, where they are clearly faster.
// They are no further from 64 bits than that kernel, on sums of few terms either (256 x 256 x 2048, relative 2-norm in units
// of 2^-24, fp32 / slices: 1 term 0.42 / 0.42, 2 0.61 / 0.60, 4 0.76 / 0.74, 16 1.06 / 0.98, 64 1.3 / 1.06, 2048 4.9 / 1.8).
// The fp32 kernel's time is a fit that is off by up to 40 %, so theirs has to be below three quarters of it: of 97 random
// sizes 36 go there, and 110 that do take 0.61 of the time on average, none more (four fifths: 195 x 292 x 7618 34.1 -> 40.0;
// nine tenths: 128 x 512 x 4032 16.1 -> 20.6).  us, replayed from a graph: 288 x 320 x 2880 36.4 / 17.9; stays: 512^3 6.0 / 7.0.
bool split_k_default(int64_t M, int64_t N, int64_t K, const GemmPlan& f, GemmPlan* g) {
  if (!split_sizes(M, N, K) || K < 128 || (double)M * N * K < (double)(1 << 26)) return false;
  const bool b16 = f.BM == 16, whole = M % f.BM == 0 && N % f.BN == 0 && K % 16 == 0;
  const double per[2][2][3] = {{{2.9, 0.0243, 0.0382}, {2.4, 0.0273, 0.0247}}, {{2.0, 0.0037, 0.0232}, {0.6, 0.0212, 0.0135}}};
  const double *c = per[b16][whole], wg = (double)cdiv(M, f.BM) * cdiv(N, f.BN) * f.S;
  const double fp32 = c[0] + (double)K / (f.WK * f.S) * (c[1] + c[2] * wg * f.WK / 1024) + (f.S > 1 ? 3.0 : 0.0);
  GemmPlan b;
  const double t = best_tile(kStep, kSplitTiles - 3, kSplitTiles, 1, M, N, K, false, 1, f.S, &b);
  if (t < 0 || t > 0.76 * fp32) return false;
  *g = b;
  return true;
}

}  // namespace detail
}  // namespace mdh
