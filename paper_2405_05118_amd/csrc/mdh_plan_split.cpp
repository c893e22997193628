// Planner rules shared by MatMul and the batched / transposed MatMul for the kernel that carries every fp32 value
// as three bf16 values (mdh_matmul_split.hip; block 32 x 32 x 16): its tiles, the sizes it takes, and when the
// library's default is one of them.
#include "mdh_internal.h"

namespace mdh {
namespace detail {

static const int kSplitMenu[][5] = {  // BM, BN, BK, WM, WN
    {256, 256, 16, 64, 128}, {256, 128, 32, 64, 64}, {128, 128, 32, 32, 64}, {128, 64, 32, 64, 32}, {64, 64, 32, 32, 32}};

// C stored transposed runs as the product of the transposed operands in the other order: the tile swaps too
bool split_inst(const GemmPlan& g, bool tc) {
  for (auto& m : kSplitMenu)
    if ((tc ? g.BN : g.BM) == m[0] && (tc ? g.BM : g.BN) == m[1] && g.BK == m[2] && (tc ? g.WN : g.WM) == m[3] &&
        (tc ? g.WM : g.WN) == m[4])
      return true;
  return false;
}

int64_t split_lds_bytes(const GemmPlan& g) { return 2ll * (g.BM + g.BN) * g.BK * 6 + 16; }

// The last k-tile is read whole, ending at the last k, so there must be one; operand addresses are a 32-bit offset
// from the tile's first element.
bool split_sizes(int64_t M, int64_t N, int64_t K) {
  return K >= 32 && K <= (1 << 20) && M <= (1 << 24) && N <= (1 << 24);
}

int split_tiles(bool tc, GemmPlan* out) {
  int n = 0;
  for (auto& m : kSplitMenu) {
    GemmPlan g{m[0], m[1], m[2], m[3], m[4], 1, 0};
    if (tc) g = GemmPlan{m[1], m[0], m[2], m[4], m[3], 1, 0};
    g.split = 1;
    out[n++] = g;
  }
  return n;
}

// Microseconds of 32 k for the workgroups a compute unit holds at once (index: how many, less one).  Measured on
// K = 300 ... 4096; with all compute units at work on a large tile the clock gives way, which the second figure adds.
struct StepTime {
  double us[3], full;
  int held, first;  // first: what the first, not overlapped k-tile and the output take, in steps
};
static const StepTime kStep[kSplitTiles] = {
    {{3.5}, 0.9, 1, 3}, {{1.95}, 0.45, 1, 3}, {{1.1}, 0.2, 1, 3}, {{0.98, 1.56}, 0, 2, 2}, {{0.57, 0.95, 1.30}, 0, 3, 1}};

static double estimate(int i, int64_t tiles, int64_t M, int64_t N, int64_t batch, int64_t K, int S) {
  const StepTime& t = kStep[i];
  const int64_t slots = 256 * t.held, work = tiles * S, rest = work % slots;
  const double fill = t.full * (work < 256 ? (double)work / 256 : 1.0);
  double round = (double)(work / slots) * (t.us[t.held - 1] + fill);
  if (rest) round += t.us[cdiv(rest, 256) - 1] + t.full * (double)(rest < 256 ? rest : 256) / 256;
  const double steps = (double)cdiv(K, 32 * S) + t.first;
  return round * steps + (S > 1 ? 2.0 + (double)(S + 1) * batch * M * N * 4e-6 / 4.0 : 0.0);
}

// Is the default one of these tiles, and which?  `S` is the number of parts the fp32 rule splits k into: not more
// parts here, so that no call needs more workspace than it does there.
// Against the fp32 kernels, us: 4096^3 566 / 1003; 3000^3 364 / 504; 2048^3 93 / 150; 1021 x 1531 x 777 28.5 / 40.4;
// 65536 x 64 x 4096 258 / 312; 16 x 1024^3 157 / 253; 8 x 200 x 333 x 650 16.7 / 24.4; 1024^3 23.8 / 24.4.  The line:
// below 128 k the first and last tile are most of the walk (4096 x 4096 x 64: 27.9 / 27.0; 16 x 512 x 512 x 64: 10.7
// / 10.5), below 2^26 products a call is its launch (16 x 128^3: 8.1 / 7.8), and less than 48 rows or columns
// leave most of a tile of 64 empty (8192 x 32 x 256: 9.6 / 9.0).  Over 1600 random sizes the split is 5-12 % ahead on
// average from 128 to 224 k and 15-30 % beyond, whatever the number of tiles; 3-4 % of them are 4-25 % behind (167 x 113
// x 1521 x 142, A and B transposed: 155 / 126), with nothing in their sizes to tell them by.
bool split_default(int64_t batch, int64_t M, int64_t N, int64_t K, bool tc, int S, GemmPlan* g) {
  if (!split_sizes(M, N, K) || K < 128 || M < 48 || N < 48 || batch < 1) return false;
  if ((double)batch * M * N * K < (double)(1 << 26)) return false;
  GemmPlan sp[kSplitTiles];
  const int n = split_tiles(tc, sp);
  double best = -1;
  for (int i = 0; i < n; ++i)
    for (int s = 1; s <= S; s *= 2) {
      sp[i].S = s;
      if ((s - 1) * split_part(K, sp[i]) >= K) break;  // a part without k
      const double t = estimate(i, batch * cdiv(M, sp[i].BM) * cdiv(N, sp[i].BN), M, N, batch, K, s);
      if (best < 0 || t < best) {
        best = t;
        *g = sp[i];
      }
    }
  return true;
}

}  // namespace detail
}  // namespace mdh
