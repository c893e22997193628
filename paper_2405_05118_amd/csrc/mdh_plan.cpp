// Host-side de-composition planner: turns a configuration of the paper's tuning
// parameters (Table "Tuning parameters of our low-level expressions") into a launch
// descriptor of one of the library's kernel instantiations and back, and checks the
// algorithmic constraint of parameter 0 (prod_l #PRT(l,d) = N_d) and the model
// constraints (lanes per workgroup, LDS budget; Appendix "Constraints of Programming
// Models").  Integer arithmetic only; no GPU call in this file.
#include <string.h>

#include "mdh_internal.h"

namespace mdh {

namespace {
constexpr int kMaxLanesPerWG = 1024;        // model constraint 0 of the CUDA/OpenCL tables
constexpr int64_t kLdsBytesPerWG = 160 * 1024;  // gfx950 LDS per workgroup
}  // namespace

namespace detail {

void clear_params(mdh_tile_params* p, int D) {
  memset(p, 0, sizeof(*p));
  p->D = D;
  for (int l = 0; l < MDH_NUM_LAYERS; ++l)
    for (int d = 0; d < MDH_MAX_D; ++d) p->prt[l][d] = 1;
  for (int d = 0; d < MDH_MAX_D; ++d) p->blk[d] = 1;
}

// Fused loop order D1=S1=R1: workgroup parts outermost (one workgroup = one iteration of
// them), then the sequential HBM-layer parts, then wavefront and lane parts (parallel
// inside the workgroup), then the LDS- and VGPR-layer sequential parts; within a layer,
// dimensions in the given order.
void set_order(mdh_tile_params* p, const int* dim_order) {
  static const int layer_order[MDH_NUM_LAYERS] = {MDH_L_WG,   MDH_L_HBM, MDH_L_WAVE,
                                                  MDH_L_LANE, MDH_L_LDS, MDH_L_VGPR};
  int n = 0;
  for (int li = 0; li < MDH_NUM_LAYERS; ++li)
    for (int di = 0; di < p->D; ++di)
      p->order[n++] = (uint8_t)(layer_order[li] * MDH_MAX_D + dim_order[di]);
}

int64_t extent(const mdh_tile_params* p, int d) {
  int64_t e = p->blk[d];
  for (int l = 0; l < MDH_NUM_LAYERS; ++l) e *= p->prt[l][d];
  return e;
}

// Algorithmic constraint of parameter 0 (with the predicated-tail extension).
mdh_status check_products(const mdh_tile_params* p, const int64_t* sizes, bool* ragged) {
  *ragged = false;
  for (int d = 0; d < p->D; ++d) {
    if (p->blk[d] < 1) return MDH_ERR_TILE_NOT_DIVIDING;
    for (int l = 0; l < MDH_NUM_LAYERS; ++l)
      if (p->prt[l][d] < 1) return MDH_ERR_TILE_NOT_DIVIDING;
    const int64_t e = extent(p, d);
    if (e == sizes[d]) continue;
    if (!p->ragged || e < sizes[d]) return MDH_ERR_TILE_NOT_DIVIDING;
    *ragged = true;
  }
  return MDH_OK;
}

mdh_status check_lanes(const mdh_tile_params* p) {
  int64_t lanes = 1;
  for (int d = 0; d < p->D; ++d) lanes *= (int64_t)p->prt[MDH_L_WAVE][d] * p->prt[MDH_L_LANE][d];
  return lanes > kMaxLanesPerWG ? MDH_ERR_TILE_RESOURCES : MDH_OK;
}

// A configuration is supported iff regenerating the table from the derived launch
// descriptor reproduces it (apart from the ragged flag).
bool same_table(const mdh_tile_params& a, const mdh_tile_params& b) {
  mdh_tile_params x = a, y = b;
  x.ragged = y.ragged = 0;
  memset(x.reserved, 0, sizeof(x.reserved));
  memset(y.reserved, 0, sizeof(y.reserved));
  return memcmp(&x, &y, sizeof(x)) == 0;
}

}  // namespace detail
using namespace detail;

// =============================================================================== stencil

static bool stencil_inst(int RJ, int TY, int LK) {
  static const int menu[][3] = {{4, 2, 128}, {2, 2, 128}, {8, 2, 128}, {4, 4, 128}, {2, 4, 128},
                                {4, 1, 128}, {8, 1, 128}, {4, 4, 64},  {2, 4, 64},  {4, 2, 64},
                                {4, 8, 32},  {4, 16, 16}};
  for (auto& m : menu)
    if (m[0] == RJ && m[1] == TY && m[2] == LK) return true;
  return false;
}

// the kernel without LDS: rows and planes a lane holds, workgroups of 256 lanes
static const int kStencilDirect[][2] = {{2, 2}, {2, 4}, {4, 2}, {4, 4}, {1, 2}, {2, 1}};

static bool stencil_direct_inst(const StencilPlan& pl) {
  if ((pl.LK != 16 && pl.LK != 32 && pl.LK != 64) || pl.TY != 256 / pl.LK) return false;
  for (auto& m : kStencilDirect)
    if (m[0] == pl.RJ && m[1] == pl.PI) return true;
  return false;
}

int64_t stencil_lds_bytes(int RJ, int TY, int LK) {
  return 2ll * (TY * RJ + 2) * (LK * 4 + 8) * 4;
}

void params_from_plan(const int64_t* sizes, const StencilPlan& pl, mdh_tile_params* p) {
  clear_params(p, 3);
  const int TJ = pl.TY * pl.RJ, KT = pl.LK * 4;
  p->prt[MDH_L_WG][0] = (int32_t)cdiv(sizes[0], pl.SI);
  p->prt[MDH_L_WG][1] = (int32_t)cdiv(sizes[1], TJ);
  p->prt[MDH_L_WG][2] = (int32_t)cdiv(sizes[2], KT);
  p->prt[pl.PI ? MDH_L_VGPR : MDH_L_HBM][0] = pl.SI;
  if (pl.LK >= 64) {
    p->prt[MDH_L_WAVE][1] = pl.TY;
    p->prt[MDH_L_WAVE][2] = pl.LK / 64;
    p->prt[MDH_L_LANE][2] = 64;
  } else {  // narrow grids: a wavefront is 64/LK lane-rows of LK lanes
    p->prt[MDH_L_WAVE][1] = pl.TY * pl.LK / 64;
    p->prt[MDH_L_LANE][1] = 64 / pl.LK;
    p->prt[MDH_L_LANE][2] = pl.LK;
  }
  p->prt[MDH_L_VGPR][1] = pl.RJ;
  p->prt[MDH_L_VGPR][2] = 4;
  static const int dims[3] = {0, 1, 2};
  set_order(p, dims);
  p->strided = 0;
  p->lane_fast_dim = 2;            // k is contiguous in both buffers
  p->in_region[0] = pl.PI ? MDH_MR_VGPR : MDH_MR_LDS;  // a lane's planes and rows at once; current plane staged in LDS
  p->out_region = MDH_MR_VGPR;     // results leave from registers
  p->ragged = (uint8_t)pl.ragged;
}

static StencilPlan stencil_direct(const int64_t* s, int RJ, int PI) {
  StencilPlan pl{RJ, 0, s[2] <= 64 ? 16 : s[2] <= 128 ? 32 : 64, PI, 0, PI};
  pl.TY = 256 / pl.LK;
  pl.ragged = (s[0] % PI) || (s[1] % (pl.TY * RJ)) || (s[2] % (pl.LK * 4));
  return pl;
}

// A launch has less than 2^32 lanes, which grids of few points a plane reach first (nx = 2^26, ny = nz = 1: 2^24 workgroups of
// 256); the marching kernel's workgroups take up to 64 planes.
static bool stencil_direct_fits(const int64_t* s, const StencilPlan& pl) {
  return cdiv(s[0], pl.PI) * cdiv(s[1], (int64_t)pl.TY * pl.RJ) * cdiv(s[2], (int64_t)pl.LK * 4) < (1 << 24);
}

static StencilPlan stencil_march(const int64_t* s) {
  StencilPlan pl;
  pl.RJ = 4;
  pl.TY = 4;
  pl.LK = s[2] <= 256 ? 64 : 128;
  // narrow grids: fewer lanes along k, more lane-rows along j, so that no lane idles beyond nz
  // (512 x 512 x 64: 0.189 ms with 64 lanes along k against 0.069 ms for the best of those tiles)
  if (s[2] <= 128) pl.LK = 32, pl.TY = 8;
  if (s[2] <= 64) pl.LK = 16, pl.TY = 16;
  pl.SI = 64;
  // Tiles of 512 columns only where they fit nz (within 10 %); otherwise 256 columns, two rows per
  // lane and at most 32 planes per workgroup -- more and smaller workgroups, whose partly filled last
  // tile costs little.  Measured: 384^3 0.234 -> 0.111 ms; 256 x 256 x 320 0.069 -> 0.043 ms; 640^3
  // 0.563 -> 0.486 ms; 1024 x 256 x 256 0.107 -> 0.095 ms; 256^3 0.0299 -> 0.0285 ms.
  if (s[2] > 128 && (s[2] <= 256 || cdiv(s[2], 512) * 512 * 10 > s[2] * 11)) {
    pl.RJ = 2;
    pl.TY = 4;
    pl.LK = 64;
    pl.SI = 32;
  }
  const int TJ = pl.TY * pl.RJ, KT = pl.LK * 4;
  // keep at least one workgroup per compute unit when the grid is small (the four-wavefront
  // workgroups of the variant above: four per compute unit, down to 16 planes each)
  if (pl.RJ == 2)
    while (pl.SI > 16 && cdiv(s[0], pl.SI) * cdiv(s[1], TJ) * cdiv(s[2], KT) < 1024) pl.SI /= 2;
  while (pl.SI > 4 && cdiv(s[0], pl.SI) * cdiv(s[1], TJ) * cdiv(s[2], KT) < 256) pl.SI /= 2;
  if (s[0] > 0 && pl.SI > s[0]) pl.SI = (int)s[0];
  pl.ragged = (s[0] % pl.SI) || (s[1] % TJ) || (s[2] % KT);
  return pl;
}

// Which kernel, and how much a lane of the one without LDS holds.  us, that one / the marching one: 86 x 72 x 69 5.0 / 15.1
// (of which 5 is the host's launch), 154 x 191 x 65 5.8 / 15.7, 226 x 214 x 89 9.3 / 20.1, 143 x 70 x 501 9.8 / 24.7, 256^3
// 21.0 / 28.1, 300^3 41 / 81, 400^3 78 / 158, 640^3 411 / 507; over 80 random grids of 64 to 512 a side 2.4 times as fast.
// Rows x planes a lane: 2 x 2 has the most wavefronts (143 x 70 x 501 9.8; 2 x 4 9.7, 4 x 4 12.1), 4 x 4 reads the least twice
// (500^3 211; 2 x 4 234, 2 x 2 272), 2 x 4 is between (168 x 307 x 146 14.4, 13.8 and 16.6; 300^3 43.0, 47.4 and 42.3).
// The marching kernel stays for large grids that its tiles of 512 columns and 16 rows fit, where every input cell comes from
// memory once, if its workgroups are whole rounds of one a compute unit.  us, it / 4 x 4, buffers in turn: 512^3 181 / 203,
// 256 x 512 x 512 93 / 105, 1024 x 512 x 512 387 / 419, 512 x 512 x 1024 383 / 394, 1024 x 1024 x 512 838 / 833; with a last
// round that is not full 512 x 544 x 512 267 / 219, 400 x 400 x 1024 282 / 249, 512 x 320 x 512 147 / 126, 640 x 640 x 512 314 /
// 311, 512 x 480 x 512 191 / 194; with a last row of tiles that is not full 512 x 520 x 512 371 / 202, 512 x 508 x 512 281 /
// 205, 1000 x 1000 x 1024 1675 / 1525; in tiles of 256 columns 384^3 109.7 / 109.2.
static StencilPlan stencil_default(const int64_t* s) {
  const double points = (double)s[0] * s[1] * s[2];
  const StencilPlan march = stencil_march(s);
  if (points >= (double)(1 << 25) && march.LK == 128 && s[2] % 512 == 0 && s[1] % (march.TY * march.RJ) == 0 &&
      cdiv(s[0], march.SI) * (s[1] / (march.TY * march.RJ)) * (s[2] / 512) % 256 == 0)
    return march;
  const StencilPlan direct = points < (double)(1 << 23) ? stencil_direct(s, 2, 2) : points < (double)(1 << 24) ? stencil_direct(s, 2, 4) : stencil_direct(s, 4, 4);
  return stencil_direct_fits(s, direct) ? direct : march;
}

int stencil_candidates(const int64_t* s, StencilPlan* out, int cap) {
  int n = 0;
  auto push = [&](int RJ, int TY, int LK, int SI) {
    if (n >= cap) return;
    if (s[0] > 0 && SI > s[0]) SI = (int)s[0];
    StencilPlan pl{RJ, TY, LK, SI, 0};
    pl.ragged = (s[0] % SI) || (s[1] % (TY * RJ)) || (s[2] % (LK * 4));
    for (int i = 0; i < n; ++i)
      if (!out[i].PI && out[i].RJ == RJ && out[i].TY == TY && out[i].LK == LK && out[i].SI == SI) return;
    out[n++] = pl;
  };
  const StencilPlan d = stencil_default(s);
  if (d.PI) out[n++] = d;
  const StencilPlan march = stencil_march(s);
  push(march.RJ, march.TY, march.LK, march.SI);
  static const int menu[][3] = {{4, 2, 128}, {2, 2, 128}, {8, 2, 128}, {4, 4, 128}, {2, 4, 128},
                                {4, 1, 128}, {8, 1, 128}, {4, 4, 64},  {2, 4, 64},  {4, 2, 64},
                                {4, 8, 32},  {4, 16, 16}};
  static const int sis[] = {16, 32, 64, 128};
  for (auto& m : menu)
    for (int si : sis) push(m[0], m[1], m[2], si);
  for (auto& m : kStencilDirect) {
    const StencilPlan pl = stencil_direct(s, m[0], m[1]);
    if (n < cap && !(d.PI == pl.PI && d.RJ == pl.RJ) && stencil_direct_fits(s, pl)) out[n++] = pl;
  }
  return n;
}

mdh_status plan_stencil(const int64_t* s, const mdh_tile_params* p, StencilPlan* out) {
  if (!p) {
    *out = stencil_default(s);
    return MDH_OK;
  }
  if (p->D != 3) return MDH_ERR_UNSUPPORTED;
  bool ragged;
  mdh_status st = check_products(p, s, &ragged);
  if (st != MDH_OK) return st;
  if ((st = check_lanes(p)) != MDH_OK) return st;
  StencilPlan pl;
  pl.RJ = p->prt[MDH_L_VGPR][1];
  pl.TY = p->prt[MDH_L_WAVE][1] * p->prt[MDH_L_LANE][1];
  pl.LK = p->prt[MDH_L_WAVE][2] * p->prt[MDH_L_LANE][2];
  pl.PI = p->in_region[0] == MDH_MR_VGPR ? p->prt[MDH_L_VGPR][0] : 0;
  pl.SI = pl.PI ? pl.PI : p->prt[MDH_L_HBM][0];
  pl.ragged = ragged;
  if (pl.PI && !stencil_direct_inst(pl)) return MDH_ERR_UNSUPPORTED;
  if (pl.PI && !stencil_direct_fits(s, pl)) return MDH_ERR_SIZE;
  if (!pl.PI && stencil_lds_bytes(pl.RJ, pl.TY, pl.LK) > kLdsBytesPerWG) return MDH_ERR_TILE_RESOURCES;
  mdh_tile_params chk;
  params_from_plan(s, pl, &chk);
  if (!same_table(chk, *p) || !(pl.PI || stencil_inst(pl.RJ, pl.TY, pl.LK))) return MDH_ERR_UNSUPPORTED;
  *out = pl;
  return MDH_OK;
}

// =============================================================================== matmul

struct GemmInst {
  int BM, BN, BK, WM, WN;
};
static const GemmInst kGemmMenu[] = {
    {128, 128, 16, 64, 64}, {256, 128, 16, 128, 64}, {128, 64, 16, 64, 32},
    {64, 64, 16, 32, 32},   {128, 128, 32, 64, 64},  {256, 128, 32, 128, 64},
    {256, 64, 16, 64, 64},  {256, 64, 32, 64, 64},   {128, 64, 32, 64, 32},
    {128, 64, 64, 64, 32},  {256, 64, 64, 64, 64},   {64, 64, 32, 32, 32},
};

// wavefront-layer split of k: (BM, BN, WK) = workgroup tile and wavefronts along k; the 16 x 16 tile is
// one 16 x 16 x 4 block, the others are made of 32 x 32 x 2 blocks
static const int kGemmKsplitMenu[][3] = {{32, 32, 8}, {32, 32, 4}, {32, 32, 16}, {64, 32, 8}, {64, 64, 4},
                                         {64, 64, 8}, {16, 16, 4}, {16, 16, 2}, {16, 16, 8}};

static bool gemm_inst(const GemmPlan& pl) {
  if (pl.split) return split_inst(pl, false);
  if (pl.WK > 1) {
    for (auto& m : kGemmKsplitMenu)
      if (pl.BM == m[0] && pl.BN == m[1] && pl.WK == m[2]) return true;
    return false;
  }
  for (auto& m : kGemmMenu)
    if (m.BM == pl.BM && m.BN == pl.BN && m.BK == pl.BK && m.WM == pl.WM && m.WN == pl.WN)
      return true;
  return false;
}

int64_t gemm_lds_bytes(int BM, int BN, int BK) {
  // two stages of an A tile [BM][BK+4] and a B tile [BK][BN+4]
  return 2ll * ((int64_t)BM * (BK + 4) + (int64_t)BK * (BN + 4)) * 4;
}

void params_from_plan(const int64_t* s, const GemmPlan& pl, mdh_tile_params* p) {
  clear_params(p, 3);
  p->blk[0] = 32;
  p->blk[1] = 32;
  const int bk = pl.split ? 16 : 2;
  p->blk[2] = bk;  // one v_mfma_f32_32x32x2_f32, or six v_mfma_f32_32x32x16_bf16
  if (pl.WK > 1 && pl.split) {
    // k on the wavefront layer, chunks of 32 as two register parts: combined in LDS
    p->prt[MDH_L_VGPR][2] = 2;
    p->prt[MDH_L_WG][0] = (int32_t)cdiv(s[0], pl.BM);
    p->prt[MDH_L_WG][1] = (int32_t)cdiv(s[1], pl.BN);
    p->prt[MDH_L_WG][2] = pl.S;
    p->prt[MDH_L_WAVE][2] = pl.WK;
    p->prt[MDH_L_HBM][2] = (int32_t)cdiv(cdiv(s[2], (int64_t)pl.S * pl.WK), 32);
    p->prt[MDH_L_VGPR][0] = pl.BM / 32;
    p->prt[MDH_L_VGPR][1] = pl.BN / 32;
    static const int kdims[3] = {0, 1, 2};
    set_order(p, kdims);
    p->strided = 0;
    p->lane_fast_dim = 1;
    p->in_region[0] = MDH_MR_VGPR;
    p->in_region[1] = MDH_MR_VGPR;
    p->out_region = MDH_MR_LDS;
    p->ragged = (uint8_t)pl.ragged;
    return;
  }
  if (pl.WK > 1) {
    // k on the wavefront layer: every wavefront owns the whole tile and walks groups of 8 k (4 MFMA
    // steps of 2; with the 16 x 16 x 4 block: groups of 16 k, 4 steps of 4) read straight into
    // registers; the wavefront results are combined in LDS
    const int b = pl.BM == 16 ? 16 : 32, kb = pl.BM == 16 ? 4 : 2;
    p->blk[0] = p->blk[1] = b;
    p->blk[2] = kb;
    p->prt[MDH_L_WG][0] = (int32_t)cdiv(s[0], pl.BM);
    p->prt[MDH_L_WG][1] = (int32_t)cdiv(s[1], pl.BN);
    p->prt[MDH_L_WG][2] = pl.S;
    p->prt[MDH_L_WAVE][2] = pl.WK;
    p->prt[MDH_L_HBM][2] = (int32_t)cdiv(cdiv(s[2], (int64_t)pl.S * pl.WK), 4 * kb);
    p->prt[MDH_L_VGPR][0] = pl.BM / b;
    p->prt[MDH_L_VGPR][1] = pl.BN / b;
    p->prt[MDH_L_VGPR][2] = 4;
    static const int kdims[3] = {0, 1, 2};
    set_order(p, kdims);
    p->strided = 0;
    p->lane_fast_dim = 1;
    p->in_region[0] = MDH_MR_VGPR;
    p->in_region[1] = MDH_MR_VGPR;
    p->out_region = MDH_MR_LDS;
    p->ragged = (uint8_t)pl.ragged;
    return;
  }
  p->prt[MDH_L_WG][0] = (int32_t)cdiv(s[0], pl.BM);
  p->prt[MDH_L_WG][1] = (int32_t)cdiv(s[1], pl.BN);
  p->prt[MDH_L_WG][2] = pl.S;
  p->prt[MDH_L_HBM][2] = (int32_t)cdiv(cdiv(s[2], pl.S), pl.BK);
  p->prt[MDH_L_WAVE][0] = pl.BM / pl.WM;
  p->prt[MDH_L_WAVE][1] = pl.BN / pl.WN;
  p->prt[MDH_L_LDS][2] = pl.BK / bk;
  p->prt[MDH_L_VGPR][0] = pl.WM / 32;
  p->prt[MDH_L_VGPR][1] = pl.WN / 32;
  static const int dims[3] = {0, 1, 2};
  set_order(p, dims);
  if (pl.jmajor) {  // workgroup layer: j before i
    p->order[0] = (uint8_t)(MDH_L_WG * MDH_MAX_D + 1);
    p->order[1] = (uint8_t)(MDH_L_WG * MDH_MAX_D + 0);
  }
  p->strided = 0;
  p->lane_fast_dim = 1;
  p->in_region[0] = MDH_MR_LDS;
  p->in_region[1] = MDH_MR_LDS;
  p->out_region = MDH_MR_VGPR;
  p->ragged = (uint8_t)pl.ragged;
}

static int gemm_ragged(const int64_t* s, const GemmPlan& pl) {
  if (pl.WK > 1)
    return (s[0] % pl.BM) || (s[1] % pl.BN) || (s[2] % ((int64_t)pl.S * pl.WK * (pl.split ? 32 : pl.BM == 16 ? 16 : 8)));
  return (s[0] % pl.BM) || (s[1] % pl.BN) || (s[2] % ((int64_t)pl.S * pl.BK));
}

// the fp32 kernels' choice
static GemmPlan gemm_default_fp32(const int64_t* s) {
  const int64_t M = s[0], N = s[1], K = s[2];
  // Outputs of few tiles: k over the wavefronts of a workgroup, one launch, tiles small enough to give
  // every compute unit a workgroup.  Kernel durations (rocprofv3 kernel trace, us; the LDS-tiled kernel
  // with 64 x 64 tiles beside it, second pass included where it splits k):
  //   128^3: 2.9 (16 x 16 tiles, 2 wavefronts) / 5.1      256^3: 3.3 (16 x 16, 4) / 8.4
  //   200 x 300 x 500: 5.1 (16 x 16, 4) / 8.6             256 x 256 x 4096: 13.7 (16 x 16, 4) / 15.3
  //   384^3: 5.5 (32 x 32, 4) / 7.5                       512^3: 6.5 (32 x 32, 4) / 9.9
  //   768^3 and 1024^3: the LDS-tiled kernel stays ahead (18.9 against 20.0; 26.3 against 28.1)
  if (K >= 32 && K <= 8192 && M > 0 && N > 0) {
    const int64_t t16 = cdiv(M, 16) * cdiv(N, 16), t32 = cdiv(M, 32) * cdiv(N, 32);
    // (up to 384 where k is short: 300^3 5.4 with 16 x 16 tiles, 6.8 with 32 x 32; 700 x 450 x 150: 7.1 / 8.5 LDS-tiled)
    const int64_t few = K <= 512 ? 384 : 320;
    if (t16 <= few || t32 <= few) {
      const int b = t16 <= few ? 16 : 32;
      GemmPlan pl{b, b, b == 16 ? 16 : 8, b, b, 1, 0};
      pl.WK = (b == 16 && K <= 128) ? 2 : 4;
      pl.ragged = gemm_ragged(s, pl);
      return pl;
    }
  }
  // Tile: the largest of 128x128, 128x64, 64x64 that still gives two workgroups per compute unit
  // (measured best at 4096^3, 2048^3 and 1024^3 respectively); narrow problems keep 128x64 / 64x64.
  GemmPlan pl{128, 128, 32, 64, 64, 1, 0};
  const bool narrow = N <= 64 || M <= 64;
  if (narrow) {
    // one tile spans the short dimension.  Measured (65536 x 64 x 4096 / 16384 x 64 x 4096 /
    // 64 x 65536 x 1024): 128x64 tiles only where they still give two workgroups per compute unit
    // (0.312 against 0.327 ms), 64x64 tiles otherwise (0.085 against 0.088 ms; 0.087 against 0.19 ms
    // when M = 64 would leave half of a 128-row tile empty)
    pl = GemmPlan{64, 64, 32, 32, 32, 1, 0};
    if (M > 64 && cdiv(M, 128) * cdiv(N, 64) >= 512) pl = GemmPlan{128, 64, 32, 64, 32, 1, 0};
  } else if (cdiv(M, 128) * cdiv(N, 128) < 512) {
    pl = GemmPlan{128, 64, 32, 64, 32, 1, 0};
    if (cdiv(M, 128) * cdiv(N, 64) < 512) pl = GemmPlan{64, 64, 32, 32, 32, 1, 0};
  } else {
    // wave quantisation: 512 tiles of 128 x 128 run at once; when the last round would be mostly
    // empty the 64 x 64 tile (about 0.8 of the rate, but four times the tiles) is faster.  Measured:
    // 3000^3 (576 tiles) 0.66 -> 0.52 ms; 4100 x 4096 x 4096 (1056 tiles) 1.32 -> 1.18 ms.
    const double rounds = (double)(cdiv(M, 128) * cdiv(N, 128)) / 512.0;
    const double whole = (double)cdiv(cdiv(M, 128) * cdiv(N, 128), 512);
    if (whole > 1.3 * rounds) pl = GemmPlan{64, 64, 32, 32, 32, 1, 0};
  }
  // Split the reduction dimension over workgroups only while there is less than one workgroup per
  // compute unit (two for the narrow shapes, whose tiles are small) AND every part keeps at least 8
  // k-tiles: below that the second pass and the shortened pipelines cost more than the parallelism
  // gains (256^3 is fastest unsplit, 8.7 us against 14.6 us with 16 parts; 256 x 256 x 4096 is
  // fastest with 16 parts; 8192 x 64 x 4096 with 4 parts: 0.046 against 0.089 ms unsplit).
  const int64_t tiles = cdiv(M, pl.BM) * cdiv(N, pl.BN);
  const int64_t want = narrow ? 512 : 256;
  int S = 1;
  while (tiles * S < want && S < 64 && K / (S * 2) >= 8 * pl.BK) S *= 2;
  // beyond 64 parts only while a part keeps 2048 elements of k (64 x 64 x 2^20: 0.22 ms with 256
  // parts against 0.55 ms with 64; 32 x 32 x 65536 is fastest with 64)
  while (tiles * S < want && S >= 64 && S < 256 && K / (S * 2) >= 2048) S *= 2;
  pl.S = S;
  pl.ragged = gemm_ragged(s, pl);
  return pl;
}

// The default without more workspace than the fp32 rule asks for; on slices in at most `most` parts of k.
static GemmPlan gemm_default_lean(const int64_t* s, int64_t most = 1 << 20) {
  GemmPlan pl = gemm_default_fp32(s);
  const int S = pl.S < most ? pl.S : (int)most;
  // outputs of few tiles stay with k over the wavefronts, on either kernel
  if (!(pl.WK > 1 ? split_k_default(s[0], s[1], s[2], pl, &pl) : split_default(1, s[0], s[1], s[2], false, S, &pl))) return pl;
  pl.ragged = gemm_ragged(s, pl);
  return pl;
}

static GemmPlan gemm_default(const int64_t* s) {
  GemmPlan pl = gemm_default_fp32(s);
  if (pl.WK <= 1) return gemm_default_lean(s);
  // Few tiles and many k: parts of k over workgroups too, as many as leave a compute unit one workgroup and a part
  // its worth of k, against the second pass (us, replayed from a graph; WK wavefronts, S parts)
  const int64_t K = s[2];
  auto parts = [&](int64_t tiles, int64_t least) {
    int S = 1;
    while (S < 8 && tiles * 2 * S <= 320 && K / (2 * S) >= least) S *= 2;
    return S;
  };
  if (pl.BM == 16) {
    // 20 x 1000 x 3000: 13.8 with S = 2, 19.4 without; 90 x 90 x 8000: 14.9 with 4 and eight wavefronts, 46 without;
    // 128 x 300 x 2000: 8.9 with eight wavefronts, 11.2 with four.  A second launch costs the host about 6 us: not
    // below 14 us, which whole blocks reach at a deeper k (64 x 64 x 4096: 10.9 in one launch, 6.6 + the launch)
    const bool whole = s[0] % 16 == 0 && s[1] % 16 == 0 && K % 16 == 0;
    if (K >= (whole ? 6000 : 2400)) pl.S = parts(cdiv(s[0], 16) * cdiv(s[1], 16), 1024);
    if (K / (8 * pl.S) >= 250) pl.WK = 8;
  } else if (K >= 1500 && (s[0] % 32 || s[1] % 32) && s[0] >= 40 && s[1] >= 40 && split_sizes(s[0], s[1], K)) {
    // ragged tiles go through the checked loads, which take twice as long: the split kernel's do not (320 x 900 x
    // 2500: 26 against 53; 40 x 2000 x 2000: 17 against 26; 512 x 512 x 4096: 28.8 against 28.7)
    const GemmPlan sp{64, 64, 32, 32, 32, 1, 0};
    const int S = parts(cdiv(s[0], 64) * cdiv(s[1], 64), 256);
    if (S >= 4 && !split_default(1, s[0], s[1], K, false, S, &pl)) {
      pl = sp;
      pl.split = 1;
      pl.S = S;
    }
  }
  if (!pl.split) split_k_default(s[0], s[1], K, pl, &pl);
  while (pl.split && pl.WK == 1 && (pl.S - 1) * split_part(K, pl) >= K) pl.S /= 2;
  pl.ragged = gemm_ragged(s, pl);
  return pl;
}

void plan_matmul_lean(const int64_t* s, size_t workspace, GemmPlan* pl) {
  const GemmPlan d = gemm_default(s);
  mdh_tile_params a, b;
  params_from_plan(s, d, &a);
  params_from_plan(s, *pl, &b);
  if (same_table(a, b)) *pl = gemm_default_lean(s, parts_held(workspace, s[0] * s[1]));
}

int matmul_candidates(const int64_t* s, GemmPlan* out, int cap) {
  int n = 0;
  auto push = [&](GemmPlan pl) {
    if (n >= cap) return;
    if (pl.S > 1 && s[2] / pl.S < pl.BK) return;
    if (pl.WK == 1 && !pl.split && gemm_lds_bytes(pl.BM, pl.BN, pl.BK) > kLdsBytesPerWG) return;
    pl.ragged = gemm_ragged(s, pl);
    for (int i = 0; i < n; ++i)
      if (out[i].BM == pl.BM && out[i].BN == pl.BN && out[i].BK == pl.BK && out[i].WM == pl.WM &&
          out[i].S == pl.S && out[i].WK == pl.WK && out[i].jmajor == pl.jmajor && out[i].split == pl.split)
        return;
    out[n++] = pl;
  };
  // (for few rows candidate 0 is shown as the small-M kernel: what it hides is the fp32 kernels' choice, as ever)
  if (small_m_matmul(s, nullptr)) push(gemm_default_fp32(s));
  for (const GemmPlan& d : {gemm_default(s), gemm_default_fp32(s)}) {
    push(d);
    // its tile with the other loop order of the workgroup layer (column bands)
    GemmPlan t = d;
    t.jmajor = !t.jmajor;
    if (t.WK == 1 && cdiv(s[0], t.BM) > 1 && cdiv(s[1], t.BN) > 1) push(t);
  }
  if (split_sizes(s[0], s[1], s[2])) {
    GemmPlan sp[kSplitTiles];
    const int ns = split_offered(1, s[0], s[1], s[2], false, sp);
    for (int i = 0; i < ns; ++i)
      for (int S : {1, 2, 4}) {
        if (S > 1 && (cdiv(s[0], sp[i].BM) * cdiv(s[1], sp[i].BN) * (S / 2) >= 2048 || s[2] / S < 128)) continue;
        sp[i].S = S;
        if (split_fits(s[0], s[1], s[2], sp[i])) push(sp[i]);
      }
  }
  // k over the wavefronts of a workgroup, for outputs of few tiles (every wavefront keeps 8 k or more)
  if (cdiv(s[0], 32) * cdiv(s[1], 32) <= 1024)
    for (auto& m : kGemmKsplitMenu)
      for (int S : {1, 2, 4}) {
        if (s[2] / ((int64_t)S * m[2]) < 16) continue;
        if (S > 1 && cdiv(s[0], m[0]) * cdiv(s[1], m[1]) * (S / 2) >= 256) continue;
        if (m[0] == 16 && cdiv(s[0], 16) * cdiv(s[1], 16) > 1024) continue;
        GemmPlan pl{m[0], m[1], m[0] == 16 ? 16 : 8, m[0], m[1], S, 0};
        pl.WK = m[2];
        push(pl);
      }
  static const int splits[] = {1, 2, 4, 8, 16};
  for (auto& m : kGemmMenu)
    for (int S : splits) {
      const int64_t tiles = cdiv(s[0], m.BM) * cdiv(s[1], m.BN);
      if (S > 1 && tiles * (S / 2) >= 2048) continue;  // splitting a full grid only adds traffic
      push(GemmPlan{m.BM, m.BN, m.BK, m.WM, m.WN, S, 0});
    }
  return n;
}

mdh_status plan_matmul(const int64_t* s, const mdh_tile_params* p, GemmPlan* out) {
  if (!p) {
    *out = gemm_default(s);
    return MDH_OK;
  }
  if (p->D != 3) return MDH_ERR_UNSUPPORTED;
  bool ragged;
  mdh_status st = check_products(p, s, &ragged);
  if (st != MDH_OK) return st;
  if ((st = check_lanes(p)) != MDH_OK) return st;
  if (p->prt[MDH_L_WAVE][2] > 1) {
    // wavefront-layer parts of k: the register-streaming kernel
    GemmPlan pl;
    const bool b16 = p->blk[0] == 16;
    pl.split = p->blk[2] == 16;
    if (!((p->blk[0] == 32 && p->blk[1] == 32 && (p->blk[2] == 2 || pl.split)) || (b16 && p->blk[1] == 16 && p->blk[2] == 4)))
      return MDH_ERR_UNSUPPORTED;
    pl.BM = pl.WM = p->prt[MDH_L_VGPR][0] * p->blk[0];
    pl.BN = pl.WN = p->prt[MDH_L_VGPR][1] * p->blk[1];
    pl.BK = pl.split ? 32 : b16 ? 16 : 8;
    pl.S = p->prt[MDH_L_WG][2];
    pl.WK = p->prt[MDH_L_WAVE][2];
    pl.ragged = ragged;
    if (pl.split && !split_inst(pl, false)) return MDH_ERR_UNSUPPORTED;
    if (pl.split && (pl.S - 1) * split_part(s[2], pl) >= s[2]) return MDH_ERR_TILE_NOT_DIVIDING;  // a part without k
    if (pl.split && !split_fits(s[0], s[1], s[2], pl)) return MDH_ERR_UNSUPPORTED;
    // model constraints: lanes per workgroup, and the LDS that holds the WK partial tiles
    if ((int64_t)pl.WK * 64 > kMaxLanesPerWG) return MDH_ERR_TILE_RESOURCES;
    if ((int64_t)pl.WK * pl.BM * pl.BN * 4 > kLdsBytesPerWG) return MDH_ERR_TILE_RESOURCES;
    mdh_tile_params chk;
    params_from_plan(s, pl, &chk);
    if (!same_table(chk, *p) || !gemm_inst(pl)) return MDH_ERR_UNSUPPORTED;
    *out = pl;
    return MDH_OK;
  }
  GemmPlan pl;
  pl.WM = p->prt[MDH_L_VGPR][0] * 32;
  pl.WN = p->prt[MDH_L_VGPR][1] * 32;
  pl.BM = p->prt[MDH_L_WAVE][0] * pl.WM;
  pl.BN = p->prt[MDH_L_WAVE][1] * pl.WN;
  pl.split = p->blk[2] == 16;
  pl.BK = p->prt[MDH_L_LDS][2] * p->blk[2];
  pl.S = p->prt[MDH_L_WG][2];
  pl.ragged = ragged;
  // parameter D1 on the workgroup layer: (WG,j) before (WG,i) selects the column-band tile order; any
  // other permutation has no instantiation (the regenerated table below differs)
  pl.jmajor = (p->order[0] == MDH_L_WG * MDH_MAX_D + 1 && p->order[1] == MDH_L_WG * MDH_MAX_D + 0) ? 1 : 0;
  if (p->blk[0] != 32 || p->blk[1] != 32 || (p->blk[2] != 2 && p->blk[2] != 16)) return MDH_ERR_UNSUPPORTED;
  if (pl.split && (!split_inst(pl, false) || !split_sizes(s[0], s[1], s[2]))) return MDH_ERR_UNSUPPORTED;
  if (pl.split && (pl.S - 1) * split_part(s[2], pl) >= s[2]) return MDH_ERR_TILE_NOT_DIVIDING;  // a part without k
  if ((pl.split ? split_lds_bytes(pl) : gemm_lds_bytes(pl.BM, pl.BN, pl.BK)) > kLdsBytesPerWG) return MDH_ERR_TILE_RESOURCES;
  if ((int64_t)p->prt[MDH_L_WAVE][0] * p->prt[MDH_L_WAVE][1] * 64 > kMaxLanesPerWG)
    return MDH_ERR_TILE_RESOURCES;
  mdh_tile_params chk;
  params_from_plan(s, pl, &chk);
  if (!same_table(chk, *p) || !gemm_inst(pl)) return MDH_ERR_UNSUPPORTED;
  *out = pl;
  return MDH_OK;
}

// ---- MatMul with few rows: the small-M kernel of the batched instance, one batch entry

bool small_m_matmul(const int64_t* s, const mdh_tile_params* p) {
  if (!p) return s[0] > 0 && s[0] <= 16 && s[1] > 0;
  // both strip widths of that kernel (64 or 16 columns per wavefront); the kernel that splits k over
  // wavefronts has 16 x 16 x 4 blocks too, but combines in LDS
  return p->D == 3 && p->blk[0] == 16 && (p->prt[MDH_L_VGPR][1] == 4 || p->out_region != MDH_MR_LDS);
}

static void move_dims(const mdh_tile_params& src, mdh_tile_params* dst, int D, int shift) {
  // dimension d of dst is dimension d + shift of src (shift = 1 drops the batch, -1 inserts it)
  clear_params(dst, D);
  for (int d = 0; d < D; ++d) {
    const int e = d + shift;
    if (e < 0 || e >= src.D) continue;  // the inserted batch dimension: one part everywhere, blk 1
    dst->blk[d] = src.blk[e];
    for (int l = 0; l < MDH_NUM_LAYERS; ++l) dst->prt[l][d] = src.prt[l][e];
  }
  int dims[MDH_MAX_D];
  for (int d = 0; d < D; ++d) dims[d] = d;
  set_order(dst, dims);
  dst->strided = src.strided;
  dst->lane_fast_dim = (uint8_t)(src.lane_fast_dim - shift);
  dst->ragged = src.ragged;
  memcpy(dst->in_region, src.in_region, sizeof(src.in_region));
  dst->out_region = src.out_region;
  memcpy(dst->in_transposed, src.in_transposed, sizeof(src.in_transposed));
  dst->out_transposed = src.out_transposed;
}

void lift_batch(const mdh_tile_params& p3, mdh_tile_params* p4) { move_dims(p3, p4, 4, -1); }
void drop_batch(const mdh_tile_params& p4, mdh_tile_params* p3) { move_dims(p4, p3, 3, 1); }

// the batched instance's view of a small-M MatMul call: sizes and (if given) the lifted table
static mdh_status plan_small_m(const int64_t* s, const mdh_tile_params* p, GemmExPlan* out) {
  const int64_t s4[7] = {1, s[0], s[1], s[2], 0, 0, 0};
  if (!p) return plan_matmul_ex(s4, nullptr, out);
  mdh_tile_params p4;
  lift_batch(*p, &p4);
  // the order entries of the caller's table must be the ones this library generates
  mdh_tile_params back;
  drop_batch(p4, &back);
  if (!same_table(back, *p)) return MDH_ERR_UNSUPPORTED;
  return plan_matmul_ex(s4, &p4, out);
}

mdh_status plan_matmul_small_m(const int64_t* s, const mdh_tile_params* p, GemmExPlan* out) {
  return plan_small_m(s, p, out);
}

// =============================================================================== MCC

int64_t mcc_flat_lds_bytes(int QB, int TP, int BN, int64_t C, int64_t R, int64_t S, int64_t sh, int64_t sw);

struct MccInst {
  int TP, TQ, BN, CK, WM, WN;
};
static const MccInst kMccMenu[] = {  // channel-chunked kernel
    {4, 32, 128, 16, 64, 64},
    {8, 32, 128, 16, 128, 64},
    {2, 32, 64, 16, 32, 32},
    {4, 32, 64, 16, 64, 32},
    {8, 16, 128, 16, 64, 64},  // blocks of 2 x 16 pixels (images narrower than 32 output columns)
    {8, 16, 64, 16, 64, 32},
    {8, 8, 128, 16, 32, 64},   // blocks of 4 x 8 pixels
    {8, 8, 64, 16, 32, 32},
    {4, 32, 128, 32, 64, 64},  // channel chunks of 32: twice the MFMAs between two barriers
    {4, 32, 64, 32, 64, 32},
    {8, 16, 128, 32, 64, 64},
    {8, 16, 64, 32, 64, 32},
    {8, 8, 128, 32, 32, 64},
    {8, 8, 64, 32, 32, 32},
};
// few-channel kernel (s and c fused): TP rows x TQ = QB columns of pixels, BN channels, WM, WN
static const MccInst kMccFlatMenu[] = {
    {8, 16, 64, 0, 32, 64},  {4, 32, 64, 0, 32, 64},   {8, 16, 32, 0, 32, 32},
    {4, 32, 32, 0, 32, 32},  {8, 16, 128, 0, 64, 64},  {4, 32, 128, 0, 64, 64},
    {8, 16, 64, 0, 32, 32},  {4, 32, 64, 0, 32, 32},   {16, 16, 32, 0, 32, 32},  {8, 32, 32, 0, 32, 32},  // eight wavefronts
};

// channel-chunked kernel that splits fp32 values into bf16 slices
static const MccInst kMccSplitMenu[] = {
    {8, 32, 128, 16, 64, 64}, {4, 32, 128, 16, 64, 64}, {4, 32, 64, 16, 64, 32}, {8, 16, 128, 16, 64, 64}, {8, 16, 64, 16, 64, 32},
    {8, 8, 128, 16, 32, 64},  {8, 8, 64, 16, 32, 32},   {8, 32, 128, 32, 64, 64}, {4, 32, 128, 32, 64, 64}, {4, 32, 64, 32, 64, 32},
    {8, 16, 128, 32, 64, 64}, {8, 16, 64, 32, 64, 32},  {16, 8, 64, 32, 64, 32}, {8, 8, 128, 32, 32, 64}, {8, 8, 64, 32, 32, 32},
};
// few-channel kernel that splits: a wavefront's block of 32 pixels x 32 or 64 channels
static const MccInst kMccFlatSplitMenu[] = {{2, 16, 64, 0, 32, 64}, {1, 32, 64, 0, 32, 64}, {4, 8, 64, 0, 32, 64},
                                            {2, 16, 32, 0, 32, 32}, {1, 32, 32, 0, 32, 32}, {4, 8, 32, 0, 32, 32}};

static bool mcc_inst(const MccPlan& pl) {
  const MccInst* menu = pl.flat ? pl.split ? kMccFlatSplitMenu : kMccFlatMenu : pl.split ? kMccSplitMenu : kMccMenu;
  const int n = (int)(pl.flat ? pl.split ? sizeof(kMccFlatSplitMenu) : sizeof(kMccFlatMenu) : pl.split ? sizeof(kMccSplitMenu) : sizeof(kMccMenu)) / (int)sizeof(MccInst);
  for (int i = 0; i < n; ++i) {
    const MccInst& m = menu[i];
    if (m.TP == pl.TP && m.TQ == pl.TQ && m.BN == pl.BN && m.CK == pl.CK && m.WM == pl.WM && m.WN == pl.WN)
      return true;
  }
  return false;
}

// sizes: N, P, Q, K, C, R, S, stride_h, stride_w
int64_t mcc_lds_bytes(const MccPlan& pl, const int64_t* s) {
  if (pl.flat && pl.split) return mcc_flat_split_lds_bytes(pl.BN, s[4], s[5], s[6]);
  if (pl.flat) return mcc_flat_lds_bytes(pl.TQ, pl.TP, pl.BN, s[4], s[5], s[6], s[7], s[8]);
  const int64_t ph = (pl.TP - 1) * s[7] + s[5], pw = (pl.TQ - 1) * s[8] + s[6];
  if (pl.split) return 6ll * pl.CK * (cdiv(ph * pw, 8) * 8 + (pl.CK == 16 ? 4 : 2)) + 12ll * pl.BN * pl.CK + 16;
  return (ph * pw * (pl.CK + 4) + 2ll * pl.BN * (pl.CK + 4)) * 4;
}

void params_from_plan(const int64_t* s, const MccPlan& pl, mdh_tile_params* p) {
  // dims: 0 n, 1 p, 2 q, 3 k, 4 c, 5 r, 6 s
  clear_params(p, 7);
  p->prt[MDH_L_WG][0] = (int32_t)s[0];
  p->prt[MDH_L_WG][1] = (int32_t)cdiv(s[1], pl.TP);
  p->prt[MDH_L_WG][2] = (int32_t)cdiv(cdiv(s[2], pl.TQ), pl.flat ? pl.QT : 1);
  p->prt[MDH_L_WG][3] = (int32_t)cdiv(s[3], pl.BN);
  if (pl.flat) p->prt[MDH_L_HBM][2] = pl.QT;  // column tiles walked with the filter slice resident
  p->prt[MDH_L_LDS][5] = (int32_t)s[5];
  p->prt[MDH_L_LDS][6] = (int32_t)s[6];
  p->prt[MDH_L_WAVE][3] = pl.BN / pl.WN;
  p->prt[MDH_L_VGPR][3] = pl.WN / 32;
  p->blk[3] = 32;  // 32 output channels
  if (pl.flat) {
    // few channels: the block is (32/QB rows of p) x (QB consecutive q); s and c are walked as one
    // sequential LDS-layer dimension of S*C single steps (two of them feed one MFMA)
    const int rb = 32 / pl.TQ, mi = pl.WM / 32;
    p->blk[1] = rb;
    p->blk[2] = pl.TQ;
    p->prt[MDH_L_LDS][4] = (int32_t)s[4];
    p->prt[MDH_L_WAVE][1] = pl.TP / (rb * mi);
    p->prt[MDH_L_VGPR][1] = mi;
  } else {
    // the block: 32 pixels = (32/TQ rows of p) x (TQ consecutive q), 2 input channels per MFMA
    const int rb = 32 / pl.TQ, mi = pl.WM / 32;
    p->blk[1] = rb;
    p->blk[2] = pl.TQ;
    p->blk[4] = 2;
    if (pl.split) p->prt[MDH_L_VGPR][4] = 8;  // 16 channels per v_mfma_f32_32x32x16_bf16
    p->prt[MDH_L_WG][4] = pl.S;  // parts of the reduction dimension c over workgroups
    p->prt[MDH_L_HBM][4] = (int32_t)cdiv(cdiv(s[4], pl.S), pl.CK);
    p->prt[MDH_L_LDS][4] = pl.split ? pl.CK / 16 : pl.CK / 2;
    // wavefront grid: TP/(mi*rb) along p, BN/WN along k; mi blocks along p per wavefront
    p->prt[MDH_L_WAVE][1] = pl.TP / (mi * rb);
    p->prt[MDH_L_VGPR][1] = mi;
  }
  static const int dims[7] = {0, 1, 2, 3, 4, 5, 6};
  set_order(p, dims);
  // few-channel kernel: 0 = a workgroup owns a run of column tiles, 1 = the tiles of (n, p, q) are dealt
  // out one at a time to the workgroups resident on the chip
  p->strided = (pl.flat && pl.dealt) ? 1 : 0;
  p->lane_fast_dim = 3;
  p->in_region[0] = pl.flat && pl.split ? MDH_MR_HBM : MDH_MR_LDS;
  p->in_region[1] = MDH_MR_LDS;
  p->out_region = MDH_MR_VGPR;
  p->ragged = (uint8_t)pl.ragged;
}

// the split kernel reads whole channel chunks, the last one ending with the last channel; a filter row's address is
// a 32-bit offset from the tile's first
static bool mcc_split_sizes(const int64_t* s, const MccPlan& pl) {
  const int64_t part = cdiv(cdiv(s[4], pl.S), pl.CK) * pl.CK;
  return s[4] >= pl.CK && (pl.S - 1) * part < s[4] && s[5] * s[6] * s[4] <= (1 << 22);
}

static int mcc_ragged(const int64_t* s, const MccPlan& pl) {
  if (pl.flat) return (s[1] % pl.TP) || (s[2] % ((int64_t)pl.TQ * pl.QT)) || (s[3] % pl.BN);
  return (s[1] % pl.TP) || (s[2] % pl.TQ) || (s[3] % pl.BN) || (s[4] % ((int64_t)pl.S * pl.CK));
}

// Column tiles per workgroup of the few-channel kernel: at most `want`, fewer while the grid would
// drop below one workgroup per compute unit; normalised so that no workgroup is without a tile.
static int flat_qt(const int64_t* s, const MccPlan& pl, int want, int min_wgs = 256) {
  const int64_t tiles = cdiv(s[2] > 0 ? s[2] : 1, pl.TQ);
  const int64_t other = (s[0] > 0 ? s[0] : 1) * cdiv(s[1] > 0 ? s[1] : 1, pl.TP) * cdiv(s[3] > 0 ? s[3] : 1, pl.BN);
  int64_t qt = want < tiles ? want : tiles;
  while (qt > 1 && other * cdiv(tiles, qt) < min_wgs) qt = cdiv(qt, 2);
  return (int)cdiv(tiles, cdiv(tiles, qt));
}

static MccPlan mcc_flat_plan(const int64_t* s) {
  // Measured on the first-layer shapes of ResNet-50, VGG-16 and MobileNet: 32 channels per
  // workgroup up to K = 64 (more workgroups, each stages a smaller filter slice; a lane stores 16
  // bytes of a pixel, so narrow channel slices still write whole 128-byte lines), a workgroup keeps
  // its filter slice and walks up to 8 column tiles (ResNet-50: 56 us against 64 us with one tile;
  // VGG-16: 66 us against 80 us with 64 channels), blocks of 8 x 16 pixels where 16 divides Q and
  // 32 does not (Q = 112), of 4 x 32 pixels otherwise.
  // Where the grid is large enough, eight wavefronts per workgroup -- two along k from 64 channels
  // on (they share one input patch), otherwise all along p -- blocks of 8 x 16 pixels, and up to 16
  // column tiles per workgroup while 192 workgroups remain.  Candidates measured in alternation
  // (medians): VGG-16 first layer, N = 16: 67.7 us against 71.2 us for the rule below; MobileNet:
  // 18.9 against 19.2 us; ResNet-50, N = 4: 20.0 against 21.7 us; N = 16 and 32: equal to the rule
  // below at 32 channels per workgroup (54.1 us, 89 us), one patch staging instead of two; with
  // N = 1 the four-wavefront workgroups below stay faster (10.0 against 11.4 us).
  {
    MccPlan w = s[3] > 32 ? MccPlan{8, 16, 64, 0, 32, 32, 0, 1} : MccPlan{16, 16, 32, 0, 32, 32, 0, 1};
    const int64_t wgs = (s[0] > 0 ? s[0] : 1) * cdiv(s[1] > 0 ? s[1] : 1, w.TP) * cdiv(s[2] > 0 ? s[2] : 1, w.TQ) *
                        cdiv(s[3] > 0 ? s[3] : 1, w.BN);
    if (wgs >= 256 && mcc_lds_bytes(w, s) <= kLdsBytesPerWG) {
      // Long walks per tile (ResNet-50's 7 x 7 filter: 21 steps of 8; the 3 x 3 filters have 6): tiles of
      // 16 x 16 pixels x 32 channels dealt out to resident workgroups instead of owned -- every compute
      // unit stays busy to the end and two workgroups per unit cover each other's tile hand-over.
      // ResNet-50 first layer, N = 16: 46.9 against 55.3 us; N = 32: 81 against 96 us; N = 4: 17.4 against
      // 19.1 us.  VGG-16 (70 against 81 us) and MobileNet (16.5 against 16.9 us) stay with owned tiles.
      MccPlan d{16, 16, 32, 0, 32, 32, 0, 1};
      d.dealt = 1;
      if (s[5] * cdiv(s[6] * s[4], 8) >= 16 && cdiv(s[3] > 0 ? s[3] : 1, d.BN) <= 8 && mcc_lds_bytes(d, s) <= kLdsBytesPerWG) {
        d.ragged = mcc_ragged(s, d);
        return d;
      }
      w.QT = flat_qt(s, w, 16, 192);
      w.ragged = mcc_ragged(s, w);
      return w;
    }
  }
  const int qb = (s[2] % 32 != 0 && s[2] % 16 == 0) ? 16 : 32;
  const int tp = qb == 16 ? 8 : 4;
  MccPlan pl{tp, qb, 32, 0, 32, 32, 0, 1};
  if (s[3] > 64) pl = MccPlan{tp, qb, 64, 0, 32, 64, 0, 1};
  pl.QT = flat_qt(s, pl, 8);
  pl.ragged = mcc_ragged(s, pl);
  return pl;
}

// The few-channel kernel reads its input in 16-byte pieces and needs an input of at least four elements;
// the smallest input these output sizes can have is N x ((P-1) sh + R) x ((Q-1) sw + S) x C.
static bool flat_input_ok(const int64_t* s) {
  return (s[0] > 0 ? s[0] : 1) * ((s[1] > 0 ? s[1] - 1 : 0) * s[7] + s[5]) * ((s[2] > 0 ? s[2] - 1 : 0) * s[8] + s[6]) * s[4] >= 4;
}

// the fp32 kernels' choice
static MccPlan mcc_default_fp32(const int64_t* s) {
  if (s[4] <= 8 && flat_input_ok(s)) {  // fewer channels than half a channel chunk: fuse s and c
    MccPlan f = mcc_flat_plan(s);
    if (mcc_lds_bytes(f, s) <= kLdsBytesPerWG) return f;
  }
  // Pixel block: 32 consecutive q of one row, 2 x 16 or 4 x 8 pixels -- the shape whose tiles (4 x 32,
  // 8 x 16, 8 x 8 pixels) pad the image least; on a tie the widest.  Squarer tiles also stage less
  // halo.  Measured against blocks of 32 columns throughout: 32 x 112 x 112 x 64 -> 32, 3 x 3: 0.144
  // against 0.191 ms; 16 x 56 x 56, 1 x 1, 256 -> 64 / 64 -> 256: 28 / 32 us against 41 / 55 us;
  // 16 x 14 x 14 x 256 -> 256, 3 x 3: 122 against 137 us.
  const int64_t P = s[1] > 0 ? s[1] : 1, Q = s[2] > 0 ? s[2] : 1;
  // (on a tie the widest that still gives two workgroups per compute unit at 64 channels per
  // workgroup and with c split as far as it goes, else the narrowest)
  int tq = 32, tp = 4;
  int64_t area = -1;
  bool enough = false;
  for (int t : {32, 16, 8}) {
    const int rows = t == 32 ? 4 : 8;
    const int64_t a = cdiv(P, rows) * rows * cdiv(Q, t) * t;
    int smax = 1;  // parts the reduction dimension c can be split into (at least one chunk each)
    while (smax < 8 && s[4] / (2 * smax) >= 16) smax *= 2;
    const bool many = (s[0] > 0 ? s[0] : 1) * cdiv(P, rows) * cdiv(Q, t) * cdiv(s[3] > 0 ? s[3] : 1, 64) * smax >= 512;
    if (area < 0 || a < area || (a == area && !enough)) area = a, tq = t, tp = rows, enough = many;
  }
  const int wm = tq == 8 ? 32 : 64;  // two blocks along p per wavefront, one for the 4 x 8 block
  MccPlan pl{tp, tq, 128, 16, wm, 64, 0, 0};
  if (s[3] <= 64) pl = MccPlan{tp, tq, 64, 16, wm, 32, 0, 0};
  // small images: narrower channel slices when there are fewer than two workgroups per compute unit
  // (16 x 28 x 28 x 128 -> 128, 3 x 3: 76 us against 124 us; 7 x 7 x 512: 283 against 462 us; fewer
  // rows per workgroup on top of that measured slower)
  auto wgs = [&](const MccPlan& m) {
    return (s[0] > 0 ? s[0] : 1) * cdiv(P, m.TP) * cdiv(Q, m.TQ) * cdiv(s[3] > 0 ? s[3] : 1, m.BN);
  };
  if (wgs(pl) < 512 && pl.BN == 128) pl = MccPlan{tp, tq, 64, 16, wm, 32, 0, 0};
  // still few workgroups: parts of the reduction dimension c over workgroups (partial outputs in the
  // workspace + second pass) up to ~450 workgroups, every part keeping at least one channel chunk.
  // 16 x 7 x 7 x 512 -> 512, 3 x 3: 85 us with 4 or 8 parts, 137 us with 2, 267 us unsplit (MIOpen
  // 118 us); 16 x 14 x 14 x 256 -> 256: 68 us with 4 parts, 80 with 2, 143 unsplit; 16 x 28 x 28 x 128
  // -> 128: 69 us with 2 parts, 73 with 4, 75 unsplit; 1 x 28 x 28 x 128: 15 us with 8 parts, 41 with 2.
  while (wgs(pl) * pl.S < 448 && pl.S < 8 && s[4] / (2 * pl.S) >= pl.CK) pl.S *= 2;
  // many channels per part: chunks of 32 channels, twice the MFMAs between two barriers (16 x 14 x 14
  // x 256 -> 256: 55.5 against 58.8 us; 16 x 7 x 7 x 2048 -> 512, 1 x 1: 37.5 against 44.3 us; with 32
  // channels in all, or 7 x 7 taps on 64, chunks of 16 are as fast or faster)
  if (s[4] / pl.S >= 128 || (s[4] / pl.S >= 64 && s[5] * s[6] <= 9)) {
    MccPlan w = pl;
    w.CK = 32;
    if (mcc_lds_bytes(w, s) <= kLdsBytesPerWG) pl = w;
  }
  // parts are whole channel chunks: no part may end up without channels (e.g. 200 channels in 8 parts)
  while (pl.S > 1 && (int64_t)(pl.S - 1) * cdiv(cdiv(s[4], pl.S), pl.CK) * pl.CK >= s[4]) pl.S /= 2;
  pl.ragged = mcc_ragged(s, pl);
  return pl;
}

// Microseconds that a filter tap of one channel chunk takes the workgroups a compute unit holds at once (index: how many,
// less one), per number of pixels, channels and CK of kMccSplitMenu; `full` is the share by which the clock gives way with
// all compute units at work.  A chunk's patch takes `patch` and `pixel` per hundred of its pixels, a call `once`.  Fitted to
// 160 random layers (16 to 512 channels, 1 x 1 to 7 x 7, stride 1 and 2, up to 4e10 operations), every tile in every number
// of parts on each: off by 6 to 8 % rms; the tile it picks takes 0.7 % longer on average than the fastest.
struct TapTime {
  int px, BN, CK, held;
  double once, patch, pixel, full, us[4];
};
static const TapTime kTap[] = {{64, 64, 16, 4, 4.7, 0.25, 0.313, 0.04, {0.292, 0.389, 0.565, 0.730}},
                               {64, 64, 32, 4, 4.6, 0.0, 0.779, 0.17, {0.310, 0.525, 0.725, 1.005}},
                               {64, 128, 16, 2, 4.9, 0.24, 0.315, 0.12, {0.326, 0.469}},
                               {64, 128, 32, 2, 5.1, 0.21, 0.656, 0.10, {0.582, 0.978}},
                               {128, 64, 16, 3, 5.1, 0.17, 0.308, 0.11, {0.339, 0.490, 0.739}},
                               {128, 64, 32, 3, 5.2, 0.12, 0.592, 0.16, {0.459, 0.761, 1.477}},
                               {128, 128, 16, 2, 6.1, 0.18, 0.319, 0.13, {0.469, 0.807}},
                               {128, 128, 32, 2, 6.2, 0.28, 0.591, 0.18, {0.837, 1.705}},
                               {256, 128, 16, 1, 7.6, 0.52, 0.148, 0.26, {0.753}},
                               {256, 128, 32, 1, 7.8, 0.0, 0.506, 0.25, {1.340}}};

// A coarser estimate, of 3 x 3 and 7 x 7 layers alone, which leans towards more parts of c: it has the least number of them.
static const TapTime kTapParts[] = {{64, 64, 16, 4, 0.0, 0.5, 0.11, 0.0, {0.319, 0.44, 0.605, 0.77}},
                                    {64, 64, 32, 4, 0.0, 0.5, 0.2, 0.0, {0.58, 0.80, 1.10, 1.40}},
                                    {64, 128, 16, 2, 0.0, 0.5, 0.11, 0.0, {0.44, 0.77}},
                                    {64, 128, 32, 2, 0.0, 0.5, 0.2, 0.0, {0.80, 1.40}},
                                    {128, 64, 16, 3, 0.0, 0.5, 0.11, 0.0, {0.385, 0.715, 1.045}},
                                    {128, 64, 32, 3, 0.0, 0.5, 0.2, 0.0, {0.70, 1.30, 1.90}},
                                    {128, 128, 16, 2, 0.0, 0.5, 0.11, 0.0, {0.77, 1.32}},
                                    {128, 128, 32, 2, 0.0, 0.5, 0.2, 0.0, {1.40, 2.40}},
                                    {256, 128, 16, 1, 0.0, 0.5, 0.11, 0.0, {1.1935}},
                                    {256, 128, 32, 1, 0.0, 0.5, 0.2, 0.0, {2.17}}};

// second pass: microseconds, per part, per 10^6 of the outputs' partial results and outputs
struct SecondPass {
  double once, part, output;
};

static double mcc_split_estimate(const int64_t* s, const MccPlan& pl, const TapTime* t, const SecondPass& pass) {
  const int64_t P = s[1] > 0 ? s[1] : 1, Q = s[2] > 0 ? s[2] : 1, N = s[0] > 0 ? s[0] : 1, K = s[3] > 0 ? s[3] : 1;
  while (t->px != pl.TP * pl.TQ || t->BN != pl.BN || t->CK != pl.CK) ++t;
  const int64_t lds = kLdsBytesPerWG / mcc_lds_bytes(pl, s);
  const int held = (int)(lds < t->held ? lds : t->held);
  const int64_t work = N * cdiv(P, pl.TP) * cdiv(Q, pl.TQ) * cdiv(K, pl.BN) * pl.S;
  const int64_t npix = ((pl.TP - 1) * s[7] + s[5]) * ((pl.TQ - 1) * s[8] + s[6]);
  const int64_t chunks = cdiv(cdiv(s[4], pl.S), pl.CK);
  auto round = [&](int r) {
    return chunks * (s[5] * s[6] * t->us[r - 1] + (t->patch + t->pixel * npix / 100) * (1 + 0.3 * (r - 1)));
  };
  double us = t->once + (double)(work / (256 * held)) * round(held) * (1 + t->full);
  const int64_t rest = work % (256 * held);
  if (rest) us += round((int)cdiv(rest, 256)) * (1 + t->full * (rest < 256 ? rest : 256) / 256);
  if (pl.S > 1) us += pass.once + pass.part * pl.S + (double)(pl.S + 1) * N * P * Q * K * pass.output * 1e-6;
  return us;
}

// Which tile of the split kernel the default is.  The fp32 rule's pixel block (TQ) is kept unless another is 3 % faster by
// the estimate (16 x 56 x 56 x 64 -> 64, 3 x 3: 30.6 with blocks of 4 x 8, 30.1 with 2 x 16).  `S` is the number of parts
// the fp32 rule splits c into: not more parts here, so that no call needs more workspace than it does there.  It is ahead of the fp32 kernels on every
// layer measured from 16 channels on (us, against theirs): 16 x 224 x 224 x 64 -> 128, 7 x 7: 2766 / 4829; 16 x 56 x
// 56 x 64 -> 64, 3 x 3: 28.8 / 51.1; 1 x 1, 256 -> 64: 21.5 / 29.6; 32 x 7 x 7 x 512 -> 512, 3 x 3: 67.5 / 109;
// 1 x 18 x 19 x 40 -> 33: 10.5 / 14.8.  Below 16 channels a chunk is mostly padding, and a reduction of less than 128 terms
// is all first and last tap (1 x 1, 64 -> 256: 29.0 / 27.8), as is a small layer of one tap (9 x 5 x 5 x 136 -> 92: 12.8
// / 12.2).  Of 400 random layers of stride 2 to 5, where much of a patch is split and not used, 1.5 % are slower by more
// than 4 % (26 x 3 x 1 x 665 -> 9, 2 x 1, stride 4: 32 / 37), the mean is 0.73.
static bool mcc_split_default(const int64_t* s, int TQ, int S, MccPlan* out) {
  if (s[4] * s[5] * s[6] < 128) return false;
  if (s[5] * s[6] == 1 && (double)s[0] * s[1] * s[2] * s[3] * s[4] < (double)(1 << 24)) return false;
  // the fastest tile in `least` parts of c or more; `other`: what another pixel block counts for
  auto fastest = [&](const TapTime* t, const SecondPass& pass, int least, double other) {
    double best = -1;
    for (auto& m : kMccSplitMenu)
      for (int parts = least; parts <= S; parts *= 2) {
        MccPlan pl{m.TP, m.TQ, m.BN, m.CK, m.WM, m.WN, 0, 0};
        pl.S = parts;
        pl.split = 1;
        if (pl.TQ != TQ && other < 1) continue;
        if (!mcc_split_sizes(s, pl) || mcc_lds_bytes(pl, s) > kLdsBytesPerWG) continue;
        const double us = mcc_split_estimate(s, pl, t, pass) * (pl.TQ == TQ ? 1.0 : other);
        if (best < 0 || us < best) best = us, *out = pl;
      }
    return best >= 0;
  };
  // A part twice as long is 1.4 times as far from 64 bits, so not fewer parts than the coarser estimate has, though the
  // other one would take fewer on 7 % of random layers and be 3 % faster there (35 of them: 0.71 of the error; 5 x 19 x 24,
  // 121 -> 235, 3 x 3: four parts; 3 x 55 x 56, 180 -> 51, 5 x 5: 55.2 us and 9.0 x 2^-24 in four, 48.6 and 12.7 in two).
  const int least = S > 1 && fastest(kTapParts, {3.0, 0.5, 1.0}, 1, 0.0) ? out->S : 1;
  return fastest(kTap, {0.4, 0.3, 2.3}, least, 1.03);
}

// the few-channel kernel that splits addresses an image with 32 bits (a stride that is not used may have any value: the
// product of what the sizes allow is no whole number of 64 bits)
static bool mcc_flat_split_sizes(const int64_t* s) {
  const double rows = (double)(s[1] > 0 ? s[1] : 1) * s[7] + s[5], columns = (double)(s[2] > 0 ? s[2] : 1) * s[8] + s[6];
  return flat_input_ok(s) && rows * columns * s[4] < (double)(1 << 28);
}

// Does a call without a table go to the few-channel kernel that splits, and in which block?  (The default's table stays
// that of the fp32 instructions: bit for bit the results it always had.)
// The line: its matrix instructions have to take at most two thirds of the time of the fp32 ones, nine tenths where there
// are fewer than 2^24 outputs.  us, against those, at 16 x 224 x 224 -> 64 / the same with stride 2 / 8 x 70 x 90 -> 24:
//   7 x 7 x 3 (0.57) 127 : 143 / 39 : 45 / 11.2 : 12.1     3 x 3 x 4 (0.67) 57 : 58 / 19.9 : 23.3 / 7.0 : 9.0
//   5 x 5 x 4 (0.64) 101 : 106 / 31 : 37 / 9.5 : 13.0      3 x 3 x 3 (0.80) 59 : 54 / 19.9 : 21.5 / 7.0 : 8.8
//   5 x 5 x 2 (0.80) 74 : 68 / 23 : 26 / 8.1 : 10.2        3 x 3 x 2 (0.89) 50 : 45 / 18.0 : 17.4 / 6.6 : 7.5
// one image of 230 x 230 x 3 -> 64, 7 x 7, stride 2: 8.8 : 9.0.  Below 18 terms the outputs' stores are most of a call (3 x
// 3 x 1: 51 : 43).  64 channels a wavefront share the split of the input, 32 leave more wavefronts: one image of the first
// layer 7.6 with 32, 10.4 with 64 (with six products).
static void mcc_flat_split_rule(const int64_t* s, MccPlan* out) {
  if (!mcc_flat_split_sizes(s)) return;
  const int64_t P = s[1] > 0 ? s[1] : 1, Q = s[2] > 0 ? s[2] : 1, SC = s[6] * s[4];
  // cycles of the matrix instructions of 32 pixels x 32 channels
  const int64_t split = cdiv(s[5] * cdiv(SC, 8), 2) * 8 * 32, fp32 = s[5] * (SC / 8 * 4 + cdiv(SC % 8, 2)) * 64;
  const bool few = (double)s[0] * P * Q * s[3] < (double)(1 << 24);
  if (s[5] * SC < 18 || split * 30 > fp32 * (few ? 27 : 20)) return;
  int64_t area = -1;
  int tq = 0;
  for (int t : {16, 32, 8}) {  // the block that pads the image least
    const int64_t a = cdiv(P, 32 / t) * (32 / t) * cdiv(Q, t) * t;
    if (area < 0 || a < area) area = a, tq = t;
  }
  const int bn = s[3] > 32 && s[0] * area / 32 >= 2048 ? 64 : 32;
  MccPlan pl{32 / tq, tq, bn, 0, 32, bn, 0, 1};
  pl.split = 1;
  pl.ragged = mcc_ragged(s, pl);
  if (mcc_lds_bytes(pl, s) <= kLdsBytesPerWG) *out = pl;
}

// on slices in at most `most` parts of c
static MccPlan mcc_default(const int64_t* s, int64_t most = 1 << 20) {
  MccPlan pl = mcc_default_fp32(s);
  if (!pl.flat && mcc_split_default(s, pl.TQ, pl.S < most ? pl.S : (int)most, &pl)) pl.ragged = mcc_ragged(s, pl);
  return pl;
}

MccPlan mcc_default_table(const int64_t* s) { return mcc_default(s); }

MccPlan mcc_default_lean(const int64_t* s, size_t workspace) { return mcc_default(s, parts_held(workspace, s[0] * s[1] * s[2] * s[3])); }

int mcc_candidates(const int64_t* s, MccPlan* out, int cap) {
  int n = 0;
  auto push = [&](MccPlan pl) {
    if (n >= cap) return;
    if (mcc_lds_bytes(pl, s) > kLdsBytesPerWG) return;
    pl.ragged = mcc_ragged(s, pl);
    for (int i = 0; i < n; ++i)
      if (out[i].flat == pl.flat && out[i].TP == pl.TP && out[i].TQ == pl.TQ && out[i].BN == pl.BN && out[i].CK == pl.CK &&
          out[i].WM == pl.WM && out[i].WN == pl.WN && out[i].QT == pl.QT && out[i].S == pl.S && out[i].dealt == pl.dealt && out[i].split == pl.split)
        return;
    out[n++] = pl;
  };
  push(mcc_default(s));
  push(mcc_default_fp32(s));
  for (auto& m : kMccMenu) push(MccPlan{m.TP, m.TQ, m.BN, m.CK, m.WM, m.WN, 0, 0});
  for (int S : {1, 2, 4, 8})
    for (auto& m : kMccSplitMenu) {
      MccPlan pl{m.TP, m.TQ, m.BN, m.CK, m.WM, m.WN, 0, 0};
      pl.S = S;
      pl.split = 1;
      const int64_t wg = (s[0] > 0 ? s[0] : 1) * cdiv(s[1] > 0 ? s[1] : 1, m.TP) * cdiv(s[2] > 0 ? s[2] : 1, m.TQ) *
                         cdiv(s[3] > 0 ? s[3] : 1, m.BN);
      if ((S > 1 && wg * (S / 2) >= 512) || !mcc_split_sizes(s, pl)) continue;
      push(pl);
    }
  // the reduction dimension c over workgroups, where the concatenation dimensions leave the chip empty
  for (int S : {2, 4, 8})
    for (auto& m : kMccMenu) {
      MccPlan pl{m.TP, m.TQ, m.BN, m.CK, m.WM, m.WN, 0, 0};
      pl.S = S;
      const int64_t wg = (s[0] > 0 ? s[0] : 1) * cdiv(s[1] > 0 ? s[1] : 1, m.TP) * cdiv(s[2] > 0 ? s[2] : 1, m.TQ) *
                         cdiv(s[3] > 0 ? s[3] : 1, m.BN);
      if (wg * (S / 2) >= 1024 || (int64_t)(S - 1) * cdiv(cdiv(s[4], S), m.CK) * m.CK >= s[4]) continue;
      push(pl);
    }
  if (s[4] <= 16 && flat_input_ok(s))
    for (int want : {1, 2, 4, 8, 16})
      for (auto& m : kMccFlatMenu) {
        MccPlan pl{m.TP, m.TQ, m.BN, m.CK, m.WM, m.WN, 0, 1};
        const int64_t tiles = cdiv(s[2] > 0 ? s[2] : 1, pl.TQ);
        const int64_t qt = want < tiles ? want : tiles;
        pl.QT = (int)cdiv(tiles, cdiv(tiles, qt));
        push(pl);
        if (want == 1 && cdiv(s[3] > 0 ? s[3] : 1, pl.BN) <= 8) {  // the same tile, dealt out
          pl.dealt = 1;
          push(pl);
        }
      }
  if (s[4] <= 16 && mcc_flat_split_sizes(s))
    for (auto& m : kMccFlatSplitMenu) {
      MccPlan pl{m.TP, m.TQ, m.BN, m.CK, m.WM, m.WN, 0, 1};
      pl.split = 1;
      push(pl);
    }
  return n;
}

mdh_status plan_mcc(const int64_t* s, const mdh_tile_params* p, MccPlan* out) {
  if (!p) {
    *out = mcc_default(s);
    if (mcc_lds_bytes(*out, s) > kLdsBytesPerWG) return MDH_ERR_TILE_RESOURCES;
    if (out->flat) mcc_flat_split_rule(s, out);
    return MDH_OK;
  }
  if (p->D != 7) return MDH_ERR_UNSUPPORTED;
  bool ragged;
  mdh_status st = check_products(p, s, &ragged);
  if (st != MDH_OK) return st;
  if ((st = check_lanes(p)) != MDH_OK) return st;
  MccPlan pl;
  pl.flat = p->blk[4] == 1 ? 1 : 0;
  pl.WN = p->prt[MDH_L_VGPR][3] * 32;
  pl.BN = p->prt[MDH_L_WAVE][3] * pl.WN;
  if (pl.flat) {
    pl.TQ = p->blk[2];
    pl.split = p->in_region[0] == MDH_MR_HBM;
    if ((pl.TQ != 16 && pl.TQ != 32 && !(pl.split && pl.TQ == 8)) || !flat_input_ok(s)) return MDH_ERR_UNSUPPORTED;
    if (pl.split && (!mcc_flat_split_sizes(s) || p->strided || p->prt[MDH_L_HBM][2] != 1)) return MDH_ERR_UNSUPPORTED;
    // tiles beyond any LDS, and beyond 32 bits further on
    if (p->prt[MDH_L_VGPR][3] > 4096 || p->prt[MDH_L_WAVE][3] > 4096) return MDH_ERR_TILE_RESOURCES;
    if (p->prt[MDH_L_VGPR][1] > 4096 || p->prt[MDH_L_WAVE][1] > 4096) return pl.split ? MDH_ERR_UNSUPPORTED : MDH_ERR_TILE_RESOURCES;
    pl.WM = p->prt[MDH_L_VGPR][1] * 32;
    pl.TP = p->prt[MDH_L_WAVE][1] * p->prt[MDH_L_VGPR][1] * (32 / pl.TQ);
    pl.CK = 0;
    pl.QT = p->prt[MDH_L_HBM][2];
    pl.dealt = p->strided ? 1 : 0;
    // dealt tiles: one column tile per part, at most 8 filter slices (one ticket counter each)
    if (pl.dealt && (pl.QT != 1 || p->prt[MDH_L_WG][3] > 8)) return MDH_ERR_UNSUPPORTED;
    // a workgroup part of q that owns no tile is not a partition of the columns
    if ((int64_t)(p->prt[MDH_L_WG][2] - 1) * pl.QT * pl.TQ >= (s[2] > 0 ? s[2] : 1)) return MDH_ERR_TILE_NOT_DIVIDING;
  } else {
    pl.TQ = p->blk[2];
    if (pl.TQ != 8 && pl.TQ != 16 && pl.TQ != 32) return MDH_ERR_UNSUPPORTED;
    pl.WM = p->prt[MDH_L_VGPR][1] * 32;
    pl.TP = p->prt[MDH_L_WAVE][1] * p->prt[MDH_L_VGPR][1] * (32 / pl.TQ);
    pl.split = p->prt[MDH_L_VGPR][4] == 8;
    // chunks beyond any LDS, and beyond 32 bits here
    if (p->prt[MDH_L_LDS][4] > 4096 || p->prt[MDH_L_VGPR][4] > 4096) return MDH_ERR_TILE_RESOURCES;
    pl.CK = p->prt[MDH_L_LDS][4] * 2 * p->prt[MDH_L_VGPR][4];
    pl.S = p->prt[MDH_L_WG][4];
    // a workgroup part of c that owns no channel would leave its partial output unset
    if (pl.S > 1 && pl.CK > 0 && (int64_t)(pl.S - 1) * cdiv(cdiv(s[4], pl.S), pl.CK) * pl.CK >= s[4])
      return MDH_ERR_TILE_NOT_DIVIDING;
    if (pl.split && (!mcc_inst(pl) || !mcc_split_sizes(s, pl))) return MDH_ERR_UNSUPPORTED;
  }
  pl.ragged = ragged;
  if (mcc_lds_bytes(pl, s) > kLdsBytesPerWG) return MDH_ERR_TILE_RESOURCES;
  mdh_tile_params chk;
  params_from_plan(s, pl, &chk);
  if (!same_table(chk, *p) || !mcc_inst(pl)) return MDH_ERR_UNSUPPORTED;
  *out = pl;
  return MDH_OK;
}

// =============================================================================== custom reduce

static bool prl_inst(const PrlPlan& pl) {
  static const int menu[][3] = {{2, 4, 1}, {4, 4, 1}, {1, 4, 1}, {2, 2, 2}, {4, 2, 2},
                                {2, 1, 4}, {4, 1, 4}, {2, 8, 1}, {4, 8, 1}};
  for (auto& m : menu)
    if (m[0] == pl.RA && m[1] == pl.WB && m[2] == pl.WA) return true;
  return false;
}

void params_from_plan(const int64_t* s, const PrlPlan& pl, mdh_tile_params* p) {
  clear_params(p, 2);
  p->prt[MDH_L_WG][0] = (int32_t)cdiv(s[0], (int64_t)pl.WA * 64 * pl.RA);
  p->prt[MDH_L_WG][1] = pl.S;
  p->prt[MDH_L_WAVE][0] = pl.WA;
  p->prt[MDH_L_WAVE][1] = pl.WB;
  p->prt[MDH_L_LANE][0] = 64;
  p->prt[MDH_L_VGPR][0] = pl.RA;
  p->prt[MDH_L_HBM][1] = (int32_t)cdiv(s[1], (int64_t)pl.S * pl.WB);
  static const int dims[2] = {0, 1};
  set_order(p, dims);
  p->strided = 0;
  p->lane_fast_dim = 0;
  p->in_region[0] = MDH_MR_VGPR;  // a lane's records of A stay in registers
  p->in_region[1] = MDH_MR_HBM;   // records of B are wavefront-uniform: scalar loads, no staging
  p->out_region = MDH_MR_VGPR;
  p->ragged = (uint8_t)pl.ragged;
}

static int prl_ragged(const int64_t* s, const PrlPlan& pl) {
  return (s[0] % ((int64_t)pl.WA * 64 * pl.RA)) || (s[1] % ((int64_t)pl.S * pl.WB));
}

static PrlPlan prl_default(const int64_t* s) {
  // two records of A per lane, four wavefronts along b (2^16 x 2^18, 8 fields: 7.04 ms with 32 parts of
  // b over workgroups, 7.22 with 16; eight wavefronts along b: 7.42 / 7.51; four records per lane: 7.16)
  PrlPlan pl{2, 4, 1, 1, 0};
  const int64_t wgs_a = cdiv(s[0], (int64_t)pl.WA * 64 * pl.RA);
  int S = 1;
  // split B over workgroups until there are ~64 wavefronts per SIMD of the chip to draw from
  // (2^16 x 2^18: 10.35 ms with 4 parts, 10.0 with 8, 9.8 with 16, 9.75 with 32) while a wavefront
  // keeps 256 records of B; with few records of A first of all a workgroup per compute unit, down to
  // 32 records of B per wavefront (2^10 x 2^14: 30 us with 32 parts, 41 with 16, 69 with 8;
  // 2^8 x 2^18: 104 us with 128 parts, 129 with 256)
  while (wgs_a * S < 256 && S < 256 && s[1] / (2ll * S * pl.WB) >= 32) S *= 2;
  while (wgs_a * S * pl.WB * pl.WA < 65536 && S < 256 && s[1] / (2ll * S * pl.WB) >= 256) S *= 2;
  pl.S = S;
  pl.ragged = prl_ragged(s, pl);
  return pl;
}

int prl_candidates(const int64_t* s, PrlPlan* out, int cap) {
  int n = 0;
  auto push = [&](PrlPlan pl) {
    if (n >= cap) return;
    if (s[1] / ((int64_t)pl.S * pl.WB) < 1) return;
    pl.ragged = prl_ragged(s, pl);
    for (int i = 0; i < n; ++i)
      if (out[i].RA == pl.RA && out[i].WB == pl.WB && out[i].WA == pl.WA && out[i].S == pl.S) return;
    out[n++] = pl;
  };
  PrlPlan d = prl_default(s);
  push(d);
  static const int menu[][3] = {{2, 4, 1}, {4, 4, 1}, {1, 4, 1}, {2, 2, 2}, {4, 2, 2},
                                {2, 1, 4}, {4, 1, 4}, {2, 8, 1}, {4, 8, 1}};
  for (auto& m : menu)
    for (int S = d.S / 2 > 0 ? d.S / 2 : 1; S <= d.S * 2; S *= 2) push(PrlPlan{m[0], m[1], m[2], S, 0});
  return n;
}

mdh_status plan_prl(const int64_t* s, const mdh_tile_params* p, PrlPlan* out) {
  if (!p) {
    *out = prl_default(s);
    return MDH_OK;
  }
  if (p->D != 2) return MDH_ERR_UNSUPPORTED;
  bool ragged;
  mdh_status st = check_products(p, s, &ragged);
  if (st != MDH_OK) return st;
  if ((st = check_lanes(p)) != MDH_OK) return st;
  PrlPlan pl;
  pl.RA = p->prt[MDH_L_VGPR][0];
  pl.WA = p->prt[MDH_L_WAVE][0];
  pl.WB = p->prt[MDH_L_WAVE][1];
  pl.S = p->prt[MDH_L_WG][1];
  pl.ragged = ragged;
  mdh_tile_params chk;
  params_from_plan(s, pl, &chk);
  if (!same_table(chk, *p) || !prl_inst(pl)) return MDH_ERR_UNSUPPORTED;
  *out = pl;
  return MDH_OK;
}

}  // namespace mdh

// =============================================================================== C ABI (host-only part)

using namespace mdh;

extern "C" {

const char* mdh_strerror(mdh_status s) {
  switch (s) {
    case MDH_OK: return "ok";
    case MDH_ERR_NULL: return "a required pointer is NULL";
    case MDH_ERR_SIZE: return "invalid size (negative, empty reduction dimension, or beyond 2^31-1 elements)";
    case MDH_ERR_TILE_NOT_DIVIDING: return "tile parameters violate prod_l #PRT(l,d) * blk[d] == N_d";
    case MDH_ERR_TILE_RESOURCES: return "tile parameters exceed lanes-per-workgroup or LDS budget";
    case MDH_ERR_WORKSPACE: return "workspace missing or too small for the split reduction";
    case MDH_ERR_UNSUPPORTED: return "no kernel instantiation for this configuration";
    case MDH_ERR_LAUNCH: return "HIP launch failed";
    case MDH_ERR_STATIC_LIMIT: return "the call needs more scratch memory than the library's static buffer holds";
  }
  return "unknown status";
}

const char* mdh_version(void) { return "0.1"; }

mdh_status mdh_part_offset(int64_t N, int32_t L, const int32_t* P, const int32_t* p,
                           int64_t* offset, int64_t* part_size) {
  if (!P || !p || !offset || !part_size) return MDH_ERR_NULL;
  if (N < 0 || L < 0) return MDH_ERR_SIZE;
  int64_t prod = 1, os = 0;
  for (int l = 0; l < L; ++l) {
    if (P[l] < 1) return MDH_ERR_TILE_NOT_DIVIDING;
    if (p[l] < 0 || p[l] >= P[l]) return MDH_ERR_SIZE;
    prod *= P[l];
    if (N % prod) return MDH_ERR_TILE_NOT_DIVIDING;
    os += (int64_t)p[l] * (N / prod);
  }
  *offset = os;
  *part_size = N / prod;
  return MDH_OK;
}

static mdh_status check_sizes(mdh_instance inst, const int64_t* s) {
  if (!s) return MDH_ERR_NULL;
  const int D = (inst == MDH_MCC || inst == MDH_MCC_CAPSULE) ? 9 : (inst == MDH_CUSTOM_REDUCE || inst == MDH_MATVEC || inst == MDH_SCAN) ? 2
                                  : inst == MDH_DOT ? 1 : inst == MDH_BMATMUL ? 7 : 3;
  for (int d = 0; d < D; ++d)
    if (s[d] < 0 || s[d] > 0x7fffffff) return MDH_ERR_SIZE;
  switch (inst) {
    case MDH_DOT:
      if (s[0] < 1) return MDH_ERR_SIZE;
      break;
    case MDH_BMATMUL:
      if (s[3] < 1 || s[0] > 65535 || s[4] > 1 || s[5] > 1 || s[6] > 1) return MDH_ERR_SIZE;
      break;
    case MDH_MATVEC:
      if (s[1] < 1) return MDH_ERR_SIZE;
      break;
    case MDH_MATMUL:
      if (s[2] < 1) return MDH_ERR_SIZE;
      break;
    case MDH_STENCIL:
    case MDH_SCAN:
      break;
    case MDH_MCC:
    case MDH_MCC_CAPSULE:
      if (s[4] < 1 || s[5] < 1 || s[6] < 1 || s[7] < 1 || s[8] < 1) return MDH_ERR_SIZE;
      break;
    case MDH_CUSTOM_REDUCE:
      if (s[1] < 1) return MDH_ERR_SIZE;
      break;
    default:
      return MDH_ERR_UNSUPPORTED;
  }
  return MDH_OK;
}

mdh_status mdh_default_params(mdh_instance inst, const int64_t* sizes, mdh_tile_params* out) {
  if (!out) return MDH_ERR_NULL;
  mdh_status st = check_sizes(inst, sizes);
  if (st != MDH_OK) return st;
  switch (inst) {
    case MDH_MATMUL: {
      if (small_m_matmul(sizes, nullptr)) {
        GemmExPlan ex;
        if ((st = plan_small_m(sizes, nullptr, &ex)) != MDH_OK) return st;
        const int64_t s4[7] = {1, sizes[0], sizes[1], sizes[2], 0, 0, 0};
        mdh_tile_params p4;
        params_from_plan(s4, ex, &p4);
        drop_batch(p4, out);
        return MDH_OK;
      }
      GemmPlan pl;
      if ((st = plan_matmul(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
    case MDH_STENCIL: {
      StencilPlan pl;
      if ((st = plan_stencil(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
    case MDH_MCC: {
      MccPlan pl;
      if ((st = plan_mcc(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, mcc_default_table(sizes), out);
      return st;
    }
    case MDH_CUSTOM_REDUCE: {
      PrlPlan pl;
      if ((st = plan_prl(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
    case MDH_DOT: {
      DotPlan pl;
      if ((st = plan_dot(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
    case MDH_BMATMUL: {
      GemmExPlan pl;
      if ((st = plan_matmul_ex(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
    case MDH_MATVEC: {
      MatVecPlan pl;
      if ((st = plan_matvec(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
    case MDH_SCAN: {
      ScanPlan pl;
      if ((st = plan_scan(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
    case MDH_MCC_CAPSULE: {
      CapsulePlan pl;
      if ((st = plan_capsule(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
      return st;
    }
  }
  return MDH_ERR_UNSUPPORTED;
}

mdh_status mdh_call_params(mdh_instance inst, const int64_t* sizes, mdh_tile_params* out) {
  mdh_status st = mdh_default_params(inst, sizes, out);
  MccPlan pl;
  if (st == MDH_OK && inst == MDH_MCC && (st = plan_mcc(sizes, nullptr, &pl)) == MDH_OK) params_from_plan(sizes, pl, out);
  return st;
}

mdh_status mdh_validate_params(mdh_instance inst, const int64_t* sizes, const mdh_tile_params* p) {
  if (!p) return MDH_ERR_NULL;
  mdh_status st = check_sizes(inst, sizes);
  if (st != MDH_OK) return st;
  switch (inst) {
    case MDH_MATMUL: {
      if (small_m_matmul(sizes, p)) {
        GemmExPlan ex;
        return plan_small_m(sizes, p, &ex);
      }
      GemmPlan pl;
      return plan_matmul(sizes, p, &pl);
    }
    case MDH_STENCIL: {
      StencilPlan pl;
      return plan_stencil(sizes, p, &pl);
    }
    case MDH_MCC: {
      MccPlan pl;
      return plan_mcc(sizes, p, &pl);
    }
    case MDH_CUSTOM_REDUCE: {
      PrlPlan pl;
      return plan_prl(sizes, p, &pl);
    }
    case MDH_DOT: {
      DotPlan pl;
      return plan_dot(sizes, p, &pl);
    }
    case MDH_BMATMUL: {
      GemmExPlan pl;
      return plan_matmul_ex(sizes, p, &pl);
    }
    case MDH_MATVEC: {
      MatVecPlan pl;
      return plan_matvec(sizes, p, &pl);
    }
    case MDH_SCAN: {
      ScanPlan pl;
      return plan_scan(sizes, p, &pl);
    }
    case MDH_MCC_CAPSULE: {
      CapsulePlan pl;
      return plan_capsule(sizes, p, &pl);
    }
  }
  return MDH_ERR_UNSUPPORTED;
}

size_t mdh_workspace_size(mdh_instance inst, const int64_t* sizes, const mdh_tile_params* params) {
  if (check_sizes(inst, sizes) != MDH_OK) return 0;
  switch (inst) {
    case MDH_MATMUL: {
      if (small_m_matmul(sizes, params)) {
        GemmExPlan ex;
        if (plan_small_m(sizes, params, &ex) != MDH_OK || ex.g.S <= 1) return 0;
        return (size_t)ex.g.S * (size_t)sizes[0] * (size_t)sizes[1] * sizeof(float);
      }
      GemmPlan pl;
      if (plan_matmul(sizes, params, &pl) != MDH_OK || pl.S <= 1) return 0;
      return (size_t)pl.S * (size_t)sizes[0] * (size_t)sizes[1] * sizeof(float);
    }
    case MDH_MCC: {
      MccPlan pl;
      if (plan_mcc(sizes, params, &pl) != MDH_OK || pl.flat || pl.S <= 1) return 0;
      return (size_t)pl.S * (size_t)(sizes[0] * sizes[1] * sizes[2] * sizes[3]) * sizeof(float);
    }
    case MDH_CUSTOM_REDUCE: {
      PrlPlan pl;
      if (plan_prl(sizes, params, &pl) != MDH_OK || pl.S <= 1) return 0;
      return (size_t)pl.S * (size_t)sizes[0] * 2 * sizeof(int32_t);
    }
    case MDH_DOT: {
      DotPlan pl;
      if (plan_dot(sizes, params, &pl) != MDH_OK || pl.S <= 1) return 0;
      return (size_t)pl.S * sizeof(float);
    }
    case MDH_BMATMUL: {
      GemmExPlan pl;
      if (plan_matmul_ex(sizes, params, &pl) != MDH_OK || pl.g.S <= 1) return 0;
      return (size_t)pl.g.S * (size_t)sizes[0] * (size_t)sizes[1] * (size_t)sizes[2] * sizeof(float);
    }
    case MDH_MATVEC: {
      MatVecPlan pl;
      if (plan_matvec(sizes, params, &pl) != MDH_OK || pl.S <= 1) return 0;
      return (size_t)pl.S * (size_t)sizes[0] * sizeof(float);
    }
    case MDH_SCAN: {
      ScanPlan pl;
      if (plan_scan(sizes, params, &pl) != MDH_OK) return 0;
      return scan_workspace_bytes(pl, sizes[0]);
    }
    default:
      return 0;
  }
}

int32_t mdh_num_candidates(mdh_instance inst, const int64_t* sizes) {
  if (check_sizes(inst, sizes) != MDH_OK) return 0;
  constexpr int CAP = 128;
  switch (inst) {
    case MDH_MATMUL: {
      GemmPlan c[CAP];
      return matmul_candidates(sizes, c, CAP);
    }
    case MDH_STENCIL: {
      StencilPlan c[CAP];
      return stencil_candidates(sizes, c, CAP);
    }
    case MDH_MCC: {
      MccPlan c[CAP];
      return mcc_candidates(sizes, c, CAP);
    }
    case MDH_CUSTOM_REDUCE: {
      PrlPlan c[CAP];
      return prl_candidates(sizes, c, CAP);
    }
    case MDH_DOT: {
      DotPlan c[CAP];
      return dot_candidates(sizes, c, CAP);
    }
    case MDH_BMATMUL: {
      GemmExPlan c[CAP];
      return matmul_ex_candidates(sizes, c, CAP);
    }
    case MDH_MATVEC: {
      MatVecPlan c[CAP];
      return matvec_candidates(sizes, c, CAP);
    }
    case MDH_SCAN: {
      ScanPlan c[CAP];
      return scan_candidates(sizes, c, CAP);
    }
    case MDH_MCC_CAPSULE: {
      CapsulePlan c[CAP];
      return capsule_candidates(sizes, c, CAP);
    }
  }
  return 0;
}

mdh_status mdh_candidate(mdh_instance inst, const int64_t* sizes, int32_t idx, mdh_tile_params* out) {
  if (!out) return MDH_ERR_NULL;
  mdh_status st = check_sizes(inst, sizes);
  if (st != MDH_OK) return st;
  constexpr int CAP = 128;
  switch (inst) {
    case MDH_MATMUL: {
      GemmPlan c[CAP];
      int n = matmul_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      // candidate 0 is the default: for few rows the small-M kernel, which the tiled menu does not hold
      if (idx == 0 && small_m_matmul(sizes, nullptr)) return mdh_default_params(inst, sizes, out);
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_STENCIL: {
      StencilPlan c[CAP];
      int n = stencil_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_MCC: {
      MccPlan c[CAP];
      int n = mcc_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_CUSTOM_REDUCE: {
      PrlPlan c[CAP];
      int n = prl_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_DOT: {
      DotPlan c[CAP];
      int n = dot_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_BMATMUL: {
      GemmExPlan c[CAP];
      int n = matmul_ex_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_MATVEC: {
      MatVecPlan c[CAP];
      int n = matvec_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_SCAN: {
      ScanPlan c[CAP];
      int n = scan_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
    case MDH_MCC_CAPSULE: {
      CapsulePlan c[CAP];
      int n = capsule_candidates(sizes, c, CAP);
      if (idx < 0 || idx >= n) return MDH_ERR_SIZE;
      params_from_plan(sizes, c[idx], out);
      return MDH_OK;
    }
  }
  return MDH_ERR_UNSUPPORTED;
}

}  // extern "C"
