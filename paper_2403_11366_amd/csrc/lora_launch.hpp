// Internal interface between the C ABI (argument checks, workspace layout) and
// the kernel launchers.  Shapes here have already been validated.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lora {

// Rank padded to the matrix-core granularity of 16 (r in 1..64 -> 16..64).
inline int pad_rank(int64_t r) { return (int)((r + 15) / 16) * 16; }

// Token count padded to the 64-token chunk of the split-K reductions.
inline int64_t pad_tokens(int64_t m) { return (m + 63) / 64 * 64; }

// Output tiles of the two large GEMMs (tokens x features): 256x256 runs 8
// waves (two per SIMD) as 2 x 4 waves of 128 x 64, the others 8 waves that
// split k.  Forward only: 128x128 shared by a pair of workgroups of 64 tokens
// each, and 128x128 staged in registers by four waves, two workgroups to a
// compute unit (TILE_REG).  dX only: 64x128 and 64x64, and 128x256 whose wave
// rows split the tokens (TILE_ROWS).
enum GemmTile {
  TILE_256x256 = 0, TILE_128x256 = 1, TILE_128x128 = 2, TILE_128x192 = 3, TILE_PAIR = 4, TILE_64x128 = 5, TILE_64x64 = 6,
  TILE_REG = 7, TILE_ROWS = 8
};

// A candidate tile: the output area a workgroup computes, and the workgroup's
// relative efficiency (larger tiles read less LDS and L2 per flop).  Every
// workgroup of these kernels fills one compute unit (LDS-limited), so a launch
// runs in ceil(workgroups / 256) rounds on 256 CUs, and its estimated cost is
// rounds x area / efficiency.
struct TileCost { GemmTile t; int bm, bn, wgs; double eff; };

// Forward tiles.  Time per 64-wide k stage with the chip full, measured at k =
// 4096 to 13824: 256x256 1.34 us, 128x256 0.85, 128x192 0.72, 128x128 0.55, a
// half of a pair 0.42.
constexpr TileCost kFwdTiles[5] = {{TILE_256x256, 256, 256, 1, 1.0}, {TILE_128x256, 128, 256, 1, 0.8},
                                   {TILE_128x128, 128, 128, 1, 0.61}, {TILE_128x192, 128, 192, 1, 0.71},
                                   {TILE_PAIR, 128, 128, 2, 0.4}};
// dX tiles (per 64-wide n stage with the chip full: 1.39 us, 0.77, 0.48, 0.61;
// with W read from memory and the chip part full 1.17, 0.80, 0.50, 0.67, and
// 0.39 and 0.28 of the 64-token tiles).
constexpr TileCost kDxTiles[6] = {{TILE_256x256, 256, 256, 1, 1.0}, {TILE_128x256, 128, 256, 1, 0.9},
                                  {TILE_128x128, 128, 128, 1, 0.72}, {TILE_128x192, 128, 192, 1, 0.82},
                                  {TILE_64x128, 64, 128, 1, 0.44},   {TILE_64x64, 64, 64, 1, 0.33}};
// Below kMidTileDepth contraction steps: 128x256 with nothing to exchange; it and
// 256x256, which has nothing to exchange either, gain 8% on the others.
constexpr TileCost kDxShallowTiles[5] = {{TILE_256x256, 256, 256, 1, 1.08}, {TILE_ROWS, 128, 256, 1, 0.97}, kDxTiles[2],
                                         kDxTiles[4], kDxTiles[5]};
// The tiles that have the dropout epilogue.
constexpr TileCost kDxDropTiles[5] = {kDxTiles[1], kDxTiles[2], kDxTiles[3], kDxTiles[4], kDxTiles[5]};
constexpr TileCost kDxDropShallowTiles[4] = {kDxShallowTiles[1], kDxTiles[2], kDxTiles[4], kDxTiles[5]};
// Tiles a call may take beside 256x256, 128x256, 128x128 and pairs.  128x192
// serves single projections of at least kMidTileDepth contraction steps (the
// forward's of fewer by estimated time, plan_fwd), and from there dX's 128x256
// splits k instead of tokens (equal at 33 to 64 stages).  Measured with 128x192
// open to all (500 drawn steps, the better plan of each call): groups 1.7%
// forward and 1.0% backward, single dX below kMidTileDepth 0.2%; groups have no
// kernel of it.  The 64-token tiles
// serve calls of few tokens, where the larger ones leave compute units idle: up to
// kFewTokens at any depth, up to kShortTokens from kShortDepth steps on.  (Whole
// backward call with the best of them against 128x128: 130 x 4096 x 4096 38 ->
// 29 us, 333 x 4096 x 4096 41 -> 36, 1024 x 4096 x 2048 54 -> 47, 256 x 512 x 512
// 16 -> 13; 257 x 1024 x 4096, outside, 19.6 and 18.1; above 1024 tokens an
// output of so few tiles has few columns.  Rounds of them past the first are no
// longer cheap: 296 x 5120 x 11008, r = 8 77.6 us on one round of 128x256, 85.7
// on two of 64x128.)
constexpr int64_t kMidTileDepth = 3072, kFewTokens = 256, kShortTokens = 1024, kShortDepth = 2048;
enum TileSet { TILES_BASE = 0, TILES_MID = 1, TILES_SHORT = 2 };
inline bool tile_allowed(GemmTile t, int set) {
  if (t == TILE_128x192) return set & TILES_MID;
  if (t == TILE_64x128 || t == TILE_64x64) return set & TILES_SHORT;
  return true;
}

inline int64_t tile_workgroups(const TileCost& c, int64_t M, int64_t N) {
  return (M + c.bm - 1) / c.bm * ((N + c.bn - 1) / c.bn) * c.wgs;
}
inline double tile_cost(const TileCost& c, int64_t M, int64_t N) {
  return (double)((tile_workgroups(c, M, N) + 255) / 256) * (c.bm * c.bn / c.wgs) / c.eff;
}

// The cheapest tile of a set for an M x N output (the first of equal ones).
template <int NT>
inline const TileCost& cheapest_tile(const TileCost (&cands)[NT], int64_t M, int64_t N, int set) {
  const TileCost* best = &cands[0];
  for (const TileCost& c : cands)
    if (tile_allowed(c.t, set) && tile_cost(c, M, N) < tile_cost(*best, M, N)) best = &c;
  return *best;
}

// Column split of one large GEMM with an M x N output: columns [0, n1) with
// tile t1, then columns [n1, N) with tile t2 in a second launch.  Taken when
// the split, whose second part is at most one round of 256 workgroups, is
// estimated more than 5% faster than the single tiling.
// Typical cases: 4096 x 5120, where 640 tiles of 128x256 take three rounds
// and 256 tiles of 256x256 plus 256 tiles of 128x128 take two; 4096 x 13824,
// where 1728 tiles of 128x256 take seven rounds and 768 tiles of 256x256 plus
// 192 of 128x256 take four (forward 607-616 -> 537 us).  The first part's cost
// depends on its rounds alone, so for each tile and number of rounds only the
// largest n1 is looked at.  n1 == N: no split.
struct GemmSplit { GemmTile t1, t2; int64_t n1; };
template <int NT>
inline GemmSplit plan_gemm_split(const TileCost (&cands)[NT], int64_t M, int64_t N, int set) {
  const TileCost& c0 = cheapest_tile(cands, M, N, set);
  GemmSplit best{c0.t, c0.t, N};
  double best_cost = 0.95 * tile_cost(c0, M, N);
  for (const TileCost& c1 : cands) {
    if (!tile_allowed(c1.t, set)) continue;
    const int64_t per_col = tile_workgroups(c1, M, 1);   // workgroups per column of tiles
    const int64_t rounds = (tile_workgroups(c1, M, N) + 255) / 256;
    for (int64_t R = 1; R <= rounds; ++R) {
      const int64_t n1 = 256 * R / per_col * c1.bn;
      if (n1 < c1.bn || n1 >= N) continue;
      for (const TileCost& c2 : cands) {
        if (!tile_allowed(c2.t, set) || tile_workgroups(c2, M, N - n1) > 256) continue;
        const double c = tile_cost(c1, M, n1) + tile_cost(c2, M, N - n1);
        if (c < best_cost || (c == best_cost && best.n1 < N && n1 > best.n1)) {
          best_cost = c;
          best = GemmSplit{c1.t, c2.t, n1};
        }
      }
    }
  }
  return best;
}

// Split-K plan of a token reduction out[t][c] = sum_i P[t][i] Q[i][c] over
// `cols` columns: columns in tiles of kRedCols, tokens in `splits` ranges of
// `span` tokens (a multiple of 64).  Splits are capped so the fp32 partial
// sums stay at most 1/8 of the bytes of Q (1/16 at rank 64, where fewer,
// longer splits measured faster: 7B down_proj backward 875 vs 891 us).
constexpr int kRedCols = 128;
struct RedPlan { int64_t span; int splits; int col_tiles; };
inline RedPlan plan_reduction(int64_t m, int64_t cols, int rp) {
  const int64_t mp = pad_tokens(m);
  const int col_tiles = (int)((cols + kRedCols - 1) / kRedCols);
  int64_t s = (1024 + col_tiles - 1) / col_tiles;
  int64_t cap = m / ((rp >= 64 ? 32 : 16) * (int64_t)rp);
  if (cap < 1) cap = 1;
  if (s > cap) s = cap;
  if (s > mp / 64) s = mp / 64;
  if (s < 1) s = 1;
  int64_t span = (mp + s - 1) / s;
  span = (span + 63) / 64 * 64;
  const int splits = (int)((mp + span - 1) / span);
  return RedPlan{span, splits, col_tiles};
}

// Backward workspace, byte offsets of each region (256-byte aligned).
struct BwdLayout {
  size_t ut2;    // Ut2  [RP][mp]     bf16: U^T
  size_t du2;    // dU2  [mp][2RP]    bf16: dU as high part (cols 0..RP) and low part
  size_t dut2;   // dUt2 [RP][mp]     bf16: s dU^T
  size_t pb;     // partial dB^T [splits_b][RP][n] fp32
  size_t pa;     // partial dA   [splits_a][RP][k] fp32
  size_t total;
  RedPlan plan_b, plan_a;
  int rp;
  int64_t mp;
};

inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }

inline BwdLayout bwd_layout(int64_t m, int64_t n, int64_t k, int64_t r) {
  BwdLayout L;
  L.rp = pad_rank(r);
  L.mp = pad_tokens(m);
  L.plan_b = plan_reduction(m, n, L.rp);
  L.plan_a = plan_reduction(m, k, L.rp);
  const size_t rp = (size_t)L.rp, mp = (size_t)L.mp;
  size_t off = 0;
  L.ut2 = off;  off = align256(off + rp * mp * 2);
  L.du2 = off;  off = align256(off + mp * 2 * rp * 2);
  L.dut2 = off; off = align256(off + rp * mp * 2);
  L.pb = off;   off = align256(off + (size_t)L.plan_b.splits * rp * (size_t)n * 4);
  L.pa = off;   off = align256(off + (size_t)L.plan_a.splits * rp * (size_t)k * 4);
  L.total = off;
  return L;
}

// Workspace of the fused backward (rank <= 16): dUt2 [16][mp] bf16 (s dU^T,
// written by the dX launch for the dA reduction), the dB^T
// partials of the dX launch [tiles_m][16][n] fp32 (one per 128-token tile
// row) and the dA partials of the token reduction [splits][16][k] fp32.
struct BwdFusedLayout {
  size_t dut2, pb, pa, total;
  RedPlan plan_a;
  int64_t mp;
  int tiles_m;
};

inline BwdFusedLayout bwd_fused_layout(int64_t m, int64_t n, int64_t k, int64_t r) {
  (void)r;
  BwdFusedLayout L;
  L.mp = pad_tokens(m);
  L.tiles_m = (int)((m + 127) / 128);
  L.plan_a = plan_reduction(m, k, 16);
  size_t off = 0;
  L.dut2 = off; off = align256(off + 16 * (size_t)L.mp * 2);
  L.pb = off;   off = align256(off + (size_t)L.tiles_m * 16 * (size_t)n * 4);
  L.pa = off;   off = align256(off + (size_t)L.plan_a.splits * 16 * (size_t)k * 4);
  L.total = off;
  return L;
}

struct FwdArgs {
  const uint16_t *X, *W, *A, *B;
  uint16_t* Y;
  float* U;
  int64_t m, n, k, r;
  float s;
  const uint8_t* keep = nullptr;   // dropout keep bits [m][k/8], or none
  float inv_keep = 1.0f;           // 1 / (1 - p)
};

struct BwdArgs {
  const uint16_t *dY, *X, *W, *A, *B;
  const float* U;
  uint16_t* dX;
  float *dA, *dB;
  char* ws;
  int64_t m, n, k, r;
  float s;
  const uint8_t* keep = nullptr;   // dropout keep bits [m][k/8], or none
  float inv_keep = 1.0f;           // 1 / (1 - p)
};

// Projections that share one input X (q, k, v of an attention block; gate and
// up of an MLP): at most kMaxGroup, one rank and alpha for the group.
constexpr int kMaxGroup = 8;

// Kernel argument (by value) of the grouped forward: per-projection pointers;
// the output tiles of all projections form one grid, projection g owning
// column tiles tile0[g] .. tile0[g+1]-1.
struct FwdGroup {
  const uint16_t* W[kMaxGroup];
  const uint16_t* A[kMaxGroup];
  const uint16_t* B[kMaxGroup];
  uint16_t* Y[kMaxGroup];
  float* U[kMaxGroup];
  int n[kMaxGroup];
  int tile0[kMaxGroup];
  int count;
};

struct GroupFwdArgs {
  const uint16_t* X;
  int count;
  int64_t n[kMaxGroup];
  const uint16_t *W[kMaxGroup], *A[kMaxGroup], *B[kMaxGroup];
  uint16_t* Y[kMaxGroup];
  float* U[kMaxGroup];
  int64_t m, k, r;
  float s;
};

struct GroupBwdArgs {
  const uint16_t* X;
  int count;
  int64_t n[kMaxGroup];
  const uint16_t *dY[kMaxGroup], *W[kMaxGroup], *A[kMaxGroup], *B[kMaxGroup];
  const float* U[kMaxGroup];
  uint16_t* dX;
  float *dA[kMaxGroup], *dB[kMaxGroup];
  char* ws;
  int64_t m, k, r;
  float s;
};

// Grouped backward workspace: one backward layout per projection, back to
// back; for groups of three or more whose padded ranks add up to at most 64
// (q, k, v at rank 16 or less), also a stacked dU^T of all members and the
// partials of one dA reduction over X for the whole group (13B q, k, v: 13.4
// us instead of three 6.4 us passes; for a pair such as gate, up the stacked
// pass measured no faster than two, 14.8 vs 12.8 us, so pairs keep theirs):
//   dut_stack [RPT][mp] bf16, RPT = count x RP: member g's rows at g RP ..
//   pa_stack  [splits][RPT][k] fp32 partial dA of all members
// (the members' own dUt2 and pa regions then stay unused).
struct GroupBwdLayout {
  BwdLayout L[kMaxGroup];
  size_t off[kMaxGroup];
  bool stacked;
  int rpt;
  size_t dut_stack, pa_stack;
  RedPlan plan_a;
  size_t total;
};

constexpr int kMaxStackedRank = 64;

inline GroupBwdLayout group_bwd_layout(int count, const int64_t* n, int64_t m, int64_t k, int64_t r) {
  GroupBwdLayout G{};
  size_t off = 0;
  for (int g = 0; g < count; ++g) {
    G.L[g] = bwd_layout(m, n[g], k, r);
    G.off[g] = off;
    off = align256(off + G.L[g].total);
  }
  G.rpt = count * pad_rank(r);
  G.stacked = count >= 3 && G.rpt <= kMaxStackedRank;
  if (G.stacked) {
    const size_t mp = (size_t)pad_tokens(m);
    G.plan_a = plan_reduction(m, k, G.rpt);
    G.dut_stack = off;
    off = align256(off + (size_t)G.rpt * mp * 2);
    G.pa_stack = off;
    off = align256(off + (size_t)G.plan_a.splits * G.rpt * (size_t)k * 4);
  }
  G.total = off;
  return G;
}

// Dropout keep mask drawn on the device (lora_mask.hip).
struct MaskArgs {
  uint64_t seed, offset;   // Philox key word 0 and the first counter
  uint32_t thr;            // keep iff the 16-bit draw is below thr (thr <= 2^16)
  uint8_t* keep;           // [m, k/8] packed bits
  int64_t m, k;
};

hipError_t launch_keep_mask(const MaskArgs& a, hipStream_t st);

struct MergeArgs {
  const uint16_t* W;       // [n, k]
  const uint16_t *A, *B;   // [r, k], [n, r]
  uint16_t* Wout;          // [n, k], may equal W
  int64_t n, k, r;
  float ss;                // sign * alpha / r
};

// Scratch of lora_linear_bwd_noalloc: a fixed device array per GPU holding
// the backward workspace (the largest Llama-2 projection shapes need 21 MiB).
constexpr size_t kNoAllocScratchBytes = size_t(32) << 20;

struct Launch;
hipError_t launch_fwd(const FwdArgs& a, hipStream_t st);
hipError_t launch_fwd_skinny(const Launch& L, const FwdArgs& a, const FwdGroup& grp, hipStream_t st);   // few tokens
hipError_t launch_bwd_noalloc(const BwdArgs& a, hipStream_t st);   // workspace: the library's scratch array
hipError_t launch_merge(const MergeArgs& a, hipStream_t st);
hipError_t launch_bwd(const BwdArgs& a, hipStream_t st);
hipError_t launch_bwd_fused(const BwdArgs& a, hipStream_t st);   // rank <= 16, no dropout
hipError_t launch_fwd_group(const GroupFwdArgs& a, hipStream_t st);
hipError_t launch_bwd_group(const GroupBwdArgs& a, hipStream_t st);

}  // namespace lora
