// Launch plans: the one place that decides which kernel instantiations a
// call runs, with which grid and over which output columns.  The launchers
// in lora_fwd.hip, lora_bwd.hip and lora_merge.hip execute these plans, and
// lora_linear_plan() in the C ABI reports them (host only, no GPU needed), so
// tools and tests see exactly what a call will launch.
#pragma once

#include <stdint.h>
#include <stdio.h>

#include <type_traits>

#include "lora_launch.hpp"

namespace lora {

enum KernelId : int {
  K_UPASS = 0,     // lora_u_kernel<RP, TPW, KEEP>: U = X A^T on its own (rank > 16, and under dropout)
  K_FWD = 1,       // lora_fwd_kernel<BM, BN, WM, WN, RP, GRP, UPRE, KFULL, BIG>
  K_FWD_KS = 2,    // lora_fwd_ks_kernel<GRP, KFULL, DMA, UPRE>: 128 x 256 up to rank 16
  K_DU = 3,        // lora_bwd_du_dma_kernel<RP, TPW> (r a multiple of 8), else lora_bwd_du_kernel<RP, TPW>
  K_TOKRED = 4,    // lora_tokred_dma_kernel<RP>, or lora_tokred_kernel<RP, true> with a keep mask
  K_DX = 5,        // lora_bwd_dx_kernel<BM, BN, WM, WN, RP, DROP, GRP, FULL>
  K_DXF = 6,       // lora_bwd_dxf_kernel<FULL, FASTB>
  K_FINALIZE = 7,  // lora_finalize_kernel
  K_MERGE = 8,     // lora_merge_kernel<RP, 64>
  K_MASK = 9,      // lora_keep_mask_kernel: the dropout keep mask from the counter-based generator
  K_FWD_PAIR = 11,     // lora_fwd_pair_ks_kernel<RP, GRP, KFULL, UPRE>: 128 x 128 tiles, two workgroups each
  K_FWD_SKINNY = 10,   // lora_fwd_skinny_ks_kernel<XR, F, AR, UPRE>: forward of few tokens
  K_DX_ROWS = 13,      // lora_bwd_rows_dx_kernel<128, 256, 2, 4, RP, DROP, GRP, FULL>: dX of few stages
  K_FWD_REG = 12,      // lora_fwd_reg_kernel<128, 128, 2, 2, RP, GRP, UPRE, KFULL>: two workgroups to a compute unit
};

// One kernel launch.  Fields a kernel does not use stay zero / false.
struct Launch {
  KernelId id;
  int bm, bn, wm, wn;          // GEMM output tile and wave layout
  int rp;                      // padded rank the instantiation is built for
  int tpw;                     // tokens per workgroup (U pass, dU)
  bool drop, grp, upre, full, dma, fastb;   // template switches (see KernelId)
  int64_t col_begin, col_end;  // GEMM output columns [col_begin, col_end)
  int tiles_m, tiles_n;        // GEMM tile grid (the grid is their product)
  int64_t grid;                // workgroups
  int block;                   // threads per workgroup
  bool finalize;               // dX: the workgroups' tails finalize dA and dB
  int member;                  // grouped calls: the projection a per-member launch serves
  int part;                    // token reductions: 0 dB and dA, 1 dB only, 2 a group's stacked dA
};

constexpr int kMaxLaunches = 4 + 2 * kMaxGroup;

struct Plan {
  int count = 0;
  Launch l[kMaxLaunches];
  void add(const Launch& x) {
    if (count < kMaxLaunches) l[count++] = x;
  }
};

inline Launch blank_launch(KernelId id) {
  Launch x{};
  x.id = id;
  return x;
}

// Forward instantiations exist for padded ranks 16, 32 and 64 (r = 33 .. 64
// all use 64); backward ones for 16, 32, 48 and 64.
inline int fwd_rank(int64_t r) { return r <= 16 ? 16 : (r <= 32 ? 32 : 64); }

// Output area of a tile, and the two wave counts of its kernel's name: waves
// along the tokens and the columns (of the k-split tiles, which run four waves a
// k share, they name a square arrangement whatever the tile runs).
inline void tile_dims(GemmTile t, int& bm, int& bn, int& wm, int& wn) {
  switch (t) {
    case TILE_256x256: bm = 256; bn = 256; wm = 2; wn = 4; break;
    case TILE_ROWS:
    case TILE_128x256: bm = 128; bn = 256; wm = 2; wn = 4; break;
    case TILE_128x192: bm = 128; bn = 192; wm = 2; wn = 2; break;
    case TILE_64x128: bm = 64; bn = 128; wm = 1; wn = 2; break;
    case TILE_64x64: bm = 64; bn = 64; wm = 1; wn = 2; break;
    default: bm = 128; bn = 128; wm = 2; wn = 2; break;
  }
}

inline Launch gemm_launch(KernelId id, GemmTile t, int64_t M, int64_t col_begin, int64_t col_end, int tiles_n) {
  Launch x = blank_launch(id);
  tile_dims(t, x.bm, x.bn, x.wm, x.wn);
  x.col_begin = col_begin;
  x.col_end = col_end;
  x.tiles_m = (int)((M + x.bm - 1) / x.bm);
  x.tiles_n = tiles_n >= 0 ? tiles_n : (int)((col_end - col_begin + x.bn - 1) / x.bn);
  x.grid = (int64_t)x.tiles_m * x.tiles_n;
  x.block = 64 * x.wm * x.wn;
  return x;
}

// U pass over the tokens of `count` projections that read one X: 32 tokens per
// workgroup (A read half as often) unless that leaves compute units idle, then
// 16, then 8.  The workgroups of all projections run together: counted per
// projection, 3663 x (512, 128, 128) x 512 at rank 32 took 5.4 rounds of 8-token
// workgroups (forward 26.4 us, 18.7 with 32 tokens).
inline Launch upass_launch(int count, int64_t m, int64_t r, bool drop) {
  Launch u = blank_launch(K_UPASS);
  u.rp = fwd_rank(r);
  u.drop = drop;
  const int64_t tokens = count * m;
  u.tpw = (tokens + 31) / 32 >= 256 ? 32 : ((tokens + 15) / 16 >= 256 ? 16 : 8);
  u.tiles_m = (int)((m + u.tpw - 1) / u.tpw);
  u.grid = (int64_t)count * u.tiles_m;
  u.block = 256;
  return u;
}

// Forward of few tokens: up to kSkinnyTokens, unless the output is so wide and
// the call of so few stages that the register-staged tile is estimated faster
// (faster_fwd), and up to kFewTokens for outputs of at most kSkinnyTiles tiles of
// 128 x 128.  There the GEMM tiles leave most compute units idle or multiply
// mostly padding, and a kernel that streams W past blocks of up to 64 tokens is
// faster (n = k = 4096: 4 tokens 39 -> 10 us,
// 64 tokens 40 -> 18; against paired 128 x 128 tiles: 128 tokens 24.2 -> 18.2,
// 256 x 2048 x 2048 14.7 -> 11.5, 256 x 512 x 512 7.4 -> 5.5; at 64 tiles, 192 x
// 4096 x 4096, 24.4 and 24.2; at 86, 128 x 11008 x 4096, 25.6 and 37.5).
constexpr int64_t kSkinnyTokens = 64, kSkinnyTiles = 32;
inline bool fwd_skinny(int count, const int64_t* n, int64_t m) {
  if (m <= kSkinnyTokens) return true;
  int64_t tiles = 0;
  for (int g = 0; g < count; ++g) tiles += (m + 127) / 128 * ((n[g] + 127) / 128);
  return m <= kFewTokens && tiles <= kSkinnyTiles;
}
inline Plan plan_fwd_skinny(int count, const int64_t* n, int64_t m, int64_t k, int64_t r, bool drop) {
  Plan p;
  Launch x = blank_launch(K_FWD_SKINNY);
  x.upre = drop || r > 16;   // the tile forms U beside W up to rank 16
  if (x.upre) p.add(upass_launch(count, m, r, drop));
  x.rp = x.upre ? 0 : 16;
  x.bm = m <= 16 ? 16 : (m <= 32 ? 32 : 64);
  x.tiles_m = (int)((m + x.bm - 1) / x.bm);
  // Features per workgroup: rounds of 256 workgroups times the rows a stage
  // copies, X and A rows (read from L2) at 0.6 of a W row: 4096 x 24 x 11008
  // takes 23.3, 25.7, 30.6 us with 48, 64, 96 features, 13824 x 40 x 5120 49.5
  // us with 32 and 56.4 with 48.
  double best = 1e300;
  for (const int f : {16, 32, 48, 64, 96}) {
    int64_t tiles = 0;
    for (int g = 0; g < count; ++g) tiles += (n[g] + f - 1) / f;
    const double cost = (double)((tiles * x.tiles_m + 255) / 256) * (f + 0.6 * (x.bm + x.rp));
    if (cost < best) {
      best = cost;
      x.bn = f;
      x.tiles_n = (int)tiles;
    }
  }
  x.grid = (int64_t)x.tiles_m * x.tiles_n;
  x.block = 512;
  x.col_end = count == 1 ? n[0] : 0;   // (as the grouped tiles: no single column range)
  p.add(x);
  return p;
}

// Forward GEMM launch(es) for output columns [cb, ce) with tile t.  `first`:
// the launch whose range starts at column 0 (it writes U, or the U pass runs
// before it).  U comes from the U pass for ranks above 16 (in the tile it
// would be recomputed by every output tile), on the 256 x 256 tile (where
// recomputing rank 16 in every tile costs more than the pass: 7B up_proj
// forward 387 -> 371 us), and under dropout (drop: the pass applies the keep
// mask, and the GEMM then runs exactly as without dropout); otherwise, and for
// a group on the register-staged tile, the tile computes it.  For a group,
// tiles_n is the summed column tiles.
inline void plan_fwd_part(Plan& p, GemmTile t, int64_t m, int64_t k, int64_t r, int64_t cb, int64_t ce,
                          bool first, bool drop, bool grp, int count, int tiles_n) {
  const bool kfull = k % 64 == 0;
  const bool upre = drop || t == TILE_256x256 || (fwd_rank(r) >= 32 && !(t == TILE_REG && grp));
  if (upre && first) p.add(upass_launch(count, m, r, drop));
  Launch x = gemm_launch(K_FWD, t, m, cb, ce, tiles_n);
  x.grp = grp;
  x.upre = upre;
  x.full = kfull;
  x.rp = fwd_rank(r);
  x.block = 512;
  if (t == TILE_128x256 && r <= 16) {
    // With whole stages the stages are copied straight into LDS and the wave
    // halves take turns (7B q_proj 73 -> 61 us; 2431 x 6656 x 4096, two rounds,
    // 136 -> 122).  The register-staged loop stays for several rounds of few
    // stages (2431 x 6656 x 128: 20.4 us, copies 21.1; x 256 equal) and for a
    // partial last stage, whose rows lie unaligned (1531 x 4104 x 3208 64.5 us,
    // copies 67.1).
    x.id = K_FWD_KS;
    x.dma = kfull && (x.grid <= 256 || k >= 512);
  } else if (t == TILE_PAIR) {
    x.id = K_FWD_PAIR;
    x.grid *= 2;
  } else if (t == TILE_REG) {
    x.id = K_FWD_REG;
    x.block = 256;
  } else if (t == TILE_256x256) {
    x.dma = true;
  } else {
    x.wm = x.wn = 2;
  }
  p.add(x);
}

// Estimated GPU time of the forward's kernels in us, for the choice between the
// turn-taking and few-token kernels on one side and the register-staged tile on
// the other.  A launch takes rounds of 256 workgroups (two half rounds of the
// register-staged tile run together) of a fixed part -- the first stages from
// memory, the exchange of sums, the epilogue, more of it beyond rank 16 -- and
// a part per 64-wide stage, where rows lie unaligned (k no multiple of 64) a
// longer one.  Fitted to 1900 calls drawn over the supported range up to k =
// 2048, weights read from memory: 6 to 9% standard error, 10 to 13 unaligned.
struct FwdTime { double fixed, wide[2], stage[2]; };   // wide: added at padded ranks 32, 64; stage: aligned, unaligned
inline FwdTime fwd_tile_time(const Launch& x) {
  if (x.id == K_FWD_PAIR) return {4.5, {0, 0.6}, {0.37, 0.43}};
  if (x.bm == 256) return {11, {1, 1.8}, {0.85, 0.95}};
  if (x.bn == 256) return {8.4, {2.5, 3.3}, {0.68, 0.90}};
  if (x.bn == 192) return {7, {1.6, 2.4}, {0.58, 0.73}};
  return {6, {0.1, 1}, {0.495, 0.58}};
}
// A group's U pass takes longer than a single projection's of as many
// workgroups, by about kGroupTokens us for every 1000 tokens of its members
// (6381 x (3 x 512) x 512, r = 8: forward 27.7 us, 22.1 without the pass); on
// deeper calls that is lost in the error of the rest.
constexpr int64_t kRegDepth = 1536;
constexpr double kGroupTokens = 0.6;
inline double fwd_time(const Plan& p, int64_t k, int64_t r) {
  const double stages = (double)((k + 63) / 64);
  const int rag = k % 64 != 0, wide = fwd_rank(r) / 32;   // 0, 1, 2
  double t = 0;
  for (int i = 0; i < p.count; ++i) {
    const Launch& x = p.l[i];
    const double rounds = (double)((x.grid + 255) / 256);
    if (x.id == K_UPASS) {
      t += 2.3 + rounds * stages * (x.tpw + x.rp) * 0.0013;
      if (x.grid > x.tiles_m && k <= kRegDepth) t += kGroupTokens * (double)(x.grid * x.tpw) / 1000;
    } else if (x.id == K_FWD_SKINNY) {
      const double ranks = (wide == 0 ? 0.45 : 0.85) * (double)r / 16;
      t += rag ? rounds * (3.25 + ranks + stages * (0.0052 * x.bn + 0.00175 * x.bm))
               : 0.24 + rounds * (3.28 + ranks + stages * (0.00474 * x.bn + 0.00117 * x.bm));
    } else if (x.id == K_FWD_REG) {
      const double both = (double)((x.grid + 255) / 256 / 2), one = rounds - 2 * both;
      const double w = x.upre ? (wide == 0 ? 0 : (wide == 1 ? 0.8 : 2)) : (wide == 0 ? 0 : (wide == 1 ? 1 : 3.6));
      const double f = x.upre || wide == 0 ? 1 : (wide == 1 ? 1.15 : 1.2);   // A rows and U products beside W
      t += 2 + both * (3.7 + w + (rag ? 1.34 : 1.04) * f * stages) + one * (1.9 + 0.6 * w + (rag ? 0.71 : 0.64) * f * stages);
    } else {
      const FwdTime c = fwd_tile_time(x);
      t += rounds * (c.fixed + (wide ? c.wide[wide - 1] : 0) + stages * c.stage[rag]);
    }
  }
  return t;
}
// The plan p, or the register-staged tile where that is estimated at least 3%
// faster.  Measured with the other kernels (forward calls, this tile second):
// 5912 x 1240 x 512, r = 20 23.1 and 21.2 us; 842 x (2 x 11008) x 928, r = 4 76.6
// and 61.4; 1735 x (2 x 5120) x 512, r = 32 50.7 and 39.2; 3663 x (512, 128, 128) x
// 512, r = 32 18.7 and 13.9.  The few-token kernel keeps calls deeper than
// kRegDepth, where its one pass over W wins even over wide outputs (5 x (2 x 13824)
// x 13824 133 and 180; 39 x (3 x 13824) x 512, r = 32 26.5 and 18.2).
inline Plan faster_fwd(const Plan& p, const Plan& reg, int64_t k, int64_t r) {
  if (p.l[p.count - 1].id == K_FWD_SKINNY && k > kRegDepth) return p;
  return fwd_time(reg, k, r) < 0.97 * fwd_time(p, k, r) ? reg : p;
}

// lora_linear_fwd / lora_linear_fwd_dropout (the same tiles and column split;
// under dropout the U pass applies the mask).  Below kMidTileDepth, where the
// rounds alone do not say which tile is faster, outputs of more than
// kNarrowCols columns take 128 x 192 where it is estimated at least 3% faster
// than the plan without it (786 x 5120 x 1064, r = 45 29.8 us on 128 x 256, 26.1;
// 330 x 13824 x 1040, r = 23 33.3 and 29.5; 1241 x 4096 x 512, r = 16 15.1 and 13.4;
// of 90 drawn calls that it changes 87 gain, 4 to 20%, and one loses, 1.5%).
// Narrower ones would gain 5 to 10% and keep their tiles.
constexpr int64_t kNarrowCols = 768;
enum FwdTiles { FWD_BY_ROUNDS, FWD_REG_TILE, FWD_MID_TILE };   // how plan_fwd_tiles chooses: by rounds, or this tile
inline Plan plan_fwd_tiles(int64_t m, int64_t n, int64_t k, int64_t r, bool drop, FwdTiles tiles) {
  if (tiles == FWD_BY_ROUNDS && fwd_skinny(1, &n, m)) return plan_fwd_skinny(1, &n, m, k, r, drop);
  Plan p;
  const GemmSplit s = tiles == FWD_REG_TILE ? GemmSplit{TILE_REG, TILE_REG, n}
                      : tiles == FWD_MID_TILE
                          ? GemmSplit{TILE_128x192, TILE_128x192, n}
                          : plan_gemm_split(kFwdTiles, m, n, k >= kMidTileDepth ? TILES_MID : TILES_BASE);
  plan_fwd_part(p, s.t1, m, k, r, 0, s.n1, true, drop, false, 1, -1);
  if (s.n1 < n) plan_fwd_part(p, s.t2, m, k, r, s.n1, n, false, drop, false, 1, -1);
  return p;
}
inline Plan plan_fwd(int64_t m, int64_t n, int64_t k, int64_t r, bool drop) {
  const Plan p = plan_fwd_tiles(m, n, k, r, false, FWD_BY_ROUNDS), reg = plan_fwd_tiles(m, n, k, r, false, FWD_REG_TILE);
  Plan best = faster_fwd(p, reg, k, r);
  FwdTiles tiles = best.l[best.count - 1].id == K_FWD_REG ? FWD_REG_TILE : FWD_BY_ROUNDS;
  if (k < kMidTileDepth && n > kNarrowCols && best.l[best.count - 1].id != K_FWD_SKINNY) {
    const Plan mid = plan_fwd_tiles(m, n, k, r, false, FWD_MID_TILE);
    if (fwd_time(mid, k, r) < 0.97 * fwd_time(best, k, r)) {
      best = mid;
      tiles = FWD_MID_TILE;
    }
  }
  return drop ? plan_fwd_tiles(m, n, k, r, true, tiles) : best;
}

// lora_linear_group_fwd: one GEMM launch over the output tiles of all members,
// the tile chosen for m x (sum of n).  A group of one is the single projection.
inline Plan plan_group_fwd_tiles(int count, const int64_t* n, int64_t m, int64_t k, int64_t r, bool reg) {
  if (!reg && fwd_skinny(count, n, m)) return plan_fwd_skinny(count, n, m, k, r, false);
  int64_t ntot = 0;
  for (int g = 0; g < count; ++g) ntot += n[g];
  const GemmTile t = reg ? TILE_REG : cheapest_tile(kFwdTiles, m, ntot, TILES_BASE).t;
  int bm, bn, wm, wn;
  tile_dims(t, bm, bn, wm, wn);
  int tiles_n = 0;
  for (int g = 0; g < count; ++g) tiles_n += (int)((n[g] + bn - 1) / bn);
  Plan p;
  plan_fwd_part(p, t, m, k, r, 0, 0, true, false, true, count, tiles_n);
  return p;
}
inline Plan plan_group_fwd(int count, const int64_t* n, int64_t m, int64_t k, int64_t r) {
  if (count == 1) return plan_fwd(m, n[0], k, r, false);
  return faster_fwd(plan_group_fwd_tiles(count, n, m, k, r, false), plan_group_fwd_tiles(count, n, m, k, r, true), k, r);
}

// dX GEMM launch over columns [cb, ce).  FULL (no bound checks on the copies)
// needs every n a multiple of 64 and whole column tiles.  The 256 x 256 tile
// runs only FULL; otherwise the range takes a 128 x 256 tile, of `depth`
// contraction steps in all.
inline void plan_dx_part(Plan& p, GemmTile t, int64_t m, int rp, int64_t depth, int64_t cb, int64_t ce, bool n_whole,
                         bool drop, bool grp, bool finalize) {
  int bm, bn, wm, wn;
  tile_dims(t, bm, bn, wm, wn);
  bool full = n_whole && (ce - cb) % bn == 0;
  if (t == TILE_256x256 && !full) {
    t = depth < kMidTileDepth ? TILE_ROWS : TILE_128x256;
    tile_dims(t, bm, bn, wm, wn);
    full = n_whole && (ce - cb) % bn == 0;
  }
  Launch x = gemm_launch(t == TILE_ROWS ? K_DX_ROWS : K_DX, t, m, cb, ce, -1);
  x.rp = rp;
  x.drop = drop;
  x.grp = grp;
  x.block = 512;
  x.full = full;
  x.finalize = finalize;
  p.add(x);
}

// Tiles open to the dX GEMM of m tokens over `depth` output features.
inline int dx_tile_set(int64_t m, int64_t depth, bool grp) {
  return (!grp && depth >= kMidTileDepth ? TILES_MID : 0) | (m <= kFewTokens || (m <= kShortTokens && depth >= kShortDepth) ? TILES_SHORT : 0);
}

inline GemmSplit dx_split(int64_t m, int64_t k, int64_t depth, bool grp) {
  const int set = dx_tile_set(m, depth, grp);
  return depth < kMidTileDepth ? plan_gemm_split(kDxShallowTiles, m, k, set) : plan_gemm_split(kDxTiles, m, k, set);
}

// dU of `count` projections of one rank and token count in one launch.
inline Launch du_launch(const BwdLayout& L, int64_t r, int count) {
  Launch x = blank_launch(K_DU);
  x.rp = L.rp;
  x.fastb = r % 8 == 0;   // 16-byte pieces of B then lie inside one row: the direct-to-LDS kernel
  // the most tokens per workgroup (each reads all of B) that still leaves no
  // compute unit idle; 32 tokens from padded rank 32 on, where B is at least
  // as many bytes per workgroup as 16 tokens of dY
  const int64_t tokens = count * L.mp;
  x.tpw = tokens / 16 < 256 ? 8 : (L.rp >= 32 && tokens / 32 >= 256 ? 32 : 16);
  x.tiles_m = (int)(L.mp / x.tpw);
  x.grid = (int64_t)count * x.tiles_m;
  x.block = x.fastb ? 256 : 512;
  x.member = count == 1 ? 0 : -1;
  return x;
}

// Token reductions run four waves per workgroup.
inline int tokred_threads(int) { return 256; }

inline Launch tokred_launch(const BwdLayout& L, bool keep, int member, int part = 0) {
  Launch x = blank_launch(K_TOKRED);
  x.rp = L.rp;
  x.drop = keep;
  x.grid = (int64_t)L.plan_b.col_tiles * L.plan_b.splits + (part == 0 ? (int64_t)L.plan_a.col_tiles * L.plan_a.splits : 0);
  x.block = tokred_threads(x.rp);
  x.member = member;
  x.part = part;
  return x;
}

// lora_linear_bwd / lora_linear_bwd_dropout: dU, the token reductions, then
// the dX GEMM (its columns split between two launches as for the forward; the
// first one's tails finalize dA and dB).
inline Plan plan_bwd(int64_t m, int64_t n, int64_t k, int64_t r, bool drop) {
  const BwdLayout L = bwd_layout(m, n, k, r);
  Plan p;
  p.add(du_launch(L, r, 1));
  p.add(tokred_launch(L, drop, 0));
  const bool n_whole = n % 64 == 0;
  if (drop) {
    const int set = dx_tile_set(m, n, false);
    const GemmTile t = (n < kMidTileDepth ? cheapest_tile(kDxDropShallowTiles, m, k, set)
                                          : cheapest_tile(kDxDropTiles, m, k, set)).t;
    plan_dx_part(p, t, m, L.rp, n, 0, k, n_whole, true, false, true);
    return p;
  }
  const GemmSplit s = dx_split(m, k, n, false);
  plan_dx_part(p, s.t1, m, L.rp, n, 0, s.n1, n_whole, false, false, true);
  if (s.n1 < k) plan_dx_part(p, s.t2, m, L.rp, n, s.n1, k, n_whole, false, false, false);
  return p;
}

// lora_linear_group_bwd: one dU launch for all members (three members of 300 x
// 4096 x 4096 step 162 -> 150 us against one each; equal at 4096 tokens), per
// member the token reductions, then one dX
// launch over the concatenated contraction (split like the single one).  For
// groups of three or more whose padded ranks add up to at most 64 the dA
// reductions of all members run as one (a stacked rank over one pass of X)
// after the members' dB reductions.
inline Plan plan_group_bwd(int count, const int64_t* n, int64_t m, int64_t k, int64_t r) {
  if (count == 1) return plan_bwd(m, n[0], k, r, false);
  const GroupBwdLayout G = group_bwd_layout(count, n, m, k, r);
  Plan p;
  bool n_whole = true;
  int64_t depth = 0;
  p.add(du_launch(G.L[0], r, count));
  for (int g = 0; g < count; ++g) {
    p.add(tokred_launch(G.L[g], false, g, G.stacked ? 1 : 0));
    n_whole = n_whole && n[g] % 64 == 0;
    depth += n[g];
  }
  if (G.stacked) {
    Launch x = blank_launch(K_TOKRED);
    x.rp = G.rpt;
    x.grid = (int64_t)G.plan_a.col_tiles * G.plan_a.splits;
    x.block = tokred_threads(x.rp);
    x.member = -1;
    x.part = 2;
    p.add(x);
  }
  const int rp = G.L[0].rp;
  const GemmSplit s = dx_split(m, k, depth, true);
  plan_dx_part(p, s.t1, m, rp, depth, 0, s.n1, n_whole, false, true, true);
  if (s.n1 < k) plan_dx_part(p, s.t2, m, rp, depth, s.n1, k, n_whole, false, true, false);
  return p;
}

// lora_linear_bwd_fused (r <= 16): the dX launch that also forms dU and the dB
// partials, the dA token reduction, the finalize.
inline Plan plan_bwd_fused(int64_t m, int64_t n, int64_t k, int64_t r) {
  const BwdFusedLayout L = bwd_fused_layout(m, n, k, r);
  Plan p;
  Launch x = gemm_launch(K_DXF, TILE_128x256, m, 0, k, -1);
  x.rp = 16;
  x.fastb = r % 8 == 0;
  x.full = x.fastb && n % 64 == 0 && k % 256 == 0;
  p.add(x);
  Launch t = blank_launch(K_TOKRED);
  t.rp = 16;
  t.grid = (int64_t)L.plan_a.col_tiles * L.plan_a.splits;
  t.block = tokred_threads(t.rp);
  p.add(t);
  Launch f = blank_launch(K_FINALIZE);
  const int64_t total = n * r + r * k;
  f.grid = (total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048;
  f.block = 256;
  p.add(f);
  return p;
}

// lora_linear_merge: 64 x 128 tiles of W.
constexpr int kMergeRows = 64;
inline Plan plan_merge(int64_t n, int64_t k, int64_t r) {
  Plan p;
  Launch x = blank_launch(K_MERGE);
  x.rp = pad_rank(r);
  x.tiles_m = (int)((n + kMergeRows - 1) / kMergeRows);
  x.tiles_n = (int)((k + 127) / 128);
  x.grid = (int64_t)x.tiles_m * x.tiles_n;
  x.block = 256;
  p.add(x);
  return p;
}

// lora_dropout_keep_mask: kMaskBytesPerThread mask bytes (two per generator
// block) per thread.
constexpr int kMaskBytesPerThread = 4;
inline Plan plan_keep_mask(int64_t m, int64_t k) {
  Plan p;
  Launch x = blank_launch(K_MASK);
  x.grid = (m * (k / 8) + kMaskBytesPerThread * 256 - 1) / (kMaskBytesPerThread * 256);
  x.block = 256;
  p.add(x);
  return p;
}

// The instantiation's name as profilers print it (demangled, without the
// argument list).
inline void launch_name(const Launch& x, char* buf, size_t len) {
  auto b = [](bool v) { return v ? "true" : "false"; };
  switch (x.id) {
    case K_UPASS: snprintf(buf, len, "lora::lora_u_kernel<%d, %d, %s>", x.rp, x.tpw, b(x.drop)); break;
    case K_FWD:
      snprintf(buf, len, "lora::lora_fwd_kernel<%d, %d, %d, %d, %d, %s, %s, %s, %s>", x.bm, x.bn, x.wm, x.wn, x.rp,
               b(x.grp), b(x.upre), b(x.full), b(x.dma));
      break;
    case K_FWD_KS:
      snprintf(buf, len, "lora::lora_fwd_ks_kernel<%s, %s, %s, %s>", b(x.grp), b(x.full), b(x.dma), b(x.upre));
      break;
    case K_DU:
      snprintf(buf, len, x.fastb ? "lora::lora_bwd_du_dma_kernel<%d, %d>" : "lora::lora_bwd_du_kernel<%d, %d>", x.rp,
               x.tpw);
      break;
    case K_TOKRED:
      if (x.drop) snprintf(buf, len, "lora::lora_tokred_kernel<%d, true>", x.rp);
      else snprintf(buf, len, "lora::lora_tokred_dma_kernel<%d>", x.rp);
      break;
    case K_DX:
      snprintf(buf, len, "lora::lora_bwd_dx_kernel<%d, %d, %d, %d, %d, %s, %s, %s>", x.bm, x.bn, x.wm, x.wn, x.rp,
               b(x.drop), b(x.grp), b(x.full));
      break;
    case K_DX_ROWS:
      snprintf(buf, len, "lora::lora_bwd_rows_dx_kernel<%d, %d, %d, %d, %d, %s, %s, %s>", x.bm, x.bn, x.wm, x.wn, x.rp,
               b(x.drop), b(x.grp), b(x.full));
      break;
    case K_DXF: snprintf(buf, len, "lora::lora_bwd_dxf_kernel<%s, %s>", b(x.full), b(x.fastb)); break;
    case K_FINALIZE: snprintf(buf, len, "lora::lora_finalize_kernel"); break;
    case K_MERGE: snprintf(buf, len, "lora::lora_merge_kernel<%d, %d>", x.rp, kMergeRows); break;
    case K_MASK: snprintf(buf, len, "lora::lora_keep_mask_kernel"); break;
    case K_FWD_PAIR:
      snprintf(buf, len, "lora::lora_fwd_pair_ks_kernel<%d, %s, %s, %s>", x.rp, b(x.grp), b(x.full), b(x.upre));
      break;
    case K_FWD_REG:
      snprintf(buf, len, "lora::lora_fwd_reg_kernel<%d, %d, %d, %d, %d, %s, %s, %s>", x.bm, x.bn, x.wm, x.wn, x.rp,
               b(x.grp), b(x.upre), b(x.full));
      break;
    case K_FWD_SKINNY:
      snprintf(buf, len, "lora::lora_fwd_skinny_ks_kernel<%d, %d, %d, %s>", x.bm, x.bn, x.rp, b(x.upre));
      break;
  }
}

// Runtime switches to compile-time constants for the launchers' dispatch.
template <typename F>
inline hipError_t with_bool(bool v, F&& f) {
  return v ? f(std::true_type{}) : f(std::false_type{});
}

template <int... Vs, typename F>
inline hipError_t with_int(int v, F&& f) {
  hipError_t e = hipErrorInvalidValue;
  (void)((v == Vs ? (e = f(std::integral_constant<int, Vs>{}), true) : false) || ...);
  return e;
}

// The GEMM tile of a launch as its width, 257 for 256x256, 65 for 64x128.
inline int tile_code(const Launch& x) { return x.bm == 256 ? 257 : (x.bm == 64 && x.bn == 128 ? 65 : x.bn); }

}  // namespace lora
