// Forward of the LoRA-adapted linear layer (Eq. 1 of JORA, Section 3):
//   U = X A^T,   Y = X W^T + s U B^T,   s = alpha / r.
//
// Kernels (one launch per call; a U pass before it for rank > 16 -- but a group's
// on the register-staged tile --, on the 256 x 256 tile and under dropout, and a
// second GEMM launch when the columns are split between two tiles):
//   lora_fwd_kernel     the 256 x 256 tile (below), and the 128-token tiles of
//                       lora_fwd_ks.hpp: 128 x 128, 128 x 192 and, beyond rank
//                       16, 128 x 256.
//   lora_fwd_ks_kernel  the 128 x 256 tile up to rank 16 (the 7B q_proj shape).
//   lora_fwd_pair_ks_kernel  128 x 128 tiles, each computed by a pair of
//                       workgroups of 64 tokens (lora_fwd_ks.hpp).
//   lora_u_kernel       U = X A^T on its own (under dropout with the keep
//                       mask applied; for a group, of every projection in one
//                       launch), followed by a GEMM tile without U columns.
//   lora_fwd_skinny_ks_kernel (lora_fwd_skinny.hip)  few tokens.
//   lora_fwd_reg_kernel (lora_fwd_reg.hpp)  128 x 128 tiles of few stages, staged
//                       in registers, two workgroups to a compute unit.
// A launch covers the output columns from n_begin on (plan_gemm_split);
// the launch whose range starts at column 0 writes U.
//
// Every tile walks k in stages of 64.  Per stage it stages k-contiguous tiles
// in LDS -- X rows, W rows and, where U is formed beside W, A padded to 16
// rows -- so each X tile is read once for both products.
//
// Matrix-core products are formed transposed
// (W as the A operand, X as the B operand), so each lane's accumulator holds
// runs of 4 consecutive output features of one token.  After the k loop the
// epilogue adds s U B^T to the accumulators with a short matrix-core pass over
// t in which s U enters as a bf16 high part and a bf16 low part, then rounds Y
// to bf16 and stores it through a per-wave LDS block so that stores write
// whole row pieces.
#include <type_traits>

#include "lora_device.hpp"
#include "lora_fwd_ks.hpp"
#include "lora_fwd_reg.hpp"
#include "lora_launch.hpp"
#include "lora_plan.hpp"

namespace lora {

constexpr int kBigStage = 512 * 128;   // bytes of a 64-wide stage of the 256 x 256 tile

// The 256 x 256 tile: eight waves of 128 x 64, two 64-wide stages in LDS, U
// from the U pass (read back in the epilogue).  The stages are copied from
// global memory straight into LDS (one 16-byte chunk per lane per copy
// instruction, the swizzle applied to the global addresses).
//
// The two wave rows take turns: waves w and w + 4 share a SIMD, and while one
// multiplies, the other reads its next fragments and issues copies; a workgroup
// barrier ends each slot, and the second row runs one slot behind.  A stage is
// four phases, each a slot of reads and a slot of sixteen products: (W half 0, X
// half 0), (W 1, X 0), (W 0, X 1), (W 1, X 1), reading X half 0, W half 1, X
// half 1 and the next stage's W half 0.  Every wave waits for its reads before
// the barrier that ends its read slot, so the quarter of a stage read in phase
// P is free from the read slots of phase P + 1 on, which refill it for the
// stage after next (seven phases before its use).  The quarter read in phase
// P + 1 is waited for (six newer ones stay in flight) in the read slot of P.
// The reads before the first slot (W half 0 of stage 0, whose quarter the first
// row's first slot refills) are closed the same way: every wave waits for them
// and all eight pass a barrier before the second row's extra one.
//
// Bound by power: with all eight waves in step (reads of the next substep
// under the products, one barrier per stage) the matrix cores were 65% busy,
// waiting after every barrier.  8192 x 4096 x 11008 at rank 64 (U pass
// included) takes 620 us so, 582 taking turns on 32x32x16 products and 533 on
// the 16x16x32 ones used here; 4096 x 11008 x 4096 at rank 16 303, 292 and 275;
// 4096 x 4096 x 5120 143, 137 and 126 (one process, in turn).  s_setprio around
// the products: no difference.
// KFULL: k a multiple of 64 (otherwise each copy checks its k bound).  With GRP
// the grid covers the output tiles of a group of projections that read the
// same X (FwdGroup): each workgroup first selects its projection's W, B, Y, U
// and n.
template <int RP, bool GRP, bool KFULL>
__device__ __forceinline__ void fwd_big_tile(const u16* __restrict__ X, const u16* __restrict__ W,
                                             const u16* __restrict__ B, u16* __restrict__ Y,
                                             const float* __restrict__ U, int m, int n, int k, int r, float s, int tm,
                                             int tn, int n_begin, const FwdGroup& grp, char* smem) {
  constexpr int BM = 256, BN = 256, WM = 2, WN = 4;
  constexpr int NW = WM * WN;
  constexpr int NT = 64 * NW;
  constexpr int WTI = BM / WM, WTJ = BN / WN;   // tokens, features per wave
  static_assert(WTI == 128 && WTJ == 64, "wave tile");
  constexpr int STAGE = kBigStage;
  static_assert(STAGE == (BM + BN) * 128 && 2 * STAGE <= 160 * 1024, "128-byte rows per 64-wide stage");
  constexpr int RPU = 2 * RP + 8, RPB = RP + 8;   // padded row lengths of the epilogue's U and B copies
  static_assert(BM * RPU * 2 + BN * RPB * 2 <= 2 * STAGE, "epilogue LDS reuse");
  if (GRP) {   // projection of this column tile (uniform; compile-time indices only)
    int sel = 0;
#pragma unroll
    for (int q = 1; q < kMaxGroup; ++q)
      if (q < grp.count && tn >= grp.tile0[q]) sel = q;
#pragma unroll
    for (int q = 0; q < kMaxGroup; ++q)
      if (q == sel) {
        W = grp.W[q]; B = grp.B[q]; Y = grp.Y[q]; U = grp.U[q];
        n = grp.n[q];
        tn -= grp.tile0[q];
      }
  }
  const int m0 = tm * BM, n0 = n_begin + tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int g = lane >> 4, c16 = lane & 15;

  const uint32_t rowbytes = (uint32_t)k * 2;
  const __amdgpu_buffer_rsrc_t rsX = make_rsrc(X + (size_t)m0 * k, (uint64_t)min(BM, m - m0) * rowbytes);
  const __amdgpu_buffer_rsrc_t rsW = make_rsrc(W + (size_t)n0 * k, (uint64_t)min(BN, n - n0) * rowbytes);

  floatx4 acc[4][8];           // 16 x 16 fragments: [features 16 a ..][tokens 16 b ..] of the wave's 64 x 128
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  short8 fw[2][2][2], fx[2][4];   // W halves [half][32-wide k][fragment], the current X half [32-wide k][fragment]
  const int nkb = (k + 63) / 64;
  // Quarters of a stage, 16 KB each: X half h = tokens 64 h .. + 63 of both
  // wave rows (tile rows 64 h .. and 128 + 64 h ..), W half h = features 32 h ..
  // + 31 of all four wave columns (rows 64 j + 32 h ..).
  // A wave copies 8 rows per instruction, two instructions per quarter: lane l
  // takes position l % 8 of row l / 8 of the eight, which holds logical chunk
  // (l % 8) ^ kc_swz(row) (the same for all of a wave's copies).
  const int l8 = lane >> 3;
  const int xrow = 8 * wave, wrow = 64 * (wave >> 2) + 8 * (wave & 3);
  const int kcol = 8 * ((lane & 7) ^ kc_swz(xrow + l8));
  const uint32_t xoff = (uint32_t)(xrow + l8) * rowbytes + (uint32_t)kcol * 2;
  const uint32_t woff = (uint32_t)(wrow + l8) * rowbytes + (uint32_t)kcol * 2;
  auto copy_x = [&](int kb, int h) LORA_INLINE {
    char* sb = smem + (kb & 1) * STAGE + xrow * 128 + h * 8192;
    const bool ok = KFULL || kb * 64 + kcol < k;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      dma16(rsX, ok ? xoff + (uint32_t)(64 * h + 128 * i) * rowbytes : kOOB, (uint32_t)kb * 128, sb + i * 16384);
  };
  auto copy_w = [&](int kb, int h) LORA_INLINE {
    char* sb = smem + (kb & 1) * STAGE + BM * 128 + wrow * 128 + h * 4096;
    const bool ok = KFULL || kb * 64 + kcol < k;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      dma16(rsW, ok ? woff + (uint32_t)(32 * h + 128 * i) * rowbytes : kOOB, (uint32_t)kb * 128, sb + i * 16384);
  };
  auto read_x = [&](int kb, int h) LORA_INLINE {
    const char* Xs = smem + (kb & 1) * STAGE;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int b = 0; b < 4; ++b) fx[kk][b] = kc_read(Xs, wm * WTI + 64 * h + 16 * b + c16, 4 * kk + g);
  };
  auto read_w = [&](int kb, int h) LORA_INLINE {
    const char* Ws = smem + (kb & 1) * STAGE + BM * 128;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int a = 0; a < 2; ++a) fw[h][kk][a] = kc_read(Ws, wn * WTJ + 32 * h + 16 * a + c16, 4 * kk + g);
  };
  auto slot_end = [&]() LORA_INLINE {
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto products = [&](int hw, int hx) LORA_INLINE {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[2 * hw + a][4 * hx + b] = mfma16x16x32(fw[hw][kk][a], fx[kk][b], acc[2 * hw + a][4 * hx + b]);
    __builtin_amdgcn_sched_barrier(0);
    slot_end();
  };
  auto ready = [&](auto left) LORA_INLINE {   // reads done; at most `left` quarters' copies in flight
    __builtin_amdgcn_sched_barrier(0);
    wait_lgkm0();
    wait_vmcnt<2 * decltype(left)::value>();
    slot_end();
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using I4 = std::integral_constant<int, 4>;
  using I5 = std::integral_constant<int, 5>;
  using I6 = std::integral_constant<int, 6>;
  auto stage = [&](int kb, auto mode) LORA_INLINE {   // 0: steady, 1: the last but one, 2: the last
    constexpr int MODE = decltype(mode)::value;
    read_x(kb, 0);
    if constexpr (MODE == 0) { copy_w(kb + 2, 0); ready(I6{}); }
    else if constexpr (MODE == 1) ready(I5{});
    else ready(I1{});
    products(0, 0);
    read_w(kb, 1);
    if constexpr (MODE == 0) { copy_x(kb + 2, 0); ready(I6{}); }
    else if constexpr (MODE == 1) ready(I4{});
    else ready(I0{});
    products(1, 0);
    read_x(kb, 1);
    if constexpr (MODE == 0) { copy_w(kb + 2, 1); ready(I6{}); }
    else if constexpr (MODE == 1) ready(I3{});
    else ready(I0{});
    products(0, 1);
    if constexpr (MODE < 2) read_w(kb + 1, 0);
    if constexpr (MODE == 0) { copy_x(kb + 2, 1); ready(I6{}); }
    else if constexpr (MODE == 1) ready(I2{});
    else ready(I0{});
    products(1, 1);
  };
  copy_w(0, 0); copy_x(0, 0); copy_w(0, 1); copy_x(0, 1);
  if (nkb > 1) {
    copy_w(1, 0); copy_x(1, 0); copy_w(1, 1); copy_x(1, 1);
    wait_vmcnt<12>();
  } else {
    wait_vmcnt<0>();
  }
  slot_end();
  read_w(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  wait_lgkm0();
  slot_end();                    // every wave has read the quarter that the first read slot refills
  if (wm == 1) slot_end();       // the second wave row runs one slot behind
  int kb = 0;
  for (; kb + 2 < nkb; ++kb) stage(kb, I0{});
  if (nkb > 1) stage(kb++, I1{});
  stage(kb, I2{});
  if (wm == 0) slot_end();

  // ---- epilogue ------------------------------------------------------------
  // LDS reuse: Us [BM][RPU] bf16, s U as its high parts (RP) and low parts (RP)
  // a row, then Bs [BN][RPB] bf16 (B rows of this tile, zero beyond r and n).
  // Split here, once a value: split by every wave that multiplies the token (each
  // lane forming both parts) the conversions alone took 5 us a tile at rank 64.
  // The rows are padded by 16 bytes so that the 16 lanes of a read group, which
  // read 16 consecutive rows, fall in different banks.  Rows n0 .. n0+jn-1 of B
  // are fetched as 16-byte chunks of 8 elements, all issued before the first
  // wait.
  u16* Us = reinterpret_cast<u16*>(smem);
  u16* Bs = reinterpret_cast<u16*>(smem + BM * RPU * 2);
  constexpr int BCH = (BN * RP / 8 + NT - 1) / NT;   // chunks per thread (r <= RP)
  const int jn = min(BN, n - n0);
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B + (size_t)n0 * r, (uint64_t)jn * r * 2);
  int4v bv[BCH];
  load_b_rows<RP, NT>(rsB, r, jn, tid, bv);
  {   // U of the tile's tokens from the U pass (zero beyond r and m), all loads issued before the first use
    const __amdgpu_buffer_rsrc_t rsU = make_rsrc(U + (size_t)m0 * r, (uint64_t)min(BM, m - m0) * r * 4);
    float uv[BM * RP / NT];
    load_u_pairs<BM, RP, NT>(rsU, r, tid, uv);
    split_u_pairs<BM, RP, NT>(uv, s, tid, Us);
  }
  store_b_rows<BN, RP, NT>(bv, r, jn, tid, Bs);
  __syncthreads();

  // acc += s U B^T, formed as Y^T += B (sU)^T over t in blocks of 16: one
  // product of 32 k holds the block twice, against the high bf16 part of sU in
  // its lower half (lanes g = 0, 1) and the low part in its upper half.
  const int tblocks = (r + 15) / 16;
  const u16* up = Us + (wm * WTI + c16) * RPU + (g < 2 ? 0 : RP) + 8 * (g & 1);
  const u16* bp = Bs + (wn * WTJ + c16) * RPB + 8 * (g & 1);
  for (int tb = 0; tb < tblocks; ++tb) {
    short8 bfr[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) bfr[a] = *reinterpret_cast<const short8*>(bp + 16 * a * RPB + 16 * tb);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const short8 uf = *reinterpret_cast<const short8*>(up + 16 * b * RPU + 16 * tb);
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[a][b] = mfma16x16x32(bfr[a], uf, acc[a][b]);
    }
  }

  // store Y: each wave's blocks of 32 tokens x 64 features through a
  // wave-private LDS region (free once every wave is past the reads above)
  constexpr int OUT = out16_bytes<4, 2>();
  static_assert(NW * OUT <= 2 * STAGE, "output staging");
  __syncthreads();
  const int j0 = n0 + wn * WTJ;
#pragma unroll
  for (int fi = 0; fi < 4; ++fi) {
    const int i0 = m0 + wm * WTI + 32 * fi;
    floatx4 v[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      v[a][0] = acc[a][2 * fi];
      v[a][1] = acc[a][2 * fi + 1];
    }
    store_out16<4, 2>(v, smem + wave * OUT, Y + (size_t)i0 * n + j0, (size_t)n, m - i0, n - j0, lane);
  }
}

// One kernel template for the 256 x 256 tile (BIG) and the 128-token tiles that
// lora_fwd_ks_kernel does not serve.  WM and WN, the waves along the tokens and
// the features of a k share, stand in the kernels' names alone.
template <int BM, int BN, int WM, int WN, int RP, bool GRP, bool UPRE, bool KFULL, bool BIG>
__global__ __launch_bounds__(512) void lora_fwd_kernel(
    const u16* __restrict__ X, const u16* __restrict__ W, const u16* __restrict__ A, const u16* __restrict__ B,
    u16* __restrict__ Y, float* __restrict__ U, int m, int n, int k, int r, float s, int tiles_m, int tiles_n,
    int n_begin, FwdGroup grp) {
  static_assert(BIG == (BM == 256) && (BM == 256 ? BN == 256 && UPRE : BM == 128), "tile shapes");
  int tm, tn;
  tile_coords(tiles_m, tiles_n, 8, (int)blockIdx.x, tm, tn);
  if constexpr (BIG) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * kBigStage];
    fwd_big_tile<RP, GRP, KFULL>(X, W, B, Y, U, m, n, k, r, s, tm, tn, n_begin, grp, smem);
  } else {
    __shared__ __attribute__((aligned(1024))) char smem[fwd_ks_smem<128, BN, RP, UPRE>()];
    fwd_ks_tile<128, BN, RP, GRP, UPRE, KFULL>(X, W, A, B, Y, U, m, n, k, r, s, tm * 128, tn, n_begin, grp, smem);
  }
}

// 128 x 128 tiles, each computed by a pair of workgroups of 64 tokens, for
// outputs of too few tiles to fill the chip.  Pair p's workgroups are 8 apart
// (the last few, when the tiles are no multiple of 8, at most 7 apart), so
// both run on the same XCD and share the tile's W rows in its L2.
template <int RP, bool GRP, bool KFULL, bool UPRE>
__global__ __launch_bounds__(512) void lora_fwd_pair_ks_kernel(
    const u16* __restrict__ X, const u16* __restrict__ W, const u16* __restrict__ A, const u16* __restrict__ B,
    u16* __restrict__ Y, float* __restrict__ U, int m, int n, int k, int r, float s, int tiles_m, int tiles_n,
    int n_begin, FwdGroup grp) {
  __shared__ __attribute__((aligned(1024))) char smem[fwd_ks_smem<64, 128, RP, UPRE>()];
  const int b = (int)blockIdx.x, tiles = tiles_m * tiles_n, whole = tiles & ~7, rest = tiles & 7;
  int p, h;
  if (b < 2 * whole) {
    p = (b >> 4) * 8 + (b & 7);
    h = (b >> 3) & 1;
  } else {
    h = (b - 2 * whole) / rest;
    p = whole + (b - 2 * whole) - h * rest;
  }
  int tm, tn;
  tile_coords(tiles_m, tiles_n, 8, p, tm, tn);
  const int m0 = tm * 128 + 64 * h;
  if (m0 >= m) return;   // (uniform) the second half of a ragged last tile row
  fwd_ks_tile<64, 128, RP, GRP, UPRE, KFULL>(X, W, A, B, Y, U, m, n, k, r, s, m0, tn, n_begin, grp, smem);
}

// ---------------------------------------------------------------------------
// U = X A^T on its own: for ranks above 16 (in the fused tile every output
// tile recomputes all RP U columns of its tokens, RP / BN more matrix-core
// work, a quarter at RP = 64 on the 256-wide tile; this pass computes them
// once), and under LoRA dropout (KEEP: U = (keep X) A^T / (1 - p), so the
// GEMM that follows needs no mask).  TPW (8, 16 or 32) tokens per workgroup,
// four waves (eight measured the same: 1024 x 5120 x 13824 step at rank 32
// 302.2 and 302.3 us).  The k loop runs in stages of 64; wave w takes stages w, w + 4,
// ... and copies each of them (its TPW X rows and RP A rows, 128 bytes a row,
// eight whole row pieces per copy instruction with the swizzle of kc_offset
// applied to the global addresses; under KEEP also the stage's keep bits, 8
// bytes a token, 4 bytes a lane) from global memory straight into a private
// ring of NSW LDS stages, NSW - 1 stages ahead.  No barrier in the loop: the
// wave waits only for its own copies.  (Loads of 16 rows x 64 bytes per
// instruction straight into matrix-core operands kept the L1 busy
// translating addresses; a shared ring with a barrier per stage was bound by
// each stage's short compute chain.)  Each wave accumulates all RP x TPW of U
// over its stages (16x16x32 products; under KEEP each X fragment of 8 k is
// masked with its keep byte first); the four partial sums are added in wave
// order through LDS at the end (bit-identical from run to run) and written
// as fp32 U [m][r], scaled by inv_keep under KEEP.  With TPW = 8 (launches
// whose 16-token workgroups would leave compute units idle) a stage still
// holds 16 X rows for the 16-token products; rows 8..15 are zeroed once and
// never copied into, and only the first 8 tokens' U is written.
template <int RP, int TPW, bool KEEP>
__global__ __launch_bounds__(256) void lora_u_kernel(const u16* __restrict__ X, const uint8_t* __restrict__ keep,
                                                     int m, int k, int r, float inv_keep, int blocks, FwdGroup grp) {
  constexpr int NWV = 4;
  constexpr int XR = TPW < 16 ? 16 : TPW;        // X rows of a stage (rows TPW .. XR-1 stay zero)
  constexpr int ROWS = XR + RP;                  // 128-byte rows per stage: X rows, then A rows
  constexpr int MOFF = ROWS * 128;               // keep bytes of the stage: [TPW][8]
  constexpr int STAGE = MOFF + (KEEP ? 256 : 0);
  constexpr int CPS = (TPW + RP) / 8;            // 1 KB copies per stage
  constexpr int CPW = CPS + (KEEP ? 1 : 0);      // copy instructions per stage (the wave's own)
  constexpr int NSW = (156 * 1024) / (NWV * STAGE) < 6 ? (156 * 1024) / (NWV * STAGE) : 6;   // ring stages per wave
  constexpr int FT = RP / 16, TG = XR / 16;
  constexpr int RED = NWV * FT * TG * 64 * 16;   // cross-wave sum: [NWV][FT][TG][64] float4
  constexpr int SMEM = NWV * NSW * STAGE > RED ? NWV * NSW * STAGE : RED;
  static_assert(TPW == 8 || TPW == 16 || TPW == 32, "tokens per workgroup");
  static_assert(NSW >= 3 && CPW * (NSW - 2) < 64, "copies in flight fit the wait counter");
  static_assert(FT * TG <= 8, "fragments per wave");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  const int sel = (int)blockIdx.x / blocks;        // the projection (its A and U)
  const u16* A = grp.A[0];
  float* U = grp.U[0];
#pragma unroll
  for (int q = 1; q < kMaxGroup; ++q)
    if (q == sel) { A = grp.A[q]; U = grp.U[q]; }
  const int i0 = ((int)blockIdx.x - sel * blocks) * TPW;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const uint32_t rowbytes = (uint32_t)k * 2;
  const int rows = uniform(max(0, min(TPW, m - i0)));
  const __amdgpu_buffer_rsrc_t rsX = make_rsrc(X + (size_t)i0 * k, (uint64_t)rows * rowbytes);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(A, (uint64_t)r * rowbytes);
  const uint32_t kb8 = (uint32_t)k / 8;          // keep bytes per token (k % 64 == 0 with dropout)
  const __amdgpu_buffer_rsrc_t rsK =
      make_rsrc(KEEP ? (const void*)(keep + (size_t)i0 * kb8) : (const void*)X, KEEP ? (uint64_t)rows * kb8 : 0);
  char* ring = smem + wave * NSW * STAGE;

  // Copy c of a stage fills 8 rows: X rows 8c .. 8c+7 (8c < TPW), else A rows
  // 8c - TPW .. +7 at stage rows XR + 8c - TPW ..; this lane's row lane/8 of
  // the eight at physical chunk lane%8, which holds logical chunk
  // (lane%8) ^ kc_swz(stage row).  Rows past m or r, k past the end and stages
  // past the wave's last read zero.
  const int c8 = lane & 7, r8 = lane >> 3;
  const int nst = (k + 63) / 64;
  auto issue = [&](int j, int buf) LORA_INLINE {   // the wave's j-th stage
    const int st = wave + NWV * j;
    const int k0 = st * 64;
    const bool live = st < nst;
    char* sb = ring + buf * STAGE;
#pragma unroll
    for (int c = 0; c < CPS; ++c) {
      const bool isx = 8 * c < TPW;   // uniform
      const int row = 8 * c + r8;
      const int srow = isx ? row : row + (XR - TPW);   // stage row
      const int lc = c8 ^ kc_swz(srow);
      const int grow = isx ? row : row - TPW;
      const uint32_t off = live && k0 + 8 * lc < k ? (uint32_t)grow * rowbytes + (uint32_t)(k0 + 8 * lc) * 2 : kOOB;
      dma16(isx ? rsX : rsA, off, 0, sb + (isx ? c : c + (XR - TPW) / 8) * 1024);
    }
    if (KEEP)   // lane l: bytes 4 (l % 2) .. +3 of token l / 2's stage bits (lanes past TPW tokens: zero)
      dma4(rsK, live && (lane >> 1) < TPW ? (uint32_t)(lane >> 1) * kb8 + (uint32_t)k0 / 8 + 4 * (lane & 1) : kOOB,
           0, sb + MOFF);
  };
  floatx4 acc[FT][TG];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) acc[ft][tg] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) LORA_INLINE {
    const char* sb = ring + buf * STAGE;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int ch = 4 * kk + g;
      short8 xf[TG], af[FT];
#pragma unroll
      for (int tg = 0; tg < TG; ++tg) {
        xf[tg] = kc_read(sb, 16 * tg + c16, ch);
        if constexpr (KEEP) xf[tg] = keep_mask8(xf[tg], (uint32_t)(uint8_t)sb[MOFF + (16 * tg + c16) * 8 + ch]);
      }
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) af[ft] = kc_read(sb, XR + 16 * ft + c16, ch);
#pragma unroll
      for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) acc[ft][tg] = mfma16x16x32(af[ft], xf[tg], acc[ft][tg]);
    }
  };

  const int nsw = wave < nst ? (nst - wave + NWV - 1) / NWV : 0;   // this wave's stages
  if constexpr (TPW < 16) {   // the zero X rows TPW .. 15 of every ring stage (8 rows: 16 bytes a lane)
    static_assert(TPW == 8, "one 1 KB block of zero rows");
#pragma unroll
    for (int b = 0; b < NSW; ++b) *reinterpret_cast<int4v*>(ring + b * STAGE + TPW * 128 + lane * 16) = int4v{0, 0, 0, 0};
  }
#pragma unroll
  for (int j = 0; j < NSW - 1; ++j) issue(j, j);
  for (int j = 0; j < nsw; ++j) {
    wait_vmcnt<CPW * (NSW - 2)>();   // the wave's stage j has landed
    issue(j + NSW - 1, (j + NSW - 1) % NSW);   // into the buffer of stage j - 1, read already
    compute(j % NSW);
  }
  wait_vmcnt<0>();   // the trailing copies (zeros) land before the LDS is reused

  // Cross-wave sum in wave order; lane of (ft, tg): rank rows 16 ft + 4 g ..
  // +3 of token 16 tg + c16.
  floatx4* red = reinterpret_cast<floatx4*>(smem);
  __syncthreads();
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) red[((wave * FT + ft) * TG + tg) * 64 + lane] = acc[ft][tg];
  __syncthreads();
  for (int e = wave; e < FT * TG; e += NWV) {
    const int ft = e / TG, tg = e - ft * TG;
    floatx4 v = red[((0 * FT + ft) * TG + tg) * 64 + lane];
#pragma unroll
    for (int w = 1; w < NWV; ++w) v += red[((w * FT + ft) * TG + tg) * 64 + lane];
    const int i = i0 + 16 * tg + c16;
    if (i < m && 16 * tg + c16 < TPW) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = 16 * ft + 4 * g + j;
        if (t < r) U[(size_t)i * r + t] = KEEP ? inv_keep * v[j] : v[j];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The 128 x 256 tile for rank <= 16, the k substeps of each stage split between
// wave pairs.  DMA (whole stages, and one round of workgroups or k from 512
// on): fwd_ks_tile.
// Otherwise the same split with both halves of a pair in step and the stages
// staged in registers two ahead, stored to the free one of two LDS buffers
// during the stage before their use.  Wave (wk, wm, wn) multiplies the 64
// tokens wm and the 128 features wn of the tile over substeps 2 wk and 2 wk + 1
// of every 64-wide stage; U as in fwd_ks_tile.  After the k loop wave wk keeps
// feature fragments 2 wk, 2 wk + 1 and sends the other two to its partner, so
// each wave then holds a complete 64 x 64 block (features wn 128 + 64 wk ..).
template <bool GRP, bool KFULL, bool DMA, bool UPRE>
__global__ __launch_bounds__(512) void lora_fwd_ks_kernel(
    const u16* __restrict__ X, const u16* __restrict__ W, const u16* __restrict__ A,
    const u16* __restrict__ B, u16* __restrict__ Y, float* __restrict__ U, int m, int n, int k, int r, float s,
    int tiles_m, int tiles_n, int n_begin, FwdGroup grp) {
  constexpr int BM = 128, BN = 256, NT = 512, RP = 16;
  constexpr int WTI = 64, WTJ = 128, FI = 2, FJ = 4;
  constexpr int GPW = 2;                          // 16-token U groups per wave
  constexpr int RPS = UPRE ? 0 : RP;              // A rows staged per stage
  constexpr int ROWS = BM + BN + RPS;
  constexpr int STAGE = ROWS * 128;
  constexpr int CX = BM * 8, CW = BN * 8, CA = RPS * 8;
  constexpr int LX = CX / NT, LW = CW / NT, LA = UPRE ? 1 : (CA + NT - 1) / NT;
  static_assert(!(UPRE && GRP), "U from the U pass only for single projections");
  constexpr int XCH = 8 * 16 * 1024;              // exchange: 8 waves x 32 fragments x 64 lanes x 4 B
  constexpr int BS_OFF = XCH + 2 * BM * RP * 4;
  constexpr int EPI = BS_OFF + BN * RP * 2;
  constexpr int SMEM = DMA ? fwd_ks_smem<128, 256, 16, UPRE>() : (EPI > 2 * STAGE ? EPI : 2 * STAGE);
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];

  int tm, tn;
  tile_coords(tiles_m, tiles_n, 8, (int)blockIdx.x, tm, tn);
  if constexpr (DMA) {
    fwd_ks_tile<128, 256, 16, GRP, UPRE, KFULL>(X, W, A, B, Y, U, m, n, k, r, s, tm * 128, tn, n_begin, grp, smem);
    return;
  } else {
  if (GRP) {
    int sel = 0;
#pragma unroll
    for (int q = 1; q < kMaxGroup; ++q)
      if (q < grp.count && tn >= grp.tile0[q]) sel = q;
#pragma unroll
    for (int q = 0; q < kMaxGroup; ++q)
      if (q == sel) {
        W = grp.W[q]; A = grp.A[q]; B = grp.B[q]; Y = grp.Y[q]; U = grp.U[q];
        n = grp.n[q];
        tn -= grp.tile0[q];
      }
  }
  const int m0 = tm * BM, n0 = n_begin + tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wk = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
  const int g = lane >> 5, c32 = lane & 31;
  const int g16 = lane >> 4, c16 = lane & 15;

  const uint32_t rowbytes = (uint32_t)k * 2;
  const __amdgpu_buffer_rsrc_t rsX = make_rsrc(X + (size_t)m0 * k, (uint64_t)min(BM, m - m0) * rowbytes);
  const __amdgpu_buffer_rsrc_t rsW = make_rsrc(W + (size_t)n0 * k, (uint64_t)min(BN, n - n0) * rowbytes);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(A, (uint64_t)r * rowbytes);

  // Register staging of one k-block (thread chunk q = tid + i NT of a region is
  // row q/8, k-chunk q%8), stored in two pieces (0 = X and A rows, 1 = W rows),
  // one per substep of the stage.
  int4v gx[LX], gw[LW], ga[LA];
  auto gload = [&](int kb, int piece) LORA_INLINE {
    const int k0 = kb * 64;
    if (piece == 0) {
#pragma unroll
      for (int i = 0; i < LX; ++i) {
        const int q = tid + i * NT;
        const int kk = k0 + 8 * (q & 7);
        gx[i] = buf_load16(rsX, (KFULL || kk < k) ? (uint32_t)(q >> 3) * rowbytes + (uint32_t)kk * 2 : kOOB);
      }
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        if (UPRE) break;
        const int q = tid + i * NT;
        if (CA % NT != 0 && wave * 64 + i * NT >= CA) break;
        const int kk = k0 + 8 * (q & 7);
        ga[i] = buf_load16(rsA, (KFULL || kk < k) ? (uint32_t)(q >> 3) * rowbytes + (uint32_t)kk * 2 : kOOB);
      }
    } else {
#pragma unroll
      for (int i = 0; i < LW; ++i) {
        const int q = tid + i * NT;
        const int kk = k0 + 8 * (q & 7);
        gw[i] = buf_load16(rsW, (KFULL || kk < k) ? (uint32_t)(q >> 3) * rowbytes + (uint32_t)kk * 2 : kOOB);
      }
    }
  };
  auto swrite = [&](int buf, int piece) LORA_INLINE {
    char* sb = smem + buf * STAGE;
    if (piece == 0) {
#pragma unroll
      for (int i = 0; i < LX; ++i) {
        const int q = tid + i * NT;
        *reinterpret_cast<int4v*>(sb + kc_offset(q >> 3, q & 7)) = gx[i];
      }
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        if (UPRE) break;
        const int q = tid + i * NT;
        if (CA % NT != 0 && wave * 64 + i * NT >= CA) break;
        *reinterpret_cast<int4v*>(sb + (BM + BN) * 128 + kc_offset(q >> 3, q & 7)) = ga[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < LW; ++i) {
        const int q = tid + i * NT;
        *reinterpret_cast<int4v*>(sb + BM * 128 + kc_offset(q >> 3, q & 7)) = gw[i];
      }
    }
  };

  floatx16 acc[FJ][FI];
#pragma unroll
  for (int a = 0; a < FJ; ++a)
#pragma unroll
    for (int b = 0; b < FI; ++b) acc[a][b] = floatx16{};
  floatx4 uacc16[GPW];
#pragma unroll
  for (int a = 0; a < GPW; ++a) uacc16[a] = floatx4{0.f, 0.f, 0.f, 0.f};
  int urow16[GPW];
#pragma unroll
  for (int gg = 0; gg < GPW; ++gg) urow16[gg] = wm * WTI + 16 * (wn * GPW + gg) + c16;

  short8 fw[2][FJ], fx[2][FI], fa16, fxu16[GPW];
  // Fragments of the wave's substep j (0, 1), global substep 2 wk + j; the
  // U operands of the wave's 32-wide k half are read with substep 0.
  auto read_frags = [&](const char* sb, int j, int p) LORA_INLINE {
    const char* Xs = sb;
    const char* Ws = sb + BM * 128;
    const char* As = sb + (BM + BN) * 128;
    const int ch = 2 * (2 * wk + j) + g;
#pragma unroll
    for (int fj = 0; fj < FJ; ++fj) fw[p][fj] = kc_read(Ws, wn * WTJ + 32 * fj + c32, ch);
#pragma unroll
    for (int fi = 0; fi < FI; ++fi) fx[p][fi] = kc_read(Xs, wm * WTI + 32 * fi + c32, ch);
    if (!UPRE && j == 0) {   // the wave's 32-wide half: chunks 4 wk + g16
      fa16 = kc_read(As, c16, 4 * wk + g16);
#pragma unroll
      for (int gg = 0; gg < GPW; ++gg) fxu16[gg] = kc_read(Xs, urow16[gg], 4 * wk + g16);
    }
  };
  auto multiply = [&](int p, int j) LORA_INLINE {
#pragma unroll
    for (int fi = 0; fi < FI; ++fi)
#pragma unroll
      for (int fj = 0; fj < FJ; ++fj) acc[fj][fi] = mfma32x32x16(fw[p][fj], fx[p][fi], acc[fj][fi]);
    if (!UPRE && j == 0) {
#pragma unroll
      for (int gg = 0; gg < GPW; ++gg) uacc16[gg] = mfma16x16x32(fa16, fxu16[gg], uacc16[gg]);
    }
  };
  // Two substeps per wave and stage: at the
  // top of stage kb the registers hold block kb+1; each piece is stored to the
  // free buffer and reloaded with block kb+2; fragments of substep 1 are read
  // while substep 0 multiplies.
  auto stage = [&](int kb, auto bufc, bool write_next, bool load_next) LORA_INLINE {
    constexpr int BUF = decltype(bufc)::value;    // -1: the buffer of kb's parity at run time
    const int cur = BUF >= 0 ? BUF : (kb & 1);
    const char* sb = smem + cur * STAGE;
    read_frags(sb, 0, 0);
    if (write_next) swrite(cur ^ 1, 0);
    if (load_next) gload(kb + 2, 0);
    read_frags(sb, 1, 1);
    multiply(0, 0);
    if (write_next) swrite(cur ^ 1, 1);
    if (load_next) gload(kb + 2, 1);
    multiply(1, 1);
    __syncthreads();
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  using BR = std::integral_constant<int, -1>;
  u16* Bs = reinterpret_cast<u16*>(smem + BS_OFF);   // B rows for the epilogue, staged in the prologue
  const int nkb = (k + 63) / 64;
  gload(0, 0);
  gload(0, 1);
  // B rows of the tile for the epilogue, staged once beside the pipeline's
  // buffers: Bs [BN][RP] bf16, zero beyond r and n; thread tid fills entries
  // t0b .. t0b + 7 of row tid / (RP / 8).
  {
    static_assert(BN * RP / 8 == NT, "one chunk of Bs per thread");
    const int j = tid / (RP / 8), t0b = 8 * (tid % (RP / 8));
    int4v v = int4v{0, 0, 0, 0};
    if (j < min(BN, n - n0) && t0b < r) {
      const u16* brow = B + (size_t)(n0 + j) * r;
      if ((r & 7) == 0) {
        v = *reinterpret_cast<const int4v*>(brow + t0b);
      } else {
        uint32_t w[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const uint32_t lo = t0b + 2 * x < r ? brow[t0b + 2 * x] : 0u;
          const uint32_t hi = t0b + 2 * x + 1 < r ? brow[t0b + 2 * x + 1] : 0u;
          w[x] = lo | (hi << 16);
        }
        v = int4v{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
      }
    }
    *reinterpret_cast<int4v*>(Bs + j * RP + t0b) = v;
  }
  swrite(0, 0);
  swrite(0, 1);
  __syncthreads();
  if (nkb > 1) {
    gload(1, 0);
    gload(1, 1);
  }
  int kb = 0;
  if constexpr (KFULL) {
    // k a multiple of 64: no bound checks on the loads, and stages in pairs
    // so that the LDS buffer of every stage is a compile-time constant (its
    // offset rides in the instructions' immediates).  kb is even after the
    // loop and at most three stages remain.
    for (; kb + 3 < nkb; kb += 2) {
      stage(kb, B0{}, true, true);
      stage(kb + 1, B1{}, true, true);
    }
    if (kb < nkb) stage(kb, B0{}, kb + 1 < nkb, kb + 2 < nkb);
    if (kb + 1 < nkb) stage(kb + 1, B1{}, kb + 2 < nkb, kb + 3 < nkb);
    if (kb + 2 < nkb) stage(kb + 2, B0{}, false, false);
  } else {
    for (; kb + 2 < nkb; ++kb) stage(kb, BR{}, true, true);
    if (kb + 1 < nkb) stage(kb++, BR{}, true, false);
    stage(kb, BR{}, false, false);
  }
  // The epilogue's lane-derived values are recomputed from the lane index
  // rather than kept live across the k loop (which runs at the register limit).
  const int lane_e = lane_fresh();
  {
  const int lane = lane_e, tid = wave * 64 + lane_e;
  const int g = lane >> 5, c32 = lane & 31;
  const int g16 = lane >> 4, c16 = lane & 15;
  int urow16[GPW];
#pragma unroll
  for (int gg = 0; gg < GPW; ++gg) urow16[gg] = wm * WTI + 16 * (wn * GPW + gg) + c16;
  // ---- epilogue (LDS is free after the loop's last barrier).  Regions:
  // [0, XCH) the exchange of the k-half partial sums, later the per-wave
  // staging of the bf16 output block; then Us [2][BM][RP] fp32 (the two
  // k-half partials of U, summed in fixed order) and Bs [BN][RP] bf16 (B rows
  // of the tile, zero beyond r and n, staged in the prologue).  Two
  // barriers in all.
  float* Us = reinterpret_cast<float*>(smem + XCH);
  // Exchange region of (pair, destination half h): the partner's fragments
  // [fjl][fi][q4] as float4 x 64 lanes; wave wk keeps feature fragments
  // 2 wk, 2 wk + 1 and sends the other two.
  float4* xb = reinterpret_cast<float4*>(smem);
  const int pair = wm * 2 + wn;
  auto region = [&](int h) LORA_INLINE { return xb + (size_t)((pair * 2 + h) * 16) * 64; };
  {
    float4* dst = region(1 - wk);
#pragma unroll
    for (int fjl = 0; fjl < 2; ++fjl)
#pragma unroll
      for (int fi = 0; fi < FI; ++fi) {
        const floatx16 v = wk == 0 ? acc[2 + fjl][fi] : acc[fjl][fi];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          dst[((fjl * FI + fi) * 4 + q4) * 64 + lane] = float4{v[4 * q4], v[4 * q4 + 1], v[4 * q4 + 2], v[4 * q4 + 3]};
      }
  }
  if (!UPRE) {
#pragma unroll
    for (int gg = 0; gg < GPW; ++gg)
#pragma unroll
      for (int q = 0; q < 4; ++q) Us[(wk * BM + urow16[gg]) * RP + 4 * g16 + q] = uacc16[gg][q];
  }
  __syncthreads();
  {
    const float4* src = region(wk);
#pragma unroll
    for (int fjl = 0; fjl < 2; ++fjl)
#pragma unroll
      for (int fi = 0; fi < FI; ++fi)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const float4 o = src[((fjl * FI + fi) * 4 + q4) * 64 + lane];
          if (wk == 0) {
            acc[fjl][fi][4 * q4] += o.x; acc[fjl][fi][4 * q4 + 1] += o.y;
            acc[fjl][fi][4 * q4 + 2] += o.z; acc[fjl][fi][4 * q4 + 3] += o.w;
          } else {
            acc[2 + fjl][fi][4 * q4] += o.x; acc[2 + fjl][fi][4 * q4 + 1] += o.y;
            acc[2 + fjl][fi][4 * q4 + 2] += o.z; acc[2 + fjl][fi][4 * q4 + 3] += o.w;
          }
        }
  }
  if (UPRE) {   // U of the tile's tokens from the U pass (zero beyond r and m), all loads issued before the first use
    constexpr int UPT = BM * RP / NT;
    static_assert(BM * RP % NT == 0, "U values per thread");
    const __amdgpu_buffer_rsrc_t rsU = make_rsrc(U + (size_t)m0 * r, (uint64_t)min(BM, m - m0) * r * 4);
    float uv[UPT];
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
      const int e = tid + i * NT, il = e / RP, t = e - il * RP;
      uv[i] = buf_load4f(rsU, t < r ? (uint32_t)(il * r + t) * 4 : kOOB);
    }
#pragma unroll
    for (int i = 0; i < UPT; ++i) Us[tid + i * NT] = uv[i];
  } else {
    // (the partial of half 1 is read here and written before the barrier above)
    for (int e = tid; e < BM * RP; e += NT) Us[e] = Us[e] + Us[BM * RP + e];
  }
  __syncthreads();
  if (n0 == 0 && !UPRE) {
    for (int e = tid; e < BM * RP; e += NT) {
      const int il = e / RP, t = e - il * RP;
      if (m0 + il < m && t < r) U[(size_t)(m0 + il) * r + t] = Us[e];
    }
  }
  // acc += s U B^T (high and low bf16 parts of s U), then Y rounded to bf16
  // on the wave's 64 x 64 block: features wn WTJ + 64 wk + 32 fjl, tokens
  // wm WTI + 32 fi, stored through a wave-private LDS region (the exchange
  // region is free after the barrier above).
  auto finish = [&](floatx16 (&a2)[FI], floatx16 (&b2)[FI]) {
    floatx16* own[2] = {a2, b2};
    const int t0 = 8 * g;
    short8 bfr[2];
#pragma unroll
    for (int fjl = 0; fjl < 2; ++fjl) {
      const int jl = wn * WTJ + 64 * wk + 32 * fjl + c32;
      bfr[fjl] = *reinterpret_cast<const short8*>(Bs + jl * RP + t0);
    }
#pragma unroll
    for (int fi = 0; fi < FI; ++fi) {
      const int il = wm * WTI + 32 * fi + c32;
      const float* up = Us + il * RP + t0;
      short8 uh, ul;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v = s * up[e];
        const u16 hi = f32_to_bf16(v);
        uh[e] = (short)hi;
        ul[e] = (short)f32_to_bf16(v - bf16_to_f32(hi));
      }
#pragma unroll
      for (int fjl = 0; fjl < 2; ++fjl) {
        own[fjl][fi] = mfma32x32x16(bfr[fjl], uh, own[fjl][fi]);
        own[fjl][fi] = mfma32x32x16(bfr[fjl], ul, own[fjl][fi]);
      }
    }
    const int j0 = n0 + wn * WTJ + 64 * wk;
#pragma unroll
    for (int fi = 0; fi < FI; ++fi) {
      const int i0 = m0 + wm * WTI + 32 * fi;
      store_block_32x64(a2[fi], b2[fi], smem + wave * kYsBytes, Y + (size_t)i0 * n + j0, (size_t)n, m - i0, n - j0,
                        lane);
    }
  };
  static_assert(8 * kYsBytes <= XCH, "output staging fits the exchange region");
  if (wk == 0) finish(acc[0], acc[1]);
  else finish(acc[2], acc[3]);
  }
  }
}

// ---------------------------------------------------------------------------
// Launchers: execute the plans of lora_plan.hpp.

static hipError_t run_fwd_launch(const Launch& L, const FwdArgs& a, const FwdGroup& grp, hipStream_t st) {
  const dim3 grid((unsigned)L.grid), block((unsigned)L.block);
  if (L.id == K_UPASS) {
    return with_int<16, 32, 64>(L.rp, [&](auto rc) {
      return with_int<8, 16, 32>(L.tpw, [&](auto tc) {
        return with_bool(L.drop, [&](auto kc) {
          hipLaunchKernelGGL((lora_u_kernel<decltype(rc)::value, decltype(tc)::value, decltype(kc)::value>), grid,
                             block, 0, st, a.X, a.keep, (int)a.m, (int)a.k, (int)a.r, a.inv_keep, L.tiles_m, grp);
          return hipGetLastError();
        });
      });
    });
  }
  if (L.id == K_FWD_KS) {
    return with_bool(L.grp, [&](auto gc) {
      return with_bool(L.full, [&](auto fc) {
        return with_bool(L.dma, [&](auto dc) {
          return with_bool(L.upre, [&](auto uc) {
            constexpr bool G = decltype(gc)::value, F = decltype(fc)::value, D = decltype(dc)::value,
                           UP = decltype(uc)::value;
            if constexpr ((D && !F) || (UP && (G || !F))) {   // (U from the pass: dropout, k a multiple of 64)
              return hipErrorInvalidValue;
            } else {
              hipLaunchKernelGGL((lora_fwd_ks_kernel<G, F, D, UP>), grid, block, 0, st, a.X, a.W, a.A, a.B, a.Y,
                                 a.U, (int)a.m, (int)a.n, (int)a.k, (int)a.r, a.s, L.tiles_m, L.tiles_n,
                                 (int)L.col_begin, grp);
              return hipGetLastError();
            }
          });
        });
      });
    });
  }
  if (L.id == K_FWD_SKINNY) return launch_fwd_skinny(L, a, grp, st);
  if (L.id == K_FWD_REG) {
    return with_int<16, 32, 64>(L.rp, [&](auto rc) {
      return with_bool(L.grp, [&](auto gc) {
        return with_bool(L.upre, [&](auto uc) {
          return with_bool(L.full, [&](auto fc) {
            constexpr int RP = decltype(rc)::value;
            constexpr bool G = decltype(gc)::value, UP = decltype(uc)::value, F = decltype(fc)::value;
            // U from the pass: single projections beyond rank 16, and under dropout (k a multiple of 64)
            if constexpr (G ? UP : (UP ? RP == 16 && !F : RP != 16)) {
              return hipErrorInvalidValue;
            } else {
              hipLaunchKernelGGL((lora_fwd_reg_kernel<128, 128, 2, 2, RP, G, UP, F>), grid, block, 0, st, a.X, a.W,
                                 a.A, a.B, a.Y, a.U, (int)a.m, (int)a.n, (int)a.k, (int)a.r, a.s, L.tiles_m,
                                 L.tiles_n, (int)L.col_begin, grp);
              return hipGetLastError();
            }
          });
        });
      });
    });
  }
  if (L.id != K_FWD && L.id != K_FWD_PAIR) return hipErrorInvalidValue;
  // U comes from the tile only at rank 16 and below the 256 x 256 tile, 128 x
  // 192 serves single projections, and 128 x 256 at rank 16 is K_FWD_KS's.
  const int tile = L.id == K_FWD_PAIR ? 64 : tile_code(L);
  return with_int<64, 128, 192, 256, 257>(tile, [&](auto tc) {
    constexpr int T = decltype(tc)::value;
    return with_int<16, 32, 64>(L.rp, [&](auto rc) {
      return with_bool(L.grp, [&](auto gr) {
        return with_bool(L.upre, [&](auto up) {
          return with_bool(L.full, [&](auto kf) {
            constexpr int RP = decltype(rc)::value;
            constexpr bool GRP = decltype(gr)::value, UPRE = decltype(up)::value, KF = decltype(kf)::value;
            if constexpr ((!UPRE && (RP != 16 || T == 257)) || (T == 256 && RP == 16) || (T == 192 && GRP) ||
                          (UPRE && RP == 16 && T != 257 && (GRP || !KF))) {
              return hipErrorInvalidValue;
            } else if constexpr (T == 64) {
              hipLaunchKernelGGL((lora_fwd_pair_ks_kernel<RP, GRP, KF, UPRE>), grid, block, 0, st, a.X, a.W, a.A, a.B,
                                 a.Y, a.U, (int)a.m, (int)a.n, (int)a.k, (int)a.r, a.s, L.tiles_m, L.tiles_n,
                                 (int)L.col_begin, grp);
              return hipGetLastError();
            } else {
              constexpr bool BIG = T == 257;
              hipLaunchKernelGGL((lora_fwd_kernel<BIG ? 256 : 128, BIG ? 256 : T, 2, BIG ? 4 : 2, RP, GRP, UPRE, KF, BIG>),
                                 grid, block, 0, st, a.X, a.W, a.A, a.B, a.Y, a.U, (int)a.m, (int)a.n, (int)a.k,
                                 (int)a.r, a.s, L.tiles_m, L.tiles_n, (int)L.col_begin, grp);
              return hipGetLastError();
            }
          });
        });
      });
    });
  });
}

hipError_t launch_fwd(const FwdArgs& a, hipStream_t st) {
  const Plan p = plan_fwd(a.m, a.n, a.k, a.r, a.keep != nullptr);
  FwdGroup one{};   // the projection as a group of one (the U pass and the few-token forward read it)
  one.W[0] = a.W; one.A[0] = a.A; one.B[0] = a.B; one.Y[0] = a.Y; one.U[0] = a.U;
  one.n[0] = (int)a.n;
  one.count = 1;
  for (int i = 0; i < p.count; ++i) {
    const hipError_t e = run_fwd_launch(p.l[i], a, one, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// One launch for the whole group: each projection owns a run of column tiles
// (tile0 filled here for the plan's tile width).
hipError_t launch_fwd_group(const GroupFwdArgs& a, hipStream_t st) {
  const Plan p = plan_group_fwd(a.count, a.n, a.m, a.k, a.r);
  if (a.count == 1) {   // a group of one is the single projection
    FwdArgs f{};
    f.X = a.X; f.W = a.W[0]; f.A = a.A[0]; f.B = a.B[0]; f.Y = a.Y[0]; f.U = a.U[0];
    f.m = a.m; f.n = a.n[0]; f.k = a.k; f.r = a.r; f.s = a.s;
    return launch_fwd(f, st);
  }
  FwdGroup grp{};
  for (int g = 0; g < a.count; ++g) {
    grp.W[g] = a.W[g]; grp.A[g] = a.A[g]; grp.B[g] = a.B[g]; grp.Y[g] = a.Y[g]; grp.U[g] = a.U[g];
    grp.n[g] = (int)a.n[g];
  }
  grp.count = a.count;
  FwdArgs f{};
  f.X = a.X;
  f.m = a.m; f.n = 0; f.k = a.k; f.r = a.r; f.s = a.s;
  for (int i = 0; i < p.count; ++i) {
    const Launch& L = p.l[i];
    int t0 = 0;
    for (int g = 0; g < a.count && L.bn > 0; ++g) {   // (the U pass has no column tiles)
      grp.tile0[g] = t0;
      t0 += (grp.n[g] + L.bn - 1) / L.bn;
    }
    const hipError_t e = run_fwd_launch(L, f, grp, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lora
