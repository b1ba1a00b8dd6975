// Forward tile of 128 x 128 with its stages staged in registers, two
// workgroups to a compute unit:
//   Y = X W^T + s U B^T,   U = X A^T formed beside W at any rank, or read back.
#pragma once

#include <type_traits>

#include "lora_device.hpp"
#include "lora_fwd_ks.hpp"
#include "lora_launch.hpp"

namespace lora {

// Four waves of 64 x 64, all in step on 32x32x16 products; k runs in stages of
// 64 in two LDS buffers.  No sums are exchanged between waves, half the LDS and
// half the waves of the turn-taking tiles, so two workgroups share a compute
// unit and one's loads and epilogue run under the other's products: the faster
// tile where a launch is few stages of up to 512 tiles, and where rows of k no
// multiple of 64 lie unaligned.
//
// U products: at RP = 16 on 16x16x32 products, a wave row's four groups of 16
// tokens split between its two waves, over the 32-wide halves of the stage
// (substeps 0-1 and 2-3); from RP = 32 on 32x32x16 products, one 32-token
// fragment per wave.  UPRE: U comes from lora_u_kernel.  GRP: the projection of
// a grouped launch is selected first.  KFULL (k a multiple of 64): no k-bound
// checks on the loads, and stages in pairs with compile-time LDS buffers.
template <int BM, int BN, int WM, int WN, int RP, bool GRP, bool UPRE, bool KFULL>
__global__ __launch_bounds__(256, 2) void lora_fwd_reg_kernel(
    const u16* __restrict__ X, const u16* __restrict__ W, const u16* __restrict__ A, const u16* __restrict__ B,
    u16* __restrict__ Y, float* __restrict__ U, int m, int n, int k, int r, float s, int tiles_m, int tiles_n,
    int n_begin, FwdGroup grp) {
  constexpr int NW = WM * WN, NT = 64 * NW;
  constexpr int WTI = BM / WM, WTJ = BN / WN, FI = 2, FJ = 2;   // tokens, features and their 32-wide fragments per wave
  static_assert(BM == 128 && BN == 128 && WM == 2 && WN == 2, "wave tile");
  constexpr bool U16 = RP == 16;
  constexpr int FT = U16 ? 1 : RP / 32;          // U row fragments (A operand)
  constexpr int GPW = 2;                         // 16-token U groups per wave
  constexpr int RPS = UPRE ? 0 : RP;             // A rows staged per stage
  constexpr int ROWS = BM + BN + RPS;            // 128-byte rows per 64-wide stage
  constexpr int STAGE = ROWS * 128;
  constexpr int CX = BM * 8, CW = BN * 8, CA = RPS * 8;  // 16-byte chunks per region
  constexpr int LX = CX / NT, LW = CW / NT, LA = UPRE ? 1 : (CA + NT - 1) / NT;
  static_assert(2 * 2 * STAGE <= 160 * 1024, "LDS of two workgroups");
  constexpr int RPU = 2 * RP + 8, RPB = RP + 8;   // padded row lengths of the epilogue's U and B copies
  static_assert(BM * RPU * 2 + BN * RPB * 2 <= 2 * STAGE, "epilogue LDS reuse");

  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];

  int tm, tn;
  tile_coords(tiles_m, tiles_n, 8, (int)blockIdx.x, tm, tn);
  if (GRP) {   // projection of this column tile (uniform; compile-time indices only)
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
  const int wm = wave / WN, wn = wave % WN;
  const int g = lane >> 5, c32 = lane & 31;
  const int g16 = lane >> 4, c16 = lane & 15;

  const uint32_t rowbytes = (uint32_t)k * 2;
  const __amdgpu_buffer_rsrc_t rsX = make_rsrc(X + (size_t)m0 * k, (uint64_t)min(BM, m - m0) * rowbytes);
  const __amdgpu_buffer_rsrc_t rsW = make_rsrc(W + (size_t)n0 * k, (uint64_t)min(BN, n - n0) * rowbytes);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(A, (uint64_t)r * rowbytes);

  // Register staging of one k-block of the three regions: thread chunk
  // q = tid + i NT of a region is row q/8, k-chunk q%8 (coalesced 128-byte
  // rows).  The block moves in four pieces, one per 16-wide substep of the
  // stage that stores it: 0 = X rows, 1 and 2 = the two halves of the W rows,
  // 3 = A rows.
  constexpr int LW1 = (LW + 1) / 2;
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
    } else if (piece <= 2) {
#pragma unroll
      for (int i = piece == 1 ? 0 : LW1; i < (piece == 1 ? LW1 : LW); ++i) {
        const int q = tid + i * NT;
        const int kk = k0 + 8 * (q & 7);
        gw[i] = buf_load16(rsW, (KFULL || kk < k) ? (uint32_t)(q >> 3) * rowbytes + (uint32_t)kk * 2 : kOOB);
      }
    } else if (!UPRE) {
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int q = tid + i * NT;
        if (CA % NT != 0 && wave * 64 + i * NT >= CA) break;   // wave-uniform
        const int kk = k0 + 8 * (q & 7);
        ga[i] = buf_load16(rsA, (KFULL || kk < k) ? (uint32_t)(q >> 3) * rowbytes + (uint32_t)kk * 2 : kOOB);
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
    } else if (piece <= 2) {
#pragma unroll
      for (int i = piece == 1 ? 0 : LW1; i < (piece == 1 ? LW1 : LW); ++i) {
        const int q = tid + i * NT;
        *reinterpret_cast<int4v*>(sb + BM * 128 + kc_offset(q >> 3, q & 7)) = gw[i];
      }
    } else if (!UPRE) {
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int q = tid + i * NT;
        if (CA % NT != 0 && wave * 64 + i * NT >= CA) break;   // wave-uniform
        *reinterpret_cast<int4v*>(sb + (BM + BN) * 128 + kc_offset(q >> 3, q & 7)) = ga[i];
      }
    }
  };

  floatx16 acc[FJ][FI];
  floatx16 uacc[FT];           // U on the 32x32x16 form (RP >= 32)
  floatx4 uacc16[GPW];         // U on the 16x16x32 form (RP = 16)
#pragma unroll
  for (int a = 0; a < GPW; ++a) uacc16[a] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int a = 0; a < FJ; ++a)
#pragma unroll
    for (int b = 0; b < FI; ++b) acc[a][b] = floatx16{};
#pragma unroll
  for (int a = 0; a < FT; ++a) uacc[a] = floatx16{};
  const int urow = wm * WTI + 32 * wn + c32;   // the wave's U tokens (RP >= 32)
  int urow16[GPW];
#pragma unroll
  for (int gg = 0; gg < GPW; ++gg) urow16[gg] = wm * WTI + 16 * (wn * GPW + gg) + c16;

  // Fragments of the next 16-wide substep are read while the current one
  // multiplies (two register sets, p = substep parity).
  short8 fw[2][FJ], fx[2][FI], fa[2][FT], fxu[2];
  short8 fa16[2], fxu16[2][GPW];
  auto read_frags = [&](const char* sb, int ks, int p) LORA_INLINE {
    const char* Xs = sb;
    const char* Ws = sb + BM * 128;
    const char* As = sb + (BM + BN) * 128;
    const int ch = 2 * ks + g;
#pragma unroll
    for (int fj = 0; fj < FJ; ++fj) fw[p][fj] = kc_read(Ws, wn * WTJ + 32 * fj + c32, ch);
#pragma unroll
    for (int fi = 0; fi < FI; ++fi) fx[p][fi] = kc_read(Xs, wm * WTI + 32 * fi + c32, ch);
    if (UPRE) {
    } else if (U16) {
      if (ks % 2 == 0) {   // the 32-wide half starting at substep ks: chunks 2 ks + g16
        fa16[p] = kc_read(As, c16, 2 * ks + g16);
#pragma unroll
        for (int gg = 0; gg < GPW; ++gg) fxu16[p][gg] = kc_read(Xs, urow16[gg], 2 * ks + g16);
      }
    } else {
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) fa[p][ft] = kc_read(As, 32 * ft + c32, ch);
      fxu[p] = kc_read(Xs, urow, ch);
    }
  };
  auto multiply = [&](int p, int ks) LORA_INLINE {
#pragma unroll
    for (int fi = 0; fi < FI; ++fi)
#pragma unroll
      for (int fj = 0; fj < FJ; ++fj) acc[fj][fi] = mfma32x32x16(fw[p][fj], fx[p][fi], acc[fj][fi]);
    if (UPRE) {
    } else if (U16) {
      if (ks % 2 == 0) {
#pragma unroll
        for (int gg = 0; gg < GPW; ++gg) uacc16[gg] = mfma16x16x32(fa16[p], fxu16[p][gg], uacc16[gg]);
      }
    } else {
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) uacc[ft] = mfma32x32x16(fa[p][ft], fxu[p], uacc[ft]);
    }
  };

  // Pipeline.  At the top of stage kb the staging registers hold k-block
  // kb+1 (loaded one stage earlier); piece ks of it is stored to the free LDS
  // buffer at substep ks, and its registers are then reloaded with block kb+2.
  // The loop is rotated by one substep: the products of substep 3 of stage kb-1
  // are issued after the barrier, while the first fragments of stage kb are being
  // read (their operands are zeroed for stage 0, adding exact zeros).  The k loop
  // is peeled so the steady state carries no conditionals.
  {
#pragma unroll
    for (int j = 0; j < FJ; ++j) fw[1][j] = short8{};
#pragma unroll
    for (int j = 0; j < FI; ++j) fx[1][j] = short8{};
#pragma unroll
    for (int j = 0; j < FT; ++j) fa[1][j] = short8{};
    fxu[1] = short8{};
    fa16[1] = short8{};
#pragma unroll
    for (int j = 0; j < GPW; ++j) fxu16[1][j] = short8{};
  }
  // bufc: the stage's LDS buffer as a compile-time constant, or -1 for the
  // parity of kb at run time
  auto stage = [&](int kb, auto bufc, bool write_next, bool load_next) LORA_INLINE {
    constexpr int BUF = decltype(bufc)::value;
    const int cur = BUF >= 0 ? BUF : (kb & 1);
    const char* sb = smem + cur * STAGE;
    read_frags(sb, 0, 0);
    multiply(1, 3);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (write_next) swrite(cur ^ 1, ks);
      if (load_next) gload(kb + 2, ks);
      if (ks < 3) read_frags(sb, ks + 1, (ks + 1) & 1);
      if (ks < 3) multiply(ks & 1, ks);
    }
    __syncthreads();
  };
  const int nkb = (k + 63) / 64;
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  using BR = std::integral_constant<int, -1>;
#pragma unroll
  for (int pc = 0; pc < 4; ++pc) gload(0, pc);
#pragma unroll
  for (int pc = 0; pc < 4; ++pc) swrite(0, pc);
  __syncthreads();
  if (nkb > 1) {
#pragma unroll
    for (int pc = 0; pc < 4; ++pc) gload(1, pc);
  }
  int kb = 0;
  if constexpr (KFULL) {
    for (; kb + 3 < nkb; kb += 2) {
      stage(kb, B0{}, true, true);
      stage(kb + 1, B1{}, true, true);
    }
  }
  for (; kb + 2 < nkb; ++kb) stage(kb, BR{}, true, true);
  if (kb + 1 < nkb) stage(kb++, BR{}, true, false);
  stage(kb, BR{}, false, false);
  multiply(1, 3);

  // ---- epilogue: LDS reuse as in the 256 x 256 tile: Us [BM][RPU] bf16 (s U as
  // high and low parts), then Bs [BN][RPB] bf16.  U goes to memory from the
  // registers of the first tile column's workgroups.
  u16* Us = reinterpret_cast<u16*>(smem);
  u16* Bs = reinterpret_cast<u16*>(smem + BM * RPU * 2);
  constexpr int BCH = (BN * RP / 8 + NT - 1) / NT;   // chunks per thread (r <= RP)
  const int jn = min(BN, n - n0);
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B + (size_t)n0 * r, (uint64_t)jn * r * 2);
  int4v bv[BCH];
  load_b_rows<RP, NT>(rsB, r, jn, tid, bv);
  // ranks t .. t + 3 of token il, from the lane that holds them
  auto put_u = [&](int il, int t, const float* v) LORA_INLINE {
    u16 hi[4], lo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float x = s * v[q];
      hi[q] = f32_to_bf16(x);
      lo[q] = f32_to_bf16(x - bf16_to_f32(hi[q]));
      if (n0 == 0 && m0 + il < m && t + q < r) U[(size_t)(m0 + il) * r + t + q] = v[q];
    }
    *reinterpret_cast<uint2*>(Us + il * RPU + t) =
        uint2{(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16)};
    *reinterpret_cast<uint2*>(Us + il * RPU + RP + t) =
        uint2{(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16)};
  };
  if constexpr (UPRE) {
    const __amdgpu_buffer_rsrc_t rsU = make_rsrc(U + (size_t)m0 * r, (uint64_t)min(BM, m - m0) * r * 4);
    float uv[BM * RP / NT];
    load_u_pairs<BM, RP, NT>(rsU, r, tid, uv);
    split_u_pairs<BM, RP, NT>(uv, s, tid, Us);
  } else if constexpr (U16) {   // lane holds token column c16 of its group, ranks 4 g16 .. +3
#pragma unroll
    for (int gg = 0; gg < GPW; ++gg) {
      const float v[4] = {uacc16[gg][0], uacc16[gg][1], uacc16[gg][2], uacc16[gg][3]};
      put_u(urow16[gg], 4 * g16, v);
    }
  } else {
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const float v[4] = {uacc[ft][4 * q4], uacc[ft][4 * q4 + 1], uacc[ft][4 * q4 + 2], uacc[ft][4 * q4 + 3]};
        put_u(urow, 32 * ft + 8 * q4 + 4 * g, v);
      }
  }
  store_b_rows<BN, RP, NT>(bv, r, jn, tid, Bs);
  __syncthreads();

  // acc += s U B^T, formed as Y^T += B (sU)^T over t in blocks of 16, each
  // block once with the high and once with the low bf16 part of sU.
  const int tblocks = (r + 15) / 16;
  for (int tb = 0; tb < tblocks; ++tb) {
    const int t0 = 16 * tb + 8 * g;
    short8 bfr[FJ];
#pragma unroll
    for (int fj = 0; fj < FJ; ++fj)
      bfr[fj] = *reinterpret_cast<const short8*>(Bs + (wn * WTJ + 32 * fj + c32) * RPB + t0);
#pragma unroll
    for (int fi = 0; fi < FI; ++fi) {
      const u16* up = Us + (wm * WTI + 32 * fi + c32) * RPU + t0;
      const short8 uh = *reinterpret_cast<const short8*>(up), ul = *reinterpret_cast<const short8*>(up + RP);
#pragma unroll
      for (int fj = 0; fj < FJ; ++fj) {
        acc[fj][fi] = mfma32x32x16(bfr[fj], uh, acc[fj][fi]);
        acc[fj][fi] = mfma32x32x16(bfr[fj], ul, acc[fj][fi]);
      }
    }
  }

  // store Y: each wave's 32-token blocks of its 64 features through a
  // wave-private LDS region (free once every wave is past the reads above)
  static_assert(FJ == 2 && NW * kYsBytes <= 2 * STAGE, "output staging");
  __syncthreads();
  const int j0 = n0 + wn * WTJ;
#pragma unroll
  for (int fi = 0; fi < FI; ++fi) {
    const int i0 = m0 + wm * WTI + 32 * fi;
    store_block_32x64(acc[0][fi], acc[1][fi], smem + wave * kYsBytes, Y + (size_t)i0 * n + j0, (size_t)n, m - i0,
                      n - j0, lane);
  }
}

}  // namespace lora
