// Forward tiles of 128 tokens x 128, 192 or 256 features with the k substeps
// of each stage split between wave pairs:
//   Y = X W^T + s U B^T,   U = X A^T formed beside W or read back.
#pragma once

#include <type_traits>

#include "lora_device.hpp"
#include "lora_launch.hpp"

namespace lora {

// Epilogue operands of the forward tiles beyond rank 16 and of the 256 x 256
// one.  U of BM tokens, in pairs of ranks (zero beyond r and the resource).
template <int BM, int RP, int NT>
__device__ __forceinline__ void load_u_pairs(__amdgpu_buffer_rsrc_t rsU, int r, int tid, float (&uv)[BM * RP / NT]) {
  static_assert(BM * RP % (2 * NT) == 0, "pairs per thread");
#pragma unroll
  for (int i = 0; i < BM * RP / NT / 2; ++i) {
    const int e = 2 * (tid + i * NT), il = e / RP, t = e - il * RP;
#pragma unroll
    for (int h = 0; h < 2; ++h) uv[2 * i + h] = buf_load4f(rsU, t + h < r ? (uint32_t)(il * r + t + h) * 4 : kOOB);
  }
}
// s U as bf16 high and low parts: Us rows of RP high, RP low and 8 unused.
template <int BM, int RP, int NT>
__device__ __forceinline__ void split_u_pairs(const float (&uv)[BM * RP / NT], float s, int tid, u16* Us) {
#pragma unroll
  for (int i = 0; i < BM * RP / NT / 2; ++i) {
    const int e = 2 * (tid + i * NT), il = e / RP, t = e - il * RP;
    uint32_t hi = 0, lo = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float v = s * uv[2 * i + h];
      const u16 top = f32_to_bf16(v);
      hi |= (uint32_t)top << (16 * h);
      lo |= (uint32_t)f32_to_bf16(v - bf16_to_f32(top)) << (16 * h);
    }
    *reinterpret_cast<uint32_t*>(Us + il * (2 * RP + 8) + t) = hi;
    *reinterpret_cast<uint32_t*>(Us + il * (2 * RP + 8) + RP + t) = lo;
  }
}
// B rows of BN features in 16-byte chunks: the tile's rows (contiguous) in order,
// or, for r a multiple of 8, where each chunk lies inside one row, by their place
// in the padded [BN][RP] block.
template <int RP, int NT, int BCH>
__device__ __forceinline__ void load_b_rows(__amdgpu_buffer_rsrc_t rsB, int r, int jn, int tid, int4v (&bv)[BCH]) {
  const bool whole = (r & 7) == 0;
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int q = tid + i * NT, j = q / (RP / 8), t0 = 8 * (q % (RP / 8));
    bv[i] = buf_load16(rsB, whole ? (t0 < r ? (uint32_t)(j * r + t0) * 2 : kOOB)
                                  : (q < jn * r / 8 ? (uint32_t)q * 16 : kOOB));   // (exact: jn is a multiple of 8)
  }
}
// The same into Bs [BN][RP + 8], zero beyond r and n.  Contains a barrier for
// other ranks (uniform).
template <int BN, int RP, int NT, int BCH>
__device__ __forceinline__ void store_b_rows(const int4v (&bv)[BCH], int r, int jn, int tid, u16* Bs) {
  constexpr int RPB = RP + 8;
  if ((r & 7) == 0) {
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
      const int q = tid + i * NT;
      if (q < BN * RP / 8) *reinterpret_cast<int4v*>(Bs + q / (RP / 8) * RPB + 8 * (q % (RP / 8))) = bv[i];
    }
    return;
  }
  for (int e = tid; e < BN * RPB / 8; e += NT) reinterpret_cast<int4v*>(Bs)[e] = int4v{0, 0, 0, 0};
  __syncthreads();
  // element idx of the chunks is B row idx / r, column idx % r; the quotient
  // comes from a float product that stays at least 0.5/r away from an integer
  const float rinv = 1.0f / (float)r;
  const int nch = jn * r / 8;
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int q = tid + i * NT;
    if (q < nch) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int idx = 8 * q + e;
        const int j = (int)(((float)idx + 0.5f) * rinv);
        const int t = idx - j * r;
        Bs[j * RPB + t] = (u16)((uint32_t)bv[i][e >> 1] >> (16 * (e & 1)));
      }
    }
  }
}

// Eight waves: wave (wk, wm, wn) multiplies the 64 tokens wm and the BN / 2
// features wn of the tile over substeps 2 wk and 2 wk + 1 of every 64-wide
// stage (the 32-wide k half wk); waves w and w + 4, the two k halves of one
// block, share a SIMD.  The stages (X[128 rows], W[BN rows] and, without UPRE,
// A padded to 16 rows, 128 bytes a row with the kc_offset swizzle) are copied
// straight into NBUF LDS buffers, NBUF - 1 stages ahead.
//
// The two halves take turns: while the waves wk = 0 multiply, the waves wk = 1
// read the fragments of their half of the stage and issue the copies of a
// later one, then they swap, with a workgroup barrier at each change (the
// waves wk = 1 run one slot behind).  So one wave of every SIMD is always
// multiplying and its partner's LDS latency is hidden, where the same loop
// with both waves in step waits for the first fragments after each barrier.
// Measured (weights rotated past the caches; forward kernel alone, U beside W,
// against the same shapes on the previous tiles): 2048 x 4096 x 4096, r = 8: 73
// -> 68 us with the halves taking turns on 32x32x16 products, 63.7 on the
// 16x16x32 ones used here, whose X fragments also feed the U products; 333 x
// 4096 x 4096: 44 us on 96 workgroups of 128 x 128 with four waves in step, 37
// with this loop, 28.8 as 192 half tiles; 1024 x 5120 x 13824, r = 32: 174 us on
// 128 x 256 tiles, 153 on 128 x 192.  A slot lasts about as long as its LDS
// traffic: at 128 x 128 36 KB of reads and 17 KB of copies, 0.23 us, against
// 0.13 us of products.  Issuing the copies before the reads is 2 to 5% slower;
// s_setprio around the products makes no difference here.
//
// Ordering.  Slot 2 kb holds the reads of half 0 and slot 2 kb + 1 those of
// half 1 of stage kb.  Every wave waits for its LDS reads before the barrier
// that ends its read slot, so a buffer is free once both read slots are over:
// the copies of stage kb + NBUF - 1 go to the buffer of stage kb - 1 in the
// read slots of stage kb.  Copies of stage kb + 1 are waited for (vmcnt,
// leaving those of NBUF - 2 later stages in flight) before the barrier that
// ends slot 2 kb + 1: by half 1 in its read slot, by half 0 after its products.
//
// BM = 64 (half of a paired 128 x 128 tile): four k shares instead of two, the
// stages 128 wide (two 64-wide pieces), waves 0 .. 3 on the first piece.
//
// After the k loop the partial sums of each output are added in k-share order
// through LDS, every wave finishing a share of the tokens of its block.  U:
// wave (wk, wm, wn) multiplies A with its own X fragments of the tokens 32 wn ..
// + 31 of its block, over its k share; the first tile column writes U.  s U B^T
// is added as in the 256 x 256 tile.  GRP selects the projection of a grouped
// launch; UPRE reads U from the U pass.  KFULL: k a multiple of 64 (otherwise
// each copy checks its k bound).
template <int BM, int BN, int RP, bool GRP, bool UPRE, bool KFULL>
__device__ __forceinline__ void fwd_ks_tile(const u16* __restrict__ X, const u16* __restrict__ W,
                                            const u16* __restrict__ A, const u16* __restrict__ B,
                                            u16* __restrict__ Y, float* __restrict__ U, int m, int n, int k, int r,
                                            float s, int m0, int tn, int n_begin, const FwdGroup& grp, char* smem) {
  constexpr int NT = 512, WTJ = BN / 2, NA = WTJ / 16;   // features per wave, in fragments of 16
  constexpr int WM = BM / 64, NK = 4 / WM;        // waves along the tokens, k shares
  constexpr int KP = NK / 2;                      // 64-wide k pieces per stage
  constexpr int ROWS = BM + BN + (UPRE ? 0 : 16);
  constexpr int PIECE = ROWS * 128, STAGE = KP * PIECE;
  constexpr bool EARLY_B = RP == 16;              // B staged beside the pipeline's buffers
  constexpr int BS_EARLY = EARLY_B ? BN * RP * 2 : 0;
  constexpr int NBUF = (160 * 1024 - BS_EARLY) / STAGE < 4 ? (160 * 1024 - BS_EARLY) / STAGE : 4;
  constexpr int NCOPY = KP * (BM / 64 + BN / 64);  // copies per wave and stage
  constexpr int NCA = UPRE ? 0 : 2 * KP;          // waves 0 .. NCA - 1: one more, for A
  constexpr int NOB = 4 / NK;                     // token fragments a wave finishes
  constexpr int XCH = 8 * (NK == 2 ? 2 : 4) * NA * 1024;   // exchanged fragments of 64 lanes x 4 floats
  static_assert((BM == 128 || (BM == 64 && BN == 128)), "tile shapes");
  static_assert(NBUF >= 3 && (UPRE || RP == 16), "pipeline depth; U beside W only up to rank 16");

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
  const int n0 = n_begin + tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wk = wave / (2 * WM), wm = (wave >> 1) % WM, wn = wave & 1;
  const bool second = wave >= 4;                   // the waves that run one slot behind
  const int g = lane >> 4, c16 = lane & 15;

  const uint32_t rowbytes = (uint32_t)k * 2;
  const __amdgpu_buffer_rsrc_t rsX = make_rsrc(X + (size_t)m0 * k, (uint64_t)min(BM, m - m0) * rowbytes);
  const __amdgpu_buffer_rsrc_t rsW = make_rsrc(W + (size_t)n0 * k, (uint64_t)min(BN, n - n0) * rowbytes);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(A, (uint64_t)r * rowbytes);
  const int nkb = (k + 64 * KP - 1) / (64 * KP);

  // Copy i of a region fills its rows 64 i + 8 wave .. + 7: lane l takes
  // position l % 8 of row l / 8 of the eight, which holds logical chunk
  // (l % 8) ^ kc_swz(row) (the same for every i).
  const int r8 = 8 * wave + (lane >> 3);
  const int kcol = 8 * ((lane & 7) ^ kc_swz(r8));
  const uint32_t voff = (uint32_t)r8 * rowbytes + (uint32_t)kcol * 2;
  auto dload = [&](int kb, int boff) LORA_INLINE {
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      const int k0 = (kb * KP + p) * 64;
      const uint32_t k0b = (uint32_t)k0 * 2;
      char* sb = smem + boff + p * PIECE + wave * 1024;
      // (a piece that starts past the end has no byte in range either way)
      const bool ok = (KFULL && KP == 1) || k0 + kcol < k;
      const uint32_t so = KP == 1 || k0 < k ? k0b : 0;
#pragma unroll
      for (int i = 0; i < BM / 64; ++i)
        dma16(rsX, ok ? voff + (uint32_t)(64 * i) * rowbytes : kOOB, so, sb + i * 8192);
#pragma unroll
      for (int i = 0; i < BN / 64; ++i)
        dma16(rsW, ok ? voff + (uint32_t)(64 * i) * rowbytes : kOOB, so, sb + BM * 128 + i * 8192);
    }
    if (wave < NCA) {   // A: rows 8 (wave % 2) .. + 7 of piece wave / 2
      const int k0 = (kb * KP + (wave >> 1)) * 64, row = 8 * (wave & 1) + (lane >> 3);
      const int kc = 8 * ((lane & 7) ^ kc_swz(row));
      dma16(rsA, k0 + kc < k ? (uint32_t)row * rowbytes + (uint32_t)(k0 + kc) * 2 : kOOB, 0,
            smem + boff + (wave >> 1) * PIECE + (BM + BN) * 128 + (wave & 1) * 1024);
    }
  };
  // Wait until only the copies of the `later` newest stages are in flight.
  auto wait_copies = [&](auto later) LORA_INLINE {
    constexpr int N = decltype(later)::value;
    if (wave < NCA) wait_vmcnt<N * (NCOPY + 1)>();
    else wait_vmcnt<N * NCOPY>();
  };
  using All = std::integral_constant<int, 0>;
  using Deep = std::integral_constant<int, NBUF - 2>;

#pragma unroll
  for (int st = 0; st < NBUF - 1; ++st)
    if (st < nkb) dload(st, st * STAGE);

  u16* Bs = reinterpret_cast<u16*>(smem + NBUF * STAGE);   // EARLY_B: [BN][RP] bf16, zero beyond r and n
  if constexpr (EARLY_B) {
    if (tid < BN * 2) {
      const int j = tid >> 1, t0b = 8 * (tid & 1);
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
  }

  // acc[a][b]: features 16 a .. of the wave's block, tokens 16 (b ^ 2 wn) .. (in
  // this order a wave's share of U is always its fragments b = 0, 1).
  floatx4 acc[NA][4];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  floatx4 uacc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};

  short8 fw[NA], fx[4], fa;
  auto reads = [&](int boff) LORA_INLINE {
    const char* Xs = smem + boff + (wk >> 1) * PIECE;
    const char* Ws = Xs + BM * 128;
    const char* As = Xs + (BM + BN) * 128;
    const int ch = 4 * (wk & 1) + g;
#pragma unroll
    for (int b = 0; b < 4; ++b) fx[b] = kc_read(Xs, wm * 64 + 16 * (b ^ (2 * wn)) + c16, ch);
#pragma unroll
    for (int a = 0; a < NA; ++a) fw[a] = kc_read(Ws, wn * WTJ + 16 * a + c16, ch);
    if (!UPRE) fa = kc_read(As, c16, ch);
  };
  auto multiply = [&]() LORA_INLINE {
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = mfma16x16x32(fw[a], fx[b], acc[a][b]);
    if (!UPRE) {
      uacc[0] = mfma16x16x32(fa, fx[0], uacc[0]);
      uacc[1] = mfma16x16x32(fa, fx[1], uacc[1]);
    }
  };
  auto slot_end = [&]() LORA_INLINE {
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  if (nkb >= NBUF - 1) wait_copies(Deep{});
  else wait_copies(All{});
  wait_lgkm0();
  slot_end();                    // stage 0 and B are staged
  if (second) slot_end();        // half 1 runs one slot behind
  int rb = 0, wb = (NBUF - 1) * STAGE;
  for (int kb = 0; kb < nkb; ++kb) {
    const bool more = kb + NBUF - 1 < nkb;
    reads(rb);
    if (more) dload(kb + NBUF - 1, wb);
    __builtin_amdgcn_sched_barrier(0);
    wait_lgkm0();
    if (second) {
      if (more) wait_copies(Deep{});
      else wait_copies(All{});
    }
    slot_end();
    multiply();
    __builtin_amdgcn_sched_barrier(0);
    if (!second) {
      if (more) wait_copies(Deep{});
      else wait_copies(All{});
    }
    slot_end();
    rb = rb + STAGE == NBUF * STAGE ? 0 : rb + STAGE;
    wb = wb + STAGE == NBUF * STAGE ? 0 : wb + STAGE;
  }
  if (!second) slot_end();

  // ---- epilogue (LDS is free of copies and reads after the last barrier).
  // Lane-derived values are recomputed rather than kept live across the loop.
  const int lane_e = lane_fresh();
  {
    const int lane = lane_e, tid = wave * 64 + lane_e;
    const int g = lane >> 4, c16 = lane & 15;
    // Regions: [0, XCH) the exchange, later the per-wave output staging; at RP =
    // 16, beside it, Us fp32 [BM][RP] (once per k share) and Bs bf16 [BN][RP]; for
    // larger ranks, over it once it has been read, Us bf16 [BM][RPU] (s U as high
    // and low parts) and Bs [BN][RPB].
    constexpr int RPU = RP == 16 ? RP : 2 * RP + 8, RPB = RP == 16 ? RP : RP + 8;
    constexpr int UPT = BM * RP / NT, BCH = (BN * RP / 8 + NT - 1) / NT;
    float* Us = reinterpret_cast<float*>(smem + (EARLY_B ? XCH : 0));
    u16* Bs2 = EARLY_B ? Bs : reinterpret_cast<u16*>(smem + BM * RPU * 2);
    float uv[UPT];
    int4v bv[EARLY_B ? 1 : BCH];
    const int jn = min(BN, n - n0);
    // The wave finishes fragments b = NOB wk .. + NOB - 1 of its block.
    // Partial sums are added in k-share order.
    // Beyond rank 16 the shares are pinned where they are formed: sunk to their next
    // use, they keep all of acc and the partner's sums in registers beside the U and
    // B loads, and 128 x 256 at rank 64 spills each U value as it arrives, one load
    // after the other (1172 x 5120 x 512, r = 54: 24.8 us against 17.1).  At rank
    // 16, where nothing is loaded here, the pins would cost 0.4 us.
    floatx4 own[NA][NOB];
    auto pin = [&](floatx4& v) LORA_INLINE { if constexpr (!EARLY_B) asm volatile("" : "+v"(v)); };
    floatx4* xb = reinterpret_cast<floatx4*>(smem);
    if constexpr (NK == 2) {
      floatx4* dst = xb + (size_t)(wave ^ 4) * NA * 2 * 64;   // the partner's region
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const floatx4 lo = acc[a][b], hi = acc[a][2 + b];
          floatx4 o;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            o[q] = wk == 0 ? hi[q] : lo[q];
            own[a][b][q] = wk == 0 ? lo[q] : hi[q];
          }
          pin(own[a][b]);
          dst[(a * 2 + b) * 64 + lane] = o;
        }
    } else {   // [wn][token fragment][k share][feature fragment]
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) xb[(size_t)(((wn * 4 + b) * 4 + wk) * NA + a) * 64 + lane] = acc[a][b];
    }
    if constexpr (UPRE) {   // U, and B beyond rank 16: all loads issued before the first use, acc half free
      const __amdgpu_buffer_rsrc_t rsU = make_rsrc(U + (size_t)m0 * r, (uint64_t)min(BM, m - m0) * r * 4);
      load_u_pairs<BM, RP, NT>(rsU, r, tid, uv);
      if constexpr (!EARLY_B) {
        const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B + (size_t)n0 * r, (uint64_t)jn * r * 2);
        load_b_rows<RP, NT>(rsB, r, jn, tid, bv);
      }
    }
    if (!UPRE) {
#pragma unroll
      for (int gg = 0; gg < 2; ++gg)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          Us[(wk * BM + wm * 64 + 16 * (2 * wn + gg) + c16) * RP + 4 * g + q] = uacc[gg][q];
    }
    __syncthreads();
    if constexpr (NK == 2) {
      const floatx4* src = xb + (size_t)wave * NA * 2 * 64;
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          own[a][b] += src[(a * 2 + b) * 64 + lane];
          pin(own[a][b]);
        }
    } else {
      const floatx4* src = xb + (size_t)(wn * 4 + wk) * 4 * NA * 64;
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        own[a][0] = src[a * 64 + lane];
#pragma unroll
        for (int q = 1; q < 4; ++q) own[a][0] += src[(q * NA + a) * 64 + lane];
      }
    }
    if constexpr (!EARLY_B) {
      __syncthreads();                             // the exchange has been read
      store_b_rows<BN, RP, NT>(bv, r, jn, tid, Bs2);
      split_u_pairs<BM, RP, NT>(uv, s, tid, reinterpret_cast<u16*>(Us));
    } else if (UPRE) {
#pragma unroll
      for (int i = 0; i < UPT / 2; ++i)
        *reinterpret_cast<float2*>(Us + 2 * (tid + i * NT)) = float2{uv[2 * i], uv[2 * i + 1]};
    } else {
      for (int e = tid; e < BM * RP; e += NT) {   // the k shares' partials, written before the barrier above
        float v = Us[e];
#pragma unroll
        for (int q = 1; q < NK; ++q) v += Us[q * BM * RP + e];
        Us[e] = v;
      }
    }
    __syncthreads();
    if (n0 == 0 && !UPRE) {
      for (int e = tid; e < BM * RP; e += NT) {
        const int il = e / RP, t = e - il * RP;
        if (m0 + il < m && t < r) U[(size_t)(m0 + il) * r + t] = Us[e];
      }
    }
    // own += s U B^T: one product of 32 k holds a block of 16 t twice, against
    // the high bf16 part of s U (lanes g = 0, 1) and the low part (g = 2, 3)
    const int i1 = wm * 64 + 16 * ((NOB * wk) ^ (2 * wn));   // the wave's first token in the tile
    const int tblocks = RP == 16 ? 1 : (r + 15) / 16;
    for (int tb = 0; tb < tblocks; ++tb) {
      const int t0 = 16 * tb + 8 * (g & 1);
      short8 uf[NOB];
#pragma unroll
      for (int b = 0; b < NOB; ++b) {
        if constexpr (!EARLY_B) {
          uf[b] = *reinterpret_cast<const short8*>(reinterpret_cast<const u16*>(Us) + (i1 + 16 * b + c16) * RPU +
                                                   (g < 2 ? 0 : RP) + t0);
        } else {
          const float* up = Us + (i1 + 16 * b + c16) * RPU + t0;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float v = s * up[e];
            const u16 hi = f32_to_bf16(v);
            uf[b][e] = (short)(g < 2 ? hi : f32_to_bf16(v - bf16_to_f32(hi)));
          }
        }
      }
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const short8 bfr = *reinterpret_cast<const short8*>(Bs2 + (wn * WTJ + 16 * a + c16) * RPB + t0);
#pragma unroll
        for (int b = 0; b < NOB; ++b) own[a][b] = mfma16x16x32(bfr, uf[b], own[a][b]);
      }
    }
    // Y rounded to bf16, through a wave-private LDS region (at RP = 16 the
    // exchange region, read before the last barrier)
    if constexpr (!EARLY_B) __syncthreads();
    constexpr int OUT = out16_bytes<NA, NOB>();
    static_assert(8 * OUT <= (EARLY_B ? XCH : 96 * 1024), "output staging");
    store_out16<NA, NOB>(own, smem + wave * OUT, Y + (size_t)(m0 + i1) * n + n0 + wn * WTJ, (size_t)n, m - m0 - i1,
                         n - n0 - wn * WTJ, lane);
  }
}

template <int BM, int BN, int RP, bool UPRE>
constexpr int fwd_ks_smem() {
  constexpr int nk = BM == 128 ? 2 : 4;
  constexpr int stage = (BM + BN + (UPRE ? 0 : 16)) * 128 * (nk / 2), early = RP == 16 ? BN * RP * 2 : 0;
  constexpr int nbuf = (160 * 1024 - early) / stage < 4 ? (160 * 1024 - early) / stage : 4;
  constexpr int loop = nbuf * stage + early, xch = 8 * (nk == 2 ? 2 : 4) * (BN / 32) * 1024;
  constexpr int epi = RP == 16 ? xch + nk * BM * RP * 4 : BM * (RP + 4) * 4 + BN * (RP + 8) * 2;
  constexpr int e1 = epi > xch ? epi : xch;
  static_assert(loop <= 160 * 1024 && e1 <= (RP == 16 ? nbuf * stage : 160 * 1024), "LDS budget");
  return loop > e1 ? loop : e1;
}

}  // namespace lora
