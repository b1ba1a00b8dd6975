// Backward of the LoRA-adapted linear layer (chain rule through Eq. 1 of JORA,
// Section 3, for the trainable A and B; W0 is frozen so no dW is formed):
//   dU = s dY B,   dX = dY W + dU A,   dB = s dY^T U,   dA = dU^T X.
//
// Kernels, in stream order (three launches, four when the dX columns are
// split between two tiles; each launch costs a few microseconds on its own,
// so small steps share launches):
//   du        dU = s dY B, reducing over n.  Writes dU2 (token-major, high |
//             low) for the dX GEMM, dUt2 (dU^T rounded to bf16) for dA and
//             Ut2 (U^T rounded to bf16, tokens padded to mp) for dB.
//   tokred    one launch, two token reductions split over token ranges:
//             dB^T partials = Ut2 . dY and dA partials = dUt2 . X; the
//             waves of a workgroup split its tokens.
//   dx        dX = [dY | dU2] . [W ; A ; A]: one GEMM whose k loop runs over
//             n and then over the 2 RP wide slab (high and low part of dU
//             against the same A rows).  W is read through LDS with the
//             transposing ds_read_b64_tr_b16, since the product contracts
//             W over its rows.  After its tile, each workgroup of this
//             launch (the first one of a split) sums a slice of the dB and dA
//             partials in a fixed order (no atomics, so results are
//             bit-identical from run to run) and applies s to dB.
#include <mutex>
#include <type_traits>

#include "lora_device.hpp"
#include "lora_launch.hpp"
#include "lora_plan.hpp"

namespace lora {

// ---------------------------------------------------------------------------
// 16x16x32 A operand (16 columns x 32 k) from a small row-major LDS tile
// whose rows are k (no swizzle, `pitch` bytes per row): lane (g = l/16,
// c = l%16) receives column col0 + c, k rows 8g .. 8g+7.
__device__ __forceinline__ short8 tr16_read(const char* tile, int pitch, int col0, int lane) {
  const int g = lane >> 4, j = lane & 15;
  const int e = j >> 2, q = j & 3;
  const char* p0 = tile + (8 * g + e) * pitch + (col0 + 4 * q) * 2;
  return join4(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)p0),
               __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)(p0 + 4 * pitch)));
}

// U^T of the tokens i0 .. i0+TPW-1 rounded to bf16 into Ut2 [RP][mp] (tokens
// at or past m and ranks at or past r zero), by NTH threads; each thread
// issues all of its loads before its first store.
template <int RP, int TPW, int NTH>
__device__ __forceinline__ void store_ut2(const float* __restrict__ U, u16* __restrict__ Ut2, int i0, int m, int r,
                                          int mp, int tid) {
  constexpr int UPT = (RP * TPW + NTH - 1) / NTH;
  const __amdgpu_buffer_rsrc_t rsU = make_rsrc(U + (size_t)i0 * r, (uint64_t)max(0, min(TPW, m - i0)) * r * 4);
  float uv[UPT];
#pragma unroll
  for (int q = 0; q < UPT; ++q) {
    const int e = tid + q * NTH, t = e / TPW, il = e % TPW;
    uv[q] = buf_load4f(rsU, (e < RP * TPW && t < r) ? (uint32_t)(il * r + t) * 4 : kOOB);
  }
#pragma unroll
  for (int q = 0; q < UPT; ++q) {
    const int e = tid + q * NTH, t = e / TPW;
    if (e < RP * TPW) Ut2[(size_t)t * mp + i0 + e % TPW] = f32_to_bf16(uv[q]);
  }
}

// Element q of a per-projection argument array (q uniform); compile-time
// indices only, so the kernel argument is never indexed dynamically.
template <typename T>
__device__ __forceinline__ T pick(const T (&v)[kMaxGroup], int q) {
  T x = v[0];
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i)
    if (q == i) x = v[i];
  return x;
}

// Kernel argument (by value) of the dU kernels: the projections of a group
// (one for a single projection), each with `blocks` workgroups of its own.
struct DuGroup {
  const u16* dY[kMaxGroup];
  const u16* B[kMaxGroup];
  const float* U[kMaxGroup];
  u16* dU2[kMaxGroup];
  u16* dUt2[kMaxGroup];
  u16* Ut2[kMaxGroup];
  int n[kMaxGroup];
};

// ---------------------------------------------------------------------------
// dU = s dY B for TPW (8, 16 or 32) tokens per workgroup, reducing over all
// of n, plus the U^T high/low split of the same tokens.  The launch takes the
// largest TPW that still gives every compute unit a workgroup: each
// workgroup reads all of B (n x r), so more tokens per workgroup means less B
// traffic per token (at rank 64 B is 4 times the dY bytes of 16 tokens).
// TPW = 8 carries 8 zero token columns in the matrix-core B operand.  The 8
// waves take interleaved 32-wide chunks of n, UNR chunks per batch with all
// of a batch's loads issued together.  A chunk's B rows (32 x r, contiguous
// in B) are staged in a wave-private LDS slot as [32][RP] (columns t >= r
// stay zero) and read back transposed into matrix-core A operands, each used
// for the TG = TPW / 16 groups of 16 tokens; dY rows go straight into B
// operands.  The waves' sums are added in wave order through LDS, so the
// result is bit-identical from run to run.  (A split of n over workgroups
// would need a cross-workgroup reduction, whose device-scope fences write
// back the per-XCD L2s -- far dearer than the work.)  Writes dU2 (token-major,
// high | low parts), dUt2 (dU^T rounded to bf16, rows of mp tokens; for a
// group whose members share one dA reduction, the member's rows of the
// stacked dU^T) and Ut2 (U^T rounded to bf16).  Index math is 32-bit:
// validation bounds every index below 2^30.
template <int RP, int TPW>
__global__ __launch_bounds__(512) void lora_bwd_du_kernel(DuGroup grp, int blocks, int m, int r, int mp,
                                                          float s) {
  constexpr int FT = RP / 16;
  constexpr int TG = TPW >= 16 ? TPW / 16 : 1;      // 16-token groups
  constexpr int NWV = 8;
  // Chunks per batch: deep batches pay off only for the short n runs of the
  // 8-token workgroups; with 16 or more tokens, batches of one or two chunks
  // keep more of them in flight across the loop (7B up_proj dU 29.8 -> 24.0 us).
  constexpr int UNR = TPW == 8 ? (RP <= 16 ? 8 : (RP <= 32 ? 4 : 2)) : (RP <= 32 && TG == 1 ? 2 : 1);
  constexpr int SLOT = 32 * RP * 2;                 // bytes of one staged chunk of B
  constexpr int BL = RP / 16;                       // 16-byte B loads per lane per chunk (4r <= 4 RP)
  constexpr int STAGE_BYTES = NWV * UNR * SLOT, RED_BYTES = NWV * TG * FT * 64 * 16;
  __shared__ __attribute__((aligned(1024))) char sm[STAGE_BYTES > RED_BYTES ? STAGE_BYTES : RED_BYTES];
  static_assert(TPW == 32 || TPW == 16 || TPW == 8, "tokens per workgroup");
  static_assert(TG * FT <= NWV, "one wave per output fragment in the epilogue");
  const int sel = (int)blockIdx.x / blocks;        // the projection
  const u16 *dY = pick(grp.dY, sel), *B = pick(grp.B, sel);
  const float* U = pick(grp.U, sel);
  u16 *dU2 = pick(grp.dU2, sel), *dUt2 = pick(grp.dUt2, sel), *Ut2 = pick(grp.Ut2, sel);
  const int n = pick(grp.n, sel);
  const int i0 = ((int)blockIdx.x - sel * blocks) * TPW;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const uint32_t rowbytes = (uint32_t)n * 2;
  const int rows = uniform(max(0, min(TPW, m - i0)));
  const __amdgpu_buffer_rsrc_t rsY = make_rsrc(dY + (size_t)i0 * n, (uint64_t)rows * rowbytes);
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B, (uint64_t)n * r * 2);
  char* slots = sm + wave * UNR * SLOT;

  for (int e = lane; e < UNR * SLOT / 16; e += 64) reinterpret_cast<int4v*>(slots)[e] = int4v{0, 0, 0, 0};

  floatx4 acc[TG][FT];
#pragma unroll
  for (int tg = 0; tg < TG; ++tg)
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) acc[tg][ft] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int nbch = 4 * r;                           // 16-byte chunks in 32 rows of B
  const bool fast = (r & 7) == 0;                   // a chunk then lies inside one row of B
  const float rinv = 1.0f / (float)r;
  // Batch b of this wave covers chunks j = 32 wave + 32 NWV (UNR b + u); the
  // loads of batch b+1 are in flight while batch b multiplies.
  short8 yf[2][UNR][TG];
  int4v bq[2][UNR][BL];
  auto load = [&](int bt, int p) LORA_INLINE {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int j = 32 * wave + 32 * NWV * (UNR * bt + u);
      const int jy = j + 8 * g;
#pragma unroll
      for (int tg = 0; tg < TG; ++tg)
        yf[p][u][tg] = __builtin_bit_cast(
            short8, buf_load16(rsY, jy < n ? (uint32_t)(16 * tg + c16) * rowbytes + (uint32_t)jy * 2 : kOOB));
#pragma unroll
      for (int v = 0; v < BL; ++v) {
        const int c = lane + 64 * v;
        bq[p][u][v] = buf_load16(rsB, (j < n && c < nbch) ? (uint32_t)j * r * 2 + (uint32_t)c * 16 : kOOB);
      }
    }
  };
  auto process = [&](int p) LORA_INLINE {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      char* slot = slots + u * SLOT;
#pragma unroll
      for (int v = 0; v < BL; ++v) {
        const int c = lane + 64 * v;
        if (c < nbch) {
          if (fast) {
            const int e0 = 8 * c, jj = e0 / r;
            *reinterpret_cast<int4v*>(slot + (jj * RP + e0 - jj * r) * 2) = bq[p][u][v];
          } else {
#pragma unroll
            for (int x = 0; x < 8; ++x) {   // quotient from a float product at least 0.5/r from an integer
              const int e = 8 * c + x;
              const int jj = (int)(((float)e + 0.5f) * rinv);
              *reinterpret_cast<u16*>(slot + (jj * RP + e - jj * r) * 2) =
                  (u16)((uint32_t)bq[p][u][v][x >> 1] >> (16 * (x & 1)));
            }
          }
        }
      }
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
        const short8 bt = tr16_read(slot, RP * 2, 16 * ft, lane);
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) acc[tg][ft] = mfma16x16x32(bt, yf[p][u][tg], acc[tg][ft]);
      }
    }
  };
  const int nbt = uniform(32 * wave < n ? (n - 32 * wave + 32 * NWV * UNR - 1) / (32 * NWV * UNR) : 0);
  if (nbt > 0) load(0, 0);
  for (int bt = 0; bt < nbt; bt += 2) {
    if (bt + 1 < nbt) load(bt + 1, 1);
    process(0);
    if (bt + 1 >= nbt) break;
    if (bt + 2 < nbt) load(bt + 2, 0);
    process(1);
  }

  store_ut2<RP, TPW, 64 * NWV>(U, Ut2, i0, m, r, mp, tid);   // U^T of this workgroup's tokens in bf16

  __syncthreads();
  floatx4* red = reinterpret_cast<floatx4*>(sm);   // [NWV][TG][FT][64]
#pragma unroll
  for (int tg = 0; tg < TG; ++tg)
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) red[((wave * TG + tg) * FT + ft) * 64 + lane] = acc[tg][ft];
  __syncthreads();
  if (wave >= TG * FT) return;
  const int tg = wave / FT, ft = wave - tg * FT;   // one wave per 16 x 16 fragment of dU^T
  floatx4 v = red[(tg * FT + ft) * 64 + lane];
#pragma unroll
  for (int w = 1; w < NWV; ++w) v += red[((w * TG + tg) * FT + ft) * 64 + lane];
  if (16 * tg + c16 >= TPW) return;   // the zero token columns of TPW = 8
  const int i = i0 + 16 * tg + c16;   // < mp: the grid covers exactly mp tokens
  u16 hi[4], lo[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float d = s * v[q];
    hi[q] = f32_to_bf16(d);
    lo[q] = f32_to_bf16(d - bf16_to_f32(hi[q]));
  }
  const int t = 16 * ft + 4 * g;
  u16* row = dU2 + (size_t)i * (2 * RP);
  *reinterpret_cast<uint2*>(row + t) =
      uint2{(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16)};
  *reinterpret_cast<uint2*>(row + RP + t) =
      uint2{(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16)};
#pragma unroll
  for (int q = 0; q < 4; ++q) dUt2[(size_t)(t + q) * mp + i] = hi[q];
}

// ---------------------------------------------------------------------------
// Wait until at most N LDS operations of this wave are outstanding, in an asm
// statement that takes a substep's fragment registers as operands (so no use
// of them can move above it): TG dY fragments, FT pairs of B^T halves.
template <int N, int FT, int TG>
__device__ __forceinline__ void du_frag_wait(short8 (&y)[TG], short4v (&bl)[FT], short4v (&bh)[FT]) {
  static_assert(N >= 0 && N <= 15, "lgkmcnt range");
#define LORA_DU_WAIT(...) asm volatile("s_waitcnt lgkmcnt(%[cnt])" : __VA_ARGS__ : [cnt] "i"(N))
  if constexpr (FT == 1 && TG == 1) LORA_DU_WAIT("+v"(y[0]), "+v"(bl[0]), "+v"(bh[0]));
  else if constexpr (FT == 1 && TG == 2) LORA_DU_WAIT("+v"(y[0]), "+v"(y[1]), "+v"(bl[0]), "+v"(bh[0]));
  else if constexpr (FT == 2 && TG == 1) LORA_DU_WAIT("+v"(y[0]), "+v"(bl[0]), "+v"(bh[0]), "+v"(bl[1]), "+v"(bh[1]));
  else if constexpr (FT == 2 && TG == 2)
    LORA_DU_WAIT("+v"(y[0]), "+v"(y[1]), "+v"(bl[0]), "+v"(bh[0]), "+v"(bl[1]), "+v"(bh[1]));
  else if constexpr (FT == 3 && TG == 1)
    LORA_DU_WAIT("+v"(y[0]), "+v"(bl[0]), "+v"(bh[0]), "+v"(bl[1]), "+v"(bh[1]), "+v"(bl[2]), "+v"(bh[2]));
  else if constexpr (FT == 3 && TG == 2)
    LORA_DU_WAIT("+v"(y[0]), "+v"(y[1]), "+v"(bl[0]), "+v"(bh[0]), "+v"(bl[1]), "+v"(bh[1]), "+v"(bl[2]),
                 "+v"(bh[2]));
  else if constexpr (FT == 4 && TG == 1)
    LORA_DU_WAIT("+v"(y[0]), "+v"(bl[0]), "+v"(bh[0]), "+v"(bl[1]), "+v"(bh[1]), "+v"(bl[2]), "+v"(bh[2]),
                 "+v"(bl[3]), "+v"(bh[3]));
  else {
    static_assert(FT == 4 && TG == 2, "fragment shapes");
    LORA_DU_WAIT("+v"(y[0]), "+v"(y[1]), "+v"(bl[0]), "+v"(bh[0]), "+v"(bl[1]), "+v"(bh[1]), "+v"(bl[2]),
                 "+v"(bh[2]), "+v"(bl[3]), "+v"(bh[3]));
  }
#undef LORA_DU_WAIT
}

// ---------------------------------------------------------------------------
// dU = s dY B for ranks that are multiples of 8 (each 16-byte piece of B then
// lies inside one row), fed by copies straight into LDS.  TPW (8, 16 or 32)
// tokens per workgroup, four waves; the n loop runs in stages of 64: wave w
// takes stages w, w + 4, ... and copies each of them (its TPW dY rows, 8 rows
// of 128 bytes per copy instruction with the swizzle of kc_offset applied to
// the global addresses, and the stage's 64 rows of B as a [64][RP] block,
// zero past r) straight into a private ring of NSW LDS stages, NSW - 1
// stages ahead, waiting only for its own copies (no barrier in the loop).
// (The register-loading kernel above reads 16 rows x 64 bytes of dY per
// instruction, which keeps the L1 busy translating addresses.)  Each wave
// accumulates all of dU^T for its stages on 16x16x32 products: B^T fragments
// by transposing reads of the B block, dY fragments as the second operand
// (TPW = 8 leaves token columns 8..15 zero); the fragment reads are issued as
// inline assembly with counted waits, since the compiler would otherwise wait
// for every copy in flight before each transposing read.  The four partial
// sums are added in wave order through LDS, then written as the register
// kernel does (dU2, dUt2, Ut2).
template <int RP, int TPW>
__global__ __launch_bounds__(256) void lora_bwd_du_dma_kernel(DuGroup grp, int blocks, int m, int r, int mp,
                                                              float s) {
  constexpr int NWV = 4;
  constexpr int FT = RP / 16;
  constexpr int TG = TPW >= 16 ? TPW / 16 : 1;
  constexpr int YR = TG * 16;                    // dY rows per stage in LDS (TPW = 8: rows 8..15 stay zero)
  constexpr int BOFF = YR * 128;                 // the B block [64][RP] after the dY rows
  constexpr int STAGE = BOFF + 64 * RP * 2;
  constexpr int CY = TPW / 8, CB = RP / 8;       // 1 KB copies per stage: dY rows, B block
  constexpr int CPW = CY + CB;
  constexpr int NSW = (156 * 1024) / (NWV * STAGE) < 6 ? (156 * 1024) / (NWV * STAGE) : 6;
  constexpr int RED = NWV * TG * FT * 64 * 16;   // cross-wave sum [NWV][TG][FT][64] float4
  constexpr int SMEM = NWV * NSW * STAGE > RED ? NWV * NSW * STAGE : RED;
  constexpr int NRD = TG + 2 * FT;               // LDS reads per wave and 32-wide substep
  static_assert(TPW == 8 || TPW == 16 || TPW == 32, "tokens per workgroup");
  static_assert(NSW >= 3 && CPW * (NSW - 2) < 64, "copies in flight fit the wait counter");
  static_assert(NRD <= 15, "reads of one substep fit the LDS wait counter");
  __shared__ __attribute__((aligned(1024))) char sm[SMEM];
  const int sel = (int)blockIdx.x / blocks;        // the projection
  const u16 *dY = pick(grp.dY, sel), *B = pick(grp.B, sel);
  const float* U = pick(grp.U, sel);
  u16 *dU2 = pick(grp.dU2, sel), *dUt2 = pick(grp.dUt2, sel), *Ut2 = pick(grp.Ut2, sel);
  const int n = pick(grp.n, sel);
  const int i0 = ((int)blockIdx.x - sel * blocks) * TPW;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const uint32_t rowbytes = (uint32_t)n * 2;
  const int rows = uniform(max(0, min(TPW, m - i0)));
  const __amdgpu_buffer_rsrc_t rsY = make_rsrc(dY + (size_t)i0 * n, (uint64_t)rows * rowbytes);
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B, (uint64_t)n * r * 2);
  char* ring = sm + wave * NSW * STAGE;
  if (YR > TPW) {   // the zero token rows of TPW = 8, in every stage of the ring
    for (int e = lane; e < NSW * (YR - TPW) * 8; e += 64) {
      const int st = e / ((YR - TPW) * 8), q = e % ((YR - TPW) * 8);
      reinterpret_cast<int4v*>(ring + st * STAGE + TPW * 128)[q] = int4v{0, 0, 0, 0};
    }
  }

  // Copy c of the dY rows: rows 8c + lane/8 at physical chunk lane%8, which
  // holds logical chunk (lane%8) ^ kc_swz(row).  Copy c of the B block: its
  // bytes 1024c + 16 lane, i.e. row (1024c + 16 lane) / (2 RP) of the stage
  // and 8-element chunk ((1024c + 16 lane) % (2 RP)) / 16.
  const int nst = (n + 63) / 64;
  auto issue = [&](int j, int buf) LORA_INLINE {
    const int st = wave + NWV * j;
    const int j0 = st * 64;
    const bool live = st < nst;
    char* sb = ring + buf * STAGE;
#pragma unroll
    for (int c = 0; c < CY; ++c) {
      const int row = 8 * c + (lane >> 3);
      const int jj = j0 + 8 * ((lane & 7) ^ kc_swz(row));
      dma16(rsY, live && jj < n ? (uint32_t)row * rowbytes + (uint32_t)jj * 2 : kOOB, 0, sb + c * 1024);
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int byte = 1024 * c + 16 * lane;
      const int row = byte / (2 * RP), t0 = (byte % (2 * RP)) / 2;
      const int jb = j0 + row;
      dma16(rsB, live && jb < n && t0 < r ? ((uint32_t)jb * (uint32_t)r + (uint32_t)t0) * 2 : kOOB, 0,
            sb + BOFF + c * 1024);
    }
  };

  // Lane addresses in stage 0 of the wave's ring.  dY fragment (second
  // operand, 32 n x 16 tokens) of substep kk: row c16 (+ 2048 bytes per token
  // group), chunk 4 kk + g.  B^T fragment (first operand, 16 t x 32 n) as in
  // tr16_read: rows 8 g + e (+ 4 rows for the second read, + 32 rows for kk),
  // columns 16 ft + 4 q.
  uint32_t ya[2], ba;
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) ya[kk] = lds_addr(ring + kc_offset(c16, 4 * kk + g));
  {
    const int j = lane & 15, e = j >> 2, q = j & 3;
    ba = lds_addr(ring + BOFF + (8 * g + e) * (2 * RP) + 4 * q * 2);
  }
  floatx4 acc[TG][FT];
#pragma unroll
  for (int tg = 0; tg < TG; ++tg)
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) acc[tg][ft] = floatx4{0.f, 0.f, 0.f, 0.f};
  short8 fy[2][TG];
  short4v fbl[2][FT], fbh[2][FT];
  auto reads = [&](uint32_t boff, auto kkc) LORA_INLINE {
    constexpr int kk = decltype(kkc)::value;
    ds_read_b128_asm<0>(fy[kk][0], ya[kk] + boff);
    if constexpr (TG > 1) ds_read_b128_asm<2048>(fy[kk][1], ya[kk] + boff);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      // (ft, kk) immediates: 32 ft bytes of columns, 32 rows of 2 RP bytes per kk
      const uint32_t a = ba + boff + (uint32_t)(32 * ft);
      ds_read_tr_b64_asm<kk * 32 * 2 * RP>(fbl[kk][ft], a);
      ds_read_tr_b64_asm<kk * 32 * 2 * RP + 4 * 2 * RP>(fbh[kk][ft], a);
    }
  };
  auto mult = [&](int kk) LORA_INLINE {
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const short8 bt = join4(fbl[kk][ft], fbh[kk][ft]);
#pragma unroll
      for (int tg = 0; tg < TG; ++tg) acc[tg][ft] = mfma16x16x32(bt, fy[kk][tg], acc[tg][ft]);
    }
  };
  using K0 = std::integral_constant<int, 0>;
  using K1 = std::integral_constant<int, 1>;
  auto compute = [&](int buf) LORA_INLINE {
    const uint32_t boff = (uint32_t)buf * STAGE;
    if constexpr (2 * NRD <= 15) {   // both substeps' reads in flight, then the products
      reads(boff, K0{});
      reads(boff, K1{});
      du_frag_wait<NRD, FT, TG>(fy[0], fbl[0], fbh[0]);   // only substep 1's reads outstanding
      mult(0);
      du_frag_wait<0, FT, TG>(fy[1], fbl[1], fbh[1]);
      mult(1);
    } else {
      reads(boff, K0{});
      du_frag_wait<0, FT, TG>(fy[0], fbl[0], fbh[0]);
      mult(0);
      reads(boff, K1{});
      du_frag_wait<0, FT, TG>(fy[1], fbl[1], fbh[1]);
      mult(1);
    }
  };

  const int nsw = wave < nst ? (nst - wave + NWV - 1) / NWV : 0;   // this wave's stages
#pragma unroll
  for (int j = 0; j < NSW - 1; ++j) issue(j, j);
  for (int j = 0; j < nsw; ++j) {
    wait_vmcnt<CPW * (NSW - 2)>();   // the wave's stage j has landed
    issue(j + NSW - 1, (j + NSW - 1) % NSW);   // into the buffer of stage j - 1, read already
    compute(j % NSW);
  }
  wait_vmcnt<0>();   // the trailing copies (zeros) land before the LDS is reused

  store_ut2<RP, TPW, 64 * NWV>(U, Ut2, i0, m, r, mp, tid);   // U^T of this workgroup's tokens in bf16

  __syncthreads();
  floatx4* red = reinterpret_cast<floatx4*>(sm);   // [NWV][TG][FT][64]
#pragma unroll
  for (int tg = 0; tg < TG; ++tg)
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) red[((wave * TG + tg) * FT + ft) * 64 + lane] = acc[tg][ft];
  __syncthreads();
  for (int e = wave; e < TG * FT; e += NWV) {   // fragment e of dU^T, summed in wave order
    const int tg = e / FT, ft = e - tg * FT;
    floatx4 v = red[(tg * FT + ft) * 64 + lane];
#pragma unroll
    for (int w = 1; w < NWV; ++w) v += red[((w * TG + tg) * FT + ft) * 64 + lane];
    if (16 * tg + c16 >= TPW) continue;   // the zero token columns of TPW = 8
    const int i = i0 + 16 * tg + c16;     // < mp: the grid covers exactly mp tokens
    u16 hi[4], lo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float d = s * v[q];
      hi[q] = f32_to_bf16(d);
      lo[q] = f32_to_bf16(d - bf16_to_f32(hi[q]));
    }
    const int t = 16 * ft + 4 * g;
    u16* row = dU2 + (size_t)i * (2 * RP);
    *reinterpret_cast<uint2*>(row + t) =
        uint2{(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16)};
    *reinterpret_cast<uint2*>(row + RP + t) =
        uint2{(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16)};
#pragma unroll
    for (int q = 0; q < 4; ++q) dUt2[(size_t)(t + q) * mp + i] = hi[q];
  }
}

// ---------------------------------------------------------------------------
// Token reduction part[sp][t][c] = sum over the tokens i of split sp of
// P[t][i] * Q[i][c], t < RP, for a tile of kRedCols = 128 columns.  P is the
// rank-r operand rounded to bf16 (U^T or s dU^T, [RP][mp]); its rounding
// error (relative 2^-9 per element) averages out in the sums to about 1e-3 of
// dA and dB.  One launch serves two such problems (dB^T from Ut2 and dY, dA
// from dUt2 and X): workgroups [0, nb0) take the first.
//
// The four waves of a workgroup take interleaved 32-token slices of the
// split.  Each reads its P fragments straight from the token-contiguous P
// into matrix-core A operands and stages its 32 x 128 slice of Q
// ([m][cols]) in a private LDS region that it reads back transposed, so the
// token loop has no barriers; the next slice is loaded while the current one
// multiplies.  At the end the four waves' sums are added in wave order
// through LDS (bit-identical from run to run).
struct RedProblem {
  const u16* P;
  const u16* Q;
  float* part;
  int ncols, span, col_tiles;
  const uint8_t* keep;   // dropout keep bits of Q ([m][ncols/8]) or null: masked Q elements count as 0
};

// Launched with KEEP, for the masked-Q path of LoRA dropout: the mask is
// applied to the Q chunks in registers before they are staged.  Without a
// mask the launch takes lora_tokred_dma_kernel below.
template <int RP, bool KEEP>
__global__ __launch_bounds__(256) void lora_tokred_kernel(RedProblem p0, RedProblem p1, int nb0, int m, int mp) {
  constexpr int CB = kRedCols;                // columns per workgroup
  constexpr int FC = CB / 16;                 // column fragments
  constexpr int FP = RP / 16;                 // row fragments
  constexpr int CPR = CB / 8;                 // 16-byte chunks per Q row
  constexpr int QL = 32 * CPR / 64;           // Q loads per lane per slice
  constexpr int REG = 32 * CB * 2;            // bytes of one staged Q slice
  // column fragments per reduction pass: the largest power of two dividing FC
  // whose partial sums (4 waves x FP x FCP fragments) fit the staging LDS
  constexpr int FCP = 16 / FP >= 8 ? 8 : (16 / FP >= 4 ? 4 : (16 / FP >= 2 ? 2 : 1));
  static_assert(FC % FCP == 0, "reduction passes cover the column fragments");
  static_assert(CB == 128 && QL * 64 == 32 * CPR, "slice shape");
  static_assert(4 * FP * FCP * 64 * 16 <= 4 * 2 * REG, "reduction fits the staging LDS");
  __shared__ __attribute__((aligned(1024))) char smem[4 * 2 * REG];

  const bool first = (int)blockIdx.x < nb0;
  const RedProblem& pr = first ? p0 : p1;
  const int bid = first ? (int)blockIdx.x : (int)blockIdx.x - nb0;
  const u16* __restrict__ P = pr.P;
  const u16* __restrict__ Q = pr.Q;
  const int ncols = pr.ncols;
  const int c0 = (bid % pr.col_tiles) * CB;
  const int sp = bid / pr.col_tiles;
  const int tb = sp * pr.span;
  const int te = min(mp, tb + pr.span);
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const uint32_t qrow = (uint32_t)ncols * 2;
  const __amdgpu_buffer_rsrc_t rsP = make_rsrc(P, (uint64_t)RP * mp * 2);
  char* wreg = smem + wave * 2 * REG;

  floatx4 acc[FP][FC];
#pragma unroll
  for (int f = 0; f < FP; ++f)
#pragma unroll
    for (int fc = 0; fc < FC; ++fc) acc[f][fc] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Slice loads: Q chunk u of this lane is row (lane + 64u) / CPR, chunk
  // (lane + 64u) % CPR; P fragment f is row 16f + c16, tokens ts + 8g .. +7.
  int4v qv[2][QL];
  uint32_t kq[KEEP ? 2 : 1][KEEP ? QL : 1];   // keep byte of each Q chunk (dropout)
  short8 pv[2][FP];
  const uint8_t* keep = KEEP ? pr.keep : nullptr;
  const uint32_t kb8 = (uint32_t)ncols / 8;
  auto load = [&](int ts, int b) LORA_INLINE {
    const int rows = uniform(max(0, min(32, m - ts)));   // keeps the resource in scalar registers
    const __amdgpu_buffer_rsrc_t rsQ = make_rsrc(Q + (size_t)ts * ncols, (uint64_t)rows * qrow);
#pragma unroll
    for (int u = 0; u < QL; ++u) {
      const int q = lane + 64 * u;
      const int cc = c0 + 8 * (q % CPR);
      qv[b][u] = buf_load16(rsQ, cc < ncols ? (uint32_t)(q / CPR) * qrow + (uint32_t)cc * 2 : kOOB);
    }
    if (KEEP && keep) {   // workgroup-uniform
      const __amdgpu_buffer_rsrc_t rsK = make_rsrc(keep + (size_t)ts * kb8, (uint64_t)rows * kb8);
#pragma unroll
      for (int u = 0; u < QL; ++u) {
        const int q = lane + 64 * u;
        const int cc = c0 + 8 * (q % CPR);
        kq[KEEP ? b : 0][KEEP ? u : 0] = buf_load_u8(rsK, cc < ncols ? (uint32_t)(q / CPR) * kb8 + (uint32_t)cc / 8 : kOOB);
      }
    }
#pragma unroll
    for (int f = 0; f < FP; ++f)
      pv[b][f] = __builtin_bit_cast(
          short8, buf_load16(rsP, ((uint32_t)(16 * f + c16) * (uint32_t)mp + (uint32_t)(ts + 8 * g)) * 2));
  };
  auto step = [&](int b) LORA_INLINE {
    char* qs = wreg + b * REG;
#pragma unroll
    for (int u = 0; u < QL; ++u) {
      const int q = lane + 64 * u;
      int4v v = qv[b][u];
      if (KEEP && keep)
        v = __builtin_bit_cast(int4v, keep_mask8(__builtin_bit_cast(short8, v), kq[KEEP ? b : 0][KEEP ? u : 0]));
      *reinterpret_cast<int4v*>(qs + mc16_offset<CB>(q / CPR, q % CPR)) = v;
    }
#pragma unroll
    for (int fc = 0; fc < FC; ++fc) {
      const short8 qf = mc16_read_tr<CB>(qs, 0, 16 * fc, lane);
#pragma unroll
      for (int f = 0; f < FP; ++f) acc[f][fc] = mfma16x16x32(pv[b][f], qf, acc[f][fc]);
    }
  };

  // Slices of this wave: ts0 + 128 j < te, ts0 = tb + 32 wave (te - tb is a
  // multiple of 64, so slices never straddle te).
  const int ts0 = tb + 32 * wave;
  const int ns = ts0 < te ? (te - ts0 + 127) / 128 : 0;
  if (ns > 0) load(ts0, 0);
  int j = 0;
  for (; j + 2 <= ns; j += 2) {
    load(ts0 + 128 * (j + 1), 1);
    step(0);
    if (j + 2 < ns) load(ts0 + 128 * (j + 2), 0);
    step(1);
  }
  if (j < ns) step(0);

  // Cross-wave sum in wave order, FCP column fragments per pass; lane holds
  // column c16 of fragment fc, rows 4g .. 4g+3 of fragment f.
  floatx4* red = reinterpret_cast<floatx4*>(smem);   // [4 waves][FP][FCP][64]
  float* part = pr.part;
#pragma unroll
  for (int f0 = 0; f0 < FC; f0 += FCP) {
    __syncthreads();
#pragma unroll
    for (int f = 0; f < FP; ++f)
#pragma unroll
      for (int q = 0; q < FCP; ++q) red[((wave * FP + f) * FCP + q) * 64 + lane] = acc[f][f0 + q];
    __syncthreads();
    for (int e = wave; e < FP * FCP; e += 4) {
      const int f = e / FCP, q = e - f * FCP;
      floatx4 v = red[((0 * FP + f) * FCP + q) * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += red[((w * FP + f) * FCP + q) * 64 + lane];
      const int col = c0 + 16 * (f0 + q) + c16;
      if (col < ncols) {
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) part[((size_t)sp * RP + 16 * f + 4 * g + qq) * ncols + col] = v[qq];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same token reduction without a keep mask, fed by copies straight into
// LDS.  Stages of 64 tokens: the stage's P block (RP rows x 64 tokens, 128
// bytes a row, kc_offset swizzle) and Q block (64 tokens x 128 columns, 256
// bytes a row, mc16_offset swizzle) are copied from global memory into a ring
// of NS LDS stages, NS - 1 stages ahead, in whole row pieces (8 rows of P or 4
// rows of Q per copy instruction; the swizzles applied to the global
// addresses), one barrier per stage.  (Register loads of 16 rows x 64 bytes
// per instruction kept the L1 busy translating addresses.)  The four waves
// split the columns, two 16-column fragments each, over all tokens of the
// split, so no cross-wave sum is needed.  The fragment reads are issued as
// inline assembly with explicit lgkmcnt waits: the compiler would otherwise
// wait for every copy still in flight before each transposing read of Q.
// At most 80 KB of LDS, so two workgroups share a compute unit.
template <int RP>
__global__ __launch_bounds__(256) void lora_tokred_dma_kernel(RedProblem p0, RedProblem p1, int nb0, int m,
                                                              int mp) {
  constexpr int CB = kRedCols, NWV = 4, TS = 64;
  constexpr int FP = RP / 16;
  constexpr int PB = RP * 128;                // P block bytes
  constexpr int QB = TS * CB * 2;             // Q block bytes
  constexpr int STAGE = PB + QB;
  constexpr int NS = (80 * 1024) / STAGE;     // ring stages
  constexpr int NP = RP / 8, NQ = TS / 4;     // 1 KB copies per stage: P rows / 8, Q rows / 4
  constexpr int QPW = NQ / NWV;               // Q copies per wave
  constexpr int NRD = FP + 4;                 // LDS reads per wave and substep
  static_assert(CB == 128 && NQ % NWV == 0 && NS >= 3, "stage shape");
  static_assert((NS - 2) * (NP / NWV + 1 + QPW) < 64, "copies in flight fit the wait counter");
  __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];

  const bool first = (int)blockIdx.x < nb0;
  const RedProblem& pr = first ? p0 : p1;
  const int bid = first ? (int)blockIdx.x : (int)blockIdx.x - nb0;
  const u16* __restrict__ P = pr.P;
  const u16* __restrict__ Q = pr.Q;
  const int ncols = pr.ncols;
  const int c0 = (bid % pr.col_tiles) * CB;
  const int sp = bid / pr.col_tiles;
  const int tb = sp * pr.span;
  const int te = min(mp, tb + pr.span);       // te - tb is a multiple of 64
  const int nst = (te - tb) / TS;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const uint32_t qrow = (uint32_t)ncols * 2;
  const __amdgpu_buffer_rsrc_t rsP = make_rsrc(P, (uint64_t)RP * mp * 2);

  // Copies of stage st into buffer buf.  P copy j (j = wave mod 4): rows
  // 8j + lane/8 at physical chunk lane%8; Q copy j = wave + 4i: rows
  // 4j + lane/16 at physical chunk lane%16.  Each position holds the logical
  // chunk given by the swizzle.  Tokens at or past m, columns past ncols and
  // stages past the split read zero.
  int pcol[NP / NWV + 1];
  uint32_t qoff[QPW];
  int qcol[QPW];
#pragma unroll
  for (int i = 0; i * NWV < NP; ++i) {
    const int row = 8 * (wave + NWV * i) + (lane >> 3);
    pcol[i] = 8 * ((lane & 7) ^ kc_swz(row));
  }
#pragma unroll
  for (int i = 0; i < QPW; ++i) {
    const int row = 4 * (wave + NWV * i) + (lane >> 4);
    const int c = (lane & 15) ^ mc16_swz(row);
    qcol[i] = c0 + 8 * c;
    qoff[i] = (uint32_t)row * qrow + (uint32_t)qcol[i] * 2;
  }
  auto issue = [&](int st, int buf) LORA_INLINE {
    const int ts = tb + TS * st;
    const bool live = st < nst;
    char* sb = smem + buf * STAGE;
#pragma unroll
    for (int i = 0; i * NWV < NP; ++i) {
      const int j = wave + NWV * i;
      if (j < NP) {   // wave-uniform
        const int row = 8 * j + (lane >> 3);
        dma16(rsP, live ? ((uint32_t)row * (uint32_t)mp + (uint32_t)(ts + pcol[i])) * 2 : kOOB, 0, sb + j * 1024);
      }
    }
    const int rows = uniform(live ? max(0, min(TS, m - ts)) : 0);
    const __amdgpu_buffer_rsrc_t rsQ = make_rsrc(Q + (size_t)ts * ncols, (uint64_t)rows * qrow);
#pragma unroll
    for (int i = 0; i < QPW; ++i)
      dma16(rsQ, qcol[i] < ncols ? qoff[i] : kOOB, 0, sb + PB + (wave + NWV * i) * 1024);
  };
  auto stage_barrier = [&]() LORA_INLINE {   // this wave's copies of the stage waited for: NS - 2 stages stay in flight
    if (wave < NP % NWV) copy_barrier<(NS - 2) * (NP / NWV + 1 + QPW)>();
    else copy_barrier<(NS - 2) * (NP / NWV + QPW)>();
  };

  // Lane addresses in buffer 0.  P fragment f (A operand, 16 rank rows x 32
  // tokens) of substep kk: row 16 f + c16, chunk 4 kk + g (f adds 2048 bytes;
  // the swizzle of kk depends on the lane).  Q fragment j of this wave
  // (column tile 2 wave + j; B operand, 32 tokens x 16 columns) as in
  // mc16_read_tr: two transposing reads 4 rows apart (+1024 bytes), substep kk
  // 32 rows further (+8192 bytes).
  uint32_t pa[2], qa[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) pa[kk] = lds_addr(smem + kc_offset(c16, 4 * kk + g));
  {
    const int j = lane & 15, e = j >> 2, q = j & 3;
#pragma unroll
    for (int jf = 0; jf < 2; ++jf) {
      const int col = 16 * (2 * wave + jf) + 4 * q;
      qa[jf] = lds_addr(smem + PB + mc16_offset<CB>(8 * g + e, col >> 3) + (col & 7) * 2);
    }
  }
  floatx4 acc[FP][2];
#pragma unroll
  for (int f = 0; f < FP; ++f) acc[f][0] = acc[f][1] = floatx4{0.f, 0.f, 0.f, 0.f};
  short8 fp[2][FP];
  short4v fql[2][2], fqh[2][2];
  auto reads = [&](uint32_t boff, int kk) LORA_INLINE {
    const uint32_t a = pa[kk] + boff;
    ds_read_b128_asm<0>(fp[kk][0], a);
    if constexpr (FP > 1) ds_read_b128_asm<2048>(fp[kk][1], a);
    if constexpr (FP > 2) ds_read_b128_asm<4096>(fp[kk][2], a);
    if constexpr (FP > 3) ds_read_b128_asm<6144>(fp[kk][3], a);
#pragma unroll
    for (int jf = 0; jf < 2; ++jf) {
      const uint32_t b = qa[jf] + boff;
      if (kk == 0) {
        ds_read_tr_b64_asm<0>(fql[kk][jf], b);
        ds_read_tr_b64_asm<1024>(fqh[kk][jf], b);
      } else {
        ds_read_tr_b64_asm<8192>(fql[kk][jf], b);
        ds_read_tr_b64_asm<9216>(fqh[kk][jf], b);
      }
    }
  };
  static_assert(FP <= 4, "rank rows per stage");
  auto mult = [&](int kk) LORA_INLINE {
#pragma unroll
    for (int jf = 0; jf < 2; ++jf) {
      const short8 qf = join4(fql[kk][jf], fqh[kk][jf]);
#pragma unroll
      for (int f = 0; f < FP; ++f) acc[f][jf] = mfma16x16x32(fp[kk][f], qf, acc[f][jf]);
    }
  };
  auto compute = [&](int buf) LORA_INLINE {
    const uint32_t boff = (uint32_t)buf * STAGE;
    reads(boff, 0);
    reads(boff, 1);
    // substep 0 once only the NRD reads of substep 1 are outstanding
    if constexpr (FP == 1)
      asm volatile("s_waitcnt lgkmcnt(5)" : "+v"(fp[0][0]), "+v"(fql[0][0]), "+v"(fqh[0][0]), "+v"(fql[0][1]),
                   "+v"(fqh[0][1]));
    else if constexpr (FP == 2)
      asm volatile("s_waitcnt lgkmcnt(6)" : "+v"(fp[0][0]), "+v"(fp[0][1]), "+v"(fql[0][0]), "+v"(fqh[0][0]),
                   "+v"(fql[0][1]), "+v"(fqh[0][1]));
    else if constexpr (FP == 3)
      asm volatile("s_waitcnt lgkmcnt(7)" : "+v"(fp[0][0]), "+v"(fp[0][1]), "+v"(fp[0][2]), "+v"(fql[0][0]),
                   "+v"(fqh[0][0]), "+v"(fql[0][1]), "+v"(fqh[0][1]));
    else
      asm volatile("s_waitcnt lgkmcnt(8)" : "+v"(fp[0][0]), "+v"(fp[0][1]), "+v"(fp[0][2]), "+v"(fp[0][3]),
                   "+v"(fql[0][0]), "+v"(fqh[0][0]), "+v"(fql[0][1]), "+v"(fqh[0][1]));
    static_assert(NRD == FP + 4, "wait counts above");
    mult(0);
    if constexpr (FP == 1)
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fp[1][0]), "+v"(fql[1][0]), "+v"(fqh[1][0]), "+v"(fql[1][1]),
                   "+v"(fqh[1][1]));
    else if constexpr (FP == 2)
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fp[1][0]), "+v"(fp[1][1]), "+v"(fql[1][0]), "+v"(fqh[1][0]),
                   "+v"(fql[1][1]), "+v"(fqh[1][1]));
    else if constexpr (FP == 3)
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fp[1][0]), "+v"(fp[1][1]), "+v"(fp[1][2]), "+v"(fql[1][0]),
                   "+v"(fqh[1][0]), "+v"(fql[1][1]), "+v"(fqh[1][1]));
    else
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fp[1][0]), "+v"(fp[1][1]), "+v"(fp[1][2]), "+v"(fp[1][3]),
                   "+v"(fql[1][0]), "+v"(fqh[1][0]), "+v"(fql[1][1]), "+v"(fqh[1][1]));
    mult(1);
  };

#pragma unroll
  for (int st = 0; st < NS - 1; ++st) issue(st, st);
  for (int st = 0; st < nst; ++st) {
    stage_barrier();   // stage st has landed; every wave is done with stage st - 1
    issue(st + NS - 1, (st + NS - 1) % NS);
    compute(st % NS);
  }
  copy_barrier<0>();   // the trailing copies land before the workgroup ends

  // lane of (f, jf): rank rows 16 f + 4 g .. +3 of column c0 + 16 (2 wave + jf) + c16
  float* part = pr.part;
#pragma unroll
  for (int jf = 0; jf < 2; ++jf) {
    const int col = c0 + 16 * (2 * wave + jf) + c16;
    if (col < ncols) {
#pragma unroll
      for (int f = 0; f < FP; ++f)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) part[((size_t)sp * RP + 16 * f + 4 * g + qq) * ncols + col] = acc[f][jf][qq];
    }
  }
}

// ---------------------------------------------------------------------------
// Fixed-order sum of the split partials of dB and dA (s applied to dB), no
// atomics.  Runs at the end of the dX workgroups, after the token reductions
// have completed in stream order.
struct FinalizeArgs {
  const float* pb;
  const float* pa;
  float* dB;
  float* dA;
  int n, k, r, rp, sb, sa;
  float s;
  float sa_scale;   // 1, or 1 / (1 - p) with dropout (dA = dU^T keep X / (1 - p))
  int rpa;          // rows of one split's dA partial block (rp, or a group's stacked rank)
};

// Sum of `count` partials spaced `step` floats apart, in index order; the
// loads of each group of eight are all issued before the first add.
__device__ __forceinline__ float sum_partials(const float* p, size_t step, int count) {
  float v = 0.f;
  for (int p0 = 0; p0 < count; p0 += 8) {
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = p0 + u < count ? p[(size_t)(p0 + u) * step] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p0 + u < count) v += x[u];
  }
  return v;
}

__device__ __forceinline__ void finalize_partials(const FinalizeArgs& f, int first, int stride) {
  const int nb = f.n * f.r, na = f.r * f.k;
  for (int e = first; e < nb + na; e += stride) {
    if (e < nb) {  // e = t * n + j: partial reads along j are contiguous
      const int t = e / f.n, j = e - t * f.n;
      const float v = sum_partials(f.pb + (size_t)t * f.n + j, (size_t)f.rp * f.n, f.sb);
      f.dB[(size_t)j * f.r + t] = f.s * v;
    } else {
      const int g = e - nb;
      const int t = g / f.k, l = g - t * f.k;
      f.dA[g] = f.sa_scale * sum_partials(f.pa + (size_t)t * f.k + l, (size_t)f.rpa * f.k, f.sa);
    }
  }
}

// Kernel argument (by value) of the grouped dX GEMM of projections that read
// one X: dX = sum_g (dY_g W_g + dU_g A_g).  The n stages of every projection
// run back to back in one k loop (ceil(n_g / 64) stages each, nkb in all);
// the rank-r terms dU_g A_g are added after the loop,
// and the workgroup tails finalize every projection's dA_g and dB_g.
struct DxGroup {
  const u16* dY[kMaxGroup];
  const u16* W[kMaxGroup];
  const u16* dU2[kMaxGroup];
  const u16* A[kMaxGroup];
  int n[kMaxGroup];
  int count, nkb;
  FinalizeArgs fin[kMaxGroup];
};

// ---------------------------------------------------------------------------
// dX tiles, formed as dX^T = W^T dY^T with v_mfma_f32_16x16x32_bf16 (W as the A
// operand, dY as the B operand).  Stages of 64 along n: dY [BM rows][64]
// (k-contiguous) and W [64 rows of n][BN] (mn-contiguous, read with the
// transposing LDS read, which is issued as inline assembly: the compiler would
// otherwise wait for every copy in flight before each), copied from global
// memory straight into LDS.  After the n stages, NSLAB stages cover the 2 RP
// wide slab: dU2 [BM][2RP] against A's rows, once for the high and once for the
// low part.
//
// With dropout (DROP) the LoRA term is keep * (dU A) / (1 - p): the mask acts
// after the rank-r product, so it cannot ride in the k loop.  The slab stages
// are skipped; after the n stages the tile's dU2 rows, A columns and keep bits
// are staged in LDS, dU A is formed per fragment into a temporary
// accumulator, and added under the mask with the 1 / (1 - p) scale.
//
// With GRP (DxGroup) the n stages of all projections of a group form the k
// loop, each stage loading from its own projection's dY_g and W_g; the slab
// stages are skipped and each dU_g A_g is added after the loop from LDS.
//
// FULL (every n a multiple of 64 and the launch's columns a multiple of BN):
// the copies carry no bound checks.
// LDS stages and bytes of the 128- and 64-token tiles.
constexpr int dx_ks_bufs(int bm, int bn) { return bm == 128 ? (bn == 256 ? 3 : 4) : (bn == 128 ? 3 : 4); }
constexpr int dx_ks_smem(int bm, int bn) { return dx_ks_bufs(bm, bn) * (bm * 128 + bn * 128) * (bm == 64 ? 2 : 1); }

struct DxArgs {
  const u16 *dY, *W, *dU2, *A;
  const uint8_t* keep;
  u16* dX;
  int m, n, k, r, mp;
  float inv_keep;
};

// Source of every STEP-th 64-wide n piece, starting `STEP - first` before its
// first one: projection, the piece's index there, its dY rows (a single
// projection's are the arguments').  Past the last piece sl * 64 >= n.
template <bool GRP, int STEP>
struct DxCursor {
  int g = 0, sl, n;
  const u16* W;
  uint32_t yr;
  __amdgpu_buffer_rsrc_t rsY;
  int m0, rows;
  __device__ __forceinline__ DxCursor(const DxArgs& p, const DxGroup& grp, int m0_, int bm, int first)
      : sl(first - STEP), n(GRP ? grp.n[0] : p.n), W(GRP ? grp.W[0] : p.W), yr((uint32_t)n * 2),
        rsY(make_rsrc((GRP ? grp.dY[0] : p.dY) + (size_t)m0_ * n, (uint64_t)min(bm, p.m - m0_) * yr)), m0(m0_),
        rows(min(bm, p.m - m0_)) {}
  __device__ __forceinline__ void advance(const DxGroup& grp) {
    sl += STEP;
    if (GRP) {
      while (sl * 64 >= n && g + 1 < grp.count) {   // next projection (uniform)
        sl -= (n + 63) / 64;
        ++g;
        n = pick(grp.n, g);
        W = pick(grp.W, g);
        yr = (uint32_t)n * 2;
        rsY = make_rsrc(pick(grp.dY, g) + (size_t)m0 * n, (uint64_t)rows * yr);
      }
    }
  }
};

// 16x16x32 A operand (16 columns x 32 k) of the rank-r rows in LDS: tile As
// [RP][BN] mn-contiguous (mc16 swizzle), k rows 32 kk + 8 g .. + 7 of [A; A].
template <int BN, int RP>
__device__ __forceinline__ short8 slab_frag(const char* As, int kk, int col0, int lane) {
  const int g = lane >> 4, c = lane & 15;
  const int r0 = (32 * kk + 8 * g) % RP + (c >> 2), col = col0 + 4 * (c & 3);   // RP is a multiple of 16
  const char* p0 = As + mc16_offset<BN>(r0, col >> 3) + (col & 7) * 2;
  const char* p1 = As + mc16_offset<BN>(r0 + 4, col >> 3) + (col & 7) * 2;
  return join4(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)p0),
               __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)p1));
}

// Stage a tile's dU2 rows (Us [BM][2 RP + 8] bf16) and A columns (As [RP][BN]
// mn-contiguous, zero beyond r and k) for the rank-r term after the k loop.
template <int BM, int BN, int RP, int NT>
__device__ __forceinline__ void stage_rank_operands(const u16* dU2, const u16* A, u16* Us, char* As, int m0, int l0,
                                                    int mp, int k, int r, int tid) {
  constexpr int KS2 = 2 * RP, UP = KS2 + 8;
  const uint32_t urow = (uint32_t)KS2 * 2, wrow = (uint32_t)k * 2;
  const __amdgpu_buffer_rsrc_t rsU = make_rsrc(dU2 + (size_t)m0 * KS2, (uint64_t)min(BM, mp - m0) * urow);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(A, (uint64_t)r * wrow);
  for (int q = tid; q < BM * (RP / 4); q += NT) {
    const int i = q / (RP / 4), c = q % (RP / 4);
    *reinterpret_cast<int4v*>(Us + i * UP + 8 * c) = buf_load16(rsU, (uint32_t)i * urow + (uint32_t)c * 16);
  }
  for (int q = tid; q < RP * (BN / 8); q += NT) {
    const int t = q / (BN / 8), c = q % (BN / 8);
    const int ll = l0 + 8 * c;
    *reinterpret_cast<int4v*>(As + mc16_offset<BN>(t, c)) =
        buf_load16(rsA, (t < r && ll < k) ? (uint32_t)t * wrow + (uint32_t)ll * 2 : kOOB);
  }
}

// Tiles of 128 tokens x 128, 192 or 256 columns.  Eight waves: wave (wk, wn)
// multiplies all 128 tokens with BN / 4 columns over the 32-wide n half wk of
// every stage (so each W column is read by one wave per half: the transposing
// reads run at half the rate of the plain ones), three or four stages in LDS.
// The two halves take turns reading and multiplying exactly as in the forward's
// 128-token tiles, with the same ordering of copies, waits and barriers; after
// the loop the halves' partial sums are exchanged through LDS, each wave
// finishing 64 tokens.
//
// Tiles of 64 tokens x 64 or 128 columns, for few tokens (the larger tiles then
// leave compute units idle): four n shares of 32 instead of two, stages of 128
// n (two 64-wide pieces), two waves along the columns.
// Measured (whole backward call, against 64 x 64 wave tiles in step on 32x32x16
// products, register-staged for partial stages and 128 x 128): 2048 x 4096 x
// 4096 (tokens x n x k), r = 8: 76 -> 70 us; 333 x 4096 x 4096 51 -> 40; 1531 x
// 4104 x 3208, r = 12: 83 -> 71; 2000 x 512 x 4096 24.8 -> 25.6 (the exchange;
// even at n = 1024).  The reads come before the copies: 5 us slower the other
// way round at 2048 x 4096 x 4096.
//
// ROWS (128 x 256): the wave rows split the tokens instead, 64 each, and multiply
// whole stages.  Nothing is exchanged after the loop (256 KB through LDS, about
// a microsecond a tile), for a third more LDS reads a stage.  Measured (whole
// backward calls, 1350 drawn; k-split time over this one's): 1.06 to 1.09 up to 8
// stages, 1.05 to 1.08 at 12, 1.03 to 1.07 at 16, 1.02 to 1.05 at 24, 1.00 at 33
// to 64, 0.97 to 1.00 above.
template <int BM, int BN, int RP, bool DROP, bool GRP, bool FULL, bool ROWS>
__device__ __forceinline__ void dx_ks_tile(const DxArgs& p, const DxGroup& grp, int m0, int l0, char* smem) {
  constexpr int NT = 512, WN = BM == 128 ? 4 : 2;   // waves along the columns
  constexpr int NK = ROWS ? 1 : 8 / WN;             // n shares
  constexpr int KP = ROWS ? 1 : NK / 2;             // 64-wide n pieces per stage
  constexpr int NKK = ROWS ? 2 : 1;                 // 32-wide n halves a wave multiplies per stage
  constexpr int NA = BN / WN / 16, NB = (ROWS ? 64 : BM) / 16;   // 16-column and 16-token fragments per wave
  constexpr int NOB = NB / NK;                      // token fragments a wave finishes
  constexpr int PIECE = BM * 128 + 64 * BN * 2, STAGE = KP * PIECE;
  constexpr int NBUF = dx_ks_bufs(BM, BN);
  constexpr int KS2 = 2 * RP, NSLAB = (KS2 + 63) / 64;
  constexpr int CPR = BN / 8;                      // 16-byte chunks per W tile row
  constexpr int NCOPY = KP * (BM / 64 + BN / 64);  // copies per wave and stage
  static_assert(BM == 128 ? BN == 128 || BN == 192 || BN == 256 : BM == 64 && (BN == 64 || BN == 128), "tile shapes");
  static_assert(!ROWS || BM == 128, "wave rows of 64 tokens");
  const int m = p.m, n = p.n, k = p.k, r = p.r;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wk = ROWS ? 0 : wave / WN, wn = wave % WN;
  const int i0 = ROWS ? 64 * (wave / WN) : 0;       // the wave's first token in the tile
  const bool second = wave >= 4;                    // the waves that run one slot behind
  const int g = lane >> 4, c16 = lane & 15;
  const uint32_t wrow = (uint32_t)k * 2, urow = (uint32_t)KS2 * 2;
  const __amdgpu_buffer_rsrc_t rsU = make_rsrc(p.dU2 + (size_t)m0 * KS2, (uint64_t)min(BM, p.mp - m0) * urow);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(p.A, (uint64_t)r * wrow);
  const int nkb = GRP ? grp.nkb : (n + 63) / 64;
  const int NM = (nkb + KP - 1) / KP;               // n stages, then the slab's
  const int T = NM + ((GRP || DROP) ? 0 : (NSLAB + KP - 1) / KP);
  using Cursor = DxCursor<GRP, KP>;
  Cursor cur[2] = {Cursor(p, grp, m0, BM, 0), Cursor(p, grp, m0, BM, KP - 1)};   // (the second: with two pieces)
  int pn0[2], pleft[2];   // per piece: first n, and its count of n (branches only here)
  auto advance = [&]() LORA_INLINE {
#pragma unroll
    for (int q = 0; q < KP; ++q) {
      cur[q].advance(grp);
      pleft[q] = KP == 1 ? 64 : uniform(min(64, max(0, cur[q].n - cur[q].sl * 64)));   // (kept in scalar registers)
      pn0[q] = pleft[q] > 0 ? cur[q].sl * 64 : 0;   // (past the last piece: no offset beyond the resource)
    }
  };

  // dY copy i: rows 64 i + 8 wave + lane / 8; W copy i: the tile's 16-byte
  // positions 64 (8 i + wave) + lane.  The lane's position holds the logical
  // chunk of the tile's swizzle (dY: the same for every i).
  const int yr0 = 8 * wave + (lane >> 3);
  const int ycol = 8 * ((lane & 7) ^ kc_swz(yr0));
  int wr[BN / 64], wcol[BN / 64];
#pragma unroll
  for (int i = 0; i < BN / 64; ++i) {
    const int pos = 64 * (8 * i + wave) + lane;
    wr[i] = pos / CPR;
    wcol[i] = l0 + 8 * ((pos % CPR) ^ mc16_swz_of<BN>(wr[i]));
  }
  auto copy_main = [&](int boff) LORA_INLINE {       // the cursors' pieces
#pragma unroll
    for (int q = 0; q < KP; ++q) {
      const Cursor& c = cur[q];
      char* sb = smem + boff + q * PIECE + wave * 1024;
      const int n0 = pn0[q];
      const bool yok = KP == 1 ? (FULL || n0 + ycol < c.n) : ycol < pleft[q];
      const uint32_t yoff = (uint32_t)yr0 * c.yr + (uint32_t)ycol * 2;
#pragma unroll
      for (int i = 0; i < BM / 64; ++i)
        dma16(c.rsY, yok ? yoff + (uint32_t)(64 * i) * c.yr : kOOB, (uint32_t)n0 * 2, sb + i * 8192);
      const int wrows = KP == 1 ? (FULL ? 64 : uniform(min(64, c.n - n0))) : pleft[q];
      const __amdgpu_buffer_rsrc_t rsW = make_rsrc(c.W + (size_t)n0 * k, (uint64_t)wrows * wrow);
#pragma unroll
      for (int i = 0; i < BN / 64; ++i)
        dma16(rsW, FULL || wcol[i] < k ? (uint32_t)wr[i] * wrow + (uint32_t)wcol[i] * 2 : kOOB, 0,
              sb + BM * 128 + i * 8192);
    }
  };
  auto copy_slab = [&](int kb, int boff) LORA_INLINE {
#pragma unroll
    for (int q = 0; q < KP; ++q) {
      char* sb = smem + boff + q * PIECE + wave * 1024;
      const int kk0 = ((kb - NM) * KP + q) * 64;
      const uint32_t uoff = (uint32_t)(kk0 + ycol) * 2;
#pragma unroll
      for (int i = 0; i < BM / 64; ++i)
        dma16(rsU, uoff < urow ? (uint32_t)(yr0 + 64 * i) * urow + uoff : kOOB, 0, sb + i * 8192);
#pragma unroll
      for (int i = 0; i < BN / 64; ++i) {
        const int kk = kk0 + wr[i], t = kk % RP;
        dma16(rsA, ((FULL || wcol[i] < k) && kk < KS2 && t < r) ? (uint32_t)t * wrow + (uint32_t)wcol[i] * 2 : kOOB, 0,
              sb + BM * 128 + i * 8192);
      }
    }
  };
  // Fragment addresses in buffer 0: W rows 32 (wk % 2) + 8 g + e of piece wk / 2
  // (second read of a pair 4 rows further), columns j1 + 16 a + 4 q; dY as
  // kc_read.
  const int j1 = wn * (BN / WN);                    // the wave's first column in the tile
  uint32_t wa[NA];
  {
    const int e = c16 >> 2, q = c16 & 3;
#pragma unroll
    for (int a = 0; a < NA; ++a)
      wa[a] = lds_addr(smem + (wk >> 1) * PIECE + BM * 128 +
                       mc16_offset<BN>(32 * (wk & 1) + 8 * g + e, (j1 + 16 * a) / 8 + (q >> 1)) + (q & 1) * 8);
  }
  floatx4 acc[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  short8 fy[NKK][NB];
  short4v wl[NKK * NA], wh[NKK * NA];
  auto slot_end = [&]() LORA_INLINE {
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int st = 0; st < NBUF - 1; ++st) {
    if (st < NM) {
      advance();
      copy_main(st * STAGE);
    } else if (st < T) {
      copy_slab(st, st * STAGE);
    }
  }
  if (T >= NBUF - 1) wait_vmcnt<(NBUF - 2) * NCOPY>();
  else wait_vmcnt<0>();
  slot_end();                    // stage 0 has landed
  if (second) slot_end();        // half 1 runs one slot behind
  int rb = 0, wb = (NBUF - 1) * STAGE;
  // Stage kb; mode 0: refills a buffer with an n stage, 1: with a slab stage,
  // 2: with none.  Nothing branches between the assembly reads and their wait.
  auto stage = [&](int kb, auto mode) LORA_INLINE {
    constexpr int MODE = decltype(mode)::value;
    if constexpr (MODE == 0) advance();
    const char* Ys = smem + rb + (wk >> 1) * PIECE;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
      for (int b = 0; b < NB; ++b) fy[kk][b] = kc_read(Ys, i0 + 16 * b + c16, 4 * ((wk & 1) + kk) + g);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      ds_read_tr_b64_asm<0>(wl[a], wa[a] + (uint32_t)rb);
      ds_read_tr_b64_asm<4 * BN * 2>(wh[a], wa[a] + (uint32_t)rb);
      if constexpr (ROWS) {
        ds_read_tr_b64_asm<32 * BN * 2>(wl[NA + a], wa[a] + (uint32_t)rb);
        ds_read_tr_b64_asm<36 * BN * 2>(wh[NA + a], wa[a] + (uint32_t)rb);
      }
    }
    if constexpr (MODE == 0) copy_main(wb);
    if constexpr (MODE == 1) copy_slab(kb + NBUF - 1, wb);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NA == 4 && ROWS)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(wl[0]), "+v"(wh[0]), "+v"(wl[1]), "+v"(wh[1]), "+v"(wl[2]), "+v"(wh[2]), "+v"(wl[3]),
                     "+v"(wh[3]), "+v"(wl[4]), "+v"(wh[4]), "+v"(wl[5]), "+v"(wh[5]), "+v"(wl[6]), "+v"(wh[6]),
                     "+v"(wl[7]), "+v"(wh[7]));
    else if constexpr (NA == 4)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(wl[0]), "+v"(wh[0]), "+v"(wl[1]), "+v"(wh[1]), "+v"(wl[2]), "+v"(wh[2]), "+v"(wl[3]),
                     "+v"(wh[3]));
    else if constexpr (NA == 3)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(wl[0]), "+v"(wh[0]), "+v"(wl[1]), "+v"(wh[1]), "+v"(wl[2]), "+v"(wh[2]));
    else
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(wl[0]), "+v"(wh[0]), "+v"(wl[1]), "+v"(wh[1]));
    static_assert(NA >= 2 && NA <= 4 && (!ROWS || NA == 4), "fragments of the wait");
    if (second) wait_vmcnt<MODE == 2 ? 0 : (NBUF - 2) * NCOPY>();
    slot_end();
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const short8 w8 = join4(wl[kk * NA + a], wh[kk * NA + a]);
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = mfma16x16x32(w8, fy[kk][b], acc[a][b]);
      }
    __builtin_amdgcn_sched_barrier(0);
    if (!second) wait_vmcnt<MODE == 2 ? 0 : (NBUF - 2) * NCOPY>();
    slot_end();
    rb = rb + STAGE == NBUF * STAGE ? 0 : rb + STAGE;
    wb = wb + STAGE == NBUF * STAGE ? 0 : wb + STAGE;
  };
  int kb = 0;
  for (; kb + NBUF - 1 < NM; ++kb) stage(kb, std::integral_constant<int, 0>{});
  if constexpr (!GRP && !DROP)
    for (; kb + NBUF - 1 < T; ++kb) stage(kb, std::integral_constant<int, 1>{});
  for (; kb < T; ++kb) stage(kb, std::integral_constant<int, 2>{});
  if (!second) slot_end();

  // Exchange: wave wk finishes its token fragments NOB wk .., moved to own[..][0
  // .. NOB - 1]; partial sums are added in n-share order.
  auto& own = acc;
  floatx4* xin = reinterpret_cast<floatx4*>(smem) + (size_t)(NK == 4 ? wn * 4 + wk : wave) * NA * 4 * 64;   // to this wave
  if constexpr (ROWS) {   // the tile's sums are whole
  } else if constexpr (NK == 2) {   // (branches on wk: selects of every element cost a microsecond)
    floatx4* dst = reinterpret_cast<floatx4*>(smem) + (size_t)(wave ^ 4) * NA * 4 * 64;
    if (wk == 0) {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) dst[(a * 4 + b) * 64 + lane] = acc[a][4 + b];
    } else {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          dst[(a * 4 + b) * 64 + lane] = acc[a][b];
          own[a][b] = acc[a][4 + b];
        }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) own[a][b] += xin[(a * 4 + b) * 64 + lane];
  } else {   // [wn][token fragment = finishing share][share][column fragment]
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        reinterpret_cast<floatx4*>(smem)[(size_t)(((wn * 4 + b) * 4 + wk) * NA + a) * 64 + lane] = acc[a][b];
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      own[a][0] = xin[a * 64 + lane];
#pragma unroll
      for (int q = 1; q < 4; ++q) own[a][0] += xin[(q * NA + a) * 64 + lane];
    }
  }
  const int i1 = i0 + 16 * NOB * wk;                // the first token that the wave finishes

  if constexpr (GRP || DROP) {
    constexpr int UP = KS2 + 8;                    // Us row pitch in elements (16-byte multiple)
    constexpr int US_BYTES = BM * UP * 2, AS_BYTES = RP * BN * 2;
    static_assert(US_BYTES + AS_BYTES + BM * BN / 8 <= NBUF * STAGE, "the rank-r operands fit the stage LDS");
    u16* Us = reinterpret_cast<u16*>(smem);
    char* As = smem + US_BYTES;
    if constexpr (GRP) {
      for (int pq = 0; pq < grp.count; ++pq) {
        __syncthreads();                           // the exchange, or the previous projection's reads, are done
        stage_rank_operands<BM, BN, RP, NT>(pick(grp.dU2, pq), pick(grp.A, pq), Us, As, m0, l0, p.mp, k, r, tid);
        __syncthreads();
#pragma unroll 1
        for (int kk = 0; kk < KS2 / 32; ++kk) {
          short8 uf[NOB];
#pragma unroll
          for (int b = 0; b < NOB; ++b)
            uf[b] = *reinterpret_cast<const short8*>(Us + (i1 + 16 * b + c16) * UP + 32 * kk + 8 * g);
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            const short8 af = slab_frag<BN, RP>(As, kk, j1 + 16 * a, lane);
#pragma unroll
            for (int b = 0; b < NOB; ++b) own[a][b] = mfma16x16x32(af, uf[b], own[a][b]);
          }
        }
      }
    } else {
      __syncthreads();                             // the exchange has been read
      stage_rank_operands<BM, BN, RP, NT>(p.dU2, p.A, Us, As, m0, l0, p.mp, k, r, tid);
      uint8_t* Kb = reinterpret_cast<uint8_t*>(smem + US_BYTES + AS_BYTES);   // keep bytes of the tile [BM][BN / 8]
      const uint32_t kb8 = (uint32_t)k / 8;
      const __amdgpu_buffer_rsrc_t rsK = make_rsrc(p.keep + (size_t)m0 * kb8, (uint64_t)min(BM, m - m0) * kb8);
      for (int q = tid; q < BM * (BN / 64); q += NT) {
        const int i = q / (BN / 64), c = q % (BN / 64);
        *reinterpret_cast<uint2*>(Kb + i * (BN / 8) + 8 * c) =
            buf_load8(rsK, (uint32_t)i * kb8 + (uint32_t)l0 / 8 + 8 * c);
      }
      __syncthreads();
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        floatx4 tmp[NOB];
#pragma unroll
        for (int b = 0; b < NOB; ++b) tmp[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KS2 / 32; ++kk) {
          const short8 af = slab_frag<BN, RP>(As, kk, j1 + 16 * a, lane);
#pragma unroll
          for (int b = 0; b < NOB; ++b)
            tmp[b] = mfma16x16x32(
                af, *reinterpret_cast<const short8*>(Us + (i1 + 16 * b + c16) * UP + 32 * kk + 8 * g), tmp[b]);
        }
        // lane: token c16 of fragment b, columns 16 a + 4 g + q
#pragma unroll
        for (int b = 0; b < NOB; ++b) {
          const uint32_t bits = (uint32_t)Kb[(i1 + 16 * b + c16) * (BN / 8) + (j1 + 16 * a) / 8 + (g >> 1)] >> (4 * (g & 1));
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if ((bits >> q) & 1u) own[a][b][q] += p.inv_keep * tmp[b][q];
        }
      }
    }
  }
  // Stored through the wave's own exchange region, which nobody else touches
  // after the exchange; the rank-r operands of a group or dropout lie there too.
  if constexpr (GRP || DROP) __syncthreads();
  constexpr int OUT = out16_bytes<NA, NOB>();
  static_assert(OUT <= NA * 4 * 1024 && 8 * NA * 4 * 1024 <= NBUF * STAGE, "output staging and exchange");
  floatx4 v[NA][NOB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NOB; ++b) v[a][b] = own[a][b];
  store_out16<NA, NOB>(v, reinterpret_cast<char*>(xin), p.dX + (size_t)(m0 + i1) * k + l0 + j1, (size_t)k, m - m0 - i1,
                       k - l0 - j1, lane);
}

// The 256 x 256 tile (whole stages and columns).
// Stages 0 .. nkb-1 over n, then the NSLAB slab stages, two in LDS.  The
// wave rows take turns as in the forward's 256 x 256 tile: per stage four
// phases of sixteen products -- (W half 0, dY half 0), (W 1, dY 0), (W 0, dY
// 1), (W 1, dY 1) -- and while one row multiplies, the other reads the dY
// half 0, W half 1, dY half 1, or the next stage's W half 0, and refills
// the quarter that both rows read in the phase before for the stage after
// next.  dY half h: tokens 64 h .. + 63 of both wave rows.  W half h:
// columns 128 h .. + 127 of the tile as [64][128] (wave column wn takes
// columns 128 h + 32 wn .. + 31), so that a copy takes whole 256-byte row
// pieces.  Nothing branches between the assembly reads and their wait.  The
// reads before the first slot are closed by a barrier of all eight waves before
// the second row's extra one.
// Measured (whole backward call, against all waves in step on 32x32x16
// products): 8192 x 4096 x 11008 (tokens x n x k), r = 64: 712 -> 650 us taking
// turns, 628 on the 16x16x32 products used here; 4096 x 11008 x 4096, r = 16:
// 305, 305 and 292.
template <int RP, bool GRP>
__device__ __forceinline__ void dx_big_tile(const DxArgs& p, const DxGroup& grp, int m0, int l0, char* smem) {
  constexpr int BM = 256, BN = 256, NT = 512, WTI = 128;
  constexpr int STAGE = BM * 128 + 64 * BN * 2;
  constexpr int KS2 = 2 * RP, NSLAB = (KS2 + 63) / 64;
  const int m = p.m, k = p.k, r = p.r;
  u16* dX = p.dX;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int g16 = lane >> 4, c16 = lane & 15;
  const uint32_t wrow = (uint32_t)k * 2, urow = (uint32_t)KS2 * 2;
  const __amdgpu_buffer_rsrc_t rsU = make_rsrc(p.dU2 + (size_t)m0 * KS2, (uint64_t)min(BM, p.mp - m0) * urow);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(p.A, (uint64_t)r * wrow);
  const int nkb = GRP ? grp.nkb : (p.n + 63) / 64;
  // acc[a][b]: columns big_col(a) .. + 15 of the tile, tokens 16 b .. of the wave row.
  floatx4 acc[4][8];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto big_col = [&](int a) LORA_INLINE { return 128 * (a >> 1) + 32 * wn + 16 * (a & 1); };
  const int T = nkb + (GRP ? 0 : NSLAB);   // (group epilogues add dU A)
  DxCursor<GRP, 1> cur(p, grp, m0, BM, 0);   // advanced once per stage
  const int l8 = lane >> 3, l16 = lane >> 4;
  const int yr0 = 8 * wave + l8;                            // dY row of this lane in copy 0 (+ 64 h + 128 i)
  const uint32_t ych = (uint32_t)(((lane & 7) ^ kc_swz(yr0)) << 4);
  const int wr0 = 4 * wave + l16;                           // W row (+ 32 i)
  const int wc = (lane & 15) ^ mc16_swz(wr0);               // logical 8-column chunk of the half
  using Slab = std::true_type;
  using Main = std::false_type;
  // Quarters of stage kb (Main: the cursor's stage).
  auto copy_y = [&](int kb, int h, auto slab) LORA_INLINE {
    char* sb = smem + (kb & 1) * STAGE + wave * 1024 + h * 8192;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t row = (uint32_t)(yr0 + 64 * h + 128 * i);
      if constexpr (decltype(slab)::value) {
        const uint32_t off = (uint32_t)(kb - nkb) * 128 + ych;
        dma16(rsU, off < urow ? row * urow + off : kOOB, 0, sb + i * 16384);
      } else {
        dma16(cur.rsY, row * cur.yr + ych, (uint32_t)cur.sl * 128, sb + i * 16384);
      }
    }
  };
  auto copy_w = [&](int kb, int h, auto slab) LORA_INLINE {
    char* sb = smem + (kb & 1) * STAGE + BM * 128 + h * 16384 + wave * 1024;
    const uint32_t col = (uint32_t)(l0 + 128 * h + 8 * wc) * 2;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = wr0 + 32 * i;
      if constexpr (decltype(slab)::value) {
        const int kk = (kb - nkb) * 64 + row, t = kk % RP;
        dma16(rsA, (kk < KS2 && t < r) ? (uint32_t)t * wrow + col : kOOB, 0, sb + i * 8192);
      } else {
        const __amdgpu_buffer_rsrc_t rsW = make_rsrc(cur.W + (size_t)cur.sl * 64 * k, (uint64_t)64 * wrow);
        dma16(rsW, (uint32_t)row * wrow + col, 0, sb + i * 8192);
      }
    }
  };
  // Fragment addresses in buffer 0: W half 0, k rows 0 .. 31 (half 1 + 16384,
  // rows 32 .. 63 + 8192, second read of a pair + 1024), dY as kc_read.
  uint32_t wa[2];
  {
    const int e = c16 >> 2, q = c16 & 3;
#pragma unroll
    for (int a = 0; a < 2; ++a)
      wa[a] = lds_addr(smem + BM * 128 + mc16_offset<128>(8 * g16 + e, 4 * wn + 2 * a + (q >> 1)) + (q & 1) * 8);
  }
  short8 fyq[2][4];                    // the current dY half: [32-wide k][token fragment]
  short4v wl[2][4], wh[2][4];          // W halves: [half][2 (32-wide k) + fragment], rows 0..3 and 4..7 of eight
  auto read_y = [&](int kb, int h) LORA_INLINE {
    const char* Ys = smem + (kb & 1) * STAGE;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int b = 0; b < 4; ++b) fyq[kk][b] = kc_read(Ys, wm * WTI + 64 * h + 16 * b + c16, 4 * kk + g16);
  };
  auto read_w = [&](int kb, auto hc) LORA_INLINE {
    constexpr int H = decltype(hc)::value;
    const uint32_t a0 = wa[0] + (uint32_t)((kb & 1) * STAGE), a1 = wa[1] + (uint32_t)((kb & 1) * STAGE);
    ds_read_tr_b64_asm<H * 16384>(wl[H][0], a0);
    ds_read_tr_b64_asm<H * 16384 + 1024>(wh[H][0], a0);
    ds_read_tr_b64_asm<H * 16384>(wl[H][1], a1);
    ds_read_tr_b64_asm<H * 16384 + 1024>(wh[H][1], a1);
    ds_read_tr_b64_asm<H * 16384 + 8192>(wl[H][2], a0);
    ds_read_tr_b64_asm<H * 16384 + 9216>(wh[H][2], a0);
    ds_read_tr_b64_asm<H * 16384 + 8192>(wl[H][3], a1);
    ds_read_tr_b64_asm<H * 16384 + 9216>(wh[H][3], a1);
  };
  auto slot_end = [&]() LORA_INLINE {
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // Reads done (the W fragments pass through the wait, so their products
  // stay behind it); at most `left` quarters' copies in flight.
  auto ready = [&](auto left, auto hc) LORA_INLINE {
    constexpr int H = decltype(hc)::value;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (H >= 0)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(wl[H][0]), "+v"(wh[H][0]), "+v"(wl[H][1]), "+v"(wh[H][1]), "+v"(wl[H][2]), "+v"(wh[H][2]),
                     "+v"(wl[H][3]), "+v"(wh[H][3]));
    else
      wait_lgkm0();
    wait_vmcnt<2 * decltype(left)::value>();
    slot_end();
  };
  auto products = [&](int hw, int hy) LORA_INLINE {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const short8 w8 = join4(wl[hw][2 * kk + a], wh[hw][2 * kk + a]);
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[2 * hw + a][4 * hy + b] = mfma16x16x32(w8, fyq[kk][b], acc[2 * hw + a][4 * hy + b]);
      }
    __builtin_amdgcn_sched_barrier(0);
    slot_end();
  };
  using N1 = std::integral_constant<int, -1>;
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using I4 = std::integral_constant<int, 4>;
  using I5 = std::integral_constant<int, 5>;
  using I6 = std::integral_constant<int, 6>;
  // mode 0: refill with n stages, 3: with slab stages, 1: the last stage but
  // one, 2: the last.
  auto stage = [&](int kb, auto mode) LORA_INLINE {
    constexpr int MODE = decltype(mode)::value;
    constexpr bool FILL = MODE == 0 || MODE == 3;
    using S = std::integral_constant<bool, MODE == 3>;
    if constexpr (MODE == 0) cur.advance(grp);
    read_y(kb, 0);
    if constexpr (FILL) { copy_w(kb + 2, 0, S{}); ready(I6{}, N1{}); }
    else if constexpr (MODE == 1) ready(I5{}, N1{});
    else ready(I1{}, N1{});
    products(0, 0);
    read_w(kb, I1{});
    if constexpr (FILL) { copy_y(kb + 2, 0, S{}); ready(I6{}, I1{}); }
    else if constexpr (MODE == 1) ready(I4{}, I1{});
    else ready(I0{}, I1{});
    products(1, 0);
    read_y(kb, 1);
    if constexpr (FILL) { copy_w(kb + 2, 1, S{}); ready(I6{}, N1{}); }
    else if constexpr (MODE == 1) ready(I3{}, N1{});
    else ready(I0{}, N1{});
    products(0, 1);
    if constexpr (MODE != 2) read_w(kb + 1, I0{});
    if constexpr (FILL) { copy_y(kb + 2, 1, S{}); ready(I6{}, I0{}); }
    else if constexpr (MODE == 1) ready(I2{}, I0{});
    else ready(I0{}, N1{});
    products(1, 1);
  };
  auto fill = [&](int kb) LORA_INLINE {
    if (kb < nkb) {
      cur.advance(grp);
      copy_w(kb, 0, Main{}); copy_y(kb, 0, Main{}); copy_w(kb, 1, Main{}); copy_y(kb, 1, Main{});
    } else {
      copy_w(kb, 0, Slab{}); copy_y(kb, 0, Slab{}); copy_w(kb, 1, Slab{}); copy_y(kb, 1, Slab{});
    }
  };
  fill(0);
  if (T > 1) {
    fill(1);
    wait_vmcnt<12>();
  } else {
    wait_vmcnt<0>();
  }
  slot_end();
  read_w(0, I0{});
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(wl[0][0]), "+v"(wh[0][0]), "+v"(wl[0][1]), "+v"(wh[0][1]), "+v"(wl[0][2]), "+v"(wh[0][2]),
                 "+v"(wl[0][3]), "+v"(wh[0][3]));
  slot_end();                    // every wave has read the quarter that the first read slot refills
  if (wm == 1) slot_end();       // the second wave row runs one slot behind
  int kb = 0;
  for (; kb + 2 < nkb; ++kb) stage(kb, I0{});
  if constexpr (!GRP)
    for (; kb + 2 < T; ++kb) stage(kb, I3{});
  if (T > 1) stage(kb++, I1{});
  stage(kb, I2{});
  if (wm == 0) slot_end();

  if constexpr (GRP) {
    // LDS after the k loop, per projection: dU_g rows (high | low) and A_g rows;
    // acc += [dU_hi | dU_lo] [A_g; A_g].
    constexpr int UP = KS2 + 8;
    constexpr int US_BYTES = BM * UP * 2, AS_BYTES = RP * BN * 2;
    static_assert(US_BYTES + AS_BYTES <= 2 * STAGE, "the rank-r operands fit the stage LDS");
    u16* Us = reinterpret_cast<u16*>(smem);
    char* As = smem + US_BYTES;
    for (int pq = 0; pq < grp.count; ++pq) {
      if (pq > 0) __syncthreads();                  // the previous projection's reads are done
      stage_rank_operands<BM, BN, RP, NT>(pick(grp.dU2, pq), pick(grp.A, pq), Us, As, m0, l0, p.mp, k, r, tid);
      __syncthreads();
#pragma unroll 1
      for (int kk = 0; kk < KS2 / 32; ++kk) {
        short8 uf[8];
#pragma unroll
        for (int b = 0; b < 8; ++b)
          uf[b] = *reinterpret_cast<const short8*>(Us + (wm * WTI + 16 * b + c16) * UP + 32 * kk + 8 * g16);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const short8 af = slab_frag<BN, RP>(As, kk, big_col(a), lane);
#pragma unroll
          for (int b = 0; b < 8; ++b) acc[a][b] = mfma16x16x32(af, uf[b], acc[a][b]);
        }
      }
    }
    __syncthreads();
  }

  // The wave's columns lie in two pieces: the tile goes through LDS as bf16 and
  // is stored in whole rows.
  static_assert(2 * STAGE >= 256 * 512, "the bf16 tile fits the stage LDS");
#pragma unroll
  for (int b = 0; b < 8; ++b)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int row = wm * WTI + 16 * b + c16, col = big_col(a) + 4 * g16;
      const floatx4 v = acc[a][b];
      const uint32_t lo = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
      const uint32_t hi = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
      // 16-byte chunk col / 8 at position (col / 8) ^ (row % 32)
      *reinterpret_cast<uint2*>(smem + row * 512 + (((col >> 3) ^ (row & 31)) << 4) + (col & 7) * 2) = uint2{lo, hi};
    }
  __syncthreads();
  for (int e = tid; e < BM * 32; e += NT) {   // (whole column tiles: FULL)
    const int row = e >> 5, ch = e & 31;
    const int4v v = *reinterpret_cast<const int4v*>(smem + row * 512 + ((ch ^ (row & 31)) << 4));
    if (m0 + row < m) *reinterpret_cast<int4v*>(dX + (size_t)(m0 + row) * k + l0 + 8 * ch) = v;
  }
}

// After its tile, every workgroup sums a slice of the dA, dB partials
// (complete: the token reductions ran before this launch in stream order).
// (WM and WN stand in the kernel's name alone.)
template <int BM, int BN, int WM, int WN, int RP, bool DROP, bool GRP, bool FULL>
__global__ __launch_bounds__(512) void lora_bwd_dx_kernel(
    const u16* __restrict__ dY, const u16* __restrict__ W, const u16* __restrict__ dU2,
    const u16* __restrict__ A, const uint8_t* __restrict__ keep, u16* __restrict__ dX, int m, int n, int k,
    int r, int mp, float inv_keep, int tiles_m, int tiles_n, int l_begin, FinalizeArgs fin, DxGroup grp) {
  static_assert(BM <= 128 || (BM == 256 && BN == 256 && FULL && !DROP), "tile shapes");
  __shared__ __attribute__((aligned(1024))) char smem[BM == 256 ? 2 * 65536 : dx_ks_smem(BM, BN)];
  int tm, tn;
  tile_coords(tiles_m, tiles_n, 8, (int)blockIdx.x, tm, tn);
  const DxArgs p{dY, W, dU2, A, keep, dX, m, n, k, r, mp, inv_keep};
  if constexpr (BM == 256) dx_big_tile<RP, GRP>(p, grp, tm * BM, l_begin + tn * BN, smem);
  else dx_ks_tile<BM, BN, RP, DROP, GRP, FULL, false>(p, grp, tm * BM, l_begin + tn * BN, smem);
  const int first = (int)blockIdx.x * 512 + (int)threadIdx.x, stride = (int)gridDim.x * 512;
  if (GRP) {
    for (int pq = 0; pq < grp.count; ++pq) finalize_partials(pick(grp.fin, pq), first, stride);
  } else {
    finalize_partials(fin, first, stride);
  }
}

template <int BM, int BN, int WM, int WN, int RP, bool DROP, bool GRP, bool FULL>
__global__ __launch_bounds__(512) void lora_bwd_rows_dx_kernel(
    const u16* __restrict__ dY, const u16* __restrict__ W, const u16* __restrict__ dU2,
    const u16* __restrict__ A, const uint8_t* __restrict__ keep, u16* __restrict__ dX, int m, int n, int k,
    int r, int mp, float inv_keep, int tiles_m, int tiles_n, int l_begin, FinalizeArgs fin, DxGroup grp) {
  static_assert(BM == 64 * WM && BN == 64 * WN && WM * WN == 8, "wave tiles of 64 x 64");
  __shared__ __attribute__((aligned(1024))) char smem[dx_ks_smem(BM, BN)];
  int tm, tn;
  tile_coords(tiles_m, tiles_n, 8, (int)blockIdx.x, tm, tn);
  const DxArgs p{dY, W, dU2, A, keep, dX, m, n, k, r, mp, inv_keep};
  dx_ks_tile<BM, BN, RP, DROP, GRP, FULL, true>(p, grp, tm * BM, l_begin + tn * BN, smem);
  const int first = (int)blockIdx.x * 512 + (int)threadIdx.x, stride = (int)gridDim.x * 512;
  if (GRP) {
    for (int pq = 0; pq < grp.count; ++pq) finalize_partials(pick(grp.fin, pq), first, stride);
  } else {
    finalize_partials(fin, first, stride);
  }
}

// ---------------------------------------------------------------------------
// Fused backward for ranks up to 16 (no dropout): the dX GEMM also forms dU
// and the dB partials from the dY tiles it stages, so no other launch reads
// dY.  Tile of 128 tokens x 256 input features, 2 x 4 waves of 64 x 64 all in
// step, stages of 64 along n in two LDS buffers, loaded two stages ahead into
// registers; each stage's last substep multiplies after its barrier, while the
// next stage's first fragments are read.
//   dU^T = B^T dY^T: each stage also stages its 64 B rows ([64][16] bf16,
//     zero beyond r and n); at substep wn of every stage, wave (wm, wn)
//     multiplies the transposed B rows (rows t >= 16 of the operand zero)
//     with its own dY fragments.  After the loop the four partial sums of each
//     token are added in wn order, s dU is split into bf16 high and low parts
//     in LDS, and the rank-r term [dU_hi | dU_lo] [A; A] is added to the dX
//     tile.  The workgroups of column tile 0 also store the parts transposed
//     (dUt2 [16][mp], the bf16 high part) for the dA reduction.
//   dB^T partials: at the stages st with st % tiles_n == tn, four waves (the
//     lower or upper four, alternately) each form U^T dY for 16 of the stage's
//     64 n over the tile's 128 tokens, with U^T as high and low bf16 parts
//     (staged in LDS in the prologue), and store the tile row's partial
//     pbt [tm][16][n] (s is applied by the finalize).
// FULL: n a multiple of 64 and k of 256 (no bound checks on the loads).
// FASTB: r a multiple of 8 (B rows staged with 16-byte loads).
template <bool FULL, bool FASTB>
__global__ __launch_bounds__(512) void lora_bwd_dxf_kernel(
    const u16* __restrict__ dY, const u16* __restrict__ W, const u16* __restrict__ A, const u16* __restrict__ B,
    const float* __restrict__ U, u16* __restrict__ dX, u16* __restrict__ dUt2, float* __restrict__ pbt, int m, int n,
    int k, int r, int mp, float s, int tiles_m, int tiles_n) {
  constexpr int BM = 128, BN = 256, WM = 2, WN = 4, RP = 16;
  constexpr int NW = WM * WN, NT = 64 * NW;
  constexpr int WTI = BM / WM, WTJ = BN / WN;
  constexpr int FI = WTI / 32, FJ = WTJ / 32;
  constexpr int YB = BM * 128, WB = 64 * BN * 2, BB = 64 * RP * 2;
  constexpr int STAGE = YB + WB + BB;
  constexpr int CPR = BN / 8;                       // 16-byte chunks per W tile row
  constexpr int CY = BM * 8, CW = 64 * CPR;
  constexpr int LY = CY / NT, LW = CW / NT, LW1 = LW / 2;
  constexpr int UTP = BM * 2 + 16;                  // U^T row pitch in bytes
  constexpr int UT_OFF = 2 * STAGE;
  static_assert(CY % NT == 0 && CW % NT == 0 && UT_OFF + 2 * RP * UTP <= 160 * 1024, "tile shape and LDS budget");
  __shared__ __attribute__((aligned(1024))) char smem[UT_OFF + 2 * RP * UTP];

  int tm, tn;
  tile_coords(tiles_m, tiles_n, 8, (int)blockIdx.x, tm, tn);
  const int m0 = tm * BM, l0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int g = lane >> 5, c32 = lane & 31;
  const int g16 = lane >> 4, c16 = lane & 15;
  const uint32_t yrow = (uint32_t)n * 2, wrow = (uint32_t)k * 2;
  const __amdgpu_buffer_rsrc_t rsY = make_rsrc(dY + (size_t)m0 * n, (uint64_t)min(BM, m - m0) * yrow);
  const __amdgpu_buffer_rsrc_t rsA = make_rsrc(A, (uint64_t)r * wrow);
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B, (uint64_t)n * r * 2);
  const int nkb = (n + 63) / 64;

  // U^T of the tile's tokens: high parts in rows 0..15, low parts in rows
  // 16..31 (zero beyond r and m), for the dB products.
  char* Uts = smem + UT_OFF;
  {
    constexpr int UPT = BM * RP / NT;   // all loads issued before the first store
    static_assert(BM * RP % NT == 0, "U values per thread");
    const __amdgpu_buffer_rsrc_t rsU = make_rsrc(U + (size_t)m0 * r, (uint64_t)min(BM, m - m0) * r * 4);
    float uv[UPT];
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int e = tid + q * NT, i = e / RP, t = e - i * RP;
      uv[q] = buf_load4f(rsU, t < r ? (uint32_t)(i * r + t) * 4 : kOOB);
    }
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int e = tid + q * NT, i = e / RP, t = e - i * RP;
      const u16 h = f32_to_bf16(uv[q]);
      *reinterpret_cast<u16*>(Uts + t * UTP + i * 2) = h;
      *reinterpret_cast<u16*>(Uts + (RP + t) * UTP + i * 2) = f32_to_bf16(uv[q] - bf16_to_f32(h));
    }
  }

  // Staging registers, stored in pieces: 0 = the dY rows and (threads below
  // 128) one 16-byte half of a B row, 1 and 2 = the two halves of the W rows.
  int4v gy[LY], gw[LW], gb = int4v{0, 0, 0, 0};
  auto gload = [&](int st, int piece) LORA_INLINE {
    const int n0 = st * 64;
    if (piece == 0) {
#pragma unroll
      for (int i = 0; i < LY; ++i) {
        const int q = tid + i * NT;
        const int nn = n0 + 8 * (q & 7);
        gy[i] = buf_load16(rsY, (FULL || nn < n) ? (uint32_t)(q >> 3) * yrow + (uint32_t)nn * 2 : kOOB);
      }
      if (tid < 128) {   // waves 0 and 1: row n0 + tid / 2, ranks 8 (tid % 2) .. +7
        const int row = n0 + (tid >> 1), t0 = 8 * (tid & 1);
        if constexpr (FASTB) {
          gb = buf_load16(rsB, (row < n && t0 < r) ? ((uint32_t)row * r + t0) * 2 : kOOB);
        } else {
          uint32_t w[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const int t = t0 + 2 * x;
            const uint32_t lo = (row < n && t < r) ? B[(size_t)row * r + t] : 0u;
            const uint32_t hi = (row < n && t + 1 < r) ? B[(size_t)row * r + t + 1] : 0u;
            w[x] = lo | (hi << 16);
          }
          gb = int4v{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
        }
      }
    } else if (piece <= 2) {
      const __amdgpu_buffer_rsrc_t rsW = make_rsrc(W + (size_t)n0 * k, (uint64_t)min(64, n - n0) * wrow);
#pragma unroll
      for (int i = piece == 1 ? 0 : LW1; i < (piece == 1 ? LW1 : LW); ++i) {
        const int q = tid + i * NT;
        const int ll = l0 + 8 * (q % CPR);
        gw[i] = buf_load16(rsW, (FULL || ll < k) ? (uint32_t)(q / CPR) * wrow + (uint32_t)ll * 2 : kOOB);
      }
    }
  };
  auto swrite = [&](int buf, int piece) LORA_INLINE {
    char* sb = smem + buf * STAGE;
    if (piece == 0) {
#pragma unroll
      for (int i = 0; i < LY; ++i) {
        const int q = tid + i * NT;
        *reinterpret_cast<int4v*>(sb + kc_offset(q >> 3, q & 7)) = gy[i];
      }
      if (tid < 128) *reinterpret_cast<int4v*>(sb + YB + WB + tid * 16) = gb;   // Bs [64][16]
    } else if (piece <= 2) {
#pragma unroll
      for (int i = piece == 1 ? 0 : LW1; i < (piece == 1 ? LW1 : LW); ++i) {
        const int q = tid + i * NT;
        *reinterpret_cast<int4v*>(sb + YB + mc32_offset<BN>(q / CPR, q % CPR)) = gw[i];
      }
    }
  };

  floatx16 acc[FJ][FI], dacc[FI];
#pragma unroll
  for (int a = 0; a < FJ; ++a)
#pragma unroll
    for (int b = 0; b < FI; ++b) acc[a][b] = floatx16{};
#pragma unroll
  for (int b = 0; b < FI; ++b) dacc[b] = floatx16{};

  // Fragments of substep ks (16 n): W read transposed, dY as rows, and at
  // this wave's substep (ks == wn) the B^T operand: lane (g, c32) row t = c32
  // (zero for c32 >= 16), k = n 16 ks + 8g .. +7, read transposed from Bs
  // (rows of 32 bytes, no swizzle: a 16-lane read covers 128 contiguous bytes).
  short8 fw[2][FJ], fy[2][FI], fb = short8{};
  auto read_frags = [&](const char* sb, int ks, int p) LORA_INLINE {
    const char* Ys = sb;
    const char* Ws = sb + YB;
#pragma unroll
    for (int fj = 0; fj < FJ; ++fj) fw[p][fj] = mc32_read_tr<BN>(Ws, 16 * ks, wn * WTJ + 32 * fj, lane);
#pragma unroll
    for (int fi = 0; fi < FI; ++fi) fy[p][fi] = kc_read(Ys, wm * WTI + 32 * fi + c32, 2 * ks + g);
    if (ks == wn) {
      const int j = lane & 15;
      const char* p0 = sb + YB + WB + (16 * ks + 8 * g + (j >> 2)) * (RP * 2) + (j & 3) * 8;
      const short8 v = join4(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)p0),
                             __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)(p0 + 4 * RP * 2)));
      fb = ((lane >> 4) & 1) ? short8{} : v;
    }
  };
  auto multiply = [&](int p, int ks) LORA_INLINE {
#pragma unroll
    for (int fi = 0; fi < FI; ++fi)
#pragma unroll
      for (int fj = 0; fj < FJ; ++fj) acc[fj][fi] = mfma32x32x16(fw[p][fj], fy[p][fi], acc[fj][fi]);
    if (ks == wn) {
#pragma unroll
      for (int fi = 0; fi < FI; ++fi) dacc[fi] = mfma32x32x16(fb, fy[p][fi], dacc[fi]);
    }
  };
  // dB^T partial of stage st (its buffer sb): wave set (st / tiles_n) % 2,
  // wave f of the set takes n columns 16 f .. 16 f + 15 of the stage.
  auto dB_part = [&](const char* sb, int st) LORA_INLINE {
    const int f = wave - 4 * ((st / tiles_n) & 1);
    if (f < 0 || f >= 4) return;
    floatx4 d = floatx4{0.f, 0.f, 0.f, 0.f};
    const int j = lane & 15, col = 16 * f + 4 * (j & 3);
#pragma unroll
    for (int kt = 0; kt < BM / 32; ++kt) {
      // B operand: lane (g16, c16) column n 16 f + c16, k = tokens 32 kt + 8 g16 .. +7
      const int r0 = 32 * kt + 8 * g16 + (j >> 2);
      const char* p0 = sb + kc_offset(r0, col >> 3) + (col & 7) * 2;
      const char* p1 = sb + kc_offset(r0 + 4, col >> 3) + (col & 7) * 2;
      const short8 yb = join4(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)p0),
                              __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v*)p1));
      const short8 uh = *reinterpret_cast<const short8*>(Uts + c16 * UTP + (32 * kt + 8 * g16) * 2);
      const short8 ul = *reinterpret_cast<const short8*>(Uts + (RP + c16) * UTP + (32 * kt + 8 * g16) * 2);
      d = mfma16x16x32(uh, yb, d);
      d = mfma16x16x32(ul, yb, d);
    }
    const int cn = st * 64 + 16 * f + c16;   // lane: column cn, ranks 4 g16 .. +3
    if (FULL || cn < n) {
#pragma unroll
      for (int q = 0; q < 4; ++q) pbt[((size_t)tm * RP + 4 * g16 + q) * n + cn] = d[q];
    }
  };

#pragma unroll
  for (int j = 0; j < FJ; ++j) fw[1][j] = short8{};
#pragma unroll
  for (int j = 0; j < FI; ++j) fy[1][j] = short8{};
  auto stage = [&](int st, auto bufc, bool write_next, bool load_next) LORA_INLINE {
    constexpr int BUF = decltype(bufc)::value;
    const int cur = BUF >= 0 ? BUF : (st & 1);
    const char* sb = smem + cur * STAGE;
    read_frags(sb, 0, 0);
    multiply(1, 3);   // substep 3 of the previous stage (zero operands before stage 0)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (write_next) swrite(cur ^ 1, ks);
      if (load_next) gload(st + 2, ks);
      if (ks < 3) {
        read_frags(sb, ks + 1, (ks + 1) & 1);
        multiply(ks & 1, ks);
      }
    }
    if (st % tiles_n == tn) dB_part(sb, st);
    __syncthreads();
  };
#pragma unroll
  for (int pc = 0; pc < 3; ++pc) gload(0, pc);
#pragma unroll
  for (int pc = 0; pc < 3; ++pc) swrite(0, pc);
  __syncthreads();
  // (stages with run-time buffer parity: a loop over pairs of stages, each
  // buffer a compile-time constant, spills here)
  using BR = std::integral_constant<int, -1>;
  int st = 0;
  if (nkb >= 2) {
#pragma unroll
    for (int pc = 0; pc < 3; ++pc) gload(1, pc);
    for (; st + 2 < nkb; ++st) stage(st, BR{}, true, true);
    stage(st++, BR{}, true, false);   // st = nkb - 2: stores the last stage
  }
  stage(st, BR{}, false, false);
  multiply(1, 3);

  // ---- epilogue (LDS stage buffers free after the loop's last barrier):
  // red [NW][FI][8][64] fp32 (rows t < 16 of each wave's dU^T partials), Us2
  // [BM][UP] bf16 (s dU high | low), As2 [RP][BN] bf16 mn-contiguous (A rows
  // of the tile, zero beyond r and k).
  constexpr int RED = NW * FI * 8 * 64 * 4;
  constexpr int UP = 2 * RP + 8;
  static_assert(RED + BM * UP * 2 + RP * BN * 2 <= UT_OFF && NW * kYsBytes <= UT_OFF, "epilogue fits the stage LDS");
  float* red = reinterpret_cast<float*>(smem);
  u16* Us2 = reinterpret_cast<u16*>(smem + RED);
  char* As2 = smem + RED + BM * UP * 2;
#pragma unroll
  for (int fi = 0; fi < FI; ++fi)
#pragma unroll
    for (int q = 0; q < 8; ++q) red[((wave * FI + fi) * 8 + q) * 64 + lane] = dacc[fi][q];
  for (int q = tid; q < RP * (BN / 8); q += NT) {
    const int t = q / (BN / 8), c = q % (BN / 8);
    const int ll = l0 + 8 * c;
    *reinterpret_cast<int4v*>(As2 + mc32_offset<BN>(t, c)) =
        buf_load16(rsA, (t < r && ll < k) ? (uint32_t)t * wrow + (uint32_t)ll * 2 : kOOB);
  }
  __syncthreads();
  // entry e: lane ln of (token half wh, fragment fi), result row q: token
  // wh 64 + 32 fi + ln % 32, rank 8 (q / 4) + 4 (ln / 32) + q % 4
  for (int e = tid; e < WM * FI * 8 * 64; e += NT) {
    const int ln = e & 63, q = (e >> 6) & 7, fi = (e >> 9) & 1, wh = e >> 10;
    float v = 0.f;
#pragma unroll
    for (int w4 = 0; w4 < WN; ++w4) v += red[(((wh * WN + w4) * FI + fi) * 8 + q) * 64 + ln];
    const int i = wh * WTI + 32 * fi + (ln & 31);
    const int t = 8 * (q >> 2) + 4 * (ln >> 5) + (q & 3);
    const float d = s * v;
    const u16 hi = f32_to_bf16(d), lo = f32_to_bf16(d - bf16_to_f32(hi));
    Us2[i * UP + t] = hi;
    Us2[i * UP + RP + t] = lo;
    if (tn == 0 && m0 + i < mp) dUt2[(size_t)t * mp + m0 + i] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int fj = 0; fj < FJ; ++fj) {
    const short8 af = mc32_read_tr<BN>(As2, 0, wn * WTJ + 32 * fj, lane);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)   // k = t of [dU_hi | dU_lo] against [A; A]
#pragma unroll
      for (int fi = 0; fi < FI; ++fi) {
        const short8 bf = *reinterpret_cast<const short8*>(Us2 + (wm * WTI + 32 * fi + c32) * UP + 16 * kk + 8 * g);
        acc[fj][fi] = mfma32x32x16(af, bf, acc[fj][fi]);
      }
  }
  __syncthreads();
  {
    const int j0 = l0 + wn * WTJ;
#pragma unroll
    for (int fi = 0; fi < FI; ++fi) {
      const int i0 = m0 + wm * WTI + 32 * fi;
      store_block_32x64(acc[0][fi], acc[1][fi], smem + wave * kYsBytes, dX + (size_t)i0 * k + j0, (size_t)k,
                        m - i0, k - j0, lane);
    }
  }
}

// Fixed-order sum of the dA and dB partials as a launch of its own (the fused
// backward's token reduction runs after its dX launch).
__global__ __launch_bounds__(256) void lora_finalize_kernel(FinalizeArgs f) {
  finalize_partials(f, (int)(blockIdx.x * 256 + threadIdx.x), (int)(gridDim.x * 256));
}

// ---------------------------------------------------------------------------
// Launchers: execute the plans of lora_plan.hpp.

// Instantiations a plan can name: the 256 x 256 tile only with whole stages and
// without dropout, 128 x 192 for single projections.
template <int BM, int BN, int RP, bool DROP, bool GRP, bool FULL>
constexpr bool dx_instantiated() {
  return !(DROP && GRP) && (BM <= 128 || (FULL && !DROP)) && !(BN == 192 && GRP);
}

static hipError_t run_dx(const Launch& L, const BwdArgs& a, const u16* dU2, int mp, const FinalizeArgs& fin,
                         const DxGroup& grp, hipStream_t st) {
  const dim3 grid((unsigned)L.grid), block((unsigned)L.block);
  if (L.id == K_DX_ROWS) {
    return with_int<16, 32, 48, 64>(L.rp, [&](auto rc) {
      return with_bool(L.drop, [&](auto dr) {
        return with_bool(L.grp, [&](auto gr) {
          return with_bool(L.full, [&](auto fu) {
            constexpr int RP = decltype(rc)::value;
            constexpr bool DROP = decltype(dr)::value, GRP = decltype(gr)::value, FULL = decltype(fu)::value;
            if constexpr (DROP && GRP) {
              return hipErrorInvalidValue;
            } else {
              hipLaunchKernelGGL((lora_bwd_rows_dx_kernel<128, 256, 2, 4, RP, DROP, GRP, FULL>), grid, block, 0, st,
                                 a.dY, a.W, dU2, a.A, a.keep, a.dX, (int)a.m, (int)a.n, (int)a.k, (int)a.r, mp,
                                 a.inv_keep, L.tiles_m, L.tiles_n, (int)L.col_begin, L.finalize ? fin : FinalizeArgs{},
                                 grp);
              return hipGetLastError();
            }
          });
        });
      });
    });
  }
  return with_int<64, 65, 128, 192, 256, 257>(tile_code(L), [&](auto tc) {
    constexpr int T = decltype(tc)::value;
    constexpr int BM = T == 257 ? 256 : (T <= 65 ? 64 : 128), BN = T == 257 ? 256 : (T == 65 ? 128 : T);
    constexpr int WM = BM == 64 ? 1 : 2, WN = BN == 256 ? 4 : 2;
    return with_int<16, 32, 48, 64>(L.rp, [&](auto rc) {
      return with_bool(L.drop, [&](auto dr) {
        return with_bool(L.grp, [&](auto gr) {
          return with_bool(L.full, [&](auto fu) {
            constexpr int RP = decltype(rc)::value;
            constexpr bool DROP = decltype(dr)::value, GRP = decltype(gr)::value, FULL = decltype(fu)::value;
            if constexpr (!dx_instantiated<BM, BN, RP, DROP, GRP, FULL>()) {
              return hipErrorInvalidValue;
            } else {
              hipLaunchKernelGGL((lora_bwd_dx_kernel<BM, BN, WM, WN, RP, DROP, GRP, FULL>), grid, block, 0, st, a.dY,
                                 a.W, dU2, a.A, a.keep, a.dX, (int)a.m, (int)a.n, (int)a.k, (int)a.r, mp, a.inv_keep,
                                 L.tiles_m, L.tiles_n, (int)L.col_begin, L.finalize ? fin : FinalizeArgs{}, grp);
              return hipGetLastError();
            }
          });
        });
      });
    });
  });
}

// Projection a (workspace layout BL) as member g of a dU launch.  dUt2: where
// dU^T goes (the projection's own region, or its rows of a group's stacked
// region).
static void set_du(DuGroup& grp, int g, const BwdArgs& a, const BwdLayout& BL, u16* dUt2) {
  grp.dY[g] = a.dY;
  grp.B[g] = a.B;
  grp.U[g] = a.U;
  grp.dU2[g] = reinterpret_cast<u16*>(a.ws + BL.du2);
  grp.dUt2[g] = dUt2 ? dUt2 : reinterpret_cast<u16*>(a.ws + BL.dut2);
  grp.Ut2[g] = reinterpret_cast<u16*>(a.ws + BL.ut2);
  grp.n[g] = (int)a.n;
}

static hipError_t run_du(const Launch& L, const DuGroup& grp, int64_t m, int64_t r, int64_t mp, float s,
                         hipStream_t st) {
  return with_int<16, 32, 48, 64>(L.rp, [&](auto rc) {
    return with_int<8, 16, 32>(L.tpw, [&](auto tc) {
      constexpr int RP = decltype(rc)::value, TPW = decltype(tc)::value;
      if (L.fastb)
        hipLaunchKernelGGL((lora_bwd_du_dma_kernel<RP, TPW>), dim3((unsigned)L.grid), dim3((unsigned)L.block), 0, st,
                           grp, L.tiles_m, (int)m, (int)r, (int)mp, s);
      else
        hipLaunchKernelGGL((lora_bwd_du_kernel<RP, TPW>), dim3((unsigned)L.grid), dim3((unsigned)L.block), 0, st, grp,
                           L.tiles_m, (int)m, (int)r, (int)mp, s);
      return hipGetLastError();
    });
  });
}

// The two token reductions of one projection in one launch: dB^T partials =
// Ut2 . dY, then dA partials = dUt2 . X (masked X under dropout).
// L.part: 0 both reductions, 1 dB only (a group member whose dA is reduced
// with the group's), 2 the group's stacked dA (pap given by the caller).
static hipError_t run_tokred(const Launch& L, const BwdArgs& a, const BwdLayout& BL, hipStream_t st,
                             const RedProblem* stacked = nullptr) {
  const u16* Ut2 = reinterpret_cast<const u16*>(a.ws + BL.ut2);
  const u16* dUt2 = reinterpret_cast<const u16*>(a.ws + BL.dut2);
  float* pb = reinterpret_cast<float*>(a.ws + BL.pb);
  float* pa = reinterpret_cast<float*>(a.ws + BL.pa);
  const RedProblem pbp0{Ut2, a.dY, pb, (int)a.n, (int)BL.plan_b.span, BL.plan_b.col_tiles, nullptr};
  const RedProblem pap0{dUt2, a.X, pa, (int)a.k, (int)BL.plan_a.span, BL.plan_a.col_tiles, a.keep};
  const RedProblem pbp = L.part == 2 ? *stacked : pbp0;
  const RedProblem pap = L.part == 0 ? pap0 : pbp;
  const int nb0 = L.part == 0 ? BL.plan_b.col_tiles * BL.plan_b.splits : (int)L.grid;
  return with_int<16, 32, 48, 64>(L.rp, [&](auto rc) {
    constexpr int RP = decltype(rc)::value;
    if (L.drop)
      hipLaunchKernelGGL((lora_tokred_kernel<RP, true>), dim3((unsigned)L.grid), dim3((unsigned)L.block), 0, st, pbp,
                         pap, nb0, (int)a.m, (int)BL.mp);
    else
      hipLaunchKernelGGL((lora_tokred_dma_kernel<RP>), dim3((unsigned)L.grid), dim3((unsigned)L.block), 0, st, pbp,
                         pap, nb0, (int)a.m, (int)BL.mp);
    return hipGetLastError();
  });
}

static FinalizeArgs finalize_args(const BwdArgs& a, const BwdLayout& L) {
  return FinalizeArgs{reinterpret_cast<const float*>(a.ws + L.pb), reinterpret_cast<const float*>(a.ws + L.pa),
                      a.dB, a.dA, (int)a.n, (int)a.k, (int)a.r, L.rp, L.plan_b.splits, L.plan_a.splits, a.s,
                      a.keep ? a.inv_keep : 1.0f, L.rp};
}

hipError_t launch_bwd(const BwdArgs& a, hipStream_t st) {
  const BwdLayout BL = bwd_layout(a.m, a.n, a.k, a.r);
  const Plan p = plan_bwd(a.m, a.n, a.k, a.r, a.keep != nullptr);
  const FinalizeArgs fin = finalize_args(a, BL);
  const DxGroup none{};
  const u16* dU2 = reinterpret_cast<const u16*>(a.ws + BL.du2);
  for (int i = 0; i < p.count; ++i) {
    const Launch& L = p.l[i];
    hipError_t e = hipErrorInvalidValue;
    switch (L.id) {
      case K_DU: {
        DuGroup one{};
        set_du(one, 0, a, BL, nullptr);
        e = run_du(L, one, a.m, a.r, BL.mp, a.s, st);
        break;
      }
      case K_TOKRED: e = run_tokred(L, a, BL, st); break;
      case K_DX:
      case K_DX_ROWS: e = run_dx(L, a, dU2, (int)BL.mp, fin, none, st); break;
      default: break;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Fused backward: the dX launch (dU, the dB partials, dX), the dA token
// reduction, then the finalize of dA and dB.
hipError_t launch_bwd_fused(const BwdArgs& a, hipStream_t st) {
  const BwdFusedLayout BL = bwd_fused_layout(a.m, a.n, a.k, a.r);
  const Plan p = plan_bwd_fused(a.m, a.n, a.k, a.r);
  u16* dUt2 = reinterpret_cast<u16*>(a.ws + BL.dut2);
  float* pb = reinterpret_cast<float*>(a.ws + BL.pb);
  float* pa = reinterpret_cast<float*>(a.ws + BL.pa);
  const int m = (int)a.m, n = (int)a.n, k = (int)a.k, r = (int)a.r, mp = (int)BL.mp;
  for (int i = 0; i < p.count; ++i) {
    const Launch& L = p.l[i];
    const dim3 grid((unsigned)L.grid), block((unsigned)L.block);
    if (L.id == K_DXF) {
      const hipError_t e = with_bool(L.full, [&](auto fc) {
        return with_bool(L.fastb, [&](auto bc) {
          constexpr bool F = decltype(fc)::value, FB = decltype(bc)::value;
          if constexpr (F && !FB) {
            return hipErrorInvalidValue;
          } else {
            hipLaunchKernelGGL((lora_bwd_dxf_kernel<F, FB>), grid, block, 0, st, a.dY, a.W, a.A, a.B, a.U, a.dX, dUt2,
                               pb, m, n, k, r, mp, a.s, L.tiles_m, L.tiles_n);
            return hipGetLastError();
          }
        });
      });
      if (e != hipSuccess) return e;
    } else if (L.id == K_TOKRED) {
      const RedProblem pap{dUt2, a.X, pa, k, (int)BL.plan_a.span, BL.plan_a.col_tiles, nullptr};
      hipLaunchKernelGGL((lora_tokred_dma_kernel<16>), grid, block, 0, st, pap, pap, (int)L.grid, m, mp);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    } else if (L.id == K_FINALIZE) {
      const FinalizeArgs fin{pb, pa, a.dB, a.dA, n, k, r, 16, BL.tiles_m, BL.plan_a.splits, a.s, 1.0f, 16};
      hipLaunchKernelGGL(lora_finalize_kernel, grid, block, 0, st, fin);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    } else {
      return hipErrorInvalidValue;
    }
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Backward without a caller-provided workspace: the workspace regions live in
// a fixed device array of this library, one per GPU, whose address is looked
// up once per device (with that device current) on the first call there.
// Host code never passes the array's name itself to a kernel or a copy: in
// host code it stands for a host-side shadow, not the device address.
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_bwd_noalloc(const BwdArgs& a, hipStream_t st) {
  if (bwd_layout(a.m, a.n, a.k, a.r).total > kNoAllocScratchBytes) return hipErrorInvalidValue;
  void* ws = nullptr;
  const hipError_t e = noalloc_scratch(&ws);
  if (e != hipSuccess) return e;
  BwdArgs b = a;
  b.ws = static_cast<char*>(ws);
  return launch_bwd(b, st);
}

// Grouped backward: one dU launch for all projections, per projection the
// token reductions (each in its own workspace region), then one dX launch over the whole group whose
// tails (of the first column range) finalize every projection's dA and dB.
hipError_t launch_bwd_group(const GroupBwdArgs& a, hipStream_t st) {
  auto member_args = [&](int g, const GroupBwdLayout& GL) {
    BwdArgs b{};
    b.dY = a.dY[g]; b.X = a.X; b.W = a.W[g]; b.A = a.A[g]; b.B = a.B[g]; b.U = a.U[g];
    b.dX = a.dX; b.dA = a.dA[g]; b.dB = a.dB[g]; b.ws = a.ws + GL.off[g];
    b.m = a.m; b.n = a.n[g]; b.k = a.k; b.r = a.r; b.s = a.s;
    return b;
  };
  if (a.count == 1) {   // a group of one is the single projection (workspace sizes agree)
    BwdArgs b{};
    b.dY = a.dY[0]; b.X = a.X; b.W = a.W[0]; b.A = a.A[0]; b.B = a.B[0]; b.U = a.U[0];
    b.dX = a.dX; b.dA = a.dA[0]; b.dB = a.dB[0]; b.ws = a.ws;
    b.m = a.m; b.n = a.n[0]; b.k = a.k; b.r = a.r; b.s = a.s;
    return launch_bwd(b, st);
  }
  const GroupBwdLayout GL = group_bwd_layout(a.count, a.n, a.m, a.k, a.r);
  const Plan p = plan_group_bwd(a.count, a.n, a.m, a.k, a.r);
  const int rp = GL.L[0].rp;
  u16* dut_stack = GL.stacked ? reinterpret_cast<u16*>(a.ws + GL.dut_stack) : nullptr;
  float* pa_stack = GL.stacked ? reinterpret_cast<float*>(a.ws + GL.pa_stack) : nullptr;
  DxGroup grp{};
  int nkb = 0;
  for (int g = 0; g < a.count; ++g) {
    const BwdArgs b = member_args(g, GL);
    grp.dY[g] = a.dY[g];
    grp.W[g] = a.W[g];
    grp.dU2[g] = reinterpret_cast<const u16*>(b.ws + GL.L[g].du2);
    grp.A[g] = a.A[g];
    grp.n[g] = (int)a.n[g];
    nkb += (int)((a.n[g] + 63) / 64);
    grp.fin[g] = finalize_args(b, GL.L[g]);
    if (GL.stacked) {   // member g's dA rows of the stacked reduction
      grp.fin[g].pa = pa_stack + (size_t)g * rp * a.k;
      grp.fin[g].rpa = GL.rpt;
      grp.fin[g].sa = GL.plan_a.splits;
    }
  }
  grp.count = a.count;
  grp.nkb = nkb;
  DxGroup rest = grp;   // later column ranges finalize nothing
  for (int g = 0; g < kMaxGroup; ++g) rest.fin[g] = FinalizeArgs{};
  BwdArgs d{};
  d.X = a.X; d.dX = a.dX; d.ws = a.ws;
  d.m = a.m; d.n = 0; d.k = a.k; d.r = a.r; d.s = a.s;
  for (int i = 0; i < p.count; ++i) {
    const Launch& L = p.l[i];
    hipError_t e = hipErrorInvalidValue;
    if (L.id == K_TOKRED && L.part == 2) {   // the stacked dA reduction over X
      const RedProblem pap{dut_stack, a.X, pa_stack, (int)a.k, (int)GL.plan_a.span, GL.plan_a.col_tiles, nullptr};
      const BwdArgs b = member_args(0, GL);
      e = with_int<32, 48, 64>(L.rp, [&](auto rc) {
        hipLaunchKernelGGL((lora_tokred_dma_kernel<decltype(rc)::value>), dim3((unsigned)L.grid),
                           dim3((unsigned)L.block), 0, st, pap, pap, (int)L.grid, (int)b.m, (int)GL.L[0].mp);
        return hipGetLastError();
      });
    } else if (L.id == K_DU) {
      DuGroup dg{};
      for (int g = 0; g < a.count; ++g)
        set_du(dg, g, member_args(g, GL), GL.L[g], GL.stacked ? dut_stack + (size_t)g * rp * GL.L[0].mp : nullptr);
      e = run_du(L, dg, a.m, a.r, GL.L[0].mp, a.s, st);
    } else if (L.id == K_TOKRED) {
      const BwdArgs b = member_args(L.member, GL);
      e = run_tokred(L, b, GL.L[L.member], st);
    } else if (L.id == K_DX || L.id == K_DX_ROWS) {
      e = run_dx(L, d, nullptr, (int)GL.L[0].mp, FinalizeArgs{}, L.finalize ? grp : rest, st);
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lora
