// Forward for few tokens (generation with the adapter kept apart from W):
//   U = X A^T,   Y = X W^T + s U B^T   for calls fwd_skinny() admits.
#include <type_traits>

#include "lora_device.hpp"
#include "lora_launch.hpp"
#include "lora_plan.hpp"

namespace lora {

// Each workgroup owns F output features of a block of up to XR tokens (all
// tokens up to 64 of them), so the call streams W once and is bound by the
// bytes of W in flight; the plan picks the F that spreads the columns over
// one round of workgroups.  (Measured with weights rotated past the caches,
// against the 128 x 128 tile, which leaves most compute units idle here:
// 4 tokens, n = k = 4096, r = 8: 39 -> 10.5 us, 3.2 TB/s of W; 24 tokens,
// n = 11008, k = 4096, r = 16: 23 us, 3.9 TB/s; 64 tokens, n = k = 4096,
// r = 16: 40 -> 18 us.  Stages twice as deep in k or two workgroups per
// compute unit with half the ring each: within 5%.)
// k runs in stages of 64 KQ; a stage holds, for each of its KQ 64-wide k
// pieces, the F rows of W, XR rows of X and (without UPRE) AR rows of A as
// 128-byte rows (kc_offset swizzle), copied straight into a ring of NS LDS
// stages, NS - 1 stages ahead, one barrier per stage.  The eight waves are
// KQ k pieces x RW row shares: wave (q, rw) multiplies the 16-row groups
// rw, rw + RW, ... of W and A with all tokens over piece q on 16x16x32
// products.  After the loop the KQ partial sums go through LDS, are added in
// piece order, and s U B^T is added in fp32 before Y is rounded.  Every
// workgroup forms U itself (A comes from L2); the first one of a projection
// writes it.  With UPRE (rank above 16, or LoRA dropout) U comes from
// lora_u_kernel.
//
// Rows of a region beyond its matrix (tokens past m, ranks past r, features
// past n) are copied as zeros.
template <int XR, int F, int AR, bool UPRE>
__global__ __launch_bounds__(512) void lora_fwd_skinny_ks_kernel(const u16* __restrict__ X, int mtot, int k, int r,
                                                                 float s, int tiles_n, FwdGroup grp) {
  static_assert(UPRE == (AR == 0), "A rows are staged unless U comes from its own pass");
  constexpr int NT = 512, NW = 8;
  constexpr int FG = F / 16;
  constexpr int KQ = FG == 1 ? 4 : 2, RW = NW / KQ;
  constexpr int TG = XR / 16, UG = AR / 16, RG = FG + UG;
  constexpr int GPW = (RG + RW - 1) / RW;          // row groups per wave
  constexpr int ROWS = F + XR + AR;
  constexpr int PIECE = ROWS * 128, STAGE = KQ * PIECE;
  constexpr int RB = ROWS / 8;                     // 1 KB copies per k piece
  constexpr int NC = KQ * RB;                      // copies per stage
  constexpr int CPW = (NC + NW - 1) / NW;
  constexpr int NSMAX = (152 * 1024) / STAGE;
  constexpr int NS = NSMAX < 8 ? NSMAX : 8;
  constexpr int TP = 16 * TG + 1;                  // padded token pitch of the partial sums
  constexpr int PR = F + (UPRE ? 64 : 16 * UG);   // rows of one k piece's partial sums (then U)
  constexpr int PART = KQ * PR * TP * 4;
  constexpr int RMAX = UPRE ? 64 : 16;
  constexpr int BCH = (F * RMAX / 8 + NT - 1) / NT;
  constexpr int UPT = UPRE ? (16 * TG * RMAX + NT - 1) / NT : 1;
  constexpr bool BT = UPRE || XR > 16;             // B^T in LDS (below, B as it lies in memory is 0.1 us faster)
  constexpr int BP = F + 2;                        // its row pitch: a rank's features contiguous
  constexpr int EPI = PART + RMAX * BP * 2;
  constexpr int SMEM = NS * STAGE > EPI ? NS * STAGE : EPI;
  static_assert(NS >= 3 && CPW * (NS - 2) < 64, "copies in flight fit the wait counter");
  static_assert(SMEM <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];

  const int tb = (int)blockIdx.x / tiles_n;        // token block
  int tn = (int)blockIdx.x - tb * tiles_n, sel = 0;
  X += (size_t)tb * XR * k;
  const int m = min(XR, mtot - tb * XR);
#pragma unroll
  for (int q = 1; q < kMaxGroup; ++q)
    if (q < grp.count && tn >= grp.tile0[q]) sel = q;
  const u16 *W = grp.W[0], *A = grp.A[0], *B = grp.B[0];
  u16* Y = grp.Y[0];
  float* U = grp.U[0];
  int n = grp.n[0], t0 = grp.tile0[0];
#pragma unroll
  for (int q = 1; q < kMaxGroup; ++q)
    if (q == sel) {
      W = grp.W[q]; A = grp.A[q]; B = grp.B[q]; Y = grp.Y[q]; U = grp.U[q];
      n = grp.n[q]; t0 = grp.tile0[q];
    }
  tn -= t0;
  Y += (size_t)tb * XR * n;
  U += (size_t)tb * XR * r;
  const int n0 = tn * F;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const int kq = wave / RW, rw = wave % RW;
  const uint32_t rowbytes = (uint32_t)k * 2;
  const int jn = min(F, n - n0);
  const u16* Wt = W + (size_t)n0 * k;

  // Copy c = wave + 8 i of a stage fills 8 rows of k piece c / RB: row block
  // c % RB (W rows, then X, then A); lane l takes row l / 8 of the eight at
  // chunk position l % 8, which holds logical chunk (l % 8) ^ kc_swz(row).
  uint32_t voff[CPW];
  int kcol[CPW];
#pragma unroll
  for (int i = 0; i < CPW; ++i) {
    const int c = wave + NW * i, rb = c % RB;
    const int row = 8 * rb + (lane >> 3);
    const int grow = row < F ? row : (row < F + XR ? row - F : row - F - XR);
    kcol[i] = 64 * (c / RB) + 8 * ((lane & 7) ^ kc_swz(row));
    voff[i] = (uint32_t)grow * rowbytes + (uint32_t)kcol[i] * 2;
  }
  const int nst = (k + 64 * KQ - 1) / (64 * KQ);
  auto issue = [&](int st, int buf) LORA_INLINE {
    const int k0 = st * 64 * KQ;
    char* sb = smem + buf * STAGE;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const int c = wave + NW * i, rb = c % RB;
      if (NC % NW != 0 && c >= NC) break;          // wave-uniform
      // (base and row count selected by masks: from conditional expressions
      // the compiler selects the address of the captured variable, loads it
      // from memory and loops over the lanes)
      const uint64_t isw = 0 - (uint64_t)(8 * rb < F), isx = 0 - (uint64_t)(8 * rb < F + XR);
      const uint64_t base = (isw & (uint64_t)Wt) | (~isw & ((isx & (uint64_t)X) | (~isx & (uint64_t)A)));
      const int rows = ((int)isw & jn) | (~(int)isw & (((int)isx & m) | (~(int)isx & r)));
      const __amdgpu_buffer_rsrc_t rs = make_rsrc((const void*)base, (uint64_t)rows * rowbytes);
      dma16(rs, k0 + kcol[i] < k ? voff[i] + (uint32_t)k0 * 2 : kOOB, 0, sb + c * 1024);
    }
  };

#pragma unroll
  for (int st = 0; st < NS - 1; ++st) issue(st, st);

  floatx4 acc[GPW][TG];
#pragma unroll
  for (int a = 0; a < GPW; ++a)
#pragma unroll
    for (int b = 0; b < TG; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) LORA_INLINE {
    const char* sb = smem + buf * STAGE + kq * PIECE;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int ch = 4 * kk + g;
      short8 xf[TG];
#pragma unroll
      for (int tg = 0; tg < TG; ++tg) xf[tg] = kc_read(sb, F + 16 * tg + c16, ch);
#pragma unroll
      for (int a = 0; a < GPW; ++a) {
        const int rg = rw + RW * a;                // past the last group: group 0, not stored
        const int row = rg < FG ? 16 * rg + c16 : F + XR + 16 * (rg - FG) + c16;
        const short8 wf = kc_read(sb, rg < RG ? row : c16, ch);
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) acc[a][tg] = mfma16x16x32(wf, xf[tg], acc[a][tg]);
      }
    }
  };
  auto stage_barrier = [&]() LORA_INLINE {
    if (NC % NW != 0 && wave >= NC % NW) copy_barrier<(NS - 2) * (NC / NW)>();
    else copy_barrier<(NS - 2) * CPW>();
  };
  int buf = 0, nbuf = NS - 1;
  for (int st = 0; st < nst; ++st) {
    stage_barrier();   // stage st has landed; every wave is done with stage st - 1
    issue(st + NS - 1, nbuf);
    compute(buf);
    buf = buf + 1 == NS ? 0 : buf + 1;
    nbuf = nbuf + 1 == NS ? 0 : nbuf + 1;
  }

  // B rows n0 .. n0 + jn - 1 (contiguous) and, with UPRE, U: all loads issued together
  const int nch = jn * r / 8;                      // exact: n and n0 are multiples of 8
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B + (size_t)n0 * r, (uint64_t)nch * 16);
  int4v bv[BCH];
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int q = tid + i * NT;
    bv[i] = buf_load16(rsB, q < nch ? (uint32_t)q * 16 : kOOB);
  }
  float uv[UPT];
  if (UPRE) {
    const __amdgpu_buffer_rsrc_t rsU = make_rsrc(U, (uint64_t)m * r * 4);
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
      const int e = tid + i * NT;
      uv[i] = buf_load4f(rsU, e < m * r ? (uint32_t)e * 4 : kOOB);
    }
  }
  copy_barrier<0>();   // the trailing copies (zeros) have landed before the LDS is reused
  float* part = reinterpret_cast<float*>(smem);    // [KQ][PR][TP]
  u16* Bt = reinterpret_cast<u16*>(smem + PART);   // B^T of the workgroup's features [r][BP], or B [jn][r]
#pragma unroll
  for (int a = 0; a < GPW; ++a) {
    const int rg = rw + RW * a;
    if (rg < RG) {
#pragma unroll
      for (int tg = 0; tg < TG; ++tg)
#pragma unroll
        for (int j = 0; j < 4; ++j) part[(kq * PR + 16 * rg + 4 * g + j) * TP + 16 * tg + c16] = acc[a][tg][j];
    }
  }
  // element 8 q of chunk q is B row 8 q / r, column 8 q % r; the quotient comes
  // from a float product that stays at least 0.5/r away from an integer
  const float rinv = 1.0f / (float)r;
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const int q = tid + i * NT;
    if (q < nch && !BT) reinterpret_cast<int4v*>(Bt)[q] = bv[i];
    if (q < nch && BT) {
      const int f0 = (int)(((float)(8 * q) + 0.5f) * rinv);
      int f = f0, t = 8 * q - f0 * r;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        Bt[t * BP + f] = (u16)((uint32_t)bv[i][e >> 1] >> (16 * (e & 1)));
        if (++t == r) { t = 0; ++f; }
      }
    }
  }
  if (UPRE) {
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
      const int e = tid + i * NT;
      if (e < m * r) part[(F + e % r) * TP + e / r] = uv[i];
    }
  }
  __syncthreads();
  if (!UPRE) {   // U: the partial sums in piece order
    for (int e = tid; e < m * r; e += NT) {
      const int i = e / r, t = e - i * r;
      float v = part[(F + t) * TP + i];
#pragma unroll
      for (int q = 1; q < KQ; ++q) v += part[(q * PR + F + t) * TP + i];
      part[(F + t) * TP + i] = v;
      if (tn == 0) U[e] = v;
    }
    __syncthreads();
  }
  // Two features of TT tokens (i, i + XR / TT, ...) per thread, as many tokens as
  // leave every thread work: per rank one read of B^T, contiguous over the lanes,
  // and TT of U, shared by the lanes of a token.  (One token per thread with B as
  // [feature][rank] read each value of B in as many LDS passes as lanes hit its
  // bank, 32 at rank 64: 2 x 13824 x 64 x 1024, r = 64, 99 us against 33.)
  constexpr int TW = XR * (F / 2) / NT;
  constexpr int TT = TW >= 4 ? 4 : (TW >= 2 ? 2 : 1), TI = XR / TT;
  for (int e = tid; e < TI * (F / 2); e += NT) {
    const int i = e / (F / 2), f = 2 * (e - i * (F / 2));
    if (f >= jn || i >= m) continue;
    float y[TT][2], d[TT][2];
#pragma unroll
    for (int x = 0; x < TT; ++x) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        y[x][h] = part[(f + h) * TP + i + TI * x];
#pragma unroll
        for (int q = 1; q < KQ; ++q) y[x][h] += part[(q * PR + f + h) * TP + i + TI * x];
        d[x][h] = 0.f;
      }
    }
    for (int t = 0; t < r; ++t) {
      const uint32_t b2 = BT ? *reinterpret_cast<const uint32_t*>(Bt + t * BP + f)
                             : (uint32_t)Bt[f * r + t] | ((uint32_t)Bt[(f + 1) * r + t] << 16);
      const float b0 = bf16_to_f32((u16)b2), b1 = bf16_to_f32((u16)(b2 >> 16));
#pragma unroll
      for (int x = 0; x < TT; ++x) {
        const float u = part[(F + t) * TP + i + TI * x];
        d[x][0] += u * b0;
        d[x][1] += u * b1;
      }
    }
#pragma unroll
    for (int x = 0; x < TT; ++x)
      if (i + TI * x < m)
        *reinterpret_cast<uint32_t*>(Y + (size_t)(i + TI * x) * n + n0 + f) =
            (uint32_t)f32_to_bf16(y[x][0] + s * d[x][0]) | ((uint32_t)f32_to_bf16(y[x][1] + s * d[x][1]) << 16);
  }
}

hipError_t launch_fwd_skinny(const Launch& L, const FwdArgs& a, const FwdGroup& grp, hipStream_t st) {
  return with_int<16, 32, 48, 64, 96>(L.bn, [&](auto fc) {
    return with_int<16, 32, 64>(L.bm, [&](auto xc) {
      return with_bool(L.upre, [&](auto uc) {
        constexpr int F = decltype(fc)::value, XR = decltype(xc)::value;
        constexpr bool UP = decltype(uc)::value;
        hipLaunchKernelGGL((lora_fwd_skinny_ks_kernel<XR, F, UP ? 0 : 16, UP>), dim3((unsigned)L.grid),
                           dim3((unsigned)L.block), 0, st, a.X, (int)a.m, (int)a.k, (int)a.r, a.s, L.tiles_n, grp);
        return hipGetLastError();
      });
    });
  });
}

}  // namespace lora
