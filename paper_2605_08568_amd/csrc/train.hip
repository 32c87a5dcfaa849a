// Router training step (Sec. 4.2, "Calibration-Decoupled Router Training"): the low-rank factors stay fixed, the
// router matrix is trained against the dense model's output with the reconstruction loss of Eq. 6; the forward
// pass uses the hard top-k mask (Eq. 7), the backward pass the K-normalised sigmoid mask (Eq. 8-9, straight
// through).  This file computes loss and gradient for one batch of prompts, groups as experts, one embedding per
// prompt, given the routed output Y_hat (parse_lowrank_forward) and the dense output Y_dense:
//   residual       g = 2 (y_hat - y_dense) per token (bf16), squared-error sum per token row
//   pair           Z = X V^T and Tm = g U over ALL stored ranks, multiplied in registers, summed over 8 ranks
//   mask_grad      dL/dm[p][group] = sum over the prompt's tokens and the group's ranks of Z * Tm
//   router_grad    dL/ds_j = k a'_j (dL/dm_j / A - B / A^2) with a = sigmoid(s / tau), a' = a (1 - a) / tau,
//                  A = sum a + eps, B = sum_g dL/dm_g a_g  (the Jacobian of Eq. 9 applied in closed form), then
//                  dL/dWr[j][:] = sum_p dL/ds_j(p) e_p, prompts added in order.
// No atomics: same inputs, same bits.
#include "prefill_common.hpp"

namespace parse {

#define PARSE_TR_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
#define PARSE_TR_GLB_PTR(p) ((const __attribute__((address_space(1))) void *)(p))

struct TrainPair {
  const uint16_t *X, *V, *g, *U;   // [rows][n] and the R x n factor in operand order; [rows][m] and the R x m factor
  float *W;                        // [R/8][rows]
  int rows, n, m, R;
};

// grid rows, block 256.
__global__ __launch_bounds__(256) void train_residual(const uint16_t *__restrict__ Yh, const uint16_t *__restrict__ Yd,
                                                      int rows, int m, uint16_t *__restrict__ g,
                                                      float *__restrict__ rowloss) {
  __shared__ float red[256];
  const int t = blockIdx.x;
  float acc = 0.f;
  for (int c = threadIdx.x * 8; c < m; c += 256 * 8) {
    const u32x4 a = *reinterpret_cast<const u32x4 *>(Yh + (size_t)t * m + c);
    const u32x4 b = *reinterpret_cast<const u32x4 *>(Yd + (size_t)t * m + c);
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float d0 = __uint_as_float(a[i] << 16) - __uint_as_float(b[i] << 16);
      const float d1 = __uint_as_float(a[i] & 0xFFFF0000u) - __uint_as_float(b[i] & 0xFFFF0000u);
      acc += d0 * d0 + d1 * d1;
      w[i] = pack_bf16x2(2.f * d0, 2.f * d1);
    }
    *reinterpret_cast<u32x4 *>(g + (size_t)t * m + c) = w;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) rowloss[t] = red[0];
}

// ---------------------------------------------------------------------------------------------------------
// train_pair.  The gradient needs, per (prompt, group), the sum of Z * Tm over the group's ranks and the prompt's tokens,
// with Z = X V^T and Tm = g U over ALL stored ranks; neither product is needed by itself.  A workgroup computes the SAME
// tile (BM tokens x BN ranks) of both, one after the other through one pipeline, multiplies the two accumulators in
// registers and writes only the fp32 sums over 8 consecutive ranks, W[R/8][rows]: the two intermediates (2 x rows x R)
// never exist, are not rounded, and are not read back.
// Bound by power, the issue of loads and the matrix cores, and built like the tile kernel of the prefill (prefill_lds_bf16.hip):
// both operands staged in LDS by loads that write LDS directly (factors in operand order, 1 KiB per instruction; token rows
// row-major with their 16-byte chunks XOR-swizzled on the way in), STAGES slices of 64 in rotation, the loads spread between
// 16x16x32 products, one barrier per slice, no branches in the steady part but the one where the second product's operands begin.
// The slices of the second product follow those of the first in the same ring: nothing drains between the two.
// Measured at 4096 rows, n = m = 4096, R = 2048: the two separate products and the pass over their outputs took 90 + 90 +
// 19 us; this kernel 109-125 us (137 GFLOP), 139-156 with 32x32x16 products and the loads of a slice in a row.
template <int BM, int BN, int WM, int WN, int STAGES>
__global__ __launch_bounds__(WM * WN * 64, 2) void train_pair(TrainPair a) {
  constexpr int NW = WM * WN;
  constexpr int FB = BN / WN / 16, TB = BM / WM / 16;          // 16-row blocks of a wavefront
  constexpr int F_BYTES = BN * 128, T_BYTES = BM * 128, STAGE_BYTES = F_BYTES + T_BYTES;
  constexpr int NI_F = F_BYTES / 1024, NI_T = T_BYTES / 1024;
  static_assert(NI_F % NW == 0 && NI_T % NW == 0, "the loads of a slice divide evenly over the wavefronts");
  constexpr int LF = NI_F / NW, LT = NI_T / NW, L = LF + LT, LU = L / 2;
  static_assert(L % 2 == 0 && (STAGES - 2) * L + LU < 64, "and over the two halves; vmcnt is a 6-bit count");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int j = lane & 15, g = lane >> 4;
  // up to 8 token tiles run through a rank tile before the next one: a die's consecutive tiles share both operands in its L2
  const int ntm = (a.rows + BM - 1) / BM, ntn = (a.R + BN - 1) / BN;
  const int tile = xcd_tile(blockIdx.x, ((a.rows + BM - 1) / BM) * ((a.R + BN - 1) / BN));
  const int grp = tile / (8 * ntn), first = grp * 8, gm = min(8, ntm - first), r = tile - grp * 8 * ntn;
  const int tm = first + r % gm, tn = r / gm;
  const int nblk = a.R / 32;

  // sources of this wavefront's load instructions in the two products
  const uint32_t loff = lane * 16;
  const char *fsrc[LF], *tsrc[LT];
  auto aim = [&](const uint16_t *F, const uint16_t *T, int K) {
#pragma unroll
    for (int i = 0; i < LF; ++i) {
      const int ins = wave * LF + i, fb = ins / 4, kk = ins % 4;
      const int gb = min(tn * (BN / 32) + fb, nblk - 1);       // blocks past the end re-read the last one (never stored)
      fsrc[i] = (const char *)F + ((size_t)gb * (K / 16) + kk) * 1024;
    }
#pragma unroll
    for (int i = 0; i < LT; ++i) {                             // LDS place: row rr, slot lane % 8; it holds chunk slot ^ swizzle of the row
      const int rr = (wave * LT + i) * 8 + (lane >> 3);
      const size_t row = min(tm * BM + rr, a.rows - 1);        // rows past the end re-read the last one (never stored)
      tsrc[i] = (const char *)T + row * K * 2 + ((lane & 7) ^ ((rr >> 1) & 7)) * 16;
    }
  };
  aim(a.V, a.X, a.n);
  const int nk1 = a.n / 64, nk = nk1 + a.m / 64;
  int issued = 0, dst = 0;
  auto load = [&](int q) {                                     // load q of L of the next slice; the last one moves on
    if (q < LF) {
      __builtin_amdgcn_global_load_lds(PARSE_TR_GLB_PTR(fsrc[q] + loff), PARSE_TR_LDS_PTR(smem + dst + (wave * LF + q) * 1024), 16, 0, 0);
      fsrc[q] += 4096;
    } else {
      __builtin_amdgcn_global_load_lds(PARSE_TR_GLB_PTR(tsrc[q - LF]), PARSE_TR_LDS_PTR(smem + dst + F_BYTES + (wave * LT + q - LF) * 1024), 16, 0, 0);
      tsrc[q - LF] += 128;
    }
    if (q == L - 1) {
      dst = dst + STAGE_BYTES == STAGES * STAGE_BYTES ? 0 : dst + STAGE_BYTES;
      if (++issued == nk1) aim(a.U, a.g, a.m);                 // uniform: on to the operands of the second product
    }
  };
  // LDS operands: lane (j, g) reads reduction indices 8 g .. 8 g + 7 of row j of a 16-row block
  const int f_lane = wn * (FB / 2) * 4096 + (g >> 1) * 1024 + (g & 1) * 512 + j * 16;
  const int t_lane = F_BYTES + wm * TB * 2048 + j * 128 + (g ^ ((j >> 1) & 7)) * 16;
  u32x4 fr[2][FB], tr[2][TB];
  int src = 0;
  auto read_half = [&](int half) {
    const char *fb = smem + src + f_lane + half * 2048, *tb = smem + src + (t_lane ^ (half * 64));
#pragma unroll
    for (int i = 0; i < FB; ++i) fr[half][i] = *reinterpret_cast<const u32x4 *>(fb + (i >> 1) * 4096 + (i & 1) * 256);
#pragma unroll
    for (int t = 0; t < TB; ++t) tr[half][t] = *reinterpret_cast<const u32x4 *>(tb + t * 2048);
  };
  // this half's operands are touched before the next half's LDS reads are issued: the wait the compiler places there then
  // covers reads that had a whole half to finish
  auto settle = [&](int half) {
#pragma unroll
    for (int i = 0; i < FB; ++i) asm volatile("" ::"v"(fr[half][i]));
#pragma unroll
    for (int t = 0; t < TB; ++t) asm volatile("" ::"v"(tr[half][t]));
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x4v accz[FB][TB], acct[FB][TB];
#pragma unroll
  for (int i = 0; i < FB; ++i)
#pragma unroll
    for (int t = 0; t < TB; ++t) accz[i][t] = acct[i][t] = f32x4v{0.f, 0.f, 0.f, 0.f};
  auto products = [&](f32x4v(&acc)[FB][TB], int half, int q0, bool more) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fr[half][i]), as_bf16x8(tr[half][t]), acc[i][t], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < LU; ++q)
          if (i * TB + t == (2 * q + 1) * FB * TB / (2 * LU)) {
            __builtin_amdgcn_sched_barrier(0);
            if (more) load(q0 + q);
            __builtin_amdgcn_sched_barrier(0);
          }
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // slice kt + STAGES is requested from the second half of slice kt on, whose start has the barrier that says that everybody has read
  // slice kt and that slice kt + 1 has landed
  auto slice = [&](f32x4v(&acc)[FB][TB], bool steady, int kt) {
    settle(0);
    read_half(1);
    products(acc, 0, LU, steady || kt - 1 + STAGES < nk);
    settle(1);
    if (steady || kt + 1 < nk) {
      if (steady) wait_vm<(STAGES - 2) * L>(); else wait_slices<STAGES - 2, L>(min(kt + STAGES - 1, nk - 1) - (kt + 1));
      wg_barrier();
      src = src + STAGE_BYTES == STAGES * STAGE_BYTES ? 0 : src + STAGE_BYTES;
      read_half(0);
    }
    products(acc, 1, 0, steady || kt + STAGES < nk);
  };
#pragma unroll
  for (int s = 0; s < STAGES; ++s) {
    if (s < nk) {
#pragma unroll
      for (int q = 0; q < (s == STAGES - 1 ? LU : L); ++q) load(q);
    }
  }
  if (nk >= STAGES) wait_vm<(STAGES - 2) * L + LU>(); else wait_vm<0>();
  wg_barrier();
  read_half(0);
  int kt = 0;
  for (; kt < nk1 && kt + STAGES < nk; ++kt) slice(accz, true, kt);
  for (; kt < nk1; ++kt) slice(accz, false, kt);
  for (; kt + STAGES < nk; ++kt) slice(acct, true, kt);
  for (; kt < nk; ++kt) slice(acct, false, kt);
  // lane (j, g) of acc[i][t] holds ranks 16 i + 4 g + (0..3) of token 16 t + j of both products; one 16-lane swap of two token blocks
  // brings the sums over 4 ranks together: groups 0 / 2 get ranks 0..7 / 8..15 of the first block, 1 / 3 of the second
#pragma unroll
  for (int i = 0; i < FB; ++i) {
    const int b16 = (tn * BN + wn * FB * 16) / 16 + i;
#pragma unroll
    for (int t = 0; t < TB; t += 2) {
      float s[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        s[u] = accz[i][t + u][0] * acct[i][t + u][0];
#pragma unroll
        for (int e = 1; e < 4; ++e) s[u] += accz[i][t + u][e] * acct[i][t + u][e];
      }
      const u32x2 sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[0]), __float_as_uint(s[1]), false, false);
      const int row = tm * BM + (wm * TB + t + (g & 1)) * 16 + j;
      if (b16 < nblk * 2 && row < a.rows) a.W[(size_t)(b16 * 2 + (g >> 1)) * a.rows + row] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
  }
}

template <int BM, int BN, int WM, int WN, int STAGES>
static int launch_train_pair(const TrainPair &a, hipStream_t s) {
  constexpr size_t smem = (size_t)STAGES * (BM + BN) * 128;
  auto kern = train_pair<BM, BN, WM, WN, STAGES>;
  PARSE_ALLOW_LDS(kern, 0, smem);
  const int grid = ((a.rows + BM - 1) / BM) * ((a.R + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WM * WN * 64), smem, s, a);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

// Tile by how many workgroups it gives a launch.  256 x 128 moves the fewest bytes per flop and wins once it fills the chip; below
// that the tile that still fills it wins, and 64 x 64 when none does
// (whole call, us, 256 x 128 / 128 x 128 / 64 x 64: 4096 rows x 2048 ranks 134 / 155 / 206; 3300 x 1024 113 / 83 / 119;
// 4000 x 768 117 / 86 / 101; 1800 x 2048 109 / 81 / 114; 1024 x 2048 99 / 69 / 64; 16 x 1024 87 / 56 / 32).
static int forward_train_pair(const TrainPair &a, hipStream_t s) {
  auto wgs = [&](int bm, int bn) { return (long long)((a.rows + bm - 1) / bm) * ((a.R + bn - 1) / bn); };
  if (wgs(256, 128) >= 192) return launch_train_pair<256, 128, 4, 2, 3>(a, s);
  if (wgs(128, 128) >= 160) return launch_train_pair<128, 128, 2, 4, 4>(a, s);
  return launch_train_pair<64, 64, 2, 2, 4>(a, s);
}

// Adds W over the group's pieces of 8 ranks and the prompt's tokens.  grid (G + 1, P), block 256; the last column of
// workgroups adds up the per-prompt losses instead.
__global__ __launch_bounds__(256) void train_mask_grad(const float *__restrict__ W, int rows, int gs,
                                                       const int32_t *__restrict__ tok_offsets, const float *__restrict__ rowloss,
                                                       float *__restrict__ dm, float *__restrict__ loss_out, int G) {
  __shared__ float red[256];
  const int g = blockIdx.x, p = blockIdx.y;
  int a = tok_offsets[p], b = tok_offsets[p + 1];
  a = a < 0 ? 0 : (a > rows ? rows : a);
  b = b < a ? a : (b > rows ? rows : b);
  float acc = 0.f;
  if (g < G) {
    const float *src = W + (size_t)g * (gs / 8) * rows;
    for (int t = a + (int)threadIdx.x; t < b; t += 256) {
#pragma unroll 8
      for (int i = 0; i < gs / 8; ++i) acc += src[(size_t)i * rows + t];
    }
  } else {
    for (int t = a + (int)threadIdx.x; t < b; t += 256) acc += rowloss[t];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (g < G) dm[(size_t)p * G + g] = red[0];
    else loss_out[p] = red[0];
  }
}

constexpr int TR_MAX_PG = 8192;   // P * G entries of dL/ds a workgroup keeps in LDS
constexpr int TR_GJ = 4;          // router rows per workgroup

// grid (ceil(d / 256), ceil(G / TR_GJ)), block 256.  Every workgroup first works out dL/ds[p][j] of its TR_GJ groups for
// the whole batch (LDS; 64 / width prompts per wavefront at a time, width = G rounded up to a power of two, one lane per
// group), then its 256 columns of its rows of the gradient, prompts added in order.
__global__ __launch_bounds__(256) void train_router_grad(const float *__restrict__ dm, const float *__restrict__ scores,
                                                         const float *__restrict__ emb, int P, int G, int d, int k,
                                                         float inv_tau, float eps, int width, float *__restrict__ grad) {
  __shared__ float ds[TR_MAX_PG];          // [p][TR_GJ]
  const int j0 = blockIdx.y * TR_GJ, nj = min(TR_GJ, G - j0);
  const int per = 256 / width, sub = threadIdx.x % width;      // prompts per round, this lane's group
  for (int p0 = 0; p0 < P; p0 += per) {
    const int p = p0 + (int)threadIdx.x / width;
    const bool on = p < P && sub < G;
    const float sg = on ? 1.f / (1.f + expf(-scores[(size_t)p * G + sub] * inv_tau)) : 0.f;
    const float dv = on ? dm[(size_t)p * G + sub] : 0.f;
    float A = sg, B = on ? dv * sg : 0.f;
    for (int o = width >> 1; o > 0; o >>= 1) { A += __shfl_xor(A, o, 64); B += __shfl_xor(B, o, 64); }
    A += eps;
    if (on && sub >= j0 && sub < j0 + nj) ds[p * nj + sub - j0] = (float)k * (sg * (1.f - sg) * inv_tau) * (dv / A - B / (A * A));
  }
  __syncthreads();
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d) return;
  float acc[TR_GJ];
#pragma unroll
  for (int j = 0; j < TR_GJ; ++j) acc[j] = 0.f;
#pragma unroll 8
  for (int p = 0; p < P; ++p) {
    const float e = emb[(size_t)p * d + c];
#pragma unroll
    for (int j = 0; j < TR_GJ; ++j) acc[j] += ds[p * nj + min(j, nj - 1)] * e;
  }
#pragma unroll
  for (int j = 0; j < TR_GJ; ++j)
    if (j < nj) grad[(size_t)(j0 + j) * d + c] = acc[j];
}

}  // namespace parse

using namespace parse;

extern "C" {

size_t parse_router_grad_workspace_bytes(const parse_layer *L, int32_t rows, int32_t P) {
  if (!L || rows <= 0 || P <= 0 || L->R <= 0 || L->G <= 0 || L->m <= 0) return 0;
  // (the middle term is room for two bf16 products over all ranks, which callers' sizes count on; their reduced product, the fp32
  // sums over 8 ranks, takes an eighth of it)
  return round_up((size_t)rows * L->m * 2, 256) + 2 * round_up((size_t)rows * L->R * 2, 256) +
         round_up((size_t)rows * sizeof(float), 256) + round_up((size_t)P * L->G * sizeof(float), 256) + 256;
}

int parse_router_grad(const parse_layer *L, const void *Ut_rankmajor, const void *X, int32_t rows,
                      const int32_t *tok_offsets, int32_t P, const void *Y_hat, const void *Y_dense,
                      const float *emb, const float *scores, int32_t d, int32_t k, float temperature, float eps,
                      float *loss_out, float *grad_Wr, void *workspace, size_t workspace_bytes,
                      parse_stream stream) {
  int st = check_layer(L);
  if (st != PARSE_OK) return st;
  if (!Ut_rankmajor || !X || !tok_offsets || !Y_hat || !Y_dense || !emb || !scores || !grad_Wr) return PARSE_EINVAL;
  if (rows <= 0 || P <= 0 || d <= 0 || k <= 0 || !(temperature > 0.f) || eps < 0.f) return PARSE_EINVAL;
  if (L->dtype != PARSE_BF16 || L->layout != PARSE_MFMA16) return PARSE_ELAYOUT;
  const int gs = L->R / L->G;
  if (k > L->G || L->G > 64 || P > rows || (long long)P * L->G > TR_MAX_PG) return PARSE_ESHAPE;
  if (L->n % 128 != 0 || L->m % 128 != 0 || L->R % 32 != 0 || gs % 8 != 0) return PARSE_ESHAPE;
  if (!aligned16(Ut_rankmajor) || !aligned16(X) || !aligned16(Y_hat) || !aligned16(Y_dense) || !aligned16(emb))
    return PARSE_EALIGN;
  if (!workspace || workspace_bytes < parse_router_grad_workspace_bytes(L, rows, P)) return PARSE_EWORKSPACE;
  if (!aligned16(workspace)) return PARSE_EALIGN;
  hipStream_t s = (hipStream_t)stream;
  char *ws = reinterpret_cast<char *>(workspace);
  uint16_t *g = reinterpret_cast<uint16_t *>(ws);            ws += round_up((size_t)rows * L->m * 2, 256);
  float *W = reinterpret_cast<float *>(ws);                  ws += round_up((size_t)rows * (L->R / 8) * sizeof(float), 256);
  float *rowloss = reinterpret_cast<float *>(ws);            ws += round_up((size_t)rows * sizeof(float), 256);
  float *dm = reinterpret_cast<float *>(ws);
  hipLaunchKernelGGL(train_residual, dim3(rows), dim3(256), 0, s, (const uint16_t *)Y_hat, (const uint16_t *)Y_dense,
                     rows, L->m, g, rowloss);
  PARSE_LAUNCH_CHECK();
  const TrainPair tp{(const uint16_t *)X, (const uint16_t *)L->Vt, g, (const uint16_t *)Ut_rankmajor, W, rows, L->n, L->m, L->R};
  st = forward_train_pair(tp, s);
  if (st != PARSE_OK) return st;
  hipLaunchKernelGGL(train_mask_grad, dim3(L->G + (loss_out ? 1 : 0), P), dim3(256), 0, s, W, rows, gs, tok_offsets, rowloss, dm,
                     loss_out, L->G);
  PARSE_LAUNCH_CHECK();
  int width = 1;
  while (width < L->G) width *= 2;
  hipLaunchKernelGGL(train_router_grad, dim3((d + 255) / 256, (L->G + TR_GJ - 1) / TR_GJ), dim3(256), 0, s, dm, scores, emb, P,
                     L->G, d, k, 1.0f / temperature, eps, width, grad_Wr);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

}  // extern "C"
