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
// Bound by the matrix cores and the load path into LDS.  Both operands are staged in LDS by loads that write LDS directly
// (factors in operand order, 1 KiB per instruction; token rows row-major with their 16-byte chunks XOR-swizzled on the way
// in), STAGES slices of BK in rotation, one barrier per slice.  The slices of the second product follow those of the
// first in the same ring: nothing drains between the two.
// Measured at 4096 rows, n = m = 4096, R = 2048: the two separate products and the pass over their outputs took 90 + 90 +
// 19 us, this kernel 139-156 us (137 GFLOP).
typedef __attribute__((ext_vector_type(2))) uint32_t tr_u32x2;

template <int BM, int BN, int WM, int WN, int BK, int STAGES>
__global__ __launch_bounds__(WM * WN * 64) void train_pair(TrainPair a) {
  constexpr int NW = WM * WN;
  constexpr int KK = BK / 16;
  constexpr int TB = BM / WM / 32, FB = BN / WN / 32;
  constexpr int F_BYTES = BN * BK * 2, T_BYTES = BM * BK * 2, STAGE_BYTES = F_BYTES + T_BYTES;
  constexpr int NI_F = F_BYTES / 1024, NI_T = T_BYTES / 1024;
  static_assert(NI_F % NW == 0 && NI_T % NW == 0, "the loads of a slice divide evenly over the wavefronts");
  static_assert(KK == 2 || KK == 4, "register double-buffering assumes an even number of steps");
  constexpr int LF = NI_F / NW, LT = NI_T / NW, L = LF + LT;
  constexpr int CPR = BK * 2 / 16, RPI = 1024 / (BK * 2);      // 16-byte chunks per staged row, rows per instruction
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int j = lane & 31, q = lane >> 5;
  // up to 8 token tiles run through a rank tile before the next one: a die's consecutive tiles share both operands in its L2
  const int ntm = (a.rows + BM - 1) / BM, ntn = (a.R + BN - 1) / BN;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int grp = tile / (8 * ntn), first = grp * 8, gm = min(8, ntm - first), r = tile - grp * 8 * ntn;
  const int tm = first + r % gm, tn = r / gm;
  const int nblk = a.R / 32;

  // sources of this wavefront's load instructions in the two products
  const char *fsrc[LF], *tsrc[LT], *fnext[LF], *tnext[LT];
  int fdst[LF], tdst[LT];
#pragma unroll
  for (int i = 0; i < LF; ++i) {
    const int ins = wave + i * NW, fb = ins / KK, kk = ins % KK;
    const int gb = min(tn * (BN / 32) + fb, nblk - 1);         // blocks past the end re-read the last one (never stored)
    fsrc[i] = (const char *)a.V + ((size_t)gb * (a.n / 16) + kk) * 1024 + lane * 16;
    fnext[i] = (const char *)a.U + ((size_t)gb * (a.m / 16) + kk) * 1024 + lane * 16;
    fdst[i] = ins * 1024;
  }
#pragma unroll
  for (int i = 0; i < LT; ++i) {
    const int ins = wave + i * NW;
    const int rr = ins * RPI + lane / CPR, cp = lane % CPR;    // LDS position (row, chunk slot)
    const int sw = CPR == 4 ? ((rr >> 2) & 3) : ((rr >> 1) & 7);
    const size_t row = min(tm * BM + rr, a.rows - 1);          // rows past the end re-read the last one (never stored)
    tsrc[i] = (const char *)a.X + row * a.n * 2 + (cp ^ sw) * 16;
    tnext[i] = (const char *)a.g + row * a.m * 2 + (cp ^ sw) * 16;
    tdst[i] = F_BYTES + ins * 1024;
  }
  const int nk1 = a.n / BK, nk = nk1 + a.m / BK;
  int issued = 0;
  auto issue = [&](int stage_buf) {
    char *base = smem + stage_buf * STAGE_BYTES;
#pragma unroll
    for (int i = 0; i < LF; ++i) {
      __builtin_amdgcn_global_load_lds(PARSE_TR_GLB_PTR(fsrc[i]), PARSE_TR_LDS_PTR(base + fdst[i]), 16, 0, 0);
      fsrc[i] += KK * 1024;
    }
#pragma unroll
    for (int i = 0; i < LT; ++i) {
      __builtin_amdgcn_global_load_lds(PARSE_TR_GLB_PTR(tsrc[i]), PARSE_TR_LDS_PTR(base + tdst[i]), 16, 0, 0);
      tsrc[i] += BK * 2;
    }
    if (++issued == nk1) {                                     // uniform: on to the operands of the second product
#pragma unroll
      for (int i = 0; i < LF; ++i) fsrc[i] = fnext[i];
#pragma unroll
      for (int i = 0; i < LT; ++i) tsrc[i] = tnext[i];
    }
  };
  int foff[FB], toff[TB], tsw[TB];
#pragma unroll
  for (int i = 0; i < FB; ++i) foff[i] = ((wn * FB + i) * KK) * 1024 + lane * 16;
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    const int rr = (wm * TB + t) * 32 + j;
    toff[t] = F_BYTES + rr * (BK * 2);
    tsw[t] = CPR == 4 ? ((rr >> 2) & 3) : ((rr >> 1) & 7);
  }
  u32x4 fr[2][FB], tr[2][TB];
  auto read_ops = [&](int buf, int stage_buf, int kk) {
    const char *base = smem + stage_buf * STAGE_BYTES;
#pragma unroll
    for (int i = 0; i < FB; ++i) fr[buf][i] = *reinterpret_cast<const u32x4 *>(base + foff[i] + kk * 1024);
#pragma unroll
    for (int t = 0; t < TB; ++t) tr[buf][t] = *reinterpret_cast<const u32x4 *>(base + toff[t] + (((kk * 2 + q) ^ tsw[t]) * 16));
  };
  // this step's operands are touched before the next step's LDS reads are issued: the wait the compiler places there then
  // covers reads that had a whole step to finish
  auto settle = [&](int buf) {
#pragma unroll
    for (int i = 0; i < FB; ++i) asm volatile("" ::"v"(fr[buf][i]));
#pragma unroll
    for (int t = 0; t < TB; ++t) asm volatile("" ::"v"(tr[buf][t]));
  };
  f32x16 accz[TB][FB], acct[TB][FB];
#pragma unroll
  for (int t = 0; t < TB; ++t)
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) { accz[t][i][e] = 0.f; acct[t][i][e] = 0.f; }
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nk) issue(s);
  if (nk >= STAGES - 1) wait_vm<(STAGES - 2) * L>(); else wait_vm<0>();
  wg_barrier();
  if (STAGES - 1 < nk) issue(STAGES - 1);
  read_ops(0, 0, 0);
  int sb = 0;
  auto slices = [&](f32x16(&acc)[TB][FB], int k0, int k1) {
    for (int kt = k0; kt < k1; ++kt) {
      const int sn = sb + 1 == STAGES ? 0 : sb + 1;
#pragma unroll
      for (int s = 0; s < KK; ++s) {
        const int cur = s & 1;
        settle(cur);
        __builtin_amdgcn_sched_barrier(0);
        if (s < KK - 1) {
          read_ops(cur ^ 1, sb, s + 1);
        } else if (kt + 1 < nk) {
          // hand-over: slice kt+1 must have landed for every wavefront; slice kt's buffer is free after the barrier
          const int later = min(kt + STAGES - 1, nk - 1) - (kt + 1);   // slices requested after kt+1
          if (later >= STAGES - 2) wait_vm<(STAGES - 2) * L>();
          else if (STAGES > 3 && later == 1) wait_vm<L>();
          else wait_vm<0>();
          wg_barrier();
          if (kt + STAGES < nk) issue(sb);
          read_ops(cur ^ 1, sn, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
          for (int t = 0; t < TB; ++t)
            acc[t][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[cur][i]), as_bf16x8(tr[cur][t]), acc[t][i], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      sb = sn;
    }
  };
  slices(accz, 0, nk1);
  slices(acct, nk1, nk);
  // lane (j, q) of acc[t][i] holds token t*32+j, ranks i*32 + 8*band + 4*q + (0..3) of both products
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    const int row = tm * BM + (wm * TB + t) * 32 + j;
#pragma unroll
    for (int i = 0; i < FB; ++i) {
      const int gb = tn * (BN / 32) + wn * FB + i;
      float s[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        s[b] = accz[t][i][b * 4] * acct[t][i][b * 4];
#pragma unroll
        for (int e = 1; e < 4; ++e) s[b] += accz[t][i][b * 4 + e] * acct[t][i][b * 4 + e];
      }
      // the two halves of a band: lane (j, 0) ends up with bands 0 and 1, lane (j, 1) with bands 2 and 3
      float w[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const tr_u32x2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[b]), __float_as_uint(s[b + 2]), false, false);
        w[b] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
      }
      if (gb < nblk && row < a.rows) {
        float *dst = a.W + (size_t)(gb * 4 + q * 2) * a.rows + row;
        dst[0] = w[0];
        dst[a.rows] = w[1];
      }
    }
  }
}

template <int BM, int BN, int WM, int WN, int BK, int STAGES>
static int launch_train_pair(const TrainPair &a, hipStream_t s) {
  constexpr size_t smem = (size_t)STAGES * (BM + BN) * BK * 2;
  auto kern = train_pair<BM, BN, WM, WN, BK, STAGES>;
  PARSE_ALLOW_LDS(kern, smem);
  const int grid = ((a.rows + BM - 1) / BM) * ((a.R + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WM * WN * 64), smem, s, a);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

// Tile by how many workgroups it gives a launch.  256 x 128 (eight wavefronts, six slices of 32) moves the fewest bytes
// per flop and wins once it fills the chip; below that the tile that still fills it wins, and 64 x 64 when none does
// (whole call, us, 256 x 128 / 128 x 128 / 64 x 64: 4096 rows x 2048 ranks 155 / 181 / 218; 3300 x 1024 128 / 95 / 113;
// 4000 x 768 273 / 190 / 235; 1024 x 2048 204 / 145 / 113; 16 x 1024 111 / 79 / 47).
static int forward_train_pair(const TrainPair &a, hipStream_t s) {
  auto wgs = [&](int bm, int bn) { return (long long)((a.rows + bm - 1) / bm) * ((a.R + bn - 1) / bn); };
  if (wgs(256, 128) >= 192) return launch_train_pair<256, 128, 4, 2, 32, 6>(a, s);
  if (wgs(128, 128) >= 160) return launch_train_pair<128, 128, 2, 2, 64, 4>(a, s);
  return launch_train_pair<64, 64, 2, 2, 64, 4>(a, s);
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
