// a1 + a2: prompt pooling and the linear router with top-k (Sec. 4.1, Eq. 5).
//
// The rows of a prompt are dealt round robin to 4 Q chains of sums (Q slices of four), the chains of a slice are added in order, then
// the slices in order; fp32, rows streamed once, the same bits whichever kernel does it:
//   pool_rows     a workgroup holds all chains of 16 lanes' (or 8) columns of a prompt and writes the means: one launch
//   pool_partial  a workgroup is one slice of 64 lanes' columns, its sums go to memory and pool_finish or route_finish adds
//                 them: long prompts that are too few for one workgroup each to fill the chip
//   route_finish  one block per prompt: the embedding, or its sum of the Q partials, scores the G groups (one
//                 wavefront per group, butterfly reduction) and selects the top k with a rank count inside one wavefront.
#include "common.hpp"
#include "topk.hpp"

namespace parse {

constexpr int kPoolThreads = 256, kPoolWaves = kPoolThreads / 64;

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

template <bool BF16, bool MEAN>
__global__ __launch_bounds__(kPoolThreads) void pool_partial(const void *__restrict__ X, int rows, int d,
                                                             const int32_t *__restrict__ tok_offsets,
                                                             int Q, float *__restrict__ partial) {
  constexpr int PER = BF16 ? 8 : 4;  // columns per lane = 16 bytes
  constexpr int U = 16;              // rows a wavefront has in flight
  __shared__ float red[kPoolWaves - 1][PER][64];
  const int p = blockIdx.z, q = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int c0 = (blockIdx.x * 64 + lane) * PER;
  const bool in = c0 < d;
  const int a = clampi(tok_offsets[p], 0, rows);
  const int b = clampi(tok_offsets[p + 1], a, rows);
  // the rows of a prompt are dealt round robin to the Q * kPoolWaves wavefronts that share a column block: at any
  // moment they read a window of consecutive rows
  const int r0 = a + q * kPoolWaves + wave, r1 = b, rstep = Q * kPoolWaves;
  float acc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = 0.f;
  // U rows at a time: all of them are requested before the first is added (left to itself the compiler waits for every
  // row before it asks for the next); rows past the end re-read the wavefront's last row and are not added; the adds
  // run in row order.  Lanes past the last column re-read the last piece of the row; their sums are not stored.
  const char *xb = reinterpret_cast<const char *>(X) + (size_t)min(c0, d - PER) * (BF16 ? 2 : 4);
  const size_t row_bytes = (size_t)d * (BF16 ? 2 : 4);
  for (int r = r0; r < r1; r += rstep * U) {
    const int rlast = r + ((r1 - 1 - r) / rstep) * rstep;
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const u32x4 *>(xb + (size_t)min(r + u * rstep, rlast) * row_bytes);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r + u * rstep < r1) {       // uniform
        if constexpr (BF16) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[2 * i] += __uint_as_float(v[u][i] << 16);
            acc[2 * i + 1] += __uint_as_float(v[u][i] & 0xFFFF0000u);
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i] += __uint_as_float(v[u][i]);
        }
      }
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int i = 0; i < PER; ++i) red[wave - 1][i][lane] = acc[i];
  }
  __syncthreads();
  if (wave == 0 && in) {
    for (int w = 0; w < kPoolWaves - 1; ++w)
#pragma unroll
      for (int i = 0; i < PER; ++i) acc[i] += red[w][i][lane];
    if (MEAN) {                                  // Q == 1: the embedding itself
      const float inv = b > a ? 1.0f / (float)(b - a) : 0.f;
#pragma unroll
      for (int i = 0; i < PER; ++i) acc[i] *= inv;
    }
    float *dst = partial + ((size_t)p * Q + q) * d + c0;
#pragma unroll
    for (int i = 0; i < PER; i += 4) *reinterpret_cast<float4 *>(dst + i) = float4{acc[i], acc[i + 1], acc[i + 2], acc[i + 3]};
  }
}

// Workgroup = (prompt, 1 << lwl lanes of 16 bytes of columns, all 4 Q chains): lane l of chain c adds rows c, c + 4 Q, ... of its
// columns.  Bound by HBM for long prompts, by a round trip to memory and the launch for short ones.
constexpr int kPoolRowsThreads = 1024;       // the most
template <bool BF16>
__global__ __launch_bounds__(kPoolRowsThreads) void pool_rows(const void *__restrict__ X, int rows, int d, const int32_t *__restrict__ tok_offsets,
                                                              int Q, int lwl, float *__restrict__ emb) {
  constexpr int PER = BF16 ? 8 : 4;  // columns per lane = 16 bytes
  constexpr int U = 16;              // rows a lane has in flight
  extern __shared__ __attribute__((aligned(16))) float red[];      // [chain][column]
  const int p = blockIdx.y;
  const int cols = PER << lwl, chains = Q * kPoolWaves;
  const int chain = (int)threadIdx.x >> lwl, lane = (int)threadIdx.x & ((1 << lwl) - 1);
  const int c0 = blockIdx.x * cols + lane * PER;
  const int a = clampi(tok_offsets[p], 0, rows);
  const int b = clampi(tok_offsets[p + 1], a, rows);
  float acc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = 0.f;
  // loads and sums as in pool_partial; U steps of a chain are at most 128 MiB
  const char *xr = reinterpret_cast<const char *>(X) + ((size_t)(a + chain) * d + min(c0, d - PER)) * (BF16 ? 2 : 4);
  const uint32_t step = (uint32_t)chains * d * (BF16 ? 2 : 4);
  for (int left = b - a - chain > 0 ? (b - a - chain - 1) / chains : -1; left >= 0; left -= U) {   // rows of the chain after this one
    u32x4 v[U];
    uint32_t at = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = *reinterpret_cast<const u32x4 *>(xr + at);
      at += u < left ? step : 0u;
    }
    xr += (size_t)U * step;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u <= left) {
        if constexpr (BF16) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[2 * i] += __uint_as_float(v[u][i] << 16);
            acc[2 * i + 1] += __uint_as_float(v[u][i] & 0xFFFF0000u);
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i] += __uint_as_float(v[u][i]);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < PER; i += 4)
    *reinterpret_cast<float4 *>(red + chain * cols + lane * PER + i) = float4{acc[i], acc[i + 1], acc[i + 2], acc[i + 3]};
  __syncthreads();
  const float inv = b > a ? 1.0f / (float)(b - a) : 0.f;
  for (int c = threadIdx.x; c < cols; c += chains << lwl) {
    if ((int)blockIdx.x * cols + c >= d) break;
    float total = 0.f;
#pragma unroll 4
    for (int q = 0; q < Q; ++q) {
      const float *s = red + q * kPoolWaves * cols + c;
      float part = s[0];
#pragma unroll
      for (int w = 1; w < kPoolWaves; ++w) part += s[w * cols];
      total += part;
    }
    emb[(size_t)p * d + blockIdx.x * cols + c] = total * inv;
  }
}

constexpr int kFinishThreads = 1024;

template <bool MEANS>                       // partial: the embeddings instead of Q slices' sums
__global__ __launch_bounds__(kFinishThreads) void route_finish(const float *__restrict__ partial, int Q, int rows, int d,
                                                               const int32_t *__restrict__ tok_offsets,
                                                               const float *__restrict__ Wr, int G, int k,
                                                               int32_t *__restrict__ subset_out, int subset_stride,
                                                               float *__restrict__ scores_out,
                                                               float *__restrict__ emb_out, int n_shared) {
  extern __shared__ float lds[];
  float *e = lds;          // [d]
  float *s = lds + d;      // [64]
  const int p = blockIdx.x;
  const int a = clampi(tok_offsets[p], 0, rows);
  const int b = clampi(tok_offsets[p + 1], a, rows);
  const float inv = (b > a) ? 1.0f / (float)(b - a) : 0.f;
  // four columns per lane, the Q slice partials added in slice order (independent loads, fixed order of adds)
  if (MEANS) {
    for (int c = threadIdx.x * 4; c < d; c += kFinishThreads * 4)
      *reinterpret_cast<float4 *>(e + c) = *reinterpret_cast<const float4 *>(partial + (size_t)p * d + c);
  } else
  for (int c = threadIdx.x * 4; c < d; c += kFinishThreads * 4) {
    const float *src = partial + (size_t)p * Q * d + c;
    float4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int q = 0; q < Q; ++q) {
      const float4 v = *reinterpret_cast<const float4 *>(src + (size_t)q * d);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    acc.x *= inv; acc.y *= inv; acc.z *= inv; acc.w *= inv;
    *reinterpret_cast<float4 *>(e + c) = acc;
    if (emb_out) *reinterpret_cast<float4 *>(emb_out + (size_t)p * d + c) = acc;
  }
  __syncthreads();
  block_router_scores(Wr, e, d, G, s, kFinishThreads / 64);
  if (scores_out)
    for (int g = threadIdx.x; g < G; g += kFinishThreads) scores_out[(size_t)p * G + g] = s[g];
  if (threadIdx.x < 64) wave_topk_ascending(s, G, k, subset_out + (size_t)p * subset_stride, n_shared);
}

// Slices per prompt: about two workgroups per compute unit, a slice of at least 32 rows (8 per wavefront), at most
// 32 slices.
static int pool_slices(int rows, int P, int d, bool bf16) {
  const int per_block = 64 * (bf16 ? 8 : 4);
  const int colblocks = (d + per_block - 1) / per_block;
  long long want = (512 + (long long)P * colblocks - 1) / ((long long)P * colblocks);
  long long avg = rows / (P > 0 ? P : 1);
  long long by_len = avg / 32 > 0 ? avg / 32 : 1;
  long long q = want < by_len ? want : by_len;
  if (q > 32) q = 32;
  if (q < 1) q = 1;
  return (int)q;
}

// Launches pool_partial into `partial` ([P][Q][d] floats)
template <bool MEAN>
static int launch_pool_partials(const void *X, bool bf16, int rows, const int32_t *tok_offsets, int P, int d, int Q, float *partial, hipStream_t s) {
  const int per_block = 64 * (bf16 ? 8 : 4);
  hipLaunchKernelGGL((bf16 ? pool_partial<true, MEAN> : pool_partial<false, MEAN>), dim3((d + per_block - 1) / per_block, Q, P), dim3(kPoolThreads),
                     0, s, X, rows, d, tok_offsets, Q, partial);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

// Lanes (their log2) that a workgroup of pool_rows gives to a row, or -1 where the slices' own launch is faster.  Sixteen lanes read whole lines of a
// row, eight where that makes fewer workgroups than units.  A workgroup no larger than one of the slices makes as many of them per prompt: taken for up
// to 24 rows a chain.  A larger one is taken for up to 16, all of which are on their way at once, and while all rows of the batch through its columns are
// 1 MiB at most (0.5 below 512 columns, where the sums of the slices are next to nothing): the lengths are not known here, and a prompt that holds most of the
// rows has an eighth to a half of the slices' workgroups.  Half of these rows a chain where rows do not start on a line of 128 bytes: the narrow pieces then take
// in up to twice their lines.  Over 2528 batches of 1 to 64 prompts of 1 to 4096 rows, 64 to 16384 columns, as long as each other, ragged, or one with half
// of the rows: 11 % less time than two launches on average, 8 % more at worst (always one launch: 160 % more).
// Embeddings, us, two launches / one: 8 x 512 rows of 4096 columns 10.4 / 8.6, 20 ragged 14.6 / 12.5, one of 77 3.6 / 3.1, of 160 6.1 / 3.3, of 700 7.3 /
// 4.7, of 4096 11.8 / 12.9, of 16000 31 / 66; 1024 columns, 8 x 512 6.4 / 4.6, one of 4096 8.4 / 9.7; fp32, 1024 columns, 4 x 64 4.7 / 2.8; one slice, 64 x 20 rows
// of 4096 columns 4.6 / 5.1; 19 of 80 columns and 1295 rows on average 7.7 / 5.7, one of them of 12600 12.9 / 24.8; 4488 columns, 8 x 466 9.9 / 11.8.
// The router's second launch comes either way, and adds the slices of few columns fast (256 columns, 8 x 512 rows 7.3 / 7.7, one of 1050 7.4 / 8.5): not below 1024
// columns, and for more than eight rows a chain only where the workgroups are half as many as units and rows start on lines.  4096 columns, 8 x 512 15.5 /
// 14.6, one of 160 9.8 / 8.4; 1024 columns, 8 x 512 9.1 / 9.0; 1120 columns, one of 2152 9.4 / 10.9; 2 % less time on average over the same batches.
static int pool_rows_lanes(int rows, int P, int d, bool bf16, int Q, bool router) {
  if (Q == 1) return -1;
  const int chains = Q * kPoolWaves, per = bf16 ? 8 : 4;
  const long long per_chain = rows / P / chains;       // rows
  const bool lines = d % (per * 8) == 0;
  auto wgs = [&](int l) { return (long long)P * ((d + (per << l) - 1) / (per << l)); };
  int l = wgs(4) < 256 ? 3 : 4;
  while ((chains << l) > kPoolRowsThreads) --l;
  if (chains << l <= kPoolThreads) {
    if (per_chain > (lines ? 24 : 12)) return -1;
  } else if (per_chain > (lines ? 16 : 8) || (long long)rows * (16 << l) > (d < 512 ? 512 : 1024) * 1024) {
    return -1;
  }
  if (router && (d < 1024 || (per_chain > 8 && (wgs(l) < 128 || !lines)))) return -1;
  return l;
}

static int launch_pool_rows(const void *X, bool bf16, int rows, const int32_t *tok_offsets, int P, int d, int Q, int l, float *emb, hipStream_t s) {
  const int per = bf16 ? 8 : 4, threads = (Q * kPoolWaves) << l;
  hipLaunchKernelGGL((bf16 ? pool_rows<true> : pool_rows<false>), dim3((d + (per << l) - 1) / (per << l), P), dim3(threads),
                     (size_t)threads * per * sizeof(float), s, X, rows, d, tok_offsets, Q, l, emb);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

int launch_pool_finish(const float *partial, int Q, int rows, int d, const int32_t *tok_offsets, int P, float *emb,
                       hipStream_t s);   // with the rank-granular router

// Embeddings of a batch, with the bits of the router's.
int launch_pool(const void *X, int xdtype, int rows, const int32_t *tok_offsets, int P, int d, float *partial, float *emb, hipStream_t s) {
  const bool bf16 = xdtype == PARSE_BF16;
  const int Q = pool_slices(rows, P, d, bf16), l = pool_rows_lanes(rows, P, d, bf16, Q, false);
  if (l >= 0) return launch_pool_rows(X, bf16, rows, tok_offsets, P, d, Q, l, emb, s);
  if (Q == 1) return launch_pool_partials<true>(X, bf16, rows, tok_offsets, P, d, 1, emb, s);
  const int st = launch_pool_partials<false>(X, bf16, rows, tok_offsets, P, d, Q, partial, s);
  if (st != PARSE_OK) return st;
  return launch_pool_finish(partial, Q, rows, d, tok_offsets, P, emb, s);
}

}  // namespace parse

using namespace parse;

extern "C" {

size_t parse_route_workspace_bytes(int32_t rows, int32_t P, int32_t d) {
  if (rows <= 0 || P <= 0 || d <= 0) return 0;
  // the slice count does not depend on the dtype beyond the column-block count; size for the larger one
  const int q = pool_slices(rows, P, d, false) > pool_slices(rows, P, d, true) ? pool_slices(rows, P, d, false)
                                                                                  : pool_slices(rows, P, d, true);
  return round_up((size_t)P * q * d * sizeof(float), 256);
}

int parse_pool(const void *X, int32_t xdtype, int32_t rows, const int32_t *tok_offsets, int32_t P, int32_t d,
               float *emb_out, void *workspace, size_t workspace_bytes, parse_stream stream) {
  if (!X || !tok_offsets || !emb_out) return PARSE_EINVAL;
  if (xdtype != PARSE_F32 && xdtype != PARSE_BF16) return PARSE_EINVAL;
  if (rows <= 0 || P <= 0 || d <= 0) return PARSE_EINVAL;
  if (d > 16384 || P > rows) return PARSE_ESHAPE;
  if (d % 8 != 0) return PARSE_EALIGN;
  if (!aligned16(X) || !aligned16(emb_out) || !aligned16(workspace)) return PARSE_EALIGN;
  if (!workspace || workspace_bytes < parse_route_workspace_bytes(rows, P, d)) return PARSE_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  float *partial = reinterpret_cast<float *>(workspace);
  return launch_pool(X, xdtype, rows, tok_offsets, P, d, partial, emb_out, s);
}

int parse_route(const void *X, int32_t xdtype, int32_t rows, const int32_t *tok_offsets, int32_t P, int32_t d,
                const float *Wr, int32_t G, int32_t k, int32_t *subset_out, int32_t subset_stride,
                float *scores_out, float *emb_out, void *workspace, size_t workspace_bytes,
                parse_stream stream) {
  return parse_route_shared(X, xdtype, rows, tok_offsets, P, d, Wr, G, k, 0, subset_out, subset_stride, scores_out,
                            emb_out, workspace, workspace_bytes, stream);
}

int parse_route_shared(const void *X, int32_t xdtype, int32_t rows, const int32_t *tok_offsets, int32_t P, int32_t d,
                       const float *Wr, int32_t G, int32_t k, int32_t n_shared, int32_t *subset_out,
                       int32_t subset_stride, float *scores_out, float *emb_out, void *workspace,
                       size_t workspace_bytes, parse_stream stream) {
  if (!X || !tok_offsets || !Wr || !subset_out) return PARSE_EINVAL;
  if (xdtype != PARSE_F32 && xdtype != PARSE_BF16) return PARSE_EINVAL;
  if (rows <= 0 || P <= 0 || d <= 0 || G <= 0 || k <= 0) return PARSE_EINVAL;
  if (n_shared < 0) return PARSE_EINVAL;
  if (k > G || G > 64 || d > 16384 || P > rows || subset_stride < k || n_shared > k) return PARSE_ESHAPE;
  if (d % 8 != 0) return PARSE_EALIGN;
  if (!aligned16(X) || !aligned16(Wr) || !aligned16(workspace)) return PARSE_EALIGN;
  if (emb_out && !aligned16(emb_out)) return PARSE_EALIGN;
  if (!workspace || workspace_bytes < parse_route_workspace_bytes(rows, P, d)) return PARSE_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  float *partial = reinterpret_cast<float *>(workspace);
  const bool bf16 = xdtype == PARSE_BF16;
  const int Q = pool_slices(rows, P, d, bf16), l = pool_rows_lanes(rows, P, d, bf16, Q, true);
  int st;
  if (l >= 0) {              // the means, where the caller or the second launch wants them
    if (emb_out) partial = emb_out;
    st = launch_pool_rows(X, bf16, rows, tok_offsets, P, d, Q, l, partial, s);
  } else {
    st = launch_pool_partials<false>(X, bf16, rows, tok_offsets, P, d, Q, partial, s);
  }
  if (st != PARSE_OK) return st;
  const size_t lds = (size_t)(d + 64) * sizeof(float);
  const auto finish = l >= 0 ? route_finish<true> : route_finish<false>;
  PARSE_ALLOW_LDS(finish, 0, lds);
  hipLaunchKernelGGL(finish, dim3(P), dim3(kFinishThreads), lds, s, partial, Q, rows, d, tok_offsets, Wr, G, k,
                     subset_out, subset_stride, scores_out, emb_out, n_shared);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

}  // extern "C"
