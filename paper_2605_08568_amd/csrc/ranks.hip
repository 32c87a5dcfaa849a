// Rank-granular routing: the paper's own formulation (Sec. 4.1, Eq. 4-5) -- every rank-1 component is an expert,
// the router maps the prompt embedding to one score per rank (R^d -> R^{r_max}) and the K best ranks are active.
// The grouped path elsewhere in this library is the special case of contiguous groups; here
//   route_ranks  pool (shared with the grouped router) -> embedding -> scores = Wr e for thousands of ranks, a
//                bandwidth-bound skinny product that reads Wr once per block of 8 prompts -> exact top-K by radix
//                select over the score bits (ties to the lower rank id), ids written ascending;
//   pack_ranks   the K selected rank rows of a row-major bf16 layer are gathered and written straight into
//                matrix-core operand order (the memory aggregation of Sec. 4.4 for scattered single ranks: K
//                row reads of n*2 / m*2 bytes become one contiguous block per pattern), after which the
//                prefill kernels run unchanged with r_S = K.
#include "common.hpp"

namespace parse {

int launch_pool(const void *X, int xdtype, int rows, const int32_t *tok_offsets, int P, int d, float *partial, float *emb, hipStream_t s);

constexpr int RK_MAXG = 8192;        // ranks the selection kernel holds in LDS

// e[p][:] = (sum of the Q slice partials, in slice order) / prompt length.  grid (ceil(d/1024), P), block 256.
__global__ __launch_bounds__(256) void pool_finish(const float *__restrict__ partial, int Q, int rows, int d,
                                                   const int32_t *__restrict__ tok_offsets, float *__restrict__ emb) {
  const int p = blockIdx.y;
  const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c >= d) return;
  int a = tok_offsets[p], b = tok_offsets[p + 1];
  a = a < 0 ? 0 : (a > rows ? rows : a);
  b = b < a ? a : (b > rows ? rows : b);
  const float inv = (b > a) ? 1.0f / (float)(b - a) : 0.f;
  const float *src = partial + (size_t)p * Q * d + c;
  float4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int q = 0; q < Q; ++q) {
    const float4 v = *reinterpret_cast<const float4 *>(src + (size_t)q * d);
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  acc.x *= inv; acc.y *= inv; acc.z *= inv; acc.w *= inv;
  *reinterpret_cast<float4 *>(emb + (size_t)p * d + c) = acc;
}

// Shared with the embedding-only entry point.
int launch_pool_finish(const float *partial, int Q, int rows, int d, const int32_t *tok_offsets, int P, float *emb,
                       hipStream_t s) {
  hipLaunchKernelGGL(pool_finish, dim3((d + 1023) / 1024, P), dim3(256), 0, s, partial, Q, rows, d, tok_offsets, emb);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

// scores[p][g] = <Wr[g], e_p>.  grid (router rows in units of WAVES RPW, prompts in units of PB), block 64 WAVES: wavefront w owns RPW rows
// for the PB prompts of the block; lane l adds columns 256 i + 4 l .. + 3 for i = 0, 1, ..., and the 64 lanes are added at the end (the
// same order for all RPW and PB: same inputs, same bits).  Bound by the stream of Wr and, for eight prompts, by the embeddings that come in beside
// it: parts of RK_PART columns, rows and embeddings of the next ones on their way while one is added up; the embeddings go through LDS,
// where the wavefronts share them.
constexpr int RK_PART = 1024, RK_STEPS = RK_PART / 256, RK_AHEAD = 2;
template <int RPW, int PB, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 1) void rank_scores(const float *__restrict__ Wr, const float *__restrict__ emb, int G,
                                                              int d, int P, float *__restrict__ scores) {
  constexpr int BUFS = RPW == 1 ? 2 : 1;                // one for three workgroups a unit instead of two
  __shared__ f32x4 es[BUFS][PB][RK_PART / 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g0 = (blockIdx.x * WAVES + wave) * RPW, p0 = blockIdx.y * PB;
  constexpr int EP = PB * 4 / WAVES;                    // embeddings of a thread: e0, e0 + WAVES / 4, ...
  const int e0 = threadIdx.x >> 8, ec = threadIdx.x & 255;
  float acc[RPW][PB];
#pragma unroll
  for (int r = 0; r < RPW; ++r)
#pragma unroll
    for (int p = 0; p < PB; ++p) acc[r][p] = 0.f;
  const float *wrow[RPW], *erow[EP];
#pragma unroll
  for (int r = 0; r < RPW; ++r) wrow[r] = Wr + (size_t)min(g0 + r, G - 1) * d;
#pragma unroll
  for (int i = 0; i < EP; ++i) erow[i] = emb + (size_t)min(p0 + e0 + i * (WAVES / 4), P - 1) * d;
  f32x4 w[RK_AHEAD][RPW][RK_STEPS], e[RK_AHEAD][EP];
  auto load = [&](int base, f32x4 (&wv)[RPW][RK_STEPS], f32x4 (&ev)[EP]) {   // columns past the end: the last four again, not used
#pragma unroll
    for (int i = 0; i < EP; ++i) ev[i] = *reinterpret_cast<const f32x4 *>(erow[i] + min(base + ec * 4, d - 4));
#pragma unroll
    for (int i = 0; i < RK_STEPS; ++i)
#pragma unroll
      for (int r = 0; r < RPW; ++r) wv[r][i] = *reinterpret_cast<const f32x4 *>(wrow[r] + min(base + i * 256 + lane * 4, d - 4));
  };
#pragma unroll
  for (int u = 0; u < RK_AHEAD; ++u)
    if (u * RK_PART < d) load(u * RK_PART, w[u], e[u]);
  int buf = 0;
  for (int b0 = 0; b0 < d; b0 += RK_AHEAD * RK_PART) {
#pragma unroll
    for (int u = 0; u < RK_AHEAD; ++u) {
      const int base = b0 + u * RK_PART;
      if (base >= d) break;                            // uniform
      if (BUFS == 1 && base > 0)                       // the part before is read
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
      for (int i = 0; i < EP; ++i) es[buf][e0 + i * (WAVES / 4)][ec] = e[u][i];
      // everybody's piece is there (of two buffers the other one is read by now).  No fence: loads on their way stay so.
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
      for (int i = 0; i < RK_STEPS; ++i)
        if (base + i * 256 + lane * 4 < d) {
#pragma unroll
          for (int p = 0; p < PB; ++p) {
            const f32x4 v = es[buf][p][i * 64 + lane];
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
              const f32x4 x = w[u][r][i];
              acc[r][p] += x[0] * v[0] + x[1] * v[1] + x[2] * v[2] + x[3] * v[3];
            }
          }
        }
      buf ^= BUFS - 1;
      if (base + RK_AHEAD * RK_PART < d) load(base + RK_AHEAD * RK_PART, w[u], e[u]);
    }
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r)
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const float v = wave_sum(acc[r][p]);
      if (lane == 0 && g0 + r < G && p0 + p < P) scores[(size_t)(p0 + p) * G + g0 + r] = v;
    }
}

// The same sums without LDS: two rows a wavefront, which reads the eight embeddings for itself, four steps of 256 columns on their way.  Many workgroups of
// few columns hide each other's waits better than loads ahead do, which come in parts of RK_PART and are for nothing past the last column.
constexpr int RK_ROWS = 8, RK_PB = 8;        // router rows and prompts of a workgroup
__global__ __launch_bounds__(256) void rank_scores_narrow(const float *__restrict__ Wr, const float *__restrict__ emb, int G,
                                                          int d, int P, float *__restrict__ scores) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g0 = blockIdx.x * RK_ROWS + wave * 2, p0 = blockIdx.y * RK_PB;
  float acc[2][RK_PB];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int p = 0; p < RK_PB; ++p) acc[r][p] = 0.f;
  const float *wrow[2], *erow[RK_PB];
#pragma unroll
  for (int r = 0; r < 2; ++r) wrow[r] = Wr + (size_t)min(g0 + r, G - 1) * d;
#pragma unroll
  for (int p = 0; p < RK_PB; ++p) erow[p] = emb + (size_t)min(p0 + p, P - 1) * d;
#pragma unroll 4
  for (int c = lane * 4; c < d; c += 256) {
    f32x4 w[2], e[RK_PB];
#pragma unroll
    for (int r = 0; r < 2; ++r) w[r] = *reinterpret_cast<const f32x4 *>(wrow[r] + c);
#pragma unroll
    for (int p = 0; p < RK_PB; ++p) e[p] = *reinterpret_cast<const f32x4 *>(erow[p] + c);
#pragma unroll
    for (int p = 0; p < RK_PB; ++p)
#pragma unroll
      for (int r = 0; r < 2; ++r) acc[r][p] += w[r][0] * e[p][0] + w[r][1] * e[p][1] + w[r][2] * e[p][2] + w[r][3] * e[p][3];
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int p = 0; p < RK_PB; ++p) {
      const float v = wave_sum(acc[r][p]);
      if (lane == 0 && g0 + r < G && p0 + p < P) scores[(size_t)(p0 + p) * G + g0 + r] = v;
    }
}

// One row a wavefront while every workgroup is at work at once (two a unit), or with so few prompts that the embeddings do not count; else two,
// which share what they read of LDS, and one buffer, so that three workgroups fit a unit.  The whole routing call, us, the kernel without LDS / one row / two
// rows, 4096 columns: 2048 ranks x 8 prompts 30.6 / 27.6 / 29.2, x 1 23.2 / 17.5 / 18.0, x 16 29.5 / 31.9 / 28.7, x 20 36.3 / 41.6 / 33.3, 512 x 8 23.3 / 17.5 /
// 20.5, 8192 x 8 63.0 / 60.9 / 50.0, 8192 x 1 56.7 / 41.7 / 42.8; 1024 columns, 512 x 8 17.8 / 13.9 / 15.7; same bits.
// Eight prompts and two workgroups of four wavefronts on some units: one of eight, and the embeddings come in once a unit.  The call, 256 workgroups of four / of
// eight: 4096 columns, 2048 ranks x 8 prompts 23.9 / 22.6, 1040 x 8 21.8 / 20.3, 1024 x 16 21.5 / 20.3; 2048 columns, 2048 x 8 19.0 / 18.6; 512 columns 14.7 /
// 14.5; with a unit to each of four the same.
// Without LDS for more than four prompts and 1024 workgroups of one row where over a fifth of the parts' columns is past the last one: 144 columns, 3576 ranks
// x 12 prompts 18.7 / 23.9 / 21.9, 1032, 6442 x 8 26.3 / 33.5 / 29.6, 2136, 6311 x 16 43.6 / 57.6 / 45.2; with fewer, 1480 workgroups x 4 prompts of 88 columns 20.2 /
// 19.2 / 18.8.  Over 300 calls of 32 to 16384 columns, 32 to 8192 ranks and 1 to 64 prompts 18 % less time than without LDS throughout, 8 % more at worst.
template <int PB>
static int launch_rank_scores(const float *Wr, const float *emb, int G, int d, int P, float *scores, hipStream_t s) {
  const int blocks = (P + PB - 1) / PB, parts = (d + RK_PART - 1) / RK_PART;
  const long long wgs = (long long)((G + 3) / 4) * blocks;
  if constexpr (PB == RK_PB) {
    if (wgs > 1024 && parts * RK_PART * 4 > d * 5) {
      hipLaunchKernelGGL(rank_scores_narrow, dim3((G + RK_ROWS - 1) / RK_ROWS, blocks), dim3(256), 0, s, Wr, emb, G, d, P, scores);
      PARSE_LAUNCH_CHECK();
      return PARSE_OK;
    }
  }
  if constexpr (PB > 2) {
    if (wgs > 512) {
      hipLaunchKernelGGL((rank_scores<2, PB, 4>), dim3((G + 7) / 8, blocks), dim3(256), 0, s, Wr, emb, G, d, P, scores);
      PARSE_LAUNCH_CHECK();
      return PARSE_OK;
    }
  }
  if constexpr (PB == RK_PB) {
    if (wgs > 256) {
      hipLaunchKernelGGL((rank_scores<1, PB, 8>), dim3((G + 7) / 8, blocks), dim3(512), 0, s, Wr, emb, G, d, P, scores);
      PARSE_LAUNCH_CHECK();
      return PARSE_OK;
    }
  }
  hipLaunchKernelGGL((rank_scores<1, PB, 4>), dim3((G + 3) / 4, blocks), dim3(256), 0, s, Wr, emb, G, d, P, scores);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

// order-preserving map of a float's bits: larger float <=> larger unsigned key (-0 counts as +0)
__device__ __forceinline__ uint32_t score_key(float f) {
  const uint32_t u = __float_as_uint(f + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exact top-K of one prompt's G scores.  One workgroup of 1024 lanes per prompt, keys in LDS.  Four radix passes
// (8 bits each, from the top) find the K-th largest key T; the selected set is {key > T} plus the lowest-id
// members of {key == T} up to K; ids come out ascending through a block prefix sum in id order.  Latency-bound by its
// barriers: the 256 bins are summed by one wavefront (four bins a lane, shuffles), the block prefix takes one shuffle scan
// per wavefront and one over the sixteen totals (2048 scores of 8 prompts: 10.4 us with scans of a barrier per step, 6.9 now).
__global__ __launch_bounds__(1024) void rank_topk(const float *__restrict__ scores, int G, int K,
                                                  int32_t *__restrict__ subset_out, int subset_stride) {
  __shared__ uint32_t keys[RK_MAXG];
  __shared__ __attribute__((aligned(16))) uint32_t hist[256];
  __shared__ uint32_t sel_prefix, sel_need;
  __shared__ int32_t wave_gt[16], wave_eq[16];
  const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int g = tid; g < G; g += 1024) keys[g] = score_key(scores[(size_t)p * G + g]);
  if (tid < 256) hist[tid] = 0u;
  uint32_t prefix = 0u, need = (uint32_t)K;
  __syncthreads();
  // after the pass for byte b, prefix holds the top bytes of T and need the number still to take among the keys that
  // share them
  for (int shift = 24; shift >= 0; shift -= 8) {
    const uint32_t himask = shift == 24 ? 0u : (0xFFFFFFFFu << (shift + 8));
    for (int g = tid; g < G; g += 1024) {
      const uint32_t kx = keys[g];
      if ((kx & himask) == (prefix & himask)) atomicAdd(&hist[(kx >> shift) & 0xFFu], 1u);
    }
    __syncthreads();
    if (wave == 0) {
      // lane l holds bins 4l..4l+3 and the number of keys above them; the wanted bin is the one whose suffix reaches
      // `need` while the next one's does not (exactly one: the total is >= need by construction)
      const uint4 h = *reinterpret_cast<const uint4 *>(&hist[lane * 4]);
      *reinterpret_cast<uint4 *>(&hist[lane * 4]) = uint4{0u, 0u, 0u, 0u};
      uint32_t suffix = h.x + h.y + h.z + h.w;
      const uint32_t own = suffix;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_down(suffix, o, 64);
        if (lane + o < 64) suffix += up;
      }
      uint32_t above = suffix - own;
      const uint32_t bin[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        if (above < need && above + bin[i] >= need) {
          sel_prefix = prefix | ((uint32_t)(lane * 4 + i) << shift);
          sel_need = need - above;
        }
        above += bin[i];
      }
    }
    __syncthreads();
    prefix = sel_prefix;
    need = sel_need;
  }
  const uint32_t T = prefix;
  const int need_eq = (int)need;                 // members of {key == T} to take, lowest ids first
  // ids in contiguous segments per lane, counts scanned over the block in id order
  const int per = (G + 1023) / 1024;
  const int s0 = min(tid * per, G), s1 = min(s0 + per, G);
  int ngt = 0, neq = 0;
  for (int g = s0; g < s1; ++g) { ngt += keys[g] > T ? 1 : 0; neq += keys[g] == T ? 1 : 0; }
  int igt = ngt, ieq = neq;                      // inclusive over the wavefront
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int a = __shfl_up(igt, o, 64), b = __shfl_up(ieq, o, 64);
    if (lane >= o) { igt += a; ieq += b; }
  }
  if (lane == 63) { wave_gt[wave] = igt; wave_eq[wave] = ieq; }
  __syncthreads();
  int before_gt = igt - ngt, before_eq = ieq - neq;   // exclusive over the block
  for (int w = 0; w < wave; ++w) { before_gt += wave_gt[w]; before_eq += wave_eq[w]; }
  for (int g = s0; g < s1; ++g) {
    const uint32_t kx = keys[g];
    const bool eq = kx == T;
    const bool take = kx > T || (eq && before_eq < need_eq);
    if (take) {
      const int pos = before_gt + min(before_eq, need_eq);
      if (pos < K) subset_out[(size_t)p * subset_stride + pos] = g;
    }
    before_gt += kx > T ? 1 : 0;
    before_eq += eq ? 1 : 0;
  }
}

// Gather + reorder into the operand-order blocks (index maps as in the offline reorder); rank r of pattern j is row
// subset[j*stride + r] of the row-major layer.  Out-of-range ids give zero rows.  Bound by the writes to memory (a pattern's
// blocks are new memory, the rows are shared by the patterns and stay in the last-level cache).

// A wavefront turns 32 ranks x GV_STEPS reduction steps, 128 bytes of each row: eight lanes take a row's whole line, and the lines come back from LDS
// as operands (places swizzled by the row), stored in 1 KiB pieces.  Lane by lane in operand order, 32 bytes of 32 rows an instruction, every line was
// asked for four times, and a unit has 256 lines outstanding at most: 1024 of 2048 ranks of a 4096 x 4096 layer for 8 patterns, both factors, 42.7 -> 38.8 us
// (stores past the caches: the same, and the products after it 1 to 2 us more; patterns next to each other in the grid: 41.2).
constexpr int GV_STEPS = 4;
__device__ __forceinline__ void gather_mfma16_v(int wg, const uint16_t *__restrict__ Vt, int R, int n,
                                                const int32_t *__restrict__ subset, int stride, int K,
                                                uint16_t *__restrict__ dst, char *lds) {
  const int nkb = n / 16, nch = (nkb + GV_STEPS - 1) / GV_STEPS;
  const size_t t = ((size_t)wg * 256 + threadIdx.x) >> 6;              // wavefront: (rank block, GV_STEPS reduction steps)
  const int lane = threadIdx.x & 63, j = lane & 31, q = lane >> 5;
  const int kb0 = (int)(t % nch) * GV_STEPS;
  const size_t rb = t / nch;
  if (rb >= (size_t)(K / 32)) return;
  const int pat = blockIdx.y;
  const int id = subset[(size_t)pat * stride + rb * 32 + j];
  char *tile = lds + (threadIdx.x >> 6) * 4096;                        // this wavefront's
  const int r8 = lane >> 3, c = lane & 7;                              // row of eight, 16-byte piece of its 128
  u32x4 v[4];
  bool ok[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = __shfl(id, u * 8 + r8, 64);
    ok[u] = row >= 0 && row < R;
    v[u] = *reinterpret_cast<const u32x4 *>(Vt + (size_t)(ok[u] ? row : 0) * n + min(kb0 * 2 + c, nkb * 2 - 1) * 8);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) *reinterpret_cast<u32x4 *>(tile + (u * 8 + r8) * 128 + ((c ^ r8) * 16)) = ok[u] ? v[u] : u32x4{0, 0, 0, 0};
  // other lanes' pieces from here on: this wavefront's writes stay ahead of its reads (LDS serves them in order, so nothing is waited for)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  char *out = (char *)dst + (size_t)pat * K * n * 2 + (rb * nkb + kb0) * 1024 + lane * 16;
#pragma unroll
  for (int u = 0; u < GV_STEPS; ++u)
    if (kb0 + u < nkb)
      *reinterpret_cast<u32x4 *>(out + (size_t)u * 1024) = *reinterpret_cast<const u32x4 *>(tile + j * 128 + (((u * 2 + q) ^ (j & 7)) * 16));
}

// A workgroup turns 16 ranks (one reduction step) x GU_COLS columns: whole pieces of the rank rows go to LDS, and come back
// as the 8 ranks of a column that make an output piece.  Same sizes: 40.9 us when every value was loaded by itself, 19.7 now.
constexpr int GU_COLS = 512, GU_LD = GU_COLS + 8;
__device__ __forceinline__ void gather_mfma16_u(int wg, const uint16_t *__restrict__ Ut, int R, int m,
                                                const int32_t *__restrict__ subset, int stride, int K,
                                                uint16_t *__restrict__ dst, uint16_t (*tile)[GU_LD]) {
  const int ncc = (m + GU_COLS - 1) / GU_COLS;
  const int kb = wg / ncc, c0 = (wg % ncc) * GU_COLS, cols = min(GU_COLS, m - c0);   // cols: a multiple of 32
  const int pat = blockIdx.y;
  const int32_t *ids = subset + (size_t)pat * stride + kb * 16;
  u32x4 v[GU_COLS / 128];                                              // 16 rows x GU_COLS / 8 pieces over 256 threads
#pragma unroll
  for (int u = 0; u < GU_COLS / 128; ++u) {
    const int piece = u * 256 + (int)threadIdx.x, r = piece / (GU_COLS / 8), c = piece % (GU_COLS / 8) * 8;
    const int row = ids[r];
    v[u] = u32x4{0, 0, 0, 0};
    if (row >= 0 && row < R && c < cols) v[u] = *reinterpret_cast<const u32x4 *>(Ut + (size_t)row * m + c0 + c);
  }
#pragma unroll
  for (int u = 0; u < GU_COLS / 128; ++u) {
    const int piece = u * 256 + (int)threadIdx.x, r = piece / (GU_COLS / 8), c = piece % (GU_COLS / 8) * 8;
    *reinterpret_cast<u32x4 *>(&tile[r][c]) = v[u];
  }
  __syncthreads();
  char *out = (char *)dst + (size_t)pat * K * m * 2 + ((size_t)kb * (m / 32) + c0 / 32) * 1024;
  for (int o = threadIdx.x; o < cols * 2; o += 256) {                  // piece (column block, q, j): ranks 8q..8q+7 of a column
    const int j = o & 31, q = (o >> 5) & 1, c = (o >> 6) * 32 + j;
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (uint32_t)tile[q * 8 + 2 * e][c] | ((uint32_t)tile[q * 8 + 2 * e + 1][c] << 16);
    *reinterpret_cast<u32x4 *>(out + (size_t)o * 16) = w;
  }
}

// Both factors in one launch: each is a chain of two loads and a store, and the workgroups of one cover the waits of the other's.
// 1024 of 2048 ranks of a 4096 x 4096 layer for 8 patterns: 22 + 20 us as two launches, 37 as one (with the right factor read lane by lane).
__global__ __launch_bounds__(256) void gather_mfma16(const uint16_t *__restrict__ Vt, const uint16_t *__restrict__ Ut, int R, int n, int m,
                                                     const int32_t *__restrict__ subset, int stride, int K,
                                                     uint16_t *__restrict__ Vt_S, uint16_t *__restrict__ Ut_S, int v_wgs) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[16][GU_LD];
  static_assert(sizeof(tile) >= 4 * 4096, "four wavefronts' tiles of the right factor");
  if ((int)blockIdx.x < v_wgs) gather_mfma16_v(blockIdx.x, Vt, R, n, subset, stride, K, Vt_S, (char *)tile);      // uniform
  else gather_mfma16_u(blockIdx.x - v_wgs, Ut, R, m, subset, stride, K, Ut_S, tile);
}

}  // namespace parse

using namespace parse;

extern "C" {

size_t parse_route_ranks_workspace_bytes(int32_t rows, int32_t P, int32_t d, int32_t G) {
  if (rows <= 0 || P <= 0 || d <= 0 || G <= 0) return 0;
  // pooling partials (as the grouped router), embeddings, scores
  return parse_route_workspace_bytes(rows, P, d) + round_up((size_t)P * d * sizeof(float), 256) +
         round_up((size_t)P * G * sizeof(float), 256);
}

int parse_route_ranks(const void *X, int32_t xdtype, int32_t rows, const int32_t *tok_offsets, int32_t P, int32_t d,
                      const float *Wr, int32_t G, int32_t K, int32_t *subset_out, int32_t subset_stride,
                      float *scores_out, float *emb_out, void *workspace, size_t workspace_bytes,
                      parse_stream stream) {
  if (!X || !tok_offsets || !Wr || !subset_out) return PARSE_EINVAL;
  if (xdtype != PARSE_F32 && xdtype != PARSE_BF16) return PARSE_EINVAL;
  if (rows <= 0 || P <= 0 || d <= 0 || G <= 0 || K <= 0) return PARSE_EINVAL;
  if (K > G || G > RK_MAXG || d > 16384 || P > rows || P > 65535 || subset_stride < K) return PARSE_ESHAPE;
  if (d % 8 != 0) return PARSE_EALIGN;
  if (!aligned16(X) || !aligned16(Wr) || !aligned16(workspace)) return PARSE_EALIGN;
  if ((emb_out && !aligned16(emb_out)) || (scores_out && !aligned16(scores_out))) return PARSE_EALIGN;
  if (!workspace || workspace_bytes < parse_route_ranks_workspace_bytes(rows, P, d, G)) return PARSE_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  char *ws = reinterpret_cast<char *>(workspace);
  const size_t pool_bytes = parse_route_workspace_bytes(rows, P, d);
  float *partial = reinterpret_cast<float *>(ws);
  float *emb = emb_out ? emb_out : reinterpret_cast<float *>(ws + pool_bytes);
  float *scores = scores_out ? scores_out
                             : reinterpret_cast<float *>(ws + pool_bytes + round_up((size_t)P * d * sizeof(float), 256));
  int st = launch_pool(X, xdtype, rows, tok_offsets, P, d, partial, emb, s);
  if (st != PARSE_OK) return st;
  st = P == 1 ? launch_rank_scores<1>(Wr, emb, G, d, P, scores, s) : P == 2 ? launch_rank_scores<2>(Wr, emb, G, d, P, scores, s)
       : P <= 4 ? launch_rank_scores<4>(Wr, emb, G, d, P, scores, s) : launch_rank_scores<8>(Wr, emb, G, d, P, scores, s);
  if (st != PARSE_OK) return st;
  hipLaunchKernelGGL(rank_topk, dim3(P), dim3(1024), 0, s, scores, G, K, subset_out, subset_stride);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

int parse_pack_ranks(const parse_layer *L, const int32_t *subset, int32_t subset_stride, int32_t K,
                     int32_t n_patterns, void *Vt_S, void *Ut_S, parse_stream stream) {
  int st = check_layer(L);
  if (st != PARSE_OK) return st;
  if (!subset || !Vt_S || !Ut_S) return PARSE_EINVAL;
  if (K <= 0 || n_patterns <= 0) return PARSE_EINVAL;
  if (L->dtype != PARSE_BF16 || L->layout != PARSE_ROWMAJOR) return PARSE_ELAYOUT;
  if (K % 32 != 0 || L->n % 16 != 0 || L->m % 32 != 0 || subset_stride < K || n_patterns > 65535) return PARSE_ESHAPE;
  if (!aligned16(Vt_S) || !aligned16(Ut_S)) return PARSE_EALIGN;
  hipStream_t s = (hipStream_t)stream;
  const size_t wv = (size_t)(K / 32) * ((L->n / 16 + GV_STEPS - 1) / GV_STEPS);     // wavefronts of a pattern
  const size_t wu = (size_t)(K / 16) * ((L->m + GU_COLS - 1) / GU_COLS);            // workgroups of a pattern
  const size_t v_wgs = (wv + 3) / 4;
  hipLaunchKernelGGL(gather_mfma16, dim3((unsigned)(v_wgs + wu), n_patterns), dim3(256), 0, s, (const uint16_t *)L->Vt, (const uint16_t *)L->Ut,
                     L->R, L->n, L->m, subset, subset_stride, K, (uint16_t *)Vt_S, (uint16_t *)Ut_S, (int)v_wgs);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

}  // extern "C"
