// a6 for fp32 layers: Y = (X Vt_S^T) Ut_S on the fp32 matrix instructions (16x16x4, full fp32 products and sums), two
// launches; the r_S-wide intermediate goes through the workspace.
//
// What bounds it: the fp32 layers are small (256 tokens x 1024 x 128 ranks: 0.13 GFLOP, 3 MB), so what counts is how much of
// the chip works at once and how many dependent memory round trips a wavefront makes.  Hence small output tiles (16 or 32
// token rows), the reduction cut over the wavefronts of a workgroup (added in wavefront order through LDS), and operands
// fetched straight into registers, several 16-deep reduction chunks at a time: lane (i = l % 16, g = l / 16) takes 16
// bytes of its row at reduction index 4 g, and the four matrix instructions of a chunk use element e of every lane, i.e.
// reduction indices {e, 4 + e, 8 + e, 12 + e} -- the same for both operands, so the order within a chunk does not matter.
// Measured at that size: both products 9.2 us (64 x 64 tiles of plain FMA through LDS, 8 workgroups for the first product: 178).
//
// Each block of token rows is cut into the segments that belong to one prompt, and a segment uses the packed factors of
// that prompt's pattern.
#include <algorithm>

#include "common.hpp"

namespace parse {

__device__ __forceinline__ f32x4 mfma_f32_16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// one block of token rows: calls body(valid, pattern, seg_lo, seg_hi) for every prompt segment of rows [row0, row_end)
template <bool TABLE, typename F>
__device__ __forceinline__ void for_segments(int row0, int row_end, int rows, const int32_t *__restrict__ tok_offsets,
                                             const int32_t *__restrict__ pattern_id, int P, int n_patterns, F body) {
  // TABLE, up to 64 prompts: offsets and patterns in one load each, side by side, then by lane, instead of a pattern read once its prompt is known: both
  // products of 4 x 64 rows of a 1024 x 1024 layer, 128 ranks, 9.7 -> 9.35 us, 1024 rows of 2048 x 2048 31.6 -> 30.8 (same bits).  Not for the first product's
  // large tiles, whose loops it makes slower: 41 prompts, 1189 rows, 3856 x 552, 588 ranks 233.5 / 250 us.
  const int lane = threadIdx.x & 63;
  int off_l = 0x7FFFFFFF, pid_l = -1;
  if (TABLE && P <= 64 && lane < P) {
    off_l = tok_offsets[lane];
    pid_l = pattern_id[lane];
  }
  int seg_lo = row0;
  while (seg_lo < row_end) {
    int p, pid, seg_hi;                                     // the last prompt owns every remaining row
    if (TABLE && P <= 64) {
      p = max(__popcll(__ballot(off_l <= seg_lo)) - 1, 0);
      pid = __builtin_amdgcn_readlane(pid_l, p);
      seg_hi = p + 1 < P ? __builtin_amdgcn_readlane(off_l, p + 1) : rows;
    } else if (TABLE) {
      p = prompt_of_row(tok_offsets, P, seg_lo);
      pid = pattern_id[p];
      seg_hi = p + 1 < P ? tok_offsets[p + 1] : rows;
    } else {                                                // the pattern last: the loop that follows comes out 7 % faster
      p = prompt_of_row_wave(tok_offsets, P, seg_lo);
      seg_hi = p + 1 < P ? tok_offsets[p + 1] : rows;
      pid = pattern_id[p];
    }
    seg_hi = min(max(seg_hi, seg_lo + 1), row_end);
    body(pid >= 0 && pid < n_patterns, pid, seg_lo, seg_hi);
    seg_lo = seg_hi;
  }
}

constexpr int FN_WAVES = 8;          // first product: wavefronts of a workgroup = parts of the reduction

// Z[rows][N] = X[rows][K] * B_p[N][K]^T.  K % 4 == 0.  RT x CT blocks of 16 token rows x 16 ranks per workgroup; a
// wavefront requests BATCH reduction chunks at a time.  KS slices of the reduction (blockIdx.z), each with its own Z.
template <int RT, int CT, int BATCH, int KS>
__global__ __launch_bounds__(FN_WAVES * 64) void sgemm_nt(const float *__restrict__ A, const float *__restrict__ Bbase,
                                                          size_t pattern_stride, int n_patterns, int rows, int N, int K,
                                                          const int32_t *__restrict__ tok_offsets,
                                                          const int32_t *__restrict__ pattern_id, int P, float *__restrict__ C) {
  constexpr int TN = CT * 16;
  __shared__ float red[FN_WAVES][RT * 16][TN];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  const int row0 = blockIdx.x * RT * 16, col0 = blockIdx.y * TN;
  int first = 0, chunks = (K + 15) / 16;
  if constexpr (KS > 1) {
    const int all = chunks;
    first = all * (int)blockIdx.z / KS;
    chunks = all * ((int)blockIdx.z + 1) / KS;
    C += (size_t)blockIdx.z * rows * N;
  }
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  for_segments<RT == 1>(row0, min(row0 + RT * 16, rows), rows, tok_offsets, pattern_id, P, n_patterns, [&](bool valid, int pid, int lo, int hi) {
    f32x4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int u = 0; u < CT; ++u) acc[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (valid) {
      const float *arow[RT], *brow[CT];
#pragma unroll
      for (int t = 0; t < RT; ++t) arow[t] = A + (size_t)min(row0 + t * 16 + i16, rows - 1) * K;
#pragma unroll
      for (int u = 0; u < CT; ++u) brow[u] = Bbase + (size_t)pid * pattern_stride + (size_t)min(col0 + u * 16 + i16, N - 1) * K;
      for (int c0 = first + wave; c0 < chunks; c0 += FN_WAVES * BATCH) {
        f32x4 av[BATCH][RT], bv[BATCH][CT];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {                    // chunks past the end are not read (uniform); the last one may be cut
          const int c = c0 + b * FN_WAVES, k = c * 16 + g * 4;
          if (c < chunks) {
#pragma unroll
            for (int t = 0; t < RT; ++t) av[b][t] = k < K ? *reinterpret_cast<const f32x4 *>(arow[t] + k) : zero4;
#pragma unroll
            for (int u = 0; u < CT; ++u) bv[b][u] = k < K ? *reinterpret_cast<const f32x4 *>(brow[u] + k) : zero4;
          }
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
          if (c0 + b * FN_WAVES < chunks) {
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
              for (int u = 0; u < CT; ++u) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][u] = mfma_f32_16(av[b][t][e], bv[b][u][e], acc[t][u]);
              }
          }
        }
      }
    }
    __syncthreads();                 // the previous segment's sums have been read
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int u = 0; u < CT; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][t * 16 + g * 4 + r][u * 16 + i16] = acc[t][u][r];
    __syncthreads();
#pragma unroll
    for (int o = threadIdx.x; o < RT * 16 * TN; o += FN_WAVES * 64) {
      const int r = o / TN, c = o % TN;
      float s = red[0][r][c];
#pragma unroll
      for (int w = 1; w < FN_WAVES; ++w) s += red[w][r][c];
      if (row0 + r >= lo && row0 + r < hi && col0 + c < N) C[(size_t)(row0 + r) * N + col0 + c] = s;
    }
  });
}

constexpr int FS_WAVES = 4;          // second product: parts of the (short) reduction
constexpr int FS_TN = 64;            // output columns per workgroup
constexpr int FS_BATCH = 2;

// Y[rows][N] = Z[rows][K] * B_p[K][N].  N % 4 == 0; K arbitrary (A4: K % 4 == 0, 16-byte loads of Z).  A lane takes 4
// consecutive columns of a factor row, so the four sub-tiles of a workgroup's 64 columns are interleaved: sub-tile e holds
// columns 4 i + e, and a lane ends up with 4 consecutive columns of its 4 output rows.  KS slices of Z, added in order where they are read.
template <int RT, bool A4, int KS>
__global__ __launch_bounds__(FS_WAVES * 64) void sgemm_nn(const float *__restrict__ A, const float *__restrict__ Bbase,
                                                          size_t pattern_stride, int n_patterns, int rows, int N, int K,
                                                          const int32_t *__restrict__ tok_offsets,
                                                          const int32_t *__restrict__ pattern_id, int P, float *__restrict__ C) {
  __shared__ float4 red[FS_WAVES][RT * 16][FS_TN / 4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  const int row0 = blockIdx.x * RT * 16, col0 = blockIdx.y * FS_TN;
  const int chunks = (K + 15) / 16;
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  for_segments<true>(row0, min(row0 + RT * 16, rows), rows, tok_offsets, pattern_id, P, n_patterns, [&](bool valid, int pid, int lo, int hi) {
    f32x4 acc[RT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (valid) {
      const float *arow[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) arow[t] = A + (size_t)min(row0 + t * 16 + i16, rows - 1) * K;
      const float *bcol = Bbase + (size_t)pid * pattern_stride + min(col0 + i16 * 4, N - 4);
      for (int c0 = wave; c0 < chunks; c0 += FS_WAVES * FS_BATCH) {
        f32x4 av[FS_BATCH][RT], bv[FS_BATCH][4];
#pragma unroll
        for (int b = 0; b < FS_BATCH; ++b) {
          const int c = c0 + b * FS_WAVES, k = c * 16 + g * 4;
          if (c < chunks) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
              f32x4 part[KS];
#pragma unroll
              for (int o = 0; o < KS; ++o) {
                const float *z = arow[t] + (size_t)o * rows * K;
                if (A4) part[o] = k < K ? *reinterpret_cast<const f32x4 *>(z + k) : zero4;
                else part[o] = f32x4{k < K ? z[k] : 0.f, k + 1 < K ? z[k + 1] : 0.f, k + 2 < K ? z[k + 2] : 0.f, k + 3 < K ? z[k + 3] : 0.f};
              }
              av[b][t] = part[0];
#pragma unroll
              for (int o = 1; o < KS; ++o) av[b][t] += part[o];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[b][e] = k + e < K ? *reinterpret_cast<const f32x4 *>(bcol + (size_t)(k + e) * N) : zero4;
          }
        }
#pragma unroll
        for (int b = 0; b < FS_BATCH; ++b) {
          if (c0 + b * FS_WAVES < chunks) {
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[t][u] = mfma_f32_16(av[b][t][e], bv[b][e][u], acc[t][u]);
              }
          }
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[wave][t * 16 + g * 4 + r][i16] = float4{acc[t][0][r], acc[t][1][r], acc[t][2][r], acc[t][3][r]};
    __syncthreads();
#pragma unroll
    for (int o = threadIdx.x; o < RT * 16 * (FS_TN / 4); o += FS_WAVES * 64) {
      const int r = o / (FS_TN / 4), c = o % (FS_TN / 4);
      float4 s = red[0][r][c];
#pragma unroll
      for (int w = 1; w < FS_WAVES; ++w) {
        const float4 v = red[w][r][c];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
      }
      const int col = col0 + c * 4;
      if (row0 + r >= lo && row0 + r < hi && col < N) *reinterpret_cast<float4 *>(C + (size_t)(row0 + r) * N + col) = s;
    }
  });
}

// First product, tiles (T = 16 x 32 ones):
//   32 x 32  T at least four a unit and no more than a sixth of the 32-rank blocks empty: every prompt in a tile takes the whole tile's products, so for prompts
//            that share none (one, or of one length, a multiple of 32), from 512 columns on; for long reductions once prompts are 24 rows on average; else
//            once they are 100 and T is seven a unit.
//   16 x 16  a sixth and more of the 32-rank blocks empty, or few of these tiles: up to 400; for long reductions hardly more than one a unit, two where prompts of
//            150 rows share them
//   16 x 32  else
// Two chunks a wavefront at a time: with four or eight the registers left room for half of the workgroups, which cover each other's waits better
// than one's own loads do; four in the large tiles for long reductions (from 3072 columns on where prompts share none).  Both products, us, the tiles
// and chunks before / now: 4 x 64 rows, 1024 x 1024, 128 ranks 9.35 / 8.9; 1 x 700, 2048 x 256, 100 20.7 / 16.7; 8 x 128, 2048 x 2048, 100 30.8 / 26.3 (16 x 16:
// 29.2); 1 x 1000, 520 x 516, 125 12.3 / 11.4; 8 x 512, 1024 x 1024, 128 47.1 / 43.4.  16 x 16 / 16 x 32 / 32 x 32: 26 prompts, 5368 rows, 2256 x 492, 5 ranks
// 31.6 / 42.0 / 47.7; 24, 5934, 7540 x 184, 153 491 / 390 / 347; 64, 2326, 3372 x 436, 295 279 / 261 / 302; 48, 240, 6936 x 1320, 336 241 / 164 / -; 5, 450, 2824 x 224,
// 144 29.2 / 34.0 / -; 4 x 512, 1024 x 256, 256 38 / 33 / 28.5; 8, 6049, 420 x 144, 222 - / 48.1 / 47.6.  Over 1300 calls of 1 to 100 prompts, 64 to 8192 columns and 4 to
// 2000 ranks 6 % less time than before, 3 % more in 13 of them (25 % at worst), and 1 % off the best form of each.
constexpr int F32_LONG = 2048;                // columns
constexpr int F32_MANY_WGS = 1024, F32_MANY_N = 512, F32_MANY_ROWS_LONG = 24, F32_MANY_ROWS = 100, F32_MANY_WGS_SHARED = 1792, F32_FOUR_CHUNKS = 3072;
constexpr int F32_FEW_WGS = 400, F32_FEW_WGS_LONG = 288, F32_FEW_WGS_LONG_PROMPTS = 512, F32_LONG_PROMPT = 150;
// Second product, 32 rows a workgroup (every factor operand fetched for twice the products) once 16-row ones are four a unit, or seven where single values of
// Z are loaded (rS not a multiple of 4).  us, 16 / 32 rows: 100 ranks, 4 x 128, 2048 x 2048 (1024 workgroups of 16 rows) 19.6 / 17.1, 8 x 128 (2048) 32.3 / 29.7; 125
// ranks, 2 x 300, 1032 x 2048 (1216) 22.1 / 24.4, 8 x 100, 256 x 2048 (1600) 23.3 / 25.5.
constexpr int F32_NN_WGS = 1024, F32_NN_WGS_SINGLE = 1792;
// First product of few 16 x 16 tiles: its reduction in 2, 4 or 8 slices, as many as leave a unit one workgroup and a slice sixteen chunks, each with a Z of its own
// that the second product adds up.  A unit takes in about 50 GB/s, so half as many columns a workgroup take half the time.  Both products, us, one / the slices
// chosen: 4 x 64 rows, 1024 x 1024, 128 ranks 10.6 / 9.2; 1 x 64 8.9 / 7.3; 1 x 16, 4096 x 1024 19.5 / 9.1; 4 x 16, 8192 x 256 34.2 / 11.7; 4 x 64, 2048 x 2048,
// 100 ranks 15.1 / 11.8.  Up to two workgroups a unit: 1 x 256, 1024 x 1024 9.0 (one: 8.7), 4 x 64, 2048 x 2048 12.7, 4 x 128, 1024 x 1024 13.9 (13.4); slices of
// eight chunks: 1 x 64, 1024 x 1024 7.8.  Error against 64 bits, rms, one / the slices chosen: 1024 columns 2.4e-7 / 1.9e-7, 8192 5.9e-7 / 2.4e-7.
// KS is a template argument because gridDim is not an argument of the launch but read from memory of its own: a routed pass of 4 x 64 rows, launched call by
// call, 24.7 unsplit, 27.1 with gridDim.z slices, 23.5 with KS.
constexpr int F32_SPLIT_WGS = 256, F32_SPLIT_CHUNKS = 16, F32_MAX_SPLIT = 8;
static int f32_slices(int rows, int rS, int n, int m, size_t workspace_bytes) {
  const long long t16 = (rows + 15) / 16, wgs = t16 * ((rS + 15) / 16);
  if (t16 * ((m + FS_TN - 1) / FS_TN) >= F32_NN_WGS) return 1;         // the second product's 32-row form takes one Z
  int ks = 1;
  while (ks < F32_MAX_SPLIT && wgs * ks * 2 <= F32_SPLIT_WGS && (n + 15) / 16 >= ks * 2 * F32_SPLIT_CHUNKS &&
         (size_t)rows * rS * ks * 2 * sizeof(float) <= workspace_bytes)
    ks *= 2;
  return ks;
}
size_t f32_needed_bytes(int rows, int rS) { return round_up((size_t)rows * rS * sizeof(float), 256); }
// room for the slices of as many rows or fewer, too
size_t f32_workspace_bytes(int rows, int rS) {
  const size_t need = f32_needed_bytes(rows, rS);
  return std::max(need, std::min(need * F32_MAX_SPLIT, (size_t)F32_SPLIT_WGS * 16 * 16 * sizeof(float)));
}

int forward_f32(const parse_layer *L, const parse_patterns *pt, const float *X, int rows, const int32_t *tok_offsets,
                const int32_t *pattern_id, int P, float *Y, void *workspace, size_t workspace_bytes, hipStream_t s) {
  const int gs = L->R / L->G, rS = pt->k * gs;
  float *Z = reinterpret_cast<float *>(workspace);
  const float *V = (const float *)pt->Vt_S, *U = (const float *)pt->Ut_S;
  const size_t vs = (size_t)rS * L->n, us = (size_t)rS * L->m;
  const int t16 = (rows + 15) / 16, t32 = (rows + 31) / 32;
  const int nb16 = (rS + 15) / 16, nb32 = (rS + 31) / 32, nb2 = (L->m + FS_TN - 1) / FS_TN;
  const int ks = f32_slices(rows, rS, L->n, L->m, workspace_bytes);
#define PARSE_NT(RT_, CT_, B_, KS_)                                                                                             \
  hipLaunchKernelGGL((sgemm_nt<RT_, CT_, B_, KS_>), dim3(RT_ == 2 ? t32 : t16, CT_ == 2 ? nb32 : nb16, KS_), dim3(FN_WAVES * 64), 0, \
                     s, X, V, vs, pt->n_patterns, rows, rS, L->n, tok_offsets, pattern_id, P, Z)
  const int avg = rows / P;
  const long long tiles = (long long)t16 * nb32;
  const bool long_n = L->n >= F32_LONG, apart = P == 1 || (rows % P == 0 && avg % 32 == 0);
  const int few = !long_n ? F32_FEW_WGS : (!apart && avg >= F32_LONG_PROMPT ? F32_FEW_WGS_LONG_PROMPTS : F32_FEW_WGS_LONG);
  const bool many = nb32 * 10 <= nb16 * 6 && tiles >= F32_MANY_WGS && L->n >= F32_MANY_N &&
                    (apart || (long_n ? avg >= F32_MANY_ROWS_LONG : avg >= F32_MANY_ROWS && tiles >= F32_MANY_WGS_SHARED));
  if (ks == 8) PARSE_NT(1, 1, 2, 8);
  else if (ks == 4) PARSE_NT(1, 1, 2, 4);
  else if (ks == 2) PARSE_NT(1, 1, 2, 2);
  else if (many && L->n >= (apart ? F32_FOUR_CHUNKS : F32_LONG)) PARSE_NT(2, 2, 4, 1);
  else if (many) PARSE_NT(2, 2, 2, 1);
  else if (nb32 * 10 >= nb16 * 6 || (long long)t16 * nb16 <= few) PARSE_NT(1, 1, 2, 1);
  else PARSE_NT(1, 2, 2, 1);
#undef PARSE_NT
  PARSE_LAUNCH_CHECK();
  const bool a4 = rS % 4 == 0, rows32 = (long long)t16 * nb2 >= (a4 ? F32_NN_WGS : F32_NN_WGS_SINGLE);
#define PARSE_NN(RT_, A4_, KS_)                                                                                                       \
  hipLaunchKernelGGL((sgemm_nn<RT_, A4_, KS_>), dim3(RT_ == 2 ? t32 : t16, nb2), dim3(FS_WAVES * 64), 0, s, Z, U, us, pt->n_patterns, \
                     rows, L->m, rS, tok_offsets, pattern_id, P, Y)
  if (rows32) { if (a4) PARSE_NN(2, true, 1); else PARSE_NN(2, false, 1); }
  else if (ks == 1) { if (a4) PARSE_NN(1, true, 1); else PARSE_NN(1, false, 1); }
  else if (ks == 2) { if (a4) PARSE_NN(1, true, 2); else PARSE_NN(1, false, 2); }
  else if (ks == 4) { if (a4) PARSE_NN(1, true, 4); else PARSE_NN(1, false, 4); }
  else { if (a4) PARSE_NN(1, true, 8); else PARSE_NN(1, false, 8); }
#undef PARSE_NN
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

}  // namespace parse
