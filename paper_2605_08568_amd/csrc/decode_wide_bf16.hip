// a7 for more than 32 sequences (a loaded server): the same two products as decode_bf16.hip over panels of 32 sequences, but a
// group selected by any sequence of up to DW_MAXP panels is streamed ONCE and applied to all of them, instead of once per
// panel.  Launches per call:
//   wide_prepare  the plan (per layer: groups in use, a 32-sequence mask per group and panel) and x in operand order
//   wide_z        CB rank blocks x a slice of the reduction per workgroup, all panels: fp32 partial sums, or z
//   wide_zsum     adds the slices in slice order, masks, rounds to bf16 (only when the reduction is cut)
//   wide_y        CB column blocks per workgroup, all used reduction blocks, all panels
// Both products keep every operand in operand order, so a wavefront loads 1 KiB per instruction straight into registers:
// per reduction step CB factor operands and NT token operands feed CB * NT matrix instructions.  The four wavefronts of a
// workgroup take every fourth step and share nothing until their sums meet in LDS: no staging, no barrier in the loop; what
// is in flight is DEPTH steps per wavefront (about 40 KiB; one wavefront per SIMD, so the registers are there).
// Bound by HBM for the factors and by what a compute unit can take in: CB + NT KiB per step, of which NT are re-read by every
// workgroup -- hence the largest CB that still gives every unit one workgroup.
// Measured, MLP of a 4096 x 11008 block (20 groups of 128 ranks), 150 sequences, six patterns: wide_z 18-20 us for gate+up and
// for down, wide_y 28 and 14 us, 100 us a step; five panels one after the other took 313-335 us.
// No atomics on floating point; fixed order of all sums: same inputs, same bits.
#include <algorithm>

#include "prefill_common.hpp"

namespace parse {

bool decode_supported(const parse_layer *L);   // what a panel at a time takes

constexpr int DW_MAXP = 6;                 // panels of 32 sequences a pass covers
constexpr int DW_MAX_LAYERS = 4;
constexpr int DW_MAXG = 64;
constexpr int DW_WAVES = 4, DW_THREADS = DW_WAVES * 64;
constexpr int DW_PLAN_WORDS = 128 + DW_MAXP * 64;      // [0] count, [1..64] used groups, [128 + 64 p + g] mask of panel p, group g
constexpr int DW_ZCB = 2;                  // rank blocks per wide_z workgroup
constexpr int DW_UNITS = 256;              // workgroups wanted per launch
constexpr int DW_MAX_KS = 8;
constexpr int DW_ESTRIDE = 66;             // floats between accumulator rows in LDS: the row-wise read-out is conflict-free

struct DwLayer {
  const uint16_t *Vt, *Ut;
  uint16_t *y;
  uint16_t *zf;              // [panel][R/16] operands of 1 KiB
  float *zpart;              // [R/32][KS][panel][16][64]
  int32_t *plan;
  const int32_t *subsets;
  int stride, k, n_patterns;
  int R, G, gs, m;
  int z_first, s_first, y_first;   // first workgroup in wide_z / first wavefront in wide_zsum / first workgroup in wide_y
};
struct DwArgs {
  DwLayer L[DW_MAX_LAYERS];
  int n_layers;
  const uint16_t *x;         // [B][n]
  uint16_t *xo;              // [panel][n/16] operands of 1 KiB
  const int32_t *pattern_id;
  int B, n, KS, panels;
};

// grid = layers + workgroups that reorder x, 256 threads
__global__ __launch_bounds__(DW_THREADS) void wide_prepare(DwArgs a) {
  if ((int)blockIdx.x < a.n_layers) {
    const DwLayer &ly = a.L[blockIdx.x];
    __shared__ uint32_t gmask[DW_MAXP][DW_MAXG];
    for (int i = threadIdx.x; i < DW_MAXP * DW_MAXG; i += DW_THREADS) gmask[i / DW_MAXG][i % DW_MAXG] = 0u;
    __syncthreads();
    for (int s = threadIdx.x; s < a.B; s += DW_THREADS) {
      const int pid = a.pattern_id[s];
      if (pid < 0 || pid >= ly.n_patterns) continue;
      for (int i = 0; i < ly.k; ++i) {
        const int g = ly.subsets[(size_t)pid * ly.stride + i];
        if (g >= 0 && g < ly.G) atomicOr(&gmask[s >> 5][g], 1u << (s & 31));
      }
    }
    __syncthreads();
    if (threadIdx.x < 64) {
      const int lane = threadIdx.x;
      uint32_t any = 0u;
      for (int p = 0; p < DW_MAXP; ++p) any |= gmask[p][lane];
      const unsigned long long votes = __ballot(lane < ly.G && any != 0u);
      if ((votes >> lane) & 1ull) ly.plan[1 + __popcll(votes & ((1ull << lane) - 1ull))] = lane;
      if (lane == 0) ly.plan[0] = __popcll(votes);
    }
    for (int i = threadIdx.x; i < DW_MAXP * DW_MAXG; i += DW_THREADS) ly.plan[128 + i] = (int32_t)gmask[i / DW_MAXG][i % DW_MAXG];
    return;
  }
  // x in operand order: piece (panel, kb, q, j) = x[panel*32 + j][kb*16 + q*8 ..+7]; sequences past the last give zeros
  const int nkb = a.n / 16;
  const int total = a.panels * nkb * 64;
  for (int o = ((int)blockIdx.x - a.n_layers) * DW_THREADS + threadIdx.x; o < total; o += ((int)gridDim.x - a.n_layers) * DW_THREADS) {
    // neighbouring threads read neighbouring pieces of a row
    const int q2 = o % (nkb * 2), row = o / (nkb * 2);
    u32x4 v = {0, 0, 0, 0};
    if (row < a.B) v = *reinterpret_cast<const u32x4 *>(a.x + (size_t)row * a.n + q2 * 8);
    *reinterpret_cast<u32x4 *>((char *)a.xo + (((size_t)(row >> 5) * nkb + (q2 >> 1)) * 64 + (q2 & 1) * 32 + (row & 31)) * 16) = v;
  }
}

constexpr int dw_depth(int CB, int NT) { return 40 / (CB + NT) < 4 ? 4 : (40 / (CB + NT) > 8 ? 8 : 40 / (CB + NT)); }

// The reduction loop of both products: steps first, first + DW_WAVES, ... (cnt of them); f(step, i) / t(step, p) = address
// of factor operand i / token operand p.
template <int CB, int NT, class F, class T>
__device__ __forceinline__ void wide_loop(f32x16 (&acc)[CB][NT], int cnt, F f, T t) {
  constexpr int D = dw_depth(CB, NT);
  u32x4 fr[D][CB], tr[D][NT];
#pragma unroll
  for (int i = 0; i < CB; ++i)
#pragma unroll
    for (int p = 0; p < NT; ++p)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][p][e] = 0.f;
  if (cnt <= 0) return;
#pragma unroll
  for (int d = 0; d < D; ++d) {              // steps past the last re-read it (switched off below)
    const int s = min(d, cnt - 1);
#pragma unroll
    for (int i = 0; i < CB; ++i) fr[d][i] = *reinterpret_cast<const u32x4 *>(f(s, i));
#pragma unroll
    for (int p = 0; p < NT; ++p) tr[d][p] = *reinterpret_cast<const u32x4 *>(t(s, p));
  }
  int s0 = 0;
  for (; s0 + D <= cnt; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int p = 0; p < NT; ++p)
          acc[i][p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[d][i]), as_bf16x8(tr[d][p]), acc[i][p], 0, 0, 0);
      const int s = min(s0 + d + D, cnt - 1);
#pragma unroll
      for (int i = 0; i < CB; ++i) fr[d][i] = *reinterpret_cast<const u32x4 *>(f(s, i));
#pragma unroll
      for (int p = 0; p < NT; ++p) tr[d][p] = *reinterpret_cast<const u32x4 *>(t(s, p));
    }
  }
#pragma unroll
  for (int d = 0; d < D - 1; ++d) {
    if (s0 + d < cnt) {                      // uniform
#pragma unroll
      for (int i = 0; i < CB; ++i)
#pragma unroll
        for (int p = 0; p < NT; ++p)
          acc[i][p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[d][i]), as_bf16x8(tr[d][p]), acc[i][p], 0, 0, 0);
    }
  }
}

// lane (j, q) holds s[e] = ranks 8*(e/4) + 4*q + e%4 of sequence j of rank block rb: mask, round, store as two z operands
__device__ __forceinline__ void wide_store_z(const float (&s)[16], uint32_t mask, int lane, char *zf, int rb) {
  const bool member = (mask >> (lane & 31)) & 1u;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = member ? cvt_pk_bf16(s[h * 8 + 2 * e], s[h * 8 + 2 * e + 1]) : 0u;
    const u32x2 sx = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
    const u32x2 sy = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
    *reinterpret_cast<u32x4 *>(zf + (size_t)(rb * 2 + h) * 1024 + lane * 16) = u32x4{sx[0], sy[0], sx[1], sy[1]};
  }
}

// grid: layers x rank blocks in units of DW_ZCB (numbered over the blocks in use; the rest leaves) x KS slices
template <int NT>
__global__ __launch_bounds__(DW_THREADS, 1) void wide_z(DwArgs a) {
  constexpr int CB = DW_ZCB;
  int li = 0;
#pragma unroll
  for (int i = 1; i < DW_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].z_first) ? 1 : 0;
  const DwLayer &ly = a.L[li];
  const int KS = a.KS, bid = blockIdx.x - ly.z_first;
  const int sl = bid % KS, i0 = bid / KS * CB;
  const int bpg = ly.gs / 32;                          // rank blocks per group
  const int nused = min(max(ly.plan[0], 0), ly.G) * bpg;
  if (i0 >= nused) return;
  __shared__ float red[2][DW_WAVES][CB][16][64];       // panels alternate: one barrier each
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nkb = a.n / 16;
  const int k0 = (int)(((long long)nkb * sl) / KS), k1 = (int)(((long long)nkb * (sl + 1)) / KS);
  int rb[CB];
#pragma unroll
  for (int i = 0; i < CB; ++i) {                       // blocks past the last re-read it (not stored)
    const int at = min(i0 + i, nused - 1);
    rb[i] = ly.plan[1 + at / bpg] * bpg + at % bpg;
  }
  const char *V = (const char *)ly.Vt + (size_t)(k0 + wave) * 1024 + lane * 16;
  const char *X = (const char *)a.xo + (size_t)(k0 + wave) * 1024 + lane * 16;
  f32x16 acc[CB][NT];
  wide_loop<CB, NT>(acc, (k1 - k0 - wave + DW_WAVES - 1) / DW_WAVES,
                    [&](int s, int i) { return V + ((size_t)rb[i] * nkb + s * DW_WAVES) * 1024; },
                    [&](int s, int p) { return X + ((size_t)p * nkb + s * DW_WAVES) * 1024; });
#pragma unroll
  for (int p = 0; p < NT; ++p) {
#pragma unroll
    for (int i = 0; i < CB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) red[p & 1][wave][i][e][lane] = acc[i][p][e];
    __syncthreads();
    // the four sums of every value, in wavefront order
    if (KS > 1) {
#pragma unroll
      for (int i = 0; i < CB; ++i) {
        const int at = min(i0 + i, nused - 1);
        float *dst = ly.zpart + (((size_t)(ly.plan[1 + at / bpg] * bpg + at % bpg) * KS + sl) * NT + p) * 1024;
        if (i0 + i < nused) {
#pragma unroll
          for (int u = 0; u < 1024 / DW_THREADS; ++u) {
            const int v = u * DW_THREADS + (int)threadIdx.x;
            float s = (&red[p & 1][0][i][0][0])[v];
#pragma unroll
            for (int w = 1; w < DW_WAVES; ++w) s += (&red[p & 1][w][i][0][0])[v];
            dst[v] = s;
          }
        }
      }
    } else if (wave < CB && i0 + wave < nused) {
      const int g = ly.plan[1 + (i0 + wave) / bpg], myrb = g * bpg + (i0 + wave) % bpg;
      float s[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        s[e] = red[p & 1][0][wave][e][lane];
#pragma unroll
        for (int w = 1; w < DW_WAVES; ++w) s[e] += red[p & 1][w][wave][e][lane];
      }
      wide_store_z(s, (uint32_t)ly.plan[128 + p * 64 + g], lane, (char *)ly.zf + (size_t)p * (ly.R / 16) * 1024, myrb);
    }
  }
}

// one wavefront per (used rank block, panel)
__global__ __launch_bounds__(DW_THREADS) void wide_zsum(DwArgs a) {
  const int id = (int)blockIdx.x * DW_WAVES + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int li = 0;
#pragma unroll
  for (int i = 1; i < DW_MAX_LAYERS; ++i) li += (i < a.n_layers && id >= a.L[i].s_first) ? 1 : 0;
  const DwLayer &ly = a.L[li];
  const int at = (id - ly.s_first) / a.panels, p = (id - ly.s_first) % a.panels;
  const int bpg = ly.gs / 32;
  if (at >= min(max(ly.plan[0], 0), ly.G) * bpg) return;
  const int lane = threadIdx.x & 63;
  const int g = ly.plan[1 + at / bpg], rb = g * bpg + at % bpg;
  const uint32_t mask = (uint32_t)ly.plan[128 + p * 64 + g];
  float s[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) s[e] = 0.f;
  const float *src = ly.zpart + ((size_t)rb * a.KS * a.panels + p) * 1024 + lane;
  const size_t step = (size_t)a.panels * 1024;
#pragma unroll 2
  for (int o = 0; o < a.KS; ++o) {
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] += src[o * step + e * 64];
  }
  wide_store_z(s, mask, lane, (char *)ly.zf + (size_t)p * (ly.R / 16) * 1024, rb);
}

// grid: layers x column blocks in units of CB
template <int CB, int NT>
__global__ __launch_bounds__(DW_THREADS, 1) void wide_y(DwArgs a) {
  int li = 0;
#pragma unroll
  for (int i = 1; i < DW_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].y_first) ? 1 : 0;
  const DwLayer &ly = a.L[li];
  __shared__ float red[DW_WAVES][CB][16][DW_ESTRIDE];
  __shared__ int32_t kb_list[1024];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int kpg = ly.gs / 16, ncb = ly.m / 32, m = ly.m;
  const int total = min(max(ly.plan[0], 0), ly.G) * kpg;           // <= R / 16 <= 1024
  for (int i = threadIdx.x; i < total; i += DW_THREADS) kb_list[i] = ly.plan[1 + i / kpg] * kpg + i % kpg;
  __syncthreads();
  const int c0 = ((int)blockIdx.x - ly.y_first) * CB;
  const char *U = (const char *)ly.Ut + lane * 16, *Z = (const char *)ly.zf + lane * 16;
  int cb[CB];
#pragma unroll
  for (int i = 0; i < CB; ++i) cb[i] = min(c0 + i, ncb - 1);       // blocks past the end re-read the last one (not stored)
  const size_t zstep = (size_t)(ly.R / 16);
  f32x16 acc[CB][NT];
  wide_loop<CB, NT>(acc, (total - wave + DW_WAVES - 1) / DW_WAVES,
                    [&](int s, int i) { return U + ((size_t)kb_list[wave + s * DW_WAVES] * ncb + cb[i]) * 1024; },
                    [&](int s, int p) { return Z + (p * zstep + kb_list[wave + s * DW_WAVES]) * 1024; });
#pragma unroll
  for (int p = 0; p < NT; ++p) {
#pragma unroll
    for (int i = 0; i < CB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) red[wave][i][e][lane] = acc[i][p][e];
    __syncthreads();
    // thread = four consecutive columns of a sequence (eight threads a row's 32 columns): sums in wavefront order
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const int quad = threadIdx.x & 7, j = threadIdx.x >> 3, seq = p * 32 + j;
      float s[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = (quad >> 1) * 4 + e, ln = (quad & 1) * 32 + j;
        s[e] = red[0][i][row][ln];
#pragma unroll
        for (int w = 1; w < DW_WAVES; ++w) s[e] += red[w][i][row][ln];
      }
      if (seq < a.B && c0 + i < ncb)
        *reinterpret_cast<u32x2 *>(ly.y + (size_t)seq * m + (c0 + i) * 32 + quad * 4) = u32x2{cvt_pk_bf16(s[0], s[1]), cvt_pk_bf16(s[2], s[3])};
    }
    __syncthreads();
  }
}

// slices of the first product's reduction: one workgroup per compute unit, at least 16 steps each
static int wide_slices(const parse_layer *layers, int n_layers) {
  int units = 0;
  for (int l = 0; l < n_layers; ++l) units += (layers[l].R / 32 + DW_ZCB - 1) / DW_ZCB;
  const int nkb = layers[0].n / 16;
  return std::max(1, std::min({DW_UNITS / std::max(units, 1), nkb / 16, DW_MAX_KS}));
}
static int panels_of(int rows) { return rows / 32 + (rows % 32 != 0); }
// panels of one pass over `rows` sequences: the passes cover about the same number each
static int wide_panels(int rows) {
  const int panels = panels_of(rows), passes = (panels + DW_MAXP - 1) / DW_MAXP;
  return (panels + passes - 1) / passes;
}

// Layers whose factors are worth streaming once for several panels; smaller ones are over in a few launches' latency.
bool decode_wide_supported(const parse_layer *layers, int n_layers) {
  if (n_layers < 1 || n_layers > DW_MAX_LAYERS) return false;
  for (int l = 0; l < n_layers; ++l) {
    const parse_layer *L = &layers[l];
    if (L->G <= 0 || L->R <= 0 || !decode_supported(L) || L->m % 32 != 0 || L->n < 256 || L->R < 256 || L->n != layers[0].n) return false;
  }
  return true;
}

static size_t wide_bytes(const parse_layer *layers, int n_layers, size_t nt) {
  const int ks = wide_slices(layers, n_layers);
  size_t t = round_up((size_t)n_layers * DW_PLAN_WORDS * sizeof(int32_t), 256) + nt * (layers[0].n / 16) * 1024;
  for (int l = 0; l < n_layers; ++l)
    t += nt * (layers[l].R / 16) * 1024 + (ks > 1 ? nt * (layers[l].R / 32) * ks * 4096 : 0);
  return t;
}
// What a call of `rows` sequences takes ...
size_t decode_wide_needed_bytes(const parse_layer *layers, int n_layers, int rows) {
  return wide_bytes(layers, n_layers, (size_t)wide_panels(rows));
}
// ... and what covers every call of up to `rows`: the balanced passes of 193 sequences are shorter than the one pass of 192.
size_t decode_wide_workspace_bytes(const parse_layer *layers, int n_layers, int rows) {
  return wide_bytes(layers, n_layers, (size_t)std::min(panels_of(rows), DW_MAXP));
}

static int wide_pass(DwArgs a, hipStream_t s) {
  int xwgs = std::min(512, (a.panels * (a.n / 16) * 64 + DW_THREADS - 1) / DW_THREADS);
  hipLaunchKernelGGL(wide_prepare, dim3(a.n_layers + xwgs), dim3(DW_THREADS), 0, s, a);
  PARSE_LAUNCH_CHECK();
  int zw = 0, sw = 0, cols = 0;
  for (int l = 0; l < a.n_layers; ++l) {
    a.L[l].z_first = zw; zw += (a.L[l].R / 32 + DW_ZCB - 1) / DW_ZCB * a.KS;
    a.L[l].s_first = sw; sw += a.L[l].R / 32 * a.panels;
    cols += a.L[l].m / 32;
  }
  int cb = 1;                                // column blocks per workgroup: the fewest that need one round of workgroups
  const int most = a.panels >= 6 ? 2 : 3;    // what the accumulators leave room for (256 registers per SIMD lane and 256 more)
  while (cb < most && (cols + cb - 1) / cb > DW_UNITS) ++cb;
  int yw = 0;
  for (int l = 0; l < a.n_layers; ++l) { a.L[l].y_first = yw; yw += (a.L[l].m / 32 + cb - 1) / cb; }
#define PARSE_DW(NT_)                                                                              \
  case NT_:                                                                                        \
    hipLaunchKernelGGL(wide_z<NT_>, dim3(zw), dim3(DW_THREADS), 0, s, a);                          \
    PARSE_LAUNCH_CHECK();                                                                          \
    if (a.KS > 1) {                                                                                \
      hipLaunchKernelGGL(wide_zsum, dim3((sw + DW_WAVES - 1) / DW_WAVES), dim3(DW_THREADS), 0, s, a); \
      PARSE_LAUNCH_CHECK();                                                                        \
    }                                                                                              \
    if (cb == 1) hipLaunchKernelGGL((wide_y<1, NT_>), dim3(yw), dim3(DW_THREADS), 0, s, a);        \
    else if (cb == 2) hipLaunchKernelGGL((wide_y<2, NT_>), dim3(yw), dim3(DW_THREADS), 0, s, a);   \
    else hipLaunchKernelGGL((wide_y<(NT_ < 6 ? 3 : 2), NT_>), dim3(yw), dim3(DW_THREADS), 0, s, a); \
    break
  switch (a.panels) {
    PARSE_DW(1); PARSE_DW(2); PARSE_DW(3); PARSE_DW(4); PARSE_DW(5); PARSE_DW(6);
    default: return PARSE_ESHAPE;
  }
#undef PARSE_DW
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

int forward_decode_wide_bf16(const parse_layer *layers, const parse_patterns *pts, int n_layers, const uint16_t *x, int rows,
                             const int32_t *pattern_id, void *const *Y, void *workspace, hipStream_t s) {
  const int per = wide_panels(rows);
  const int ks = wide_slices(layers, n_layers);
  DwArgs a{};
  a.n_layers = n_layers;
  a.n = layers[0].n;
  a.KS = ks;
  char *ws = reinterpret_cast<char *>(workspace);
  int32_t *plan = reinterpret_cast<int32_t *>(ws);
  ws += round_up((size_t)n_layers * DW_PLAN_WORDS * sizeof(int32_t), 256);
  a.xo = reinterpret_cast<uint16_t *>(ws);
  ws += (size_t)per * (a.n / 16) * 1024;
  for (int l = 0; l < n_layers; ++l) {
    const parse_layer *L = &layers[l];
    DwLayer &d = a.L[l];
    d.Vt = (const uint16_t *)L->Vt; d.Ut = (const uint16_t *)L->Ut;
    d.zf = reinterpret_cast<uint16_t *>(ws);
    ws += (size_t)per * (L->R / 16) * 1024;
    d.zpart = reinterpret_cast<float *>(ws);
    ws += ks > 1 ? (size_t)per * (L->R / 32) * ks * 4096 : 0;
    d.plan = plan + (size_t)l * DW_PLAN_WORDS;
    d.subsets = pts[l].subsets; d.stride = pts[l].subset_stride; d.k = pts[l].k; d.n_patterns = pts[l].n_patterns;
    d.R = L->R; d.G = L->G; d.gs = L->R / L->G; d.m = L->m;
  }
  for (int r0 = 0; r0 < rows; r0 += per * 32) {
    a.B = std::min(rows - r0, per * 32);
    a.panels = (a.B + 31) / 32;
    a.x = x + (size_t)r0 * a.n;
    a.pattern_id = pattern_id + r0;
    for (int l = 0; l < n_layers; ++l) a.L[l].y = (uint16_t *)Y[l] + (size_t)r0 * a.L[l].m;
    const int st = wide_pass(a, s);
    if (st != PARSE_OK) return st;
  }
  return PARSE_OK;
}

}  // namespace parse
