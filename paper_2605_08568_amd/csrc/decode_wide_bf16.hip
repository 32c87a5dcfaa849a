// a7 for more than 32 sequences (a loaded server): the same two products as decode_bf16.hip over panels of 32 sequences, but a
// group selected by any sequence of up to DW_MAXP panels is streamed ONCE and applied to all of them, instead of once per
// panel.  Launches per call:
//   wide_z        the plan (per layer the groups in use, a 32-sequence mask per group and panel), then two rank blocks x a slice of
//                 the reduction per workgroup, all panels: fp32 partial sums, or z
//   wide_zsum     adds the slices in slice order, masks, rounds to bf16 (only when the reduction is cut)
//   wide_y        CB column blocks x NT panels per workgroup, all used reduction blocks
// wide_z is a tile kernel like the prefill's (see prefill_lds_bf16.hip): both operands staged in LDS, the loads between 16x16x32
// products; x is read as it is, row-major.  wide_y keeps every operand in operand order, so a wavefront loads 1 KiB per instruction
// straight into registers: per reduction step CB factor operands and NT token operands feed CB * NT matrix instructions; its four
// wavefronts take every fourth step and share nothing until their sums meet in LDS: no staging, no barrier in the loop; what
// is in flight is DEPTH steps per wavefront (about 40 KiB; one wavefront per SIMD, so the registers are there).
// Bound by HBM for the factors and by what a compute unit can take in: the token operands are re-read by every workgroup.
// Measured, MLP of a 4096 x 11008 block (20 groups of 128 ranks), 150 sequences, six patterns, 100 us a step, three states in turn: wide_z 19.3 us for gate+up
// and 24.0 for down, 5.2 of them until the first slice is there (2.3 for the plan; a launch of its own for it and operands straight into registers, with one more launch
// that brought x into operand order, came to 27-30), then half a microsecond a slice of 28 KiB, which is what a unit takes in where lines from memory are among
// those from the L2 (55 GB/s: 32 KiB outstanding, back in order), 1.6 for the sums; wide_zsum 4.8 each; wide_y 34 us, 24 of them the 467 KiB of factor and 778 KiB of z that
// a unit takes in, and 13.6 us; five panels one after the other took 313-335 us.
// No atomics on floating point; fixed order of all sums: same inputs, same bits.
#include <algorithm>

#include "prefill_common.hpp"

namespace parse {

bool decode_supported(const parse_layer *L);   // what a panel at a time takes
bool past_caches(const parse_layer *layers, int n_layers);   // whether a call's factors are read past the caches

constexpr int DW_MAXP = 6;                 // panels of 32 sequences a pass covers
constexpr int DW_MAX_LAYERS = 4;
constexpr int DW_MAXG = 64;
constexpr int DW_WAVES = 4, DW_THREADS = DW_WAVES * 64;
constexpr int DW_PLAN_WORDS = 128 + DW_MAXP * 64;      // [0] count, [1..64] used groups, [128 + 64 p + g] mask of panel p, group g
constexpr int DW_ZCB = 2;                  // rank blocks per wide_z workgroup
constexpr int DW_UNITS = 256;              // workgroups wanted per launch
constexpr int DW_MAX_KS = 8;
constexpr int DWY_PAST = 3;                // most panels of a wide_y workgroup that reads its factor past the caches
// Tiles of wide_y whose sums meet at a time: 16 KiB each, nine where the registers leave room for one workgroup a compute unit only
constexpr int dw_round(int tiles) { return tiles <= 4 ? tiles : (tiles < 6 ? 4 : (tiles < 9 ? tiles : 9)); }

struct DwLayer {
  const uint16_t *Vt, *Ut;
  uint16_t *y;
  uint16_t *zf;              // [panel][R/16] operands of 1 KiB
  float *zpart;              // [R/16][KS][16 sequences][64][4]
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
  const int32_t *pattern_id;
  int B, n, KS, panels;
  int groups;                // of panels in wide_y
};

constexpr int dw_depth(int CB, int NT) { return 40 / (CB + NT) < 4 ? 4 : (40 / (CB + NT) > 8 ? 8 : 40 / (CB + NT)); }

// The reduction loop of the second product over cnt steps; k(step) = its reduction block, f(block, i) / t(block, p) = address of factor
// operand i / token operand p.
template <int CB, int NT, bool PAST, class K, class F, class T>
__device__ __forceinline__ void wide_loop(f32x16 (&acc)[CB][NT], int cnt, K k, F f, T t) {
  constexpr int D = dw_depth(CB, NT);
  u32x4 fr[D][CB], tr[D][NT];
  auto factor = [](const void *p) { return PAST ? __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p)) : *reinterpret_cast<const u32x4 *>(p); };
#pragma unroll
  for (int i = 0; i < CB; ++i)
#pragma unroll
    for (int p = 0; p < NT; ++p)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][p][e] = 0.f;
  if (cnt <= 0) return;
#pragma unroll
  for (int d = 0; d < D; ++d) {              // steps past the last re-read it (switched off below)
    const int s = k(min(d, cnt - 1));
#pragma unroll
    for (int i = 0; i < CB; ++i) fr[d][i] = factor(f(s, i));
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
      const int s = k(min(s0 + d + D, cnt - 1));
#pragma unroll
      for (int i = 0; i < CB; ++i) fr[d][i] = factor(f(s, i));
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

// lane (j, g) holds ranks 4 g + (0..3) of sequences j (lo) and 16 + j (hi) of a panel: mask, round, pair, store one z operand
__device__ __forceinline__ void wide_store_z(const f32x4v &lo, const f32x4v &hi, uint32_t mask, int lane, char *dst) {
  const u32x2 s0 = __builtin_amdgcn_permlane16_swap(cvt_pk_bf16(lo[0], lo[1]), cvt_pk_bf16(hi[0], hi[1]), false, false);
  const u32x2 s1 = __builtin_amdgcn_permlane16_swap(cvt_pk_bf16(lo[2], lo[3]), cvt_pk_bf16(hi[2], hi[3]), false, false);
  const bool member = (mask >> (lane & 31)) & 1u;      // after the swap the lane's sequence is lane & 31
  *reinterpret_cast<u32x4 *>(dst + lane * 16) = member ? u32x4{s0[0], s1[0], s0[1], s1[1]} : u32x4{0, 0, 0, 0};
}

#define PARSE_DW_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
#define PARSE_DW_GLB_PTR(p) ((const __attribute__((address_space(1))) void *)(p))

// Stages of NT panels' slices (8 KiB of factor, 4 KiB of x per panel): all of the LDS, up to eight: there is little to multiply, what
// counts is how much of the factor stream is on its way.
constexpr int dw_stages(int NT) { return 160 / (8 + 4 * NT) > 8 ? 8 : 160 / (8 + 4 * NT); }
constexpr int DWZ_WAVES = 8, DWZ_THREADS = DWZ_WAVES * 64;   // two per SIMD, whose waits cover each other
static_assert(DW_MAXP * 32 <= 256, "a thread of each 256 looks at one sequence");

// The groups in use and the mask of sequences of every (panel, group), worked out by every workgroup of wide_z in LDS: 1 us of two dependent
// loads and a vote where a launch of its own took 4-5.  The first workgroup of a layer leaves them in memory for the launches that follow.
constexpr int DW_PREP_BYTES = (DW_MAXP + 1) * DW_MAXG * 4;
struct DwUsed {
  const uint32_t *gmask;     // [DW_MAXP][DW_MAXG]
  const int32_t *ids;        // ascending
  int count;
};
__device__ __forceinline__ DwUsed wide_used(const DwArgs &a, const DwLayer &ly, char *lds, bool keep) {
  uint32_t *gmask = reinterpret_cast<uint32_t *>(lds);
  int32_t *ids = reinterpret_cast<int32_t *>(lds) + DW_MAXP * DW_MAXG;
  constexpr int PARTS = DWZ_THREADS / 256;             // threads that share a sequence's groups (at most 192 sequences)
  const int s = threadIdx.x & 255, part = threadIdx.x >> 8, lane = threadIdx.x & 63;
  const int pid = s < a.B ? a.pattern_id[s] : -1;
  for (int i = threadIdx.x; i < DW_MAXP * DW_MAXG; i += DWZ_THREADS) gmask[i] = 0u;
  __syncthreads();
  if (pid >= 0 && pid < ly.n_patterns) {
    const int32_t *sub = ly.subsets + (size_t)pid * ly.stride;
    for (int i0 = part; i0 < ly.k; i0 += 8 * PARTS) {
      int g[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) g[u] = sub[min(i0 + u * PARTS, ly.k - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i0 + u * PARTS < ly.k && g[u] >= 0 && g[u] < ly.G) atomicOr(&gmask[(s >> 5) * DW_MAXG + g[u]], 1u << (s & 31));
    }
  }
  __syncthreads();
  uint32_t any = 0u;
#pragma unroll
  for (int p = 0; p < DW_MAXP; ++p) any |= gmask[p * DW_MAXG + lane];
  const unsigned long long votes = __ballot(any != 0u);          // groups below G only
  const int count = __popcll(votes), at = __popcll(votes & ((1ull << lane) - 1ull));
  if (threadIdx.x < 64 && any != 0u) ids[at] = lane;
  if (keep) {
    if (threadIdx.x < 64 && any != 0u) ly.plan[1 + at] = lane;
    if (threadIdx.x == 0) ly.plan[0] = count;
    for (int i = threadIdx.x; i < DW_MAXP * DW_MAXG; i += DWZ_THREADS) ly.plan[128 + i] = (int32_t)gmask[i];
  }
  __syncthreads();
  return DwUsed{gmask, ids, count};
}

// grid: layers x rank blocks in units of DW_ZCB (numbered over the blocks in use; the rest leaves) x KS slices.
// Slices of 64 reduction indices in a ring: slice kt + STAGES is requested once slice kt has been read by everybody.  A wavefront owns
// 16 of the 64 ranks and half of the panels (the middle one of an odd number twice), so nothing is added between wavefronts.  A last slice of fewer than 64 indices re-reads the
// last operands in their place, and both are cleared before they are multiplied (an infinite weight times zero is no number).
template <int NT, bool PAST>
__global__ __launch_bounds__(DWZ_THREADS, 2) void wide_z(DwArgs a) {
  constexpr int CB = DW_ZCB, PW = (NT + 1) / 2, TB = 2 * PW, STAGES = dw_stages(NT);
  constexpr int F_BYTES = CB * 4096, STAGE_BYTES = F_BYTES + NT * 4096;
  constexpr int LT = (4 * NT + DWZ_WAVES - 1) / DWZ_WAVES, L = 1 + LT, H = L / 2;   // loads of a wavefront per slice; after its last half
  static_assert(F_BYTES == DWZ_WAVES * 1024 && (STAGES - 2) * L + H < 64, "vmcnt is a 6-bit count");
  int li = 0;
#pragma unroll
  for (int i = 1; i < DW_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].z_first) ? 1 : 0;
  const DwLayer &ly = a.L[li];
  const int KS = a.KS, bid = blockIdx.x - ly.z_first;
  const int sl = bid % KS, i0 = bid / KS * CB;
  const int bpg = ly.gs / 32;                          // rank blocks per group
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const DwUsed use = wide_used(a, ly, smem, bid == 0);
  const int nused = use.count * bpg;
  if (i0 >= nused) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int j = lane & 15, g = lane >> 4;
  const int n = a.n, nkb = n / 16, slices = (n + 63) / 64;
  const int kt0 = (int)(((long long)slices * sl) / KS), nk = (int)(((long long)slices * (sl + 1)) / KS) - kt0;
  const bool ragged = (n & 63) != 0 && kt0 + nk == slices;
  const int wr = wave & 3, p0 = wave >> 2 ? NT - PW : 0;                 // its 16 ranks, its first panel
  auto rank_block = [&](int i, int &grp) -> int {                        // blocks past the last one re-read it (not stored)
    const int at = min(i0 + i, nused - 1);
    grp = __builtin_amdgcn_readfirstlane(use.ids[at / bpg]);
    return grp * bpg + at % bpg;
  };
  int grp, lgrp;
  const int rb = rank_block(wr >> 1, grp), lrb = rank_block(wave >> 2, lgrp);
  uint32_t mask[PW];                                   // of its panels, for z that is stored here
#pragma unroll
  for (int p = 0; p < PW; ++p) mask[p] = __builtin_amdgcn_readfirstlane(use.gmask[(p0 + p) * DW_MAXG + grp]);
  __syncthreads();                                     // the lists are read: the stages take their place

  // sources: one of the eight factor operands of a slice, and of its groups of 8 rows of x every eighth (the last one again where
  // they do not divide: the same data to the same place)
  const uint32_t loff = lane * 16;
  const char *V = (const char *)ly.Vt + ((size_t)lrb * nkb + kt0 * 4 + wr) * 1024;
  const char *xs[LT];
  int chunk[LT], xdst[LT];                             // 16-byte piece of a row's 128 bytes; place of the group in the slice
#pragma unroll
  for (int i = 0; i < LT; ++i) {
    const int grp8 = min(i * DWZ_WAVES + wave, 4 * NT - 1), rr = grp8 * 8 + (lane >> 3);
    xdst[i] = F_BYTES + grp8 * 1024;
    chunk[i] = (lane & 7) ^ ((rr >> 1) & 7);           // LDS place: row rr, slot lane % 8; it holds chunk slot ^ swizzle of the row
    xs[i] = (const char *)a.x + (size_t)min(rr, a.B - 1) * n * 2 + (size_t)kt0 * 128;  // rows past the last sequence re-read it
  }
  int issued = 0, dst = 0;
  // load q of L of the next slice; the last one moves on.  PAST: the factor past the caches (aux 2)
  auto load = [&](int q, bool steady) {
    const bool cut = !steady && ragged && issued == nk - 1;              // uniform
    if (q == 0) {
      const int over = cut ? max((kt0 + issued) * 4 + wr - (nkb - 1), 0) : 0;
      __builtin_amdgcn_global_load_lds(PARSE_DW_GLB_PTR(V - over * 1024 + loff), PARSE_DW_LDS_PTR(smem + dst + wave * 1024), 16, 0, PAST ? 2 : 0);
    } else {
      const int i = q - 1;
      const int c = cut ? min(chunk[i], n / 8 - 1 - (kt0 + issued) * 8) : chunk[i];
      __builtin_amdgcn_global_load_lds(PARSE_DW_GLB_PTR(xs[i] + c * 16), PARSE_DW_LDS_PTR(smem + dst + xdst[i]), 16, 0, 0);
      xs[i] += 128;
    }
    if (q == L - 1) {
      V += 4096;
      dst = dst + STAGE_BYTES == STAGES * STAGE_BYTES ? 0 : dst + STAGE_BYTES;
      ++issued;
    }
  };
  // LDS operands: lane (j, g) reads reduction indices 8 g .. 8 g + 7 of row j of a 16-row block
  const int f_lane = (wr >> 1) * 4096 + (g >> 1) * 1024 + (g & 1) * 512 + (wr & 1) * 256 + j * 16;
  const int t_lane = F_BYTES + p0 * 4096 + j * 128 + ((g ^ ((j >> 1) & 7)) * 16);
  u32x4 fr[2], tr[2][TB];
  int src = 0;
  auto read_half = [&](int half) {
    fr[half] = *reinterpret_cast<const u32x4 *>(smem + src + f_lane + half * 2048);
    const char *tb = smem + src + (t_lane ^ (half * 64));
#pragma unroll
    for (int t = 0; t < TB; ++t) tr[half][t] = *reinterpret_cast<const u32x4 *>(tb + t * 2048);
  };
  auto settle = [&](int half) {                        // the reads have arrived before anything else is issued (see gemm_lds)
    asm volatile("" ::"v"(fr[half]));
#pragma unroll
    for (int t = 0; t < TB; ++t) asm volatile("" ::"v"(tr[half][t]));
    __builtin_amdgcn_sched_barrier(0);
  };
  // Four sums of a value, added at the end: the two halves of even and of odd slices.  One alone is farther from the exact value (z rounded
  // the other way to bf16, 4096 x 4096 ranks: 223 values in a million with one, 129 with four; 0.5 us of 113).
  f32x4v acc[4][TB];
#pragma unroll
  for (int t = 0; t < TB; ++t) acc[0][t] = acc[1][t] = acc[2][t] = acc[3][t] = f32x4v{0.f, 0.f, 0.f, 0.f};
  auto products = [&](int odd, int half, int q0, int q1, bool more, bool steady) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      f32x4v &sum = acc[odd * 2 + half][t];
      sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fr[half]), as_bf16x8(tr[half][t]), sum, 0, 0, 0);
#pragma unroll
      for (int q = q0; q < q1; ++q)
        if (t == (q - q0) * TB / (q1 - q0)) {
          __builtin_amdgcn_sched_barrier(0);
          if (more) load(q, steady);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto clear_past = [&](int half, int kt) {            // reduction indices past the last one
    if ((kt0 + kt) * 64 + half * 32 + g * 8 >= n) {
      fr[half] = u32x4{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < TB; ++t) tr[half][t] = u32x4{0, 0, 0, 0};
    }
  };
  auto slice = [&](bool steady, int odd, int kt) {
    const bool cut = !steady && ragged && kt == nk - 1;
    settle(0);
    read_half(1);
    if (cut) clear_past(0, kt);
    products(odd, 0, H, L, steady || kt - 1 + STAGES < nk, steady);
    settle(1);
    if (cut) clear_past(1, kt);
    if (steady || kt + 1 < nk) {                       // slice kt + 1 has landed for everybody, slice kt has been read by everybody
      if (steady) wait_vm<(STAGES - 2) * L>(); else wait_slices<STAGES - 2, L>(min(kt + STAGES - 1, nk - 1) - (kt + 1));
      wg_barrier();
      src = src + STAGE_BYTES == STAGES * STAGE_BYTES ? 0 : src + STAGE_BYTES;
      read_half(0);
    }
    products(odd, 1, 0, H, steady || kt + STAGES < nk, steady);
  };
#pragma unroll
  for (int s = 0; s < STAGES; ++s) {
    if (s < nk) {
#pragma unroll
      for (int q = 0; q < (s == STAGES - 1 ? H : L); ++q) load(q, false);
    }
  }
  if (nk >= STAGES) wait_vm<(STAGES - 2) * L + H>(); else wait_vm<0>();
  wg_barrier();
  read_half(0);
  int kt = 0;
  for (; kt + STAGES + 2 < nk; kt += 2) {              // what they request are whole slices
    slice(true, 0, kt);
    slice(true, 1, kt + 1);
  }
  for (; kt < nk; kt += 2) {
    slice(false, 0, kt);
    if (kt + 1 < nk) slice(false, 1, kt + 1);
  }

  if (i0 + (wr >> 1) >= nused) return;
#pragma unroll
  for (int t = 0; t < TB; ++t) acc[0][t] = (acc[0][t] + acc[1][t]) + (acc[2][t] + acc[3][t]);
  const int rb16 = rb * 2 + (wr & 1), skip = wave >> 2 ? 2 * PW - NT : 0;        // the other half stores the middle panel
  if (KS > 1) {
    float *dst4 = ly.zpart + (((size_t)rb16 * KS + sl) * NT + p0) * 512 + lane * 4;
#pragma unroll
    for (int t = 0; t < TB; ++t)
      if (t >= 2 * skip) *reinterpret_cast<f32x4v *>(dst4 + t * 256) = acc[0][t];
  } else {
#pragma unroll
    for (int p = 0; p < PW; ++p)
      if (p >= skip)
        wide_store_z(acc[0][2 * p], acc[0][2 * p + 1], mask[p], lane, (char *)ly.zf + ((size_t)(p0 + p) * (ly.R / 16) + rb16) * 1024);
  }
}

// one wavefront per (16 used ranks, panel)
__global__ __launch_bounds__(DW_THREADS) void wide_zsum(DwArgs a) {
  const int id = (int)blockIdx.x * DW_WAVES + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int li = 0;
#pragma unroll
  for (int i = 1; i < DW_MAX_LAYERS; ++i) li += (i < a.n_layers && id >= a.L[i].s_first) ? 1 : 0;
  const DwLayer &ly = a.L[li];
  const int at = (id - ly.s_first) / a.panels, p = (id - ly.s_first) % a.panels;
  const int bpg = ly.gs / 16;
  if (at >= min(max(ly.plan[0], 0), ly.G) * bpg) return;
  const int lane = threadIdx.x & 63;
  const int g = ly.plan[1 + at / bpg], rb16 = g * bpg + at % bpg;
  const uint32_t mask = (uint32_t)ly.plan[128 + p * 64 + g];
  const size_t step = (size_t)a.panels * 512;
  const float *src = ly.zpart + (size_t)rb16 * a.KS * step + p * 512 + lane * 4;
  f32x4v lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int o = 0; o < a.KS; ++o) {
    lo += *reinterpret_cast<const f32x4v *>(src + o * step);
    hi += *reinterpret_cast<const f32x4v *>(src + o * step + 256);
  }
  wide_store_z(lo, hi, mask, lane, (char *)ly.zf + ((size_t)p * (ly.R / 16) + rb16) * 1024);
}

// grid: layers x groups of NT panels x column blocks in units of CB (their number rounded up to whole rounds of the dies, so that the groups of one
// column block run on one die and its factor comes from memory once).  The last group of panels ends with the last panel: the ones it shares with the
// group before are computed by both and stored once.
template <int CB, int NT, bool PAST>
__global__ __launch_bounds__(DW_THREADS, 1) void wide_y(DwArgs a) {
  int li = 0;
#pragma unroll
  for (int i = 1; i < DW_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].y_first) ? 1 : 0;
  const DwLayer &ly = a.L[li];
  constexpr int TILES = CB * NT, ROUND = dw_round(TILES);          // tiles whose sums meet in LDS at a time
  __shared__ __attribute__((aligned(16))) f32x4v red[ROUND][DW_WAVES][4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int kpg = ly.gs / 16, ncb = ly.m / 32, m = ly.m;
  // the blocks in use, counted through: the ids are a register of the 64 lanes, a block's place follows by arithmetic and a lane read.  Exact: i < 1024, and
  // (i + 1/2) / kpg is at least 1/2048 off every integer
  const int ids = ly.plan[1 + lane];
  const int total = min(max(ly.plan[0], 0), ly.G) * kpg;           // <= R / 16 <= 1024
  const float inv = 1.0f / (float)kpg;
  auto block = [&](int s) {                                        // of step s of this wavefront
    const int i = wave + s * DW_WAVES, g = __builtin_amdgcn_readfirstlane((int)(((float)i + 0.5f) * inv));
    return max(__builtin_amdgcn_readlane(ids, g), 0) * kpg + i - g * kpg;
  };
  const int units = (ncb + CB - 1) / CB, units8 = a.groups > 1 ? (units + 7) / 8 * 8 : units;
  const int unit = ((int)blockIdx.x - ly.y_first) % units8, group = ((int)blockIdx.x - ly.y_first) / units8;
  const int c0 = unit * CB, p0 = min(group * NT, a.panels - NT), skip = group * NT - p0;
  if (unit >= units) return;
  const char *U = (const char *)ly.Ut + lane * 16, *Z = (const char *)ly.zf + (size_t)p0 * (ly.R / 16) * 1024 + lane * 16;
  int cb[CB];
#pragma unroll
  for (int i = 0; i < CB; ++i) cb[i] = min(c0 + i, ncb - 1);       // blocks past the end re-read the last one (not stored)
  const size_t zstep = (size_t)(ly.R / 16);
  f32x16 acc[CB][NT];
  wide_loop<CB, NT, PAST>(acc, (total - wave + DW_WAVES - 1) / DW_WAVES, block,
                    [&](int b, int i) { return U + ((size_t)b * ncb + cb[i]) * 1024; },
                    [&](int b, int p) { return Z + (p * zstep + b) * 1024; });
  // The wavefronts' sums meet in LDS, ROUND tiles at a time, and wavefront w adds and stores every fourth tile (all fifteen of three column blocks and five
  // panels, panel by panel, took 4.4 us of 36).  Lane (sequence, q) holds columns 8 b + 4 q .. + 3 of band b of its tile.
#pragma unroll
  for (int t0 = 0; t0 < TILES; t0 += ROUND) {
    if (t0 > 0) __syncthreads();
#pragma unroll
    for (int t = t0; t < TILES && t < t0 + ROUND; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const f32x16 &v = acc[t % CB][t / CB];
        red[t - t0][wave][b][lane] = f32x4v{v[b * 4], v[b * 4 + 1], v[b * 4 + 2], v[b * 4 + 3]};
      }
    __syncthreads();
    for (int t = t0 + wave; t < TILES && t < t0 + ROUND; t += DW_WAVES) {              // uniform
      const int i = t % CB, p = t / CB, seq = (p0 + p) * 32 + (lane & 31);
      if (p < skip || c0 + i >= ncb) continue;
      f32x4v y[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        y[b] = red[t - t0][0][b][lane];
#pragma unroll
        for (int w = 1; w < DW_WAVES; ++w) y[b] += red[t - t0][w][b][lane];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {          // after the swap lane (sequence, q) holds the 8 columns 16 h + 8 q .. + 7
        const u32x2 x0 = __builtin_amdgcn_permlane32_swap(cvt_pk_bf16(y[2 * h][0], y[2 * h][1]), cvt_pk_bf16(y[2 * h + 1][0], y[2 * h + 1][1]), false, false);
        const u32x2 x1 = __builtin_amdgcn_permlane32_swap(cvt_pk_bf16(y[2 * h][2], y[2 * h][3]), cvt_pk_bf16(y[2 * h + 1][2], y[2 * h + 1][3]), false, false);
        if (seq < a.B)
          *reinterpret_cast<u32x4 *>(ly.y + (size_t)seq * m + (c0 + i) * 32 + h * 16 + (lane >> 5) * 8) = u32x4{x0[0], x1[0], x0[1], x1[1]};
      }
    }
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
  size_t t = round_up((size_t)n_layers * DW_PLAN_WORDS * sizeof(int32_t), 256);
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

template <int NT, bool PAST>
static int launch_wide_z(const DwArgs &a, int wgs, hipStream_t s) {
  constexpr int smem = dw_stages(NT) * (8 + 4 * NT) * 1024;
  static_assert(smem >= DW_PREP_BYTES, "the plan's lists stand where the stages do");
  static bool attr_done[64] = {false};       // the limit holds for the kernel on a device, not for a launch
  int dev = 0;
  PARSE_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return PARSE_EINVAL;
  if (!attr_done[dev]) {
    PARSE_HIP_TRY(hipFuncSetAttribute((const void *)wide_z<NT, PAST>, hipFuncAttributeMaxDynamicSharedMemorySize, smem));
    attr_done[dev] = true;
  }
  hipLaunchKernelGGL((wide_z<NT, PAST>), dim3(wgs), dim3(DWZ_THREADS), smem, s, a);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

static int wide_pass(DwArgs a, bool past, hipStream_t s) {
  int st, zw = 0, sw = 0;
  for (int l = 0; l < a.n_layers; ++l) {
    a.L[l].z_first = zw; zw += (a.L[l].R / 32 + DW_ZCB - 1) / DW_ZCB * a.KS;
    a.L[l].s_first = sw; sw += a.L[l].R / 16 * a.panels;
  }
  // Column blocks x panels of a wide_y workgroup: every round of workgroups takes in as many operands a step as their sum; of equals the one with
  // fewer panels, whose sums meet one after the other at the end.  All panels in each workgroup left half of the units idle where columns are few: 150
  // sequences through 11008 -> 4096 columns, 2560 ranks, a call, us, column blocks x panels 1 x 5 38.5, 2 x 5 40.8 and the equals 1 x 3 35.2, 2 x 2 34.7, 3 x 1
  // 34.3; 1024 -> 448, 2048 ranks, 238 sequences 37.8 (1 x 4), 30.1 (1 x 2); 4096 -> 2 x 11008, 192 sequences 82 (2 x 6), 68 (3 x 3), 150 sequences 46 (3 x 5),
  // 52 (3 x 3).  Over 122 calls of up to 17 forms each the one taken is 1 % off the best on average, 10 % at worst (few ranks, where two workgroups a unit run
  // side by side); in the 21 with equals of unlike panels the one with fewer took 2 % less.
  int cb = 1, nt = a.panels;
  long long least = 0;
  for (int c = 1; c <= 3; ++c)
    for (int g = 1; g <= a.panels; ++g) {
      const int t = (a.panels + g - 1) / g;
      if (c * t > 15 || (t * (g - 1) >= a.panels)) continue;       // what the accumulators leave room for
      long long wgs = 0;
      for (int l = 0; l < a.n_layers; ++l) wgs += (long long)((a.L[l].m / 32 + c - 1) / c) * g;
      const long long cost = (wgs + DW_UNITS - 1) / DW_UNITS * (c + t);
      if (least == 0 || cost < least || (cost == least && t < nt)) { least = cost; cb = c; nt = t; a.groups = g; }
    }
  int yw = 0;
  for (int l = 0; l < a.n_layers; ++l) {
    const int units = (a.L[l].m / 32 + cb - 1) / cb;
    a.L[l].y_first = yw;
    yw += (a.groups > 1 ? (units + 7) / 8 * 8 : units) * a.groups;
  }
#define PARSE_DWZ(NT_) case NT_: st = past ? launch_wide_z<NT_, true>(a, zw, s) : launch_wide_z<NT_, false>(a, zw, s); break
  switch (a.panels) {
    PARSE_DWZ(1); PARSE_DWZ(2); PARSE_DWZ(3); PARSE_DWZ(4); PARSE_DWZ(5); PARSE_DWZ(6);
    default: return PARSE_ESHAPE;
  }
#undef PARSE_DWZ
  if (st != PARSE_OK) return st;
  if (a.KS > 1) {
    hipLaunchKernelGGL(wide_zsum, dim3((sw + DW_WAVES - 1) / DW_WAVES), dim3(DW_THREADS), 0, s, a);
    PARSE_LAUNCH_CHECK();
  }
  // Past the caches where one group of panels reads a column block (several share what the first one brings into the die's L2) and has up to three panels:
  // a workgroup of more takes in more z than factor.  MLP of 4096 x 11008, us a step, ordinary loads / first product past the caches / both, by states in turn:
  //    64 sequences  one 68.3 / 68.5 / 71.6   three 78.6 / 77.4 / 71.8    32 78.9 / 77.0 / 75.6
  //    96            one 74.2 / 77.9 / 82.2   three 91.5 / 89.6 / 83.0    32 92.2 / 90.1 / 89.0
  //   128            one 76.7 / 80.7 / 88.2   three 97.4 / 94.5 / 88.6    32 97.3 / 94.4 / 95.3
  //   150            one 91.0 / 89.0 / 99.9   three 107.3 / 105.4 / 99.9  32 106.7 / 104.6 / 107.9
  // (of few states a part stays in the last-level cache when nothing drives it out, which a program of tens of layers, or with other work in between, does not see).
  past = past && a.groups == 1 && nt <= DWY_PAST;
#define PARSE_DWY2(CB_, NT_)                                                                                     \
  do {                                                                                                           \
    if (past) hipLaunchKernelGGL((wide_y<CB_, NT_, (NT_ <= DWY_PAST)>), dim3(yw), dim3(DW_THREADS), 0, s, a);    \
    else hipLaunchKernelGGL((wide_y<CB_, NT_, false>), dim3(yw), dim3(DW_THREADS), 0, s, a);                     \
  } while (0)
#define PARSE_DWY(NT_)                                                                                           \
  case NT_:                                                                                                      \
    if (cb == 1) PARSE_DWY2(1, NT_); else if (cb == 2) PARSE_DWY2(2, NT_); else PARSE_DWY2((NT_ < 6 ? 3 : 2), NT_); \
    break
  switch (nt) {
    PARSE_DWY(1); PARSE_DWY(2); PARSE_DWY(3); PARSE_DWY(4); PARSE_DWY(5); PARSE_DWY(6);
    default: return PARSE_ESHAPE;
  }
#undef PARSE_DWY
#undef PARSE_DWY2
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
    const int st = wide_pass(a, past_caches(layers, n_layers), s);
    if (st != PARSE_OK) return st;
  }
  return PARSE_OK;
}

}  // namespace parse
