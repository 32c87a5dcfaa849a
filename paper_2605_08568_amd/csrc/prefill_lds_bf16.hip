// a6, planned form of the bf16 prefill product (Sec. 4.4, Eq. 10):  launch 1  Z = X Vt_S^T,  launch 2  Y = Z Ut_S,
// both with one tile kernel, `gemm_lds` (first products of many tiles: `gemm_first256`), over the virtual rows of a
// prefill plan (plan.hip): a tile of token rows belongs to one pattern, so a workgroup runs one reduction with one factor block, whatever the prompt lengths.
//
// Data path.  Both operands of a tile are staged in LDS by loads that write LDS directly (no register round trip,
// 1 KiB per wavefront instruction), STAGES reduction slices of KS deep; the matrix-core operands are then 16-byte
// LDS reads.  Factor operands are stored in operand order in memory (PARSE_MFMA16), so a 1 KiB load lands as one
// ready operand and is read back linearly (conflict-free).  The intermediate Z is written by launch 1 in the same
// operand order (token block x reduction block), so launch 2 stages it exactly like a factor.  Only X is row-major:
// its rows are loaded 16 bytes per lane, whole cache lines per row, and the 16-byte chunks of a row are XOR-swizzled
// on the way in (the swizzle is applied to the global address, the LDS write is linear) so that the operand reads --
// 16 rows x four chunks -- spread over all banks.
// Pipeline: a unit is 32 reduction indices of a wavefront's share of the tile; its operands are read from LDS into
// registers during the unit before, and the loads of later slices are requested one by one between its matrix
// instructions.  Before the last unit of a slice the wavefront waits for its own loads of the next slice and meets the
// others at a barrier (so everybody's loads have landed and everybody has read the current slice); from then on the
// slice STAGES ahead is requested into the place just freed.
// Output: the accumulator of the 16x16x32 instruction gives a lane 4 consecutive factor rows (output columns) of one
// token; one 16-lane swap of two blocks pairs them up to 8 consecutive columns = 16 bytes, which is one piece of a Z
// operand (launch 1: stored linearly, 1 KiB per instruction) or a 16-byte store into the token's row of Y (launch 2).
#include <algorithm>

#include "prefill_common.hpp"

namespace parse {

#define PARSE_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
#define PARSE_GLB_PTR(p) ((const __attribute__((address_space(1))) void *)(p))

constexpr int LG_MAX_LAYERS = 4;

// One product of one layer.  A launch covers up to LG_MAX_LAYERS of them (layers that share their token rows and the
// plan: the stacked first product and the batched second product of Sec. 4.4, Eq. 11-12): the column tiles of the
// layers are numbered through, tn_first is a layer's first.
struct LgLayer {
  const uint16_t *Tk;      // TROW 1: row-major [rows][K] (X);  TROW 0: Z in operand order [(virtual rows)/32][K/16][1 KiB]
  const uint16_t *F;       // factor operands of all patterns
  uint16_t *O;             // OROW 0: Z (operand order);  OROW 1: Y row-major [rows][M]
  float *Pz;               // SPLIT: fp32 partial sums of Z, [slice][token block][reduction block][64 lanes][8]
  size_t pattern_stride;   // elements of F per pattern
  int K, M;                // reduction length, factor rows (= output columns)
  // shared head (Sec. 4.4: shared experts at the head of memory, stored once): the first sh_blocks 32-rank blocks of
  // every pattern's selection come from Fsh (same operand order, as many rank rows as the head has), the per-pattern
  // blocks in F hold the rest, renumbered from 0.  FORD 0: the leading factor-row blocks; FORD 1 (KS == 32 only): the
  // leading reduction slices.  0 = everything per pattern.
  const uint16_t *Fsh;
  int sh_blocks;
  int tn_first;            // first column tile of this layer in the launch
};
struct LgArgs {
  LgLayer L[LG_MAX_LAYERS];
  int n_layers;
  const int32_t *plan;     // header | tile patterns | row map (plan.hip); ONE: none
  const int32_t *tok_offsets, *pattern_id;     // ONE: the prompt
  int rows, NP;
  int cap;                 // plan capacity in 256-row tiles (fixes where the row map starts)
  int ntn, gm, ngroups;    // column tiles (all layers), token tiles per locality group, groups
  int compact;             // the padding tiles are left out of the numbering (plans of at most 256 tiles of BM rows)
  int ks;                  // SPLIT: slices of the reduction range, one workgroup each
};

// What a workgroup asks of the plan: read from memory, or (ONE) the same answers for a single prompt, whose virtual rows are its token rows: that saves the
// plan's own launch where a call makes its plan for itself, and two dependent loads (one prompt of 57 rows, 1024 x 1024, 224 ranks, both products
// 13.7 -> 10.9 us a call; 34 rows, 4096 x 4096 17.1 -> 14.1; 2048 rows x 1024 ranks, n = 11008, 87 -> 81).  More prompts are not worth it: up to four in scalar registers
// take 1-2 us of a call's 3 (two launches, all wavefronts), up to 16 by lane readings 2-7.
template <int ONE>
struct LgPlan {
  const LgArgs &a;
  const int32_t *rowmap;
  int off, len, pid;                           // first token row, rows, pattern (-1: none)
  __device__ __forceinline__ explicit LgPlan(const LgArgs &args) : a(args) {
    if (!ONE) {
      rowmap = a.plan + 16 + (a.cap + 15) / 16 * 16;
    } else {
      const int b = a.tok_offsets[0], e = a.tok_offsets[1], v = a.pattern_id[0];
      off = b < 0 ? 0 : (b > a.rows ? a.rows : b);
      len = max((e < 0 ? 0 : (e > a.rows ? a.rows : e)) - off, 0);
      pid = v >= 0 && v < a.NP ? v : -1;
    }
  }
  __device__ __forceinline__ int virtual_rows() const { return ONE ? (len + 255) / 256 * 256 : a.plan[1]; }
  __device__ __forceinline__ int pattern(int tile) const { return ONE ? pid : a.plan[16 + tile]; }   // of a 256-row tile below virtual_rows, -1: none
  __device__ __forceinline__ int token_row(int v) const { return ONE ? (v < len ? off + v : -1) : rowmap[v]; }   // of a virtual row, -1: padding
};

// Numbering of a launch's tiles: consecutive ids share a die (and its L2); within a locality group the token tile runs fastest.
// The grid is sized for the plan's capacity; the real tile count comes from the plan.  Workgroups past it leave at once, the others
// are renumbered over the REAL count so that every die gets its share.  The last locality group is as high as the tiles it has: with its
// missing ones numbered too, the dies of the full groups got up to twice the tiles of the others (one prompt of 2306 rows, n = 11008, 672 ranks, both
// products 101 -> 75 us; 1500 rows x 3 x 768 ranks 95 -> 74; seven of 734, 11008 columns 74 -> 67).  False: nothing to do.
// a.compact: tiles of nothing but padding (the rows of a pattern come first, its padding last: such a tile starts with it)
// are left out of the numbering.  Workgroups are dealt to the dies before anything is known of them; with the padding
// numbered, one die can get more tiles than it has compute units while another one's leave at once (20 prompts of 30-640
// tokens, 220 of 264 tiles real: the launch took two rounds, 118 us against 82).
template <int BM, int ONE>
__device__ __forceinline__ bool lg_find_tile(const LgArgs &a, const LgPlan<ONE> &plan, int bid, int lane, int &tm, int &tn, int &li) {
  const int per = a.gm * a.ntn;
  int n_tiles = (plan.virtual_rows() + BM - 1) / BM;
  unsigned long long real[4];                  // bit l of real[u]: tile 64 u + l holds tokens
  if (BM < 256 && a.compact) {
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = u * 64 + lane;
      real[u] = __ballot(t < a.cap * (256 / BM) && plan.token_row(min(t, a.cap * (256 / BM) - 1) * BM) >= 0 && t < n_tiles);
      cnt += __popcll(real[u]);
    }
    n_tiles = cnt;
  }
  const int n_real = n_tiles * a.ntn;
  if (bid >= n_real) return false;
  const int tile = xcd_tile(bid, n_real);
  const int g = tile / per, r = tile % per, high = min(a.gm, n_tiles - g * a.gm);
  tm = g * a.gm + r % high;
  tn = r / high;                               // column tile over all layers of the launch
  li = 0;
#pragma unroll
  for (int i = 1; i < LG_MAX_LAYERS; ++i) li += (i < a.n_layers && tn >= a.L[i].tn_first) ? 1 : 0;
  tn -= a.L[li].tn_first;
  if (BM < 256 && a.compact) {                 // the tm-th tile that holds tokens
    int at = tm, found = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int n = __popcll(real[u]);
      if (at >= 0 && at < n) {                 // uniform
        const bool is = ((real[u] >> lane) & 1ull) && __popcll(real[u] & ((1ull << lane) - 1ull)) == at;
        found = u * 64 + __ffsll((unsigned long long)__ballot(is)) - 1;
      }
      at -= n;
    }
    tm = __builtin_amdgcn_readfirstlane(found);
  }
  return true;
}

// Rows of a tile whose prompts have no valid pattern: the first product has nothing to do, the second one writes zero rows
template <int BM, int BN, int ONE>
__device__ __forceinline__ void lg_zero_rows(const LgLayer &ly, const LgPlan<ONE> &plan, int tm, int tn, int wave, int n_waves, int lane) {
  for (int rr = wave; rr < BM; rr += n_waves) {
    const int orow = plan.token_row(tm * BM + rr);
    if (orow < 0) continue;
    for (int c = lane * 8; c < BN; c += 512) {
      const int col = tn * BN + c;
      if (col < ly.M) *reinterpret_cast<u32x4 *>(ly.O + (size_t)orow * ly.M + col) = u32x4{0, 0, 0, 0};
    }
  }
}

// Lane (j, g) of an accumulator holds factor rows 4 g + (0..3) of token j.  One 16-lane swap of two blocks pairs them up to 8
// consecutive factor rows, 16 bytes: groups 0 / 2 get rows 0..7 / 8..15 of the first block, groups 1 / 3 of the second.
__device__ __forceinline__ u32x4 lg_pair(const f32x4v &u, const f32x4v &v) {
  const u32x2 s0 = __builtin_amdgcn_permlane16_swap(cvt_pk_bf16(u[0], u[1]), cvt_pk_bf16(v[0], v[1]), false, false);
  const u32x2 s1 = __builtin_amdgcn_permlane16_swap(cvt_pk_bf16(u[2], u[3]), cvt_pk_bf16(v[2], v[3]), false, false);
  return u32x4{s0[0], s1[0], s0[1], s1[1]};
}

// Tile kernel.  What bounds it is power and the issue of loads: a load that writes LDS holds its wavefront until the address unit
// takes it, so the loads of a slice in a row after the barrier, by every wavefront at once, left the matrix pipes idle for a third
// of a slice.  Here they are spread between the matrix instructions.  16x16x32 instead of 32x32x16 instructions: twice the
// reduction per accumulator access, 5-8 % less power (a slice of 64 of a 256 x 256 tile in a loop on normal data, us: matrix
// instructions and operand reads alone 1.31, loads in a burst 1.60, between the products 1.49, with 16x16x32 1.40).
//
// FORD: factor order, 0 = right factor (operand (rb, kb) at rb*(K/16)+kb), 1 = left factor (operand (kb, cb) at kb*(M/32)+cb).
// TROW: token operand 1 = row-major rows looked up through the plan's row map (X), 0 = operand order over the plan's virtual
//       rows (Z).   OROW: output 1 = row-major through the row map, 0 = operand order.
// First product: <FORD 0, TROW 1, OROW 0>, slices of KS = 64 (whole cache lines of a row of X); second product: <1, 0, 1>, KS = 32
// (64 in launches of few tiles without a shared head).
// A unit of work is 32 reduction indices of a wavefront's share of the tile; its operands are read from LDS into registers during
// the unit before.  WK 2: two wavefronts share an output tile, each takes one half of every slice, and the halves are added at the
// end through LDS: a tile of 128 x 128 or less then still has eight wavefronts, two per SIMD, whose waits cover each other.
// Slice kt + STAGES is requested once slice kt has been read by everybody: from the last unit of slice kt on, whose start has the
// barrier that also says that slice kt + 1 has landed.
// SPLIT (first product only): the reduction range is cut in a.ks slices, one workgroup each; a workgroup stores its fp32
// sums as slice s of the partial sums and z_combine adds the slices (in slice order) and rounds -- for launches whose
// tiles alone would leave most compute units idle (one short prompt).
template <int BM, int BN, int WM, int WN, int KS, int STAGES, int FORD, int TROW, int OROW, int SPLIT, int WK, int ONE>
__global__ __launch_bounds__(WM * WN * WK * 64, 2) void gemm_lds(LgArgs a) {
  static_assert(!SPLIT || (FORD == 0 && OROW == 0), "only the first product is split");
  static_assert(WK == 1 || (OROW == 0 && KS == 64), "halves of slices of 64, added for Z");
  // FORD 1 with a shared head: KS = 32, the head ends between slices
  static_assert(TROW == 0 || KS == 64, "token rows are swizzled in chunks of 128 bytes");
  static_assert(256 % BM == 0, "token tiles subdivide the plan's 256-row tiles");
  constexpr int NW = WM * WN * WK;
  constexpr int KK = KS / 16;                 // operands of a 32-row block in a slice
  constexpr int NU = KS / 32 / WK;            // units of a slice
  constexpr int FB = BN / WN / 16, TB = BM / WM / 16;   // 16-row blocks of a wavefront
  constexpr int F_BYTES = BN * KS * 2, T_BYTES = BM * KS * 2, STAGE_BYTES = F_BYTES + T_BYTES;
  constexpr int NI_F = F_BYTES / 1024, NI_T = T_BYTES / 1024;   // 1 KiB load instructions per slice
  static_assert(NI_F % NW == 0 && NI_T % NW == 0, "the loads of a slice divide evenly over the wavefronts");
  constexpr int LF = NI_F / NW, LT = NI_T / NW, L = LF + LT, LU = L / NU;
  static_assert(L % NU == 0 && LU <= FB * TB, "and over the units");
  static_assert((STAGES - 2) * L + LU < 64, "vmcnt is a 6-bit count");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wk = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;
  const int j = lane & 15, g = lane >> 4;

  const LgPlan<ONE> plan(a);
  const int ks = SPLIT ? a.ks : 1;
  const int bid = SPLIT ? (int)blockIdx.x / ks : (int)blockIdx.x, sl = SPLIT ? (int)blockIdx.x % ks : 0;
  int tm, tn, li;
  if (!lg_find_tile<BM>(a, plan, bid, lane, tm, tn, li)) return;
  const LgLayer &ly = a.L[li];
  const int K = ly.K, M = ly.M;
  const int kt0 = SPLIT ? (int)(((long long)(K / KS) * sl) / ks) : 0;           // first slice of this workgroup
  const int nk = (SPLIT ? (int)(((long long)(K / KS) * (sl + 1)) / ks) : K / KS) - kt0;
  const int pat = plan.pattern(tm * BM / 256);
  if (pat < 0) {
    if (OROW == 1) lg_zero_rows<BM, BN>(ly, plan, tm, tn, wave, NW, lane);
    return;
  }
  if (BM < 256 && !a.compact && plan.token_row(tm * BM) < 0) return;
  const uint16_t *Fp = ly.F + (size_t)pat * ly.pattern_stride;

  // ---- sources of this wavefront's load instructions; they advance by a constant per slice ----
  const uint32_t loff = lane * 16;
  const char *fsrc[LF], *fsrc_own[LF];         // own: FORD 1 with a shared head: where the pattern's own slices start
  const int shb = ly.sh_blocks;
  const size_t fstep = FORD == 0 ? (size_t)KK * 1024 : (size_t)KK * (M / 32) * 1024;
#pragma unroll
  for (int i = 0; i < LF; ++i) {
    const int ins = wave * LF + i, fb = ins / KK, kk = ins % KK;   // LDS order of the factor part: [block of 32][operand]
    const int gb = min(tn * (BN / 32) + fb, M / 32 - 1);           // blocks past the end re-read the last one (never stored)
    if (FORD == 0) {
      fsrc[i] = (gb < shb ? (const char *)ly.Fsh + (size_t)gb * (K / 16) * 1024 : (const char *)Fp + (size_t)(gb - shb) * (K / 16) * 1024) +
                (size_t)kk * 1024 + (SPLIT ? (size_t)kt0 * fstep : 0);
      fsrc_own[i] = fsrc[i];
    } else {
      fsrc_own[i] = (const char *)Fp + ((size_t)kk * (M / 32) + gb) * 1024;
      fsrc[i] = shb > 0 ? (const char *)ly.Fsh + ((size_t)kk * (M / 32) + gb) * 1024 : fsrc_own[i];
    }
  }
  const char *tsrc[LT];
#pragma unroll
  for (int i = 0; i < LT; ++i) {
    const int ins = wave * LT + i;
    if (TROW == 0) {                           // LDS order: [block of 32][operand]
      const int tb = ins / KK, kk = ins % KK;
      tsrc[i] = (const char *)ly.Tk + ((size_t)(tm * (BM / 32) + tb) * (K / 16) + kk) * 1024;
    } else {                                   // LDS place: row rr, slot lane % 8; it holds chunk slot ^ swizzle of the row
      const int rr = ins * 8 + (lane >> 3);
      const int row = max(plan.token_row(tm * BM + rr), 0);        // padding rows read row 0; their results are never stored to Y
      tsrc[i] = (const char *)ly.Tk + (size_t)row * K * 2 + (((lane & 7) ^ ((rr >> 1) & 7)) * 16) + (SPLIT ? (size_t)kt0 * 128 : 0);
    }
  }
  int issued = 0, dst = 0;                     // slices requested so far; place of the next one
  auto load = [&](int q) {                     // load q of L of the next slice; the last one moves on
    if (q < LF) {
      __builtin_amdgcn_global_load_lds(PARSE_GLB_PTR(fsrc[q] + loff), PARSE_LDS_PTR(smem + dst + (wave * LF + q) * 1024), 16, 0, 0);
      fsrc[q] += fstep;
    } else {
      const int i = q - LF;
      __builtin_amdgcn_global_load_lds(PARSE_GLB_PTR(TROW == 0 ? tsrc[i] + loff : tsrc[i]),
                                       PARSE_LDS_PTR(smem + dst + F_BYTES + (wave * LT + i) * 1024), 16, 0, 0);
      tsrc[i] += TROW == 0 ? KK * 1024 : KS * 2;
    }
    if (q == L - 1) {
      dst = dst + STAGE_BYTES == STAGES * STAGE_BYTES ? 0 : dst + STAGE_BYTES;
      ++issued;
      if (FORD == 1 && issued == shb) {        // the reduction leaves the shared head: continue in the pattern's own block
#pragma unroll
        for (int i = 0; i < LF; ++i) fsrc[i] = fsrc_own[i];
      }
    }
  };

  // ---- LDS operands: lane (j, g) reads reduction indices 8 g .. 8 g + 7 of row j of a 16-row block ----
  const int oplane = (g >> 1) * 1024 + (g & 1) * 512 + j * 16;     // in operand order
  const int f_lane = wn * (FB / 2) * KK * 1024 + oplane;
  const int t_lane = F_BYTES + (TROW == 0 ? wm * (TB / 2) * KK * 1024 + oplane : wm * TB * 2048 + j * 128 + ((g ^ ((j >> 1) & 7)) * 16));
  f32x4v acc[FB][TB];
#pragma unroll
  for (int i = 0; i < FB; ++i)
#pragma unroll
    for (int t = 0; t < TB; ++t) acc[i][t] = f32x4v{0.f, 0.f, 0.f, 0.f};
  u32x4 fr[2][FB], tr[2][TB];
  auto read_unit = [&](int buf, int src, int half) {               // half of the slice at src
    const char *fb = smem + src + f_lane + half * 2048;
#pragma unroll
    for (int i = 0; i < FB; ++i) fr[buf][i] = *reinterpret_cast<const u32x4 *>(fb + (i >> 1) * KK * 1024 + (i & 1) * 256);
    const char *tb = smem + src + (TROW == 0 ? t_lane + half * 2048 : t_lane ^ (half * 64));
#pragma unroll
    for (int t = 0; t < TB; ++t)
      tr[buf][t] = *reinterpret_cast<const u32x4 *>(tb + (TROW == 0 ? (t >> 1) * KK * 1024 + (t & 1) * 256 : t * 2048));
  };
  // The compiler treats a load that writes LDS directly like a flat access that may complete out of order with LDS
  // reads, so after one of them every wait it inserts for LDS data is a wait for ALL outstanding LDS reads.  Placed by
  // the compiler that wait sits between the reads of the next unit and the matrix instructions of this one and exposes
  // the LDS latency.  Touching this unit's operands BEFORE the next unit's reads are issued moves the wait
  // to where nothing is outstanding but reads that had a whole unit to finish.
  auto settle = [&](int buf) {
#pragma unroll
    for (int i = 0; i < FB; ++i) asm volatile("" ::"v"(fr[buf][i]));
#pragma unroll
    for (int t = 0; t < TB; ++t) asm volatile("" ::"v"(tr[buf][t]));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto products = [&](int buf, int q0, bool more) {                // ... with loads q0 .. q0 + LU - 1 between them
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fr[buf][i]), as_bf16x8(tr[buf][t]), acc[i][t], 0, 0, 0);
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

  // prologue: what the units before the first one would have requested
#pragma unroll
  for (int s = 0; s < STAGES; ++s) {
    if (s < nk) {
#pragma unroll
      for (int q = 0; q < (s == STAGES - 1 ? LU : L); ++q) load(q);
    }
  }
  if (nk >= STAGES) wait_vm<(STAGES - 2) * L + LU>(); else wait_vm<0>();
  wg_barrier();
  int src = 0;                                 // place of the slice that is read
  read_unit(0, src, wk);
  auto hand_over = [&](bool steady, int kt) {  // slice kt + 1 has landed for everybody, slice kt has been read by everybody
    if (steady) wait_vm<(STAGES - 2) * L>(); else wait_slices<STAGES - 2, L>(min(kt + STAGES - 1, nk - 1) - (kt + 1));
    wg_barrier();
    src = src + STAGE_BYTES == STAGES * STAGE_BYTES ? 0 : src + STAGE_BYTES;
  };
  // the units of slice kt (NU 1: p its parity); steady: slice kt + STAGES exists.  The loop over those has no branches: between
  // the barriers of a 128 x 128 tile a wavefront has but sixteen products, and every taken branch delays all eight of them
  auto slice = [&](bool steady, int p, int kt) {
    if (NU == 2) {
      settle(0);
      read_unit(1, src, 1);
      products(0, LU, steady || kt - 1 + STAGES < nk);
      settle(1);
      if (steady || kt + 1 < nk) { hand_over(steady, kt); read_unit(0, src, 0); }
      products(1, 0, steady || kt + STAGES < nk);
    } else {
      settle(p);
      if (steady || kt + 1 < nk) { hand_over(steady, kt); read_unit(p ^ 1, src, wk); }
      products(p, 0, steady || kt + STAGES < nk);
    }
  };
  int kt = 0;
  for (; kt + STAGES + 1 < nk; kt += 2) {
    slice(true, 0, kt);
    slice(true, 1, kt + 1);
  }
  for (; kt < nk; kt += 2) {
    slice(false, 0, kt);
    if (kt + 1 < nk) slice(false, 1, kt + 1);
  }

  if constexpr (WK == 2) {
    // the two halves of the reduction: each takes half of the accumulators over from the other (the staged slices are dead)
    float *ex = reinterpret_cast<float *>(smem) + (size_t)(wave % (WM * WN)) * (FB * TB * 256) + lane * 4;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int t = 0; t < TB; ++t)
        if (i * 2 / FB != wk) *reinterpret_cast<f32x4v *>(ex + (i * TB + t) * 256) = acc[i][t];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
      for (int t = 0; t < TB; ++t)
        if (i * 2 / FB == wk) acc[i][t] += *reinterpret_cast<const f32x4v *>(ex + (i * TB + t) * 256);
  }
  if (OROW == 0) {                             // Z operands: two token blocks together are one operand, lane's piece at lane * 16
#pragma unroll
    for (int i = 0; i < FB; ++i) {
      const int kb = (tn * BN + wn * FB * 16) / 16 + i;            // 16 factor rows = one operand of the second product
      if (kb >= M / 16 || (WK == 2 && i * 2 / FB != wk)) continue;
#pragma unroll
      for (int t = 0; t < TB; t += 2) {
        const int tbg = tm * (BM / 32) + (wm * TB + t) / 2;
        if (SPLIT) {                           // the same exchange on the fp32 sums
          float *dst8 = ly.Pz + (((size_t)sl * (a.cap * 8) + tbg) * (M / 16) + kb) * 512 + lane * 8;
          f32x4v lo, hi;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const u32x2 sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[i][t][e]), __float_as_uint(acc[i][t + 1][e]), false, false);
            lo[e] = __uint_as_float(sw[0]); hi[e] = __uint_as_float(sw[1]);
          }
          *reinterpret_cast<f32x4v *>(dst8) = lo;
          *reinterpret_cast<f32x4v *>(dst8 + 4) = hi;
        } else {
          *reinterpret_cast<u32x4 *>((char *)ly.O + ((size_t)tbg * (M / 16) + kb) * 1024 + lane * 16) = lg_pair(acc[i][t], acc[i][t + 1]);
        }
      }
    }
  } else {                                     // rows of Y: two column blocks together, 64 bytes of a row
    int orow[TB];
    const LgPlan<ONE> again(a);                // not kept in registers over the reduction
#pragma unroll
    for (int t = 0; t < TB; ++t) orow[t] = again.token_row(tm * BM + (wm * TB + t) * 16 + j);
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int i = 0; i < FB; i += 2) {
        const int cb = (tn * BN + wn * FB * 16) / 32 + i / 2;      // block of 32 columns
        if (cb < M / 32 && orow[t] >= 0)
          *reinterpret_cast<u32x4 *>(ly.O + (size_t)orow[t] * M + cb * 32 + (g & 1) * 16 + (g >> 1) * 8) = lg_pair(acc[i][t], acc[i + 1][t]);
      }
  }
}

// First product on 256 x 256 tiles, for launches with many of them.  Slices of 64 of both operands would leave room for two only;
// here token operands are staged in slices of 64, three of them, and factor operands in halves of 32, four of them: 160 KiB, all of
// the LDS.  Time h runs the products of half h from registers, reads half h + 1 from LDS and requests factor half h + 4 (into the
// place of half h, read at time h - 1) and half of the token slice three after the one whose last half was read at time h - 1.  At
// the start of time h everything requested up to time h - 3 has landed (8 loads a wavefront may be outstanding; fewer are requested
// near the end), so a load has two halves, 2000 cycles, to arrive.  The sums are those of the other tiles, in the same order.
// 32768 rows x 1024 ranks of eight patterns, n = m = 4096, both products on large tiles: 526 us with slices of 64, two stages and
// 32x32x16 instructions, 462-480 now; 1280 ranks, 11008 columns: 1264 and 1160.
template <int ONE>
__global__ __launch_bounds__(512) void gemm_first256(LgArgs a) {
  constexpr int F_HALF = 16384, T_SLICE = 32768, T_BASE = 4 * F_HALF;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;     // 128 token rows x 64 factor rows each
  const int j = lane & 15, g = lane >> 4;
  const LgPlan<ONE> plan(a);
  int tm, tn, li;
  if (!lg_find_tile<256>(a, plan, blockIdx.x, lane, tm, tn, li)) return;
  const LgLayer &ly = a.L[li];
  const int K = ly.K, M = ly.M;
  const int pat = plan.pattern(tm);
  if (pat < 0) return;
  const int nk = K / 64, nh = nk * 2;

  // ---- sources: wavefront w loads factor block w of a half (two operands) and token rows 32 w .. +31 of a slice ----
  const int gb = min(tn * 8 + wave, M / 32 - 1);         // blocks past the end re-read the last one (never stored)
  const int shb = ly.sh_blocks;
  const char *fsrc = gb < shb ? (const char *)ly.Fsh + (size_t)gb * (K / 16) * 1024
                              : (const char *)(ly.F + (size_t)pat * ly.pattern_stride) + (size_t)(gb - shb) * (K / 16) * 1024;
  const uint32_t loff = lane * 16;
  const char *tsrc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rr = wave * 32 + i * 8 + (lane >> 3);      // LDS place: row rr, slot lane % 8; it holds chunk slot ^ swizzle of the row
    const int row = max(plan.token_row(tm * 256 + rr), 0);       // padding rows read row 0; their results are never stored to Y
    tsrc[i] = (const char *)ly.Tk + (size_t)row * K * 2 + (((lane & 7) ^ ((rr >> 1) & 7)) * 16);
  }
  int f_dst = wave * 2048, t_dst = T_BASE + wave * 4096; // place of the next half / slice that is requested
  auto load_f = [&](int i) {                             // operand i of the next half; i == 1 moves on
    __builtin_amdgcn_global_load_lds(PARSE_GLB_PTR(fsrc + i * 1024 + loff), PARSE_LDS_PTR(smem + f_dst + i * 1024), 16, 0, 0);
    if (i == 1) {
      fsrc += 2048;
      f_dst += F_HALF;
      if (f_dst >= T_BASE) f_dst -= T_BASE;
    }
  };
  auto load_t = [&](int i) {                             // row group i of the next slice; i == 3 moves on
    __builtin_amdgcn_global_load_lds(PARSE_GLB_PTR(tsrc[i]), PARSE_LDS_PTR(smem + t_dst + i * 1024), 16, 0, 0);
    tsrc[i] += 128;
    if (i == 3) {
      t_dst += T_SLICE;
      if (t_dst >= T_BASE + 3 * T_SLICE) t_dst -= 3 * T_SLICE;
    }
  };

  // ---- LDS operands: as in gemm_lds ----
  const int f_lane = wn * 4096 + (g >> 1) * 1024 + (g & 1) * 512 + j * 16;         // half: [block of 32][2 operands]
  const int t_lane = wm * 16384 + j * 128 + ((g ^ ((j >> 1) & 7)) * 16);
  f32x4v acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[i][t] = f32x4v{0.f, 0.f, 0.f, 0.f};
  u32x4 fr[2][4], tr[2][8];
  int f_rd = 0, t_rd = T_BASE;                           // places of the half / slice that is read next
  auto read_half = [&](int buf) {                        // buf = parity of the half
    const char *fb = smem + f_rd + f_lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) fr[buf][i] = *reinterpret_cast<const u32x4 *>(fb + (i >> 1) * 2048 + (i & 1) * 256);
    const char *tb = smem + t_rd + (t_lane ^ (buf * 64));
#pragma unroll
    for (int t = 0; t < 8; ++t) tr[buf][t] = *reinterpret_cast<const u32x4 *>(tb + t * 2048);
    f_rd += F_HALF;
    if (f_rd >= T_BASE) f_rd -= T_BASE;
    if (buf == 1) {
      t_rd += T_SLICE;
      if (t_rd >= T_BASE + 3 * T_SLICE) t_rd -= 3 * T_SLICE;
    }
  };
  auto settle = [&](int buf) {                           // as in gemm_lds
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" ::"v"(fr[buf][i]));
#pragma unroll
    for (int t = 0; t < 8; ++t) asm volatile("" ::"v"(tr[buf][t]));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto products = [&](int p, bool more_f, bool more_t) { // one load after every eight products
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fr[p][i]), as_bf16x8(tr[p][t]), acc[i][t], 0, 0, 0);
        if (t == 3) {
          __builtin_amdgcn_sched_barrier(0);
          if (i < 2) { if (more_f) load_f(i); }
          else if (more_t) load_t(p == 0 ? i : i - 2);   // even times: the second half of a slice
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // prologue: T0 F0 | F1 T1 | F2 F3, half of T2
#pragma unroll
  for (int i = 0; i < 4; ++i) load_t(i);
  load_f(0); load_f(1);
  load_f(0); load_f(1);
  if (nk > 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) load_t(i);
    load_f(0); load_f(1);
    load_f(0); load_f(1);
  }
  if (nk > 2) { load_t(0); load_t(1); wait_vm<12>(); } else wait_vm<0>();
  wg_barrier();
  read_half(0);
  auto slice = [&](bool steady, int h) {                 // steady: everything that a slice requests exists
    settle(0);
    if (steady || h < nh - 4) wait_vm<8>(); else if (h == nh - 4) wait_vm<6>(); else wait_vm<0>();
    wg_barrier();
    read_half(1);
    products(0, steady || h + 4 < nh, steady || h / 2 + 2 < nk);
    settle(1);
    if (steady || h + 2 < nh) {
      if (steady || h < nh - 5) wait_vm<8>(); else wait_vm<2>();
      wg_barrier();
      read_half(0);
    }
    products(1, steady || h + 5 < nh, steady || h / 2 + 3 < nk);
  };
  int h = 0;
  for (; h < nh - 6; h += 2) slice(true, h);
  for (; h < nh; h += 2) slice(false, h);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int kb = tn * 16 + wn * 4 + i;       // 16 factor rows = one operand of the second product
    if (kb >= M / 16) continue;
#pragma unroll
    for (int t = 0; t < 8; t += 2)
      *reinterpret_cast<u32x4 *>((char *)ly.O + ((size_t)(tm * 8 + wm * 4 + t / 2) * (M / 16) + kb) * 1024 + lane * 16) = lg_pair(acc[i][t], acc[i][t + 1]);
  }
}

// Adds the ks partial sums of every 16-byte piece of Z (8 consecutive ranks of a token) in slice order and rounds to
// bf16.  One thread per piece, over the plan's virtual rows and all layers of the call (grid.y); padding rows hold nothing
// and are passed over (the second product's results for them are not stored either).
template <int ONE>
__global__ __launch_bounds__(256) void z_combine(LgArgs a, int wgs) {
  const LgLayer &ly = a.L[blockIdx.y];
  const int M = ly.M, ks = a.ks;
  const LgPlan<ONE> plan(a);
  const size_t pieces = (size_t)(plan.virtual_rows() / 32) * (M / 16) * 64;    // virtual rows / 32 token blocks x reduction blocks x lanes
  const size_t slice = (size_t)a.cap * 8 * (M / 16) * 512;           // floats per slice
  for (size_t o = (size_t)blockIdx.x * 256 + threadIdx.x; o < pieces; o += (size_t)wgs * 256) {
    const size_t tb = o / ((size_t)(M / 16) * 64);
    if (plan.token_row((int)(tb * 32 + (o & 31))) < 0) continue;
    const float *src = ly.Pz + o * 8;
    float4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < ks; s0 += 4) {      // four slices requested at a time (slices past the last re-read it)
      float4 l4[4], h4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float *ps = src + (size_t)min(s0 + u, ks - 1) * slice;
        l4[u] = *reinterpret_cast<const float4 *>(ps);
        h4[u] = *reinterpret_cast<const float4 *>(ps + 4);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (s0 + u < ks) {
          lo.x += l4[u].x; lo.y += l4[u].y; lo.z += l4[u].z; lo.w += l4[u].w;
          hi.x += h4[u].x; hi.y += h4[u].y; hi.z += h4[u].z; hi.w += h4[u].w;
        }
      }
    }
    *reinterpret_cast<u32x4 *>(ly.O + o * 8) =
        u32x4{cvt_pk_bf16(lo.x, lo.y), cvt_pk_bf16(lo.z, lo.w), cvt_pk_bf16(hi.x, hi.y), cvt_pk_bf16(hi.z, hi.w)};
  }
}

// kern on tiles of BM x BN: the column tiles of the layers are numbered through, the grid covers what the plan can hold
template <int BM, int BN>
static int launch_tiles(void (*kern)(LgArgs), int threads, int smem, bool (&attr_done)[64], LgArgs a, int avg_tiles_per_pattern, int slices, hipStream_t s) {
  int dev = 0;
  PARSE_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return PARSE_EINVAL;
  if (!attr_done[dev]) {
    PARSE_HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem));
    attr_done[dev] = true;
  }
  const int ntm = a.cap * (256 / BM);          // token tiles the plan can hold (the kernel exits past the real count)
  a.ntn = 0;
  for (int l = 0; l < a.n_layers; ++l) {
    a.L[l].tn_first = a.ntn;
    a.ntn += (a.L[l].M + BN - 1) / BN;
  }
  int gm = avg_tiles_per_pattern * (256 / BM);
  a.gm = gm < 1 ? 1 : (gm > 8 ? 8 : gm);
  a.ngroups = (ntm + a.gm - 1) / a.gm;
  a.compact = BM < 256 && ntm <= 256 && a.compact;
  hipLaunchKernelGGL(kern, dim3(a.ngroups * a.gm * a.ntn * slices), dim3(threads), smem, s, a);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

template <int ONE, int BM, int BN, int WM, int WN, int KS, int STAGES, int FORD, int TROW, int OROW, int SPLIT, int WK>
static int launch_gemm_lds_as(const LgArgs &a, int avg_tiles_per_pattern, hipStream_t s) {
  constexpr int staged = STAGES * (BM + BN) * KS * 2, sums = WK > 1 ? BM * BN * 4 : 0;
  static bool attr_done[64] = {false};
  return launch_tiles<BM, BN>(gemm_lds<BM, BN, WM, WN, KS, STAGES, FORD, TROW, OROW, SPLIT, WK, ONE>, WM * WN * WK * 64,
                              staged > sums ? staged : sums, attr_done, a, avg_tiles_per_pattern, SPLIT ? a.ks : 1, s);
}
template <int BM, int BN, int WM, int WN, int KS, int STAGES, int FORD, int TROW, int OROW, int SPLIT = 0, int WK = 1>
static int launch_gemm_lds(const LgArgs &a, int avg_tiles_per_pattern, hipStream_t s) {
  return a.plan ? launch_gemm_lds_as<0, BM, BN, WM, WN, KS, STAGES, FORD, TROW, OROW, SPLIT, WK>(a, avg_tiles_per_pattern, s)
                : launch_gemm_lds_as<1, BM, BN, WM, WN, KS, STAGES, FORD, TROW, OROW, SPLIT, WK>(a, avg_tiles_per_pattern, s);
}

template <int ONE>
static int launch_first256(const LgArgs &a, int avg_tiles_per_pattern, hipStream_t s) {
  static bool attr_done[64] = {false};
  return launch_tiles<256, 256>(gemm_first256<ONE>, 512, 160 * 1024, attr_done, a, avg_tiles_per_pattern, 1, s);
}

// Token tiles of bm rows, as far as the host can tell: it does not know which prompts share a pattern, and a pattern starts on a
// tile of its own.  Prompts of one length that are a multiple of bm leave nothing open; otherwise full tiles and one more are
// taken for the number.  (Half a tile more for every prompt is closer when every prompt has its own pattern, but many prompts of
// few patterns then get tiles that are too large: 24 prompts of 20-300 tokens, n = m = 2048, 512 ranks, both products, us, first one
// on 64 x 128 / 128 x 128 tiles: 29.8 / 32.4 with two patterns, 44.6 / 38.8 with 24.  Over 70 batches of 1 to 40 prompts the tile chosen is
// 2.7 % off the best of each on average, 29 % at worst: ragged prompts, nearly every one with its own pattern or nearly none.)
static long long token_tiles(int rows, int P, int bm) {
  if (rows % P == 0 && rows / P % bm == 0) return rows / bm;
  return (rows + bm - 1) / bm + (P > 1 ? 1 : 0);
}

// Slices of the first product's reduction range that the smallest workspace has room for (1 = no split) ...
int prefill_planned_split(int rows, int n) {
  const int tiles = (rows + 63) / 64;
  if (tiles <= 0 || tiles > 16) return 1;
  int ks = 32 / tiles;
  if (ks > 8) ks = 8;
  if (ks > n / 64 / 8) ks = n / 64 / 8;
  return ks < 2 ? 1 : ks;
}
// ... and that the queried one has: also longer batches on long reductions that are cut (see split_slices), of which few prompts
// with few tiles are: everybody else is not asked for four fp32 copies of the intermediate (4096 rows of 64 prompts x 1280 ranks:
// 52 MB with the room left out, 472 MB with it).
constexpr int SHORT_ROWS = 4096;
int prefill_planned_cut_prompts(int rows, int n) { return rows > 1024 && rows <= SHORT_ROWS && n >= 8192 ? rows / 384 : 0; }
int prefill_planned_room(int rows, int P, int n, int rS) {
  if (P <= prefill_planned_cut_prompts(rows, n) && token_tiles(rows, P, 128) * ((rS + 255) / 256) <= 96) return 4;
  return prefill_planned_split(rows, n);
}
// Z of one layer (bf16, operand order over the plan's capacity), then -- when the first product is split -- the fp32
// partial sums of its ks slices
static size_t planned_z_only_bytes(int cap_tiles, int rS) { return round_up((size_t)cap_tiles * 256 * rS * sizeof(uint16_t), 256); }
size_t prefill_planned_z_bytes(int cap_tiles, int rS, int ks) {
  return planned_z_only_bytes(cap_tiles, rS) + (ks > 1 ? round_up((size_t)ks * cap_tiles * 256 * rS * sizeof(float), 256) : 0);
}

bool prefill_planned_supported(int n, int m, int rS) { return n % 64 == 0 && rS % 32 == 0 && m % 32 == 0 && n >= 64 && rS >= 32; }

// Time of the first product with tile i, in units of a round of 128 x 128 tiles, one per compute unit (30 us at K = 4096).
// Fitted to earlier forms of these kernels, over shapes of 77 to 57 000 rows and 512 to 3072 ranks; over 34 calls of 150 to 4096 rows of the present ones
// the tile taken is 0.4 % off the best of each on average, 16 % at worst (ragged prompts).  n = m = 4096, both products, us, 256 x 256 / 128 x 256 / 128 x 128 /
// 64 x 128 / 64 x 64: one prompt of 2048 rows x 768 ranks 95 / 62 / 46 / 38 / 42; eight of 512 x 1024 111 / 78 / 68 / 76 / 82, of 1024 x 1024 147 / 124 / 138 / 151 /
// 161, of 4096 x 1024 462 / 517 / 573 / 651 / 694.  128 x 192 between them, up to SHORT_ROWS, 128 x 256 / 128 x 192 / 128 x 128 / 64 x 128: three layers of
// 768 ranks that share 2048 rows 93 / 88 / 101 / 101 (192 tiles of three quarters of the work, instead of 144), 2 x 1024 rows 107 / 99 / 112 / 114; n = m = 2048, 3 x 384
// ranks, 4096 rows 60 / 55.5 / 62 / 63.
enum { T64, T64x128, T128, T128x192, T128x256, T256, N_TILES };
static double tile_rounds(int i, const PfArgs *const *p, int n_layers, int split = 1) {
  static const int bm[N_TILES] = {64, 64, 128, 128, 128, 256}, bn[N_TILES] = {64, 128, 128, 192, 256, 256};
  long long t = 0;
  for (int l = 0; l < n_layers; ++l) t += (p[l]->rS + bn[i] - 1) / bn[i];
  t *= token_tiles(p[0]->rows, p[0]->P, bm[i]) * split;
  const double rounds = (double)((t + 255) / 256), two_each = (double)((t + 511) / 512);
  switch (i) {
    case T64: return t <= 256 ? 0.45 : (split > 1 ? 0.69 * two_each : 0.69 + 0.9 * (two_each - 1));
    case T64x128: return rounds - 0.4;
    case T128: return rounds;
    case T128x192: return 1.3 * rounds;
    case T128x256: return 1.57 * rounds;
    default: return 2.5 * rounds;
  }
}
static int best_tile(const PfArgs *const *p, int n_layers) {
  int best = T64;
  for (int i = 1; i < N_TILES; ++i)
    if (i != (p[0]->rows <= SHORT_ROWS ? T256 : T128x192) && tile_rounds(i, p, n_layers) < tile_rounds(best, p, n_layers)) best = i;
  return best;
}
// Slices of one layer's first product: as many (up to four) as pay for the second launch, which adds the fp32 partial sums (2 us
// and a pass over them).  77 rows, n = 4096, 1024 ranks, both products: 18.6 us with four, 20.1 and 19.1 with two and three, 22.2
// without; 300 rows x 1024 ranks 23.4 (two), 25.1 (three) and 24.8; 700 x 1024 32.6 (two) and 28.3; n = 11008: 534 rows x 384 ranks 35.8 (three)
// and 41.3, 643 x 384 32.1 (two) and 41.6, 1024 x 1280 76 (two) and 63; n = 5632, 546 x 640 27-29 and 27.  A function of the batch and of this
// layer alone, so that a call over several layers splits each like its single-layer call and gives the same bits -- as long as
// both have their queried workspace: with more than 1024 rows and no room for the partial sums a call is not cut.
// Batches of more than 1024 rows are split on reductions of 8192 and more, in four slices of 128 x 256 tiles: those move the
// fewest bytes per flop, and in slices they fill the chip, as long as they are few and the prompts fill them.  n = 11008, both products, us,
// without / with: 2048 rows x 1024 ranks 96 / 83, 1300 x 1024 91 / 72, 2048 x 640 91 / 68, 2 x 700 rows x 1024 96 / 75, 3 x 1300 x 768 145 / 141;
// three slices of 100 and 128 tiles 137 / 141 and 195 / 195; 16 x 200 x 1024 169 / 200; n = 8192, 2048 x 1024 77 / 70; n = 5632,
// 2048 x 512 39 / 44; n = 4096, 2048 x 1024 56 / 62.
static int split_slices(const PfArgs &p) {
  const int room = std::min(4, p.split_room);
  if (p.n < 4096) return 1;
  if (p.rows > 1024) return room;        // four where prefill_planned_room says so and the workspace is large enough
  const PfArgs *one[1] = {&p};
  const double round_us = 30.0 * p.n / 4096;
  int best = 1;
  double least = tile_rounds(best_tile(one, 1), one, 1) * round_us;
  for (int ks = 2; ks <= room; ++ks) {
    const double us = tile_rounds(T64, one, 1, ks) / ks * round_us + 2.0 + 4e-6 * p.rows * p.rS * ks;
    if (us < least) { least = us; best = ks; }
  }
  return best;
}

// A call that would make its plan for itself needs none.
bool prefill_needs_plan(int P) { return P > 1; }

// n_layers layers that share X [rows][n] (row-major) and the plan (none unless prefill_needs_plan; built for the tok_offsets and pattern ids of these
// patterns); Z[l] = layer l's intermediate (operand order over the plan's virtual rows); p[l].Y [rows][m_l].
// Two launches for all layers together: the stacked first product, the batched second product (Sec. 4.4, Eq. 11-12); where the
// first one is split, one more that adds the slices (layers that are split differently: as many of each).
int forward_prefill_planned_multi_bf16(const PfArgs *p, int n_layers, const int32_t *plan, int cap, uint16_t *const *Z,
                                       int avg_prompt_rows, hipStream_t s) {
  if (n_layers < 1 || n_layers > LG_MAX_LAYERS) return PARSE_ESHAPE;
  LgArgs g1{};
  g1.n_layers = n_layers;
  g1.plan = plan;
  g1.tok_offsets = p[0].tok_offsets; g1.pattern_id = p[0].pattern_id;
  g1.rows = p[0].rows; g1.NP = p[0].n_patterns;
  g1.cap = cap;
  const int rows = p[0].rows, P = p[0].P;
  // one prompt has less than a 256-row tile of padding, prompts of one length in whole tiles (most likely) have none: leaving
  // padding tiles out of the numbering costs a launch 1 us
  g1.compact = P > 1 && !(rows % P == 0 && rows / P % 256 == 0);
  LgArgs g2 = g1;
  bool slices64 = true;                        // the second product can take slices of 64
  for (int l = 0; l < n_layers; ++l) {
    if (p[l].sh_ranks % 32 != 0 || p[l].sh_ranks >= p[l].rS) return PARSE_ESHAPE;
    const int own = p[l].rS - p[l].sh_ranks;   // ranks in a pattern's own block
    g1.L[l] = LgLayer{p[l].X, p[l].Vt_S, Z[l], nullptr, (size_t)own * p[l].n, p[l].n, p[l].rS, p[l].Vt_sh, p[l].sh_ranks / 32, 0};
    g2.L[l] = LgLayer{Z[l], p[l].Ut_S, p[l].Y, nullptr, (size_t)own * p[l].m, p[l].rS, p[l].m, p[l].Ut_sh, p[l].sh_ranks / 32, 0};
    slices64 = slices64 && p[l].sh_ranks == 0 && p[l].rS % 64 == 0;
  }
  const int per_pattern = avg_prompt_rows / 256;
  // First product, layers of one number of slices together.  Up to SHORT_ROWS rows every tile takes the reduction in two halves
  // (WK 2, slices of 64), beyond it none does: which tile a call takes depends on the layers it fuses, its bits do not.
  int slices[LG_MAX_LAYERS];
  for (int l = 0; l < n_layers; ++l) slices[l] = split_slices(p[l]);
  for (int ks = 1; ks <= 4; ++ks) {
    LgArgs g = g1;
    const PfArgs *lay[LG_MAX_LAYERS];
    int most = 0, st;
    g.n_layers = 0;
    for (int l = 0; l < n_layers; ++l) {
      if (slices[l] != ks) continue;
      lay[g.n_layers] = &p[l];
      g.L[g.n_layers] = g1.L[l];
      if (ks > 1)      // the partial sums follow the layer's Z in the workspace
        g.L[g.n_layers].Pz = reinterpret_cast<float *>(reinterpret_cast<char *>(Z[l]) + planned_z_only_bytes(cap, p[l].rS));
      most = std::max(most, p[l].rS);
      ++g.n_layers;
    }
    if (g.n_layers == 0) continue;
    if (ks > 1) {
      g.ks = ks;
      if (rows > 1024) st = launch_gemm_lds<128, 256, 2, 2, 64, 3, 0, 1, 0, 1, 2>(g, per_pattern, s);
      else st = launch_gemm_lds<64, 64, 2, 2, 64, 4, 0, 1, 0, 1, 2>(g, per_pattern, s);
      if (st != PARSE_OK) return st;
      const size_t pieces = (size_t)cap * 8 * (most / 16) * 64;
      const int wgs = (int)std::min<size_t>((pieces + 255) / 256, 2048);
      hipLaunchKernelGGL((g.plan ? z_combine<0> : z_combine<1>), dim3(wgs, g.n_layers), dim3(256), 0, s, g, wgs);
      PARSE_LAUNCH_CHECK();
      continue;
    }
    const int tile = best_tile(lay, g.n_layers);
    if (rows <= SHORT_ROWS) {
      if (tile == T64) st = launch_gemm_lds<64, 64, 2, 2, 64, 4, 0, 1, 0, 0, 2>(g, per_pattern, s);
      else if (tile == T64x128) st = launch_gemm_lds<64, 128, 2, 2, 64, 4, 0, 1, 0, 0, 2>(g, per_pattern, s);
      else if (tile == T128) st = launch_gemm_lds<128, 128, 2, 2, 64, 4, 0, 1, 0, 0, 2>(g, per_pattern, s);
      else if (tile == T128x192) st = launch_gemm_lds<128, 192, 2, 2, 64, 4, 0, 1, 0, 0, 2>(g, per_pattern, s);
      else st = launch_gemm_lds<128, 256, 2, 2, 64, 3, 0, 1, 0, 0, 2>(g, per_pattern, s);
    } else if (tile == T64) st = launch_gemm_lds<64, 64, 2, 2, 64, 5, 0, 1, 0>(g, per_pattern, s);      // many rows, few ranks
    else if (tile == T64x128) st = launch_gemm_lds<64, 128, 2, 2, 64, 4, 0, 1, 0>(g, per_pattern, s);
    else if (tile == T128) st = launch_gemm_lds<128, 128, 2, 4, 64, 5, 0, 1, 0>(g, per_pattern, s);
    else if (tile == T128x256) st = launch_gemm_lds<128, 256, 2, 4, 64, 3, 0, 1, 0>(g, per_pattern, s);
    else st = g.plan ? launch_first256<0>(g, per_pattern, s) : launch_first256<1>(g, per_pattern, s);
    if (st != PARSE_OK) return st;
  }

  auto tiles2 = [&](int bm, int bn) { long long t = 0; for (int l = 0; l < n_layers; ++l) t += (p[l].m + bn - 1) / bn; return t * token_tiles(rows, P, bm); };
  // Second product: 256 x 256 tiles where their number is as good as known and they fill their rounds, or there are many; else 128 x 256,
  // two to a compute unit, whose stores and starts overlap and whose last round is shorter; smaller tiles as these run out
  // (both products, n = 4096, us, 256 x 256 / 128 x 256 / 128 x 128 / 64 x 128 / 64 x 64: eight prompts of 512 rows x 4096 columns, 1024 ranks 68 / 68 / 70 /
  // 76 / 87, of 4096 465 / 474 / 487 / 553 / 638; one prompt, 768 ranks: 2048 rows x 12288 columns 69 / 59 / 62 / 69 / 83, 2048 x 4096 45 / 39 / 39 / 40 / 45,
  // 1100 x 4096 47 / 40 / 40 / 38 / 42; 77 x 4096, 1024 ranks 34 / 27 / 22 / 20 / 18; n = 1024, 1533 rows of 40 prompts x 1024 columns, 512 ranks 32 / 27 / 27 / 26 / 29).
  const long long u256 = tiles2(256, 256);
  const bool full = rows % P == 0 && rows / P % 256 == 0 && (double)u256 >= 0.88 * 256 * ((u256 + 255) / 256);
  if (full || u256 >= 1792) return launch_gemm_lds<256, 256, 2, 4, 32, 5, 1, 0, 1>(g2, per_pattern, s);
  if (tiles2(128, 256) >= 384) return launch_gemm_lds<128, 256, 2, 2, 32, 3, 1, 0, 1>(g2, per_pattern, s);
  if (tiles2(128, 128) >= 384) return launch_gemm_lds<128, 128, 2, 2, 32, 3, 1, 0, 1>(g2, per_pattern, s);
  if (slices64 && tiles2(64, 128) <= 160) return launch_gemm_lds<64, 64, 2, 2, 64, 4, 1, 0, 1>(g2, per_pattern, s);
  return launch_gemm_lds<64, 128, 2, 2, 32, 4, 1, 0, 1>(g2, per_pattern, s);
}

int forward_prefill_planned_bf16(const PfArgs &p, const int32_t *plan, int cap, uint16_t *Z, int avg_prompt_rows,
                                 hipStream_t s) {
  uint16_t *Zs[1] = {Z};
  return forward_prefill_planned_multi_bf16(&p, 1, plan, cap, Zs, avg_prompt_rows, s);
}

}  // namespace parse
