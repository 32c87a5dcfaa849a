// a7: decode step for bf16 PARSE_MFMA16 layers (Sec. 4.3, "Rank Reuse for Decoding"): every sequence keeps the
// rank subset chosen at prefill; one token per sequence.  Bandwidth-bound: the kernels stream each rank group that
// ANY sequence of the batch selected exactly once, straight from the layer's factor store in operand order
// (1 KiB coalesced per wavefront instruction, no packed copies), and apply it to all sequences at once on the
// matrix cores (32 sequences = the N side of a 32x32x16 instruction).  A sequence whose pattern does not hold a
// group gets a zero in that group's part of z, so it contributes nothing.
//
// Decode plan (Sec. 4.3: the subsets are fixed after prefill, so everything derived from them is computed once per
// batch, not once per step): per layer the sequence mask of every group, the ascending list of groups selected by at
// least one sequence and their count, plus the arrival counters of decode_zr's split reduction.  decode_plan_build
// writes it; the kernels below read it (decode_zr also draws and resets its tickets there).
//
// Two launches per step:
//   decode_zr  one workgroup per 32-rank block of a used group (operand-order layers have groups of whole blocks) and slice
//              of the reduction range: the Vt operands go straight into registers, all of a wavefront's at once; the x
//              rows of the slice are staged in LDS; long reductions are cut in slices whose partial sums the last
//              workgroup of a ticket adds in slice order.  z ends up masked, rounded to bf16 and stored as operands of
//              the second product.
//   decode_y   NC (1..4) 32-column output blocks per workgroup; the eight wavefronts split the used reduction blocks,
//              all Ut operands requested up front; LDS reduction in wavefront order.
// Up to sixteen sequences leave half or more of the 32-wide N side empty and take other kernels with a finer split of the
// work: decode_zv / decode_zp (eight ranks a task on the 16 x 16 x 32 matrix instruction) while x fits the LDS, decode_y16 (sixteen columns), and one to
// four sequences with little to do decode_yv on the vector units (sixteen or thirty-two columns).  More than 32 sequences: decode_wide_bf16.hip.
// What bounds all of them: HBM, and what a compute unit takes in.  A unit has at most 32 KiB outstanding and gets it back in order, 57 GB/s of a mixture of
// cached and uncached lines, so every byte of x or z that a workgroup reads again counts like one of the factor; a launch costs 1.9 us, and the plan, the first
// loads and the sums about 4 more.
// Horizontal fusion (Sec. 4.4, Eq. 11-12): up to DEC_MAX_LAYERS layers that read the SAME x (Q/K/V, gate/up) go
// through the same two launches together -- each launch's grid is the concatenation of the layers' task lists.
// No floating-point atomics; the summation order is fixed: same inputs, same bits.
#include <algorithm>

#include "prefill_common.hpp"
#include "decode_tasks.hpp"

namespace parse {

constexpr int DY_WAVES = 8, DY_THREADS = DY_WAVES * 64;
constexpr int DEC_MAXG = 64;
constexpr int DY_CHUNK = 4;                // decode_y: operands per chunk after the first block
constexpr int DY_MAXKB = 1024;             // selected reduction blocks a decode_y workgroup can list
constexpr int DEC_TICKETS = 512;           // 32-rank blocks of the largest layer (R = 16384)
constexpr int DEC_PLAN_WORDS = 192 + DEC_TICKETS;   // per layer: [0] count, [1..64] used group ids, [65..128] sequence masks,
                                                    // [192..) arrival counters of the split reduction (zero between calls)

#define PARSE_DEC_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
#define PARSE_DEC_GLB_PTR(p) ((const __attribute__((address_space(1))) void *)(p))

struct DecLayer {
  const uint16_t *Vt, *Ut;
  uint16_t *y;
  uint16_t *zf;                // workspace: z of this layer in operand order
  const int32_t *plan;         // this layer's DEC_PLAN_WORDS of the decode plan
  float *zpart;                // workspace: partial sums of z, [R/32][KS][16][64] floats (KS > 1)
  int32_t *ticket;             // [DEC_TICKETS] arrival counters in the plan, one per 32-rank block
  int R, G, gs, m;
  int z_first, y_first;        // first workgroup of this layer in decode_zr and decode_zp / decode_y
  int z_wgs;                   // decode_zp: workgroups of this layer
};
struct DecArgs {
  DecLayer L[DEC_MAX_LAYERS];
  int n_layers;
  const uint16_t *x;
  int B, n;
  int KS;                      // decode_zr: slices of the reduction range
};

struct DecPlanArgs {
  const int32_t *subsets[DEC_MAX_LAYERS];
  int stride[DEC_MAX_LAYERS], k[DEC_MAX_LAYERS], n_patterns[DEC_MAX_LAYERS], G[DEC_MAX_LAYERS];
  const int32_t *pattern_id;
  int B;
  int32_t *plan;
};

// Factor operands: each line is read once in the launch.  NT: past the caches (which calls, is decided where the kernels are launched).
template <bool NT>
__device__ __forceinline__ u32x4 stream_load(const void *p) {
  const u32x4 *q = reinterpret_cast<const u32x4 *>(p);
  return NT ? __builtin_nontemporal_load(q) : *q;
}
__device__ __forceinline__ bf16x8 dec_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// The blocks (of 16 or 32 ranks, `per` to a group) of the groups in use, counted through: one load of the plan puts the used ids
// in a register of the 64 lanes, a block's place follows by arithmetic and a lane read.  A list in LDS put two barriers and two LDS
// round trips between the plan and the first factor load: decode_y16 5.5 -> 5.0 and 8.4 -> 7.8 us a launch.  (decode_y keeps its list: the
// step of 32 sequences was 0.4 us slower without; so does decode_yv, which asks for the blocks of four lanes' groups at a time.)
struct DecUsed {
  int ids, count, per;
  float inv;
  __device__ __forceinline__ DecUsed(const DecLayer &ly, int lane, int per_group) : per(per_group), inv(1.0f / (float)per_group) {
    ids = ly.plan[1 + lane];
    count = max(0, min(ly.plan[0], ly.G)) * per;
  }
  // exact: i < 1024, and (i + 1/2) / per is at least 1/2048 off every integer
  __device__ __forceinline__ int block(int i) const {        // i the same for all lanes, below count
    const int g = __builtin_amdgcn_readfirstlane((int)(((float)i + 0.5f) * inv));
    return max(__builtin_amdgcn_readlane(ids, g), 0) * per + i - g * per;
  }
};

// A task of a first product: 2^shift ranks of a group in use.  Each layer's tasks are counted through over its groups in use.  decode_zv, a workgroup a task:
// the layers take turns, so that the workgroups without one are the last of the grid (of layers with equally many): up to one task a compute unit is then one task a
// unit (numbered over all groups some units got two and some none: 11008 -> 4096 columns, one sequence, four ranks a workgroup, 11.0 us, 8.5 this way).
// decode_zp, several tasks a workgroup: each layer has workgroups of its own (dec_share).
struct DecTask {
  int unit;                    // unit < 0: none
  uint32_t mask;               // sequences whose pattern holds the unit's group
};
__device__ __forceinline__ int dec_layer_of(const DecArgs &a, int bid, int &at) {
  at = a.n_layers == 1 ? bid : a.n_layers == 2 ? bid >> 1 : a.n_layers == 4 ? bid >> 2 : bid / 3;
  return bid - at * a.n_layers;
}
// ids and masks: the plan's words of the lane
__device__ __forceinline__ DecTask dec_task(const DecLayer &ly, int used, int ids, int masks, int at, int shift) {
  const int per = ly.gs >> shift, count = max(0, min(used, ly.G)) * per;
  const int g = min(__builtin_amdgcn_readfirstlane(dec_group_of(at, per)), DEC_MAXG - 1);
  const int id = min(max(__builtin_amdgcn_readlane(ids, g), 0), ly.G - 1);
  return DecTask{at < count ? id * per + at - g * per : -1, (uint32_t)__builtin_amdgcn_readlane(masks, id)};
}

// a barrier without the usual one's fence, which waits for every outstanding load: what this wavefront wrote to LDS is there
__device__ __forceinline__ void dec_lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// grid = layers, one wavefront each: lane b < B looks at its sequence's k group ids and ORs its bit into the groups'
// masks (LDS, integer OR: order-free); then the used groups are listed in ascending order by a vote.
__global__ __launch_bounds__(64) void decode_plan_build(DecPlanArgs a) {
  __shared__ uint32_t gmask[DEC_MAXG];
  const int l = blockIdx.x, lane = threadIdx.x;
  int32_t *out = a.plan + (size_t)l * DEC_PLAN_WORDS;
  gmask[lane] = 0u;
  __syncthreads();
  const int G = a.G[l];
  if (lane < a.B && lane < 32) {
    const int pid = a.pattern_id[lane];
    if (pid >= 0 && pid < a.n_patterns[l]) {
      for (int i = 0; i < a.k[l]; ++i) {
        const int g = a.subsets[l][(size_t)pid * a.stride[l] + i];
        if (g >= 0 && g < G) atomicOr(&gmask[g], 1u << lane);
      }
    }
  }
  __syncthreads();
  __shared__ int32_t used_l[DEC_MAXG];
  const bool u = lane < G && gmask[lane] != 0u;
  const unsigned long long votes = __ballot(u);
  used_l[lane] = -1;
  __syncthreads();
  if (u) used_l[__popcll(votes & ((1ull << lane) - 1ull))] = lane;
  __syncthreads();
  out[1 + lane] = used_l[lane];
  out[65 + lane] = (int32_t)gmask[lane];
  if (lane == 0) out[0] = __popcll(votes);
  for (int i = lane; i < DEC_TICKETS; i += 64) out[192 + i] = 0;
}

// ---------------------------------------------------------------------------------------------------------
// decode_zr.  Workgroup = (layer, 32-rank block, slice s of KS of the reduction range).  A slice is at most 256 reduction steps (4096 columns): each of the eight wavefronts
// owns an eighth of it and requests ALL its Vt operands at once, straight into registers (1 KiB coalesced per
// instruction, up to 32 of them): the registers of the eight wavefronts are the staging buffer.  Up to 256 KiB are asked for, of which a
// unit has 32 KiB on their way; the others wait in its queue, so that it never runs dry, and LDS is left to x.
// The x rows of the slice are staged in LDS (loads that write LDS directly; 512-byte row segments, 16-byte pieces
// XOR-swizzled by the row so that an operand read -- 32 rows x the same piece -- spreads over the banks), at most 128
// steps at a time.  TWO == false (slices of up to 128 steps): one wait, one barrier, then the products run from registers
// and LDS.  TWO == true: the slice is staged in two halves; a wavefront's operands are ordered first half, second half,
// so the products of the first half run while the second half of the factor stream is still arriving, and the second
// half of x -- requested as soon as the first is consumed, long before the stream ends -- is there when it does.
// The eight wavefronts' sums are added in wavefront order through LDS.
// KS == 1: the block's z is masked, rounded to bf16 and stored as operands of the second product.
// KS  > 1: the workgroup stores its partial sum (fp32) and takes a ticket of its rank block; the workgroup that draws
// the last ticket adds the KS partial sums in slice order (not in arrival order: same inputs, same bits) and stores the
// operands.  Nobody waits for anybody: a workgroup that is not the last simply ends.  The tickets live in the decode plan
// (zeroed when the plan is built, reset by the last workgroup), so a plan serves one decode call at a time.
constexpr int DR_WAVES = 8, DR_THREADS = DR_WAVES * 64;
constexpr int DR_MAXK = 32;                  // Vt operands a wavefront requests (its eighth of the slice)
constexpr int DR_SEG_KB = 16;                // reduction steps per staged x segment (256 columns, 512 bytes per row)
constexpr int DR_SEG_BYTES = 32 * 512;       // 16 KiB
constexpr int DR_MAXSEG = 8;                 // segments staged at a time: 128 steps, 128 KiB
constexpr int DR_HALF_KB = DR_MAXSEG * DR_SEG_KB;    // 128
constexpr int DR_MAX_KS = 16;
constexpr int DR_TARGET_WGS = 240;           // workgroups wanted per launch: a little under one per compute unit

// lane (j, q) holds s[e] = ranks 8*(e/4) + 4*q + e%4 of sequence j of a 32-rank block: mask, round, pair the bands into
// 8 consecutive ranks and store the two z operands (reduction blocks rb*2, rb*2+1 of the second product)
__device__ __forceinline__ void dec_store_z_operands(const float (&s)[16], uint32_t mask, int lane, uint16_t *zf, int rb) {
  const bool member = (mask >> (lane & 31)) & 1u;     // a sequence outside the group's mask gets zeros
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t p0x = member ? cvt_pk_bf16(s[(2 * h) * 4 + 0], s[(2 * h) * 4 + 1]) : 0u;
    const uint32_t p0y = member ? cvt_pk_bf16(s[(2 * h) * 4 + 2], s[(2 * h) * 4 + 3]) : 0u;
    const uint32_t p1x = member ? cvt_pk_bf16(s[(2 * h + 1) * 4 + 0], s[(2 * h + 1) * 4 + 1]) : 0u;
    const uint32_t p1y = member ? cvt_pk_bf16(s[(2 * h + 1) * 4 + 2], s[(2 * h + 1) * 4 + 3]) : 0u;
    // after the swap lane (j, q) holds the 8 consecutive ranks rb*32 + 16h + 8q + (0..7) of sequence j
    const u32x2 sx = __builtin_amdgcn_permlane32_swap(p0x, p1x, false, false);
    const u32x2 sy = __builtin_amdgcn_permlane32_swap(p0y, p1y, false, false);
    *reinterpret_cast<u32x4 *>((char *)zf + (size_t)(rb * 2 + h) * 1024 + lane * 16) = u32x4{sx[0], sy[0], sx[1], sy[1]};
  }
}

// ROWS: 32, or 16 where no more sequences are there: half of x's loads, 15.6 -> 14.5 us for twelve sequences of 11008 columns, 2048 ranks (the upper rows of the
// staged segments are then whatever was there, and so are the sums of sequences that nobody stores)
template <bool TWO, int ROWS, bool NT>
__global__ __launch_bounds__(DR_THREADS) void decode_zr(DecArgs a) {
  constexpr int HK = DR_MAXK / 2;            // TWO: operands per half and wavefront
  int li = 0;
#pragma unroll
  for (int i = 1; i < DEC_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].z_first) ? 1 : 0;
  const DecLayer &ly = a.L[li];
  const int KS = a.KS;
  const int bid = blockIdx.x - ly.z_first;
  const int rb = bid / KS, sl = bid % KS;
  const int n = a.n, B = a.B, gs = ly.gs;
  // sequences whose pattern holds this block's group; a block nobody selected is neither read nor written
  const uint32_t mask = (uint32_t)ly.plan[65 + (rb * 32) / gs];
  if (mask == 0u) return;
  __shared__ __attribute__((aligned(1024))) char xs[DR_MAXSEG * DR_SEG_BYTES];
  __shared__ int32_t am_last;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int j = lane & 31, q = lane >> 5;
  const int nkb = n / 16;
  const int ks0 = (int)(((long long)nkb * sl) / KS), ks1 = (int)(((long long)nkb * (sl + 1)) / KS);
  const int cnt_wg = ks1 - ks0;                         // <= 8 * DR_MAXK, and <= DR_HALF_KB unless TWO (the host picks KS so)
  // the slice in one part (A) or two (A, B); x segments are counted from the start of the slice
  const int nseg = (cnt_wg + DR_SEG_KB - 1) / DR_SEG_KB;
  const int nsegA = TWO ? (nseg + 1) / 2 : nseg;        // <= DR_MAXSEG
  const int cntA = min(cnt_wg, nsegA * DR_SEG_KB), cntB = cnt_wg - cntA;
  const int a0 = (cntA * wave) / DR_WAVES, cntAw = (cntA * (wave + 1)) / DR_WAVES - a0;   // this wavefront's steps of part A
  const int b0 = (cntB * wave) / DR_WAVES, cntBw = (cntB * (wave + 1)) / DR_WAVES - b0;   // ... of part B (<= HK each if TWO)
  const int last_piece = n / 8 - 1;
  // x segments [s0, s0 + ns) of the slice into LDS slots 0..ns-1: a segment is 16 instructions of 1 KiB (two rows of 512
  // bytes each).  Lane l writes slot l % 32 of row 2*ins + l / 32 and fetches the piece (slot ^ (row & 15)) of that row's
  // segment; pieces past the end of the row re-read its last one (their products are switched off below)
  auto stage_x = [&](int s0, int ns) {
#pragma unroll
    for (int u = 0; u < DR_MAXSEG * ROWS / 2 / DR_WAVES; ++u) {
      const int t = wave + u * DR_WAVES;                 // instruction id: segment, row pair
      if (t < ns * (ROWS / 2)) {                         // uniform
        const int seg = t / (ROWS / 2), ins = t % (ROWS / 2);
        const int r = ins * 2 + (lane >> 5);
        const int piece = min(ks0 * 2 + (s0 + seg) * 32 + ((lane & 31) ^ (r & 15)), last_piece);
        __builtin_amdgcn_global_load_lds(PARSE_DEC_GLB_PTR((const char *)a.x + (size_t)min(r, B - 1) * n * 2 + (size_t)piece * 16),
                                         PARSE_DEC_LDS_PTR(xs + seg * DR_SEG_BYTES + ins * 1024), 16, 0, 0);
      }
    }
  };
  // lane's x operand of step kl (counted from the first staged segment)
  auto x_operand = [&](int kl) -> u32x4 {
    return *reinterpret_cast<const u32x4 *>(xs + (kl >> 4) * DR_SEG_BYTES + j * 512 + ((((kl & 15) * 2 + q) ^ (j & 15)) * 16));
  };
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  const u32x4 zero = {0, 0, 0, 0};
  const char *vrow = (const char *)ly.Vt + ((size_t)rb * nkb + ks0) * 1024;   // uniform; operand k of the slice at + k KiB
  const int vlane = lane * 16;
  u32x4 vr[DR_MAXK];
  if (!TWO) {
    // ---- all Vt operands of this wavefront, requested at once (steps past the count re-read the last one) ----
#pragma unroll
    for (int g = 0; g < HK / 4; ++g) {                   // a slice of up to 128 steps: up to HK per wavefront
      if (g * 4 < cntAw) {                               // uniform
#pragma unroll
        for (int ii = 0; ii < 4; ++ii)
          vr[g * 4 + ii] = stream_load<NT>(vrow + (size_t)(a0 + min(g * 4 + ii, cntAw - 1)) * 1024 + vlane);
      } else {
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) vr[g * 4 + ii] = zero;
      }
    }
    stage_x(0, nsegA);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                     // everybody's x rows are in LDS
#pragma unroll
    for (int g = 0; g < HK / 4; ++g) {
      if (g * 4 < cntAw) {                               // uniform
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) {
          const int i = g * 4 + ii;
          const u32x4 xv = x_operand(min(a0 + i, cntA - 1));
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dec_bf16x8(vr[i]), dec_bf16x8(i < cntAw ? xv : zero), acc, 0, 0, 0);
        }
      }
    }
  } else {
    // ---- Two stagings.  Here the x rows go through registers (16 loads of 1 KiB per wavefront and half, then 16 LDS
    // writes): with plain loads the compiler counts every outstanding load exactly, so the products of part A start while
    // the operands of part B are still in flight (it does not do that across loads that write LDS directly).  Every
    // wavefront issues the same number of loads whatever the counts are -- instructions past the end repeat the last
    // one (same data to the same place) -- first half of x, operands of part A, operands of part B ----
    constexpr int XI = DR_MAXSEG * 16 / DR_WAVES * ROWS / 32;        // x instructions per wavefront and half
    auto x_src = [&](int s0, int ns, int u) -> const char * {
      const int t = min(wave + u * DR_WAVES, ns * (ROWS / 2) - 1);
      const int seg = t / (ROWS / 2), ins = t % (ROWS / 2);
      const int r = ins * 2 + (lane >> 5);
      const int piece = min(ks0 * 2 + (s0 + seg) * 32 + ((lane & 31) ^ (r & 15)), last_piece);
      return (const char *)a.x + (size_t)min(r, B - 1) * n * 2 + (size_t)piece * 16;
    };
    auto x_dst = [&](int ns, int u) -> char * {          // wave-uniform slot + the lane's 16 bytes
      const int t = min(wave + u * DR_WAVES, ns * (ROWS / 2) - 1);
      return xs + t / (ROWS / 2) * DR_SEG_BYTES + t % (ROWS / 2) * 1024 + lane * 16;
    };
    auto bare_barrier = [&]() {     // the usual barrier comes with a fence that waits for every outstanding load
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    u32x4 xr[XI];
#pragma unroll
    for (int u = 0; u < XI; ++u) xr[u] = *reinterpret_cast<const u32x4 *>(x_src(0, nsegA, u));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < HK; ++i)
      vr[i] = stream_load<NT>(vrow + (size_t)(a0 + min(i, max(cntAw - 1, 0))) * 1024 + vlane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < HK; ++i)
      vr[HK + i] = stream_load<NT>(vrow + (size_t)min(cntA + b0 + min(i, max(cntBw - 1, 0)), cnt_wg - 1) * 1024 + vlane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < XI; ++u) *reinterpret_cast<u32x4 *>(x_dst(nsegA, u)) = xr[u];
    bare_barrier();                                      // everybody's share of the first half of x is in LDS
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < HK; ++i) {
      const u32x4 xv = x_operand(min(a0 + i, cntA - 1));
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dec_bf16x8(vr[i]), dec_bf16x8(i < cntAw ? xv : zero), acc, 0, 0, 0);
      if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);     // a few x operands in registers at a time, not all sixteen
    }
    bare_barrier();                                      // everybody is done with the first half of x
    __builtin_amdgcn_sched_barrier(0);
    const int nsegB = max(nseg - nsegA, 1);
#pragma unroll
    for (int u = 0; u < XI; ++u) xr[u] = *reinterpret_cast<const u32x4 *>(x_src(min(nsegA, nseg - 1), nsegB, u));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < XI; ++u) *reinterpret_cast<u32x4 *>(x_dst(nsegB, u)) = xr[u];
    bare_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int offB = cntA - nsegA * DR_SEG_KB;           // first step of part B counted from the first segment staged now (0)
#pragma unroll
    for (int i = 0; i < HK; ++i) {
      const u32x4 xv = x_operand(max(0, min(offB + b0 + i, offB + cntB - 1)));
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dec_bf16x8(vr[HK + i]), dec_bf16x8(i < cntBw ? xv : zero), acc, 0, 0, 0);
      if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();        // the staged rows are dead: their LDS now takes the wavefronts' sums
  float(*red)[16][64] = reinterpret_cast<float(*)[16][64]>(xs);               // [8][16][64] floats = 32 KiB
  float *sums = reinterpret_cast<float *>(xs + 32768);                        // [16][64]
#pragma unroll
  for (int e = 0; e < 16; ++e) red[wave][e][lane] = acc[e];
  __syncthreads();
  // the eight sums of each value, in wavefront order; value v = (e, lane)
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int v = (int)threadIdx.x + u * DR_THREADS;
    const float *r0 = &red[0][0][0] + v;
    float sum = r0[0];
#pragma unroll
    for (int w = 1; w < DR_WAVES; ++w) sum += r0[w * 1024];
    if (KS == 1) sums[v] = sum;
    else           // device-scope store: written through to memory, past this die's (non-coherent) L2
      __hip_atomic_store(&ly.zpart[((size_t)rb * KS + sl) * 1024 + v], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (KS == 1) {
    __syncthreads();
    if (wave == 0) {
      float s[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = sums[e * 64 + lane];
      dec_store_z_operands(s, mask, lane, ly.zf, rb);
    }
    return;
  }
  // ---- ticket.  The partial sums and the ticket are device-scope accesses (they go past the die's L2, which is not
  // coherent with the other dies'), so no cache has to be written back or invalidated as a device-scope fence would do
  // (that would also throw away the x rows and factor lines the other workgroups of the die are using): every thread
  // waits until its own stores are acknowledged, the barrier collects all of them, then thread 0 draws ----
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int t = __hip_atomic_fetch_add(&ly.ticket[rb], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = t == KS - 1 ? 1 : 0;
    if (last) __hip_atomic_store(&ly.ticket[rb], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
    am_last = last;
  }
  __syncthreads();
  if (!am_last) return;
  // the last workgroup of the block: all KS partial sums are in memory; read them past the L2 as well, add in slice order
  if (wave == 0) {
    float s[16];
    const float *zp = ly.zpart + (size_t)rb * KS * 1024 + lane;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = __hip_atomic_load(zp + e * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int o = 1; o < KS; ++o) {
      float t[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) t[e] = __hip_atomic_load(zp + (size_t)o * 1024 + e * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] += t[e];
    }
    dec_store_z_operands(s, mask, lane, ly.zf, rb);
  }
}

// ---------------------------------------------------------------------------------------------------------
// decode_zv: z for a handful of sequences (B <= 4; which calls of two to four come here is decided where the kernels are launched).
// With one to four sequences the 32-wide N side of the matrix instruction is almost empty and, worse, a
// 32-rank block per workgroup leaves most compute units without work (one sequence selects k groups: a 4096x4096 layer with 8 groups of 96 ranks has 24 blocks for 256 units).  Here a
// task is EIGHT ranks of a block (or four: JW) over the whole reduction range: in the operand order the 16-byte pieces of 8
// consecutive ranks are 128 contiguous bytes, so a wavefront instruction reads 8 such lines (4 reduction steps x 2
// halves), every line exactly once in the launch.  The 16 x 16 x 32 matrix instruction multiplies them: its sixteen rows are the
// task's ranks in 16 / JW parts of the reduction range, its sixteen columns the sequences (all of x sits in LDS) in the same parts, and what row and
// column of one part make is of use.  On the vector units, 36 instructions a load, this was the slower (one sequence, four calls of a 4096 x 11008 block, us:
// 7.9 + 5.6 + 7.6 + 9.7, with workgroups numbered over all groups; 7.1 + 4.6 + 5.8 + 7.3 now).  The result is masked, rounded and stored like decode_zr's; no
// partial sums leave the workgroup.
// The sums: an instruction's product of 32 columns goes to one of its lane's four running sums, and those, the parts and the wavefronts (in LDS) are added by pairs.
// What the roundings add up to, rms, in units of 2^-24 of the root of the sum of the products' squares (products that cancel, so that all of the result is
// rounding), 1024 / 2048 / 4096 / 11008 columns: 0.91 / 1.01 / 1.11 / 1.28.  One running sum a lane, parts and wavefronts in order: 1.11 / 1.21 / 1.25 to 1.32 /
// 1.54 to 1.69; on the vector units 0.90 / 1.00 / 1.15 / 1.47; a 16-wide kernel with one sum over all columns 1.06 / 1.45 / 2.05 / 3.49; decode_zr 0.97 / 1.11 / 1.30
// / 2.10.
constexpr int DV_SUMS = 4;                   // running sums of a lane, one for every fourth instruction

// v[0..N), a power of two of them, by pairs, pairs of pairs, ...
template <int N, class T>
__device__ __forceinline__ T pair_sum(T (&v)[N]) {
#pragma unroll
  for (int d = 1; d < N; d *= 2)
#pragma unroll
    for (int i = 0; i < N; i += 2 * d) v[i] += v[i + d];
  return v[0];
}

constexpr int DV_WAVES = 8, DV_THREADS = DV_WAVES * 64;
constexpr int DV_XBYTES = 96 * 1024;         // most LDS the x rows may take
constexpr int DV_MAXB = 4;
constexpr int dv_red_bytes(int JW) { return DV_WAVES * 16 * JW * 4; }       // the wavefronts' sums

__device__ __host__ __forceinline__ int dv_xstride(int n) { return n * 2 + ((n & 127) == 0 ? 128 : 0); }   // bytes between x rows in LDS

// XP pieces of x and DEPTH factor operands a lane: what is past the counts repeats the last one, so that no load stands behind a branch (the compiler
// waits for all loads where the two sides of one meet)
template <int JW, int XP, int DEPTH, bool NT>
__global__ __launch_bounds__(DV_THREADS) void decode_zv(DecArgs a) {
  constexpr int C = 16 / JW;                 // parts of an instruction's reduction range
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int at;
  const int li = dec_layer_of(a, blockIdx.x, at);
  const DecLayer &ly = a.L[li];
  // eight ranks; JW == 4: one half of them, the other half (of the same 128-byte lines) goes to a workgroup of the same die
  const int half = JW == 4 ? (at >> 3) & 1 : 0;
  const DecTask task = dec_task(ly, ly.plan[0], ly.plan[1 + lane], ly.plan[65 + lane], JW == 4 ? (at >> 4) * 8 + (at & 7) : at, 3);
  if (task.unit < 0) return;
  const int rb = task.unit >> 2, j0 = (task.unit & 3) * 8 + half * 4;
  const int n = a.n, B = a.B, nkb = n / 16;
  extern __shared__ __attribute__((aligned(16))) char xs[];      // B rows of x: several workgroups fit a compute unit
  __shared__ __attribute__((aligned(16))) float red[DV_WAVES][C][JW][JW];            // [wavefront][part][sequence][rank]
  static_assert(sizeof(red) == dv_red_bytes(JW), "");
  const int r = (lane & 15) % JW, part = (lane & 15) / JW, kq = lane >> 4;           // rank and sequence, part, 8 of its 32 reduction indices
  const int pieces = n / 8, xstride = dv_xstride(n), all = B * pieces;
  u32x4 xr[XP];
#pragma unroll
  for (int u = 0; u < XP; ++u) xr[u] = *reinterpret_cast<const u32x4 *>((const char *)a.x + (size_t)min(u * DV_THREADS + (int)threadIdx.x, all - 1) * 16);
  const char *vbase = (const char *)ly.Vt + (size_t)rb * nkb * 1024 + ((kq & 1) * 32 + j0 + r) * 16;
  auto step = [&](int i) { return ((wave + i * DV_WAVES) * C + part) * 2 + (kq >> 1); };       // of this wavefront's instruction i, this lane
  u32x4 v[DEPTH];
  auto request = [&](int i0) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) v[u] = stream_load<NT>(vbase + (size_t)min(step(i0 + u), nkb - 1) * 1024);
  };
  __builtin_amdgcn_sched_barrier(0);
  request(0);
  __builtin_amdgcn_sched_barrier(0);
  const float inv = 1.0f / (float)pieces;
  auto keep = [&](int i, u32x4 w) {          // piece i of the rows; exact: i < 2^14, and (i + 1/2) / pieces is at least 2^-14 off every integer
    const int row = (int)(((float)i + 0.5f) * inv);
    *reinterpret_cast<u32x4 *>(xs + row * xstride + (i - row * pieces) * 16) = w;
  };
#pragma unroll
  for (int u = 0; u < XP; ++u) keep(min(u * DV_THREADS + (int)threadIdx.x, all - 1), xr[u]);
#pragma unroll 1
  for (int i = XP * DV_THREADS + (int)threadIdx.x; i < all; i += DV_THREADS)
    keep(i, *reinterpret_cast<const u32x4 *>((const char *)a.x + (size_t)i * 16));
  dec_lds_barrier();
  const char *xrow = xs + min(r, B - 1) * xstride + (kq & 1) * 16;
  f32x4 acc[DV_SUMS];
#pragma unroll
  for (int i = 0; i < DV_SUMS; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0;;) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      const int kb = step(i0 + u);
      const u32x4 xv = *reinterpret_cast<const u32x4 *>(xrow + min(kb, nkb - 1) * 32);
      const bool on = kb < nkb;              // else both are cleared: an infinite weight times zero is no number
      acc[u % DV_SUMS] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(dec_bf16x8(on ? v[u] : u32x4{0, 0, 0, 0}), dec_bf16x8(on ? xv : u32x4{0, 0, 0, 0}), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    i0 += DEPTH;
    if ((wave + i0 * DV_WAVES) * C * 2 >= nkb) break;      // uniform
    request(i0);
  }
  // lane (column lane % 16, g) holds rows 4 g .. 4 g + 3: of use where row and column are of the same part
  if ((kq * 4) / JW == part) *reinterpret_cast<f32x4 *>(&red[wave][part][r][(kq * 4) % JW]) = pair_sum(acc);
  __syncthreads();
  if (threadIdx.x < JW * JW) {               // thread (sequence, rank)
    const int b = threadIdx.x / JW, e = threadIdx.x % JW;
    float zs[DV_WAVES * C];
#pragma unroll
    for (int i = 0; i < DV_WAVES * C; ++i) zs[i] = red[i / C][i % C][b][e];
    const float z = pair_sum(zs);
    const float next = __shfl_down(z, 1, 64);
    if (b < B && !(e & 1))                   // zeros outside the group's mask
      *reinterpret_cast<uint32_t *>((char *)ly.zf + (size_t)(rb * 2 + (j0 >> 4)) * 1024 + (((j0 >> 3) & 1) * 32 + b) * 16 + ((j0 & 7) + e) * 2) =
          ((task.mask >> b) & 1u) ? cvt_pk_bf16(z, next) : 0u;
  }
}

// ---------------------------------------------------------------------------------------------------------
// decode_zp: decode_zv's tasks of eight ranks for up to sixteen sequences, with x, all of it, staged once per compute unit: one workgroup a unit takes
// tasks of its layer in turn.  A task is done in chunks of DEPTH factor operands a wavefront; the next chunk, of this task or the next one, is on its way while
// one is multiplied.  Bound by what a unit takes in: x once and its share of the factor, where a workgroup of sixteen ranks that reads x for itself takes
// in as much of x as of the factor and a unit with two of them twice that (twelve sequences, a 4096 x 11008 block, us: q/k/v 14.1 -> 10.5, o 8.2 -> 6.1,
// gate/up 9.6 -> 9.0; a call of 512 ranks 15.2 (32-wide) / 10.9 / 9.2).
constexpr int DP_MAXB = 16;
constexpr int DP_LDS = 160 * 1024 - 512;     // x and the wavefronts' sums

__device__ __host__ constexpr int dp_red_bytes(int NX) { return 2 * DV_WAVES * 2 * NX * 8 * 8 * 4; }

// NX groups of eight sequences, XP pieces of x a thread asks for at once; ONE: a task is one chunk
template <int NX, int XP, int DEPTH, bool ONE, bool NT>
__global__ __launch_bounds__(DV_THREADS) void decode_zp(DecArgs a) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n = a.n, B = a.B, nkb = n / 16;
  extern __shared__ __attribute__((aligned(16))) char xs[];      // B rows of x
  __shared__ __attribute__((aligned(16))) float red[2][DV_WAVES][2][NX * 8][8];      // [turn][wavefront][part][sequence][rank]
  static_assert(sizeof(red) == dp_red_bytes(NX), "");
  const int r = lane & 7, part = (lane >> 3) & 1, kq = lane >> 4;                    // rank and sequence, part, 8 of its 32 reduction indices
  const int pieces = n / 8, xstride = dv_xstride(n), all = B * pieces;
  const int chunks = ONE ? 1 : (nkb + 4 * DV_WAVES * DEPTH - 1) / (4 * DV_WAVES * DEPTH);
  auto step = [&](int i) { return ((wave + i * DV_WAVES) * 2 + part) * 2 + (kq >> 1); };       // of this wavefront's instruction i of a task, this lane
  int li = 0;
#pragma unroll
  for (int i = 1; i < DEC_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].z_first) ? 1 : 0;
  const DecLayer &ly = a.L[li];
  const int used = ly.plan[0], ids = ly.plan[1 + lane], masks = ly.plan[65 + lane];
  __builtin_amdgcn_sched_barrier(0);
  struct Task {
    int unit;                                // < 0: none
    uint32_t mask;
    const char *V;                           // this lane's factor; without a task all lanes read the same 16 bytes
    int stride;
  };
  auto task_of = [&](int at) {
    const DecTask t = dec_task(ly, used, ids, masks, at, 3);
    const bool on = t.unit >= 0;
    return Task{t.unit, t.mask,
                on ? (const char *)ly.Vt + (size_t)(t.unit >> 2) * nkb * 1024 + ((kq & 1) * 32 + (t.unit & 3) * 8 + r) * 16 : (const char *)a.x,
                on ? 1024 : 0};
  };
  u32x4 xr[XP], v0[DEPTH], v1[DEPTH];
  auto request = [&](const Task &t, int chunk, u32x4 (&v)[DEPTH]) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) v[u] = stream_load<NT>(t.V + (size_t)min(step(chunk * DEPTH + u), nkb - 1) * t.stride);
  };
  const float inv = 1.0f / (float)pieces;
  auto keep = [&](int i, u32x4 w) {          // piece i of the rows; exact: i < 2^14, and (i + 1/2) / pieces is at least 2^-14 off every integer
    const int row = (int)(((float)i + 0.5f) * inv);
    *reinterpret_cast<u32x4 *>(xs + row * xstride + (i - row * pieces) * 16) = w;
  };
#pragma unroll
  for (int u = 0; u < XP; ++u) xr[u] = *reinterpret_cast<const u32x4 *>((const char *)a.x + (size_t)min(u * DV_THREADS + (int)threadIdx.x, all - 1) * 16);
  __builtin_amdgcn_sched_barrier(0);
  int at = (int)blockIdx.x - ly.z_first, chunk = 0;
  Task task = task_of(at);
  if (task.unit < 0) return;                 // uniform; no later place has a task either
  request(task, 0, v0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < XP; ++u) keep(min(u * DV_THREADS + (int)threadIdx.x, all - 1), xr[u]);
#pragma unroll 1
  for (int i = XP * DV_THREADS + (int)threadIdx.x; i < all; i += DV_THREADS)
    keep(i, *reinterpret_cast<const u32x4 *>((const char *)a.x + (size_t)i * 16));
  dec_lds_barrier();
  const char *xrow[NX];
  f32x4 acc[NX][DV_SUMS];
  auto clear = [&]() {
#pragma unroll
    for (int h = 0; h < NX; ++h)
#pragma unroll
      for (int i = 0; i < DV_SUMS; ++i) acc[h][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
#pragma unroll
  for (int h = 0; h < NX; ++h) xrow[h] = xs + min(h * 8 + r, B - 1) * xstride + (kq & 1) * 16;
  clear();
  int which = 0;
  // multiplies the chunk in v, the next one on its way into w; false after the last task
  auto turn = [&](const u32x4 (&v)[DEPTH], u32x4 (&w)[DEPTH]) -> bool {
    const Task now = task;
    const int c = ONE ? 0 : chunk;
    if (ONE || ++chunk == chunks) {          // uniform
      chunk = 0;
      at += ly.z_wgs;
      task = task_of(at);
    }
    request(task, ONE ? 0 : chunk, w);
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      const int kb = step(c * DEPTH + u), xat = min(kb, nkb - 1) * 32;
      const bool on = kb < nkb;              // else both are cleared: an infinite weight times zero is no number
      const u32x4 vv = on ? v[u] : u32x4{0, 0, 0, 0};
#pragma unroll
      for (int h = 0; h < NX; ++h) {
        const u32x4 xv = *reinterpret_cast<const u32x4 *>(xrow[h] + xat);
        acc[h][u % DV_SUMS] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(dec_bf16x8(vv), dec_bf16x8(on ? xv : u32x4{0, 0, 0, 0}), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      }
    }
    if (!ONE && chunk != 0) return true;     // uniform
    if ((kq >> 1) == part) {
#pragma unroll
      for (int h = 0; h < NX; ++h) *reinterpret_cast<f32x4 *>(&red[which][wave][part][h * 8 + r][(kq & 1) * 4]) = pair_sum(acc[h]);
    }
    dec_lds_barrier();
    if (threadIdx.x < NX * 64) {             // thread (sequence, rank)
      const int b = threadIdx.x >> 3, e = threadIdx.x & 7;
      float zs[DV_WAVES * 2];
#pragma unroll
      for (int i = 0; i < DV_WAVES * 2; ++i) zs[i] = red[which][i >> 1][i & 1][b][e];
      const float z = pair_sum(zs);
      const float next = __shfl_down(z, 1, 64);
      if (b < B && !(e & 1))                 // zeros outside the group's mask
        *reinterpret_cast<uint32_t *>((char *)ly.zf + (size_t)(now.unit >> 1) * 1024 + ((now.unit & 1) * 32 + b) * 16 + e * 2) =
            ((now.mask >> b) & 1u) ? cvt_pk_bf16(z, next) : 0u;
    }
    which ^= 1;                              // the other place: this one is read until the next barrier
    clear();
    return task.unit >= 0;
  };
  while (turn(v0, v1) && turn(v1, v0)) {}
}

// ---------------------------------------------------------------------------------------------------------
// decode_y: y.  grid = ceil(ncb / NC) workgroups per layer, each owns NC consecutive 32-column output blocks;
// wavefront w owns an eighth of the used reduction blocks for all NC column blocks, so one z operand (cache-resident)
// feeds NC products; the Ut operands of its first MAXK reduction blocks are requested at once (MAXK sized so that
// everything stays in registers), the rest is streamed in chunks; the eight wavefronts add up through LDS.
template <int NC, bool NT>
__global__ __launch_bounds__(DY_THREADS) void decode_y(DecArgs a) {
  int li = 0;
#pragma unroll
  for (int i = 1; i < DEC_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].y_first) ? 1 : 0;
  const DecLayer &ly = a.L[li];
  const uint16_t *__restrict__ Ut = ly.Ut;
  const uint16_t *__restrict__ zf = ly.zf;
  const int32_t *__restrict__ plan = ly.plan;
  uint16_t *__restrict__ y = ly.y;
  const int B = a.B, m = ly.m, G = ly.G, gs = ly.gs;
  const int bid = blockIdx.x - ly.y_first;
  __shared__ float red[DY_WAVES][16][64];
  __shared__ int32_t kb_list[DY_MAXKB];
  __shared__ int32_t used[DEC_MAXG];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, q = lane >> 5;
  const int ncb = m / 32;
  const int c0 = bid * NC;
  const int nc = min(NC, ncb - c0);
  // count and ids come from the plan in one round trip (ids past the count are -1 and not used)
  const int n_used_raw = plan[0];
  if (threadIdx.x < DEC_MAXG) used[threadIdx.x] = plan[1 + threadIdx.x];
  const int n_used = max(0, min(n_used_raw, G));
  __syncthreads();
  const int kpg = gs / 16;                 // reduction blocks per group
  const int total_kb = n_used * kpg;       // selected reduction blocks
  for (int i = threadIdx.x; i < total_kb; i += DY_THREADS) kb_list[i] = max(used[i / kpg], 0) * kpg + i % kpg;
  __syncthreads();
  const int k0 = (total_kb * wave) / DY_WAVES, k1 = (total_kb * (wave + 1)) / DY_WAVES;
  const int cnt = k1 - k0;
  const uint16_t *ubase = Ut + ((size_t)c0 * 64 + lane) * 8;
  const uint16_t *zbase = zf + (size_t)lane * 8;
  const size_t ustep = (size_t)ncb * 512;
  int coff[NC];   // element offset of column block j's operand; blocks past the end re-read block 0 (result unused)
#pragma unroll
  for (int j = 0; j < NC; ++j) coff[j] = j < nc ? j * 512 : 0;
  f32x16 acc[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
  const u32x4 zero = {0, 0, 0, 0};
  constexpr int DY_MAXK = NC == 1 ? 20 : (NC == 2 ? 16 : (NC == 3 ? 12 : 8));
  constexpr int DEC_CHUNK = DY_CHUNK;
  if (cnt > 0) {
    u32x4 ur[DY_MAXK][NC], zr[DY_MAXK];
#pragma unroll
    for (int i = 0; i < DY_MAXK; ++i) zr[i] = *reinterpret_cast<const u32x4 *>(zbase + (size_t)kb_list[k0 + min(i, cnt - 1)] * 512);
    __builtin_amdgcn_sched_barrier(0);       // z, which is cached, ahead of the factor: loads come back in order (one column block a workgroup 9.0 -> 8.1 us)
#pragma unroll
    for (int i = 0; i < DY_MAXK; ++i) {
      const int kb = kb_list[k0 + min(i, cnt - 1)];
#pragma unroll
      for (int j = 0; j < NC; ++j) ur[i][j] = stream_load<NT>(ubase + (size_t)kb * ustep + coff[j]);
    }
    __builtin_amdgcn_sched_barrier(0);   // every fetch above is in flight before the first product
#pragma unroll
    for (int i = 0; i < DY_MAXK; ++i) {
      const u32x4 zv = i < cnt ? zr[i] : zero;
#pragma unroll
      for (int j = 0; j < NC; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dec_bf16x8(ur[i][j]), dec_bf16x8(zv), acc[j], 0, 0, 0);
    }
    for (int c = DY_MAXK; c < cnt; c += DEC_CHUNK) {
      u32x4 uu[DEC_CHUNK][NC], zz[DEC_CHUNK];
#pragma unroll
      for (int i = 0; i < DEC_CHUNK; ++i) {
        const int kb = kb_list[k0 + min(c + i, cnt - 1)];
#pragma unroll
        for (int j = 0; j < NC; ++j) uu[i][j] = stream_load<NT>(ubase + (size_t)kb * ustep + coff[j]);
        zz[i] = *reinterpret_cast<const u32x4 *>(zbase + (size_t)kb * 512);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < DEC_CHUNK; ++i) {
        const u32x4 zv = (c + i < cnt) ? zz[i] : zero;
#pragma unroll
        for (int j = 0; j < NC; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dec_bf16x8(uu[i][j]), dec_bf16x8(zv), acc[j], 0, 0, 0);
      }
    }
  }
  // per column block: add the wavefronts' contributions in wave order and store
#pragma unroll
  for (int jl = 0; jl < NC; ++jl) {
    if (jl < nc) {   // uniform
#pragma unroll
      for (int e = 0; e < 16; ++e) red[wave][e][lane] = acc[jl][e];
      __syncthreads();
      for (int i = threadIdx.x; i < 16 * 64; i += DY_THREADS) {
        const int e = i >> 6, ln = i & 63;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < DY_WAVES; ++w) sum += red[w][e][ln];
        red[0][e][ln] = sum;   // each (e, ln) is read and written by this thread only
      }
      __syncthreads();
      if (wave == 0 && l32 < B) {
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
          u32x2 w;
          w[0] = pack_bf16x2(red[0][blk * 4 + 0][lane], red[0][blk * 4 + 1][lane]);
          w[1] = pack_bf16x2(red[0][blk * 4 + 2][lane], red[0][blk * 4 + 3][lane]);
          *reinterpret_cast<u32x2 *>(y + (size_t)l32 * m + (c0 + jl) * 32 + blk * 8 + q * 4) = w;
        }
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// decode_yv: y for a handful of sequences (B <= 4, while there is little to do), on the vector units -- the counterpart of
// decode_zv.  decode_y feeds z to the matrix cores as a 32-sequence operand (1 KiB per reduction block whatever B is) that every workgroup re-reads;
// here z is a few values per rank: a workgroup copies the B sequences' pieces of the used reduction blocks into LDS once
// (16 bytes per block half and sequence) and then streams nothing but Ut.  Workgroup = 8 * CG consecutive output columns
// of one layer (CG = 2 or 4 groups of 8 columns: 128-byte lines of the operand order, each read once in the launch);
// wavefront w owns column group w % CG and every (8 / CG)-th instruction of the used reduction blocks, 4 blocks per
// instruction: lane (block s of 4, half q, column j of 8) multiplies its 8 Ut values with the 8 matching z values of
// each sequence.  The 8 lanes of a column are added by a butterfly, the wavefronts of a column group through LDS in
// wavefront order; one 16-byte store per sequence and column group.
constexpr int DYV_WAVES = 8, DYV_THREADS = DYV_WAVES * 64;
constexpr int DYV_DEPTH = 16;                // Ut loads a lane has in flight
constexpr int DYV_ZBYTES = 96 * 1024;        // most LDS the z pieces may take
constexpr int dyv_own_bytes(int NB) { return (DY_MAXKB + DEC_MAXG + DYV_WAVES * NB * 8) * 4; }         // the kernel's own arrays

template <int NB, int CG, bool NT>
__global__ __launch_bounds__(DYV_THREADS) void decode_yv(DecArgs a) {
  constexpr int PARTS = DYV_WAVES / CG;      // wavefronts that share a column group
  int li = 0;
#pragma unroll
  for (int i = 1; i < DEC_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].y_first) ? 1 : 0;
  const DecLayer &ly = a.L[li];
  const int32_t *__restrict__ plan = ly.plan;
  const int B = a.B, m = ly.m, G = ly.G, gs = ly.gs;
  const int bid = blockIdx.x - ly.y_first;
  extern __shared__ __attribute__((aligned(16))) char zs[];          // [used reduction block][half][NB] pieces of 16 bytes
  __shared__ int32_t kb_list[DY_MAXKB];
  __shared__ int32_t used[DEC_MAXG];
  __shared__ float red[DYV_WAVES][NB][8];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int jl = lane & 7, q = (lane >> 3) & 1, ks = lane >> 4;
  const int cg = wave % CG, part = wave / CG;
  const int ncb = m / 32;
  const int col0 = (bid * CG + cg) * 8;                              // first column of this wavefront's group
  const int n_used_raw = plan[0];
  if (threadIdx.x < DEC_MAXG) used[threadIdx.x] = plan[1 + threadIdx.x];
  const int n_used = max(0, min(n_used_raw, G));
  __syncthreads();
  const int kpg = gs / 16;
  const int total_kb = n_used * kpg;
  for (int i = threadIdx.x; i < total_kb; i += DYV_THREADS) kb_list[i] = max(used[i / kpg], 0) * kpg + i % kpg;
  __syncthreads();
  // z pieces of the used blocks: piece (i, h, b) = ranks kb_list[i]*16 + 8h .. +7 of sequence b (zeros for b >= B)
  for (int t = threadIdx.x; t < total_kb * 2 * NB; t += DYV_THREADS) {
    const int b = t % NB, h = (t / NB) & 1, i = t / (2 * NB);
    u32x4 w = {0, 0, 0, 0};
    if (b < B) w = *reinterpret_cast<const u32x4 *>((const char *)ly.zf + (size_t)kb_list[i] * 1024 + (h * 32 + b) * 16);
    *reinterpret_cast<u32x4 *>(zs + (size_t)t * 16) = w;
  }
  const int ninstr = (total_kb + 3) / 4;
  const int nw = col0 < m ? (ninstr - part + PARTS - 1) / PARTS : 0;  // instructions of this wavefront: part, part + PARTS, ...
  // column col0 + jl sits in column block c / 32 at place c % 32 of the operand
  const int cc = min(col0, m - 8) + jl;
  const char *ubase = (const char *)ly.Ut + (size_t)(cc >> 5) * 1024 + (q * 32 + (cc & 31)) * 16;
  const size_t ustep = (size_t)ncb * 1024;
  u32x4 v[DYV_DEPTH];
  auto request = [&](int i0) {               // lanes past the last block re-read it (switched off when used)
#pragma unroll
    for (int u = 0; u < DYV_DEPTH; ++u) {
      if (i0 + u < nw) {                     // uniform
        const int i = min(((part + (i0 + u) * PARTS) << 2) + ks, total_kb - 1);
        v[u] = stream_load<NT>(ubase + (size_t)kb_list[i] * ustep);
      }
    }
  };
  request(0);
  __syncthreads();                           // the z pieces are in LDS
  float acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = 0.f;
  for (int i0 = 0; i0 < nw; i0 += DYV_DEPTH) {
#pragma unroll
    for (int u = 0; u < DYV_DEPTH; ++u) {
      if (i0 + u >= nw) break;               // uniform
      const int ir = ((part + (i0 + u) * PARTS) << 2) + ks;
      const bool on = ir < total_kb;
      const int i = min(ir, total_kb - 1);
      const u32x4 uv = v[u];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const u32x4 zv = *reinterpret_cast<const u32x4 *>(zs + (size_t)((i * 2 + q) * NB + b) * 16);
        float t = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          t += __uint_as_float(uv[e] << 16) * __uint_as_float(zv[e] << 16);
          t += __uint_as_float(uv[e] & 0xFFFF0000u) * __uint_as_float(zv[e] & 0xFFFF0000u);
        }
        acc[b] += on ? t : 0.f;
      }
    }
    if (i0 + DYV_DEPTH < nw) request(i0 + DYV_DEPTH);   // uniform
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    float t = acc[b];
    t += __shfl_xor(t, 8, 64);
    t += __shfl_xor(t, 16, 64);
    t += __shfl_xor(t, 32, 64);
    if (lane < 8) red[wave][b][lane] = t;
  }
  __syncthreads();
  if ((int)threadIdx.x < CG * NB) {          // thread (column group, sequence): 8 columns = one 16-byte store
    const int g2 = threadIdx.x / NB, b = threadIdx.x % NB;
    const int c = (bid * CG + g2) * 8;
    if (b < B && c < m) {
      u32x4 out;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int pt = 0; pt < PARTS; ++pt) { s0 += red[pt * CG + g2][b][2 * e]; s1 += red[pt * CG + g2][b][2 * e + 1]; }
        out[e] = pack_bf16x2(s0, s1);
      }
      *reinterpret_cast<u32x4 *>(ly.y + (size_t)b * m + c) = out;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// decode_y16: y for up to sixteen sequences (which calls of two to four come here is decided where the kernels are launched), on the 16x16x32 matrix
// instruction.  The 32-wide kernel leaves half of its N side empty there and owns 32 columns per workgroup (too few workgroups: a 4096-column
// layer has 128 column blocks for 256 units).  Here the M side is 16
// columns: in the operand order 16 rows x 32 reduction indices are four runs of 256 bytes, a wavefront instruction reads
// whole lines, every line once in the launch.  Everything goes straight from memory into registers; the eight wavefronts
// of a workgroup split the reduction and share nothing until their sums meet in LDS.
// Same rounding points, plan and workspace as the other decode kernels.  Bound by HBM and by the launch's latency: 5.0 us for 11 MB, 8.8 for 33 MB.
// A wavefront's steps take SUMS running sums in turn, those and the wavefronts are added by pairs: roundings as above, 512 / 1024 / 1536 / 2048 ranks 0.77 / 0.90 / 1.00 /
// 1.05 (two blocks and more a workgroup 1.18), one sum a wavefront and wavefronts in order 0.80 / 1.05 / 1.24 / 1.44, decode_yv 0.76 / 0.90 / 0.98 / 1.05; no more
// than 0.1 us of 5.
typedef __attribute__((ext_vector_type(4))) float f32x4_acc;
constexpr int D16_WAVES = 8, D16_THREADS = D16_WAVES * 64, D16_MAXB = 16;

// NC blocks of 16 columns per workgroup; wavefront w takes every eighth 32-rank block in use.
template <int NC>
__global__ __launch_bounds__(D16_THREADS) void decode_y16(DecArgs a) {
  constexpr int DEPTH = NC <= 2 ? 12 : (NC == 3 ? 10 : (NC == 4 ? 8 : 6)), SUMS = NC == 3 || NC == 6 ? 2 : 4;
  int li = 0;
#pragma unroll
  for (int i = 1; i < DEC_MAX_LAYERS; ++i) li += (i < a.n_layers && (int)blockIdx.x >= a.L[i].y_first) ? 1 : 0;
  const DecLayer &ly = a.L[li];
  const int B = a.B, m = ly.m;
  const int c0 = ((int)blockIdx.x - ly.y_first) * NC, ncb = m / 32;
  __shared__ float red[D16_WAVES][NC][4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int r = lane & 15, kq = lane >> 4;
  const DecUsed blocks(ly, lane, ly.gs / 32);                      // 32-rank blocks in use
  const int total = blocks.count;
  const int cnt = (total - wave + D16_WAVES - 1) / D16_WAVES;
  const char *U = (const char *)ly.Ut + (size_t)(kq >> 1) * ncb * 1024 + ((kq & 1) * 32 + r) * 16;
  const char *Z = (const char *)ly.zf + (kq >> 1) * 1024 + ((kq & 1) * 32 + r) * 16;
  int coff[NC];                                                    // blocks past the end re-read the last one (not stored)
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = min(c0 + i, ncb * 2 - 1);
    coff[i] = (c >> 1) * 1024 + (c & 1) * 256;
  }
  f32x4_acc acc0[NC], acc1[NC], acc2[NC], acc3[NC];                // arrays of their own: one of all of them is moved about as a whole at every branch
#pragma unroll
  for (int i = 0; i < NC; ++i) acc0[i] = acc1[i] = acc2[i] = acc3[i] = f32x4_acc{0.f, 0.f, 0.f, 0.f};
  u32x4 ur[DEPTH][NC], zr[DEPTH];
  auto request = [&](int d, int s) {
    const int rb = blocks.block(wave + s * D16_WAVES);
#pragma unroll
    for (int i = 0; i < NC; ++i) ur[d][i] = *reinterpret_cast<const u32x4 *>(U + (size_t)rb * 2 * ncb * 1024 + coff[i]);
    zr[d] = *reinterpret_cast<const u32x4 *>(Z + (size_t)rb * 2048);
  };
  auto multiply = [&](int d, f32x4_acc (&acc)[NC]) {
#pragma unroll
    for (int i = 0; i < NC; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dec_bf16x8(ur[d][i]), dec_bf16x8(zr[d]), acc[i], 0, 0, 0);
  };
  auto in_turn = [&](auto f) {                                     // f(step, running sum) of all DEPTH steps
#pragma unroll
    for (int d = 0; d < DEPTH; d += SUMS) {
      f(d, acc0);
      f(d + 1, acc1);
      if constexpr (SUMS == 4) {
        f(d + 2, acc2);
        f(d + 3, acc3);
      }
    }
  };
  if (cnt > 0) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) request(d, min(d, cnt - 1));
    int s = 0;
    for (; s + DEPTH < cnt; s += DEPTH)
      in_turn([&](int d, f32x4_acc (&acc)[NC]) {
        __builtin_amdgcn_sched_barrier(0);
        multiply(d, acc);
        request(d, min(s + d + DEPTH, cnt - 1));
      });
    in_turn([&](int d, f32x4_acc (&acc)[NC]) {
      __builtin_amdgcn_sched_barrier(0);
      if (s + d < cnt) multiply(d, acc);                           // uniform
    });
  }
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const f32x4_acc sum = (acc0[i] + acc1[i]) + (acc2[i] + acc3[i]);
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][i][e][lane] = sum[e];
  }
  __syncthreads();
  // thread (column block, g, sequence): columns 4g..4g+3
  for (int t = threadIdx.x; t < NC * 64; t += D16_THREADS) {
    const int i = t >> 6, ln = t & 63, seq = ln & 15;
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float ys[D16_WAVES];
#pragma unroll
      for (int w = 0; w < D16_WAVES; ++w) ys[w] = red[w][i][e][ln];
      y[e] = pair_sum(ys);
    }
    if (seq < B && c0 + i < ncb * 2)
      *reinterpret_cast<u32x2 *>(ly.y + (size_t)seq * m + (c0 + i) * 16 + (ln >> 4) * 4) = u32x2{cvt_pk_bf16(y[0], y[1]), cvt_pk_bf16(y[2], y[3])};
  }
}

// workspace of one layer: z in operand order (R/16 operands of 1 KiB), then the partial sums of decode_zr
static size_t dec_zf_bytes(const parse_layer *L) { return round_up((size_t)(L->R / 16) * 1024, 256); }
// decode_zr takes reductions of up to DR_MAX_KS slices of 8 * DR_MAXK steps (n <= 65536) and layers of up to DEC_TICKETS
// rank blocks whose groups are whole 32-rank blocks (which the operand-order layout requires anyway)
static bool dec_zr_ok(const parse_layer *L) {
  if (L->G <= 0 || L->R % L->G != 0 || (L->R / L->G) % 32 != 0) return false;
  if (L->R / 32 > DEC_TICKETS) return false;
  const int nkb = L->n / 16;
  return (nkb + 8 * DR_MAXK - 1) / (8 * DR_MAXK) <= DR_MAX_KS;
}
// slices of the reduction range: enough that a slice fits a workgroup (8 * DR_MAXK steps), and enough workgroups to give
// every compute unit one
static int dec_zr_slices(const parse_layer *layers, int n_layers) {
  const int nkb = layers[0].n / 16;
  int blocks = 0;
  for (int l = 0; l < n_layers; ++l) blocks += layers[l].R / 32;
  const int need = (nkb + 8 * DR_MAXK - 1) / (8 * DR_MAXK);
  int ks = blocks > 0 ? DR_TARGET_WGS / blocks : 1;
  if (ks > nkb / 8) ks = nkb / 8;          // at least one step per wavefront
  if (ks < need) ks = need;
  if (ks > DR_MAX_KS) ks = DR_MAX_KS;
  return ks < 1 ? 1 : ks;
}
static size_t dec_zpart_bytes(const parse_layer *L, int ks) { return ks > 1 ? (size_t)(L->R / 32) * ks * 4096 : 0; }
size_t decode_plan_bytes(int n_layers) { return round_up((size_t)n_layers * DEC_PLAN_WORDS * sizeof(int32_t), 256); }
// z workspace of several layers that go through one call: per layer z, then its partial sums
size_t decode_z_bytes(const parse_layer *layers, int n_layers) {
  const int ks = dec_zr_slices(layers, n_layers);
  size_t t = 0;
  for (int l = 0; l < n_layers; ++l) t += dec_zf_bytes(&layers[l]) + dec_zpart_bytes(&layers[l], ks);
  return t;
}
// one layer's intermediates, then room for a one-layer plan (used when the caller brings no plan)
size_t decode_workspace_bytes(const parse_layer *L) { return decode_z_bytes(L, 1) + decode_plan_bytes(1); }

bool decode_supported(const parse_layer *L) {
  return L->R / 16 <= DY_MAXKB && L->G <= DEC_MAXG && L->n % 16 == 0 && L->n >= 16 && dec_zr_ok(L);
}

int build_decode_plan(const parse_layer *layers, const parse_patterns *pts, int n_layers, const int32_t *pattern_id,
                      int B, int32_t *plan, hipStream_t s) {
  if (n_layers < 1 || n_layers > DEC_MAX_LAYERS) return PARSE_ESHAPE;
  DecPlanArgs pa{};
  for (int l = 0; l < n_layers; ++l) {
    pa.subsets[l] = pts[l].subsets; pa.stride[l] = pts[l].subset_stride; pa.k[l] = pts[l].k;
    pa.n_patterns[l] = pts[l].n_patterns; pa.G[l] = layers[l].G;
  }
  pa.pattern_id = pattern_id; pa.B = B; pa.plan = plan;
  hipLaunchKernelGGL(decode_plan_build, dim3(n_layers), dim3(64), 0, s, pa);
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

// Which kernel makes z.  Up to sixteen sequences whose x fits the LDS: decode_zv, many small workgroups that each stage x, for one sequence, for so few tasks that
// none waits for a unit (up to 128 units of eight ranks, which decode_zv halves), or for many tasks of little x; decode_zp, x once per unit, otherwise.
// The 32-wide kernel where x does not fit.  us a call of one layer (or three) with 512 columns of output, half of the groups in up to three patterns, over layers of 0.7
// gigabytes in turn, decode_zv / decode_zp / 32-wide, by sequences x columns (decode_zv takes four sequences):
//    512 ranks: 1 x 2816  6.7 / 7.6 / 13.1     4 x 2816   7.8 / 8.4 / 15.1     4 x 11008 13.2 / 14.6 / 17.8    12 x 2816  - / 9.2 / 15.7
//   1024 ranks: 1 x 2816  7.4 / 8.1 / 10.8     2 x 11008 13.1 / 14.4 / 15.7    4 x 5632  12.4 / 12.4 / 15.2    4 x 11008 14.2 / 15.5 / 16.8
//               6 x 11008  - / 15.3 / 16.7     12 x 5632   - / 13.2 / 15.1
//   2048 ranks: 1 x 4096  9.0 / 9.2 / 12.6     2 x 4096  12.1 / 11.4 / 14.3    4 x 4096  12.3 / 11.4 / 14.9    12 x 4096  - / 12.5 / 15.2
//               1 x 11008 12.1 / 13.8 / 17.2   2 x 11008 19.4 / 16.2 / 19.5    4 x 8192  18.5 / 15.3 / 19.2
//   2560 ranks: 1 x 11008 12.9 / 13.1 / 17.0   2 x 11008 17.3 / 16.1 / 19.8    4 x 11008 22.8 / 19.9 / 19.7    6 x 11008  - / 19.8 / 19.7
//   3 x 1536:   1 x 4096  11.3 / 11.4 / 15.7   2 x 4096  13.1 / 13.3 / 17.3    4 x 4096  15.0 / 14.7 / 17.8    12 x 4096  - / 15.5 / 18.0
// Unlike layers: decode_zv's take turns, so beyond the shorter ones' ends only every second to fourth workgroup has a task, and the dispatcher hands those
// to a half or a quarter of the units.  decode_zv / decode_zp, one sequence x columns, tasks of the layers: x 12624, 24 + 16 + 32 + 176 24.8 / 13.9; x 12832, 192 + 64 19.7 / 14.6;
// x 8592, 128 + 152 + 176 + 80 26.0 / 17.8; x 4096, 192 + 64 + 64 11.2 / 10.4; x 4096, 256 + 64 10.5 / 11.0; x 5504, 80 + 96 + 64 9.8 / 10.3.
static bool z_many_workgroups(int B, int n, int n_layers, int units, int most) {
  if (most * n_layers != units && ((n_layers > 2 && units > 256) || most * n_layers * (units <= 256 ? 2 : 1) > 640)) return false;
  return B == 1 || units <= 128 || (units > 256 && B * n <= 12288);
}

// Factors past the caches: a call whose layers are about a fifth of the last-level cache (256 MiB) or more.  What a call cannot see is whether the program's
// factors all stay in that cache: then it costs, and beyond it gains.  A program with calls of this size fits the cache only if it has no more than five of them, so the
// line is drawn for those that do not.  It goes by what is stored: the groups in use are known on the device only.  us a pass, ordinary loads / as chosen, the factors
// of one state again and again, of three and of 32 (seven gigabytes) in turn, 4096 x 11008:
//   block (273 MiB)   1 sequence  49.5 / 48.8   55.2 / 52.7   57.7 / 55.5        MLP (221 MiB)   1  34.7 / 35.7   39.8 / 36.1    40.6 / 38.0
//                    12           82.0 / 81.5   88.8 / 82.7   88.6 / 86.8                       12  55.6 / 59.2   64.2 / 59.1    64.0 / 61.8
//                    32          100.5 / 101.1 108.0 / 100.6 107.7 / 105.6                      32  62.1 / 66.6   71.7 / 66.6    71.4 / 66.4
//   MLP              64           68.0 / 74.2   79.2 / 71.7   78.9 / 75.8                       96  76.0 / 85.0   92.0 / 81.1    92.0 / 88.0
//                   128           79.0 / 82.9   97.3 / 94.7   97.3 / 94.2                      150  87.4 / 90.1  106.5 / 103.9  106.0 / 103.5
// 83 random calls above the line (one to 200 sequences) take 0.83 to 1.02 of the time beyond the cache, 0.95 in the middle, one 1.05; one call repeated, its factors in
// the cache, 1.05 in the middle, up to 1.28, one 1.45.  Smaller calls are those of programs that may fit the cache.  Ordinary / past the caches for all calls, one state, three, as many as make 0.9 to 1.5 gigabytes:
//   block of 2048 x 5632 (61 MiB)    1 sequence  34.2 / 33.5  35.6 / 36.1  41.5 / 37.2    32  64.8 / 66.6  65.1 / 70.4  72.1 / 70.5
//   block of 1024 x 2816 (19 MiB)    1           28.7 / 28.7  31.2 / 30.4  36.8 / 32.9    32  58.1 / 59.6  60.2 / 63.5  66.2 / 65.1
// decode_y16 keeps ordinary loads in either: 32 states, without / with, block of 4 78.6 / 79.0, of 12 86.9 / 87.0, MLP of 12 61.8 / 59.7.
bool past_caches(const parse_layer *layers, int n_layers) {
  size_t bytes = 0;
  for (int l = 0; l < n_layers; ++l) bytes += (size_t)layers[l].R * ((size_t)layers[l].n + layers[l].m) * 2;
  return bytes >= (size_t)48 << 20;
}

// PARSE_ALLOW_LDS, raised to the most that any call asks for: it holds for the kernel on a device, so once is enough
#define DEC_ALLOW_LDS(kernel, own, most, bytes, dev)                                                                                     \
  do {                                                                                                                                   \
    static bool done[64] = {false};                                                                                                      \
    if ((size_t)(own) + (size_t)(bytes) > (size_t)65536 && !done[dev]) {                                                                 \
      PARSE_HIP_TRY(hipFuncSetAttribute((const void *)(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(most)));               \
      done[dev] = true;                                                                                                                  \
    }                                                                                                                                    \
  } while (0)

// n_layers layers that share x (same n); plan = n_layers consecutive layer plans; Y[l] and the z part of layer l in the
// workspace follow the order of `layers`.
int forward_decode_planned_bf16(const parse_layer *layers, int n_layers, const uint16_t *x, int B, int32_t *plan,
                                uint16_t *const *Y, void *workspace, hipStream_t s) {
  if (n_layers < 1 || n_layers > DEC_MAX_LAYERS) return PARSE_ESHAPE;
  static int n_cu_of[64] = {0};
  int dev = 0;
  PARSE_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return PARSE_EINVAL;
  if (n_cu_of[dev] == 0) {
    hipDeviceProp_t prop;
    PARSE_HIP_TRY(hipGetDeviceProperties(&prop, dev));
    n_cu_of[dev] = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  }
  const int n_cu = n_cu_of[dev];
  DecArgs a{};
  a.n_layers = n_layers;
  a.x = x;
  a.B = B;
  a.n = layers[0].n;
  for (int l = 0; l < n_layers; ++l) {
    if (!decode_supported(&layers[l])) return PARSE_ESHAPE;
    if (layers[l].n != a.n) return PARSE_ESHAPE;
  }
  // column blocks per workgroup (one z operand feeds NC products): the smallest count that puts at most one
  // workgroup on a compute unit -- a unit with two streams runs both at half the rate and sets the kernel's time
  int NC = 1;
  for (; NC < 4; ++NC) {
    int wgs = 0;
    for (int l = 0; l < n_layers; ++l) wgs += (layers[l].m / 32 + NC - 1) / NC;
    if (wgs <= n_cu) break;
  }
  const int KS = dec_zr_slices(layers, n_layers);
  a.KS = KS;
  char *ws = reinterpret_cast<char *>(workspace);
  int zb = 0, yb = 0;
  for (int l = 0; l < n_layers; ++l) {
    const parse_layer *L = &layers[l];
    DecLayer &d = a.L[l];
    d.Vt = (const uint16_t *)L->Vt;
    d.Ut = (const uint16_t *)L->Ut;
    d.y = Y[l];
    d.zf = reinterpret_cast<uint16_t *>(ws);
    ws += dec_zf_bytes(L);
    d.zpart = reinterpret_cast<float *>(ws);
    ws += dec_zpart_bytes(L, KS);
    d.plan = plan + (size_t)l * DEC_PLAN_WORDS;
    d.ticket = plan + (size_t)l * DEC_PLAN_WORDS + 192;
    d.R = L->R; d.G = L->G; d.gs = L->R / L->G; d.m = L->m;
    d.z_first = zb; zb += (L->R / 32) * KS;
    d.y_first = yb; yb += (L->m / 32 + NC - 1) / NC;
  }
  const int nkb = a.n / 16;
  const int NB = B <= 1 ? 1 : (B <= 2 ? 2 : 4);
  const bool nt = past_caches(layers, n_layers);
  int units = 0, most = 0;                                 // tasks of eight ranks in the first product, of all layers and of the largest
  for (int l = 0; l < n_layers; ++l) { units += layers[l].R / 8; most = std::max(most, layers[l].R / 8); }
  const bool zv = B <= DV_MAXB && (size_t)B * dv_xstride(a.n) <= (size_t)DV_XBYTES && z_many_workgroups(B, a.n, n_layers, units, most);
  const bool zp = !zv && B <= DP_MAXB && (size_t)B * dv_xstride(a.n) + dp_red_bytes(B <= 8 ? 1 : 2) <= (size_t)DP_LDS;
  if (zv) {
    // a handful of sequences: eight ranks per workgroup, four where that leaves units without work
    const int jw = units <= n_cu ? 4 : 8;
    int wgs = 0;
    for (int l = 0; l < n_layers; ++l) wgs = std::max(wgs, jw == 4 ? (layers[l].R / 8 + 7) / 8 * 16 : layers[l].R / 8);
    wgs *= n_layers;
    const int share = ((nkb + 32 / jw - 1) / (32 / jw) + DV_WAVES - 1) / DV_WAVES;       // instructions of a wavefront
    const size_t lds = (size_t)B * dv_xstride(a.n);
    const int xp = (B * (a.n / 8) + DV_THREADS - 1) / DV_THREADS;                        // pieces of x of a thread
#define PARSE_ZV(JW_, XP_, D_)                                                                                                              \
  do {                                                                                                                                     \
    if (nt) {                                                                                                                              \
      DEC_ALLOW_LDS((decode_zv<JW_, XP_, D_, true>), dv_red_bytes(JW_), DV_XBYTES, lds, dev);                                             \
      hipLaunchKernelGGL((decode_zv<JW_, XP_, D_, true>), dim3(wgs), dim3(DV_THREADS), lds, s, a);                                         \
    } else {                                                                                                                               \
      DEC_ALLOW_LDS((decode_zv<JW_, XP_, D_, false>), dv_red_bytes(JW_), DV_XBYTES, lds, dev);                                            \
      hipLaunchKernelGGL((decode_zv<JW_, XP_, D_, false>), dim3(wgs), dim3(DV_THREADS), lds, s, a);                                        \
    }                                                                                                                                      \
  } while (0)
#define PARSE_ZVX(JW_, D_)                                                                     \
  do {                                                                                         \
    if (xp <= 1) PARSE_ZV(JW_, 1, D_);                                                         \
    else if (xp <= 4) PARSE_ZV(JW_, 4, D_);                                                    \
    else PARSE_ZV(JW_, 12, D_);                                                                \
  } while (0)
    if (jw == 4) { if (share <= 2) PARSE_ZVX(4, 2); else if (share <= 4) PARSE_ZVX(4, 4); else PARSE_ZVX(4, 12); }
    else { if (share <= 4) PARSE_ZVX(8, 4); else if (share <= 8) PARSE_ZVX(8, 8); else if (share <= 12) PARSE_ZVX(8, 12); else PARSE_ZVX(8, 24); }
#undef PARSE_ZVX
#undef PARSE_ZV
  } else if (zp) {
    int tasks[DEC_MAX_LAYERS], share_of[DEC_MAX_LAYERS], first = 0;
    for (int l = 0; l < n_layers; ++l) tasks[l] = layers[l].R / 8;
    const int wgs = dec_share(tasks, n_layers, n_cu, share_of);
    for (int l = 0; l < n_layers; ++l) { a.L[l].z_first = first; a.L[l].z_wgs = share_of[l]; first += share_of[l]; }
    const int share = ((nkb + 3) / 4 + DV_WAVES - 1) / DV_WAVES;
    const size_t lds = (size_t)B * dv_xstride(a.n);
    const int xp = (B * (a.n / 8) + DV_THREADS - 1) / DV_THREADS;                        // pieces of x of a thread
#define PARSE_ZP(NX_, XP_, D_, ONE_)                                                                                                        \
  do {                                                                                                                                     \
    if (nt) {                                                                                                                              \
      DEC_ALLOW_LDS((decode_zp<NX_, XP_, D_, ONE_, true>), dp_red_bytes(NX_), DP_LDS - dp_red_bytes(NX_), lds, dev);                        \
      hipLaunchKernelGGL((decode_zp<NX_, XP_, D_, ONE_, true>), dim3(wgs), dim3(DV_THREADS), lds, s, a);                                   \
    } else {                                                                                                                               \
      DEC_ALLOW_LDS((decode_zp<NX_, XP_, D_, ONE_, false>), dp_red_bytes(NX_), DP_LDS - dp_red_bytes(NX_), lds, dev);                       \
      hipLaunchKernelGGL((decode_zp<NX_, XP_, D_, ONE_, false>), dim3(wgs), dim3(DV_THREADS), lds, s, a);                                  \
    }                                                                                                                                      \
  } while (0)
    if (B <= 8) {
      if (share <= 2) PARSE_ZP(1, 2, 2, true);
      else if (share <= 4) PARSE_ZP(1, 4, 4, true);
      else if (share <= 8) PARSE_ZP(1, 8, 8, true);
      else if (share <= 12) PARSE_ZP(1, 12, 12, true);
      else PARSE_ZP(1, 16, 8, false);
    } else {
      if (share <= 2) PARSE_ZP(2, 4, 2, true);
      else if (share <= 4) PARSE_ZP(2, 8, 4, true);
      else if (share <= 8 && xp <= 12) PARSE_ZP(2, 12, 8, true);
      else if (share <= 8) PARSE_ZP(2, 16, 8, true);
      else if (share <= 12) PARSE_ZP(2, 16, 12, true);
      else PARSE_ZP(2, 16, 8, false);
    }
#undef PARSE_ZP
  } else {
    const bool two = (nkb + KS - 1) / KS > DR_HALF_KB;     // the longest slice needs two stagings of x
#define PARSE_ZR(TWO_, ROWS_)                                                                                     \
  do {                                                                                                           \
    if (nt) hipLaunchKernelGGL((decode_zr<TWO_, ROWS_, true>), dim3(zb), dim3(DR_THREADS), 0, s, a);             \
    else hipLaunchKernelGGL((decode_zr<TWO_, ROWS_, false>), dim3(zb), dim3(DR_THREADS), 0, s, a);               \
  } while (0)
    if (B <= 16) { if (two) PARSE_ZR(true, 16); else PARSE_ZR(false, 16); }
    else { if (two) PARSE_ZR(true, 32); else PARSE_ZR(false, 32); }
#undef PARSE_ZR
  }
  PARSE_LAUNCH_CHECK();
  size_t max_kb = 0;
  for (int l = 0; l < n_layers; ++l) max_kb = std::max(max_kb, (size_t)layers[l].R / 16);
  const size_t zs_bytes = max_kb * 2 * NB * 16;            // z pieces of every reduction block a layer has
  // ... and which one y: the vector units up to four sequences while there is little to do (sequences x columns x stored ranks;
  // 13 M 5.0 / 5.8, 25 M 8.0 / 6.6, 46 M 10.1 / 7.3 vector / 16-wide; four sequences, 2048 ranks and few columns 9.1 / 7.5), 16-wide up to sixteen
  // (4096 columns 6.4, 32-wide 8.1) while up to four blocks a workgroup make one round.  Beyond, six blocks a workgroup or 32-wide (us a call of 512 columns of input, three or
  // twelve sequences, factors from memory, six / 32-wide, by columns x ranks): while six make one round, up to 45 M (columns x ranks) 17408 x 64 6.5 / 9.1,
  // 2 x 9920 x 512 11.6 / 13.7, 24576 x 1536 18.1 / 18.9; 24576 x 2048 23.2 / 22.8, 2 x 11008 x 2048 26.9 / 26.2; while four 32-wide ones do and six not, up to
  // 6 M only, 28672 x 64 8.4 / 9.4, x 128 9.8 / 10.4, x 192 12.2 / 12.2, x 256 13.6 / 12.7, x 1024 19.7 / 15.7; where neither does always, 36864 x 64 8.5 / 14.0, 40960 x 1024 21.0 / 24.6,
  // 49152 x 2048 32.3 / 36.7, 65536 x 256 18.5 / 20.3, x 2048 41.7 / 40.7.
  long long y_work = 0;
  for (int l = 0; l < n_layers; ++l) y_work += (long long)layers[l].m * layers[l].R;
  // 16-column blocks per workgroup: the fewest that make one round of workgroups
  auto rounds = [&](int columns) {
    int wgs = 0;
    for (int l = 0; l < n_layers; ++l) wgs += (layers[l].m + columns - 1) / columns;
    return (wgs + n_cu - 1) / n_cu;
  };
  int nc16 = 1;
  while (nc16 <= 4 && rounds(nc16 * 16) > 1) ++nc16;
  if (nc16 > 4) {
    const bool one6 = rounds(96) == 1, one32 = rounds(128) == 1;
    nc16 = (one6 ? y_work <= 45000000 : one32 ? y_work <= 6000000 : true) ? 6 : 0;                 // 0: 32-wide
  }
  if (B <= DV_MAXB && zs_bytes <= (size_t)DYV_ZBYTES && (B == 1 || (NB * y_work <= (16ll << 20) && (B == 2 || max_kb <= 64)))) {
    // a handful of sequences: z as a few values per rank in LDS, the launch streams only Ut.  16 columns per workgroup
    // unless that makes more than about four workgroups per compute unit
    int cols = 0;
    for (int l = 0; l < n_layers; ++l) cols += layers[l].m;
    const int CG = cols / 16 > 4 * n_cu ? 4 : 2;
    yb = 0;
    for (int l = 0; l < n_layers; ++l) { a.L[l].y_first = yb; yb += (layers[l].m + 8 * CG - 1) / (8 * CG); }
#define PARSE_YV(NB_, CG_)                                                                                        \
  do {                                                                                                           \
    if (nt) {                                                                                                    \
      PARSE_ALLOW_LDS((decode_yv<NB_, CG_, true>), dyv_own_bytes(NB_), zs_bytes);                                \
      hipLaunchKernelGGL((decode_yv<NB_, CG_, true>), dim3(yb), dim3(DYV_THREADS), zs_bytes, s, a);              \
    } else {                                                                                                     \
      PARSE_ALLOW_LDS((decode_yv<NB_, CG_, false>), dyv_own_bytes(NB_), zs_bytes);                               \
      hipLaunchKernelGGL((decode_yv<NB_, CG_, false>), dim3(yb), dim3(DYV_THREADS), zs_bytes, s, a);             \
    }                                                                                                            \
  } while (0)
    if (NB == 1) { if (CG == 2) PARSE_YV(1, 2); else PARSE_YV(1, 4); }
    else if (NB == 2) { if (CG == 2) PARSE_YV(2, 2); else PARSE_YV(2, 4); }
    else { if (CG == 2) PARSE_YV(4, 2); else PARSE_YV(4, 4); }
#undef PARSE_YV
  } else if (B <= D16_MAXB && nc16 > 0) {
    yb = 0;
    for (int l = 0; l < n_layers; ++l) { a.L[l].y_first = yb; yb += (layers[l].m / 16 + nc16 - 1) / nc16; }
    if (nc16 == 1) hipLaunchKernelGGL(decode_y16<1>, dim3(yb), dim3(D16_THREADS), 0, s, a);
    else if (nc16 == 2) hipLaunchKernelGGL(decode_y16<2>, dim3(yb), dim3(D16_THREADS), 0, s, a);
    else if (nc16 == 3) hipLaunchKernelGGL(decode_y16<3>, dim3(yb), dim3(D16_THREADS), 0, s, a);
    else if (nc16 == 4) hipLaunchKernelGGL(decode_y16<4>, dim3(yb), dim3(D16_THREADS), 0, s, a);
    else hipLaunchKernelGGL(decode_y16<6>, dim3(yb), dim3(D16_THREADS), 0, s, a);
  } else {
#define PARSE_Y(NC_)                                                                                              \
  do {                                                                                                           \
    if (nt) hipLaunchKernelGGL((decode_y<NC_, true>), dim3(yb), dim3(DY_THREADS), 0, s, a);                      \
    else hipLaunchKernelGGL((decode_y<NC_, false>), dim3(yb), dim3(DY_THREADS), 0, s, a);                        \
  } while (0)
    if (NC == 1) PARSE_Y(1); else if (NC == 2) PARSE_Y(2); else if (NC == 3) PARSE_Y(3); else PARSE_Y(4);
#undef PARSE_Y
  }
  PARSE_LAUNCH_CHECK();
  return PARSE_OK;
}

// Without a caller's plan: the plan is built into the workspace (after the z parts), one more small launch.
int forward_decode_multi_bf16(const parse_layer *layers, const parse_patterns *pts, int n_layers, const uint16_t *x,
                              int B, const int32_t *pattern_id, uint16_t *const *Y, void *workspace, hipStream_t s) {
  if (n_layers < 1 || n_layers > DEC_MAX_LAYERS) return PARSE_ESHAPE;
  int32_t *plan = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(workspace) + decode_z_bytes(layers, n_layers));
  int st = build_decode_plan(layers, pts, n_layers, pattern_id, B, plan, s);
  if (st != PARSE_OK) return st;
  return forward_decode_planned_bf16(layers, n_layers, x, B, plan, Y, workspace, s);
}

int forward_decode_bf16(const parse_layer *L, const parse_patterns *pt, const uint16_t *x, int B,
                        const int32_t *pattern_id, uint16_t *y, void *workspace, hipStream_t s) {
  uint16_t *Y[1] = {y};
  return forward_decode_multi_bf16(L, pt, 1, x, B, pattern_id, Y, workspace, s);
}

}  // namespace parse
