// Body of the bucketing kernel (one workgroup of T >= P lanes, a multiple of 64), shared by the stand-alone launch and
// the launch that also builds the prefill plan.
#pragma once
#include "common.hpp"

namespace parse {

constexpr int kBucketMaxK = 64;
constexpr int kBucketMaxP = 1024;
// Up to here buckets and prefill plans are worked out in registers (bucket_wave, plan_wave).  The host chooses: with both forms in one
// kernel the other one was 0.3-0.6 us slower.
constexpr int kFewPrompts = 16;

// inclusive scan of v[0..T) in LDS, T the workgroup's lanes, a multiple of 64; every lane takes part
__device__ __forceinline__ void block_scan_inclusive(int32_t *v, int T) {
  const int p = threadIdx.x;
  for (int o = 1; o < T; o <<= 1) {
    const int add = (p >= o) ? v[p - o] : 0;
    __syncthreads();
    v[p] += add;
    __syncthreads();
  }
}

// Few prompts: one wavefront, everything in registers (P readings of a lane in place of scans in LDS, some forty barriers
// in a workgroup of 256).  All 64 lanes of the wavefront take part.  The readings are a chain that grows with P, the scans do not (us, scans /
// registers, k = 4, all alike and all different: 4 prompts 4.1 / 2.7 and 3.9 / 2.3, 16 4.4 / 4.1 and 5.3 / 3.9, 24 4.5 / 5.1 and 6.3 / 5.0, 64
// 5.1 / 10.2; k = 64, pairs alike: 16 55.9 / 55.8, 24 80 / 82).
__device__ __forceinline__ void bucket_wave(const int32_t *__restrict__ subset, int P, int k, int stride, int32_t *__restrict__ pattern_id,
                                            int32_t *__restrict__ perm, int32_t *__restrict__ bucket_off,
                                            int32_t *__restrict__ n_patterns, int32_t *__restrict__ rep) {
  const int p = threadIdx.x & 63;
  const int32_t *mine = subset + (size_t)min(p, P - 1) * stride;
  uint32_t h = 0x9E3779B9u;
#pragma unroll 8
  for (int i = 0; i < k; ++i) {
    h ^= (uint32_t)mine[i];
    h *= 0xED558CCDu;
    h ^= h >> 15;
  }
  int first = p;                           // the first prompt with the same subset
  for (int q = 0; q + 1 < P; ++q) {
    bool same = q < p && first == p && h == (uint32_t)__builtin_amdgcn_readlane((int)h, q);
    if (__ballot(same) == 0ull) continue;  // uniform
    for (int i = 0; i < k; ++i) same = same && subset[(size_t)q * stride + i] == mine[i];
    if (same) first = q;
  }
  const unsigned long long reps = __ballot(p < P && first == p);
  const int npat = __popcll(reps);
  const int pid = p < P ? __popcll(reps & ((1ull << first) - 1ull)) : 64;      // rank of the representative
  int below = 0, upto = 0, rank = 0;       // prompts of earlier patterns; of patterns up to number p; earlier ones of this pattern
  for (int q = 0; q < P; ++q) {
    const int other = __builtin_amdgcn_readlane(pid, q);
    below += other < pid ? 1 : 0;
    upto += other <= p ? 1 : 0;
    rank += q < p && other == pid ? 1 : 0;
  }
  if (p < P) {
    perm[below + rank] = p;
    pattern_id[p] = pid;
    if (first == p) rep[pid] = p;
    bucket_off[p + 1] = p < npat ? upto : P;
    if (p >= npat) rep[p] = -1;
  }
  if (p == 0) {
    bucket_off[0] = 0;
    *n_patterns = npat;
  }
}

template <bool FEW>
__device__ __forceinline__ void bucket_body(const int32_t *__restrict__ subset, int P, int k, int stride,
                                                        int32_t *__restrict__ pattern_id, int32_t *__restrict__ perm,
                                                        int32_t *__restrict__ bucket_off,
                                                        int32_t *__restrict__ n_patterns, int32_t *__restrict__ rep, int T) {
  if constexpr (FEW) {
    if (threadIdx.x < 64) bucket_wave(subset, P, k, stride, pattern_id, perm, bucket_off, n_patterns, rep);
    return;
  }
  __shared__ unsigned long long sig[1024];
  __shared__ int32_t scan[1024];   // inclusive scan of "is representative", later of the pattern sizes
  __shared__ int32_t pid[1024];
  __shared__ int32_t cnt[1025];
  const int p = threadIdx.x;
  const int32_t *mine = subset + (size_t)min(p, P - 1) * stride;
  unsigned long long h = 0x9E3779B97F4A7C15ull;
  for (int i = 0; i < k; ++i) {   // independent loads, then a sequential mix
    h ^= (unsigned long long)(uint32_t)mine[i];
    h *= 0xFF51AFD7ED558CCDull;
    h ^= h >> 29;
  }
  sig[p] = h;
  cnt[p] = 0;
  if (p == 0) cnt[T] = 0;
  __syncthreads();
  int first = p;
  if (p < P) {
    for (int q = 0; q < p; ++q) {
      if (sig[q] != h) continue;
      bool same = true;
      for (int i = 0; i < k; ++i) same = same && (subset[(size_t)q * stride + i] == mine[i]);
      if (same) { first = q; break; }
    }
  }
  const int is_rep = (p < P && first == p) ? 1 : 0;
  scan[p] = is_rep;
  __syncthreads();
  block_scan_inclusive(scan, T);
  const int npat = scan[T - 1];
  if (p < P) pid[p] = scan[first] - 1;   // representative's exclusive rank
  __syncthreads();
  if (p < P) atomicAdd(&cnt[pid[p] + 1], 1);
  __syncthreads();
  scan[p] = cnt[p + 1];                  // size of pattern p
  __syncthreads();
  block_scan_inclusive(scan, T);
  // scan[j] = number of prompts in patterns 0..j  =>  bucket_off[j+1]
  if (p < P) {
    const int j = pid[p];
    const int base = j > 0 ? scan[j - 1] : 0;
    int rank = 0;
    for (int q = 0; q < p; ++q) rank += (pid[q] == j) ? 1 : 0;
    perm[base + rank] = p;
    pattern_id[p] = j;
    if (is_rep) rep[j] = p;
    bucket_off[p + 1] = (p < npat) ? scan[p] : P;
    if (p >= npat) rep[p] = -1;
  }
  if (p == 0) {
    bucket_off[0] = 0;
    *n_patterns = npat;
  }
}

}  // namespace parse
