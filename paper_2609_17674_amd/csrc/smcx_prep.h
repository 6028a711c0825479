// The ordering pass: validates the particles, writes the outputs of those without
// a pass, and lists the others longest K first. Included by the sources whose
// launches share the pass with other work.
#pragma once
#include "smcx_internal.h"

namespace smcx {
namespace {

// ---------------------------------------------------------------- prep
// Ordering pass: validates every particle, settles the ones without work (K = 0
// outside the birth pass, invalid ones) and lists the rest longest-K first.
// One launch: each workgroup sorts a slice of at most kPrepSlice particles
// by itself (a counting sort in LDS), and the work list takes the slices'
// p-th particles in turn (rank p S + (b + p) mod S for slice b of S), which hands
// the long particles out first as one sorted list would: a slice of thousands
// holds about the same mix of K as the next. The turn by p keeps a slice from
// falling to the same dies (workgroups go round the eight) every time, whose work
// would differ as the slices' does: logL of 65536 sinusoid particles, K on 0..50,
// 65536 samples: 8.68 ms without it, 8.60 with. A slice with fewer than its share
// of particles to list leaves its last ranks empty (-1). (Two launches, a
// histogram per slice and then one global order, took 5.3 + 5.0 us at N =
// 16384.) Each thread loads all of its particles before it uses any, so the
// pass pays about one memory latency. Particles of equal K are listed in no
// particular order (results do not depend on it).
constexpr int kPrepBlock = 256;
constexpr int kPrepUnroll = 8;
constexpr int kPrepSlice = kPrepBlock * kPrepUnroll;

// Work-list key of particle i: K, or -1 when it needs no pass. With `settle`,
// also writes the outputs of invalid and K = 0 particles.
__device__ __forceinline__ int prep_key(const PrepArgs& a, int64_t i, int64_t o0, int64_t o1,
                                        int32_t dj, double beta_i, int bad_global, bool settle) {
  const int64_t K = o1 - o0;
  int bits = 0;
  if (bad_global) bits |= kFlagOffsets;
  if (K < 0 || o0 < 0 || o1 > a.M) bits |= kFlagOffsets;
  if (K > a.k_max) bits |= kFlagKMax;
  if (a.dlogl_death && a.death_idx && (dj < -1 || (int64_t)dj >= K)) bits |= kFlagDeath;
  if (bits) {
    if (settle) {
      const double nan = __builtin_nan("");
      if (!bad_global) atomicOr(a.flag, bits);
      if (a.logl) a.logl[i] = nan;
      if (a.dlogl_birth) a.dlogl_birth[i] = nan;
      if (a.dlogl_death) a.dlogl_death[i] = nan;
      if (a.grad && !bad_global && K > 0) {
        for (int64_t m = o0 < 0 ? 0 : o0; m < o1 && m < a.M; ++m)
          for (int p = 0; p < a.P; ++p) a.grad[m * a.P + p] = nan;
      }
    }
    return -1;
  }
  if (K == 0 && !a.include_k0) {
    if (settle && a.logl) a.logl[i] = a.k0_lo + beta_i * (a.k0_dev ? *a.k0_dev : a.k0_value);
    return -1;
  }
  return (int)K;
}

// Rank of the p-th listed particle of this workgroup's slice.
__device__ __forceinline__ int64_t prep_rank(int p, int64_t S) {
  return p * S + (blockIdx.x + (uint32_t)p) % (uint32_t)S;
}

// Particles per slice: S slices of (almost) equal size.
__host__ __device__ inline int64_t prep_slice_len(int64_t N, int64_t S) { return (N + S - 1) / S; }

// One slice (workgroup blockIdx.x < S) of the pass.
template <bool DEATH>
__device__ __forceinline__ void prep_block(const PrepArgs& a, int64_t S) {
  extern __shared__ int hist[];  // [k_max + 1] particles with K = k, then their next list position
  __shared__ int wsum[kPrepBlock / 64];
  __shared__ int bad_global;
  const int tid = threadIdx.x, lane = tid & 63;
  const int nk = a.k_max + 1;  // at most 4 * kPrepBlock
  const int64_t len = prep_slice_len(a.N, S), base = blockIdx.x * len;
  const int64_t end = base + len < a.N ? base + len : a.N;
  int64_t o0[kPrepUnroll], o1[kPrepUnroll];
  int32_t dj[kPrepUnroll];
  double bt[kPrepUnroll];
  // the loads are unconditional, on a clamped index, so that they are all in
  // flight together
#pragma unroll
  for (int u = 0; u < kPrepUnroll; ++u) {
    int64_t i = base + (int64_t)u * kPrepBlock + tid;
    i = i < a.N ? i : a.N - 1;
    o0[u] = a.offsets[i];
    o1[u] = a.offsets[i + 1];
    dj[u] = DEATH ? a.death_idx[i] : 0;
    bt[u] = 1.0;
  }
  // the K = 0 outputs are tempered: fetch beta with the rest
  if (a.tempered && a.beta && a.logl) {
#pragma unroll
    for (int u = 0; u < kPrepUnroll; ++u) {
      const int64_t i = base + (int64_t)u * kPrepBlock + tid;
      bt[u] = a.beta[i < a.N ? i : a.N - 1];
    }
  }
  for (int k = tid; k < nk; k += kPrepBlock) hist[k] = 0;
  if (tid == 0) {
    // offsets[0] != 0 or offsets[N] != M: every particle is then invalid
    const int bad = a.offsets[0] != 0 || a.offsets[a.N] != a.M ? 1 : 0;
    bad_global = bad;
    if (bad && blockIdx.x == 0) atomicOr(a.flag, a.offsets[0] != 0 ? kFlagOffsets : kFlagMMax);
  }
  __syncthreads();
  int key[kPrepUnroll];
#pragma unroll
  for (int u = 0; u < kPrepUnroll; ++u) {
    const int64_t i = base + (int64_t)u * kPrepBlock + tid;
    key[u] = i < end ? prep_key(a, i, o0[u], o1[u], dj[u], bt[u], bad_global, true) : -1;
    if (key[u] >= 0) atomicAdd(&hist[key[u]], 1);
  }
  __syncthreads();
  // exclusive prefix over K in descending order: 4 entries per thread, then a
  // scan over the threads
  int loc[4], sum = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = 4 * tid + q;  // j-th K in descending order
    loc[q] = j < nk ? hist[a.k_max - j] : 0;
    sum += loc[q];
  }
  int run = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(run, o);
    if (lane >= o) run += y;
  }
  if (lane == 63) wsum[tid >> 6] = run;
  __syncthreads();
  int total = 0;
  run -= sum;
#pragma unroll
  for (int w = 0; w < kPrepBlock / 64; ++w) {
    if (w < tid >> 6) run += wsum[w];
    total += wsum[w];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = 4 * tid + q;
    if (j < nk) hist[a.k_max - j] = run;
    run += loc[q];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPrepUnroll; ++u)
    if (key[u] >= 0)
      a.order[prep_rank(atomicAdd(&hist[key[u]], 1), S)] =
          (int32_t)(base + (int64_t)u * kPrepBlock + tid);
  for (int64_t p = total + tid; p < len; p += kPrepBlock) a.order[prep_rank((int)p, S)] = -1;
}

}  // namespace
}  // namespace smcx
