// SMC steps around the likelihood (Sec. "Sequential Monte Carlo",
// Sec. "Algorithm and implementation"): the ESS choice of the next
// inverse temperature with its weights and evidence increment, systematic
// resampling, the accept/reject of birth and death moves (eq. rj_acceptance),
// and the CSR rebuild the last two share.
//
// Population-wide sums of reals have a fixed order of additions (butterfly
// within a wave, then waves, then workgroups in order), so results do not
// depend on timing. Resampling works on integer weights so that its prefix
// sums, and therefore the ancestors, are exact however they are grouped.
#include "smcx_internal.h"

#include <math.h>

#include <algorithm>

namespace smcx {
namespace {

constexpr int kBlock = 1024;  // single-block kernels
constexpr int kBlockWaves = kBlock / 64;
constexpr double kWeightUnit = 1099511627776.0;  // 2^40: integer weight units

// Sum of a and b over the block, the same bits in every thread.
__device__ void block_sum2(double& a, double& b, double* sh) {
  for (int o = 32; o >= 1; o >>= 1) {  // butterfly: each step is commutative, so all lanes agree
    a += __shfl_xor(a, o);
    b += __shfl_xor(b, o);
  }
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    sh[w] = a;
    sh[kBlockWaves + w] = b;
  }
  __syncthreads();
  a = 0.0;
  b = 0.0;
  for (int i = 0; i < kBlockWaves; ++i) {
    a += sh[i];
    b += sh[kBlockWaves + i];
  }
}

// ---------------------------------------------------------------- prefix sums over tiles
// The rebuild passes cut the items into at most kScanTiles tiles of a whole
// number of workgroup widths, one workgroup per tile: it leaves prefix sums
// within its tile and the tile's sum, and the next launch's workgroups add the
// sums of the tiles before theirs. Integer sums are exact, so the grouping
// does not change them. (One workgroup over the whole population, with the
// loads of 16 waves to hide its latency: 40000 items took 39 and 50 us per
// prefix pass; these launches take 3 to 7.)
constexpr int kScanBlock = 256;
constexpr int kScanTiles = 1024;

__host__ __device__ inline int64_t scan_tile(int64_t N) {
  const int64_t per = (int64_t)kScanBlock * kScanTiles;
  return kScanBlock * ((N + per - 1) / per);
}

// Inclusive prefix sum of v over the workgroup's threads; sum receives the
// total. All threads call it; wsum is kScanBlock / 64 words of LDS.
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t& sum, int64_t* wsum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(v, o);
    if (lane >= o) v += y;
  }
  __syncthreads();  // the previous call's words have been read
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  sum = 0;
#pragma unroll
  for (int i = 0; i < kScanBlock / 64; ++i) {
    const int64_t x = wsum[i];
    v += i < w ? x : 0;
    sum += x;
  }
  return v;
}

__device__ double block_max(double a, double* sh) {
  for (int o = 32; o >= 1; o >>= 1) a = fmax(a, __shfl_xor(a, o));
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = a;
  __syncthreads();
  a = -INFINITY;
  for (int i = 0; i < kBlockWaves; ++i) a = fmax(a, sh[i]);
  return a;
}

// The search stops when the bracket is 1e-14 of the step or a few units in
// the last place of beta, whichever is wider (a step much smaller than
// beta_prev cannot be resolved to 1e-14 of itself).
constexpr double kBracketUlps = 8.0 * 2.220446049250313e-16;
// ... or when the lower end itself meets the condition to 1e-12 in log ESS
// (ESS >= alpha N still holds there).
constexpr double kRootTol = 1e-12;

struct NextBetaArgs {
  int64_t N;
  const double* logl;
  const double* logw_prev;
  double beta_prev, alpha;
  double* beta_out;
  double* logw;
  double* w_norm;
  double* scalars;
};

__device__ __forceinline__ double log_weight(const NextBetaArgs& a, int64_t i, double db) {
  return (a.logw_prev ? a.logw_prev[i] : 0.0) + db * a.logl[i];
}

// ESS of the weights at increment db (eq. ess), with the shift and sum.
__device__ double ess_at(const NextBetaArgs& a, double db, double* sh, double* m_out,
                         double* s1_out) {
  double m = -INFINITY;
  for (int64_t i = threadIdx.x; i < a.N; i += kBlock) m = fmax(m, log_weight(a, i, db));
  m = block_max(m, sh);
  double s1 = 0.0, s2 = 0.0;
  for (int64_t i = threadIdx.x; i < a.N; i += kBlock) {
    const double e = exp(log_weight(a, i, db) - m);
    s1 += e;
    s2 += e * e;
  }
  block_sum2(s1, s2, sh);
  if (m_out) *m_out = m;
  if (s1_out) *s1_out = s1;
  return s1 * s1 / s2;
}

// One block: the root of ESS = alpha N on [beta_prev, 1] (eq. ess_target),
// then the weights of eq. incremental_weight and the evidence increment.
__global__ __launch_bounds__(kBlock) void next_beta_kernel(NextBetaArgs a) {
  __shared__ double sh[2 * kBlockWaves];
  const double target = a.alpha * (double)a.N;
  double beta = 1.0;
  int evals = 0;
  const double e1 = ess_at(a, 1.0 - a.beta_prev, sh, nullptr, nullptr);
  if (!(e1 >= target)) {
    // The root of ESS(beta) = target in [beta_prev, 1], kept bracketed:
    // ESS(lo) >= target > ESS(hi). Each step tries the regula-falsi point of
    // f = log(ESS / target) (the Illinois variant halves the value kept at an
    // end that stays twice in a row), or the midpoint where that point is not
    // strictly inside; about ten evaluations reach the bracket width the
    // plain bisection reaches in fifty. The result is lo, a tested point, so
    // ESS(beta) >= target holds as for the bisection.
    double lo = a.beta_prev, hi = 1.0;
    const double f0 = a.logw_prev ? log(ess_at(a, 0.0, sh, nullptr, nullptr) / target)
                                  : log((double)a.N / target);
    double flo = f0, fhi = log(e1 / target);
    if (!(flo >= 0.0)) {
      // the previous weights alone are below the target: plain bisection
      // (it ends next to beta_prev)
      bool moved = false;
      for (int it = 0; it < 60; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi)) break;
        const double e = ess_at(a, mid - a.beta_prev, sh, nullptr, nullptr);
        ++evals;
        if (e >= target) {
          lo = mid;
          moved = true;
        } else {
          hi = mid;
        }
      }
      beta = moved ? lo : hi;
    } else {
      int side = 0;
      for (int it = 0; it < 100; ++it) {
        double x = fhi == fhi && flo - fhi > 0.0 ? hi - fhi * (hi - lo) / (fhi - flo) : 0.5 * (lo + hi);
        if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);
        if (!(x > lo && x < hi)) break;
        const double fx = log(ess_at(a, x - a.beta_prev, sh, nullptr, nullptr) / target);
        ++evals;
        if (fx >= 0.0) {
          lo = x;
          flo = fx;
          if (side == 1) fhi *= 0.5;
          side = 1;
        } else {
          hi = x;
          fhi = fx == fx ? fx : -INFINITY;
          if (side == -1) flo *= 0.5;
          side = -1;
        }
        if (hi - lo <= fmax(1e-14 * (hi - a.beta_prev), kBracketUlps * hi) ||
            (fx >= 0.0 && fx <= kRootTol))
          break;
      }
      beta = lo;
    }
  }
  const double db = beta - a.beta_prev;
  double m, s1;
  const double ess = ess_at(a, db, sh, &m, &s1);
  for (int64_t i = threadIdx.x; i < a.N; i += kBlock) {
    const double lw = log_weight(a, i, db);
    a.logw[i] = lw;
    a.w_norm[i] = exp(lw - m) / s1;
    if (a.beta_out) a.beta_out[i] = beta;
  }
  double lse_prev = log((double)a.N);
  if (a.logw_prev) {
    double mp = -INFINITY;
    for (int64_t i = threadIdx.x; i < a.N; i += kBlock) mp = fmax(mp, a.logw_prev[i]);
    mp = block_max(mp, sh);
    double sp = 0.0, unused = 0.0;
    for (int64_t i = threadIdx.x; i < a.N; i += kBlock) sp += exp(a.logw_prev[i] - mp);
    block_sum2(sp, unused, sh);
    lse_prev = mp + log(sp);
  }
  if (threadIdx.x == 0) {
    a.scalars[0] = beta;
    a.scalars[1] = ess;
    a.scalars[2] = m + log(s1) - lse_prev;
    a.scalars[3] = (double)evals;
  }
}

// ---------------------------------------------------------------- next beta, many workgroups
// The same search for uniform previous weights (no logw_prev), spread over
// the device: one launch per ESS evaluation. A launch's workgroups each sum
// exp(db l_i - m) and its square over their slice of particles (m = db
// max_i l_i, exact since db >= 0); the next launch's workgroups first add the
// range sums in slice order and take the search's next step from them, every
// workgroup computing the same bits (so they agree on the point to evaluate),
// and workgroup 0 records the step. A fixed number of evaluation launches is
// queued; the ones after the search has ended return at once, and a one-block
// pass finishes a search that would still be running. The evaluation at the
// bracket's lower end is kept, so the weights need no further pass.
constexpr int kNbBlock = 256;
constexpr int kNbPer = 4;                      // particles per thread per launch
constexpr int kNbSlice = kNbBlock * kNbPer;    // particles per workgroup
constexpr int kNbLaunches = 12;                // evaluation launches queued
constexpr int kNbState = 16;                   // doubles per search state

// search state (doubles): lo, hi, flo, fhi, x (point evaluated by the launch),
// side, evals, phase (0: evaluate beta = 1; 1: bracketing search; 2: done),
// beta, s1_lo, s2_lo (sums at beta), L (max l)
enum { kLo, kHi, kFlo, kFhi, kX, kSide, kEvals, kPhase, kBeta, kS1, kS2, kL };

struct NbMultiArgs {
  int64_t N;
  const double* logl;
  double beta_prev, alpha, target;
  double* beta_out;
  double* logw;
  double* w_norm;
  double* scalars;
  double* state;  // [2][kNbState]
  double* pmax;   // [G]
  double* psum;   // [2][G][2]
  int G;
};

// The search's step after an evaluation at st[kX] with sums (s1, s2); the
// same arithmetic as next_beta_kernel's bracketing search.
__device__ void nb_advance(const NbMultiArgs& a, double* st, double s1, double s2) {
  const double ess = s1 * s1 / s2;
  if (st[kPhase] == 0.0) {  // the evaluation at beta = 1
    if (ess >= a.target) {
      st[kPhase] = 2.0;
      st[kBeta] = 1.0;
      st[kS1] = s1;
      st[kS2] = s2;
      return;
    }
    st[kLo] = a.beta_prev;
    st[kHi] = 1.0;
    st[kFlo] = log((double)a.N / a.target);
    st[kFhi] = log(ess / a.target);
    st[kSide] = 0.0;
    st[kPhase] = 1.0;
    // sums at beta_prev: uniform weights
    st[kS1] = (double)a.N;
    st[kS2] = (double)a.N;
  } else {
    const double x = st[kX];
    const double fx = log(ess / a.target);
    st[kEvals] += 1.0;
    if (fx >= 0.0) {
      st[kLo] = x;
      st[kFlo] = fx;
      if (st[kSide] == 1.0) st[kFhi] *= 0.5;
      st[kSide] = 1.0;
      st[kS1] = s1;
      st[kS2] = s2;
    } else {
      st[kHi] = x;
      st[kFhi] = fx == fx ? fx : -INFINITY;
      if (st[kSide] == -1.0) st[kFlo] *= 0.5;
      st[kSide] = -1.0;
    }
    if (st[kHi] - st[kLo] <= fmax(1e-14 * (st[kHi] - a.beta_prev), kBracketUlps * st[kHi]) ||
        (fx >= 0.0 && fx <= kRootTol) || st[kEvals] >= 100.0) {
      st[kPhase] = 2.0;
      st[kBeta] = st[kLo];
      return;
    }
  }
  const double lo = st[kLo], hi = st[kHi], flo = st[kFlo], fhi = st[kFhi];
  double x = fhi == fhi && flo - fhi > 0.0 ? hi - fhi * (hi - lo) / (fhi - flo) : 0.5 * (lo + hi);
  if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);
  if (!(x > lo && x < hi)) {
    st[kPhase] = 2.0;
    st[kBeta] = lo;
    return;
  }
  st[kX] = x;
}

// The search state before launch k in st: launch k - 1's, advanced by its
// evaluation. All threads call it. The workgroups' sums come in by all threads
// and are added in workgroup order, s1 by thread 0 and s2 by thread 1: a
// thread that also loaded them took most of an evaluation launch (7.6 -> 5.0 us
// with 40 workgroups). ch is 2 NT words of LDS.
template <int NT>
__device__ void nb_state(const NbMultiArgs& a, int k, double* st, double* ch) {
  const int tid = threadIdx.x;
  if (k == 0) {
    double L = -INFINITY;
    for (int g = tid; g < a.G; g += NT) L = fmax(L, a.pmax[g]);
    for (int o = 32; o >= 1; o >>= 1) L = fmax(L, __shfl_xor(L, o));
    if ((tid & 63) == 0) ch[tid >> 6] = L;
    if (tid < kNbState) st[tid] = 0.0;
    __syncthreads();
    if (tid == 0) {
      for (int w = 1; w < NT / 64; ++w) L = fmax(L, ch[w]);
      st[kX] = 1.0;
      st[kL] = L;
    }
    __syncthreads();
    return;
  }
  const double* ps = a.psum + (size_t)((k - 1) & 1) * a.G * 2;
  const double* prev = a.state + ((k - 1) & 1) * kNbState;
  if (tid < kNbState) st[tid] = prev[tid];
  if (prev[kPhase] == 2.0) {
    __syncthreads();
    return;
  }
  double s = 0.0;
  for (int g0 = 0; g0 < a.G; g0 += NT) {
    const int n = a.G - g0 < NT ? a.G - g0 : NT;
    if (g0) __syncthreads();
    if (tid < n) {
      ch[tid] = ps[2 * (g0 + tid)];
      ch[NT + tid] = ps[2 * (g0 + tid) + 1];
    }
    __syncthreads();
    if (tid < 2) {
#pragma unroll 8
      for (int g = 0; g < n; ++g) s += ch[tid * NT + g];
    }
  }
  const double s2 = __shfl(s, 1);
  if (tid == 0) nb_advance(a, st, s, s2);
  __syncthreads();
}

__global__ __launch_bounds__(kNbBlock) void nb_max_kernel(NbMultiArgs a) {
  __shared__ double sh[kNbBlock / 64];
  const int64_t base = (int64_t)blockIdx.x * kNbSlice;
  double m = -INFINITY;
#pragma unroll
  for (int u = 0; u < kNbPer; ++u) {
    const int64_t i = base + u * kNbBlock + threadIdx.x;
    if (i < a.N) m = fmax(m, a.logl[i]);
  }
  for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = sh[0];
    for (int w = 1; w < kNbBlock / 64; ++w) r = fmax(r, sh[w]);
    a.pmax[blockIdx.x] = r;
  }
}

// Launch k: take the step after launch k - 1's evaluation (k > 0), then
// evaluate the new point.
__global__ __launch_bounds__(kNbBlock) void nb_eval_kernel(NbMultiArgs a, int k) {
  __shared__ double st[kNbState];
  __shared__ double sh[2 * kNbBlock];
  // the particles' values come in under the search's step
  const int64_t base = (int64_t)blockIdx.x * kNbSlice;
  double l[kNbPer];
#pragma unroll
  for (int u = 0; u < kNbPer; ++u) {
    const int64_t i = base + u * kNbBlock + threadIdx.x;
    l[u] = i < a.N ? a.logl[i] : 0.0;
  }
  nb_state<kNbBlock>(a, k, st, sh);
  if (blockIdx.x == 0 && threadIdx.x < kNbState)
    a.state[(k & 1) * kNbState + threadIdx.x] = st[threadIdx.x];
  if (st[kPhase] == 2.0) return;
  const double db = st[kX] - a.beta_prev;
  const double m = db * st[kL];
  double s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int u = 0; u < kNbPer; ++u) {
    const int64_t i = base + u * kNbBlock + threadIdx.x;
    if (i < a.N) {
      const double e = exp(db * l[u] - m);
      s1 += e;
      s2 += e * e;
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    s1 += __shfl_xor(s1, o);
    s2 += __shfl_xor(s2, o);
  }
  __syncthreads();  // sh has been read
  if ((threadIdx.x & 63) == 0) {
    sh[threadIdx.x >> 6] = s1;
    sh[kNbBlock / 64 + (threadIdx.x >> 6)] = s2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t1 = 0.0, t2 = 0.0;
    for (int w = 0; w < kNbBlock / 64; ++w) {
      t1 += sh[w];
      t2 += sh[kNbBlock / 64 + w];
    }
    double* ps = a.psum + (size_t)(k & 1) * a.G * 2;
    ps[2 * blockIdx.x] = t1;
    ps[2 * blockIdx.x + 1] = t2;
  }
}

// After the last queued evaluation: every workgroup takes the step from it
// and, should the search still be running, finishes it over the whole
// population (the same bits in each, so at most kNbFinish of them); then the
// weights at the chosen beta (eq. incremental_weight), normalised by the kept
// sums, and the scalars.
constexpr int kNbFinish = 256;

__global__ __launch_bounds__(kBlock) void nb_weights_kernel(NbMultiArgs a) {
  __shared__ double st[kNbState];
  __shared__ double sh[2 * kBlock];
  nb_state<kBlock>(a, kNbLaunches, st, sh);
  while (st[kPhase] != 2.0) {
    const double db = st[kX] - a.beta_prev;
    const double m = db * st[kL];
    double s1 = 0.0, s2 = 0.0;
    for (int64_t i = threadIdx.x; i < a.N; i += kBlock) {
      const double e = exp(db * a.logl[i] - m);
      s1 += e;
      s2 += e * e;
    }
    block_sum2(s1, s2, sh);  // the same bits in every thread
    __syncthreads();
    if (threadIdx.x == 0) nb_advance(a, st, s1, s2);
    __syncthreads();
  }
  const double beta = st[kBeta], db = beta - a.beta_prev;
  const double m = db * st[kL], s1 = st[kS1];
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < a.N;
       i += (int64_t)gridDim.x * kBlock) {
    const double lw = db * a.logl[i];
    a.logw[i] = lw;
    a.w_norm[i] = exp(lw - m) / s1;
    if (a.beta_out) a.beta_out[i] = beta;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.scalars[0] = beta;
    a.scalars[1] = s1 * s1 / st[kS2];
    a.scalars[2] = m + log(s1) - log((double)a.N);
    a.scalars[3] = st[kEvals];
  }
}

// ---------------------------------------------------------------- CSR rebuild
// Output particle j takes rows src_row[j] .. src_row[j] + src_len[j] - 1 of
// theta, without row skip[j] (local index, -1 = none), followed by row j of
// theta_add when append[j] != 0. Resampling neither skips nor appends (skip and
// append null), and the tiles' sums lie in an array that the call has no other
// use for, so that they add nothing to what a handle holds.
struct RebuildArgs {
  int64_t N, M;
  int P;
  int32_t k_max;
  const int64_t* offsets;  // source population
  const double* theta;
  int64_t* src_row;   // [N] workspace
  int32_t* src_len;   // [N]
  int32_t* skip;      // [N] or nullptr
  int32_t* append;    // [N] or nullptr
  int64_t* first;     // [N] first output row of particle j within its tile
  int32_t* rows;      // [tiles] output rows of each tile (of at most 2^20 particles)
  const double* theta_add;  // [N][P] rows appended (births)
  int64_t* offsets_out;     // [N + 1]
  double* theta_out;        // [m_cap][P]
  int64_t m_cap;
  int* flag;
};

// Rows of source particle i, validated against [0, M] and k_max (an invalid
// particle contributes no rows and raises the flag).
__device__ __forceinline__ bool source_rows(const RebuildArgs& a, int64_t i, int64_t& row,
                                            int32_t& len) {
  const int64_t o0 = a.offsets[i], o1 = a.offsets[i + 1];
  if (!(o0 >= 0 && o1 >= o0 && o1 <= a.M && o1 - o0 <= a.k_max)) {
    atomicOr(a.flag, (o1 - o0 > a.k_max && o0 >= 0 && o1 <= a.M) ? kFlagKMax : kFlagOffsets);
    row = 0;
    len = 0;
    return false;
  }
  row = o0;
  len = (int32_t)(o1 - o0);
  return true;
}

// Output particle j's first row within its tile (n rows; -1: no particle j),
// and after the tile's last pass its sum.
__device__ __forceinline__ void place_rows(const RebuildArgs& a, int64_t j, int32_t n,
                                           int64_t& carry, int64_t* wsum) {
  int64_t sum;
  const int64_t through = block_scan(n > 0 ? n : 0, sum, wsum);
  if (n >= 0) a.first[j] = carry + through - n;
  carry += sum;
}

// Copies the output particles' rows, 16 lanes per particle, and places them
// after the rows of the tiles before; rows at or past m_cap are not written
// (the capacity flag is raised). A chain of dependent loads bounds it, so 16
// particles share a workgroup and a lane has four loads in flight: 40000
// particles of 5.5 rows of 8 doubles: 13 -> 10 us (a wave per particle before;
// its 28 MB take 5.4 at the rate of a copy).
constexpr int kGatherLanes = 16;
constexpr int kGatherItems = kScanBlock / kGatherLanes;  // divides a tile

__global__ __launch_bounds__(kScanBlock) void csr_gather_kernel(RebuildArgs a) {
  __shared__ int64_t wsum[kScanBlock / 64];
  const int64_t j = (int64_t)blockIdx.x * kGatherItems + threadIdx.x / kGatherLanes;
  const int lane = threadIdx.x % kGatherLanes;
  const bool live = j < a.N;
  int64_t start = 0, row = 0;
  int32_t len = 0, skip = -1, add = 0;
  if (live) {
    start = a.first[j];
    row = a.src_row[j];
    len = a.src_len[j];
    if (a.skip) skip = a.skip[j];
    if (a.append) add = a.append[j];
  }
  // the rows are one run of values: the first batch comes in under the base
  const int P = a.P;
  const double* src = a.theta + row * P;
  const int n = len * P;
  double v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int x = lane + u * kGatherLanes;
    v[u] = x < n ? src[x] : 0.0;
  }
  const int tiles = (int)((int64_t)blockIdx.x * kGatherItems / scan_tile(a.N));
  int64_t before = 0;
#pragma unroll
  for (int u = 0; u < kScanTiles / kScanBlock; ++u) {
    const int g = u * kScanBlock + threadIdx.x;
    before += g < tiles ? a.rows[g] : 0;
  }
  int64_t base;
  block_scan(before, base, wsum);
  if (!live) return;
  start += base;
  const int64_t end = start + len - (skip >= 0 ? 1 : 0) + (add ? 1 : 0);
  if (lane == 0) {
    a.offsets_out[j] = start;
    if (j == a.N - 1) {
      a.offsets_out[a.N] = end;
      if (end > a.m_cap) atomicOr(a.flag, kFlagCapacity);
    }
  }
  // the values after the skipped row move up by P
  double* dst = a.theta_out + start * P;
  const int64_t room = (a.m_cap - start) * P;  // values that may be written from dst on
  const int s0 = skip >= 0 ? skip * P : n, s1 = s0 + P;
  for (int x0 = lane;;) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int x = x0 + u * kGatherLanes, y = x < s0 ? x : x - P;
      if (x < n && (x < s0 || x >= s1) && y < room) dst[y] = v[u];
    }
    x0 += 4 * kGatherLanes;
    if (x0 >= n) break;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int x = x0 + u * kGatherLanes;
      v[u] = x < n ? src[x] : 0.0;
    }
  }
  if (add && end <= a.m_cap)
    for (int p = lane; p < P; p += kGatherLanes) a.theta_out[(end - 1) * P + p] = a.theta_add[j * P + p];
}

// ---------------------------------------------------------------- resampling
struct ResampleArgs {
  RebuildArgs r;
  const double* w_norm;
  double u;
  int64_t* cum;       // [N] prefix sums, through i, of its tile's integer weights
  int32_t* ancestors; // [N]
};

// Integer weights c_i = round(w_i 2^40) (0 unless w_i > 0) and their inclusive
// prefix sums within a tile, exact in int64.
__device__ __forceinline__ int64_t weight_units(double w) {
  return w > 0.0 ? (int64_t)rint((w < 1.0 ? w : 1.0) * kWeightUnit) : 0;
}

__global__ __launch_bounds__(kScanBlock) void resample_prefix_kernel(ResampleArgs a) {
  __shared__ int64_t wsum[kScanBlock / 64];
  const int64_t N = a.r.N, tile = scan_tile(N), t0 = blockIdx.x * tile;
  int64_t carry = 0;
  for (int64_t i = t0 + threadIdx.x; i - threadIdx.x < t0 + tile; i += kScanBlock) {
    int64_t sum;
    const int64_t through = block_scan(i < N ? weight_units(a.w_norm[i]) : 0, sum, wsum);
    if (i < N) a.cum[i] = carry + through;
    carry += sum;
  }
}

// Offspring j: position U_j = floor(((j + u) C) / N), ancestor = first i whose
// prefix sum exceeds U_j, by bisection of the tile sums in LDS and of the
// tile (16-way steps, whose loads are in flight together, touch more lines and
// took 12 us, this 7); then its rows for the rebuild.
__global__ __launch_bounds__(kScanBlock) void resample_ancestor_kernel(ResampleArgs a) {
  __shared__ int64_t wsum[kScanBlock / 64];
  __shared__ int64_t through[kScanTiles];  // integer weight of the tiles through g
  const int64_t N = a.r.N, tile = scan_tile(N), t0 = blockIdx.x * tile;
  const int G = (int)((N + tile - 1) / tile);
  int64_t total = 0;
  for (int g0 = 0; g0 < G; g0 += kScanBlock) {
    const int g = g0 + threadIdx.x;
    int64_t sum;
    const int64_t end = (g + 1) * tile < N ? (g + 1) * tile : N;
    const int64_t x = block_scan(g < G ? a.cum[end - 1] : 0, sum, wsum);
    if (g < G) through[g] = total + x;
    total += sum;
  }
  __syncthreads();
  if (total <= 0 && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(a.r.flag, kFlagWeights);
  int64_t carry = 0;
  for (int64_t j = t0 + threadIdx.x; j - threadIdx.x < t0 + tile; j += kScanBlock) {
    int32_t len = -1;
    if (j < N) {
      int64_t anc = j;  // no positive weight: every particle keeps itself (flagged)
      if (total > 0) {
        int64_t U = (int64_t)floor(((double)j + a.u) * (double)total / (double)N);
        if (U >= total) U = total - 1;
        int g = 0;
        for (int hi = G - 1; g < hi;) {  // through[hi] > U
          const int mid = (g + hi) / 2;
          if (through[mid] > U) hi = mid;
          else g = mid + 1;
        }
        if (g) U -= through[g - 1];
        int64_t lo = g * tile, last = lo + tile < N ? lo + tile - 1 : N - 1;
        while (lo < last) {  // cum[last] > U
          const int64_t mid = lo + (last - lo) / 2;
          if (a.cum[mid] > U) last = mid;
          else lo = mid + 1;
        }
        anc = lo;
      }
      a.ancestors[j] = (int32_t)anc;
      int64_t row;
      source_rows(a.r, anc, row, len);
      a.r.src_row[j] = row;
      a.r.src_len[j] = len;
    }
    place_rows(a.r, j, len, carry, wsum);
  }
  if (threadIdx.x == 0) a.r.rows[blockIdx.x] = (int32_t)carry;
}

// ---------------------------------------------------------------- birth/death
struct RjArgs {
  RebuildArgs r;
  const int8_t* move;
  const int32_t* death_idx;
  const double* dlogl_birth;
  const double* dlogl_death;
  const double* log_u;
  int32_t k_lo, k_hi;
  double log_pd_over_pb;
  int8_t* accepted;
};

// Accept/reject per particle: log alpha = dlogl_birth + log(p_death/p_birth)
// for a birth with K + 1 <= k_hi, dlogl_death - log(p_death/p_birth) for a
// death of a valid index with K - 1 >= k_lo (the reading of eq. rj_acceptance
// for exchangeable components, a birth proposal equal to the prior and a
// uniform prior on K); accepted when log_u < log alpha.
__global__ __launch_bounds__(kScanBlock) void rj_decide_kernel(RjArgs a) {
  __shared__ int64_t wsum[kScanBlock / 64];
  const int64_t N = a.r.N, tile = scan_tile(N), t0 = blockIdx.x * tile;
  int64_t carry = 0;
  for (int64_t i = t0 + threadIdx.x; i - threadIdx.x < t0 + tile; i += kScanBlock) {
    int32_t n = -1;
    if (i < N) {
      int64_t row;
      int32_t K;
      const bool ok = source_rows(a.r, i, row, K);
      const int mv = a.move[i];
      bool acc = false;
      int32_t skip = -1;
      if (ok && mv == 1 && a.r.theta_add && a.dlogl_birth && K + 1 <= a.k_hi) {
        acc = a.log_u[i] < a.dlogl_birth[i] + a.log_pd_over_pb;
      } else if (ok && mv == 2 && a.death_idx && a.dlogl_death && K - 1 >= a.k_lo) {
        const int32_t j = a.death_idx[i];
        if (j >= 0 && j < K) {
          acc = a.log_u[i] < a.dlogl_death[i] - a.log_pd_over_pb;
          if (acc) skip = j;
        }
      }
      a.accepted[i] = acc ? 1 : 0;
      a.r.src_row[i] = row;
      a.r.src_len[i] = K;
      a.r.skip[i] = skip;
      a.r.append[i] = (acc && mv == 1) ? 1 : 0;
      n = K + (acc ? (mv == 1 ? 1 : -1) : 0);
    }
    place_rows(a.r, i, n, carry, wsum);
  }
  if (threadIdx.x == 0) a.r.rows[blockIdx.x] = (int32_t)carry;
}

hipError_t launch_gather(const RebuildArgs& r, hipStream_t st) {
  hipLaunchKernelGGL(csr_gather_kernel, dim3((unsigned)((r.N + kGatherItems - 1) / kGatherItems)),
                     dim3(kScanBlock), 0, st, r);
  return hipGetLastError();
}

unsigned scan_tiles(int64_t N) { return (unsigned)((N + scan_tile(N) - 1) / scan_tile(N)); }

}  // namespace

hipError_t launch_next_beta(int64_t N, const double* logl, const double* logw_prev,
                            double beta_prev, double alpha, double* beta_out, double* logw,
                            double* w_norm, double* scalars, double* work, size_t work_cap,
                            hipStream_t st) {
  const int64_t G = (N + kNbSlice - 1) / kNbSlice;
  if (logw_prev || !work || work_cap < (size_t)(2 * kNbState + 5 * G)) {
    NextBetaArgs a{N, logl, logw_prev, beta_prev, alpha, beta_out, logw, w_norm, scalars};
    hipLaunchKernelGGL(next_beta_kernel, dim3(1), dim3(kBlock), 0, st, a);
    return hipGetLastError();
  }
  NbMultiArgs a;
  a.N = N;
  a.logl = logl;
  a.beta_prev = beta_prev;
  a.alpha = alpha;
  a.target = alpha * (double)N;
  a.beta_out = beta_out;
  a.logw = logw;
  a.w_norm = w_norm;
  a.scalars = scalars;
  a.state = work;
  a.pmax = work + 2 * kNbState;
  a.psum = a.pmax + G;
  a.G = (int)G;
  const dim3 grid((unsigned)G), block(kNbBlock);
  hipLaunchKernelGGL(nb_max_kernel, grid, block, 0, st, a);
  for (int k = 0; k < kNbLaunches; ++k) hipLaunchKernelGGL(nb_eval_kernel, grid, block, 0, st, a, k);
  const int64_t gw = std::min<int64_t>((N + kBlock - 1) / kBlock, kNbFinish);
  hipLaunchKernelGGL(nb_weights_kernel, dim3((unsigned)gw), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_resample(const SmcWork& w, int model, int32_t k_max, int64_t N,
                           const int64_t* offsets, int64_t M, const double* theta,
                           const double* w_norm, double u, int64_t m_cap, int32_t* ancestors,
                           int64_t* offsets_out, double* theta_out, int* flag, hipStream_t st) {
  ResampleArgs a;
  a.r = RebuildArgs{N, M, n_params(model), k_max, offsets, theta, w.src_row, w.src_len, nullptr,
                    nullptr, w.count, w.skip, nullptr, offsets_out, theta_out, m_cap, flag};
  a.w_norm = w_norm;
  a.u = u;
  a.cum = w.cum;
  a.ancestors = ancestors;
  hipLaunchKernelGGL(resample_prefix_kernel, dim3(scan_tiles(N)), dim3(kScanBlock), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(resample_ancestor_kernel, dim3(scan_tiles(N)), dim3(kScanBlock), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_gather(a.r, st);
}

hipError_t launch_rj_apply(const SmcWork& w, int model, int32_t k_max, int64_t N,
                           const int64_t* offsets, int64_t M, const double* theta,
                           const int8_t* move, const double* theta_birth, const int32_t* death_idx,
                           const double* dlogl_birth, const double* dlogl_death,
                           const double* log_u, int32_t k_lo, int32_t k_hi, double log_pd_over_pb,
                           int64_t m_cap, int64_t* offsets_out, double* theta_out,
                           int8_t* accepted, int* flag, hipStream_t st) {
  RjArgs a;
  a.r = RebuildArgs{N, M, n_params(model), k_max, offsets, theta, w.src_row, w.src_len, w.skip,
                    w.append, w.count, (int32_t*)w.cum, theta_birth, offsets_out, theta_out, m_cap, flag};
  a.move = move;
  a.death_idx = death_idx;
  a.dlogl_birth = dlogl_birth;
  a.dlogl_death = dlogl_death;
  a.log_u = log_u;
  a.k_lo = k_lo;
  a.k_hi = k_hi;
  a.log_pd_over_pb = log_pd_over_pb;
  a.accepted = accepted;
  hipLaunchKernelGGL(rj_decide_kernel, dim3(scan_tiles(N)), dim3(kScanBlock), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_gather(a.r, st);
}

}  // namespace smcx
