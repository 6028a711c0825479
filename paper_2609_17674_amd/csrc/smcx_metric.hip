// Gauss-Newton (Fisher) metric of every particle on the matrix cores.
//
// F_i = (beta_i / sigma^2) sum_s J_s J_s^T with J_s the template partials
// dh_k(t_s)/dtheta_{k,p} of particle i (coordinate k P + p): the Hessian of the
// tempered negative log-likelihood without its residual term, the mass matrix
// the NUTS section of the paper asks for (the Hessian of the negative log
// posterior; a uniform prior adds nothing inside its box).
//
// A wave owns up to 32 components, those of one particle or of several small
// ones (pack_groups packs them), and walks the samples in steps of 8.
// Lane l stands for component row l % 32 and per step forms the P partials of
// its component at four samples, in natural units (J~ = J * s with s =
// (1, w, w) for pulses and (1, 1/T_obs, 1/T_obs^2, 1) for sinusoids, so every
// entry is of order one), so that the exponential or the phase of a component
// is taken once per sample and not once per parameter. The values are rounded
// to FP16 and feed both operands of v_mfma_f32_32x32x8_f16, one product per
// pair of parameters (6 for pulses, 10 for sinusoids): with A[i][k] held by
// lane i + 32 (k/4), element k%4, and B[k][j] by lane j + 32 (k/4), a lane's
// own values of parameter p are its row of A and those of p' its column of
// B, and D_pp' = J~_p^T J~_p' over the wave's rows; the entries between rows
// of different particles are dropped. The FP32 accumulators
// are flushed into the FP64 output after each window of 4096 samples, each
// entry owned by one lane and the windows in order (read-add-write, no
// atomics), so the result is deterministic; entries
// below the diagonal are written as copies of those above it.
// Few particles, and k_max P > 64, take the coordinate form instead: one wave
// per particle, lanes over its coordinates k P + p in NB blocks of 32,
// NB (NB + 1) / 2 products per step; see launch_metric for where the line lies.
// What bounds the grouped form: per step about 195 cycles of vector work (8 of
// the 39 instructions are the conversions, 9 cycles each) beside 6 x 32 of the
// matrix cores, overlapped to about 300 at three waves per SIMD. Measured on
// 16384 pulse particles, K uniform on 0..20, T = 4096, dense blocks: 0.41 ms
// a call against 1.30 ms for the coordinate form; sinusoids, 8192 particles,
// K on 0..16, T = 4096: 0.45 against 1.02 ms.
// Error: FP16 rounding of J~ (2^-11 relative) bounds |dF~_ac| by about
// 2^-10 sqrt(F~_aa F~_cc), plus FP32 accumulation over 512 steps.
#include "smcx_internal.h"

#include <algorithm>

#include <math.h>

namespace smcx {
namespace {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr double kTwoPiM = 6.283185307179586476925286766559;
constexpr double kPiM = 3.141592653589793238462643383279;
constexpr double kHalfLog2eRoot = 0.84932180028801904272150283410289;  // sqrt(log2(e) / 2)
constexpr int kFlushSamples = 4096;

// Orders the LDS accesses of one wave around it.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct MetricArgs {
  int P;
  int64_t N, M, T;
  double t_start, dt, inv_sigma2, t_obs;
  int32_t k_max;
  const int64_t* offsets;
  const double* theta;
  const double* beta;
  const int64_t* f_offsets;
  int64_t f_size;  // entries of F: every block must fit
  double* F;
  int* flag;
  int64_t w0, w1;  // coordinate form: the sample window of this launch; the first window
                   // writes F, later ones add
  int tempered;    // coordinate form: 1: the window's samples carry beta_i (0: before a
                   // bridge split)
  int blocks;      // 1: only each component's P x P block, at F + m P P (source row m)
  const uint8_t* mask;  // [N] or nullptr: particles with mask[i] == 0 get zero blocks
  int64_t split;   // samples before it carry weight 1, later ones beta_i
  int nblk;        // grouped form: blocks of kGroupBlock particles,
  int slots;       // and waves (or, with several windows, sets of waves) of each
};

// Whether particle i's rows, and its output block, are as they should be; its
// components in K, its block's start in fo. Raises the flag if not.
__device__ __forceinline__ bool metric_particle(const MetricArgs& a, int64_t i, int64_t& o0, int& K,
                                                int64_t& fo, bool raise) {
  o0 = a.offsets[i];
  const int64_t o1 = a.offsets[i + 1];
  bool ok = o0 >= 0 && o1 >= o0 && o1 <= a.M && o1 - o0 <= a.k_max;
  K = ok ? (int)(o1 - o0) : 0;
  const int64_t n = (int64_t)K * a.P;
  fo = a.blocks ? o0 * a.P * a.P : a.f_offsets[i];
  if (ok && !a.blocks)
    ok = a.f_offsets[i + 1] - fo == n * n && fo >= 0 && fo + n * n <= a.f_size;
  if (!ok && raise) atomicOr(a.flag, kFlagOffsets);
  return ok;
}

// ---------------------------------------------------------------- groups
// Packs the particles of a block of kGroupBlock into groups of at most 32
// components, first-fit decreasing: a counting sort by K, then the wave opens
// a group and keeps adding the largest particle that still fits. A group is
// a range of perm (particles of the block). The placing is a serial chain per
// particle, which a wave takes with its scans in registers. Every wave packs its
// block for itself, into LDS: the groups in memory, from a pass of its own, would
// be workspace that the handle's calls on other streams share. It costs no
// more than that pass did (16384 particles, K on 0..20, dense blocks: T = 4096
// 468 us in two launches, 455 in one; T = 1000 172, 175; T = 8 80, 88). For K
// uniform on 0..20 the rows are 93% filled (96% in blocks of 128, 79% when
// neighbours are taken as they come). Particles without components, and with a
// mask those not selected, are in no group.
constexpr int kGroupBlock = 64;

struct GroupPack {
  int64_t row[kGroupBlock];  // per particle of the block: its first row,
  int64_t fo[kGroupBlock];   // its output block in F
  int K[kGroupBlock];        // and its components
  int perm[kGroupBlock];
  int start[kGroupBlock + 1];  // group g is perm[start[g]] .. perm[start[g + 1] - 1]
  int groups;
  unsigned long long zero;   // particles that get zero blocks
  int sorted[kGroupBlock];
};

// By one wave, for the particles from i0 on; every wave that packs a block comes
// to the same groups (equal K in particle order). raise: flag invalid particles.
__device__ __forceinline__ void pack_groups(const MetricArgs& a, int64_t i0, int lane, bool raise,
                                            GroupPack& pk) {
  const int64_t i = i0 + lane;
  int K = 0;
  bool zero = false;
  if (i < a.N) {
    int64_t o0, fo;
    if (!metric_particle(a, i, o0, K, fo, raise)) K = 0;
    zero = K > 0 && a.mask && !a.mask[i];
    pk.row[lane] = o0;
    pk.fo[lane] = fo;
    pk.K[lane] = K;
    if (zero) K = 0;
  }
  int rank = 0, left = 0;  // lane k: particles with K = k still to place
  for (int k = 1; k <= a.k_max; ++k) {
    const unsigned long long same = __builtin_amdgcn_ballot_w64(K == k);
    if (K == k) rank = __popcll(same & ((1ull << lane) - 1ull));
    if (lane == k) left = __popcll(same);
  }
  int pos = left;
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(pos, o);
    if (lane >= o) pos += y;
  }
  pos -= left;  // lane k: the first place of K = k in sorted order
  const int at = __shfl(pos, K) + rank;
  if (K > 0) pk.sorted[at] = lane;
  wave_lds_order();
  int mine = 0, o = 0, g = 0;  // lane o keeps the o-th particle of the groups
  unsigned long long any = __builtin_amdgcn_ballot_w64(left > 0);
  while (any) {
    if (lane == 0) pk.start[g] = o;
    int rem = 32;
    for (;;) {
      const unsigned long long fit = any & ((2ull << rem) - 1ull);
      if (!fit) break;
      const int k = 63 - __builtin_clzll(fit);
      const int p = __builtin_amdgcn_readlane(pos, k);
      mine = lane == o ? p : mine;
      ++o;
      rem -= k;
      left -= lane == k ? 1 : 0;
      pos += lane == k ? 1 : 0;
      any = __builtin_amdgcn_ballot_w64(left > 0);
    }
    ++g;
  }
  if (lane < o) pk.perm[lane] = pk.sorted[mine];
  if (lane == 0) {
    pk.start[g] = o;
    pk.groups = g;
  }
  const unsigned long long z = __builtin_amdgcn_ballot_w64(zero);
  if (lane == 0) pk.zero = z;
  wave_lds_order();
}

// ---------------------------------------------------------------- grouped form
// Per-lane description of one component. Rows past the group's components
// have zero coefficients.
template <int MODEL>
struct Comp;

// pulse: x = s - nf (exact), z = x a - fa, e = 2^(-z^2),
// J~ = (e, e (c1 z), e (c2 z^2)): c1 = A k, c2 = A k^2 with
// k = 1 / sqrt(log2(e)/2), so that k z = (t - t0)/w. A width so small that z
// is not finite on some sample has fa = NaN, an empty row a = 0 and fa so
// large that e is zero.
template <>
struct Comp<SMCX_PULSE> {
  float nf = 0.f, a = 0.f, fa = 1e6f, c1 = 0.f, c2 = 0.f;
};

// sinusoid: phase in cycles ph0 + ph1 s + ph2 s^2 (FP64), tr = t / T_obs =
// tr0 + s dtr, J~ = (c0 sin, cos (k1 tr), cos (k2 tr^2), cos k3) with k1 =
// 2 pi A', k2 = pi A', k3 = A'
template <>
struct Comp<SMCX_GBSINE> {
  double ph0 = 0.0, ph1 = 0.0, ph2 = 0.0;
  float c0 = 0.f, k1 = 0.f, k2 = 0.f, k3 = 0.f;
};

__device__ __forceinline__ void make_comp(const MetricArgs& a, const double* r, Comp<SMCX_PULSE>& q,
                                          double* scale) {
  const double A = r[0], t0 = r[1], w = r[2];
  const double cc = (t0 - a.t_start) / a.dt;
  double nn = floor(cc);
  nn = fmin(fmax(nn, -4194304.0), 4194304.0);
  const double al = kHalfLog2eRoot * a.dt / w;
  const double k = 1.0 / kHalfLog2eRoot;
  q.nf = (float)nn;
  q.a = (float)al;
  q.fa = (float)((cc - nn) * al);
  const float x_max = fmaxf(fabsf(q.nf), fabsf((float)(a.T - 1) - q.nf));
  if (!(fabsf(x_max * q.a) < INFINITY && fabsf(q.fa) < INFINITY)) q.fa = __builtin_nanf("");
  q.c1 = (float)(A * k);
  q.c2 = (float)(A * k * k);
  scale[0] = 1.0;
  scale[1] = scale[2] = w;
}
__device__ __forceinline__ void make_comp(const MetricArgs& a, const double* r, Comp<SMCX_GBSINE>& q,
                                          double* scale) {
  const double A = r[0], f0 = r[1], fd = r[2], phi0 = r[3];
  const double ts = a.t_start, dt = a.dt;
  q.ph0 = f0 * ts + 0.5 * fd * ts * ts + phi0 / kTwoPiM;
  q.ph1 = (f0 + fd * ts) * dt;
  q.ph2 = 0.5 * fd * dt * dt;
  q.c0 = 1.f;
  q.k1 = (float)(kTwoPiM * A);
  q.k2 = (float)(kPiM * A);
  q.k3 = (float)A;
  scale[0] = scale[3] = 1.0;
  scale[1] = 1.0 / a.t_obs;
  scale[2] = 1.0 / (a.t_obs * a.t_obs);
}

// The partials of one component at sample s (sf = s - nf for pulses).
__device__ __forceinline__ void jvalues(const Comp<SMCX_PULSE>& q, float x, int, float, float,
                                        float (&j)[3]) {
  const float z = __builtin_fmaf(x, q.a, -q.fa);
  const float e = __builtin_amdgcn_exp2f(-(z * z));
  j[0] = e;
  j[1] = e * (q.c1 * z);
  j[2] = e * (q.c2 * z * z);
}
__device__ __forceinline__ void jvalues(const Comp<SMCX_GBSINE>& q, float, int s, float tr0,
                                        float dtr, float (&j)[4]) {
  const double sd = (double)s;
  const double ph = fma(fma(q.ph2, sd, q.ph1), sd, q.ph0);
  const float rev = (float)(ph - rint(ph));  // revolutions in [-0.5, 0.5]
  const float tr = __builtin_fmaf((float)s, dtr, tr0);
  const float c = __builtin_amdgcn_sinf(rev + 0.25f);  // the cosine, a quarter cycle on
  j[0] = __builtin_amdgcn_sinf(rev) * q.c0;
  j[1] = c * (q.k1 * tr);
  j[2] = c * (q.k2 * tr * tr);
  j[3] = c * q.k3;
}
__device__ __forceinline__ float centre(const Comp<SMCX_PULSE>& q) { return q.nf; }
__device__ __forceinline__ float centre(const Comp<SMCX_GBSINE>&) { return 0.f; }

// The partials at this half's four samples of a step from s0 on (x = s0 minus
// the pulse's centre index, exact), in FP16. TAIL: samples from w1 on are
// left out.
template <int MODEL, int P, bool TAIL>
__device__ __forceinline__ void step_partials(const Comp<MODEL>& q, float x, int s0, int w1, float tr0,
                                              float dtr, half4 (&h)[P]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float j[P];
    jvalues(q, x + (float)e, s0 + e, tr0, dtr, j);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      // a value that ends in a product is converted with it (one rounding);
      // the empty asm on the first of two keeps the compiler from converting
      // such values in pairs, with the products rounded to FP32 first
      _Float16 v = (_Float16)(!TAIL || s0 + e < w1 ? j[p] : 0.f);
      if ((MODEL != SMCX_PULSE || p > 0) && (TAIL || e % 2 == 0)) asm volatile("" : "+v"(v));
      h[p][e] = v;
    }
  }
}

template <int P>
__device__ __forceinline__ void step_products(const half4 (&h)[P], float16v (&acc)[P * (P + 1) / 2]) {
  int y = 0;
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int r = p; r < P; ++r, ++y)
      acc[y] = __builtin_amdgcn_mfma_f32_32x32x8f16(h[p], h[r], acc[y], 0, 0, 0);
}

// The products of one wave's group for one window, in LDS for the flush.
template <int P>
struct FlushTile {
  float d[P * (P + 1) / 2][32 * 33];  // D_pp', rows of p by rows of p'
};
// What the flush needs to know of a wave's group.
template <int P>
struct FlushGroup {
  double scale[32 * P];  // inverse natural scales of the rows
  double beta[32];       // per particle of the group
  int64_t fo[32];        // its block in F
  int r0[32], K[32];     // its rows
  int parts;             // particles
};

// One window's products into F, by the whole workgroup: rows of the output
// over the waves and its columns over the lanes, so that every store covers
// a stretch of an output row (written straight from the accumulators the
// columns lie P entries apart and the mirrored half n entries, 110 us for
// the 157 MB of a pulse population instead of 60). Of a symmetric product only
// the upper triangle is read, so that the result is exactly symmetric.
template <int P>
__device__ __forceinline__ void flush_group(const MetricArgs& a, const FlushTile<P>& t,
                                            const FlushGroup<P>& g, bool tempered, bool first) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int l = 0; l < g.parts; ++l) {
    const int K = g.K[l], r0 = g.r0[l];
    const double bs = (tempered ? g.beta[l] : 1.0) * a.inv_sigma2;
    double* Fi = a.F + g.fo[l];
    // entry (row r, p) x (row c, pc), p <= pc after ordering
    auto entry = [&](int r, int p, int c, int pc) {
      const bool up = p < pc || (p == pc && r <= c);
      const int u = up ? r : c, pu = up ? p : pc, v = up ? c : r, pv = up ? pc : p;
      const int y = pu * P - pu * (pu - 1) / 2 + (pv - pu);
      // scaled in the order of the coordinate form
      const int a0 = u * P + pu, a1 = v * P + pv, lo = a0 < a1 ? a0 : a1, hi = a0 < a1 ? a1 : a0;
      return (double)t.d[y][u * 33 + v] * (bs * g.scale[hi]) * g.scale[lo];
    };
    if (a.blocks) {
      for (int e = threadIdx.x; e < K * P * P; e += 256) {
        const int k = e / (P * P), p = e / P % P, pc = e % P;
        const double v = entry(r0 + k, p, r0 + k, pc);
        Fi[e] = first ? v : Fi[e] + v;
      }
      continue;
    }
    const int n = K * P;
    if (lane >= n) continue;  // n <= 64
    const int c = r0 + lane / P, pc = lane % P;
    if (first) {
#pragma unroll 4
      for (int x = wid; x < n; x += 4)
        Fi[(int64_t)x * n + lane] = entry(r0 + x / P, x % P, c, pc);
    } else {
      for (int x = wid; x < n; x += 4)
        Fi[(int64_t)x * n + lane] += entry(r0 + x / P, x % P, c, pc);
    }
  }
}

// Waves of a workgroup that share a group, one window each in turn: with
// several windows of samples a group's windows run side by side and are
// flushed in order.
// The step loop takes the partials of the next step while the products of
// the current one are in the matrix cores, two steps to a turn, which saves the
// copies from one to the next (39 vector instructions a step instead of 46).
// A wave takes group `slot` of block `blk`, and with more groups than slots every
// `slots`-th from there. The waves of a workgroup go to neighbouring blocks, so
// that it is full wherever the blocks have about as many groups.
template <int MODEL, int WPG>
__global__ __launch_bounds__(256, (MODEL == SMCX_PULSE ? 3 : 2)) void metric_group_kernel(MetricArgs a) {
  constexpr int P = n_params(MODEL);
  constexpr int NP = P * (P + 1) / 2;
  __shared__ FlushTile<P> tile;
  __shared__ FlushGroup<P> groups[4];
  __shared__ GroupPack packs[4];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  FlushGroup<P>& gr = groups[wid];
  GroupPack& pk = packs[wid];
  const int half = lane >> 5;  // which group of 4 samples of a step this lane feeds
  const int row = lane & 31;
  // the first groups of all blocks come first
  const unsigned item = (blockIdx.x * 4u + (unsigned)wid) / WPG;
  int slot = (int)(item / (unsigned)a.nblk);
  const int64_t i0 = (int64_t)(item - (unsigned)slot * (unsigned)a.nblk) * kGroupBlock;
  int ngroups = 0;
  if (slot < a.slots) {
    pack_groups(a, i0, lane, slot == 0, pk);
    ngroups = __builtin_amdgcn_readfirstlane(pk.groups);
    // not selected: zero blocks (the factor's ridge makes them definite)
    int t = 0;
    for (unsigned long long z = pk.zero; z; z &= z - 1, ++t) {
      if (t % a.slots != slot || wid % WPG) continue;
      const int l = __builtin_ctzll(z);
      const int64_t n = (int64_t)pk.K[l] * P, cnt = a.blocks ? n * P : n * n;
      for (int64_t e = lane; e < cnt; e += 64) a.F[pk.fo[l] + e] = 0.0;
    }
  }
  for (;; slot += a.slots) {
    const bool have = slot < ngroups;
    if (!__syncthreads_or(have)) return;
    const int g = slot;
    const int first = have ? pk.start[g] : 0, parts = have ? pk.start[g + 1] - first : 0;
    // lane l < parts holds the group's l-th particle
    int Kl = 0, end = 0;
    int64_t ol = 0;
    if (lane < parts) {
      const int l = pk.perm[first + lane];
      ol = pk.row[l];
      Kl = pk.K[l];
      gr.beta[lane] = a.beta ? a.beta[i0 + l] : 1.0;
      gr.fo[lane] = pk.fo[l];
      gr.K[lane] = Kl;
    }
    if (lane == 0) gr.parts = parts;
    end = Kl;
    for (int o = 1; o < 32; o <<= 1) {
      const int y = __shfl_up(end, o);
      if (lane >= o) end += y;
    }
    if (lane < parts) gr.r0[lane] = end - Kl;
    // this lane's component: row `row` of the group
    Comp<MODEL> q;
    int64_t src = -1;  // its row of theta
    for (int l = 0; l < parts; ++l) {
      const int e = __builtin_amdgcn_readlane(end, l), k = __builtin_amdgcn_readlane(Kl, l);
      const int64_t o = ((int64_t)__builtin_amdgcn_readlane((int)(ol >> 32), l) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)ol, l);
      if (row >= e - k && row < e) src = o + row - (e - k);
    }
    if (src >= 0) {
      double natural[P];
      make_comp(a, a.theta + src * P, q, natural);
      if (half == 0)
        for (int p = 0; p < P; ++p) gr.scale[row * P + p] = 1.0 / natural[p];
    }
    const float tr0 = (float)(a.t_start / a.t_obs), dtr = (float)(a.dt / a.t_obs);
    const float nf = centre(q);
    // windows of at most 4096 samples, none across the split
    const int nlo = (int)((a.split + kFlushSamples - 1) / kFlushSamples);
    const int nwin = nlo + (int)((a.T - a.split + kFlushSamples - 1) / kFlushSamples);
    for (int w = 0; w < nwin; w += WPG) {
      const int win = w + wid % WPG;
      float16v acc[NP];
#pragma unroll
      for (int y = 0; y < NP; ++y) acc[y] = float16v{};
      if (have && win < nwin) {
        const bool lo = win < nlo;
        // sample indices fit in 32 bits (T <= 2^22)
        const int w0 = lo ? win * kFlushSamples : (int)a.split + (win - nlo) * kFlushSamples;
        const int last = lo ? (int)a.split : (int)a.T;
        const int w1 = w0 + kFlushSamples < last ? w0 + kFlushSamples : last;
        const int full = w0 + (w1 - w0) / 8 * 8;
        float x = (float)(w0 + 4 * half) - nf;  // exact: integers below 2^24
        half4 h[P];
        if (full > w0) {
          step_partials<MODEL, P, false>(q, x, w0 + 4 * half, w1, tr0, dtr, h);
          int s = w0 + 8;
          // the products of one step, the partials of the next
          const auto step = [&](const half4(&hc)[P], half4(&hn)[P]) {
            x += 8.f;
            step_partials<MODEL, P, false>(q, x, s + 4 * half, w1, tr0, dtr, hn);
            step_products<P>(hc, acc);
#pragma unroll
            for (int y = 0; y < NP; ++y) {
              // one product, then a share of the next step's vector work
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x402, MODEL == SMCX_PULSE ? 7 : 9, 0);
            }
            s += 8;
          };
          half4 hn[P];
#pragma unroll 1
          while (s + 8 < full) {  // two steps: no copies from one to the next
            step(h, hn);
            step(hn, h);
          }
          if (s < full) {
            step(h, hn);
#pragma unroll
            for (int p = 0; p < P; ++p) h[p] = hn[p];
          }
          step_products<P>(h, acc);
          x += 8.f;
        }
        if (full < w1) {
          step_partials<MODEL, P, true>(q, x, full + 4 * half, w1, tr0, dtr, h);
          step_products<P>(h, acc);
        }
      }
      // flush, one wave's products after the other: lane holds D[i][j] of rows
      // j = lane % 32 and i = 8 (r/4) + 4 half + r % 4
      for (int turn = 0; turn < 4; ++turn) {
        __syncthreads();
        if (wid == turn)
#pragma unroll
          for (int y = 0; y < NP; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              tile.d[y][(8 * (r >> 2) + 4 * half + (r & 3)) * 33 + row] = acc[y][r];
        __syncthreads();
        const int wt = w + turn % WPG;  // that wave's window
        if (wt < nwin) flush_group<P>(a, tile, groups[turn], wt >= nlo, wt == 0);
      }
    }
  }
}

// ---------------------------------------------------------------- coordinate form
// Per-lane description of one coordinate (component k, parameter p), set up
// so that J~ needs no branch on p; padding lanes get zero coefficients.
template <int MODEL>
struct Coord;

// pulse: x = s - nf (exact), z = x a - fa, J~ = e (c0 + c1 z + c2 z^2) with
// e = 2^(-z^2): (c0, c1, c2) = (1, 0, 0), (0, A k, 0), (0, 0, A k^2) for
// p = 0, 1, 2, k = 1 / sqrt(log2(e)/2) so that k z = (t - t0)/w
template <>
struct Coord<SMCX_PULSE> {
  float nf, a, fa, c0, c1, c2;
};

// sinusoid: phase in cycles ph0 + ph1 s + ph2 s^2 (FP64);
// J~ = sin(2 pi (phase + shift)) (k0 + k1 tr + k2 tr^2), tr = t / T_obs
// = tr0 + s dtr: shift 0 and (1, 0, 0) for A'; a quarter cycle (the cosine)
// and (0, 2 pi A', 0), (0, 0, pi A'), (A', 0, 0) for f0, fdot, phi0
template <>
struct Coord<SMCX_GBSINE> {
  double ph0, ph1, ph2;
  float shift, k0, k1, k2, tr0, dtr;
};

template <int MODEL>
__device__ Coord<MODEL> make_coord(const MetricArgs& a, const double* th, int c, int n,
                                   double* scale) {
  Coord<MODEL> q{};
  *scale = 1.0;
  if (c >= n) return q;  // all coefficients zero
  const int p = c % a.P;
  const double* r = th + (int64_t)(c / a.P) * a.P;
  if constexpr (MODEL == SMCX_PULSE) {
    const double A = r[0], t0 = r[1], w = r[2];
    const double cc = (t0 - a.t_start) / a.dt;
    double nn = floor(cc);
    nn = fmin(fmax(nn, -4194304.0), 4194304.0);
    const double al = kHalfLog2eRoot * a.dt / w;
    const double k = 1.0 / kHalfLog2eRoot;
    q.nf = (float)nn;
    q.a = (float)al;
    q.fa = (float)((cc - nn) * al);
    q.c0 = p == 0 ? 1.f : 0.f;
    q.c1 = p == 1 ? (float)(A * k) : 0.f;
    q.c2 = p == 2 ? (float)(A * k * k) : 0.f;
    *scale = p == 0 ? 1.0 : w;
  } else {
    const double A = r[0], f0 = r[1], fd = r[2], phi0 = r[3];
    const double ts = a.t_start, dt = a.dt;
    q.ph0 = f0 * ts + 0.5 * fd * ts * ts + phi0 / kTwoPiM;
    q.ph1 = (f0 + fd * ts) * dt;
    q.ph2 = 0.5 * fd * dt * dt;
    q.shift = p == 0 ? 0.f : 0.25f;
    q.k0 = p == 0 ? 1.f : (p == 3 ? (float)A : 0.f);
    q.k1 = p == 1 ? (float)(kTwoPiM * A) : 0.f;
    q.k2 = p == 2 ? (float)(kPiM * A) : 0.f;
    q.tr0 = (float)(ts / a.t_obs);
    q.dtr = (float)(dt / a.t_obs);
    *scale = p == 1 ? 1.0 / a.t_obs : (p == 2 ? 1.0 / (a.t_obs * a.t_obs) : 1.0);
  }
  return q;
}

// J~ of one coordinate at sample s.
template <int MODEL>
__device__ __forceinline__ float jvalue(const Coord<MODEL>& q, int s) {
  if constexpr (MODEL == SMCX_PULSE) {
    const float z = __builtin_fmaf((float)s - q.nf, q.a, -q.fa);
    const float e = __builtin_amdgcn_exp2f(-(z * z));
    return e * __builtin_fmaf(__builtin_fmaf(q.c2, z, q.c1), z, q.c0);
  } else {
    const double sd = (double)s;
    const double ph = fma(fma(q.ph2, sd, q.ph1), sd, q.ph0);
    const float rev = (float)(ph - rint(ph)) + q.shift;  // revolutions in [-0.5, 0.75]
    const float tr = __builtin_fmaf((float)s, q.dtr, q.tr0);
    return __builtin_amdgcn_sinf(rev) * __builtin_fmaf(__builtin_fmaf(q.k2, tr, q.k1), tr, q.k0);
  }
}

template <int MODEL, int NB>
__global__ __launch_bounds__(256) void metric_kernel(MetricArgs a) {
  constexpr int NP = NB * (NB + 1) / 2;
  extern __shared__ double scl[];  // [4 waves][32 NB] inverse natural scales of the coordinates
  const int lane = threadIdx.x & 63;
  const int wid = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 4 + wid;
  if (i >= a.N) return;
  const int64_t o0 = a.offsets[i], o1 = a.offsets[i + 1];
  if (!(o0 >= 0 && o1 >= o0 && o1 <= a.M && o1 - o0 <= a.k_max)) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  const int n = (int)(o1 - o0) * a.P;
  const int64_t fo = a.blocks ? o0 * a.P * a.P : a.f_offsets[i];
  if (n > 32 * NB ||
      (!a.blocks && (a.f_offsets[i + 1] - fo != (int64_t)n * n || fo < 0 ||
                     fo + (int64_t)n * n > a.f_size))) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  if (n == 0) return;
  if (a.mask && !a.mask[i]) {
    // not selected: zero blocks (the factor's ridge makes them definite),
    // written by the first window; later windows add nothing
    if (a.w0 == 0) {
      const int64_t cnt = a.blocks ? (int64_t)n * a.P : (int64_t)n * n;
      for (int64_t e = lane; e < cnt; e += 64) a.F[fo + e] = 0.0;
    }
    return;
  }
  const double* th = a.theta + o0 * a.P;
  Coord<MODEL> q[NB];
  double* my = scl + wid * 32 * NB;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    double sc;
    q[b] = make_coord<MODEL>(a, th, 32 * b + (lane & 31), n, &sc);
    if (lane < 32) my[32 * b + lane] = 1.0 / sc;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const double bs = (a.tempered && a.beta ? a.beta[i] : 1.0) * a.inv_sigma2;
  const int half = lane >> 5;  // which group of 4 samples of a step this lane feeds
  float16v acc[NP];
#pragma unroll
  for (int x = 0; x < NP; ++x) acc[x] = float16v{};
  const int w1 = (int)a.w1;  // sample indices fit in 32 bits (T <= 2^22)
#pragma unroll 1
  for (int s0 = (int)a.w0 + 4 * half; s0 < w1 + 4 * half; s0 += 8) {
    half4 j[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = jvalue<MODEL>(q[b], s0 + e);
        j[b][e] = (_Float16)(s0 + e < w1 ? v : 0.f);
      }
    int x = 0;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
      for (int bj = bi; bj < NB; ++bj, ++x)
        acc[x] = __builtin_amdgcn_mfma_f32_32x32x8f16(j[bi], j[bj], acc[x], 0, 0, 0);
  }
  // flush: lane holds D[r_i][c_j] with c_j = lane % 32, r_i = 8 (r/4) + 4 half + r % 4
  const bool first = a.w0 == 0;
  int x = 0;
#pragma unroll
  for (int bi = 0; bi < NB; ++bi)
#pragma unroll
    for (int bj = bi; bj < NB; ++bj, ++x) {
      const int c = 32 * bj + (lane & 31);
      if (c >= n) continue;
      const double sc = bs * my[c];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rr = 32 * bi + 8 * (r >> 2) + 4 * half + (r & 3);
        // inside a diagonal block only the upper triangle is taken and
        // mirrored, so the result is exactly symmetric
        if (rr >= n || (bi == bj && rr > c)) continue;
        const double v = (double)acc[x][r] * sc * my[rr];
        if (a.blocks) {
          // a component's block starts at coordinate P k: entries (rr, c) of
          // one component only, at F + (o0 + k) P P
          if (rr / a.P != c / a.P) continue;
          const int64_t bo = fo + (int64_t)(rr / a.P) * a.P * a.P;
          const int pr = rr % a.P, pc = c % a.P;
          double* e1 = a.F + bo + pr * a.P + pc;
          *e1 = first ? v : *e1 + v;
          if (pr != pc) {
            double* e2 = a.F + bo + pc * a.P + pr;
            *e2 = first ? v : *e2 + v;
          }
          continue;
        }
        double* e1 = a.F + fo + (int64_t)rr * n + c;
        *e1 = first ? v : *e1 + v;
        if (rr != c) {
          double* e2 = a.F + fo + (int64_t)c * n + rr;
          *e2 = first ? v : *e2 + v;
        }
      }
    }
}

// ---------------------------------------------------------------- factor
// W = L^{-1} of M = F + diag(ridge) (M = L L^T), the NUTS mass matrix's
// factor with M^{-1} = W^T W. One workgroup of one wave per particle keeps
// the lower triangle of its block packed in LDS (row r at r (r + 1) / 2):
// right-looking Cholesky, one column per step (the subtractions into each
// entry come in column order, as in the row-by-row textbook form), then the
// in-place inversion of the triangle from the last column to the first with
// W_rj = -(sum_{j<k<=r} W_rk L_kj) / L_jj, W_jj = 1 / L_jj. Lanes own rows;
// barriers separate the steps. A pivot that is not > 0 (or NaN) stops the
// factorisation: the block is filled with NaN and a flag is raised.
struct FactorArgs {
  int P;
  int64_t N, M;
  int32_t k_max;
  const int64_t* offsets;
  const int64_t* f_offsets;
  int64_t f_size;
  const double* F;
  double* W;
  double ridge[8];  // per parameter, P <= 8
  int block;        // 0: the whole block; b: its block-diagonal part in b x b blocks
  int* flag;
  const uint8_t* mask;  // [N] or nullptr: particles with mask[i] == 0 are skipped
  int slices;       // register form: 1: slices of kFactorSlice particles, each handed out
                    // largest K first; 0: particle order
};

__device__ __forceinline__ int tri(int r, int c) { return r * (r + 1) / 2 + c; }

// Factor of the diagonal block [o, o + m) of particle block Fi (n x n), its
// W written into Wi at the same place; L is the LDS triangle (m (m+1)/2
// doubles). Returns false (in every lane) if a pivot is not > 0.
__device__ bool factor_block(const FactorArgs& a, const double* Fi, double* Wi, int n, int o, int m,
                             double* L, int lane) {
  for (int r = 0; r < m; ++r)
    for (int c = lane; c <= r; c += 64)
      L[tri(r, c)] = Fi[(int64_t)(o + r) * n + o + c] + (r == c ? a.ridge[(o + c) % a.P] : 0.0);
  __syncthreads();
  for (int j = 0; j < m; ++j) {
    const double d = L[tri(j, j)];
    if (!(d > 0.0)) {  // the same value in every lane: a uniform exit
      __syncthreads();
      return false;
    }
    const double ljj = sqrt(d);
    __syncthreads();
    for (int r = j + 1 + lane; r < m; r += 64) L[tri(r, j)] = L[tri(r, j)] / ljj;
    if (lane == 0) L[tri(j, j)] = ljj;
    __syncthreads();
    for (int r = j + 1 + lane; r < m; r += 64) {
      const double lrj = L[tri(r, j)];
      for (int c = j + 1; c <= r; ++c) L[tri(r, c)] = fma(-lrj, L[tri(c, j)], L[tri(r, c)]);
    }
    __syncthreads();
  }
  for (int j = m - 1; j >= 0; --j) {
    const double ljj = L[tri(j, j)];
    double acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int r = j + 1 + lane + 64 * t;
      double s = 0.0;
      if (r < m)
        for (int k = j + 1; k <= r; ++k) s = fma(L[tri(r, k)], L[tri(k, j)], s);
      acc[t] = s;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int r = j + 1 + lane + 64 * t;
      if (r < m) L[tri(r, j)] = -acc[t] / ljj;
    }
    if (lane == 0) L[tri(j, j)] = 1.0 / ljj;
    __syncthreads();
  }
  for (int e = lane; e < m * m; e += 64) {
    const int r = e / m, c = e % m;
    Wi[(int64_t)(o + r) * n + o + c] = c <= r ? L[tri(r, c)] : 0.0;
  }
  __syncthreads();  // L is reused by the next block
  return true;
}

__global__ __launch_bounds__(64) void factor_kernel(FactorArgs a) {
  extern __shared__ double L[];
  const int lane = threadIdx.x;
  const int64_t i = blockIdx.x;
  if (i >= a.N) return;
  const int64_t o0 = a.offsets[i], o1 = a.offsets[i + 1];
  if (!(o0 >= 0 && o1 >= o0 && o1 <= a.M && o1 - o0 <= a.k_max)) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  const int n = (int)(o1 - o0) * a.P;
  const int64_t fo = a.f_offsets[i];
  if (a.f_offsets[i + 1] - fo != (int64_t)n * n || fo < 0 || fo + (int64_t)n * n > a.f_size) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  if (a.mask && !a.mask[i]) return;
  if (n == 0) return;
  const double* Fi = a.F + fo;
  double* Wi = a.W + fo;
  bool ok = true;
  if (a.block == 0) {
    ok = factor_block(a, Fi, Wi, n, 0, n, L, lane);
  } else {
    // block-diagonal part only: the blocks between diagonal blocks are zero
    // in W (when W is F itself they are overwritten after every read)
    for (int o = 0; o < n && ok; o += a.block) ok = factor_block(a, Fi, Wi, n, o, a.block, L, lane);
    if (ok)
      for (int64_t e = lane; e < (int64_t)n * n; e += 64) {
        const int r = (int)(e / n), c = (int)(e % n);
        if (r / a.block != c / a.block) Wi[e] = 0.0;
      }
  }
  if (!ok) {
    if (lane == 0) atomicOr(a.flag, kFlagNotPD);
    for (int64_t e = lane; e < (int64_t)n * n; e += 64) Wi[e] = __builtin_nan("");
  }
}

// ---- blocks of up to 64 rows, in registers
// factor_block's LDS form spends its time in serial LDS chains: 577 us for 8192
// blocks of 3 K coordinates, K uniform on 0..20, whose bytes take 31 us. This
// form takes 96 us (85 repeated), bound by the latency of its chains; one wave
// per workgroup, so that a long block holds no other's slot, and the long
// blocks first.
// Here lane r keeps row r of the block in registers and one sweep over the
// columns both eliminates and inverts, in place: with F + diag(ridge) =
// U^{-1} D U^{-T} (U unit lower triangular), step j takes m_r = -A_rj / A_jj
// in every lane r > j and adds m_r times one vector b to the whole row, where
// b_c is A_cj (the column, held by the lanes) for c > j and U_jc (lane j's
// finished row) for c < j; column j then becomes U_rj = m_r. At the end
// W = D^{-1/2} U.
// Eight steps at a time: on the block's own eight columns step by step, the
// vector from lane to scalar registers; on the others all at once, since the
// eight columns of U that the steps leave are just the row's multiples of the
// eight vectors as they were before (150 us with every step on every column,
// an LDS round trip and a row written by one lane in each). Those go through LDS
// once per eight steps and come back 16 entries to a register, one per lane
// of a row of 16, from where v_fmac_f64 broadcasts each entry by itself (DPP
// row_newbcast): one instruction per entry and step, where a read of every
// entry by all lanes would keep the LDS busy longer than the FMAs take.
// The register array is rotated by eight columns after every eight steps,
// so that the block's columns sit at a fixed place: register i of block jb
// holds column (jb + i) mod NR.
#define SMCX_FMAC8(r, o, b, m, c0, c1, c2, c3, c4, c5, c6, c7)                                     \
  asm("s_nop 1\n\t" /* b may come from a register copy: two wait states before DPP */            \
      "v_fmac_f64_dpp %0, %8, %9 row_newbcast:" #c0 " row_mask:0xf bank_mask:0xf\n\t"            \
      "v_fmac_f64_dpp %1, %8, %9 row_newbcast:" #c1 " row_mask:0xf bank_mask:0xf\n\t"            \
      "v_fmac_f64_dpp %2, %8, %9 row_newbcast:" #c2 " row_mask:0xf bank_mask:0xf\n\t"            \
      "v_fmac_f64_dpp %3, %8, %9 row_newbcast:" #c3 " row_mask:0xf bank_mask:0xf\n\t"            \
      "v_fmac_f64_dpp %4, %8, %9 row_newbcast:" #c4 " row_mask:0xf bank_mask:0xf\n\t"            \
      "v_fmac_f64_dpp %5, %8, %9 row_newbcast:" #c5 " row_mask:0xf bank_mask:0xf\n\t"            \
      "v_fmac_f64_dpp %6, %8, %9 row_newbcast:" #c6 " row_mask:0xf bank_mask:0xf\n\t"            \
      "v_fmac_f64_dpp %7, %8, %9 row_newbcast:" #c7 " row_mask:0xf bank_mask:0xf"                  \
      : "+v"(r[(o) + 0]), "+v"(r[(o) + 1]), "+v"(r[(o) + 2]), "+v"(r[(o) + 3]), "+v"(r[(o) + 4]),  \
        "+v"(r[(o) + 5]), "+v"(r[(o) + 6]), "+v"(r[(o) + 7])                                       \
      : "v"(b), "v"(m))

__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

constexpr int kRowPad = 17;  // doubles per row of the 16-column stage

// Factor of the n x n block Fi (n <= NR <= 64, NR - n < 8) into Wi by one
// full wave; sh: the wave's LDS, NR rows of kRowPad doubles. Returns false
// (in every lane, Wi untouched) if a pivot is not > 0.
template <int NR>
__device__ __forceinline__ bool factor_rows(const FactorArgs& a, const double* Fi, double* Wi, int n,
                                            double* sh, int lane) {
  double r[NR];
  const int sub = lane & 15;
  // rows in whole lines, 16 columns at a time through LDS; only the lower
  // triangle is read, all of it in flight together (the row registers are
  // not live yet): group g, its t-th set of four rows, at entry kAt(g) + t
  constexpr auto kAt = [](int g) { return g * (NR / 4) - 4 * (g * (g - 1) / 2); };
  constexpr int kGroups = (NR + 15) / 16;
  double in[kAt(kGroups)];
#pragma unroll
  for (int g = 0; g < kGroups; ++g)
#pragma unroll
    for (int t = 0; t < (NR - 16 * g) / 4; ++t) {
      const int row = 16 * g + 4 * t + (lane >> 4), c = 16 * g + sub;
      in[kAt(g) + t] = row < n && c <= row ? Fi[row * n + c] : 0.0;
    }
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int c0 = 16 * g, c = c0 + sub;
    const double ridge = a.ridge[c % a.P];
#pragma unroll
    for (int t = 0; t < (NR - c0) / 4; ++t) {
      const int row = c0 + 4 * t + (lane >> 4);
      sh[row * kRowPad + sub] = in[kAt(g) + t] + (c == row && row < n ? ridge : 0.0);
    }
    wave_lds_order();
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (c0 + u < NR) r[c0 + u] = sh[min(lane, NR - 1) * kRowPad + u];
    wave_lds_order();
  }
  double pivot = 1.0;
#pragma unroll 1
  for (int jb = 0; jb < NR; jb += 8) {
    // the block's rows before its steps, for the update of the other columns:
    // entry i of row u is A_c,jb+u (the column, held by the lanes) for a column
    // still to come, the finished row's entry for one before the block
    if constexpr (NR > 8) {
      if (lane >= jb + 8 && lane < NR)
#pragma unroll
        for (int u = 0; u < 8; ++u) sh[u * NR + lane - jb] = r[u];
      if (lane >= jb && lane < jb + 8)
#pragma unroll
        for (int g = 8; g < NR; g += 8)
          if (g >= NR - jb)
#pragma unroll
            for (int i = g; i < g + 8; ++i) sh[(lane - jb) * NR + i] = r[i];
      wave_lds_order();
    }
    // the eight steps on the block's own columns, r[0..7]
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = jb + u;
      if (j < n) {
        const double x = r[u];
        const double d = lane_value(x, j);
        if (!(d > 0.0)) return false;
        if (lane == j) pivot = d;
        double e[8];
#pragma unroll
        for (int v = 0; v < 8; ++v)
          if (v != u) e[v] = v > u ? lane_value(x, jb + v) : lane_value(r[v], j);
        double t = x * (-1.0 / d);
        asm("" : "+v"(t));  // in every lane, without a branch around the division
        const double m = lane > j && lane < n ? t : 0.0;
#pragma unroll
        for (int v = 0; v < 8; ++v)
          if (v != u) r[v] = fma(m, e[v], r[v]);
        r[u] = lane == j ? 1.0 : m;
      }
    }
    // the other columns: a lane's steps are its entries of U against the rows as
    // they were
    if constexpr (NR > 8) {
      // a row's entry group is read again, for the next row, right after its use
      constexpr int kQ = (NR + 15) / 16;
      double b[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) b[q] = sh[16 * q + sub];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double m = lane > jb + u ? r[u] : 0.0;
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          if (q > 0) SMCX_FMAC8(r, 16 * q, b[q], m, 0, 1, 2, 3, 4, 5, 6, 7);
          if (16 * q + 8 < NR)
            SMCX_FMAC8(r, (16 * q + 8 < NR ? 16 * q + 8 : 0), b[q], m, 8, 9, 10, 11, 12, 13, 14, 15);
          __builtin_amdgcn_sched_barrier(0);
          if (u < 7) b[q] = sh[(u + 1) * NR + 16 * q + sub];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      wave_lds_order();
    }
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = r[u];
#pragma unroll
    for (int i = 0; i + 8 < NR; ++i) r[i] = r[i + 8];
#pragma unroll
    for (int u = 0; u < 8; ++u) r[NR - 8 + u] = t[u];
  }
  const double s = 1.0 / sqrt(pivot);
  asm volatile("" : "+v"(lane));  // what the output takes from it is formed anew, not held
#pragma unroll
  for (int c0 = 0; c0 < NR; c0 += 16) {
    if (lane < NR)
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (c0 + u < NR) sh[lane * kRowPad + u] = r[c0 + u] * s;
    wave_lds_order();
    const int c = c0 + (lane & 15);
    if (c < n)
      for (int row = lane >> 4; row < n; row += 4) Wi[row * n + c] = sh[row * kRowPad + (lane & 15)];
    wave_lds_order();
  }
  return true;
}

// The p-th longest particle of the slice of 64 that starts at i0, by one wave: its
// index, or -1 where the slice has fewer. Handing out the longest of every slice,
// then the second longest and so on starts the long blocks first, as one sorted
// list would, and needs no list: a wave finds its own particle from one load of
// the slice's offsets. With blocks of n = 3 to 60 in particle order the last,
// long ones left the device idle for a quarter of the time (8192 blocks: 113 us
// repeated; with a list from a launch of its own 86, and workspace that the
// handle's calls on other streams share; this way 86. 20000 blocks: 205 to 213
// with the list, 210 to 220). Particles of equal K come in index order, and every
// particle is some wave's: an invalid one counts as the longest or as empty,
// and the factor validates for itself.
constexpr int kFactorSlice = 64;

__device__ __forceinline__ int64_t slice_particle(const FactorArgs& a, int64_t i0, int p) {
  const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int64_t i = i0 + lane, j = i < a.N ? i : a.N - 1;
  const int64_t K = a.offsets[j + 1] - a.offsets[j];
  const int key = i < a.N ? (int)min(max(K, (int64_t)0), (int64_t)a.k_max + 1) : -1;
  for (int k = a.k_max + 1; k >= 0; --k) {
    const unsigned long long same = __builtin_amdgcn_ballot_w64(key == k);
    const int n = __popcll(same);
    if (p >= n) {
      p -= n;
      continue;
    }
    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((unsigned)same, 0u));
    return i0 + __builtin_ctzll(__builtin_amdgcn_ballot_w64(key == k && before == p));
  }
  return -1;
}

// One wave per particle, CAP >= k_max P rows at most.
template <int CAP>
__global__ __launch_bounds__(64, (CAP <= 32 ? 5 : 3)) void factor_rows_kernel(FactorArgs a) {
  __shared__ double sh[CAP * kRowPad];
  const int lane = threadIdx.x;
  int64_t i = blockIdx.x;
  if (a.slices) {
    // row p of the grid takes the slices' p-th particles, turned by p, so that a
    // slice does not fall to the same dies every time
    unsigned s = blockIdx.x + blockIdx.y;
    while (s >= gridDim.x) s -= gridDim.x;
    i = slice_particle(a, (int64_t)s * kFactorSlice, (int)blockIdx.y);
    if (i < 0) return;
  }
  const int64_t o0 = a.offsets[i], o1 = a.offsets[i + 1];
  if (!(o0 >= 0 && o1 >= o0 && o1 <= a.M && o1 - o0 <= a.k_max)) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  const int n = __builtin_amdgcn_readfirstlane((int)(o1 - o0) * a.P);
  const int64_t fo = a.f_offsets[i];
  if (a.f_offsets[i + 1] - fo != (int64_t)n * n || fo < 0 || fo + (int64_t)n * n > a.f_size) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  if (n == 0 || (a.mask && !a.mask[i])) return;
  const double* Fi = a.F + fo;
  double* Wi = a.W + fo;
  bool ok = false;
  switch ((n + 7) / 8) {
    case 1: ok = factor_rows<8>(a, Fi, Wi, n, sh, lane); break;
    case 2: ok = factor_rows<16>(a, Fi, Wi, n, sh, lane); break;
    case 3: ok = factor_rows<24>(a, Fi, Wi, n, sh, lane); break;
    case 4: ok = factor_rows<32>(a, Fi, Wi, n, sh, lane); break;
    default:
      if constexpr (CAP > 32) {
        switch ((n + 7) / 8) {
          case 5: ok = factor_rows<40>(a, Fi, Wi, n, sh, lane); break;
          case 6: ok = factor_rows<48>(a, Fi, Wi, n, sh, lane); break;
          case 7: ok = factor_rows<56>(a, Fi, Wi, n, sh, lane); break;
          case 8: ok = factor_rows<64>(a, Fi, Wi, n, sh, lane); break;
        }
      }
  }
  if (!ok) {
    if (lane == 0) atomicOr(a.flag, kFlagNotPD);
    for (int e = lane; e < n * n; e += 64) Wi[e] = __builtin_nan("");
  }
}

// One P x P block per thread, W_m = L^{-1} with L L^T = F_m + diag(ridge),
// in registers: the same steps in the same order as factor_block, so a block
// comes out bitwise as the workgroup factor's block mode gives it. A pivot
// that is not > 0 (or NaN) fills the block with NaN and raises the flag.
struct RidgeP {
  double r[8];
};

template <int P>
__global__ __launch_bounds__(256) void factor_blocks_kernel(const double* F, double* W, int64_t M,
                                                            RidgeP rg, int* flag) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= M) return;
  const double* f = F + m * P * P;
  double L[P][P];
#pragma unroll
  for (int r = 0; r < P; ++r)
#pragma unroll
    for (int c = 0; c <= r; ++c) L[r][c] = f[r * P + c] + (r == c ? rg.r[c] : 0.0);
  bool ok = true;
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const double d = L[j][j];
    ok = ok && d > 0.0;
    const double ljj = sqrt(d);
#pragma unroll
    for (int r = j + 1; r < P; ++r) L[r][j] = L[r][j] / ljj;
    L[j][j] = ljj;
#pragma unroll
    for (int r = j + 1; r < P; ++r) {
      const double lrj = L[r][j];
#pragma unroll
      for (int c = j + 1; c <= r; ++c) L[r][c] = fma(-lrj, L[c][j], L[r][c]);
    }
  }
#pragma unroll
  for (int j = P - 1; j >= 0; --j) {
    const double ljj = L[j][j];
    double acc[P];
#pragma unroll
    for (int r = j + 1; r < P; ++r) {
      double s = 0.0;
#pragma unroll
      for (int k = j + 1; k <= r; ++k) s = fma(L[r][k], L[k][j], s);
      acc[r] = s;
    }
#pragma unroll
    for (int r = j + 1; r < P; ++r) L[r][j] = -acc[r] / ljj;
    L[j][j] = 1.0 / ljj;
  }
  double* w = W + m * P * P;
#pragma unroll
  for (int r = 0; r < P; ++r)
#pragma unroll
    for (int c = 0; c < P; ++c) w[r * P + c] = !ok ? __builtin_nan("") : (c <= r ? L[r][c] : 0.0);
  if (!ok) atomicOr(flag, kFlagNotPD);
}

}  // namespace

// The population-level mass matrix: the mean of M P x P blocks. Stage one
// sums contiguous row ranges, one lane per entry and four waves taking every
// fourth row, the waves combined in order; stage two adds the range sums in
// order and divides by M. The partition depends only on M and the scratch
// size, so the result is reproducible bit for bit.
constexpr int kPoolWaves = 4;

__global__ __launch_bounds__(64 * kPoolWaves) void pool_partial_kernel(int PP, int64_t M,
                                                                         int64_t rows, const double* F,
                                                                         double* part) {
  __shared__ double sh[kPoolWaves][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  const int64_t r1 = min(M, r0 + rows);
  // four running sums per lane (rows r0 + wid + kPoolWaves (4 j + u) go to
  // sum u), so that four loads are in flight; combined in a fixed order
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  if (lane < PP) {
    int64_t m = r0 + wid;
    for (; m + 3 * kPoolWaves < r1; m += 4 * kPoolWaves)
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += F[(m + u * kPoolWaves) * PP + lane];
    for (int u = 0; m < r1; m += kPoolWaves, ++u) s[u] += F[m * PP + lane];
  }
  sh[wid][lane] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (wid == 0 && lane < PP) {
    double t = sh[0][lane];
    for (int w = 1; w < kPoolWaves; ++w) t += sh[w][lane];
    part[(size_t)blockIdx.x * PP + lane] = t;
  }
}

// The range sums of the G workgroups: 16 waves take every 16th range each,
// then the first wave adds the 16 wave sums in order.
constexpr int kFinalWaves = 16;
__global__ __launch_bounds__(64 * kFinalWaves) void pool_final_kernel(int PP, int G, int64_t M,
                                                                      const double* part,
                                                                      double* out) {
  __shared__ double sh[kFinalWaves][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  double s[2] = {0.0, 0.0};
  if (lane < PP) {
    int g = wid, u = 0;
    for (; g < G; g += kFinalWaves, u ^= 1) s[u] += part[(size_t)g * PP + lane];
  }
  sh[wid][lane] = s[0] + s[1];
  __syncthreads();
  if (wid == 0 && lane < PP) {
    double t = sh[0][lane];
    for (int w = 1; w < kFinalWaves; ++w) t += sh[w][lane];
    out[lane] = t / (double)M;
  }
}

hipError_t launch_metric_factor_blocks(int P, int64_t M, const double* F, const double* ridge,
                                       double* W, int* flag, hipStream_t st) {
  if (M == 0) return hipSuccess;
  RidgeP rg{};
  if (P > 8) return hipErrorInvalidValue;
  for (int p = 0; p < P; ++p) rg.r[p] = ridge[p];
  const dim3 grid((unsigned)((M + 255) / 256)), block(256);
  switch (P) {
    case 3: hipLaunchKernelGGL(factor_blocks_kernel<3>, grid, block, 0, st, F, W, M, rg, flag); break;
    case 4: hipLaunchKernelGGL(factor_blocks_kernel<4>, grid, block, 0, st, F, W, M, rg, flag); break;
    case 8: hipLaunchKernelGGL(factor_blocks_kernel<8>, grid, block, 0, st, F, W, M, rg, flag); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_metric_pool(int P, int64_t M, const double* F, double* F_mean, double* part,
                              size_t part_cap, hipStream_t st) {
  const int PP = P * P;
  if (PP > 64 || M < 1) return hipErrorInvalidValue;
  // about 256 rows per workgroup, at most 1024 workgroups and what the scratch
  // holds; with no room for a range sum, one workgroup sums into F_mean itself
  int64_t G = std::min<int64_t>((M + 255) / 256, 1024);
  G = std::min<int64_t>(G, (int64_t)(part_cap / PP));
  if (G < 1) {
    G = 1;
    part = F_mean;
  }
  const int64_t rows = (M + G - 1) / G;
  G = (M + rows - 1) / rows;
  hipLaunchKernelGGL(pool_partial_kernel, dim3((unsigned)G), dim3(64 * kPoolWaves), 0, st, PP, M,
                     rows, F, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pool_final_kernel, dim3(1), dim3(64 * kFinalWaves), 0, st, PP, (int)G, M, part,
                     F_mean);
  return hipGetLastError();
}

size_t factor_lds_bytes(int nmax) { return (size_t)nmax * (nmax + 1) / 2 * sizeof(double); }

hipError_t launch_metric_factor(int P, int64_t N, int64_t M, int32_t k_max,
                                const int64_t* offsets, const int64_t* f_offsets, int64_t f_size,
                                const double* F, const double* ridge, int block, double* W,
                                int* flag, int n_cu, hipStream_t st, const uint8_t* mask) {
  FactorArgs a{};
  a.P = P;
  a.N = N;
  a.M = M;
  a.k_max = k_max;
  a.offsets = offsets;
  a.f_offsets = f_offsets;
  a.f_size = f_size;
  a.F = F;
  a.W = W;
  if (P > 8) return hipErrorInvalidValue;
  for (int p = 0; p < P; ++p) a.ridge[p] = ridge[p];
  a.flag = flag;
  a.mask = mask;
  a.block = block;
  // whole blocks of up to 64 coordinates in registers, a wave per particle;
  // larger ones do not fit a row per lane, and the block mode's small blocks
  // leave most lanes of either form idle
  if (block == 0 && k_max * P <= 64) {
    // more particles than the device holds at once (three waves per SIMD of
    // the 64-row form): longest first
    a.slices = N > 12 * (int64_t)n_cu;
    const dim3 grid = a.slices ? dim3((unsigned)((N + kFactorSlice - 1) / kFactorSlice), kFactorSlice)
                               : dim3((unsigned)N);
    if (k_max * P <= 32)
      hipLaunchKernelGGL(factor_rows_kernel<32>, grid, dim3(64), 0, st, a);
    else
      hipLaunchKernelGGL(factor_rows_kernel<64>, grid, dim3(64), 0, st, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(factor_kernel, dim3((unsigned)N), dim3(64),
                     factor_lds_bytes(block > 0 ? block : k_max * P), st, a);
  return hipGetLastError();
}

namespace {
template <int MODEL>
hipError_t launch_groups(MetricArgs a, int64_t windows, hipStream_t st) {
  // one wave per group on a single window, else up to four windows of a group
  // at once (a long record of few particles has few groups)
  const int wpg = windows == 1 ? 1 : (windows == 2 ? 2 : 4);
  // slots per block: its groups on average, and a quarter more for the blocks
  // above it (beyond, a wave takes further groups; an idle one costs its
  // packing); above 16 components a group holds one particle
  const int64_t per = std::min<int64_t>(a.N, kGroupBlock);
  const int64_t rows = (a.M * per + a.N - 1) / a.N;
  const int64_t full = a.M > 16 * a.N ? per : (rows + 31) / 32;
  a.slots = (int)std::min(per, full + (full + 3) / 4 + 1);
  const dim3 grid((unsigned)(((int64_t)a.nblk * a.slots * wpg + 3) / 4)), block(256);
  if (wpg == 1)
    hipLaunchKernelGGL((metric_group_kernel<MODEL, 1>), grid, block, 0, st, a);
  else if (wpg == 2)
    hipLaunchKernelGGL((metric_group_kernel<MODEL, 2>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((metric_group_kernel<MODEL, 4>), grid, block, 0, st, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_metric(int model, int P, int64_t N, int64_t M, int64_t T, double t_start,
                         double dt, double inv_sigma2, int32_t k_max, const int64_t* offsets,
                         const double* theta, const double* beta, const int64_t* f_offsets,
                         int64_t f_size, double* F, int64_t split, int blocks, int* flag,
                         int n_cu, hipStream_t st, const uint8_t* mask) {
  MetricArgs a{P, N, M, T, t_start, dt, inv_sigma2, (double)T * dt, k_max, offsets, theta,
               beta, f_offsets, f_size, F, flag, 0, 0, 1, blocks, mask, split,
               (int)((N + kGroupBlock - 1) / kGroupBlock), 1};
  const int nmax = k_max * P;
  if (nmax > 128) return hipErrorInvalidValue;
  const int nb = nmax <= 32 ? 1 : (nmax <= 64 ? 2 : 4);
  {
    // The grouped form saves vector work and takes several windows at once,
    // but spends about 40 us on packing and flushing and more per step of
    // a lone wave (0.15 us against 0.09 with one block of coordinates). It wins
    // where the coordinate form would put four waves of work or more on each
    // SIMD, with 1024 samples or more for their products (in us, coordinate
    // against grouped form; pulses, K on 0..10: 6000 particles, T = 500: 60, 63,
    // T = 1000: 95, 73; 4096, T = 500: 46, 64, T = 1000: 71, 71, T = 4096: 223,
    // 115; 2048, T = 1500: 58, 73. K on 0..20, three products a sample: 2048,
    // T = 500: 54, 58, T = 1000: 73, 65; 1024, T = 4096: 140, 115, left with the
    // coordinate form. Sinusoids, K on 0..8: 4096, T = 500: 57, 74, T = 1500:
    // 125, 104), or on more than two windows (256 pulse particles, T = 16384: 264,
    // 131). Its flush into whole matrices costs as much as 100 samples or more,
    // twice that where the particles fill the coordinate form's blocks (dense, 40000
    // sinusoid particles, T = 138, K on 1..8, 18 of 32 coordinates: 142, 190;
    // T = 250: 215, 209; K on 0..10, 20 of 64, T = 138: 223, 197; 30000, T = 100: 0.96).
    // Beyond 64 coordinates the compiler rounds some of the coordinate
    // form's products to FP32 before FP16 and others once, depending on the
    // block; the grouped form would change F by 2e-7 there (below it gives the
    // same bits), so those keep the coordinate form.
    const int64_t windows = (split + kFlushSamples - 1) / kFlushSamples +
                            (T - split + kFlushSamples - 1) / kFlushSamples;
    const int64_t waves = 16 * (int64_t)n_cu, products = N * (nb * (nb + 1) / 2);  // per sample
    const int64_t t_dense = 5 * M * P > 64 * nb * N ? 224 : 120;  // above or below 0.4 filled
    if (nb <= 2 && (windows > 2 || (N * nb >= waves && products * T >= 1024 * waves &&
                                    (blocks || T >= t_dense))))
      return model == SMCX_PULSE ? launch_groups<SMCX_PULSE>(a, windows, st)
                                 : launch_groups<SMCX_GBSINE>(a, windows, st);
  }
  const dim3 grid((unsigned)((N + 3) / 4)), block(256);
  const size_t lds = 4 * 32 * (size_t)nb * sizeof(double);
  // one launch per window of samples: later windows add to what earlier ones
  // wrote; with a bridge split the windows stop at the split, and only those
  // after it are tempered
  for (int64_t w0 = 0; w0 < T; w0 = a.w1) {
    const int64_t end = split > 0 && w0 < split ? split : T;  // windows never straddle the split
    a.w0 = w0;
    a.w1 = w0 + kFlushSamples < end ? w0 + kFlushSamples : end;
    a.tempered = split == 0 || w0 >= split ? 1 : 0;
    if (model == SMCX_PULSE) {
      if (nb == 1) hipLaunchKernelGGL((metric_kernel<SMCX_PULSE, 1>), grid, block, lds, st, a);
      else if (nb == 2) hipLaunchKernelGGL((metric_kernel<SMCX_PULSE, 2>), grid, block, lds, st, a);
      else hipLaunchKernelGGL((metric_kernel<SMCX_PULSE, 4>), grid, block, lds, st, a);
    } else {
      if (nb == 1) hipLaunchKernelGGL((metric_kernel<SMCX_GBSINE, 1>), grid, block, lds, st, a);
      else if (nb == 2) hipLaunchKernelGGL((metric_kernel<SMCX_GBSINE, 2>), grid, block, lds, st, a);
      else hipLaunchKernelGGL((metric_kernel<SMCX_GBSINE, 4>), grid, block, lds, st, a);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace smcx
