// LISA Galactic binaries in the frequency domain (Sec. "LISA Galactic
// binaries"): eight parameters per source (f0, fdot, log10 A, ecliptic
// latitude and longitude, psi, iota, phi0), the A and E channels in the
// long-wavelength limit of the constellation, and the likelihood of
// eq. gw_likelihood with a constant PSD over a band of bins [k0, k0 + B):
//   logL = -(1/2) (4 / (T_obs S)) sum_c sum_k |d_c[k] - h_c[k]|^2.
//
// Templates use the fast/slow decomposition the paper's waveforms come from:
// the heterodyned envelope z_c(t) = a_c(t) e^{i(Phi(tau) - 2 pi q t / T_obs)} / 2
// (carrier bin q = floor(f0 T_obs), tau the retarded time at the guiding
// centre) is sampled at t_j = j T_obs / 64 and its 64-point DFT fills bins
// q - 32 .. q + 31:  h_c[q + m] = (T_obs / 64) sum_j z_c(t_j) e^{-2 pi i m j / 64}.
//
// Mapping: one wave per particle; lane j owns envelope sample j and band
// bins j + 64 r. A source's 64 samples go through one FFT across the wave
// (radix 2, six stages over lane pairs lane ^ h, both channels at once,
// FP64), then each lane fetches the window value of its own bins from the
// lane holding it.
// The residual stays in registers; the adjoint contracts the inverse FFT of
// each source's residual window with the analytic envelope derivatives, so
// d logL / d theta = beta (4 / (T_obs S)) (T_obs / 64) Re sum_j conj(w_j) dz_j.
// Everything is FP64: a source concentrates its signal in a few bins, where
// an FP32 template would not hold the likelihood to 1e-6.
#include "smcx_nuts.h"
#include "smcx_prep.h"

#include <math.h>

#include <algorithm>

// The library is built without floating-point contraction so that the
// time-domain kernels round as written. These FP64 kernels are held to a
// tolerance and rely on no particular rounding of a product followed by a
// sum, so here a * b + c may fuse into one FMA.
#pragma clang fp contract(fast)

namespace smcx {
namespace {

constexpr int kNs = 64;
constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr double kLn10 = 2.302585092994045684017991454684;
constexpr double kAuLight = 1.495978707e11 / 299792458.0;  // R / c [s]

// Per-lane constants of the coarse time grid: symmetric detector tensors
// of A and E (xx, yy, zz, xy, xz, yz), cos and sin of the orbital phase,
// t_j. Each workgroup stages them in LDS as [field][lane], so that a wave
// reads one field of all its lanes without bank conflicts; g points at this
// lane's column. Read where used, they keep 15 doubles out of the registers
// of the particle's whole pass.
constexpr int kGeoFields = 15;
struct LaneGeom {
  const double* g;
  __device__ __forceinline__ double d(int c, int x) const { return g[(6 * c + x) * 64]; }
  __device__ __forceinline__ double ca() const { return g[12 * 64]; }
  __device__ __forceinline__ double sa() const { return g[13 * 64]; }
  __device__ __forceinline__ double t() const { return g[14 * 64]; }
};

// The lane tables of a workgroup, in the dynamic LDS of the launch: the FFT
// twiddles, forward then inverse, [stage][lane][re, im] each; the phase
// table of the envelope; the grid of the handle's record; under a bridge
// that of its partner (otherwise geo[1] aliases geo[0] and takes no space).
// The gradient kernel adds one residual copy per wave after them
// (fd_lds_words).
constexpr int kTwWords = 2 * 6 * 128;
constexpr int kTrigWords = 2 * (kFdTrigSteps + 1);
constexpr int kGeoWords = kGeoFields * 64;
struct FdTables {
  const double* tw;
  const double* trig;
  const double* geo[2];
};

extern __shared__ double fd_lds[];

// Doubles of dynamic LDS a frequency-domain launch needs: the tables, plus
// resid_words per wave.
constexpr size_t fd_lds_words(bool bridge, int waves, int resid_words) {
  return (size_t)kTwWords + kTrigWords + (bridge ? 2 : 1) * kGeoWords + (size_t)waves * resid_words;
}

// Every thread of the workgroup calls this before any of them returns.
// Returns the first word after the tables.
__device__ __forceinline__ double* stage_tables(FdTables& t, const double* own, const double* partner) {
  double* tw = fd_lds;
  double* trig = tw + kTwWords;
  double* g0 = trig + kTrigWords;
  double* g1 = partner ? g0 + kGeoWords : g0;
  for (int x = threadIdx.x; x < kGeoWords; x += blockDim.x) {
    const int f = x >> 6, l = x & 63;
    g0[x] = own[l * kFdTableStride + f];
    if (partner) g1[x] = partner[l * kFdTableStride + f];
  }
  for (int x = threadIdx.x; x < kTwWords; x += blockDim.x) tw[x] = own[kFdTwiddleFwd + x];
  for (int x = threadIdx.x; x < kTrigWords; x += blockDim.x) trig[x] = own[kFdTrig + x];
  __syncthreads();
  t.tw = tw;
  t.trig = trig;
  t.geo[0] = g0;
  t.geo[1] = g1;
  return (partner ? g1 : g0) + kGeoWords;
}

// Orders the LDS accesses of one wave around it (they complete in order;
// this keeps the compiler from moving them across).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct V3 {
  double x, y, z;
};
__device__ __forceinline__ double dot3(const V3& a, const V3& b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 mul_sym(const double* d, const V3& v) {
  return {d[0] * v.x + d[3] * v.y + d[4] * v.z, d[3] * v.x + d[1] * v.y + d[5] * v.z,
          d[4] * v.x + d[5] * v.y + d[2] * v.z};
}

// Source constants, the same in every lane.
struct Src {
  double f0, fd, A, cb, sb, cl, sl, c2p, s2p, ci, si, cyc0;
  double Ap, Ax;  // amplitudes of h+ and hx
  // The antenna patterns Fp = cos(2 psi) P + sin(2 psi) X and
  // Fx = -sin(2 psi) P + cos(2 psi) X of the quadratic forms P = u.D u - v.D v
  // and X = 2 u.D v of a detector tensor D, as weights of its six components
  // (xx, yy, zz, xy, xz, yz): Fp = sum fpw[e] D[e], Fx = sum fxw[e] D[e].
  double fpw[6], fxw[6];
  // The weights of the forms n.D u and n.D v in the same way (the
  // zz weight of n.D v is zero, v having no z component: five words).
  double wnu[6], wnv[5];
  V3 n, u, v;  // v = (-sin l, cos l, 0)
  int64_t q;
};

// Source constants, one row of kSrcWords doubles per row of theta, written
// before each frequency-domain launch (with the ordering pass or by
// fd_src_kernel, one lane per source) and read by the kernels at wave-uniform addresses through a
// restrict-qualified pointer, so they arrive by scalar loads into scalar
// registers instead of occupying vector registers in every lane. Words 0-32
// hold the constants with the carrier bin q of the handle's record, word 33
// the carrier bin under the bridge partner's observation time, words 34-44
// the weights of n.D u and n.D v, word 45 is zero.
constexpr int kSrcWords = kFdSrcWords;
constexpr int kQOwn = 32, kQPartner = 33, kWnu = 34, kWnv = 40;

// All words but the partner's carrier bin.
__device__ __forceinline__ void src_store(double* c, const Src& s) {
  const double v[33] = {s.f0,    s.fd,    s.A,     s.cb,    s.sb,    s.cl,    s.sl,
                        s.c2p,    s.s2p,    s.ci,     s.si,     s.cyc0,   s.Ap,     s.Ax,
                        s.fpw[0], s.fpw[1], s.fpw[2], s.fpw[3], s.fpw[4], s.fpw[5], s.fxw[0],
                        s.fxw[1], s.fxw[2], s.fxw[3], s.fxw[4], s.fxw[5], s.n.x,    s.n.y,
                        s.n.z,   s.u.x,   s.u.y,   s.u.z,   __builtin_bit_cast(double, s.q)};
#pragma unroll
  for (int x = 0; x < 33; ++x) c[x] = v[x];
#pragma unroll
  for (int x = 0; x < 6; ++x) c[kWnu + x] = s.wnu[x];
#pragma unroll
  for (int x = 0; x < 5; ++x) c[kWnv + x] = s.wnv[x];
  c[kSrcWords - 1] = 0.0;
}

__device__ __forceinline__ Src src_load(const double* c, int qslot) {
  Src s;
  s.f0 = c[0]; s.fd = c[1]; s.A = c[2]; s.cb = c[3]; s.sb = c[4]; s.cl = c[5]; s.sl = c[6];
  s.c2p = c[7]; s.s2p = c[8]; s.ci = c[9]; s.si = c[10]; s.cyc0 = c[11]; s.Ap = c[12]; s.Ax = c[13];
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    s.fpw[e] = c[14 + e];
    s.fxw[e] = c[20 + e];
  }
  s.n = {c[26], c[27], c[28]};
  s.u = {c[29], c[30], c[31]};
  s.v = {-s.sl, s.cl, 0.0};
  s.q = __builtin_bit_cast(int64_t, c[qslot]);  // stored as its bit pattern
#pragma unroll
  for (int x = 0; x < 6; ++x) s.wnu[x] = c[kWnu + x];
#pragma unroll
  for (int x = 0; x < 5; ++x) s.wnv[x] = c[kWnv + x];
  return s;
}

// The constants from the parameters with the sines and cosines given.
__device__ __forceinline__ Src make_src_from(const double* th, double T_obs, double sb, double cb,
                                             double sl, double cl, double s2p, double c2p, double si,
                                             double ci) {
  Src s;
  s.f0 = th[0];
  s.fd = th[1];
  s.A = exp10(th[2] + 21.0);
  s.sb = sb;
  s.cb = cb;
  s.sl = sl;
  s.cl = cl;
  s.s2p = s2p;
  s.c2p = c2p;
  s.si = si;
  s.ci = ci;
  s.cyc0 = th[7] / kTwoPi;
  s.n = {s.cb * s.cl, s.cb * s.sl, s.sb};
  s.u = {s.sb * s.cl, s.sb * s.sl, -s.cb};
  s.v = {-s.sl, s.cl, 0.0};
  s.q = (int64_t)floor(s.f0 * T_obs);
  s.Ap = s.A * (1.0 + s.ci * s.ci);
  s.Ax = -2.0 * s.A * s.ci;
  const V3& u = s.u;
  const V3& v = s.v;
  // weights of P and X, then of the antenna patterns
  const double ep[6] = {u.x * u.x - v.x * v.x,         u.y * u.y - v.y * v.y,
                        u.z * u.z - v.z * v.z,         2.0 * (u.x * u.y - v.x * v.y),
                        2.0 * (u.x * u.z - v.x * v.z), 2.0 * (u.y * u.z - v.y * v.z)};
  const double ex[6] = {2.0 * u.x * v.x,               2.0 * u.y * v.y,
                        2.0 * u.z * v.z,               2.0 * (u.x * v.y + u.y * v.x),
                        2.0 * (u.x * v.z + u.z * v.x), 2.0 * (u.y * v.z + u.z * v.y)};
  for (int x = 0; x < 6; ++x) {
    s.fpw[x] = s.c2p * ep[x] + s.s2p * ex[x];
    s.fxw[x] = -s.s2p * ep[x] + s.c2p * ex[x];
  }
  const V3& n = s.n;
  s.wnu[0] = n.x * u.x;
  s.wnu[1] = n.y * u.y;
  s.wnu[2] = n.z * u.z;
  s.wnu[3] = n.x * u.y + n.y * u.x;
  s.wnu[4] = n.x * u.z + n.z * u.x;
  s.wnu[5] = n.y * u.z + n.z * u.y;
  s.wnv[0] = n.x * v.x;  // xx, yy, xy, xz, yz
  s.wnv[1] = n.y * v.y;
  s.wnv[2] = n.x * v.y + n.y * v.x;
  s.wnv[3] = n.z * v.x;
  s.wnv[4] = n.z * v.y;
  return s;
}

__device__ __forceinline__ Src make_src(const double* th, double T_obs) {
  double sb, cb, sl, cl, s2p, c2p, si, ci;
  sincos(th[3], &sb, &cb);
  sincos(th[4], &sl, &cl);
  sincos(2.0 * th[5], &s2p, &c2p);
  sincos(th[6], &si, &ci);
  return make_src_from(th, T_obs, sb, cb, sl, cl, s2p, c2p, si, ci);
}

// Envelope of one source at this lane's sample, both channels (no (-1)^j).
struct Env {
  double zr[2], zi[2];  // z_c
  double ar[2], ai[2];  // complex amplitude a_c
  double Fp[2], Fx[2];  // antenna patterns
  double cph, sph, tau, doppler;  // doppler = cos(a - l) (R/c)
};

// The amplitude part of the envelope: antenna patterns, complex amplitudes,
// Doppler delay and retarded time (no phase).
__device__ __forceinline__ Env envelope_amp(const Src& s, const LaneGeom& g) {
  Env e;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double Fp = 0.0, Fx = 0.0;
#pragma unroll
    for (int x = 0; x < 6; ++x) {
      const double D = g.d(c, x);
      Fp = fma(s.fpw[x], D, Fp);
      Fx = fma(s.fxw[x], D, Fx);
    }
    e.Fp[c] = Fp;
    e.Fx[c] = Fx;
    e.ar[c] = e.Fp[c] * s.Ap;
    e.ai[c] = -e.Fx[c] * s.Ax;
  }
  e.doppler = kAuLight * (g.ca() * s.cl + g.sa() * s.sl);
  e.tau = g.t() + s.cb * e.doppler;
  return e;
}

// cos and sin of 2 pi cyc: the nearest step k / 128 of the phase (t = 128 cyc
// and its nearest integer are exact, and so is their difference), turned
// by the remainder x = 2 pi (cyc - k / 128), |x| <= pi / 128, whose sine
// and cosine are their Taylor series cut after x^7 and x^6 (the next terms
// are below 1e-20 and 4e-18). The cut is relative to the double-precision
// ulp far smaller than the rounding of the two products that turn the step.
// The table (trig) holds cos, sin of 2 pi k / 128 for k = -64..64; the step
// is taken modulo 128, so any phase (a NaN one converts to some integer)
// indexes inside it.
__device__ __forceinline__ void cis_cycles(double cyc, const double* trig, double* c, double* s) {
  const double t = cyc * (double)kFdTrigSteps;  // exact
  const double kf = rint(t);
  const double x = (t - kf) * (kTwoPi / kFdTrigSteps);  // t - kf is exact
  const double x2 = x * x;
  const double sx = fma(x * x2, fma(x2, fma(x2, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0), x);
  const double cx = fma(x2, fma(x2, fma(x2, -1.0 / 720.0, 1.0 / 24.0), -0.5), 1.0);
  const int k = ((int)kf + kFdTrigSteps / 2) & (kFdTrigSteps - 1);  // entry of the step modulo 128
  const double ck = trig[2 * k], sk = trig[2 * k + 1];
  *c = fma(ck, cx, -(sk * sx));
  *s = fma(sk, cx, ck * sx);
}

// zs: the factor of z (1/2 for the envelope itself).
__device__ __forceinline__ Env envelope(const Src& s, const LaneGeom& g, const double* trig,
                                        int lane, double zs = 0.5) {
  Env e = envelope_amp(s, g);
  // phase in cycles (heterodyned at the carrier bin q), reduced by cis_cycles
  // before the product with 2 pi
  const double cyc = fma(e.tau, fma(0.5 * s.fd, e.tau, s.f0),
                         fma(-(double)(int)(s.q & (kNs - 1)), (double)lane * (1.0 / kNs), s.cyc0));
  cis_cycles(cyc, trig, &e.cph, &e.sph);
  // zs (a_c e^{i ph}) with a_c = Ap Fp_c - i Ax Fx_c
  const double zp = zs * s.Ap, zx = zs * s.Ax;
  const double pc = zp * e.cph, ps = zp * e.sph, xc = zx * e.cph, xs = zx * e.sph;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    e.zr[c] = e.Fp[c] * pc + e.Fx[c] * xs;
    e.zi[c] = e.Fp[c] * ps - e.Fx[c] * xc;
  }
  return e;
}

// The value of lane (lane ^ H), H a power of two below 64, with no trip
// through the LDS crossbar: DPP row permutations for H <= 8 (H = 4 and 8 as
// the half-row mirror i -> i ^ 7 followed by i -> i ^ 3 or the row mirror
// i -> i ^ 15) and the row-swap instructions for H = 16 and 32.
template <int H>
__device__ __forceinline__ int xor_lane_u32(int v, int lane) {
  if constexpr (H == 1) {
    return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
  } else if constexpr (H == 2) {
    return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
  } else if constexpr (H == 4) {
    const int t = __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);  // row_half_mirror
    return __builtin_amdgcn_mov_dpp(t, 0x1B, 0xF, 0xF, true);          // quad_perm [3,2,1,0]
  } else if constexpr (H == 8) {
    const int t = __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);  // row_half_mirror
    return __builtin_amdgcn_mov_dpp(t, 0x140, 0xF, 0xF, true);         // row_mirror
  } else if constexpr (H == 16) {
    // both operands a copy of v: the first ends with rows (0, 0, 2, 2), the
    // second with rows (1, 1, 3, 3)
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    return (int)((lane & 16) ? r[0] : r[1]);
  } else {
    static_assert(H == 32, "xor distance");
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return (int)((lane & 32) ? r[0] : r[1]);
  }
}

template <int H>
__device__ __forceinline__ double xor_lane(double v, int lane) {
  const int64_t b = __builtin_bit_cast(int64_t, v);
  const int lo = xor_lane_u32<H>((int)(uint32_t)b, lane), hi = xor_lane_u32<H>((int)(b >> 32), lane);
  return __builtin_bit_cast(double, (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

__device__ __forceinline__ double join_words(unsigned lo, unsigned hi) {
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

// Half-lane moves at distance H = 4 or 8, where a DPP row shift can write
// only the lanes of one side (its bank mask selects groups of four lanes):
// from_above gives the lanes with bit H clear the value src of lane L + H and
// leaves old in the others; from_below gives the lanes with bit H set src of
// lane L - H and leaves old in the rest. Two of them make a trade between
// lane pairs with no select.
template <int H, bool ABOVE>
__device__ __forceinline__ double half_move(double old, double src) {
  static_assert(H == 4 || H == 8, "bank-masked move distance");
  constexpr int kCtrl = ABOVE ? 0x100 + H : 0x110 + H;  // row_shl:H or row_shr:H
  constexpr int kBanks = ABOVE ? (H == 8 ? 0x3 : 0x5) : (H == 8 ? 0xC : 0xA);
  const uint64_t uo = __builtin_bit_cast(uint64_t, old), us = __builtin_bit_cast(uint64_t, src);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)uo, (int)(unsigned)us,
                                                            kCtrl, 0xF, kBanks, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(uo >> 32),
                                                            (int)(unsigned)(us >> 32), kCtrl, 0xF,
                                                            kBanks, false);
  return join_words(lo, hi);
}
template <int H>
__device__ __forceinline__ double from_above(double old, double src) { return half_move<H, true>(old, src); }
template <int H>
__device__ __forceinline__ double from_below(double old, double src) { return half_move<H, false>(old, src); }

// v of lane L - N within the row of 16 lanes (lanes with L mod 16 < N get 0).
template <int N>
__device__ __forceinline__ double row_shr(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, 0x110 + N, 0xF, 0xF, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), 0x110 + N, 0xF, 0xF, true);
  return join_words(lo, hi);
}

// Transposed sums: a stage over lane pairs (L, L ^ H) takes two partial sums
// per lane and leaves one, lanes with bit H clear keeping the first value's
// pair sum and the others the second's. Each value's total is formed over
// the same pairs, level by level, as in a butterfly, so it is bitwise the
// same; a stage costs one exchange per pair of values instead of one per
// value. At H = 32 and 16 the row swaps do it without selects: after
// swapping the upper rows of a with the lower rows of b, a + b holds a's pair
// sum in the lower rows and b's in the upper ones; at H = 8 and 4 the
// half-lane moves do the same.
template <int H>
__device__ __forceinline__ double pair_sum(double a, double b, int lane) {
  if constexpr (H == 32 || H == 16) {
    const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
    const unsigned alo = (unsigned)ua, ahi = (unsigned)(ua >> 32), blo = (unsigned)ub, bhi = (unsigned)(ub >> 32);
    if constexpr (H == 32) {
      const auto lo = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
      const auto hi = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
      return join_words(lo[0], hi[0]) + join_words(lo[1], hi[1]);
    } else {
      const auto lo = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
      return join_words(lo[0], hi[0]) + join_words(lo[1], hi[1]);
    }
  } else if constexpr (H == 8 || H == 4) {
    // lanes with bit H clear: (own a, a of L + H); set: (b of L - H, own b)
    return from_below<H>(a, b) + from_above<H>(b, a);
  } else {
    const bool up = lane & H;
    const double send = up ? a : b, keep = up ? b : a;
    return keep + xor_lane<H>(send, lane);
  }
}

// Wave totals of eight values: lane L with L mod 8 = 7 ends with the total
// of v[L >> 3]. The last three levels add the value of lane L - 4, L - 2 and
// L - 1, which pairs the same partial sums as a butterfly would.
__device__ __forceinline__ double transposed_sum8(const double v[8], int lane) {
  double t5[4], t4[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) t5[i] = pair_sum<32>(v[i], v[i + 4], lane);
#pragma unroll
  for (int i = 0; i < 2; ++i) t4[i] = pair_sum<16>(t5[i], t5[i + 2], lane);
  double t = pair_sum<8>(t4[0], t4[1], lane);
  t += row_shr<4>(t);
  t += row_shr<2>(t);
  t += row_shr<1>(t);
  return t;
}

// Wave totals of 36 values. Value x is given the lane slot kSlot36[x]; the
// slots are R5 and R5 + 32 with R5 = R4 and R4 + 16, R4 = {0,1,2,4,5,8,9,10,12},
// so each stage halves the number of live partial sums (36, 18, 9, 5, 3, 2,
// 1) and pairs absent from a stage are zero. Lane L ends with the total of
// the value whose slot is L.
__constant__ const int kSlot36[36] = {0,  1,  2,  4,  5,  8,  9,  10, 12, 16, 17, 18,
                                      20, 21, 24, 25, 26, 28, 32, 33, 34, 36, 37, 40,
                                      41, 42, 44, 48, 49, 50, 52, 53, 56, 57, 58, 60};

__device__ __forceinline__ double transposed_sum36(const double v[36], int lane) {
  double t5[18], t4[9], t3[5], t2[3], t1[2];
#pragma unroll
  for (int i = 0; i < 18; ++i) t5[i] = pair_sum<32>(v[i], v[i + 18], lane);
#pragma unroll
  for (int i = 0; i < 9; ++i) t4[i] = pair_sum<16>(t5[i], t5[i + 9], lane);
#pragma unroll
  for (int i = 0; i < 5; ++i) t3[i] = pair_sum<8>(t4[i], i + 5 < 9 ? t4[i + 5] : 0.0, lane);
#pragma unroll
  for (int i = 0; i < 3; ++i) t2[i] = pair_sum<4>(t3[i], i + 3 < 5 ? t3[i + 3] : 0.0, lane);
#pragma unroll
  for (int i = 0; i < 2; ++i) t1[i] = pair_sum<2>(t2[i], i + 2 < 3 ? t2[i + 2] : 0.0, lane);
  return pair_sum<1>(t1[0], t1[1], lane);
}

// The 64-point transforms keep two complex values per lane, A and B; at the
// start A is channel A's and B channel E's sample of the lane. A stage of
// span H first trades values between lanes L and L ^ H so that a lane with
// bit H clear holds (its A, the partner's A) and one with bit H set (the
// partner's B, its B): a butterfly pair of one sub-transform. The lane then
// forms both outputs of that butterfly, so no lane computes a result it
// throws away. At H = 32 and 16 the row swaps make the trade, one
// instruction per register; at H = 8 and 4 two half-lane moves; at H = 2
// and 1 one DPP exchange and selects. After the
// six forward stages lane 32c + i holds channel c's window bins bitrev5(i)
// and 32 + bitrev5(i); one more row swap at span 32 leaves lane 32s + i with
// both channels of bin 32s + bitrev5(i). Each trade is its own inverse, so
// the inverse transform runs the stages backwards. The twiddles come from
// the table, one complex number per lane and stage.
struct Pair {
  double ar, ai, br, bi;  // A = ar + i ai, B = br + i bi
};

// the trade at span 32 or 16 of one register pair
template <int H>
__device__ __forceinline__ void row_swap(double& a, double& b) {
  const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
  const unsigned alo = (unsigned)ua, ahi = (unsigned)(ua >> 32), blo = (unsigned)ub, bhi = (unsigned)(ub >> 32);
  if constexpr (H == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
    a = join_words(lo[0], hi[0]);
    b = join_words(lo[1], hi[1]);
  } else {
    static_assert(H == 16, "row swap span");
    const auto lo = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
    a = join_words(lo[0], hi[0]);
    b = join_words(lo[1], hi[1]);
  }
}

template <int H>
__device__ __forceinline__ void trade(Pair& p, int lane) {
  if constexpr (H >= 16) {
    row_swap<H>(p.ar, p.br);
    row_swap<H>(p.ai, p.bi);
  } else if constexpr (H >= 4) {
    // lanes with bit H clear keep A and take the B of lane L + H; the others
    // keep B and take the A of lane L - H
    const double nbr = from_above<H>(p.br, p.ar), nbi = from_above<H>(p.bi, p.ai);
    p.ar = from_below<H>(p.ar, p.br);
    p.ai = from_below<H>(p.ai, p.bi);
    p.br = nbr;
    p.bi = nbi;
  } else {
    const bool set = lane & H;
    const double rr = xor_lane<H>(set ? p.ar : p.br, lane), ri = xor_lane<H>(set ? p.ai : p.bi, lane);
    p.ar = set ? rr : p.ar;
    p.ai = set ? ri : p.ai;
    p.br = set ? p.br : rr;
    p.bi = set ? p.bi : ri;
  }
}

// Forward stage S (span 32 >> S), decimation in frequency: (a, b) ->
// (a + b, (a - b) w). Down to span 4 the pair arrives in order (x the
// element of the lower index). At spans 2 and 1 the lane keeps x (its A, or
// its B with bit H set) and receives y, so the pair is (x, y) or (y, x); the
// sign of the difference in the second case is folded into the lane's
// twiddle, which at span 1 is that sign alone (the root is 1), applied by
// flipping the sign bit.
template <int S>
__device__ __forceinline__ void fwd_stage(Pair& p, const double* tw, int lane) {
  constexpr int H = 32 >> S;
  double xr, xi, yr, yi;
  if constexpr (H >= 16) {
    row_swap<H>(p.ar, p.br);
    row_swap<H>(p.ai, p.bi);
    xr = p.ar;
    xi = p.ai;
    yr = p.br;
    yi = p.bi;
  } else if constexpr (H >= 4) {
    // lanes with bit H clear: (own A, A of lane L + H); set: (B of L - H, own B)
    xr = from_below<H>(p.ar, p.br);
    xi = from_below<H>(p.ai, p.bi);
    yr = from_above<H>(p.br, p.ar);
    yi = from_above<H>(p.bi, p.ai);
  } else {
    const bool set = lane & H;
    xr = set ? p.br : p.ar;
    xi = set ? p.bi : p.ai;
    yr = xor_lane<H>(set ? p.ar : p.br, lane);
    yi = xor_lane<H>(set ? p.ai : p.bi, lane);
  }
  const double dr = xr - yr, di = xi - yi;
  p.ar = xr + yr;
  p.ai = xi + yi;
  if constexpr (H == 1) {
    const uint64_t sgn = (uint64_t)(lane & 1) << 63;
    p.br = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, dr) ^ sgn);
    p.bi = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, di) ^ sgn);
  } else {
    const double wr = tw[S * 128 + 2 * lane], wi = tw[S * 128 + 2 * lane + 1];
    p.br = dr * wr - di * wi;
    p.bi = dr * wi + di * wr;
  }
}

// Inverse stage S: (s, d) -> (s + conj(w) d, s - conj(w) d), then the trade
// (at span 1 the root is 1).
template <int S>
__device__ __forceinline__ void inv_stage(Pair& p, const double* tw, int lane) {
  constexpr int H = 32 >> S;
  double tr = p.br, ti = p.bi;
  if constexpr (H > 1) {
    const double wr = tw[S * 128 + 2 * lane], wi = tw[S * 128 + 2 * lane + 1];
    tr = p.br * wr - p.bi * wi;
    ti = p.br * wi + p.bi * wr;
  }
  const double sr = p.ar, si = p.ai;
  p.ar = sr + tr;
  p.ai = si + ti;
  p.br = sr - tr;
  p.bi = si - ti;
  trade<H>(p, lane);
}

__device__ __forceinline__ int bitrev5(int x) { return (int)(__builtin_bitreverse32((unsigned)x) >> 27); }

// The lane holding window bin m (0 <= m < 64) after the forward transform,
// and the bin a lane holds: the map is its own inverse.
__device__ __forceinline__ int bin_lane(int m) { return (m & 32) | bitrev5(m & 31); }

// Forward DFT of both channels over the wave: lane j holds sample j of each
// channel in (re[c], im[c]); lane bin_lane(m) ends with bin m of each.
// tw: the forward twiddles ([stage][lane][re, im]).
__device__ __forceinline__ void fft_fwd(double re[2], double im[2], const double* tw, int lane) {
  Pair p{re[0], im[0], re[1], im[1]};
  fwd_stage<0>(p, tw, lane);
  fwd_stage<1>(p, tw, lane);
  fwd_stage<2>(p, tw, lane);
  fwd_stage<3>(p, tw, lane);
  fwd_stage<4>(p, tw, lane);
  fwd_stage<5>(p, tw, lane);
  row_swap<32>(p.ar, p.br);
  row_swap<32>(p.ai, p.bi);
  re[0] = p.ar;
  im[0] = p.ai;
  re[1] = p.br;
  im[1] = p.bi;
}

// Inverse (unnormalised, e^{+2 pi i m j / 64}) DFT of both channels: lane L
// holds bin bin_lane(L) of each channel, or with SPLIT lane 32c + i holds
// channel c's bins bitrev5(i) in (re[0], im[0]) and 32 + bitrev5(i) in
// (re[1], im[1]) (the layout of the forward stages before their last row
// swap); lane j ends with sample j. tw: the inverse twiddles.
template <bool SPLIT = false>
__device__ __forceinline__ void fft_inv(double re[2], double im[2], const double* tw, int lane) {
  Pair p{re[0], im[0], re[1], im[1]};
  if constexpr (!SPLIT) {
    row_swap<32>(p.ar, p.br);
    row_swap<32>(p.ai, p.bi);
  }
  inv_stage<5>(p, tw, lane);
  inv_stage<4>(p, tw, lane);
  inv_stage<3>(p, tw, lane);
  inv_stage<2>(p, tw, lane);
  inv_stage<1>(p, tw, lane);
  inv_stage<0>(p, tw, lane);
  re[0] = p.ar;
  im[0] = p.ai;
  re[1] = p.br;
  im[1] = p.bi;
}

// Butterfly sum: every lane ends with the same (bitwise) total, since each
// stage adds the same two values in both lanes of a pair.
__device__ __forceinline__ double wave_sum(double v, int lane) {
  v += xor_lane<32>(v, lane);
  v += xor_lane<16>(v, lane);
  v += xor_lane<8>(v, lane);
  v += xor_lane<4>(v, lane);
  v += xor_lane<2>(v, lane);
  v += xor_lane<1>(v, lane);
  return v;
}

// The source's window spectrum (times T_obs / 64) across the wave: lane L
// holds bin q - 32 + bin_lane(L).
__device__ __forceinline__ void window_spectrum(const Src& s, const LaneGeom& g, const double* tw,
                                                const double* trig, double scale, int lane,
                                                double re[2], double im[2]) {
  // (-1)^j centres the window on q
  const Env e = envelope(s, g, trig, lane, (lane & 1) ? -0.5 * scale : 0.5 * scale);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    re[c] = e.zr[c];
    im[c] = e.zi[c];
  }
  fft_fwd(re, im, tw, lane);
}

// Value of the window spectrum at band bin b (0 outside the window), read
// from the lane that holds it. All lanes must call this together.
__device__ __forceinline__ void window_at(const double re[2], const double im[2], int64_t b_abs,
                                          int64_t q, double out_re[2], double out_im[2]) {
  const int64_t m = b_abs - (q - kNs / 2);
  const bool in = m >= 0 && m < kNs;
  const int src = bin_lane((int)(m & (kNs - 1)));
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const double vr = __shfl(re[c], src), vi = __shfl(im[c], src);
    out_re[c] = in ? vr : 0.0;
    out_im[c] = in ? vi : 0.0;
  }
}

// One data set of the likelihood: the handle's own, or under a bridge
// (eq. reuse_bridge between two records) also its partner's.
struct FdSide {
  const double* data;
  const double* tw;  // twiddles in LDS, forward then inverse
  const double* trig;  // phase table in LDS
  LaneGeom g;        // this lane's grid constants in LDS
  int64_t k0, B;
  double T_obs, scale, cnorm;
  int qslot;         // word of the source rows with this record's carrier bin
};

__device__ __forceinline__ FdSide own_side(const PopArgs& a, const FdTables& t, int lane) {
  return {a.fd_data, t.tw, t.trig, LaneGeom{t.geo[0] + lane}, a.fd_k0, a.fd_B, a.fd_T_obs,
          a.fd_scale, a.inv_sigma2, kQOwn};
}
__device__ __forceinline__ FdSide partner_side(const PopArgs& a, const FdTables& t, int lane) {
  return {a.fd2_data, t.tw, t.trig, LaneGeom{t.geo[1] + lane}, a.fd2_k0, a.fd2_B, a.fd2_T_obs,
          a.fd2_T_obs / 64.0, a.fd2_cnorm, kQPartner};
}

template <int NR>
struct Resid {
  double re[2][NR], im[2][NR];
};

template <int NR>
__device__ __forceinline__ void load_resid(const FdSide& sd, int lane, Resid<NR>& R) {
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int b = lane + kNs * r;
      R.re[c][r] = sd.data[(c * kFdBandStride + b) * 2];
      R.im[c][r] = sd.data[(c * kFdBandStride + b) * 2 + 1];
    }
}

// Band index of the source's window bin 0 (wave-uniform), clamped to
// [-2 kNs, B], which leaves every test of a band bin against the window and
// the band as it was and keeps the index arithmetic in 32 bits.
__device__ __forceinline__ int window_start(int64_t q, const FdSide& sd) {
  const int64_t lo = q - kNs / 2 - sd.k0;
  return (int)(lo < -2 * kNs ? -2 * kNs : (lo > sd.B ? sd.B : lo));
}

// R -= sign h over the band (sign = +-1). Each band bin takes the window
// value from the lane holding it, weighted by sign where the bin lies in both
// the window and the band and by 0 elsewhere: one FMA per value, which
// rounds as R - sign v.
template <int NR>
__device__ __forceinline__ void subtract_source(const FdSide& sd, const Src& s, const LaneGeom& g,
                                                int lane, Resid<NR>& R, double sign) {
  double re[2], im[2];
  window_spectrum(s, g, sd.tw, sd.trig, sd.scale, lane, re, im);
  const int lo = window_start(s.q, sd);  // band index of window bin 0
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int b = lane + kNs * r, m = b - lo;
    const double f = ((unsigned)m < (unsigned)kNs && b < (int)sd.B) ? -sign : 0.0;
    const int from = bin_lane(m & (kNs - 1));
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      R.re[c][r] = fma(f, __shfl(re[c], from), R.re[c][r]);
      R.im[c][r] = fma(f, __shfl(im[c], from), R.im[c][r]);
    }
  }
}

// Re<R, h> and |h|^2 over the band for one source (both channels).
template <int NR>
__device__ __forceinline__ void overlap(const FdSide& sd, const Src& s, const LaneGeom& g, int lane,
                                        const Resid<NR>& R, double* rh, double* hh) {
  double re[2], im[2];
  window_spectrum(s, g, sd.tw, sd.trig, sd.scale, lane, re, im);
  double x = 0.0, y = 0.0;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int64_t b = lane + kNs * r;
    double vr[2], vi[2];
    window_at(re, im, sd.k0 + b, s.q, vr, vi);
    if (b < sd.B)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        x = fma(R.re[c][r], vr[c], fma(R.im[c][r], vi[c], x));
        y = fma(vr[c], vr[c], fma(vi[c], vi[c], y));
      }
  }
  *rh = wave_sum(x, lane);
  *hh = wave_sum(y, lane);
}

// Derivatives of the envelope z_c = a_c e^{i ph} / 2 (channel c) with respect
// to the eight parameters at this lane's sample: dz_p = (da_p e^{i ph}) / 2 +
// i dphi_p z = (e^{i ph} / 2) g_p with g_p = da_p + i dphi_p a_c, a the complex
// amplitude and ph the heterodyned phase. This returns g_p; the phase factor
// has modulus one and drops out of the metric entries Re(conj(dz_a) dz_b).
__device__ __forceinline__ void amp_phase_derivs(const Src& s, const LaneGeom& g, const Env& e, int c,
                                                 double gr[8], double gi[8]) {
  const double Ap = s.Ap, Ax = s.Ax;
  const double fi = s.f0 + s.fd * e.tau;
  const double dphi[8] = {kTwoPi * e.tau, 0.5 * kTwoPi * e.tau * e.tau, 0.0,
                          kTwoPi * fi * (-s.sb * e.doppler),
                          kTwoPi * fi * (s.cb * kAuLight * (g.sa() * s.cl - g.ca() * s.sl)), 0.0, 0.0,
                          1.0};
  const V3 ul = {s.sb * s.v.x, s.sb * s.v.y, 0.0};
  const V3 vl = {-s.cl, -s.sl, 0.0};
  double D[6];
#pragma unroll
  for (int x = 0; x < 6; ++x) D[x] = g.d(c, x);
  const V3 Du = mul_sym(D, s.u), Dv = mul_sym(D, s.v);
  const double dPb = 2.0 * dot3(s.n, Du), dXb = 2.0 * dot3(s.n, Dv);
  const double dPl = 2.0 * (dot3(ul, Du) - dot3(vl, Dv));
  const double dXl = 2.0 * (dot3(ul, Dv) + dot3(vl, Du));
  double da_r[8], da_i[8];
  da_r[0] = da_i[0] = da_r[1] = da_i[1] = da_r[7] = da_i[7] = 0.0;
  da_r[2] = kLn10 * e.ar[c];
  da_i[2] = kLn10 * e.ai[c];
  da_r[3] = (s.c2p * dPb + s.s2p * dXb) * Ap;
  da_i[3] = -(-s.s2p * dPb + s.c2p * dXb) * Ax;
  da_r[4] = (s.c2p * dPl + s.s2p * dXl) * Ap;
  da_i[4] = -(-s.s2p * dPl + s.c2p * dXl) * Ax;
  da_r[5] = 2.0 * e.Fx[c] * Ap;
  da_i[5] = 2.0 * e.Fp[c] * Ax;
  da_r[6] = e.Fp[c] * (-2.0 * s.A * s.ci * s.si);
  da_i[6] = -e.Fx[c] * (2.0 * s.A * s.si);
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    gr[p] = da_r[p] - dphi[p] * e.ai[c];
    gi[p] = da_i[p] + dphi[p] * e.ar[c];
  }
}



// This lane's share of the gradient of one source, sum_c Re(conj(w_c) dz_c,p)
// for the eight parameters, without forming dz_c,p = (da_c,p / 2) e^{i ph} +
// i dphi_p z_c (amp_phase_derivs): per channel
//   Re(conj(w) dz_p) = Re(da_p) ur + Im(da_p) ui + dphi_p (Im w Re z - Re w Im z),
// ur = (Re w cos ph + Im w sin ph) / 2, ui = (Im w cos ph - Re w sin ph) / 2.
// The caller passes w up to a sign, which half (+-1/2) restores. With the
// amplitudes a_c = Ap Fp_c - i Ax Fx_c, every amplitude and phase term is a
// combination of four channel sums S1 = sum Fp ur, S2 = sum Fp ui,
// S3 = sum Fx ur, S4 = sum Fx ui: the phase factor shared by the dphi terms
// is G = sum (Im w Re z - Re w Im z) = sum (Re a ui - Im a ur) = Ap S2 + Ax S3,
// the amplitude's own term sum (Re a ur + Im a ui) = Ap S1 - Ax S4, the
// polarisation angle's sum (Fx Ap ur + Fp Ax ui) = Ap S3 + Ax S2 and the
// inclination's sum (cos(i) Fp ur + Fx ui) = cos(i) S1 + S4. The two sky
// derivatives are linear in (dP, dX), which are bilinear in the detector
// tensor D_c, so with the weights alpha_c = c2p Ap ur + s2p Ax ui,
// beta_c = s2p Ap ur - c2p Ax ui that the polarisation angle and the
// amplitudes give dP and dX they contract to 2 n.D y1 (latitude) and
// 2 (ul.D y1 + vl.D y2) (longitude), y1 = alpha u + beta v, y2 = beta u - alpha v,
// ul = sin(b) v and vl = -(cos(b) n + sin(b) u) the derivatives of u and v
// with respect to the longitude. With D symmetric these reduce to the forms
// n.D u and n.D v and the patterns P and X:
//   latitude:  2 sum (alpha n.D u + beta n.D v)
//   longitude: 2 sum (alpha (sin(b) X + cos(b) n.D v) - beta (sin(b) P + cos(b) n.D u)),
// where sum (alpha X - beta P) is the polarisation angle's sum above (P and X
// rotated by 2 psi are Fp and Fx), and the rest is linear in the four sums
// U1 = sum ur n.D u, U2 = sum ui n.D u, V1 = sum ur n.D v, V2 = sum ui n.D v.
__device__ __forceinline__ void grad_terms(const Src& s, const LaneGeom& g, const Env& e,
                                           const double wr[2], const double wi[2], double half,
                                           double gp[8]) {
  const double Ap = s.Ap, Ax = s.Ax;
  const double hc = half * e.cph, hs = half * e.sph;
  double ur[2], ui[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    ur[c] = wr[c] * hc + wi[c] * hs;
    ui[c] = wi[c] * hc - wr[c] * hs;
  }
  const double S1 = e.Fp[0] * ur[0] + e.Fp[1] * ur[1], S2 = e.Fp[0] * ui[0] + e.Fp[1] * ui[1];
  const double S3 = e.Fx[0] * ur[0] + e.Fx[1] * ur[1], S4 = e.Fx[0] * ui[0] + e.Fx[1] * ui[1];
  const double G = Ap * S2 + Ax * S3;
  const double t5 = Ap * S3 + Ax * S2;
  // the phase derivatives times G: 2 pi (tau, tau^2 / 2) and 2 pi f_i times
  // the Doppler delay's derivatives, f_i = f0 + fdot tau
  const double G2 = kTwoPi * G;
  const double Gf = (s.f0 + s.fd * e.tau) * G2;
  gp[0] = e.tau * G2;
  gp[1] = (0.5 * e.tau) * gp[0];
  gp[2] = kLn10 * (Ap * S1 - Ax * S4);
  gp[5] = 2.0 * t5;
  gp[6] = -2.0 * s.A * s.si * (s.ci * S1 + S4);
  gp[7] = G;
  // the sky derivatives, one channel at a time (the barrier keeps the two
  // channels' temporaries from being live together)
  static constexpr int kVx[5] = {0, 1, 3, 4, 5};  // the tensor entries of the n.D v weights
  double U1 = 0.0, U2 = 0.0, V1 = 0.0, V2 = 0.0;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double nDu = 0.0, nDv = 0.0;
#pragma unroll
    for (int x = 0; x < 6; ++x) nDu = fma(s.wnu[x], g.d(c, x), nDu);
#pragma unroll
    for (int x = 0; x < 5; ++x) nDv = fma(s.wnv[x], g.d(c, kVx[x]), nDv);
    U1 = fma(ur[c], nDu, U1);
    U2 = fma(ui[c], nDu, U2);
    V1 = fma(ur[c], nDv, V1);
    V2 = fma(ui[c], nDv, V2);
    __builtin_amdgcn_sched_barrier(0);
  }
  const double kPa = s.c2p * Ap, kXa = s.s2p * Ax, kPb = s.s2p * Ap, kXb = s.c2p * Ax;
  const double lat = (kPa * U1 + kXa * U2) + (kPb * V1 - kXb * V2);
  const double lon = (kPa * V1 + kXa * V2) - (kPb * U1 - kXb * U2);
  gp[3] = (-s.sb * e.doppler) * Gf + 2.0 * lat;
  gp[4] = (s.cb * kAuLight) * (g.sa() * s.cl - g.ca() * s.sl) * Gf + 2.0 * (s.sb * t5 + s.cb * lon);
}

struct FdItem {
  int64_t i, m0;
  int K;
};

// Work items of a launch: the ranks of the ordering pass (valid particles with
// K > 0, or all valid ones for birth/death), else N.
__device__ __forceinline__ int64_t fd_count(const PopArgs& a) {
  return a.order ? a.n_ranks : a.N;
}

// Work item at rank < fd_count(a); false for an empty rank and for a particle
// whose offsets are invalid or exceed k_max.
__device__ __forceinline__ bool fd_item_at(const PopArgs& a, int64_t rank, FdItem& it) {
  it.i = a.order ? (int64_t)a.order[rank] : rank;
  if (it.i < 0) return false;  // an empty rank
  const int64_t o0 = a.offsets[it.i], o1 = a.offsets[it.i + 1];
  if (!(o0 >= 0 && o1 >= o0 && o1 <= a.M && o1 - o0 <= a.k_max)) return false;
  it.m0 = o0;
  it.K = (int)(o1 - o0);
  return true;
}

__device__ __forceinline__ bool fd_active_at(const PopArgs& a, int64_t rank, FdItem& it) {
  return fd_item_at(a, rank, it) && !(a.active && !a.active[it.i]);
}

// A wave's residual copy in LDS (the gradient pass): four rows (re, im of
// A, re, im of E) of kNs NR band bins and one zero word that gathers from
// outside the band read.
template <int NR>
constexpr int resid_row() { return kNs * NR + 2; }
template <int NR>
constexpr int resid_words() { return 4 * resid_row<NR>(); }

// |R|^2 over the band and both channels.
template <int NR>
__device__ __forceinline__ double resid_square(const Resid<NR>& R, int lane) {
  double ss = 0.0;
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < NR; ++r) ss = fma(R.re[c][r], R.re[c][r], fma(R.im[c][r], R.im[c][r], ss));
  return wave_sum(ss, lane);
}

// The residual into the wave's LDS copy ([re, im of A, re, im of E][band
// position]).
template <int NR>
__device__ __forceinline__ void stage_resid(const Resid<NR>& R, int lane, double* rl) {
  constexpr int Bp = kNs * NR, rs = resid_row<NR>();
  wave_lds_sync();
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      rl[(2 * c) * rs + lane + kNs * r] = R.re[c][r];
      rl[(2 * c + 1) * rs + lane + kNs * r] = R.im[c][r];
    }
  if (lane < 4) rl[lane * rs + Bp] = 0.0;
  wave_lds_sync();
}

// The gradient of a source from the residual in LDS: lane 8p + 7 ends with
// parameter p's.
template <int NR>
__device__ __forceinline__ double fd_adjoint(const FdSide& sd, const Src& s, int lane, double wc,
                                             const double* rl) {
  constexpr int Bp = kNs * NR, rs = resid_row<NR>();
  // the window bins this lane gathers, in the split layout of the inverse
  // transform: channel lane >> 5, bins m0 and m0 + 32
  const int wc0 = (lane >> 5) * 2, m0 = bitrev5(lane & 31);
  // residual window of the source in the inverse transform's input order
  const int lo = window_start(s.q, sd);  // band index of window bin 0
  double wr[2], wi[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int bw = lo + m0 + 32 * h;  // band index this lane gathers
    const int bi = (unsigned)bw < (unsigned)sd.B ? bw : Bp;  // the zero word outside the band
    wr[h] = rl[wc0 * rs + bi];
    wi[h] = rl[(wc0 + 1) * rs + bi];
  }
  fft_inv<true>(wr, wi, sd.tw + 6 * 128, lane);
  // w_j = sum_m R[q + m] e^{2 pi i m j / 64} = (-1)^j times the inverse DFT
  // of the window (indexed from q - 32); the sign goes with the factor 1/2
  // Re(conj(w) dz) per parameter
  const Env e = envelope(s, sd.g, sd.trig, lane);
  double gp[8];
  grad_terms(s, sd.g, e, wr, wi, (lane & 1) ? -0.5 : 0.5, gp);
  return transposed_sum8(gp, lane) * (wc * sd.scale);
}

// Stores it for source row m, added to the first side's after it, with the
// closing kick of a leapfrog step (he) after the last side.
__device__ __forceinline__ void store_gradient(const PopArgs& a, int64_t m, int lane, double gv, double he,
                                               bool first, bool last) {
  if ((lane & 7) == 7) {
    const int64_t x = m * 8 + (lane >> 3);
    if (!first && a.grad) gv += a.grad[x];
    if (a.grad) a.grad[x] = gv;
    if (last && a.p_half) a.p_out[x] = fma(he, gv, a.p_half[x]);
  }
}

// The change of logL by the particle's birth candidate, and by the death of a
// component, from its residual.
template <int NR>
__device__ __forceinline__ void fd_birth(const PopArgs& a, const FdSide& sd, const FdItem& it, int lane,
                                         const Resid<NR>& R, double wc, bool first) {
  const int64_t i = it.i;
  if (a.theta_birth && a.dlogl_birth) {
    const Src s = make_src(a.theta_birth + i * 8, sd.T_obs);
    double rh, hh;
    overlap<NR>(sd, s, sd.g, lane, R, &rh, &hh);
    const double v = wc * (rh - 0.5 * hh);
    if (lane == 0) a.dlogl_birth[i] = first ? v : a.dlogl_birth[i] + v;
  }
}

template <int NR>
__device__ __forceinline__ void fd_death(const PopArgs& a, const FdSide& sd, const FdItem& it, int lane,
                                         const Resid<NR>& R, double wc, bool first,
                                         const double* __restrict__ src) {
  const int64_t i = it.i;
  if (a.death_idx && a.dlogl_death) {
    const int j = a.death_idx[i];
    if (j >= 0 && j < it.K) {
      const int row = __builtin_amdgcn_readfirstlane((int)(it.m0 + j));
      const Src s = src_load(src + (int64_t)row * kSrcWords, sd.qslot);
      double rh, hh;
      overlap<NR>(sd, s, sd.g, lane, R, &rh, &hh);
      const double v = -(wc * (rh + 0.5 * hh));
      if (lane == 0) a.dlogl_death[i] = first ? v : a.dlogl_death[i] + v;
    } else if (lane == 0 && first) {
      a.dlogl_death[i] = j == -1 ? 0.0 : __builtin_nan("");
      if (j != -1) atomicOr(a.flag, kFlagDeath);
    }
  }
}

// One particle on one data set, weighted by w; the first side writes the
// outputs, a second one adds to them, and the leapfrog kick (p_half set)
// follows the last side's gradient. rl: the wave's residual copy in LDS
// (MODE 1).
template <int MODE, int NR>
__device__ __forceinline__ void fd_particle(const PopArgs& a, const FdSide& sd, const FdItem& it,
                                            int lane, double w, bool first, bool last,
                                            const double* __restrict__ src, double* rl) {
  const int64_t i = it.i;
  const double wc = w * sd.cnorm;  // weight * 4 / (T_obs S)
  const LaneGeom g = sd.g;
  Resid<NR> R;
  load_resid<NR>(sd, lane, R);
  for (int k = 0; k < it.K; ++k) {
    const int row = __builtin_amdgcn_readfirstlane((int)(it.m0 + k));
    // the lane index, opaque in each pass, so that the lane's grid constants
    // are read from LDS for every source instead of held in 30 registers
    // through the loop
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const LaneGeom gk{g.g + (ln - lane)};
    subtract_source<NR>(sd, src_load(src + (int64_t)row * kSrcWords, sd.qslot), gk, lane, R, 1.0);
  }
  if constexpr (MODE == 2) {
    fd_birth<NR>(a, sd, it, lane, R, wc, first);
    fd_death<NR>(a, sd, it, lane, R, wc, first, src);
    return;
  }
  const double ss = resid_square<NR>(R, lane);
  if (lane == 0 && a.logl) {
    const double v = -0.5 * wc * ss;
    a.logl[i] = first ? v : a.logl[i] + v;
  }
  if constexpr (MODE == 1) {
    const double he = a.p_half ? 0.5 * a.eps * (a.dir ? (double)a.dir[i] : 1.0) : 0.0;
    // the loop gathers each source's window from the wave's LDS copy of the
    // residual, whose registers are free for the adjoint
    stage_resid<NR>(R, lane, rl);
    for (int k = 0; k < it.K; ++k) {
      const int row = __builtin_amdgcn_readfirstlane((int)(it.m0 + k));
      const double gv = fd_adjoint<NR>(sd, src_load(src + (int64_t)row * kSrcWords, sd.qslot), lane, wc, rl);
      store_gradient(a, it.m0 + k, lane, gv, he, first, last);
    }
  }
}

// MODE 0: logL; 1: logL and gradient (with the leapfrog kick when p_half
// is set); 2: birth / death changes. Under a bridge (fd_bridge) the target
// is (1 - beta) logL_partner + beta logL_own, so each particle runs on both
// data sets.
template <int MODE, int NR, bool BRIDGE>
__device__ __forceinline__ void fd_run(const PopArgs& a, const FdTables& tabs, const FdItem& it,
                                       int lane, const double* __restrict__ src, double* rl) {
  const double b = a.beta ? a.beta[it.i] : 1.0;
  if constexpr (BRIDGE) {
    fd_particle<MODE, NR>(a, partner_side(a, tabs, lane), it, lane, 1.0 - b, true, false, src, rl);
    fd_particle<MODE, NR>(a, own_side(a, tabs, lane), it, lane, b, false, true, src, rl);
  } else {
    fd_particle<MODE, NR>(a, own_side(a, tabs, lane), it, lane, b, true, true, src, rl);
  }
}

// Waves per SIMD the kernel is compiled for. The gradient's LDS (a residual copy
// per wave) holds four; the likelihood alone gains from more (128 bins, 40000
// particles, K on 0..10: 168 us at four, 159 at five, 154 at six), and more
// waves still would leave few particles' latency exposed (eight: 41 us for 1000
// particles, K on 0..16, against 35 at six and 33 at four). 0: the compiler's
// choice, for two records (held to four the schedule loses more than a wave gains:
// gradient of 1441 particles, K on 0..26, 151 us at four, 126 left alone;
// birth/death over 200 bins 111, 98; 40000, K on 1..10: gradient 598, 553).
template <int MODE, int NR, bool BRIDGE>
constexpr int fd_occupancy() {
  return BRIDGE ? 0 : (MODE == 0 && NR == 2 ? 6 : 4);
}

// One particle per wave; the hardware hands the workgroups out in the K-sorted
// order. (BRIDGE apart: the two sides' constants together spill.)
template <int MODE, int NR, bool BRIDGE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    fd_occupancy<MODE, NR, BRIDGE>() ? fd_occupancy<MODE, NR, BRIDGE>() : 1,
    fd_occupancy<MODE, NR, BRIDGE>() ? fd_occupancy<MODE, NR, BRIDGE>() : 8))) void fd_kernel(PopArgs a, const double* __restrict__ src) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  FdTables tabs;
  FdItem it;
  const int64_t rank = (int64_t)blockIdx.x * waves + wave;
  const bool work = rank < fd_count(a) && fd_active_at(a, rank, it);
  // a workgroup without an active particle leaves at once
  if (!__syncthreads_or(work)) return;
  double* rl = stage_tables(tabs, a.fd_table, BRIDGE ? a.fd2_table : nullptr) + wave * resid_words<NR>();
  if (work) fd_run<MODE, NR, BRIDGE>(a, tabs, it, lane, src, rl);
}

// Few particles: a workgroup of four waves per particle, the sources shared out.
// Waves take the window spectra of four sources at a time; each then subtracts
// them, in source order, from its quarter of the band (channel, real or
// imaginary part); the adjoint, or the two candidates' overlaps, go wave by
// wave again. Every value is formed by the operations of fd_kernel in their
// order. A wave's serial pass over its sources is what few particles wait for:
// 300 particles, K on 0..10: gradient 33 -> 20 us, likelihood 23 -> 16,
// birth/death 25 -> 18.
template <int MODE, int NR>
__device__ __forceinline__ void fd_split_side(const PopArgs& a, const FdSide& sd, const FdItem& it, int lane,
                                              int wave, double w, bool first, bool last,
                                              const double* __restrict__ src, double* rl, double* spec) {
  constexpr int Bp = kNs * NR, rs = resid_row<NR>();
  const double wc = w * sd.cnorm;
  const double* row0 = src + (int64_t)__builtin_amdgcn_readfirstlane((int)it.m0) * kSrcWords;
  double q[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r)
    q[r] = sd.data[((wave >> 1) * kFdBandStride + lane + kNs * r) * 2 + (wave & 1)];
  for (int c0 = 0; c0 < it.K; c0 += 4) {
    const int n = it.K - c0 < 4 ? it.K - c0 : 4;
    if (c0) __syncthreads();  // the spectra have been read
    if (wave < n) {
      double re[2], im[2];
      window_spectrum(src_load(row0 + (c0 + wave) * kSrcWords, sd.qslot), sd.g, sd.tw, sd.trig, sd.scale,
                      lane, re, im);
      double* o = spec + wave * 4 * kNs + lane;
      o[0] = re[0];
      o[kNs] = im[0];
      o[2 * kNs] = re[1];
      o[3 * kNs] = im[1];
    }
    __syncthreads();
    for (int k = 0; k < n; ++k) {
      const int lo =
          window_start(__builtin_bit_cast(int64_t, row0[(c0 + k) * kSrcWords + sd.qslot]), sd);
      const double* o = spec + (k * 4 + wave) * kNs;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int b = lane + kNs * r, m = b - lo;
        const double f = ((unsigned)m < (unsigned)kNs && b < (int)sd.B) ? -1.0 : 0.0;
        q[r] = fma(f, o[bin_lane(m & (kNs - 1))], q[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) rl[wave * rs + lane + kNs * r] = q[r];
  if (lane == 0) rl[wave * rs + Bp] = 0.0;
  __syncthreads();
  if (MODE == 2 ? wave < 2 : wave == 3) {  // the whole residual
    Resid<NR> R;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        R.re[c][r] = rl[2 * c * rs + lane + kNs * r];
        R.im[c][r] = rl[(2 * c + 1) * rs + lane + kNs * r];
      }
    if constexpr (MODE == 2) {
      if (wave == 0) fd_birth<NR>(a, sd, it, lane, R, wc, first);
      else fd_death<NR>(a, sd, it, lane, R, wc, first, src);
    } else {
      const double ss = resid_square<NR>(R, lane);
      if (lane == 0 && a.logl) {
        const double v = -0.5 * wc * ss;
        a.logl[it.i] = first ? v : a.logl[it.i] + v;
      }
    }
  }
  if constexpr (MODE == 1) {
    const double he = a.p_half ? 0.5 * a.eps * (a.dir ? (double)a.dir[it.i] : 1.0) : 0.0;
    for (int k = wave; k < it.K; k += 4) {
      const double gv = fd_adjoint<NR>(sd, src_load(row0 + k * kSrcWords, sd.qslot), lane, wc, rl);
      store_gradient(a, it.m0 + k, lane, gv, he, first, last);
    }
  }
}

template <int MODE, int NR, bool BRIDGE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void fd_split_kernel(
    PopArgs a, const double* __restrict__ src) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  FdTables tabs;
  FdItem it;
  if (!((int64_t)blockIdx.x < fd_count(a) && fd_active_at(a, blockIdx.x, it))) return;
  double* rl = stage_tables(tabs, a.fd_table, BRIDGE ? a.fd2_table : nullptr);
  double* spec = rl + resid_words<NR>();
  const double b = a.beta ? a.beta[it.i] : 1.0;
  if constexpr (BRIDGE) {
    fd_split_side<MODE, NR>(a, partner_side(a, tabs, lane), it, lane, wave, 1.0 - b, true, false, src, rl, spec);
    __syncthreads();
    fd_split_side<MODE, NR>(a, own_side(a, tabs, lane), it, lane, wave, b, false, true, src, rl, spec);
  } else {
    fd_split_side<MODE, NR>(a, own_side(a, tabs, lane), it, lane, wave, b, true, true, src, rl, spec);
  }
}

// ---------------------------------------------------------------- NUTS trajectories
// A whole No-U-Turn transition: a wave takes a particle from the queue and runs
// its trajectory to the end, leaf by leaf, without a barrier. A trajectory is a
// chain of dependent gradients; most end after one doubling while a few of
// small K take fifty steps. In lockstep (a launch each for source rows, gradient
// and leaf over the particles still extending) the late leaves cost 20 to 37 us
// of launches for little work, and the host had to read after each doubling
// whether any were left. Here the long chains, taken first, overlap the short
// ones. Every value is formed by the operations of
// the lockstep steps (smcx_nuts.h) in their order. 24000 particles, K on 1..10,
// depth 6: 1210 us and six host reads in lockstep, 456 here, 250 to 330 of them the
// longest trajectories' latency.
//
// One workgroup of traj_waves waves per compute unit: two waves per SIMD hide
// most of each other's latency, and more would not fit the LDS. (A workgroup
// of four waves per particle, sharing its sources, took 714 us: most leaves
// have fewer sources than waves, and three waves wait for the leaf step.)
//
// A particle of at most kResK sources, one coordinate per lane, keeps its
// frontier on chip from leaf to leaf: through global memory (the general form,
// the steps of smcx_nuts.h) a leaf waits for one dependent round trip after
// another, 16000 of its 28000 cycles. The ends of the trajectory and the
// subtree's proposal, which a leaf does not read, stay in the state vectors;
// the trajectory's proposal is written to the caller's arrays at once.
constexpr int kResK = 8;
constexpr int kResCk = 3;     // checkpoint levels in LDS
constexpr int kWPitch = 9;    // words per row of W in LDS
constexpr int kTrajRows = 16;  // source rows in LDS at a time, general form
template <int NR>
struct TrajLds {              // of one wave
  double rl[resid_words<NR>()];
  double q[64], h[64], g[64];
  double ck[kResCk][2][64];
  double rows[kResK * kSrcWords];
  double w[64 * kWPitch];     // the general form's further rows
};
static_assert(kResK * kSrcWords + 64 * kWPitch >= kTrajRows * kSrcWords, "rows of the general form");
static_assert(sizeof(TrajLds<2>::q) + sizeof(TrajLds<2>::h) >= 8 * kNutsMetricMax, "vector of the general form");
template <int NR>
constexpr int traj_waves() { return NR == 2 ? 8 : 6; }

struct TrajArgs {
  PopArgs a;
  NutsArgs na;
  int* queue;
};

// The kernel's arguments, read again from the kernarg segment by each phase:
// held across phases they would spill by the hundred. The lane index goes
// through opaque_lane for the same reason (table addresses derived from it).
__device__ __forceinline__ TrajArgs traj_args() {
#ifdef __HIP_DEVICE_COMPILE__  // (the host pass has no address spaces to convert between)
  using Arg = const __attribute__((address_space(4))) TrajArgs;
  Arg* p = (Arg*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *p;
#else
  return TrajArgs();
#endif
}
__device__ __forceinline__ int opaque_lane(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

// v of lane 4 (lane / 4) + T.
template <int T>
__device__ __forceinline__ double quad_lane(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  return join_words((unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, 0x55 * T, 0xF, 0xF, true),
                    (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), 0x55 * T, 0xF, 0xF, true));
}

// The rows of n <= kTrajRows sources with parameters th[n][8] into LDS, four
// lanes per source, each with one of the four angles.
__device__ __forceinline__ void traj_rows(const double* th, int n, int lane, double* rows) {
  static_assert(4 * kTrajRows <= 64, "lanes of the rows");
  if (lane < 4 * n) {  // whole quads
    const TrajArgs z = traj_args();
    const int t = lane & 3;
    const double* c = th + (lane >> 2) * 8;
    double sn, cs;
    sincos(t == 2 ? 2.0 * c[5] : c[t == 3 ? 6 : 3 + t], &sn, &cs);
    const Src s = make_src_from(c, z.a.fd_T_obs, quad_lane<0>(sn), quad_lane<0>(cs), quad_lane<1>(sn),
                                quad_lane<1>(cs), quad_lane<2>(sn), quad_lane<2>(cs), quad_lane<3>(sn),
                                quad_lane<3>(cs));
    if (t == 0) {
      double* w = rows + (lane >> 2) * kSrcWords;
      src_store(w, s);
      w[kQPartner] =
          z.a.fd_bridge ? __builtin_bit_cast(double, (int64_t)floor(s.f0 * z.a.fd2_T_obs)) : w[kQOwn];
    }
  }
  wave_lds_sync();
}

// Likelihood (returned, added to logl) and gradient of the particle on one
// data set, as fd_particle<1>: RES with the rows in LDS and the gradient into L.g,
// else with the rows made here, kTrajRows at a time, and the gradient into
// global memory with the closing kick.
template <int NR, bool RES>
__device__ __forceinline__ double traj_side(const FdTables& tabs, const FdItem& it, int lane, double w,
                                            bool partner, bool first, bool last, double logl,
                                            TrajLds<NR>& L) {
  const TrajArgs z = traj_args();
  const auto side = [&](int ln) { return partner ? partner_side(z.a, tabs, ln) : own_side(z.a, tabs, ln); };
  constexpr int kRows = RES ? kResK : kTrajRows;
  const double* th = z.a.theta + it.m0 * 8;
  const double wc = w * side(lane).cnorm;
  Resid<NR> R;
  load_resid<NR>(side(lane), lane, R);
  for (int c0 = 0; c0 < it.K; c0 += kRows) {
    const int n = it.K - c0 < kRows ? it.K - c0 : kRows;
    if (!RES) traj_rows(th + c0 * 8, n, lane, L.rows);
    for (int k = 0; k < n; ++k) {
      const int ln = opaque_lane(lane);
      const FdSide sd = side(ln);
      subtract_source<NR>(sd, src_load(L.rows + k * kSrcWords, sd.qslot), sd.g, ln, R, 1.0);
    }
  }
  const double ss = resid_square<NR>(R, lane);
  const double v = -0.5 * wc * ss;
  logl = first ? v : logl + v;
  stage_resid<NR>(R, lane, L.rl);
  const double he = !RES && z.a.p_half ? 0.5 * z.a.eps * (double)z.a.dir[it.i] : 0.0;
  for (int c0 = 0; c0 < it.K; c0 += kRows) {
    const int n = it.K - c0 < kRows ? it.K - c0 : kRows;
    if (!RES && it.K > kRows) traj_rows(th + c0 * 8, n, lane, L.rows);
    for (int k = 0; k < n; ++k) {
      const int ln = opaque_lane(lane);
      const FdSide sd = side(ln);
      const double gv = fd_adjoint<NR>(sd, src_load(L.rows + k * kSrcWords, sd.qslot), ln, wc, L.rl);
      if constexpr (RES) {
        double* g = L.g + k * 8 + (ln >> 3);
        if ((ln & 7) == 7) *g = first ? gv : gv + *g;
      } else {
        store_gradient(z.a, it.m0 + c0 + k, ln, gv, he, first, last);
      }
    }
  }
  wave_lds_sync();
  return logl;
}

template <int NR, bool RES>
__device__ __forceinline__ double traj_gradient(const FdTables& tabs, const FdItem& it, int lane,
                                                TrajLds<NR>& L) {
  const TrajArgs z = traj_args();
  const double b = z.a.beta ? z.a.beta[it.i] : 1.0;
  double logl = 0.0;
  if (RES) traj_rows(L.q, it.K, opaque_lane(lane), L.rows);
  for (int side = z.a.fd_bridge ? 0 : 1; side < 2; ++side)
    logl = traj_side<NR, RES>(tabs, it, opaque_lane(lane), side ? b : 1.0 - b, !side,
                              !side || !z.a.fd_bridge, side != 0, logl, L);
  return logl;
}

// y[0] = (W x)_c, or (W^T x)_c, at c = lane < n, as nuts::wmul.
template <int NR, bool TRANS>
__device__ __forceinline__ double resident_mul(const NutsArgs& a, const nuts::View& v, const TrajLds<NR>& L,
                                               const double* x, int n) {
  double s = 0.0;
  if (v.lane < n) {
    if (a.w_blocks) {
      const int r = v.lane & 7, b = v.lane - r;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        s = fma(TRANS ? L.w[(b + k) * kWPitch + r] : L.w[v.lane * kWPitch + k], x[b + k], s);
    } else {
      double y[2];
      nuts::wmul<TRANS>(nuts::wblock(a, v), n, 0, x, v.lane, y);
      s = y[0];
    }
  }
  return s;
}

// The transition of a particle of at most kResK sources (nuts::init_step, the
// leaves and merges, nuts::finalize_step), a coordinate per lane.
template <int NR>
__device__ __forceinline__ void resident_trajectory(const FdTables& tabs, const FdItem& it, int lane,
                                                    TrajLds<NR>& L) {
#pragma clang fp contract(off)
  const int n = it.K * 8;
  const bool in = lane < n;
  const int64_t x = it.m0 * 8 + lane, i = it.i;
  nuts::View v;
  v.lane = lane;
  v.i = i;
  v.x0 = it.m0 * 8;
  v.x1 = v.x0 + n;
  v.K = it.K;
  v.ok = true;
  double q = 0.0, p = 0.0, g = 0.0, wg, lo = -INFINITY, hi = INFINITY;
  double H0, lw_tree, lw_sub = -INFINITY, logl_prop, logl_sub, e;
  int d;
  bool move = true, bad_w = false, box;
  {
    const NutsArgs a = traj_args().na;
    if (in) {
      q = a.q[x];
      p = a.momentum[x];
      g = a.grad[x];
    }
    logl_prop = a.logl[i];
    d = a.dirs[i * a.D];
    box = a.prior_lo != nullptr;
    if (box) {
      lo = a.prior_lo[lane & 7];
      hi = a.prior_hi[lane & 7];
    }
    if (a.w_blocks) {
      const double* W = nuts::wblock(a, v);
#pragma unroll
      for (int u = 0; u < kResK; ++u) {
        const int c = lane + 64 * u;
        if (u < it.K) L.w[(c >> 3) * kWPitch + (c & 7)] = W[c];
      }
    } else if (a.wmat) {
      const int64_t w0 = a.w_off[i], w1 = a.w_off[i + 1];
      bad_w = w1 - w0 != (int64_t)n * n || w0 < 0 || w1 > a.w_size;
      if (bad_w && lane == 0) atomicOr(a.flag, kFlagOffsets);
    }
    if (bad_w || (a.mask && !a.mask[i])) {
      if (bad_w && lane == 0 && a.status_out) a.status_out[i] = -1;
      move = false;
    }
  }
  logl_sub = logl_prop;
  L.g[lane] = g;
  wave_lds_sync();
  {
    const double pp = wave_sum(p * p, lane);
    const bool out = __any(in && box && !(q >= lo && q <= hi));
    H0 = -logl_prop + 0.5 * pp;
    lw_tree = -H0;
    if (move && !(!out && (H0 == H0) && fabs(H0) < INFINITY)) {
      const NutsArgs a = traj_args().na;
      if (lane == 0 && a.status_out) a.status_out[i] = 2;
      move = false;
    }
  }
  if (!move) return;

  const auto times_w = [&]() {  // W g of the gradient in L.g (g itself without a metric)
    const NutsArgs a = traj_args().na;
    return a.wmat ? resident_mul<NR, false>(a, v, L, L.g, n) : g;
  };
  // h = p + (e/2) W g, q += e W^T h
  const auto drift = [&]() {
    const NutsArgs a = traj_args().na;
    const double h = fma(0.5 * e, wg, p);
    L.h[lane] = h;
    wave_lds_sync();
    q = fma(e, a.wmat ? resident_mul<NR, true>(a, v, L, L.h, n) : h, q);
    L.q[lane] = q;
    wave_lds_sync();
  };
  e = traj_args().na.eps * (double)d;
  wg = times_w();
  drift();

  int steps = 0, status = 4, depth = 0;
  while (status == 4) {  // doubling at depth j
    const int j = depth;
    double rs = 0.0, ut, u64;
    int dn;
    bool take = false;
    {
      const NutsArgs a = traj_args().na;
      ut = a.u_tree[i * a.D + j];
      dn = j + 1 < a.D ? a.dirs[i * a.D + j + 1] : 1;
    }
    for (int m0 = 0; m0 < (1 << j) && status == 4; ++m0) {  // leaf m0
      const bool end = m0 == (1 << j) - 1;
      if ((m0 & 63) == 0) {  // the next 64 leaves' uniforms, one per lane
        const NutsArgs a = traj_args().na;
        u64 = m0 + lane < (1 << j) ? a.u_leaf[i * ((1ll << a.D) - 1) + ((1ll << j) - 1) + m0 + lane] : 0.0;
      }
      const double lf = traj_gradient<NR, true>(tabs, it, lane, L);
      g = in ? L.g[lane] : 0.0;
      wg = times_w();
      p = in ? fma(0.5 * e, wg, L.h[lane]) : 0.0;
      const double pp = wave_sum(p * p, lane);
      const bool out = __any(in && box && !(q >= lo && q <= hi));
      const double H = out ? INFINITY : -lf + 0.5 * pp;
      ++steps;
      if (!(H - H0 <= 1000.0)) {  // divergence (also NaN)
        status = 2;
        break;
      }
      const double lw = -H;
      const double lws = nuts::logaddexp(lw_sub, lw);
      take = __shfl(u64, m0 & 63) < exp(lw - lws);
      lw_sub = lws;
      logl_sub = take ? lf : logl_sub;
      const double before = rs;
      rs = before + p;
      const NutsArgs a = traj_args().na;
      if (in && take && !end) {
        nuts::slot(a, nuts::qS)[x] = q;
        nuts::slot(a, nuts::gS)[x] = g;
      }
      // checkpoints of the blocks of 2^m leaves that start here, and the
      // U-turn tests of those that end here
      for (int m = 1; m <= j && (m0 & ((1 << m) - 1)) == 0; ++m) {
        if (m <= kResCk) {
          L.ck[m - 1][0][lane] = p;
          L.ck[m - 1][1][lane] = before;
        } else if (in) {
          nuts::slot(a, nuts::kFirstCk + (m - 1))[x] = p;
          nuts::slot(a, nuts::kFirstCk + a.D + (m - 1))[x] = before;
        }
      }
      for (int m = 1; m <= j && ((m0 + 1) & ((1 << m) - 1)) == 0; ++m) {
        double ckp = 0.0, ckr = 0.0;
        if (m <= kResCk) {
          ckp = L.ck[m - 1][0][lane];
          ckr = L.ck[m - 1][1][lane];
        } else if (in) {
          ckp = nuts::slot(a, nuts::kFirstCk + (m - 1))[x];
          ckr = nuts::slot(a, nuts::kFirstCk + a.D + (m - 1))[x];
        }
        const double rb = rs - ckr;
        const double dl = wave_sum(rb * ckp, lane), dr = wave_sum(rb * p, lane);
        if (dl <= 0.0 || dr <= 0.0) {
          status = 1;
          break;
        }
      }
      if (status == 4 && !end) drift();
    }
    if (status != 4) break;
    // merge the subtree into the trajectory
    const NutsArgs a = traj_args().na;
    const int e0 = d > 0 ? nuts::qR : nuts::qL, e1 = d > 0 ? nuts::qL : nuts::qR;  // this end, the other
    // the other end: the start point in the first doubling
    double oq = 0.0, op = 0.0, og = 0.0, rt = 0.0, sq = q, sg = g;
    if (in) {
      oq = j ? nuts::slot(a, e1)[x] : a.q[x];
      op = j ? nuts::slot(a, e1 + 1)[x] : a.momentum[x];
      og = j ? nuts::slot(a, e1 + 2)[x] : a.grad[x];
      rt = j ? nuts::slot(a, nuts::rhoT)[x] : op;
      if (!take) {
        sq = nuts::slot(a, nuts::qS)[x];
        sg = nuts::slot(a, nuts::gS)[x];
      }
    }
    const bool take_tree = ut < exp(lw_sub - lw_tree);
    lw_tree = nuts::logaddexp(lw_tree, lw_sub);
    if (take_tree) logl_prop = logl_sub;
    rt = rt + rs;
    const double da = wave_sum(rt * op, lane), db = wave_sum(rt * p, lane);
    ++depth;
    if (da <= 0.0 || db <= 0.0) status = 1;
    else if (depth == a.D) status = 3;
    if (in && take_tree) {
      a.q[x] = sq;
      a.grad[x] = sg;
    }
    if (status != 4) break;
    if (in) {
      nuts::slot(a, nuts::rhoT)[x] = rt;
      nuts::slot(a, e0)[x] = q;
      nuts::slot(a, e0 + 1)[x] = p;
      nuts::slot(a, e0 + 2)[x] = g;
      if (j == 0) {
        nuts::slot(a, e1)[x] = oq;
        nuts::slot(a, e1 + 1)[x] = op;
        nuts::slot(a, e1 + 2)[x] = og;
      }
    }
    lw_sub = -INFINITY;
    if ((dn > 0) != (d > 0)) {  // the next doubling goes on from the other end
      q = oq;
      p = op;
      g = og;
      L.g[lane] = g;
      wave_lds_sync();
      wg = times_w();
    }
    d = dn;
    e = a.eps * (double)dn;
    drift();
  }
  const NutsArgs a = traj_args().na;
  if (lane == 0) {
    a.logl[i] = logl_prop;
    if (a.depth_out) a.depth_out[i] = depth;
    if (a.steps_out) a.steps_out[i] = steps;
    if (a.status_out) a.status_out[i] = status;
  }
}

// The transition of any particle, its state in global memory.
template <int NR>
__device__ __forceinline__ void general_trajectory(const FdTables& tabs, const FdItem& it, int lane,
                                                   TrajLds<NR>& L) {
  nuts::View v;
  v.lane = lane;
  v.i = it.i;
  v.x0 = it.m0 * 8;
  v.x1 = v.x0 + it.K * 8;
  v.K = it.K;
  v.ok = true;
  bool on = nuts::init_step(traj_args().na, v, L.q);
  for (int j = 0; on; ++j) {
    for (int n = 0; n < (1 << j) && on; ++n) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // the drift, for the rows' lanes
      const double lf = traj_gradient<NR, false>(tabs, it, lane, L);
      const NutsArgs a = traj_args().na;
      a.logl_front[v.i] = lf;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // the gradient, for its coordinates' lanes
      on = nuts::leaf_step(a, v, j, n, L.q);
      if (on && n == (1 << j) - 1) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // lane 0's state
        on = nuts::merge_step(a, v, j, L.q);
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  nuts::finalize_step(traj_args().na, v);
}

template <int NR>
__global__ __launch_bounds__(64 * traj_waves<NR>(), 1) void fd_trajectory_kernel(TrajArgs t) {
  const int lane = threadIdx.x & 63;
  FdTables tabs;
  double* lds = stage_tables(tabs, t.a.fd_table, t.a.fd_bridge ? t.a.fd2_table : nullptr);
  TrajLds<NR>& L = ((TrajLds<NR>*)lds)[__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))];
  for (;;) {
    const TrajArgs z = traj_args();
    const int cnt = (int)(z.a.order ? z.a.n_ranks : z.a.N);
    int r = 0;
    if (lane == 0) r = atomicAdd(z.queue, 1);
    r = __builtin_amdgcn_readfirstlane(r);
    if (r >= cnt) return;
    FdItem it;
    // with a mass matrix smallest K first (the order's last rank), whose trees run
    // deepest; without one nearly all run to the end, and the largest K takes
    // longest (3000 particles, K on 10..40, depth 6, 58 steps on average: 13.8 ms
    // smallest first, 9.5 largest first; 40000, K on 1..10: 27.2, 26.1)
    if (!fd_item_at(z.a, z.na.wmat ? cnt - 1 - r : r, it) || it.K == 0) continue;
    it.i = __builtin_amdgcn_readfirstlane((int)it.i);  // particles and rows are below 2^31
    it.m0 = __builtin_amdgcn_readfirstlane((int)it.m0);
    it.K = __builtin_amdgcn_readfirstlane(it.K);
    if (it.K <= kResK)
      resident_trajectory<NR>(tabs, it, lane, L);
    else
      general_trajectory<NR>(tabs, it, lane, L);
  }
}

// The outputs of the particles without a trajectory (no components, or
// invalid: status -1) and of those that do not move, and the queue's start.
// Offsets that do not span [0, M] make every particle invalid, as in the
// ordering pass, which lists none then.
__global__ __launch_bounds__(256) void fd_settle_kernel(NutsArgs a, int* queue) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0) *queue = 0;
  if (i >= a.N) return;
  const int64_t o0 = a.offsets[i], o1 = a.offsets[i + 1];
  const bool span = a.offsets[0] == 0 && a.offsets[a.N] == a.M;
  const bool ok = span && o0 >= 0 && o1 >= o0 && o1 <= a.M;
  const bool bad_k = ok && o1 - o0 > a.k_max;
  if (bad_k) atomicOr(a.flag, kFlagKMax);
  if (a.depth_out) a.depth_out[i] = 0;
  if (a.steps_out) a.steps_out[i] = 0;
  if (a.status_out) a.status_out[i] = !ok || bad_k ? -1 : 0;
}

// Per-source Gauss-Newton metric: block k of particle i is
//   beta (4 / (T_obs S)) Re sum_c sum_m conj(dh_c / dtheta_a) dh_c / dtheta_b
// over the source's 64-bin window, which by Parseval's identity for the
// 64-point DFT equals beta (4 / (T_obs S)) (T_obs / 64)^2 64 Re sum_c sum_j
// conj(dz_c,a(t_j)) dz_c,b(t_j) = (1/4) Re sum_c sum_j conj(g_c,a) g_c,b (the
// phase drops out, see amp_phase_derivs); blocks between sources are zero.
// One wave per particle; 36 sums per source.
// blocks: F is [M][8][8], block k of particle i at F + (o0 + k) 64 (nothing
// between blocks is written); otherwise the dense n x n block at F + f_off[i].
// Held to 168 VGPRs (it needs 171 unconstrained; the excess goes to SGPR
// spills into VGPR lanes, no scratch), which gives three waves per SIMD.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void fd_metric_kernel(PopArgs a, const double* __restrict__ src,
                                                        const int64_t* f_off, int64_t f_size, double* F,
                                                        int blocks) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  FdTables tabs;
  stage_tables(tabs, a.fd_table, a.fd_bridge ? a.fd2_table : nullptr);
  if (i >= a.N) return;
  const int64_t o0 = a.offsets[i], o1 = a.offsets[i + 1];
  if (!(o0 >= 0 && o1 >= o0 && o1 <= a.M && o1 - o0 <= a.k_max)) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  const int K = (int)(o1 - o0), n = 8 * K;
  const int64_t fo = blocks ? o0 * 64 : f_off[i];
  if (!blocks && (f_off[i + 1] - fo != (int64_t)n * n || fo < 0 || fo + (int64_t)n * n > f_size)) {
    if (lane == 0) atomicOr(a.flag, kFlagOffsets);
    return;
  }
  if (n == 0) return;
  double* Fi = F + fo;
  if (a.active && !a.active[i]) {
    // not selected: zero blocks, which the factor's ridge makes definite
    const int64_t cnt = blocks ? (int64_t)K * 64 : (int64_t)n * n;
    for (int64_t x = lane; x < cnt; x += 64) Fi[x] = 0.0;
    return;
  }
  if (!blocks)
    for (int64_t x = lane; x < (int64_t)n * n; x += 64) {
      const int r = (int)(x / n), c = (int)(x % n);
      if ((r >> 3) != (c >> 3)) Fi[x] = 0.0;
    }
  const double b = a.beta ? a.beta[i] : 1.0;
  const int ra = lane >> 3, rb = lane & 7;  // the block entry this lane writes
  const int lo = ra < rb ? ra : rb, hi = ra < rb ? rb : ra;
  // the lane holding entry (lo, hi) of the upper triangle after the sums
  const int holder = kSlot36[lo * 8 - lo * (lo - 1) / 2 + (hi - lo)];
  for (int side = a.fd_bridge ? 0 : 1; side < 2; ++side) {
  const FdSide sd = side == 0 ? partner_side(a, tabs, lane) : own_side(a, tabs, lane);
  const double gs = (side == 0 ? 1.0 - b : b) * sd.cnorm * sd.scale * sd.scale * kNs * 0.25;
  const bool first = side == 0 || !a.fd_bridge;
  const LaneGeom g = sd.g;
  for (int k = 0; k < K; ++k) {
    const int row = __builtin_amdgcn_readfirstlane((int)(o0 + k));
    const Src s = src_load(src + (int64_t)row * kSrcWords, sd.qslot);
    const Env e = envelope_amp(s, g);
    double acc[36];
#pragma unroll
    for (int x = 0; x < 36; ++x) acc[x] = 0.0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      double gr[8], gi[8];
      amp_phase_derivs(s, g, e, c, gr, gi);
      int x = 0;
#pragma unroll
      for (int p = 0; p < 8; ++p)
#pragma unroll
        for (int q = p; q < 8; ++q, ++x) acc[x] = fma(gr[p], gr[q], fma(gi[p], gi[q], acc[x]));
    }
    const double v = __shfl(transposed_sum36(acc, lane), holder);
    double* dst = blocks ? Fi + 64 * k + 8 * ra + rb : Fi + (int64_t)(8 * k + ra) * n + 8 * k + rb;
    *dst = first ? gs * v : *dst + gs * v;
  }
  }
}

// The band spectrum of K sources (out [2][B][2]): one wave.
__global__ __launch_bounds__(64) void fd_spectrum_kernel(PopArgs a, int64_t K, double* out) {
  const int lane = threadIdx.x;
  FdTables tabs;
  stage_tables(tabs, a.fd_table, nullptr);
  const FdSide sd = own_side(a, tabs, lane);
  Resid<4> R;
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) R.re[c][r] = R.im[c][r] = 0.0;
  for (int64_t k = 0; k < K; ++k) {
    const Src s = make_src(a.theta + k * 8, a.fd_T_obs);
    subtract_source<4>(sd, s, sd.g, lane, R, -1.0);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t b = lane + kNs * r;
      if (b < a.fd_B) {
        out[(c * a.fd_B + b) * 2] = R.re[c][r];
        out[(c * a.fd_B + b) * 2 + 1] = R.im[c][r];
      }
    }
}

// The source rows of all of theta, one lane per row, by workgroup `block`: a
// launch without a mask works on (nearly) all of them, and a lane per row
// keeps every lane busy where a group of lanes per particle (below) leaves two
// thirds idle at K = 5.5. Rows go out through LDS in two halves, so that a store
// covers consecutive words. The rows share the ordering pass's launch, which
// reads nothing of them. Bound by the 368 bytes written per row: 40000
// particles, K on 1..10, 81 MB: 29 + 6 us -> 25, of which 16 at the rate of a copy.
__device__ __forceinline__ void fd_src_rows(int64_t block, const double* theta, int64_t M, double T1,
                                            double T2, double* out) {
  constexpr int kHalf = kSrcWords / 2;  // odd: rows start in different banks
  __shared__ double stage[4][64 * kHalf];
  const int lane = threadIdx.x & 63;
  double* st = stage[threadIdx.x >> 6];
  const int64_t m0 = block * 256 + (threadIdx.x & ~63);
  const int rows = (int)min(M - m0, (int64_t)64);
  if (rows <= 0) return;
  double w[kSrcWords];
  if (lane < rows) {
    const Src s = make_src(theta + (m0 + lane) * 8, T1);
    src_store(w, s);
    w[kQPartner] = T2 > 0.0 ? __builtin_bit_cast(double, (int64_t)floor(s.f0 * T2)) : w[kQOwn];
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (lane < rows) {
#pragma unroll
      for (int x = 0; x < kHalf; ++x) st[lane * kHalf + x] = w[h * kHalf + x];
    }
    wave_lds_sync();
    for (int x = lane; x < rows * kHalf; x += 64) {
      const int r = x / kHalf, c = x - r * kHalf;
      out[(m0 + r) * kSrcWords + h * kHalf + c] = st[x];
    }
    wave_lds_sync();
  }
}

template <bool DEATH>
__global__ __launch_bounds__(kPrepBlock) void fd_prep_kernel(PrepArgs p, int64_t S, const double* theta,
                                                             double T1, double T2, double* out) {
  static_assert(kPrepBlock == 256, "source rows per workgroup");
  if (blockIdx.x < S)
    prep_block<DEATH>(p, S);
  else
    fd_src_rows(blockIdx.x - S, theta, p.M, T1, T2, out);
}

// The source rows of the particles the following launch works on (the same
// work items and activity mask): constants with the carrier bins of both
// records (T2 = 0: no partner, word 33 repeats word 32). A group of
// kSrcGroup lanes per particle, one lane per source, four particles to a
// wave: a whole wave per particle left most lanes idle at K <= 10, and one
// thread per particle measured slower in late NUTS leaves, where few
// particles are active. The cost follows the active set.
constexpr int kSrcGroup = 16;

__global__ __launch_bounds__(256) void fd_src_kernel(PopArgs a, double T2) {
  // The rows of a group's particle are contiguous ([K][46] doubles): each
  // lane builds its source's row in registers, and the group writes the
  // rows out through LDS in two halves of 23 words, so that a store of the
  // group covers 128 consecutive bytes instead of one word of each of 16
  // rows. The group's lanes are in one wave, whose LDS accesses complete in
  // order.
  constexpr int kHalf = kSrcWords / 2;
  __shared__ double stage[256 / kSrcGroup][kSrcGroup][kHalf];
  const int sub = threadIdx.x & (kSrcGroup - 1);
  double(*st)[kHalf] = stage[threadIdx.x / kSrcGroup];
  const int64_t n = fd_count(a);
  const int64_t stride = (int64_t)gridDim.x * (blockDim.x / kSrcGroup);
  for (int64_t rank = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kSrcGroup; rank < n;
       rank += stride) {
    FdItem it;
    if (!fd_active_at(a, rank, it)) continue;
    for (int c0 = 0; c0 < it.K; c0 += kSrcGroup) {
      const int rows = it.K - c0 < kSrcGroup ? it.K - c0 : kSrcGroup;
      double w[kSrcWords];
      if (sub < rows) {
        const Src s = make_src(a.theta + (it.m0 + c0 + sub) * 8, a.fd_T_obs);
        src_store(w, s);
        w[kQPartner] = T2 > 0.0 ? __builtin_bit_cast(double, (int64_t)floor(s.f0 * T2)) : w[kQOwn];
      }
      double* out = a.fd_src + (it.m0 + c0) * kSrcWords;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (sub < rows) {
#pragma unroll
          for (int x = 0; x < kHalf; ++x) st[sub][x] = w[h * kHalf + x];
        }
        wave_lds_sync();
        for (int x = sub; x < rows * kHalf; x += kSrcGroup) {
          const int r = x / kHalf, c = x - r * kHalf;
          out[r * kSrcWords + h * kHalf + c] = st[r][c];
        }
        wave_lds_sync();
      }
    }
  }
}

hipError_t launch_src_pass(const PopArgs& a, hipStream_t st) {
  if (a.N == 0) return hipSuccess;
  constexpr int per = 256 / kSrcGroup;
  hipLaunchKernelGGL(fd_src_kernel, dim3((unsigned)((launch_ranks(a) + per - 1) / per)), dim3(256), 0, st, a,
                     a.fd_bridge ? a.fd2_T_obs : 0.0);
  return hipGetLastError();
}

// Whether a launch gives each particle a workgroup: up to one wave per SIMD (1000
// particles, K on 0..10: gradient 35 against 27 us, likelihood 24 / 21,
// birth/death 26 / 25; 2000: 38 / 44, 25 / 31, 28 / 41). Half of those workgroups are
// resident at once, and the second round costs more than it gives where no
// particle keeps a wave of its own much longer than the others do: all of about
// one K, up to six (1024 bridged particles, K = 1: gradient 17 against 28 us, birth/death
// 22 / 33; K = 5: 34 / 43, 30 / 42), for birth/death up to 16 (11: 42 / 52; 20, over more
// than 128 bins: 80 / 77), for the gradient over more than 128 bins up to three (4:
// 34 / 30 of 600); and of 800 or more, K of three at most.
template <int MODE>
bool fd_split(const PopArgs& a, bool nr2) {
  const int64_t n_cu = a.n_cu > 0 ? a.n_cu : 256;
  if (a.N <= 2 * n_cu || a.N > 4 * n_cu) return a.N <= 2 * n_cu;
  const int k_alike = MODE == 2 ? 16 : (MODE == 1 && !nr2 ? 3 : 6);
  const bool alike = 5 * a.M >= 4 * a.N * a.k_max && a.M <= k_alike * a.N;
  return !alike && (a.k_max > 3 || a.N <= 3 * n_cu);
}

template <int MODE>
hipError_t launch_fd_mode(const PopArgs& a, hipStream_t st) {
  if (a.N == 0) return hipSuccess;
  if (!a.fd_src_ready) {
    hipError_t e = launch_src_pass(a, st);
    if (e != hipSuccess) return e;
  }
  const dim3 block(256);
  const bool br = a.fd_bridge != 0;
  // two band bins per lane cover up to 128 bins; the wider of two bridged
  // bands decides
  const bool nr2 = a.fd_B <= 2 * kNs && !(br && a.fd2_B > 2 * kNs);
  // LDS bytes: the tables, and for the gradient a residual copy per wave
  const size_t lds2 = 8 * fd_lds_words(br, 4, MODE == 1 ? resid_words<2>() : 0);
  const size_t lds4 = 8 * fd_lds_words(br, 4, MODE == 1 ? resid_words<4>() : 0);
  if (fd_split<MODE>(a, nr2)) {
    const size_t s2 = 8 * fd_lds_words(br, 1, resid_words<2>() + 4 * 4 * kNs);
    const size_t s4 = 8 * fd_lds_words(br, 1, resid_words<4>() + 4 * 4 * kNs);
    const dim3 each((unsigned)launch_ranks(a));
    if (nr2 && br)
      hipLaunchKernelGGL((fd_split_kernel<MODE, 2, true>), each, block, s2, st, a, a.fd_src);
    else if (nr2)
      hipLaunchKernelGGL((fd_split_kernel<MODE, 2, false>), each, block, s2, st, a, a.fd_src);
    else if (br)
      hipLaunchKernelGGL((fd_split_kernel<MODE, 4, true>), each, block, s4, st, a, a.fd_src);
    else
      hipLaunchKernelGGL((fd_split_kernel<MODE, 4, false>), each, block, s4, st, a, a.fd_src);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((launch_ranks(a) + 3) / 4));
  if (nr2 && br)
    hipLaunchKernelGGL((fd_kernel<MODE, 2, true>), grid, block, lds2, st, a, a.fd_src);
  else if (nr2)
    hipLaunchKernelGGL((fd_kernel<MODE, 2, false>), grid, block, lds2, st, a, a.fd_src);
  else if (br)
    hipLaunchKernelGGL((fd_kernel<MODE, 4, true>), grid, block, lds4, st, a, a.fd_src);
  else
    hipLaunchKernelGGL((fd_kernel<MODE, 4, false>), grid, block, lds4, st, a, a.fd_src);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fd_src(const PopArgs& a, hipStream_t st) { return launch_src_pass(a, st); }

hipError_t launch_fd_prep(const PrepArgs& p, const PopArgs& a, hipStream_t st) {
  if (p.k_max + 1 > 4 * kPrepBlock) return hipErrorInvalidValue;
  const int64_t S = prep_slices(p.N);
  const dim3 grid((unsigned)(S + (p.M + 255) / 256)), block(kPrepBlock);
  const size_t lds = (size_t)(p.k_max + 1) * sizeof(int);
  const double T2 = a.fd_bridge ? a.fd2_T_obs : 0.0;
  if (p.dlogl_death && p.death_idx)
    hipLaunchKernelGGL(fd_prep_kernel<true>, grid, block, lds, st, p, S, a.theta, a.fd_T_obs, T2, a.fd_src);
  else
    hipLaunchKernelGGL(fd_prep_kernel<false>, grid, block, lds, st, p, S, a.theta, a.fd_T_obs, T2, a.fd_src);
  return hipGetLastError();
}

hipError_t launch_fd(int mode, const PopArgs& a, hipStream_t st) {
  if (a.fd_B < 1 || a.fd_B > 4 * kNs) return hipErrorInvalidValue;
  switch (mode) {
    case 0: return launch_fd_mode<0>(a, st);
    case 1: return launch_fd_mode<1>(a, st);
    case 2: return launch_fd_mode<2>(a, st);
    default: return hipErrorInvalidValue;
  }
}

template <int NR>
hipError_t launch_trajectories(const TrajArgs& t, hipStream_t st) {
  constexpr int nw = traj_waves<NR>();
  const int64_t n_cu = t.a.n_cu > 0 ? t.a.n_cu : 256;
  const dim3 grid((unsigned)std::min<int64_t>(t.a.N, n_cu));
  hipLaunchKernelGGL(fd_trajectory_kernel<NR>, grid, dim3(64 * nw),
                     8 * fd_lds_words(t.a.fd_bridge != 0, nw, sizeof(TrajLds<NR>) / 8), st, t);
  return hipGetLastError();
}

hipError_t launch_fd_trajectory(const PopArgs& a, const NutsArgs& na, int* queue, hipStream_t st) {
  if (a.fd_B < 1 || a.fd_B > 4 * kNs) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fd_settle_kernel, dim3((unsigned)((a.N + 255) / 256)), dim3(256), 0, st, na, queue);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool nr2 = a.fd_B <= 2 * kNs && !(a.fd_bridge && a.fd2_B > 2 * kNs);
  const TrajArgs t{a, na, queue};
  return nr2 ? launch_trajectories<2>(t, st) : launch_trajectories<4>(t, st);
}

hipError_t launch_fd_metric(const PopArgs& a, const int64_t* f_offsets, int64_t f_size, double* F,
                            int blocks, hipStream_t st) {
  if (a.N == 0) return hipSuccess;
  // the metric walks every particle in natural order (no ordering pass ran);
  // a.active (or nullptr) selects the particles it evaluates
  PopArgs all = a;
  all.order = nullptr;
  hipError_t e = launch_src_pass(all, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fd_metric_kernel, dim3((unsigned)((a.N + 3) / 4)), dim3(256),
                     8 * fd_lds_words(a.fd_bridge != 0, 4, 0), st, a, a.fd_src, f_offsets, f_size, F,
                     blocks);
  return hipGetLastError();
}

hipError_t launch_fd_spectrum(const PopArgs& a, int64_t K, double* out, hipStream_t st) {
  if (a.fd_B < 1 || a.fd_B > 4 * kNs) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fd_spectrum_kernel, dim3(1), dim3(64), 8 * fd_lds_words(false, 1, 0), st, a, K,
                     out);
  return hipGetLastError();
}

}  // namespace smcx
