// Batched No-U-Turn transition kernels (Sec. "No-U-Turn-Sampler") of the
// time-domain models.
//
// Every particle builds its own trajectory by repeated doubling; since a
// doubling at depth j always has 2^j leapfrog steps, all particles that are
// still extending sit at the same (depth, leaf) position and advance in
// lockstep, one batched gradient evaluation per leaf. A particle that stops
// (U-turn, divergence, maximum depth) simply drops out of the active mask,
// so trajectory lengths are ragged. (The frequency-domain model runs each
// trajectory on its own, in one launch of smcx_gblisa.hip.) The variant is
// multinomial NUTS:
//  * within a subtree, leaf n replaces the subtree proposal with probability
//    w_n / (sum of subtree weights so far), w = exp(-H);
//  * a completed subtree replaces the trajectory proposal with probability
//    min(1, W_subtree / W_trajectory);
//  * the generalised U-turn test on a segment with momentum sum rho and end
//    momenta p_a, p_b stops when rho.p_a <= 0 or rho.p_b <= 0; it is applied
//    to every balanced block of the subtree as the block completes, and to
//    the whole trajectory after each doubling;
//  * a leaf whose energy exceeds the initial one by more than 1000, or that
//    leaves the prior box, is a divergence and stops the trajectory;
//  * a subtree that turns or diverges is discarded.
// Random numbers are inputs: one direction per doubling, one uniform per
// leaf and one per doubling.
//
// With a mass matrix M = (W^T W)^{-1} (the section's Hessian metric, W the
// inverse Cholesky factor of the Gauss-Newton metric) the state carries the
// whitened momentum r = W p_M, drawn N(0, I): kicks add (e/2) W g, drifts add
// e W^T r, and the energy and U-turn test keep the identity form in r. The
// closing kick of a leapfrog step then needs the whole gradient of the
// particle, so it moves from the gradient pass's epilogue into the leaf
// kernel.
//
// One workgroup of one wave handles one particle at a time; lanes run over its K*P
// coordinates (at most two each when a metric is used).
#include "smcx_nuts.h"

#include <algorithm>

namespace smcx {
namespace {

using namespace nuts;

__global__ __launch_bounds__(64) void nuts_init_kernel(NutsArgs a) {
  __shared__ double sh[kNutsMetricMax];
  if (blockIdx.x == 0 && (int)threadIdx.x <= a.D) a.count[threadIdx.x] = 0;
  const View v = view_of(a);
  if (!v.ok) {
    if (v.i < a.N && v.lane == 0) {
      a.active[v.i] = 0;
      a.state[v.i].status = -1;
    }
    return;
  }
  init_step(a, v, sh);
}

// Leaf and merge, one workgroup of one wave per particle. (A loop around the
// step would keep about twice the registers live, 64 -> 127 VGPRs for the leaf.)
__global__ __launch_bounds__(64) void nuts_leaf_kernel(NutsArgs a, int j, int n) {
  __shared__ double sh[kNutsMetricMax];
  const View v = view_of(a);
  if (v.ok && a.active[v.i]) leaf_step(a, v, j, n, sh);
}

__global__ __launch_bounds__(64) void nuts_merge_kernel(NutsArgs a, int j) {
  __shared__ double sh[kNutsMetricMax];
  const View v = view_of(a);
  if (v.ok && a.active[v.i]) merge_step(a, v, j, sh);
}

__global__ __launch_bounds__(64) void nuts_finalize_kernel(NutsArgs a) {
  const View v = view_of(a);
  if (!v.ok) {
    if (v.i < a.N && v.lane == 0) {
      if (a.status_out) a.status_out[v.i] = -1;
      if (a.depth_out) a.depth_out[v.i] = 0;
      if (a.steps_out) a.steps_out[v.i] = 0;
    }
    return;
  }
  finalize_step(a, v);
}

dim3 grid_of(int64_t N) { return dim3((unsigned)N); }  // one wave-sized workgroup per particle

}  // namespace

hipError_t launch_nuts_init(const NutsArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(nuts_init_kernel, grid_of(a.N), dim3(64), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_nuts_leaf(const NutsArgs& a, int j, int n, hipStream_t st) {
  hipLaunchKernelGGL(nuts_leaf_kernel, grid_of(a.N), dim3(64), 0, st, a, j, n);
  return hipGetLastError();
}
hipError_t launch_nuts_merge(const NutsArgs& a, int j, hipStream_t st) {
  hipLaunchKernelGGL(nuts_merge_kernel, grid_of(a.N), dim3(64), 0, st, a, j);
  return hipGetLastError();
}
hipError_t launch_nuts_finalize(const NutsArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(nuts_finalize_kernel, grid_of(a.N), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace smcx
