// gfx950 kernels that evaluate arbitrary trajectories: cost and gradient,
// guidance steps, sphere centres.
#include <hip/hip_runtime.h>

#include "dsopt_eval.h"

namespace dsk {
namespace {

// Seed of this wavefront in k_cost / k_guide: W = 1, one seed per
// wavefront (WAVES_PER_BLOCK per workgroup); W > 1, one seed per workgroup
// of W wavefronts (a team, for batches too small to fill the chip; FULL: one
// of MAX_TEAM).
template <bool FULL>
__device__ __forceinline__ int seed_of(int W, float* team_lds, Team& tm) {
  tm.buf = 0;
  if (FULL || W > 1) {
    tm.W = W;
    tm.w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    tm.lds = team_lds;
    tm.kin = FULL ? team_lds + 2 * W * PART * WAVE : nullptr;
    return blockIdx.x;
  }
  tm.W = 1;
  tm.w = 0;
  tm.lds = nullptr;
  tm.kin = nullptr;
  return (blockIdx.x * BLOCK + threadIdx.x) / WAVE;
}

// Waypoint t of a trajectory (zeros past the horizon or the last seed).
// Called ahead of the staging, so its memory round trip overlaps theirs.
__device__ __forceinline__ void load_waypoint(const float* __restrict__ X, int seed, int S, int T,
                                              int t, float* x) {
  const bool in = seed < S && t < T;
#pragma unroll
  for (int j = 0; j < NJ; ++j) x[j] = in ? X[((size_t)seed * T + t) * NJ + j] : 0.f;
}

// The problem is a kernel argument of k_cost and k_guide: a table in device
// memory costs a copy ahead of the kernel and an event behind it.
// Objective (and gradient) of arbitrary trajectories: one wavefront (or a
// team) per seed group of G lanes (G = smallest of 16/32/64 holding T).
template <bool EXT, bool FULL>
__global__ void __launch_bounds__(MAX_TEAM * WAVE)
k_cost(const RobotDev* __restrict__ rb, const ParamsDev* __restrict__ pp, const ProbDev pb,
       const float* __restrict__ X, int S, int T, int G, const float* __restrict__ dJ,
       float* __restrict__ J_out, float* __restrict__ dX, int with_grad, int W) {
  extern __shared__ float s_team[];
  __shared__ __attribute__((aligned(16))) uint8_t s_cm[COARSE_BYTES];
  const int lane = threadIdx.x & (WAVE - 1);
  Team tm;
  const int seed = seed_of<FULL>(W, s_team, tm);
  const int t = lane & (G - 1);
  const bool owner = tm.w == 0 && lane < G;
  const bool active = t < T;
  float x[NJ];
  load_waypoint(X, seed, S, T, t, x);
  if (pp->skip) stage_coarse(pb.sc, lds(s_cm), threadIdx.x, blockDim.x);
  stage_robot(rb);
  if (seed >= S) return;   // whole wavefront (team: whole workgroup) past the end
  ParamsDev P = *pp;
  Sampler Sm = make_sampler(pb.sc, rb);
  Sm.cm = lds(s_cm);
  put_goal(pb);
  float J;
  if (with_grad) {
    EvalOut e = eval_any<EV_GRAD, EXT, FULL>(use_pipe(rb, tm, G), rb, P, Sm, x, t, T, G, active, tm);
    J = grp_sum(e.cost, G);
    float w = dJ ? dJ[seed] : 1.f;
    if (active && owner) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) dX[((size_t)seed * T + t) * NJ + j] = w * e.g[j];
    }
  } else {
    EvalOut e = eval_any<EV_COST, EXT, FULL>(use_pipe(rb, tm, G), rb, P, Sm, x, t, T, G, active, tm);
    J = grp_sum(e.cost, G);
  }
  if (J_out && tm.w == 0 && lane == 0) J_out[seed] = J;
}

// Guidance: n gradient steps x <- x - alpha * g on every trajectory, one
// wavefront (or a team) per seed (same evaluation as the optimiser).
template <bool EXT, bool FULL>
__global__ void __launch_bounds__(MAX_TEAM * WAVE)
k_guide(const RobotDev* __restrict__ rb, const ParamsDev* __restrict__ pp, const ProbDev pb,
        float* __restrict__ X, int S, int T, int G, float alpha, int n_steps,
        float* __restrict__ J_out, int W) {
  extern __shared__ float s_team[];
  __shared__ __attribute__((aligned(16))) uint8_t s_cm[COARSE_BYTES];
  const int lane = threadIdx.x & (WAVE - 1);
  Team tm;
  const int seed = seed_of<FULL>(W, s_team, tm);
  const int t = lane & (G - 1);
  const bool owner = tm.w == 0 && lane < G;
  const bool active = t < T;
  float x[NJ];
  load_waypoint(X, seed, S, T, t, x);
  if (pp->skip) stage_coarse(pb.sc, lds(s_cm), threadIdx.x, blockDim.x);
  stage_robot(rb);
  if (seed >= S) return;   // whole wavefront (team: whole workgroup) past the end
  ParamsDev P = *pp;
  Sampler Sm = make_sampler(pb.sc, rb);
  Sm.cm = lds(s_cm);
  put_goal(pb);
  const bool pipe = use_pipe(rb, tm, G);
  for (int k = 0; k < n_steps; ++k) {
    EvalOut e = eval_any<EV_GRAD, EXT, FULL>(pipe, rb, P, Sm, x, t, T, G, active, tm);
#pragma unroll
    for (int j = 0; j < NJ; ++j) x[j] -= alpha * e.g[j];
  }
  if (J_out) {
    EvalOut e = eval_any<EV_COST, EXT, FULL>(pipe, rb, P, Sm, x, t, T, G, active, tm);
    float J = grp_sum(e.cost, G);
    if (tm.w == 0 && lane == 0) J_out[seed] = J;
  }
  if (active && owner) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) X[((size_t)seed * T + t) * NJ + j] = x[j];
  }
}

// Sphere centres (parity dump), one thread per seed-waypoint.
__global__ void k_spheres(const RobotDev* __restrict__ rb, const float* __restrict__ X, int n,
                          float* __restrict__ out) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float q[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) q[j] = X[(size_t)i * NJ + j];
  float R[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
  float p[3] = {0.f, 0.f, 0.f};
  const int ns = rb->ns;
  for (int l = 0; l < NJ; ++l) {
    const float* F = rb->F[l];
    float A[9], pa[3];
    for (int r = 0; r < 3; ++r) {
      for (int c = 0; c < 3; ++c)
        A[3 * r + c] = R[3 * r] * F[c] + R[3 * r + 1] * F[4 + c] + R[3 * r + 2] * F[8 + c];
      pa[r] = R[3 * r] * F[3] + R[3 * r + 1] * F[7] + R[3 * r + 2] * F[11] + p[r];
    }
    float sn, cs;
    sincosf(q[l], &sn, &cs);
    for (int r = 0; r < 3; ++r) {
      float a0 = A[3 * r], a1 = A[3 * r + 1];
      R[3 * r] = cs * a0 + sn * a1;
      R[3 * r + 1] = cs * a1 - sn * a0;
      R[3 * r + 2] = A[3 * r + 2];
      p[r] = pa[r];
    }
    for (int s = rb->link_begin[l]; s < rb->link_begin[l + 1]; ++s) {
      float4 sp = rb->sph[s];
      float* o = out + ((size_t)i * ns + rb->perm[s]) * 3;
      o[0] = R[0] * sp.x + R[1] * sp.y + R[2] * sp.z + p[0];
      o[1] = R[3] * sp.x + R[4] * sp.y + R[5] * sp.z + p[1];
      o[2] = R[6] * sp.x + R[7] * sp.y + R[8] * sp.z + p[2];
    }
  }
}

}  // namespace

// Team size for k_cost / k_guide: wavefronts per seed, doubled while all the
// seeds' wavefronts are fewer than eight per CU (two per SIMD, which is what
// the registers allow), up to MAX_TEAM.  The last doubling may go past that:
// 257 to 511 seeds in teams of eight and 513 to 1023 in teams of four take two
// rounds (gradient of 48 waypoints, 60 spheres: 256 seeds 12.7 us, 257 18.4,
// 511 19.2, 512 14.3, 513 22.2, 1023 25.1, 1024 18.8, 2048 26.8).
static int cost_team(int S, int cu_count) {
  int W = 1;
  while (W < MAX_TEAM && (long long)S * W < (long long)2 * WAVES_PER_BLOCK * cu_count) W *= 2;
  return W;
}

hipError_t launch_cost(const RobotDev* rb, const ParamsDev* pp, const ProbDev& prob,
                       const float* X, int S, int T, const float* dJ, float* J_out, float* dX,
                       int with_grad, bool ext, int cu_count, hipStream_t s) {
  const int G = T <= 16 ? 16 : (T <= 32 ? 32 : 64);
  const int W = cost_team(S, cu_count);
  const int blocks = W > 1 ? S : (S + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
  const size_t lds_bytes = eval_lds(W);
  const auto kernel = W == MAX_TEAM ? (ext ? k_cost<true, true> : k_cost<false, true>)
                                    : (ext ? k_cost<true, false> : k_cost<false, false>);
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(W > 1 ? W * WAVE : BLOCK), lds_bytes, s, rb, pp,
                     prob, X, S, T, G, dJ, J_out, dX, with_grad, W);
  return hipGetLastError();
}

hipError_t launch_guide(const RobotDev* rb, const ParamsDev* pp, const ProbDev& prob, float* X,
                        int S, int T, float alpha, int n_steps, float* J_out, bool ext,
                        int cu_count, hipStream_t s) {
  const int G = T <= 16 ? 16 : (T <= 32 ? 32 : 64);
  const int W = cost_team(S, cu_count);
  const int blocks = W > 1 ? S : (S + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
  const size_t lds_bytes = eval_lds(W);
  const auto kernel = W == MAX_TEAM ? (ext ? k_guide<true, true> : k_guide<false, true>)
                                    : (ext ? k_guide<true, false> : k_guide<false, false>);
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(W > 1 ? W * WAVE : BLOCK), lds_bytes, s, rb, pp,
                     prob, X, S, T, G, alpha, n_steps, J_out, W);
  return hipGetLastError();
}

hipError_t launch_spheres(const RobotDev* rb, const float* X, int S, int T, float* out,
                          hipStream_t s) {
  int n = S * T;
  hipLaunchKernelGGL(k_spheres, dim3((n + 255) / 256), dim3(256), 0, s, rb, X, n, out);
  return hipGetLastError();
}

}  // namespace dsk
