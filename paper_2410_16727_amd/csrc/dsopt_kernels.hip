// gfx950 kernels around the optimiser: the plain variants of the persistent
// kernel, best seed, queue order, resets, and their launches.
#include <hip/hip_runtime.h>

#include "dsopt_optimize.h"

namespace dsk {
namespace {

// Best seed per problem: lowest cost among successful seeds (ties: lowest
// index), else lowest cost among valid seeds.
__global__ void __launch_bounds__(256) k_best(const ProbDev* __restrict__ probs,
                                              const int* __restrict__ list) {
  if (list && (int)blockIdx.x >= list[0]) return;
  const ProbDev& pb = probs[list ? list[1 + blockIdx.x] : blockIdx.x];
  __shared__ int s_any;
  __shared__ unsigned long long s_key[2];
  __shared__ int s_valid;
  if (threadIdx.x == 0) { s_any = 0; s_key[0] = ~0ull; s_key[1] = ~0ull; s_valid = 0; }
  __syncthreads();
  for (int s = threadIdx.x; s < pb.S; s += blockDim.x) {
    const ds_seed_result& r = pb.seed_res[s];
    if (r.valid) {
      atomicAdd(&s_valid, 1);
      // order-preserving key of a finite float cost, then the index
      unsigned u = __float_as_uint(r.cost);
      u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
      unsigned long long key = ((unsigned long long)u << 32) | (unsigned)s;
      atomicMin(&s_key[0], key);
      if (r.success) { atomicMin(&s_key[1], key); s_any = 1; }
    }
  }
  __syncthreads();
  const unsigned long long key = s_any ? s_key[1] : s_key[0];
  const int best = (key == ~0ull) ? -1 : (int)(key & 0xffffffffu);
  float* land_traj = pb.landing ? reinterpret_cast<float*>(pb.landing + 256) : nullptr;
  if (best >= 0)
    for (int e = threadIdx.x; e < pb.T * NJ; e += blockDim.x) {
      const float v = pb.final_traj[(size_t)best * pb.T * NJ + e];
      pb.best_traj[e] = v;
      if (land_traj) land_traj[e] = v;
    }
  if (threadIdx.x == 0) {
    ds_result out;
    out.best_seed = best;
    out.n_valid_seeds = s_valid;
    out.n_iters = pb.n_iters;
    if (best >= 0) {
      const ds_seed_result& r = pb.seed_res[best];
      out.success = r.success;
      out.collision_free = r.collision_free;
      out.pos_err_m = r.pos_err;
      out.rot_err_rad = r.rot_err;
      out.cost = r.cost;
      out.min_clearance_m = r.clearance;
      out.max_jerk = r.max_jerk;
      out.max_vel = r.max_vel;
      out.motion_time = r.motion_time;
    } else {
      out.success = 0;
      out.collision_free = 0;
      out.pos_err_m = out.rot_err_rad = out.cost = out.min_clearance_m = out.max_jerk = NAN;
      out.max_vel = out.motion_time = NAN;
    }
    *pb.result = out;
    if (pb.landing) *reinterpret_cast<ds_result*>(pb.landing) = out;
  }
}

// Fresh tiles: each tile's iteration counters (so the optimiser starts from
// the seed) and its seed's result record (counters accumulate over
// launches).  One workgroup of one wavefront per tile.
// Queue order of a batched launch after the tiles' initial evaluation: one
// workgroup per XCD queue sorts its tiles, longest expected first -- by
// lane group (a G = 64 tile walks twice the spheres per lane of a G = 32
// one), then by the cost at the seed (seeds far from a good trajectory
// tend to need more line-search candidates) -- with a counting sort over
// ORDER_BINS keys.  Ties land in any order: the order only decides when a
// seed runs, never what it computes.
constexpr int ORDER_BINS = 4096;
constexpr int ORDER_THREADS = 1024;
__device__ __forceinline__ int order_key(const TileDev& t) {
  const float J = t.state[ST_J];
  const int grp = t.G >= 64 ? 2 : (t.G >= 32 ? 1 : 0);
  // log2(1 + J) in 1/48 steps, 1024 per group; a NaN cost sorts last
  const float l = J > 0.f ? __log2f(1.f + J) * 48.f : 0.f;
  const int b = l >= 0.f ? (int)fminf(l, 1023.f) : 0;
  return grp * 1024 + b;
}
__global__ void __launch_bounds__(ORDER_THREADS) k_queue_order(const TileDev* __restrict__ tiles,
                                                               const int* __restrict__ ranges,
                                                               int* __restrict__ list,
                                                               int* __restrict__ counter) {
  __shared__ int bins[ORDER_BINS];
  const int x = blockIdx.x;
  const int b = ranges[x], e = ranges[x + 1];
  for (int i = threadIdx.x; i < ORDER_BINS; i += blockDim.x) bins[i] = 0;
  if (threadIdx.x == 0) counter[x] = 0;
  __syncthreads();
  for (int i = b + threadIdx.x; i < e; i += blockDim.x) atomicAdd(&bins[order_key(tiles[i])], 1);
  __syncthreads();
  // start of each key's run, largest key first: an exclusive scan of the
  // bins in descending key order.  Thread t owns the PER keys from
  // ORDER_BINS - 1 - PER t downwards; the threads' totals are scanned per
  // wavefront (shuffles), then across the wavefronts (LDS).
  constexpr int PER = ORDER_BINS / ORDER_THREADS;
  constexpr int NW = ORDER_THREADS / WAVE;
  __shared__ int wsum[NW];
  const int t = threadIdx.x, lane = t & (WAVE - 1), wv = t / WAVE;
  int cnt[PER], tot = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    cnt[q] = bins[ORDER_BINS - 1 - (PER * t + q)];
    tot += cnt[q];
  }
  int inc = tot;   // inclusive scan of the totals inside the wavefront
#pragma unroll
  for (int off = 1; off < WAVE; off <<= 1) {
    const int o = __shfl_up(inc, off);
    if (lane >= off) inc += o;
  }
  if (lane == WAVE - 1) wsum[wv] = inc;
  __syncthreads();
  int base = 0;
  for (int w = 0; w < wv; ++w) base += wsum[w];
  int run = base + inc - tot;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    bins[ORDER_BINS - 1 - (PER * t + q)] = run;
    run += cnt[q];
  }
  __syncthreads();
  for (int i = b + threadIdx.x; i < e; i += blockDim.x)
    list[b + atomicAdd(&bins[order_key(tiles[i])], 1)] = i;
}

__global__ void __launch_bounds__(64) k_tile_reset(const TileDev* __restrict__ tiles,
                                                   const ProbDev* __restrict__ probs,
                                                   int* __restrict__ counter) {
  if (blockIdx.x == 0 && threadIdx.x < N_XCD) counter[threadIdx.x] = 0;   // the tile queues
  const TileDev td = tiles[blockIdx.x];
  reinterpret_cast<int*>(td.state)[ST_ITER + threadIdx.x] = 0;
  reinterpret_cast<int*>(td.state)[ST_EVG + threadIdx.x] = 0;
  constexpr int W = (int)(sizeof(ds_seed_result) / sizeof(int));
  if (threadIdx.x < W)
    reinterpret_cast<int*>(probs[td.prob].seed_res + td.seed0)[threadIdx.x] = 0;
}

__global__ void k_zero_i32(int* p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

}  // namespace

int team_block(int W) { return (W > 1 ? W : WAVES_PER_BLOCK) * WAVE; }
// dynamic LDS of an optimiser workgroup: a team's evaluation, history ring,
// coarse table and direction broadcast; single wavefronts: one coarse table
// each
size_t team_lds(int W) {
  return W > 1 ? eval_lds(W) + (H_FLOATS + COARSE_FLOATS + DL_FLOATS) * sizeof(float)
               : (size_t)WAVES_PER_BLOCK * COARSE_FLOATS * sizeof(float);
}

const void* optimize_kernel_ext(int W);   // dsopt_optimize_ext.hip

// (With one bare link in seven the plain kernels are as fast or faster; a full
// team's tests cost nothing beside its kinematics; with the optional terms the
// sweeps are a smaller part.)
static OptKernel optimize_kernel(const OptForm& f) {
  if (f.ext) return reinterpret_cast<OptKernel>(const_cast<void*>(optimize_kernel_ext(f.waves)));
  if (f.exact && f.waves == 1) return k_optimize<false, false, false, false, true>;
  if (f.exact && f.waves < MAX_TEAM) return k_optimize<true, false, false, true, true>;
  if (f.bare && f.waves == 1) return k_optimize<false, false, false, true>;
  if (f.bare && f.waves == MAX_TEAM) return k_optimize<true, false, true, true>;
  return optimize_variant<false>(f.waves);
}

hipError_t launch_optimize(const RobotDev* rb, const ParamsDev* pp, const ProbDev* probs,
                           const TileDev* tiles, int n_tiles, int* counter, int grid_blocks,
                           int max_iters, const OptForm& form, hipStream_t s,
                           const int* xcd_ranges, const int* tile_list) {
  hipLaunchKernelGGL(optimize_kernel(form), dim3(grid_blocks), dim3(team_block(form.waves)),
                     team_lds(form.waves), s, rb, pp, probs, tiles, tile_list, (const int*)nullptr,
                     n_tiles, counter, max_iters, (const int*)nullptr, xcd_ranges);
  return hipGetLastError();
}

hipError_t launch_queue_order(const TileDev* tiles, const int* xcd_ranges, int* list,
                              int* counter, hipStream_t s) {
  hipLaunchKernelGGL(k_queue_order, dim3(N_XCD), dim3(ORDER_THREADS), 0, s, tiles, xcd_ranges,
                     list, counter);
  return hipGetLastError();
}

hipError_t launch_serve_step(const RobotDev* rb, const ParamsDev* pp, const ProbDev* probs,
                             const TileDev* tiles, const int* tile_list, int* counter,
                             int max_tiles, int grid_blocks, const int* max_iters_dev,
                             const OptForm& form, hipStream_t s) {
  // tile_list[0] holds the number of listed tiles, the indices follow; the
  // iterations of this replay are read from max_iters_dev
  hipLaunchKernelGGL(optimize_kernel(form), dim3(grid_blocks), dim3(team_block(form.waves)),
                     team_lds(form.waves), s, rb, pp, probs, tiles, tile_list + 1, tile_list, max_tiles,
                     counter, 0, max_iters_dev, (const int*)nullptr);
  return hipGetLastError();
}

int optimize_blocks_per_cu(const OptForm& f) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, optimize_kernel(f), team_block(f.waves),
                                                   team_lds(f.waves)) != hipSuccess)
    return 1;
  return n > 0 ? n : 1;
}

hipError_t launch_tile_reset(const TileDev* tiles, const ProbDev* probs, int n_tiles, int* counter,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_tile_reset, dim3(n_tiles), dim3(64), 0, s, tiles, probs, counter);
  return hipGetLastError();
}

hipError_t launch_best(const ProbDev* probs, int n_probs, const int* list, hipStream_t s) {
  hipLaunchKernelGGL(k_best, dim3(n_probs), dim3(256), 0, s, probs, list);
  return hipGetLastError();
}

hipError_t launch_zero_i32(int* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_i32, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace dsk
