// Device code of the objective: one evaluation of a trajectory by a wavefront
// or a team (included by the translation units with kernels that evaluate).
//
// Mapping: one wavefront (or a team of W wavefronts) owns one tile = one
// seed of one problem; lane t of each lane group holds waypoint t (group
// size G = 64, 32 or 16 >= T) and the 64 / G groups of a wavefront are
// copies of the seed that split its spheres.  Per lane the kernel runs the whole per-waypoint chain of the
// objective (App. A.6): forward kinematics (sincos + 3x4 compositions with
// the robot table read through the scalar cache), sphere centres, an ESDF
// gather of one 32-byte corner record per sphere (two 16-byte buffer
// loads), the smooth hinge, and -- for the gradient -- the joint-axis
// adjoint: sphere forces f = w_c phi'(D) grad d accumulated per link into
// a wrench and projected on every preceding joint twist, recomputing the
// kinematics instead of storing transforms.  Finite differences of the
// trajectory (smoothness) move between lanes with cross-lane shuffles;
// per-seed sums (cost, L-BFGS dot products, Armijo tests) are butterfly
// reductions inside the lane group, so every lane ends with bitwise the same
// value and the reduction order depends only on G.  Nothing here is a dense
// contraction: no MFMA.
#pragma once

#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <cstddef>
#include <type_traits>

#include "dsopt_internal.h"

namespace dsk {
namespace {

constexpr unsigned RSRC_DWORD3 = 0x00020000u;   // raw buffer, gfx9 family

// Pointers read from tables are generic to the compiler; these casts state
// that they address global memory, so accesses use global (not flat)
// instructions.
#define DS_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ DS_GLOBAL T* glb(T* p) {
  return (DS_GLOBAL T*)p;
}
template <class T>
__device__ __forceinline__ const DS_GLOBAL T* glb(const T* p) {
  return (const DS_GLOBAL T*)p;
}
// ... and that a pointer into a __shared__ array addresses LDS (ds_read /
// ds_write rather than flat accesses).
#define DS_LDS __attribute__((address_space(3)))
template <class T>
__device__ __forceinline__ DS_LDS T* lds(T* p) {
  return (DS_LDS T*)p;
}
#ifndef DSOPT_CH
#define DSOPT_CH 4
#endif
constexpr int CH = DSOPT_CH;                     // sphere gathers in flight per lane
static_assert(CH >= 2, "a chunk's short form has two");
// s_waitcnt operand: vector memory count 0, the export and LDS/scalar
// counts at their maxima (not waited on)
constexpr int WAIT_VMEM_ALL = 0x0F70;

// Butterfly reductions over a lane group of G = 16, 32 or 64 lanes.  The
// first four stages pair lanes inside a 16-lane row with DPP (quad
// permutations 1<->0 / 2<->0, then the half-row and row mirrors), the
// remaining ones exchange rows (lane ^ 16) and halves (lane ^ 32) with the
// permlane swaps -- VALU instructions, no LDS round trip.  Every pairing is
// an involution, so both partners add the same two numbers and every lane of
// the group ends with bitwise the same result.
constexpr int DPP_QUAD_XOR1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int DPP_QUAD_XOR2 = 0x4E;   // quad_perm [2,3,0,1]
constexpr int DPP_HALF_MIRROR = 0x141;
constexpr int DPP_MIRROR = 0x140;

constexpr int DPP_WAVE_SHL1 = 0x130;   // lane i reads lane i + 1
constexpr int DPP_WAVE_SHR1 = 0x138;   // lane i reads lane i - 1

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// The value of lane i + 1 / lane i - 1 (one DPP move; the lane past either
// end of the wavefront reads 0).  Callers only use lanes whose neighbour is
// in the same lane group.
__device__ __forceinline__ float from_next(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), DPP_WAVE_SHL1, 0xF, 0xF, true));
}
__device__ __forceinline__ float from_prev(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), DPP_WAVE_SHR1, 0xF, 0xF, true));
}

struct OpSum { __device__ static float f(float a, float b) { return a + b; } };
struct OpMax { __device__ static float f(float a, float b) { return fmaxf(a, b); } };
struct OpMin { __device__ static float f(float a, float b) { return fminf(a, b); } };

// v combined with lane ^ 16's v (v_permlane16_swap with v as both operands
// exchanges the odd rows of the first with the even rows of the second: in
// every lane one result is its own value and the other its partner's) and
// with lane ^ 32's (v_permlane32_swap: the upper half of the first operand
// with the lower half of the second).  The operations are commutative, so
// combining the two results needs no per-lane select.
template <class Op>
__device__ __forceinline__ float xor16_reduce(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), true,
                                                  false);
  return Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float xor32_reduce(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), true,
                                                  false);
  return Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float xor_reduce(float v, int off) {
  return off == 16 ? xor16_reduce<Op>(v) : xor32_reduce<Op>(v);
}

template <class Op>
__device__ __forceinline__ float grp_reduce(float v, int G) {
  v = Op::f(v, dpp<DPP_QUAD_XOR1>(v));
  v = Op::f(v, dpp<DPP_QUAD_XOR2>(v));
  v = Op::f(v, dpp<DPP_HALF_MIRROR>(v));
  v = Op::f(v, dpp<DPP_MIRROR>(v));
  if (G > 16) v = xor16_reduce<Op>(v);
  if (G > 32) v = xor32_reduce<Op>(v);
  return v;
}

__device__ __forceinline__ float grp_sum(float v, int G) { return grp_reduce<OpSum>(v, G); }
__device__ __forceinline__ float grp_max(float v, int G) { return grp_reduce<OpMax>(v, G); }
__device__ __forceinline__ float grp_min(float v, int G) { return grp_reduce<OpMin>(v, G); }
__device__ __forceinline__ float dot7(const float* a, const float* b) {
  float s = a[0] * b[0];
#pragma unroll
  for (int j = 1; j < NJ; ++j) s += a[j] * b[j];
  return s;
}

// The goal pose of a wavefront's tile lives in LDS: twelve values that one
// section of the evaluation reads (in registers they were live across all of
// it).
struct Goal {
  float pd[3];
  float Rd[9];
};
constexpr int MAX_WAVES = 8;   // wavefronts of a workgroup
__shared__ Goal s_goal[MAX_WAVES];

// Unit goal quaternion (w, x, y, z) -> rotation matrix (uniform per tile).
__device__ __forceinline__ void put_goal(const ProbDev& pb) {
  Goal g;
  float w = pb.quat[0], x = pb.quat[1], y = pb.quat[2], z = pb.quat[3];
  float n = sqrtf(w * w + x * x + y * y + z * z);
  w /= n; x /= n; y /= n; z /= n;
  g.Rd[0] = 1.f - 2.f * (y * y + z * z); g.Rd[1] = 2.f * (x * y - w * z); g.Rd[2] = 2.f * (x * z + w * y);
  g.Rd[3] = 2.f * (x * y + w * z); g.Rd[4] = 1.f - 2.f * (x * x + z * z); g.Rd[5] = 2.f * (y * z - w * x);
  g.Rd[6] = 2.f * (x * z - w * y); g.Rd[7] = 2.f * (y * z + w * x); g.Rd[8] = 1.f - 2.f * (x * x + y * y);
  g.pd[0] = pb.pd[0]; g.pd[1] = pb.pd[1]; g.pd[2] = pb.pd[2];
  // (a wavefront's LDS accesses complete in order: no barrier)
  if ((threadIdx.x & (WAVE - 1)) == 0) s_goal[threadIdx.x / WAVE] = g;
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ Goal get_goal() {
  return s_goal[__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE))];
}

// The robot's sphere ranges, packed into three scalar registers: read from
// the table at every use they were a scalar memory round trip per link and
// evaluation (the compiler repeats invariant loads when it is short of
// scalar registers, unless their value is opaque to it).
struct Links {
  unsigned lo, hi, misc;
  // spheres of link l (0..6): [begin(l), begin(l + 1))
  __device__ __forceinline__ int begin(int l) const {
    return (int)((l < 4 ? lo >> (8 * l) : hi >> (8 * (l - 4))) & 255u);
  }
  __device__ __forceinline__ int last() const { return begin(NJ) - 1; }
  // whether every sphere of link l sits on its z axis
  __device__ __forceinline__ bool axis(int l) const { return (misc >> l) & 1u; }
  __device__ __forceinline__ bool all_axis() const { return (misc & 0x7Fu) == 0x7Fu; }
  __device__ __forceinline__ int most() const { return (int)(misc >> 8); }   // on one link
};
static_assert(DS_MAX_SPHERES <= 255, "sphere positions are bytes");

__device__ __forceinline__ Links make_links(const RobotDev* __restrict__ rb) {
  Links k{0, 0, (unsigned)rb->axis_links | ((unsigned)rb->max_per_link << 8)};
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    k.lo |= (unsigned)rb->link_begin[l] << (8 * l);
    k.hi |= (unsigned)rb->link_begin[l + 4] << (8 * l);
  }
  k.lo = __builtin_amdgcn_readfirstlane(k.lo);
  k.hi = __builtin_amdgcn_readfirstlane(k.hi);
  k.misc = __builtin_amdgcn_readfirstlane(k.misc);
  asm("" : "+s"(k.lo), "+s"(k.hi), "+s"(k.misc));
  return k;
}

struct Sampler {
  Links ln;
  __amdgpu_buffer_rsrc_t rsrc;
  float ox, oy, oz, inv_h, h, nxm1, nym1, nzm1;
  float fxm2, fym2, fzm2;          // last cell index per axis, as floats
  int cx, cy;                      // cells along x and y
  const DS_LDS uint8_t* cm;        // the scene's coarse table (4-bit levels), staged in LDS
  float cq;                        // distance of one level
  int cshift, cdx, cdy;
};

__device__ __forceinline__ Sampler make_sampler(const SceneDev& sc, const RobotDev* __restrict__ rb) {
  Sampler s;
  s.ln = make_links(rb);
  s.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)sc.rec, (short)0, (int)sc.bytes, RSRC_DWORD3);
  s.ox = sc.ox; s.oy = sc.oy; s.oz = sc.oz; s.inv_h = sc.inv_h; s.h = 1.f / sc.inv_h;
  s.nxm1 = (float)(sc.nx - 1); s.nym1 = (float)(sc.ny - 1); s.nzm1 = (float)(sc.nz - 1);
  s.fxm2 = (float)(sc.nx - 2); s.fym2 = (float)(sc.ny - 2); s.fzm2 = (float)(sc.nz - 2);
  s.cx = sc.nx - 1;
  s.cy = sc.ny - 1;
  s.cm = nullptr;
  s.cq = sc.cq;
  s.cshift = sc.cshift;
  s.cdx = sc.cdx;
  s.cdy = sc.cdy;
  return s;
}

// Copy the scene's coarse table into LDS (threads tid = 0..nth-1 of the
// group that shares it; the caller synchronises them afterwards) in
// 16-byte pieces, STAGE_UNROLL loads in flight per thread before their LDS
// stores (one load at a time made every piece a memory round trip).  The
// table's allocation and both ends are 16-byte aligned.
constexpr int STAGE_UNROLL = 4;
__device__ __forceinline__ void stage_coarse(const SceneDev& sc, DS_LDS uint8_t* dst, int tid,
                                             int nth) {
  const int n = (sc.cdx * sc.cdy * sc.cdz + 31) / 32;   // 32 levels per piece
  const DS_GLOBAL uint32_t* src = glb(reinterpret_cast<const uint32_t*>(sc.coarse));
  DS_LDS uint32_t* d = (DS_LDS uint32_t*)dst;
  for (int i0 = tid; i0 < n; i0 += STAGE_UNROLL * nth) {
    uint32_t v[STAGE_UNROLL][4];
#pragma unroll
    for (int u = 0; u < STAGE_UNROLL; ++u) {
      const int i = i0 + u * nth;
      if (i < n) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[u][q] = src[4 * i + q];
      }
    }
#pragma unroll
    for (int u = 0; u < STAGE_UNROLL; ++u) {
      const int i = i0 + u * nth;
      if (i < n) {
#pragma unroll
        for (int q = 0; q < 4; ++q) d[4 * i + q] = v[u][q];
      }
    }
  }
}

// A coarse-table entry as a distance: level * cq, at most the block's
// minimum node distance.
__device__ __forceinline__ float coarse_at(const Sampler& S, int idx) {
  const unsigned b = S.cm[idx >> 1];
  return (float)((b >> ((idx & 1) << 2)) & 15u) * S.cq;
}

// A sample's place in the grid.  u = (c - origin) / voxel is the sphere
// centre c in grid units; the sample's cell is trunc(clamp(u, 0, n-2)) per
// axis (the cell whose corners bracket the clamped point), its fractional
// position clamp(u, 0, n-1) - cell, and the gradient is zero along axes
// where u was clamped.
//
// A link frame (R, p) maps a sphere offset o to c = p + R o.  For a link
// whose spheres all lie on its z axis (o = (0, 0, oz)) the link's part is
// formed once -- u = u0 + oz az with u0 = (p - origin) / voxel and
// az = R e_z / voxel -- so a sphere costs one FMA per axis.
struct LinkGrid {
  float u0[3], az[3];
};

// (z: the third column of R)
__device__ __forceinline__ LinkGrid link_grid(const Sampler& S, const float* z, const float* p) {
  LinkGrid g;
  g.u0[0] = (p[0] - S.ox) * S.inv_h;
  g.u0[1] = (p[1] - S.oy) * S.inv_h;
  g.u0[2] = (p[2] - S.oz) * S.inv_h;
  g.az[0] = z[0] * S.inv_h;
  g.az[1] = z[1] * S.inv_h;
  g.az[2] = z[2] * S.inv_h;
  return g;
}

// World centre of a sphere at oz on its link's z axis, per component, as the
// full product gives it with zeros in x and y (rounded before p is added).
__device__ __forceinline__ float axis_centre(float z, float oz, float p) {
#pragma clang fp contract(off)
  const float c = z * oz;
  return c + p;
}

// Grid position of a sphere at oz on its link's z axis ...
__device__ __forceinline__ void axis_pos(const LinkGrid& g, float oz, float* u) {
#pragma unroll
  for (int r = 0; r < 3; ++r) u[r] = fmaf(oz, g.az[r], g.u0[r]);
}
// ... and of any sphere on the link (R, p).
__device__ __forceinline__ void frame_pos(const Sampler& S, const float* R, const float* p,
                                          float4 sp, float* u) {
  const float cx = R[0] * sp.x + R[1] * sp.y + R[2] * sp.z + p[0];
  const float cy = R[3] * sp.x + R[4] * sp.y + R[5] * sp.z + p[1];
  const float cz = R[6] * sp.x + R[7] * sp.y + R[8] * sp.z + p[2];
  u[0] = (cx - S.ox) * S.inv_h;
  u[1] = (cy - S.oy) * S.inv_h;
  u[2] = (cz - S.oz) * S.inv_h;
}

// The sample's cell: trunc(clamp(u, 0, n-2)) per axis (for u >= 0,
// min(trunc(min(u, n-1)), n-2) == trunc(min(u, n-2)): one v_med3 and one
// conversion per axis).
__device__ __forceinline__ void cell_of(const Sampler& S, const float* u, int* i) {
  i[0] = (int)__builtin_amdgcn_fmed3f(u[0], 0.f, S.fxm2);
  i[1] = (int)__builtin_amdgcn_fmed3f(u[1], 0.f, S.fym2);
  i[2] = (int)__builtin_amdgcn_fmed3f(u[2], 0.f, S.fzm2);
}

// The cell's block in the coarse table and its record's byte offset.
// Every product fits 24 bits: the upload keeps (ny-1)(nz-1) below 2^24,
// and the coarse table has at most COARSE_MAX blocks (stating the bounds
// keeps both products 24-bit multiply-adds).
__device__ __forceinline__ int block_index(const Sampler& S, const int* i) {
  const unsigned crow =
      __umul24((unsigned)S.cdy, (unsigned)(i[2] >> S.cshift)) + (unsigned)(i[1] >> S.cshift);
  __builtin_assume(crow < (1u << 24));
  return (int)(__umul24((unsigned)S.cdx, crow) + (unsigned)(i[0] >> S.cshift));
}

__device__ __forceinline__ int record_offset(const Sampler& S, const int* i) {
  const unsigned row = __umul24((unsigned)S.cy, (unsigned)i[2]) + (unsigned)i[1];
  __builtin_assume(row < (1u << 24));
  return (int)((__umul24((unsigned)S.cx, row) + (unsigned)i[0]) << 5);
}

// Trilinear blend of a cell record (a: z0 corners, b: z1 corners) at the
// fractional position (fx, fy, fz): the value, and the differences its
// spatial gradient is formed from.
struct Blend {
  float d;                          // interpolated distance
  float dx00, dx10, dx01, dx11;     // x differences of the four x edges
  float dy0, dy1, dz;               // y differences at z0/z1, z difference
};

__device__ __forceinline__ Blend blend_value(float fx, float fy, float fz, float4 a, float4 b) {
  Blend r;
  r.dx00 = a.y - a.x; r.dx10 = a.w - a.z; r.dx01 = b.y - b.x; r.dx11 = b.w - b.z;
  float c00 = a.x + fx * r.dx00;
  float c10 = a.z + fx * r.dx10;
  float c01 = b.x + fx * r.dx01;
  float c11 = b.z + fx * r.dx11;
  r.dy0 = c10 - c00;
  r.dy1 = c11 - c01;
  float c0 = c00 + fy * r.dy0;
  float c1 = c01 + fy * r.dy1;
  r.dz = c1 - c0;
  r.d = c0 + fz * r.dz;
  return r;
}

// Its spatial gradient in grid units (times 1/voxel by the caller).
__device__ __forceinline__ void blend_grad(float fy, float fz, const Blend& r, float& gx,
                                           float& gy, float& gz) {
  float e0 = r.dx00 + fy * (r.dx10 - r.dx00);
  float e1 = r.dx01 + fy * (r.dx11 - r.dx01);
  gx = e0 + fz * (e1 - e0);
  gy = r.dy0 + fz * (r.dy1 - r.dy0);
  gz = r.dz;
}

__device__ __forceinline__ float4 load_rec(const Sampler& S, int off) {
  auto v = __builtin_amdgcn_raw_buffer_load_b128(S.rsrc, off, 0, 0);
  return *reinterpret_cast<float4*>(&v);
}

enum { EV_COST = 0, EV_GRAD = 1, EV_RESULT = 2 };

// The robot's sphere table (offset, radius; sorted by link) staged in LDS
// by every kernel that evaluates the objective: the sphere a lane takes
// depends on its copy index, so the reads are per-lane and would otherwise
// be vector memory round trips ahead of every record gather.
__shared__ float4 s_sph[DS_MAX_SPHERES];

// The fixed transforms before the joints, rows of 3x4: read by the wavefronts
// that form a team's frames (scalar loads would be five round trips along
// the chain).
__shared__ float4 s_frame[3 * NJ + 3];   // and the end effector's

// Fill s_sph and s_frame; every thread of the workgroup must call it.
__device__ __forceinline__ void stage_robot(const RobotDev* __restrict__ rb) {
  for (int i = threadIdx.x; i < rb->ns; i += blockDim.x) s_sph[i] = rb->sph[i];
  static_assert(offsetof(RobotDev, Fee) == sizeof(RobotDev::F), "the frames are one array");
  if (threadIdx.x < 3 * NJ + 3) {
    const float* f = &rb->F[0][0] + 4 * threadIdx.x;
    s_frame[threadIdx.x] = make_float4(f[0], f[1], f[2], f[3]);
  }
  __syncthreads();
}

// Joint twists (axis z_i, origin o_i) of the swept joints, kept for the
// wrench projections of the adjoint.
struct Twists {
  float z[NJ][3], o[NJ][3];
  __device__ __forceinline__ void put(int i, const float* R, const float* p) {
    z[i][0] = R[2]; z[i][1] = R[5]; z[i][2] = R[8];
    o[i][0] = p[0]; o[i][1] = p[1]; o[i][2] = p[2];
  }
  __device__ __forceinline__ void get(int i, float* zi, float* oi) const {
    zi[0] = z[i][0]; zi[1] = z[i][1]; zi[2] = z[i][2];
    oi[0] = o[i][0]; oi[1] = o[i][1]; oi[2] = o[i][2];
  }
};

struct EvalOut {
  float cost;        // this lane's share of the seed objective (0 when inactive)
  float g[NJ];       // gradient row (EV_GRAD; zero at t = 0 and inactive lanes)
  float clr;         // min (distance - radius) at this waypoint (EV_RESULT)
  float perr, rerr;  // goal errors at this lane's waypoint (EV_RESULT)
  int ng;            // cell records this lane gathered
};

// Smoothness on the lane group: v_t = q_{t+1} - q_t (t <= T-2),
// a_t = v_t - v_{t-1} (t < T), j_t = a_{t+1} - a_t (t < T) plus
// j_{-1} = a_0 at t = 0 -- the first/second/third differences of the
// sequence padded with two copies of q_0 and of q_{T-1}.  The gradient
// applies the transposed stencils with the same lane shifts (DPP moves; the
// masks keep every read inside the lane group).
template <bool GRAD>
__device__ __forceinline__ float smoothness(const ParamsDev& P, const float* q, int t, int T,
                                            float* g) {
  float c = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    float qn = from_next(q[j]);
    float v = (t <= T - 2) ? qn - q[j] : 0.f;
    float vp = from_prev(v);
    float a = (t < T) ? v - (t >= 1 ? vp : 0.f) : 0.f;
    float an = from_next(a);
    float jk = (t < T) ? ((t + 1 < T ? an : 0.f) - a) : 0.f;
    float jm = (t == 0) ? a : 0.f;   // j_{-1}
    c += P.lv * (v * v) + P.la * (a * a) + P.lj * (jk * jk) + P.lj * (jm * jm);
    if (GRAD) {
      float jb = 2.f * P.lj * jk;
      float jbp = from_prev(jb);
      float ab = (t < T) ? 2.f * P.la * a + ((t == 0) ? 2.f * P.lj * jm : jbp) - jb : 0.f;
      float abn = from_next(ab);
      float vb = (t <= T - 2) ? 2.f * P.lv * v + ab - abn : 0.f;
      float vbp = from_prev(vb);
      g[j] += ((t >= 1) ? vbp : 0.f) - vb;
    }
  }
  return c;
}

// Joint-limit penalty (its gradient into g).
template <bool GRAD>
__device__ __forceinline__ float limits(const RobotDev* __restrict__ rb, const ParamsDev& P,
                                        const float* q, float* g) {
  float lim = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    float hi = q[j] - rb->qhi[j], lo = rb->qlo[j] - q[j];
    float hp = fmaxf(hi, 0.f), lp = fmaxf(lo, 0.f);
    lim += hp * hp + lp * lp;
    if (GRAD) g[j] += 2.f * P.wl * (hp - lp);
  }
  return P.wl * lim;
}

// A team of W wavefronts (one workgroup) optimises one seed: every
// wavefront holds the whole trajectory (one waypoint per lane group) and
// takes every (W*L)-th sphere of each link; the partial sums meet in
// double-buffered LDS with one barrier per evaluation.  W = 1: independent
// wavefronts, no barrier.
constexpr int MAX_TEAM = 8;
constexpr int PART = NJ + 2;   // partial sums per lane: hinge sum, gradient row, clearance

struct Team {
  int W, w;       // team size, this wavefront's index
  float* lds;     // [2][W][PART][64]
  float* kin;     // [KIN_ROWS][64] of a full team, else null
  int buf;
  __device__ __forceinline__ void sync() const {
    if (W > 1) __syncthreads();
  }
};

// Kinematics of a full team (MAX_TEAM wavefronts), shared through LDS.  With
// every wavefront forming the whole chain (about 530 VALU instructions of
// 1270 per evaluation, two wavefronts on each SIMD) the SIMDs issued in 80 %
// of the cycles; here three wavefronts form a row of every frame each (the
// rows of R and the components of p follow the chain independently of each
// other) and all of them read what they need.  One more barrier, the same
// arithmetic per element: the results are those of the whole chain.
// Rows of 64 lanes: per link the joint axis (third column of R) and the
// origin; per link the first two columns of R; the goal's part of the sums.
// Smaller teams keep the whole chain: there are fewer copies of it to save,
// and the rows would halve the workgroups that fit a CU.
constexpr int KIN_ZO = 0, KIN_XY = KIN_ZO + 6 * NJ, KIN_GOAL = KIN_XY + 6 * NJ,
              KIN_ROWS = KIN_GOAL + 1;

// Hinge cost of one sphere sample (grid position u, cell record ra/rz,
// radius r) and, with GRAD, its force accumulated into the link
// wrench (F, M about the world origin).  Returns whether the force terms
// ran (some lane of the wavefront inside the hinge band).
template <int MODE>
__device__ __forceinline__ bool sphere_term(const ParamsDev& P, const Sampler& S, const float* u,
                                            float4 ra, float4 rz, float r,
                                            float& phisum, float& clr, float* FM) {
  constexpr bool GRAD = (MODE == EV_GRAD);
  const float cx = __builtin_amdgcn_fmed3f(u[0], 0.f, S.nxm1);
  const float cy = __builtin_amdgcn_fmed3f(u[1], 0.f, S.nym1);
  const float cz = __builtin_amdgcn_fmed3f(u[2], 0.f, S.nzm1);
  // the cell, as cell_of gives it
  const float fx0 = cx - truncf(__builtin_amdgcn_fmed3f(u[0], 0.f, S.fxm2));
  const float fy = cy - truncf(__builtin_amdgcn_fmed3f(u[1], 0.f, S.fym2));
  const float fz = cz - truncf(__builtin_amdgcn_fmed3f(u[2], 0.f, S.fzm2));
  const Blend bl = blend_value(fx0, fy, fz, ra, rz);
  float D = bl.d - r;
  float De = D - P.eps;
  float phi = (D < P.eps) ? De * De * P.half_inv_eps : 0.f;
  phi = (D < 0.f) ? 0.5f * P.eps - D : phi;
  phisum += phi;
  if (MODE == EV_RESULT) clr = fminf(clr, D);
  // the force is zero outside the hinge band: when no lane of the
  // wavefront has a sample inside it, the gradient and the wrench terms
  // (which would add zeros) are skipped
  const bool band = GRAD && __any(D < P.eps);
  if (band) {
    float gx, gy, gz;
    blend_grad(fy, fz, bl, gx, gy, gz);
    // world units; zero along axes where the point was clamped
    gx *= (cx == u[0]) ? S.inv_h : 0.f;
    gy *= (cy == u[1]) ? S.inv_h : 0.f;
    gz *= (cz == u[2]) ? S.inv_h : 0.f;
    float dphi = (D < P.eps) ? De * P.inv_eps : 0.f;
    dphi = (D < 0.f) ? -1.f : dphi;
    float w = P.wc * dphi;
    float fx = w * gx, fyy = w * gy, fzz = w * gz;
    // the sphere centre (the moment arm) back from its grid position
    const float px = fmaf(u[0], S.h, S.ox);
    const float py = fmaf(u[1], S.h, S.oy);
    const float pz = fmaf(u[2], S.h, S.oz);
    FM[0] += fx; FM[1] += fyy; FM[2] += fzz;
    FM[3] += py * fzz - pz * fyy;
    FM[4] += pz * fx - px * fzz;
    FM[5] += px * fyy - py * fx;
  }
  return band;
}

// Project a link wrench on the joints 0..l: g_i += z_i . (M - o_i x F).
__device__ __forceinline__ void project(const Twists& tw, int l, const float* FM, float* g) {
#pragma unroll
  for (int i = 0; i < NJ; ++i) {
    if (i > l) break;
    float zi[3], oi[3];
    tw.get(i, zi, oi);
    float tx = FM[3] - (oi[1] * FM[2] - oi[2] * FM[1]);
    float ty = FM[4] - (oi[2] * FM[0] - oi[0] * FM[2]);
    float tz = FM[5] - (oi[0] * FM[1] - oi[1] * FM[0]);
    g[i] += zi[0] * tx + zi[1] * ty + zi[2] * tz;
  }
}

// Sines and cosines of N joint angles.  Below 2^17 the library's sincosf is a
// short straight line; above it reduces the argument by a long one, and with
// both in the code every call is two branches around it, which cost about as
// much as the line itself.  Angles that large only come from a caller's
// seeds: one test for the wavefront takes the short form for all of them
// (the same instructions, hence the same results), or the whole one for all.
template <int N>
__device__ __forceinline__ void sincos_n(const float* q, float* sn, float* cs) {
  constexpr float SHORT = 0x1p17f;
  unsigned most = 0;   // as bits, so that a NaN counts as large
#pragma unroll
  for (int j = 0; j < N; ++j) most = max(most, __float_as_uint(q[j]) & 0x7FFFFFFFu);
  if (__any(most >= __float_as_uint(SHORT))) {
    // (one copy of the long form: the angles pass through it in turn)
    float x[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      x[j] = q[j];
      sn[j] = cs[j] = 0.f;
    }
#pragma unroll 1
    for (int k = 0; k < N; ++k) {
      float s, c;
      sincosf(x[0], &s, &c);
#pragma unroll
      for (int j = 0; j + 1 < N; ++j) {
        x[j] = x[j + 1];
        sn[j] = sn[j + 1];
        cs[j] = cs[j + 1];
      }
      sn[N - 1] = s;
      cs[N - 1] = c;
    }
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const bool is_short = __builtin_fabsf(q[j]) < SHORT;
      __builtin_assume(is_short);
      sincosf(q[j], &sn[j], &cs[j]);
    }
  }
}

// The next frame of the chain: (R, p) of a link from its predecessor's and the
// link's fixed transform F, turned by the joint (sine sn, cosine cs).  One
// row of it (row r of R, component r of p):
__device__ __forceinline__ void frame_row(const float* F, float sn, float cs, float* R, float& p) {
  float A[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) A[c] = R[0] * F[c] + R[1] * F[4 + c] + R[2] * F[8 + c];
  p = R[0] * F[3] + R[1] * F[7] + R[2] * F[11] + p;
  R[0] = cs * A[0] + sn * A[1];
  R[1] = cs * A[1] - sn * A[0];
  R[2] = A[2];
}

// The kinematics of q by a full team: the twists of every joint on return,
// the frames' rows in tm.kin.  `between` runs while three wavefronts form the
// frames (work of the others that needs no frame).  Every wavefront calls it.
template <class Between>
__device__ __forceinline__ void team_kinematics(const Team& tm, const float* q, Twists& tw,
                                                Between between) {
  const int lane = threadIdx.x & (WAVE - 1);
  DS_LDS float* kin = lds(tm.kin) + lane;
  // rows on wavefronts 4..6: three different SIMDs, beside wavefronts that
  // wait, and not that of the smoothness (3)
  constexpr int ROW0 = 4;
  const int r = tm.w - ROW0;
  if (r >= 0 && r < 3) {
    float4 F[NJ][3];
#pragma unroll
    for (int l = 0; l < NJ; ++l)
#pragma unroll
      for (int k = 0; k < 3; ++k) F[l][k] = s_frame[3 * l + k];
    float sn[NJ], cs[NJ];
    sincos_n<NJ>(q, sn, cs);
    float R[3] = {r == 0 ? 1.f : 0.f, r == 1 ? 1.f : 0.f, r == 2 ? 1.f : 0.f}, p = 0.f;
#pragma unroll
    for (int l = 0; l < NJ; ++l) {
      frame_row(&F[l][0].x, sn[l], cs[l], R, p);
      kin[(KIN_ZO + 6 * l + r) * WAVE] = R[2];
      kin[(KIN_ZO + 6 * l + 3 + r) * WAVE] = p;
      kin[(KIN_XY + 6 * l + 2 * r) * WAVE] = R[0];
      kin[(KIN_XY + 6 * l + 2 * r + 1) * WAVE] = R[1];
    }
  } else {
    between();
  }
  tm.sync();
#pragma unroll
  for (int l = 0; l < NJ; ++l)
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      tw.z[l][r] = kin[(KIN_ZO + 6 * l + r) * WAVE];
      tw.o[l][r] = kin[(KIN_ZO + 6 * l + 3 + r) * WAVE];
    }
}

// A link's frame from the team's rows (R whole).
__device__ __forceinline__ void team_frame(const Team& tm, const Twists& tw, int l, float* R,
                                           float* p) {
  const DS_LDS float* kin = lds(tm.kin) + (threadIdx.x & (WAVE - 1));
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    R[3 * r] = kin[(KIN_XY + 6 * l + 2 * r) * WAVE];
    R[3 * r + 1] = kin[(KIN_XY + 6 * l + 2 * r + 1) * WAVE];
    R[3 * r + 2] = tw.z[l][r];
    p[r] = tw.o[l][r];
  }
}

// Self-collision share of this lane (App. A.6 C_self): every pair of spheres
// on links at least two apart, hinge on D = |c_a - c_b| - r_a - r_b; the
// pairs of each link pair are split over the W*L copies.  Forces go into
// per-link wrenches that are projected on the joint axes at the end.
// Inlined, with the frames of the sweep before it: as a function of its own it
// formed them again and, taking the parameters by reference, put the whole
// tile context in scratch memory, where every gather of the sweep read its
// descriptor lane by lane.  A call is bound by latency and instruction fetch:
// 64 trajectories of 47 waypoints with 56 spheres and two swept samples, with
// gradient: 92 us as that function, 39 us here.
// Spheres on their links' axes (AXIS) need the twists only; else xy[l] holds
// the first two columns of R of link l, by rows.
// A pair's distance is compared squared first, with a margin well above its
// rounding: pairs out of reach in the whole wavefront (they add zeros) take
// neither the root nor the rest.  (The negated test lets NaN through.)
template <int MODE, bool AXIS>
__device__ __forceinline__ void self_pairs(const ParamsDev& P, const Links& ln, const Twists& tw,
                                           const float (*xy)[6], int cp, int LW, bool active,
                                           float& selfsum, float& clr, float* g) {
  constexpr bool GRAD = (MODE == EV_GRAD);
  constexpr float MARGIN = 1.00001f;
  float FM[NJ][6];
#pragma unroll
  for (int l = 0; l < NJ; ++l)
#pragma unroll
    for (int k = 0; k < 6; ++k) FM[l][k] = 0.f;
  auto centre = [&](int l, float4 sp, float* c) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      if constexpr (AXIS)
        c[r] = axis_centre(tw.z[l][r], sp.z, tw.o[l][r]);
      else
        c[r] = xy[l][2 * r] * sp.x + xy[l][2 * r + 1] * sp.y + tw.z[l][r] * sp.z + tw.o[l][r];
    }
  };
#pragma unroll
  for (int la = 0; la < NJ; ++la) {
#pragma unroll
    for (int lb = la + 2; lb < NJ; ++lb) {
      const int a0 = ln.begin(la), na = ln.begin(la + 1) - a0;
      const int b0 = ln.begin(lb), nb = ln.begin(lb + 1) - b0;
      // k / nb below: exact, the quotient being under 256 and k + 1/2 at
      // least 1/(2 nb) of a step away from the next whole number
      const float inb = __builtin_amdgcn_rcpf((float)nb);
      for (int k0 = 0; k0 < na * nb; k0 += LW) {
        const int k = min(k0 + cp, na * nb - 1);
        const int ia = (int)(((float)k + 0.5f) * inb), ib = k - ia * nb;
        const float4 sa = s_sph[a0 + ia], sb = s_sph[b0 + ib];
        float ca[3], cb[3];
        centre(la, sa, ca);
        centre(lb, sb, cb);
        float dx = ca[0] - cb[0], dy = ca[1] - cb[1], dz = ca[2] - cb[2];
        const float d2 = dx * dx + dy * dy + dz * dz;
        const float reach = sa.w + sb.w + P.eps;
        const bool mine = active & (k0 + cp < na * nb);
        const bool near = mine & (MODE == EV_RESULT || !(d2 >= reach * reach * MARGIN));
        if (!__any(near)) continue;
        if (near) {
          float dist = sqrtf(d2);
          float D = dist - sa.w - sb.w;
          float De = D - P.eps;
          float phi = (D < P.eps) ? De * De * P.half_inv_eps : 0.f;
          phi = (D < 0.f) ? 0.5f * P.eps - D : phi;
          selfsum += phi;
          if (MODE == EV_RESULT) clr = fminf(clr, D);
          if (GRAD) {
            float dphi = (D < P.eps) ? De * P.inv_eps : 0.f;
            dphi = (D < 0.f) ? -1.f : dphi;
            float w = (dist > 0.f) ? P.ws * dphi / dist : 0.f;
            float fx = w * dx, fy = w * dy, fz = w * dz;
            FM[la][0] += fx; FM[la][1] += fy; FM[la][2] += fz;
            FM[la][3] += ca[1] * fz - ca[2] * fy;
            FM[la][4] += ca[2] * fx - ca[0] * fz;
            FM[la][5] += ca[0] * fy - ca[1] * fx;
            FM[lb][0] -= fx; FM[lb][1] -= fy; FM[lb][2] -= fz;
            FM[lb][3] -= cb[1] * fz - cb[2] * fy;
            FM[lb][4] -= cb[2] * fx - cb[0] * fz;
            FM[lb][5] -= cb[0] * fy - cb[1] * fx;
          }
        }
      }
    }
  }
  if (GRAD) {
#pragma unroll
    for (int l = 0; l < NJ; ++l) project(tw, l, FM[l], g);
  }
}

// ... with the frames of q: the team's rows, or the whole chain again where
// some sphere lies off its link's axis.
template <int MODE, bool KIN>
__device__ __forceinline__ void self_collision(const ParamsDev& P, const Links& ln, const Team& tm,
                                               const float* q, const Twists& tw, int cp, int LW,
                                               bool active, float& selfsum, float& clr, float* g) {
  if (ln.all_axis()) {
    self_pairs<MODE, true>(P, ln, tw, nullptr, cp, LW, active, selfsum, clr, g);
    return;
  }
  float xy[NJ][6];
  if constexpr (KIN) {
    const DS_LDS float* kin = lds(tm.kin) + (threadIdx.x & (WAVE - 1));
#pragma unroll
    for (int l = 0; l < NJ; ++l)
#pragma unroll
      for (int k = 0; k < 6; ++k) xy[l][k] = kin[(KIN_XY + 6 * l + k) * WAVE];
  } else {
    float sn[NJ], cs[NJ];
    sincos_n<NJ>(q, sn, cs);
    float R[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f}, p[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int l = 0; l < NJ; ++l) {
      float F[12];
#pragma unroll
      for (int r = 0; r < 3; ++r) *reinterpret_cast<float4*>(F + 4 * r) = s_frame[3 * l + r];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        frame_row(F, sn[l], cs[l], R + 3 * r, p[r]);
        xy[l][2 * r] = R[3 * r];
        xy[l][2 * r + 1] = R[3 * r + 1];
      }
    }
  }
  self_pairs<MODE, false>(P, ln, tw, xy, cp, LW, active, selfsum, clr, g);
}

// A sample's coarse minimum.
__device__ __forceinline__ float coarse_min(const Sampler& S, const float* u) {
  int ci[3];
  cell_of(S, u, ci);
  return coarse_at(S, block_index(S, ci));
}

// The sweep over the chain for one configuration q: FK, this lane's share
// of the sphere samples (hinge sum into phisum, min clearance into clr) and,
// with GRAD, the link wrenches projected on the joint axes into g.  On
// return R, p hold the frame of link 7 and tw the joint twists.
// KIN: the twists are there already (a full team's shared kinematics), and
// R, p are left alone.
// A sample whose coarse block holds no node nearer than radius + eps (+
// margin) has a zero hinge (a trilinear blend stays within its corners'
// range): it loads no record.  EXACT: no sample is tested (for plans that
// gather them all; with the tests made and not used these take up to 5 %
// longer, and a branch around the tests costs the other plans 1 to 4 %).
// PIPE (every lane holds at most one sphere of each link, W*L >= spheres
// per link): the tests of all links, then their record loads, then the
// hinges, so one memory round trip covers the whole configuration.
// Otherwise each link is processed in chunks of CH spheres per lane, with
// the next link's frame formed while the last chunk's records are on their
// way.  The tests are straight lines: their table and coarse reads from LDS
// are in flight together, where a branch per sample made each of them wait
// for its own two (lanes without a sample go through the motions with the
// last sphere of the table at the most).
template <int MODE, bool PIPE, bool KIN, bool SMALL, bool EXACT>
__device__ __forceinline__ void sweep(const ParamsDev& P, const Sampler& S, const float* q, int cp,
                                      int LW, const Team& tm, Twists& tw, float* R, float* p,
                                      float& phisum, float& clr, float* g, int& ng, bool active) {
  constexpr bool GRAD = (MODE == EV_GRAD);
  // the result pass gathers every sample: the clearance is a minimum over
  // all of them
  const bool SKIP = MODE != EV_RESULT && !EXACT && P.skip;
  const Links ln = S.ln;
  float sn[NJ], cs[NJ];
  // the frame of link l from that of its predecessor
  auto fixed = [&](int l, float* F) {
#pragma unroll
    for (int r = 0; r < 3; ++r) *reinterpret_cast<float4*>(F + 4 * r) = s_frame[3 * l + r];
  };
  auto advance_by = [&](int l, const float* F) {
#pragma unroll
    for (int r = 0; r < 3; ++r) frame_row(F, sn[l], cs[l], R + 3 * r, p[r]);
    tw.put(l, R, p);
  };
  auto advance = [&](int l) {
    float F[12];
    fixed(l, F);
    advance_by(l, F);
  };
  if constexpr (!KIN) {
    sincos_n<NJ>(q, sn, cs);
    R[0] = 1.f; R[1] = 0.f; R[2] = 0.f; R[3] = 0.f; R[4] = 1.f; R[5] = 0.f;
    R[6] = 0.f; R[7] = 0.f; R[8] = 1.f;
    p[0] = p[1] = p[2] = 0.f;
  }
  if constexpr (PIPE) {
    // the lane's sample of every link: sphere, grid position, coarse minimum,
    // record
    int sk[NJ];
    float oz[NJ], r[NJ], u[NJ][3], cm[NJ];
    bool use[NJ];
#pragma unroll
    for (int l = 0; l < NJ; ++l) {
      // copy cp takes sphere (cp - rot) mod LW of the link (LW: a power of
      // two), rot advancing by the longest link's sphere count from link to
      // link: when there are more copies than spheres, consecutive links
      // land on different copies and the samples spread evenly over the
      // wavefronts
      sk[l] = ln.begin(l) + ((cp - l * ln.most()) & (LW - 1));
      use[l] = active & (sk[l] < ln.begin(l + 1));   // lanes past the horizon gather nothing
      sk[l] = min(sk[l], ln.last());
      oz[l] = s_sph[sk[l]].z;
      r[l] = s_sph[sk[l]].w;
    }
#pragma unroll
    for (int l = 0; l < NJ; ++l) {
      if constexpr (!KIN) advance(l);
      axis_pos(link_grid(S, tw.z[l], tw.o[l]), oz[l], u[l]);
      if (!KIN && !ln.axis(l)) frame_pos(S, R, p, s_sph[sk[l]], u[l]);
    }
    if (KIN && !ln.all_axis()) {
#pragma unroll
      for (int l = 0; l < NJ; ++l) {
        if (ln.axis(l)) continue;
        float Rl[9], pl[3];
        team_frame(tm, tw, l, Rl, pl);
        frame_pos(S, Rl, pl, s_sph[sk[l]], u[l]);
      }
    }
#pragma unroll
    for (int l = 0; l < NJ; ++l) cm[l] = coarse_min(S, u[l]);
#pragma unroll
    for (int l = 0; l < NJ; ++l) use[l] &= !(SKIP & (cm[l] >= r[l] + P.far));
    // issue the record loads of the samples that can reach the hinge
    float4 ra[NJ], rz[NJ];
#pragma unroll
    for (int l = 0; l < NJ; ++l) {
      if (use[l]) {
        int ci[3];
        cell_of(S, u[l], ci);
        const int off = record_offset(S, ci);
        ra[l] = load_rec(S, off);
        rz[l] = load_rec(S, off + 16);
        ++ng;
      }
    }
#pragma unroll
    for (int l = 0; l < NJ; ++l) {
      float FM[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      bool forced = false;
      if (use[l])
        forced = sphere_term<MODE>(P, S, u[l], ra[l], rz[l], r[l], phisum, clr, FM);
      // a link with no force in this wavefront has a zero wrench
      // everywhere: its projection would add zeros
      if (GRAD && __any(forced)) project(tw, l, FM, g);
    }
  } else {
    constexpr int C = KIN ? 2 : CH;   // (a full team has eight copies at least)
    // SMALL (teams of 2 and 4, and robots with bare links): a team's later
    // wavefronts run out of a link's spheres before its first one does, and make
    // fewer tests: what counts is left from their own first copy on; where
    // nothing is, or on a link without spheres, the next frame is formed at
    // once, its fixed transform being read ahead.  (50 iterations of 10 seeds
    // with nine spheres on some links: W = 2 893 us with a branch per sample,
    // 908 with the tests in straight lines, 887 from the first copy on; W = 4
    // 700, 718 and 704.  30 iterations of 300 seeds of 32 waypoints, 0, 1, 17,
    // 3, 0, 9 and 0 spheres on the links: W = 1 718, 765 and 699, W = 2 657,
    // 710 and 642, W = 4 557, 622 and 554, W = 8 750, 766 and 642.  One
    // wavefront per seed of a robot with spheres on every link has nothing to
    // gain and loses 1 to 4 % to the longer code, a full team 1 to 2 %.)
    const int cp0 = SMALL ? __builtin_amdgcn_readfirstlane(cp) : 0;
    if constexpr (!KIN) advance(0);
#pragma unroll
    for (int l = 0; l < NJ; ++l) {
      const int s1 = ln.begin(l + 1);
      if (KIN && SMALL && ln.begin(l) >= s1) continue;
      const LinkGrid lg = link_grid(S, tw.z[l], tw.o[l]);
      if (KIN && !ln.axis(l)) team_frame(tm, tw, l, R, p);
      float FM[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      bool forced = false;   // some sample of this link added a force
      // this lane takes every (W*L)-th sphere of the link
      int s = ln.begin(l);
      float Fn[12];
      if (SMALL && !KIN && l + 1 < NJ) fixed(l + 1, Fn);
      do {
        int sk[C];
        float oz[C], r[C], u[C][3], cm[C];
        bool use[C], some = false;
        float4 ra[C], rz[C];
        auto test = [&](auto count) {
          constexpr int N = decltype(count)::value;
#pragma unroll
          for (int k = 0; k < N; ++k) {
            sk[k] = s + k * LW + cp;
            use[k] = active & (sk[k] < s1);
            sk[k] = min(sk[k], ln.last());
            oz[k] = s_sph[sk[k]].z;
            r[k] = s_sph[sk[k]].w;
          }
#pragma unroll
          for (int k = 0; k < N; ++k) axis_pos(lg, oz[k], u[k]);
          if (!ln.axis(l)) {
#pragma unroll
            for (int k = 0; k < N; ++k) frame_pos(S, R, p, s_sph[sk[k]], u[k]);
          }
#pragma unroll
          for (int k = 0; k < N; ++k) cm[k] = coarse_min(S, u[k]);
#pragma unroll
          for (int k = 0; k < N; ++k) use[k] &= !(SKIP & (cm[k] >= r[k] + P.far));
        };
#pragma unroll
        for (int k = 0; k < C; ++k) use[k] = false;
        if (!SMALL || s < s1 - cp0) {   // (else no sphere for this wavefront)
          if (C == 2 || s + 2 * LW < s1 - cp0)
            test(std::integral_constant<int, C>());
          else if (!SMALL || s + LW < s1 - cp0)   // at most two spheres per lane are left
            test(std::integral_constant<int, 2>());
          else
            test(std::integral_constant<int, 1>());
#pragma unroll
          for (int k = 0; k < C; ++k) {
            some |= use[k];
            if (use[k]) {
              int ci[3];
              cell_of(S, u[k], ci);
              const int off = record_offset(S, ci);
              ra[k] = load_rec(S, off);
              rz[k] = load_rec(S, off + 16);
              ++ng;
            }
          }
        }
        s += LW * C;
        if constexpr (!KIN)
          if (l + 1 < NJ && s >= s1) {
            if constexpr (SMALL)
              advance_by(l + 1, Fn);
            else
              advance(l + 1);
          }
        if (__any(some)) {
#pragma unroll
          for (int k = 0; k < C; ++k)
            if (use[k])
              forced |= sphere_term<MODE>(P, S, u[k], ra[k], rz[k], r[k], phisum, clr, FM);
          // every load of the chunk has been consumed: saying so keeps the
          // next chunk's loads in flight together.  (The loads and their uses
          // sit in separate wavefront-uniform branches, so without it the
          // compiler cannot tell which of them are outstanding at the loop's
          // back edge and drains them all before each sphere's loads.)
          __builtin_amdgcn_s_waitcnt(WAIT_VMEM_ALL);
        }
      } while (s < s1);
      // a link with no force in this wavefront has a zero wrench everywhere:
      // its projection would add zeros
      if (GRAD && __any(forced)) project(tw, l, FM, g);
    }
  }
}

// One evaluation of the objective at this lane's configuration q (its
// waypoint) and, with swept sub-samples, at the configurations interpolated
// towards the next waypoint.
template <int MODE, bool PIPE, bool EXT, bool KIN, bool SMALL, bool EXACT>
__device__ __forceinline__ EvalOut evaluate(const RobotDev* __restrict__ rb,
                                            const ParamsDev& P, const Sampler& S, const float* q,
                                            int t, int T, int G, bool active,
                                            Team& tm) {
  constexpr bool GRAD = (MODE == EV_GRAD);
  // the L = 64/G lanes holding the same waypoint in each of the W
  // wavefronts split its spheres: copy index and stride
  const int L = WAVE / G;
  const int lane = threadIdx.x & (WAVE - 1);
  const int cp = tm.w * L + lane / G;
  const int LW = tm.W * L;
  EvalOut o;
  o.ng = 0;
  o.perr = o.rerr = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) o.g[j] = 0.f;
  float phisum = 0.f, clr = FLT_MAX;
  // goal pose, joint limits and smoothness: the same for every copy of the
  // waypoint, so one wavefront of the team computes each and only its first
  // copy adds them to its share before the sums below -- the goal on the
  // second wavefront, the limits on the third and the smoothness on the
  // fourth (off the first one's path; smaller teams fold them onto fewer
  // wavefronts), except in the result pass, whose goal errors the first
  // one writes
  const int xg = (MODE == EV_RESULT || tm.W == 1) ? 0 : 1;
  const int xl = (MODE == EV_RESULT || tm.W < 3) ? xg : 2;
  const int xs = (MODE == EV_RESULT || tm.W < 4) ? xl : 3;
  // a full team's gradient pass forms the goal on the last wavefront, which
  // leaves it in LDS for the sums to add to the second wavefront's share
  constexpr bool FAR_GOAL = KIN && GRAD;
  const int wg = FAR_GOAL ? MAX_TEAM - 1 : xg;
  float ge[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) ge[j] = 0.f;
  float extra_g = 0.f, extra_l = 0.f;
  float R[9], p[3];
  Twists tw;
  static_assert(!KIN || MODE != EV_RESULT, "the result pass keeps its terms on one wavefront");
  // the limits and the smoothness of a full team on their own wavefronts while
  // the frames are formed
  auto own_terms = [&]() {
    if (tm.w == xl) extra_l = limits<GRAD>(rb, P, q, ge);
    if (tm.w == xs) extra_l += smoothness<GRAD>(P, q, t, T, ge);
  };
  if constexpr (!EXT) {
    if constexpr (KIN) team_kinematics(tm, q, tw, own_terms);
    sweep<MODE, PIPE, KIN, SMALL, EXACT>(P, S, q, cp, LW, tm, tw, R, p, phisum, clr, o.g, o.ng, active);
  } else {
    // swept collision: q + tau (q_next - q), tau = i / (nsub + 1), i = 1 ..
    // nsub; the gradient splits (1 - tau) here and tau onto the next
    // waypoint.  Then the waypoint itself, by the same code (a second copy of
    // it would not fit the instruction cache beside the first).
    float qn[NJ], gsh[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      qn[j] = __shfl_down(q[j], 1);
      gsh[j] = 0.f;
    }
    const bool seg = active && t <= T - 2;
    // The tables in LDS are read again in every round: without the statement
    // the compiler reads the frames (84 registers) and the lane's spheres ahead
    // of the loop and, being short of registers, keeps them in scratch memory
    // instead (k_cost for smaller teams: 336 bytes per lane, 140 so; 600
    // trajectories of 12 waypoints, 28 spheres, eight swept samples, with
    // gradient: 142 us, 87 us so).
#pragma unroll 1
    for (int i = 1;; ++i) {
      asm volatile("" ::: "memory");
      const bool own = i > P.nsub;
      const float tau = (float)i / (float)(P.nsub + 1);
      float qi[NJ], gi[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        qi[j] = own ? q[j] : q[j] + tau * (qn[j] - q[j]);
        gi[j] = own ? o.g[j] : 0.f;
      }
      float ph = own ? phisum : 0.f, cl = own ? clr : FLT_MAX;
      if constexpr (KIN) {
        team_kinematics(tm, qi, tw, [&]() {
          if (own) own_terms();
        });
      }
      sweep<MODE, PIPE, KIN, SMALL, EXACT>(P, S, qi, cp, LW, tm, tw, R, p, ph, cl, gi, o.ng, own ? active : seg);
      if (own) {
        phisum = ph;
        clr = cl;
#pragma unroll
        for (int j = 0; j < NJ; ++j) o.g[j] = gi[j];
        break;
      }
      if constexpr (KIN) tm.sync();   // the frames are read before the next ones are formed
      if (seg) {
        phisum += ph;
        clr = fminf(clr, cl);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          o.g[j] += (1.f - tau) * gi[j];
          gsh[j] += tau * gi[j];
        }
      }
      if (GRAD && i == P.nsub) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          float up = __shfl_up(gsh[j], 1);
          o.g[j] += (t >= 1) ? up : 0.f;
        }
      }
    }
  }
  // collision cost share: world hinge sum, plus the self-collision pairs
  // when that term is on
  float coll = P.wc * phisum;
  if (EXT && P.ws != 0.f) {
    float selfsum = 0.f;
    self_collision<MODE, KIN>(P, S.ln, tm, q, tw, cp, LW, active, selfsum, clr, o.g);
    coll += P.ws * selfsum;
  }
  if (tm.w == wg || tm.w == xl || tm.w == xs) {
    const bool first = lane < G;
    const bool last = (t == T - 1);
    if (tm.w == wg) {
    // end effector and goal pose
    // (a full team: the last waypoint's frame in every lane, and joint i's
    // part of the gradient on lane i)
    float zl[3], ol[3];
    if constexpr (KIN) {
      const DS_LDS float* kin = lds(tm.kin) + (T - 1);
      const int i = min(lane, NJ - 1);
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        R[3 * r] = kin[(KIN_XY + 6 * (NJ - 1) + 2 * r) * WAVE];
        R[3 * r + 1] = kin[(KIN_XY + 6 * (NJ - 1) + 2 * r + 1) * WAVE];
        R[3 * r + 2] = kin[(KIN_ZO + 6 * (NJ - 1) + r) * WAVE];
        p[r] = kin[(KIN_ZO + 6 * (NJ - 1) + 3 + r) * WAVE];
        zl[r] = kin[(KIN_ZO + 6 * i + r) * WAVE];
        ol[r] = kin[(KIN_ZO + 6 * i + 3 + r) * WAVE];
      }
    }
    const Goal goal = get_goal();
    float E[12];
#pragma unroll
    for (int r = 0; r < 3; ++r) *reinterpret_cast<float4*>(E + 4 * r) = s_frame[3 * NJ + r];
    float Re[9], pe[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
        Re[3 * r + c] = R[3 * r] * E[c] + R[3 * r + 1] * E[4 + c] + R[3 * r + 2] * E[8 + c];
      pe[r] = R[3 * r] * E[3] + R[3 * r + 1] * E[7] + R[3 * r + 2] * E[11] + p[r];
    }
    float ex = pe[0] - goal.pd[0], ey = pe[1] - goal.pd[1], ez = pe[2] - goal.pd[2];
    float tr = 0.f;
#pragma unroll
    for (int k = 0; k < 9; ++k) tr += goal.Rd[k] * Re[k];
    const float goal_cost = P.wp * (ex * ex + ey * ey + ez * ez) + P.wr * (3.f - tr) * 0.25f;
    extra_g = !FAR_GOAL && last ? goal_cost : 0.f;
    if (GRAD && (KIN || last)) {
      // force 2 w_p e at p_ee and torque -(w_r/4) w, w = vee(M - M^T), M = R_ee R_d^T
      float M[9];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
          M[3 * a + b] = Re[3 * a] * goal.Rd[3 * b] + Re[3 * a + 1] * goal.Rd[3 * b + 1] +
                         Re[3 * a + 2] * goal.Rd[3 * b + 2];
      float wx = M[5] - M[7], wy = M[6] - M[2], wz = M[1] - M[3];
      float k2 = 2.f * P.wp, k4 = -0.25f * P.wr;
      float fx = k2 * ex, fy = k2 * ey, fz = k2 * ez;
      auto part = [&](const float* zi, const float* oi) {
        float rx = pe[0] - oi[0], ry = pe[1] - oi[1], rz = pe[2] - oi[2];
        float tx = ry * fz - rz * fy + k4 * wx;
        float ty = rz * fx - rx * fz + k4 * wy;
        float tz = rx * fy - ry * fx + k4 * wz;
        return zi[0] * tx + zi[1] * ty + zi[2] * tz;
      };
      if constexpr (KIN) {
        DS_LDS float* out = lds(tm.kin) + KIN_GOAL * WAVE;
        if (lane < NJ) out[1 + lane] = part(zl, ol);
        if (lane == NJ) out[0] = goal_cost;
      } else {
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
          float zi[3], oi[3];
          tw.get(i, zi, oi);
          ge[i] += part(zi, oi);
        }
      }
    }
    if (MODE == EV_RESULT) {
      o.perr = sqrtf(ex * ex + ey * ey + ez * ez);
      // angle of R_d^T R_ee: cos = (tr - 1) / 2, sin = |vee(R_ee R_d^T)| / 2
      float M5, M7, M6, M2, M1, M3;
      M5 = Re[3] * goal.Rd[6] + Re[4] * goal.Rd[7] + Re[5] * goal.Rd[8];
      M7 = Re[6] * goal.Rd[3] + Re[7] * goal.Rd[4] + Re[8] * goal.Rd[5];
      M6 = Re[6] * goal.Rd[0] + Re[7] * goal.Rd[1] + Re[8] * goal.Rd[2];
      M2 = Re[0] * goal.Rd[6] + Re[1] * goal.Rd[7] + Re[2] * goal.Rd[8];
      M1 = Re[0] * goal.Rd[3] + Re[1] * goal.Rd[4] + Re[2] * goal.Rd[5];
      M3 = Re[3] * goal.Rd[0] + Re[4] * goal.Rd[1] + Re[5] * goal.Rd[2];
      float wx = M5 - M7, wy = M6 - M2, wz = M1 - M3;
      o.rerr = atan2f(0.5f * sqrtf(wx * wx + wy * wy + wz * wz), 0.5f * (tr - 1.f));
    }
    }
    if constexpr (!KIN) {
      if (tm.w == xl) extra_l = limits<GRAD>(rb, P, q, ge);
      if (tm.w == xs) extra_l += smoothness<GRAD>(P, q, t, T, ge);
    }
    coll += first ? extra_l + extra_g : 0.f;
    if (GRAD) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) o.g[j] += first ? ge[j] : 0.f;
    }
  }
  phisum = coll;
  // a team's gradient pass sums the copies inside its reduce-scatter below
  const bool scatter = GRAD && tm.W > 1;
  // sum the shares of the L lanes of this waypoint (butterfly: every copy
  // ends with the same value)
  if (!scatter)
  for (int off = G; off < WAVE; off <<= 1) {
    phisum = xor_reduce<OpSum>(phisum, off);
    if (MODE == EV_RESULT) clr = xor_reduce<OpMin>(clr, off);
    if (GRAD) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) o.g[j] = xor_reduce<OpSum>(o.g[j], off);
    }
  }
  if (scatter) {
    // ... and of the W wavefronts, summed in wavefront order: wavefront w
    // sums the components c = w mod W of the team (into wavefront 0's row)
    // -- each copy's lanes separately, then the copies by the butterfly --
    // and every wavefront takes the sums
    constexpr int NC = NJ + 1;
    float* base = tm.lds + (tm.buf * tm.W * PART) * WAVE + lane;
    float* mine = base + tm.w * PART * WAVE;
    mine[0] = phisum;
#pragma unroll
    for (int j = 0; j < NJ; ++j) mine[(1 + j) * WAVE] = o.g[j];
    tm.sync();
    if constexpr (KIN) {
      // a full team: one component per wavefront, its shares read together
      static_assert(NC == MAX_TEAM, "one component per wavefront");
      float sh[MAX_TEAM];
#pragma unroll
      for (int u = 0; u < MAX_TEAM; ++u) sh[u] = base[(u * PART + tm.w) * WAVE];
      const float goal_part = lds(tm.kin)[KIN_GOAL * WAVE + tm.w];
      sh[1] += lane == T - 1 ? goal_part : 0.f;
      float v = sh[0];
#pragma unroll
      for (int u = 1; u < MAX_TEAM; ++u) v += sh[u];
      for (int off = G; off < WAVE; off <<= 1) v = xor_reduce<OpSum>(v, off);
      base[tm.w * WAVE] = v;
    } else {
      for (int cc = tm.w; cc < NC; cc += tm.W) {
        float v = base[cc * WAVE];
        for (int u = 1; u < tm.W; ++u) v += base[(u * PART + cc) * WAVE];
        for (int off = G; off < WAVE; off <<= 1) v = xor_reduce<OpSum>(v, off);
        base[cc * WAVE] = v;
      }
    }
    tm.sync();
    phisum = base[0];
#pragma unroll
    for (int j = 0; j < NJ; ++j) o.g[j] = base[(1 + j) * WAVE];
    tm.buf ^= 1;
  } else if (tm.W > 1) {
    // (cost and result passes: every wavefront sums all shares)
    float* mine = tm.lds + ((tm.buf * tm.W + tm.w) * PART) * WAVE + lane;
    mine[0] = phisum;
    if (MODE == EV_RESULT) mine[(1 + NJ) * WAVE] = clr;
    tm.sync();
    const float* all = tm.lds + (tm.buf * tm.W * PART) * WAVE + lane;
    if constexpr (KIN) {
      float sh[MAX_TEAM];
#pragma unroll
      for (int u = 0; u < MAX_TEAM; ++u) sh[u] = all[u * PART * WAVE];
      phisum = sh[0];
#pragma unroll
      for (int u = 1; u < MAX_TEAM; ++u) phisum += sh[u];
    } else {
      phisum = all[0];
      if (MODE == EV_RESULT) clr = all[(1 + NJ) * WAVE];
      for (int v = 1; v < tm.W; ++v) {
        const float* pv = all + v * PART * WAVE;
        phisum += pv[0];
        if (MODE == EV_RESULT) clr = fminf(clr, pv[(1 + NJ) * WAVE]);
      }
    }
    tm.buf ^= 1;
  }
  if (MODE == EV_RESULT) o.clr = clr;
  o.cost = active ? phisum : 0.f;
  if (GRAD) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) o.g[j] = (active && t > 0) ? o.g[j] : 0.f;
  }
  return o;
}

// The evaluation form for this team: PIPE when every lane holds at most one
// sphere per link; shared kinematics for a full team (FULL: MAX_TEAM
// wavefronts; SMALL: the optimiser's smaller ones, and any with bare links).
// Full teams have kernels
// of their own: a kernel with both forms pays for both in registers and in
// instruction fetch (100 iterations of 32 seeds in teams of eight: 1060 us,
// 1000 us with the full team's alone).
template <int MODE, bool EXT, bool FULL, bool SMALL = false, bool EXACT = false>
__device__ __forceinline__ EvalOut eval_any(bool pipe, const RobotDev* __restrict__ rb,
                                            const ParamsDev& P, const Sampler& S, const float* q,
                                            int t, int T, int G, bool active,
                                            Team& tm) {
  constexpr bool KIN = FULL && MODE != EV_RESULT;
  if (pipe) return evaluate<MODE, true, EXT, KIN, SMALL, EXACT>(rb, P, S, q, t, T, G, active, tm);
  return evaluate<MODE, false, EXT, KIN, SMALL, EXACT>(rb, P, S, q, t, T, G, active, tm);
}

__device__ __forceinline__ bool use_pipe(const RobotDev* __restrict__ rb, const Team& tm, int G) {
  return tm.W * (WAVE / G) >= rb->max_per_link;
}

// dynamic LDS of a team's evaluation: its partial sums (double buffered) and,
// for a full team, the shared kinematics
inline size_t eval_lds(int W) {
  return W > 1 ? ((size_t)2 * W * PART + (W == MAX_TEAM ? KIN_ROWS : 0)) * WAVE * sizeof(float) : 0;
}
}  // namespace
}  // namespace dsk
