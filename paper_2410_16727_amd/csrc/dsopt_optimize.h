// Device code of the optimiser: L-BFGS directions, the tile loop and the
// persistent kernel (included by the translation units that instantiate it).
#pragma once

#include "dsopt_eval.h"

namespace dsk {
namespace {

struct TileCtx {
  const RobotDev* rb;
  ParamsDev P;
  const ProbDev* pb;
  Sampler S;
  DS_GLOBAL float* st;
  int lane, G, t, T, seed;
  bool owner;    // first copy of the waypoint: writes outputs and traces
  bool pipe;     // all-gathers-in-flight evaluation form
  bool active;   // t < T
};

__device__ __forceinline__ DS_GLOBAL float* col(DS_GLOBAL float* st, int base, int j, int lane) {
  return st + base + j * WAVE + lane;
}

// History ring (rho, y^T y, s, y per slot) of one seed, laid out like the
// tile state's history section: in the tile state (global) for single
// wavefronts, or in LDS for a team for the duration of a launch.
constexpr int H_RHO = 0, H_YY = H_RHO + DS_MAX_HISTORY * WAVE, H_S = H_YY + DS_MAX_HISTORY * WAVE,
              H_Y = H_S + DS_MAX_HISTORY * NJ * WAVE, H_FLOATS = H_Y + DS_MAX_HISTORY * NJ * WAVE;
static_assert(ST_YY - ST_RHO == H_YY && ST_S - ST_RHO == H_S && ST_Y - ST_RHO == H_Y &&
                  ST_FLOATS - ST_RHO == H_FLOATS,
              "history layout must match the tile state");

template <class Ptr>
struct Hist {
  Ptr h;      // base of the history section
  int lane;
  __device__ __forceinline__ float s(int k, int j) const { return h[H_S + (k * NJ + j) * WAVE + lane]; }
  __device__ __forceinline__ float y(int k, int j) const { return h[H_Y + (k * NJ + j) * WAVE + lane]; }
  __device__ __forceinline__ float rho(int k) const { return h[H_RHO + k * WAVE + lane]; }
  __device__ __forceinline__ float yy(int k) const { return h[H_YY + k * WAVE + lane]; }
  __device__ __forceinline__ void push(int k, const float* sv, const float* yv, float r, float q) const {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      h[H_S + (k * NJ + j) * WAVE + lane] = sv[j];
      h[H_Y + (k * NJ + j) * WAVE + lane] = yv[j];
    }
    h[H_RHO + k * WAVE + lane] = r;
    h[H_YY + k * WAVE + lane] = q;
  }
};
using LHist = Hist<float*>;

// The ring in the tile state, read and written through a buffer resource:
// the lane's column is the vector offset and slot and joint a scalar one,
// so an access needs no per-lane 64-bit address arithmetic.  Slots are
// wave-uniform (one seed per wavefront).  Only the first copy's lanes that
// hold a waypoint touch memory for s and y: the other copies read the first
// copy's column (the same bits: every copy carries the same s and y), and
// lanes past the horizon (s = y = 0 there) use an offset past the end of
// the buffer, which reads zeros and drops stores without a memory access.
// rho and y^T y, the same in every lane, are read by all lanes from column
// 0 (one broadcast access).
constexpr int HIST_OFF_NONE = 0x7FFFFF00;
struct BHist {
  __amdgpu_buffer_rsrc_t r;
  int vo;   // column * 4 for loads, or HIST_OFF_NONE
  int vw;   // column * 4 for stores (first copy only), or HIST_OFF_NONE
  __device__ __forceinline__ float ld(int idx) const {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, vo, idx * 4, 0));
  }
  __device__ __forceinline__ float ld0(int idx) const {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, 0, idx * 4, 0));
  }
  __device__ __forceinline__ void st(int idx, float v) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, vw, idx * 4, 0);
  }
  __device__ __forceinline__ float s(int k, int j) const { return ld(H_S + (k * NJ + j) * WAVE); }
  __device__ __forceinline__ float y(int k, int j) const { return ld(H_Y + (k * NJ + j) * WAVE); }
  __device__ __forceinline__ float rho(int k) const { return ld0(H_RHO + k * WAVE); }
  __device__ __forceinline__ float yy(int k) const { return ld0(H_YY + k * WAVE); }
  __device__ __forceinline__ void push(int k, const float* sv, const float* yv, float r, float q) const {
    k = __builtin_amdgcn_readfirstlane(k);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      st(H_S + (k * NJ + j) * WAVE, sv[j]);
      st(H_Y + (k * NJ + j) * WAVE, yv[j]);
    }
    st(H_RHO + k * WAVE, r);
    st(H_YY + k * WAVE, q);
  }
};

// Steepest-descent step scaled so that its largest entry is delta0 (the
// restart direction).
__device__ __forceinline__ void steepest(const TileCtx& c, const float* g, float* d) {
  float gmax = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) gmax = fmaxf(gmax, fabsf(g[j]));
  gmax = grp_max(gmax, c.G);
  const float sc = c.P.delta0 / fmaxf(gmax, 1e-30f);
#pragma unroll
  for (int j = 0; j < NJ; ++j) d[j] = -g[j] * sc;
}

// The largest |d| of the seed.
__device__ __forceinline__ float largest(const TileCtx& c, const float* d) {
  float dn = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) dn = fmaxf(dn, fabsf(d[j]));
  return grp_max(dn, c.G);
}

// A direction's descent test, restart and infinity-norm cap; returns g . d of
// the direction as it is then (formed again only where d was changed).  The
// seed's values are the same in every lane, so the tests are taken
// wave-uniformly, and both reductions run side by side.
__device__ __forceinline__ float restart_and_cap(const TileCtx& c, const float* g, int& cnt,
                                                 float* d) {
  float gtd = grp_sum(dot7(g, d), c.G), dn = largest(c, d);
  bool changed = false;
  if (!__builtin_amdgcn_readfirstlane(gtd < 0.f ? 1 : 0)) {
    cnt = 0;
    steepest(c, g, d);
    dn = largest(c, d);
    changed = true;
  }
  if (__builtin_amdgcn_readfirstlane(dn > c.P.dmax ? 1 : 0)) {
    const float f = c.P.dmax / dn;
#pragma unroll
    for (int j = 0; j < NJ; ++j) d[j] *= f;
    changed = true;
  }
  if (changed) gtd = grp_sum(dot7(g, d), c.G);
  return gtd;
}

// Ring slot of the entry of a given age (0 = newest), 0 <= head < m and
// 0 <= age < m: one conditional wrap, no integer division.
__device__ __forceinline__ int ring_slot(int head, int age, int m) {
  const int s = head - 1 - age;
  return s < 0 ? s + m : s;
}

// a . b with the product of component FIRST (0 or 1) rounded by itself and the
// others fused into the sum.
template <int FIRST>
__device__ __forceinline__ float dot7_from(const float* a, const float* b) {
  float s = a[FIRST] * b[FIRST];
  asm("" : "+v"(s));
  s += a[1 - FIRST] * b[1 - FIRST];
#pragma unroll
  for (int j = 2; j < NJ; ++j) s += a[j] * b[j];
  return s;
}

// L-BFGS direction (two-loop recursion over the history ring),
// steepest-descent restart and infinity-norm cap; returns g . d.  cnt/head are
// the seed's history count and ring head (the same in every lane of the
// wavefront).
template <class H>
__device__ __forceinline__ float direction(const TileCtx& c, const H& hist, const float* g, int& cnt,
                                          int head, float* d) {
  const int m = c.P.m;
  // one seed per wavefront: count and head are wave-uniform
  const int cmax = __builtin_amdgcn_readfirstlane(cnt);
  const int hd = __builtin_amdgcn_readfirstlane(head);
  // A history of all eight entries (all = true, every iteration but the first
  // few; a plan with a shorter memory takes the other form) has no branches on
  // the count of ages (100 iterations of 32 seeds of one wavefront
  // each: 1580 us, 1520 us so).  The products that stay rounded by themselves
  // are stated, so that both forms give the same bits.
  float q[NJ];
  auto recursion = [&](auto all) {
    constexpr bool ALL = decltype(all)::value;
    // the ring's live slots are read once, all loads in flight together,
    // and both passes of the recursion run on registers
    float hs[DS_MAX_HISTORY][NJ], hy[DS_MAX_HISTORY][NJ], hr[DS_MAX_HISTORY];
    float yy_n = 0.f;
#pragma unroll
    for (int k = 0; k < DS_MAX_HISTORY; ++k) {
      if (ALL || k < cmax) {
        const int slot = ring_slot(hd, k, m);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          hs[k][j] = hist.s(slot, j);
          hy[k][j] = hist.y(slot, j);
        }
        hr[k] = hist.rho(slot);
        if (k == 0) yy_n = hist.yy(slot);
      }
    }
    float a[DS_MAX_HISTORY];
#pragma unroll
    for (int j = 0; j < NJ; ++j) q[j] = g[j];
#pragma unroll
    for (int k = 0; k < DS_MAX_HISTORY; ++k) {
      a[k] = 0.f;
      if (ALL || k < cmax) {
        const float sq = k == 0 ? dot7_from<0>(hs[k], q) : dot7_from<1>(hs[k], q);
        const float ak = hr[k] * grp_sum(sq, c.G);
        a[k] = ak;
        asm("" : "+v"(a[k]));
#pragma unroll
        for (int j = 0; j < NJ; ++j) q[j] -= ak * hy[k][j];
      }
    }
    if (ALL || cmax > 0) {
      const float gamma = 1.f / (hr[0] * yy_n);   // s^T y / y^T y
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        q[j] *= gamma;
        asm("" : "+v"(q[j]));
      }
    }
#pragma unroll
    for (int k = DS_MAX_HISTORY - 1; k >= 0; --k) {
      if (ALL || k < cmax) {
        const float b = hr[k] * grp_sum(dot7_from<1>(hy[k], q), c.G);
#pragma unroll
        for (int j = 0; j < NJ; ++j) q[j] += hs[k][j] * (a[k] - b);
      }
    }
  };
  if (cmax == DS_MAX_HISTORY)
    recursion(std::true_type());
  else
    recursion(std::false_type());
  if (cmax > 0) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) d[j] = -q[j];
  } else {
    steepest(c, g, d);
  }
  return restart_and_cap(c, g, cnt, d);
}

// A team's direction block in LDS: the columns of d, the 2m dot products
// of the history with g, and the ring-slot matrices s_a.y_b and y_a.y_b
// (element (a, b) at a * DS_MAX_HISTORY + b).
constexpr int DL_D = 0, DL_AB = NJ * WAVE, DL_SY = DL_AB + 2 * DS_MAX_HISTORY,
              DL_YY = DL_SY + DS_MAX_HISTORY * DS_MAX_HISTORY,
              DL_FLOATS = DL_YY + DS_MAX_HISTORY * DS_MAX_HISTORY;

// The same direction for a team (W > 1), spread over its wavefronts.  The
// two-loop recursion's result written with inner products (ages k = 0
// newest .. cnt-1; a_k = s_k.g, b_k = y_k.g; SY(k,j) = s_k.y_j,
// YY(k,j) = y_k.y_j):
//   alpha_k = rho_k (a_k - sum_{j<k} alpha_j SY(k,j)),
//   beta_k  = rho_k (gamma (b_k - sum_i alpha_i YY(k,i))
//                    + sum_{j>k} (alpha_j - beta_j) SY(j,k)),
//   H g     = gamma g - sum_k gamma alpha_k y_k + sum_k (alpha_k - beta_k) s_k,
// gamma = s_0.y_0 / y_0.y_0.  Wavefront w reduces a_k, b_k of the ages
// k = w mod W; every wavefront then runs the two triangular recurrences
// (lane i < cnt holds row i) and forms the columns j = w mod W of d.  Every
// wavefront ends with bitwise the same d and cnt.
template <class H>
__device__ __forceinline__ float team_direction(const TileCtx& c, const H& hist, const Team& tm,
                                                const float* g, int& cnt, int head, float* d,
                                                DS_LDS float* dl) {
  const int m = c.P.m;
  const int cu = __builtin_amdgcn_readfirstlane(cnt);
  const int hd = __builtin_amdgcn_readfirstlane(head);

  // wavefront w: ages k = w mod W -- a_k, b_k and the newest pair's row and
  // column of the slot matrices (the same values again when nothing was
  // pushed since the last direction; older pairs were formed when the
  // newer of the two was pushed)
  const int s0 = ring_slot(hd, 0, m);
  for (int k = tm.w; k < cu; k += tm.W) {
    const int b = ring_slot(hd, k, m);
    float sv[NJ], yv[NJ], s0v[NJ], y0v[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      sv[j] = hist.s(b, j);
      yv[j] = hist.y(b, j);
      s0v[j] = hist.s(s0, j);
      y0v[j] = hist.y(s0, j);
    }
    const float a = grp_sum(dot7(sv, g), c.G);
    const float bb = grp_sum(dot7(yv, g), c.G);
    const float p0b = grp_sum(dot7(s0v, yv), c.G);   // s_0 . y_k
    const float pb0 = grp_sum(dot7(sv, y0v), c.G);   // s_k . y_0
    const float q0b = grp_sum(dot7(y0v, yv), c.G);   // y_0 . y_k
    if (c.lane == 0) {
      dl[DL_AB + k] = a;
      dl[DL_AB + DS_MAX_HISTORY + k] = bb;
      dl[DL_SY + s0 * DS_MAX_HISTORY + b] = p0b;
      dl[DL_SY + b * DS_MAX_HISTORY + s0] = pb0;
      dl[DL_YY + s0 * DS_MAX_HISTORY + b] = q0b;
      dl[DL_YY + b * DS_MAX_HISTORY + s0] = q0b;
    }
  }
  tm.sync();

  // lane i < cnt holds age i: row i of SY and YY, column i of SY.  Every
  // operand is loaded unconditionally (valid LDS addresses) and entries of
  // ages >= cnt are replaced by zeros, so no stale value reaches a sum.  A
  // history of all eight entries (all = true, every iteration but the first
  // few; a plan with a shorter memory takes the other form) has none, and the
  // lanes past it are not read: no selects, 60 instructions less of a phase
  // bound by issue (100 iterations of 32 seeds in teams of eight: 868 us, 840
  // us so).
  auto columns = [&](auto all) {
    constexpr bool ALL = decltype(all)::value;
    const int li = c.lane < m ? c.lane : 0;
    const bool lrow = ALL || c.lane < cu;
    const int sli = ring_slot(hd, li, m);
    float syr[DS_MAX_HISTORY], syc[DS_MAX_HISTORY], yyr[DS_MAX_HISTORY], rh[DS_MAX_HISTORY];
    float al[DS_MAX_HISTORY], ee[DS_MAX_HISTORY];
    float acc = lrow ? dl[DL_AB + li] : 0.f;
    float bq = lrow ? dl[DL_AB + DS_MAX_HISTORY + li] : 0.f;
#pragma unroll
    for (int k = 0; k < DS_MAX_HISTORY; ++k) {
      const bool v = ALL || k < cu;
      const int sk = ring_slot(hd, ALL || k < m ? k : 0, m);
      const float a = dl[DL_SY + sli * DS_MAX_HISTORY + sk];
      const float b = dl[DL_SY + sk * DS_MAX_HISTORY + sli];
      const float e = dl[DL_YY + sli * DS_MAX_HISTORY + sk];
      const float r = hist.rho(sk);
      syr[k] = (v && lrow) ? a : 0.f;
      syc[k] = (v && lrow) ? b : 0.f;
      yyr[k] = (v && lrow) ? e : 0.f;
      rh[k] = v ? r : 0.f;
    }
    // alpha: forward substitution, one age per step (lane k is final at step k)
#pragma unroll
    for (int k = 0; k < DS_MAX_HISTORY; ++k) {
      al[k] = rh[k] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(acc), k));
      acc -= al[k] * syr[k];
    }
#pragma unroll
    for (int k = 0; k < DS_MAX_HISTORY; ++k) bq -= al[k] * yyr[k];
    const float gamma = cu > 0 ? 1.f / (hist.rho(s0) * hist.yy(s0)) : 0.f;
    // beta: backward substitution from the oldest age
    float acc2 = gamma * bq;
#pragma unroll
    for (int k = DS_MAX_HISTORY - 1; k >= 0; --k) {
      const float be = rh[k] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(acc2), k));
      ee[k] = al[k] - be;
      acc2 += ee[k] * syc[k];
    }
    // the columns j = w mod W of d: all operands loaded before the sums
    for (int j0 = tm.w; j0 < NJ; j0 += tm.W) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j != j0) continue;
        float sv[DS_MAX_HISTORY], yv[DS_MAX_HISTORY];
#pragma unroll
        for (int k = 0; k < DS_MAX_HISTORY; ++k) {
          const int sk = ring_slot(hd, ALL || k < m ? k : 0, m);
          const bool v = ALL || k < cu;
          const float a = hist.s(sk, j), b = hist.y(sk, j);
          sv[k] = v ? a : 0.f;
          yv[k] = v ? b : 0.f;
        }
        float r = gamma * g[j];
        asm("" : "+v"(r));   // a rounded product, whatever is added to it
#pragma unroll
        for (int k = 0; k < DS_MAX_HISTORY; ++k) {
          r += (-gamma * al[k]) * yv[k];
          r += ee[k] * sv[k];
        }
        dl[DL_D + j * WAVE + c.lane] = -r;
      }
    }
  };
  if (cu == DS_MAX_HISTORY)
    columns(std::true_type());
  else
    columns(std::false_type());
  tm.sync();
  if (cu > 0) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) d[j] = dl[DL_D + j * WAVE + c.lane];
  } else {
    steepest(c, g, d);
  }
  return restart_and_cap(c, g, cnt, d);
}

// The slot matrices of the cnt valid ring entries, formed from the ring
// (a team resuming a seed in a later launch): the same grp_sum(dot7(.))
// products the direction forms, so a resumed run is bitwise the same.
template <class H>
__device__ __forceinline__ void team_rebuild_products(const TileCtx& c, const H& hist,
                                                      const Team& tm, int cnt, int head,
                                                      DS_LDS float* dl) {
  const int m = c.P.m;
  const int cu = __builtin_amdgcn_readfirstlane(cnt);
  const int hd = __builtin_amdgcn_readfirstlane(head);
  for (int ka = tm.w; ka < cu; ka += tm.W) {
    const int a = ring_slot(hd, ka, m);
    float sa[NJ], ya[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      sa[j] = hist.s(a, j);
      ya[j] = hist.y(a, j);
    }
    for (int kb = 0; kb < cu; ++kb) {
      const int b = ring_slot(hd, kb, m);
      float yb[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) yb[j] = hist.y(b, j);
      const float v = grp_sum(dot7(sa, yb), c.G);
      const float w = grp_sum(dot7(ya, yb), c.G);
      if (c.lane == 0) {
        dl[DL_SY + a * DS_MAX_HISTORY + b] = v;
        dl[DL_YY + a * DS_MAX_HISTORY + b] = w;
      }
    }
  }
}

__device__ __forceinline__ void trace_row(float* buf, const TileCtx& c, int k, const float* v) {
  if (!buf || !c.owner || c.t >= c.T) return;
  size_t base = (((size_t)k * c.pb->S + c.seed) * c.T + c.t) * NJ;
#pragma unroll
  for (int j = 0; j < NJ; ++j) glb(buf)[base + j] = v[j];
}
__device__ __forceinline__ void trace_scalar(float* buf, const TileCtx& c, int k, float v) {
  if (!buf || !c.owner || c.t != 0) return;
  glb(buf)[(size_t)k * c.pb->S + c.seed] = v;
}

// Final per-seed results and output trajectory.
template <bool EXT, bool FULL>
__device__ __forceinline__ int finalize(const TileCtx& c, const float* x, Team& tm) {
  EvalOut r = eval_any<EV_RESULT, EXT, FULL>(c.pipe, c.rb, c.P, c.S, x, c.t, c.T, c.G, c.active, tm);
  float Jr = grp_sum(r.cost, c.G);
  float clr = grp_min(c.active ? r.clr : FLT_MAX, c.G);
  float perr = grp_sum((c.t == c.T - 1) ? r.perr : 0.f, c.G);
  float rerr = grp_sum((c.t == c.T - 1) ? r.rerr : 0.f, c.G);
  int inlim = 1;
#pragma unroll
  for (int j = 0; j < NJ; ++j) inlim &= (x[j] >= c.rb->qlo[j] && x[j] <= c.rb->qhi[j]) ? 1 : 0;
  float okf = grp_min((c.active && !inlim) ? 0.f : 1.f, c.G);
  // trajectory metrics: largest first, second and third differences
  float vm = 0.f, am = 0.f, jm = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    float q1 = __shfl_down(x[j], 1), q2 = __shfl_down(x[j], 2), q3 = __shfl_down(x[j], 3);
    float v1 = q1 - x[j];
    float v2 = q2 - 2.f * q1 + x[j];
    float v3 = q3 - 3.f * q2 + 3.f * q1 - x[j];
    vm = fmaxf(vm, (c.t + 1 < c.T) ? fabsf(v1) : 0.f);
    am = fmaxf(am, (c.t + 2 < c.T) ? fabsf(v2) : 0.f);
    jm = fmaxf(jm, (c.t + 3 < c.T) ? fabsf(v3) : 0.f);
  }
  vm = grp_max(vm, c.G);
  am = grp_max(am, c.G);
  jm = grp_max(jm, c.G);
  if (c.owner && c.t < c.T) {
    DS_GLOBAL float* ft = glb(c.pb->final_traj) + ((size_t)c.seed * c.T + c.t) * NJ;
#pragma unroll
    for (int j = 0; j < NJ; ++j) ft[j] = x[j];
    if (c.pb->out_traj) {
      DS_GLOBAL float* ot = glb(c.pb->out_traj) + ((size_t)c.seed * c.T + c.t) * NJ;
#pragma unroll
      for (int j = 0; j < NJ; ++j) ot[j] = x[j];
    }
  }
  if (c.owner && c.t == 0) {
    ds_seed_result sr;
    sr.cost = Jr;
    sr.clearance = clr;
    sr.pos_err = perr;
    sr.rot_err = rerr;
    const float dt = c.P.dt;
    sr.max_jerk = jm / (dt * dt * dt);
    sr.max_vel = vm / dt;
    sr.max_acc = am / (dt * dt);
    sr.within_vel = sr.max_vel <= c.P.vlim ? 1 : 0;
    // the uniform slow-down s >= 1 that meets the velocity, acceleration and
    // jerk limits (they scale as 1/s, 1/s^2, 1/s^3)
    const float sc = fmaxf(fmaxf(1.f, sr.max_vel / c.P.vlim),
                           fmaxf(sqrtf(sr.max_acc / c.P.alim), cbrtf(sr.max_jerk / c.P.jlim)));
    sr.motion_time = sc * (float)(c.T - 1) * dt;
    sr.valid = isfinite(Jr) ? 1 : 0;
    sr.collision_free = clr > 0.f ? 1 : 0;
    sr.within_limits = okf > 0.5f ? 1 : 0;
    sr.success = (sr.valid && sr.collision_free && sr.within_limits && perr < c.P.tol_pos &&
                  rerr < c.P.tol_rot) ? 1 : 0;
    sr.n_evals_cost = ((const DS_GLOBAL int*)c.st)[ST_EVC + c.lane];
    sr.n_evals_grad = ((const DS_GLOBAL int*)c.st)[ST_EVG + c.lane];
    // field by field: the implicit struct copy has no global-address form
    DS_GLOBAL ds_seed_result* o = glb(c.pb->seed_res) + c.seed;
    o->cost = sr.cost; o->clearance = sr.clearance; o->pos_err = sr.pos_err;
    o->rot_err = sr.rot_err; o->max_jerk = sr.max_jerk;
    o->collision_free = sr.collision_free; o->within_limits = sr.within_limits;
    o->success = sr.success; o->valid = sr.valid; o->n_evals_cost = sr.n_evals_cost;
    o->n_evals_grad = sr.n_evals_grad;
    o->max_vel = sr.max_vel; o->max_acc = sr.max_acc; o->motion_time = sr.motion_time;
    o->within_vel = sr.within_vel;
  }
  return r.ng;
}

enum { PH_INIT = 0, PH_DIR = 1, PH_TRIAL = 2, PH_ACCEPT = 3 };

// Run up to max_iters iterations of one tile (state persists in the arena).
// The wavefront loops over phases around a single cost+gradient evaluation:
//   INIT   evaluate the seed (first launch of the tile only);
//   DIR    direction from the history, trial point x + d;
//   TRIAL  Armijo test of alpha = 1 (its gradient is already there); further
//          cost-only candidates while a seed of the tile has no Armijo step;
//          if a seed accepted alpha < 1, evaluate there (ACCEPT), else update;
//   ACCEPT take the accepted point's cost and gradient, update.
template <bool LDS_HIST, bool EXT, bool FULL, bool SMALL, bool EXACT>
__device__ __forceinline__ void run_tile(const RobotDev* __restrict__ rb, const ParamsDev* __restrict__ pp,
                         const ProbDev* __restrict__ probs, const TileDev& td, int max_iters,
                         Team& tm, float* hist_lds, uint8_t* coarse_lds, float* dir_lds) {
  TileCtx c;
  c.rb = rb;
  c.P = *pp;
  c.pb = probs + td.prob;
  c.S = make_sampler(c.pb->sc, rb);
  put_goal(*c.pb);
  c.st = glb(td.state);
  c.lane = threadIdx.x & (WAVE - 1);
  c.G = td.G;
  c.t = c.lane & (c.G - 1);
  c.T = c.pb->T;
  c.seed = td.seed0;
  c.owner = tm.w == 0 && c.lane < c.G;
  c.pipe = use_pipe(rb, tm, c.G);
  c.active = c.t < c.T;
  const bool writer = tm.w == 0;   // the team's first wavefront writes state
  const int n_iters = c.pb->n_iters;
  DS_GLOBAL int* sti = (DS_GLOBAL int*)c.st;
  const ProbDev& pb = *c.pb;
  // the trace buffers are all set or all null: one flag per tile, so the
  // iteration does not reload the pointers
  const bool tracing = pb.tr_x != nullptr;

  float x[NJ], g[NJ], d[NJ], xe[NJ], gt[NJ];
  float J = 0.f, Jt = 0.f, gtd = 0.f, alpha = 0.f;
  int cnt, head, evc, evg, chosen = 0;
  int ngath = 0;   // cell records gathered by this lane in this launch
  int iter = sti[ST_ITER + c.lane];
  int phase;
  // a tile whose initial evaluation ran in an earlier launch (iteration 0,
  // one gradient evaluation counted) resumes from its state like any other
  if (iter == 0 && sti[ST_EVG + c.lane] == 0) {
    if (c.active) {
      const DS_GLOBAL float* sp = glb(pb.seeds) + ((size_t)c.seed * c.T + c.t) * NJ;
#pragma unroll
      for (int j = 0; j < NJ; ++j) xe[j] = (c.t == 0) ? pb.qs[j] : sp[j];
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j) xe[j] = 0.f;
    }
    cnt = head = evc = evg = 0;
    phase = PH_INIT;
  } else {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      x[j] = *col(c.st, ST_X, j, c.lane);
      g[j] = *col(c.st, ST_G, j, c.lane);
    }
    J = c.st[ST_J + c.lane];
    cnt = sti[ST_CNT + c.lane];
    head = sti[ST_HEAD + c.lane];
    evc = sti[ST_EVC + c.lane];
    evg = sti[ST_EVG + c.lane];
    phase = PH_DIR;
  }
  int n_left = min(max_iters, n_iters - iter);
  // the history ring: LDS copy for a team, else the tile state
  typename std::conditional<LDS_HIST, LHist, BHist>::type hist;
  // the scene's coarse table: shared by the team, else this wavefront's own
  c.S.cm = lds(coarse_lds);
  if constexpr (LDS_HIST) {
    hist.lane = c.lane;
    hist.h = hist_lds;
    if (iter > 0 && n_left > 0) {   // resume: bring the ring into LDS
      const DS_GLOBAL float* src = c.st + ST_RHO;
      for (int i = threadIdx.x; i < H_FLOATS; i += tm.W * WAVE) hist_lds[i] = src[i];
    }
    if (c.P.skip) stage_coarse(pb.sc, lds(coarse_lds), threadIdx.x, tm.W * WAVE);
    tm.sync();
    // the slot matrices of a resumed ring (read after the direction's first
    // barrier)
    if (iter > 0 && n_left > 0) team_rebuild_products(c, hist, tm, cnt, head, lds(dir_lds));
  } else {
    hist.r = __builtin_amdgcn_make_buffer_rsrc((void*)(float*)(c.st + ST_RHO), (short)0,
                                               (int)(H_FLOATS * sizeof(float)), RSRC_DWORD3);
    hist.vo = c.active ? (c.lane & (c.G - 1)) * 4 : HIST_OFF_NONE;
    hist.vw = (c.active && c.lane < c.G) ? c.lane * 4 : HIST_OFF_NONE;
    // one wavefront: its LDS accesses complete in order, no barrier needed
    if (c.P.skip) stage_coarse(pb.sc, lds(coarse_lds), c.lane, WAVE);
  }

  for (;;) {
    if (phase == PH_DIR) {
      if (n_left <= 0) break;
      if (tracing) {
        trace_row(pb.tr_x, c, iter, x);
        trace_row(pb.tr_g, c, iter, g);
        trace_scalar(pb.tr_J, c, iter, J);
      }
      if constexpr (LDS_HIST) {
        gtd = team_direction(c, hist, tm, g, cnt, head, d, lds(dir_lds));
      } else {
        gtd = direction(c, hist, g, cnt, head, d);
      }
      if (tracing) trace_row(pb.tr_d, c, iter, d);
#pragma unroll
      for (int j = 0; j < NJ; ++j) xe[j] = x[j] + d[j];
      phase = PH_TRIAL;
    }
    // the one cost+gradient evaluation of this pass
    EvalOut e = eval_any<EV_GRAD, EXT, FULL, SMALL, EXACT>(c.pipe, rb, c.P, c.S, xe, c.t, c.T, c.G,
                                                    c.active, tm);
    ++evg;
    ngath += e.ng;
    const float Je = grp_sum(e.cost, c.G);
    if (phase == PH_INIT) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) { x[j] = xe[j]; g[j] = e.g[j]; }
      J = Je;
      phase = PH_DIR;
      continue;
    }
    bool update_now = true;
    if (phase == PH_TRIAL) {
      Jt = Je;
#pragma unroll
      for (int j = 0; j < NJ; ++j) gt[j] = e.g[j];
      chosen = (Jt <= J + c.P.c1 * gtd) ? 0 : -1;
      float Jmin = Jt;
      int kmin = 0;
      for (int kk = 1; kk < c.P.nls; ++kk) {
        bool need = chosen < 0;
        if (!__any(need)) break;
        float al = ldexpf(1.f, -kk);
        float xk[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) xk[j] = x[j] + al * d[j];
        EvalOut ek = eval_any<EV_COST, EXT, FULL, SMALL, EXACT>(c.pipe, rb, c.P, c.S, xk, c.t, c.T, c.G,
                                                         c.active, tm);
        ++evc;
        ngath += ek.ng;
        float Jk = grp_sum(ek.cost, c.G);
        if (need && Jk <= J + c.P.c1 * al * gtd) chosen = kk;
        if (need && Jk < Jmin) { Jmin = Jk; kmin = kk; }
      }
      if (chosen < 0 && Jmin < J) chosen = kmin;
      alpha = chosen >= 0 ? ldexpf(1.f, -chosen) : 0.f;
      if (__any(chosen > 0)) {
        // evaluate the accepted step (seeds that took alpha = 1 recompute
        // the same point and keep their trial values)
        float al = chosen > 0 ? alpha : 1.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) xe[j] = x[j] + al * d[j];
        phase = PH_ACCEPT;
        update_now = false;
      }
    } else {   // PH_ACCEPT
      if (chosen > 0) {
        Jt = Je;
#pragma unroll
        for (int j = 0; j < NJ; ++j) gt[j] = e.g[j];
      }
    }
    if (!update_now) continue;
    // history update and step
    if (tracing) trace_scalar(pb.tr_a, c, iter, alpha);
    if (__builtin_amdgcn_readfirstlane(chosen) >= 0) {
      float s[NJ], y[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float xn = x[j] + alpha * d[j];
        s[j] = xn - x[j];
        y[j] = gt[j] - g[j];
        asm("" : "+v"(y[j]));   // a rounded difference, whatever is formed from it
      }
      float sy = grp_sum(dot7(s, y), c.G);
      float ss = grp_sum(dot7(s, s), c.G);
      float yy = grp_sum(dot7(y, y), c.G);
      if (__builtin_amdgcn_readfirstlane(sy > 1e-10f * sqrtf(ss) * sqrtf(yy) ? 1 : 0)) {
        if (writer) hist.push(head, s, y, 1.f / sy, yy);
        head = head + 1 == c.P.m ? 0 : head + 1;
        cnt = min(cnt + 1, c.P.m);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) { x[j] = x[j] + alpha * d[j]; g[j] = gt[j]; }
      J = Jt;
    } else {
      cnt = 0;
    }
    ++iter;
    --n_left;
    phase = PH_DIR;
    tm.sync();   // the writer's history is visible to the team
  }
  // persist the state (a team writes its LDS ring back for a later launch)
  if constexpr (LDS_HIST) {
    if (iter < n_iters) {
      DS_GLOBAL float* dst = c.st + ST_RHO;
      for (int i = threadIdx.x; i < H_FLOATS; i += tm.W * WAVE) dst[i] = hist_lds[i];
    }
  }
  if (writer) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      *col(c.st, ST_X, j, c.lane) = x[j];
      *col(c.st, ST_G, j, c.lane) = g[j];
    }
    c.st[ST_J + c.lane] = J;
    sti[ST_CNT + c.lane] = cnt;
    sti[ST_HEAD + c.lane] = head;
    sti[ST_ITER + c.lane] = iter;
    sti[ST_EVC + c.lane] = evc;
    sti[ST_EVG + c.lane] = evg;
  }
  if (iter == n_iters) {
    trace_row(pb.tr_x, c, iter, x);
    trace_row(pb.tr_g, c, iter, g);
    trace_scalar(pb.tr_J, c, iter, J);
    ngath += finalize<EXT, FULL>(c, x, tm);
  }
  // this launch's gathers into the seed's counter: every lane adds its own
  // count.  No lane-dependent branch here -- one at the end of the tile body
  // turns the persistent tile loop into a divergent loop, and the wavefront's
  // tile fetch below must run with the whole wavefront.
  __hip_atomic_fetch_add(&glb(pb.seed_res)[c.seed].n_gathers, (unsigned)ngath,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The next tile for this workgroup: from one atomic counter over the
// whole table, or -- with per-XCD queues (xcd_ranges[x] .. xcd_ranges[x+1]
// is queue x, counter[x] its position) -- from the queue of the XCD the
// workgroup runs on (workgroups are dispatched to the 8 XCDs in turn), so
// a problem's tiles, and its scene's records, stay in one XCD's L2; an
// exhausted queue sends the workgroup on to the others.  -1: nothing left.
__device__ __forceinline__ int next_tile(int* counter, const int* __restrict__ xcd_ranges,
                                         int nt) {
  if (!xcd_ranges) {
    const int i = atomicAdd(counter, 1);
    return i < nt ? i : -1;
  }
  const int home = (int)(blockIdx.x % N_XCD);
  for (int q = 0; q < N_XCD; ++q) {
    const int x = (home + q) % N_XCD;
    const int b = xcd_ranges[x], len = xcd_ranges[x + 1] - b;
    if (len <= 0) continue;
    const int i = atomicAdd(&counter[x], 1);
    if (i < len) return b + i;
  }
  return -1;
}

// Persistent optimiser: every team (W = 1: every wavefront) takes tiles
// (next_tile) until the table is exhausted (tile_list, if given, indirects
// the table; n_tiles_dev, if given, overrides n_tiles).  Every member of a
// team sees the same tile sequence and the same decisions, so all of them
// reach every barrier.  Variants: TEAM (W > 1, history ring in LDS), FULL
// (W = 8, shared kinematics), SMALL and EXACT (see the sweep) and EXT
// (self-collision and swept terms compiled in); the plain variant carries no
// code for the optional terms.
template <bool TEAM, bool EXT, bool FULL, bool SMALL, bool EXACT = false>
__global__ void __launch_bounds__(TEAM ? MAX_TEAM * WAVE : BLOCK, TEAM ? 1 : 2)
k_optimize(const RobotDev* __restrict__ rb, const ParamsDev* __restrict__ pp,
           const ProbDev* __restrict__ probs, const TileDev* __restrict__ tiles,
           const int* __restrict__ tile_list, const int* __restrict__ n_tiles_dev, int n_tiles,
           int* counter, int max_iters, const int* __restrict__ max_iters_dev,
           const int* __restrict__ xcd_ranges) {
  extern __shared__ float s_dyn[];
  __shared__ int s_tile;
  stage_robot(rb);
  const int lane = threadIdx.x & (WAVE - 1);
  const int nt = n_tiles_dev ? *n_tiles_dev : n_tiles;
  if (max_iters_dev) max_iters = *max_iters_dev;   // serving: set per replay
  Team tm;
  tm.W = TEAM ? pp->waves : 1;
  // wave-uniform (scalar) index, so loops over a wavefront's share stay scalar
  tm.w = TEAM ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE)) : 0;
  tm.lds = s_dyn;
  tm.kin = FULL ? s_dyn + 2 * tm.W * PART * WAVE + H_FLOATS + COARSE_FLOATS + DL_FLOATS : nullptr;
  tm.buf = 0;
  for (;;) {
    int mine = 0;
    if constexpr (TEAM) {
      if (threadIdx.x == 0) s_tile = next_tile(counter, xcd_ranges, nt);
      __syncthreads();
      mine = s_tile;
      __syncthreads();
    } else {
      // one fetch per wavefront, by its first active lane, broadcast from
      // that lane (correct for any set of active lanes)
      const int first = __ffsll((long long)__ballot(1)) - 1;
      if (lane == first) mine = next_tile(counter, xcd_ranges, nt);
      mine = __builtin_amdgcn_readfirstlane(__shfl(mine, first));
    }
    if (mine < 0) break;
    const int ti = tile_list ? tile_list[mine] : mine;
    TileDev td = tiles[ti];
    if constexpr (TEAM) {
      run_tile<true, EXT, FULL, SMALL, EXACT>(rb, pp, probs, td, max_iters, tm, s_dyn + 2 * tm.W * PART * WAVE,
                                reinterpret_cast<uint8_t*>(s_dyn + 2 * tm.W * PART * WAVE + H_FLOATS),
                                s_dyn + 2 * tm.W * PART * WAVE + H_FLOATS + COARSE_FLOATS);
      __syncthreads();   // the LDS ring is free for the next tile
    } else {
      // this wavefront's coarse table (uniform)
      const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
      run_tile<false, EXT, FULL, SMALL, EXACT>(rb, pp, probs, td, max_iters, tm, nullptr,
                                 reinterpret_cast<uint8_t*>(s_dyn + wv * COARSE_FLOATS), nullptr);
    }
  }
}

using OptKernel = void (*)(const RobotDev*, const ParamsDev*, const ProbDev*, const TileDev*,
                           const int*, const int*, int, int*, int, const int*, const int*);

template <bool EXT>
OptKernel optimize_variant(int W) {
  if (W == MAX_TEAM) return k_optimize<true, EXT, true, false>;
  return W > 1 ? k_optimize<true, EXT, false, true> : k_optimize<false, EXT, false, false>;
}

}  // namespace
}  // namespace dsk
