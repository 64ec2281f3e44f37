// gfx950 kernels that make a scene resident: the distance field from an
// occupancy grid, and a field's gather layout (8-corner cell records and the
// coarse table of block minima).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>

#include "dsopt_internal.h"

namespace dsk {
namespace {

// ------------------------------------------------------ records and table --
// One workgroup makes the records of a run of up to PACK_BLOCKS coarse blocks
// (2^shift cells per axis; a part of a row along x, or whole rows, or whole
// layers: a run in the table's order in any case) and their table entries, so
// that the field is read once for both.  A thread owns a block's column of
// cells along z: it keeps the plane of four nodes it has and loads the next
// one (four loads per record instead of eight), writes the 32-byte record, and
// adds the column's minimum to its block's in LDS.
//
// Table entry: the minimum node value m over the block's cells (the far
// faces included: a cell's corners), kept as the 4-bit level L = the largest
// L <= 15 with L * cq <= m (0 for a negative m), two blocks per byte, the
// even block (linear index bx + cdx (by + cdy bz)) in the low nibble.  The
// workgroup that owns a byte's even block writes the byte; where the odd one
// is not in its run it forms that block's minimum from the nodes as well, so
// no byte has two writers and the table needs no clearing.
//
// Bound: HBM, 36 bytes a cell (4 read, 32 written).  200^3, behind the kernel
// that wrote the field: 56 us, 5.1 TB/s of the 5.2 a large copy reaches here
// (one thread per record and a second kernel that read the field again for the
// table: 54 + 33 us, and 5 us to clear it).  Stores past the caches: 146.
constexpr int PACK_BLOCKS = 32;
constexpr int PACK_THREADS = 512;
constexpr int PACK_Z = 4;

// Records that the memory-side cache does not hold are written to memory in the
// order of the workgroups.
bool past_cache(int nx, int ny, int nz) {
  return (long long)(nx - 1) * (ny - 1) * (nz - 1) * 32 > 256 << 20;
}

// Blocks of a workgroup along each axis: about a column of cells per thread.
// Of a long row a part, of an even number of blocks; of short ones as many
// rows, and then layers, as fill the threads.  With whole rows for every
// workgroup, grids thin in x left most threads idle (4 x 4 x 100000: 86 us a
// call, 20 so; 3 x 700 x 700: 106 and 21), and larger ones had too few
// workgroups, or rows cut into a long and a short part of which one half of
// the XCDs got all the long ones (400^3: 884 us, 730 so; 300 x 250 x 200: 248
// and 163).  Parts of four times that, 400^3: 893 us, 300 x 250 x 200: 186;
// of half, 186 for the latter; of blocks thin in y as many as fill the threads
// (500000 x 2 x 9: 56 us a call with two blocks of 32 cells, 39 so).  A whole
// row where one per workgroup comes to about the same number for every CU and
// the records stay in the cache (196 x 185 x 154, 460 rows: 35 us of the
// kernel, 43 in parts; 155 x 137 x 147, 342 rows: 25 and 24; 256^3, 1024 rows:
// 188 and 158).
struct PackTile {
  int x, y, z;
};
PackTile pack_tile(int nx, int ny, int nz, int shift, int cdx, int cdy, int cdz, int cu_count) {
  const int b = 1 << shift;
  const int most = std::clamp(PACK_THREADS / (b * std::min(b, ny - 1)), 2, PACK_BLOCKS);
  if (cdx > most) {
    const int rows = cdy * cdz, slots = (rows + cu_count - 1) / cu_count * cu_count;
    if (cdx <= PACK_BLOCKS && !past_cache(nx, ny, nz) && rows >= 0.85 * slots) return {cdx, 1, 1};
    const int parts = (cdx + most - 1) / most, each = (cdx + parts - 1) / parts;
    return {each + (each & 1), 1, 1};
  }
  const int columns = (nx - 1) * std::min(b, ny - 1);   // of a row of blocks
  PackTile t{cdx, std::max(1, std::min({cdy, PACK_BLOCKS / cdx, PACK_THREADS / columns})), 1};
  if (t.y == cdy)
    t.z = std::max(1, std::min({cdz, PACK_BLOCKS / (cdx * cdy), PACK_THREADS / ((nx - 1) * (ny - 1))}));
  return t;
}

// Whether the records and the table get a kernel each.  Past the cache the
// records are best written in their own order, at the price of a second reading
// of the field:
// 40 x 600 x 700 230 us in one pass, 126 + 38 in two; 204^3 84, 53 + 14;
// 700 x 600 x 40 185, 137 + 23.  Not where the one pass keeps its lanes busy,
// by the columns of its tiles and the last round of its workgroups (256^3 148,
// 140 + 23; 400^3 701, 637 + 90; equal at about 0.85 of the lanes), or where
// every row of records begins at a cache line, which no two workgroups then
// share (741 x 377 x 140 380, 379 + 54).  Below 256 MB: 215 x 85 x 416 54,
// 51 + 14; 128^3 16, 15 + 5.
bool pack_apart(int nx, int ny, int nz, int shift, const PackTile& t, int parts, int cdy, int cdz,
                int cu_count) {
  const int cx = nx - 1, cy = ny - 1;
  if (!past_cache(nx, ny, nz) || cx % 4 == 0 || t.z > 1) return false;
  // lanes that the workgroups have, and those with a column
  const int rows = (cdy + t.y - 1) / t.y;
  const int w = parts > 1 ? t.x << shift : cx, wl = cx - (parts - 1) * w;
  const int h = rows > 1 ? t.y << shift : cy, hl = cy - (rows - 1) * h;
  auto lanes = [](long long a, long long b) {
    return (a * b + PACK_THREADS - 1) / PACK_THREADS * PACK_THREADS;
  };
  const long long all = (parts - 1) * ((rows - 1) * lanes(w, h) + lanes(w, hl)) +
                        (rows - 1) * lanes(std::max(wl, 0), h) + lanes(std::max(wl, 0), hl);
  const long long slots = 2048 / PACK_THREADS * (long long)cu_count;
  const long long wgs = (long long)parts * rows * cdz;
  const double busy = (double)cx * cy / all * wgs / ((wgs + slots - 1) / slots * slots);
  return busy < 0.86;
}

// Order-preserving integer key of a float (for a minimum by LDS atomics).
__device__ __forceinline__ int min_key(float v) {
  const int i = __float_as_int(v);
  return i < 0 ? i ^ 0x7FFFFFFF : i;
}
__device__ __forceinline__ float key_value(int k) {
  return __int_as_float(k < 0 ? k ^ 0x7FFFFFFF : k);
}

__device__ __forceinline__ unsigned level_of(float m, float cq) {
  if (!(m >= 0.f)) return 0;
  unsigned L = (unsigned)fminf(floorf(m / cq), 15.f);
  while (L > 0 && (float)L * cq > m) --L;   // the quotient may have rounded up
  return L;
}

// The blocks of a workgroup, [bx0, bx0 + bxn) x [by0, by0 + byn) x
// [bz0, bz0 + bzn): [first, last) in the table's order.  (A row's parts begin at
// even indices of the table, but for the first; the last, shorter ones of the
// rows are dealt to the XCDs in turn.)
struct PackRun {
  int bx0, by0, bz0, bxn, byn, bzn, first, last;
};
template <bool LAYERS>
__device__ __forceinline__ PackRun pack_run(const PackTile& tile, int cdx, int cdy, int cdz) {
  PackRun r;
  r.by0 = blockIdx.y * tile.y;
  r.byn = min(tile.y, cdy - r.by0);
  r.bz0 = LAYERS ? blockIdx.z * tile.z : blockIdx.z;
  r.bzn = LAYERS ? min(tile.z, cdz - r.bz0) : 1;
  r.bx0 = 0;
  r.bxn = cdx;
  if (gridDim.x > 1) {
    const int part = (blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x;
    const int odd = (cdx * (r.by0 + cdy * r.bz0)) & 1;
    r.bx0 = max(part * tile.x - odd, 0);
    r.bxn = min((part + 1) * tile.x - odd, cdx) - r.bx0;
  }
  r.first = r.bx0 + cdx * (r.by0 + cdy * r.bz0);
  r.last = r.first + r.bxn * r.byn * r.bzn;
  return r;
}

// The minima of a run's blocks and of the one after them.
__shared__ int s_min[PACK_BLOCKS + 1];
__device__ __forceinline__ void clear_minima() {
  for (int i = threadIdx.x; i < PACK_BLOCKS + 1; i += PACK_THREADS) s_min[i] = min_key(FLT_MAX);
  __syncthreads();
}

// The bytes whose even block is one of this workgroup's, once its threads have
// added their columns.
__device__ __forceinline__ void put_levels(const PackRun& r, const float* __restrict__ v, int nx,
                                           int ny, int nz, int shift, int cdx, int cdy, int cdz,
                                           float cq, uint8_t* __restrict__ table) {
  // the odd block after the run, if that byte is its own
  if ((r.last & 1) && r.last < cdx * cdy * cdz) {
    const int ex = r.last % cdx, ey = (r.last / cdx) % cdy, ez = r.last / (cdx * cdy);
    const int ex0 = ex << shift, ey0 = ey << shift, ez0 = ez << shift;
    const int lx = min((ex + 1) << shift, nx - 1) - ex0 + 1,
              ly = min((ey + 1) << shift, ny - 1) - ey0 + 1,
              lz = min((ez + 1) << shift, nz - 1) - ez0 + 1;
    float m = FLT_MAX;
    for (int e = threadIdx.x; e < lx * ly * lz; e += PACK_THREADS) {
      const int i = e % lx, j = (e / lx) % ly, k = e / (lx * ly);
      m = fminf(m, v[(size_t)(ex0 + i) + (size_t)nx * (ey0 + j) + (size_t)nx * ny * (ez0 + k)]);
    }
    for (int off = 1; off < WAVE; off <<= 1) m = fminf(m, __shfl_xor(m, off));
    if ((threadIdx.x & (WAVE - 1)) == 0) atomicMin(&s_min[r.last - r.first], min_key(m));
  }
  __syncthreads();
  for (int b = (r.first + 1) / 2 + threadIdx.x; 2 * b < r.last; b += PACK_THREADS) {
    const int e = 2 * b - r.first;
    const unsigned lo = level_of(key_value(s_min[e]), cq);
    const unsigned hi = 2 * b + 1 < cdx * cdy * cdz ? level_of(key_value(s_min[e + 1]), cq) : 0u;
    table[b] = (uint8_t)(lo | (hi << 4));
  }
}

template <bool LAYERS>
__global__ void __launch_bounds__(PACK_THREADS)
k_esdf_pack(const float* __restrict__ v, int nx, int ny, int nz, int shift, int cdx, int cdy,
            int cdz, PackTile tile, float cq, float4* __restrict__ rec,
            uint8_t* __restrict__ table) {
  const int cx = nx - 1, cy = ny - 1, cz = nz - 1;
  const PackRun run = pack_run<LAYERS>(tile, cdx, cdy, cdz);
  if (run.bxn <= 0) return;
  const int x0 = run.bx0 << shift, xn = min((run.bx0 + run.bxn) << shift, cx) - x0;
  const int y0 = run.by0 << shift, yn = min((run.by0 + run.byn) << shift, cy) - y0;
  clear_minima();
  const size_t row = nx, plane = (size_t)nx * ny;
  for (int c = threadIdx.x; c < xn * yn * run.bzn; c += PACK_THREADS) {
    const int q = c / xn, xi = c - q * xn, zi = LAYERS ? q / yn : 0, yi = q - zi * yn;
    const int x = x0 + xi, y = y0 + yi;
    const int z0 = (run.bz0 + zi) << shift, z1 = min((run.bz0 + zi + 1) << shift, cz);
    const float* p = v + x + row * y + plane * z0;
    float a0 = p[0], a1 = p[1], a2 = p[row], a3 = p[row + 1];
    float m = FLT_MAX;   // (fminf drops NaN nodes)
    float4* r = rec + 2 * ((size_t)x + (size_t)cx * ((size_t)y + (size_t)cy * z0));
    const size_t step = 2 * (size_t)cx * cy;
    for (int z = z0; z < z1; z += PACK_Z) {
      // PACK_Z planes' loads in flight together
      float b[PACK_Z][4];
#pragma unroll
      for (int k = 0; k < PACK_Z; ++k) {
        const float* q = p + plane * min(z + k + 1 - z0, z1 - z0);
        b[k][0] = q[0]; b[k][1] = q[1]; b[k][2] = q[row]; b[k][3] = q[row + 1];
      }
#pragma unroll
      for (int k = 0; k < PACK_Z; ++k, r += step) {
        if (z + k < z1) {
          r[0] = make_float4(a0, a1, a2, a3);
          r[1] = make_float4(b[k][0], b[k][1], b[k][2], b[k][3]);
        }
        m = fminf(m, fminf(fminf(a0, a1), fminf(a2, a3)));
        a0 = b[k][0]; a1 = b[k][1]; a2 = b[k][2]; a3 = b[k][3];
      }
    }
    m = fminf(m, fminf(fminf(a0, a1), fminf(a2, a3)));
    atomicMin(&s_min[(xi >> shift) + run.bxn * ((yi >> shift) + run.byn * zi)], min_key(m));
  }
  put_levels(run, v, nx, ny, nz, shift, cdx, cdy, cdz, cq, table);
}

// The records alone, one per thread in their own order.  Bound: HBM
// (40 x 600 x 700, 588 MB: 126 us, 4.7 TB/s).
constexpr int RECORD_THREADS = 256;
__global__ void __launch_bounds__(RECORD_THREADS)
k_esdf_records(const float* __restrict__ v, int nx, int ny, unsigned cells, float4* __restrict__ rec) {
  const unsigned r = blockIdx.x * RECORD_THREADS + threadIdx.x;   // (below 2^26)
  if (r >= cells) return;
  const unsigned cx = nx - 1, cy = ny - 1;
  const unsigned q = r / cx, x = r - q * cx, z = q / cy, y = q - z * cy;
  const size_t row = nx, plane = (size_t)nx * ny;
  const float *p = v + x + row * y + plane * z, *n = p + plane;
  rec[2 * (size_t)r] = make_float4(p[0], p[1], p[row], p[row + 1]);
  rec[2 * (size_t)r + 1] = make_float4(n[0], n[1], n[row], n[row + 1]);
}

// The table alone: a thread per column of nodes, which adds its minimum to
// every block that has it (two along an axis on their common face).  Bound:
// latency of one column's loads (40 x 600 x 700, 67 MB: 38 us; a workgroup per
// block and a thread per node took 44, and 5 to clear the table).
__global__ void __launch_bounds__(PACK_THREADS)
k_esdf_table(const float* __restrict__ v, int nx, int ny, int nz, int shift, int cdx, int cdy,
             int cdz, PackTile tile, float cq, uint8_t* __restrict__ table) {
  const PackRun run = pack_run<false>(tile, cdx, cdy, cdz);
  if (run.bxn <= 0) return;
  const int x0 = run.bx0 << shift, xn = min((run.bx0 + run.bxn) << shift, nx - 1) - x0 + 1;
  const int y0 = run.by0 << shift, yn = min((run.by0 + run.byn) << shift, ny - 1) - y0 + 1;
  const int z0 = run.bz0 << shift, zn = min((run.bz0 + 1) << shift, nz - 1) - z0 + 1;
  clear_minima();
  const size_t row = nx, plane = (size_t)nx * ny;
  const int in_block = (1 << shift) - 1;
  for (int c = threadIdx.x; c < xn * yn; c += PACK_THREADS) {
    const int yi = c / xn, xi = c - yi * xn;
    const float* p = v + (x0 + xi) + row * (y0 + yi) + plane * z0;
    float m = FLT_MAX;
    for (int z = 0; z < zn; z += 8) {
      float b[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) b[k] = p[plane * min(z + k, zn - 1)];
#pragma unroll
      for (int k = 0; k < 8; ++k) m = fminf(m, b[k]);
    }
    const int bx = xi >> shift, by = yi >> shift;
    const bool lx = (xi & in_block) == 0 && xi > 0, ly = (yi & in_block) == 0 && yi > 0;
    const bool hx = bx < run.bxn, hy = by < run.byn;
    if (hx && hy) atomicMin(&s_min[bx + run.bxn * by], min_key(m));
    if (lx && hy) atomicMin(&s_min[bx - 1 + run.bxn * by], min_key(m));
    if (hx && ly) atomicMin(&s_min[bx + run.bxn * (by - 1)], min_key(m));
    if (lx && ly) atomicMin(&s_min[bx - 1 + run.bxn * (by - 1)], min_key(m));
  }
  put_levels(run, v, nx, ny, nz, shift, cdx, cdy, cdz, cq, table);
}

// ---------------------------------------------- ESDF from an occupancy grid --
// Exact squared Euclidean distance transform by separable passes (along x,
// y and z), f'(p) = min over q on the line of f(q) + (p - q)^2 in voxels.
// Every value is an integer below 2^24 (or the "none" sentinel), so float
// arithmetic is exact.
//
// Both signs in one field: a free voxel needs the distance to the occupied
// ones and an occupied voxel that to the free ones, and its other distance
// is zero.  One signed float per voxel therefore holds both fields --
// positive the squared distance of a free voxel, negative that of an
// occupied one -- and max(+-f, 0) is either field.
//
// Along y and z a line is done by divide and conquer: the position q that
// minimises f(q) + (p - q)^2 does not decrease with p, so once the
// minimisers of every (4 S)-th position are known, the positions between
// two of them need only the range between theirs.  Strides 64, 16, 4, 1 make
// about 14 candidates per voxel for a line of 200, whatever the distances
// are (a scan outward from p takes twice the distance, the whole line where
// the line holds no obstacle).  The positions of one gap are scanned
// together, so one LDS read serves three or four of them, and a block of
// candidates whose smallest value cannot win is passed over: a wavefront
// takes as long as its widest range, and wide ranges lie where the nearest
// surface changes, with little between.
//
// Bound: VALU of the candidates (half of the issue slots; the rest is the
// latency of one round of workgroups, five per CU).  200^3 shelf scene: bits
// 6 us, x and y 54 us, z 50 us; before, with a field for each sign and a scan
// outward from every voxel, six passes of 27 to 428 us (829 together) and
// 50 us of kernels around them.
constexpr float EDT_NONE = 1e20f;
// Lines of a workgroup, side by side along x, and its threads.
constexpr int EDT_X = 32, EDT_THREADS = 256;
// ... where such workgroups would be a quarter of the CUs or fewer, and a thread
// of them would have more than one gap of four positions: the time is then that
// of one workgroup, whose threads take the gaps in turn.  A quarter of the
// lines and four times the threads, and still no more than one workgroup per
// CU.  8 x 8 x 1024, half of the voxels
// occupied: z pass 159 us, 27 so (256 threads with 8 lines: 48; 1024 with 32:
// 73); 2 x 200 x 200: 39 and 18.  With more workgroups the narrow ones lose
// what their short rows cost in memory and in barriers (100^3, 313 workgroups
// of 32 lines: 29 us, 52 narrow; 1024 x 1024 x 16: 146 and 1660).
constexpr int EDT_XN = 8, EDT_THREADSN = 1024;
bool edt_narrow(int n, long long workgroups, int cu_count) {
  return n > 4 * (EDT_THREADS / EDT_X) && 4 * workgroups <= cu_count;
}

// Candidates per block: the block minima fit into LDS beside a line of 1024.
__host__ __device__ inline int edt_block_shift(int n) { return n <= 512 ? 3 : 4; }

// In LDS, X lines side by side, element [i * X + column]: the candidates s[q],
// q < n; the minimum of each block of 2^bs of them, signed like them (0 where
// the block holds both kinds: a zero of either field); the minimisers of the
// positions that are multiples of four.
template <int X_>
struct EdtLines {
  static constexpr int X = X_;
  float *s, *blk;
  unsigned short* opt;
  int n, bs, col;
  __device__ __forceinline__ EdtLines(float* lds, int n_)
      : s(lds), n(n_), bs(edt_block_shift(n_)), col((int)threadIdx.x % X) {
    blk = s + n * X;
    opt = reinterpret_cast<unsigned short*>(blk + (((n - 1) >> bs) + 1) * X);
  }
  __device__ __forceinline__ float at(int q) const { return s[q * X + col]; }
};

size_t edt_lds(int n, int x) {
  return (size_t)x * ((n + ((n - 1) >> edt_block_shift(n)) + 1) * sizeof(float) +
                      (n + 3) / 4 * sizeof(unsigned short));
}

// A row of a tile of k_edt_xy: its word, and the nearest occupied and free
// position before and after that word.
struct EdtRow {
  unsigned own;
  short po, pf, no, nf;
};
size_t edt_xy_lds(int ny, int x) {
  return std::max(edt_lds(ny, x), (size_t)ny * (x * sizeof(float) + sizeof(EdtRow)));
}

// N positions p0 + i step of one field (sg > 0: that of the free voxels):
// the smallest sum of each so far and, with ARG, where.  With d = q - p0 a
// sum is f(q) + d^2 - 2 i step d + (i step)^2; the last part is added at the
// end, so a candidate costs a multiply-add and a minimum for each position.
template <int N, bool ARG>
struct EdtBest {
  float p0, step, sg, best[N];
  int arg[N];
  __device__ __forceinline__ EdtBest(int p0_, int step_, float sg_)
      : p0((float)p0_), step((float)step_), sg(sg_) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      best[i] = FLT_MAX;
      arg[i] = 0;
    }
  }
  template <class Lines>
  __device__ __forceinline__ void take(const Lines& L, int q) {
    const float d = (float)q - p0, c0 = fmaf(d, d, fmaxf(sg * L.at(q), 0.f));
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float c = i ? fmaf(-2.f * i * step, d, c0) : c0;
      if (ARG) arg[i] = c < best[i] ? q : arg[i];
      best[i] = fminf(best[i], c);
    }
  }
  __device__ __forceinline__ float sum(int i) const {
    return fmaf(i * step, i * step, best[i]);
  }
  // The candidates of block b, unless its smallest value at its nearest
  // place to the positions is no less than the largest sum so far.  All of
  // them, eight reads in flight, also where only some were asked for: more
  // candidates never change a minimum.
  template <class Lines>
  __device__ __forceinline__ void block(const Lines& L, int b) {
    const float q0 = (float)(b << L.bs), q1 = q0 + (float)((1 << L.bs) - 1);
    const float d = fmaxf(fmaxf(q0 - (p0 + (N - 1) * step), p0 - q1), 0.f);
    float most = best[0];
#pragma unroll
    for (int i = 1; i < N; ++i) most = fmaxf(most, sum(i));
    if (fmaf(d, d, fmaxf(sg * L.blk[b * Lines::X + L.col], 0.f)) >= most) return;
    for (int q = b << L.bs; q < (b + 1) << L.bs; q += 8) {
#pragma unroll
      for (int k = 0; k < 8; ++k) take(L, min(q + k, L.n - 1));
    }
  }
};

// The N positions p0, p0 + step, ... (those before n): put(i, sum, minimiser)
// of each in the field its own kind needs, over the candidates between the
// minimisers of a and b (b past the end: the end of the line).  An a or b of
// the other kind is a zero of that field, and so its own minimiser.
template <int N, bool ARG, class Lines, class Put>
__device__ __forceinline__ void edt_gap(const Lines& L, int a, int b, int p0, int step,
                                        Put put) {
  const bool past = b >= L.n;
  const int be = past ? L.n - 1 : b;
  const bool fa = L.at(a) > 0.f, fb = past || L.at(be) > 0.f;
  const int oa = L.opt[(a >> 2) * Lines::X + L.col];
  const int ob = past ? be : L.opt[(be >> 2) * Lines::X + L.col];
  bool fr[N], some = false, other = false;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int p = p0 + i * step;
    fr[i] = L.at(min(p, L.n - 1)) > 0.f;
    some |= p < L.n && fr[i];
    other |= p < L.n && !fr[i];
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const bool field = t == 0;
    if (!(field ? some : other)) continue;
    const int lo = fa == field ? oa : a, hi = fb == field ? ob : be;
    EdtBest<N, ARG> r(p0, step, field ? 1.f : -1.f);
    r.take(L, lo);
    r.take(L, hi);
    if (lo + 1 < hi)
      for (int k = (lo + 1) >> L.bs; k <= (hi - 1) >> L.bs; ++k) r.block(L, k);
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (fr[i] == field && p0 + i * step < L.n) put(i, field ? r.sum(i) : -r.sum(i), r.arg[i]);
  }
}

// All lines of the workgroup: put(p, signed minimum) for every position.
// Every thread must call it, after s is filled.
template <int THREADS, class Lines, class Put>
__device__ __forceinline__ void edt_lines(const Lines& L, Put put) {
  constexpr int X = Lines::X, ROWS = THREADS / X;
  const int n = L.n, g0 = threadIdx.x / X, nb = ((n - 1) >> L.bs) + 1;
  __syncthreads();
  for (int b = g0; b < nb; b += ROWS) {
    const int q1 = min(n, (b + 1) << L.bs);
    float mo = EDT_NONE, mf = EDT_NONE;   // minima of the two fields
    for (int q = b << L.bs; q < q1; ++q) {
      const float v = L.at(q);
      mo = fminf(mo, fmaxf(v, 0.f));
      mf = fminf(mf, fmaxf(-v, 0.f));
    }
    L.blk[b * X + L.col] = mo - mf;   // one of them is zero
  }
  __syncthreads();
  // every 64th position: its block, then outward while a block is near enough
  for (int p = g0 * 64; p < n; p += ROWS * 64) {
    const float v = L.at(p);
    EdtBest<1, true> r(p, 0, v > 0.f ? 1.f : -1.f);
    r.best[0] = fabsf(v);
    r.arg[0] = p;
    const int b0 = p >> L.bs;
    r.block(L, b0);
    for (int k = 1; k < nb; ++k) {
      const float d = (float)(((k - 1) << L.bs) + 1);   // the nearest voxel of block b0 +- k
      if (d * d >= r.best[0]) break;
      if (b0 - k >= 0) r.block(L, b0 - k);
      if (b0 + k < nb) r.block(L, b0 + k);
    }
    L.opt[(p >> 2) * X + L.col] = (unsigned short)r.arg[0];
  }
  __syncthreads();
  for (int S = 16; S >= 4; S >>= 2) {
    for (int a = g0 * 4 * S; a + S < n; a += ROWS * 4 * S) {
      edt_gap<3, true>(L, a, a + 4 * S, a + S, S, [&](int i, float, int arg) {
        L.opt[((a + (i + 1) * S) >> 2) * X + L.col] = (unsigned short)arg;
      });
    }
    __syncthreads();
  }
  for (int a = g0 * 4; a < n; a += ROWS * 4) {
    edt_gap<4, false>(L, a, a + 4, a, 1, [&](int i, float f, int) { put(a + i, f); });
  }
}

// Occupancy as bits: 2 * ceil(nx / 64) words of 32 voxels per row.  A lane
// reads four voxels (rows start at any byte, so these are unaligned words;
// only a row's last, partial one is read byte by byte) and eight lanes join
// their four bits each to a word.  BITS_ROWS rows' loads are in flight
// together: the kernel is a round or two of memory latency for the grid.
constexpr int BITS_ROWS = 4;
__global__ void __launch_bounds__(EDT_THREADS)
k_edt_bits(const uint8_t* __restrict__ occ, int nx, int rows, unsigned* __restrict__ bits) {
  const int lane = threadIdx.x & (WAVE - 1), words = 2 * ((nx + WAVE - 1) / WAVE);
  const int r0 = (blockIdx.x * (EDT_THREADS / WAVE) +
                  __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE))) * BITS_ROWS;
  for (int x = 4 * lane; x < 32 * words; x += 4 * WAVE) {
    unsigned v[BITS_ROWS];
#pragma unroll
    for (int r = 0; r < BITS_ROWS; ++r) {
      v[r] = 0;
      if (r0 + r >= rows) continue;
      const uint8_t* p = occ + (size_t)(r0 + r) * nx + x;
      if (x + 4 <= nx) {
        __builtin_memcpy(&v[r], p, 4);
      } else {
        for (int k = 0; x + k < nx; ++k) v[r] |= (unsigned)p[k] << (8 * k);
      }
    }
#pragma unroll
    for (int r = 0; r < BITS_ROWS; ++r) {
      unsigned b = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) b |= (v[r] >> (8 * k) & 255u) ? 1u << k : 0u;
      b <<= 4 * (lane & 7);
      b |= __shfl_xor(b, 1);
      b |= __shfl_xor(b, 2);
      b |= __shfl_xor(b, 4);
      if ((lane & 7) == 0 && r0 + r < rows) bits[(size_t)(r0 + r) * words + x / 32] = b;
    }
  }
}

// Passes along x and y: one workgroup per tile of X columns of one z plane.
// The tile is in one word of each row's bits, so the nearest opposite voxel on
// the row is in that word or is one of four positions that the whole row of
// the tile shares (the nearest occupied and free one before and after the
// word), found by one thread per row.
template <int THREADS, int X>
__global__ void __launch_bounds__(THREADS)
k_edt_xy(const unsigned* __restrict__ bits, int nx, int ny, float* __restrict__ out) {
  extern __shared__ float s_line[];
  const EdtLines<X> L(s_line, ny);
  const int x = blockIdx.x * X + L.col, w0 = blockIdx.x * X / 32;
  const int x0 = w0 * 32, bit = x - x0;   // the tile is in one word of each row
  const int words = 2 * ((nx + WAVE - 1) / WAVE);
  // (the rows are where the block minima and minimisers will be)
  EdtRow* rows = reinterpret_cast<EdtRow*>(L.blk);
  for (int y = threadIdx.x; y < ny; y += THREADS) {
    const unsigned* w = bits + ((size_t)blockIdx.y * ny + y) * words;
    EdtRow r = {w[w0], -2048, -2048, 4096, 4096};
    for (int k = 0; k < w0; ++k) {
      const unsigned o = w[k], f = ~o;
      if (o) r.po = (short)(k * 32 + 31 - __builtin_clz(o));
      if (f) r.pf = (short)(k * 32 + 31 - __builtin_clz(f));
    }
    for (int k = (nx - 1) / 32; k > w0; --k) {
      const unsigned o = w[k], f = ~o & (0xFFFFFFFFu >> max(0, (k + 1) * 32 - nx));
      if (o) r.no = (short)(k * 32 + __builtin_ctz(o));
      if (f) r.nf = (short)(k * 32 + __builtin_ctz(f));
    }
    rows[y] = r;
  }
  __syncthreads();
  const unsigned valid = 0xFFFFFFFFu >> max(0, x0 + 32 - nx), below = (1u << bit) - 1u;
  for (int y = threadIdx.x / X; y < ny; y += THREADS / X) {
    const EdtRow r = rows[y];
    const bool is_occ = (r.own >> bit) & 1;
    const unsigned opp = is_occ ? valid & ~r.own : r.own;
    const unsigned lo = opp & below, hi = opp & ~below;
    const int before = lo ? x0 + 31 - __builtin_clz(lo) : (is_occ ? r.pf : r.po);
    const int after = hi ? x0 + __builtin_ctz(hi) : (is_occ ? r.nf : r.no);
    const int d = min(x - before, after - x);
    // (columns past the row's end get a value that is not used)
    const float v = d < 1024 ? (float)(d * d) : EDT_NONE;
    L.s[y * X + L.col] = is_occ ? -v : v;
  }
  float* o = out + ((size_t)blockIdx.y * ny) * nx + x;
  edt_lines<THREADS>(L, [&](int p, float f) {
    if (x < nx) o[(size_t)p * nx] = f;
  });
}

// Pass along z over X neighbouring lines, and the distance itself: the
// root of the squared distance in metres, negative inside.  In place: a
// workgroup has its lines in LDS before it writes them.  The caller's copy, if
// any, is written beside it, without another pass over the field.
template <int THREADS, int X>
__global__ void __launch_bounds__(THREADS)
k_edt_z(float* f, long long plane, int nz, float voxel, float* copy) {
  extern __shared__ float s_line[];
  const EdtLines<X> L(s_line, nz);
  const long long l = (long long)blockIdx.x * X + L.col;
  const bool in = l < plane;
  for (int z = threadIdx.x / X; z < nz; z += THREADS / X)
    L.s[z * X + L.col] = in ? f[l + z * plane] : 1.f;
  edt_lines<THREADS>(L, [&](int p, float s) {
    if (!in) return;
    const float d = s < 0.f ? -voxel * sqrtf(-s) : voxel * sqrtf(s);
    f[l + p * plane] = d;
    if (copy) copy[l + p * plane] = d;
  });
}

}  // namespace

hipError_t launch_esdf_pack(const float* vals, int nx, int ny, int nz, int shift, int cdx,
                            int cdy, int cdz, float cq, float4* rec, uint8_t* table,
                            int cu_count, hipStream_t s) {
  const PackTile t = pack_tile(nx, ny, nz, shift, cdx, cdy, cdz, cu_count);
  // (in odd rows of an odd length the parts begin one block earlier)
  const int parts = t.x == cdx ? 1 : (cdx + (cdx & 1) + t.x - 1) / t.x;
  const dim3 grid(parts, (cdy + t.y - 1) / t.y, (cdz + t.z - 1) / t.z), block(PACK_THREADS);
  if (!pack_apart(nx, ny, nz, shift, t, parts, cdy, cdz, cu_count)) {
    hipLaunchKernelGGL(t.z > 1 ? k_esdf_pack<true> : k_esdf_pack<false>, grid, block, 0, s, vals,
                       nx, ny, nz, shift, cdx, cdy, cdz, t, cq, rec, table);
    return hipGetLastError();
  }
  const unsigned cells = (unsigned)(nx - 1) * (ny - 1) * (nz - 1);
  hipLaunchKernelGGL(k_esdf_records, dim3((cells + RECORD_THREADS - 1) / RECORD_THREADS),
                     dim3(RECORD_THREADS), 0, s, vals, nx, ny, cells, rec);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  hipLaunchKernelGGL(k_esdf_table, grid, block, 0, s, vals, nx, ny, nz, shift, cdx, cdy, cdz, t, cq,
                     table);
  return hipGetLastError();
}

size_t edt_bits_bytes(int nx, int ny, int nz) {
  return (size_t)((nx + WAVE - 1) / WAVE) * ny * nz * sizeof(unsigned long long);
}

hipError_t launch_esdf_from_occupancy(const uint8_t* occ, int nx, int ny, int nz, float voxel,
                                      unsigned long long* bits, float* dist, float* copy,
                                      int cu_count, hipStream_t s) {
  const long long plane = (long long)nx * ny;
  const int per = EDT_THREADS / WAVE * BITS_ROWS;
  unsigned* words = reinterpret_cast<unsigned*>(bits);
  hipLaunchKernelGGL(k_edt_bits, dim3((ny * nz + per - 1) / per), dim3(EDT_THREADS), 0, s, occ, nx,
                     ny * nz, words);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 xy((nx + EDT_X - 1) / EDT_X, nz), xyn((nx + EDT_XN - 1) / EDT_XN, nz);
  if (edt_narrow(ny, (long long)xy.x * nz, cu_count))
    hipLaunchKernelGGL((k_edt_xy<EDT_THREADSN, EDT_XN>), xyn, dim3(EDT_THREADSN),
                       edt_xy_lds(ny, EDT_XN), s, words, nx, ny, dist);
  else
    hipLaunchKernelGGL((k_edt_xy<EDT_THREADS, EDT_X>), xy, dim3(EDT_THREADS),
                       edt_xy_lds(ny, EDT_X), s, words, nx, ny, dist);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long long z = (plane + EDT_X - 1) / EDT_X, zn = (plane + EDT_XN - 1) / EDT_XN;
  if (edt_narrow(nz, z, cu_count))
    hipLaunchKernelGGL((k_edt_z<EDT_THREADSN, EDT_XN>), dim3((unsigned)zn), dim3(EDT_THREADSN),
                       edt_lds(nz, EDT_XN), s, dist, plane, nz, voxel, copy);
  else
    hipLaunchKernelGGL((k_edt_z<EDT_THREADS, EDT_X>), dim3((unsigned)z), dim3(EDT_THREADS),
                       edt_lds(nz, EDT_X), s, dist, plane, nz, voxel, copy);
  return hipGetLastError();
}

}  // namespace dsk
