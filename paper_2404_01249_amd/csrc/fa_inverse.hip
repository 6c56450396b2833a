// The post hoc inverse of a warp (include/fa_inverse.h): psi = id + e fitted
// to minimise the mean of |psi(phi(x)) - x|^2 + |phi(psi(x)) - x|^2 (Section
// 4.4.3, "Alternative formulations for Eulerian differential") with
// Algorithm 1's loop.  Two kernels of this file form the direction; the
// smoothing, composition and loss record are the registration's kernels.
#include <algorithm>
#include <cmath>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "fa.h"
#include "fa_host.h"
#include "fa_internal.h"
#include "fa_inverse.h"

using fa::clamp_med3;
using fa::Ctl;
using fa::fail;
using fa::Tiling;

namespace {

// The splat accumulates sum_x 2 r1(x) w_j(x + d(x)) in 64-bit integers, in
// units of 2^-32: integer addition is associative, so the sum does not depend
// on the order in which the atomics land.  Each term is clamped to 2^30 in
// magnitude (only non-finite or absurd displacements reach it).
constexpr double kFixScale = 4294967296.0;
constexpr double kFixUnit = 1.0 / 4294967296.0;
constexpr float kFixClamp = 1073741824.0f;
constexpr int kInvThreads = 256;
constexpr int kInvMaxBlocks = 4096;
constexpr int64_t kSmallTileVoxels = 300000;
constexpr int kDirMaxBlocks = 2 * kInvMaxBlocks;   // workgroups of k_inv_direction; one loss partial more

// Trilinear cell of position p on an n0 x n1 x n2 grid: flat corner indices
// and weights in the order (b0, b1, b2) = 000, 001, ..., 111; corners off the
// grid have weight 0 and index 0 (zero extension).
struct Cell {
  int idx[8];
  float w[8];
  float t0, t1, t2;
  unsigned ok;
};

__device__ __forceinline__ Cell cell_of(float p0, float p1, float p2, int n0, int n1, int n2) {
  Cell c;
  const float f0 = floorf(p0), f1 = floorf(p1), f2 = floorf(p2);
  c.t0 = p0 - f0;
  c.t1 = p1 - f1;
  c.t2 = p2 - f2;
  // far outside, the clamp keeps the integers small; every corner is then off the grid anyway
  const int i0 = (int)clamp_med3(f0, -2.0f, (float)n0);
  const int i1 = (int)clamp_med3(f1, -2.0f, (float)n1);
  const int i2 = (int)clamp_med3(f2, -2.0f, (float)n2);
  c.ok = 0u;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int b0 = (k >> 2) & 1, b1 = (k >> 1) & 1, b2 = k & 1;
    const int z = i0 + b0, y = i1 + b1, x = i2 + b2;
    const bool in = z >= 0 && z < n0 && y >= 0 && y < n1 && x >= 0 && x < n2;
    c.idx[k] = in ? (z * n1 + y) * n2 + x : 0;
    c.w[k] = in ? (b0 ? c.t0 : 1.0f - c.t0) * (b1 ? c.t1 : 1.0f - c.t1) * (b2 ? c.t2 : 1.0f - c.t2) : 0.0f;
    c.ok |= in ? (1u << k) : 0u;
  }
  return c;
}

__device__ __forceinline__ float sample(const float* __restrict__ f, const Cell& c) {
  float s = 0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) s += ((c.ok >> k) & 1u) ? c.w[k] * f[c.idx[k]] : 0.0f;
  return s;
}

// The same cell as four rows of two neighbouring corners: where the pair starts
// (clamped onto the grid, so that both of its loads are in bounds), and which
// corners are on the grid.
struct PairCell {
  int off[4];          // rows (b0, b1) = 00, 01, 10, 11
  bool upper, lower;   // the pair was clamped: its second (first) value is the first (second) corner's
  unsigned ok;
  float t0, t1, t2;
};

__device__ __forceinline__ PairCell pair_cell(float p0, float p1, float p2, int n0, int n1, int n2) {
  PairCell c;
  const float f0 = floorf(p0), f1 = floorf(p1), f2 = floorf(p2);
  c.t0 = p0 - f0;
  c.t1 = p1 - f1;
  c.t2 = p2 - f2;
  const int i0 = (int)clamp_med3(f0, -2.0f, (float)n0);
  const int i1 = (int)clamp_med3(f1, -2.0f, (float)n1);
  const int i2 = (int)clamp_med3(f2, -2.0f, (float)n2);
  const int xb = min(max(i2, 0), n2 - 2);
  c.upper = i2 > xb;
  c.lower = i2 < xb;
  const unsigned mx = ((unsigned)i2 < (unsigned)n2 ? 0x55u : 0u) | ((unsigned)(i2 + 1) < (unsigned)n2 ? 0xAAu : 0u);
  const unsigned my = ((unsigned)i1 < (unsigned)n1 ? 0x33u : 0u) | ((unsigned)(i1 + 1) < (unsigned)n1 ? 0xCCu : 0u);
  const unsigned mz = ((unsigned)i0 < (unsigned)n0 ? 0x0Fu : 0u) | ((unsigned)(i0 + 1) < (unsigned)n0 ? 0xF0u : 0u);
  c.ok = mx & my & mz;
  const int z0 = min(max(i0, 0), n0 - 1), z1 = min(max(i0 + 1, 0), n0 - 1);
  const int y0 = min(max(i1, 0), n1 - 1), y1 = min(max(i1 + 1, 0), n1 - 1);
  c.off[0] = (z0 * n1 + y0) * n2 + xb;
  c.off[1] = (z0 * n1 + y1) * n2 + xb;
  c.off[2] = (z1 * n1 + y0) * n2 + xb;
  c.off[3] = (z1 * n1 + y1) * n2 + xb;
  return c;
}

typedef float float2_any __attribute__((ext_vector_type(2), aligned(4)));

// Value and position derivative of the trilinear sample (the derivative from
// the right at an integer coordinate, as the cell is chosen by floor).
__device__ __forceinline__ float sample_grad(const float* __restrict__ f, const PairCell& c, float& g0, float& g1,
                                             float& g2) {
  float v[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float2_any p = *reinterpret_cast<const float2_any*>(f + c.off[k]);
    v[2 * k] = (c.ok >> (2 * k)) & 1u ? (c.upper ? p.y : p.x) : 0.0f;
    v[2 * k + 1] = (c.ok >> (2 * k + 1)) & 1u ? (c.lower ? p.x : p.y) : 0.0f;
  }
  const float dx00 = v[1] - v[0], dx01 = v[3] - v[2], dx10 = v[5] - v[4], dx11 = v[7] - v[6];
  const float e00 = __builtin_fmaf(c.t2, dx00, v[0]), e01 = __builtin_fmaf(c.t2, dx01, v[2]);
  const float e10 = __builtin_fmaf(c.t2, dx10, v[4]), e11 = __builtin_fmaf(c.t2, dx11, v[6]);
  const float dy0 = e01 - e00, dy1 = e11 - e10;
  const float f0 = __builtin_fmaf(c.t1, dy0, e00), f1 = __builtin_fmaf(c.t1, dy1, e10);
  const float dxy0 = __builtin_fmaf(c.t1, dx01 - dx00, dx00), dxy1 = __builtin_fmaf(c.t1, dx11 - dx10, dx10);
  g0 = f1 - f0;
  g1 = __builtin_fmaf(c.t0, dy1 - dy0, dy0);
  g2 = __builtin_fmaf(c.t0, dxy1 - dxy0, dxy0);
  return __builtin_fmaf(c.t0, f1 - f0, f0);
}

// v in units of 2^-32, rounded to nearest (ties to even).  |v| = hi + lo with hi
// its integer part and lo exact in fp32, so the two 32-bit halves convert
// separately: 12 full-rate instructions; the conversion through fp64 takes about
// as many at half the rate.
__device__ __forceinline__ unsigned long long to_fixed(float v) {
  const float vc = clamp_med3(v, -kFixClamp, kFixClamp);
  const float a = fabsf(vc);
  const unsigned hi = (unsigned)a;
  const unsigned lo = (unsigned)rintf((a - (float)hi) * 4294967296.0f);
  const unsigned long long u = ((unsigned long long)hi << 32) | lo;
  return vc < 0.0f ? 0ull - u : u;
}

template <int NT>
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) s += red[i];
  return s;
}

// r1(x) = d(x) + e(x + d(x)), the residual of psi o phi.  Its derivative in e
// is the splat of 2 r1 at x + d(x), accumulated in acc ([3][N], fixed point,
// zero on entry).  part[block] = -sum of |r1|^2 over the block's voxels.
__global__ void __launch_bounds__(kInvThreads)
k_inv_splat(const float* __restrict__ d, const float* __restrict__ e, unsigned long long* __restrict__ acc,
            double* __restrict__ part, int n0, int n1, int n2) {
  __shared__ double red[kInvThreads / 64];
  const int N = n0 * n1 * n2;
  double loss = 0.0;
  for (int i = blockIdx.x * kInvThreads + threadIdx.x; i < N; i += gridDim.x * kInvThreads) {
    const int x = i % n2, y = (i / n2) % n1, z = i / (n1 * n2);
    const float d0 = d[i], d1 = d[N + i], d2 = d[2 * N + i];
    const Cell c = cell_of((float)z + d0, (float)y + d1, (float)x + d2, n0, n1, n2);
    const float r0 = d0 + sample(e, c);
    const float r1 = d1 + sample(e + N, c);
    const float r2 = d2 + sample(e + 2 * N, c);
    loss += (double)(r0 * r0 + r1 * r1 + r2 * r2);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (((c.ok >> k) & 1u) && c.w[k] != 0.0f) {
        const float w2 = 2.0f * c.w[k];
        atomicAdd(&acc[c.idx[k]], to_fixed(w2 * r0));
        atomicAdd(&acc[N + c.idx[k]], to_fixed(w2 * r1));
        atomicAdd(&acc[2 * N + c.idx[k]], to_fixed(w2 * r2));
      }
    }
  }
  const double s = block_sum<kInvThreads>(loss, red);
  if (threadIdx.x == 0) part[blockIdx.x] = -s;
}

// r2(x) = e(x) + d(x + e(x)), the residual of phi o psi, whose derivative in
// e(x) is 2 (I + grad d)^T r2; with the splat's sum sp at x and the 1/N of the
// mean this is dU/de.  grad_only: write it to out.  Otherwise Adam on it
// (moments m, v; reciprocal bias corrections ibc1, ibc2): out = the direction.
// Returns |r2|^2.
struct DirArgs {
  const float* d;
  const float* e;
  float* m;
  float* v;
  float* out;
  Ctl* ctl;
  double* part;   // per-workgroup loss partials (minus the sum)
  int n0, n1, n2;
  float inv_n, beta1, beta2, adam_eps;
  int grad_only;
};

__device__ __forceinline__ float node_direction(const DirArgs& A, int z, int y, int x, const float sp[3], float e0,
                                                float e1, float e2, float ibc1, float ibc2) {
  const int N = A.n0 * A.n1 * A.n2, i = (z * A.n1 + y) * A.n2 + x;
  const PairCell c = pair_cell((float)z + e0, (float)y + e1, (float)x + e2, A.n0, A.n1, A.n2);
  float J[3][3];   // J[q][a] = d d_q / d p_a at x + e(x)
  const float v0 = sample_grad(A.d, c, J[0][0], J[0][1], J[0][2]);
  const float v1 = sample_grad(A.d + N, c, J[1][0], J[1][1], J[1][2]);
  const float v2 = sample_grad(A.d + 2 * N, c, J[2][0], J[2][1], J[2][2]);
  const float r[3] = {e0 + v0, e1 + v1, e2 + v2};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float g =
        __builtin_fmaf(2.0f, __builtin_fmaf(J[2][a], r[2], __builtin_fmaf(J[1][a], r[1], __builtin_fmaf(J[0][a], r[0], r[a]))),
                       sp[a]) *
        A.inv_n;
    const int ia = a * N + i;
    if (A.grad_only) {
      A.out[ia] = g;
    } else {
      const float mm = __builtin_fmaf(A.beta1, A.m[ia], (1.0f - A.beta1) * g);
      const float vv = __builtin_fmaf(A.beta2, A.v[ia], (1.0f - A.beta2) * g * g);
      A.m[ia] = mm;
      A.v[ia] = vv;
      A.out[ia] = fa::adam_direction(mm, vv, ibc1, ibc2, A.adam_eps);
    }
  }
  return r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
}

__device__ __forceinline__ float from_fixed(unsigned long long s) {
  return (float)((double)(long long)s * kFixUnit);
}

// The direction from the splat of k_inv_splat (acc, cleared here for the next iteration).
__global__ void __launch_bounds__(kInvThreads) k_inv_dir(const DirArgs A, unsigned long long* __restrict__ acc) {
  __shared__ double red[kInvThreads / 64];
  const int N = A.n0 * A.n1 * A.n2;
  if (!A.grad_only && blockIdx.x == 0 && threadIdx.x < fa::kMSlots) A.ctl->mslot[threadIdx.x * fa::kMStride] = 0u;
  const float ibc1 = A.grad_only ? 1.0f : 1.0f / A.ctl->bc1;
  const float ibc2 = A.grad_only ? 1.0f : 1.0f / A.ctl->bc2;
  double loss = 0.0;
  for (int i = blockIdx.x * kInvThreads + threadIdx.x; i < N; i += gridDim.x * kInvThreads) {
    const int x = i % A.n2, y = (i / A.n2) % A.n1, z = i / (A.n1 * A.n2);
    float s[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      s[q] = from_fixed(acc[q * N + i]);
      acc[q * N + i] = 0ull;
    }
    loss += (double)node_direction(A, z, y, x, s, A.e[i], A.e[N + i], A.e[2 * N + i], ibc1, ibc2);
  }
  const double t = block_sum<kInvThreads>(loss, red);
  if (threadIdx.x == 0) A.part[blockIdx.x] = -t;
}

// ---- the splat by owner ------------------------------------------------------
// d is the same in every iteration of a level, so the cell that x + d(x) falls
// into is listed once per level (k_inv_plan): up to kSlots voxels per cell of
// the grid extended by one cell below, in `slots` ([2][cells] int4), and their
// number in `count`.  k_inv_direction then gives each tile of nodes to one
// workgroup, which takes every voxel listed in the tile's cells, sums its
// contributions in LDS and goes on to the direction: no global atomics and no
// sums in memory.  (Gradient at 160x192x224: 904 us when bricks of
// voxels were summed in LDS and added to memory with one 64-bit atomic per
// touched node and component, six per voxel, and a second kernel read the sums;
// 297 us here.  96x112x112: 174 -> 64; 40x48x56: 35 -> 25.)
//
// A cell with more than kSlots voxels (a contracting or wild warp) is "crowded":
// it is not walked through its list, its tile goes over the bricks of voxels
// whose box of cells meets the tile.  Where a map contracts, that would give a
// few tiles all of the work, so a level with many such voxels (crowded_level)
// takes the bricks themselves as items (brick_body).
constexpr int kSlots = 8;
constexpr int kBZ = 4, kBY = 8, kBX = 16, kBrick = kBZ * kBY * kBX;
constexpr int kTX = 16;         // nodes of a tile along n2
constexpr int kBoxTiles = 128;  // tiles that a brick's box may meet in a crowded level
constexpr int kReady = 16;      // tiles whose nodes a workgroup takes between barriers

struct Plan {
  unsigned* count;      // [cells]
  int* need;            // [tiles]: bricks whose box meets the tile
  int* left;            // [tiles]: of them, done so far; left at zero
  int* crowded;         // [tiles]: whether a cell of the tile is crowded
  int* total;           // voxels past kSlots of their cells, whether a box meets more than kBoxTiles tiles
                        // (count, need, left, crowded and total lie one after the other and are cleared for each level)
  int4* slots;          // [2][cells]
  int4* box;            // [2][bricks]: lowest cell, highest cell (+1 each), empty where low > high
  double* outside;      // [blocks]: sum of |d|^2 over voxels whose sample has no corner on the grid
  double* tile_loss;    // [tiles]
  unsigned* tickets;    // of a crowded level's tiles
  size_t cells;
  int bricks, tiles;
  int tile_log;         // tiles are 2^tile_log nodes along n0 and n1
};

// Cells are numbered -1 .. n-1 per axis; cell index of (c0, c1, c2).
__device__ __forceinline__ size_t cell_index(int c0, int c1, int c2, int n1, int n2) {
  return ((size_t)(c0 + 1) * (n1 + 1) + (c1 + 1)) * (n2 + 1) + (c2 + 1);
}

// Cell of position p; false if no corner is on the grid (or p is not a number).
__device__ __forceinline__ bool plan_cell(float p0, float p1, float p2, int n0, int n1, int n2, int& c0, int& c1,
                                          int& c2) {
  c0 = (int)clamp_med3(floorf(p0), -2.0f, (float)n0);
  c1 = (int)clamp_med3(floorf(p1), -2.0f, (float)n1);
  c2 = (int)clamp_med3(floorf(p2), -2.0f, (float)n2);
  return c0 >= -1 && c0 < n0 && c1 >= -1 && c1 < n1 && c2 >= -1 && c2 < n2;
}

// Adds one to *c and returns what this thread found; one atomic where the whole
// wavefront counts into one cell.
__device__ __forceinline__ unsigned count_in(unsigned* c) {
  const unsigned long long active = __ballot(true);
  unsigned* const first = reinterpret_cast<unsigned*>(
      ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned long long)c >> 32)) << 32) |
      (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned long long)c));
  if (__ballot(c == first) != active) return atomicAdd(c, 1u);
  const int lane = threadIdx.x & 63, before = __popcll(active & ((1ull << lane) - 1));
  unsigned r = 0u;
  if (before == 0) r = atomicAdd(c, (unsigned)__popcll(active));
  return (unsigned)__builtin_amdgcn_readfirstlane((int)r) + before;
}

// The tiles that hold a node which a brick contributes to: its box of cells
// (Plan::box) widened by one node above, clipped to the grid.
struct TileRange {
  int z, y, x, nz, ny, nx;   // first tile, and how many per axis
  __device__ __forceinline__ int count() const { return nz * ny * nx; }
};
__device__ __forceinline__ TileRange tiles_of(int4 lo, int4 hi, int n0, int n1, int n2, int tile_log) {
  auto axis = [](int l, int h, int n, int size, int& first, int& many) {
    first = max(l - 1, 0) / size;
    many = min(h, n - 1) / size - first + 1;
  };
  TileRange r;
  const int size = 1 << tile_log;
  axis(lo.x, hi.x, n0, size, r.z, r.nz);
  axis(lo.y, hi.y, n1, size, r.y, r.ny);
  axis(lo.z, hi.z, n2, kTX, r.x, r.nx);
  if (lo.x > hi.x) r.nz = 0;   // no voxel of the brick falls on the grid
  return r;
}
__device__ __forceinline__ int tile_at(const TileRange& r, int k, int tiles_y, int tiles_x) {
  const int x = k % r.nx, y = k / r.nx % r.ny, z = k / (r.nx * r.ny);
  return ((r.z + z) * tiles_y + r.y + y) * tiles_x + r.x + x;
}

__global__ void __launch_bounds__(kInvThreads) k_inv_plan(const float* __restrict__ d, const Plan P, int n0, int n1,
                                                          int n2) {
  __shared__ int bb[kInvThreads / 64][6];
  __shared__ double red[kInvThreads / 64];
  const int N = n0 * n1 * n2;
  const int ty = (n1 + kBY - 1) / kBY, tx = (n2 + kBX - 1) / kBX;
  const int tid = threadIdx.x;
  const int size = 1 << P.tile_log;
  const int tzs = (n0 + size - 1) / size, tys = (n1 + size - 1) / size, txs = (n2 + kTX - 1) / kTX;
  double outside = 0.0;
  int past = 0;
  for (int b = blockIdx.x; b < P.bricks; b += gridDim.x) {
    const int bx = b % tx, by = (b / tx) % ty, bz = b / (tx * ty);
    int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {-1, -1, -1};
#pragma unroll
    for (int l = tid; l < kBrick; l += kInvThreads) {
      const int z = bz * kBZ + l / (kBY * kBX), y = by * kBY + (l / kBX) % kBY, x = bx * kBX + l % kBX;
      if (z >= n0 || y >= n1 || x >= n2) continue;
      const int i = (z * n1 + y) * n2 + x;
      const float d0 = d[i], d1 = d[N + i], d2 = d[2 * N + i];
      int c[3];
      if (!plan_cell((float)z + d0, (float)y + d1, (float)x + d2, n0, n1, n2, c[0], c[1], c[2])) {
        outside += (double)(d0 * d0 + d1 * d1 + d2 * d2);
        continue;
      }
      const size_t ci = cell_index(c[0], c[1], c[2], n1, n2);
      const unsigned r = count_in(&P.count[ci]);
      past += r >= kSlots;
      if (r == kSlots)   // the cell's own tile, and those whose lower border it is
        for (int q = max(c[0], 0) >> P.tile_log; q <= min((c[0] + 1) >> P.tile_log, tzs - 1); ++q)
          for (int v = max(c[1], 0) >> P.tile_log; v <= min((c[1] + 1) >> P.tile_log, tys - 1); ++v)
            for (int u = max(c[2], 0) / kTX; u <= min((c[2] + 1) / kTX, txs - 1); ++u)
              P.crowded[(q * tys + v) * txs + u] = 1;
      if (r < kSlots) reinterpret_cast<int*>(P.slots + (r < 4 ? 0 : P.cells) + ci)[r & 3] = i;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[a] = min(lo[a], c[a] + 1);
        hi[a] = max(hi[a], c[a] + 1);
      }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        lo[a] = min(lo[a], __shfl_xor(lo[a], o, 64));
        hi[a] = max(hi[a], __shfl_xor(hi[a], o, 64));
      }
    if ((tid & 63) == 0)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        bb[tid >> 6][a] = lo[a];
        bb[tid >> 6][3 + a] = hi[a];
      }
    __syncthreads();
    int4 low = make_int4(bb[0][0], bb[0][1], bb[0][2], 0), high = make_int4(bb[0][3], bb[0][4], bb[0][5], 0);
#pragma unroll
    for (int w = 1; w < kInvThreads / 64; ++w) {
      low = make_int4(min(low.x, bb[w][0]), min(low.y, bb[w][1]), min(low.z, bb[w][2]), 0);
      high = make_int4(max(high.x, bb[w][3]), max(high.y, bb[w][4]), max(high.z, bb[w][5]), 0);
    }
    if (tid == 0) {
      P.box[b] = low;
      P.box[(size_t)P.bricks + b] = high;
    }
    const TileRange r = tiles_of(low, high, n0, n1, n2, P.tile_log);
    if (r.count() > kBoxTiles) {
      if (tid == 0) P.total[1] = 1;
    } else if (tid < r.count()) {
      atomicAdd(&P.need[tile_at(r, tid, tys, txs)], 1);
    }
    __syncthreads();
  }
  const double s = block_sum<kInvThreads>(outside, red);
  if (tid == 0) P.outside[blockIdx.x] = s;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) past += __shfl_xor(past, o, 64);
  if ((tid & 63) == 0 && past) atomicAdd(&P.total[0], past);
}

// Whether the bricks are the items of a level of N voxels: where one in 128 is
// past kSlots of its cell, and no brick's box meets more tiles than kBoxTiles
// (a wild map; its direction then walks, however crowded it is).  Maps p -> c +
// (1 - k)(p - c) with some noise, gradient in us by lists and by bricks: at
// 160x192x224 k = 0.48 (one in 360) 592 and 694, k = 0.5 (one in 42) 822 and 788;
// at 128^3 k = 0.48 276 and 291, k = 0.5 320 and 291; at 64^3 k = 0.45 (one in 145)
// 84 and 86, k = 0.48 (one in 33) 105 and 87.
__device__ __forceinline__ bool crowded_level(const Plan& P, int N) {
  return __builtin_amdgcn_readfirstlane(P.total[0]) > N / 128 && __builtin_amdgcn_readfirstlane(P.total[1]) == 0;
}

// The splat by bricks, for a crowded level.  A brick's voxels go into a box of few
// nodes: the workgroup sums them there in LDS (the same integers, so the sums are
// the same) and adds the box to acc with one atomic per node and component; a
// brick whose box is larger than that adds directly.  Then it counts itself in at
// the tiles that its box meets, and a tile whose last brick this is goes on to the
// direction here.  Which workgroup that is differs from run to run, so a tile's
// loss goes to memory and the last tile's workgroup sums them in order; nothing
// waits for another workgroup.  Tiles that no brick meets come at the end.  (The
// maps above, k = 0.55, 0.7, 0.9 and all voxels in one cell: at 160x192x224 639,
// 606, 654 and 905 us, with the tiles' walks alone 897, 1158, 10277 and 26706, as
// two kernels with an accumulator for every map 629, 609, 688 and 891; at 128^3
// 249, 221, 217 and 298, 386, 727, 3636 and 8136, 203, 200, 221 and 263; at 64^3
// 69, 63, 55 and 80, 118, 191, 703 and 1586, 37, 38, 45 and 53: few bricks, whose
// steps wait for one another here.)
template <int TZ, int TY, int NT, int BOX>   // BOX: nodes that `box` holds
__device__ __forceinline__ void brick_body(const DirArgs& A, const Plan& P, unsigned long long* __restrict__ acc,
                                           unsigned long long* box, int* ready, int* word, double* red, float ibc1,
                                           float ibc2, double& loss) {
  constexpr int VPT = kBrick / NT;
  const int n0 = A.n0, n1 = A.n1, n2 = A.n2, N = n0 * n1 * n2;
  const int tys = (n1 + TY - 1) / TY, txs = (n2 + kTX - 1) / kTX;
  const int bty = (n1 + kBY - 1) / kBY, btx = (n2 + kBX - 1) / kBX;
  const int tid = threadIdx.x;

  // the direction at the nodes of the n tiles in `ready`, whose sums are complete
  __shared__ double part[kReady][NT / 64];
  auto finish = [&](int n) {
    for (int k0 = 0; k0 < n; k0 += kReady) {
      const int m = min(kReady, n - k0);
      for (int k = 0; k < m; ++k) {
        const int t = __builtin_amdgcn_readfirstlane(ready[k0 + k]);
        const int x0 = t % txs * kTX, y0 = t / txs % tys * TY, z0 = t / (txs * tys) * TZ;
        double mine = 0.0;
        for (int q = tid; q < TZ * TY * kTX; q += NT) {
          const int z = z0 + q / (TY * kTX), y = y0 + q / kTX % TY, x = x0 + q % kTX;
          if (z >= n0 || y >= n1 || x >= n2) continue;
          const int i = (z * n1 + y) * n2 + x;
          float s[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            unsigned long long* const sum = &acc[(size_t)c * N + i];
            const unsigned long long v = __hip_atomic_load(sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v) __hip_atomic_store(sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s[c] = from_fixed(v);
          }
          mine += (double)node_direction(A, z, y, x, s, A.e[i], A.e[N + i], A.e[2 * N + i], ibc1, ibc2);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mine += __shfl_down(mine, o, 64);
        if ((tid & 63) == 0) part[k][tid >> 6] = mine;
      }
      if (tid == 0) *word = 0;
      __syncthreads();
      if (tid < m) {
        double tile = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) tile += part[tid][w];
        const int t = ready[k0 + tid];
        __hip_atomic_store(&P.tile_loss[t], tile, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (fa::last_workgroup(P.tickets, t, P.tiles)) *word = 1;
      }
      __syncthreads();
      if (*word) {
        double all = 0.0;
        for (int k = tid; k < P.tiles; k += NT)
          all += __hip_atomic_load(&P.tile_loss[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        all = block_sum<NT>(all, red);
        if (tid == 0) A.part[gridDim.x] = -all;
      }
      __syncthreads();   // part, word and ready are written again
    }
  };

  for (int b = blockIdx.x; b < P.bricks; b += gridDim.x) {
    const int4 lo = P.box[b], hi = P.box[(size_t)P.bricks + b];   // cells + 1
    const TileRange tr = tiles_of(lo, hi, n0, n1, n2, P.tile_log);
    if (tr.count() == 0) continue;   // its voxels' loss is in P.outside
    // the box's nodes, clipped to the grid
    const int b0 = max(lo.x - 1, 0), b1 = max(lo.y - 1, 0), b2 = max(lo.z - 1, 0);
    const int s0 = min(hi.x, n0 - 1) - b0 + 1, s1 = min(hi.y, n1 - 1) - b1 + 1, s2 = min(hi.z, n2 - 1) - b2 + 1;
    const int nb = s0 * s1 * s2;
    const bool in_lds = nb <= BOX;
    if (in_lds)
      for (int q = tid; q < 3 * nb; q += NT) box[q] = 0ull;
    if (tid == 0) *word = 0;
    __syncthreads();
    const int bx = b % btx, by = b / btx % bty, bz = b / (btx * bty);
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const int l = tid + u * NT;
      const int z = bz * kBZ + l / (kBY * kBX), y = by * kBY + (l / kBX) % kBY, x = bx * kBX + l % kBX;
      if (z >= n0 || y >= n1 || x >= n2) continue;
      const int i = (z * n1 + y) * n2 + x;
      const float d0 = A.d[i], d1 = A.d[N + i], d2 = A.d[2 * N + i];
      const float p0 = (float)z + d0, p1 = (float)y + d1, p2 = (float)x + d2;
      int cz, cy, cx;
      if (!plan_cell(p0, p1, p2, n0, n1, n2, cz, cy, cx)) continue;
      const Cell c = cell_of(p0, p1, p2, n0, n1, n2);
      const float r[3] = {d0 + sample(A.e, c), d1 + sample(A.e + N, c), d2 + sample(A.e + 2 * N, c)};
      loss += (double)(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (!((c.ok >> k) & 1u) || c.w[k] == 0.0f) continue;
        const float w2 = 2.0f * c.w[k];
        if (in_lds) {
          const int q = ((cz + (k >> 2) - b0) * s1 + (cy + ((k >> 1) & 1) - b1)) * s2 + (cx + (k & 1) - b2);
#pragma unroll
          for (int a = 0; a < 3; ++a) atomicAdd(&box[a * nb + q], to_fixed(w2 * r[a]));
        } else {
#pragma unroll
          for (int a = 0; a < 3; ++a) atomicAdd(&acc[(size_t)a * N + c.idx[k]], to_fixed(w2 * r[a]));
        }
      }
    }
    __syncthreads();
    if (in_lds)
      for (int q = tid; q < nb; q += NT) {
        const int x = b2 + q % s2, y = b1 + q / s2 % s1, z = b0 + q / (s1 * s2);
#pragma unroll
        for (int a = 0; a < 3; ++a)
          if (const unsigned long long v = box[a * nb + q]) atomicAdd(&acc[(size_t)a * N + (z * n1 + y) * n2 + x], v);
      }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's sums have reached memory
    __syncthreads();
    if (tid < tr.count()) {
      const int t = tile_at(tr, tid, tys, txs);
      if (__hip_atomic_fetch_add(&P.left[t], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == P.need[t]) {
        __hip_atomic_store(&P.left[t], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ready[atomicAdd(word, 1)] = t;
      }
    }
    __syncthreads();
    const int n = __builtin_amdgcn_readfirstlane(*word);
    __syncthreads();   // word is written again
    finish(n);
  }
  for (int t = blockIdx.x; t < P.tiles; t += gridDim.x)
    if (__builtin_amdgcn_readfirstlane(P.need[t]) == 0) {
      if (tid == 0) ready[0] = t;
      __syncthreads();
      finish(1);
    }
}

// Exact i / dv for 0 <= i < 2^31 (launch: mul = floor(2^(31 + s) / dv) + 1, s = ceil(log2 dv)).
struct FastDiv {
  unsigned mul, shift;
};
__device__ __forceinline__ int fast_div(int i, FastDiv f) { return (int)(__umulhi((unsigned)i, f.mul) >> f.shift); }

// Per tile: 24 B per node of accumulators and 12 B per node of the tile and its
// one-node border (e) in LDS, 46 KB at 8 x 8 x 16 nodes.  Bound by latency and
// VALU work rather than by memory: each listed voxel takes 24 LDS reads, 24
// conversions and up to 24 LDS atomics, and the tile's lower border cells (a
// third of its cells) are also taken by its neighbours.  At 160x192x224, of 297
// us: 80 the lists and d, 86 the contributions, 90 the nodes.  Six wavefronts
// per SIMD (80 VGPRs, a few spilled) hide more of the latency than the five of
// an unbounded allocation (322 us); 4 x 8 x 16 tiles take 355, 8 x 8 x 32 575.
template <int TZ, int TY, int TX, int NT>
__global__ void __launch_bounds__(NT, 6) k_inv_direction(const DirArgs A, const Plan P, unsigned long long* all_acc,
                                                         FastDiv by_row, FastDiv by_plane) {
  static_assert(TX == kTX && kBrick % NT == 0 && NT >= kBoxTiles, "tile and workgroup shape");
  constexpr int CY = TY + 1, CX = TX + 1, CELLS = (TZ + 1) * CY * CX, NODES = TZ * TY * TX;
  constexpr int SY = TY + 2, SX = TX + 2, SN = (TZ + 2) * SY * SX;
  constexpr int BOX = NODES < 512 ? 512 : NODES;   // nodes that a brick's box may have in LDS
  __shared__ unsigned long long acc[3 * BOX];
  __shared__ float es[3 * SN];
  __shared__ int ready[kBoxTiles];
  __shared__ double red[NT / 64];
  __shared__ unsigned long long hit[NT / 64];
  __shared__ int word;
  const int n0 = A.n0, n1 = A.n1, n2 = A.n2, N = n0 * n1 * n2;
  const int tid = threadIdx.x;
  if (!A.grad_only && blockIdx.x == 0 && tid < fa::kMSlots) A.ctl->mslot[tid * fa::kMStride] = 0u;
  const float ibc1 = A.grad_only ? 1.0f : 1.0f / A.ctl->bc1;
  const float ibc2 = A.grad_only ? 1.0f : 1.0f / A.ctl->bc2;
  const int ty = (n1 + TY - 1) / TY, tx = (n2 + TX - 1) / TX, tiles = (n0 + TZ - 1) / TZ * ty * tx;
  double loss = tid == 0 ? P.outside[blockIdx.x] : 0.0;
  // every XCD takes a contiguous range of tiles (neighbours share border cells and gathers in its L2)
  const int G = gridDim.x;
  const int past = __builtin_amdgcn_readfirstlane(P.total[0]);

  // The nodes of tile t, from the lists of its cells or, where one is crowded, from
  // the bricks (walk).  Two bodies, as the walk in the middle of the one for lists
  // cost it registers (328 us against 319 at 160x192x224).
  auto body = [&](int t, auto walk) __attribute__((always_inline)) {
    const int x0 = t % tx * TX, y0 = t / tx % ty * TY, z0 = t / (tx * ty) * TZ;
    for (int q = tid; q < 3 * NODES; q += NT) acc[q] = 0ull;
    for (int q = tid; q < SN; q += NT) {
      const int z = z0 - 1 + q / (SY * SX), y = y0 - 1 + q / SX % SY, x = x0 - 1 + q % SX;
      const bool in = (unsigned)z < (unsigned)n0 && (unsigned)y < (unsigned)n1 && (unsigned)x < (unsigned)n2;
      const int i = in ? (z * n1 + y) * n2 + x : 0;
#pragma unroll
      for (int c = 0; c < 3; ++c) es[c * SN + q] = in ? A.e[c * N + i] : 0.0f;
    }
    __syncthreads();

    // voxel with displacement (d0, d1, d2) to position p in the tile's cell (lz, ly, lx), 0 = the border
    auto take = [&](float d0, float d1, float d2, float p0, float p1, float p2, int lz, int ly, int lx) {
      const float t0 = p0 - floorf(p0), t1 = p1 - floorf(p1), t2 = p2 - floorf(p2);
      const int base = (lz * SY + ly) * SX + lx;
      float w[8], r[3];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        w[k] = ((k >> 2) & 1 ? t0 : 1.0f - t0) * ((k >> 1) & 1 ? t1 : 1.0f - t1) * (k & 1 ? t2 : 1.0f - t2);
      const float dd[3] = {d0, d1, d2};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
#pragma clang fp contract(off)
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) s += w[k] * es[c * SN + base + ((k >> 2) * SY + ((k >> 1) & 1)) * SX + (k & 1)];
        r[c] = dd[c] + s;
      }
      // a border cell's voxels count where that cell is not another tile's own
      if ((lz > 0 || z0 == 0) && (ly > 0 || y0 == 0) && (lx > 0 || x0 == 0))
        loss += (double)(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int z = lz - 1 + (k >> 2), y = ly - 1 + ((k >> 1) & 1), x = lx - 1 + (k & 1);
        if ((unsigned)z < (unsigned)TZ && (unsigned)y < (unsigned)TY && (unsigned)x < (unsigned)TX && w[k] != 0.0f) {
          const int q = (z * TY + y) * TX + x;
          const float w2 = 2.0f * w[k];
#pragma unroll
          for (int c = 0; c < 3; ++c) atomicAdd(&acc[c * NODES + q], to_fixed(w2 * r[c]));
        }
      }
    };

    if constexpr (!decltype(walk)::value) {
      for (int q = tid; q < CELLS; q += NT) {
        const int lz = q / (CY * CX), ly = q / CX % CY, lx = q % CX;
        const int cz = z0 - 1 + lz, cy = y0 - 1 + ly, cx = x0 - 1 + lx;
        if (cz >= n0 || cy >= n1 || cx >= n2) continue;
        const size_t ci = cell_index(cz, cy, cx, n1, n2);
        const int4 a = P.slots[ci];   // not waiting for the count: entries past it are ignored
        const int n = (int)min(P.count[ci], (unsigned)kSlots);   // never more in a tile that is not crowded
        if (n == 0) continue;
        // in the order of the voxels, so that the loss does not depend on the order of the listing
        int i = -1;
        for (int j = 0; j < n; ++j) {
          int next = 0x7fffffff;
          auto after = [&](int v, int k) { next = k < n && v > i ? min(next, v) : next; };
          after(a.x, 0), after(a.y, 1), after(a.z, 2), after(a.w, 3);
          if (n > 4) {
            const int4 b = P.slots[P.cells + ci];
            after(b.x, 4), after(b.y, 5), after(b.z, 6), after(b.w, 7);
          }
          i = next;
          const int z = fast_div(i, by_plane), yx = i - z * (n1 * n2), y = fast_div(yx, by_row), x = yx - y * n2;
          const float d0 = A.d[i], d1 = A.d[N + i], d2 = A.d[2 * N + i];
          take(d0, d1, d2, (float)z + d0, (float)y + d1, (float)x + d2, lz, ly, lx);
        }
      }
      __syncthreads();
    } else {
      const int bty = (n1 + kBY - 1) / kBY, btx = (n2 + kBX - 1) / kBX;
      for (int b0 = 0; b0 < P.bricks; b0 += NT) {
        bool meets = false;
        if (b0 + tid < P.bricks) {
          const int4 lo = P.box[b0 + tid], hi = P.box[(size_t)P.bricks + b0 + tid];   // cells + 1
          meets = lo.x <= z0 + TZ && hi.x >= z0 && lo.y <= y0 + TY && hi.y >= y0 && lo.z <= x0 + TX && hi.z >= x0;
        }
        const unsigned long long mask = __ballot(meets);
        if ((tid & 63) == 0) hit[tid >> 6] = mask;
        __syncthreads();
        for (int w = 0; w < NT / 64; ++w)
          for (unsigned long long bits = hit[w]; bits; bits &= bits - 1) {
            const int b = b0 + 64 * w + __ffsll(bits) - 1;
            const int bx = b % btx, by = b / btx % bty, bz = b / (btx * bty);
            for (int l = tid; l < kBrick; l += NT) {
              const int z = bz * kBZ + l / (kBY * kBX), y = by * kBY + (l / kBX) % kBY, x = bx * kBX + l % kBX;
              if (z >= n0 || y >= n1 || x >= n2) continue;
              const int i = (z * n1 + y) * n2 + x;
              const float d0 = A.d[i], d1 = A.d[N + i], d2 = A.d[2 * N + i];
              const float p0 = (float)z + d0, p1 = (float)y + d1, p2 = (float)x + d2;
              int cz, cy, cx;
              if (!plan_cell(p0, p1, p2, n0, n1, n2, cz, cy, cx)) continue;
              const int lz = cz - z0 + 1, ly = cy - y0 + 1, lx = cx - x0 + 1;
              if ((unsigned)lz > (unsigned)TZ || (unsigned)ly > (unsigned)TY || (unsigned)lx > (unsigned)TX) continue;
              take(d0, d1, d2, p0, p1, p2, lz, ly, lx);
            }
          }
        __syncthreads();   // hit is written again
      }
      // (the last barrier also ends the accumulation)
    }
    for (int q = tid; q < NODES; q += NT) {
      const int lz = q / (TY * TX), ly = q / TX % TY, lx = q % TX;
      const int z = z0 + lz, y = y0 + ly, x = x0 + lx;
      if (z >= n0 || y >= n1 || x >= n2) continue;
      const float s[3] = {from_fixed(acc[q]), from_fixed(acc[NODES + q]), from_fixed(acc[2 * NODES + q])};
      const int u = ((lz + 1) * SY + ly + 1) * SX + lx + 1;
      loss += (double)node_direction(A, z, y, x, s, es[u], es[SN + u], es[2 * SN + u], ibc1, ibc2);
    }
    __syncthreads();   // acc and es are written again
  };

  if (crowded_level(P, N)) {
    brick_body<TZ, TY, NT, BOX>(A, P, all_acc, acc, ready, &word, red, ibc1, ibc2, loss);
  } else {
    // every XCD takes a contiguous range of tiles (neighbours share border cells and gathers in its L2)
    const int G = gridDim.x, xq = G / 8, xr = G % 8, xb = blockIdx.x % 8;
    const int first = xb * xq + min(xb, xr) + blockIdx.x / 8;
    for (int t = first; t < tiles; t += G)
      if (past == 0 || __builtin_amdgcn_readfirstlane(P.crowded[t]) == 0) body(t, std::false_type{});
    if (past)
      for (int t = first; t < tiles; t += G)
        if (__builtin_amdgcn_readfirstlane(P.crowded[t])) body(t, std::true_type{});
    if (blockIdx.x == 0 && tid == 0) A.part[G] = 0.0;
  }
  const double s = block_sum<NT>(loss, red);
  if (tid == 0) A.part[blockIdx.x] = -s;
}

int inv_blocks(int64_t n) {
  return (int)std::min<int64_t>((n + kInvThreads - 1) / kInvThreads, kInvMaxBlocks);
}

template <typename T>
fa_status ialloc(T** out, size_t count, const char* what) {
  *out = nullptr;
  if (count == 0) count = 1;
  const hipError_t e = hipMalloc((void**)out, count * sizeof(T));
  if (e != hipSuccess) {
    *out = nullptr;
    (void)hipGetLastError();
    return fail(FA_ENOMEM, std::string("hipMalloc failed for ") + what + " (" + std::to_string(count * sizeof(T)) +
                               " bytes): " + hipGetErrorString(e));
  }
  return FA_OK;
}

struct ILevel {
  fa_shape shape{};
  int64_t n = 0;
  float scale = 1.0f;
  int iters = 0;
  float* d = nullptr;   // the warp's field on this grid (owned unless it aliases the input copy)
  bool owns = false;
  Tiling tsg{}, tsc{}, tsw{};
};

}  // namespace

struct fa_inverse_s {
  hipStream_t stream = nullptr;
  fa_shape shape{};
  int64_t n = 0;
  fa_params p{};
  float* in_d = nullptr;   // [3][n] copy of the input field
  std::vector<ILevel> levels;
  int64_t cap = 0;
  float* e = nullptr;      // psi - id at the current level, [3][n]
  float* m = nullptr;
  float* v = nullptr;
  float* a = nullptr;      // Adam direction
  float* tmp = nullptr;    // smoothed direction, then the composed field
  float* wide = nullptr;   // [3][cap] scratch of the smoothing passes with a radius above 6
  unsigned long long* acc = nullptr;   // sums of the splat by bricks and the direct one [3][cap], zero between iterations
  Plan plan{};             // voxels by cell of level plan_level
  size_t plan_words = 0, plan_cells = 0;   // capacities of its buffers
  int plan_bricks = 0, plan_tiles = 0;
  int plan_level = -1;     // -1: none listed (or only inside a captured graph)
  bool captured = false;   // a call was captured: its replays list their own level, so each call lists anew
  Ctl* ctl = nullptr;
  float* loss_hist = nullptr;
  int loss_cap = 0;
  double* partials = nullptr;
  float* scalar = nullptr;  // device float (eval_gradient's cost)
  float* wts = nullptr;
  std::vector<float> wts_host;   // what wts holds
  int rg = 0, rw = 0, off_g = 0, off_w = 0, off_one = 0;
  int cur_level = 0, cur_iter = 0, t_done = 0, iters_done = 0;
  bool scheduled = false;
  bool splat_direct = false;   // the per-voxel global-atomic splat instead of the listed one
};

namespace {

void free_levels(fa_inverse H) {
  for (auto& L : H->levels)
    if (L.owns && L.d) (void)hipFree(L.d);
  H->levels.clear();
}

void free_plan(fa_inverse H) {
  const Plan& P = H->plan;
  void* const bufs[] = {P.count, P.slots, P.box, P.outside, P.tile_loss, P.tickets};
  for (void* b : bufs)
    if (b) (void)hipFree(b);
  H->plan = Plan{};
  H->plan_words = H->plan_cells = 0;
  H->plan_bricks = H->plan_tiles = 0;
  H->plan_level = -1;
}

int64_t cells_of(const fa_shape& s) { return (int64_t)(s.n0 + 1) * (s.n1 + 1) * (s.n2 + 1); }
int bricks_of(const fa_shape& s) {
  return (s.n0 + kBZ - 1) / kBZ * ((s.n1 + kBY - 1) / kBY) * ((s.n2 + kBX - 1) / kBX);
}

// Tiles of k_inv_direction: 8 x 8 x 16 nodes, or 4 x 4 x 16 below
// kSmallTileVoxels, where the larger ones give a CU less than one workgroup
// (40x48x56: 25 us against 30 with the larger; 80x96x112, 860,000 voxels: 58
// with either).
bool small_tiles(const fa_shape& s) { return fa::voxels(s) < kSmallTileVoxels; }

int dir_tiles(const fa_shape& s) {
  const int t = small_tiles(s) ? 4 : 8;
  return (s.n0 + t - 1) / t * ((s.n1 + t - 1) / t) * ((s.n2 + kTX - 1) / kTX);
}
int dir_blocks(const fa_shape& s) { return std::min(dir_tiles(s), kDirMaxBlocks); }

// Words that are cleared for each level: Plan::count, need, left, crowded and total.
size_t plan_words(const fa_shape& s) { return (size_t)cells_of(s) + 3 * (size_t)dir_tiles(s) + 2; }

// The lists' extents on a level, in buffers that hold its largest.
Plan plan_of(Plan P, const fa_shape& s) {
  P.cells = (size_t)cells_of(s);
  P.bricks = bricks_of(s);
  P.tiles = dir_tiles(s);
  P.tile_log = small_tiles(s) ? 2 : 3;
  P.need = reinterpret_cast<int*>(P.count) + P.cells;
  P.left = P.need + P.tiles;
  P.crowded = P.left + P.tiles;
  P.total = P.crowded + P.tiles;
  return P;
}

// The sums in memory, zeroed.
fa_status ensure_acc(fa_inverse H) {
  if (H->acc) return FA_OK;
  FA_TRY(ialloc(&H->acc, (size_t)(3 * H->cap), "splat accumulator"));
  FA_HIP(hipMemsetAsync(H->acc, 0, (size_t)(3 * H->cap) * sizeof(unsigned long long), H->stream));
  return FA_OK;
}

void free_all(fa_inverse H) {
  free_levels(H);
  float* fb[] = {H->in_d, H->e, H->m, H->v, H->a, H->tmp, H->wide, H->loss_hist, H->scalar, H->wts};
  for (float* b : fb)
    if (b) (void)hipFree(b);
  free_plan(H);
  if (H->acc) (void)hipFree(H->acc);
  if (H->ctl) (void)hipFree(H->ctl);
  if (H->partials) (void)hipFree(H->partials);
}

// e scaled by rho, the Adam moments unscaled, trilinear at corner-aligned
// positions of the next (finer) grid.
fa_status transition(fa_inverse H) {
  const ILevel& C = H->levels[H->cur_level];
  const ILevel& F = H->levels[H->cur_level + 1];
  auto rho = [](int nf, int nc) { return nc > 1 ? (float)((double)(nf - 1) / (double)(nc - 1)) : 1.0f; };
  const int c[3] = {C.shape.n0, C.shape.n1, C.shape.n2}, f[3] = {F.shape.n0, F.shape.n1, F.shape.n2};
  const float r[3] = {rho(f[0], c[0]), rho(f[1], c[1]), rho(f[2], c[2])}, one[3] = {1.0f, 1.0f, 1.0f};
  const float* in[2] = {H->e, H->m};
  float* out[2] = {H->tmp, H->a};
  FA_HIP(fa::launch_resample(in, out, 2, c, f, r, H->stream));
  std::swap(H->e, H->tmp);
  std::swap(H->m, H->a);
  // v goes to the buffer that held the coarse e
  const float* in_v = H->v;
  FA_HIP(fa::launch_resample(&in_v, &H->tmp, 1, c, f, one, H->stream));
  std::swap(H->v, H->tmp);
  return FA_OK;
}

bool schedule_done(const fa_inverse H) {
  return H->cur_level == (int)H->levels.size() - 1 && H->cur_iter >= H->levels.back().iters;
}

// Loss partials of one direction (launch_direction).
int direction_partials(const fa_inverse H, const ILevel& L) {
  return H->splat_direct ? 2 * inv_blocks(L.n) : dir_blocks(L.shape) + 1;
}

FastDiv fast_divisor(unsigned dv) {   // dv >= 2
  unsigned s = 0;
  while ((1ull << s) < dv) ++s;
  return {(unsigned)((1ull << (31 + s)) / dv + 1), s - 1};
}

fa_status launch_direction(fa_inverse H, const ILevel& L, float* out, int grad_only) {
  const fa_shape& s = L.shape;
  DirArgs A{};
  A.d = L.d;
  A.e = H->e;
  A.m = H->m;
  A.v = H->v;
  A.out = out;
  A.ctl = H->ctl;
  A.part = H->partials;
  A.n0 = s.n0;
  A.n1 = s.n1;
  A.n2 = s.n2;
  A.inv_n = (float)(1.0 / (double)L.n);
  A.beta1 = H->p.adam_beta1;
  A.beta2 = H->p.adam_beta2;
  A.adam_eps = H->p.adam_eps;
  A.grad_only = grad_only;
  if (H->splat_direct) {
    const int b = inv_blocks(L.n);
    hipLaunchKernelGGL(k_inv_splat, dim3(b), dim3(kInvThreads), 0, H->stream, L.d, H->e, H->acc, H->partials,
                       s.n0, s.n1, s.n2);
    FA_HIP(hipGetLastError());
    A.part = H->partials + b;
    hipLaunchKernelGGL(k_inv_dir, dim3(b), dim3(kInvThreads), 0, H->stream, A, H->acc);
    FA_HIP(hipGetLastError());
    return FA_OK;
  }
  const int b = dir_blocks(s);
  const Plan P = plan_of(H->plan, s);
  H->captured |= fa::capturing(H->stream);
  if (H->captured || H->plan_level != H->cur_level) {
    FA_HIP(fa::launch_fill(reinterpret_cast<float*>(P.count), 0.0f, (int64_t)plan_words(s), H->stream));
    hipLaunchKernelGGL(k_inv_plan, dim3(b), dim3(kInvThreads), 0, H->stream, L.d, P, s.n0, s.n1, s.n2);
    FA_HIP(hipGetLastError());
    H->plan_level = H->captured ? -1 : H->cur_level;
  }
  const FastDiv by_row = fast_divisor(s.n2), by_plane = fast_divisor((unsigned)(s.n1 * s.n2));
  if (small_tiles(s))
    hipLaunchKernelGGL((k_inv_direction<4, 4, 16, 256>), dim3(b), dim3(256), 0, H->stream, A, P, H->acc, by_row, by_plane);
  else
    hipLaunchKernelGGL((k_inv_direction<8, 8, 16, 512>), dim3(b), dim3(512), 0, H->stream, A, P, H->acc, by_row, by_plane);
  FA_HIP(hipGetLastError());
  return FA_OK;
}

fa_status launch_iteration(fa_inverse H, const ILevel& L) {
  FA_TRY(launch_direction(H, L, H->a, 0));
  fa::GaussArgs gs{};
  gs.ctl = H->ctl;
  gs.n0 = L.shape.n0;
  gs.n1 = L.shape.n1;
  gs.n2 = L.shape.n2;
  gs.eta = H->p.eta;
  gs.inv_n = (float)(1.0 / (double)L.n);

  fa::GaussArgs g1 = gs;   // s = G * a, M = max |s|
  g1.in = H->a;
  g1.out = H->tmp;
  g1.wts = H->wts + H->off_g;
  g1.wide_tmp = H->wide;
  g1.zc = L.tsg.zc;
  g1.tiles_y = L.tsg.tiles_y;
  g1.tiles_x = L.tsg.tiles_x;
  FA_HIP(fa::launch_gauss(g1, H->rg, fa::EPI_SMOOTH_MAX, L.tsg, H->stream));

  fa::GaussArgs g2 = gs;   // e' = u + e(x + u), u = -eta s / (2M), in place over s
  g2.in = H->tmp;
  g2.out = H->tmp;
  g2.d = H->e;
  g2.wts = H->wts + H->off_one;
  g2.zc = L.tsc.zc;
  g2.tiles_y = L.tsc.tiles_y;
  g2.tiles_x = L.tsc.tiles_x;

  fa::GaussArgs g3 = gs;   // e = G * e'
  g3.in = H->tmp;
  g3.out = H->e;
  g3.wts = H->wts + H->off_w;
  g3.wide_tmp = H->wide;
  g3.zc = L.tsw.zc;
  g3.tiles_y = L.tsw.tiles_y;
  g3.tiles_x = L.tsw.tiles_x;

  // the cost record and step count, in the launch the registration uses
  fa::GaussArgs& gr = fa::record_launch(L.tsw) == 2 ? g3 : g2;
  gr.partials = H->partials;
  gr.n_partials = direction_partials(H, L);
  gr.loss_hist = H->loss_hist;
  gr.loss_cap = H->loss_cap;

  FA_HIP(fa::launch_gauss(g2, 0, H->p.eta <= 2.0f ? fa::EPI_COMPOSE_LDS : fa::EPI_COMPOSE, L.tsc, H->stream));

  FA_HIP(fa::launch_gauss(g3, H->rw, fa::EPI_STORE, L.tsw, H->stream));
  return FA_OK;
}

}  // namespace

namespace fa {

fa_status inverse_restart(fa_inverse H, const float* d, const fa_params* params) {
  FA_TRY(check_params(params));
  H->p = *params;
  H->scheduled = false;
  FA_HIP(hipMemcpyAsync(H->in_d, d, (size_t)(3 * H->n) * sizeof(float), hipMemcpyDeviceToDevice, H->stream));
  return FA_OK;
}

}  // namespace fa

extern "C" {

fa_status fa_inverse_create(const float* d, fa_shape shape, const fa_params* params, void* stream,
                            fa_inverse* out) {
  if (!out) return fail(FA_EINVAL, "out is NULL");
  *out = nullptr;
  if (!d) return fail(FA_EINVAL, "d must be a device pointer");
  FA_TRY(fa::check_shape(shape));
  FA_TRY(fa::check_params(params));
  fa_inverse H = new (std::nothrow) fa_inverse_s();
  if (!H) return fail(FA_ENOMEM, "host allocation failed");
  H->stream = (hipStream_t)stream;
  H->shape = shape;
  H->n = fa::voxels(shape);
  H->p = *params;
  fa_status st = FA_OK;
  if ((st = ialloc(&H->in_d, (size_t)(3 * H->n), "input field")) != FA_OK ||
      (st = ialloc(&H->ctl, 1, "control block")) != FA_OK || (st = ialloc(&H->scalar, 1, "scalar")) != FA_OK) {
    free_all(H);
    delete H;
    return st;
  }
  const hipError_t e = hipMemcpyAsync(H->in_d, d, (size_t)(3 * H->n) * sizeof(float), hipMemcpyDeviceToDevice,
                                      H->stream);
  if (e != hipSuccess) {
    free_all(H);
    delete H;
    return fail(FA_EHIP, std::string("copying the field: ") + hipGetErrorString(e));
  }
  *out = H;
  return FA_OK;
}

fa_status fa_inverse_set_schedule(fa_inverse H, int n_levels, const float* scales, const int* iters) {
  if (!H) return fail(FA_EINVAL, "handle is NULL");
  if (n_levels < 1 || n_levels > 16) return fail(FA_EINVAL, "n_levels must be in [1, 16]");
  if (!scales || !iters) return fail(FA_EINVAL, "scales and iters must not be NULL");
  std::vector<ILevel> lv(n_levels);
  int64_t total = 0, nmax = 0;
  H->rg = fa::tap_radius(H->p.sigma_grad);
  H->rw = fa::tap_radius(H->p.sigma_warp);
  for (int i = 0; i < n_levels; ++i) {
    if (!(scales[i] >= 1.0f) || !(scales[i] <= 20.0f)) return fail(FA_EINVAL, "scales must be in [1, 20]");
    if (iters[i] < 0) return fail(FA_EINVAL, "iters must be >= 0");
    lv[i].scale = scales[i];
    lv[i].iters = iters[i];
    lv[i].shape = fa::level_shape(H->shape, scales[i]);
    lv[i].n = fa::voxels(lv[i].shape);
    if (lv[i].shape.n0 < 2 || lv[i].shape.n1 < 2 || lv[i].shape.n2 < 2)
      return fail(FA_ESHAPE, "level " + std::to_string(i) + " has a dimension < 2");
    lv[i].tsg = fa::choose_tiling(lv[i].shape, fa::KIND_SMOOTH_MAX, fa::Tuning(),
                                  fa::gauss_cube_supported(H->rg, fa::EPI_SMOOTH_MAX));
    lv[i].tsw = fa::choose_tiling(lv[i].shape, fa::KIND_WARP_SMOOTH, fa::Tuning(),
                                  fa::gauss_cube_supported(H->rw, fa::EPI_STORE));
    lv[i].tsc = fa::choose_tiling(lv[i].shape, fa::KIND_COMPOSE, fa::Tuning(),
                                  H->p.eta <= 2.0f && fa::gauss_cube_supported(0, fa::EPI_COMPOSE_LDS));
    total += iters[i];
    nmax = std::max(nmax, lv[i].n);
  }
  if (total > (int64_t)1 << 30) return fail(FA_EINVAL, "too many iterations");

  // the level fields of an earlier schedule over the same grids are used again
  H->scheduled = false;
  auto full = [&](const fa_shape& a) { return a.n0 == H->shape.n0 && a.n1 == H->shape.n1 && a.n2 == H->shape.n2; };
  bool same = (int)H->levels.size() == n_levels;
  for (int i = 0; same && i < n_levels; ++i) {
    const ILevel& o = H->levels[i];
    same = o.d && o.owns == !(lv[i].scale == 1.0f && full(lv[i].shape)) && o.shape.n0 == lv[i].shape.n0 &&
           o.shape.n1 == lv[i].shape.n1 && o.shape.n2 == lv[i].shape.n2;
  }
  if (same) {
    for (int i = 0; i < n_levels; ++i) {
      lv[i].d = H->levels[i].d;
      lv[i].owns = H->levels[i].owns;
    }
    H->levels = lv;
  } else {
    FA_HIP(hipStreamSynchronize(H->stream));
    free_levels(H);
  }

  // tap tables: sigma_grad, sigma_warp, the single tap, then one blur per level
  std::vector<float> host;
  auto push = [&](const std::vector<float>& t) {
    const int off = (int)host.size();
    host.insert(host.end(), t.begin(), t.end());
    while (host.size() % 16) host.push_back(0.0f);
    return off;
  };
  H->off_g = push(fa::gaussian_taps(H->p.sigma_grad));
  H->off_w = push(fa::gaussian_taps(H->p.sigma_warp));
  H->off_one = push(std::vector<float>{1.0f});
  std::vector<int> off_blur(n_levels);
  for (int i = 0; i < n_levels; ++i) off_blur[i] = push(fa::gaussian_taps(lv[i].scale / 2.0f));
  if (!H->wts || host != H->wts_host) {
    FA_HIP(hipStreamSynchronize(H->stream));
    if (H->wts) (void)hipFree(H->wts);
    H->wts = nullptr;
    FA_TRY(ialloc(&H->wts, host.size(), "tap tables"));
    H->wts_host = host;
    const hipError_t e = hipMemcpyAsync(H->wts, H->wts_host.data(), host.size() * sizeof(float), hipMemcpyHostToDevice,
                                        H->stream);
    if (e != hipSuccess) {   // wts holds nothing: the next schedule uploads again
      H->wts_host.clear();
      return fail(FA_EHIP, std::string("copying the tap tables: ") + hipGetErrorString(e));
    }
  }

  // state, sized for the largest level, and the sums in memory
  const int64_t need = std::max(nmax, H->n);   // m and e hold three input volumes each below
  const bool wide = H->rg > fa::kMaxRadius || H->rw > fa::kMaxRadius;
  if (need > H->cap || (wide && !H->wide)) {
    FA_HIP(hipStreamSynchronize(H->stream));
    float** bufs[] = {&H->e, &H->m, &H->v, &H->a, &H->tmp, &H->wide};
    for (float** b : bufs) {
      if (*b) (void)hipFree(*b);
      *b = nullptr;
    }
    if (H->acc) (void)hipFree(H->acc);
    H->acc = nullptr;
    if (H->partials) (void)hipFree(H->partials);
    H->partials = nullptr;
    H->cap = 0;
    for (int k = 0; k < (wide ? 6 : 5); ++k) FA_TRY(ialloc(bufs[k], (size_t)(3 * need), "state"));
    FA_TRY(ialloc(&H->partials, (size_t)kDirMaxBlocks + 1, "cost partials"));
    H->cap = need;
  }
  size_t words = 0, cells = 0;
  int bricks = 0, tiles = 0;
  for (auto& L : lv) {
    words = std::max(words, plan_words(L.shape));
    cells = std::max(cells, (size_t)cells_of(L.shape));
    bricks = std::max(bricks, bricks_of(L.shape));
    tiles = std::max(tiles, dir_tiles(L.shape));
  }
  if (words > H->plan_words || cells > H->plan_cells || bricks > H->plan_bricks || tiles > H->plan_tiles) {
    FA_HIP(hipStreamSynchronize(H->stream));
    free_plan(H);
    const size_t tickets = (size_t)(fa::kTicketSlots + 1) * fa::kTicketStride;
    FA_TRY(ialloc(&H->plan.count, words, "cell counts"));
    FA_TRY(ialloc(&H->plan.slots, 2 * cells, "voxels by cell"));
    FA_TRY(ialloc(&H->plan.box, (size_t)(2 * bricks), "brick boxes"));
    FA_TRY(ialloc(&H->plan.outside, (size_t)kDirMaxBlocks, "cost partials"));
    FA_TRY(ialloc(&H->plan.tile_loss, (size_t)tiles, "cost partials"));
    FA_TRY(ialloc(&H->plan.tickets, tickets, "tickets"));
    FA_HIP(fa::launch_fill(reinterpret_cast<float*>(H->plan.tickets), 0.0f, (int64_t)tickets, H->stream));
    H->plan_words = words;
    H->plan_cells = cells;
    H->plan_bricks = bricks;
    H->plan_tiles = tiles;
  }
  H->plan_level = -1;
  FA_TRY(ensure_acc(H));
  if (H->splat_direct)
    FA_HIP(hipMemsetAsync(H->acc, 0, (size_t)(3 * H->cap) * sizeof(unsigned long long), H->stream));
  if (total > H->loss_cap) {
    FA_HIP(hipStreamSynchronize(H->stream));
    if (H->loss_hist) (void)hipFree(H->loss_hist);
    H->loss_hist = nullptr;
    H->loss_cap = 0;
    FA_TRY(ialloc(&H->loss_hist, (size_t)total, "loss history"));
    H->loss_cap = (int)total;
  }

  // pyramid of the warp's field; m and e serve as scratch before the state is set
  if (!same) H->levels = lv;
  for (int i = 0; i < n_levels; ++i) {
    ILevel& L = H->levels[i];
    if (L.scale == 1.0f && full(L.shape)) {
      L.d = H->in_d;
      L.owns = false;
      continue;
    }
    if (!L.d) FA_TRY(ialloc(&L.d, (size_t)(3 * L.n), "level field"));
    L.owns = true;
    const fa_shape& s = H->shape;
    const float* src[3];
    float* dst[3];
    for (int c = 0; c < 3; ++c) {
      src[c] = H->in_d + c * H->n;
      dst[c] = L.d + c * L.n;
    }
    auto inv_rho = [](int nf, int nc) { return nc > 1 ? (float)((double)(nc - 1) / (double)(nf - 1)) : 1.0f; };
    const float rho[3] = {inv_rho(s.n0, L.shape.n0), inv_rho(s.n1, L.shape.n1), inv_rho(s.n2, L.shape.n2)};
    FA_HIP(fa::launch_level_images(src, dst, rho, 3, H->m, H->e, s.n0, s.n1, s.n2, L.shape.n0, L.shape.n1, L.shape.n2,
                                   H->wts + off_blur[i], fa::tap_radius(L.scale / 2.0f), H->stream));
  }

  // psi = id, m = v = 0, t = 0
  const int64_t n0 = H->levels[0].n;
  float* const zeroed[4] = {H->e, H->m, H->v, H->a};
  FA_HIP(fa::launch_start(zeroed, 3 * n0, H->ctl, H->p.adam_beta1, H->p.adam_beta2, nullptr, H->stream));
  H->cur_level = 0;
  H->cur_iter = 0;
  H->t_done = 0;
  H->iters_done = 0;
  H->scheduled = true;
  return FA_OK;
}

fa_status fa_inverse_step(fa_inverse H, int max_iters, int* iters_done, int* finished) {
  if (iters_done) *iters_done = 0;
  if (finished) *finished = 0;
  if (!H) return fail(FA_EINVAL, "handle is NULL");
  if (!H->scheduled) return fail(FA_ESTATE, "fa_inverse_set_schedule has not been called");
  if (max_iters < 0) return fail(FA_EINVAL, "max_iters must be >= 0");
  int done = 0;
  while (done < max_iters) {
    while (H->cur_level + 1 < (int)H->levels.size() && H->cur_iter >= H->levels[H->cur_level].iters) {
      FA_TRY(transition(H));
      H->cur_level += 1;
      H->cur_iter = 0;
    }
    if (schedule_done(H)) break;
    FA_TRY(launch_iteration(H, H->levels[H->cur_level]));
    H->cur_iter += 1;
    H->t_done += 1;
    H->iters_done += 1;
    done += 1;
  }
  if (iters_done) *iters_done = done;
  if (finished) *finished = schedule_done(H) ? 1 : 0;
  return FA_OK;
}

fa_status fa_inverse_get_field(fa_inverse H, float* dev_out, int* level, fa_shape* shape) {
  if (!H) return fail(FA_EINVAL, "handle is NULL");
  if (!H->scheduled) return fail(FA_ESTATE, "fa_inverse_set_schedule has not been called");
  const ILevel& L = H->levels[H->cur_level];
  if (level) *level = H->cur_level;
  if (shape) *shape = L.shape;
  if (dev_out)
    FA_HIP(hipMemcpyAsync(dev_out, H->e, (size_t)(3 * L.n) * sizeof(float), hipMemcpyDeviceToDevice, H->stream));
  return FA_OK;
}

fa_status fa_inverse_get_loss(fa_inverse H, float* host_out, int capacity, int* n_written) {
  if (n_written) *n_written = 0;
  if (!H) return fail(FA_EINVAL, "handle is NULL");
  if (!host_out && capacity > 0) return fail(FA_EINVAL, "host_out is NULL");
  const int cnt = std::min(std::max(capacity, 0), H->scheduled ? std::min(H->iters_done, H->loss_cap) : 0);
  FA_HIP(hipStreamSynchronize(H->stream));
  if (cnt > 0) FA_HIP(hipMemcpy(host_out, H->loss_hist, (size_t)cnt * sizeof(float), hipMemcpyDeviceToHost));
  if (n_written) *n_written = cnt;
  return FA_OK;
}

fa_status fa_inverse_eval_gradient(fa_inverse H, float* g_dev, float* loss_host) {
  if (!H) return fail(FA_EINVAL, "handle is NULL");
  if (!g_dev) return fail(FA_EINVAL, "g_dev is NULL");
  if (!H->scheduled) return fail(FA_ESTATE, "fa_inverse_set_schedule has not been called");
  const ILevel& L = H->levels[H->cur_level];
  FA_TRY(launch_direction(H, L, g_dev, 1));
  FA_HIP(fa::launch_partials_ratio(H->partials, direction_partials(H, L), -(double)L.n, H->scalar, H->stream));
  if (loss_host) {
    FA_HIP(hipMemcpyAsync(loss_host, H->scalar, sizeof(float), hipMemcpyDeviceToHost, H->stream));
    FA_HIP(hipStreamSynchronize(H->stream));
  }
  return FA_OK;
}

fa_status fa_inverse_set_splat(fa_inverse H, int direct) {
  if (!H) return fail(FA_EINVAL, "handle is NULL");
  if (direct != 0 && direct != 1) return fail(FA_EINVAL, "direct must be 0 or 1");
  if (direct && H->scheduled) FA_TRY(ensure_acc(H));   // else set_schedule allocates it
  H->splat_direct = direct != 0;
  return FA_OK;
}

void fa_inverse_destroy(fa_inverse H) {
  if (!H) return;
  (void)hipStreamSynchronize(H->stream);
  free_all(H);
  delete H;
}

}  // extern "C"
