// HIP kernels (gfx950) of the FireANTs dense matching step.
//
// One iteration of Algorithm 1 runs as four streaming launches:
//
//   grad   : LNCC window statistics of I_f and the warped image J = I_m(x + d),
//            LNCC adjoint, the Gateaux gradient g = dL/dJ * grad_p I_m
//            (Jacobian-free Eulerian descent, Section 4.4.2) and the Adam
//            update (Section 4.4) -> m, v, direction a; loss partials.
//   gauss  : s = G_sigma_grad * a stored, M = max |s|     (EPI_SMOOTH_MAX)
//   gauss  : single tap: u = -eta s / (2M) (Appendix E), d' = u + d(x + u)
//            (the retraction phi o (id + u) of Algorithm 1)  (EPI_COMPOSE_LDS)
//   gauss  : d = G_sigma_warp * d', and for the next iteration J = I_m(x + d)
//            with its slope grad_p I_m                       (EPI_STORE_WARP)
// The first workgroup of the composition, or of the warp smoothing where that
// is a brick launch, also records the loss and advances the Adam step count.
//
// Every streaming kernel gives a workgroup an in-plane tile (TY x TX columns
// along n1, n2) and marches it along n0 over a chunk of planes.  Window sums
// and Gaussian taps along n0 come from per-column register rings; the in-plane
// parts are separable passes over halo tiles staged in LDS.  The path is a
// stencil-and-gather workload bound by HBM bandwidth; there is no dense
// contraction, so no MFMA.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "fa_internal.h"

namespace fa {
namespace {

__device__ __forceinline__ int vidx(int z, int y, int x, int n1, int n2) {
  return (z * n1 + y) * n2 + x;
}

// M = max |s| over the slots of Ctl::mslot: cleared by threads 0..kMSlots-1
// of one workgroup, raised with one atomicMax per workgroup on the slot of
// its XCD (workgroups go to the XCDs round robin by linear index), read as
// the largest slot.
__device__ __forceinline__ void m_clear(Ctl* c, int tid) {
  if (tid < kMSlots) c->mslot[tid * kMStride] = 0u;
}
__device__ __forceinline__ void m_raise(Ctl* c, float bm, unsigned linear_block) {
  atomicMax(&c->mslot[(linear_block % kMSlots) * kMStride], __float_as_uint(bm));
}
__device__ __forceinline__ float m_value(const Ctl* c) {
  unsigned m = c->mslot[0];
#pragma unroll
  for (int j = 1; j < kMSlots; ++j) m = max(m, c->mslot[j * kMStride]);
  return __uint_as_float(m);
}

// Cell index and fraction of a sample coordinate, plus whether the lower and
// upper corners lie on the grid.  Coordinates far outside are clamped first
// (all corners are then off the grid anyway), which also keeps the integer
// conversion defined.
__device__ __forceinline__ void cell(float p, int n, int& i, float& t, bool& lo, bool& hi) {
  p = clamp_med3(p, -2.0f, (float)n + 1.0f);
  const float f = floorf(p);
  i = (int)f;
  t = p - f;
  lo = (i >= 0) & (i < n);
  hi = (i >= -1) & (i + 1 < n);
}

// The same for a sample at grid point x displaced by dd.  The cell index is
// x + floor(dd) and the fraction dd - floor(dd), so no precision is lost to
// forming x + dd in fp32: the cell is exactly the cell of the exact position
// (the trilinear derivative jumps between cells, so the cell matters) and the
// fraction is exact up to at most half an ulp of 1.
__device__ __forceinline__ void cell_at(int x, float dd, int n, int& i, float& t, bool& lo, bool& hi) {
  dd = clamp_med3(dd, (float)(-x - 2), (float)(n + 1 - x));
  const float f = floorf(dd);
  i = x + (int)f;
  t = dd - f;
  lo = (i >= 0) & (i < n);
  hi = (i >= -1) & (i + 1 < n);
}

struct Corners {
  int i0, i1, i2;
  bool a0, b0, a1, b1, a2, b2;
  float t0, t1, t2;
};

__device__ __forceinline__ Corners make_corners(int n0, int n1, int n2, float p0, float p1, float p2) {
  Corners c;
  cell(p0, n0, c.i0, c.t0, c.a0, c.b0);
  cell(p1, n1, c.i1, c.t1, c.a1, c.b1);
  cell(p2, n2, c.i2, c.t2, c.a2, c.b2);
  return c;
}

// Trilinear sample from its corners' values in the order 000, 001, ..., 111
// (zero where a corner is off the grid).
__device__ __forceinline__ float tri(const float v[8], const Corners& c) {
  const float e00 = v[0] + c.t2 * (v[1] - v[0]);
  const float e01 = v[2] + c.t2 * (v[3] - v[2]);
  const float e10 = v[4] + c.t2 * (v[5] - v[4]);
  const float e11 = v[6] + c.t2 * (v[7] - v[6]);
  const float f0 = e00 + c.t1 * (e01 - e00);
  const float f1 = e10 + c.t1 * (e11 - e10);
  return f0 + c.t0 * (f1 - f0);
}


// Number of grid points of [i - r, i + r] inside [0, n).
__device__ __forceinline__ float clipped_count(int i, int n, int r) {
  return (float)(min(i + r, n - 1) - max(i - r, 0) + 1);
}

// f(std::integral_constant<int, i>) for i = 0 .. N-1, each i a compile-time
// constant in f's body.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Box sums of two neighbouring outputs along a row: out[0] = in[0] + ... +
// in[W-1] and out[1] = in[1] + ... + in[W], each added left to right as a
// single output would be.  W is odd and in and out are 8-byte aligned, so the
// W + 1 inputs arrive as (W + 1) / 2 pair reads and the outputs as one pair
// write.
template <int W>
__device__ __forceinline__ void box_pair_x(const float* in, float* out) {
  float v[W + 1];
#pragma unroll
  for (int k = 0; k < (W + 1) / 2; ++k) {
    const float2 t = reinterpret_cast<const float2*>(in)[k];
    v[2 * k] = t.x;
    v[2 * k + 1] = t.y;
  }
  float a = v[0], b = v[1];
#pragma unroll
  for (int k = 1; k < W; ++k) {
    a += v[k];
    b += v[k + 1];
  }
  reinterpret_cast<float2*>(out)[0] = make_float2(a, b);
}

// The same with tap weights w[0..L-1]: out[0] = sum_k w[k] in[k] and out[1]
// = sum_k w[k] in[k + 1], each accumulated from k = 0 upwards.
template <int L>
__device__ __forceinline__ void tap_pair_x(const float* in, float* out, const float* w) {
  float v[L + 1];
#pragma unroll
  for (int k = 0; k < (L + 1) / 2; ++k) {
    const float2 t = reinterpret_cast<const float2*>(in)[k];
    v[2 * k] = t.x;
    v[2 * k + 1] = t.y;
  }
  float a = w[0] * v[0], b = w[0] * v[1];
#pragma unroll
  for (int k = 1; k < L; ++k) {
    a += w[k] * v[k];
    b += w[k] * v[k + 1];
  }
  reinterpret_cast<float2*>(out)[0] = make_float2(a, b);
}

template <int NT>
__device__ double block_sum(double v, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    for (int i = 0; i < NT / 64; ++i) s += red[i];
  }
  return s;  // meaningful on thread 0
}

template <int NT>
__device__ float block_max(float v, float* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_down(v, o, 64));
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  float s = 0.0f;
  if (threadIdx.x == 0) {
    for (int i = 0; i < NT / 64; ++i) s = fmaxf(s, red[i]);
  }
  return s;
}

// ---------------------------------------------------------------------------
// Fused LNCC + adjoint + Adam.
//
// Stage 1 (window statistics) runs on the tile plus a 2r halo: each column
// keeps the last W planes of I and J in registers, sums them along n0, and
// the in-plane box sums are two passes over LDS.  Stage 2 (adjoint box sums of
// the per-centre coefficients A, B, C) runs on the tile plus an r halo:
// in-plane passes first, then running sums along n0.  The output plane lags
// the input plane by 2r.
//
// The warped image J and its slope are sampled once per voxel, where d is made
// (EPI_STORE_WARP, k_warp), not on every halo column of the march: a tile of
// 16 x 32 outputs marches 24 x 40 columns over its chunk plus 4r planes, 2.4
// samples per voxel at 160x192x224 and window 5, each a chain of dependent
// loads whose registers and 24 KB of LDS (the slope's delay line) held the
// kernel at 4 waves per SIMD.  Without it window 5 fits 64 VGPRs and 37 KB,
// and 1024 threads share a tile's columns, one each: 8 waves per SIMD, which
// is what hides the LDS and memory latency that bound it.  Measured (us per
// launch at 160x192x224, events): window 3 162 -> 113, window 5 198 -> 125
// (582 MB, 4.7 TB/s), window 7 375 -> 179, window 9 441 -> 269.
// ---------------------------------------------------------------------------

// Trilinear gathers as 32-bit byte offsets from a uniform base pointer (the
// global loads then take the scalar-base form, with no per-lane 64-bit address
// arithmetic).  Every offset stays inside the volume (an axis whose corner is
// off the grid contributes offset 0), and an 8-bit mask zeroes the off-grid
// corners when the values are consumed.
__device__ __forceinline__ float load_at(const float* __restrict__ base, unsigned byte_off) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + (size_t)byte_off);
}

__device__ __forceinline__ void store_at(float* __restrict__ base, unsigned byte_off, float v) {
  *reinterpret_cast<float*>(reinterpret_cast<char*>(base) + (size_t)byte_off) = v;
}

// A uniform base pointer that stays in scalar registers.  The compiler may
// otherwise fold a component's offset (q * N) into the per-lane part of the
// address, which then takes 64-bit vector arithmetic and two vector registers
// per access; the empty asm hides where the pointer comes from.
typedef __attribute__((address_space(1))) float global_float;
__device__ __forceinline__ global_float* scalar_base(const float* p) {
  global_float* g = (global_float*)(uintptr_t)p;
  asm("" : "+s"(g));
  return g;
}
__device__ __forceinline__ float load_at(const global_float* base, unsigned byte_off) {
  typedef __attribute__((address_space(1))) char global_char;
  return *(const global_float*)((const global_char*)base + (size_t)byte_off);
}
__device__ __forceinline__ void store_at(global_float* base, unsigned byte_off, float v) {
  typedef __attribute__((address_space(1))) char global_char;
  *(global_float*)((global_char*)base + (size_t)byte_off) = v;
}

// Waits here for the load behind v.  Loads and stores share one in-order
// counter, and after a branch that may have skipped a store the compiler waits
// for all of them: a march therefore collects the loads of its next plane
// before it issues a plane's stores, instead of at the top of the next plane
// step, where the wait would include the stores just issued.
__device__ __forceinline__ void arrived(float& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ void axis_offsets(int x, float dd, int n, int stride_bytes, unsigned& lo,
                                             unsigned& hi, bool& lo_ok, bool& hi_ok, float& t) {
  dd = clamp_med3(dd, (float)(-x - 2), (float)(n + 1 - x));
  const float f = floorf(dd);
  const int i = x + (int)f;
  t = dd - f;
  lo_ok = i >= 0 && i < n;
  hi_ok = i >= -1 && i + 1 < n;
  lo = lo_ok ? (unsigned)(i * stride_bytes) : 0u;
  hi = hi_ok ? (unsigned)((i + 1) * stride_bytes) : 0u;
}

// The 8 corner offsets, validity mask and fractions of the sample at grid
// point (z, y, x) displaced by (d0, d1, d2); the cell is x + floor(d) as in
// cell_at.
struct Cell8 {
  unsigned off[8];
  unsigned mask;
  float t0, t1, t2;
};

__device__ __forceinline__ Cell8 cell8_at(int n0, int n1, int n2, int z, int y, int x, float d0, float d1,
                                          float d2) {
  Cell8 c;
  unsigned l0, h0, l1, h1, l2, h2;
  bool a0, b0, a1, b1, a2, b2;
  axis_offsets(z, d0, n0, n1 * n2 * 4, l0, h0, a0, b0, c.t0);
  axis_offsets(y, d1, n1, n2 * 4, l1, h1, a1, b1, c.t1);
  axis_offsets(x, d2, n2, 4, l2, h2, a2, b2, c.t2);
  const unsigned a00 = l0 + l1, a01 = l0 + h1, a10 = h0 + l1, a11 = h0 + h1;
  c.off[0] = a00 + l2;
  c.off[1] = a00 + h2;
  c.off[2] = a01 + l2;
  c.off[3] = a01 + h2;
  c.off[4] = a10 + l2;
  c.off[5] = a10 + h2;
  c.off[6] = a11 + l2;
  c.off[7] = a11 + h2;
  const unsigned mz = (a0 ? 0x0Fu : 0u) | (b0 ? 0xF0u : 0u);
  const unsigned my = (a1 ? 0x33u : 0u) | (b1 ? 0xCCu : 0u);
  const unsigned mx = (a2 ? 0x55u : 0u) | (b2 ? 0xAAu : 0u);
  c.mask = mz & my & mx;
  return c;
}

// Eight corner values of a trilinear sample (loaded; consumed later so that
// issuing the loads does not wait for them).
struct Gather {
  float c[8];
  unsigned mask;
  float t0, t1, t2;
};

// The same corners as four pairs of row neighbours: half the addresses of
// gather_issue for the same bytes, for kernels bound by them.  (Composition of
// two fields of 6.9 M voxels: 87 us against 95.)  A pair is clamped
// onto the grid, so that both its loads are in bounds (n2 >= 2).
struct CellPairs {
  unsigned off[4];
  bool up, down;   // clamped: both corners' values are the pair's second (first)
  unsigned mask;
  float t0, t1, t2;
};

__device__ __forceinline__ CellPairs pairs_at(int n0, int n1, int n2, int z, int y, int x, float d0, float d1,
                                              float d2) {
  CellPairs c;
  int i0, i1, i2;
  bool a0, b0, a1, b1, a2, b2;
  cell_at(z, d0, n0, i0, c.t0, a0, b0);
  cell_at(y, d1, n1, i1, c.t1, a1, b1);
  cell_at(x, d2, n2, i2, c.t2, a2, b2);
  const int x0 = min(max(i2, 0), n2 - 2);
  c.up = i2 > x0;
  c.down = i2 < x0;
  const int za = min(max(i0, 0), n0 - 1), zb = min(max(i0 + 1, 0), n0 - 1);
  const int ya = min(max(i1, 0), n1 - 1), yb = min(max(i1 + 1, 0), n1 - 1);
  c.off[0] = (unsigned)((za * n1 + ya) * n2 + x0) * 4u;
  c.off[1] = (unsigned)((za * n1 + yb) * n2 + x0) * 4u;
  c.off[2] = (unsigned)((zb * n1 + ya) * n2 + x0) * 4u;
  c.off[3] = (unsigned)((zb * n1 + yb) * n2 + x0) * 4u;
  const unsigned mz = (a0 ? 0x0Fu : 0u) | (b0 ? 0xF0u : 0u);
  const unsigned my = (a1 ? 0x33u : 0u) | (b1 ? 0xCCu : 0u);
  const unsigned mx = (a2 ? 0x55u : 0u) | (b2 ? 0xAAu : 0u);
  c.mask = mz & my & mx;
  return c;
}

typedef float float2_any __attribute__((ext_vector_type(2), aligned(4)));

struct PairGather {
  float2_any p[4];
};

__device__ __forceinline__ void gather_issue(const float* __restrict__ f, const CellPairs& c, PairGather& g) {
#pragma unroll
  for (int k = 0; k < 4; ++k)
    g.p[k] = *reinterpret_cast<const float2_any*>(reinterpret_cast<const char*>(f) + c.off[k]);
}

__device__ __forceinline__ Gather corners_of(const PairGather& p, const CellPairs& c) {
  Gather g;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    g.c[2 * k] = c.up ? p.p[k].y : p.p[k].x;
    g.c[2 * k + 1] = c.down ? p.p[k].x : p.p[k].y;
  }
  g.mask = c.mask;
  g.t0 = c.t0;
  g.t1 = c.t1;
  g.t2 = c.t2;
  return g;
}

__device__ __forceinline__ void gather_issue(const float* __restrict__ f, const Cell8& c, Gather& g) {
#pragma unroll
  for (int k = 0; k < 8; ++k) g.c[k] = load_at(f, c.off[k]);
  g.mask = c.mask;
  g.t0 = c.t0;
  g.t1 = c.t1;
  g.t2 = c.t2;
}

// The moving image of a level as row pairs with a zero border of kPad voxels
// on every side (launch_row_pairs): entry (z, y, x) of the padded grid holds
// the padded values at (z, y, x) and (z, y + 1, x).  A trilinear sample then
// takes two 16-byte loads (two neighbouring entries in the planes z and z + 1
// of its cell) instead of eight 4-byte ones with masks.  The cell is clamped
// to [-kPad, n], so every corner lies in the padded volume; a sample clamped
// this way lies wholly in the border, where value and derivative are 0 as with
// the masked form.  Byte offsets are 32-bit unsigned, and the padded plane
// size and every padded index stay below 2^24, so the index products are
// full-rate 24-bit multiplies (row_pairs_supported).
__device__ __forceinline__ void pair_axis(int x, float dd, int n, unsigned stride, unsigned& lo, float& t) {
  dd = clamp_med3(dd, (float)(-x - kPad), (float)(n - x));
  const float f = floorf(dd);
  lo = __umul24((unsigned)(x + kPad + (int)f), stride);   // padded index in [0, n + kPad]
  t = dd - f;
}

__device__ __forceinline__ void gather_issue_pairs(const float* __restrict__ q, int n0, int n1, int n2, int z, int y,
                                                   int x, float d0, float d1, float d2, Gather& g) {
  struct alignas(8) Two { float v[4]; };   // two entries, 8-byte aligned
  const unsigned p2 = (unsigned)(n2 + 2 * kPad), p1 = (unsigned)(n1 + 2 * kPad);
  unsigned l0, l1, l2;
  pair_axis(z, d0, n0, p1 * p2, l0, g.t0);
  pair_axis(y, d1, n1, p2, l1, g.t1);
  pair_axis(x, d2, n2, 1u, l2, g.t2);
  const char* b = reinterpret_cast<const char*>(q);
  const unsigned off = (l0 + l1 + l2) * 8u;
  const Two lo = *reinterpret_cast<const Two*>(b + (size_t)off);
  const Two hi = *reinterpret_cast<const Two*>(b + (size_t)(off + p1 * p2 * 8u));
  g.c[0] = lo.v[0];
  g.c[1] = lo.v[2];
  g.c[2] = lo.v[1];
  g.c[3] = lo.v[3];
  g.c[4] = hi.v[0];
  g.c[5] = hi.v[2];
  g.c[6] = hi.v[1];
  g.c[7] = hi.v[3];
  g.mask = 0xFFu;
}

__device__ __forceinline__ float gather_value(const Gather& g) {
  float v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = ((g.mask >> k) & 1u) ? g.c[k] : 0.0f;
  const float e00 = v[0] + g.t2 * (v[1] - v[0]);
  const float e01 = v[2] + g.t2 * (v[3] - v[2]);
  const float e10 = v[4] + g.t2 * (v[5] - v[4]);
  const float e11 = v[6] + g.t2 * (v[7] - v[6]);
  const float f0 = e00 + g.t1 * (e01 - e00);
  const float f1 = e10 + g.t1 * (e11 - e10);
  return f0 + g.t0 * (f1 - f0);
}

__device__ __forceinline__ float gather_value_grad(const Gather& g, float& g0, float& g1, float& g2) {
  float v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = ((g.mask >> k) & 1u) ? g.c[k] : 0.0f;
  const float dx00 = v[1] - v[0], dx01 = v[3] - v[2], dx10 = v[5] - v[4], dx11 = v[7] - v[6];
  const float e00 = v[0] + g.t2 * dx00;
  const float e01 = v[2] + g.t2 * dx01;
  const float e10 = v[4] + g.t2 * dx10;
  const float e11 = v[6] + g.t2 * dx11;
  const float dy0 = e01 - e00, dy1 = e11 - e10;
  const float f0 = e00 + g.t1 * dy0;
  const float f1 = e10 + g.t1 * dy1;
  const float dxy0 = dx00 + g.t1 * (dx01 - dx00);
  const float dxy1 = dx10 + g.t1 * (dx11 - dx10);
  g0 = f1 - f0;
  g1 = dy0 + g.t0 * (dy1 - dy0);
  g2 = dxy0 + g.t0 * (dxy1 - dxy0);
  return f0 + g.t0 * (f1 - f0);
}

// Stage-1 column c as (row, column) of the halo tile.  Columns 0 .. TY * TX - 1
// are the tile's own (column c belongs to output thread c); the rest enumerate
// the halo bands (top, bottom, left, right).
template <int TY, int TX, int H>
__device__ __forceinline__ bool column_coords(int c, int& ey, int& ex) {
  constexpr int NC = TY * TX;
  constexpr int EX = TX + 2 * H;
  if (c < NC) {
    ey = H + c / TX;
    ex = H + c % TX;
    return true;
  }
  if constexpr (H == 0) {
    ey = ex = 0;
    return false;
  } else {
    const int h = c - NC;
    constexpr int TB = H * EX;       // one horizontal band
    constexpr int LB = TY * H;       // one vertical band
    if (h < TB) {
      ey = h / EX;
      ex = h % EX;
    } else if (h < 2 * TB) {
      ey = H + TY + (h - TB) / EX;
      ex = (h - TB) % EX;
    } else if (h < 2 * TB + LB) {
      ey = H + (h - 2 * TB) / H;
      ex = (h - 2 * TB) % H;
    } else if (h < 2 * TB + 2 * LB) {
      ey = H + (h - 2 * TB - LB) / H;
      ex = H + TX + (h - 2 * TB - LB) % H;
    } else {
      ey = ex = 0;
      return false;
    }
    return true;
  }
}

// Extents of a march launch.  The loss alone (MODE 2) needs the window
// statistics of the tile's own centres, so its input halo is r instead of 2r
// and there is no second stage.
template <int W, int TY, int TX, int MODE>
struct GradShape {
  static constexpr int R = W / 2;
  static constexpr int H2 = MODE == 2 ? 0 : R;    // halo of the centres
  static constexpr int H1 = H2 + R;               // halo of the inputs
  static constexpr int E1Y = TY + 2 * H1, E1X = TX + 2 * H1, E1 = E1Y * E1X;
  static constexpr int E2Y = TY + 2 * H2, E2X = TX + 2 * H2, E2 = E2Y * E2X;
  static constexpr int XS1 = E1Y * E2X;
  static constexpr int XS2 = E2Y * TX;
  static constexpr size_t lds_bytes = sizeof(float) * (size_t)(5 * E1 + 5 * XS1);
};

// Two LDS offsets (in floats, below 2^16) that stay packed in one register:
// the asm keeps the compiler from unpacking them ahead of the march, where
// they would occupy two.
struct PackedOffsets {
  unsigned v;
  __device__ __forceinline__ void set(int lo, int hi) { v = (unsigned)lo | ((unsigned)hi << 16); }
  __device__ __forceinline__ void get(int& lo, int& hi) const {
    unsigned t = v;
    asm volatile("" : "+v"(t));
    lo = (int)(t & 0xffffu);
    hi = (int)(t >> 16);
  }
};

// NT threads per workgroup (at least TY * TX: thread c < TY * TX writes output
// column c).  MODE = A.mode: 0 gradient and Adam, 1 gradient, 2 loss.
template <int W, int TY, int TX, int NT, int MODE>
__device__ __forceinline__ void grad_body(const GradArgs& A, const int tile) {
  using S = GradShape<W, TY, TX, MODE>;
  constexpr int R = S::R, H1 = S::H1, H2 = S::H2;
  constexpr int E1X = S::E1X, E1 = S::E1;
  constexpr int E2X = S::E2X, E2 = S::E2;
  constexpr int XS1 = S::XS1, XS2 = S::XS2;
  constexpr int NC = TY * TX;
  constexpr int CPT1 = (E1 + NT - 1) / NT;
  // The in-plane x passes give each thread two neighbouring outputs (pair
  // reads along rows): every row length and array offset below is even.
  static_assert(TX % 2 == 0 && W % 2 == 1 && NT >= NC && NT % 64 == 0, "tile and workgroup shape");
  extern __shared__ __attribute__((aligned(16))) float glds[];
  float* buf = glds;             // [5][E1], later [3][E2]
  float* bufx = glds + 5 * E1;   // [5][XS1], later [3][XS2]
  __shared__ double red[NT / 64];

  const int tid = threadIdx.x;
  int b = tile;
  const int bx = b % A.tiles_x;
  b /= A.tiles_x;
  const int by = b % A.tiles_y;
  b /= A.tiles_y;
  const int n0 = A.n0, n1 = A.n1, n2 = A.n2;
  const int N = n0 * n1 * n2;
  const int plane = n1 * n2;
  const int z0 = b * A.zc;
  const int z1 = min(z0 + A.zc, n0);
  const int y0 = by * TY, x0 = bx * TX;

  int cl[CPT1];            // LDS offset of the column
  unsigned cpos[CPT1];     // its offset in a plane
  bool cin[CPT1], cuse[CPT1];
#pragma unroll
  for (int k = 0; k < CPT1; ++k) {
    int ey, ex;
    cuse[k] = column_coords<TY, TX, H1>(tid + k * NT, ey, ex);
    cl[k] = ey * E1X + ex;
    const int yy = y0 - H1 + ey, xx = x0 - H1 + ex;
    cin[k] = cuse[k] && yy >= 0 && yy < n1 && xx >= 0 && xx < n2;
    cpos[k] = cin[k] ? (unsigned)(yy * n2 + xx) : 0u;
  }
  const int oy = tid / TX, ox = tid % TX;
  const int gy = y0 + oy, gx = x0 + ox;
  const bool out_thread = NT == NC || tid < NC;
  const bool out_col = out_thread && gy < n1 && gx < n2;   // == cin[0] of an output thread

  // per-thread entries of the window-statistics pass (tile + H2 halo), the
  // tile's own first as for the columns: LDS offset and in-plane window count
  // (0 off the grid); fixed across planes
  constexpr int CPT2 = (E2 + NT - 1) / NT;
  int e2off[CPT2];
  float e2cnt[CPT2];
#pragma unroll
  for (int k = 0; k < CPT2; ++k) {
    int yo, xo;
    const bool use = column_coords<TY, TX, H2>(tid + k * NT, yo, xo);
    const int yy = y0 - H2 + yo, xx = x0 - H2 + xo;
    e2off[k] = yo * E2X + xo;
    const bool ok = use && yy >= 0 && yy < n1 && xx >= 0 && xx < n2;
    e2cnt[k] = ok ? clipped_count(yy, n1, R) * clipped_count(xx, n2, R) : 0.0f;
  }

  // x passes: X1P (X2P) pairs of outputs.  With threads to spare, groups of
  // threads share the quantities of a pair: X1G groups take every X1G-th of
  // the five, and three groups one each of A, B, C.
  constexpr int X1H = E2X / 2, X1P = S::E1Y * X1H;
  constexpr int X1G = NT >= 5 * X1P ? 5 : (NT >= X1P ? NT / X1P : 1);
  constexpr bool X1ONE = NT >= X1P;
  constexpr int X2H = TX / 2, X2P = S::E2Y * X2H;
  constexpr bool X2ONE = NT >= 3 * X2P;
  PackedOffsets x1{0u}, x2{0u};
  if constexpr (X1ONE) {
    const int g = tid / X1P, p = tid - g * X1P, yy = p / X1H, xo = 2 * (p - yy * X1H);
    if (g < X1G) x1.set(g * E1 + yy * E1X + xo, g * XS1 + yy * E2X + xo);
  }
  if constexpr (X2ONE) {
    const int g = tid / X2P, p = tid - g * X2P, yy = p / X2H, xo = 2 * (p - yy * X2H);
    if (g < 3) x2.set(g * E2 + yy * E2X + xo, g * XS2 + yy * TX + xo);
  }
  // LDS offsets of the thread's first column and first centre
  PackedOffsets own;
  own.set(cl[0], e2off[0]);

  float ringI[CPT1][W], ringJ[CPT1][W];
  // stage-2 sums along n0 in progress: entry j holds the sum of the last j + 1
  // planes, so a plane adds to each in turn and the window sum (oldest plane
  // first) leaves with one more add; no entry moves
  constexpr int WA = W > 1 ? W - 1 : 1;
  float accA[WA], accB[WA], accC[WA];
#pragma unroll
  for (int j = 0; j < W; ++j) {
#pragma unroll
    for (int k = 0; k < CPT1; ++k) { ringI[k][j] = 0.0f; ringJ[k][j] = 0.0f; }
  }
#pragma unroll
  for (int j = 0; j < WA; ++j) accA[j] = accB[j] = accC[j] = 0.0f;

  const float ibc1 = 1.0f / A.ctl->bc1, ibc2 = 1.0f / A.ctl->bc2;
  if (MODE == 0 && tile == 0) m_clear(A.ctl, tid);  // M of this iteration
  const float si = A.ctl->shift_i, sj = A.ctl->shift_j;
  const float gsc = (MODE == 1 && A.gscale) ? *A.gscale : 1.0f;
  float lacc = 0.0f;   // the own column's cc sum

  const int zs = z0 - H1, ze = z1 + H1;

  // I and J of the next plane, loaded one plane step ahead (zero off the grid)
  float nI[CPT1], nJ[CPT1];
  auto load_plane = [&](int z) {
    const bool zin = z >= 0 && z < n0;
    // byte offsets from uniform bases (volumes hold < 2^29 voxels)
    const unsigned zoff = (unsigned)((zin ? z : 0) * plane);
#pragma unroll
    for (int k = 0; k < CPT1; ++k) {
      nI[k] = si;
      nJ[k] = sj;
      if (zin && cin[k]) {
        const unsigned off = (zoff + cpos[k]) * 4u;
        nI[k] = load_at(A.fixed, off);
        nJ[k] = load_at(A.warped, off);
      }
    }
  };
  auto plane_arrived = [&]() {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < CPT1; ++k) {
      arrived(nI[k]);
      arrived(nJ[k]);
    }
  };
  load_plane(zs);
  plane_arrived();
  // the slope of the moving image and the Adam moments of the output plane
  float pg[3] = {0.f, 0.f, 0.f}, pm[3] = {0.f, 0.f, 0.f}, pv[3] = {0.f, 0.f, 0.f};
  global_float *bg[3], *bm[3], *bv[3], *bo[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (MODE != 2) bg[q] = scalar_base(A.slope + (size_t)q * N);
    if (MODE != 2) bo[q] = scalar_base(A.out + (size_t)q * N);
    if (MODE == 0) bm[q] = scalar_base(A.m + (size_t)q * N);
    if (MODE == 0) bv[q] = scalar_base(A.v + (size_t)q * N);
  }
  auto load_out = [&](unsigned off) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      pg[q] = load_at(bg[q], off);
      if (MODE == 0) {
        pm[q] = load_at(bm[q], off);
        pv[q] = load_at(bv[q], off);
      }
    }
  };

  // The register rings of I, J (per column) hold the last W planes and rotate
  // by moves each plane step.  Window 7 unrolls the march by W instead: at
  // phase ph of W the newest entry goes to slot ph, so the j-th oldest entry
  // sits at a slot fixed at compile time and no entry moves.  The sums run
  // oldest first.
  constexpr int UNZ = (W == 7 && TY == 16) ? W : 1;   // not the 8-row tiles of thin volumes
  auto step = [&](const int zin, auto PH) __attribute__((always_inline)) {
    constexpr int ph = decltype(PH)::value;
    // slot of the j-th oldest entry of the I/J rings
    auto ri = [](int j) constexpr { return UNZ == 1 ? j : (ph + 1 + j) % W; };
#pragma unroll
    for (int k = 0; k < CPT1; ++k) {
      if constexpr (UNZ == 1) {
#pragma unroll
        for (int j = 0; j < W - 1; ++j) {
          ringI[k][j] = ringI[k][j + 1];
          ringJ[k][j] = ringJ[k][j + 1];
        }
        ringI[k][W - 1] = nI[k] - si;
        ringJ[k][W - 1] = nJ[k] - sj;
      } else {
        ringI[k][ph] = nI[k] - si;
        ringJ[k][ph] = nJ[k] - sj;
      }
    }
    if (zin + 1 < ze) load_plane(zin + 1);

    if (zin >= z0 - H2 + R) {
#pragma unroll
      for (int k = 0; k < CPT1; ++k) {
        if (cuse[k]) {
          // sums start from the first term: 0 + x is not foldable in IEEE
          // arithmetic (signed zero) and would cost an add per sum
          const float i0 = ringI[k][ri(0)], j0 = ringJ[k][ri(0)];
          float s0 = i0, s1 = j0, s2 = i0 * i0, s3 = j0 * j0, s4 = i0 * j0;
          // Fused multiply-adds spelled out: which of the oldest two planes'
          // products is rounded and which fused into it is otherwise the
          // compiler's choice, in an unrolled march one by phase, and shows in
          // the last bits.  The oldest's is rounded at every plane, so that a
          // voxel's sums do not depend on where its chunk begins.
#pragma unroll
          for (int j = 1; j < W; ++j) {
            const float i_ = ringI[k][ri(j)], j_ = ringJ[k][ri(j)];
            s0 += i_;
            s1 += j_;
            s2 = __builtin_fmaf(i_, i_, s2);
            s3 = __builtin_fmaf(j_, j_, s3);
            s4 = __builtin_fmaf(i_, j_, s4);
          }
          int c = cl[k], c2;
          if (k == 0) own.get(c, c2);
          buf[c] = s0;
          buf[E1 + c] = s1;
          buf[2 * E1 + c] = s2;
          buf[3 * E1 + c] = s3;
          buf[4 * E1 + c] = s4;
        }
      }
      __syncthreads();
      {
        // one quantity at a time, in a rolled loop (unrolled over the five
        // quantities the pass measured slower, and it crowds the register
        // budget)
        if constexpr (X1ONE) {
          if (tid < X1G * X1P) {
            int src, dst;
            x1.get(src, dst);
            const int g = X1G == 1 ? 0 : tid / X1P;
#pragma unroll 1
            for (int q = g; q < 5; q += X1G) {
              box_pair_x<W>(buf + src, bufx + dst);
              src += X1G * E1;
              dst += X1G * XS1;
            }
          }
        } else {
          for (int p = tid; p < X1P; p += NT) {
            const int yy = p / X1H, xo = 2 * (p - yy * X1H);
            const float* src = buf + yy * E1X + xo;
            float* dst = bufx + yy * E2X + xo;
#pragma unroll 1
            for (int q = 0; q < 5; ++q) box_pair_x<W>(src + q * E1, dst + q * XS1);
          }
        }
      }
      __syncthreads();
      const int zc1 = zin - R;
      const bool z1ok = zc1 >= 0 && zc1 < n0;
      const float cz = clipped_count(zc1, n0, R);
      const bool z1out = zc1 >= z0 && zc1 < z1;
#pragma unroll
      for (int k2 = 0; k2 < CPT2; ++k2) {
        const int c = tid + k2 * NT;
        if (c >= E2) break;
        int c1, c2 = e2off[k2];
        if (k2 == 0) own.get(c1, c2);
        const float* src = bufx + c2;
        float SI = src[0], SJ = src[XS1], SII = src[2 * XS1], SJJ = src[3 * XS1], SIJ = src[4 * XS1];
#pragma unroll
        for (int k = 1; k < W; ++k) {
          SI += src[k * E2X];
          SJ += src[XS1 + k * E2X];
          SII += src[2 * XS1 + k * E2X];
          SJJ += src[3 * XS1 + k * E2X];
          SIJ += src[4 * XS1 + k * E2X];
        }
        float ca = 0.f, cb = 0.f, cc_ = 0.f;
        // A one-voxel window has zero variance and zero covariance exactly, so
        // its correlation and every coefficient are 0 (W == 1 skips the
        // arithmetic that would leave rounding residue).
        if (W > 1 && z1ok && e2cnt[k2] > 0.0f) {
          const float icnt = __builtin_amdgcn_rcpf(cz * e2cnt[k2]);
          const float muI = SI * icnt, muJ = SJ * icnt;
          const float cross = SIJ - muI * SJ;
          const float vI = SII - muI * SI;
          const float vJ = SJJ - muJ * SJ;
          const float D = vI * vJ + A.eps_cc;
          if (D != 0.0f) {
            const float invD = __builtin_amdgcn_rcpf(D);
            const float cc = cross * cross * invD;
            ca = 2.0f * cross * invD;
            cb = -2.0f * cc * vI * invD;
            cc_ = ca * muI + cb * muJ;
            if (k2 == 0 && z1out && out_thread) lacc += cc;   // the loss sums the tile's own centres
          }
        }
        if (MODE != 2) {
          buf[c2] = ca;
          buf[E2 + c2] = cb;
          buf[2 * E2 + c2] = cc_;
        }
      }
      // the loss alone: the next step's writes of buf come after the barrier
      // behind every read of it, and its x pass after the barrier behind the
      // reads of bufx above
      if constexpr (MODE != 2) {
        __syncthreads();
        {
          if constexpr (X2ONE) {
            if (tid < 3 * X2P) {
              int src, dst;
              x2.get(src, dst);
              box_pair_x<W>(buf + src, bufx + dst);
            }
          } else {
            for (int p = tid; p < X2P; p += NT) {
              const int yy = p / X2H, xo = 2 * (p - yy * X2H);
              const float* src = buf + yy * E2X + xo;
              float* dst = bufx + yy * TX + xo;
#pragma unroll
              for (int q = 0; q < 3; ++q) box_pair_x<W>(src + q * E2, dst + q * XS2);
            }
          }
        }
        const int zc2 = zc1 - R;
        if (zc2 >= z0 && out_col) load_out((unsigned)vidx(zc2, gy, gx, n1, n2) * 4u);
        __syncthreads();
        float SA = 0.0f, SB = 0.0f, SC = 0.0f;   // window sums of A, B, C around zc2
        if (out_thread) {
          const float* src = bufx + oy * TX + ox;
          float sa = src[0], sb = src[XS2], sc = src[2 * XS2];
#pragma unroll
          for (int k = 1; k < W; ++k) {
            sa += src[k * TX];
            sb += src[XS2 + k * TX];
            sc += src[2 * XS2 + k * TX];
          }
          if constexpr (W == 1) {
            SA = sa;
            SB = sb;
            SC = sc;
          } else {
            SA = accA[W - 2] + sa;
            SB = accB[W - 2] + sb;
            SC = accC[W - 2] + sc;
#pragma unroll
            for (int j = W - 2; j > 0; --j) {
              accA[j] = accA[j - 1] + sa;
              accB[j] = accB[j - 1] + sb;
              accC[j] = accC[j - 1] + sc;
            }
            accA[0] = sa;
            accB[0] = sb;
            accC[0] = sc;
          }
        }
        plane_arrived();
        if (zc2 >= z0 && out_col) {
          const unsigned off = (unsigned)vidx(zc2, gy, gx, n1, n2) * 4u;
          // oldest ring entries of the own column hold plane zc2
          // (spelled out, with the second product rounded: what is fused here
          // is otherwise the compiler's choice and shows in the last bits)
          float js = ringJ[0][ri(0)] * SB;
          asm("" : "+v"(js));
          const float dl = -A.inv_n * (__builtin_fmaf(ringI[0][ri(0)], SA, js) - SC);
          const float g[3] = {dl * pg[0], dl * pg[1], dl * pg[2]};
          if (MODE == 0) {
            const float b1 = A.beta1, b2 = A.beta2;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
              const float mm = b1 * pm[q] + (1.0f - b1) * g[q];
              const float vv = b2 * pv[q] + (1.0f - b2) * g[q] * g[q];
              store_at(bm[q], off, mm);
              store_at(bv[q], off, vv);
              store_at(bo[q], off, adam_direction(mm, vv, ibc1, ibc2, A.adam_eps));
            }
          } else {
#pragma unroll
            for (int q = 0; q < 3; ++q) store_at(bo[q], off, g[q] * gsc);
          }
        }
      }
    }
  };
  if constexpr (UNZ == 1) {
    for (int zin = zs; zin < ze; ++zin) step(zin, std::integral_constant<int, 0>{});
  } else {
    // the guard is uniform across the workgroup, so the barriers inside
    // are reached by every thread or by none
    for (int zb = zs; zb < ze; zb += UNZ)
      static_for<UNZ>([&](auto PH) __attribute__((always_inline)) {
        if (zb + decltype(PH)::value < ze) step(zb + decltype(PH)::value, PH);
      });
  }
  const double tot = block_sum<NT>((double)lacc, red);
  if (tid == 0) A.partials[tile] = tot;
}

// Threads and waves per SIMD of the march kernels.  Two threads per output
// column (one per column of the halo tile) where that fits 64 VGPRs, two
// workgroups per CU: windows 3 and 5.  Window 7 keeps 512 threads at 128 VGPRs,
// two workgroups per CU (one at 210 before).  Window 9 with Adam spills 30
// registers that way (463 us at 160x192x224) and takes 1024 threads, one
// workgroup per CU (269 us); its gradient alone (LNCC) spills 11 outside the
// passes and is still the faster form (127 against 139 us a pass at 128^3).
template <int W, int TY, int TX, int MODE>
struct GradLaunch {
  static constexpr bool TWO = TY == 16 && (W == 3 || W == 5 || (W == 9 && MODE == 0));
  static constexpr int NT = TWO ? 2 * TY * TX : TY * TX;
  static constexpr int WAVES = (W <= 5 && TY == 16) ? 8 : (TY == 16 ? 4 : 2);
};

template <int W, int TY, int TX, int MODE>
__global__ void __launch_bounds__((GradLaunch<W, TY, TX, MODE>::NT))
__attribute__((amdgpu_waves_per_eu(GradLaunch<W, TY, TX, MODE>::WAVES))) k_grad(const GradArgs A) {
  grad_body<W, TY, TX, GradLaunch<W, TY, TX, MODE>::NT, MODE>(A, xcd_tile(blockIdx.x, gridDim.x));
}

// ---------------------------------------------------------------------------
// Separable Gaussian (replicate boundary) on a 3-channel field, streaming.
// In-plane passes over a clamped halo tile in LDS, then a register ring of
// 2R+1 planes per output column along n0.  The next plane's loads are issued
// before the current plane's passes; the composition epilogue issues its
// gathers of d in one plane step and consumes them in the next.
// ---------------------------------------------------------------------------
// The iteration's loss record and Adam step count, run before its own work by
// the first workgroup of one launch after the gradient kernel (the launch
// whose GaussArgs carry the partials): the composition, or the warp smoothing
// where that is a brick launch (it costs the brick composition 0.6 us and the
// brick smoothing 0.1 us).  The gradient kernel of the iteration has written
// every loss partial, and no launch reads t or the bias corrections before
// the next iteration's gradient kernel.  No other workgroup waits for it, and
// the first workgroup is dispatched first.  The streaming smoothing launches
// never take it: inlined there, its registers cost occupancy or load
// pipelining at some radii.  The composition has registers to spare.  The partials are summed as 64-element
// chunks, each by one wave with the same shuffle tree, and the chunk sums in
// order by one thread: the sum does not depend on the workgroup size.
template <int NT>
__device__ __forceinline__ void record_iteration(const GaussArgs& A) {
  static_assert(NT % 64 == 0, "whole waves");
  constexpr int NW = NT / 64;
  __shared__ double csum[64];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int n = A.n_partials, nch = (n + 63) / 64;
  // the counters are fetched with the partials: one memory round trip
  Ctl* C = A.ctl;
  const int it = C->iter, t = C->t;
  const double bp1 = C->bp1, bp2 = C->bp2;
  const float b1 = C->beta1, b2 = C->beta2;
  double s = 0.0;
  for (int c0 = 0; c0 < nch; c0 += 64) {   // rounds of at most 64 chunks
    const int cend = min(nch, c0 + 64);
    for (int c = c0 + wid; c < cend; c += NW) {
      const int i = c * 64 + lane;
      double v = i < n ? A.partials[i] : 0.0;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
      if (lane == 0) csum[c - c0] = v;
    }
    __syncthreads();
    if (tid == 0)
      for (int c = c0; c < cend; ++c) s += csum[c - c0];
    __syncthreads();
  }
  if (tid == 0) {
    if (A.loss_hist && it >= 0 && it < A.loss_cap) A.loss_hist[it] = (float)(-s * (double)A.inv_n);
    C->iter = it + 1;
    C->t = t + 1;
    const double p1 = bp1 * (double)b1, p2 = bp2 * (double)b2;
    C->bp1 = p1;
    C->bp2 = p2;
    C->bc1 = (float)(1.0 - p1);
    C->bc2 = (float)(1.0 - p2);
  }
}

// J and its slope from a gathered cell of the moving image.
__device__ __forceinline__ void store_warp(const GaussArgs& A, const Gather& g, unsigned off, int N) {
  float g0, g1, g2;
  store_at(A.warped, off, gather_value_grad(g, g0, g1, g2));
  store_at(A.slope, off, g0);
  store_at(A.slope + N, off, g1);
  store_at(A.slope + 2 * N, off, g2);
}

template <int R, int TY, int TX, int EPI>
__device__ __forceinline__ void gauss_body(const GaussArgs& A, const int tile, const int nblocks) {
  constexpr int L = 2 * R + 1;
  constexpr int NT = TY * TX;
  constexpr int EY = TY + 2 * R, EX = TX + 2 * R, E = EY * EX;
  constexpr int XS = EY * TX;
  constexpr int CPT = (E + NT - 1) / NT;
  constexpr int DY = TY + 2, DX = TX + 2, DE = DY * DX;  // staged d planes (EPI_COMPOSE_LDS)
  // stride of the staged planes and components: DE rounded up to a multiple
  // of the 32 LDS banks, so that lanes of one row whose samples fall in
  // different planes (the sign of u0 flips along the row) read different
  // banks for different columns
  constexpr int DEP = (DE + 31) / 32 * 32;
  constexpr int CPTD = (DE + NT - 1) / NT;
  // the x pass gives each thread two neighbouring outputs (pair reads along
  // rows): EX, E, XS and every row offset are even
  static_assert(TX % 2 == 0, "pairs need an even tile width");
  extern __shared__ __attribute__((aligned(16))) float glds[];
  float* buf = glds;           // [3][E]
  float* bufx = glds + 3 * E;  // [3][XS]
  float* dring = glds + 3 * E + 3 * XS;  // [3 planes][3][DEP] (EPI_COMPOSE_LDS)
  __shared__ double red[NT / 64];

  const int tid = threadIdx.x;
  // the first tile of the composition records the iteration before its own work
  if ((EPI == EPI_COMPOSE_LDS || EPI == EPI_COMPOSE) && A.partials && tile == 0) record_iteration<NT>(A);
  int b = tile;
  const int bx = b % A.tiles_x;
  b /= A.tiles_x;
  const int by = b % A.tiles_y;
  b /= A.tiles_y;
  const int n0 = A.n0, n1 = A.n1, n2 = A.n2;
  const int N = n0 * n1 * n2;
  const int z0 = b * A.zc;
  const int z1 = min(z0 + A.zc, n0);
  const int y0 = by * TY, x0 = bx * TX;
  const int oy = tid / TX, ox = tid % TX;
  const int gy = y0 + oy, gx = x0 + ox;
  const bool out_col = gy < n1 && gx < n2;

  // clamped in-plane offsets of this thread's halo-tile columns
  int coff[CPT];
  bool cuse[CPT];
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = tid + k * NT;
    cuse[k] = c < E;
    const int yy = min(max(y0 - R + c / EX, 0), n1 - 1);
    const int xx = min(max(x0 - R + c % EX, 0), n2 - 1);
    coff[k] = yy * n2 + xx;
  }

  float w[L];
#pragma unroll
  for (int k = 0; k < L; ++k) w[k] = A.wts[k];
  float ring[3][L];
#pragma unroll
  for (int k = 0; k < L; ++k) ring[0][k] = ring[1][k] = ring[2][k] = 0.0f;

  float scale = 0.0f;
  if (EPI == EPI_COMPOSE || EPI == EPI_COMPOSE_LDS) {
    const float M = m_value(A.ctl);
    scale = M > 0.0f ? -A.eta / (2.0f * M) : 0.0f;
  }
  float mx = 0.0f;

  const int plane = n1 * n2;
  float pre[CPT][3];
  auto load_plane = [&](int z) {
    const int base = min(max(z, 0), n0 - 1) * plane;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      if (cuse[k]) {
        // byte offsets from uniform bases (volumes hold < 2^29 voxels)
        const unsigned off = (unsigned)(base + coff[k]) * 4u;
        pre[k][0] = load_at(A.in, off);
        pre[k][1] = load_at(A.in + N, off);
        pre[k][2] = load_at(A.in + 2 * N, off);
      }
    }
  };

  // d planes for the LDS composition: plane p lives in slot p mod 3 and
  // covers the tile plus one voxel on each side, zero off the grid (the
  // zero extension of the trilinear sample)
  float pd[CPTD][3];
  auto load_dplane = [&](int pz) {
#pragma unroll
    for (int k = 0; k < CPTD; ++k) {
      const int c = tid + k * NT;
      const int yy = y0 - 1 + c / DX, xx = x0 - 1 + c % DX;
      const bool ok = c < DE && pz >= 0 && pz < n0 && yy >= 0 && yy < n1 && xx >= 0 && xx < n2;
      const unsigned off = ok ? (unsigned)((pz * n1 + yy) * n2 + xx) * 4u : 0u;
      pd[k][0] = ok ? load_at(A.d, off) : 0.0f;
      pd[k][1] = ok ? load_at(A.d + N, off) : 0.0f;
      pd[k][2] = ok ? load_at(A.d + 2 * N, off) : 0.0f;
    }
  };
  auto store_dplane = [&](int pz) {
    const int slot = ((pz % 3) + 3) % 3;
#pragma unroll
    for (int k = 0; k < CPTD; ++k) {
      const int c = tid + k * NT;
      if (c < DE) {
        dring[(slot * 3 + 0) * DEP + c] = pd[k][0];
        dring[(slot * 3 + 1) * DEP + c] = pd[k][1];
        dring[(slot * 3 + 2) * DEP + c] = pd[k][2];
      }
    }
  };
  if (EPI == EPI_COMPOSE_LDS) {
    const int p0 = z0 - 2 * R + 1;   // plane stored by the first step (zin - R + 1)
    load_dplane(p0 - 2);
    store_dplane(p0 - 2);
    load_dplane(p0 - 1);
    store_dplane(p0 - 1);
    load_dplane(p0);
  }

  // composition gathers in flight (EPI_COMPOSE)
  Gather cg[3];
  float cu[3] = {0.f, 0.f, 0.f};
  int cidx = -1;
  auto finish_compose = [&]() {
    if (cidx >= 0) {
      A.out[cidx] = cu[0] + gather_value(cg[0]);
      A.out[N + cidx] = cu[1] + gather_value(cg[1]);
      A.out[2 * N + cidx] = cu[2] + gather_value(cg[2]);
      cidx = -1;
    }
  };

  // the sample of the moving image at the new d in flight (EPI_STORE_WARP)
  Gather wg;
  unsigned woff = 0u;
  bool wlive = false;
  auto finish_warp = [&]() {
    if (wlive) {
      store_warp(A, wg, woff, N);
      wlive = false;
    }
  };

  auto planes_arrived = [&]() {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      arrived(pre[k][0]);
      arrived(pre[k][1]);
      arrived(pre[k][2]);
    }
    if (EPI == EPI_COMPOSE_LDS) {
#pragma unroll
      for (int k = 0; k < CPTD; ++k) {
        arrived(pd[k][0]);
        arrived(pd[k][1]);
        arrived(pd[k][2]);
      }
    }
  };
  load_plane(z0 - R);
  planes_arrived();
  for (int zin = z0 - R; zin < z1 + R; ++zin) {
    if constexpr (R == 0) {
      // a single tap: the thread's own column is the output; no LDS passes
      ring[0][0] = pre[0][0];
      ring[1][0] = pre[0][1];
      ring[2][0] = pre[0][2];
      if (zin + 1 < z1) load_plane(zin + 1);
      if (EPI == EPI_COMPOSE_LDS) {
        __syncthreads();   // the previous step's reads of the d ring are done
        store_dplane(zin + 1);
        if (zin + 1 < z1) load_dplane(zin + 2);
        __syncthreads();
      }
      if (EPI == EPI_COMPOSE) finish_compose();
    } else {
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      if (cuse[k]) {
        const int c = tid + k * NT;
        buf[c] = pre[k][0];
        buf[E + c] = pre[k][1];
        buf[2 * E + c] = pre[k][2];
      }
    }
    if (zin + 1 < z1 + R) load_plane(zin + 1);
    __syncthreads();
    if (EPI == EPI_COMPOSE_LDS) {
      // plane zo + 1 joins the ring (slot of zo - 2, last read before the
      // barrier above); the next plane's loads go out now
      store_dplane(zin - R + 1);
      if (zin + 1 < z1 + R) load_dplane(zin - R + 2);
    }
    {
      constexpr int HX = TX / 2, PX = EY * HX;
      for (int p = tid; p < PX; p += NT) {
        const int yy = p / HX, xo = 2 * (p - yy * HX);
        const float* src = buf + yy * EX + xo;
        float* dst = bufx + yy * TX + xo;
#pragma unroll
        for (int q = 0; q < 3; ++q) tap_pair_x<L>(src + q * E, dst + q * XS, w);
      }
    }
    __syncthreads();
    if (EPI == EPI_COMPOSE) finish_compose();
    {
      const float* src = bufx + oy * TX + ox;
      float s0 = w[0] * src[0], s1 = w[0] * src[XS], s2 = w[0] * src[2 * XS];
#pragma unroll
      for (int k = 1; k < L; ++k) {
        s0 += w[k] * src[k * TX];
        s1 += w[k] * src[XS + k * TX];
        s2 += w[k] * src[2 * XS + k * TX];
      }
#pragma unroll
      for (int j = 0; j < L - 1; ++j) {
        ring[0][j] = ring[0][j + 1];
        ring[1][j] = ring[1][j + 1];
        ring[2][j] = ring[2][j + 1];
      }
      ring[0][L - 1] = s0;
      ring[1][L - 1] = s1;
      ring[2][L - 1] = s2;
    }
    }
    const int zo = zin - R;
    // the next plane's loads, and the previous plane's sample, before the stores
    planes_arrived();
    if (EPI == EPI_STORE_WARP) finish_warp();
    if (zo >= z0 && out_col) {
      float v0 = w[0] * ring[0][0], v1 = w[0] * ring[1][0], v2 = w[0] * ring[2][0];
#pragma unroll
      for (int j = 1; j < L; ++j) {
        v0 += w[j] * ring[0][j];
        v1 += w[j] * ring[1][j];
        v2 += w[j] * ring[2][j];
      }
      const int idx = vidx(zo, gy, gx, n1, n2);
      const unsigned off = (unsigned)idx * 4u;
      if (EPI == EPI_STORE || EPI == EPI_STORE_WARP) {
        if (EPI == EPI_STORE_WARP) {
          // finished next plane step; issued ahead of the stores, which the
          // wait for it would otherwise include (one counter, in order)
          gather_issue_pairs(A.moving_pairs, n0, n1, n2, zo, gy, gx, v0, v1, v2, wg);
          woff = off;
          wlive = true;
          __builtin_amdgcn_sched_barrier(0);
        }
        store_at(A.out, off, v0);
        store_at(A.out + N, off, v1);
        store_at(A.out + 2 * N, off, v2);
      } else if (EPI == EPI_SMOOTH_MAX) {
        store_at(A.out, off, v0);
        store_at(A.out + N, off, v1);
        store_at(A.out + 2 * N, off, v2);
        mx = fmaxf(mx, v0 * v0 + v1 * v1 + v2 * v2);
      } else if (EPI == EPI_COMPOSE_LDS) {
        // d' = u + d(x + u) from the staged planes zo - 1 .. zo + 1; the
        // cell offset floor(u) is -1 or 0 for |u| <= 1 (u = 1 exactly uses
        // offset 0 with fraction 1, which selects the same corner value)
        const float u0 = scale * v0, u1 = scale * v1, u2 = scale * v2;
        const float f0 = clamp_med3(floorf(u0), -1.0f, 0.0f);
        const float f1 = clamp_med3(floorf(u1), -1.0f, 0.0f);
        const float f2 = clamp_med3(floorf(u2), -1.0f, 0.0f);
        const float t0 = u0 - f0, t1 = u1 - f1, t2 = u2 - f2;
        const int sA = (((zo + (int)f0) % 3) + 3) % 3;
        const int sB = (sA + 1) % 3;
        const int cb = (oy + 1 + (int)f1) * DX + (ox + 1 + (int)f2);
        float res[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const float* pa = dring + (sA * 3 + q) * DEP + cb;
          const float* pb = dring + (sB * 3 + q) * DEP + cb;
          const float e00 = pa[0] + t2 * (pa[1] - pa[0]);
          const float e01 = pa[DX] + t2 * (pa[DX + 1] - pa[DX]);
          const float e10 = pb[0] + t2 * (pb[1] - pb[0]);
          const float e11 = pb[DX] + t2 * (pb[DX + 1] - pb[DX]);
          const float g0 = e00 + t1 * (e01 - e00);
          const float g1 = e10 + t1 * (e11 - e10);
          res[q] = g0 + t0 * (g1 - g0);
        }
        store_at(A.out, off, u0 + res[0]);
        store_at(A.out + N, off, u1 + res[1]);
        store_at(A.out + 2 * N, off, u2 + res[2]);
      } else {  // EPI_COMPOSE: d' = u + d(x + u); finished next plane step
        cu[0] = scale * v0;
        cu[1] = scale * v1;
        cu[2] = scale * v2;
        const Cell8 c = cell8_at(n0, n1, n2, zo, gy, gx, cu[0], cu[1], cu[2]);
        gather_issue(A.d, c, cg[0]);
        gather_issue(A.d + N, c, cg[1]);
        gather_issue(A.d + 2 * N, c, cg[2]);
        cidx = idx;
      }
    }
  }
  if (EPI == EPI_COMPOSE) finish_compose();
  if (EPI == EPI_STORE_WARP) finish_warp();

  if (EPI == EPI_SMOOTH_MAX) {
    const float bm = block_max<NT>(mx, reinterpret_cast<float*>(red));
    if (tid == 0) m_raise(A.ctl, sqrtf(bm), blockIdx.x);
  }
}

// ---------------------------------------------------------------------------
// Brick form of the gradient kernel for small volumes.  A workgroup takes a
// TZ x TY x TX brick: it loads I and J = I_m(x + d) on the brick plus a 2r
// halo, forms the window sums of I, J, I^2, J^2 and IJ with separable passes
// (x and y together, then z), the per-centre coefficients A, B, C on the
// brick plus an r halo, their window sums with three more passes, and the
// output as in k_grad.  No plane-by-plane march: the launch is a short chain
// of dependent steps, which is what bounds small volumes.  The sums run in a
// different order from the streaming form (x, y, z instead of z, x, y), so
// the two agree to rounding, not bitwise.
//
// Bound by LDS traffic and by the waits between the steps.  An item of a pass
// forms two to four neighbouring sums from one run of values, so a value is
// read about twice instead of w times.  Two threads per voxel fill the passes
// over the halo.  The x sums stay in registers and I and J are staged half the
// planes at a time (held in registers until then), so that two workgroups fit
// a CU's LDS (79 KiB at window 5 instead of 131) and one computes while the
// other loads or waits.  (Window 5: 64^3 18.4 -> 13.4 us, eight volumes of
// 48x56x52 135 -> 75; with the sums along x in LDS and one workgroup per CU
// 13.4 and 97.)
// ---------------------------------------------------------------------------
template <int W, int TZ, int TY, int TX>
struct GradCubeShape {
  static constexpr int R = W / 2;
  static constexpr int QZ = TZ + 4 * R, QY = TY + 4 * R, QX = TX + 4 * R, NQ = QZ * QY * QX;  // I, J
  static constexpr int CZ = TZ + 2 * R, CY = TY + 2 * R, CX = TX + 2 * R, NC = CZ * CY * CX;  // centres
  static constexpr int HZ = QZ / 2, NH = HZ * QY * QX;   // half the planes of I, J
  static constexpr int NY1 = QZ * CY * CX;   // stage-1 sums after the x and y passes
  static constexpr int NX2 = CZ * CY * TX;   // stage-2 sums after the x pass
  static constexpr int NY2 = CZ * TY * TX;   // ... after the y pass
  static constexpr int cmax(int a, int b) { return a > b ? a : b; }
  static constexpr int SA = cmax(5 * NY1, 3 * NX2);   // stage-1 xy -> stage-2 x
  static constexpr int SB = cmax(2 * NH, cmax(3 * NC, 3 * NY2));   // half of I, J -> A, B, C -> stage-2 y
  static constexpr size_t lds_bytes = sizeof(float) * (size_t)(SA + SB);
  static constexpr int NT = 2 * TZ * TY * TX;   // threads
  static constexpr int XT = CX % 4 == 0 ? 4 : 2;   // floats per vector read of a row of centres
  static_assert(QZ % 2 == 0 && CY % 2 == 0 && CZ % 2 == 0 && CX % XT == 0 && TX % 4 == 0 && TY % 4 == 0, "brick");
  static_assert(SA % 4 == 0 && NC % 4 == 0 && NX2 % 4 == 0, "vector alignment");
};

// N consecutive floats from LDS, A of them aligned to their size (2 or 4).
template <int N, int A>
__device__ __forceinline__ void lds_run(const float* p, float* v) {
  typedef float vec __attribute__((ext_vector_type(A)));
#pragma unroll
  for (int k = 0; k < N / A; ++k) {
    const vec u = reinterpret_cast<const vec*>(p)[k];
#pragma unroll
    for (int i = 0; i < A; ++i) v[A * k + i] = u[i];
  }
#pragma unroll
  for (int k = N / A * A; k < N; ++k) v[k] = p[k];
}
template <int A>
__device__ __forceinline__ void lds_put(float* p, const float* v) {
  typedef float vec __attribute__((ext_vector_type(A)));
  vec u;
#pragma unroll
  for (int i = 0; i < A; ++i) u[i] = v[i];
  *reinterpret_cast<vec*>(p) = u;
}

// MODE = A.mode (0 gradient and Adam, 1 gradient, 2 loss).
template <int W, int TZ, int TY, int TX, int MODE>
__device__ __forceinline__ void grad_cube_body(const GradArgs& A, const int tile) {
  using S = GradCubeShape<W, TZ, TY, TX>;
  constexpr int R = S::R;
  constexpr int NT = S::NT;
  constexpr int QY = S::QY, QX = S::QX, NQ = S::NQ;
  constexpr int CY = S::CY, CX = S::CX, NC = S::NC;
  constexpr int HZ = S::HZ, NH = S::NH, NY1 = S::NY1, NX2 = S::NX2, NY2 = S::NY2, XT = S::XT;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* bufA = lds;
  float* bufB = lds + S::SA;
  __shared__ double red[NT / 64];

  const int tid = threadIdx.x;
  int b = tile;
  const int bx = b % A.tiles_x;
  b /= A.tiles_x;
  const int by = b % A.tiles_y;
  b /= A.tiles_y;
  const int n0 = A.n0, n1 = A.n1, n2 = A.n2;
  const int N = n0 * n1 * n2;
  const int z0 = b * TZ, y0 = by * TY, x0 = bx * TX;
  const float si = A.ctl->shift_i, sj = A.ctl->shift_j;
  if (MODE == 0 && tile == 0) m_clear(A.ctl, tid);  // M of this iteration

  // stage-1 inputs on the brick plus 2r (zero off the grid): every load is
  // issued before any is consumed
  constexpr int KQ = (NQ + NT - 1) / NT;   // voxels per thread
  float qI[KQ], qJ[KQ];
#pragma unroll
  for (int j = 0; j < KQ; ++j) {
    const int c = tid + j * NT;
    const int qz = c / (QY * QX), r = c - qz * (QY * QX);
    const int qy = r / QX, qx = r - qy * QX;
    const int z = z0 - 2 * R + qz, y = y0 - 2 * R + qy, x = x0 - 2 * R + qx;
    const bool ok = c < NQ && z >= 0 && z < n0 && y >= 0 && y < n1 && x >= 0 && x < n2;
    qI[j] = si;
    qJ[j] = sj;
    if (ok) {
      const unsigned off = (unsigned)vidx(z, y, x, n1, n2) * 4u;
      qI[j] = load_at(A.fixed, off);
      qJ[j] = load_at(A.warped, off);
    }
  }

  // the thread's own output voxel: I, J, the slope and the Adam moments
  const int tz = tid / (TY * TX), tr = tid - tz * (TY * TX);
  const int ty = tr / TX, tx = tr - ty * TX;
  const int oz = z0 + tz, oy = y0 + ty, ox = x0 + tx;
  const bool own = tid < TZ * TY * TX && oz < n0 && oy < n1 && ox < n2;
  // byte offset of the own voxel from uniform bases (volumes hold < 2^29 voxels)
  const unsigned ooff = own ? (unsigned)vidx(oz, oy, ox, n1, n2) * 4u : 0u;
  float oI = 0.f, oJ = 0.f;
  float pg[3] = {0.f, 0.f, 0.f}, pm[3] = {0.f, 0.f, 0.f}, pv[3] = {0.f, 0.f, 0.f};
  if (MODE != 2 && own) {
    oI = load_at(A.fixed, ooff) - si;
    oJ = load_at(A.warped, ooff) - sj;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      pg[q] = load_at(A.slope + q * N, ooff);
      if (MODE == 0) {
        pm[q] = load_at(A.m + q * N, ooff);
        pv[q] = load_at(A.v + q * N, ooff);
      }
    }
  }
  // Stage 1, x and y, half of the planes at a time: an item forms the x sums of
  // I, J, I^2, J^2, IJ of a column's W + 1 rows and from them its two sums along y.
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h) __syncthreads();   // the first half's reads are done
#pragma unroll
    for (int j = 0; j < KQ; ++j) {
      const int c = tid + j * NT - h * NH;
      if (c >= 0 && c < NH) {
        bufB[c] = qI[j] - si;
        bufB[NH + c] = qJ[j] - sj;
      }
    }
    __syncthreads();
    constexpr int YG = CY / 2;
    for (int c = tid; c < HZ * YG * CX; c += NT) {
      const int zg = c / CX, xo = c - zg * CX;
      const int zq = zg / YG, yo = (zg - zq * YG) * 2;
      const float* pI = bufB + (zq * QY + yo) * QX + xo;
      const float* pJ = pI + NH;
      float sum[2][5];
#pragma unroll
      for (int r = 0; r < W + 1; ++r) {
        float i_[W], j_[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
          i_[k] = pI[r * QX + k];
          j_[k] = pJ[r * QX + k];
        }
        // the second product is rounded and the first fused into it: which is
        // otherwise the compiler's choice and shows in the last bits
        constexpr int k0 = W > 1 ? 1 : 0;
        float s[5] = {i_[0], j_[0], i_[k0] * i_[k0], j_[k0] * j_[k0], i_[k0] * j_[k0]};
#pragma unroll
        for (int k = 1; k < W; ++k) {
          s[0] += i_[k];
          s[1] += j_[k];
          const float ia = i_[k == 1 ? 0 : k], ja = j_[k == 1 ? 0 : k];
          s[2] = __builtin_fmaf(ia, ia, s[2]);
          s[3] = __builtin_fmaf(ja, ja, s[3]);
          s[4] = __builtin_fmaf(ia, ja, s[4]);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int q = 0; q < 5; ++q) {
            if (r == t) sum[t][q] = s[q];
            if (r > t && r < t + W) sum[t][q] += s[q];
          }
      }
      float* o = bufA + ((h * HZ + zq) * CY + yo) * CX + xo;
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        o[q * NY1] = sum[0][q];
        o[q * NY1 + CX] = sum[1][q];
      }
    }
  }
  __syncthreads();
  // stage 1, z, and the per-centre coefficients on the brick plus r
  float lacc = 0.0f;
  constexpr int ZT = 2;   // planes per item
  for (int ci = tid; ci < NC / ZT; ci += NT) {
    const int zi = ci / (CY * CX), r = ci - zi * (CY * CX);
    const int cy = r / CX, cx = r - cy * CX;
    const float* src = bufA + zi * ZT * CY * CX + r;
    float Sz[ZT][5];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const float* p = src + q * NY1;
      float v[ZT + W - 1];
#pragma unroll
      for (int k = 0; k < ZT + W - 1; ++k) v[k] = p[k * CY * CX];
#pragma unroll
      for (int t = 0; t < ZT; ++t) {
        float sum = v[t];
#pragma unroll
        for (int k = 1; k < W; ++k) sum += v[t + k];
        Sz[t][q] = sum;
      }
    }
#pragma unroll
    for (int t = 0; t < ZT; ++t) {
    const int cz = zi * ZT + t, c = cz * (CY * CX) + r;
    const float* St = Sz[t];
    const int z = z0 - R + cz, y = y0 - R + cy, x = x0 - R + cx;
    const bool ok = z >= 0 && z < n0 && y >= 0 && y < n1 && x >= 0 && x < n2;
    float ca = 0.f, cb = 0.f, cc_ = 0.f;
    // a one-voxel window has zero variance and covariance: every coefficient is 0
    if (W > 1 && ok) {
      const float cnt = clipped_count(z, n0, R) * (clipped_count(y, n1, R) * clipped_count(x, n2, R));
      const float icnt = __builtin_amdgcn_rcpf(cnt);
      const float muI = St[0] * icnt, muJ = St[1] * icnt;
      const float cross = St[4] - muI * St[1];
      const float vI = St[2] - muI * St[0];
      const float vJ = St[3] - muJ * St[1];
      const float D = vI * vJ + A.eps_cc;
      if (D != 0.0f) {
        const float invD = __builtin_amdgcn_rcpf(D);
        const float cc = cross * cross * invD;
        ca = 2.0f * cross * invD;
        cb = -2.0f * cc * vI * invD;
        cc_ = ca * muI + cb * muJ;
        if (cz >= R && cz < R + TZ && cy >= R && cy < R + TY && cx >= R && cx < R + TX) lacc += cc;
      }
    }
    bufB[c] = ca;
    bufB[NC + c] = cb;
    bufB[2 * NC + c] = cc_;
    }
  }
  if constexpr (MODE != 2) {
  __syncthreads();
  // stage 2 (sums of A, B, C over the window around each brick voxel), x
  constexpr int G2 = TX / 4, NXI = NX2 / 4;
  for (int c = tid; c < 3 * NXI; c += NT) {
    const int q = c / NXI, cq = c - q * NXI;
    const int row = cq / G2, xo = (cq - row * G2) * 4;
    float v[4 + W - 1], o[4];
    lds_run<4 + W - 1, XT>(bufB + q * NC + row * CX + xo, v);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float sum = v[t];
#pragma unroll
      for (int k = 1; k < W; ++k) sum += v[t + k];
      o[t] = sum;
    }
    lds_put<4>(bufA + q * NX2 + row * TX + xo, o);
  }
  __syncthreads();
  // stage 2, y
  constexpr int G3 = TY / 4, NYJ = NY2 / 4;
  for (int c = tid; c < 3 * NYJ; c += NT) {
    const int q = c / NYJ, cq = c - q * NYJ;
    const int zg = cq / TX, xo = cq - zg * TX;
    const int zc = zg / G3, yo = (zg - zc * G3) * 4;
    const float* p = bufA + q * NX2 + (zc * CY + yo) * TX + xo;
    float v[4 + W - 1];
#pragma unroll
    for (int k = 0; k < 4 + W - 1; ++k) v[k] = p[k * TX];
    float* o = bufB + q * NY2 + (zc * TY + yo) * TX + xo;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float sum = v[t];
#pragma unroll
      for (int k = 1; k < W; ++k) sum += v[t + k];
      o[t * TX] = sum;
    }
  }
  __syncthreads();
  // stage 2, z, and the output
  if (own) {
    const float* src = bufB + (tz * TY + ty) * TX + tx;
    float SA = src[0], SB = src[NY2], SC = src[2 * NY2];
#pragma unroll
    for (int k = 1; k < W; ++k) {
      SA += src[k * TY * TX];
      SB += src[NY2 + k * TY * TX];
      SC += src[2 * NY2 + k * TY * TX];
    }
    const float dl = -A.inv_n * (oI * SA + oJ * SB - SC);
    const float g[3] = {dl * pg[0], dl * pg[1], dl * pg[2]};
    if (MODE == 0) {
      const float ibc1 = 1.0f / A.ctl->bc1, ibc2 = 1.0f / A.ctl->bc2;
      const float b1 = A.beta1, b2 = A.beta2;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float mm = b1 * pm[q] + (1.0f - b1) * g[q];
        const float vv = b2 * pv[q] + (1.0f - b2) * g[q] * g[q];
        store_at(A.m + q * N, ooff, mm);
        store_at(A.v + q * N, ooff, vv);
        store_at(A.out + q * N, ooff, adam_direction(mm, vv, ibc1, ibc2, A.adam_eps));
      }
    } else {
      const float gsc = A.gscale ? *A.gscale : 1.0f;
#pragma unroll
      for (int q = 0; q < 3; ++q) store_at(A.out + q * N, ooff, g[q] * gsc);
    }
  }
  }
  const double tot = block_sum<NT>((double)lacc, red);
  if (tid == 0) A.partials[tile] = tot;
}

// ---------------------------------------------------------------------------
// Brick forms of the smoothing and composition kernels for small volumes.
// A workgroup takes a TZ x TY x TX brick, loads its clamped halo region into
// LDS and runs the three separable passes there (x, then y, then z, the
// order and summation of k_gauss, so the results are bitwise those of the
// streaming form).  With no march along n0, a launch is a few dependent
// steps long instead of one step per plane of a chunk plus its halo.
// ---------------------------------------------------------------------------
// Threads of a brick launch of the smoothing.  Two per voxel fill the passes
// over the halo (R = 3, 64^3: 5.9 us against 6.2 with one); where half of them
// would then wait for the others' samples, one (R = 2, eight volumes of
// 48x56x52: 22 us against 26 with two).  An item of a pass forms four sums from
// one run of values, of which each is then read from LDS two to three times
// instead of 2R + 1 (with one sum per item: 7.5 us and 23).
template <int TZ, int TY, int TX, int EPI>
constexpr int kCubeThreads = (EPI == EPI_SMOOTH_MAX ? 2 : 1) * TZ * TY * TX;

// Sum of L taps.  The second product is rounded and the first fused into it:
// which is otherwise the compiler's choice and shows in the last bits.
template <int L>
__device__ __forceinline__ float tap_sum(const float* w, const float* v) {
  if constexpr (L == 1) return w[0] * v[0];
  float s = __builtin_fmaf(w[0], v[0], w[1] * v[1]);
#pragma unroll
  for (int k = 2; k < L; ++k) s = __builtin_fmaf(w[k], v[k], s);
  return s;
}

template <int R, int TZ, int TY, int TX, int EPI>
__device__ __forceinline__ void gauss_cube_body(const GaussArgs& A, const int tile, const int nblocks) {
  constexpr int L = 2 * R + 1;
  constexpr int NT = kCubeThreads<TZ, TY, TX, EPI>;
  constexpr int RZ = TZ + 2 * R, RY = TY + 2 * R, RX = TX + 2 * R;
  constexpr int NR = RZ * RY * RX;   // halo region
  constexpr int NX = RZ * RY * TX;   // after the x-pass
  constexpr int NY = RZ * TY * TX;   // after the y-pass
  static_assert(NY <= NR, "y-pass output reuses the region buffer");
  static_assert(RX % 2 == 0 && NR % 2 == 0 && 3 * NR % 4 == 0 && NX % 4 == 0, "vector alignment");
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* reg = lds;            // [3][NR], later [3][NY]
  float* xo = lds + 3 * NR;    // [3][NX]
  __shared__ double red[NT / 64];

  const int tid = threadIdx.x;
  // the first brick of a warp smoothing that records the iteration does so first
  if ((EPI == EPI_STORE || EPI == EPI_STORE_WARP) && A.partials && tile == 0) record_iteration<NT>(A);
  int b = tile;
  const int bx = b % A.tiles_x;
  b /= A.tiles_x;
  const int by = b % A.tiles_y;
  b /= A.tiles_y;
  const int n0 = A.n0, n1 = A.n1, n2 = A.n2;
  const int N = n0 * n1 * n2;
  const int z0 = b * TZ, y0 = by * TY, x0 = bx * TX;

  float w[L];
#pragma unroll
  for (int k = 0; k < L; ++k) w[k] = A.wts[k];

  // the region's loads are all issued before any is consumed
  constexpr int KR = (NR + NT - 1) / NT;
  float rv[KR][3];
#pragma unroll
  for (int k = 0; k < KR; ++k) {
    const int c = min(tid + k * NT, NR - 1);
    const int zz = c / (RY * RX), r = c - zz * (RY * RX);
    const int yy = r / RX, xx = r - yy * RX;
    const int gz = min(max(z0 - R + zz, 0), n0 - 1);
    const int gy = min(max(y0 - R + yy, 0), n1 - 1);
    const int gx = min(max(x0 - R + xx, 0), n2 - 1);
    const unsigned off = (unsigned)((gz * n1 + gy) * n2 + gx) * 4u;
    rv[k][0] = load_at(A.in, off);
    rv[k][1] = load_at(A.in + N, off);
    rv[k][2] = load_at(A.in + 2 * N, off);
  }
#pragma unroll
  for (int k = 0; k < KR; ++k) {
    const int c = tid + k * NT;
    if (c < NR) {
      reg[c] = rv[k][0];
      reg[NR + c] = rv[k][1];
      reg[2 * NR + c] = rv[k][2];
    }
  }
  __syncthreads();
  // x, four neighbours of a row and one component per item
  constexpr int XG = TX / 4, NXI = NX / 4;
  for (int c = tid; c < 3 * NXI; c += NT) {
    const int q = c / NXI, cq = c - q * NXI;
    const int row = cq / XG, xx = (cq - row * XG) * 4;
    float v[4 + L - 1], o[4];
    lds_run<4 + L - 1, 2>(reg + q * NR + row * RX + xx, v);
#pragma unroll
    for (int t = 0; t < 4; ++t) o[t] = tap_sum<L>(w, v + t);
    lds_put<4>(xo + q * NX + row * TX + xx, o);
  }
  __syncthreads();
  // y, four outputs of a column per item
  constexpr int YG = TY / 4, NYI = NY / 4;
  for (int c = tid; c < 3 * NYI; c += NT) {
    const int q = c / NYI, cq = c - q * NYI;
    const int zg = cq / TX, xx = cq - zg * TX;
    const int zz = zg / YG, yy = (zg - zz * YG) * 4;
    const float* src = xo + q * NX + (zz * RY + yy) * TX + xx;
    float v[4 + L - 1];
#pragma unroll
    for (int k = 0; k < 4 + L - 1; ++k) v[k] = src[k * TX];
    float* o = reg + q * NY + (zz * TY + yy) * TX + xx;
#pragma unroll
    for (int t = 0; t < 4; ++t) o[t * TX] = tap_sum<L>(w, v + t);
  }
  __syncthreads();
  const int tz = tid / (TY * TX), r = tid - tz * (TY * TX);
  const int ty = r / TX, tx = r - ty * TX;
  const int gz = z0 + tz, gy = y0 + ty, gx = x0 + tx;
  float mx = 0.0f;
  if (tid < TZ * TY * TX && gz < n0 && gy < n1 && gx < n2) {
    const float* src = reg + (tz * TY + ty) * TX + tx;
    float vz[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      float v[L];
#pragma unroll
      for (int j = 0; j < L; ++j) v[j] = src[q * NY + j * TY * TX];
      vz[q] = tap_sum<L>(w, v);
    }
    const float v0 = vz[0], v1 = vz[1], v2 = vz[2];
    const unsigned off = (unsigned)vidx(gz, gy, gx, n1, n2) * 4u;
    store_at(A.out, off, v0);
    store_at(A.out + N, off, v1);
    store_at(A.out + 2 * N, off, v2);
    if (EPI == EPI_SMOOTH_MAX) mx = v0 * v0 + v1 * v1 + v2 * v2;
    if (EPI == EPI_STORE_WARP) {
      Gather g;
      gather_issue_pairs(A.moving_pairs, n0, n1, n2, gz, gy, gx, v0, v1, v2, g);
      store_warp(A, g, off, N);
    }
  }
  if (EPI == EPI_SMOOTH_MAX) {
    const float bm = block_max<NT>(mx, reinterpret_cast<float*>(red));
    if (tid == 0) m_raise(A.ctl, sqrtf(bm), blockIdx.x);
  }
}

// d' = u + d(x + u), u = -eta s / (2M), |u| <= 1 voxel, on a brick: d is
// staged in LDS on the brick plus one voxel (zero off the grid).  Runs in
// place over s: each thread reads s only at the voxel it writes.
template <int TZ, int TY, int TX>
__device__ __forceinline__ void compose_cube_body(const GaussArgs& A, const int tile) {
  constexpr int NT = TZ * TY * TX;
  constexpr int DZ = TZ + 2, DY = TY + 2, DX = TX + 2, DE = DZ * DY * DX;
  extern __shared__ __attribute__((aligned(16))) float lds[];   // [3][DE]
  const int tid = threadIdx.x;
  // the first brick records the iteration before its own work
  if (A.partials && tile == 0) record_iteration<NT>(A);
  int b = tile;
  const int bx = b % A.tiles_x;
  b /= A.tiles_x;
  const int by = b % A.tiles_y;
  b /= A.tiles_y;
  const int n0 = A.n0, n1 = A.n1, n2 = A.n2;
  const int N = n0 * n1 * n2;
  const int z0 = b * TZ, y0 = by * TY, x0 = bx * TX;
  constexpr int KD = (DE + NT - 1) / NT;
  float dv[KD][3];
#pragma unroll
  for (int k = 0; k < KD; ++k) {
    const int c = tid + k * NT;
    const int zz = c / (DY * DX), r = c - zz * (DY * DX);
    const int yy = r / DX, xx = r - yy * DX;
    const int gz = z0 - 1 + zz, gy = y0 - 1 + yy, gx = x0 - 1 + xx;
    const bool ok = c < DE && gz >= 0 && gz < n0 && gy >= 0 && gy < n1 && gx >= 0 && gx < n2;
    const unsigned off = ok ? (unsigned)((gz * n1 + gy) * n2 + gx) * 4u : 0u;
    dv[k][0] = ok ? load_at(A.d, off) : 0.0f;
    dv[k][1] = ok ? load_at(A.d + N, off) : 0.0f;
    dv[k][2] = ok ? load_at(A.d + 2 * N, off) : 0.0f;
  }
#pragma unroll
  for (int k = 0; k < KD; ++k) {
    const int c = tid + k * NT;
    if (c < DE) {
      lds[c] = dv[k][0];
      lds[DE + c] = dv[k][1];
      lds[2 * DE + c] = dv[k][2];
    }
  }
  const float M = m_value(A.ctl);
  const float scale = M > 0.0f ? -A.eta / (2.0f * M) : 0.0f;
  const int tz = tid / (TY * TX), r = tid - tz * (TY * TX);
  const int ty = r / TX, tx = r - ty * TX;
  const int gz = z0 + tz, gy = y0 + ty, gx = x0 + tx;
  const bool own = gz < n0 && gy < n1 && gx < n2;
  const unsigned off = own ? (unsigned)vidx(gz, gy, gx, n1, n2) * 4u : 0u;
  float sv[3] = {0.f, 0.f, 0.f};
  if (own) {
    sv[0] = load_at(A.in, off);
    sv[1] = load_at(A.in + N, off);
    sv[2] = load_at(A.in + 2 * N, off);
  }
  __syncthreads();
  if (own) {
    // the arithmetic of k_gauss<0, EPI_COMPOSE_LDS>: floor(u) is -1 or 0
    const float u0 = scale * sv[0], u1 = scale * sv[1], u2 = scale * sv[2];
    const float f0 = clamp_med3(floorf(u0), -1.0f, 0.0f);
    const float f1 = clamp_med3(floorf(u1), -1.0f, 0.0f);
    const float f2 = clamp_med3(floorf(u2), -1.0f, 0.0f);
    const float t0 = u0 - f0, t1 = u1 - f1, t2 = u2 - f2;
    const int cb = ((tz + 1 + (int)f0) * DY + (ty + 1 + (int)f1)) * DX + (tx + 1 + (int)f2);
    float res[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const float* pa = lds + q * DE + cb;
      const float* pb = pa + DY * DX;
      const float e00 = pa[0] + t2 * (pa[1] - pa[0]);
      const float e01 = pa[DX] + t2 * (pa[DX + 1] - pa[DX]);
      const float e10 = pb[0] + t2 * (pb[1] - pb[0]);
      const float e11 = pb[DX] + t2 * (pb[DX + 1] - pb[DX]);
      const float g0 = e00 + t1 * (e01 - e00);
      const float g1 = e10 + t1 * (e11 - e10);
      res[q] = g0 + t0 * (g1 - g0);
    }
    store_at(A.out, off, u0 + res[0]);
    store_at(A.out + N, off, u1 + res[1]);
    store_at(A.out + 2 * N, off, u2 + res[2]);
  }
}

// ---------------------------------------------------------------------------
// Kernels of the iteration, in two forms.  The plain form runs one
// registration, with its arguments in the kernel arguments.  The batch form
// runs several registrations in one launch: entry e of a table in device
// memory holds the arguments of one registration and its range of
// workgroups in the launch, and owner[g] names the entry of workgroup g
// (after the XCD renumbering, so each XCD takes a contiguous range of the
// batch's tiles).  A workgroup loads its entry's arguments once, with scalar
// loads, and then runs the same body as the plain form.
// ---------------------------------------------------------------------------
// A pointer loaded from memory is generic to the compiler, and accesses
// through it become flat instructions (which also count against the LDS
// wait counter, so every LDS wait would wait for them too).  Each pointer is
// rebuilt from its integer value as a global-address-space pointer, which
// tells the compiler what it knows for kernel arguments: the body then uses
// global instructions.  (A plain cast to the global space and back is folded
// away before the address spaces are inferred.)
template <class T>
__device__ __forceinline__ T* as_global(T* p) {
  typedef __attribute__((address_space(1))) T GT;
  return (T*)(GT*)(uintptr_t)p;
}

__device__ __forceinline__ void load_args(const GradArgs* __restrict__ s, GradArgs& A) {
  A.fixed = as_global(s->fixed);
  A.warped = as_global(s->warped);
  A.slope = as_global(s->slope);
  A.m = as_global(s->m);
  A.v = as_global(s->v);
  A.out = as_global(s->out);
  A.gscale = as_global(s->gscale);
  A.partials = as_global(s->partials);
  A.ctl = as_global(s->ctl);
  A.n0 = s->n0;
  A.n1 = s->n1;
  A.n2 = s->n2;
  A.zc = s->zc;
  A.tiles_y = s->tiles_y;
  A.tiles_x = s->tiles_x;
  A.eps_cc = s->eps_cc;
  A.beta1 = s->beta1;
  A.beta2 = s->beta2;
  A.adam_eps = s->adam_eps;
  A.inv_n = s->inv_n;
  A.mode = s->mode;
}

__device__ __forceinline__ void load_args(const GaussArgs* __restrict__ s, GaussArgs& A) {
  A.in = as_global(s->in);
  A.out = as_global(s->out);
  A.d = as_global(s->d);
  A.moving_pairs = as_global(s->moving_pairs);
  A.warped = as_global(s->warped);
  A.slope = as_global(s->slope);
  A.wts = as_global(s->wts);
  A.ctl = as_global(s->ctl);
  A.partials = as_global(s->partials);
  A.loss_hist = as_global(s->loss_hist);
  A.loss_cap = s->loss_cap;
  A.n_partials = s->n_partials;
  A.inv_n = s->inv_n;
  A.eta = s->eta;
  A.n0 = s->n0;
  A.n1 = s->n1;
  A.n2 = s->n2;
  A.zc = s->zc;
  A.tiles_y = s->tiles_y;
  A.tiles_x = s->tiles_x;
}

template <class Args>
__device__ __forceinline__ int batch_entry(const BatchEntry<Args>* __restrict__ E, const int* __restrict__ owner,
                                           Args& A, int& nblocks) {
  const int g = xcd_tile(blockIdx.x, gridDim.x);
  const int e = owner[g];
  load_args(&E[e].a, A);
  nblocks = E[e].nblocks;
  return g - E[e].first;
}

template <int W, int TY, int TX, int MODE>
__global__ void __launch_bounds__((GradLaunch<W, TY, TX, MODE>::NT))
__attribute__((amdgpu_waves_per_eu(GradLaunch<W, TY, TX, MODE>::WAVES)))
k_grad_batch(const BatchEntry<GradArgs>* __restrict__ E, const int* __restrict__ owner) {
  GradArgs A;
  int nb;
  const int tile = batch_entry(E, owner, A, nb);
  grad_body<W, TY, TX, GradLaunch<W, TY, TX, MODE>::NT, MODE>(A, tile);
}

template <int R, int TY, int TX, int EPI>
__global__ void __launch_bounds__(TY * TX) k_gauss(const GaussArgs A) {
  gauss_body<R, TY, TX, EPI>(A, xcd_tile(blockIdx.x, gridDim.x), gridDim.x);
}

template <int R, int TY, int TX, int EPI>
__global__ void __launch_bounds__(TY * TX) k_gauss_batch(const BatchEntry<GaussArgs>* __restrict__ E,
                                                         const int* __restrict__ owner) {
  GaussArgs A;
  int nb;
  const int tile = batch_entry(E, owner, A, nb);
  gauss_body<R, TY, TX, EPI>(A, tile, nb);
}

template <int W, int TZ, int TY, int TX, int MODE>
__global__ void __launch_bounds__((GradCubeShape<W, TZ, TY, TX>::NT)) k_grad_cube(const GradArgs A) {
  grad_cube_body<W, TZ, TY, TX, MODE>(A, xcd_tile(blockIdx.x, gridDim.x));
}

template <int W, int TZ, int TY, int TX, int MODE>
__global__ void __launch_bounds__((GradCubeShape<W, TZ, TY, TX>::NT)) k_grad_cube_batch(const BatchEntry<GradArgs>* __restrict__ E,
                                                                  const int* __restrict__ owner) {
  GradArgs A;
  int nb;
  const int tile = batch_entry(E, owner, A, nb);
  grad_cube_body<W, TZ, TY, TX, MODE>(A, tile);
}

template <int R, int TZ, int TY, int TX, int EPI>
__global__ void __launch_bounds__((kCubeThreads<TZ, TY, TX, EPI>)) k_gauss_cube(const GaussArgs A) {
  gauss_cube_body<R, TZ, TY, TX, EPI>(A, xcd_tile(blockIdx.x, gridDim.x), gridDim.x);
}

template <int R, int TZ, int TY, int TX, int EPI>
__global__ void __launch_bounds__((kCubeThreads<TZ, TY, TX, EPI>)) k_gauss_cube_batch(const BatchEntry<GaussArgs>* __restrict__ E,
                                                                   const int* __restrict__ owner) {
  GaussArgs A;
  int nb;
  const int tile = batch_entry(E, owner, A, nb);
  gauss_cube_body<R, TZ, TY, TX, EPI>(A, tile, nb);
}

template <int TZ, int TY, int TX>
__global__ void __launch_bounds__(TZ * TY * TX) k_compose_cube(const GaussArgs A) {
  compose_cube_body<TZ, TY, TX>(A, xcd_tile(blockIdx.x, gridDim.x));
}

template <int TZ, int TY, int TX>
__global__ void __launch_bounds__(TZ * TY * TX) k_compose_cube_batch(const BatchEntry<GaussArgs>* __restrict__ E,
                                                                     const int* __restrict__ owner) {
  GaussArgs A;
  int nb;
  const int tile = batch_entry(E, owner, A, nb);
  compose_cube_body<TZ, TY, TX>(A, tile);
}

// ---------------------------------------------------------------------------
// Off-loop kernels: pyramid blur and resampling, warp, fills, layout copies.
// ---------------------------------------------------------------------------
// Algorithm 1 with use_jac: the descent direction is J(phi)^T dU/dphi
// (Section 4.4.2, Eulerian descent), J(phi) = I + grad d; component a is
// g_a + sum_c (d d_c / d x_a) g_c, with grad d by central differences inside
// the grid and one-sided differences on its faces.  Adam follows, as in the
// gradient kernel's own epilogue.  In place: each thread reads g only at the
// voxel whose direction it writes.
__global__ void __launch_bounds__(256)
k_eulerian_adam(float* __restrict__ ga, const float* __restrict__ d, float* __restrict__ m,
                float* __restrict__ v, Ctl* ctl, int n0, int n1, int n2, float beta1, float beta2,
                float adam_eps) {
  const int N = n0 * n1 * n2;
  if (blockIdx.x == 0) m_clear(ctl, threadIdx.x);   // M of this iteration
  const float ibc1 = 1.0f / ctl->bc1, ibc2 = 1.0f / ctl->bc2;
  const int plane = n1 * n2;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
    const int x2 = i % n2, t = i / n2;
    const int x1 = t % n1, x0 = t / n1;
    const int xs[3] = {x0, x1, x2}, ns[3] = {n0, n1, n2}, st[3] = {plane, n2, 1};
    float g[3], out[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) g[c] = ga[c * N + i];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const bool has_lo = xs[a] > 0, has_hi = xs[a] < ns[a] - 1;
      const int lo = has_lo ? i - st[a] : i, hi = has_hi ? i + st[a] : i;
      const float h = (has_lo && has_hi) ? 0.5f : 1.0f;
      float r = g[a];
#pragma unroll
      for (int c = 0; c < 3; ++c) r += (d[c * N + hi] - d[c * N + lo]) * h * g[c];
      out[a] = r;
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int iq = q * N + i;
      const float mm = beta1 * m[iq] + (1.0f - beta1) * out[q];
      const float vv = beta2 * v[iq] + (1.0f - beta2) * out[q] * out[q];
      m[iq] = mm;
      v[iq] = vv;
      ga[iq] = adam_direction(mm, vv, ibc1, ibc2, adam_eps);
    }
  }
}

// Voxel (z, y, x) and flat index i of this thread in an n0 x n1 x n2 launch:
// on a (n2 / blockDim, n1, n0) grid (G3) from the block indices, with no
// integer divisions; else from a flat index.  False past the end of a row or
// of the volume.
template <bool G3>
__device__ __forceinline__ bool grid_voxel(int n0, int n1, int n2, int& z, int& y, int& x, int& i) {
  if constexpr (G3) {
    x = blockIdx.x * blockDim.x + threadIdx.x;
    y = blockIdx.y;
    z = blockIdx.z;
    i = (z * n1 + y) * n2 + x;
    return x < n2;
  } else {
    i = blockIdx.x * blockDim.x + threadIdx.x;
    x = i % n2;
    y = (i / n2) % n1;
    z = i / (n1 * n2);
    return i < n0 * n1 * n2;
  }
}

// Row pairs of the padded image (gather_issue_pairs), from the image itself:
// grid (ceil(p2 / blockDim), p1, p0) over the padded extents, or flat.
template <bool G3>
__global__ void k_row_pairs(const float* __restrict__ in, float2* __restrict__ out, int n0, int n1, int n2) {
  int z, y, x, i;
  if (!grid_voxel<G3>(n0 + 2 * kPad, n1 + 2 * kPad, n2 + 2 * kPad, z, y, x, i)) return;
  z -= kPad;
  y -= kPad;
  x -= kPad;
  const bool zx = z >= 0 && z < n0 && x >= 0 && x < n2;
  const bool lo = zx && y >= 0 && y < n1, hi = zx && y >= -1 && y + 1 < n1;
  const int at = vidx(z, y, x, n1, n2);
  float2 v;
  v.x = lo ? in[at] : 0.0f;
  v.y = hi ? in[at + n2] : 0.0f;
  out[i] = v;
}

__global__ void k_fill(float* __restrict__ p, float value, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

// ---- Gaussian smoothing of a field with a radius above kMaxRadius ----------
// One separable pass of a 3-component field [3][n0][n1][n2] along one axis:
// out_c(x) = sum_{k=-R..R} w[k+R] in_c(x + k e_axis), the index clamped to the
// grid (replicate), the taps summed in that order.  The radius is a run-time
// value up to kMaxWideRadius.  A workgroup stages its line segment (outputs
// plus R on each side) in LDS once and every output reads its 2R+1 taps from
// there.
//
// Along n2: a workgroup of 256 threads takes 256 consecutive voxels of one
// row (grid: ceil(n2/256), n1, n0).
__global__ void __launch_bounds__(256) k_field_wide_x(const float* __restrict__ in, float* __restrict__ out,
                                                      int n0, int n1, int n2, const float* __restrict__ w, int R) {
  extern __shared__ float wl[];   // [3][256 + 2R]
  const int L = 256 + 2 * R;
  const int x0 = blockIdx.x * 256, y = blockIdx.y, z = blockIdx.z;
  const int64_t N = (int64_t)n0 * n1 * n2;
  const int64_t row = ((int64_t)z * n1 + y) * n2;
  // L <= 512: two values per thread and component, all loads in flight at once
  float pre[3][2];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      pre[c][u] = in[c * N + row + min(max(x0 - R + (int)threadIdx.x + 256 * u, 0), n2 - 1)];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = threadIdx.x + 256 * u;
      if (i < L) wl[c * L + i] = pre[c][u];
    }
  __syncthreads();
  const int x = x0 + threadIdx.x;
  if (x >= n2) return;
  for (int c = 0; c < 3; ++c) {
    const float* src = wl + c * L + threadIdx.x;
    float acc = w[0] * src[0];
    for (int k = 1; k <= 2 * R; ++k) acc += w[k] * src[k];
    out[c * N + row + x] = acc;
  }
}

// Along n1 (axis 1) or n0 (axis 0): a workgroup of 64 x 8 threads takes 64
// consecutive n2 columns and kWideRun consecutive positions along the axis
// (grid: ceil(n2/64), ceil(n_axis/kWideRun), the remaining axis); thread
// (lane, j) forms the 8 consecutive outputs 8j .. 8j+7 of its column from a
// sliding window of 8 registers: taps go in blocks of 8 (the tap tables are
// zero-padded to a multiple of 16, so the block past 2R + 1 adds exact
// zeros), and each staged input is read from LDS once per thread instead of
// once per tap.  One component is staged at a time.  The last pass (axis 0)
// also runs the smoothing's epilogue (EPI): the max norm M of the result
// (EPI_SMOOTH_MAX), as the streaming kernels do; E carries the control block.
// (64 positions: at radius 18 a run of 32 re-read 36 halo positions for
// every 32 outputs; runs of up to 96, as few as cover the axis, hold too few
// wavefronts: 429 us an iteration at 131x177x219 against 411)
constexpr int kWideRun = 64, kWideRows = kWideRun / 8, kWideThreads = 64 * kWideRows;
constexpr int kWideLoads = (kWideRun + (2 * kMaxWideRadius + 8) / 8 * 8) / kWideRows;   // staged values per thread
template <int AX, int EPI>
__global__ void __launch_bounds__(kWideThreads) k_field_wide_yz(const float* __restrict__ in, float* __restrict__ out,
                                                       int n0, int n1, int n2, const float* __restrict__ w, int R,
                                                       const GaussArgs E) {
  extern __shared__ float wl[];   // [kWideRun + L8][64], one component at a time
  __shared__ float red[kWideRows];
  const int L8 = (2 * R + 1 + 7) / 8 * 8;
  const int LS = kWideRun + L8;
  const int lane = threadIdx.x & 63, j0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: scalar addresses
  const int x = blockIdx.x * 64 + lane;
  const int a0 = blockIdx.y * kWideRun;
  const int na = AX == 0 ? n0 : n1;
  const int other = blockIdx.z;   // y for AX == 0, z for AX == 1
  const int64_t N = (int64_t)n0 * n1 * n2;
  const int64_t astride = AX == 0 ? (int64_t)n1 * n2 : (int64_t)n2;
  const int64_t base = AX == 0 ? (int64_t)other * n2 : (int64_t)other * n1 * n2;
  const bool xin = x < n2;
  const int bo = 8 * j0;          // this thread's outputs, relative to a0
  float v[3][8];
  // A component's staged values are loaded together, while the one before is
  // formed: a load and its LDS write in turn cost a memory latency each, 13 per
  // component.  (An iteration with sigma_grad 6 at 131x177x219: 437 -> 405 us,
  // at 33x44x55 60 -> 48.)
  float pre[kWideLoads];
  auto fetch = [&](int c) {
    const float* src = in + c * N + base + min(x, n2 - 1);
#pragma unroll
    for (int u = 0; u < kWideLoads; ++u)
      pre[u] = src[min(max(a0 - R + min(j0 + u * kWideRows, LS - 1), 0), na - 1) * astride];
  };
  fetch(0);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (c > 0) __syncthreads();   // the previous component's reads are done
#pragma unroll
    for (int u = 0; u < kWideLoads; ++u)
      if (j0 + u * kWideRows < LS) wl[(j0 + u * kWideRows) * 64 + lane] = pre[u];
    __syncthreads();
    if (c < 2) fetch(c + 1);
    float acc[8], xr[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) {
      acc[o] = 0.0f;
      xr[o] = wl[(bo + o) * 64 + lane];
    }
    for (int k = 0; k < L8; k += 8) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const float wk = w[k + m];
#pragma unroll
        for (int o = 0; o < 8; ++o) acc[o] += wk * xr[(m + o) & 7];
        xr[m] = wl[(bo + k + m + 8) * 64 + lane];
      }
    }
#pragma unroll
    for (int o = 0; o < 8; ++o) {
      v[c][o] = acc[o];
      if (xin && a0 + bo + o < na) out[c * N + base + (int64_t)(a0 + bo + o) * astride + x] = acc[o];
    }
  }
  float mx = 0.0f;
  if (EPI == EPI_SMOOTH_MAX && xin) {
#pragma unroll
    for (int o = 0; o < 8; ++o)
      if (a0 + bo + o < na) mx = fmaxf(mx, v[0][o] * v[0][o] + v[1][o] * v[1][o] + v[2][o] * v[2][o]);
  }
  if (EPI == EPI_SMOOTH_MAX) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_down(mx, o, 64));
    if (lane == 0) red[j0] = mx;
    __syncthreads();
    float bm = 0.0f;
    if (threadIdx.x == 0)
      for (int j = 0; j < kWideRows; ++j) bm = fmaxf(bm, red[j]);
    if (threadIdx.x == 0) m_raise(E.ctl, sqrtf(bm), blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
  }
}

__device__ __forceinline__ float aligned_pos(int i, int nin, int nout) {
  return nout > 1 ? (float)(i * (nin - 1)) / (float)(nout - 1) : 0.0f;
}

// ---- level images ------------------------------------------------------------
// A level's image is the input blurred along n0, n1, n2 and sampled trilinearly
// at corner-aligned positions.  Along an axis of n inputs and m samples only
// the 2m entries floor(pos) and floor(pos) + 1 of the blurred input are read,
// so where 2m < n ("compact", and wherever the radius is above 3) the passes along n0 and n1 form only those, entry
// 2k + b at input floor(pos(k)) + b, and the last pass blurs along n2 just the
// eight corners it samples.  The taps, their order and the sample are those of
// the full blur, so the values are the same.  At scale 8 the first pass writes
// a quarter of the volume and the second a sixteenth.  (512^3, scales 8, 4, 2,
// two images: 2.2 ms; 13.9 when every entry was blurred and then resampled, the
// radius-12 passes 10.3 of them.)  Up to three images go through one launch per pass.
struct Images {
  const float* in[3];
  float* out[3];
};

// Splits a launch over `outer` rows of `inner` consecutive items: whole
// workgroups per row (BLK), so that everything but the item is uniform, or flat
// over all items where a row is too short to fill a wavefront.
template <bool BLK>
__device__ __forceinline__ bool row_item(unsigned block, unsigned inner, unsigned outer, unsigned& row,
                                         unsigned& item) {
  if constexpr (BLK) {
    const unsigned nb = (inner + blockDim.x - 1) / blockDim.x;
    row = block / nb;
    item = (block - row * nb) * blockDim.x + threadIdx.x;
    return item < inner;
  } else {
    const unsigned t = block * blockDim.x + threadIdx.x;
    row = t / inner;
    item = t - row * inner;
    return row < outer;
  }
}

// floor of the position of sample k
__device__ __forceinline__ int aligned_cell(int k, int nin, int nout) {
  int i;
  float t;
  bool lo, hi;
  cell(aligned_pos(k, nin, nout), nin, i, t, lo, hi);
  return i;
}

// Entries 2k and 2k + 1 (inputs floor(pos(k)) and the next) of the blur along
// n0 (AX 0) or n1 (AX 1) of `count` images [n0][n1][n2]: na is the blurred axis'
// inputs, nm its samples, n_other the other of the two axes.  Both entries take
// the 2R + 2 inputs they share; radius RT, or R at run time (RT = 0).  A thread
// takes kg consecutive k, so that the inputs that neighbouring k share (26 - 8
// of 26 at scale 8) come from the caches.
template <int AX, int RT, bool BLK>
__global__ void __launch_bounds__(256) k_blur_pairs(const Images im, unsigned count, int na, int nm, int n_other,
                                                    int n2, const float* __restrict__ w, int Rr, int kg) {
  const int R = RT ? RT : Rr;
  // a row: the items [n_other][n2] (AX 0) or [n2] at one n0 (AX 1) of one image and one group of k
  const unsigned inner = AX == 0 ? (unsigned)n_other * n2 : (unsigned)n2;
  const unsigned groups = (unsigned)(nm + kg - 1) / kg;
  const unsigned per_image = AX == 0 ? groups : n_other * groups;
  unsigned row, item;
  if (!row_item<BLK>(blockIdx.x, inner, per_image * count, row, item)) return;
  const unsigned img = row / per_image, r = row - img * per_image, z = AX == 0 ? 0u : r / groups;
  const int k0 = (int)(r - z * groups) * kg;
  const size_t stride = inner;
  const float* src = im.in[img] + (size_t)z * na * stride + item;
  float* dst = im.out[img] + ((size_t)z * (2 * nm) + 2 * k0) * stride + item;
  for (int k = k0; k < min(k0 + kg, nm); ++k, dst += 2 * stride) {
    const int f = aligned_cell(k, na, nm);
    float s0 = 0.0f, s1 = 0.0f;
    float x = src[(size_t)min(max(f - R, 0), na - 1) * stride];
#pragma unroll(RT ? 2 * RT + 1 : 4)
    for (int j = 0; j <= 2 * R; ++j) {
      const float y = src[(size_t)min(max(f - R + 1 + j, 0), na - 1) * stride];
      s0 += w[j] * x;
      s1 += w[j] * y;
      x = y;
    }
    dst[0] = s0;
    dst[stride] = s1;
  }
}

// The blur along n0 or n1 of every entry, T consecutive outputs per thread: the
// T + 2R inputs of a run are loaded once into registers instead of 2R + 1
// times per output through the caches.  Consecutive threads take consecutive
// lines (x fastest), so every load is coalesced.
template <int R, int T>
__global__ void __launch_bounds__(256) k_blur_axis_run(const Images im, int n0, int n1, int n2, int axis,
                                                       const float* __restrict__ w) {
  const int n = axis == 0 ? n0 : n1;
  const int stride = axis == 0 ? n1 * n2 : n2;
  const int lines = axis == 0 ? n1 * n2 : n0 * n2;
  const int runs = (n + T - 1) / T;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= lines * runs) return;
  const float* __restrict__ in = im.in[blockIdx.y];
  float* __restrict__ out = im.out[blockIdx.y];
  const int l = t % lines, r = t / lines;
  const int base = axis == 0 ? l : (l / n2) * (n1 * n2) + l % n2;
  const int p0 = r * T;
  float wt[2 * R + 1];
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) wt[k] = w[k];
  float v[T + 2 * R];
#pragma unroll
  for (int j = 0; j < T + 2 * R; ++j) v[j] = in[base + min(max(p0 - R + j, 0), n - 1) * stride];
#pragma unroll
  for (int j = 0; j < T; ++j) {
    if (p0 + j < n) {
      float s = 0.0f;
#pragma unroll
      for (int k = 0; k <= 2 * R; ++k) s += wt[k] * v[j + k];
      out[base + (p0 + j) * stride] = s;
    }
  }
}

// The blur along n2 of the eight corners of each sample, and the sample, times
// rho[image].  im.in holds the images after the passes along n0 and n1,
// [p0][p1][n2] (p0 = 2 m0 where compact, else n0; p1 likewise).
// Bound by the addresses of its loads, 32 to 104 per sample with one per value:
// four neighbours to a load took the three levels of 512^3 from 958 to 475 us.
template <int RT, bool BLK>
__global__ void __launch_bounds__(256) k_level_sample(const Images im, unsigned count, int n0, int n1, int n2, int m0, int m1, int m2,
                                                      bool c0, bool c1, float rho0, float rho1, float rho2,
                                                      const float* __restrict__ w, int Rr) {
  const int R = RT ? RT : Rr;
  unsigned row, item;
  const unsigned per_image = (unsigned)m0 * m1;
  if (!row_item<BLK>(blockIdx.x, (unsigned)m2, per_image * count, row, item)) return;
  const unsigned img = row / per_image, r = row - img * per_image;
  const int k1 = (int)(r % m1), k0 = (int)(r / m1), k2 = (int)item;
  Corners c = make_corners(n0, n1, n2, aligned_pos(k0, n0, m0), aligned_pos(k1, n1, m1), aligned_pos(k2, n2, m2));
  const int p1 = c1 ? 2 * m1 : n1;
  const float* rows[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int z = c0 ? 2 * k0 + (b >> 1) : min(max(c.i0 + (b >> 1), 0), n0 - 1);
    const int y = c1 ? 2 * k1 + (b & 1) : min(max(c.i1 + (b & 1), 0), n1 - 1);
    rows[b] = im.in[img] + ((size_t)z * p1 + y) * n2;
  }
  float v[8];
  auto corner = [&](int b, float s0, float s1) {
    const bool in0 = b >> 1 ? c.b0 : c.a0, in1 = b & 1 ? c.b1 : c.a1;
    v[2 * b] = in0 & in1 & c.a2 ? s0 : 0.0f;
    v[2 * b + 1] = in0 & in1 & c.b2 ? s1 : 0.0f;
  };
  if constexpr (RT > 0) {
    // a row's 2R + 2 neighbours, four to a load (any 4-byte alignment) but near the ends of a row
    typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int NV = 2 * RT + 2;
    float x[4][NV];
    if (c.i2 >= RT && c.i2 + RT + 1 < n2) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const float* p = rows[b] + (c.i2 - RT);
#pragma unroll
        for (int j = 0; j + 4 <= NV; j += 4) {
          const float4_any q = *reinterpret_cast<const float4_any*>(p + j);
          x[b][j] = q.x, x[b][j + 1] = q.y, x[b][j + 2] = q.z, x[b][j + 3] = q.w;
        }
#pragma unroll
        for (int j = NV / 4 * 4; j < NV; ++j) x[b][j] = p[j];
      }
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int j = 0; j < NV; ++j) x[b][j] = rows[b][min(max(c.i2 - RT + j, 0), n2 - 1)];
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
      for (int j = 0; j <= 2 * RT; ++j) {
        s0 += w[j] * x[b][j];
        s1 += w[j] * x[b][j + 1];
      }
      corner(b, s0, s1);
    }
  } else {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      float s0 = 0.0f, s1 = 0.0f;
      float x = rows[b][min(max(c.i2 - R, 0), n2 - 1)];
#pragma unroll 4
      for (int j = 0; j <= 2 * R; ++j) {
        const float t = rows[b][min(max(c.i2 - R + 1 + j, 0), n2 - 1)];
        s0 += w[j] * x;
        s1 += w[j] * t;
        x = t;
      }
      corner(b, s0, s1);
    }
  }
  const float rho = img == 0 ? rho0 : (img == 1 ? rho1 : rho2);
  im.out[img][(size_t)r * m2 + k2] = rho * tri(v, c);
}

// Trilinear samples at corner-aligned positions of up to three [3][N] fields
// (displacement and Adam moments at a level's end).  A thread takes one field's
// three components along a run of zc samples in n0: the sample in a plane
// (along n2, then n1) is the same for every sample between two planes, so it is
// formed once per input plane and a sample costs one more interpolation and its
// store.  Forming each sample by itself takes some 150 instructions a wavefront,
// 1.5 times what the stores cost.  (Three fields, 64^3 to 512^3 in three steps:
// 1.69 ms; a launch per field and a thread per sample 2.80.  Eight pairs,
// 48x56x52 to 96x112x104: 125 us against 307.)
struct Resample {
  const float* in[3];
  float* out[3];
  float rho[3];   // of the first field's components; the others' are 1
};

template <bool BLK>
__global__ void __launch_bounds__(256) k_resample(const Resample A, unsigned fields, int ni0, int ni1, int ni2,
                                                  int no0, int no1, int no2, int zc) {
  unsigned row, item;   // a row: one field, one run along n0, one y
  const unsigned runs = (unsigned)(no0 + zc - 1) / zc;
  if (!row_item<BLK>(xcd_tile(blockIdx.x, gridDim.x), (unsigned)no2, fields * runs * no1, row, item)) return;
  const unsigned f = row / (runs * no1), run = row / no1 % runs;
  const int y = (int)(row % no1), x = (int)item;
  int iy, ix;
  float ty, tx;
  bool a1, b1, a2, b2;
  cell(aligned_pos(y, ni1, no1), ni1, iy, ty, a1, b1);
  cell(aligned_pos(x, ni2, no2), ni2, ix, tx, a2, b2);
  const int ya = min(max(iy, 0), ni1 - 1) * ni2, yb = min(max(iy + 1, 0), ni1 - 1) * ni2;
  const int xa = min(max(ix, 0), ni2 - 1), xb = min(max(ix + 1, 0), ni2 - 1);
  const int off[4] = {ya + xa, ya + xb, yb + xa, yb + xb};
  const bool ok[4] = {a1 && a2, a1 && b2, b1 && a2, b1 && b2};
  const float* const in = f == 0 ? A.in[0] : (f == 1 ? A.in[1] : A.in[2]);
  float* const out = (f == 0 ? A.out[0] : (f == 1 ? A.out[1] : A.out[2])) + (size_t)y * no2 + x;
  const size_t Ni = (size_t)ni0 * ni1 * ni2, No = (size_t)no0 * no1 * no2;

  float lo[3], hi[3];   // the samples in planes at and at + 1
  auto plane = [&](int z, float p[3]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) p[q] = 0.0f;
    if (z < 0 || z >= ni0) return;
    const float* g = in + (size_t)z * ni1 * ni2;
    float v[3][4];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[q][k] = g[q * Ni + off[k]];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[q][k] = ok[k] ? v[q][k] : 0.0f;
      const float e0 = v[q][0] + tx * (v[q][1] - v[q][0]);
      const float e1 = v[q][2] + tx * (v[q][3] - v[q][2]);
      p[q] = e0 + ty * (e1 - e0);
    }
  };
  int at = -100;   // no plane yet
  const int z1 = min((int)(run + 1) * zc, no0);
  for (int z = (int)run * zc; z < z1; ++z) {
    int iz;
    float tz;
    bool a0, b0;
    cell(aligned_pos(z, ni0, no0), ni0, iz, tz, a0, b0);
    if (iz != at) {
      if (iz == at + 1)
#pragma unroll
        for (int q = 0; q < 3; ++q) lo[q] = hi[q];
      else
        plane(iz, lo);
      plane(iz + 1, hi);
      at = iz;
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const float s = lo[q] + tz * (hi[q] - lo[q]);
      // written once and far more than the L2 holds: past it (1.82 -> 1.69 ms)
      __builtin_nontemporal_store((f == 0 ? A.rho[q] : 1.0f) * s, &out[q * No + (size_t)z * no1 * no2]);
    }
  }
}

// J = I_m(x + d) and, with SLOPE, its position derivative ([3][N]): one
// trilinear sample per voxel, zero outside the grid.
template <bool SLOPE>
__device__ __forceinline__ void warp_voxel(const float* __restrict__ img, const float* __restrict__ d,
                                           float* __restrict__ out, float* __restrict__ slope, int n0, int n1, int n2,
                                           int z, int y, int x) {
  const int N = n0 * n1 * n2;
  const unsigned off = (unsigned)((z * n1 + y) * n2 + x) * 4u;
  const CellPairs c = pairs_at(n0, n1, n2, z, y, x, load_at(d, off), load_at(d + N, off), load_at(d + 2 * N, off));
  PairGather p;
  gather_issue(img, c, p);
  const Gather g = corners_of(p, c);
  if constexpr (SLOPE) {
    float g0, g1, g2;
    store_at(out, off, gather_value_grad(g, g0, g1, g2));
    store_at(slope, off, g0);
    store_at(slope + N, off, g1);
    store_at(slope + 2 * N, off, g2);
  } else {
    store_at(out, off, gather_value(g));
  }
}

template <bool SLOPE>
__global__ void __launch_bounds__(256) k_warp(const float* __restrict__ img, const float* __restrict__ d,
                                              float* __restrict__ out, float* __restrict__ slope, int n0, int n1,
                                              int n2, int bs) {
  int z, y, x;
  if (row_voxel(blockIdx.x, n0, n1, n2, bs, z, y, x))
    warp_voxel<SLOPE>(img, d, out, slope, n0, n1, n2, z, y, x);
}

// out = u + d(x + u): the displacement of phi o (id + u) for phi = id + d,
// with d sampled trilinearly per component (zero outside the grid).
__global__ void __launch_bounds__(256) k_compose_fields(const float* __restrict__ u, const float* __restrict__ d,
                                                        float* __restrict__ out, int n0, int n1, int n2, int bs) {
  const int N = n0 * n1 * n2;
  int z, y, x;
  if (!row_voxel(blockIdx.x, n0, n1, n2, bs, z, y, x)) return;
  const int i = (z * n1 + y) * n2 + x;
  const float u0 = u[i], u1 = u[N + i], u2 = u[2 * N + i];
  const CellPairs c = pairs_at(n0, n1, n2, z, y, x, u0, u1, u2);
  PairGather p0, p1, p2;
  gather_issue(d, c, p0);
  gather_issue(d + N, c, p1);
  gather_issue(d + 2 * N, c, p2);
  out[i] = u0 + gather_value(corners_of(p0, c));
  out[N + i] = u1 + gather_value(corners_of(p1, c));
  out[2 * N + i] = u2 + gather_value(corners_of(p2, c));
}

__global__ void k_soa_to_aos(const float* __restrict__ in, float* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  out[3 * i] = in[i];
  out[3 * i + 1] = in[n + i];
  out[3 * i + 2] = in[2 * n + i];
}

__device__ __forceinline__ void ctl_init(Ctl* ctl, float beta1, float beta2, int t_done, int iter) {
  const int t = t_done + 1;
  ctl->t = t;
  if (iter >= 0) ctl->iter = iter;
  ctl->beta1 = beta1;
  ctl->beta2 = beta2;
  ctl->bp1 = pow((double)beta1, (double)t);
  ctl->bp2 = pow((double)beta2, (double)t);
  ctl->bc1 = (float)(1.0 - ctl->bp1);
  ctl->bc2 = (float)(1.0 - ctl->bp2);
  for (int j = 0; j < kMSlots; ++j) ctl->mslot[j * kMStride] = 0u;
}

__global__ void k_ctl_init(Ctl* ctl, float beta1, float beta2, int t_done, int iter, unsigned* tickets) {
  if (threadIdx.x == 0 && blockIdx.x == 0) ctl_init(ctl, beta1, beta2, t_done, iter);
  if (tickets && threadIdx.x < kTicketCount) tickets[threadIdx.x * kTicketStride] = 0u;
}

// The start of a schedule in one launch: four arrays of n floats cleared (y
// picks one, four values per thread), the control block and the means' tickets.
struct Clear4 {
  float* p[4];
};
__global__ void __launch_bounds__(256) k_start(const Clear4 A, int64_t n, Ctl* ctl, float beta1, float beta2,
                                               unsigned* tickets) {
  const unsigned a = blockIdx.y;
  float* p = a == 0 ? A.p[0] : (a == 1 ? A.p[1] : (a == 2 ? A.p[2] : A.p[3]));
  const int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  if (i + 4 <= n) {
    *reinterpret_cast<float4*>(p + i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  } else {
    for (int64_t j = i; j < n; ++j) p[j] = 0.0f;
  }
  if (a == 0 && blockIdx.x == 0) {
    if (threadIdx.x == 255) ctl_init(ctl, beta1, beta2, 0, 0);
    if (tickets && threadIdx.x < kTicketCount) tickets[threadIdx.x * kTicketStride] = 0u;
  }
}

// The means of two images in one launch: the sums of each image's workgroups go
// to memory, and the last workgroup to finish adds them up, in the order of the
// workgroups.  Bound by launches at the usual sizes: an LNCC loss
// and gradient takes 97 us at 24^3 and at 128^3 with k_means_warp, 122 and 119
// with a sum and a division per image and the warp in launches of their own.
__device__ __forceinline__ void mean_block(const Means& A, int img, int blk, int np) {
  __shared__ double red[4];
  __shared__ int last;
  const float* __restrict__ x = img ? A.x[1] : A.x[0];
  double* part = A.part + (size_t)img * kMeanBlocks;
  double s = 0.0;
  for (int64_t i = (int64_t)blk * 256 + threadIdx.x; i < A.n; i += (int64_t)kMeanBlocks * 256) s += (double)x[i];
  s = block_sum<256>(s, red);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&part[blk], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the sum has to have reached memory before this workgroup counts
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    last = last_workgroup(A.tickets + (size_t)img * (kTicketSlots + 1) * kTicketStride, blk, np);
  }
  __syncthreads();
  if (!last) return;
  asm volatile("" ::: "memory");
  double t = 0.0;
  for (int i = threadIdx.x; i < np; i += 256)
    t += __hip_atomic_load(&part[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  t = block_sum<256>(t, red);
  if (threadIdx.x == 0) *(img ? A.dst[1] : A.dst[0]) = (float)(t / (double)A.n);
}

// Workgroups with values, of kMeanBlocks (the sums of the others would be zero).
__host__ __device__ inline int mean_blocks(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return b < kMeanBlocks ? (int)b : kMeanBlocks;
}

__global__ void __launch_bounds__(256) k_means(const Means A, int np) {
  mean_block(A, blockIdx.x >= (unsigned)np, blockIdx.x % np, np);
}

// The same together with J (and its slope), which needs neither, in the
// workgroups after the means'.
template <bool SLOPE>
__global__ void __launch_bounds__(256) k_means_warp(const Means A, int np, const float* __restrict__ img,
                                                    const float* __restrict__ d, float* __restrict__ out,
                                                    float* __restrict__ slope, int n0, int n1, int n2, int bs) {
  if (blockIdx.x < 2u * np) {
    mean_block(A, blockIdx.x >= (unsigned)np, blockIdx.x % np, np);
    return;
  }
  int z, y, x;
  if (row_voxel(blockIdx.x - 2 * np, n0, n1, n2, bs, z, y, x))
    warp_voxel<SLOPE>(img, d, out, slope, n0, n1, n2, z, y, x);
}

__global__ void k_mean_final(const double* __restrict__ part, int np, double n, float* __restrict__ dst) {
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < np; i += blockDim.x) s += part[i];
  s = block_sum<256>(s, red);
  if (threadIdx.x == 0) *dst = (float)(s / n);
}

__global__ void k_sum_final(const double* __restrict__ part, int np, double* __restrict__ dst) {
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < np; i += blockDim.x) s += part[i];
  s = block_sum<256>(s, red);
  if (threadIdx.x == 0) *dst = s;
}

// ---------------------------------------------------------------------------
// Dispatch tables
// ---------------------------------------------------------------------------
template <int R, int TY, int TX>
constexpr size_t gauss_lds(bool staged_d) {
  return sizeof(float) * (3 * (TY + 2 * R) * (TX + 2 * R) + 3 * (TY + 2 * R) * TX +
                          (staged_d ? 9 * (((TY + 2) * (TX + 2) + 31) / 32 * 32) : 0));
}

template <int W, int TY, int TX, int MODE>
hipError_t grad_launch_m(const GradArgs& a, const Tiling& t, hipStream_t s) {
  constexpr size_t sh = GradShape<W, TY, TX, MODE>::lds_bytes;
  static_assert(sh <= 65536, "gradient kernel LDS exceeds 64 KiB");
  k_grad<W, TY, TX, MODE><<<dim3(t.blocks()), dim3(GradLaunch<W, TY, TX, MODE>::NT), sh, s>>>(a);
  return hipGetLastError();
}

template <int W, int TY, int TX>
hipError_t grad_launch_t(const GradArgs& a, const Tiling& t, hipStream_t s) {
  switch (a.mode) {
    case 0: return grad_launch_m<W, TY, TX, 0>(a, t, s);
    case 1: return grad_launch_m<W, TY, TX, 1>(a, t, s);
    default: return grad_launch_m<W, TY, TX, 2>(a, t, s);
  }
}

template <int TY, int TX>
hipError_t grad_launch_tile(const GradArgs& a, int window, const Tiling& t, hipStream_t s) {
  switch (window) {
    case 1: return grad_launch_t<1, TY, TX>(a, t, s);
    case 3: return grad_launch_t<3, TY, TX>(a, t, s);
    case 5: return grad_launch_t<5, TY, TX>(a, t, s);
    case 7: return grad_launch_t<7, TY, TX>(a, t, s);
    case 9: return grad_launch_t<9, TY, TX>(a, t, s);
    default: return hipErrorInvalidValue;
  }
}

template <int R, int TY, int TX>
hipError_t gauss_launch_r(const GaussArgs& a, int epi, const Tiling& t, hipStream_t s) {
  const dim3 g(t.blocks()), blk(TY * TX);
  const size_t sh = gauss_lds<R, TY, TX>(epi == EPI_COMPOSE_LDS);
  switch (epi) {
    case EPI_STORE: k_gauss<R, TY, TX, EPI_STORE><<<g, blk, sh, s>>>(a); break;
    case EPI_STORE_WARP: k_gauss<R, TY, TX, EPI_STORE_WARP><<<g, blk, sh, s>>>(a); break;
    case EPI_SMOOTH_MAX: k_gauss<R, TY, TX, EPI_SMOOTH_MAX><<<g, blk, sh, s>>>(a); break;
    case EPI_COMPOSE:
    case EPI_COMPOSE_LDS:
      // the composition runs with the single tap (radius 0) only
      if constexpr (R == 0) {
        if (epi == EPI_COMPOSE_LDS) k_gauss<0, TY, TX, EPI_COMPOSE_LDS><<<g, blk, sh, s>>>(a);
        else k_gauss<0, TY, TX, EPI_COMPOSE><<<g, blk, sh, s>>>(a);
        break;
      } else {
        return hipErrorInvalidValue;
      }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int TY, int TX>
hipError_t gauss_launch_tile(const GaussArgs& a, int radius, int epi, const Tiling& t, hipStream_t s) {
  switch (radius) {
    case 0: return gauss_launch_r<0, TY, TX>(a, epi, t, s);
    case 1: return gauss_launch_r<1, TY, TX>(a, epi, t, s);
    case 2: return gauss_launch_r<2, TY, TX>(a, epi, t, s);
    case 3: return gauss_launch_r<3, TY, TX>(a, epi, t, s);
    case 4: return gauss_launch_r<4, TY, TX>(a, epi, t, s);
    case 5: return gauss_launch_r<5, TY, TX>(a, epi, t, s);
    case 6: return gauss_launch_r<6, TY, TX>(a, epi, t, s);
    default: return hipErrorInvalidValue;
  }
}

template <int R>
hipError_t gauss_cube_r(const GaussArgs& a, int epi, const Tiling& t, hipStream_t s) {
  constexpr int TZ = kCubeZ, TY = kCubeY, TX = kCubeX;
  constexpr size_t sh = sizeof(float) * 3 *
                        ((TZ + 2 * R) * (TY + 2 * R) * (TX + 2 * R) + (TZ + 2 * R) * (TY + 2 * R) * TX);
  static_assert(sh <= 65536, "brick smoothing LDS exceeds 64 KiB");
  const dim3 g(t.blocks()), one(kCubeThreads<TZ, TY, TX, EPI_STORE>), two(kCubeThreads<TZ, TY, TX, EPI_SMOOTH_MAX>);
  switch (epi) {
    case EPI_SMOOTH_MAX: k_gauss_cube<R, TZ, TY, TX, EPI_SMOOTH_MAX><<<g, two, sh, s>>>(a); break;
    case EPI_STORE: k_gauss_cube<R, TZ, TY, TX, EPI_STORE><<<g, one, sh, s>>>(a); break;
    case EPI_STORE_WARP: k_gauss_cube<R, TZ, TY, TX, EPI_STORE_WARP><<<g, one, sh, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t gauss_launch_cube(const GaussArgs& a, int radius, int epi, const Tiling& t, hipStream_t s) {
  if (epi == EPI_COMPOSE_LDS) {
    if (radius != 0) return hipErrorInvalidValue;
    constexpr int TZ = kCubeZ, TY = kCubeY, TX = kCubeX;
    constexpr size_t sh = sizeof(float) * 3 * (TZ + 2) * (TY + 2) * (TX + 2);
    k_compose_cube<TZ, TY, TX><<<dim3(t.blocks()), dim3(TZ * TY * TX), sh, s>>>(a);
    return hipGetLastError();
  }
  switch (radius) {
    case 0: return gauss_cube_r<0>(a, epi, t, s);
    case 1: return gauss_cube_r<1>(a, epi, t, s);
    case 2: return gauss_cube_r<2>(a, epi, t, s);
    case 3: return gauss_cube_r<3>(a, epi, t, s);
    default: return hipErrorInvalidValue;
  }
}

template <int W, int MODE>
hipError_t grad_cube_m(const GradArgs& a, const Tiling& t, hipStream_t s) {
  constexpr int TZ = kCubeZ, TY = kCubeY, TX = kCubeX;
  constexpr size_t sh = GradCubeShape<W, TZ, TY, TX>::lds_bytes;
  static_assert(sh <= 160 * 1024 - 1024, "brick gradient LDS exceeds the 160 KiB of a CU");
  static bool attr_set = false;   // raise the dynamic LDS limit once per process
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_grad_cube<W, TZ, TY, TX, MODE>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  k_grad_cube<W, TZ, TY, TX, MODE><<<dim3(t.blocks()), dim3(GradCubeShape<W, TZ, TY, TX>::NT), sh, s>>>(a);
  return hipGetLastError();
}

template <int W>
hipError_t grad_cube_w(const GradArgs& a, const Tiling& t, hipStream_t s) {
  switch (a.mode) {
    case 0: return grad_cube_m<W, 0>(a, t, s);
    case 1: return grad_cube_m<W, 1>(a, t, s);
    default: return grad_cube_m<W, 2>(a, t, s);
  }
}

hipError_t grad_launch_cube(const GradArgs& a, int window, const Tiling& t, hipStream_t s) {
  switch (window) {
    case 1: return grad_cube_w<1>(a, t, s);
    case 3: return grad_cube_w<3>(a, t, s);
    case 5: return grad_cube_w<5>(a, t, s);
    default: return hipErrorInvalidValue;
  }
}

// ---- batched launches ------------------------------------------------------
template <int W, int TY, int TX>
hipError_t grad_batch_t(const BatchEntry<GradArgs>* E, const int* owner, int total, bool adam, hipStream_t s) {
  constexpr size_t sh = GradShape<W, TY, TX, 0>::lds_bytes;
  const dim3 g(total);
  if (adam) k_grad_batch<W, TY, TX, 0><<<g, dim3(GradLaunch<W, TY, TX, 0>::NT), sh, s>>>(E, owner);
  else k_grad_batch<W, TY, TX, 1><<<g, dim3(GradLaunch<W, TY, TX, 1>::NT), sh, s>>>(E, owner);
  return hipGetLastError();
}

template <int TY, int TX>
hipError_t grad_batch_tile(const BatchEntry<GradArgs>* E, const int* owner, int total, int window, bool adam,
                           hipStream_t s) {
  switch (window) {
    case 1: return grad_batch_t<1, TY, TX>(E, owner, total, adam, s);
    case 3: return grad_batch_t<3, TY, TX>(E, owner, total, adam, s);
    case 5: return grad_batch_t<5, TY, TX>(E, owner, total, adam, s);
    case 7: return grad_batch_t<7, TY, TX>(E, owner, total, adam, s);
    case 9: return grad_batch_t<9, TY, TX>(E, owner, total, adam, s);
    default: return hipErrorInvalidValue;
  }
}

template <int W, int MODE>
hipError_t grad_cube_batch_m(const BatchEntry<GradArgs>* E, const int* owner, int total, hipStream_t s) {
  constexpr int TZ = kCubeZ, TY = kCubeY, TX = kCubeX;
  constexpr size_t sh = GradCubeShape<W, TZ, TY, TX>::lds_bytes;
  static bool attr_set = false;   // raise the dynamic LDS limit once per process
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_grad_cube_batch<W, TZ, TY, TX, MODE>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  k_grad_cube_batch<W, TZ, TY, TX, MODE><<<dim3(total), dim3(GradCubeShape<W, TZ, TY, TX>::NT), sh, s>>>(E, owner);
  return hipGetLastError();
}

template <int W>
hipError_t grad_cube_batch_w(const BatchEntry<GradArgs>* E, const int* owner, int total, bool adam, hipStream_t s) {
  return adam ? grad_cube_batch_m<W, 0>(E, owner, total, s) : grad_cube_batch_m<W, 1>(E, owner, total, s);
}

template <int R, int TY, int TX>
hipError_t gauss_batch_r(const BatchEntry<GaussArgs>* E, const int* owner, int total, int epi, hipStream_t s) {
  const dim3 g(total), blk(TY * TX);
  const size_t sh = gauss_lds<R, TY, TX>(epi == EPI_COMPOSE_LDS);
  switch (epi) {
    case EPI_SMOOTH_MAX: k_gauss_batch<R, TY, TX, EPI_SMOOTH_MAX><<<g, blk, sh, s>>>(E, owner); break;
    case EPI_STORE_WARP: k_gauss_batch<R, TY, TX, EPI_STORE_WARP><<<g, blk, sh, s>>>(E, owner); break;
    case EPI_COMPOSE_LDS:
    case EPI_COMPOSE:
      // the composition runs with the single tap (radius 0) only
      if constexpr (R == 0) {
        if (epi == EPI_COMPOSE_LDS) k_gauss_batch<0, TY, TX, EPI_COMPOSE_LDS><<<g, blk, sh, s>>>(E, owner);
        else k_gauss_batch<0, TY, TX, EPI_COMPOSE><<<g, blk, sh, s>>>(E, owner);
        break;
      } else {
        return hipErrorInvalidValue;
      }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int TY, int TX>
hipError_t gauss_batch_tile(const BatchEntry<GaussArgs>* E, const int* owner, int total, int radius, int epi,
                            hipStream_t s) {
  switch (radius) {
    case 0: return gauss_batch_r<0, TY, TX>(E, owner, total, epi, s);
    case 1: return gauss_batch_r<1, TY, TX>(E, owner, total, epi, s);
    case 2: return gauss_batch_r<2, TY, TX>(E, owner, total, epi, s);
    case 3: return gauss_batch_r<3, TY, TX>(E, owner, total, epi, s);
    case 4: return gauss_batch_r<4, TY, TX>(E, owner, total, epi, s);
    case 5: return gauss_batch_r<5, TY, TX>(E, owner, total, epi, s);
    case 6: return gauss_batch_r<6, TY, TX>(E, owner, total, epi, s);
    default: return hipErrorInvalidValue;
  }
}

template <int R>
hipError_t gauss_cube_batch_r(const BatchEntry<GaussArgs>* E, const int* owner, int total, int epi,
                              hipStream_t s) {
  constexpr int TZ = kCubeZ, TY = kCubeY, TX = kCubeX;
  constexpr size_t sh = sizeof(float) * 3 *
                        ((TZ + 2 * R) * (TY + 2 * R) * (TX + 2 * R) + (TZ + 2 * R) * (TY + 2 * R) * TX);
  const dim3 g(total), one(kCubeThreads<TZ, TY, TX, EPI_STORE>), two(kCubeThreads<TZ, TY, TX, EPI_SMOOTH_MAX>);
  switch (epi) {
    case EPI_SMOOTH_MAX: k_gauss_cube_batch<R, TZ, TY, TX, EPI_SMOOTH_MAX><<<g, two, sh, s>>>(E, owner); break;
    case EPI_STORE_WARP: k_gauss_cube_batch<R, TZ, TY, TX, EPI_STORE_WARP><<<g, one, sh, s>>>(E, owner); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t gauss_cube_batch(const BatchEntry<GaussArgs>* E, const int* owner, int total, int radius, int epi,
                            hipStream_t s) {
  if (epi == EPI_COMPOSE_LDS) {
    if (radius != 0) return hipErrorInvalidValue;
    constexpr int TZ = kCubeZ, TY = kCubeY, TX = kCubeX;
    constexpr size_t sh = sizeof(float) * 3 * (TZ + 2) * (TY + 2) * (TX + 2);
    k_compose_cube_batch<TZ, TY, TX><<<dim3(total), dim3(TZ * TY * TX), sh, s>>>(E, owner);
    return hipGetLastError();
  }
  switch (radius) {
    case 0: return gauss_cube_batch_r<0>(E, owner, total, epi, s);
    case 1: return gauss_cube_batch_r<1>(E, owner, total, epi, s);
    case 2: return gauss_cube_batch_r<2>(E, owner, total, epi, s);
    case 3: return gauss_cube_batch_r<3>(E, owner, total, epi, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool grad_tile_supported(int ty, int tx) { return (ty == 16 && tx == 32) || (ty == 8 && tx == 32); }
bool grad_cube_supported(int window) { return window == 1 || window == 3 || window == 5; }

bool gauss_cube_supported(int radius, int epilogue) {
  if (epilogue == EPI_COMPOSE_LDS) return radius == 0;
  return (epilogue == EPI_SMOOTH_MAX || epilogue == EPI_STORE || epilogue == EPI_STORE_WARP) && radius >= 0 &&
         radius <= 3;
}

bool gauss_tile_supported(int ty, int tx) {
  return (ty == 16 && tx == 32) || (ty == 8 && tx == 32) || (ty == 8 && tx == 64);
}

size_t gauss_lds_bytes(int radius, int ty, int tx) {
  return sizeof(float) * (size_t)(3 * (ty + 2 * radius) * (tx + 2 * radius) + 3 * (ty + 2 * radius) * tx +
                                  9 * (((ty + 2) * (tx + 2) + 31) / 32 * 32));
}

hipError_t launch_grad(const GradArgs& a, int window, const Tiling& t, hipStream_t s) {
  if (t.cube) return grad_launch_cube(a, window, t, s);
  if (t.ty == 16 && t.tx == 32) return grad_launch_tile<16, 32>(a, window, t, s);
  if (t.ty == 8 && t.tx == 32) return grad_launch_tile<8, 32>(a, window, t, s);
  return hipErrorInvalidValue;
}

bool grad_batch_supported(int window, const Tiling& t) {
  if (t.cube) return grad_cube_supported(window);
  return grad_tile_supported(t.ty, t.tx) && window >= 1 && window <= kMaxWindow && window % 2 == 1;
}

bool gauss_batch_supported(int radius, int epilogue, const Tiling& t) {
  if (t.cube) return epilogue != EPI_STORE && gauss_cube_supported(radius, epilogue);
  if (!gauss_tile_supported(t.ty, t.tx) || radius < 0 || radius > kMaxRadius) return false;
  if (epilogue == EPI_SMOOTH_MAX || epilogue == EPI_STORE_WARP) return true;
  return (epilogue == EPI_COMPOSE_LDS || epilogue == EPI_COMPOSE) && radius == 0;
}

hipError_t launch_grad_batch(const BatchEntry<GradArgs>* E, const int* owner, int total, int window,
                             const Tiling& t, bool adam, hipStream_t s) {
  if (total <= 0) return hipSuccess;
  if (t.cube) {
    switch (window) {
      case 1: return grad_cube_batch_w<1>(E, owner, total, adam, s);
      case 3: return grad_cube_batch_w<3>(E, owner, total, adam, s);
      case 5: return grad_cube_batch_w<5>(E, owner, total, adam, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (t.ty == 16 && t.tx == 32) return grad_batch_tile<16, 32>(E, owner, total, window, adam, s);
  if (t.ty == 8 && t.tx == 32) return grad_batch_tile<8, 32>(E, owner, total, window, adam, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gauss_batch(const BatchEntry<GaussArgs>* E, const int* owner, int total, int radius,
                              int epilogue, const Tiling& t, hipStream_t s) {
  if (total <= 0) return hipSuccess;
  if (t.cube) return gauss_cube_batch(E, owner, total, radius, epilogue, s);
  if (t.ty == 16 && t.tx == 32) return gauss_batch_tile<16, 32>(E, owner, total, radius, epilogue, s);
  if (t.ty == 8 && t.tx == 32) return gauss_batch_tile<8, 32>(E, owner, total, radius, epilogue, s);
  if (t.ty == 8 && t.tx == 64) return gauss_batch_tile<8, 64>(E, owner, total, radius, epilogue, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gauss_narrow(const GaussArgs& a, int radius, int epilogue, const Tiling& t, hipStream_t s) {
  if (t.cube) return gauss_launch_cube(a, radius, epilogue, t, s);
  if (t.ty == 16 && t.tx == 32) return gauss_launch_tile<16, 32>(a, radius, epilogue, t, s);
  if (t.ty == 8 && t.tx == 32) return gauss_launch_tile<8, 32>(a, radius, epilogue, t, s);
  if (t.ty == 8 && t.tx == 64) return gauss_launch_tile<8, 64>(a, radius, epilogue, t, s);
  return hipErrorInvalidValue;
}

// Radius above kMaxRadius (sigma_grad or sigma_warp or the inverse's widths
// above 2 voxels): three separable passes, the last with the epilogue (max
// norm, or a plain store):
//   in -> out (n2), out -> wide_tmp (n1), wide_tmp -> out (n0).
// Needs a.wide_tmp distinct from a.in and a.out, a.in != a.out, and a tap
// table a.wts of 2R + 1 taps followed by zeros up to a multiple of 16 (the
// runtime's tables are laid out so).
hipError_t launch_gauss_wide(const GaussArgs& a, int radius, int epilogue, const Tiling& t, hipStream_t s) {
  (void)t;
  if (radius > kMaxWideRadius || !a.wide_tmp || a.wide_tmp == a.in || a.wide_tmp == a.out || a.in == a.out ||
      (epilogue != EPI_SMOOTH_MAX && epilogue != EPI_STORE))
    return hipErrorInvalidValue;
  const int n0 = a.n0, n1 = a.n1, n2 = a.n2;
  if (n0 > 65535 || n1 > 65535) return hipErrorInvalidValue;
  const int l8 = (2 * radius + 1 + 7) / 8 * 8;
  const size_t shx = sizeof(float) * 3 * (256 + 2 * radius);
  // one component staged at a time: the run plus the taps rounded up to 8
  const size_t shyz = sizeof(float) * (kWideRun + l8) * 64;
  k_field_wide_x<<<dim3((n2 + 255) / 256, n1, n0), dim3(256), shx, s>>>(a.in, a.out, n0, n1, n2, a.wts, radius);
  k_field_wide_yz<1, EPI_STORE><<<dim3((n2 + 63) / 64, (n1 + kWideRun - 1) / kWideRun, n0), dim3(kWideThreads), shyz, s>>>(
      a.out, a.wide_tmp, n0, n1, n2, a.wts, radius, a);
  const dim3 g0((n2 + 63) / 64, (n0 + kWideRun - 1) / kWideRun, n1);
  switch (epilogue) {
    case EPI_SMOOTH_MAX:
      k_field_wide_yz<0, EPI_SMOOTH_MAX><<<g0, dim3(kWideThreads), shyz, s>>>(a.wide_tmp, a.out, n0, n1, n2, a.wts,
                                                                           radius, a);
      break;
    default:
      k_field_wide_yz<0, EPI_STORE><<<g0, dim3(kWideThreads), shyz, s>>>(a.wide_tmp, a.out, n0, n1, n2, a.wts, radius,
                                                                      a);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_gauss(const GaussArgs& a, int radius, int epilogue, const Tiling& t, hipStream_t s) {
  if (epilogue == EPI_STORE_WARP && !a.moving_pairs) {
    // a volume whose row pairs 32-bit offsets do not reach: sampled by a launch of its own
    const hipError_t e = launch_gauss(a, radius, EPI_STORE, t, s);
    return e != hipSuccess ? e : launch_warp_slope(a.moving, a.out, a.warped, a.slope, a.n0, a.n1, a.n2, s);
  }
  if (radius > kMaxRadius) {
    if (epilogue != EPI_STORE_WARP) return launch_gauss_wide(a, radius, epilogue, t, s);
    const hipError_t e = launch_gauss_wide(a, radius, EPI_STORE, t, s);
    return e != hipSuccess ? e : launch_warp_slope(a.moving, a.out, a.warped, a.slope, a.n0, a.n1, a.n2, s);
  }
  return launch_gauss_narrow(a, radius, epilogue, t, s);
}


static inline unsigned grid1(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

hipError_t launch_eulerian_adam(float* ga, const float* d, float* m, float* v, Ctl* ctl, int n0, int n1,
                                int n2, float beta1, float beta2, float adam_eps, hipStream_t s) {
  const int64_t n = (int64_t)n0 * n1 * n2;
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(k_eulerian_adam, dim3(blocks), dim3(256), 0, s, ga, d, m, v, ctl, n0, n1, n2, beta1, beta2,
                     adam_eps);
  return hipGetLastError();
}

hipError_t launch_row_pairs(const float* in, float* out, int n0, int n1, int n2, hipStream_t s) {
  const int p0 = n0 + 2 * kPad, p1 = n1 + 2 * kPad, p2 = n2 + 2 * kPad;
  float2* o = reinterpret_cast<float2*>(out);
  if (p0 <= 65535 && p1 <= 65535)
    hipLaunchKernelGGL(k_row_pairs<true>, dim3(grid1(p2, 128), p1, p0), dim3(128), 0, s, in, o, n0, n1, n2);
  else
    hipLaunchKernelGGL(k_row_pairs<false>, dim3(grid1((int64_t)p0 * p1 * p2, 256)), dim3(256), 0, s, in, o, n0, n1, n2);
  return hipGetLastError();
}

hipError_t launch_fill(float* p, float value, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill, dim3(grid1(n, 256)), dim3(256), 0, s, p, value, n);
  return hipGetLastError();
}

template <int R>
hipError_t blur_axis_run(const Images& im, int count, int n0, int n1, int n2, int axis, const float* wts,
                         hipStream_t s) {
  constexpr int T = 8;
  const int n = axis == 0 ? n0 : n1;
  const int64_t threads = (int64_t)n0 * n1 * n2 / n * ((n + T - 1) / T);
  hipLaunchKernelGGL((k_blur_axis_run<R, T>), dim3(grid1(threads, 256), count), dim3(256), 0, s, im, n0, n1, n2, axis,
                     wts);
  return hipGetLastError();
}

template <int AX, int RT>
hipError_t blur_pairs(const Images& im, int count, int na, int nm, int n_other, int n2, const float* wts, int R,
                      hipStream_t s) {
  const int64_t inner = AX == 0 ? (int64_t)n_other * n2 : n2;
  const int64_t rows = (int64_t)count * (AX == 0 ? 1 : n_other);   // times the groups of k
  // a thread takes up to eight k while that leaves every CU its 2048 threads
  const int kg = (int)std::min<int64_t>(8, std::max<int64_t>(1, rows * inner * nm / (256 * 2048)));
  const int64_t all = rows * ((nm + kg - 1) / kg);
  if (const int bs = row_span((int)std::min<int64_t>(inner, 256)))
    hipLaunchKernelGGL((k_blur_pairs<AX, RT, true>), dim3((unsigned)(all * ((inner + bs - 1) / bs))), dim3(bs), 0, s,
                       im, count, na, nm, n_other, n2, wts, R, kg);
  else
    hipLaunchKernelGGL((k_blur_pairs<AX, RT, false>), dim3(grid1(all * inner, 256)), dim3(256), 0, s, im, count, na,
                       nm, n_other, n2, wts, R, kg);
  return hipGetLastError();
}

// One pass of the blur along n0 or n1: the entries that are sampled (compact) or all.
template <int AX>
hipError_t blur_pass(const Images& im, int count, int n0, int n1, int n2, int nm, bool compact, const float* wts, int R,
                     hipStream_t s) {
  const int na = AX == 0 ? n0 : n1, other = AX == 0 ? n1 : n0;
  if (compact) {
    switch (R) {   // radii of the usual scales (4 and 8) unrolled
      case 6: return blur_pairs<AX, 6>(im, count, na, nm, other, n2, wts, R, s);
      case 12: return blur_pairs<AX, 12>(im, count, na, nm, other, n2, wts, R, s);
      default: return blur_pairs<AX, 0>(im, count, na, nm, other, n2, wts, R, s);
    }
  }
  switch (R) {   // compact where R > 3
    case 1: return blur_axis_run<1>(im, count, n0, n1, n2, AX, wts, s);
    case 2: return blur_axis_run<2>(im, count, n0, n1, n2, AX, wts, s);
    case 3: return blur_axis_run<3>(im, count, n0, n1, n2, AX, wts, s);
    default: return hipErrorInvalidValue;
  }
}

template <int RT>
hipError_t level_sample(const Images& im, int count, int n0, int n1, int n2, int m0, int m1, int m2, bool c0, bool c1,
                        const float* rho, const float* wts, int R, hipStream_t s) {
  const int64_t rows = (int64_t)count * m0 * m1;
  if (const int bs = row_span(m2))
    hipLaunchKernelGGL((k_level_sample<RT, true>), dim3((unsigned)(rows * ((m2 + bs - 1) / bs))), dim3(bs), 0, s, im,
                       count, n0, n1, n2, m0, m1, m2, c0, c1, rho[0], rho[1], rho[2], wts, R);
  else
    hipLaunchKernelGGL((k_level_sample<RT, false>), dim3(grid1(rows * m2, 256)), dim3(256), 0, s, im, count, n0, n1,
                       n2, m0, m1, m2, c0, c1, rho[0], rho[1], rho[2], wts, R);
  return hipGetLastError();
}

hipError_t launch_level_images(const float* const* src, float* const* dst, const float* rho, int count, float* tmp0,
                               float* tmp1, int n0, int n1, int n2, int m0, int m1, int m2, const float* wts, int R,
                               hipStream_t s) {
  if (count < 1 || count > 3 || R < 1) return hipErrorInvalidValue;
  // Scale 2 and below (2m >= n, radius at most 3) leave out so little that the
  // run form's shared loads win; a larger radius always has 2m <= n.
  const bool c0 = 2 * m0 < n0 || R > 3, c1 = 2 * m1 < n1 || R > 3;
  const int p0 = c0 ? 2 * m0 : n0, p1 = c1 ? 2 * m1 : n1;
  Images a{}, b{}, c{};
  for (int i = 0; i < count; ++i) {
    a.in[i] = src[i];
    a.out[i] = tmp0 + (size_t)i * p0 * n1 * n2;
    b.in[i] = a.out[i];
    b.out[i] = tmp1 + (size_t)i * p0 * p1 * n2;
    c.in[i] = b.out[i];
    c.out[i] = dst[i];
  }
  hipError_t e = blur_pass<0>(a, count, n0, n1, n2, m0, c0, wts, R, s);
  if (e == hipSuccess) e = blur_pass<1>(b, count, p0, n1, n2, m1, c1, wts, R, s);
  if (e != hipSuccess) return e;
  switch (R) {   // scales 2, 4 and 8 unrolled
    case 3: return level_sample<3>(c, count, n0, n1, n2, m0, m1, m2, c0, c1, rho, wts, R, s);
    case 6: return level_sample<6>(c, count, n0, n1, n2, m0, m1, m2, c0, c1, rho, wts, R, s);
    case 12: return level_sample<12>(c, count, n0, n1, n2, m0, m1, m2, c0, c1, rho, wts, R, s);
    default: return level_sample<0>(c, count, n0, n1, n2, m0, m1, m2, c0, c1, rho, wts, R, s);
  }
}

hipError_t launch_resample(const float* const* in, float* const* out, int fields, const int ni[3], const int no[3],
                           const float rho[3], hipStream_t s) {
  if (fields < 1 || fields > 3) return hipErrorInvalidValue;
  Resample A{};
  for (int f = 0; f < fields; ++f) {
    A.in[f] = in[f];
    A.out[f] = out[f];
  }
  for (int q = 0; q < 3; ++q) A.rho[q] = rho[q];
  // runs of 4 to 16 samples: as long as every CU keeps its 2048 threads
  const int64_t threads = (int64_t)fields * no[0] * no[1] * no[2];
  const int zc = (int)std::min<int64_t>(16, std::max<int64_t>(4, threads / (256 * 2048)));
  const int64_t rows = (int64_t)fields * no[1] * ((no[0] + zc - 1) / zc);
  if (const int bs = row_span(no[2]))
    hipLaunchKernelGGL(k_resample<true>, dim3((unsigned)(rows * ((no[2] + bs - 1) / bs))), dim3(bs), 0, s, A, fields,
                       ni[0], ni[1], ni[2], no[0], no[1], no[2], zc);
  else
    hipLaunchKernelGGL(k_resample<false>, dim3(grid1(rows * no[2], 256)), dim3(256), 0, s, A, fields, ni[0], ni[1],
                       ni[2], no[0], no[1], no[2], zc);
  return hipGetLastError();
}

template <bool SLOPE>
hipError_t warp_launch(const float* img, const float* d, float* out, float* slope, int n0, int n1, int n2,
                       hipStream_t s) {
  const int bs = row_span(n2);
  hipLaunchKernelGGL((k_warp<SLOPE>), dim3(row_blocks((int64_t)n0 * n1, n2, bs)), dim3(256), 0, s, img, d, out, slope, n0,
                     n1, n2, bs);
  return hipGetLastError();
}

hipError_t launch_warp(const float* img, const float* d, float* out, int n0, int n1, int n2, hipStream_t s) {
  return warp_launch<false>(img, d, out, nullptr, n0, n1, n2, s);
}

hipError_t launch_warp_slope(const float* img, const float* d, float* out, float* slope, int n0, int n1, int n2,
                             hipStream_t s) {
  return warp_launch<true>(img, d, out, slope, n0, n1, n2, s);
}

hipError_t launch_compose_fields(const float* u, const float* d, float* out, int n0, int n1, int n2,
                                hipStream_t s) {
  const int bs = row_span(n2);
  hipLaunchKernelGGL(k_compose_fields, dim3(row_blocks((int64_t)n0 * n1, n2, bs)), dim3(256), 0, s, u, d, out, n0, n1, n2,
                     bs);
  return hipGetLastError();
}

hipError_t launch_soa_to_aos(const float* in, float* out, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_soa_to_aos, dim3(grid1(n, 256)), dim3(256), 0, s, in, out, n);
  return hipGetLastError();
}

hipError_t launch_ctl_init(Ctl* ctl, float beta1, float beta2, int t_done, int iter, unsigned* tickets,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_ctl_init, dim3(1), dim3(128), 0, s, ctl, beta1, beta2, t_done, iter, tickets);
  return hipGetLastError();
}

hipError_t launch_start(float* const p[4], int64_t n, Ctl* ctl, float beta1, float beta2, unsigned* tickets,
                        hipStream_t s) {
  Clear4 A{{p[0], p[1], p[2], p[3]}};
  hipLaunchKernelGGL(k_start, dim3(grid1((n + 3) / 4, 256), 4), dim3(256), 0, s, A, n, ctl, beta1, beta2, tickets);
  return hipGetLastError();
}

hipError_t launch_means(const Means& A, hipStream_t s) {
  const int np = mean_blocks(A.n);
  hipLaunchKernelGGL(k_means, dim3(2 * np), dim3(256), 0, s, A, np);
  return hipGetLastError();
}

hipError_t launch_means_warp(const Means& A, const float* img, const float* d, float* out, float* slope, int n0, int n1,
                             int n2, hipStream_t s) {
  const int np = mean_blocks(A.n), bs = row_span(n2);
  const dim3 g(2 * np + row_blocks((int64_t)n0 * n1, n2, bs));
  if (slope)
    hipLaunchKernelGGL(k_means_warp<true>, g, dim3(256), 0, s, A, np, img, d, out, slope, n0, n1, n2, bs);
  else
    hipLaunchKernelGGL(k_means_warp<false>, g, dim3(256), 0, s, A, np, img, d, out, slope, n0, n1, n2, bs);
  return hipGetLastError();
}

hipError_t launch_sum_partials(const double* partials, int n, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s, partials, n, dst);
  return hipGetLastError();
}

hipError_t launch_partials_ratio(const double* partials, int n, double denom, float* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_mean_final, dim3(1), dim3(256), 0, s, partials, n, denom, dst);
  return hipGetLastError();
}

}  // namespace fa
