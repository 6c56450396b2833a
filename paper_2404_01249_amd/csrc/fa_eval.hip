// Evaluation of a registration result (include/fa_eval.h): label transfer by
// nearest neighbour, per-class overlap counts, and det(I + grad d).
//
// All three are single passes over the volume, bound by HBM bandwidth; they
// run once per registration, not per iteration.  Integer results are exact:
// the rounding of a sample position is decided from the fp32 displacement
// without rounding error, and the determinant is evaluated in double
// precision in a fixed order, without contraction into fused multiply-adds.
#include <algorithm>
#include <vector>

#include "fa_eval.h"
#include "fa_host.h"

using fa::fail;

namespace {

constexpr int kThreads = 256;
constexpr int kMaxBlocks = 2048;
constexpr int kMaxClasses = 127;

int grid_for(int64_t n) {
  const int64_t b = (n + kThreads - 1) / kThreads;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, kMaxBlocks));
}

// round(x + d) along one axis, half up, decided exactly: with q = floor(d),
// d - q is exact in fp32, so the comparison with 1/2 carries no rounding.
__device__ __forceinline__ bool rounded_coord(int x, float dv, int n, int& p) {
  if (!(fabsf(dv) < 1.0e9f)) return false;   // also rejects NaN
  const float q = floorf(dv);
  const int r = (int)q + ((dv - q) >= 0.5f ? 1 : 0);
  p = x + r;
  return p >= 0 && p < n;
}

__global__ void __launch_bounds__(kThreads)
k_warp_labels(const int8_t* __restrict__ lab, const float* __restrict__ d, int8_t* __restrict__ out,
              int n0, int n1, int n2, int bs) {
  const int N = n0 * n1 * n2;
  int x0, x1, x2;
  if (!fa::row_voxel(blockIdx.x, n0, n1, n2, bs, x0, x1, x2)) return;
  const int i = (x0 * n1 + x1) * n2 + x2;
  int p0 = 0, p1 = 0, p2 = 0;
  const float d0 = d[i], d1 = d[N + i], d2 = d[2 * N + i];
  const bool in0 = rounded_coord(x0, d0, n0, p0), in1 = rounded_coord(x1, d1, n1, p1);
  const bool ok = rounded_coord(x2, d2, n2, p2) && in0 && in1;
  out[i] = ok ? lab[(p0 * n1 + p1) * n2 + p2] : (int8_t)-1;
}

// Per-workgroup class counts in LDS, written to part[block][3 * nc].  A thread
// takes 16 neighbouring voxels at a time and counts runs of equal labels: one
// LDS atomic per run and counter instead of one per voxel, which serialise
// where a wavefront's labels are the same (6.9 M voxels: 8 us against 38).
// vec: both arrays are 16-byte aligned.
__global__ void __launch_bounds__(kThreads)
k_overlap_partial(const int8_t* __restrict__ a, const int8_t* __restrict__ b, int64_t n, int nc, int vec,
                  unsigned* __restrict__ part) {
  __shared__ unsigned cnt[3 * kMaxClasses];
  for (int j = threadIdx.x; j < 3 * nc; j += kThreads) cnt[j] = 0u;
  __syncthreads();
  auto flush = [&](int va, int vb, unsigned run) {
    const bool ia = (unsigned)va < (unsigned)nc, ib = (unsigned)vb < (unsigned)nc;
    if (ia) atomicAdd(&cnt[3 * va], run);
    if (ib) atomicAdd(&cnt[3 * vb + 1], run);
    if (ia && va == vb) atomicAdd(&cnt[3 * va + 2], run);
  };
  const int64_t groups = (n + 15) / 16;
  for (int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x; g < groups; g += (int64_t)gridDim.x * kThreads) {
    if (vec && 16 * g + 16 <= n) {
      const int4 A = reinterpret_cast<const int4*>(a)[g], B = reinterpret_cast<const int4*>(b)[g];
      const int wa[4] = {A.x, A.y, A.z, A.w}, wb[4] = {B.x, B.y, B.z, B.w};
      int va = (int8_t)wa[0], vb = (int8_t)wb[0];
      unsigned run = 0u;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int ca = (int8_t)(wa[k / 4] >> (8 * (k % 4))), cb = (int8_t)(wb[k / 4] >> (8 * (k % 4)));
        if (ca != va || cb != vb) {
          flush(va, vb, run);
          va = ca;
          vb = cb;
          run = 0u;
        }
        ++run;
      }
      flush(va, vb, run);
    } else {
      for (int64_t i = 16 * g; i < n && i < 16 * g + 16; ++i) flush(a[i], b[i], 1u);
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < 3 * nc; j += kThreads) part[(size_t)blockIdx.x * 3 * nc + j] = cnt[j];
}

// One workgroup per counter: the sum over the workgroups' partial counts.
__global__ void __launch_bounds__(kThreads)
k_overlap_final(const unsigned* __restrict__ part, int nblocks, int nc, unsigned long long* __restrict__ out) {
  __shared__ unsigned long long red[kThreads];
  const int j = blockIdx.x;
  unsigned long long s = 0ull;
  for (int k = threadIdx.x; k < nblocks; k += kThreads) s += part[(size_t)k * 3 * nc + j];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[j] = red[0];
}

// det(I + grad d) by central differences at interior voxels, in double.
// The expression is the cofactor expansion along the first row, evaluated
// left to right with separate multiplies and adds.  A thread takes V
// neighbours of a row, with rows of a power of two of threads: with V = 4 a
// component's 24 values come in six loads of up to 16 bytes (any 4-byte
// alignment), and no voxel takes an integer division.  The last group of a row is moved
// back onto it and skips the voxels of the group before.  V = 1 for rows below
// four voxels.  (6.9 M voxels with the determinants stored: 35 us against 64
// with a thread per voxel.)
template <int V>
__global__ void __launch_bounds__(kThreads)
k_jacdet(const float* __restrict__ d, int n0, int n1, int n2, int lanes, double* __restrict__ det,
         unsigned* __restrict__ part) {
#pragma clang fp contract(off)
  typedef float floatv __attribute__((ext_vector_type(V), aligned(4)));
  __shared__ unsigned nonpos;
  if (threadIdx.x == 0) nonpos = 0u;
  __syncthreads();
  const int m0 = n0 - 2, m1 = n1 - 2, m2 = n2 - 2;
  const size_t N = (size_t)n0 * n1 * n2;
  const int s1 = n2, s0 = n1 * n2;
  const unsigned groups = (unsigned)(m2 + V - 1) / V, nb = (groups + lanes - 1) / lanes, rows = m0 * m1;
  const unsigned rpb = kThreads / (unsigned)lanes;
  unsigned mine = 0u;
  for (unsigned b = blockIdx.x; b < (rows + rpb - 1) / rpb * nb; b += gridDim.x) {
    const unsigned rb = b / nb, row = rb * rpb + threadIdx.x / (unsigned)lanes;
    const unsigned g = (b - rb * nb) * lanes + threadIdx.x % (unsigned)lanes;
    if (row >= rows || g >= groups) continue;
    const int k0 = (int)(row / m1), k1 = (int)(row - (unsigned)k0 * m1);
    const int first = (int)g * V, k2 = V == 1 ? first : min(first, m2 - V);
    const size_t c = ((size_t)(k0 + 1) * n1 + (k1 + 1)) * n2 + (k2 + 1);
    float z[3][2][V], y[3][2][V], x[3][V + 2];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const float* f = d + q * N + c;
      auto row_of = [](const float* at, float* o) {
        const floatv v = *reinterpret_cast<const floatv*>(at);
#pragma unroll
        for (int i = 0; i < V; ++i) o[i] = v[i];
      };
      row_of(f - s0, z[q][0]);
      row_of(f + s0, z[q][1]);
      row_of(f - s1, y[q][0]);
      row_of(f + s1, y[q][1]);
      row_of(f - 1, x[q]);
      x[q][V] = f[V - 1];
      x[q][V + 1] = f[V];
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
      double J[3][3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        J[q][0] = 0.5 * ((double)z[q][1][i] - (double)z[q][0][i]);
        J[q][1] = 0.5 * ((double)y[q][1][i] - (double)y[q][0][i]);
        J[q][2] = 0.5 * ((double)x[q][i + 2] - (double)x[q][i]);
        J[q][q] = J[q][q] + 1.0;
      }
      const double c0 = J[1][1] * J[2][2] - J[1][2] * J[2][1];
      const double c1 = J[1][0] * J[2][2] - J[1][2] * J[2][0];
      const double c2 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
      const double v = J[0][0] * c0 - J[0][1] * c1 + J[0][2] * c2;
      if (k2 + i < first) continue;   // the group before has it
      if (det) det[((size_t)k0 * m1 + k1) * m2 + k2 + i] = v;
      mine += v <= 0.0 ? 1u : 0u;
    }
  }
  if (mine) atomicAdd(&nonpos, mine);
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = nonpos;
}

__global__ void __launch_bounds__(kThreads)
k_count_final(const unsigned* __restrict__ part, int nblocks, unsigned long long* __restrict__ out) {
  __shared__ unsigned long long red[kThreads];
  unsigned long long s = 0ull;
  for (int k = threadIdx.x; k < nblocks; k += kThreads) s += part[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

// Stream-ordered scratch freed on every return path.
struct Scratch {
  void* p = nullptr;
  hipStream_t s = nullptr;
  ~Scratch() {
    if (p) (void)hipFreeAsync(p, s);
  }
};

}  // namespace

extern "C" {

fa_status fa_warp_labels(const int8_t* labels_dev, const float* d_dev, fa_shape shape, int8_t* out_dev,
                         void* hip_stream) {
  if (!labels_dev || !d_dev || !out_dev) return fail(FA_EINVAL, "labels, d and out must not be NULL");
  FA_TRY(fa::check_shape(shape));
  if ((const void*)labels_dev == (const void*)out_dev) return fail(FA_EINVAL, "out must not alias labels");
  const hipStream_t s = (hipStream_t)hip_stream;
  const int bs = fa::row_span(shape.n2);
  hipLaunchKernelGGL(k_warp_labels, dim3(fa::row_blocks((int64_t)shape.n0 * shape.n1, shape.n2, bs)), dim3(kThreads), 0, s,
                     labels_dev, d_dev, out_dev, shape.n0, shape.n1, shape.n2, bs);
  FA_HIP(hipGetLastError());
  return FA_OK;
}

fa_status fa_label_overlap(const int8_t* a_dev, const int8_t* b_dev, int64_t n, int n_classes,
                           int64_t* counts_host, void* hip_stream) {
  if (!counts_host) return fail(FA_EINVAL, "counts_host is NULL");
  if (n_classes < 1 || n_classes > kMaxClasses) return fail(FA_EINVAL, "n_classes must be in [1, 127]");
  if (n < 0) return fail(FA_EINVAL, "n must be >= 0");
  if (n > 0 && (!a_dev || !b_dev)) return fail(FA_EINVAL, "a and b must not be NULL");
  std::fill(counts_host, counts_host + 3 * n_classes, (int64_t)0);
  if (n == 0) return FA_OK;
  const hipStream_t s = (hipStream_t)hip_stream;
  const int nb = grid_for((n + 15) / 16);
  const int vec = (((uintptr_t)a_dev | (uintptr_t)b_dev) & 15u) == 0;
  const size_t part_bytes = ((size_t)nb * 3 * n_classes * sizeof(unsigned) + 255) & ~(size_t)255;
  Scratch sc;
  sc.s = s;
  FA_HIP(hipMallocAsync(&sc.p, part_bytes + 3 * kMaxClasses * sizeof(unsigned long long), s));
  unsigned* part = (unsigned*)sc.p;
  unsigned long long* tot = (unsigned long long*)((char*)sc.p + part_bytes);
  hipLaunchKernelGGL(k_overlap_partial, dim3(nb), dim3(kThreads), 0, s, a_dev, b_dev, n, n_classes, vec, part);
  FA_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_overlap_final, dim3(3 * n_classes), dim3(kThreads), 0, s, part, nb, n_classes, tot);
  FA_HIP(hipGetLastError());
  std::vector<unsigned long long> h((size_t)3 * n_classes);
  FA_HIP(hipMemcpyAsync(h.data(), tot, h.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
  FA_HIP(hipStreamSynchronize(s));
  for (size_t j = 0; j < h.size(); ++j) counts_host[j] = (int64_t)h[j];
  return FA_OK;
}

fa_status fa_jacobian_det(const float* d_dev, fa_shape shape, double* det_dev, int64_t* n_nonpos_host,
                          int64_t* n_interior_host, void* hip_stream) {
  if (!d_dev) return fail(FA_EINVAL, "d must not be NULL");
  if (shape.n0 < 1 || shape.n1 < 1 || shape.n2 < 1) return fail(FA_ESHAPE, "every dimension must be >= 1");
  if ((double)shape.n0 * shape.n1 * shape.n2 > 536870911.0)
    return fail(FA_ESHAPE, "volume too large: n0*n1*n2 must be < 2^29");
  const int64_t m = shape.n0 < 3 || shape.n1 < 3 || shape.n2 < 3
                        ? 0
                        : (int64_t)(shape.n0 - 2) * (shape.n1 - 2) * (shape.n2 - 2);
  if (n_interior_host) *n_interior_host = m;
  if (n_nonpos_host) *n_nonpos_host = 0;
  if (m == 0) return FA_OK;
  const hipStream_t s = (hipStream_t)hip_stream;
  const int v = shape.n2 - 2 >= 4 ? 4 : 1;
  int lanes = 1;
  while (lanes < 64 && lanes * v < shape.n2 - 2) lanes *= 2;
  const int64_t groups = (shape.n2 - 2 + v - 1) / v, rows = (int64_t)(shape.n0 - 2) * (shape.n1 - 2);
  const int64_t blocks = (rows + kThreads / lanes - 1) / (kThreads / lanes) * ((groups + lanes - 1) / lanes);
  const int nb = (int)std::min<int64_t>(blocks, 16384);
  Scratch sc;
  sc.s = s;
  const size_t part_bytes = ((size_t)nb * sizeof(unsigned) + 255) & ~(size_t)255;
  FA_HIP(hipMallocAsync(&sc.p, part_bytes + sizeof(unsigned long long), s));
  unsigned* part = (unsigned*)sc.p;
  unsigned long long* tot = (unsigned long long*)((char*)sc.p + part_bytes);
  if (v == 4)
    hipLaunchKernelGGL(k_jacdet<4>, dim3(nb), dim3(kThreads), 0, s, d_dev, shape.n0, shape.n1, shape.n2, lanes, det_dev,
                       part);
  else
    hipLaunchKernelGGL(k_jacdet<1>, dim3(nb), dim3(kThreads), 0, s, d_dev, shape.n0, shape.n1, shape.n2, lanes, det_dev,
                       part);
  FA_HIP(hipGetLastError());
  if (!n_nonpos_host) return FA_OK;
  hipLaunchKernelGGL(k_count_final, dim3(1), dim3(kThreads), 0, s, part, nb, tot);
  FA_HIP(hipGetLastError());
  unsigned long long h = 0;
  FA_HIP(hipMemcpyAsync(&h, tot, sizeof(h), hipMemcpyDeviceToHost, s));
  FA_HIP(hipStreamSynchronize(s));
  *n_nonpos_host = (int64_t)h;
  return FA_OK;
}

fa_status fa_compose_fields(const float* u_dev, const float* d_dev, fa_shape shape, float* out_dev,
                            void* hip_stream) {
  if (!u_dev || !d_dev || !out_dev) return fail(FA_EINVAL, "u, d and out must not be NULL");
  if (out_dev == d_dev) return fail(FA_EINVAL, "out must not alias d");
  FA_TRY(fa::check_shape(shape));
  FA_HIP(fa::launch_compose_fields(u_dev, d_dev, out_dev, shape.n0, shape.n1, shape.n2, (hipStream_t)hip_stream));
  return FA_OK;
}

}  // extern "C"
