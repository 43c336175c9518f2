// Global moments (Sec. III-B: centroid, covariance and its largest
// eigenvalue, for the scale).  The local shape descriptors (Sec. III-A) come
// from the grid search in knn_grid.hip.
#include "common.h"
#include "launch.h"

namespace sgr {

struct P3 {
  float x, y, z;
};

// Thread t's share of the coordinate sums, and of the second moments about c.
template <int U>
__device__ inline void moment1(const float* __restrict__ X, const float* __restrict__ Y, const float* __restrict__ Z,
                               int64_t n, int64_t t, double (&s)[3]) {
  s[0] = s[1] = s[2] = 0.0;
  strided<U>(t, n, [&](int64_t i) { return P3{X[i], Y[i], Z[i]}; },
             [&](const P3& p) {
               s[0] += p.x;
               s[1] += p.y;
               s[2] += p.z;
             });
}
template <int U>
__device__ inline void moment2(const float* __restrict__ X, const float* __restrict__ Y, const float* __restrict__ Z,
                               int64_t n, int64_t t, double cx, double cy, double cz, double (&v)[6]) {
  for (int c = 0; c < 6; ++c) v[c] = 0.0;
  strided<U>(t, n, [&](int64_t i) { return P3{X[i], Y[i], Z[i]}; },
             [&](const P3& p) {
               const double ex = p.x - cx, ey = p.y - cy, ez = p.z - cz;
               v[0] += ex * ex;
               v[1] += ey * ey;
               v[2] += ez * ez;
               v[3] += ex * ey;
               v[4] += ex * ez;
               v[5] += ey * ez;
             });
}

// C: the second moments / n.
__device__ inline void moments_store(const double cen[3], const double (&C)[6], double* __restrict__ out) {
  double lam[3];
  eig_psd3(C, lam);
  for (int c = 0; c < 3; ++c) out[c] = cen[c];
  for (int c = 0; c < 6; ++c) out[3 + c] = C[c];
  out[9] = lam[0];
}

// Centroid, covariance (1/n) and its largest eigenvalue; two passes over
// the cloud in one block with a fixed-order FP64 reduction (deterministic).
// Bound by the latency of each thread's loads: eight in flight.
__device__ inline __attribute__((always_inline)) void moments_body(const float* __restrict__ X,
                                                                   const float* __restrict__ Y,
                                                                   const float* __restrict__ Zc, int64_t n,
                                                                   double* __restrict__ out, double* lds,
                                                                   double* cen) {
  double s[3];
  moment1<8>(X, Y, Zc, n, threadIdx.x, s);
  block_sum<3, 1024>(s, lds);
  if (threadIdx.x == 0) {
    for (int c = 0; c < 3; ++c) cen[c] = s[c] / (double)n;
  }
  __syncthreads();
  double v[6];
  moment2<8>(X, Y, Zc, n, threadIdx.x, cen[0], cen[1], cen[2], v);
  block_sum<6, 1024>(v, lds);
  if (threadIdx.x == 0) {
    double C[6];
    for (int c = 0; c < 6; ++c) C[c] = v[c] / (double)n;
    moments_store(cen, C, out);
  }
}

__global__ __launch_bounds__(1024) void moments_kernel(const float* __restrict__ X, const float* __restrict__ Y,
                                                       const float* __restrict__ Zc, int64_t n, double* __restrict__ out) {
  __shared__ double lds[16 * 6];
  __shared__ double cen[3];
  moments_body(X, Y, Zc, n, out, lds, cen);
}

// One block per cloud; cloud c writes out[10 c .. 10 c + 9].
__global__ __launch_bounds__(1024) void moments_batch_kernel(const CloudDesc* __restrict__ clouds,
                                                             double* __restrict__ out) {
  __shared__ double lds[16 * 6];
  __shared__ double cen[3];
  const CloudDesc& c = clouds[blockIdx.x];
  moments_body(gptr(c.x), gptr(c.y), gptr(c.z), c.n, out + 10 * (int64_t)blockIdx.x, lds, cen);
}

// The same with the 16 waves of that block as 16 blocks on as many CUs (the
// additions and their order are the block's): part [0, 48) the sums, [48,
// 144) the second moments.
__global__ __launch_bounds__(64) void moments_wide1_kernel(const float* __restrict__ X, const float* __restrict__ Y,
                                                           const float* __restrict__ Zc, int64_t n,
                                                           double* __restrict__ part) {
  double s[3];
  moment1<20>(X, Y, Zc, n, blockIdx.x * 64 + threadIdx.x, s);
  wave_part<3>(s, part, blockIdx.x);
}
__global__ __launch_bounds__(64) void moments_wide2_kernel(const float* __restrict__ X, const float* __restrict__ Y,
                                                           const float* __restrict__ Zc, int64_t n,
                                                           double* __restrict__ part) {
  const double c = threadIdx.x < 3 ? part_sum(part, 3, threadIdx.x) / (double)n : 0.0;
  double v[6];
  moment2<20>(X, Y, Zc, n, blockIdx.x * 64 + threadIdx.x, lane_value(c, 0), lane_value(c, 1), lane_value(c, 2), v);
  wave_part<6>(v, part + 48, blockIdx.x);
}
__global__ __launch_bounds__(64) void moments_wide3_kernel(int64_t n, const double* __restrict__ part,
                                                           double* __restrict__ out) {
  const double c = threadIdx.x < 3 ? part_sum(part, 3, threadIdx.x) / (double)n : 0.0;
  const double v = threadIdx.x < 6 ? part_sum(part + 48, 6, threadIdx.x) / (double)n : 0.0;
  double cen[3], C[6];
  for (int k = 0; k < 3; ++k) cen[k] = lane_value(c, k);
  for (int k = 0; k < 6; ++k) C[k] = lane_value(v, k);
  if (threadIdx.x == 0) moments_store(cen, C, out);
}

hipError_t launch_moments_batch(const CloudDesc* clouds, int n_clouds, double* out, hipStream_t st) {
  hipLaunchKernelGGL(moments_batch_kernel, dim3(n_clouds), dim3(1024), 0, st, clouds, out);
  return hipGetLastError();
}

hipError_t launch_moments(const float* x, const float* y, const float* z, int64_t n, double* part, double* out,
                          hipStream_t st) {
  if (part && n > WIDE_N) {
    const dim3 waves(16), bt(64);
    hipLaunchKernelGGL(moments_wide1_kernel, waves, bt, 0, st, x, y, z, n, part);
    hipLaunchKernelGGL(moments_wide2_kernel, waves, bt, 0, st, x, y, z, n, part);
    hipLaunchKernelGGL(moments_wide3_kernel, dim3(1), bt, 0, st, n, part, out);
  } else {
    hipLaunchKernelGGL(moments_kernel, dim3(1), dim3(1024), 0, st, x, y, z, n, out);
  }
  return hipGetLastError();
}

}  // namespace sgr
