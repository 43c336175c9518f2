// Registration residual (the RMSE of Sec. V): with correspondences,
// sqrt(mean |T(y_i) - x_corr(i)|^2) over i with corr(i) >= 0; without, the
// one-sided nearest-neighbour RMSE template -> reference.  The nearest
// neighbour is chosen by float32 squared distance of the float32-rounded
// transformed point (ties by index), by a search over all of a small
// reference streamed through LDS or through the grid of a larger one; the
// distance that enters the mean is recomputed in FP64.
#include "common.h"
#include "launch.h"

namespace sgr {

constexpr int RS_BT = 256;

__device__ inline void posed(const float* __restrict__ yx, const float* __restrict__ yy, const float* __restrict__ yz,
                             int i, const double* __restrict__ pose, double T[3]) {
  const double s = pose[0];
  const double p0 = yx[i], p1 = yy[i], p2 = yz[i];
  for (int r = 0; r < 3; ++r)
    T[r] = s * (pose[1 + 3 * r] * p0 + pose[2 + 3 * r] * p1 + pose[3 + 3 * r] * p2) + pose[10 + r];
}

__global__ __launch_bounds__(RS_BT) void residual_kernel(const float* __restrict__ yx, const float* __restrict__ yy,
                                                         const float* __restrict__ yz, int M,
                                                         const float* __restrict__ xx, const float* __restrict__ xy,
                                                         const float* __restrict__ xz, int N,
                                                         const double* __restrict__ pose,
                                                         const int32_t* __restrict__ corr, double* __restrict__ part) {
  __shared__ float4 tile[RS_BT];
  __shared__ double lds[(RS_BT / 64) * 2];
  const int i = blockIdx.x * RS_BT + threadIdx.x;
  const bool valid = i < M;
  double T[3] = {0, 0, 0};
  if (valid) posed(yx, yy, yz, i, pose, T);
  double v[2] = {0, 0};
  if (corr) {
    if (valid && corr[i] >= 0 && corr[i] < N) {
      const int j = corr[i];
      const double dx = T[0] - xx[j], dy = T[1] - xy[j], dz = T[2] - xz[j];
      v[0] = dx * dx + dy * dy + dz * dz;
      v[1] = 1.0;
    }
  } else {
    const float qx = (float)T[0], qy = (float)T[1], qz = (float)T[2];
    float best = INFINITY;
    int bj = -1;
    for (int base = 0; base < N; base += RS_BT) {
      const int j = base + threadIdx.x;
      __syncthreads();
      tile[threadIdx.x] = (j < N) ? make_float4(xx[j], xy[j], xz[j], 0.f) : make_float4(0.f, 0.f, 0.f, 0.f);
      __syncthreads();
      const int cnt = min(RS_BT, N - base);
      for (int jj = 0; jj < cnt; ++jj) {
        const float4 p = tile[jj];
        const float dx = __fsub_rn(p.x, qx), dy = __fsub_rn(p.y, qy), dz = __fsub_rn(p.z, qz);
        // the fused form the compiler's contraction gave these sums, kept so
        // that both searches pick the same point
        const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dx, dx, __fmul_rn(dy, dy)));
        if (d2 < best) {
          best = d2;
          bj = base + jj;
        }
      }
    }
    if (valid && bj >= 0) {
      const double dx = T[0] - xx[bj], dy = T[1] - xy[bj], dz = T[2] - xz[bj];
      v[0] = dx * dx + dy * dy + dz * dz;
      v[1] = 1.0;
    }
  }
  block_sum<2, RS_BT>(v, lds);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = v[0];
    part[2 * blockIdx.x + 1] = v[1];
  }
}

// T(y_i) rounded to FP32, as residual_kernel's search rounds it.
__global__ __launch_bounds__(RS_BT) void residual_pose_kernel(const float* __restrict__ yx, const float* __restrict__ yy,
                                                              const float* __restrict__ yz, int M,
                                                              const double* __restrict__ pose, float* __restrict__ qx,
                                                              float* __restrict__ qy, float* __restrict__ qz) {
  const int i = blockIdx.x * RS_BT + threadIdx.x;
  if (i >= M) return;
  double T[3];
  posed(yx, yy, yz, i, pose, T);
  qx[i] = (float)T[0];
  qy[i] = (float)T[1];
  qz[i] = (float)T[2];
}

__global__ __launch_bounds__(256) void residual_final_kernel(const double* __restrict__ part, int nblk,
                                                             double* __restrict__ out) {
  __shared__ double lds[4 * 2];
  double v[2] = {0, 0};
  for (int b = threadIdx.x; b < nblk; b += 256) {
    v[0] += part[2 * b];
    v[1] += part[2 * b + 1];
  }
  block_sum<2, 256>(v, lds);
  if (threadIdx.x == 0) out[0] = v[1] > 0 ? sqrt(v[0] / v[1]) : NAN;
}

int residual_blocks(int M) { return (M + RS_BT - 1) / RS_BT; }

// Without correspondences the nearest points come from the grid search
// unless the reference is small.  The search over all of it takes 37 us per
// 1 000 reference points (its blocks run side by side: 1 168 us for 32 400
// against 36 000); the grid 30 to 45 us at 2 000, 56 to 385 us at 32 400
// against 36 000 by how far the clouds lie apart.
constexpr int RS_GRID_N = 1024;
bool residual_grid(int N, bool has_corr) { return !has_corr && N > RS_GRID_N; }
static size_t rs_up(size_t b) { return (b + 255) & ~size_t(255); }

size_t residual_workspace(int M, int N, bool grid) {
  const size_t part = rs_up(sizeof(double) * 2 * (size_t)residual_blocks(M));
  return grid ? part + 5 * rs_up(4 * (size_t)M) + grid_nn_workspace(N, M) : part;
}

hipError_t launch_residual(const float* yx, const float* yy, const float* yz, int M, const float* xx, const float* xy,
                           const float* xz, int N, const double* pose, const int32_t* corr, bool grid, void* ws,
                           double* rmse_out, hipStream_t st) {
  const int nblk = residual_blocks(M);
  char* p = (char*)ws;
  double* part = (double*)p;
  if (grid) {
    p += rs_up(sizeof(double) * 2 * (size_t)nblk);
    float* q[5];
    for (int a = 0; a < 5; ++a) {
      q[a] = (float*)p;
      p += rs_up(4 * (size_t)M);
    }
    int32_t* nn = (int32_t*)q[3];
    hipLaunchKernelGGL(residual_pose_kernel, dim3(nblk), dim3(RS_BT), 0, st, yx, yy, yz, M, pose, q[0], q[1], q[2]);
    if (hipError_t e = launch_grid_nn(xx, xy, xz, N, q[0], q[1], q[2], M, INFINITY, true, nn, q[4], p, st)) return e;
    corr = nn;
  }
  hipLaunchKernelGGL(residual_kernel, dim3(nblk), dim3(RS_BT), 0, st, yx, yy, yz, M, xx, xy, xz, N, pose, corr, part);
  hipLaunchKernelGGL(residual_final_kernel, dim3(1), dim3(256), 0, st, part, nblk, rmse_out);
  return hipGetLastError();
}

}  // namespace sgr
