// Pose-independent pair sums of the p = 1 law (eq. 5 with h = 1; eqs. 3, 10).
//
// With p = 1 the pair weight c_ij = exp2(lw_j - (b_i - b_j)^2), lw_j the
// log2 of the reference mass (times a_j / abar for eq. 10), depends on the
// descriptors and masses only, never on the pose.  The force on template
// point i is then linear in its posed position y_i:
//   f_i = -(G / Z) g_i sum_j c_ij (y_i - x_j) = -(G / Z) g_i (y_i S0_i - S1_i),
// with S0_i = sum_j c_ij and S1_i = sum_j c_ij x_j, and its energy term is
// g_i ((|y_i|^2 + eps^2) S0_i - 2 y_i . S1_i + S2_i) with S2_i = sum_j c_ij
// |x_j|^2 (x_j relative to the reference centroid, as everywhere).
//
// psum_kernel forms S0, S1, S2 once per registration (scalar descriptors;
// the vector-descriptor kernel writes the same sums itself), one pass over all
// pairs: a block of 1 024 template points (visiting order, four per lane)
// against one chunk of the reference, staged through LDS 256 points at a
// time; every lane sums a tile's 256 terms per point in FP32 and adds them
// to FP64 sums, as the force kernel does.  psum_reduce_kernel adds the chunks in a fixed order.  pinv_kernel
// is then the whole per-iteration force: O(M) work that poses the template
// exactly as the force kernel does (FP64 pose, FP32 posed point), forms the
// forces in FP64 and writes the same per-block wrench partials for the
// update kernel.
#include <algorithm>

#include "common.h"
#include "launch.h"
#include "update.h"

namespace sgr {

namespace {

constexpr int PS_BT = 256;
constexpr int PS_NQ = 5;  // S0, S1 (3), S2
// Reference points whose weights are formed before any of them is added: the
// exponentials' latency stays off the sums, which are added in the same order
// whatever U.
constexpr int PS_U = 4;

// Sums of R template points per lane (positions ip0 + r * PS_BT) over the
// reference points [j0, j1) of one LDS tile after the other, written to
// out[5 ip ..]; every staged point is read from LDS once for the lane's R
// points.  Q: with S2, which only the energy reads (left 0 otherwise).  Each
// point meets a tile's terms in order in FP32 and adds the tile's sums to
// FP64, so its sums depend neither on R nor on where whole tiles are cut
// into chunks beyond FP64 rounding.
template <int R, bool Q>
__device__ inline void psum_block(const float4* __restrict__ tm4, int M, const float4* __restrict__ ref4,
                                  const float* __restrict__ lw, int j0, int j1, int ip0, float4* s_x, float2* s_l,
                                  double* __restrict__ out) {
  constexpr int NQ = Q ? PS_NQ : PS_NQ - 1;
  constexpr int U = PS_U;
  float bi[R];
#pragma unroll
  for (int r = 0; r < R; ++r) bi[r] = ip0 + r * PS_BT < M ? tm4[ip0 + r * PS_BT].w : 0.f;
  double t[R][NQ];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < NQ; ++q) t[r][q] = 0.0;
  for (int base = j0; base < j1; base += PS_BT) {
    __syncthreads();
    {
      const int j = base + threadIdx.x;
      float4 X = make_float4(0.f, 0.f, 0.f, 0.f);
      float l = -INFINITY;  // exp2(-inf) = 0: beyond the range
      if (j < j1) {
        X = ref4[j];
        l = lw[j];
      }
      s_x[threadIdx.x] = X;
      s_l[threadIdx.x] = make_float2(l, __builtin_fmaf(X.x, X.x, __builtin_fmaf(X.y, X.y, X.z * X.z)));
    }
    __syncthreads();
    // whole groups of U: points beyond the range have zero weight
    const int n = min(PS_BT, j1 - base);
    float a[R][NQ];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < NQ; ++q) a[r][q] = 0.f;
    for (int jj = 0; jj < n; jj += U) {
      float4 X[U];
      float c[U][R];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        X[u] = s_x[jj + u];
        const float2 l = s_l[jj + u];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float d = bi[r] - X[u].w;
          c[u][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(-d, d, l.x));
        }
        if constexpr (Q) X[u].w = l.y;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          a[r][0] += c[u][r];
          a[r][1] = __builtin_fmaf(c[u][r], X[u].x, a[r][1]);
          a[r][2] = __builtin_fmaf(c[u][r], X[u].y, a[r][2]);
          a[r][3] = __builtin_fmaf(c[u][r], X[u].z, a[r][3]);
          if constexpr (Q) a[r][4] = __builtin_fmaf(c[u][r], X[u].w, a[r][4]);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < NQ; ++q) t[r][q] += (double)a[r][q];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int ip = ip0 + r * PS_BT;
    if (ip < M) {
      double* o = out + (int64_t)ip * PS_NQ;
#pragma unroll
      for (int q = 0; q < PS_NQ; ++q) o[q] = q < NQ ? t[r][q < NQ ? q : 0] : 0.0;
    }
  }
}

// One registration: PS_R * 256 template points per block against one chunk.
constexpr int PS_R = 4;

template <bool Q>
__global__ __launch_bounds__(PS_BT) void psum_kernel(const float4* __restrict__ tm4, int M,
                                                     const float4* __restrict__ ref4, const float* __restrict__ lw,
                                                     int N, int chunk_len, double* __restrict__ part) {
  __shared__ float4 s_x[PS_BT];
  __shared__ float2 s_l[PS_BT];
  const int n_iblk = (M + PS_BT * PS_R - 1) / (PS_BT * PS_R);
  const int iblk = blockIdx.x % n_iblk, chunk = blockIdx.x / n_iblk;
  const int j0 = chunk * chunk_len, j1 = min(N, j0 + chunk_len);
  psum_block<PS_R, Q>(tm4, M, ref4, lw, j0, j1, iblk * PS_BT * PS_R + threadIdx.x, s_x, s_l,
                      part + (int64_t)chunk * M * PS_NQ);
}

// A batch: block = one item (registration, block of PS_RB * 256 template
// points, reference chunk) of a list in decreasing cost, so that the long
// items start first and the short ones fill the end of the launch.  A
// registration with one chunk writes its sums at once.
constexpr int PS_RB = 3;

__global__ __launch_bounds__(PS_BT) void psum_batch_kernel(const PsumReg* __restrict__ regs,
                                                           const int4* __restrict__ items, int chunk_len,
                                                           const float4* __restrict__ ref4,
                                                           const float* __restrict__ lw) {
  __shared__ float4 s_x[PS_BT];
  __shared__ float2 s_l[PS_BT];
  const int4 it = items[blockIdx.x];
  const PsumReg g = regs[it.x];
  const int j0 = it.z * chunk_len, j1 = min(g.N, j0 + chunk_len);
  double* out = g.n_chunks == 1 ? g.S : g.part + (int64_t)it.z * g.M * PS_NQ;
  psum_block<PS_RB, true>(gptr(g.tm4), g.M, ref4 + g.ref_off, lw + g.ref_off, j0, j1,
                          it.y * PS_BT * PS_RB + threadIdx.x, s_x, s_l, gptr(out));
}

// One sum over the chunks, in chunk order, eight loads in flight.
__device__ inline double chunk_sum(const double* __restrict__ p, int64_t stride, int n) {
  constexpr int U = 8;
  double s = 0.0;
  for (int c = 0; c < n; c += U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[min(c + u, n - 1) * stride];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < n) s += v[u];
  }
  return s;
}

// Chunk sums of the registrations with several chunks, in chunk order; the
// grid covers (registration, 256 values) through blockIdx.y and a stride.
__global__ __launch_bounds__(256) void psum_reduce_batch_kernel(const PsumReg* __restrict__ regs) {
  const PsumReg g = regs[blockIdx.y];
  if (g.n_chunks == 1) return;
  const double* __restrict__ part = gptr(g.part);
  const int64_t ne = (int64_t)g.M * PS_NQ;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < ne; e += (int64_t)gridDim.x * 256) {
    gptr(g.S)[e] = chunk_sum(part + e, ne, g.n_chunks);
  }
}

__global__ __launch_bounds__(256) void psum_reduce_kernel(const double* __restrict__ part, int M, int n_chunks,
                                                          double* __restrict__ S) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)M * PS_NQ) return;
  S[e] = chunk_sum(part + e, (int64_t)M * PS_NQ, n_chunks);
}

// Wrench terms of template point ip (visiting order) of one registration:
// the posed point as the force kernel forms it (FP64 pose, rounded once to
// FP32), then its force and energy from the pair sums s, in FP64.
template <bool WU>
__device__ inline void pinv_point(const float4* __restrict__ tm4, const float2* __restrict__ tmx, const double* s,
                                  int ip, const double* __restrict__ pose, const Derived& D, int t, double* w) {
  double sR[9], cv[3];
  const double sc = pose[0];
#pragma unroll
  for (int e = 0; e < 9; ++e) sR[e] = sc * pose[1 + e];
#pragma unroll
  for (int r = 0; r < 3; ++r)
    cv[r] = sR[3 * r] * D.ybar0[0] + sR[3 * r + 1] * D.ybar0[1] + sR[3 * r + 2] * D.ybar0[2] + pose[10 + r] -
            D.xbar[r];
  // eq. (12), reading: iteration t uses 0.1 G1 + 0.9 G1 / (1 + exp(-(t - 1 - E/2)))
  const double G = 0.1 * D.G1 + 0.9 * D.G1 / (1.0 + exp(-(((double)t - 1.0) - 0.5 * D.E)));
  const double coef = -(G / D.Z) * D.coefL;
  const double ucoef = (G / D.Z) * D.coefL / (D.p + 1.0);
  const float4 T = tm4[ip];
  const double ex = (double)T.x - D.ybar0[0], ey = (double)T.y - D.ybar0[1], ez = (double)T.z - D.ybar0[2];
  // the posed point relative to xbar, rounded once to FP32
  const float pxf = (float)(sR[0] * ex + sR[1] * ey + sR[2] * ez + cv[0]);
  const float pyf = (float)(sR[3] * ex + sR[4] * ey + sR[5] * ez + cv[1]);
  const float pzf = (float)(sR[6] * ex + sR[7] * ey + sR[8] * ez + cv[2]);
  const double px = pxf, py = pyf, pz = pzf;
  const double tx = px * s[0] - s[1], ty = py * s[0] - s[2], tz = pz * s[0] - s[3];
  const float2 A2 = tmx[ip];
  const double gi = D.g_mode == 1.0 ? (double)A2.x / D.abar : 1.0;
  const double mi = (double)A2.y;
  const double fx = coef * gi * tx, fy = coef * gi * ty, fz = coef * gi * tz;
  const double cx = px - cv[0], cy = py - cv[1], cz = pz - cv[2];
  w[WR_F + 0] = mi * fx;
  w[WR_F + 1] = mi * fy;
  w[WR_F + 2] = mi * fz;
  w[WR_K + 0] = fx * cx;
  w[WR_K + 1] = fx * cy;
  w[WR_K + 2] = fx * cz;
  w[WR_K + 3] = fy * cx;
  w[WR_K + 4] = fy * cy;
  w[WR_K + 5] = fy * cz;
  w[WR_K + 6] = fz * cx;
  w[WR_K + 7] = fz * cy;
  w[WR_K + 8] = fz * cz;
  if constexpr (WU)
    w[WR_U] = ucoef * gi * ((px * px + py * py + pz * pz + D.eps2) * s[0] - 2.0 * (px * s[1] + py * s[2] + pz * s[3]) +
                            s[4]);
}

__global__ __launch_bounds__(256) void pack_plain_kernel(const float* __restrict__ x, const float* __restrict__ y,
                                                         const float* __restrict__ z, const float* __restrict__ mY, int M,
                                                         float4* __restrict__ tm4, float2* __restrict__ tmx) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= M) return;
  tm4[i] = make_float4(x[i], y[i], z[i], 0.f);
  tmx[i] = make_float2(0.f, mY ? mY[i] : 1.f);
}

template <bool WU>
__global__ __launch_bounds__(PS_BT) void pinv_kernel(const float4* __restrict__ tm4, const float2* __restrict__ tmx,
                                                     const double* __restrict__ S, int M,
                                                     const double* __restrict__ pose, const Derived* __restrict__ dv,
                                                     int t, double* __restrict__ wpart) {
  __shared__ double s_red[(PS_BT / 64) * 13];
  double w[13];
#pragma unroll
  for (int e = 0; e < 13; ++e) w[e] = 0.0;
  const int ip = blockIdx.x * PS_BT + threadIdx.x;
  if (ip < M) pinv_point<WU>(tm4, tmx, S + (int64_t)ip * PS_NQ, ip, pose, *dv, t, w);
  block_sum<13, PS_BT>(w, s_red);
  if (threadIdx.x == 0) {
    double* o = wpart + (int64_t)blockIdx.x * WR_STRIDE;
#pragma unroll
    for (int e = 0; e < 13; ++e) o[e] = w[e];
  }
}

// Batched form: block (r, b) of tblk, wrench slot regs[r].wslot0 + b (regs
// here describe the slot layout of this kernel: one slot per 256 points).
template <bool WU>
__global__ __launch_bounds__(PS_BT) void pinv_batch_kernel(const RegDesc* __restrict__ regs,
                                                           const int2* __restrict__ tblk,
                                                           const PsumReg* __restrict__ sums,
                                                           const double* __restrict__ poses,
                                                           const Derived* __restrict__ dvs, int t,
                                                           double* __restrict__ wpart) {
  __shared__ double s_red[(PS_BT / 64) * 13];
  const int2 rb = tblk[blockIdx.x];
  const RegDesc g = reg_at(regs, rb.x);
  double w[13];
#pragma unroll
  for (int e = 0; e < 13; ++e) w[e] = 0.0;
  const int ip = rb.y * PS_BT + threadIdx.x;
  if (ip < g.M)
    pinv_point<WU>(g.tm4, g.tmx, gptr(sums[rb.x].S) + (int64_t)ip * PS_NQ, ip, poses + 13 * (int64_t)rb.x, dvs[rb.x],
                   t, w);
  block_sum<13, PS_BT>(w, s_red);
  if (threadIdx.x == 0) {
    double* o = wpart + ((int64_t)g.wslot0 + rb.y) * WR_STRIDE;
#pragma unroll
    for (int e = 0; e < 13; ++e) o[e] = w[e];
  }
}

// ------------------------------------------------------ iteration loop
// All iterations of a registration in one launch.  An iteration is O(M) and
// bound by latency and launches: with the per-iteration kernels the
// 32 400-point scan took 17 us per iteration (pinv_kernel 4.5, update_kernel
// 7.7, and the gaps), of which the arithmetic is below 1 us; with this kernel
// it takes 5.3 us, and a one-block registration 3.3 us.  Here a block of LP_BT threads keeps LP_PPT template points per
// thread in registers (their coordinates and pair sums) for the whole loop;
// per iteration it poses them as the force kernel does (FP64 pose, rounded
// once to FP32), sums the wrench, and runs the FP64 update itself.
//
// A registration of more than LP_BT * LP_PPT points is spread over up to
// LP_MAX_BLOCKS blocks that exchange their 13 partial sums through memory.
// Every block sums all partials in block order and runs the same update on
// the same numbers, so there is one exchange and no second barrier per
// iteration.  A grid barrier would make every block write back and
// invalidate its XCD's L2 (7.4 us measured for one); instead each 64-bit word
// of the exchange carries half a double and the iteration's tag, is stored
// and polled with relaxed atomics at device scope, and so is valid by itself:
// no ordering between words is needed.  Two slots per block alternate: a
// block can only write iteration t + 2's words after reading every block's
// t + 1 words, which their writers store after having read iteration t's.
//
// Progress: block indices are tickets taken at the start, so the blocks of
// the lowest unfinished registration are running or finished; at most
// LP_MAX_BLOCKS of a registration wait for each other, a quarter of the
// chip's CUs.  Should they still not be resident together (a stream
// confined to a few CUs), the poll gives up after `spins` tries, every wave
// ends, ST_STALLED is set, and the caller runs the per-iteration kernels
// instead, from the pose saved in pose0 (a block that has all partials of the
// last iteration may have stored its result).
constexpr int LP_BT = 512;
constexpr int LP_WAVES = LP_BT / 64;
constexpr int LP_WORDS = 26;  // two tagged words per wrench component

// The iterations of one block: add(sR, cv, b, wu, v) adds the wrench terms of
// the thread's points, posed with s R, cv about the centroid b, to v[0, 13)
// (the energy only with wu), without the factors of G.
template <class Add>
__device__ inline void loop_run(const LoopReg& g, int sub, int t0, int t1, int spins, Add&& add) {
  __shared__ double s_part[LP_WAVES][16];
  __shared__ double s_x[LP_MAX_BLOCKS][13];
  __shared__ double s_pose[12];  // s R (9), cv (3)
  __shared__ double s_G[2], s_coef[2], s_ucoef[2];  // G and the force and energy factors, by iteration parity
  __shared__ UpdateIn s_u;                          // the update's state
  __shared__ int s_dead;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const Derived& D = *g.dv;
  // s R and cv of the pose in s_u (thread 0)
  auto share_pose = [&]() {
    double sR[9];
    for (int e = 0; e < 9; ++e) sR[e] = s_u.P[0] * s_u.P[1 + e];
    for (int e = 0; e < 9; ++e) s_pose[e] = sR[e];
    for (int r = 0; r < 3; ++r)
      s_pose[9 + r] = sR[3 * r] * s_u.ybar0[0] + sR[3 * r + 1] * s_u.ybar0[1] + sR[3 * r + 2] * s_u.ybar0[2] +
                      s_u.P[10 + r] - D.xbar[r];
  };
  // thread 64: the factors of iteration t, beside the update of the one before
  auto set_G = [&](int t) {
    const double G = G_sched(D, t);
    s_G[t & 1] = G;
    s_coef[t & 1] = -(G / D.Z) * D.coefL;
    s_ucoef[t & 1] = (G / D.Z) * D.coefL / (D.p + 1.0);
  };
  if (tid == 0) {
    UpdateIn u;
    update_load(g.dv, g.pose, t0, 1.0, u);
    s_u = u;
    share_pose();
    if (sub == 0)
      for (int e = 0; e < 13; ++e) g.pose0[e] = u.P[e];
  }
  if (tid == 64) {
    set_G(t0);
    s_dead = 0;
  }
  __syncthreads();
  for (int t = t0; t < t1; ++t) {
    const bool wu = g.stats != nullptr || (g.energy != nullptr && t == t1 - 1);
    double v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = 0.0;
    double sR[9], cv[3];
    const double b[3] = {D.ybar0[0], D.ybar0[1], D.ybar0[2]};
#pragma unroll
    for (int e = 0; e < 9; ++e) sR[e] = s_pose[e];
#pragma unroll
    for (int r = 0; r < 3; ++r) cv[r] = s_pose[9 + r];
    add(sR, cv, b, wu, v);
    wave_sum_many<16>(v);
    if ((lane & 3) == 0) s_part[wave][lane >> 2] = v[0];
    __syncthreads();
    // this block's wrench sums in threads 0..12
    double w = 0.0;
    if (tid < 13)
      for (int q = 0; q < LP_WAVES; ++q) w += s_part[q][tid];
    if (g.nb > 1) {
      unsigned long long* slot = g.xch + (size_t)(t & 1) * g.nb * LP_WORDS;
      const unsigned tag = (unsigned)(t - t0 + 1);
      if (tid < 13) {
        const unsigned long long bits = (unsigned long long)__double_as_longlong(w);
        unsigned long long* o = slot + (size_t)sub * LP_WORDS + 2 * tid;
        __hip_atomic_store(o, (bits & 0xffffffff00000000ull) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(o + 1, (bits << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      for (int e = tid; e < g.nb * 13; e += LP_BT) {
        const unsigned long long* a = slot + 2 * (size_t)e;  // 13 pairs of words per block, contiguous
        unsigned long long hi = 0, lo = 0;
        int left = spins;
        do {
          hi = __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          lo = __hip_atomic_load(a + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } while (((unsigned)hi != tag || (unsigned)lo != tag) && --left > 0);
        if ((unsigned)hi != tag || (unsigned)lo != tag) s_dead = 1;
        s_x[e / 13][e % 13] = __longlong_as_double((long long)((hi & 0xffffffff00000000ull) | (lo >> 32)));
      }
      __syncthreads();
      if (s_dead) {  // the same value in every thread: set before the barrier, never cleared
        if (tid == 0) atomicOr(&g.dv->status, (int32_t)ST_STALLED);
        return;
      }
      if (tid < 13) {
        w = 0.0;
        for (int q = 0; q < g.nb; ++q) w += s_x[q][tid];
      }
    }
    if (wave == 0) {
      if (tid < 13) w *= tid == WR_U ? s_ucoef[t & 1] : s_coef[t & 1];
      double W[13];
#pragma unroll
      for (int e = 0; e < 13; ++e) W[e] = lane_value(w, e);
      if (tid == 0) {
        const double c = update_core<true>(W, s_u);
        share_pose();
        if (sub == 0) {
          if (g.stats) stats_write(W, s_u, s_G[t & 1], c, g.stats + (size_t)t * STATS_STRIDE);
          if (g.energy && t == t1 - 1) *g.energy = W[WR_U];
        }
      }
    }
    if (tid == 64 && t + 1 < t1) set_G(t + 1);
    __syncthreads();
  }
  if (sub == 0 && tid == 0) {
    update_store(s_u, g.dv);
    for (int e = 0; e < 13; ++e) g.pose[e] = s_u.P[e];
  }
}

template <int PPT>
__device__ inline void loop_body(const LoopReg& g, int sub, int t0, int t1, int spins) {
  const int tid = threadIdx.x;
  const Derived& D = *g.dv;
  // this thread's points: coordinates, g S0 and g S1, mass (the offsets from
  // the centroid are formed again in every iteration, which leaves the update
  // its registers with 8 points)
  float x0[PPT], y0[PPT], z0[PPT], mi[PPT];
  double A0[PPT], Ax[PPT], Ay[PPT], Az[PPT];
  const int p0 = sub * LP_BT * PPT + tid;
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int ip = p0 + u * LP_BT;
    x0[u] = y0[u] = z0[u] = mi[u] = 0.f;
    A0[u] = Ax[u] = Ay[u] = Az[u] = 0.0;
    if (ip < g.M) {
      const float4 T = g.tm4[ip];
      const float2 X = g.tmx[ip];
      const double* S = g.S + (int64_t)ip * PS_NQ;
      const double gi = D.g_mode == 1.0 ? (double)X.x / D.abar : 1.0;
      x0[u] = T.x;
      y0[u] = T.y;
      z0[u] = T.z;
      A0[u] = gi * S[0];
      Ax[u] = gi * S[1];
      Ay[u] = gi * S[2];
      Az[u] = gi * S[3];
      mi[u] = X.y;
    }
  }
  const double eps2 = D.eps2;
  loop_run(g, sub, t0, t1, spins, [&](const double (&sR)[9], const double (&cv)[3], const double (&b)[3], bool wu,
                                      double (&v)[16]) {
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      asm volatile("" : "+v"(x0[k]), "+v"(y0[k]), "+v"(z0[k]));  // kept as floats, not hoisted as doubles
      const double ex = (double)x0[k] - b[0], ey = (double)y0[k] - b[1], ez = (double)z0[k] - b[2];
      const double px = (double)(float)(sR[0] * ex + sR[1] * ey + sR[2] * ez + cv[0]);
      const double py = (double)(float)(sR[3] * ex + sR[4] * ey + sR[5] * ez + cv[1]);
      const double pz = (double)(float)(sR[6] * ex + sR[7] * ey + sR[8] * ez + cv[2]);
      const double fx = px * A0[k] - Ax[k], fy = py * A0[k] - Ay[k], fz = pz * A0[k] - Az[k];
      const double cx = px - cv[0], cy = py - cv[1], cz = pz - cv[2];
      const double m = (double)mi[k];
      v[WR_F + 0] += m * fx;
      v[WR_F + 1] += m * fy;
      v[WR_F + 2] += m * fz;
      v[WR_K + 0] += fx * cx;
      v[WR_K + 1] += fx * cy;
      v[WR_K + 2] += fx * cz;
      v[WR_K + 3] += fy * cx;
      v[WR_K + 4] += fy * cy;
      v[WR_K + 5] += fy * cz;
      v[WR_K + 6] += fz * cx;
      v[WR_K + 7] += fz * cy;
      v[WR_K + 8] += fz * cz;
      if (wu) {
        const int ip = p0 + k * LP_BT;
        if (ip < g.M) {
          const double gi = D.g_mode == 1.0 ? (double)g.tmx[ip].x / D.abar : 1.0;
          v[WR_U] += (px * px + py * py + pz * pz + eps2) * A0[k] - 2.0 * (px * Ax[k] + py * Ay[k] + pz * Az[k]) +
                     gi * g.S[(int64_t)ip * PS_NQ + 4];
        }
      }
    }
  });
}

template <int PPT>
__global__ __launch_bounds__(LP_BT) void pinv_loop_kernel(LoopReg g, int* __restrict__ ticket, int t0, int t1,
                                                          int spins) {
  __shared__ int s_id;
  if (threadIdx.x == 0) s_id = g.nb > 1 ? atomicAdd(ticket, 1) : 0;
  __syncthreads();
  loop_body<PPT>(g, s_id, t0, t1, spins);
}

// blocks: (registration, block within it) in ticket order.
template <int PPT>
__global__ __launch_bounds__(LP_BT) void pinv_loop_batch_kernel(const LoopReg* __restrict__ regs,
                                                                const int2* __restrict__ blocks,
                                                                int* __restrict__ ticket, int t0, int t1, int spins) {
  __shared__ int s_id;
  if (threadIdx.x == 0) s_id = atomicAdd(ticket, 1);
  __syncthreads();
  const int2 rb = blocks[s_id];
  LoopReg g = regs[rb.x];
  g.tm4 = gptr(g.tm4), g.tmx = gptr(g.tmx), g.S = gptr(g.S), g.pose = gptr(g.pose), g.dv = gptr(g.dv);
  g.pose0 = gptr(g.pose0), g.stats = gptr(g.stats), g.energy = gptr(g.energy), g.xch = gptr(g.xch);
  loop_body<PPT>(g, rb.y, t0, t1, spins);
}

// ------------------------------------------ iteration loop of small forces
// The p = 1 force of a small pair, every pair evaluated in every iteration, all
// iterations in one launch.  With the per-iteration kernels 1 024 points took
// 10.8 us an iteration (force_kernel 5.5, update_kernel 5.3), of which the
// pairs are below 1 us; here they take 7.5, bound by the chain of sums,
// exchange and update.  The reference chunks
// are force_kernel's, and the FP32 sums of a point over a chunk's tiles are
// formed in its order with its exponent, so they have its bits; the FP64 sums
// over chunks and points differ by their rounding.  A block of LP_BT threads
// has 256 template points twice, each half of it every other chunk of the
// block's share, which stays in LDS (exponents centred for the block's points)
// with the point's constants in registers.
constexpr int FL_PTS = 256;  // force_kernel's block and tile
constexpr int FL_PAD = 1;     // points of zero weight behind a block's share

__global__ __launch_bounds__(LP_BT) void force_loop_kernel(LoopReg g, ForceLoop F, int* __restrict__ ticket, int t0,
                                                           int t1, int spins) {
  extern __shared__ float4 s_ref[];                      // [F.share + FL_PAD]
  float* s_lw = reinterpret_cast<float*>(s_ref + F.share + FL_PAD);
  __shared__ double s_red[2 * LP_BT / 64];
  __shared__ int s_id;
  if (threadIdx.x == 0) s_id = g.nb > 1 ? atomicAdd(ticket, 1) : 0;
  __syncthreads();
  const int sub = s_id, tid = threadIdx.x;
  const Derived& D = *g.dv;
  const int iblk = sub % F.n_iblk, grp = sub / F.n_iblk;
  const int64_t n_sub = (F.N + F.gran - 1) / F.gran;
  auto chunk0 = [&](int c) { return min(F.N, (int)(c * n_sub / F.n_chunks) * F.gran); };
  const int c0 = (int)((int64_t)grp * F.n_chunks / F.groups), c1 = (int)((int64_t)(grp + 1) * F.n_chunks / F.groups);
  const int J0 = chunk0(c0), J1 = chunk0(c1);
  const int ip = iblk * FL_PTS + tid % FL_PTS;
  const bool on = ip < g.M;
  const float4 T = on ? g.tm4[ip] : make_float4(0.f, 0.f, 0.f, 0.f);
  const float2 TX = on ? g.tmx[ip] : make_float2(0.f, 0.f);
  const float bi = T.w;
  float lo = on ? bi : INFINITY, hi = on ? bi : -INFINITY, beta = 0.f;
  block_range<LP_BT>(lo, hi, s_red);
  const bool expd = expanded_centre(lo, hi, D, false, beta);
  const float al = 2.f * (bi - beta);
  const double dl = (double)(bi - beta);
  const double gi = D.g_mode == 1.0 ? (double)TX.x / D.abar : 1.0;
  const double gs = gi * (expd ? exp2(-dl * dl) : 1.0), mi = (double)TX.y;
  // the chunks' first points within the share (a 64-bit division each)
  int* s_c = reinterpret_cast<int*>(s_lw + F.share + FL_PAD);  // [F.share / F.gran + 1]
  for (int c = tid; c <= c1 - c0; c += LP_BT) s_c[c] = chunk0(c0 + c) - J0;
  for (int j = J0 + tid; j < J1 + FL_PAD; j += LP_BT) {
    float4 X = make_float4(0.f, 0.f, 0.f, 0.f);  // behind the share: zero weight
    float l = -INFINITY;
    if (j < J1) {
      X = F.ref4[j];
      l = F.lw[j];
    }
    if (expd) {
      float d = X.w - beta;
      if (fabsf(d) > 1e18f) d = copysignf(1e18f, d);
      X.w = d;
      l = __builtin_fmaf(-d, d, l);
    }
    s_ref[j - J0] = X;
    s_lw[j - J0] = l;
  }
  __syncthreads();
  loop_run(g, sub, t0, t1, spins, [&](const double (&sR)[9], const double (&cv)[3], const double (&b)[3], bool,
                                      double (&v)[16]) {
    if (!on) return;  // a block's expanded exponent may overflow for others' b
    double S0 = 0.0, Sx = 0.0, Sy = 0.0, Sz = 0.0;
    for (int c = tid / FL_PTS; c < c1 - c0; c += LP_BT / FL_PTS) {
      const int j1 = s_c[c + 1];
      for (int base = s_c[c]; base < j1; base += FL_PTS) {
        const int tn = min(FL_PTS, j1 - base);
        const float4* X = s_ref + base;
        const float* L = s_lw + base;
        float a0 = 0.f, ax = 0.f, ay = 0.f, az = 0.f;
        if (expd) {
          // in pairs, as force_kernel adds them; an odd last point (the
          // reference's) with the zero weight behind it
#pragma unroll 4
          for (int jj = 0; jj < tn; jj += 2) {
            const float4 X0 = X[jj], X1 = X[jj + 1];
            const float w0 = __builtin_amdgcn_exp2f(__builtin_fmaf(al, X0.w, L[jj]));
            const float w1 = __builtin_amdgcn_exp2f(__builtin_fmaf(al, X1.w, L[jj + 1]));
            a0 += w0 + w1;
            ax = __builtin_fmaf(w0, X0.x, __builtin_fmaf(w1, X1.x, ax));
            ay = __builtin_fmaf(w0, X0.y, __builtin_fmaf(w1, X1.y, ay));
            az = __builtin_fmaf(w0, X0.z, __builtin_fmaf(w1, X1.z, az));
          }
        } else {
#pragma unroll 4
          for (int jj = 0; jj < tn; ++jj) {
            const float4 P = X[jj];
            const float db = bi - P.w;
            const float w = __builtin_amdgcn_exp2f(__builtin_fmaf(-db, db, L[jj]));
            a0 += w;
            ax = __builtin_fmaf(w, P.x, ax);
            ay = __builtin_fmaf(w, P.y, ay);
            az = __builtin_fmaf(w, P.z, az);
          }
        }
        S0 += (double)a0;
        Sx += (double)ax;
        Sy += (double)ay;
        Sz += (double)az;
      }
    }
    const double ex = (double)T.x - b[0], ey = (double)T.y - b[1], ez = (double)T.z - b[2];
    const double px = (double)(float)(sR[0] * ex + sR[1] * ey + sR[2] * ez + cv[0]);
    const double py = (double)(float)(sR[3] * ex + sR[4] * ey + sR[5] * ez + cv[1]);
    const double pz = (double)(float)(sR[6] * ex + sR[7] * ey + sR[8] * ez + cv[2]);
    const double fx = gs * (px * S0 - Sx), fy = gs * (py * S0 - Sy), fz = gs * (pz * S0 - Sz);
    const double cx = px - cv[0], cy = py - cv[1], cz = pz - cv[2];
    v[WR_F + 0] = mi * fx;
    v[WR_F + 1] = mi * fy;
    v[WR_F + 2] = mi * fz;
    v[WR_K + 0] = fx * cx;
    v[WR_K + 1] = fx * cy;
    v[WR_K + 2] = fx * cz;
    v[WR_K + 3] = fy * cx;
    v[WR_K + 4] = fy * cy;
    v[WR_K + 5] = fy * cz;
    v[WR_K + 6] = fz * cx;
    v[WR_K + 7] = fz * cy;
    v[WR_K + 8] = fz * cz;
  });
}

}  // namespace

// Reference chunks of psum_kernel, of whole tiles: the cut that costs least by
// the tiles of the CU that has most (14 us each, and a quarter of one for a
// block's start and end) and the chunks' sums to be added (40 bytes a point at
// 4 TB/s), among those that give a CU 3 to 24 blocks where there are enough
// tiles for that.  32 400 x 36 000: 24 chunks, 3 blocks of 6 tiles per CU,
// 268 us; 29 chunks, 4 blocks of 5, took 284.
int pinv_chunks(int M, int N, int n_cu) {
  const int n_iblk = (M + PS_BT * PS_R - 1) / (PS_BT * PS_R);
  const int n_t = (N + PS_BT - 1) / PS_BT;
  int best = 0;
  double best_us = 0.0;
  for (int t = 1; t <= n_t; ++t) {
    const int nc = (n_t + t - 1) / t;
    const int64_t per_cu = ((int64_t)n_iblk * nc + n_cu - 1) / n_cu;
    if (per_cu > 24 && t < n_t) continue;
    if (per_cu < 3 && best > 0) break;
    const double us = 14.0 * (double)per_cu * (t + 0.25) + 1e-5 * (double)nc * M;
    if (best == 0 || us < best_us) best = nc, best_us = us;
  }
  return best;
}

int pinv_blocks(int M) { return (M + PS_BT - 1) / PS_BT; }

hipError_t launch_psum(const float4* tm4, int M, const float4* ref4, const float* lw, int N, int n_chunks,
                       bool want_s2, double* part, double* S, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  const int n_t = (N + PS_BT - 1) / PS_BT;
  const int chunk_len = (n_t + n_chunks - 1) / n_chunks * PS_BT;  // whole tiles
  const int nc = (N + chunk_len - 1) / chunk_len;                // chunks actually used
  const int n_iblk = (M + PS_BT * PS_R - 1) / (PS_BT * PS_R);
  double* out = nc == 1 ? S : part;
  const dim3 grid((unsigned)(n_iblk * nc)), block(PS_BT);
  if (want_s2)
    hipLaunchKernelGGL(psum_kernel<true>, grid, block, 0, st, tm4, M, ref4, lw, N, chunk_len, out);
  else
    hipLaunchKernelGGL(psum_kernel<false>, grid, block, 0, st, tm4, M, ref4, lw, N, chunk_len, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nc == 1) return e;
  return launch_psum_reduce(part, M, nc, S, st);
}

hipError_t launch_psum_reduce(const double* part, int M, int n_chunks, double* S, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  const int64_t ne = (int64_t)M * PS_NQ;
  hipLaunchKernelGGL(psum_reduce_kernel, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st, part, M, n_chunks, S);
  return hipGetLastError();
}

hipError_t launch_pack_plain(const float* x, const float* y, const float* z, const float* mY, int M, float4* tm4,
                             float2* tmx, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  hipLaunchKernelGGL(pack_plain_kernel, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, st, x, y, z, mY, M, tm4, tmx);
  return hipGetLastError();
}

int psum_batch_points() { return PS_BT * PS_RB; }

hipError_t launch_psum_batch(const PsumReg* regs, int n_regs, const int4* items, int n_items, int chunk_len,
                             bool chunked, const float4* ref4, const float* lw, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  hipLaunchKernelGGL(psum_batch_kernel, dim3((unsigned)n_items), dim3(PS_BT), 0, st, regs, items, chunk_len, ref4, lw);
  if (chunked)
    hipLaunchKernelGGL(psum_reduce_batch_kernel, dim3(64, (unsigned)n_regs), dim3(256), 0, st, regs);
  return hipGetLastError();
}

hipError_t launch_pinv_batch(const RegDesc* regs_p, const int2* tblk, int n_tblk, const PsumReg* sums,
                             const double* poses, const Derived* dvs, int t, bool wu, double* wpart, hipStream_t st) {
  if (n_tblk <= 0) return hipSuccess;
  const dim3 grid((unsigned)n_tblk), block(PS_BT);
  if (wu)
    hipLaunchKernelGGL(pinv_batch_kernel<true>, grid, block, 0, st, regs_p, tblk, sums, poses, dvs, t, wpart);
  else
    hipLaunchKernelGGL(pinv_batch_kernel<false>, grid, block, 0, st, regs_p, tblk, sums, poses, dvs, t, wpart);
  return hipGetLastError();
}

hipError_t launch_pinv(const float4* tm4, const float2* tmx, const double* S, int M, const double* pose,
                       const Derived* dv, int t, bool wu, double* wpart, hipStream_t st) {
  const dim3 grid((unsigned)pinv_blocks(M)), block(PS_BT);
  if (wu)
    hipLaunchKernelGGL(pinv_kernel<true>, grid, block, 0, st, tm4, tmx, S, M, pose, dv, t, wpart);
  else
    hipLaunchKernelGGL(pinv_kernel<false>, grid, block, 0, st, tm4, tmx, S, M, pose, dv, t, wpart);
  return hipGetLastError();
}

// Points per thread of the loop kernel.  One registration: few while its
// blocks stay few; an iteration's arithmetic is serial in the points of a
// thread, and the exchange grows with the blocks (us per iteration with 2 / 4
// / 8 points: 3.3 / 3.6 / 4.3 at 1 000 points, one block; 4.7 / 4.8 / 5.4 at
// 16 000; 5.3 / 5.3 / 6.0 at 32 768; 8.7 / 6.2 / 7.1 at 131 072; 8.3 with 8
// at 250 000, where the others no longer fit LP_MAX_BLOCKS).  A batch takes
// the fewest whose blocks all fit on the chip's 256 CUs at once, one each:
// blocks that wait for a second round run all their iterations after the
// first (2.7 / 1.4 / 0.8 ms for 48 registrations of 12 700 points on average).
int loop_points(int64_t M_total, int n_regs) {
  if (n_regs > 1) {
    for (int ppt = 2; ppt < 8; ppt *= 2)
      if (M_total / ((int64_t)LP_BT * ppt) + n_regs / 2 <= 240) return ppt;
    return 8;
  }
  return M_total <= 16384 ? 2 : (M_total <= 131072 ? 4 : 8);
}

// Blocks of a registration; 0: too many points for LP_MAX_BLOCKS blocks, the
// caller keeps the per-iteration kernels.
int loop_blocks(int M, int ppt) {
  const int64_t nb = ((int64_t)M + (int64_t)LP_BT * ppt - 1) / ((int64_t)LP_BT * ppt);
  return nb <= LP_MAX_BLOCKS ? (int)nb : 0;
}

size_t loop_words(int nb) { return nb > 1 ? (size_t)2 * nb * LP_WORDS : 0; }

// The loop's shape for a force launch of n_chunks reference chunks with one
// point a lane; blocks 0: it stays with the per-iteration kernels.  The loop
// has 64 CUs, so its pairs take four times as long: a block's share of the
// reference is limited to FL_SHARE points.  An iteration in the loop and with
// the per-iteration kernels, by the share: 64 points 7.5 and 10.8 us, 256
// 11.8 and 13.6, 512 17.5 and 19.1, 1 024 24.7 and 20.2.
constexpr int FL_SHARE = 512;

ForceLoop force_loop_shape(int M, int N, int n_chunks) {
  ForceLoop F{};
  F.N = N;
  F.gran = force_chunk_gran();
  F.n_chunks = n_chunks;
  F.n_iblk = (M + FL_PTS - 1) / FL_PTS;
  if (force_points_per_block(1) != FL_PTS || force_tile_j() != FL_PTS || F.n_iblk > LP_MAX_BLOCKS) return F;
  F.groups = std::min(n_chunks, LP_MAX_BLOCKS / F.n_iblk);
  const int64_t n_sub = (N + F.gran - 1) / F.gran;
  for (int q = 0; q < F.groups; ++q) {
    const int64_t c0 = (int64_t)q * n_chunks / F.groups, c1 = (int64_t)(q + 1) * n_chunks / F.groups;
    F.share = std::max(F.share, (int)(c1 * n_sub / n_chunks - c0 * n_sub / n_chunks) * F.gran);
  }
  F.blocks = F.share <= FL_SHARE ? F.n_iblk * F.groups : 0;
  return F;
}

hipError_t launch_force_loop(const LoopReg& g, const ForceLoop& F, int* ticket, int t0, int t1, int spins,
                             hipStream_t st) {
  const size_t lds = (size_t)(F.share + FL_PAD) * (sizeof(float4) + sizeof(float)) +
                     (size_t)(F.share / F.gran + 2) * sizeof(int);
  hipLaunchKernelGGL(force_loop_kernel, dim3((unsigned)g.nb), dim3(LP_BT), lds, st, g, F, ticket, t0, t1, spins);
  return hipGetLastError();
}

hipError_t launch_pinv_loop(const LoopReg& g, int ppt, int* ticket, int t0, int t1, int spins, hipStream_t st) {
  const dim3 grid((unsigned)g.nb), block(LP_BT);
  if (ppt == 2)
    hipLaunchKernelGGL(pinv_loop_kernel<2>, grid, block, 0, st, g, ticket, t0, t1, spins);
  else if (ppt == 4)
    hipLaunchKernelGGL(pinv_loop_kernel<4>, grid, block, 0, st, g, ticket, t0, t1, spins);
  else
    hipLaunchKernelGGL(pinv_loop_kernel<8>, grid, block, 0, st, g, ticket, t0, t1, spins);
  return hipGetLastError();
}

hipError_t launch_pinv_loop_batch(const LoopReg* regs, const int2* blocks, int n_blocks, int ppt, int* ticket, int t0,
                                  int t1, int spins, hipStream_t st) {
  const dim3 grid((unsigned)n_blocks), block(LP_BT);
  if (ppt == 2)
    hipLaunchKernelGGL(pinv_loop_batch_kernel<2>, grid, block, 0, st, regs, blocks, ticket, t0, t1, spins);
  else if (ppt == 4)
    hipLaunchKernelGGL(pinv_loop_batch_kernel<4>, grid, block, 0, st, regs, blocks, ticket, t0, t1, spins);
  else
    hipLaunchKernelGGL(pinv_loop_batch_kernel<8>, grid, block, 0, st, regs, blocks, ticket, t0, t1, spins);
  return hipGetLastError();
}

}  // namespace sgr
