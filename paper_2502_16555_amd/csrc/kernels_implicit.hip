// Pieces of the fully implicit electron step (eq. bte_fully_implicit) that the
// semi-implicit kernels do not already provide: the forward spatial operator
// A_x F D_x^T in the speed eigenbasis and the vector kernels of the Newton-Krylov driver (batched dot products with
// deterministic two-stage sums, linear combinations).
#include <stdexcept>

#include "internal.h"
#include "lu_common.h"

namespace bte {
namespace {

constexpr int kThreads = 256;
constexpr int kDotBlocks = 256;

// Y_ia <- lambda_i cos(theta_a) D_x Y_ia for every mode of every discharge
// (mode-major Y of the X step: the modes of discharge d at Y + x_off[d] n, one
// row of nx_d per mode); A_x = U Lambda U^-1 (x) diag(cos theta).  D_x is read
// column-major (entry (x, k) at k nx + x).  A block takes 16 modes, the rows of
// MFMA f64 products with D_x^T; its eight wavefronts take the tiles of 16 points
// in turn (TW tiles each at most, held until all have read their modes).  Bound
// by latency and D_x's way through the vector cache: 100 points x 1024 modes
// 14 -> 10.7 us (a thread per point and eight modes before: 100 threads of 256).
template <int TW>
__global__ __launch_bounds__(512) void k_x_fwd(double* __restrict__ Y, const double* __restrict__ DT,
                                               const size_t* __restrict__ dx_off, const double* __restrict__ lam,
                                               const double* __restrict__ mu, const int* __restrict__ x_off,
                                               const int* __restrict__ nx_of, int nth, int n) {
  constexpr int NW = 512 / 64;
  const int o0 = blockIdx.x * 16, d = blockIdx.y, nx = nx_of[d];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  double* y0 = Y + (size_t)x_off[d] * n;
  const double* D = DT + dx_off[d];
  const double* yr = y0 + (size_t)min(o0 + li, n - 1) * nx;
  int xc[TW];   // this lane's point in each tile (beyond the last: repeated, dropped below)
#pragma unroll
  for (int t = 0; t < TW; ++t) xc[t] = min(16 * (w + NW * t) + li, nx - 1);
  f64x4 acc[TW];
#pragma unroll
  for (int t = 0; t < TW; ++t) acc[t] = f64x4{0, 0, 0, 0};
  const int steps = (nx + 3) / 4;
  constexpr int UN = 16 / TW;   // steps whose loads are on their way together
  for (int q0 = 0; q0 < steps; q0 += UN) {
    double yv[UN], dv[UN][TW];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int k = 4 * (q0 + u) + lk, kc = min(k, nx - 1);
      yv[u] = yr[kc];
#pragma unroll
      for (int t = 0; t < TW; ++t) dv[u][t] = D[(size_t)kc * nx + xc[t]];
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const double y = 4 * (q0 + u) + lk < nx ? yv[u] : 0.0;
#pragma unroll
      for (int t = 0; t < TW; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(y, dv[u][t], acc[t], 0, 0, 0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    const int x = 16 * (w + NW * t) + li;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = o0 + lk + 4 * i;   // result row of item i
      if (x < nx && o < n) y0[(size_t)o * nx + x] = lam[o / nth] * mu[o % nth] * acc[t][i];
    }
  }
}

// partial[b][v] = sum over block b's slice of w . V_v   (v < nvec, V_v = V + v stride)
__global__ __launch_bounds__(kThreads) void k_dots(const double* __restrict__ w, const double* __restrict__ V,
                                                   int nvec, size_t stride, size_t N, double* __restrict__ partial) {
  __shared__ double red[kThreads / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int v = 0; v < nvec; ++v) {
    const double* vv = V + (size_t)v * stride;
    double s = 0.0;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x)
      s += w[i] * vv[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) red[wid] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int u = 0; u < kThreads / 64; ++u) t += red[u];
      partial[(size_t)blockIdx.x * nvec + v] = t;
    }
    __syncthreads();
  }
}

// y = beta y + sum_v coef[v] V_v
__global__ __launch_bounds__(kThreads) void k_comb(double* __restrict__ y, double beta, const double* __restrict__ V,
                                                   const double* __restrict__ coef, int nvec, size_t stride,
                                                   size_t N) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x) {
    double s = (beta == 0.0) ? 0.0 : beta * y[i];
    for (int v = 0; v < nvec; ++v) s += coef[v] * V[(size_t)v * stride + i];
    y[i] = s;
  }
}

// Sum of k_dots' partial sums of one vector, one thread per block of k_dots, in a
// fixed order (a serial sum of the 256 took 27 us of latency); on every thread.
__device__ inline double dot_sum(const double* __restrict__ partial, int stride) {
  static_assert(kDotBlocks == kThreads, "one partial sum per thread");
  __shared__ double red[kThreads / 64];
  double t = partial[(size_t)threadIdx.x * stride];
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// The Gram-Schmidt coefficients of one pass from k_dots' partial sums, a block
// per vector: h[v] = t_v (first pass) or h[v] + t_v (second pass), coef[v] =
// -t_v for k_comb.
__global__ __launch_bounds__(kThreads) void k_gs_reduce(const double* __restrict__ partial, int nvec, int accumulate,
                                                        double* __restrict__ h, double* __restrict__ coef) {
  const int v = blockIdx.x;
  const double t = dot_sum(partial + v, nvec);
  if (threadIdx.x == 0) {
    h[v] = accumulate ? h[v] + t : t;
    coef[v] = -t;
  }
}

// *h = sqrt(t), t = w . w from k_dots' partial sums; y = y / *h where *h > 0
// (else y is left as it is).  Every block sums the partials itself.
__global__ __launch_bounds__(kThreads) void k_normalize(double* __restrict__ y, const double* __restrict__ partial,
                                                        double* __restrict__ h, size_t N) {
  const double hv = sqrt(dot_sum(partial, 1));
  if (blockIdx.x == 0 && threadIdx.x == 0) *h = hv;
  if (!(hv > 0.0)) return;
  const double a = 1.0 / hv;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x)
    y[i] = a * y[i];
}

// y = a y + b x
__global__ __launch_bounds__(kThreads) void k_axpby(double* __restrict__ y, const double* __restrict__ x, double a,
                                                    double b, size_t N) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x)
    y[i] = a * y[i] + b * x[i];
}

}  // namespace

void launch_x_forward(const DevOps& d, hipStream_t s) {
  if (d.max_nx > 1024) throw std::invalid_argument("Nx above 1024");
  dim3 g((d.n + 15) / 16, d.nd);
  auto go = [&](auto tw) {
    k_x_fwd<decltype(tw)::value><<<g, 512, 0, s>>>(d.Y, d.dxT, d.p_off, d.lam, d.mu_th, d.x_off, d.nx_of, d.nth, d.n);
  };
  // 16-point tiles per wavefront
  if (d.max_nx <= 128) go(std::integral_constant<int, 1>());
  else if (d.max_nx <= 256) go(std::integral_constant<int, 2>());
  else if (d.max_nx <= 512) go(std::integral_constant<int, 4>());
  else go(std::integral_constant<int, 8>());
}

int dot_blocks() { return kDotBlocks; }

void launch_dots(const double* w, const double* V, int nvec, size_t stride, size_t N, double* partial,
                 hipStream_t s) {
  k_dots<<<kDotBlocks, kThreads, 0, s>>>(w, V, nvec, stride, N, partial);
}

void launch_comb(double* y, double beta, const double* V, const double* coef, int nvec, size_t stride, size_t N,
                 hipStream_t s) {
  k_comb<<<1024, kThreads, 0, s>>>(y, beta, V, coef, nvec, stride, N);
}

void launch_gs_reduce(const double* partial, int nvec, int accumulate, double* h, double* coef, hipStream_t s) {
  k_gs_reduce<<<nvec, kThreads, 0, s>>>(partial, nvec, accumulate, h, coef);
}

void launch_normalize(double* y, const double* partial, double* h, size_t N, hipStream_t s) {
  k_normalize<<<1024, kThreads, 0, s>>>(y, partial, h, N);
}

void launch_axpby(double* y, const double* x, double a, double b, size_t N, hipStream_t s) {
  k_axpby<<<1024, kThreads, 0, s>>>(y, x, a, b, N);
}

}  // namespace bte
