// Spatial advection X(dt/2) (Alg. bte_spatial_adv of the paper), the field
// E^{1/2} (eq. bte_semi_implicit_efield), the moments (eq. hybrid_discrete_c and
// the k_i definition of the hybrid model) and the Maxwellian initial state.
//
// X(dt/2):  Y = (U^-1 (x) I) F      -> mode-major Y[i][a][x] (x contiguous)
//           Y_ia <- Q_ia Y_ia        (HBM-bound batched GEMV; Q streamed once per
//                                     ordinate pair thanks to Q(-mu) = J Q(mu) J)
//           F = (U (x) I) Y
#include <cmath>

#include "internal.h"
#include "lu_common.h"

namespace bte {
namespace {

constexpr int kThreads = 256;

__device__ inline bool finite_d(double v) { return (v - v) == 0.0; }

// State to modes, Y_d[i][a][xl] = sum_k W[i][k] F[x][k][a] (TO_X = 0), and back,
// F[x][k][a] = sum_i W[k][i] Y_d[i][a][xl] (TO_X = 1); transposeW: W^T in W's
// place (the X^T path contracts with U^T).  TO_X = 2 adds the sums to the rows of
// the fully implicit system: F <- F + dt sum - Fn (Fn may be NULL), and F = X at
// the inflow entries (x = 0 for cos theta > 0, x = L for cos theta < 0).  A block takes 16 points of one
// discharge, two ordinates and 64 output speeds (16 per wavefront): the points
// of one ordinate are the columns of MFMA f64 products with W, staged in LDS 64
// contracted speeds at a time.  Bound by latency (a few MB and 27 MFLOP per
// transform at 100 x 64 x 16); the tile is what turns the modes' strided
// entries into whole lines: one block per point, as before, wrote Y eight bytes
// at a time and kept 100 of 256 CUs.  The ordinate pairs of 16 points run on
// one XCD, whose L2 joins their parts of the state's lines.
// The contraction ends at Nr (rounded up to 16), and one discharge's place is an
// argument: on small grids a chain of loads, divisions and products on zeros was
// half of the time.  Per transform to modes / back, against one block per point:
// 16 x 16 x 8 3.5 / 3.2 -> 3.6 / 3.2 us (5.2 / 5.1 with 64 speeds contracted always), 180
// x 16 x 8 3.8 / 3.6 (5.4 / 4.6), 18 x 48 x 16 5.0 / 4.8 (6.2 / 6.9), 100 x 64 x 16
// 13.7 / 12.3 -> 6.7 / 6.1 (7.1 / 8.1), 256 x 64 x 32 23 / 22 -> 7.8 / 7.9 (8.4 / 9.4).
constexpr int kModeX = 16, kModeA = 2, kModeK = 64;
template <int TO_X>
__global__ __launch_bounds__(kThreads) void k_modes(double* __restrict__ F, double* __restrict__ Y,
                                                    const double* __restrict__ W, const int* __restrict__ x_off,
                                                    const int* __restrict__ nx_of, int nr, int nth, int transposeW,
                                                    int tiles, int nd, int nx_one, int* __restrict__ status,
                                                    const double* __restrict__ X, const double* __restrict__ Fn,
                                                    const double* __restrict__ mu, double dt) {
  using V2 = double __attribute__((ext_vector_type(2), aligned(8)));   // (F is the caller's: any double address)
  constexpr int XP = kModeX + 2;
  __shared__ double sF[kModeA][kModeK][XP];
  const int groups = (nr + 63) / 64, pairs = nth / kModeA;
  int tile, item;
  xcd_map(blockIdx.x, pairs * groups, tiles * nd, &tile, &item);
  if (tile >= tiles * nd) return;
  // (one discharge: no loads before those of the state)
  const int d = nd == 1 ? 0 : tile / tiles;
  const int nx = nd == 1 ? nx_one : nx_of[d], xo = nd == 1 ? 0 : x_off[d];
  const int xt = (tile - d * tiles) * kModeX;
  if (xt >= nx) return;
  const int grp = groups == 1 ? 0 : item / pairs;
  const int a0 = (item - grp * pairs) * kModeA, n = nr * nth;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  double* Yd = Y + (size_t)xo * n;
  double* Fd = F + (size_t)xo * n;
  const int m0 = grp * 64 + 16 * w;   // this wavefront's output speeds
  const int mrow = min(m0 + li, nr - 1);
  const double* wr = W + (transposeW ? (size_t)mrow : (size_t)mrow * nr);
  const int ws = transposeW ? nr : 1;
  f64x4 acc[kModeA];
#pragma unroll
  for (int a = 0; a < kModeA; ++a) acc[a] = f64x4{0, 0, 0, 0};
  bool bad = false;
  for (int k0 = 0; k0 < nr; k0 += kModeK) {
    double wv[kModeK / 4];
#pragma unroll
    for (int q = 0; q < kModeK / 4; ++q) {
      if (q % 4 == 0 && k0 + 4 * q >= nr) break;   // (the contraction ends at Nr, rounded up to 16)
      wv[q] = wr[(size_t)min(k0 + 4 * q + lk, nr - 1) * ws];
    }
    if (k0 > 0) __syncthreads();
    // (loads without branches, from entries of the discharge; all before the first store)
    if constexpr (TO_X) {
      constexpr int NU = kModeA * kModeK * kModeX / kThreads, KU = kModeK / NU;
      double v[NU];
      const int x = tid % kModeX, a = tid / kModeX % kModeA, k = k0 + tid / (kModeX * kModeA);
      const double* p = Yd + (size_t)(a0 + a) * nx + min(xt + x, nx - 1);
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (u % (16 / KU) == 0 && k0 + KU * u >= nr) break;
        v[u] = p[(size_t)min(k + KU * u, nr - 1) * (nth * nx)];
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (u % (16 / KU) == 0 && k0 + KU * u >= nr) break;
        sF[a][k - k0 + KU * u][x] = (k + KU * u < nr && xt + x < nx) ? v[u] : 0.0;
      }
    } else {
      constexpr int NU = kModeK * kModeX / kThreads, XU = kModeX / NU;
      V2 v[NU];
      const int k = tid % kModeK, x = tid / kModeK;
      const double* p = Fd + (size_t)min(k0 + k, nr - 1) * nth + a0;
#pragma unroll
      for (int u = 0; u < NU; ++u) v[u] = *reinterpret_cast<const V2*>(p + (size_t)min(xt + x + XU * u, nx - 1) * n);
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        bad |= !finite_d(v[u][0]) | !finite_d(v[u][1]);
        const bool in = k0 + k < nr && xt + x + XU * u < nx;
        sF[0][k][x + XU * u] = in ? v[u][0] : 0.0;
        sF[1][k][x + XU * u] = in ? v[u][1] : 0.0;
      }
    }
    __syncthreads();
    if (m0 < nr) {
#pragma unroll
      for (int q = 0; q < kModeK / 4; ++q) {
        if (q % 4 == 0 && k0 + 4 * q >= nr) break;
#pragma unroll
        for (int a = 0; a < kModeA; ++a)
          acc[a] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv[q], sF[a][4 * q + lk][li], acc[a], 0, 0, 0);
      }
    }
  }
  if (!TO_X && bad) atomicOr(status, kStNonFinite);
  const int x = xt + li;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int m = m0 + lk + 4 * t;   // result row of item t
    if (m >= nr || x >= nx) continue;
    if constexpr (TO_X) {
      const size_t o = (size_t)x * n + (size_t)m * nth + a0, og = (size_t)xo * n + o;
      V2 v = V2{acc[0][t], acc[1][t]};
      if constexpr (TO_X == 2) {
        const V2 f = *reinterpret_cast<const V2*>(Fd + o), xv = *reinterpret_cast<const V2*>(X + og);
        const V2 fn = Fn ? *reinterpret_cast<const V2*>(Fn + og) : V2{0.0, 0.0};
#pragma unroll
        for (int a = 0; a < kModeA; ++a) {
          const double c = mu[a0 + a];
          const bool inflow = (x == 0 && c > 0.0) | (x == nx - 1 && c < 0.0);
          v[a] = inflow ? xv[a] : f[a] + dt * v[a] - fn[a];
        }
      }
      *reinterpret_cast<V2*>(Fd + o) = v;
    } else {
#pragma unroll
      for (int a = 0; a < kModeA; ++a) Yd[(size_t)(m * nth + a0 + a) * nx + x] = acc[a][t];
    }
  }
}

// Batched Chebyshev-system application for one (eigen-speed i, ordinate pair).
// Qt holds Q_{i,a} transposed (Qt[c][r] = Q[r][c]) for the ordinates with cos > 0;
// the mirrored ordinate uses Q(-mu) y = J Q(mu) J y.  transpose=1 applies Q^T.
// Q is read once per half-step (537 MB at 256 x 64 x 32 in FP64) by non-temporal
// loads, which bound it: sums of 33 to 128 columns are split over two or four
// groups of threads (shorter ones are on their way at once already), and the
// transposed product takes eight columns per wavefront, so that enough of them
// are in flight.  Per half-step: 100 x 64 x 16 13.2 -> 10.2 us, 256 x 64 x 32 83 ->
// 79 (6.8 TB/s); transposed, 128 x 32 x 16, 39 -> 11.
template <typename QT, int TRANSPOSE>
__global__ __launch_bounds__(kThreads) void k_advect(double* __restrict__ Y, const QT* __restrict__ Qt,
                                                     const size_t* __restrict__ q_off, const int* __restrict__ x_off,
                                                     const int* __restrict__ nx_of, int nr, int nth) {
  extern __shared__ double sy[];
  const int m = blockIdx.x;
  const int d = blockIdx.y;
  const int nh = nth / 2;
  const int i = m / nh, h = m % nh;
  const int nx = nx_of[d];
  const int n = nr * nth;
  double* Yd = Y + (size_t)x_off[d] * n;
  double* yp = Yd + (size_t)(i * nth + nh + h) * nx;
  double* yn = Yd + (size_t)(i * nth + nh - 1 - h) * nx;
  const QT* Q = Qt + q_off[d] + (size_t)m * nx * nx;
  for (int c = threadIdx.x; c < nx; c += blockDim.x) {
    sy[c] = yp[c];
    sy[nx + c] = yn[nx - 1 - c];
  }
  __syncthreads();
  if (!TRANSPOSE) {
    // out[r] = sum_c Q[r][c] y[c] = sum_c Qt[c][r] y[c]: coalesced over r
    static_assert(kThreads == 256, "threads per group");
    __shared__ double s_sum[2][kThreads];
    const int lg = nx <= 32 ? 0 : (nx <= 64 ? 2 : (nx <= 128 ? 1 : 0)), groups = 1 << lg, tg = kThreads >> lg;
    const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> (8 - lg));
    const int len = (nx + groups - 1) >> lg, c0 = g * len, c1 = min(nx, c0 + len);
    for (int r = threadIdx.x & (tg - 1); r < nx; r += tg) {
      double ap = 0.0, an = 0.0;
#pragma unroll 16
      for (int c = c0; c < c1; ++c) {
        const double q = static_cast<double>(__builtin_nontemporal_load(&Q[(size_t)c * nx + r]));
        ap += q * sy[c];
        an += q * sy[nx + c];
      }
      if (groups > 1) {
        s_sum[0][threadIdx.x] = ap;
        s_sum[1][threadIdx.x] = an;
      } else {
        yp[r] = ap;
        yn[nx - 1 - r] = an;
      }
    }
    if (groups > 1) {
      __syncthreads();
      const int r = threadIdx.x;
      if (r < nx) {
        double ap = 0.0, an = 0.0;
        for (int u = 0; u < groups; ++u) {
          ap += s_sum[0][u * tg + r];
          an += s_sum[1][u * tg + r];
        }
        yp[r] = ap;
        yn[nx - 1 - r] = an;
      }
    }
  } else {
    // out[c] = sum_r Q[r][c] y[r] = sum_r Qt[c][r] y[r]: eight outputs c per wavefront
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int c = 8 * wid; c < nx; c += 8 * (kThreads / 64)) {
      double ap[8], an[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) ap[u] = an[u] = 0.0;
#pragma unroll 2
      for (int r0 = 0; r0 < nx; r0 += 64) {
        const int r = r0 + lane, rc = min(r, nx - 1);
        double q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          q[u] = static_cast<double>(__builtin_nontemporal_load(&Q[(size_t)min(c + u, nx - 1) * nx + rc]));
        const double zp = r < nx ? sy[rc] : 0.0, zn = r < nx ? sy[nx + rc] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          ap[u] += q[u] * zp;
          an[u] += q[u] * zn;
        }
      }
      const double tp = fold8(ap, lane), tn = fold8(an, lane);
      const int cc = c + lane;
      if (lane < 8 && cc < nx) {
        yp[cc] = tp;
        yn[nx - 1 - cc] = tn;
      }
    }
  }
}

// Poisson field over all points: rhs[x] = -(e/eps0)(n_i - u^T F) at interior
// points, the electrode voltage / 0 at the walls (one wavefront per point);
// then E[x] = (P_d rhs_d)[x] (one wavefront per point, lanes along P's row).
__global__ __launch_bounds__(kThreads) void k_field_rhs(double t_half, double freq, double V0,
                                                        const double* __restrict__ Fh, const double* __restrict__ ni,
                                                        double* __restrict__ rhs, const int* __restrict__ x_disc,
                                                        const int* __restrict__ x_off, const int* __restrict__ nx_of,
                                                        const double* __restrict__ mom, int nx_total, int n) {
  const int x = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (x >= nx_total) return;
  const int d = x_disc[x], xl = x - x_off[d];
  const double kE = 1.602176634e-19, kEps0 = 8.8541878128e-12, kPi = 3.14159265358979323846;
  const double* f = Fh + (size_t)x * n;
  double s = 0.0;
  for (int c = lane; c < n; c += 64) s += mom[c] * f[c];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) {
    double v = -(kE / kEps0) * (ni[x] - s);
    if (xl == 0) v = V0 * sin(2.0 * kPi * freq * t_half);
    if (xl == nx_of[d] - 1) v = 0.0;
    rhs[x] = v;
  }
}

__global__ __launch_bounds__(kThreads) void k_field_apply(const double* __restrict__ rhs, double* __restrict__ E,
                                                          const int* __restrict__ x_disc,
                                                          const int* __restrict__ x_off, const int* __restrict__ nx_of,
                                                          const double* __restrict__ P,
                                                          const size_t* __restrict__ p_off, int nx_total) {
  const int x = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (x >= nx_total) return;
  const int d = x_disc[x], x0 = x_off[d], nx = nx_of[d], j = x - x0;
  const double* row = P + p_off[d] + (size_t)j * nx;
  double s = 0.0;
  for (int c = lane; c < nx; c += 64) s += row[c] * rhs[x0 + c];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) E[x] = s;
}

// E^{1/2} for the specified modes (one block per discharge).
__global__ __launch_bounds__(kThreads) void k_field(int mode, double t_half, double freq, double a1, double V0,
                                                    const double* __restrict__ Fh, const double* __restrict__ Eg,
                                                    const double* __restrict__ ni, double* __restrict__ E,
                                                    const int* __restrict__ x_off, const int* __restrict__ nx_of,
                                                    const double* __restrict__ E0_of, const double* __restrict__ xhat,
                                                    const double* __restrict__ mom, const double* __restrict__ P,
                                                    const size_t* __restrict__ p_off, int n) {
  const int d = blockIdx.x;
  const int x0 = x_off[d], nx = nx_of[d];
  const double kPi = 3.14159265358979323846;
  if (mode == 0 || mode == 1 || mode == 2) {
    const double s = (mode == 1) ? sin(2.0 * kPi * freq * t_half) : 1.0;
    for (int j = threadIdx.x; j < nx; j += blockDim.x) {
      const int x = x0 + j;
      E[x] = (mode == 2) ? Eg[x] : (mode == 0 ? E0_of[d] : E0_of[d] * s * (1.0 + a1 * xhat[x]));
    }
  }
  // Poisson (mode 3) runs as k_field_rhs and k_field_apply
}

// gE0[d] += sum_{x in d} gE[x] dE_x/dE0_d
__global__ void k_field_dE0(int mode, double t_half, double freq, double a1, const double* __restrict__ gE,
                            double* __restrict__ gE0, const int* __restrict__ x_off, const int* __restrict__ nx_of,
                            const double* __restrict__ xhat) {
  const int d = blockIdx.x;
  const double kPi = 3.14159265358979323846;
  const double s = (mode == 1) ? sin(2.0 * kPi * freq * t_half) : 1.0;
  double acc = 0.0;
  for (int j = threadIdx.x; j < nx_of[d]; j += blockDim.x) {
    const int x = x_off[d] + j;
    acc += gE[x] * (mode == 1 ? s * (1.0 + a1 * xhat[x]) : 1.0);
  }
  __shared__ double red[kThreads / 64];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
    gE0[d] += t;
  }
}

__device__ inline void block_sum3(double& a, double& b, double& c, double* red) {
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off);
    b += __shfl_xor(b, off);
    c += __shfl_xor(c, off);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if (lane == 0) {
    red[3 * wid] = a;
    red[3 * wid + 1] = b;
    red[3 * wid + 2] = c;
  }
  __syncthreads();
  a = b = c = 0.0;
  for (int w = 0; w < nw; ++w) {
    a += red[3 * w];
    b += red[3 * w + 1];
    c += red[3 * w + 2];
  }
}

// Moments per x: n_e = u.F, mean energy = e.F / n_e, k_i = k.F / n_e
__global__ __launch_bounds__(kThreads) void k_moments(const double* __restrict__ F, const double* __restrict__ mom,
                                                      double* __restrict__ out, int n, int nx_total) {
  __shared__ double red[3 * (kThreads / 64)];
  const int x = blockIdx.x;
  const double* f = F + (size_t)x * n;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    const double v = f[j];
    a += mom[j] * v;
    b += mom[n + j] * v;
    c += mom[2 * n + j] * v;
  }
  block_sum3(a, b, c, red);
  if (threadIdx.x == 0) {
    out[x] = a;
    out[nx_total + x] = (a != 0.0) ? b / a : 0.0;
    out[2 * nx_total + x] = (a != 0.0) ? c / a : 0.0;
  }
}

// lam[x] += g0 u + g1 (e - ebar u)/ne + g2 (k - kbar u)/ne
__global__ __launch_bounds__(kThreads) void k_moments_vjp(const double* __restrict__ F, const double* __restrict__ mom,
                                                          const double* __restrict__ g, double* __restrict__ lam, int n,
                                                          int nx_total) {
  __shared__ double red[3 * (kThreads / 64)];
  const int x = blockIdx.x;
  const double* f = F + (size_t)x * n;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    const double v = f[j];
    a += mom[j] * v;
    b += mom[n + j] * v;
    c += mom[2 * n + j] * v;
  }
  block_sum3(a, b, c, red);
  const double g0 = g[x], g1 = g[nx_total + x], g2 = g[2 * nx_total + x];
  const double inv = (a != 0.0) ? 1.0 / a : 0.0;
  const double eb = b * inv, kb = c * inv;
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    const double u = mom[j];
    lam[(size_t)x * n + j] += g0 * u + g1 * (mom[n + j] - eb * u) * inv + g2 * (mom[2 * n + j] - kb * u) * inv;
  }
}

__global__ void k_maxwellian(const double* __restrict__ ne, const double* __restrict__ coeff, double* __restrict__ F,
                             int nr, int nth, int nx_total) {
  const size_t n = (size_t)nr * nth;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n * nx_total;
       idx += (size_t)gridDim.x * blockDim.x) {
    const size_t x = idx / n;
    const int k = static_cast<int>((idx % n) / nth);
    F[idx] = ne[x] * coeff[k];
  }
}

}  // namespace

template <int TO_X>
static void run_modes(const DevOps& d, double* F, const double* W, int transposeW, hipStream_t s,
                      const double* X = nullptr, const double* Fn = nullptr) {
  const int tiles = (d.max_nx + kModeX - 1) / kModeX;
  const int grid = xcd_grid(d.nth / kModeA * ((d.nr + 63) / 64), tiles * d.nd);
  k_modes<TO_X><<<grid, kThreads, 0, s>>>(F, d.Y, W, d.x_off, d.nx_of, d.nr, d.nth, transposeW, tiles, d.nd, d.max_nx, d.status,
                                         X, Fn, d.mu_th, d.dt);
}

void launch_x_to_modes(const DevOps& d, const double* F, hipStream_t s) {
  run_modes<0>(d, const_cast<double*>(F), d.Uinv, 0, s);
}

void launch_x_to_modes_T(const DevOps& d, const double* F, hipStream_t s) {
  run_modes<0>(d, const_cast<double*>(F), d.U, 1, s);
}

void launch_modes_to_x(const DevOps& d, double* F, hipStream_t s) { run_modes<1>(d, F, d.U, 0, s); }

void launch_modes_to_rows(const DevOps& d, double* R, const double* X, const double* Fn, hipStream_t s) {
  run_modes<2>(d, R, d.U, 0, s, X, Fn);
}

void launch_modes_to_x_T(const DevOps& d, double* F, hipStream_t s) { run_modes<1>(d, F, d.Uinv, 1, s); }

void launch_advect(const DevOps& d, bool fp32, bool transpose, hipStream_t s, const double* Qt) {
  dim3 grid(d.nr * d.nh, d.nd);
  const size_t sh = sizeof(double) * 2 * d.max_nx;
  if (Qt) {   // other FP64 inverses in the layout of d.Qt (forward only)
    k_advect<double, 0><<<grid, kThreads, sh, s>>>(d.Y, Qt, d.q_off, d.x_off, d.nx_of, d.nr, d.nth);
  } else if (fp32) {
    if (transpose) k_advect<float, 1><<<grid, kThreads, sh, s>>>(d.Y, d.Qt32, d.q_off, d.x_off, d.nx_of, d.nr, d.nth);
    else k_advect<float, 0><<<grid, kThreads, sh, s>>>(d.Y, d.Qt32, d.q_off, d.x_off, d.nx_of, d.nr, d.nth);
  } else {
    if (transpose) k_advect<double, 1><<<grid, kThreads, sh, s>>>(d.Y, d.Qt, d.q_off, d.x_off, d.nx_of, d.nr, d.nth);
    else k_advect<double, 0><<<grid, kThreads, sh, s>>>(d.Y, d.Qt, d.q_off, d.x_off, d.nx_of, d.nr, d.nth);
  }
}

void launch_field(const DevOps& d, int mode, double t_half, double freq, double a1, double V0, const double* Fh,
                  const double* E_given, const double* ni, double* E, hipStream_t s, double* rhs) {
  if (mode == 3) {
    if (!rhs) rhs = d.field_rhs;
    const int gb = (d.nx_total + kThreads / 64 - 1) / (kThreads / 64);
    k_field_rhs<<<gb, kThreads, 0, s>>>(t_half, freq, V0, Fh, ni, rhs, d.x_disc, d.x_off, d.nx_of, d.mom,
                                        d.nx_total, d.n);
    k_field_apply<<<gb, kThreads, 0, s>>>(rhs, E, d.x_disc, d.x_off, d.nx_of, d.poisson, d.p_off,
                                          d.nx_total);
    return;
  }
  k_field<<<d.nd, kThreads, 0, s>>>(mode, t_half, freq, a1, V0, Fh, E_given, ni, E, d.x_off, d.nx_of, d.E0_of,
                                    d.xhat, d.mom, d.poisson, d.p_off, d.n);
}

void launch_field_dE0(const DevOps& d, int mode, double t_half, double freq, double a1, const double* gE, double* gE0,
                      hipStream_t s) {
  k_field_dE0<<<d.nd, kThreads, 0, s>>>(mode, t_half, freq, a1, gE, gE0, d.x_off, d.nx_of, d.xhat);
}

void launch_moments(const DevOps& d, const double* F, double* out, hipStream_t s) {
  k_moments<<<d.nx_total, kThreads, 0, s>>>(F, d.mom, out, d.n, d.nx_total);
}

void launch_moments_vjp(const DevOps& d, const double* F, const double* gbar, double* lam, hipStream_t s) {
  k_moments_vjp<<<d.nx_total, kThreads, 0, s>>>(F, d.mom, gbar, lam, d.n, d.nx_total);
}

void launch_maxwellian(const DevOps& d, const double* ne, const double* coeff, double* F, hipStream_t s) {
  const size_t total = (size_t)d.n * d.nx_total;
  const int blocks = static_cast<int>(std::min<size_t>((total + kThreads - 1) / kThreads, 65535));
  k_maxwellian<<<blocks, kThreads, 0, s>>>(ne, coeff, F, d.nr, d.nth, d.nx_total);
}

}  // namespace bte
