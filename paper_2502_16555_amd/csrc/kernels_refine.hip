// FP64 refinement of the mixed-precision V step and the adjoint gradient
// contractions.  The residual r = b - (I - dt (n0 C + E A)) x is the operator
// action of Alg. vspace_action of the paper evaluated in FP64 with MFMA f64;
// the refinement x += LU^-1 r repeats until max|r| <= rtol max|b| (a device
// flag stops the remaining sweeps without a host synchronization).
#include <algorithm>
#include <cmath>

#include "internal.h"
#include "lu_common.h"
#include "tile_products.h"

namespace bte {
namespace {

// Rows of n entries (the caller's, at any double address) <-> rows padded with
// zeros to npad, a block per row (n is even: two ordinates per mu).
__global__ __launch_bounds__(256) void k_pad(const double* __restrict__ F, double* __restrict__ Bp, int n, int npad) {
  const double* f = F + (size_t)blockIdx.x * n;
  double* b = Bp + (size_t)blockIdx.x * npad;
  for (int j = 2 * threadIdx.x; j < npad; j += 512)
    *reinterpret_cast<V2u*>(b + j) = j < n ? *reinterpret_cast<const V2u*>(f + j) : V2u{0.0, 0.0};
}

__global__ __launch_bounds__(256) void k_unpad(const double* __restrict__ Bp, double* __restrict__ F, int n, int npad) {
  const double* b = Bp + (size_t)blockIdx.x * npad;
  double* f = F + (size_t)blockIdx.x * n;
  for (int j = 2 * threadIdx.x; j < n; j += 512)
    *reinterpret_cast<V2u*>(f + j) = *reinterpret_cast<const V2u*>(b + j);
}

// Ordinates <-> harmonics of every point: harmonic coefficients
// Bh[l * nr + k] = sum_a TS[l][a] F[k][a] (P_S of eq. (proj_ops), l-major, padded
// rows of npad, l < nl) and back.  With nl = nth, P_O P_S = I and the way back is
// F[k][a] = sum_l TO[a][l] Xh[l * nr + k] (P_O).  With nl < nth the operator part
// of the V system has rank nr nl, (I - P_O K P_S)^-1 = I - P_O P_S + P_O (I - K)^-1 P_S
// (T_S T_O = I_nl), so the way back adds the solution's harmonic change to the
// state: F[k][a] += sum_l TO[a][l] (Xh - Bh)[l * nr + k].
__global__ __launch_bounds__(256) void k_to_harm(const double* __restrict__ F, const double* __restrict__ TS,
                                                 double* __restrict__ Bh, int nr, int nth, int nl, int npad) {
  extern __shared__ double sh[];
  const int n = nr * nth, x = blockIdx.x;
  double* sF = sh;
  double* sT = sh + n;
  for (int i = threadIdx.x; i < n; i += blockDim.x) sF[i] = F[(size_t)x * n + i];
  for (int i = threadIdx.x; i < nl * nth; i += blockDim.x) sT[i] = TS[i];
  __syncthreads();
  for (int o = threadIdx.x; o < npad; o += blockDim.x) {
    double v = 0.0;
    if (o < nr * nl) {
      const int l = o / nr, k = o % nr;
      for (int a = 0; a < nth; ++a) v += sT[l * nth + a] * sF[k * nth + a];
    }
    Bh[(size_t)x * npad + o] = v;
  }
}

__global__ __launch_bounds__(256) void k_from_harm(const double* __restrict__ Xh, const double* __restrict__ Bh,
                                                   const double* __restrict__ TO, double* __restrict__ F, int nr,
                                                   int nth, int nl, int npad) {
  extern __shared__ double sh[];
  const int n = nr * nth, nhm = nr * nl, x = blockIdx.x;
  const bool reduced = nl < nth;
  double* sX = sh;
  double* sT = sh + nhm;
  for (int i = threadIdx.x; i < nhm; i += blockDim.x)
    sX[i] = reduced ? Xh[(size_t)x * npad + i] - Bh[(size_t)x * npad + i] : Xh[(size_t)x * npad + i];
  for (int i = threadIdx.x; i < nth * nl; i += blockDim.x) sT[i] = TO[i];
  __syncthreads();
  for (int o = threadIdx.x; o < n; o += blockDim.x) {
    const int k = o / nth, a = o % nth;
    double v = 0.0;
    for (int l = 0; l < nl; ++l) v += sT[a * nl + l] * sX[l * nr + k];
    F[(size_t)x * n + o] = reduced ? F[(size_t)x * n + o] + v : v;
  }
}

// ---------------------------------------------------------------------------
// FP64 residual R = B - X + dt n0_x (X C^T) + dt E_x (X A^T)  (TRANSPOSE: C, A)
// rows = collocation points, ld doubles apart.  MODE 0: the refinement residual, with the
// per-point maxima (skipped once the refinement is done); MODE 1: R = B - M X
// only; MODE 2: R = M X (operator action of Alg. vspace_action, for the Krylov
// solver); MODE 3: R = B - dt E (X A^T) (the field-coupling term of the fully
// implicit Jacobian, eq. 1dbte_jac_action).
//
// A block computes 16 PT points x 16 OT outputs by tile_products, whose partial
// tiles meet in LDS.  Bound by the FP64 matrix rate (64 cycles per 16 x 16 x 4 product and SIMD)
// where the tiles fill the chip: hence two shapes.  64 x 32 tiles of four
// wavefronts load half as much per product, and run where they give every CU a
// block; otherwise 32 x 16 tiles of eight wavefronts make eight times as many
// blocks' worth of parallel work from a small grid.  The blocks of one output
// tile run on one XCD, so that its rows of C and A come from HBM once.
// Per residual (32 x 64 tiles staged in LDS, one barrier pair per 64 of k, no
// split before): 100 points, n = 1024 57 -> 19 us; 200 points, n = 512 33 -> 11; 256
// points, n = 2048 122 -> 83 (53 us at 69 TFLOP/s).  Three chunks in flight took
// 22 us at the first, five 28: they push each other out of the 32 KB vector cache.
// ---------------------------------------------------------------------------
template <int TRANSPOSE, int MODE, int PT, int OT, int NW>
__global__ __launch_bounds__(NW * 64) void k_residual(const double* __restrict__ Bv, const double* __restrict__ Xv,
                                                      double* __restrict__ Rv, const double* __restrict__ C,
                                                      const double* __restrict__ Aop, const double* __restrict__ E,
                                                      const double* __restrict__ n0x,
                                                      unsigned long long* __restrict__ rmax,
                                                      unsigned long long* __restrict__ bmax,
                                                      unsigned long long* __restrict__ xmax,
                                                      const int* __restrict__ done, double dt, int n, int ld,
                                                      int nx, const int* __restrict__ skip) {
  if (MODE == 0 && *done) return;   // (no launch that may run beside this one writes it)
  constexpr int BM = 16 * PT, BN = 16 * OT;
  constexpr int NOP = MODE == 3 ? 1 : 2;         // operators: A, then C
  int bx, by;
  xcd_map(blockIdx.x, (nx + BM - 1) / BM, (n + BN - 1) / BN, &bx, &by);
  if (bx * BN >= n) return;
  const int x0 = by * BM, i0 = bx * BN;
  if (MODE != 0 && skip) {  // points already converged need no operator action
    bool all = true;
    for (int u = 0; u < BM && x0 + u < nx; ++u)
      if (!skip[x0 + u]) all = false;
    if (all) return;
  }
  __shared__ double s_part[NW][NOP][BM][BN];
  const int tid = threadIdx.x;
  const double* M[NOP];
  M[0] = Aop;
  if constexpr (NOP == 2) M[1] = C;
  tile_products<TRANSPOSE, NOP, PT, OT, NW>(Xv, ld, M, n, n, nx, x0, i0, s_part);
  // sums, result, and (MODE 0) max |r|, |b| and |x| per point, reduced over the
  // tile's outputs before one atomic per point (bit patterns of non-negative
  // doubles order like the values, and a NaN orders above +inf)
  using u64 = unsigned long long;
#pragma unroll
  for (int e = tid; e < BM * BN; e += NW * 64) {
    const int xl = e / BN, il = e % BN, x = x0 + xl, i = i0 + il;
    u64 rb = 0, bb = 0, xb = 0;
    if (x < nx && i < n) {
      double sA = 0.0, sC = 0.0;
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        sA += s_part[u][0][xl][il];
        if constexpr (NOP == 2) sC += s_part[u][NOP - 1][xl][il];
      }
      const size_t o = (size_t)x * ld + i;
      if (MODE == 0) {
        const double bv = Bv[o], xv = Xv[o];
        const double r = bv - xv + dt * n0x[x] * sC + dt * E[x] * sA;
        Rv[o] = r;
        rb = static_cast<u64>(__double_as_longlong(fabs(r)));
        bb = static_cast<u64>(__double_as_longlong(fabs(bv)));
        xb = static_cast<u64>(__double_as_longlong(fabs(xv)));
      } else if (MODE == 3) {
        Rv[o] = Bv[o] - dt * E[x] * sA;
      } else {
        const double mx = Xv[o] - dt * n0x[x] * sC - dt * E[x] * sA;
        Rv[o] = (MODE == 1) ? Bv[o] - mx : mx;
      }
    }
    if constexpr (MODE == 0) {
#pragma unroll
      for (int off = 1; off < BN; off <<= 1) {
        const u64 orb = __shfl_xor(rb, off), obb = __shfl_xor(bb, off), oxb = __shfl_xor(xb, off);
        rb = orb > rb ? orb : rb;
        bb = obb > bb ? obb : bb;
        xb = oxb > xb ? oxb : xb;
      }
      if (il == 0 && x < nx) {
        atomicMax(&rmax[x], rb);
        atomicMax(&bmax[x], bb);
        atomicMax(&xmax[x], xb);
      }
    }
  }
}

template <int TRANSPOSE, int MODE>
void run_residual(const DevOps& d, const double* B, const double* X, double* R, const double* E, const int* skip,
                  int ld, hipStream_t s, int sweep = 0) {
  auto go = [&](auto pt, auto ot, auto nw) {
    constexpr int PT = decltype(pt)::value, OT = decltype(ot)::value, NW = decltype(nw)::value;
    const int grid = xcd_grid((d.nx_total + 16 * PT - 1) / (16 * PT), (d.n + 16 * OT - 1) / (16 * OT));
    const size_t o = (size_t)(sweep & 1) * d.nx_total;
    const int* done = d.status + done_slot(sweep + 1);   // of the sweep before
    k_residual<TRANSPOSE, MODE, PT, OT, NW><<<grid, NW * 64, 0, s>>>(B, X, R, d.Cord, d.Aord, E, d.n0x,
                                                                    d.rmax + o, d.bmax + o, d.xmax + o, done, d.dt,
                                                                    d.n, ld, d.nx_total,
                                                                    skip);
  };
  using std::integral_constant;
  // one 64 x 32 tile per CU or more: the larger tiles
  if (((d.nx_total + 63) / 64) * ((d.n + 31) / 32) >= 256)
    go(integral_constant<int, 4>(), integral_constant<int, 2>(), integral_constant<int, 4>());
  else
    go(integral_constant<int, 2>(), integral_constant<int, 1>(), integral_constant<int, 8>());
}

// The test after the last sweep: status[2] = sweeps used, resid[0] = max_x eta_x
// (the sweeps before are tested by the solves, which set the same).
__global__ __launch_bounds__(256) void k_refine_check(RefineCheck c) {
  if (*c.done) return;
  const double worst = refine_worst<256>(c);
  if (threadIdx.x == 0) {
    c.resid[0] = worst;
    c.status[2] = c.sweep;
    if (!(worst <= c.rtol)) atomicOr(c.status, kStNoConv);
  }
}

__global__ void k_reset_refine(unsigned long long* rmax, unsigned long long* bmax, unsigned long long* xmax,
                               int* status, int n) {
  for (int x = threadIdx.x; x < n; x += blockDim.x) {
    rmax[x] = 0ull;
    bmax[x] = 0ull;
    xmax[x] = 0ull;
  }
  if (threadIdx.x == 0) {
    status[done_slot(0)] = status[done_slot(1)] = 0;
    status[2] = 0;
  }
}

// grad_scal[op] += dt sum_x n0_x mu_x^T C^(op) F*_x  and  grad_E[x] = dt mu_x^T A F*_x.
// Tiled like the residual: out[x][i] = sum_k F*[x][k] M[i][k] (tile_products), then
// the epilogue contracts with mu[x][i].  gx tiles of outputs, gy of points and
// n_params + 1 operators, the blocks of one operator's output tile on one XCD.
// Every block writes its partial sums to slots of its own (no atomics), and
// k_adjoint_reduce adds the slots in a fixed order, so the gradients are the same
// bit for bit from run to run:
//   pscal[(op * gy + by) * gx + bx]  = dt sum_{x in block} n0_x (mu_x . out_x)   (op < n_params)
//   pE[x * gx + bx]                  = dt (mu_x . out_x) over the block's i range  (op = n_params)
// 128 points, n = 512, 24 parameters: 193 -> 62 us (32 x 64 tiles through LDS, no load
// in flight during the products, before).
template <int PT, int OT, int NW>
__global__ __launch_bounds__(NW * 64) void k_adjoint_grads(const double* __restrict__ Mu,
                                                           const double* __restrict__ Fs,
                                                           const double* __restrict__ Csb,
                                                           const double* __restrict__ Aop,
                                                           const double* __restrict__ n0x, double* __restrict__ pscal,
                                                           double* __restrict__ pE, double dt, int n, int nx,
                                                           int nparams) {
  constexpr int BM = 16 * PT, BN = 16 * OT;
  const int gx = (n + BN - 1) / BN, gy = (nx + BM - 1) / BM;
  int mi, by;
  xcd_map(blockIdx.x, gy, gx * (nparams + 1), &mi, &by);
  if (mi >= gx * (nparams + 1)) return;
  const int op = mi / gx, bx = mi % gx, x0 = by * BM, i0 = bx * BN, tid = threadIdx.x;
  __shared__ double s_part[NW][1][BM][BN];
  __shared__ double s_pt[BM];
  const double* M[1] = {(op < nparams) ? Csb + (size_t)op * n * n : Aop};
  tile_products<0, 1, PT, OT, NW>(Fs, n, M, n, n, nx, x0, i0, s_part);
  // dt mu . out per point, over the tile's outputs
#pragma unroll
  for (int e = tid; e < BM * BN; e += NW * 64) {
    const int xl = e / BN, il = e % BN, x = x0 + xl, i = i0 + il;
    double v = 0.0;
    if (x < nx && i < n) {
#pragma unroll
      for (int u = 0; u < NW; ++u) v += s_part[u][0][xl][il];
      v *= Mu[(size_t)x * n + i];
    }
#pragma unroll
    for (int off = 1; off < BN; off <<= 1) v += __shfl_xor(v, off);
    if (il == 0) {
      if (op == nparams && x < nx) pE[(size_t)x * gx + bx] = dt * v;
      s_pt[xl] = x < nx ? dt * n0x[x] * v : 0.0;
    }
  }
  __syncthreads();
  if (op < nparams && tid < 64) {
    double v = tid < BM ? s_pt[tid] : 0.0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
    if (tid == 0) pscal[((size_t)op * gy + by) * gx + bx] = v;
  }
}

// Second pass: gscal[op] += sum over the (by, bx) slots, gE[x] = sum over bx, a
// wavefront each, in a fixed order.
__global__ __launch_bounds__(64) void k_adjoint_reduce(const double* __restrict__ pscal,
                                                       const double* __restrict__ pE, double* __restrict__ gscal,
                                                       double* __restrict__ gE, int nparams, int gx, int gy) {
  const int t = blockIdx.x, lane = threadIdx.x;
  const bool sc = t < nparams;
  const double* p = sc ? pscal + (size_t)t * gy * gx : pE + (size_t)(t - nparams) * gx;
  double s = 0.0;
  for (int q = lane; q < (sc ? gx * gy : gx); q += 64) s += p[q];
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) s += __shfl_xor(s, off);
  if (lane == 0) {
    if (sc) gscal[t] += s;
    else gE[t - nparams] = s;
  }
}

}  // namespace

void launch_to_harm(const DevOps& d, int nl, int npad_h, const double* F, const double* TS, double* Bh,
                    hipStream_t s) {
  const size_t sh = (size_t)(d.n + nl * d.nth) * sizeof(double);
  k_to_harm<<<d.nx_total, 256, sh, s>>>(F, TS, Bh, d.nr, d.nth, nl, npad_h);
}

void launch_from_harm(const DevOps& d, int nl, int npad_h, const double* Xh, const double* Bh, const double* TO,
                      double* F, hipStream_t s) {
  const size_t sh = (size_t)(d.nr * nl + nl * d.nth) * sizeof(double);
  k_from_harm<<<d.nx_total, 256, sh, s>>>(Xh, Bh, TO, F, d.nr, d.nth, nl, npad_h);
}

void launch_pad_rows(const DevOps& d, const double* F, double* Bp, hipStream_t s) {
  k_pad<<<d.nx_total, 256, 0, s>>>(F, Bp, d.n, d.npad);
}

void launch_unpad_rows(const DevOps& d, const double* Bp, double* F, hipStream_t s) {
  k_unpad<<<d.nx_total, 256, 0, s>>>(Bp, F, d.n, d.npad);
}

void launch_apply(const DevOps& d, int mode, const double* B, const double* X, double* R, const int* skip,
                  hipStream_t s) {
  if (mode == 1) run_residual<0, 1>(d, B, X, R, d.E, skip, d.npad, s);
  else run_residual<0, 2>(d, B, X, R, d.E, skip, d.npad, s);
}

void launch_apply_field(const DevOps& d, int mode, const double* B, const double* X, double* R, const double* E,
                        hipStream_t s) {
  if (mode == 3) run_residual<0, 3>(d, B, X, R, E, nullptr, d.n, s);
  else run_residual<0, 2>(d, B, X, R, E, nullptr, d.n, s);
}

void launch_residual(const DevOps& d, bool transpose, int sweep, hipStream_t s) {
  if (transpose) run_residual<1, 0>(d, d.B, d.X, d.R, d.E, nullptr, d.npad, s, sweep);
  else run_residual<0, 0>(d, d.B, d.X, d.R, d.E, nullptr, d.npad, s, sweep);
}

namespace {
__global__ void k_fill(double* __restrict__ p, double v, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
}  // namespace

void launch_fill(double* p, double v, size_t n, hipStream_t s) {
  if (n == 0) return;
  const int blocks = static_cast<int>(std::min<size_t>((n + 255) / 256, 1024));
  k_fill<<<blocks, 256, 0, s>>>(p, v, n);
}

void launch_refine_check(const RefineCheck& c, hipStream_t s) { k_refine_check<<<1, 256, 0, s>>>(c); }

void launch_reset_refine(const DevOps& d, hipStream_t s) {
  k_reset_refine<<<1, 256, 0, s>>>(d.rmax, d.bmax, d.xmax, d.status, 2 * d.nx_total);
}

void launch_adjoint_grads(const DevOps& d, double* grad_scal, double* grad_E, hipStream_t s) {
  const int nop = d.n_params + 1;
  auto go = [&](auto pt, auto ot, auto nw) {
    constexpr int PT = decltype(pt)::value, OT = decltype(ot)::value, NW = decltype(nw)::value;
    const int gx = (d.n + 16 * OT - 1) / (16 * OT), gy = (d.nx_total + 16 * PT - 1) / (16 * PT);
    double* pE = d.adj_part + (size_t)d.n_params * gx * gy;
    k_adjoint_grads<PT, OT, NW><<<xcd_grid(gy, gx * nop), NW * 64, 0, s>>>(d.mu, d.Fs, d.Csb, d.Aord, d.n0x, d.adj_part,
                                                                          pE, d.dt, d.n, d.nx_total, d.n_params);
    k_adjoint_reduce<<<d.n_params + d.nx_total, 64, 0, s>>>(d.adj_part, pE, grad_scal, grad_E, d.n_params, gx, gy);
  };
  using std::integral_constant;
  // the residual's tiles, by the same rule over all operators' tiles
  if (((d.nx_total + 63) / 64) * ((d.n + 31) / 32) * nop >= 256)
    go(integral_constant<int, 4>(), integral_constant<int, 2>(), integral_constant<int, 4>());
  else
    go(integral_constant<int, 2>(), integral_constant<int, 1>(), integral_constant<int, 8>());
}

}  // namespace bte
