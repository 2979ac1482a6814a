// Heavies' update of the hybrid model (eq. fluid_step): for every discharge,
//   (n_i^{n+1} - n_i^n)/dt + D_x J_i(E^n, n_i^{n+1}) = (k_i^T F^n) n0 (u^T F^n),
//   J_i = mu_i n_i E - D_i D_x n_i   (eq. hybrid_cnt_a_flux), E = E^n frozen,
// on the CGL collocation points, with the drift outflow condition at the two
// walls (eq. fl_ion_bc, outward normal: J_i . n = n_i max(0, mu_i E . n), no
// inflow) in place of the equation at the wall nodes.  The constant ion
// coefficients are those of the table of modeling parameters (n0 mu_i and
// n0 D_i).  One Nx x Nx dense system per discharge, formed and solved by
// Gaussian elimination with partial pivoting in one block per discharge.
#include <mutex>
#include <type_traits>

#include "internal.h"
#include "lu_common.h"
#include "pivot_steps.h"

namespace bte {
namespace {

constexpr double kIonN0Mu = 4.65e21;  // n0 mu_i [1/(V m s)]
constexpr double kIonN0D = 2.07e20;   // n0 D_i [1/(m s)]
constexpr int kIonThreads = 256;

// M (column-major, Nx x Nx per discharge) and b of the ion system.  Interior
// rows: I/dt + D_x diag(mu E) - D D_x^2; wall rows: the outflow condition (the
// solve scales them to the size of the interior rows, 1/dt -- an equilibration
// that does not change the solution); b = n_i/dt + n0 (k_i weights . F), 0 at
// the walls.  Each block forms 8 columns (all rows, from the column-major
// copies of D_x and D_x^2, so that reads and writes run down the columns) and
// the right-hand sides of the same 8 points.
constexpr int kIonFormCols = 8;
__global__ __launch_bounds__(kIonThreads) void k_ion_form(const double* __restrict__ F, const double* __restrict__ ni,
                                                          const double* __restrict__ E, const double* __restrict__ DxT,
                                                          const double* __restrict__ D2T,
                                                          const double* __restrict__ kiw,
                                                          const double* __restrict__ n0_of,
                                                          const int* __restrict__ x_off, const int* __restrict__ nx_of,
                                                          const size_t* __restrict__ m_off, double* __restrict__ M,
                                                          double* __restrict__ b, double dt, int n) {
  const int d = blockIdx.y, N = nx_of[d], x0 = x_off[d];
  const int cb = blockIdx.x * kIonFormCols;
  if (cb >= N) return;
  const int ce = min(N, cb + kIonFormCols);
  const double n0 = n0_of[d], mu = kIonN0Mu / n0, D = kIonN0D / n0;
  const double* dx = DxT + m_off[d];   // column-major: dx[c * N + r] = (D_x)_{rc}
  const double* d2 = D2T + m_off[d];
  double* A = M + m_off[d];
  const double e0 = E[x0], eL = E[x0 + N - 1];
  for (int e = threadIdx.x; e < (ce - cb) * N; e += blockDim.x) {
    const int c = cb + e / N, r = e % N;
    const size_t o = (size_t)c * N + r;
    double v;
    if (r == 0) {
      v = D * dx[o] + (c == 0 ? -mu * e0 - fmax(0.0, -mu * e0) : 0.0);
    } else if (r == N - 1) {
      v = -D * dx[o] + (c == N - 1 ? mu * eL - fmax(0.0, mu * eL) : 0.0);
    } else {
      v = (r == c ? 1.0 / dt : 0.0) + dx[o] * (mu * E[x0 + c]) - D * d2[o];
    }
    A[o] = v;
  }
  // right-hand sides: one wavefront per point
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int j = cb + w; j < ce; j += nw) {
    const double* f = F + (size_t)(x0 + j) * n;
    double s = 0.0;
    for (int c = lane; c < n; c += 64) s += kiw[c] * f[c];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) b[x0 + j] = (j == 0 || j == N - 1) ? 0.0 : ni[x0 + j] / dt + n0 * s;
  }
}

// ---------------------------------------------------------------------------
// Gaussian elimination with partial pivoting (max |a|, ties to the lowest row)
// on [M | b] of one discharge in one block, 16 columns at a time.  The block is
// bound by its chain of N pivot steps, so these run on rows held in registers
// (NF wavefronts, RPT rows per lane; 0.3 to 0.5 us a step in one wavefront, 0.8
// to 1.2 across several), and rows are not moved: a pivot row stays where it is and is
// found by its step (s_row).  Per group: the columns to the rows' lanes and the
// pivot steps; then, CW columns at a time, the new pivot rows' entries of the
// columns to the right and of b, U12 = L11^-1 of them (a thread per
// column, stored in place), and the rank-16 update of the rest by MFMA.  Back substitution by the same blocks of 16.
// The last group is filled up with columns of the identity, whose rows are
// lanes without memory.
// Measured, one discharge: Nx = 200 911 -> 397 us, per group 8 us of pivot steps
// and 9 us of updates (MFMA-bound in one CU: 4.3 us).  Ion steps with the field
// and the formation: Nx = 16 77 -> 27 us, 100 485 -> 129, 512 4990 -> 2780, 1024 30 ->
// 18 ms (before: panels of 16 or 8 columns factored in LDS by all threads, four
// barriers a step).
// ---------------------------------------------------------------------------
constexpr int kIonSolveThreads = 512;
template <int RPT, int NF>
__global__ __launch_bounds__(kIonSolveThreads) void k_ion_solve(double* __restrict__ M, double* __restrict__ b,
                                                                double* __restrict__ out,
                                                                const int* __restrict__ x_off,
                                                                const int* __restrict__ nx_of,
                                                                const size_t* __restrict__ m_off,
                                                                int* __restrict__ status, double dt) {
  constexpr int NT = kIonSolveThreads, NW = NT / 64, R = 64 * RPT * NF, CW = R > 512 ? 128 : 256;
  constexpr int BF = 4;   // update tiles a wavefront has on their way
  const int d = blockIdx.x, N = nx_of[d], x0 = x_off[d];
  double* A = M + m_off[d];
  double* r = b + x0;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  __shared__ __align__(16) double sP[SW][R + 2];    // multipliers, negated (0: retired rows)
  __shared__ __align__(16) double sU[SW][CW + 16];
  __shared__ __align__(16) double sL11[SW][SW];
  __shared__ __align__(16) PivotLds<NF> s_pl;
  __shared__ int s_piv[R + SW];
  __shared__ short s_row[R + SW];                   // the row of every pivot step
  __shared__ bool s_act[R];                         // rows of the system not yet chosen as a pivot
  bool singular = false, nonfinite = false;
  // equilibration of the two wall rows (wavefront 0: row 0, wavefront 1: row
  // N-1) to the size of the interior rows; their right-hand sides are 0
  if (w < 2) {
    const int rr = (w == 0) ? 0 : N - 1;
    double m = 0.0;
    for (int c = lane; c < N; c += 64) m = fmax(m, fabs(A[(size_t)c * N + rr]));
    m = wave_max(m);
    const double sc = (m > 0.0) ? 1.0 / (dt * m) : 1.0;
    for (int c = lane; c < N; c += 64) A[(size_t)c * N + rr] *= sc;
  }
  Rows<RPT> x;
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    x.pos[q] = tid + 64 * NF * q;
    x.act[q] = x.pos[q] < (N + SW - 1) / SW * SW ? ~0u : 0u;
  }
  __syncthreads();
  for (int k0 = 0; k0 < N; k0 += SW) {
    if (w < NF) {
      // (loads without branches, from entries of the system)
      UniformCols<double> cols(A + (size_t)k0 * N, N);
#pragma unroll
      for (int j = 0; j < SW; ++j) {
        const double* p = cols.next();
        if (k0 + j >= N) p = A;
#pragma unroll
        for (int q = 0; q < RPT; ++q) x.a[q][j] = p[static_cast<unsigned>(min(tid + 64 * NF * q, N - 1))];
      }
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const int row = tid + 64 * NF * q;
        const bool in = row < N;
#pragma unroll
        for (int j = 0; j < SW; ++j) {
          const int c = k0 + j;
          x.a[q][j] = (in & (c < N)) ? x.a[q][j] : (row == c ? 1.0 : 0.0);
        }
      }
      pivot_steps<RPT, NF>(x, k0, &s_pl, s_piv, singular, nonfinite);
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const int row = tid + 64 * NF * q, st = x.pos[q] - k0;
        const bool act = x.act[q] != 0u;
#pragma unroll
        for (int j = 0; j < SW; ++j) sP[j][row] = act ? -x.a[q][j] : 0.0;
        s_act[row] = act & (row < N);
        if (!act & (st >= 0) & (st < SW)) {   // (rows without a place in the system lie past the last step)
          s_row[k0 + st] = static_cast<short>(row);
          double* p = A + (size_t)k0 * N + row;
#pragma unroll
          for (int j = 0; j < SW; ++j) {
            sL11[j][st] = x.a[q][j];   // entries k < st are read
            if (k0 + j < N && row < N) *p = x.a[q][j];
            p += N;
          }
        }
      }
    } else if constexpr (NF > 1) {
      for (int j = 0; j < SW; ++j) lds_barrier();   // the steps' barriers
    }
    lds_barrier();
    // the columns to the right, then b
    const int c1 = k0 + SW, nc = max(0, N - c1) + 1;
    auto col = [&](int q) { return c1 + q < N ? A + (size_t)(c1 + q) * N : r; };
    for (int q0 = 0; q0 < nc; q0 += CW) {
      const int qn = min(CW, nc - q0);
      if (tid < CW) {
        double uc[SW];
        int rows[SW];   // (rows without memory: the last, not written)
        double* p = col(q0 + min(tid, qn - 1));
#pragma unroll
        for (int i = 0; i < SW; ++i) {
          rows[i] = s_row[k0 + i];
          const double v = p[min(rows[i], N - 1)];
          uc[i] = ((tid < qn) & (rows[i] < N)) ? v : 0.0;
        }
        unit_lower_16(sL11, uc);
#pragma unroll
        for (int i = 0; i < SW; ++i) {
          sU[i][tid] = uc[i];
          if ((tid < qn) & (rows[i] < N)) p[rows[i]] = uc[i];   // (read again by the back substitution only)
        }
      }
      lds_barrier();
      const int nrt = (N + 15) / 16, tiles = nrt * ((qn + 15) / 16);
      // (the products transposed, rows along the lanes: an item is 4 columns' 16
      // consecutive rows)
      for (int t0 = w; t0 < tiles; t0 += BF * NW) {
        f64x4 acc[BF];
#pragma unroll
        for (int f = 0; f < BF; ++f) {
          const int tile = min(t0 + f * NW, tiles - 1), q = 16 * (tile / nrt) + lk, row = 16 * (tile % nrt) + li;
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[f][i] = col(q0 + min(q + 4 * i, qn - 1))[min(row, N - 1)];
        }
#pragma unroll
        for (int f = 0; f < BF; ++f) {
          const int tile = t0 + f * NW, q = 16 * (tile / nrt), row = 16 * (tile % nrt) + li;
          if (tile >= tiles) break;
#pragma unroll
          for (int k = 0; k < 4; ++k)
            acc[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(sU[4 * k + lk][q + li], sP[4 * k + lk][row], acc[f], 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (q + lk + 4 * i < qn && s_act[row]) col(q0 + q + lk + 4 * i)[row] = acc[f][i];
        }
      }
      __syncthreads();
    }
  }
  // back substitution U x = y by blocks of 16 steps from the last, y in LDS in
  // the steps' order: one wavefront solves a block (values passed by lane
  // reads), then every thread subtracts the block's columns from the rows above
  double* sy = &sP[0][0];
  for (int i = tid; i < N; i += NT) sy[i] = r[s_row[i]];
  __syncthreads();
  for (int k0 = (N - 1) / SW * SW; k0 >= 0; k0 -= SW) {
    const int nb = min(SW, N - k0);
    if (w == 0) {
      const bool own = lane < nb;
      double v = own ? sy[k0 + lane] : 0.0;
      const double* p = A + (size_t)k0 * N + s_row[k0 + min(lane, nb - 1)];
      double u[SW];   // (entries below the diagonal are not read)
#pragma unroll
      for (int t = 0; t < SW; ++t) u[t] = p[(size_t)min(t, nb - 1) * N];
#pragma unroll
      for (int t = SW - 1; t >= 0; --t) {
        if (t < nb) {
          if (lane == t) v = v / u[t];
          const double xt = readlane_f64(v, t);
          if (lane < t) v -= u[t] * xt;
        }
      }
      if (own) sy[k0 + lane] = v;
    }
    __syncthreads();
    for (int i = tid; i < k0; i += NT) {
      const double* p = A + (size_t)k0 * N + s_row[i];
      double t[SW], ri = sy[i];
#pragma unroll
      for (int j = 0; j < SW; ++j) t[j] = p[(size_t)min(j, nb - 1) * N];
#pragma unroll
      for (int j = SW - 1; j >= 0; --j)
        if (j < nb) ri -= t[j] * sy[k0 + j];
      sy[i] = ri;
    }
    __syncthreads();
  }
  for (int i = tid; i < N; i += NT) out[x0 + i] = sy[i];
  if (singular && tid == 0) atomicOr(status, kStSingular);
  if (nonfinite && tid == 0) atomicOr(status, kStNonFinite);
}

}  // namespace

void launch_ion_update_ws(const DevOps& d, const double* F, const double* ni_in, double* ni_out, double* M, double* b,
                          const double* E, hipStream_t s) {
  const dim3 gf((d.max_nx + kIonFormCols - 1) / kIonFormCols, d.nd);
  k_ion_form<<<gf, kIonThreads, 0, s>>>(F, ni_in, E, d.dxT, d.dx2, d.mom + 2 * (size_t)d.n, d.n0_of, d.x_off,
                                        d.nx_of, d.p_off, M, b, d.dt, d.n);
  auto solve = [&](auto rpt, auto nf) {
    k_ion_solve<decltype(rpt)::value, decltype(nf)::value><<<d.nd, kIonSolveThreads, 0, s>>>(
        M, b, ni_out, d.x_off, d.nx_of, d.p_off, d.status, d.dt);
  };
  using std::integral_constant;
  // the fewest wavefronts that hold the rows of the largest discharge: a step of
  // 16 columns takes 4.9 us with two rows per lane of one wavefront, 7.9 with four
  // (13 with one row per lane of four wavefronts, at 256 rows); at 512 rows 12.5 with
  // two per lane of four, 16 with four per lane of two
  if (d.max_nx <= 128) solve(integral_constant<int, 2>(), integral_constant<int, 1>());
  else if (d.max_nx <= 256) solve(integral_constant<int, 4>(), integral_constant<int, 1>());
  else if (d.max_nx <= 512) solve(integral_constant<int, 2>(), integral_constant<int, 4>());
  else solve(integral_constant<int, 2>(), integral_constant<int, 8>());   // (Nx <= 1024)
}

void launch_ion_update(const DevOps& d, const double* F, const double* ni_in, double* ni_out, hipStream_t s) {
  launch_ion_update_ws(d, F, ni_in, ni_out, d.ion_M, d.ion_b, d.ion_E, s);
}

// Scratch of the allocation-free ion step: one copy per GPU, alive until the
// process ends.  Host code never uses the array's name as an address; it takes
// the device address that hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) double scratch[kIonScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t ion_scratch(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    double* p = nullptr;
    e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace bte
