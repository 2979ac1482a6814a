// FP64 panel factorization of the batched LU (partial pivoting: max |a|, ties
// to the lowest row).  A panel is a chain of 128 dependent pivot steps, one
// matrix per block, so its time is the latency of a step plus every trip to
// memory between steps.  Rows are never moved while columns are factored:
// each row keeps the position it would have after the interchanges so far, a
// chosen pivot row retires with its step, and the rows go to their positions
// once, on the way out.
//   k_panel_reg   panels of at most 256 rows: the whole panel stays in the
//                 block's MFMA accumulators (256 x 128 doubles, half of the
//                 CU's registers), 16 columns at a time pass through LDS to
//                 one thread per row for their pivot steps, and the columns to
//                 their right take one rank-16 MFMA update.  Memory is touched
//                 at load and store only.
//   k_panel_tall  taller panels: 16 columns per launch, up to four rows per
//                 thread in registers; the interchanges and the U rows of the
//                 panel's other columns follow in the same launch, and
//   k_panel_upd   the rank-16 update of the columns to the right, over many
//                 blocks per matrix.
// All of them also write the inverses of L11's 16 x 16 diagonal blocks, which
// the formation of L11^-1 starts from.
// (The tall panels of many matrices, which these passes over memory would bind,
// go to the left-looking kernel: the rule is at the factorization's dispatch.)
// Measured per panel, 64 matrices, against the former kernel (one block per
// matrix, 8 or 16 columns in registers, the rest of the panel re-read from
// memory between them; it did not get faster with fewer rows): 128 rows 72 us
// (266), 256 rows 129 us (284), 512 rows 215 us (298), 640 to 1024 rows 290 us
// (409), 1152 to 2048 rows 450 us (600).  A step costs 680 cycles in one
// wavefront and 1.3k to 2k across wavefronts (two LDS trips and a barrier).
#include "internal.h"
#include "lu_common.h"
#include "pivot_steps.h"

namespace bte {
namespace {

constexpr int NB = kNB;
constexpr int kUPitch = NB + 16;   // row pitch of the staged U rows (operand reads of two rows on different banks)

// ---------------------------------------------------------------------------
// Panels of R = 128 RT rows (RT = 2 or 1), one 512-thread block per matrix.
// Wavefront w holds rows 16 RT w + 16 rt + 4 lk + t (row tile rt, item t of the
// accumulator, lane group lk) of column 16 ct + li: the MFMA's result row
// lk + 4 t is free to name any row, and this choice lets a lane load and store
// four consecutive rows.  The accumulators rotate by one column tile per group
// of 16 columns, so that the loop body is compiled once (unrolled over the
// eight groups it would not fit the instruction cache).
// Per group: the group's tile through LDS to the rows' lanes for the 16 pivot
// steps (128 rows: two per lane of wavefront 0, which needs no barrier; 256
// rows: one per lane of four wavefronts, 1.2k cycles per step otherwise), and
// back (final values); the 16 new pivot rows' entries to the right through LDS, U12 =
// L11^-1 of them (a thread per column, and the inverse of L11's diagonal block
// as 16 more columns), straight to the matrix, and A22 -= L21 U12 by MFMA with
// zero rows for retired ones.
// ---------------------------------------------------------------------------
template <int RT>
__global__ __launch_bounds__(512) void k_panel_reg(double* __restrict__ LU, double* __restrict__ linv,
                                                   int* __restrict__ piv, int* __restrict__ perm,
                                                   int* __restrict__ status, int npad, int k0) {
  constexpr int NT = 512, R = 128 * RT, NCT = NB / SW, LP = R + 2;
  constexpr int RPT = RT == 1 ? 2 : 1, NF = R / 64 / RPT;   // rows per lane of the pivot steps, their wavefronts
  const int mat = blockIdx.x;
  double* A = LU + (size_t)mat * npad * npad + (size_t)k0 * npad + k0;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  __shared__ __align__(16) double sP[SW][LP];
  __shared__ __align__(16) double sU[SW][kUPitch];   // columns to the right, then the identity
  __shared__ __align__(16) double sL11[SW][SW];
  __shared__ __align__(16) PivotLds<NF> s_pl;
  __shared__ __align__(16) int s_step[R];   // step of this group, -1 active, -2 retired earlier; positions at the end
  __shared__ int s_piv[NB];
  __shared__ int s_cnt;
  bool singular = false, nonfinite = false;
  f64x4 acc[RT][NCT];
  const int rw = 16 * RT * w;
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const double* p = A + (size_t)(SW * ct + li) * npad + rw + 16 * rt + 4 * lk;
      const f64x2 lo = *reinterpret_cast<const f64x2*>(p), hi = *reinterpret_cast<const f64x2*>(p + 2);
      acc[rt][ct] = f64x4{lo[0], lo[1], hi[0], hi[1]};
    }
  if (tid < SW * SW) sU[tid / SW][NB - SW + tid % SW] = tid / SW == tid % SW ? 1.0 : 0.0;
  Rows<RPT> x;
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    x.pos[q] = tid + 64 * q;
    x.act[q] = ~0u;
  }
  double* dinv = linv + (size_t)mat * kLinvElems;
  for (int sp = 0; sp < NCT; ++sp) {
    const int c0 = SW * sp, nrem = NCT - 1 - sp;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      double* p = &sP[li][rw + 16 * rt + 4 * lk];
      *reinterpret_cast<f64x2*>(p) = f64x2{acc[rt][0][0], acc[rt][0][1]};
      *reinterpret_cast<f64x2*>(p + 2) = f64x2{acc[rt][0][2], acc[rt][0][3]};
    }
    lds_barrier();
    if (w < NF) {
#pragma unroll
      for (int q = 0; q < RPT; ++q)
#pragma unroll
        for (int j = 0; j < SW; ++j) x.a[q][j] = sP[j][tid + 64 * q];
      pivot_steps<RPT, NF>(x, c0, &s_pl, s_piv, singular, nonfinite);
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const int r = tid + 64 * q;
        const int st = x.act[q] ? -1 : (x.pos[q] < c0 ? -2 : x.pos[q] - c0);
        s_step[r] = st;
#pragma unroll
        for (int j = 0; j < SW; ++j) sP[j][r] = x.a[q][j];
        if (st >= 0) {
#pragma unroll
          for (int j = 0; j < SW; ++j) sL11[j][st] = x.a[q][j];   // entries k < st are read
        }
      }
    } else if constexpr (NF > 1) {
      for (int j = 0; j < SW; ++j) lds_barrier();   // the steps' barriers
    }
    // (the first group's U rows go to the matrix where other wavefronts' first loads come from)
    if (sp == 0) loads_barrier();
    else lds_barrier();
    // final values of the group's columns; L21 operands, zero for retired rows;
    // the new pivot rows' entries to the right
    double av[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const double* p = &sP[li][rw + 16 * rt + 4 * lk];
      const f64x2 lo = *reinterpret_cast<const f64x2*>(p), hi = *reinterpret_cast<const f64x2*>(p + 2);
      acc[rt][0] = f64x4{lo[0], lo[1], hi[0], hi[1]};
      const int ar = rw + 16 * rt + 4 * (li & 3) + (li >> 2);   // the row of MFMA row li
      const bool on = s_step[ar] == -1;
#pragma unroll
      for (int q = 0; q < 4; ++q) av[rt][q] = on ? -sP[4 * q + lk][ar] : 0.0;
      const int4 js = *reinterpret_cast<const int4*>(&s_step[rw + 16 * rt + 4 * lk]);
      const int jt[4] = {js.x, js.y, js.z, js.w};
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (jt[t] >= 0) {
#pragma unroll
          for (int ct = 1; ct < NCT; ++ct) sU[jt[t]][SW * (ct - 1) + li] = acc[rt][ct][t];   // (past nrem: not read)
        }
    }
    lds_barrier();
    if ((tid < SW * nrem) | ((tid >= NB - SW) & (tid < NB))) {
      double u[SW];
#pragma unroll
      for (int i = 0; i < SW; ++i) u[i] = sU[i][tid];
      unit_lower_16(sL11, u);
      if (tid < SW * nrem) {
        f64x2* o = reinterpret_cast<f64x2*>(A + (size_t)(c0 + SW + tid) * npad + c0);
#pragma unroll
        for (int i = 0; i < SW; ++i) sU[i][tid] = u[i];
#pragma unroll
        for (int i = 0; i < SW / 2; ++i) o[i] = f64x2{u[2 * i], u[2 * i + 1]};
      } else {
#pragma unroll
        for (int i = 0; i < SW; ++i) dinv[sp * 256 + i * SW + tid - (NB - SW)] = u[i];
      }
    }
    lds_barrier();
#pragma unroll
    for (int ct = 1; ct < NCT; ++ct) {
      if (ct <= nrem) {
        double b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = sU[4 * q + lk][SW * (ct - 1) + li];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) acc[rt][ct] = Mma<double>::step(av[rt][q], b[q], acc[rt][ct]);
      }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const f64x4 f = acc[rt][0];
#pragma unroll
      for (int ct = 0; ct + 1 < NCT; ++ct) acc[rt][ct] = acc[rt][ct + 1];
      acc[rt][NCT - 1] = f;
    }
  }
  // out: every row at its position, 16 columns at a time through LDS (above a
  // column tile's own rows: the U rows, which are out already)
  if (tid == 0) s_cnt = 0;
  if (w < NF) {
#pragma unroll
    for (int q = 0; q < RPT; ++q) s_step[tid + 64 * q] = x.pos[q];
  }
  lds_barrier();
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int4 pt = *reinterpret_cast<const int4*>(&s_step[rw + 16 * rt + 4 * lk]);
      sP[li][pt.x] = acc[rt][ct][0];
      sP[li][pt.y] = acc[rt][ct][1];
      sP[li][pt.z] = acc[rt][ct][2];
      sP[li][pt.w] = acc[rt][ct][3];
    }
    lds_barrier();
#pragma unroll
    for (int e = tid; e < SW * R / 2; e += NT) {
      const int j = e / (R / 2), r = e % (R / 2) * 2;
      if (r >= SW * ct)
        *reinterpret_cast<f64x2*>(A + (size_t)(SW * ct + j) * npad + r) = *reinterpret_cast<const f64x2*>(&sP[j][r]);
    }
    lds_barrier();
  }
  // pivots, and the panel's permutation: its own rows first, then the displaced rows below
  if (tid < NB) piv[(size_t)mat * npad + k0 + tid] = k0 + s_piv[tid];
  int* pm = perm + ((size_t)mat * kMaxPanels + k0 / NB) * kPermStride;
  if (tid < R) {
    const int po = s_step[tid];
    if (po < NB) {
      pm[1 + po] = k0 + po;
      pm[1 + kMaxSwapRows + po] = k0 + tid;
    } else if (po != tid) {
      const int t = NB + atomicAdd(&s_cnt, 1);
      pm[1 + t] = k0 + po;
      pm[1 + kMaxSwapRows + t] = k0 + tid;
    }
  }
  if (singular && tid == 0) atomicOr(status, kStSingular);
  if (nonfinite && tid == 0) atomicOr(status, kStNonFinite);
  lds_barrier();
  if (tid == 0) pm[0] = NB + s_cnt;
}

// ---------------------------------------------------------------------------
// Columns c0 .. c0 + 15 (relative to the panel) of a panel of R rows, one
// 512-thread block per matrix, rows c0 .. R - 1 in registers (RPT per thread).
// row_of[r] (device scratch, R per matrix): the row of the unpermuted panel at
// position r, carried from group to group.  After the steps the rows of the
// panel's other columns are interchanged (gather, then scatter), the columns
// to the right take U = L11^-1 of the new pivot rows, and the last group
// writes the panel's permutation.
// ---------------------------------------------------------------------------
template <int RPT, int NW>
__global__ __launch_bounds__(64 * NW) void k_panel_tall(double* __restrict__ LU, double* __restrict__ linv,
                                                    int* __restrict__ piv, int* __restrict__ perm,
                                                    int* __restrict__ row_of, size_t row_of_stride,
                                                    int* __restrict__ status, int npad, int k0, int R, int c0) {
  constexpr int NT = 64 * NW;
  const int mat = blockIdx.x;
  double* A = LU + (size_t)mat * npad * npad + (size_t)k0 * npad + k0;
  int* ro = row_of + (size_t)mat * row_of_stride;
  const int tid = threadIdx.x;
  __shared__ __align__(16) PivotLds<NW> s;
  __shared__ __align__(16) double sL11[SW][SW];
  __shared__ double sX[SW][kUPitch];   // pivot rows of the columns to the right, then the identity
  __shared__ int s_piv[NB];
  __shared__ int s_src[2 * SW], s_dst[2 * SW];
  __shared__ int s_cnt;
  bool singular = false, nonfinite = false;
  Rows<RPT> x;
  int org[RPT];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const unsigned r = c0 + tid + q * NT;
    const bool in = r < static_cast<unsigned>(R);
    x.pos[q] = in ? r : -1;
    x.act[q] = in ? ~0u : 0u;
#pragma unroll
    for (int j = 0; j < SW; ++j) {
      const double* col = A + (size_t)(c0 + j) * npad;
      x.a[q][j] = in ? col[r] : 0.0;
    }
    org[q] = c0 == 0 ? r : (in ? ro[r] : 0);
  }
  if (tid == 0) s_cnt = SW;
  if (tid < SW * SW) sX[tid / SW][NB - SW + tid % SW] = tid / SW == tid % SW ? 1.0 : 0.0;
  pivot_steps<RPT, NW>(x, c0, &s, s_piv, singular, nonfinite);
  loads_barrier();   // the rows and ro go out below at positions that other wavefronts hold
  const bool last = c0 + SW == NB;
  int* pm = perm + ((size_t)mat * kMaxPanels + k0 / NB) * kPermStride;
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = c0 + tid + q * NT, po = x.pos[q];
    if (r >= R) continue;
#pragma unroll
    for (int j = 0; j < SW; ++j) {
      double* col = A + (size_t)(c0 + j) * npad;
      col[static_cast<unsigned>(po)] = x.a[q][j];
    }
    ro[po] = org[q];
    if (po < c0 + SW) {
      s_src[po - c0] = r;
      s_dst[po - c0] = po;
#pragma unroll
      for (int j = 0; j < SW; ++j) sL11[j][po - c0] = x.a[q][j];
    } else if (po != r) {
      const int t = atomicAdd(&s_cnt, 1);
      s_src[t] = r;
      s_dst[t] = po;
    }
  }
  lds_barrier();
  if (tid < SW) piv[(size_t)mat * npad + k0 + c0 + tid] = k0 + s_piv[c0 + tid];
  // the panel's other columns: all reads, then all writes; the pivot rows of
  // the columns to the right go to LDS for U
  {
    const int nT = s_cnt;
    constexpr int NOC = NB - SW, NV = (NOC * 2 * SW + NT - 1) / NT;
    double v[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = tid + u * NT, t = e % nT, cc = e / nT;
      const int col = cc < c0 ? cc : cc + SW;
      if (e < NOC * nT && (cc >= c0 || s_src[t] != s_dst[t])) v[u] = A[(size_t)col * npad + s_src[t]];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = tid + u * NT, t = e % nT, cc = e / nT;
      const int col = cc < c0 ? cc : cc + SW;
      if (e < NOC * nT) {
        if (cc >= c0 && t < SW) sX[t][cc - c0] = v[u];
        else if (s_src[t] != s_dst[t]) A[(size_t)col * npad + s_dst[t]] = v[u];
      }
    }
  }
  lds_barrier();
  const int nright = NB - SW - c0;
  if ((tid < nright) | ((tid >= NB - SW) & (tid < NB))) {
    double u[SW];
#pragma unroll
    for (int i = 0; i < SW; ++i) u[i] = sX[i][tid];
    unit_lower_16(sL11, u);
    if (tid < nright) {
      double* o = A + (size_t)(c0 + SW + tid) * npad + c0;
#pragma unroll
      for (int i = 0; i < SW; ++i) o[i] = u[i];
    } else {
      double* o = linv + (size_t)mat * kLinvElems + (c0 / SW) * 256 + tid - (NB - SW);
#pragma unroll
      for (int i = 0; i < SW; ++i) o[i * SW] = u[i];
    }
  }
  if (singular && tid == 0) atomicOr(status, kStSingular);
  if (nonfinite && tid == 0) atomicOr(status, kStNonFinite);
  if (!last) return;
  // the panel's permutation: its own rows, then the displaced rows below
  __syncthreads();
  if (tid == 0) s_cnt = NB;
  lds_barrier();
  if (tid < c0) {   // rows retired by the earlier groups
    pm[1 + tid] = k0 + tid;
    pm[1 + kMaxSwapRows + tid] = k0 + ro[tid];
  }
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = c0 + tid + q * NT, po = x.pos[q];
    if (r >= R) continue;
    int t = po;
    if (po >= NB) {
      if (po == org[q]) continue;
      t = atomicAdd(&s_cnt, 1);
    }
    pm[1 + t] = k0 + po;
    pm[1 + kMaxSwapRows + t] = k0 + org[q];
  }
  lds_barrier();
  if (tid == 0) pm[0] = s_cnt;
}

// ---------------------------------------------------------------------------
// Rank-16 update of the panel's columns c0 + 16 .. 127 below the group at c0:
// A[r][c] -= sum_k L[r][c0 + k] U[c0 + k][c], 128 rows per block (32 per
// wavefront), straight from and to memory in the lane layout of k_panel_reg.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_panel_upd(double* __restrict__ LU, int npad, int k0, int R, int c0, int nrt,
                                                   int nmat) {
  int mat, tile;
  xcd_map(blockIdx.x, nrt, nmat, &mat, &tile);
  if (mat >= nmat) return;
  double* A = LU + (size_t)mat * npad * npad + (size_t)k0 * npad + k0;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  constexpr int MT = NB / SW - 1;
  const int rem = NB / SW - 1 - c0 / SW;   // 16-column tiles to the right
  const int r0 = c0 + SW + tile * 128 + 32 * w;   // R - c0 is a multiple of 16
  double av[2][4];
  bool on[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    on[rt] = r0 + 16 * rt < R;
    const int ar = r0 + 16 * rt + 4 * (li & 3) + (li >> 2);
#pragma unroll
    for (int q = 0; q < 4; ++q) av[rt][q] = on[rt] ? -A[(size_t)(c0 + 4 * q + lk) * npad + ar] : 0.0;
  }
  if (!on[0]) return;
  f64x4 acc[2][MT];
  double b[MT][4];
#pragma unroll
  for (int ct = 0; ct < MT; ++ct) {
    if (ct >= rem) break;
    const double* col = A + (size_t)(c0 + SW + SW * ct + li) * npad;
#pragma unroll
    for (int q = 0; q < 4; ++q) b[ct][q] = col[c0 + 4 * q + lk];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      if (!on[rt]) continue;
      const f64x2 lo = *reinterpret_cast<const f64x2*>(col + r0 + 16 * rt + 4 * lk);
      const f64x2 hi = *reinterpret_cast<const f64x2*>(col + r0 + 16 * rt + 4 * lk + 2);
      acc[rt][ct] = f64x4{lo[0], lo[1], hi[0], hi[1]};
    }
  }
#pragma unroll
  for (int ct = 0; ct < MT; ++ct) {
    if (ct >= rem) break;
    double* col = A + (size_t)(c0 + SW + SW * ct + li) * npad;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      if (!on[rt]) continue;
      f64x4 d = acc[rt][ct];
#pragma unroll
      for (int q = 0; q < 4; ++q) d = Mma<double>::step(av[rt][q], b[ct][q], d);
      *reinterpret_cast<f64x2*>(col + r0 + 16 * rt + 4 * lk) = f64x2{d[0], d[1]};
      *reinterpret_cast<f64x2*>(col + r0 + 16 * rt + 4 * lk + 2) = f64x2{d[2], d[3]};
    }
  }
}

}  // namespace

void launch_panel_f64(double* LU, double* linv, void* xscr, int* piv, int* perm, int* status, int npad, int k0,
                      int rend, int nmat, hipStream_t s) {
  const int R = rend - k0;
  if (R <= 128) {
    k_panel_reg<1><<<nmat, 512, 0, s>>>(LU, linv, piv, perm, status, npad, k0);
    return;
  }
  if (R <= 256) {
    k_panel_reg<2><<<nmat, 512, 0, s>>>(LU, linv, piv, perm, status, npad, k0);
    return;
  }
  int* ro = static_cast<int*>(xscr);   // free until the panel's U12
  const size_t stride = (size_t)npad * NB * (sizeof(double) / sizeof(int));
  for (int c0 = 0; c0 < NB; c0 += SW) {
    if (R <= 512) k_panel_tall<2, 4><<<nmat, 256, 0, s>>>(LU, linv, piv, perm, ro, stride, status, npad, k0, R, c0);
    else if (R <= 1024) k_panel_tall<2, 8><<<nmat, 512, 0, s>>>(LU, linv, piv, perm, ro, stride, status, npad, k0, R, c0);
    else k_panel_tall<4, 8><<<nmat, 512, 0, s>>>(LU, linv, piv, perm, ro, stride, status, npad, k0, R, c0);
    if (c0 + SW < NB) {
      const int nrt = (R - c0 - SW + 127) / 128;
      k_panel_upd<<<xcd_grid(nrt, nmat), 256, 0, s>>>(LU, npad, k0, R, c0, nrt, nmat);
    }
  }
}

}  // namespace bte
