// FP64 products of rows by operators on MFMA, shared by the residuals, the
// adjoint gradients and the Hessenberg form's basis changes.
#pragma once

#include "lu_common.h"

namespace bte {
namespace {

// 16 bytes at any double address
using V2u = double __attribute__((ext_vector_type(2), aligned(8)));

// Result row of item t of lane group lk for MFMA f64 16x16x4 (measured layout).
__device__ inline int f64_row(int lk, int t) { return lk + 4 * t; }

// s_part[w][q] = this wavefront's part of the tile X[x0 ..][.] M_q^T[.][i0 ..]
// (TRANSPOSE: M_q) for the operators q: 16 PT rows of X (ld doubles apart) x 16 OT
// outputs, the sum over k shared by the block's NW wavefronts (each takes every
// NW-th chunk of 16), operands straight from memory in 16-byte vectors.  M's
// rows are ldm doubles apart (ldm > n for an odd n, whose last vector reaches past it).
template <int TRANSPOSE, int NOP, int PT, int OT, int NW>
__device__ __forceinline__ void tile_products(const double* __restrict__ Xv, int ld, const double* const (&M)[NOP],
                                              int ldm, int n, int nx, int x0, int i0,
                                              double (&s_part)[NW][NOP][16 * PT][16 * OT]) {
  constexpr int CK = 16, DEPTH = 2;   // chunks in registers: one in use, one on its way
  using V2 = double __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  // operand rows of this lane (rows beyond the last repeat it; their results are dropped)
  const double* xp[PT];
  const double* op[NOP][OT];
#pragma unroll
  for (int p = 0; p < PT; ++p) xp[p] = Xv + (size_t)min(x0 + p * 16 + li, nx - 1) * ld;
#pragma unroll
  for (int o = 0; o < OT; ++o) {
    const size_t i = min(i0 + o * 16 + li, n - 1);
#pragma unroll
    for (int q = 0; q < NOP; ++q) op[q][o] = M[q] + (TRANSPOSE ? i : i * ldm);
  }
  const int nch = (n + CK - 1) / CK, cnt = (nch - w + NW - 1) / NW;
  struct Chunk {
    V2 x[PT][2], m[NOP][OT][2];
  } buf[DEPTH];
  // k of a lane's vector j: 8 j + 2 lk, + 1 within the chunk
  auto load = [&](Chunk& c, int it) {
    const int kc = CK * (w + NW * min(it, cnt - 1)) + 2 * lk;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int k = min(kc + 8 * j, n + (n & 1) - 2);
#pragma unroll
      for (int p = 0; p < PT; ++p) c.x[p][j] = *reinterpret_cast<const V2u*>(xp[p] + k);
#pragma unroll
      for (int q = 0; q < NOP; ++q)
#pragma unroll
        for (int o = 0; o < OT; ++o) {
          if constexpr (TRANSPOSE) c.m[q][o][j] = V2{op[q][o][(size_t)k * ldm], op[q][o][(size_t)(k + 1) * ldm]};
          else c.m[q][o][j] = *reinterpret_cast<const V2*>(op[q][o] + k);
        }
    }
  };
  f64x4 acc[NOP][PT][OT];
#pragma unroll
  for (int q = 0; q < NOP; ++q)
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
      for (int o = 0; o < OT; ++o) acc[q][p][o] = f64x4{0, 0, 0, 0};
  auto product = [&](Chunk& c, int it) {
    if (CK * (w + NW * it) + CK > n) {   // the last chunk of an n that 16 does not divide
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int k = CK * (w + NW * it) + 2 * lk + 8 * j;
#pragma unroll
        for (int p = 0; p < PT; ++p) c.x[p][j] = V2{k < n ? c.x[p][j][0] : 0.0, k + 1 < n ? c.x[p][j][1] : 0.0};
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < NOP; ++q)
#pragma unroll
          for (int p = 0; p < PT; ++p)
#pragma unroll
            for (int o = 0; o < OT; ++o)
              acc[q][p][o] = __builtin_amdgcn_mfma_f64_16x16x4f64(c.x[p][j][e], c.m[q][o][j][e], acc[q][p][o], 0, 0, 0);
  };
  if (cnt > 0) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(buf[d], d);
    for (int it = 0; it < cnt; it += DEPTH)
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (it + d < cnt) product(buf[d], it + d);
        load(buf[d], it + d + DEPTH);
      }
  }
#pragma unroll
  for (int q = 0; q < NOP; ++q)
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
      for (int o = 0; o < OT; ++o)
#pragma unroll
        for (int t = 0; t < 4; ++t) s_part[w][q][p * 16 + f64_row(lk, t)][o * 16 + li] = acc[q][p][o][t];
  __syncthreads();
}

}  // namespace
}  // namespace bte
