// The 16 dependent pivot steps of a group of columns (partial pivoting: max |a|,
// ties to the lowest row), shared by the FP64 panels and the ion system's
// elimination.  Rows are held in registers, one or two per lane, and are never
// moved: each keeps the position it would have after the interchanges so far.
#pragma once

#include <cfloat>
#include <climits>
#include <cmath>

#include "lu_common.h"

namespace bte {
namespace {

constexpr int SW = 16;   // columns per pivot-step group

// maximum over the wavefront of 32-bit unsigned keys; uniform result
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
  v = dpp_max<0x140>(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(v))));
  const unsigned r0 = __builtin_amdgcn_readlane(static_cast<int>(v), 0), r1 = __builtin_amdgcn_readlane(static_cast<int>(v), 16);
  const unsigned r2 = __builtin_amdgcn_readlane(static_cast<int>(v), 32), r3 = __builtin_amdgcn_readlane(static_cast<int>(v), 48);
  return max(max(r0, r1), max(r2, r3));
}

// Rows of a panel held RPT per thread: a[q][.] the row's 16 entries of the
// current group, pos[q] its position after the interchanges so far (-1: no
// row), act[q] all ones until the row is chosen as a pivot.
template <int RPT>
struct Rows {
  double a[RPT][SW];
  int pos[RPT];
  unsigned act[RPT];
};

// What the wavefronts publish for one pivot step (two copies, by step parity:
// a copy is written again two steps later, past the barrier of the step between).
template <int NW>
struct PivotLds {
  double cand[2][NW][SW];   // the wavefront's candidate row
  int2 kp[2][NW];           // its key and position
};

// The 16 pivot steps of the columns at position c0 (relative to the panel).
// s_piv[c]: the position that step c interchanges with position c.  A step is a
// chain of latencies and, with one wavefront per SIMD, of issue slots, so it is
// kept short: a candidate's key is the high word of |a| (its bits order like
// the values; a NaN is larger than all and is reported as the pivot), the
// wavefront's maximum takes four DPP steps, and only where several rows share
// the largest key do the full values and the positions decide.  NW = 1: the
// rows of one wavefront, the pivot row passed on by lane reads; else the
// wavefronts' candidates meet in LDS.
template <int RPT, int NW>
__device__ __forceinline__ void pivot_steps(Rows<RPT>& x, int c0, PivotLds<NW>* s, int* s_piv, bool& singular,
                                            bool& nonfinite) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  static_for(std::make_integer_sequence<int, SW>(), [&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    constexpr int par = j & 1;
    const int c = c0 + j;
    unsigned key[RPT], km = 0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      key[q] = ((static_cast<unsigned>(__double2hiint(x.a[q][j])) << 1) | 1u) & x.act[q];
      km = max(km, key[q]);
    }
    km = wave_max_u32(km);
    unsigned long long m[RPT];
    int cnt = 0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      m[q] = __ballot(key[q] == km);
      cnt += __popcll(m[q]);
    }
    if (__builtin_expect(cnt != 1, 0)) {
      // equal keys: the largest |a| (a NaN counts as infinite), then the lowest position
      double v[RPT], vm = -2.0;
      int pm = INT_MAX;
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const double av = fabs(x.a[q][j]);
        v[q] = key[q] == km ? (av == av ? av : HUGE_VAL) : -2.0;
        vm = v[q] > vm ? v[q] : vm;
      }
      vm = wave_max(vm);
#pragma unroll
      for (int q = 0; q < RPT; ++q) pm = v[q] == vm ? min(pm, x.pos[q]) : pm;
      pm = wave_min(pm);
      bool found = false;
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        m[q] = found ? 0 : __ballot((v[q] == vm) & (x.pos[q] == pm));
        m[q] &= -m[q];   // (a wavefront without candidates: one lane all the same)
        found |= m[q] != 0;
      }
    }
    double pr[SW];
    int p;
    if constexpr (NW == 1) {
      p = c;
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        if (m[q]) {
          const int sel = __builtin_ctzll(m[q]);
          p = __builtin_amdgcn_readlane(x.pos[q], sel);
#pragma unroll
          for (int jj = j; jj < SW; ++jj) pr[jj] = readlane_f64(x.a[q][jj], sel);
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        if (m[q]) {
          if (lane == __builtin_ctzll(m[q])) {
            s->kp[par][w] = make_int2(static_cast<int>(key[q]), x.pos[q]);
#pragma unroll
            for (int jj = j; jj < SW; ++jj) s->cand[par][w][jj] = x.a[q][jj];
          }
        }
      }
      lds_barrier();
      // the block's pivot, a wavefront's candidate per lane; all candidate rows
      // come in one read, 16 bytes per lane, and the pivot row is passed on by
      // lane reads (16 entries broadcast to 8 wavefronts would fill the LDS pipe)
      const int2 kp = s->kp[par][lane % NW];
      const f64x2 cr = *reinterpret_cast<const f64x2*>(&s->cand[par][(lane / 8) % NW][2 * (lane % 8)]);
      unsigned kw = static_cast<unsigned>(kp.x);
      if constexpr (NW > 1) kw = dpp_max<0xB1>(kw);
      if constexpr (NW > 2) kw = dpp_max<0x4E>(kw);
      if constexpr (NW > 4) kw = dpp_max<0x141>(kw);
      unsigned long long mw = __ballot(static_cast<unsigned>(kp.x) == kw) & ((1ull << NW) - 1ull);
      if (__builtin_expect(__popcll(mw) != 1, 0)) {
        const double av = fabs(s->cand[par][lane % NW][j]);
        const double v = static_cast<unsigned>(kp.x) == kw ? (av == av ? av : HUGE_VAL) : -2.0;
        const double vm = wave_max(v);
        const int pm = wave_min(v == vm ? kp.y : INT_MAX);
        mw = __ballot((v == vm) & (kp.y == pm));
      }
      const int pw = __builtin_ctzll(mw);
      p = __builtin_amdgcn_readlane(kp.y, pw);
#pragma unroll
      for (int jj = j; jj < SW; ++jj) pr[jj] = readlane_f64(cr[jj & 1], 8 * pw + jj / 2);
    }
    if (tid == 0) s_piv[c] = p;
    // multipliers by the reciprocal of the pivot: the hardware's estimate and
    // two Newton steps, or divisions where those could leave the normal range
    // (as for zero and non-finite pivots)
    const double pv = pr[j];
    const unsigned ex = (static_cast<unsigned>(__builtin_amdgcn_readfirstlane(__double2hiint(pv))) >> 20) & 0x7FFu;
    double rp = __builtin_amdgcn_rcp(pv);
    rp = fma(rp, fma(-pv, rp, 1.0), rp);
    rp = fma(rp, fma(-pv, rp, 1.0), rp);
    double l[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int po = x.pos[q];
      x.pos[q] = po == p ? c : (po == c ? p : po);
      x.act[q] = po == p ? 0u : x.act[q];
      l[q] = x.a[q][j] * rp;
    }
    if (__builtin_expect(ex - 63u >= 1920u, 0)) {
      singular |= pv == 0.0;
      nonfinite |= !(fabs(pv) <= DBL_MAX);
#pragma unroll
      for (int q = 0; q < RPT; ++q) l[q] = pv != 0.0 ? x.a[q][j] / pv : 0.0;
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const bool on = x.act[q] != 0u;
      l[q] = on ? l[q] : 0.0;
      x.a[q][j] = on ? l[q] : x.a[q][j];
#pragma unroll
      for (int jj = j + 1; jj < SW; ++jj) x.a[q][jj] = fma(-l[q], pr[jj], x.a[q][jj]);
    }
  });
}

// x <- L^-1 x for the unit lower 16 x 16 block sL[k][i] = L[i][k]; one column of
// L ahead in registers (all of them would spill)
__device__ __forceinline__ void unit_lower_16(const double (*sL)[SW], double (&x)[SW]) {
  double l[SW], ln[SW];
#pragma unroll
  for (int i = 0; i < SW; ++i) l[i] = sL[0][i];
#pragma unroll
  for (int k = 0; k < SW - 1; ++k) {
#pragma unroll
    for (int i = k + 2; i < SW; ++i) ln[i] = sL[k + 1][i];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = k + 1; i < SW; ++i) x[i] -= l[i] * x[k];
#pragma unroll
    for (int i = k + 2; i < SW; ++i) l[i] = ln[i];
  }
}

}  // namespace
}  // namespace bte
