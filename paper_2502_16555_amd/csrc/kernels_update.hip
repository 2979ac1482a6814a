// Trailing update of the batched LU: A22 -= L21 U12 for every matrix, 128 x 128
// tiles on MFMA (FP64, FP32, or FP32 storage with operands split into 16-bit
// parts).  The tile's
// old values are read and written once (the LDS-staged epilogue), L21 and U12
// are read once per tile; blocks of one matrix stay on one XCD so that its L21
// and U12 come from that XCD's L2.
#include <stdexcept>

#include "internal.h"
#include "lu_common.h"

namespace bte {
namespace {

constexpr int NB = kNB;

// ---------------------------------------------------------------------------
// Trailing update on the 16-bit matrix units, FP32 storage and accumulation:
// the operands are split into a high and a low 16-bit part on their way to LDS
// (hi = round(a), lo = round(a - hi)) and the product takes hi*hi (NT = 1) or
// lo*hi + hi*lo + hi*hi (NT = 3).
//   BF16: the reduced precisions' operands.
//   F16:  the FP32 update.  Each row of L21 and column of U12 is scaled by a
//         power of two that brings its largest entry (rmax, cmax: over the
//         panels applied, kept by the kernels that form L21 and U12) to
//         [2^13, 2^14), where hi + lo keeps 23 bits of every entry down to
//         2^-15 of the largest (below that an absolute 2^-39 of it); the scale
//         is taken back on the way out.  An FP32 operand holds 24 bits whatever
//         its size, so the product is not bounded entry by entry as one on the FP32
//         matrix unit is: random operands graded oppositely along k over six decades
//         or more lose to it (7.6e-7 against 4.0e-7 of the result at six, 7e-5 at
//         eight; 1.1e-7 at five).  With 32 products per rounding of the accumulator instead of 4, it
//         is otherwise the closer one to a 64-bit evaluation: 2.4e-7 against 4.0e-7
//         relative (1.2e-7 against 2.0e-7 of |L||U|, largest) on random operands, K =
//         512; a fourth product, lo*lo, changes neither figure.  In factors of the
//         velocity systems (16 configurations of n = 400 to 2048, both ends of the
//         time step, field and gas) the error of L U, entry by entry against |L||U|,
//         is that of the FP32 unit to three digits: 5.6e-8 to 1.1e-7 in the mean,
//         6.9e-6 at the worst entry; and so it is with collision rates spread over
//         twelve decades of energy bins.
// Operands of MFMA 16x16x32: lane l holds 8 consecutive k of row l%16 (A) and
// of column l%16 (B), k = 8 (l/16) + e; the result has the FP32 16x16x4 layout.
// LDS rows hold a chunk of 32 k, 64 bytes per plane, as four 16-byte units, unit
// u of row r at u ^ f(r), f(r) = -(r / 4) mod 4: the 16 rows of an operand read
// then fall on all 64 banks in each of its phases.
// Tiles of 128 x 128, four wavefronts of 64 x 64.  With 32-bit lane offsets
// beside uniform bases three or four blocks fit on a CU, so that one block's
// loads and read-modify-write run under another's products.  K = 512 on 256
// matrices, 1536 trailing columns, in a loop of its own: 2.07 ms (3.1 TB/s of tile
// and operand bytes; split bf16 1.91) against 4.64 ms on the FP32 matrix unit, which
// is bound by its rate; the L-shaped updates of 1920, 1792 and 1664 rows 335, 414 and
// 489 us, 4.4 TB/s, against 344, 542 and 671.  In the step, behind the kernels that
// write L21 and U12: 2.23 ms, and 325, 424 and 504 us.  The epilogue without LDS
// (16 bytes per lane, 64 per column) took 2.26 ms and 370, 449, 515 us; tiles of 256 x 256
// in one block per CU, with no products under the read-modify-write, 2.6 ms.
// ---------------------------------------------------------------------------
using bf16x8 = __bf16 __attribute__((ext_vector_type(8)));
using f16x8 = _Float16 __attribute__((ext_vector_type(8)));
template <bool F16>
struct Op16;
template <>
struct Op16<true> {
  using E = _Float16;
  using V = f16x8;
  __device__ static inline f32x4 mma(V a, V b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};
template <>
struct Op16<false> {
  using E = __bf16;
  using V = bf16x8;
  __device__ static inline f32x4 mma(V a, V b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};

// exponent (biased) of the power of two that brings m to [2^13, 2^14); the
// inverse power has the exponent 254 minus it
__device__ inline int scale_exp(float m) {
  return min(max(267 - static_cast<int>((__float_as_uint(m) >> 23) & 0xFFu), 2), 252);
}

template <int KD, bool F16, int NT>
__global__ __launch_bounds__(256, 3) void k_update_split(float* __restrict__ LU, const float* __restrict__ rmax,
                                                         const float* __restrict__ cmax, int npad, int k0, int mtr,
                                                         int mtc, int tj0, int nmat, int lrow) {
  using E = typename Op16<F16>::E;
  using V = typename Op16<F16>::V;
  constexpr int KC = 32, NP = NT == 1 ? 1 : 2;
  constexpr int PL = 128 * KC;   // entries of a plane
  int mat, tile;
  xcd_map(blockIdx.x, mtr * mtc + lrow, nmat, &mat, &tile);
  if (mat >= nmat) return;
  // mtr x mtc tiles, then lrow more in the first tile row (columns mtc ..)
  const bool band = tile >= mtr * mtc;
  const int ti = band ? 0 : tile % mtr, tj = band ? mtc + (tile - mtr * mtc) : tile / mtr;
  float* A = LU + (size_t)mat * npad * npad;
  const int r0 = k0 + KD + ti * 128, c0 = k0 + KD + (tj0 + tj) * 128;
  constexpr int RP = 32, LDC = RP + 4;   // the epilogue's passes
  constexpr int OPB = 2 * NP * PL * 2, EPB = 128 * LDC * 4;
  __shared__ __align__(16) unsigned char smem[OPB > EPB ? OPB : EPB];
  E (*sh)[NP][PL] = reinterpret_cast<E (*)[NP][PL]>(smem);   // L21 / U12, plane
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wr = (w >> 1) * 64, wc = (w & 1) * 64;
  auto unit = [](int r, int u) { return (r * 4 + (u ^ ((-(r >> 2)) & 3))) * 8; };
  // staging: thread t takes 16 consecutive k of row t mod 128 of L21 (loads run
  // down the columns), and four k of the columns t / 8 + 32 i of U12 (eight
  // lanes read one column's 128 bytes); offsets in 32 bits beside uniform bases
  const unsigned lrw = tid & 127;
  const int lkh = __builtin_amdgcn_readfirstlane(tid >> 7) * 16;
  const unsigned uc = tid >> 3, uq = tid & 7;
  const unsigned uo = uc * npad + 4 * uq;
  float sl = 1.0f, su[4] = {1.0f, 1.0f, 1.0f, 1.0f};
  const float* rm = rmax + (size_t)mat * npad + r0;
  const float* cm = cmax + (size_t)mat * npad + c0;
  if constexpr (F16) {
    sl = __uint_as_float(scale_exp(rm[lrw]) << 23);
#pragma unroll
    for (int i = 0; i < 4; ++i) su[i] = __uint_as_float(scale_exp(cm[uc + 32 * i]) << 23);
  }
  float ra[16];
  float4 rb[4];
  auto load = [&](int kk) {
    const float* base = A + (size_t)(k0 + kk + lkh) * npad + r0;
#pragma unroll
    for (int k = 0; k < 16; ++k) ra[k] = (base + (size_t)k * npad)[lrw];
    const float* bu = A + (size_t)c0 * npad + k0 + kk;
#pragma unroll
    for (int i = 0; i < 4; ++i) rb[i] = *reinterpret_cast<const float4*>((bu + (size_t)(32 * i) * npad) + uo);
  };
  auto split = [&](float x, float s, E& h, E& l) {
    h = static_cast<E>(x * s);
    if constexpr (NP == 2) l = static_cast<E>(fmaf(x, s, -static_cast<float>(h)));
  };
  auto store = [&]() {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      V h, l;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        E hh, ll;
        split(ra[8 * u + e], sl, hh, ll);
        h[e] = hh;
        if constexpr (NP == 2) l[e] = ll;
      }
      const int o = unit(lrw, lkh / 8 + u);
      *reinterpret_cast<V*>(&sh[0][0][o]) = h;
      if constexpr (NP == 2) *reinterpret_cast<V*>(&sh[0][NP - 1][o]) = l;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      using E4 = E __attribute__((ext_vector_type(4)));
      const float x[4] = {rb[i].x, rb[i].y, rb[i].z, rb[i].w};
      E4 h, l;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        E hh, ll;
        split(x[e], su[i], hh, ll);
        h[e] = hh;
        if constexpr (NP == 2) l[e] = ll;
      }
      const int o = unit(uc + 32 * i, uq >> 1) + 4 * (uq & 1);
      *reinterpret_cast<E4*>(&sh[1][0][o]) = h;
      if constexpr (NP == 2) *reinterpret_cast<E4*>(&sh[1][NP - 1][o]) = l;
    }
  };
  f32x4 acc[4][4];
#pragma unroll
  for (int bi = 0; bi < 4; ++bi)
#pragma unroll
    for (int bj = 0; bj < 4; ++bj) acc[bi][bj] = f32x4{0, 0, 0, 0};
  auto chunk = [&]() __attribute__((always_inline)) {
    V bh[4], bl[4];
#pragma unroll
    for (int bj = 0; bj < 4; ++bj) {
      const int o = unit(wc + bj * 16 + li, lk);
      bh[bj] = *reinterpret_cast<const V*>(&sh[1][0][o]);
      if constexpr (NP == 2) bl[bj] = *reinterpret_cast<const V*>(&sh[1][NP - 1][o]);
    }
#pragma unroll
    for (int bi = 0; bi < 4; ++bi) {
      const int o = unit(wr + bi * 16 + li, lk);
      const V ah = *reinterpret_cast<const V*>(&sh[0][0][o]);
      if constexpr (NP == 2) {
        const V al = *reinterpret_cast<const V*>(&sh[0][NP - 1][o]);
#pragma unroll
        for (int bj = 0; bj < 4; ++bj) acc[bi][bj] = Op16<F16>::mma(al, bh[bj], acc[bi][bj]);
#pragma unroll
        for (int bj = 0; bj < 4; ++bj) acc[bi][bj] = Op16<F16>::mma(ah, bl[bj], acc[bi][bj]);
      }
#pragma unroll
      for (int bj = 0; bj < 4; ++bj) acc[bi][bj] = Op16<F16>::mma(ah, bh[bj], acc[bi][bj]);
    }
  };
  load(0);
#pragma unroll 1
  for (int kk = 0; kk + KC < KD; kk += KC) {
    store();
    __syncthreads();
    load(kk + KC);
    chunk();
    __syncthreads();   // every read of this chunk is done
  }
  store();
  __syncthreads();
  // A22 -= acc through LDS in four passes of 32 rows, so that the tile is read
  // and written by whole 128-byte lines; the first pass's old values come during
  // the last chunk's products, each later pass's before its accumulators are staged
  float* sC = reinterpret_cast<float*>(smem);
  float* tp = A + (size_t)c0 * npad + r0;
  const unsigned to = (tid >> 3) * npad + 4 * (tid & 7);
  float4 old[2][4];
  auto fetch = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 4; ++u) old[p & 1][u] = ntload(reinterpret_cast<const float4*>((tp + (size_t)(32 * u) * npad + RP * p) + to));
  };
  fetch(0);
  chunk();
  float ci[4];
#pragma unroll
  for (int bj = 0; bj < 4; ++bj) ci[bj] = F16 ? __uint_as_float((254 - scale_exp(cm[wc + bj * 16 + li])) << 23) : 1.0f;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    __syncthreads();
    if (p < 3) fetch(p + 1);
    if (wr == 64 * (p >> 1)) {
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2) {
        const int bi = 2 * (p & 1) + b2;
        float ri[4] = {1.0f, 1.0f, 1.0f, 1.0f};
        if constexpr (F16) {
          const float4 mm = *reinterpret_cast<const float4*>(rm + wr + 16 * bi + 4 * lk);
          ri[0] = __uint_as_float((254 - scale_exp(mm.x)) << 23);
          ri[1] = __uint_as_float((254 - scale_exp(mm.y)) << 23);
          ri[2] = __uint_as_float((254 - scale_exp(mm.z)) << 23);
          ri[3] = __uint_as_float((254 - scale_exp(mm.w)) << 23);
        }
#pragma unroll
        for (int bj = 0; bj < 4; ++bj) {
          f32x4 v = acc[bi][bj];
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = v[t] * ri[t] * ci[bj];
          *reinterpret_cast<f32x4*>(sC + (wc + bj * 16 + li) * LDC + 16 * b2 + 4 * lk) = v;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(sC + (tid / 8 + 32 * u) * LDC + 4 * (tid & 7));
      float4 o = old[p & 1][u];
      o.x -= v[0];
      o.y -= v[1];
      o.z -= v[2];
      o.w -= v[3];
      *reinterpret_cast<float4*>((tp + (size_t)(32 * u) * npad + RP * p) + to) = o;
    }
  }
}

// ---------------------------------------------------------------------------
// Trailing update A22 -= L21 U12: 128 x 128 tiles, K = KD (one panel, 128, or
// two, 256) in chunks of KC staged
// through double-buffered LDS, four wavefronts of 64 x 64 (4 x 4 MFMA blocks).
// The epilogue goes through LDS in P passes of 128 / P rows, which bounds the
// LDS of a block by the K-chunk buffers and lets MINB blocks share a CU; the
// old values of the first NPP passes are loaded before the last K chunk, those
// of every later pass before its accumulators are staged, so that their
// latency hides behind the products or the staging.
// ---------------------------------------------------------------------------
template <typename T, int KC, int P, int MINB, int NPP, int KD>
__global__ __launch_bounds__(256, MINB) void k_update(T* __restrict__ LU, int npad, int k0, int mtr, int mtc, int tj0,
                                                      int nmat, int lrow) {
  using V = typename Vec4<T>::type;
  constexpr int PER = Vec4<T>::per;
  // LDS rows of the K chunk (64 banks of 4 bytes).  FP32: a pitch of 144 puts
  // an operand read (lanes li + 16 lk, rows k + lk, 16 columns) on 64 distinct
  // banks, and U12's transposed stores (16 columns, rows 4 q + m) write column
  // j of row r at j ^ SW(r), SW(r) = 16 ((r / 4) mod 4), so that the four q
  // fall on different banks too; the swizzle is uniform over a wave at each
  // k step of the product, whose reads take column block bj ^ (k / 4 mod 4).
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int LD = F32 ? 128 + 16 : 128 + 4;
  auto sw = [](int r) { return F32 ? 16 * ((r >> 2) & 3) : 0; };
  constexpr int RP = 128 / P;
  constexpr int LDC = RP + 4 / (sizeof(T) / 4);
  int mat, tile;
  xcd_map(blockIdx.x, mtr * mtc + lrow, nmat, &mat, &tile);
  if (mat >= nmat) return;
  // mtr x mtc tiles, then lrow more in the first tile row (columns mtc ..)
  const bool band = tile >= mtr * mtc;
  const int ti = band ? 0 : tile % mtr, tj = band ? mtc + (tile - mtr * mtc) : tile / mtr;
  T* A = LU + (size_t)mat * npad * npad;
  const int r0 = k0 + KD + ti * 128, c0 = k0 + KD + (tj0 + tj) * 128;
  constexpr int OPER = 2 * 2 * KC * LD;
  constexpr int EPI = 128 * LDC;
  __shared__ __align__(16) T smem[OPER > EPI ? OPER : EPI];
  T (*sA)[KC][LD] = reinterpret_cast<T (*)[KC][LD]>(smem);
  T (*sB)[KC][LD] = reinterpret_cast<T (*)[KC][LD]>(smem + 2 * KC * LD);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wr = (w >> 1) * 64, wc = (w & 1) * 64;
  constexpr int NA = KC * 128 / PER / 256, NBV = KC * 128 / PER / 256;
  V ra[NA], rb[NBV];
  auto load = [&](int kk) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int e = tid + u * 256;
      const int k = e / (128 / PER), i = (e % (128 / PER)) * PER;
      ra[u] = *reinterpret_cast<const V*>(A + (size_t)(k0 + kk + k) * npad + r0 + i);
    }
#pragma unroll
    for (int u = 0; u < NBV; ++u) {
      const int e = tid + u * 256;
      const int j = e / (KC / PER), k = (e % (KC / PER)) * PER;
      rb[u] = *reinterpret_cast<const V*>(A + (size_t)(c0 + j) * npad + k0 + kk + k);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int e = tid + u * 256;
      const int k = e / (128 / PER), i = (e % (128 / PER)) * PER;
      const T* v = reinterpret_cast<const T*>(&ra[u]);
#pragma unroll
      for (int m = 0; m < PER; ++m) sA[buf][k][i + m] = v[m];
    }
#pragma unroll
    for (int u = 0; u < NBV; ++u) {
      const int e = tid + u * 256;
      const int j = e / (KC / PER), k = (e % (KC / PER)) * PER;
      const T* v = reinterpret_cast<const T*>(&rb[u]);
#pragma unroll
      for (int m = 0; m < PER; ++m) sB[buf][k + m][j ^ sw(k + m)] = v[m];
    }
  };
  typename Mma<T>::acc acc[4][4];
#pragma unroll
  for (int bi = 0; bi < 4; ++bi)
#pragma unroll
    for (int bj = 0; bj < 4; ++bj) acc[bi][bj] = typename Mma<T>::acc{0, 0, 0, 0};
  load(0);
  store(0);
  __syncthreads();
  constexpr int NCH = KD / KC;
  constexpr int NV = 128 * RP / PER / 256;   // vectors per thread per pass
  V pre[NPP > 0 ? NPP : 1][NV];
  auto prefetch = [&](int pass, V (&dst)[NV]) {
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = tid + u * 256;
      const int col = e / (RP / PER), rr = (e % (RP / PER)) * PER;
      dst[u] = ntload(reinterpret_cast<const V*>(A + (size_t)(c0 + col) * npad + r0 + pass * RP + rr));
    }
  };
  for (int ch = 0; ch < NCH; ++ch) {
    const int buf = ch & 1;
    if (ch + 1 < NCH) load((ch + 1) * KC);
    else {
#pragma unroll
      for (int pp = 0; pp < NPP; ++pp) prefetch(pp, pre[pp]);
    }
#pragma unroll
    for (int k = 0; k < KC; k += 4) {
      T av[4], bv[4];
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) av[bi] = sA[buf][k + lk][wr + bi * 16 + li];
#pragma unroll
      for (int bj = 0; bj < 4; ++bj) bv[bj] = sB[buf][k + lk][wc + (bj * 16 ^ sw(k)) + li];
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int bj = 0; bj < 4; ++bj) acc[bi][bj] = Mma<T>::step(av[bi], bv[bj], acc[bi][bj]);
    }
    if (ch + 1 < NCH) {
      store(buf ^ 1);
      __syncthreads();
    }
  }
  T* sC = smem;
#pragma unroll
  for (int pass = 0; pass < P; ++pass) {
    V old[NV];
    if (pass >= NPP) prefetch(pass, old);
    __syncthreads();
#pragma unroll
    for (int bi = 0; bi < 4; ++bi) {
      if ((wr + bi * 16) / RP == pass) {
#pragma unroll
        for (int bj = 0; bj < 4; ++bj)
#pragma unroll
          for (int it = 0; it < 4; ++it)
            sC[(wc + bj * 16 + li) * LDC + wr + bi * 16 - pass * RP + Mma<T>::row(lk, it)] = acc[bi][bj][it];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = tid + u * 256;
      const int col = e / (RP / PER), rr = (e % (RP / PER)) * PER;
      V* p = reinterpret_cast<V*>(A + (size_t)(c0 + col) * npad + r0 + pass * RP + rr);
      V o;
      if (pass < NPP) o = pre[pass < NPP ? pass : 0][u];
      else o = old[u];
      const V a = *reinterpret_cast<const V*>(sC + col * LDC + rr);
      T* po = reinterpret_cast<T*>(&o);
      const T* pa = reinterpret_cast<const T*>(&a);
#pragma unroll
      for (int m = 0; m < PER; ++m) po[m] -= pa[m];
      *p = o;
    }
  }
}

template <int KD>
void launch_update_k(int kind, void* LU, int npad, int k0, int mtr, int mtc, int tj0, int nmat, bool alt_kc,
                     hipStream_t s, int lrow, const float* rmax, const float* cmax) {
  const dim3 gu = xcd_grid(mtr * mtc + lrow, nmat);
  float* A = static_cast<float*>(LU);
  if (kind == 2) {
    k_update_split<KD, false, 1><<<gu, 256, 0, s>>>(A, nullptr, nullptr, npad, k0, mtr, mtc, tj0, nmat, lrow);
  } else if (kind == 3) {
    k_update_split<KD, false, 3><<<gu, 256, 0, s>>>(A, nullptr, nullptr, npad, k0, mtr, mtc, tj0, nmat, lrow);
  } else if (kind == 1 && rmax) {
    k_update_split<KD, true, 3><<<gu, 256, 0, s>>>(A, rmax, cmax, npad, k0, mtr, mtc, tj0, nmat, lrow);
  } else if constexpr (KD <= 2 * NB) {   // (groups of four take the forms above)
    double* D = static_cast<double*>(LU);
    if (kind == 0 && alt_kc) k_update<double, 8, 4, 2, 1, KD><<<gu, 256, 0, s>>>(D, npad, k0, mtr, mtc, tj0, nmat, lrow);
    else if (kind == 0) k_update<double, 16, 4, 2, 1, KD><<<gu, 256, 0, s>>>(D, npad, k0, mtr, mtc, tj0, nmat, lrow);
    else if (alt_kc) k_update<float, 32, 1, 2, 1, KD><<<gu, 256, 0, s>>>(A, npad, k0, mtr, mtc, tj0, nmat, lrow);
    else k_update<float, 16, 4, 4, 1, KD><<<gu, 256, 0, s>>>(A, npad, k0, mtr, mtc, tj0, nmat, lrow);
  } else {
    throw std::logic_error("no trailing update of this depth without the row and column maxima");
  }
}

}  // namespace

void launch_update(int kind, void* LU, int npad, int k0, int mtr, int mtc, int tj0, int nmat, bool alt_kc,
                   hipStream_t s, int kd, int lrow, const float* rmax, const float* cmax) {
  auto go = [&](auto kdc) {
    launch_update_k<decltype(kdc)::value>(kind, LU, npad, k0, mtr, mtc, tj0, nmat, alt_kc, s, lrow, rmax, cmax);
  };
  switch (kd) {
    case 4 * NB: go(std::integral_constant<int, 4 * NB>{}); break;
    case 3 * NB: go(std::integral_constant<int, 3 * NB>{}); break;
    case 2 * NB: go(std::integral_constant<int, 2 * NB>{}); break;
    case NB: go(std::integral_constant<int, NB>{}); break;
    default: throw std::logic_error("trailing update of an unknown depth");
  }
}

}  // namespace bte
