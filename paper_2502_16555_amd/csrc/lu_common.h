// Device helpers shared by the LU kernels: MFMA tile conventions, XCD-aware
// block mapping and 16-byte vector types.  Each translation unit gets its own
// copies (internal linkage).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "internal.h"

namespace bte {
namespace {

using f64x4 = double __attribute__((ext_vector_type(4)));
using f32x4 = float __attribute__((ext_vector_type(4)));
using f64x2 = double __attribute__((ext_vector_type(2)));

constexpr int kXcd = 8;  // XCDs of an MI355X; workgroups are dealt to them round-robin

// Non-temporal 16-byte load of data read once (the solves' factors, a
// trailing update's old tile), so that it does not displace what is reused.
template <typename V>
__device__ inline V ntload(const V* p) {
  using I = int __attribute__((ext_vector_type(sizeof(V) / 4)));
  return __builtin_bit_cast(V, __builtin_nontemporal_load(reinterpret_cast<const I*>(p)));
}

// f(integral_constant<int, I>) for I in the sequence, in order: loop bodies
// whose indices must be compile-time constants (register arrays, unrolled
// steps) without relying on the unroller
template <int... I, class F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// MFMA 16x16x4 tiles: operand lanes hold A[i = lane%16][k = lane/16] and
// B[k = lane/16][j = lane%16]; result item t of lane l holds D[row(l, t)][l%16]
// with row = 4*(l/16) + t for f32 and row = l/16 + 4*t for f64 (measured).
template <typename T>
struct Mma;
template <>
struct Mma<double> {
  using acc = f64x4;
  __device__ static inline acc step(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lk, int t) { return lk + 4 * t; }
};
template <>
struct Mma<float> {
  using acc = f32x4;
  __device__ static inline acc step(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lk, int t) { return 4 * lk + t; }
};

// Block id -> (matrix, item) such that all items of a matrix run on one XCD.
__device__ inline void xcd_map(int bid, int items, int nmat, int* mat, int* item) {
  const int xcd = bid % kXcd, j = bid / kXcd;
  *mat = xcd + kXcd * (j / items);
  *item = j % items;
}

inline int xcd_grid(int items, int nmat) { return kXcd * items * ((nmat + kXcd - 1) / kXcd); }

// Columns at a wavefront-uniform address: next() gives each one's and steps on.
// Kept in scalar registers, so that a load takes the lane's 32-bit offset alone
// (the compiler makes a 64-bit address per load and lane of it otherwise).
template <typename T>
struct UniformCols {
  uint64_t p;
  const uint64_t stride;
  __device__ __forceinline__ UniformCols(const T* base, size_t elems)
      : p(reinterpret_cast<uint64_t>(base)), stride(elems * sizeof(T)) {}
  __device__ __forceinline__ const T* next() {
    using G = const T __attribute__((address_space(1)))*;
    asm("" : "+s"(p));
    const uint64_t q = p;
    p += stride;
    return (const T*)(G)q;
  }
};

// Barrier for data exchanged through LDS only: the block's global loads
// and stores stay in flight (a full fence would wait for them every time).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Barrier past which every global load that the block issued before it has its
// value: for stores to locations that other wavefronts have read (lds_barrier
// orders no global access, and a load may still be on its way behind it).
__device__ __forceinline__ void loads_barrier() {
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt 0, the other counters free
  __syncthreads();
}

// Wavefront reductions through DPP lane permutations (quad swaps, half-row and
// row mirrors) inside each row of 16 lanes, then the four row results by lane
// reads: no LDS round trip on the pivot search's critical path.
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp(static_cast<int>(b), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(static_cast<int>(b >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
__device__ inline double readlane_f64(double v, int l) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(b), l);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), l);
  return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
// maximum over the wavefront of values that are never NaN; uniform result
__device__ inline double wave_max(double v) {
  double o = dpp_f64<0xB1>(v);  // quad_perm [1,0,3,2]
  v = o > v ? o : v;
  o = dpp_f64<0x4E>(v);         // quad_perm [2,3,0,1]
  v = o > v ? o : v;
  o = dpp_f64<0x141>(v);        // row_half_mirror
  v = o > v ? o : v;
  o = dpp_f64<0x140>(v);        // row_mirror
  v = o > v ? o : v;
  const double r0 = readlane_f64(v, 0), r1 = readlane_f64(v, 16), r2 = readlane_f64(v, 32), r3 = readlane_f64(v, 48);
  const double m0 = r1 > r0 ? r1 : r0, m1 = r3 > r2 ? r3 : r2;
  return m1 > m0 ? m1 : m0;
}
// v max of the lane that DPP control CTRL names (0 for none)
template <int CTRL>
__device__ __forceinline__ unsigned dpp_max(unsigned v) {
  return max(v, static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, false)));
}
// maximum over the 16 lanes of a DPP row of non-negative floats (whose bits
// order like the values)
__device__ __forceinline__ float row16_max(float v) {
  const unsigned u = __float_as_uint(v);
  return __uint_as_float(dpp_max<0x140>(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(u)))));
}
// maximum over the wavefront of 64-bit unsigned keys; uniform result
template <int CTRL>
__device__ inline unsigned long long dpp_u64(unsigned long long v) {
  const int lo = __builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(static_cast<int>(v >> 32), CTRL, 0xF, 0xF, false);
  return (static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) | static_cast<unsigned>(lo);
}
__device__ inline unsigned long long readlane_u64(unsigned long long v, int l) {
  const unsigned lo = __builtin_amdgcn_readlane(static_cast<int>(v), l);
  const unsigned hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), l);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}
__device__ inline unsigned long long wave_max_u64(unsigned long long v) {
  unsigned long long o = dpp_u64<0xB1>(v);
  v = o > v ? o : v;
  o = dpp_u64<0x4E>(v);
  v = o > v ? o : v;
  o = dpp_u64<0x141>(v);
  v = o > v ? o : v;
  o = dpp_u64<0x140>(v);
  v = o > v ? o : v;
  const unsigned long long r0 = readlane_u64(v, 0), r1 = readlane_u64(v, 16), r2 = readlane_u64(v, 32),
                           r3 = readlane_u64(v, 48);
  const unsigned long long m0 = r1 > r0 ? r1 : r0, m1 = r3 > r2 ? r3 : r2;
  return m1 > m0 ? m1 : m0;
}
__device__ inline int wave_min(int v) {
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false));
  return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
  using type = float4;
  static constexpr int per = 4;
};
template <>
struct Vec4<double> {
  using type = double2;
  static constexpr int per = 2;
};
// FP16 storage of factors that only precondition (the Krylov solver's bins)
using half8 = _Float16 __attribute__((ext_vector_type(8)));
template <>
struct Vec4<_Float16> {
  using type = half8;
  static constexpr int per = 8;
};

// Sums of the wavefront for eight values per lane: lane l returns value l mod 8's
// (the values are halved three times as the lanes pair up, then summed).
__device__ __forceinline__ double fold8(const double (&v)[8], int lane) {
  double a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool up = lane & 1;
    a[i] = (up ? v[2 * i + 1] : v[2 * i]) + __shfl_xor(up ? v[2 * i] : v[2 * i + 1], 1);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool up = lane & 2;
    b[i] = (up ? a[2 * i + 1] : a[2 * i]) + __shfl_xor(up ? a[2 * i] : a[2 * i + 1], 2);
  }
  const bool up = lane & 4;
  double c = (up ? b[1] : b[0]) + __shfl_xor(up ? b[0] : b[1], 4);
  c += __shfl_xor(c, 8);
  c += __shfl_xor(c, 16);
  return c + __shfl_xor(c, 32);
}

// Stop test of the refinement: the largest normwise backward error of the points,
//   eta_x = max|r_x| / (||M_x|| max|x_x| + max|b_x|),
// with ||M_x|| <= 1 + dt (n0_x ||C|| + |E_x| ||A||) in the norm that matches
// max-norms of the vectors (inf-norm for M, 1-norm for M^T).  The residual's own
// FP64 rounding is of order sqrt(n) eps ||M|| |x|, so a bound relative to |b|
// alone is unreachable once dt |E| ||A|| grows; eta is not.  On every thread of
// the block.
template <int NT>
__device__ __forceinline__ double refine_worst(const RefineCheck& c) {
  __shared__ double red[NT / 64];
  double worst = 0.0;
  for (int x = threadIdx.x; x < c.nx; x += NT) {
    const double r = __longlong_as_double(static_cast<long long>(c.r[x]));
    const double b = __longlong_as_double(static_cast<long long>(c.b[x]));
    const double xm = __longlong_as_double(static_cast<long long>(c.x[x]));
    const double mn = 1.0 + c.dt * (c.n0x[x] * c.cnorm + fabs(c.E[x]) * c.anorm);
    const double den = mn * xm + b;
    const double q = (den > 0.0) ? r / den : (r > 0.0 ? INFINITY : 0.0);
    worst = fmax(worst, (q == q) ? q : INFINITY);
  }
  worst = wave_max(worst);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = worst;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) worst = fmax(worst, red[w]);
  return worst;
}

}  // namespace
}  // namespace bte
