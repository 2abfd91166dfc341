// Helpers shared by the HIP kernel files: vector types over VEC columns, row loads, the
// wavefront-private LDS strip barrier, and the host-side choice of the (VEC, LPR) shape.
// Everything has internal linkage; include inside a .hip file only.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "arrow_internal.h"

namespace arrow {
namespace {

constexpr int kBlock = 64 * kChunksPerGroup;  // threads per workgroup = 4 wavefronts

template <int VEC> struct Vec;
template <> struct Vec<1> { using type = float; };
template <> struct Vec<2> { using type = float2; };
template <> struct Vec<4> { using type = float4; };

template <int VEC> __device__ __forceinline__ typename Vec<VEC>::type vzero();
template <> __device__ __forceinline__ float vzero<1>() { return 0.f; }
template <> __device__ __forceinline__ float2 vzero<2>() { return make_float2(0.f, 0.f); }
template <> __device__ __forceinline__ float4 vzero<4>() { return make_float4(0.f, 0.f, 0.f, 0.f); }

__device__ __forceinline__ void vfma(float& a, float s, float x) { a = fmaf(s, x, a); }
__device__ __forceinline__ void vfma(float2& a, float s, float2 x) {
  a.x = fmaf(s, x.x, a.x); a.y = fmaf(s, x.y, a.y);
}
__device__ __forceinline__ void vfma(float4& a, float s, float4 x) {
  a.x = fmaf(s, x.x, a.x); a.y = fmaf(s, x.y, a.y); a.z = fmaf(s, x.z, a.z); a.w = fmaf(s, x.w, a.w);
}
__device__ __forceinline__ void vadd(float& a, float x) { a += x; }
__device__ __forceinline__ void vadd(float2& a, float2 x) { a.x += x.x; a.y += x.y; }
__device__ __forceinline__ void vadd(float4& a, float4 x) { a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w; }

__device__ __forceinline__ float vshfl_xor(float v, int m) { return __shfl_xor(v, m, 64); }
__device__ __forceinline__ float2 vshfl_xor(float2 v, int m) {
  return make_float2(__shfl_xor(v.x, m, 64), __shfl_xor(v.y, m, 64));
}
__device__ __forceinline__ float4 vshfl_xor(float4 v, int m) {
  return make_float4(__shfl_xor(v.x, m, 64), __shfl_xor(v.y, m, 64), __shfl_xor(v.z, m, 64),
                     __shfl_xor(v.w, m, 64));
}

template <int VEC>
__device__ __forceinline__ typename Vec<VEC>::type vload(const float* p) {
  return *reinterpret_cast<const typename Vec<VEC>::type*>(p);
}
template <int VEC>
__device__ __forceinline__ void vstore(float* p, typename Vec<VEC>::type v) {
  *reinterpret_cast<typename Vec<VEC>::type*>(p) = v;
}

// The same for global memory at any 4-byte boundary: one 16-byte instruction does it there, so rows
// whose length is no multiple of 4 columns are still moved four columns per lane (lane_columns).
typedef float stream_v2f __attribute__((ext_vector_type(2), aligned(4)));
typedef float stream_v4f __attribute__((ext_vector_type(4), aligned(4)));
template <int VEC> __device__ __forceinline__ typename Vec<VEC>::type gload(const float* p);
template <> __device__ __forceinline__ float gload<1>(const float* p) { return *p; }
template <> __device__ __forceinline__ float2 gload<2>(const float* p) {
  const stream_v2f t = *reinterpret_cast<const stream_v2f*>(p); return make_float2(t.x, t.y);
}
template <> __device__ __forceinline__ float4 gload<4>(const float* p) {
  const stream_v4f t = *reinterpret_cast<const stream_v4f*>(p); return make_float4(t.x, t.y, t.z, t.w);
}
template <int VEC> __device__ __forceinline__ void gstore(float* p, typename Vec<VEC>::type v);
template <> __device__ __forceinline__ void gstore<1>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void gstore<2>(float* p, float2 v) {
  stream_v2f t; t.x = v.x; t.y = v.y;
  *reinterpret_cast<stream_v2f*>(p) = t;
}
template <> __device__ __forceinline__ void gstore<4>(float* p, float4 v) {
  stream_v4f t; t.x = v.x; t.y = v.y; t.z = v.z; t.w = v.w;
  *reinterpret_cast<stream_v4f*>(p) = t;
}

// First column of lane l's VEC columns in the slice of `width` columns that starts at column c0; a lane whose columns
// would run past the last one is moved back so that they end there.  It then shares `shared` columns
// with the lane before it: both hold and store the same values for them.  Lanes that start at or
// beyond column k have none (ok = false) and read column 0.
struct LaneColumns {
  int c;         // first column
  int shared;    // columns that the lane before holds as well
  bool ok;
};
template <int VEC>
__device__ __forceinline__ LaneColumns lane_columns(int l, int c0, int k, int width = 1 << 20) {
  LaneColumns r;
  r.c = c0 + l * VEC;
  r.shared = 0;
  r.ok = r.c < k && l * VEC < width;
  if (VEC > 1 && r.ok && r.c + VEC > k) { r.shared = r.c + VEC - k; r.c = k - VEC; }
  return r;
}

// Store of a result row that this product does not read again: the non-temporal hint keeps the
// 4 k bytes per output row from displacing rows of X in the L2 (measured on the R-MAT workload:
// short rows 3.97 -> 3.71 ms, reduction 0.38 -> 0.33 ms; the same hint on loads of X rows made the
// product slower; for the entries see stream_load).
template <int VEC>
__device__ __forceinline__ void vstore_stream(float* p, typename Vec<VEC>::type v);
template <> __device__ __forceinline__ void vstore_stream<1>(float* p, float v) { __builtin_nontemporal_store(v, p); }
template <> __device__ __forceinline__ void vstore_stream<2>(float* p, float2 v) {
  stream_v2f t; t.x = v.x; t.y = v.y;
  __builtin_nontemporal_store(t, reinterpret_cast<stream_v2f*>(p));
}
template <> __device__ __forceinline__ void vstore_stream<4>(float* p, float4 v) {
  stream_v4f t; t.x = v.x; t.y = v.y; t.z = v.z; t.w = v.w;
  __builtin_nontemporal_store(t, reinterpret_cast<stream_v4f*>(p));
}

// Load of a row that is read exactly once (a partial vector in the reduction, the old value of a
// Y row a later level adds to), same hint.
template <int VEC>
__device__ __forceinline__ typename Vec<VEC>::type vload_stream(const float* p);
template <> __device__ __forceinline__ float vload_stream<1>(const float* p) { return __builtin_nontemporal_load(p); }
template <> __device__ __forceinline__ float2 vload_stream<2>(const float* p) {
  stream_v2f t = __builtin_nontemporal_load(reinterpret_cast<const stream_v2f*>(p)); return make_float2(t.x, t.y);
}
template <> __device__ __forceinline__ float4 vload_stream<4>(const float* p) {
  stream_v4f t = __builtin_nontemporal_load(reinterpret_cast<const stream_v4f*>(p)); return make_float4(t.x, t.y, t.z, t.w);
}

// Load VEC columns of row `row` of a row-major matrix.  `base` is wavefront-uniform,
// col_bytes the lane's byte offset inside a row, row_bytes = 4 k.
// SMALL: the matrix has at most 2^24 rows and 2^32 bytes, so the byte offset is one 24-bit
// multiply-add and the load can use (uniform base + 32-bit lane offset) addressing.
template <bool SMALL>
__device__ __forceinline__ auto row_offset(int32_t row, uint32_t row_bytes, uint32_t col_bytes) {
  if constexpr (SMALL) return __umul24((uint32_t)row, row_bytes) + col_bytes;
  else return (uint64_t)(uint32_t)row * row_bytes + col_bytes;
}
template <int VEC, bool SMALL>
__device__ __forceinline__ typename Vec<VEC>::type load_row(const char* base, int32_t row,
                                                            uint32_t row_bytes, uint32_t col_bytes) {
  return gload<VEC>(reinterpret_cast<const float*>(base + row_offset<SMALL>(row, row_bytes, col_bytes)));
}

// A load of what is read once: it leaves the rows of X in the L2 alone.  Entries of the order-3 product and of
// window rows always, those of the product's short rows from a size on (kEntriesOnce); the entries of the wave
// list, which a column pass reads again, never.
template <typename T> __device__ __forceinline__ T stream_load(const T* p) {
  if constexpr (sizeof(T) == 8) {
    const unsigned long long v = __builtin_nontemporal_load(reinterpret_cast<const unsigned long long*>(p));
    T t;
    __builtin_memcpy(&t, &v, 8);
    return t;
  } else {
    return __builtin_nontemporal_load(p);
  }
}

__device__ __forceinline__ void strip_sync() {
  // the strip is written and read by lanes of ONE wavefront: LDS executes a wavefront's
  // instructions in order, so only the compiler has to be kept from reordering
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// dot products across the lanes of a group
// ---------------------------------------------------------------------------
__device__ __forceinline__ float vdot(float u, float x) { return u * x; }
__device__ __forceinline__ float vdot(float2 u, float2 x) { return fmaf(u.y, x.y, u.x * x.x); }
__device__ __forceinline__ float vdot(float4 u, float4 x) {
  return fmaf(u.w, x.w, fmaf(u.z, x.z, fmaf(u.y, x.y, u.x * x.x)));
}

// A lane that shares columns with the one before it (lane_columns) leaves them out of its dot products.
__device__ __forceinline__ void drop_shared(float&, int) {}
__device__ __forceinline__ void drop_shared(float2& v, int shared) { if (shared) v.x = 0.f; }
__device__ __forceinline__ void drop_shared(float4& v, int shared) {
  if (shared > 0) v.x = 0.f;
  if (shared > 1) v.y = 0.f;
  if (shared > 2) v.z = 0.f;
}

// v of a lane whose bit M differs from this lane's (M = 1, 2, 4, 8: the partner differs in lower bits
// too where M = 4; a reduction over those bits does not mind).  A DPP operand, no LDS access.
template <int M> __device__ __forceinline__ float across(float v) {
  static_assert(M == 1 || M == 2 || M == 4 || M == 8, "within sixteen lanes");
  constexpr int ctrl = M == 1 ? 0xB1 /* quad_perm 1,0,3,2 */ : M == 2 ? 0x4E /* quad_perm 2,3,0,1 */
                     : M == 4 ? 0x141 /* row_half_mirror */ : 0x128 /* row_ror 8 */;
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, false));
}

// One exchange of the transposing butterfly: lanes with bit M clear get the sum over bit M of `a`,
// lanes with it set that of `b`.
template <int M> __device__ __forceinline__ float exchange(float a, float b, int lane) {
  if constexpr (M == 32 || M == 16) {
    // swaps the halves (rows of sixteen) of one register with the other halves of the second
    const auto r = M == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false)
                           : __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
    return __int_as_float(r[0]) + __int_as_float(r[1]);
  } else {
    const bool upper = (lane & M) != 0;
    return (upper ? b : a) + across<M>(upper ? a : b);
  }
}

// The sum over all lanes, in every lane: over bit 0 first, then bits 1 to 5.
__device__ __forceinline__ float wave_sum(float v) {
  v += across<1>(v);
  v += across<2>(v);
  v += across<4>(v);
  v += across<8>(v);
  v = exchange<16>(v, v, 0);
  return exchange<32>(v, v, 0);
}

// The same sums of eight values in the same order of additions, each in eight lanes: lane l has that of value
// 4 (l & 1) + (l & 2) + (l >> 2 & 1).
__device__ __forceinline__ float wave_sum8(const float (&v)[8], int lane) {
  const float a0 = exchange<1>(v[0], v[4], lane), a1 = exchange<1>(v[1], v[5], lane), a2 = exchange<1>(v[2], v[6], lane),
              a3 = exchange<1>(v[3], v[7], lane);
  const float b0 = exchange<2>(a0, a2, lane), b1 = exchange<2>(a1, a3, lane);
  // the partner across four lanes by the mirror image of eight and that of four of it
  const bool upper = (lane & 4) != 0;
  const float other = across<4>(upper ? b0 : b1);
  float c = (upper ? b1 : b0) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(other), 0x1B /* quad_perm 3,2,1,0 */, 0xf, 0xf, false));
  c += across<8>(c);
  c = exchange<16>(c, c, 0);
  return exchange<32>(c, c, 0);
}

// Sums of NB values over the LPR lanes of a group: the upper lanes keep the upper half of the values at
// every exchange, so that lane l ends up with the sum of value l / (LPR / NB).  With shuffles through
// LDS instead of permlane swaps and DPP operands it took 40 vector instructions and 6 LDS accesses for
// four values, now 10 and none.
template <int NB, int LPR>
__device__ __forceinline__ float group_reduce(float (&p)[NB], int l) {
  if constexpr (LPR == 1) {
    return p[0];
  } else if constexpr (NB > 1) {
    float q[NB / 2];
#pragma unroll
    for (int e = 0; e < NB / 2; ++e) q[e] = exchange<LPR / 2>(p[e], p[e + NB / 2], l);
    return group_reduce<NB / 2, LPR / 2>(q, l);
  } else {
    float q[1] = {exchange<LPR / 2>(p[0], p[0], l)};
    return group_reduce<1, LPR / 2>(q, l);
  }
}

// ---------------------------------------------------------------------------
// host-side dispatch on (VEC, LPR)
// ---------------------------------------------------------------------------
struct Shape {
  int vec, lpr, slices;
  int width;             // columns per slice where the slices are made even (a multiple of vec); lpr * vec at most
};

// Columns per lane: 4 wherever a row has that many (the last lane of a row may share columns with
// its neighbour, see lane_columns): a 16-byte load moves four times as much per instruction as the
// 4-byte load an odd k would otherwise take, and a row needs a quarter of the lanes.  `exact` asks
// for lanes that share nothing: kernels that lay lanes' columns out side by side in LDS, and
// launches that add to Y whose last slice would reach back into the one before (two workgroups
// would then add to the same elements).
[[maybe_unused]] Shape pick_shape(int k, int kc, bool exact = false) {
  Shape s;
  s.vec = k >= 4 ? 4 : (k == 2 ? 2 : 1);
  if (exact) s.vec = (k % 4 == 0) ? 4 : (k % 2 == 0) ? 2 : 1;
  int width = k;                                   // columns per slice
  if (kc > 0 && kc < width) width = kc;
  if (width > 64 * s.vec) width = 64 * s.vec;
  int lanes = (width + s.vec - 1) / s.vec;
  int lpr = 1;
  while (lpr < lanes) lpr <<= 1;
  s.lpr = lpr;
  s.slices = (k + lpr * s.vec - 1) / (lpr * s.vec);
  // slices of about the same width; where rows are whole 128-byte lines, so are the slices (k = 96 in
  // 48 and 48 columns reads four lines of a row, in 64 and 32 three: R-MAT 1.1m 1026 and 880 us)
  const int step = k % 32 == 0 && s.vec == 4 && lpr >= 8 ? 32 : s.vec;
  s.width = ((k + s.slices - 1) / s.slices + step - 1) / step * step;
  return s;
}

template <typename F>
int dispatch_shape(const Shape& s, F&& f) {
#define ARROW_CASE(V, L) \
  if (s.vec == V && s.lpr == L) return f(std::integral_constant<int, V>{}, std::integral_constant<int, L>{});
#define ARROW_CASES(V) \
  ARROW_CASE(V, 1) ARROW_CASE(V, 2) ARROW_CASE(V, 4) ARROW_CASE(V, 8) ARROW_CASE(V, 16) ARROW_CASE(V, 32) ARROW_CASE(V, 64)
  ARROW_CASES(4)
  ARROW_CASES(2)
  ARROW_CASES(1)
#undef ARROW_CASES
#undef ARROW_CASE
  return (int)hipErrorInvalidValue;
}

// the shape of a launch that writes Y: exact where it adds to Y and its last slice holds fewer than 4 columns
[[maybe_unused]] Shape pick_output_shape(int k, int kc, bool accumulate) {
  const Shape s = pick_shape(k, kc);
  const int last = k - (s.slices - 1) * s.width;
  return accumulate && s.slices > 1 && last < s.vec ? pick_shape(k, kc, true) : s;
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// 32-bit offsets are enough when a matrix of `rows` rows and k columns stays below 2^24 rows
// and 2^32 bytes (and a row below 2^24 bytes, for the 24-bit multiply)
inline bool small_matrix(int64_t rows, int32_t k) {
  return rows <= (1LL << 24) && rows * (int64_t)k * 4 <= (1LL << 32) && (int64_t)k * 4 < (1LL << 24);
}

}  // namespace
}  // namespace arrow
