// HIP kernel for gfx950 of the order-3 MTTKRP
//     A(i, a) = sum_{j,k} T(i, j, k) B(j, a) C(k, a)
// in the factorize-and-fuse form (the paper's sections "Pairwise Contraction" and "Performance
// Evaluation"): per fibre (i, j) the sum x(a) = sum_k T(i,j,k) C(k,a) is formed first -- the same
// scaled vector update over the dense index as the matrix product's leaf -- and then multiplied
// elementwise by B(j, :) and added to the slice's accumulator, so the intermediate never leaves
// registers and the products with B are paid per fibre, not per entry.
//
// A lane owns VEC consecutive columns of the rank index, LPR lanes cover a slice of LPR * VEC
// columns, a wavefront holds G = 64 / LPR lane groups.  One wavefront per work item (a run of
// segments of one slice i, at most kCsfItemNnz entries and kCsfItemSegs segments, each segment
// being at most 64 entries of one fibre).  The wavefront first copies the item's entries and
// segment descriptors into LDS with coalesced loads and reads them from there, so that the only
// memory latency inside the loop is that of the gathered rows.
//
// The build sorts an item's segments by length, longest first, so the segments that the lane groups
// take side by side are equally long nearly everywhere: such a round needs no masks and no load slot
// stays unused.  Short segments are taken two or four per lane group at a time, which keeps four
// to eight row loads in flight whatever their length (more of them cost registers: six wavefronts per
// SIMD instead of eight is 12 % slower).  In the order of j a round lasted as long as the
// longest of G random lengths, and with the masks 16 vector instructions stood for every row load, of
// which 5 do the work: the kernel was bound by instruction issue (83 % of the cycles).  Uniform 4096^3
// tensor, 68.7 M entries in 16.5 M fibres, R = 64: 1078 -> 850 us; what it gathers (21.8 GB from the L2 at
// 64 B per cycle and compute unit) takes 630 us, which is why factors that fit the LDS are read from there
// (resident_kernel).  A skewed tensor of 16.4 M fibres of one entry, R = 32, gained
// nothing (507 us): B and C are 8 MiB each and an L2 is 4 MiB, so that 68 % of the requests missed it, 3.3 GB that
// came at 6.6 TB/s; such tensors have a form of their own too (streams_kernel).
//
// At the end the lane groups are combined with wavefront shuffles and the result goes to row i of A
// or, for a slice cut into several items, to a partial vector that the reduction kernel sums in a
// fixed order.  No atomics.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <type_traits>

#include "arrow_internal.h"
#include "kernel_common.h"

namespace arrow {
namespace {

__device__ __forceinline__ void vmuladd(float& a, float x, float b) { a = fmaf(x, b, a); }
__device__ __forceinline__ void vmuladd(float2& a, float2 x, float2 b) {
  a.x = fmaf(x.x, b.x, a.x); a.y = fmaf(x.y, b.y, a.y);
}
__device__ __forceinline__ void vmuladd(float4& a, float4 x, float4 b) {
  a.x = fmaf(x.x, b.x, a.x); a.y = fmaf(x.y, b.y, a.y); a.z = fmaf(x.z, b.z, a.z); a.w = fmaf(x.w, b.w, a.w);
}

// The staged item and what a lane needs to load rows of the factors.
struct ItemView {
  const Entry* ent;
  const uint16_t* ptr;      // segment offsets relative to the item's first entry
  const int32_t* j;
  const char* B;
  const char* C;
  uint32_t row_bytes, col_bytes;
};

// Segments s0 + p * G + g, p < P, of at most U entries each (P = 1: any number, U at a time);
// ALIKE: all of them exist and hold `len` entries.
template <int VEC, int LPR, int P, int U, bool SMALL, bool ALIKE>
__device__ __forceinline__ void segments(const ItemView& v, uint32_t s0, uint32_t n_seg, uint32_t len, uint32_t g,
                                         typename Vec<VEC>::type& acc) {
  using V = typename Vec<VEC>::type;
  constexpr uint32_t G = 64 / LPR;
  uint32_t lo[P], n[P];
  V b[P], x[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint32_t s = s0 + p * G + g;
    const bool there = ALIKE || s < n_seg;
    lo[p] = there ? (uint32_t)v.ptr[s] : 0u;
    n[p] = ALIKE ? len : (there ? (uint32_t)v.ptr[s + 1] - lo[p] : 0u);
    b[p] = x[p] = vzero<VEC>();
    if (there) b[p] = load_row<VEC, SMALL>(v.B, v.j[s], v.row_bytes, v.col_bytes);
  }
  uint32_t done = 0;
  do {
    Entry e[P][U];
    V c[P][U];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (done + u < n[p]) e[p][u] = v.ent[lo[p] + done + u];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (done + u < n[p]) c[p][u] = load_row<VEC, SMALL>(v.C, e[p][u].xrow, v.row_bytes, v.col_bytes);
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (done + u < n[p]) vfma(x[p], e[p][u].val, c[p][u]);
    done += U;
  } while (P == 1 && done < n[0]);
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (ALIKE || n[p] > 0) vmuladd(acc, x[p], b[p]);
}

constexpr int64_t kResidentItems = 8192;  // wavefronts the chip holds

// TOGETHER: the four wavefronts of a workgroup share an item and stage all of it together.  (What a wavefront stages for itself is the segments of its share, whose
// entries it knows only when their offsets have come: one more memory latency, 250 x 231 x 307 of 17,720, R = 25, 5.3 -> 5.0 us, 1086 x 338 x 234 of
// 86 K, 32, 5.3 -> 4.9; 300 x 200 x 307 of 18.4 K, 8, 3.7 -> 3.45.  Where items are many the wavefronts would wait for each other: skewed 5897 x 491 x 536, 8, 13.9 -> 14.2.)
template <int VEC, int LPR, bool SMALL, bool TOGETHER>
__global__ __launch_bounds__(kBlock, 8) void mttkrp_kernel(
    const uint32_t* __restrict__ item_seg, const uint32_t* __restrict__ item_ent,
    const int32_t* __restrict__ item_dst, const uint32_t* __restrict__ seg_ptr,
    const int32_t* __restrict__ seg_j, const Entry* __restrict__ ent, int64_t n_items,
    const float* __restrict__ B, const float* __restrict__ C, float* __restrict__ A,
    float* __restrict__ partials, int R, int team_log) {
  using V = typename Vec<VEC>::type;
  constexpr uint32_t G = 64 / LPR;
  constexpr int WPB = kBlock / 64;
  __shared__ __attribute__((aligned(16))) Entry s_ent[WPB][kCsfItemNnz];
  __shared__ uint16_t s_ptr[WPB][kCsfItemSegs + 2];     // (16 bits: the eighth workgroup then fits the compute unit)
  __shared__ int32_t s_j[WPB][kCsfItemSegs];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  // 1 << team_log wavefronts share an item (the last workgroup's may have none)
  const int64_t slot = ((int64_t)blockIdx.x * WPB + wave) >> team_log;
  const int team = 1 << team_log, part = wave & (team - 1);
  int64_t it = slot;
  if (slot >= n_items) {
    if (team == 1) return;                              // whole wavefront leaves together
    it = n_items - 1;
  }
  uint32_t s_lo = item_seg[it], e_lo = item_ent[it];
  uint32_t n_seg = item_seg[it + 1] - s_lo, n_ent = item_ent[it + 1] - e_lo;
  const int32_t dst = item_dst[it];
  // An item beyond what the staging arrays hold cannot come out of csf3_build, which is the one
  // place that enforces the limits; if an image ever carried one, its destination row is filled
  // with NaN (a result that announces itself) instead of being left with whatever it held.
  const bool over_limit = n_seg > (uint32_t)kCsfItemSegs || n_ent > (uint32_t)kCsfItemNnz;
  if (over_limit) { n_seg = 0; n_ent = 0; }
  if (!TOGETHER && team > 1) {          // this wavefront's share of the segments
    const uint32_t first = n_seg * part >> team_log, last = n_seg * (part + 1) >> team_log, s_item = s_lo;
    const uint32_t e_end = last < n_seg ? seg_ptr[s_item + last] : e_lo + n_ent;
    if (first > 0) e_lo = seg_ptr[s_item + first];
    s_lo += first;
    n_seg = last - first;
    n_ent = e_end - e_lo;
  }
  const uint32_t lane = threadIdx.x % 64;
  const uint32_t g = lane / LPR;
  const LaneColumns lc = lane_columns<VEC>(lane % LPR, blockIdx.y * (LPR * VEC), R);
  const int at = TOGETHER ? 0 : wave;
  const ItemView v{s_ent[at], s_ptr[at], s_j[at], reinterpret_cast<const char*>(B),
                   reinterpret_cast<const char*>(C), 4u * (uint32_t)R, lc.ok ? 4u * (uint32_t)lc.c : 0u};
  // stage the item, the loads of up to 128 segments and 256 entries before the first wait
  static_assert(kCsfItemSegs == 128 && kCsfItemNnz == 512, "the staging covers these sizes");
  if constexpr (TOGETHER) {
    const uint32_t me = threadIdx.x;
    Entry e[kCsfItemNnz / kBlock];
    uint32_t pt = 0;
    int32_t jt = 0;
    if (me < n_seg) { pt = stream_load(&seg_ptr[s_lo + me]); jt = stream_load(&seg_j[s_lo + me]); }
#pragma unroll
    for (uint32_t q = 0; q < kCsfItemNnz / kBlock; ++q) if (me + q * kBlock < n_ent) e[q] = stream_load(&ent[e_lo + me + q * kBlock]);
    if (me < n_seg) { s_ptr[0][me] = (uint16_t)(pt - e_lo); s_j[0][me] = jt; }
    if (me == 0) s_ptr[0][n_seg] = (uint16_t)n_ent;
#pragma unroll
    for (uint32_t q = 0; q < kCsfItemNnz / kBlock; ++q) if (me + q * kBlock < n_ent) s_ent[0][me + q * kBlock] = e[q];
    __syncthreads();
  } else {
    Entry e[4];
    uint32_t pt[2];
    int32_t jt[2];
#pragma unroll
    for (uint32_t q = 0; q < 2; ++q)
      if (lane + q * 64 < n_seg) { pt[q] = stream_load(&seg_ptr[s_lo + lane + q * 64]); jt[q] = stream_load(&seg_j[s_lo + lane + q * 64]); }
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) if (lane + q * 64 < n_ent) e[q] = stream_load(&ent[e_lo + lane + q * 64]);
#pragma unroll
    for (uint32_t q = 0; q < 2; ++q)
      if (lane + q * 64 < n_seg) { s_ptr[wave][lane + q * 64] = (uint16_t)(pt[q] - e_lo); s_j[wave][lane + q * 64] = jt[q]; }
    if (lane == 0) s_ptr[wave][n_seg] = (uint16_t)n_ent;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) if (lane + q * 64 < n_ent) s_ent[wave][lane + q * 64] = e[q];
    if (n_ent > 256) {
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) if (lane + (q + 4) * 64 < n_ent) e[q] = stream_load(&ent[e_lo + lane + (q + 4) * 64]);
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) if (lane + (q + 4) * 64 < n_ent) s_ent[wave][lane + (q + 4) * 64] = e[q];
    }
  }
  strip_sync();
  V acc = vzero<VEC>();
  uint32_t s = 0;
  if constexpr (TOGETHER) {                             // this wavefront's share of the segments
    s = n_seg * part / WPB;
    n_seg = n_seg * (part + 1) / WPB;
  }
  while (s < n_seg) {
    // lengths of the next 64 segments, one per lane; the first is the longest of them
    const uint32_t mine = s + lane < n_seg ? (uint32_t)v.ptr[s + lane + 1] - (uint32_t)v.ptr[s + lane] : 0u;
    const uint32_t len = (uint32_t)__builtin_amdgcn_readfirstlane((int)mine);
    const unsigned long long alike = __ballot(mine == len);
    auto take = [&](auto Pc, auto Uc) {
      constexpr int P = decltype(Pc)::value, U = decltype(Uc)::value;
      constexpr uint32_t N = P * G;                 // at most 64
      constexpr unsigned long long mask = ~0ULL >> (64 - N);
      if ((alike & mask) == mask) segments<VEC, LPR, P, U, SMALL, true>(v, s, n_seg, len, g, acc);
      else segments<VEC, LPR, P, U, SMALL, false>(v, s, n_seg, len, g, acc);
      s += N;
    };
    using std::integral_constant;
    constexpr int P4 = LPR >= 4 ? 4 : LPR, P2 = LPR >= 2 ? 2 : LPR;
    if (len == 1) take(integral_constant<int, P4>{}, integral_constant<int, 1>{});
    else if (len == 2) take(integral_constant<int, P2>{}, integral_constant<int, 2>{});
        else take(integral_constant<int, 1>{}, integral_constant<int, 4>{});
  }
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1) vadd(acc, vshfl_xor(acc, m));
  if (team > 1) {
    // each wavefront's sum in the memory of its own entries, which it has read (TOGETHER: which no entries are in)
    strip_sync();
    if (part > 0 && g == 0) vstore<VEC>(reinterpret_cast<float*>(s_ent[wave]) + lane * VEC, acc);
    __syncthreads();
    if (part > 0 || slot >= n_items) return;
    for (int w = 1; w < team; ++w) vadd(acc, vload<VEC>(reinterpret_cast<const float*>(s_ent[wave + w]) + lane % LPR * VEC));
  }
  if (over_limit) vfma(acc, __builtin_nanf(""), acc);
  if (g == 0 && lc.ok)
    gstore<VEC>(dst >= 0 ? A + (size_t)dst * (size_t)R + lc.c : partials + (size_t)(-1 - dst) * (size_t)R + lc.c, acc);
}

// ---------------------------------------------------------------------------------------------------------
// resident kernel: both factors in LDS, four or eight columns at a time.  A workgroup copies its columns of all rows
// of C and B (16 bytes a row and four columns, at most 10200 of them) and keeps them while its sixteen wavefronts go through
// items.  A lane owns a segment: in every step it reads one row of C from LDS and adds it, times the value, to
// the segment's sum, until the step that multiplies the sum by the row of B.  All lanes of a batch do this in
// the same step, so the choice is a scalar one; the image holds the offsets and values in this order (ResidentBlock), so
// the entries come with coalesced 16-byte loads and no lane waits for anything but LDS.
//
// Why: with the rows gathered from the L2 an entry moves 4 R bytes over the path of 64 bytes per cycle into the
// compute unit; from LDS they come twice as fast, random 16-byte rows at 51 TB/s against 26.  The price is
// that the entries are read R / 4 times, 6 bytes a step; the workgroups of one die that
// differ in their columns go through the same items at the same time, so that 95 % of these loads hit the L2.
// Uniform 4096^3 tensor, 68.7 M entries in 16.5 M fibres: R = 64 850 -> 443 us, R = 8 378 -> 107, R = 128 1636 ->
// 822.  What bounds it is what comes back to the registers, 16 bytes of a row and 6 of the image per lane and
// step: 943 k cycles at 128 bytes a cycle, of 955 k that pass.  LDS works 735 k of them (bank conflicts included; an order of the
// entries with a third fewer of those gained 1 %), the vector units 625 k.  Entry and offset as a pair of eight bytes
// per step: 593 us.  Rows of the next half block read from LDS ahead of the sums: 465 us (smaller tensors gained 1 to 2 %).
//
// Where items are short, what an item ends with counts: its 64 sums were added with 24 shuffles through LDS, six latencies in
// a row, behind which the rows of the next block waited.  DPP operands and permlane swaps instead (the same sums), and
// two blocks on their way instead of three: 3000 x 500 x 2500, 3.75 M entries, R = 96: 68.2 -> 56.9 us; 1300^3, 2.2 M,
// R = 64: 31.0 -> 26.7; 1000 x 2000 x 3000, 6 M, R = 32: 29.2 -> 27.5; 4096^3, R = 64: 450.6 -> 448.0.  What items are left
// after whole turns of all wavefronts are spread over the workgroups, not given to the first of them: 2100 x 1500 x 2000, 6.3 M,
// R = 8: 18.2 -> 16.0; 900 x 2000 x 3000, 5.4 M, R = 9: 15.6 -> 13.8; 700 x 2000 x 1500, 2.1 M, R = 100: 34.9 -> 32.8.
//
// Half as many rows fit with eight columns of each, in two planes (the banks of a step stay those that the image was ordered
// for): 38 bytes come back for eight columns instead of 44, and the offsets are taken apart once.  Fewer rows read ahead of the
// sums are better, the other wavefronts of a SIMD fill the wait: eight columns, rows of 4 / 2 / 1 steps together: 4096 x 2500 x
// 2500 of 25.6 M, R = 64, 165.3 / 161.3 / 150.5 us (four columns: 8 / 4 / 2 steps 170.6 / 166.9 / 172.3; 4096^3 453.0 / 449.8 /
// 466.4, and with a third block on its way 443.6).  Eight sums of an item are reduced together, halving what a lane holds with every
// exchange (some 30 instructions instead of 96), and the steps that fill up its last block are left out, which are half a block on average (both for
// eight columns only): 3000 x 500 x
// 2500, R = 96, 48.0 -> 44.9 us; 4000 x 1000 x 1000, 128, 72.3 -> 67.6; 2734 x 640 x 509 of 890 K, 96, 24.3 -> 20.4 (some of it by the choice between four and eight).
//
// The scheduler prefers the oldest wavefronts of a SIMD; of the longest shares the first were through after 394 of 430 us.  With priorities that fall with
// every quarter of their items they stay together, and what they read of the image (the form with a third block on its way; both sides timed in turn on two
// cards, runs of one side 0.1 to 0.2 % apart): 4096^3, R = 64, 443.5 -> 439.7 and 446.1 -> 442.8; R = 128, 823.3 -> 818.6 and 828.1 -> 825.1; 4000^3 of 50 M,
// R = 100, 521.7 -> 518.8 and 524.9 -> 522.4.
// (A barrier after every item: 467.  Windows of B, five of them, so that eight columns fit for 4096^3: R = 64 415, but R = 4 / 12 / 20 97 -> 107, 139 -> 157, 190 -> 214 us;
// batches of a window mix the lengths of more segments, which takes 5 to 8 % more steps, and there is one image for all ranks.)
// ---------------------------------------------------------------------------------------------------------
constexpr int kResidentBlock = 1024;

// One step: a record of a batch adds its row to the sums of the fibres, the one that ends it adds their products
// with the row of B to acc.  The bit is the same for the whole wavefront; written out because the compiler
// turned the choice into sixteen register moves a step.
template <int BIT>
__device__ __forceinline__ void resident_step(float4 (&acc)[1], float4 (&x)[1], uint32_t bits, float v, const float4 (&c)[1]) {
  asm volatile(
      "s_bitcmp1_b32 %[m], %[bit]\n\t"
      "s_cbranch_scc1 1f\n\t"
      "v_fmac_f32 %[x0], %[v], %[c0]\n\t"
      "v_fmac_f32 %[x1], %[v], %[c1]\n\t"
      "v_fmac_f32 %[x2], %[v], %[c2]\n\t"
      "v_fmac_f32 %[x3], %[v], %[c3]\n\t"
      "s_branch 2f\n"
      "1:\n\t"
      "v_fmac_f32 %[a0], %[x0], %[c0]\n\t"
      "v_fmac_f32 %[a1], %[x1], %[c1]\n\t"
      "v_fmac_f32 %[a2], %[x2], %[c2]\n\t"
      "v_fmac_f32 %[a3], %[x3], %[c3]\n\t"
      "v_mov_b32 %[x0], 0\n\t"
      "v_mov_b32 %[x1], 0\n\t"
      "v_mov_b32 %[x2], 0\n\t"
      "v_mov_b32 %[x3], 0\n"
      "2:"
      : [x0] "+v"(x[0].x), [x1] "+v"(x[0].y), [x2] "+v"(x[0].z), [x3] "+v"(x[0].w),
        [a0] "+v"(acc[0].x), [a1] "+v"(acc[0].y), [a2] "+v"(acc[0].z), [a3] "+v"(acc[0].w)
      : [m] "s"(bits), [bit] "n"(BIT), [v] "v"(v), [c0] "v"(c[0].x), [c1] "v"(c[0].y), [c2] "v"(c[0].z), [c3] "v"(c[0].w)
      : "scc");
}
template <int BIT>
__device__ __forceinline__ void resident_step(float4 (&acc)[2], float4 (&x)[2], uint32_t bits, float v, const float4 (&c)[2]) {
  asm volatile(
      "s_bitcmp1_b32 %[m], %[bit]\n\t"
      "s_cbranch_scc1 1f\n\t"
      "v_fmac_f32 %[x0], %[v], %[c0]\n\t"
      "v_fmac_f32 %[x1], %[v], %[c1]\n\t"
      "v_fmac_f32 %[x2], %[v], %[c2]\n\t"
      "v_fmac_f32 %[x3], %[v], %[c3]\n\t"
      "v_fmac_f32 %[x4], %[v], %[c4]\n\t"
      "v_fmac_f32 %[x5], %[v], %[c5]\n\t"
      "v_fmac_f32 %[x6], %[v], %[c6]\n\t"
      "v_fmac_f32 %[x7], %[v], %[c7]\n\t"
      "s_branch 2f\n"
      "1:\n\t"
      "v_fmac_f32 %[a0], %[x0], %[c0]\n\t"
      "v_fmac_f32 %[a1], %[x1], %[c1]\n\t"
      "v_fmac_f32 %[a2], %[x2], %[c2]\n\t"
      "v_fmac_f32 %[a3], %[x3], %[c3]\n\t"
      "v_fmac_f32 %[a4], %[x4], %[c4]\n\t"
      "v_fmac_f32 %[a5], %[x5], %[c5]\n\t"
      "v_fmac_f32 %[a6], %[x6], %[c6]\n\t"
      "v_fmac_f32 %[a7], %[x7], %[c7]\n\t"
      "v_mov_b32 %[x0], 0\n\t"
      "v_mov_b32 %[x1], 0\n\t"
      "v_mov_b32 %[x2], 0\n\t"
      "v_mov_b32 %[x3], 0\n\t"
      "v_mov_b32 %[x4], 0\n\t"
      "v_mov_b32 %[x5], 0\n\t"
      "v_mov_b32 %[x6], 0\n\t"
      "v_mov_b32 %[x7], 0\n"
      "2:"
      : [x0] "+v"(x[0].x), [x1] "+v"(x[0].y), [x2] "+v"(x[0].z), [x3] "+v"(x[0].w),
        [x4] "+v"(x[1].x), [x5] "+v"(x[1].y), [x6] "+v"(x[1].z), [x7] "+v"(x[1].w),
        [a0] "+v"(acc[0].x), [a1] "+v"(acc[0].y), [a2] "+v"(acc[0].z), [a3] "+v"(acc[0].w),
        [a4] "+v"(acc[1].x), [a5] "+v"(acc[1].y), [a6] "+v"(acc[1].z), [a7] "+v"(acc[1].w)
      : [m] "s"(bits), [bit] "n"(BIT), [v] "v"(v), [c0] "v"(c[0].x), [c1] "v"(c[0].y), [c2] "v"(c[0].z), [c3] "v"(c[0].w),
        [c4] "v"(c[1].x), [c5] "v"(c[1].y), [c6] "v"(c[1].z), [c7] "v"(c[1].w)
      : "scc");
}

constexpr int kResidentGroups = 256;     // workgroups: one per compute unit, which holds one window of rows
// A third block on its way, four columns at a time: gains where both a wavefront's share and its items are long (two / three blocks, us, by
// steps a wavefront and blocks an item: 6147, 24: 489.5 / 479.7; 5382, 42: 449.6 / 448.2), not in shorter shares (4075, 32: 343.7 / 343.9; 3074, 24: 255.7
// / 258.0; 2691, 42: 250.2 / 255.3) or items (6647, 13: 477.6 / 480.3; 5973, 12: 420.1 / 423.6; 4725, 16: 337.0 / 338.0).
constexpr int kResidentLong = 4096, kResidentLongItem = 20;
// Blocks of an item on average from which on four of them are a chain of additions, below that two.  Error against 64 bits with two / four, 1e-7
// of the norm: 13 blocks 0.99 / 1.04, 16 0.96 / 1.01, 24 1.02 / 1.05, 32 1.04 / 1.06, 42 1.08 / 1.07 and 1.12 / 1.08 (the other kernel, R = 12 / 64: 0.94 to 1.03 /
// 0.97 to 1.38); four are up to 1 % faster.  By the image alone: a column of A does not depend on the number of columns.
constexpr int kResidentChain = 32;

// P: quads of columns of a workgroup, each in a plane of its own of all rows; UR: steps whose rows are read together; N: blocks
// on their way; CHAIN: blocks whose additions are a chain (as an argument of the launch it cost 4096^3 half a percent).
template <int P, int UR, int N, uint32_t CHAIN>
__global__ __launch_bounds__(kResidentBlock) void resident_kernel(
    const ResidentItem* __restrict__ items, const ResidentBlock* __restrict__ blocks, const uint32_t* __restrict__ last, int n_items,
    const float* __restrict__ B, int J, const float* __restrict__ C, int K, float* __restrict__ A,
    float* __restrict__ partials, int R, int slices, int replicas) {
  __shared__ float4 s_row[kCsfRowsInLds];
  const int per_die = gridDim.x / 8, q = (int)(blockIdx.x % 8) * per_die + (int)(blockIdx.x / 8);
  if (q >= slices * replicas) return;
  const int rows = K + 1 + J;                           // (P planes of them fit, the launch sees to that)
  const int slice = q % slices, c0 = R >= 4 * P ? min(4 * P * slice, R - 4 * P) : 0;
  auto copy = [&](const float* M, int r, int at) {
    const float* p = M + (size_t)r * (size_t)R + c0;
    if (P > 1 || R >= 4) {
      float4 v[P];
#pragma unroll
      for (int e = 0; e < P; ++e) v[e] = gload<4>(p + 4 * e);
#pragma unroll
      for (int e = 0; e < P; ++e) s_row[e * rows + at] = v[e];
    } else {
      s_row[at] = make_float4(p[0], R > 1 ? p[1] : 0.f, R > 2 ? p[2] : 0.f, 0.f);
    }
  };
  for (int r = threadIdx.x; r < K; r += kResidentBlock) copy(C, r, r);
  for (int r = threadIdx.x; r < J; r += kResidentBlock) copy(B, r, K + 1 + r);
  if (threadIdx.x < P) s_row[threadIdx.x * rows + K] = vzero<4>();
  __syncthreads();
  const char* lds = reinterpret_cast<const char*>(s_row);
  const uint32_t plane = (uint32_t)rows * (uint32_t)sizeof(float4);
  constexpr int U = kCsfBlockSteps;
  static_assert(U == 8, "the steps of a block");
  const uint32_t lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  const int workers = replicas * (kResidentBlock / 64);
  int it = wave * replicas + q / slices;                // what is left after whole turns goes to all workgroups
  if (it >= n_items) return;
  // The blocks of this wavefront's items as one sequence, N of them on their way: `f` is the item that is
  // fetched from, `d` the one that is summed; what follows an item is loaded while there is time.
  auto item = [&](int i) { return items[min(i, n_items - 1)]; };
  // (for the eight columns, whose steps are read one by one; in front of the second half of a block, four columns lost 2 to 4 % by the branch)
  auto steps = [&](int i) { return P == 2 && last ? (int)last[min(i, n_items - 1)] : U; };
  int d_last = steps(it);
  ResidentItem d = item(it), d_next = item(it + workers), f = d, f_next = d_next;
  int f_it = it;
  const ResidentBlock* p = blocks + f.block;
  uint4 of[N];
  float4 lo[N], hi[N];
  auto fetch = [&](int h) {
    of[h] = *reinterpret_cast<const uint4*>(&p->offsets[lane]);
    lo[h] = *reinterpret_cast<const float4*>(&p->values[0][lane]);
    hi[h] = *reinterpret_cast<const float4*>(&p->values[1][lane]);
    ++p;
    if (--f.blocks == 0) {
      f = f_next;
      f_it = min(f_it, n_items) + workers;
      f_next = item(f_it + workers);
      p = blocks + f.block;
    }
  };
#pragma unroll
  for (int h = 0; h < N; ++h) fetch(h);
  float4 sum[P], part[P], acc[P], x[P];
#pragma unroll
  for (int e = 0; e < P; ++e) sum[e] = part[e] = acc[e] = x[e] = vzero<4>();
  auto store = [&] {
    if constexpr (P == 2) {
      const float v[8] = {sum[0].x, sum[0].y, sum[0].z, sum[0].w, sum[1].x, sum[1].y, sum[1].z, sum[1].w};
      const float total = wave_sum8(v, (int)lane);
      float* out = (d.dst >= 0 ? A + (size_t)d.dst * (size_t)R : partials + (size_t)(-1 - d.dst) * (size_t)R) + c0;
      if (lane < 8) out[4 * (lane & 1) + (lane & 2) + (lane >> 2)] = total;
      sum[0] = sum[1] = vzero<4>();
      return;
    }
#pragma unroll
    for (int e = 0; e < P; ++e) sum[e] = make_float4(wave_sum(sum[e].x), wave_sum(sum[e].y), wave_sum(sum[e].z), wave_sum(sum[e].w));
    if (lane == 0) {
      float* out = (d.dst >= 0 ? A + (size_t)d.dst * (size_t)R : partials + (size_t)(-1 - d.dst) * (size_t)R) + c0;
      if (P > 1 || R >= 4) {
#pragma unroll
        for (int e = 0; e < P; ++e) gstore<4>(out + 4 * e, sum[e]);
      } else {
        out[0] = sum[0].x;
        if (R > 1) out[1] = sum[0].y;
        if (R > 2) out[2] = sum[0].z;
      }
    }
#pragma unroll
    for (int e = 0; e < P; ++e) sum[e] = vzero<4>();
  };
  const int first = it, quarter = (n_items - it + 3) / 4;    // (N == 3: the longest shares)
  if (N == 3) __builtin_amdgcn_s_setprio(3);
  while (true) {
#pragma unroll
    for (int h = 0; h < N; ++h) {
      const uint32_t w[4] = {of[h].x, of[h].y, of[h].z, of[h].w};
      const float v[U] = {lo[h].x, lo[h].y, lo[h].z, lo[h].w, hi[h].x, hi[h].y, hi[h].z, hi[h].w};
      uint32_t ends[U / 2];
#pragma unroll
      for (int u0 = 0; u0 < U; u0 += UR) {
        if (P == 2 && u0 > 0 && u0 % 2 == 0 && d.blocks == 1 && u0 >= d_last) break;
        float4 c[UR][P];
#pragma unroll
        for (int u = u0; u < u0 + UR; ++u)
#pragma unroll
          for (int e = 0; e < P; ++e)
            c[u - u0][e] = *reinterpret_cast<const float4*>(lds + ((u % 2 ? w[u / 2] >> 14 : w[u / 2]) & 0x3fff0u) + e * plane);
        if (u0 == 0) {
#pragma unroll
          for (int u = 0; u < U / 2; ++u) ends[u] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[u]);
        }
#pragma unroll
        for (int u = u0; u < u0 + UR; ++u) {
          if (u % 2 == 0) resident_step<0>(acc, x, ends[u / 2], v[u], c[u - u0]);
          else resident_step<1>(acc, x, ends[u / 2], v[u], c[u - u0]);
        }
      }
      fetch(h);
      if (--d.blocks % CHAIN == 0) {                    // short chains of additions: as exact as the other kernel
#pragma unroll
        for (int e = 0; e < P; ++e) {
          vadd(part[e], acc[e]);
          acc[e] = vzero<4>();
        }
        if (d.blocks % (4 * CHAIN) == 0) {
#pragma unroll
          for (int e = 0; e < P; ++e) {
            vadd(sum[e], part[e]);
            part[e] = vzero<4>();
          }
        }
      }
      if (d.blocks == 0) {
        store();
        it += workers;
        if (N == 3) {
          if (it - first >= 3 * quarter) __builtin_amdgcn_s_setprio(0);
          else if (it - first >= 2 * quarter) __builtin_amdgcn_s_setprio(1);
          else if (it - first >= quarter) __builtin_amdgcn_s_setprio(2);
        }
        if (it >= n_items) return;
        d = d_next;
        d_last = steps(it);
        d_next = item(it + workers);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// streams kernel: sums in LDS, entries in the order of one factor's rows.  Where slices are small and the factors do
// not fit an L2, rows of B and C come from behind it whatever the order of the slices: what is in flight at a
// time touches more rows than an L2 holds.  Here a wavefront owns up to 71 rows of A for the whole launch, so its
// entries may come in any order, and all wavefronts go through the rows of one factor together, window by window: a
// part of that factor is in the L2 while everyone needs it, and the rest of the L2 is left to the other factor.  The scheduler
// prefers a compute unit's older wavefronts; a barrier every 32 entries of a lane group keeps them in step
// (338 -> 288 us with sums in 32 bits).  Sixteen wavefronts of 10 KiB fill the LDS.  Records are taken from LDS, rows of four
// entries per lane group are on their way while four others are added.
//
// A sum in LDS is read when its row comes up and written after every entry; what follows of the row meanwhile is
// added in 64 bits, whose additions and products take no longer here than those of 32: rounded once per run of a
// row's entries, not per entry (in 32 bits with chains of 8 and 32 entries 290 us instead of 293, but the error
// below was 0.85e-7).
//
// Skewed 512k x 64k x 64k tensor, 16.8 M entries, R = 32: 506 -> 293 us; 40 % of the requests miss the L2 instead of 68 %,
// 1.84 GB instead of 3.3, which still bounds it (6.3 TB/s).  R = 128: 2164 -> 1170.  Rows that are no whole
// lines touch more of them than they need to in every slice of columns: laid out anew (slices_kernel, 33 MB in
// 15 us) R = 50 takes 644 instead of 1353 us, in the other form 1136.  Error against 64 bits, R = 32: 2-norm
// 0.82 -> 0.61e-7, largest over root mean square 4.2 -> 1.6e-5; 400k x 2000 x 2000 uniform, R = 25: 0.60 -> 0.54e-7.
// ---------------------------------------------------------------------------------------------------------
constexpr int kStreamBlock = 64 * kCsfStreamTeam;

template <int VEC, bool SMALL, bool SHARED>
__global__ __launch_bounds__(kStreamBlock) void streams_kernel(
    const StreamWave* __restrict__ waves, const StreamBlock* __restrict__ blocks, const int32_t* __restrict__ dsts,
    const int32_t* __restrict__ zero_rows, int64_t n_waves, const float* __restrict__ B, const float* __restrict__ C,
    float* __restrict__ A, float* __restrict__ partials, int R, int stride, int64_t slice_floats) {
  using V = typename Vec<VEC>::type;
  constexpr uint32_t LPR = 8;
  constexpr int WPB = kStreamBlock / 64, U = 4;        // U: entries of a lane group whose rows are loaded together
  __shared__ V s_sum[WPB][(kCsfStreamRows + 1) * LPR];
  __shared__ uint4 s_rec[WPB][64];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  const int64_t w = (int64_t)blockIdx.x * WPB + wave;
  if (w >= n_waves) return;
  const StreamWave d = waves[w];
  const uint32_t lane = threadIdx.x % 64, g = lane / LPR, l = lane % LPR;
  // this lane's columns: a part of them may lie beyond R in factors laid out anew; in the caller's (SHARED) such a
  // lane is moved back and holds columns of the one before it as well (R >= VEC)
  int c = (int)(blockIdx.y * LPR + l) * VEC;
  const bool ok = c < R;
  if (SHARED && ok) c = min(c, R - VEC);
  const uint32_t row_bytes = 4u * (uint32_t)stride, col_bytes = ok ? 4u * (SHARED ? (uint32_t)c : l * VEC) : 0u;
  const char* Bc = reinterpret_cast<const char*>(B + (int64_t)blockIdx.y * slice_floats);
  const char* Cc = reinterpret_cast<const char*>(C + (int64_t)blockIdx.y * slice_floats);
  V* sums = s_sum[wave] + l;
#pragma unroll
  for (uint32_t r = 0; r < (kCsfStreamRows + 1) / 8; ++r) sums[(r * 8 + g) * LPR] = vzero<VEC>();
  strip_sync();
  struct Batch { V b[U], c[U]; float val[U]; uint32_t at[U]; } q[2];
  double acc[VEC] = {};
  uint32_t prev = ~0u;
  auto issue = [&](Batch& t, int s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint4 r = s_rec[wave][g * 8 + s0 + u];
      t.at[u] = (r.x & 127u) * LPR;
      t.val[u] = __uint_as_float(r.z);
      t.b[u] = load_row<VEC, SMALL>(Bc, (int32_t)(r.x >> 7), row_bytes, col_bytes);
      t.c[u] = load_row<VEC, SMALL>(Cc, (int32_t)r.y, row_bytes, col_bytes);
    }
  };
  auto sum = [&](const Batch& t) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const V old = sums[t.at[u]];
      const bool other = t.at[u] != prev;
      prev = t.at[u];
      float was[VEC], b[VEC], x[VEC], now[VEC];
      V p = vzero<VEC>();
      vfma(p, t.val[u], t.c[u]);
      __builtin_memcpy(was, &old, sizeof was);
      __builtin_memcpy(b, &t.b[u], sizeof b);
      __builtin_memcpy(x, &p, sizeof x);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        acc[e] = fma((double)x[e], (double)b[e], other ? (double)was[e] : acc[e]);
        now[e] = (float)acc[e];
      }
      __builtin_memcpy(&sums[t.at[u]], now, sizeof now);
    }
  };
  StreamBlock::Record next;
  auto load = [&](uint32_t n) {
    const StreamBlock::Record* p = &blocks[d.block + min(n, d.blocks - 1)].rec[lane];
    return StreamBlock::Record{stream_load(&p->j_slot), stream_load(&p->k), stream_load(&p->val)};
  };
  auto put = [&] { s_rec[wave][lane] = make_uint4(next.j_slot, (uint32_t)next.k, __float_as_uint(next.val), 0u); };
  if (d.blocks > 0) {
    next = load(0);
    put();
    strip_sync();
    next = load(1);
    issue(q[0], 0);
    for (uint32_t n = 0; n < d.blocks; ++n) {
      issue(q[1], U);
      strip_sync();
      put();
      strip_sync();
      next = load(n + 2);
      sum(q[0]);
      if (n + 1 < d.blocks) issue(q[0], 0);
      sum(q[1]);
      if ((n + 1) % kCsfStreamTurn == 0) __builtin_amdgcn_s_barrier();      // (nothing is handed over)
    }
  }
  for (uint32_t n = d.blocks / kCsfStreamTurn; n < d.turns; ++n) __builtin_amdgcn_s_barrier();
  strip_sync();
  auto store = [&](float* row, V v) {
    if (c + VEC <= R) { vstore_stream<VEC>(row + c, v); return; }
    float f[VEC];
    __builtin_memcpy(f, &v, sizeof f);
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      if (c + e < R) row[c + e] = f[e];
  };
#pragma unroll
  for (uint32_t r = 0; r < (kCsfStreamRows + 1) / 8; ++r) {
    const uint32_t slot = r * 8 + g;
    const int32_t dst = slot < (uint32_t)kCsfStreamRows ? dsts[w * kCsfStreamRows + slot] : kCsfNoRow;
    if (dst != kCsfNoRow) store(dst >= 0 ? A + (size_t)dst * (size_t)R : partials + (size_t)(-1 - dst) * (size_t)R, sums[slot * LPR]);
  }
  for (uint32_t z = g; z < d.zeros; z += 8) store(A + (size_t)zero_rows[d.zero + z] * (size_t)R, vzero<VEC>());
}

// Rows of B, then of C, in slices of `width` columns one after the other; zeros in the columns from R on.
__global__ __launch_bounds__(kBlock) void slices_kernel(const float* __restrict__ B, int64_t J, const float* __restrict__ C,
                                                        int64_t K, int R, int width, float4* __restrict__ out, int64_t n) {
  const int64_t at = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (at >= n) return;
  const int quads = width / 4;
  const int64_t row = at / quads % (J + K);
  const int c = (int)(at / quads / (J + K)) * width + (int)(at % quads) * 4;
  const float* p = row < J ? B + row * R : C + (row - J) * R;
  float4 v = vzero<4>();
  if (c + 4 <= R) v = gload<4>(p + c);
  else {
    if (c < R) v.x = p[c];
    if (c + 1 < R) v.y = p[c + 1];
    if (c + 2 < R) v.z = p[c + 2];
  }
  out[at] = v;
}

}  // namespace

int launch_mttkrp_streams(const StreamWave* waves, const StreamBlock* blocks, const int32_t* dst, const int32_t* zero_rows,
                          int64_t n_waves, const float* B, int64_t b_rows, const float* C, int64_t c_rows, float* A,
                          float* partials, float* scratch, int32_t R, void* stream) {
  if (n_waves <= 0) return 0;
  // Where rows are no whole lines of 128 bytes, or parts of one, the factors are laid out anew in slices that are,
  // if there is room for that.  (512k x 64k x 64k, R = 33 / 50 / 100: 609 / 644 / 1243 us, without room 996 / 1353 / 2525.)
  const int width = stream_slice(R), vec = width / 8;
  const int64_t slices = ceil_div(R, width);
  const bool lines = stream_lines(R), anew = scratch && !(lines && ((uintptr_t)B | (uintptr_t)C) % 128 == 0);
  const int stride = anew ? width : R;
  const bool small = small_matrix(b_rows, stride) && small_matrix(c_rows, stride), shared = !anew && !lines;
  int64_t slice_floats = shared ? 0 : width;             // (lanes that share columns count them from the row's first)
  if (anew) {
    const int64_t n = (b_rows + c_rows) * slices * width / 4, blocks = ceil_div(n, kBlock);
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(slices_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, (hipStream_t)stream, B, b_rows, C, c_rows, (int)R,
                       width, reinterpret_cast<float4*>(scratch), n);
    slice_floats = (b_rows + c_rows) * width;
    B = scratch;
    C = scratch + b_rows * width;
  }
  const int64_t groups = ceil_div(n_waves, kStreamBlock / 64);
  if (groups > 0x7fffffffLL || slices > 65535) return (int)hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)groups, (unsigned)slices);
#define ARROW_LAUNCH(V, SM, SH)                                                                                         \
  hipLaunchKernelGGL((streams_kernel<V, SM, SH>), grid, dim3(kStreamBlock), 0, (hipStream_t)stream, waves, blocks, dst, zero_rows, \
                     n_waves, B, C, A, partials, (int)R, stride, slice_floats)
#define ARROW_VEC(SM, SH) if (vec == 4) ARROW_LAUNCH(4, SM, SH); else if (vec == 2) ARROW_LAUNCH(2, SM, SH); else ARROW_LAUNCH(1, SM, SH)
#define ARROW_SHARED(SM) if (shared) { ARROW_VEC(SM, true); } else { ARROW_VEC(SM, false); }
  if (small) { ARROW_SHARED(true) } else { ARROW_SHARED(false) }
#undef ARROW_SHARED
#undef ARROW_VEC
#undef ARROW_LAUNCH
  return (int)hipGetLastError();
}

int launch_mttkrp_resident(const ResidentItem* items, const ResidentBlock* blocks, int64_t n_items, int64_t n_blocks,
                           const float* B, int64_t b_rows, const float* C, int64_t c_rows, float* A, float* partials,
                           int32_t R, void* stream, const uint32_t* last) {
  if (n_items <= 0) return 0;
  if (b_rows + c_rows + 1 > kCsfRowsInLds || n_items > INT_MAX) return (int)hipErrorInvalidValue;
  // Replicas: workgroups that share the items of a column slice.  One round of workgroups where the slices divide
  // the compute units well; else more of them, each of which copies the factors again, four rows in about
  // the time of a wavefront's step.  (1300^3, R = 520, 130 slices: 338 -> 218 us with three
  // workgroups per slice in two rounds.  Fewer items than workgroups: some of these copy for nothing, beside the others; no more workgroups than items took 0
  // to 1 % longer, 128 x 300 x 200 of 70 K, R = 3, 4.4 -> 4.6 us, 144 x 415 x 1945 of 116 K, 4.9 -> 5.0.)
  struct Split { int64_t slices, replicas; double cost; };
  const double copy = (double)((b_rows + c_rows) / 4), steps = (double)(n_blocks * kCsfBlockSteps);
  constexpr int64_t waves = kResidentBlock / 64;
  auto split = [&](int quads, double step, int64_t tail, double copied) {
    Split s{ceil_div(R, 4 * quads), 1, 0.0};
    double best = 0.0;
    // (more slices than four rounds hold: as many rounds as give each a workgroup.  Four / eight
    // columns, us, 2000 x 1000 x 1000 of 1 M: R = 5120 1129 / 1150, 6144 1355 / 1156, 8192 1803 / 1538)
    const int64_t most = std::max<int64_t>(4, ceil_div(s.slices, kResidentGroups));
    for (int64_t rounds = 1; rounds <= most; ++rounds) {
      const int64_t n = kResidentGroups * rounds / s.slices;
      if (n < 1) continue;
      const double cost = (double)rounds * (steps / (double)n + copy);
      if (best != 0.0 && cost >= best) continue;
      best = cost;
      s.replicas = n;
      // the items of a workgroup: `tail` of them at least in a last turn, of which each takes as long on its own
      const int64_t turns = n_items / (n * waves), rest = n_items - turns * n * waves;
      const int64_t load = turns * waves + (rest > 0 ? std::max(ceil_div(rest, n), tail) : 0);
      s.cost = (double)rounds * (step * (double)load * steps / (double)n_items + copied * copy);
    }
    return s;
  };
  // Eight columns at a time where the rows fit the LDS so: the entries are read half as often, and a step takes 1.78 times as long instead of
  // twice, less what an item saves, whose sums are reduced together and whose last block is not filled up: 0.8 of a block.  Half as many slices leave twice as many
  // wavefronts for the items, though, and a wavefront that has its SIMD to itself waits longer for each of its rows.  Both measured at 14,116 products with uniform
  // tensors of 200 to 4096 rows a side, R = 8 to 128, others than the numbers were chosen with: they take 0.16 % longer than the better of the two on average.  With 1.57 and
  // nothing by the item it was 0.29 % and 332 products lost more than 2 % against what was chosen before sums were reduced together (1.72, a tail of 10, a copy of 0.7: 0.80 %);
  // now 135 do and 1218 gain that much.  Four / eight columns, us: 4096 x 2500 x 2500 of 25.6 M, R = 64, 166 / 150; 4000 x 1000 x 1000 of 4 M, 128, 84.9 / 67.6;
  // 1606 x 528 x 1024 of 868 K, 64, 17.8 / 13.6; 3122 x 868 x 472 of 646 K, 17, 8.7 / 7.3; but long items 700 x 2000 x 1500 of 2.1 M, 100, 35.9 / 37.0; 679 x 1410 x 2131 of
  // 3.6 M, 64, 27.9 / 31.0; and few 1018 x 2781 x 1602 of 4.5 M, 16, 15.5 / 18.4; 487 x 2818 x 1884 of 2.6 M, 32, 16.6 / 19.8.
  // None of these takes more slices than one round holds; where eight columns do, the earlier numbers stand, all three.
  Split s = split(1, 1.0, 5, 0.6);
  bool two = false;
  if (R >= 8 && 2 * (b_rows + c_rows + 1) <= kCsfRowsInLds) {
    const Split t = ceil_div(R, 8) > kResidentGroups ? split(2, 1.72, 10, 0.7)
                                                          : split(2, 1.78 - 0.8 * (double)n_items / (double)n_blocks, 11, 0.6);
    two = t.cost < s.cost;
    if (two) s = t;
  }
  const int64_t groups = ceil_div(s.slices * s.replicas, 8) * 8;
  if (groups > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
#define ARROW_CHAIN(CHAIN, ...)                                                                                            \
  hipLaunchKernelGGL((resident_kernel<__VA_ARGS__, CHAIN>), dim3((unsigned)groups), dim3(kResidentBlock), 0, (hipStream_t)stream, items, blocks, \
                     last, (int)n_items, B, (int)b_rows, C, (int)c_rows, A, partials, (int)R, (int)s.slices, (int)s.replicas)
#define ARROW_LAUNCH(...) if (chain4) ARROW_CHAIN(4, __VA_ARGS__); else ARROW_CHAIN(2, __VA_ARGS__)
  const bool chain4 = n_blocks >= n_items * kResidentChain;
  const bool third = steps >= (double)(s.replicas * waves) * kResidentLong && n_blocks >= n_items * kResidentLongItem;
  if (two) { ARROW_LAUNCH(2, 1, 2); }
  else if (third) { ARROW_LAUNCH(1, 4, 3); }
  else { ARROW_LAUNCH(1, 4, 2); }
#undef ARROW_CHAIN
#undef ARROW_LAUNCH
  return (int)hipGetLastError();
}

int launch_mttkrp(const uint32_t* item_seg, const uint32_t* item_ent, const int32_t* item_dst,
                  const uint32_t* seg_ptr, const int32_t* seg_j, const Entry* entries, int64_t n_items, const float* B,
                  int64_t b_rows, const float* C, int64_t c_rows, float* A, float* partials, int32_t R,
                  int32_t longest, int32_t average, void* stream) {
  if (n_items <= 0) return 0;
  const Shape s = pick_shape(R, 0);
  // Few items leave most wavefront slots empty, and the longest chain of row loads decides: wavefronts of a
  // workgroup then share an item and add up in LDS.  Four where they all find a slot on the chip (250 x 231
  // x 307 tensor of 17,720 entries, R = 25: 8.4 -> 6.9 us), two where two of them do and a lane group has
  // more than a few rows to go through (1322 x 161 x 3035 of 646 K, R = 32, 45 rows: 17.0 -> 14.3 us; 1704 x
  // 389 x 887 of 588 K, R = 14, 20 rows: 11.6 -> 11.9).  Four again where items are few enough for a slot
  // each and the longest are much longer than most (hub slices, skewed 5882 x 1176 x 588 of 188 K, R = 30:
  // 21.3 -> 17.5 us).
  const int64_t chain = (int64_t)longest * s.lpr / 64;   // rows one after the other in a lane group
  int team_log = 0;
  if (n_items <= kResidentItems / 4) team_log = 2;
  else if (n_items <= kResidentItems && chain >= 64 && longest > 4 * average) team_log = 2;
  else if (n_items <= kResidentItems / 2 && chain >= 32) team_log = 1;
  const bool small = small_matrix(b_rows, R) && small_matrix(c_rows, R);
  return dispatch_shape(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value;
    const int64_t blocks = ceil_div(n_items << team_log, kBlock / 64);
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)blocks, (unsigned)s.slices);
    const bool together = small && n_items <= kResidentItems / 4;      // (four wavefronts an item)
#define ARROW_LAUNCH(SM, TOGETHER)                                                                  \
  hipLaunchKernelGGL((mttkrp_kernel<VEC, LPR, SM, TOGETHER>), grid, dim3(kBlock), 0, (hipStream_t)stream,     \
                     item_seg, item_ent, item_dst, seg_ptr, seg_j, entries, n_items, B, C, A, partials, (int)R, team_log)
    if (together) ARROW_LAUNCH(true, true); else if (small) ARROW_LAUNCH(true, false); else ARROW_LAUNCH(false, false);
#undef ARROW_LAUNCH
    return (int)hipGetLastError();
  });
}

}  // namespace arrow
