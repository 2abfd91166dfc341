// HIP kernels for gfx950 (CDNA4, 64-wide wavefronts) of the arrow SpMM
//     Y = sum_i P_i^T B_i (P_i X).
//
// Every kernel keeps the dense index innermost and contiguous across lanes:
// one stored entry a(p,q) triggers one scaled vector update
//     acc[0:k] += a * X[perm[q], 0:k]
// which is the axpy leaf of the paper's loop nests (figure "Loop nest for an
// order 4 TTMc kernel") at order 2, with rows then nonzeros as outer loops
// (section "SpTTN-Cyclops Framework": sparse indices in stored order).  The
// row gather P_i X is fused into the loads: entries carry perm[q] directly
// (or the row of the staged head buffer).  The scatter P_i^T is fused into the
// epilogue: results go to row perm[p] of Y.
//
// A lane owns VEC consecutive columns; LPR lanes ("a lane group") cover one
// slice of LPR*VEC columns; a wavefront holds G = 64 / LPR lane groups.
//   product kernel - the work lists of a level in one launch: a wavefront per chunk of a
//                   long row (the head rows), its G lane groups taking entries round-robin
//                   and combined with wavefront shuffles; a lane group per run of short rows
//                   (first-block-column and diagonal-block entries of the body rows, short
//                   head rows, pieces of long rows)
//   reduce kernel - sums the partial vectors of rows that were split into
//                   several chunks, in a fixed order, and scatters to Y
//   window kernel - diagonal-block tiles with their window of P_i X staged in LDS
//   gather kernel - rows of P_i X materialised (the staged head X_0, or a whole level)
//   panel kernels - optional: head-block entries of sparse head rows with the rows'
//                   accumulators in LDS, one column class per accelerator die
//   corner kernels - the dense top-left corner of the head block in tiles of 256 x 256: the
//                   tile's staged head rows and the row panel's accumulators both live in LDS
//   sddmm_panel, sddmm_corner kernels - the sampled product S = A .* (U V^T) over the two optional
//                   lists; the others are in sddmm.hip
// The product kernel fetches its entries with coalesced loads into LDS (short
// rows: all entries of a workgroup's items at once; chunks: 64 to 256 at a time
// into a wavefront-private strip, the next ones already on their way)
// and read them back per lane group, so that U row loads are in flight before
// the first FMA and a lane group only ever waits for the rows it gathers; the
// SIMDs are 16 lanes wide (4 cycles per wavefront instruction), so the inner
// loops are written to need one address instruction per row load.
// Rows written or read exactly once per product (results, partial vectors)
// carry the non-temporal hint and leave the L2 to the rows of X.
// No floating-point atomics: results are bitwise reproducible run to run.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "arrow_internal.h"
#include "kernel_common.h"

namespace arrow {
namespace {

// ---------------------------------------------------------------------------
// product kernel: one launch runs the wave list, the pieces and the short rows of a level; a
// workgroup's place in the grid says which of them it works on.  The parts write different rows of
// Y and partial slots, so they need no order among themselves, and one grid has one ramp and one
// tail instead of three (a launch on its own costs 2 - 3 us on the stream, which is most of the
// time of a product over a few thousand rows).
// ---------------------------------------------------------------------------
constexpr int64_t kPieceWavesMax = 4096;
constexpr int kFlowBatches = 4;        // batches of a workgroup of the flow kernel; fewer where that leaves
constexpr int64_t kFlowBlocks = 1536;  // less than these workgroups, the ones the chip holds at a time
constexpr int64_t kFlowLeast = 1024;   // fewest batches it takes (100489 rows, k = 32: 13.2 -> 10.2 us; 40000, k = 16: 5.3 and 5.6)
constexpr int64_t kDieSetsLeast = 8LL << 20;     // smallest X whose column slices are dealt to sets of dies,
constexpr int64_t kDieSetsMost = 512LL << 20;    // ... and the largest
constexpr int kRowsStage = 1024;   // entries of the group list a workgroup stages at once (8 KiB)

template <int LPR> constexpr int strip_entries() {     // entries of the wave list a wavefront parks per batch
  constexpr int full = 64 / LPR * 8;                   // eight rows in flight for each of its lane groups
  return full < 64 ? 64 : (full > 128 ? 128 : full);
}

struct alignas(16) RowsShared {
  Entry stage[kRowsStage];
  uint32_t ptr[kItemsPerGroupBlock + 1];
  uint32_t mid[kItemsPerGroupBlock];
  int32_t dst[kItemsPerGroupBlock];
};

// Items [0, n_it) of a batch of the group list whose descriptors are at ptr, mid and dst, one lane group
// per item, taken round-robin.  Entries [lo, mid) of an item read rows of the staged head buffer Xh,
// entries [mid, hi) rows of X.  `staged`: the batch's entries, or null where they are read from memory.
template <int VEC, int LPR, bool SMALL>
__device__ __forceinline__ void row_items(const uint32_t* ptr, const uint32_t* mids, const int32_t* dsts,
                                          const Entry* staged, const ProductArgs& a, int n_it, const LaneColumns lc) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  constexpr uint32_t U = 8;
  const int tid = threadIdx.x;
  const uint32_t col_bytes = lc.ok ? 4u * (uint32_t)lc.c : 0u;
  const uint32_t e0 = ptr[0];
  auto run = [&](auto entry) {
    for (int it = tid / LPR; it < n_it; it += GPB) {
      const int32_t dst = dsts[it];
      if (dst == INT32_MIN) continue;             // padding slot of the die queues
      const uint32_t lo = ptr[it], mid = mids[it], hi = ptr[it + 1];
      V acc = vzero<VEC>();
      for (int seg = 0; seg < 2; ++seg) {
        const char* base = reinterpret_cast<const char*>(seg == 0 ? a.Xh : a.X);
        const uint32_t row_bytes = 4u * (uint32_t)(seg == 0 ? a.head_stride : a.k);
        const uint32_t j_hi = seg == 0 ? mid : hi;
        for (uint32_t j = seg == 0 ? lo : mid; j < j_hi; j += U) {
          Entry e[U];
          V x[U];
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) e[u] = entry(j + u < j_hi ? j + u : j);
#pragma unroll
          for (uint32_t u = 0; u < U; ++u)
            x[u] = (j + u < j_hi) ? load_row<VEC, SMALL>(base, e[u].xrow, row_bytes, col_bytes) : vzero<VEC>();
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) vfma(acc, (j + u < j_hi) ? e[u].val : 0.f, x[u]);
        }
      }
      if (lc.ok) {
        float* y = dst >= 0 ? a.Y + (size_t)dst * (size_t)a.k + lc.c
                            : a.partials + (size_t)(-1 - dst) * (size_t)a.k + lc.c;
        if (a.accumulate && dst >= 0) vadd(acc, vload_stream<VEC>(y));
        vstore_stream<VEC>(y, acc);
      }
    }
  };
  if (staged) run([&](uint32_t t) { return staged[t - e0]; });
  else run([&](uint32_t t) { return a.ent[t]; });
}

// The items [first, first + n_it) of the group list.  The workgroup first copies the descriptors of its
// items and, when they fit the staging buffer, all their entries -- one contiguous range -- into LDS with
// coalesced loads; after that the only memory latency a lane group waits for is that of the rows it
// gathers.  Items that do not fit are read from memory entry by entry.  Which entries these are is read beside the descriptors, not out
// of LDS behind a barrier: five products of Chung-Lu 2m, k = 32, 2465 -> 2439 us; R-MAT 200k, 16, 38.9 -> 38.4; grid 90k, 64, 16.7 -> 16.5.
template <int VEC, int LPR, bool SMALL>
__device__ __forceinline__ void rows_part(RowsShared& sh, const ProductArgs& a, int64_t first, int n_it,
                                          const LaneColumns lc) {
  const int tid = threadIdx.x;
  uint32_t ptr = 0, mid = 0;
  int32_t dst = 0;
  if (tid <= n_it) ptr = a.rows_ptr[first + tid];
  if (tid < n_it) { mid = a.rows_mid[first + tid]; dst = a.rows_dst[first + tid]; }
  const uint32_t e0 = a.rows_ptr[first];
  const uint32_t total = a.rows_ptr[first + n_it] - e0;
  const bool staged = total <= (uint32_t)kRowsStage;
  if (staged) {
    // all loads before the first wait (one at a time they were up to four memory latencies in a row)
    constexpr uint32_t Q = kRowsStage / kBlock;
    Entry e[Q];
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q)
      if (tid + q * kBlock < total) e[q] = a.entries_once ? stream_load(a.ent + e0 + tid + q * kBlock) : a.ent[e0 + tid + q * kBlock];
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) if (tid + q * kBlock < total) sh.stage[tid + q * kBlock] = e[q];
  }
  if (tid <= n_it) sh.ptr[tid] = ptr;
  if (tid < n_it) { sh.mid[tid] = mid; sh.dst[tid] = dst; }
  __syncthreads();
  row_items<VEC, LPR, SMALL>(sh.ptr, sh.mid, sh.dst, staged ? sh.stage : nullptr, a, n_it, lc);
}

// One chunk of the wave list per wavefront.  Entries [lo, mid) of a chunk read rows of the staged
// head buffer Xh, entries [mid, hi) read rows of X (the chunk's entries are ordered by column
// position, head columns first), so the base pointer is uniform inside a batch.  The G lane groups
// take the entries round-robin and are combined with a butterfly over the lane groups; the wavefronts
// of a team (kTeamDst) then add up in LDS, in slot order (sums: LDS for that, or null where the list
// has no teams).
// (Several chunks per wavefront, the next one's descriptor and entries fetched ahead, measured 3 %
// slower for two and 10 % for four: the chunks in flight then reach over more column windows.)
template <int VEC, int LPR, bool SMALL>
__device__ __forceinline__ void chunk_part(Entry* mine, const ProductArgs& a, const uint32_t* ptr,
                                           const uint32_t* mids, const int32_t* dsts, int64_t ch, float* sums,
                                           const LaneColumns lc) {
  using V = typename Vec<VEC>::type;
  constexpr int G = 64 / LPR;
  constexpr uint32_t U = 8;
  constexpr uint32_t STRIP = strip_entries<LPR>();
  constexpr int NA = STRIP / 64;
  const uint32_t lo = ptr[ch];
  const uint32_t hi = ptr[ch + 1];
  const uint32_t mid = mids[ch];
  const int32_t dst = dsts[ch];
  if (lo == hi) return;                // padding slot of the die queues
  const uint32_t lane = threadIdx.x % 64;
  const uint32_t g = lane / LPR;
  const uint32_t col_bytes = lc.ok ? 4u * (uint32_t)lc.c : 0u;
  const Entry* grp = mine + g;
  const int64_t ch0 = ch - ch % kChunksPerGroup;
  const bool team = sums && ch0 + 1 < a.n_chunks && dsts[ch0 + 1] == kTeamDst;
  V acc = vzero<VEC>();
  // the next entries of the chunk are fetched while the current batch is being worked on (the two
  // segments are consecutive in the entry array, so the fetch runs across their boundary)
  Entry ahead[NA];
#pragma unroll
  for (int q = 0; q < NA; ++q) ahead[q] = a.ent[lo + lane + q * 64 < hi ? lo + lane + q * 64 : lo];
  for (int seg = 0; seg < 2; ++seg) {
    const char* base = reinterpret_cast<const char*>(seg == 0 ? a.Xh : a.X);
    const uint32_t row_bytes = 4u * (uint32_t)(seg == 0 ? a.head_stride : a.k);
    const uint32_t s_lo = seg == 0 ? lo : mid;
    const uint32_t s_hi = seg == 0 ? mid : hi;
    for (uint32_t b0 = s_lo; b0 < s_hi; b0 += STRIP) {
      const uint32_t nb = s_hi - b0 < STRIP ? s_hi - b0 : STRIP;
#pragma unroll
      for (int q = 0; q < NA; ++q) {   // entries b0 .. b0 + STRIP - 1 (those past the chunk's end are not used)
        mine[lane + q * 64] = ahead[q];
        const uint32_t nx = b0 + nb + lane + q * 64;     // next batch, of this or the next segment
        ahead[q] = a.ent[nx < hi ? nx : lo];
      }
      strip_sync();
      uint32_t s = 0;                  // step: lane group g handles entry s * G + g
      for (; (s + U) * G <= nb; s += U) {
        Entry e[U];
        V x[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) e[u] = grp[(s + u) * G];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) x[u] = load_row<VEC, SMALL>(base, e[u].xrow, row_bytes, col_bytes);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) vfma(acc, e[u].val, x[u]);
      }
      if (s * G < nb) {                // last, partly filled round of this batch
        Entry e[U];
        V x[U];
        bool ok[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          ok[u] = (s + u) * G + g < nb;
          e[u] = mine[((s + u) * G + g) % STRIP];
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
          x[u] = ok[u] ? load_row<VEC, SMALL>(base, e[u].xrow, row_bytes, col_bytes) : vzero<VEC>();
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) vfma(acc, ok[u] ? e[u].val : 0.f, x[u]);
      }
      strip_sync();                    // the strip is rewritten by the next batch
    }
  }
  // combine the G lane groups: butterfly over lane-id bits LPR, 2 LPR, ..., 32
#pragma unroll
  for (int m = LPR; m < 64; m <<= 1) vadd(acc, vshfl_xor(acc, m));
  const int wave = (int)(ch % kChunksPerGroup);
  if (team) {                          // all four wavefronts of the workgroup are here
    if (wave > 0 && g == 0) vstore<VEC>(sums + (wave * 64 + lane) * VEC, acc);
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 1; w < kChunksPerGroup; ++w) vadd(acc, vload<VEC>(sums + (w * 64 + lane % LPR) * VEC));
  }
  if (g == 0 && lc.ok) {
    float* y = dst >= 0 ? a.Y + (size_t)dst * (size_t)a.k + lc.c
                        : a.partials + (size_t)(-1 - dst) * (size_t)a.k + lc.c;
    if (a.accumulate && dst >= 0) vadd(acc, vload_stream<VEC>(y));
    vstore_stream<VEC>(y, acc);
  }
}

// The column slices are dealt to the dies in 1 << sets_log sets of neighbours: a die of set t works on the t-th share of
// the slices, one after the other, so that its L2 holds rows of X of that many columns only and fetches them for that many.
// Which slice and which of its `blocks` workgroups the id-th workgroup of a part is (a multiple of kDies per slice; the
// part begins at die 0):
struct SliceBlock { uint32_t slice, block; };
__device__ __forceinline__ SliceBlock slice_block(const ProductArgs& a, uint32_t id, uint32_t blocks) {
  const uint32_t dies_log = kDiesLog - a.sets_log, die = id % kDies;
  uint32_t at = (id / kDies << dies_log) + (die & ((1u << dies_log) - 1u));
  uint32_t slice = (die >> dies_log) * (a.slices >> a.sets_log);
  if (a.slices > 8) {
    const uint32_t more = at / blocks;
    return {slice + more, at - more * blocks};
  }
  for (; at >= blocks; at -= blocks) ++slice;       // (few slices: a division costs more)
  return {slice, at};
}

// Six wavefronts per SIMD: with seven the compiler spills in the narrow shapes (A^5 X of a 2m-vertex
// Chung-Lu graph, k = 32: 2675 -> 2747 us).
// grid: [wave list][pieces][short rows][rows without entries], each slice by slice on every set of dies
// (slice_block); every part is a multiple of 8 workgroups per slice, so that workgroup w of every slice
// runs on die w mod 8 where there is one set (the die queues of both lists rely on it).
template <int VEC, int LPR, bool SMALL>
__global__ __launch_bounds__(kBlock, 6) void product_kernel(const ProductArgs a) {
  constexpr int GPB = kBlock / LPR;
  constexpr int WPB = kBlock / 64;
  union Shared {
    RowsShared rows;
    struct { Entry strip[WPB][strip_entries<LPR>()]; float sums[WPB * 64 * VEC]; } chunk;
    __device__ Shared() {}
  };
  __shared__ Shared sh;
  const int tid = threadIdx.x;
  uint32_t id = blockIdx.x;
  int part = 0;
  while (part < 3 && id >= a.blocks[part] * a.slices) { id -= a.blocks[part] * a.slices; ++part; }
  const SliceBlock at = slice_block(a, id, a.blocks[part]);
  id = at.block;
  const LaneColumns lc = lane_columns<VEC>(tid % LPR, (int)at.slice * a.width, a.k, a.width);
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  if (part == 0 || (part == 1 && a.piece_waves)) {
    const bool list = part == 0;
    const int64_t ch = (int64_t)id * WPB + wave;
    if (ch < a.count[part])
      chunk_part<VEC, LPR, SMALL>(sh.chunk.strip[wave], a, list ? a.chunk_ptr : a.rows_ptr,
                                  list ? a.chunk_mid : a.rows_mid, list ? a.chunk_dst : a.rows_dst, ch,
                                  list ? sh.chunk.sums : nullptr, lc);
    return;
  }
  const int64_t first = (int64_t)id * a.items[part] + a.begin[part];
  const int64_t left = a.begin[part] + a.count[part] - first;
  const int n_it = left < a.items[part] ? (int)left : a.items[part];
  if (n_it <= 0) return;
  if (part < 3) {
    rows_part<VEC, LPR, SMALL>(sh.rows, a, first, n_it, lc);
    return;
  }
  for (int it = tid / LPR; it < n_it; it += GPB)   // level 0 stores every row of Y
    if (lc.ok) vstore_stream<VEC>(a.Y + (size_t)a.rows_dst[first + it] * (size_t)a.k + lc.c, vzero<VEC>());
}

// Copies the lanes' 4 or 16 bytes from `from` to consecutive places at `to` in LDS (the same for the whole
// wavefront) without registers in between.  In assembly because the compiler waits for such a copy before
// the next read of LDS, whatever it reads: the caller waits (vmcnt) before it reads what was copied.
// m0, which holds the place in LDS, gets back what it held: the compiler reserves the register and does
// not heed it in a list of clobbers.
#define ARROW_TO_LDS(INSTRUCTION)                                                                                     \
  int m0_was;                                                                                                         \
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\t" INSTRUCTION " %1, off\n\ts_mov_b32 m0, %0"        \
               : "=&s"(m0_was)                                                                                        \
               : "v"(from), "s"(__builtin_amdgcn_readfirstlane((int)(uint32_t)reinterpret_cast<uintptr_t>(to)))       \
               : "memory")
__device__ __forceinline__ void copy_to_lds16(const void* from, const void* to) { ARROW_TO_LDS("global_load_lds_dwordx4"); }
__device__ __forceinline__ void copy_to_lds4(const void* from, const void* to) { ARROW_TO_LDS("global_load_lds_dword"); }
#undef ARROW_TO_LDS

struct alignas(16) FlowShared {
  Entry stage[2][kRowsStage + 8];      // a batch's entries from an even one on; up to seven past the last are read
  struct { uint32_t lo[kItemsPerGroupBlock], hi[kItemsPerGroupBlock], mid[kItemsPerGroupBlock]; int32_t dst[kItemsPerGroupBlock]; } of[3];
};
static_assert(kItemsPerGroupBlock == 64 && kBlock == 256, "one wavefront per descriptor array, one lane per item");

// The short rows on their own, where they are nearly all of the product and every batch of them fits the
// staging buffer.  A workgroup works on every gridDim.x-th batch; the next batch's entries and the
// descriptors of the one after it are copied to LDS meanwhile.  Of the row of X that an entry of a stencil
// reads, one in five comes from memory and the others from the L2, so it is the latency of few bytes that
// bounds the time: three latencies per batch with the copies ahead, of which two are for rows of X, where
// there were four.  (Grid of 1024 x 1024, k = 32, X and Y not in any cache: 80.1 -> 65.4 us, 4.8 TB/s; when
// it was built four batches took 69.7, one 73.8, two 70.6, eight 74.5.  Beside long rows, whose misses fill the memory pipes, the
// launch of its own costs more than this gives: three products of R-MAT 1m, k = 64, 1184 -> 1227 us.)
template <int VEC, int LPR, bool SMALL>
__global__ __launch_bounds__(kBlock, 6) void flow_kernel(const ProductArgs a) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  constexpr uint32_t U = 8;
  __shared__ FlowShared sh;
  const int tid = threadIdx.x;
  const int lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const LaneColumns lc = lane_columns<VEC>(tid % LPR, (int)blockIdx.y * a.width, a.k, a.width);
  const uint32_t col_bytes = lc.ok ? 4u * (uint32_t)lc.c : 0u;
  const int64_t step = gridDim.x;
  auto items_of = [&](int64_t bt) {
    const int64_t left = a.count[2] - bt * kItemsPerGroupBlock;
    return left < 0 ? 0 : (left < kItemsPerGroupBlock ? (int)left : kItemsPerGroupBlock);
  };
  const uint32_t* mine = wave == 0 ? a.rows_ptr : wave == 1 ? a.rows_ptr + 1 : wave == 2 ? a.rows_mid
                                                : reinterpret_cast<const uint32_t*>(a.rows_dst);
  auto describe = [&](int to, int64_t bt) {
    if (lane < items_of(bt)) copy_to_lds4(mine + a.begin[2] + bt * kItemsPerGroupBlock + lane, &sh.of[to].lo[0] + wave * 64);
  };
  auto fetch = [&](int buf, int to, int n) {         // two entries per lane
    const uint32_t e0 = sh.of[to].lo[0] & ~1u, e1 = sh.of[to].hi[n - 1];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int at = (q * 4 + wave) * 64;
      if (q < 2 || wave == 0)
        if (e0 + 2u * (uint32_t)(at + lane) < e1) copy_to_lds16(a.ent + e0 + 2 * (at + lane), sh.stage[buf] + 2 * at);
    }
  };
  // (__syncthreads would wait for the stores of Y as well)
  auto arrived = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  auto sync = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  int64_t bt = blockIdx.x;
  int n = items_of(bt);
  if (n == 0) return;
  describe(0, bt);
  describe(1, bt + step);
  arrived();
  sync();
  fetch(0, 0, n);
  arrived();
  sync();
  for (int cur = 0, buf = 0;; buf ^= 1) {
    const int nxt = cur == 2 ? 0 : cur + 1;
    const int n_next = items_of(bt + step);
    if (n_next > 0) {
      fetch(buf ^ 1, nxt, n_next);
      describe(nxt == 2 ? 0 : nxt + 1, bt + 2 * step);
    }
    const auto& b = sh.of[cur];
    const uint32_t e0 = b.lo[0] & ~1u;
    for (int it = tid / LPR; it < n; it += GPB) {
      const uint32_t mid = b.mid[it], hi = b.hi[it];
      V acc = vzero<VEC>();
      for (int seg = 0; seg < 2; ++seg) {
        const char* base = reinterpret_cast<const char*>(seg == 0 ? a.Xh : a.X);
        const uint32_t row_bytes = 4u * (uint32_t)(seg == 0 ? a.head_stride : a.k);
        const uint32_t j_hi = seg == 0 ? mid : hi;
        for (uint32_t j = seg == 0 ? b.lo[it] : mid; j < j_hi; j += U) {
          Entry e[U];
          V x[U];
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) e[u] = sh.stage[buf][j - e0 + u];
#pragma unroll
          for (uint32_t u = 0; u < U; ++u)
            x[u] = (j + u < j_hi) ? load_row<VEC, SMALL>(base, e[u].xrow, row_bytes, col_bytes) : vzero<VEC>();
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) vfma(acc, (j + u < j_hi) ? e[u].val : 0.f, x[u]);
        }
      }
      arrived();                                     // older than the rows just used: no wait but for the first item's store
      if (lc.ok) {
        float* y = a.Y + (size_t)b.dst[it] * (size_t)a.k + lc.c;
        if (a.accumulate) vadd(acc, vload_stream<VEC>(y));
        vstore_stream<VEC>(y, acc);
      }
    }
    if (n_next == 0) return;
    if (wave * (64 / LPR) >= n) arrived();           // a wavefront without items has not waited yet
    sync();
    bt += step; n = n_next; cur = nxt;
  }
}

// The wave list on its own, for lists in window order: a chunk is over in two or three rounds of row
// loads, so what a wavefront does before the first of them counts (finding its part of the product
// kernel's grid and looking for a team cost the chunks of the Chung-Lu graph above 7 %).
template <int VEC, int LPR, bool SMALL>
__global__ __launch_bounds__(kBlock) void chunks_kernel(const ProductArgs a) {
  constexpr int WPB = kBlock / 64;
  __shared__ Entry strip[WPB][strip_entries<LPR>()];
  // The same order of slices as slice_block's, but by the grid: a row of it is a slice of every set.  (With slice_block, a
  // loop or a division, the shape of 17 to 32 columns took 78 registers instead of 72 and six wavefronts per SIMD
  // instead of seven, also with one slice: A^5 of Chung-Lu 2m, k = 32, 2478 us instead of 2464.)
  const uint32_t dies_log = kDiesLog - a.sets_log, dies = 1u << dies_log, die = blockIdx.x % kDies;
  uint32_t id = (blockIdx.x / kDies << dies_log) + (die & (dies - 1u));
  const uint32_t slice = (die >> dies_log) * gridDim.y + blockIdx.y;
  // Runs of some 256 workgroups (die_run) go to one die each: the eight dies then work on different column
  // windows at a time, and a row of X that several chunks of a run read is fetched into one L2
  // instead of several (the same chunks: 255 -> 231 us per product; R-MAT 8m, k = 128: 1 %; eighths
  // of the whole list are slower, the dies then finish at different times).
  id = in_runs(id, dies_log, a.run, a.blocks[0]);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int64_t ch = (int64_t)id * WPB + wave;
  if (ch >= a.n_chunks) return;
  const LaneColumns lc = lane_columns<VEC>(threadIdx.x % LPR, (int)slice * a.width, a.k, a.width);
  chunk_part<VEC, LPR, SMALL>(strip[wave], a, a.chunk_ptr, a.chunk_mid, a.chunk_dst, ch, nullptr, lc);
}

// ---------------------------------------------------------------------------
// window kernel: one workgroup per tile of a diagonal block and column slice.  The tile's window of
// P_i X (win_count consecutive positions of the level, `width` columns) is gathered through perm into
// LDS once -- the permutation gather of these rows happens here -- and every diagonal-block entry of
// the tile's rows then reads its X row from LDS; the rows' other entries (first block column, other
// blocks once levels are fused) read rows of X from memory.
//
// Sixteen lanes own a row of Y, whatever the number of columns (VEC = 4, 2 or 1 of them per lane), so
// that they are one DPP row: the lanes load sixteen entries at a time, one each, and an entry reaches
// all of them as an operand modifier of the address addition and the multiply-adds (row_newbcast).
// An entry costs five vector instructions and one LDS read for four rows of Y.  The next row's
// entries are on their way while the current one is worked on.  With the entries read four at a time
// by every lane and windows of 64 KiB in slices of 32 columns, two memory latencies stood before
// every fourth entry; 512 blocks of 512 with 48 entries per row, k = 128: 250 -> 145 us, of which the
// LDS reads (6.4 GB at the 78 TB/s that all compute units together reach) take 82.
// ---------------------------------------------------------------------------
constexpr int kWinBlock = 1024;   // threads of a window-kernel workgroup: 16 wavefronts share one staged window,
constexpr int kWinBlockHalf = 512;   // ... or 8 where a compute unit holds two windows and registers are short
constexpr int64_t kWinHalfTiles = 768;   // fewest workgroups of 8 wavefronts
constexpr int kWinLanes = 16;
constexpr int kWinParts = 8;      // most workgroups that share the rows of a tile
constexpr int kComputeUnits = 256;
constexpr int kWinFloats = 38400; // LDS floats of a window: 150 KiB, one workgroup per compute unit,
constexpr int kWinFloatsHalf = 19200;   // ... or two
constexpr double kWinStage = 6.0; // entries that a row of Y adds in the time that a row of the window takes to arrive
constexpr int kWinColumns = 64;   // most columns of a slice

template <int U>
__device__ __forceinline__ int row16_bcast(int v) {   // lane U's value in every lane of its sixteen
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + U, 0xf, 0xf, false);
}
// acc += (the v of lane U + u) * x[u] for u = 0 .. 3 in turn, the broadcast being an operand modifier of the
// multiply-adds themselves (out of the builtin the compiler makes a move per entry).  The compiler does not
// look into the statement, so the wait that the modifier needs stands in it as well: the register that is
// read must not have been written by the two instructions before, nor the lane mask by a vector instruction among the
// five before; the mask can change before the first and the third four of a batch, and which kind of instruction does that
// is the compiler's choice.  (512 blocks of 512, k = 128: with one
// wait per batch, which nothing ties to the multiply-adds, 158.2 us, so 159.4.)
#define ARROW_BCAST(A, V, X, U) "v_fmac_f32_dpp %" #A ", %" #V ", %" #X " row_newbcast:%" #U " row_mask:0xf bank_mask:0xf\n\t"
template <int U> __device__ __forceinline__ void fma_bcast4(float& a, float v, const float* x) {
  asm("s_nop %10\n\t"
      ARROW_BCAST(0, 1, 2, 6) ARROW_BCAST(0, 1, 3, 7) ARROW_BCAST(0, 1, 4, 8) ARROW_BCAST(0, 1, 5, 9)
      : "+&v"(a) : "v"(v), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "n"(U), "n"(U + 1), "n"(U + 2), "n"(U + 3), "n"(U % 8 ? 1 : 4));
}
template <int U> __device__ __forceinline__ void fma_bcast4(float2& a, float v, const float2* x) {
  asm("s_nop %15\n\t"
      ARROW_BCAST(0, 2, 3, 11) ARROW_BCAST(1, 2, 4, 11) ARROW_BCAST(0, 2, 5, 12) ARROW_BCAST(1, 2, 6, 12)
      ARROW_BCAST(0, 2, 7, 13) ARROW_BCAST(1, 2, 8, 13) ARROW_BCAST(0, 2, 9, 14) ARROW_BCAST(1, 2, 10, 14)
      : "+&v"(a.x), "+&v"(a.y)
      : "v"(v), "v"(x[0].x), "v"(x[0].y), "v"(x[1].x), "v"(x[1].y), "v"(x[2].x), "v"(x[2].y), "v"(x[3].x), "v"(x[3].y),
        "n"(U), "n"(U + 1), "n"(U + 2), "n"(U + 3), "n"(U % 8 ? 1 : 4));
}
template <int U> __device__ __forceinline__ void fma_bcast4(float4& a, float v, const float4* x) {
  asm("s_nop %25\n\t"
      ARROW_BCAST(0, 4, 5, 21) ARROW_BCAST(1, 4, 6, 21) ARROW_BCAST(2, 4, 7, 21) ARROW_BCAST(3, 4, 8, 21)
      ARROW_BCAST(0, 4, 9, 22) ARROW_BCAST(1, 4, 10, 22) ARROW_BCAST(2, 4, 11, 22) ARROW_BCAST(3, 4, 12, 22)
      ARROW_BCAST(0, 4, 13, 23) ARROW_BCAST(1, 4, 14, 23) ARROW_BCAST(2, 4, 15, 23) ARROW_BCAST(3, 4, 16, 23)
      ARROW_BCAST(0, 4, 17, 24) ARROW_BCAST(1, 4, 18, 24) ARROW_BCAST(2, 4, 19, 24) ARROW_BCAST(3, 4, 20, 24)
      : "+&v"(a.x), "+&v"(a.y), "+&v"(a.z), "+&v"(a.w)
      : "v"(v), "v"(x[0].x), "v"(x[0].y), "v"(x[0].z), "v"(x[0].w), "v"(x[1].x), "v"(x[1].y), "v"(x[1].z), "v"(x[1].w),
        "v"(x[2].x), "v"(x[2].y), "v"(x[2].z), "v"(x[2].w), "v"(x[3].x), "v"(x[3].y), "v"(x[3].z), "v"(x[3].w),
        "n"(U), "n"(U + 1), "n"(U + 2), "n"(U + 3), "n"(U % 8 ? 1 : 4));
}
#undef ARROW_BCAST

template <int VEC, bool SMALL, int BLOCK, int FLOATS>
__global__ __launch_bounds__(BLOCK, BLOCK / 256 * (kWinFloats / FLOATS)) void window_kernel(
    const WindowTile* __restrict__ tiles, int64_t n_tiles, const uint32_t* __restrict__ wrow_ptr,
    const uint32_t* __restrict__ wrow_mid, const int32_t* __restrict__ wrow_y,
    const Entry* __restrict__ ent, const int32_t* __restrict__ perm, const float* __restrict__ X,
    float* __restrict__ Y, int k, int width, int slices, int parts, int accumulate) {
  using V = typename Vec<VEC>::type;
  constexpr uint32_t GPB = BLOCK / kWinLanes;
  constexpr int QB = 4;                              // batches of sixteen window entries a row has on their way
  constexpr uint32_t NO = 4;                         // entries outside the window loaded ahead
  // The window, and behind it a row of zeros for the lanes that hold no entry: with a row of the window in
  // its place an infinity or NaN there would reach rows of Y that have no entry in its column (0 * inf).
  __shared__ __attribute__((aligned(16))) float win[FLOATS + kWinColumns];
  // the slices of a tile follow each other on one die: its entries are read from memory once
  const int64_t id = blockIdx.x;
  const int64_t tile = id / (kDies * slices * parts) * kDies + id % kDies;
  const int slice = (int)(id / (kDies * parts) % slices);
  if (tile >= n_tiles) return;
  WindowTile t = tiles[tile];
  if (parts > 1) {                                   // this workgroup's share of the tile's rows
    const uint32_t part = (uint32_t)(id / kDies % parts), rows = t.row_end - t.row_begin, first = t.row_begin;
    t.row_begin = first + rows * part / parts;
    t.row_end = first + rows * (part + 1) / parts;
    if (t.row_begin == t.row_end) return;
  }
  const uint32_t l = threadIdx.x % kWinLanes;
  const uint32_t grp = threadIdx.x / kWinLanes;
  const LaneColumns lc = lane_columns<VEC>((int)l, slice * width, k, width);   // lane l's columns sit at [l * VEC] of an LDS row
  const uint32_t row_bytes = 4u * (uint32_t)k;
  const uint32_t col_bytes = lc.ok ? 4u * (uint32_t)lc.c : 0u;
  const char* Xb = reinterpret_cast<const char*>(X);
  const bool has_lds = (int)l * VEC < width;         // lanes beyond the slice own no part of an LDS row
  // everything of the tile is addressed relative to its first row and first entry: 32-bit offsets
  const uint32_t n_rows = t.row_end - t.row_begin;
  const uint32_t* __restrict__ t_ptr = wrow_ptr + t.row_begin;
  const uint32_t* __restrict__ t_mid = wrow_mid + t.row_begin;
  const int32_t* __restrict__ t_y = wrow_y + t.row_begin;
  const uint32_t e0 = t_ptr[0];
  const Entry* __restrict__ t_ent = ent + e0;
  struct Row { uint32_t lo, mid, hi; int32_t y; };
  auto describe = [&](uint32_t i) {
    Row r{0, 0, 0, 0};
    if (i < n_rows) { r.lo = t_ptr[i] - e0; r.mid = t_mid[i] - e0; r.hi = t_ptr[i + 1] - e0; r.y = t_y[i]; }
    return r;
  };
  auto fetch = [&](const Row& r, Entry& out, Entry (&e)[QB]) {
    if (l < r.mid - r.lo) out = t_ent[r.lo + l];
#pragma unroll
    for (uint32_t q = 0; q < QB; ++q)
      if (r.mid + l + q * kWinLanes < r.hi) e[q] = t_ent[r.mid + l + q * kWinLanes];
  };
  Row r = describe(grp), r_n = describe(grp + GPB);
  if (threadIdx.x < kWinColumns) win[FLOATS + threadIdx.x] = 0.f;
  // stage: lane group j loads window rows j, j + GPB, ... eight at a time
  for (uint32_t i0 = grp; i0 < t.win_count; i0 += 8 * GPB) {
    int32_t src[8];
    V v[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) {
      const uint32_t i = i0 + u * GPB;
      src[u] = i < t.win_count ? perm[t.win_begin + i] : -1;
    }
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u)
      v[u] = (src[u] >= 0 && lc.ok) ? load_row<VEC, SMALL>(Xb, src[u], row_bytes, col_bytes) : vzero<VEC>();
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) {
      const uint32_t i = i0 + u * GPB;
      if (i < t.win_count && has_lds) vstore<VEC>(win + i * width + l * VEC, v[u]);
    }
  }
  Entry o{0, 0.f}, o_n{0, 0.f}, e[QB] = {}, e_n[QB] = {};
  fetch(r, o, e);
  __syncthreads();
  const char* lane_win = reinterpret_cast<const char*>(win) + (has_lds ? l * VEC * 4 : 0);
  const int row_step = width * 4;
  V acc;
  // sixteen window entries, one per lane (`n` of them there)
  auto batch = [&](const Entry& mine, uint32_t n) {
    const int off = l < n ? mine.xrow * row_step : FLOATS * 4;
    const float val = l < n ? mine.val : 0.f;
    V x[8], x2[8];                                   // all reads on their way before the first is used
#define ARROW_READ(U) vload<VEC>(reinterpret_cast<const float*>(lane_win + row16_bcast<U>(off)))
    x[0] = ARROW_READ(0); x[1] = ARROW_READ(1); x[2] = ARROW_READ(2); x[3] = ARROW_READ(3);
    x[4] = ARROW_READ(4); x[5] = ARROW_READ(5); x[6] = ARROW_READ(6); x[7] = ARROW_READ(7);
    if (n > 8) {
      x2[0] = ARROW_READ(8); x2[1] = ARROW_READ(9); x2[2] = ARROW_READ(10); x2[3] = ARROW_READ(11);
      x2[4] = ARROW_READ(12); x2[5] = ARROW_READ(13); x2[6] = ARROW_READ(14); x2[7] = ARROW_READ(15);
    }
#undef ARROW_READ
    fma_bcast4<0>(acc, val, x);
    fma_bcast4<4>(acc, val, x + 4);
    if (n > 8) {
      fma_bcast4<8>(acc, val, x2);
      fma_bcast4<12>(acc, val, x2 + 4);
    }
  };
  // The scheduler prefers the oldest wavefronts of a SIMD: they were through with their rows after 17.6 us, the youngest after
  // 27.6, alone at the end.  With lower priorities for those that have fewer rows left they end after 20 to 22.7 us (512
  // blocks of 512 with 48 entries per row, k = 128, 136.1 -> 123.8 us of a product; 300k, 50 entries, 96: 176.5 -> 160.2).  Where two
  // workgroups share a compute unit the one that sums may hold up the other one's staging, and it depends on the operand: a product without / with
  // priorities, us, 500k, 60, 16, 82.2 / 75.4; 700k, 30, 8, 73.4 / 69.7; 437k, 62, 16, 83.2 / 91.8; in the form of eight wavefronts 600k, 26, 32, 97 / 98.
  // None there: what tells the first two from the third is not known.
  constexpr bool RANKED = FLOATS == kWinFloats;
  uint32_t left = (n_rows + GPB - 1) / GPB;          // rows to go, this one included
  if (RANKED && left > 3) __builtin_amdgcn_s_setprio(3);
  for (uint32_t i = grp; i < n_rows; i += GPB, --left) {
    if (RANKED && left == 3) __builtin_amdgcn_s_setprio(2);
    if (RANKED && left == 2) __builtin_amdgcn_s_setprio(1);
    if (RANKED && left == 1) __builtin_amdgcn_s_setprio(0);
    const Row r_nn = describe(i + 2 * GPB);
    fetch(r_n, o_n, e_n);
    acc = vzero<VEC>();
    // the first entries outside the window: their rows of X arrive while the window entries are summed
    const uint32_t n_out = r.mid - r.lo;
    V xo[NO];
#define ARROW_OUT(O)                                                                    \
    {                                                                                   \
      const int xrow = row16_bcast<O>(o.xrow);                                          \
      xo[O] = vzero<VEC>();                                                             \
      if (O < n_out) xo[O] = load_row<VEC, SMALL>(Xb, xrow, row_bytes, col_bytes);      \
    }
    if (n_out > 0) { ARROW_OUT(0) ARROW_OUT(1) ARROW_OUT(2) ARROW_OUT(3) }
#undef ARROW_OUT
    const uint32_t n_win = r.hi - r.mid;
#pragma unroll
    for (uint32_t q = 0; q < QB; ++q)
      if (q * kWinLanes < n_win) batch(e[q], n_win - q * kWinLanes);
    for (uint32_t at = QB * kWinLanes; at < n_win; at += kWinLanes) {           // rows of more than 64 window entries
      Entry m{0, 0.f};
      if (at + l < n_win) m = t_ent[r.mid + at + l];
      batch(m, n_win - at);
    }
    if (n_out > 0) {
      const float vo = l < n_out ? o.val : 0.f;
#define ARROW_OUT(O) vfma(acc, __int_as_float(row16_bcast<O>(__float_as_int(vo))), xo[O]);
      ARROW_OUT(0) ARROW_OUT(1) ARROW_OUT(2) ARROW_OUT(3)
#undef ARROW_OUT
      for (uint32_t j = r.lo + NO; j < r.mid; j += 4) {                         // further entries outside the window
        Entry m[4];
        V x[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) m[u] = t_ent[j + u < r.mid ? j + u : j];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) x[u] = j + u < r.mid ? load_row<VEC, SMALL>(Xb, m[u].xrow, row_bytes, col_bytes) : vzero<VEC>();
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) vfma(acc, j + u < r.mid ? m[u].val : 0.f, x[u]);
      }
    }
    if (lc.ok) {
      float* y = reinterpret_cast<float*>(reinterpret_cast<char*>(Y) + row_offset<SMALL>(r.y, row_bytes, col_bytes));
      if (accumulate) vadd(acc, vload_stream<VEC>(y));
      vstore_stream<VEC>(y, acc);
    }
    r = r_n; r_n = r_nn; o = o_n;
#pragma unroll
    for (int q = 0; q < QB; ++q) e[q] = e_n[q];
  }
}

// ---------------------------------------------------------------------------
// panel kernel: workgroup w = group * 8 + class keeps the accumulators of the group's kPanelRows
// head rows (one column slice of LPR * VEC columns) in LDS and runs on accelerator die w mod 8, so
// its entries -- those of the group whose staged head row is of that class -- only touch the
// die's eighth of the staged head.  Each of its kPanelBins lane groups streams one entry list,
// ordered by column window, then row: products are summed in registers while the row stays the
// same and added to the row's LDS accumulator when it changes (all class entries of a row are in
// one stream, so only one lane group ever touches an accumulator and no barrier is needed while
// streaming).  At the end the accumulators go to part[class][slot]; the combine kernel adds the
// eight class results of a row to Y in class order.
// ---------------------------------------------------------------------------
template <int VEC, int LPR, int U, bool SMALL>
__global__ __launch_bounds__(kPanelBins * LPR) void panel_kernel(
    const uint32_t* __restrict__ panel_ptr, const int32_t* __restrict__ panel_y,
    const Entry* __restrict__ ent, int64_t n_bins, int64_t n_slots, const float* __restrict__ Xh,
    float* __restrict__ part, int k) {
  using V = typename Vec<VEC>::type;
  constexpr int W = LPR * VEC;
  constexpr uint32_t kRowMask = (1u << kPanelRowShift) - 1u;
  constexpr int SG = 4 * LPR < 8 ? 8 : (4 * LPR > 32 ? 32 : 4 * LPR);
  constexpr int UU = U < SG ? U : SG;
  constexpr uint32_t kNone = 0xffffffffu;
  __shared__ __attribute__((aligned(16))) float acc[kPanelRows * W];
  __shared__ Entry strip[kPanelBins * SG];
  const int tid = threadIdx.x;
  const int l = tid % LPR;
  const int g = tid / LPR;
  const int c = l * VEC + blockIdx.y * W;
  const bool col_ok = c < k;
  const uint32_t row_bytes = 4u * (uint32_t)k;
  const uint32_t col_bytes = col_ok ? 4u * (uint32_t)c : 0u;
  for (int i = tid; i < kPanelRows * LPR; i += kPanelBins * LPR) vstore<VEC>(acc + i * VEC, vzero<VEC>());
  __syncthreads();
  const int64_t bin = (int64_t)blockIdx.x * kPanelBins + g;
  if (bin < n_bins) {
    const uint32_t lo = panel_ptr[bin], hi = panel_ptr[bin + 1];
    const char* base = reinterpret_cast<const char*>(Xh);
    Entry* grp = strip + g * SG;
    uint32_t cur = kNone;
    V a = vzero<VEC>();
    auto flush_to = [&](uint32_t r) {               // add the register sum to its accumulator, start row r
      if (cur != kNone) {
        float* ap = acc + cur * W + l * VEC;
        V t = vload<VEC>(ap);
        vadd(t, a);
        vstore<VEC>(ap, t);
      }
      cur = r;
      a = vzero<VEC>();
    };
    for (uint32_t b0 = lo; b0 < hi; b0 += SG) {
      const uint32_t nb = hi - b0 < (uint32_t)SG ? hi - b0 : (uint32_t)SG;
#pragma unroll
      for (int t = 0; t < SG / LPR; ++t) {
        const uint32_t idx = (uint32_t)(l + t * LPR);
        if (idx < nb) grp[idx] = ent[b0 + idx];
      }
      strip_sync();
      uint32_t j = 0;
      for (; j + UU <= nb; j += UU) {               // full rounds: nothing is predicated
        Entry e[UU];
        V x[UU];
#pragma unroll
        for (int u = 0; u < UU; ++u) e[u] = grp[j + u];
#pragma unroll
        for (int u = 0; u < UU; ++u)
          x[u] = load_row<VEC, SMALL>(base, (int32_t)((uint32_t)e[u].xrow & kRowMask), row_bytes, col_bytes);
        const uint32_t r0 = (uint32_t)e[0].xrow >> kPanelRowShift;
        const uint32_t r1 = (uint32_t)e[UU - 1].xrow >> kPanelRowShift;
        if (r0 == r1) {                             // the stream is ordered by row: the whole round is one row
          if (r0 != cur) flush_to(r0);
#pragma unroll
          for (int u = 0; u < UU; ++u) vfma(a, e[u].val, x[u]);
        } else {
#pragma unroll
          for (int u = 0; u < UU; ++u) {
            const uint32_t r = (uint32_t)e[u].xrow >> kPanelRowShift;
            if (r != cur) flush_to(r);
            vfma(a, e[u].val, x[u]);
          }
        }
      }
      for (; j < nb; ++j) {                         // the last, partly filled round of the stream
        const Entry e = grp[j];
        const V x = load_row<VEC, SMALL>(base, (int32_t)((uint32_t)e.xrow & kRowMask), row_bytes, col_bytes);
        const uint32_t r = (uint32_t)e.xrow >> kPanelRowShift;
        if (r != cur) flush_to(r);
        vfma(a, e.val, x);
      }
      strip_sync();
    }
    flush_to(kNone);
  }
  __syncthreads();
  const int64_t slot0 = (int64_t)(blockIdx.x / kDies) * kPanelRows;
  const int32_t* py = panel_y + slot0;
  float* out = part + ((size_t)(blockIdx.x % kDies) * (size_t)n_slots + (size_t)slot0) * (size_t)k;
  for (int r = g; r < kPanelRows; r += kPanelBins) {
    if (py[r] < 0 || !col_ok) continue;
    vstore<VEC>(out + (size_t)r * (size_t)k + c, vload<VEC>(acc + r * W + l * VEC));
  }
}

// Y[panel_y[slot]] += part[0][slot] + ... + part[7][slot], lane group per slot.
template <int VEC, int LPR>
__global__ __launch_bounds__(kBlock) void panel_combine_kernel(
    const int32_t* __restrict__ panel_y, int64_t n_slots, const float* __restrict__ part,
    float* __restrict__ Y, int k) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  const int64_t slot = (int64_t)blockIdx.x * GPB + threadIdx.x / LPR;
  const int c = (threadIdx.x % LPR) * VEC + blockIdx.y * (LPR * VEC);
  if (slot >= n_slots || c >= k) return;
  const int32_t y = panel_y[slot];
  if (y < 0) return;
  V p[kDies];
#pragma unroll
  for (int x = 0; x < kDies; ++x)
    p[x] = vload<VEC>(part + ((size_t)x * (size_t)n_slots + (size_t)slot) * (size_t)k + c);
  V acc = p[0];
#pragma unroll
  for (int x = 1; x < kDies; ++x) vadd(acc, p[x]);
  float* yp = Y + (size_t)y * (size_t)k + c;
  vadd(acc, vload<VEC>(yp));
  vstore_stream<VEC>(yp, acc);
}

// Sampled product over the panel entries: lane group per bin, NB entries at a time; the row
// vertex of an entry is looked up through the accumulator table.
template <int VEC, int LPR, int NB, bool SMALL>
__global__ __launch_bounds__(kBlock) void sddmm_panel_kernel(
    const uint32_t* __restrict__ panel_ptr, const int32_t* __restrict__ panel_y,
    const Entry* __restrict__ ent, const uint32_t* __restrict__ emap, int64_t n_bins,
    const float* __restrict__ U, const float* __restrict__ Vh, float* __restrict__ S, int k,
    int slices) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  constexpr int W = LPR * VEC;
  constexpr int SPAN = LPR / NB;
  constexpr uint32_t kRowMask = (1u << kPanelRowShift) - 1u;
  const int l = threadIdx.x % LPR;
  const int64_t bin = (int64_t)blockIdx.x * GPB + threadIdx.x / LPR;
  if (bin >= n_bins) return;
  const uint32_t lo = panel_ptr[bin], hi = panel_ptr[bin + 1];
  const int32_t* py = panel_y + (bin / (kDies * kPanelBins)) * kPanelRows;
  const uint32_t row_bytes = 4u * (uint32_t)k;
  const char* base = reinterpret_cast<const char*>(Vh);
  for (uint32_t j = lo; j < hi; j += NB) {
    int32_t xr[NB], ur[NB];
    float p[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const uint32_t code = (uint32_t)ent[j + u < hi ? j + u : lo].xrow;
      xr[u] = (int32_t)(code & kRowMask);
      ur[u] = py[code >> kPanelRowShift];
      p[u] = 0.f;
    }
    for (int sl = 0; sl < slices; ++sl) {
      const int c = l * VEC + sl * W;
      const bool col_ok = c < k;
      const uint32_t col_bytes = col_ok ? 4u * (uint32_t)c : 0u;
      V x[NB], uu[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const bool ok = j + u < hi && col_ok;
        x[u] = ok ? load_row<VEC, SMALL>(base, xr[u], row_bytes, col_bytes) : vzero<VEC>();
        uu[u] = ok ? vload<VEC>(U + (size_t)ur[u] * (size_t)k + c) : vzero<VEC>();
      }
#pragma unroll
      for (int u = 0; u < NB; ++u) p[u] += vdot(uu[u], x[u]);
    }
    const float dot = group_reduce<NB, LPR>(p, l);
    const uint32_t mine = j + (uint32_t)(l / SPAN);
    if (l % SPAN == 0 && mine < hi) S[emap ? emap[mine] : mine] = ent[mine].val * dot;
  }
}

// ---------------------------------------------------------------------------
// corner kernel: workgroup = one work item = a run of tiles of one row panel (kCornerTile head rows)
// of the dense corner.  The panel's accumulators (one column slice of W = LPR * VEC columns) stay
// in LDS for the whole item.  Per tile the kCornerTile staged head rows it covers are copied into
// LDS with coalesced loads (the next tile's rows are already on their way while the current tile
// is worked on), then every lane group streams one run of the tile's entries: an entry costs one
// LDS row read instead of a row gathered through the caches, and products are summed in registers
// while the row stays the same.  Runs never share a row, so an accumulator has one owner per tile
// and the workgroup barriers between tiles order the owners: no atomics, a fixed summation order.
// Results go to part[item]; the combine kernel adds the items of a panel to Y in item order.
// (A form with one wavefront per run, its 64 lanes across the slice and every entry broadcast
// from a lane so that row changes are scalar branches, was measured at 2.8 ms against 1.8 ms for
// this one on the same 60 M entries.)
// ---------------------------------------------------------------------------
constexpr int kCornerBlock = 1024;

template <int VEC, int LPR, int U>
__global__ __launch_bounds__(kCornerBlock) void corner_kernel(
    const uint32_t* __restrict__ tiles, const uint32_t* __restrict__ items,
    const Entry* __restrict__ ent, const float* __restrict__ Xh, float* __restrict__ part, int k) {
  using V = typename Vec<VEC>::type;
  constexpr int W = LPR * VEC;
  constexpr int GPB = kCornerBlock / LPR;
  constexpr int SG = 4 * LPR < 8 ? 8 : (4 * LPR > 32 ? 32 : 4 * LPR);
  constexpr int UU = U < SG ? U : SG;
  constexpr int NL = (kCornerTile * LPR + kCornerBlock - 1) / kCornerBlock;   // tile elements a thread copies
  constexpr int NA = SG / LPR > 0 ? SG / LPR : 1;     // entries of a batch a lane fetches
  constexpr uint32_t kNone = 0xffffffffu;
  __shared__ __attribute__((aligned(16))) float acc[kCornerTile * W];
  __shared__ __attribute__((aligned(16))) float xt[kCornerTile * W];
  __shared__ Entry strip[GPB * SG];
  const int tid = threadIdx.x;
  const int l = tid % LPR;
  const int g = tid / LPR;
  const int c = l * VEC + blockIdx.y * W;
  const bool col_ok = c < k;
  const uint32_t t_begin = items[blockIdx.x], t_end = items[blockIdx.x + 1];
  for (int i = tid; i < kCornerTile * LPR; i += kCornerBlock) vstore<VEC>(acc + i * VEC, vzero<VEC>());
  // element i of a tile copy: staged row i / LPR, lane slot i % LPR (consecutive threads read
  // consecutive columns of one row)
  V nxt[NL];
  auto fetch = [&](uint32_t t) {
    const uint32_t col0 = tiles[(size_t)t * kCornerTileWords + kCornerRuns + 1];
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int i = tid + j * kCornerBlock;
      const int r = i / LPR, cc = (i % LPR) * VEC + blockIdx.y * W;
      nxt[j] = (i < kCornerTile * LPR && cc < k) ? vload<VEC>(Xh + (size_t)(col0 + r) * (size_t)k + cc) : vzero<VEC>();
    }
  };
  fetch(t_begin);
  Entry* grp = strip + g * SG;
  // The first run a lane group takes from a tile, and the first SG entries of that run, are fetched
  // one tile ahead: a run holds about that many entries, so without this every tile would start
  // with two dependent memory latencies (run offsets, then entries) before its first LDS read.
  uint32_t lo_c = 0, hi_c = 0, lo_n = 0, hi_n = 0;
  Entry ahead_c[NA], ahead_n[NA];
  auto fetch_bounds = [&](uint32_t t, uint32_t& lo, uint32_t& hi) {
    lo = hi = 0;
    if (g < kCornerRuns) { lo = tiles[(size_t)t * kCornerTileWords + g]; hi = tiles[(size_t)t * kCornerTileWords + g + 1]; }
  };
  auto fetch_entries = [&](uint32_t lo, uint32_t hi, Entry (&out)[NA]) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const uint32_t idx = lo + (uint32_t)(l + q * LPR);
      out[q] = ent[idx < hi ? idx : (lo < hi ? lo : 0u)];
    }
  };
  fetch_bounds(t_begin, lo_c, hi_c);
  fetch_entries(lo_c, hi_c, ahead_c);
  for (uint32_t t = t_begin; t < t_end; ++t) {
    const bool more = t + 1 < t_end;
    if (more) fetch_bounds(t + 1, lo_n, hi_n);
    __syncthreads();                                  // the previous tile's reads and flushes are done
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int i = tid + j * kCornerBlock;
      if (i < kCornerTile * LPR) vstore<VEC>(xt + i * VEC, nxt[j]);
    }
    if (more) fetch(t + 1);
    __syncthreads();
    if (more) fetch_entries(lo_n, hi_n, ahead_n);
    const uint32_t* tw = tiles + (size_t)t * kCornerTileWords;
    for (int run = g; run < kCornerRuns; run += GPB) {
      const bool first = run == g;
      const uint32_t lo = first ? lo_c : tw[run], hi = first ? hi_c : tw[run + 1];
      uint32_t cur = kNone;
      V a = vzero<VEC>();
      auto flush_to = [&](uint32_t r) {               // add the register sum to its accumulator, start row r
        if (cur != kNone) {
          float* ap = acc + cur * W + l * VEC;
          V s = vload<VEC>(ap);
          vadd(s, a);
          vstore<VEC>(ap, s);
        }
        cur = r;
        a = vzero<VEC>();
      };
      for (uint32_t b0 = lo; b0 < hi; b0 += SG) {
        const uint32_t nb = hi - b0 < (uint32_t)SG ? hi - b0 : (uint32_t)SG;
        if (first && b0 == lo) {                      // this batch was fetched while the previous tile ran
#pragma unroll
          for (int q = 0; q < NA; ++q) {
            const uint32_t idx = (uint32_t)(l + q * LPR);
            if (idx < nb) grp[idx] = ahead_c[q];
          }
        } else {
#pragma unroll
          for (int q = 0; q < NA; ++q) {
            const uint32_t idx = (uint32_t)(l + q * LPR);
            if (idx < nb) grp[idx] = ent[b0 + idx];
          }
        }
        strip_sync();
        uint32_t j = 0;
        for (; j + UU <= nb; j += UU) {               // full rounds: nothing is predicated
          Entry e[UU];
          V x[UU];
#pragma unroll
          for (int u = 0; u < UU; ++u) e[u] = grp[j + u];
#pragma unroll
          for (int u = 0; u < UU; ++u) x[u] = vload<VEC>(xt + ((uint32_t)e[u].xrow & 0xffffu) * W + l * VEC);
#pragma unroll
          for (int u = 0; u < UU; ++u) {
            const uint32_t r = (uint32_t)e[u].xrow >> 16;
            if (r != cur) flush_to(r);
            vfma(a, e[u].val, x[u]);
          }
        }
        for (; j < nb; ++j) {                         // the last, partly filled round of the batch
          const Entry e = grp[j];
          const V x = vload<VEC>(xt + ((uint32_t)e.xrow & 0xffffu) * W + l * VEC);
          const uint32_t r = (uint32_t)e.xrow >> 16;
          if (r != cur) flush_to(r);
          vfma(a, e.val, x);
        }
        strip_sync();
      }
      flush_to(kNone);
    }
    lo_c = lo_n; hi_c = hi_n;
#pragma unroll
    for (int q = 0; q < NA; ++q) ahead_c[q] = ahead_n[q];
  }
  __syncthreads();
  float* out = part + (size_t)blockIdx.x * kCornerTile * (size_t)k;
  if (col_ok)
    for (int r = g; r < kCornerTile; r += GPB)
      vstore_stream<VEC>(out + (size_t)r * (size_t)k + c, vload<VEC>(acc + r * W + l * VEC));
}

// Y[corner_y[p]] += part[it][p % kCornerTile] summed over the items it of p's row panel, in item
// order.  Lane group per corner row.
template <int VEC, int LPR>
__global__ __launch_bounds__(kBlock) void corner_combine_kernel(
    const uint32_t* __restrict__ panel_ptr, const int32_t* __restrict__ corner_y, int64_t corner,
    const float* __restrict__ part, float* __restrict__ Y, int k) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  const int64_t p = (int64_t)blockIdx.x * GPB + threadIdx.x / LPR;
  const int c = (threadIdx.x % LPR) * VEC + blockIdx.y * (LPR * VEC);
  if (p >= corner || c >= k) return;
  const uint32_t it0 = panel_ptr[p / kCornerTile], it1 = panel_ptr[p / kCornerTile + 1];
  if (it0 == it1) return;
  const float* src = part + ((size_t)it0 * kCornerTile + (size_t)(p % kCornerTile)) * (size_t)k + c;
  V acc = vload_stream<VEC>(src);
  for (uint32_t it = it0 + 1; it < it1; ++it) {
    src += (size_t)kCornerTile * (size_t)k;
    vadd(acc, vload_stream<VEC>(src));
  }
  float* yp = Y + (size_t)corner_y[p] * (size_t)k + c;
  vadd(acc, vload_stream<VEC>(yp));
  vstore_stream<VEC>(yp, acc);
}

// Sampled product over the corner tiles: workgroup per tile, lane group per run, NB entries at a
// time; the row vertex of an entry comes from the corner row table, its V row from the staged head.
template <int VEC, int LPR, int NB, bool SMALL>
__global__ __launch_bounds__(kBlock) void sddmm_corner_kernel(
    const uint32_t* __restrict__ tiles, const int32_t* __restrict__ corner_y,
    const Entry* __restrict__ ent, const uint32_t* __restrict__ emap, const float* __restrict__ U,
    const float* __restrict__ Vh, float* __restrict__ S, int k, int slices) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  constexpr int W = LPR * VEC;
  constexpr int SPAN = LPR / NB;
  const int l = threadIdx.x % LPR;
  const uint32_t* tw = tiles + (size_t)blockIdx.x * kCornerTileWords;
  const uint32_t col0 = tw[kCornerRuns + 1];
  const int32_t* py = corner_y + (size_t)tw[kCornerRuns + 2] * kCornerTile;
  const uint32_t row_bytes = 4u * (uint32_t)k;
  const char* base = reinterpret_cast<const char*>(Vh);
  for (int run = threadIdx.x / LPR; run < kCornerRuns; run += GPB) {
    const uint32_t lo = tw[run], hi = tw[run + 1];
    for (uint32_t j = lo; j < hi; j += NB) {
      int32_t xr[NB], ur[NB];
      float p[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const uint32_t code = (uint32_t)ent[j + u < hi ? j + u : lo].xrow;
        xr[u] = (int32_t)(col0 + (code & 0xffffu));
        ur[u] = py[code >> 16];
        p[u] = 0.f;
      }
      for (int sl = 0; sl < slices; ++sl) {
        const int c = l * VEC + sl * W;
        const bool col_ok = c < k;
        const uint32_t col_bytes = col_ok ? 4u * (uint32_t)c : 0u;
        V x[NB], uu[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          const bool ok = j + u < hi && col_ok;
          x[u] = ok ? load_row<VEC, SMALL>(base, xr[u], row_bytes, col_bytes) : vzero<VEC>();
          uu[u] = ok ? vload<VEC>(U + (size_t)ur[u] * (size_t)k + c) : vzero<VEC>();
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) p[u] += vdot(uu[u], x[u]);
      }
      const float dot = group_reduce<NB, LPR>(p, l);
      const uint32_t mine = j + (uint32_t)(l / SPAN);
      if (l % SPAN == 0 && mine < hi) S[emap ? emap[mine] : mine] = ent[mine].val * dot;
    }
  }
}

// One wavefront per split row: its partial vectors (consecutive slots) are summed slot-strided by the G lane groups, then
// combined by the same butterfly.  Rows of many partial vectors are shared by the wavefronts of the workgroup, and eight
// loads are on their way instead of four: the launch lasted as long as one wavefront took for the longest row
// (a hub of 2048 partial vectors, 64 rounds of loads one after the other).  Such rows are usually neighbours, so
// a workgroup takes rows that are far apart.  Partial vectors shorter than a line are left to one wavefront per row, neighbours
// beside each other: they share lines, and 16 and more lane groups take them (Chung-Lu 500k, k = 16, 5.6 us a launch, shared
// 7.6).  Chung-Lu 2m k = 32 25.9 -> 13.4 us, R-MAT 1m k = 64 13.3 -> 10.9,
// R-MAT 8m k = 128, where memory bounds it, 320 -> 308.  (Sixteen wavefronts per workgroup: 18, 16 and 346 us; a lane
// group per short row: 22, 18 and 343.)
template <int VEC, int LPR>
__global__ __launch_bounds__(kBlock) void reduce_kernel(
    const uint32_t* __restrict__ split_ptr, const int32_t* __restrict__ split_y, int64_t n_split,
    const float* __restrict__ partials, float* __restrict__ Y, int k, int width, int accumulate) {
  using V = typename Vec<VEC>::type;
  constexpr int WPB = kBlock / 64;
  constexpr uint32_t G = 64 / LPR, kLong = 16 * G;
  __shared__ V s_part[2][WPB][LPR];
  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  const uint32_t g = lane / LPR, l = lane % LPR;
  const LaneColumns lc = lane_columns<VEC>((int)l, blockIdx.y * width, k, width);
  const float* __restrict__ Pc = partials + (lc.ok ? lc.c : 0);
  const bool apart = LPR * VEC >= 32 && k >= 32;
  // lane t holds what belongs to the row of wavefront t
  const int64_t mine = !apart ? (int64_t)blockIdx.x * WPB + lane % WPB : (int64_t)blockIdx.x + (int64_t)(lane % WPB) * gridDim.x;
  uint32_t lo_of = 0, hi_of = 0;
  int32_t y_of = 0;
  if (mine < n_split) { lo_of = split_ptr[mine]; hi_of = split_ptr[mine + 1]; y_of = split_y[mine]; }
  auto of = [](auto v, int t) { return (decltype(v))__builtin_amdgcn_readlane((int)v, t); };
  auto sum = [&](uint32_t s, uint32_t end, uint32_t step) {
    V acc = vzero<VEC>();
    if constexpr (LPR * VEC >= 16) {
      for (; s + 7 * step < end; s += 8 * step) {
        V p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = vload_stream<VEC>(Pc + (size_t)(s + u * step) * (size_t)k);
#pragma unroll
        for (int m = 1; m < 8; m *= 2)
#pragma unroll
          for (int u = 0; u < 8; u += 2 * m) vadd(p[u], p[u + m]);
        vadd(acc, p[0]);
      }
    }
    for (; s + 3 * step < end; s += 4 * step) {
      V p[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) p[u] = vload_stream<VEC>(Pc + (size_t)(s + u * step) * (size_t)k);
      vadd(p[0], p[1]); vadd(p[2], p[3]); vadd(p[0], p[2]); vadd(acc, p[0]);
    }
    V p[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) if (s + u * step < end) p[u] = vload_stream<VEC>(Pc + (size_t)(s + u * step) * (size_t)k);
#pragma unroll
    for (int u = 0; u < 3; ++u) if (s + u * step < end) vadd(acc, p[u]);
#pragma unroll
    for (int m = LPR; m < 64; m <<= 1) vadd(acc, vshfl_xor(acc, m));
    return acc;
  };
  auto store = [&](int32_t row, V acc) {
    if (g != 0 || !lc.ok) return;
    float* to = Y + (size_t)row * (size_t)k + lc.c;
    if (accumulate) vadd(acc, vload_stream<VEC>(to));
    vstore_stream<VEC>(to, acc);
  };
  uint32_t shared = (uint32_t)__ballot(apart && lane < WPB && hi_of - lo_of >= kLong);
  if (!(shared >> wave & 1u)) {
    const uint32_t lo = of(lo_of, wave), hi = of(hi_of, wave);
    if (lo < hi) store(of(y_of, wave), sum(lo + g, hi, G));
  }
  for (int half = 0; shared; half ^= 1, shared &= shared - 1) {
    const int t = __ffs(shared) - 1;
    const V part = sum(of(lo_of, t) + (uint32_t)wave * G + g, of(hi_of, t), WPB * G);
    if (g == 0) s_part[half][wave][l] = part;
    __syncthreads();                     // (the other half is read no more: its readers have come this far)
    if (wave == t) {
      V acc = s_part[half][0][l];
      for (int w = 1; w < WPB; ++w) vadd(acc, s_part[half][w][l]);
      store(of(y_of, t), acc);
    }
  }
}

template <int VEC, int LPR>
__global__ __launch_bounds__(kBlock) void gather_kernel(const int32_t* __restrict__ perm,
                                                        int64_t n_i, const float* __restrict__ X,
                                                        float* __restrict__ Xp, int k, int stride) {
  constexpr int GPB = kBlock / LPR;
  const int64_t p = (int64_t)blockIdx.x * GPB + threadIdx.x / LPR;
  const LaneColumns lc = lane_columns<VEC>(threadIdx.x % LPR, blockIdx.y * (LPR * VEC), k);
  const int c = lc.c;
  if (p >= n_i || !lc.ok) return;
  gstore<VEC>(Xp + (size_t)p * (size_t)stride + c, gload<VEC>(X + (size_t)perm[p] * (size_t)k + c));
}

}  // namespace

int launch_product(ProductArgs a, int parts, int64_t n_pieces, int64_t n_rows, int64_t n_empty, bool die_queues,
                   bool windows, int64_t x_rows, int32_t kc, void* stream) {
  const Shape s = pick_output_shape(a.k, kc, a.accumulate != 0);
  const bool small = small_matrix(x_rows, a.k);    // the staged buffer has at most as many rows as X
  const int64_t n_long = a.n_chunks;
  if (!(parts & kPartChunks)) a.n_chunks = 0;
  a.begin[0] = 0; a.count[0] = a.n_chunks;
  a.items[0] = kBlock / 64;
  a.begin[1] = 0; a.count[1] = parts & kPartPieces ? n_pieces : 0;
  a.begin[2] = n_pieces; a.count[2] = parts & kPartShort ? n_rows - n_pieces - n_empty : 0;
  a.begin[3] = n_rows - n_empty; a.count[3] = parts & kPartShort ? n_empty : 0;
  // Items per workgroup: as many as the descriptor arrays hold where that still gives a few thousand
  // workgroups, fewer (down to one per lane group) for short lists, which would otherwise leave most
  // of the 256 compute units without one (71 K pieces of R-MAT 1m, k = 64: 56 -> 44 us).  Pieces are
  // up to three times as long as short rows.
  const int least = kBlock / s.lpr < kItemsPerGroupBlock ? kBlock / s.lpr : kItemsPerGroupBlock;
  auto items_of = [&](int p, int64_t count) {
    int items = kItemsPerGroupBlock;
    if (!(p == 1 && die_queues)) {
      if (p == 1) items = kItemsPerGroupBlock / 4;
      while (items > least && count < (int64_t)items * 2048) items >>= 1;
    }
    return items;
  };
  for (int p = 1; p < 4; ++p) a.items[p] = items_of(p, a.count[p]);
  // A piece is some 30 entries: eight to sixteen lane groups finish one in a round or two of row
  // loads where a lane group on its own needs four to six in a row.  Worth the idle lanes only where
  // latency decides, in a list of at most a few pieces per SIMD.
  a.piece_waves = !die_queues && s.lpr <= 8 && a.count[1] <= kPieceWavesMax;
  // Four lane groups too (33 to 64 columns, and slices of wider rows) where four workgroups to a compute unit or fewer come of it, or more than the six that it holds
  // but no more than some three rounds; just below six two ranks in five lose by up to 10 %.  (Ten thousand lists of 2500 to 100 K vertices, R-MAT and Chung-Lu: up
  // to 1024 workgroups 0.74 to 1.05 times the time, 0.93 on average, 1024 to 1536 0.98, 1536 to 4000 0.97, beyond 1.0 to 1.04.  us: R-MAT 2504, k = 40, 6.7 -> 5.2;
  // 12.6 K, 10.3 -> 9.3; Chung-Lu 15 K, 14.2 -> 13.1; but R-MAT 3850, k = 200, 8.0 and 8.8, Chung-Lu 97 K, k = 40, 29.6 and 31.9.)
  // Of the workgroups of all lists that share the launch of a product that is not profiled: what adds up a piece decides about the bits of its sum.
  if (!die_queues && !windows && s.lpr == 16 && a.count[1] > 0) {
    const int together = a.together ? a.together : parts;
    const int64_t counts[3] = {together & kPartChunks ? n_long : 0, n_pieces, together & kPartShort ? n_rows - n_pieces - n_empty : 0};
    int64_t groups = 0;
    for (int p = 0; p < 3; ++p) groups += ceil_div(ceil_div(counts[p], p < 2 ? kBlock / 64 : items_of(p, counts[p])), kDies) * kDies * s.slices;
    a.piece_waves = groups <= 4 * kComputeUnits || (groups > 6 * kComputeUnits && groups <= 4000);
  }
  if (a.piece_waves) a.items[1] = kBlock / 64;
  a.run = windows && !die_queues ? die_run(ceil_div(a.count[0], a.items[0])) : 0;
  int64_t total = 0;
  for (int p = 0; p < 4; ++p) {
    const int64_t blocks = ceil_div(ceil_div(a.count[p], a.items[p]), kDies) * kDies;
    total += blocks * s.slices;
    if (total > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    a.blocks[p] = (uint32_t)blocks;
  }
  a.slices = (uint32_t)s.slices;
  a.width = s.width;
  // Two sets of dies (slice_block) wherever there is an even number of slices that share no lines, or hardly any: an L2
  // then holds and fetches half of every row of X (us, all slices on every die / two sets / four; R-MAT unless said
  // otherwise): 10k, k = 256: 20.7 / 20.0 / 17.1; 65k, 256: 76.7 / 68.1 / 71.5; 131k, 256: 200 / 190 / 174; 180k, 256: 256 /
  // 245 / 251; 200k, 384: 325 / 313 / 324; 65k, 512: 174 / 152 / 146; 524k, 128: 419 / 412; Chung-Lu 60k, 256: 82.5 / 76.9 / 74.2,
  // 250k: 336 / 318 / 327.  Narrow slices that end inside a line are fetched by both sets (R-MAT 17.5k, k = 70: 15.1 / 16.5;
  // but 65k, k = 260, 102 / 94).  Beyond twice the cache behind the L2s it depends on the graph (k = 128: Chung-Lu 900k, 460 MB,
  // 725 / 718, 1.5m 1224 / 1228, 2m 1728 / 1737; R-MAT 1.5m 1568 / 1520, 4m 5537 / 5500, 8m 11620 / 11680; 800k, k = 256, 820 MB,
  // 907 / 921).
  // Slices of unequal width would leave dies idle (k = 96, 64 + 32 columns: 20.9 / 22.4).
  const bool lines = s.width % 32 == 0 || s.width >= 128, equal = a.k > (s.slices - 1) * s.width + s.width * 3 / 4;
  // And an X that an L2 nearly holds gains nothing (10k, k = 128: 14.7 / 15.0).
  const int64_t x_bytes = x_rows * a.k * (int64_t)sizeof(float);
  const bool sets = !die_queues && s.slices % 2 == 0 && lines && equal && x_bytes >= kDieSetsLeast && x_bytes <= kDieSetsMost;
  a.sets_log = sets ? 1 : 0;
  // Stencils, meshes, bands: hardly any long rows or pieces of them, whichever launch those are in, and enough
  // batches for every compute unit to have several in turn.  (1m rows of 3 to 8 random entries and one in
  // twenty of 20 to 40, k = 96: 448 us with the flow kernel, 443 without; one in five: 735 and 727; 200k rows,
  // one in fifty of 20 to 40 and one in 500 of 300, k = 128: 116 and 119.)
  const bool flow = a.longest_short * (int64_t)kItemsPerGroupBlock <= kRowsStage &&
                    a.count[2] >= kItemsPerGroupBlock * kFlowLeast && a.count[2] >= 64 * (n_long + n_pieces);
  return dispatch_shape(s, [&](auto V, auto L) -> int {
    constexpr int VEC = decltype(V)::value, LPR = decltype(L)::value;
    if (windows && a.blocks[0] > 0) {
      dim3 grid(a.blocks[0] << a.sets_log, a.slices >> a.sets_log);
      if (small) hipLaunchKernelGGL((chunks_kernel<VEC, LPR, true>), grid, dim3(kBlock), 0, (hipStream_t)stream, a);
      else hipLaunchKernelGGL((chunks_kernel<VEC, LPR, false>), grid, dim3(kBlock), 0, (hipStream_t)stream, a);
      total -= (int64_t)a.blocks[0] * a.slices;
      a.blocks[0] = 0;
    }
    if (flow) {
      const int64_t batches = ceil_div(a.count[2], (int64_t)kItemsPerGroupBlock);
      const int64_t blocks = std::max(ceil_div(batches, (int64_t)kFlowBatches), std::min(batches, kFlowBlocks));
      dim3 grid((unsigned)(ceil_div(blocks, kDies) * kDies), a.slices);
      if (small) hipLaunchKernelGGL((flow_kernel<VEC, LPR, true>), grid, dim3(kBlock), 0, (hipStream_t)stream, a);
      else hipLaunchKernelGGL((flow_kernel<VEC, LPR, false>), grid, dim3(kBlock), 0, (hipStream_t)stream, a);
      total -= (int64_t)a.blocks[2] * a.slices;
      a.blocks[2] = 0;
    }
    if (total > 0) {
      if (small) hipLaunchKernelGGL((product_kernel<VEC, LPR, true>), dim3((unsigned)total), dim3(kBlock), 0, (hipStream_t)stream, a);
      else hipLaunchKernelGGL((product_kernel<VEC, LPR, false>), dim3((unsigned)total), dim3(kBlock), 0, (hipStream_t)stream, a);
    }
    return (int)hipGetLastError();
  });
}

bool same_shape(int32_t k, int32_t kc_a, int32_t kc_b, bool accumulate) {
  const Shape a = pick_output_shape(k, kc_a, accumulate), b = pick_output_shape(k, kc_b, accumulate);
  return a.vec == b.vec && a.lpr == b.lpr && a.width == b.width;
}

int launch_reduce(const uint32_t* split_ptr, const int32_t* split_y, int64_t n_split,
                  const float* partials, float* Y, int32_t k, bool accumulate, void* stream) {
  if (n_split <= 0) return 0;
  const Shape s = pick_output_shape(k, 0, accumulate);
  return dispatch_shape(s, [&](auto V, auto L) -> int {
    constexpr int VEC = decltype(V)::value, LPR = decltype(L)::value;
    const int64_t blocks = ceil_div(n_split, kBlock / 64);
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)blocks, (unsigned)s.slices);
    hipLaunchKernelGGL((reduce_kernel<VEC, LPR>), grid, dim3(kBlock), 0, (hipStream_t)stream,
                       split_ptr, split_y, n_split, partials, Y, (int)k, s.width, accumulate ? 1 : 0);
    return (int)hipGetLastError();
  });
}

int launch_gather(const int32_t* perm, int64_t n_i, const float* X, float* Xp, int32_t k,
                  int32_t stride, void* stream) {
  if (n_i <= 0) return 0;
  const Shape s = pick_shape(k, 0);
  return dispatch_shape(s, [&](auto V, auto L) -> int {
    constexpr int VEC = decltype(V)::value, LPR = decltype(L)::value;
    const int64_t blocks = ceil_div(n_i, kBlock / LPR);
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)blocks, (unsigned)s.slices);
    hipLaunchKernelGGL((gather_kernel<VEC, LPR>), grid, dim3(kBlock), 0, (hipStream_t)stream, perm,
                       n_i, X, Xp, (int)k, (int)stride);
    return (int)hipGetLastError();
  });
}

int launch_window(const WindowTile* tiles, int64_t n_tiles, int64_t max_span, int64_t nnz, const uint32_t* wrow_ptr,
                  const uint32_t* wrow_mid, const int32_t* wrow_y, const Entry* entries,
                  const int32_t* perm, const float* X, int64_t x_rows, float* Y, int32_t k, bool accumulate,
                  void* stream) {
  if (n_tiles <= 0) return 0;
  // the widest slice whose window fits: 64, 32 or 16 columns (4, 2 or 1 per lane), 8 for the widest
  // spans; no wider than k needs
  int vec = 4, most = kWinColumns;
  while (vec > 1 && (k <= most / 2 || max_span * most > kWinFloats)) { vec >>= 1; most >>= 1; }
  if (max_span * most > kWinFloats) most = 8;
  if (max_span * most > kWinFloats) return (int)hipErrorInvalidValue;
  // a slice that adds to Y must not reach back into the one before it (see pick_shape)
  int slices = (int)ceil_div(k, most);
  int width = (int)ceil_div(ceil_div(k, slices), vec) * vec;
  if (accumulate && slices > 1 && k - (slices - 1) * width < vec) {
    vec = 1;
    if (most > 16) most = 16;
    slices = (int)ceil_div(k, most);
    width = (int)ceil_div(k, slices);
  }
  // Several workgroups stage the same window and share its rows where that fills the compute units better: by the number of
  // rounds of workgroups times the time that one takes for its window and its share of the entries.  A tile's workgroups run on
  // one die, so the rounds are those of the die with most tiles (14 tiles in three slices, k = 141: six workgroups a tile are
  // 252, but 36 for the 32 compute units of six dies: 29.6 us, with four a tile 24.5).  (Tiles of 512 rows
  // with 30 to 60 entries, 1 / 2 / 3 / 4 / 6 workgroups a tile, us: k = 64, 130 tiles 44 / 45 / 36 / 41 / 42, 180 47 / 49 / 51 / 44 /
  // 53, 258 74 / 63 / 60 / 62 / 67, 380 78 / 67 / 75 / 74 / 85, 700 129 / 137 / 141 / 153 / 174; k = 32, 70 tiles 37 / 23 / 19 / 18 / 16,
  // 130 49 / 32 / 26 / 29 / 29; k = 128, 512 tiles 155 / - ; two workgroups of one compute unit share its time: k = 16, 380
  // tiles 39 / 37 / 39 / 38 / 43, 700 65 / 70 / 72 / 72 / 82.)
  int parts = 1;
  double best = 0.0;
  const double tile_nnz = (double)nnz / (double)n_tiles;
  for (int p = 1; p <= kWinParts; p += p < 4 ? 1 : 2) {
    const double rounds = (double)ceil_div(ceil_div(n_tiles, kDies) * slices * p, kComputeUnits / kDies);
    const double cost = rounds * (kWinStage * (double)max_span + tile_nnz / p);
    if (p == 1 || cost < best) { best = cost; parts = p; }
  }
  const int64_t blocks = ceil_div(n_tiles, kDies) * kDies * slices * parts;
  if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
  const bool small = small_matrix(x_rows, k);
  // A compute unit takes two workgroups where two windows fit it: one sums while the other waits for its window.  Of 16
  // wavefronts each where a lane has one column (of 64 registers it misses one or two, stored once and loaded once a row; 512 tiles, k = 8 / 16: 59.6 -> 43.0, 61.1 -> 45.3
  // us; 1367, 16: 130 -> 93), of 8 each where it has two, which pays from three a compute unit on (781 tiles, k = 24: 89.7 ->
  // 86.6; 976, 20: 120.5 -> 114.1; 1953, 32: 184 -> 176; but 511, 32: 66.9 -> 71.3).  Where no die has more workgroups than compute units there is nothing
  // for a second one (196 tiles, k = 8, 21.4 us in the large form, 22.3 in this one).
  const bool shared = ceil_div(n_tiles, kDies) * slices * parts > kComputeUnits / kDies;
  const bool half = shared && max_span * (int64_t)width <= kWinFloatsHalf && (vec == 1 || (vec == 2 && n_tiles * slices * parts >= kWinHalfTiles));
#define ARROW_LAUNCH(VEC, SM, BLOCK, FLOATS)                                                                              \
  hipLaunchKernelGGL((window_kernel<VEC, SM, BLOCK, FLOATS>), dim3((unsigned)blocks), dim3(BLOCK), 0, (hipStream_t)stream, tiles, \
                     n_tiles, wrow_ptr, wrow_mid, wrow_y, entries, perm, X, Y, (int)k, width, slices, parts, accumulate ? 1 : 0)
#define ARROW_SMALL(VEC, BLOCK, FLOATS) \
  if (small) ARROW_LAUNCH(VEC, true, BLOCK, FLOATS); else ARROW_LAUNCH(VEC, false, BLOCK, FLOATS)
  if (vec == 4) { ARROW_SMALL(4, kWinBlock, kWinFloats); }
  else if (vec == 2 && half) { ARROW_SMALL(2, kWinBlockHalf, kWinFloatsHalf); }
  else if (vec == 2) { ARROW_SMALL(2, kWinBlock, kWinFloats); }
  else if (half) { ARROW_SMALL(1, kWinBlock, kWinFloatsHalf); }
  else { ARROW_SMALL(1, kWinBlock, kWinFloats); }
#undef ARROW_SMALL
#undef ARROW_LAUNCH
  return (int)hipGetLastError();
}

namespace {
// (VEC, LPR) with at most 32 lanes per row: the panel kernel runs kPanelBins lane groups per workgroup
template <typename F>
int dispatch_narrow(const Shape& s, F&& f) {
#define ARROW_CASE(V, L) \
  if (s.vec == V && s.lpr == L) return f(std::integral_constant<int, V>{}, std::integral_constant<int, L>{});
#define ARROW_CASES(V) ARROW_CASE(V, 1) ARROW_CASE(V, 2) ARROW_CASE(V, 4) ARROW_CASE(V, 8) ARROW_CASE(V, 16) ARROW_CASE(V, 32)
  ARROW_CASES(4)
  ARROW_CASES(2)
  ARROW_CASES(1)
#undef ARROW_CASES
#undef ARROW_CASE
  return (int)hipErrorInvalidValue;
}
}  // namespace

int launch_panel(const uint32_t* panel_ptr, const int32_t* panel_y, const Entry* entries,
                 int64_t n_groups, const float* Xh, int64_t xh_rows, float* part, int32_t k, void* stream) {
  if (n_groups <= 0) return 0;
  const int vec = (k % 4 == 0) ? 4 : (k % 2 == 0) ? 2 : 1;
  const Shape s = pick_shape(k, 32 * vec, true);         // at most 32 lanes per row: LDS rows of at most 128 floats
  const bool small = small_matrix(xh_rows, k);
  return dispatch_narrow(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value;
    const int64_t blocks = n_groups * kDies;          // workgroup id mod 8 = column class = die
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    const int64_t n_bins = blocks * kPanelBins, n_slots = n_groups * kPanelRows;
    dim3 grid((unsigned)blocks, (unsigned)s.slices);
    if (small)
      hipLaunchKernelGGL((panel_kernel<VEC, LPR, 8, true>), grid, dim3(kPanelBins * LPR), 0, (hipStream_t)stream,
                         panel_ptr, panel_y, entries, n_bins, n_slots, Xh, part, (int)k);
    else
      hipLaunchKernelGGL((panel_kernel<VEC, LPR, 8, false>), grid, dim3(kPanelBins * LPR), 0, (hipStream_t)stream,
                         panel_ptr, panel_y, entries, n_bins, n_slots, Xh, part, (int)k);
    return (int)hipGetLastError();
  });
}

int launch_panel_combine(const int32_t* panel_y, int64_t n_slots, const float* part, float* Y, int32_t k,
                         void* stream) {
  if (n_slots <= 0) return 0;
  const Shape s = pick_shape(k, 0, true);
  return dispatch_shape(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value;
    const int64_t blocks = ceil_div(n_slots, kBlock / LPR);
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)blocks, (unsigned)s.slices);
    hipLaunchKernelGGL((panel_combine_kernel<VEC, LPR>), grid, dim3(kBlock), 0, (hipStream_t)stream, panel_y,
                       n_slots, part, Y, (int)k);
    return (int)hipGetLastError();
  });
}

int launch_sddmm_panel(const uint32_t* panel_ptr, const int32_t* panel_y, const Entry* entries,
                       const uint32_t* emap, int64_t n_bins, const float* U, const float* Vh,
                       int64_t vh_rows, float* S, int32_t k, void* stream) {
  if (n_bins <= 0) return 0;
  const Shape s = pick_shape(k, 0, true);
  const bool small = small_matrix(vh_rows, k);
  return dispatch_shape(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value, NB = LPR < kSampledBatch ? LPR : kSampledBatch;
    const int64_t blocks = ceil_div(n_bins, kBlock / LPR);
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)blocks);
    if (small)
      hipLaunchKernelGGL((sddmm_panel_kernel<VEC, LPR, NB, true>), grid, dim3(kBlock), 0, (hipStream_t)stream,
                         panel_ptr, panel_y, entries, emap, n_bins, U, Vh, S, (int)k, (int)s.slices);
    else
      hipLaunchKernelGGL((sddmm_panel_kernel<VEC, LPR, NB, false>), grid, dim3(kBlock), 0, (hipStream_t)stream,
                         panel_ptr, panel_y, entries, emap, n_bins, U, Vh, S, (int)k, (int)s.slices);
    return (int)hipGetLastError();
  });
}


namespace {
// (VEC, LPR) with at most 64 columns per slice: the corner kernel keeps 2 x 256 rows of a slice in LDS
template <typename F>
int dispatch_w64(const Shape& s, F&& f) {
#define ARROW_CASE(V, L) \
  if (s.vec == V && s.lpr == L) return f(std::integral_constant<int, V>{}, std::integral_constant<int, L>{});
  ARROW_CASE(4, 1) ARROW_CASE(4, 2) ARROW_CASE(4, 4) ARROW_CASE(4, 8) ARROW_CASE(4, 16)
  ARROW_CASE(2, 1) ARROW_CASE(2, 2) ARROW_CASE(2, 4) ARROW_CASE(2, 8) ARROW_CASE(2, 16) ARROW_CASE(2, 32)
  ARROW_CASE(1, 1) ARROW_CASE(1, 2) ARROW_CASE(1, 4) ARROW_CASE(1, 8) ARROW_CASE(1, 16) ARROW_CASE(1, 32) ARROW_CASE(1, 64)
#undef ARROW_CASE
  return (int)hipErrorInvalidValue;
}
}  // namespace

int launch_corner(const uint32_t* tiles, const uint32_t* items, int64_t n_items, const Entry* entries,
                  const float* Xh, int64_t xh_rows, float* part, int32_t k, void* stream) {
  if (n_items <= 0) return 0;
  (void)xh_rows;
  // 64-column slices: accumulators and tile copy take 64 KiB of LDS each
  const Shape s = pick_shape(k, 64, true);
  return dispatch_w64(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value;
    if (n_items > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)n_items, (unsigned)s.slices);
    hipLaunchKernelGGL((corner_kernel<VEC, LPR, 8>), grid, dim3(kCornerBlock), 0, (hipStream_t)stream, tiles,
                       items, entries, Xh, part, (int)k);
    return (int)hipGetLastError();
  });
}

int launch_corner_combine(const uint32_t* panel_ptr, const int32_t* corner_y, int64_t corner,
                          const float* part, float* Y, int32_t k, void* stream) {
  if (corner <= 0) return 0;
  const Shape s = pick_shape(k, 0, true);
  return dispatch_shape(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value;
    const int64_t blocks = ceil_div(corner, kBlock / LPR);
    if (blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)blocks, (unsigned)s.slices);
    hipLaunchKernelGGL((corner_combine_kernel<VEC, LPR>), grid, dim3(kBlock), 0, (hipStream_t)stream,
                       panel_ptr, corner_y, corner, part, Y, (int)k);
    return (int)hipGetLastError();
  });
}

int launch_sddmm_corner(const uint32_t* tiles, int64_t n_tiles, const int32_t* corner_y, const Entry* entries,
                        const uint32_t* emap, const float* U, const float* Vh, int64_t vh_rows, float* S,
                        int32_t k, void* stream) {
  if (n_tiles <= 0) return 0;
  const Shape s = pick_shape(k, 0, true);
  const bool small = small_matrix(vh_rows, k);
  return dispatch_shape(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value, NB = LPR < kSampledBatch ? LPR : kSampledBatch;
    if (n_tiles > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    dim3 grid((unsigned)n_tiles);
    if (small)
      hipLaunchKernelGGL((sddmm_corner_kernel<VEC, LPR, NB, true>), grid, dim3(kBlock), 0, (hipStream_t)stream,
                         tiles, corner_y, entries, emap, U, Vh, S, (int)k, (int)s.slices);
    else
      hipLaunchKernelGGL((sddmm_corner_kernel<VEC, LPR, NB, false>), grid, dim3(kBlock), 0, (hipStream_t)stream,
                         tiles, corner_y, entries, emap, U, Vh, S, (int)k, (int)s.slices);
    return (int)hipGetLastError();
  });
}

}  // namespace arrow
