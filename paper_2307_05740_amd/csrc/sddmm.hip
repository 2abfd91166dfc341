// HIP kernels for gfx950 of the sampled dense-dense product on the arrow layout:
//     S[src(e)] = a_e * <U[i, :], V[j, :]>       for every stored entry e = (i, j).
// It walks the same work lists as the matrix product (kernels.hip).  A lane owns VEC consecutive columns,
// LPR lanes (a lane group) a row.  Per entry the LPR lanes of a group hold partial dot products of their
// columns; NB entries are reduced together by a transposing butterfly (group_reduce), after which lane l
// of the group holds the dot product of entry l / (LPR / NB) of the batch.  All k columns are covered
// inside the kernels (a loop over column slices of LPR * VEC), so the result needs no second pass.
//
// What bounds it: every entry reads one row of V through the L1, four times the bytes per column pass of
// the matrix product's 64-column slices (a dot product needs the whole row), and writes 4 bytes to a
// place of its own.  The entries' places in S used to be loaded when their dot products were ready, a
// second memory latency after every batch of rows, and the entries of a list one batch at a time; both
// are now on their way while the batch before is worked on (R-MAT 1m, k = 128: chunks 944 -> 868 us, short
// rows and pieces 448 -> 363 us, at 6.4 and 7.1 TB/s of what crosses the L2's boundary; R-MAT 30k, k = 24: 47 ->
// 19 us, 12 since wavefronts share chunks, 10.2 since the pieces of long rows come before the short rows, launch_sddmm).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "arrow_internal.h"
#include "kernel_common.h"

namespace arrow {
namespace {

constexpr int64_t kResidentWaves = 8192;   // wavefronts the chip holds
constexpr int kSampledStage = 1024;   // entries of the group list a workgroup stages at once
// Bytes of U (V has as many) from which on the rows of U that short rows read carry the streaming hint: they then leave
// the caches to the rows of V, and where everything still fits the cache behind the L2s they are better kept there.  R-MAT 100k, k = 96 (37
// MiB) 61.2 us, with the hint 63.6; k = 128 (49 MiB) 74.1 and 75.5; 300k, k = 50 (57 MiB) 162.4 and 155.0; 200k, k = 100 (76 MiB)
// 199.0 and 190.0; 1m, k = 128 1233 and 1227; grid of 350 x 350, k = 96 (45 MiB) 35.2 and 37.2, 500 x 500, k = 100 (95 MiB) 71.5
// and 62.2; dense blocks, 150k, k = 128 (73 MiB) 217.6 and 212.8.  (Not in the launch
// of both lists together: the choice alone costs 30k, k = 24, 0.6 % there.)
constexpr int64_t kSampledOnce = 56 << 20;

struct alignas(16) SampledShared {
  Entry ent[kSampledStage];
  uint32_t at[kSampledStage];                       // the entries' places in S
  uint32_t ptr[kItemsPerGroupBlock + 1];
  uint32_t mid[kItemsPerGroupBlock];
  int32_t row[kItemsPerGroupBlock];
  uint32_t win[kItemsPerGroupBlock];               // window-row list: first position of the row's window
};

// NB entries' rows of V (valid where ok) against the row of U, all k columns.  `get(u)` names the row of
// entry u; rows of entries that are not ok are not read.
template <int VEC, int LPR, int NB, bool SMALL, typename Row, typename Ok>
__device__ __forceinline__ float dots(const SampledArgs& a, const char* base, uint32_t row_bytes, const float* Urow,
                                      typename Vec<VEC>::type u0, int l, const LaneColumns lc0, Row&& row, Ok&& ok) {
  using V = typename Vec<VEC>::type;
  float p[NB];
  {
    V x[NB];
    const uint32_t col_bytes = lc0.ok ? 4u * (uint32_t)lc0.c : 0u;
#pragma unroll
    for (int u = 0; u < NB; ++u)
      x[u] = ok(u) && lc0.ok ? load_row<VEC, SMALL>(base, row(u), row_bytes, col_bytes) : vzero<VEC>();
    if (a.k % VEC != 0) {
#pragma unroll
      for (int u = 0; u < NB; ++u) drop_shared(x[u], lc0.shared);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) p[u] = vdot(u0, x[u]);
  }
  for (int c0 = LPR * VEC; c0 < a.k; c0 += LPR * VEC) {
    const LaneColumns lc = lane_columns<VEC>(l, c0, a.k);
    const uint32_t col_bytes = lc.ok ? 4u * (uint32_t)lc.c : 0u;
    V uu = lc.ok ? gload<VEC>(Urow + lc.c) : vzero<VEC>();
    drop_shared(uu, lc.shared);
    V x[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u)
      x[u] = ok(u) && lc.ok ? load_row<VEC, SMALL>(base, row(u), row_bytes, col_bytes) : vzero<VEC>();
    if (a.k % VEC != 0) {
#pragma unroll
      for (int u = 0; u < NB; ++u) drop_shared(x[u], lc.shared);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) p[u] += vdot(uu, x[u]);
  }
  return group_reduce<NB, LPR>(p, l);
}

// One chunk of the wave list per wavefront: the G lane groups take the entries round-robin, NB rounds at
// a time; nothing is combined across lane groups.  Entries [lo, mid) read rows of the staged head Vh.
template <int VEC, int LPR, int NB, bool SMALL, bool AHEAD>
__device__ __forceinline__ void sampled_chunk(Entry* ents, uint32_t* ats, const SampledArgs& a, int64_t ch, uint32_t part) {
  using V = typename Vec<VEC>::type;
  constexpr uint32_t G = 64 / LPR;
  constexpr uint32_t SPAN = LPR / NB;               // lanes that end up with the same entry's sum
  uint32_t lo = a.chunk_ptr[ch];
  uint32_t hi = a.chunk_ptr[ch + 1];
  uint32_t mid = a.chunk_mid[ch];
  const int32_t row = a.chunk_row[ch];
  if (a.chunk_parts > 1) {                          // this wavefront's share of the chunk
    const uint32_t len = hi - lo, first = lo;
    lo = first + len * part / a.chunk_parts;
    hi = first + len * (part + 1) / a.chunk_parts;
    mid = mid < lo ? lo : (mid > hi ? hi : mid);
  }
  if (lo == hi) return;                             // padding slot of the die queues
  const uint32_t lane = threadIdx.x % 64;
  const uint32_t g = lane / LPR;
  const uint32_t l = lane % LPR;
  const LaneColumns lc0 = lane_columns<VEC>((int)l, 0, a.k);
  const float* Urow = a.U + (size_t)row * (size_t)a.k;
  Entry ahead = a.ent[lo + lane < hi ? lo + lane : lo];
  uint32_t ahead_at = lo + lane < hi ? lo + lane : lo;
  if (a.emap) ahead_at = a.emap[ahead_at];
  V u0 = lc0.ok ? gload<VEC>(Urow + lc0.c) : vzero<VEC>();
  drop_shared(u0, lc0.shared);
  for (int seg = 0; seg < 2; ++seg) {
    const char* base = reinterpret_cast<const char*>(seg == 0 ? a.Vh : a.V);
    const uint32_t row_bytes = 4u * (uint32_t)(seg == 0 ? a.head_stride : a.k);
    const uint32_t s_lo = seg == 0 ? lo : mid;
    const uint32_t s_hi = seg == 0 ? mid : hi;
    for (uint32_t b0 = s_lo; b0 < s_hi; b0 += 64) {
      const uint32_t nb = s_hi - b0 < 64u ? s_hi - b0 : 64u;
      ents[lane] = ahead;
      ats[lane] = ahead_at;
      {
        const uint32_t nx = b0 + nb + lane < hi ? b0 + nb + lane : lo;   // next batch, of this or the next segment
        ahead = a.ent[nx];
        ahead_at = a.emap ? a.emap[nx] : nx;
      }
      strip_sync();
      // A chunk that a wavefront has to itself in a short list is many rounds of rows one after the other: the next
      // round's rows arrive while this one's are multiplied.  (R-MAT 60k, k = 32: 18.4 -> 16.4 us; 100k, 200: 148 -> 132; shared
      // chunks lose, 16k, 64: 8.9 -> 9.3, and the registers cost the long lists and the rows their occupancy.)
      if (AHEAD && a.k <= LPR * VEC) {
        const uint32_t col_bytes = lc0.ok ? 4u * (uint32_t)lc0.c : 0u;
        auto load = [&](V (&x)[NB], uint32_t s) {
#pragma unroll
          for (int u = 0; u < NB; ++u) {
            const uint32_t i = (s + u) * G + g;
            x[u] = i < nb && lc0.ok ? load_row<VEC, SMALL>(base, ents[i % 64].xrow, row_bytes, col_bytes) : vzero<VEC>();
          }
        };
        auto finish = [&](V (&x)[NB], uint32_t s) {
          float p[NB];
          if (a.k % VEC != 0) {
#pragma unroll
            for (int u = 0; u < NB; ++u) drop_shared(x[u], lc0.shared);
          }
#pragma unroll
          for (int u = 0; u < NB; ++u) p[u] = vdot(u0, x[u]);
          const float dot = group_reduce<NB, LPR>(p, (int)l);
          const uint32_t idx = (s + l / SPAN) * G + g;
          if (l % SPAN == 0 && idx < nb) a.S[ats[idx]] = ents[idx].val * dot;
        };
        V x0[NB], x1[NB];
        load(x0, 0);
        for (uint32_t s = 0;; s += 2 * NB) {
          const bool more = (s + NB) * G < nb, more2 = (s + 2 * NB) * G < nb;
          if (more) load(x1, s + NB);
          finish(x0, s);
          if (!more) break;
          if (more2) load(x0, s + 2 * NB);
          finish(x1, s + NB);
          if (!more2) break;
        }
        strip_sync();
        continue;
      }
      for (uint32_t s = 0; s * G < nb; s += NB) {   // round s + u: lane group g handles entry (s + u) * G + g
        float dot;
        if ((s + NB) * G <= nb)
          dot = dots<VEC, LPR, NB, SMALL>(a, base, row_bytes, Urow, u0, (int)l, lc0,
                                          [&](int u) { return ents[(s + u) * G + g].xrow; }, [](int) { return true; });
        else
          dot = dots<VEC, LPR, NB, SMALL>(a, base, row_bytes, Urow, u0, (int)l, lc0,
                                          [&](int u) { return ents[((s + u) * G + g) % 64].xrow; },
                                          [&](int u) { return (s + u) * G + g < nb; });
        const uint32_t idx = (s + l / SPAN) * G + g;
        if (l % SPAN == 0 && idx < nb) a.S[ats[idx]] = ents[idx].val * dot;
      }
      strip_sync();
    }
  }
}

// Which items the id-th workgroup of the rows has: pieces first.  (In 32 bits, n is below 2^31; with 64 grids of 500 K vertices took 1 % longer.)
struct ItemRange { uint32_t first; int n; };
__device__ __forceinline__ ItemRange items_at(const SampledArgs& a, uint32_t id) {
  const bool piece = id < a.piece_blocks;
  const uint32_t items = (uint32_t)(piece ? a.piece_items : a.items), end = (uint32_t)(piece ? a.n_pieces : a.n_rows);
  const uint32_t first = id * items + (piece ? 0u : a.short_base);
  return {first, first < end ? (int)(end - first < items ? end - first : items) : 0};
}

// Items [first, first + n_it) of the group list (WINDOW false: entries before `mid` read the staged head
// Vh, the rest rows of V) or of the window-row list (WINDOW true: entries before `mid` name rows of V, the
// rest positions inside the row's tile window, translated through perm).  The workgroup copies the items'
// descriptors into LDS and then, as many items at a time as fit, their entries and places in S (part of
// an item where it is longer than that).  As many lane groups as there are to spare share an item.
// (With entries that do not fit read from memory one batch after the other instead: the 55-entry rows of
// dense diagonal blocks, 2.9 M rows, k = 16, 3510 us; 2180 us with a strip of 16 entries per lane group.)
template <int VEC, int LPR, int NB, bool SMALL, bool WINDOW, bool ONCE>
__device__ __forceinline__ void sampled_rows(SampledShared& sh, const SampledArgs& a, int64_t first, int n_it) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  constexpr uint32_t SPAN = LPR / NB;
  constexpr uint32_t Q = kSampledStage / kBlock;
  constexpr int WPB = kBlock / 64;
  const int tid = threadIdx.x;
  const uint32_t lane = tid % 64, wave = tid / 64;
  const uint32_t l = tid % LPR;
  const LaneColumns lc0 = lane_columns<VEC>((int)l, 0, a.k);
  uint32_t ptr = 0, mids = 0, wins = 0;
  int32_t rows = 0;
  if (tid <= n_it) ptr = a.rows_ptr[first + tid];
  if (tid < n_it) { mids = a.rows_mid[first + tid]; rows = a.rows_row[first + tid]; }
  if (WINDOW && tid < n_it) wins = a.rows_win[first + tid];
  auto describe = [&] {
    if (tid <= n_it) sh.ptr[tid] = ptr;
    if (tid < n_it) { sh.mid[tid] = mids; sh.row[tid] = rows; }
    if (WINDOW && tid < n_it) sh.win[tid] = wins;
  };
  // Where all entries fit, as nearly everywhere, they are loaded beside the descriptors, not behind a barrier: grid of 622 x 622, k = 16,
  // 23.2 -> 21.9 us; R-MAT 60k, 50, 24.6 -> 23.2; 163k, 64, 54.1 -> 53.0.  (With 64-bit offsets it would cost a wavefront per SIMD.)
  const uint32_t begin = a.rows_ptr[first], end = a.rows_ptr[first + n_it];
  const bool together = SMALL && !WINDOW && end - begin <= (uint32_t)kSampledStage;
  if (!together) {
    describe();
    __syncthreads();
  }
  int i0 = 0;
  for (uint32_t b0 = begin; b0 < end;) {
    // entries [b0, b1) of items [i0, i1)
    static_assert(kItemsPerGroupBlock <= 64, "one lane per item");
    int fit = n_it, i1 = n_it;
    uint32_t b1 = end;
    if (!together) {
      const int i = i0 + 1 + (int)lane;
      fit = __popcll(__ballot(i <= n_it && sh.ptr[i <= n_it ? i : n_it] - b0 <= (uint32_t)kSampledStage));
      i1 = i0 + (fit > 0 ? fit : 1);
      b1 = fit > 0 ? sh.ptr[i1] : b0 + (uint32_t)kSampledStage;
    }
    Entry e[Q];
    uint32_t at[Q];
    if (WINDOW) {                                   // a wavefront per item, which knows its window
      for (int j0 = i0 + (int)wave; j0 < i1; j0 += WPB * Q) {
        uint32_t from[Q], to[Q], win[Q], longest = 0;
#pragma unroll
        for (uint32_t q = 0; q < Q; ++q) {
          const int it = j0 + (int)q * WPB;
          from[q] = to[q] = win[q] = 0;
          if (it < i1) {
            from[q] = sh.ptr[it] > b0 ? sh.ptr[it] : b0;
            to[q] = sh.ptr[it + 1] < b1 ? sh.ptr[it + 1] : b1;
            win[q] = sh.win[it];
          }
          if (to[q] - from[q] > longest) longest = to[q] - from[q];
        }
        for (uint32_t t0 = lane; t0 < longest + lane; t0 += 64) {
#pragma unroll
          for (uint32_t q = 0; q < Q; ++q) {
            const uint32_t t = from[q] + t0;
            if (t < to[q]) { e[q] = stream_load(&a.ent[t]); at[q] = a.emap ? stream_load(&a.emap[t]) : t; }
          }
#pragma unroll
          for (uint32_t q = 0; q < Q; ++q)
            if (from[q] + t0 < to[q] && from[q] + t0 >= sh.mid[j0 + (int)q * WPB]) e[q].xrow = a.perm[win[q] + (uint32_t)e[q].xrow];
#pragma unroll
          for (uint32_t q = 0; q < Q; ++q) {
            const uint32_t t = from[q] + t0;
            if (t < to[q]) { sh.ent[t - b0] = e[q]; sh.at[t - b0] = at[q]; }
          }
        }
      }
    } else {
#pragma unroll
      for (uint32_t q = 0; q < Q; ++q) {
        const uint32_t t = b0 + tid + q * kBlock;
        if (t < b1) { e[q] = a.ent[t]; at[q] = a.emap ? a.emap[t] : t; }
      }
#pragma unroll
      for (uint32_t q = 0; q < Q; ++q) {
        const uint32_t t = b0 + tid + q * kBlock;
        if (t < b1) { sh.ent[t - b0] = e[q]; sh.at[t - b0] = at[q]; }
      }
    }
    if (together) describe();
    __syncthreads();
    int share = 1;                                  // lane groups per item
    while (share * 2 * (i1 - i0) <= GPB) share *= 2;
    for (int it = i0 + tid / LPR / share; it < i1; it += GPB / share) {
      const int32_t row = sh.row[it];
      if (row < 0) continue;                        // padding slot of the die queues
      const uint32_t lo = sh.ptr[it] > b0 ? sh.ptr[it] : b0, hi = sh.ptr[it + 1] < b1 ? sh.ptr[it + 1] : b1;
      const uint32_t mid = sh.mid[it] < lo ? lo : (sh.mid[it] > hi ? hi : sh.mid[it]);
      const uint32_t skip = (uint32_t)(tid / LPR % share) * NB;
      const float* Urow = a.U + (size_t)row * (size_t)a.k;
      V u0 = vzero<VEC>();
      if (lc0.ok) u0 = ONCE ? vload_stream<VEC>(Urow + lc0.c) : gload<VEC>(Urow + lc0.c);
      drop_shared(u0, lc0.shared);
      for (int seg = WINDOW ? 1 : 0; seg < 2; ++seg) {
        const char* base = reinterpret_cast<const char*>(seg == 0 ? a.Vh : a.V);
        const uint32_t row_bytes = 4u * (uint32_t)(seg == 0 ? a.head_stride : a.k);
        const uint32_t j_lo = WINDOW || seg == 0 ? lo : mid, j_hi = seg == 0 ? mid : hi;
        for (uint32_t j = j_lo + skip; j < j_hi; j += NB * (uint32_t)share) {
          const float dot = dots<VEC, LPR, NB, SMALL>(
              a, base, row_bytes, Urow, u0, (int)l, lc0, [&](int u) { return sh.ent[(j + u < j_hi ? j + u : j) - b0].xrow; },
              [&](int u) { return j + u < j_hi; });
          const uint32_t mine = j + l / SPAN;
          if (l % SPAN == 0 && mine < j_hi) a.S[sh.at[mine - b0]] = sh.ent[mine - b0].val * dot;
        }
      }
    }
    b0 = b1;
    i0 += fit;
    if (b0 < end) __syncthreads();
  }
}

template <int VEC, int LPR, int NB, bool SMALL>
__global__ __launch_bounds__(kBlock) void sddmm_chunks_kernel(const SampledArgs a) {
  constexpr int WPB = kBlock / 64;
  __shared__ Entry ents[WPB][64];
  __shared__ uint32_t ats[WPB][64];
  // runs of workgroups to one die each, as in the product's chunks kernel
  const uint32_t id = in_runs(blockIdx.x, kDiesLog, a.run, gridDim.x);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int64_t ch = (int64_t)id * WPB + wave;      // (a list in window order is never short)
  if (ch < a.n_chunks) sampled_chunk<VEC, LPR, NB, SMALL, false>(ents[wave], ats[wave], a, ch, 0);
}

template <int VEC, int LPR, int NB, bool SMALL, bool WINDOW, bool ONCE>
__global__ __launch_bounds__(kBlock) void sddmm_rows_kernel(const SampledArgs a) {
  __shared__ SampledShared sh;
  const ItemRange it = items_at(a, blockIdx.x);
  if (it.n > 0) sampled_rows<VEC, LPR, NB, SMALL, WINDOW, ONCE>(sh, a, it.first, it.n);
}

// Both lists in one launch (short lists: the second launch would be most of the time).  AHEAD: see sampled_chunk.
template <int VEC, int LPR, int NB, bool SMALL, bool AHEAD>
__global__ __launch_bounds__(kBlock) void sddmm_kernel(const SampledArgs a) {
  constexpr int WPB = kBlock / 64;
  union Shared {
    SampledShared rows;
    struct { Entry ents[WPB][64]; uint32_t ats[WPB][64]; } chunk;
    __device__ Shared() {}
  };
  __shared__ Shared sh;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  if (blockIdx.x < a.chunk_blocks) {
    const uint32_t slot = blockIdx.x * WPB + wave;  // fewer than 2^31, the launch sees to that
    const int64_t ch = slot / a.chunk_parts;
    if (ch < a.n_chunks)
      sampled_chunk<VEC, LPR, NB, SMALL, AHEAD>(sh.chunk.ents[wave], sh.chunk.ats[wave], a, ch, slot % a.chunk_parts);
    return;
  }
  const ItemRange it = items_at(a, blockIdx.x - a.chunk_blocks);
  if (it.n > 0) sampled_rows<VEC, LPR, NB, SMALL, false, false>(sh.rows, a, it.first, it.n);
}

}  // namespace

namespace {

// Items of the group list (or window rows) per workgroup.  Few of them leave several lane groups for each, so that all
// of its rounds of row loads are on their way at once, and balance rows of unequal length; many of them pay once for what
// a workgroup does before its first row arrives.  Measured with 2 to 64 of them on 2605 lists (grids, R-MAT, Chung-Lu, dense blocks of 26 to 62
// entries a row; 1.5 K to 450 K vertices, k = 8 to 256): what follows is within 1 % of the best on average, 2 % for the widest equal rows.  (By the square
// root of the list's length single lists lost up to 16 %: Chung-Lu 50 K, k = 48, 23.0 us, now 19.8; dense blocks 14 K, 48, 20.4 / 18.1; grid 120 K, 64, 27.3 / 24.7.)
//
// Short rows behind pieces of long ones, which are several times as long: the two have workgroups of their own, by the number of each from which on 4, 8, 16, 32 and
// 64 short rows and 2, 4, 8 and 16 pieces are the best, by lanes per row.  (One number for both, by the root of rows times entries, let the first workgroups,
// which are all pieces, end the launch, or gave short rows more workgroups than the chip holds beside the chunks: R-MAT 30 K, k = 24, started them after 3 to 6 of 11 us.
// 441 lists of 3 K to 1.5 M vertices, R-MAT and Chung-Lu, at five ranks each, rows without entries left out: 0.96 times the time on average, within 1 % of the
// best numbers.  us before / now: R-MAT 30 K, k = 24, 10.9 / 9.5; 6 K, 96, 6.1 / 5.5; 14 K, 43, 8.8 / 8.0; 70 K, 66, 45.8 / 44.0; 1.5 M, 20, 364.5 / 356.3; Chung-Lu 25 K, 37,
// 12.4 / 10.8; 67 K, 32, 17.7 / 16.9.)  Wider lists of more than 131072 vertices gain less than they scatter (Chung-Lu 540 K, k = 64, 175.8 us, apart 178.2) and
// lists of more pieces than short rows lose (dense blocks, 12 K vertices of 44 entries, k = 128, 23.9 us, apart 27.3; 17 K, 43, 65, 24.9 and 28.1): one number for both,
// by the root of rows times entries.  Its lines were measured with rows without entries in the list, which are left out since: the root is smaller, and lists
// near a line get half as many items.  Those are the better: of 52 lists, R-MAT and Chung-Lu of 140 K to 1.5 M vertices at 40 to 200 columns, 16 take 2 to 8 % longer with
// the number that all rows gave and the others the same within a percent (k = 64, all rows / those with entries, us: R-MAT 300 K of 8 edges a vertex 109.4 / 105.4; 600 K 219.2 / 206.8; 650 K of 6
// 188.9 / 177.2; directed 300 K of 12, 88.6 / 82.6, k = 128 167.7 / 155.3; 700 K, 128, 375.6 / 366.0).
// Rows of dense blocks, of which a lane group takes one or two, by rows: 450 K, 26 entries, k = 48,  8: 244.3  16: 221.5  32: 254.4;
// 250 K, 40 entries, k = 128,  4: 298.9  8: 293.6  16: 365.1; 27 K, 42 entries, k = 8,  4: 18.5  8: 14.4  16: 12.2  32: 16.4.
// (Lines as close as 10 % are one: short rows at four and eight lanes go from 4 items to 16, with 8 between 1700 and 1900 rows nothing was faster by more than runs differ.  Pieces at two
// lanes gain from theirs: 2 / 4 of 4679, Chung-Lu 36 K, k = 8, 10.7 / 10.0 us, 16 / 8 of 5742, 45 K, 11.5 / 11.1, though 5183, R-MAT 60 K, 12.4 / 12.7.)
struct ItemsFrom { int lpr; double from[5]; };      // ... items at least from[0], from[1], ... rows
constexpr double kNever = 1e18;
constexpr ItemsFrom kUnequalItems[] = {{2, {0, 5800, 21400, 226000, 909000}},       {4, {0, 12100, 31400, 186000, 909000}},
                                       {8, {0, 7900, 50000, 253000, 962000}},       {16, {8700, 25900, 90700, 498000, 1090000}},
                                       {32, {13500, 44800, 156000, 498000, 1090000}}, {64, {21400, 90700, 226000, 720000, kNever}}};
constexpr ItemsFrom kShortItems[] = {{2, {0, 1700, 5500, 17500, 49500}},            {4, {0, 1800, 1800, 10800, 70000}},
                                     {8, {0, 1800, 1800, 17800, 60000}},            {16, {0, 2000, 10400, 40800, 145000}},
                                     {32, {0, 5600, 15500, 90000, 690000}},         {64, {0, 20000, 46000, 263000, kNever}}};
constexpr ItemsFrom kPieceItems[] = {{2, {0, 3900, 4800, 6000, kNever}},            {4, {0, 900, 1450, 3400, kNever}},
                                     {8, {0, 300, 1100, 4000, kNever}},             {16, {0, 950, 2500, 11000, kNever}},
                                     {32, {0, 1200, 3600, 8600, kNever}},           {64, {0, 2400, 20000, kNever, kNever}}};
constexpr ItemsFrom kWindowItems[] = {{4, {0, 4000, 16000, kNever, kNever}},        {8, {2500, 8000, 16000, kNever, kNever}},
                                      {16, {2500, 8000, kNever, kNever, kNever}},   {32, {4000, 8000, kNever, kNever, kNever}},
                                      {64, {4000, kNever, kNever, kNever, kNever}}};

int items_from(const ItemsFrom* row, int least, int lpr, double n) {
  while (row->lpr < lpr) ++row;
  int items = least / 2;
  for (double from : row->from)
    if (n >= from) items *= 2;
  return items;
}

// Of a list of n rows with nnz entries: rows of dense blocks, long and short rows, pieces of long rows, short rows behind those, or rows that are all alike.  chunks: behind some of those.
enum class Rows { kWindow, kUnequal, kPieces, kShort, kAlike };
int items_of(int64_t n, int64_t nnz, int lpr, Rows rows, bool chunks) {
  const double average = (double)nnz / (double)std::max<int64_t>(1, n);
  int items;
  if (rows != Rows::kAlike) {
    items = rows == Rows::kPieces    ? items_from(kPieceItems, 2, lpr, (double)n)
            : rows == Rows::kUnequal ? items_from(kUnequalItems, 4, lpr, std::sqrt((double)n * (double)nnz))
                                     : items_from(rows == Rows::kWindow ? kWindowItems : kShortItems, 4, lpr, (double)n);
    // (What dense blocks leave beside their tiles are rows of 30 to 48 entries.  Behind chunks they end the launch, and two of the widest are better for longer: k = 256,
    // us, 2 / 4 items, 12 K vertices of 50 entries 43.6 / 46.4, 14 K 52.1 / 55.3, 20 K 66.8 / 69.9, 24 K (root 39 K) 78.3 / 82.2; k = 150, 14 K, 44.4 / 45.2, 12 K 37.4 /
    // 36.8; but without chunks k = 150, 14 K of 46 entries 42.2 / 40.3, 17 K of 36 40.8 / 38.9.)
    if ((rows == Rows::kWindow || rows == Rows::kUnequal) && chunks && lpr == 64 && average >= 32.0 && items == 4 && std::sqrt((double)n * (double)nnz) < 45000.0) items = 2;
    if (rows == Rows::kWindow && lpr == 16 && average < 35.0 && n >= 15000) items = 16;
    // (Eight long rows of 32 lanes to a workgroup are one to one and a half rounds of the 1536 workgroups that the chip holds of them: the second round is
    // mostly empty.  k = 128, us, 4 / 8 items: 54 entries, 9.4 K rows 31.9 / 30.2, 14.0 K 41.0 / 42.9, 16.5 K 49.4 / 53.8; 62, 19.0 K 58.5 / 64.0; 46, 15.1 K
    // 39.6 / 42.0, 23.4 K 38.2 / 37.3; 36, 19.4 K 31.0 / 31.4; 26, 21.4 K 29.2 / 27.8.)
    if (rows == Rows::kWindow && lpr == 32 && average >= 40.0 && n > 8 * 1536 && n <= 8 * 1536 * 8 / 5) items = 4;
  } else {
    // All about alike: as few as give one round of the workgroups that the chip holds, 256 entries at first (32 of a grid's rows) and 64 items at most, 32
    // of the widest rows.  A second round that is nearly empty costs most: grid 30 K, k = 128, 16 items (1871 workgroups) 15.1 us, 32 12.9; 120 K, k = 64, 64 items (1871)
    // 27.3, 32 24.7, but 90 K, 64 (1407) 17.6, 32 18.2; 200 K, 64 (3123) 33.7, 32 35.1; 60 K, k = 150, 32 (1861) 35.2, 16 31.0.  (74.5 K: k = 48 12.5 with 64, 13.7 with
    // 32, k = 64 15.9 and 14.9.)
    constexpr int64_t kRound = 1792;                // 256 compute units, seven wavefronts a SIMD
    const int most = lpr == 64 ? kItemsPerGroupBlock / 2 : kItemsPerGroupBlock;
    items = lpr <= 4 || (lpr == 8 && n >= 14000) ? 32 : lpr == 8 || (lpr == 16 && n >= 7400) ? 16 : lpr == 64 || (lpr == 32 && n < 3000) ? 4 : 8;
    while (items > 2 && items * average > 256.0) items /= 2;
    while (items < most && n > kRound * items) items *= 2;
    if (items == most && lpr >= 8 && n > kRound * items && n <= kRound * items * 7 / 5) items /= 2;
  }
  while (items < kItemsPerGroupBlock && n > (kMostGroups - kDies) * items) items *= 2;   // (what a grid holds)
  return items;
}

}  // namespace

int launch_sddmm(SampledArgs a, bool window_rows, bool die_queues, bool windows, bool unequal, int64_t v_rows, void* stream) {
  const Shape s = pick_shape(a.k, 0);
  const bool small = small_matrix(v_rows, a.k);
  const hipStream_t st = (hipStream_t)stream;
  if (window_rows || die_queues || (windows && s.lpr >= 16) || 2 * a.n_pieces > a.n_rows) a.n_pieces = 0;
  // Few chunks leave wavefront slots empty, and a chunk of 256 entries is four to 64 rounds of row loads one
  // after the other: wavefronts share it as far as that leaves each a few rounds (nothing has to be
  // combined).  R-MAT 7419, k = 73: 30.7 -> 10.5 us; 12527, k = 128: 33.2 -> 13.7; 51952, k = 128: 50.2 ->
  // 28.4; 30011, k = 24: 16.5 -> 12.0.  Up to twice as many wavefronts as the chip holds where each is left three and a half rounds
  // (1 / 2 / 4 wavefronts, us: R-MAT 60k, k = 64 / 100 / 200: 29.3 / 25.4 / 28.6, 55.5 / 38.8 / 42.7, 113 / 69 / 75; 30k, 128: - /
  // 24.4 / 19.8, but 64: - / 13.7 / 14.4; Chung-Lu 80k, 50: 35.1 / 30.0 / 32.2; 130k, 64: 61.2 / 65.5).
  // Beyond 1.3 times what it holds six rounds, where short rows of much the same weight are in the launch to fill the slots (as they were / shared
  // further, Chung-Lu 60k, k = 96: 31.5 / 35.2; 20k, 200: 28.0 / 30.1; but 75k, 150, 8.5 rounds: 57.5 / 55.2; R-MAT 30k, 150, few short rows: 47.3 / 31.0).
  // Four wavefronts where a row takes eight lanes: R-MAT 30k, k = 24, 3369 chunks, 10.2 -> 11.8, 20k 6.9 -> 7.4; they would gain where there are fewer than some
  // 1000 chunks (9k 6.7 -> 5.3); two with the next round on its way 10.2.
  // Chunks that are one strip each (rows of 49 to 64 entries, as dense blocks leave them) are alike and leave nothing to even out: a list of them that
  // fills half of the chip is not shared, and its widest rows run without the next round on its way (shared / not / nor ahead; 58 or 62 entries a row:
  // 14k, k = 200, 52.9 / 49.5 / 48.4, 20k, 150, 61.6 / 59.4 / 56.1, 20k, 256, 82.4 / 80.1 / 74.4 us, 14k, 40, not shared before either, 17.4 / 16.8, but 28k, 64, 36.5 / 37.2).
  const bool single = a.nnz_chunks <= 64 * a.n_chunks;
  a.chunk_parts = 1;
  const uint32_t most = s.lpr < 4 ? 1u : (s.lpr < 8 ? 2u : (uint32_t)s.lpr / 4);
  const int64_t round = 64 / s.lpr * kSampledBatch;  // entries
  const bool filled = a.nnz_rows * 5 >= a.nnz_chunks * 3;
  if (!window_rows && !windows && !die_queues)
    while (a.chunk_parts < most) {
      const int64_t waves = a.n_chunks * a.chunk_parts * 2;
      const bool few = waves <= kResidentWaves || (!single && waves <= 2 * kResidentWaves && 2 * a.nnz_chunks >= 7 * round * waves &&
                                                   (!filled || 10 * waves <= 13 * kResidentWaves || a.nnz_chunks >= 6 * round * waves));
      if (!few) break;
      a.chunk_parts *= 2;
    }
  const int64_t chunk_blocks = ceil_div(ceil_div(a.n_chunks * a.chunk_parts, kBlock / 64), kDies) * kDies;
  int64_t piece_blocks, row_blocks;
  auto divide = [&] {
    const Rows rows = window_rows ? Rows::kWindow : a.n_pieces > 0 ? Rows::kShort : unequal ? Rows::kUnequal : Rows::kAlike;
    const int64_t n_short = a.n_rows - a.n_pieces;
    a.piece_items = items_of(a.n_pieces, a.nnz_rows, s.lpr, Rows::kPieces, a.n_chunks > 0);
    a.items = die_queues ? (window_rows ? kItemsPerGroupBlock / 4 : kItemsPerGroupBlock) : items_of(n_short, a.nnz_rows, s.lpr, rows, a.n_chunks > 0);
    piece_blocks = ceil_div(ceil_div(a.n_pieces, a.piece_items), kDies) * kDies;
    row_blocks = piece_blocks + ceil_div(ceil_div(n_short, a.items), kDies) * kDies;
  };
  divide();
  if (a.n_pieces > 0 && row_blocks + (windows ? 0 : chunk_blocks) > kMostGroups) {   // (more than a grid holds, with workgroups for both it may)
    a.n_pieces = 0;
    divide();
  }
  a.piece_blocks = (uint32_t)piece_blocks;
  a.short_base = (uint32_t)a.n_pieces - a.piece_blocks * (uint32_t)a.items;
  if (chunk_blocks + row_blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
  a.run = windows && !die_queues ? die_run(chunk_blocks) : 0;
  const bool once = v_rows * a.k * (int64_t)sizeof(float) >= kSampledOnce;
  return dispatch_shape(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value;
    constexpr int NB = LPR < kSampledBatch ? LPR : kSampledBatch;
#define ARROW_LAUNCH(KERNEL, BLOCKS, ...)                                                                           \
  if (small) hipLaunchKernelGGL((KERNEL<VEC, LPR, NB, true __VA_ARGS__>), dim3((unsigned)(BLOCKS)), dim3(kBlock), 0, st, a); \
  else hipLaunchKernelGGL((KERNEL<VEC, LPR, NB, false __VA_ARGS__>), dim3((unsigned)(BLOCKS)), dim3(kBlock), 0, st, a)
#define ARROW_COMMA ,
    if (window_rows) {
      if (row_blocks > 0 && once) { ARROW_LAUNCH(sddmm_rows_kernel, row_blocks, ARROW_COMMA true ARROW_COMMA true); }
      else if (row_blocks > 0) { ARROW_LAUNCH(sddmm_rows_kernel, row_blocks, ARROW_COMMA true ARROW_COMMA false); }
    } else if (!windows && chunk_blocks > 0) {
      a.chunk_blocks = (uint32_t)chunk_blocks;
      if (a.chunk_parts == 1 && !(single && s.lpr >= 32)) { ARROW_LAUNCH(sddmm_kernel, chunk_blocks + row_blocks, ARROW_COMMA true); }
      else { ARROW_LAUNCH(sddmm_kernel, chunk_blocks + row_blocks, ARROW_COMMA false); }
    } else {
      if (chunk_blocks > 0) { ARROW_LAUNCH(sddmm_chunks_kernel, chunk_blocks, ); }
      if (row_blocks > 0 && once) { ARROW_LAUNCH(sddmm_rows_kernel, row_blocks, ARROW_COMMA false ARROW_COMMA true); }
      else if (row_blocks > 0) { ARROW_LAUNCH(sddmm_rows_kernel, row_blocks, ARROW_COMMA false ARROW_COMMA false); }
    }
#undef ARROW_COMMA
#undef ARROW_LAUNCH
    return (int)hipGetLastError();
  });
}

}  // namespace arrow
