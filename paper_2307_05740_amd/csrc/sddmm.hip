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
// are now on their way while the batch before is worked on (R-MAT 1m, k = 128: chunks 944 -> 867 us, short
// rows and pieces 448 -> 416 us, both then at 6.7 TB/s of rows that miss the L2; R-MAT 30k, k = 24: 47 -> 19 us).
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "arrow_internal.h"
#include "kernel_common.h"

namespace arrow {
namespace {

constexpr int kSampledStage = 1024;   // entries of the group list a workgroup stages at once

struct alignas(16) SampledShared {
  Entry ent[kSampledStage];
  uint32_t at[kSampledStage];                       // the entries' places in S
  uint32_t ptr[kItemsPerGroupBlock + 1];
  uint32_t mid[kItemsPerGroupBlock];
  int32_t row[kItemsPerGroupBlock];
};

// NB entries' rows of V (valid where ok) against the row of U, all k columns.  `get(u)` names the row of
// entry u; rows of entries that are not ok are not read.
template <int VEC, int LPR, int NB, bool SMALL, typename Row, typename Ok>
__device__ __forceinline__ float dots(const SampledArgs& a, const char* base, const float* Urow,
                                      typename Vec<VEC>::type u0, int l, const LaneColumns lc0, Row&& row, Ok&& ok) {
  using V = typename Vec<VEC>::type;
  const uint32_t row_bytes = 4u * (uint32_t)a.k;
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
template <int VEC, int LPR, int NB, bool SMALL>
__device__ __forceinline__ void sampled_chunk(Entry* ents, uint32_t* ats, const SampledArgs& a, int64_t ch) {
  using V = typename Vec<VEC>::type;
  constexpr uint32_t G = 64 / LPR;
  constexpr uint32_t SPAN = LPR / NB;               // lanes that end up with the same entry's sum
  const uint32_t lo = a.chunk_ptr[ch];
  const uint32_t hi = a.chunk_ptr[ch + 1];
  const uint32_t mid = a.chunk_mid[ch];
  const int32_t row = a.chunk_row[ch];
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
      for (uint32_t s = 0; s * G < nb; s += NB) {   // round s + u: lane group g handles entry (s + u) * G + g
        float dot;
        if ((s + NB) * G <= nb)
          dot = dots<VEC, LPR, NB, SMALL>(a, base, Urow, u0, (int)l, lc0,
                                          [&](int u) { return ents[(s + u) * G + g].xrow; }, [](int) { return true; });
        else
          dot = dots<VEC, LPR, NB, SMALL>(a, base, Urow, u0, (int)l, lc0,
                                          [&](int u) { return ents[((s + u) * G + g) % 64].xrow; },
                                          [&](int u) { return (s + u) * G + g < nb; });
        const uint32_t idx = (s + l / SPAN) * G + g;
        if (l % SPAN == 0 && idx < nb) a.S[ats[idx]] = ents[idx].val * dot;
      }
      strip_sync();
    }
  }
}

// Items [first, first + n_it) of the group list (WINDOW false: entries before `mid` read the staged head
// Vh, the rest rows of V) or of the window-row list (WINDOW true: entries before `mid` name rows of V, the
// rest positions inside the row's tile window, translated through perm), one lane group per item.  The
// workgroup copies the items' descriptors and, when they fit, entries and places in S into LDS first;
// entries that do not fit are read from memory.
template <int VEC, int LPR, int NB, bool SMALL, bool WINDOW>
__device__ __forceinline__ void sampled_rows(SampledShared& sh, const SampledArgs& a, int64_t first, int n_it) {
  using V = typename Vec<VEC>::type;
  constexpr int GPB = kBlock / LPR;
  constexpr uint32_t SPAN = LPR / NB;
  const int tid = threadIdx.x;
  const uint32_t l = tid % LPR;
  const LaneColumns lc0 = lane_columns<VEC>((int)l, 0, a.k);
  if (tid <= n_it) sh.ptr[tid] = a.rows_ptr[first + tid];
  if (tid < n_it) { sh.mid[tid] = a.rows_mid[first + tid]; sh.row[tid] = a.rows_row[first + tid]; }
  __syncthreads();
  const uint32_t e0 = sh.ptr[0];
  const uint32_t total = sh.ptr[n_it] - e0;
  const bool staged = total <= (uint32_t)kSampledStage;
  if (staged) {
    constexpr uint32_t Q = kSampledStage / kBlock;
    Entry e[Q];
    uint32_t at[Q];
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) {
      const uint32_t t = tid + q * kBlock;
      if (t < total) { e[q] = a.ent[e0 + t]; at[q] = a.emap ? a.emap[e0 + t] : e0 + t; }
    }
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) {
      const uint32_t t = tid + q * kBlock;
      if (t < total) { sh.ent[t] = e[q]; sh.at[t] = at[q]; }
    }
    __syncthreads();
    if (WINDOW) {                                   // window positions -> rows of V, all items before the first is used
      for (int it = tid / LPR; it < n_it; it += GPB) {
        const uint32_t win = a.rows_win[first + it];
        for (uint32_t t = sh.mid[it] - e0 + l; t < sh.ptr[it + 1] - e0; t += LPR)
          sh.ent[t].xrow = a.perm[win + (uint32_t)sh.ent[t].xrow];
      }
      strip_sync();
    }
  }
  auto run = [&](auto entry, auto place) {
    for (int it = tid / LPR; it < n_it; it += GPB) {
      const int32_t row = sh.row[it];
      if (row < 0) continue;                        // padding slot of the die queues
      const uint32_t lo = sh.ptr[it], mid = sh.mid[it], hi = sh.ptr[it + 1];
      const uint32_t win = WINDOW && !staged ? a.rows_win[first + it] : 0u;
      const float* Urow = a.U + (size_t)row * (size_t)a.k;
      V u0 = lc0.ok ? gload<VEC>(Urow + lc0.c) : vzero<VEC>();
      drop_shared(u0, lc0.shared);
      for (int seg = 0; seg < 2; ++seg) {
        const char* base = reinterpret_cast<const char*>(seg == 0 && !WINDOW ? a.Vh : a.V);
        const uint32_t j_hi = seg == 0 ? mid : hi;
        for (uint32_t j = seg == 0 ? lo : mid; j < j_hi; j += NB) {
          const float dot = dots<VEC, LPR, NB, SMALL>(
              a, base, Urow, u0, (int)l, lc0,
              [&](int u) {
                const int32_t x = entry(j + u < j_hi ? j + u : j).xrow;
                return WINDOW && !staged && seg == 1 ? a.perm[win + (uint32_t)x] : x;
              },
              [&](int u) { return j + u < j_hi; });
          const uint32_t mine = j + l / SPAN;
          if (l % SPAN == 0 && mine < j_hi) a.S[place(mine)] = entry(mine).val * dot;
        }
      }
    }
  };
  if (staged) run([&](uint32_t t) { return sh.ent[t - e0]; }, [&](uint32_t t) { return sh.at[t - e0]; });
  else run([&](uint32_t t) { return a.ent[t]; }, [&](uint32_t t) { return a.emap ? a.emap[t] : t; });
}

template <int VEC, int LPR, int NB, bool SMALL>
__global__ __launch_bounds__(kBlock) void sddmm_chunks_kernel(const SampledArgs a) {
  constexpr int WPB = kBlock / 64;
  __shared__ Entry ents[WPB][64];
  __shared__ uint32_t ats[WPB][64];
  // runs of kDieRun workgroups to one die each, as in the product's chunks kernel
  uint32_t id = blockIdx.x;
  const uint32_t span = kDies * kDieRun;
  const uint32_t base = id / span * span;
  if (a.runs && base + span <= gridDim.x) id = base + id % kDies * kDieRun + (id - base) / kDies;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int64_t ch = (int64_t)id * WPB + wave;
  if (ch < a.n_chunks) sampled_chunk<VEC, LPR, NB, SMALL>(ents[wave], ats[wave], a, ch);
}

template <int VEC, int LPR, int NB, bool SMALL, bool WINDOW>
__global__ __launch_bounds__(kBlock) void sddmm_rows_kernel(const SampledArgs a) {
  __shared__ SampledShared sh;
  const int64_t first = (int64_t)blockIdx.x * a.items;
  const int n_it = a.n_rows - first < a.items ? (int)(a.n_rows - first) : a.items;
  if (n_it > 0) sampled_rows<VEC, LPR, NB, SMALL, WINDOW>(sh, a, first, n_it);
}

// Both lists in one launch (short lists: the second launch would be most of the time).
template <int VEC, int LPR, int NB, bool SMALL>
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
    const int64_t ch = (int64_t)blockIdx.x * WPB + wave;
    if (ch < a.n_chunks) sampled_chunk<VEC, LPR, NB, SMALL>(sh.chunk.ents[wave], sh.chunk.ats[wave], a, ch);
    return;
  }
  const int64_t first = (int64_t)(blockIdx.x - a.chunk_blocks) * a.items;
  const int n_it = a.n_rows - first < a.items ? (int)(a.n_rows - first) : a.items;
  if (n_it > 0) sampled_rows<VEC, LPR, NB, SMALL, false>(sh.rows, a, first, n_it);
}

}  // namespace

int launch_sddmm(SampledArgs a, bool window_rows, bool die_queues, bool windows, int64_t v_rows, void* stream) {
  const Shape s = pick_shape(a.k, 0);
  const bool small = small_matrix(v_rows, a.k);
  const hipStream_t st = (hipStream_t)stream;
  // items per workgroup as in launch_product
  const int least = kBlock / s.lpr < kItemsPerGroupBlock ? kBlock / s.lpr : kItemsPerGroupBlock;
  a.items = kItemsPerGroupBlock;
  if (!die_queues)
    while (a.items > least && a.n_rows < (int64_t)a.items * 2048) a.items >>= 1;
  const int64_t chunk_blocks = ceil_div(ceil_div(a.n_chunks, kBlock / 64), kDies) * kDies;
  const int64_t row_blocks = ceil_div(ceil_div(a.n_rows, a.items), kDies) * kDies;
  if (chunk_blocks + row_blocks > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
  a.runs = windows && !die_queues;
  return dispatch_shape(s, [&](auto Vc, auto L) -> int {
    constexpr int VEC = decltype(Vc)::value, LPR = decltype(L)::value;
    constexpr int NB = LPR < kSampledBatch ? LPR : kSampledBatch;
#define ARROW_LAUNCH(KERNEL, BLOCKS, ...)                                                                           \
  if (small) hipLaunchKernelGGL((KERNEL<VEC, LPR, NB, true __VA_ARGS__>), dim3((unsigned)(BLOCKS)), dim3(kBlock), 0, st, a); \
  else hipLaunchKernelGGL((KERNEL<VEC, LPR, NB, false __VA_ARGS__>), dim3((unsigned)(BLOCKS)), dim3(kBlock), 0, st, a)
#define ARROW_COMMA ,
    if (window_rows) {
      if (row_blocks > 0) { ARROW_LAUNCH(sddmm_rows_kernel, row_blocks, ARROW_COMMA true); }
    } else if (!windows && chunk_blocks > 0 && row_blocks > 0) {
      a.chunk_blocks = (uint32_t)chunk_blocks;
      ARROW_LAUNCH(sddmm_kernel, chunk_blocks + row_blocks, );
    } else {
      if (chunk_blocks > 0) { ARROW_LAUNCH(sddmm_chunks_kernel, chunk_blocks, ); }
      if (row_blocks > 0) { ARROW_LAUNCH(sddmm_rows_kernel, row_blocks, ARROW_COMMA false); }
    }
#undef ARROW_COMMA
#undef ARROW_LAUNCH
    return (int)hipGetLastError();
  });
}

}  // namespace arrow
