// Order-3 MTTKRP: host-side compressed-sparse-fibre build and the C boundary.
// The arithmetic of a product happens in the HIP kernels this file launches (mttkrp.hip and the
// shared partial-vector reduction); nothing here falls back to the CPU.
//
// Image: the entries as {k, value} pairs, by slice i; SEGMENTS, runs of at most
// kSegMax entries of one fibre (i, j) with the fibre's j (a long fibre is cut: the product with
// B(j, :) distributes over the pieces); ITEMS, runs of consecutive segments of one slice i with at
// most kItemNnz entries and kItemSegs segments, one per wavefront, with a destination: row i of A when the slice is one
// item, else a partial-vector slot that the reduction pass sums in a fixed order.  Every i in
// [0, I) has at least one item (an empty one stores zeros), so A is fully overwritten.
// Tensors whose factors fit the LDS, and tensors of many small slices whose factors do not fit an L2, get
// other forms (pack_resident, pack_streams).
#include <hip/hip_runtime.h>
#include <omp.h>

#include <algorithm>
#include <array>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "arrow.h"
#include "arrow_internal.h"
#include "csf3.h"

namespace {

thread_local std::string g_err3;

int fail3(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err3 = buf;
  return code;
}

constexpr size_t kAlign3 = 256;
size_t align3(size_t x) { return (x + kAlign3 - 1) / kAlign3 * kAlign3; }
constexpr int64_t kSegMax = arrow::kCsfSegMax;      // most entries of a segment
constexpr int64_t kItemNnz = arrow::kCsfItemNnz;    // an item is closed before it would hold more entries
constexpr int64_t kItemSegs = arrow::kCsfItemSegs;  // ... or more segments than this

}  // namespace

struct csf3_handle {
  int64_t I = 0, J = 0, K = 0, nnz = 0;
  int64_t longest = 0;       // entries and segments of the longest item
  int64_t slices = 0, fibers = 0, n_seg = 0, n_items = 0, n_split = 0, n_partials = 0;
  int64_t distinct_j = 0, distinct_k = 0;
  double build_seconds = 0.0;
  std::vector<unsigned char> bytes;   // packed host copy of the image
  size_t off_seg_ptr = 0, off_seg_j = 0, off_item_seg = 0, off_item_dst = 0, off_item_ent = 0, off_split_ptr = 0,
         off_split_y = 0, off_entries = 0;
  bool resident = false;              // the image is in the form for factors that fit the LDS
  size_t off_items = 0, off_last = 0;
  int64_t n_blocks = 0;
  bool streams = false;               // the form for many small slices and factors that do not fit an L2
  size_t off_waves = 0, off_dst = 0, off_zero = 0;
  int64_t n_waves = 0;
  unsigned char* dev = nullptr;
  unsigned char* ws = nullptr;
  size_t ws_bytes = 0;
  bool profiling = false, profiled = false;
  hipEvent_t ev[3] = {nullptr, nullptr, nullptr};   // before the kernel, between, after the reduction
};

namespace {

// Where the resident form pays.  Both forms measured on 2854 uniform tensors of 128 to 4096 rows a side and 30 K to 8 M entries, R = 8, 12,
// 25, 32, 50, 64, 100 and 128: of the 1293 that this rule takes all gain on average over the ranks, 0.38 to 0.90 times the
// other form's time, and four lose at a single rank, the worst 157 x 3694 x 1451 of 841 K, R = 32, 15.2 -> 17.3 us.
//   608 x 1224 x 1970 of 1.47 M, 1.18 steps per 64 rows, R = 8 / 64 / 128   13.9 / 29.8 / 49.7 -> 7.2 / 18.9 / 29.2
//   2414 x 1806 x 310 of 1.35 M, 1.47                                       14.3 / 32.8 / 55.5 -> 6.4 / 22.4 / 39.1
//   144 x 415 x 1945 of 116 K, 1.36, 144 items                               8.3 / 13.5 / 19.3 -> 4.5 /  6.6 /  7.9
//   282 x 223 x 1855 of 117 K, 1.74                                          7.7 / 12.2 / 17.0 -> 4.4 /  6.9 /  8.5
// Fill is what loses at high ranks (beside thousands of slices that are shorter than a block: 4055 x 994 x 147 of 592 K, 1.85:
// 10.5 / 18.2 / 27.3 -> 5.0 / 18.9 / 32.6; 4061 x 347 x 430 of 606 K, 2.02: 10.3 / 18.4 / 27.3 -> 5.1 / 18.6 / 32.8); from 2.1 on single tensors
// lose on average.  Fewer items were not measured; tensors of 30 K to 64 K entries gained too and keep the form that they had.
constexpr int64_t kResidentNnz = 1 << 16;
constexpr int64_t kResidentItems = 128;
constexpr double kResidentFill = 1.8;
// And every workgroup copies all J + K rows, which has to be paid for by the rows that are read, entries and segments,
// where they are so many that eight columns of them do not fit the LDS (below that nothing was lost down to 30 rows read per row
// copied).  The rank is not known here; 32 gains least (whole lines for the other form, and all compute units copy).  us, R = 8 / 32 /
// 64 / 128; in brackets rows read per row copied, geometric mean over those ranks and 12, 24, 50 and 100:
//   600 x 1000 x 9100 of 500 K  [83,  -6 %]       9.8 / 11.4 / 15.2 / 30.4 ->  7.2 / 15.0 / 17.4 / 26.7
//   520 x 9000 x 1000 of 560 K [109,  -8 %]       9.7 / 12.2 / 16.7 / 30.9 ->  7.0 / 15.8 / 18.7 / 28.5
//   783 x 1736 x 7090 of 806 K [160, -20 %]      11.7 / 14.0 / 20.4 / 38.3 ->  7.4 / 15.1 / 19.4 / 30.6
//   3000 x 2525 x 7575 of 1.2 M [229, -27 %]     17.0 / 20.4 / 32.1 / 64.6 ->  7.9 / 21.1 / 30.1 / 50.4
//   785 x 8113 x 1294 of 1.2 M [244, -35 %]      15.7 / 20.0 / 31.2 / 59.5 ->  8.3 / 18.3 / 24.5 / 39.0
//   757 x 1673 x 3882 of 874 K [271, -32 %]      11.9 / 14.9 / 21.1 / 35.6 ->  7.3 / 12.4 / 16.5 / 26.9
//   3000 x 2525 x 7575 of 2.5 M [458, -42 %]     28.1 / 34.6 / 55.7 / 115  -> 11.8 / 27.7 / 41.2 / 73.2
// so from 200 on, where rank 32 loses 9 % at most; below that the others gain on average but it loses up to a third (24, 50, 100 at [109]: 13.6 / 18.7 /
// 29.6 -> 12.1 / 18.5 / 24.5).  Where there is hardly more than an item per wavefront the other form is not filled either, and the first 2600 rows are
// free: 299 x 503 x 3305 of 371 K [134, -34 %] gains at every rank, 520 x 5000 x 5000 of 600 K [114], 900 K [166] and 1.2 M [216] 14, 22 and 26 %
// on average (R = 32: 13.0 / 15.0 / 18.0 -> 16.3 / 18.2 / 19.7).
constexpr int64_t kResidentReuse = 200, kResidentFew = 640, kResidentFree = 2600;
constexpr int64_t kResidentSegs = 4096;    // segments of an item
// Lanes whose 16-byte reads of LDS are served together (found by timing reads whose rows lie in different banks
// for one grouping only: 2.7 ns a wavefront's read against 3.7 to 7 for the other groupings and 5.0 at random).
constexpr uint8_t kSixteens[4][16] = {{0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27},
                                      {4, 5, 6, 7, 8, 9, 10, 11, 16, 17, 18, 19, 28, 29, 30, 31},
                                      {32, 33, 34, 35, 44, 45, 46, 47, 52, 53, 54, 55, 56, 57, 58, 59},
                                      {36, 37, 38, 39, 40, 41, 42, 43, 48, 49, 50, 51, 60, 61, 62, 63}};

// Packs the segments in the resident form (arrow_internal.h), or leaves the image alone and returns false where that form does
// not pay: factors that do not fit the LDS, too few entries to pay for copying them there, or so few fibres per
// slice, or of so unequal length, that the lanes would work on fill.  `at` gives the caller's index of an entry.
//
// An item's segments go to batches of 64 by length, longest first, one per lane; what a lane reads in a step is
// free to choose.  Sixteen lanes are served together and wait for the bank that most of them want, 3.1 of them
// at random: so a batch's segments are dealt to the sixteens by the bank of their row of B, and of its entries
// a lane takes first the one whose bank is wanted least in this step and most in those to come, which leaves 2.0
// (uniform 4096^3, R = 64: 529 -> 463 us; entries and rows of B are added in this order, not in that of j and k).
template <typename At>
bool pack_resident(csf3_handle& h, const std::vector<uint32_t>& seg_ptr, const std::vector<int32_t>& seg_j,
                   const std::vector<int32_t>& seg_i, At at, const int32_t* tk, const float* tv) {
  if (h.J + h.K + 1 > arrow::kCsfRowsInLds || h.nnz < kResidentNnz) return false;
  const double most = kResidentFill * (double)(h.nnz + h.n_seg);           // rows read, fill included
  if (64.0 * arrow::kCsfBlockSteps * (double)h.I > most) return false;     // (a block per slice at least)
  struct Part { uint32_t seg, n, block, blocks, steps; int32_t dst; };
  std::vector<Part> parts;
  std::vector<uint32_t> split_ptr{0};
  std::vector<int32_t> split_y;
  int64_t slots = 0;
  // A slice is cut where it holds more segments than an item may, or much more rows than the items' average.
  // (Whole slices where possible: every cut adds fill, at the lengths of its own, and a partial vector.)
  const int64_t cost_max = std::max<int64_t>(4096, (h.nnz + h.n_seg) / 2048);
  for (int64_t i = 0, s = 0; i < h.I; ++i) {
    int64_t end = s;
    while (end < h.n_seg && seg_i[end] == i) ++end;
    const int64_t segs = end - s, cost = segs ? (int64_t)(seg_ptr[end] - seg_ptr[s]) + segs : 0;
    const int64_t n = std::max<int64_t>({1, (segs + kResidentSegs - 1) / kResidentSegs, cost / cost_max});
    for (int64_t t = 0; t < n; ++t) {
      const int64_t lo = s + segs * t / n, hi = s + segs * (t + 1) / n;
      parts.push_back({(uint32_t)lo, (uint32_t)(hi - lo), 0, 0, 0, n == 1 ? (int32_t)i : (int32_t)(-1 - (slots + t))});
    }
    if (n > 1) {
      slots += n;
      split_ptr.push_back((uint32_t)slots);
      split_y.push_back((int32_t)i);
    }
    s = end;
  }
  if (slots > 0x7fffffffLL || parts.size() > 0x7fffff00ULL) return false;
  if ((int64_t)parts.size() < kResidentItems) return false;
  const int64_t copied = h.J + h.K - ((int64_t)parts.size() <= kResidentFew ? kResidentFree : 0);
  if (2 * (h.J + h.K + 1) > arrow::kCsfRowsInLds && h.nnz + h.n_seg < kResidentReuse * copied) return false;
  // segments by length, longest first: at_len[l] = where those of length kSegMax - l begin
  auto by_length = [&](const Part& p, std::array<uint32_t, kSegMax + 2>& at_len) {
    at_len.fill(0);
    for (uint32_t q = p.seg; q < p.seg + p.n; ++q) ++at_len[(size_t)(kSegMax - (seg_ptr[q + 1] - seg_ptr[q])) + 1];
    for (size_t q = 1; q < at_len.size(); ++q) at_len[q] += at_len[q - 1];
  };
  const int64_t n_parts = (int64_t)parts.size();
#pragma omp parallel for schedule(dynamic, 16)
  for (int64_t t = 0; t < n_parts; ++t) {
    std::array<uint32_t, kSegMax + 2> at_len;
    by_length(parts[t], at_len);
    uint32_t steps = 0;
    for (uint32_t first = 0, l = 0; first < parts[t].n; first += 64) {     // l: kSegMax - the length of segment `first`
      while (at_len[l + 1] <= first) ++l;
      steps += (uint32_t)kSegMax - l + 1;
    }
    parts[t].steps = steps;
    parts[t].blocks = std::max(1u, (steps + arrow::kCsfBlockSteps - 1) / arrow::kCsfBlockSteps);
  }
  int64_t blocks = 0;
  for (Part& p : parts) {
    if (blocks > 0xffffffffLL) return false;
    p.block = (uint32_t)blocks;
    blocks += p.blocks;
  }
  if ((double)(blocks * 64 * arrow::kCsfBlockSteps) > most) return false;
  size_t total = 0;
  h.off_items = total;     total = align3(total + sizeof(arrow::ResidentItem) * parts.size());
  h.off_last = total;      total = align3(total + sizeof(uint32_t) * parts.size());
  h.off_split_ptr = total; total = align3(total + sizeof(uint32_t) * split_ptr.size());
  h.off_split_y = total;   total = align3(total + sizeof(int32_t) * split_y.size());
  h.off_entries = total;   total = align3(total + sizeof(arrow::ResidentBlock) * (size_t)blocks);
  h.bytes.assign(total, 0);
  unsigned char* base = h.bytes.data();
  std::memcpy(base + h.off_split_ptr, split_ptr.data(), sizeof(uint32_t) * split_ptr.size());
  if (!split_y.empty()) std::memcpy(base + h.off_split_y, split_y.data(), sizeof(int32_t) * split_y.size());
  // the longest items first: the wavefronts take them in turn
  std::vector<uint32_t> turn(parts.size());
  for (size_t t = 0; t < turn.size(); ++t) turn[t] = (uint32_t)t;
  std::stable_sort(turn.begin(), turn.end(), [&](uint32_t a, uint32_t b) { return parts[a].blocks > parts[b].blocks; });
  arrow::ResidentItem* items = reinterpret_cast<arrow::ResidentItem*>(base + h.off_items);
  uint32_t* last = reinterpret_cast<uint32_t*>(base + h.off_last);
  for (size_t t = 0; t < turn.size(); ++t) {
    const Part& p = parts[turn[t]];
    items[t] = {p.block, p.blocks, p.dst};
    last[t] = p.steps - std::min(p.steps, (p.blocks - 1) * (uint32_t)arrow::kCsfBlockSteps);
  }
  arrow::ResidentBlock* image = reinterpret_cast<arrow::ResidentBlock*>(base + h.off_entries);
  const uint32_t zeros = (uint32_t)h.K;
#pragma omp parallel for schedule(dynamic, 16)
  for (int64_t t = 0; t < n_parts; ++t) {                        // (nothing in here may throw)
    const Part& p = parts[t];
    std::array<uint32_t, kSegMax + 2> at_len;
    std::array<uint16_t, kResidentSegs> order;
    by_length(p, at_len);
    for (uint32_t q = 0; q < p.n; ++q) order[at_len[(size_t)(kSegMax - (seg_ptr[p.seg + q + 1] - seg_ptr[p.seg + q]))]++] = (uint16_t)q;
    auto put = [&](uint32_t step, uint32_t lane, uint32_t row, float v, bool end = false) {
      arrow::ResidentBlock& b = image[p.block + step / 8];
      b.offsets[lane].pair[step % 8 / 2] |= row << (step % 2 ? 18 : 4) | (uint32_t)end << step % 2;
      b.values[step % 8 / 4][lane].v[step % 4] = v;
    };
    uint32_t step = 0;
    for (uint32_t first = 0; first < p.n; first += 64) {
      const uint32_t longest = seg_ptr[p.seg + order[first] + 1] - seg_ptr[p.seg + order[first]];
      const uint32_t m = std::min<uint32_t>(64, p.n - first);
      // lanes: the segments by the bank of their row of B, dealt to the sixteens
      std::array<uint32_t, 17> at_bank{};
      auto end_of = [&](uint32_t q) { return zeros + 1 + (uint32_t)seg_j[p.seg + order[first + q]]; };
      for (uint32_t q = 0; q < m; ++q) ++at_bank[end_of(q) % 16 + 1];
      for (size_t q = 1; q < 17; ++q) at_bank[q] += at_bank[q - 1];
      std::array<uint8_t, 64> dealt;
      for (uint32_t q = 0; q < m; ++q) dealt[at_bank[end_of(q) % 16]++] = (uint8_t)q;
      for (uint32_t g = 0; g < 4; ++g) {
        std::array<std::array<uint32_t, kSegMax>, 16> src;      // caller's index of the entries of the sixteen lanes
        std::array<std::array<uint8_t, kSegMax>, 16> bank;
        std::array<uint32_t, 16> n{};
        std::array<uint32_t, 16> left{};                        // entries still to come, by bank
        for (uint32_t x = 0; x < 16; ++x) {
          const uint32_t lane = kSixteens[g][x];
          uint32_t end = zeros;
          if (x * 4 + g < m) {
            const uint32_t q = p.seg + order[first + dealt[x * 4 + g]], from = seg_ptr[q];
            n[x] = seg_ptr[q + 1] - from;
            end = zeros + 1 + (uint32_t)seg_j[q];
            for (uint32_t l = 0; l < n[x]; ++l) {
              src[x][l] = (uint32_t)at(from + l);
              bank[x][l] = (uint8_t)(tk[src[x][l]] % 16);
              ++left[bank[x][l]];
            }
          }
          put(step + longest, lane, end, 0.f, true);
        }
        for (uint32_t l = 0; l < longest; ++l) {
          std::array<uint32_t, 16> taken{};                     // lanes of this step, by bank
          for (uint32_t x = 0; x < 16; ++x) {
            const uint32_t lane = kSixteens[g][x];
            if (l >= n[x]) { put(step + l, lane, zeros, 0.f); continue; }
            uint32_t best = l, cost = ~0u;
            for (uint32_t c = l; c < n[x]; ++c) {
              const uint32_t b = bank[x][c], at_b = taken[b] * 1024 + 1023 - std::min(left[b], 1023u);
              if (at_b < cost) { cost = at_b; best = c; }
            }
            std::swap(src[x][l], src[x][best]);
            std::swap(bank[x][l], bank[x][best]);
            ++taken[bank[x][l]];
            --left[bank[x][l]];
            put(step + l, lane, (uint32_t)tk[src[x][l]], tv[src[x][l]]);
          }
        }
      }
      step += longest + 1;
    }
    for (; step < p.blocks * 8; ++step)
      for (uint32_t lane = 0; lane < 64; ++lane) put(step, lane, zeros, 0.f);
  }
  h.n_items = n_parts;
  h.n_split = (int64_t)split_y.size();
  h.n_partials = slots;
  h.n_blocks = blocks;
  h.resident = true;
  return true;
}

// Where the streams form pays (both forms measured, us, R = 8 / 32 / 50 / 128; skewed tensors of 32 entries per slice unless
// said otherwise):
//   524288 x 65536 x 65536 of 16.8 M           329 / 505 / 1149 / 2179 -> 199 / 293 / 624 / 1180
//   180000 x 22500 x 22500 of 5.8 M            110 / 144 /  253 /  621 ->  72 /  96 / 201 /  364
//   800000 x  2000 x  2000 of 4.2 M, uniform   R = 33 / 66 / 100 / 128: 397 / 458 / 464 / 467 -> 201 / 332 / 473 / 362
// The rank is not known here, and ranks that are no multiple of 32 pay for the columns that fill the last slice: R = 33 / 66 /
// 100 take 192 / 291 / 388 instead of 197 / 350 / 545 us at 180000 x 22500 x 22500.  So it stays away where they would lose
// to factors that an L2 holds (90000 x 7500 x 18000: 94 / 149 / 208 -> 108 / 162 / 212, although R = 32 takes 55 instead of
// 72; 120000 x 20000 x 24000: 134 / 235 / 364 -> 139 / 210 / 280), unless slices are short, whose items the other form cannot fill
// (400000 x 2000 x 2000 of 4.2 M: 228 / 271 / 285 -> 160 / 255 / 356), and from long
// slices, whose items go through B in order by themselves (500 x 30000 x 30000 of 8.4 M: 84 / 149 / 406 / 905 -> 139 /
// 197 / 327 / 571), and fibres of several entries, for each of which it reads the row of B again.
// Where the factors have many rows for the tensor's entries, hardly one is read again while it is in an L2, and at
// ranks that are no whole lines every pass over the columns touches lines of its neighbours (this form over the
// ordinary one at R = 8 / 24 / 32 / 50 / 100 / 128; geometric mean with R = 4, 12 and 64; uniform tensors):
//   500k slices, 16 M, rows 1/8 of the entries  .86 / .79 / .95 / 1.02 / 1.27 /  .98   .94
//                           1/4                 .93 / .89 / 1.0 / 1.20 / 1.32 /  .90   .99
//                           1/2                 .96 / .98 / .95 / 1.57 / 1.63 /  .86   1.05
//   500k slices,  8 M       1/8                 .81 / .77 / .86 / 1.03 / 1.26 / 1.04   .90
//                           1/2                 .95 / .95 / .86 / 1.75 / 1.69 /  .88   1.05
//   800k slices,  6.4 M     1/8                 .52 / .64 / .63 / 1.00 / 1.35 / 1.12   .74
//                           1/1                 .68 / .76 / .58 / 1.61 / 1.81 /  .88   .87
//   4 M  slices,  8 M       1/1                 R = 6 / 12 / 24 / 50 / 100: .23 / .25 / .35 / 1.02 / 1.54
// so from 1/4 on it stays away unless slices have fewer than kStreamLong entries.
// Empty slices do not make the others short.  200k slices of which few hold 8.4 M entries, J = K = 30000 (this form over the
// ordinary one, R = 8 / 12 / 25 / 32 / 50 / 64 / 100 / 128; geometric mean):
//   500, 16800 entries each   1.33 / 1.79 / 1.24 / 1.39 / .91 / .90 / .79 / .70   1.08
//   5000, 1680                1.15 / 1.47 / 1.00 / 1.18 / .88 / .92 / .81 / .74   1.00
//   10000, 840                1.00 / 1.25 /  .89 / 1.06 / .81 / .84 / .79 / .73   .91
//   60000, 140                 .65 /    -  /  .60 /  .65 / .59 /   -  /   -  / .55
// but the ordinary form takes a wavefront for each of them too: 500 of 600k slices .79 / 1.15 / 1.04 / 1.07 / 1.03 / .94 / .91 /
// .73 (.95), 500 of 1.1 M with 4.2 M entries .32 to 1.39 (.72).
constexpr int64_t kStreamNnz = 1 << 21;
constexpr int64_t kStreamSlice = 64;       // most entries of a slice on average,
constexpr int64_t kStreamFull = 1024;      // ... of those that are not empty, unless
constexpr int64_t kStreamEmpty = 16;       // ... there is an empty one for so many entries,
constexpr int64_t kStreamShort = 4;        // ... and where the factors have fewer rows than this:
constexpr int64_t kStreamRows = 45000;
constexpr int64_t kStreamReuse = 4;        // fewest entries per row of the factors, and where there are fewer:
constexpr int64_t kStreamLong = 12;        // most entries of a slice on average
constexpr int64_t kStreamWaves = 4096;     // wavefronts that are resident at a time
// Windows of one factor's rows, each with the same share of the entries.  Few of them leave more rows in use at a time,
// many leave a row's entries one by one, and its sum is rounded for each (they are added up by window first): 8 / 16 windows
// 293 / 286 us, 2-norm of the error 0.61 / 0.74e-7 (512k x 64k x 64k, R = 32; 0.82e-7 in the other form).
constexpr int kStreamWindows = 8;

// Packs the entries in the streams form (arrow_internal.h), or leaves the image alone and returns false.
// Rows of A (pieces of the longest) are dealt to the lane groups of all wavefronts so that every group has
// about the same number of entries, and groups to wavefronts so that none has more rows than it has room for.
template <typename At>
bool pack_streams(csf3_handle& h, At at, const int32_t* ti, const int32_t* tj, const int32_t* tk, const float* tv) {
  constexpr int64_t G = arrow::kCsfStreamGroups, room = arrow::kCsfStreamRows;
  if (h.nnz < kStreamNnz || h.J > arrow::kCsfStreamRowsOfB || h.fibers * 4 < h.nnz * 3 || h.nnz > kStreamSlice * h.I) return false;
  if (h.nnz > kStreamFull * h.slices && h.nnz > kStreamEmpty * (h.I - h.slices)) return false;
  if (h.J + h.K < kStreamRows && h.nnz > kStreamShort * h.I) return false;
  if (h.nnz < kStreamReuse * (h.J + h.K) && h.nnz > kStreamLong * h.I) return false;
  struct Row { uint32_t first, n; int32_t i; };                   // a slice with entries
  std::vector<Row> rows;
  std::vector<int32_t> zero;
  rows.reserve((size_t)h.slices);
  zero.reserve((size_t)(h.I - h.slices));
  for (int64_t p = 0, i = 0; i < h.I; ++i) {
    const int64_t first = p;
    while (p < h.nnz && ti[at(p)] == i) ++p;
    if (p > first) rows.push_back({(uint32_t)first, (uint32_t)(p - first), (int32_t)i});
    else zero.push_back((int32_t)i);
  }
  struct Piece { uint32_t first, n; int32_t dst; };
  std::vector<Piece> pieces;
  std::vector<uint32_t> split_ptr, group_of, order;
  std::vector<int32_t> split_y;
  std::vector<uint32_t> group_rows;
  int64_t slots = 0, n_waves = 0;
  for (int64_t rounds = ((int64_t)rows.size() + kStreamWaves * room - 1) / (kStreamWaves * room);; ++rounds) {
    n_waves = kStreamWaves * rounds;
    if (n_waves * G > 0x7fffffffLL || rounds > 64) return false;
    const uint32_t share = (uint32_t)std::max<int64_t>(16, (h.nnz + n_waves * G - 1) / (n_waves * G));   // entries of a group
    pieces.clear(); split_y.clear(); split_ptr.assign(1, 0);
    slots = 0;
    for (const Row& r : rows) {
      const uint32_t n = (r.n + share - 1) / share;
      for (uint32_t t = 0; t < n; ++t) {
        const uint32_t lo = (uint32_t)((uint64_t)r.n * t / n), hi = (uint32_t)((uint64_t)r.n * (t + 1) / n);
        pieces.push_back({r.first + lo, hi - lo, n == 1 ? r.i : (int32_t)(-1 - (slots + t))});
      }
      if (n > 1) {
        slots += n;
        split_ptr.push_back((uint32_t)slots);
        split_y.push_back(r.i);
      }
    }
    if (slots > 0x7fffffffLL) return false;
    if ((int64_t)pieces.size() > n_waves * room) continue;
    // longest piece first to the group with the fewest entries, groups in lists by how many they have
    std::vector<uint32_t> at_len(share + 2, 0);
    for (const Piece& p : pieces) ++at_len[share - p.n + 1];
    for (size_t q = 1; q < at_len.size(); ++q) at_len[q] += at_len[q - 1];
    order.resize(pieces.size());
    for (size_t q = 0; q < pieces.size(); ++q) order[at_len[share - pieces[q].n]++] = (uint32_t)q;
    const size_t n_groups = (size_t)(n_waves * G);
    constexpr uint32_t none = ~0u;
    std::vector<uint32_t> next(n_groups), head(2 * (size_t)share + 2, none);
    for (size_t q = 0; q < n_groups; ++q) next[q] = q + 1 < n_groups ? (uint32_t)(q + 1) : none;
    head[0] = 0;
    size_t least = 0;
    group_of.resize(pieces.size());
    group_rows.assign(n_groups, 0);
    for (const uint32_t q : order) {
      while (head[least] == none) ++least;
      const uint32_t g = head[least];
      head[least] = next[g];
      const size_t load = least + pieces[q].n;                     // (at most twice the share: the least load is no more than it)
      next[g] = head[load];
      head[load] = g;
      group_of[q] = g;
      ++group_rows[g];
    }
    // eight groups to a wavefront, those with many rows beside those with few
    const uint32_t most = *std::max_element(group_rows.begin(), group_rows.end());
    std::vector<uint32_t> at_rows(most + 2, 0), place(n_groups);
    for (const uint32_t r : group_rows) ++at_rows[most - r + 1];
    for (size_t q = 1; q < at_rows.size(); ++q) at_rows[q] += at_rows[q - 1];
    for (size_t g = 0; g < n_groups; ++g) {
      const size_t rank = at_rows[most - group_rows[g]]++, turn = rank / (size_t)n_waves, w = rank % (size_t)n_waves;
      place[g] = (uint32_t)((turn % 2 ? (size_t)n_waves - 1 - w : w) * G + turn);
    }
    std::vector<uint32_t> wave_rows((size_t)n_waves, 0);
    for (size_t g = 0; g < n_groups; ++g) wave_rows[place[g] / G] += group_rows[g];
    if (*std::max_element(wave_rows.begin(), wave_rows.end()) > (uint32_t)room) continue;
    for (uint32_t& g : group_of) g = place[g];
    break;
  }
  // pieces by group, and their entries by window of the rows of the factor with more of them
  const size_t n_groups = (size_t)(n_waves * G);
  std::vector<uint32_t> group_ptr(n_groups + 1, 0), by_group(pieces.size());
  for (const uint32_t g : group_of) ++group_ptr[g + 1];
  for (size_t g = 0; g < n_groups; ++g) group_ptr[g + 1] += group_ptr[g];
  {
    std::vector<uint32_t> to(group_ptr.begin(), group_ptr.end() - 1);
    for (size_t q = 0; q < pieces.size(); ++q) by_group[to[group_of[q]]++] = (uint32_t)q;
  }
  const bool by_k = h.distinct_k >= h.distinct_j;
  const int32_t* key = by_k ? tk : tj;
  std::vector<uint8_t> window((size_t)(by_k ? h.K : h.J));
  {
    std::vector<uint32_t> uses(window.size(), 0);
    for (int64_t p = 0; p < h.nnz; ++p) ++uses[key[p]];
    uint64_t before = 0;
    for (size_t r = 0; r < window.size(); ++r) {
      window[r] = (uint8_t)(before * kStreamWindows / (uint64_t)h.nnz);
      before += uses[r];
    }
  }
  std::vector<arrow::StreamWave> waves((size_t)n_waves);
  std::vector<uint32_t> group_nnz(n_groups, 0);
  for (size_t q = 0; q < pieces.size(); ++q) group_nnz[group_of[q]] += pieces[q].n;
  uint64_t blocks = 0;
  for (int64_t w = 0; w < n_waves; ++w) {
    uint32_t longest = 0;
    for (int64_t g = 0; g < G; ++g) longest = std::max(longest, group_nnz[(size_t)(w * G + g)]);
    const uint32_t n = (longest + 7) / 8;
    const uint64_t z = zero.size();
    waves[(size_t)w] = {(uint32_t)blocks, n, 0, (uint32_t)(z * w / n_waves), (uint32_t)(z * (w + 1) / n_waves - z * w / n_waves)};
    blocks += n;
  }
  if (blocks > 0xffffffffULL) return false;
  for (size_t w = 0; w < waves.size(); ++w)
    for (size_t t = w / arrow::kCsfStreamTeam * arrow::kCsfStreamTeam; t < waves.size() && t / arrow::kCsfStreamTeam == w / arrow::kCsfStreamTeam; ++t)
      waves[w].turns = std::max(waves[w].turns, waves[t].blocks / arrow::kCsfStreamTurn);
  size_t total = 0;
  h.off_waves = total;     total = align3(total + sizeof(arrow::StreamWave) * waves.size());
  h.off_dst = total;       total = align3(total + sizeof(int32_t) * (size_t)(n_waves * room));
  h.off_zero = total;      total = align3(total + sizeof(int32_t) * zero.size());
  h.off_split_ptr = total; total = align3(total + sizeof(uint32_t) * split_ptr.size());
  h.off_split_y = total;   total = align3(total + sizeof(int32_t) * split_y.size());
  h.off_entries = total;   total = align3(total + sizeof(arrow::StreamBlock) * (size_t)blocks);
  h.bytes.assign(total, 0);
  unsigned char* base = h.bytes.data();
  std::memcpy(base + h.off_waves, waves.data(), sizeof(arrow::StreamWave) * waves.size());
  if (!zero.empty()) std::memcpy(base + h.off_zero, zero.data(), sizeof(int32_t) * zero.size());
  std::memcpy(base + h.off_split_ptr, split_ptr.data(), sizeof(uint32_t) * split_ptr.size());
  if (!split_y.empty()) std::memcpy(base + h.off_split_y, split_y.data(), sizeof(int32_t) * split_y.size());
  int32_t* dst = reinterpret_cast<int32_t*>(base + h.off_dst);
  arrow::StreamBlock* image = reinterpret_cast<arrow::StreamBlock*>(base + h.off_entries);
#pragma omp parallel for schedule(static)
  for (int64_t w = 0; w < n_waves; ++w) {                          // (nothing in here may throw)
    const arrow::StreamWave& d = waves[(size_t)w];
    uint32_t place = 0;
    for (uint32_t g = 0; g < (uint32_t)G; ++g) {
      const size_t group = (size_t)(w * G + g);
      std::array<uint32_t, kStreamWindows + 1> to{};
      for (uint32_t q = group_ptr[group]; q < group_ptr[group + 1]; ++q) {
        const Piece& p = pieces[by_group[q]];
        for (uint32_t e = p.first; e < p.first + p.n; ++e) ++to[window[(size_t)key[at(e)]] + 1];
      }
      for (size_t v = 1; v < to.size(); ++v) to[v] += to[v - 1];
      auto record = [&](uint32_t s) -> arrow::StreamBlock::Record& { return image[d.block + s / 8].rec[g * 8 + s % 8]; };
      for (uint32_t q = group_ptr[group]; q < group_ptr[group + 1]; ++q, ++place) {
        const Piece& p = pieces[by_group[q]];
        dst[w * room + place] = p.dst;
        for (uint32_t e = p.first; e < p.first + p.n; ++e) {
          const int64_t src = at(e);
          record(to[window[(size_t)key[src]]]++) = {(uint32_t)tj[src] << 7 | place, tk[src], tv[src]};
        }
      }
      for (uint32_t s = group_nnz[group]; s < d.blocks * 8; ++s) record(s) = {(uint32_t)room, 0, 0.f};
    }
    for (; place < (uint32_t)room; ++place) dst[w * room + place] = arrow::kCsfNoRow;
  }
  h.n_items = (int64_t)(pieces.size() + zero.size());
  h.n_split = (int64_t)split_y.size();
  h.n_partials = slots;
  h.n_waves = n_waves;
  h.streams = true;
  return true;
}

// workspace layout: [partial vectors][factors laid out anew]
size_t partial_bytes(const csf3_handle& h, int32_t R) { return align3((size_t)h.n_partials * (size_t)R * sizeof(float)); }
// Entries for every row of the factors from which on laying them out anew pays: it copies all J + K of them, whether an entry
// refers to them or not (us, in place / laid out anew; the ordinary form):
//   1M x 20M x 20M of 2.3 M    [0.06]   R = 25 272 / 1806 (529), 50 668 / 5099 (571)
//   500k x 4M x 4M of 16 M     [2]      R = 12 +4 %, 24 +8 %, 50 -14 %, 100 -2 %
//   500k x 2M x 2M of 16 M     [4]      R = 12 -3 %, 24 -8 %, 50 -31 %, 100 -21 %
//   500k x 500k x 500k of 8 M  [8]      R = 12 -4 %, 24 -15 %, 50 -41 %, 100 -33 %
constexpr int64_t kStreamCopied = 3;
size_t laid_out_bytes(const csf3_handle& h, int32_t R) {
  if (!h.streams || h.nnz < kStreamCopied * (h.J + h.K)) return 0;
  return align3(sizeof(float) * (size_t)arrow::stream_scratch(h.J, h.K, R));
}

}  // namespace

extern "C" {

const char* csf3_last_error(void) { return g_err3.c_str(); }

int csf3_build(int64_t I, int64_t J, int64_t K, int64_t nnz, const int32_t* ti, const int32_t* tj,
               const int32_t* tk, const float* tv, csf3_handle** out) {
  if (!out) return fail3(ARROW_EINVAL, "out is NULL");
  *out = nullptr;
  if (I < 1 || J < 1 || K < 1 || I > 2147483647LL || J > 2147483647LL || K > 2147483647LL)
    return fail3(ARROW_EINVAL, "mode sizes must be in [1, 2^31 - 1]");
  if (nnz < 0 || nnz >= 0xffffffffLL) return fail3(ARROW_EINVAL, "nnz must be in [0, 2^32 - 2]");
  if (nnz > 0 && (!ti || !tj || !tk || !tv)) return fail3(ARROW_EINVAL, "a coordinate or value array is NULL");
  auto t0 = std::chrono::steady_clock::now();
  try {
    int64_t bad = -1;
    bool sorted = true;
#pragma omp parallel for schedule(static) reduction(&& : sorted)
    for (int64_t p = 0; p < nnz; ++p) {
      if (ti[p] < 0 || ti[p] >= I || tj[p] < 0 || tj[p] >= J || tk[p] < 0 || tk[p] >= K) {
#pragma omp critical
        if (bad < 0 || p < bad) bad = p;
      }
      if (p > 0) {
        const bool le = ti[p - 1] != ti[p] ? ti[p - 1] < ti[p]
                        : (tj[p - 1] != tj[p] ? tj[p - 1] < tj[p] : tk[p - 1] <= tk[p]);
        sorted = sorted && le;
      }
    }
    if (bad >= 0) return fail3(ARROW_EINVAL, "entry %lld has a coordinate out of range", (long long)bad);
    // order of the entries by (i, j, k); equal coordinates keep the caller's order
    std::vector<uint32_t> order;
    if (!sorted) {
      order.resize((size_t)nnz);
      for (int64_t p = 0; p < nnz; ++p) order[p] = (uint32_t)p;
      std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
        if (ti[x] != ti[y]) return ti[x] < ti[y];
        if (tj[x] != tj[y]) return tj[x] < tj[y];
        return tk[x] < tk[y];
      });
    }
    auto at = [&](int64_t p) -> int64_t { return sorted ? p : (int64_t)order[p]; };

    auto h = std::make_unique<csf3_handle>();
    h->I = I; h->J = J; h->K = K; h->nnz = nnz;
    // segments: a new one starts where the fibre changes or the current one is full
    std::vector<uint32_t> seg_ptr;
    std::vector<int32_t> seg_j, seg_i;
    seg_ptr.reserve((size_t)(nnz / 2 + 16)); seg_j.reserve((size_t)(nnz / 2 + 16)); seg_i.reserve((size_t)(nnz / 2 + 16));
    for (int64_t p = 0; p < nnz; ++p) {
      const int64_t q = at(p);
      const bool new_fiber = p == 0 || ti[at(p - 1)] != ti[q] || tj[at(p - 1)] != tj[q];
      if (new_fiber) {
        ++h->fibers;
        if (p == 0 || ti[at(p - 1)] != ti[q]) ++h->slices;
      }
      if (new_fiber || (int64_t)(p - seg_ptr.back()) >= kSegMax) {
        seg_ptr.push_back((uint32_t)p);
        seg_j.push_back(tj[q]);
        seg_i.push_back(ti[q]);
      }
    }
    seg_ptr.push_back((uint32_t)nnz);
    h->n_seg = (int64_t)seg_j.size();
    {
      std::vector<uint8_t> seen_j((size_t)J, 0), seen_k((size_t)K, 0);
      for (int64_t p = 0; p < nnz; ++p) { seen_j[tj[p]] = 1; seen_k[tk[p]] = 1; }
      for (uint8_t v : seen_j) h->distinct_j += v;
      for (uint8_t v : seen_k) h->distinct_k += v;
    }
    if (pack_resident(*h, seg_ptr, seg_j, seg_i, at, tk, tv) || pack_streams(*h, at, ti, tj, tk, tv)) {
      h->build_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
      *out = h.release();
      return ARROW_OK;
    }
    // items: per slice i (empty slices included), consecutive segments up to kItemNnz entries
    // and kItemSegs segments
    std::vector<uint32_t> item_seg, split_ptr;
    std::vector<int32_t> item_dst, split_y;
    split_ptr.push_back(0);
    // How many items a slice needs when each takes what it can hold, and then as many that cost about the
    // same (rows gathered: one per entry and one per segment).
    auto fits = [&](int64_t at_seg, int64_t cnt, int64_t segs) {
      return at_seg < h->n_seg && seg_i[at_seg] == seg_i[at_seg - segs] && segs < kItemSegs &&
             (cnt == 0 || cnt + (seg_ptr[at_seg + 1] - seg_ptr[at_seg]) <= kItemNnz);
    };
    std::vector<std::pair<int64_t, int64_t>> need;   // of the slices with entries: (end, items)
    need.reserve((size_t)h->slices);
    bool split = false;
    int64_t wanted = I - h->slices;
    for (int64_t at_seg = 0; at_seg < h->n_seg;) {
      const int32_t i = seg_i[at_seg];
      int64_t items = 0;
      while (at_seg < h->n_seg && seg_i[at_seg] == i) {
        ++items;
        for (int64_t cnt = 0, segs = 0; fits(at_seg, cnt, segs); ++segs, ++at_seg) cnt += seg_ptr[at_seg + 1] - seg_ptr[at_seg];
      }
      need.push_back({at_seg, items});
      split = split || items > 1;
      wanted += items;
    }
    // A tensor that does not fill the chip's wavefronts with full items gets shorter ones, as many as there
    // are wavefronts: the longest chain of row loads decides then.  (Not where no slice has to be split: the
    // launch that adds up the parts would cost more; nor below 1024 items, which four wavefronts share
    // each.)  697 x 254 x 2633 of 466 K, R = 128: 26.1 -> 22.3 us;
    // skewed 16640 x 2080 x 2377 of 532 K, R = 32: 24.7 -> 20.4 us; items of 128 rows are slower again.
    const int64_t cost_max = split && wanted >= 1024 ? std::max<int64_t>(192, (nnz + h->n_seg) / 7168) : kItemNnz + kItemSegs;
    int64_t s = 0, slots = 0;
    size_t slice = 0;
    for (int64_t i = 0; i < I; ++i) {
      const size_t first_item = item_dst.size();
      if (s >= h->n_seg || seg_i[s] != i) {          // empty slice: one item without segments
        item_seg.push_back((uint32_t)s);
        item_dst.push_back((int32_t)i);
        continue;
      }
      const int64_t end = need[slice].first, cost = (int64_t)(seg_ptr[end] - seg_ptr[s]) + (end - s);
      const int64_t items = std::max(need[slice].second, (cost + cost_max - 1) / cost_max);
      const int64_t share = (cost + items - 1) / items;
      ++slice;
      while (s < end) {
        item_seg.push_back((uint32_t)s);
        item_dst.push_back((int32_t)i);
        for (int64_t cnt = 0, segs = 0; cnt + segs < share && fits(s, cnt, segs); ++segs, ++s) cnt += seg_ptr[s + 1] - seg_ptr[s];
      }
      const size_t n_it = item_dst.size() - first_item;
      if (n_it > 1) {                                  // split slice: consecutive partial slots
        for (size_t t = 0; t < n_it; ++t) item_dst[first_item + t] = (int32_t)(-1 - (slots + (int64_t)t));
        slots += (int64_t)n_it;
        split_ptr.push_back((uint32_t)slots);
        split_y.push_back((int32_t)i);
      }
    }
    item_seg.push_back((uint32_t)h->n_seg);
    // the kernel stages an item in fixed-size LDS arrays: make sure no item exceeds them
    for (size_t t = 0; t + 1 < item_seg.size(); ++t) {
      const int64_t segs = (int64_t)item_seg[t + 1] - (int64_t)item_seg[t];
      const int64_t ents = (int64_t)seg_ptr[item_seg[t + 1]] - (int64_t)seg_ptr[item_seg[t]];
      h->longest = std::max(h->longest, segs + ents);
      if (segs < 0 || segs > kItemSegs || ents < 0 || ents > kItemNnz) {
        return fail3(ARROW_EINTERNAL, "work item %zu holds %lld segments / %lld entries", t, (long long)segs, (long long)ents);
      }
    }
    if (slots > 0x7fffffffLL || item_dst.size() > 0x7fffff00ULL) return fail3(ARROW_EINVAL, "too many work items");
    h->n_items = (int64_t)item_dst.size();
    h->n_split = (int64_t)split_y.size();
    h->n_partials = slots;
    size_t total = 0;
    h->off_seg_ptr = total;   total = align3(total + sizeof(uint32_t) * seg_ptr.size());
    h->off_seg_j = total;     total = align3(total + sizeof(int32_t) * seg_j.size());
    h->off_item_seg = total;  total = align3(total + sizeof(uint32_t) * item_seg.size());
    h->off_item_dst = total;  total = align3(total + sizeof(int32_t) * item_dst.size());
    h->off_item_ent = total;  total = align3(total + sizeof(uint32_t) * item_seg.size());
    h->off_split_ptr = total; total = align3(total + sizeof(uint32_t) * split_ptr.size());
    h->off_split_y = total;   total = align3(total + sizeof(int32_t) * split_y.size());
    h->off_entries = total;   total = align3(total + sizeof(arrow::Entry) * (size_t)nnz);
    h->bytes.assign(total, 0);
    unsigned char* base = h->bytes.data();
    std::memcpy(base + h->off_item_seg, item_seg.data(), sizeof(uint32_t) * item_seg.size());
    std::memcpy(base + h->off_item_dst, item_dst.data(), sizeof(int32_t) * item_dst.size());
    {
      uint32_t* item_ent = reinterpret_cast<uint32_t*>(base + h->off_item_ent);
      for (size_t t = 0; t < item_seg.size(); ++t) item_ent[t] = seg_ptr[item_seg[t]];
    }
    std::memcpy(base + h->off_split_ptr, split_ptr.data(), sizeof(uint32_t) * split_ptr.size());
    if (!split_y.empty()) std::memcpy(base + h->off_split_y, split_y.data(), sizeof(int32_t) * split_y.size());
    // Inside every item the segments are ordered by length, longest first (equal ones by j), so that the
    // lane groups of the wavefront that owns it work on equally long ones; the entries move along.  Items
    // whose segments are in that order already, as where nearly all of them hold one entry, are copied as
    // they are.  (A second pass over all segments that sorted the lengths and kept where each came from: 16 M
    // segments of one entry 0.56 s with eight threads, so 0.45, without any order 0.43.)
    uint32_t* img_ptr = reinterpret_cast<uint32_t*>(base + h->off_seg_ptr);
    int32_t* img_j = reinterpret_cast<int32_t*>(base + h->off_seg_j);
    arrow::Entry* ent = reinterpret_cast<arrow::Entry*>(base + h->off_entries);
    img_ptr[h->n_seg] = (uint32_t)nnz;
    const int64_t n_it = h->n_items;
#pragma omp parallel for schedule(static)
    for (int64_t it = 0; it < n_it; ++it) {                     // (nothing in here may throw)
      const uint32_t s0 = item_seg[it], n_s = item_seg[it + 1] - s0;
      const uint32_t* ptr = seg_ptr.data() + s0;
      auto length = [&](uint32_t q) { return ptr[q + 1] - ptr[q]; };
      std::array<uint8_t, kItemSegs> order;
      bool ordered = true;
      for (uint32_t q = 1; q < n_s; ++q) ordered = ordered && length(q - 1) >= length(q);
      if (!ordered) {
        std::array<uint32_t, kSegMax + 2> at_len{};             // where the segments of a length begin
        for (uint32_t q = 0; q < n_s; ++q) ++at_len[(size_t)(kSegMax - length(q)) + 1];
        for (size_t q = 1; q < at_len.size(); ++q) at_len[q] += at_len[q - 1];
        for (uint32_t q = 0; q < n_s; ++q) order[at_len[(size_t)(kSegMax - length(q))]++] = (uint8_t)q;
      }
      uint32_t e = ptr[0];                                      // the item's entry range stays where it is
      for (uint32_t q = 0; q < n_s; ++q) {
        const uint32_t from = ordered ? q : order[q];
        img_ptr[s0 + q] = e;
        img_j[s0 + q] = seg_j[s0 + from];
        for (uint32_t p = ptr[from]; p < ptr[from + 1]; ++p, ++e) {
          const int64_t src = at(p);
          ent[e].xrow = tk[src];
          ent[e].val = tv[src];
        }
      }
    }
    h->build_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    *out = h.release();
    return ARROW_OK;
  } catch (const std::bad_alloc&) {
    return fail3(ARROW_ENOMEM, "out of host memory while building the fibre image");
  }
}

size_t csf3_device_bytes(const csf3_handle* h) { return h ? h->bytes.size() : 0; }

int csf3_upload(csf3_handle* h, void* dev_buf, size_t bytes, void* stream) {
  if (!h) return fail3(ARROW_EINVAL, "handle is NULL");
  if (!dev_buf) return fail3(ARROW_EINVAL, "dev_buf is NULL");
  if ((uintptr_t)dev_buf % kAlign3) return fail3(ARROW_EINVAL, "dev_buf must be 256-byte aligned");
  if (bytes < h->bytes.size()) return fail3(ARROW_ETOOSMALL, "image needs %zu bytes, buffer has %zu", h->bytes.size(), bytes);
  if (!h->bytes.empty()) {
    hipError_t e = hipMemcpyAsync(dev_buf, h->bytes.data(), h->bytes.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e != hipSuccess) return fail3(ARROW_EHIP, "image upload: %s", hipGetErrorString(e));
  }
  h->dev = static_cast<unsigned char*>(dev_buf);
  return ARROW_OK;
}

size_t csf3_workspace_bytes(const csf3_handle* h, int32_t R) {
  if (!h || R < 1) return 0;
  return partial_bytes(*h, R) + (arrow::stream_lines(R) ? 0 : laid_out_bytes(*h, R)) + kAlign3;
}

int csf3_set_workspace(csf3_handle* h, void* dev_ws, size_t bytes) {
  if (!h) return fail3(ARROW_EINVAL, "handle is NULL");
  if (!dev_ws) return fail3(ARROW_EINVAL, "dev_ws is NULL");
  if ((uintptr_t)dev_ws % kAlign3) return fail3(ARROW_EINVAL, "dev_ws must be 256-byte aligned");
  h->ws = static_cast<unsigned char*>(dev_ws);
  h->ws_bytes = bytes;
  return ARROW_OK;
}

int csf3_mttkrp(csf3_handle* h, const float* B, const float* C, float* A, int32_t R, void* stream) {
  if (!h) return fail3(ARROW_EINVAL, "handle is NULL");
  if (R < 1) return fail3(ARROW_EINVAL, "R must be >= 1 (got %d)", R);
  if (!h->dev) return fail3(ARROW_ENOTREADY, "csf3_upload has not been called");
  if (!h->ws) return fail3(ARROW_ENOTREADY, "csf3_set_workspace has not been called");
  if (h->ws_bytes < partial_bytes(*h, R) + kAlign3)
    return fail3(ARROW_ETOOSMALL, "workspace holds %zu bytes, R = %d needs %zu", h->ws_bytes, R, partial_bytes(*h, R) + kAlign3);
  if (!B || !C || !A) return fail3(ARROW_EINVAL, "B, C or A is NULL");
  if (A == B || A == C) return fail3(ARROW_EINVAL, "A must not overlap B or C");
  if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) % 16) return fail3(ARROW_EINVAL, "A, B and C must be 16-byte aligned");
  float* partials = reinterpret_cast<float*>(h->ws);
  // Where the workspace has room for it, also at ranks that need it only for a factor which does not begin at a line.
  const size_t laid_out = laid_out_bytes(*h, R);
  const bool room = laid_out > 0 && h->ws_bytes >= partial_bytes(*h, R) + laid_out;
  float* scratch = room ? reinterpret_cast<float*>(h->ws + partial_bytes(*h, R)) : nullptr;
  auto at = [&](size_t off) { return h->dev + off; };
  const bool prof = h->profiling && h->ev[0];
  if (prof) (void)hipEventRecord(h->ev[0], (hipStream_t)stream);
  int rc;
  if (h->resident)
    rc = arrow::launch_mttkrp_resident(reinterpret_cast<const arrow::ResidentItem*>(at(h->off_items)),
                                       reinterpret_cast<const arrow::ResidentBlock*>(at(h->off_entries)), h->n_items,
                                       h->n_blocks, B, h->J, C, h->K, A, partials, R, stream,
                                       reinterpret_cast<const uint32_t*>(at(h->off_last)));
  else if (h->streams)
    rc = arrow::launch_mttkrp_streams(reinterpret_cast<const arrow::StreamWave*>(at(h->off_waves)),
                                      reinterpret_cast<const arrow::StreamBlock*>(at(h->off_entries)),
                                      reinterpret_cast<const int32_t*>(at(h->off_dst)),
                                      reinterpret_cast<const int32_t*>(at(h->off_zero)), h->n_waves, B, h->J, C, h->K, A,
                                      partials, scratch, R, stream);
  else
    rc = arrow::launch_mttkrp(reinterpret_cast<const uint32_t*>(at(h->off_item_seg)),
                              reinterpret_cast<const uint32_t*>(at(h->off_item_ent)),
                              reinterpret_cast<const int32_t*>(at(h->off_item_dst)),
                              reinterpret_cast<const uint32_t*>(at(h->off_seg_ptr)),
                              reinterpret_cast<const int32_t*>(at(h->off_seg_j)),
                              reinterpret_cast<const arrow::Entry*>(at(h->off_entries)), h->n_items, B, h->J, C, h->K, A,
                              partials, R, (int32_t)h->longest, (int32_t)((h->nnz + h->n_seg) / h->n_items), stream);
  if (rc) return fail3(ARROW_EHIP, "mttkrp kernel launch: %s", hipGetErrorString((hipError_t)rc));
  if (prof) (void)hipEventRecord(h->ev[1], (hipStream_t)stream);
  rc = arrow::launch_reduce(reinterpret_cast<const uint32_t*>(at(h->off_split_ptr)),
                            reinterpret_cast<const int32_t*>(at(h->off_split_y)), h->n_split, partials, A, R,
                            false, stream);
  if (rc) return fail3(ARROW_EHIP, "reduce kernel launch: %s", hipGetErrorString((hipError_t)rc));
  if (prof) { (void)hipEventRecord(h->ev[2], (hipStream_t)stream); h->profiled = true; }
  return ARROW_OK;
}

int csf3_set_profiling(csf3_handle* h, int32_t enabled) {
  if (!h) return fail3(ARROW_EINVAL, "handle is NULL");
  if (enabled && !h->ev[0]) {
    for (hipEvent_t& e : h->ev)
      if (hipEventCreate(&e) != hipSuccess) { e = nullptr; return fail3(ARROW_EHIP, "event creation failed"); }
  }
  h->profiling = enabled != 0;
  h->profiled = false;
  return ARROW_OK;
}

int csf3_get_profile(csf3_handle* h, float* kernel_ms, float* reduce_ms) {
  if (!h || !kernel_ms || !reduce_ms) return fail3(ARROW_EINVAL, "NULL argument");
  if (!h->profiled) return fail3(ARROW_ENOTREADY, "no profiled product has run");
  hipError_t e = hipEventSynchronize(h->ev[2]);
  if (e == hipSuccess) e = hipEventElapsedTime(kernel_ms, h->ev[0], h->ev[1]);
  if (e == hipSuccess) e = hipEventElapsedTime(reduce_ms, h->ev[1], h->ev[2]);
  if (e != hipSuccess) return fail3(ARROW_EHIP, "event timing: %s", hipGetErrorString(e));
  return ARROW_OK;
}

int csf3_info(const csf3_handle* h, csf3_info_t* out) {
  if (!h || !out) return fail3(ARROW_EINVAL, "NULL argument");
  out->I = h->I; out->J = h->J; out->K = h->K; out->nnz = h->nnz;
  out->slices = h->slices; out->fibers = h->fibers; out->segments = h->n_seg; out->items = h->n_items;
  out->split_rows = h->n_split; out->partials = h->n_partials;
  out->distinct_j = h->distinct_j; out->distinct_k = h->distinct_k;
  out->build_seconds = h->build_seconds;
  return ARROW_OK;
}

int csf3_form(const csf3_handle* h) {
  if (!h) return fail3(ARROW_EINVAL, "handle is NULL");
  return h->resident ? CSF3_FORM_FACTORS_IN_LDS : h->streams ? CSF3_FORM_SUMS_IN_LDS : CSF3_FORM_ITEMS;
}

void csf3_destroy(csf3_handle* h) {
  if (!h) return;
  for (hipEvent_t e : h->ev)
    if (e) (void)hipEventDestroy(e);
  delete h;
}

}  // extern "C"
