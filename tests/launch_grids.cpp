// Launches of the library recorded instead of made: HIP takes a grid dimension of fewer than 2^32 work items, and
// operands that a card has room for must not be refused for the shape of a grid.  No device memory is touched, so the
// pointers are made up.  `launch_grids <case>`; exit status 0 = accepted, and the grid holds all of the work.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "arrow.h"
#include "arrow_internal.h"

namespace {

struct Launch { dim3 grid, block; uint64_t groups() const { return (uint64_t)grid.x * grid.y * grid.z; } };
std::vector<Launch>& launches() { static std::vector<Launch> l; return l; }
hipError_t last = hipSuccess;
dim3 pushed_grid, pushed_block;

}  // namespace

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) { pushed_grid = grid; pushed_block = block; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = pushed_grid; *block = pushed_block; *shared = 0; *stream = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  launches().push_back({grid, block});
  const uint64_t items[3] = {(uint64_t)grid.x * block.x, (uint64_t)grid.y * block.y, (uint64_t)grid.z * block.z};
  bool fits = grid.x > 0 && grid.y > 0 && grid.z > 0 && grid.y < 65536 && grid.z < 65536;
  for (uint64_t n : items) fits = fits && n < 1ull << 32;
  last = fits ? hipSuccess : hipErrorInvalidConfiguration;
  return last;
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int*) { return hipErrorNoDevice; }
}

namespace {

float* address(int which) { return reinterpret_cast<float*>((uintptr_t)(which + 1) << 44); }

// Chunks of long rows in window order, `slices` of them.
int chunks(int64_t n, int32_t k, int32_t kc, int64_t n_chunks, uint64_t slices) {
  arrow::ProductArgs a{};
  a.X = a.Xh = address(0); a.Y = address(1); a.partials = address(2);
  a.n_chunks = n_chunks; a.k = k;
  const int rc = arrow::launch_product(a, arrow::kPartChunks, 0, 0, 0, false, true, n, kc, nullptr);
  std::printf("rc %d, %zu launches, %u x %u groups\n", rc, launches().size(), launches()[0].grid.x, launches()[0].grid.y);
  return rc == 0 && launches().size() == 1 && launches()[0].groups() * arrow::kChunksPerGroup >= (uint64_t)n_chunks * slices ? 0 : 1;
}

// Pieces of long rows and short rows of a product in row order, four lane groups to a wavefront: `groups` workgroups.
int product_pieces(int64_t n_pieces, int64_t n_short, uint32_t groups) {
  arrow::ProductArgs a{};
  a.X = a.Xh = address(0); a.Y = address(1); a.partials = address(2);
  a.k = 64;
  const int rc = arrow::launch_product(a, arrow::kPartAll, n_pieces, n_pieces + n_short, 0, false, false, 100000, 0, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].grid.x == groups ? 0 : 1;
}

// A product in row order whose rows have so many columns that slices of 64 for all of its parts are too many for one grid.
int short_rows() {
  const int64_t n = 32768;
  const int32_t k = 1 << 19;
  std::vector<int64_t> ptr(n + 1, 0);
  std::vector<int32_t> col;
  for (int64_t i = 0; i < n; ++i) {
    const int64_t entries = i < 64 ? 2048 : 3;
    for (int64_t e = 0; e < entries; ++e) col.push_back((int32_t)((e * (n / entries) + i) % (n / entries) + e * (n / entries)));
    ptr[i + 1] = (int64_t)col.size();
  }
  const std::vector<float> val(col.size(), 1.f);
  arrow_handle* h = nullptr;
  int rc = arrow_decompose(n, ptr.data(), col.data(), val.data(), 1024, &h);
  if (rc == 0) rc = arrow_upload(h, address(0), arrow_device_bytes(h), nullptr);
  if (rc == 0) rc = arrow_set_workspace(h, address(1), arrow_workspace_bytes(h, k));
  if (rc == 0) rc = arrow_spmm(h, address(2), address(3), k, nullptr);
  std::printf("rc %d (%s)\n", rc, arrow_last_error());
  for (const Launch& l : launches()) std::printf("%u x %u groups\n", l.grid.x, l.grid.y);
  arrow_destroy(h);
  return rc == 0 ? 0 : 1;
}

// Rows of dense blocks of a sampled product: `groups` workgroups, if given.
int window_rows(int64_t n, int32_t k, int64_t nnz = 0, uint32_t groups = 0) {
  arrow::SampledArgs a{};
  a.U = address(0); a.V = a.Vh = address(1); a.S = address(2);
  a.n_rows = n; a.nnz_rows = nnz; a.k = k;
  const int rc = arrow::launch_sddmm(a, true, false, true, false, n, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].groups() * arrow::kItemsPerGroupBlock >= (uint64_t)n &&
         (groups == 0 || launches()[0].grid.x == groups) ? 0 : 1;
}

// Rows of a sampled product that are all alike, five entries each: `groups` workgroups.
int equal_rows(int64_t n, int32_t k, uint32_t groups) {
  arrow::SampledArgs a{};
  a.U = address(0); a.V = a.Vh = address(1); a.S = address(2);
  a.n_rows = n; a.nnz_rows = 5 * n; a.k = k;
  const int rc = arrow::launch_sddmm(a, false, false, false, false, n, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].grid.x == groups ? 0 : 1;
}

// Rows of a sampled product that are not all short, `groups` workgroups of them, behind some chunks.
int unequal_rows(int64_t n, int64_t nnz, int32_t k, uint32_t groups, int64_t n_chunks) {
  arrow::SampledArgs a{};
  a.U = address(0); a.V = a.Vh = address(1); a.S = address(2);
  a.n_rows = n; a.nnz_rows = nnz; a.n_chunks = n_chunks; a.nnz_chunks = 50 * n_chunks; a.k = k;
  const int rc = arrow::launch_sddmm(a, false, false, false, true, n, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].grid.x == groups ? 0 : 1;
}

// Pieces of long rows of a sampled product before its short rows, eight entries each: `groups` workgroups.
int pieces(int64_t n_pieces, int64_t n_short, int32_t k, bool windows, uint32_t groups) {
  arrow::SampledArgs a{};
  a.U = address(0); a.V = a.Vh = address(1); a.S = address(2);
  a.n_rows = n_pieces + n_short; a.n_pieces = n_pieces; a.nnz_rows = 8 * a.n_rows; a.k = k;
  const int rc = arrow::launch_sddmm(a, false, false, windows, true, a.n_rows, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].grid.x == groups ? 0 : 1;
}

// Pieces and short rows in window order that one grid holds with workgroups for both, but not with workgroups of their own.
int pieces_apart(int64_t n_pieces, int64_t n_short, int32_t k) {
  arrow::SampledArgs a{};
  a.U = address(0); a.V = a.Vh = address(1); a.S = address(2);
  a.n_rows = n_pieces + n_short; a.n_pieces = n_pieces; a.nnz_rows = 8 * a.n_rows; a.k = k;
  const int rc = arrow::launch_sddmm(a, false, false, true, true, a.n_rows, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].groups() * arrow::kItemsPerGroupBlock >= (uint64_t)a.n_rows ? 0 : 1;
}

// Chunks of long rows of a sampled product, in row order: `groups` workgroups of four wavefronts.
int sampled_chunks(int64_t n_chunks, int64_t nnz, int32_t k, uint32_t groups) {
  arrow::SampledArgs a{};
  a.U = address(0); a.V = a.Vh = address(1); a.S = address(2);
  a.n_chunks = n_chunks; a.nnz_chunks = nnz; a.k = k;
  const int rc = arrow::launch_sddmm(a, false, false, false, false, 20000, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].grid.x == groups ? 0 : 1;
}

// The order-3 product with the factors in LDS, 2000 items of 2.75 blocks: `slices` of columns with `replicas` workgroups each.
int factors_in_lds(int32_t R, uint32_t slices, uint32_t replicas) {
  const int rc = arrow::launch_mttkrp_resident(nullptr, nullptr, 2000, 5500, address(0), 1000, address(1), 1000, address(2), address(3), R, nullptr);
  std::printf("rc %d, %zu launches, %u groups\n", rc, launches().size(), launches()[0].grid.x);
  return rc == 0 && launches().size() == 1 && launches()[0].grid.x == (slices * replicas + 7) / 8 * 8 ? 0 : 1;
}

}  // namespace

int main(int, char** argv) {
  const std::string c = argv[1];
  if (c == "chunks") return chunks(8 << 20, 1024, 64, 4400000, 16);
  if (c == "chunks in narrow slices") return chunks(8 << 20, 512, 32, 4400000, 16);
  if (c == "chunks, two sets of dies") return chunks(1 << 20, 128, 64, 16000000, 2);
  if (c == "short rows") return short_rows();
  // a wavefront to a piece up to 1024 workgroups, sixteen pieces to a workgroup beyond, a wavefront again from 1537 to 4000
  if (c == "pieces of a product, four workgroups a unit") return product_pieces(2000, 8320, 1024);
  if (c == "pieces of a product, a row more") return product_pieces(2000, 8321, 128 + 528);
  if (c == "pieces of a product, six and more") return product_pieces(4000, 8600, 1000 + 544);
  if (c == "pieces of a product, too many") return product_pieces(13000, 12000, 816 + 752);
  if (c == "window rows") return window_rows(80000000, 128);
  // one round of 1536 workgroups of eight rows, then half as many rows each, then eight again; shorter rows eight always
  if (c == "window rows, one round") return window_rows(12288, 128, 12288 * 50, 1536);
  if (c == "window rows, a row more") return window_rows(12289, 128, 12289 * 50, 3080);
  if (c == "window rows, three fifths more") return window_rows(19661, 128, 19661 * 50, 2464);
  if (c == "window rows, short") return window_rows(12289, 128, 12289 * 39, 1544);
  // one round of 1792 workgroups, then two rather than one and a little, then what 64 items give
  if (c == "equal rows, one round") return equal_rows(114688, 64, 1792);
  if (c == "equal rows, a row more") return equal_rows(114689, 64, 3592);
  if (c == "equal rows, two fifths more") return equal_rows(160600, 64, 2512);
  if (c == "equal rows, the widest") return equal_rows(250000, 192, 7816);
  // two of the widest to a workgroup behind chunks (32 of these, which 16 wavefronts share), or four where they are many, shorter or alone
  if (c == "unequal rows, long") return unequal_rows(6000, 6000 * 45, 200, 128 + 3000, 32);
  if (c == "unequal rows, many") return unequal_rows(6800, 6800 * 45, 200, 128 + 1704, 32);
  if (c == "unequal rows, short") return unequal_rows(16000, 16000 * 8, 200, 128 + 4000, 32);
  if (c == "unequal rows, alone") return unequal_rows(6000, 6000 * 45, 200, 1504, 0);
  // eight pieces and 32 short rows to a workgroup; eight of both where pieces are more than half; in window order 16 and 64, or 32 of both in wide rows
  if (c == "pieces, fewer") return pieces(3000, 20000, 24, false, 376 + 632);
  if (c == "pieces, more") return pieces(7000, 6000, 24, false, 1632);
  if (c == "pieces, in window order") return pieces(9000, 300000, 24, true, 568 + 4688);
  if (c == "pieces, in window order, wide") return pieces(9000, 300000, 64, true, 9664);
  if (c == "pieces and short rows, many") return pieces_apart(200000000, 280000000, 8);
  if (c == "pieces and short rows, most") return pieces_apart(240000000, 700000000, 24);
  // a wavefront each, or two where chunks are more than a strip, or four where they leave the chip half empty
  if (c == "chunks of a strip") return sampled_chunks(5000, 5000 * 64, 200, 1256);
  if (c == "chunks of a strip and more") return sampled_chunks(5000, 5000 * 64 + 1, 200, 2504);
  if (c == "chunks of a strip, few") return sampled_chunks(2000, 2000 * 56, 200, 2000);
  // beyond 1024 slices of four columns: four columns, or eight where those take fewer rounds of workgroups
  if (c == "factors in LDS, 4096 columns") return factors_in_lds(4096, 512, 1);
  if (c == "factors in LDS, 5120 columns") return factors_in_lds(5120, 1280, 1);
  if (c == "factors in LDS, 6144 columns") return factors_in_lds(6144, 768, 1);
  if (c == "factors in LDS, 9000 columns") return factors_in_lds(9000, 1125, 1);
  return 2;
}
