// What the library's calls hand to their kernels: the launches are recorded instead of made, by name and with the arguments that the
// cases below look at.  No device memory is touched, so the pointers are made up.  `launch_arguments <case>`; exit status 0 = as it has to be.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

#include "arrow.h"
#include "arrow_internal.h"

namespace {

struct Launch {
  std::string kernel;
  dim3 grid;
  arrow::ProductArgs product;      // of a kernel that takes one
  arrow::SampledArgs sampled;      // of a kernel that takes one
  const unsigned char* head;       // of gather_kernel: its result, rows of it, and the floats between those
  int64_t rows;
  int stride;
};
std::vector<Launch>& launches() { static std::vector<Launch> l; return l; }
std::map<const void*, std::string>& names() { static std::map<const void*, std::string> n; return n; }
dim3 pushed_grid, pushed_block;

}  // namespace

extern "C" {
void __hipRegisterFunction(void**, const void* function, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) { names()[function] = name; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) { pushed_grid = grid; pushed_block = block; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = pushed_grid; *block = pushed_block; *shared = 0; *stream = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* function, dim3 grid, dim3, void** args, size_t, hipStream_t) {
  Launch l{};
  l.kernel = names()[function];
  l.grid = grid;
  if (l.kernel.find("ProductArgs") != std::string::npos) l.product = *static_cast<const arrow::ProductArgs*>(args[0]);
  if (l.kernel.find("SampledArgs") != std::string::npos) l.sampled = *static_cast<const arrow::SampledArgs*>(args[0]);
  if (l.kernel.find("13gather_kernel") != std::string::npos) {
    l.rows = *static_cast<const int64_t*>(args[1]);
    l.head = *static_cast<unsigned char* const*>(args[3]);
    l.stride = *static_cast<const int*>(args[5]);
  }
  launches().push_back(l);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int*) { return hipErrorNoDevice; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorNoDevice; }
}

namespace {

unsigned char* address(int which) { return reinterpret_cast<unsigned char*>((uintptr_t)(which + 1) << 44); }
float* floats(int which) { return reinterpret_cast<float*>(address(which)); }
size_t up(size_t bytes) { return (bytes + 255) / 256 * 256; }
bool disjoint(const unsigned char* a, size_t a_bytes, const unsigned char* b, size_t b_bytes) { return a + a_bytes <= b || b + b_bytes <= a; }

uint64_t state = 1;
uint32_t below(uint32_t n) { state = state * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)((state >> 33) % n); }

// An operand with the given number of entries in every row.
arrow_handle* operand(const std::vector<int>& entries, uint32_t columns, int32_t b, const arrow_options_t& options) {
  const int64_t n = (int64_t)entries.size();
  std::vector<int64_t> ptr(1, 0);
  std::vector<int32_t> col;
  for (int m : entries) {
    std::vector<int32_t> row;
    while ((int)row.size() < m) {
      row.push_back((int32_t)below(columns));
      std::sort(row.begin(), row.end());
      row.erase(std::unique(row.begin(), row.end()), row.end());
    }
    col.insert(col.end(), row.begin(), row.end());
    ptr.push_back((int64_t)col.size());
  }
  const std::vector<float> val(col.size(), 1.f);
  arrow_handle* h = nullptr;
  if (arrow_decompose_with(n, ptr.data(), col.data(), val.data(), b, &options, &h) != 0) std::printf("%s\n", arrow_last_error());
  return h;
}

// An operand whose head is staged, and the least workspace of a product with it.
constexpr int64_t kRows = 4096;
arrow_handle* staged_operand() {
  arrow_options_t o;
  arrow_options_default(&o);
  o.stage_short = 1; o.window_rows = 1024;
  std::vector<int> entries(kRows);
  for (int& m : entries) m = 4 + (int)below(30);
  arrow_handle* h = operand(entries, kRows, 512, o);
  if (h && (arrow_upload(h, address(0), arrow_device_bytes(h), nullptr) || arrow_sddmm_upload(h, address(1), arrow_sddmm_device_bytes(h), nullptr))) return nullptr;
  return h;
}
size_t least_workspace(arrow_handle* h, int32_t k) {
  size_t low = 0, least = arrow_workspace_bytes(h, k) / 256;
  while (least - low > 1) {
    const size_t m = (low + least) / 2;
    arrow_set_workspace(h, address(2), 256 * m);
    if (arrow_spmm(h, floats(3), floats(4), k, nullptr) == 0) least = m; else low = m;
  }
  launches().clear();
  return 256 * least;
}

// Every call that stages a head; each has to leave [kept, kept + bytes) alone.  `whole`: counts the heads laid out in whole lines.
bool leaves_alone(arrow_handle* h, int32_t k, const unsigned char* kept, size_t bytes, int* whole) {
  launches().clear();
  int rc = arrow_spmm(h, floats(3), floats(4), k, nullptr);
  if (rc == 0) rc = arrow_sddmm(h, floats(3), floats(4), floats(5), k, nullptr);
  if (rc) { std::printf("rc %d (%s)\n", rc, arrow_last_error()); return false; }
  int heads = 0;
  for (const Launch& l : launches()) {
    if (!l.head) continue;
    ++heads;
    if (l.stride > k) ++*whole;
    if (!disjoint(l.head, (size_t)l.rows * (size_t)l.stride * 4, kept, bytes)) { std::printf("a head over what is kept, %d floats a row\n", l.stride); return false; }
  }
  return heads == 2;
}

// The head in whole lines lies where only the workspace asked for it, whatever else a caller keeps in a workspace larger than the least.
int buffers_in_the_workspace() {
  arrow_handle* h = staged_operand();
  if (!h) return 1;
  int whole = 0;
  for (int32_t k : {17, 50, 63, 127}) {
    const size_t least = least_workspace(h, k), xy = up((size_t)kRows * (size_t)k * 4), full = arrow_workspace_bytes(h, k);
    unsigned char* ws = address(2);
    if (least != up(arrow_scratch_bytes(h, k))) return 1;
    // an operand of another call in the part that only chained products write
    arrow_set_workspace(h, ws, full);
    if (!leaves_alone(h, k, ws + least, xy, &whole) || whole == 0) return 1;
    const size_t map = arrow_sddmm_device_bytes(h), image = arrow_device_bytes(h);
    for (size_t at : {least, least + xy / 2 / 256 * 256, least + xy, full - 256, full}) {
      arrow_set_workspace(h, ws, full + std::max(map, image));
      arrow_sddmm_upload(h, ws + at, map, nullptr);
      if (!leaves_alone(h, k, ws + at, map, &whole)) { std::printf("entry map, k = %d\n", k); return 1; }
      arrow_sddmm_upload(h, address(1), map, nullptr);
      if (at < least + xy) continue;             // (products are refused where Y overlaps the image, chained ones write all before)
      arrow_upload(h, ws + at, image, nullptr);
      if (!leaves_alone(h, k, ws + at, image, &whole)) { std::printf("image, k = %d\n", k); return 1; }
      arrow_upload(h, address(0), image, nullptr);
    }
  }
  arrow_destroy(h);
  return 0;
}

// A workspace asked for `most` columns: with k columns the head is laid out in whole lines, as in one asked for k.
int fewer_columns(int32_t most, int32_t k) {
  arrow_handle* h = staged_operand();
  if (!h) return 1;
  for (int32_t asked : {k, most}) {
    arrow_set_workspace(h, address(2), arrow_workspace_bytes(h, asked));
    launches().clear();
    int rc = arrow_spmm(h, floats(3), floats(4), k, nullptr);
    if (rc == 0) rc = arrow_sddmm(h, floats(3), floats(4), floats(5), k, nullptr);
    if (rc == 0) rc = arrow_spmm_iter(h, floats(3), k, 2, nullptr);
    int heads = 0, whole = 0;
    for (const Launch& l : launches())
      if (l.head) { ++heads; whole += l.stride % 32 == 0; }
    std::printf("rc %d, asked for %d columns: %d of %d heads in whole lines\n", rc, asked, whole, heads);
    if (rc || heads != 4 || whole != heads) return 1;
  }
  arrow_destroy(h);
  return 0;
}

// Whether the heads of a product and of a sampled product with k columns are in rows of whole lines where there is room, `columns` floats apart.
int head_rows(int32_t k, int columns) {
  arrow_handle* h = staged_operand();
  if (!h) return 1;
  const size_t full = arrow_workspace_bytes(h, k), least = up(arrow_scratch_bytes(h, k));
  for (size_t bytes : {full, least}) {
    arrow_set_workspace(h, address(2), bytes);
    launches().clear();
    int rc = arrow_spmm(h, floats(3), floats(4), k, nullptr);
    if (rc == 0) rc = arrow_sddmm(h, floats(3), floats(4), floats(5), k, nullptr);
    int heads = 0;
    for (const Launch& l : launches()) {
      if (!l.head) continue;
      std::printf("%d columns, rows %d apart\n", k, l.stride);
      if (l.stride != (bytes == full ? columns : k) || l.head < address(2) || l.head + (size_t)l.rows * (size_t)l.stride * 4 > address(2) + bytes) return 1;
      ++heads;
    }
    bool read = false;
    for (const Launch& l : launches()) read = read || l.product.head_stride == (bytes == full ? columns : k);
    if (rc || heads != 2 || !read) return 1;
  }
  arrow_destroy(h);
  return 0;
}

// Pieces of long rows, short rows and rows of several chunks of a product: the launch that holds the pieces gives them the same
// wavefronts and workgroups where the product is profiled, which launches the lists apart.
int profiled(int64_t n, int pieces, int shorts, int longs, int32_t k, bool wave) {
  std::vector<int> entries((size_t)n, 0);
  for (int64_t i = 0; i < pieces + shorts + longs; ++i) entries[(size_t)i] = i < pieces ? 17 + (int)below(31) : i < pieces + shorts ? 1 + (int)below(15) : 700;
  arrow_options_t o;
  arrow_options_default(&o);
  arrow_handle* h = operand(entries, (uint32_t)n, (int32_t)(n / 16), o);
  if (!h || arrow_upload(h, address(0), arrow_device_bytes(h), nullptr)) return 1;
  arrow_set_workspace(h, address(2), (size_t)1 << 40);
  arrow::ProductArgs seen[2] = {};
  for (int p = 0; p < 2; ++p) {
    launches().clear();
    if (arrow_set_profiling(h, p) || arrow_spmm(h, floats(3), floats(4), k, nullptr)) { std::printf("%s\n", arrow_last_error()); return 1; }
    for (const Launch& l : launches())
      if (l.product.count[1] > 0) seen[p] = l.product;
  }
  arrow_destroy(h);
  for (const arrow::ProductArgs& a : seen)
    std::printf("%lld pieces, %d to a workgroup, a wavefront each: %d\n", (long long)a.count[1], a.items[1], a.piece_waves);
  return seen[0].count[1] >= pieces && seen[0].count[1] == seen[1].count[1] && seen[0].piece_waves == (wave ? 1 : 0) && seen[1].piece_waves == seen[0].piece_waves &&
         seen[1].items[1] == seen[0].items[1] ? 0 : 1;
}

// A sampled product of long and short rows in window order: `items` of them to a workgroup, which go by the rows that have entries.
int sampled_items(int64_t n, int pieces, int shorts, int32_t k, int items) {
  std::vector<int> entries((size_t)n, 0);
  for (int i = 0; i < pieces + shorts; ++i) entries[(size_t)i] = i < pieces ? 20 : 2;
  arrow_options_t o;
  arrow_options_default(&o);
  arrow_handle* h = operand(entries, (uint32_t)n, (int32_t)(n / 16), o);
  if (!h || arrow_upload(h, address(0), arrow_device_bytes(h), nullptr) || arrow_sddmm_upload(h, address(1), arrow_sddmm_device_bytes(h), nullptr)) return 1;
  arrow_set_workspace(h, address(2), (size_t)1 << 40);
  if (arrow_sddmm(h, floats(3), floats(4), floats(5), k, nullptr)) { std::printf("%s\n", arrow_last_error()); return 1; }
  int rc = 1;
  for (const Launch& l : launches())
    if (l.sampled.n_rows > 0) {
      std::printf("%lld rows, %lld pieces apart, %d items to a workgroup\n", (long long)l.sampled.n_rows, (long long)l.sampled.n_pieces, l.sampled.items);
      rc = l.sampled.n_rows >= pieces + shorts && l.sampled.n_rows < n / 2 && l.sampled.n_pieces == 0 && l.sampled.items == items ? 0 : 1;
    }
  arrow_destroy(h);
  return rc;
}

// The order-3 product with the factors in LDS: four or eight columns of them.
int columns(int64_t items, int64_t blocks, int64_t rows, int32_t R, int quads) {
  const uint32_t last = 0;
  const int rc = arrow::launch_mttkrp_resident(nullptr, nullptr, items, blocks, floats(0), rows / 2, floats(1), rows - rows / 2, floats(2), floats(3), R, nullptr, &last);
  std::printf("rc %d, %s\n", rc, launches()[0].kernel.c_str());
  return rc == 0 && launches().size() == 1 && launches()[0].kernel.find("resident_kernelILi" + std::to_string(quads) + "E") != std::string::npos ? 0 : 1;
}

// The workgroups of a wave list in window order, of a product (k columns in slices of kc) and of a sampled one: every one is taken
// once, `run` of them one after the other by the same die, as far as whole runs go.
int runs(int64_t n_chunks, int32_t k, int32_t kc, uint32_t run, uint32_t sets_log) {
  arrow::ProductArgs p{};
  p.X = p.Xh = floats(0); p.Y = floats(1); p.partials = floats(2);
  p.n_chunks = n_chunks; p.k = k;
  arrow::SampledArgs s{};
  s.U = floats(0); s.V = s.Vh = floats(1); s.S = floats(2);
  s.n_chunks = n_chunks; s.nnz_chunks = 100 * n_chunks; s.k = k;
  if (arrow::launch_product(p, arrow::kPartChunks, 0, 0, 0, false, true, 300000, kc, nullptr) || arrow::launch_sddmm(s, false, false, true, false, 300000, nullptr)) return 1;
  if (launches().size() != 2 || launches()[0].product.run != run || launches()[1].sampled.run != run || launches()[0].product.sets_log != sets_log) return 1;
  for (int which = 0; which < 2; ++which) {
    const uint32_t dies_log = 3 - (which == 0 ? sets_log : 0), dies = 1u << dies_log;
    const uint32_t blocks = which == 0 ? launches()[0].product.blocks[0] : launches()[1].grid.x;
    if ((int64_t)blocks * arrow::kChunksPerGroup < n_chunks) return 1;
    std::vector<int> taken(blocks, 0);
    for (uint32_t id = 0; id < blocks; ++id) {
      const uint32_t at = arrow::in_runs(id, dies_log, run, blocks);
      if (at >= blocks || taken[at]++) { std::printf("workgroup %u of %u\n", at, blocks); return 1; }
      const bool whole = id / (dies * run) * dies * run + dies * run <= blocks;
      if (whole && at / run % dies != id % dies) { std::printf("workgroup %u on die %u\n", at, id % dies); return 1; }
    }
  }
  return 0;
}

}  // namespace

int main(int, char** argv) {
  const std::string c = argv[1];
  if (c == "profiled, one launch") return profiled(11000, 2000, 8321, 0, 64, false);
  if (c == "profiled, one launch, a wavefront each") return profiled(11000, 2000, 8320, 0, 64, true);
  if (c == "profiled, seven workgroups a unit") return profiled(15000, 4001, 8601, 0, 50, true);
  if (c == "profiled, slices and chunks") return profiled(11000, 2000, 8321, 40, 200, false);
  if (c == "profiled, two launches") return profiled(140000, 3000, 60000, 20, 96, true);
  if (c == "buffers in the workspace") return buffers_in_the_workspace();
  // the root of 200 K rows times 160 K entries is 179 K; of the 35 K rows with entries alone 75 K
  if (c == "items of a sampled product, 48 columns") return sampled_items(200000, 5000, 30000, 48, 8);
  if (c == "items of a sampled product, 100 columns") return sampled_items(200000, 5000, 30000, 100, 8);
  if (c == "items of a sampled product, 200 columns") return sampled_items(200000, 5000, 30000, 200, 4);
  if (c == "eight columns, 4000 items of 2.5 blocks, rank 128") return columns(4000, 10000, 2000, 128, 2);
  if (c == "four columns, 1018 items of 12 blocks, rank 16") return columns(1018, 12216, 4383, 16, 1);
  if (c == "eight columns, 2000 items of 1.2 blocks, rank 64") return columns(2000, 2444, 1900, 64, 2);
  if (c == "four columns, 2000 items of 1.2 blocks, rank 4") return columns(2000, 2444, 1900, 4, 1);
  if (c == "four columns, 700 items of 10 blocks, rank 100") return columns(700, 6986, 3500, 100, 1);
  if (c == "eight columns, 1403 items of 2 blocks, rank 43") return columns(1403, 2806, 1324, 43, 2);
  if (c == "four columns, 430 items, rank 4742") return columns(430, 480, 2370, 4742, 1);
  if (c == "eight columns, 229 items, rank 6881") return columns(229, 3436, 3356, 6881, 2);
  if (c == "127 columns in a workspace for 128") return fewer_columns(128, 127);
  if (c == "31 columns in a workspace for 32") return fewer_columns(32, 31);
  if (c == "20 columns in a workspace for 25") return fewer_columns(25, 20);
  if (c == "runs of 64, a few workgroups") return runs(20, 128, 128, 64, 0);
  if (c == "runs of 64, the shortest that has one") return runs(4 * 512, 128, 128, 64, 0);
  if (c == "runs of 64, the longest") return runs(4 * 7296, 50, 50, 64, 0);
  if (c == "runs of 128, the shortest") return runs(4 * 7299 + 1, 50, 50, 128, 0);
  if (c == "runs of 128, two sets of dies") return runs(4 * 9592, 128, 64, 128, 1);
  if (c == "runs of 256, the shortest") return runs(4 * 9599 + 1, 50, 50, 256, 0);
  if (c == "runs of 256, two sets of dies") return runs(1000003, 128, 64, 256, 1);
  if (c.rfind("head rows of ", 0) == 0) {
    const int k = std::atoi(c.c_str() + 13);
    const bool whole = k == 17 || k == 20 || k == 63 || k == 90 || k == 127 || k == 150;
    return head_rows(k, whole ? (k + 31) / 32 * 32 : k);
  }
  return 2;
}
