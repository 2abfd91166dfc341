// Internal C++ declarations shared by the host decomposition, the image
// packer / C-ABI and the HIP kernel launchers.  Nothing here is exported.
#pragma once

#include <cstddef>
#include <cstdint>
#include <memory>
#include <string>
#include <utility>
#include <vector>

namespace arrow {

// std::vector whose resize() leaves new elements uninitialised: the entry arrays of a level are
// hundreds of megabytes and are filled by parallel loops right after they are sized, so a serial
// zero-fill (and its page faults) would only cost time.
template <typename T>
struct default_init_allocator : std::allocator<T> {
  template <typename U> struct rebind { using other = default_init_allocator<U>; };
  using std::allocator<T>::allocator;
  template <typename U, typename... Args>
  void construct(U* p, Args&&... args) {
    if constexpr (sizeof...(Args) == 0) ::new (static_cast<void*>(p)) U;
    else ::new (static_cast<void*>(p)) U(std::forward<Args>(args)...);
  }
};
template <typename T> using raw_vector = std::vector<T, default_init_allocator<T>>;

// One arrow matrix B_i in position coordinates, CSR by row position.
struct HostLevel {
  int64_t n_i = 0;                 // active vertices of this level
  std::vector<int32_t> perm;       // position -> original vertex id, n_i entries
  std::vector<int64_t> rowptr;     // n_i + 1
  raw_vector<int32_t> colpos;      // column positions, ascending inside a row
  raw_vector<float> vals;
  raw_vector<uint32_t> src;        // index of every entry in the caller's CSR arrays
  int64_t nnz_head_head = 0, nnz_head_row = 0, nnz_head_col = 0, nnz_diag = 0;
  bool separator_rule = false;
};

struct DecomposeOptions {
  double hub_factor = 8.0;   // a vertex is a hub when its degree exceeds hub_factor * mean degree
  bool separators = true;    // try the block-separator rule before the plain top-degree head
  bool bfs_tail = true;      // levels >= 1 arrange the non-head vertices in BFS order
  bool head_by_id = true;    // plain rule: head vertices in id order (else by falling degree)
  int64_t hubs_first = 0;    // ... after this many of the highest degrees, which lead the head by falling degree
};

// Peels arrow matrices of width b off A until nothing is left.  Returns 0 or a
// negative arrow_status; `err` receives a description on failure.
int decompose(int64_t n, const int64_t* rowptr, const int32_t* colidx, const float* vals,
              int32_t b, const DecomposeOptions& opt, std::vector<HostLevel>& levels,
              std::string& err);

// ---------------------------------------------------------------------------
// Device image.  All offsets are byte offsets from the image base, 256-aligned.
// ---------------------------------------------------------------------------

// Entry of a work list: the row to read (perm already applied, or a staged head row) and the value.
struct Entry {
  int32_t xrow;
  float val;
};

constexpr int kDies = 8;             // MI355X: 8 accelerator dies, workgroups are dealt to them round-robin
constexpr uint32_t kDiesLog = 3;
static_assert(kDies == 1 << kDiesLog, "a power of two of dies");
constexpr int kChunksPerGroup = 4;   // wave-list items (one per wavefront) per workgroup of the chunk kernel
// Destination of a wave-list item whose sum is added to that of its workgroup's first item: the four
// wavefronts of a workgroup then work on one item together (slots 4 i .. 4 i + 3, all or none).
// INT32_MIN marks padding; partial slots end below both.
constexpr int32_t kTeamDst = INT32_MIN + 1;
constexpr int kItemsPerGroupBlock = 64;  // most group-list items per workgroup, and exactly that many of a die queue
constexpr int64_t kMostGroups = (1LL << 24) - 1;   // workgroups of 256 in a dimension of a grid: HIP takes fewer than 2^32 work items
// Consecutive wave-list workgroups that one die takes where the list has no die queues (a power of two): long enough for its L2 to gain, and several of
// them for every die of a short list, whose last ones else go round-robin or leave dies idle.  (On 604 lists of 132 K to 900 K vertices, R-MAT and
// Chung-Lu, at two ranks each: 64 take 0.96 times the time of 256 below 4000 workgroups and 0.99 to 7300, 128 0.99 to 9600, beyond that nothing gains on
// average; us, 256 / 128 / 64: directed 300 K, k = 50, 136.1 / 136.0 / 133.6; Chung-Lu 250 K, 48, 84.3 / 81.0 / 81.5; sampled product, Chung-Lu 400 K, 32, 95.7 /
// 92.5 / 91.2; R-MAT 500 K, 128, 331.6 / 335.6 / 337.8.)
inline uint32_t die_run(int64_t blocks) { return blocks < 7300 ? 64 : blocks < 9600 ? 128 : 256; }
// The workgroup of the wave list that the id-th place is for, of `blocks` places that are dealt to 1 << dies_log dies round-robin: runs of `run` of
// them to one die each, as far as every die has a whole one (run = 0: the id-th).
constexpr uint32_t in_runs(uint32_t id, uint32_t dies_log, uint32_t run, uint32_t blocks) {
  const uint32_t dies = 1u << dies_log, span = dies * run, base = id & ~(span - 1u);
  return run && base + span <= blocks ? base + (id & (dies - 1u)) * run + ((id - base) >> dies_log) : id;
}
// head panels: kPanelRows head rows form a group; the group's head-block entries are dealt by column
// class (staged head row mod kDies) to kDies workgroups, one per accelerator die, each keeping the
// group's accumulators in LDS and streaming its entries in kPanelBins lane-group streams
constexpr int kPanelBins = 32;
constexpr int kPanelRows = 128;
constexpr int kPanelClassShift = 6;       // staged head rows are dealt to the column classes 64 at a time
inline int panel_class(uint32_t staged_row) { return (int)((staged_row >> kPanelClassShift) & (kDies - 1)); }
constexpr int kPanelRowShift = 24;       // panel entry code = (row inside the workgroup << 24) | staged head row

// dense corner of the head block: rows and columns [0, corner) of level 0, cut into tiles of
// kCornerTile x kCornerTile positions.  A workgroup owns the accumulators of one row panel
// (kCornerTile rows) in LDS and sweeps a run of the panel's tiles, each with its kCornerTile
// staged head rows copied into LDS; a tile's entries are dealt to kCornerRuns lane-group streams
// that never share a row.  Entry code = (row inside the panel << 16) | column inside the tile.
constexpr int kCornerTile = 256;
constexpr int kCornerRuns = 64;
constexpr int kCornerTileWords = kCornerRuns + 3;   // per tile: run offsets (kCornerRuns + 1), first column, panel

struct LevelImage {
  int64_t n_i = 0;
  // permutation (int32 n_i)
  size_t off_perm = 0;
  // staged head: rows of X gathered into a contiguous buffer before the level runs
  bool staged = false;
  bool stage_used = false;      // an entry reads the buffer (else it need not be filled)
  int64_t n_stage = 0;          // rows of the staging buffer (min(b, n_i) or 0)
  int64_t stage_class_rows = 0; // rows of the first column class in the buffer
  size_t off_stage_perm = 0;    // int32 n_stage : buffer row -> X row
  bool row_major = false;       // the wave list is ordered by length, not by column window
  int32_t classes = 0;          // column classes used for the chunk queues (0 = none)
  // group list: items handled one per lane group (class pieces in die queues, then the short rows)
  int64_t n_rows = 0, n_real_rows = 0, rows_partials = 0, nnz_rows = 0;
  int64_t piece_slots = 0;   // slots [0, piece_slots) hold the class pieces (die queues), the rest the short rows
  int64_t longest_short = 0; // entries of the longest short row of the group list (pieces apart)
  int64_t empty_slots = 0;   // the last empty_slots slots are rows of Y without entries
  size_t off_rows_ptr = 0;   // uint32 n_rows + 1 (offsets into the level's entry array)
  size_t off_rows_mid = 0;   // uint32 n_rows : entries before it read the staged head buffer, the rest read X
  size_t off_rows_dst = 0;   // int32  n_rows : >= 0 -> Y row, < 0 -> partial slot (-1 - slot), INT32_MIN -> padding
  size_t off_rows_row = 0;   // int32  n_rows : the vertex (row of A) the item belongs to, -1 for padding
  // wave list: items handled one per wavefront (the list may contain empty padding slots)
  int64_t n_chunks = 0, n_real_chunks = 0, chunks_partials = 0, nnz_chunks = 0;
  size_t off_chunk_ptr = 0;  // uint32 n_chunks + 1
  size_t off_chunk_mid = 0;  // uint32 n_chunks : entries before it read the staged head buffer, the rest read X
  size_t off_chunk_dst = 0;  // int32  n_chunks : >= 0 -> Y row (whole row in one chunk), < 0 -> partial slot (-1 - slot), kTeamDst, INT32_MIN -> padding
  size_t off_chunk_row = 0;  // int32  n_chunks : the vertex the item belongs to, -1 for padding
  // rows assembled from several chunks
  int64_t n_split = 0, n_partials = 0;
  size_t off_split_ptr = 0;  // uint32 n_split + 1 (partial slots of a row are consecutive)
  size_t off_split_y = 0;    // int32  n_split
  // entries: first nnz_rows for the row list, then nnz_chunks for the chunk list
  size_t off_entries = 0;
  int64_t x_rows_rows = 0, x_rows_chunks = 0;  // distinct X rows each list references
  // diagonal-block tiles processed with their window of P_i X staged in LDS; their entries
  // follow the chunk entries in the level's entry array
  int64_t n_wtiles = 0, n_wrows = 0, nnz_w = 0;
  size_t off_wtiles = 0;     // WindowTile n_wtiles
  size_t off_wrow_ptr = 0;   // uint32 n_wrows + 1
  size_t off_wrow_mid = 0;   // uint32 n_wrows : entries before it read X rows, the rest index the LDS window
  size_t off_wrow_y = 0;     // int32  n_wrows
  size_t off_wrow_win = 0;   // uint32 n_wrows : first position of the row's tile window
  // head panels: head rows whose head-block entries are swept window by window with the rows'
  // accumulators resident in LDS; their entries follow the window entries in the entry array.
  // Workgroup w = group * kDies + class owns bins [w * kPanelBins, (w + 1) * kPanelBins).
  int64_t n_panel_rows = 0, n_panel_groups = 0, n_panel_bins = 0, nnz_panel = 0;
  size_t off_panel_ptr = 0;  // uint32 n_panel_bins + 1 (entry offsets; a bin is one lane group's stream)
  size_t off_panel_y = 0;    // int32  n_panel_groups * kPanelRows : Y row of every accumulator, -1 = unused
  // dense corner (see kCornerTile): its entries follow the panel entries in the entry array
  int64_t corner = 0;        // rows = columns of the corner (a multiple of kCornerTile), 0 = none
  int64_t n_corner_tiles = 0, n_corner_items = 0, nnz_corner = 0;
  size_t off_corner_tiles = 0;   // uint32 n_corner_tiles * kCornerTileWords
  size_t off_corner_items = 0;   // uint32 n_corner_items * 2 + 2 : first tile of every item (+ end), then ...
  size_t off_corner_panel = 0;   // uint32 panels + 1 : first item of every row panel (items of a panel are consecutive)
  size_t off_corner_y = 0;       // int32  corner : Y row of every corner row position
  int64_t map_offset = 0;    // first element of this level in the entry map (one uint32 per entry, image order)
  int64_t nnz_fused = 0;     // level 0 with fused levels: entries of later levels listed with its rows
};

// Rows [row_begin, row_end) of the window-row list belong to one diagonal block and touch only
// column positions [win_begin, win_begin + win_count) of it.
struct WindowTile {
  uint32_t row_begin, row_end;
  uint32_t win_begin, win_count;
};

struct PackOptions {
  int32_t short_max = 16;     // rows with at most this many entries go to the lane-group list
  int32_t chunk_nnz = 256;    // most nonzeros per wavefront chunk
  int32_t chunk_min = 64;     // windows of a row are merged until a chunk holds this many
  int32_t window_rows = 4096; // column positions per window of the chunk ordering (0 = row-major chunks)
  int32_t classes = 0;        // column classes (rounded up to a multiple of 8; 0 = no die queues)
  int32_t class_gran = 512;   // column positions dealt to a class at a time
  int32_t class_min = 32;     // a row is split by class when it holds classes * class_min entries
  int32_t piece_max = 48;     // a class piece with at most this many entries is a group-list item
  int32_t stage_head = 1;     // gather the head rows of level 0 into a contiguous buffer
  int32_t stage_short = -1;   // short rows read their head columns from the staged head too (-1 = when the head is scattered over X)
  int32_t empty_last = 1;     // level 0: the short rows without entries are listed after all others
  int32_t panel = 0;          // run the head block of sparse head rows in panels (accumulators in LDS, one column class per die)
  int32_t panel_min = 8;      // fewest head-block entries of a row that joins a panel
  int32_t window_span = 2048; // widest column span of an LDS-window tile (0 = no such tiles)
  int32_t window_tile_rows = 1024;  // most rows per tile
  double window_reuse = 8.0;  // a tile is kept when its diagonal-block entries >= this x span
  double window_level_share = 0.05;  // ... and the tiles of a level when they hold this share of its entries
  int32_t fuse_levels = 1;    // list the entries of later levels with the level-0 rows of their vertices
  int32_t corner = 0;         // run the dense top-left corner of the head block in LDS tiles (off: measured slower than the chunk list)
  int32_t corner_max = 65536; // largest corner considered (rows = columns)
  int32_t corner_min_tile = 768;  // the corner grows while the tiles it gains hold at least this many entries on average
};

struct Image {
  std::vector<LevelImage> levels;
  std::vector<unsigned char> bytes;  // packed host copy
  int64_t max_partials = 0;
  int64_t max_stage_rows = 0;
  int64_t max_window_span = 0;
  int64_t max_panel_slots = 0;       // most panel accumulators (groups * kPanelRows) of a level
  int64_t max_corner_items = 0;      // most corner work items of a level (each writes kCornerTile result rows)
  std::vector<uint32_t> entry_src;   // per entry in image order: its index in the caller's CSR arrays
  bool fused = false;                // the image was packed from the fused execution form of the levels
};

int pack_image(int64_t n, int32_t b, const std::vector<HostLevel>& levels, const PackOptions& opt,
               Image& img, std::string& err);
// host-side consistency check of a packed image (used by arrow_self_check)
int verify_image(int64_t n, int32_t b, const std::vector<HostLevel>& levels, const Image& img,
                 std::string& err);

// ---------------------------------------------------------------------------
// Kernel launchers (kernels.hip).  All pointers are device pointers; `stream`
// is a hipStream_t.  Each returns a hipError_t cast to int.
// ---------------------------------------------------------------------------
struct LaunchTuning {
  int32_t kc = 0;          // column slice width per pass (0 = automatic)
  int64_t l2_resident_bytes = 2 << 20;  // share of a die's 4 MiB L2 a resident slice of X_0 may take
};

// The work lists of one level for one launch (device pointers; launch_product fills in the grid).
struct ProductArgs {
  const uint32_t* chunk_ptr; const uint32_t* chunk_mid; const int32_t* chunk_dst;   // wave list
  const uint32_t* rows_ptr; const uint32_t* rows_mid; const int32_t* rows_dst;      // group list
  const Entry* ent;
  const float* X; const float* Xh;      // dense operand; staged head (X where nothing is staged)
  float* Y; float* partials;
  int64_t n_chunks;
  int64_t longest_short;                // entries of the longest short row
  int32_t head_stride;                  // floats from one row of Xh to the next (those of X are k apart)
  int32_t k, accumulate;                // accumulate: add to the rows of Y instead of storing them
  // parts 0 .. 3: wave list, pieces, short rows, rows without entries
  int64_t begin[4], count[4];           // slots of the part
  uint32_t blocks[4];                   // workgroups per column slice
  int32_t items[4];                     // slots per workgroup
  uint32_t slices;
  uint32_t sets_log;                    // logarithm of the sets of dies that the slices are dealt to (0: every die works on all)
  int32_t width;                        // columns per slice
  int32_t piece_waves;                  // a piece per wavefront instead of per lane group
  int32_t together;                     // parts that share a launch where the product is not profiled (0: those of this launch)
  int32_t entries_once;                 // the entries are too many to be found in a cache the next time
  uint32_t run;                         // workgroups of the wave list that a die takes one after the other (die_run), or 0
};
enum { kPartChunks = 1, kPartPieces = 2, kPartShort = 4, kPartAll = 7 };
// Launches the given parts.  n_pieces, n_rows, n_empty: pieces, all items and trailing empty rows of
// the group list; x_rows = rows of X (it decides whether 32-bit offsets are enough); kc = columns per
// pass (0: the whole row); windows: the wave list is ordered by column window.
int launch_product(ProductArgs a, int parts, int64_t n_pieces, int64_t n_rows, int64_t n_empty, bool die_queues,
                   bool windows, int64_t x_rows, int32_t kc, void* stream);
// whether launches with these two kc have the same shape, so that their parts can share one
bool same_shape(int32_t k, int32_t kc_a, int32_t kc_b, bool accumulate);
int launch_reduce(const uint32_t* split_ptr, const int32_t* split_y, int64_t n_split,
                  const float* partials, float* Y, int32_t k, bool accumulate, void* stream);
// Rows of k columns; those of Xp are `stride` floats apart.
int launch_gather(const int32_t* perm, int64_t n_i, const float* X, float* Xp, int32_t k, int32_t stride,
                  void* stream);
// Head panels.  launch_panel: every workgroup (group, class) sums its entries times rows of the
// staged head Xh into LDS accumulators and stores them to part[class][slot][0:k].
// launch_panel_combine: Y[panel_y[slot]] += sum over the kDies classes, in class order.
int launch_panel(const uint32_t* panel_ptr, const int32_t* panel_y, const Entry* entries,
                 int64_t n_groups, const float* Xh, int64_t xh_rows, float* part, int32_t k, void* stream);
int launch_panel_combine(const int32_t* panel_y, int64_t n_slots, const float* part, float* Y, int32_t k,
                         void* stream);
int launch_sddmm_panel(const uint32_t* panel_ptr, const int32_t* panel_y, const Entry* entries,
                       const uint32_t* emap, int64_t n_bins, const float* U, const float* Vh,
                       int64_t vh_rows, float* S, int32_t k, void* stream);
// Dense corner.  launch_corner: workgroup = item; sums the item's tiles into LDS accumulators and
// stores kCornerTile rows to part[item].  launch_corner_combine: Y[corner_y[p]] += the parts of the
// items of p's panel, in item order.  launch_sddmm_corner: the sampled product over the corner tiles.
int launch_corner(const uint32_t* tiles, const uint32_t* items, int64_t n_items, const Entry* entries,
                  const float* Xh, int64_t xh_rows, float* part, int32_t k, void* stream);
int launch_corner_combine(const uint32_t* panel_ptr, const int32_t* corner_y, int64_t corner,
                          const float* part, float* Y, int32_t k, void* stream);
int launch_sddmm_corner(const uint32_t* tiles, int64_t n_tiles, const int32_t* corner_y, const Entry* entries,
                        const uint32_t* emap, const float* U, const float* Vh, int64_t vh_rows, float* S,
                        int32_t k, void* stream);
// max_span = widest window of the tiles (sizes the LDS allocation and the column slice), nnz = entries of all of them
int launch_window(const WindowTile* tiles, int64_t n_tiles, int64_t max_span, int64_t nnz, const uint32_t* wrow_ptr,
                  const uint32_t* wrow_mid, const int32_t* wrow_y, const Entry* entries,
                  const int32_t* perm, const float* X, int64_t x_rows, float* Y, int32_t k, bool accumulate,
                  void* stream);


// Sampled dense-dense product S[emap[e]] = a_e <U[row(e)], V[col(e)]> over the wave list and the group
// list of a level, or over its window-row list (rows_*, rows_win and perm then describe that one).
// emap points at the level's slice of the entry map, or is null: S in image order.
struct SampledArgs {
  uint32_t chunk_parts;                 // wavefronts that share a chunk (filled in by the launch)
  const uint32_t* chunk_ptr; const uint32_t* chunk_mid; const int32_t* chunk_row;
  const uint32_t* rows_ptr; const uint32_t* rows_mid; const int32_t* rows_row;
  const uint32_t* rows_win; const int32_t* perm;
  int32_t head_stride;                  // floats from one row of Vh to the next (those of V are k apart)
  const Entry* ent; const uint32_t* emap;
  const float* U; const float* V; const float* Vh;
  float* S;
  int64_t n_chunks, n_rows;             // (rows without entries, the last ones of a group list, are left out)
  int64_t n_pieces;                     // the first n_pieces of the rows are pieces of long rows
  int64_t nnz_chunks, nnz_rows;
  int32_t k;
  int32_t items;                        // group-list slots per workgroup (filled in by the launch),
  int32_t piece_items;                  // ... of the pieces,
  uint32_t piece_blocks;                // ... which have the first of the workgroups of the rows; the short rows'
  uint32_t short_base;                  // ... begin at item id * items + short_base (mod 2^32)
  uint32_t chunk_blocks;
  uint32_t run;                         // as in ProductArgs
};
// v_rows = rows of V; windows, die_queues: as in launch_product (the grid is filled in here); unequal: the group list
// holds pieces of long rows, not only short ones.
int launch_sddmm(SampledArgs a, bool window_rows, bool die_queues, bool windows, bool unequal, int64_t v_rows, void* stream);
constexpr int kSampledBatch = 4;        // entries a lane group reduces together (= row loads in flight per lane)

// Device address of the current device's copy of the static scratch array of arrow_spmm_static
// (static_scratch.hip); NULL and a description in `err` on failure.  A lookup, never an allocation.
unsigned char* static_scratch(std::string& err);

// Bare row gather (probe.hip), the yardstick of the measurements: `gathers` pseudo-random rows of
// the n x k matrix X drawn from its first region_rows rows (per_die: from a region of its own for
// every accelerator die; from_lds: the region is copied into LDS first) are read and summed.
int64_t probe_out_floats(int64_t gathers);
int launch_probe_gather(const float* X, int64_t x_rows, int32_t k, int64_t region_rows, int per_die,
                        int from_lds, int64_t gathers, float* out, void* stream);

// Order-3 MTTKRP over the compressed-sparse-fibre image (mttkrp.hip): one wavefront per item.
// b_rows, c_rows = rows of the factor matrices (they decide whether 32-bit offsets are enough).
// Limits of one work item of the fibre image: the wavefront that owns the item stages its entries
// and segment descriptors in LDS, so both are bounded.
constexpr int kCsfSegMax = 64;      // most entries of a segment
constexpr int kCsfItemNnz = 512;    // most entries of an item
constexpr int kCsfItemSegs = 128;   // most segments of an item
// item_ent[it] = index of the item's first entry (the items' entries are consecutive).
int launch_mttkrp(const uint32_t* item_seg, const uint32_t* item_ent, const int32_t* item_dst,
                  const uint32_t* seg_ptr,
                  const int32_t* seg_j, const Entry* entries, int64_t n_items, const float* B,
                  int64_t b_rows, const float* C, int64_t c_rows, float* A, float* partials, int32_t R,
                  int32_t longest, int32_t average, void* stream);   // entries and segments of the longest item and of one on average

// The other form of the fibre image, for factors whose rows all fit the LDS of a compute unit four (or even eight) columns at a
// time (resident_kernel in mttkrp.hip): the segments of an item side by side, one per lane, as a sequence of
// STEPS, in each of which a lane reads one row from LDS and has a value for it.  In LDS lie the K rows of C, a
// row of zeros (which the steps that fill up read) and the J rows of B.  A bit per step says that its rows are
// rows of B, which end a batch of 64 segments.  Steps come in blocks of eight, an item has at least one: what the kernel
// loads ahead of an item is the next one's, at last the last one's again, and never lies beyond the blocks.
constexpr int kCsfRowsInLds = 10200;    // rows of four columns, 16 bytes each
constexpr int kCsfBlockSteps = 8;
struct ResidentBlock {
  // of two steps: the first one's row << 4, the second one's << 18; bits 0 and 1: their rows are of B
  struct alignas(16) Offsets { uint32_t pair[4]; };
  struct alignas(16) Values { float v[4]; };
  Offsets offsets[64];                  // by lane
  Values values[2][64];
};
static_assert(kCsfRowsInLds < 1 << 14, "bits of a row");
struct ResidentItem {
  uint32_t block, blocks;   // first block and their number
  int32_t dst;              // as in the other form
};
// last: steps of each item's last block that do not only fill it up (null: not known)
int launch_mttkrp_resident(const ResidentItem* items, const ResidentBlock* blocks, int64_t n_items, int64_t n_blocks,
                           const float* B, int64_t b_rows, const float* C, int64_t c_rows, float* A, float* partials,
                           int32_t R, void* stream, const uint32_t* last = nullptr);

// A third form, for tensors of many small slices and fibres of about one entry, whose factors do not fit an L2
// (streams_kernel in mttkrp.hip): a wavefront owns rows of A and keeps their sums in LDS; each of its eight lane
// groups goes through the entries of rows of its own, ordered by windows of one factor's rows, so that all lane
// groups of the chip read the same part of that factor at a time.
constexpr int kCsfStreamRows = 71;      // most rows of a wavefront; one more takes what fills up
constexpr int kCsfStreamGroups = 8;     // lane groups
constexpr int kCsfStreamTeam = 16;      // wavefronts of a workgroup, which wait for each other
constexpr uint32_t kCsfStreamTurn = 4;  // ... after so many blocks
constexpr int64_t kCsfStreamRowsOfB = 1 << 25;   // most rows of B: an index shares a word with the place of the sum
struct StreamBlock {                    // eight entries of each lane group: word 8 g + s is entry s of group g
  struct Record { uint32_t j_slot; int32_t k; float val; };   // row of B << 7 | place of the sum
  Record rec[64];
};
struct StreamWave {
  uint32_t block, blocks;               // first block and their number
  uint32_t turns;                       // of kCsfStreamTurn blocks, in the wavefront of the team that has most
  uint32_t zero, zeros;                 // its part of the rows of A without entries
};
// dst[kCsfStreamRows * w + place]: row of A, -1 - partial vector, or kCsfNoRow
constexpr int32_t kCsfNoRow = INT32_MIN;
int launch_mttkrp_streams(const StreamWave* waves, const StreamBlock* blocks, const int32_t* dst, const int32_t* zero_rows,
                          int64_t n_waves, const float* B, int64_t b_rows, const float* C, int64_t c_rows, float* A,
                          float* partials, float* scratch, int32_t R, void* stream);
// Columns a wavefront of that form sums at a time; whether rows of R columns are whole lines or parts of one, so that
// slices of them are too where the factor begins at a line; and floats of the scratch that factors take
// which are laid out anew because they are not (may be null: they are read where they are).
constexpr int stream_slice(int32_t R) { return R > 16 ? 32 : R > 8 ? 16 : 8; }
constexpr bool stream_lines(int32_t R) { return R % stream_slice(R) == 0 || stream_slice(R) % R == 0; }
constexpr int64_t stream_scratch(int64_t b_rows, int64_t c_rows, int32_t R) {
  return (b_rows + c_rows) * ((R + (int64_t)stream_slice(R) - 1) / stream_slice(R)) * stream_slice(R);
}

}  // namespace arrow
