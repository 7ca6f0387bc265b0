// Internal interface of the ragged batched path: the device-side header and
// row table a batch is described by, the workspace pointers the kernels use,
// and the launch plan. Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nrm.h"
#include "nrm_internal.h"

namespace nrm {

// One row as the kernels see it (same layout as the public nrm_row).
struct RowDesc {
  const char* in;
  char* out;
  int64_t n;
  int32_t in_dt;
  int32_t out_dt;
};
static_assert(sizeof(RowDesc) == sizeof(nrm_row), "RowDesc must match nrm_row");

enum { BATCH_CSR = 0, BATCH_TABLE = 1 };

// Per-call inputs, passed as a kernel argument.
struct BatchHeader {
  int64_t nrows;
  int32_t mode;            // BATCH_CSR or BATCH_TABLE
  int32_t csr_in_dt, csr_out_dt;
  int32_t rows_per_block;  // rows each block of batch_rows_kernel takes: 1..8 or ROWS_MAX
  const int64_t* offsets;  // CSR: rows + 1 offsets (device)
  const char* csr_in;
  char* csr_out;
  int64_t capacity;        // CSR: elements addressable through csr_in / csr_out
  const RowDesc* table;    // TABLE: the row table (pinned host memory)
  float* lse;              // softmax: each row's log-sum-exp (device), or NULL
  int64_t run_max;         // rows of wave_max < n <= run_max are run by a block of batch_rows_kernel
  int64_t grid_x;          // blocks of batch_rows_kernel in one row of its grid
};

// Device error bits (OR-ed by the kernels, read by nrm_get_device_error).
enum {
  NRM_DEVERR_OFFSETS = 1,   // CSR offsets negative, decreasing or past capacity
  NRM_DEVERR_ROW = 2,       // a table row with n < 0, bad dtype, NULL pointer, or too many tiles
  NRM_DEVERR_CAPACITY = 4,  // more rows or list entries than the workspace holds
  NRM_DEVERR_TARGET = 8,    // NLL loss: a target outside [0, C) that is not ignore_index
  NRM_DEVERR_STALL = 16,    // a resident row's segments did not all arrive within the spin limit
};

constexpr int64_t MAX_ROW_TILES = 65536;  // partials the per-row combine merges

// One entry of a work list: a tile of a long row, a segment of a resident
// row, or a whole single-pass row (tile 0), with the row's descriptor (a
// reader needs no second load). row -1: an empty entry.
struct Item {
  RowDesc d;
  int32_t row;
  int32_t tile;
};

// Words the kernels of one call share (device memory, zero at first; 64-bit).
// The counters of the work lists are in two sets, used by calls in turn, each
// counter on a 128-byte line of its own.
constexpr int CNT_LINE = 16;
enum {
  CNT_CALL = 0,      // the last call's number
  CNT_CALL_RUN = 1,  // the number of the call that runs, for its later launches
  CNT_LSE = 2,       // softmax: the header's lse pointer, for the later launches
  CNT_ORDERED = 4,   // blocks whose entries block_shorts orders (0: more than it holds)
  CNT_STALL = 3,     // the tag of the last call in which a wait gave up
  CNT_TAKEN = CNT_LINE,  // list entries taken so far by the resident rows' kernel
  CNT_SET0 = 2 * CNT_LINE,
};
enum { LIST_TILES = 0, LIST_SHORT = 1, LIST_LONG_ROWS = 2, LIST_COUNTERS = 3 };
constexpr int CNT_SET_STRIDE = LIST_COUNTERS * CNT_LINE;
constexpr int CNT_COUNT = CNT_SET0 + 2 * CNT_SET_STRIDE;

// The entries of `shorts` that one block of batch_rows_kernel appended.
struct BlockShorts {
  int64_t base, count;
};
// (65536 rows, 32 per block: rows long enough to be listed, 4 GB and more)
constexpr int ORDERED_BLOCKS = 2048;

// One row's reduction result: the sum (a) for normalize, or the exponent and
// the scaled sum (a = k, b = s) for softmax.
struct RowRes {
  float a, b;
};

// Kernel arguments: workspace pointers, fixed for a context's workspace, and
// the call's header (batch_rows_kernel only).
struct BatchArgs {
  BatchHeader header;
  Item* tiles;           // [cap_items]: the long rows' tiles
  Item* shorts;          // [cap_items]: the resident rows' segments, or the single-pass rows
  BlockShorts* block_shorts;  // [ORDERED_BLOCKS]
  int64_t* lrow_first;   // [cap_rows]: each long row's first entry, -1: it did not fit (resident rows off, or apart)
  int64_t* cnt;          // [CNT_COUNT]
  int* error;            // [1]
  int64_t cap_rows;
  int64_t cap_items;
  int64_t tile;          // elements per tile of a long row: 2^tile_log2
  int tile_log2;
  int64_t short_max;     // longer rows are long
  int64_t keep_tiles;    // the last this many tiles are summed with temporal loads
  // rows of 0 < n <= wave_max elements are taken by 16 lanes or one wavefront
  // (0: none; at most WAVE_MAX_ELEMS)
  int64_t wave_max;
  // resident rows (res_on): a row of 2^RES_LOG2 < n <= short_max elements is
  // cut into segments of 2^RES_LOG2 elements, one entry each, each held in one
  // block's registers from its read to its write
  int res_on;
  int apart;  // long rows in launches of their own, not in the resident rows' kernel
  // by a row's first entry: its entries' partials (two tagged words each),
  // its total (two tagged words), and the count of its published partials (0
  // between calls)
  unsigned long long* tagged;       // [2 * cap_items], shorts
  unsigned long long* rowtot;       // [2 * cap_items]
  unsigned* arrivals;               // [cap_items]
  unsigned long long* tile_tagged;  // [2 * cap_items], tiles
  unsigned long long* tile_total;   // [2 * cap_items]
  unsigned* tile_arrivals;          // [cap_items]
  // without resident rows: each tile's partial, and by a row's first tile its
  // result, plain (apart from the tagged words, of which any bits that equal a
  // call's tag count as published)
  void* partials;    // [cap_items] x 8 bytes
  RowRes* results;   // [cap_items]
};

// batch_rows_kernel: blocks of ROWS_BLOCK threads, at most ROWS_MAX rows each
// (four per wavefront).
constexpr int ROWS_BLOCK = 512;
constexpr int ROWS_WAVES = ROWS_BLOCK / 64;
constexpr int ROWS_MAX = 4 * ROWS_WAVES;

// Its grid, for `blocks` blocks: one row of them, or rows of at most
// ROWS_GRID_X, since a launch's extent in threads is a 32-bit number in each
// dimension (2^23 blocks of 512 are one too many) and a batch may have up to
// 2^31 - 1 rows. Block (x, y) is number y * x_extent + x; the few numbers past
// the last block find no rows.
constexpr int64_t ROWS_GRID_X = int64_t(1) << 20;
inline int64_t rows_grid_y(int64_t blocks) { return (blocks + ROWS_GRID_X - 1) / ROWS_GRID_X; }
inline int64_t rows_grid_x(int64_t blocks) { return (blocks + rows_grid_y(blocks) - 1) / rows_grid_y(blocks); }

// Elements of one resident segment: 512 threads x 8 vectors of 4 binary32
// (4 vectors of 8 for 2-byte inputs); three blocks fit a CU's registers.
constexpr int RES_LOG2 = 14;
constexpr int RES_BLOCK = 512;
constexpr int RES_MAX_SEGMENTS = 64;  // one wavefront lane per segment in the merge

// Long rows' tile sums beside the resident rows: vectors per thread per
// iteration, chains per thread, and the elements of a part. A longer tile is
// summed part by part, so that its threads' chains, and with them the row's
// summation tree, stay low.
constexpr int TILE_U = 4;
constexpr int TILE_NA = 8;
constexpr int64_t TILE_PART = int64_t(1) << 19;

// Height of such a row's summation tree (binary32 sums): a thread's part
// (CHAIN_ADDS + 1 additions in a chain, the merge of its chains, one addition
// per CHAIN_ADDS elements of every chain), the block's (wavefront 6, its
// wavefronts 3), the tile's parts one after the other, and the row's tiles (RES_BLOCK at a
// time by a block, then up to MAX_ROW_TILES / RES_BLOCK totals by a wavefront,
// two per lane). The published bound is gamma_62.
constexpr int log2_of(int64_t x) { return x <= 1 ? 0 : 1 + log2_of(x / 2); }
constexpr int long_row_height(int tile_log2) {
  const int64_t tile = int64_t(1) << tile_log2, part = tile < TILE_PART ? tile : TILE_PART;
  const int64_t flush = (int64_t)RES_BLOCK * CHAIN_ADDS * TILE_NA;
  return (int)(CHAIN_ADDS + 1 + log2_of(TILE_NA) + (part + flush - 1) / flush + log2_of(RES_BLOCK) + (tile / part - 1) +
               log2_of(RES_BLOCK) + log2_of(MAX_ROW_TILES / RES_BLOCK));
}

// The longest row of one wavefront (2048 binary32: eight 16-byte vectors per lane).
constexpr int64_t WAVE_MAX_ELEMS = 2048;

struct BatchPlan {
  int acc;
  int64_t rows_grid;    // blocks of batch_rows_kernel in x
  int64_t rows_grid_y;  // and rows of them
  bool lists;         // rows may be listed: launch the lists' kernels
  int64_t res_grid;   // persistent blocks of the resident rows' kernel
  // resident rows off: the three list kernels' shapes
  int block;
  int unroll;       // tile sums: vectors per thread per iteration
  int map_unroll;   // tile divides
  int short_regs;   // vectors per thread held for a single-pass row
  int64_t grid;     // blocks of phase 1 and of the row sums
  int map_block;    // phase 2
  int64_t map_grid;
};

// The first launch of a sequence, for a graph's node.
const void* rows_kernel(int acc);
hipError_t launch_batch(const BatchPlan& p, const BatchArgs& a, hipStream_t s);

}  // namespace nrm
