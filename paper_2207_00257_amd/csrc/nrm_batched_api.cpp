// C ABI of the ragged batched path (include/nrm.h): workspace and pinned
// staging management, host validation, the launch sequence (the rows, then
// the lists of the longer ones) and its optional capture in a hipGraph. A row
// table is written to pinned, coherent host memory that the first launch reads
// in place; a ring of such buffers (one graph each) lets a call be enqueued
// while the previous ones still run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "nrm_ctx.h"

using nrm::BatchArgs;
using nrm::BatchHeader;
using nrm::BatchPlan;
using nrm::BatchWorkspace;
using nrm::DeviceGuard;
using nrm::RowDesc;
using nrm::fail;
using nrm::hip_fail;

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The call's words and counters, then the device error word, in one region.
constexpr size_t kErrorOffset = sizeof(int64_t) * nrm::CNT_COUNT;
constexpr size_t kSmallBytes = kErrorOffset + 128;
int64_t align_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

// Batches of at least this many elements are replayed from a captured graph
// (parameter graph = 1), smaller ones launched kernel by kernel. On MI355X
// hipGraphLaunch takes 15.8 us of the host whatever the graph holds, a kernel
// launch 1.1 us, and a replay of the two launches about 10 us more of the device
// than the launches themselves (4096 rows of up to 2^20: 587 and 577 us; 2^20 x 256:
// 358 and 348). No size was found where a replay is the faster one; it is kept where
// it costs 3 % at most, for callers that ask for one submission per batch.
constexpr int64_t kGraphElems = int64_t(1) << 27;

// Batches of at least this many elements, most of them in long rows, run the
// long rows in launches of their own (the results are the same). us per call on
// MI355X, in the persistent kernel and apart:
//                         rows of 2,000,000, 32       64         128
//   binary32                        128 and 127  258 and 246  545 and 492
//   bfloat16                         92 and  73  189 and 135
//   bfloat16 to binary32             99 and 133  218 and 217
// and 16 rows of 20,000,000 676 and 611, 424 and 318, 569 and 551. (At most 8 rows
// are also a little faster apart, 29 and 26 us for 4 of them, for three launches
// more on the host.)
constexpr int64_t kApartElems = int64_t(1) << 26;
constexpr int64_t kApartElemsWide = int64_t(1) << 27;  // with outputs wider than inputs among them

// From 2^27 elements on a quarter of the resident limit is enough of a mean: with
// lengths spread over a few powers of two most elements are in long rows then
// (1000 rows of 32 to 2^22 binary32, mean 350,000: 773 and 722 us; bfloat16 499 and
// 441), and equal rows of that mean, none of them long, do not lose by the idle
// launches more than they gain without a replay (1000 x 300,000: 418 and 415).
bool apart_rows(const BatchArgs& a, int64_t elems, int64_t mean, bool wide) {
  if (!a.res_on) return false;
  return elems >= kApartElemsWide ? mean > a.short_max / 4 : !wide && elems >= kApartElems && mean > a.short_max;
}

// Blocks of their divide, at least: a block's tiles are dealt to it beforehand,
// so that more blocks than run at once even out the last round. us per call by
// 1024, 2048, 4096 and 8192 blocks: 64 x 2,000,000 binary32 246, 241, 248, 249; 16 x
// 20,000,000 614, 603, 603, 603, bfloat16 to binary32 552, 544, 517, 556; softmax of
// 267 x 1,521,478 845, 832, 822, 802.
int64_t apart_map_grid(int64_t elems, int acc) {
  return elems < int64_t(1) << 28 ? 2048 : acc == nrm::ACC_SOFTMAX ? 8192 : 4096;
}

nrm_batch_params default_batch_params() {
  nrm_batch_params p;
  std::memset(&p, 0, sizeof(p));
  // On MI355X: within a few percent of the tuner's best for the 4096-row
  // ragged workload, and with persistent grids small enough that small
  // batches (serving) do not pay for dispatching idle blocks.
  p.block = 256;
  p.unroll = 8;
  p.map_unroll = 4;
  p.grid = 2048;
  p.tile_log2 = 15;
  p.short_regs = 4;
  p.graph = 1;  // replay captured graphs (one per staging buffer and reduction kind)
  p.map_block = 1024;
  p.map_grid = 1024;
  p.keep_mib = 256;
  // rows up to 64 segments of 2^14 elements (2^20) are held on chip between
  // their read and their write; three 512-thread blocks per CU
  p.resident_segments = 64;
  p.resident_grid = 768;
  // rows of up to 2048 elements one per wavefront
  p.wave_max = 2048;
  p.wave_grid = 1024;  // without effect
  return p;
}

int check_batch_params(const nrm_batch_params& p) {
  auto ok_u = [](int u) { return u == 1 || u == 2 || u == 4 || u == 8; };
  if (p.block < 64 || p.block > 1024 || p.block % 64 || p.map_block < 64 || p.map_block > 1024 || p.map_block % 64)
    return fail(NRM_EINVAL, "block and map_block must be 64..1024, multiples of 64");
  if (p.map_grid < 1 || p.map_grid > (1 << 20)) return fail(NRM_EINVAL, "map_grid must be 1..2^20");
  if (!ok_u(p.unroll) || !ok_u(p.map_unroll) || !ok_u(p.short_regs))
    return fail(NRM_EINVAL, "unroll, map_unroll and short_regs must be 1, 2, 4 or 8");
  if (p.grid < 1 || p.grid > (1 << 20)) return fail(NRM_EINVAL, "grid must be 1..2^20");
  if (p.tile_log2 < 10 || p.tile_log2 > 22) return fail(NRM_EINVAL, "tile_log2 must be 10..22");
  if (p.graph != 0 && p.graph != 1) return fail(NRM_EINVAL, "graph must be 0 or 1");
  if (p.keep_mib < 0 || p.keep_mib > 4096) return fail(NRM_EINVAL, "keep_mib must be 0..4096");
  if (p.resident_segments < 0 || p.resident_segments > nrm::RES_MAX_SEGMENTS)
    return fail(NRM_EINVAL, "resident_segments must be 0..64");
  if (p.resident_grid < 1 || p.resident_grid > (1 << 20)) return fail(NRM_EINVAL, "resident_grid must be 1..2^20");
  // the blocks of one resident row wait for each other: the kernel must be
  // able to hold a whole row's segments in running blocks at once
  if (p.resident_grid < p.resident_segments)
    return fail(NRM_EINVAL, "resident_grid must be at least resident_segments");
  if (p.wave_max < 0 || p.wave_max > nrm::WAVE_MAX_ELEMS) return fail(NRM_EINVAL, "wave_max must be 0..2048");
  if (p.wave_grid < 1 || p.wave_grid > (1 << 20)) return fail(NRM_EINVAL, "wave_grid must be 1..2^20");
  // a tile's per-thread summation tree must stay within the plain path's
  // height bound (36) for every input dtype: 4-byte elements give the most
  // iterations, 2-byte elements the most additions per iteration
  const int64_t tile = int64_t(1) << p.tile_log2;
  for (int dt : {NRM_F32, NRM_BF16}) {
    int64_t iters = ceil_div(tile, (int64_t)p.block * p.unroll * nrm::dtype_vec(dt));
    if (nrm::thread_tree_height(dt, NRM_ACC_F32, p.unroll, iters) > 36)
      return fail(NRM_EINVAL, "tile too long for block * unroll: a thread's summation tree would exceed height 36");
  }
  return NRM_OK;
}

// Rows of at most this many elements are not long: single-pass rows, or
// resident rows when those are on.
int64_t short_max_of(const nrm_batch_params& p) {
  return p.resident_segments > 0 ? (int64_t)p.resident_segments << nrm::RES_LOG2 : (int64_t)p.block * p.short_regs * 4;
}

bool any_graph(const BatchWorkspace& w) {
  for (const auto& per_kind : w.graph)
    for (const nrm::BatchGraph& g : per_kind)
      if (g.exec) return true;
  return false;
}

void destroy_graph(BatchWorkspace& w) {
  for (auto& per_kind : w.graph)
    for (nrm::BatchGraph& g : per_kind) {
      if (g.exec) (void)hipGraphExecDestroy(g.exec);
      if (g.graph) (void)hipGraphDestroy(g.graph);
      g = nrm::BatchGraph();
    }
}

// Layout of the single device allocation.
struct Layout {
  size_t tiles, shorts, block_shorts, lrow_first, partials, results, small, tagged, rowtot, arrivals, tile_tagged, tile_total,
      tile_arrivals, total;
};

Layout layout_for(int64_t cap_rows, int64_t cap_items) {
  Layout L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t at = off;
    off = (size_t)align_up((int64_t)(off + bytes), 256);
    return at;
  };
  L.tiles = take(sizeof(nrm::Item) * cap_items);
  L.shorts = take(sizeof(nrm::Item) * cap_items);
  L.block_shorts = take(sizeof(nrm::BlockShorts) * nrm::ORDERED_BLOCKS);
  L.lrow_first = take(sizeof(int64_t) * cap_rows);
  L.partials = take(8 * cap_items);
  L.results = take(sizeof(nrm::RowRes) * cap_items);
  // zeroed from here on
  L.small = take(kSmallBytes);
  L.tagged = take(16 * cap_items);
  L.rowtot = take(16 * cap_items);
  L.arrivals = take(4 * cap_items);
  L.tile_tagged = take(16 * cap_items);
  L.tile_total = take(16 * cap_items);
  L.tile_arrivals = take(4 * cap_items);
  L.total = off;
  return L;
}

int reserve(nrm_ctx* c, int64_t rows, int64_t items) {
  BatchWorkspace& w = c->batch;
  if (rows <= w.cap_rows && items <= w.cap_items && w.dev) return NRM_OK;
  int64_t cap_rows = std::max<int64_t>({rows, w.cap_rows, 64});
  int64_t cap_items = std::max<int64_t>({items, w.cap_items, 1024});
  Layout L = layout_for(cap_rows, cap_items);
  // the old buffers may still be in use by enqueued work
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
  destroy_graph(w);
  void* dev = nullptr;
  e = hipMalloc(&dev, L.total);
  if (e != hipSuccess) return fail(NRM_ENOMEM, std::string("batched workspace hipMalloc: ") + hipGetErrorString(e));
  // Row tables: pinned, coherent host memory that the kernels read directly
  // (no copy, no DMA latency per call).
  void* host = nullptr;
  const size_t staging = (size_t)align_up((int64_t)(sizeof(RowDesc) * (size_t)cap_rows), 256);
  e = hipHostMalloc(&host, staging * nrm::kStagingRing, hipHostMallocCoherent | hipHostMallocMapped);
  if (e != hipSuccess) {
    (void)hipFree(dev);  // already failing
    return fail(NRM_ENOMEM, std::string("pinned staging hipHostMalloc: ") + hipGetErrorString(e));
  }
  void* host_dev = nullptr;
  e = hipHostGetDevicePointer(&host_dev, host, 0);
  if (e != hipSuccess) {
    (void)hipFree(dev);
    (void)hipHostFree(host);
    return hip_fail(e, "hipHostGetDevicePointer");
  }
  int err_word = 0;
  if (w.dev) {
    // keep a pending device error of the old workspace
    e = hipMemcpy(&err_word, w.args.error, sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) {  // the old workspace stays as it was
      (void)hipFree(dev);
      (void)hipHostFree(host);
      return hip_fail(e, "hipMemcpy (device error word)");
    }
    (void)hipFree(w.dev);
  }
  if (w.host) (void)hipHostFree(w.host);
  char* d = static_cast<char*>(dev);
  w.dev = dev;
  w.host = host;
  w.staging = staging;
  w.next = 0;
  for (int b = 0; b < nrm::kStagingRing; ++b)
    w.table[b] = reinterpret_cast<RowDesc*>(static_cast<char*>(host_dev) + staging * b);
  BatchArgs& a = w.args;
  a.tiles = reinterpret_cast<nrm::Item*>(d + L.tiles);
  a.shorts = reinterpret_cast<nrm::Item*>(d + L.shorts);
  a.block_shorts = reinterpret_cast<nrm::BlockShorts*>(d + L.block_shorts);
  a.lrow_first = reinterpret_cast<int64_t*>(d + L.lrow_first);
  a.partials = d + L.partials;
  a.results = reinterpret_cast<nrm::RowRes*>(d + L.results);
  a.cnt = reinterpret_cast<int64_t*>(d + L.small);
  a.error = reinterpret_cast<int*>(d + L.small + kErrorOffset);
  a.tagged = reinterpret_cast<unsigned long long*>(d + L.tagged);
  a.rowtot = reinterpret_cast<unsigned long long*>(d + L.rowtot);
  a.arrivals = reinterpret_cast<unsigned*>(d + L.arrivals);
  a.tile_tagged = reinterpret_cast<unsigned long long*>(d + L.tile_tagged);
  a.tile_total = reinterpret_cast<unsigned long long*>(d + L.tile_total);
  a.tile_arrivals = reinterpret_cast<unsigned*>(d + L.tile_arrivals);
  a.cap_rows = cap_rows;
  a.cap_items = cap_items;
  w.cap_rows = cap_rows;
  w.cap_items = cap_items;
  w.dirty = false;
  for (bool& p : w.staged_pending) p = false;
  // the call's words and counters, the tags, totals and arrival counts
  e = hipMemset(d + L.small, 0, L.total - L.small);
  if (e == hipSuccess && err_word) e = hipMemcpy(a.error, &err_word, sizeof(int), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "hipMemset");
  for (hipEvent_t& ev : w.staged)
    if (!ev) {
      e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
      if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
    }
  return NRM_OK;
}

// Items a batch of `rows` rows and at most `elems` elements can need.
int64_t items_bound(const nrm_batch_params& p, int64_t rows, int64_t elems) {
  // a long row has ceil(n / tile) items, a resident row ceil(n / 2^RES_LOG2)
  const int lg = p.resident_segments > 0 ? std::min(p.tile_log2, nrm::RES_LOG2) : p.tile_log2;
  return rows + ceil_div(std::max<int64_t>(elems, 0), int64_t(1) << lg);
}

BatchArgs args_of(const nrm_ctx* c) {
  BatchArgs a = c->batch.args;
  const nrm_batch_params& p = c->bparams;
  a.tile_log2 = p.tile_log2;
  a.tile = int64_t(1) << a.tile_log2;
  a.short_max = short_max_of(p);
  // tiles counted at 4 bytes per element: at most keep_mib MiB for any dtype
  a.keep_tiles = ((int64_t)p.keep_mib << 20) / (a.tile * 4);
  a.wave_max = p.wave_max;
  a.res_on = p.resident_segments > 0;
  a.apart = 0;
  return a;
}

// Whether a batch's listed rows are mostly of one segment each.
bool single_segments(const nrm_batch_params& q, const BatchHeader& h, int64_t mean) {
  return q.resident_segments > 0 && h.run_max == 0 && mean <= int64_t(1) << nrm::RES_LOG2;
}

// The plan of a batch of `rows` rows of at most `elems` elements, the longest
// at most `longest`, cut up as `h` says.
BatchPlan plan_of(const nrm_ctx* c, const BatchHeader& h, int64_t rows, int64_t elems, int64_t longest, int acc) {
  const nrm_batch_params& q = c->bparams;
  BatchPlan p;
  p.acc = acc;
  p.rows_grid = h.grid_x;
  p.rows_grid_y = nrm::rows_grid_y(ceil_div(rows, h.rows_per_block));
  // no row can be longer than those run on the spot: nothing is listed
  p.lists = longest > std::max<int64_t>(h.run_max, q.wave_max);
  // no more blocks than a small batch can list entries: a listed row of more
  // than 2^RES_LOG2 elements has fewer than two entries per 2^RES_LOG2 of them
  p.res_grid = std::min<int64_t>(q.resident_grid, (h.run_max > 0 ? 0 : rows) + 2 * (elems >> nrm::RES_LOG2) + 1);
  // long rows stream better from two blocks per CU (2^26 binary32 in one row:
  // 145 against 148 us; 16 rows of up to 2^24: 64.3 and 66.8 us)
  // and so do listed rows that are single segments, which wait for nothing (30000
  // x 16000: 614 and 660 us; 16000 x 16384 343 and 369; rows of more segments want
  // three, 20000 x 20000 643 and 580)
  if (elems / rows > short_max_of(q) || single_segments(q, h, elems / rows))
    p.res_grid = std::min<int64_t>(p.res_grid, std::max(512, q.resident_segments));
  p.block = q.block;
  p.unroll = q.unroll;
  p.map_unroll = q.map_unroll;
  p.short_regs = q.short_regs;
  p.grid = q.grid;
  p.map_block = q.map_block;
  p.map_grid = q.map_grid;
  return p;
}

// Capture the sequence of a large batch; each replay sets the arguments and
// grid of its first launch (set_rows_node).
int capture_graph(nrm_ctx* c, const BatchPlan& p, const BatchArgs& a, nrm::BatchGraph* out) {
  BatchWorkspace& w = c->batch;
  hipError_t e;
  if (!w.capture_stream) {
    e = hipStreamCreateWithFlags(&w.capture_stream, hipStreamNonBlocking);
    if (e != hipSuccess) return hip_fail(e, "hipStreamCreate");
  }
  e = hipStreamBeginCapture(w.capture_stream, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
  hipError_t e2 = nrm::launch_batch(p, a, w.capture_stream);
  nrm::BatchGraph g;
  e = hipStreamEndCapture(w.capture_stream, &g.graph);
  size_t roots = 1;
  if (e == hipSuccess && e2 == hipSuccess) e = hipGraphGetRootNodes(g.graph, &g.rows, &roots);
  if (e == hipSuccess && e2 == hipSuccess) e = hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0);
  if (e != hipSuccess || e2 != hipSuccess) {
    if (g.graph) (void)hipGraphDestroy(g.graph);  // already failing
    return e2 != hipSuccess ? hip_fail(e2, "batched launch (capture)") : hip_fail(e, "capturing the batched launches");
  }
  *out = g;
  return NRM_OK;
}

hipError_t set_rows_node(const nrm::BatchGraph& g, const BatchPlan& p, BatchArgs a) {
  void* args[] = {&a};
  hipKernelNodeParams k;
  std::memset(&k, 0, sizeof(k));
  k.func = const_cast<void*>(nrm::rows_kernel(p.acc));
  k.gridDim = dim3((unsigned)p.rows_grid, (unsigned)p.rows_grid_y);
  k.blockDim = dim3(nrm::ROWS_BLOCK);
  k.kernelParams = args;
  return hipGraphExecKernelNodeSetParams(g.exec, g.rows, &k);
}

// How batch_rows_kernel is cut up; the results are the same. A wavefront costs
// the dispatcher about 0.4 ns, so many short rows go four to a wavefront (2^20
// rows of 64 binary32: 159 us with 32 rows per block, 489 us with 8). Rows of
// several hundred elements, up to about the longest that a wavefront takes, get
// one each: 8 per block (2^18 x 1000: 350 us, with 32 377 us; 65536 x 1536 133 us, 4
// per block 170; 2^17 x 2048 bfloat16 177 and 244; of binary32 of that length those
// in whole lines gain, 2^17 x 2048 365 and 402, others lose, 2^17 x 2000 387 and
// 374, and keep 4 per block). Longer rows are run by
// the block and take turns in it: 4 per block (65536 x 3000 290 us, 8 per block
// 299), and from 4096 elements on nearly a block each: 16384 x 10000 in 237 us
// with 2 per block, 257 us with 4, and 4 log-uniform up to 65536 in 288 and 280 us
// (2-byte inputs would keep 8 per block up to 4096 elements: 32768 x 4096 bfloat16
// 140 us, 2 per block 156); and a batch of few rows one block per row.
//
// Where the mean row is of more than 2^RES_LOG2 elements, most are in listed
// rows, and so are those of wave_max < n <= 2^RES_LOG2 then. The listed segments
// are taken in row order where the batch has at most ORDERED_BLOCKS blocks: many
// such rows go 32 per block (16384 x 20000: 475 us, 8 per block 489, run by their
// blocks 2 at a time 590; 12000 of 32 to 2^18 482, 493 and 537; 7895 x 17000 230,
// 235 and 276). In large batches of binary32 in and out the same pays from three
// quarters of that mean on (16384 rows of 32 to 2^17: 372 us listed, 404 us run;
// 39431 x 13074 647 and 755), from 2^27 elements on from two thirds (36363 x 11000
// 545 and 569; 6100 x 11000 103 and 97), not in small ones (2000 x 12000: 50 and 38) nor where
// a segment is fewer bytes (10000 x 13074 to bfloat16: 165 and 138; 13421 x 10000
// bfloat16: 191 and 103). Above 2^14 2-byte rows gain like the others if they are
// alike (16384 x 20000 bfloat16 443 us listed, 533 run), and lose if most are below
// it (14532 rows of 1320 to 71892 float16, mean 17806: 323 and 299).
// Below that it depends on how the lengths spread, which the host does not know
// (32768 rows of 32 to 2^16, mean 8600: 398 listed, 447 run; 16384 x 8192: 239 and
// 194).
// Without resident rows the single-pass rows are run here whatever the batch is
// (listed they take another kernel, whose sums have another order): 65536 x 4096
// 363 us, 533 listed; 200,000 up to 4096 167 us, 291 listed.
void cut_rows(const nrm_batch_params& p, int64_t rows, int64_t elems, BatchHeader* h) {
  const int64_t mean = elems / rows;
  const int64_t block_max = int64_t(1) << nrm::RES_LOG2;
  const bool f32 = h->mode == nrm::BATCH_CSR && h->csr_in_dt == NRM_F32 && h->csr_out_dt == NRM_F32;
  const int64_t listed_mean = f32 && elems >= (int64_t(1) << 27)   ? block_max / 3 * 2
                              : f32 && elems >= (int64_t(1) << 26) ? block_max / 4 * 3
                                                                   : block_max + 1;
  const int64_t wave_mean = h->mode == nrm::BATCH_CSR && nrm::dtype_size(h->csr_in_dt) == 2 ? nrm::WAVE_MAX_ELEMS
                                                                                        : nrm::WAVE_MAX_ELEMS / 8 * 7;
  h->run_max = std::min(block_max, short_max_of(p));
  if (rows <= 512) {
    h->rows_per_block = 1;
  } else if (mean >= listed_mean) {
    h->rows_per_block = rows <= 4096 ? nrm::ROWS_WAVES : nrm::ROWS_MAX;
    if (p.resident_segments > 0) h->run_max = 0;
  } else {
    h->rows_per_block = mean >= 4096                 ? 2
                        : mean > wave_mean           ? 4
                        : mean > 512 || rows <= 4096 ? nrm::ROWS_WAVES
                                                     : nrm::ROWS_MAX;
  }
  h->grid_x = nrm::rows_grid_x(ceil_div(rows, h->rows_per_block));
}

// After a failed launch: the rows' kernel may have run without the launches
// that take its lists' entries and zero the counters, and the next call would
// append behind entries that point at the failed call's arrays.
int empty_lists(BatchWorkspace& w) {
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess)
    e = hipMemset(w.args.cnt + nrm::CNT_SET0, 0, sizeof(int64_t) * (nrm::CNT_COUNT - nrm::CNT_SET0));
  if (e != hipSuccess) return hip_fail(e, "emptying the work lists after a failed launch");
  w.dirty = false;
  return NRM_OK;
}

// A row table of its own for a call that a caller's graph captures: the
// replays read it in place, whatever later calls stage. Held until the context
// is destroyed.
int keep_table(BatchWorkspace& w, const nrm_row* table, int64_t nrows, const RowDesc** dev) {
  const size_t bytes = sizeof(RowDesc) * (size_t)nrows;
  void *host = nullptr, *view = nullptr;
  // allocating is not a stream operation: allowed beside any kind of capture
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  hipError_t e = hipThreadExchangeStreamCaptureMode(&mode);
  if (e != hipSuccess) return hip_fail(e, "hipThreadExchangeStreamCaptureMode");
  e = hipHostMalloc(&host, bytes, hipHostMallocCoherent | hipHostMallocMapped);
  const hipError_t e2 = hipThreadExchangeStreamCaptureMode(&mode);  // the caller's again
  if (e != hipSuccess) return fail(NRM_ENOMEM, std::string("pinned row table hipHostMalloc: ") + hipGetErrorString(e));
  w.captured.push_back(host);
  if (e2 != hipSuccess) return hip_fail(e2, "hipThreadExchangeStreamCaptureMode");
  e = hipHostGetDevicePointer(&view, host, 0);
  if (e != hipSuccess) return hip_fail(e, "hipHostGetDevicePointer");
  std::memcpy(host, table, bytes);
  *dev = static_cast<const RowDesc*>(view);
  return NRM_OK;
}

// Run the launch sequence on `s` for a batch of at most `elems` elements whose
// longest row has at most `longest`; `wide`: some rows' outputs are wider than
// their inputs. A row table is staged in the next ring buffer first.
int run_batch(nrm_ctx* c, const BatchHeader& h, const nrm_row* table, int64_t nrows, int64_t elems, int64_t longest,
              bool wide, int acc, hipStream_t s) {
  BatchWorkspace& w = c->batch;
  hipError_t e;
  if (w.dirty) {
    int st = empty_lists(w);
    if (st != NRM_OK) return st;
  }
  BatchArgs a = args_of(c);
  a.header = h;
  cut_rows(c->bparams, nrows, elems, &a.header);
  BatchPlan p = plan_of(c, a.header, nrows, elems, longest, acc);
  a.apart = apart_rows(a, elems, elems / nrows, wide);
  if (a.apart) p.map_grid = std::max(p.map_grid, apart_map_grid(elems, acc));
  // (a replay has the persistent blocks that it was captured with)
  bool replay = c->bparams.graph && elems >= kGraphElems && !a.apart &&
                !single_segments(c->bparams, a.header, elems / nrows);
  bool ring = replay || table;
  if (ring) {
    hipStreamCaptureStatus state = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &state) != hipSuccess) {
      // (the null stream beside a capture on a blocking one): the launch says so
      (void)hipGetLastError();
      state = hipStreamCaptureStatusNone;
    }
    if (state != hipStreamCaptureStatusNone) {
      // the launches themselves go into the caller's graph (a graph launched
      // on a capturing stream leaves it empty)
      replay = ring = false;
      if (table) {
        int st = keep_table(w, table, nrows, &a.header.table);
        if (st != NRM_OK) return st;
      }
    }
  }
  const int buf = w.next;
  if (ring && w.staged_pending[buf]) {  // the call that used this buffer or graph before must be done with it
    e = hipEventSynchronize(w.staged[buf]);
    if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize");
    w.staged_pending[buf] = false;
  }
  if (ring && table) {
    std::memcpy(static_cast<char*>(w.host) + w.staging * buf, table, sizeof(RowDesc) * (size_t)nrows);
    a.header.table = w.table[buf];
  }
  hipEvent_t* ev = nullptr;
  if (c->timing) {
    ev = &w.events[2 * (w.timed_calls % nrm::kTimingRing)];
    w.timed_calls++;
    (void)hipEventRecord(ev[0], s);  // timing only
  }
  if (replay) {
    // the sequence of any large batch: all launches, the lists' at full size
    p.lists = true;
    p.res_grid = c->bparams.resident_grid;
    nrm::BatchGraph& g = w.graph[acc][buf];
    if (!g.exec) {
      int st = capture_graph(c, p, a, &g);
      if (st != NRM_OK) return st;
    }
    e = set_rows_node(g, p, a);
    if (e != hipSuccess) return hip_fail(e, "hipGraphExecKernelNodeSetParams");
    e = hipGraphLaunch(g.exec, s);
  } else {
    e = nrm::launch_batch(p, a, s);
  }
  if (e != hipSuccess) {
    w.dirty = true;
    return hip_fail(e, replay ? "hipGraphLaunch" : "batched kernel launch");
  }
  if (ev) (void)hipEventRecord(ev[1], s);
  if (ring) {
    e = hipEventRecord(w.staged[buf], s);
    if (e != hipSuccess) return hip_fail(e, "hipEventRecord");
    w.staged_pending[buf] = true;
    w.next = (buf + 1) % nrm::kStagingRing;
  }
  return NRM_OK;
}

bool valid_dtype(int dt) { return dt == NRM_F32 || dt == NRM_BF16 || dt == NRM_F16; }

}  // namespace

namespace nrm {
void batch_free(nrm_ctx* c) {
  BatchWorkspace& w = c->batch;
  destroy_graph(w);
  if (w.capture_stream) (void)hipStreamDestroy(w.capture_stream);
  for (hipEvent_t ev : w.staged)
    if (ev) (void)hipEventDestroy(ev);
  for (hipEvent_t ev : w.events) (void)hipEventDestroy(ev);
  if (w.dev) (void)hipFree(w.dev);
  if (w.host) (void)hipHostFree(w.host);
  for (void* p : w.captured) (void)hipHostFree(p);
  w = BatchWorkspace();
}
}  // namespace nrm

extern "C" {

int nrm_default_batch_params(nrm_batch_params* params) {
  if (!params) return fail(NRM_EINVAL, "NULL argument");
  *params = default_batch_params();
  return NRM_OK;
}

int nrm_set_batch_params(nrm_ctx* c, const nrm_batch_params* params) {
  if (!c || !params) return fail(NRM_EINVAL, "NULL argument");
  nrm::CtxLock lk(c->mu);
  int st = check_batch_params(*params);
  if (st != NRM_OK) return st;
  if (std::memcmp(params, &c->bparams, sizeof(*params)) != 0) {
    DeviceGuard g(c->device);
    if (any_graph(c->batch)) {
      hipError_t e = hipDeviceSynchronize();  // a replay may still be running
      if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
      destroy_graph(c->batch);
    }
    c->bparams = *params;
  }
  return NRM_OK;
}

int nrm_get_batch_params(const nrm_ctx* c, nrm_batch_params* params) {
  if (!c || !params) return fail(NRM_EINVAL, "NULL argument");
  nrm::CtxLock lk(c->mu);
  *params = c->bparams;
  return NRM_OK;
}

int nrm_batch_reserve(nrm_ctx* c, int64_t max_rows, int64_t max_elems) {
  if (!c) return fail(NRM_EINVAL, "ctx is NULL");
  nrm::CtxLock lk(c->mu);
  if (max_rows < 0 || max_elems < 0) return fail(NRM_EINVAL, "negative reservation");
  if (max_rows > INT32_MAX) return fail(NRM_EINVAL, "more than 2^31 - 1 rows");
  DeviceGuard g(c->device);
  return reserve(c, max_rows, items_bound(c->bparams, max_rows, max_elems));
}

namespace {
int check_csr_buffers(const void* out, int out_dtype, const void* in, int in_dtype, int64_t capacity) {
  const int64_t si = nrm::dtype_size(in_dtype), so = nrm::dtype_size(out_dtype);
  if (!in || !out) return fail(NRM_EINVAL, "NULL data pointer");
  if (capacity > INT64_MAX / 8) return fail(NRM_EINVAL, "capacity too large");
  if ((reinterpret_cast<uintptr_t>(in) % si) || (reinterpret_cast<uintptr_t>(out) % so))
    return fail(NRM_EINVAL, "in or out is not aligned to its element size");
  uintptr_t a0 = (uintptr_t)in, a1 = a0 + (uintptr_t)(capacity * si);
  uintptr_t b0 = (uintptr_t)out, b1 = b0 + (uintptr_t)(capacity * so);
  if (a0 < b1 && b0 < a1 && !(a0 == b0 && si == so))
    return fail(NRM_EOVERLAP, "in and out overlap without being the same array");
  return NRM_OK;
}
}  // namespace

namespace {
// lse[rows] must not overlap in or out (capacity elements each).
int check_lse(const void* out, int out_dtype, const void* in, int in_dtype, int64_t capacity, const float* lse,
              int64_t rows) {
  const int64_t si = nrm::dtype_size(in_dtype), so = nrm::dtype_size(out_dtype);
  const uintptr_t l0 = (uintptr_t)lse, l1 = l0 + (uintptr_t)(rows * (int64_t)sizeof(float));
  const uintptr_t a0 = (uintptr_t)in, a1 = a0 + (uintptr_t)(capacity * si);
  const uintptr_t b0 = (uintptr_t)out, b1 = b0 + (uintptr_t)(capacity * so);
  if ((l0 < a1 && a0 < l1) || (l0 < b1 && b0 < l1)) return fail(NRM_EOVERLAP, "lse overlaps in or out");
  return NRM_OK;
}

// The CSR form of both operations: validation before any HIP call, the
// capacity read from offsets[rows] when not given, then one batched run of
// the reduction kind `acc` (with lse written for softmax when non-NULL).
int run_csr(nrm_ctx* c, void* out, int out_dtype, const void* in, int in_dtype, const int64_t* offsets,
            int64_t rows, int64_t capacity, int acc, float* lse, void* stream) {
  if (rows < 0) return fail(NRM_EINVAL, "rows < 0");
  if (!valid_dtype(in_dtype) || !valid_dtype(out_dtype)) return fail(NRM_EINVAL, "unknown dtype");
  if (rows == 0) return NRM_OK;
  if (rows > INT32_MAX) return fail(NRM_EINVAL, "more than 2^31 - 1 rows");
  if (!offsets) return fail(NRM_EINVAL, "offsets is NULL");
  if (lse && (reinterpret_cast<uintptr_t>(lse) % sizeof(float)))
    return fail(NRM_EINVAL, "lse is not aligned to 4 bytes");
  if (capacity == 0 && !lse) return NRM_OK;  // every row is empty (or invalid)
  if (capacity > 0) {
    int st = check_csr_buffers(out, out_dtype, in, in_dtype, capacity);
    if (st == NRM_OK && lse) st = check_lse(out, out_dtype, in, in_dtype, capacity, lse, rows);
    if (st != NRM_OK) return st;
  }
  if (!c) {
    int st = nrm::default_ctx(&c);
    if (st != NRM_OK) return st;
  }
  nrm::CtxLock lk(c->mu);
  DeviceGuard g(c->device);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (capacity < 0) {
    int64_t last = 0;
    hipError_t e = hipMemcpyAsync(&last, offsets + rows, sizeof(int64_t), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "reading offsets[rows]");
    if (last <= 0 && !lse) return NRM_OK;
    capacity = last > 0 ? last : 0;
    if (capacity > 0) {
      int st = check_csr_buffers(out, out_dtype, in, in_dtype, capacity);
      if (st != NRM_OK) return st;
    }
  }
  if (lse && capacity > 0) {
    int st = check_lse(out, out_dtype, in, in_dtype, capacity, lse, rows);
    if (st != NRM_OK) return st;
  }
  int st = reserve(c, rows, items_bound(c->bparams, rows, capacity));
  if (st != NRM_OK) return st;
  BatchHeader h;
  std::memset(&h, 0, sizeof(h));
  h.nrows = rows;
  h.mode = nrm::BATCH_CSR;
  h.csr_in_dt = in_dtype;
  h.csr_out_dt = out_dtype;
  h.offsets = offsets;
  h.csr_in = static_cast<const char*>(in);
  h.csr_out = static_cast<char*>(out);
  h.capacity = capacity;
  h.lse = lse;
  const bool wide = nrm::dtype_size(out_dtype) > nrm::dtype_size(in_dtype);
  return run_batch(c, h, nullptr, rows, capacity, capacity, wide, acc, s);
}
}  // namespace

int nrm_normalize_batched_ex(nrm_ctx* c, void* out, int out_dtype, const void* in, int in_dtype,
                             const int64_t* offsets, int64_t rows, int64_t capacity, int accum,
                             void* stream) {
  if (accum != NRM_ACC_F32 && accum != NRM_ACC_KAHAN) return fail(NRM_EINVAL, "unknown accumulation mode");
  return run_csr(c, out, out_dtype, in, in_dtype, offsets, rows, capacity, accum, nullptr, stream);
}

int nrm_softmax_batched(nrm_ctx* c, float* out, const float* in, const int64_t* offsets, int64_t rows,
                        int64_t capacity, float* lse, void* stream) {
  return run_csr(c, out, NRM_F32, in, NRM_F32, offsets, rows, capacity, nrm::ACC_SOFTMAX, lse, stream);
}

int normalize_batched(float* out, const float* in, const int64_t* offsets, int64_t rows) {
  return nrm_normalize_batched_ex(nullptr, out, NRM_F32, in, NRM_F32, offsets, rows, -1, NRM_ACC_F32, nullptr);
}

int nrm_normalize_rows(nrm_ctx* c, const nrm_row* rows, int64_t nrows, int accum, void* stream) {
  if (nrows < 0) return fail(NRM_EINVAL, "nrows < 0");
  if (accum != NRM_ACC_F32 && accum != NRM_ACC_KAHAN) return fail(NRM_EINVAL, "unknown accumulation mode");
  if (nrows == 0) return NRM_OK;
  if (nrows > INT32_MAX) return fail(NRM_EINVAL, "more than 2^31 - 1 rows");
  if (!rows) return fail(NRM_EINVAL, "rows is NULL");
  int64_t total = 0, longest = 0;
  bool wide = false;
  for (int64_t r = 0; r < nrows; ++r) {
    const nrm_row& d = rows[r];
    if (d.n < 0) return fail(NRM_EINVAL, "row with n < 0");
    if (!valid_dtype(d.in_dtype) || !valid_dtype(d.out_dtype)) return fail(NRM_EINVAL, "row with unknown dtype");
    if (d.n == 0) continue;
    if (!d.in || !d.out) return fail(NRM_EINVAL, "row with NULL data pointer");
    const int64_t si = nrm::dtype_size(d.in_dtype), so = nrm::dtype_size(d.out_dtype);
    if ((reinterpret_cast<uintptr_t>(d.in) % si) || (reinterpret_cast<uintptr_t>(d.out) % so))
      return fail(NRM_EINVAL, "row pointer not aligned to its element size");
    uintptr_t a0 = (uintptr_t)d.in, a1 = a0 + (uintptr_t)(d.n * si);
    uintptr_t b0 = (uintptr_t)d.out, b1 = b0 + (uintptr_t)(d.n * so);
    if (a0 < b1 && b0 < a1 && !(a0 == b0 && si == so))
      return fail(NRM_EOVERLAP, "a row's in and out overlap without being the same array");
    total += d.n;
    longest = std::max(longest, d.n);
    wide = wide || so > si;
  }
  if (!c) {
    int st = nrm::default_ctx(&c);
    if (st != NRM_OK) return st;
  }
  nrm::CtxLock lk(c->mu);
  if (longest > (int64_t(1) << c->bparams.tile_log2) * nrm::MAX_ROW_TILES)
    return fail(NRM_EINVAL, "row too long for the batched path's tile size");
  DeviceGuard g(c->device);
  int st = reserve(c, nrows, items_bound(c->bparams, nrows, total));
  if (st != NRM_OK) return st;
  BatchHeader h;
  std::memset(&h, 0, sizeof(h));
  h.nrows = nrows;
  h.mode = nrm::BATCH_TABLE;
  return run_batch(c, h, rows, nrows, total, longest, wide, accum, static_cast<hipStream_t>(stream));
}

int nrm_get_device_error(nrm_ctx* c, void* stream) {
  if (!c) {
    int st = nrm::default_ctx(&c);
    if (st != NRM_OK) return st;
  }
  nrm::CtxLock lk(c->mu);
  DeviceGuard g(c->device);
  hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  // the batched workspace's word and the context's word of the other kernels
  int word = 0;
  for (int* p : {c->batch.dev ? c->batch.args.error : nullptr, c->dev_error}) {
    if (!p) continue;
    int w = 0;
    e = hipMemcpy(&w, p, sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "reading the device error flag");
    if (w) {
      e = hipMemset(p, 0, sizeof(int));
      if (e != hipSuccess) return hip_fail(e, "clearing the device error flag");
    }
    word |= w;
  }
  if (!word) return NRM_OK;
  if (word & nrm::NRM_DEVERR_STALL) {
    // a wait that gave up may have left arrival counts behind: start them over
    if (c->batch.dev) {
      e = hipMemset(c->batch.args.arrivals, 0, sizeof(unsigned) * (size_t)c->batch.cap_items);
      if (e == hipSuccess)
        e = hipMemset(c->batch.args.tile_arrivals, 0, sizeof(unsigned) * (size_t)c->batch.cap_items);
    }
    if (e != hipSuccess) return hip_fail(e, "clearing the arrival counts");
  }
  std::string why;
  if (word & nrm::NRM_DEVERR_OFFSETS) why += "CSR offsets negative, decreasing or past capacity; ";
  if (word & nrm::NRM_DEVERR_ROW) why += "invalid table row or row with too many tiles; ";
  if (word & nrm::NRM_DEVERR_CAPACITY) why += "batch larger than the workspace; ";
  if (word & nrm::NRM_DEVERR_TARGET) why += "NLL target outside [0, classes); ";
  if (word & nrm::NRM_DEVERR_STALL) why += "a resident row's segment sums did not all arrive within the spin limit; ";
  return fail(NRM_EDEVICE, why + "those rows or samples were skipped");
}

int nrm_batch_times(nrm_ctx* c, double* total_ms, int64_t* calls) {
  if (!c) return fail(NRM_EINVAL, "ctx is NULL");
  nrm::CtxLock lk(c->mu);
  BatchWorkspace& w = c->batch;
  double t = 0;
  int64_t k = std::min<int64_t>(w.timed_calls, nrm::kTimingRing);
  for (int64_t i = 0; i < k; ++i) {
    hipError_t e = hipEventSynchronize(w.events[2 * i + 1]);
    if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize");
    float ms = 0;
    e = hipEventElapsedTime(&ms, w.events[2 * i], w.events[2 * i + 1]);
    if (e != hipSuccess) return hip_fail(e, "hipEventElapsedTime");
    t += ms;
  }
  if (total_ms) *total_ms = t;
  if (calls) *calls = k;
  return NRM_OK;
}

}  // extern "C"
