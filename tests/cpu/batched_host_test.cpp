// CPU tests of the batched path's host code (paper_2207_00257_amd/csrc/
// nrm_batched_api.cpp, included below so that its file-local rules can be
// called): a HIP runtime over host memory, and a launch that records what it
// is given, stand in for the GPU. Built with g++ and run, one test per process,
// by tests/test_batched_host_cpu.py. Exit status 0: passed.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <functional>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "nrm_batched_api.cpp"

static int g_failures = 0;
#define CHECK(cond)                                                          \
  do {                                                                       \
    if (!(cond)) {                                                           \
      fprintf(stderr, "%s:%d: CHECK failed: %s\n", __FILE__, __LINE__, #cond); \
      ++g_failures;                                                          \
    }                                                                        \
  } while (0)

// ---- the stand-ins -----------------------------------------------------------------

static BatchPlan g_plan;   // what the last launch was given
static BatchArgs g_args;
static int g_launches = 0;
static bool g_capturing = false;
static std::function<hipError_t(const BatchPlan&, const BatchArgs&)> g_launch;

namespace nrm {
std::string& last_error() {
  static std::string text;
  return text;
}
int default_ctx(nrm_ctx**) { return NRM_EINVAL; }
const void* rows_kernel(int) { return nullptr; }
hipError_t launch_batch(const BatchPlan& p, const BatchArgs& a, hipStream_t) {
  g_plan = p;
  g_args = a;
  ++g_launches;
  return g_launch ? g_launch(p, a) : hipSuccess;
}
}  // namespace nrm

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  static hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
  std::swap(mode, *m);
  return hipSuccess;
}
// no graph can be made here: tests use batches that are launched directly
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphGetRootNodes(hipGraph_t, hipGraphNode_t*, size_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecKernelNodeSetParams(hipGraphExec_t, hipGraphNode_t, const hipKernelNodeParams*) {
  return hipErrorNotSupported;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

struct Ctx : nrm_ctx {
  Ctx() { bparams = default_batch_params(); }
  ~Ctx() { nrm::batch_free(this); }
};

// ---- tests -------------------------------------------------------------------------

// Whatever a batch has rows and elements, its first launch is one that the
// hardware takes (fewer than 2^32 threads in each dimension) and that has a
// block for every row.
static void test_rows_grid() {
  Ctx c;
  for (int segments : {64, 0}) {
    c.bparams.resident_segments = segments;
    for (int64_t rows : {int64_t(1), int64_t(512), int64_t(513), int64_t(5000), (int64_t(1) << 20) - 1, int64_t(1) << 21,
                         (int64_t(1) << 21) + 1, (int64_t(1) << 24) + 7, int64_t(1) << 25, int64_t(1) << 28,
                         (int64_t(1) << 28) + 1, int64_t(INT32_MAX)})
      for (int64_t mean : {0, 1, 17, 256, 600, 2048, 4096, 20000, 1 << 21}) {
        const int64_t elems = rows * mean;
        BatchHeader h;
        memset(&h, 0, sizeof(h));
        h.nrows = rows;
        cut_rows(c.bparams, rows, elems, &h);
        const BatchPlan p = plan_of(&c, h, rows, elems, elems, NRM_ACC_F32);
        CHECK(p.rows_grid >= 1 && p.rows_grid * nrm::ROWS_BLOCK < int64_t(1) << 32);
        CHECK(p.rows_grid_y >= 1 && p.rows_grid_y <= 65535);
        CHECK(h.grid_x == p.rows_grid);
        CHECK(p.rows_grid * p.rows_grid_y * h.rows_per_block >= rows);
        CHECK((p.rows_grid * p.rows_grid_y - p.rows_grid_y) * h.rows_per_block < rows);  // hardly any without rows
        CHECK(p.res_grid >= 1 && p.res_grid <= c.bparams.resident_grid);
      }
  }
}

// A captured call's replays see its own row table, whatever was staged since,
// and a large batch on a capturing stream is launched, not replayed.
static void test_captured_tables() {
  Ctx c;
  std::vector<float> in(100000), out(100000);
  auto call = [&](int64_t first, int64_t n) {
    std::vector<nrm_row> rows(3);
    for (int64_t k = 0; k < 3; ++k) {
      rows[k].in = in.data() + first + k * n;
      rows[k].out = out.data() + first + k * n;
      rows[k].n = n;
      rows[k].in_dtype = rows[k].out_dtype = NRM_F32;
    }
    CHECK(nrm_normalize_rows(&c, rows.data(), 3, NRM_ACC_F32, nullptr) == NRM_OK);
    CHECK(g_args.header.table[2].n == n);
    return g_args.header.table;
  };
  call(0, 5);
  g_capturing = true;
  std::vector<const RowDesc*> captured;
  for (int k = 0; k < 6; ++k) captured.push_back(call(100 * k, 10 + k));
  g_capturing = false;
  for (int k = 0; k < 9; ++k) call(50000, 1000 + k);
  CHECK(nrm_batch_reserve(&c, 1 << 16, 1 << 20) == NRM_OK);
  call(50000, 7);
  for (int k = 0; k < 6; ++k)
    for (int r = 0; r < 3; ++r) {
      CHECK(captured[k][r].n == 10 + k);
      CHECK(captured[k][r].in == reinterpret_cast<const char*>(in.data() + 100 * k + r * (10 + k)));
    }
  const int launches = g_launches;
  const std::vector<int64_t> offsets(1001, 0);
  CHECK(nrm_normalize_batched_ex(&c, in.data(), NRM_F32, in.data(), NRM_F32, offsets.data(), 1000, kGraphElems, NRM_ACC_F32,
                                 nullptr) != NRM_OK);  // a replay: no graph can be made here
  g_capturing = true;
  CHECK(nrm_normalize_batched_ex(&c, in.data(), NRM_F32, in.data(), NRM_F32, offsets.data(), 1000, kGraphElems, NRM_ACC_F32,
                                 nullptr) == NRM_OK);
  g_capturing = false;
  CHECK(g_launches == launches + 1 && g_args.header.offsets == offsets.data());
}

// A call whose later launches fail leaves its list entries behind: the next
// call finds the lists empty.
static void test_failed_launch() {
  Ctx c;
  std::vector<float> in(1 << 16);
  const int64_t offsets[2] = {0, 1 << 16};
  auto call = [&] {
    return nrm_normalize_batched_ex(&c, in.data(), NRM_F32, in.data(), NRM_F32, offsets, 1, 1 << 16, NRM_ACC_F32, nullptr);
  };
  auto listed = [](const BatchArgs& a) {
    int64_t n = 0;
    for (int set = 0; set < 2; ++set)
      for (int k = 0; k < nrm::LIST_COUNTERS; ++k) n += a.cnt[nrm::CNT_SET0 + set * nrm::CNT_SET_STRIDE + k * nrm::CNT_LINE];
    return n;
  };
  CHECK(call() == NRM_OK);
  for (int set = 0; set < 2; ++set) {
    g_launch = [&](const BatchPlan&, const BatchArgs& a) {
      CHECK(listed(a) == 0);
      for (int k = 0; k < nrm::LIST_COUNTERS; ++k) a.cnt[nrm::CNT_SET0 + set * nrm::CNT_SET_STRIDE + k * nrm::CNT_LINE] = 4;
      return hipErrorLaunchFailure;
    };
    CHECK(call() == NRM_EHIP);
  }
  g_launch = [&](const BatchPlan&, const BatchArgs& a) {
    CHECK(listed(a) == 0);
    return hipSuccess;
  };
  CHECK(call() == NRM_OK);
  g_launch = nullptr;
}

// No array of the workspace reaches into another. The tagged words are then
// written by publishing alone: plain floats among them (the partials and results
// of calls without resident rows) could pass for a later call's.
static void test_workspace_layout() {
  Ctx c;
  for (int64_t rows : {1, 1000, 70000}) {
    CHECK(nrm_batch_reserve(&c, rows, rows * 100000) == NRM_OK);
    const BatchArgs& a = c.batch.args;
    const size_t n = (size_t)a.cap_items;
    const struct {
      const void* at;
      size_t bytes;
    } arrays[] = {{a.tiles, sizeof(nrm::Item) * n},
                  {a.shorts, sizeof(nrm::Item) * n},
                  {a.block_shorts, sizeof(nrm::BlockShorts) * nrm::ORDERED_BLOCKS},
                  {a.lrow_first, sizeof(int64_t) * (size_t)a.cap_rows},
                  {a.cnt, sizeof(int64_t) * nrm::CNT_COUNT},
                  {a.error, sizeof(int)},
                  {a.partials, 8 * n},
                  {a.results, sizeof(nrm::RowRes) * n},
                  {a.tagged, 16 * n},
                  {a.rowtot, 16 * n},
                  {a.arrivals, 4 * n},
                  {a.tile_tagged, 16 * n},
                  {a.tile_total, 16 * n},
                  {a.tile_arrivals, 4 * n}};
    const size_t total = layout_for(a.cap_rows, a.cap_items).total;
    for (const auto& x : arrays) {
      CHECK((const char*)x.at >= (const char*)c.batch.dev && (const char*)x.at + x.bytes <= (const char*)c.batch.dev + total);
      for (const auto& y : arrays)
        CHECK(&x == &y || (const char*)x.at + x.bytes <= (const char*)y.at || (const char*)y.at + y.bytes <= (const char*)x.at);
    }
    for (const unsigned long long* tagged : {a.tagged, a.rowtot, a.tile_tagged, a.tile_total})
      for (size_t k = 0; k < 2 * n; ++k) CHECK(tagged[k] == 0);
  }
}

// The published error bound is that of a summation tree of height 62, for every
// tile size that the parameters take.
static void test_tree_height() {
  Ctx c;
  for (int t = 10; t <= 22; ++t) {
    nrm_batch_params p = c.bparams;
    p.tile_log2 = t;
    CHECK(t >= 18 || check_batch_params(p) == NRM_OK);
    CHECK(nrm::long_row_height(t) <= 62);
  }
  nrm_batch_params p = c.bparams;
  p.tile_log2 = 22;
  p.block = 1024;
  p.unroll = 8;
  CHECK(check_batch_params(p) == NRM_OK);
}

// Rows of about a segment are listed in large batches of binary32 in and out, on
// two blocks per CU and without a replay; elsewhere they are run by their blocks.
static void test_cuts_of_one_segment_rows() {
  Ctx c;
  const std::vector<int64_t> offsets(40001, 0);
  auto cut = [&](int64_t rows, int64_t mean, int in_dt, int out_dt) {
    const int64_t half = int64_t(1) << 45;  // addresses only: nothing is read here
    CHECK(nrm_normalize_batched_ex(&c, reinterpret_cast<void*>(half + half / 2), out_dt, reinterpret_cast<void*>(half), in_dt,
                                   offsets.data(), rows, rows * mean, NRM_ACC_F32, nullptr) == NRM_OK);
    return g_args.header.run_max == 0;
  };
  for (int64_t mean : {12288, 13074, 16384}) {
    CHECK(cut(40000, mean, NRM_F32, NRM_F32) && g_args.header.rows_per_block == nrm::ROWS_MAX && g_plan.res_grid == 512);
    CHECK(cut(5462, mean, NRM_F32, NRM_F32) && g_plan.res_grid == 512);
    c.bparams.graph = 0;
    CHECK(!cut(40000, mean, NRM_F32, NRM_BF16) && g_args.header.rows_per_block == 2);
    CHECK(!cut(40000, mean, NRM_BF16, NRM_BF16) && !cut(2000, mean, NRM_F32, NRM_F32));
    c.bparams.graph = 1;
  }
  c.bparams.graph = 0;
  CHECK(cut(40000, 10922, NRM_F32, NRM_F32) && !cut(40000, 10921, NRM_F32, NRM_F32));  // 2^27 elements and more
  CHECK(cut(6000, 12288, NRM_F32, NRM_F32) && !cut(6000, 12287, NRM_F32, NRM_F32));    // 2^26 and more
  CHECK(cut(40000, 16385, NRM_BF16, NRM_BF16) && g_plan.res_grid == 768);
}

// Without resident rows a single-pass row of at most 2^RES_LOG2 elements is run by
// its block in every batch (its bits must not depend on the other rows), and
// batches of short rows are cut up as they are with resident rows.
static void test_cuts_without_resident_rows() {
  Ctx on, off;
  off.bparams.resident_segments = 0;
  for (const auto& shape : std::vector<std::pair<int, int>>{{256, 4}, {1024, 8}, {64, 1}}) {
    off.bparams.block = shape.first;
    off.bparams.short_regs = shape.second;
    const int64_t run = std::min<int64_t>(shape.first * shape.second * 4, int64_t(1) << nrm::RES_LOG2);
    for (int64_t rows : {1, 512, 513, 4096, 4097, 200000, 1 << 20})
      for (int64_t mean : {0, 17, 256, 600, 2048, 5000, 20000, 40000, 1 << 21}) {
        BatchHeader a, b;
        memset(&a, 0, sizeof(a));
        memset(&b, 0, sizeof(b));
        cut_rows(on.bparams, rows, rows * mean, &a);
        cut_rows(off.bparams, rows, rows * mean, &b);
        CHECK(b.run_max == run);
        CHECK(b.rows_per_block == a.rows_per_block);
      }
  }
}

// Which batches run their long rows in launches of their own: never without
// resident rows, never a small batch or one of short rows, and then not as a replay.
static void test_apart_rule() {
  Ctx c;
  std::vector<float> in(16);
  const std::vector<int64_t> offsets(100001, 0);
  auto apart = [&](int64_t rows, int64_t capacity, int in_dt, int out_dt) {
    const int64_t half = int64_t(1) << 45;  // addresses only: nothing is read here
    void* from = reinterpret_cast<void*>(half);
    void* to = reinterpret_cast<void*>(half + half / 2);
    return nrm_normalize_batched_ex(&c, to, out_dt, from, in_dt, offsets.data(), rows, capacity, NRM_ACC_F32, nullptr) ==
               NRM_OK && g_args.apart;
  };
  const int64_t b = kApartElems, w = kApartElemsWide;
  c.bparams.graph = 0;
  CHECK(!apart(63, b - 1, NRM_F32, NRM_F32) && apart(63, b, NRM_F32, NRM_F32) && apart(63, b, NRM_BF16, NRM_BF16));
  CHECK(!apart(64, b, NRM_F32, NRM_F32));  // mean 2^20
  CHECK(apart(1, b, NRM_F32, NRM_BF16) && !apart(1, b, NRM_BF16, NRM_F32) && !apart(1, w - 1, NRM_F16, NRM_F32));
  CHECK(apart(1, w, NRM_BF16, NRM_F32));
  CHECK(apart(511, w, NRM_F32, NRM_F32) && g_plan.map_grid == 2048 && !apart(512, w, NRM_F32, NRM_F32));  // mean 2^18
  CHECK(apart(1, 2 * w, NRM_F32, NRM_F32) && g_plan.map_grid == 4096);
  c.bparams.map_grid = 10000;
  CHECK(apart(1, 2 * w, NRM_F32, NRM_F32) && g_plan.map_grid == 10000);
  c.bparams.map_grid = 1024;
  c.bparams.resident_segments = 0;
  CHECK(!apart(1, w, NRM_F32, NRM_F32));
  c.bparams.resident_segments = 64;
  c.bparams.graph = 1;  // a replay fails here
  CHECK(apart(1, w, NRM_F32, NRM_F32));
  CHECK(nrm_normalize_batched_ex(&c, in.data(), NRM_F32, in.data(), NRM_F32, offsets.data(), 512, w, NRM_ACC_F32, nullptr) != NRM_OK);
}

// A block's eight wavefronts have a row each while the mean row is about one
// wavefront's.
static void test_cuts_of_wavefront_rows() {
  Ctx c;
  for (int dt : {NRM_F32, NRM_BF16, NRM_F16})
    for (int64_t rows : {5000, 1 << 17})
      for (int64_t mean : {513, 1000, 1536, 1792, 1793, 2000, 2048, 2049, 3000}) {
        BatchHeader h;
        memset(&h, 0, sizeof(h));
        h.csr_in_dt = dt;
        cut_rows(c.bparams, rows, rows * mean, &h);
        CHECK(h.rows_per_block == (mean <= (dt == NRM_F32 ? 1792 : 2048) ? nrm::ROWS_WAVES : 4));
      }
}

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> tests = {
      {"rows_grid", test_rows_grid},
      {"captured_tables", test_captured_tables},
      {"failed_launch", test_failed_launch},
      {"workspace_layout", test_workspace_layout},
      {"tree_height", test_tree_height},
      {"apart_rule", test_apart_rule},
      {"cuts_of_one_segment_rows", test_cuts_of_one_segment_rows},
      {"cuts_of_wavefront_rows", test_cuts_of_wavefront_rows},
      {"cuts_without_resident_rows", test_cuts_without_resident_rows},
  };
  const auto t = tests.find(argc > 1 ? argv[1] : "");
  if (t == tests.end()) {
    fprintf(stderr, "no such test\n");
    return 2;
  }
  t->second();
  if (g_failures) {
    fprintf(stderr, "%d check(s) failed\n", g_failures);
    return 1;
  }
  printf("%s: passed\n", argv[1]);
  return 0;
}
