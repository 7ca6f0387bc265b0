// Ragged batched normalize on gfx950: every row of a batch is normalized on
// its own, out_r[i] = in_r[i] / sum(in_r), with the per-row sum hoisted out
// of the element-wise divide exactly as in the plain path (arXiv 2207.00257,
// Fig. 1 and Sec. IV-C), in two launches for the batch.
//
//   batch_rows_kernel    a grid over the rows themselves (1 to 32 consecutive
//                        rows per block, in dispatch order): resolves and
//                        validates each row (from CSR offsets or a descriptor
//                        table) and runs the rows of at most 2^14 elements on
//                        the spot: up to 256 elements on 16 lanes, up to
//                        wave_max (2048) on one wavefront, the rest on the
//                        block, each read into registers, summed, divided and
//                        written. The longer rows are appended to two work
//                        lists, one atomic per block and list.
//   batch_resident_kernel  persistent blocks take the lists' units from a
//                        counter: tile sums of the long rows, the segments
//                        of the rows of up to 2^20 elements (held on chip
//                        between their read and their write), then the tiles
//                        of the long rows again for the divide.
// In a large batch mostly of long rows, that kernel takes the segments only and
//   batch_tile_sums_kernel, batch_tile_totals_kernel, batch_phase2_kernel
// take the long rows, each with as many blocks as stream best.
// With resident_segments = 0 the lists are instead walked by three launches:
//   batch_phase1_kernel  single-pass rows and tile sums;
//   batch_rowsum_kernel  one block per long row merges the row's tile sums in
//                        a fixed order (the kernel boundary is the barrier
//                        that makes them visible);
//   batch_phase2_kernel  the long rows' tiles again, divided.
//
// All of a call's inputs are arguments of batch_rows_kernel: the launches can
// be captured once in a hipGraph and replayed with that one launch's arguments
// and grid set anew. A row's summation order depends only on its length, its
// start alignment modulo 128 bytes, its dtypes, the accumulation mode and the
// launch parameters: never on the other rows or its position in the batch.
#include <type_traits>

#include "nrm_batch.h"
#include "nrm_device.h"
#include "nrm_rows.h"

namespace nrm {
namespace {

using namespace dev;

// The lse output of a softmax call (device float[rows]), or NULL.
__device__ __forceinline__ float* lse_out(const BatchArgs& a) { return reinterpret_cast<float*>(a.cnt[CNT_LSE]); }

// ---- rows ------------------------------------------------------------------------

__device__ __forceinline__ bool valid_dt(int dt) { return dt == NRM_F32 || dt == NRM_BF16 || dt == NRM_F16; }

// Tiles are 2^tile_log2 elements: a shift, not a 64-bit division (which the
// GPU emulates in about a hundred instructions, per lane).
__device__ __forceinline__ int64_t long_tiles(int64_t n, int64_t short_max, int tile_log2) {
  return n <= short_max ? 0 : (n + (int64_t(1) << tile_log2) - 1) >> tile_log2;
}

// Row r resolved and validated: n = 0 if it is invalid (error bits in err) or
// has more tiles than a row's combine merges.
__device__ __forceinline__ RowDesc resolve_row(const BatchArgs& a, const BatchHeader& h, int64_t r, int& err) {
  RowDesc d;
  if (h.mode == BATCH_CSR) {
    const int64_t b = h.offsets[r], e = h.offsets[r + 1];
    const int si = h.csr_in_dt == NRM_F32 ? 4 : 2, so = h.csr_out_dt == NRM_F32 ? 4 : 2;
    d.in = h.csr_in + b * si;
    d.out = h.csr_out + b * so;
    d.n = e - b;
    d.in_dt = h.csr_in_dt;
    d.out_dt = h.csr_out_dt;
    if (b < 0 || e < b || e > h.capacity) {
      err |= NRM_DEVERR_OFFSETS;
      d.n = 0;
    }
  } else {
    d = h.table[r];
    if (d.n < 0 || !valid_dt(d.in_dt) || !valid_dt(d.out_dt) || (d.n > 0 && (!d.in || !d.out))) {
      err |= NRM_DEVERR_ROW;
      d.n = 0;
    }
  }
  if (long_tiles(d.n, a.short_max, a.tile_log2) > MAX_ROW_TILES) {
    err |= NRM_DEVERR_ROW;
    d.n = 0;
  }
  return d;
}

// Values the same in every lane, moved to scalar registers: a segment's
// addresses are then a scalar base plus a 32-bit offset per lane.
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ RowDesc uniform_desc(const RowDesc& d) {
  RowDesc x;
  x.in = reinterpret_cast<const char*>(uniform64(reinterpret_cast<int64_t>(d.in)));
  x.out = reinterpret_cast<char*>(uniform64(reinterpret_cast<int64_t>(d.out)));
  x.n = uniform64(d.n);
  x.in_dt = __builtin_amdgcn_readfirstlane(d.in_dt);
  x.out_dt = __builtin_amdgcn_readfirstlane(d.out_dt);
  return x;
}

__device__ __forceinline__ Item uniform_item(const Item& i) {
  return Item{uniform_desc(i.d), __builtin_amdgcn_readfirstlane(i.row), __builtin_amdgcn_readfirstlane(i.tile)};
}

// Inclusive scan over the 64 lanes of a wavefront by DPP lane moves: row_shr
// by 1, 2, 4 and 8 scans each row of 16 lanes (lanes shifted in from outside
// the row read 0); the totals of rows 0..2 (lanes 15, 31, 47) are then added
// to the rows after them.
template <int N>
__device__ __forceinline__ uint32_t row_shr(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x110 + N, 0xF, 0xF, false);
}

__device__ __forceinline__ uint32_t wave_scan32(uint32_t x, int lane) {
  x += row_shr<1>(x);
  x += row_shr<2>(x);
  x += row_shr<4>(x);
  x += row_shr<8>(x);
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
  if (lane >= 16) x += r0;
  if (lane >= 32) x += r1;
  if (lane >= 48) x += r2;
  return x;
}

// Entries of a resident row.
__device__ __forceinline__ int64_t row_segments(int64_t n) { return (n + (int64_t(1) << RES_LOG2) - 1) >> RES_LOG2; }

// The call number travels in two words so that no launch reads a word that
// it writes: batch_rows_kernel reads CNT_CALL and leaves CNT_CALL + 1 in
// CNT_CALL_RUN, which the launches after it read; the last of them copies
// it back to CNT_CALL. The call's parity picks one of two sets of list counters;
// the last launch zeroes the set that the next call uses. (CNT_TAKEN is zeroed
// by batch_rows_kernel, which does not use it.)
__device__ __forceinline__ int64_t* list_counters(const BatchArgs& a, int64_t call) {
  return a.cnt + CNT_SET0 + (call & 1) * CNT_SET_STRIDE;
}

__device__ __forceinline__ void end_call(const BatchArgs& a, int64_t call) {
  int64_t* other = list_counters(a, call + 1);
  for (int k = 0; k < LIST_COUNTERS; ++k) other[k * CNT_LINE] = 0;
  a.cnt[CNT_CALL] = call;
}

// The call's tag for published partials, never 0 (the value of a slot that
// was never written).
__device__ __forceinline__ uint32_t call_tag(int64_t call) { return (uint32_t)((uint64_t)call % 0xFFFFFFFFull) + 1u; }

// ---- single-pass rows (held in registers) --------------------------------------------

template <int DTI, int DTO, int ACC, int KB>
__device__ __forceinline__ void single_pass(const RowDesc& d, Acc<ACC>* slots, RowRes* s_bcast, float* lse,
                                            int64_t row) {
  constexpr int VEC = Elem<DTI>::VEC;
  constexpr int NA = accumulators(DTI, ACC, KB);
  const int B = blockDim.x, t = threadIdx.x;
  const Geom g = geometry<DTI>(d.in, (int)d.n);
  const u4* body = reinterpret_cast<const u4*>(d.in + g.head * Elem<DTI>::SIZE);
  u4 r[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    const int v = t + k * B;
    if (v < g.nvec) r[k] = load_vec<false>(body + v);
  }
  Acc<ACC> acc[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) acc[k].zero();
  if constexpr (ACC == ACC_SOFTMAX) {
    softmax_add_held<DTI, NA, KB>(acc, r, t, B, g.nvec);
  } else {
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if (t + k * B < g.nvec) {
        float x[VEC];
        widen<DTI>(r[k], x);
#pragma unroll
        for (int c = 0; c < VEC; ++c) acc[(k * VEC + c) % NA].add(x[c]);
      }
    }
  }
  if (t < g.head) acc[0].add(load_one<DTI>(d.in, t));
  if (t < (int)d.n - g.tail_begin) acc[0].add(load_one<DTI>(d.in, g.tail_begin + t));
  merge_chains<ACC, NA>(acc);
  Acc<ACC> tot = block_reduce<ACC>(acc[0], slots);
  if (t == 0) {
    const RowMap<ACC> f0 = RowMap<ACC>::of(tot);
    *s_bcast = f0.result();
    if constexpr (ACC == ACC_SOFTMAX) {
      if (lse) lse[row] = f0.lse();
    }
  }
  lds_barrier();
  const RowMap<ACC> f = RowMap<ACC>::of(*s_bcast);
  const bool vec_ok = out_vector_ok<DTI, DTO>(d.out, g.head);
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    const int v = t + k * B;
    if (v < g.nvec) {
      float x[VEC], q[VEC];
      widen<DTI>(r[k], x);
#pragma unroll
      for (int c = 0; c < VEC; ++c) q[c] = f(x[c]);
      store_quotients<DTI, DTO>(d.out, g.head, v, vec_ok, q);
    }
  }
  if (t < g.head) store_one<DTO>(d.out, t, f(load_one<DTI>(d.in, t)));
  if (t < (int)d.n - g.tail_begin) {
    const int i = g.tail_begin + t;
    store_one<DTO>(d.out, i, f(load_one<DTI>(d.in, i)));
  }
}

// ---- tiles of long rows ------------------------------------------------------------

// Sum of elements [b, e) of a row; valid in thread 0. NT: non-temporal loads
// (a temporal tile stays in the last-level cache for phase 2).
// NA independent chains per thread, each vector's elements dealt to them in
// turn: the bits depend on NA, not on U.
template <int DTI, int ACC, int U, bool NT, int NA>
__device__ __forceinline__ Acc<ACC> tile_reduce(const char* in_row, int64_t b, int64_t e,
                                                Acc<ACC>* slots) {
  constexpr int VEC = Elem<DTI>::VEC;
  const int t = thread_index();
  static_assert(CHAIN_ADDS * NA % (U * VEC) == 0 && U * VEC % NA == 0, "whole iterations between flushes");
  constexpr int FLUSH = CHAIN_ADDS * NA / (U * VEC);
  const char* seg = in_row + b * Elem<DTI>::SIZE;
  const int n = (int)(e - b);
  const Geom g = geometry<DTI>(seg, n);
  const u4* p = reinterpret_cast<const u4*>(seg + g.head * Elem<DTI>::SIZE) + t;
  const int B = blockDim.x, step = B * U;
  Acc<ACC> acc[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) acc[k].zero();
  Acc<ACC> run;
  run.zero();
  int since_flush = 0;
  // the unaligned head and the short tail, loaded before the stream so their
  // latency overlaps it
  const bool has_head = t < g.head;
  const bool has_tail = t < n - g.tail_begin;
  const float xh = has_head ? load_one<DTI>(seg, t) : 0.0f;
  const float xt = has_tail ? load_one<DTI>(seg, g.tail_begin + t) : 0.0f;
  for (int base = 0; base < g.nvec; base += step) {
    if (base + step <= g.nvec) {
      u4 r[U];
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = load_vec<NT>(p + base + u * B);
      if constexpr (ACC == ACC_SOFTMAX) {
        // full iterations keep the chains' k equal (see raise_shared); only
        // the last iteration of a tile can be partial, and it and the head
        // and tail raise their chains element by element
        float x[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) widen<DTI>(r[u], x[u]);
        float m = x[0][0];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int c = 0; c < VEC; ++c) m = fmaxf(m, x[u][c]);
        raise_shared<NA>(acc, m);
        const float nk = -acc[0].k;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int c = 0; c < VEC; ++c)
            acc[(u * VEC + c) % NA].s += __builtin_amdgcn_exp2f(__builtin_fmaf(x[u][c], LOG2E_F, nk));
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float x[VEC];
          widen<DTI>(r[u], x);
#pragma unroll
          for (int c = 0; c < VEC; ++c) acc[(u * VEC + c) % NA].add(x[c]);
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (base + u * B + t < g.nvec) {
          float x[VEC];
          widen<DTI>(load_vec<NT>(p + base + u * B), x);
#pragma unroll
          for (int c = 0; c < VEC; ++c) acc[(u * VEC + c) % NA].add(x[c]);
        }
      }
    }
    if constexpr (ACC != NRM_ACC_KAHAN) {
      if (++since_flush == FLUSH) {
        since_flush = 0;
        merge_chains<ACC, NA>(acc);
        run.merge(acc[0]);
#pragma unroll
        for (int k = 0; k < NA; ++k) acc[k].zero();
      }
    }
  }
  if (has_head) acc[0].add(xh);
  if (has_tail) acc[0].add(xt);
  merge_chains<ACC, NA>(acc);
  run.merge(acc[0]);
  return block_reduce<ACC>(run, slots);
}

// out[i] = f(in[i]) for elements [b, e) of a row.
template <int DTI, int DTO, int U, class F>
__device__ __forceinline__ void tile_map(const RowDesc& d, int64_t b, int64_t e, const F& f) {
  constexpr int VEC = Elem<DTI>::VEC;
  const int t = thread_index();
  const char* in_seg = d.in + b * Elem<DTI>::SIZE;
  char* out_seg = d.out + b * Elem<DTO>::SIZE;
  const int n = (int)(e - b);
  const Geom g = geometry<DTI>(in_seg, n);
  const u4* body = reinterpret_cast<const u4*>(in_seg + g.head * Elem<DTI>::SIZE);
  const bool vec_ok = out_vector_ok<DTI, DTO>(out_seg, g.head);
  const int B = blockDim.x, step = B * U;
  const bool has_head = t < g.head;
  const int ti = g.tail_begin + t;
  const bool has_tail = ti < n;
  const float xh = has_head ? load_one<DTI>(in_seg, t) : 0.0f;
  const float xt = has_tail ? load_one<DTI>(in_seg, ti) : 0.0f;
  for (int base = 0; base < g.nvec; base += step) {
    const int v0 = base + t;
    if (base + step <= g.nvec) {
      u4 r[U];
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = load_vec<true>(body + v0 + u * B);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float x[VEC], q[VEC];
        widen<DTI>(r[u], x);
#pragma unroll
        for (int c = 0; c < VEC; ++c) q[c] = f(x[c]);
        store_quotients<DTI, DTO>(out_seg, g.head, v0 + u * B, vec_ok, q);
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (v0 + u * B < g.nvec) {
          float x[VEC], q[VEC];
          widen<DTI>(load_vec<true>(body + v0 + u * B), x);
#pragma unroll
          for (int c = 0; c < VEC; ++c) q[c] = f(x[c]);
          store_quotients<DTI, DTO>(out_seg, g.head, v0 + u * B, vec_ok, q);
        }
      }
    }
  }
  if (has_head) store_one<DTO>(out_seg, t, f(xh));
  if (has_tail) store_one<DTO>(out_seg, ti, f(xt));
}

// ---- dtype dispatch of one item --------------------------------------------------------
// The softmax kind is binary32 in and out only (the host rejects anything else).

template <int ACC, int KB>
__device__ __forceinline__ void dispatch_single(const RowDesc& d, Acc<ACC>* slots, RowRes* s_bcast, float* lse,
                                                int64_t row) {
  if constexpr (ACC == ACC_SOFTMAX) {
    single_pass<NRM_F32, NRM_F32, ACC, KB>(d, slots, s_bcast, lse, row);
  } else {
#define NRM_SP(I, O) single_pass<I, O, ACC, KB>(d, slots, s_bcast, lse, row)
    switch (d.in_dt * 3 + d.out_dt) {
      case NRM_F32 * 3 + NRM_F32: NRM_SP(NRM_F32, NRM_F32); break;
      case NRM_F32 * 3 + NRM_BF16: NRM_SP(NRM_F32, NRM_BF16); break;
      case NRM_F32 * 3 + NRM_F16: NRM_SP(NRM_F32, NRM_F16); break;
      case NRM_BF16 * 3 + NRM_F32: NRM_SP(NRM_BF16, NRM_F32); break;
      case NRM_BF16 * 3 + NRM_BF16: NRM_SP(NRM_BF16, NRM_BF16); break;
      case NRM_BF16 * 3 + NRM_F16: NRM_SP(NRM_BF16, NRM_F16); break;
      case NRM_F16 * 3 + NRM_F32: NRM_SP(NRM_F16, NRM_F32); break;
      case NRM_F16 * 3 + NRM_BF16: NRM_SP(NRM_F16, NRM_BF16); break;
      default: NRM_SP(NRM_F16, NRM_F16); break;
    }
#undef NRM_SP
  }
}

// NA 0: one chain per element of an iteration, as the plain reduce has them.
template <int ACC, int U, bool NT, int NA = 0>
__device__ __forceinline__ Acc<ACC> dispatch_tile_reduce(const RowDesc& d, int64_t b, int64_t e,
                                                         Acc<ACC>* slots) {
#define NRM_TR(I) return tile_reduce<I, ACC, U, NT, NA ? NA : accumulators(I, ACC, U)>(d.in, b, e, slots)
  if constexpr (ACC == ACC_SOFTMAX) {
    NRM_TR(NRM_F32);
  } else {
    switch (d.in_dt) {
      case NRM_F32: NRM_TR(NRM_F32);
      case NRM_BF16: NRM_TR(NRM_BF16);
      default: NRM_TR(NRM_F16);
    }
  }
#undef NRM_TR
}

template <int ACC, int U>
__device__ __forceinline__ void dispatch_tile_map(const RowDesc& d, int64_t b, int64_t e, const RowMap<ACC>& f) {
  if constexpr (ACC == ACC_SOFTMAX) {
    tile_map<NRM_F32, NRM_F32, U>(d, b, e, f);
  } else {
#define NRM_TM(I, O) tile_map<I, O, U>(d, b, e, f)
    switch (d.in_dt * 3 + d.out_dt) {
      case NRM_F32 * 3 + NRM_F32: NRM_TM(NRM_F32, NRM_F32); break;
      case NRM_F32 * 3 + NRM_BF16: NRM_TM(NRM_F32, NRM_BF16); break;
      case NRM_F32 * 3 + NRM_F16: NRM_TM(NRM_F32, NRM_F16); break;
      case NRM_BF16 * 3 + NRM_F32: NRM_TM(NRM_BF16, NRM_F32); break;
      case NRM_BF16 * 3 + NRM_BF16: NRM_TM(NRM_BF16, NRM_BF16); break;
      case NRM_BF16 * 3 + NRM_F16: NRM_TM(NRM_BF16, NRM_F16); break;
      case NRM_F16 * 3 + NRM_F32: NRM_TM(NRM_F16, NRM_F32); break;
      case NRM_F16 * 3 + NRM_BF16: NRM_TM(NRM_F16, NRM_BF16); break;
      default: NRM_TM(NRM_F16, NRM_F16); break;
    }
#undef NRM_TM
  }
}

// ---- the long rows' tiles and the resident rows, persistently -------------------------------

constexpr int TILE_MAP_U = 4;  // tile divides: vectors per thread per iteration
// elements of one unit of the divide: one block-iteration of 4-byte elements
constexpr int64_t MAP_UNIT = (int64_t)RES_BLOCK * TILE_MAP_U * 4;

// The block that published a long row's last tile sum: read and merge the
// row's `count` tagged partials (at most MAX_ROW_TILES), RES_BLOCK at a time,
// one per thread, in a fixed order that depends only on count: each round by
// block_reduce, then the rounds' totals by wavefront 0 (height 9 + 7).
// Every thread must call it; the result is valid in thread 0.
constexpr int TILE_ROUNDS = (int)(MAX_ROW_TILES / RES_BLOCK);
static_assert(TILE_ROUNDS <= 128, "two rounds' totals per lane");
static_assert(long_row_height(22) <= 62, "the published bound");
template <int ACC>
__device__ __forceinline__ Acc<ACC> gather_tiles(const ResExchange& x, int64_t count, Acc<ACC>* slots,
                                                 Acc<ACC>* rounds) {
  const int t = threadIdx.x, n = (int)((count + RES_BLOCK - 1) / RES_BLOCK);
  for (int j = 0; j < n; ++j) {
    const int64_t i = (int64_t)j * RES_BLOCK + t;
    Acc<ACC> v;
    v.zero();
    if (i < count) v = wait_tagged<ACC>(x, x.slots + 2 * i);
    lds_barrier();  // slots: of the call before, or of the round before
    const Acc<ACC> r = block_reduce<ACC>(v, slots);
    if (t == 0) rounds[j] = r;
  }
  lds_barrier();
  Acc<ACC> v;
  v.zero();
  if (t < 64) {
    if (t < n) v = rounds[t];
    if (t + 64 < n) v.merge(rounds[t + 64]);
    v = wave_reduce<ACC>(v);
  }
  return v;
}

// The sum of one tile of a long row; valid in thread 0. The last keep_tiles
// tiles of a batch are read with a temporal hint (keep): the divide finds them
// in the last-level cache.
template <int ACC>
__device__ __forceinline__ Acc<ACC> tile_sum(const BatchArgs& a, const Item& it, bool keep, Acc<ACC>* slots) {
  const RowDesc& d = it.d;
  const int64_t b = (int64_t)it.tile << a.tile_log2;
  const int64_t e = b + a.tile < d.n ? b + a.tile : d.n;
  Acc<ACC> p;
  p.zero();
  for (int64_t c = b; c < e; c += TILE_PART) {
    const int64_t ce = c + TILE_PART < e ? c + TILE_PART : e;
    p.merge(keep ? dispatch_tile_reduce<ACC, TILE_U, false, TILE_NA>(d, c, ce, slots)
                 : dispatch_tile_reduce<ACC, TILE_U, true, TILE_NA>(d, c, ce, slots));
    if (ce < e) lds_barrier();  // slots are reused
  }
  return p;
}

// The entries that one block of batch_rows_kernel appended: where in the list,
// and which in row order.
struct ListRange {
  int64_t base;
  uint32_t start, count;
};
static_assert(ORDERED_BLOCKS % RES_BLOCK == 0, "a whole number of ranges per thread");

// Persistent blocks: the units are the long rows' tile sums, then the
// segments of the resident rows, both taken one at a time from a counter in
// list order; then the long rows' tiles once more, in units of MAP_UNIT
// elements dealt out statically. A tile sum waits for nothing. A resident
// segment waits for its row (see the resident rows' progress argument; tile
// sums only come before). A divide unit waits for its row's total, whose
// tile sums were all taken before by blocks that run. The wait is bounded
// like the resident rows'.
//
// HBM bounds it: resident rows move 8 bytes per binary32 element, long rows
// 12. 4096 rows of up to 2^20 binary32 (3.43 GB) take 577 us per call launched
// directly (587 replayed) with three blocks per CU (80 registers; with the plain
// reduce's 16 chains in the tile sums 128 and two blocks, 616 us; four blocks
// spilled: 597-622 us), BF16 ones 404 against 478 us, the latency of their smaller
// segments (claim, entry, elements, exchange) not hidden. The tiles of the divide
// are dealt statically because nothing waits for them, and in units of 2^13
// elements so that the last round of 512 blocks is short (whole tiles of 2^15
// left up to half of the blocks idle in it). Large batches of long rows are
// faster apart (below).
template <int ACC>
__global__ void __launch_bounds__(RES_BLOCK) __attribute__((amdgpu_waves_per_eu(6, 6))) batch_resident_kernel(BatchArgs a) {
  __shared__ Acc<ACC> slots[MAX_WAVES];
  __shared__ RowRes s_bcast;
  __shared__ int64_t s_claim;
  __shared__ Acc<ACC> rounds[TILE_ROUNDS];
  __shared__ int s_last;
  __shared__ uint32_t s_scan[RES_BLOCK / 64];
  __shared__ ListRange s_range[ORDERED_BLOCKS];
  __shared__ int64_t s_pos;
  unsigned long long* counter = reinterpret_cast<unsigned long long*>(a.cnt + CNT_TAKEN);
  auto take = [&] {
    return (int64_t)__hip_atomic_fetch_add(counter, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // every word the start needs in one round trip: both sets of counters, of
  // which the call's number picks one
  const int64_t call = a.cnt[CNT_CALL_RUN], ordered = a.cnt[CNT_ORDERED];
  const int64_t* set0 = list_counters(a, 0);
  const int64_t* set1 = list_counters(a, 1);
  const int64_t t0 = set0[LIST_TILES * CNT_LINE], s0 = set0[LIST_SHORT * CNT_LINE];
  const int64_t t1 = set1[LIST_TILES * CNT_LINE], s1 = set1[LIST_SHORT * CNT_LINE];
  const BlockShorts mine0 = a.block_shorts[threadIdx.x];
  int64_t n_long = call & 1 ? t1 : t0, n_short = call & 1 ? s1 : s0;
  // (entries past the capacity were not written; in row order they are passed
  // over one by one)
  if (n_long > a.cap_items) n_long = a.cap_items;
  if (a.apart) n_long = 0;
  if (n_short > a.cap_items && ordered == 0) n_short = a.cap_items;
  if (blockIdx.x == 0 && threadIdx.x == 0) end_call(a, call);
  const int64_t units = n_long + n_short;
  if (units <= 0) return;
  // the first unit only now: one counter serves about one block per 14 ns, so
  // with nothing listed 768 blocks that took one first ended after 11 us, and
  // end after 4.3 us this way
  if (threadIdx.x == 0) s_claim = take();
  const uint32_t ep = call_tag(call);
  float* lse = lse_out(a);
  unsigned long long* stall = reinterpret_cast<unsigned long long*>(a.cnt + CNT_STALL);
  // Up to ORDERED_BLOCKS blocks: the segments are taken in the rows' order,
  // whatever the order in which the blocks of batch_rows_kernel appended them:
  // thread t holds the ranges of the list of blocks t, t + RES_BLOCK, ... and
  // where they start in row order. (4096 rows, 1.7 GB: 642 us in memory order, 666
  // us shuffled; 8192 x 40000 451 and 499, 16384 x 40000 867 and 963.)
  if (ordered > 0) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t before = 0;
    for (int k = 0; k < ordered; k += RES_BLOCK) {
      const int64_t b = k + threadIdx.x;
      BlockShorts mine = mine0;
      if (k > 0) {
        mine = b < ordered ? a.block_shorts[b] : BlockShorts{0, 0};
        lds_barrier();  // s_scan is reused
      }
      const uint32_t count = b < ordered ? (uint32_t)mine.count : 0u;
      const uint32_t incl = wave_scan32(count, lane);
      if (lane == 63) s_scan[wave] = incl;
      lds_barrier();
      uint32_t start = before + incl - count;
      for (int w = 0; w < RES_BLOCK / 64; ++w) {
        if (w < wave) start += s_scan[w];
        before += s_scan[w];
      }
      s_range[b] = ListRange{mine.base, start, count};
    }
  }
  lds_barrier();
  int64_t u = uniform64(s_claim);
  while (u < units) {
    int64_t pos = u - n_long;  // in the list of segments
    if (pos >= 0 && ordered > 0) {
      for (int k = 0; k < ordered; k += RES_BLOCK) {
        const ListRange r = s_range[k + threadIdx.x];
        const uint32_t off = (uint32_t)pos - r.start;
        if ((uint32_t)pos >= r.start && off < r.count) s_pos = r.base + off;
      }
      lds_barrier();
      pos = uniform64(s_pos);
    }
    Item it;
    it.row = -1;
    if (pos < a.cap_items) it = uniform_item(u < n_long ? a.tiles[u] : a.shorts[pos]);
    if (it.row >= 0) {  // an entry of a row that did not fit the list is empty
      const RowDesc& d = it.d;
      if (u < n_long) {
        const int64_t first = u - it.tile;
        const Acc<ACC> p = tile_sum<ACC>(a, it, u >= n_long - a.keep_tiles, slots);
        const ResExchange x{a.tile_tagged + 2 * first, a.tile_total + 2 * first, a.tile_arrivals + first, ep, a.error, stall};
        const int64_t count = (d.n + a.tile - 1) >> a.tile_log2;
        if (threadIdx.x == 0) {
          publish_tagged<ACC>(x.slots + 2 * it.tile, ep, p);
          s_last = __hip_atomic_fetch_add(x.arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   (unsigned)count - 1;
        }
        lds_barrier();
        if (s_last) {
          const Acc<ACC> total = gather_tiles<ACC>(x, count, slots, rounds);
          if (threadIdx.x == 0) {
            __hip_atomic_store(x.arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            publish_tagged<ACC>(x.total, ep, total);
            if constexpr (ACC == ACC_SOFTMAX) {
              if (lse) lse[it.row] = RowMap<ACC>::of(total).lse();
            }
          }
        }
      } else {
        // the row's entries are consecutive: its first is at pos - tile
        const int64_t first = pos - it.tile;
        const ResExchange x{a.tagged + 2 * first, a.rowtot + 2 * first, a.arrivals + first, ep, a.error, stall};
        dispatch_resident<ACC>(d, it.tile, x, slots, &s_bcast, lse ? lse + it.row : nullptr);
      }
    }
    // the next unit once this one is done (claiming it as soon as the row's
    // sum was known, to overlap the claim with the writes, measured slower)
    lds_barrier();  // slots, s_bcast and s_claim are reused
    if (threadIdx.x == 0) s_claim = take();
    lds_barrier();
    u = uniform64(s_claim);
  }
  const int64_t per_tile = a.tile > MAP_UNIT ? a.tile / MAP_UNIT : 1;  // powers of two
  const int64_t unit = a.tile / per_tile;
  for (int64_t m = blockIdx.x; m < n_long * per_tile; m += gridDim.x) {
    const int64_t pos = m / per_tile, part = m - pos * per_tile;
    const Item it = uniform_item(a.tiles[pos]);
    if (it.row < 0) continue;
    const RowDesc& d = it.d;
    const int64_t b = ((int64_t)it.tile << a.tile_log2) + part * unit;
    if (b >= d.n) continue;
    const int64_t e = b + unit < d.n ? b + unit : d.n;
    const int64_t first = pos - it.tile;
    const ResExchange x{a.tile_tagged + 2 * first, a.tile_total + 2 * first, a.tile_arrivals + first, ep, a.error, stall};
    lds_barrier();  // s_bcast is reused
    if (threadIdx.x == 0) s_bcast = RowMap<ACC>::of(wait_tagged<ACC>(x, x.total)).result();
    lds_barrier();
    dispatch_tile_map<ACC, TILE_MAP_U>(d, b, e, RowMap<ACC>::of(s_bcast));
  }
}

// ---- the long rows in launches of their own --------------------------------------------------
// A large batch mostly of long rows (args.apart): the same tile sums, published
// in the same tagged words and merged in the same order, so that a row's bits do
// not depend on it, then the divide by batch_phase2_kernel.
//
// HBM bounds it, three transfers. The persistent kernel takes the tiles from a
// counter, which serves one per 14 to 17 ns, holds 80 registers for the segments,
// and waits for each unit's row total: 16 rows of 20,000,000 binary32 676 us there,
// 603 us here (6.4 TB/s over 3.84 GB, less what the cache keeps), bfloat16 424 and
// 313 us. Small batches lose here to the launches' starts, and those with wider
// outputs than inputs to phase 2's two stores per vector: see the host's rule.

template <int ACC>
__global__ void __launch_bounds__(RES_BLOCK) batch_tile_sums_kernel(BatchArgs a) {
  __shared__ Acc<ACC> slots[MAX_WAVES];
  const int64_t call = a.cnt[CNT_CALL_RUN];
  const int64_t listed = list_counters(a, call)[LIST_TILES * CNT_LINE];
  const int64_t n_long = listed < a.cap_items ? listed : a.cap_items;
  for (int64_t pos = blockIdx.x; pos < n_long; pos += gridDim.x) {
    const Item it = uniform_item(a.tiles[pos]);
    if (it.row < 0) continue;
    const Acc<ACC> p = tile_sum<ACC>(a, it, pos >= n_long - a.keep_tiles, slots);
    if (threadIdx.x == 0) publish_tagged<ACC>(a.tile_tagged + 2 * pos, call_tag(call), p);
    lds_barrier();  // slots are reused
  }
}

// One block per long row at a time.
template <int ACC>
__global__ void __launch_bounds__(RES_BLOCK) batch_tile_totals_kernel(BatchArgs a) {
  __shared__ Acc<ACC> slots[MAX_WAVES];
  __shared__ Acc<ACC> rounds[TILE_ROUNDS];
  const int64_t call = a.cnt[CNT_CALL_RUN];
  const int64_t n_rows = list_counters(a, call)[LIST_LONG_ROWS * CNT_LINE];
  float* lse = lse_out(a);
  for (int64_t k = blockIdx.x; k < n_rows; k += gridDim.x) {
    const int64_t first = a.lrow_first[k];
    if (first < 0) continue;  // the row did not fit the list
    const Item it = uniform_item(a.tiles[first]);
    const ResExchange x{a.tile_tagged + 2 * first, nullptr, nullptr, call_tag(call), a.error,
                        reinterpret_cast<unsigned long long*>(a.cnt + CNT_STALL)};
    const Acc<ACC> total = gather_tiles<ACC>(x, (it.d.n + a.tile - 1) >> a.tile_log2, slots, rounds);
    if (threadIdx.x == 0) {
      const RowMap<ACC> f = RowMap<ACC>::of(total);
      a.results[first] = f.result();
      if constexpr (ACC == ACC_SOFTMAX) {
        if (lse) lse[it.row] = f.lse();
      }
    }
    lds_barrier();  // rounds are reused
  }
}

// ---- the same lists in three launches (resident_segments = 0) ---------------------------------

template <int ACC, int U, int KB>
__global__ void __launch_bounds__(1024) batch_phase1_kernel(BatchArgs a) {
  __shared__ Acc<ACC> slots[MAX_WAVES];
  __shared__ RowRes s_bcast;
  const int64_t* lists = list_counters(a, a.cnt[CNT_CALL_RUN]);
  const int64_t n_long = lists[LIST_TILES * CNT_LINE] < a.cap_items ? lists[LIST_TILES * CNT_LINE] : a.cap_items;
  const int64_t n_short = lists[LIST_SHORT * CNT_LINE] < a.cap_items ? lists[LIST_SHORT * CNT_LINE] : a.cap_items;
  const int64_t n_items = n_long + n_short;
  const int64_t keep_item = n_long - a.keep_tiles;
  float* lse = lse_out(a);
  Acc<ACC>* part = static_cast<Acc<ACC>*>(a.partials);
  for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    const Item it = uniform_item(item < n_long ? a.tiles[item] : a.shorts[item - n_long]);
    if (it.row < 0) continue;
    const RowDesc& d = it.d;
    if (item >= n_long) {
      dispatch_single<ACC, KB>(d, slots, &s_bcast, lse, it.row);
    } else {
      const int64_t b = (int64_t)it.tile << a.tile_log2;
      const int64_t e = b + a.tile < d.n ? b + a.tile : d.n;
      // the last keep_tiles tiles are read with a temporal hint: phase 2
      // finds them in the last-level cache
      const Acc<ACC> p = item >= keep_item ? dispatch_tile_reduce<ACC, U, false>(d, b, e, slots)
                                           : dispatch_tile_reduce<ACC, U, true>(d, b, e, slots);
      if (threadIdx.x == 0) part[item] = p;  // read after the kernel boundary
    }
    lds_barrier();  // the block's LDS is reused by the next item
  }
}

// Each long row's result from its tile partials, in a fixed order that
// depends only on the number of tiles (combine_partials: one wavefront for up
// to 1024 partials, the LDS tree beyond). One block per long row at a time.
template <int ACC>
__global__ void __launch_bounds__(1024) batch_rowsum_kernel(BatchArgs a) {
  __shared__ Acc<ACC> tree[COMBINE_TILE];
  __shared__ Acc<ACC> tiles[MAX_COMBINE_TILES];
  const int64_t* lists = list_counters(a, a.cnt[CNT_CALL_RUN]);
  const int64_t n_lrows = lists[LIST_LONG_ROWS * CNT_LINE];
  float* lse = lse_out(a);
  const Acc<ACC>* part = static_cast<const Acc<ACC>*>(a.partials);
  for (int64_t k = blockIdx.x; k < n_lrows; k += gridDim.x) {
    const int64_t first = a.lrow_first[k];
    if (first < 0) continue;  // the row did not fit the list
    const int32_t row = a.tiles[first].row;
    const int64_t count = (a.tiles[first].d.n + a.tile - 1) >> a.tile_log2;
    Acc<ACC> tot = combine_partials<ACC>(part + first, count, tree, tiles);
    if (threadIdx.x == 0) {
      const RowMap<ACC> f = RowMap<ACC>::of(tot);
      a.results[first] = f.result();
      if constexpr (ACC == ACC_SOFTMAX) {
        if (lse) lse[row] = f.lse();
      }
    }
    lds_barrier();  // the trees are reused by the next row
  }
}

template <int ACC, int U>
__global__ void __launch_bounds__(1024) batch_phase2_kernel(BatchArgs a) {
  const int64_t call = a.cnt[CNT_CALL_RUN];
  const int64_t* lists = list_counters(a, call);
  const int64_t n_long = lists[LIST_TILES * CNT_LINE] < a.cap_items ? lists[LIST_TILES * CNT_LINE] : a.cap_items;
  if (blockIdx.x == 0 && threadIdx.x == 0) end_call(a, call);
  for (int64_t pos = blockIdx.x; pos < n_long; pos += gridDim.x) {
    const Item it = uniform_item(a.tiles[pos]);
    if (it.row < 0) continue;
    const RowDesc& d = it.d;
    const int64_t b = (int64_t)it.tile << a.tile_log2;
    const int64_t e = b + a.tile < d.n ? b + a.tile : d.n;
    dispatch_tile_map<ACC, U>(d, b, e, RowMap<ACC>::of(a.results[pos - it.tile]));
  }
}

template <int ACC, int U>
hipError_t phase1_kb(const BatchPlan& p, const BatchArgs& a, hipStream_t s) {
  switch (p.short_regs) {
    case 1: hipLaunchKernelGGL((batch_phase1_kernel<ACC, U, 1>), dim3(p.grid), dim3(p.block), 0, s, a); break;
    case 2: hipLaunchKernelGGL((batch_phase1_kernel<ACC, U, 2>), dim3(p.grid), dim3(p.block), 0, s, a); break;
    case 4: hipLaunchKernelGGL((batch_phase1_kernel<ACC, U, 4>), dim3(p.grid), dim3(p.block), 0, s, a); break;
    default: hipLaunchKernelGGL((batch_phase1_kernel<ACC, U, 8>), dim3(p.grid), dim3(p.block), 0, s, a); break;
  }
  return hipGetLastError();
}

template <int ACC>
hipError_t phase1_u(const BatchPlan& p, const BatchArgs& a, hipStream_t s) {
  switch (p.unroll) {
    case 1: return phase1_kb<ACC, 1>(p, a, s);
    case 2: return phase1_kb<ACC, 2>(p, a, s);
    case 4: return phase1_kb<ACC, 4>(p, a, s);
    default: return phase1_kb<ACC, 8>(p, a, s);
  }
}

constexpr int64_t ROWSUM_GRID = 1024;
// the long rows' own launches: 16 blocks per CU, a tile at a time (four per CU:
// compensated sums of 200 rows of 2^18 to 2^22 binary32 625 us, with 16 602); a
// block per row
constexpr unsigned SUMS_GRID = 4096, TOTALS_GRID = 256;

template <int ACC>
hipError_t rowsum_acc(const BatchPlan& p, const BatchArgs& a, hipStream_t s) {
  // one 64-thread block per long row at a time; more blocks than this only
  // add dispatch work for small batches
  const int64_t grid = p.grid < ROWSUM_GRID ? p.grid : ROWSUM_GRID;
  hipLaunchKernelGGL((batch_rowsum_kernel<ACC>), dim3(grid), dim3(64), 0, s, a);
  return hipGetLastError();
}

template <int ACC>
hipError_t phase2_acc(const BatchPlan& p, const BatchArgs& a, hipStream_t s) {
  switch (p.map_unroll) {
    case 1: hipLaunchKernelGGL((batch_phase2_kernel<ACC, 1>), dim3(p.map_grid), dim3(p.map_block), 0, s, a); break;
    case 2: hipLaunchKernelGGL((batch_phase2_kernel<ACC, 2>), dim3(p.map_grid), dim3(p.map_block), 0, s, a); break;
    case 4: hipLaunchKernelGGL((batch_phase2_kernel<ACC, 4>), dim3(p.map_grid), dim3(p.map_block), 0, s, a); break;
    default: hipLaunchKernelGGL((batch_phase2_kernel<ACC, 8>), dim3(p.map_grid), dim3(p.map_block), 0, s, a); break;
  }
  return hipGetLastError();
}

// ---- rows run by batch_rows_kernel ------------------------------------------------------
// A row of 0 < n <= wave_max elements (at most WAVE_MAX_ELEMS) is taken by one
// wavefront: its head, 16-byte vectors and tail are read into registers, summed
// in each lane's chains and across the lanes by DPP moves (no LDS, no barrier),
// divided from the registers and written: two HBM transfers, and a wavefront
// never waits for another.
// Whether n elements from p are whole 128-byte lines: rows that share no line
// with their neighbours are read (and on 16 lanes also written)
// non-temporally, the others temporally, since the neighbour's wavefront finds
// the shared line in the L2. (2^20 rows of 250 binary32: 475 us non-temporal,
// 371 us temporal; 200,000 rows of up to 4096: 187 and 177 us; 2^17 rows of
// 2048, whole lines, at 4 per block: 369 us non-temporal, 397 us temporal.)
template <int DT>
__device__ __forceinline__ bool whole_lines(const char* p, int n) {
  return (((uint32_t)reinterpret_cast<uintptr_t>(p) | (uint32_t)(n * Elem<DT>::SIZE)) & (BODY_ALIGN - 1)) == 0;
}

template <int DTI, int DTO, int ACC>
__device__ __forceinline__ void wave_row(const RowDesc& d, float* lse) {
  constexpr int VEC = Elem<DTI>::VEC;
  constexpr int KW = (int)(WAVE_MAX_ELEMS / (64 * VEC));
  constexpr int NA = ACC == NRM_ACC_F32 ? 8 : 4;  // chains per lane (few: registers go to the held row)
  const int lane = threadIdx.x & 63;
  const Geom g = geometry<DTI>(d.in, (int)d.n);
  const u4* body = reinterpret_cast<const u4*>(d.in + g.head * Elem<DTI>::SIZE);
  u4 r[KW];
  if (whole_lines<DTI>(d.in, (int)d.n)) {
#pragma unroll
    for (int k = 0; k < KW; ++k)
      if (lane + k * 64 < g.nvec) r[k] = load_vec<true>(body + lane + k * 64);
  } else {
#pragma unroll
    for (int k = 0; k < KW; ++k)
      if (lane + k * 64 < g.nvec) r[k] = load_vec<false>(body + lane + k * 64);
  }
  const bool has_head = lane < g.head;
  const bool has_tail = lane < (int)d.n - g.tail_begin;
  const float xh = has_head ? load_one<DTI>(d.in, lane) : 0.0f;
  const float xt = has_tail ? load_one<DTI>(d.in, g.tail_begin + lane) : 0.0f;
  Acc<ACC> acc[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) acc[k].zero();
  if constexpr (ACC == ACC_SOFTMAX) {
    softmax_add_held<DTI, NA, KW>(acc, r, lane, 64, g.nvec);
  } else {
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      if (lane + k * 64 < g.nvec) {
        float x[VEC];
        widen<DTI>(r[k], x);
#pragma unroll
        for (int c = 0; c < VEC; ++c) acc[(k * VEC + c) % NA].add(x[c]);
      }
    }
  }
  if (has_head) acc[0].add(xh);
  if (has_tail) acc[0].add(xt);
  merge_chains<ACC, NA>(acc);
  const RowMap<ACC> f = RowMap<ACC>::of(wave_reduce<ACC>(acc[0]));  // the same in every lane
  if constexpr (ACC == ACC_SOFTMAX) {
    if (lse && lane == 0) *lse = f.lse();
  }
  const bool vec_ok = out_vector_ok<DTI, DTO>(d.out, g.head);
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int v = lane + k * 64;
    if (v < g.nvec) {
      float x[VEC], q[VEC];
      widen<DTI>(r[k], x);
#pragma unroll
      for (int c = 0; c < VEC; ++c) q[c] = f(x[c]);
      store_quotients<DTI, DTO>(d.out, g.head, v, vec_ok, q);
    }
  }
  if (has_head) store_one<DTO>(d.out, lane, f(xh));
  if (has_tail) store_one<DTO>(d.out, g.tail_begin + lane, f(xt));
}

template <int ACC>
__device__ __forceinline__ void dispatch_wave(const RowDesc& d, float* lse) {
  if constexpr (ACC == ACC_SOFTMAX) {
    wave_row<NRM_F32, NRM_F32, ACC>(d, lse);
  } else {
#define NRM_WR(I, O) wave_row<I, O, ACC>(d, lse)
    switch (d.in_dt * 3 + d.out_dt) {
      case NRM_F32 * 3 + NRM_F32: NRM_WR(NRM_F32, NRM_F32); break;
      case NRM_F32 * 3 + NRM_BF16: NRM_WR(NRM_F32, NRM_BF16); break;
      case NRM_F32 * 3 + NRM_F16: NRM_WR(NRM_F32, NRM_F16); break;
      case NRM_BF16 * 3 + NRM_F32: NRM_WR(NRM_BF16, NRM_F32); break;
      case NRM_BF16 * 3 + NRM_BF16: NRM_WR(NRM_BF16, NRM_BF16); break;
      case NRM_BF16 * 3 + NRM_F16: NRM_WR(NRM_BF16, NRM_F16); break;
      case NRM_F16 * 3 + NRM_F32: NRM_WR(NRM_F16, NRM_F32); break;
      case NRM_F16 * 3 + NRM_BF16: NRM_WR(NRM_F16, NRM_BF16); break;
      default: NRM_WR(NRM_F16, NRM_F16); break;
    }
#undef NRM_WR
  }
}

// Rows of at most QUARTER_MAX elements take a row of 16 lanes (a DPP row)
// each, four of them per wavefront at once. The head before the first 16-byte
// boundary (fewer than one vector) and the tail are one element per lane; each
// lane holds at most QUARTER_MAX / (16 VEC) vectors; the sum is the 16 lanes'
// chains merged by row16_reduce, in every lane of the row.
constexpr int64_t QUARTER_MAX = 256;

template <int DTI, int DTO, int ACC>
__device__ __forceinline__ void quarter_row(const RowDesc& d, float* lse) {
  constexpr int SI = Elem<DTI>::SIZE, VEC = Elem<DTI>::VEC;
  constexpr int KQ = (int)(QUARTER_MAX / (16 * VEC));
  constexpr int NA = ACC == NRM_ACC_F32 ? 8 : 4;
  const int j = threadIdx.x & 15;
  // at most QUARTER_MAX elements: 32-bit indexes
  const int n = (int)d.n, mis = (int)(reinterpret_cast<uintptr_t>(d.in) & 15);
  const int to_line = mis ? (16 - mis) / SI : 0, head = to_line < n ? to_line : n;
  const int nvec = (n - head) / VEC, tail_begin = head + nvec * VEC;
  const u4* body = reinterpret_cast<const u4*>(d.in + head * SI);
  const bool nt = __all(whole_lines<DTI>(d.in, n));
  u4 r[KQ];
  if (nt) {
#pragma unroll
    for (int k = 0; k < KQ; ++k)
      if (j + k * 16 < nvec) r[k] = load_vec<true>(body + j + k * 16);
  } else {
#pragma unroll
    for (int k = 0; k < KQ; ++k)
      if (j + k * 16 < nvec) r[k] = load_vec<false>(body + j + k * 16);
  }
  const bool has_head = j < head, has_tail = j < n - tail_begin;
  const float xh = has_head ? load_one<DTI>(d.in, j) : 0.0f;
  const float xt = has_tail ? load_one<DTI>(d.in, tail_begin + j) : 0.0f;
  Acc<ACC> acc[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) acc[k].zero();
  if constexpr (ACC == ACC_SOFTMAX) {
    softmax_add_held<DTI, NA, KQ>(acc, r, j, 16, nvec);
  } else {
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
      if (j + k * 16 < nvec) {
        float x[VEC];
        widen<DTI>(r[k], x);
#pragma unroll
        for (int c = 0; c < VEC; ++c) acc[(k * VEC + c) % NA].add(x[c]);
      }
    }
  }
  if (has_head) acc[0].add(xh);
  if (has_tail) acc[0].add(xt);
  merge_chains<ACC, NA>(acc);
  const RowMap<ACC> f = RowMap<ACC>::of(row16_reduce<ACC>(acc[0]));  // the same in the row's 16 lanes
  if constexpr (ACC == ACC_SOFTMAX) {
    if (lse && j == 0) *lse = f.lse();
  }
  const bool vec_ok = out_vector_ok<DTI, DTO>(d.out, head);
  auto write = [&](auto non_temporal) {
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
      const int v = j + k * 16;
      if (v < nvec) {
        float x[VEC], q[VEC];
        widen<DTI>(r[k], x);
#pragma unroll
        for (int c = 0; c < VEC; ++c) q[c] = f(x[c]);
        store_quotients<DTI, DTO, decltype(non_temporal)::value>(d.out, head, v, vec_ok, q);
      }
    }
  };
  if (nt) write(std::true_type());
  else write(std::false_type());
  if (has_head) store_one<DTO>(d.out, j, f(xh));
  if (has_tail) store_one<DTO>(d.out, tail_begin + j, f(xt));
}

// The dtype switch of a row of each 16-lane group: it may differ between the
// groups (row tables), never within one.
template <int ACC>
__device__ __forceinline__ void dispatch_quarter(const RowDesc& d, float* lse) {
  if constexpr (ACC == ACC_SOFTMAX) {
    quarter_row<NRM_F32, NRM_F32, ACC>(d, lse);
  } else {
#define NRM_QR(I, O) quarter_row<I, O, ACC>(d, lse)
    switch (d.in_dt * 3 + d.out_dt) {
      case NRM_F32 * 3 + NRM_F32: NRM_QR(NRM_F32, NRM_F32); break;
      case NRM_F32 * 3 + NRM_BF16: NRM_QR(NRM_F32, NRM_BF16); break;
      case NRM_F32 * 3 + NRM_F16: NRM_QR(NRM_F32, NRM_F16); break;
      case NRM_BF16 * 3 + NRM_F32: NRM_QR(NRM_BF16, NRM_F32); break;
      case NRM_BF16 * 3 + NRM_BF16: NRM_QR(NRM_BF16, NRM_BF16); break;
      case NRM_BF16 * 3 + NRM_F16: NRM_QR(NRM_BF16, NRM_F16); break;
      case NRM_F16 * 3 + NRM_F32: NRM_QR(NRM_F16, NRM_F32); break;
      case NRM_F16 * 3 + NRM_BF16: NRM_QR(NRM_F16, NRM_BF16); break;
      default: NRM_QR(NRM_F16, NRM_F16); break;
    }
#undef NRM_QR
  }
}

// Block b takes rows [b * R, (b + 1) * R), R = rows_per_block (1..8: one row
// per wavefront; 32: four), chosen by the host from the batch's size. No block
// waits for another, so the grid is as large as the batch and streams the rows
// in dispatch order.
//
// First each wavefront runs its own rows of at most QUARTER_MAX elements, all
// at once on 16 lanes each, then rows of at most wave_max: with one row per
// wavefront its own, with four the block's, dealt out in turn, since one
// wavefront may hold four of them and its neighbour none. For that the block's
// barrier stands before the rows there (200,000 rows of up to 4096: 163 us, 175
// with own rows only; 2^20 rows of 17: 118 and 138; 2^20 of 256: 346 and 353);
// with one row each it stands behind them (8 rows per block, 100,000 rows of 100
// to 3000: 149 us, before them 160; 2^17 rows of 2048: 356 either way. Blocks that
// rows of that length do not fill lose by it, 4 per block 398 and 355 us, but such
// blocks are left to longer rows, which the block runs: 65536 x 3000 290 either way).
// It then appends its rows of more than run_max elements to the lists:
// the segments of a resident row (one for a row of at most 2^RES_LOG2 elements;
// resident rows off, a single-pass row's one entry) to `shorts`, a long row's
// tiles to `tiles`; a row's entries are consecutive, the order of the rows in
// a list does not matter to any result. Then the block runs its rows of up to
// run_max one after the other.
//
// What bounds it: with many short rows HBM (2^20 rows of 256 binary32, 2.16 GB:
// 348 us per call launched directly, 6.2 TB/s, 358 replayed, against 572 us in six
// launches over planned tables), with few the launch and the chain of dependent loads (offsets,
// elements; 64 rows of up to 256: 4.1 us per call). 80 registers, three blocks
// per CU: spilling any of them cost more than a block less (2^20 rows of 256:
// 361 us with none, 523 us with 29).
template <int ACC>
__global__ void __launch_bounds__(ROWS_BLOCK) __attribute__((amdgpu_waves_per_eu(6))) batch_rows_kernel(BatchArgs a) {
  __shared__ Acc<ACC> slots[MAX_WAVES];
  __shared__ RowRes s_bcast;
  __shared__ RowDesc s_rows[ROWS_MAX];   // by the row's place in the block
  __shared__ uint32_t s_at[ROWS_MAX];    // each listed row's first entry after the block's base
  __shared__ int64_t s_base_tiles, s_base_shorts, s_base_lrows;
  const BatchHeader& h = a.header;
  const int t = threadIdx.x, lane = t & 63, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t nrows = h.nrows;
  const int R = h.rows_per_block;
  const int64_t block = (int64_t)blockIdx.y * h.grid_x + blockIdx.x;
  if (block == 0 && t == 0) {
    const int64_t blocks = (nrows + R - 1) / R;
    a.cnt[CNT_CALL_RUN] = a.cnt[CNT_CALL] + 1;
    a.cnt[CNT_TAKEN] = 0;
    a.cnt[CNT_LSE] = reinterpret_cast<int64_t>(h.lse);
    a.cnt[CNT_ORDERED] = blocks <= ORDERED_BLOCKS ? blocks : 0;
    if (nrows < 0 || nrows > a.cap_rows) atomicOr(a.error, NRM_DEVERR_CAPACITY);
  }
  if (nrows < 0 || nrows > a.cap_rows) return;
  const int64_t r0 = block * R;
  if (r0 >= nrows) return;
  const int here = nrows - r0 < R ? (int)(nrows - r0) : R;     // the block's rows
  const int rw = R > ROWS_WAVES ? ROWS_MAX / ROWS_WAVES : 1;   // rows per wavefront
  {
    const int own = wave * rw + grp;  // the 16 lanes' row
    RowDesc d;
    d.n = 0;
    if (grp < rw && own < here) {
      int err = 0;
      d = resolve_row(a, h, r0 + own, err);
      if ((lane & 15) == 0) {
        if (err) atomicOr(a.error, err);
        if (d.n == 0 && h.lse) h.lse[r0 + own] = -__builtin_inff();  // the log of an empty sum
        s_rows[own] = d;
      }
    }
    if (rw > 1) lds_barrier();
    if (d.n > 0 && d.n <= QUARTER_MAX && d.n <= a.wave_max)
      dispatch_quarter<ACC>(d, h.lse ? h.lse + (r0 + own) : nullptr);
  }
  // every wavefront sees the same rows: lane j the block's row j
  int64_t n = lane < here && (rw > 1 || lane == wave) ? s_rows[lane].n : 0;
  {
    const uint32_t waves = (uint32_t)__ballot(n > QUARTER_MAX && n <= a.wave_max);
    uint32_t k = rw > 1 ? 0 : wave;
    for (uint32_t m = waves; m; m &= m - 1, ++k) {
      if (k % ROWS_WAVES != wave) continue;
      const int j = __builtin_ctz(m);
      dispatch_wave<ACC>(uniform_desc(s_rows[j]), h.lse ? h.lse + (r0 + j) : nullptr);
    }
  }
  if (rw == 1) {
    lds_barrier();
    n = lane < here ? s_rows[lane].n : 0;
  }
  if (n <= a.wave_max) n = 0;
  const uint32_t kept = (uint32_t)__ballot(n > 0), list = (uint32_t)__ballot(n > h.run_max);
  if (list) {
    const int64_t call = a.cnt[CNT_CALL] + 1;
    // where kernels of their own take the long rows, these are listed too
    const uint32_t longs = !a.res_on || a.apart ? (uint32_t)__ballot(n > h.run_max && n > a.short_max) : 0u;
    if (wave == 0) {
      const bool listed = n > h.run_max, is_long = listed && n > a.short_max;
      const uint32_t tiles = is_long ? (uint32_t)long_tiles(n, a.short_max, a.tile_log2) : 0u;
      const uint32_t shorts = listed && !is_long ? (a.res_on ? (uint32_t)row_segments(n) : 1u) : 0u;
      const uint32_t it = wave_scan32(tiles, lane), is = wave_scan32(shorts, lane);
      if (lane < ROWS_MAX) s_at[lane] = is_long ? it - tiles : is - shorts;
      if (lane == 63) {
        unsigned long long* lists = reinterpret_cast<unsigned long long*>(list_counters(a, call));
        unsigned long long bt = 0, bs = 0;
        if (it)
          bt = __hip_atomic_fetch_add(lists + LIST_TILES * CNT_LINE, (unsigned long long)it, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
        if (is)
          bs = __hip_atomic_fetch_add(lists + LIST_SHORT * CNT_LINE, (unsigned long long)is, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
        if (longs)
          s_base_lrows = (int64_t)__hip_atomic_fetch_add(lists + LIST_LONG_ROWS * CNT_LINE,
                                                         (unsigned long long)__popc(longs), __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
        s_base_tiles = (int64_t)bt;
        s_base_shorts = (int64_t)bs;
        if (block < ORDERED_BLOCKS) a.block_shorts[block] = BlockShorts{(int64_t)bs, (int64_t)is};
      }
    }
    lds_barrier();
    int k = 0;
    for (uint32_t m = list; m; m &= m - 1, ++k) {
      if (k % ROWS_WAVES != wave) continue;
      const int j = __builtin_ctz(m);
      const RowDesc x = uniform_desc(s_rows[j]);
      const int32_t row = (int32_t)(r0 + j);
      const bool is_long = x.n > a.short_max;
      const int64_t count = is_long ? long_tiles(x.n, a.short_max, a.tile_log2)
                            : a.res_on ? row_segments(x.n)
                                       : 1;
      const int64_t first = (is_long ? s_base_tiles : s_base_shorts) + s_at[j];
      Item* to = is_long ? a.tiles : a.shorts;
      // rows that overlap one another can need more entries than the capacity
      // allows for: such a row is skipped, its entries inside the list empty
      const bool fits = first + count <= a.cap_items;
      for (int64_t i = lane; i < count && first + i < a.cap_items; i += 64)
        to[first + i] = Item{x, fits ? row : -1, (int32_t)i};
      if (lane == 0) {
        if (!fits) atomicOr(a.error, NRM_DEVERR_CAPACITY);
        if (longs >> j & 1) a.lrow_first[s_base_lrows + __popc(longs & ((1u << j) - 1))] = fits ? first : -1;
      }
    }
  } else if (t == 0 && block < ORDERED_BLOCKS) {
    a.block_shorts[block] = BlockShorts{0, 0};
  }
  for (uint32_t m = kept & ~list; m; m &= m - 1) {
    const int j = __builtin_ctz(m);
    const ResExchange none{nullptr, nullptr, nullptr, 0, nullptr, nullptr};
    dispatch_resident<ACC, true>(uniform_desc(s_rows[j]), 0, none, slots, &s_bcast, h.lse ? h.lse + (r0 + j) : nullptr);
    lds_barrier();  // slots and s_bcast are reused
  }
}

template <int ACC>
hipError_t launch_lists(const BatchPlan& p, const BatchArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((batch_rows_kernel<ACC>), dim3((unsigned)p.rows_grid, (unsigned)p.rows_grid_y), dim3(ROWS_BLOCK), 0,
                     s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !p.lists) return e;
  if (a.res_on) {
    hipLaunchKernelGGL((batch_resident_kernel<ACC>), dim3((unsigned)p.res_grid), dim3(RES_BLOCK), 0, s, a);
    e = hipGetLastError();
    if (e != hipSuccess || !a.apart) return e;
    hipLaunchKernelGGL((batch_tile_sums_kernel<ACC>), dim3(SUMS_GRID), dim3(RES_BLOCK), 0, s, a);
    hipLaunchKernelGGL((batch_tile_totals_kernel<ACC>), dim3(TOTALS_GRID), dim3(RES_BLOCK), 0, s, a);
    return phase2_acc<ACC>(p, a, s);
  }
  e = phase1_u<ACC>(p, a, s);
  if (e != hipSuccess) return e;
  e = rowsum_acc<ACC>(p, a, s);
  if (e != hipSuccess) return e;
  return phase2_acc<ACC>(p, a, s);
}

// ---- the plain path's single-launch form for small n ---------------------------------
// One 1024-thread block holds the whole input in registers (SMALL_ELEMS
// elements: 16 vectors per thread for binary32, 8 for 2-byte inputs, which
// keeps the widened values in registers), reduces it, and divides from the
// registers: one read, one write, one launch. The sum is left in sum_out for
// nrm_get_last_sum.
constexpr int64_t SMALL_ELEMS = 65536;

template <int DTI, int DTO, int ACC>
__global__ void __launch_bounds__(1024) small_normalize_kernel(RowDesc d, float* sum_out) {
  __shared__ Acc<ACC> slots[MAX_WAVES];
  __shared__ RowRes s_bcast;
  constexpr int KB = (int)(SMALL_ELEMS / 1024 / Elem<DTI>::VEC);
  single_pass<DTI, DTO, ACC, KB>(d, slots, &s_bcast, nullptr, 0);
  if (threadIdx.x == 0) sum_out[0] = s_bcast.a;  // single_pass ended after the broadcast's barrier
}

template <int ACC>
hipError_t small_acc(const RowDesc& d, float* sum_out, hipStream_t s) {
#define NRM_SK(I, O) hipLaunchKernelGGL((small_normalize_kernel<I, O, ACC>), dim3(1), dim3(1024), 0, s, d, sum_out)
  switch (d.in_dt * 3 + d.out_dt) {
    case NRM_F32 * 3 + NRM_F32: NRM_SK(NRM_F32, NRM_F32); break;
    case NRM_F32 * 3 + NRM_BF16: NRM_SK(NRM_F32, NRM_BF16); break;
    case NRM_F32 * 3 + NRM_F16: NRM_SK(NRM_F32, NRM_F16); break;
    case NRM_BF16 * 3 + NRM_F32: NRM_SK(NRM_BF16, NRM_F32); break;
    case NRM_BF16 * 3 + NRM_BF16: NRM_SK(NRM_BF16, NRM_BF16); break;
    case NRM_BF16 * 3 + NRM_F16: NRM_SK(NRM_BF16, NRM_F16); break;
    case NRM_F16 * 3 + NRM_F32: NRM_SK(NRM_F16, NRM_F32); break;
    case NRM_F16 * 3 + NRM_BF16: NRM_SK(NRM_F16, NRM_BF16); break;
    default: NRM_SK(NRM_F16, NRM_F16); break;
  }
#undef NRM_SK
  return hipGetLastError();
}

// ---- the plain path's single-launch form for mid-size n ---------------------------------
// n in (small_n, 2^20]: one block per segment of the input, at most
// PRES_MAX_SEGMENTS of them, each held in registers from its read to its write
// while the blocks exchange their segment sums: every block reads every sum,
// one lane of a wavefront per segment. Two transfers and one launch instead of
// three and two. The call number that tags the sums lives in the workspace; the
// last block to arrive moves it on (every block read it before arriving), so
// consecutive calls on one workspace never read each other's sums.
//
// The blocks need not all be able to run at once. A segment belongs to the block
// that publishes its sum, by a compare-and-swap against the slot's word as it
// read it meanwhile. A block that has waited PRES_PATIENCE polls takes a segment
// whose sum is missing, reads it and publishes its sum, waits again, and in the
// end divides all segments that are its own: one running block alone ends the
// call. Nothing is written before every sum is published, so a block that starts
// late, and reads elements already divided in place, finds its slot taken or its
// swap fails.
//
// Launch and exchange latency bound it. A short input takes segments of 2^12
// elements on 256 threads (more CUs load at once), one of more than
// PRES_SHORT_MAX segments of 2^14 on 512, which keeps the sums of 2^20
// elements within one wavefront's lanes and the launch within 64 blocks.
// Per call back to back, one box: 2^16 binary32 4.7 us, 2^18 5.2, 2^19 6.3, 2^20 6.9
// (8.1 us at 2^19 and 8.4 at 2^20 for the two kernels); 2^20 bfloat16 6.8. The
// compensated sum's longer chains lose from 2^20 on (8.2 against 7.7 us; 2^19: 7.3
// and 7.7), so it stops at 2^19. The call that takes over is kept off the common
// path: in one loop with it, 2^19 binary32 took 6.4 to 7.0 us and 2^20 bfloat16 7.3
// to 7.8. The slot is looked at after the elements are requested (before: 6.6 and 6.9).
constexpr int PRES_BLOCK = 256;
constexpr int PRES_LOG2 = 12;
constexpr int PRES_MAX_SEGMENTS = 64;
constexpr int64_t PRES_SHORT_MAX = (int64_t)PRES_MAX_SEGMENTS << PRES_LOG2;
// Polls (about 1 us each) before a block takes another segment: longer than
// blocks of one launch start apart on a free device, short beside a foreign
// kernel that keeps some of them out.
constexpr uint32_t PRES_PATIENCE = 1u << 10;

// Wavefront 0, lane l: wait for the sum of segment l. Returns the mask of the
// segments without one after `patience` polls; 0: *total is the sum of all,
// in every lane, in an order that depends only on nseg.
template <int ACC>
__device__ __forceinline__ uint64_t gather_segments(const unsigned long long* words, uint32_t ep, int nseg,
                                                    uint32_t patience, Acc<ACC>* total) {
  const int lane = threadIdx.x & 63;
  float f[2] = {0.0f, 0.0f};
  bool have = lane >= nseg;
  for (uint32_t spin = 0;; ++spin) {
    if (!have) {
      have = true;
#pragma unroll
      for (int w = 0; w < Tagged<ACC>::WORDS; ++w) {
        const unsigned long long v =
            __hip_atomic_load(words + 2 * lane + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        f[w] = f32_bits((uint32_t)v);
        have = have && (uint32_t)(v >> 32) == ep;
      }
    }
    const uint64_t missing = __ballot(!have);
    if (missing && spin < patience) {
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    if (missing) return missing;
    Acc<ACC> v;
    if (lane < nseg) v = Tagged<ACC>::join(f);
    else v.zero();
    *total = wave_reduce<ACC>(v);
    return 0;
  }
}

// One thread: publish a segment's sum in place of the words seen before; true
// if the segment is now this block's. (Each word on its own: two blocks that
// both find a word unpublished have summed the same elements.)
template <int ACC>
__device__ __forceinline__ bool claim_tagged(unsigned long long* words, unsigned long long (&seen)[2], uint32_t ep,
                                             const Acc<ACC>& v) {
  float f[2];
  Tagged<ACC>::split(v, f);
  bool won[2] = {false, false};
#pragma unroll
  for (int w = 0; w < Tagged<ACC>::WORDS; ++w)
    if ((uint32_t)(seen[w] >> 32) != ep)
      won[w] = __hip_atomic_compare_exchange_strong(words + w, &seen[w], ((unsigned long long)ep << 32) | bits_f32(f[w]),
                                                    __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return won[0];
}

// What the blocks of one call meet over.
template <int ACC>
struct PlainExchange {
  PlainResidentWs w;
  uint32_t ep;  // the call's tag: never 0, the value of a slot that was never written
  int nseg;
  Acc<ACC>* slots;
  RowRes* s_bcast;
  uint64_t* s_mine;  // the segments that are this block's
  int* s_next;       // the one to take next, -1: every sum is known

  // The slot's words, before the segment's sum is known; thread 0.
  __device__ __forceinline__ void look(int seg, unsigned long long (&seen)[2]) const {
    seen[0] = seen[1] = 0;
    if (threadIdx.x == 0) {
#pragma unroll
      for (int k = 0; k < Tagged<ACC>::WORDS; ++k)
        seen[k] = __hip_atomic_load(w.slots + 2 * seg + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // Publish the segment's sum, then wait for the others: the result in *s_bcast
  // and this block's arrival, or the segment to take next. Every thread.
  __device__ __forceinline__ int meet(int seg, unsigned long long (&seen)[2], const Acc<ACC>& tot, uint64_t& mine,
                                      uint32_t patience) const {
    if (threadIdx.x < 64) {
      bool won = false;
      if (threadIdx.x == 0) won = claim_tagged<ACC>(w.slots + 2 * seg, seen, ep, tot);
      Acc<ACC> total;
      uint64_t missing = gather_segments<ACC>(w.slots, ep, nseg, patience, &total);
      if (won) mine |= 1ull << seg;
      if (threadIdx.x == 0) {
        *s_mine = mine;
        *s_next = -1;
        if (missing) {
          // blocks that wait for the same segments take different ones first
          for (int skip = blockIdx.x % __popcll(missing); skip > 0; --skip) missing &= missing - 1;
          *s_next = __ffsll((unsigned long long)missing) - 1;
        } else {
          *s_bcast = RowMap<ACC>::of(total).result();
          if (__hip_atomic_fetch_add(w.arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == w.blocks - 1) {
            __hip_atomic_store(w.arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(w.call, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
    }
    lds_barrier();
    return __builtin_amdgcn_readfirstlane(*s_next);
  }
};

template <int DTI, int DTO, int ACC, int BLOCK, int LOG2>
__global__ void __launch_bounds__(BLOCK) plain_resident_kernel(RowDesc d, PlainResidentWs w) {
  __shared__ Acc<ACC> slots[MAX_WAVES];
  __shared__ RowRes s_bcast;
  __shared__ uint64_t s_mine;
  __shared__ int s_next;
  const unsigned long long call = __hip_atomic_load(w.call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const PlainExchange<ACC> x{w,     (uint32_t)(call % 0xFFFFFFFFull) + 1u, (int)((d.n + (1 << LOG2) - 1) >> LOG2),
                             slots, &s_bcast, &s_mine, &s_next};
  const int seg = blockIdx.x;
  unsigned long long seen[2];
  Held<DTI, DTO, ACC, BLOCK, LOG2> h;
  h.load(d, seg);
  x.look(seg, seen);
  const Acc<ACC> tot = h.sum(slots);
  uint64_t mine = 0;
  int next = -1;
  if (x.nseg > 1) {
    next = x.meet(seg, seen, tot, mine, PRES_PATIENCE);
  } else {  // nothing to exchange
    if (threadIdx.x == 0) {
      s_bcast = RowMap<ACC>::of(tot).result();
      s_mine = 1;
    }
    lds_barrier();
  }
  if (__builtin_expect(next < 0, 1)) {
    if (uniform64((int64_t)s_mine) != 0) h.divide(RowMap<ACC>::of(s_bcast));
  } else {
    while (next >= 0) {
      const int take = next;
      lds_barrier();  // slots, s_mine and s_next are reused
      x.look(take, seen);
      h.load(d, take);
      next = x.meet(take, seen, h.sum(slots), mine, 1);  // having waited once, one after the other
    }
    for (uint64_t own = (uint64_t)uniform64((int64_t)s_mine); own; own &= own - 1) {
      h.load(d, __ffsll((unsigned long long)own) - 1);
      h.divide(RowMap<ACC>::of(s_bcast));
    }
  }
  if (threadIdx.x == 0 && blockIdx.x == 0) w.sum_out[0] = s_bcast.a;  // the invariant, for nrm_get_last_sum
}

template <int ACC, int BLOCK, int LOG2>
hipError_t plain_resident_acc(const RowDesc& d, PlainResidentWs w, hipStream_t s) {
  const unsigned segments = (unsigned)((d.n + (int64_t(1) << LOG2) - 1) >> LOG2);
  if (w.blocks == 0 || w.blocks > segments) w.blocks = segments;
#define NRM_PR(I, O) \
  hipLaunchKernelGGL((plain_resident_kernel<I, O, ACC, BLOCK, LOG2>), dim3(w.blocks), dim3(BLOCK), 0, s, d, w)
  switch (d.in_dt * 3 + d.out_dt) {
    case NRM_F32 * 3 + NRM_F32: NRM_PR(NRM_F32, NRM_F32); break;
    case NRM_F32 * 3 + NRM_BF16: NRM_PR(NRM_F32, NRM_BF16); break;
    case NRM_F32 * 3 + NRM_F16: NRM_PR(NRM_F32, NRM_F16); break;
    case NRM_BF16 * 3 + NRM_F32: NRM_PR(NRM_BF16, NRM_F32); break;
    case NRM_BF16 * 3 + NRM_BF16: NRM_PR(NRM_BF16, NRM_BF16); break;
    case NRM_BF16 * 3 + NRM_F16: NRM_PR(NRM_BF16, NRM_F16); break;
    case NRM_F16 * 3 + NRM_F32: NRM_PR(NRM_F16, NRM_F32); break;
    case NRM_F16 * 3 + NRM_BF16: NRM_PR(NRM_F16, NRM_BF16); break;
    default: NRM_PR(NRM_F16, NRM_F16); break;
  }
#undef NRM_PR
  return hipGetLastError();
}

template <int ACC>
hipError_t plain_resident_size(const RowDesc& d, const PlainResidentWs& w, hipStream_t s) {
  return d.n <= PRES_SHORT_MAX ? plain_resident_acc<ACC, PRES_BLOCK, PRES_LOG2>(d, w, s)
                               : plain_resident_acc<ACC, RES_BLOCK, RES_LOG2>(d, w, s);
}

}  // namespace

int64_t small_capacity(int) { return SMALL_ELEMS; }
int64_t plain_resident_capacity(int acc) {
  return ((int64_t)PRES_MAX_SEGMENTS << RES_LOG2) >> (acc == NRM_ACC_KAHAN ? 1 : 0);
}

hipError_t launch_plain_resident(const void* in, int in_dt, void* out, int out_dt, int64_t n, int acc,
                                 const PlainResidentWs& w, hipStream_t s) {
  RowDesc d;
  d.in = static_cast<const char*>(in);
  d.out = static_cast<char*>(out);
  d.n = n;
  d.in_dt = in_dt;
  d.out_dt = out_dt;
  return acc == NRM_ACC_KAHAN ? plain_resident_size<NRM_ACC_KAHAN>(d, w, s) : plain_resident_size<NRM_ACC_F32>(d, w, s);
}

hipError_t launch_small(const void* in, int in_dt, void* out, int out_dt, int64_t n, int acc, float* sum_out,
                        hipStream_t s) {
  RowDesc d;
  d.in = static_cast<const char*>(in);
  d.out = static_cast<char*>(out);
  d.n = n;
  d.in_dt = in_dt;
  d.out_dt = out_dt;
  return acc == NRM_ACC_KAHAN ? small_acc<NRM_ACC_KAHAN>(d, sum_out, s) : small_acc<NRM_ACC_F32>(d, sum_out, s);
}

hipError_t launch_batch(const BatchPlan& p, const BatchArgs& a, hipStream_t s) {
  switch (p.acc) {
    case NRM_ACC_KAHAN: return launch_lists<NRM_ACC_KAHAN>(p, a, s);
    case ACC_SOFTMAX: return launch_lists<ACC_SOFTMAX>(p, a, s);
    default: return launch_lists<NRM_ACC_F32>(p, a, s);
  }
}

const void* rows_kernel(int acc) {
  switch (acc) {
    case NRM_ACC_KAHAN: return reinterpret_cast<const void*>(&batch_rows_kernel<NRM_ACC_KAHAN>);
    case ACC_SOFTMAX: return reinterpret_cast<const void*>(&batch_rows_kernel<ACC_SOFTMAX>);
    default: return reinterpret_cast<const void*>(&batch_rows_kernel<NRM_ACC_F32>);
  }
}

}  // namespace nrm
