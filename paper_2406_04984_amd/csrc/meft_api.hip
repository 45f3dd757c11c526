// Host side of libmeft: argument validation, workspace layout and kernel launches behind the C ABI
// declared in include/meft.h.  Nothing here computes on the host; every step of the layer runs in
// the kernels of the headers included below.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/meft.h"
#include "adam.h"
#include "common.h"
#include "dense_path.h"
#include "dispatch.h"
#include "few_tokens.h"
#include "gather.h"
#include "gemm_nt.h"
#include "router.h"
#include "scatter.h"
#include "select.h"
#include "small_groups.h"
#include "union_path.h"

// Device memory of meft_route_static: part of the library's image, one copy on every GPU the library runs on.  In
// host code this name is only a handle for hipGetSymbolAddress; kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[MEFT_ROUTE_STATIC_BYTES];

namespace meft {
namespace {

// The host side of every entry point that enqueues work or touches the library's few pieces of process-wide state
// (the timing list, the side stream and events of the host-resident variant, the table of staged workspaces) runs
// under this lock, so the entry points may be called from several host threads.
std::mutex g_api_mutex;
#define MEFT_API_LOCK() std::lock_guard<std::mutex> api_lock_(g_api_mutex)

// ---- per-kernel timing ----------------------------------------------------------------------
struct ProfEntry {
  const char* name;
  hipEvent_t start, stop;
};
bool g_prof_on = false;
std::vector<ProfEntry> g_prof;

struct LaunchScope {
  hipStream_t st;
  bool on;
  hipEvent_t stop{};
  LaunchScope(const char* name, hipStream_t s) : st(s), on(g_prof_on) {
    if (!on) return;
    ProfEntry e{name, nullptr, nullptr};
    if (hipEventCreate(&e.start) != hipSuccess || hipEventCreate(&e.stop) != hipSuccess) {
      on = false;
      return;
    }
    (void)hipEventRecord(e.start, st);
    stop = e.stop;
    g_prof.push_back(e);
  }
  ~LaunchScope() {
    if (on) (void)hipEventRecord(stop, st);
  }
};

#define MEFT_LAUNCH(name, kernel, grid, block, shmem, stream, ...)            \
  do {                                                                        \
    LaunchScope scope_(name, stream);                                         \
    hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);      \
  } while (0)

// ---- shape checks ---------------------------------------------------------------------------
constexpr int kMaxD = 16384, kMaxBlocks = 16384;
constexpr int kMaxC = 1 << 22;      // candidates per token (top_e * block_size)
// few out of more candidates than this: topk_select_bound_kernel, whose 1024 threads need four each.  Forward without the
// value sum, 2048 tokens, registers / bound: 16 of 4160 75 / 60 us, 64 of 4160 78 / 68, 256 of 4160 85 / 82, 256 of 12288
// 168 / 142.
constexpr int kBoundMinC = 4096;
constexpr int kMaxLdsC = 12288;     // up to here the top-k selection keeps a token's keys in LDS

meft_status check_shape(const meft_shape* s) {
  if (!s) return MEFT_ERR_INVALID_ARG;
  if (s->T < 0 || s->d < 1 || s->n_blocks < 1 || s->block_size < 1 || s->N < 1) return MEFT_ERR_INVALID_ARG;
  if ((int64_t)s->n_blocks * s->block_size != (int64_t)s->N) return MEFT_ERR_INVALID_ARG;
  if (s->top_e < 1 || s->top_e > s->n_blocks) return MEFT_ERR_INVALID_ARG;
  const int64_t C = (int64_t)s->top_e * s->block_size;
  if (s->top_k < 1 || s->top_k > C) return MEFT_ERR_INVALID_ARG;
  if ((int64_t)s->T * s->top_k >= (1ll << 31) || (int64_t)s->T * C >= (1ll << 31)) return MEFT_ERR_INVALID_ARG;
  if (s->dtype != MEFT_F32 && s->dtype != MEFT_BF16) return MEFT_ERR_INVALID_ARG;
  if (s->activation != 0) return MEFT_ERR_INVALID_ARG;
  if (s->flags & ~(uint32_t)(MEFT_FLAG_HOST_KV | MEFT_FLAG_KEEP_STAGED | MEFT_FLAG_PRESTAGED | MEFT_FLAG_REUSE_FWD))
    return MEFT_ERR_INVALID_ARG;
  if ((s->flags & (MEFT_FLAG_KEEP_STAGED | MEFT_FLAG_PRESTAGED)) && !(s->flags & MEFT_FLAG_HOST_KV))
    return MEFT_ERR_INVALID_ARG;
  if (s->d % 8 != 0 || s->d > kMaxD || C > kMaxC || s->n_blocks > kMaxBlocks) return MEFT_ERR_UNSUPPORTED;
  return MEFT_OK;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---- workspace layout -----------------------------------------------------------------------
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base(static_cast<char*>(b)) {}
  template <typename T>
  T* take(size_t n) {
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += (n * sizeof(T) + 255) & ~(size_t)255;
    return p;
  }
};

// The matrix-core formulation (dense_path.h) is used for bf16 when the hidden size fits its k tiling and
// the selection is dense enough inside the chosen blocks; otherwise, and for fp32, the per-pair gather
// kernels are used.
// The score contraction alone runs on the matrix-core kernel of the block-dense path also for bf16 shapes that
// are not dense enough for the rest of it, when the groups are large enough to fill its 128-row tiles.
bool use_mfma_scores(const meft_shape& s) {
  return s.dtype == MEFT_BF16 && s.d % kTK == 0 && (int64_t)s.T * s.top_e >= (int64_t)128 * s.n_blocks;
}

bool use_dense(const meft_shape& s) {
  const int64_t C = (int64_t)s.top_e * s.block_size;
  return s.dtype == MEFT_BF16 && s.d % kTK == 0 && s.block_size >= 16 && (int64_t)s.top_k * 64 >= C &&
         C <= kMaxLdsC;
}

// The forward of a few tokens (few_tokens.h): as many entries as one workgroup looks through, and on average at most
// two 16-token tiles per block.  Such a forward leaves nothing in the workspace for the backward.
bool few_tokens(const meft_shape& s) {
  const int64_t n_ent = (int64_t)s.T * s.top_e;
  return n_ent <= kFewEntries && n_ent <= (int64_t)32 * s.n_blocks && s.top_e <= kFewMaxE && s.top_k <= kTopkEmitLds &&
         (int64_t)s.top_e * s.block_size <= kMaxLdsC;
}

int round64(int v) { return (v + 63) & ~63; }
// Block-dense path: groups of at most this many tokens go to the per-pair kernels of small_groups.h (0: none).  The
// tile schedule knows the small groups only where it deals the groups out longest first.
// A contraction reads all block_size rows of the block for a group, the per-pair kernels about top_k / top_e rows for
// each of its tokens: at top_e * block_size / top_k tokens both move the same bytes, so the limit is no larger.
int small_rows_of(const meft_shape& s) {
  if (!use_dense(s) || s.n_blocks > kSchedSortMax) return 0;
  const int64_t even = (int64_t)s.top_e * s.block_size / s.top_k;   // >= 1: top_k <= top_e * block_size
  return (int)(even < kSmallRows ? even : kSmallRows);
}
// per XCD: at most n_blocks groups (+1 end entry) and, as a bound that needs no knowledge of the deal, all m tiles
int sched_cap(const meft_shape& s) { return s.n_blocks + 1; }
int sched_max_tiles(const meft_shape& s) { return (int)(((int64_t)s.T * s.top_e) / kTMTok + s.n_blocks); }
// bound of the tile ids of a launch with tn n tiles per m tile (ids beyond the real ones find no tile)
int tile_bound(const meft_shape& s, int tn) {
  const int64_t b = (int64_t)kXcd * sched_max_tiles(s) * tn;
  return (int)(b < (int64_t)INT32_MAX ? b : (int64_t)INT32_MAX);
}

constexpr int kRouterSplitMax = 4;

// Slices of the hidden dimension in the untiled router contraction (router.h): at least four 64-byte steps per wave of a
// slice, one batch of loads.
int route_slices(const meft_shape& s) {
  const int steps = (int)(((int64_t)s.d * (s.dtype == MEFT_BF16 ? 2 : 4) + 63) / 64), want = steps / (4 * kRouteWaves);
  return want < 1 ? 1 : (want > kRouterSplitMax ? kRouterSplitMax : want);
}

// Whether the router contraction runs on LDS tiles: ProbRouter for bf16 rows of whole 64-element k tiles, gemm_nt.h
// otherwise.  The untiled one wins while the problem is small and then re-reads h (once per 64 blocks) and the router too
// often.  All times are of the whole route call, us, untiled / tiled.
bool route_on_tiles(const meft_shape& s) {
  // 64-byte steps of a row, and the steps the untiled one's waves go through: whole batches of four per wave and slice
  const int es = s.dtype == MEFT_BF16 ? 2 : 4;
  const int64_t steps = ((int64_t)s.d * es + 63) / 64, slices = (int64_t)route_slices(s) * kRouteWaves;
  const int64_t per = (steps + slices - 1) / slices, padded = slices * ((per + 3) / 4 * 4);
  if (s.dtype == MEFT_BF16 && s.d % kTK == 0) {
    // d 4096, 64 blocks: 11.0 / 18.6 at 1024 tokens, 20.3 / 20.1 at 4096, 39.1 / 23.5 at 8192; 256 blocks: 22.6 / 23.4 at
    // 1024, 69.5 / 27.6 at 4096
    if ((int64_t)s.T * s.n_blocks > 4096 * 64) return true;
    // Few blocks, many long rows: by two models in us, fitted to 60 shapes.  Untiled: by the steps, those that are only padding
    // counted half.  Tiled: the serial k tiles of a slice (one of `parts`; 1 or 2 where d / 64 is no multiple of 4), or h at
    // the copy rate.  8 blocks: d 4096 14.2 / 18.6 at 4096 tokens, 31.2 / 20.6 at 8192; d 4160 33.6 / 47 at 8192, 78 / 57 at
    // 20000; d 5120 (160 steps go as 256) 12.7 / 19 at 2048, 29.2 / 21 at 5000; d 8192 24.4 / 28.4 at 4096, 46.7 / 33.5 at
    // 8192; d 2048 14.0 / 15.0 at 8192, 50.4 / 42.3 at 32768.  Below d 2048 the ring's start outweighs a slice's few k tiles:
    // 28.4 / 32.1 at d 1024 and 32768 tokens.
    if (s.d < 2048 || (int64_t)s.T * s.d <= (int64_t)5 << 22) return false;
    const int kt = s.d / kTK, parts = kt % 4 == 0 ? 4 : (kt % 2 == 0 ? 2 : 1);
    const double untiled = 6.0 + (16.0 + s.n_blocks / 4.0) * 1e-6 * s.T * 0.5 * (double)(steps + padded);
    const double chain = 9.0 + 0.62 * kt / parts, stream = 6.0 + 2.0 * s.T * (double)s.d / 4.6e6;
    return untiled > 1.05 * (chain > stream ? chain : stream);
  }
  // The untiled time goes by tokens x groups of 64 blocks, and by the steps.  fp32: 64 blocks, d 768 18.4 / 19.5 at 4096 tokens,
  // 23.4 / 20.4 at 8192, 81 / 46 at 32768, d 4096 81 / 75 at 8192; 256 blocks, d 1024 24.5 / 24.7 at 2048, 80 / 54 at 8192;
  // 1024 blocks, d 512 51 / 42 at 2048; 8 blocks, d 1024 69 / 53 at 32768 (the tiled one is level from about 6000 tokens on;
  // the line takes it where it is ahead by a third at every size measured).  bf16, 16384 and 65536 tokens: d 1000 19.5 / 25.5
  // and 65 / 42, d 4104 85 / 68 and 385 / 142 (1024 blocks, 16384 tokens: 1404 / 274).
  const int64_t reads = (int64_t)s.T * ((s.n_blocks + 63) / 64);
  return reads * padded > (es == 2 ? 28672 : 16384) * steps;
}

struct RouteWs {
  float* p;
  size_t bytes;
  RouteWs(const meft_shape& s, void* ws) {
    Carver c(ws);
    p = c.take<float>((size_t)kRouterSplitMax * s.T * s.n_blocks);
    bytes = c.off;
  }
};

// the dispatch over chunks of whole tokens, at most 1024 entries each (dispatch.h): up to 1024 blocks and 2^20 entries
int disp_chunk_entries(const meft_shape& s) { return 1024 / s.top_e * s.top_e; }   // n_blocks <= 1024 only
int disp_chunks(const meft_shape& s) {
  const int epc = disp_chunk_entries(s);
  return (int)(((int64_t)s.T * s.top_e + epc - 1) / epc);
}
bool fast_dispatch(const meft_shape& s) { return s.n_blocks <= kDispMaxBlocks && (int64_t)s.T * s.top_e <= kDispMaxEntries; }

// index structures of the (token, block) dispatch, common to forward and backward
struct DispatchWs {
  int32_t* chunk_hist = nullptr;   // three-pass dispatch: [chunks][n_blocks]
  int32_t *sblk = nullptr, *cnt = nullptr, *group_off = nullptr, *tile_off = nullptr, *perm = nullptr,
          *tok_of_slot = nullptr, *slot_of_ent = nullptr, *sched_len = nullptr;
  int4* sched_pairs = nullptr;
  int2* sched_tiles = nullptr;
  // the groups of at most small_rows_of(s) tokens and their entries (small_groups.h), and the two list lengths
  int2* small_ent = nullptr;
  int32_t *small_grp = nullptr, *small_cnt = nullptr;
  void carve(const meft_shape& s, Carver& c) {
    const size_t n_ent = (size_t)s.T * s.top_e;
    sblk = c.take<int32_t>(n_ent);
    cnt = c.take<int32_t>(s.n_blocks);
    group_off = c.take<int32_t>((size_t)s.n_blocks + 1);
    tile_off = c.take<int32_t>((size_t)s.n_blocks + 1);
    perm = c.take<int32_t>(n_ent);
    tok_of_slot = c.take<int32_t>(n_ent + kSlotPad);   // padded: see kSlotPad
    slot_of_ent = c.take<int32_t>(n_ent);
    sched_len = c.take<int32_t>(kSchedLenInts);   // list lengths per XCD, the split flag, lengths without small groups
    sched_pairs = c.take<int4>((size_t)kXcd * sched_cap(s));
    sched_tiles = c.take<int2>((size_t)kXcd * sched_cap(s));
    chunk_hist = c.take<int32_t>(fast_dispatch(s) ? (size_t)disp_chunks(s) * s.n_blocks : 0);
    const size_t small = (size_t)small_rows_of(s);
    small_ent = c.take<int2>(small ? small * s.n_blocks : 0);
    small_grp = c.take<int32_t>(small ? (size_t)s.n_blocks : 0);
    small_cnt = c.take<int32_t>(small ? 2 : 0);
  }
};

// Block-dense path: what forward and backward both hold, at the same place in the workspace, so that a backward may
// take the forward's dispatch tables and activation rows as they are (MEFT_FLAG_REUSE_FWD).
struct DenseWs : DispatchWs {
  int32_t *flag = nullptr, *chunk_cnt = nullptr;
  uint16_t *zrow = nullptr, *Ap = nullptr, *DS = nullptr, *part = nullptr;
  float* ds32 = nullptr;   // activation gradients of the pairs of small groups, [T, top_k]
  // the touched flags and the row of zeros start from zero (adjacent in the workspace)
  size_t clear_words() const { return (size_t)(reinterpret_cast<char*>(Ap) - reinterpret_cast<char*>(flag)) / 4; }
  void carve_dense(const meft_shape& s, Carver& c) {
    carve(s, c);
    const size_t n_ent = (size_t)s.T * s.top_e;
    chunk_cnt = c.take<int32_t>((size_t)(s.N + kFlagChunk - 1) / kFlagChunk);
    flag = c.take<int32_t>(s.N);                               // flag and zrow adjacent: cleared by one fill
    // one piece: the row of zeros, A', DS', each row bsp elements, so that the zero row is row -1 of A' and row
    // -(n_ent + 1) of DS'
    const size_t bsp = round64(s.block_size);
    zrow = c.take<uint16_t>(bsp * (1 + 2 * n_ent));
    Ap = zrow ? zrow + bsp : nullptr;
    DS = zrow ? Ap + n_ent * bsp : nullptr;
    part = c.take<uint16_t>(n_ent * s.d);   // per-entry partial rows [T*e, d] bf16
    ds32 = c.take<float>((size_t)s.T * s.top_k);
  }
};

struct FwdWs : DenseWs {
  float* sc;
  size_t bytes;
  FwdWs(const meft_shape& s, void* ws) {
    Carver c(ws);
    if (use_dense(s)) carve_dense(s, c);
    else carve(s, c);
    sc = c.take<float>((size_t)s.T * s.top_e * s.block_size);
    bytes = c.off;
  }
};

// upper bound of the chunks of neurons with more than one chunk: such a neuron has more than kSegChunk pairs, so its
// ceil(L / kSegChunk) chunks are fewer than 2 L / kSegChunk
size_t seg_multi_chunks(const meft_shape& s) { return 2 * (((size_t)s.T * s.top_k) / kSegChunk) + 1; }

// Per-pair backward: whether the pairs are grouped by one launch (pair_one_kernel), and its buckets' neurons as a power of two
int pair_one_shift(const meft_shape& s) {
  int shift = 0;
  while ((s.N - 1) >> shift >= kPairOneBuckets) ++shift;
  return shift;
}
bool pair_one(const meft_shape& s) { return (int64_t)s.T * s.top_k <= kPairOneP && pair_one_shift(s) + kPairBits <= 32; }

struct BwdWs : DenseWs {
  // gather path
  float* ds;
  int32_t *cnt_n, *seg_off, *pair_list, *pair_sorted, *totals, *first;   // pair_sorted also holds the pairs' places (pair_count)
  int2* seg;         // (token, activation) of the pairs, segment by segment
  float* ds_part;    // partial activation gradients in the same order, one piece per group of column slices
  PairSums* sums;
  SegWork* work;     // at most one chunk per touched neuron plus one per kSegChunk pairs; pair_one: an entry per pair
  int4* multi;       // neurons of more than one chunk
  float* seg_part;   // fp32 chunk sums of the neurons with more than kSegChunk pairs: [chunk][dV | dK][d]
  size_t bytes;
  BwdWs(const meft_shape& s, void* ws) {
    Carver c(ws);
    const size_t P = (size_t)s.T * s.top_k;
    ds = nullptr; cnt_n = seg_off = pair_list = pair_sorted = totals = first = nullptr; seg_part = nullptr;
    sums = nullptr; work = nullptr; multi = nullptr; seg = nullptr; ds_part = nullptr;
    if (use_dense(s)) {
      carve_dense(s, c);
    } else {
      ds = c.take<float>(P);
      cnt_n = c.take<int32_t>(s.N);
      seg_off = c.take<int32_t>((size_t)s.N + 1);
      pair_list = c.take<int32_t>(P);
      pair_sorted = c.take<int32_t>(P);
      totals = c.take<int32_t>(3);
      sums = c.take<PairSums>(s.N > kScanSelfMax ? (size_t)(s.N + kScanChunk - 1) / kScanChunk : 0);
      const size_t n_seg = (size_t)s.N < P ? (size_t)s.N : P;
      work = c.take<SegWork>(pair_one(s) ? P : n_seg + P / kSegChunk + 1);
      first = c.take<int32_t>(pair_one(s) ? P : 0);
      multi = c.take<int4>(P / kSegChunk + 1);
      seg_part = c.take<float>(seg_multi_chunks(s) * 2 * (size_t)s.d);
      seg = c.take<int2>(P);
      const size_t slices = ((size_t)s.d * (s.dtype == MEFT_BF16 ? 2 : 4) + 1023) / 1024;
      ds_part = c.take<float>(P * (slices < kDsParts ? slices : kDsParts));
    }
    bytes = c.off;
  }
};

size_t compute_bytes(const meft_shape& s) {
  const size_t a = RouteWs(s, nullptr).bytes, b = FwdWs(s, nullptr).bytes, c = BwdWs(s, nullptr).bytes;
  const size_t m = a > b ? (a > c ? a : c) : (b > c ? b : c);
  return m < 256 ? 256 : m;
}

// With MEFT_FLAG_HOST_KV the workspace also holds device copies of K, V and device staging for dK, dV.
struct HostKvWs {
  char *Kd, *Vd, *dKd, *dVd;
  int32_t *pair_blk, *pair_blk_cnt;   // backward: block of every pair, pairs per block
  size_t bytes;
  HostKvWs(const meft_shape& s, void* ws) {
    Carver c(ws);
    c.off = compute_bytes(s);
    const size_t row_bytes = (size_t)s.d * (s.dtype == MEFT_BF16 ? 2 : 4);
    Kd = c.take<char>((size_t)s.N * row_bytes);
    Vd = c.take<char>((size_t)s.N * row_bytes);
    dKd = c.take<char>((size_t)s.N * row_bytes);
    dVd = c.take<char>((size_t)s.N * row_bytes);
    pair_blk = c.take<int32_t>((size_t)s.T * s.top_k);
    pair_blk_cnt = c.take<int32_t>(s.n_blocks);
    bytes = c.off;
  }
};

size_t workspace_bytes(const meft_shape& s) {
  return (s.flags & MEFT_FLAG_HOST_KV) ? HostKvWs(s, nullptr).bytes : compute_bytes(s);
}

// ---- host-resident keys/values: side streams, events, pinned read-back buffer (created on first use) ----
struct HostKvState {
  hipStream_t side = nullptr;   // K, V on their way in
  hipStream_t back = nullptr;   // dV on its way out while a later layer's blocks are on their way in (rows_stream)
  hipEvent_t ev_entry = nullptr, ev_cnt = nullptr, ev_k = nullptr, ev_v = nullptr, ev_dv = nullptr, ev_out = nullptr;
  int32_t* host_cnt = nullptr;
  bool ready = false;
};
HostKvState g_hkv;

bool hostkv_init() {
  if (g_hkv.ready) return true;
  hipStream_t* streams[2] = {&g_hkv.side, &g_hkv.back};
  for (hipStream_t* st : streams)
    if (!*st && hipStreamCreateWithFlags(st, hipStreamNonBlocking) != hipSuccess) return false;
  hipEvent_t* evs[6] = {&g_hkv.ev_entry, &g_hkv.ev_cnt, &g_hkv.ev_k, &g_hkv.ev_v, &g_hkv.ev_dv, &g_hkv.ev_out};
  for (hipEvent_t* e : evs)
    if (!*e && hipEventCreateWithFlags(e, hipEventDisableTiming) != hipSuccess) return false;
  if (hipHostMalloc(reinterpret_cast<void**>(&g_hkv.host_cnt), (size_t)kMaxBlocks * sizeof(int32_t), hipHostMallocDefault) !=
      hipSuccess)
    return false;
  g_hkv.ready = true;
  return true;
}

// Workspaces whose K, V copies were requested ahead of their forward (meft_hostkv_stage), each with the events
// that follow its K and its V copies.
struct StageSlot {
  const void* ws = nullptr;
  hipEvent_t ev_k = nullptr, ev_v = nullptr;
};
constexpr int kStageSlots = 16;
StageSlot g_slots[kStageSlots];
int g_slot_next = 0;

StageSlot* stage_slot(const void* ws, bool create) {
  for (StageSlot& sl : g_slots)
    if (sl.ws == ws) return &sl;
  if (!create) return nullptr;
  StageSlot& sl = g_slots[g_slot_next];
  g_slot_next = (g_slot_next + 1) % kStageSlots;
  if (!sl.ev_k && hipEventCreateWithFlags(&sl.ev_k, hipEventDisableTiming) != hipSuccess) return nullptr;
  if (!sl.ev_v && hipEventCreateWithFlags(&sl.ev_v, hipEventDisableTiming) != hipSuccess) return nullptr;
  sl.ws = ws;
  return &sl;
}

// The stream on which dV leaves early: on the one that carries blocks in it would queue behind those that were requested
// for a forward still to come.  Where there are none it is the better one (10.10 against 10.12 ms for a step of 2048 tokens,
// d 4096, 32 blocks of 512: a stream that has been idle takes a while to start).
hipStream_t rows_stream() {
  for (const StageSlot& sl : g_slots)
    if (sl.ws) return g_hkv.back;
  return g_hkv.side;
}

// Reads the per-block entry counts back (the host blocks until the work queued on `st` so far has produced them),
// then copies the blocks that some token uses, in runs of neighbouring blocks, from the pinned host matrices to their
// device copies on the side stream: `first` before `second`, each followed by its event.
meft_status hostkv_fetch(const meft_shape& s, const int32_t* cnt_dev, const void* first_host, char* first_dev,
                         hipEvent_t first_ev, const void* second_host, char* second_dev, hipEvent_t second_ev,
                         hipStream_t st) {
  HostKvState& k = g_hkv;
  if (hipMemcpyAsync(k.host_cnt, cnt_dev, (size_t)s.n_blocks * sizeof(int32_t), hipMemcpyDeviceToHost, st) != hipSuccess)
    return MEFT_ERR_DEVICE;
  if (hipEventRecord(k.ev_cnt, st) != hipSuccess || hipEventSynchronize(k.ev_cnt) != hipSuccess) return MEFT_ERR_DEVICE;
  const size_t block_bytes = (size_t)s.block_size * s.d * (s.dtype == MEFT_BF16 ? 2 : 4);
  const void* host[2] = {first_host, second_host};
  char* dev[2] = {first_dev, second_dev};
  hipEvent_t ev[2] = {first_ev, second_ev};
  for (int m = 0; m < 2; ++m) {
    for (int b = 0; b < s.n_blocks; ++b) {   // neighbouring blocks in use travel in one copy
      if (k.host_cnt[b] <= 0) continue;
      int n = 1;
      while (b + n < s.n_blocks && k.host_cnt[b + n] > 0) ++n;
      if (hipMemcpyAsync(dev[m] + (size_t)b * block_bytes, static_cast<const char*>(host[m]) + (size_t)b * block_bytes,
                         (size_t)n * block_bytes, hipMemcpyHostToDevice, k.side) != hipSuccess)
        return MEFT_ERR_DEVICE;
      b += n - 1;
    }
    if (hipEventRecord(ev[m], k.side) != hipSuccess) return MEFT_ERR_DEVICE;
  }
  return MEFT_OK;
}

// ---- batch-union variant: virtual blocks over the compacted rows --------------------------------
struct UnionGeom {
  int cap;        // capacity of S: min(N, T*top_k)
  int vbs, nvb;   // rows per virtual block, number of virtual blocks (nvb * vbs >= cap)
  meft_shape vs;  // the shape the grouped GEMMs see: nvb blocks of vbs rows, every token in every block
};

// false: the variant is not available for this shape (it runs on the bf16 matrix-core kernels only)
bool union_geom(const meft_shape& s, UnionGeom& g) {
  if (s.dtype != MEFT_BF16 || s.d % kTK != 0 || (s.flags & MEFT_FLAG_HOST_KV)) return false;
  const int64_t cap = (int64_t)s.T * s.top_k < (int64_t)s.N ? (int64_t)s.T * s.top_k : (int64_t)s.N;
  g.cap = (int)(cap < 1 ? 1 : cap);
  g.vbs = g.cap >= 1024 ? 1024 : round64(g.cap);
  g.nvb = (g.cap + g.vbs - 1) / g.vbs;
  if (g.nvb > 4096 || (int64_t)g.nvb * (s.T > 0 ? s.T : 1) > ((int64_t)1 << 30)) return false;
  g.vs = s;
  g.vs.n_blocks = g.nvb; g.vs.block_size = g.vbs; g.vs.N = g.nvb * g.vbs; g.vs.top_e = g.nvb; g.vs.top_k = 1;
  return true;
}

struct UnionWs : DispatchWs {
  int32_t *flag, *chunk_cnt, *rowtag;
  uint16_t *Kc, *Vc, *zrow, *Ap, *DS, *part;
  size_t bytes;
  UnionWs(const meft_shape& s, const UnionGeom& g, void* ws) {
    Carver c(ws);
    carve(g.vs, c);
    const size_t n_ent = (size_t)s.T * g.nvb, rows = (size_t)g.nvb * g.vbs;
    chunk_cnt = c.take<int32_t>((size_t)(s.N + kFlagChunk - 1) / kFlagChunk);
    flag = c.take<int32_t>(s.N);
    rowtag = c.take<int32_t>(rows + kTagPad);
    Kc = c.take<uint16_t>(rows * s.d);
    Vc = c.take<uint16_t>(rows * s.d);
    zrow = c.take<uint16_t>((size_t)g.vbs * (1 + 2 * n_ent));   // one piece: row of zeros, A', DS' (see BwdWs)
    Ap = zrow ? zrow + g.vbs : nullptr;
    DS = zrow ? Ap + n_ent * g.vbs : nullptr;
    part = c.take<uint16_t>(n_ent * s.d);
    bytes = c.off < 256 ? 256 : c.off;
  }
};

// every entry point asks for the same size, the one meft_workspace_bytes() reports
meft_status check_ws(const meft_shape& s, const void* ws, size_t have) {
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) || have < workspace_bytes(s)) return MEFT_ERR_WORKSPACE;
  return MEFT_OK;
}

thread_local hipError_t g_last_device_error = hipSuccess;   // what the last MEFT_ERR_DEVICE of this thread was
meft_status launch_status() {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return MEFT_OK;
  g_last_device_error = e;
  return MEFT_ERR_DEVICE;
}
// The runtime keeps the last error of the thread until it is read: an entry point reads it away before its first
// launch, so that MEFT_ERR_DEVICE reports this call's own launches and not a failure some other code left behind.
void clear_stale_error() { (void)hipGetLastError(); }

// threads per workgroup and 8-column groups per thread for the row kernels
void row_launch(int d, int& nthr, int& nv) {
  const int vecs = d / 8;
  nthr = vecs >= 256 ? 256 : ((vecs + 63) / 64) * 64;
  const int need = (vecs + nthr - 1) / nthr;
  nv = need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : 8;
}

// Rows of a tile of the fp32 score kernel: 64, which take fewer bytes per flop, once that gives every compute unit four tiles.
// Forward, us, 64 / 32 rows: one block of 16384, 1000 tokens, d 1024 366 / 404; 16 blocks of 256, d 4096, 2000 tokens 330 / 269.
int gemm_f32_rows(int64_t rows, int groups, int cols) {
  return (rows / 64 + groups / 2) * ((cols + kGemmF32BN - 1) / kGemmF32BN) >= 1024 ? 64 : 32;
}

// `rows` rows in `groups` groups, each of which may end with a partial tile
void launch_gemm_nt(const meft_shape& s, const GemmNTArgs& a, int64_t rows, int groups, const char* name, hipStream_t st) {
  if (s.dtype == MEFT_BF16) {
    dim3 grid((unsigned)(rows / kGemmBM + groups), (a.Ng + kGemmBN - 1) / kGemmBN);
    MEFT_LAUNCH(name, gemm_nt_bf16_kernel, grid, dim3(256), 0, st, a);
    return;
  }
  const int bm = gemm_f32_rows(rows, groups, a.Ng);
  const dim3 grid((unsigned)(((rows / bm + groups) * ((a.Ng + kGemmF32BN - 1) / kGemmF32BN) + 7) / 8 * 8));
  if (bm == 64) MEFT_LAUNCH(name, gemm_nt_f32_kernel<64>, grid, dim3(256), 0, st, a);
  else MEFT_LAUNCH(name, gemm_nt_f32_kernel<32>, grid, dim3(256), 0, st, a);
}

// A launch of n workgroups of 256 threads, n rounded up to a multiple of 8 (they go to the XCDs in turn), along x and then y
// (a launch takes fewer than 2^32 threads along x).
dim3 grid_xcd(int64_t n) {
  const int64_t all = (n + 7) / 8 * 8, x = all < (1 << 23) ? all : 1 << 23;
  return dim3((unsigned)x, (unsigned)((all + x - 1) / x));
}

template <typename T>
int row_slices(const meft_shape& s) { return (s.d + 64 * Vec16<T>::kElems - 1) / (64 * Vec16<T>::kElems); }   // of 1 KB

template <typename T, int kAcc>
void launch_pair_rows(const char* name, const meft_shape& s, const void* W, const int32_t* idx, const float* coef,
                      const float* gate, void* row, const SegFinish<T>& f, hipStream_t st) {
  const int64_t groups = row ? ((int64_t)s.T + 3) / 4 * row_slices<T>(s) : 0;
  if (groups + f.n_wg == 0) return;
  auto kernel = s.top_k == 1 ? pair_rows_kernel<T, kAcc, 1> : s.top_k == 2 ? pair_rows_kernel<T, kAcc, 2>
                : s.top_k <= 4 ? pair_rows_kernel<T, kAcc, 4> : pair_rows_kernel<T, kAcc, 8>;
  MEFT_LAUNCH(name, kernel, grid_xcd(f.n_wg + (groups + 7) / 8 * 8), dim3(256), 0, st, static_cast<const T*>(W), idx, coef,
              gate, row ? s.T : 0, s.d, s.top_k, s.N, static_cast<T*>(row), f);
}

// Whether dV, ds and dK of a chunk come out of one kernel (seg_rows_kernel) or of two, by the bytes of the rows of one operand that
// are touched at most; with more slices than waves to a chunk, only where most neurons have one pair.  Backward, us, two kernels /
// one.  Pairs grouped by one launch: 512 tokens x 16 of 16384 neurons (8192 rows) x 1 KB 26.7 / 22.1, x 2 KB 31.3 / 30.4, x 3 KB 36.4 /
// 38.9; 250 x 64 of 65536 x 1.4 KB 44.8 / 44.7, x 2 KB 49.1 / 51.0; 1000 x 16 of 4096 x 3 KB 39.8 / 42.4; 300 x 50 of 2000 x 3 KB
// 36.8 / 33.1; 1500 x 4 of 1500 x 4 KB 27.8 / 27.8, x 6 KB 35.1 / 38.2; 100 x 8 of 5000 x 6 KB 20.9 / 16.6, x 16 KB 28.2 / 24.9; 200 x
// 20 of 4096 x 6 KB 31.3 / 32.8.  By five: 1500 x 16 of 3000 x 1 KB 36.0 / 32.3, of 20000 40.0 / 41.7; 2500 x 25 of 1664 x 2 KB 63.9 /
// 62.2, x 3 KB 78.3 / 85.3; 8192 x 8 of 4000 x 2 KB 71.5 / 74.4; 65536 x 16 of 1000 x 1 KB 691 / 703.
bool seg_rows_fused(const meft_shape& s, int slices) {
  const int64_t P = (int64_t)s.T * s.top_k, bytes = (s.N < P ? s.N : P) * s.d * (s.dtype == MEFT_BF16 ? 2 : 4), MB = 1 << 20;
  if (!pair_one(s)) return slices <= 2 && bytes <= (slices == 1 ? 8 : 6) * MB && P <= 131072;
  if (slices <= 2) return bytes <= 24 * MB;
  if (slices <= 4) return bytes <= 12 * MB && P * slices <= 65536;
  return bytes <= 16 * MB && 4 * P <= s.N;
}

// The backward of the per-pair path.
template <typename T>
void launch_pair_bwd(const meft_shape& s, const BwdWs& w, const void* h, const void* K, const void* V, const int32_t* idx,
                     const float* act, const void* dOut, void* dh, void* dK, void* dV, int32_t* touched, int32_t* n_touched,
                     hipStream_t st) {
  const int P = s.T * s.top_k;
  const size_t n_pairs = (size_t)P;
  const dim3 pairs((unsigned)(((int64_t)P + 255) / 256));
  const int64_t n_seg = s.N < P ? s.N : P;
  // (a token's ids may repeat where they were clamped: more than kSegChunk pairs may have one neuron whatever T is)
  const int n_multi = P <= kSegChunk ? 0 : P / kSegChunk < 512 ? P / kSegChunk + 1 : 512;
  PairLists lists{};
  if (pair_one(s)) {
    lists = PairLists{w.first, P, touched, n_touched, w.multi, w.totals};
    static std::once_flag configured;   // 80 KB of pairs
    std::call_once(configured, [] {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&pair_one_kernel<kPairOneBatch>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                kPairOneP * (int)sizeof(uint32_t));
    });
    auto one = P <= 8 * kScanThreads ? pair_one_kernel<8> : pair_one_kernel<kPairOneBatch>;
    MEFT_LAUNCH("pair_one", one, dim3(kPairOneWgs), dim3(kScanThreads), (size_t)P * sizeof(uint32_t), st, idx, act, P, s.N, s.top_k,
                pair_one_shift(s), w.work, w.multi, w.first, w.pair_sorted, w.seg);
  } else {
    MEFT_LAUNCH("fill_i32", fill_i32_kernel, dim3((unsigned)(((size_t)s.N + 255) / 256)), dim3(256), 0, st, w.cnt_n, (size_t)s.N, 0);
    MEFT_LAUNCH("pair_count", pair_count_kernel, pairs, dim3(256), 0, st, idx, P, s.N, w.cnt_n, w.pair_sorted);
    const int n_chunks = (s.N + kScanChunk - 1) / kScanChunk;
    if (w.sums && s.N > kScanSelfMax)
      MEFT_LAUNCH("pair_sums", pair_sums_kernel, dim3(n_chunks), dim3(kScanThreads), 0, st, w.cnt_n, s.N, w.sums);
    MEFT_LAUNCH("pair_scan", pair_scan_kernel, dim3(n_chunks), dim3(kScanThreads), 0, st, w.cnt_n, s.N,
                s.N > kScanSelfMax ? w.sums : nullptr, w.seg_off, touched, n_touched, w.work, w.multi, w.totals);
    MEFT_LAUNCH("pair_fill", pair_fill_kernel, pairs, dim3(256), 0, st, idx, P, s.N, w.seg_off, w.pair_sorted, w.pair_list);
    MEFT_LAUNCH("seg_sort", seg_sort_kernel, dim3((unsigned)(n_multi + ((int64_t)P + 255) / 256)), dim3(256), 0, st, w.multi, w.totals,
                w.seg_off, w.pair_list, idx, act, P, s.N, s.top_k, n_multi, w.pair_sorted, w.seg);
  }
  const int slices = row_slices<T>(s), parts = slices < kDsParts ? slices : kDsParts;
  const int64_t n_work = lists.first ? P : n_seg + P / kSegChunk;   // work entries at most
  if (seg_rows_fused(s, slices)) {
    const int lg = slices >= 3 ? 2 : slices - 1;
    const int64_t wgs = ((n_work << lg) + 3) / 4;
    const int grid = (int)(wgs < kSegRowsWgs ? wgs : kSegRowsWgs) + (lists.first ? 1 : 0);
    MEFT_LAUNCH("seg_rows", seg_rows_kernel<T>, dim3(grid), dim3(256), 0, st, w.work, w.totals, P, w.seg, w.pair_sorted,
                static_cast<const T*>(V), static_cast<const T*>(dOut), static_cast<const T*>(h), s.d, slices, lg, static_cast<T*>(dV),
                static_cast<T*>(dK), w.seg_part, dh ? w.ds : nullptr, lists);
  } else {
    // work entries per chunk, if the pairs fall on the neurons alike
    const double chunks = s.N * -std::expm1(-(double)P / s.N);
    const int entries = lists.first ? (int)(P / chunks + 0.5) : 1;
    auto launch = [&](auto dv, auto dk) {
      const int64_t groups = (n_work + 3) / 4;   // four entries per workgroup
      auto grid = [&](int n, int more) {   // (no workgroup beyond what runs at once: it would have to wait for another)
        return grid_xcd((groups * n < kSegWorkgroups - more ? groups * n : kSegWorkgroups - more) + more);
      };
      MEFT_LAUNCH("seg_dv", dv, grid(parts, lists.first ? 8 : 0), dim3(256), 0, st, w.work, w.totals, w.seg, static_cast<const T*>(V),
                  static_cast<const T*>(dOut), s.d, slices, n_pairs, static_cast<T*>(dV), w.seg_part, w.ds_part, entries, lists);
      MEFT_LAUNCH("seg_dk", dk, grid(slices, 0), dim3(256), 0, st, w.work, w.totals, w.seg, w.pair_sorted, w.ds_part,
                  static_cast<const T*>(h), s.d, slices, n_pairs, static_cast<T*>(dK), w.seg_part, dh ? w.ds : nullptr, entries);
    };
    if (lists.first) launch(seg_dv_kernel<T, true>, seg_dk_kernel<T, true>);
    else launch(seg_dv_kernel<T, false>, seg_dk_kernel<T, false>);
  }
  const int n_fin = n_multi == 0 ? 0 : P / kSegChunk < 4096 ? (P / kSegChunk + 8) / 8 * 8 : 4096;
  const SegFinish<T> f{n_fin, w.multi, w.totals, w.seg_part, static_cast<T*>(dK), static_cast<T*>(dV)};
  launch_pair_rows<T, 4>("pair_dh", s, K, idx, w.ds, act, dh, f, st);
}

constexpr int kPersistentWgs = 256;   // compute units of an MI355X; a multiple of the 8 XCDs

// Bytes readable from an operand's lowest address; buffer loads (32-bit offsets) where both fit.  Setting
// MEFT_GLOBAL_LOADS=1 in the environment selects the global-load kernels (those for operands of 4 GB and more)
// at any size, so that tests reach them with small inputs.
// (the environment is read once, when the library is loaded; meft_debug_global_loads overrides it.  Read and written under
// g_api_mutex only: the launches of one call depend on each other's choice, so it may not change between them.)
bool g_force_global_loads = [] {
  const char* env = getenv("MEFT_GLOBAL_LOADS");
  return env && env[0] == '1';
}();

constexpr uint64_t kBufLimit = 0xFFFF0000ull;   // bytes that a buffer resource's 32-bit offsets reach

template <class P>
void set_gemm_extents(P& p, uint64_t a_bytes, uint64_t b_bytes) {
  p.buf = !g_force_global_loads && a_bytes < kBufLimit && b_bytes < kBufLimit;
  p.a_bytes = p.buf ? (uint32_t)a_bytes : 0u;
  p.b_bytes = p.buf ? (uint32_t)b_bytes : 0u;
}

template <class P>
void launch_gemm_mfma(const char* name, const P& prob, int grid, hipStream_t st) {
  static std::once_flag configured;  // raise the dynamic LDS limit of both instantiations once
  std::call_once(configured, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_mfma_kernel<P, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, gemm_lds_bytes<P>());
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_mfma_kernel<P, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, gemm_lds_bytes<P>());
  });
  // persistent workgroups: one per compute unit (the LDS footprint allows no more), each walking the tile ids
  // wg, wg + 256, ... below `grid`
  const int launch = grid < kPersistentWgs ? grid : kPersistentWgs;
  if (prob.buf) {
    MEFT_LAUNCH(name, (gemm_mfma_kernel<P, true>), dim3(launch), dim3(gemm_threads<P>()), gemm_lds_bytes<P>(), st, prob, grid);
  } else {
    MEFT_LAUNCH(name, (gemm_mfma_kernel<P, false>), dim3(launch), dim3(gemm_threads<P>()), gemm_lds_bytes<P>(), st, prob, grid);
  }
}

template <class P>
void launch_gemm_wide(const char* name, const P& prob, int grid, hipStream_t st) {
  static std::once_flag configured;
  std::call_once(configured, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_wide_kernel<P>), hipFuncAttributeMaxDynamicSharedMemorySize,
                              kWideLds);
  });
  const int launch = grid < kPersistentWgs ? grid : kPersistentWgs;
  MEFT_LAUNCH(name, gemm_wide_kernel<P>, dim3(launch), dim3(256), kWideLds, st, prob, grid);
}

// for policies that exist with buffer loads only
template <class P>
void launch_gemm_mfma_buf(const char* name, const P& prob, int grid, hipStream_t st) {
  static std::once_flag configured;
  std::call_once(configured, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_mfma_kernel<P, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, gemm_lds_bytes<P>());
  });
  const int launch = grid < kPersistentWgs ? grid : kPersistentWgs;
  MEFT_LAUNCH(name, (gemm_mfma_kernel<P, true>), dim3(launch), dim3(gemm_threads<P>()), gemm_lds_bytes<P>(), st, prob, grid);
}

template <class P>
void launch_gemm_tile(const char* name, const P& prob, int64_t tiles, hipStream_t st) {
  static std::once_flag configured;
  std::call_once(configured, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tile_kernel<P>), hipFuncAttributeMaxDynamicSharedMemorySize,
                              gemm_tile_lds<P>());
  });
  const int bound = (int)(tiles < (int64_t)INT32_MAX ? tiles : (int64_t)INT32_MAX);
  const int launch = bound < 2 * kPersistentWgs ? bound : 2 * kPersistentWgs;   // two workgroups per compute unit
  MEFT_LAUNCH(name, gemm_tile_kernel<P>, dim3(launch), dim3(256), gemm_tile_lds<P>(), st, prob, bound);
}

// Whether a token-major contraction over `cols` output columns runs on small tiles.  What a compute unit's time goes by
// is the kilobytes per k tile it takes into LDS: 48 for each of its 128 x 256 tiles, 24 for each 64 x 128 tile; large
// tiles come in whole rounds of one per compute unit, small ones two at a time.  Groups are taken to be alike, each
// with half a tile to spare.
bool small_tiles(const meft_shape& s, int cols) {
  const int64_t n_ent = (int64_t)s.T * s.top_e, groups = s.n_blocks < n_ent ? s.n_blocks : n_ent;
  const int64_t large = (n_ent / kTMTok + (groups + 1) / 2) * ((cols + kTN - 1) / kTN);
  const int64_t small = (n_ent / 64 + (groups + 1) / 2) * ((cols + 127) / 128);
  const int64_t cost_large = (large + kPersistentWgs - 1) / kPersistentWgs * kPersistentWgs * 48;
  return (small < kPersistentWgs ? kPersistentWgs : small) * 24 < cost_large;
}

// Whether a token-major contraction of nk k tiles over `cols` output columns runs on tiles of 256 rows (gemm_wide_kernel) rather
// than of 128 (gemm_mfma_kernel), by what one compute unit takes for a k tile and for a tile, in hundredths of a whole tile's k
// tile (1.7-2.4 us): 256 rows 100 and 150, the short tile at the end of a group 74 and 120 (its columns' lines are nobody else's by then),
// 128 rows 56 and 50.  Whole tiles come first and short ones fill up their last round (WideFinder).  Groups are taken
// to lie within 30 % of their average, as the router's do, or to be alike where every token is in every block.  us on 128 / 256
// rows: 64 blocks of 1024 x 4096, activation gradient at 512 rows a group 316 / 294, at 256 rows 203 / 222 (half of the groups a few
// rows too long); 64 blocks of 512 x 1024, scores at 96 to 192 rows 22 / 29 (two columns of tiles: 128 whole tiles leave half of the
// compute units idle); one block of 9984 x 3264, 138 tokens 40 / 64, of 34560 x 2560 83 / 58.
// Between one and four groups per XCD the XCD with one more counts: union of 879 tokens over 10 x 1024, 1344 columns 48 / 59; 18 blocks
// of 816, 444 rows a group, 1472 columns 38 / 41.
// Over 330 contractions of random layers and unions this takes 3 % longer than the better form of each would, 128 rows always 7 %.
//
// Groups of fewer than 224 rows, but enough tiles for every compute unit, are bound by the block's rows out of HBM, which fewer
// and deeper requests bring faster: 256 columns' rows of 32 k tiles and more (64 blocks of 1024 x 4096, scores at 128 rows 154 / 136),
// or four rounds of tiles, whose last one is a small part (256 unbalanced blocks of 1024 x 4096, values 550 / 440).  With fewer
// tiles of fewer k tiles the rounds decide here too (28 blocks of 864 x 2688 at 104 rows, values 38 / 44).
bool wide_tiles(const meft_shape& s, int cols, int nk) {
  const int64_t n_ent = (int64_t)s.T * s.top_e, groups = s.n_blocks < n_ent ? s.n_blocks : n_ent, rows = n_ent / groups;
  if (rows < 96) return false;
  const int64_t tn = (cols + kTN - 1) / kTN, per = groups * tn;
  if (rows < 224 && (per >= 4 * kPersistentWgs || (per >= kPersistentWgs && nk >= 32))) return nk >= 8;
  struct Tiles {
    int64_t whole, shorts, of128;   // of one XCD
    void add(int64_t r, int64_t n) {
      const int64_t f = (r + 127) / 256;
      whole += f * n;
      shorts += r > f * kWideM ? n : 0;
      of128 += (r + 127) / 128 * n;
    }
  };
  int64_t cost_wide = 0, cost_128 = 0;
  auto count = [&](const Tiles& t) {   // an XCD has 32 compute units
    const int64_t cu = kPersistentWgs / kXcd, rounds = (t.whole + cu - 1) / cu, room = rounds * cu - t.whole;
    const int64_t late = t.shorts > room ? t.shorts - room : 0;
    const int64_t wide = rounds * (nk * 100 + 150) + (late + cu - 1) / cu * (nk * 74 + 120);
    const int64_t small = (t.of128 + cu - 1) / cu * (nk * 56 + 50);
    cost_wide = wide > cost_wide ? wide : cost_wide;
    cost_128 = small > cost_128 ? small : cost_128;
  };
  Tiles t{};
  if (s.top_e == s.n_blocks) {
    const int64_t by = groups > kXcd ? 1 : kXcd;   // whole groups, or tiles of each
    t.add(rows, groups > kXcd ? (groups + kXcd - 1) / kXcd * tn : per);
    count({(t.whole + by - 1) / by, (t.shorts + by - 1) / by, (t.of128 + by - 1) / by});
  } else if (groups > kXcd && groups < 4 * kXcd && groups % kXcd != 0) {   // dealt longest first (build_sched_body)
    int64_t load[kXcd] = {};
    Tiles x[kXcd] = {};
    for (int64_t i = 0; i < groups; ++i) {
      const int64_t r = rows * (130 - 60 * i / (groups - 1)) / 100;
      int k = 0;
      for (int j = 1; j < kXcd; ++j) k = load[j] < load[k] ? j : k;
      load[k] += (r + 63) / 64 + 2;
      x[k].add(r, tn);
    }
    for (const Tiles& one : x) count(one);
  } else {
    const int64_t by = 7 * kXcd;
    for (int z = 7; z <= 13; ++z) t.add(rows * z / 10, per);
    count({(t.whole + by - 1) / by, (t.shorts + by - 1) / by, (t.of128 + by - 1) / by});
  }
  return cost_wide * 101 <= cost_128 * 100;   // (a tie: 28 blocks of 896 at 268 rows, 4992 columns 102 / 115)
}

// Launches a token-major policy that exists with buffer loads only, with the tiles that suit the problem.
template <class Large, class F>
void launch_tok_buf(const char* name, const meft_shape& s, int cols, int nk, F&& fill, hipStream_t st) {
  if (wide_tiles(s, cols, nk)) {
    WideTok<Large> p{};
    fill(p);
    launch_gemm_wide(name, p, tile_bound(s, (cols + kTN - 1) / kTN), st);
  } else {
    Large p{};
    fill(p);
    launch_gemm_mfma_buf(name, p, tile_bound(s, (cols + kTN - 1) / kTN), st);
  }
}

// Fills in a token-major policy's fields and launches it with the tiles that suit the problem.
template <class Large, class Small, class F>
void launch_tok(const char* name, const meft_shape& s, int cols, int nk, uint64_t a_bytes, uint64_t b_bytes, uint64_t o_bytes, F&& fill,
                hipStream_t st) {
  Small q{};
  set_gemm_extents(q, a_bytes, b_bytes);
  if (q.buf && o_bytes < kBufLimit && (s.block_size & 1) == 0 && small_tiles(s, cols)) {
    q.o_bytes = (uint32_t)o_bytes;
    fill(q);
    const int64_t m_tiles = (int64_t)s.T * s.top_e / Small::kTM + s.n_blocks;
    launch_gemm_tile(name, q, kXcd * m_tiles * ((cols + Small::kTNt - 1) / Small::kTNt), st);
    return;
  }
  if (q.buf && wide_tiles(s, cols, nk)) {
    WideTok<Large> p{};
    set_gemm_extents(p, a_bytes, b_bytes);
    fill(p);
    launch_gemm_wide(name, p, tile_bound(s, (cols + kTN - 1) / kTN), st);
    return;
  }
  Large p{};
  set_gemm_extents(p, a_bytes, b_bytes);
  fill(p);
  launch_gemm_mfma(name, p, tile_bound(s, (cols + kTN - 1) / kTN), st);
}
template <int MODE> using TokKCLarge = ProbTokKC<MODE>;
template <int MODE> using TokKCSmall = TileTokKC<MODE, 64, 128>;
using TokNCSmall = TileTokNC<64, 128>;

// (token, block) dispatch: groups, slot maps, XCD tile schedule; with block_idx the per-token block lists are sorted
// first (otherwise w.sblk holds them).  `clear`: words set to zero on the way.
void launch_dispatch(const meft_shape& s, const DispatchWs& w, const int32_t* block_idx, int BM, bool dense, bool want_sched,
                     int32_t* clear, size_t clear_words, hipStream_t st) {
  const int n_ent = s.T * s.top_e;
  const int small = dense ? small_rows_of(s) : 0;
  const DispatchTables tab{w.cnt, w.group_off, w.tile_off, BM, sched_cap(s), want_sched ? w.sched_pairs : nullptr,
                           w.sched_tiles, w.sched_len, small, small ? w.small_ent : nullptr, w.small_grp, w.small_cnt};
  int32_t* tok = dense || want_sched ? w.tok_of_slot : nullptr;
  if (const int form = dispatch_one_form(s.T, s.top_e, s.n_blocks)) {
    const int n_iter = (s.T + 1023) / 1024;
    const size_t lds = (size_t)n_iter * (1024 + 16) * sizeof(int);   // up to 65 KB
    static std::once_flag configured_one;
    std::call_once(configured_one, [] {
      const int most = kDispOneTokens / 1024 * (1024 + 16) * (int)sizeof(int);
      const void* forms[] = {reinterpret_cast<const void*>(&dispatch_one_kernel<true, true>), reinterpret_cast<const void*>(&dispatch_one_kernel<false, true>),
                             reinterpret_cast<const void*>(&dispatch_one_kernel<true, false>), reinterpret_cast<const void*>(&dispatch_one_kernel<false, false>)};
      for (const void* f : forms) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    });
    const int room = form == 1 ? 64 / s.n_blocks : 1, parts = room < n_iter ? room : n_iter;   // >= 1
    const dim3 grid(s.n_blocks * parts + 1);
    auto go = [&](auto kernel, const int32_t* in, int32_t* sorted) {
      MEFT_LAUNCH("dispatch", kernel, grid, dim3(1024), lds, st, in, s.T, s.top_e, s.n_blocks, tab, sorted, w.perm, tok, w.slot_of_ent,
                  kSlotPad, clear, clear_words);
    };
    if (block_idx && form == 1) go(dispatch_one_kernel<true, true>, block_idx, w.sblk);
    else if (block_idx) go(dispatch_one_kernel<true, false>, block_idx, w.sblk);
    else if (form == 1) go(dispatch_one_kernel<false, true>, w.sblk, nullptr);
    else go(dispatch_one_kernel<false, false>, w.sblk, nullptr);
    return;
  }
  if (fast_dispatch(s)) {
    const int epc = disp_chunk_entries(s), n_chunks = disp_chunks(s);
    const size_t lds = (size_t)16 * s.n_blocks * sizeof(int);
    static std::once_flag configured;   // 64 KB of counters at 1024 blocks, and the static arrays
    std::call_once(configured, [] {
      const int most = 16 * kDispMaxBlocks * (int)sizeof(int);
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&dispatch_count_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&dispatch_count_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&dispatch_place_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
    });
    if (block_idx)
      MEFT_LAUNCH("dispatch_count", dispatch_count_kernel<true>, dim3(n_chunks), dim3(1024), lds, st, block_idx, n_ent,
                  s.top_e, epc, s.n_blocks, w.sblk, w.chunk_hist, clear, clear_words);
    else
      MEFT_LAUNCH("dispatch_count", dispatch_count_kernel<false>, dim3(n_chunks), dim3(1024), lds, st, w.sblk, n_ent,
                  s.top_e, epc, s.n_blocks, nullptr, w.chunk_hist, clear, clear_words);
    int lg = 0;
    while ((1 << lg) < s.n_blocks) ++lg;
    if (s.n_blocks <= kDispScanBlocks && (int64_t)n_chunks * s.n_blocks <= kDispScanMax) {
      MEFT_LAUNCH("dispatch_place", dispatch_place_kernel<true>, dim3(n_chunks + 1), dim3(1024), lds, st, w.sblk, n_ent,
                  s.top_e, epc, s.n_blocks, lg, n_chunks, w.chunk_hist, tab, w.perm, tok, w.slot_of_ent, kSlotPad);
    } else {
      MEFT_LAUNCH("dispatch_scan", dispatch_scan_kernel, dim3(1), dim3(1024), 0, st, w.chunk_hist, n_chunks, s.n_blocks, tab);
      MEFT_LAUNCH("dispatch_place", dispatch_place_kernel<false>, dim3(n_chunks), dim3(1024), lds, st, w.sblk, n_ent,
                  s.top_e, epc, s.n_blocks, lg, n_chunks, w.chunk_hist, tab, w.perm, tok, w.slot_of_ent, kSlotPad);
    }
    return;
  }
  if (clear_words)
    MEFT_LAUNCH("fill_i32", fill_i32_kernel, dim3((unsigned)((clear_words + 255) / 256)), dim3(256), 0, st, clear,
                clear_words, 0);
  if (block_idx)
    MEFT_LAUNCH("sort_blocks", sort_blocks_kernel, dim3((s.T + 255) / 256), dim3(256), 0, st, block_idx, s.T, s.top_e,
                s.n_blocks, w.sblk);
  MEFT_LAUNCH("count_blocks", count_blocks_kernel, dim3(s.n_blocks), dim3(1024), 0, st, w.sblk, n_ent, w.cnt);
  MEFT_LAUNCH("fill_groups", fill_groups_kernel, dim3(s.n_blocks), dim3(1024), 0, st, w.sblk, n_ent, w.cnt,
              s.n_blocks, BM, w.group_off, w.tile_off, w.perm);
  if (dense || want_sched) {
    MEFT_LAUNCH("slot_maps", slot_maps_kernel, dim3((n_ent + kSlotPad + 255) / 256), dim3(256), 0, st, w.perm, w.group_off,
                s.n_blocks, s.top_e, w.sblk, small, w.tok_of_slot, w.slot_of_ent);
  }
  if (want_sched) {
    MEFT_LAUNCH("build_sched", build_sched_kernel, dim3(1), dim3(1024), 0, st, w.group_off, s.n_blocks,
                sched_cap(s), w.sched_pairs, w.sched_tiles, w.sched_len, small);
  }
  if (small) {
    MEFT_LAUNCH("small_lists", small_lists_kernel, dim3(1), dim3(1024), 0, st, w.group_off, s.n_blocks, small,
                w.small_ent, w.small_grp, w.small_cnt);
  }
}

// Launch widths of the work on the lists of small groups: enough workgroups for the lists of a skewed batch to be taken
// in one pass, few enough that a launch on a batch without small groups costs next to nothing.
constexpr int kSmallEntGrid = 256, kSmallGrpGrid = 128;

// few tokens: a workgroup per (token, 512 columns), so that small groups, whose pairs are a chain of row reads, get more waves
bool rows_split(const meft_shape& s) { return s.T * ((s.d + kSmallCols - 1) / kSmallCols) <= 16 * kPersistentWgs; }

// Whether the dV / dK rows of the small groups share the launch of the dh rows.  That launch then has four waves per
// workgroup, of which a token's short row uses as many as it has 512 columns; an idle one costs 0.2 to 0.3 ns, the launch that
// is saved 4 to 6 us.  One launch / two, us: 37 / 28 at 32768 tokens x 512, 166 / 97 at 100000 x 256, 393 / 166 at 300000 x
// 64; 20.8 for one at 8192 x 1024, where the rows alone take 18.
bool dvdk_beside_rows(const meft_shape& s) {
  int nthr, nv;
  row_launch(s.d, nthr, nv);
  return rows_split(s) || (int64_t)s.T * (4 - nthr / 64) <= 16384;
}

// The tokens' rows of out (W = V, coef = act) or dh (W = K, coef = ds) from the entries' partial rows and the pairs of
// the small groups; `dv`: the dV / dK work of the small groups, or none.
// Whether token_rows reads its partial rows, each of them once, past L2, out of the way of the next contraction's operands, by the
// bytes of all partial rows.  us per pass through / past L2.
//   From 60 MB on past it: 7757 tokens, 8 of 41 blocks of 144 x 1856 (230 MB) 936 / 889; 1289 tokens, 7 of 67 blocks of 416 x 5056
// (91 MB) 711 / 671; 4079 tokens, 8 of 29 blocks of 224 x 2048 (134 MB) 406 / 388; unions within 1 %.  But where a contraction of
// up to three k tiles has just written 60 to 190 MB, the reads that go through L2 are the faster ones by more than the contractions
// gain: 2003 tokens, 8 of 64 blocks of 96 x 4096 (131 MB) 328 / 339; 4666 tokens, 6 of 230 blocks of 96 x 1664 (93 MB) 350 / 364
// (more of the same: 4000 x 4096, 262 MB 600 / 594).
//   Below, rows of up to 4 KB: 5823 tokens, 4 of 19 blocks of 912 x 704 (33 MB) 474 / 463; 777 tokens, 4 of 64 blocks of 1024 x 4096
// (25 MB) 281 / 283.
bool rows_past_l2(const meft_shape& s) {
  const int64_t bytes = (int64_t)s.T * s.top_e * s.d * 2;
  if (bytes < (60ll << 20)) return s.d <= 2048;
  return bytes > (190ll << 20) || s.block_size > 3 * kTK;
}

void launch_token_rows(const char* name, const meft_shape& s, const uint16_t* part, const DispatchWs& w, const void* W,
                       const int32_t* idx, const float* coef, void* out, const SmallDvdk& dv, hipStream_t st) {
  const TokenRows a{part, w.sblk, w.slot_of_ent, idx, coef, static_cast<const bf16_t*>(W), s.d, s.top_e, s.top_k, s.N,
                    s.block_size, static_cast<bf16_t*>(out), rows_past_l2(s)};
  const size_t lds = small_rows_of(s) ? (size_t)(s.top_k < kTokenRowsPairs ? s.top_k : kTokenRowsPairs) * sizeof(int2) : 0;
  const int chunks = (s.d + kSmallCols - 1) / kSmallCols;
  if (rows_split(s)) {
    if (dv.n_wg) MEFT_LAUNCH(name, (token_rows_kernel<1, true, true>), dim3(dv.n_wg + s.T * chunks), dim3(256), lds, st, a, dv);
    else MEFT_LAUNCH(name, (token_rows_kernel<1, true, false>), dim3(s.T * chunks), dim3(256), lds, st, a, dv);
    return;
  }
  int nthr, nv;
  row_launch(s.d, nthr, nv);
  if (dv.n_wg) { nthr = 256; nv = s.d <= 2048 ? 1 : s.d <= 4096 ? 2 : s.d <= 8192 ? 4 : 8; }   // the dV / dK work takes four waves
#define RP(NV) MEFT_LAUNCH(name, (token_rows_kernel<NV, false>), dim3(dv.n_wg + s.T), dim3(nthr), lds, st, a, dv)
  switch (nv) { case 1: RP(1); break; case 2: RP(2); break; case 4: RP(4); break; default: RP(8); }
#undef RP
}

// touched list, and in the same launch (small: w holds lists of small groups) the activation gradients of their pairs
void launch_bwd_head(const meft_shape& s, const int32_t* flag, int32_t* chunk_cnt, int32_t* touched, int32_t* n_touched,
                     const DenseWs* w, const void* V, const void* dOut, const int32_t* idx, const float* act,
                     hipStream_t st) {
  const int n_chunks = (s.N + kFlagChunk - 1) / kFlagChunk;
  const bool counts = s.N > kFlagCountMax;
  if (counts)
    MEFT_LAUNCH("count_flags", count_flags_kernel, dim3(n_chunks), dim3(256), 0, st, flag, s.N, chunk_cnt);
  const int small = w ? small_rows_of(s) : 0;
  const int nx = s.n_blocks * small < kSmallEntGrid ? s.n_blocks * small : kSmallEntGrid;
  MEFT_LAUNCH("bwd_head", bwd_head_kernel, dim3(n_chunks + nx * kSmallPairSplit), dim3(256), small ? (size_t)s.top_k * 4 : 0, st,
              flag, s.N, counts ? chunk_cnt : nullptr, n_chunks, touched, n_touched, nx, static_cast<const bf16_t*>(V),
              static_cast<const bf16_t*>(dOut), idx, act, w ? w->small_ent : nullptr, w ? w->small_cnt : nullptr,
              w ? w->tok_of_slot : nullptr, s.d, s.top_k, s.block_size, w ? w->ds32 : nullptr);
}

// Whether the dV / dK contractions of s's groups run on tiles of 256 rows (gemm_wide_kernel) rather than of 128 (gemm_mfma_kernel):
// where that computes no more padded rows of the block, and by what an XCD's 32 compute units take for a k tile (64 tokens) and for a
// tile, as in wide_tiles: 256 rows 100 and 150, 128 rows 56 and 54, or 72 where most compute units have a tile of 256 rows and 40
// tokens or more for it (then both wait for the stores of the rows).  Every group has the same tiles.  us per launch on 128 / 256 rows:
// 64 blocks of 1024 x 4096, 512 tokens each 355 / 320; 256 unbalanced ones, 128 each on average 314 / 303; 64 blocks of 256 x 1024, 128
// each 15.3 / 14.6; 72 blocks of 144 x 640, 21 each 7.8 / 9.4 (a tile's end takes longer than its k tile); 15 blocks of 1024 x 1280, 168
// each 19 / 22; one block of 960 x 1216, 1328 tokens 19 / 33 (20 tiles of 256 rows).  Over 111 contractions of random layers and unions
// with smaller gradients this takes 1 % longer than the better form of each would, 256 rows always 34 %.
//   Gradients of 48 MB and more each go to 256 rows, whose stores pass the caches by: those of the 128 rows push K and V out of the
// memory-side cache (256 MB), from where the other contractions read them.  us per pass on 128 / 256 rows: 388 tokens, 4 of 120 blocks
// of 208 x 4288 (214 MB) 418 / 381, of which dV and dK 104 / 111; 3579 tokens, 3 of 220 blocks of 224 x 3584 (353 MB) 710 / 645; 448
// tokens, 6 of 236 blocks of 192 x 640 (58 MB) 171 / 166; 808 tokens, 2 of 40 blocks of 720 x 768 (44 MB) 128 / 127.  Groups of up to
// four tokens are summed pair by pair but for a few, and nothing is found sooner by fewer waves (70 blocks, one token each 3.8 / 2.2
// per launch).
bool wide_neu(const meft_shape& s) {
  const int64_t n_ent = (int64_t)s.T * s.top_e, groups = s.n_blocks < n_ent ? s.n_blocks : n_ent, rows = n_ent / groups;
  const int64_t tm256 = (s.block_size + 255) / 256, tm128 = (s.block_size + 127) / 128;
  if (2 * tm256 != tm128) return false;
  if (rows <= 4 || (int64_t)s.N * s.d * 2 >= (48ll << 20)) return true;
  const int64_t nk = (rows + kTK - 1) / kTK, tn = (s.d + kTN - 1) / kTN, cu = kPersistentWgs / kXcd;
  auto rounds = [&](int64_t tm) {   // lists of fewer groups than XCDs: each XCD takes a part of every group's tiles
    const int64_t tiles = groups < kXcd ? (groups * tm * tn + kXcd - 1) / kXcd : (groups + kXcd - 1) / kXcd * tm * tn;
    return (tiles + cu - 1) / cu;
  };
  const bool stores = 4 * groups * tm256 * tn >= 3 * kPersistentWgs && rows >= 40;
  return rounds(tm256) * (nk * 100 + 150) <= rounds(tm128) * (nk * 56 + (stores ? 72 : 54));
}

// One weight-gradient contraction (dV: A = A', X = dOut; dK: A = DS', X = h) over the groups of a tile schedule
struct NeuArgs {
  const uint16_t* A; int zrow; const uint16_t* X; uint16_t* G;
  const int32_t *tok_of_slot, *flag;
  TokenSched sched;
  int big_only, n_groups, bs, bsp, d;
  bool wide;
  uint64_t a_bytes, x_bytes;   // bytes readable from the lowest address of either operand
};

template <template <int> class P = ProbNeuTN>
void launch_neu(const char* name, const NeuArgs& a, hipStream_t st) {
  auto launch = [&](auto pn) {
    constexpr int TM = decltype(pn)::kTM;
    pn.A = a.A; pn.zrow = a.zrow; pn.X = a.X; pn.G = a.G;
    pn.tok_of_slot = a.tok_of_slot; pn.flag = a.flag;
    pn.sched = a.sched; pn.big_only = a.big_only; pn.bs = a.bs; pn.bsp = a.bsp; pn.d = a.d;
    set_gemm_extents(pn, a.a_bytes, a.x_bytes);
    if (TM == 256 && !pn.buf) return false;
    // every listed group has the same tiles; in the worst case one XCD holds all groups
    const int64_t tiles = (int64_t)kXcd * a.n_groups * ((a.bs + TM - 1) / TM) * ((a.d + kTN - 1) / kTN);
    const int bound = (int)(tiles < (int64_t)INT32_MAX ? tiles : (int64_t)INT32_MAX);
    if constexpr (TM == 256) launch_gemm_wide(name, pn, bound, st);
    else launch_gemm_mfma(name, pn, bound, st);
    return true;
  };
  if (a.wide && launch(P<256>{})) return;
  launch(P<128>{});
}

}  // namespace
}  // namespace meft

using namespace meft;

// the few-token forward: scores, then selection and value sum
template <typename T>
static meft_status launch_few(const meft_shape& s, const void* h, const void* K, const void* V, const int32_t* block_idx, void* out,
                       int32_t* idx, float* act, float* sc, hipStream_t st, hipEvent_t wait_v) {
  const int n_ent = s.T * s.top_e, C = s.top_e * s.block_size;
  const int by_block = s.n_blocks <= n_ent ? 1 : 0, rows = by_block ? s.n_blocks : n_ent;
  const T *hh = static_cast<const T*>(h), *kk = static_cast<const T*>(K), *vv = static_cast<const T*>(V);
  // two 16-neuron tiles per workgroup (they share the loads of h) where that leaves a workgroup for every compute unit
#define FS(NA) MEFT_LAUNCH("few_score", (few_score_kernel<T, NA>), dim3((s.block_size + 16 * (NA) - 1) / (16 * (NA)), rows), dim3(64 * kFewWaves), 0, st, hh, kk, block_idx, n_ent, s.top_e, s.n_blocks, s.block_size, s.d, by_block, sc)
  if (rows * ((s.block_size + 31) / 32) >= kPersistentWgs) FS(2);
  else FS(1);
#undef FS
  if (wait_v && hipStreamWaitEvent(st, wait_v, 0) != hipSuccess) return MEFT_ERR_DEVICE;
  T* o = static_cast<T*>(out);
  // 512 columns per workgroup, 128 where that leaves compute units without one
  const bool wide = (int64_t)s.T * ((s.d + 511) / 512) >= kPersistentWgs;
  const int cols = wide ? 512 : 128;
  const dim3 grid(out ? (s.d + cols - 1) / cols : 1, s.T);
#define FO3(KPT, FULL, CL) MEFT_LAUNCH("few_out", (few_out_kernel<T, KPT, FULL, CL>), grid, dim3(256), 0, st, sc, block_idx, vv, C, s.block_size, s.top_e, s.top_k, s.n_blocks, s.d, idx, act, o)
#define FO2(KPT, FULL) do { if (wide) FO3(KPT, FULL, 64); else FO3(KPT, FULL, 16); } while (0)
#define FO(KPT) do { if (C == 256 * (KPT)) FO2(KPT, true); else FO2(KPT, false); } while (0)
  if (C <= 256 * 4) FO(4);
  else if (C <= 256 * 8) FO(8);
  else if (C <= 256 * 16) FO(16);
  else if (C <= 256 * 32) FO(32);
  else FO(48);
#undef FO
#undef FO2
#undef FO3
  return launch_status();
}

// Partial router scores without LDS tiles; returns the number of slices of the hidden dimension (at most
// kRouterSplitMax).
template <typename T>
static int launch_route_part(const meft_shape& s, const void* h, const void* Wg, float* p, hipStream_t st) {
  const T *hh = static_cast<const T*>(h), *ww = static_cast<const T*>(Wg);
  const int n_part = route_slices(s);
#define RP(NA, TT) MEFT_LAUNCH("route_part", (route_part_kernel<T, NA, TT>), dim3((unsigned)((s.n_blocks + 16 * (NA) - 1) / (16 * (NA))) * ((s.T + 16u * (TT) - 1) / (16 * (TT))), 1, n_part), dim3(64 * kRouteWaves), 0, st, hh, ww, s.T, s.d, s.n_blocks, p)
  // one 16-block tile per workgroup for the few tokens that would leave the chip idle, else four (they share the
  // loads of h), and two token tiles (they share the loads of the router) once that still fills it
  const int64_t wg = (int64_t)((s.T + 15) / 16) * ((s.n_blocks + 63) / 64) * n_part;
  if (wg < kPersistentWgs / 4) RP(1, 1);
  else if (wg < 2 * kPersistentWgs) RP(4, 1);
  else RP(4, 2);
#undef RP
  return n_part;
}

// Router scores (as up to kRouterSplitMax partial sums over slices of the hidden dimension, in `p`) and the top-e
// selection over their sum.
static meft_status route_impl(const meft_shape& s, const void* h, const void* Wg, const float* bias,
                              int32_t* block_idx, float* block_score, float* p, hipStream_t st) {
  int n_part = 1;
  if (!route_on_tiles(s)) {
    n_part = s.dtype == MEFT_BF16 ? launch_route_part<bf16_t>(s, h, Wg, p, st) : launch_route_part<float>(s, h, Wg, p, st);
  } else if (s.dtype == MEFT_BF16 && s.d % kTK == 0) {
    const int kt = s.d / kTK;
    n_part = kt % 4 == 0 ? 4 : (kt % 2 == 0 ? 2 : 1);
    ProbRouter pr{static_cast<const uint16_t*>(h), static_cast<const uint16_t*>(Wg), p, s.T, s.d, s.n_blocks, n_part};
    set_gemm_extents(pr, (uint64_t)s.T * s.d * 2, (uint64_t)s.n_blocks * s.d * 2);
    launch_gemm_mfma("router_gemm", pr, n_part * ((s.T + ProbRouter::kTM - 1) / ProbRouter::kTM) * ((s.n_blocks + kTN - 1) / kTN), st);
  } else {
    GemmNTArgs a{};
    a.A = h; a.Bm = Wg; a.C = p; a.perm = nullptr; a.group_off = nullptr; a.tile_off = nullptr;
    a.n_groups = 1; a.M = s.T; a.Ng = s.n_blocks; a.Kdim = s.d; a.lda = s.d; a.ldb = s.d; a.ldc = s.n_blocks;
    a.e = 1;
    launch_gemm_nt(s, a, s.T, 1, "router_gemm", st);
  }
  const size_t stride = (size_t)s.T * s.n_blocks;
#define PK(Z) MEFT_LAUNCH("route_pick", (route_pick_kernel<Z>), dim3((s.T + 3) / 4), dim3(256), 0, st, p, n_part, stride, bias, s.T, s.n_blocks, s.top_e, block_idx, block_score)
  if (s.n_blocks <= 64) PK(1);
  else if (s.n_blocks <= 128) PK(2);
  else if (s.n_blocks <= 256) PK(4);
  // beyond 256 blocks the keys take sixteen registers per lane: better for several rounds on few tokens (route call, LDS
  // keys / registers, 1024 blocks and 2048 tokens: 39.9 / 28.7 us for 16 blocks, 23.4 / 22.2 for 4, 19.1 / 20.7 for 1),
  // worse once the tokens fill the chip (16384 tokens: 112 / 153, 55 / 104, 40 / 92)
  else if (s.n_blocks <= 1024 && s.top_e >= 8 && s.T <= 2048) PK(16);
  else
#undef PK
  MEFT_LAUNCH("route_topk", route_topk_kernel, dim3(s.T), dim3(64), (size_t)s.n_blocks * 4, st, p, n_part,
              (size_t)s.T * s.n_blocks, bias,
              s.n_blocks, s.top_e, block_idx, block_score);
  return launch_status();
}

// Forward on device-resident K, V.  wait_k / wait_v (may be null): events the stream must wait for before
// the first kernel that reads K / V (used when they are being staged from host memory).
static meft_status fwd_impl(const meft_shape& s, const void* h, const void* K, const void* V,
                            const int32_t* block_idx, void* out, int32_t* idx, float* act, const FwdWs& w,
                            hipStream_t st, hipEvent_t wait_k, hipEvent_t wait_v) {
  const int n_ent = s.T * s.top_e;
  const int C = s.top_e * s.block_size;
  const int nb_used = s.n_blocks < n_ent ? s.n_blocks : n_ent;
  const int BM = s.dtype == MEFT_BF16 ? kGemmBM : gemm_f32_rows(n_ent, nb_used, s.block_size);

  if (few_tokens(s)) {
    if (wait_k && hipStreamWaitEvent(st, wait_k, 0) != hipSuccess) return MEFT_ERR_DEVICE;
    return s.dtype == MEFT_BF16 ? launch_few<bf16_t>(s, h, K, V, block_idx, out, idx, act, w.sc, st, wait_v)
                                : launch_few<float>(s, h, K, V, block_idx, out, idx, act, w.sc, st, wait_v);
  }
  const bool dense = use_dense(s);
  const bool mfma_scores = dense || use_mfma_scores(s);
  launch_dispatch(s, w, block_idx, BM, dense, mfma_scores, dense ? w.flag : nullptr, dense ? w.clear_words() : 0, st);
  const int bsp = round64(s.block_size);
  const TokenSched sched{w.sched_pairs, w.sched_tiles, w.sched_len, sched_cap(s), sched_max_tiles(s)};
  const uint16_t *hh = static_cast<const uint16_t*>(h), *kk = static_cast<const uint16_t*>(K),
                 *vv = static_cast<const uint16_t*>(V);
  if (wait_k && hipStreamWaitEvent(st, wait_k, 0) != hipSuccess) return MEFT_ERR_DEVICE;
  if (mfma_scores) {
    auto fill = [&](auto& ps) {
      ps.X = hh; ps.W = kk; ps.perm = w.perm; ps.tok_of_slot = w.tok_of_slot; ps.sched = sched;
      ps.e = s.top_e; ps.bs = s.block_size; ps.bsp = bsp; ps.d = s.d; ps.sc = w.sc;
    };
    if (dense) {
      launch_tok<TokKCLarge<kTokSlotScores>, TokKCSmall<kTokSlotScores>>("score_gemm", s, s.block_size, s.d / kTK, (uint64_t)s.T * s.d * 2, (uint64_t)s.N * s.d * 2, (uint64_t)n_ent * s.block_size * 4, fill, st);
    } else {
      ProbTokKC<kTokScores> ps{};
      set_gemm_extents(ps, (uint64_t)s.T * s.d * 2, (uint64_t)s.N * s.d * 2);
      fill(ps);
      if (ps.buf && wide_tiles(s, s.block_size, s.d / kTK)) {
        WideTok<ProbTokKC<kTokScores>> pw{ps};
        launch_gemm_wide("score_gemm", pw, tile_bound(s, (s.block_size + kTN - 1) / kTN), st);
      } else {
        launch_gemm_mfma("score_gemm", ps, tile_bound(s, (s.block_size + kTN - 1) / kTN), st);
      }
    }
  } else {
    GemmNTArgs a{};
    a.A = h; a.Bm = K; a.C = w.sc; a.perm = w.perm; a.group_off = w.group_off; a.tile_off = w.tile_off;
    a.n_groups = s.n_blocks; a.M = 0; a.Ng = s.block_size; a.Kdim = s.d; a.lda = s.d; a.ldb = s.d;
    a.ldc = s.block_size; a.e = s.top_e;
    launch_gemm_nt(s, a, n_ent, nb_used, "score_gemm", st);
  }
  if (!dense && s.top_k <= kBoundMaxK && C > kBoundMinC && C <= 1024 * 64) {
    MEFT_LAUNCH("topk_select_bound", topk_select_bound_kernel, dim3(s.T), dim3(1024), 0, st, w.sc, w.sblk, C, s.block_size,
                s.top_e, s.top_k, idx, act);
  } else if (C <= kMaxLdsC) {
    // keys in registers, the smallest per-thread count that covers the C candidates with 256 threads
    uint16_t* ap = dense ? w.Ap : nullptr;
#define TK2(KPT, FULL) MEFT_LAUNCH("topk_select", (topk_select_reg_kernel<KPT, FULL>), dim3(s.T), dim3(256), 0, st, w.sc, w.sblk, C, s.block_size, s.top_e, s.top_k, idx, act, w.slot_of_ent, bsp, ap, dense ? w.flag : nullptr)
#define TK(KPT) do { if (C == 256 * (KPT)) TK2(KPT, true); else TK2(KPT, false); } while (0)
    if (C <= 256 * 4) TK(4);
    else if (C <= 256 * 8) TK(8);
    else if (C <= 256 * 16) TK(16);
    else if (C <= 256 * 32) TK(32);
    else TK(48);
#undef TK
#undef TK2
  }
  else if (C <= 1024 * 64) {
    // e.g. one block holding every neuron: 1024 threads per token, still with the keys in registers
#define TK(KPT) MEFT_LAUNCH("topk_select_big", (topk_select_reg1024_kernel<KPT>), dim3(s.T), dim3(1024), 0, st, w.sc, w.sblk, C, s.block_size, s.top_e, s.top_k, idx, act)
    if (C <= 1024 * 16) TK(16);
    else if (C <= 1024 * 32) TK(32);
    else TK(64);
#undef TK
  } else {   // beyond that the keys stay in global memory and are read once per pass
    MEFT_LAUNCH("topk_select_big", topk_select_big_kernel, dim3(s.T), dim3(1024), 0, st, w.sc, w.sblk, C,
                s.block_size, s.top_e, s.top_k, idx, act);
  }
  // (also when only the selection is wanted: a backward that reuses the staged copies relies on this wait)
  if (wait_v && hipStreamWaitEvent(st, wait_v, 0) != hipSuccess) return MEFT_ERR_DEVICE;
  if (!out) return launch_status();   // selection only
  if (dense) {
    launch_tok<ProbTokNC, TokNCSmall>("value_gemm", s, s.d, bsp / kTK, (uint64_t)n_ent * bsp * 2, (uint64_t)s.N * s.d * 2, (uint64_t)n_ent * s.d * 2, [&](auto& pv) {
      pv.A = w.Ap; pv.W = vv; pv.sched = sched; pv.bs = s.block_size; pv.bsp = bsp;
      pv.d = s.d; pv.part = w.part; pv.big_only = small_rows_of(s) > 0;
    }, st);
    launch_token_rows("out_rows", s, w.part, w, V, idx, act, out, SmallDvdk{}, st);
  } else if (s.dtype == MEFT_BF16) {
    launch_pair_rows<bf16_t, 1>("pair_out", s, V, idx, act, nullptr, out, SegFinish<bf16_t>{}, st);
  } else {
    launch_pair_rows<float, 1>("pair_out", s, V, idx, act, nullptr, out, SegFinish<float>{}, st);
  }
  return launch_status();
}

// Writes the touched rows of a gradient matrix in device staging to the host matrix.
static void launch_rows_to_host(const meft_shape& s, const int32_t* touched, const int32_t* n_touched, const void* src,
                                void* dst, hipStream_t st) {
  const int n_rows = s.N < s.T * s.top_k ? s.N : s.T * s.top_k;
  const int vec = s.d * (s.dtype == MEFT_BF16 ? 2 : 4) / 16;
  MEFT_LAUNCH("rows_to_host", rows_to_host_kernel, dim3(n_rows), dim3(256), 0, st, touched, n_touched,
              static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), vec);
}

// Where the rows of a dV in device staging go: dst, the host matrix (nullptr: dV is not staging), on `stream`.  On another
// stream than the backward's they leave as soon as they are complete, under the rest of the backward, and the caller waits
// for g_hkv.ev_out.
struct HostRows {
  void* dst = nullptr;
  hipStream_t stream = nullptr;
};

// Backward on device-resident K, V, dK, dV.  wait_v / wait_k as in fwd_impl.
static meft_status bwd_impl(const meft_shape& s, const void* h, const void* K, const void* V, const int32_t* idx,
                            const float* act, const void* dOut, void* dh, void* dK, void* dV, int32_t* touched,
                            int32_t* n_touched, const BwdWs& w, hipStream_t st, hipEvent_t wait_k,
                            hipEvent_t wait_v, HostRows dV_rows) {
  if (use_dense(s)) {
    const int bsp = round64(s.block_size);
    const uint16_t *hh = static_cast<const uint16_t*>(h), *kk = static_cast<const uint16_t*>(K),
                   *vv = static_cast<const uint16_t*>(V), *gg = static_cast<const uint16_t*>(dOut);
    // With MEFT_FLAG_REUSE_FWD the dispatch tables and the activation rows A' are the ones the forward of this step
    // left in the workspace; otherwise they are rebuilt from (idx, act).
    const bool reuse = (s.flags & MEFT_FLAG_REUSE_FWD) != 0 && !few_tokens(s);
    if (!reuse) {
      MEFT_LAUNCH("blocks_from_idx", blocks_from_idx_kernel, dim3(s.T), dim3(64), (size_t)((s.n_blocks + 31) / 32) * 4,
                  st, idx, s.top_k, s.N, s.block_size, s.n_blocks, s.top_e, w.sblk);
      launch_dispatch(s, w, nullptr, kGemmBM, true, true, w.flag, w.clear_words(), st);
      // a token's rows take top_e * bsp * 2 bytes of LDS: up to 96 KB where blocks are small and many (the default
      // limit of a launch is 64 KB)
      static std::once_flag act_rows_configured;
      std::call_once(act_rows_configured, [] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&act_rows_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 4 * kMaxLdsC * 2);
      });
      MEFT_LAUNCH("act_rows", act_rows_kernel, dim3(s.T), dim3(256), (size_t)s.top_e * bsp * 2, st, idx, act, s.top_k,
                  s.N, s.block_size, bsp, s.top_e, w.sblk, w.slot_of_ent, w.Ap, w.flag);
    }
    const int small = small_rows_of(s);
    // (with host-resident V still on its way the small groups' gradients wait for it)
    launch_bwd_head(s, w.flag, w.chunk_cnt, touched, n_touched, small && !wait_v ? &w : nullptr, V, dOut, idx, act, st);
    const TokenSched sched{w.sched_pairs, w.sched_tiles, w.sched_len, sched_cap(s), sched_max_tiles(s)};
    const int big_only = small > 0;   // the small groups: computed pair by pair
    const int n_ent = s.T * s.top_e;
    NeuArgs pn{};
    pn.tok_of_slot = w.tok_of_slot; pn.flag = w.flag;
    pn.sched = sched; pn.big_only = big_only; pn.n_groups = s.n_blocks; pn.bs = s.block_size; pn.bsp = bsp; pn.d = s.d;
    pn.wide = wide_neu(s);
    pn.a_bytes = (uint64_t)(1 + 2 * (uint64_t)n_ent) * bsp * 2; pn.x_bytes = (uint64_t)s.T * s.d * 2;
    // dV first: it needs neither K nor V (so it also runs while host-resident K, V are still on their way), and it
    // gathers the same dOut rows as the activation-gradient GEMM that follows it
    pn.A = w.Ap; pn.zrow = -1; pn.X = gg; pn.G = static_cast<uint16_t*>(dV);
    launch_neu("dV_gemm", pn, st);
    SmallDvdk dv{};
    if (small) {
      dv.nx = (s.block_size + kSmallRowChunk - 1) / kSmallRowChunk;
      dv.ny = s.n_blocks < kSmallGrpGrid ? s.n_blocks : kSmallGrpGrid;
      dv.n_wg = dv.nx * dv.ny;
      dv.h = reinterpret_cast<const bf16_t*>(hh); dv.dOut = reinterpret_cast<const bf16_t*>(gg);
      dv.act = act; dv.ds32 = w.ds32;
      dv.small_grp = w.small_grp; dv.small_cnt = w.small_cnt; dv.group_off = w.group_off; dv.tok_of_slot = w.tok_of_slot;
      dv.dK = static_cast<bf16_t*>(dK); dv.dV = static_cast<bf16_t*>(dV);
    }
    auto launch_small_dvdk = [&]() {
      TokenRows a{};
      a.idx = idx; a.d = s.d; a.k = s.top_k; a.N = s.N; a.bs = s.block_size;
      MEFT_LAUNCH("small_dvdk", small_dvdk_kernel, dim3(dv.n_wg), dim3(256), 0, st, a, dv);
      dv.n_wg = 0;
    };
    auto dv_to_host = [&]() -> bool {   // dV is complete in its staging
      if (small) launch_small_dvdk();
      const hipStream_t to = dV_rows.stream;
      if (to != st && (hipEventRecord(g_hkv.ev_dv, st) != hipSuccess || hipStreamWaitEvent(to, g_hkv.ev_dv, 0) != hipSuccess)) return false;
      launch_rows_to_host(s, touched, n_touched, dV, dV_rows.dst, to);
      return to == st || hipEventRecord(g_hkv.ev_out, to) == hipSuccess;
    };
    if (dV_rows.dst && !(small && wait_v) && !dv_to_host()) return MEFT_ERR_DEVICE;
    if (wait_v && hipStreamWaitEvent(st, wait_v, 0) != hipSuccess) return MEFT_ERR_DEVICE;
    launch_tok<TokKCLarge<kTokMasked>, TokKCSmall<kTokMasked>>("dact_gemm", s, s.block_size, s.d / kTK, (uint64_t)s.T * s.d * 2, (uint64_t)s.N * s.d * 2, (uint64_t)n_ent * bsp * 2, [&](auto& pg) {
      pg.X = gg; pg.W = vv; pg.perm = w.perm; pg.tok_of_slot = w.tok_of_slot; pg.sched = sched;
      pg.e = s.top_e; pg.bs = s.block_size; pg.bsp = bsp; pg.d = s.d; pg.Ap = w.Ap; pg.DS = w.DS;
      pg.big_only = big_only;
    }, st);
    if (small && wait_v) {
      launch_bwd_head(s, w.flag, w.chunk_cnt, touched, n_touched, &w, V, dOut, idx, act, st);
      if (dV_rows.dst && !dv_to_host()) return MEFT_ERR_DEVICE;
    }
    if (wait_k && hipStreamWaitEvent(st, wait_k, 0) != hipSuccess) return MEFT_ERR_DEVICE;
    if (dh) {
      launch_tok<ProbTokNC, TokNCSmall>("dh_gemm", s, s.d, bsp / kTK, (uint64_t)n_ent * bsp * 2, (uint64_t)s.N * s.d * 2, (uint64_t)n_ent * s.d * 2, [&](auto& ph) {
        ph.A = w.DS; ph.W = kk; ph.sched = sched; ph.bs = s.block_size; ph.bsp = bsp;
        ph.d = s.d; ph.part = w.part; ph.big_only = big_only;
      }, st);
      if (dv.n_wg && !dvdk_beside_rows(s)) launch_small_dvdk();
      launch_token_rows("dh_rows", s, w.part, w, K, idx, w.ds32, dh, dv, st);
    } else if (dv.n_wg) {
      launch_small_dvdk();
    }
    pn.A = w.DS; pn.zrow = -(n_ent + 1); pn.X = hh; pn.G = static_cast<uint16_t*>(dK);
    launch_neu("dK_gemm", pn, st);
    return launch_status();
  }

  if (wait_v && hipStreamWaitEvent(st, wait_v, 0) != hipSuccess) return MEFT_ERR_DEVICE;
  if (wait_k && hipStreamWaitEvent(st, wait_k, 0) != hipSuccess) return MEFT_ERR_DEVICE;
  if (s.dtype == MEFT_BF16) launch_pair_bwd<bf16_t>(s, w, h, K, V, idx, act, dOut, dh, dK, dV, touched, n_touched, st);
  else launch_pair_bwd<float>(s, w, h, K, V, idx, act, dOut, dh, dK, dV, touched, n_touched, st);
  if (dV_rows.dst) launch_rows_to_host(s, touched, n_touched, dV, dV_rows.dst, st);   // complete with dK: nothing to gain
  return launch_status();
}

// Whether the contractions of the batch union gather K's and V's rows themselves instead of reading compacted copies: the
// large tiles by buffer loads do.  The copies cost 2 x 43 us of 747 at 1023 tokens, 16384 rows x 2048.
static bool union_direct(const meft_shape& s, const UnionGeom& g) {
  return !g_force_global_loads && (uint64_t)s.N * s.d * 2 < kBufLimit &&
         (uint64_t)s.T * s.d * 2 < kBufLimit && (uint64_t)s.T * g.nvb * g.vbs * 2 < kBufLimit && !small_tiles(g.vs, g.vbs) &&
         !small_tiles(g.vs, s.d);
}

template <class P>
static void fill_union_kc(P& p, const meft_shape& s, const UnionGeom& g, const UnionWs& w, const TokenSched& sched, const void* X,
                          const void* W, uint16_t* DS, const uint16_t* Ap) {
  set_gemm_extents(p, (uint64_t)s.T * s.d * 2, (uint64_t)s.N * s.d * 2);
  p.X = static_cast<const uint16_t*>(X); p.W = static_cast<const uint16_t*>(W); p.tag = w.rowtag;
  p.perm = w.perm; p.tok_of_slot = w.tok_of_slot; p.sched = sched; p.e = g.nvb; p.bs = g.vbs; p.bsp = g.vbs; p.d = s.d;
  p.DS = DS; p.Ap = Ap;
}

static void launch_union_nc(const char* name, const meft_shape& s, const UnionGeom& g, const UnionWs& w, const TokenSched& sched,
                            const uint16_t* A, const void* W, hipStream_t st) {
  launch_tok_buf<ProbTokNCRows>(name, g.vs, s.d, g.vbs / kTK, [&](auto& p) {
    set_gemm_extents(p, (uint64_t)s.T * g.nvb * g.vbs * 2, (uint64_t)s.N * s.d * 2);
    p.A = A; p.W = static_cast<const uint16_t*>(W); p.tag = w.rowtag; p.sched = sched; p.bs = g.vbs; p.bsp = g.vbs; p.d = s.d;
    p.part = w.part;
  }, st);
}

// Shared front part of the batch-union forward and backward: index structure from n_S, tile schedule, compacted
// K and V, and A' = ReLU(h K[S]^T).
static void union_front(const meft_shape& s, const UnionGeom& g, const UnionWs& w, bool direct, const void* h, const void* K,
                        const void* V, const int32_t* S, const int32_t* n_S, hipStream_t st) {
  const size_t n_slots = (size_t)g.nvb * s.T, n_rows = (size_t)g.nvb * g.vbs;
  const size_t n_thr = (n_slots + kSlotPad) > n_rows + kTagPad ? (n_slots + kSlotPad) : n_rows + kTagPad;
  MEFT_LAUNCH("union_maps", union_maps_kernel, dim3((unsigned)((n_thr + 255) / 256)), dim3(256), 0, st, S, n_S, g.cap,
              s.N, s.T, g.vbs, g.nvb, w.sblk, w.perm, w.tok_of_slot, w.slot_of_ent, w.group_off, w.rowtag,
              reinterpret_cast<int32_t*>(w.zrow));   // (vbs % 64 == 0)
  MEFT_LAUNCH("build_sched", build_sched_kernel, dim3(1), dim3(1024), 0, st, w.group_off, g.nvb, sched_cap(g.vs),
              w.sched_pairs, w.sched_tiles, w.sched_len, 0);
  const TokenSched sched{w.sched_pairs, w.sched_tiles, w.sched_len, sched_cap(g.vs), sched_max_tiles(g.vs)};
  if (direct) {
    launch_tok_buf<ProbTokKCRows<kTokRelu>>("union_score_gemm", g.vs, g.vbs, s.d / kTK, [&](auto& pr) {
      fill_union_kc(pr, s, g, w, sched, h, K, w.Ap, nullptr);
    }, st);
    return;
  }
  const int rows_grid = (int)(n_rows < 4096 ? n_rows : 4096);
  MEFT_LAUNCH("gather_rows", gather_rows_kernel, dim3(rows_grid, 2), dim3(256), 0, st, static_cast<const uint16_t*>(K),
              static_cast<const uint16_t*>(V), S, n_S, g.cap, s.N, s.d, g.vbs, w.Kc, w.Vc);
  launch_tok<TokKCLarge<kTokRelu>, TokKCSmall<kTokRelu>>("union_score_gemm", g.vs, g.vbs, s.d / kTK, (uint64_t)s.T * s.d * 2, (uint64_t)n_rows * s.d * 2, (uint64_t)s.T * g.nvb * g.vbs * 2, [&](auto& pr) {
    pr.X = static_cast<const uint16_t*>(h); pr.W = w.Kc; pr.perm = w.perm; pr.tok_of_slot = w.tok_of_slot;
    pr.sched = sched; pr.e = g.nvb; pr.bs = g.vbs; pr.bsp = g.vbs; pr.d = s.d;
    pr.DS = w.Ap;
  }, st);
}

extern "C" {

size_t meft_union_workspace_bytes(const meft_shape* shape) {
  UnionGeom g;
  if (check_shape(shape) != MEFT_OK || !union_geom(*shape, g)) return 0;
  return UnionWs(*shape, g, nullptr).bytes;
}

meft_status meft_union_fwd(const meft_shape* shape, const void* h, const void* K, const void* V, const int32_t* idx,
                           void* out, int32_t* S, int32_t* n_S, void* ws, size_t ws_bytes, void* stream) {
  meft_status rc = check_shape(shape);
  if (rc != MEFT_OK) return rc;
  const meft_shape& s = *shape;
  UnionGeom g;
  if (!union_geom(s, g)) return MEFT_ERR_UNSUPPORTED;
  if (!h || !K || !V || !idx || !out || !S || !n_S) return MEFT_ERR_INVALID_ARG;
  if (!aligned16(h) || !aligned16(K) || !aligned16(V) || !aligned16(out)) return MEFT_ERR_INVALID_ARG;
  const UnionWs w(s, g, ws);
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) || ws_bytes < w.bytes) return MEFT_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  if (s.T == 0) {
    MEFT_LAUNCH("fill_i32", fill_i32_kernel, dim3(1), dim3(64), 0, st, n_S, (size_t)1, 0);
    return launch_status();
  }
  // S = ascending ids of the neurons that some token selected
  const int P = s.T * s.top_k;
  MEFT_LAUNCH("fill_i32", fill_i32_kernel, dim3((unsigned)(((size_t)s.N + 255) / 256)), dim3(256), 0, st, w.flag,
              (size_t)s.N, 0);
  MEFT_LAUNCH("mark_idx", mark_idx_kernel, dim3((P + 255) / 256), dim3(256), 0, st, idx, P, s.N, w.flag);
  launch_bwd_head(s, w.flag, w.chunk_cnt, S, n_S, nullptr, nullptr, nullptr, nullptr, nullptr, st);
  const bool direct = union_direct(s, g);
  union_front(s, g, w, direct, h, K, V, S, n_S, st);
  const TokenSched sched{w.sched_pairs, w.sched_tiles, w.sched_len, sched_cap(g.vs), sched_max_tiles(g.vs)};
  if (direct) launch_union_nc("union_value_gemm", s, g, w, sched, w.Ap, V, st);
  else launch_tok<ProbTokNC, TokNCSmall>("union_value_gemm", g.vs, s.d, g.vbs / kTK, (uint64_t)s.T * g.nvb * g.vbs * 2, (uint64_t)g.nvb * g.vbs * s.d * 2, (uint64_t)s.T * g.nvb * s.d * 2, [&](auto& pv) {
    pv.A = w.Ap; pv.W = w.Vc; pv.sched = sched; pv.bs = g.vbs; pv.bsp = g.vbs;
    pv.d = s.d; pv.part = w.part;
  }, st);
  launch_token_rows("union_out_rows", g.vs, w.part, w, nullptr, nullptr, nullptr, out, SmallDvdk{}, st);
  return launch_status();
}

meft_status meft_union_bwd(const meft_shape* shape, const void* h, const void* K, const void* V, const int32_t* S,
                           const int32_t* n_S, const void* dOut, void* dh, void* dK, void* dV, void* ws,
                           size_t ws_bytes, void* stream) {
  meft_status rc = check_shape(shape);
  if (rc != MEFT_OK) return rc;
  const meft_shape& s = *shape;
  UnionGeom g;
  if (!union_geom(s, g)) return MEFT_ERR_UNSUPPORTED;
  if (!h || !K || !V || !S || !n_S || !dOut || !dK || !dV) return MEFT_ERR_INVALID_ARG;
  if (!aligned16(h) || !aligned16(K) || !aligned16(V) || !aligned16(dOut) || !aligned16(dK) || !aligned16(dV) ||
      (dh && !aligned16(dh)))
    return MEFT_ERR_INVALID_ARG;
  const UnionWs w(s, g, ws);
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) || ws_bytes < w.bytes) return MEFT_ERR_WORKSPACE;
  if (s.T == 0) return MEFT_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  const bool direct = union_direct(s, g);
  union_front(s, g, w, direct, h, K, V, S, n_S, st);
  const TokenSched sched{w.sched_pairs, w.sched_tiles, w.sched_len, sched_cap(g.vs), sched_max_tiles(g.vs)};
  const uint16_t *hh = static_cast<const uint16_t*>(h), *gg = static_cast<const uint16_t*>(dOut);
  if (direct) {
    launch_tok_buf<ProbTokKCRows<kTokMasked>>("union_dact_gemm", g.vs, g.vbs, s.d / kTK, [&](auto& pg) {
      fill_union_kc(pg, s, g, w, sched, gg, V, w.DS, w.Ap);
    }, st);
  } else
  launch_tok<TokKCLarge<kTokMasked>, TokKCSmall<kTokMasked>>("union_dact_gemm", g.vs, g.vbs, s.d / kTK, (uint64_t)s.T * s.d * 2, (uint64_t)g.nvb * g.vbs * s.d * 2, (uint64_t)s.T * g.nvb * g.vbs * 2, [&](auto& pg) {
    pg.X = gg; pg.W = w.Vc; pg.perm = w.perm; pg.tok_of_slot = w.tok_of_slot; pg.sched = sched;
    pg.e = g.nvb; pg.bs = g.vbs; pg.bsp = g.vbs; pg.d = s.d; pg.Ap = w.Ap; pg.DS = w.DS;
  }, st);
  if (dh) {
    if (direct) launch_union_nc("union_dh_gemm", s, g, w, sched, w.DS, K, st);
    else launch_tok<ProbTokNC, TokNCSmall>("union_dh_gemm", g.vs, s.d, g.vbs / kTK, (uint64_t)s.T * g.nvb * g.vbs * 2, (uint64_t)g.nvb * g.vbs * s.d * 2, (uint64_t)s.T * g.nvb * s.d * 2, [&](auto& ph) {
      ph.A = w.DS; ph.W = w.Kc; ph.sched = sched; ph.bs = g.vbs; ph.bsp = g.vbs;
      ph.d = s.d; ph.part = w.part;
    }, st);
    launch_token_rows("union_dh_rows", g.vs, w.part, w, nullptr, nullptr, nullptr, dh, SmallDvdk{}, st);
  }
  NeuArgs pn{};
  pn.tok_of_slot = w.tok_of_slot; pn.flag = w.rowtag;
  pn.sched = sched; pn.big_only = 0; pn.n_groups = g.nvb; pn.bs = g.vbs; pn.bsp = g.vbs; pn.d = s.d;
  pn.wide = wide_neu(g.vs);
  pn.a_bytes = (1 + 2 * (uint64_t)s.T * g.nvb) * g.vbs * 2; pn.x_bytes = (uint64_t)s.T * s.d * 2;
  // written to the rows of S directly: a pass over compacted gradients took 2 x 24 us at 16384 rows x 2048
  pn.A = w.Ap; pn.zrow = -1; pn.X = gg; pn.G = static_cast<uint16_t*>(dV);
  launch_neu<ProbNeuTNRows>("union_dV_gemm", pn, st);
  pn.A = w.DS; pn.zrow = -(s.T * g.nvb + 1); pn.X = hh; pn.G = static_cast<uint16_t*>(dK);
  launch_neu<ProbNeuTNRows>("union_dK_gemm", pn, st);
  return launch_status();
}

meft_status meft_check_shape(const meft_shape* shape) { return check_shape(shape); }

size_t meft_workspace_bytes(const meft_shape* shape) {
  if (check_shape(shape) != MEFT_OK) return 0;
  return workspace_bytes(*shape);
}

const char* meft_status_string(meft_status status) {
  switch (status) {
    case MEFT_OK: return "ok";
    case MEFT_ERR_INVALID_ARG: return "invalid argument";
    case MEFT_ERR_UNSUPPORTED: return "unsupported shape or flag";
    case MEFT_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case MEFT_ERR_DEVICE: return "device error";
  }
  return "unknown status";
}

meft_status meft_route(const meft_shape* shape, const void* h, const void* Wg, const float* bias,
                       int32_t* block_idx, float* block_score, void* ws, size_t ws_bytes, void* stream) {
  meft_status rc = check_shape(shape);
  if (rc != MEFT_OK) return rc;
  const meft_shape& s = *shape;
  if (!h || !Wg || !block_idx || !aligned16(h) || !aligned16(Wg)) return MEFT_ERR_INVALID_ARG;
  RouteWs w(s, ws);
  if ((rc = check_ws(s, ws, ws_bytes)) != MEFT_OK) return rc;
  if (s.T == 0) return MEFT_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  return route_impl(s, h, Wg, bias, block_idx, block_score, w.p, st);
}

// Address of `scratch` on the current device, looked up on the first call with that device current.
static float* static_scratch_ptr() {
  constexpr int kMaxDevices = 64;
  static void* ptr[kMaxDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  if (!ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    ptr[dev] = p;
  }
  return static_cast<float*>(ptr[dev]);
}

meft_status meft_route_static(const meft_shape* shape, const void* h, const void* Wg, const float* bias,
                              int32_t* block_idx, float* block_score, void* stream) {
  meft_status rc = check_shape(shape);
  if (rc != MEFT_OK) return rc;
  const meft_shape& s = *shape;
  if (!h || !Wg || !block_idx || !aligned16(h) || !aligned16(Wg)) return MEFT_ERR_INVALID_ARG;
  if (RouteWs(s, nullptr).bytes > MEFT_ROUTE_STATIC_BYTES) return MEFT_ERR_WORKSPACE;
  if (s.T == 0) return MEFT_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  float* p = static_scratch_ptr();
  if (!p) { (void)launch_status(); return MEFT_ERR_DEVICE; }
  const bool timing = g_prof_on;   // per-kernel timing creates events: off inside this call
  g_prof_on = false;
  rc = route_impl(s, h, Wg, bias, block_idx, block_score, p, st);
  g_prof_on = timing;
  return rc;
}

meft_status meft_sparse_fwd(const meft_shape* shape, const void* h, const void* K, const void* V,
                            const int32_t* block_idx, void* out, int32_t* idx, float* act, void* ws,
                            size_t ws_bytes, void* stream) {
  meft_status rc = check_shape(shape);
  if (rc != MEFT_OK) return rc;
  const meft_shape& s = *shape;
  if (!h || !K || !V || !block_idx || !idx || !act) return MEFT_ERR_INVALID_ARG;
  if (!aligned16(h) || !aligned16(K) || !aligned16(V) || (out && !aligned16(out))) return MEFT_ERR_INVALID_ARG;
  FwdWs w(s, ws);
  if ((rc = check_ws(s, ws, ws_bytes)) != MEFT_OK) return rc;
  if (s.T == 0) return MEFT_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  if (!(s.flags & MEFT_FLAG_HOST_KV)) return fwd_impl(s, h, K, V, block_idx, out, idx, act, w, st, nullptr, nullptr);

  // K, V in pinned host memory: find the blocks in use, fetch them on the side stream (K first, then V) while
  // the dispatch runs, and let the scoring wait for K and the value stage for V.
  if (!hostkv_init()) return MEFT_ERR_DEVICE;
  HostKvWs hw(s, ws);
  if (s.flags & MEFT_FLAG_PRESTAGED) {   // the copies were requested by meft_hostkv_stage
    StageSlot* sl = stage_slot(ws, false);
    if (!sl) return MEFT_ERR_INVALID_ARG;
    sl->ws = nullptr;   // one stage call serves one forward
    return fwd_impl(s, h, hw.Kd, hw.Vd, block_idx, out, idx, act, w, st, sl->ev_k, sl->ev_v);
  }
  if (hipEventRecord(g_hkv.ev_entry, st) != hipSuccess || hipStreamWaitEvent(g_hkv.side, g_hkv.ev_entry, 0) != hipSuccess)
    return MEFT_ERR_DEVICE;   // the device copies may still be read by work queued earlier on this stream
  MEFT_LAUNCH("sort_blocks", sort_blocks_kernel, dim3((s.T + 255) / 256), dim3(256), 0, st, block_idx, s.T,
              s.top_e, s.n_blocks, w.sblk);
  MEFT_LAUNCH("count_blocks", count_blocks_kernel, dim3(s.n_blocks), dim3(1024), 0, st, w.sblk, s.T * s.top_e, w.cnt);
  if ((rc = hostkv_fetch(s, w.cnt, K, hw.Kd, g_hkv.ev_k, V, hw.Vd, g_hkv.ev_v, st)) != MEFT_OK) return rc;
  return fwd_impl(s, h, hw.Kd, hw.Vd, block_idx, out, idx, act, w, st, g_hkv.ev_k, g_hkv.ev_v);
}

meft_status meft_hostkv_stage(const meft_shape* shape, const int32_t* block_idx, const void* K, const void* V, void* ws,
                              size_t ws_bytes, void* stream) {
  meft_status rc = check_shape(shape);
  if (rc != MEFT_OK) return rc;
  const meft_shape& s = *shape;
  if (!(s.flags & MEFT_FLAG_HOST_KV) || !block_idx || !K || !V || !aligned16(K) || !aligned16(V)) return MEFT_ERR_INVALID_ARG;
  FwdWs w(s, ws);
  if ((rc = check_ws(s, ws, ws_bytes)) != MEFT_OK) return rc;
  if (s.T == 0) return MEFT_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  if (!hostkv_init()) return MEFT_ERR_DEVICE;
  HostKvWs hw(s, ws);
  StageSlot* sl = stage_slot(ws, true);
  if (!sl) return MEFT_ERR_DEVICE;
  if (hipEventRecord(g_hkv.ev_entry, st) != hipSuccess || hipStreamWaitEvent(g_hkv.side, g_hkv.ev_entry, 0) != hipSuccess)
    return MEFT_ERR_DEVICE;   // the device copies may still be read by work queued earlier on this stream
  MEFT_LAUNCH("sort_blocks", sort_blocks_kernel, dim3((s.T + 255) / 256), dim3(256), 0, st, block_idx, s.T,
              s.top_e, s.n_blocks, w.sblk);
  MEFT_LAUNCH("count_blocks", count_blocks_kernel, dim3(s.n_blocks), dim3(1024), 0, st, w.sblk, s.T * s.top_e, w.cnt);
  if ((rc = hostkv_fetch(s, w.cnt, K, hw.Kd, sl->ev_k, V, hw.Vd, sl->ev_v, st)) != MEFT_OK) return rc;
  return launch_status();
}

meft_status meft_sparse_bwd(const meft_shape* shape, const void* h, const void* K, const void* V,
                            const int32_t* idx, const float* act, const void* dOut, void* dh, void* dK,
                            void* dV, int32_t* touched, int32_t* n_touched, void* ws, size_t ws_bytes,
                            void* stream) {
  meft_status rc = check_shape(shape);
  if (rc != MEFT_OK) return rc;
  const meft_shape& s = *shape;
  if (!h || !K || !V || !idx || !act || !dOut || !dK || !dV || !touched || !n_touched) return MEFT_ERR_INVALID_ARG;
  if (!aligned16(h) || !aligned16(K) || !aligned16(V) || !aligned16(dOut) || !aligned16(dK) || !aligned16(dV) ||
      (dh && !aligned16(dh)))
    return MEFT_ERR_INVALID_ARG;
  BwdWs w(s, ws);
  if ((rc = check_ws(s, ws, ws_bytes)) != MEFT_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  if (s.T == 0) {
    MEFT_LAUNCH("fill_i32", fill_i32_kernel, dim3(1), dim3(64), 0, st, n_touched, (size_t)1, 0);
    return launch_status();
  }
  if (!(s.flags & MEFT_FLAG_HOST_KV))
    return bwd_impl(s, h, K, V, idx, act, dOut, dh, dK, dV, touched, n_touched, w, st, nullptr, nullptr, HostRows{});

  // K, V, dK, dV in pinned host memory: fetch the blocks that hold a selected neuron (V first: the activation
  // gradient needs it before dh needs K), compute into device staging, then write the touched rows back.
  if (!hostkv_init()) return MEFT_ERR_DEVICE;
  HostKvWs hw(s, ws);
  // Under capture everything stays on the caller's stream: a stream of the library's that joined a capture would stay part
  // of it until it ends, and other calls' work on that stream would be recorded instead of run.
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool early = use_dense(s) && hipStreamIsCapturing(st, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone;
  const HostRows dV_rows{dV, early ? rows_stream() : st};
  if (s.flags & MEFT_FLAG_KEEP_STAGED) {
    // the forward of this step left the blocks in use in the workspace, and its copies are ordered before
    // anything enqueued here (the forward made `st` wait for them)
    rc = bwd_impl(s, h, hw.Kd, hw.Vd, idx, act, dOut, dh, hw.dKd, hw.dVd, touched, n_touched, w, st, nullptr, nullptr, dV_rows);
  } else {
  if (hipEventRecord(g_hkv.ev_entry, st) != hipSuccess || hipStreamWaitEvent(g_hkv.side, g_hkv.ev_entry, 0) != hipSuccess)
    return MEFT_ERR_DEVICE;
  int32_t* sblk_tmp = hw.pair_blk;
  int32_t* cnt_tmp = hw.pair_blk_cnt;
  MEFT_LAUNCH("blocks_of_pairs", blocks_of_pairs_kernel, dim3((s.T * s.top_k + 255) / 256), dim3(256), 0, st, idx,
              s.T * s.top_k, s.N, s.block_size, sblk_tmp);
  MEFT_LAUNCH("count_blocks", count_blocks_kernel, dim3(s.n_blocks), dim3(1024), 0, st, sblk_tmp, s.T * s.top_k,
              cnt_tmp);
  if ((rc = hostkv_fetch(s, cnt_tmp, V, hw.Vd, g_hkv.ev_v, K, hw.Kd, g_hkv.ev_k, st)) != MEFT_OK) return rc;
  rc = bwd_impl(s, h, hw.Kd, hw.Vd, idx, act, dOut, dh, hw.dKd, hw.dVd, touched, n_touched, w, st, g_hkv.ev_k,
                g_hkv.ev_v, dV_rows);
  }
  if (rc == MEFT_OK) launch_rows_to_host(s, touched, n_touched, hw.dKd, dK, st);
  // (also after an error: what has been enqueued still reads the workspace and writes dV)
  if (early && hipStreamWaitEvent(st, g_hkv.ev_out, 0) != hipSuccess) return MEFT_ERR_DEVICE;
  return rc != MEFT_OK ? rc : launch_status();
}

meft_status meft_adam_rows(const meft_shape* shape, const meft_adam* hp, void* W, const void* G, float* m,
                           float* v, float* master, const int32_t* touched, const int32_t* n_touched,
                           void* stream) {
  const meft_status cs = check_shape(shape);
  if (cs != MEFT_OK) return cs;
  const meft_shape& s = *shape;
  if (s.flags & MEFT_FLAG_HOST_KV) return MEFT_ERR_UNSUPPORTED;   // the kernel reads and writes device memory
  if (!hp || !W || !G || !m || !v || !touched || !n_touched) return MEFT_ERR_INVALID_ARG;
  if (!aligned16(W) || !aligned16(G) || !aligned16(m) || !aligned16(v) || (master && !aligned16(master)))
    return MEFT_ERR_INVALID_ARG;
  if (hp->step < 1 || !(hp->beta1 >= 0.f && hp->beta1 < 1.f) || !(hp->beta2 >= 0.f && hp->beta2 < 1.f) ||
      !(hp->eps >= 0.f) || !(hp->lr == hp->lr))
    return MEFT_ERR_INVALID_ARG;
  if (s.T == 0) return MEFT_OK;
  AdamScalars a;
  const double b1 = hp->beta1, b2 = hp->beta2;
  a.lr = hp->lr; a.b1 = hp->beta1; a.b2 = hp->beta2; a.eps = hp->eps;
  a.omb1 = (float)(1.0 - b1); a.omb2 = (float)(1.0 - b2);
  a.inv_c1 = (float)(1.0 / (1.0 - std::pow(b1, (double)hp->step)));
  a.inv_c2 = (float)(1.0 / (1.0 - std::pow(b2, (double)hp->step)));
  const int64_t cap = (int64_t)s.T * s.top_k < (int64_t)s.N ? (int64_t)s.T * s.top_k : (int64_t)s.N;
  const int grid = (int)(cap < 4096 ? cap : 4096);   // rows are walked with a grid stride
  hipStream_t st = static_cast<hipStream_t>(stream);
  MEFT_API_LOCK();
  clear_stale_error();
  if (s.dtype == MEFT_BF16)
    MEFT_LAUNCH("adam_rows", adam_rows_kernel<bf16_t>, dim3(grid), dim3(256), 0, st, static_cast<bf16_t*>(W),
                static_cast<const bf16_t*>(G), m, v, master, touched, n_touched, s.N, s.d, a);
  else
    MEFT_LAUNCH("adam_rows", adam_rows_kernel<float>, dim3(grid), dim3(256), 0, st, static_cast<float*>(W),
                static_cast<const float*>(G), m, v, master, touched, n_touched, s.N, s.d, a);
  return launch_status();
}

meft_status meft_probe_copy(void* dst, const void* src, size_t bytes, void* stream) {
  if (!dst || !src || !aligned16(dst) || !aligned16(src) || bytes % 16 != 0) return MEFT_ERR_INVALID_ARG;
  if (bytes == 0) return MEFT_OK;
  const size_t n = bytes / 16;
  MEFT_API_LOCK();
  clear_stale_error();
  MEFT_LAUNCH("probe_copy", probe_copy_kernel, dim3(256 * 16), dim3(256), 0, static_cast<hipStream_t>(stream),
              static_cast<u32x4*>(dst), static_cast<const u32x4*>(src), n);
  return launch_status();
}

meft_status meft_probe_mfma(float* out, int workgroups, int iters, void* stream) {
  if (!out || workgroups < 1 || workgroups > 65536 || iters < 1) return MEFT_ERR_INVALID_ARG;
  MEFT_API_LOCK();
  clear_stale_error();
  MEFT_LAUNCH("probe_mfma", probe_mfma_kernel, dim3(workgroups), dim3(256), 0, static_cast<hipStream_t>(stream), out,
              iters);
  return launch_status();
}

const char* meft_last_device_error(void) { return hipGetErrorString(g_last_device_error); }

void meft_debug_global_loads(int on) {
  MEFT_API_LOCK();
  g_force_global_loads = on != 0;
}

void meft_profile_enable(int on) {
  MEFT_API_LOCK();
  for (auto& e : g_prof) {
    (void)hipEventDestroy(e.start);
    (void)hipEventDestroy(e.stop);
  }
  g_prof.clear();
  g_prof_on = on != 0;
}

int meft_profile_read(const char** names, int32_t* launches, float* total_ms, int cap) {
  MEFT_API_LOCK();
  int n = 0;
  for (auto& e : g_prof) {
    if (hipEventSynchronize(e.stop) != hipSuccess) continue;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, e.start, e.stop) != hipSuccess) continue;
    int slot = -1;
    for (int i = 0; i < n; ++i)
      if (std::strcmp(names[i], e.name) == 0) { slot = i; break; }
    if (slot < 0) {
      if (n >= cap) continue;
      slot = n++;
      names[slot] = e.name;
      launches[slot] = 0;
      total_ms[slot] = 0.f;
    }
    launches[slot] += 1;
    total_ms[slot] += ms;
  }
  return n;
}

}  // extern "C"
