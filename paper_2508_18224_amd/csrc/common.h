// Shared declarations of the gfx950 selected-attention library: workspace layout, launch prototypes and
// small device helpers.  Everything here is internal; the public surface is include/nsa_sel.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <atomic>

#include "../../include/nsa_sel.h"

namespace nsa {

constexpr int kBlock = 64;         // tokens of the smaller of the two block sizes (B_K = 64 or 2 * 64)
constexpr int kD = 128;            // head dimension
constexpr int kMaxUnit = 2048;     // most list entries of one work unit (the size used for long inputs)
constexpr int kMinUnit = 256;       // the smallest a caller may ask for (the library itself goes lower for tiny inputs)
constexpr int kMaxTopk = 32;
constexpr int kTileTokens = 64;    // query tokens of a tile of the dense forward path (whatever B_K is)
constexpr int kDenseMax = 32;      // most 64-key pieces one (query tile, kv head) routes through the dense path
constexpr int kDenseHash = 1024;   // per-wavefront counters of the detection pass (block id modulo this)

// Host-computed description of the index workspace (byte offsets from its base, all 256-aligned).
struct IndexLayout {
  int32_t T, nseq, hkv, topk, causal;
  int32_t window;       // 0 or the sliding-window length in tokens
  int32_t bk;           // B_K: tokens per KV block, 64 or 128
  int32_t b_cap;        // list stride: T / bk + nseq  (>= real number of blocks)
  int32_t n_lists;      // hkv * b_cap
  int32_t n_chunks;     // chunks of query tiles the inversion works by (index_chunks)
  int32_t n_groups;     // groups of 64 lists of a kv head: ceil(b_cap / 64)
  int64_t p_max;        // T * hkv * topk
  int32_t unit;         // list entries per work unit of the attention kernels (see work_unit_entries)
  int32_t units_max;    // upper bound of the number of work units
  int32_t dense;        // 1: (query tile, KV block) pairs most of the tile's tokens keep go through the dense path
  int32_t brief;        // 1: the forward is k_fwd_short (see short_forward)
  int32_t t_cap;        // query tiles of kTileTokens tokens: T / kTileTokens + nseq (>= real number of tiles)
  size_t blk_base, blk_tok0, blk_len, chunk_off, cnt, off, qent, vmask, slotpos;
  size_t u_nu, u_rec, group_sum;
  size_t tile_base, tile_tok0, tile_len, tile_seq, dmask, d_cnt, d_piece, d_mask;
  size_t total;
};

// One work unit of the attention kernels: up to `unit` consecutive entries of one list.  A workgroup finds everything it
// needs to request its keys, values and entries in this one record.
struct UnitRec {
  int32_t e0, ne;      // first entry (position in qent) and number of entries
  int32_t tok0, blen;  // the list's KV block: first token and number of keys
  int32_t j;           // kv head
  int32_t n_units;     // units of the list
  int32_t pad[2];
};

struct IndexPtrs {
  int32_t* blk_base;
  int32_t* blk_tok0;
  int32_t* blk_len;
  int32_t* chunk_off;  // [hkv][n_chunks][b_cap]: entries a list receives from the chunks before this one (index_folds: from this one)
  int32_t* cnt;        // [n_lists] list lengths
  int32_t* off;        // [n_lists + 1] exclusive scan of cnt: first position of every list in qent
  int2* qent;        // list entries: (token, column of idx it came from)
  uint32_t* vmask;
  int32_t* slotpos;  // [T, hkv, topk]: position in qent of the entry a kept column produced
  // work units (shared by forward and backward): scanned units per list, and a record per unit in list order
  int32_t* u_nu;
  UnitRec* u_rec;
  int2* group_sum;     // [hkv, n_groups] (entries, work units) of 64 lists (index_folds: not written)
  // dense forward path: query tiles (kTileTokens consecutive tokens of one sequence) and, per (tile, kv head), the
  // 64-key pieces of the KV blocks at least half of the tile's tokens keep, each with the 64-bit mask of the tokens
  // that keep its block
  int32_t *tile_base, *tile_tok0, *tile_len, *tile_seq;
  uint32_t* dmask;     // [T, hkv]: columns of idx the dense path takes over (a subset of vmask)
  int32_t* d_cnt;      // [t_cap, hkv]
  int2* d_piece;       // [t_cap, hkv, kDenseMax] (first key token, number of keys <= 64)
  unsigned long long* d_mask;  // [t_cap, hkv, kDenseMax]
};

inline IndexPtrs index_ptrs(const IndexLayout& L, void* base) {
  char* p = static_cast<char*>(base);
  IndexPtrs r;
  r.blk_base = (int32_t*)(p + L.blk_base);
  r.blk_tok0 = (int32_t*)(p + L.blk_tok0);
  r.blk_len = (int32_t*)(p + L.blk_len);
  r.chunk_off = (int32_t*)(p + L.chunk_off);
  r.cnt = (int32_t*)(p + L.cnt);
  r.off = (int32_t*)(p + L.off);
  r.qent = (int2*)(p + L.qent);
  r.vmask = (uint32_t*)(p + L.vmask);
  r.slotpos = (int32_t*)(p + L.slotpos);
  r.u_nu = (int32_t*)(p + L.u_nu);
  r.u_rec = (UnitRec*)(p + L.u_rec);
  r.group_sum = (int2*)(p + L.group_sum);
  r.tile_base = (int32_t*)(p + L.tile_base);
  r.tile_tok0 = (int32_t*)(p + L.tile_tok0);
  r.tile_len = (int32_t*)(p + L.tile_len);
  r.tile_seq = (int32_t*)(p + L.tile_seq);
  r.dmask = (uint32_t*)(p + L.dmask);
  r.d_cnt = (int32_t*)(p + L.d_cnt);
  r.d_piece = (int2*)(p + L.d_piece);
  r.d_mask = (unsigned long long*)(p + L.d_mask);
  return r;
}

// Problem description handed to the attention kernels.
struct Problem {
  int32_t T, nseq, hq, hkv, g, topk, causal, b_cap, bk;
  int32_t window;    // 0, or: key u is visible to token t only if u > t - window
  uint32_t g_magic;  // floor(2^32 / g) + 1, or 0 when g == 1: row / g as one multiply-high (see div_g)
  int32_t unit;    // list entries per work unit
  int32_t dense;   // 1: the dense forward path is on (the index carries dense flags and tables)
  int32_t t_cap;   // stride of the per-(tile, kv head) dense tables
  int32_t j0, nj;  // KV heads [j0, j0 + nj) handled by this launch (all of them unless the workspace is capped)
  int32_t l0, l1;  // lists [l0, l1): those of the heads, or a range of one head's (see launch_bwd)
  int32_t units_max;  // last index the table of work units has room for
  float scale;
};

// List entries per work unit.  Long inputs use kMaxUnit (splitting lists further only adds dK/dV partial sums); shorter
// ones use smaller units so that the ~512 workgroup slots of the chip each get several and the sink block's list (every
// token) does not become one slot's whole share: the largest power of two <= pairs / 2048, swept on the paper's
// 8K .. 64K grid.  Below 2048 x 256 pairs that would cut lists into many partial sums for nothing, so it stops at 256 -
// unless there would then be fewer than 400 units, or, for units of more than 1024 rows, fewer than 1024: slots that
// would stand idle are worth the partial sums, down to the size at which a unit's fp32 dK/dV sums (2 x 64 rows of 512
// bytes) take the room of its partial dQ rows (unit x g rows of 256 bytes): beyond it the backward workspace would be
// mostly sums.  Measured, forward + backward main + dK/dV reduction: 1024 tokens x 1 kv head, g = 4, top-k 8:
// 73 / 49 / 41 us for units of 256 / 128 / 64; 2048 x 2, g = 4, top-k 16: 79 / 71 / 86; 8192 x 1, g = 8: 297 / 259 for
// 256 / 128; but 4096 x 2, g = 4: 117 / 131 and 16384 x 1, g = 4: 269 / 311.  Blocks of 128 tokens stay at 256: their
// backward has half the workgroup slots, and its sums are twice as large.
// Units of 32 need a top-k of 4: a list of every token must not have more units than the smallest backward workspace has room
// for (see bwd_units_min).
inline int work_unit_entries(int64_t total_pairs, int topk, int g, int bk) {
  int u = bk == kBlock ? (topk < 4 ? 64 : 32) : kMinUnit;
  while (u < kMaxUnit && (u * g < 4 * kBlock || (int64_t)u * 2 * (u < kMinUnit ? 400 : 2048) <= total_pairs) &&
         (u < kMinUnit || (int64_t)u * 2 * 2048 <= total_pairs))
    u *= 2;
  if (bk == kBlock && u == kMinUnit && u * g > 1024 && total_pairs < (int64_t)u * 1024) u /= 2;
  return u;
}

// Whether the inversion walks a packed batch 64 consecutive tokens at a time instead of by query tile, one wavefront each.  By
// tile it has T / 64 + nseq wavefronts and a row of counters (one per block) for every eight of them: while sequences average
// 256 tokens that is at most 1.25 x what the tokens alone need, far beyond it grows with the square of nseq.  The 16 keep
// small batches by tile, where the launch that finds the dense pairs by itself would be felt.  Measured by tile / by token:
// 65536 tokens x 8 kv heads, top-k 16, in 273 sequences 110 / 113 us, in 1024 104 / 102, in 4096 214 / 142 us; 160000
// tokens in 10000 sequences 1128 / 420 us and 938 / 438 MB of index workspace.
inline bool index_by_token(int T, int nseq) { return nseq > 16 + T / 256; }

// Chunks of the inversion: kTilesPerChunk query tiles, or as many times 64 tokens, each.
constexpr int kTilesPerChunk = 8;
inline int index_chunks(int T, int nseq) {
  const int tiles = index_by_token(T, nseq) ? (T + kTileTokens - 1) / kTileTokens : T / kTileTokens + nseq;
  return (tiles + kTilesPerChunk - 1) / kTilesPerChunk;
}
// Whether the scatter sums the histogram's counters by itself instead of a launch before it: while a workgroup reads no more of them
// than a few loads a thread.  Inversion with and without that launch, us: 1000 tokens x 1 kv head 14.3 -> 12.4, 2000 x 2 23.7 -> 21.7, 4096 x 8
// 25.9 -> 24.1 (4680 counters), 8192 x 8 29.2 -> 28.7 (17 544), 8192 x 32 55 -> 65 (70 176).
inline bool index_folds(int T, int nseq, int hkv, int bk) {
  const int64_t chunks = index_chunks(T, nseq), lists = T / bk + nseq;
  return !index_by_token(T, nseq) && hkv * chunks * lists <= (1 << 14) && chunks <= 32 && lists <= 1024;
}

// Whether the library's choice of forward is the one of short inputs (k_fwd_short), which computes every (row group, 64 keys) pair that any
// of the group's tokens keeps: by x, the blocks of the whole input for every column (twice that where nothing hides the later ones).
// A packed batch counts as one sequence: its rows see fewer blocks than that.  Measured, whole forward with the inversion, gather or dense
// route -> short, us; 64-token blocks, causal, x = 2 / 3 / 4 / 6: 4 heads, g = 4 44 -> 40, 55 -> 50, 59 -> 60, 78 -> 123; 8 heads, g = 4 58 -> 42,
// 79 -> 73, 90 -> 97, 126 -> 144; 32 heads, g = 4 139 -> 81, 179 -> 131, 235 -> 198, 342 -> 361 (top-k 16, 2000, 3000, 4096 and 6000 tokens); top-k 8,
// 2000 tokens (x = 4) 4 heads 31 -> 35, 32 heads 90 -> 71.  All keys, x = 4 / 6 / 8: 4 heads 45 -> 40, 56 -> 52, 65 -> 73; 32 heads 159 -> 99, 233
// -> 183, 281 -> 293.  Blocks of 128 tokens, of which the other routes gather half as many: x = 1 / 2 / 3, 8 heads 38 -> 24, 45 -> 36, 51 -> 67; 4 heads,
// g = 1, 31 -> 35 at x = 2.  (k_fwd_short takes 2 to 6 % longer since it rescales for every piece; 184 inputs drawn inside the rule took 16 % less and more
// than by the other routes with either.)
inline bool short_forward(int T, int nseq, int hq, int topk, int bk, bool causal, int window) {
  if (T > 8192 || nseq > 64 || index_by_token(T, nseq)) return false;  // what k_fwd_short has room for
  const int64_t rows = (int64_t)T * hq, blocks = (int64_t)(window > 0 && window < T ? window : T) * (causal ? 1 : 2);
  const int64_t x10 = bk == kBlock ? (!causal ? 60 : rows >= 50000 ? 42 : 30) : (rows >= (1 << 14) ? 20 : 10);
  return blocks * 10 <= x10 * topk * bk;
}

// Upper bound of the work units of nj KV heads (one per non-empty list plus one per full unit of entries); the
// real count is only known on the device.  It is never reached, and the backward keeps its queue of units in the room of the last
// one's sums (see UnitQueue).
inline int64_t units_bound(int nj, int b_cap, int T, int topk, int unit) {
  return (int64_t)nj * b_cap + (int64_t)nj * T * topk / unit + 1;
}

// Whether the forward main kernels take the first units of all `heads` KV heads of a pass, then the second ones and so on, instead of
// head by head.  Causal, a head's first lists are its longest (the sink's, then the early blocks'), and those of the last head would
// otherwise start last: at 8192 tokens x 32 heads, g = 1, they ran alone for a seventh of the kernel.  Against that, head by head every XCD
// has one head's Q in its L2; in turn it has that of the heads whose workgroups it is dealt, few where their number is a multiple of eight
// and all of them where it is odd.  Measured head by head -> in turn, us (top-k 16, tokens x KV heads):
//   g = 1   8192 x 32 with a sink 331 -> 309, without one 339 -> 297; 16000 x 16 316 -> 322; 30000 x 8 282 -> 293
//           all keys: 4096 x 16 95 -> 90, 8192 x 16 155 -> 156, x 24 229 -> 225, x 32 311 -> 325, 4096 x 64 304 -> 322
//           other numbers of heads: 8192 x 20 186 -> 184, 26360 x 5 152 -> 166, 6660 x 31 226 -> 264, 5843 x 30, all keys, 198 -> 235
//   g = 2   8192 x 32 480 -> 432, 9000 x 24 -8 %, 11000 x 16 -5 %, 16000 x 16 507 -> 537, 16384 x 8 -9 %, 28000 x 8 +2 %, 24000 x 4 -6 %
//           all keys: 16384 x 8 -8 %, 14500 x 16 +6 %; other numbers: 8849 x 21 298 -> 338, 24815 x 6 279 -> 302
//   g >= 4  8192 x 16 444 -> 354, g = 5, 12000 x 8 419 -> 347, g = 7, 16000 x 4 412 -> 386, 12729 x 6 274 -> 260, 34739 x 2 286 -> 262, 65536 x 2
//           526 -> 568; all keys: 16384 x 8 574 -> 562, 7887 x 10 333 -> 379, 5688 x 12 368 -> 390; other numbers: 6523 x 19 +4 %, 6416 x 14 +4 %, 4323 x 15 194 -> 225
//   128-token blocks, of which a head has half as many: g = 1, 8192 x 32 251 -> 230, x 28 232 -> 234; g = 2, 16384 x 8 198 -> 181, 4920 x 41
//           212 -> 190, 28000 x 8 +1 %; g = 4, 8192 x 16 264 -> 238, 6667 x 13 88 -> 81, 10936 x 11 301 -> 282; all keys: 7708 x 19 225 -> 233
inline bool units_in_turn(int T, int heads, int hq, int g, int bk, bool causal) {
  const bool even = heads % (g == 1 || !causal ? 8 : 4) == 0 || (g >= 2 && heads == 4) || (causal && g >= 4 && (heads == 2 || heads == 6)) ||
                    (causal && g >= 2 && bk == 2 * kBlock && T <= 24576);
  const int64_t rows = (int64_t)T * hq, near = (int64_t)(g < 4 ? g : 4) << 17;
  return even && T <= 40960 && (rows <= near || (causal && T <= 12288 && rows <= min(2 * near, (int64_t)1 << 19)));
}

// Work units whose dK/dV sums the smallest backward workspace holds: those of one KV head at units of at least kMinUnit.  The
// smaller units of tiny inputs have more; where they do not fit, the backward goes through the head's lists in ranges.  One
// list always fits: it has at most ceil(T / unit) units, and that is no more than the blocks of T tokens (units of 64 and
// 128) or, for units of 32, the blocks and T topk / 256.
inline int64_t bwd_units_min(int b_cap, int T, int topk, int unit) {
  return units_bound(1, b_cap, T, topk, unit < kMinUnit ? kMinUnit : unit);
}

// ---- optional per-kernel timing (off unless nsa_sel_profile_enable was called) ---------------------------
enum KernelId {
  KID_INDEX_PREP = 0, KID_INDEX_HIST, KID_INDEX_DENSE, KID_INDEX_SCAN, KID_INDEX_SCATTER, KID_FWD_MAIN, KID_FWD_MERGE,
  KID_FWD_DENSE, KID_FWD_SHORT, KID_FWD_QUERY_OUTER, KID_BWD_DELTA, KID_BWD_MAIN, KID_BWD_DQ_REDUCE, KID_BWD_DKV_REDUCE, KID_SELECT_BLOCKS,
  KID_COUNT
};
// Records a HIP event on `st` at construction and destruction when profiling is on; does nothing otherwise.
struct ProfScope {
  int slot;
  hipStream_t st;
  ProfScope(int kid, hipStream_t stream);
  ~ProfScope();
};

// Raises a kernel's dynamic-LDS limit to `bytes`, once per device (`done` holds one bit per device id), so that
// later launches - also those recorded into a HIP graph - make no attribute call at all.
inline hipError_t allow_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// Optional gated combination with the other attention branches (Eq. (2)); all null for the plain entry points.
struct GateArgs {
  const float* gate;  // [T, hq]
  const void* o_acc;  // bf16 [T, hq, d] or null
  void* o_out;        // bf16 [T, hq, d]
  float* dgate;       // [T, hq] (backward)
};

// ---- launchers (each enqueues on `st` and returns hipGetLastError()) -------------------------------------
hipError_t launch_build_index(const IndexLayout& L, const int32_t* idx, const int32_t* cu, void* index_ws,
                              hipStream_t st);
// heads_per_pass: KV heads whose partial results the workspace can hold at once (1 .. hkv)
hipError_t launch_fwd(const Problem& P, const IndexLayout& L, int heads_per_pass, const void* Q, const void* K,
                      const void* V, const void* index_ws, void* opart, float* lse_part, void* O, float* LSE,
                      const GateArgs& G, hipStream_t st);
// the forward of short inputs, with (build) the index; without, it reads the one that is there (see short.hip)
hipError_t launch_fwd_short(const Problem& P, const IndexLayout& L, bool build, const void* Q, const void* K, const void* V,
                            const int32_t* idx, const int32_t* cu, void* index_ws, void* O, float* LSE, const GateArgs& G,
                            hipStream_t st);
// the same forward in query-outer loop order (no workspaces, no index): see qouter.hip
hipError_t launch_fwd_query_outer(const Problem& P, const void* Q, const void* K, const void* V, const int32_t* idx,
                                  const int32_t* cu, void* O, float* LSE, hipStream_t st);
// lists_per_pass: lists of a KV head whose dK/dV sums the workspace can hold at once (only with one head per pass; 0: all)
hipError_t launch_bwd(const Problem& P, const IndexLayout& L, int heads_per_pass, int lists_per_pass, const void* Q,
                      const void* K, const void* V, const void* O, const float* LSE, const void* dO, const void* index_ws,
                      void* dqpart, float* delta, float* dkv_part, void* dQ, void* dK, void* dV, const GateArgs& G,
                      hipStream_t st);

// ---- device helpers ------------------------------------------------------------------------------------
#if defined(__HIPCC__)
typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // 16 bytes in flight as a plain vector (rows being gathered)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// r / g for 0 <= r < 2^20 and g in [1, 8] without an integer division: the error of the rounded-up reciprocal,
// r (magic - 2^32 / g) < r, stays far below 2^32 / g, so the high word of the product is the exact quotient.
// g = 1 has no 32-bit reciprocal; its magic is 0 and r is added instead (a select, not a branch).
__device__ __forceinline__ int div_g(int r, int g, uint32_t g_magic) {
  return (int)(((uint64_t)(uint32_t)r * g_magic) >> 32) + (g == 1 ? r : 0);
}

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __builtin_bit_cast(float, u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __builtin_bit_cast(float, u & 0xffff0000u); }

// 16-byte accesses with the non-temporal hint.
__device__ __forceinline__ u32x4 load_streaming(const bf16_t* src) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src));
}
__device__ __forceinline__ void store_streaming(bf16_t* dst, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
}

// ---- rows of 256 bytes through buffer instructions ------------------------------------------------------
// A tile's rows are moved with raw buffer loads and stores: base in scalar registers, 32-bit offset per lane, and an access
// past the end of the buffer is dropped by the hardware.  That last point matters most: the accesses need no branch
// (rows past the end of a list are given kNoRow), so the compiler knows exactly how many are outstanding and a wait
// for the loads of the next tile does not also wait for the stores of this one.
constexpr uint32_t kNoRow = 1u << 30;  // byte offset past the end of every buffer it is used with
constexpr int kNonTemporal = 2;           // cache policy bit of the buffer instructions

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// N dropped stores.  In front of a loop whose iterations issue loads first and N stores later they make both ways into the
// loop agree on what is outstanding, so that the wait for the loads at its top leaves the last iteration's stores in flight.
template <int N>
__device__ __forceinline__ void pad_stores(__amdgpu_buffer_rsrc_t b) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) __builtin_amdgcn_raw_buffer_store_b32(0u, b, kNoRow + 16 * i, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
}

// Value of `v` in lane `src` (any lane of the wavefront).
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int src) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)v);
}

// The rows of one kv head's block of K or V: rows past the end of a ragged block read as zero.  Row r at r * row_bytes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t block_buffer(const bf16_t* x, const Problem& P, const UnitRec& U) {
  return buffer_of(x + ((size_t)U.tok0 * P.hkv + U.j) * kD, (uint32_t)((U.blen - 1) * P.hkv + 1) * (kD * 2));
}
__device__ __forceinline__ bf16x8 load_frag(__amdgpu_buffer_rsrc_t b, uint32_t off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
}

// The unit of this workgroup of a main kernel, or false when the launch (sized by an upper bound) has no unit left
// for it.  By number, the record is requested before the unit count is known: the two loads are independent and every
// index up to the bound is allocated.  With the heads in turn (the forward's, see units_in_turn) consecutive workgroups take the same place among the
// units of each of the pass's heads, and the launch has room for as many units as one head can have, for each.
// pos0 = the first list position of the pass's KV heads (partial rows are relative to it).
template <bool kInTurn>
__device__ __forceinline__ bool load_unit(const Problem& P, const UnitRec* __restrict__ u_rec,
                                          const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ off,
                                          UnitRec& U, int& pos0) {
  pos0 = P.j0 > 0 ? off[P.j0 * P.b_cap] : 0;
  int u, end;
  if constexpr (kInTurn) {
    const int i = (int)(blockIdx.x / (unsigned)P.nj), l = (P.j0 + (int)blockIdx.x - i * P.nj) * P.b_cap;
    u = nu_scan[l] + i;
    end = nu_scan[l + P.b_cap];
  } else {
    u = (P.l0 > 0 ? nu_scan[P.l0] : 0) + (int)blockIdx.x;
    end = nu_scan[P.l1];
  }
  const int ur = min(u, P.units_max);
  const int4 a = *reinterpret_cast<const int4*>(u_rec + ur);
  const int2 b = *reinterpret_cast<const int2*>(&u_rec[ur].j);
  U.e0 = a.x; U.ne = a.y; U.tok0 = a.z; U.blen = a.w; U.j = b.x; U.n_units = b.y;
  asm volatile("" : "+s"(U.e0), "+s"(U.ne), "+s"(U.tok0), "+s"(U.blen), "+s"(U.j), "+s"(U.n_units));  // requested here
  return u < end;
}

// LDS by 32-bit address.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)(uint32_t)(uintptr_t)p;
}
__device__ __forceinline__ bf16x8 lds_read_frag(uint32_t a) {
  return *(__attribute__((address_space(3))) const bf16x8*)a;
}
__device__ __forceinline__ u32x4 lds_read_16(uint32_t a) { return *(__attribute__((address_space(3))) const u32x4*)a; }
__device__ __forceinline__ void lds_write_16(uint32_t a, u32x4 v) { *(__attribute__((address_space(3))) u32x4*)a = v; }
__device__ __forceinline__ void lds_write_8(uint32_t a, uint2 v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  *(__attribute__((address_space(3))) u32x2*)a = u32x2{v.x, v.y};
}
// Rows of 128 bf16 lie in LDS unpadded, the 16-byte chunk c of row r at place c ^ row_turn(r).  That spreads over all 64 banks both
// shapes in which the matrix operands are read: 16 bytes of one chunk in 16 consecutive rows (the low four bits of r all count),
// and the transposing read, which takes four consecutive rows x 64 bytes in a cycle (their two low bits select the quarter of the
// row).  Measured per CU: 256 bytes a clock for the former and twice the 128 of a 304-byte pitch for the latter, for which no
// padding serves both (64 at 256 + 16, 64 with c ^ (r & 15)).  Where rows of a read differ by multiples of 16, its places differ by
// an immediate offset; other steps flip bits of the address.
__device__ __forceinline__ int row_turn(int r) { return (r & 3) << 2 | ((r >> 2) & 3); }
// ds_read_b64_tr_b16: every lane passes the address of 8 bytes (four 16-bit elements); within each group of 16 lanes, lane
// i receives element (i % 4) of the 8 bytes addressed by lanes 4e + i / 4, e = 0..3.  With lane s of a group pointing at row
// (s / 4), columns 4 (s % 4).. of a row-major tile, lane i gets column i of four consecutive rows: the MFMA operand layout
// (lane = column, elements = rows) without a transposed copy.
__device__ __forceinline__ bf16x4 lds_read_tr_at(uint32_t a) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
  return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)a));
}
__device__ __forceinline__ bf16x4 lds_read_tr(const bf16_t* p) { return lds_read_tr_at((uint32_t)(uintptr_t)p); }

// 16 bytes per lane from memory straight to LDS: lane l's, from byte `off` of the buffer, go to lds + 16 l (lds is
// wave-uniform); lanes past the end of the buffer get zero.  The whole offset is per lane: the instruction's scalar offset is
// left out of the bounds check, or taken off the buffer's size before it, so a row step put there could read past the end.
// The bytes are there once the wavefront's wait_loads() and, for other wavefronts, a barrier
// after it have passed.  Written as assembly because the compiler would make every LDS read after it wait for it, also
// reads of another tile: the double use of one tile set rests on the reads being ordered by the barriers alone.
// The load takes its LDS address from m0 and needs a wait state after the scalar write of m0; inside an assembly block the
// compiler inserts none, hence the s_nop.
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t b, uint32_t lds, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds), "v"(off), "s"(b) : "memory", "m0");
}
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A gathered bf16 [rows, 128] tensor.  kWide: 4 GB or more, which a 32-bit offset does not reach.
template <bool kWide>
struct RowTensor {
  const char* base;
  uint32_t bytes;
  __device__ __forceinline__ RowTensor(const void* p, int64_t rows)
      : base(static_cast<const char*>(p)), bytes(kWide ? 0u : (uint32_t)(rows * (kD * 2))) {}
  __device__ __forceinline__ u32x4 load(uint32_t row, uint32_t lane_off) const {
    if constexpr (kWide)
      return *reinterpret_cast<const u32x4*>(base + ((size_t)row * (kD * 2) + lane_off));
    else
      return __builtin_amdgcn_raw_buffer_load_b128(buffer_of(base, bytes), row * (kD * 2) + lane_off, 0, 0);
  }
};
inline bool rows_are_wide(int64_t rows) { return rows * (kD * 2) >= ((int64_t)1 << 32) - 65536; }

// ---- the two reduction kernels ---------------------------------------------------------------------------
// k_fwd_merge and k_bwd_dq_reduce read sixteen rows for every row they write, and what bounds them is the memory side: a kernel that
// only gathers these rows reads 7.0 TB/s with non-temporal loads (6.2 with plain ones), and the sixteenth of writes takes it
// down to 5.4 when they are strewn among the reads, to 5.7 as non-temporal stores, and to 6.4 when a workgroup keeps 128 KB of results
// and writes them at once.  So a workgroup parks its rows in LDS and writes them after its last gather: dQ reduction at
// 65536 tokens, g = 4: 1.72 -> 1.50 ms, at 8192, g = 1: 222 -> 182 us; merge there 233 -> 207 us.  Small inputs, and sequences too
// short for their rows to have most columns, leave a burst little to read between its writes and take 16 rows a workgroup instead,
// written as they are done: merge_in_bursts and dq_in_bursts say where either is faster.
// Rows of a pass are (token, head of its KV heads), token-major.  A workgroup of kThreads threads takes at most kRows steps of
// kThreads / 16 consecutive ones, 16 lanes a row, and every XCD (they get workgroups in turn) works through one contiguous eighth of
// them, so that its L2 keeps the lines of log-sum-exps that neighbouring tokens share.  The LDS holds one burst workgroup a compute
// unit: up to four turns of all 256 of them the steps are spread evenly, so that no turn is nearly empty (16875 tokens, 16 heads: merge 256
// -> 224 us, dQ reduction 222 -> 205; 25000: 348 -> 315, 314 -> 285); beyond that full workgroups are as fast or up to 5 % faster.
struct ReduceSpan {
  uint32_t first;  // of the workgroup's steps, kThreads / 16 consecutive rows each
  int count;       // at most kRows
};
template <int kRows, int kThreads>
__device__ __forceinline__ ReduceSpan reduce_span(const Problem& P, uint32_t group, uint32_t groups) {
  constexpr uint32_t kStep = kThreads / 16;
  const uint32_t steps = ((uint32_t)P.T * (uint32_t)(P.nj * P.g) + kStep - 1) / kStep;  // total_tokens * hq < 2^31 is checked on the host
  const uint32_t blk = (group & 7) * (groups >> 3) + (group >> 3);
  if constexpr (kRows == 1) return {blk, blk < steps ? 1 : 0};
  const uint32_t each = steps / groups, more = steps - each * groups;
  return {blk * each + min(blk, more), (int)(each + (blk < more ? 1 : 0))};
}
struct ReduceRow {
  int t, j, hh;   // token, KV head, head of the group; rows past the last one repeat it
  bool on;
};
template <int kThreads>
__device__ __forceinline__ ReduceRow reduce_row(const Problem& P, uint32_t step) {
  const uint32_t hp = (uint32_t)(P.nj * P.g), rows = (uint32_t)P.T * hp;
  const uint32_t r = step * (kThreads / 16) + (threadIdx.x >> 4), rc = min(r, rows - 1);
  ReduceRow x;
  x.t = (int)(rc / hp);
  const int h = (int)(rc - (uint32_t)x.t * hp);
  x.j = h / P.g;
  x.hh = h - x.j * P.g;
  x.j += P.j0;
  x.on = r < rows;
  return x;
}
// Positions of the row's columns in the partial rows (-1: not kept, or past the last column): lane sub of the 16 holds columns
// sub and 16 + sub.
struct SlotRow {
  int lo, hi;
};
__device__ __forceinline__ SlotRow load_slots(const int32_t* __restrict__ slotpos, const Problem& P, const ReduceRow& R) {
  const int32_t* sp = slotpos + ((size_t)R.t * P.hkv + R.j) * P.topk;
  const int sub = threadIdx.x & 15;
  SlotRow s;
  s.lo = sp[min(sub, P.topk - 1)];
  s.hi = P.topk > 16 ? sp[min(16 + sub, P.topk - 1)] : -1;
  if (sub >= P.topk) s.lo = -1;
  if (16 + sub >= P.topk) s.hi = -1;
  return s;
}
__device__ __forceinline__ int slot_of(const SlotRow& s, int m0, int i) {  // of column m0 + i: m0 a wave-uniform multiple of 8, i < 8
  return (int)lane_value((uint32_t)(m0 < 16 ? s.lo : s.hi), (int)(threadIdx.x & 48) + (m0 & 8) + i);
}
// The kept columns of a wavefront's four rows, 16 bits a row.  Columns are gathered eight at a time.  In bursts, which serve
// sequences long enough that nearly all rows keep all columns, a dropped column requests the kept one before it again, without
// a branch.  One row at a time, batches of which no row keeps anything are skipped and dropped columns request nothing; batches
// that all four rows keep whole go without branches.  6762 tokens in 23 sequences, 16 heads, g = 1, top-k 16, merge / dQ
// reduction: 58 / 51 us as in the bursts, now 39 / 36.  (In the bursts of long sequences the second way costs up to 8 %.)
struct KeptColumns {
  uint64_t lo, hi;
  __device__ __forceinline__ explicit KeptColumns(const SlotRow& s)
      : lo(__builtin_amdgcn_ballot_w64(s.lo >= 0)), hi(__builtin_amdgcn_ballot_w64(s.hi >= 0)) {}
  __device__ __forceinline__ bool none() const { return (((lo | hi) >> (threadIdx.x & 48)) & 0xffffu) == 0; }  // of this lane's row
  static constexpr uint64_t kAll = 0x00ff00ff00ff00ffull;
  __device__ __forceinline__ uint64_t eight_from(int m) const { return ((m < 16 ? lo : hi) >> (m & 8)) & kAll; }  // m a multiple of 8
};
constexpr int kBurstThreads = 1024, kBurstRows = 8, kBurstRowsGated = 4;  // gated: two tensors share the LDS
inline bool reduce_in_bursts(const Problem& P, int64_t rows, int64_t tokens) {  // at least: rows of the pass, mean length of a sequence
  return (int64_t)P.T * P.nj * P.g >= rows && P.T >= tokens * P.nseq;
}
// The merge: by what it reads, rows * top-k; gated it has two tensors to write and half the rows a workgroup.  (one row at a time ->
// bursts, us; 16 heads, g = 1: top-k 16 8192 tokens 109 -> 109, 12500 169 -> 168, 16384 224 -> 208; top-k 8 25000 tokens 175 -> 185, 33080
// 252 -> 240; gated, top-k 16 25000 376 -> 396, 33080 523 -> 490; top-k 5 and 6 62500 286 -> 334 and 334 -> 357.)  Sequences of 870 / 1440 /
// 2030 tokens in the mean, 35000 in all: top-k 8 220 -> 230 / 223 -> 229 / 244 -> 239, top-k 16 377 -> 390 / 381 -> 399 / 451 -> 429, top-k
// 32 594 -> 656 / 609 -> 689 / 784 -> 772.
inline bool merge_in_bursts(const Problem& P, bool gated) {
  return P.topk >= 8 && reduce_in_bursts(P, (gated ? 1 << 23 : 1 << 22) / P.topk, 1536);
}
// The dQ reduction: a row of the sum is half the work of a merged one.  (16 heads, g = 1, top-k 16: 5600 tokens 69 -> 68, 8192 101 -> 92, 12500
// 159 -> 140; top-k 8 8192 tokens 56 -> 54; top-k 6 25000 tokens 133 -> 138, 37500 200 -> 192; top-k 5 25000 tokens 113 -> 129, 62500 282 -> 291.)
// Sequences of 470 / 670 / 870 tokens: top-k 8 165 -> 173 / 196 -> 188 / 212 -> 200, top-k 16 221 -> 273 / 307 -> 297 / 347 -> 322; of 670 / 870 /
// 2030 tokens: top-k 32 418 -> 497 / 542 -> 538 / 722 -> 651.
inline bool dq_in_bursts(const Problem& P) {
  return P.topk >= 6 && reduce_in_bursts(P, P.topk >= 8 ? 1 << 17 : 1 << 19, (int64_t)P.topk * P.bk * 5 / 8);
}
// LDS of a workgroup: 16 bytes a thread and row for every tensor written, and a float a row for LSE.
constexpr int reduce_lds(int threads, int rows, int tensors, bool lse) { return rows * threads * (16 * tensors) + (lse ? rows * threads / 4 : 0); }
template <int kRows, int kThreads>
inline unsigned reduce_groups(const Problem& P) {
  constexpr int64_t kStep = kThreads / 16, kTurn = kRows == 1 ? 8 : 256;
  const int64_t steps = ((int64_t)P.T * P.nj * P.g + kStep - 1) / kStep, turns = (steps + kTurn * kRows - 1) / (kTurn * kRows);
  return (unsigned)(kRows == 1 || turns <= 4 ? turns * kTurn : ((steps + kRows - 1) / kRows + 7) / 8 * 8);
}

// Sequence bounds of token t in a packed batch (cu may be null for a single sequence).
__device__ __forceinline__ void seq_bounds(const int32_t* cu, int nseq, int T, int t, int& s, int& c0, int& c1) {
  if (cu == nullptr || nseq == 1) {
    s = 0;
    c0 = 0;
    c1 = T;
    return;
  }
  int lo = 0, hi = nseq;  // invariant: cu[lo] <= t < cu[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (cu[mid] <= t) lo = mid; else hi = mid;
  }
  s = lo;
  c0 = cu[lo];
  c1 = cu[lo + 1];
}
#endif

}  // namespace nsa
