// Block selection in front of the attention path: per (token, KV head) the forced sink / most-recent blocks and
// then the visible blocks with the highest scores (see nsa_sel_select_blocks in nsa_sel.h for the rule).
//
// One wavefront takes a row at a time and looks at it in chunks of up to 1024 blocks, 16 scores per lane held in registers.  The fast method (select_by_threshold) bounds the picks from below with the
// r-th largest lane maximum, compacts the few elements above that bound into the LDS and ranks them against each
// other: ~530 instructions per row.  Rows where too many scores agree in the bound's bits fall back to the general method
// (select_by_rounds): one pick per round, each round two wave-wide reductions.  Each visible score is read from
// HBM once, with 16-byte loads when the rows are 16-byte aligned.
#include "common.h"

namespace nsa {
namespace {

constexpr int kSelWaves = 4;                  // wavefronts per workgroup
// Rows of a wavefront: one, or eight in a loop.  The kernel is bound by the instructions a row takes (270 vector, 260 scalar; a
// compute unit issues one scalar instruction a clock for its four SIMDs), and a token's bounds and the row's divisions are a fifth of
// the scalar ones: eight rows share them where a token has several heads.  Against that the loop keeps more alive than the scalar
// registers hold, and eight rows in turn need more rows before every SIMD has wavefronts enough.  Measured, one -> eight, 64 ..
// 1024 blocks, causal: 8 heads 65536 rows 36.8 .. 40.2 -> 40.6 .. 39.5 us, 131072 rows 74.8 .. 78.2 -> 77.9 .. 74.0, 524288 rows 296 ..
// 385 -> 291 .. 340; 2 heads 65536 rows 38.2 .. 42.6 -> 44.8 .. 48.5, 131072 rows 76.2 .. 94.2 -> 84.2 .. 96.0, 262144 rows 150 ..
// 210 -> 158 .. 200; one head 131072 rows 76.8 .. 105.9 -> 89.3 .. 113.8, 524288 rows 299 .. 446 -> 328 .. 430.  16 rows cost
// 3 % against eight, ending the bound's search early by a branch or requesting the next row ahead (16 more registers
// and moves) 20 %.
constexpr uint32_t kSelRows = 8;
inline bool eight_rows(int64_t rows, int hkv) { return rows >= (hkv > 1 ? 1 << 17 : 1 << 19); }
constexpr int kChunkBlocks = 1024;            // blocks examined at a time: 16 keys per lane
constexpr int kKeys = kChunkBlocks / 64;
constexpr int kMaxChunks = 16;                // rows of up to 16384 blocks
constexpr int kCandPerLane = kMaxChunks * kMaxTopk / 64;   // chunk picks each lane holds in the final selection
// The bound is searched on the upper 16 bits of the keys: sign, exponent and 7 bits of the score.  Two bits of it, a grid of a quarter
// octave, let everything within 25 % of the bound survive, and ordinary scores of a narrower range than exp(1.5 z) outgrew the list of
// survivors: exp(0.1 z) took 1470 us at 65536 tokens x 8 heads x 1024 blocks instead of 344, uniform ones 592 instead of 343.
constexpr int kTauLowBit = 16;
// Survivors the fast method ranks; rows with more take the general one.  A chunk in which fewer than r lanes hold a score, r <= 35,
// keeps all of its up to 136 without a search, after what the chunks before it left: with room for 128 all rows of 129 to 136 blocks
// (top-k 32, all keys) took the general method, 3540 us for 65536 tokens x 8 heads.
constexpr int kMaxSurv = 256;

// All four steps stay inside a row of 16 lanes (quad swaps, then mirrors of 8 and of 16 lanes), after which every
// lane of a row holds the row's result; the four rows are combined on the scalar unit.
template <bool kMax>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v) {
  auto comb = [](uint32_t a, uint32_t b) { return kMax ? (a > b ? a : b) : (a < b ? a : b); };
  v = comb(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));   // lanes ^ 1
  v = comb(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));   // lanes ^ 2
  v = comb(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));  // mirror of 8
  v = comb(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));  // mirror of 16
  const uint32_t a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
  return comb(comb(a, b), comb(c, d));
}

// fp32 bits -> unsigned key with the same order as the values; NaN ranks with -infinity, -0 with +0, and every
// key is > 0 so that 0 can mean "no candidate".
__device__ __forceinline__ uint32_t order_key(uint32_t u) {
  if ((u & 0x7fffffffu) > 0x7f800000u) u = 0xff800000u;   // NaN -> -inf
  if (u == 0x80000000u) u = 0u;                            // -0 -> +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Picks up to `want` candidates in descending (key, then ascending block) order.  key[e] belongs to block
// blk_of(e), which must ascend with e inside a lane; ne bounds the e that can hold candidates (wave-uniform).
// emit(i, block, key) is called wave-uniformly for the i-th pick.  Returns the number of picks.
template <int E, class BlkOf, class Emit>
__device__ __forceinline__ int pick_rounds(uint32_t (&key)[E], int ne, int want, BlkOf blk_of, Emit emit) {
  int got = 0;
  for (; got < want; ++got) {
    uint32_t best = 0, bblk = 0x7fffffffu;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (e < ne) {
        const bool up = key[e] > best;      // strict: of equal keys the lane keeps its smallest block
        best = up ? key[e] : best;
        bblk = up ? (uint32_t)blk_of(e) : bblk;
      }
    }
    const uint32_t m = wave_reduce<true>(best);
    if (m == 0) break;                      // no candidate left
    const uint32_t wb = wave_reduce<false>(best == m ? bblk : 0x7fffffffu);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (e < ne) key[e] = ((uint32_t)blk_of(e) == wb) ? 0u : key[e];   // block ids are unique: clears the winner only
    }
    emit(got, (int)wb, m);
  }
  return got;
}

// What one row needs to know about itself.
struct RowInfo {
  const float* srow;  // the row's scores
  int b_vis;          // visible blocks are [0, b_vis)
  int ns;             // forced sinks are [0, ns)
  int nl, loc_lo, loc_hi;   // forced local blocks are [loc_lo, loc_hi] when nl > 0
  int n_forced;       // columns taken by forced blocks
  int want;           // columns to fill by score
  __device__ __forceinline__ bool forced(int b) const { return b < ns || (nl > 0 && b >= loc_lo && b <= loc_hi); }
};

// Block of element e of a lane in the chunk that starts at `base`: four consecutive blocks per 16-byte load, or
// one block per 4-byte load.  Ascends with e inside a lane in both layouts.
template <bool kVec>
__device__ __forceinline__ int blk_of(int base, int lane, int e) {
  return kVec ? base + ((e >> 2) << 8) + (lane << 2) + (e & 3) : base + (e << 6) + lane;
}

// Raw score bits of E elements per lane; what lies at or past b_vis in a lane's FIRST element is not loaded and
// reads as `fill` (a 16-byte load may bring up to three blocks past b_vis along; callers deal with those).
template <bool kVec, int E>
__device__ __forceinline__ void load_bits(const RowInfo& R, int base, int lane, uint32_t fill, uint32_t (&x)[E]) {
  if (kVec) {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      const int b = base + (q << 8) + (lane << 2);
      u32x4 v = {fill, fill, fill, fill};
      if (b < R.b_vis) v = *reinterpret_cast<const u32x4*>(R.srow + b);   // b + 3 < stride: both multiples of 4
#pragma unroll
      for (int i = 0; i < 4; ++i) x[q * 4 + i] = v[i];
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int b = base + (e << 6) + lane;
      x[e] = b < R.b_vis ? __builtin_bit_cast(uint32_t, R.srow[b]) : fill;
    }
  }
}

// What lies in a wavefront's LDS is written and read as 32-bit words by all methods.  An entry of the survivor list is the pair
// (score bits or key, ~block), in the order in which its two words compare as one number.
struct alignas(8) Survivor {
  uint32_t not_blk, score;
  __device__ __forceinline__ uint64_t both() const { return (uint64_t)score << 32 | not_blk; }
};

// Orders a wavefront's own LDS traffic: what its lanes wrote before is what any of them reads after, and the other way round.
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- the general method: `want` rounds of "take the largest remaining key".  Exact for any input, also when
// most scores are equal; ~150 instructions per pick, so it only serves rows the fast method hands over.
template <bool kVec>
__device__ __forceinline__ int select_by_rounds(const RowInfo& R, int lane, uint32_t* lds_wave, int mine) {
  uint32_t* cand_key = lds_wave;
  int32_t* cand_blk = reinterpret_cast<int32_t*>(lds_wave + kMaxChunks * kMaxTopk);
  const int n_chunks = (R.b_vis + kChunkBlocks - 1) / kChunkBlocks;
  int n_cand = 0;                          // chunk picks parked in the LDS (only when n_chunks > 1)
  for (int c = 0; c < n_chunks; ++c) {
    const int base = c * kChunkBlocks;
    const int left = R.b_vis - base;       // > 0
    const int ne = left >= kChunkBlocks ? kKeys : (kVec ? ((left + 255) >> 8) << 2 : (left + 63) >> 6);
    uint32_t key[kKeys];
    load_bits<kVec, kKeys>(R, base, lane, 0u, key);
#pragma unroll
    for (int e = 0; e < kKeys; ++e) {
      const int b = blk_of<kVec>(base, lane, e);
      key[e] = (b < R.b_vis && !R.forced(b)) ? order_key(key[e]) : 0u;
    }
    auto blk = [&](int e) { return blk_of<kVec>(base, lane, e); };
    if (n_chunks == 1) {
      pick_rounds<kKeys>(key, ne, R.want, blk, [&](int i, int b, uint32_t) {
        if (lane == R.n_forced + i) mine = b;
      });
    } else {
      const int got = pick_rounds<kKeys>(key, ne, R.want, blk, [&](int i, int b, uint32_t k) {
        if (lane == 0) {
          cand_key[n_cand + i] = k;
          cand_blk[n_cand + i] = b;
        }
      });
      n_cand += got;
    }
  }
  if (n_chunks > 1) {
    // final selection over the chunk picks (written by lane 0 of this wavefront, read by all of its lanes)
    wave_sync_lds();
    uint32_t key[kCandPerLane];
    int32_t blk[kCandPerLane];
#pragma unroll
    for (int e = 0; e < kCandPerLane; ++e) {
      const int q = (e << 6) + lane;
      key[e] = q < n_cand ? cand_key[q] : 0u;
      blk[e] = q < n_cand ? cand_blk[q] : 0x7fffffff;
    }
    // within a lane the candidates of later chunks have larger block ids, so blocks ascend with e as required
    pick_rounds<kCandPerLane>(key, (n_cand + 63) >> 6, R.want, [&](int e) { return blk[e]; },
                              [&](int i, int b, uint32_t) {
                                if (lane == R.n_forced + i) mine = b;
                              });
  }
  return mine;
}

// ---- the fast method.  Per chunk of up to 1024 blocks:
//   1. every lane takes the largest of its scores; tau = the r-th largest of the 64 lane maxima, found bit by bit
//      with ballots (scalar work).  r = want + (forced blocks) + 3, so at least `want` selectable blocks of the
//      chunk have a score >= tau (forced blocks and the up to three blocks a 16-byte load brings along past b_vis
//      are not masked beforehand: they are dropped in step 3), hence no block with a score < tau can be a pick;
//   2. the elements not below tau ("survivors", a few more than r unless many scores agree in the bits of tau) are compacted into
//      an LDS list of (score, ~block) pairs;
//   3. after all chunks the survivors' scores become order-preserving keys and every survivor counts the survivors that beat
//      it; that rank is its output column.
// The scores are compared as floats up to step 3, so that only the 64 maxima and the survivors are turned into keys.  A lane's
// maximum leaves out its NaNs (or reads as -inf for one, which only lowers the bound), and a NaN survives only where -inf does;
// -0 equals +0.  chunk_survivors does steps 1 and 2; n_surv above kMaxSurv says that the survivors do not fit the list.
template <bool kVec, int E>
__device__ __forceinline__ void chunk_survivors(const RowInfo& R, int base, int lane, int r, Survivor* surv, int& n_surv) {
  uint32_t x[E];
  load_bits<kVec, E>(R, base, lane, 0xff800000u, x);
  float lmax = -__builtin_inff();
#pragma unroll
  for (int e = 0; e < E; e += 2)
    asm("v_max3_f32 %0, %0, %1, %2" : "+v"(lmax) : "v"(x[e]), "v"(x[e + 1]));
  const uint32_t key = blk_of<kVec>(base, lane, 0) < R.b_vis ? order_key(__builtin_bit_cast(uint32_t, lmax)) : 0u;
  uint32_t tau = 0;
  if (E > 4 || R.b_vis - base > (kVec ? 4 : 1) * (r - 1)) {  // else fewer than r lanes hold anything
#pragma unroll
    for (int bit = 31; bit >= kTauLowBit; --bit) {
      const uint32_t trial = tau | (1u << bit);
      const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(key >= trial));
      tau = c >= r ? trial : tau;
    }
  }
  // tau as a score; with fewer than r lanes that hold more than -inf everything loaded survives, its NaNs as the -inf they rank with
  float thr = __builtin_bit_cast(float, (tau & 0x80000000u) ? tau ^ 0x80000000u : ~tau);
  if (tau <= 0x007fffffu) {  // the key of -inf
    thr = -__builtin_inff();
#pragma unroll
    for (int e = 0; e < E; ++e) {  // what was not loaded reads as -inf and would survive here, so it becomes a NaN
      asm volatile("" : "+v"(x[e]));  // keeps this in its branch: worked out for every row it was 47 instructions of 16 scores a lane
      const bool loaded = blk_of<kVec>(base, lane, kVec ? (e & ~3) : e) < R.b_vis;
      x[e] = loaded ? __builtin_bit_cast(uint32_t, __builtin_fmaxf(__builtin_bit_cast(float, x[e]), thr)) : 0x7fc00000u;
    }
  }
  const uint32_t not_blk = ~(uint32_t)blk_of<kVec>(base, lane, 0);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const bool sv = __builtin_bit_cast(float, x[e]) >= thr;
    const uint64_t m = __builtin_amdgcn_ballot_w64(sv);
    // (a list that overflows is discarded: its writes only have to stay inside the wavefront's LDS)
    const int at = min(n_surv, kMaxChunks * kMaxTopk - 64);
    const int pos = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)at));
    if (sv) {
      surv[pos].not_blk = not_blk - (uint32_t)blk_of<kVec>(0, 0, e);
      surv[pos].score = x[e];
    }
    n_surv += __builtin_popcountll(m);
  }
}

// Step 3: the survivors' columns.
__device__ __forceinline__ void rank_survivors(const RowInfo& R, int lane, Survivor* surv, int n_surv, int32_t* out_row) {
  // keys in place of the scores; 0 for what may not be picked, forced blocks and blocks past the visible range, and for the
  // entries that fill the list up to a multiple of eight
  for (int q = lane; q < ((n_surv + 7) & ~7); q += 64) {
    Survivor v = surv[q];
    const int b = (int)~v.not_blk;
    v.score = order_key(v.score);
    if (q >= n_surv || b >= R.b_vis || R.forced(b)) v.score = v.not_blk = 0;
    surv[q] = v;
  }
  wave_sync_lds();
  for (int q0 = 0; q0 < n_surv; q0 += 64) {
    const int q = q0 + lane;
    const uint64_t my = q < n_surv ? surv[q].both() : 0;
    int rank = 0;
    for (int s = 0; s < n_surv; s += 8) {
#pragma unroll
      for (int i = 0; i < 8; ++i) rank += surv[s + i].both() > my ? 1 : 0;   // same address in every lane: a broadcast
    }
    if (my != 0 && rank < R.want) out_row[R.n_forced + rank] = (int32_t)~(uint32_t)my;
  }
}

template <bool kVec>
__device__ __forceinline__ bool select_by_threshold(const RowInfo& R, int lane, Survivor* surv, int32_t* out_row) {
  const int r = R.want + R.ns + R.nl + 3;   // <= topk + 3 whenever want > 0
  const int n_chunks = (R.b_vis + kChunkBlocks - 1) / kChunkBlocks;
  int n_surv = 0;
  for (int c = 0; c < n_chunks; ++c) {
    const int base = c * kChunkBlocks;
    const int nq = (R.b_vis - base + 255) >> 8;   // quarter chunks with visible blocks (>= 1)
    if (nq >= 4) chunk_survivors<kVec, 16>(R, base, lane, r, surv, n_surv);
    else if (nq == 3) chunk_survivors<kVec, 12>(R, base, lane, r, surv, n_surv);
    else if (nq == 2) chunk_survivors<kVec, 8>(R, base, lane, r, surv, n_surv);
    else chunk_survivors<kVec, 4>(R, base, lane, r, surv, n_surv);
    if (n_surv > kMaxSurv) return false;
  }
  wave_sync_lds();
  rank_survivors(R, lane, surv, n_surv, out_row);
  return true;
}

}  // namespace

template <bool kVec, bool kMany>
__global__ void __launch_bounds__(64 * kSelWaves)
k_select_blocks(const float* __restrict__ scores, int64_t stride, const int32_t* __restrict__ cu, int T, int nseq,
                int hkv, int bk, int topk, int causal, int n_sink, int n_local, int32_t* __restrict__ idx) {
  // per wavefront: the survivor list of the fast method, or the chunk picks of the general one
  __shared__ Survivor lds[kSelWaves][kMaxChunks * kMaxTopk];
  static_assert(kMaxSurv <= kMaxChunks * kMaxTopk, "survivor list must fit");
  int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr uint32_t kRows = kMany ? kSelRows : 1;
  // consecutive rows a wavefront (T * hkv < 2^31 is checked on the host); what they share, a token's bounds, is worked out
  // once per token
  const uint32_t rows = (uint32_t)T * (uint32_t)hkv, first = ((uint32_t)blockIdx.x * kSelWaves + w) * kRows;
  if (first >= rows) return;               // whole wavefront leaves together
  const uint32_t end = kMany ? min(first + kRows, rows) : first + 1;
  int t = (int)(first / (uint32_t)hkv), j = (int)(first - (uint32_t)t * (uint32_t)hkv), t_known = -1;
  RowInfo R;
  R.srow = scores + (int64_t)first * stride;
  int32_t* out_row = idx + (int64_t)first * topk;
#pragma unroll 1
  for (uint32_t row = first; kMany ? row < end : row == first; ++row, R.srow += stride, out_row += topk) {
    if constexpr (kMany) asm volatile("" : "+v"(lane));  // what derives from it is not kept in registers from row to row
    if (t != t_known) {
      t_known = t;
      int s, c0, c1;
      seq_bounds(cu, nseq, T, t, s, c0, c1);
      const int cur = (t - c0) / bk;
      const int b_s = (c1 - c0 + bk - 1) / bk;
      R.b_vis = causal ? (cur + 1 < b_s ? cur + 1 : b_s) : b_s;
      if ((int64_t)R.b_vis > stride) R.b_vis = (int)stride;   // never read past a row, whatever cu says
      // forced blocks: sinks 0 .. ns-1, then cur - r0, cur - r0 - 1, ... (nl of them, all >= ns and < b_vis)
      R.ns = n_sink < R.b_vis ? n_sink : R.b_vis;
      const int r0 = cur - R.b_vis + 1 > 0 ? cur - R.b_vis + 1 : 0;
      const int r_last = n_local - 1 < cur - R.ns ? n_local - 1 : cur - R.ns;
      R.nl = r_last - r0 + 1 > 0 ? r_last - r0 + 1 : 0;
      R.loc_hi = cur - r0;
      R.loc_lo = R.loc_hi - R.nl + 1;
      R.n_forced = R.ns + R.nl < topk ? R.ns + R.nl : topk;
      R.want = topk - R.n_forced;
    }
    if (++j == hkv) {
      j = 0;
      ++t;
    }
    int mine = -1;                           // lane i holds column i of the output row: forced blocks, then -1
    if (lane < R.n_forced) mine = lane < R.ns ? lane : R.loc_hi - (lane - R.ns);
    const int n_free = R.b_vis - R.ns - R.nl;                  // selectable blocks
    int n_picks = R.want < n_free ? R.want : n_free;           // columns the selection fills
    bool by_rank = true;                     // pick columns already written, each by the lane that ranked there
    if (n_picks > 0 && scores == nullptr) {
      n_picks = 0;                           // forced blocks only: the rest of the row is padding
    }
    if (n_picks > 0) {
      by_rank = select_by_threshold<kVec>(R, lane, lds[w], out_row);
      if (!by_rank) mine = select_by_rounds<kVec>(R, lane, reinterpret_cast<uint32_t*>(lds[w]), mine);
      wave_sync_lds();                       // the next row writes there
    }
    if (lane < topk && (!by_rank || lane < R.n_forced || lane >= R.n_forced + n_picks)) out_row[lane] = mine;
  }
}

}  // namespace nsa

using namespace nsa;

extern "C" int nsa_sel_select_blocks(const nsa_sel_shape* shape, const float* scores, int64_t score_stride,
                                     const int32_t* cu_seqlens, int32_t n_sink, int32_t n_local, int32_t* idx,
                                     void* stream) {
  if (!shape) return NSA_SEL_EINVAL;
  if (shape->total_tokens < 0 || shape->nseq < 1 || shape->hkv < 1 || n_sink < 0 || n_local < 0) return NSA_SEL_EINVAL;
  if (shape->block != kBlock && shape->block != 2 * kBlock) return NSA_SEL_EUNSUPPORTED;
  if (shape->topk < 1 || shape->topk > kMaxTopk) return NSA_SEL_EUNSUPPORTED;
  if (!scores) score_stride = (int64_t)kMaxChunks * kChunkBlocks;   // no rows to stay inside
  if (score_stride < 1 || score_stride > (int64_t)kMaxChunks * kChunkBlocks) return NSA_SEL_EUNSUPPORTED;
  if (!idx || ((uintptr_t)scores & 3) || ((uintptr_t)idx & 3)) return NSA_SEL_EINVAL;   // scores may be NULL
  if (!cu_seqlens && shape->nseq != 1) return NSA_SEL_EINVAL;
  const int64_t rows = (int64_t)shape->total_tokens * shape->hkv;
  if (rows == 0) return NSA_SEL_OK;
  if (rows * shape->topk >= ((int64_t)1 << 31)) return NSA_SEL_EUNSUPPORTED;
  const bool many = eight_rows(rows, shape->hkv);
  const int64_t per = many ? kSelRows : 1;
  const int64_t grid = (rows + kSelWaves * per - 1) / (kSelWaves * per);
  if (grid >= ((int64_t)1 << 31)) return NSA_SEL_EUNSUPPORTED;
  hipStream_t st = (hipStream_t)stream;
  ProfScope prof(KID_SELECT_BLOCKS, st);
  const bool vec = (score_stride & 3) == 0 && ((uintptr_t)scores & 15) == 0;
  auto kern = many ? (vec ? k_select_blocks<true, true> : k_select_blocks<false, true>)
                   : (vec ? k_select_blocks<true, false> : k_select_blocks<false, false>);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * kSelWaves), 0, st, scores, score_stride, cu_seqlens,
                     shape->total_tokens, shape->nseq, shape->hkv, shape->block, shape->topk, shape->causal ? 1 : 0,
                     (int)n_sink, (int)n_local, idx);
  return hipGetLastError() == hipSuccess ? NSA_SEL_OK : NSA_SEL_EHIP;
}
