// Index inversion for selected-block attention: from the selection table idx[token, kv head, column] build, for
// every (kv head, KV block), the ascending list of query tokens that select it (the paper's index tensor I_i,
// Sec. 3.2, the paragraph on the token-selection kernel) together with the column each entry came from, and, per kept
// (token, kv head, column), the entry's position in its list, which is where its partial result lives in the
// compact partial buffers (the role of the paper's O_i), plus the work-unit tables of the attention kernels.
//
// Three launches (for packed batches k_prep before them, and k_dense where the tokens are walked without regard to sequences; small
// inputs without the dense route go without k_prefix, see index_folds; the forward of short inputs does the work of the launches
// before it in its own, see short.hip):
//   k_hist     per (kv head, chunk, block) counts, kept columns per token, dense (query tile, KV block) pairs
//   k_prefix   per list: prefix over the chunks, length; per 64 lists: sums
//   k_scatter  exclusive scan of the list lengths (redone by every workgroup from the 64-list sums), list entries and
//              their positions, work units
// Everything is organised by query tile: 64 consecutive tokens of one sequence, one wavefront, lane = token.  A chunk
// is kTilesPerChunk tiles = one workgroup.  The counters are stored chunk-major, [kv head][chunk][block], so that
// the histogram and the scatter of one (chunk, kv head) touch one contiguous row.
// Batches of many short sequences (index_by_token) would have a tile, mostly empty, per sequence, and counters that grow with
// the square of the number of sequences: there a wavefront takes 64 consecutive tokens whatever sequences they belong to
// (the lists come out the same), and only the dense pairs, which are defined by query tile, are found tile by tile, in k_dense.
// Lists come out ascending without a sort and without order-dependent atomics: a token's rank inside its tile is a
// popcount over a 64-bit membership mask, the tiles of a chunk are ordered by a byte count per (block, tile).
//
// The inversion reads a few MB and is bound by latency and launches, not by bandwidth: 137 us at 65536 tokens x 8 kv heads (52
// histogram, 8 prefix, 76 scatter).  An earlier cut (12 launches; one wavefront walked a chunk's 512 tokens in eight dependent
// rounds; separate scan, dense-detection and unit kernels) took 233 us there.
#include "inversion.h"

namespace nsa {

constexpr int kPrefixWaves = 16;                     // wavefronts of a k_prefix workgroup (64 lists each)
constexpr int kScatterWindow = 1024;                 // most blocks k_scatter handles at a time (its LDS tables)

template <bool kByToken>
__device__ __forceinline__ Tile load_tile(const IndexGeom& G, int qt, int lane, const int32_t* cu, const IndexPtrs& p) {
  Tile t = {0, 0, 0, 0, 0};
  if constexpr (kByToken) {
    t.tok0 = qt * kTileTokens;
    t.len = max(min(G.T - t.tok0, kTileTokens), 0);
    if (t.len == 0) return t;
    int s;
    seq_bounds(cu, G.nseq, G.T, t.tok0 + min(lane, t.len - 1), s, t.c0, t.c1);
    t.bb = p.blk_base[s];
    return t;
  }
  if (qt >= G.t_cap) return t;
  if (G.nseq == 1) {
    t.tok0 = qt * kTileTokens;
    t.len = max(min(G.T - t.tok0, kTileTokens), 0);
    t.c1 = G.T;
    return t;
  }
  t.len = p.tile_len[qt];
  if (t.len == 0) return t;
  const int s = p.tile_seq[qt];
  t.tok0 = p.tile_tok0[qt];
  t.c0 = cu[s];
  t.c1 = cu[s + 1];
  t.bb = p.blk_base[s];
  return t;
}

// The window [lo, hi) of global blocks the tokens of a chunk can keep; block-wide (every wavefront passes its own tile).
// Blocks ascend with the tokens: the first lane knows where a tile's begin, the last where they end.
__device__ __forceinline__ void chunk_window(const IndexGeom& G, const Tile& t, int wave, int* s_win, int& lo, int& hi) {
  const int lane = threadIdx.x & 63;
  if (lane == 0) s_win[2 * wave] = t.len > 0 ? t.bb : 0x7fffffff;
  if (lane == 63) s_win[2 * wave + 1] = t.len > 0 ? t.bb + last_block(G, t, t.tok0 + t.len - 1) + 1 : 0;
  __syncthreads();
  lo = 0x7fffffff;
  hi = 0;
#pragma unroll
  for (int w = 0; w < kTilesPerChunk; ++w) {
    lo = min(lo, s_win[2 * w]);
    hi = max(hi, s_win[2 * w + 1]);
  }
  if (lo > hi) lo = hi;
}

// ------------------------------------------------------------------------------------------------ prep
// Packed batches: blk_base[s] / tile_base[s] = number of KV blocks / query tiles of sequences < s; per global block its
// first token and its key count, per tile its first token, length and sequence.  One workgroup.  (For a single sequence
// the tables are closed forms that k_hist writes.)  The tiles cover every token up to T, whatever the last of cu says: tokens
// past it (a padded batch) are queries of the last sequence, so that no row of the per-token tables stays unwritten.
__global__ void __launch_bounds__(1024) k_prep(IndexGeom G, const int32_t* __restrict__ cu, IndexPtrs p) {
  __shared__ int s_sum[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int carry_b = 0, carry_t = 0;
  for (int s0 = 0; s0 < G.nseq; s0 += 1024) {
    const int s = s0 + tid;
    const int len = s < G.nseq ? cu[s + 1] - cu[s] : 0, queries = s == G.nseq - 1 ? max(G.T - cu[s], 0) : len;
    const int nb = (len + G.bk - 1) / G.bk, nt = (queries + kTileTokens - 1) / kTileTokens;
    int ib = nb, it = nt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int xb = __shfl_up(ib, d), xt = __shfl_up(it, d);
      if (lane >= d) { ib += xb; it += xt; }
    }
    __syncthreads();  // the previous round's sums are no longer read
    if (lane == 63) { s_sum[0][wave] = ib; s_sum[1][wave] = it; }
    __syncthreads();
    int before_b = carry_b, before_t = carry_t;
    for (int w = 0; w < 16; ++w) {
      if (w < wave) { before_b += s_sum[0][w]; before_t += s_sum[1][w]; }
      carry_b += s_sum[0][w];
      carry_t += s_sum[1][w];
    }
    if (s < G.nseq) {
      p.blk_base[s] = before_b + ib - nb;
      p.tile_base[s] = before_t + it - nt;
    }
  }
  if (tid == 0) {
    p.blk_base[G.nseq] = carry_b;
    p.tile_base[G.nseq] = carry_t;
  }
  __threadfence_block();
  __syncthreads();
  auto owner = [&](const int32_t* base, int i) {  // base[s] <= i < base[s + 1]
    int lo = 0, hi = G.nseq;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (base[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
  };
  for (int gb = tid; gb < G.b_cap; gb += 1024) {
    int tok0 = 0, len = 0;
    if (gb < carry_b) {
      const int s = owner(p.blk_base, gb);
      tok0 = cu[s] + (gb - p.blk_base[s]) * G.bk;
      len = min(G.bk, cu[s + 1] - tok0);
    }
    p.blk_tok0[gb] = tok0;
    p.blk_len[gb] = len;
  }
  for (int qt = tid; qt < G.t_cap; qt += 1024) {
    int tok0 = 0, len = 0, s = 0;
    if (qt < carry_t) {
      s = owner(p.tile_base, qt);
      tok0 = cu[s] + (qt - p.tile_base[s]) * kTileTokens;
      len = min(kTileTokens, (s == G.nseq - 1 ? G.T : cu[s + 1]) - tok0);
    }
    p.tile_tok0[qt] = tok0;
    p.tile_len[qt] = len;
    p.tile_seq[qt] = s;
  }
}

// ------------------------------------------------------------------------------------------------ dense detection
// Dense forward path: which (query tile, KV block) pairs skip the gather route.  One wavefront per (tile, kv head), lane =
// token: a KV block that at least `need` = half of the tile's tokens keep (the attention-sink block, the tokens' own
// block and the blocks next to it are kept by all of them) becomes a dense pair: the forward computes it for the whole
// tile with the query tile read once and the output accumulated on chip, a 64-bit mask saying which tokens really keep
// it.  The tokens' columns that hold such a block are recorded in dmask; the scatter flags their list entries, and the
// gather route of the forward skips them.  Nothing here is assumed about the selection: pairs come from counting, and
// any pair may take either route.  Candidates are the kept blocks of three tokens of the tile (first, middle, last); a
// block that qualifies but is kept by none of the three simply stays on the gather route.  A per-wavefront table of
// counters (block id modulo kDenseHash, LDS atomics: counts are order-free) tells which candidates can reach `need`:
// only the few that pass get the exact count (a ballot).
// The dense table lists 64-key pieces (a 128-token block gives two) by first key and key count, in the order found;
// pieces no token of the tile can see (wholly in the future, or wholly before every token's window) are left out.
// Returns the lane's dense columns.
template <int KMAX>
__device__ __forceinline__ uint32_t dense_detect(const IndexGeom& G, const Tile& t, const int32_t (&row)[KMAX], uint32_t vm,
                                                 int lane, size_t slot, int32_t* hash, const IndexPtrs& p) {
  for (int i = lane; i < kDenseHash / 4; i += 64) reinterpret_cast<int4*>(hash)[i] = make_int4(0, 0, 0, 0);
  wave_lds_sync();
  int kept[KMAX];  // -1 where the column is not kept: no candidate matches it
#pragma unroll
  for (int m = 0; m < KMAX; ++m) {
    const bool on = (vm >> m) & 1u;
    kept[m] = on ? row[m] : -1;
    if (m < G.k) count_column(hash, row[m] & (kDenseHash - 1), on, lane);
  }
  wave_lds_sync();
  const int need = (t.len + 1) >> 1;
  const int prop[3] = {0, t.len >> 1, t.len - 1};
  int nd = 0;
  uint32_t dm = 0;
  for (int pi = 0; pi < 3; ++pi) {
    const int pr = prop[pi];
    if ((pi == 1 && pr == prop[0]) || (pi == 2 && (pr == prop[0] || pr == prop[1]))) continue;
    const uint32_t pvm = (uint32_t)__builtin_amdgcn_readlane((int)vm, pr);
    // lane m: column m of token pr's row
    int cand_blk = 0;
#pragma unroll
    for (int m = 0; m < KMAX; ++m) {
      const int x = __builtin_amdgcn_readlane(row[m], pr);
      cand_blk = lane == m ? x : cand_blk;
    }
    const bool mine = lane < G.k && ((pvm >> (lane & 31)) & 1u);
    const int cand_cnt = mine ? hash[cand_blk & (kDenseHash - 1)] : 0;
    unsigned long long cand = __builtin_amdgcn_ballot_w64(cand_cnt >= need);
    while (cand != 0ull) {
      const int m = __builtin_ctzll(cand);
      cand &= cand - 1ull;
      const int c = __builtin_amdgcn_readlane(cand_blk, m);
      int mycol = -1;
#pragma unroll
      for (int mm = KMAX - 1; mm >= 0; --mm) mycol = kept[mm] == c ? mm : mycol;
      const unsigned long long members = __builtin_amdgcn_ballot_w64(mycol >= 0);
      // an earlier proposer that keeps c has already dealt with it
      bool seen = false;
      for (int pj = 0; pj < pi; ++pj) seen |= ((members >> prop[pj]) & 1ull) != 0ull;
      if (seen || __popcll(members) < need) continue;
      // the block's 64-key pieces some token of the tile can see
      const int btok0 = t.c0 + c * G.bk, blen = min(G.bk, t.c1 - btok0);
      int np = 0, ptok[2], plen[2];
      for (int sub = 0; sub < (G.bk >> 6); ++sub) {
        const int pt = btok0 + 64 * sub, pl = min(64, blen - 64 * sub);
        if (pl <= 0) continue;
        if (G.causal && pt > t.tok0 + t.len - 1) continue;
        if (G.window > 0 && pt + pl - 1 < t.tok0 - G.window + 1) continue;
        ptok[np] = pt;
        plen[np] = pl;
        ++np;
      }
      if (nd + np > kDenseMax) continue;
      if (lane == 0)
        for (int q = 0; q < np; ++q) {
          p.d_piece[slot * kDenseMax + nd + q] = make_int2(ptok[q], plen[q]);
          p.d_mask[slot * kDenseMax + nd + q] = members;
        }
      if (mycol >= 0) dm |= 1u << mycol;  // also when no piece is visible: the pair then contributes nothing
      nd += np;
    }
  }
  if (lane == 0) p.d_cnt[slot] = nd;
  return dm;
}

// The same for every tile of the grid's, also the empty ones at its end, with the lanes' dense columns recorded.
template <int KMAX>
__device__ __forceinline__ void dense_tile(const IndexGeom& G, const Tile& t, const int32_t (&row)[KMAX], uint32_t vm, int lane,
                                           int qt, int j, int32_t* hash, const IndexPtrs& p) {
  const size_t slot = (size_t)qt * G.hkv + j;
  if (t.len > 0) {
    const uint32_t dm = dense_detect<KMAX>(G, t, row, vm, lane, slot, hash, p);
    if (lane < t.len) p.dmask[(size_t)(t.tok0 + lane) * G.hkv + j] = dm;
  } else if (lane == 0) {
    p.d_cnt[slot] = 0;
  }
}

// Detection as a launch of its own, where the histogram does not go by query tile.  grid (ceil(t_cap / kTilesPerChunk), hkv).
// Dynamic LDS: kTilesPerChunk * kDenseHash ints.
template <int KMAX>
__global__ void __launch_bounds__(kChunkThreads) k_dense(IndexGeom G, const int32_t* __restrict__ idx,
                                                         const int32_t* __restrict__ cu, IndexPtrs p) {
  extern __shared__ __attribute__((aligned(16))) int32_t lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), j = blockIdx.y;
  const int qt = blockIdx.x * kTilesPerChunk + wave;
  if (qt >= G.t_cap) return;  // no block-wide barrier below
  const Tile t = load_tile<false>(G, qt, lane, cu, p);
  int32_t row[KMAX];
#pragma unroll
  for (int m = 0; m < KMAX; ++m) row[m] = -1;
  uint32_t vm = 0;
  if (lane < t.len) {
    const size_t at = (size_t)(t.tok0 + lane) * G.hkv + j;
    load_row<KMAX>(idx + at * G.k, G.k, rows_are_vec4(idx, G.k), row);
    vm = p.vmask[at];
  }
  dense_tile<KMAX>(G, t, row, vm, lane, qt, j, lds + wave * kDenseHash, p);
}

// ------------------------------------------------------------------------------------------------ histogram
// grid (n_chunks, hkv).  chunk_off[(j*n_chunks + chunk)*b_cap + gb] = number of tokens of the chunk that keep block gb
// for kv head j; the whole row is written (zeros outside the chunk's window), so the array needs no clearing.  The rows
// of idx stay in registers (one 16-byte load per four columns); the duplicate test is k^2/2 register compares.
// Dynamic LDS: b_cap ints, with the dense route (by tile) + kTilesPerChunk * kDenseHash ints.
template <int KMAX, bool kByToken>
__global__ void __launch_bounds__(kChunkThreads) k_hist(IndexGeom G, const int32_t* __restrict__ idx,
                                                        const int32_t* __restrict__ cu, IndexPtrs p) {
  extern __shared__ __attribute__((aligned(16))) int32_t lds[];
  __shared__ int s_win[2 * kTilesPerChunk];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int chunk = blockIdx.x, j = blockIdx.y;
  const int qt = chunk * kTilesPerChunk + wave;
  const Tile t = load_tile<kByToken>(G, qt, lane, cu, p);
  const int tok = t.tok0 + lane;
  const bool live = lane < t.len;
  int32_t row[KMAX];
#pragma unroll
  for (int m = 0; m < KMAX; ++m) row[m] = -1;
  if (live) load_row<KMAX>(idx + ((size_t)tok * G.hkv + j) * G.k, G.k, rows_are_vec4(idx, G.k), row);
  int gb_lo, gb_hi;
  chunk_window(G, t, wave, s_win, gb_lo, gb_hi);
  int32_t* hash = lds + wave * kDenseHash;
  int32_t* hist = lds + (G.dense && !kByToken ? kTilesPerChunk * kDenseHash : 0);
  for (int i = tid; i < gb_hi - gb_lo; i += kChunkThreads) hist[i] = 0;
  if (G.nseq == 1 && j == 0) {  // block and tile tables of a single sequence
    if (lane == 0 && qt < G.t_cap) {
      p.tile_tok0[qt] = t.tok0;
      p.tile_len[qt] = t.len;
    }
    const int per = kTilesPerChunk * kTileTokens / G.bk;
    for (int gb = chunk * per + tid; gb < min((chunk + 1) * per, G.b_cap); gb += kChunkThreads) {
      const int len = max(min(G.bk, G.T - gb * G.bk), 0);
      p.blk_tok0[gb] = len > 0 ? gb * G.bk : 0;
      p.blk_len[gb] = len;
    }
  }
  uint32_t vm = 0;
  if (live) {
    vm = kept_columns<KMAX>(G, t, tok, row);
    p.vmask[(size_t)tok * G.hkv + j] = vm;
  }
  __syncthreads();
  const int base = t.bb - gb_lo;
#pragma unroll
  for (int m = 0; m < KMAX; ++m)
    if (m < G.k) count_column(hist, base + row[m], (vm >> m) & 1u, lane);
  if constexpr (!kByToken)
    if (G.dense && qt < G.t_cap) dense_tile<KMAX>(G, t, row, vm, lane, qt, j, hash, p);
  __syncthreads();
  int32_t* out = p.chunk_off + ((size_t)j * G.n_chunks + chunk) * G.b_cap;
  for (int i = tid; i < G.b_cap; i += kChunkThreads) out[i] = (i >= gb_lo && i < gb_hi) ? hist[i - gb_lo] : 0;
}

// ------------------------------------------------------------------------------------------------ prefix
// For every list (kv head j, block gb): chunk_off[j][chunk][gb] becomes the number of entries the list gets from
// earlier chunks, cnt receives the list's length, group_sum the (entries, work units) of 64 lists.  A workgroup owns 64
// consecutive blocks of one kv head; its wavefronts take a share of the chunks each (sum, exchange through LDS, then
// prefix), so the column walk is a handful of coalesced row accesses per thread.  grid (n_groups, hkv).
__global__ void __launch_bounds__(64 * kPrefixWaves) k_prefix(IndexGeom G, int32_t* __restrict__ counters,
                                                              int32_t* __restrict__ cnt, int2* __restrict__ group_sum) {
  __shared__ int32_t part[kPrefixWaves][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6, j = blockIdx.y;
  const int gb = blockIdx.x * 64 + lane;
  const bool live = gb < G.b_cap;
  const int per = (G.n_chunks + kPrefixWaves - 1) / kPrefixWaves;
  const int c0 = min(q * per, G.n_chunks), c1 = min(c0 + per, G.n_chunks);
  int32_t* col = counters + (size_t)j * G.n_chunks * G.b_cap + (live ? gb : 0);
  int32_t sum = 0;
  if (live) {
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
      int32_t v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = col[(size_t)(c + i) * G.b_cap];
#pragma unroll
      for (int i = 0; i < 8; ++i) sum += v[i];
    }
    for (; c < c1; ++c) sum += col[(size_t)c * G.b_cap];
  }
  part[q][lane] = sum;
  __syncthreads();
  int32_t run = 0;
  for (int w = 0; w < q; ++w) run += part[w][lane];
  if (live) {
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
      int32_t v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = col[(size_t)(c + i) * G.b_cap];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        col[(size_t)(c + i) * G.b_cap] = run;
        run += v[i];
      }
    }
    for (; c < c1; ++c) {
      const int32_t v = col[(size_t)c * G.b_cap];
      col[(size_t)c * G.b_cap] = run;
      run += v;
    }
  }
  if (q == kPrefixWaves - 1) {
    if (live) cnt[j * G.b_cap + gb] = run;
    int e = live ? run : 0, nu = (e + G.unit - 1) / G.unit;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      e += __shfl_xor(e, d);
      nu += __shfl_xor(nu, d);
    }
    if (lane == 0) group_sum[j * G.n_groups + blockIdx.x] = make_int2(e, nu);
  }
}

// Block-wide (kChunkThreads threads) sums of two values; ends with a barrier.
__device__ __forceinline__ int2 block_sum(int2 v, int2* s_red) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    v.x += __shfl_xor(v.x, d);
    v.y += __shfl_xor(v.y, d);
  }
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  int2 r = make_int2(0, 0);
#pragma unroll
  for (int w = 0; w < kTilesPerChunk; ++w) {
    r.x += s_red[w].x;
    r.y += s_red[w].y;
  }
  __syncthreads();
  return r;
}

// Block-wide exclusive scan of two values per thread; `total` receives the sums.  Ends with a barrier.
__device__ __forceinline__ int2 block_scan(int2 v, int2* s_red, int2& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int2 inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int x = __shfl_up(inc.x, d), y = __shfl_up(inc.y, d);
    if (lane >= d) { inc.x += x; inc.y += y; }
  }
  if (lane == 63) s_red[wave] = inc;
  __syncthreads();
  int2 before = make_int2(0, 0);
  total = make_int2(0, 0);
#pragma unroll
  for (int w = 0; w < kTilesPerChunk; ++w) {
    const int2 x = s_red[w];
    if (w < wave) { before.x += x.x; before.y += x.y; }
    total.x += x.x;
    total.y += x.y;
  }
  __syncthreads();
  return make_int2(before.x + inc.x - v.x, before.y + inc.y - v.y);
}

// ------------------------------------------------------------------------------------------------ scatter
// grid (n_chunks + 1, hkv).  Workgroup x = 0 of a kv head writes its scanned list offsets and work units; workgroup
// x = 1 + chunk writes the chunk's list entries and, per token, the row of their positions.  The exclusive scan over the
// lists is not a pass of its own: every workgroup sums the 64-list sums in front of its first list and scans the lengths
// of the lists it needs (a few KB from L2).
// A chunk's blocks are taken `win` at a time (one pass unless a sequence has more than kScatterWindow blocks).  Per
// pass: every wavefront marks its tokens in its own 64-bit mask per block; the lowest member of a mask leaves the count
// as the wavefront's byte of the block's word; a token's position is list offset + entries of earlier chunks +
// the bytes of the wavefronts before its own + popcount(mask below its lane).
// Dynamic LDS: win * (8 masks + 1 word of bytes + 1 offset) = 76 win bytes.
// kFold: the prefix over the chunks is not a launch before this one; the counters are still k_hist's, and every workgroup
// sums the few it needs by itself (see index_folds).
template <int KMAX, bool kByToken, bool kFold>
__global__ void __launch_bounds__(kChunkThreads) k_scatter(IndexGeom G, int win, const int32_t* __restrict__ idx,
                                                           const int32_t* __restrict__ cu, IndexPtrs p) {
  extern __shared__ __attribute__((aligned(16))) int32_t lds[];
  __shared__ int s_win[2 * kTilesPerChunk];
  __shared__ int2 s_red[kTilesPerChunk];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = blockIdx.y;
  const int2* gsum = p.group_sum + j * G.n_groups;  // the 64-list sums of this kv head, those of the others before it
  // (length, entries of the chunks before `upto`) of list gb of kv head jj, from the histogram's counters
  auto list_counts = [&](int jj, int gb, int upto) {
    const int32_t* c = p.chunk_off + (size_t)jj * G.n_chunks * G.b_cap + gb;
    int2 r = make_int2(0, 0);
#pragma unroll 4
    for (int i = 0; i < G.n_chunks; ++i, c += G.b_cap) {
      const int x = *c;
      r.x += x;
      r.y += i < upto ? x : 0;
    }
    return r;
  };
  if (blockIdx.x == 0) {
    int2 run = make_int2(0, 0);
    if constexpr (kFold) {
      for (int i = tid; i < j * G.b_cap; i += kChunkThreads) {
        const int len = list_counts(i / G.b_cap, i % G.b_cap, 0).x;
        run.x += len;
        run.y += (len + G.unit - 1) / G.unit;
      }
    } else {
      for (int i = tid - j * G.n_groups; i < 0; i += kChunkThreads) {
        const int2 x = gsum[i];
        run.x += x.x;
        run.y += x.y;
      }
    }
    run = block_sum(run, s_red);
    for (int b0 = 0; b0 < G.b_cap; b0 += kChunkThreads) {
      const int gb = b0 + tid, L = j * G.b_cap + gb;
      const int len = gb < G.b_cap ? (kFold ? list_counts(j, gb, 0).x : p.cnt[L]) : 0, nu = (len + G.unit - 1) / G.unit;
      int2 total;
      const int2 ex = block_scan(make_int2(len, nu), s_red, total);
      const int e0 = run.x + ex.x, u0 = run.y + ex.y;
      if (gb < G.b_cap) {
        p.off[L] = e0;
        p.u_nu[L] = u0;
        if constexpr (kFold) p.cnt[L] = len;
        const int tok0 = p.blk_tok0[gb], blen = p.blk_len[gb];
        for (int u = 0; u < nu; ++u) {
          int4* rec = reinterpret_cast<int4*>(p.u_rec + u0 + u);
          rec[0] = make_int4(e0 + u * G.unit, min(G.unit, len - u * G.unit), tok0, blen);
          rec[1] = make_int4(j, nu, 0, 0);
        }
      }
      run.x += total.x;
      run.y += total.y;
    }
    if (j == G.hkv - 1 && tid == 0) {
      p.off[G.hkv * G.b_cap] = run.x;
      p.u_nu[G.hkv * G.b_cap] = run.y;
    }
    return;
  }
  const int chunk = blockIdx.x - 1;
  const Tile t = load_tile<kByToken>(G, chunk * kTilesPerChunk + wave, lane, cu, p);
  const int tok = t.tok0 + lane;
  const bool live = lane < t.len;
  int32_t row[KMAX];
#pragma unroll
  for (int m = 0; m < KMAX; ++m) row[m] = -1;
  uint32_t vm = 0, dm = 0;
  if (live) {
    load_row<KMAX>(idx + ((size_t)tok * G.hkv + j) * G.k, G.k, rows_are_vec4(idx, G.k), row);
    vm = p.vmask[(size_t)tok * G.hkv + j];               // kept columns, decided by the histogram pass
    if (G.dense) dm = p.dmask[(size_t)tok * G.hkv + j];  // those of them the dense forward path takes over
  }
  int gb_lo, gb_hi;
  chunk_window(G, t, wave, s_win, gb_lo, gb_hi);
  unsigned long long* masks = reinterpret_cast<unsigned long long*>(lds);
  unsigned long long* bytes = masks + kTilesPerChunk * win;
  int32_t* cursor = reinterpret_cast<int32_t*>(bytes + win);
  unsigned long long* mask = masks + wave * win;
  const unsigned long long below = (1ull << lane) - 1ull;
  int32_t pos[KMAX];
#pragma unroll
  for (int m = 0; m < KMAX; ++m) pos[m] = -1;

  const int w_first = kFold ? 0 : gb_lo & ~63;  // passes start at a 64-list boundary
  int2 part = make_int2(0, 0);
  if constexpr (kFold) {
#pragma unroll 4
    for (int i = tid; i < j * G.n_chunks * G.b_cap; i += kChunkThreads) part.x += p.chunk_off[i];
  } else {
    for (int i = tid - j * G.n_groups; i < (w_first >> 6); i += kChunkThreads) part.x += gsum[i].x;
  }
  int run = block_sum(part, s_red).x;  // first position of list (j, w_first)
  const int32_t* chunk_off = p.chunk_off + ((size_t)j * G.n_chunks + chunk) * G.b_cap;
  for (int w0 = w_first; w0 < gb_hi; w0 += win) {
    // list offsets of the window's blocks: two consecutive blocks per thread
    const int i0 = 2 * tid, gb = w0 + i0;
    const bool on0 = i0 < win && gb < G.b_cap, on1 = i0 + 1 < win && gb + 1 < G.b_cap;
    int len0 = 0, len1 = 0, co0 = 0, co1 = 0;
    if constexpr (kFold) {
      const int2 a = on0 ? list_counts(j, gb, chunk) : make_int2(0, 0), b = on1 ? list_counts(j, gb + 1, chunk) : make_int2(0, 0);
      len0 = a.x; co0 = a.y; len1 = b.x; co1 = b.y;
    } else {
      if (on0) { len0 = p.cnt[j * G.b_cap + gb]; co0 = chunk_off[gb]; }
      if (on1) { len1 = p.cnt[j * G.b_cap + gb + 1]; co1 = chunk_off[gb + 1]; }
    }
    for (int i = tid; i < 9 * win / 2; i += kChunkThreads)  // masks and bytes, 16 bytes at a time
      reinterpret_cast<uint4*>(lds)[i] = make_uint4(0, 0, 0, 0);
    int2 total;
    const int2 ex = block_scan(make_int2(len0 + len1, 0), s_red, total);
    if (i0 < win) cursor[i0] = run + ex.x + co0;
    if (i0 + 1 < win) cursor[i0 + 1] = run + ex.x + len0 + co1;
    run += total.x;
    __syncthreads();
    const int base = t.bb - w0;
    int at[KMAX];  // the column's block inside the window, -1 where it is not kept or belongs to another pass
#pragma unroll
    for (int m = 0; m < KMAX; ++m) {
      const int b = base + row[m];
      at[m] = (((vm >> m) & 1u) && b >= 0 && b < win) ? b : -1;
      if (m >= G.k) continue;
      const unsigned long long act = __builtin_amdgcn_ballot_w64(at[m] >= 0);
      if (act == 0ull) continue;
      const int lead = __builtin_ctzll(act);
      const int x0 = __builtin_amdgcn_readlane(at[m], lead);
      if (__builtin_amdgcn_ballot_w64(at[m] == x0) == act) {  // a column all lanes agree on: one atomic (see count_column)
        if (lane == lead) atomicOr(&mask[x0], act);
      } else if (at[m] >= 0) {
        atomicOr(&mask[at[m]], 1ull << lane);
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < KMAX; ++m) {
      if (at[m] < 0) continue;
      const unsigned long long mk = mask[at[m]];
      if ((mk & below) == 0ull) reinterpret_cast<uint8_t*>(bytes + at[m])[wave] = (uint8_t)__popcll(mk);
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < KMAX; ++m) {
      if (at[m] < 0) continue;
      // tokens of this tile before the lane, then of the chunk's earlier tiles (v_sad_u8 adds four bytes)
      int q = cursor[at[m]] + __popcll(mask[at[m]] & below);
      const unsigned long long earlier = bytes[at[m]] & ((1ull << (8 * wave)) - 1ull);
      q = (int)__builtin_amdgcn_sad_u8((uint32_t)earlier, 0u, (uint32_t)q);
      q = (int)__builtin_amdgcn_sad_u8((uint32_t)(earlier >> 32), 0u, (uint32_t)q);
      // the sign bit of the column flags an entry of a dense (tile, block) pair: the forward's gather route skips
      // it, the backward (which walks whole lists) ignores the flag
      p.qent[q] = make_int2(tok, m | (int)(((dm >> m) & 1u) << 31));
      pos[m] = q;
    }
    if (w0 + win < gb_hi) __syncthreads();  // the tables are rewritten by the next pass
  }
  if (live) {
    int32_t* dst = p.slotpos + ((size_t)tok * G.hkv + j) * G.k;
    if (rows_are_vec4(p.slotpos, G.k)) {
#pragma unroll
      for (int m = 0; m < KMAX; m += 4)
        if (m < G.k) *reinterpret_cast<int4*>(dst + m) = make_int4(pos[m], pos[m + 1], pos[m + 2], pos[m + 3]);
    } else {
#pragma unroll
      for (int m = 0; m < KMAX; ++m)
        if (m < G.k) dst[m] = pos[m];
    }
  }
}

template <int KMAX, bool kByToken, bool kFold>
static hipError_t launch_scatter(const IndexGeom& G, const int32_t* idx, const int32_t* cu, const IndexPtrs& p, hipStream_t st) {
  const int win = min((G.b_cap + 63) & ~63, kScatterWindow);
  const int lds = 76 * win;
  if (lds > 60 * 1024) {  // beyond the default 64 KB
    static std::atomic<uint64_t> ready;
    const hipError_t e = allow_dynamic_lds((const void*)(k_scatter<KMAX, kByToken, kFold>), 150 * 1024, ready);
    if (e != hipSuccess) return e;
  }
  ProfScope ps(KID_INDEX_SCATTER, st);
  hipLaunchKernelGGL((k_scatter<KMAX, kByToken, kFold>), dim3(G.n_chunks + 1, G.hkv), dim3(kChunkThreads), lds, st, G, win, idx, cu, p);
  return hipGetLastError();
}

// From the histogram's counters to the lists.
template <int KMAX, bool kByToken>
static hipError_t launch_lists(const IndexGeom& G, const int32_t* idx, const int32_t* cu, const IndexPtrs& p, hipStream_t st) {
  if constexpr (!kByToken)
    if (!G.dense && index_folds(G.T, G.nseq, G.hkv, G.bk)) return launch_scatter<KMAX, false, true>(G, idx, cu, p, st);
  {
    ProfScope ps(KID_INDEX_SCAN, st);
    hipLaunchKernelGGL(k_prefix, dim3(G.n_groups, G.hkv), dim3(64 * kPrefixWaves), 0, st, G, p.chunk_off, p.cnt,
                       p.group_sum);
  }
  return launch_scatter<KMAX, kByToken, false>(G, idx, cu, p, st);
}

template <int KMAX, bool kByToken>
static hipError_t launch_inversion(const IndexGeom& G, const int32_t* idx, const int32_t* cu, const IndexPtrs& p,
                                   hipStream_t st) {
  const int lds_dense = 4 * kTilesPerChunk * kDenseHash, lds_hist = 4 * G.b_cap + (G.dense && !kByToken ? lds_dense : 0);
  if (lds_hist > 60 * 1024) {  // beyond the default 64 KB
    static std::atomic<uint64_t> ready;
    const hipError_t e = allow_dynamic_lds((const void*)(k_hist<KMAX, kByToken>), 150 * 1024, ready);
    if (e != hipSuccess) return e;
  }
  {
    ProfScope ps(KID_INDEX_HIST, st);
    hipLaunchKernelGGL((k_hist<KMAX, kByToken>), dim3(G.n_chunks, G.hkv), dim3(kChunkThreads), lds_hist, st, G, idx, cu, p);
  }
  if constexpr (kByToken) {
    if (G.dense) {
      ProfScope ps(KID_INDEX_DENSE, st);
      hipLaunchKernelGGL(k_dense<KMAX>, dim3((G.t_cap + kTilesPerChunk - 1) / kTilesPerChunk, G.hkv), dim3(kChunkThreads),
                         lds_dense, st, G, idx, cu, p);
    }
  }
  return launch_lists<KMAX, kByToken>(G, idx, cu, p, st);
}

IndexGeom index_geom(const IndexLayout& L) {
  IndexGeom G;
  G.nseq = L.nseq;
  G.T = L.T;
  G.hkv = L.hkv;
  G.k = L.topk;
  G.bk = L.bk;
  G.causal = L.causal;
  G.window = L.window;
  G.b_cap = L.b_cap;
  G.t_cap = L.t_cap;
  G.n_chunks = L.n_chunks;
  G.n_groups = L.n_groups;
  G.unit = L.unit;
  G.dense = L.dense;
  return G;
}

hipError_t launch_build_index(const IndexLayout& L, const int32_t* idx, const int32_t* cu, void* index_ws,
                              hipStream_t st) {
  const IndexPtrs p = index_ptrs(L, index_ws);
  const IndexGeom G = index_geom(L);
  if (G.nseq > 1) {
    ProfScope ps(KID_INDEX_PREP, st);
    hipLaunchKernelGGL(k_prep, dim3(1), dim3(1024), 0, st, G, cu, p);
  }
  // rows of idx live in registers: a variant per width
  if (index_by_token(L.T, L.nseq)) {
    if (G.k <= 8) return launch_inversion<8, true>(G, idx, cu, p, st);
    if (G.k <= 16) return launch_inversion<16, true>(G, idx, cu, p, st);
    return launch_inversion<32, true>(G, idx, cu, p, st);
  }
  if (G.k <= 8) return launch_inversion<8, false>(G, idx, cu, p, st);
  if (G.k <= 16) return launch_inversion<16, false>(G, idx, cu, p, st);
  return launch_inversion<32, false>(G, idx, cu, p, st);
}

// The same after a kernel that did the histogram's work and the tables' (k_fwd_short).
hipError_t launch_short_lists(const IndexLayout& L, const int32_t* idx, const int32_t* cu, void* index_ws, hipStream_t st) {
  const IndexPtrs p = index_ptrs(L, index_ws);
  const IndexGeom G = index_geom(L);
  if (G.k <= 8) return launch_lists<8, false>(G, idx, cu, p, st);
  if (G.k <= 16) return launch_lists<16, false>(G, idx, cu, p, st);
  return launch_lists<32, false>(G, idx, cu, p, st);
}

}  // namespace nsa
