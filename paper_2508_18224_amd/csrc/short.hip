// Forward of short inputs for gfx950: where a token keeps a good part of all the blocks it sees, the gather of query rows by block, the
// partial rows and their reduction cost more than computing every (query tile, KV block) pair with a mask; and where the whole input is
// small, what bounds the forward is its chain of dependent launches (prep, histogram, prefix, scatter, main, merge).  Here one launch
// reads the selection tensor itself and writes O and LSE; the workgroups in front of it do the histogram and the tables of the
// inversion, which k_scatter finishes in a second launch (the index is an output that the backward and later calls read).
// Same definition of what a row attends to as the other forwards, fp32 accumulation over all of a row's keys.
#include "dense_piece.h"
#include "inversion.h"

namespace nsa {

hipError_t launch_short_lists(const IndexLayout& L, const int32_t* idx, const int32_t* cu, void* index_ws, hipStream_t st);

constexpr int kShortWaves = 4;
constexpr int kShortThreads = 64 * kShortWaves;

// Sequence bounds, and a place among equal parts of the sequences (query tiles, groups of rows), without the tables of the index: lane s
// looks at sequence s (at most 64 of them).
struct Sequences {
  int c0, c1, queries;   // of the lane's sequence; tokens past the last sequence are queries of it
  bool on;
  __device__ __forceinline__ Sequences(const IndexGeom& G, int lane, const int32_t* cu) {
    const int s = min(lane, G.nseq - 1);
    on = lane < G.nseq;
    c0 = G.nseq == 1 ? 0 : cu[s];
    c1 = G.nseq == 1 ? G.T : cu[s + 1];
    queries = s == G.nseq - 1 ? max(G.T - c0, 0) : c1 - c0;
  }
  __device__ __forceinline__ int blocks(const IndexGeom& G) const { return on ? (c1 - c0 + G.bk - 1) / G.bk : 0; }
  __device__ __forceinline__ int tiles() const { return on ? (queries + kTileTokens - 1) / kTileTokens : 0; }
};
__device__ __forceinline__ int wave_scan(int x, int lane) {  // inclusive
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  return x;
}
// The sequence that holds part i of those counted by `scan` (inclusive): its lane, or -1.
__device__ __forceinline__ int sequence_of(int scan, int i) {
  const unsigned long long after = __builtin_amdgcn_ballot_w64(scan > i);
  return after == 0ull ? -1 : __builtin_ctzll(after);
}

__device__ __forceinline__ Tile short_tile(const IndexGeom& G, int qt, int lane, const int32_t* cu) {
  Tile t = {0, 0, 0, 0, 0};
  const Sequences Q(G, lane, cu);
  const int nt = Q.tiles(), it = wave_scan(nt, lane), nb = Q.blocks(G), ib = wave_scan(nb, lane), o = sequence_of(it, qt);
  if (o < 0) return t;
  t.bb = __builtin_amdgcn_readlane(ib - nb, o);
  t.c0 = __builtin_amdgcn_readlane(Q.c0, o);
  t.c1 = __builtin_amdgcn_readlane(Q.c1, o);
  const int at = (qt - __builtin_amdgcn_readlane(it - nt, o)) * kTileTokens;
  t.tok0 = t.c0 + at;
  t.len = min(kTileTokens, __builtin_amdgcn_readlane(Q.queries, o) - at);
  return t;
}

// The tables k_prep and k_hist would write: per block first token and length, per tile first token, length and sequence.  One
// workgroup; a wavefront takes 64 blocks or tiles at a time, one after the other where several sequences share them.
__device__ void short_tables(const IndexGeom& G, const int32_t* cu, const IndexPtrs& p) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (G.nseq == 1) {
    for (int gb = tid; gb < G.b_cap; gb += kShortThreads) {
      const int len = max(min(G.bk, G.T - gb * G.bk), 0);
      p.blk_tok0[gb] = len > 0 ? gb * G.bk : 0;
      p.blk_len[gb] = len;
    }
    for (int qt = tid; qt < G.t_cap; qt += kShortThreads) {
      p.tile_tok0[qt] = qt * kTileTokens;
      p.tile_len[qt] = max(min(G.T - qt * kTileTokens, kTileTokens), 0);
    }
    return;
  }
  const Sequences Q(G, lane, cu);
  const int nb = Q.blocks(G), nt = Q.tiles(), ib = wave_scan(nb, lane), it = wave_scan(nt, lane);
  if (tid < G.nseq) {
    p.blk_base[tid] = ib - nb;
    p.tile_base[tid] = it - nt;
    if (tid == G.nseq - 1) {
      p.blk_base[G.nseq] = ib;
      p.tile_base[G.nseq] = it;
    }
  }
  auto owner = [&](int scan, int i) {  // the sequence that holds item i (the number of sequences: none)
    int o = 0;
    for (int q = 0; q < G.nseq; ++q) o += __builtin_amdgcn_readlane(scan, q) <= i ? 1 : 0;
    return o;
  };
  for (int i0 = tid - lane; i0 < G.b_cap; i0 += kShortThreads) {
    const int gb = i0 + lane, o = owner(ib, gb), from = min(o, G.nseq - 1);
    const int first = __shfl(ib - nb, from), a = __shfl(Q.c0, from), b = __shfl(Q.c1, from);
    if (gb < G.b_cap) {
      const int tok0 = a + (gb - first) * G.bk;
      p.blk_tok0[gb] = o < G.nseq ? tok0 : 0;
      p.blk_len[gb] = o < G.nseq ? min(G.bk, b - tok0) : 0;
    }
  }
  for (int i0 = tid - lane; i0 < G.t_cap; i0 += kShortThreads) {
    const int qt = i0 + lane, o = owner(it, qt), from = min(o, G.nseq - 1);
    const int first = __shfl(it - nt, from), a = __shfl(Q.c0, from), n = __shfl(Q.queries, from);
    if (qt < G.t_cap) {
      const int at = (qt - first) * kTileTokens;
      p.tile_tok0[qt] = o < G.nseq ? a + at : 0;
      p.tile_len[qt] = o < G.nseq ? min(kTileTokens, n - at) : 0;
      p.tile_seq[qt] = o < G.nseq ? o : 0;
    }
  }
}

// One chunk of k_hist's work: kept columns per token and the chunk's counters.
template <int KMAX>
__device__ void short_histogram(const IndexGeom& G, int chunk, int j, const int32_t* __restrict__ idx, const int32_t* cu,
                                const IndexPtrs& p, int32_t* hist) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int i = tid; i < G.b_cap; i += kShortThreads) hist[i] = 0;
  __syncthreads();
  for (int q = wave; q < kTilesPerChunk; q += kShortWaves) {
    const int qt = chunk * kTilesPerChunk + q;
    if (qt >= G.t_cap) break;
    const Tile t = short_tile(G, qt, lane, cu);
    const int tok = t.tok0 + lane;
    int32_t row[KMAX];
#pragma unroll
    for (int m = 0; m < KMAX; ++m) row[m] = -1;
    uint32_t vm = 0;
    if (lane < t.len) {
      const size_t at = (size_t)tok * G.hkv + j;
      load_row<KMAX>(idx + at * G.k, G.k, rows_are_vec4(idx, G.k), row);
      vm = kept_columns<KMAX>(G, t, tok, row);
      p.vmask[at] = vm;
    }
#pragma unroll
    for (int m = 0; m < KMAX; ++m)
      if (m < G.k) count_column(hist, t.bb + row[m], (vm >> m) & 1u, lane);
  }
  __syncthreads();
  int32_t* out = p.chunk_off + ((size_t)j * G.n_chunks + chunk) * G.b_cap;
  for (int i = tid; i < G.b_cap; i += kShortThreads) out[i] = hist[i];
}

// Dynamic LDS: per split two pairs of K and V tiles (afterwards the wavefronts' sums), then which of the workgroup's tokens keep a block (two
// 64-bit words), then a (max, sum) per row and split.
constexpr int kShortBlocks = 128;  // most blocks, and 64-key pieces, of a sequence
template <int S>
struct ShortLds {
  static constexpr int Masks = S * 4 * kPieceBytes;
  static constexpr int Stats = Masks + kShortBlocks * 16;
  static constexpr int Bytes = Stats + 32 * kShortWaves * 8;
};

// Workgroups [0, n_index) build the histogram and the tables of the inversion.  Every other one takes 128 / S consecutive (token, head)
// rows of one (sequence, KV head).  It marks, per block, which of its tokens keep it (a bit each; repeated, future and foreign ids
// fall out here), and walks the 64-key pieces of the blocks that some token keeps: with S = 2 two wavefronts each take every other
// piece of the sequence, and their sums are combined at the end.  A piece goes to the split of its place in the sequence, and one
// that a row does not keep leaves the row's sums as they are, so a row's bits do not depend on its neighbours.
// Rows that see nothing of a piece get +inf for a maximum there: their probabilities come out as exp2(-inf) = 0 without a select a score.
// Where K or V of a piece holds an infinity or a NaN, that shows in rows that never selected it.  So when anything the workgroup is
// about to write is not finite it walks its pieces again with selects, and with the sums of rows that do not keep a piece set back.
template <int S, int KMAX>
__global__ void __launch_bounds__(kShortThreads, 2)
k_fwd_short(Problem P, IndexGeom G, int n_index, int groups, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
            const bf16_t* __restrict__ V, const int32_t* __restrict__ idx, const int32_t* __restrict__ cu, IndexPtrs p,
            bf16_t* __restrict__ O, float* __restrict__ LSE, const float* __restrict__ gate, const bf16_t* Oacc, bf16_t* Oout) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int kGroups = kShortWaves / S, kRows = 32 * kGroups;  // wavefronts of a split, rows of the workgroup
  typedef ShortLds<S> Lds;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((int)blockIdx.x < n_index) {
    const int b = blockIdx.x, chunks = G.hkv * G.n_chunks;
    if (b < chunks) short_histogram<KMAX>(G, b % G.n_chunks, b / G.n_chunks, idx, cu, p, reinterpret_cast<int32_t*>(smem));
    else if (b == chunks) short_tables(G, cu, p);
    return;
  }
  // The chip's 8 XCDs get workgroups in turn.  The row groups of a KV head are dealt into eight classes (group % 8), later ones,
  // which see more blocks, first; an XCD takes hkv consecutive (head, class) pairs, so that its L2 holds the K and V of few
  // heads and all XCDs have as much to do.
  int j, item;
  {
    const int lid = (int)blockIdx.x - n_index, per_class = (groups + 7) >> 3;
    const int i = (lid & 7) * (P.hkv * per_class) + (lid >> 3);
    const int cls = i / per_class;
    j = cls >> 3;
    item = 8 * (per_class - 1 - (i - cls * per_class)) + (cls & 7);
  }
  Tile t = {0, 0, 0, 0, 0};  // the tokens of the workgroup's rows
  int row0, n_rows;          // its first row, counted from the first token's first head, and their number (1 .. kRows)
  {
    const Sequences X(G, lane, cu);
    const int n = X.on ? (X.queries * P.g + kRows - 1) / kRows : 0, in = wave_scan(n, lane), nb = X.blocks(G), ib = wave_scan(nb, lane);
    const int o = sequence_of(in, item);
    if (o < 0) return;
    t.bb = __builtin_amdgcn_readlane(ib - nb, o);
    t.c0 = __builtin_amdgcn_readlane(X.c0, o);
    t.c1 = __builtin_amdgcn_readlane(X.c1, o);
    const int first = (item - __builtin_amdgcn_readlane(in - n, o)) * kRows;
    const int last = min(first + kRows, __builtin_amdgcn_readlane(X.queries, o) * P.g) - 1;
    const int e0 = div_g(first, P.g, P.g_magic);
    t.tok0 = t.c0 + e0;
    t.len = div_g(last, P.g, P.g_magic) - e0 + 1;
    row0 = first - e0 * P.g;
    n_rows = last - first + 1;
  }
  const int col = lane & 31, qh = lane >> 5, rg = wave % kGroups, split = wave / kGroups;

  // this wavefront's rows of Q as B-operand fragments (past the last row: that row again, it sees no key)
  const bool valid = 32 * rg + col < n_rows;
  const int rc = row0 + min(32 * rg + col, n_rows - 1);
  const int e_row = div_g(rc, P.g, P.g_magic), tok = t.tok0 + e_row;
  bf16x8 qf[8];
  {
    const bf16_t* src = Q + ((size_t)tok * P.hq + j * P.g + (rc - e_row * P.g)) * kD + 8 * qh;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(src + 16 * s);
  }

  // which tokens keep a block
  unsigned long long* masks = reinterpret_cast<unsigned long long*>(smem + Lds::Masks);
  const int n_keys = t.c1 - t.c0, n_blocks = (n_keys + G.bk - 1) / G.bk;
  for (int i = tid; i < 2 * n_blocks; i += kShortThreads) masks[i] = 0ull;
  __syncthreads();
  {
    const int words = t.len > 64 ? 2 : 1, word = wave % words, part = wave / words, parts = kShortWaves / words;
    const int e = 64 * word + lane;
    const bool mine = e < t.len;
    const int tk = t.tok0 + min(e, t.len - 1);
    const int first = first_block(G, t, tk), last = last_block(G, t, tk);
    const size_t at = ((size_t)tk * G.hkv + j) * G.k;
    auto mark = [&](int x) {
      const bool on = mine && x >= first && x <= last;
      const unsigned long long act = __builtin_amdgcn_ballot_w64(on);
      if (act == 0ull) return;
      const int lead = __builtin_ctzll(act), x0 = __builtin_amdgcn_readlane(x, lead);
      if (__builtin_amdgcn_ballot_w64(on && x == x0) == act) {  // all agree, as on the sink: one atomic
        if (lane == lead) atomicOr(&masks[2 * x0 + word], act);
      } else if (on) {
        atomicOr(&masks[2 * x + word], 1ull << lane);
      }
    };
    if (idx != nullptr) {
      const bool vec4 = rows_are_vec4(idx, G.k);
      for (int m = 4 * part; m < G.k; m += 4 * parts) {
        int4 x = make_int4(-1, -1, -1, -1);
        if (vec4) {
          x = *reinterpret_cast<const int4*>(idx + at + m);
        } else {
          x.x = idx[at + m];
          if (m + 1 < G.k) x.y = idx[at + m + 1];
          if (m + 2 < G.k) x.z = idx[at + m + 2];
          if (m + 3 < G.k) x.w = idx[at + m + 3];
        }
        mark(x.x); mark(x.y); mark(x.z); mark(x.w);
      }
    } else {  // from the index: the list that holds the column's position
      const int32_t* off = p.off + j * G.b_cap + t.bb;
      for (int m = part; m < G.k; m += parts) {
        const int pos = p.slotpos[at + m];
        int lo = 0, hi = n_blocks;  // off[lo] <= pos < off[hi]
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (off[mid] <= pos) lo = mid; else hi = mid;
        }
        mark(pos >= 0 ? lo : -1);
      }
    }
  }
  __syncthreads();
  // the pieces of every split that some token keeps and sees: bit i of split s is piece s + S i of the sequence
  const int per = G.bk == kBlock ? 0 : 1;  // log2 of the pieces of a block
  constexpr int kWords = kShortBlocks / (64 * S);
  unsigned long long pieces[kWords];
  int steps = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    int count = 0;
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
      const int q = s + S * (64 * w + lane), k0 = 64 * q;
      bool on = k0 < n_keys;
      if (on) on = (masks[2 * (q >> per)] | masks[2 * (q >> per) + 1]) != 0ull;
      if (P.causal && t.c0 + k0 > t.tok0 + t.len - 1) on = false;
      if (P.window > 0 && t.c0 + k0 + 63 < t.tok0 - P.window + 1) on = false;
      const unsigned long long bits = __builtin_amdgcn_ballot_w64(on);
      count += __popcll(bits);
      if (s == split) pieces[w] = bits;
    }
    steps = max(steps, count);
  }

  const float c2 = P.scale * 1.4426950408889634f;
  const uint32_t k_lds = lds_address(smem) + split * 4 * kPieceBytes, v_lds = k_lds + 2 * kPieceBytes;
  uint32_t kaddr[8], vaddr[2][4];
  piece_addresses(k_lds, v_lds, lane, kaddr, vaddr);
  // access i of the split's wavefronts fills rows 4 kGroups i + 4 rg + lane / 16 of a tile (see load_to_lds)
  const int srow = 4 * rg + (lane >> 4);
  const uint32_t row_bytes = (uint32_t)P.hkv * kPieceRow;
  const uint32_t stage_off = srow * row_bytes + (((lane & 15) ^ row_turn(srow)) << 4);
  constexpr int kLoads = 16 / kGroups;
  // the rows of piece q of K or V, with -1 none: they arrive as zeros
  auto piece_of = [&](const bf16_t* X, int q) __attribute__((always_inline)) {
    const int len = q < 0 ? 0 : min(64, n_keys - 64 * q);
    return buffer_of(X + ((size_t)(t.c0 + 64 * max(q, 0)) * P.hkv + j) * kD, len > 0 ? (uint32_t)((len - 1) * P.hkv + 1) * kPieceRow : 0u);
  };
  auto load = [&](__amdgpu_buffer_rsrc_t buf, uint32_t lds, int i) __attribute__((always_inline)) {
    uint32_t from = stage_off;
    asm volatile("" : "+v"(from));  // the offsets are not kept in registers; row_turn(row + 8) = row_turn(row) ^ 2, row_turn(row + 16) = row_turn(row)
    load_to_lds(buf, lds + (4 * kGroups * i + 4 * rg) * kPieceRow, (kGroups == 2 ? from ^ (32 * (i & 1)) : from) + 4 * kGroups * i * row_bytes);
  };
  auto stage = [&](const bf16_t* X, uint32_t lds, int q) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t buf = piece_of(X, q);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load(buf, lds, i);
  };
  // the split's pieces in order; -1 past the last
  struct Walk {
    unsigned long long lo, hi;  // (hi: with one split a sequence may have more than 64 pieces)
    __device__ __forceinline__ explicit Walk(const unsigned long long (&pieces)[kWords]) : lo(pieces[0]), hi(pieces[kWords - 1]) {}
    __device__ __forceinline__ int take(int split) {
      if (kWords == 1) hi = 0ull;
      const bool second = lo == 0ull;
      const unsigned long long word = second ? hi : lo, rest = word & (word - 1ull);
      lo = second ? 0ull : rest;
      hi = second ? rest : hi;
      return __builtin_amdgcn_readfirstlane(word != 0ull ? split + S * ((second ? 64 : 0) + __builtin_ctzll(word)) : -1);
    }
  };
  // which of the workgroup's tokens of this lane's word keep piece q's block
  auto members_of = [&](int q) __attribute__((always_inline)) { return masks[2 * (max(q, 0) >> per) + (e_row >> 6)]; };
  // keys [lo, lim) of piece q are visible to this lane's row: none if its token does not keep the block
  auto visible = [&](int q, unsigned long long members, int& lo, int& lim) __attribute__((always_inline)) {
    const int k0 = t.c0 + 64 * q;
    lim = min(64, n_keys - 64 * q);
    if (P.causal) lim = min(lim, tok - k0 + 1);
    if (q < 0 || !valid || !((members >> (e_row & 63)) & 1ull)) lim = 0;
    lo = P.window > 0 ? max(tok - P.window + 1 - k0, 0) : 0;
  };

  f32x16 oacc[4];
  float mc_run = -INFINITY, l_run = 0.f;
  // The row's running maximum takes in that of a piece.  It is kept as the exponents use it, times c2 and rounded: where it stays, the sums
  // stay to the bit, and over a sequence's 128 pieces nothing adds up (taken anew from the raw maximum, what the rounding leaves of m * c2
  // went into the sums with every piece: LSE off by 1.7e-5 instead of 4e-6 over 8000 tokens with wide scores).
  auto take_in = [&](float m, bool sees, float& alpha) __attribute__((always_inline)) {
    const float mc = sees ? fmaxf(mc_run, m * c2) : mc_run;
    alpha = mc == mc_run ? 1.f : __builtin_amdgcn_exp2f(mc_run - mc);
    mc_run = mc;
    return !sees ? INFINITY : mc == -INFINITY ? 0.f : mc;  // what the piece's exponents are taken against
  };
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
    mc_run = -INFINITY;
    l_run = 0.f;
  };
  clear();
  {
    Walk walk(pieces);
    int q0 = walk.take(split), q1 = walk.take(split);  // this piece and the next
    stage(K, k_lds, q0);
    stage(V, v_lds, q0);
    stage(K, k_lds + kPieceBytes, q1);
    unsigned long long members = members_of(q0);
    await_rows(qf);
    wait_loads();
    __syncthreads();
    f32x16 even[2], odd[2];
    piece_scores(kaddr, qf, even);
    float m = row_max(max_scores(even));
    auto step = [&](f32x16 (&cur)[2], f32x16 (&next)[2], int side) __attribute__((always_inline)) {
      // this piece's K tile has been read in the step before: K of the piece after the next flies there, V of the next to the other tile
      const int q2 = walk.take(split);
      const __amdgpu_buffer_rsrc_t kbuf = piece_of(K, q2), vbuf = piece_of(V, q1);
      keep_addresses(kaddr, vaddr);
      uint32_t ka[8], va[2][4];
#pragma unroll
      for (int s = 0; s < 8; ++s) ka[s] = kaddr[s] + (side ^ 1) * kPieceBytes;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        va[0][d] = vaddr[0][d] + side * kPieceBytes;
        va[1][d] = vaddr[1][d] + side * kPieceBytes;
      }
      int lo, lim;
      visible(q0, members, lo, lim);
      const bool sees = lim > lo;
      if (__builtin_amdgcn_ballot_w64(sees && (lim < 64 || lo > 0)) != 0ull) m = row_max(mask_scores(cur, lo, lim, qh));
      float alpha;
      const float mc = take_in(m, sees, alpha);
      members = members_of(q1);
      m = piece_values_and_next_scores(ka, va, qf, c2, mc, alpha, cur, next, l_run, oacc,
                                       [&](int i) __attribute__((always_inline)) {
                                         if (i < kLoads) load(vbuf, v_lds + (side ^ 1) * kPieceBytes, i);
                                         else if (i < 2 * kLoads) load(kbuf, k_lds + side * kPieceBytes, i - kLoads);
                                       });
      m = row_max(m);
      wait_loads();
      __syncthreads();
      q0 = q1;
      q1 = q2;
    };
    __syncthreads();  // every wavefront has read the first K
    for (int n = 0; n < steps; n += 2) {
      step(even, odd, 0);
      if (n + 1 < steps) step(odd, even, 1);
    }
  }
  float finite = l_run * 0.f;  // a NaN as soon as anything is not finite
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) finite = fmaf(oacc[db][v], 0.f, finite);
  if (__syncthreads_or(finite != finite) != 0) {
    clear();
    Walk walk(pieces);
    for (int n = 0; n < steps; ++n) {
      const int q = walk.take(split);
      stage(K, k_lds, q);
      stage(V, v_lds, q);
      wait_loads();
      __syncthreads();
      if (q >= 0) {
        int lo, lim;
        visible(q, members_of(q), lo, lim);
        const bool sees = lim > lo;
        f32x16 sacc[2];
        piece_scores(kaddr, qf, sacc);
        float alpha;
        const float mc = take_in(row_max(mask_scores(sacc, lo, lim, qh)), sees, alpha);
        bf16x8 pf[4];
        float l = 0.f;
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) pf[sp] = piece_probabilities(sacc, sp, c2, mc, l);
        l_run = fmaf(l_run, alpha, l + __shfl_xor(l, 32));
#pragma unroll
        for (int db = 0; db < 4; ++db) {
          f32x16 sum;
#pragma unroll
          for (int v = 0; v < 16; ++v) sum[v] = oacc[db][v] * alpha;
#pragma unroll
          for (int sp = 0; sp < 4; ++sp)
            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(value_frag(vaddr, sp, db), pf[sp], sum, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[db][v] = sees ? sum[v] : oacc[db][v];
        }
      }
      __syncthreads();
    }
  }

  int lane_b = threadIdx.x & 63;
  asm volatile("" : "+v"(lane_b));  // what follows is not worked out ahead of the loop
  const int col_b = lane_b & 31, qh_b = lane_b >> 5;
  // combine the splits: row sums scaled to the row's maximum over them, 512 bytes a row, 16-byte chunk c of row r at place c ^ r
  float2* stats = reinterpret_cast<float2*>(smem + Lds::Stats);
  if (qh_b == 0) stats[32 * wave + col_b] = make_float2(mc_run, l_run);
  __syncthreads();
  {
    float M = -INFINITY;
#pragma unroll
    for (int s = 0; s < S; ++s) M = fmaxf(M, stats[32 * (s * kGroups + rg) + col_b].x);
    const float f = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc_run - M);
    unsigned char* dst = smem + wave * 32 * 512 + col_b * 512;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 x = {oacc[db][4 * a] * f, oacc[db][4 * a + 1] * f, oacc[db][4 * a + 2] * f, oacc[db][4 * a + 3] * f};
        *reinterpret_cast<f32x4*>(dst + (((8 * db + 2 * a + qh_b) ^ col_b) << 4)) = x;
      }
  }
  __syncthreads();
  const int sub = lane_b & 15;
  for (int rr = 4 * wave + (lane_b >> 4); rr < n_rows; rr += 4 * kShortWaves) {
    const int e = div_g(row0 + rr, P.g, P.g_magic);
    const size_t grow = (size_t)(t.tok0 + e) * P.hq + j * P.g + (row0 + rr - e * P.g);
    float2 st[S];
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      st[s] = stats[32 * kGroups * s + rr];
      M = fmaxf(M, st[s].x);
    }
    // nothing visible: O = 0, LSE = -inf, and the gated sum is what the other branches gave (where the visible scores are all -inf,
    // LSE is that too and O is not a number)
    bool empty = M == -INFINITY;
    for (int b = 0; empty && b < n_blocks; ++b) empty = ((masks[2 * b + (e >> 6)] >> (e & 63)) & 1ull) == 0ull;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < S; ++s) {
      L += st[s].x == -INFINITY ? 0.f : st[s].y * __builtin_amdgcn_exp2f(st[s].x - M);
      const unsigned char* src = smem + (kGroups * s + (rr >> 5)) * 32 * 512 + (rr & 31) * 512;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(src + (((2 * sub + h) ^ (rr & 31)) << 4));
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[4 * h + c] += x[c];
      }
    }
    const float inv = empty ? 0.f : 1.f / L;
    const u32x4 o = {pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv),
                     pack_bf16x2(acc[4] * inv, acc[5] * inv), pack_bf16x2(acc[6] * inv, acc[7] * inv)};
    *reinterpret_cast<u32x4*>(O + grow * kD + 8 * sub) = o;
    if (sub == 0) LSE[grow] = empty ? -INFINITY : (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
    if (gate != nullptr) {
      // Eq. (2): O_out = O_acc + gate * O, from the fp32 result (Oout may be the buffer Oacc points to: every lane
      // reads its own 16 bytes before it writes them)
      const float tau = gate[grow] * inv;
      u32x4 a = {0, 0, 0, 0};
      if (Oacc != nullptr) a = *reinterpret_cast<const u32x4*>(Oacc + grow * kD + 8 * sub);
      if (!empty) {
        a.x = pack_bf16x2(bf16_lo(a.x) + tau * acc[0], bf16_hi(a.x) + tau * acc[1]);
        a.y = pack_bf16x2(bf16_lo(a.y) + tau * acc[2], bf16_hi(a.y) + tau * acc[3]);
        a.z = pack_bf16x2(bf16_lo(a.z) + tau * acc[4], bf16_hi(a.z) + tau * acc[5]);
        a.w = pack_bf16x2(bf16_lo(a.w) + tau * acc[6], bf16_hi(a.w) + tau * acc[7]);
      }
      *reinterpret_cast<u32x4*>(Oout + grow * kD + 8 * sub) = a;
    }
  }
}

// Most row groups a KV head can have.
static int short_groups(const Problem& P, int splits) { return P.T * P.g / (32 * kShortWaves / splits) + P.nseq; }

template <int S, int KMAX>
static hipError_t launch_short(const Problem& P, const IndexGeom& G, bool build, const void* Q, const void* K, const void* V,
                               const int32_t* idx, const int32_t* cu, const IndexPtrs& p, void* O, float* LSE, const GateArgs& A,
                               hipStream_t st) {
  static std::atomic<uint64_t> ready;
  const hipError_t e = allow_dynamic_lds((const void*)(k_fwd_short<S, KMAX>), ShortLds<S>::Bytes, ready);
  if (e != hipSuccess) return e;
  const int groups = short_groups(P, S), n_index = build ? (G.hkv * G.n_chunks + 1 + 7) & ~7 : 0;
  ProfScope ps(KID_FWD_SHORT, st);
  hipLaunchKernelGGL((k_fwd_short<S, KMAX>), dim3(n_index + 8 * P.hkv * ((groups + 7) / 8)), dim3(kShortThreads), ShortLds<S>::Bytes, st, P, G,
                     n_index, groups, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, build ? idx : nullptr, cu, p, (bf16_t*)O, LSE,
                     A.gate, (const bf16_t*)A.o_acc, (bf16_t*)A.o_out);
  return hipGetLastError();
}

hipError_t launch_fwd_short(const Problem& P, const IndexLayout& L, bool build, const void* Q, const void* K, const void* V,
                            const int32_t* idx, const int32_t* cu, void* index_ws, void* O, float* LSE, const GateArgs& A, hipStream_t st) {
  const IndexGeom G = index_geom(L);
  const IndexPtrs p = index_ptrs(L, index_ws);
  // few workgroups: two splits, which leave one workgroup (a wavefront a SIMD) on a compute unit
  const bool few = (int64_t)P.hkv * short_groups(P, 2) <= 320;
  hipError_t e;
  if (few) e = G.k <= 8 ? launch_short<2, 8>(P, G, build, Q, K, V, idx, cu, p, O, LSE, A, st)
             : G.k <= 16 ? launch_short<2, 16>(P, G, build, Q, K, V, idx, cu, p, O, LSE, A, st)
                         : launch_short<2, 32>(P, G, build, Q, K, V, idx, cu, p, O, LSE, A, st);
  else e = G.k <= 8 ? launch_short<1, 8>(P, G, build, Q, K, V, idx, cu, p, O, LSE, A, st)
         : G.k <= 16 ? launch_short<1, 16>(P, G, build, Q, K, V, idx, cu, p, O, LSE, A, st)
                     : launch_short<1, 32>(P, G, build, Q, K, V, idx, cu, p, O, LSE, A, st);
  if (e != hipSuccess || !build) return e;
  return launch_short_lists(L, idx, cu, index_ws, st);
}

}  // namespace nsa
