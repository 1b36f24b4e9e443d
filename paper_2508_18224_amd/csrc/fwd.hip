// Forward selected-block attention for gfx950 (paper Sec. 3.2, the KV-outer token-selection step and the
// reduction step; Eq. (2), c = sel).
//
// k_fwd_main (B_K = 64): one work unit = (kv head j, KV block i, up to P.unit entries of the block's query list).
//   The block's K_i stays in registers for the whole unit (the A operand of S^T = K_i Q^T) and V_i^T sits in LDS,
//   transposed and key-permuted once per unit (the A operand of O^T = V_i^T P^T), so the inner loop reads no K/V
//   from memory: each wavefront walks tiles of 32 query rows (row = (list entry, head of the group), flattened so
//   any g packs densely).  The kernel is held to 256 registers per wavefront so that TWO workgroups share a CU:
//   one's unit prologue, gather waits and softmax overlap the other's MFMA and stores (with V_i^T in registers too
//   only one workgroup fitted and the kernel ran 30 % slower).  The rows of Q are gathered coalesced (16 lanes x 16
//   bytes per row) one tile ahead and re-laid out into the B-operand layout
//   through a wave-private LDS tile; 16 + 16 MFMA 32x32x16 bf16 per tile; the softmax of the 64 scores of a row
//   runs inside the accumulator layout (a lane holds 32 keys of one query; one cross-lane exchange with
//   lane ^ 32 completes max and sum).  Because S^T leaves each lane holding keys of ONE query, the probabilities
//   are already in B-operand layout for the PV product; no transposition of P is needed.
//   The result of a (token, head, block) triple is a partial output normalised by its own sum, plus the
//   log-sum-exp of its 64 scores; both are stored at the entry's own position in the list order (the compact
//   buffer the paper addresses through O_i), so a tile's 32 rows are one contiguous 8 KB (non-temporal) write.
// k_fwd_main128 (B_K = 128): see the comment above it.
// k_fwd_merge: per (token, head) combines the kept slots: LSE = ln sum_s exp(lse_s), O = sum_s exp(lse_s-LSE) O_s.
//   This replaces the paper's separate statistics pre-pass: per-slot log-sum-exps make the merge exact.
#include "dense_piece.h"
#include <type_traits>

namespace nsa {

constexpr int kVtStride = 72;     // bf16 per row of the transposed V tile in LDS: 64 keys + 8 pad
constexpr int kTileStride = 136;  // bf16 per row of a wave's private 32-row tile in LDS: 128 + 8 pad

// Place of a key in the contraction order of the PV product.  The accumulator of a 32x32 MFMA gives lane
// (col, q) the rows 8a + 4q + c (a, c in 0..3) of each 32-key half mb; contraction step s' = 2 mb + a / 2 takes
// element e = 4 (a & 1) + c from lane group q.
__device__ __forceinline__ int key_pos(int key) {
  const int mb = key >> 5, a = (key >> 3) & 3, q = (key >> 2) & 1, c = key & 3;
  return 16 * (2 * mb + (a >> 1)) + 8 * q + 4 * (a & 1) + c;
}

// Orders a wavefront's own LDS traffic (no cross-wave meaning): a wave-private tile is written by some lanes and
// read by others of the same wave.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}


// Tokens of a work unit's list entries that take the gather route, compacted into `ent`, with each one's index
// inside the unit in `epos` (its partial rows live at the entry's list position, dense entries leave holes there).
// Entries of dense (tile, block) pairs carry the sign bit in their column (see k_scatter) and are skipped.  Block-wide:
// every thread takes entries i0 + tid of up to kMaxUnit / kThreads rounds, a round's survivors of a wavefront are
// ranked by ballot, and the (round, wavefront) counts are prefix-summed through `cnts`.  Returns the number of
// entries kept; ends with a barrier.
template <int kThreads>
__device__ __forceinline__ int load_sparse_entries(const int2* __restrict__ qent, int e0, int ne, int32_t* ent,
                                                   uint16_t* epos, int32_t* cnts) {
  constexpr int kRounds = kMaxUnit / kThreads, kWaves = kThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int tok[kRounds];
  unsigned long long keep[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int i = r * kThreads + tid;
    int2 e = make_int2(0, -1);
    if (i < ne) e = qent[e0 + i];
    tok[r] = e.x;
    keep[r] = __builtin_amdgcn_ballot_w64(e.y >= 0);
    if (lane == 0) cnts[r * kWaves + wave] = __popcll(keep[r]);
  }
  __syncthreads();
  int run = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    int before = 0;  // survivors of earlier rounds and of the lower wavefronts of this round
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w == wave) before = run;
      run += cnts[r * kWaves + w];
    }
    if ((keep[r] >> lane) & 1ull) {
      const int pos = before + __popcll(keep[r] & ((1ull << lane) - 1ull));
      ent[pos] = tok[r];
      epos[pos] = (uint16_t)(r * kThreads + tid);
    }
  }
  __syncthreads();
  return run;
}

// One row (list entry, head of the group) of a unit.  It is found once per tile by the lane that owns it (both halves of
// the wavefront alike) and handed to the lanes that move it by lane_value.
struct GatherRow {
  uint32_t src;   // (token, head) row of Q; total_tokens * hq < 2^31 is checked on the host
  uint32_t part;  // row inside the unit's partial rows: list position in the unit * g + head
  int t;          // token, -1 past the end of the list (those re-read the last row, are masked out and never stored)
};

__device__ __forceinline__ GatherRow find_row(const Problem& P, int r, int rows_total, int hbase, const int32_t* ent,
                                              const uint16_t* epos) {
  const int rc = min(r, rows_total - 1);
  const int e = div_g(rc, P.g, P.g_magic), hh = rc - e * P.g;
  const int tok = ent[e];
  GatherRow x;
  x.src = (uint32_t)tok * (uint32_t)P.hq + (uint32_t)(hbase + hh);
  x.part = (uint32_t)(epos[e] * P.g + hh);
  x.t = r < rows_total ? tok : -1;
  return x;
}

// A tile's 32 partial rows (wave-private LDS tile) to their list positions: consecutive entries of the unit give one
// contiguous run, broken only where a dense pair's entries were left out.
__device__ __forceinline__ void store_partial_rows(const bf16_t* tile_lds, const GatherRow& x, bool valid, int crow,
                                                   int cchunk, __amdgpu_buffer_rsrc_t o_buf) {
  const uint32_t dst = valid ? x.part : kNoRow / (kD * 2);
  uint32_t to[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) to[i] = lane_value(dst, 4 * i + crow);
#pragma unroll
  for (int i = 0; i < 8; ++i)
    __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(&tile_lds[(4 * i + crow) * kTileStride + cchunk]),
                                           o_buf, to[i] * (kD * 2) + cchunk * 2, 0, kNonTemporal);
}

__device__ __forceinline__ void store_partial_lse(float lse, const GatherRow& x, bool on, __amdgpu_buffer_rsrc_t l_buf) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, lse), l_buf, on ? x.part * 4 : kNoRow, 0, 0);
}

// LDS of k_fwd_main (dynamic: 66 KB, two workgroups per CU)
constexpr int kF64Vt = 0;
constexpr int kF64Tiles = kF64Vt + kD * kVtStride * 2;
constexpr int kF64Ent = kF64Tiles + 4 * 32 * kTileStride * 2;
constexpr int kF64Epos = kF64Ent + kMaxUnit * 4;
constexpr int kF64Cnts = kF64Epos + kMaxUnit * 2;
constexpr int kF64Bytes = kF64Cnts + (kMaxUnit / 64) * 4;
static_assert(2 * kF64Bytes <= 160 * 1024, "two workgroups of the 64-key forward must fit one CU's LDS");

// Bound by the traffic between the XCDs and the memory side: 14.3 GB per launch at 65536 tokens, g = 4, which this kernel
// moves at 7.0 TB/s.  Rows move by branch-free buffer instructions with the row's place worked out once per tile and lane: with
// branches around the stores and 64-bit addresses per access every wait for the next rows also drained the stores and the tile
// cost a third more vector instructions (2.14 -> 2.04 ms; at 8192 tokens, g = 1: 367 -> 330 us).
template <bool kWide, bool kInTurn>
__global__ void __launch_bounds__(256, 2)  // two workgroups per CU: 256 registers per wavefront
k_fwd_main(Problem P, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
           const UnitRec* __restrict__ u_rec, const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ off,
           const int2* __restrict__ qent, bf16_t* __restrict__ opart, float* __restrict__ lse_part) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* Vt = reinterpret_cast<bf16_t*>(smem + kF64Vt);
  int32_t* ent = reinterpret_cast<int32_t*>(smem + kF64Ent);     // tokens of the unit's list entries that take this route
  uint16_t* epos = reinterpret_cast<uint16_t*>(smem + kF64Epos);  // and their index inside the unit
  int32_t* cnts = reinterpret_cast<int32_t*>(smem + kF64Cnts);
  UnitRec U;
  int pos0;
  if (!load_unit<kInTurn>(P, u_rec, nu_scan, off, U, pos0)) return;
  const int j = U.j, e0 = U.e0, ne_all = U.ne, tok0 = U.tok0, blen = U.blen;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, qh = lane >> 5;
  const int crow = lane >> 4, cchunk = (lane & 15) * 8;  // coalesced layout: 16 lanes per row, 4 rows per access
  const uint32_t row_bytes = (uint32_t)P.hkv * (kD * 2);
  // The block's V (thread = key, 32 channels) and K fragments.  They are requested before the entries are looked at, except
  // with a window and the dense route, where nearly every unit turns out to have no entry left.
  bf16x8 vreg[4], kf[2][8];
  auto load_block = [&]() __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t k_buf = block_buffer(K, P, U), v_buf = block_buffer(V, P, U);
#pragma unroll
    for (int i = 0; i < 4; ++i) vreg[i] = load_frag(v_buf, (tid >> 2) * row_bytes + (tid & 3) * 64 + 16 * i);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int s = 0; s < 8; ++s) kf[mb][s] = load_frag(k_buf, (32 * mb + col) * row_bytes + 16 * qh + 32 * s);
  };
  const bool late = P.window > 0 && P.dense;
  if (!late) load_block();
  // entries of dense (tile, block) pairs are the dense kernel's: a unit made of them only (the sink block's) ends here
  const int ne = load_sparse_entries<256>(qent, e0, ne_all, ent, epos, cnts);
  if (ne == 0) return;
  if (late) load_block();
  {  // V_i -> LDS, transposed and key-permuted
    const int d0 = (tid & 3) * 32, pos = key_pos(tid >> 2);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) Vt[(d0 + 8 * i + e) * kVtStride + pos] = vreg[i][e];
  }
  __syncthreads();
  const bf16_t* vbase = &Vt[col * kVtStride + 8 * qh];  // this lane's V^T fragments: + 32 db rows, + 16 sp keys

  const int rows_total = ne * P.g;
  const int n_tiles = (rows_total + 31) >> 5;
  if (wave >= n_tiles) return;  // no block-wide barrier below this point
  const float c2 = P.scale * 1.4426950408889634f;  // scores in the log2 domain
  bf16_t* tile_lds = reinterpret_cast<bf16_t*>(smem + kF64Tiles) + wave * 32 * kTileStride;
  const int hbase = j * P.g;
  const RowTensor<kWide> Qrows(Q, (int64_t)P.T * P.hq);
  // the unit's partial rows and log-sum-exps: list positions e0 .. of the pass, row = position * g + head
  const size_t part0 = (size_t)(e0 - pos0) * P.g;
  const __amdgpu_buffer_rsrc_t o_buf = buffer_of(opart + part0 * kD, (uint32_t)(ne_all * P.g) * (kD * 2));
  const __amdgpu_buffer_rsrc_t l_buf = buffer_of(lse_part + part0, (uint32_t)(ne_all * P.g) * 4);

  auto row_of = [&](int tile) __attribute__((always_inline)) {
    return find_row(P, tile * 32 + col, rows_total, hbase, ent, epos);
  };
  // gather the 32 rows of Q of a tile in coalesced form (a row = 16 lanes x 16 bytes, 4 rows per access)
  u32x4 qc[8];
  auto issue_q = [&](const GatherRow& x) __attribute__((always_inline)) {
    uint32_t row[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) row[i] = lane_value(x.src, 4 * i + crow);
#pragma unroll
    for (int i = 0; i < 8; ++i) qc[i] = Qrows.load(row[i], cchunk * 2);
  };

  GatherRow cur = row_of(wave), next = row_of(wave + 4);
  issue_q(cur);
  pad_stores<9>(l_buf);
  int tile = wave;
  do {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      *reinterpret_cast<u32x4*>(&tile_lds[(4 * i + crow) * kTileStride + cchunk]) = qc[i];
    // this wave's next tile: its rows fly during the compute (past the last tile: the list's last row again, unused)
    issue_q(next);
    wave_sync();
    bf16x8 qf[8];
#pragma unroll
    for (int s = 0; s < 8; ++s)
      qf[s] = *reinterpret_cast<const bf16x8*>(&tile_lds[col * kTileStride + 16 * s + 8 * qh]);

    f32x16 sacc[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) sacc[mb][v] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
        sacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[mb][s], qf[s], sacc[mb], 0, 0, 0);

    // keys [0, lim) of the block are visible to this row
    const int t = cur.t;
    const bool valid = t >= 0;
    int lim = P.causal ? min(blen, t - tok0 + 1) : blen;
    if (!valid) lim = 0;
    const int lo = P.window > 0 ? t - P.window + 1 - tok0 : 0;  // with a window, keys before lo are hidden (<= 0: none)
    // Only tiles with a row in the block itself (causal diagonal), a ragged block end or a window edge need the
    // key mask; the test is wave-uniform.  The maximum is taken over the raw scores (the scale is positive) and the scale is
    // folded into the exponent: p = 2^(s c2 - m c2).
    float m = -INFINITY;
    if (__builtin_amdgcn_ballot_w64(lim < kBlock || lo > 0) == 0) {
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) m = fmaxf(m, sacc[mb][v]);
    } else {
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = 32 * mb + 8 * (v >> 2) + 4 * qh + (v & 3);
          const float x = (key < lim && key >= lo) ? sacc[mb][v] : -INFINITY;
          sacc[mb][v] = x;
          m = fmaxf(m, x);
        }
    }
    m = fmaxf(m, __shfl_xor(m, 32));
    const float mc = (m == -INFINITY) ? 0.f : m * c2;  // row maximum in the log2 domain
    float l = 0.f;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[mb][v], c2, -mc));
        sacc[mb][v] = p;
        l += p;
      }
    l += __shfl_xor(l, 32);

    bf16x8 pf[4];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int e2 = 0; e2 < 8; ++e2) pf[sp][e2] = (bf16_t)sacc[sp >> 1][8 * (sp & 1) + e2];

    f32x16 oacc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const bf16x8 vf = *reinterpret_cast<const bf16x8*>(vbase + 32 * db * kVtStride + 16 * sp);
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[sp], oacc[db], 0, 0, 0);
      }

    // normalised partial rows -> wave tile in LDS -> coalesced 256-byte row stores
    const float inv = valid ? 1.f / l : 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        uint2 w;
        w.x = pack_bf16x2(oacc[db][4 * a + 0] * inv, oacc[db][4 * a + 1] * inv);
        w.y = pack_bf16x2(oacc[db][4 * a + 2] * inv, oacc[db][4 * a + 3] * inv);
        *reinterpret_cast<uint2*>(&tile_lds[col * kTileStride + 32 * db + 8 * a + 4 * qh]) = w;
      }
    wave_sync();
    store_partial_rows(tile_lds, cur, valid, crow, cchunk, o_buf);
    store_partial_lse((mc + __builtin_amdgcn_logf(l)) * 0.6931471805599453f, cur, valid && qh == 0, l_buf);
    wave_sync();
    cur = next;
    next = row_of(tile + 8);
    tile += 4;
  } while (tile < n_tiles);
}

// ---- B_K = 128 -----------------------------------------------------------------------------------------------
// Same work split, but a 128-key block does not fit the register file next to the tile state, so K_i and V_i sit
// row-major in LDS: K fragments are plain 16-byte reads, V^T fragments are LDS transpose reads (no transposed
// copy).  A tile computes S^T for all 128 keys (4 x 8 MFMA), one softmax over the 128 scores of a row, and
// O^T = V_i^T P^T (8 x 4 MFMA); one partial row and one log-sum-exp per (token, head, selected 128-block).
constexpr int kPitch128 = 152;  // bf16 per LDS row of K / V (128 + 24 pad): conflict-free operand and transpose reads
constexpr int kWaves128 = 8;    // two wavefronts per SIMD: one wave's LDS / memory waits are covered by the other
constexpr int kF128K = 0;
constexpr int kF128V = kF128K + 128 * kPitch128 * 2;
constexpr int kF128Tiles = kF128V + 128 * kPitch128 * 2;
constexpr int kF128Ent = kF128Tiles + kWaves128 * 32 * kTileStride * 2;
constexpr int kF128Epos = kF128Ent + kMaxUnit * 4;
constexpr int kF128Cnts = kF128Epos + kMaxUnit * 2;
constexpr int kF128Bytes = kF128Cnts + (kMaxUnit / 64) * 4;
static_assert(kF128Bytes <= 160 * 1024, "forward 128-key tile set must fit the CU's LDS");

template <bool kWide, bool kInTurn>
__global__ void __launch_bounds__(64 * kWaves128)
k_fwd_main128(Problem P, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
              const UnitRec* __restrict__ u_rec, const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ off,
              const int2* __restrict__ qent, bf16_t* __restrict__ opart, float* __restrict__ lse_part) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* Ks = reinterpret_cast<bf16_t*>(smem + kF128K);
  bf16_t* Vs = reinterpret_cast<bf16_t*>(smem + kF128V);
  int32_t* ent = reinterpret_cast<int32_t*>(smem + kF128Ent);
  uint16_t* epos = reinterpret_cast<uint16_t*>(smem + kF128Epos);
  int32_t* cnts = reinterpret_cast<int32_t*>(smem + kF128Cnts);
  UnitRec U;
  int pos0;
  if (!load_unit<kInTurn>(P, u_rec, nu_scan, off, U, pos0)) return;
  const int j = U.j, e0 = U.e0, ne_all = U.ne, tok0 = U.tok0, blen = U.blen;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int col = lane & 31, qh = lane >> 5;                 // not const: see the top of the tile loop
  int crow = lane >> 4, cchunk = (lane & 15) * 8;
  bf16_t* tile_lds = reinterpret_cast<bf16_t*>(smem + kF128Tiles) + wave * 32 * kTileStride;
  // K_i, V_i (thread = key, 32 channels), requested before the entries are looked at (see k_fwd_main)
  bf16x8 kreg[4], vreg[4];
  auto load_block = [&]() __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t k_buf = block_buffer(K, P, U), v_buf = block_buffer(V, P, U);
    const uint32_t o = (uint32_t)(tid >> 2) * (uint32_t)P.hkv * (kD * 2) + (tid & 3) * 64;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      kreg[i] = load_frag(k_buf, o + 16 * i);
      vreg[i] = load_frag(v_buf, o + 16 * i);
    }
  };
  const bool late = P.window > 0 && P.dense;
  if (!late) load_block();
  // entries of dense (tile, block) pairs belong to the dense kernel (see load_sparse_entries)
  const int ne = load_sparse_entries<64 * kWaves128>(qent, e0, ne_all, ent, epos, cnts);
  if (ne == 0) return;
  if (late) load_block();
  {
    const int o = (tid >> 2) * kPitch128 + (tid & 3) * 32;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *reinterpret_cast<bf16x8*>(&Ks[o + 8 * i]) = kreg[i];
      *reinterpret_cast<bf16x8*>(&Vs[o + 8 * i]) = vreg[i];
    }
  }
  __syncthreads();

  const int rows_total = ne * P.g;
  const int n_tiles = (rows_total + 31) >> 5;
  if (wave >= n_tiles) return;  // no block-wide barrier below this point
  const float c2 = P.scale * 1.4426950408889634f;
  const int hbase = j * P.g;
  // this lane's share of a transposing read of four key rows x 16 channels; lane half qh = grp / 2 holds keys
  // k0 + 4 qh + {0..3} (first read) and the same + 8 (second read) of contraction step sp, k0 = 32 (sp/2) + 16 (sp&1)
  const int grp = lane >> 4, sl = lane & 15;
  int tr_v = ((sl >> 2) + 4 * (grp >> 1)) * kPitch128 + 16 * (grp & 1) + 4 * (sl & 3);

  const RowTensor<kWide> Qrows(Q, (int64_t)P.T * P.hq);
  const size_t part0 = (size_t)(e0 - pos0) * P.g;  // the unit's first partial row
  const __amdgpu_buffer_rsrc_t o_buf = buffer_of(opart + part0 * kD, (uint32_t)(ne_all * P.g) * (kD * 2));
  const __amdgpu_buffer_rsrc_t l_buf = buffer_of(lse_part + part0, (uint32_t)(ne_all * P.g) * 4);
  auto row_of = [&](int tile) __attribute__((always_inline)) {
    return find_row(P, tile * 32 + col, rows_total, hbase, ent, epos);
  };
  u32x4 qc[8];
  auto issue_q = [&](const GatherRow& x) __attribute__((always_inline)) {
    uint32_t row[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) row[i] = lane_value(x.src, 4 * i + crow);
#pragma unroll
    for (int i = 0; i < 8; ++i) qc[i] = Qrows.load(row[i], cchunk * 2);
  };
  GatherRow cur = row_of(wave), next = row_of(wave + kWaves128);
  issue_q(cur);
  pad_stores<9>(l_buf);
  int tile = wave;
  do {
    // register budget (256 per wave): keep the lane-derived LDS addresses from being precomputed across the loop
    asm volatile("" : "+v"(col), "+v"(qh), "+v"(crow), "+v"(cchunk), "+v"(tr_v));
#pragma unroll
    for (int i = 0; i < 8; ++i)
      *reinterpret_cast<u32x4*>(&tile_lds[(4 * i + crow) * kTileStride + cchunk]) = qc[i];
    issue_q(next);  // next rows fly during this tile's compute
    wave_sync();
    bf16x8 qf[8];
#pragma unroll
    for (int s = 0; s < 8; ++s)
      qf[s] = *reinterpret_cast<const bf16x8*>(&tile_lds[col * kTileStride + 16 * s + 8 * qh]);

    f32x16 sacc[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) sacc[mb][v] = 0.f;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Ks[(32 * mb + col) * kPitch128 + 16 * s + 8 * qh]);
        sacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], sacc[mb], 0, 0, 0);
      }

    const int t = cur.t;
    const bool valid = t >= 0;
    int lim = P.causal ? min(blen, t - tok0 + 1) : blen;
    if (!valid) lim = 0;
    const int lo = P.window > 0 ? t - P.window + 1 - tok0 : 0;  // with a window, keys before lo are hidden
    // key mask only where a row lies in the block itself, the block is ragged or a window edge falls into it (wave-uniform test); maximum over
    // the raw scores, scale folded into the exponent
    float m = -INFINITY;
    if (__builtin_amdgcn_ballot_w64(lim < 2 * kBlock || lo > 0) == 0) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) m = fmaxf(m, sacc[mb][v]);
    } else {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = 32 * mb + 8 * (v >> 2) + 4 * qh + (v & 3);
          const float x = (key < lim && key >= lo) ? sacc[mb][v] : -INFINITY;
          sacc[mb][v] = x;
          m = fmaxf(m, x);
        }
    }
    m = fmaxf(m, __shfl_xor(m, 32));
    const float mc = (m == -INFINITY) ? 0.f : m * c2;  // row maximum in the log2 domain
    float l = 0.f;
    bf16x8 pf[8];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[mb][v], c2, -mc));
        l += p;
        pf[2 * mb + (v >> 3)][v & 7] = (bf16_t)p;
      }
    l += __shfl_xor(l, 32);

    f32x16 oacc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
#pragma unroll
    for (int sp = 0; sp < 8; ++sp) {
      const int k0 = 32 * (sp >> 1) + 16 * (sp & 1);
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const bf16x4 a0 = lds_read_tr(&Vs[k0 * kPitch128 + tr_v + 32 * db]);
        const bf16x4 a1 = lds_read_tr(&Vs[(k0 + 8) * kPitch128 + tr_v + 32 * db]);
        const bf16x8 vf = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[sp], oacc[db], 0, 0, 0);
      }
    }

    const float inv = valid ? 1.f / l : 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        uint2 w;
        w.x = pack_bf16x2(oacc[db][4 * a + 0] * inv, oacc[db][4 * a + 1] * inv);
        w.y = pack_bf16x2(oacc[db][4 * a + 2] * inv, oacc[db][4 * a + 3] * inv);
        *reinterpret_cast<uint2*>(&tile_lds[col * kTileStride + 32 * db + 8 * a + 4 * qh]) = w;
      }
    wave_sync();
    store_partial_rows(tile_lds, cur, valid, crow, cchunk, o_buf);
    store_partial_lse((mc + __builtin_amdgcn_logf(l)) * 0.6931471805599453f, cur, valid && qh == 0, l_buf);
    wave_sync();
    cur = next;
    next = row_of(tile + 2 * kWaves128);
    tile += kWaves128;
  } while (tile < n_tiles);
}

// ---- dense (query-tile-outer) forward, fused with the merge ---------------------------------------------------------
// The (query tile, KV block) pairs the index marked dense - blocks that at least half of the tile's 64 tokens keep:
// the attention-sink block and the tokens' own and neighbouring blocks (App. E, the paragraph on the attention sink;
// the whole band of the sliding-window term of Eq. (2)) - are contiguous token ranges on both sides, so they need no
// gather and no partial row in memory at all.  One workgroup takes 128 rows (row = (token of the tile, head of the
// group)) of one (tile, kv head):
//   phase 1  keeps the rows' Q fragments in registers and walks the tile's dense blocks, 64 keys at a time (the index
//            lists them as pieces) through LDS, with a running (max, sum) per row and the output accumulated in
//            registers across the pieces (dense_piece.h).  The 64-bit mask of a piece says which tokens of the tile keep its
//            block; the others see none of its keys.  K and V go from memory straight to LDS, to two pairs of tiles: a
//            piece's PV product runs beside the next piece's S product, and beside both the K after that and the next V arrive.  The
//            result, normalised, goes to LDS with its log-sum-exp.
//   phase 2  is the reduction step of Sec. 3.2 for the same rows: 16 lanes per row gather the partial rows the gather
//            route left for the row's other kept columns (two rows and up to eight columns at a time per lane: the few
//            wavefronts of this kernel need that many loads in flight) and combine them, together with the row of
//            phase 1, by their log-sum-exps; O, LSE and the optional gated sum of Eq. (2) are written once.  The
//            rows' kept-column masks and slot positions are fetched at the very start of the kernel and parked in
//            LDS, so that phase 2 starts with its addresses known and the only memory latency left in it is that of the
//            gathers themselves.  A row's columns are taken from its bit mask, so that dense ones cost no place in a batch; the
//            finished rows wait in LDS until the workgroup writes them all (see "the two reduction kernels" in common.h).  With
//            the columns in place, plain loads and every row written as it was done: 1.79 instead of 1.62 ms at 65536 tokens, g = 4,
//            1.78 instead of 1.54 with 9 of 16 columns dense at g = 7, 1.02 instead of 0.91 gated at 32768 tokens.
// Tiles without a dense piece skip phase 1, so with the dense route on this kernel is the merge of every row.
// Phase 2 is bound by memory (65536 tokens, g = 4: 8.9 GB in 1.62 ms for the whole kernel), phase 1 by what two
// wavefronts a SIMD issue: for a window of 512 over 32768 tokens, where nothing is left to gather, 15 vector instructions go with a product, the
// matrix pipe is 32 % busy, and the wavefronts wait 29 % of their time; the piece loop itself keeps the pipe busy (see
// piece_values_and_next_scores), the rest is tables, Q, the first piece's scores, the reduction and the write.  One pair of tiles, with two barriers a
// piece and the S product, softmax and PV product one after the other, took 1.55 instead of 1.40 ms with 9 of 16 columns dense at g
// = 7, 65536 tokens, and 532 instead of 514 us for a window of 512 at 32768; there every access of the piece loop also waited for the loads just
// sent on their way (see await_rows).  The last piece goes without scores of a next one, which tiles of one or two pieces paid for with
// what the order gained them: one piece, 32768 tokens, g = 4, own block 310 us with them, 290 without; a window of 100 142 and 139.  Three workgroups per CU leave 168 registers, 30 of them spilled.
// LDS: unpadded, turned rows (see row_turn): 0.55 -> 0.51 ms for a window of
// 512 at 32768 tokens, 6.3 -> 6.1 ms at 131072, g = 8, against a turn of the low three bits, which left the transposing reads at a
// quarter of their rate.  Phase 1's result takes the same area afterwards (place c ^ (r & 15)), and with a gate the gated rows.
constexpr int kDnRow = kD * 2;
constexpr int kDnK = 0;
constexpr int kDnV = kDnK + 2 * kPieceBytes;
constexpr int kDnLse = kDnV + 2 * kPieceBytes;
constexpr int kDnMeta = kDnLse + 4 * 32 * 4;
static_assert(2 * 4 * 32 * kDnRow <= kDnLse, "phase 1's result and the gated rows must fit the K / V area");
// words of phase 2's index data of one wavefront: (kept, dense, positions) of every token its 32 rows can touch
inline __host__ __device__ int dense_meta_words(int g, int topk) { return (31 / g + 2) * (topk + 2); }
inline int dense_lds_bytes(int g, int topk) { return kDnMeta + (g == 1 ? 8 : 16) * dense_meta_words(g, topk); }  // g = 1: two wavefronts have rows
// Columns of a row gathered next in phase 2 when `left` are: at most eight, as few rounds as possible, of like size.  A place in a
// round that no row fills costs nearly as much as a column: 16384 tokens, g = 4, with 15 columns to gather 427 us in rounds of
// seven, 403 as eight and seven; with 14 columns 392 in rounds of seven, 419 as eight and six; with 30 columns 774 in rounds of seven, 759 as
// eight, eight, seven and seven; with 2 columns 212 in a round of seven, 192 in one of four.  Rounds that all rows of a wavefront fill go
// without a branch a column: 386, 386, 751 us with 15 (bidirectional), 14 and 30 columns, and 362 for 382 with 7 local picks of 16.
constexpr int kMergeBatch = 8;
__device__ __forceinline__ int batch_of(int left) {
  constexpr int b = kMergeBatch;
  return left <= b ? left : left <= 2 * b ? (left + 1) / 2 : left <= 3 * b ? (left + 2) / 3 : (left + 3) / 4;
}
static_assert(4 * kMergeBatch >= kMaxTopk, "at most four rounds");

__global__ void __launch_bounds__(256, 2)
k_fwd_dense_merge(Problem P, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
                  const int32_t* __restrict__ tile_tok0, const int32_t* __restrict__ tile_len,
                  const int32_t* __restrict__ d_cnt, const int2* __restrict__ d_piece,
                  const unsigned long long* __restrict__ d_mask, const bf16_t* __restrict__ opart,
                  const float* __restrict__ lse_part, const uint32_t* __restrict__ vmask,
                  const uint32_t* __restrict__ dmask, const int32_t* __restrict__ slotpos,
                  const int32_t* __restrict__ off, bf16_t* __restrict__ O, float* __restrict__ LSE,
                  const float* __restrict__ gate, const bf16_t* Oacc, bf16_t* Oout) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int chunks = (kTileTokens * P.g + 127) >> 7;  // 128-row chunks of a tile's rows
  // Workgroups are handed to the chip's 8 XCDs (each with its own L2) round-robin by their index; the work is
  // ordered kv head -> tile -> chunk, and every XCD takes one contiguous eighth of that order, so that the
  // workgroups running side by side on an XCD share K / V pieces (neighbouring tiles of one head, the sink block).
  const int total = P.nj * P.t_cap * chunks, per = (total + 7) >> 3;
  const int lid = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (lid >= total) return;
  const int chunk = lid % chunks, qt = (lid / chunks) % P.t_cap;
  const int j = P.j0 + lid / (chunks * P.t_cap);
  const size_t slot = (size_t)qt * P.hkv + j;
  // everything the prologue needs from the tables is requested at once: lane i holds the tile's piece i and its member
  // mask (the slots exist whatever the piece count), so that the loop over the pieces waits for no table
  const int nd = d_cnt[slot];
  const int tlen = tile_len[qt];
  const int ttok0 = tile_tok0[qt];
  const int2 my_piece = d_piece[slot * kDenseMax + (threadIdx.x & (kDenseMax - 1))];
  const unsigned long long my_mask = d_mask[slot * kDenseMax + (threadIdx.x & (kDenseMax - 1))];
  const int rows_total = tlen * P.g;
  if (chunk * 128 >= rows_total) return;
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, qh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: what derives from it stays out of the VGPRs
  float* lse_lds = reinterpret_cast<float*>(smem + kDnLse) + wave * 32;
  unsigned char* od_lds = smem + wave * 32 * kDnRow;  // phase 1's result for phase 2 (the K / V area after the last piece)
  const int row0 = chunk * 128 + wave * 32;        // first row of this wavefront
  const bool wave_on = row0 < rows_total;          // idle wavefronts still help to stage K / V
  const int hbase = j * P.g;

  // Phase 2's index data for this wavefront's tokens: per token (kept columns, dense columns, slot positions).
  // Requested now (up to 4 words per lane in registers, the rest - many tokens per wave, long rows - later).
  const int e_lo = div_g(min(row0, rows_total - 1), P.g, P.g_magic);
  const int e_hi = div_g(min(row0 + 31, rows_total - 1), P.g, P.g_magic);
  const int mstride = P.topk + 2;
  const int mwords = wave_on ? (e_hi - e_lo + 1) * mstride : 0;
  int32_t* meta = reinterpret_cast<int32_t*>(smem + kDnMeta) + wave * dense_meta_words(P.g, P.topk);
  auto meta_word = [&](int i) -> int32_t {
    const int tk = i / mstride, c = i - tk * mstride;
    const size_t tj = (size_t)(ttok0 + e_lo + tk) * P.hkv + j;
    return c == 0 ? (int32_t)vmask[tj] : c == 1 ? (int32_t)dmask[tj] : slotpos[tj * P.topk + (c - 2)];
  };
  int32_t mreg[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) mreg[q] = lane + 64 * q < mwords ? meta_word(lane + 64 * q) : 0;
  auto park_meta = [&]() {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (lane + 64 * q < mwords) meta[lane + 64 * q] = mreg[q];
    for (int i = lane + 256; i < mwords; i += 64) meta[i] = meta_word(i);
    wave_sync();
  };

  if (nd > 0) {  // ---------------------------------------------------------------------------------- phase 1
    const float c2 = P.scale * 1.4426950408889634f;
    // Staging goes from memory straight to LDS (no register, no LDS store instruction): access i of a wavefront fills rows
    // 16 i + 4 wave + lane / 16, lane l the place l % 16 of its row, so the lane fetches chunk (l % 16) ^ row_turn(row).
    // Rows past the end of a ragged block lie past the end of the buffer and arrive as zero.
    const int srow = 4 * wave + (lane >> 4);
    const uint32_t row_bytes = (uint32_t)P.hkv * kDnRow;
    const uint32_t stage_off = srow * row_bytes + (((lane & 15) ^ row_turn(srow)) << 4);
    // the rows of piece `step` of K or V; of K past the last piece none: they arrive as zeros
    auto piece_of = [&](const bf16_t* X, int step) __attribute__((always_inline)) {
      const int first = __builtin_amdgcn_readlane(my_piece.x, min(step, nd - 1)), len = __builtin_amdgcn_readlane(my_piece.y, min(step, nd - 1));
      return buffer_of(X + ((size_t)first * P.hkv + j) * kD, step < nd ? (uint32_t)((len - 1) * P.hkv + 1) * kDnRow : 0u);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t buf, int lds_off, int i) __attribute__((always_inline)) {
      uint32_t from = stage_off;
      asm volatile("" : "+v"(from));  // the offsets are not kept in registers
      load_to_lds(buf, lds_address(smem + lds_off) + (16 * i + 4 * wave) * kDnRow, from + 16 * i * row_bytes);
    };
    auto stage = [&](const bf16_t* X, int lds_off, int step) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t buf = piece_of(X, step);
#pragma unroll
      for (int i = 0; i < 4; ++i) load(buf, lds_off, i);
    };
    stage(K, kDnK, 0);
    stage(V, kDnV, 0);
    if (nd > 1) stage(K, kDnK + kPieceBytes, 1);
    // this wavefront's 32 rows of Q as B-operand fragments, kept for the whole tile
    const int r = row0 + col;                        // this lane's row
    const bool valid = r < rows_total;
    const int e_row = div_g(min(r, rows_total - 1), P.g, P.g_magic);
    const int t = ttok0 + e_row;
    bf16x8 qf[8];
    {  // (a wavefront without rows goes along with the last row: it sees no key)
      const uint32_t grow = (uint32_t)t * (uint32_t)P.hq + (uint32_t)(hbase + min(r, rows_total - 1) - e_row * P.g);
      const bf16_t* src = Q + (size_t)grow * kD + 8 * qh;
#pragma unroll
      for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(src + 16 * s);
      park_meta();
    }

    f32x16 oacc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;            // running maximum (raw scores) and sum of the row
    uint32_t kaddr[8], vaddr[2][4];
    piece_addresses(lds_address(smem + kDnK), lds_address(smem + kDnV), lane, kaddr, vaddr);

    await_rows(qf);
    wait_loads();
    __syncthreads();  // the first piece and the second one's K are staged
    f32x16 even[2], odd[2];
    piece_scores(kaddr, qf, even);
    float m = max_scores(even);
    if (nd > 1) __syncthreads();  // every wavefront has read the first K
    // visibility and maximum of piece `step`, whose scores are `cur` (see new_maximum)
    auto prepare = [&](int step, f32x16 (&cur)[2], float& alpha) __attribute__((always_inline)) {
      const unsigned long long members =
          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_mask, step) |
          (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_mask >> 32), step) << 32;
      // first key of the piece and its number of keys
      const int ktok0 = __builtin_amdgcn_readlane(my_piece.x, step), klen = __builtin_amdgcn_readlane(my_piece.y, step);
      // keys [lo, lim) of the piece are visible to this row: none if the token does not keep the block
      int lim = P.causal ? min(klen, t - ktok0 + 1) : klen;
      if (!valid || !((members >> e_row) & 1ull)) lim = 0;
      const int lo = P.window > 0 ? max(t - P.window + 1 - ktok0, 0) : 0;
      const bool sees = lim > lo;
      if (__builtin_amdgcn_ballot_w64(sees && (lim < 64 || lo > 0)) != 0ull) {
        m = mask_scores(cur, lo, lim, qh);
      } else if (__builtin_amdgcn_ballot_w64(!sees) != 0ull) {  // rows see all of the piece or nothing of it
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int v = 0; v < 16; ++v) cur[mb][v] = sees ? cur[mb][v] : -INFINITY;
      }
      return new_maximum(row_max(m), sees, c2, m_run, alpha);
    };
    // every piece but the last: with the scores of the next one
    auto piece = [&](int step, f32x16 (&cur)[2], f32x16 (&next)[2], int side) __attribute__((always_inline)) {
      // this piece's K tile has been read in the step before: K of the piece after the next flies there, V of the next to the
      // other tile
      const __amdgpu_buffer_rsrc_t kbuf = piece_of(K, step + 2), vbuf = piece_of(V, step + 1);
      keep_addresses(kaddr, vaddr);
      uint32_t ka[8], va[2][4];
#pragma unroll
      for (int s = 0; s < 8; ++s) ka[s] = kaddr[s] + (side ^ 1) * kPieceBytes;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        va[0][d] = vaddr[0][d] + side * kPieceBytes;
        va[1][d] = vaddr[1][d] + side * kPieceBytes;
      }
      float alpha;
      const float mc = prepare(step, cur, alpha);
      m = piece_values_and_next_scores(ka, va, qf, c2, mc, alpha, cur, next, l_run, oacc, [&](int i) __attribute__((always_inline)) {
        if (i < 4) load(vbuf, kDnV + (side ^ 1) * kPieceBytes, i);
        else if (i < 8) load(kbuf, kDnK + side * kPieceBytes, i - 4);
      });
      wait_loads();
      __syncthreads();  // this piece has been read, the next one is staged
    };
    for (int step = 0; step + 1 < nd; step += 2) {
      piece(step, even, odd, 0);
      if (step + 2 < nd) {
        piece(step + 1, odd, even, 1);
      } else {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) even[mb] = odd[mb];
      }
    }
    {
      keep_addresses(kaddr, vaddr);
      uint32_t va[2][4];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        va[0][d] = vaddr[0][d] + ((nd - 1) & 1) * kPieceBytes;
        va[1][d] = vaddr[1][d] + ((nd - 1) & 1) * kPieceBytes;
      }
      float alpha;
      const float mc = prepare(nd - 1, even, alpha);
      piece_values(va, c2, mc, alpha, even, l_run, oacc);
      __syncthreads();  // the K / V area is free
    }
    if (wave_on) {
      // the rows' dense result, normalised, and its log-sum-exp (natural log; -inf for a row that keeps none of the
      // tile's dense blocks) -> this wavefront's quarter of the K / V area, where phase 2 picks them up in its own
      // lane layout
      const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          uint2 w;
          w.x = pack_bf16x2(oacc[db][4 * a + 0] * inv, oacc[db][4 * a + 1] * inv);
          w.y = pack_bf16x2(oacc[db][4 * a + 2] * inv, oacc[db][4 * a + 3] * inv);
          *reinterpret_cast<uint2*>(od_lds + col * kDnRow + (((4 * db + a) ^ (col & 15)) << 4) + 8 * qh) = w;
        }
      if (qh == 0) {
        const float mcf = (m_run == -INFINITY) ? 0.f : m_run * c2;
        lse_lds[col] = l_run > 0.f ? (mcf + __builtin_amdgcn_logf(l_run)) * 0.6931471805599453f : -INFINITY;
      }
      wave_sync();
    }
  }
  // ------------------------------------------------------------------------------------------------ phase 2
  // lane-derived indices of this phase, recomputed here so that they do not occupy registers during phase 1
  int lane_b = threadIdx.x & 63;
  asm volatile("" : "+v"(lane_b));
  const int sub = lane_b & 15, crow_b = lane_b >> 4;
  unsigned char* gated_lds = smem + (4 + wave) * 32 * kDnRow;
  if (wave_on) {
    if (nd == 0) park_meta();
    const int pos0 = off[P.j0 * P.b_cap];  // first list position of the pass: partial rows are relative to it
    for (int pass = 0; pass < 4; ++pass) {
      // two rows per lane group: wave rows 4 pass + crow and 16 more
      int hh[2];
      uint32_t vm_all[2], vm[2];
      const int32_t* sp[2];  // the row's slot positions (LDS)
      float acc[2][8], M[2], Ls[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int wrow = 4 * pass + crow_b + 16 * x;
        const int rr = row0 + wrow;
        const bool ok = rr < rows_total;
        const int rc = min(rr, rows_total - 1);
        const int e = div_g(rc, P.g, P.g_magic);
        hh[x] = rc - e * P.g;
        const int32_t* mrow = meta + (e - e_lo) * mstride;
        vm_all[x] = ok ? (uint32_t)mrow[0] : 0u;
        const uint32_t dm = ok ? (uint32_t)mrow[1] : 0u;
        vm[x] = vm_all[x] & ~dm;
        sp[x] = mrow + 2;
        M[x] = -INFINITY;
        Ls[x] = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[x][c] = 0.f;
        if (dm != 0u && nd > 0) {  // the row of phase 1 starts the sum
          const float ls = lse_lds[wrow];
          if (ls > -INFINITY) {
            const uint4 v = *reinterpret_cast<const uint4*>(od_lds + wrow * kDnRow + ((sub ^ (wrow & 15)) << 4));
            M[x] = ls;
            Ls[x] = 1.f;
            acc[x][0] = bf16_lo(v.x); acc[x][1] = bf16_hi(v.x); acc[x][2] = bf16_lo(v.y); acc[x][3] = bf16_hi(v.y);
            acc[x][4] = bf16_lo(v.z); acc[x][5] = bf16_hi(v.z); acc[x][6] = bf16_lo(v.w); acc[x][7] = bf16_hi(v.w);
          }
        }
      }
      int n[2];  // columns of the round
      // the next n[x] <= count columns of both rows; with `all`, exactly count of them
      auto gather = [&](auto count, auto all) __attribute__((always_inline)) {
        constexpr int kBatch = decltype(count)::value;
        u32x4 xv[2][kBatch];
        float ls[2][kBatch];
        int at[2][kBatch];  // position, -1 past the row's last column
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int i = 0; i < kBatch; ++i) {
            const bool on = all || i < n[x];
            at[x][i] = on ? sp[x][__builtin_ctz(vm[x] | 0x80000000u)] : -1;
            if (on) vm[x] &= vm[x] - 1u;
          }
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int i = 0; i < kBatch; ++i) {
            xv[x][i] = u32x4{0, 0, 0, 0};
            ls[x][i] = -INFINITY;
            if (all || at[x][i] >= 0) {
              const size_t pr = (size_t)(at[x][i] - pos0) * P.g + hh[x];
              xv[x][i] = load_streaming(opart + pr * kD + 8 * sub);
              ls[x][i] = lse_part[pr];
            }
          }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          float Mb = M[x];
#pragma unroll
          for (int i = 0; i < kBatch; ++i) Mb = fmaxf(Mb, ls[x][i]);
          if (Mb == -INFINITY) continue;  // no kept column in this batch or before it
          const float rescale = __expf(M[x] - Mb);  // 0 on the first non-empty batch
          Ls[x] *= rescale;
#pragma unroll
          for (int c = 0; c < 8; ++c) acc[x][c] *= rescale;
          M[x] = Mb;
#pragma unroll
          for (int i = 0; i < kBatch; ++i) {
            const float w = __expf(ls[x][i] - Mb);  // exp(-inf) = 0 for columns that are off
            Ls[x] += w;
            acc[x][0] += w * bf16_lo(xv[x][i].x); acc[x][1] += w * bf16_hi(xv[x][i].x);
            acc[x][2] += w * bf16_lo(xv[x][i].y); acc[x][3] += w * bf16_hi(xv[x][i].y);
            acc[x][4] += w * bf16_lo(xv[x][i].z); acc[x][5] += w * bf16_hi(xv[x][i].z);
            acc[x][6] += w * bf16_lo(xv[x][i].w); acc[x][7] += w * bf16_hi(xv[x][i].w);
          }
        }
      };
      // every row takes what its own columns call for, so that its bits do not depend on the wavefront's other rows; where all
      // eight have as many left, as far from the start of a sequence, that is one size and no branch a column
      while (true) {
        const int left0 = __builtin_popcount(vm[0]), left1 = __builtin_popcount(vm[1]);
        const int left = __builtin_amdgcn_readfirstlane(left0);
        const bool even = __builtin_amdgcn_ballot_w64(left0 != left || left1 != left) == 0ull;
        if (even && left == 0) break;
        n[0] = batch_of(left0);
        n[1] = batch_of(left1);
        switch (even ? batch_of(left) : 0) {
          case 8: gather(std::integral_constant<int, 8>{}, std::true_type{}); break;
          case 7: gather(std::integral_constant<int, 7>{}, std::true_type{}); break;
          case 6: gather(std::integral_constant<int, 6>{}, std::true_type{}); break;
          case 5: gather(std::integral_constant<int, 5>{}, std::true_type{}); break;
          case 4: gather(std::integral_constant<int, 4>{}, std::true_type{}); break;
          case 0: gather(std::integral_constant<int, 8>{}, std::false_type{}); break;
          default: gather(std::integral_constant<int, 3>{}, std::false_type{});
        }
      }
      // the finished rows wait in LDS, in the place of phase 1's, until the workgroup writes all of them
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int wrow = 4 * pass + crow_b + 16 * x;
        const bool empty = vm_all[x] == 0u;  // nothing visible: O = 0, LSE = -inf, and the gated sum is what the other branches gave
        const float inv = empty ? 0.f : 1.f / Ls[x];
        const int place = wrow * kDnRow + ((sub ^ (wrow & 15)) << 4);
        const u32x4 o = {pack_bf16x2(acc[x][0] * inv, acc[x][1] * inv), pack_bf16x2(acc[x][2] * inv, acc[x][3] * inv),
                         pack_bf16x2(acc[x][4] * inv, acc[x][5] * inv), pack_bf16x2(acc[x][6] * inv, acc[x][7] * inv)};
        const float lse = empty ? -INFINITY : M[x] + __logf(Ls[x]);
        *reinterpret_cast<u32x4*>(od_lds + place) = o;
        if (sub == 0) lse_lds[wrow] = lse;
        if (gate != nullptr) {
          // Eq. (2): O_out = O_acc + gate * O, from the fp32 result (Oout may be the buffer Oacc points to: every lane
          // reads its own 16 bytes before it writes them)
          const int64_t grow = (int64_t)(ttok0 + div_g(min(row0 + wrow, rows_total - 1), P.g, P.g_magic)) * P.hq + hbase + hh[x];
          const float tau = gate[grow] * inv;
          u32x4 a = {0, 0, 0, 0};
          if (Oacc != nullptr) a = *reinterpret_cast<const u32x4*>(Oacc + grow * kD + 8 * sub);
          if (!empty) {
            a.x = pack_bf16x2(bf16_lo(a.x) + tau * acc[x][0], bf16_hi(a.x) + tau * acc[x][1]);
            a.y = pack_bf16x2(bf16_lo(a.y) + tau * acc[x][2], bf16_hi(a.y) + tau * acc[x][3]);
            a.z = pack_bf16x2(bf16_lo(a.z) + tau * acc[x][4], bf16_hi(a.z) + tau * acc[x][5]);
            a.w = pack_bf16x2(bf16_lo(a.w) + tau * acc[x][6], bf16_hi(a.w) + tau * acc[x][7]);
          }
          *reinterpret_cast<u32x4*>(gated_lds + place) = a;
        }
      }
    }
  }
  __syncthreads();
  if (!wave_on) return;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int wrow = 4 * q + crow_b;
    if (row0 + wrow >= rows_total) break;
    const int e = div_g(row0 + wrow, P.g, P.g_magic);
    const int64_t grow = (int64_t)(ttok0 + e) * P.hq + hbase + (row0 + wrow - e * P.g);
    const int place = wrow * kDnRow + ((sub ^ (wrow & 15)) << 4);
    store_streaming(O + grow * kD + 8 * sub, *reinterpret_cast<const u32x4*>(od_lds + place));
    if (sub == 0) LSE[grow] = lse_lds[wrow];
    if (gate != nullptr) store_streaming(Oout + grow * kD + 8 * sub, *reinterpret_cast<const u32x4*>(gated_lds + place));
  }
}

// The reduction alone (dense route off); rows and workgroups: see "the two reduction kernels" in common.h.  16 lanes per (token,
// head) row, 8 output channels per lane; columns are taken kBatch at a time (see KeptColumns), all their log-sum-exps and rows
// requested before any is used, the positions of the next row before this one's; batches are chained by the usual running-max
// rescale.
template <int kRows, int kThreads, bool kGate>
__global__ void __launch_bounds__(kThreads)
k_fwd_merge(Problem P, const bf16_t* __restrict__ opart, const float* __restrict__ lse_part,
            const int32_t* __restrict__ slotpos, const int32_t* __restrict__ off, bf16_t* __restrict__ O,
            float* __restrict__ LSE, const float* __restrict__ gate, const bf16_t* Oacc, bf16_t* Oout) {
  constexpr int kBatch = 8;  // columns of a row gathered at a time
  const int sub = threadIdx.x & 15;
  const int pos0 = off[P.j0 * P.b_cap];
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // what the workgroup's rows leave with: the sum, LSE, and with a gate the gated sum
  u32x4* const out = reinterpret_cast<u32x4*>(smem) + threadIdx.x;
  u32x4* const gated = out + kRows * kThreads;
  float* const lse = reinterpret_cast<float*>(smem + kRows * kThreads * (kGate ? 32 : 16)) + (threadIdx.x >> 4);
  const ReduceSpan span = reduce_span<kRows, kThreads>(P, blockIdx.x, gridDim.x);
  if (span.count == 0) return;  // the whole workgroup
  ReduceRow R = reduce_row<kThreads>(P, span.first);
  SlotRow slots = load_slots(slotpos, P, R);
#pragma unroll 1
  for (int q = 0; q < span.count; ++q) {
    const ReduceRow R_next = reduce_row<kThreads>(P, span.first + min(q + 1, span.count - 1));
    const SlotRow slots_next = load_slots(slotpos, P, R_next);
    const int64_t row = (int64_t)R.t * P.hq + R.j * P.g + R.hh;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float M = -INFINITY, Ls = 0.f;
    int pos = pos0;  // of the last kept column
    const KeptColumns kept(slots);
    auto gather = [&](int m0, auto all_kept) __attribute__((always_inline)) {
      int at[kBatch];
      u32x4 x[kBatch];
      float ls[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) at[i] = slot_of(slots, m0, i);
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        x[i] = u32x4{0, 0, 0, 0};
        ls[i] = -INFINITY;
        if constexpr (kRows > 1) {
          pos = at[i] >= 0 ? at[i] : pos;
          asm volatile("" : "+v"(at[i]), "+v"(pos));  // keeps the loads free of branches
        } else {
          pos = at[i];
        }
        if (kRows > 1 || all_kept || at[i] >= 0) {
          const size_t pr = (size_t)(uint32_t)(pos - pos0) * (uint32_t)P.g + (uint32_t)R.hh;
          x[i] = load_streaming(opart + pr * kD + 8 * sub);
          ls[i] = lse_part[pr];
        }
      }
      float Mb = M;
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (kRows > 1 && at[i] < 0) {
          x[i] = u32x4{0, 0, 0, 0};
          ls[i] = -INFINITY;
        }
        Mb = fmaxf(Mb, ls[i]);
      }
      const float Mf = Mb == -INFINITY ? 0.f : Mb;  // no kept slot in this batch or before it: all factors below are 0
      const float rescale = __expf(M - Mf);         // 0 on the first non-empty batch
      Ls *= rescale;
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[c] *= rescale;
      M = Mb;
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const float w = __expf(ls[i] - Mf);  // exp(-inf) = 0 for slots that are off
        Ls += w;
        acc[0] += w * bf16_lo(x[i].x); acc[1] += w * bf16_hi(x[i].x);
        acc[2] += w * bf16_lo(x[i].y); acc[3] += w * bf16_hi(x[i].y);
        acc[4] += w * bf16_lo(x[i].z); acc[5] += w * bf16_hi(x[i].z);
        acc[6] += w * bf16_lo(x[i].w); acc[7] += w * bf16_hi(x[i].w);
      }
    };
    for (int m0 = 0; m0 < P.topk; m0 += kBatch) {
      const uint64_t eight = kept.eight_from(m0);
      if (kRows == 1 && eight == KeptColumns::kAll) gather(m0, std::true_type{});
      else if (kRows > 1 || eight != 0) gather(m0, std::false_type{});
    }
    const bool empty = kept.none();  // nothing visible: O = 0, LSE = -inf, and the gated sum is what the other branches gave
    const float inv = empty ? 0.f : 1.f / Ls;
    out[q * kThreads] = u32x4{pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv),
                              pack_bf16x2(acc[4] * inv, acc[5] * inv), pack_bf16x2(acc[6] * inv, acc[7] * inv)};
    if (sub == 0) lse[q * (kThreads / 16)] = empty ? -INFINITY : M + __logf(Ls);
    if constexpr (kGate) {
      // Eq. (2): O_out = O_acc + gate * O, from the fp32 result (Oout may be the buffer Oacc points to: every lane
      // reads its own 16 bytes before it writes them)
      const float tau = gate[row] * inv;
      u32x4 a = {0, 0, 0, 0};
      if (Oacc != nullptr) a = *reinterpret_cast<const u32x4*>(Oacc + row * kD + 8 * sub);
      if (!empty) {
        a.x = pack_bf16x2(bf16_lo(a.x) + tau * acc[0], bf16_hi(a.x) + tau * acc[1]);
        a.y = pack_bf16x2(bf16_lo(a.y) + tau * acc[2], bf16_hi(a.y) + tau * acc[3]);
        a.z = pack_bf16x2(bf16_lo(a.z) + tau * acc[4], bf16_hi(a.z) + tau * acc[5]);
        a.w = pack_bf16x2(bf16_lo(a.w) + tau * acc[6], bf16_hi(a.w) + tau * acc[7]);
      }
      gated[q * kThreads] = a;
    }
    R = R_next;
    slots = slots_next;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    if (q >= span.count) break;
    const ReduceRow R = reduce_row<kThreads>(P, span.first + q);
    if (!R.on) continue;
    const int64_t row = (int64_t)R.t * P.hq + R.j * P.g + R.hh;
    store_streaming(O + row * kD + 8 * sub, out[q * kThreads]);
    if (sub == 0) LSE[row] = lse[q * (kThreads / 16)];
    if constexpr (kGate) store_streaming(Oout + row * kD + 8 * sub, gated[q * kThreads]);
  }
}

hipError_t launch_fwd(const Problem& P0, const IndexLayout& L, int heads_per_pass, const void* Q, const void* K,
                      const void* V, const void* index_ws, void* opart, float* lse_part, void* O, float* LSE,
                      const GateArgs& G, hipStream_t st) {
  IndexPtrs p = index_ptrs(L, const_cast<void*>(index_ws));
  const bool wide = rows_are_wide((int64_t)P0.T * P0.hq);
  const bool in_turn = units_in_turn(P0.T, heads_per_pass, P0.hq, P0.g, P0.bk, P0.causal != 0);  // (far fewer rows than the wide forms are for)
  auto* main64 = in_turn ? k_fwd_main<false, true> : wide ? k_fwd_main<true, false> : k_fwd_main<false, false>;
  auto* main128 = in_turn ? k_fwd_main128<false, true> : wide ? k_fwd_main128<true, false> : k_fwd_main128<false, false>;
  if (P0.dense) {
    static std::atomic<uint64_t> ready_dense;
    const hipError_t e = allow_dynamic_lds((const void*)k_fwd_dense_merge, 80 * 1024, ready_dense);
    if (e != hipSuccess) return e;
  } else {
    static std::atomic<uint64_t> ready_merge[2];
    hipError_t e = allow_dynamic_lds((const void*)(k_fwd_merge<kBurstRows, kBurstThreads, false>),
                                     reduce_lds(kBurstThreads, kBurstRows, 1, true), ready_merge[0]);
    if (e == hipSuccess)
      e = allow_dynamic_lds((const void*)(k_fwd_merge<kBurstRowsGated, kBurstThreads, true>),
                            reduce_lds(kBurstThreads, kBurstRowsGated, 2, true), ready_merge[1]);
    if (e != hipSuccess) return e;
  }
  {
    static std::atomic<uint64_t> ready[6];
    const int form = in_turn ? 2 : wide;
    hipError_t e = P0.bk == 128 ? allow_dynamic_lds((const void*)main128, kF128Bytes, ready[3 + form])
                                : allow_dynamic_lds((const void*)main64, kF64Bytes, ready[form]);
    if (e != hipSuccess) return e;
  }
  // KV heads are processed heads_per_pass at a time; every pass reuses the same partial buffers (the lists of
  // one KV head are contiguous in list-position order, so a pass owns a contiguous range of positions).
  for (int j0 = 0; j0 < P0.hkv; j0 += heads_per_pass) {
    Problem P = P0;
    P.j0 = j0;
    P.nj = min(heads_per_pass, P0.hkv - j0);
    P.l0 = j0 * P.b_cap;
    P.l1 = (j0 + P.nj) * P.b_cap;
    // upper bound of the work units of the pass (the real count is only known on the device)
    const unsigned units_max = (unsigned)(in_turn ? P.nj * units_bound(1, P.b_cap, P.T, P.topk, P.unit)
                                                    : units_bound(P.nj, P.b_cap, P.T, P.topk, P.unit));
    if (P.bk == 128) {
      ProfScope ps(KID_FWD_MAIN, st);
      hipLaunchKernelGGL(main128, dim3(units_max), dim3(64 * kWaves128), kF128Bytes, st, P, (const bf16_t*)Q,
                         (const bf16_t*)K, (const bf16_t*)V, p.u_rec, p.u_nu, p.off, p.qent, (bf16_t*)opart, lse_part);
    } else {
      ProfScope ps(KID_FWD_MAIN, st);
      hipLaunchKernelGGL(main64, dim3(units_max), dim3(256), kF64Bytes, st, P, (const bf16_t*)Q, (const bf16_t*)K,
                         (const bf16_t*)V, p.u_rec, p.u_nu, p.off, p.qent, (bf16_t*)opart, lse_part);
    }
    if (P.dense) {
      // dense pairs and the reduction step in one kernel (every row of the pass's heads)
      const int chunks = (kTileTokens * P.g + 127) / 128;
      const int per = (P.nj * P.t_cap * chunks + 7) / 8;
      ProfScope ps(KID_FWD_DENSE, st);
      hipLaunchKernelGGL(k_fwd_dense_merge, dim3((unsigned)(8 * per)), dim3(256), dense_lds_bytes(P.g, P.topk), st, P, (const bf16_t*)Q,
                         (const bf16_t*)K, (const bf16_t*)V, p.tile_tok0, p.tile_len, p.d_cnt, p.d_piece, p.d_mask,
                         (const bf16_t*)opart, (const float*)lse_part, p.vmask, p.dmask, p.slotpos, p.off, (bf16_t*)O,
                         LSE, G.gate, (const bf16_t*)G.o_acc, (bf16_t*)G.o_out);
    } else {
      ProfScope ps(KID_FWD_MERGE, st);
      auto launch = [&](auto rows, auto threads, auto gated) {
        constexpr int kRows = decltype(rows)::value, kThreads = decltype(threads)::value;
        constexpr bool kGate = decltype(gated)::value;
        hipLaunchKernelGGL((k_fwd_merge<kRows, kThreads, kGate>), dim3(reduce_groups<kRows, kThreads>(P)), dim3(kThreads),
                           reduce_lds(kThreads, kRows, kGate ? 2 : 1, true), st, P, (const bf16_t*)opart,
                           (const float*)lse_part, p.slotpos, p.off, (bf16_t*)O, LSE, G.gate, (const bf16_t*)G.o_acc,
                           (bf16_t*)G.o_out);
      };
      using std::integral_constant;
      const integral_constant<int, kBurstThreads> burst;
      const integral_constant<int, 1> one;
      const integral_constant<int, 256> few;
      if (merge_in_bursts(P, G.gate != nullptr)) {
        if (G.gate != nullptr) launch(integral_constant<int, kBurstRowsGated>{}, burst, std::true_type{});
        else launch(integral_constant<int, kBurstRows>{}, burst, std::false_type{});
      } else {
        if (G.gate != nullptr) launch(one, few, std::true_type{});
        else launch(one, few, std::false_type{});
      }
    }
  }
  return hipGetLastError();
}

}  // namespace nsa
