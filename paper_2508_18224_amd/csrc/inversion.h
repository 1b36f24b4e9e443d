// What the kernels that read the selection tensor share (the inversion in index.hip, the forward of short inputs in short.hip).
#pragma once
#include "common.h"

namespace nsa {

constexpr int kChunkThreads = 64 * kTilesPerChunk;   // of a k_hist / k_scatter workgroup: a wavefront a tile

struct IndexGeom {
  int32_t nseq, T, hkv, k, bk, causal, window, b_cap, t_cap, n_chunks, n_groups, unit, dense;
};

IndexGeom index_geom(const IndexLayout& L);

// The tokens of a wavefront: the first one and their number (0: none); bounds and first global block of their sequence.  In
// a query tile the latter are the same for all lanes; by token they are those of the lane's token (of the last one past it).
struct Tile {
  int tok0, len, c0, c1, bb;
};

// Last block of its sequence the token can keep, -1 if none.  (A token past the last sequence's end lies past its blocks.)
__device__ __forceinline__ int last_block(const IndexGeom& G, const Tile& t, int tok) {
  const int last = (t.c1 - t.c0 + G.bk - 1) / G.bk - 1;
  return G.causal ? min((tok - t.c0) / G.bk, last) : last;
}

// First block of its sequence the token can keep: that of the oldest key a window of G.window tokens shows to it, position
// tok - c0 - window + 1 of its sequence.
__device__ __forceinline__ int first_block(const IndexGeom& G, const Tile& t, int tok) {
  return G.window > 0 ? max(tok - t.c0 - G.window + 1, 0) / G.bk : 0;
}

// One row of idx in registers; columns past k hold -1.
template <int KMAX>
__device__ __forceinline__ void load_row(const int32_t* __restrict__ src, int k, bool vec4, int32_t (&row)[KMAX]) {
  if (vec4) {
#pragma unroll
    for (int m = 0; m < KMAX; m += 4) {
      int4 x = make_int4(-1, -1, -1, -1);
      if (m < k) x = *reinterpret_cast<const int4*>(src + m);
      row[m] = x.x; row[m + 1] = x.y; row[m + 2] = x.z; row[m + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int m = 0; m < KMAX; ++m) row[m] = m < k ? src[m] : -1;
  }
}

__device__ __forceinline__ bool rows_are_vec4(const void* a, int k) {
  return (k & 3) == 0 && (reinterpret_cast<uintptr_t>(a) & 15) == 0;
}

__device__ __forceinline__ void wave_lds_sync() {  // orders a wavefront's own LDS traffic
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// table[x] += 1 for every lane with `on`.  The forced columns (sink, own block) hold the same id in every lane, which
// would serialise 64 atomics on one address: a column all of whose lanes agree is counted by one of them.
__device__ __forceinline__ void count_column(int32_t* table, int x, bool on, int lane) {
  const unsigned long long act = __builtin_amdgcn_ballot_w64(on);
  if (act == 0ull) return;
  const int lead = __builtin_ctzll(act);
  const int x0 = __builtin_amdgcn_readlane(x, lead);
  if (__builtin_amdgcn_ballot_w64(on && x == x0) == act) {
    if (lane == lead) atomicAdd(&table[x0], __popcll(act));
  } else if (on) {
    atomicAdd(&table[x], 1);
  }
}

// Bit m of the result: column m is a kept selection - in range for the sequence, not in the token's future when causal, not
// wholly before the token's window, and not a repeat of an earlier column.
template <int KMAX>
__device__ __forceinline__ uint32_t kept_columns(const IndexGeom& G, const Tile& t, int tok, const int32_t (&row)[KMAX]) {
  uint32_t vm = 0;
  const int first = first_block(G, t, tok), last = last_block(G, t, tok);
#pragma unroll
  for (int m = 0; m < KMAX; ++m) {
    bool dup = false;
#pragma unroll
    for (int mp = 0; mp < m; ++mp) dup |= row[mp] == row[m];
    if (m < G.k && row[m] >= first && row[m] <= last && !dup) vm |= 1u << m;
  }
  return vm;
}

}  // namespace nsa
