// Backward selected-block attention for gfx950.  The paper (Sec. 3.2) only says that the backward pass follows
// the forward's KV-outer logic, gathers the queries again through the cached index tensors and stores
// intermediate query gradients to a buffer that a reduction kernel sums; dK/dV accumulation is not described.
// This file is that pass, with dK/dV accumulated without atomics:
//
//   k_bwd_delta       delta[t,h] = <dO[t,h], O[t,h]>, stored next to LSE[t,h] log2(e) as one 8-byte pair so that the
//                     main kernel fetches both row statistics with one gather
//   k_bwd_tiled       the main kernel for B_K = 64.  One work unit = (kv head j, KV block i, up to
//                     P.unit list entries): four wavefronts and half of a CU's LDS, so two workgroups share a CU and
//                     cover each other's barriers and waits.  The waves share tiles of 64 gathered rows and take three
//                     roles per tile (see the comment above the kernel): S = Q K_i^T, dP = dO V_i^T,
//                     P = exp(S - LSE), dS = P (dP - delta) scale; then dV_i += P^T dO and dK_i += dS^T Q
//                     (accumulators in registers for the whole unit) and dQ^T = K_i^T dS^T.  Operands are row-major
//                     tiles in LDS; "lane = column" operands are LDS transpose reads.  Partial dQ rows go to the
//                     compact buffer at the rows' list position; the unit's dK_i, dV_i go out as bf16 (list fitted
//                     the unit) or to a per-unit fp32 buffer.
//   k_bwd_pipe128     the main kernel for B_K = 128, same work units and outputs.  The fp32 dK_i / dV_i accumulators
//                     of a 128-key block fill the registers of four wavefronts, so one eight-wave workgroup owns the
//                     CU; its waves specialise (four compute P / dS of tile n, four accumulate tile n - 1) instead
//                     of all stepping through the same phases (see the comment above the kernel).
//   k_bwd_dq_reduce   dQ[t,h] = sum over kept slots of the partial rows
//   k_bwd_dkv_reduce  (with k_bwd_dq_reduce) dK_i, dV_i = sum over the list's units in unit order (fixed order: bit-reproducible); a list
//                     that fitted one unit was already written by that unit, a list with no entry gets zeros
#include "common.h"
#include <type_traits>

namespace nsa {

__device__ __forceinline__ void wave_sync_bwd() {  // orders a wavefront's own LDS traffic
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// delta[t, h] = <dO[t, h], O[t, h]> next to LSE[t, h] log2(e).  The pair is gathered by the main kernels once per (pair,
// head), so it is laid out head-major, [kv head][token][head of the group]: one kv head's pairs (8 g bytes a token, 2 MB
// at 65536 tokens and g = 4) stay in an XCD's L2 while the main kernels work on that head.  In token-major order every
// gather of 8 g bytes fetched a line of its own (2 GB per pass at 65536 tokens, 32 kv heads, g = 1).
// A workgroup takes kDeltaTokens tokens x the query heads of kDeltaKv KV heads: rows are read in memory order (16 lanes x 16 bytes a
// row, four rows per lane in flight), the pairs are turned around in LDS and leave as runs of 8 g kDeltaTokens bytes.
constexpr int kDeltaTokens = 8;
constexpr int kDeltaKv = 8;   // kv heads per workgroup: at most 64 query heads

// ---- the order in which the main kernels take the work units -----------------------------------------------------
// With a workgroup a unit the hardware deals the units out to the XCDs in turn, by number: at 65536 tokens, g = 4, the first
// XCD had finished 6 % before the last one, a slot stood empty for 5 us or more between two workgroups, and the sink's long
// units of the last KV head, started last, ran alone at the end (8192 tokens, g = 1: 540 us of work a slot in 660 us).  So where there are several
// units for each of the workgroups that the chip holds, the kernels stay resident, draw their units from a counter, and the long
// units come first.  The first workgroup of k_bwd_delta prepares counters and order in the room of the one unit's dK / dV
// sums that the bound on the number of units always leaves free (a list of c entries has less than c / unit + 1 units).
struct UnitQueue {
  int32_t* next;         // tickets drawn beyond the first one of every workgroup
  const int32_t* order;  // unit by ticket; null: by number
};
constexpr int kQueuePasses = 64;                                                // counters, one a pass over KV heads
constexpr int kQueueUnits = 2 * kBlock * kD - kQueuePasses;                     // entries of the order: 64 KB in all
// Where there is a queue.  Main kernel with a workgroup a unit -> from the queue, in us (tokens x query heads, top-k 16):
//   64-token blocks, causal: 8192 x 32, g = 1 529 -> 503, 32768 x 32, g = 4 2077 -> 1984, 19897 x 26, g = 1 1075 -> 1047, 4096 x 32, g = 4 243 -> 236; but
//     65536 x 32, g = 4 4086 -> 4078 in one run and 4168 -> 4199 in another, 65536 x 28, g = 7 3526 -> 3548: the tail is a small part of so long a kernel,
//     and what the idle slots gave up the others may have had as clock rate (the chip runs these kernels at 1.8 of its 2.4 GHz).  On shorter
//     inputs a KV head with more than half a unit's entries for each slot leaves little of a tail, and the classes go through the heads'
//     Q and dO three times: 27033 x 20, g = 4, top-k 8 527 -> 538, 18046 x 7, g = 1 289 -> 296, 33223 x 20, g = 4, top-k 8 633 -> 656, 34873 x 3 241 -> 250; not so
//     with three units and more for each slot (54612 x 8, g = 4, packed 823 -> 792, 52116 x 4, g = 4 231 -> 224), with lists of four units and more (14455 x 8, g = 2
//     247 -> 237, 14094 x 8, g = 4 228 -> 221) and from g = 5 on (16760 x 10 340 -> 330, 49467 x 5, top-k 32 930 -> 916, at worst 5493 x 50 484 -> 492)
//   all keys, where the lists are alike: with full units and remainders 16384 x 32, g = 4 1049 -> 993, 38968 x 10, g = 2 785 -> 732; lists of one unit
//     (top-k x block entries below 3/4 of it) leave nothing to start early, 31821 x 28, g = 2 1644 -> 1684; packed short documents, lists of several
//     units: 6831 x 26, g = 2 352 -> 362, 16743 x 24, g = 8 733 -> 753, of one 20741 x 18, g = 2 707 -> 686, few heads 40760 x 4, g = 4, top-k 32 600 -> 565
//   windows: 512 over 32768 x 32, g = 4 1155 -> 1117, over 47450 x 32, g = 2 1708 -> 1640, 256 over 30277 x 16, g = 4 419 -> 335; 100 over 25385 x 40, g = 8 349 -> 357
//   128-token blocks, one workgroup a compute unit: window of 512 at 32768 tokens 1455 -> 1123, 8192 x 32, g = 1 532 -> 487, 65536 x 32, g = 4 3240 -> 3188,
//     15810 x 56, g = 4, all keys 1474 -> 1363; at worst +0.6 %
// Fewer units than 2048 are a few a slot: 2000 x 32, g = 4 117 -> 118.
constexpr int kQueueMinUnits = 2048;
inline bool queue_pays(const Problem& P) {
  if (P.bk == 2 * kBlock) return true;
  const int64_t rows = (int64_t)P.T * P.hq * P.topk;  // (token, query head, column) triples
  const int list = P.topk * P.bk;                     // entries of an average list
  const int64_t head = (int64_t)P.T * P.topk, round = 512 * (int64_t)P.unit;  // entries of a KV head, and a unit for each slot
  if (rows > (int64_t)3 << 23) return false;
  if (!P.causal) return 4 * list >= 3 * P.unit && (P.nseq == 1 || rows >= (1 << 23) || list <= P.unit || head >= 4 * round);
  return P.window > 0 || rows >= (1 << 23) || P.g >= 5 || list >= 4 * P.unit || 2 * head <= round || head >= 3 * round;
}

// Units in order of their length class, longest first: more than 3/8, 3/16 and less of a full unit.  A thread takes a run of units,
// so that a class stays in the order of the KV heads, whose Q, dO and statistics the main kernels find in L2; the lengths are read once,
// 16 at a time, and kept as classes of two bits.  Lists of like length (no causal mask) have about top-k x block entries, for units of
// a power of two mostly a power of two of a unit too: the classes part where such lists don't, at 1/2 and 1/4 they went through the heads
// once for each class (32768 tokens, g = 4, all keys: 1855 us with a workgroup a unit, 1980 so).
__device__ __forceinline__ void prepare_queue(const Problem& P, const UnitRec* __restrict__ u_rec, const int32_t* __restrict__ nu_scan,
                                              int32_t* __restrict__ queue, bool ordered) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < kQueuePasses) queue[tid] = 0;
  if (!ordered) return;
  const int n = min(nu_scan[P.hkv * P.b_cap], kQueueUnits);
  const int per = (n + 255) / 256, first = tid * per, mine = max(0, min(per, n - first));
  constexpr int kB = 16, kMost = (kQueueUnits + 255) / 256;
  static_assert(kMost <= 4 * kB, "four words of classes a thread");
  uint32_t cls[4] = {0, 0, 0, 0};
  uint64_t counts = 0;  // of the three classes, 21 bits each
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    if (b * kB >= per) break;
    int ne[kB];
#pragma unroll
    for (int i = 0; i < kB; ++i) ne[i] = u_rec[min(first + b * kB + i, n - 1)].ne;
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const uint32_t c = 8 * ne[i] > 3 * P.unit ? 0 : 16 * ne[i] > 3 * P.unit ? 1 : 2;
      cls[b] |= c << (2 * i);
      if (b * kB + i < mine) counts += (uint64_t)1 << (21 * c);
    }
  }
  uint64_t before = counts;  // of the threads up to this one
#pragma unroll
  for (int d = 1; d < 64; d *= 2) {
    const uint64_t x = __shfl_up((unsigned long long)before, d);
    if (lane >= d) before += x;
  }
  __shared__ uint64_t wave_sum[4];
  if (lane == 63) wave_sum[wave] = before;
  __syncthreads();
  before -= counts;
  uint64_t all = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) before += wave_sum[w];
    all += wave_sum[w];
  }
  constexpr uint64_t kMask = (1 << 21) - 1;
  const int n0 = (int)(all & kMask), n1 = (int)(all >> 21 & kMask);
  int at0 = (int)(before & kMask), at1 = n0 + (int)(before >> 21 & kMask), at2 = n0 + n1 + (int)(before >> 42);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    if (b * kB >= per) break;
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      if (b * kB + i >= mine) break;
      const uint32_t c = cls[b] >> (2 * i) & 3;
      queue[kQueuePasses + (c == 0 ? at0 : c == 1 ? at1 : at2)] = first + b * kB + i;
      at0 += c == 0;
      at1 += c == 1;
      at2 += c == 2;
    }
  }
}

__global__ void __launch_bounds__(256)
k_bwd_delta(Problem P, const bf16_t* __restrict__ O, const bf16_t* __restrict__ dO, const float* __restrict__ LSE,
            float2* __restrict__ stats, const float* __restrict__ gate, float* __restrict__ dgate, const UnitRec* __restrict__ u_rec,
            const int32_t* __restrict__ nu_scan, int32_t* __restrict__ queue, bool ordered) {
  __shared__ float deltas[kDeltaTokens * kDeltaKv * 8];
  if (queue != nullptr && blockIdx.x == 0) {
    if (blockIdx.y == 0) prepare_queue(P, u_rec, nu_scan, queue, ordered);
    return;
  }
  const int t0 = (blockIdx.x - (queue != nullptr)) * kDeltaTokens, j0 = blockIdx.y * kDeltaKv;
  const int nt = min(kDeltaTokens, P.T - t0), nj = min(kDeltaKv, P.hkv - j0), nh = nj * P.g;
  const int sub = threadIdx.x & 15, rows = nt * nh;
  constexpr int kB = 4, kOut = kDeltaTokens * kDeltaKv * 8 / 256;
  // the pairs this thread writes, in (kv head, token, head of the group) order; their LSE is requested before the rows
  int from[kOut];
  int64_t row_out[kOut];
  size_t to[kOut];
  float lse2[kOut];
#pragma unroll
  for (int q = 0; q < kOut; ++q) {
    const int i = min((int)threadIdx.x + 256 * q, rows - 1);
    const int jl = i / (nt * P.g), rem = i - jl * nt * P.g, tt = rem / P.g, hh = rem - tt * P.g;
    from[q] = tt * nh + jl * P.g + hh;
    row_out[q] = (int64_t)(t0 + tt) * P.hq + (j0 + jl) * P.g + hh;
    to[q] = ((size_t)(j0 + jl) * P.T + t0 + tt) * P.g + hh;
    lse2[q] = LSE[row_out[q]] * 1.4426950408889634f;
  }
  for (int r0 = threadIdx.x >> 4; r0 < rows; r0 += 16 * kB) {
    uint4 a[kB], b[kB];
    int64_t row[kB];
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const int r = min(r0 + 16 * i, rows - 1), tt = r / nh;
      row[i] = (int64_t)(t0 + tt) * P.hq + j0 * P.g + (r - tt * nh);
      a[i] = *reinterpret_cast<const uint4*>(O + row[i] * kD + 8 * sub);
      b[i] = *reinterpret_cast<const uint4*>(dO + row[i] * kD + 8 * sub);
    }
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      float acc = bf16_lo(a[i].x) * bf16_lo(b[i].x) + bf16_hi(a[i].x) * bf16_hi(b[i].x) +
                  bf16_lo(a[i].y) * bf16_lo(b[i].y) + bf16_hi(a[i].y) * bf16_hi(b[i].y) +
                  bf16_lo(a[i].z) * bf16_lo(b[i].z) + bf16_hi(a[i].z) * bf16_hi(b[i].z) +
                  bf16_lo(a[i].w) * bf16_lo(b[i].w) + bf16_hi(a[i].w) * bf16_hi(b[i].w);
      acc += __shfl_xor(acc, 8);
      acc += __shfl_xor(acc, 4);
      acc += __shfl_xor(acc, 2);
      acc += __shfl_xor(acc, 1);
      if (sub == 0 && r0 + 16 * i < rows) deltas[r0 + 16 * i] = acc;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kOut; ++q) {
    if ((int)threadIdx.x + 256 * q >= rows) break;
    const float delta = deltas[from[q]];
    if (gate != nullptr) {
      // Gated output (Eq. (2)): the gradient that reaches this branch is gate * dO.  Every place the main kernel
      // uses it carries a factor P = exp2(s - lse2) (dV += P^T dO, dS = P (dP - delta)), so the gate is folded into
      // the row's log-sum-exp, lse2 - log2(gate), and dO and delta stay as they are; a zero gate gives +inf, P = 0.
      // d(loss)/d(gate) is the same <dO, O> as delta.
      if (lse2[q] > -INFINITY) lse2[q] -= log2f(gate[row_out[q]]);
      dgate[row_out[q]] = delta;
    }
    stats[to[q]] = make_float2(lse2[q], delta);
  }
}

// ---- the tiled backward main kernel ----------------------------------------------------------------------------
// B_K = 64: four wavefronts (256 registers each) and half of a CU's LDS, so TWO workgroups share a CU and run out of
// phase: one's barriers, gather waits, unit prologue and LDS-bound phases are covered by the other's MFMA work (with one
// eight-wave workgroup per CU all waves sat in the same phase, and LDS, MFMA and VALU time simply added up).
// Tiles of 64 gathered rows; per tile, wave (rb = w / 2, kb = w % 2) takes three roles in turn:
//   rows/keys   S = Q K_i^T, dP = dO V_i^T, P, dS for rows 32 rb.. and keys 32 kb..; K_i fragments from LDS, V_i fragments
//               of the wave's 32 keys held in registers for the whole unit (only this role uses V_i).  The products are
//               taken with lane = key, so that a lane holds four consecutive rows of P^T / dS^T per register quad (one
//               8-byte LDS store); the rows' statistics come from a record per row that the staging waves leave in LDS
//   keys/chans  dV_i, dK_i accumulators for keys 32 rb.. and channels 64 kb.. (two 32-channel blocks share every
//               P^T / dS^T operand read)
//   rows/chans  dQ^T for rows 32 rb.. and channels 64 kb..; the same wave stages / prefetches that part of the Q and dO
//               tiles and stores that part of dQ
// K_i, Q, dO (turned rows of 256 bytes, see row_turn) and P^T, dS^T (144-byte pitch) are row-major tiles in LDS; "lane =
// column" operands are LDS transpose reads.  The products start from
// zero and the row statistics come in afterwards, P = 2^(S scale log2 e - LSE), dS = P (dP scale - delta scale): partial sums of S that
// start from -LSE / scale carry a term several times their size (the error of P before it is rounded to bf16 doubles) and are no
// faster (4.07 and 4.08 ms at 65536 tokens, g = 4).  Keys are hidden in a branch that tiles seeing the whole block skip.  The list's token ids are kept in LDS 1024
// entries at a time.
// A row's place in memory is worked out once, by the lane that owns it, one tile before its loads are issued, and handed
// to the lanes that move it; rows move through buffer instructions without branches (see RowTensor), so the wait for a
// tile's rows does not wait for the stores of the tile before.  That took 40 % of the vector instructions out of the loop
// and a full drain of the memory queue out of every tile: 4.59 -> 4.2 ms at 65536 tokens, g = 4.  What bounds the kernel is on
// the CU, LDS first (with the gathers served by one XCD's L2 and the stores dropped it still took 3.7 ms of 4.4): the turned
// rows in place of a 304-byte pitch and the masks in a branch together took 4.30 -> 3.98 ms (8192 tokens, g = 1: 568 -> 542 us; g = 7,
// 65536 tokens: 3.73 -> 3.42 ms).  Staging the next tile before the dQ rows are stored,
// through the P^T / dS^T area, gave nothing (g = 1: +4 %).
constexpr int kTile = 64;      // rows per tile
constexpr int kPStride = 72;   // bf16 per row of the P^T / dS^T tiles: 64 rows + 8 pad
constexpr int kEntSeg = 1024;  // list entries whose token ids are resident in LDS

struct BwdLds {
  static constexpr int Row = kD * 2;
  static constexpr int K = 0;
  static constexpr int Q = K + 64 * Row;
  static constexpr int DO = Q + kTile * Row;
  static constexpr int Pt = DO + kTile * Row;
  static constexpr int DSt = Pt + 64 * kPStride * 2;
  static constexpr int Ent = DSt + 64 * kPStride * 2;
  static constexpr int Rec = Ent + kEntSeg * 4;      // per row of the tile: LSE (log2 domain), delta * scale, visible keys
  static constexpr int Next = Rec + 3 * kTile * 4;   // the unit after this one, two words in turn
  static constexpr int Bytes = Next + 16;            // 72464
};
static_assert(2 * BwdLds::Bytes <= 160 * 1024, "two workgroups of the 64-key backward must fit one CU's LDS");

// A workgroup's way through the units (the same in all its threads).  kQueue: one after the other from the queue; otherwise the unit of
// its number alone, in a kernel without the loop: what the loop carries round costs registers, and the forms that have none to spare spill
// them (k_bwd_pipe128 with 64-bit row addresses: 12 bytes a lane).
template <bool kQueue>
struct UnitTurn {
  const Problem& P;
  const UnitQueue q;
  int32_t* const next;  // two words of LDS in turn: a wavefront may read one while the first already writes the other
  UnitRec only;
  int base, count, pos0, ticket, par, unit;
  __device__ __forceinline__ UnitTurn(const Problem& P_, const UnitRec* __restrict__ u_rec, const int32_t* nu_scan, const int32_t* off,
                                      const UnitQueue& q_, int32_t* next_)
      : P(P_), q(q_), next(next_), ticket((int)blockIdx.x), par(0) {
    if constexpr (!kQueue) {
      unit = load_unit<false>(P, u_rec, nu_scan, off, only, pos0) ? ticket : -1;
    } else {
      base = P.l0 > 0 ? nu_scan[P.l0] : 0;
      pos0 = P.j0 > 0 ? off[P.j0 * P.b_cap] : 0;
      count = nu_scan[P.l1] - base;
      unit = ticket >= count ? -1 : q.order != nullptr ? q.order[ticket] : ticket;
    }
  }
  __device__ __forceinline__ UnitRec record(const UnitRec* __restrict__ u_rec) const {
    if constexpr (!kQueue) return only;
    UnitRec U;
    const int4 a = *reinterpret_cast<const int4*>(u_rec + base + unit);
    const int2 b = *reinterpret_cast<const int2*>(&u_rec[base + unit].j);
    U.e0 = a.x; U.ne = a.y; U.tok0 = a.z; U.blen = a.w; U.j = b.x; U.n_units = b.y;
    asm volatile("" : "+s"(U.e0), "+s"(U.ne), "+s"(U.tok0), "+s"(U.blen), "+s"(U.j), "+s"(U.n_units));  // requested here
    return U;
  }
  // Once a unit, between its first requests and its first block-wide barrier.
  __device__ __forceinline__ void draw() {
    if constexpr (!kQueue) return;
    if (threadIdx.x == 0) {
      const int t = (int)gridDim.x + atomicAdd(q.next, 1);
      next[par] = t >= count ? -1 : q.order != nullptr ? q.order[t] : t;
    }
  }
  __device__ __forceinline__ void advance() {  // with a block-wide barrier: the unit's LDS is free after it
    if constexpr (!kQueue) {
      unit = -1;
      return;
    }
    __syncthreads();
    unit = __builtin_amdgcn_readfirstlane(next[par]);
    par ^= 1;
  }
};

template <bool kWin, bool kWide, bool kQueue>
__global__ void __launch_bounds__(256, 2)
k_bwd_tiled(Problem P, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
            const bf16_t* __restrict__ dO, const float2* __restrict__ stats, const UnitRec* __restrict__ u_rec,
            const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ off, const int2* __restrict__ qent,
            bf16_t* __restrict__ dqpart, float* __restrict__ dkv_part, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV,
            UnitQueue queue) {
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  int32_t* ent = reinterpret_cast<int32_t*>(smem + BwdLds::Ent);
  UnitTurn<kQueue> turn(P, u_rec, nu_scan, off, queue, reinterpret_cast<int32_t*>(smem + BwdLds::Next));
  const int pos0 = turn.pos0;
  for (; turn.unit >= 0; turn.advance()) {  // (once without the queue)
  const UnitRec U = turn.record(u_rec);
  constexpr int kRow = BwdLds::Row;
  const int j = U.j, ne = U.ne, tok0 = U.tok0, blen = U.blen;
  int tid = threadIdx.x;
  if constexpr (kQueue) asm volatile("" : "+v"(tid));  // keeps what depends on it inside the loop over units
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, qh = lane >> 5, rb = wave >> 1, kb = wave & 1;
  const uint32_t hbase = (uint32_t)(j * P.g), row_bytes = (uint32_t)P.hkv * (kD * 2);

  // first segment's token ids, K_i (thread = key, 32 channels) and V_i fragments: all requested before any is waited for
  int ids[kEntSeg / 256];
#pragma unroll
  for (int i = 0; i < kEntSeg / 256; ++i) ids[i] = tid + 256 * i < ne ? qent[U.e0 + tid + 256 * i].x : 0;
  bf16x8 kreg[4], vf[8];
  {
    const __amdgpu_buffer_rsrc_t k_buf = block_buffer(K, P, U), v_buf = block_buffer(V, P, U);
#pragma unroll
    for (int i = 0; i < 4; ++i) kreg[i] = load_frag(k_buf, (tid >> 2) * row_bytes + (tid & 3) * 64 + 16 * i);
#pragma unroll
    for (int s = 0; s < 8; ++s) vf[s] = load_frag(v_buf, (32 * kb + col) * row_bytes + 16 * qh + 32 * s);
  }
  turn.draw();
#pragma unroll
  for (int i = 0; i < kEntSeg / 256; ++i) ent[tid + 256 * i] = ids[i];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    *reinterpret_cast<bf16x8*>(smem + BwdLds::K + (tid >> 2) * kRow + (((4 * (tid & 3) + i) ^ row_turn(tid >> 2)) << 4)) = kreg[i];

  f32x16 dkacc[2], dvacc[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      dkacc[cb][v] = 0.f;
      dvacc[cb][v] = 0.f;
    }
  const float c2 = P.scale * 1.4426950408889634f;
  constexpr uint32_t kAllSeen = kWin ? 64u << 16 : 64u;

  // this lane's places in the LDS tiles (everything else is an immediate offset)
  const int grp = lane >> 4, sl = lane & 15, srow = lane >> 3;
  const uint32_t lds = lds_address(smem);
  const uint32_t stage = lds + BwdLds::Q + (32 * rb + srow) * kRow + (((8 * kb + (lane & 7)) ^ row_turn(srow)) << 4);
  const uint32_t frag = col * kRow + ((qh ^ row_turn(col)) << 4);
  uint32_t qfrag = lds + BwdLds::Q + 32 * rb * kRow + frag, kfrag = lds + BwdLds::K + 32 * kb * kRow + frag;
  const float* const rec_rd = reinterpret_cast<const float*>(smem + BwdLds::Rec) + 32 * rb + 4 * qh;
  float* const rec_wr = reinterpret_cast<float*>(smem + BwdLds::Rec) + 32 * rb + col;
  unsigned char* const pt_wr = smem + BwdLds::Pt + (32 * kb + col) * (kPStride * 2) + (32 * rb + 4 * qh) * 2;
  const unsigned char* const pt_rd = smem + BwdLds::Pt + (32 * rb + col) * (kPStride * 2) + 16 * qh;
  // transposing reads of four rows x 16 columns (see lds_read_tr), for the two row pitches
  const int tr_r = (sl >> 2) + 8 * (grp >> 1);
  uint32_t tr_row = lds + tr_r * kRow + (((8 * kb + 2 * (grp & 1) + ((sl & 3) >> 1)) ^ row_turn(tr_r)) << 4) + 8 * (sl & 1);
  const bf16_t* const tr_ds = reinterpret_cast<const bf16_t*>(smem + BwdLds::DSt) +
                              ((sl >> 2) + 8 * (grp >> 1)) * kPStride + 16 * (grp & 1) + 4 * (sl & 3) + 32 * rb;
  uint32_t dq_wr = lds + BwdLds::Q + (32 * rb + col) * kRow + (((8 * kb) ^ row_turn(col)) << 4) + 8 * qh;
  constexpr int kDoOff = BwdLds::DO - BwdLds::Q, kDsOff = BwdLds::DSt - BwdLds::Pt;

  const RowTensor<kWide> Qrows(Q, (int64_t)P.T * P.hq), dOrows(dO, (int64_t)P.T * P.hq);
  const uint32_t lane_off = 128 * kb + 16 * (lane & 7);  // 8 lanes cover the wave's 64 channels of a row
  u32x4 qc[4], dc[4];
  const float2* const head_stats = stats + (size_t)j * P.T * P.g;
  float2 st;                // (LSE in the log2 domain, delta) of row col
  int seg0 = 0, rows_end = 0;

  // Row 32 rb + col of the tile at row tile0 of the unit: its (token, head) row in Q / dO (in 32 bits: total_tokens * hq <
  // 2^31 is checked on the host), its place in the kv head's statistics and the keys of the block it sees.  Rows past the end of the list re-read its
  // last row: they see no key, so their P and dS are zero, and their dQ is dropped by the store.
  auto find_row = [&](int tile0, uint32_t& row, uint32_t& sidx, uint32_t& vis) __attribute__((always_inline)) {
    const int r = tile0 + 32 * rb + col, rc = min(r, rows_end - 1);
    const int e = div_g(rc, P.g, P.g_magic);
    const int t = ent[e - seg0];
    const uint32_t hh = (uint32_t)(rc - e * P.g);
    row = (uint32_t)t * (uint32_t)P.hq + hbase + hh;
    sidx = (uint32_t)t * (uint32_t)P.g + hh;
    int lim = P.causal ? min(blen, t - tok0 + 1) : blen;  // keys [lo, lim)
    if (r >= rows_end) lim = 0;
    if constexpr (kWin) {
      const int lo = min(max(t - P.window + 1 - tok0, 0), 64);
      vis = (uint32_t)(lo | (max(lim - lo, 0) << 16));
    } else {
      vis = (uint32_t)lim;
    }
  };
  auto issue_rows = [&](uint32_t row, uint32_t sidx) __attribute__((always_inline)) {
    uint32_t r4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r4[i] = lane_value(row, 8 * i + srow);
    st = head_stats[sidx];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      qc[i] = Qrows.load(r4[i], lane_off);
      dc[i] = dOrows.load(r4[i], lane_off);
    }
  };
  // the unit's partial dQ rows, one tile at a time: stores past the tile's last row are dropped
  bf16_t* const dq_unit = dqpart + (size_t)(U.e0 - pos0) * P.g * kD;
  const uint32_t dq_lane = (32 * rb + srow) * (kD * 2) + lane_off;

  for (seg0 = 0; seg0 < ne; seg0 += kEntSeg) {
    const int seg_n = min(kEntSeg, ne - seg0);
    if (seg0 > 0) {
      __syncthreads();  // the previous segment's ids are no longer read
      for (int i = tid; i < seg_n; i += 256) ent[i] = qent[U.e0 + seg0 + i].x;
    }
    __syncthreads();  // ids (and K_i on the first pass) visible
    rows_end = (seg0 + seg_n) * P.g;
    uint32_t row_n, sidx_n, vis_c, vis_n;
    find_row(seg0 * P.g, row_n, sidx_n, vis_c);
    issue_rows(row_n, sidx_n);
    find_row(seg0 * P.g + kTile, row_n, sidx_n, vis_n);
    pad_stores<4>(buffer_of(dq_unit, 0));
    int tile0 = seg0 * P.g;
    do {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t to = (stage ^ (32 * (i & 1))) + 8 * i * kRow;
        lds_write_16(to, qc[i]);
        lds_write_16(to + kDoOff, dc[i]);
      }
      if (kb == 0 && qh == 0) {  // this row's record, for the lanes of the rows/keys role (which hold keys, not rows)
        rec_wr[0] = st.x;
        rec_wr[kTile] = st.y * P.scale;
        reinterpret_cast<uint32_t*>(rec_wr)[2 * kTile] = vis_c;
      }
      // the reads below are these addresses with bits flipped and immediate offsets added
      asm volatile("" : "+v"(qfrag), "+v"(kfrag), "+v"(tr_row), "+v"(dq_wr));
      const bool part_seen = __builtin_amdgcn_ballot_w64(vis_c != kAllSeen) != 0ull;  // some row does not see the whole block
      issue_rows(row_n, sidx_n);  // the next tile's rows fly while this one computes (past the last: its last row, unused)
      vis_c = vis_n;
      __syncthreads();  // Q / dO tile and the row records staged by all waves

      {  // role rows/keys: S = Q K_i^T, dP = dO V_i^T for rows 32 rb.. x keys 32 kb..: lane = key, register v = row
         // 8 (v >> 2) + 4 qh + (v & 3), so four consecutive rows of P^T / dS^T leave each lane as one 8-byte LDS store
        f32x16 sacc, dpacc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sacc[v] = dpacc[v] = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const bf16x8 qf = lds_read_frag(qfrag ^ (32 * s));
          const bf16x8 dof = lds_read_frag((qfrag ^ (32 * s)) + kDoOff);
          const bf16x8 kfa = lds_read_frag(kfrag ^ (32 * s));
          sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kfa, sacc, 0, 0, 0);
          dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dof, vf[s], dpacc, 0, 0, 0);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const f32x4 lse4 = *reinterpret_cast<const f32x4*>(rec_rd + 8 * a);
#pragma unroll
          for (int c = 0; c < 4; ++c) sacc[4 * a + c] = __builtin_amdgcn_exp2f(fmaf(sacc[4 * a + c], c2, -lse4[c]));
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {  // (dP - delta) scale, ahead of the branch so that the reads run beside the products
          const f32x4 dls4 = *reinterpret_cast<const f32x4*>(rec_rd + kTile + 8 * a);
#pragma unroll
          for (int c = 0; c < 4; ++c) dpacc[4 * a + c] = fmaf(dpacc[4 * a + c], P.scale, -dls4[c]);
        }
        if (part_seen) {
          const uint32_t key = 32 * kb + col;
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const u32x4 vis4 = *reinterpret_cast<const u32x4*>(rec_rd + 2 * kTile + 8 * a);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const bool seen = kWin ? key - (vis4[c] & 0xffffu) < (vis4[c] >> 16) : (int)key < (int)vis4[c];
              sacc[4 * a + c] = seen ? sacc[4 * a + c] : 0.f;
            }
          }
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          float p[4], ds[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            p[c] = sacc[4 * a + c];
            ds[c] = p[c] * dpacc[4 * a + c];
          }
          uint2 pw, sw2;
          pw.x = pack_bf16x2(p[0], p[1]);
          pw.y = pack_bf16x2(p[2], p[3]);
          sw2.x = pack_bf16x2(ds[0], ds[1]);
          sw2.y = pack_bf16x2(ds[2], ds[3]);
          *reinterpret_cast<uint2*>(pt_wr + 16 * a) = pw;
          *reinterpret_cast<uint2*>(pt_wr + kDsOff + 16 * a) = sw2;
        }
      }
      __syncthreads();  // P^T, dS^T complete
      find_row(tile0 + 2 * kTile, row_n, sidx_n, vis_n);
      {  // role keys/chans: dV_i += P^T dO, dK_i += dS^T Q for keys 32 rb.., channels 64 kb + 32 cb..
#pragma unroll
        for (int qs = 0; qs < 4; ++qs) {
          const bf16x8 pa = *reinterpret_cast<const bf16x8*>(pt_rd + 32 * qs);
          const bf16x8 sa = *reinterpret_cast<const bf16x8*>(pt_rd + kDsOff + 32 * qs);
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) {
            const uint32_t lo = (tr_row ^ (64 * cb)) + BwdLds::Q + 16 * qs * kRow;  // four rows, and the four below
            const uint32_t hi = (tr_row ^ (64 * cb + 16)) + BwdLds::Q + (16 * qs + 4) * kRow;
            const bf16x4 d0 = lds_read_tr_at(lo + kDoOff), d1 = lds_read_tr_at(hi + kDoOff);
            const bf16x4 q0 = lds_read_tr_at(lo), q1 = lds_read_tr_at(hi);
            const bf16x8 dob = __builtin_shufflevector(d0, d1, 0, 1, 2, 3, 4, 5, 6, 7);
            const bf16x8 qb = __builtin_shufflevector(q0, q1, 0, 1, 2, 3, 4, 5, 6, 7);
            dvacc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa, dob, dvacc[cb], 0, 0, 0);
            dkacc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa, qb, dkacc[cb], 0, 0, 0);
          }
        }
      }
      f32x16 dqacc[2];
      {  // role rows/chans: dQ^T[64 kb.., 32 rb..] = K_i^T dS^T over the block's keys
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
          for (int v = 0; v < 16; ++v) dqacc[db][v] = 0.f;
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) {
          const bf16x4 b0 = lds_read_tr(tr_ds + 16 * sp * kPStride), b1 = lds_read_tr(tr_ds + (16 * sp + 4) * kPStride);
          const bf16x8 dsb = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
          for (int db = 0; db < 2; ++db) {
            const bf16x4 a0 = lds_read_tr_at((tr_row ^ (64 * db)) + BwdLds::K + 16 * sp * kRow);
            const bf16x4 a1 = lds_read_tr_at((tr_row ^ (64 * db + 16)) + BwdLds::K + (16 * sp + 4) * kRow);
            const bf16x8 ktf = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
            dqacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktf, dsb, dqacc[db], 0, 0, 0);
          }
        }
      }
      __syncthreads();  // every wave is done reading the Q / dO / P^T / dS^T tiles
      // dQ rows (32 rows x 64 channels) -> the part of the Q tile this wave staged -> contiguous row segments
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          uint2 w;
          w.x = pack_bf16x2(dqacc[db][4 * a + 0], dqacc[db][4 * a + 1]);
          w.y = pack_bf16x2(dqacc[db][4 * a + 2], dqacc[db][4 * a + 3]);
          lds_write_8(dq_wr ^ (64 * db + 16 * a), w);
        }
      wave_sync_bwd();
      const __amdgpu_buffer_rsrc_t dq_buf =
          buffer_of(dq_unit + (size_t)tile0 * kD, (uint32_t)min(rows_end - tile0, kTile) * (kD * 2));
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(lds_read_16((stage ^ (32 * (i & 1))) + 8 * i * kRow), dq_buf,
                                               dq_lane + 8 * i * (kD * 2), 0, kNonTemporal);
      wave_sync_bwd();
      tile0 += kTile;
    } while (tile0 < rows_end);
  }

  if (U.n_units == 1) {
    // the whole list fitted this unit: dK_i, dV_i are final, write them as bf16 (keys of a ragged tail excluded)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      bf16_t* outk = dK + ((size_t)tok0 * P.hkv + j) * kD + 64 * kb + 32 * cb + col;
      bf16_t* outv = dV + ((size_t)tok0 * P.hkv + j) * kD + 64 * kb + 32 * cb + col;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = 32 * rb + 8 * (v >> 2) + 4 * qh + (v & 3);
        if (key < blen) {
          outk[(size_t)key * P.hkv * kD] = (bf16_t)dkacc[cb][v];
          outv[(size_t)key * P.hkv * kD] = (bf16_t)dvacc[cb][v];
        }
      }
    }
    continue;
  }
  // unit partial: [u][0 = dK, 1 = dV][key][d] fp32, summed by k_bwd_dkv_reduce in unit order
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    float* outk = dkv_part + (size_t)(kQueue ? turn.unit : (int)blockIdx.x) * 2 * 64 * kD + 64 * kb + 32 * cb + col;
    float* outv = outk + 64 * kD;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = 32 * rb + 8 * (v >> 2) + 4 * qh + (v & 3);
      outk[key * kD] = dkacc[cb][v];
      outv[key * kD] = dvacc[cb][v];
    }
  }
  }
}

// ---- pipelined backward main kernel for 128-key blocks -----------------------------------------------------------
// With B_K = 128 the fp32 dK / dV accumulators of a block (128 KB) need the registers of four wavefronts and leave room
// for one eight-wave workgroup per CU.  If all eight waves step through the same phases of a tile (products, exponentials,
// accumulation), MFMA, VALU and LDS time add up and every LDS read waits out its latency: two waves per SIMD cannot
// cover each other.  Here the waves specialise and work one tile apart:
//   waves 0-3 (S-waves, one per SIMD): wave w keeps the K and V fragments of keys 32 w.. in registers and computes, for
//       the 64 rows of tile n, S = Q K^T, dP = dO V^T, P = exp(S - LSE), dS = P (dP - delta) scale, and writes
//       P^T, dS^T (bf16, [key][row]) to LDS; they also request and stage the gathered Q / dO rows;
//   waves 4-7 (A-waves, the other wave of each SIMD): wave a keeps the fp32 dK, dV accumulators of keys 32 a.. (all 128
//       channels) and the K^T fragments of channels 32 a.., and for tile n - 1 computes dV += P^T dO, then
//       dQ^T = K^T dS^T (channels 32 a.., all 128 keys; its 64-byte slice of every dQ row is stored at once), then
//       dK += dS^T Q; they also work out the row addresses of tile n + 3 for the S-waves.
// Q / dO tiles (turned rows, see row_turn) and P^T / dS^T tiles are double-buffered in LDS (142 KB in all), so the S-waves' MFMA and exponential work
// on tile n runs beside the A-waves' LDS-bound products on tile n - 1 on the same SIMD; two block-wide barriers per
// tile order the hand-over.  Rows are requested three tiles ahead into two register sets and staged after the second
// barrier.  Measured at 65536 tokens, g = 4, (128, 8): 3.5 ms against 4.1 ms for the eight-waves-in-step kernel, 3.3 ms
// since rows move by buffer instructions (no 64-bit address per access on the P/dS waves' staging path), 3.30 -> 3.20 ms with
// turned rows and one compare a key.  The masks in a branch instead (3.25 ms) or products that
// start from the row statistics as in the 64-key kernel (+1.5 %) break up the order the P/dS waves' steps are issued in.
struct PipeLds {
  static constexpr int Row = kD * 2;
  static constexpr int QB = kTile * Row;              // one Q or dO tile: 16384 bytes
  static constexpr int PB = 128 * kPStride * 2;       // one P^T or dS^T tile: 18432 bytes
  static constexpr int Q0 = 0;
  static constexpr int DO0 = Q0 + 2 * QB;
  static constexpr int Pt0 = DO0 + 2 * QB;
  static constexpr int DSt0 = Pt0 + 2 * PB;
  static constexpr int Ent = DSt0 + 2 * PB;
  static constexpr int St0 = Ent + kEntSeg * 4;       // per-row records of a staged tile, two buffers: three arrays
  static constexpr int SB = 3 * kTile * 4;            // of 64: LSE (log2 domain), delta * scale, visible key range
  static constexpr int Tb0 = St0 + 2 * SB;            // per row of the tile to request next: row of Q / dO, place in
  static constexpr int Next = Tb0 + kTile * 12;       // the kv head's statistics, visible keys
  static constexpr int Bytes = Next + 16;             // as in BwdLds; 145680 in all
};
static_assert(PipeLds::Bytes <= 160 * 1024, "the pipelined 128-key backward must fit one CU's LDS");
constexpr int kDqPitch = 36;  // bf16 per row of an A-wave's dQ staging (64 rows x 32 channels + pad = 4608 bytes)
static_assert(64 * kDqPitch <= 32 * kPStride, "dQ staging must fit the wave's 32 rows of a P^T tile");

// Built with -DNSA_PIPE_TIMING the pipelined kernel adds up, per role, the clocks its waves spend waiting at the two
// barriers, computing, and between them (a measuring build only: the stamps drain the LDS queue and cost a few percent).
#ifdef NSA_PIPE_TIMING
__device__ unsigned long long g_pipe_t[2][8];
#define PT_STAMP(k) { const unsigned long long now_ = clock64(); pt[k] += now_ - pt_last; pt_last = now_; }
#else
#define PT_STAMP(k)
#endif
// f(integral_constant<int, I>) for I = kBegin .. kEnd - 1, every index a compile-time constant
template <int kBegin, int kEnd, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (kBegin < kEnd) {
    f(std::integral_constant<int, kBegin>{});
    static_for<kBegin + 1, kEnd>(f);
  }
}

// What one workgroup of k_bwd_pipe128 works on.
struct PipeUnit : UnitRec {
  int pos0, number;
};

// One role of the pipeline (kS: an S-wave, else an A-wave).  Both roles run this same skeleton, so they execute the same
// sequence of block-wide barriers: every loop bound below depends only on the unit, never on the role or the lane.
template <bool kWin, bool kWide, bool kS, bool kQueue>
__device__ __forceinline__ void
pipe_role(const Problem& P, const PipeUnit& U, UnitTurn<kQueue>& turn, unsigned char* smem, const int sw, const bf16_t* __restrict__ Q,
          const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO,
          const float2* __restrict__ stats, const int2* __restrict__ qent, bf16_t* __restrict__ dqpart, float* __restrict__ dkv_part, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV) {
  int32_t* ent = reinterpret_cast<int32_t*>(smem + PipeLds::Ent);
  int tid = threadIdx.x;
  if constexpr (kQueue) asm volatile("" : "+v"(tid));  // keeps what depends on it inside the loop over units: carried round it, it spills
  const int lane = tid & 63;
  int col = lane & 31, qh = lane >> 5;
  const int j = U.j, tok0 = U.tok0, blen = U.blen;
  const float c2 = P.scale * 1.4426950408889634f;
  const int hbase = j * P.g;
  const int grp = lane >> 4, sl = lane & 15;
  // this lane's place in the Q / dO tiles (turned rows, see row_turn): as operand rows, and in a transposing read of four rows
  constexpr int kRow = PipeLds::Row;
  const int tr_r = (sl >> 2) + 8 * (grp >> 1);
  uint32_t tr_lane = lds_address(smem) + tr_r * kRow + (((2 * (grp & 1) + ((sl & 3) >> 1)) ^ row_turn(tr_r)) << 4) + 8 * (sl & 1);
  uint32_t frag_lane = lds_address(smem) + col * kRow + ((qh ^ row_turn(col)) << 4);
  int tr_lane_p = ((sl >> 2) + 8 * (grp >> 1)) * kPStride + 16 * (grp & 1) + 4 * (sl & 3);
  const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

  // register-resident operands.  S-wave: kf = K_i, vf = V_i fragments of keys 32 sw.. (A operands of S^T and dP^T).
  // A-wave: kf = K_i^T fragments of channels 32 sw.. (A operand of dQ^T; element e of step sp = key 16 sp + 8 qh + e).
  bf16x8 kf[8], vf[kS ? 8 : 1];
  if constexpr (kS) {
    const int key = 32 * sw + col;
    const size_t o = ((size_t)(tok0 + min(key, blen - 1)) * P.hkv + j) * kD + 8 * qh;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const bf16x8 kk = *reinterpret_cast<const bf16x8*>(K + o + 16 * s);
      const bf16x8 vv = *reinterpret_cast<const bf16x8*>(V + o + 16 * s);
      kf[s] = key < blen ? kk : zero8;
      vf[s] = key < blen ? vv : zero8;
    }
  } else {
    const bf16_t* src = K + ((size_t)tok0 * P.hkv + j) * kD + 32 * sw + col;
#pragma unroll
    for (int sp = 0; sp < 8; ++sp)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int key = 16 * sp + 8 * qh + e;
        const bf16_t kk = src[(size_t)min(key, blen - 1) * P.hkv * kD];
        kf[sp][e] = key < blen ? kk : (bf16_t)0.f;
      }
  }
  turn.draw();
  f32x16 dkacc[kS ? 1 : 4], dvacc[kS ? 1 : 4];  // A-wave: keys 32 sw.., by 32-channel block
  if constexpr (!kS) {
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        dkacc[cb][v] = 0.f;
        dvacc[cb][v] = 0.f;
      }
  }

  // S-waves stage the 64-row tiles: access i of thread t covers row 16 i + (t >> 4), 16 bytes at channel 8 (t & 15).
  // Rows are requested three tiles ahead of the S-waves' own use into two register sets (tile parity), so two tiles
  // (64 KB per CU) are in flight while one is computed: one tile in flight leaves the loop waiting on HBM latency.
  const int srow = (tid & 255) >> 4, schunk = (tid & 15) * 8;
  u32x4 qc[kS ? 2 : 1][kS ? 4 : 1], dc[kS ? 2 : 1][kS ? 4 : 1];
  // row record of row (t >> 2) of a requested tile, staged like the rows: (LSE in the log2 domain, delta) and the
  // block's keys the row sees: [0, lim) as lim, with a window [lo, lo + span) as lo | span << 16
  float2 st_set[2];
  int vis_set[2];
  int seg0 = 0, rows_end = 0;
  // The row table of a tile: for each of its 64 rows the (token, head) row index into Q / dO / stats and the block's
  // keys the row sees.  It is worked out one phase before the loads are issued, by whichever waves have the time
  // (all of them before the pipeline starts, the A-waves inside it) and handed over in LDS, so that the S-waves carry
  // no addresses through their products and issue the loads right after the barrier that frees the registers.
  uint32_t* row_table = reinterpret_cast<uint32_t*>(smem + PipeLds::Tb0);  // [3][kTile]
  const RowTensor<kWide> Qrows(Q, (int64_t)P.T * P.hq), dOrows(dO, (int64_t)P.T * P.hq);
  const float2* const head_stats = stats + (size_t)j * P.T * P.g;
  auto prepare_rows = [&](int tile0) __attribute__((always_inline)) {
    // rows past the end of the list re-read its last row: their P and dS are forced to zero and their dQ is never stored
    const int rr = tile0 + ((tid & 255) >> 2);
    const int rc = min(rr, rows_end - 1);
    const int ec = div_g(rc, P.g, P.g_magic);
    const int t = ent[ec - seg0];
    int lim = P.causal ? min(blen, t - tok0 + 1) : blen;  // keys [lo, lim) of the block are visible to this row
    if (rr >= rows_end) lim = 0;
    const int lo = kWin ? min(max(t - P.window + 1 - tok0, 0), 128) : 0;
    if ((tid & 3) == 0) {
      uint32_t* e = row_table + ((tid & 255) >> 2);
      e[0] = (uint32_t)t * (uint32_t)P.hq + (uint32_t)(hbase + (rc - ec * P.g));
      e[kTile] = (uint32_t)t * (uint32_t)P.g + (uint32_t)(rc - ec * P.g);
      e[2 * kTile] = kWin ? (uint32_t)(lo | (max(lim - lo, 0) << 16)) : (uint32_t)lim;
    }
  };
  auto issue_rows = [&](auto setc) __attribute__((always_inline)) {
    constexpr int set = kS ? decltype(setc)::value : 0;
    uint32_t grow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) grow[i] = row_table[16 * i + srow];
    const uint32_t* mine = row_table + ((tid & 255) >> 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      qc[set][i] = Qrows.load(grow[i], schunk * 2);
      dc[set][i] = dOrows.load(grow[i], schunk * 2);
    }
    st_set[set] = head_stats[mine[kTile]];
    vis_set[set] = (int)mine[2 * kTile];
  };
  const uint32_t stage = lds_address(smem) + srow * kRow + (((tid & 15) ^ row_turn(srow)) << 4);
  auto stage_rows = [&](auto bufc, auto setc) __attribute__((always_inline)) {
    constexpr int set = kS ? decltype(setc)::value : 0, buf = decltype(bufc)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lds_write_16(stage + PipeLds::Q0 + buf * PipeLds::QB + 16 * i * kRow, qc[set][i]);
      lds_write_16(stage + PipeLds::DO0 + buf * PipeLds::QB + 16 * i * kRow, dc[set][i]);
    }
    if ((tid & 3) == 0) {
      float* rec = reinterpret_cast<float*>(smem + PipeLds::St0 + buf * PipeLds::SB) + ((tid & 255) >> 2);
      rec[0] = st_set[set].x;
      rec[kTile] = st_set[set].y * P.scale;
      reinterpret_cast<int*>(rec)[2 * kTile] = vis_set[set];
    }
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;

#ifdef NSA_PIPE_TIMING
  unsigned long long pt[8] = {0, 0, 0, 0, 0, 0, 0, 0}, pt_last = clock64();
#endif
  for (seg0 = 0; seg0 < U.ne; seg0 += kEntSeg) {
    const int seg_n = min(kEntSeg, U.ne - seg0);
    __syncthreads();  // the previous segment's ids and tiles are no longer read
    for (int i = tid; i < seg_n; i += 512) ent[i] = qent[U.e0 + seg0 + i].x;
    __syncthreads();
    const int row_first = seg0 * P.g;
    rows_end = (seg0 + seg_n) * P.g;
    const int ntiles = (rows_end - row_first + kTile - 1) / kTile;
    // start of the pipeline: tiles 0, 1, 2 requested, tile 0 staged (one table, so a barrier pair per tile)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if constexpr (kS) prepare_rows(row_first + k * kTile);
      __syncthreads();
      if constexpr (kS) {
        if (k == 0) {
          issue_rows(Set0{});
          stage_rows(Set0{}, Set0{});
        } else if (k == 1) {
          issue_rows(Set1{});
        } else {
          issue_rows(Set0{});
        }
      }
      __syncthreads();
    }

    // one pipeline step: S-waves work on tile `it`, A-waves on tile `it - 1`; `par` = parity of `it`
    auto step = [&](const int it, auto par) __attribute__((always_inline)) {
      using Other = std::integral_constant<int, 1 - decltype(par)::value>;
      asm volatile("" : "+v"(col), "+v"(qh), "+v"(tr_lane), "+v"(tr_lane_p), "+v"(frag_lane));
      PT_STAMP(3)
      __syncthreads();  // tile `it` staged; P^T / dS^T of tile `it - 1` complete
      PT_STAMP(0)
      if constexpr (kS) {
        if (it < ntiles) {  // ---- S, dP, P, dS of tile `it`: keys 32 sw.., all 64 rows
          constexpr int buf = decltype(par)::value;
          bf16_t* Pt = reinterpret_cast<bf16_t*>(smem + PipeLds::Pt0 + buf * PipeLds::PB);
          bf16_t* dSt = reinterpret_cast<bf16_t*>(smem + PipeLds::DSt0 + buf * PipeLds::PB);
          // S = Q K_i^T, dP = dO V_i^T for rows 32 rb.. x keys 32 sw..: lane = key, register v = row 8 (v >> 2) + 4 qh
          // + (v & 3), so four consecutive rows of P^T / dS^T leave each lane as one 8-byte LDS store.
          // Issue order, fixed by hand: a wave issues in order and only two waves share a SIMD, so an LDS read that
          // is waited for right before its MFMA exposes the whole LDS latency each time.  The four products (S, dP of
          // two row blocks) run as one software pipeline over a ring of eight fragment registers: step s issues the
          // MFMA on fragment s, refills that register with fragment s of the NEXT product, and does one eighth of the
          // elementwise work on the PREVIOUS product's result.
          f32x16 sacc[2], dpacc[2];
          float pv[2][16];
          bf16x8 fr[8];
          const float* rec = reinterpret_cast<const float*>(smem + PipeLds::St0 + buf * PipeLds::SB);
          const int key = 32 * sw + col;
          auto q_frag = [&](int rb, int st) { return lds_read_frag((frag_lane ^ (32 * st)) + PipeLds::Q0 + buf * PipeLds::QB + 32 * rb * kRow); };
          auto d_frag = [&](int rb, int st) { return lds_read_frag((frag_lane ^ (32 * st)) + PipeLds::DO0 + buf * PipeLds::QB + 32 * rb * kRow); };
          f32x4 lse4, dls4;
          u32x4 vis4;
          auto probs = [&](int rb, int st) __attribute__((always_inline)) {  // P = exp(S scale - LSE) on visible keys
            const int a = st >> 1, r4 = 32 * rb + 8 * a + 4 * qh;
            if ((st & 1) == 0) {
              lse4 = *reinterpret_cast<const f32x4*>(rec + r4);
              vis4 = *reinterpret_cast<const u32x4*>(rec + 2 * kTile + r4);
            }
#pragma unroll
            for (int c = 2 * (st & 1); c < 2 * (st & 1) + 2; ++c) {
              const bool seen = kWin ? (uint32_t)key - (vis4[c] & 0xffffu) < (vis4[c] >> 16) : (uint32_t)key < vis4[c];
              pv[rb][4 * a + c] = seen ? __builtin_amdgcn_exp2f(fmaf(sacc[rb][4 * a + c], c2, -lse4[c])) : 0.f;
            }
          };
          auto emit = [&](int rb, int st) __attribute__((always_inline)) {  // dS = P (dP - delta) scale; bf16 to LDS
            const int a = st >> 1, r4 = 32 * rb + 8 * a + 4 * qh;
            if ((st & 1) == 0) {
              dls4 = *reinterpret_cast<const f32x4*>(rec + kTile + r4);
              uint2 pw;
              pw.x = pack_bf16x2(pv[rb][4 * a + 0], pv[rb][4 * a + 1]);
              pw.y = pack_bf16x2(pv[rb][4 * a + 2], pv[rb][4 * a + 3]);
              *reinterpret_cast<uint2*>(&Pt[key * kPStride + r4]) = pw;
            } else {
              float ds[4];
#pragma unroll
              for (int c = 0; c < 4; ++c) ds[c] = pv[rb][4 * a + c] * fmaf(dpacc[rb][4 * a + c], P.scale, -dls4[c]);
              uint2 sw2;
              sw2.x = pack_bf16x2(ds[0], ds[1]);
              sw2.y = pack_bf16x2(ds[2], ds[3]);
              *reinterpret_cast<uint2*>(&dSt[key * kPStride + r4]) = sw2;
            }
          };
#pragma unroll
          for (int v = 0; v < 16; ++v) sacc[0][v] = dpacc[0][v] = sacc[1][v] = dpacc[1][v] = 0.f;
#pragma unroll
          for (int st = 0; st < 8; ++st) fr[st] = q_frag(0, st);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int st = 0; st < 8; ++st) {  // S, rows 0..31; refill with dO, rows 0..31
            sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[st], kf[st], sacc[0], 0, 0, 0);
            fr[st] = d_frag(0, st);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int st = 0; st < 8; ++st) {  // dP, rows 0..31; refill with Q, rows 32..63; P of rows 0..31
            dpacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[st], vf[st], dpacc[0], 0, 0, 0);
            fr[st] = q_frag(1, st);
            probs(0, st);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int st = 0; st < 8; ++st) {  // S, rows 32..63; refill with dO, rows 32..63; P, dS of rows 0..31 to LDS
            sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[st], kf[st], sacc[1], 0, 0, 0);
            fr[st] = d_frag(1, st);
            emit(0, st);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int st = 0; st < 8; ++st) {  // dP, rows 32..63; P of rows 32..63
            dpacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[st], vf[st], dpacc[1], 0, 0, 0);
            probs(1, st);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int st = 0; st < 8; ++st) emit(1, st);
        }
        PT_STAMP(1)
        __syncthreads();  // every wave is done with the tiles of `it - 1`: stage tile `it + 1` there, request `it + 2`
        PT_STAMP(2)
        // unconditional (tiles past the end re-read the list's last row and are never used): with no branch around
        // the loads the compiler's wait counts stay exact and the newer set's loads are left in flight here
        stage_rows(Other{}, Other{});
        issue_rows(Other{});
      } else {
        constexpr int buf = 1 - decltype(par)::value;
        prepare_rows(row_first + (it + 3) * kTile);  // read by the S-waves after this step's second barrier
        if (it >= 1 && it <= ntiles) {  // ---- tile `it - 1`
          const bf16_t* Pt = reinterpret_cast<const bf16_t*>(smem + PipeLds::Pt0 + buf * PipeLds::PB);
          const bf16_t* dSt = reinterpret_cast<const bf16_t*>(smem + PipeLds::DSt0 + buf * PipeLds::PB);
          // Three products of 16 MFMAs each, in this order:
          //   ops  0..15  dV_i += P^T dO          (op = 4 qs + cb: rows 16 qs.., channels 32 cb..)
          //   ops 16..31  dQ^T  = K_i^T dS^T      (op = 16 + 2 sp + rb: keys 16 sp.., rows 32 rb..)
          //   ops 32..47  dK_i += dS^T Q          (as the first, with Q)
          // Every op's "lane = column" operand is a pair of transposing LDS reads.  As in the S-waves the issue order
          // is fixed by hand: the operands run through a ring of kRing registers, op i issues its MFMA and refills its
          // slot with the operand of op i + kRing, across the product boundaries, so only the first kRing reads of a
          // tile are waited for at full LDS latency.  The dQ slices are stored between the second and third product.
          constexpr int kRing = 4;
          const bf16_t* parow = Pt + (32 * sw + col) * kPStride + 8 * qh;   // rows 32 sw.. of P^T: read by this wave only
          const bf16_t* sarow = dSt + (32 * sw + col) * kPStride + 8 * qh;
          const bf16_t* ds_tr = dSt + tr_lane_p;
          auto operand = [&](auto opc) __attribute__((always_inline)) {
            constexpr int op = decltype(opc)::value;
            bf16x4 lo4, hi4;
            if constexpr (op >= 16 && op < 32) {
              const bf16_t* p0 = ds_tr + (16 * ((op - 16) >> 1) * kPStride + 32 * (op & 1));
              lo4 = lds_read_tr(p0);
              hi4 = lds_read_tr(p0 + 4 * kPStride);
            } else {
              constexpr int at = (op < 16 ? PipeLds::DO0 : PipeLds::Q0) + buf * PipeLds::QB + 16 * ((op & 15) >> 2) * kRow;
              lo4 = lds_read_tr_at((tr_lane ^ (64 * (op & 3))) + at);
              hi4 = lds_read_tr_at((tr_lane ^ (64 * (op & 3) + 16)) + at + 4 * kRow);
            }
            return __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
          };
          bf16x8 ring[kRing], af[4];  // af: the "lane = row of the result" operand of the first / third product
          f32x16 dqacc[2];
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int v = 0; v < 16; ++v) dqacc[rb][v] = 0.f;
#pragma unroll
          for (int qs = 0; qs < 4; ++qs) af[qs] = *reinterpret_cast<const bf16x8*>(parow + 16 * qs);
          static_for<0, kRing>([&](auto opc) { ring[decltype(opc)::value] = operand(opc); });
          __builtin_amdgcn_sched_barrier(0);
          static_for<0, 48>([&](auto opc) __attribute__((always_inline)) {
            constexpr int op = decltype(opc)::value;
            if constexpr (op < 16)
              dvacc[op & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[op >> 2], ring[op % kRing], dvacc[op & 3], 0, 0, 0);
            else if constexpr (op < 32)
              dqacc[op & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[(op - 16) >> 1], ring[op % kRing],
                                                                      dqacc[op & 1], 0, 0, 0);
            else
              dkacc[op & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[(op - 32) >> 2], ring[op % kRing],
                                                                      dkacc[op & 3], 0, 0, 0);
            if constexpr (op + kRing < 48) ring[op % kRing] = operand(std::integral_constant<int, op + kRing>{});
            if constexpr (op >= 24 && op < 28)  // the first product is done with af: refill it for the third
              af[op - 24] = *reinterpret_cast<const bf16x8*>(sarow + 16 * (op - 24));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (op == 31) {
              // this wave's 64-byte slice of the tile's dQ rows: accumulator layout (lane = row) -> rows 32 sw.. of
              // the P^T tile, which this wave has finished reading and the S-waves rewrite only after the next
              // barrier -> 16-byte row pieces
              bf16_t* stg = reinterpret_cast<bf16_t*>(smem + PipeLds::Pt0 + buf * PipeLds::PB) + 32 * sw * kPStride;
#pragma unroll
              for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                  uint2 w;
                  w.x = pack_bf16x2(dqacc[rb][4 * a + 0], dqacc[rb][4 * a + 1]);
                  w.y = pack_bf16x2(dqacc[rb][4 * a + 2], dqacc[rb][4 * a + 3]);
                  *reinterpret_cast<uint2*>(&stg[(32 * rb + col) * kDqPitch + 8 * a + 4 * qh]) = w;
                }
              wave_sync_bwd();
              const int tile0 = row_first + (it - 1) * kTile;
              const __amdgpu_buffer_rsrc_t dq_buf =
                  buffer_of(dqpart + ((size_t)(U.e0 - U.pos0) * P.g + (size_t)tile0) * kD,
                            (uint32_t)min(rows_end - tile0, kTile) * (kD * 2));  // rows past the list's end are dropped
              int ln = lane;
              asm volatile("" : "+v"(ln));  // keeps the row addresses from being precomputed and held (register budget)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int row = 16 * i + (ln >> 2), piece = (ln & 3) * 8;
                const uint2 lo2 = *reinterpret_cast<const uint2*>(&stg[row * kDqPitch + piece]);
                const uint2 hi2 = *reinterpret_cast<const uint2*>(&stg[row * kDqPitch + piece + 4]);
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{lo2.x, lo2.y, hi2.x, hi2.y}, dq_buf,
                                                       row * (kD * 2) + 64 * sw + piece * 2, 0, kNonTemporal);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          });
        }
        PT_STAMP(1)
        __syncthreads();  // every wave is done with the tiles of `it - 1`
        PT_STAMP(2)
      }
    };
    // both roles take the same number of steps: the barriers inside `step` pair up across the roles
    // (an even number of steps; a last step past the end computes nothing)
    for (int it = 0; it <= ntiles; it += 2) {
      step(it, Set0{});
      step(it + 1, Set1{});
    }
  }

#ifdef NSA_PIPE_TIMING
  if (lane == 0)
    for (int k = 0; k < 8; ++k)
      if (k != 4) atomicAdd(&g_pipe_t[kS ? 0 : 1][k], pt[k]);
  if (lane == 0) atomicAdd(&g_pipe_t[kS ? 0 : 1][4], 1ull);
#endif
  if constexpr (!kS) {
    if (U.n_units == 1) {
      // the whole list fitted this unit: dK_i, dV_i are final, write them as bf16 (keys of a ragged tail excluded)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        bf16_t* outk = dK + ((size_t)tok0 * P.hkv + j) * kD + 32 * cb + col;
        bf16_t* outv = dV + ((size_t)tok0 * P.hkv + j) * kD + 32 * cb + col;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = 32 * sw + 8 * (v >> 2) + 4 * qh + (v & 3);
          if (key < blen) {
            outk[(size_t)key * P.hkv * kD] = (bf16_t)dkacc[cb][v];
            outv[(size_t)key * P.hkv * kD] = (bf16_t)dvacc[cb][v];
          }
        }
      }
      return;
    }
    // unit partial: [u][0 = dK, 1 = dV][key][d] fp32, summed by k_bwd_dkv_reduce in unit order
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      float* outk = dkv_part + (size_t)(kQueue ? U.number : (int)blockIdx.x) * 2 * 128 * kD + 32 * cb + col;
      float* outv = outk + 128 * kD;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = 32 * sw + 8 * (v >> 2) + 4 * qh + (v & 3);
        outk[key * kD] = dkacc[cb][v];
        outv[key * kD] = dvacc[cb][v];
      }
    }
  }
}

template <bool kWin, bool kWide, bool kQueue>
__global__ void __launch_bounds__(512, 1)
k_bwd_pipe128(Problem P, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
              const bf16_t* __restrict__ dO, const float2* __restrict__ stats, const UnitRec* __restrict__ u_rec,
              const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ off, const int2* __restrict__ qent,
              bf16_t* __restrict__ dqpart, float* __restrict__ dkv_part, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV,
              UnitQueue queue) {
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  UnitTurn<kQueue> turn(P, u_rec, nu_scan, off, queue, reinterpret_cast<int32_t*>(smem + PipeLds::Next));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (turn.unit < 0) return;
  do {
    const PipeUnit U = {turn.record(u_rec), turn.pos0, turn.unit};
    if (wave < 4)
      pipe_role<kWin, kWide, true>(P, U, turn, smem, wave, Q, K, V, dO, stats, qent, dqpart, dkv_part, dK, dV);
    else
      pipe_role<kWin, kWide, false>(P, U, turn, smem, wave - 4, Q, K, V, dO, stats, qent, dqpart, dkv_part, dK, dV);
    if constexpr (kQueue) turn.advance();
  } while (kQueue && turn.unit >= 0);  // (without the queue no loop, which a condition on the unit alone would leave)
}

// dK / dV of the lists whose units left partial sums: the sum runs in unit order, four units in flight.  A piece of this work is
// (`per` <= 64 lists, dK or dV, 8 keys), so that the units of a long list (the sink block's list has 32 of them) are walked by
// B_K / 8 pieces side by side, 256 threads each; thread = 4 consecutive channels of one key.  Most lists fit one unit, which wrote the
// final values itself: a piece looks at its lists at once (one per lane) and walks only those that need it, so that there are some
// thousand of them and not one per list and key group (25 900 lists: 414 000 workgroups, 174 us).
// (Its pointers are arguments of the kernels themselves: out of a structure the compiler does not take them to be distinct, and the table
// reads of a list wait for the stores of the one before.)
__device__ __forceinline__ void dkv_reduce(const Problem& P, int per, int group, int which, int part, int tid,
                                           const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ blk_tok0,
                                           const int32_t* __restrict__ blk_len, const float* __restrict__ dkv_part,
                                           bf16_t* __restrict__ dK, bf16_t* __restrict__ dV) {
  const int lane = tid & 63, l0 = P.l0 + group * per;
  const int ubase = P.l0 > 0 ? nu_scan[P.l0] : 0;
  const int mine = min(l0 + lane, P.l1 - 1);
  const int my_u0 = nu_scan[mine], my_nu = nu_scan[mine + 1] - my_u0;
  unsigned long long todo = __builtin_amdgcn_ballot_w64(lane < per && l0 + lane < P.l1 && my_nu != 1);
  bf16_t* out = which ? dV : dK;
  const int d4 = (tid & 31) * 4;
  const int key = 8 * part + (tid >> 5);
  const size_t unit_stride = (size_t)2 * P.bk * kD;
  while (todo != 0ull) {
    const int i = __builtin_ctzll(todo);
    todo &= todo - 1ull;
    const int u0 = __builtin_amdgcn_readlane(my_u0, i), nu = __builtin_amdgcn_readlane(my_nu, i);
    const int j = (l0 + i) / P.b_cap, gb = l0 + i - j * P.b_cap;
    if (key >= blk_len[gb]) continue;
    const float* src = dkv_part + (size_t)(u0 - ubase) * unit_stride + (size_t)which * P.bk * kD + key * kD + d4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int u = 0;
    for (; u + 4 <= nu; u += 4, src += 4 * unit_stride) {
      float4 x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = *reinterpret_cast<const float4*>(src + q * unit_stride);
#pragma unroll
      for (int q = 0; q < 4; ++q) { acc.x += x[q].x; acc.y += x[q].y; acc.z += x[q].z; acc.w += x[q].w; }
    }
    for (; u < nu; ++u, src += unit_stride) {
      const float4 x = *reinterpret_cast<const float4*>(src);
      acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
    }
    uint2 w;
    w.x = pack_bf16x2(acc.x, acc.y);
    w.y = pack_bf16x2(acc.z, acc.w);
    *reinterpret_cast<uint2*>(out + ((size_t)(blk_tok0[gb] + key) * P.hkv + j) * kD + d4) = w;
  }
}

// The pieces alone: beside a dQ reduction in bursts, and where a head's KV blocks are taken in ranges, of all ranges but the last.
__global__ void __launch_bounds__(256)
k_bwd_dkv_reduce(Problem P, int per, const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ blk_tok0,
                 const int32_t* __restrict__ blk_len, const float* __restrict__ dkv_part, bf16_t* __restrict__ dK,
                 bf16_t* __restrict__ dV) {
  dkv_reduce(P, per, blockIdx.x, blockIdx.y, blockIdx.z, threadIdx.x, nu_scan, blk_tok0, blk_len, dkv_part, dK, dV);
}

// dQ of every (token, head) row from its columns' partial rows: plain sums, in column order.  Rows and workgroups: see "the two
// reduction kernels" in common.h.  (k_fwd_merge is the same with weights.)  Row by row, on smaller inputs, its first `before` workgroups
// do the dK / dV sums, which are independent of it, instead of a launch for them: 12.6 -> 7.2 us for both at 1024 tokens, 31 -> 28 on a
// batch of short documents.  In bursts they would leave the others one workgroup a compute unit less: 214 -> 250 us at 8192 tokens, 32
// heads, g = 1.
template <int kRows, int kThreads>
__global__ void __launch_bounds__(kThreads)
k_bwd_dq_reduce(Problem P, const bf16_t* __restrict__ dqpart, const int32_t* __restrict__ slotpos,
                const int32_t* __restrict__ off, bf16_t* __restrict__ dQ, int before, int per, int groups,
                const int32_t* __restrict__ nu_scan, const int32_t* __restrict__ blk_tok0, const int32_t* __restrict__ blk_len,
                const float* __restrict__ dkv_part, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV) {
  if constexpr (kRows == 1) {
    static_assert(kThreads == 256, "one piece of the dK / dV sums a workgroup");
    if ((int)blockIdx.x < before) {
      const int side = blockIdx.x / groups;  // the lists side by side, then dK and dV, then the keys
      if (side < P.bk / 4)
        dkv_reduce(P, per, blockIdx.x - side * groups, side & 1, side >> 1, threadIdx.x, nu_scan, blk_tok0, blk_len, dkv_part, dK, dV);
      return;
    }
  }
  constexpr int kBatch = 8;  // independent 256-byte gathers in flight per row
  const int sub = threadIdx.x & 15;
  const int pos0 = off[P.j0 * P.b_cap];
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* const out = reinterpret_cast<u32x4*>(smem) + threadIdx.x;
  const ReduceSpan span = reduce_span<kRows, kThreads>(P, blockIdx.x - before, gridDim.x - before);
  if (span.count == 0) return;  // the whole workgroup
  ReduceRow R = reduce_row<kThreads>(P, span.first);
  SlotRow slots = load_slots(slotpos, P, R);
#pragma unroll 1
  for (int q = 0; q < span.count; ++q) {
    const ReduceRow R_next = reduce_row<kThreads>(P, span.first + min(q + 1, span.count - 1));
    const SlotRow slots_next = load_slots(slotpos, P, R_next);
    const bf16_t* base = dqpart + R.hh * kD + 8 * sub;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int pos = pos0;  // of the last kept column
    const KeptColumns kept(slots);
    auto gather = [&](int m0, auto all_kept) __attribute__((always_inline)) {
      int at[kBatch];
      u32x4 x[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) at[i] = slot_of(slots, m0, i);
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        x[i] = u32x4{0, 0, 0, 0};
        if constexpr (kRows > 1) {
          pos = at[i] >= 0 ? at[i] : pos;
          asm volatile("" : "+v"(at[i]), "+v"(pos));  // keeps the loads free of branches
        } else {
          pos = at[i];
        }
        if (kRows > 1 || all_kept || at[i] >= 0) x[i] = load_streaming(base + (size_t)(uint32_t)(pos - pos0) * (uint32_t)P.g * kD);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (kRows > 1 && at[i] < 0) x[i] = u32x4{0, 0, 0, 0};
        acc[0] += bf16_lo(x[i].x); acc[1] += bf16_hi(x[i].x);
        acc[2] += bf16_lo(x[i].y); acc[3] += bf16_hi(x[i].y);
        acc[4] += bf16_lo(x[i].z); acc[5] += bf16_hi(x[i].z);
        acc[6] += bf16_lo(x[i].w); acc[7] += bf16_hi(x[i].w);
      }
    };
    for (int m0 = 0; m0 < P.topk; m0 += kBatch) {
      const uint64_t eight = kept.eight_from(m0);
      if (kRows == 1 && eight == KeptColumns::kAll) gather(m0, std::true_type{});
      else if (kRows > 1 || eight != 0) gather(m0, std::false_type{});
    }
    out[q * kThreads] = u32x4{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]), pack_bf16x2(acc[4], acc[5]),
                              pack_bf16x2(acc[6], acc[7])};
    R = R_next;
    slots = slots_next;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    if (q >= span.count) break;
    const ReduceRow R = reduce_row<kThreads>(P, span.first + q);
    if (R.on) store_streaming(dQ + ((int64_t)R.t * P.hq + R.j * P.g + R.hh) * kD + 8 * sub, out[q * kThreads]);
  }
}

#ifdef NSA_PIPE_TIMING
// Measuring build only: copies the 2 x 8 counters (role x {phase 0..3 clocks, waves counted, unused}) to the host `out`
// (synchronous, on the current device) and, with `reset`, zeroes them.  Returns 0, or -1 if a HIP call failed.
extern "C" int nsa_sel_pipe_timing_read(unsigned long long* out, int reset) {
  if (hipMemcpyFromSymbol(out, HIP_SYMBOL(g_pipe_t), sizeof(unsigned long long) * 16) != hipSuccess) return -1;
  if (reset) {
    unsigned long long z[16] = {};
    if (hipMemcpyToSymbol(HIP_SYMBOL(g_pipe_t), z, sizeof(z)) != hipSuccess) return -1;
  }
  return 0;
}
#endif
hipError_t launch_bwd(const Problem& P0, const IndexLayout& L, int heads_per_pass, int lists_per_pass, const void* Q,
                      const void* K, const void* V, const void* O, const float* LSE, const void* dO, const void* index_ws,
                      void* dqpart, float* delta, float* dkv_part, void* dQ, void* dK, void* dV, const GateArgs& G,
                      hipStream_t st) {
  IndexPtrs p = index_ptrs(L, const_cast<void*>(index_ws));
  // 64-token blocks: four waves, two workgroups per CU; 128-token blocks: eight waves, one workgroup per CU
  const bool b128 = P0.bk == 128;
  const bool win = P0.window > 0;
  const bool wide = rows_are_wide((int64_t)P0.T * P0.hq);
  const int main_threads = b128 ? 512 : 256;
  const int main_lds = b128 ? PipeLds::Bytes : BwdLds::Bytes;
  const int passes = (P0.hkv + heads_per_pass - 1) / heads_per_pass;
  const int64_t pass_units = units_bound(heads_per_pass, P0.b_cap, P0.T, P0.topk, P0.unit);
  // (Q of 4 GB and more: units by the hundred a slot)
  const bool queued = lists_per_pass == 0 && passes <= kQueuePasses && pass_units >= kQueueMinUnits && !wide &&
                      queue_pays(P0);
  int32_t* const queue = queued ? reinterpret_cast<int32_t*>(dkv_part + (size_t)(pass_units - 1) * 2 * P0.bk * kD) : nullptr;
  const bool ordered = queued && passes == 1 && pass_units <= kQueueUnits;
  auto form = [&](auto* keys64, auto* keys128) { return b128 ? keys128 : keys64; };
  auto* main_kernel = win ? queued ? form(k_bwd_tiled<true, false, true>, k_bwd_pipe128<true, false, true>)
                            : wide ? form(k_bwd_tiled<true, true, false>, k_bwd_pipe128<true, true, false>)
                                   : form(k_bwd_tiled<true, false, false>, k_bwd_pipe128<true, false, false>)
                          : queued ? form(k_bwd_tiled<false, false, true>, k_bwd_pipe128<false, false, true>)
                            : wide ? form(k_bwd_tiled<false, true, false>, k_bwd_pipe128<false, true, false>)
                                   : form(k_bwd_tiled<false, false, false>, k_bwd_pipe128<false, false, false>);
  {
    static std::atomic<uint64_t> ready[16];
    static std::atomic<uint64_t> ready_reduce;
    hipError_t e = allow_dynamic_lds((const void*)main_kernel, main_lds, ready[win + 2 * wide + 4 * b128 + 8 * queued]);
    if (e == hipSuccess)
      e = allow_dynamic_lds((const void*)(k_bwd_dq_reduce<kBurstRows, kBurstThreads>), reduce_lds(kBurstThreads, kBurstRows, 1, false),
                            ready_reduce);
    if (e != hipSuccess) return e;
  }
  {
    ProfScope ps(KID_BWD_DELTA, st);
    hipLaunchKernelGGL(k_bwd_delta, dim3((P0.T + kDeltaTokens - 1) / kDeltaTokens + queued, (P0.hkv + kDeltaKv - 1) / kDeltaKv),
                       dim3(256), 0, st, P0, (const bf16_t*)O,
                       (const bf16_t*)dO, LSE, (float2*)delta, G.gate, G.dgate, p.u_rec, p.u_nu, queue, ordered);
  }
  // KV heads are processed heads_per_pass at a time, every pass reusing the partial-dQ and unit-sum buffers; of one head,
  // where its unit sums do not fit, lists_per_pass lists at a time, every range reusing the unit sums.
  for (int j0 = 0; j0 < P0.hkv; j0 += heads_per_pass) {
    Problem P = P0;
    P.j0 = j0;
    P.nj = min(heads_per_pass, P0.hkv - j0);
    const int first = j0 * P.b_cap, end = (j0 + P.nj) * P.b_cap;
    const int step = lists_per_pass > 0 ? lists_per_pass : end - first;
    for (P.l0 = first; P.l0 < end; P.l0 += step) {
      P.l1 = min(P.l0 + step, end);
      // upper bound of the work units of the launch (the real count is only known on the device): also what the workspace holds
      const int64_t bound = units_bound(P.nj, P.b_cap, P.T, P.topk, P.unit);
      const unsigned units_max =
          (unsigned)(lists_per_pass > 0 ? min(bound, (int64_t)step * ((P.T + P.unit - 1) / P.unit)) : bound);
      const UnitQueue turns = {queued ? queue + j0 / heads_per_pass : nullptr, ordered ? queue + kQueuePasses : nullptr};
      const unsigned slots = b128 ? 256 : 512;  // workgroups that the chip holds
      { ProfScope ps(KID_BWD_MAIN, st);
      hipLaunchKernelGGL(main_kernel, dim3(queued ? min(units_max, slots) : units_max), dim3(main_threads), main_lds, st, P, (const bf16_t*)Q,
                         (const bf16_t*)K, (const bf16_t*)V, (const bf16_t*)dO, (const float2*)delta, p.u_rec, p.u_nu,
                         p.off, p.qent, (bf16_t*)dqpart, dkv_part, (bf16_t*)dK, (bf16_t*)dV, turns); }
      const int lists = P.l1 - P.l0, per = max(1, min(64, lists * (P.bk / 4) / 4096));
      const int groups = (lists + per - 1) / per;
      const bool last = P.l1 == end, bursts = dq_in_bursts(P);
      if (last) {
        ProfScope ps(KID_BWD_DQ_REDUCE, st);
        auto launch = [&](auto rows, auto threads, int before) {
          constexpr int kRows = decltype(rows)::value, kThreads = decltype(threads)::value;
          hipLaunchKernelGGL((k_bwd_dq_reduce<kRows, kThreads>), dim3(before + reduce_groups<kRows, kThreads>(P)), dim3(kThreads),
                             reduce_lds(kThreads, kRows, 1, false), st, P, (const bf16_t*)dqpart, p.slotpos, p.off, (bf16_t*)dQ, before, per,
                             groups, p.u_nu, p.blk_tok0, p.blk_len, (const float*)dkv_part, (bf16_t*)dK, (bf16_t*)dV);
        };
        if (bursts)
          launch(std::integral_constant<int, kBurstRows>{}, std::integral_constant<int, kBurstThreads>{}, 0);
        else  // (a multiple of eight, so that the XCDs of the workgroups after them stay the same)
          launch(std::integral_constant<int, 1>{}, std::integral_constant<int, 256>{}, (groups * (P.bk / 4) + 7) & ~7);
      }
      if (!last || bursts) {
        ProfScope ps(KID_BWD_DKV_REDUCE, st);
        hipLaunchKernelGGL(k_bwd_dkv_reduce, dim3(groups, 2, P.bk / 8), dim3(256), 0, st, P, per, p.u_nu, p.blk_tok0, p.blk_len,
                           (const float*)dkv_part, (bf16_t*)dK, (bf16_t*)dV);
      }
    }
  }
  return hipGetLastError();
}

}  // namespace nsa
