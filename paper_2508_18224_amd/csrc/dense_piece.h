// One 64-key piece against 32 query rows of a wavefront, as the kernels that walk contiguous keys do it (k_fwd_dense_merge, k_fwd_short):
// the piece's K and V lie in LDS as unpadded, turned rows (see row_turn), the rows' Q in registers, the output is accumulated there.
#pragma once
#include "common.h"

namespace nsa {

constexpr int kPieceRow = kD * 2;               // bytes of a row of K or V in LDS
constexpr int kPieceBytes = 64 * kPieceRow;     // a piece's K, or its V

// This lane's operand reads: K fragment of contraction step s, keys 32 mb.., is chunk 2 s + qh of row 32 mb + col; V^T fragments are
// transposing reads of rows (sl / 4) + 4 (grp / 2) + 16 sp (+ 8), channels 32 db + 16 (grp & 1) + 4 (sl & 3).
__device__ __forceinline__ void piece_addresses(uint32_t k_lds, uint32_t v_lds, int lane, uint32_t (&kaddr)[8], uint32_t (&vaddr)[2][4]) {
  const int col = lane & 31, qh = lane >> 5, grp = lane >> 4, sl = lane & 15;
#pragma unroll
  for (int s = 0; s < 8; ++s) kaddr[s] = k_lds + col * kPieceRow + (((2 * s + qh) ^ row_turn(col)) << 4);
  const int vrow = (sl >> 2) + 4 * (grp >> 1), vchunk = 2 * (grp & 1) + ((sl & 3) >> 1);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int d = 0; d < 4; ++d)
      vaddr[h][d] = v_lds + (vrow + 8 * h) * kPieceRow + (((4 * d + vchunk) ^ row_turn(vrow + 8 * h)) << 4) + 8 * (sl & 1);
}

// S^T = K Q^T of the piece: lane = row, register v of half mb = key 32 mb + 8 (v >> 2) + 4 qh + (v & 3).
__device__ __forceinline__ void piece_scores(const uint32_t (&kaddr)[8], const bf16x8 (&qf)[8], f32x16 (&sacc)[2]) {
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) sacc[mb][v] = 0.f;
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      const bf16x8 kf = lds_read_frag(kaddr[s] + 32 * mb * kPieceRow);
      sacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], sacc[mb], 0, 0, 0);
    }
}

// The row's maximum from the maxima over the keys of its two lanes.
__device__ __forceinline__ float row_max(float m) { return fmaxf(m, __shfl_xor(m, 32)); }

// Scores of keys outside [lo, lim) become -inf; returns the maximum over this lane's keys.
__device__ __forceinline__ float mask_scores(f32x16 (&sacc)[2], int lo, int lim, int qh) {
  float m = -INFINITY;
  lo -= 4 * qh;
  lim -= 4 * qh;
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int key = 32 * mb + 8 * (v >> 2) + (v & 3);
      const float x = (key < lim && key >= lo) ? sacc[mb][v] : -INFINITY;
      sacc[mb][v] = x;
      m = fmaxf(m, x);
    }
  return m;
}
__device__ __forceinline__ float max_scores(const f32x16 (&sacc)[2]) {
  float m = -INFINITY;
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) m = fmaxf(m, sacc[mb][v]);
  return m;
}

// Online softmax: the row's running maximum m_run takes in that of a piece, `m`, unless the row sees nothing of it.  Returns what the
// piece's exponents are taken against, and in alpha what the sums so far are to be multiplied by.  For every piece: a rescale put off until
// a maximum has grown by some factor (FlashAttention-4 does so) takes a fifth of a piece's vector instructions out, but the largest
// probability is then no longer 1, which bf16 holds exactly, and the error of O grew by 7 % for a window of 512 over 32768 tokens (2.18e-3
// -> 2.33e-3 of its norm) and by 21 % with scores four times as wide (1.73e-3 -> 2.10e-3).
__device__ __forceinline__ float new_maximum(float m, bool sees, float c2, float& m_run, float& alpha) {
  const float m_new = sees ? fmaxf(m_run, m) : m_run;
  const float mc = m_new == -INFINITY ? 0.f : m_new * c2;
  alpha = __builtin_amdgcn_exp2f(fmaf(m_run, c2, -mc));  // exp2(-inf) = 0 on the first piece with a score
  m_run = m_new;
  return mc;
}

// Probabilities of contraction step sp, rounded to bf16 as the B operand of the PV product; their sum goes to l.
__device__ __forceinline__ bf16x8 piece_probabilities(const f32x16 (&sacc)[2], int sp, float c2, float mc, float& l) {
  bf16x8 pf;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float p = __builtin_amdgcn_exp2f(fmaf(sacc[sp >> 1][8 * (sp & 1) + e], c2, -mc));
    l += p;
    pf[e] = (bf16_t)p;
  }
  return pf;
}

__device__ __forceinline__ bf16x8 value_frag(const uint32_t (&vaddr)[2][4], int sp, int db) {
  const bf16x4 a0 = lds_read_tr_at(vaddr[0][db] + 16 * sp * kPieceRow), a1 = lds_read_tr_at(vaddr[1][db] + 16 * sp * kPieceRow);
  return __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
}
// The rest of a piece, O^T += V^T P^T, beside the scores of the next one (of whatever lies in its K tile) and their maximum over this lane's
// keys, which is returned.  A wavefront issues in order, and left to themselves the two products and the exponentials come one after the
// other, and every product waits for its own LDS read.  So the order is fixed by hand: 32 steps of one product, the LDS read of the
// product four steps on, the exponentials that are due (those of contraction step sp of the PV product four products before it), the rescale of the
// sums before the PV product and whatever `beside(step)` issues: the loads of pieces to come, which would hold the wavefront up if they were issued at once.  Without
// the rescale it measured 1040 clocks, of which the products need 1024; with it the kernels take 0.5 % (k_fwd_dense_merge, nine pieces) to 6 %
// (k_fwd_short, 6000 tokens) longer.
template <class Beside>
__device__ __forceinline__ float piece_values_and_next_scores(const uint32_t (&kaddr)[8], const uint32_t (&vaddr)[2][4],
                                                              const bf16x8 (&qf)[8], float c2, float mc, float alpha, const f32x16 (&cur)[2],
                                                              f32x16 (&next)[2], float& l_run, f32x16 (&oacc)[4], Beside beside) {
  constexpr int kAhead = 4;
  bf16x8 frag[kAhead], pf[4];
  float p[8], l = 0.f, m = -INFINITY;
  auto read = [&](int i) __attribute__((always_inline)) {  // operand of product i
    return i < 16 ? lds_read_frag(kaddr[i >> 1] + 32 * (i & 1) * kPieceRow) : value_frag(vaddr, (i - 16) >> 2, (i - 16) & 3);
  };
#pragma unroll
  for (int i = 0; i < kAhead; ++i) frag[i] = read(i);
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) next[mb][v] = 0.f;
  int done = 0;  // exponentials
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    __builtin_amdgcn_sched_barrier(0);
    if (i < 16) next[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i % kAhead], qf[i >> 1], next[i & 1], 0, 0, 0);
    else oacc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i % kAhead], pf[(i - 16) >> 2], oacc[i & 3], 0, 0, 0);
    if (i + kAhead < 32) frag[i % kAhead] = read(i + kAhead);
    beside(i);
    if (i < 16) {
#pragma unroll
      for (int v = 0; v < 4; ++v) oacc[i >> 2][4 * (i & 3) + v] *= alpha;
    }
    const int due = i < 28 ? (32 * (i + 1) + 27) / 28 : 32;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (done >= due) break;
      p[done & 7] = __builtin_amdgcn_exp2f(fmaf(cur[done >> 4][done & 15], c2, -mc));
      l += p[done & 7];
      ++done;
      if ((done & 7) == 0) {
#pragma unroll
        for (int c = 0; c < 8; ++c) pf[(done >> 3) - 1][c] = (bf16_t)p[c];
      }
    }
    if (i >= 18 && i < 26) m = fmaxf(fmaxf(m, next[0][2 * i - 36]), next[0][2 * i - 35]);
    if (i >= 24) m = fmaxf(fmaxf(m, next[1][2 * i - 48]), next[1][2 * i - 47]);
    asm volatile("" : "+v"(l), "+v"(m));  // sum and maximum are taken here, not after the last product
  }
  __builtin_amdgcn_sched_barrier(0);
  l_run = fmaf(l_run, alpha, l + __shfl_xor(l, 32));
  return m;
}

// The same for the last piece, after which no scores are wanted.
__device__ __forceinline__ void piece_values(const uint32_t (&vaddr)[2][4], float c2, float mc, float alpha, const f32x16 (&cur)[2],
                                             float& l_run, f32x16 (&oacc)[4]) {
  float l = 0.f;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[db][v] *= alpha;
#pragma unroll
  for (int sp = 0; sp < 4; ++sp) {
    __builtin_amdgcn_sched_barrier(0);
    const bf16x8 pf = piece_probabilities(cur, sp, c2, mc, l);
#pragma unroll
    for (int db = 0; db < 4; ++db) oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(value_frag(vaddr, sp, db), pf, oacc[db], 0, 0, 0);
  }
  l_run = fmaf(l_run, alpha, l + __shfl_xor(l, 32));
}

// Q's fragments are there.  In front of a loop whose loads go to LDS by assembly: the compiler does not count those and would
// wait inside the loop for as many accesses as Q's loads were, which are then the ones in flight for the next piece.
__device__ __forceinline__ void await_rows(bf16x8 (&qf)[8]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(qf[s]));
}

// The reads of a piece differ from these addresses by immediate offsets only: keeps the compiler from working out more of them.
__device__ __forceinline__ void keep_addresses(uint32_t (&kaddr)[8], uint32_t (&vaddr)[2][4]) {
  asm volatile("" : "+v"(kaddr[0]), "+v"(kaddr[1]), "+v"(kaddr[2]), "+v"(kaddr[3]), "+v"(kaddr[4]), "+v"(kaddr[5]),
               "+v"(kaddr[6]), "+v"(kaddr[7]));
  asm volatile("" : "+v"(vaddr[0][0]), "+v"(vaddr[0][1]), "+v"(vaddr[0][2]), "+v"(vaddr[0][3]), "+v"(vaddr[1][0]),
               "+v"(vaddr[1][1]), "+v"(vaddr[1][2]), "+v"(vaddr[1][3]));
}

}  // namespace nsa
