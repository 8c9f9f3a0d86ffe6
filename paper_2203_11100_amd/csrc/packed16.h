// Packed half-precision cell arithmetic shared by the inter-task kernels.  A
// 32-bit register holds two independent cells (bits 0..15 and 16..31) as
// IEEE binary16 values.
//
// Exactness.  Every quantity of the recurrence is an integer, and binary16
// holds every integer of magnitude <= 2048 exactly, so sums, differences and
// maxima of such values are exact while they stay in that range.  Let the
// rescoring limit be L <= 2048 and the gap penalties o, e <= 2048 (larger
// ones are passed as 2048: in the exact regime H < 2048, so H - o and
// E - e are negative either way and meet a max with 0).  Suppose every
// cell that (i, j) depends on has H < L and was computed exactly.  Then
// E(i, j) and F(i, j) are maxima of 0 and differences of integers in
// [0, 2048], all exact and below L; and H_diag + S, exact or not, is at most
// the true H(i, j).  So if the true H(i, j) < L, the sum is below 2048 and
// exact, and H(i, j) is exact; if the true H(i, j) >= L, then H_diag + S >= L
// and its rounding (monotone, 2048 representable) is still >= L, so the
// computed maximum reaches L.  By induction: a sequence whose true score is
// below L is scored exactly, and one whose score is L or more ends with a
// computed maximum >= L and is rescored exactly in 32-bit integers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plans.h"

namespace swdb {

typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ h16x2 as_h2(uint32_t a) { return __builtin_bit_cast(h16x2, a); }
__device__ __forceinline__ uint32_t as_u32(h16x2 a) { return __builtin_bit_cast(uint32_t, a); }

// per half: a + b, a - b (v_pk_add_f16)
__device__ __forceinline__ uint32_t hadd(uint32_t a, uint32_t b) { return as_u32(as_h2(a) + as_h2(b)); }
__device__ __forceinline__ uint32_t hsub(uint32_t a, uint32_t b) { return as_u32(as_h2(a) - as_h2(b)); }
// per half: a * b + c (v_pk_fma_f16).  With a = (S_x, 1) and b = (1, S_y)
// it is c + (S_x, S_y): the products by 1 are exact and the sum rounds
// once, exactly as the add would.
__device__ __forceinline__ uint32_t hfma(uint32_t a, uint32_t b, uint32_t c) {
  return as_u32(__builtin_elementwise_fma(as_h2(a), as_h2(b), as_h2(c)));
}
// per half: max(a, b) and max(a, b, c) (v_pk_maximum3_f16)
__device__ __forceinline__ uint32_t hmax2(uint32_t a, uint32_t b) {
  return as_u32(__builtin_elementwise_maximum(as_h2(a), as_h2(b)));
}
__device__ __forceinline__ uint32_t hmax3(uint32_t a, uint32_t b, uint32_t c) {
  return as_u32(__builtin_elementwise_maximum(__builtin_elementwise_maximum(as_h2(a), as_h2(b)),
                                              as_h2(c)));
}

// Score in one half of a register of maxima, as an integer, or -1 when it
// reaches `limit` (infinity included) and the sequence must be rescored.
__device__ __forceinline__ int half_score(uint32_t v, int half, int limit) {
  const float f = (float)__builtin_bit_cast(_Float16, (uint16_t)(v >> (16 * half)));
  return f < (float)limit ? (int)f : -1;
}

// One cell of Gotoh's recurrence on both halves, with E and F kept as
// max(E, 0) and max(F, 0) (then H = max(H_diag + S, E, F) needs no 0):
//   h = max(d, E, F);  t = h - o;  E = max(E - e, t, 0);  F = max(F - e, t, 0)
// where d = H(i-1, j-1) + S(a_i, b_j).  Returns h.
__device__ __forceinline__ uint32_t cell_from_diag(uint32_t d, uint32_t& E, uint32_t& F,
                                                   uint32_t go, uint32_t ge) {
  const uint32_t h = hmax3(d, E, F);
  const uint32_t t = hsub(h, go);
  E = hmax3(hsub(E, ge), t, 0u);
  F = hmax3(hsub(F, ge), t, 0u);
  return h;
}

// The cell with packed scores p: hd enters as H(i-1, j-1) and leaves as
// H(i, j-1) (the next row's diagonal); H enters as H(i, j-1) and leaves as
// H(i, j).  Returns h.
__device__ __forceinline__ uint32_t cell(uint32_t& hd, uint32_t& H, uint32_t& E, uint32_t& F,
                                         uint32_t p, uint32_t go, uint32_t ge) {
  const uint32_t h = cell_from_diag(hadd(hd, p), E, F, go, ge);
  hd = H;
  H = h;
  return h;
}

// Scores one 4-column chunk of an R-row strip, column by column.  The
// running maximum takes two rows per 3-input max.  (Sweeping bands of two or
// four columns along anti-diagonals, which removes the wait states between
// dependent packed ops, measured 5 % and 7 % slower on gfx950.)
//   prof(jj, p)  fills p[0..R-1] with the packed scores of column jj
//   hdiag        H of the row above the strip at the column before the chunk;
//                leaves as that of the chunk's last column
//   up_h, up_f   H and F of the row above the strip, per column
//   emit(jj, h, f)  takes H and F of the strip's bottom row at column jj as
//                soon as the column is done
template <int R, class Prof, class Emit>
__device__ __forceinline__ void sweep_chunk(uint32_t (&H)[R], uint32_t (&E)[R], uint32_t& hdiag,
                                            const uint32_t (&up_h)[4], const uint32_t (&up_f)[4],
                                            uint32_t& best, uint32_t go, uint32_t ge, Prof prof,
                                            Emit emit) {
  static_assert(R % 2 == 0, "rows are taken in pairs for the maximum");
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    uint32_t p[R];
    prof(jj, p);
    uint32_t hd = hdiag;
    hdiag = up_h[jj];
    uint32_t F = up_f[jj];
    uint32_t hprev = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t h = cell_from_diag(hadd(hd, p[k]), E[k], F, go, ge);
      hd = H[k];
      H[k] = h;
      if (k & 1) best = hmax3(best, hprev, h);
      else hprev = h;
    }
    emit(jj, H[R - 1], F);
  }
}

// sweep_chunk with the profile reads issued one column ahead: while row pair
// k2 of column jj is computed, row pair k2 of column jj + 1 is read, so the
// reads' latency hides behind a column of arithmetic (the chunk's first
// column is read at its start).  The registers held stay those of one
// column: a row pair's old values die as its new ones are read.  (Reading
// the next chunk's first column during the last column as well keeps those
// registers live across the chunk boundary and spills.)
//   prof_pair(jj, k2, a, b)  reads row pair k2 of column jj: with kSplit,
//                a = the low table's two (S, 1) dwords and b = the high
//                table's two (1, S) dwords, one fused multiply-add per cell
//                forming H_diag + S (see hfma); without, a = the two rows'
//                packed scores, added to H_diag (b unused)
//   emit(jj, h, f)  takes H and F of the strip's bottom row at column jj as
//                soon as the column is done (stored at once, the registers
//                of the four columns' results are not held to the chunk's end)
template <int R, bool kSplit, class ProfPair, class Emit>
__device__ __forceinline__ void sweep_chunk_ahead(uint32_t (&H)[R], uint32_t (&E)[R],
                                                  uint32_t& hdiag, const uint32_t (&up_h)[4],
                                                  const uint32_t (&up_f)[4], uint32_t& best,
                                                  uint32_t go, uint32_t ge, ProfPair prof_pair,
                                                  Emit emit) {
  static_assert(R % 2 == 0, "rows are taken in pairs");
  // VALU and SALU may cross the scheduling barriers; LDS reads may not
  constexpr int kMayCross = 0x0002 | 0x0004;
  uint2 a[R / 2], b[R / 2];
#pragma unroll
  for (int k2 = 0; k2 < R / 2; ++k2) prof_pair(0, k2, a[k2], b[k2]);
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    uint32_t hd = hdiag;
    hdiag = up_h[jj];
    uint32_t F = up_f[jj];
#pragma unroll
    for (int k2 = 0; k2 < R / 2; ++k2) {
      // an empty asm taking the F that enters the row pair keeps the first
      // use of its scores (read a column earlier) where the F chain reaches it
      if (kSplit) asm volatile("" : "+v"(a[k2]), "+v"(b[k2]) : "v"(F));
      else asm volatile("" : "+v"(a[k2]) : "v"(F));
      const uint2 ca = a[k2], cb = b[k2];
      if (jj < 3) {
        prof_pair(jj + 1, k2, a[k2], b[k2]);
        __builtin_amdgcn_sched_barrier(kMayCross);
      }
      const uint32_t d0 = kSplit ? hfma(ca.x, cb.x, hd) : hadd(hd, ca.x);
      const uint32_t h0 = cell_from_diag(d0, E[2 * k2], F, go, ge);
      hd = H[2 * k2];
      H[2 * k2] = h0;
      const uint32_t d1 = kSplit ? hfma(ca.y, cb.y, hd) : hadd(hd, ca.y);
      const uint32_t h1 = cell_from_diag(d1, E[2 * k2 + 1], F, go, ge);
      hd = H[2 * k2 + 1];
      H[2 * k2 + 1] = h1;
      best = hmax3(best, h0, h1);
    }
    emit(jj, H[R - 1], F);
  }
}

// ---------------------------------------------------------------------------
// Drift cells: the same recurrence in packed 16-bit integers, every value
// stored with ge added once per row and once per column:
//   X~(i, j) = X(i, j) + base + ge * (i + j).
// A gap that is extended moves one row or one column, so what it costs is
// what the drift adds and E~ and F~ need no subtraction:
//   E~' = max(E~, H~ - c, Z)   F~' = max(F~, H~ - c)   c = go - ge
//   H~  = max(H~diag + S + 2 ge, E~, F~)
// where Z(i, j) = base + ge * (i + j) stands for 0; only E is floored (H~ is
// at least E~, and an F~ below Z never wins).  A cell pair takes 5 packed ops
// and half of one for the running maximum, against the 7 and a half of the
// form above, and one of them, the subtraction of c, is a 32-bit one on two
// registers, which gfx950 issues at nearly twice the packed rate (2.6 against
// 4.4 cycles a wave and SIMD, measured; not with a scalar operand).
//
// The maxima are v_pk_maximum3_f16 and compare the integers as binary16 bit
// patterns: for 0 .. 31743 (0x7bff, the largest finite pattern) that order is
// the integers' own.  Range: the host (drift_plan in runtime.hip) takes this
// form only when every value stays within 0 .. 31743: base = kDriftBase keeps
// H~ - c and H~diag + S above 0 (c is passed as at most 2048, which no score
// below the limit survives), and the drift starts again at base every
// `group` strips.  A sequence that reaches the limit is rescored, so from
// then on its values need only stay in range: either no score can leave it
// (min(m, columns) * max S fits, the usual case), or `guard` sets the state of
// such a half back to Z at the end of every chunk.
//
// Global and semi-global scores (k_inter.hip) have no floor; their values stay
// above base because a gap along a border costs its opening only, so `base` is
// 3 go + 256 for them, and below it plus a bounded gain (mode_plan).
//
// The running maximum is of H = H~ - Z.  All cells of an anti-diagonal have
// the same Z, so A[k] carries the maximum of the anti-diagonal through row k
// of the last odd column: at odd columns A[k] = max(A[k + 2], the cell, the
// cell left and below of it), two cells an op, in place, and an anti-diagonal
// that has reached row 0 is complete and enters `best` less its Z.
enum { kCellHalf = 0, kCellDrift = 1, kCellGlobal = 2, kCellSemi = 3 };   // cell forms

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_u2(uint32_t a) { return __builtin_bit_cast(u16x2, a); }
__device__ __forceinline__ uint32_t from_u2(u16x2 a) { return __builtin_bit_cast(uint32_t, a); }
// per half: a * b, max(a, b), min(a, b), max(a - b, 0)
__device__ __forceinline__ uint32_t umul2(uint32_t a, uint32_t b) {
  return from_u2(as_u2(a) * as_u2(b));
}
__device__ __forceinline__ uint32_t umax2(uint32_t a, uint32_t b) {
  return from_u2(__builtin_elementwise_max(as_u2(a), as_u2(b)));
}
__device__ __forceinline__ uint32_t umin2(uint32_t a, uint32_t b) {
  return from_u2(__builtin_elementwise_min(as_u2(a), as_u2(b)));
}
__device__ __forceinline__ uint32_t usub2_sat(uint32_t a, uint32_t b) {
  return from_u2(__builtin_elementwise_sub_sat(as_u2(a), as_u2(b)));
}
__device__ __forceinline__ uint32_t twice(uint32_t v) { return v | (v << 16); }

// Score in one half of a register of maxima, or -1 at the limit and above.
__device__ __forceinline__ int drift_score(uint32_t v, int half, int limit) {
  const int s = (int)((v >> (16 * half)) & 0xffffu);
  return s < limit ? s : -1;
}

// The row above a strip, where its values need more than reading: the first
// strip (delta2 = 0xffff in both halves: the border, H = 0, whatever was
// read), the first strip of a drift group (delta2 = the group's drift) and
// every strip under `guard` (values cut at the limit).  zu = Z of the row
// above and the chunk's first column, lim2 = the limit in both halves.
__device__ __forceinline__ void drift_adjust(uint32_t (&up_h)[4], uint32_t (&up_f)[4],
                                             uint32_t delta2, uint32_t zu, uint32_t ge2,
                                             uint32_t lim2) {
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const uint32_t z = zu + ge2 * (uint32_t)jj;
    up_h[jj] = umin2(umax2(usub2_sat(up_h[jj], delta2), z), z + lim2);
    up_f[jj] = umin2(usub2_sat(up_f[jj], delta2), z + lim2);
  }
}

// Starts a strip: the cells left of column 0 (H = 0, E floored), z0 = Z of
// row 0 and column 0.
template <int R>
__device__ __forceinline__ void drift_start(uint32_t (&H)[R], uint32_t (&E)[R], uint32_t (&A)[R],
                                            uint32_t& hdiag, uint32_t z0, uint32_t ge2) {
#pragma unroll
  for (int k = 0; k < R; ++k) {
    E[k] = z0 + ge2 * (uint32_t)k;
    H[k] = E[k] - ge2;
    A[k] = 0;
  }
  hdiag = z0 - 2 * ge2;
}

// Ends a strip: the anti-diagonals that have not reached row 0, z = Z of row
// 0 and the last column.
template <int R>
__device__ __forceinline__ void drift_finish(const uint32_t (&A)[R], uint32_t& best, uint32_t z,
                                             uint32_t ge2) {
#pragma unroll
  for (int k = 1; k < R; ++k) best = umax2(best, A[k] - (z + ge2 * (uint32_t)k));
}

// One 4-column chunk of an R-row strip.  prof_pair and emit as in
// sweep_chunk_ahead, the profile read one column ahead in the same way; with
// kSplit a and b hold the two tables' dwords, S + 2 ge as a 32-bit integer and
// the same shifted up 16 bits (one three-input 32-bit addition forms H~diag + S
// for both halves: every half's result is in 0 .. 65535, so what a negative
// score borrows from the high half the sum gives back), without a = both
// queries' scores in one such sum.  cv is c2 in a vector register, zc = Z of
// row 0 and the chunk's first column.  Nothing crosses the barrier between two
// row pairs: let the arithmetic cross and the compiler fills the wait states
// between dependent packed ops from the next pairs (6 instead of 60 a chunk at
// 14 rows) for registers that are not there, 20 rows spilling 25 of them, and
// 1-3 % of the time.
// Without kLocal (global and semi-global scores) there is no floor and no
// running maximum: 5 ops, and A, best and the Z are not used.
template <int R, bool kSplit, bool kLocal, class ProfPair, class Emit>
__device__ __forceinline__ void drift_chunk(uint32_t (&H)[R], uint32_t (&E)[R], uint32_t (&A)[R],
                                            uint32_t& hdiag, const uint32_t (&up_h)[4],
                                            const uint32_t (&up_f)[4], uint32_t& best,
                                            uint32_t cv, uint32_t zc, uint32_t ge2,
                                            ProfPair prof_pair, Emit emit) {
  static_assert(R % 2 == 0, "rows are taken in pairs");
  uint2 a[R / 2], b[R / 2];
#pragma unroll
  for (int k2 = 0; k2 < R / 2; ++k2) prof_pair(0, k2, a[k2], b[k2]);
  uint32_t x = 0;
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    uint32_t hd = hdiag;
    hdiag = up_h[jj];
    uint32_t F = up_f[jj];
    // Z of each row at the next column, from scalar adds
    uint32_t z = zc + ge2 * (uint32_t)jj;
#pragma unroll
    for (int k2 = 0; k2 < R / 2; ++k2) {
      if (kSplit) asm volatile("" : "+v"(a[k2]), "+v"(b[k2]) : "v"(F));
      else asm volatile("" : "+v"(a[k2]) : "v"(F));
      const uint2 ca = a[k2], cb = b[k2];
      if (jj < 3) {
        prof_pair(jj + 1, k2, a[k2], b[k2]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        const int k = 2 * k2 + t2;
        const uint32_t pa = t2 ? ca.y : ca.x, pb = t2 ? cb.y : cb.x;
        const uint32_t d = kSplit ? hd + pa + pb : hd + pa;
        const uint32_t h = hmax3(d, E[k], F);
        const uint32_t t = h - cv;
        if (kLocal && k == 0 && !(jj & 1)) x = umax2(A[1], h) - z;
        if (kLocal && (jj & 1)) {
          if (k + 2 < R) A[k] = hmax3(A[k + 2], h, H[k + 1]);
          else if (k + 1 < R) A[k] = umax2(h, H[k + 1]);
          else A[k] = h;
          if (k == 0) best = hmax3(best, x, A[0] - z);
        }
        z += ge2;
        E[k] = kLocal ? hmax3(E[k], t, z) : umax2(E[k], t);
        F = umax2(F, t);
        hd = H[k];
        H[k] = h;
      }
    }
    emit(jj, H[R - 1], F);
  }
}

// guard: a half whose maximum has reached the limit is rescored whatever its
// later cells hold; its state goes back to Z (z = Z of row 0 and the next
// chunk's first column).  A cell enters `best` at most R - 1 columns after it
// was computed and the row above is cut at the limit, so no value passes the
// limit by more than (R + 5) * max S.  over2 = 32768 - limit in both halves.
template <int R>
__device__ __forceinline__ void drift_guard(uint32_t (&H)[R], uint32_t (&E)[R], uint32_t (&A)[R],
                                            uint32_t& hdiag, uint32_t best, uint32_t over2,
                                            uint32_t z, uint32_t ge2) {
  const uint32_t over = (best + over2) & 0x80008000u;
  if (over == 0) return;
  asm volatile("");     // a branch, not selects on every chunk
  const uint32_t m = (over >> 15) * 0xffffu;     // 0xffff in the halves to reset
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const uint32_t zk = z + ge2 * (uint32_t)k;
    E[k] = (E[k] & ~m) | (zk & m);
    H[k] = (H[k] & ~m) | ((zk - ge2) & m);
    A[k] = (A[k] & ~m) | ((zk - ge2) & m);
  }
  hdiag = (hdiag & ~m) | ((z - 2 * ge2) & m);
}

}  // namespace swdb
