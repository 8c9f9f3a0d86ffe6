// Long-pair kernel: pairs of database sequences, the two 16-bit halves of every
// register holding the two sequences of a pair, each pair on the waves of one
// workgroup (paper section 2.2: intra-task parallelism, all processing elements
// work on one alignment matrix and neighbours exchange border elements).  It
// scores the long list of single searches, the longest short bins of searches
// that would otherwise wait for them, and the very long sequences of batches, in
// the drift form of the cells (packed16.h); gap penalties that form does not take
// go through k_intra_f16.
//
// Wavefront.  The query is cut into passes of 64 R rows; lane l of a wave owns
// R consecutive rows of its pass and at step t computes column t - l of them.
// H and F of the row above come from lane l - 1, which computed them the step
// before, by one cross-lane move each (DPP wave_shr:1); lane 0 takes them, and
// the residue codes, from a line of 64 columns in LDS that every lane reads
// (one broadcast read a step in the place of a rotating register for each of
// the three), and lane 63 writes its bottom row to a second line.
//
// Drift.  A superstep is 64 steps.  Lane l carries base + ge * (tau + k) in its
// row k at step tau of the superstep: what passes from row R - 1 of lane l - 1 at
// step tau - 1 to row 0 of lane l at step tau is ge (R - 1) too high, which F
// pays by a subtraction and H~diag inside the constant added with row 0's score.
// At a superstep's end 64 ge comes off all state, so columns do not count
// against the 16-bit range, and halves at the rescoring limit go back to Z.
// The anti-diagonals of a lane are steps plus rows, so the running maximum works
// as in the strips.
//
// Profile: bytes S + 2 ge + bias (unsigned), [code][row] within a pass: a lane
// reads its R rows for each sequence's residue as one 2-, 4- or 8-byte read, 64
// consecutive pieces of one code row per wave, and one byte permute a row puts
// the two sequences' scores into the halves (zero bytes above them); the bias
// comes off in the three-input add that joins them to H~diag.  All passes of a
// query up to several thousand rows fit in LDS at once and serve every wave; of
// longer ones, and in batches, each wave stages the rows of its pass.
//
// Stream.  Workgroups take pairs, longest first, from a queue and their waves
// take the pairs' passes round robin, pair after pair without a seam, ordered by
// progress words (stream.h), two supersteps behind the pass above; a pair's passes
// hand their bottom rows on through a row buffer of its own in device memory,
// overwritten in place.
//
// Global and semi-global (kForm): no floor and no running maximum, H and F drift
// over the rows too (base + ge * (row + column): a gap along the left border
// costs its opening only, so that border is one value), and nothing comes off
// between lanes.  The global top border is one value as well and its columns'
// drift stays, the values being bounded by the gain of min(rows, columns); the
// semi-global one, H = 0, rises with the columns, whose drift comes off every
// superstep.  Before its column 0 a lane's cells keep the left border: they read
// the pad code, S = -2 ge in these forms.  The query is shifted down by less than
// R rows, as in the strips, so that its last row is the last of a lane; that
// lane's bottom row goes to the line in the last pass, and the score is taken from
// there, a superstep at a time.  Lanes below it compute what nobody reads.
//
// A step takes 8 + 6.5 R vector ops for 2 R cells (k_intra_f16: 24 + 8 R with
// the byte permutes, and barriers every 64 steps).  Bound by a pair's own chain
// of steps where pairs are few (columns times the time of a step), else by the
// VALU.  Against k_intra_f16: 211 residues, 20,001 sequences 1.10 ms a search ->
// 0.51; 1,001 bases, 3,000 sequences 1.92 -> 1.28; 2,000 residues, the long mix
// 7.05 -> 5.7; against k_intra_i32, global, 310 residues, 100,000 sequences
// 5.48 -> 2.49.
#include <type_traits>

#include "internal.h"
#include "packed16.h"
#include "stream.h"

namespace swdb {
namespace {

constexpr int kWaveShr1 = 0x138;  // DPP wave_shr:1  (lane l <- lane l-1)

// lane l <- lane l-1; lane 0 keeps `first`
__device__ __forceinline__ uint32_t shr_in(uint32_t v, uint32_t first) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, kWaveShr1, 0xf, 0xf, false);
}

template <int R> struct ByteRows;
template <> struct ByteRows<2> { typedef uint16_t T; };
template <> struct ByteRows<4> { typedef uint32_t T; };
template <> struct ByteRows<8> { typedef uint2 T; };
__device__ __forceinline__ uint32_t word_of(const uint16_t& v, int) { return v; }
__device__ __forceinline__ uint32_t word_of(const uint32_t& v, int) { return v; }
__device__ __forceinline__ uint32_t word_of(const uint2& v, int x) { return x ? v.y : v.x; }

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <int R, int W, int kForm>
__global__ __launch_bounds__(64 * W) void k_pairs(PairArgs a) {
  constexpr bool kLocal = kForm == kCellDrift;
  constexpr int ROWS = 64 * R;             // query rows per pass, bytes per code row
  constexpr int kPassBytes = kIntraCodes * ROWS;
  typedef typename ByteRows<R>::T PV;
  extern __shared__ __align__(16) char lprof_all[];
  __shared__ uint4 lfeed[W][64];           // {code offsets, H, F, -} of a superstep's columns
  // the bottom row, step by step from 1.  Every lane writes, lane 63 (in general:
  // the one whose row it is) at the step's place and the others ahead of it, where
  // the steps to come write over them: no exec mask to change, and the compiler
  // counts the store among the reads it waits for
  __shared__ uint2 lcoll[W][128];
  __shared__ uint32_t lprog[W];            // each wave's progress
  __shared__ int2 lpos[W];                 // its item: {ordinal, pass}
  __shared__ int litem[kRing];             // ordinal n's entry of the list, at n % ring
  __shared__ int lend;                     // the list is empty: items from here on hold nothing
  __shared__ int lfin[kRing];              // its finished passes
  __shared__ int lfree[kRing];             // the ordinal that may take this place next
  __shared__ uint32_t lbest[kRing][2];     // its maxima, low and high halves apart

  const uint32_t lane = threadIdx.x & 63;
  const int w = uniform(threadIdx.x >> 6);
  const int pred = w > 0 ? w - 1 : W - 1;
  const uint32_t ge2 = a.ge2;
  const uint32_t gr_s = kLocal ? ge2 * (uint32_t)(R - 1) : 0;
  uint32_t cv = a.c2, gr = gr_s;
  asm("" : "+v"(cv), "+v"(gr));            // 32-bit subtractions on two vector registers
  const uint32_t base2 = twice(kDriftBase);
  // what joins a row's byte and H~diag: less the bias, and in row 0 the drift
  // between lanes (opaque, or the compiler makes two ops of the three-input add)
  uint32_t bias_k = 0u - a.bias2, bias_0 = bias_k - gr_s;
  asm("" : "+s"(bias_k), "+s"(bias_0));
  // H and F of a zero row above, as lane 0 takes them at step `lane`
  uint32_t zero_h = base2 + ge2 * (lane + R) - 2 * ge2;
  uint32_t zero_f = base2 + ge2 * (lane + R) - ge2;
  // global and semi-global: the left border, the lane that holds the last row
  const ModeShape& md = a.mode;
  const uint32_t mbase2 = twice((uint32_t)md.base);
  const uint32_t left2 = twice((uint32_t)(md.base - md.go - md.ge + md.ge * md.pad));
  const uint32_t top2 = twice((uint32_t)(md.base - md.go + md.ge * (md.pad - 1)));
  const int last_lane = kLocal ? 63 : (md.m + md.pad) / R - 1 - (a.n_pass - 1) * 64;
  if constexpr (!kLocal) {
    zero_h = kForm == kCellGlobal ? top2 : mbase2 + ge2 * lane - ge2;
    zero_f = zero_h - a.c2;
  }

  auto stage = [&](char* dst, const uint8_t* prof, int m_pad2, int pass, int from, int step) {
    constexpr int per_code = ROWS / 16;    // uint4 per code row
    uint4* d = reinterpret_cast<uint4*>(dst);
    for (int x = from; x < kIntraCodes * per_code; x += step) {
      const int code = x / per_code, r = x - code * per_code;
      d[x] = *reinterpret_cast<const uint4*>(prof + (size_t)code * m_pad2 + (size_t)pass * ROWS +
                                             16 * r);
    }
  };
  if (a.shared)
    for (int p = 0; p < a.n_pass; ++p)
      stage(lprof_all + p * kPassBytes, a.prof, a.m_pad2, p, threadIdx.x, 64 * W);
  if (threadIdx.x < W) lprog[threadIdx.x] = ~0u;       // before its first item's start, 0
  if (threadIdx.x == 0) lend = 0;
  if (threadIdx.x < kRing) {
    lfin[threadIdx.x] = 0;
    lfree[threadIdx.x] = (int)threadIdx.x;
    lbest[threadIdx.x][0] = lbest[threadIdx.x][1] = 0;
  }
  __syncthreads();

  uint32_t known = ~0u;                    // the predecessor's progress as last read
  auto wait_pred = [&](uint32_t need) { wait_progress(&lprog[pred], known, need); };
  auto passes_of = [&](int it) {
    return a.batch_items ? uniform(a.queries[a.batch_items[it].y].n_pass3) : a.n_pass;
  };

  for (uint32_t k = 0;; ++k) {
    // Item g = k * W + w follows item g - 1: the next pass of its pair, or the
    // first of the next entry of the list.  Items start in that order (so that
    // entries are taken in order, the longest first, and every wave ends at its
    // first item past the list's end) and wait for smaller ones only - a pass
    // for the one before it, superstep by superstep, a pair's first for the pair a
    // ring before to be finished - so every wait ends.
    const uint32_t here = k << kProgBits;
    const uint32_t there = (w > 0 ? k : k - 1) << kProgBits;   // item g - 1 in its wave's count
    int n = 0, p = 0;
    if (k > 0 || w > 0) {
      wait_pred(there);
      if (!peek(&lend)) {
        n = peek(&lpos[pred].x);
        p = peek(&lpos[pred].y) + 1;
        if (p >= passes_of(peek(&litem[n % a.ring]))) {
          p = 0;
          ++n;
        }
      }
    }
    const int slot = n % a.ring;
    int it = -1;
    if (!peek(&lend)) {
      if (p > 0) {
        it = peek(&litem[slot]);
      } else {
        while (peek(&lfree[slot]) != n) poll_pause();
        if (lane == 0) it = atomicAdd(a.counter, 1);
        it = uniform(it);
        if (it >= a.count) {
          it = -1;
          publish(&lend, 1);
        } else if (lane == 0) {
          litem[slot] = it;
        }
      }
    }
    it = uniform(it);
    if (it < 0) {
      publish(&lprog[w], here + (1u << kProgBits) - 1);
      break;
    }
    if (lane == 0) lpos[w] = make_int2(n, p);
    publish(&lprog[w], here);
    const int P = passes_of(it);

    const int2 seg = a.seg_items ? a.seg_items[it] : make_int2(it, 0);
    const int2 bitem = a.batch_items ? a.batch_items[it] : make_int2(seg.x, 0);
    const uint8_t* prof = a.prof;
    int m_pad2 = a.m_pad2;
    int64_t out_off = 0;
    if (a.batch_items) {
      const QueryDesc qd = a.queries[bitem.y];
      prof += qd.prof3_off;
      m_pad2 = qd.m_pad2;
      out_off = qd.out_off;
    }
    const int2 item = a.items[bitem.x];
    const int sa = uniform(item.x), sb = uniform(item.y);
    const int64_t ba = a.offs[sa];
    int na = uniform((int)(a.offs[sa + 1] - ba));
    const int64_t bb = sb >= 0 ? a.offs[sb] : 0;
    int nb = sb >= 0 ? uniform((int)(a.offs[sb + 1] - bb)) : 0;
    const uint8_t* __restrict__ sqa = a.res + ba;
    const uint8_t* __restrict__ sqb = a.res + bb;
    if (a.seg_items) {
      // the segment's window: columns [c0, hi) of both sequences, each cut to
      // its own length (a is the longer one: na = 0 only for two empty sequences)
      const int lo = uniform(seg.y) * a.seg_cols;
      const int hi = min(na, lo + a.seg_cols);
      const int c0 = max(0, lo - a.seg_overlap);
      na = hi - c0;
      nb = max(0, min(nb, hi) - c0);
      sqa += c0;
      sqb += c0;
    }
    if (nb == 0) sqb = sqa;       // an empty b reads a's residues (clamped, in bounds)
    const int cols = max(na, nb);
    // two empty sequences: no superstep, no residue or boundary row read
    const int C = cols > 0 ? (cols + 63 + 63) >> 6 : 0;
    uint2* __restrict__ rb =
        a.scratch + ((size_t)blockIdx.x * a.ring + (size_t)slot) * a.scratch_stride;
    char* const lprof = lprof_all + (a.shared ? p : w) * kPassBytes;
    if (!a.shared) {
      stage(lprof, prof, m_pad2, p, (int)lane, 64);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);   // LDS of one wave executes in order
    }
    const char* lb = lprof + lane * R;

    // the next superstep's inputs, loaded a superstep ahead: the raw residue
    // bytes and the row above, every index clamped into bounds, what lies
    // outside replaced where they are used
    uint32_t ca_n = 0, cb_n = 0;
    uint2 up_n = make_uint2(0, 0);
    auto fetch = [&](int c) {
      const int jf = c * 64 + (int)lane;
      ca_n = sqa[min(jf, na - 1)];
      cb_n = sqb[min(jf, max(nb - 1, 0))];
      if (p > 0) up_n = rb[min(jf, cols - 1)];
    };

    uint32_t H[R], E[R], A[R];
    uint32_t best = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      E[r] = base2 + ge2 * (uint32_t)r;
      H[r] = E[r] - ge2;
      A[r] = 0;
    }
    // true 0 as lane l - 1 passes it on; an F far below Z, above 0 after gr
    uint32_t hdiag = base2 + ge2 * (uint32_t)R - 3 * ge2;
    const uint32_t low_f = base2 - twice(2048) + gr_s;
    uint32_t fbot = low_f;
    uint32_t score = 0;
    const int out_lane = p == P - 1 ? last_lane : 63;
    if constexpr (!kLocal) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        H[r] = left2;
        E[r] = left2 - a.c2;
      }
      hdiag = left2;
      fbot = left2 - a.c2;
      if (p == 0 && lane == 0) {
        const uint32_t corner2 = mbase2 + ge2 * (uint32_t)md.pad - 2 * ge2;   // H(0, 0) = 0
        hdiag = kForm == kCellGlobal && md.pad > 0 ? top2 : mbase2 - 2 * ge2;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (r < md.pad) {
            if (kForm == kCellGlobal) {
              H[r] = r == md.pad - 1 ? corner2 : top2;
              E[r] = top2;
            } else {
              H[r] = mbase2 + ge2 * (uint32_t)r - ge2;
              E[r] = H[r] - a.c2;
            }
          }
        }
      }
    }
    uint32_t code = twice((uint32_t)(SW_PAD_CODE * ROWS));
    if (C > 0) {
      if (p > 0) wait_pred(there + (uint32_t)min(2, C));
      fetch(0);
    }
    for (int c = 0; c < C; ++c) {
      {
        const int jf = c * 64 + (int)lane;
        const uint32_t x = jf < na ? ca_n : (uint32_t)SW_PAD_CODE;
        const uint32_t y = jf < nb ? cb_n : (uint32_t)SW_PAD_CODE;
        const bool up = p > 0 && jf < cols;
        // cut at the limit: such a sequence is rescored, its values only have to
        // stay in range
        const uint32_t up_h = kLocal ? umin2(up_n.x, zero_h + a.lim2) : up_n.x;
        const uint32_t up_f = kLocal ? umin2(up_n.y, zero_f + a.lim2) : up_n.y;
        lfeed[w][lane] = make_uint4(x * ROWS | (y * ROWS) << 16, up ? up_h : zero_h,
                                    up ? up_f : zero_f, 0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
      }
      if (c + 1 < C) {
        if (p > 0) wait_pred(there + (uint32_t)min(c + 3, C));
        fetch(c + 1);
      }
      if (kForm != kCellGlobal && c > 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          H[r] -= 64 * ge2;
          E[r] -= 64 * ge2;
          if (kLocal) A[r] -= 64 * ge2;
        }
        hdiag -= 64 * ge2;
        fbot -= 64 * ge2;
      }
      // the codes of step tau + 1 are those of step tau a lane on, so each
      // step's profile rows are read two steps ahead, the first two at the
      // start (and the line's entries four steps ahead, past its end the first
      // again): a read takes about as long as a step of few rows (one and two
      // steps ahead: 0.219 ms instead of 0.190 at 144 residues against 2,000
      // sequences, two rows)
      // (the three words used of an entry alone: a fourth would be a register in
      // flight that holds nothing and is given out again, behind a wait)
      auto feed = [&](int i) { return *reinterpret_cast<const u32x3*>(&lfeed[w][i]); };
      u32x3 f0 = feed(0), f1 = feed(1), f2 = feed(2), f3 = feed(3);
      PV va[2], vb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        code = shr_in(code, i == 0 ? f0.x : f1.x);
        va[i] = *reinterpret_cast<const PV*>(lb + (code & 0xffffu));
        vb[i] = *reinterpret_cast<const PV*>(lb + (code >> 16));
      }
      uint2* coll = &lcoll[w][(out_lane - (int)lane) & 63];
      uint32_t code_63 = 0;
      uint32_t x = 0;
      for (int g = 0; g < 8; ++g) {
        const uint32_t zg = base2 + ge2 * (uint32_t)(8 * g);
        auto step = [&](auto uc) {
          constexpr int u = decltype(uc)::value;
          // the last step's bottom row, then this step's reads; nothing of the next
          // step may be scheduled before them
          coll[u] = make_uint2(H[R - 1], fbot);
          code = shr_in(code, f2.x);
          if (u == 5) code_63 = code;
          const u32x3 f4 = feed((8 * g + u + 4) & 63);
          const PV va_n = *reinterpret_cast<const PV*>(lb + (code & 0xffffu));
          const PV vb_n = *reinterpret_cast<const PV*>(lb + (code >> 16));
          const uint32_t hup = shr_in(H[R - 1], f0.y);
          const uint32_t fup = shr_in(fbot, f0.z);
          __builtin_amdgcn_sched_barrier(0);
          uint32_t hd = hdiag;
          hdiag = hup;
          uint32_t F = kLocal ? fup - gr : fup;
          uint32_t z = zg + ge2 * (uint32_t)u;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const uint32_t s = __builtin_amdgcn_perm(
                word_of(vb[0], r >> 2), word_of(va[0], r >> 2),
                0x0c000c00u | (uint32_t)(r & 3) | (uint32_t)(4 + (r & 3)) << 16);
            const uint32_t d = hd + s + (r == 0 ? bias_0 : bias_k);
            const uint32_t h = hmax3(d, E[r], F);
            const uint32_t t = h - cv;
            if (kLocal && r == 0 && !(u & 1)) x = umax2(A[1], h) - z;
            if (kLocal && (u & 1)) {
              if (r + 2 < R) A[r] = hmax3(A[r + 2], h, H[r + 1]);
              else if (r + 1 < R) A[r] = umax2(h, H[r + 1]);
              else A[r] = h;
              if (r == 0) best = hmax3(best, x, A[0] - z);
            }
            z += ge2;
            E[r] = kLocal ? hmax3(E[r], t, z) : umax2(E[r], t);
            F = umax2(F, t);
            hd = H[r];
            H[r] = h;
          }
          fbot = F;
          __builtin_amdgcn_sched_barrier(0);
          va[0] = va[1];
          vb[0] = vb[1];
          va[1] = va_n;
          vb[1] = vb_n;
          f0 = f1;
          f1 = f2;
          f2 = f3;
          f3 = f4;
        };
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
        step(std::integral_constant<int, 2>());
        step(std::integral_constant<int, 3>());
        step(std::integral_constant<int, 4>());
        step(std::integral_constant<int, 5>());
        step(std::integral_constant<int, 6>());
        step(std::integral_constant<int, 7>());
        coll += 8;
      }
      coll[0] = make_uint2(H[R - 1], fbot);
      code = code_63;   // `code` ran two steps ahead: back to the last step's own
      asm volatile("" ::: "memory");
      const uint2 low = lcoll[w][lane + 1];
      const int jo = c * 64 + (int)lane - out_lane;
      if (p < P - 1 && jo >= 0 && jo < cols) {
        // what the next pass finds there in its superstep, by this one's drift:
        // lane 63's column is the first of the superstep after (local cells), or
        // the others' are a superstep back (semi-global)
        uint32_t off = lane == 63 ? 64 * ge2 : 0u;
        if (kForm == kCellSemi) off -= 64 * ge2;
        if (kForm == kCellGlobal) off = 0;
        rb[jo] = make_uint2(low.x - off, low.y - off);
      }
      if constexpr (!kLocal) {
        if (p == P - 1) {
          // 0xffff in the halves whose sequence ends with this column or has it
          const bool ina = kForm == kCellGlobal ? jo == na - 1 : jo >= 0 && jo < na;
          const bool inb = kForm == kCellGlobal ? jo == nb - 1 : jo >= 0 && jo < nb;
          const uint32_t in = (ina && na > 0 ? 0xffffu : 0u) | (inb && nb > 0 ? 0xffff0000u : 0u);
          const uint32_t v =
              kForm == kCellGlobal ? low.x : low.x + ge2 * (uint32_t)(out_lane - (int)lane);
          score = umax2(score, v & in);
        }
      }
      publish(&lprog[w], here + (uint32_t)c + 1);
      // a lane whose maximum has reached the limit starts again from Z in that
      // half: what a lane takes from the one above it enters its maximum at once,
      // so no value passes the limit by more than two supersteps' gain
      const uint32_t over = kLocal ? (best + a.over2) & 0x80008000u : 0;
      if (over != 0) {
        drift_guard<R>(H, E, A, hdiag, best, a.over2, base2 + 64 * ge2, ge2);
        const uint32_t m = (over >> 15) * 0xffffu;
        fbot = (fbot & ~m) | ((low_f + 64 * ge2) & m);
      }
    }
    if (kLocal && C > 0) drift_finish<R>(A, best, base2 + 63 * ge2, ge2);
    if (!kLocal) best = score;

#pragma unroll
    for (int off = 32; off > 0; off >>= 1) best = umax2(best, (uint32_t)__shfl_xor((int)best, off, 64));
    int fin = 0;
    if (!kLocal && p == P - 1 && lane == 0) {
      // H~ less base and the drift of the last row (and, global, of the last column)
      const int rows = md.base + md.ge * (md.m + md.pad - 1);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int sid = half ? sb : sa, n_h = half ? nb : na;
        if (sid < 0) continue;
        const int v = (int)(half ? best >> 16 : best & 0xffffu);
        a.out[sid] = n_h == 0 ? -(md.go + (md.m - 1) * md.ge)
                              : v - rows - (kForm == kCellGlobal ? md.ge * (n_h - 1) : 0);
      }
    }
    if (lane == 0) {
      atomicMax(&lbest[slot][0], best & 0xffffu);
      atomicMax(&lbest[slot][1], best >> 16);
      fin = __hip_atomic_fetch_add(&lfin[slot], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (uniform(fin) == P - 1 && lane == 0) {
      // the pair's last pass: a segment's maximum, or per half the score or, at
      // the rescoring limit, an entry of the rescoring list
      const uint32_t b0 = lbest[slot][0], b1 = lbest[slot][1];
      lbest[slot][0] = lbest[slot][1] = 0;
      if (!kLocal) {
        // the scores are out
      } else if (a.seg_best) {
        a.seg_best[it] = b0 | (b1 << 16);
      } else {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int sid = half ? sb : sa;
          if (sid < 0) continue;
          const int score = drift_score(half ? b1 : b0, 0, a.sat_limit);
          if (score < 0) {
            const int idx = atomicAdd(a.flag_count, 1);
            a.flag_list[idx] = make_int2(sid, bitem.y);
          } else {
            a.out[out_off + sid] = score;
          }
        }
      }
      lfin[slot] = 0;
      publish(&lfree[slot], n + a.ring);
    }
  }
}

template <int R, int W>
hipError_t launch_rw(int grid, size_t lds, const PairArgs& a, hipStream_t s) {
  const dim3 block(64 * W);
  if (a.mode.mode == SW_MODE_GLOBAL)
    hipLaunchKernelGGL((k_pairs<R, W, kCellGlobal>), dim3(grid), block, lds, s, a);
  else if (a.mode.mode == SW_MODE_SEMIGLOBAL)
    hipLaunchKernelGGL((k_pairs<R, W, kCellSemi>), dim3(grid), block, lds, s, a);
  else
    hipLaunchKernelGGL((k_pairs<R, W, kCellDrift>), dim3(grid), block, lds, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pairs(int R, int W, int grid, const PairArgs& a, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  const size_t lds = pairs_lds(R, W, a.n_pass, a.shared != 0);
#define SWDB_CASE(r, w) \
  if (R == r && W == w) return launch_rw<r, w>(grid, lds, a, s);
  SWDB_CASE(2, 1) SWDB_CASE(4, 1) SWDB_CASE(8, 1)
  SWDB_CASE(2, 2) SWDB_CASE(4, 2) SWDB_CASE(8, 2)
  SWDB_CASE(2, 4) SWDB_CASE(4, 4) SWDB_CASE(8, 4)
  SWDB_CASE(2, 8) SWDB_CASE(4, 8) SWDB_CASE(8, 8)
  SWDB_CASE(2, 16) SWDB_CASE(4, 16) SWDB_CASE(8, 16)
#undef SWDB_CASE
  return hipErrorInvalidValue;
}

}  // namespace swdb
