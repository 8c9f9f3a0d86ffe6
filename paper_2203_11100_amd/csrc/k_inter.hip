// Inter-task Smith-Waterman/Gotoh kernel: every lane scores two database
// sequences against the query (paper section 2.2: inter-task parallelism,
// one independent alignment matrix per processing element, no communication
// between elements), in packed 16-bit arithmetic.
//
// Cells follow Gotoh's recurrence over query rows i and database columns j:
//   E(i,j) = max(E(i,j-1) - e, H(i,j-1) - o)
//   F(i,j) = max(F(i-1,j) - e, H(i-1,j) - o)
//   H(i,j) = max(0, H(i-1,j-1) + S(a_i,b_j), E(i,j), F(i,j)),  score = max H.
// Two forms of the cell compute it in packed 16-bit arithmetic (packed16.h):
// the drift form, in integers, 5 packed ops and half of one for the running
// maximum, and the binary16 form, 7 and a half, for gap penalties whose drift
// leaves the 16-bit range.  Both are exact below the rescoring limit; sequences
// whose maximum reaches it are handed to the exact 32-bit kernel.
//
// Work decomposition.  A bin is 128 length-sorted sequences (lane l holds the
// sequences of slots 2l and 2l+1 in the low and high 16-bit halves).  The query
// is cut into strips of R rows; the H and E state of a strip's R rows lives in
// registers while the strip sweeps every column of the bin.  The bottom row of
// a strip (H and the F flowing into the next row) is written to a per-bin
// boundary buffer and read back by the next strip, which overwrites it in
// place: every strip reads a chunk of 4 columns before writing it.
//
// The kernel is persistent.  A workgroup takes bins, longest first, from a
// queue and its W waves take the strips of those bins round robin, bin after
// bin without a seam: a wave that is done with its last strip of one bin starts
// on the next while other waves still work on the one before.  So no wave
// idles in the last round of a query that is no multiple of W strips, no
// pipeline fills and drains with every bin, and the last bins of the search are
// short ones.  Splitting a bin's strips over W waves divides its latency by W,
// which keeps the longest bins from trailing the rest of the grid.
// Waves are kept in order by progress words in LDS alone, chunk by chunk, each
// waiting for its predecessor only; a workgroup barrier every chunk had the
// four waves of a SIMD start and end every chunk together, the last of them
// alone on it.  Bound by the VALU: on the plain database (71 M residues, m =
// 5,478, 14 x 16) the kernel takes 38.8 ms, 85 % of the VALU's issue slots at
// the clock the card holds (2.2 GHz); binary16 cells with barriers and one bin
// a workgroup took 52.6 ms, drift cells alone 45.6, without the barriers 43
// (36.7 with the long pairs in drift cells beside it).
//
// The query profile rows of the current strip are staged in LDS as two
// tables (internal.h, prof_strip_dwords), one dword a row and code, for 26 codes
// (24 residues, pad, spare), rows in pairs and code-major within a pair: the low
// table's dword holds the score for the low half, the high table's the one for
// the high half.  Per row pair a lane reads one 64-bit entry for its low
// sequence's residue from the low table and one for its high sequence's from
// the high table, and a single three-input add (drift) or fused multiply-add
// (binary16) per cell forms H_diag + S for both sequences, with no byte permute.
// Each column's entries are read while the previous column is computed
// (sweep_chunk_ahead), so the LDS latency hides behind a column of arithmetic.
// The next strip's rows are copied in during the current strip's last chunks,
// one or two dwords per lane per chunk, so the copy holds few registers.
#include "internal.h"
#include "packed16.h"
#include "stream.h"

namespace swdb {
namespace {

// The cell form: binary16 or drift local scores, global or semi-global scores
// (drift form, without the floor and the maximum).
//
// Global and semi-global: with H(i, 0) = -w(i), w(k) = go + (k - 1) ge, and the
// drift ge * (row + column) over 0-based rows and columns, the left border is
// the constant base - go - ge (a border gap costs its opening only) and so is
// the global mode's top border; the semi-global top border, H = 0, is base + ge *
// (column - 1).  E and F start c below the borders.  The query's rows are
// shifted down by `pad`, so that its last row is the last strip's last and its
// H comes out of the strip's sweep; the rows above it repeat the top border:
// in semi-global mode they score 0 against everything (0 along the diagonals),
// in global mode they score -2 ge and E holds the border.  The score is the last
// row's H at the sequence's last column (global) or its maximum over the
// sequence's columns, both taken by the last strip.
template <int R, int W, int kForm>
__global__ __launch_bounds__(64 * W) void k_inter(InterArgs a) {
  constexpr bool kDrift = kForm == kCellDrift;
  constexpr bool kMode = kForm == kCellGlobal || kForm == kCellSemi;
  constexpr int kSlot = prof_strip_dwords(R);
  constexpr int kHighBytes = R * kProfRowDwords * 4;   // the high table's offset
  constexpr int kStage = (kSlot + 63) / 64;            // dwords per lane per strip
  constexpr int kPer = (kStage + 15) / 16;             // staged per chunk
  constexpr int kStageChunks = (kStage + kPer - 1) / kPer;
  static_assert(kStageChunks <= SW_MIN_BIN_LEN / 4, "the staging needs kStageChunks chunks");
  __shared__ __attribute__((aligned(16))) uint32_t lprof[W][2][kStage * 64];
  __shared__ uint32_t lprog[W];         // each wave's progress
  __shared__ int lbin[kRing];           // ordinal n's bin at n % kRing
  __shared__ int lend;                  // the queue is empty: items from here on hold nothing
  __shared__ int lfin[kRing];           // its finished strips
  __shared__ int lfree[kRing];          // the ordinal that may take this place next
  __shared__ uint32_t lbest[kRing][2][64];   // its maxima, low and high halves apart

  const uint32_t lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int S = a.n_strips;
  const int pred = w > 0 ? w - 1 : W - 1;

  // the workgroup's items are the strips of its bins in order; wave w takes
  // items w, w + W, ...: strip s of the workgroup's n-th bin
  int n = w / S, s = w % S;
  const int dn = W / S, ds = W % S;
  {
    const uint32_t* src = a.prof + (size_t)s * kSlot;
#pragma unroll
    for (int x = 0; x < kStage; ++x) lprof[w][0][x * 64 + lane] = src[x * 64 + lane];
  }
  if (threadIdx.x < W) lprog[threadIdx.x] = ~0u;       // before its first item's start, 0
  if (threadIdx.x < kRing) {
    lfin[threadIdx.x] = 0;
    lfree[threadIdx.x] = (int)threadIdx.x;
  }
  if (threadIdx.x == 0) lend = 0;
  if (w == 0) {
#pragma unroll
    for (int x = 0; x < kRing; ++x) lbest[x][0][lane] = lbest[x][1][lane] = 0;
  }
  __syncthreads();

  const uint32_t go = a.go2, ge = a.ge2;
  const DriftArgs dr = a.drift;
  uint32_t cv = dr.c2;      // in a vector register: a 32-bit subtraction with a
  asm("" : "+v"(cv));       // scalar operand runs at the packed ops' rate only

  uint32_t known = ~0u;          // the predecessor's progress as last read
  auto wait_pred = [&](uint32_t need) { wait_progress(&lprog[pred], known, need); };

  // one 64-bit LDS read per row pair and sequence gives both rows' dwords,
  // from the low table for the low half's residue and from the high table for
  // the high half's; the residue bytes hold 8 x code, the byte offset of the
  // code's dword pair in a row pair
  auto read_pair = [&](const uint32_t* sl, uint2 res, int jj, int k2, uint2& pa, uint2& pb) {
    const uint2* plo = reinterpret_cast<const uint2*>(
        reinterpret_cast<const char*>(sl) + ((res.x >> (8 * jj)) & 0xffu));
    const uint2* phi = reinterpret_cast<const uint2*>(
        reinterpret_cast<const char*>(sl) + kHighBytes + ((res.y >> (8 * jj)) & 0xffu));
    pa = plo[k2 * kProfRowDwords];
    pb = phi[k2 * kProfRowDwords];
  };

  int buf = 0;                   // the profile buffer that holds this strip's rows
  for (uint32_t k = 0;; ++k) {
    // Item g = k * W + w needs item g - 1: a strip reads the rows the strip
    // above it leaves (chunk by chunk, below), and the first strip of a bin
    // starts after the last of the bin before has started, so that bins are
    // taken from the queue in order and every wave ends at its first item past
    // the queue's end.  Waits end: an item waits for smaller items only
    // (the bin kRing before consists of such), and the wave of the smallest
    // unfinished one has nothing else to do.
    const uint32_t here = k << kProgBits;
    const uint32_t there = (w > 0 ? k : k - 1) << kProgBits;   // item g - 1 in its wave's count
    const int slot = n & (kRing - 1);
    int b = -1;
    if (s == 0) {
      if (k > 0 || w > 0) wait_pred(there);
      if (!peek(&lend)) {
        while (peek(&lfree[slot]) != n) poll_pause();
        if (lane == 0) b = atomicAdd(a.counter, 1);
        b = __builtin_amdgcn_readfirstlane(b);
        if (b >= a.n_bins) {
          b = -1;
          publish(&lend, 1);
        }
        if (lane == 0) lbin[slot] = b;
      }
    } else {
      wait_pred(there + 1);
      if (!peek(&lend)) b = peek(&lbin[slot]);
    }
    if (b < 0) {
      publish(&lprog[w], here + (1u << kProgBits) - 1);
      break;
    }
    publish(&lprog[w], here);

    const BinDesc bin = a.bins[a.bin_begin + b];
    const int C = (int)(bin.len >> 2);
    // uniform bases, advanced chunk by chunk, and the lane's constant offsets
    const char* __restrict__ rbin = reinterpret_cast<const char*>(a.res2 + (bin.res_off >> 1));
    char* __restrict__ rbb = reinterpret_cast<char*>(a.rb + (bin.rb_off - a.rb_base));

    // inputs of the next chunk, fetched one chunk ahead.  The first strip
    // reads the boundary buffer too and drops what it reads, so every chunk
    // issues the same memory operations and the compiler can count them exactly.
    uint2 rr_n;
    uint4 b0_n, b1_n;
    auto fetch = [&](int c) {
      rr_n = *reinterpret_cast<const uint2*>(rbin + (size_t)c * 512 + lane * 8u);
      const uint4* p = reinterpret_cast<const uint4*>(rbb + (size_t)c * 2048 + lane * 16u);
      b0_n = p[0];
      b1_n = p[64];
    };
    fetch(0);

    uint32_t H[R], E[R], A[R];
    uint32_t best = 0, hdiag = 0;
    // Z of row 0 and the chunk's first column, and the row above's correction
    const int in_group = kDrift ? s % dr.group : 0;
    uint32_t zc = twice(kDriftBase) + dr.ge2 * (uint32_t)(in_group * R);
    const uint32_t delta2 = s == 0 ? 0xffffffffu : in_group == 0 ? dr.group2 : 0u;
    const bool adjust = delta2 != 0 || dr.guard;
    const ModeShape& md = a.mode;
    const uint32_t base2 = twice((uint32_t)md.base);
    // the row above the query's first in global mode: H~ there, F~ below it c less
    const uint32_t top2 = twice((uint32_t)(md.base - md.go + md.ge * (md.pad - 1)));
    uint32_t n2 = 0, score = 0;      // modes, last strip: both sequences' lengths, their scores
    int sid_lo = -1, sid_hi = -1;
    if constexpr (kMode) {
      const uint32_t left2 = twice((uint32_t)(md.base - md.go - md.ge + md.ge * md.pad));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        H[r] = left2;
        E[r] = left2 - dr.c2;
      }
      hdiag = left2;
      if (s == 0) {
        const uint32_t corner2 = base2 + dr.ge2 * (uint32_t)md.pad - 2 * dr.ge2;   // H(0, 0) = 0
        hdiag = kForm == kCellGlobal && md.pad > 0 ? top2 : base2 - 2 * dr.ge2;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (r < md.pad) {
            if (kForm == kCellGlobal) {
              H[r] = r == md.pad - 1 ? corner2 : top2;
              E[r] = top2;
            } else {
              H[r] = base2 + dr.ge2 * (uint32_t)r - dr.ge2;
              E[r] = H[r] - dr.c2;
            }
          }
        }
      }
      if (s == S - 1) {
        sid_lo = a.slot_seq[bin.slot0 + 2 * lane];
        sid_hi = a.slot_seq[bin.slot0 + 2 * lane + 1];
        const int n_lo = sid_lo >= 0 ? (int)(md.offs[sid_lo + 1] - md.offs[sid_lo]) : 0;
        const int n_hi = sid_hi >= 0 ? (int)(md.offs[sid_hi + 1] - md.offs[sid_hi]) : 0;
        n2 = (uint32_t)n_lo | ((uint32_t)n_hi << 16);
      }
    } else if constexpr (kDrift) {
      drift_start<R>(H, E, A, hdiag, zc, dr.ge2);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) { H[r] = 0; E[r] = 0; }
    }
    const uint32_t* slotp = &lprof[w][buf][0];
    // the wave's next item: its profile rows are staged in the other buffer
    // during this item's last chunks, unless it is the same strip again
    const int s_next = s + ds >= S ? s + ds - S : s + ds;
    const bool more = s_next != s;
    // nothing may be pending when the chunk loop starts: the compiler merges
    // the loop's entry with its back edge, and scalar loads return out of
    // order, so a load pending on entry would make every chunk wait for
    // memory or for all of its first column's LDS reads at its start
    __builtin_amdgcn_s_waitcnt(0);   // vmcnt(0) expcnt(0) lgkmcnt(0)
    for (int c = 0; c < C; ++c) {
      const uint2 rr = rr_n;
      uint32_t up_h[4] = {b0_n.x, b0_n.z, b1_n.x, b1_n.z};
      uint32_t up_f[4] = {b0_n.y, b0_n.w, b1_n.y, b1_n.w};
      if constexpr (kMode) {
        if (s == 0) {
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            up_h[jj] = kForm == kCellGlobal ? top2 : base2 + dr.ge2 * (uint32_t)(4 * c + jj) - dr.ge2;
            up_f[jj] = kForm == kCellGlobal
                           ? top2 - dr.c2
                           : base2 + dr.ge2 * (uint32_t)(4 * c + jj) - twice((uint32_t)md.go);
          }
        }
      } else if constexpr (kDrift) {
        if (adjust) drift_adjust(up_h, up_f, delta2, zc - dr.ge2, dr.ge2, dr.lim2);
      } else if (s == 0) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) up_h[jj] = up_f[jj] = 0;
      }
      // the next chunk (after the last a harmless reload)
      const int c_n = min(c + 1, C - 1);
      if (s > 0) wait_pred(there + (uint32_t)c_n + 1);
      fetch(c_n);
      // next strip's profile, pieces kPer * x .. kPer * x + kPer - 1 of
      // kStage with x = c - (C - kStageChunks): the global loads now (always
      // issued, from this strip's own profile when there is nothing to
      // stage), the LDS stores after the compute
      const int x_st = c - (C - kStageChunks);
      const bool stage = more && x_st >= 0;
      const uint32_t* st_src =
          a.prof + ((size_t)(stage ? s_next : s) * kSlot + (size_t)(kPer * max(x_st, 0)) * 64);
      uint32_t st[kPer];
#pragma unroll
      for (int y = 0; y < kPer; ++y) st[y] = st_src[y * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);   // keep the loads ahead of the compute
      // the strip's bottom row, (H, F) per column, stored two columns at a time,
      // a kilobyte in one piece (8 bytes a column and lane, 32 apart, took four
      // times the cache's write requests and bound the 12-row strips)
      uint4* pbd = reinterpret_cast<uint4*>(rbb + (size_t)c * 2048 + lane * 16u);
      uint32_t h_even = 0, f_even = 0;
      uint32_t bottom[4];            // modes: the bottom row's H~
      auto prof_pair = [&](int jj, int k2, uint2& pa, uint2& pb) {
        read_pair(slotp, rr, jj, k2, pa, pb);
      };
      auto emit = [&](int jj, uint32_t h, uint32_t f) {
        if (kMode) bottom[jj] = h;
        if (jj & 1) {
          pbd[jj / 2 * 64] = make_uint4(h_even, f_even, h, f);
        } else {
          h_even = h;
          f_even = f;
        }
      };
      if constexpr (kMode) {
        drift_chunk<R, true, false>(H, E, A, hdiag, up_h, up_f, best, cv, zc, dr.ge2, prof_pair,
                                    emit);
        if (s == S - 1) {
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            // 0xffff in the halves whose sequence has this column
            const uint32_t j2 = twice((uint32_t)(4 * c + jj));
            const uint32_t in = umul2(umin2(usub2_sat(n2, j2), 0x00010001u), 0xffffffffu);
            if (kForm == kCellGlobal) score = (score & ~in) | (bottom[jj] & in);
            else score = umax2(score, (bottom[jj] - dr.ge2 * (uint32_t)(4 * c + jj)) & in);
          }
        }
      } else if constexpr (kDrift) {
        drift_chunk<R, true, true>(H, E, A, hdiag, up_h, up_f, best, cv, zc, dr.ge2, prof_pair,
                                   emit);
        zc += 4 * dr.ge2;
        if (dr.guard) drift_guard<R>(H, E, A, hdiag, best, dr.over2, zc, dr.ge2);
      } else {
        sweep_chunk_ahead<R, true>(H, E, hdiag, up_h, up_f, best, go, ge, prof_pair, emit);
      }
      // the next chunk's inputs are first needed here: without this use the
      // compiler copies them to the loop's registers right after the loads,
      // and every chunk starts by waiting for the memory
      asm volatile("" : "+v"(rr_n.x), "+v"(rr_n.y), "+v"(b0_n.x), "+v"(b0_n.y), "+v"(b0_n.z),
                   "+v"(b0_n.w), "+v"(b1_n.x), "+v"(b1_n.y), "+v"(b1_n.z), "+v"(b1_n.w));
      if (stage) {
#pragma unroll
        for (int y = 0; y < kPer; ++y)
          if (kStage % kPer == 0 || kPer * x_st + y < kStage)
            lprof[w][buf ^ 1][(kPer * x_st + y) * 64 + lane] = st[y];
      }
      publish(&lprog[w], here + (uint32_t)c + 1);
    }
    if constexpr (kDrift) drift_finish<R>(A, best, zc - dr.ge2, dr.ge2);
    if (more) buf ^= 1;

    // modes: the last strip has the scores
    if constexpr (kMode) {
      if (s == S - 1) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int sid = half ? sid_hi : sid_lo;
          if (sid < 0) continue;
          const int n_h = (int)(half ? n2 >> 16 : n2 & 0xffffu);
          const int v = (int)(half ? score >> 16 : score & 0xffffu);
          // H~ less base and the drift of the last row (and, global, of the last column)
          const int rows = md.base + md.ge * (S * R - 1);
          a.out[sid] = n_h == 0 ? -(md.go + (md.m - 1) * md.ge)
                                : v - rows - (kForm == kCellGlobal ? md.ge * (n_h - 1) : 0);
        }
      }
    }
    // the strip's maxima join the bin's; the wave that brings the last strip
    // writes the scores and gives the place in the ring to the next bin
    uint32_t ln = threadIdx.x & 63;
    asm volatile("" : "+v"(ln));      // its addresses are made here, not kept over the chunks
    if constexpr (!kMode) {
      atomicMax(&lbest[slot][0][ln], best & 0xffffu);
      atomicMax(&lbest[slot][1][ln], best >> 16);
    }
    int fin = 0;
    if (lane == 0)
      fin = __hip_atomic_fetch_add(&lfin[slot], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__builtin_amdgcn_readfirstlane(fin) == S - 1) {
      const int64_t slot0 = bin.slot0 + 2 * ln;
#pragma unroll
      for (int half = 0; half < (kMode ? 0 : 2); ++half) {
        const uint32_t top = lbest[slot][half][ln];
        lbest[slot][half][ln] = 0;
        const int sid = a.slot_seq[slot0 + half];
        if (sid < 0) continue;
        const int score =
            kDrift ? drift_score(top, 0, a.sat_limit) : half_score(top, 0, a.sat_limit);
        if (score < 0) {
          const int idx = atomicAdd(a.flag_count, 1);
          a.flag_list[idx] = make_int2(sid, 0);
        } else {
          a.out[sid] = score;
        }
      }
      if (lane == 0) {
        lfin[slot] = 0;
        publish(&lfree[slot], n + kRing);
      }
    }
    n += dn;
    s += ds;
    if (s >= S) { s -= S; ++n; }
  }
}

template <int R, int W, int kForm>
hipError_t launch_rwd(const InterArgs& a, int n_cus, hipStream_t s) {
  // one workgroup for every place on the device, at most one per bin
  static const int per_cu = [] {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, reinterpret_cast<const void*>(&k_inter<R, W, kForm>), 64 * W, 0) != hipSuccess) {
      (void)hipGetLastError();
      n = 1;
    }
    return n > 0 ? n : 1;
  }();
  const int grid = (int)std::min<int64_t>(a.n_bins, (int64_t)n_cus * per_cu);
  hipLaunchKernelGGL((k_inter<R, W, kForm>), dim3(grid), dim3(64 * W), 0, s, a);
  return hipGetLastError();
}

template <int R, int W>
hipError_t launch_rw(const InterArgs& a, int n_cus, hipStream_t s) {
  return a.drift.group > 0 ? launch_rwd<R, W, kCellDrift>(a, n_cus, s)
                           : launch_rwd<R, W, kCellHalf>(a, n_cus, s);
}

template <int R, int W>
hipError_t launch_mode_rw(const InterArgs& a, int n_cus, hipStream_t s) {
  return a.mode.mode == SW_MODE_GLOBAL ? launch_rwd<R, W, kCellGlobal>(a, n_cus, s)
                                       : launch_rwd<R, W, kCellSemi>(a, n_cus, s);
}

}  // namespace

hipError_t launch_inter(int R, int W, int n_cus, const InterArgs& a, hipStream_t s) {
  if (a.n_bins <= 0) return hipSuccess;
  if (a.mode.mode != SW_MODE_LOCAL) {
#define SWDB_CASE(r, w) \
  if (R == r && W == w) return launch_mode_rw<r, w>(a, n_cus, s);
    SWDB_CASE(12, 16) SWDB_CASE(14, 16) SWDB_CASE(16, 16)
#undef SWDB_CASE
    return hipErrorInvalidValue;
  }
#define SWDB_CASE(r, w) \
  if (R == r && W == w) return launch_rw<r, w>(a, n_cus, s);
  SWDB_CASE(16, 1) SWDB_CASE(16, 2) SWDB_CASE(16, 4) SWDB_CASE(16, 8) SWDB_CASE(16, 12)
  SWDB_CASE(32, 1) SWDB_CASE(32, 2) SWDB_CASE(32, 4) SWDB_CASE(32, 8)
  SWDB_CASE(12, 12) SWDB_CASE(14, 12) SWDB_CASE(18, 12) SWDB_CASE(20, 12)
  SWDB_CASE(12, 16) SWDB_CASE(14, 16)
#undef SWDB_CASE
  return hipErrorInvalidValue;
}

}  // namespace swdb
