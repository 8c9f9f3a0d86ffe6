// Batched inter-task Smith-Waterman/Gotoh kernel: many queries against the
// resident database in one persistent launch (paper section 2.2, database
// search; section 4.1 runs 20 queries against one database).
//
// Queries are sorted by length and paired; the two 16-bit halves of every
// register hold the two queries of a pair, scored against the same database
// sequence, so each lane owns one sequence and a wave 64.  The profile of a
// pair stores, for query row i and residue code c, one dword with both halves'
// scores, rows in pairs and code-major within a pair: one 64-bit LDS read per
// row pair returns both halves' scores for two rows with no packing op (all
// lanes read the same 208-byte row pair).  The two cell forms, the R-row
// strips, the stream of strips over the W waves and the boundary rows are those
// of the single-query inter-task kernel (k_inter.hip).
//
// Work is a list of (pair, half bin) entries, costliest first; a half bin is
// the 64 even or odd slots of a 128-sequence bin of the interleaved store.
// Workgroups take entries from a device counter until the list is exhausted,
// and their waves take the entries' strips one after the other without a seam.
// The strips of the entries in flight keep their boundary rows in the
// workgroup's own buffer, given out round and round in entry order: as large as
// the longest bin's, it holds several of the usual ones at once.
#include "internal.h"
#include "packed16.h"
#include "stream.h"

namespace swdb {
namespace {

template <int R, int W, bool kDrift>
__global__ __launch_bounds__(64 * W) void k_batch(BatchArgs a) {
  constexpr int kSlot = R * kBatchRowDwords;
  constexpr int kStage = (kSlot + 63) / 64;
  __shared__ __attribute__((aligned(16))) uint32_t lprof[W][kStage * 64];
  __shared__ uint32_t lprog[W];         // each wave's progress
  __shared__ int2 lpos[W];              // its item: {ordinal, strip}
  __shared__ int litem[kRing];          // ordinal n's entry of the work list at n % kRing
  __shared__ int lchunk[kRing];         // and the first chunk of its boundary rows,
  __shared__ int lvirt[kRing];          // the same before the buffer's end wrapped it
  __shared__ int lfin[kRing];           // its finished strips
  __shared__ int lfree[kRing];          // the ordinal that may take this place next
  __shared__ int lend;                  // the list is empty: items from here on hold nothing
  __shared__ int lold, lhead;           // oldest unfinished ordinal, end of the boundary rows given out
  __shared__ uint32_t lbest[kRing][2][64];   // maxima, the first and the second query's apart

  const uint32_t lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pred = w > 0 ? w - 1 : W - 1;
  char* __restrict__ rows = reinterpret_cast<char*>(a.rb + (size_t)blockIdx.x * a.rb_stride);
  const int cap = (int)(a.rb_stride / 128);   // chunks the workgroup's boundary rows hold
  const uint32_t go = a.go2, ge = a.ge2;
  const DriftArgs dr = a.drift;
  uint32_t cv = dr.c2;      // in a vector register: a 32-bit subtraction with a
  asm("" : "+v"(cv));       // scalar operand runs at the packed ops' rate only

  if (threadIdx.x < W) lprog[threadIdx.x] = ~0u;       // before its first item's start, 0
  if (threadIdx.x < kRing) {
    lfin[threadIdx.x] = 0;
    lfree[threadIdx.x] = (int)threadIdx.x;
  }
  if (threadIdx.x == 0) lend = lold = lhead = 0;
  for (int x = w; x < kRing; x += W) lbest[x][0][lane] = lbest[x][1][lane] = 0;
  __syncthreads();

  uint32_t known = ~0u;          // the predecessor's progress as last read
  auto wait_pred = [&](uint32_t need) { wait_progress(&lprog[pred], known, need); };

  for (uint32_t k = 0;; ++k) {
    // Item g = k * W + w follows item g - 1: the next strip of its matrix (pair
    // of queries, half bin), or the first of the next entry of the work list.
    // Items start in that order (so that entries are taken in order and every
    // wave ends at its first item past the list's end) and wait for smaller
    // ones only, so every wait ends.
    const uint32_t here = k << kProgBits;
    const uint32_t there = (w > 0 ? k : k - 1) << kProgBits;   // item g - 1 in its wave's count
    int n = 0, s = 0;
    if (k > 0 || w > 0) {
      wait_pred(there);
      if (!peek(&lend)) {
        n = peek(&lpos[pred].x);
        s = peek(&lpos[pred].y) + 1;
        const int2 iv = a.items[peek(&litem[n & (kRing - 1)])];
        if (s >= a.pairs[iv.x].n_strips) {
          s = 0;
          ++n;
        }
      }
    }
    const int slot = n & (kRing - 1);
    int it = -1;
    if (!peek(&lend)) {
      if (s > 0) {
        wait_pred(there + 1);
        it = peek(&litem[slot]);
      } else {
        while (peek(&lfree[slot]) != n) poll_pause();
        if (lane == 0) it = atomicAdd(a.counter, 1);
        it = __builtin_amdgcn_readfirstlane(it);
        if (it >= a.n_items) {
          it = -1;
          publish(&lend, 1);
        } else {
          // boundary rows: the next chunks of the workgroup's buffer, round
          // and round, once no unfinished matrix holds them
          const int C = (int)(a.bins[a.items[it].y >> 1].len >> 2);
          int v = peek(&lhead);
          if (v % cap + C > cap) v += cap - v % cap;
          int old = peek(&lold);
          for (;;) {
            while (old < n && peek(&lfree[old & (kRing - 1)]) == old + kRing) ++old;
            if (old == n) {        // nothing is held: the count starts again
              v = 0;
              break;
            }
            if (v < (1 << 30) && v + C - cap <= peek(&lvirt[old & (kRing - 1)])) break;
            poll_pause();
          }
          if (lane == 0) {
            lold = old;
            lhead = v + C;
            lvirt[slot] = v;
            lchunk[slot] = v % cap;
            litem[slot] = it;
          }
        }
      }
    }
    it = __builtin_amdgcn_readfirstlane(it);
    if (it < 0) {
      publish(&lprog[w], here + (1u << kProgBits) - 1);
      break;
    }
    if (lane == 0) lpos[w] = make_int2(n, s);
    publish(&lprog[w], here);

    const int2 iv = a.items[it];
    const PairDesc pd = a.pairs[iv.x];
    const BinDesc bin = a.bins[iv.y >> 1];
    const int half = iv.y & 1;
    const int C = (int)(bin.len >> 2);
    const int S = pd.n_strips;
    // lane's residues: dword res_off + c*128 + 2*lane + half
    const char* __restrict__ rbin = reinterpret_cast<const char*>(a.res + bin.res_off + half);
    char* __restrict__ rbb = rows + (size_t)peek(&lchunk[slot]) * 2048;

    uint32_t rr_n;
    uint4 b0_n, b1_n;
    // the first strip reads the boundary rows too and drops what it reads
    auto fetch = [&](int c) {
      rr_n = *reinterpret_cast<const uint32_t*>(rbin + (size_t)c * 512 + lane * 8u);
      const uint4* p = reinterpret_cast<const uint4*>(rbb + (size_t)c * 2048 + lane * 16u);
      b0_n = p[0];
      b1_n = p[64];
    };
    fetch(0);
    {
      const uint32_t* src = a.prof + pd.prof_off + (size_t)s * kSlot;
#pragma unroll
      for (int x = 0; x < kStage; ++x) lprof[w][x * 64 + lane] = src[x * 64 + lane];
    }

    uint32_t H[R], E[R], A[R];
    uint32_t best = 0, hdiag = 0;
    const int in_group = kDrift ? s % dr.group : 0;
    uint32_t zc = twice(kDriftBase) + dr.ge2 * (uint32_t)(in_group * R);
    const uint32_t delta2 = s == 0 ? 0xffffffffu : in_group == 0 ? dr.group2 : 0u;
    bool guard = false;
    if constexpr (kDrift) {
      // scores of this matrix that could leave the range (drift_plan)
      const int gev = (int)(dr.ge2 & 0xffffu), cols = 4 * C;
      const int score = max(min(S * R, cols) * a.max_s, (int)(dr.lim2 & 0xffffu));
      guard = dr.guard && score > kDriftTop - (int)kDriftBase - 256 -
                                      gev * (cols + R * min(dr.group, S) + R + 8);
      drift_start<R>(H, E, A, hdiag, zc, dr.ge2);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) { H[r] = 0; E[r] = 0; }
    }
    const bool adjust = delta2 != 0 || guard;
    const uint32_t* slotp = &lprof[w][0];
    // nothing may be pending when the chunk loop starts (k_inter.hip)
    __builtin_amdgcn_s_waitcnt(0);   // vmcnt(0) expcnt(0) lgkmcnt(0)
    for (int c = 0; c < C; ++c) {
      const uint32_t rr = rr_n;
      uint32_t up_h[4] = {b0_n.x, b0_n.z, b1_n.x, b1_n.z};
      uint32_t up_f[4] = {b0_n.y, b0_n.w, b1_n.y, b1_n.w};
      if constexpr (kDrift) {
        if (adjust) drift_adjust(up_h, up_f, delta2, zc - dr.ge2, dr.ge2, dr.lim2);
      } else if (s == 0) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) up_h[jj] = up_f[jj] = 0;
      }
      const int c_n = min(c + 1, C - 1);
      if (s > 0) wait_pred(there + (uint32_t)c_n + 1);
      fetch(c_n);
      __builtin_amdgcn_sched_barrier(0);   // keep the loads ahead of the compute
      // the strip's bottom row, (H, F) per column, stored two columns at a time,
      // a kilobyte in one piece (8 bytes a column and lane, 32 apart, took four
      // times the cache's write requests and bound the 12-row strips)
      uint4* pbd = reinterpret_cast<uint4*>(rbb + (size_t)c * 2048 + lane * 16u);
      uint32_t h_even = 0, f_even = 0;
      auto emit = [&](int jj, uint32_t h, uint32_t f) {
        if (jj & 1) {
          pbd[jj / 2 * 64] = make_uint4(h_even, f_even, h, f);
        } else {
          h_even = h;
          f_even = f;
        }
      };
      // residue bytes hold 8 x code, the byte offset of the code's dword pair in
      // a row pair: one 64-bit LDS read gives two rows
      if constexpr (kDrift) {
        drift_chunk<R, false, true>(H, E, A, hdiag, up_h, up_f, best, cv, zc, dr.ge2,
                              [&](int jj, int k2, uint2& pa, uint2&) {
          pa = reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(slotp) +
                                              ((rr >> (8 * jj)) & 0xffu))[k2 * kBatchRowDwords];
        }, emit);
        zc += 4 * dr.ge2;
        if (guard) drift_guard<R>(H, E, A, hdiag, best, dr.over2, zc, dr.ge2);
      } else {
        // (reading a column ahead measured 2 % slower here: one table, half
        // the reads to hide)
        sweep_chunk<R>(H, E, hdiag, up_h, up_f, best, go, ge,
                       [&](int jj, uint32_t (&p)[R]) {
          const uint2* pc = reinterpret_cast<const uint2*>(
              reinterpret_cast<const char*>(slotp) + ((rr >> (8 * jj)) & 0xffu));
#pragma unroll
          for (int k2 = 0; k2 < R / 2; ++k2) {
            const uint2 v = pc[k2 * kBatchRowDwords];
            p[2 * k2] = v.x;
            p[2 * k2 + 1] = v.y;
          }
        }, emit);
      }
      // the next chunk's inputs are first needed here (k_inter.hip)
      asm volatile("" : "+v"(rr_n), "+v"(b0_n.x), "+v"(b0_n.y), "+v"(b0_n.z), "+v"(b0_n.w),
                   "+v"(b1_n.x), "+v"(b1_n.y), "+v"(b1_n.z), "+v"(b1_n.w));
      publish(&lprog[w], here + (uint32_t)c + 1);
    }
    if constexpr (kDrift) drift_finish<R>(A, best, zc - dr.ge2, dr.ge2);

    // the strip's maxima join the matrix's; the wave that brings the last strip
    // writes the scores and gives the place in the ring to the next
    uint32_t ln = threadIdx.x & 63;
    asm volatile("" : "+v"(ln));      // its addresses are made here, not kept over the chunks
    atomicMax(&lbest[slot][0][ln], best & 0xffffu);
    atomicMax(&lbest[slot][1][ln], best >> 16);
    int fin = 0;
    if (ln == 0)
      fin = __hip_atomic_fetch_add(&lfin[slot], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__builtin_amdgcn_readfirstlane(fin) == S - 1) {
      const int sid = a.slot_seq[bin.slot0 + 2 * ln + half];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const uint32_t top = lbest[slot][hh][ln];
        lbest[slot][hh][ln] = 0;
        const int qi = hh ? pd.qb : pd.qa;
        if (qi < 0 || sid < 0) continue;
        const int score =
            kDrift ? drift_score(top, 0, a.sat_limit) : half_score(top, 0, a.sat_limit);
        if (score < 0) {
          const int idx = atomicAdd(a.flag_count, 1);
          a.flag_list[idx] = make_int2(sid, qi);
        } else {
          a.out[(size_t)qi * a.n_seqs + sid] = score;
        }
      }
      if (ln == 0) {
        lfin[slot] = 0;
        publish(&lfree[slot], n + kRing);
      }
    }
  }
}

template <int R, int W>
hipError_t launch_rw(int grid, const BatchArgs& a, hipStream_t s) {
  if (a.drift.group > 0)
    hipLaunchKernelGGL((k_batch<R, W, true>), dim3(grid), dim3(64 * W), 0, s, a);
  else
    hipLaunchKernelGGL((k_batch<R, W, false>), dim3(grid), dim3(64 * W), 0, s, a);
  return hipGetLastError();
}

template <int R, int W>
int occupancy() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &n, reinterpret_cast<const void*>(&k_batch<R, W, true>), 64 * W, 0) != hipSuccess) {
    (void)hipGetLastError();
    return 1;
  }
  return n > 0 ? n : 1;
}

}  // namespace

hipError_t launch_batch(int R, int W, int grid, const BatchArgs& a, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
#define SWDB_CASE(r, w) \
  if (R == r && W == w) return launch_rw<r, w>(grid, a, s);
  SWDB_CASE(16, 4) SWDB_CASE(16, 8) SWDB_CASE(16, 12) SWDB_CASE(32, 4) SWDB_CASE(32, 8)
  SWDB_CASE(12, 12) SWDB_CASE(14, 12) SWDB_CASE(18, 12) SWDB_CASE(20, 12) SWDB_CASE(12, 16) \
  SWDB_CASE(14, 16) SWDB_CASE(16, 16) SWDB_CASE(24, 12)
#undef SWDB_CASE
  return hipErrorInvalidValue;
}

int batch_workgroups_per_cu(int R, int W) {
#define SWDB_CASE(r, w) \
  if (R == r && W == w) return occupancy<r, w>();
  SWDB_CASE(16, 4) SWDB_CASE(16, 8) SWDB_CASE(16, 12) SWDB_CASE(32, 4) SWDB_CASE(32, 8)
  SWDB_CASE(12, 12) SWDB_CASE(14, 12) SWDB_CASE(18, 12) SWDB_CASE(20, 12) SWDB_CASE(12, 16) \
  SWDB_CASE(14, 16) SWDB_CASE(16, 16) SWDB_CASE(24, 12)
#undef SWDB_CASE
  return 1;
}

}  // namespace swdb
