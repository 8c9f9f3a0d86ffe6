// Traceback walk: from each alignment's end back through the codes that the
// int32 wavefront left in device memory (k_intra.hip), one wave per sequence.
//
// A walk is one chain of dependent reads, so its cells come in tiles of 64
// columns and 64 rows through LDS (4 KB, four 16-byte reads a lane), the cell
// at the walk's place near the tile's last row and column; the state is scalar.
// Along a diagonal, which most steps follow, each lane looks at one cell and the
// walk goes to the first that leaves it (a step at a time, a read, a decision and
// a branch or two each, took 0.086 ms in the place of 0.007).  What leaves the device are the runs of
// operations, a few words an alignment, in the place of the codes of every column
// up to the end (half a kilobyte a column and more, through pageable memory,
// walked by host threads: of a traceback of ten alignments, 310 residues against
// up to 1,572, 0.30 ms of 0.73).
#include "internal.h"
#include "trace_walk.h"

namespace swdb {
namespace {

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// kRows: rows a code word holds, as many bytes
template <int kRows>
__global__ __launch_bounds__(64) void k_trace_walk(TraceWalkArgs a) {
  __shared__ __align__(16) uint8_t tile[64 * 64];    // [column][row]
  const int lane = threadIdx.x, it = blockIdx.x;
  const int4 end = a.ends[it];
  if (end.y <= 0) {
    if (lane == 0) a.heads[it] = make_int4(0, -1, -1, 0);
    return;
  }
  const uint8_t* dir = a.dir + a.dir_off[it] + kTracePad * a.dir_ld;
  uint32_t* rev = a.rev + a.rev_off[it];

  int r0 = 0, c0 = 0, c1 = -1;                       // the tile's rows from, columns from, to
  auto load = [&](int row, int col) {
    if (col < c0 || col > c1 || row < r0 || row > r0 + 63) {
      c1 = col;
      c0 = max(0, col - 63);
      r0 = max(0, (row & ~15) - 48);
      __syncthreads();
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int e = 64 * x + lane, c = e >> 2, part = e & 3;
        if (c0 + c <= c1)
          *reinterpret_cast<uint4*>(tile + 64 * c + 16 * part) = *reinterpret_cast<const uint4*>(
              dir + (size_t)(c0 + c) * a.dir_ld + (size_t)(r0 + 16 * part));
      }
      __syncthreads();
    }
  };
  // the code of a cell in the tile
  auto cell = [&](int row, int col) -> uint32_t {
    const uint8_t* at = tile + 64 * (col - c0) + ((row - r0) & ~(kRows - 1));
    const uint32_t word = kRows == 2 ? *reinterpret_cast<const uint16_t*>(at)
                                     : *reinterpret_cast<const uint32_t*>(at);
    const uint32_t v = word >> (5 * (kRows - 1 - (row & (kRows - 1))));
    // signs {d - H, F - H, 0 - H, (H - go) - (E - ge), (H - go) - (F - ge)}
    const uint32_t src = !(v & 4) ? 0u : !(v & 16) ? 1u : !(v & 8) ? 3u : 2u;
    return src | (v & 2 ? 0u : 4u) | (v & 1 ? 0u : 8u);
  };
  auto code = [&](int row, int col) -> uint32_t {
    load(row, col);
    return (uint32_t)uniform((int)cell(row, col));
  };
  auto diagonal = [&](int row, int col) -> int {
    load(row, col);
    const int r = row - lane, c = col - lane;
    const bool in = r >= r0 && c >= c0;
    const uint64_t leaves = __ballot(!in || (cell(in ? r : row, in ? c : col) & 3) != 1);
    return leaves ? uniform(__builtin_ctzll(leaves)) : 64;
  };
  uint32_t run = 0;
  int n = 0;
  auto emit = [&](uint32_t op, uint32_t times) {
    if (run != 0 && (run & 3u) == op) {
      run += 4u * times;
    } else {
      if (run != 0) {
        if (lane == 0) rev[n] = run;
        ++n;
      }
      run = 4u * times | op;
    }
  };
  int32_t qb = -1, db = -1;
  const bool ok =
      walk_path(uniform(end.z) + 1, uniform(end.w) + 1, code, diagonal, emit, &qb, &db);
  if (run != 0) {
    if (lane == 0) rev[n] = run;
    ++n;
  }
  if (!ok) {
    if (lane == 0) a.heads[it] = make_int4(-1, -1, -1, 0);
    return;
  }
  int at = 0;
  if (lane == 0) {
    at = atomicAdd(a.total, n);
    a.heads[it] = make_int4(n, qb, db, at);
  }
  at = uniform(at);
  __syncthreads();
  for (int x = lane; x < n; x += 64) a.runs[at + x] = rev[n - 1 - x];
}

}  // namespace

hipError_t launch_trace_walk(int R, int count, const TraceWalkArgs& a, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (R == 2) hipLaunchKernelGGL(k_trace_walk<2>, dim3(count), dim3(64), 0, s, a);
  else hipLaunchKernelGGL(k_trace_walk<4>, dim3(count), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace swdb
