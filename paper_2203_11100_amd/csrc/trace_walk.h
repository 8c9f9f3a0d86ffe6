// The traceback's walk back through the per-cell codes of the int32 intra-task
// kernel's traceback variant (k_intra.hip): the steps, shared by the device's
// walk (k_trace.hip) and the host's.
#pragma once
#include <stdint.h>

#include <vector>

#ifdef __HIP__
#define SWDB_WALK __host__ __device__ __forceinline__
#else
#define SWDB_WALK inline
#endif

namespace swdb {

// Three states, H, F and E, stepping from cell (i, j) (1-based) toward the
// alignment's first matched pair.  code(row, column) gives a 0-based cell's code:
// bits 0-1 where H came from - 0 it is 0, 1 the diagonal, 2 E, 3 F; bit 2 E of the
// next column opens a gap; bit 3 F of the next row opens a gap.  diagonal(row,
// column) says for how many cells from there on, up and left, H is known to come
// from the diagonal (0: not for this one).  emit(op, n) takes the operations, last
// first: 0 = M, 1 = I (query residue against a gap), 2 = D (database residue
// against a gap).  Sets the 0-based first positions.  Returns false on codes that
// do not form a path.
template <class Code, class Diagonal, class Emit>
SWDB_WALK bool walk_path(int32_t i, int32_t j, Code&& code, Diagonal&& diagonal, Emit&& emit,
                         int32_t* q_begin, int32_t* db_begin) {
  int state = 0;                                              // 0 H, 1 F, 2 E
  const int32_t bound = 2 * (i + j) + 4;
  for (int32_t step = 0; step <= bound; ++step) {
    if (state != 0 && (i < 1 || j < 1)) return false;
    if (state == 0) {
      const int n = i < 1 || j < 1 ? 0 : diagonal(i - 1, j - 1);
      if (n > 0) {
        emit(0u, (uint32_t)n);
        i -= n;
        j -= n;
        continue;
      }
      // H is 0 on the borders (row 0, column 0): the alignment starts there too
      const int src = i < 1 || j < 1 ? 0 : code(i - 1, j - 1) & 3;
      if (src == 0) {
        *q_begin = i;
        *db_begin = j;
        return true;
      }
      state = src == 3 ? 1 : 2;
    } else if (state == 1) {
      emit(1u, 1u);
      if (i < 2) return false;
      state = (code(i - 2, j - 1) >> 3) & 1 ? 0 : 1;
      --i;
    } else {
      emit(2u, 1u);
      if (j < 2) return false;
      state = (code(i - 1, j - 2) >> 2) & 1 ? 0 : 2;
      --j;
    }
  }
  return false;
}

// Walks an optimal local alignment back from its end (0-based q_end, db_end)
// through one sequence's codes ([column][row] bytes, ld bytes per column) and
// appends it, first operation first, as runs (length << 2 | op).
bool walk_alignment(const uint8_t* dir, int64_t ld, int32_t q_end, int32_t db_end,
                    int32_t* q_begin, int32_t* db_begin, std::vector<uint32_t>* runs);

}  // namespace swdb
