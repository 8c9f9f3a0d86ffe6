// The traceback walk over codes in host memory (see trace_walk.h).
#include "trace_walk.h"

#include <stddef.h>

namespace swdb {

bool walk_alignment(const uint8_t* dir, int64_t ld, int32_t q_end, int32_t db_end,
                    int32_t* q_begin, int32_t* db_begin, std::vector<uint32_t>* runs) {
  std::vector<uint8_t> rev;
  auto code = [&](int32_t row, int32_t col) { return (uint32_t)dir[(int64_t)col * ld + row]; };
  auto diagonal = [&](int32_t row, int32_t col) { return (code(row, col) & 3) == 1 ? 1 : 0; };
  auto emit = [&](uint32_t op, uint32_t) { rev.push_back((uint8_t)op); };
  if (!walk_path(q_end + 1, db_end + 1, code, diagonal, emit, q_begin, db_begin)) return false;
  for (size_t x = rev.size(); x-- > 0;) {
    const uint32_t op = rev[x];
    if (!runs->empty() && (runs->back() & 3u) == op) runs->back() += 4u;
    else runs->push_back(4u | op);
  }
  return true;
}

}  // namespace swdb
