// Small helper kernels: query profile construction and buffer fill.
#include "internal.h"

namespace swdb {
namespace {

__device__ __forceinline__ int profile_score(const uint8_t* __restrict__ q, int m,
                                             const Matrix& mat, int i, int c) {
  if (i >= m || c >= SW_ALPHA) return kPadScore;
  const int qc = q[i];
  return qc < SW_ALPHA ? (int)mat.v[qc * SW_ALPHA + c] : kPadScore;
}

// Builds the query profiles from the query codes and the substitution
// matrix: the inter-task layout for strips of R rows (see prof_strip_dwords),
// the intra-task layout [25][m_pad2] int8 and, when prof3 is given, the
// packed intra-task layout [25][m_pad2 / 2] of binary16 row pairs (dword
// (c, r) = S(a_2r, c) low, S(a_2r+1, c) high); codes 0..23 and the pad code.
// Entry (i, c) is S(a_i, c); rows past the query end and the pad/spare codes
// get kPadScore.  Thread 0 also clears the rescoring list's count.
// pb.add >= 0: prof3 is instead the long-pair kernel's [25][m_pad2] bytes
// S + p.add, four rows a dword, with p's bytes for the rows above and past the
// query and for the pad code.
__device__ __forceinline__ uint32_t pair_bytes(const uint8_t* __restrict__ q, int m,
                                               const Matrix& mat, int row, int c,
                                               const PairBytes& p) {
  uint32_t v = 0;
  for (int t = 0; t < 4; ++t) {
    const int i = row + t - p.top;
    const uint32_t b = i < 0           ? (uint32_t)p.top_byte
                       : c >= SW_ALPHA ? (uint32_t)p.code_byte
                       : i >= m || q[i] >= SW_ALPHA
                           ? (uint32_t)p.row_byte
                           : (uint32_t)(mat.v[q[i] * SW_ALPHA + c] + p.add);
    v |= (b & 0xffu) << (8 * t);
  }
  return v;
}

__global__ void k_profile(const uint8_t* __restrict__ q, int m, Matrix mat,
                          uint32_t* __restrict__ prof, int m_pad, int R, int drift,
                          int top, int top_score, int8_t* __restrict__ prof2, uint32_t* __restrict__ prof3,
                          PairBytes pb, int m_pad2,
                          int32_t* __restrict__ flag_count) {
  const int64_t n1 = (int64_t)(m_pad / R) * prof_strip_dwords(R);
  const int64_t n2 = (int64_t)kIntraCodes * m_pad2;
  const int64_t n3 = prof3 ? (int64_t)kIntraCodes * (m_pad2 / (pb.add >= 0 ? 4 : 2)) : 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < kFlagWords && flag_count) flag_count[idx] = 0;
  for (; idx < n1 + n2 + n3; idx += stride) {
    if (idx < n1) {
      // idx = ((strip * 2 + table) * R / 2 + pair) * kProfPairDwords + 2 * c + t
      const int rem = (int)(idx % kProfPairDwords);
      const int64_t pr = idx / kProfPairDwords;
      const int pair = (int)(pr % (R / 2));
      const int64_t st = pr / (R / 2);
      const int i = (int)(st >> 1) * R + 2 * pair + (rem & 1), c = rem >> 1;
      const int sc = i < top ? top_score : profile_score(q, m, mat, i - top, c);
      if (drift >= 0) {
        const uint32_t v = (uint32_t)(sc + 2 * drift);
        prof[idx] = (st & 1) ? v << 16 : v;
      } else {
        const uint32_t v = half_bits(sc);
        prof[idx] = (st & 1) ? kHalfOne | (v << 16) : v | (kHalfOne << 16);
      }
    } else if (idx < n1 + n2) {
      const int64_t j = idx - n1;
      const int c = (int)(j / m_pad2), i = (int)(j % m_pad2);
      prof2[j] = (int8_t)profile_score(q, m, mat, i, c);
    } else {
      const int64_t j = idx - n1 - n2;
      if (pb.add >= 0) {
        const int words = m_pad2 / 4;
        prof3[j] = pair_bytes(q, m, mat, (int)(j % words) * 4, (int)(j / words), pb);
        continue;
      }
      const int half_rows = m_pad2 / 2;
      const int c = (int)(j / half_rows), r = (int)(j % half_rows);
      const uint32_t lo = half_bits(profile_score(q, m, mat, 2 * r, c));
      const uint32_t hi = half_bits(profile_score(q, m, mat, 2 * r + 1, c));
      prof3[j] = lo | (hi << 16);
    }
  }
}

// Pair profiles and intra-task profiles of a batch.  blockIdx.y < n_pairs
// selects a pair: the dword of row i and code c of its profile (n_strips * R
// rows in the kProfRowDwords layout) holds (S(a_i, c), S(b_i, c)) as
// binary16 or, with drift >= 0, the 32-bit sum of S(a_i, c) + 2 drift and,
// shifted up 16 bits, S(b_i, c) + 2 drift; kPadScore past either query's end.  Larger
// blockIdx.y select a query's intra-task [25][m_pad2] int8 profile and, when
// prof3 is given, its packed [25][m_pad2 / 2] binary16 row pairs.
__global__ void k_batch_profiles(const uint8_t* __restrict__ queries,
                                 const int64_t* __restrict__ qoffs, Matrix mat,
                                 const PairDesc* __restrict__ pairs, int n_pairs, int R,
                                 int drift, uint32_t* __restrict__ prof,
                                 const QueryDesc* __restrict__ qdesc, int8_t* __restrict__ prof2,
                                 uint32_t* __restrict__ prof3, PairBytes pb) {
  const int y = blockIdx.y;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t start = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (y < n_pairs) {
    const PairDesc pd = pairs[y];
    const int64_t total = (int64_t)pd.n_strips * R * kBatchRowDwords;
    const uint8_t* qa = queries + qoffs[pd.qa];
    const int ma = (int)(qoffs[pd.qa + 1] - qoffs[pd.qa]);
    const uint8_t* qb = pd.qb >= 0 ? queries + qoffs[pd.qb] : nullptr;
    const int mb = pd.qb >= 0 ? (int)(qoffs[pd.qb + 1] - qoffs[pd.qb]) : 0;
    for (int64_t idx = start; idx < total; idx += stride) {
      const int rem = (int)(idx % kProfPairDwords);
      const int i = 2 * (int)(idx / kProfPairDwords) + (rem & 1), c = rem >> 1;
      const int sa = profile_score(qa, ma, mat, i, c), sb = profile_score(qb, mb, mat, i, c);
      prof[pd.prof_off + idx] =
          drift >= 0 ? (uint32_t)(sa + 2 * drift) + ((uint32_t)(sb + 2 * drift) << 16)
                     : half_bits(sa) | ((uint32_t)half_bits(sb) << 16);
    }
  } else {
    const int qi = y - n_pairs;
    const QueryDesc qd = qdesc[qi];
    const uint8_t* q = queries + qoffs[qi];
    const int m = (int)(qoffs[qi + 1] - qoffs[qi]);
    const int64_t total = (int64_t)kIntraCodes * qd.m_pad2;
    for (int64_t idx = start; idx < total; idx += stride) {
      const int c = (int)(idx / qd.m_pad2), i = (int)(idx % qd.m_pad2);
      prof2[qd.prof2_off + idx] = (int8_t)profile_score(q, m, mat, i, c);
    }
    if (prof3 && pb.add >= 0) {   // bytes, prof3_off in bytes
      const int words = qd.m_pad2 / 4;
      for (int64_t idx = start; idx < (int64_t)kIntraCodes * words; idx += stride)
        prof3[qd.prof3_off / 4 + idx] =
            pair_bytes(q, m, mat, (int)(idx % words) * 4, (int)(idx / words), pb);
    } else if (prof3) {   // packed binary16 row pairs [25][m_pad2 / 2] (the layout of k_profile)
      const int half_rows = qd.m_pad2 / 2;
      for (int64_t idx = start; idx < (int64_t)kIntraCodes * half_rows; idx += stride) {
        const int c = (int)(idx / half_rows), r = (int)(idx % half_rows);
        const uint32_t lo = half_bits(profile_score(q, m, mat, 2 * r, c));
        const uint32_t hi = half_bits(profile_score(q, m, mat, 2 * r + 1, c));
        prof3[qd.prof3_off + idx] = lo | (hi << 16);
      }
    }
  }
}

__global__ void k_fill(int32_t* __restrict__ p, int64_t n, int32_t v) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

}  // namespace

hipError_t launch_profile(const uint8_t* d_query, int m, const Matrix& mat, uint32_t* prof,
                          int m_pad, int R, int drift, int top, int top_score, int8_t* prof2,
                          uint32_t* prof3, const PairBytes& pb, int m_pad2, int32_t* flag_count,
                          hipStream_t s) {
  if (R <= 0 || R % 2 != 0 || m_pad % R != 0) return hipErrorInvalidValue;
  const int64_t total = (int64_t)(m_pad / R) * prof_strip_dwords(R) +
                        (int64_t)kIntraCodes * m_pad2 +
                        (prof3 ? (int64_t)kIntraCodes * (m_pad2 / (pb.add >= 0 ? 4 : 2)) : 0);
  int grid = (int)std::min<int64_t>((total + 255) / 256, 2048);
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(k_profile, dim3(grid), dim3(256), 0, s, d_query, m, mat, prof, m_pad, R,
                     drift, top, top_score, prof2, prof3, pb, m_pad2, flag_count);
  return hipGetLastError();
}

hipError_t launch_batch_profiles(const uint8_t* d_queries, const int64_t* d_qoffs, int n_queries,
                                 const Matrix& mat, const PairDesc* d_pairs, int n_pairs, int R,
                                 int drift, int64_t max_work, uint32_t* prof, const QueryDesc* d_qdesc,
                                 int8_t* prof2, uint32_t* prof3, const PairBytes& pb,
                                 hipStream_t s) {
  const int ys = n_pairs + n_queries;
  if (ys <= 0) return hipSuccess;
  if (ys > 65535) return hipErrorInvalidValue;
  const int gx = (int)std::max<int64_t>(1, std::min<int64_t>((max_work + 255) / 256, 256));
  hipLaunchKernelGGL(k_batch_profiles, dim3(gx, ys), dim3(256), 0, s, d_queries, d_qoffs, mat,
                     d_pairs, n_pairs, R, drift, prof, d_qdesc, prof2, prof3, pb);
  return hipGetLastError();
}

hipError_t launch_fill(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int grid = (int)std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_fill, dim3(grid), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

}  // namespace swdb
