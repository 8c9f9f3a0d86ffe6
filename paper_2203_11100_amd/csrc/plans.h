// The rules by which the host chooses the packed kernels' forms and launches:
// ranges of 16-bit values, profile bytes, workgroups and their row buffers.
// Plain C++, so that CPU tests compile and call them.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/swdb.h"

namespace swdb {

// Scoring matrix passed by value to the profile kernel.
struct Matrix {
  int8_t v[SW_ALPHA * SW_ALPHA];
};

// Intra-task profile (int8, [code][row]) has the 24 codes plus the pad code.
constexpr int kIntraCodes = 25;

// The packed inter-task kernels compute in IEEE binary16, which holds every
// integer of magnitude <= 2048 exactly.
constexpr int kHalfExact = 2048;

// Values of the drift form (packed16.h): what they start from, and the largest
// one the maxima order as integers.
constexpr uint32_t kDriftBase = 2560;
constexpr int kDriftTop = 31743;

// Matrices (ordinals) whose results are being gathered in one workgroup at
// once: the wave that would start one further ahead waits for the oldest to be
// finished.  At least as many as a workgroup has waves, so that queries of a
// single strip keep every wave busy.
constexpr int kRing = 16;

// The parameters of a drift sweep (packed16.h), the same in both halves of
// each word; group = 0: the binary16 form is used instead.
struct DriftArgs {
  int32_t group;              // strips until the drift starts again at its base
  int32_t guard;              // values need the guard to stay in range
  uint32_t c2;                // gap_open - gap_extend, at most 2048
  uint32_t ge2;               // the drift of one row or column
  uint32_t group2;            // the drift of a group's rows
  uint32_t lim2, over2;       // the rescoring limit; 32768 - the limit
};

// A global or semi-global search in the drift form (k_inter.hip): H~ = H + base
// + ge * (row + column), the query's rows shifted down so that its last row is
// the last strip's last.
struct ModeShape {
  int32_t mode;               // SW_MODE_LOCAL: the fields below are not used
  int32_t pad;                // rows above the query's first, < R
  int32_t base;
  int32_t go, ge, m;
  const int64_t* offs;        // sequence offsets
};

// The long-pair kernel's profile: bytes S + add of a query's rows, shifted down
// by `top` rows of top_byte; add -1: not the byte form.
struct PairBytes {
  int32_t add = -1;
  int32_t top = 0, top_byte = 0;
  int32_t code_byte = 0;      // the pad code's
  int32_t row_byte = 0;       // of rows past the query's end
};

// LDS of one workgroup of the long-pair kernel: profiles (dynamic) and the rest.
constexpr size_t kLdsBytes = 160 * 1024;
constexpr size_t pairs_lds(int R, int W, int n_pass, bool shared) {
  return (size_t)(shared ? n_pass : W) * kIntraCodes * 64 * R;
}
constexpr size_t pairs_lds_static(int W) { return (size_t)W * (1024 + 1024 + 12) + 512; }

// Rescoring limit of the packed kernels: the requested limit, at most 2048,
// below which every value is computed exactly (packed16.h).
inline int32_t effective_limit(int32_t requested) {
  return std::max<int32_t>(0, std::min<int32_t>(requested, kHalfExact));
}

// The matrix's largest score, at least 0.
inline int max_score(const Matrix& mat) {
  int max_s = 0;
  for (int x = 0; x < SW_ALPHA * SW_ALPHA; ++x) max_s = std::max<int>(max_s, mat.v[x]);
  return max_s;
}

// The drift form's parameters for a kernel whose bins have at most `cols`
// columns and whose strips have R rows (the arithmetic and the meaning of the
// range: packed16.h), or group = 0 where it does not fit and the binary16 form
// is used: gap_extend so large that the drift over the columns and one strip
// leaves no room (above 12 at 2,048 columns and the default limit).  The drift over the rows starts
// again every `group` strips, as many as fit (all of a usual query's).
// Batches give the columns of the short bins too: the groups are then sized so
// that these need no guard where that leaves at least 8 strips, and the kernel
// guards the matrices that do.
inline DriftArgs drift_plan(int m, int64_t cols, int R, const Matrix& mat, int32_t go, int32_t ge,
                     int32_t sat_limit, int64_t short_cols = 0) {
  DriftArgs d{};
  const int64_t limit = effective_limit(sat_limit);
  const int max_s = max_score(mat);
  // room for the drift of columns and rows, when scores stay below what the
  // lengths allow, or (guard) within some columns' gain of the limit
  const int64_t top = kDriftTop - (int64_t)kDriftBase - 256;
  auto score = [&](int64_t n) {
    return std::max<int64_t>(std::min<int64_t>((m + R - 1) / R * R, n) * max_s, limit);
  };
  const int64_t guarded = limit + (int64_t)(R + 8) * max_s;
  auto groups = [&](int64_t highest, int64_t n) -> int64_t {
    if (highest > top) return 0;
    if (ge == 0) return INT32_MAX / R;
    return ((top - highest) / ge - n - R - 8) / R;
  };
  int64_t g = groups(score(cols), cols);
  if (g < 1) {
    g = groups(guarded, cols);
    d.guard = 1;
    const int64_t gs = short_cols > 0 ? groups(score(short_cols), short_cols) : 0;
    if (gs >= 8) g = std::min(g, gs);
  }
  if (g < 1) return DriftArgs{};
  d.group = (int32_t)std::min<int64_t>(g, (m + R - 1) / R);
  auto both = [](int64_t v) { return (uint32_t)v | ((uint32_t)v << 16); };
  d.c2 = both(std::min<int32_t>(go - ge, kHalfExact));
  d.ge2 = both(ge);
  d.group2 = both((int64_t)ge * R * d.group);
  d.lim2 = both(limit);
  d.over2 = both(32768 - limit);
  return d;
}

// The long-pair kernel's drift form (k_pairs.hip) for one set of scores: `add`
// is what its profile bytes hold beside S (2 ge + bias), -1 where the form does
// not fit - the drift of a superstep and two supersteps' gain past the limit
// within the 16-bit range, scores within a byte - and k_intra_f16 is used.
struct PairForm : PairBytes {
  int bias = 0;
};
inline PairForm pair_form(const Matrix& mat, int32_t ge, int32_t sat_limit) {
  PairForm f;
  int lo = 0, hi = 0;
  for (int x = 0; x < SW_ALPHA * SW_ALPHA; ++x) {
    lo = std::min<int>(lo, mat.v[x]);
    hi = std::max<int>(hi, mat.v[x]);
  }
  const int64_t top = (int64_t)kDriftBase + effective_limit(sat_limit) + 140 * (int64_t)hi +
                      (int64_t)ge * (64 + 2 * 8 + 8) + 512;
  const int bias = std::max(0, -(lo + 2 * std::min(ge, 1024)));
  if (top > kDriftTop || hi + 2 * (int64_t)ge + bias > 255) return f;
  f.bias = bias;
  f.add = 2 * ge + bias;
  f.code_byte = f.row_byte = lo + f.add;     // the smallest score, or 0
  return f;
}

// Pairs one workgroup holds at once: each keeps a row buffer when it has more
// than one pass.
inline int pair_ring(int n_pass, int W) {
  return n_pass > 1 ? std::min(kRing, (W + n_pass - 1) / n_pass + 1) : kRing;
}

// A schedule of an inter-task kernel: strips of R rows, W waves, relative efficiency.
struct Sched {
  int R, W;
  double eff;
};

// The batched kernel's fitted schedules, with relative efficiencies: padded
// rows / kernel time of 24 queries of 50 .. 5,000 residues against 100,000
// plain sequences, every form forced (186.8 ms at 24 x 12, 200.0 at 12 x 12).
// Taller strips pay less for boundary rows and chunk starts, four waves a SIMD
// (16 waves, <= 128 VGPRs) hide more than three.
constexpr Sched kBatchScheds[] = {{24, 12, 1.000}, {16, 16, 0.997}, {20, 12, 0.987},
                                  {14, 16, 0.973}, {18, 12, 0.964}, {16, 12, 0.964},
                                  {14, 12, 0.951}, {12, 16, 0.951}, {12, 12, 0.932}};

// The batched kernel's rows and waves (0: any; false if none matches) for queries of
// these lengths, longest first, over half bins of `cols` columns together: the least
// of the work on all CUs, the pairs' padded rows, and the longest half bin with the
// longest pair on its one workgroup, whose strips lie on the four SIMDs round robin:
// the fullest one's rows set its time.  Two queries of 144 residues against 100,000
// plain sequences (longest half bin 8,188 columns), kernel ms: 24 x 12 (6 strips) 4.06,
// 16 x 12 (9) 4.03, 14 x 12 (11) 3.65, 18 x 12 (8) 3.26, 12 x 12 (12) 2.94.
inline bool batch_schedule(const int64_t* lens, int64_t n, double cols, double longest, int cus,
                           int rows, int waves, int* R_out, int* W_out) {
  double best = 1e300;
  for (const Sched& c : kBatchScheds) {
    if ((rows && c.R != rows) || (waves && c.W != waves)) continue;
    double padded = 0;
    for (int64_t i = 0; i < n; i += 2) padded += (double)((lens[i] + c.R - 1) / c.R * c.R);
    const int64_t strips = n > 0 ? (lens[0] + c.R - 1) / c.R : 0;
    const double work = padded / 4 * cols / std::max(cus, 1);
    const double chain = (double)((strips + 3) / 4 * c.R) * longest;
    const double cost = (std::max(work, chain) + 0.1 * std::min(work, chain)) / c.eff;
    if (cost < best) {
      best = cost;
      *R_out = c.R;
      *W_out = c.W;
    }
  }
  return best < 1e300;
}

// What the long-pair kernel is to score, and beside what.
struct PairLoad {
  int m = 0;                  // query rows (batches: the longest query's)
  double items = 0;           // pairs, segments of pairs, or pairs times queries
  double cols = 0;            // their columns together
  double longest = 0;         // and the longest one's
  double beside = 0;          // seconds the bins beside it take on the whole device
  const int64_t* bins = nullptr;   // their descriptors, longest first (BinDesc's words),
  int64_t n_bins = 0;
  double bin_col = 0;         // seconds one of them takes per column, alone on a CU
  int cus = 256;
  int rows = 0, waves = 0;    // 0: any, else fixed
  bool own = false;           // each wave stages its own pass's rows (batches)
};
struct PairLaunch {
  int R = 8, W = 1, grid = 1;   // rows per lane, waves per workgroup, workgroups
};

// Cycles between two steps of a SIMD's waves, all together, with one, two and
// four waves on it (300 pairs of long sequences on 24 CUs; 2.4 GHz).
struct StepCost {
  int R;
  double at1, at2, at4;
};
constexpr StepCost kStepCosts[] = {{2, 181, 124, 107}, {4, 238, 170, 154}, {8, 370, 288, 271}};
inline double step_cycles(const StepCost& c, double waves) {   // per SIMD
  if (waves <= 1) return c.at1 / std::max(waves, 1e-3);
  if (waves <= 2) return c.at1 + (c.at2 - c.at1) * (waves - 1);
  return c.at2 + (c.at4 - c.at2) * std::min(1.0, (waves - 2) / 2);
}

// Rows, waves and workgroups of the drift long-pair kernel: the least expected
// time of the pairs and the bins together.  One workgroup a CU (of waves that an
// option fixes below 8, up to 16 waves), spread over the CUs however few passes
// there are: packed so that every wave has a pass, 881 items of one pass took 56 CUs
// and 0.81 ms, over 224 of them 0.39 (47 residues, 12,500 sequences of the long mix).
// The pairs take the work on the CUs they get, or the longest one's chain: its
// columns times the rounds its passes take on one workgroup's waves.  Beside bins,
// whose workgroups share a CU with no other, at most 7/8 of the CUs, and fewer where
// the longest bin that waits for one of them would end last: a bin that waits for
// every pair's workgroup starts when the search is all but over (6,000 residues
// against 50,000 sequences of the long mix: 48 ms with every CU taken, 37 so).
// Against fixed counts of CUs, rows and waves swept over 37 searches of eight
// databases, 47 .. 10,000 residues: 2 % above the best of them on average, 13 % at
// most (without the spreading and the fullest SIMD's share in the chain: 17 %, 114 %).
inline PairLaunch pair_launch(const PairLoad& p) {
  PairLaunch best;
  double least = 1e300;
  const double cus = std::max(p.cus, 1);
  for (const StepCost& c : kStepCosts) {
    if (p.rows && c.R != p.rows) continue;
    const int P = std::max(1, (p.m + 64 * c.R - 1) / (64 * c.R));
    for (int W : {16, 8, 4, 2, 1}) {
      if (p.waves ? W != p.waves : W < 8) continue;
      const size_t lds = std::min(p.own ? kLdsBytes + 1 : pairs_lds(c.R, W, P, true),
                                  pairs_lds(c.R, W, P, false));
      if (lds + pairs_lds_static(W) > kLdsBytes) continue;
      const int conc = std::min(P, W);
      constexpr double kSixteenths[] = {14, 10, 8, 6, 5, 4, 3, 1.5};
      constexpr int kParts = sizeof(kSixteenths) / sizeof(*kSixteenths);
      for (int choice = W < 8 ? 0 : kParts; choice < 2 * kParts; ++choice) {
        // the CUs that get workgroups, and how many each
        const int per_cu = choice < kParts ? 16 / W : 1;
        const double sixteenths = kSixteenths[choice % kParts];
        const double most = std::max(1.0, p.beside > 0 ? cus * sixteenths / 16 : cus);
        const double grid = std::max(1.0, std::min(p.items, most * per_cu));
        const double on = std::min(grid, most);
        const double waves = std::min((double)W * per_cu, std::max<double>(conc, p.items * P / on));
        const double step = step_cycles(c, waves / 4);
        const double lead = p.longest + 128.0 * (conc - 1);
        // a round of passes takes the fullest SIMD's steps; a last round of fewer
        // starts while the one before still runs
        auto round = [&](int passes) {
          const double held = (passes + 3) / 4;
          return held * step_cycles(c, held);
        };
        const int full = P / W, rest = P % W;
        double chain = lead * (full * round(W) + (rest ? (full ? 0.5 : 1.0) * round(rest) : 0));
        // other pairs' waves on the same SIMDs
        chain *= 1 + 0.004 * (waves - conc) + (per_cu > 1 ? 0.1 : 0);
        const double work = 1.2 * p.cols * P * step / (4 * on);
        const double pairs = std::max(chain, work) + 0.1 * std::min(chain, work);
        double all = pairs;
        if (p.beside > 0) {
          const double busy = std::min(pairs * on, work * on + 0.2 * chain * on);
          all = std::max(pairs, p.beside * 2.4e9 + busy / cus);
          const int64_t now = (int64_t)(cus - on);    // bins that start at once
          if (now < p.n_bins)
            all = std::max(all, 0.7 * pairs + p.bin_col * 2.4e9 * (double)p.bins[4 * now + 2]);
        }
        // (where two agree the more CUs; 16 waves beside bins, 8 alone)
        const bool same = best.R == c.R && best.W == W;
        if (p.beside > 0 ? all < (same ? 0.995 : 1.0) * least : all <= least) {
          least = all;
          best.R = c.R;
          best.W = W;
          best.grid = (int)grid;
        }
        if (p.beside <= 0) choice += kParts - 1;     // alone: on all CUs
      }
    }
  }
  return best;
}

// Whether searches with a launch that measuring found (milliseconds of whole
// searches) are to use it: clearly shorter than with the one fitted to each query.
inline bool tuned_beats_fitted(double tuned, double fitted) { return tuned < 0.97 * fitted; }

// The binary16 long-pair kernel (k_intra_f16): a workgroup's W waves take one
// pair's passes in rounds, three supersteps a wave apart with their barriers.  The
// expected time of a search's pairs, in units of an instruction: the longest one's
// chain, or the work on 256 CUs, which idle waves in a last round (they issue
// little and hold their place: 0.35 of a pass), the start and end of a pair, and few
// waves on a CU (the profiles in LDS) lengthen.
inline double half_estimate(int m, double items, double cols, double longest, int R, int W) {
  const int P = std::max(1, (m + 64 * R - 1) / (64 * R)), rounds = (P + W - 1) / W;
  const double step = 8.0 * R + 32;
  const double steps = std::max(1.0, cols / std::max(items, 1.0) / 64);   // supersteps a pair
  const int per_cu = std::max(1, std::min<int>(16 / W, (int)(kLdsBytes / (W * 3200 * R + 2000))));
  const double few = 1 + 0.05 * std::max(0, 12 - per_cu * W);
  const double slots = 0.35 * rounds * W + 0.65 * P;
  const double work = cols * slots * step / 1024 * (steps + 3 * (W - 1)) / steps * few;
  const double chain = longest * rounds * step * 1.6;
  return std::max(chain, work) + 0.1 * std::min(chain, work);
}
// The rows and waves that end first by that estimate where they do so clearly,
// else R and W as they are (the shortest chain of one pair), also where the bins
// beside the pairs (`beside` residues) are most of the search.  Many short pairs ask
// for few waves: gaps 200/130, 20,001 plain sequences, 977 residues 3.24 ms with 4 x
// 4, 2.35 with 8 x 2.  Of 38 searches of seven databases for which full rounds in the
// place of `slots` named another form, 10 were 1 to 30 % slower with it (long mix of
// 50,000, 690 residues: 7.89 ms with 4 x 4, 9.00 with 4 x 1); of these, one still
// takes it and loses more than 3 % (two pairs of 2,000,000 residues, 450 residues:
// 1.26 ms with 2 x 4, 1.42 with 4 x 2), and one gain above 6 % is given up.
inline void half_rows(int m, double items, double cols, double longest, int* R, int* W,
                      double beside = 0) {
  if (beside > 4 * cols) return;
  double least = 0.8 * half_estimate(m, items, cols, longest, *R, *W);
  int r = *R, w = *W;
  for (int rows : {2, 4, 8})
    for (int waves : {1, 2, 4}) {
      const double est = half_estimate(m, items, cols, longest, rows, waves);
      if (est < least) {
        least = est;
        r = rows;
        w = waves;
      }
    }
  *R = r;
  *W = w;
}

// The row buffers of a launch of the long-pair kernel over `items` pairs (or
// segments, or pairs times queries) of `stride` columns at most: `ring` for each
// of `grid` workgroups, for the workgroups that are launched and no others.  Fewer
// pairs in flight, down to one, where all of them would take more than 512 MiB and
// more than one row for each of the items or 1,024 (what k_intra_f16 takes, and the
// binary16 searches took: at 2^24 residues a row has 134 MB); with `have` rows
// given instead, what fits in those.
constexpr int kIntraGridLong = 1024;   // workgroups sweeping the long list
constexpr int64_t kPairRowBytes = int64_t(512) << 20;
struct PairRows {
  int ring = 1, grid = 1;
  int64_t rows = 0;           // all of them; none for queries of one pass
};
inline PairRows pair_rows(int ring, int grid, int n_pass, int64_t items, int64_t stride,
                          int64_t have = -1) {
  PairRows r;
  r.ring = ring;
  r.grid = grid;
  if (n_pass <= 1) return r;
  const int64_t most = std::max<int64_t>(
      1, have >= 0 ? have
                   : std::max<int64_t>(std::min<int64_t>(items, kIntraGridLong),
                                       kPairRowBytes / (8 * std::max<int64_t>(stride, 1))));
  while (r.ring > 1 && (int64_t)r.ring * r.grid > most) --r.ring;
  r.grid = (int)std::min<int64_t>(r.grid, std::max<int64_t>(1, most / r.ring));
  r.rows = (int64_t)r.ring * r.grid;
  return r;
}

// A global or semi-global search's inter-task form: the packed drift kernel
// (k_inter.hip) where every value stays within 16 bits, else R = 0 and the int32
// kernel.  Values lie above base - 2 go (borders, and gaps from them) and below
// base plus what the cells of a path can gain: max S + 2 ge for each of at most
// min(rows, columns) matched pairs from the corner (global), or max S + ge from
// anywhere on the top border, which itself rises to ge * columns (semi-global).
// BLOSUM62 with gaps 10/2 fits for every query up to 2,047 columns.
struct ModePlan {
  int R = 0, W = 0, n_strips = 0;
  ModeShape shape{};
};
inline ModePlan mode_plan(int m, int64_t cols, const Matrix& mat, int64_t go, int64_t ge, int mode) {
  ModePlan p;
  const int64_t max_s = max_score(mat);
  // padded rows over relative rate, as for batches
  struct Form {
    int R, W;
    double eff;
  };
  static const Form forms[] = {{16, 16, 1.0}, {14, 16, 0.98}, {12, 16, 0.95}};
  double best = 1e300;
  for (const Form& c : forms) {
    const double cost = (double)((m + c.R - 1) / c.R * c.R) / c.eff;
    if (cost < best) { best = cost; p.R = c.R; p.W = c.W; }
  }
  p.n_strips = (m + p.R - 1) / p.R;
  const int64_t rows = (int64_t)p.n_strips * p.R;
  const int64_t base = 3 * go + 256;
  const int64_t pairs = std::min<int64_t>(rows, cols);
  const int64_t gain = mode == SW_MODE_GLOBAL ? pairs * (max_s + 2 * ge)
                                              : pairs * (max_s + ge) + ge * cols;
  if (base + ge * p.R + gain + 512 > kDriftTop || cols > kDriftTop) {
    p.R = 0;
    return p;
  }
  p.shape.mode = mode;
  p.shape.pad = (int32_t)(rows - m);
  p.shape.base = (int32_t)base;
  p.shape.go = (int32_t)go;
  p.shape.ge = (int32_t)ge;
  p.shape.m = m;
  return p;
}

// The long-pair kernel's form for a global or semi-global search and R rows a
// lane: the profile's bytes, and values within the 16-bit range (k_pairs.hip):
// above 0 from `base` on (a superstep's columns may lie before a lane's), and
// below the maxima's top by the gain of the shorter side.  add -1: the long list
// goes through the int32 kernel.
inline PairForm mode_pairs(int m, int64_t longest, const Matrix& mat, int32_t go, int32_t ge, int mode,
                    int R, ModeShape* shape) {
  PairForm f = pair_form(mat, ge, 1);
  if (f.add < 0) return f;
  const int64_t max_s = max_score(mat);
  const int64_t rows = (int64_t)(m + R - 1) / R * R;
  const int64_t pairs = std::min(rows, longest);
  const bool global = mode == SW_MODE_GLOBAL;
  const int64_t base = 3 * (int64_t)go + 256 + (global ? 0 : 128 * (int64_t)ge);
  const int64_t gain = global ? pairs * (max_s + 2 * ge) : pairs * max_s + ge * (rows + 136);
  if (base + ge * R + gain + 512 > kDriftTop) {
    f.add = -1;
    return f;
  }
  f.top = (int32_t)(rows - m);
  f.top_byte = f.bias + (global ? 0 : 2 * ge);
  f.code_byte = f.bias;
  shape->mode = mode;
  shape->pad = f.top;
  shape->base = (int32_t)base;
  shape->go = go;
  shape->ge = ge;
  shape->m = m;
  return f;
}

}  // namespace swdb
