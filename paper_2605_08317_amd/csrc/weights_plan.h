// How many workgroups cut the key tiles into runs in the first weights pass, and whether the second one makes the rows' log-sum-exp
// itself, as host code that needs no HIP header.
#pragma once

#include <algorithm>
#include <cstdint>

namespace rdkv {

constexpr int kFewRuns = 34;           // of an item, that the second pass reads itself

struct RunPlan {
  int workgroups;                      // of the first pass
  bool few;                            // no item has more than kFewRuns runs: no launch for the log-sum-exp
};

// one round of workgroups (per_cu of them stay resident on a compute unit), at least one tile each
inline int workgroups_of(int64_t n_tiles, int per_cu) { return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(n_tiles, 256 * per_cu))); }

// n_tiles: key tiles of all items; most_tiles: of the longest; rows: window rows of an item.
inline RunPlan run_plan(int64_t n_tiles, int64_t most_tiles, int rows, int per_cu) {
  const int all = workgroups_of(n_tiles, per_cu);
  // Runs that an item of most_tiles tiles can meet: as many as tiles where each has a workgroup; otherwise runs of at least
  // n_tiles / workgroups tiles and a part of one at either end; of two tiles (the first has one where n_tiles is odd) half as many
  // and a half-run at one end.
  const int64_t alone = all == n_tiles ? most_tiles : most_tiles * all / n_tiles + 2, paired = (most_tiles + 1) / 2 + 1;
  const bool known = n_tiles < (1 << 22);
  if (!known || alone <= kFewRuns) return RunPlan{all, known};
  // Where every tile has a workgroup, half as many if that spares the launch of the log-sum-exp: compressing 8 x 3800 tokens 60.6 ->
  // 56.9 us, 2 x 4K 55.9 -> 53.6.  (Three or four tiles a run: 2 x 7000 tokens 56.8 -> 59.5; 256 rows, whose sums every
  // workgroup reads: 4 x 4000 tokens 54.4 -> 55.4.)
  if (rows <= 128 && all == n_tiles && paired <= kFewRuns) return RunPlan{static_cast<int>((n_tiles + 1) / 2), true};
  return RunPlan{all, false};
}

// Whether the second pass makes the log-sum-exp.  With channel weights, which go along with whichever launch makes it, their
// workgroups (four an item) have the second pass's LDS and registers, two to a compute unit, and come behind it: with up to 128 window
// rows and many items they take longer than the launch (microseconds, launch and second pass; 128 rows: 128 x 300 tokens of 8 heads
// 91.2, 95.3, 64 x 300 60.8, 61.1, 32 x 300 43.3, 41.2; 32 rows: 256 x 200 of 2 heads 50.0, 54.1, 64 x 500 of 4 30.9, 32.0, 128 x 300 of 2 40.2,
// 41.0, 64 x 300 of 2 35.6, 34.5; 256 rows: 128 x 300 of 8 124.9, 118.8).
inline bool lse_in_second_pass(const RunPlan& plan, int64_t n_items, int rows, bool channels) {
  return plan.few && !(channels && rows <= 128 && n_items > (rows <= 64 ? 128 : 256));
}

}  // namespace rdkv
