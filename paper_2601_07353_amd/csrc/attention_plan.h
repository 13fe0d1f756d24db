// Launch plan of tree attention.  Host code without HIP, so that tests can evaluate it on a machine
// without a GPU; attention.hip launches what it says.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "talon.h"

namespace talon {

constexpr int kKeyTile = 64;
// Fewest key tiles of a run (of a prefix that has more than that): the fewer keys a run has, the
// larger its normalised outputs are against the row's result, and their rounding to bf16 with them.
constexpr int kLeastRun = 4;

struct AttnPlan {
  int waves;             // wavefronts per workgroup
  int row_tiles, run_bound, run_single, split_max, split_likely, capacity_per_head, balance;   // as in AttnArgs
  size_t partial;        // bytes of the partial results ...
  size_t bytes;          // ... and with the table of run counts
};

// ---- Launch plan: rows per workgroup and the number of KV splits.
// A workgroup is 4 wavefronts (128 packed rows, two workgroups per compute unit) or 8 wavefronts
// (256 rows, one per compute unit: a K/V tile is loaded once for 256 rows instead of twice).  A split
// takes a run of key tiles; more splits shorten the runs but add workgroups, which run in rounds of
// what the chip holds, and partial results, which are written and read back by the merge.
// The plan is the one that fills the chip (as many splits as that takes, rounded up; 8 wavefronts from
// 512 rows on) unless another (width, splits) is estimated to be at least a tenth cheaper; with more
// than 64 splits, where the chip is filled by a costly merge, unless another is cheaper at all.  The
// estimate, in microseconds, is fitted to 330 measured plans of 22 shapes, 1 x 8 to 16 x 16 (sequence,
// KV head) pairs and 300 to 16000 keys (the cheapest by it are 0.7 % off the fastest plans on average, 7 %
// at most), and the merge of many splits to 1 to 8 KV heads of one sequence at 16384 to 262144 keys:
//   a round     a run of key tiles, plus 2.3 (queries, first tile, last stores)
//   a tile      8 wavefronts: 1.88; 4: 1.98 while two workgroups share a compute unit, 1.70 alone
//               (1.28 when the keys are in the Infinity Cache, which a model's many layers do not
//               leave them in); Dh = 64: 1.15, 1.20 and 1.10
//   merge       3.5, 0.07 per split beyond six and 0.05 more beyond 64, and the partial results' bytes,
//               twice, at 5 TB/s
// The filling plan alone leaves 288 workgroups on 256 places: 3 sequences of 200 nodes x 2 heads at 6000
// keys 76 us against 52, 6 x 250 x 4 at 9000 keys 186 against 140, 5 x 100 x 3 of 64 at 3001 keys 22 (ragged)
// against 19; and 410 splits of one head of 64 rows at 131072 keys: 65 us against 42 with 158.

inline int legacy_waves(int rows) { return rows >= 512 ? 8 : 4; }

inline size_t partial_bytes(long long row_tiles_all, int splits, int row_tile, int Dh) {
  if (splits == 1) return 256;   // nothing is staged, keep a token size
  return static_cast<size_t>(row_tiles_all) * splits * row_tile * (Dh * sizeof(uint16_t) + 2 * sizeof(float));
}

inline int key_tiles(int N_pad, int max_prefix_len) { return (max_prefix_len + kKeyTile - 1) / kKeyTile + N_pad / kKeyTile; }

inline double plan_us(int waves, long long wgs, int run, int splits, int Dh, size_t bytes) {
  const long long slots = waves == 8 ? 256 : 512;
  const long long full = wgs / slots, rest = wgs % slots;
  const double shared = Dh == 64 ? (waves == 8 ? 1.15 : 1.20) : (waves == 8 ? 1.88 : 1.98);
  const double alone = waves == 8 ? shared : (Dh == 64 ? 1.10 : 1.70);
  double us = full * (run * shared + 2.3);
  if (rest) us += run * (rest > 256 ? shared : alone) + 2.3;   // the last round's workgroups
  if (splits > 1)
    us += 3.5 + 0.07 * (splits > 6 ? splits - 6 : 0) + 0.05 * (splits > 64 ? splits - 64 : 0) + 2.0 * static_cast<double>(bytes) / 5e6;
  return us;
}

// Splits that fill the chip, rounded up: where the estimate starts from.
inline int filling_splits(long long pairs, int waves, int tiles) {
  long long want = ((waves == 8 ? 256 : 512) + pairs - 1) / pairs;
  const long long cap = tiles / kLeastRun > 1 ? tiles / kLeastRun : 1;
  if (want > cap) want = cap;
  const int run = static_cast<int>((tiles + want - 1) / want);
  return (tiles + run - 1) / run;
}

// Bytes of workspace that a call must bring.
inline size_t attention_least_workspace(int B, int N_pad, int Hq, int Hkv, int Dh, int max_prefix_len) {
  const int rows = N_pad * (Hq / Hkv);
  const int waves = legacy_waves(rows);
  const int mt = 32 * waves;
  const int row_tiles = (rows + mt - 1) / mt;
  const long long pairs = static_cast<long long>(B) * Hkv * row_tiles;
  return partial_bytes(pairs, filling_splits(pairs, waves, key_tiles(N_pad, max_prefix_len)), mt, Dh);
}

// Workspace whose splits a plan may choose from beyond what a call must bring: short prefixes gain from
// more splits than that, as long as the partial results stay small.  A caller whose workspace was sized
// for another (longer) prefix gets the best plan that fits it.
constexpr size_t kAttnPlanBytes = static_cast<size_t>(16) << 20;
inline size_t attention_plan_limit(size_t least) {
  return (least > kAttnPlanBytes ? least : kAttnPlanBytes) + TALON_B_MAX * sizeof(int32_t);   // + the table of run counts
}

// The plan of a call that may use `bytes` of workspace (at least attention_least_workspace; a plan needs
// plan.bytes of them).
inline AttnPlan attention_plan(int B, int N_pad, int Hq, int Hkv, int Dh, int max_prefix_len, size_t bytes) {
  const size_t limit = attention_plan_limit(attention_least_workspace(B, N_pad, Hq, Hkv, Dh, max_prefix_len));
  const size_t search_bytes = bytes < limit ? bytes : limit;
  const int rows = N_pad * (Hq / Hkv);
  const int tiles = key_tiles(N_pad, max_prefix_len);
  const size_t table = (static_cast<size_t>(B) * sizeof(int32_t) + 15) & ~static_cast<size_t>(15);   // runs per sequence
  AttnPlan best = {};
  int best_splits = 1;
  double best_us = 0.0;
  bool other = false;   // another plan than the one that fills the chip
  bool staged;   // may partial results be staged?  They are rounded to bf16: only where the plan that fills the chip has them too
  // Another plan than the one that fills the chip has to promise a tenth less: differences of a few
  // percent are within the estimate's error (8 -> 4 wavefronts promised 5 % at 3 sequences of 227
  // nodes x 4 heads and 376 keys and cost 7 %), the plans it is for gain a quarter or more.
  {
    const int waves = legacy_waves(rows);
    const int mt = 32 * waves;
    const int row_tiles = (rows + mt - 1) / mt;
    const long long all = static_cast<long long>(B) * Hkv * row_tiles;
    const int splits = filling_splits(all, waves, tiles);
    staged = splits > 1;
    best.run_single = staged ? (tiles + splits - 1) / splits : 0;
    best.waves = waves;
    best.row_tiles = row_tiles;
    best.run_bound = (tiles + splits - 1) / splits;
    best_splits = splits;
    best_us = (splits <= 64 ? 0.9 : 1.0) * plan_us(waves, all * splits, best.run_bound, splits, Dh, partial_bytes(all, splits, mt, Dh));
  }
  for (int waves = 8; waves >= 4; waves -= 4) {
    const int mt = 32 * waves;
    const int row_tiles = (rows + mt - 1) / mt;
    const long long all = static_cast<long long>(B) * Hkv * row_tiles;
    const int most = !staged || tiles < 2 * kLeastRun ? 1 : tiles / kLeastRun;
    for (int splits = 1; splits <= most;) {   // the fewest splits of every run length
      const int run = (tiles + splits - 1) / splits;
      const size_t need = partial_bytes(all, splits, mt, Dh);
      if (splits > 1 && need > search_bytes) break;
      const double us = plan_us(waves, all * splits, run, splits, Dh, need);
      if (us < best_us) {
        best.waves = waves;
        best.row_tiles = row_tiles;
        best.run_bound = run;
        best_splits = splits;
        best_us = us;
        other = true;
      }
      if (run == 1) break;
      splits = (tiles + run - 2) / (run - 1);
    }
  }
  // Balancing of unequal sequences: a row tile may take up to twice as many runs, as far as the
  // workspace goes, and the grid grows to what its rounds hold, short of what would give full-length
  // sequences one split more.  It costs a workgroup about 0.5 us before its first load, so runs
  // have to be long enough for it to matter.
  // The plan that fills the chip balances within the workspace of the search only: at heads of 128 that
  // leaves it as it is for 2, 4, 8 or 16 sequences of 8 KV heads, whose partial results fill it.
  // Another plan of two runs or more may take what twice its runs need (one of a single run would stage
  // rows that it otherwise passes to the output in fp32).  It was chosen for full-length prefixes, and
  // unequal ones can leave it slower than the filling one: 3 sequences of 68 nodes, 64/16 heads of 64,
  // prefixes of 4525, 6643 and 9213 of 14916 keys took 119 us unbalanced, 97 with the filling plan, 100 balanced; 7 of
  // 93 nodes, 16/2 heads of 128, up to 9396 keys 64, 108 and 50.
  const int mt = 32 * best.waves;
  const long long all = static_cast<long long>(B) * Hkv * best.row_tiles;
  const long long slots = best.waves == 8 ? 256 : 512;
  best.split_max = best.split_likely = best_splits;
  long long wgs = all * best_splits;
  if (B > 1 && staged && best.run_bound >= 2 * kLeastRun) {
    const long long rounds = (wgs + slots - 1) / slots;
    const size_t room = other && best_splits > 1 ? bytes : search_bytes;
    for (int m = 2 * best_splits; m > best_splits; --m)
      if (partial_bytes(all, m, mt, Dh) + table <= room) { best.split_max = m; break; }
    if (best.split_max > best_splits) {
      best.balance = 1;
      long long grown = all * (best_splits + 1) - 1;
      if (grown > rounds * slots) grown = rounds * slots;
      if (grown > wgs) wgs = grown;
    }
  }
  best.capacity_per_head = static_cast<int>(wgs / Hkv);   // (wgs >= all * splits, a multiple of Hkv)
  best.partial = partial_bytes(all, best.split_max, mt, Dh);
  best.bytes = best.balance ? best.partial + table : best.partial;
  return best;
}

}  // namespace talon
