// Launch plan of the kernel that scans rows ahead of the tree (ahead.hip).  Host code without HIP, so
// that tests can evaluate it on a machine without a GPU.
#pragma once

#include "talon.h"

namespace talon {

struct AheadPlan {
  bool layered;      // scan one layer after the other instead (talon_build_tree)
  int rows;          // rows 0 .. rows - 1 of every sequence are scanned ...
  int head;          // ... the first of them in chunks_head runs of blocks each, the others in chunks
  int chunks_head, chunks;
  int scanners;      // workgroups that scan
};

// Rows a tree can expand at most: N - 1 (the budget's last node has no children), and no more than its
// layers 0 .. max_depth - 1 can hold.  A layer has at most k children per parent, K_init in all on
// top-K layers.
inline int ahead_rows(int N, int k, int K_init, int init_layers, int max_depth) {
  long long rows = 0, width = 1;
  for (int d = 0; d < max_depth && rows < N - 1; ++d) {
    rows += width;
    width *= k;
    if (d < init_layers && width > K_init) width = K_init;
    if (width > N) width = N;
  }
  return static_cast<int>(rows < N - 1 ? rows : N - 1);
}

// blocks: of a row; resident: workgroups the device holds at once.
inline AheadPlan ahead_plan(int B, int N, int blocks, int k, int K_init, int init_layers, int max_depth, int resident) {
  AheadPlan p;
  p.layered = false;
  p.rows = ahead_rows(N, k, K_init, init_layers, max_depth);
  const long long rows_all = static_cast<long long>(B) * p.rows;
  long long scanners = resident - B > resident / 2 ? resident - B : resident / 2;
  // Runs of blocks per row: as many as give every scanner of a full grid at most one item.  Items
  // that nobody has to queue for need no counter, and every further item of a workgroup costs it
  // about 10 us between two streams (ranking, partial results, tickets): 508 rows of 304 KB take
  // 52 us as 1016 items and 55-57 us as 1524 or 2032; 4080 rows 250 us whole and 280 us in two.
  auto runs = [&](long long want) {   // a number of equal runs of whole blocks
    const int c = want < 1 ? 1 : (want > blocks ? blocks : static_cast<int>(want));
    const int bpc = (blocks + c - 1) / c;
    return (blocks + bpc - 1) / bpc;
  };
  p.chunks = runs(scanners / rows_all);
  p.head = 0;
  p.chunks_head = 1;
  const long long two_layers = 1 + (init_layers > 0 && K_init < k ? K_init : k);   // rows of the root and of layer 1
  const bool long_runs = p.chunks * 10 < blocks;   // runs of more than ten blocks, 35 us and more at the full rate
  // Scanned one layer after the other instead:
  // * trees of which a top-K layer is all there is to select (it spends the budget, or max_depth is 1):
  //   nothing can be scanned ahead, and a row or many are scanned in vain.  26 x 19 nodes, rows of
  //   257 KB, k 32: 26 us, 52 ahead; 8 x 30 of 304 KB: 24, 41; 3 x 12 of 64 KB, k 16: 16, 19.5.  Except where
  //   rows have 32 blocks or more and the grid allows longer runs: a layer of few rows is cut into
  //   single blocks, and merging those costs more than the scan in vain: 4 x 30 of 608 KB: 87, 38 ahead.
  //   (Without a top-K layer the rows decide whether the first layer spends the budget: 8 x 30 flat
  //   rows 28 us, 41 ahead, mixed ones 81, 46 ahead; one layer by the gate alone 18.5, 15.5 ahead.)
  // * with long runs, budgets of at most five times the first layer's width, which are usually spent
  //   when that layer is expanded: most of the scan would be in vain.  13 or 16 x 72 rows of 513 KB
  //   of which 17 per sequence are expanded: 74 us layer by layer, 82 and 87 ahead.  (Budgets above
  //   that, or rows that fit in one round, are faster ahead: 4 x 127 rows of 513 KB 78 against
  //   104, 16 x 29 of 304 KB 49 against 65.)
  // * at most three layers and more than 20 blocks per scanner: the hand-over between two layers that the
  //   scan ahead saves weighs less than the rows it may read in vain.  16 x 199 rows of 304 KB of which
  //   54 are expanded: 108 us, 149 ahead; 10 x 73 of 608 KB, 18 expanded: 75, 104.  (Below that: 4 x 73 of
  //   608 KB, 14 expanded: 70 us, 48 ahead; 8 x 73 of 304 KB, all expanded: 86, 68.)
  const bool one_layer = init_layers > 0 && (two_layers >= N || p.rows == 1);
  p.layered = (one_layer && (blocks < 32 || p.chunks == blocks)) || (long_runs && N - 1 <= 5 * (two_layers - 1)) ||
              (max_depth <= 3 && rows_all * blocks > 20 * scanners);
  if (long_runs) {
    // A tree that ends after two or three layers would wait for whole rows of all sequences to be
    // read before its root's row is there.  The first rows, as many as fill the grid once, are cut
    // into shorter runs: of five blocks, or as long as it takes for the rows of the first two
    // layers to fit.
    const long long one_round = scanners / (B * two_layers);
    const long long shortest = (blocks + 4) / 5;
    p.chunks_head = runs(one_round < shortest ? one_round : shortest);
    const long long fill = scanners / (static_cast<long long>(B) * p.chunks_head);
    const long long head = fill > two_layers ? fill : two_layers;
    p.head = head < p.rows ? static_cast<int>(head) : p.rows;
    const long long rest = static_cast<long long>(B) * (p.rows - p.head);
    const int by_size = (blocks + 19) / 20;   // at most twenty blocks per run
    const long long by_grid = rest > 0 ? scanners / rest : 1;
    p.chunks = runs(by_grid > by_size ? by_grid : by_size);
  }
  const long long items = static_cast<long long>(B) * (static_cast<long long>(p.head) * p.chunks_head +
                                                       static_cast<long long>(p.rows - p.head) * p.chunks);
  p.scanners = static_cast<int>(scanners < items ? scanners : items);
  return p;
}

// Does an uncapped call whose rows are all in place go layer by layer all the same?  least: layers it may build; blocks: of
// all rows it would scan; capped: trees of at most 64 nodes, whose layered form is the capped loop, first with `cap_tried`
// candidates per row.
// * Fewer than four layers: three launches a layer weigh less than rows scanned in vain.  2 x 250 nodes, rows of 257 KB: two
//   layers 53 us (peaked rows; flat 101), 55 ahead (113), three 83 (107), 56 (114), four 119 (112), 64 (114); 4 x 250 of
//   304 KB: 56 (109), 91 (147); 90 (115), 95 (147); 130 (121), 101 (149).  (At most eight blocks per scanner would gain from two
//   or three layers on: 1 x 60 of 257 KB 48, 29; they stay as they were.)
// * More than 8 blocks per scanner for every layer beyond the first: trees of few layers read a part of what is scanned.
//   16 x 250 of 128 KB (31 blocks), peaked / flat / every other one: four layers 174, 166, 218 us, 185, 210, 209 ahead; five 238, 172, 266, 206, 209,
//   214.  8 x 250 of 304 KB (37): four 170, 139, 200, 179, 177, 203; six 282, 151, 291, 207, 178, 211.  16 x 250 of 304 KB (74): five 325,
//   233, 333, 320, 256, 301; eight 539, 251, 504, 360, 256, 313; twelve 629, 275, 529, 363, 257, 313.  16 x 250 of 513 KB (125): eight 567, 230,
//   487, 599, 333, 447; twenty-four 707, 326, 582, 608, 335, 448.
// * Trees of which a top-K layer is all there is to select.  The capped loop has them in one launch where its first number of
//   candidates holds all children (8 x 33 of 257 KB 32 us, 68 ahead; 26 x 24 33, 116), and needs a second launch beyond (8 x 36: 100,
//   68; 26 x 48 159, 116).  Above 64 nodes one row is read again by few workgroups, and the other rows are scanned in
//   vain: 1 x 128 of 257 KB 88, 66; 4 x 100 88, 78; 16 x 100 (25 blocks) 122, 152; 8 x 128 (16) 91, 106; 8 x 144 of 40 KB 79, 90; 1 x 250 of 40 KB 77, 98; 4 x 250 of
//   257 KB 97, 107.
inline bool literal_layered(int N, int K_init, int init_layers, int least, long long blocks, int resident, bool capped, int cap_tried) {
  if (least < 4) return true;
  if (init_layers > 0 && K_init >= N - 1) return (capped && N - 1 <= cap_tried) || N > 128 || blocks > 12ll * resident;
  return blocks > 8ll * (least - 1) * resident;
}

}  // namespace talon
