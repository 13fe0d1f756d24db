// Internal declarations shared by the translation units of libtalon (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "talon.h"

namespace talon {

constexpr int kThreads = 256;       // every kernel here runs 4 wavefronts per workgroup
constexpr int kScanTiles = 4;       // 16-byte vectors per thread per vocab chunk
constexpr int kChunkBytes = kThreads * kScanTiles * 16;  // 16 KiB of a logits row per workgroup pass
constexpr int kMergeCap = 2048;     // chunks * k keys one row merge stages in LDS
constexpr uint32_t kDoneMask = TALON_STATUS_DONE_BUDGET | TALON_STATUS_DONE_DEPTH | TALON_STATUS_ABORTED;

void set_error(const char* fmt, ...);
int check_hip(hipError_t e, const char* what);

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct SelectArgs {
  talon_tree_state st;
  int k;
  const int32_t* cand_token;
  const float* cand_prob;
  const double* cand_edge_logp;
  double log_mu;
  int K_init, init_layers, max_depth;
  // Optional: set to 1 when a selection keeps the last (k-th) candidate of a row, i.e. when the
  // per-row cap may have cut the pool of Alg. 2 short.  While it stays 0 the tree is the one the
  // uncapped pool gives: a selection that wants more than k tokens of a row also wants the row's
  // k best, all of which the capped pool holds.
  uint32_t* cap_hit;
};

// Workgroups leave the single-launch kernel through a two-level ticket (one counter for all
// of them would serialise several hundred atomics on one address at the end of the launch).
// Measured over 8 to 255 groups on grids of 300 to 700 workgroups: 128 is the fastest; fewer
// groups lengthen the first level, more lengthen the second.
constexpr int kExitGroups = 128;
// Words of the exit-ticket array: the groups' count, one count per group, the item counter of the
// launch that scans ahead, and a counter of selections (one layer per launch) or sequences (scan
// ahead) that have finished.
constexpr int kItemWord = kExitGroups + 1;
constexpr int kSelectedWord = kExitGroups + 2;
constexpr int kExitWords = kExitGroups + 3;
// One more word behind them, which no launch clears: the cap_hit flag of a speculative run.
constexpr int kCapHitWord = kExitWords;
constexpr unsigned long long kDescReady = 1ull << 63;

struct ExpandArgs {
  const void* logits;
  int64_t row_stride, seq_stride;
  int row_mode;
  int B, N_pad, vocab, k;
  int chunks;            // 16 KiB blocks per row = most chunks a row is ever cut into
  int target_items;      // (row, chunk) items a launch aims for when it cuts rows into chunks
  const int32_t* frontier_begin;
  const int32_t* frontier_count;
  uint32_t* status;
  int32_t* cand_token;
  float* cand_logit;
  float* cand_prob;
  double* cand_edge_logp;
  float* row_max;
  double* row_lse;
  float* part_max;       // [rows][chunks]
  double* part_sum;      // [rows][chunks]
  unsigned long long* part_keys;  // [rows][chunks][k]
  int32_t* ticket;       // [rows]
  // Fused modes (the scan runs the budget selection of a sequence in its tail, when the last
  // row of that sequence's frontier has been written): selection parameters, the index of
  // this launch in the loop, per-sequence row tickets and per-layer frontier descriptors
  // [N_pad][B], one 8-byte word each: begin in the low half, count and kDescReady in the
  // high half.  In the single launch, layer i reads desc[i] (desc[0] is copied from the public
  // tree state, or known when the launch starts the trees itself) and its selections write
  // desc[i+1], so a workgroup that is late still sees the frontier of its own layer.  A launch
  // of one layer reads the public tree state instead and holds its selections back until every
  // workgroup has done so.
  SelectArgs sel;
  int launch_idx;
  int32_t* seq_ticket;   // [B]
  unsigned long long* desc;
  // Single-launch mode: one grid walks all layers.  A descriptor is stored once everything
  // its selection wrote has been performed, with kDescReady set; a workgroup enters layer i
  // when every desc[i][b] is ready (it polls them; the wait is bounded by spin_ticks of the
  // 100 MHz wall clock).  Descriptors of layers >= 1 are zero between launches.
  // The launch leaves its workspace as it found it: every workgroup takes an exit ticket
  // when it has finished with tickets and descriptors and the last one clears them.  With
  // root_token set the launch also starts the trees itself (Alg. 2 line 1): layer 0 is the
  // root row of every sequence, and the workgroup that writes that row initialises the
  // sequence's state first.
  int layers;
  uint32_t* exit_ticket; // [kExitWords] workgroups that have left, counted per group, then the groups; see kItemWord
  unsigned long long spin_ticks;
  uint64_t* tree_mask;   // optional: ancestor masks written at the end of the single launch
  const int32_t* root_token;   // optional [B]
  const uint32_t* run_if;      // optional: the single launch does nothing unless this word is non-zero
  // Launch that scans rows ahead of the tree: rows 0 .. ahead_rows - 1 of every sequence; the first
  // ahead_head of them in ahead_chunks_head runs of blocks each, the others in ahead_chunks.
  int ahead_rows, ahead_head, ahead_chunks_head, ahead_chunks;
};

// Start of a single launch that continues trees: what it does with the five per-sequence words
// of the tree state (nodes, frontier begin and count, depth, status) besides reading them.
constexpr int kInitPlain = 0;     // nothing
constexpr int kInitSave = 1;      // copy them to `saved` [5][B] first
constexpr int kInitRestoreIf = 2; // if *flag is non-zero: put them back from `saved`, then start; else do nothing
struct FusedInitArgs {
  int mode;
  int32_t* saved;
  const uint32_t* flag;
  uint32_t* clear;   // optional: kExitWords + 1 words (exit tickets, layer counters, cap_hit) set to zero with kInitSave
};

// Uncapped ("paper-literal") layer of Alg. 2: the pool of a parent is its whole row.
#ifndef TALON_LITERAL_CHUNKS
#define TALON_LITERAL_CHUNKS 8
#endif
constexpr int kLiteralChunks = TALON_LITERAL_CHUNKS;     // parts a row is streamed in at most (their survivors, 8 * 255 keys, are merged in LDS)
constexpr int kLiteralRowCap = 256;   // survivors of one row that can still be chosen: at most N - 1 <= 255
struct LiteralPlan {   // what a layer does for one sequence
  double thr;          // gate threshold on the path score, log(mu) + anchor (-inf on top-K layers)
  int32_t active, F, fb, n, d, limit;
  uint32_t status;
  int32_t pad;
};
struct LiteralArgs {
  const void* logits;
  int64_t row_stride, seq_stride;
  int row_mode, vocab;
  talon_tree_state st;
  double log_mu;
  int K_init, init_layers, max_depth;
  int k_scan;                      // candidates per row the scan ranks (K_init on top-K layers, else 1)
  const int32_t* scan_token;       // [B*N_pad][k_scan] the scan's candidates ...
  const float* top_logit;          // [B*N_pad][k_scan] ... and their logits; the first is the row's largest
  const double* row_lse;           // [B*N_pad]
  int32_t* row_count;              // [B*N_pad] survivors kept of a row
  unsigned long long* row_key;     // [B*N_pad][kLiteralRowCap] their keys (sortable logit << 32 | ~token)
  // A row of a sequence with few rows is streamed in up to kLiteralChunks parts by as many
  // workgroups: part c of frontier row j of a layer that takes at most `limit` nodes leaves its
  // survivors at part_key[b * part_keys_per_seq + (j * parts + c) * limit] (rows * limit never
  // exceeds (N / 2)^2) and their number in part_count.
  unsigned long long* part_key;
  size_t part_keys_per_seq;
  int32_t* part_count;             // [B*N_pad][kLiteralChunks]
  int32_t* row_ticket;             // [B*N_pad] parts of a row that have finished; zero between launches
};

// The uncapped pool with rows scanned ahead (ahead.hip): `kLiteralScanK` best of every row.  A row is read again where its last
// one is kept, and a layer keeps at most N - 1: at most 15 rows, in kDeepParts parts together.
constexpr int kLiteralScanK = 16;
constexpr int kDeepParts = 64;
static_assert((TALON_N_MAX - 1) / kLiteralScanK <= kDeepParts, "a part for every row that is read again");
static_assert(kDeepParts <= 64 * kLiteralChunks, "their counts lie in 64 rows' part counts");
struct LiteralAhead {
  int helpers;                     // workgroups that read parts of rows again ...
  int late_helpers;                // ... and those that start when others have left, and stay while there is work
  int parts_per_seq;               // most parts of a sequence's request, at most kDeepParts (more only for more rows)
  int32_t* first_row;              // [B] first row to scan
  unsigned long long* request;     // [B][N_pad + 1] rows to read again: header, then node << 32 | logit bound; behind them [B][320] floors of the parts
  unsigned long long* part_key;    // [B][part_keys_per_seq] keys of the parts
  size_t part_keys_per_seq;
  int32_t* part_count;             // [B][N_pad * kLiteralChunks]
};

// Target argmax over every node of every tree.
struct ArgmaxArgs {
  const void* logits;
  int64_t row_stride, seq_stride;
  const int32_t* n_nodes;          // [B]
  int N_pad, vocab;
  int blocks;                      // 16 KiB blocks of a row
  int runs, blocks_per_run;        // runs a row is cut into
  float* part_max;                 // [B*N_pad][blocks] per run: maximum ...
  double* part_sum;                // ... sum of exp(logit - maximum) ...
  unsigned long long* part_key;    // ... and (sortable maximum << 32 | ~token); 0: nothing but NaN
  int32_t* target_token;           // [B][N_pad]
  float* target_prob;              // [B][N_pad] or NULL
  uint32_t* scan_status;           // [B]
};

// (Kernel arguments are fetched in lines of 64 bytes, a round trip each: with a fourth line a call of
// 15 us took 0.2 us longer.  What the kernels use together lies together.)
struct AttnArgs {
  const uint16_t* q;
  const uint16_t* k_prefix;
  const uint16_t* v_prefix;
  const uint16_t* k_tree;
  const uint16_t* v_tree;
  const uint64_t* mask;
  const int32_t* n_nodes;
  const int32_t* prefix_len;
  int B, N_pad, Hkv, G;  // G: query heads per KV head
  int max_prefix_len;
  float scale_log2e;     // scale * log2(e): scores are kept in base-2 units
  int64_t kv_stride_b, kv_stride_t, kv_stride_h;
  uint16_t* out;
  float* out_lse;
  // Split-KV: a (sequence, KV head, row tile) is cut into runs of key tiles, see attention.hip.
  uint16_t* part_o;      // [B][Hkv][split_max][Dh/8][rows_pad][8] bf16: each run's output, normalised by its own denominator
  float* part_m;         // [B][Hkv][split_max][rows_pad]  running max (base-2 units)
  float* part_l;         // the same: running denominator
  int32_t* part_count;   // [B] runs per row tile of the sequence (where the run length is worked out on the device)
  int capacity_per_head; // most workgroups per KV head (there)
  int run_bound;         // run length that fits the grid whatever the prefixes are
  int run_single;        // a sequence of at most this many key tiles is one run, whatever the run length is
  int split_max;         // most runs of one row tile (1: nothing is staged)
  int split_likely;      // runs of a full-length prefix
  int row_tiles;         // row tiles per (sequence, KV head)
  int rows_pad;          // rows of all of them
  int total_items;       // row_tiles * split_likely * B * Hkv: workgroups of full-length prefixes
};
static_assert(sizeof(AttnArgs) <= 192, "three lines");

// launchers (each checks nothing: arguments were validated by the ABI layer)
hipError_t launch_tree_init(const talon_tree_state& st, const int32_t* root_token, hipStream_t s);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);
hipError_t launch_prune(const talon_tree_state& st, int n_keep, int32_t* kept_ids, hipStream_t s);
hipError_t launch_argmax(const ArgmaxArgs& a, int dtype, int B, hipStream_t s);
hipError_t launch_accept(const talon_tree_state& st, const int32_t* target_token, const uint32_t* scan_status,
                         int32_t* path, int32_t* accept_len, int32_t* bonus_token, hipStream_t s);
hipError_t launch_compact_kv(const uint16_t* k_tree, const uint16_t* v_tree, const int32_t* path, const int32_t* accept_len,
                             const int32_t* prefix_len, int32_t* new_prefix_len, uint16_t* k_prefix, uint16_t* v_prefix,
                             int B, int N_pad, int Hkv, int Dh, int capacity, int64_t sb, int64_t st_, int64_t sh,
                             hipStream_t s);
hipError_t launch_read_probe(const void* buf, size_t bytes, void* sink, hipStream_t s);
hipError_t launch_mfma_probe(int workgroups, int iters, void* sink, hipStream_t s);
hipError_t launch_issue_probe(int mode, int waves, int iters, void* cycles, void* sink, hipStream_t s);
hipError_t launch_tile_load_probe(int loads, bool with_mfma, int waves, int iters, const void* window, void* cycles, void* sink, hipStream_t s);
hipError_t launch_fused_init(const talon_tree_state& st, const ExpandArgs& a, const FusedInitArgs& f, hipStream_t s);
hipError_t launch_expand_tree(const ExpandArgs& a, int dtype, int grid, hipStream_t s);
int expand_tree_max_grid(int dtype);
hipError_t launch_build_ahead(const ExpandArgs& a, int dtype, int grid, hipStream_t s);
hipError_t launch_literal_ahead(const ExpandArgs& a, const LiteralAhead& la, int dtype, int grid, void* counters, size_t counter_bytes, hipStream_t s);
int build_ahead_resident(int dtype);
int literal_ahead_resident(int dtype);
hipError_t launch_expand(const ExpandArgs& a, int dtype, int grid, bool fused, hipStream_t s);
hipError_t launch_select(const SelectArgs& a, hipStream_t s);
hipError_t launch_mask(const talon_tree_state& st, uint64_t* mask, hipStream_t s);
hipError_t launch_literal_layer(const LiteralArgs& a, int dtype, hipStream_t s);
hipError_t launch_attention(const AttnArgs& a, int Dh, int waves, bool balance, hipStream_t s);

int expand_chunk_elems(int dtype);

}  // namespace talon
