// Rows scanned ahead of the trees that will ask for them: the scanner workgroups, shared by the
// launches that build capped and uncapped trees (ahead.hip).
#pragma once

#include "scan_device.h"

namespace talon {

constexpr int32_t kRowReady = 1 << 30;   // row ticket: merged results are in the workspace ...
constexpr int32_t kRowBad = 1;           // ... and the row could not be normalised

// LDS: a workgroup is a scanner or a selector.
struct ScannerLds {
  unsigned char pool[kScanBytes];
  unsigned long long topw[4][TALON_K_MAX];
  unsigned long long top[TALON_K_MAX];
  double wsum[4];
  float wmax[4];
  int wcnt[4];
  int nc, last, next, stop;
};
// Words that scanners look at: the item counter, and the sequences' stop words, each on a memory
// line of its own (in the descriptors of layers >= 1 of the other launch forms, zero between
// launches; those of layer 0 are not).
__device__ __forceinline__ uint32_t* item_counter(const ExpandArgs& a) { return a.exit_ticket + kItemWord; }
__device__ __forceinline__ int32_t* stop_word(const ExpandArgs& a, int b) {
  return reinterpret_cast<int32_t*>(a.desc + a.B + static_cast<size_t>(b) * (a.N_pad - 1));
}

__device__ __forceinline__ int ahead_items(const ExpandArgs& a) {
  return a.B * (a.ahead_head * a.ahead_chunks_head + (a.ahead_rows - a.ahead_head) * a.ahead_chunks);
}

// ---- scanner: workgroup `wg` of `n_wg`.  Its first item is its own number; the next ones come from
// a counter, in order: workgroups (and whole compute dies) progress at different speeds, and a
// row that a slow one holds back may be the one a selector waits for.  (Counters per die were
// tried: the slowest die's rows came 30 us late in a launch of 250 us.)
// FROM: rows are counted from first_row[b] on (past the last row that a tree of N nodes can expand
// there is none left to scan).
template <int EPL, bool FROM>
__device__ __forceinline__ void scan_rows(const ExpandArgs& a, ScannerLds& s, const int wg, const int n_wg, const int32_t* first_row) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int k = a.k;
  const ScanLds L{reinterpret_cast<uint4 (*)[kHitCap]>(s.pool), reinterpret_cast<int (*)[kHitCap]>(s.pool + kHitvBytes),
                  reinterpret_cast<unsigned long long (*)[kSubKeys]>(s.pool + kHitvBytes + kHithBytes), s.topw, s.top,
                  s.wmax, s.wsum, s.wcnt};
  unsigned long long* s_keys = reinterpret_cast<unsigned long long*>(s.pool);   // row merge: partial keys,
  unsigned long long* s_cand = s_keys + kMergeCap;                              // ... then those that can still be chosen
  static_assert(kScanBytes >= static_cast<int>(sizeof(unsigned long long)) * (kMergeCap + kCandCap + 16), "the scan buffers stage a row merge");
  const int blocks_per_row = a.chunks;
  const int head_items = a.ahead_head * a.B * a.ahead_chunks_head;
  const int n_items = ahead_items(a);
  int item = wg;
  if (tid == 0) s.stop = 0;
  __syncthreads();
  while (item < n_items) {
    const bool head = item < head_items;
    const int chunks = head ? a.ahead_chunks_head : a.ahead_chunks;
    const int bpc = (blocks_per_row + chunks - 1) / chunks;
    const int per_row = a.B * chunks;                 // items of one row id, all sequences
    const int in_part = head ? item : item - head_items;
    const int row_id = in_part / per_row;
    const int rest = in_part - row_id * per_row;
    const int b = rest / chunks;
    int node = head ? row_id : a.ahead_head + row_id;
    bool exists = true;
    if constexpr (FROM) { node += first_row[b]; exists = node <= a.sel.st.N - 2; }
    const int ch = rest - b * chunks;
    const int out_row = b * a.N_pad + node;
    const char* row = static_cast<const char*>(a.logits) +
                      (static_cast<int64_t>(b) * a.seq_stride + static_cast<int64_t>(node) * a.row_stride) * (16 / EPL);
    const int blk0 = ch * bpc;
    const int blk1 = blk0 + bpc < blocks_per_row ? blk0 + bpc : blocks_per_row;
    float m = kNegInf;
    double sum = 0.0;
    const bool scanned = exists && scan_chunk<EPL, false, true>(row, a.vocab, k, blk0, blk1, L, m, sum, stop_word(a, b), &s.stop);
    // (the counter is asked here: at the start of an item the row's first loads would wait behind a
    // thousand atomics on one word, about 20 ns each)
    int next = n_items;
    if (tid == 0 && n_items > n_wg)
      next = n_wg + static_cast<int>(__hip_atomic_fetch_add(item_counter(a), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (scanned) {
      const size_t slot0 = static_cast<size_t>(out_row) * blocks_per_row;
      unsigned long long* keys = a.part_keys + slot0 * k;
      bool row_done = chunks == 1;
      if (chunks > 1) {
        if (tid < k) store_agent(keys + static_cast<size_t>(ch) * k + tid, s.top[tid]);
        if (tid == 0) {
          store_agent(a.part_max + slot0 + ch, m);
          store_agent(a.part_sum + slot0 + ch, sum);
        }
        stores_performed();   // every partial store has completed before the ticket is taken
        __syncthreads();
        if (tid == 0) s.last = __hip_atomic_fetch_add(&a.ticket[out_row], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == chunks - 1;
        __syncthreads();
        if (s.last) {
          // (statistics: one chunk per lane, in every wavefront; more only for very long rows)
          row_done = true;
          const int nkeys = chunks * k;
          const int nkeys_pad = (nkeys + 15) & ~15;
          float mc0 = kNegInf;
          double sc0 = 0.0;
          if (lane < chunks) { mc0 = load_agent(a.part_max + slot0 + lane); sc0 = load_agent(a.part_sum + slot0 + lane); }
          for (int i = tid; i < nkeys_pad; i += kThreads) s_keys[i] = i < nkeys ? load_agent(keys + i) : 0ull;
          m = mc0;
          for (int c = lane + 64; c < chunks; c += 64) m = fmaxf(m, load_agent(a.part_max + slot0 + c));
          m = wave_max_f32(m);
          sum = rescaled_sum(sc0, mc0, m);
          for (int c = lane + 64; c < chunks; c += 64)
            sum += rescaled_sum(load_agent(a.part_sum + slot0 + c), load_agent(a.part_max + slot0 + c), m);
          sum = wave_sum_f64(sum);
          __syncthreads();   // the partial results have been read: slot 0 may be written
        }
      }
      if (row_done) {
        // ---- the row's results: k keys in descending order (zero: none), log-sum-exp, maximum
        int t = tid;
        asm volatile("" : "+v"(t));   // addresses are computed here, not kept across the streaming loop
        if (chunks == 1) {
          if (t < k) store_agent(keys + t, s.top[t]);
        } else {
          const int valid = a.vocab < k ? a.vocab : k;
          if (t >= valid && t < k) store_agent(keys + t, 0ull);
          rank_lists(k, s_keys, chunks, t, s_cand, &s.nc, [&](unsigned long long key, int r) { store_agent(keys + r, key); });
        }
        const double lse = static_cast<double>(m) + log_of_sum(sum);
        const bool bad = !(fabs(lse) <= 1.7e308);
        if (t == 0) {
          store_agent(a.part_max + slot0, m);
          store_agent(a.part_sum + slot0, lse);
        }
        stores_performed();
        __syncthreads();
        if (t == 0) store_agent(a.ticket + out_row, bad ? (kRowReady | kRowBad) : kRowReady);
      }
    }
    __syncthreads();   // every wavefront has looked at the stop flag
    if (tid == 0) { s.next = next; s.stop = 0; }
    __syncthreads();   // LDS is reused by the next item
    item = s.next;
  }
}

}  // namespace talon
