// Alg. 2 for trees whose draft rows are all resident: rows are scanned ahead of the tree.
//
// With rows addressed by node id (TALON_ROWS_BY_NODE) the softmax statistics and the k best
// tokens of row i do not depend on which token node i turns out to carry, so nothing about a row
// has to wait for the selection that creates its node.  One launch, two roles:
//   scanners   take (row, chunk) items in row order -- row 0 of every sequence, row 1 of every
//              sequence, ... -- at the rate of memory, without ever waiting for anything; the
//              workgroup that finishes a row's last chunk leaves the row's k best keys and its
//              log-sum-exp in the workspace and marks the row ready;
//   selectors  (one workgroup per sequence, the last ones of the grid) run the sequence's whole
//              loop: wait until the frontier's rows are ready, select, append, next layer; the
//              tree under construction lives in LDS, and the ancestor mask is written from
//              there.  A finished sequence raises a word that its scanners poll, so rows that
//              the tree does not need are given up.
// A layer of the loop in expand.hip is a chain of about six memory round trips (descriptor, row
// chunks, partial results, row ticket, sequence ticket, selection) during which little is read:
// 10-14 us per layer whatever its width.  Here the scan is one stream and a layer costs the
// selection alone (two round trips and a few barriers), most of it under the scan.
//
// Scanners come first in the grid and never wait, so selectors always get what they wait for,
// whether or not the grid is resident as a whole; the wait is bounded all the same, and a
// selector that gives up marks every sequence TALON_STATUS_ABORTED as the other launch does.
//
// Scanners run four workgroups per compute unit without prefetching across blocks (three with
// prefetch: 8 % slower at 4080 rows, equal below).  Bound: memory while rows are scanned
// (4.4 TB/s over 4080 rows of 304 KB), then 2 us per layer that is left to select.
// Measured, this launch against the loop of expand.hip (tree and mask, resident inputs):
//   1 x 1024 f32, 16 nodes: 17 us (42);  1 x 128256 bf16, 60 nodes: 24 us (54);
//   4 x 151936, 128 nodes: 53 us (107);  16 x 151936, 256 nodes: 233-250 us (280).
#include "scan_device.h"

namespace talon {

namespace {

constexpr int32_t kRowReady = 1 << 30;   // row ticket: merged results are in the workspace ...
constexpr int32_t kRowBad = 1;           // ... and the row could not be normalised

// LDS: a workgroup is a scanner or a selector.
struct ScannerLds {
  unsigned char pool[kScanBytes];
  unsigned long long topw[4][TALON_K_MAX];
  int part[4][64];
  unsigned long long top[TALON_K_MAX];
  double wsum[4];
  float wmax[4];
  int wcnt[4];
  int nc, last, next, stop;
};
// Slots of the selector's key array: the threads of a row hold at most k + 2^lt - 1 candidates
// between them, and every thread's slots are padded to an odd number; F * k <= kMaxCand and
// F * 2^lt <= kThreads.
constexpr int kAheadKeySlots = kMaxCand + 2 * kThreads;
struct SelectorLds {
  unsigned long long key[kAheadKeySlots];
  double logp[TALON_N_MAX];   // path scores of the tree's nodes
  unsigned char parent[TALON_N_MAX];   // (not of the root)
  int hist[256];
  unsigned long long red_u64[8];
  int red_i32[8];
  int misc[2];
  int state;                  // what the wait for a layer's rows found
  unsigned long long ready[TALON_N_MAX / 64];   // rows known to be ready (and normalised)
};
constexpr size_t kAheadLds = sizeof(ScannerLds) > sizeof(SelectorLds) ? sizeof(ScannerLds) : sizeof(SelectorLds);

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
template <int EPL>
__device__ __forceinline__ void scan_rows(const ExpandArgs& a, ScannerLds& s, const int wg, const int n_wg) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int k = a.k;
  const ScanLds L{reinterpret_cast<uint4 (*)[kHitCap]>(s.pool), reinterpret_cast<int (*)[kHitCap]>(s.pool + kHitvBytes),
                  reinterpret_cast<unsigned long long (*)[kSubKeys]>(s.pool + kHitvBytes + kHithBytes), s.topw, s.part, s.top,
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
    const int node = head ? row_id : a.ahead_head + row_id;
    const int b = rest / chunks;
    const int ch = rest - b * chunks;
    const int out_row = b * a.N_pad + node;
    const char* row = static_cast<const char*>(a.logits) +
                      (static_cast<int64_t>(b) * a.seq_stride + static_cast<int64_t>(node) * a.row_stride) * (16 / EPL);
    const int blk0 = ch * bpc;
    const int blk1 = blk0 + bpc < blocks_per_row ? blk0 + bpc : blocks_per_row;
    float m;
    double sum;
    const bool scanned = scan_chunk<EPL, false, true>(row, a.vocab, k, blk0, blk1, L, m, sum, stop_word(a, b), &s.stop);
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
          sum = (mc0 != kNegInf) ? sc0 * static_cast<double>(__expf(mc0 - m)) : 0.0;
          for (int c = lane + 64; c < chunks; c += 64) {
            const float mc = load_agent(a.part_max + slot0 + c);
            if (mc != kNegInf) sum += load_agent(a.part_sum + slot0 + c) * static_cast<double>(__expf(mc - m));
          }
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

// ---- selector: the loop of Alg. 2 for sequence b.  
// exit_ticket(ok): takes the workgroup's exit ticket; called when everything other workgroups
// of the launch look at has been performed.
template <typename Exit>
__device__ __forceinline__ void select_layers(const ExpandArgs& a, SelectorLds& s, const int b, Exit&& exit_ticket) {
  const SelectArgs& sa = a.sel;
  const talon_tree_state& st = sa.st;
  const int tid = threadIdx.x;
  const int k = a.k;
  const size_t base = static_cast<size_t>(b) * st.N_pad;
  const int blocks_per_row = a.chunks;
  // Alg. 2 line 1: T = {x_t}, p(x_t) = 1
  if (tid == 0) {
    st.token[base] = a.root_token[b];
    st.parent[base] = -1;
    st.depth[base] = 0;
    st.prob[base] = 1.f;
    st.logp[base] = 0.0;
    s.logp[0] = 0.0;
    s.state = 0;
  }
  if (tid < TALON_N_MAX / 64) s.ready[tid] = 0ull;
  bool own_ready = false;   // row `tid` of the sequence is known to be ready
  int n = 1, fb = 0, F = 1, d = 0;
  uint32_t status = 0u;
  bool waited_out = false;
  __syncthreads();
  while (true) {
    // ---- scores of the pool.  A frontier row is shared by 2^lt consecutive threads; thread t owns
    // `per` <= 32 consecutive candidates of row t >> lt, so that the threads' candidates follow
    // one another in (parent, rank) order.  Every thread waits for its own row and goes on from
    // there without waiting for the others: the candidates of rows that are ready early are
    // scored while the last row is still being scanned.
    int lt = 0;
    while ((2 << lt) * F <= kThreads && (1 << lt) < k) ++lt;
    const int p = tid >> lt;
    const int share = (k + (1 << lt) - 1) >> lt;
    const int stride = share | 1;         // odd: the 64-bit LDS accesses of a wavefront fall on distinct banks
    const int per = p < F ? share : 0;    // (threads without a row own no slots)
    const int rank0 = (tid - (p << lt)) * share;
    unsigned long long* my = s.key + tid * stride;
    unsigned long long anchor = 0ull;
    int tok_r[kRegCand];                  // token, edge probability and score of the first candidates stay in registers
    float prob_r[kRegCand];
    double score_r[kRegCand];
    const size_t slot0 = (base + fb + (p < F ? p : 0)) * blocks_per_row;
    const unsigned long long* row_keys = a.part_keys + slot0 * k;
    double plogp = 0.0, lse = 0.0;
    if (p < F) plogp = s.logp[fb + p];
    if (p < F && !((s.ready[(fb + p) >> 6] >> ((fb + p) & 63)) & 1ull)) {
      const int32_t* word = a.ticket + base + fb + p;
      int32_t v = load_agent(word);
      if (v < kRowReady) {
        const unsigned long long t0 = wall_clock64();
        do {
          if (wall_clock64() - t0 > a.spin_ticks) { atomicOr(&s.state, 2); break; }
          __builtin_amdgcn_s_sleep(1);
          v = load_agent(word);
        } while (v < kRowReady);
      }
      if (v >= kRowReady && (v & kRowBad)) atomicOr(&s.state, 1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // the row's results are loaded after its ready mark has been seen
    lse = load_agent(a.part_sum + slot0);
    auto score_group = [&](const int i0, int (&tok)[kRegCand], float (&prob)[kRegCand], double (&scr)[kRegCand]) __attribute__((always_inline)) {
      unsigned long long kk[kRegCand];
#pragma unroll
      for (int u = 0; u < kRegCand; ++u) {   // all loads of a group in flight together
        const bool mine = i0 + u < per && rank0 + i0 + u < k;
        kk[u] = load_agent(row_keys + (mine ? rank0 + i0 + u : 0));
        if (!mine) kk[u] = 0ull;
      }
#pragma unroll
      for (int u = 0; u < kRegCand; ++u) {
        if (i0 + u < per) {
          const double edge = static_cast<double>(unsortable_f32(static_cast<uint32_t>(kk[u] >> 32))) - lse;
          const double score = plogp + edge;
          tok[u] = static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(kk[u]));
          prob[u] = __expf(static_cast<float>(edge));
          scr[u] = score;
          unsigned long long key = 0ull;
          if (kk[u] != 0ull && score == score) {
            key = sortable_u64(score);
            if (key == 0ull) key = 1ull;
          }
          my[i0 + u] = key;
          anchor = key > anchor ? key : anchor;
        }
      }
    };
    score_group(0, tok_r, prob_r, score_r);
    for (int i0 = kRegCand; i0 < per; i0 += kRegCand) {
      int tok_x[kRegCand];
      float prob_x[kRegCand];
      double score_x[kRegCand];
      score_group(i0, tok_x, prob_x, score_x);
    }
    anchor = block_max_u64(anchor, s.red_u64);   // (its barriers: every thread's wait has ended)
    const int found = s.state;
    if (found & 2) { waited_out = true; break; }
    if (found & 1) { status |= TALON_STATUS_BAD_ROW; break; }   // a row that cannot be normalised: stop here

    // Which of all rows are ready by now?  Thread t asks for row t; the answer arrives under the
    // selection and spares the next layer a round trip in front of its loads.
    int32_t own = 0;
    if (!own_ready && tid < a.ahead_rows) own = load_agent(a.ticket + base + tid);
    const int R = st.N - n;
    const bool init = d < sa.init_layers;
    const int limit = init ? (sa.K_init < R ? sa.K_init : R) : R;
    unsigned long long thr = 1ull;
    if (!init && anchor != 0ull) {
      thr = sortable_u64(sa.log_mu + unsortable_f64(anchor));
      if (thr == 0ull) thr = 1ull;
    }
    const SelectLds lds{s.key, s.hist, s.red_u64, s.red_i32, s.misc};
    int n_keep;
    int pos;
    const unsigned int keep_bits = keep_best(my, per, anchor, thr, limit, lds, &pos, &n_keep);
    auto append = [&](const int tok, const float prob, const double score) __attribute__((always_inline)) {
      const int id = n + pos;
      s.parent[id] = static_cast<unsigned char>(fb + p);
      s.logp[id] = score;
      st.token[base + id] = tok;
      st.parent[base + id] = fb + p;
      st.depth[base + id] = d + 1;
      st.prob[base + id] = prob;
      st.logp[base + id] = score;
      ++pos;
    };
#pragma unroll
    for (int i = 0; i < kRegCand; ++i)
      if (keep_bits & (1u << i)) append(tok_r[i], prob_r[i], score_r[i]);
    for (int i = kRegCand; i < per; ++i) {
      if (!(keep_bits & (1u << i))) continue;
      const unsigned long long key = load_agent(row_keys + rank0 + i);
      const double edge = static_cast<double>(unsortable_f32(static_cast<uint32_t>(key >> 32))) - lse;
      append(static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(key)), __expf(static_cast<float>(edge)), plogp + edge);
    }
    fb = n;
    F = n_keep;
    n += n_keep;
    ++d;
    if (n >= st.N) status |= TALON_STATUS_DONE_BUDGET;
    else if (d >= sa.max_depth) status |= TALON_STATUS_DONE_DEPTH;
    if (status != 0u || F == 0 || d >= a.layers) break;
    own_ready = own_ready || own == kRowReady;
    const unsigned long long ready = __ballot(own_ready);
    if ((tid & 63) == 0) s.ready[tid >> 6] = ready;
    __syncthreads();   // this layer's scores, parents and ready marks are read by the next one
  }
  // ---- the sequence needs no further rows; this workgroup has finished with tickets and counters
  if (tid == 0) {
    store_agent(stop_word(a, b), 1);
    if (ahead_items(a) > static_cast<int>(gridDim.x) - a.B) {   // scanners take items from the counter
      // the last sequence to finish ends the list of items: nobody looks at the remaining ones
      const uint32_t finished = __hip_atomic_fetch_add(a.exit_ticket + kSelectedWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (finished == static_cast<uint32_t>(a.B) - 1u)
        __hip_atomic_fetch_add(item_counter(a), 1u << 30, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    store_agent(st.status + b, waited_out ? (status | TALON_STATUS_ABORTED) : status);   // (the last workgroup may add to it)
  }
  stores_performed();
  __syncthreads();
  exit_ticket(a.exit_ticket, !waited_out);
  const bool bad_row = (status & TALON_STATUS_BAD_ROW) != 0u;
  if (tid == 0) {
    st.n_nodes[b] = n;
    st.frontier_begin[b] = fb;
    st.frontier_count[b] = bad_row ? 0 : F;
    st.depth_cur[b] = d;
  }
  if (waited_out) return;
  // ---- candidate arrays and statistics of the rows that were expanded: rows 0 .. rows-1
  const int rows = bad_row ? fb + F : fb;
  for (int r = tid; r < rows; r += kThreads) {
    const size_t slot = (base + r) * blocks_per_row;
    a.row_max[base + r] = load_agent(a.part_max + slot);
    a.row_lse[base + r] = load_agent(a.part_sum + slot);
  }
  for (int c0 = 0; c0 < rows * k; c0 += 4 * kThreads) {
    unsigned long long kk[4];
    double row_lse[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * kThreads + tid < rows * k ? c0 + u * kThreads + tid : 0;
      const int r = c / k;
      const size_t slot = (base + r) * blocks_per_row;
      kk[u] = load_agent(a.part_keys + slot * k + (c - r * k));
      row_lse[u] = load_agent(a.part_sum + slot);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * kThreads + tid;
      if (c < rows * k) {
        const bool have = kk[u] != 0ull;
        const float lg = have ? key_logit(kk[u]) : kNegInf;
        const double edge = have ? static_cast<double>(lg) - row_lse[u] : -__builtin_huge_val();
        const size_t ci = base * k + c;
        a.cand_token[ci] = have ? static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(kk[u])) : -1;
        a.cand_logit[ci] = lg;
        a.cand_prob[ci] = have ? __expf(static_cast<float>(edge)) : 0.f;
        a.cand_edge_logp[ci] = edge;
      }
    }
  }
  // ---- ancestor mask (Fig. 5(b), App. B): one thread per node walks its parent chain in LDS
  if (a.tree_mask && tid < st.N_pad) {
    uint64_t w[4] = {0, 0, 0, 0};
    int j = tid;
    for (int step = 0; step < TALON_N_MAX && tid < n; ++step) {
      const uint64_t bit = 1ull << (j & 63);
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] |= (j >> 6) == u ? bit : 0ull;
      if (j == 0) break;
      j = s.parent[j];
    }
    const int words = st.N_pad / 64;
    uint64_t* row = a.tree_mask + (base + tid) * words;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < words) row[u] = w[u];
  }
}

template <int EPL>
__global__ __launch_bounds__(kThreads, 4) void build_ahead_kernel(ExpandArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char s_lds[kAheadLds];
  __shared__ int s_go;
  // Exit ticket: taken when everything a workgroup has written to row tickets, stop words and the
  // counter has been performed.  Scanners count in kExitGroups groups whose last arrivals count
  // the group (one word for all would serialise a thousand atomics); selectors, which leave last
  // and whose way out is the launch's tail, count at the top themselves.
  uint32_t before = 0u;
  bool gave_up = false;
  auto exit_ticket = [&](uint32_t* word, bool ok) __attribute__((always_inline)) {
    gave_up = !ok;
    if (threadIdx.x == 0) before = __hip_atomic_fetch_add(word, ok ? 1u : 0x10001u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  const int scanners = static_cast<int>(gridDim.x) - a.B;
  const bool scanner = static_cast<int>(blockIdx.x) < scanners;
  const uint32_t group = blockIdx.x % kExitGroups;
  if (scanner) {
    scan_rows<EPL>(a, *reinterpret_cast<ScannerLds*>(s_lds), blockIdx.x, scanners);
    stores_performed();
    __syncthreads();
    exit_ticket(a.exit_ticket + 1 + group, true);
  } else {
    __builtin_amdgcn_s_setprio(3);   // its instructions are the launch's critical path; the scanners it shares a compute unit with wait for memory anyway
    select_layers(a, *reinterpret_cast<SelectorLds*>(s_lds), static_cast<int>(blockIdx.x) - scanners, exit_ticket);
  }
  // ---- the last workgroup to leave puts row tickets, sequence words and counters back to zero
  if (threadIdx.x == 0) {
    const uint32_t n_groups = scanners < static_cast<int>(kExitGroups) ? scanners : kExitGroups;
    const uint32_t in_group = (scanners - group + kExitGroups - 1) / kExitGroups;
    uint32_t top = before;
    bool counted = !scanner;
    if (scanner && (before & 0xFFFFu) == in_group - 1u) {   // last of its group
      top = __hip_atomic_fetch_add(a.exit_ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      counted = true;
    }
    int go = 0;   // (low 16 bits: arrivals; above: selectors that gave up)
    if (counted && (top & 0xFFFFu) == n_groups + a.B - 1u) go = ((top >> 16) != 0u || gave_up) ? 2 : 1;
    s_go = go;
  }
  __syncthreads();
  if (s_go == 0) return;
  const int t = threadIdx.x;
  for (int i = t; i < a.B * a.N_pad; i += kThreads) store_agent(a.ticket + i, 0);
  for (int i = t; i < a.B; i += kThreads) {
    store_agent(stop_word(a, i), 0);
    if (s_go == 2) atomicOr(&a.status[i], TALON_STATUS_ABORTED);
  }
  for (int i = t; i < kExitWords; i += kThreads) store_agent(a.exit_ticket + i, 0u);
}

}  // namespace

hipError_t launch_build_ahead(const ExpandArgs& a, int dtype, int grid, hipStream_t s) {
  if (dtype == TALON_DTYPE_F32) hipLaunchKernelGGL(build_ahead_kernel<4>, dim3(grid), dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(build_ahead_kernel<8>, dim3(grid), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

int build_ahead_resident(int dtype) {
  int dev = 0, per_cu = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
  const hipError_t e = dtype == TALON_DTYPE_F32
      ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, build_ahead_kernel<4>, kThreads, 0)
      : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, build_ahead_kernel<8>, kThreads, 0);
  if (e != hipSuccess) return 0;
  return per_cu * prop.multiProcessorCount;
}

}  // namespace talon
