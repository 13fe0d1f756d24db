// Vocabulary scan: per frontier row, softmax statistics and the k largest logits in one
// pass over the row (candidate pool of Eq. 3 restricted to each parent's k best tokens;
// Alg. 2 "gather" loop).  HBM-bandwidth bound: every logit is read exactly once.
//
// Work decomposition.  A row is a sequence of 16 KiB blocks (8192 bf16 / 4096 f32 logits);
// a block is what one workgroup holds in registers at a time (4 x 16-byte loads per
// thread).  A row is cut into `chunks` runs of consecutive blocks; one (row, chunk) item is
// streamed by one workgroup.  The number of chunks per row is chosen on the device from the total number
// of frontier rows of the launch (few rows: many short chunks, so that a one-row layer
// still spreads over the chip; many rows: one long chunk per row, so that the per-item
// fixed work vanishes).  A fixed-size grid walks the items with a grid stride; nothing
// about the frontier sizes is needed on the host.
//
// Inside a workgroup the four wavefronts stream independently, without barriers:
//   - softmax: every lane keeps its own running max and a double-precision running sum of
//     exp(logit - max), rescaled only when its max grows (rare after the first blocks);
//   - top-k: every wavefront keeps its k best keys so far and a threshold tau.  The first
//     group of 4 tiles sets tau from the 64 per-lane maxima, to a value that at least k of
//     them reach.  A lane whose 16-byte vector holds a logit that
//     reaches tau drops the whole vector into an LDS buffer (a few instructions, no
//     per-logit work); when the buffer runs full, and at the end, the buffered vectors are
//     expanded, ranked against the k best, and tau rises to the new k-th best.  After such
//     a cut a later logit EQUAL to the k-th best cannot enter (the wavefront meets tokens
//     in ascending id order, so it loses the tie): tau becomes the next float above it,
//     and rows full of ties cost nothing extra.
// The workgroup then merges its four lists and statistics.  With one chunk per row it
// writes the row's outputs directly; otherwise it stores a partial result and the
// workgroup that completes the row's last chunk (atomic ticket) merges the partials.
//
// Three ways to run it.  Scan only (talon_expand_layer).  Scan with the budget selection
// (Sec. 5.2, Alg. 2 "Hybrid Expansion Strategy" and "Budget Check") in its tail: the
// workgroup that writes the last row of a sequence's frontier selects for that sequence, one
// launch per layer (talon_expand_select_layer).  Or one launch for the whole loop of Alg. 2
// (talon_expand_tree): the grid walks the layers and enters the next one when all selections
// of the current one are published.
//
// Exactness.  Ordering is by the 64-bit integer key (sortable(logit) << 32 | ~token), so
// the order (logit descending, token ascending) is exact; floating point only enters the
// softmax statistics.
#include "scan_device.h"

// Time-stamp marks exist only in tuning builds (-DTALON_TUNING pulls in tuning.h).
#ifdef TALON_TUNING
#define TALON_TUNING_MARKS
#include "tuning.h"
#else
#define TL_MARK(d, i) do { } while (0)
#define TL_ANY(d, i) do { } while (0)
#endif

namespace talon {

namespace {

// Write the outputs of one row from its candidate keys (in LDS) and softmax statistics.
// `keys` holds `lists` lists of k keys, each sorted in descending order, zero keys in unused
// slots and up to the next multiple of 16.  s_cand: kCandCap + 16 keys of LDS, 16-byte aligned.
// FUSED: the candidates are read by another workgroup of this launch (the one that runs the
// sequence's selection), so they are stored at the device-coherent level.
// Returns whether the row could not be normalised (the same value in every thread).
template <bool FUSED>
__device__ __forceinline__ bool write_row(const ExpandArgs& a, int b, int out_row, const unsigned long long* keys,
                                          int lists, float m, double sum, unsigned long long* s_cand, int* s_nc) {
  // (thread index taken afresh, through an empty asm statement: addresses derived from it are
  // then computed here, at their use, instead of being kept alive or spilled across the
  // caller's streaming loop)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int k = a.k;
  const double lse = static_cast<double>(m) + log_of_sum(sum);
  const size_t ob = static_cast<size_t>(out_row) * k;
  auto emit = [&](unsigned long long ki, int r) {
    const float lg = key_logit(ki);
    const double edge = static_cast<double>(lg) - lse;
    const int32_t tok = static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(ki));
    const float pr = __expf(static_cast<float>(edge));
    a.cand_logit[ob + r] = lg;
    if constexpr (FUSED) {
      store_agent(a.cand_token + ob + r, tok);
      store_agent(a.cand_edge_logp + ob + r, edge);
      store_agent(a.cand_prob + ob + r, pr);
    } else {
      a.cand_token[ob + r] = tok;
      a.cand_edge_logp[ob + r] = edge;
      a.cand_prob[ob + r] = pr;
    }
  };
  rank_lists(k, keys, lists, tid, s_cand, s_nc, emit);
  const int valid = a.vocab < k ? a.vocab : k;
  if (tid >= valid && tid < k) {
    a.cand_logit[ob + tid] = kNegInf;
    if constexpr (FUSED) {
      store_agent(a.cand_token + ob + tid, -1);
      store_agent(a.cand_edge_logp + ob + tid, -__builtin_huge_val());
      store_agent(a.cand_prob + ob + tid, 0.f);
    } else {
      a.cand_token[ob + tid] = -1;
      a.cand_edge_logp[ob + tid] = -__builtin_huge_val();
      a.cand_prob[ob + tid] = 0.f;
    }
  }
  const bool bad = !(fabs(lse) <= 1.7e308);
  if (tid == 0) {
    a.row_max[out_row] = m;
    a.row_lse[out_row] = lse;
    if (bad) atomicOr(&a.status[b], TALON_STATUS_BAD_ROW);
  }
  return bad;
}

// How a launch is used: scan only; scan with the selection in its tail (one layer per launch);
// or one launch that walks all layers.
constexpr int kModeSplit = 0, kModeFused = 1, kModeTree = 2;

// Launches of one layer: workgroups that have read the frontier, counted in kStartedWords words spread
// evenly over the descriptors of layers >= 1 (which these launches do not use and every launch leaves
// zero): on memory lines of their own from B * (N_pad - 1) = 128 descriptors on, two or three to a
// line for one sequence of 64 nodes.  An atomic on one word takes about 20 ns: 900 workgroups on a
// single counter kept a selection waiting for 18 us, longer than the layer's scan.
constexpr int kStartedWords = 8;
__device__ __forceinline__ uint32_t* started_word(const ExpandArgs& a, int x) {
  return reinterpret_cast<uint32_t*>(a.desc + a.B + static_cast<size_t>(x) * (a.B * (a.N_pad - 1) / kStartedWords));
}

// One layer: returns the number of frontier rows it found (0: every sequence is finished).
template <int EPL, int MODE>
__device__ __forceinline__ int expand_body(const ExpandArgs& a, const int launch_idx) {
  constexpr bool FUSED = MODE != kModeSplit;
  constexpr bool TREE = MODE == kModeTree;
  __shared__ int s_prefix[TALON_B_MAX + 1];     // exclusive prefix of frontier sizes
  __shared__ int s_begin[TALON_B_MAX];          // first frontier node of every sequence
  __shared__ uint32_t s_stat[FUSED && !TREE ? TALON_B_MAX : 1];   // its status when the launch began
  // One LDS pool: the scan's buffers (buffered vectors per wavefront, their tile*64+lane tags,
  // ranking scratch per wavefront; the vector buffers double as row-merge staging) and, in
  // fused mode, the key array and histogram of the budget selection, which runs when the
  // scan buffers are idle.
  constexpr int kSelBytes = sizeof(unsigned long long) * kSelectKeySlots + sizeof(int) * 256;
  constexpr int kPoolBytes = (FUSED && kSelBytes > kScanBytes) ? kSelBytes : kScanBytes;
  __shared__ __attribute__((aligned(16))) unsigned char s_pool[kPoolBytes];
  __shared__ unsigned long long s_red_u64[8];
  __shared__ int s_misc[2];
  __shared__ __attribute__((aligned(16))) unsigned long long s_topw[4][TALON_K_MAX]; // k best keys of each wavefront, sorted
  __shared__ unsigned long long s_top[TALON_K_MAX];
  __shared__ int s_red_i32[8];
  __shared__ float s_wmax[4];
  __shared__ double s_wsum[4];
  __shared__ int s_wcnt[4];
  __shared__ int s_last;
  static_assert(kScanBytes >= static_cast<int>(sizeof(unsigned long long)) * kMergeCap,
                "the scan buffers double as the row-merge staging array");
  static_assert(kScanBytes >= static_cast<int>(sizeof(unsigned long long)) * (kMergeCap + kCandCap + 16),
                "... and hold the filtered candidates of a row merge behind it");
  unsigned long long* s_keys = reinterpret_cast<unsigned long long*>(s_pool);
  unsigned long long* s_cand = s_keys + kMergeCap;
  __shared__ int s_nc;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;

  // ---- frontier sizes of all sequences -> item map (identical in every workgroup)
  __shared__ int s_gave_up;
  {
    static_assert(TALON_B_MAX <= kThreads, "one thread per sequence");
    if (TREE && tid == 0) s_gave_up = 0;
    if constexpr (TREE) __syncthreads();
    int c = 0;
    if (tid < a.B) {
      if (TREE && a.root_token && launch_idx == 0) {   // fresh trees: the frontier is the root
        s_begin[tid] = 0;
        c = 1;
      } else if constexpr (TREE) {   // {begin, count} in one 8-byte load
        const unsigned long long* dp = a.desc + (launch_idx * a.B + tid);
        unsigned long long d2 = ld<TREE, unsigned long long>(dp);
        if constexpr (TREE) {
          // the selection of the layer before stores this word when all it wrote has been
          // performed: wait for it (bounded)
          if (!(d2 & kDescReady)) {
            const unsigned long long t0 = wall_clock64();
            do {
              if (wall_clock64() - t0 > a.spin_ticks) { s_gave_up = 1; break; }
              __builtin_amdgcn_s_sleep(2);
              d2 = ld<true, unsigned long long>(dp);
            } while (!(d2 & kDescReady));
          }
        }
        s_begin[tid] = static_cast<int>(static_cast<uint32_t>(d2));
        c = static_cast<int>(static_cast<uint32_t>(d2 >> 32) & 0x7FFFFFFFu);
      } else {  // the loads are issued together; the select below is register-only
        // (In a launch of one layer with the selection in its tail, that selection rewrites this
        // state while workgroups of the same launch may still be starting, and every workgroup
        // must see the same item map: a workgroup says below that it has read the state, and a
        // selection touches nothing before every workgroup of the grid has said so.)
        const uint32_t stat = a.status[tid];
        const int fc = a.frontier_count[tid];
        s_begin[tid] = a.frontier_begin[tid];
        if constexpr (FUSED) s_stat[tid] = stat;
        c = (stat & kDoneMask) ? 0 : fc;
      }
      // a finished sequence gets no selection in this launch: carry its empty frontier over
      if (TREE && blockIdx.x == 0 && c == 0 && launch_idx + 1 < a.N_pad)
        st_<true, unsigned long long>(a.desc + ((launch_idx + 1) * a.B + tid),
                                      kDescReady | static_cast<unsigned long long>(static_cast<uint32_t>(s_begin[tid])));
    }
    int total;
    const int base = block_exclusive_scan_i32(c, s_red_i32, &total);
    if (tid < a.B) s_prefix[tid] = base;
    if (tid == 0) s_prefix[a.B] = total;
    __syncthreads();
    if constexpr (TREE) {
      if (s_gave_up) return -1;
    }
  }
  const int total_rows = s_prefix[a.B];
  if (total_rows == 0) return 0;   // (nothing will be selected in this launch: nobody waits for anybody)
  if constexpr (FUSED && !TREE) {
    // this workgroup has read the frontier (the loads fed the prefix sums that thread 0 has
    // waited for at the barrier above)
    if (tid == 0) __hip_atomic_fetch_add(started_word(a, blockIdx.x % kStartedWords), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int k = a.k;

  // ---- chunks per row from the width of this layer
  const int blocks_per_row = a.chunks;
  int chunks = (a.target_items + total_rows - 1) / total_rows;
  {   // ... and at least as many as give every workgroup of the grid an item in the first round
    const int fill = static_cast<int>(gridDim.x) / total_rows;
    chunks = fill > chunks ? fill : chunks;
  }
  chunks = chunks < 1 ? 1 : (chunks > blocks_per_row ? blocks_per_row : chunks);
  const int bpc = (blocks_per_row + chunks - 1) / chunks;   // blocks per chunk
  chunks = (blocks_per_row + bpc - 1) / bpc;
  const long long n_items = static_cast<long long>(total_rows) * chunks;
  const ScanLds L{reinterpret_cast<uint4 (*)[kHitCap]>(s_pool), reinterpret_cast<int (*)[kHitCap]>(s_pool + kHitvBytes),
                  reinterpret_cast<unsigned long long (*)[kSubKeys]>(s_pool + kHitvBytes + kHithBytes), s_topw, s_top,
                  s_wmax, s_wsum, s_wcnt};

  for (long long item = blockIdx.x; item < n_items; item += gridDim.x) {
    const int rg = static_cast<int>(item / chunks);
    const int ch = static_cast<int>(item - static_cast<long long>(rg) * chunks);
    int lo = 0, hi = a.B;  // largest b with s_prefix[b] <= rg
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_prefix[mid] <= rg) lo = mid; else hi = mid;
    }
    // (scalars in the launch over all layers: the row's addresses as vectors made it spill.  The launches of one layer have
    // the registers, and were 1 % slower with scalars.)
    const auto scalar = [](int v) { return TREE ? uniform(v) : v; };
    const int b = scalar(lo);
    const int local = rg - scalar(s_prefix[b]);
    const int fbegin = scalar(s_begin[b]);
    const int node = fbegin + local;
    const int in_row = a.row_mode == TALON_ROWS_BY_FRONTIER ? local : node;
    const char* row = static_cast<const char*>(a.logits) +
                      (static_cast<int64_t>(b) * a.seq_stride + static_cast<int64_t>(in_row) * a.row_stride) * (16 / EPL);
    const int out_row = b * a.N_pad + node;
    const int blk0 = ch * bpc;
    const int blk1 = blk0 + bpc < blocks_per_row ? blk0 + bpc : blocks_per_row;

    float cm;      // the run's maximum and sum of exp(logit - maximum)
    double csum;
    scan_chunk<EPL, FUSED, false>(row, a.vocab, k, blk0, blk1, L, cm, csum);

    bool row_written = false;   // this workgroup has just written a whole row's outputs
    bool row_bad = false;       // ... and the row could not be normalised
    // Alg. 2 line 1 inside the single launch: T = {x_t}, p(x_t) = 1, d = 0.  The workgroup that
    // writes the root's row (and then runs the sequence's first selection) sets the state up.
    auto start_tree = [&]() {
      if constexpr (TREE) {
        if (a.root_token && launch_idx == 0) {
          if (tid == 0) {
            const talon_tree_state& st = a.sel.st;
            const size_t o = static_cast<size_t>(b) * st.N_pad;
            store_agent(st.token + o, a.root_token[b]);
            store_agent(st.parent + o, -1);
            store_agent(st.depth + o, 0);
            store_agent(st.prob + o, 1.f);
            store_agent(st.logp + o, 0.0);
            store_agent(st.n_nodes + b, 1);
            store_agent(st.frontier_begin + b, 0);
            store_agent(st.frontier_count + b, 1);
            store_agent(st.depth_cur + b, 0);
            store_agent(st.status + b, 0u);
          }
          __syncthreads();
        }
      }
    };
    if (chunks == 1) {
      start_tree();
      row_bad = write_row<FUSED>(a, b, out_row, s_top, 1, cm, csum, s_cand, &s_nc);
      row_written = true;
    } else {
      unsigned long long* pk = a.part_keys + (static_cast<size_t>(out_row) * blocks_per_row + ch) * k;
      if (tid < k) store_agent(pk + tid, s_top[tid]);
      if (tid == 0) {
        store_agent(a.part_max + static_cast<size_t>(out_row) * blocks_per_row + ch, cm);
        store_agent(a.part_sum + static_cast<size_t>(out_row) * blocks_per_row + ch, csum);
      }
      // every partial store of this workgroup has completed before the ticket is taken
      stores_performed();
      __syncthreads();
      if (tid == 0) {
        const int old = __hip_atomic_fetch_add(&a.ticket[out_row], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = (old == chunks - 1) ? 1 : 0;
      }
      __syncthreads();
      if (s_last) {
        const float* pm = a.part_max + static_cast<size_t>(out_row) * blocks_per_row;
        const double* ps = a.part_sum + static_cast<size_t>(out_row) * blocks_per_row;
        const unsigned long long* keys = a.part_keys + static_cast<size_t>(out_row) * blocks_per_row * k;
        const int nkeys = chunks * k;
        const int nkeys_pad = (nkeys + 15) & ~15;   // zero keys rank below every real key
        // softmax statistics of the row: every wavefront merges the chunk statistics on its own
        // (one chunk per lane, more only for very long rows), so that no workgroup-wide
        // reduction is needed.  All loads of the first sweep are issued before any is used.
        float mc0 = kNegInf;
        double sc0 = 0.0;
        if (lane < chunks) { mc0 = load_agent(pm + lane); sc0 = load_agent(ps + lane); }
        const unsigned long long key0 = tid < nkeys ? load_agent(keys + tid) : 0ull;
        if (tid < nkeys_pad) s_keys[tid] = key0;
        for (int i = tid + kThreads; i < nkeys_pad; i += kThreads) s_keys[i] = i < nkeys ? load_agent(keys + i) : 0ull;
        float m = mc0;
        for (int c = lane + 64; c < chunks; c += 64) m = fmaxf(m, load_agent(pm + c));
        m = wave_max_f32(m);
        double sum = rescaled_sum(sc0, mc0, m);
        for (int c = lane + 64; c < chunks; c += 64) sum += rescaled_sum(load_agent(ps + c), load_agent(pm + c), m);
        sum = wave_sum_f64(sum);
        __syncthreads();   // s_keys is staged
        start_tree();
        row_bad = write_row<FUSED>(a, b, out_row, s_keys, chunks, m, sum, s_cand, &s_nc);
        if (tid == 0) store_agent(a.ticket + out_row, 0);  // leave the workspace clean for the next layer
        row_written = true;
      }
    }
    if constexpr (FUSED) {
      if (row_written) {
        // ---- sequence ticket: the workgroup that writes the last row of a sequence's frontier
        // runs that sequence's budget selection
        const int F = s_prefix[b + 1] - s_prefix[b];
        if (F > 1) {
          stores_performed();
          __syncthreads();
          if (tid == 0) {
            // low 16 bits: rows written; above: how many of them could not be normalised
            const int old = __hip_atomic_fetch_add(&a.seq_ticket[b], row_bad ? 0x10001 : 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool last = (old & 0xFFFF) == F - 1;
            s_last = last ? ((old >> 16) != 0 || row_bad ? 2 : 1) : 0;
            if (last) store_agent(a.seq_ticket + b, 0);
          }
        } else {
          stores_performed();   // the selection reads the row's candidates back from global memory
          if (tid == 0) s_last = row_bad ? 2 : 1;   // a one-row frontier: the workgroup that wrote the row selects right away
        }
        __syncthreads();
        if (s_last) {
          TL_ANY(launch_idx, 2);
          // One layer per launch: the selection rewrites the state the item map is made from, so it
          // writes nothing before every workgroup of the grid has read it (workgroups that have not
          // started yet start as others leave; only the at most B selecting workgroups wait, so the
          // others always get their turn).  The wait is bounded like the single launch's: a
          // workgroup that gives up marks the sequence aborted and selects nothing.
          // A selection's time is its chain of memory round trips.  The counters
          // are read here, so that they arrive with the candidates, and looked at before the first
          // write; the status is the one read when the launch began (this launch itself can only
          // have added a bad row, which the ticket tells); and which selection is the launch's last
          // is asked before the writes, and only where there are several.  (Each in its own turn, with
          // the counters awaited before the selection began: 70.5 us for 12 layers of one sequence of 60
          // nodes, three of them with rows; this: 68.4, and 65.9 with a grid that is resident at once.)
          int started = 0;
          uint32_t selected_before = 0u;
          int active = 1;
          bool gave_up = false;
          auto read_started = [&]() { return lane < kStartedWords ? static_cast<int>(load_agent(started_word(a, lane))) : 0; };
          if constexpr (!TREE) {
            if (wave == 0) started = read_started();
          }
          auto all_started = [&]() -> bool {
            if constexpr (TREE) return true;
            if (wave == 0) {
              const unsigned long long t0 = wall_clock64();
              bool all = true;
              while (wave_sum_i32(started) != static_cast<int>(gridDim.x)) {
                if (wall_clock64() - t0 > a.spin_ticks) { all = false; break; }
                __builtin_amdgcn_s_sleep(2);
                started = read_started();
              }
              if (a.B > 1) {   // which selection of the launch is the last to come by here
                active = 0;
                for (int q = lane; q < a.B; q += 64) active += s_prefix[q + 1] > s_prefix[q] ? 1 : 0;
                active = wave_sum_i32(active);
                if (lane == 0) selected_before = __hip_atomic_fetch_add(a.exit_ticket + kSelectedWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
              if (lane == 0) s_misc[0] = all ? 0 : 1;
            }
            __syncthreads();
            gave_up = s_misc[0] != 0;
            return !gave_up;
          };
          // A launch that started the tree itself knows the sequence's status (nothing but a
          // row that cannot be normalised can have touched it), its size and its layer
          // without asking memory.
          const bool own = TREE && a.root_token != nullptr;
          uint32_t status;
          if constexpr (TREE) {
            status = own ? (s_last == 2 ? static_cast<uint32_t>(TALON_STATUS_BAD_ROW) : 0u)
                         : __hip_atomic_load(&a.status[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          } else {
            status = s_stat[b] | (s_last == 2 ? static_cast<uint32_t>(TALON_STATUS_BAD_ROW) : 0u);
          }
          unsigned long long next = static_cast<unsigned long long>(static_cast<uint32_t>(fbegin));   // count 0
          if (status & TALON_STATUS_BAD_ROW) {   // a row could not be normalised: stop the sequence here
            if (all_started() && tid == 0) st_<TREE, int32_t>(a.sel.st.frontier_count + b, 0);
          } else {
            const SelectLds lds{reinterpret_cast<unsigned long long*>(s_pool),
                                reinterpret_cast<int*>(s_pool + sizeof(unsigned long long) * kSelectKeySlots),
                                s_red_u64, s_red_i32, s_misc};
            next = select_sequence<true>(a.sel, b, F, fbegin, status, lds, own ? fbegin + F : -1,
                                         own ? launch_idx : -1, all_started);
          }
          if constexpr (TREE) {
            // everything this layer wrote for the sequence has been performed before the
            // descriptor that lets the grid into the next layer is stored
            stores_performed();
            __syncthreads();
            if (tid == 0 && launch_idx + 1 < a.N_pad)
              st_<true, unsigned long long>(a.desc + ((launch_idx + 1) * a.B + b), next | kDescReady);
            TL_ANY(launch_idx, 3);
          } else {   // (a launch of one layer leaves no descriptor: the next call starts from the public state)
            if (tid == 0) {
              if (gave_up) atomicOr(&a.status[b], static_cast<uint32_t>(TALON_STATUS_ABORTED));
              // the last selection of the launch puts the counters back to zero (every workgroup has
              // started by now and every selection has seen it, so nobody counts or looks after this;
              // unless a wait has run out: workgroups that start later count themselves in words that
              // stay so, which is why the workspace has to be initialised again then)
              if (static_cast<int>(selected_before) + 1 == active) {
                for (int x = 0; x < kStartedWords; ++x) store_agent(started_word(a, x), 0u);
                if (a.B > 1) store_agent(a.exit_ticket + kSelectedWord, 0u);
              }
            }
          }
        }
      }
    }
    __syncthreads();  // s_keys / s_top / s_w* are reused by the next item
  }
  return total_rows;
}

// With the selection in its tail the kernel needs about 160 vector registers: three
// workgroups per compute unit instead of four, rather than spilling.
template <int EPL, int MODE>
__global__ __launch_bounds__(kThreads, MODE == kModeSplit ? 4 : 3) void expand_kernel(ExpandArgs a) {
  static_assert(MODE != kModeTree, "the single-launch loop has its own kernel");
  expand_body<EPL, MODE>(a, a.launch_idx);
}

// All layers in one launch.  The grid must be resident as a whole (the host sizes it from the
// occupancy of this kernel): a workgroup waits, between two layers, for the selections of the
// layer it has just left, which other workgroups run.  The wait is bounded; a workgroup that
// gives up marks every sequence TALON_STATUS_ABORTED and leaves, and so do all others.
template <int EPL>
__global__ __launch_bounds__(kThreads, 3) void expand_tree_kernel(ExpandArgs a) {
  __shared__ int s_go;
  // a launch that is only wanted when an earlier one of the same call has raised its flag
  if (a.run_if && load_agent(a.run_if) == 0u) return;
  bool gave_up = false;
  // One pass more than there are layers: the pass after the last layer finds every sequence
  // finished (depth cap or budget), which is also the proof that every selection is
  // published.  A pass starts by waiting for the descriptors of its layer.
  int d = 0;
  for (; d <= a.layers; ++d) {
    TL_MARK(d, 0);
    const int rows = expand_body<EPL, kModeTree>(a, d);
    TL_MARK(d, 1);
    if (rows < 0) {   // the wait for a descriptor ran out
      for (int b = threadIdx.x; b < a.B; b += kThreads) atomicOr(&a.status[b], TALON_STATUS_ABORTED);
      gave_up = true;
      break;
    }
    if (rows == 0) break;   // uniform over the grid: every workgroup reads the same descriptors
  }
  TL_MARK(31, 0);
  // ---- exit ticket: this workgroup has finished with the tickets and layer counters (all its
  // own updates of them have completed).  The answer is needed only after the masks.
  stores_performed();
  __syncthreads();
  // Two levels: workgroup i counts in group i % kExitGroups; the last of a group counts the
  // group.  Low 16 bits: arrivals; above: how many of them gave up.
  const uint32_t group = blockIdx.x % kExitGroups;
  const uint32_t group_size = (gridDim.x - group + kExitGroups - 1) / kExitGroups;
  const uint32_t n_groups = gridDim.x < kExitGroups ? gridDim.x : kExitGroups;
  uint32_t left_before = 0u;
  if (threadIdx.x == 0)
    left_before = __hip_atomic_fetch_add(a.exit_ticket + 1 + group, gave_up ? 0x10001u : 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // ---- ancestor masks (Fig. 5(b), App. B): every selection of every layer is published by
  // now.  Bit j of row i is set iff j is i or an ancestor of i; one thread per node walks its
  // parent chain in LDS.
  __shared__ int s_par[TALON_N_MAX];
  const talon_tree_state& st = a.sel.st;
  const int words = st.N_pad / 64;
  for (int b = blockIdx.x; a.tree_mask && !gave_up && b < a.B; b += gridDim.x) {
    const int tid = threadIdx.x;
    const int n = load_agent(st.n_nodes + b);
    const size_t base = static_cast<size_t>(b) * st.N_pad;
    __syncthreads();
    if (tid < st.N_pad) s_par[tid] = tid < n ? load_agent(st.parent + base + tid) : -1;
    __syncthreads();
    if (tid < st.N_pad) {
      uint64_t w[4] = {0, 0, 0, 0};
      if (tid < n) {
        int j = tid;
        for (int step = 0; step < TALON_N_MAX && j >= 0; ++step) {
          const uint64_t bit = 1ull << (j & 63);
          const int q = j >> 6;
#pragma unroll
          for (int u = 0; u < 4; ++u) w[u] |= q == u ? bit : 0ull;
          j = s_par[j];
        }
      }
      uint64_t* row = a.tree_mask + (base + tid) * words;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (u < words) row[u] = w[u];
    }
  }
  TL_MARK(31, 1);
  // ---- the last workgroup to leave puts the counters back to zero for the next launch; if
  // any workgroup gave up, tickets may be half taken: clear them all, and mark every sequence
  // (a tree started late in the launch may have overwritten the mark)
  if (threadIdx.x == 0) {
    int go = 0;
    if ((left_before & 0xFFFFu) == group_size - 1u) {   // last of its group
      const bool bad = (left_before >> 16) != 0u || gave_up;
      const uint32_t groups_before = __hip_atomic_fetch_add(a.exit_ticket, bad ? 0x10001u : 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((groups_before & 0xFFFFu) == n_groups - 1u) go = ((groups_before >> 16) != 0u || bad) ? 2 : 1;
    }
    s_go = go;
  }
  __syncthreads();
  if (s_go == 0) return;
  const int t = threadIdx.x;
  // descriptors of the layers this launch has written (all of them if a workgroup gave up)
  const int used = s_go == 2 ? a.N_pad - 1 : (d + 1 < a.N_pad ? d + 1 : a.N_pad - 1);
  for (int i = t; i < used * a.B; i += kThreads) store_agent(a.desc + a.B + i, 0ull);
  if (s_go == 2) {
    for (int i = t; i < a.B * a.N_pad; i += kThreads) store_agent(a.ticket + i, 0);
    for (int i = t; i < a.B; i += kThreads) {
      store_agent(a.seq_ticket + i, 0);
      atomicOr(&a.status[i], TALON_STATUS_ABORTED);
    }
  }
  for (int i = t; i < kExitWords; i += kThreads) store_agent(a.exit_ticket + i, 0u);
}

__global__ __launch_bounds__(kThreads) void fill_zero_kernel(uint32_t* p, size_t n) {
  for (size_t i = blockIdx.x * static_cast<size_t>(kThreads) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * kThreads)
    p[i] = 0u;
}

__global__ __launch_bounds__(kThreads) void tree_init_kernel(talon_tree_state st, const int32_t* root_token) {
  const int b = blockIdx.x * kThreads + threadIdx.x;
  if (b >= st.B) return;
  const size_t o = static_cast<size_t>(b) * st.N_pad;
  st.token[o] = root_token[b];
  st.parent[o] = -1;
  st.depth[o] = 0;
  st.prob[o] = 1.f;
  st.logp[o] = 0.0;
  st.n_nodes[b] = 1;
  st.frontier_begin[b] = 0;
  st.frontier_count[b] = 1;
  st.depth_cur[b] = 0;
  st.status[b] = st.N <= 1 ? TALON_STATUS_DONE_BUDGET : 0u;
}

}  // namespace

int expand_chunk_elems(int dtype) { return dtype == TALON_DTYPE_F32 ? kChunkBytes / 4 : kChunkBytes / 2; }

// Start of a fused call that continues trees already begun: frontier descriptors of its first
// layer from the public tree state, none for the later layers; zero tickets (nothing leaves
// them taken, but a caller may hand over a workspace that other launch forms have used).
__global__ void fused_init_kernel(talon_tree_state st, unsigned long long* desc, int32_t* ticket, int32_t* seq_ticket,
                                  FusedInitArgs f) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (f.mode == kInitRestoreIf && *f.flag == 0u) return;
  if (f.mode == kInitSave && f.clear && i <= kExitWords) f.clear[i] = 0u;   // (the grid has at least 256 threads)
  if (i >= st.B * st.N_pad) return;
  ticket[i] = 0;
  if (i >= st.B) { desc[i] = 0ull; return; }
  seq_ticket[i] = 0;
  if (f.mode == kInitSave) {
    f.saved[i] = st.n_nodes[i];
    f.saved[st.B + i] = st.frontier_begin[i];
    f.saved[2 * st.B + i] = st.frontier_count[i];
    f.saved[3 * st.B + i] = st.depth_cur[i];
    f.saved[4 * st.B + i] = static_cast<int32_t>(st.status[i]);
  } else if (f.mode == kInitRestoreIf) {
    st.n_nodes[i] = f.saved[i];
    st.frontier_begin[i] = f.saved[st.B + i];
    st.frontier_count[i] = f.saved[2 * st.B + i];
    st.depth_cur[i] = f.saved[3 * st.B + i];
    st.status[i] = static_cast<uint32_t>(f.saved[4 * st.B + i]);
  }
  const uint32_t count = (st.status[i] & kDoneMask) ? 0u : static_cast<uint32_t>(st.frontier_count[i]);
  desc[i] = kDescReady | (static_cast<unsigned long long>(count) << 32) | static_cast<uint32_t>(st.frontier_begin[i]);
}

hipError_t launch_fused_init(const talon_tree_state& st, const ExpandArgs& a, const FusedInitArgs& f, hipStream_t s) {
  const int n = st.B * st.N_pad;
  hipLaunchKernelGGL(fused_init_kernel, dim3((n + 255) / 256), dim3(256), 0, s, st, a.desc, a.ticket, a.seq_ticket, f);
  return hipGetLastError();
}

hipError_t launch_expand_tree(const ExpandArgs& a, int dtype, int grid, hipStream_t s) {
  if (dtype == TALON_DTYPE_F32) hipLaunchKernelGGL(expand_tree_kernel<4>, dim3(grid), dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(expand_tree_kernel<8>, dim3(grid), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

// Workgroups of the single-launch kernel that the current device holds at once.
int expand_tree_max_grid(int dtype) {
  int dev = 0, per_cu = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
  const hipError_t e = dtype == TALON_DTYPE_F32
      ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, expand_tree_kernel<4>, kThreads, 0)
      : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, expand_tree_kernel<8>, kThreads, 0);
  if (e != hipSuccess) return 0;
  return per_cu * prop.multiProcessorCount;
}

hipError_t launch_expand(const ExpandArgs& a, int dtype, int grid, bool fused, hipStream_t s) {
  if (dtype == TALON_DTYPE_F32) {
    if (fused) hipLaunchKernelGGL((expand_kernel<4, kModeFused>), dim3(grid), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL((expand_kernel<4, kModeSplit>), dim3(grid), dim3(kThreads), 0, s, a);
  } else {
    if (fused) hipLaunchKernelGGL((expand_kernel<8, kModeFused>), dim3(grid), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL((expand_kernel<8, kModeSplit>), dim3(grid), dim3(kThreads), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 4;
  int grid = static_cast<int>((n + kThreads - 1) / kThreads);
  if (grid > 1024) grid = 1024;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(kThreads), 0, s, static_cast<uint32_t*>(p), n);
  return hipGetLastError();
}

hipError_t launch_tree_init(const talon_tree_state& st, const int32_t* root_token, hipStream_t s) {
  hipLaunchKernelGGL(tree_init_kernel, dim3((st.B + kThreads - 1) / kThreads), dim3(kThreads), 0, s, st,
                     root_token);
  return hipGetLastError();
}

}  // namespace talon
