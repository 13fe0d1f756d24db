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
//
// The same launch builds trees from the uncapped pool (talon_expand_literal_ahead): scanners rank the 16
// best of every row, and a layer that keeps a row's 16th reads that row once more (see below).  What was three
// launches per layer of the depth cap (or, up to 64 nodes, the capped loop with 32 and more candidates per row), tree
// and mask of resident inputs, before and now: 1 x 128256 bf16, 60 nodes: 72 us, 43;  4 x 151936, 128 nodes,
// two of the sequences flat: 250, 97;  8 x 100003, 100 nodes: 248, 115;  2 x 128256, 250 nodes, flat: 203, 95.
#include "ahead_device.h"
#include "literal_device.h"

namespace talon {

namespace {

// LDS: a workgroup is a scanner or a selector.
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
  // uncapped pool only (want: also whether a row has to be read again)
  int digit, want, nkeep, nfin;
};
// A part of a row read again: every wavefront keeps the keys above the bound in a buffer of its own
// and cuts it to the `limit` best when half of it is full (a step adds at most 512 keys).
constexpr int kPartBuf = 960;
struct PartLds {
  unsigned long long buf[4][kPartBuf];
  int hist[4][256];
  unsigned long long floor[4];
  int count[4];
  int item;
};
constexpr int kAheadLists = 320;   // 255 rows, and up to kDeepParts parts of rows that are read again
static_assert(TALON_N_MAX - 1 + kDeepParts <= kAheadLists, "a list each");
constexpr int kDeepPool = 2048;
struct DeepPickLds {
  PickLds<kDeepPool, kAheadLists> pick;
  double lse[TALON_N_MAX];
  unsigned int src[kAheadLists];   // where a list's keys are: frontier row, or kDeepList + part
  unsigned char par[kAheadLists];
};
constexpr unsigned int kDeepList = 1u << 31;
__device__ __forceinline__ DeepPickLds& deep_lds(SelectorLds& s) { return *reinterpret_cast<DeepPickLds*>(s.key); }
static_assert(sizeof(PartLds) <= sizeof(unsigned long long) * kAheadKeySlots && sizeof(DeepPickLds) <= sizeof(unsigned long long) * kAheadKeySlots,
              "both lie over the key array");
constexpr size_t kAheadLds = sizeof(ScannerLds) > sizeof(SelectorLds) ? sizeof(ScannerLds) : sizeof(SelectorLds);

// ---- uncapped pool: is there anything to expand in sequence b?
__device__ __forceinline__ bool has_frontier(const talon_tree_state& st, int b) {
  const int n = st.n_nodes[b], fb = st.frontier_begin[b], F = st.frontier_count[b];
  return !(st.status[b] & (kDoneMask | TALON_STATUS_BAD_ROW)) && F > 0 && fb >= 0 && fb + F <= n && n < st.N;
}

// ---- uncapped pool: rows that are read again.
// The selection takes the `limit` best of the rows' 16 best.  Where it keeps a row's 16th, tokens beyond
// it may belong to the tree, and exactly those whose path score reaches the lowest one kept (or, with
// budget left, the gate).  That bound turns into one on the row's logits, and the row is streamed
// again, in parts: by helper workgroups, which wait for such work, and by the selector itself, whoever
// claims a part first.  The request lies in the workspace: a header (most and least keys, parts per row) and one word
// per row (node, logit bound); the claim word holds the number of parts and the next one, and storing
// it is the signal.  A part leaves at most `most` keys: as many as let all parts' keys lie in LDS when the selection
// is made again, or all of `limit` where that left out one that could have been chosen.
__device__ __forceinline__ unsigned long long* claim_word(const ExpandArgs& a, int b) {
  return a.desc + a.B + static_cast<size_t>(b) * (a.N_pad - 1) + 16;
}
__device__ __forceinline__ uint32_t* parts_done_word(const ExpandArgs& a, int b) {
  return reinterpret_cast<uint32_t*>(a.desc + a.B + static_cast<size_t>(b) * (a.N_pad - 1) + 32);
}
__device__ __forceinline__ unsigned long long* request_words(const LiteralAhead& la, const ExpandArgs& a, int b) {
  return la.request + static_cast<size_t>(b) * (a.N_pad + 1);
}

// Where a part has left keys out: none of them is above this word (else 0).
__device__ __forceinline__ unsigned long long* part_floor(const LiteralAhead& la, const ExpandArgs& a, int b) {
  return la.request + static_cast<size_t>(a.B) * (a.N_pad + 1) + static_cast<size_t>(b) * kAheadLists;
}

// One wavefront: cuts the n keys in `keys` (LDS, unique) to the best ones, at least `want` and at most `room` of them,
// in place, in any order; returns how many are left and their smallest.  hist: 256 words of LDS of this
// wavefront.  (LDS operations of one wavefront complete in order.)
__device__ __forceinline__ int wave_cut(unsigned long long* keys, const int n, const int want, const int room, int* hist, unsigned long long* smallest) {
  const int lane = threadIdx.x & 63;
  unsigned long long prefix = 0ull;
  if (n > room) {
    int remaining = want;
    for (int sh = 56; sh >= 0; sh -= 8) {
#pragma unroll
      for (int j = 0; j < 4; ++j) hist[4 * lane + j] = 0;
      for (int i = lane; i < n; i += 64) {
        const unsigned long long key = keys[i];
        if (sh == 56 || ((key ^ prefix) >> (sh + 8)) == 0ull) atomicAdd(&hist[static_cast<int>(key >> sh) & 255], 1);
      }
      int h[4], lane_sum = 0;   // lane l owns digits 255-4l .. 252-4l
#pragma unroll
      for (int j = 0; j < 4; ++j) { h[j] = hist[255 - 4 * lane - j]; lane_sum += h[j]; }
      const int incl = wave_inclusive_scan_i32(lane_sum);
      const unsigned long long hit = __ballot(incl >= remaining);
      const int first = hit ? __ffsll(static_cast<long long>(hit)) - 1 : 63;
      int before = incl - lane_sum, dg = 255 - 4 * lane, j = 0;
#pragma unroll
      for (; j < 3; ++j) {
        if (before + h[j] < remaining) { before += h[j]; --dg; } else break;
      }
      const int left = remaining - before;
      const int word = __builtin_amdgcn_readlane(dg | ((h[j] - left <= room - want) ? 256 : 0), first);
      remaining = __builtin_amdgcn_readlane(left, first);
      prefix |= static_cast<unsigned long long>(word & 255) << sh;
      if (word & 256) break;
    }
  }
  int kept = 0;
  unsigned long long inv = 0ull;
  for (int i0 = 0; i0 < n; i0 += 64) {   // (a key moves to a place at or before its own)
    const unsigned long long key = i0 + lane < n ? keys[i0 + lane] : 0ull;
    const bool keep = i0 + lane < n && key >= prefix;
    const unsigned long long bal = __ballot(keep);
    if (keep) {
      keys[kept + __popcll(bal & ((1ull << lane) - 1ull))] = key;
      inv = ~key > inv ? ~key : inv;
    }
    kept += __popcll(bal);
  }
  *smallest = ~wave_max_u64(inv);
  return kept;
}

// Part `item` of sequence b's request.  Starts without and ends with a barrier.
template <int EPL>
__device__ __forceinline__ void read_part(const ExpandArgs& a, const LiteralAhead& la, PartLds& s, const int b, const int item) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned long long* request = request_words(la, a, b);
  const unsigned long long header = load_agent(request);
  const int most = static_cast<int>(header & 0xFFFFu), least = static_cast<int>((header >> 16) & 0xFFFFu), parts = static_cast<int>(header >> 32);
  const int o = item / parts, part = item - o * parts;
  const unsigned long long row_word = load_agent(request + 1 + o);
  const int node = static_cast<int>(row_word >> 32);
  float x_lo = unsortable_f32(static_cast<uint32_t>(row_word));
  const uint4* row = reinterpret_cast<const uint4*>(
      static_cast<const char*>(a.logits) +
      (static_cast<int64_t>(b) * a.seq_stride + static_cast<int64_t>(node) * a.row_stride) * (16 / EPL));
  const int nvec = a.vocab / EPL;   // whole vectors; the tokens behind the last one are the last part's, one by one (see below)
  const int per = (nvec + parts - 1) / parts;
  const int v_end = (part + 1) * per < nvec ? (part + 1) * per : nvec;
  unsigned long long* buf = s.buf[wave];
  int count = 0;
  unsigned long long floor = 0ull;   // where keys above the bound have been left out: the smallest that was not
  unsigned long long smallest;
  // Four vectors of a lane are in flight, each in registers of its own (moved on from one to the next, a vector
  // would be waited for when it is moved).
  auto load = [&](int v) { return v < v_end ? row[v] : make_uint4(0u, 0u, 0u, 0u); };
  auto take = [&](const uint4& r, int v) __attribute__((always_inline)) {
    float x[EPL];
    unpack_vec<EPL>(r, x);
    unsigned int bits = 0u;
    float top = kNegInf;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      if (x[e] >= x_lo && v < v_end) { bits |= 1u << e; top = fmaxf(top, x[e]); }
    }
    const unsigned long long hits = __ballot(bits != 0u);
    if (hits == 0ull) return;
    if (most <= 64 && __popcll(hits) > most + kRaiseHits) {
      // (flat rows) at least `most` lanes hold a logit that reaches the `most`-th of the lanes' largest ones
      const float raised = kth_of_lanes(top, most);
      if (raised > x_lo) {
        x_lo = raised;
        const unsigned long long below = static_cast<unsigned long long>(sortable_u32(x_lo)) << 32;
        floor = below > floor ? below : floor;
        unsigned int keep = 0u;
#pragma unroll
        for (int e = 0; e < EPL; ++e) keep |= x[e] >= x_lo ? 1u << e : 0u;
        bits &= keep;
      }
    }
    const int incl = wave_inclusive_scan_i32(__popc(bits));
    int pos = count + incl - __popc(bits);
#pragma unroll
    for (int e = 0; e < EPL; ++e)
      if (bits & (1u << e)) buf[pos++] = make_key(x[e], v * EPL + e);
    count += __builtin_amdgcn_readlane(incl, 63);
    if (count > kPartBuf - 64 * EPL) {
      count = wave_cut(buf, count, most, 4 * most < kPartBuf - 64 * EPL ? 4 * most : kPartBuf - 64 * EPL, s.hist[wave], &smallest);
      x_lo = float_above(key_logit(smallest));   // a later equal logit has a larger token id and loses
      floor = smallest > floor ? smallest : floor;
    }
  };
  int v = part * per + wave * 64 + lane;
  uint4 r0 = load(v), r1 = load(v + kThreads), r2 = load(v + 2 * kThreads), r3 = load(v + 3 * kThreads);
  for (int v0 = part * per + wave * 64; v0 < v_end; v0 += 4 * kThreads) {
    take(r0, v); r0 = load(v + 4 * kThreads); v += kThreads;
    take(r1, v); r1 = load(v + 4 * kThreads); v += kThreads;
    take(r2, v); r2 = load(v + 4 * kThreads); v += kThreads;
    take(r3, v); r3 = load(v + 4 * kThreads); v += kThreads;
  }
  const bool over = count > 255;
  count = wave_cut(buf, count, most, 255, s.hist[wave], &smallest);
  if (over && smallest > floor) floor = smallest;
  if (lane == 0) { s.count[wave] = count; s.floor[wave] = floor; }
  __syncthreads();
  // the four lists behind one another (each at most 255 keys: up to four per lane), and cut once more
  const int c0 = s.count[0], c1 = s.count[1], c2 = s.count[2], c3 = s.count[3];
  unsigned long long mine[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) mine[j] = 64 * j + lane < count ? buf[64 * j + lane] : 0ull;
  __syncthreads();
  unsigned long long* all = s.buf[0];
  const int at = wave == 0 ? 0 : (wave == 1 ? c0 : (wave == 2 ? c0 + c1 : c0 + c1 + c2));
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (64 * j + lane < count) all[at + 64 * j + lane] = mine[j];
  __syncthreads();
  if (wave == 0) {
    for (int w = 0; w < 4; ++w) floor = s.floor[w] > floor ? s.floor[w] : floor;
    int n_all = c0 + c1 + c2 + c3;
    if (part == parts - 1 && nvec * EPL < a.vocab) {   // fewer than EPL tokens, the last ones of the row: nothing is read beyond them
      const int tok = nvec * EPL + lane;
      float x = kNegInf;
      if (tok < a.vocab) {
        if constexpr (EPL == 4) x = reinterpret_cast<const float*>(row)[tok];
        else x = __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(row)[tok]) << 16);
      }
      const bool in = tok < a.vocab && x >= x_lo;
      const unsigned long long ins = __ballot(in);
      if (in) all[n_all + __popcll(ins & ((1ull << lane) - 1ull))] = make_key(x, tok);
      n_all += __popcll(ins);
    }
    const int n = wave_cut(all, n_all, least, most, s.hist[0], &smallest);
    unsigned long long* out = la.part_key + static_cast<size_t>(b) * la.part_keys_per_seq + static_cast<size_t>(item) * most;
    for (int i = lane; i < n; i += 64) store_agent(out + i, all[i]);
    if (lane == 0) {
      store_agent(la.part_count + static_cast<size_t>(b) * a.N_pad * kLiteralChunks + item, n);
      store_agent(part_floor(la, a, b) + item, n < n_all && smallest > floor ? smallest : floor);
    }
    stores_performed();
    if (lane == 0) __hip_atomic_fetch_add(parts_done_word(a, b), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
}

// ---- helper: parts of any sequence's request, its own number's sequence first, until every selector has
// finished or, with `leave`, until there are none.  (Helpers are the last workgroups of the grid: whoever they wait
// for has started before them.)
template <int EPL>
__device__ __forceinline__ void help_read(const ExpandArgs& a, const LiteralAhead& la, PartLds& s, const int h, const bool leave) {
  const int tid = threadIdx.x;
  while (true) {
    if (tid < 64) {
      int found = -1, item = 0, nb = 0;
      for (int c = 0; c < a.B && found == -1; c += 64) {
        const int bb = (h + c + tid) % a.B;
        unsigned long long w = c + tid < a.B ? load_agent(claim_word(a, bb)) : 0ull;
        const unsigned long long work = __ballot(static_cast<uint32_t>(w) < static_cast<uint32_t>(w >> 32));
        if (work != 0ull) {
          const int first = __ffsll(static_cast<long long>(work)) - 1;
          nb = __builtin_amdgcn_readlane(bb, first);
          if (tid == 0) w = __hip_atomic_fetch_add(claim_word(a, nb), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const uint32_t next = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(w));
          const uint32_t parts = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(w >> 32));
          found = next < parts ? nb : -2;   // (-2: somebody else was faster; look again)
          item = static_cast<int>(next);
        }
      }
      if (found == -1) {
        if (leave || load_agent(a.exit_ticket + kSelectedWord) == static_cast<uint32_t>(a.B)) found = -3;
        else __builtin_amdgcn_s_sleep(16);
      }
      if (tid == 0) { s.item = found >= 0 ? item : found; s.count[0] = nb; }
    }
    __syncthreads();
    const int item = uniform(s.item), b = uniform(s.count[0]);
    __syncthreads();
    if (item == -3) return;
    if (item >= 0) read_part<EPL>(a, la, s, b, item);
  }
}

// The selection of a layer some of whose rows have to be read again (their log-sum-exps in deep_lds, no barrier since):
// `low`, the lowest path score that can still be chosen; kept (in the threads of row p): candidates that the capped pool keeps of the row up to
// this thread's.  Appends the nodes and returns their number, -1 if the wait for parts ran out.
template <int EPL>
__device__ __forceinline__ int deep_select(const ExpandArgs& a, const LiteralAhead& la, SelectorLds& s, const int b, const int F, const int fb,
                                           const int n, const int d, const int limit, double low, const int kept, const int p) {
  const talon_tree_state& st = a.sel.st;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int k = a.k;
  const size_t base = static_cast<size_t>(b) * st.N_pad;
  // candidates kept per row; the rows to read again, in order
  s.hist[tid] = 0;
  __syncthreads();
  if (kept > 0) atomicMax(&s.hist[p], kept);
  __syncthreads();
  const int row_kept = tid < F ? s.hist[tid] : 0;
  const bool open = row_kept == k;
  int n_open;
  const int o = block_exclusive_scan_i32(open ? 1 : 0, s.red_i32, &n_open);
  const int nvec = (a.vocab + EPL - 1) / EPL;
  int parts = la.parts_per_seq / n_open;
  const int by_size = nvec / 512;
  parts = parts < by_size ? parts : by_size;
  parts = parts < 1 ? 1 : (parts > kLiteralChunks ? kLiteralChunks : parts);
  const int n_items = n_open * parts;
  unsigned long long* request = request_words(la, a, b);
  int most = (kDeepPool - TALON_N_MAX) / n_items;   // (at most kDeepParts parts; other rows keep at most 255 in all)
  most = most < 64 ? most : 64;
  most = most < limit ? most : limit;
  int n_keep = 0;
  while (true) {
    if (open) {
      // inside a row the path score rises with the logit: the smallest logit image whose score reaches
      // `low`, by bisection with the very expression the score is computed with
      const double lp = s.logp[fb + tid], lse = deep_lds(s).lse[tid];
      uint32_t l = 0x007FFFFFu, h = 0xFF800000u;   // images of -inf and +inf
      while (l < h) {
        const uint32_t mid = l + ((h - l) >> 1);
        if (lp + (static_cast<double>(unsortable_f32(mid)) - lse) >= low) h = mid; else l = mid + 1u;
      }
      store_agent(request + 1 + o, (static_cast<unsigned long long>(fb + tid) << 32) | l);
    }
    if (tid == 0) {
      const int least = most == limit ? most : most - most / 4;   // (a cut that need not be exact takes half as long)
      store_agent(request, static_cast<unsigned long long>(parts) << 32 | static_cast<unsigned long long>(least << 16 | most));
      store_agent(parts_done_word(a, b), 0u);
    }
    stores_performed();
    __syncthreads();
    if (tid == 0) store_agent(claim_word(a, b), static_cast<unsigned long long>(n_items) << 32);
    PartLds& part = *reinterpret_cast<PartLds*>(s.key);
    // (This barrier keeps thread 0's store apart from thread 0's claim below.  Without it the compiler joined the two
    // conditions, the loop got two entries, and its barriers ran for thread 0 and for the others separately.)
    __syncthreads();
    while (true) {
      if (tid == 0) part.item = static_cast<int>(static_cast<uint32_t>(__hip_atomic_fetch_add(claim_word(a, b), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
      __syncthreads();
      const int item = uniform(part.item);
      __syncthreads();
      if (item >= n_items) break;
      read_part<EPL>(a, la, part, b, item);
    }
    // parts that helpers have claimed (they are being worked on: this wait ends)
    if (tid == 0) {
      const unsigned long long t0 = wall_clock64();
      while (load_agent(parts_done_word(a, b)) != static_cast<uint32_t>(n_items)) {
        if (wall_clock64() - t0 > a.spin_ticks) { s.state |= 2; break; }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __syncthreads();
    if (s.state & 2) return -1;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    // ---- lists of keys: a row's kept candidates, or what its parts left
    DeepPickLds& L = deep_lds(s);
    const int32_t* part_count = la.part_count + static_cast<size_t>(b) * a.N_pad * kLiteralChunks;
    const unsigned long long* floors = part_floor(la, a, b);
    const int own_lists = open ? parts : (row_kept > 0 ? 1 : 0);
    int n_lists;
    const int first_list = block_exclusive_scan_i32(own_lists, s.red_i32, &n_lists);
    if (tid < F) L.lse[tid] = load_agent(a.part_sum + (base + fb + tid) * a.chunks);
    for (int c = 0; c < own_lists; ++c) {
      const int l = first_list + c;
      L.par[l] = static_cast<unsigned char>(tid);
      L.src[l] = open ? kDeepList + static_cast<unsigned int>(o * parts + c) : static_cast<unsigned int>(tid);
      L.pick.cnt[l] = open ? load_agent(part_count + o * parts + c) : row_kept;
    }
    __syncthreads();
    const int l0 = 2 * tid;   // (two lists per thread: up to 320 of them)
    const int n0 = l0 < n_lists ? L.pick.cnt[l0] : 0, n1 = l0 + 1 < n_lists ? L.pick.cnt[l0 + 1] : 0;
    int total;
    const int off = block_exclusive_scan_i32(n0 + n1, s.red_i32, &total);
    if (l0 < n_lists) L.pick.off[l0] = off;
    if (l0 + 1 < n_lists) L.pick.off[l0 + 1] = off + n0;
    if (tid == 0) s.state &= 2;
    __syncthreads();
    const unsigned long long* part_key = la.part_key + static_cast<size_t>(b) * la.part_keys_per_seq;
    n_keep = pick_best<kThreads>(
        n_lists, total, limit, L.pick, s, s.logp + fb, L.lse, [&](int list) { return static_cast<int>(L.par[list]); },
        [&](int list, int i) {
          const unsigned int src = L.src[list];
          const unsigned long long* keys = src & kDeepList ? part_key + static_cast<size_t>(src - kDeepList) * most
                                                           : a.part_keys + (base + fb + src) * a.chunks * k;
          return load_agent(keys + i);
        },
        [&](int rank, int j, unsigned long long key, double edge) {
          const int id = n + rank;
          const double score = s.logp[fb + j] + edge;
          s.logp[id] = score;
          st.token[base + id] = static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(key));
          st.parent[base + id] = fb + j;
          st.depth[base + id] = d + 1;
          st.prob[base + id] = __expf(static_cast<float>(edge));
          st.logp[base + id] = score;
        });
    if (most == limit) break;
    // Could a key that a part has left out have been chosen?
    unsigned long long inv_low = 0ull;   // of the lowest score chosen
    if (tid < n_keep) {
      const int j = L.pick.kj[tid];
      inv_low = ~sortable_u64(s.logp[fb + j] + (static_cast<double>(key_logit(L.pick.kkey[tid])) - L.lse[j]));
    }
    inv_low = block_max_u64(inv_low, s.red_u64);
    bool missed = false;
#pragma unroll
    for (int c = 0; c < kLiteralChunks; ++c) {
      const unsigned long long floor = open && c < parts ? load_agent(floors + o * parts + c) : 0ull;
      if (floor != 0ull)
        missed = missed || n_keep < limit || sortable_u64(s.logp[fb + tid] + (static_cast<double>(key_logit(floor)) - L.lse[tid])) >= ~inv_low;
    }
    if (missed) atomicOr(&s.state, 4);
    __syncthreads();
    if (!(s.state & 4)) break;
    // (the lowest score chosen bounds what can be chosen, closely: this time the parts are short)
    if (n_keep == limit) low = unsortable_f64(~inv_low);
    most = limit;
    __syncthreads();
  }
  return n_keep;
}

// ---- selector: the loop of Alg. 2 for sequence b.
// exit_ticket(ok): takes the workgroup's exit ticket; called when everything other workgroups
// of the launch look at has been performed.
// UNCAPPED: the pool as Alg. 2 writes it, from the tree state as it stands, at most a.layers layers.
template <int EPL, bool UNCAPPED, typename Exit>
__device__ __forceinline__ void select_layers(const ExpandArgs& a, const LiteralAhead& la, SelectorLds& s, const int b, Exit&& exit_ticket) {
  const SelectArgs& sa = a.sel;
  const talon_tree_state& st = sa.st;
  const int tid = threadIdx.x;
  const int k = a.k;
  const size_t base = static_cast<size_t>(b) * st.N_pad;
  const int blocks_per_row = a.chunks;
  int n = 1, fb = 0, F = 1, d = 0;
  uint32_t status = 0u;
  bool waited_out = false, active = true;
  if constexpr (UNCAPPED) {
    status = st.status[b];
    n = st.n_nodes[b];
    fb = st.frontier_begin[b];
    F = st.frontier_count[b];
    d = st.depth_cur[b];
    active = has_frontier(st, b);
    if (active && tid < F) s.logp[fb + tid] = st.logp[base + fb + tid];
    if (tid == 0) s.state = 0;
  } else if (tid == 0) {
    // Alg. 2 line 1: T = {x_t}, p(x_t) = 1
    st.token[base] = a.root_token[b];
    st.parent[base] = -1;
    st.depth[base] = 0;
    st.prob[base] = 1.f;
    st.logp[base] = 0.0;
    s.logp[0] = 0.0;
    s.state = 0;
  }
  const int d_end = UNCAPPED ? d + a.layers : a.layers;
  if (tid < TALON_N_MAX / 64) s.ready[tid] = 0ull;
  bool own_ready = false;   // row `tid` of the sequence is known to be ready
  __syncthreads();
  // Appends have been made: the next layer's frontier, and whether there is one.  (known: row `tid` is known to be ready.)
  auto next_layer = [&](const int n_keep, const bool known) __attribute__((always_inline)) {
    fb = n;
    F = n_keep;
    n += n_keep;
    ++d;
    if (n >= st.N) status |= TALON_STATUS_DONE_BUDGET;
    else if (d >= sa.max_depth) status |= TALON_STATUS_DONE_DEPTH;
    if (status != 0u || F == 0 || d >= d_end) return false;
    const unsigned long long ready = __ballot(known);
    if ((threadIdx.x & 63) == 0) s.ready[threadIdx.x >> 6] = ready;
    __syncthreads();   // this layer's scores, parents and ready marks are read by the next one
    return true;
  };
  // Uncapped pool: a layer some of whose rows have to be read again is finished outside of the loop, and branches are
  // taken on scalars.  With the reading inside, what the loop needs after it was spilled in every layer, read again or not
  // (55 vector registers; four peaked trees of 128 nodes 71.6 us, now 69.4; one of 250 in 13 layers 66.0, 62.2).
  bool again;
  int deep_limit = 0, deep_kept = 0, deep_row = 0;
  double deep_low = 0.0;
  do {
  again = false;
  while (active) {
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
    if (UNCAPPED && tid == 0) s.want = 0;   // (no row has to be read again)
    anchor = block_max_u64(anchor, s.red_u64);   // (its barriers: every thread's wait has ended)
    const int found = uniform(s.state);
    if (found & 2) { waited_out = true; break; }
    if (found & 1) { status |= TALON_STATUS_BAD_ROW; break; }   // a row that cannot be normalised: stop here

    // Which of all rows are ready by now?  Thread t asks for row t; the answer arrives under the
    // selection and spares the next layer a round trip in front of its loads.
    int32_t own = 0;
    if (!own_ready && tid < (UNCAPPED ? st.N - 1 : a.ahead_rows)) own = load_agent(a.ticket + base + tid);
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
    const unsigned int keep_bits = keep_best<!UNCAPPED>(my, per, anchor, thr, limit, lds, &pos, &n_keep);
    n_keep = uniform(n_keep);
    if constexpr (UNCAPPED) {
      // Was a row's last candidate kept?  (Of a single row the `limit` best are its first ones.)
      const int last = k - 1 - rank0;
      if (a.vocab > k && !(F == 1 && n_keep == limit) && last >= 0 && last < per && ((keep_bits >> last) & 1u)) s.want = 1;
      __syncthreads();
      again = uniform(s.want) != 0;
    }
    if (UNCAPPED && again) {
      double low = init || anchor == 0ull ? -__builtin_huge_val() : sa.log_mu + unsortable_f64(anchor);
      // Once it is sure that the budget will be spent no further rows are needed.  How many tokens of a row that is
      // read again pass at least?  Its probabilities add up to one: the k best hold at most k times the best one's, tokens
      // that do not pass less than the bound's each, and what is left is shared by tokens of at most the k-th's.  (0.99:
      // far above the rounding of the three terms, so that a rest of nothing cannot pass for one.)
      int sure = n_keep;
      if (sure < limit && n + limit >= st.N) {
        if (tid == 0) s.nfin = 0;
        if (p < F && rank0 == 0) s.hist[p] = __float_as_int(prob_r[0]);
        __syncthreads();
        const int at = k - 1 - rank0;
#pragma unroll
        for (int i = 0; i < kRegCand; ++i) {
          if (i != at || i >= per || !((keep_bits >> i) & 1u)) continue;
          const float bound = __expf(static_cast<float>(low - plogp));
          const float rest = 0.9f * (0.99f - static_cast<float>(k) * __int_as_float(s.hist[p]) - static_cast<float>(a.vocab) * bound) / prob_r[i];
          if (rest > 0.f) atomicAdd(&s.nfin, rest < 256.f ? static_cast<int>(rest) : 256);
        }
        __syncthreads();
        sure += uniform(s.nfin);
      }
      if (tid == 0 && sure >= limit && n + limit >= st.N) store_agent(stop_word(a, b), 1);
      const int kept_last = 31 - __clz(static_cast<int>(keep_bits));   // a row's kept candidates are its first ones
      if (n_keep == limit) {   // nothing below the lowest score kept can be chosen
        unsigned long long inv_low = 0ull;
        if (keep_bits != 0u) {
          const unsigned long long key = load_agent(row_keys + rank0 + kept_last);
          inv_low = ~sortable_u64(plogp + (static_cast<double>(unsortable_f32(static_cast<uint32_t>(key >> 32))) - lse));
        }
        low = unsortable_f64(~block_max_u64(inv_low, s.red_u64));
      }
      if (p < F && rank0 == 0) deep_lds(s).lse[p] = lse;
      deep_limit = limit;
      deep_low = low;
      deep_kept = keep_bits != 0u ? rank0 + kept_last + 1 : 0;
      deep_row = p;
      break;
    }
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
    own_ready = own_ready || own == kRowReady;
    if (!next_layer(n_keep, own_ready)) break;
  }
  if constexpr (UNCAPPED) {
    if (again) {
      const int n_keep = uniform(deep_select<EPL>(a, la, s, b, F, fb, n, d, deep_limit, deep_low, deep_kept, deep_row));
      own_ready = ((s.ready[threadIdx.x >> 6] >> (threadIdx.x & 63)) & 1ull) != 0ull;
      if (n_keep < 0) waited_out = true;
      if (n_keep < 0 || !next_layer(n_keep, own_ready)) break;
    }
  }
  } while (UNCAPPED && again);
  // ---- the sequence needs no further rows; this workgroup has finished with tickets and counters
  if (tid == 0) {
    store_agent(stop_word(a, b), 1);
    if (UNCAPPED || ahead_items(a) > static_cast<int>(gridDim.x) - a.B) {   // scanners take items from the counter, helpers look at it
      // the last sequence to finish ends the list of items: nobody looks at the remaining ones
      const uint32_t finished = __hip_atomic_fetch_add(a.exit_ticket + kSelectedWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (finished == static_cast<uint32_t>(a.B) - 1u)
        __hip_atomic_fetch_add(item_counter(a), 1u << 30, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!UNCAPPED || active) store_agent(st.status + b, waited_out ? (status | TALON_STATUS_ABORTED) : status);   // (the last workgroup may add to it)
  }
  stores_performed();
  __syncthreads();
  exit_ticket(a.exit_ticket, !waited_out);
  const bool bad_row = (status & TALON_STATUS_BAD_ROW) != 0u;
  if constexpr (UNCAPPED) {
    if (!active) {   // nothing to expand; a row of an earlier layer could not be normalised: the sequence stops here
      if (tid == 0 && bad_row && !(status & kDoneMask) && F > 0) st.frontier_count[b] = 0;
      return;
    }
  }
  if (tid == 0) {
    st.n_nodes[b] = n;
    st.frontier_begin[b] = fb;
    st.frontier_count[b] = bad_row ? 0 : F;
    st.depth_cur[b] = d;
  }
  if (UNCAPPED || waited_out) return;
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

// Workgroups: scanners, then one selector per sequence, then (uncapped pool) helpers, those that wait first.
template <int EPL, bool UNCAPPED>
__device__ __forceinline__ void ahead_body(const ExpandArgs& a, const LiteralAhead& la) {
  __shared__ __attribute__((aligned(16))) unsigned char s_lds[kAheadLds];
  __shared__ int s_go;
  // Exit ticket: taken when everything a workgroup has written to row tickets, stop words and the
  // counter has been performed.  Scanners (and helpers) count in kExitGroups groups whose last arrivals count
  // the group (one word for all would serialise a thousand atomics); selectors, which leave last
  // and whose way out is the launch's tail, count at the top themselves.
  uint32_t before = 0u;
  bool gave_up = false;
  auto exit_ticket = [&](uint32_t* word, bool ok) __attribute__((always_inline)) {
    gave_up = !ok;
    if (threadIdx.x == 0) before = __hip_atomic_fetch_add(word, ok ? 1u : 0x10001u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  const int others = static_cast<int>(gridDim.x) - a.B;                  // scanners and helpers
  const int scanners = UNCAPPED ? others - la.helpers - la.late_helpers : others;
  const int wg = static_cast<int>(blockIdx.x);
  const bool selector = wg >= scanners && wg < scanners + a.B;
  const uint32_t group = (wg < scanners ? wg : wg - a.B) % kExitGroups;
  if (!selector) {
    if (!UNCAPPED || wg < scanners) scan_rows<EPL, UNCAPPED>(a, *reinterpret_cast<ScannerLds*>(s_lds), wg, scanners, la.first_row);
    else help_read<EPL>(a, la, *reinterpret_cast<PartLds*>(s_lds), wg, wg >= scanners + a.B + la.helpers);
    stores_performed();
    __syncthreads();
    exit_ticket(a.exit_ticket + 1 + group, true);
  } else {
    __builtin_amdgcn_s_setprio(3);   // its instructions are the launch's critical path; the scanners it shares a compute unit with wait for memory anyway
    select_layers<EPL, UNCAPPED>(a, la, *reinterpret_cast<SelectorLds*>(s_lds), wg - scanners, exit_ticket);
  }
  // ---- the last workgroup to leave puts row tickets, sequence words and counters back to zero
  if (threadIdx.x == 0) {
    const uint32_t n_groups = others < static_cast<int>(kExitGroups) ? others : kExitGroups;
    const uint32_t in_group = (others - group + kExitGroups - 1) / kExitGroups;
    uint32_t top = before;
    bool counted = selector;
    if (!selector && (before & 0xFFFFu) == in_group - 1u) {   // last of its group
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
    if constexpr (UNCAPPED) {
      store_agent(claim_word(a, i), 0ull);
      store_agent(parts_done_word(a, i), 0u);
      store_agent(la.first_row + i, 0);
    }
    if (s_go == 2) atomicOr(&a.status[i], TALON_STATUS_ABORTED);
  }
  for (int i = t; i < kExitWords; i += kThreads) store_agent(a.exit_ticket + i, 0u);
}

template <int EPL>
__global__ __launch_bounds__(kThreads, 4) void build_ahead_kernel(ExpandArgs a) {
  ahead_body<EPL, false>(a, LiteralAhead{});
}

// The uncapped pool (talon_expand_literal_ahead).
template <int EPL>
__global__ __launch_bounds__(kThreads, 4) void literal_ahead_kernel(ExpandArgs a, LiteralAhead la) {
  ahead_body<EPL, true>(a, la);
}

// In front of it: the counters at zero, and the first row of every sequence that has to be scanned.
__global__ __launch_bounds__(kThreads) void literal_ahead_init_kernel(talon_tree_state st, uint32_t* words, int n_words, int32_t* first_row) {
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n_words; i += gridDim.x * kThreads) {
    const int b = i - static_cast<int>(first_row - reinterpret_cast<int32_t*>(words));
    uint32_t v = 0u;
    if (b >= 0 && b < st.B) {
      v = has_frontier(st, b) ? static_cast<uint32_t>(st.frontier_begin[b]) : static_cast<uint32_t>(st.N);
    }
    words[i] = v;
  }
}

}  // namespace

hipError_t launch_build_ahead(const ExpandArgs& a, int dtype, int grid, hipStream_t s) {
  if (dtype == TALON_DTYPE_F32) hipLaunchKernelGGL(build_ahead_kernel<4>, dim3(grid), dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(build_ahead_kernel<8>, dim3(grid), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_literal_ahead(const ExpandArgs& a, const LiteralAhead& la, int dtype, int grid, void* counters, size_t counter_bytes, hipStream_t s) {
  const int n_words = static_cast<int>(counter_bytes / 4);
  hipLaunchKernelGGL(literal_ahead_init_kernel, dim3((n_words + kThreads - 1) / kThreads), dim3(kThreads), 0, s, a.sel.st,
                     static_cast<uint32_t*>(counters), n_words, la.first_row);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (dtype == TALON_DTYPE_F32) hipLaunchKernelGGL(literal_ahead_kernel<4>, dim3(grid), dim3(kThreads), 0, s, a, la);
  else hipLaunchKernelGGL(literal_ahead_kernel<8>, dim3(grid), dim3(kThreads), 0, s, a, la);
  return hipGetLastError();
}

namespace {
template <typename Kernel>
int resident_workgroups(Kernel* kernel) {
  int dev = 0, per_cu = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, 0) != hipSuccess) return 0;
  return per_cu * prop.multiProcessorCount;
}
}  // namespace

int build_ahead_resident(int dtype) {
  return dtype == TALON_DTYPE_F32 ? resident_workgroups(build_ahead_kernel<4>) : resident_workgroups(build_ahead_kernel<8>);
}

int literal_ahead_resident(int dtype) {
  return dtype == TALON_DTYPE_F32 ? resident_workgroups(literal_ahead_kernel<4>) : resident_workgroups(literal_ahead_kernel<8>);
}

}  // namespace talon
