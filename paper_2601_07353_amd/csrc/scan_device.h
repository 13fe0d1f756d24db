// One pass over a run of a logits row: softmax statistics and the k largest logits, by one
// workgroup of 256 threads.  Shared by the kernels that scan a layer's frontier (expand.hip) and
// the kernel that scans rows ahead of the tree (ahead.hip); what the streaming does and why is
// described at the top of expand.hip.
#pragma once

#include "select_device.h"

namespace talon {

constexpr float kNegInf = -__builtin_huge_valf();
constexpr int kHitTrigger = 64;                  // buffered vectors that trigger a cut before the next tile
constexpr int kHitCap = kHitTrigger + 64;        // a tile adds at most 64 vectors
constexpr int kRaiseHits = 8;                    // lanes beyond k that may hold new candidates before a group raises the threshold
constexpr int kSubBatch = 32;                    // vectors expanded per ranking round (two lanes per vector)
constexpr int kSubKeys = kSubBatch * 8 + TALON_K_MAX + 16;  // keys ranked per round (<= 8 logits per vector) + zero padding

// One 16-byte vector of a logits row, with -inf in the lanes past the end of the row.
template <int EPL>
__device__ __forceinline__ uint4 load_vec(const char* row, int e0, int vocab) {
  if (e0 + EPL <= vocab) return *reinterpret_cast<const uint4*>(row + static_cast<size_t>(e0) * (16 / EPL));
  uint32_t w[4];
  if constexpr (EPL == 4) {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(row);
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (e0 + e < vocab) ? p[e0 + e] : 0xFF800000u;
  } else {
    const uint16_t* p = reinterpret_cast<const uint16_t*>(row);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t lo = (e0 + 2 * q < vocab) ? p[e0 + 2 * q] : 0xFF80u;
      const uint32_t hi = (e0 + 2 * q + 1 < vocab) ? p[e0 + 2 * q + 1] : 0xFF80u;
      w[q] = lo | (hi << 16);
    }
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

template <int EPL>
__device__ __forceinline__ void unpack_vec(const uint4& v, float* x) {
  if constexpr (EPL == 4) {
    x[0] = __uint_as_float(v.x); x[1] = __uint_as_float(v.y);
    x[2] = __uint_as_float(v.z); x[3] = __uint_as_float(v.w);
  } else {
    x[0] = __uint_as_float(v.x << 16); x[1] = __uint_as_float(v.x & 0xFFFF0000u);
    x[2] = __uint_as_float(v.y << 16); x[3] = __uint_as_float(v.y & 0xFFFF0000u);
    x[4] = __uint_as_float(v.z << 16); x[5] = __uint_as_float(v.z & 0xFFFF0000u);
    x[6] = __uint_as_float(v.w << 16); x[7] = __uint_as_float(v.w & 0xFFFF0000u);
  }
}

// Partial results cross workgroups (and the per-XCD L2 caches) inside one launch.  They are
// written and read with agent-scope atomic accesses, which go to the device-coherent level
// directly, so no whole-cache write-back or invalidate is needed around the ticket.
template <typename T>
__device__ __forceinline__ void store_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_agent(const T* p) {
  return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Release half of a ticket: every global store and atomic this wavefront has issued so far
// has been performed at the device-coherent level when this returns.  A workgroup-scope
// fence does not give that (the compiler emits no wait on the vector memory counter for
// it), and without the wait a ticket's atomic can overtake the partial results it
// announces, even those of its own wavefront.  An agent-scope fence would also write the
// whole L2 back, which nothing here needs: everything that crosses workgroups is stored at
// agent scope.  Every wavefront of the workgroup calls this before the barrier that
// precedes the ticket.
__device__ __forceinline__ void stores_performed() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

__device__ __forceinline__ unsigned long long make_key(float x, int token) {
  return (static_cast<unsigned long long>(sortable_u32(x)) << 32) |
         static_cast<unsigned long long>(0xFFFFFFFFu - static_cast<uint32_t>(token));
}

// Smallest float greater than x (x finite or -inf, not NaN): "v > x" is "v >= float_above(x)".
__device__ __forceinline__ float float_above(float x) {
  x = x + 0.0f;
  const uint32_t u = __float_as_uint(x);
  return __uint_as_float((u >> 31) ? u - 1u : u + 1u);
}

__device__ __forceinline__ float key_logit(unsigned long long key) {
  return unsortable_f32(static_cast<uint32_t>(key >> 32));
}

// log of a softmax denominator (1 <= sum <= vocabulary size, or 0 / inf / NaN for a row that
// cannot be normalised): sum = 2^e * f with f in [0.5, 1), log(sum) = e*ln2 + log(f); the
// second term is small, so single precision gives it to about 1e-7 absolute.
__device__ __forceinline__ double log_of_sum(double sum) {
  if (!(sum > 0.0) || !(sum <= 1.7e308)) return log(sum);
  int e;
  const double f = frexp(sum, &e);
  return static_cast<double>(e) * 0.69314718055994530942 + static_cast<double>(__logf(static_cast<float>(f)));
}

// The least maximum that logits are exponentiated against: below it, maximum * log2(e) is no finite float, and a
// lane that met nothing but a mask of the type's lowest value would make the row's sum a NaN.  (Against
// this bound such logits add zero, as -inf does; a row without a larger logit cannot be normalised.)
constexpr float kLeastMax = -2.358e38f;

// A partial sum of exp(logit - m), taken to a maximum `to` >= m.  Where m is -inf the sum is zero, or NaN if
// there was a NaN among the logits (the maximum passes over it): it stays what it is, so that the row is
// found out whatever else it holds.
__device__ __forceinline__ double rescaled_sum(double sum, float m, float to) {
  return m == kNegInf ? sum : sum * static_cast<double>(__expf(m - to));
}

constexpr int kCandCap = 512;   // keys of a row merge that can still be among the k best, after the filter below

// Rank the keys of `lists` lists of k keys each (in LDS, every list sorted in descending order, zero
// keys in unused slots and up to the next multiple of 16) and hand the k best to emit(key, rank).
// s_cand: kCandCap + 16 keys of LDS, 16-byte aligned.
template <typename Emit>
__device__ __forceinline__ void rank_lists(const int k, const unsigned long long* keys, const int lists, const int tid,
                                           unsigned long long* s_cand, int* s_nc, Emit&& emit) {
  const int nkeys = lists * k;
  if (lists == 1) {   // a single sorted list: a key's position is its rank
    for (int i = tid; i < k; i += kThreads) {
      const unsigned long long ki = keys[i];
      if (ki != 0ull) emit(ki, i);
    }
  } else {
    // Rank by counting keys greater than mine.  First a filter: with q = ceil(k / lists), the
    // q-th key of every list is >= T = their minimum, so at least k keys are >= T and only keys
    // >= T can be among the k best; usually that leaves little more than k of the lists * k keys.
    bool done = false;
    if (lists <= 64) {
      const int q = (k + lists - 1) / lists;
      const int lane = tid & 63;
      unsigned long long inv = 0ull;   // ~key of this lane's list (0 beyond the lists: no effect on the max)
      if (lane < lists) inv = ~keys[lane * k + q - 1];
      const unsigned long long T = ~wave_max_u64(inv);   // 0 if a list is shorter than q: no filter then
      if (tid == 0) *s_nc = 0;
      __syncthreads();
      for (int i = tid; i < nkeys; i += kThreads) {
        const unsigned long long ki = keys[i];
        if (ki != 0ull && ki >= T) {
          const int slot = atomicAdd(s_nc, 1);
          if (slot < kCandCap) s_cand[slot] = ki;
        }
      }
      __syncthreads();
      const int nc = *s_nc;
      if (nc <= kCandCap) {
        if (tid < 16) s_cand[nc + tid] = 0ull;
        __syncthreads();
        for (int j = tid; j < nc; j += kThreads) {
          const unsigned long long ki = s_cand[j];
          const int r = count_greater_pad16(s_cand, nc, ki);
          if (r < k) emit(ki, r);
        }
        done = true;
      }
    }
    if (!done) {   // every key against every key
      for (int i = tid; i < nkeys; i += kThreads) {
        const unsigned long long ki = keys[i];
        if (ki == 0ull) continue;
        const int r = count_greater_pad16(keys, nkeys, ki);
        if (r < k) emit(ki, r);
      }
    }
  }
}

// The largest value with a 16-bit (sign, exponent, 7 mantissa bits) pattern that at least k of
// the 64 values v reach, found bit by bit on their order-preserving integer images (-inf if
// fewer than k lanes hold a logit).  For bf16 logits this is the k-th largest of them itself.
// With the lane maxima of a group it bounds the k best of all logits met so far from below.
__device__ __forceinline__ float kth_of_lanes(const float v, const int k) {
  const uint32_t u = sortable_u32(v);
  uint32_t prefix = 0u;
#pragma unroll
  for (int bit = 31; bit >= 16; --bit) {
    const uint32_t cand = prefix | (1u << bit);
    if (__popcll(__ballot(u >= cand)) >= k) prefix = cand;
  }
  return prefix <= 0x007FFFFFu ? kNegInf : unsortable_f32(prefix);   // at or below the image of -inf
}

// LDS of a scan, provided by the kernel.
struct ScanLds {
  uint4 (*hitv)[kHitCap];                    // [4] buffered vectors per wavefront
  int (*hith)[kHitCap];                      // [4] their tile * 64 + lane tags
  unsigned long long (*ck)[kSubKeys];        // [4] ranking scratch
  unsigned long long (*topw)[TALON_K_MAX];   // [4] k best keys of each wavefront, sorted (16-byte aligned)
  unsigned long long* top;                   // [TALON_K_MAX] the run's k best keys, sorted, zero keys in unused slots
  float* wmax;                               // [4]
  double* wsum;                              // [4]
  int* wcnt;                                 // [4]
};
constexpr int kHitvBytes = sizeof(uint4) * 4 * kHitCap;
constexpr int kHithBytes = sizeof(int) * 4 * kHitCap;
constexpr int kCkBytes = sizeof(unsigned long long) * 4 * kSubKeys;
constexpr int kScanBytes = kHitvBytes + kHithBytes + kCkBytes;

// Blocks [blk0, blk1) of `row` (a block: 4 x 16-byte loads per thread).  Leaves the k best keys in
// L.top and returns the run's maximum and sum of exp(logit - maximum) in every thread; starts
// without and ends with a barrier behind which L.top may be read.
// PREFETCH: issue the loads of the next block before the current one is processed.
// WATCH: the first wavefront polls `stop` every kWatchBlocks blocks (the load travels with the block's
// own loads) and tells the others through *s_stop (LDS, zero on entry); once the word is non-zero the
// run is given up, and the call returns false in every thread.  (Not together with PREFETCH: the
// scanners that watch have no registers for it.)
constexpr int kWatchBlocks = 2;   // a thousand workgroups polling a word per block and wavefront hold up its memory channel
template <int EPL, bool PREFETCH, bool WATCH>
__device__ __forceinline__ bool scan_chunk(const char* row, const int vocab, const int k, const int blk0, const int blk1,
                                           const ScanLds& L, float& cm, double& csum, const int32_t* stop = nullptr,
                                           int* s_stop = nullptr) {
  static_assert(!(PREFETCH && WATCH), "the word is polled with a block's own loads");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  uint4* hitv = L.hitv[wave];
  int* hith = L.hith[wave];
  unsigned long long* ck = L.ck[wave];
  unsigned long long* topw = L.topw[wave];
  // ---- wavefront-local streaming state
  int cnt = 0;            // buffered vectors
  int tcnt = 0;           // keys in topw (<= k)
  float tau = __builtin_huge_valf();   // a vector is buffered iff one of its logits is >= tau (set by the first step)
  float m_l = kNegInf;    // this lane's running max
  double s_l = 0.0;       // this lane's running sum of exp(logit - m_l)

  // A tile is one 16-byte vector per thread (256 * EPL logits); a block is 4 tiles, and the
  // scan advances by groups of 4 tiles.  A group that lies wholly inside the row is loaded
  // with plain vector loads; the group at the ragged end of the row (only in the row's last
  // chunk) with guarded loads that return -inf past the end.
  const int t0 = blk0 * kScanTiles;
  const int tiles_in_row = (vocab + kThreads * EPL - 1) / (kThreads * EPL);
  const int full_tiles = vocab / (kThreads * EPL);
  const int t1 = blk1 * kScanTiles < tiles_in_row ? blk1 * kScanTiles : tiles_in_row;
  const char* lane_ptr = row + static_cast<size_t>(tid) * 16;
  constexpr size_t kTileBytes = static_cast<size_t>(kThreads) * 16;

  // Buffer this lane's vector if one of its logits reaches tau.  Returns false (and buffers
  // nothing) when the wavefront's buffer has no room for all hits of the tile.
  auto buffer_hits = [&](const uint4& raw, float vmax, int tile) -> bool {
    const bool hit = vmax >= tau;
    const unsigned long long bal = __ballot(hit);
    if (bal != 0ull) {
      const int nh = __popcll(bal);
      if (cnt + nh > kHitCap) return false;
      const int pos = cnt + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(bal >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(bal), 0));
      if (hit) { hitv[pos] = raw; hith[pos] = tile * 64 + lane; }
      cnt += nh;
    }
    return true;
  };

  // Streaming state machine.  A step is a group of 4 tiles.  Tiles whose hits do not fit the
  // buffer are deferred, together with all later tiles of the group, to the single slow
  // section below, which cuts the buffer and then re-reads them.
  // One group of 4 tiles of this thread: plain vector loads where the group lies wholly inside
  // the row, guarded loads (-inf past the end) at the ragged end.
  auto load_group = [&](int t, uint4 (&r)[kScanTiles]) {
    if (t + kScanTiles <= full_tiles) {
#pragma unroll
      for (int q = 0; q < kScanTiles; ++q)
        r[q] = *reinterpret_cast<const uint4*>(lane_ptr + (t + q) * kTileBytes);
    } else {
#pragma unroll
      for (int q = 0; q < kScanTiles; ++q)
        r[q] = load_vec<EPL>(row, ((t + q) * kThreads + tid) * EPL, vocab);
    }
  };
  // Sums are of 2^(x*log2e - c) with c = fl(m*log2e); the rounding of c is a common factor
  // 2^(c - m*log2e) of a whole group, applied once at its end.  (Kept with the maximum where there are registers for it: 23
  // launches of one layer for 16 sequences of 250 nodes 347 us with c worked out in every group, 343; the
  // scans at four workgroups per compute unit are 0.3 % faster the other way.)
  const float kLog2e = 1.4426950408889634f;
  float c = kLeastMax * kLog2e, c_err = 0.f;   // m*log2e and, exactly, m*log2e - c
  auto against = [&](const float m) {
    const float mm = fmaxf(m, kLeastMax);
    c = mm * kLog2e;
    c_err = __builtin_fmaf(mm, kLog2e, -c);
  };
  int tb = t0;
  bool done = false;
  // With the selection in the launch the kernel runs three workgroups per compute unit and has
  // registers to spare: the loads of the next group are issued before the current one is
  // processed, so that a chunk of several blocks does not pay the memory latency per block.
  // The scan-only launch runs four workgroups per compute unit on 128 registers and relies on
  // those for the overlap.
  uint4 raw_next[kScanTiles];
  bool given_up = false;
  // (before a block's loads are issued / when they have arrived)
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto watch_issue = [&](int t) -> int32_t {
    return wave_u == 0 && ((t - t0) / kScanTiles) % kWatchBlocks == 0 ? load_agent(stop) : 0;
  };
  auto watch_test = [&](int32_t word) -> bool {
    if (wave_u == 0 && __builtin_amdgcn_readfirstlane(word) != 0) *reinterpret_cast<volatile int*>(s_stop) = 1;
    return *reinterpret_cast<volatile int*>(s_stop) != 0;
  };
  if constexpr (PREFETCH) {
    if (tb < t1) load_group(tb, raw_next);
  }
  while (!done) {
    uint32_t deferred = 0;   // bit q: tile def_base + q still has to be buffered
    int def_base = tb;
    bool force = false;
    if (tb < t1) {
      uint4 raw[kScanTiles];
      if constexpr (PREFETCH) {
#pragma unroll
        for (int q = 0; q < kScanTiles; ++q) raw[q] = raw_next[q];
        if (tb + kScanTiles < t1) load_group(tb + kScanTiles, raw_next);
      } else {
        int32_t stop_now = 0;
        if constexpr (WATCH) stop_now = watch_issue(tb);
        load_group(tb, raw);
        if constexpr (WATCH) {
          if (watch_test(stop_now)) { given_up = true; break; }
        }
      }
      // lane maxima of the 4 tiles first; the running max moves at most once per group
      float vmax4[kScanTiles];
#pragma unroll
      for (int q = 0; q < kScanTiles; ++q) {
        float x[EPL];
        unpack_vec<EPL>(raw[q], x);
        float vmax = x[0];
#pragma unroll
        for (int e = 1; e < EPL; ++e) vmax = fmaxf(vmax, x[e]);
        vmax4[q] = vmax;
      }
      const float gmax = fmaxf(fmaxf(vmax4[0], vmax4[1]), fmaxf(vmax4[2], vmax4[3]));
      if (gmax > m_l) {
        s_l = rescaled_sum(s_l, m_l, gmax);
        m_l = gmax;
        if constexpr (PREFETCH) against(gmax);
      }
      if constexpr (!PREFETCH) against(m_l);
      float acc = 0.f;
#pragma unroll
      for (int q = 0; q < kScanTiles; ++q) {
        // unpack again from the raw vector instead of keeping the 4 * EPL floats of the
        // maximum pass alive (the empty asm hides the value's origin from the optimiser)
        uint4 r = raw[q];
        asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w));
        float x[EPL];
        unpack_vec<EPL>(r, x);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc += __builtin_amdgcn_exp2f(__builtin_fmaf(x[e], kLog2e, -c));
      }
      s_l += static_cast<double>(acc * __builtin_amdgcn_exp2f(-c_err));
      if (tb == t0) {
        tau = kth_of_lanes(gmax, k);
        force = true;
      } else if (__popcll(__ballot(gmax >= tau)) > k + kRaiseHits) {
        // Many lanes hold a new candidate: the row rises along the token ids (a sorted row, or a
        // permutation with a short period).  The group's own maxima raise the threshold before
        // anything is buffered, so that such a row does not rank every one of its vectors.
        tau = fmaxf(tau, kth_of_lanes(gmax, k));
      }
      // Lanes that hold a candidate, per tile: all four tiles at once where the buffer has room for them
      // (one test for a group without any, and straight-line code for one with a few; a test per tile
      // before: 4080 rows of 304 KB 229 us, now 225; three sequences of 48 nodes by the separate calls 66.0, now 65.2).
      unsigned long long hits[kScanTiles];
      int n_hits = 0;
#pragma unroll
      for (int q = 0; q < kScanTiles; ++q) {
        hits[q] = __ballot(vmax4[q] >= tau);
        n_hits += __popcll(hits[q]);
      }
      if (n_hits != 0) {
        if (cnt + n_hits <= kHitCap) {
#pragma unroll
          for (int q = 0; q < kScanTiles; ++q) {
            const int pos = cnt + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(hits[q] >> 32),
                                                            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(hits[q]), 0));
            if (vmax4[q] >= tau) { hitv[pos] = raw[q]; hith[pos] = (tb + q) * 64 + lane; }
            cnt += __popcll(hits[q]);
          }
        } else {
#pragma unroll
          for (int q = 0; q < kScanTiles; ++q)
            if (deferred != 0u || !buffer_hits(raw[q], vmax4[q], tb + q)) deferred |= 1u << q;
        }
      }
      tb += kScanTiles;
    } else {
      force = cnt > 0;
      done = true;
    }

    if (force || deferred != 0u || cnt > kHitTrigger) {
      // ---- slow section: cut the buffer to the k best; then buffer the deferred tiles
      while (true) {
        // Expand the buffered vectors, rank their logits that reach tau together with the k
        // best so far, keep the k best.  Every buffered token id is below every id still to
        // come (deferred tiles included), so afterwards a logit equal to the k-th best loses
        // the tie and tau becomes the next float above it.
        for (int base = 0; base < cnt; base += kSubBatch) {
          constexpr int HPL = EPL / 2;   // logits per lane: a lane expands half a vector
          float x[HPL];
          int e0 = 0;
          uint32_t hbits = 0;
          if (base + (lane >> 1) < cnt) {
            const int slot = base + (lane >> 1), half = lane & 1;
            const uint2 raw = reinterpret_cast<const uint2*>(&hitv[slot])[half];
            const int hdr = hith[slot];
            e0 = (((hdr >> 6) * 4 + wave) * 64 + (hdr & 63)) * EPL + half * HPL;
            if constexpr (EPL == 4) {
              x[0] = __uint_as_float(raw.x); x[1] = __uint_as_float(raw.y);
            } else {
              x[0] = __uint_as_float(raw.x << 16); x[1] = __uint_as_float(raw.x & 0xFFFF0000u);
              x[2] = __uint_as_float(raw.y << 16); x[3] = __uint_as_float(raw.y & 0xFFFF0000u);
            }
#pragma unroll
            for (int e = 0; e < HPL; ++e)
              if (x[e] >= tau && e0 + e < vocab) hbits |= 1u << e;
          }
          const int nh = __popc(hbits);
          const int incl = wave_inclusive_scan_i32(nh);
          const int total = __builtin_amdgcn_readlane(incl, 63);
          if (lane < tcnt) ck[lane] = topw[lane];
          int pos = tcnt + incl - nh;
#pragma unroll
          for (int e = 0; e < HPL; ++e)
            if (hbits & (1u << e)) ck[pos++] = make_key(x[e], e0 + e);
          const int n = tcnt + total;
          if (lane < 16) ck[n + lane] = 0ull;   // zero keys up to the next multiple of 16
          // LDS operations of one wavefront complete in order: ck is complete before it is read
          for (int i = lane; i < n; i += 64) {
            const unsigned long long key = ck[i];
            const int r = count_greater_pad16(ck, n, key);
            if (r < k) topw[r] = key;
          }
          tcnt = n < k ? n : k;
          if (base + kSubBatch < cnt && tcnt >= k) tau = fmaxf(tau, key_logit(topw[k - 1]));
        }
        cnt = 0;
        if (deferred == 0u && tb >= t1) break;   // nothing is left that tau would be compared with
        if (tcnt >= k) tau = float_above(key_logit(topw[k - 1]));
        if (deferred == 0u) break;
#pragma unroll 1
        for (int q = 0; q < kScanTiles; ++q) {
          if (!((deferred >> q) & 1u)) continue;
          const int tile = def_base + q;
          const uint4 raw = load_vec<EPL>(row, (tile * kThreads + tid) * EPL, vocab);
          float x[EPL];
          unpack_vec<EPL>(raw, x);
          float vmax = x[0];
#pragma unroll
          for (int e = 1; e < EPL; ++e) vmax = fmaxf(vmax, x[e]);
          if (!buffer_hits(raw, vmax, tile)) break;   // full again: cut first
          deferred &= ~(1u << q);
        }
      }
    }
  }

  // ---- wavefront statistics
  {
    const float wmax = wave_max_f32(m_l);
    // rescale factors are <= 1 and only need fp32 accuracy: their error is relative to a part of the sum
    const double wsum = wave_sum_f64(rescaled_sum(s_l, m_l, wmax));
    if (lane == 0) { L.wmax[wave] = wmax; L.wsum[wave] = wsum; L.wcnt[wave] = given_up ? -(1 << 20) : tcnt; }
    static_assert(TALON_K_MAX == 64, "a list has one slot per lane");
    if (lane >= tcnt) topw[lane] = 0ull;   // unused slots of the list: zero keys
  }
  __syncthreads();

  // ---- merge the four lists (each <= k keys, zero keys in the unused slots) into the
  // chunk's k best, sorted.  Lane 16g+i of wavefront w holds key i of list w and counts how many keys of
  // list g are greater; the four lanes' counts add up to the rank.
  const int ctot = L.wcnt[0] + L.wcnt[1] + L.wcnt[2] + L.wcnt[3];
  if constexpr (WATCH) {
    if (ctot < 0) return false;   // one wavefront saw the word: the workgroup gives the run up
  }
  if (k <= 16) {
    const int group = lane >> 4;
    const unsigned long long mkey = topw[lane & 15];
    const ulonglong2* kp = reinterpret_cast<const ulonglong2*>(L.topw[group]);
    ulonglong2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = kp[(u + 2 * group) & 7];   // the four lists start on the same bank
    int r = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) r += ((v[u].x > mkey) ? 1 : 0) + ((v[u].y > mkey) ? 1 : 0);
    auto p16 = __builtin_amdgcn_permlane16_swap(r, r, false, false);
    r = static_cast<int>(p16[0]) + static_cast<int>(p16[1]);
    auto p32 = __builtin_amdgcn_permlane32_swap(r, r, false, false);
    r = static_cast<int>(p32[0]) + static_cast<int>(p32[1]);
    if (lane < 16 && mkey != 0ull && r < k) L.top[r] = mkey;
    if (tid >= ctot && tid < k) L.top[tid] = 0ull;   // fewer than k logits in this chunk
  } else {
    // long lists: thread t holds key t % 64 of its own wavefront's list and counts against all four
    const unsigned long long mkey = L.topw[wave][lane];
    int r = 0;
#pragma unroll 1   // a rare path: keep it small in registers
    for (int w = 0; w < 4; ++w) r += count_greater_pad16(L.topw[w], 64, mkey);
    if (mkey != 0ull && r < k) L.top[r] = mkey;
    if (tid >= ctot && tid < k) L.top[tid] = 0ull;
  }
  cm = fmaxf(fmaxf(L.wmax[0], L.wmax[1]), fmaxf(L.wmax[2], L.wmax[3]));
  csum = 0.0;
#pragma unroll
  for (int w = 0; w < 4; ++w) csum += rescaled_sum(L.wsum[w], L.wmax[w], cm);
  __syncthreads();
  return true;
}

}  // namespace talon
