// Pieces of the uncapped pool of Alg. 2 shared by the layer-by-layer launches (literal.hip) and the
// launch that scans rows ahead (ahead.hip): searches for the n-th largest of many 64-bit keys, and
// the budget check over lists of keys.
#pragma once

#include "scan_device.h"

namespace talon {

__device__ __forceinline__ double key_to_f64(unsigned long long s) {
  const unsigned long long u = (s >> 63) ? (s ^ 0x8000000000000000ull) : ~s;
  return __longlong_as_double(static_cast<long long>(u));
}

// Histogram of 8-bit digits in LDS, fed one wavefront-wide call at a time.  Keys of one row
// often share their leading digits: when all lanes that count hit the same bin, their number
// is added by one lane, and runs of such calls on the same bin are added up in a register
// first (flush() hands the rest over; call it before the histogram is read).
struct WaveHist {
  int* hist;
  int pend_digit = -1;
  int pend_count = 0;
  __device__ __forceinline__ explicit WaveHist(int* h) : hist(h) {}
  __device__ __forceinline__ void flush() {
    if (pend_count > 0 && (threadIdx.x & 63) == 0) atomicAdd(&hist[pend_digit], pend_count);
    pend_count = 0;
    pend_digit = -1;
  }
  __device__ __forceinline__ void add(bool c, int digit) {
    const unsigned long long m = __ballot(c);
    if (m == 0ull) return;
    const int lead = __ffsll(static_cast<long long>(m)) - 1;
    const int d0 = __builtin_amdgcn_readlane(digit, lead);
    const unsigned long long same = __ballot(c && digit == d0);
    if (same == m) {
      if (d0 != pend_digit) { flush(); pend_digit = d0; }
      pend_count += __popcll(m);
    } else if (c) {
      atomicAdd(&hist[digit], 1);
    }
  }
};

// One slot of a counter in LDS for every lane with c set (-1 for the others): one atomic per
// wavefront, the lanes' slots in lane order.
__device__ __forceinline__ int claim_slots(int* counter, bool c) {
  const unsigned long long m = __ballot(c);
  if (m == 0ull) return -1;
  const int lane = threadIdx.x & 63;
  const int lead = __ffsll(static_cast<long long>(m)) - 1;
  int base = 0;
  if (lane == lead) base = atomicAdd(counter, __popcll(m));
  base = __shfl(base, lead);
  return c ? base + __popcll(m & ((1ull << lane) - 1ull)) : -1;
}

// Walks the 256 bins from the largest digit down to the bin that holds the `remaining`-th
// key.  Returns that digit, plus 256 if the bin holds exactly the keys still wanted (then
// all of them are kept and the search is over); *s_want = keys wanted from the bin.  Starts
// with a barrier (the histogram is complete) and ends with one (the result is visible); the
// caller places another before the histogram or the result words are written again.
__device__ __forceinline__ int find_bin(const int* s_hist, int remaining, int* s_digit, int* s_want) {
  const int tid = threadIdx.x;
  __syncthreads();
  if (tid < 64) {   // lane l owns digits 255-4l .. 252-4l
    int h[4], lane_sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) { h[j] = s_hist[255 - 4 * tid - j]; lane_sum += h[j]; }
    const int incl = wave_inclusive_scan_i32(lane_sum);
    const unsigned long long hit = __ballot(incl >= remaining);
    const int first = hit ? __ffsll(static_cast<long long>(hit)) - 1 : 63;
    if (tid == first) {
      int before = incl - lane_sum;
      int dg = 255 - 4 * tid;
      int j = 0;
#pragma unroll
      for (; j < 3; ++j) {
        if (before + h[j] < remaining) { before += h[j]; --dg; } else break;
      }
      const int want = remaining - before;
      *s_digit = dg | ((h[j] == want) ? 256 : 0);
      *s_want = want;
    }
  }
  __syncthreads();
  return *s_digit;
}

template <int NT>
__device__ __forceinline__ unsigned long long block_max_u64_nt(unsigned long long v, unsigned long long* scratch) {
  v = wave_max_u64(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long m = scratch[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) m = scratch[w] > m ? scratch[w] : m;
  return m;
}

// Exclusive prefix sum over the NT threads; *total receives the workgroup sum.
template <int NT>
__device__ __forceinline__ int block_exclusive_scan_nt(int v, int* scratch, int* total) {
  const int incl = wave_inclusive_scan_i32(v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 63) scratch[wave] = incl;
  __syncthreads();
  int base = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const int x = scratch[w];
    if (w < wave) base += x;
    sum += x;
  }
  *total = sum;
  return base + incl - v;
}

constexpr int kFinCap = 256;     // keys of the last bin that the budget check ranks by counting

// LDS of the budget check; the caller fills in the lists' sizes and offsets.
template <int POOL, int LISTS>
struct PickLds {
  unsigned long long pool[POOL];
  unsigned long long kkey[256];
  unsigned long long fin_hi[kFinCap], fin_lo[kFinCap];
  int cnt[LISTS], off[LISTS];   // keys of a list, and of the lists before it
  int kj[256];
  unsigned char pool_j[POOL];
};

// The `limit` best (at most 255) of the `total` keys in n_lists lists of at most 256 keys each, by (path
// score descending, parent ascending, token ascending), handed to emit(rank, parent, key, edge log-probability)
// in (parent, in-row) order; returns their number.  All NT threads; starts after and ends without a
// barrier.  lp, lse: path score and log-sum-exp of the parents, by local index; parent_of(list);
// load_key(list, i).  cm: words of LDS (hist[256], digit, want, nkeep, nfin, red_u64).
template <int NT, int POOL, int LISTS, typename Words, typename ParentOf, typename LoadKey, typename Emit>
__device__ __forceinline__ int pick_best(const int n_lists, const int total, const int limit, PickLds<POOL, LISTS>& L, Words& cm,
                                         const double* lp, const double* lse, ParentOf&& parent_of, LoadKey&& load_key, Emit&& emit) {
  static_assert(NT >= 256, "a list is read by one thread per key");
  const int tid = threadIdx.x;
  if (tid == 0) cm.nkeep = 0;
  __syncthreads();
  // The pool in LDS, lists one after the other, when it fits (it does unless many rows are
  // flat); otherwise every pass reads it from memory, list by list.
  const bool dense = total <= POOL;
  if (dense) {
    // One pool position per thread and round: the list of a position is the last one that starts
    // at or before it (empty lists start where the next one does, and the last list that starts at
    // or before a position below `total` has some keys).
    for (int i0 = 0; i0 < total; i0 += NT) {
      const int i = i0 + tid;
      if (i < total) {
        int lo_j = 0, hi_j = n_lists - 1;
        while (lo_j < hi_j) {
          const int mid = (lo_j + hi_j + 1) >> 1;
          if (L.off[mid] <= i) lo_j = mid; else hi_j = mid - 1;
        }
        L.pool[i] = load_key(lo_j, i - L.off[lo_j]);
        L.pool_j[i] = static_cast<unsigned char>(parent_of(lo_j));
      }
    }
    __syncthreads();
  }
  // f(valid, parent j, key): the same number of calls in every thread
  auto for_each = [&](auto&& f) {
    if (dense) {
      for (int i0 = 0; i0 < total; i0 += NT) {
        const int i = i0 + tid;
        const bool valid = i < total;
        f(valid, valid ? static_cast<int>(L.pool_j[i]) : 0, valid ? L.pool[i] : 0ull);
      }
    } else {
      for (int l = 0; l < n_lists; ++l) {
        const bool valid = tid < L.cnt[l];
        f(valid, parent_of(l), valid ? load_key(l, tid) : 0ull);
      }
    }
  };
  // path score of a candidate as a sortable key, and the order among equal scores (parent
  // ascending, then token ascending = in-row rank ascending) as a second key
  auto score_key = [&](int j, unsigned long long key) {
    return sortable_u64(lp[j] + (static_cast<double>(unsortable_f32(static_cast<uint32_t>(key >> 32))) - lse[j]));
  };
  auto order_key = [&](int j, unsigned long long key) {
    return ((static_cast<unsigned long long>(255 - j) << 32) | (key & 0xFFFFFFFFull)) << 24;
  };

  unsigned long long pre_hi = 0ull, pre_lo = 0ull, low = 0ull;
  int sh = 0;
  const bool cut = total > limit;
  if (cut) {
    // move the score keys to the range they span, so that their digits spread over the bins
    unsigned long long mx = 0ull, inv_mn = 0ull;
    for_each([&](bool valid, int j, unsigned long long key) {
      if (valid) {
        const unsigned long long hi = score_key(j, key);
        mx = hi > mx ? hi : mx;
        inv_mn = ~hi > inv_mn ? ~hi : inv_mn;
      }
    });
    mx = block_max_u64_nt<NT>(mx, cm.red_u64);
    low = ~block_max_u64_nt<NT>(inv_mn, cm.red_u64);
    sh = __clzll(static_cast<long long>(mx - low + 1ull));
    int remaining = limit;
    for (int pass = 0; pass < 13; ++pass) {
      const bool first_key = pass < 8;
      const int shift = first_key ? 56 - 8 * pass : 56 - 8 * (pass - 8);
      if (tid < 256) cm.hist[tid] = 0;
      __syncthreads();
      WaveHist wh(cm.hist);
      for_each([&](bool valid, int j, unsigned long long key) {
        const unsigned long long hi = (score_key(j, key) - low + 1ull) << sh;
        const unsigned long long lo2 = order_key(j, key);
        bool match;
        int digit;
        if (first_key) {
          match = pass == 0 || ((hi ^ pre_hi) >> (shift + 8)) == 0ull;
          digit = static_cast<int>(hi >> shift) & 255;
        } else {
          match = hi == pre_hi && (pass == 8 || ((lo2 ^ pre_lo) >> (shift + 8)) == 0ull);
          digit = static_cast<int>(lo2 >> shift) & 255;
        }
        wh.add(valid && match, digit);
      });
      wh.flush();
      const int r = find_bin(cm.hist, remaining, &cm.digit, &cm.want);
      const int population = cm.hist[r & 255];
      if (first_key) pre_hi |= static_cast<unsigned long long>(r & 255) << shift;
      else pre_lo |= static_cast<unsigned long long>(r & 255) << shift;
      remaining = cm.want;
      __syncthreads();
      if (r & 256) break;
      if (population <= kFinCap) {
        // The bin fits one key per thread: rank its keys by counting and take the cut from
        // there.  (Scores of bf16 rows tie in whole groups, and a cut inside such a group
        // would otherwise walk every remaining digit of both keys.)
        if (tid == 0) cm.nfin = 0;
        __syncthreads();
        for_each([&](bool valid, int j, unsigned long long key) {
          const unsigned long long hi = (score_key(j, key) - low + 1ull) << sh;
          const unsigned long long lo2 = order_key(j, key);
          const bool in_bin = valid && (first_key ? ((hi ^ pre_hi) >> shift) == 0ull
                                                  : (hi == pre_hi && ((lo2 ^ pre_lo) >> shift) == 0ull));
          const int slot = claim_slots(&cm.nfin, in_bin);
          if (slot >= 0 && slot < kFinCap) { L.fin_hi[slot] = hi; L.fin_lo[slot] = lo2; }
        });
        __syncthreads();
        const int nf = cm.nfin < kFinCap ? cm.nfin : kFinCap;
        if (tid < nf) {
          const unsigned long long mh = L.fin_hi[tid], ml = L.fin_lo[tid];
          int rank = 0;
          int i = 0;
          for (; i + 8 <= nf; i += 8) {   // eight broadcast reads in flight: the loop is bound by LDS latency
            unsigned long long oh[8], ol[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) { oh[u] = L.fin_hi[i + u]; ol[u] = L.fin_lo[i + u]; }
#pragma unroll
            for (int u = 0; u < 8; ++u) rank += (oh[u] > mh || (oh[u] == mh && ol[u] > ml)) ? 1 : 0;
          }
          for (; i < nf; ++i) {
            const unsigned long long oh = L.fin_hi[i], ol = L.fin_lo[i];
            rank += (oh > mh || (oh == mh && ol > ml)) ? 1 : 0;
          }
          if (rank == remaining - 1) { cm.red_u64[0] = mh; cm.red_u64[1] = ml; }   // keys are unique: one thread
        }
        __syncthreads();
        pre_hi = cm.red_u64[0];
        pre_lo = cm.red_u64[1];
        __syncthreads();
        break;
      }
    }
  }

  // kept candidates, in any order
  for_each([&](bool valid, int j, unsigned long long key) {
    bool keep = valid;
    if (cut && valid) {
      const unsigned long long hi = (score_key(j, key) - low + 1ull) << sh;
      keep = hi > pre_hi || (hi == pre_hi && order_key(j, key) >= pre_lo);
    }
    const int slot = claim_slots(&cm.nkeep, keep);
    if (slot >= 0 && slot < 256) { L.kkey[slot] = key; L.kj[slot] = j; }
  });
  __syncthreads();
  const int n_keep = cm.nkeep < limit ? cm.nkeep : limit;

  // node ids in (parent ascending, in-row rank ascending) order: rank by counting
  if (tid < n_keep) {
    const int myj = L.kj[tid];
    const unsigned long long myk = L.kkey[tid];
    int rank = 0;
    int i = 0;
    for (; i + 8 <= n_keep; i += 8) {
      int oj[8];
      unsigned long long ok[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { oj[u] = L.kj[i + u]; ok[u] = L.kkey[i + u]; }
#pragma unroll
      for (int u = 0; u < 8; ++u) rank += (oj[u] < myj || (oj[u] == myj && ok[u] > myk)) ? 1 : 0;
    }
    for (; i < n_keep; ++i) {
      const int oj = L.kj[i];
      rank += (oj < myj || (oj == myj && L.kkey[i] > myk)) ? 1 : 0;
    }
    const float lg = unsortable_f32(static_cast<uint32_t>(myk >> 32));
    emit(rank, myj, myk, static_cast<double>(lg) - lse[myj]);
  }
  return n_keep;
}

}  // namespace talon
