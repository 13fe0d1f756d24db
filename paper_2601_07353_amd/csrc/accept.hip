// Verification outcome at temperature 0 (App. B "Token-Tree Verification", step (2); Sec. 2:
// the verifier accepts the longest matched prefix): from the target model's greedy token
// after every tree node, the longest root path on which every drafted token is the target's
// own choice, the token the target adds after it, and the move of the accepted tokens' keys
// and values into the prefix cache.
//
// The target's greedy tokens take two kernels: one streams the rows, the other puts the pieces of
// a row together.
#include "scan_device.h"

namespace talon {

namespace {

// ---- target argmax, first kernel: softmax statistics and the largest logit of a run of a row.
// Bound: memory.  A workgroup takes one run of `blocks_per_run` blocks of 16 KiB of one row and
// leaves its maximum, sum and key; nothing is shared between workgroups, so there is no ticket to
// prepare beforehand and none to wait for, and a lane keeps only its best vector so far (which of
// its logits it was is found at the end).  The loads of the next block are in flight while a block
// is worked on.  It took the place of the k-best scan with k = 1 (ranking buffers, tickets, and a
// launch in front of it that cleared them): with the
// accepting walk and the cache's compaction 60 rows of 257 KB 21.0 -> 13.8 us of GPU time, 512 of 304 KB 47.9 -> 43.4,
// 4096 of them 238.8 -> 230.7 (5.4 TB/s).
// The sums are formed as the k-best scan forms them: at most 32 exponentials of a lane in single
// precision, everything above in double.
template <int EPL>
__global__ __launch_bounds__(kThreads, 6) void argmax_scan_kernel(ArgmaxArgs a) {
  __shared__ unsigned long long s_key[4];
  __shared__ double s_sum[4];
  __shared__ float s_max[4];
  const int b = blockIdx.y;
  const int node = blockIdx.x / a.runs;
  const int run = blockIdx.x - node * a.runs;
  if (node >= a.n_nodes[b]) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const char* row = static_cast<const char*>(a.logits) +
                    (static_cast<int64_t>(b) * a.seq_stride + static_cast<int64_t>(node) * a.row_stride) * (16 / EPL);
  const int vocab = a.vocab;
  const int full_tiles = vocab / (kThreads * EPL);   // a tile: one 16-byte vector per thread; a block: kScanTiles of them
  const int tiles_in_row = (vocab + kThreads * EPL - 1) / (kThreads * EPL);
  int t = run * a.blocks_per_run * kScanTiles;
  const int t_stop = t + a.blocks_per_run * kScanTiles;
  const int t1 = t_stop < tiles_in_row ? t_stop : tiles_in_row;
  const char* lane_ptr = row + static_cast<size_t>(tid) * 16;
  constexpr size_t kTileBytes = static_cast<size_t>(kThreads) * 16;
  auto load_block = [&](int t, uint4 (&r)[kScanTiles]) {
    if (t + kScanTiles <= full_tiles) {
#pragma unroll
      for (int q = 0; q < kScanTiles; ++q) r[q] = *reinterpret_cast<const uint4*>(lane_ptr + (t + q) * kTileBytes);
    } else {
#pragma unroll
      for (int q = 0; q < kScanTiles; ++q) r[q] = load_vec<EPL>(row, ((t + q) * kThreads + tid) * EPL, vocab);
    }
  };
  float m_l = kNegInf;    // this lane's running max ...
  double s_l = 0.0;       // ... and running sum of exp(logit - m_l)
  uint4 best = make_uint4(0u, 0u, 0u, 0u);   // the vector that holds m_l, and its tile
  int best_tile = -1;
  uint4 raw[kScanTiles];
  if (t < t1) load_block(t, raw);
  while (t < t1) {
    uint4 next[kScanTiles];
    if (t + kScanTiles < t1) load_block(t + kScanTiles, next);
    float vmax[kScanTiles];
#pragma unroll
    for (int q = 0; q < kScanTiles; ++q) {
      float x[EPL];
      unpack_vec<EPL>(raw[q], x);
      vmax[q] = x[0];
#pragma unroll
      for (int e = 1; e < EPL; ++e) vmax[q] = fmaxf(vmax[q], x[e]);
    }
    const float gmax = fmaxf(fmaxf(vmax[0], vmax[1]), fmaxf(vmax[2], vmax[3]));
    if (gmax > m_l || (best_tile < 0 && gmax == m_l)) {   // (a row of -inf alone has a token too, its first)
      s_l = rescaled_sum(s_l, m_l, gmax);
      m_l = gmax;
#pragma unroll
      for (int q = kScanTiles - 1; q >= 0; --q)   // the first of equal ones
        if (vmax[q] == gmax) { best = raw[q]; best_tile = t + q; }
    }
    // sum of 2^(x*log2e - c) with c = fl(m*log2e); the rounding of c is taken out once per block
    const float kLog2e = 1.4426950408889634f;
    const float mm = fmaxf(m_l, kLeastMax);
    const float c = mm * kLog2e;
    const float c_err = __builtin_fmaf(mm, kLog2e, -c);
    float acc = 0.f;
#pragma unroll
    for (int q = 0; q < kScanTiles; ++q) {
      uint4 r = raw[q];
      asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w));   // unpacked again instead of kept: see scan_chunk
      float x[EPL];
      unpack_vec<EPL>(r, x);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc += __builtin_amdgcn_exp2f(__builtin_fmaf(x[e], kLog2e, -c));
    }
    s_l += static_cast<double>(acc * __builtin_amdgcn_exp2f(-c_err));
#pragma unroll
    for (int q = 0; q < kScanTiles; ++q) raw[q] = next[q];
    t += kScanTiles;
  }
  unsigned long long key = 0ull;
  if (best_tile >= 0) {
    float x[EPL];
    unpack_vec<EPL>(best, x);
    int e0 = 0;
#pragma unroll
    for (int e = EPL - 1; e >= 0; --e)
      if (x[e] == m_l) e0 = e;
    const int token = (best_tile * kThreads + tid) * EPL + e0;
    if (token < vocab) key = make_key(m_l, token);   // (not the -inf that stands behind the row's end)
  }
  key = wave_max_u64(key);
  const float wmax = wave_max_f32(m_l);
  const double wsum = wave_sum_f64(rescaled_sum(s_l, m_l, wmax));
  if (lane == 0) { s_key[wave] = key; s_max[wave] = wmax; s_sum[wave] = wsum; }
  __syncthreads();
  if (tid == 0) {
    const float cm = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    double csum = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      csum += rescaled_sum(s_sum[w], s_max[w], cm);
      key = s_key[w] > key ? s_key[w] : key;
    }
    const size_t slot = (static_cast<size_t>(b) * a.N_pad + node) * a.blocks + run;
    a.part_max[slot] = cm;
    a.part_sum[slot] = csum;
    a.part_key[slot] = key;
  }
}

// ---- second kernel: one workgroup per sequence, 16 lanes per row.
constexpr int kMergeThreads = 1024;
__global__ __launch_bounds__(kMergeThreads) void argmax_merge_kernel(ArgmaxArgs a) {
  const int b = blockIdx.x;
  const int n = a.n_nodes[b] < a.N_pad ? a.n_nodes[b] : a.N_pad;
  const int l = threadIdx.x & 15;
  int any_bad = 0;
  for (int node = threadIdx.x >> 4; node < n; node += kMergeThreads / 16) {
    const size_t row = static_cast<size_t>(b) * a.N_pad + node;
    const size_t slot = row * a.blocks;
    float m = kNegInf;
    double sum = 0.0;
    unsigned long long key = 0ull;
    if (l < a.runs) { m = a.part_max[slot + l]; sum = a.part_sum[slot + l]; key = a.part_key[slot + l]; }
    for (int r = l + 16; r < a.runs; r += 16) {
      const float mr = a.part_max[slot + r];
      const double sr = a.part_sum[slot + r];
      const unsigned long long kr = a.part_key[slot + r];
      const float mn = fmaxf(m, mr);
      sum = rescaled_sum(sum, m, mn) + rescaled_sum(sr, mr, mn);
      m = mn;
      key = kr > key ? kr : key;
    }
    const float own = m;
    m = row16_max_f32(m);
    sum = row16_sum_f64(rescaled_sum(sum, own, m));
    key = row16_max_u64(key);
    if (l == 0) {
      const double lse = static_cast<double>(m) + log_of_sum(sum);
      if (key != 0ull) {
        a.target_token[row] = static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(key));
        if (a.target_prob) a.target_prob[row] = __expf(static_cast<float>(static_cast<double>(key_logit(key)) - lse));
      }
      if (!(fabs(lse) <= 1.7e308)) any_bad = 1;
    }
  }
  any_bad = __syncthreads_or(any_bad);
  if (threadIdx.x == 0) a.scan_status[b] = any_bad ? TALON_STATUS_BAD_ROW : 0u;
}

// One workgroup per sequence, one thread per node.  A node is on the accepted path iff every
// edge from the root down to it carries the target's greedy token of the edge's upper end;
// such nodes form one chain (siblings carry distinct tokens), one per depth.
__global__ __launch_bounds__(kThreads) void accept_kernel(talon_tree_state st, const int32_t* target_token,
                                                          const uint32_t* scan_status, int32_t* path,
                                                          int32_t* accept_len, int32_t* bonus_token) {
  static_assert(TALON_N_MAX <= kThreads, "one thread per node");
  __shared__ int s_parent[TALON_N_MAX];
  __shared__ int s_target[TALON_N_MAX];
  __shared__ unsigned char s_match[TALON_N_MAX];
  __shared__ int s_red[8];
  const int b = blockIdx.x;
  const int i = threadIdx.x;
  const int n = st.n_nodes[b];
  const size_t base = static_cast<size_t>(b) * st.N_pad;
  int tok = -1;
  if (i < n) {
    s_parent[i] = st.parent[base + i];
    s_target[i] = target_token[base + i];
    tok = st.token[base + i];
  }
  __syncthreads();
  if (i < n) s_match[i] = (i == 0) || (tok == s_target[s_parent[i]]);
  __syncthreads();
  bool valid = i < n;
  int steps = 0;   // depth of node i
  for (int j = i; valid && j > 0 && steps < TALON_N_MAX; ++steps) {
    valid = s_match[j] != 0;
    j = s_parent[j];
  }
  // the deepest valid node ends the path
  int key = valid ? ((steps << 16) | i) : -1;
  key = wave_max_i32(key);
  if ((i & 63) == 0) s_red[i >> 6] = key;
  __syncthreads();
  key = max(max(s_red[0], s_red[1]), max(s_red[2], s_red[3]));
  const int len = key >> 16;          // accepted draft tokens (the root is not counted)
  const int last = key & 0xFFFF;
  if (valid) path[base + steps] = i;
  if (i < st.N_pad && i > len) path[base + i] = -1;
  if (i == 0) {
    accept_len[b] = len;
    bonus_token[b] = s_target[last];
    if (scan_status[b] & TALON_STATUS_BAD_ROW) atomicOr(&st.status[b], TALON_STATUS_BAD_ROW);
  }
}

// Block (j, b) copies the K and V rows of the j-th accepted node of sequence b (all KV heads)
// to position prefix_len[b] + j of the prefix cache.
__global__ __launch_bounds__(kThreads) void compact_kv_kernel(const uint16_t* k_tree, const uint16_t* v_tree,
                                                              const int32_t* path, const int32_t* accept_len,
                                                              const int32_t* prefix_len, int32_t* new_prefix_len,
                                                              uint16_t* k_prefix, uint16_t* v_prefix, int N_pad, int Hkv,
                                                              int Dh, int capacity, int64_t sb, int64_t st_, int64_t sh) {
  const int j = blockIdx.x;
  const int b = blockIdx.y;
  const int len = accept_len[b];
  int L = prefix_len[b];
  L = L < 0 ? 0 : L;
  if (j == 0 && threadIdx.x == 0) {
    const int want = L + len + 1;
    new_prefix_len[b] = want < capacity ? want : capacity;
  }
  if (j > len || L + j >= capacity) return;
  const int node = path[static_cast<size_t>(b) * N_pad + j];
  if (node < 0 || node >= N_pad) return;
  const int cpr = Dh / 8;                       // 16-byte chunks per head row
  const int chunks = Hkv * cpr;
  const size_t src = (static_cast<size_t>(b) * N_pad + node) * Hkv * Dh;
  const int64_t dst = static_cast<int64_t>(b) * sb + static_cast<int64_t>(L + j) * st_;
  for (int c = threadIdx.x; c < 2 * chunks; c += kThreads) {
    const bool is_v = c >= chunks;
    const int cc = is_v ? c - chunks : c;
    const int h = cc / cpr, q = cc - h * cpr;
    const uint4 v = *reinterpret_cast<const uint4*>((is_v ? v_tree : k_tree) + src + static_cast<size_t>(h) * Dh + q * 8);
    *reinterpret_cast<uint4*>((is_v ? v_prefix : k_prefix) + dst + static_cast<int64_t>(h) * sh + q * 8) = v;
  }
}

}  // namespace

hipError_t launch_argmax(const ArgmaxArgs& a, int dtype, int B, hipStream_t s) {
  const dim3 grid(a.N_pad * a.runs, B);
  if (dtype == TALON_DTYPE_F32) hipLaunchKernelGGL(argmax_scan_kernel<4>, grid, dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(argmax_scan_kernel<8>, grid, dim3(kThreads), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(argmax_merge_kernel, dim3(B), dim3(kMergeThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_accept(const talon_tree_state& st, const int32_t* target_token, const uint32_t* scan_status,
                         int32_t* path, int32_t* accept_len, int32_t* bonus_token, hipStream_t s) {
  hipLaunchKernelGGL(accept_kernel, dim3(st.B), dim3(kThreads), 0, s, st, target_token, scan_status, path, accept_len,
                     bonus_token);
  return hipGetLastError();
}

hipError_t launch_compact_kv(const uint16_t* k_tree, const uint16_t* v_tree, const int32_t* path, const int32_t* accept_len,
                             const int32_t* prefix_len, int32_t* new_prefix_len, uint16_t* k_prefix, uint16_t* v_prefix,
                             int B, int N_pad, int Hkv, int Dh, int capacity, int64_t sb, int64_t st_, int64_t sh,
                             hipStream_t s) {
  hipLaunchKernelGGL(compact_kv_kernel, dim3(N_pad, B), dim3(kThreads), 0, s, k_tree, v_tree, path, accept_len, prefix_len,
                     new_prefix_len, k_prefix, v_prefix, N_pad, Hkv, Dh, capacity, sb, st_, sh);
  return hipGetLastError();
}

}  // namespace talon
