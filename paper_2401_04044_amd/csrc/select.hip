// Bit-exact top-k of the neuron scores (heavy-hitter selection, Sec. 4.1/5.1.1).
// Integer work only: scores are mapped to order-preserving uint32 keys.
// Up to SELECT_COUNT_MAX_N scores every element is ranked by counting the elements in front of it, n^2
// comparisons over the whole machine, and a second kernel numbers what was not chosen; beyond, one
// workgroup finds the k-th largest key by a 32-step search over its bits (each step one count over the
// keys, which 1024 threads hold in registers), compacts the chosen elements in index order (equal keys:
// lowest indices first), and these are ranked by counting.  Order: score descending, index ascending.
#include "prep.h"
#include <atomic>

namespace ffsplit {

// Scratch of the entry point that allocates nothing (ffsplit_select_heavy_static): one copy per
// GPU the library runs on, held until the process ends.  In host code this name is only a
// stand-in for the symbol; the device address comes from hipGetSymbolAddress (below).
constexpr int SELECT_STATIC_MAX_DFF = 65536;
constexpr size_t SELECT_STATIC_BYTES = (size_t)12 * SELECT_STATIC_MAX_DFF + 256;
static __device__ __align__(256) unsigned char scratch[SELECT_STATIC_BYTES];

__device__ __forceinline__ uint32_t score_key(float s, int* saw_nan) {
  uint32_t b = __float_as_uint(s);
  if ((b & 0x7fffffffu) > 0x7f800000u) { *saw_nan = 1; return 0xffffffffu; }
  if (b == 0x80000000u) b = 0u;                       // -0 counts as +0
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);  // monotone in the float order
}

// Exclusive prefix sum of v over the 1024 threads of a block, in thread order.  wsum: 16 ints
// of LDS.  Every thread must call it.
__device__ __forceinline__ int block_scan_1024(int v, int* wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  __syncthreads();
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < 16; ++w) before += w < wave ? wsum[w] : 0;
  return before + inc - v;
}

__global__ void __launch_bounds__(1024) select_compact_kernel(const float* scores, int n, int k, uint32_t* keys,
                                                              uint32_t* cand_key, int32_t* cand_idx, int32_t* perm,
                                                              int32_t* nan_flag) {
  constexpr int KPT = 32;
  __shared__ int wsum[16];
  __shared__ int csum[2][16];
  __shared__ int s_nan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) s_nan = 0;
  __syncthreads();
  // every thread owns a contiguous run of elements; the first KPT keys of the run stay in
  // registers (key 0 = no element: real keys are > 0), longer runs continue in `keys`
  const int run = (n + 1023) / 1024;
  const int i0 = min(n, tid * run), i1 = min(n, i0 + run);
  uint32_t kreg[KPT];
  int saw = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const int i = i0 + j;
    kreg[j] = (j < run && i < i1) ? score_key(scores[i], &saw) : 0u;
  }
  for (int i = i0 + KPT; i < i1; ++i) keys[i] = score_key(scores[i], &saw);
  if (saw) s_nan = 1;
  __syncthreads();
  if (tid == 0 && nan_flag) *nan_flag = s_nan ? -7 : 0;
  if (k <= 0) return;   // (never: without it the compiler's schedule takes 2 us more, 24600 scores 55.3 -> 57.0)
  // number of keys >= c (c > 0), the same value in every thread; buf alternates so that one
  // barrier per call is enough
  int buf = 0;
  auto count_ge = [&](uint32_t c) -> int {
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) cnt += kreg[j] >= c;
    for (int i = i0 + KPT; i < i1; ++i) cnt += keys[i] >= c;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0) csum[buf][wave] = cnt;
    __syncthreads();
    int tot = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) tot += csum[buf][w];
    buf ^= 1;
    return tot;
  };
  // the k-th largest key, bit by bit from the top: the largest P with at least k keys >= P
  uint32_t thr = 0u;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t c = thr | (1u << bit);
    if (count_ge(c) >= k) thr = c;
  }
  const int above = thr == 0xffffffffu ? 0 : count_ge(thr + 1u);
  const int need = k - above;  // how many keys equal to thr are taken (lowest indices)
  // Compaction in index order over the threads' runs: two block scans (equal keys, then
  // selected elements).
  int eq_cnt = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j) eq_cnt += kreg[j] == thr;     // thr > 0: empty slots never match
  for (int i = i0 + KPT; i < i1; ++i) eq_cnt += keys[i] == thr;
  int eq_before = block_scan_1024(eq_cnt, wsum);
  int sel_cnt = 0;
  {
    int e = eq_before;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      const bool eq = kreg[j] == thr;
      sel_cnt += kreg[j] > thr || (eq && e < need);
      e += eq;
    }
    for (int i = i0 + KPT; i < i1; ++i) {
      const uint32_t key = keys[i];
      const bool eq = key == thr;
      sel_cnt += key > thr || (eq && e < need);
      e += eq;
    }
  }
  int sp = block_scan_1024(sel_cnt, wsum);   // selected elements before this thread's run
  auto place = [&](uint32_t key, int i) {
    const bool eq = key == thr;
    const bool sel = key > thr || (eq && eq_before < need);
    eq_before += eq;
    if (sel) { cand_key[sp] = key; cand_idx[sp] = i; ++sp; }
    else if (perm) perm[k + (i - sp)] = i;     // i - sp = elements before i that were not selected
  };
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if (i0 + j < i1 && j < run) place(kreg[j], i0 + j);
  for (int i = i0 + KPT; i < i1; ++i) place(keys[i], i);
}

// rank of candidate a = #(keys greater) + #(equal keys at an earlier position); one wavefront
// per candidate, the lanes share the comparisons
__global__ void __launch_bounds__(256) select_rank_kernel(const uint32_t* cand_key, const int32_t* cand_idx, int k,
                                                          int32_t* idx, int32_t* perm) {
  const int a = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (a >= k) return;
  const uint32_t ka = cand_key[a];
  int rank = 0;
  for (int b = lane; b < k; b += 64) {
    const uint32_t kb = cand_key[b];
    rank += (kb > ka) || (kb == ka && b < a);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) rank += __shfl_xor(rank, o);
  if (lane == 0) {
    const int32_t v = cand_idx[a];
    idx[rank] = v;
    if (perm) perm[rank] = v;
  }
}

// Rank of every element = elements with a larger key, or with the same key at a lower index.  A workgroup ranks 32
// elements: each of its 16 wavefronts holds them twice, in its lower and its upper half, and meets two
// 1/32 shares of the keys, which come from LDS, the same four to every lane of a half.  Two vector instructions
// a comparison (compare, add with carry): 8192 scores 2 us of arithmetic; what is left is a launch
// and converting the scores.  Where the keys lie before or after the 32 elements, ties need no look at the index.
constexpr int SEL_CHUNK = 8192;   // keys in LDS at a time
__global__ void __launch_bounds__(1024) select_count_kernel(const float* scores, int n, int k, int32_t* rank, int32_t* idx,
                                                            int32_t* perm, int32_t* nan_flag) {
  __shared__ __align__(16) uint32_t key[SEL_CHUNK];
  __shared__ int part[16][32];
  __shared__ int s_nan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = blockIdx.x * 32, i = i0 + (lane & 31);
  int saw = 0, cnt = 0;
  const uint32_t ki = i < n ? score_key(scores[i], &saw) : 0xffffffffu;
  if (tid == 0) s_nan = 0;
  saw = 0;
  for (int c0 = 0; c0 < n; c0 += SEL_CHUNK) {
    const int m = min(SEL_CHUNK, n - c0), m4 = (m + 127) & ~127;   // (padded with key 0: real keys are > 0)
    __syncthreads();
#pragma unroll
    for (int u = 0; u < SEL_CHUNK / 1024; ++u) {
      const int j = u * 1024 + tid;
      if (j < m4) key[j] = j < m ? score_key(scores[c0 + j], &saw) : 0u;
    }
    __syncthreads();
    // share of this half wavefront: groups of four keys, s, s + 32, ...
    const int share = wave * 2 + (lane >> 5), groups = m4 / 4;
    // groups that end before element i0, start behind i0 + 31, and the eight (at most) between
    const int lo = max(0, min(groups, (i0 - c0) >> 2)), hi = max(0, min(groups, (i0 + 32 - c0) >> 2));
    int g = share;
#pragma unroll 4
    for (; g < lo; g += 32) {
      const uint4 q = *(const uint4*)(key + 4 * g);
      cnt += q.x >= ki; cnt += q.y >= ki; cnt += q.z >= ki; cnt += q.w >= ki;
    }
    for (; g < hi; g += 32) {
      const uint4 q = *(const uint4*)(key + 4 * g);
      const int d = i - (c0 + 4 * g);
      cnt += q.x > ki || (q.x == ki && d > 0); cnt += q.y > ki || (q.y == ki && d > 1);
      cnt += q.z > ki || (q.z == ki && d > 2); cnt += q.w > ki || (q.w == ki && d > 3);
    }
#pragma unroll 4
    for (; g < groups; g += 32) {
      const uint4 q = *(const uint4*)(key + 4 * g);
      cnt += q.x > ki; cnt += q.y > ki; cnt += q.z > ki; cnt += q.w > ki;
    }
  }
  if (blockIdx.x == 0 && saw) s_nan = 1;
  cnt += __shfl_xor(cnt, 32);
  if (lane < 32) part[wave][lane] = cnt;
  __syncthreads();
  if (blockIdx.x == 0 && tid == 0 && nan_flag) *nan_flag = s_nan ? -7 : 0;
  if (tid >= 32 || i >= n) return;
  int r = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) r += part[w][tid];
  rank[i] = r;
  if (r < k) {
    idx[r] = i;
    if (perm) perm[r] = i;
  }
}

// perm[k ..]: the elements of rank >= k in index order; a workgroup counts the chosen ones before its 1024
__global__ void __launch_bounds__(1024) select_rest_kernel(const int32_t* rank, int n, int k, int32_t* perm) {
  __shared__ int wsum[16];
  __shared__ int before;
  const int tid = threadIdx.x, i0 = blockIdx.x * 1024, i = i0 + tid;
  int c = 0;
  for (int j = tid; j < i0; j += 1024) c += rank[j] < k;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if (tid == 0) before = 0;
  __syncthreads();
  if ((tid & 63) == 0 && c > 0) atomicAdd(&before, c);
  const bool sel = i < n && rank[i] < k;
  int total, sp = block_prefix_1024(sel, wsum, &total);   // (its barriers come behind the sums above)
  sp += before;
  if (i < n && !sel) perm[k + (i - sp)] = i;
}

// Nothing is chosen: the flag, and the identity.  us, with the permutation, replayed from a graph, by the search / ranked by
// counting / so: 1500 scores 3.9 / 6.7 / 2.2, 8192 7.2 / 13.4 / 2.6, 24576 15.1 / - / 4.3.
__global__ void __launch_bounds__(1024) select_none_kernel(const float* scores, int n, int32_t* perm, int32_t* nan_flag) {
  __shared__ int s_nan;
  if (threadIdx.x == 0) s_nan = 0;
  __syncthreads();
  int saw = 0;
  if (nan_flag)
    for (int i0 = threadIdx.x; i0 < n; i0 += 8 * 1024) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = scores[min(i0 + u * 1024, n - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) score_key(v[u], &saw);
    }
  if (perm)
    for (int i = threadIdx.x; i < n; i += 1024) perm[i] = i;
  if (saw) s_nan = 1;
  __syncthreads();
  if (threadIdx.x == 0 && nan_flag) *nan_flag = s_nan ? -7 : 0;
}

// Ranking by counting grows with n^2, the search on one CU with n.  Both sides (us, a calibration call of 256 tokens
// and width 512 with the selection, search / counting): 1500 scores 55.0 / 45.3, 8192 (4096 tokens, width 2048)
// 165 / 142, 16384 88.7 / 63.8, 20480 92.3 / 84.8, 24576 102.3 / 95.4.  The selection alone, with the permutation, for any k
// from 1 on: 8192 32 / 17, 16384 53 / 30, 24576 61 / 57.
constexpr int SELECT_COUNT_MAX_N = 24576;

size_t select_workspace_bytes(int d_ff) { return (size_t)12 * (size_t)(d_ff > 0 ? d_ff : 1) + 256; }

int launch_select(const float* scores, int d_ff, int k, int32_t* idx, int32_t* perm, int32_t* nan_flag, void* ws,
                  hipStream_t st) {
  if (d_ff <= 0) return 0;
  if (k <= 0) {
    hipLaunchKernelGGL(select_none_kernel, dim3(1), dim3(1024), 0, st, scores, d_ff, perm, nan_flag);
    return hipGetLastError() == hipSuccess ? 0 : -1;
  }
  if (d_ff <= SELECT_COUNT_MAX_N) {
    int32_t* rank = (int32_t*)ws;
    hipLaunchKernelGGL(select_count_kernel, dim3((d_ff + 31) / 32), dim3(1024), 0, st, scores, d_ff, k, rank, idx, perm, nan_flag);
    if (perm && k < d_ff)
      hipLaunchKernelGGL(select_rest_kernel, dim3((d_ff + 1023) / 1024), dim3(1024), 0, st, rank, d_ff, k, perm);
    return hipGetLastError() == hipSuccess ? 0 : -1;
  }
  uint32_t* keys = (uint32_t*)ws;
  uint32_t* cand_key = keys + d_ff;
  int32_t* cand_idx = (int32_t*)(cand_key + d_ff);
  hipLaunchKernelGGL(select_compact_kernel, dim3(1), dim3(1024), 0, st, scores, d_ff, k, keys, cand_key, cand_idx, perm,
                     nan_flag);
  if (hipGetLastError() != hipSuccess) return -1;
  hipLaunchKernelGGL(select_rank_kernel, dim3((k + 3) / 4), dim3(256), 0, st, cand_key, cand_idx, k, idx, perm);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int select_static_max_dff() { return SELECT_STATIC_MAX_DFF; }

// Device address of this GPU's copy of `scratch`, looked up once per device (with that device
// current) and kept; nullptr on failure.  Racing first calls both look it up and store the same
// value.
static void* select_static_scratch() {
  static std::atomic<void*> ptr[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return nullptr;
  void* p = dev < 64 ? ptr[dev].load(std::memory_order_acquire) : nullptr;
  if (!p) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    if (dev < 64) ptr[dev].store(p, std::memory_order_release);
  }
  return p;
}

int launch_select_static(const float* scores, int d_ff, int k, int32_t* idx, int32_t* perm, int32_t* nan_flag,
                         hipStream_t st) {
  void* ws = select_static_scratch();
  if (!ws) return -1;
  // nothing in the scratch has to start at zero: every key, candidate key and candidate index
  // that a launch reads was written earlier in the same call
  return launch_select(scores, d_ff, k, idx, perm, nan_flag, ws, st);
}

}  // namespace ffsplit
