// One-off and small kernels around the GEMMs: zero fill, permuted transposes
// (neuron gather + packing of Eq. 2's partition), the fixed-order reduction of
// the score partials and the W2 row-norm / score finalisation of Eq. 3.
#include "prep.h"

namespace ffsplit {

__global__ void fill_zero_kernel(uint4* p, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

int launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return 0;
  const size_t n16 = bytes / 16;  // callers keep sizes a multiple of 16
  int blocks = (int)((n16 + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, st, (uint4*)p, n16);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// dst[f(n)][coff + c] = src[cmap(c)][nmap(n)],  n < n_count, c < c_count.
template <typename T>
__global__ void permute_transpose_kernel(const PermArgs a) {
  __shared__ T tile[32][33];
  const int n0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
  const int tx = threadIdx.x, ty = threadIdx.y;
  const T* src = (const T*)a.src;
  T* dst = (T*)a.dst;
  const int n = n0 + tx;
  int64_t scol = -1;
  if (n < a.n_count) scol = a.nmap ? a.nmap[a.nmap_off + n] : n;
  for (int cc = ty; cc < 32; cc += 8) {
    const int c = c0 + cc;
    T v = 0;
    if (c < a.c_count && scol >= 0) {
      const int64_t srow = a.cmap ? a.cmap[a.cmap_off + c] : c;
      v = src[srow * a.lds + scol];
    }
    tile[cc][tx] = v;
  }
  __syncthreads();
  const int c = c0 + tx;
  for (int nn = ty; nn < 32; nn += 8) {
    const int nq = n0 + nn;
    if (nq < a.n_count && c < a.c_count) {
      int64_t drow;
      if (a.glu_mode == 0) drow = a.row_off + nq;
      else drow = a.row_off + (int64_t)(nq >> 5) * 64 + (nq & 31) + (a.glu_mode == 2 ? 32 : 0);
      const int64_t dcol = a.coff + c;
      dst[drow * a.ldd + dcol] = tile[tx][nn];
    }
  }
}

// The same for 16-bit elements into the tiled layout: 64 columns n x 64 rows c per workgroup through
// LDS, 16-byte stores (a wavefront writes two runs of 512 bytes).  The element-wise form above moved
// 67 MB (2048 x 8192 in and out) in 28 us.  Where a row is 16-byte aligned and the columns
// are not permuted (VEC) the loads are 16 bytes too; elsewhere they are single elements, 32 rows per
// workgroup: small matrices are bound by their latency, and with 64 rows, sixteen loads a thread, a
// 512 x 1327 one took 7.8 us, longer than element-wise (4.6 us and its share of a fill).
// Zeros are written up to n_pad and c_pad (at least to the end of a chunk).
template <bool VEC>
__global__ void __launch_bounds__(256) permute_transpose_tiled_kernel(const PermArgs a) {
  constexpr int CT = VEC ? 64 : 32;   // rows c per workgroup
  constexpr int LD = 72;   // elements per LDS row: 16-byte aligned, rows shifted by four banks
  __shared__ __align__(16) uint16_t tile[CT * LD];
  const int n0 = blockIdx.x * 64, c0 = blockIdx.y * CT, t = threadIdx.x;
  const uint16_t* src = (const uint16_t*)a.src;
  if (VEC) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int cc = i * 32 + t / 8, n = n0 + (t & 7) * 8, c = c0 + cc;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (c < a.c_count && n < a.n_count) {
        const int64_t srow = a.cmap ? a.cmap[a.cmap_off + c] : c;
        v = *(const uint4*)(src + srow * a.lds + n);
      }
      *(uint4*)(tile + cc * LD + (t & 7) * 8) = v;
    }
  } else {
    const int n = n0 + (t & 63);
    // (unconditional loads of clamped indices: none waits for another)
    const int nc = min(n, a.n_count - 1);
    const int64_t scol = a.nmap ? a.nmap[a.nmap_off + nc] : nc;
    uint16_t v[CT / 4];
#pragma unroll
    for (int i = 0; i < CT / 4; ++i) {
      const int cc = min(c0 + i * 4 + (t >> 6), a.c_count - 1);
      v[i] = src[(int64_t)(a.cmap ? a.cmap[a.cmap_off + cc] : cc) * a.lds + scol];
    }
#pragma unroll
    for (int i = 0; i < CT / 4; ++i) {
      const int c = i * 4 + (t >> 6);
      tile[c * LD + (t & 63)] = (c0 + c < a.c_count && n < a.n_count) ? v[i] : (uint16_t)0;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < CT / 32; ++i) {
    const int nn = t & 63, c8 = (i * 4 + (t >> 6)) * 8, nq = n0 + nn;
    if (nq >= max(a.n_count, a.n_pad) || c0 + c8 >= max(a.c_count, a.c_pad)) continue;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = (uint32_t)tile[(c8 + 2 * e) * LD + nn] | ((uint32_t)tile[(c8 + 2 * e + 1) * LD + nn] << 16);
    int64_t drow;
    if (a.glu_mode == 0) drow = a.row_off + nq;
    else drow = a.row_off + (int64_t)(nq >> 5) * 64 + (nq & 31) + (a.glu_mode == 2 ? 32 : 0);
    const int64_t dcol = a.coff + c0 + c8;
    *(uint4*)((uint16_t*)a.dst + ((drow >> 5) * (a.ldd >> 4) + (dcol >> 4)) * 512 + ((dcol >> 3) & 1) * 256 + (drow & 31) * 8) =
        make_uint4(w[0], w[1], w[2], w[3]);
  }
}

int launch_permute_transpose(const PermArgs& a, int esize, hipStream_t st) {
  if (a.n_count <= 0 || a.c_count <= 0) return 0;
  if (esize == 2 && a.dst_tiled && (a.coff & 7) == 0) {
    const int nn = a.n_pad > a.n_count ? a.n_pad : a.n_count, cn = a.c_pad > a.c_count ? a.c_pad : a.c_count;
    const bool vec = a.nmap == nullptr && (a.lds & 7) == 0 && (a.n_count & 7) == 0 && ((uintptr_t)a.src & 15) == 0;
    const dim3 grid((nn + 63) / 64, vec ? (cn + 63) / 64 : (cn + 31) / 32);
    if (vec) hipLaunchKernelGGL(permute_transpose_tiled_kernel<true>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(permute_transpose_tiled_kernel<false>, grid, dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
  }
  if (esize != 4) return -1;   // 16-bit matrices are always tiled
  dim3 grid((a.n_count + 31) / 32, (a.c_count + 31) / 32), block(32, 8);
  hipLaunchKernelGGL(permute_transpose_kernel<uint32_t>, grid, block, 0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// acc[j] += sum_t part_s2[t][j] ; acc[d_ff + j] += sum_t part_s1[t][j]  (t ascending)
__global__ void reduce_partials_kernel(const float* part_s2, const float* part_s1, int tiles, int n_out,
                                       int d_ff, float* acc) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d_ff) return;
  float s2 = 0.f, s1 = 0.f;
  for (int t = 0; t < tiles; ++t) {
    s2 += part_s2[(int64_t)t * n_out + j];
    s1 += part_s1[(int64_t)t * n_out + j];
  }
  acc[j] += s2;
  acc[d_ff + j] += s1;
}

int launch_reduce_partials(const float* p2, const float* p1, int tiles, int n_out, int d_ff, float* acc,
                           hipStream_t st) {
  if (d_ff <= 0) return 0;
  hipLaunchKernelGGL(reduce_partials_kernel, dim3((d_ff + 255) / 256), dim3(256), 0, st, p2, p1, tiles, n_out,
                     d_ff, acc);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// n2 = sum_c W2[j,c]^2 by one wavefront per neuron (lane-strided partial sums and a fixed butterfly of
// wavefront shuffles), then the score of the given kind.  Bound by reading W2 once.
// ADDS: the call's partial sums of the activations are added to the accumulator first (reduce_partials, requested ahead of
// the rows; as a launch of its own 6.8 us of latency); a workgroup takes 16 neurons for it, its wavefronts two each, eight
// loads in flight.  Without, a neuron a wavefront, twice the wavefronts: bf16 8192 x 8192 26.4 -> 22.1 us, 24576 neurons of 512
// 6.2 -> 5.7.
struct ScoreArgs {
  const void* W2;
  int d_model, d_ff;
  float* acc;
  const float *part_s2, *part_s1;
  int tiles, n_out;
  float t_total;
  int kind;
  float* scores;
};
template <bool BF16, bool ADDS>
__global__ void __launch_bounds__(ADDS ? 512 : 256) finalize_scores_kernel(const ScoreArgs a) {
  __shared__ float s_acc[2][16];
  constexpr int PT = 8, R = ADDS ? 2 : 1;   // neurons a wavefront
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), j0 = blockIdx.x * (ADDS ? 16 : 4);
  // thread (which sum, neuron): tiles in ascending order, PT in flight
  const int which = threadIdx.x >> 4, jp = j0 + (threadIdx.x & 15);
  const bool adds = ADDS && threadIdx.x < 32 && jp < a.d_ff;
  const float* part = (which ? a.part_s1 : a.part_s2) + jp;
  float s = 0.f, old = 0.f;
  if (adds) {
    old = a.acc[which * a.d_ff + jp];
    for (int t = 0; t < a.tiles; t += PT) {
      float v[PT];
#pragma unroll
      for (int u = 0; u < PT; ++u) v[u] = part[(int64_t)min(t + u, a.tiles - 1) * a.n_out];
#pragma unroll
      for (int u = 0; u < PT; ++u)
        if (t + u < a.tiles) s += v[u];
    }
  }
  float n2[R] = {};
  if (a.kind != 2) {
    constexpr int E = BF16 ? 8 : 4, ESZ = BF16 ? 2 : 4, U = ADDS ? 4 : 1;   // 16 bytes a lane, U loads of a row at once
    const char* row[R];
#pragma unroll
    for (int i = 0; i < R; ++i) row[i] = (const char*)a.W2 + (int64_t)min(j0 + wave * R + i, a.d_ff - 1) * a.d_model * ESZ;
    for (int c0 = lane * E; c0 < a.d_model; c0 += 64 * E * U) {
      uint4 v[U][R];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * 64 * E;
#pragma unroll
        for (int i = 0; i < R; ++i) v[u][i] = c < a.d_model ? *(const uint4*)(row[i] + (int64_t)c * ESZ) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const uint32_t w[4] = {v[u][i].x, v[u][i].y, v[u][i].z, v[u][i].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (BF16) {
              const float lo = __uint_as_float(w[e] << 16), hi = __uint_as_float(w[e] & 0xffff0000u);
              n2[i] = fmaf(lo, lo, n2[i]);
              n2[i] = fmaf(hi, hi, n2[i]);
            } else {
              n2[i] = fmaf(__uint_as_float(w[e]), __uint_as_float(w[e]), n2[i]);
            }
          }
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) n2[i] += __shfl_xor(n2[i], o);
  }
  if (adds) {
    a.acc[which * a.d_ff + jp] = old + s;
    s_acc[which][threadIdx.x & 15] = old + s;
  }
  if (ADDS) __syncthreads();
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int jl = wave * R + i, j = j0 + jl;
    if (lane != 0 || j >= a.d_ff) continue;
    const float sum = ADDS ? s_acc[a.kind == 1][jl] : a.acc[(a.kind == 1 ? a.d_ff : 0) + j];
    float v;
    if (a.kind == 0) v = sum * n2[i];
    else if (a.kind == 1) v = (sum / fmaxf(a.t_total, 1.f)) * sqrtf(n2[i]);
    else v = sum;
    a.scores[j] = v + 0.f;
  }
}

int launch_finalize_scores(const void* W2, int bf16, int d_model, int d_ff, float* acc, const float* p2, const float* p1,
                           int tiles, int n_out, float t_total, int kind, float* scores, hipStream_t st) {
  if (d_ff <= 0) return 0;
  const ScoreArgs a = {W2, d_model, d_ff, acc, p2, p1, tiles, n_out, t_total, kind, scores};
  const dim3 grid(tiles > 0 ? (d_ff + 15) / 16 : (d_ff + 3) / 4), blk(tiles > 0 ? 512 : 256);
  if (tiles > 0) {
    if (bf16) hipLaunchKernelGGL((finalize_scores_kernel<true, true>), grid, blk, 0, st, a);
    else hipLaunchKernelGGL((finalize_scores_kernel<false, true>), grid, blk, 0, st, a);
  } else {
    if (bf16) hipLaunchKernelGGL((finalize_scores_kernel<true, false>), grid, blk, 0, st, a);
    else hipLaunchKernelGGL((finalize_scores_kernel<false, false>), grid, blk, 0, st, a);
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ------------------------------------------------------------------ stack harness kernels

// out[t, :] = x[t, :] / sqrt(mean(x[t, :]^2) + eps), one workgroup per token, fp32 sums added in
// a fixed order (lane-strided partials, wavefront butterfly, then the four wavefronts in order).
template <bool BF16>
__global__ void __launch_bounds__(256) token_rmsnorm_kernel(const float* x, int d, float eps, void* out) {
  __shared__ float wsum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* row = x + (int64_t)blockIdx.x * d;
  // rows of up to 8192 elements stay in registers between the sum and the scaling (one read
  // of the stream); longer rows are read a second time
  constexpr int NV = 8;
  float4 v[NV];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = tid * 4 + i * 1024;
    v[i] = c < d ? *(const float4*)(row + c) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    s = fmaf(v[i].x, v[i].x, s); s = fmaf(v[i].y, v[i].y, s); s = fmaf(v[i].z, v[i].z, s); s = fmaf(v[i].w, v[i].w, s);
  }
  for (int c = tid * 4 + NV * 1024; c < d; c += 1024) {
    const float4 w = *(const float4*)(row + c);
    s = fmaf(w.x, w.x, s); s = fmaf(w.y, w.y, s); s = fmaf(w.z, w.z, s); s = fmaf(w.w, w.w, s);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) wsum[wave] = s;
  __syncthreads();
  const float tot = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
  auto emit = [&](int c, const float4& w) {
    if (BF16) {
      *(uint2*)((bf16_t*)out + (int64_t)blockIdx.x * d + c) =
          make_uint2(pack_bf16x2(w.x * inv, w.y * inv), pack_bf16x2(w.z * inv, w.w * inv));
    } else {
      *(float4*)((float*)out + (int64_t)blockIdx.x * d + c) = make_float4(w.x * inv, w.y * inv, w.z * inv, w.w * inv);
    }
  };
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = tid * 4 + i * 1024;
    if (c < d) emit(c, v[i]);
  }
  for (int c = tid * 4 + NV * 1024; c < d; c += 1024) emit(c, *(const float4*)(row + c));
}

int launch_token_rmsnorm(const float* x, int64_t T, int d, float eps, int bf16, void* out, hipStream_t st) {
  if (T <= 0) return 0;
  if (bf16) hipLaunchKernelGGL(token_rmsnorm_kernel<true>, dim3((unsigned)T), dim3(256), 0, st, x, d, eps, out);
  else hipLaunchKernelGGL(token_rmsnorm_kernel<false>, dim3((unsigned)T), dim3(256), 0, st, x, d, eps, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// packed[i] = b1[idx[i]] for i < k, 0 up to kp; packed[kp + i] = b1[rest[i]] for i < m, 0 up to kp + mp
template <typename T>
__global__ void pack_neuron_bias_kernel(const T* b1, const int32_t* idx, const int32_t* rest, int k, int kp, int m,
                                        int mp, float* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kp + mp) return;
  int src = -1;
  if (i < k) src = idx[i];
  else if (i >= kp && i - kp < m) src = rest[i - kp];
  float v = 0.f;
  if (src >= 0) {
    if (sizeof(T) == 2) v = bf16_to_f32((bf16_t)b1[src]);
    else v = __uint_as_float((uint32_t)b1[src]);
  }
  out[i] = v;
}

int launch_pack_neuron_bias(const void* b1, int bf16, const int32_t* idx, const int32_t* rest, int k, int kp, int m,
                            int mp, float* out, hipStream_t st) {
  const int n = kp + mp;
  if (n <= 0) return 0;
  if (bf16) hipLaunchKernelGGL(pack_neuron_bias_kernel<uint16_t>, dim3((n + 255) / 256), dim3(256), 0, st,
                               (const uint16_t*)b1, idx, rest, k, kp, m, mp, out);
  else hipLaunchKernelGGL(pack_neuron_bias_kernel<uint32_t>, dim3((n + 255) / 256), dim3(256), 0, st,
                          (const uint32_t*)b1, idx, rest, k, kp, m, mp, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ffsplit
