// Rank-r factors of the remainder matrices, computed on the device so that a split can be
// built without a host factorisation (Sec. 4.2 / 5.1.1: a low-rank decomposition of U2 and V2,
// each on its own).  Instead of a full SVD: the randomised range finder of Halko, Martinsson
// and Tropp (2011, Alg. 4.1) on the d_model side of every matrix,
//     Z [d, m] (W1[:, rest], Wg[:, rest] or W2[rest, :]^T),  Y^T = Omega Z^T  [r, d],
//     B^T = orthonormal rows spanning the rows of Y^T,       C = B^T Z  [r, m],
// so that Z ~= B C.  Omega [r, m] is a counter-based Rademacher matrix (the same signs on any
// machine).  The rows of Y^T are orthonormalised by an odd matrix iteration for the polar factor,
// X <- (a I + b X X^T + c (X X^T)^2) X from X = Y^T / ||Y||_F (polar.hip), which consists of products only.
//
// Precision and where the work runs.  The sketch of bf16 weights has exact products (bf16 times +-1)
// and fp32 sums, so it is a product for the bf16 matrix cores; the projection takes the fp32 basis
// as three bf16 terms (8 + 8 + 8 bits, all of it) against the bf16 weights, again exact products
// and fp32 sums.  The iteration is fp32 throughout, the matrices of a layer side by side in
// one launch.  fp32 weights are gathered and multiplied in fp32.
#include "factor.h"
#include "polar.h"
#include "prep.h"
#include <algorithm>

namespace ffsplit {

namespace {

__device__ __forceinline__ uint32_t fmix32(uint32_t h) {   // finaliser of the public MurmurHash3
  h ^= h >> 16; h *= 0x85EBCA6Bu; h ^= h >> 13; h *= 0xC2B2AE35u; h ^= h >> 16;
  return h;
}

// fp32 weights: Z [d, m4] and / or Zt [m4, d] (zero in the padding columns):
// down = 0: Z[c][j] = W[c][rest[j]] (W [d, d_ff]);  down = 1: Z[c][j] = W[rest[j]][c] (W [d_ff, d])
__global__ void gather_z_kernel(const float* W, int d, int d_ff, const int32_t* rest, int m, int m4, int down, float* Z,
                                float* Zt) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)d * m4) return;
  // consecutive threads along the contiguous side of what is written
  const int c = Z ? (int)(id / m4) : (int)(id % d), j = Z ? (int)(id % m4) : (int)(id / d);
  float v = 0.f;
  if (j < m) {
    const int n = rest[j];
    v = down ? W[(int64_t)n * d + c] : W[(int64_t)c * d_ff + n];
  }
  if (Z) Z[id] = v;
  else Zt[id] = v;
}

// fp32: Omega [r4, m4]: entry (i, j) = +-1 from the top bit of fmix32(index * 0x9E3779B1 + key),
// index = i * m + j; zero in the padding
__global__ void rademacher_kernel(float* Om, int r, int m, int r4, int m4, uint32_t key) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)r4 * m4) return;
  const int i = (int)(id / m4), j = (int)(id % m4);
  float v = 0.f;
  if (i < r && j < m) {
    const uint32_t h = fmix32((uint32_t)(i * m + j) * 0x9E3779B1u + key);
    v = (h >> 31) ? -1.f : 1.f;
  }
  Om[id] = v;
}

// the same test matrix in bf16 in the tiled layout [r32, Kp] (K = m), zero in the padding; one
// wavefront per column block, walking down the row blocks
__global__ void __launch_bounds__(256) rademacher_tiled_kernel(uint16_t* Om, int r, int m, int r32, int kp, uint32_t key) {
  const int kb = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (kb * 16 >= kp) return;
  const int k0 = kb * 16 + (lane >> 5) * 8;
  for (int rb = blockIdx.y; rb < r32 / 32; rb += gridDim.y) {
    const int i = rb * 32 + (lane & 31);
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      uint32_t v = 0;
      if (i < r && k0 + e < m) v = (fmix32((uint32_t)(i * m + k0 + e) * 0x9E3779B1u + key) >> 31) ? 0xBF80u : 0x3F80u;
      w[e >> 1] = (e & 1) ? (w[e >> 1] | (v << 16)) : v;
    }
    *(uint4*)(Om + (((int64_t)rb * (kp / 16) + kb) * 64 + lane) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// dst (tiled [., ldd], 16-bit) row i, column j = src[row(i)][col(j)] with one of the two mapped by
// `rest`: rows (by_rows) or columns.  rows x cols valid, zeros up to the padding.
// 32 rows x 64 columns per workgroup through LDS.
__global__ void __launch_bounds__(256) gather_tiled_kernel(const uint16_t* src, int64_t lds, const int32_t* rest, int by_rows,
                                                           int rows, int cols, int cols_pad, uint16_t* dst) {
  constexpr int LD = 72;
  __shared__ __align__(16) uint16_t tile[32 * LD];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 64, t = threadIdx.x, l = t & 63;
  if (by_rows) {   // (lds a multiple of 8: 16 bytes a thread, 26 -> 12 us for 7946 x 2048)
    const int r = r0 + (t >> 3), c = c0 + (t & 7) * 8;
    uint4 w = make_uint4(0, 0, 0, 0);
    if (r < rows && c < cols) w = *(const uint4*)(src + (int64_t)rest[r] * lds + c);
    *(uint4*)(tile + (t >> 3) * LD + (t & 7) * 8) = w;
    __syncthreads();
    const int row = t & 31, c8 = (t >> 5) * 8;
    if (c0 + c8 >= cols_pad) return;
    *(uint4*)(dst + (((int64_t)blockIdx.y * (cols_pad / 16) + (c0 + c8) / 16) * 64 + ((c8 >> 3) & 1) * 32 + row) * 8) =
        *(const uint4*)(tile + row * LD + c8);
    return;
  }
  const int c = c0 + l;
  const int64_t sc = c < cols ? rest[c] : -1;
  uint16_t v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = r0 + i * 4 + (t >> 6);
    v[i] = 0;
    if (r < rows && sc >= 0) v[i] = src[(int64_t)r * lds + sc];
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) tile[(i * 4 + (t >> 6)) * LD + l] = v[i];
  __syncthreads();
  const int row = t & 31, c8 = (t >> 5) * 8;
  if (c0 + c8 >= cols_pad) return;
  const uint4 w = *(const uint4*)(tile + row * LD + c8);
  *(uint4*)(dst + (((int64_t)blockIdx.y * (cols_pad / 16) + (c0 + c8) / 16) * 64 + ((c8 >> 3) & 1) * 32 + row) * 8) = w;
}

// X [r8, ldx] fp32 (row r and beyond zero; in the copy that the state names) -> three bf16 terms whose sum is X to
// the last bit of fp32 (each takes the leading 8 bits of what is left), side by side in one tiled matrix
// [r32, 3 dk], the smallest first
__global__ void __launch_bounds__(256) split_terms_kernel(const float* X, const PolarState* state, int64_t flip, int64_t ldx,
                                                          int r8, int d, int r32, int dk, uint16_t* terms) {
  X += state->parity * flip;
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;   // one 16-byte chunk of each term
  const int kbs = dk / 16;
  if (id >= (int64_t)(r32 / 32) * kbs * 64) return;
  const int lane = (int)(id & 63), kb = (int)((id >> 6) % kbs), rb = (int)((id >> 6) / kbs);
  const int row = rb * 32 + (lane & 31), k0 = kb * 16 + (lane >> 5) * 8;
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float v = (row < r8 && k0 + e < d) ? X[(int64_t)row * ldx + k0 + e] : 0.f;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const uint32_t b = f32_to_bf16(v);
      v -= bf16_to_f32((bf16_t)b);
      w[t][e >> 1] = (e & 1) ? (w[t][e >> 1] | (b << 16)) : b;
    }
  }
#pragma unroll
  for (int t = 0; t < 3; ++t)
    *(uint4*)(terms + (((int64_t)rb * 3 * kbs + (2 - t) * kbs + kb) * 64 + lane) * 8) = make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]);
}

// sum of squares in two fixed-order stages: 256 block partials, then one block (blockIdx.y: matrix)
__global__ void __launch_bounds__(256) sumsq_stage1_kernel(const float* x, int64_t n, float* part) {
  __shared__ float red[256];
  x += n * blockIdx.y;
  float s = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)256 * gridDim.x) s += x[i] * x[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.y * 260 + blockIdx.x] = red[0];
}
__global__ void __launch_bounds__(256) sumsq_stage2_kernel(float* part, int n_part) {
  __shared__ float red[256];
  part += blockIdx.x * 260;
  red[threadIdx.x] = (int)threadIdx.x < n_part ? part[threadIdx.x] : 0.f;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[256] = red[0] > 0.f ? 1.0f / sqrtf(red[0]) : 0.f;   // scale for the next kernel
}

// dst[a][b] = src[b][a] * scale (fp32; a < rows_dst, b < cols_dst), zero for cols_dst <= b < ldd;
// blockIdx.z: matrix (both contiguous)
__global__ void scale_transpose_kernel(const float* src, int64_t lds, float* dst, int64_t ldd, int rows_dst, int cols_dst,
                                       const float* part) {
  __shared__ float tile[32][33];
  const float scale = part[blockIdx.z * 260 + 256];
  src += (int64_t)blockIdx.z * cols_dst * lds;
  dst += (int64_t)blockIdx.z * rows_dst * ldd;
  const int a0 = blockIdx.y * 32, b0 = blockIdx.x * 32;
  for (int i = threadIdx.y; i < 32; i += 8) {
    const int b = b0 + i, a = a0 + threadIdx.x;
    tile[i][threadIdx.x] = b < cols_dst && a < rows_dst ? src[(int64_t)b * lds + a] * scale : 0.f;
  }
  __syncthreads();
  for (int i = threadIdx.y; i < 32; i += 8) {
    const int a = a0 + i, b = b0 + threadIdx.x;
    if (a < rows_dst && b < ldd) dst[(int64_t)a * ldd + b] = tile[threadIdx.x][i];
  }
}

// dst [rows, cols] (bf16 or fp32, contiguous) = src[a][b], or src[b][a] through LDS; with a state, src is the
// copy that it names
template <typename T>
__global__ void emit_kernel(const float* src, const PolarState* state, int64_t flip, int64_t lds, int transposed, T* dst,
                            int rows, int cols) {
  __shared__ float tile[32][33];
  if (state) src += state->parity * flip;
  const int a0 = blockIdx.y * 32, b0 = blockIdx.x * 32;
  auto put = [&](int a, int b, float v) {
    if constexpr (sizeof(T) == 4) dst[(int64_t)a * cols + b] = v;
    else dst[(int64_t)a * cols + b] = (T)(pack_bf16x2(v, 0.f) & 0xffffu);
  };
  if (transposed) {
    for (int i = threadIdx.y; i < 32; i += 8) {
      const int b = b0 + i, a = a0 + threadIdx.x;
      if (b < cols && a < rows) tile[i][threadIdx.x] = src[(int64_t)b * lds + a];
    }
    __syncthreads();
  }
  for (int i = threadIdx.y; i < 32; i += 8) {
    const int a = a0 + i, b = b0 + threadIdx.x;
    if (a < rows && b < cols) put(a, b, transposed ? tile[threadIdx.x][i] : src[(int64_t)a * lds + b]);
  }
}

struct FactorWs {
  int mats, m4, r8, r32, mk, dk;
  size_t off_z, off_zt, off_om, off_part, off_terms, off_xt, off_c, off_red, off_polar, total;
  PolarWs polar;
  size_t part_bytes;
};

FactorWs make_factor_ws(const ffsplit_desc_t& d) {
  FactorWs w = {};
  const bool bf = d.dtype == FFSPLIT_BF16;
  const int m = d.d_ff - d.k > 0 ? d.d_ff - d.k : 4, r = d.rank > 0 ? d.rank : 4, dm = d.d_model;
  w.mats = d.act == FFSPLIT_ACT_SWIGLU ? 3 : 2;
  w.m4 = round_up(m, 4);
  w.r8 = round_up(r, 8);
  w.r32 = round_up(r, 32);
  w.mk = round_up(m, 64);
  w.dk = round_up(dm, 64);
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off = align256(off + bytes); return o; };
  if (bf) {
    // one remainder matrix at a time: tiled [d_model, m] for the sketch, [m, d_model] for the projection
    w.off_z = take(std::max((size_t)round_up(dm, 32) * w.mk, (size_t)round_up(m, 32) * w.dk) * 2);
    w.off_om = take((size_t)w.r32 * w.mk * 2);
    const GemmPlan p = gemm_plan(dm, w.r8, m, false, false, true, true);
    w.part_bytes = p.split > 1 ? (size_t)p.split * dm * w.r32 * 4 : 0;
    w.off_part = take(w.part_bytes);
    w.off_terms = take((size_t)w.r32 * 3 * w.dk * 2);
    w.off_c = take((size_t)m * w.r8 * 4);   // (B^T Z)^T
  } else {
    w.off_z = take((size_t)dm * w.m4 * 4);
    w.off_zt = take((size_t)dm * w.m4 * 4);
    w.off_om = take((size_t)w.r8 * w.m4 * 4);
    w.off_c = take((size_t)w.r8 * w.m4 * 4);   // B^T Z
  }
  w.off_xt = take((size_t)w.mats * w.r8 * dm * 4);
  w.polar = make_polar_ws(w.mats, r, dm);
  w.off_polar = take(w.polar.bytes);
  w.off_red = take((size_t)w.mats * 260 * 4);
  w.total = off;
  return w;
}

GemmArgs gemm_nt(const void* A, int64_t lda, const void* Bt, int64_t ldb, int M, int N, int K, float* C, int64_t ldc) {
  GemmArgs g = {};
  g.A = A; g.lda = lda; g.Bt = Bt; g.ldb = ldb; g.M = M; g.N = N; g.K = K;
  g.split_col = N; g.C0 = C; g.ldc0 = ldc; g.n_store = N;
  return g;
}

#define FK(expr)                 \
  do {                           \
    if ((expr) != 0) return -1;  \
  } while (0)
#define FKL()                                        \
  do {                                               \
    if (hipGetLastError() != hipSuccess) return -1;  \
  } while (0)

}  // namespace

size_t factorize_ws_bytes(const ffsplit_desc_t& d) { return make_factor_ws(d).total; }

int launch_factorize(const ffsplit_desc_t& d, const void* W1, const void* Wg, const void* W2, const int32_t* rest,
                     uint32_t seed, void* const* factors, char* ws, hipStream_t st) {
  const int dm = d.d_model, m = d.d_ff - d.k, r = d.rank;
  if (m <= 0 || r <= 0) return 0;
  const FactorWs w = make_factor_ws(d);
  const int m4 = w.m4, r8 = w.r8;
  float* C = (float*)(ws + w.off_c);
  float* red = (float*)(ws + w.off_red);
  char* Z = ws + w.off_z;
  const bool bf = d.dtype == FFSPLIT_BF16;
  const PolarWs& pw = w.polar;
  const int64_t nx = (int64_t)r8 * dm;
  const void* Ws[3] = {W1, d.act == FFSPLIT_ACT_SWIGLU ? Wg : W2, W2};   // the last one is the down projection
  const uint32_t stream_of[3] = {0, d.act == FFSPLIT_ACT_SWIGLU ? 1u : 2u, 2};

  // ---- sketches: (Y^T)^T = Z Omega^T  [d, r8] per matrix
  float* XT = (float*)(ws + w.off_xt);
  float* X = (float*)(ws + w.off_polar + pw.off_x);
  for (int i = 0; i < w.mats; ++i) {
    const bool down = i == w.mats - 1;
    const uint16_t* W = (const uint16_t*)Ws[i];
    uint32_t key = seed + 0x9E3779B9u * stream_of[i];
    key ^= key >> 16; key *= 0x85EBCA6Bu; key ^= key >> 13; key *= 0xC2B2AE35u; key ^= key >> 16;
    if (bf) {
      if (down) {
        PermArgs pa = {};
        pa.src = W; pa.lds = dm; pa.dst = Z; pa.ldd = w.mk; pa.dst_tiled = 1;
        pa.n_count = dm; pa.c_count = m; pa.cmap = rest; pa.c_pad = w.mk;
        FK(launch_permute_transpose(pa, 2, st));
      } else {
        hipLaunchKernelGGL(gather_tiled_kernel, dim3(w.mk / 64, (dm + 31) / 32), dim3(256), 0, st, W, (int64_t)d.d_ff, rest, 0,
                           dm, m, w.mk, (uint16_t*)Z);
        FKL();
      }
      const int kb = w.mk / 16;
      hipLaunchKernelGGL(rademacher_tiled_kernel, dim3((kb + 3) / 4, 4), dim3(256), 0, st, (uint16_t*)(ws + w.off_om), r, m,
                         w.r32, w.mk, key);
      FKL();
      GemmArgs g = gemm_nt(Z, w.mk, ws + w.off_om, w.mk, dm, r8, m, XT + i * nx, r8);
      g.a_tiled = 1; g.out_f32 = 1;
      const GemmPlan p = gemm_plan(dm, r8, m, false, false, true, true);
      if (p.split > 1) {
        GemmArgs gp = g;
        gp.partial = 1; gp.C0 = ws + w.off_part; gp.ldc0 = w.r32; gp.split_col = w.r32; gp.out_f32 = 0;
        FK(launch_gemm_bf16(gp, ACT_NONE, false, p.shape, p.split, st));
        FK(launch_splitk_epilogue((const float*)(ws + w.off_part), p.split, w.r32, g, ACT_NONE, st));
      } else {
        FK(launch_gemm_bf16(g, ACT_NONE, false, p.shape, 1, st));
      }
    } else {
      const unsigned gz = (unsigned)(((int64_t)dm * m4 + 255) / 256);
      hipLaunchKernelGGL(gather_z_kernel, dim3(gz), dim3(256), 0, st, (const float*)Ws[i], dm, d.d_ff, rest, m, m4, (int)down,
                         (float*)Z, (float*)nullptr);
      const int64_t no = (int64_t)r8 * m4;
      hipLaunchKernelGGL(rademacher_kernel, dim3((unsigned)((no + 255) / 256)), dim3(256), 0, st, (float*)(ws + w.off_om), r, m,
                         r8, m4, key);
      FKL();
      FK(launch_gemm_f32(gemm_nt(Z, m4, ws + w.off_om, m4, dm, r8, m4, XT + i * nx, r8), ACT_NONE, false, st));
    }
  }
  // ---- unit Frobenius norm, rows of d, polar factor
  hipLaunchKernelGGL(sumsq_stage1_kernel, dim3(256, w.mats), dim3(256), 0, st, XT, nx, red);
  hipLaunchKernelGGL(sumsq_stage2_kernel, dim3(w.mats), dim3(256), 0, st, red, 256);
  hipLaunchKernelGGL(scale_transpose_kernel, dim3(pw.dk / 32, (r8 + 31) / 32, w.mats), dim3(32, 8), 0, st, XT, (int64_t)r8, X,
                     (int64_t)pw.dk, r8, dm, red);
  FKL();
  const PolarState* state = nullptr;
  FK(launch_polar(pw, ws + w.off_polar, &state, st));
  if (!bf) FK(launch_polar_settle(pw, ws + w.off_polar, state, st));
  const int64_t flip = w.mats * pw.nx;
  // ---- projections and factors in the caller's convention and type:
  // P = B [d, r], Q = B^T Z [r, m] (up, gate);  P = Z^T B [m, r], Q = B^T [r, d] (down)
  for (int i = 0; i < w.mats; ++i) {
    const bool down = i == w.mats - 1;
    void* Pf = factors[down ? 4 : (i == 0 ? 0 : 2)];
    void* Qf = factors[down ? 5 : (i == 0 ? 1 : 3)];
    const float* Xi = X + i * pw.nx;
    const PolarState* si = bf ? state + i : nullptr;
    if (bf) {
      if (down) {
        hipLaunchKernelGGL(gather_tiled_kernel, dim3(w.dk / 64, (m + 31) / 32), dim3(256), 0, st, (const uint16_t*)Ws[i],
                           (int64_t)dm, rest, 1, m, dm, w.dk, (uint16_t*)Z);
        FKL();
      } else {
        PermArgs pa = {};
        pa.src = Ws[i]; pa.lds = d.d_ff; pa.dst = Z; pa.ldd = w.dk; pa.dst_tiled = 1;
        pa.n_count = m; pa.c_count = dm; pa.nmap = rest; pa.c_pad = w.dk;
        FK(launch_permute_transpose(pa, 2, st));
      }
      char* term = ws + w.off_terms;
      const int64_t chunks = (int64_t)(w.r32 / 32) * (w.dk / 16) * 64;
      hipLaunchKernelGGL(split_terms_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st, Xi, si, flip,
                         (int64_t)pw.dk, r8, dm, w.r32, w.dk, (uint16_t*)term);
      FKL();
      // all three terms in one reduction: three launches that each read back the sums took 73 us, one 53
      // (7946 x 512 x 2048)
      GemmArgs g = gemm_nt(Z, w.dk, term, 3 * w.dk, m, r8, 3 * w.dk, C, r8);
      g.a_tiled = 1; g.out_f32 = 1; g.a_wrap = w.dk;
      FK(launch_gemm_bf16(g, ACT_NONE, false, gemm_plan(m, r8, 3 * w.dk, false, false, true, false).shape, 1, st));
    } else {
      const unsigned gz = (unsigned)(((int64_t)dm * m4 + 255) / 256);
      hipLaunchKernelGGL(gather_z_kernel, dim3(gz), dim3(256), 0, st, (const float*)Ws[i], dm, d.d_ff, rest, m, m4, (int)down,
                         (float*)nullptr, (float*)(ws + w.off_zt));
      FKL();
      FK(launch_gemm_f32(gemm_nt(Xi, pw.dk, ws + w.off_zt, dm, r8, m4, dm, C, m4), ACT_NONE, false, st));
    }
    // C is [m, r8] (bf16) or [r8, m4] (fp32)
    const int64_t ldc = bf ? r8 : m4;
    auto emit = [&](const float* src, const PolarState* s, int64_t lds, int transposed, void* dst, int rows, int cols) {
      const dim3 grid((cols + 31) / 32, (rows + 31) / 32), block(32, 8);
      if (bf) hipLaunchKernelGGL(emit_kernel<bf16_t>, grid, block, 0, st, src, s, flip, lds, transposed, (bf16_t*)dst, rows, cols);
      else hipLaunchKernelGGL(emit_kernel<float>, grid, block, 0, st, src, s, flip, lds, transposed, (float*)dst, rows, cols);
    };
    if (down) {
      emit(C, nullptr, ldc, bf ? 0 : 1, Pf, m, r);
      emit(Xi, si, pw.dk, 0, Qf, r, dm);
    } else {
      emit(Xi, si, pw.dk, 1, Pf, dm, r);
      emit(C, nullptr, ldc, bf ? 1 : 0, Qf, r, m);
    }
    FKL();
  }
  return 0;
}

}  // namespace ffsplit
