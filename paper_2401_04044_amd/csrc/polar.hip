// Polar factor of the sketches of the remainder factorisation (factor.hip): the rows of X [r, d] fp32 become
// orthonormal by X <- (c0 I + c1 G + c2 G^2) X, G = X X^T, with coefficients chosen step by step on the
// device (polar_steps.h).  Per step three products for all matrices of a layer:
//   gram    S = X X^T (one triangle, mirrored) and the tiles' shares of ||S - I||_F^2,
//   poly    the step's coefficients, T - I for T = c0 I + c1 S + c2 S^2 (one triangle, mirrored),
//   apply   X' = X + (T - I) X into the other buffer: near the end T - I is small, and with it the rounding of the sums.
// The host cannot know how many steps a matrix takes and must not wait.  It launches the first steps product by
// product (polar_launched); the steps after those, which flat and mildly decaying spectra do not need, are one
// launch of a work queue that returns at once when nothing is left.  (A launch that does nothing costs 3.5 us:
// three for every step of the worst sketch of rank 512 were 115 us of 816.)  Measured, us, a layer compressed and
// tried (two matrices): 2048 x 7946 rank 512 1235 -> 715, 1536 x 4800 rank 400 gated 1130 -> 655, 512 x 1450 rank 64 276 -> 240 (with the
// projections in one launch each 672, 616, 229).
// Factorisation alone at 2048 x 7946 with singular values i^-a: a = 0 1140 -> 620, 1/2 1140 -> 720, 1 1140 -> 950;
// the other way round where the queue does most of the steps: a = 2 1620, rank one 1990.
// All products are true fp32 (v_mfma_f32_16x16x4_f32, 256 flop per clock and CU), staged through LDS by loads
// without registers.  A tile asks the caches for 16 (64x64) or 32 bytes per clock of 61: what bounds them is
// the matrix rate, and at the usual ranks the start of a launch and the latency of its first loads.  So the
// triangles take 32x32 tiles (272 workgroups for two matrices of rank 512: 25 us; 64x64 ones cut into seven ranges of
// d, summed by the last to arrive: 31), rings are seven slabs deep, and every launch requests its first slabs
// before it looks at the state: buffer s & 1 holds the X of step s of every matrix that takes that step.
// Of a step's 65 us gram is 25, poly 16, apply 25 (24, 12.5 and 29 with the operands straight from registers).
// Rows of X and S are padded to 32 floats of zeros, so no product looks at its last slab of K.
#include "polar.h"
#include "common.h"
#include "layout.h"
#include <algorithm>

namespace ffsplit {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((address_space(3))) void* lptr_t;

__device__ __forceinline__ void to_lds(const void* base, lptr_t dst, uint32_t lane_off, uint32_t scalar_off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00027000), dst, 16,
                                           lane_off, scalar_off, 0, 0);
}
// at most N loads still in flight, and every LDS read done
template <int N>
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}

// A product acc += A[rows][K] * B^T over K in slabs of 32, a (32 TL)^2 tile on 2 x 2 wavefronts of (16 TL)^2.
//   A: row-major, K contiguous.  B: the same (rows = output columns), or with COLS K x N, N contiguous.
// Stage: 32 TL rows x 128 bytes of A, then of B; the 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7)
// (16 lanes then read 16 different bank groups).  COLS: 32 rows (k) of 256 bytes, chunk c of row k at
// c ^ (4 ((k >> 2) & 3)), read a float at a time without conflicts.
// a_rows, b_rows: rows from the tile's first (rows past the operands repeat the last one: their results are not
// stored); COLS: b_rows is the columns of B from the tile's first, k_rows its rows.
template <int TL, bool COLS>
struct TileProduct {
  static_assert(!COLS || TL == 2, "a row of 64 columns is 256 bytes");
  static constexpr int OPER = TL * 1024;               // floats of one operand in a stage
  static constexpr int STAGES = TL == 1 ? 7 : 3;       // 56 or 48 KiB: two workgroups a CU and more
  static constexpr int LDS = STAGES * 2 * OPER * 4;
  const float *A, *B;
  float* smem;
  int64_t ldb;
  int k_rows, n, lane, wave;
  int put, get;   // stage that the next slab goes to, that the next one is read from
  uint32_t a_off[TL], b_off[TL];

  // requests the first STAGES - 1 slabs
  __device__ __forceinline__ void start(const float* A_, int64_t lda, int a_rows, const float* B_, int64_t ldb_, int b_rows,
                                        int k_rows_, int slabs, float* smem_) {
    A = A_; B = B_; smem = smem_; ldb = ldb_; k_rows = k_rows_; n = slabs;
    put = get = 0;
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int i = 0; i < TL; ++i) {
      const int blk = wave * TL + i, row = blk * 8 + (lane >> 3);
      const uint32_t col = 16 * ((lane & 7) ^ ((row >> 1) & 7));
      a_off[i] = (uint32_t)min(row, a_rows - 1) * (uint32_t)(lda * 4) + col;
      if (COLS) {
        const int c = (lane & 15) ^ (4 * (blk & 3));
        b_off[i] = (uint32_t)(c * 4 < b_rows ? c : 0) * 16;
      } else {
        b_off[i] = (uint32_t)min(row, b_rows - 1) * (uint32_t)(ldb * 4) + col;
      }
    }
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
      if (s < n) issue(s);
  }
  __device__ __forceinline__ void issue(int s) {
    float* const st = smem + put * 2 * OPER;
    put = put + 1 == STAGES ? 0 : put + 1;
#pragma unroll
    for (int i = 0; i < TL; ++i) {
      const int blk = wave * TL + i;
      to_lds(A, (lptr_t)(st + blk * 256), a_off[i], (uint32_t)s * 128);
      if (COLS) {   // (k rows past the last repeat it: A is zero there)
        const int k = min(s * 32 + blk * 4 + (lane >> 4), k_rows - 1);
        to_lds(B, (lptr_t)(st + OPER + blk * 256), b_off[i] + (uint32_t)k * (uint32_t)(ldb * 4), 0);
      } else {
        to_lds(B, (lptr_t)(st + OPER + blk * 256), b_off[i], (uint32_t)s * 128);
      }
    }
  }
  // the loads requested so far have landed: the workgroup may end, or use its LDS for another product
  static __device__ __forceinline__ void drain() { wait_loads<0>(); }

  struct Frags { f32x4_t a[2][TL], b[2][TL]; };
  __device__ __forceinline__ void read(Frags& f) {
    const int wm = wave >> 1, wn = wave & 1, r16 = lane & 15, quad = lane >> 4;
    const float* const st = smem + get * 2 * OPER;
    get = get + 1 == STAGES ? 0 : get + 1;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int pos = (quad + 4 * h) ^ ((r16 >> 1) & 7);
#pragma unroll
      for (int i = 0; i < TL; ++i) f.a[h][i] = *(const f32x4_t*)(st + (wm * 16 * TL + i * 16 + r16) * 32 + pos * 4);
#pragma unroll
      for (int j = 0; j < TL; ++j) {
        if (COLS) {
          const int c = wn * 32 + j * 16 + r16, at = ((c >> 2) ^ (4 * quad)) * 4 + (c & 3);
#pragma unroll
          for (int t = 0; t < 4; ++t) f.b[h][j][t] = st[OPER + (4 * (quad + 4 * h) + t) * 64 + at];
        } else {
          f.b[h][j] = *(const f32x4_t*)(st + OPER + (wn * 16 * TL + j * 16 + r16) * 32 + pos * 4);
        }
      }
    }
  }
  // Sums in NS accumulators of a tile, added in pairs at the end: with one, a chain of 512 roundings at d = 2048, the
  // basis was 6.8e-7 off orthonormal.  (2048 x 7946 rank 512 in fp32, root mean square: 2.3e-7 with these, 1.7e-7 with T - I
  // applied; the products straight from registers had 2.2e-7.)
  static constexpr int NS = TL == 1 ? 8 : 4;
  typedef f32x4_t Sums[NS][TL][TL];
  __device__ __forceinline__ static void mma(const Frags& f, Sums& acc) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < TL; ++i)
#pragma unroll
          for (int j = 0; j < TL; ++j) {
            f32x4_t& c = acc[(h * 4 + t) % NS][i][j];
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(f.b[h][j][t], f.a[h][i][t], c, 0, 0, 0);
          }
  }
  // slab s has landed for every wavefront, and slab s - 1 is in everyone's registers: the ring moves on
  __device__ __forceinline__ void advance(int s) {
    if (s + STAGES - 2 < n) wait_loads<(STAGES - 2) * 2 * TL>();
    else wait_loads<0>();
    asm volatile("s_barrier" ::: "memory");
    if (s + STAGES - 1 < n) issue(s + STAGES - 1);
  }
  // the fragments of a slab are read while the one before is multiplied
  __device__ __forceinline__ void run(f32x4_t (&out)[TL][TL]) {
    Sums acc = {};
    Frags f0, f1;
    advance(0);
    read(f0);
    int s = 1;
    for (; s + 1 < n; s += 2) {
      advance(s);
      read(f1);
      mma(f0, acc);
      advance(s + 1);
      read(f0);
      mma(f1, acc);
    }
    if (s < n) {
      advance(s);
      read(f1);
      mma(f0, acc);
      mma(f1, acc);
    } else {
      mma(f0, acc);
    }
#pragma unroll
    for (int n = NS / 2; n > 0; n /= 2)
#pragma unroll
      for (int k = 0; k < n; ++k)
#pragma unroll
        for (int i = 0; i < TL; ++i)
#pragma unroll
          for (int j = 0; j < TL; ++j) acc[k][i][j] += acc[k + n][i][j];
#pragma unroll
    for (int i = 0; i < TL; ++i)
#pragma unroll
      for (int j = 0; j < TL; ++j) out[i][j] = acc[0][i][j];
  }
};

struct PolarArgs {
  PolarPlan plan;
  PolarState* state;     // [max_steps + 1][mats]: state[s] is what step s starts from
  PolarState* result;    // [mats]: behind the last step carried out
  int step, mats, r, r8, rk, d, dk;
  float* X;              // [2][mats][r8, dk]
  int64_t flip;          // elements between the two buffers
  float* S;              // [mats][r8, rk]
  float* T;              // (T - I)
  int gram_tiles, poly_tiles, apply_tiles;
  float* share;          // [mats][gram_tiles]: the tiles' shares of ||S - I||_F^2
  float* rows;           // [mats][2][r8]: sums of |S| and of S^2 along its rows
  unsigned* queue;       // [product][POLAR_SHARDS drawn, POLAR_SHARDS done, 1 finished][POLAR_SHARD_WORDS], zero
};

// lower triangle, row by row: tile t is (i, j <= i)
__device__ __forceinline__ void triangle(int t, int& i, int& j) {
  i = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  while (i * (i + 1) / 2 > t) --i;
  j = t - i * (i + 1) / 2;
}

// sum over the 256 threads in a fixed order, in every thread
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// DEV (within the queue's launch): device-scope stores, which go through to where all XCDs see them
template <bool DEV>
__device__ __forceinline__ void put4(float* p, f32x4_t v) {
  if (DEV) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      __hip_atomic_store((unsigned long long*)p + h, (unsigned long long)__float_as_uint(v[2 * h]) |
                                                         ((unsigned long long)__float_as_uint(v[2 * h + 1]) << 32),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    *(f32x4_t*)p = v;
  }
}
template <bool DEV, typename V>
__device__ __forceinline__ void put1(V* p, V v) {
  if (DEV) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

// four columns col .. of a row of a symmetric matrix [r8, rk], and their mirror images; what lies in
// the padding columns is written as zero
template <bool DEV>
__device__ __forceinline__ void store_sym(float* S, int r8, int rk, int row, int col, bool mirror, f32x4_t v) {
  if (row < r8 && col < rk) put4<DEV>(S + (int64_t)row * rk + col, col < r8 ? v : f32x4_t{0.f, 0.f, 0.f, 0.f});
  if (mirror && row < rk && col < r8) {
#pragma unroll
    for (int e = 0; e < 4; ++e) put1<DEV>(S + (int64_t)(col + e) * rk + row, row < r8 ? v[e] : 0.f);
  }
}

__device__ __forceinline__ PolarState load_state(const PolarState* s) {
  // (device scope: within the queue's launch it may have been written by another XCD)
  PolarState v;
  const int* q = (const int*)s;
  int* o = (int*)&v;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(PolarState) / 4); ++i) o[i] = __hip_atomic_load(q + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return v;
}

__device__ __forceinline__ void store_state(PolarState* s, const PolarState& v) {
  int* q = (int*)s;
  const int* o = (const int*)&v;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(PolarState) / 4); ++i) put1<true>(q + i, o[i]);
}

// tile `tile` of the S that step `step` starts from
template <int TL, bool DEV>
__device__ __forceinline__ void gram_tile(const PolarArgs& p, int step, int mat, int tile, float* smem, float* red) {
  constexpr int B = 32 * TL;
  int tm, tn;
  triangle(tile, tm, tn);
  const float* X = p.X + (step & 1) * p.flip + (int64_t)mat * p.r8 * p.dk;
  TileProduct<TL, false> prod;
  prod.start(X + (int64_t)tm * B * p.dk, p.dk, p.r8 - tm * B, X + (int64_t)tn * B * p.dk, p.dk, p.r8 - tn * B, 0, p.dk / 32, smem);
  if (step > 0) {
    const PolarState s = load_state(p.state + (int64_t)step * p.mats + mat);
    if (!s.act || s.last) { prod.drain(); return; }
  }
  f32x4_t acc[TL][TL] = {};
  prod.run(acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* S = p.S + (int64_t)mat * p.r8 * p.rk;
  float dev = 0.f;
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j) {
      const int row = tm * B + (wave >> 1) * 16 * TL + i * 16 + (lane & 15);
      const int col = tn * B + (wave & 1) * 16 * TL + j * 16 + 4 * (lane >> 4);
      store_sym<DEV>(S, p.r8, p.rk, row, col, tm != tn, acc[i][j]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = acc[i][j][e] - (row == col + e ? 1.f : 0.f);
        if (row < p.r && col + e < p.r) dev = fmaf(x, x, dev);
      }
    }
  dev = block_sum(dev, red);
  if (threadIdx.x == 0) put1<DEV>(p.share + (int64_t)mat * p.gram_tiles + tile, tm != tn ? 2.f * dev : dev);
}

// sums of |S| and of S^2 along the rows: the largest of the first bounds the largest eigenvalue, as
// does the root of the total of the second
__global__ void __launch_bounds__(256) polar_rows_kernel(const PolarArgs p) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, mat = blockIdx.y;
  if (row >= p.r8) return;
  const float* S = p.S + ((int64_t)mat * p.r8 + row) * p.rk;
  float a = 0.f, q = 0.f;
  for (int c = lane; c < p.r8; c += 64) { a += fabsf(S[c]); q = fmaf(S[c], S[c], q); }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { a += __shfl_xor(a, o); q += __shfl_xor(q, o); }
  if (lane == 0) { p.rows[(int64_t)mat * 2 * p.r8 + row] = a; p.rows[((int64_t)mat * 2 + 1) * p.r8 + row] = q; }
}

// tile `tile` of T for step `step`
template <int TL, bool DEV>
__device__ __forceinline__ void poly_tile(const PolarArgs& p, int step, int mat, int tile, float* smem, float* red) {
  constexpr int B = 32 * TL;
  int tm, tn;
  triangle(tile, tm, tn);
  const float* S = p.S + (int64_t)mat * p.r8 * p.rk;
  TileProduct<TL, false> prod;
  prod.start(S + (int64_t)tm * B * p.rk, p.rk, p.r8 - tm * B, S + (int64_t)tn * B * p.rk, p.rk, p.r8 - tn * B, 0, p.rk / 32, smem);
  // (everything the tile needs is requested at once: the loads' latency is most of this kernel)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row0 = tm * B + (wave >> 1) * 16 * TL + (lane & 15), col0 = tn * B + (wave & 1) * 16 * TL + 4 * (lane >> 4);
  f32x4_t g[TL][TL];
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j)
      g[i][j] = row0 + i * 16 < p.r8 && col0 + j * 16 < p.rk ? *(const f32x4_t*)(S + (int64_t)(row0 + i * 16) * p.rk + col0 + j * 16)
                                                             : f32x4_t{0.f, 0.f, 0.f, 0.f};
  PolarState s = {};
  float most = 0.f, sum = 0.f;
  if (step == 0) {
    const float* rows = p.rows + (int64_t)mat * 2 * p.r8;
    for (int i = threadIdx.x; i < p.r; i += 256) { most = fmaxf(most, rows[i]); sum += rows[p.r8 + i]; }
  } else {
    for (int i = threadIdx.x; i < p.gram_tiles; i += 256) sum += p.share[(int64_t)mat * p.gram_tiles + i];
    s = load_state(p.state + (int64_t)step * p.mats + mat);
    if (s.mode == POLAR_ENDED || s.last) {
      prod.drain();
      s.mode = POLAR_ENDED; s.act = s.last = 0;
      if (tile == 0 && threadIdx.x == 0) store_state(p.state + (int64_t)(step + 1) * p.mats + mat, s);
      return;
    }
  }
  float fig = block_sum(sum, red);
  if (step == 0) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = fmaxf(most, __shfl_xor(most, o));
    __syncthreads();
    if (lane == 0) red[wave] = most;
    __syncthreads();
    most = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    fig = sqrtf(fminf(most, sqrtf(fig)));
  }
  float c[3];
  s = polar_decide(p.plan, step, p.r, s, fig, c);
  if (tile == 0 && threadIdx.x == 0) {
    store_state(p.state + (int64_t)(step + 1) * p.mats + mat, s);
    store_state(p.result + mat, s);
  }
  f32x4_t acc[TL][TL] = {};
  prod.run(acc);
  float* T = p.T + (int64_t)mat * p.r8 * p.rk;
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j) {
      const int row = row0 + i * 16, col = col0 + j * 16;
      f32x4_t v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = c[2] * acc[i][j][e] + c[1] * g[i][j][e] + (row == col + e ? c[0] - 1.f : 0.f);
      store_sym<DEV>(T, p.r8, p.rk, row, col, tm != tn, v);
    }
}

// tile `tile` of the X behind step `step`
template <bool DEV>
__device__ __forceinline__ void apply_tile(const PolarArgs& p, int step, int mat, int tile, float* smem) {
  constexpr int TL = 2;
  const int tiles_m = (p.r8 + 63) / 64, tm = tile % tiles_m, tn = tile / tiles_m;
  const int64_t at = (int64_t)mat * p.r8 * p.dk;
  const float* T = p.T + (int64_t)mat * p.r8 * p.rk + (int64_t)tm * 64 * p.rk;
  const float* X = p.X + (step & 1) * p.flip + at;
  TileProduct<TL, true> prod;
  prod.start(T, p.rk, p.r8 - tm * 64, X + tn * 64, p.dk, p.dk - tn * 64, p.r8, p.rk / 32, smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  f32x4_t x[TL][TL];
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j) {
      const int row = tm * 64 + (wave >> 1) * 32 + i * 16 + (lane & 15);
      const int col = tn * 64 + (wave & 1) * 32 + j * 16 + 4 * (lane >> 4);
      x[i][j] = row < p.r8 && col < p.dk ? *(const f32x4_t*)(X + (int64_t)row * p.dk + col) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  const PolarState s = load_state(p.state + (int64_t)(step + 1) * p.mats + mat);
  if (!s.act) { prod.drain(); return; }
  f32x4_t acc[TL][TL] = {};
  prod.run(acc);
  float* O = p.X + ((step & 1) ^ 1) * p.flip + at;
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j) {
      const int row = tm * 64 + (wave >> 1) * 32 + i * 16 + (lane & 15);
      const int col = tn * 64 + (wave & 1) * 32 + j * 16 + 4 * (lane >> 4);
      if (row < p.r8 && col < p.dk) put4<DEV>(O + (int64_t)row * p.dk + col, col < p.d ? x[i][j] + acc[i][j] : f32x4_t{0.f, 0.f, 0.f, 0.f});
    }
}

template <int TL>
__global__ void __launch_bounds__(256) polar_gram_kernel(const PolarArgs p) {
  extern __shared__ float polar_smem[];
  __shared__ float red[4];
  gram_tile<TL, false>(p, p.step, blockIdx.y, blockIdx.x, polar_smem, red);
}
template <int TL>
__global__ void __launch_bounds__(256) polar_poly_kernel(const PolarArgs p) {
  extern __shared__ float polar_smem[];
  __shared__ float red[4];
  poly_tile<TL, false>(p, p.step, blockIdx.y, blockIdx.x, polar_smem, red);
}
__global__ void __launch_bounds__(256) polar_apply_kernel(const PolarArgs p) {
  extern __shared__ float polar_smem[];
  apply_tile<false>(p, p.step, blockIdx.y, blockIdx.x, polar_smem);
}

// Steps p.step .. max_steps - 1 in one launch.  The tiles of a product are cut into chunks, one or more per
// workgroup of the launch, which the workgroups draw from POLAR_SHARDS counters (their own, then any that has some
// left; one counter for all of them took 70 us a step more).  A workgroup moves on to the next product when every
// chunk of this one has been drawn, and starts on it when every chunk is done.  The chunks it waits for are then all
// in the hands of workgroups that run and wait for earlier products only: every wait ends, however few workgroups
// are resident.
// Results go out with device-scope stores that every thread waits for before its chunk is counted done; a
// workgroup that starts on a product invalidates what its caches hold from before.  Everyone leaves at the
// first step that finds all matrices ended.
template <int TL>
__global__ void __launch_bounds__(256) polar_queue_kernel(const PolarArgs p) {
  extern __shared__ float polar_smem[];
  __shared__ float red[4];
  __shared__ int s_chunk;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int own = (int)blockIdx.x % POLAR_SHARDS;
  auto load = [](const unsigned* q) { return (int)__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto add1 = [](unsigned* q) { return (int)__hip_atomic_fetch_add(q, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  int waiting_for = 0;   // shards of the product before, counted at `before`
  unsigned *drawn = p.queue, *before = nullptr;
  for (int step = p.step; step < p.plan.max_steps; ++step)
    for (int product = 0; product < 3; ++product) {
      if (product == 2 && step + 1 == p.plan.max_steps) return;   // (no step follows)
      const int per_mat = product == 0 ? p.poly_tiles : product == 1 ? p.apply_tiles : p.gram_tiles;
      const int tasks = per_mat * p.mats, size = (tasks + (int)gridDim.x - 1) / (int)gridDim.x, chunks = (tasks + size - 1) / size;
      unsigned* const done = drawn + POLAR_SHARDS * POLAR_SHARD_WORDS;
      unsigned* const finished = done + POLAR_SHARDS * POLAR_SHARD_WORDS;   // shards all of whose chunks are done
      int ahead = 0;   // (the first draw travels while the workgroup waits)
      if (threadIdx.x == 0) ahead = add1(drawn + own * POLAR_SHARD_WORDS);
      if (before != nullptr) {
        if (wave == 0) {
          while (load(before) < waiting_for) __builtin_amdgcn_s_sleep(8);
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // (the wavefronts share the caches)
        }
        __syncthreads();
      }
      if (product == 0) {
        bool all = true;
        for (int m = 0; m < p.mats; ++m) {
          const PolarState s = load_state(p.state + (int64_t)step * p.mats + m);
          all = all && (s.mode == POLAR_ENDED || s.last);
        }
        if (all) return;
      }
      for (bool first = true;; first = false) {
        if (wave == 0) {
          int shard = own, chunk = -1;
          for (bool look = !first;; look = true) {
            if (look) {   // a shard with chunks left, the own one first
              const int l = lane % POLAR_SHARDS, sh = (own + l) % POLAR_SHARDS;
              const unsigned long long some = __ballot(sh + POLAR_SHARDS * load(drawn + sh * POLAR_SHARD_WORDS) < chunks);
              if (some == 0) break;
              shard = (own + (int)__builtin_ctzll(some)) % POLAR_SHARDS;
            }
            int v = ahead;
            if (look && lane == 0) v = add1(drawn + shard * POLAR_SHARD_WORDS);
            v = shard + POLAR_SHARDS * __builtin_amdgcn_readfirstlane(v);
            if (v < chunks) { chunk = v; break; }
          }
          if (lane == 0) s_chunk = chunk;
        }
        __syncthreads();
        const int chunk = __builtin_amdgcn_readfirstlane(s_chunk);
        if (chunk < 0) break;
        for (int t = chunk * size; t < min(tasks, (chunk + 1) * size); ++t) {
          const int mat = t / per_mat, tile = t % per_mat;
          if (product == 0) poly_tile<TL, true>(p, step, mat, tile, polar_smem, red);
          else if (product == 1) apply_tile<true>(p, step, mat, tile, polar_smem);
          else gram_tile<TL, true>(p, step + 1, mat, tile, polar_smem, red);
          __syncthreads();   // the LDS is free again
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) {
          const int shard = chunk % POLAR_SHARDS, of = (chunks - shard + POLAR_SHARDS - 1) / POLAR_SHARDS;
          if (add1(done + shard * POLAR_SHARD_WORDS) == of - 1) add1(finished);
        }
      }
      __syncthreads();   // (s_chunk has been read by all)
      waiting_for = chunks < POLAR_SHARDS ? chunks : POLAR_SHARDS;
      before = finished;
      drawn = finished + POLAR_SHARD_WORDS;
    }
}

constexpr int POLAR_QUEUE_WGS = 512;   // (256: a step of rank 512 takes a third longer)

__global__ void __launch_bounds__(256) polar_settle_kernel(const PolarState* state, float* X, int64_t flip, int64_t n) {
  if (!state[blockIdx.y].parity) return;
  float4* dst = (float4*)(X + blockIdx.y * n);
  const float4* src = (const float4*)(X + flip + blockIdx.y * n);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n / 4; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}

// lower triangle tiles of side b
inline int tri_tiles(int r8, int b) { const int n = (r8 + b - 1) / b; return n * (n + 1) / 2; }

}  // namespace

PolarWs make_polar_ws(int mats, int r, int d) {
  PolarWs w = {};
  w.mats = mats; w.r = r; w.d = d;
  w.r8 = round_up(r, 8);
  w.rk = round_up(r, 32);
  w.dk = round_up(d, 32);
  // triangles on 64x64 tiles once those fill the machine (from a rank of about 1000 on)
  w.side = tri_tiles(w.r8, 64) * mats >= 256 ? 64 : 32;
  w.tri = tri_tiles(w.r8, w.side);
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off = align256(off + bytes); return o; };
  w.nx = (int64_t)w.r8 * w.dk;
  w.off_x = take((size_t)2 * mats * w.nx * 4);
  w.off_s = take((size_t)mats * w.r8 * w.rk * 4);
  w.off_t = take((size_t)mats * w.r8 * w.rk * 4);
  const PolarPlan plan = polar_plan(r, d);
  const int queued = plan.max_steps - std::min(polar_launched(plan), plan.max_steps);
  w.queue_words = 3 * queued * (2 * POLAR_SHARDS + 1) * POLAR_SHARD_WORDS;
  w.off_queue = take((size_t)w.queue_words * 4);
  w.off_share = take((size_t)mats * w.tri * 4);
  w.off_rows = take((size_t)mats * 2 * w.r8 * 4);
  w.off_state = take((size_t)(plan.max_steps + 2) * mats * sizeof(PolarState));
  w.bytes = off;
  return w;
}

template <int TL>
static int launch_polar_tl(PolarArgs p, hipStream_t st) {
  constexpr int lds1 = TileProduct<TL, false>::LDS, lds2 = TileProduct<2, true>::LDS;
  const dim3 blk(256), g_tri(p.gram_tiles, p.mats), g_apply(p.apply_tiles, p.mats);
  float coef[POLAR_MAX_STEPS][3];
  if (p.plan.fixed) polar_steps(p.r, coef);
  const int launched = std::min(polar_launched(p.plan), p.plan.max_steps);
  hipLaunchKernelGGL(polar_gram_kernel<TL>, g_tri, blk, lds1, st, p);
  hipLaunchKernelGGL(polar_rows_kernel, dim3((p.r8 + 3) / 4, p.mats), blk, 0, st, p);
  for (int s = 0; s < launched; ++s) {
    p.step = s;
    if (p.plan.fixed) std::copy(coef[s], coef[s] + 3, p.plan.coef);
    hipLaunchKernelGGL(polar_poly_kernel<TL>, g_tri, blk, lds1, st, p);
    hipLaunchKernelGGL(polar_apply_kernel, g_apply, blk, lds2, st, p);
    p.step = s + 1;
    if (s + 1 < p.plan.max_steps) hipLaunchKernelGGL(polar_gram_kernel<TL>, g_tri, blk, lds1, st, p);
    if (hipGetLastError() != hipSuccess) return -1;
  }
  if (launched < p.plan.max_steps) {
    const int tasks = std::max(p.gram_tiles, p.apply_tiles) * p.mats;
    hipLaunchKernelGGL(polar_queue_kernel<TL>, dim3(std::min(POLAR_QUEUE_WGS, tasks)), blk, std::max(lds1, lds2), st, p);
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_polar(const PolarWs& w, char* ws, const PolarState** state, hipStream_t st) {
  PolarArgs p = {};
  p.plan = polar_plan(w.r, w.d);
  p.mats = w.mats; p.r = w.r; p.r8 = w.r8; p.rk = w.rk; p.d = w.d; p.dk = w.dk;
  p.X = (float*)(ws + w.off_x); p.flip = w.mats * w.nx;
  p.S = (float*)(ws + w.off_s); p.T = (float*)(ws + w.off_t);
  p.gram_tiles = p.poly_tiles = w.tri;
  p.apply_tiles = (w.r8 + 63) / 64 * ((w.dk + 63) / 64);
  p.share = (float*)(ws + w.off_share); p.rows = (float*)(ws + w.off_rows);
  p.queue = (unsigned*)(ws + w.off_queue);
  p.result = (PolarState*)(ws + w.off_state);
  p.state = p.result + w.mats;
  *state = p.result;
  return w.side == 64 ? launch_polar_tl<2>(p, st) : launch_polar_tl<1>(p, st);
}

int launch_polar_settle(const PolarWs& w, char* ws, const PolarState* state, hipStream_t st) {
  const int blocks = (int)std::min<int64_t>(1024, (w.nx / 4 + 255) / 256);
  hipLaunchKernelGGL(polar_settle_kernel, dim3(blocks, w.mats), dim3(256), 0, st, state, (float*)(ws + w.off_x),
                     w.mats * w.nx, w.nx);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ffsplit
