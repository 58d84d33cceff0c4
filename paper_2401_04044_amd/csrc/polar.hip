// Polar factor of the sketches of the remainder factorisation (factor.hip): the rows of X [r, d] fp32 become
// orthonormal by X <- (c0 I + c1 G + c2 G^2) X, G = X X^T, with coefficients chosen step by step on the
// device (polar_steps.h).  Per step three products for all matrices of a layer:
//   gram    S = X X^T (one triangle, mirrored) and the tiles' shares of ||S - I||_F^2,
//   poly    the step's coefficients, T - I for T = c0 I + c1 S + c2 S^2 (one triangle, mirrored),
//   apply   X' = X + (T - I) X into the other buffer: near the end T - I is small, and with it the rounding of the sums.
// The host cannot know how many steps a matrix takes and must not wait: it launches as many as the worst sketch may need,
// and the kernels of a step behind a matrix's last return at their first load.  Such a launch costs 3.8 us; up to rank 128
// poly and apply are one.  (The steps from the seventh on in one launch of a work queue, which returned at once when nothing
// was left, took 1.4 to 2.8 times as long a step as launches: 2048 x 7944 rank 512 with singular values i^-2 2030 us, 1608 x
// 4849 rank 800 4530.)
// Measured, us, a factorisation with singular values i^-a, a = 0, 1, 2, two matrices, the steps of polar_steps for every sketch
// / these: 2048 x 7944 rank 512 1130 / 570, 785, 1055; 1536 x 4849 rank 400 gated 1065 / 545, 720, 985; 4096 x 10675 rank 1024
// gated 8150 / 3420, 4940, 6840; 1608 x 4849 rank 800 2097 / 855, 1238, 1812; 512 x 1455 rank 64 260 / 184, 198, 236; 2048 x 7944
// rank 128 478 / 329, -, 480; of rank one, 2048 x 7944 rank 512, 1126 / 1000.  Where every matrix decays like i^-2, which takes one or
// two steps more than the fixed schedule, small ones are slower: 128 x 1000 rank 100 191 / 159, 176, 211; 768 x 2976 rank 128 319 /
// 238, 273, 332; 256 x 776 rank 200 275 / 208, 253, 299; 2048 x 7944 rank 512 1123 / 564, 774, 1038.  (Growth not left any more in its
// last two steps: 202, 328 and 272 there, but 283 with i^-1 at rank 200, which then resumes growth.)
// All products are true fp32 (v_mfma_f32_16x16x4_f32, 256 flop per clock and CU), staged through LDS by loads
// without registers.  A tile asks the caches for 16 (64x64) or 32 bytes per clock of 61: what bounds them is
// the matrix rate, and at the usual ranks the start of a launch and the latency of its first loads.  So the
// triangles take 32x32 tiles (272 workgroups for two matrices of rank 512: 25 us; 64x64 ones cut into seven ranges of
// d, summed by the last to arrive: 31; two or four groups of wavefronts that share a tile's reduction: within 1 %), or 16x16 ones
// where those are few, and rings are seven slabs deep.  Buffer s & 1 holds the X of step s of every matrix that takes that step.
// Of a step's 62 us at rank 512 gram is 25, poly 11, apply 25.
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
// (16 lanes then read 16 different bank groups).  COLS: 32 rows (k) of 32 TL columns, read a float at a time
// without conflicts: TL 2, chunk c of row k at c ^ (4 ((k >> 2) & 3)); TL 1, row k in place k ^ ((k >> 2) & 1) and its
// chunk c at c ^ (4 ((k >> 3) & 1)).
// a_rows, b_rows: rows from the tile's first (rows past the operands repeat the last one: their results are not
// stored); COLS: b_rows is the columns of B from the tile's first, k_rows its rows.
template <int TL, bool COLS>
struct TileProduct {
  static constexpr int OPER = TL * 1024;               // floats of one operand in a stage
  static constexpr int STAGES = TL == 1 ? 7 : 3;       // 56 or 48 KiB: two workgroups a CU and more
  static constexpr int LDS = STAGES * 2 * OPER * 4;
  const float *A, *B;
  float* smem;
  int64_t ldb;
  int k_rows, n, lane, wave;
  int put, get;   // stage that the next slab goes to, that the next one is read from
  uint32_t a_off[TL], b_off[TL], b_last[TL];   // (b_last, COLS: of the last slab)

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
        const int c = TL == 2 ? (lane & 15) ^ (4 * (blk & 3)) : (lane & 7) ^ (4 * (blk & 1));
        const int place = blk * 8 + (lane >> 3), k = TL == 2 ? blk * 4 + (lane >> 4) : place ^ ((place >> 2) & 1);
        const uint32_t col = (uint32_t)(c * 4 < b_rows ? c : 0) * 16;
        b_off[i] = col + (uint32_t)k * (uint32_t)(ldb * 4);
        b_last[i] = col + (uint32_t)min(k, k_rows - 1 - (n - 1) * 32) * (uint32_t)(ldb * 4);
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
        to_lds(B, (lptr_t)(st + OPER + blk * 256), s + 1 < n ? b_off[i] : b_last[i], 0);
      } else {
        to_lds(B, (lptr_t)(st + OPER + blk * 256), b_off[i], (uint32_t)s * 128);
      }
    }
    if (COLS) B += 32 * ldb;   // (X may be larger than the 4 GiB that an offset reaches; slabs are requested in order)
  }

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
          const int c = wn * 16 * TL + j * 16 + r16;
          const int at = ((c >> 2) ^ (TL == 2 ? 4 * quad : 4 * (quad >> 1))) * 4 + (c & 3);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int k = 4 * (quad + 4 * h) + t;
            f.b[h][j][t] = st[OPER + (TL == 2 ? k * 64 : (k ^ (quad & 1)) * 32) + at];
          }
        } else {
          f.b[h][j] = *(const f32x4_t*)(st + OPER + (wn * 16 * TL + j * 16 + r16) * 32 + pos * 4);
        }
      }
    }
  }
  // Sums in NS accumulators of a tile, added in pairs at the end: with one, a chain of 512 roundings at d = 2048, the
  // basis was 6.8e-7 off orthonormal.  (2048 x 7946 rank 512 in fp32, root mean square: 2.3e-7 with these, 1.7e-7 with T - I
  // applied; the products straight from registers had 2.2e-7.)  Every 4096 elements of K they are added up and start again: the
  // matrix unit's roundings do not average out over long chains (32768 x 700: 8.9e-8, 1.5e-6 with products straight from
  // registers; 1048608 x 1100: 2.1e-7, and 5.8e-5 with chains of 65536).
  static constexpr int NS = TL == 1 ? 8 : 4, FOLD = 64;   // (pairs of slabs)
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
  // out += the accumulators, which start again
  __device__ __forceinline__ static void fold(Sums& acc, f32x4_t (&out)[TL][TL]) {
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
      for (int j = 0; j < TL; ++j) {
        out[i][j] += acc[0][i][j];
#pragma unroll
        for (int k = 0; k < NS; ++k) acc[k][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
  }
  // out (zero) = the product; the fragments of a slab are read while the one before is multiplied
  __device__ __forceinline__ void run(f32x4_t (&out)[TL][TL]) {
    Sums acc = {};
    Frags f0, f1;
    advance(0);
    read(f0);
    int s = 1;
    auto pairs = [&](int end) {
      for (; s + 1 < end; s += 2) {
        advance(s);
        read(f1);
        mma(f0, acc);
        advance(s + 1);
        read(f0);
        mma(f1, acc);
      }
    };
    // (a loop of its own: with the fold inside the one that short products take these were 5 % slower)
    while (__builtin_expect(n - s > 2 * FOLD, 0)) {
      pairs(s + 2 * FOLD);
      fold(acc, out);
    }
    pairs(n);
    if (s < n) {
      advance(s);
      read(f1);
      mma(f0, acc);
      mma(f1, acc);
    } else {
      mma(f0, acc);
    }
    fold(acc, out);
  }
};

struct PolarArgs {
  PolarPlan plan;
  PolarState* state;     // [max_steps + 1][mats]: state[s] is what step s starts from, for steps carried out
  PolarState* result;    // [mats]: behind the last step carried out
  int* ended;            // [mats]: that step, a large number before it is known
  int step, mats, r, r8, rk, d, dk;
  float* X;              // [2][mats][r8, dk]
  int64_t flip;          // elements between the two buffers
  float* S;              // [mats][r8, rk]
  float* T;              // (T - I)
  int shares;
  float* share;          // [mats][shares]: the gram tiles' shares of ||S - I||_F^2
  float* rows;           // [mats][2][r8]: sums of |S| and of S^2 along its rows
  int may_be_idle;       // matrices may have ended before this step: its kernels look before they request anything
};

// lower triangle, row by row: tile t is (i, j <= i)
__device__ __forceinline__ void triangle(int t, int& i, int& j) {
  i = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  while (i * (i + 1) / 2 > t) --i;
  j = t - i * (i + 1) / 2;
}

// sum over a wavefront in a fixed order, in every lane
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// four columns col .. of a row of a symmetric matrix [r8, rk], and their mirror images; what lies in
// the padding columns is written as zero
__device__ __forceinline__ void store_sym(float* S, int r8, int rk, int row, int col, bool mirror, f32x4_t v) {
  if (row < r8 && col < rk) *(f32x4_t*)(S + (int64_t)row * rk + col) = col < r8 ? v : f32x4_t{0.f, 0.f, 0.f, 0.f};
  if (mirror && row < rk && col < r8) {
#pragma unroll
    for (int e = 0; e < 4; ++e) S[(int64_t)(col + e) * rk + row] = row < r8 ? v[e] : 0.f;
  }
}

// the S that step p.step starts from
template <int TL>
__global__ void __launch_bounds__(256) polar_gram_kernel(const PolarArgs p) {
  constexpr int B = 32 * TL;
  extern __shared__ float polar_smem[];
  __shared__ float red[4];
  const int mat = blockIdx.y, tile = blockIdx.x;
  if (p.may_be_idle && p.ended[mat] < p.step) return;
  int tm, tn;
  triangle(tile, tm, tn);
  const float* X = p.X + (p.step & 1) * p.flip + (int64_t)mat * p.r8 * p.dk;
  TileProduct<TL, false> prod;
  prod.start(X + (int64_t)tm * B * p.dk, p.dk, p.r8 - tm * B, X + (int64_t)tn * B * p.dk, p.dk, p.r8 - tn * B, 0, p.dk / 32,
             polar_smem);
  f32x4_t acc[TL][TL] = {};
  prod.run(acc);
  const int lane = prod.lane, wave = prod.wave;
  float* S = p.S + (int64_t)mat * p.r8 * p.rk;
  float dev = 0.f;
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j) {
      const int row = tm * B + (wave >> 1) * 16 * TL + i * 16 + (lane & 15);
      const int col = tn * B + (wave & 1) * 16 * TL + j * 16 + 4 * (lane >> 4);
      store_sym(S, p.r8, p.rk, row, col, tm != tn, acc[i][j]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = acc[i][j][e] - (row == col + e ? 1.f : 0.f);
        if (row < p.r && col + e < p.r) dev = fmaf(x, x, dev);
      }
    }
  dev = wave_sum(dev);
  if (lane == 0) red[wave] = dev;
  __syncthreads();
  if (threadIdx.x == 0) {
    dev = ((red[0] + red[1]) + red[2]) + red[3];
    p.share[(int64_t)mat * p.shares + tile] = tm != tn ? 2.f * dev : dev;
  }
}

// A 16 x 16 block of a row-major operand for the MFMA, straight from the caches.  Four neighbouring lanes load one 64-byte
// piece, lane l chunk l & 3 of row l >> 2 (where every lane has a row of its own, as the MFMA wants it, the vector cache
// delivers 16 bytes a clock instead of 61), and the wavefront turns the block round in 1 KiB of LDS of its own: lane
// (r16, quad) gets the elements 4 quad .. + 3 of row r16.
__device__ __forceinline__ f32x4_t turn_round(f32x4_t v, f32x4_t* area) {
  const int l = threadIdx.x & 63, r = l & 15;
  area[(l & ~3) | ((l & 3) ^ ((l >> 4) & 3))] = v;
  return area[r * 4 + ((l >> 4) ^ (r >> 2))];
}

// The same for few tiles: 16x16 ones on 16 wavefronts, which take every 16th slab of 16, eight in flight, and meet in LDS.
// (32x32 tiles of rank 128 are 20 workgroups for two matrices, and a chain of 64 slabs at d = 2048.)
__global__ void __launch_bounds__(1024) polar_gram16_kernel(const PolarArgs p) {
  __shared__ f32x4_t area[2][16][64];
  const int mat = blockIdx.y, tile = blockIdx.x, lane = threadIdx.x & 63, r16 = lane & 15, quad = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (p.may_be_idle && p.ended[mat] < p.step) return;
  int tm, tn;
  triangle(tile, tm, tn);
  const float* const X = p.X + (p.step & 1) * p.flip + (int64_t)mat * p.r8 * p.dk + 4 * (lane & 3);
  const float* const xa = X + (int64_t)min(tm * 16 + (lane >> 2), p.r8 - 1) * p.dk;
  const float* const xb = X + (int64_t)min(tn * 16 + (lane >> 2), p.r8 - 1) * p.dk;
  f32x4_t acc[4] = {};
  const int slabs = p.dk / 16;
  for (int s0 = wave; s0 < slabs; s0 += 16 * 8) {
    f32x4_t a[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {   // (past the last slab: it again, not used)
      const int s = min(s0 + 16 * u, slabs - 1);
      a[u] = *(const f32x4_t*)(xa + s * 16);
      b[u] = *(const f32x4_t*)(xb + s * 16);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (s0 + 16 * u < slabs) {
        const f32x4_t ta = turn_round(a[u], area[0][wave]), tb = turn_round(b[u], area[1][wave]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(tb[e], ta[e], acc[e], 0, 0, 0);
      }
  }
  area[0][wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (wave != 0) return;
  f32x4_t v = area[0][0][lane];
#pragma unroll
  for (int w = 1; w < 16; ++w) v += area[0][w][lane];
  const int row = tm * 16 + r16, col = tn * 16 + 4 * quad;
  store_sym(p.S + (int64_t)mat * p.r8 * p.rk, p.r8, p.rk, row, col, tm != tn, v);
  float dev = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = v[e] - (row == col + e ? 1.f : 0.f);
    if (row < p.r && col + e < p.r) dev = fmaf(x, x, dev);
  }
  dev = wave_sum(dev);
  if (lane == 0) p.share[(int64_t)mat * p.shares + tile] = tm != tn ? 2.f * dev : dev;
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

// What the choice of step p.step needs: the state and the first 256 shares, requested ahead of everything else.  Then the
// choice itself: its coefficients, and from the thread that `writes` the state behind the step.  Every wavefront adds up
// the shares by itself, so that no LDS is read: loads return in order, and those on their way into LDS need not be
// waited for.
__device__ __forceinline__ void request_choice(const PolarArgs& p, int mat, PolarState& s, float (&first)[4]) {
  const int lane = threadIdx.x & 63;
  if (p.step > 0) s = p.state[(int64_t)p.step * p.mats + mat];
  const float* const share = p.share + (int64_t)mat * p.shares;
#pragma unroll
  for (int u = 0; u < 4; ++u) first[u] = p.step > 0 && lane + 64 * u < p.shares ? share[lane + 64 * u] : 0.f;
}
__device__ __forceinline__ void choose(const PolarArgs& p, int mat, bool writes, PolarState s, const float (&first)[4], float (&c)[3]) {
  const int lane = threadIdx.x & 63;
  float fig, sum = ((first[0] + first[1]) + first[2]) + first[3];
  if (p.step == 0) {
    const float* rows = p.rows + (int64_t)mat * 2 * p.r8;
    float most = 0.f;
    for (int i = lane; i < p.r; i += 64) { most = fmaxf(most, rows[i]); sum += rows[p.r8 + i]; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = fmaxf(most, __shfl_xor(most, o));
    fig = sqrtf(fminf(most, sqrtf(wave_sum(sum))));
  } else {
    for (int i = lane + 256; i < p.shares; i += 64) sum += p.share[(int64_t)mat * p.shares + i];
    fig = wave_sum(sum);
  }
  s = polar_decide(p.plan, p.step, p.r, s, fig, c);
  if (writes && threadIdx.x == 0) {
    p.state[(int64_t)(p.step + 1) * p.mats + mat] = s;
    p.result[mat] = s;
    p.ended[mat] = s.last ? p.step : 1 << 30;
  }
}

// an element of T - I.  In the last steps the three terms of the diagonal, 0.875 - 1.25 + 0.375, cancel: in this order the
// one rounding that stays is that of their difference.  (|| B B^T - I ||_F / sqrt(r) at 2048 x 2600 rank 512: 1.6e-7; with
// c1 g rounded by itself 1.8e-7.)
__device__ __forceinline__ float t_minus_i(const float (&c)[3], float ss, float s, bool diagonal) {
  return fmaf(c[2], ss, fmaf(c[1], s, diagonal ? c[0] - 1.f : 0.f));
}

// T - I for step p.step
template <int TL>
__global__ void __launch_bounds__(256) polar_poly_kernel(const PolarArgs p) {
  constexpr int B = 32 * TL;
  extern __shared__ float polar_smem[];
  const int mat = blockIdx.y, tile = blockIdx.x, lane = threadIdx.x & 63;
  // (the launch's first tile may have named this very step by now; where there is nothing to do nothing is stored, which
  // would cost the end of the launch 2 us)
  if (p.may_be_idle && p.ended[mat] < p.step) return;
  PolarState s = {};
  float first[4];
  request_choice(p, mat, s, first);
  int tm, tn;
  triangle(tile, tm, tn);
  const float* S = p.S + (int64_t)mat * p.r8 * p.rk;
  TileProduct<TL, false> prod;
  prod.start(S + (int64_t)tm * B * p.rk, p.rk, p.r8 - tm * B, S + (int64_t)tn * B * p.rk, p.rk, p.r8 - tn * B, 0, p.rk / 32,
             polar_smem);
  const int row0 = tm * B + (prod.wave >> 1) * 16 * TL + (lane & 15), col0 = tn * B + (prod.wave & 1) * 16 * TL + 4 * (lane >> 4);
  f32x4_t g[TL][TL];
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j)
      g[i][j] = row0 + i * 16 < p.r8 && col0 + j * 16 < p.rk ? *(const f32x4_t*)(S + (int64_t)(row0 + i * 16) * p.rk + col0 + j * 16)
                                                             : f32x4_t{0.f, 0.f, 0.f, 0.f};
  float c[3];
  choose(p, mat, tile == 0, s, first, c);
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
      for (int e = 0; e < 4; ++e) v[e] = t_minus_i(c, acc[i][j][e], g[i][j][e], row == col + e);
      store_sym(T, p.r8, p.rk, row, col, tm != tn, v);
    }
}

// the X behind step p.step
template <int TL>
__global__ void __launch_bounds__(256) polar_apply_kernel(const PolarArgs p) {
  constexpr int B = 32 * TL;
  extern __shared__ float polar_smem[];
  const int mat = blockIdx.y, tiles_m = (p.r8 + B - 1) / B, tm = blockIdx.x % tiles_m, tn = blockIdx.x / tiles_m;
  if (p.may_be_idle && p.ended[mat] < p.step) return;
  const int64_t at = (int64_t)mat * p.r8 * p.dk;
  const float* T = p.T + (int64_t)mat * p.r8 * p.rk + (int64_t)tm * B * p.rk;
  const float* X = p.X + (p.step & 1) * p.flip + at;
  TileProduct<TL, true> prod;
  prod.start(T, p.rk, p.r8 - tm * B, X + tn * B, p.dk, p.dk - tn * B, p.r8, p.rk / 32, polar_smem);
  const int lane = prod.lane, wave = prod.wave;
  f32x4_t x[TL][TL];
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j) {
      const int row = tm * B + (wave >> 1) * 16 * TL + i * 16 + (lane & 15);
      const int col = tn * B + (wave & 1) * 16 * TL + j * 16 + 4 * (lane >> 4);
      x[i][j] = row < p.r8 && col < p.dk ? *(const f32x4_t*)(X + (int64_t)row * p.dk + col) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  f32x4_t acc[TL][TL] = {};
  prod.run(acc);
  float* O = p.X + ((p.step & 1) ^ 1) * p.flip + at;
#pragma unroll
  for (int i = 0; i < TL; ++i)
#pragma unroll
    for (int j = 0; j < TL; ++j) {
      const int row = tm * B + (wave >> 1) * 16 * TL + i * 16 + (lane & 15);
      const int col = tn * B + (wave & 1) * 16 * TL + j * 16 + 4 * (lane >> 4);
      if (row < p.r8 && col < p.dk) *(f32x4_t*)(O + (int64_t)row * p.dk + col) = col < p.d ? x[i][j] + acc[i][j] : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
}

// poly and apply in one launch for r <= RK: a workgroup works out the 32 rows of T - I that its 32x32 tile of X' needs
// (turn_round) and keeps them in LDS.  Up to rank 128 that is 1 MFLOP a workgroup, and a launch less a step, carried out or not.
template <int RK>
__global__ void __launch_bounds__(256, 2) polar_poly_apply_kernel(const PolarArgs p) {
  constexpr int NK = RK / 16, CB = RK / 64, LD = RK + 4;   // slabs of K; blocks of 16 columns of T a wavefront
  __shared__ __align__(16) float t[32 * LD];
  __shared__ f32x4_t area[4][64];
  const int mat = blockIdx.y, tiles_m = (p.r8 + 31) / 32, tm = blockIdx.x % tiles_m, tn = blockIdx.x / tiles_m;
  const int lane = threadIdx.x & 63, r16 = lane & 15, quad = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1;
  if (p.may_be_idle && p.ended[mat] < p.step) return;
  PolarState s = {};
  float first[4];
  request_choice(p, mat, s, first);
  const float* S = p.S + (int64_t)mat * p.r8 * p.rk;
  const float* X = p.X + (p.step & 1) * p.flip + (int64_t)mat * p.r8 * p.dk + tn * 32 + wn * 16;
  auto at_s = [&](int row, int col) {   // (past rk: zero; past r8: the last row, not used)
    return col < p.rk ? *(const f32x4_t*)(S + (int64_t)min(row, p.r8 - 1) * p.rk + col) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  f32x4_t sa[2][NK], sb[CB][NK], g[2][CB];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
#pragma unroll
    for (int i = 0; i < 2; ++i) sa[i][k] = at_s(tm * 32 + i * 16 + (lane >> 2), k * 16 + 4 * (lane & 3));
#pragma unroll
    for (int j = 0; j < CB; ++j) sb[j][k] = at_s((wave * CB + j) * 16 + (lane >> 2), k * 16 + 4 * (lane & 3));
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) g[i][j] = at_s(tm * 32 + i * 16 + r16, (wave * CB + j) * 16 + 4 * quad);
  const int row = tm * 32 + wm * 16 + r16;   // of X'
  const f32x4_t old = *(const f32x4_t*)(X + (int64_t)min(row, p.r8 - 1) * p.dk + 4 * quad);
  f32x4_t x[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) x[k][e] = X[(int64_t)min(k * 16 + 4 * quad + e, p.r8 - 1) * p.dk + r16];   // (T is zero past r8)
  float c[3];
  choose(p, mat, blockIdx.x == 0, s, first, c);
  f32x4_t acc[2][2][CB] = {};
#pragma unroll
  for (int k = 0; k < NK; ++k) {
#pragma unroll
    for (int i = 0; i < 2; ++i) sa[i][k] = turn_round(sa[i][k], area[wave]);
#pragma unroll
    for (int j = 0; j < CB; ++j) sb[j][k] = turn_round(sb[j][k], area[wave]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j)
          acc[e & 1][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(sb[j][k][e], sa[i][k][e], acc[e & 1][i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const int col = (wave * CB + j) * 16 + 4 * quad;
      f32x4_t v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float sum = acc[0][i][j][e] + acc[1][i][j][e];
        v[e] = col + e < p.r8 ? t_minus_i(c, sum, g[i][j][e], tm * 32 + i * 16 + r16 == col + e) : 0.f;
      }
      *(f32x4_t*)(t + (i * 16 + r16) * LD + col) = v;
    }
  __syncthreads();
  f32x4_t y[4] = {};
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const f32x4_t a = *(const f32x4_t*)(t + (wm * 16 + r16) * LD + k * 16 + 4 * quad);
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[k][e], a[e], y[e], 0, 0, 0);
  }
  const f32x4_t v = old + ((y[0] + y[1]) + (y[2] + y[3]));
  const int col = tn * 32 + wn * 16 + 4 * quad;
  float* O = p.X + ((p.step & 1) ^ 1) * p.flip + (int64_t)mat * p.r8 * p.dk;
  if (row < p.r8) *(f32x4_t*)(O + (int64_t)row * p.dk + col) = col < p.d ? v : f32x4_t{0.f, 0.f, 0.f, 0.f};
}

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
  // X X^T on 64x64 tiles once those fill the machine (from a rank of about 1000 on), on 16x16 ones where those are few; up
  // to 512 of them where the reduction is long.  Both sides (us, a factorisation of a flat / an i^-2 remainder, two matrices,
  // 32x32 / 16x16): 4096 x 10675 rank 256, 272 tiles, 765 / 733 and 1156 / 1046; 2048 x 7944 rank 300, 380 tiles, 473 / 464 and
  // 755 / 707; 512 x 1455 rank 300 379 / 392.
  const int t16 = tri_tiles(w.r8, 16) * mats;
  w.side = tri_tiles(w.r8, 64) * mats >= 256 ? 64 : t16 <= (d >= 1024 ? 512 : 256) ? 16 : 32;
  w.tri = tri_tiles(w.side == 16 ? w.rk : w.r8, w.side);   // (they write the padding columns of S)
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off = align256(off + bytes); return o; };
  w.nx = (int64_t)w.r8 * w.dk;
  w.off_x = take((size_t)2 * mats * w.nx * 4);
  w.off_s = take((size_t)mats * w.r8 * w.rk * 4);
  w.off_t = take((size_t)mats * w.r8 * w.rk * 4);
  w.off_share = take((size_t)mats * w.tri * 4);
  w.off_rows = take((size_t)mats * 2 * w.r8 * 4);
  w.off_state = take((size_t)(polar_plan(r, d).max_steps + 2) * mats * sizeof(PolarState));
  w.off_ended = take((size_t)mats * 4);
  w.bytes = off;
  return w;
}

// GRAM: side of the tiles of S, 16 to 64; FUSED: 0, or the rank up to which poly and apply are one launch
template <int GRAM, int TA, int FUSED>
static int launch_polar_as(PolarArgs p, hipStream_t st) {
  constexpr int TL = GRAM == 64 ? 2 : 1, lds1 = TileProduct<TL, false>::LDS, lds2 = TileProduct<TA, true>::LDS;
  const dim3 blk(256), g_gram(p.shares, p.mats), g_poly(tri_tiles(p.r8, 32 * TL), p.mats);
  const dim3 g_apply((p.r8 + 32 * TA - 1) / (32 * TA) * ((p.dk + 32 * TA - 1) / (32 * TA)), p.mats);
  float coef[POLAR_MAX_STEPS][3];
  if (p.plan.fixed) polar_steps(p.r, coef);
  auto gram = [&] {
    if constexpr (GRAM == 16) hipLaunchKernelGGL(polar_gram16_kernel, g_gram, dim3(1024), 0, st, p);
    else hipLaunchKernelGGL(polar_gram_kernel<TL>, g_gram, blk, lds1, st, p);
  };
  gram();
  hipLaunchKernelGGL(polar_rows_kernel, dim3((p.r8 + 3) / 4, p.mats), blk, 0, st, p);
  for (int s = 0; s < p.plan.max_steps; ++s) {
    p.step = s;
    p.may_be_idle = !p.plan.fixed && s >= POLAR_LEAST_STEPS;
    if (p.plan.fixed) std::copy(coef[s], coef[s] + 3, p.plan.coef);
    if constexpr (FUSED > 0) {
      hipLaunchKernelGGL(polar_poly_apply_kernel<FUSED>, g_apply, blk, 0, st, p);
    } else {
      hipLaunchKernelGGL(polar_poly_kernel<TL>, g_poly, blk, lds1, st, p);
      hipLaunchKernelGGL(polar_apply_kernel<TA>, g_apply, blk, lds2, st, p);
    }
    p.step = s + 1;
    p.may_be_idle = !p.plan.fixed && s + 1 >= POLAR_LEAST_STEPS;
    if (s + 1 < p.plan.max_steps) gram();
    if (hipGetLastError() != hipSuccess) return -1;
  }
  return 0;
}

int launch_polar(const PolarWs& w, char* ws, const PolarState** state, hipStream_t st) {
  PolarArgs p = {};
  p.plan = polar_plan(w.r, w.d);
  p.mats = w.mats; p.r = w.r; p.r8 = w.r8; p.rk = w.rk; p.d = w.d; p.dk = w.dk;
  p.X = (float*)(ws + w.off_x); p.flip = w.mats * w.nx;
  p.S = (float*)(ws + w.off_s); p.T = (float*)(ws + w.off_t);
  p.shares = w.tri;
  p.share = (float*)(ws + w.off_share); p.rows = (float*)(ws + w.off_rows);
  p.result = (PolarState*)(ws + w.off_state);
  p.state = p.result + w.mats;
  p.ended = (int*)(ws + w.off_ended);
  *state = p.result;
  if (w.side == 64) return launch_polar_as<64, 2, 0>(p, st);
  // poly and apply together while the workgroups (four of rank 64 a CU, two of rank 128) are one round of the machine: us as
  // above, apart / together, 512 x 1455 rank 64 224 / 186 and 287 / 255, 1024 x 3972 rank 128 292 / 258 and 398 / 401, 4096 x 10675
  // rank 64 (512 workgroups) 513 / 485 and 635 / 613, 2048 x 7944 rank 128 (512) 344 / 329 and 460 / 480
  const int wgs = (w.r8 + 31) / 32 * (w.dk / 32) * w.mats;
  // the last product on 32x32 tiles where 64x64 ones do not fill the machine (512 x 1455 rank 300: 412 -> 373)
  const bool small = (w.r8 + 63) / 64 * ((w.dk + 63) / 64) * w.mats < 256;
  if (w.side == 16) {
    if (w.r <= 64 && wgs <= 1024) return launch_polar_as<16, 1, 64>(p, st);
    if (w.r > 64 && w.r <= 128 && wgs <= 512) return launch_polar_as<16, 1, 128>(p, st);
    return small ? launch_polar_as<16, 1, 0>(p, st) : launch_polar_as<16, 2, 0>(p, st);
  }
  return small ? launch_polar_as<32, 1, 0>(p, st) : launch_polar_as<32, 2, 0>(p, st);
}

int launch_polar_settle(const PolarWs& w, char* ws, const PolarState* state, hipStream_t st) {
  const int blocks = (int)std::min<int64_t>(1024, (w.nx / 4 + 255) / 256);
  hipLaunchKernelGGL(polar_settle_kernel, dim3(blocks, w.mats), dim3(256), 0, st, state, (float*)(ws + w.off_x),
                     w.mats * w.nx, w.nx);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ffsplit
