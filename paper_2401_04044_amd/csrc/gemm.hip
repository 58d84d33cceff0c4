// fp32 GEMM of the split feed-forward path (the bf16 MFMA kernel is gemm_bf16.hip).
//
//   D[M, N] = A[M, K] * Bt[N, K]^T        (both operands row-major, K-contiguous)
//
// followed by one of the fused epilogues the path needs:
//   - store (optionally exact GeLU, or SwiGLU on (gate, up) pairs of 32-column
//     blocks), with the output columns routed to two destinations;
//   - score: per-row-tile column sums of h^2 and |h| (the neuron-norm reduction
//     of Sec. 4.1, Eq. 3), h never leaving registers.
// True fp32 products (v_mfma_f32_16x16x4_f32) and the erf form of GeLU: the error bar is 1e-5.
//
// Every wavefront moves its own operands, no barrier in the loop: the fp32 matrix rate is a
// sixteenth of the bf16 one, so even a 32x32 wave tile asks for 32 bytes per clock and CU where the
// vector cache delivers 61.  It does so only if four neighbouring lanes read one 64-byte piece
// (16 bytes per clock where every lane has its own row, the order the MFMA wants), so lane l loads chunk l & 3 of row l >> 2 of a 16 x 16 block and the wavefront
// turns the block round in 1 KiB of LDS of its own: lane l then holds k elements 4 (l >> 4) .. + 3 of row
// l & 15, and element t of both operands' registers feeds MFMA t of the slab (any pairing of k
// works as long as both sides use the same).  PF slabs are in flight per wavefront.
// A workgroup is WGM x WGN wavefronts per k group and KW k groups, which take every KW-th slab and
// add their accumulators through LDS in a fixed order: products of a hundred tokens are bound by
// the latency of their chain of slabs, and this shortens it without partial sums in memory or a
// second launch.  (BERT-base layer, 128 tokens: six launches with split reductions took 63 us, four 26.6, with short
// and long reductions on tiles and ranges of their own 20.6.)
#include "common.h"
#include <algorithm>

namespace ffsplit {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// 16 bytes at base + lane_off + scalar_off; a lane offset of ~0 is out of range and reads zero
__device__ __forceinline__ f32x4_t buffer_f32x4(const float* base, uint32_t lane_off, uint32_t scalar_off) {
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
  const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(
      __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0xfffffff0u, 0x00027000), lane_off, scalar_off, 0);
  f32x4_t f;
  __builtin_memcpy(&f, &v, 16);
  return f;
}

// FIX: the reduction is cut into gridDim.y ranges, added in range order by the last workgroup of a tile to
// arrive (one wavefront a tile: its store, its arrival and its reads are in order by themselves).
constexpr int F32_MAX_SPLIT = 8;
template <int TM, int TN, int WGM, int WGN, int KW, int PF, int ACT, bool DUAL, bool SCORE, bool FIX>
__global__ void __launch_bounds__(WGM* WGN* KW * 64) gemm_f32_kernel(const GemmArgs p) {
  constexpr int BM = WGM * TM * 16, BN = WGN * TN * 16;
  constexpr int NA = DUAL ? 2 : 1;
  static_assert(ACT != ACT_GLU || TN == 4, "a (gate, up) pair of 32-column blocks per wavefront");
  extern __shared__ float f32_smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = wave / (WGM * WGN), wt = wave % (WGM * WGN), wm = wt / WGN, wn = wt % WGN;
  static_assert(!FIX || (TM * TN * WGM * WGN == 1 && KW > 1 && ACT == ACT_NONE && !SCORE), "");
  if (!FIX && blockIdx.x == 0)
    for (int i = tid; i < p.n_clear; i += WGM * WGN * KW * 64) p.clear[i] = 0u;
  const int tiles_n = (p.N + BN - 1) / BN;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int m0 = tm * BM + wm * TM * 16, n0 = tn * BN + wn * TN * 16;   // the wavefront's corner
  const int r16 = lane & 15, quad = lane >> 4;

  // Buffer loads: the wavefront's corner in scalar registers, one byte offset per row tile, a scalar
  // offset along K (rows past the end repeat the last one).  A chunk past K takes an offset beyond the range, which reads as zero: no branch
  // stands between the loads, so the waits for them stay exact.
  uint32_t a_off[TM], b_off[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    a_off[i] = (uint32_t)(min(i * 16 + (lane >> 2), max(p.M - 1 - m0, 0)) * (int)p.lda + 4 * (lane & 3)) * 4;
#pragma unroll
  for (int j = 0; j < TN; ++j)
    b_off[j] = (uint32_t)(min(j * 16 + (lane >> 2), max(p.N - 1 - n0, 0)) * (int)p.ldb + 4 * (lane & 3)) * 4;
  const float* const a_base = (const float*)p.A + (int64_t)min(m0, p.M - 1) * p.lda;
  const float* const a1_base = DUAL ? (const float*)p.A1 + (int64_t)min(m0, p.M - 1) * p.lda : a_base;
  const float* const b_base = (const float*)p.Bt + (int64_t)min(n0, p.N - 1) * p.ldb;

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int all = (p.K + 15) / 16;
  const int base = FIX ? (int)((uint32_t)all * blockIdx.y / gridDim.y) : 0;
  const int slabs = (FIX ? (int)((uint32_t)all * (blockIdx.y + 1) / gridDim.y) : all) - base;
  const int k_end = FIX ? min(p.K, (base + slabs) * 16) : p.K;
  const int n = (slabs - kw + KW - 1) / KW;   // this k group's slabs: kw, kw + KW, ...
  f32x4_t ga[PF][NA][TM], gb[PF][TN];   // in flight, as loaded
  f32x4_t fa[2][NA][TM], fb[2][TN];     // the slab being multiplied and the next one
  auto load = [&](int slot, int i) {
    const int k0 = (base + kw + i * KW) * 16;
    const bool ok = k0 + 4 * (lane & 3) < k_end;   // (K is a multiple of 4: whole chunks)
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      ga[slot][0][t] = buffer_f32x4(a_base, ok ? a_off[t] : ~0u, k0 * 4);
      if (DUAL) ga[slot][NA - 1][t] = buffer_f32x4(a1_base, ok ? a_off[t] : ~0u, k0 * 4);
    }
#pragma unroll
    for (int t = 0; t < TN; ++t) gb[slot][t] = buffer_f32x4(b_base, ok ? b_off[t] : ~0u, k0 * 4);
  };
  // Chunk c of row r of a block sits at 4 r + (c ^ (r >> 2)): 16 consecutive lanes write 256
  // contiguous bytes and read 16 different 16-byte bank groups.  A wavefront's LDS accesses stay in order.
  constexpr int BLKS = NA * TM + TN;
  f32x4_t* const turn = (f32x4_t*)f32_smem + wave * BLKS * 64;
  const int put_at = (lane & ~3) | ((lane & 3) ^ ((lane >> 4) & 3));
  const int get_at = r16 * 4 + (quad ^ (r16 >> 2));
  auto turn_round = [&](int slot, int set) {
#pragma unroll
    for (int s = 0; s < NA; ++s)
#pragma unroll
      for (int t = 0; t < TM; ++t) turn[(s * TM + t) * 64 + put_at] = ga[slot][s][t];
#pragma unroll
    for (int t = 0; t < TN; ++t) turn[(NA * TM + t) * 64 + put_at] = gb[slot][t];
#pragma unroll
    for (int s = 0; s < NA; ++s)
#pragma unroll
      for (int t = 0; t < TM; ++t) fa[set][s][t] = turn[(s * TM + t) * 64 + get_at];
#pragma unroll
    for (int t = 0; t < TN; ++t) fb[set][t] = turn[(NA * TM + t) * 64 + get_at];
  };
  auto mma = [&](int set) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const float a = fa[set][DUAL ? (j >> 1) & 1 : 0][i][t], b = fb[set][j][t];
          acc[i][j] = SCORE ? __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[i][j], 0, 0, 0)
                            : __builtin_amdgcn_mfma_f32_16x16x4f32(b, a, acc[i][j], 0, 0, 0);
        }
  };
  static_assert(PF % 2 == 0, "the register set of slab i is i & 1");
#pragma unroll
  for (int u = 0; u < PF; ++u) load(u, u);
  turn_round(0, 0);
  load(0, PF);
  int i = 0;
  for (; i + PF <= n; i += PF)
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      __builtin_amdgcn_sched_barrier(0);   // keeps PF slabs in flight: the loads are not gathered
      turn_round((u + 1) % PF, (u + 1) & 1);   // slab i + u + 1 (zeros past the end)
      load((u + 1) % PF, i + u + 1 + PF);
      mma(u & 1);
    }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < PF - 1; ++u)
    if (i + u < n) {
      mma(u & 1);
      if (u + 1 < PF - 1) turn_round((u + 1) % PF, (u + 1) & 1);
    }

  if constexpr (KW > 1) {
    // Sum over the k groups: all but the first park their accumulators, then every wavefront adds
    // up its share of the tiles and hands the sums to the first group.
    constexpr int TILES = WGM * WGN * TM * TN;
    f32x4_t* sm = (f32x4_t*)f32_smem;   // [KW][TILES][64], over the wavefronts' turning blocks
    __syncthreads();
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b) sm[((kw * WGM * WGN + wt) * TM * TN + a * TN + b) * 64 + lane] = acc[a][b];
    __syncthreads();
    for (int t = wave; t < TILES; t += WGM * WGN * KW) {
      f32x4_t v = sm[t * 64 + lane];
#pragma unroll
      for (int g = 1; g < KW; ++g) v += sm[(g * TILES + t) * 64 + lane];
      sm[t * 64 + lane] = v;
    }
    __syncthreads();
    if (kw != 0 && !SCORE) return;
    if (kw == 0) {
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = sm[(wt * TM * TN + a * TN + b) * 64 + lane];
    }
  }
  if constexpr (FIX) {
    unsigned long long* q = (unsigned long long*)p.fix_part + ((int64_t)blockIdx.x * gridDim.y * 64 + lane) * 2;
    auto bits = [](float a, float b) { return (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32); };
#pragma unroll
    for (int h = 0; h < 2; ++h)
      __hip_atomic_store(q + (int64_t)blockIdx.y * 128 + h, bits(acc[0][0][2 * h], acc[0][0][2 * h + 1]), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    unsigned before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(p.fix_cnt + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) != gridDim.y - 1) return;
    if (lane == 0) __hip_atomic_store(p.fix_cnt + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long v[F32_MAX_SPLIT][2];
#pragma unroll
    for (int s = 0; s < F32_MAX_SPLIT; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        v[s][h] = __hip_atomic_load(q + (int64_t)min(s, (int)gridDim.y - 1) * 128 + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    f32x4_t t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < F32_MAX_SPLIT; ++s)
      if (s < (int)gridDim.y)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] += __uint_as_float((unsigned)(v[s][e >> 1] >> (32 * (e & 1))));
    acc[0][0] = t;
  }

  if (!SCORE) {
    // lane: row r16, columns 4 quad + 0..3 of each 16x16 tile
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int cb = n0 + j * 16;
      if (cb >= p.N) continue;
      const bool glu_here = ACT == ACT_GLU && cb < p.act_cols;
      if (glu_here && j >= 2) continue;
      const int oc = ACT == ACT_GLU ? (glu_here ? (cb >> 6) * 32 + (cb & 31) : cb - p.act_cols / 2) : cb;
      const bool to_c0 = oc < p.split_col;
      float* base = to_c0 ? (float*)p.C0 + oc : (float*)p.C1 + (oc - p.split_col);
      const int64_t ld = to_c0 ? p.ldc0 : p.ldc1;
#pragma unroll
      for (int i2 = 0; i2 < TM; ++i2) {
        const int row = m0 + i2 * 16 + r16;
        if (row >= p.M) continue;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int c = cb + 4 * quad + e;
          // (a neuron's bias before the activation; the output bias of an un-activated product)
          const float bz = (ACT != ACT_GLU && p.bias != nullptr && c < p.bias_cols) ? p.bias[c] : 0.f;
          const float z = acc[i2][j][e];
          if (ACT == ACT_GLU) v[e] = glu_here ? silu_f(z) * acc[i2][(j + 2) % TN][e] : z;
          else if (ACT == ACT_GELU) v[e] = c < p.act_cols ? gelu_f(z + bz) : z + bz;
          else v[e] = z + bz;
          if (p.resid != nullptr && to_c0 && c < p.N) v[e] += p.resid[(int64_t)row * p.ldr + oc + 4 * quad + e];
        }
        float* dst = base + (int64_t)row * ld + 4 * quad;
        // (the columns of one 16-byte piece share a destination: split_col is a multiple of 4)
        if (cb + 4 * quad + 3 < p.N) {
          *(f32x4_t*)dst = f32x4_t{v[0], v[1], v[2], v[3]};
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (cb + 4 * quad + e < p.N) dst[e] = v[e];
        }
      }
    }
  } else {
    // lane: column r16, rows 4 quad + 0..3 of each tile; one workgroup covers BM = 64 rows
    constexpr int BNO = (ACT == ACT_GLU) ? BN / 2 : BN;
    float* red2 = f32_smem;             // [WGM][BNO] (after the sum over the k groups has been read)
    float* red1 = red2 + WGM * BNO;
    __syncthreads();
    if (kw == 0) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (ACT == ACT_GLU && j >= 2) continue;
        float s2 = 0.f, s1 = 0.f;
#pragma unroll
        for (int i2 = 0; i2 < TM; ++i2)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float z = acc[i2][j][e];
            float h = (ACT == ACT_GLU) ? silu_f(z) * acc[i2][(j + 2) % TN][e] : gelu_f(z);
            h = m0 + i2 * 16 + 4 * quad + e < p.M ? h : 0.f;
            s2 += h * h;
            s1 += fabsf(h);
          }
        s2 += __shfl_xor(s2, 16); s2 += __shfl_xor(s2, 32);
        s1 += __shfl_xor(s1, 16); s1 += __shfl_xor(s1, 32);
        if (lane < 16) {
          const int c = wn * TN * 16 + j * 16;
          const int cl = ((ACT == ACT_GLU) ? (c >> 6) * 32 + (c & 31) : c) + lane;
          red2[wm * BNO + cl] = s2;
          red1[wm * BNO + cl] = s1;
        }
      }
    }
    __syncthreads();
    if (tid < BNO) {
      const int col = tn * BNO + tid;
      if (col < p.n_out) {
        float a2 = 0.f, a1 = 0.f;
#pragma unroll
        for (int w = 0; w < WGM; ++w) { a2 += red2[w * BNO + tid]; a1 += red1[w * BNO + tid]; }
        p.part_s2[(int64_t)tm * p.n_out + col] = a2;
        p.part_s1[(int64_t)tm * p.n_out + col] = a1;
      }
    }
  }
}

// ------------------------------------------------------------------ host launchers

template <int TM, int TN, int WGM, int WGN, int KW, int PF, int ACT, bool DUAL, bool SCORE, bool FIX = false>
static int launch_f32(const GemmArgs& a, hipStream_t st) {
  constexpr int BM = WGM * TM * 16, BN = WGN * TN * 16;
  constexpr size_t waves = WGM * WGN * KW;
  constexpr size_t lds = std::max(waves * ((DUAL ? 2 : 1) * TM + TN) * 1024,
                                  std::max(KW > 1 ? waves * TM * TN * 1024 : (size_t)0, (size_t)(SCORE ? WGM * BN * 8 : 0)));
  static_assert(lds <= 64 * 1024, "within the default limit of dynamic LDS");
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, WGM, WGN, KW, PF, ACT, DUAL, SCORE, FIX>), dim3(tiles, FIX ? a.fix_split : 1),
                     dim3(WGM * WGN * KW * 64), lds, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Tile by estimated clocks: ceil(W / 256) workgroups one after the other on the fullest CU, each
// bound by the matrix rate (256 flop per clock and CU) or by its loads (61 bytes per clock), plus
// about 3000 clocks of launch, first loads, sum and store.
struct F32Shape { int bm, bn, wgm, wgn; };
template <int N>
static int pick_f32(const F32Shape (&c)[N], int64_t M, int64_t Nn, int64_t K) {
  int best = 0;
  double best_t = 1e30;
  for (int i = 0; i < N; ++i) {
    const int64_t w = ((M + c[i].bm - 1) / c[i].bm) * ((Nn + c[i].bn - 1) / c[i].bn);
    const double mfma = (double)c[i].bm * c[i].bn * K / 128, ld = 4.0 * K * (c[i].bm * c[i].wgn + c[i].bn * c[i].wgm) / 61;
    const double t = (double)((w + 255) / 256) * (std::max(mfma, ld) + 3000.0);
    if (t < best_t) { best_t = t; best = i; }
  }
  return best;
}

template <int ACT, bool DUAL>
static int launch_f32_act(const GemmArgs& a, hipStream_t st) {
  if constexpr (ACT == ACT_GLU) {
    static const F32Shape c[] = {{64, 128, 2, 2}, {32, 64, 1, 1}, {16, 64, 1, 1}};
    switch (pick_f32(c, a.M, a.N, a.K)) {
      case 0: return launch_f32<2, 4, 2, 2, 1, 2, ACT, DUAL, false>(a, st);
      case 1: return launch_f32<2, 4, 1, 1, 8, 2, ACT, DUAL, false>(a, st);
      default: return launch_f32<1, 4, 1, 1, 8, 4, ACT, DUAL, false>(a, st);
    }
  } else {
    // (128 x 128 on four wavefronts was slower everywhere: one wavefront per SIMD shows every wait)
    static const F32Shape c[] = {{64, 64, 2, 2}, {32, 32, 1, 1}, {16, 32, 1, 1}, {16, 16, 1, 1}};
    const int pick = pick_f32(c, a.M, a.N, a.K);
    // A short reduction has no k groups to share, and a 64x64 tile leaves its erf to few wavefronts (128 x 2944 x 64:
    // 8.5 us, 4.7 on 32x32 tiles).  Not where the tiles fill the machine (512 x 3072 x 64: 36.4 and more).
    if (pick == 0 && a.K <= 128 && (a.M + 63) / 64 * ((a.N + 63) / 64) <= 256)
      return launch_f32<1, 1, 2, 2, 1, 4, ACT, DUAL, false>(a, st);
    if constexpr (ACT == ACT_NONE) {
      // few 16x16 tiles and a long reduction: ranges of at least 32 slabs on the idle CUs (a BERT-base-sized layer of
      // 128 tokens, 32 tiles: 23.5 -> 20.6 us; 1024 wide, 16 tokens 26.1 -> 21.2), where each of the 16 wavefronts is
      // spared four slabs (2048 x 256, 128 tokens 17.2 -> 17.0, 1536 x 256, 1 token 9.2 either way; two slabs, 1024 x 256, 1 and
      // 128 tokens: 8.6 -> 9.05 and 13.5 -> 14.0)
      const int tiles = (a.M + 15) / 16 * ((a.N + 15) / 16);
      const int s = std::min({F32_MAX_SPLIT, 256 / tiles, (a.K + 15) / 16 / 32});
      if (pick == 3 && a.fix_cnt != nullptr && (a.K + 15) / 16 * (s - 1) >= 64 * s) {
        GemmArgs g = a;
        g.fix_split = s;
        return launch_f32<1, 1, 1, 1, 16, 4, ACT, DUAL, false, true>(g, st);
      }
    }
    switch (pick) {
      case 0: return launch_f32<2, 2, 2, 2, 2, 4, ACT, DUAL, false>(a, st);
      case 1: return launch_f32<2, 2, 1, 1, 8, 4, ACT, DUAL, false>(a, st);
      case 2: return launch_f32<1, 2, 1, 1, 8, 4, ACT, DUAL, false>(a, st);
      default: return launch_f32<1, 1, 1, 1, 16, 4, ACT, DUAL, false>(a, st);
    }
  }
}

size_t gemm_f32_part_bytes() { return (size_t)256 * 1024; }   // 256 workgroups, one KiB each

int launch_gemm_f32(const GemmArgs& a, int act, bool score, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return 0;
  if ((a.K & 3) || (a.lda & 3) || (a.ldb & 3) || (a.split_col & 3)) return -1;
  const bool dual = a.A1 != nullptr;
  if (score) {
    if (act == ACT_GELU) return launch_f32<2, 4, 2, 2, 1, 2, ACT_GELU, false, true>(a, st);
    if (act == ACT_GLU) return launch_f32<2, 4, 2, 2, 1, 2, ACT_GLU, false, true>(a, st);
    return -1;
  }
  if (act == ACT_NONE) return launch_f32_act<ACT_NONE, false>(a, st);
  if (act == ACT_GELU) return launch_f32_act<ACT_GELU, false>(a, st);
  if (act == ACT_GLU && !dual) return launch_f32_act<ACT_GLU, false>(a, st);
  if (act == ACT_GLU && dual) return launch_f32_act<ACT_GLU, true>(a, st);
  return -1;
}

}  // namespace ffsplit
