// bf16 MFMA GEMM of the split feed-forward path, gfx950 only.
//
//   D[M, N] = A[M, K] * B[N, K]^T ,  fp32 accumulation, fused epilogue.
//
// Data layouts
//   "tiled": the matrix is cut into blocks of 32 rows x 16 k-elements (1 KiB).
//     Inside a block the 16-byte chunk of lane l = 32 c + r holds row r,
//     k-elements 8 c .. 8 c + 7.  Blocks are ordered [row block][k block], so a K slab of one
//     row block is contiguous.  All packed weights and all intermediates between the chained
//     products use this layout: a load or LDS read of a wavefront is a contiguous 1 KiB, and the
//     operand of v_mfma_f32_16x16x32_bf16 (row l & 15, k elements 8 (l >> 4) .. + 7 in lane l) is
//     four contiguous 256-byte pieces of two neighbouring blocks: free of bank conflicts.
//   "row-major": ordinary [rows, ld] (the caller's X and Y).
//
// Kernel: BM x BN workgroup tile; 32-deep slabs go from global memory straight into a ring of
// LDS stages (buffer loads with LDS destination, one 1 KiB operand block per wavefront
// instruction, addresses in scalar registers); each wavefront owns a (BM/WGM) x (BN/WGN) sub-tile
// of 16x16 MFMA tiles.  The MFMA is issued with the weights as the first operand so that a lane
// ends up with 4 consecutive output columns of one row; one v_permlane16_swap of two row tiles
// turns that into 8 consecutive columns = one 16-byte chunk of the tiled (or row-major) output.
//
// What bounds it, and why it looks like this (measured on random normal operands):
//   - Power.  A register-only loop of 32x32x16 MFMAs sustains 1.83 PFLOP/s (2.45 on zeros), of
//     16x16x32 ones 2.09: hence the 16x16 shape.  4096 x 8192 x 8192 in this kernel: 1.52 PFLOP/s
//     (1.96 on zeros); the 32x32 kernel it replaces ran the same chain of products at 1.2 at best.
//   - The vector cache hands a CU 61 bytes per clock, the matrix cores eat a 128x128 tile's slab
//     (16 KiB) in 256 clocks: small tiles are bound by loads, 256-wide ones are not.  LDS reads
//     (250 bytes per clock) are not the limit with wave tiles of 64x64 or more.
//   - Barriers.  Each step has one barrier, in its middle, where every read it must wait for was
//     issued hundreds of clocks earlier; a wait for reads just issued stalled all eight wavefronts
//     at the same point (the replaced kernel: 68 % MFMA busy at best).
//   - Instruction order is written out and fenced; left to the scheduler the reads bunch up.
// Epilogues: plain / GeLU / SwiGLU (on (gate, up) pairs of 32-column blocks)
// with two output destinations, fp32 split-K partials, and the neuron-norm
// column reduction of Sec. 4.1 (Eq. 3) for the calibration pass.
#include "common.h"
#include <atomic>
#include <algorithm>
#include <math.h>
#include <type_traits>

namespace ffsplit {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;  // native vector: stays in registers

union Frag {
  u32x4_t u;
  bf16x8_t v;
};

__device__ __forceinline__ int xcd_remap(int i, int total) {
  const int q = total >> 3, rem = total & 7, x = i & 7;
  return x * q + (x < rem ? x : rem) + (i >> 3);
}

template <int ACT>
__device__ __forceinline__ float act_bf16(float z, float g) {
  if (ACT == ACT_GELU) return gelu_fast(z);
  if (ACT == ACT_GLU) return silu_fast(g) * z;
  return z;
}

// swap the odd 16-lane rows of a with the even ones of b
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
  auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// The wavefront's accumulators: acc[i][j] is the 16x16 MFMA tile of token rows 16 i and GEMM
// columns 16 j of its sub-tile.  Forward (SCORE = false): weights are the first MFMA operand, so
// lane l holds row l & 15, columns 4 (l >> 4) + 0..3.  SCORE: lane l holds column l & 15, rows
// 4 (l >> 4) + 0..3.
//
// Epilogue: activation, bf16 packing and the stores (or the neuron-norm column sums).
// EPI: the optional additions of GemmArgs (bias, residual stream, fp32 destination) are compiled
// in; the plain instantiations carry none of their instructions.
template <int BM, int BN, int WGM, int WGN, int ACT, bool SCORE, bool EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& p, f32x4_t (&acc)[BM / WGM / 16][BN / WGN / 16], int m0,
                                              int n0, int tm, int wm, int wn, int lane, int tid, u32x4_t* smem) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 16, TN = WN / 16;
  const int quad = lane >> 4;
  if (!SCORE) {
    const int r0 = m0 + wm * WM;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int cb = n0 + wn * WN + j * 16;  // GEMM column of this tile
      if (cb >= p.N) continue;
      const bool act_here = cb < p.act_cols;
      int oc;       // output column of the tile
      if (ACT == ACT_GLU) {
        // (gate, up) pairs of 32-column blocks: the pair is written when its gate tile comes up
        if (act_here) {
          if (j & 2) continue;
          oc = (cb >> 6) * 32 + (cb & 31);
        } else {
          oc = cb - p.act_cols / 2;
        }
      } else {
        oc = cb;
      }
      char* base;
      int64_t ld;
      int occ, tiled;
      const bool to_c0 = oc < p.split_col;
      if (to_c0) { base = (char*)p.C0; ld = p.ldc0; occ = oc; tiled = p.c0_tiled; }
      else { base = (char*)p.C1; ld = p.ldc1; occ = oc - p.split_col; tiled = p.c1_tiled; }
      if (p.partial) {
        // fp32 split-K partial, row-major [split][M][ld]
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int row = r0 + i * 16 + (lane & 15);
          if (row < p.M)
            *(f32x4_t*)((float*)base + ((int64_t)blockIdx.y * p.M + row) * ld + occ + 4 * quad) = acc[i][j];
        }
        continue;
      }
      // a neuron's bias (the lane's GEMM columns cb + 4 quad + e), added before the activation
      float4 bz = make_float4(0.f, 0.f, 0.f, 0.f);
      if (EPI && ACT != ACT_GLU && p.bias != nullptr && cb + 4 * quad + 3 < p.bias_cols)
        bz = *(const float4*)(p.bias + cb + 4 * quad);
      const bool f32o = EPI && p.out_f32 && to_c0 && !tiled;
      const bool col4_ok = occ + 4 * quad < p.n_store;
#pragma unroll
      for (int ip = 0; ip < TM; ip += 2) {
        uint32_t pk[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int i = ip + h, row = r0 + i * 16 + (lane & 15);
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            // (static tile indices: an activated pair is (gate j, value j + 2))
            constexpr int TNM1 = TN - 1;
            const int j1 = j + 2 < TN ? j + 2 : TNM1;
            float gt = acc[i][j][e];
            if (EPI) gt += e == 0 ? bz.x : e == 1 ? bz.y : e == 2 ? bz.z : bz.w;
            const float z = (ACT == ACT_GLU && act_here) ? acc[i][j1][e] : gt;
            v[e] = act_here ? act_bf16<ACT>(z, gt) : z;
          }
          // the residual stream of an activated product (un-activated ones start from it: see the kernel)
          if (EPI && ACT != ACT_NONE && p.resid != nullptr && to_c0 && !tiled && row < p.M && col4_ok) {
            const float4 r4 = *(const float4*)(p.resid + (int64_t)row * p.ldr + occ + 4 * quad);
            v[0] += r4.x; v[1] += r4.y; v[2] += r4.z; v[3] += r4.w;
          }
          if (EPI && f32o) {
            if (row < p.M && col4_ok)
              *(float4*)((float*)base + (int64_t)row * ld + occ + 4 * quad) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
            pk[h][0] = pack_bf16x2(v[0], v[1]);
            pk[h][1] = pack_bf16x2(v[2], v[3]);
          }
        }
        if (EPI && f32o) continue;
        // Swapping the odd 16-lane rows of the first tile's registers with the even ones of the
        // second's leaves lane l with row (l & 31) of the 32-row block and columns 8 (l >> 5) + 0..7:
        // one 16-byte chunk of the tiled (or row-major) output.
        swap16(pk[0][0], pk[1][0]);
        swap16(pk[0][1], pk[1][1]);
        const u32x4_t val = {pk[0][0], pk[0][1], pk[1][0], pk[1][1]};
        const int rblk = r0 / 32 + ip / 2;
        const int row = rblk * 32 + (lane & 31);
        if (tiled) {
          if (rblk * 32 < p.m_pad)
            *(u32x4_t*)(base + (((int64_t)rblk * (ld / 16) + occ / 16) * 64 + lane) * 16) = val;
        } else {
          if (row < p.M && occ + 8 * (lane >> 5) < p.n_store)
            *(u32x4_t*)(base + ((int64_t)row * ld + occ + 8 * (lane >> 5)) * 2) = val;
        }
      }
    }
  } else {
    constexpr int BNO = (ACT == ACT_GLU) ? BN / 2 : BN;
    float* red2 = (float*)smem;  // [WGM][BNO]
    float* red1 = red2 + WGM * BNO;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (ACT == ACT_GLU && (j & 2)) continue;
      float s2 = 0.f, s1 = 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = m0 + wm * WM + i * 16 + 4 * quad + e;
          constexpr int TNM1 = TN - 1;
          const int j1 = j + 2 < TN ? j + 2 : TNM1;
          const float z = acc[i][(ACT == ACT_GLU) ? j1 : j][e];
          const float gt = acc[i][j][e];
          // same activation forms as the forward epilogue: the scores rank what the forward computes
          // (the erf form costs about a fifth of the calibration pass, nothing hides it at one
          // workgroup per CU)
          float h = act_bf16<ACT>(z, gt);
          h = row < p.M ? h : 0.f;
          s2 += h * h;
          s1 += fabsf(h);
        }
      s2 += __shfl_xor(s2, 16); s2 += __shfl_xor(s2, 32);
      s1 += __shfl_xor(s1, 16); s1 += __shfl_xor(s1, 32);
      if (lane < 16) {
        const int c = wn * WN + j * 16;
        const int cl = ((ACT == ACT_GLU) ? (c >> 6) * 32 + (c & 31) : c) + lane;
        red2[wm * BNO + cl] = s2;
        red1[wm * BNO + cl] = s1;
      }
    }
    __syncthreads();
    for (int t = tid; t < BNO; t += NT) {
      const int col = ((ACT == ACT_GLU) ? n0 / 2 : n0) + t;
      if (col < p.n_out) {
        float a2 = 0.f, a1 = 0.f;
#pragma unroll
        for (int w = 0; w < WGM; ++w) { a2 += red2[w * BNO + t]; a1 += red1[w * BNO + t]; }
        p.part_s2[(int64_t)tm * p.n_out + col] = a2;
        p.part_s1[(int64_t)tm * p.n_out + col] = a1;
      }
    }
  }
}

typedef __attribute__((address_space(3))) void* lptr_t;
// 16 bytes per lane from base + lane offset + scalar offset straight into LDS (1 KiB per
// wavefront instruction, lane l to dst + 16 l); the buffer resource spans the address space: the
// callers' offsets never leave the operands
__device__ __forceinline__ void buffer_to_lds(const void* base, lptr_t dst, uint32_t lane_off, uint32_t scalar_off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00027000), dst, 16,
                                           lane_off, scalar_off, 0, 0);
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in
// imm[3:0] and imm[15:14], expcnt imm[6:4], lgkmcnt imm[11:8])
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  __builtin_amdgcn_s_waitcnt(0xc07f | ((N < 15 ? N : 15) << 8));
}
// workgroup barrier without a memory fence (the kernel orders its loads with explicit counters);
// the memory clobber keeps the compiler from moving LDS accesses across it
__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }
#define FFS_ORDER __builtin_amdgcn_sched_barrier(0)   // instructions keep the written order

// The accumulators of a tile's ranges (blockIdx.y) added by the last workgroup to arrive, which gets them in
// acc and true; the others are done.  The XCDs' L2 caches are not coherent within a launch: device-scope
// stores and loads.  Every thread waits for its own stores before the barrier, and only behind it is the
// workgroup counted in, so that the last one finds every range in place.  All ranges come from memory, its own
// too, in one round trip, and are added in range order: the result does not depend on the order of arrival.
enum { MODE_PLAIN = 0, MODE_FIX = 1, MODE_WRAP = 2 };
constexpr int DEV_SCOPE = 16;   // sc1
template <int NT, int NR>
__device__ __forceinline__ bool last_range(const GemmArgs& p, f32x4_t* acc, int tile, int tid, int* flag) {
  const int n = p.fix_split;
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((char*)p.fix_part + (int64_t)tile * n * NR * NT * 16, 0,
                                                                     n * NR * NT * 16, 0x00027000);
#pragma unroll
  for (int i = 0; i < NR; ++i)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[i]), r, tid * 16, ((int)blockIdx.y * NR + i) * (NT * 16),
                                           DEV_SCOPE);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    const bool last = __hip_atomic_fetch_add(p.fix_cnt + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(n - 1);
    if (last) __hip_atomic_store(p.fix_cnt + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = last;
  }
  __syncthreads();
  if (!*flag) return false;
  u32x4_t v[GEMM_FIX_MAX_SPLIT][NR];
#pragma unroll
  for (int s = 0; s < GEMM_FIX_MAX_SPLIT; ++s)
#pragma unroll
    for (int i = 0; i < NR; ++i)
      v[s][i] = __builtin_amdgcn_raw_buffer_load_b128(r, tid * 16, ((s < n ? s : n - 1) * NR + i) * (NT * 16), DEV_SCOPE);
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    acc[i] = __builtin_bit_cast(f32x4_t, v[0][i]);
#pragma unroll
    for (int s = 1; s < GEMM_FIX_MAX_SPLIT; ++s)
      if (s < n) acc[i] += __builtin_bit_cast(f32x4_t, v[s][i]);
  }
  return true;
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool DBLA, int ACT, bool DUAL, bool SCORE, bool A_TILED,
          bool EPI, int MODE>
__global__ void __launch_bounds__(WGM* WGN * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
gemm_bf16_dl_kernel(const GemmArgs p) {
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 16, TN = WN / 16;    // 16x16 MFMA tiles of a wavefront
  constexpr int NA = DUAL ? 2 : 1;
  constexpr int A_BLK = NA * (BM / 16);        // 1 KiB operand blocks of one 32-deep slab
  constexpr int B_BLK = BN / 16;
  // loads per wavefront and slab; where the weights' blocks do not divide over the wavefronts the
  // last round is padded with repeats of the tile's last block, which land in spare slots that
  // nothing reads (every wavefront then issues the same number of loads, which the wait counts
  // below rely on)
  constexpr int LA = A_BLK / NW, LB = (B_BLK + NW - 1) / NW, LPW = LA + LB;
  constexpr int STAGE = (A_BLK + LB * NW) * 64;  // 16-byte chunks per stage
  static_assert(A_BLK % NW == 0, "the tokens' blocks must divide over the wavefronts");
  static_assert(STAGES >= 3 && STAGES * LPW <= 63, "loads in flight must fit the counter");
  static_assert(ACT != ACT_GLU || WN % 64 == 0, "(gate, up) pairs must lie inside one wavefront");
  static_assert(TM % 2 == 0 && (!DUAL || A_TILED), "row tiles are stored in pairs; two left operands are tiled");

  constexpr bool FIX = MODE == MODE_FIX, WRAP = MODE == MODE_WRAP;   // GemmArgs::fix_split, a_wrap
  static_assert(MODE == MODE_PLAIN || (ACT == ACT_NONE && A_TILED && !DUAL && !SCORE), "");

  extern __shared__ u32x4_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  if (!A_TILED && blockIdx.x == 0)
    for (int i = tid; i < p.n_clear; i += NW * 64) p.clear[i] = 0u;
  const int tiles_n = (p.N + BN - 1) / BN;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int logical = xcd_remap(blockIdx.x, tiles_m * tiles_n);
  const int gsz = p.group_m * tiles_n;
  const int first_m = (logical / gsz) * p.group_m;
  const int gm = min(tiles_m - first_m, p.group_m);
  const int tm = first_m + (logical % gsz) % gm, tn = (logical % gsz) / gm;
  const int m0 = tm * BM, n0 = tn * BN;

  // K range of this split (whole slabs)
  const int kt_total = (p.K + 31) / 32;
  const int kt_per = (kt_total + (int)gridDim.y - 1) / (int)gridDim.y;
  const int kt0 = blockIdx.y * kt_per;
  const int nk = min(kt_total, kt0 + kt_per) - kt0;

  // ---- the LPW blocks this wavefront moves per slab: block b = wave + i NW of the stage
  // Tiled operands: the block's address is uniform, the lane adds 16 bytes times its number.
  // Row-major A: one load instruction covers 16 rows x the slab's four 16-byte chunks; chunk c of
  // row r goes to position 4 r + (c ^ (r >> 2)), so that the fragment reads (16 rows, one chunk
  // number) of 16 consecutive lanes fall into 16 different 16-byte bank groups.  (The counters
  // still show conflicts on this form alone: 6.9e6 cycles over the machine at 4096 x 3200 x 4096, a sixth
  // of the kernel's; tiled operands have none.  So the lanes of a pass are probably not consecutive ones.)
  // All loads are buffer loads: the tile's base in scalar registers, a byte offset per lane that the
  // loop never changes, and a scalar offset that walks along K.
  uint32_t soff[LPW];       // uniform: the block's offset inside the tile
  uint32_t a_row[LA];       // row-major A: offset of the lane's row from row m0
  const uint32_t a_col = ((lane & 3) ^ ((lane >> 4) & 3)) * 8;   // row-major A: the lane's chunk (column in the slab)
  const int mrb_last = (p.M + 31) / 32 - 1, nrb_last = (p.N + 31) / 32 - 1;
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int b = wave + i * NW;
    soff[i] = 0; a_row[i] = 0;
    if (A_TILED) {
      const int rb = min(m0 / 32 + (b / 2) % (BM / 32), mrb_last) - m0 / 32;
      soff[i] = ((uint32_t)rb * (uint32_t)(p.lda / 16) + (b & 1)) * 1024;
    } else {
      a_row[i] = (uint32_t)(min(m0 + b * 16 + (lane >> 2), p.M - 1) - m0) * (uint32_t)(p.lda * 2);
    }
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int b = min(wave + i * NW, B_BLK - 1);
    const int rb = min(n0 / 32 + b / 2, nrb_last) - n0 / 32;
    soff[LA + i] = ((uint32_t)rb * (uint32_t)(p.ldb / 16) + (b & 1)) * 1024;
  }
  const uint32_t lane16 = lane * 16;
  const int wrap = WRAP ? p.a_wrap / 32 : 0;   // slabs
  auto tile_base = [&](const void* a) {
    return A_TILED ? (const char*)a + ((int64_t)(m0 / 32) * (p.lda / 16) + 2 * kt0) * 1024
                   : (const char*)a + (int64_t)m0 * p.lda * 2;
  };
  const char* const base_a = tile_base(p.A);
  const char* const base_a1 = tile_base(DUAL ? p.A1 : p.A);
  const char* const base_b = (const char*)p.Bt + ((int64_t)(n0 / 32) * (p.ldb / 16) + 2 * kt0) * 1024;

  // load number i of slab rel into a stage; check: the slab may reach past K (row-major A)
  auto issue = [&](int i, int rel, int stage, bool check) {
    const int slot = i < LA ? wave + i * NW : A_BLK + wave + (i - LA) * NW;
    const lptr_t dst = (lptr_t)(smem + stage * STAGE + slot * 64);
    if (i >= LA) {
      buffer_to_lds(base_b, dst, lane16, soff[i] + rel * 2048);
    } else if (A_TILED) {
      // (with two left operands the first BM / 16 blocks are A's, the others A1's: uniform per i)
      static_assert(!DUAL || (BM / 16) % NW == 0, "a load belongs to one left operand");
      int ra = rel;
      if (WRAP) ra -= rel >= 2 * wrap ? 2 * wrap : rel >= wrap ? wrap : 0;   // (the whole reduction: kt0 = 0)
      buffer_to_lds((DUAL && i >= LA / 2) ? base_a1 : base_a, dst, lane16, soff[i] + ra * 2048);
    } else if (!check) {
      buffer_to_lds(base_a, dst, a_row[i] + a_col * 2, (kt0 + rel) * 64);
    } else {
      // a chunk past K reads the start of the row instead: the weights are zero there
      const uint32_t col = (kt0 + rel) * 32 + a_col;
      buffer_to_lds(base_a, dst, a_row[i] + (col < (uint32_t)p.K ? col * 2 : 0), 0);
    }
  };

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // Residual stream of an un-activated product: the accumulators start from it (same lane
  // layout as the store epilogue), so its loads overlap the filling of the ring instead of forming
  // one dependent round trip per tile between the last product and the stores.  This workgroup
  // alone reads and later writes these elements, so the destination may be the residual buffer.
  if (EPI && ACT == ACT_NONE && !SCORE) {
    if (p.resid != nullptr && !p.partial && !p.c0_tiled && (!FIX || blockIdx.y == 0)) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int cb = n0 + wn * WN + j * 16;
        if (cb >= p.N || cb >= p.split_col) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int row = m0 + wm * WM + i * 16 + (lane & 15);
          if (row < p.M && cb + 4 * (lane >> 4) < p.n_store)
            acc[i][j] = *(const f32x4_t*)(p.resid + (int64_t)row * p.ldr + cb + 4 * (lane >> 4));
        }
      }
    }
  }

  // Fragments: lane l of a 16-row tile holds row l & 15, k elements 8 (l >> 4) .. + 7 of the slab.
  // Tiled operands: two 32x16 blocks per 32 rows, the tile's half of each.
  Frag fa[DBLA ? 2 : 1][NA][TM], fb[2][TN];
  const int tfrag = (lane >> 5) * 64 + ((lane >> 4) & 1) * 32 + (lane & 15);
  const int rfrag = (lane & 15) * 4 + ((lane >> 4) ^ ((lane >> 2) & 3));
  auto tile_off = [](int x) { return (x >> 1) * 128 + (x & 1) * 16; };   // tiled operand: 16-row tile x
  const int a_off = A_TILED ? tfrag + wm * (TM / 2) * 128 : rfrag + wm * TM * 64;
  const int b_off0 = A_BLK * 64 + tfrag + tile_off(wn * TN), b_off1 = A_BLK * 64 + tfrag + tile_off(wn * TN + 1);
  auto read_a = [&](int set, int i, const u32x4_t* st) {
#pragma unroll
    for (int s = 0; s < NA; ++s)
      fa[DBLA ? set : 0][s][i].u = A_TILED ? st[a_off + s * (BM / 16) * 64 + tile_off(i)] : st[a_off + i * 64];
  };
  auto read_b = [&](int set, int j, const u32x4_t* st) {
    fb[set][j].u = st[((j & 1) ? b_off1 : b_off0) + (j >> 1) * 128];
  };
  auto mma = [&](int set, int i, int j) {
    const Frag& a = fa[DBLA ? set : 0][DUAL ? (j >> 1) & 1 : 0][i];
    const Frag& b = fb[set][j];
    if (SCORE) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, acc[i][j], 0, 0, 0);
    else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.v, a.v, acc[i][j], 0, 0, 0);
  };
  // at most `later` slabs of loads may still be in flight
  auto wait_slabs = [&](int later) {
    if (later <= 0) wait_vmcnt<0>();
    else if (later == 1) wait_vmcnt<LPW>();
    else if (later == 2) wait_vmcnt<2 * LPW>();
    else wait_vmcnt<3 * LPW>();
  };
  static_assert(STAGES <= 5, "wait_slabs covers three slabs in flight");

  // Step s multiplies slab s from registers, reads the fragments of slab s + 1 and has one barrier,
  // placed where the reads it depends on were issued long before (waiting for reads that were only
  // just issued stalls every wavefront of the workgroup at the same point).
  //   DBLA: all reads of slab s + 1 are dealt out over the first five eighths of the MFMAs; the
  //     barrier after three quarters retires slab s + 1 (it is in registers now) and publishes
  //     slab s + 2; slab s + 1 + STAGES goes out behind it.
  //   otherwise: fragment row i of the left operand is overwritten as soon as its MFMAs are issued,
  //     so the reads of slab s + 1 end with the step; the barrier in the middle retires slab s and
  //     publishes slab s + 2; slab s + STAGES goes out behind it.
  constexpr int AHEAD = DBLA ? 1 : 0;
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < nk) {
#pragma unroll
      for (int i = 0; i < LPW; ++i) issue(i, s, s, true);
    }
  int stage = 0;   // stage of slab s
  if (nk > 0) {
    wait_slabs(min(nk, STAGES) - 2);   // slabs 0 and 1
    lds_barrier();
#pragma unroll
    for (int j = 0; j < TN; ++j) read_b(0, j, smem);
#pragma unroll
    for (int i = 0; i < TM; ++i) read_a(0, i, smem);
    if (DBLA) {
      wait_lgkmcnt<0>();
      lds_barrier();
      if (STAGES < nk) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) issue(i, STAGES, 0, true);
      }
    }
  }
  auto step = [&](int s, auto setc, auto fullc) {
    constexpr int set = decltype(setc)::value;
    constexpr bool FULL = decltype(fullc)::value;   // every slab referred to exists, none reaches past K
    const int ns = stage + 1 == STAGES ? 0 : stage + 1;
    const u32x4_t* nx = smem + ns * STAGE;          // (past the end: stale data that is never used)
    const int put = s + AHEAD + STAGES;             // the slab whose loads go out in this step
    auto sync = [&](auto younger) {
      if (FULL) wait_vmcnt<(STAGES - 3 + AHEAD) * LPW>();
      else wait_slabs(min(nk - 1, put - 1) - (s + 2));
      wait_lgkmcnt<decltype(younger)::value>();
      lds_barrier();
      FFS_ORDER;
    };
    FFS_ORDER;
    if constexpr (DBLA) {
      constexpr int NM = TM * TN, NR = TM + TN, RD = NM * 5 / 8, SB = NM * 3 / 4;
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int i = q / TN, j = (i & 1) ? TN - 1 - q % TN : q % TN;
        mma(set, i, j);
        FFS_ORDER;
#pragma unroll
        for (int r = 0; r < NR; ++r)
          if (r * RD / NR == q) {
            if (r < TN) read_b(set ^ 1, r, nx);
            else read_a(set ^ 1, r - TN, nx);
          }
        FFS_ORDER;
        if (q == SB - 1) sync(std::integral_constant<int, 0>{});
#pragma unroll
        for (int l = 0; l < LPW; ++l)
          if (SB + l * (NM - SB) / LPW == q && (FULL || put < nk)) issue(l, put, ns, !FULL);
        FFS_ORDER;
      }
    } else {
      constexpr int RB = TM / 2 - 1;   // the barrier follows this row
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int jj = 0; jj < TN; ++jj) {
          mma(set, i, (i & 1) ? TN - 1 - jj : jj);
          FFS_ORDER;
          // the row's share of the next slab's weight fragments, spread over its MFMAs
#pragma unroll
          for (int q = 0; q < TN; ++q)
            if (q * TM == i * TN + jj) read_b(set ^ 1, q, nx);
          FFS_ORDER;
        }
        read_a(0, i, nx);
        FFS_ORDER;
        if (i == RB) sync(std::integral_constant<int, NA*(RB + 1) + ((RB + 1) * TN + TM - 1) / TM>{});
        if (i > RB) {
#pragma unroll
          for (int l = 0; l < LPW; ++l)
            if (l * (TM - RB - 1) / LPW == i - RB - 1 && (FULL || put < nk)) issue(l, put, stage, !FULL);
          FFS_ORDER;
        }
      }
    }
    stage = ns;
  };
  int s = 0;
  for (; s + 2 + AHEAD + STAGES < nk; s += 2) {
    step(s, std::integral_constant<int, 0>{}, std::true_type{});
    step(s + 1, std::integral_constant<int, 1>{}, std::true_type{});
  }
  for (; s < nk; s += 2) {
    step(s, std::integral_constant<int, 0>{}, std::false_type{});
    if (s + 1 < nk) step(s + 1, std::integral_constant<int, 1>{}, std::false_type{});
  }
  if (SCORE) {
    wait_lgkmcnt<0>();
    lds_barrier();   // the epilogue reuses the stage memory
  }
  if constexpr (FIX) {
    if (!last_range<NW * 64, TM * TN>(p, &acc[0][0], logical, tid, (int*)smem)) return;
  }
  gemm_epilogue<BM, BN, WGM, WGN, ACT, SCORE, EPI>(p, acc, m0, n0, tm, wm, wn, lane, tid, smem);
}

// Sum of fp32 split-K partials [n_split][M][ldp] of a whole product (GEMM column order) followed
// by the store epilogue of the large-batch kernel: activation (GeLU, or SwiGLU on (gate, up)
// pairs of 32-column blocks), routing to two destinations, bf16, tiled or row-major.  Used for
// products with few tiles at a few hundred rows, which are split along the reduction to fill
// the machine.  One thread per (row, 8 output columns).
struct SplitEpiArgs {
  const float* part;
  int n_split, M, ldp, n_out, rows;   // rows: rows to write (padded to 32 for tiled destinations)
  int act, act_cols, split_col;
  void* C0;
  void* C1;
  int64_t ldc0, ldc1;
  int c0_tiled, c1_tiled, n_store;
  const float* bias;   // as in GemmArgs
  int bias_cols;
  const float* resid;
  int64_t ldr;
  int out_f32;
  unsigned* clear;
  int n_clear;
};

__global__ void __launch_bounds__(256) splitk_epilogue_kernel(const SplitEpiArgs p) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < p.n_clear; i += 256) p.clear[i] = 0u;
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int cpr = p.n_out / 8;
  if (id >= (int64_t)p.rows * cpr) return;
  const int row = (int)(id / cpr), oc = (int)(id % cpr) * 8;
  const bool glu = p.act == ACT_GLU;
  const bool pair = glu && oc < p.act_cols / 2;
  int c = oc;                                   // GEMM column of the (gate) values
  if (glu) c = pair ? (oc / 32) * 64 + (oc & 31) : oc + p.act_cols / 2;
  float v[8] = {0, 0, 0, 0, 0, 0, 0, 0}, u[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (row < p.M) {
    for (int s = 0; s < p.n_split; ++s) {
      const float* src = p.part + ((int64_t)s * p.M + row) * p.ldp + c;
      const float4 a = *(const float4*)src, b = *(const float4*)(src + 4);
      v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w; v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
      if (pair) {
        const float4 e = *(const float4*)(src + 32), f = *(const float4*)(src + 36);
        u[0] += e.x; u[1] += e.y; u[2] += e.z; u[3] += e.w; u[4] += f.x; u[5] += f.y; u[6] += f.z; u[7] += f.w;
      }
    }
    if (!glu && p.bias != nullptr && c + 7 < p.bias_cols) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += p.bias[c + e];
    }
    if (pair) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = silu_fast(v[e]) * u[e];
    } else if (p.act == ACT_GELU && c < p.act_cols) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = gelu_fast(v[e]);
    }
  }
  char* base;
  int64_t ld;
  int col, tiled;
  const bool to_c0 = oc < p.split_col;
  if (to_c0) { base = (char*)p.C0; ld = p.ldc0; col = oc; tiled = p.c0_tiled; }
  else { base = (char*)p.C1; ld = p.ldc1; col = oc - p.split_col; tiled = p.c1_tiled; }
  if (to_c0 && !tiled && row < p.M && col < p.n_store) {
    if (p.resid != nullptr) {
      const float* r = p.resid + (int64_t)row * p.ldr + col;
      const float4 a = *(const float4*)r, b = *(const float4*)(r + 4);
      v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w; v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
    }
    if (p.out_f32) {
      float* dst = (float*)base + (int64_t)row * ld + col;
      *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
      *(float4*)(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
      return;
    }
  }
  const uint4 val = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                               pack_bf16x2(v[6], v[7]));
  if (tiled) {
    const int64_t blk = (int64_t)(row / 32) * (ld / 16) + col / 16;
    *(uint4*)(base + ((blk * 64) + ((col >> 3) & 1) * 32 + (row & 31)) * 16) = val;
  } else if (row < p.M && col < p.n_store) {
    *(uint4*)(base + ((int64_t)row * ld + col) * 2) = val;
  }
}

int launch_splitk_epilogue(const float* part, int n_split, int ldp, const GemmArgs& g, int act, hipStream_t st) {
  SplitEpiArgs a = {};
  a.part = part; a.n_split = n_split; a.M = g.M; a.ldp = ldp;
  a.n_out = act == ACT_GLU ? g.N - g.act_cols / 2 : g.N;
  a.rows = (g.c0_tiled || g.c1_tiled) ? (g.M + 31) / 32 * 32 : g.M;
  a.act = act; a.act_cols = g.act_cols; a.split_col = g.split_col;
  a.C0 = g.C0; a.C1 = g.C1; a.ldc0 = g.ldc0; a.ldc1 = g.ldc1;
  a.c0_tiled = g.c0_tiled; a.c1_tiled = g.c1_tiled; a.n_store = g.n_store;
  a.bias = g.bias; a.bias_cols = g.bias_cols; a.resid = g.resid; a.ldr = g.ldr; a.out_f32 = g.out_f32;
  a.clear = g.clear; a.n_clear = g.n_clear;
  if ((a.n_out & 7) || (g.split_col & 7) || (g.act_cols & 63)) return -1;
  const int64_t n = (int64_t)a.rows * (a.n_out / 8);
  if (n <= 0) return 0;
  hipLaunchKernelGGL(splitk_epilogue_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ------------------------------------------------------------------ host launcher

template <int BM, int BN, int WGM, int WGN, int STAGES, bool DBLA, int ACT, bool DUAL, bool SCORE, bool A_TILED,
          bool EPI, int MODE>
static int launch_dl_epi(const GemmArgs& a, int n_split, hipStream_t st) {
  constexpr int NWH = WGM * WGN;
  constexpr size_t lds = (size_t)STAGES * 1024 * ((DUAL ? 2 : 1) * (BM / 16) + (BN / 16 + NWH - 1) / NWH * NWH);
  static_assert(lds <= 160 * 1024, "LDS budget of a CU");
  auto kern = gemm_bf16_dl_kernel<BM, BN, WGM, WGN, STAGES, DBLA, ACT, DUAL, SCORE, A_TILED, EPI, MODE>;
  // The kernel needs more dynamic LDS than the default limit: the attribute is set once per
  // device and instantiation.  The only state kept is this set-once bit mask (one bit per
  // device ordinal); setting the attribute twice from racing first calls is harmless.
  static std::atomic<uint64_t> configured{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -1;
  const uint64_t bit = 1ull << (dev & 63);
  if (dev >= 64 || !(configured.load(std::memory_order_acquire) & bit)) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return -1;
    if (dev < 64) configured.fetch_or(bit, std::memory_order_release);
  }
  const int tiles_m = (a.M + BM - 1) / BM, tiles = tiles_m * ((a.N + BN - 1) / BN);
  // Tiles are numbered down groups of group_m row tiles, consecutive ones on one XCD.  The R tiles
  // that an XCD runs at a time then read group_m BM + (R / group_m) BN rows per slab into its L2:
  // least at group_m = sqrt(R BN / BM).  (With group_m = 1 a product of 1000 tokens with a 22144-wide
  // weight pulled all weights into every XCD: 225 us instead of 164.)
  GemmArgs g = a;
  if (g.group_m <= 0) {
    const int per_cu = lds <= 80 * 1024 ? 2 : 1;
    const int r = std::max(1, std::min(32 * per_cu, tiles / 8));
    g.group_m = std::max(1, std::min(tiles_m, (int)(sqrt((double)r * BN / BM) + 0.5)));
  }
  hipLaunchKernelGGL(kern, dim3(tiles, n_split), dim3(NWH * 64), lds, st, g);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool DBLA, int ACT, bool DUAL, bool SCORE, bool A_TILED>
static int launch_dl_cfg(const GemmArgs& a, int n_split, hipStream_t st) {
  // (the calibration product, the gated products and the two-operand product take no additions)
  const bool adds = a.bias != nullptr || a.resid != nullptr || a.out_f32;
  if constexpr (ACT == ACT_NONE && A_TILED && !DUAL && !SCORE && BM == 64 && BN == 64) {
    if (a.fix_split > 1) {
      if (a.partial || a.fix_split != n_split || a.fix_split > GEMM_FIX_MAX_SPLIT) return -1;
      if ((int64_t)((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN) > FIX_COUNTERS) return -1;   // (a counter a tile)
      return adds ? launch_dl_epi<BM, BN, WGM, WGN, STAGES, DBLA, ACT, DUAL, SCORE, A_TILED, true, MODE_FIX>(a, n_split, st)
                  : launch_dl_epi<BM, BN, WGM, WGN, STAGES, DBLA, ACT, DUAL, SCORE, A_TILED, false, MODE_FIX>(a, n_split, st);
    }
  }
  if (a.fix_split > 1) return -1;
  if constexpr (ACT == ACT_NONE && A_TILED && !DUAL && !SCORE) {
    if (a.a_wrap > 0) {
      if (n_split != 1 || (a.a_wrap & 31) || a.K > 3 * a.a_wrap) return -1;
      return launch_dl_epi<BM, BN, WGM, WGN, STAGES, DBLA, ACT, DUAL, SCORE, A_TILED, true, MODE_WRAP>(a, 1, st);
    }
  }
  if (a.a_wrap > 0) return -1;
  if constexpr (!SCORE && !DUAL && ACT != ACT_GLU) {
    if (adds) return launch_dl_epi<BM, BN, WGM, WGN, STAGES, DBLA, ACT, DUAL, SCORE, A_TILED, true, MODE_PLAIN>(a, n_split, st);
  } else {
    if (adds) return -1;
  }
  return launch_dl_epi<BM, BN, WGM, WGN, STAGES, DBLA, ACT, DUAL, SCORE, A_TILED, false, MODE_PLAIN>(a, n_split, st);
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool DBLA>
static int launch_dl_shape(const GemmArgs& a, int act, int n_split, hipStream_t st) {
  const bool dual = a.A1 != nullptr;
  const bool at = a.a_tiled != 0;
  if (dual) return -1;
  if (act == ACT_NONE)
    return at ? launch_dl_cfg<BM, BN, WGM, WGN, STAGES, DBLA, ACT_NONE, false, false, true>(a, n_split, st)
              : launch_dl_cfg<BM, BN, WGM, WGN, STAGES, DBLA, ACT_NONE, false, false, false>(a, n_split, st);
  if (act == ACT_GELU)
    return at ? launch_dl_cfg<BM, BN, WGM, WGN, STAGES, DBLA, ACT_GELU, false, false, true>(a, 1, st)
              : launch_dl_cfg<BM, BN, WGM, WGN, STAGES, DBLA, ACT_GELU, false, false, false>(a, 1, st);
  // (a gated product reads the caller's row-major tokens; the tiled one has two left operands)
  if constexpr ((BN / WGN) % 64 == 0) {
    if (act == ACT_GLU && !at) return launch_dl_cfg<BM, BN, WGM, WGN, STAGES, DBLA, ACT_GLU, false, false, false>(a, 1, st);
  }
  return -1;
}

// the gated product with two left operands (A1)
template <int BM, int BN, int WGM, int WGN, int STAGES, bool DBLA>
static int launch_dl_dual(const GemmArgs& a, int act, hipStream_t st) {
  if (act != ACT_GLU || !a.a_tiled) return -1;
  return launch_dl_cfg<BM, BN, WGM, WGN, STAGES, DBLA, ACT_GLU, true, false, true>(a, 1, st);
}

int bf16_score_tile_m() { return 256; }

int launch_gemm_bf16(const GemmArgs& a, int act, bool score, int shape, int n_split, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return 0;
  if (score) {
    // calibration: row-major tokens, column sums of the activations in the epilogue
    if (a.a_tiled) return -1;
    if (act == ACT_GELU) return launch_dl_cfg<256, 256, 2, 4, 4, false, ACT_GELU, false, true, false>(a, 1, st);
    if (act == ACT_GLU) return launch_dl_cfg<256, 256, 2, 4, 4, false, ACT_GLU, false, true, false>(a, 1, st);
    return -1;
  }
  if (a.A1 != nullptr) {
    switch (shape) {
      case GEMM_128x128: return launch_dl_dual<128, 128, 2, 2, 3, true>(a, act, st);
      case GEMM_256x256: return act == ACT_GLU ? launch_gemm_dual(a, st) : -1;
    }
    return -1;
  }
  switch (shape) {
    case GEMM_128x128: return launch_dl_shape<128, 128, 2, 2, 4, true>(a, act, n_split, st);
    case GEMM_128x256: return launch_dl_shape<128, 256, 1, 4, 3, true>(a, act, n_split, st);
    case GEMM_128x320: return launch_dl_shape<128, 320, 2, 4, 4, true>(a, act, n_split, st);
    case GEMM_256x256: return launch_dl_shape<256, 256, 2, 4, 4, false>(a, act, n_split, st);
    case GEMM_256x320: return launch_dl_shape<256, 320, 2, 4, 4, false>(a, act, n_split, st);
    case GEMM_64x64: return launch_dl_shape<64, 64, 2, 2, 5, true>(a, act, n_split, st);
    case GEMM_64x128: return launch_dl_shape<64, 128, 2, 2, 5, true>(a, act, n_split, st);
  }
  return -1;
}

}  // namespace ffsplit
