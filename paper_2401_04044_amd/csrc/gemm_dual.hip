// Gated product with two left operands, 256 x 256 tiles, gfx950 only:
//   D[M, N/2] = silu(A[M, K] Bg[N/2, K]^T) * (A1[M, K] Bu[N/2, K]^T)
// where the weights hold Bg and Bu in alternating 32-row blocks.  All operands and the result are in
// the tiled layout of gemm_bf16.hip.  This is the remainder's expanding product of a gated low-rank
// layer; smaller grids take the 128 x 128 tiles of gemm_bf16.hip (gemm_plan.h).
//
// Eight wavefronts as 4 x 2, wave tiles of 64 x 128 (each token fragment meets two gate or two up
// blocks), v_mfma_f32_32x32x16_bf16, slabs of 32 straight from global memory into a ring of three LDS
// stages (144 KiB: a fourth does not fit beside two left operands).  Fragments are read one 16-deep
// step ahead; a slab's barrier follows the reads of its last step, and the loads that refill its stage
// are dealt out over the two steps after it.
// With three stages a slab is awaited one step of the ring after its loads went out.  The 16x16x32 form
// of gemm_bf16.hip issues them behind a barrier in the middle of a step, which leaves half of one to
// arrive in: whole layers with it take 4 to 9 % longer (us, that -> this): Llama-2-7B-sized, rank 1024:
// 1280 tokens 186 -> 173, 2048 266 -> 249, 4096 449 -> 425; rank 256, 6000 tokens 314 -> 288;
// 5120 x 13824, rank 1280, 4096 tokens 625 -> 601.  Issuing all its loads right behind that barrier
// was slower still.
#include "common.h"
#include <atomic>
#include <type_traits>

namespace ffsplit {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

union DFrag {
  u32x4_t u;
  bf16x8_t v;
};

constexpr int DBM = 256, DBN = 256, DWGM = 4, DWGN = 2, DSTAGES = 3;
constexpr int DTM = DBM / DWGM / 32, DTN = DBN / DWGN / 32;   // 32x32 tiles of a wavefront
constexpr int DNW = DWGM * DWGN;
constexpr int DA_BLK = 2 * (DBM / 32) * 2, DB_BLK = (DBN / 32) * 2;   // 1 KiB blocks of a slab
constexpr int DLA = DA_BLK / DNW, DLPW = DLA + DB_BLK / DNW;          // loads per wavefront and slab
constexpr int DSTAGE = (DA_BLK + DB_BLK) * 64;                        // 16-byte chunks of a stage
static_assert(DA_BLK % DNW == 0 && DB_BLK % DNW == 0 && DSTAGES * DLPW <= 63, "loads of a slab");

template <int N>
__device__ __forceinline__ void dual_wait_vmcnt() {   // gfx9 encoding, as in gemm_bf16.hip
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}
__device__ __forceinline__ void dual_swap32(uint32_t& a, uint32_t& b) {
  auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

__global__ void __launch_bounds__(DNW * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
gemm_dual_kernel(const GemmArgs p) {
  extern __shared__ u32x4_t dual_smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / DWGN, wn = wave % DWGN;
  const int tiles_n = (p.N + DBN - 1) / DBN, tiles_m = (p.M + DBM - 1) / DBM, tiles = tiles_m * tiles_n;
  // consecutive tiles on one XCD, down groups of group_m row tiles
  const int q8 = tiles >> 3, rem8 = tiles & 7, x = blockIdx.x & 7;
  const int logical = x * q8 + (x < rem8 ? x : rem8) + (int)(blockIdx.x >> 3);
  const int gsz = p.group_m * tiles_n;
  const int first_m = (logical / gsz) * p.group_m;
  const int gm = min(tiles_m - first_m, p.group_m);
  const int m0 = (first_m + (logical % gsz) % gm) * DBM, n0 = (logical % gsz) / gm * DBN;
  const int nk = (p.K + 31) / 32;

  // the blocks this wavefront moves per slab: number wave + i DNW of (A, A1, weights); row blocks past
  // the end repeat the last one
  const char* src[DLPW];
  const int mrb_last = (p.M + 31) / 32 - 1, nrb_last = (p.N + 31) / 32 - 1;
#pragma unroll
  for (int i = 0; i < DLPW; ++i) {
    const int b = wave + (i < DLA ? i : i - DLA) * DNW, kb = b & 1;
    const bool w = i >= DLA;
    const char* base = (const char*)(w ? p.Bt : b >= DA_BLK / 2 ? p.A1 : p.A);
    const int rb = w ? min(n0 / 32 + b / 2, nrb_last) : min(m0 / 32 + (b / 2) % (DBM / 32), mrb_last);
    src[i] = base + (((int64_t)rb * ((w ? p.ldb : p.lda) / 16) + kb) * 64 + lane) * 16;
  }
  // half q (of two) of the loads of slab s
  auto issue = [&](int s, int stage, int q) {
#pragma unroll
    for (int i = 0; i < DLPW; ++i) {
      if (i * 2 / DLPW != q) continue;
      const int slot = i < DLA ? wave + i * DNW : DA_BLK + wave + (i - DLA) * DNW;
      __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + (int64_t)s * 2048), (lptr_t)(dual_smem + stage * DSTAGE + slot * 64),
                                       16, 0, 0);
    }
  };

  f32x16_t acc[DTM][DTN];
#pragma unroll
  for (int i = 0; i < DTM; ++i)
#pragma unroll
    for (int j = 0; j < DTN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  DFrag fa[2][2][DTM], fb[2][DTN];
  auto read_frags = [&](int set, int stage, int ks) {
    const u32x4_t* sA = dual_smem + stage * DSTAGE;
    const u32x4_t* sB = sA + DA_BLK * 64;
#pragma unroll
    for (int i = 0; i < DTM; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) fa[set][s][i].u = sA[((s * (DBM / 32) + wm * DTM + i) * 2 + ks) * 64 + lane];
#pragma unroll
    for (int j = 0; j < DTN; ++j) fb[set][j].u = sB[((wn * DTN + j) * 2 + ks) * 64 + lane];
  };
  auto mfma_step = [&](int set) {
#pragma unroll
    for (int i = 0; i < DTM; ++i)
#pragma unroll
      for (int j = 0; j < DTN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j].v, fa[set][j & 1][i].v, acc[i][j], 0, 0, 0);
  };
  // the step's LDS reads, then its loads, dealt out evenly between the MFMAs
  auto order_step = [&]() {
    constexpr int NR = 2 * DTM + DTN, NM = DTM * DTN, TOT = NR + DLPW / 2, PER = TOT / NM, REM = TOT % NM;
    int done = 0;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      const int cnt = PER + (m < REM ? 1 : 0);
#pragma unroll
      for (int q = 0; q < cnt; ++q) {
        if (done < NR) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        else __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        ++done;
      }
    }
  };
  // slab s has landed once at most the loads of the slabs issued after it (up to `last`) are outstanding
  auto wait_landed = [&](int s, int last, auto full) {
    if (decltype(full)::value) {
      dual_wait_vmcnt<(DSTAGES - 2) * DLPW>();
    } else {
      const int later = min(nk - 1, last) - s;
      if (later <= 0) dual_wait_vmcnt<0>();
      else if (later == 1) dual_wait_vmcnt<DLPW>();
      else dual_wait_vmcnt<2 * DLPW>();
    }
  };

  // Steps n = 0, 1, ... (slab n / 2, half n % 2).  During step n the fragments of step n + 1 are read.
  // Right after the reads of a slab's second half comes its barrier: it publishes the next slab and
  // retires this one, whose stage is refilled three slabs ahead by the two steps that follow.
  const int nsteps = nk * 2;
  // (the last stage gets its first half here; the second goes out with step 0, like every later slab's)
#pragma unroll
  for (int s = 0; s < DSTAGES; ++s)
    if (s < nk) {
      issue(s, s, 0);
      if (s < DSTAGES - 1) issue(s, s, 1);
    }
  if (nk > 0) {
    wait_landed(0, DSTAGES - 2, std::false_type{});
    asm volatile("s_barrier" ::: "memory");
    read_frags(0, 0, 0);
  }
  int slab = 0, stage = 0;
  auto slab_steps = [&](auto full) {   // the two steps of one slab; full: every load referred to exists
    constexpr bool FULL = decltype(full)::value;
    const int nstage = stage + 1 == DSTAGES ? 0 : stage + 1, pstage = stage == 0 ? DSTAGES - 1 : stage - 1;
    read_frags(1, stage, 1);
    if (FULL || slab - 1 + DSTAGES < nk) issue(slab - 1 + DSTAGES, pstage, 1);
    mfma_step(0);
    if (FULL) order_step();
    wait_landed(slab + 1, slab + DSTAGES - 1, full);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    read_frags(0, nstage, 0);   // (past the end: stale data that is never used)
    if (FULL || slab + DSTAGES < nk) issue(slab + DSTAGES, stage, 0);
    mfma_step(1);
    if (FULL) order_step();
    slab += 1;
    stage = nstage;
  };
  int n = 0;
  for (; (n + 1) / 2 + 1 + DSTAGES < nk; n += 2) slab_steps(std::true_type{});
  for (; n < nsteps; n += 2) slab_steps(std::false_type{});

  // lane: row lane & 31, columns 8 g + 4 (lane >> 5) + 0..3 of a 32x32 tile; tile j the gate, j + 1 the up half
#pragma unroll
  for (int j = 0; j < DTN; j += 2) {
    const int cb = n0 + wn * (DBN / DWGN) + j * 32;
    if (cb >= p.N) continue;
#pragma unroll
    for (int i = 0; i < DTM; ++i) {
      const int rblk = m0 / 32 + wm * DTM + i;
      uint32_t pk[4][2];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = silu_fast(acc[i][j][4 * g + e]) * acc[i][j + 1][4 * g + e];
        pk[g][0] = pack_bf16x2(v[0], v[1]);
        pk[g][1] = pack_bf16x2(v[2], v[3]);
      }
      // after the swap the lower lanes hold columns 0..7, the upper ones 8..15 of 16: a chunk each
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        dual_swap32(pk[2 * t][0], pk[2 * t + 1][0]);
        dual_swap32(pk[2 * t][1], pk[2 * t + 1][1]);
        if (rblk * 32 < p.m_pad)
          *(u32x4_t*)((char*)p.C0 + (((int64_t)rblk * (p.ldc0 / 16) + cb / 32 + t) * 64 + lane) * 16) =
              u32x4_t{pk[2 * t][0], pk[2 * t][1], pk[2 * t + 1][0], pk[2 * t + 1][1]};
      }
    }
  }
}

}  // namespace

int launch_gemm_dual(const GemmArgs& a, hipStream_t st) {
  if (a.A1 == nullptr || !a.a_tiled || !a.c0_tiled || a.partial || a.bias != nullptr || a.resid != nullptr || a.out_f32 ||
      a.act_cols != a.N || (a.N & 63) || a.split_col < a.N / 2)
    return -1;
  constexpr size_t lds = (size_t)DSTAGES * DSTAGE * 16;
  static_assert(lds <= 160 * 1024, "LDS budget of a CU");
  // (more dynamic LDS than the default limit: set once per device, as in gemm_bf16.hip)
  static std::atomic<uint64_t> configured{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -1;
  const uint64_t bit = 1ull << (dev & 63);
  if (dev >= 64 || !(configured.load(std::memory_order_acquire) & bit)) {
    if (hipFuncSetAttribute((const void*)gemm_dual_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess)
      return -1;
    if (dev < 64) configured.fetch_or(bit, std::memory_order_release);
  }
  GemmArgs g = a;
  // Eight row tiles to a group.  Four, the least traffic with two left operands, were 0.6 to 1 % faster at
  // 3072 tokens and on the 5120-wide layer and 1 % slower at 4096 tokens; sixteen 1 to 3 % slower.
  g.group_m = 8;
  const int tiles = ((a.M + DBM - 1) / DBM) * ((a.N + DBN - 1) / DBN);
  hipLaunchKernelGGL(gemm_dual_kernel, dim3(tiles), dim3(DNW * 64), lds, st, g);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ffsplit
