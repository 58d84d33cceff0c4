// Small-batch products of the split feed-forward path, gfx950 only: the decode regime, where every
// product is bound by streaming its weights from HBM once.
//   D[M, N] = A[M, K] * Bt[N, K]^T
// rows16_kernel: bf16 weights in the 32 x 16-block tiled layout, M <= 64, one launch per product.
// quant16_up_kernel, quant16_down_kernel: 8- and 3-bit weights (qformat.h), M <= 16, one launch per product.
// skinny_stream_q2_kernel + skinny_reduce_kernel: the same weights, M <= 32.
#include "common.h"
#include "layout.h"
#include "qformat.h"

namespace ffsplit {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

namespace {

union SFrag {
  u32x4_t u;
  bf16x8_t v;
};

// The same product with the weights in the quantised tiled format (32 x 64 blocks of 8- or
// 3-bit codes plus fp16 group scales; qformat.h).  The packed blocks are the only traffic that
// comes from HBM; they are unpacked in the integer domain: a shift, a rotate and two and-or
// per operand register give the pair (magic + u) directly.
//   UP    (one scale per row and 128 reduction elements; activations = the caller's bf16 X):
//         the unscaled codes go through the MFMA, one group of 128 at a time, and the group's
//         fp32 result is scaled per row afterwards.  3 bits: operands are the bf16 values
//         128 + u.  8 bits: the codes do not fit a bf16 mantissa; X is converted to fp16 (exact)
//         and the operands are the fp16 values 1024 + u.
//   DOWN  (one scale per reduction element and 128 rows; activations fp16, written by the UP
//         products' reduce step): the scale multiplies the activations (one packed multiply per
//         register, shared by the row blocks of the group) and the operands are the fp16 values
//         1024 + u.
//   In both, the constant 128 + 4, 1024 + 4 or 1024 + 128 leaves through a second MFMA per
//   operand block whose left operand holds the negated constant in every row.
// Work split: a workgroup of four wavefronts owns RB adjacent row blocks (they share the
// activation blocks, and for DOWN the scales) over one range of the reduction; the wavefronts
// take a quarter of the range each and add their accumulators through LDS in a fixed order.
// A wavefront requests the packed weights of up to SKQ_UNITS units (its whole share at the
// usual shapes) in one batch, so that they cost one round trip to memory, and then the
// activations and scales (cache resident) unit by unit, one unit ahead of the arithmetic.
struct SkinnyQArgs {
  const void* A;
  int64_t lda;
  int M, n_rb, n_split, nu_total, nu_per, slot0;   // units: UP groups of two blocks, DOWN blocks
  int rb_out0, n_rb_part;                          // partial tiles: first row block, row blocks per range
  const char* codes;
  const uint16_t* scales;
  int G, Kp;
  float* part;
};

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
union QFrag {
  u32x4_t u;
  bf16x8_t b;
  f16x8_t h;
};
union H2 {
  uint32_t u;
  f16x2_t h;
};

// Units whose weights a wavefront holds at once, and row blocks per workgroup of the 3-bit parts.
// Both are set by registers: at most 168 per lane keeps three workgroups per CU resident, which
// matters more here than sharing the activation loads among more row blocks (measured: four
// units and four row blocks, two workgroups per CU, 47 us per step at the Llama shape against 41.5).
constexpr int SKQ_UNITS = 2;
constexpr int SKQ_RB_UP3 = 2, SKQ_RB_DOWN3 = 2;

// row blocks per workgroup (they share the activation blocks and, for DOWN, the scales)
constexpr int skq_rb(int bits, bool down) { return bits == 3 ? (down ? SKQ_RB_DOWN3 : SKQ_RB_UP3) : (down ? 2 : 1); }

template <int BITS, bool DOWN>
struct QShape {
  static constexpr int RB = skq_rb(BITS, DOWN);
  static constexpr int UB = DOWN ? 1 : 2;                                  // blocks per unit
};

template <int BITS, bool DOWN>
struct QWts {
  QPacked<BITS> w[QShape<BITS, DOWN>::RB][QShape<BITS, DOWN>::UB];
};

template <int BITS, bool DOWN>
struct QAct {
  u32x4_t a[QShape<BITS, DOWN>::UB * 4];
  u32x4_t sd[DOWN ? 4 : 1];                                  // DOWN: scale pairs of the block's 64 elements
  u32x2_t su[DOWN ? 1 : QShape<BITS, DOWN>::RB][4];          // UP: the lane's 16 row scales per row block
};

template <int BITS, bool DOWN>
__device__ __forceinline__ void skinny_q_body(const SkinnyQArgs& p, int wg, float* red_mem) {
  constexpr int RB = QShape<BITS, DOWN>::RB, UB = QShape<BITS, DOWN>::UB;
  constexpr int BB = BITS == 8 ? 2048 : 768;
  constexpr bool F16 = DOWN || BITS == 8;                    // fp16 MFMA
  float (*red)[RB][16][64] = (float (*)[RB][16][64])red_mem;   // [4][RB][16][64]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_rbg = p.n_rb / RB;
  const int rb = (wg % n_rbg) * RB, sp = wg / n_rbg;
  const int U0 = sp * p.nu_per;
  const int U1 = min(p.nu_total, U0 + p.nu_per);             // U0 < U1 by construction of the grid
  const int per = (U1 - U0 + 3) / 4;
  const int u0 = U0 + wave * per;
  const int u1 = min(U1, u0 + per);                          // may be empty: the wavefront then adds zeros
  const int r = lane & 31, c2 = lane >> 5;

  const char* wbase = p.codes + (int64_t)rb * p.nu_total * UB * BB;
  const int64_t wrow = (int64_t)p.nu_total * UB * BB;        // bytes from one row block to the next
  const char* abase = (const char*)p.A;
  if (DOWN) abase += (int64_t)lane * 16;                              // tiled, one row block
  else abase += ((int64_t)min(r, p.M - 1) * p.lda + c2 * 8) * 2;      // the caller's row-major X

  // (a unit past the range reads some valid unit of it and is not computed)
  auto load_w = [&](QWts<BITS, DOWN>& q, int u) {
    const int uc = max(U0, min(u, U1 - 1));
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int x = 0; x < UB; ++x) {
        const char* blk = wbase + i * wrow + (int64_t)(uc * UB + x) * BB;
        if constexpr (BITS == 8) q.w[i][x] = q_load8(blk, lane);
        else q.w[i][x] = q_load3(blk, lane);
      }
  };
  auto load_a = [&](QAct<BITS, DOWN>& q, int u) {
    const int uc = max(U0, min(u, U1 - 1));
#pragma unroll
    for (int kb = 0; kb < UB * 4; ++kb)
      q.a[kb] = *(const u32x4_t*)(abase + (int64_t)(uc * UB * 4 + kb) * (DOWN ? 1024 : 32));
    if constexpr (DOWN) {
      const uint16_t* sb = p.scales + (int64_t)(rb >> 2) * p.Kp + uc * 64 + 8 * c2;
#pragma unroll
      for (int j = 0; j < 4; ++j) q.sd[j] = *(const u32x4_t*)(sb + 16 * j);
    } else {
      // rows 8 g + 4 c2 + i of a row block live in accumulator registers 4 g + i
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const uint16_t* sb = p.scales + ((int64_t)(rb + i) * p.G + uc) * 32 + 4 * c2;
#pragma unroll
        for (int g = 0; g < 4; ++g) q.su[i][g] = *(const u32x2_t*)(sb + 8 * g);
      }
    }
  };

  const f32x16_t zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  f32x16_t tot[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) tot[i] = zero;

  auto compute = [&](const QWts<BITS, DOWN>& qw, const QAct<BITS, DOWN>& q) {
    QFrag a[UB * 4];
#pragma unroll
    for (int kb = 0; kb < UB * 4; ++kb) {
      a[kb].u = q.a[kb];
      if constexpr (!DOWN && BITS == 8) {
        // bf16 -> fp16: eight significant bits, exact (round toward zero never rounds)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const auto h = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(a[kb].u[i] << 16),
                                                    __uint_as_float(a[kb].u[i] & 0xffff0000u));
          uint32_t hb;
          __builtin_memcpy(&hb, &h, 4);
          a[kb].u[i] = hb;
        }
      }
    }
    // The unpacked operands are the integers magic + u (u the offset-binary code); the constant
    // magic + 2^(bits-1) is removed by a second MFMA whose left operand is that constant,
    // negated, in every row: the vector ALU, which bounds these kernels, only unpacks.
    QFrag negc;
    {
      const uint32_t c = F16 ? (BITS == 8 ? 0xE480E480u /* -1152 */ : 0xE404E404u /* -1028 */) : 0xC304C304u /* bf16 -132 */;
      negc.u = u32x4_t{c, c, c, c};
    }
    if constexpr (DOWN) {
      // the scale depends on the reduction element (and the group of 128 rows, which the RB row
      // blocks share): it multiplies the activations, one packed multiply per register
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          H2 v, s2;
          v.u = a[j].u[i];
          s2.u = q.sd[j][i];
          v.h = v.h * s2.h;
          a[j].u[i] = v.u;
        }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int rbi = 0; rbi < RB; ++rbi) {
          QFrag wf;
#pragma unroll
          for (int i = 0; i < 4; ++i) wf.u[i] = q_pair(qw.w[rbi][0], j, i, BITS == 8 ? 0x64646464u : 0x64006400u);
          tot[rbi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf.h, a[j].h, tot[rbi], 0, 0, 0);
        }
#pragma unroll
        for (int rbi = 0; rbi < RB; ++rbi)
          tot[rbi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(negc.h, a[j].h, tot[rbi], 0, 0, 0);
      }
    } else {
      f32x16_t ag[RB];
#pragma unroll
      for (int i = 0; i < RB; ++i) ag[i] = zero;
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) {
#pragma unroll
        for (int rbi = 0; rbi < RB; ++rbi) {
          QFrag wf;
#pragma unroll
          for (int i = 0; i < 4; ++i) wf.u[i] = q_pair(qw.w[rbi][kb >> 2], kb & 3, i, BITS == 8 ? 0x64646464u : 0x43004300u);
          if constexpr (F16) ag[rbi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf.h, a[kb].h, ag[rbi], 0, 0, 0);
          else ag[rbi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf.b, a[kb].b, ag[rbi], 0, 0, 0);
        }
#pragma unroll
        for (int rbi = 0; rbi < RB; ++rbi) {
          if constexpr (F16) ag[rbi] = __builtin_amdgcn_mfma_f32_32x32x16_f16(negc.h, a[kb].h, ag[rbi], 0, 0, 0);
          else ag[rbi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(negc.b, a[kb].b, ag[rbi], 0, 0, 0);
        }
      }
      // the group's integer dot products times the rows' scales for this group
#pragma unroll
      for (int rbi = 0; rbi < RB; ++rbi)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const u32x2_t sc = q.su[rbi][g];
          const float s4[4] = {q_half((uint16_t)(sc[0] & 0xffffu)), q_half((uint16_t)(sc[0] >> 16)),
                               q_half((uint16_t)(sc[1] & 0xffffu)), q_half((uint16_t)(sc[1] >> 16))};
#pragma unroll
          for (int i = 0; i < 4; ++i) tot[rbi][4 * g + i] = fmaf(s4[i], ag[rbi][4 * g + i], tot[rbi][4 * g + i]);
        }
    }
  };

  for (int ub = u0; ub < u1; ub += SKQ_UNITS) {
    QWts<BITS, DOWN> qw[SKQ_UNITS];
    QAct<BITS, DOWN> qa[2];
#pragma unroll
    for (int i = 0; i < SKQ_UNITS; ++i) load_w(qw[i], ub + i);
    load_a(qa[0], ub);
#pragma unroll
    for (int i = 0; i < SKQ_UNITS; ++i) {
      // (the scheduling barriers keep each batch of loads ahead of the arithmetic of the unit before)
      if (i + 1 < SKQ_UNITS) load_a(qa[(i + 1) & 1], ub + i + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (ub + i < u1) compute(qw[i], qa[i & 1]);   // (wavefront-uniform)
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // fixed-order sum over the four wavefronts; wavefront w finishes accumulator registers 4 w ..
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][i][v][lane] = tot[i][v];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = red[0][i][4 * wave + e][lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) o[e] += red[w][i][4 * wave + e][lane];
    }
    float4* dst = (float4*)p.part + ((int64_t)((p.slot0 + sp) * p.n_rb_part + p.rb_out0 + rb + i) * 4 + wave) * 64 + lane;
    *dst = make_float4(o[0], o[1], o[2], o[3]);
  }
}

// One launch for the 8-bit and the 3-bit part of a product: workgroups [0, wg8) take the
// first, the rest the second.
struct SkinnyQ2Args {
  SkinnyQArgs s8, s3;
  int wg8;
};

template <bool DOWN>
__global__ void __launch_bounds__(256) skinny_stream_q2_kernel(const SkinnyQ2Args p) {
  extern __shared__ float red_mem[];
  if ((int)blockIdx.x < p.wg8) skinny_q_body<8, DOWN>(p.s8, (int)blockIdx.x, red_mem);
  else skinny_q_body<3, DOWN>(p.s3, (int)blockIdx.x - p.wg8, red_mem);
}

__device__ __forceinline__ float sk_silu(float z) { return silu_fast(z); }   // exp2 and rcp: no division sequence

// Sum over the ranges (fixed order), activation, bf16 stores.  One thread per (block, lane,
// g): token row = lane & 31, four consecutive columns.
struct SkinnyReduceArgs {
  const float* part;
  int n_rb, n_split, M, N;
  int act, act_cols, split_col;
  void* C0;
  void* C1;
  int64_t ldc0, ldc1;
  int c0_tiled, c1_tiled, n_store;
  int f16_out;   // destinations hold fp16 (saturating) instead of bf16
  int rb_split, n_split_b;   // row blocks from rb_split on have n_split_b ranges
  const float* bias;         // as in GemmArgs
  int bias_cols;
  const float* resid;
  int64_t ldr;
  int out_f32;
};

__device__ __forceinline__ uint32_t pack_f16x2_sat(float lo, float hi) {
  H2 v;
  v.h = f16x2_t{(_Float16)fminf(fmaxf(lo, -65504.f), 65504.f), (_Float16)fminf(fmaxf(hi, -65504.f), 65504.f)};
  return v.u;
}

// Activation and store of four consecutive output columns (columns c .. c + 3 of row block rb, of
// token `row`): v the block's sums, u the up block's sums for a (gate, up) pair.
__device__ __forceinline__ void sk_emit(const SkinnyReduceArgs& p, int rb, int c4, int row, float v[4],
                                        const float u[4]) {
  const int cb = rb * 32;
  const bool act_here = cb < p.act_cols;
  const bool glu = p.act == ACT_GLU;
  int oc = cb;
  if (glu) oc = act_here ? cb / 2 : cb - p.act_cols / 2;
  {
    // a neuron's bias (GEMM column cb + c4 + e), before the activation
    const int c = cb + c4;
    if (!glu && p.bias != nullptr && c + 3 < p.bias_cols) {
      const float4 b4 = *(const float4*)(p.bias + c);
      v[0] += b4.x; v[1] += b4.y; v[2] += b4.z; v[3] += b4.w;
    }
  }
  if (act_here) {
    if (glu) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = sk_silu(v[e]) * u[e];
    } else if (p.act == ACT_GELU) {
#pragma unroll
      // the bf16 path's GeLU (common.h); erff here costs the kernels that inline this 60 registers per
      // lane and with them a workgroup per CU
      for (int e = 0; e < 4; ++e) v[e] = gelu_fast(v[e]);
    }
  }
  const int col0 = oc + c4;   // first of this thread's four output columns
  char* base;
  int64_t ld;
  int col, tiled;
  const bool to_c0 = col0 < p.split_col;
  if (to_c0) { base = (char*)p.C0; ld = p.ldc0; col = col0; tiled = p.c0_tiled; }
  else { base = (char*)p.C1; ld = p.ldc1; col = col0 - p.split_col; tiled = p.c1_tiled; }
  if (to_c0 && !tiled && row < p.M && col < p.n_store) {
    if (p.resid != nullptr) {
      const float4 r4 = *(const float4*)(p.resid + (int64_t)row * p.ldr + col);
      v[0] += r4.x; v[1] += r4.y; v[2] += r4.z; v[3] += r4.w;
    }
    if (p.out_f32) {
      *(float4*)((float*)base + (int64_t)row * ld + col) = make_float4(v[0], v[1], v[2], v[3]);
      return;
    }
  }
  const uint2 val = p.f16_out ? make_uint2(pack_f16x2_sat(v[0], v[1]), pack_f16x2_sat(v[2], v[3]))
                              : make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
  if (tiled) {
    // (rows past M hold repeats of row M - 1; past the last block of 16 rows nothing is written or read)
    const int64_t chunk = ((int64_t)(row >> 5) * (ld / 16) + col / 16) * 64 + ((col >> 3) & 1) * 32 + (row & 31);
    *(uint2*)(base + chunk * 16 + (col & 7) * 2) = val;
  } else if (row < p.M && col < p.n_store) {
    *(uint2*)(base + ((int64_t)row * ld + col) * 2) = val;
  }
}

__global__ void __launch_bounds__(256) skinny_reduce_kernel(const SkinnyReduceArgs p) {
  // one workgroup per row block, one wavefront per g: both uniform, so that the partial sums' addresses
  // are scalar but for the lane
  const int rb = blockIdx.x, lane = threadIdx.x & 63;
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool pair = p.act == ACT_GLU && rb * 32 < p.act_cols;
  if (pair && (rb & 1)) return;   // the pair is written from its gate block
  auto sum_block = [&](int b) {
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4* src = (const float4*)p.part + ((int64_t)b * 4 + g) * 64 + lane;
    // eight independent loads at a time, added in range order (24 at a time, all ranges of the
    // usual products in one round trip, measured slower: 5.9 vs 4.3 us, and 8.4 vs 5.0 us where
    // there are few ranges and most of the 24 were repeats)
    const int64_t step = (int64_t)p.n_rb * 256;
    const int ns = b < p.rb_split ? p.n_split : p.n_split_b;
    constexpr int NB = 8;
    for (int sp = 0; sp < ns; sp += NB) {
      float4 v[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) v[u] = src[(int64_t)min(sp + u, ns - 1) * step];
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (sp + u < ns) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
    }
    return s;
  };
  const float4 z0 = sum_block(rb);
  float v[4] = {z0.x, z0.y, z0.z, z0.w};
  float uu[4] = {0.f, 0.f, 0.f, 0.f};
  if (pair) {
    const float4 u = sum_block(rb + 1);
    uu[0] = u.x; uu[1] = u.y; uu[2] = u.z; uu[3] = u.w;
  }
  sk_emit(p, rb, 8 * g + 4 * (lane >> 5), lane & 31, v, uu);
}

// A product of at most 64 tokens in one launch, bound by streaming its weights once.
// A workgroup of four wavefronts owns 16 weight rows (RB = 1) or two such pieces (RB = 2: a 32-row
// block, or 16 gate rows and their 16 up rows) over one range of the reduction.  The wavefronts share
// the range evenly and keep a ring of U steps of 32 reduction elements in registers, each refilled as
// it is used; a step past the range is an out-of-range buffer load (zero), so nothing in the loop is
// masked, and the last round of the ring loads nothing.  The accumulators meet in LDS and are added
// in a fixed order.  Pieces of 16 rows and 16 tokens (v_mfma_f32_16x16x32_bf16) make twice as many
// workgroups of the same rows as 32 x 32 ones, and with up to 16 tokens half the activation loads.
// With n_split > 1 the ranges of one unit are added by the last of its workgroups to arrive, in range
// order: the second launch that this replaces cost 4-5 us, more than the sums are worth, and the
// result does not depend on the order of arrival.
// Measured (us; 32 x 32 blocks with a reduce launch or 4-8 wavefronts before -> now): Llama-2-7B-sized
// low-rank layer, 8 tokens 47.6 -> 34.1, 32 tokens 49.9 -> 45.4, 64 tokens 71.7 -> 60.9; four
// OPT-13B-sized layers, 16 tokens 248 -> 185 (3.1 TB/s of weights); OPT-1.3B-sized layer, 1 token
// 36 -> 21, 48 tokens 46.5 -> 28.6.  Sixteen wavefronts per workgroup instead of four: 41.8 and 244
// at the first and the fourth; eight: 39.7 and 219 (with a ring of eight); a ring of 12 costs 2 % more
// than one of 4-6, because what it holds past the range is loaded for nothing.
constexpr int ROWS16_MAX_SPLIT = 8;
constexpr int ROWS16_NW = 4;      // wavefronts of a workgroup
constexpr int ROWS16_WGS = 256;   // workgroups of a full machine
static_assert(ROWS16_WGS / 2 <= SKINNY_COUNTERS, "a product is cut only if two ranges of it fit one round");

struct Rows16Args {
  const void* A;
  const void* A1;      // DUAL: the up rows' left operand
  const void* Bt;
  int64_t lda, ldb;
  int M, K, steps;     // steps of 32 reduction elements
  int pair_units;      // GLU: units below this are (gate, up) pairs
  int n_units, n_split;
  float* part;         // [unit][n_split][pieces][64] float4
  unsigned* counters;  // one per unit
  unsigned* clear;     // counters of later launches to zero
  int n_clear;
  SkinnyReduceArgs e;
};

typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t sk_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, bytes, 0x00027000);
}
__device__ __forceinline__ u32x4_t sk_load(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
// partial sums cross workgroups of one launch: device-scope accesses go to the point where the
// per-XCD L2 caches are coherent
__device__ __forceinline__ void sk_st_dev(float4* p, float4 v) {
  unsigned long long* q = (unsigned long long*)p;
  __hip_atomic_store(q, (unsigned long long)__float_as_uint(v.x) | ((unsigned long long)__float_as_uint(v.y) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(q + 1, (unsigned long long)__float_as_uint(v.z) | ((unsigned long long)__float_as_uint(v.w) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float4 sk_ld_dev(const float4* p) {
  const unsigned long long* q = (const unsigned long long*)p;
  const unsigned long long a = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long b = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float4(__uint_as_float((unsigned)a), __uint_as_float((unsigned)(a >> 32)), __uint_as_float((unsigned)b),
                     __uint_as_float((unsigned)(b >> 32)));
}

// One unit: pieces at rows 16 sub[i] of the 32-row blocks rb[i].
template <bool A_TILED, int TB, int RB, int NW, int U, bool DUAL, bool SPLIT>
__device__ __forceinline__ void rows16_unit(const Rows16Args& p, int unit, int sp, const int (&rb)[RB],
                                            const int (&sub)[RB], bool pair, float4* red, int* flag) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  constexpr int NA = DUAL ? 2 : 1;
  constexpr bool TURN = !A_TILED && (TB > 1 || SPLIT);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this workgroup's range, then this wavefront's share of it (may be empty: it then adds zeros)
  const uint32_t steps = p.steps, parts = SPLIT ? p.n_split : 1;
  const int w0 = SPLIT ? (int)(steps * (uint32_t)sp / parts) : 0;
  const int wn = (SPLIT ? (int)(steps * (uint32_t)(sp + 1) / parts) : p.steps) - w0;
  const int s0 = w0 + wn * wave / NW, s1 = w0 + wn * (wave + 1) / NW;
  const int r = lane & 15, q8 = (lane >> 4) * 8;

  // tiled: a step is two 1 KiB blocks of 32 rows x 16 reduction elements; the lane's 16 bytes are
  // row r of a 16-row half, elements q8 ..
  const uint32_t lofs = (uint32_t)((lane >> 5) * 1024 + ((lane >> 4) & 1) * 512 + r * 16);
  rsrc_t wr[RB];
  uint32_t wofs[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    wr[i] = sk_rsrc((const char*)p.Bt + (int64_t)rb[i] * (p.ldb / 16) * 1024, (uint32_t)s1 * 2048u);
    wofs[i] = lofs + (uint32_t)sub[i] * 256u;
  }
  const int k_end = min(p.K, s1 * 32);
  rsrc_t ar[NA][(TB + 1) / 2];   // tiled: one per block of 32 tokens
  const int ac = TURN ? (lane & 3) * 8 : q8;   // row-major: the lane's chunk of a step
  uint32_t aofs[TB];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int t = 0; t < TB; t += 2) {
      const char* base = (const char*)(i ? p.A1 : p.A);
      ar[i][t / 2] = A_TILED ? sk_rsrc(base + (int64_t)(t / 2) * (p.lda / 16) * 1024, (uint32_t)s1 * 2048u)
                             : sk_rsrc(base, (uint32_t)(p.M * (int)p.lda * 2));
    }
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    if (A_TILED) aofs[t] = lofs + (uint32_t)(t & 1) * 256u;
    else aofs[t] = (uint32_t)(min(t * 16 + (TURN ? lane >> 2 : r), p.M - 1) * (int)p.lda + ac) * 2u;
  }
  // Row-major tokens (not gated ones up to 16): four neighbouring lanes read 64 bytes of a row (a row per lane, as the MFMA wants
  // them, comes at 16 bytes a clock instead of 61), and the wavefront turns the step round in LDS of its
  // own, where its sums go at the end: lane l holds chunk l & 3 of token l >> 2 and gets chunk l >> 4 of token
  // l & 15.  us, a Llama-2-7B-sized layer: 32 tokens 35.4 -> 33.2, 64 tokens 47.6 -> 42.2 (8 tokens 29.0 either way, 1 token
  // 29.0 -> 29.4).  Ungated, with a ring of eight instead of four, which pays only then: four layers of 2048 x 8192,
  // 16 tokens 94.9 -> 91.3, of 5120 x 20480, 1 token 177.5 -> 171.9, 16 tokens 183.8 -> 183.5.
  u32x4_t* const turn = (u32x4_t*)red + wave * RB * TB * 64;
  const int put_at = (lane & ~3) | ((lane & 3) ^ ((lane >> 4) & 3)), get_at = r * 4 + ((lane >> 4) ^ (r >> 2));
  u32x4_t w[U][RB], a[U][NA][TB];
  auto load = [&](int u, int s) {
#pragma unroll
    for (int i = 0; i < RB; ++i) w[u][i] = sk_load(wr[i], wofs[i] + (uint32_t)s * 2048u);
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        if (A_TILED) a[u][i][t] = sk_load(ar[i][t / 2], aofs[t] + (uint32_t)s * 2048u);
        else a[u][i][t] = sk_load(ar[i][t / 2], s * 32 + ac < k_end ? aofs[t] + (uint32_t)s * 64u : 0xfffffff0u);
      }
  };
  f32x4_t acc[RB][TB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int t = 0; t < TB; ++t) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  u32x4_t turned[TB];   // TURN: the tokens of the step that is multiplied next
  auto turn_round = [&](int u) {
#pragma unroll
    for (int t = 0; t < TB; ++t) turn[t * 64 + put_at] = a[u][0][t];
#pragma unroll
    for (int t = 0; t < TB; ++t) turned[t] = turn[t * 64 + get_at];
  };
  // (next: the ring's following step, -1 past the last)
  auto step = [&](int u, int next) {
    __builtin_amdgcn_sched_barrier(0);
    u32x4_t now[TB];
    if (TURN) {
#pragma unroll
      for (int t = 0; t < TB; ++t) now[t] = turned[t];
      if (next >= 0) turn_round(next);
    }
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        SFrag wf, af;
        wf.u = w[u][i];
        af.u = TURN ? now[t] : a[u][DUAL ? i : 0][t];
        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf.v, af.v, acc[i][t], 0, 0, 0);
      }
  };
  if (s0 < s1) {
#pragma unroll
    for (int u = 0; u < U; ++u) load(u, s0 + u);
    if (TURN) turn_round(0);
    for (int s = s0 + U; s < s1; s += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        step(u, (u + 1) % U);
        load(u, s + u);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) step(u, u + 1 < U ? u + 1 : -1);
  }
  // lane: token t * 16 + r, rows 4 (lane >> 4) + 0..3 of the piece
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int t = 0; t < TB; ++t)
      red[((wave * RB + i) * TB + t) * 64 + lane] = make_float4(acc[i][t][0], acc[i][t][1], acc[i][t][2], acc[i][t][3]);
  __syncthreads();
  auto lds_sum = [&](int piece) {
    float4 v = red[piece * 64 + lane];
#pragma unroll
    for (int w2 = 1; w2 < NW; ++w2) {
      const float4 x = red[(w2 * RB * TB + piece) * 64 + lane];
      v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w;
    }
    return v;
  };
  const int c4 = 4 * (lane >> 4);
  const float none[4] = {0.f, 0.f, 0.f, 0.f};
  if (SPLIT && p.n_split > 1) {
    float4* mine = (float4*)p.part + ((int64_t)unit * p.n_split + sp) * RB * TB * 64 + lane;
    for (int pc = wave; pc < RB * TB; pc += NW) sk_st_dev(mine + pc * 64, lds_sum(pc));
    // Every thread waits for its own device-scope stores before the barrier, and only after it does
    // thread 0 count this workgroup in: whoever reads n_split - 1 finds all partial sums in place.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      const bool last = __hip_atomic_fetch_add(&p.counters[unit], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                        (unsigned)(p.n_split - 1);
      if (last) __hip_atomic_store(&p.counters[unit], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *flag = last;
    }
    __syncthreads();
    if (!*flag) return;
    for (int pc = wave; pc < RB * TB; pc += NW) {
      const float4* src = (const float4*)p.part + (int64_t)unit * p.n_split * RB * TB * 64 + pc * 64 + lane;
      float4 x[ROWS16_MAX_SPLIT];
#pragma unroll
      for (int s = 0; s < ROWS16_MAX_SPLIT; ++s)
        x[s] = sk_ld_dev(src + (int64_t)min(s, p.n_split - 1) * RB * TB * 64);
      float v[4] = {x[0].x, x[0].y, x[0].z, x[0].w};
#pragma unroll
      for (int s = 1; s < ROWS16_MAX_SPLIT; ++s)
        if (s < p.n_split) { v[0] += x[s].x; v[1] += x[s].y; v[2] += x[s].z; v[3] += x[s].w; }
      const int i = RB > 1 ? pc / TB : 0, t = pc % TB;
      sk_emit(p.e, i ? rb[RB - 1] : rb[0], 16 * (i ? sub[RB - 1] : sub[0]) + c4, t * 16 + r, v, none);
    }
    return;
  }
  if (RB == 2 && pair) {
    for (int t = wave; t < TB; t += NW) {
      const float4 g = lds_sum(t), up = lds_sum(TB + t);
      float v[4] = {g.x, g.y, g.z, g.w};
      const float uu[4] = {up.x, up.y, up.z, up.w};
      sk_emit(p.e, rb[0], 16 * sub[0] + c4, t * 16 + r, v, uu);
    }
    return;
  }
  for (int pc = wave; pc < RB * TB; pc += NW) {
    const float4 sum = lds_sum(pc);
    float v[4] = {sum.x, sum.y, sum.z, sum.w};
    const int i = RB > 1 ? pc / TB : 0, t = pc % TB;
    sk_emit(p.e, i ? rb[RB - 1] : rb[0], 16 * (i ? sub[RB - 1] : sub[0]) + c4, t * 16 + r, v, none);
  }
}

// GLU: units below pair_units are (gate, up) pairs, the others hold RB pieces
template <bool A_TILED, int TB, int RB, int NW, int U, bool GLU, bool DUAL>
__global__ void __launch_bounds__(NW * 64) rows16_kernel(const Rows16Args p) {
  extern __shared__ float4 red4[];
  __shared__ int flag;
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < p.n_clear; i += NW * 64) p.clear[i] = 0u;
  const int unit = (int)blockIdx.x % p.n_units, sp = (int)blockIdx.x / p.n_units;
  if (GLU && unit < p.pair_units) {
    const int rb[2] = {unit & ~1, unit | 1}, sub[2] = {unit & 1, unit & 1};
    rows16_unit<A_TILED, TB, 2, NW, U, DUAL, false>(p, unit, 0, rb, sub, true, red4, &flag);
    return;
  }
  if constexpr (!DUAL) {
    const int v = unit - p.pair_units;
    if constexpr (RB == 2) {
      const int rb[2] = {p.pair_units + v, p.pair_units + v}, sub[2] = {0, 1};
      rows16_unit<A_TILED, TB, 2, NW, U, false, false>(p, unit, 0, rb, sub, false, red4, &flag);
    } else {
      const int rb[1] = {p.pair_units + (v >> 1)}, sub[1] = {v & 1};
      rows16_unit<A_TILED, TB, 1, NW, U, false, !GLU>(p, unit, sp, rb, sub, false, red4, &flag);
    }
  }
}

// ---- 8- and 3-bit weights, at most 16 tokens: one launch per product, no sums across workgroups.
// A piece is 16 weight rows: lane (r, q) = (lane & 15, lane >> 4) takes what lane 32 (q & 1) + r of the piece's half
// holds of the 32 x 64 block 2 u + (q >> 1), so that one 12-byte (8 bits: two 16-byte) load a lane is a unit of
// 16 rows x 128 reduction elements and, unpacked, the operands of four v_mfma_f32_16x16x32: MFMA j covers the
// elements 64 (q >> 1) + 16 j + 8 (q & 1) + 0..7 of quad q, and the activations are loaded to match.
//   UP    A workgroup of eight wavefronts keeps all 16 tokens in registers, wavefront w the groups w, w + 8, ..
//         of 128 inputs, and walks over pairs of pieces (16 gate and their 16 up rows, or the two halves of a row block);
//         a group's registers are refilled for the next pair as soon as it is multiplied.  The constant of the
//         offset-binary codes enters as the accumulator's start value, -132 (-1152) times the group's sum
//         of the tokens, computed once.  3 bits: the four pairs of an operand share one rotated dword of third
//         bits, pair i as 128 + 2^i u, and the tokens it meets are scaled by 2^-i (exact) beforehand: 52
//         vector instructions for 16 x 128 codes instead of 64.  The wavefronts' sums meet in LDS, where
//         one of them adds, activates and stores the pair while the others go on.
//   DOWN  A workgroup owns one piece of 16 outputs (4096 outputs: one each CU) over the whole reduction, its wavefronts
//         an eighth each; the 3-bit codes alternate between two sets of registers, the 8-bit ones have one, and so have
//         activations and scales: they are requested when the unit before is multiplied and needed at once, so that their
//         latency is covered by the other wavefronts only.  Deeper rings are slower (six sets of codes and two of activations:
//         2 us a launch): the code is run once or twice over, and twice its size costs more than the loads it has in flight.
//         The codes become exact fp16 integers in one more packed operation each (3 bits: 2^i u with the rotation shared as in UP,
//         scaled and shifted by one v_pk_fma_f16), which costs no time: the MFMA on the negated constant that went with operands
//         of 1024 + u goes.  With these the sums passed through 1024 times those of activations of one sign: relative error of an fp32
//         result, 2048 x 16384 GeLU, 16 tokens, 3.9e-4 in the kernels below, 2.9e-4 here, all of it the activations' own rounding.
// The kernels below spend half of their 32-row MFMAs on absent tokens, a second MFMA on the constant of UP, and two
// launches on sums across workgroups.  us, a layer of 16 tokens with its norm, those -> these: 4096 x 11008 gated 44.9 ->
// 32.0 (up 19.9 + 5.0 -> 16.6, down 13.8 + 4.1 -> 11.0), 2048 x 8192 25.7 -> 19.0, 1280 x 4000 22.3 -> 14.3; the operands
// scaled by powers of two are 1.2 of up's us, one set of registers instead of two another 1.2 (8.5 us of 124 for four
// layers of one token).  Bound by the unpacking (half of the time), the ramp of each launch, and in DOWN the
// 8 KB of activations and scales that every 1.5 KB of codes meets.
constexpr int Q16_NW = 8, Q16_DOWN_NW = 8;   // (sixteen for DOWN: 2 % slower, twelve: 1 % faster at one shape, slower at others)
constexpr int Q16_MAX_GPW = 5;   // groups of 128 inputs a wavefront holds

struct Q16UpArgs {
  const void* X;
  int64_t lda;
  int M, G;
  const char* codes[2];          // 8 bits, 3 bits
  const uint16_t* scales[2];
  int units8, units3, wgs3, rb3;   // rb3: first row block of the 3-bit part in the output's order
  SkinnyReduceArgs e;
};

typedef __attribute__((ext_vector_type(4))) float q16_f32x4;

template <int BITS, int GPW, bool GLU>
__device__ __forceinline__ void quant16_up(const Q16UpArgs& p, int u0, int step, int units, float4* red) {
  constexpr int PART = BITS == 8 ? 0 : 1, BB = BITS == 8 ? 2048 : 768;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the tokens: groups wave, wave + 8, .. (zeros past the last group)
  QFrag x[GPW][4];
  {
    const char* xr = (const char*)p.X + ((int64_t)min(r, p.M - 1) * p.lda + (q >> 1) * 64 + (q & 1) * 8) * 2;
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
      const int gi = wave + g * Q16_NW;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        x[g][j].u = gi < p.G ? *(const u32x4_t*)(xr + (int64_t)gi * 256 + j * 32) : u32x4_t{0, 0, 0, 0};
    }
  }
  // One set of registers for the packed codes and the lane's four row scales of both pieces, refilled piece by piece:
  // as soon as a group is multiplied its registers are loaded for the next pair.  (A second set, filled ahead, has the code
  // twice and no room to spare.)  Past the last pair the loads are out of range: zero, and no traffic.  A
  // group past the last repeats it: its tokens are zero.
  struct Wts {
    QPacked<BITS> w[2][GPW];
    u32x2_t s[2][GPW];
  } wts;
  auto load = [&](int i, int g, int u, uint32_t limit) {
    const rsrc_t cr = sk_rsrc(p.codes[PART], limit), sr = sk_rsrc(p.scales[PART], limit);
    const int rb = GLU ? (u & ~1) + i : u, sub = GLU ? (u & 1) : i;
    const int gi = min(wave + g * Q16_NW, p.G - 1);
    const uint32_t blk = ((uint32_t)rb * p.G + gi) * 2 * BB, lo = (uint32_t)(q >> 1) * BB + (uint32_t)(32 * (q & 1) + r) * (BITS == 8 ? 16 : 12);
    if constexpr (BITS == 8) {
      wts.w[i][g].h[0] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(cr, lo, blk + sub * 256, 0));
      wts.w[i][g].h[1] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(cr, lo, blk + sub * 256 + 1024, 0));
    } else {
      typedef __attribute__((ext_vector_type(3))) uint32_t u32x3_t;
      const u32x3_t v = __builtin_bit_cast(u32x3_t, __builtin_amdgcn_raw_buffer_load_b96(cr, lo, blk + sub * 192, 0));
      wts.w[i][g].lo[0] = v[0]; wts.w[i][g].lo[1] = v[1]; wts.w[i][g].hi = v[2];
    }
    wts.s[i][g] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(sr, 8 * q, ((uint32_t)rb * p.G + gi) * 64 + sub * 32, 0));
  };
  constexpr uint32_t ALL = 0xfffffff0u;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int g = 0; g < GPW; ++g) load(i, g, u0, ALL);
  // start values: every row of the operand holds the negated constants, so a token's is the same in all rows
  float start[GPW];
  {
    QFrag negc;
    if (BITS == 8) negc.u = u32x4_t{0xE480E480u, 0xE480E480u, 0xE480E480u, 0xE480E480u};   // fp16 -1152
    else negc.u = u32x4_t{0xC304C304u, 0xC308C308u, 0xC310C310u, 0xC320C320u};             // bf16 -(128 + 4 2^i)
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
      q16_f32x4 st = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (BITS == 8) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {   // bf16 -> fp16: eight significant bits, exact
            const auto h = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(x[g][j].u[i] << 16), __uint_as_float(x[g][j].u[i] & 0xffff0000u));
            uint32_t hb;
            __builtin_memcpy(&hb, &h, 4);
            x[g][j].u[i] = hb;
          }
          st = __builtin_amdgcn_mfma_f32_16x16x32_f16(negc.h, x[g][j].h, st, 0, 0, 0);
        } else {
#pragma unroll
          for (int i = 1; i < 4; ++i) {
            const float s = i == 1 ? 0.5f : i == 2 ? 0.25f : 0.125f;
            x[g][j].u[i] = pack_bf16x2(__uint_as_float(x[g][j].u[i] << 16) * s, __uint_as_float(x[g][j].u[i] & 0xffff0000u) * s);
          }
          st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(negc.b, x[g][j].b, st, 0, 0, 0);
        }
      }
      start[g] = st[0];
    }
  }
  int buf = 0, owner = 0;
  auto unit = [&](int u, int next, bool more) {
    const uint32_t limit = more ? ALL : 0u;
    q16_f32x4 tot[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      tot[i] = q16_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < GPW; ++g) {
        q16_f32x4 ag = {start[g], start[g], start[g], start[g]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          QFrag wf;
          if constexpr (BITS == 8) {
#pragma unroll
            for (int e = 0; e < 4; ++e) wf.u[e] = q_pair(wts.w[i][g], j, e, 0x64646464u);
          } else {
            q_pairs_scaled(wts.w[i][g], j, 0x43004300u, wf.u);
          }
          if constexpr (BITS == 8) ag = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf.h, x[g][j].h, ag, 0, 0, 0);
          else ag = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf.b, x[g][j].b, ag, 0, 0, 0);
        }
        const u32x2_t sc = wts.s[i][g];
        tot[i][0] = fmaf(q_half((uint16_t)(sc[0] & 0xffffu)), ag[0], tot[i][0]);
        tot[i][1] = fmaf(q_half((uint16_t)(sc[0] >> 16)), ag[1], tot[i][1]);
        tot[i][2] = fmaf(q_half((uint16_t)(sc[1] & 0xffffu)), ag[2], tot[i][2]);
        tot[i][3] = fmaf(q_half((uint16_t)(sc[1] >> 16)), ag[3], tot[i][3]);
        if constexpr (BITS == 3) {
          __builtin_amdgcn_sched_barrier(0);
          load(i, g, next, limit);
        }
      }
    }
    // (two buffers: nobody is more than one barrier ahead of the wavefront that adds)
    float4* const m = red + buf * Q16_NW * 2 * 64;
#pragma unroll
    for (int i = 0; i < 2; ++i) m[(wave * 2 + i) * 64 + lane] = make_float4(tot[i][0], tot[i][1], tot[i][2], tot[i][3]);
    __syncthreads();
    if (wave == owner) {
      float v[2][4];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float4 t = m[i * 64 + lane];
#pragma unroll
        for (int w2 = 1; w2 < Q16_NW; ++w2) {
          const float4 o = m[(w2 * 2 + i) * 64 + lane];
          t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
        }
        v[i][0] = t.x; v[i][1] = t.y; v[i][2] = t.z; v[i][3] = t.w;
      }
      const int rb0 = PART ? p.rb3 : 0;
      if (GLU) {
        sk_emit(p.e, rb0 + (u & ~1), 16 * (u & 1) + 4 * q, r, v[0], v[1]);
      } else {
        const float none[4] = {0.f, 0.f, 0.f, 0.f};
        sk_emit(p.e, rb0 + u, 4 * q, r, v[0], none);
        sk_emit(p.e, rb0 + u, 16 + 4 * q, r, v[1], none);
      }
    }
    buf ^= 1;
    owner = (owner + 1) % Q16_NW;
  };
  if constexpr (BITS == 8) {   // (one pair a workgroup)
    unit(u0, u0, false);
  } else {
    for (int u = u0; u < units; u += step) unit(u, u + step < units ? u + step : u, u + step < units);
  }
}

template <int GPW, bool GLU>
__global__ void __launch_bounds__(Q16_NW * 64) quant16_up_kernel(const Q16UpArgs p) {
  __shared__ float4 red[2 * Q16_NW * 2 * 64];
  if ((int)blockIdx.x < p.units8) quant16_up<8, GPW, GLU>(p, blockIdx.x, 0, 0, red);
  else quant16_up<3, GPW, GLU>(p, (int)blockIdx.x - p.units8, p.wgs3, p.units3, red);
}

struct Q16DownArgs {
  const void* H;                 // [32, k4] tiled fp16
  const char* codes[2];
  const uint16_t* scales[2];
  int Kp[2];                     // padded neurons of the 8- and the 3-bit part; the second follows the first in H
  SkinnyReduceArgs e;
};

// this wavefront's share of one part of the reduction, in units of 128 neurons
template <int BITS>
__device__ __forceinline__ void quant16_down(const Q16DownArgs& p, int piece, q16_f32x4& tot) {
  constexpr int PART = BITS == 8 ? 0 : 1, BB = BITS == 8 ? 2048 : 768, UW = BITS == 8 ? 1 : 2, UA = 1;
  const int Kp = p.Kp[PART], units = (Kp + 127) / 128;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = units * wave / Q16_DOWN_NW, c1 = units * (wave + 1) / Q16_DOWN_NW;
  if (c0 >= c1) return;
  const int rb = piece >> 1, sub = piece & 1;
  // (past the last block of 64 neurons, and past the share, loads are out of range: zero)
  const rsrc_t wr = sk_rsrc(p.codes[PART] + (int64_t)rb * (Kp / 64) * BB, (uint32_t)min(c1 * 2, Kp / 64) * BB);
  const rsrc_t hr = sk_rsrc((const char*)p.H + (PART ? (size_t)p.Kp[0] * 64 : 0), (uint32_t)min(c1 * 128, Kp) * 64u);
  const rsrc_t sr = sk_rsrc(p.scales[PART] + (int64_t)(rb >> 2) * Kp, (uint32_t)min(c1 * 128, Kp) * 2u);
  const uint32_t wofs = (uint32_t)(q >> 1) * BB + (uint32_t)(32 * (q & 1) + 16 * sub + r) * (BITS == 8 ? 16 : 12);
  const uint32_t hofs = (uint32_t)((q >> 1) * 4 * 64 + (q & 1) * 32 + r) * 16;
  const uint32_t sofs = (uint32_t)((q >> 1) * 64 + (q & 1) * 8) * 2;
  QPacked<BITS> w[UW];
  QFrag h[UA][4], sc[UA][4];
  auto load_w = [&](QPacked<BITS>& d, int c) {
    const uint32_t o = wofs + (uint32_t)c * 2 * BB;
    if constexpr (BITS == 8) {
      d.h[0] = sk_load(wr, o);
      d.h[1] = sk_load(wr, o + 1024);
    } else {
      typedef __attribute__((ext_vector_type(3))) uint32_t u32x3_t;
      const u32x3_t v = __builtin_bit_cast(u32x3_t, __builtin_amdgcn_raw_buffer_load_b96(wr, o, 0, 0));
      d.lo[0] = v[0]; d.lo[1] = v[1]; d.hi = v[2];
    }
  };
  auto load_a = [&](QFrag (&hh)[4], QFrag (&ss)[4], int c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      hh[j].u = sk_load(hr, hofs + (uint32_t)c * 8192 + j * 1024);
      ss[j].u = sk_load(sr, sofs + (uint32_t)c * 256 + j * 32);
    }
  };
  auto unit = [&](const QPacked<BITS>& d, QFrag (&hh)[4], const QFrag (&ss)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      QFrag wf, a;
      if constexpr (BITS == 3) q_pairs_scaled(d, j, 0x64006400u, wf.u);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        H2 v, s2, q, one, off;
        v.u = hh[j].u[i];
        s2.u = ss[j].u[i];
        v.h = v.h * s2.h;
        a.u[i] = v.u;
        if constexpr (BITS == 3) {   // (1024 + 2^i u) 2^-i - (1024 2^-i + 4)
          constexpr uint32_t ONE[4] = {0x3C003C00u, 0x38003800u, 0x34003400u, 0x30003000u};
          constexpr uint32_t OFF[4] = {0xE404E404u, 0xE008E008u, 0xDC10DC10u, 0xD820D820u};
          q.u = wf.u[i]; one.u = ONE[i]; off.u = OFF[i];
          q.h = __builtin_elementwise_fma(q.h, one.h, off.h);
        } else {                     // 1024 + 128 + code
          q.u = q_pair(d, j, i, 0x64646464u); off.u = 0xE480E480u;
          q.h = q.h + off.h;
        }
        wf.u[i] = q.u;
      }
      tot = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf.h, a.h, tot, 0, 0, 0);
    }
  };
  static_assert(UW % UA == 0, "");
#pragma unroll
  for (int i = 0; i < UA; ++i) load_a(h[i], sc[i], c0 + i);
#pragma unroll
  for (int i = 0; i < UW; ++i) load_w(w[i], c0 + i);
  for (int c = c0; c < c1; c += UW) {
#pragma unroll
    for (int i = 0; i < UW; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (c + i < c1) {   // (uniform)
        unit(w[i], h[i % UA], sc[i % UA]);
        if (c + i + UW < c1) load_w(w[i], c + i + UW);
        if (c + i + UA < c1) load_a(h[i % UA], sc[i % UA], c + i + UA);
      }
    }
  }
}

__global__ void __launch_bounds__(Q16_DOWN_NW * 64) quant16_down_kernel(const Q16DownArgs p) {
  __shared__ float4 red[Q16_DOWN_NW * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int piece = blockIdx.x;
  q16_f32x4 tot = {0.f, 0.f, 0.f, 0.f};
  quant16_down<3>(p, piece, tot);
  quant16_down<8>(p, piece, tot);
  red[wave * 64 + lane] = make_float4(tot[0], tot[1], tot[2], tot[3]);
  __syncthreads();
  if (wave != 0) return;
  float4 t = red[lane];
#pragma unroll
  for (int w = 1; w < Q16_DOWN_NW; ++w) {
    const float4 o = red[w * 64 + lane];
    t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
  }
  float v[4] = {t.x, t.y, t.z, t.w};
  const float none[4] = {0.f, 0.f, 0.f, 0.f};
  sk_emit(p.e, piece >> 1, 16 * (piece & 1) + 4 * (lane >> 4), lane & 15, v, none);
}

}  // namespace

size_t skinny_part_bytes(int M) {
  // where a reduction is cut, at most ROWS16_WGS workgroups, one KiB each per block of 16 tokens
  return (size_t)ROWS16_WGS * 1024 * (M <= 16 ? 1 : M <= 32 ? 2 : 4);
}

static void fill_reduce_args(SkinnyReduceArgs& r, const GemmArgs& g, int act) {
  r.n_rb = g.N / 32; r.M = g.M; r.N = g.N;
  r.act = act; r.act_cols = g.act_cols; r.split_col = g.split_col;
  r.C0 = g.C0; r.C1 = g.C1; r.ldc0 = g.ldc0; r.ldc1 = g.ldc1;
  r.c0_tiled = g.c0_tiled; r.c1_tiled = g.c1_tiled; r.n_store = g.n_store;
  r.bias = g.bias; r.bias_cols = g.bias_cols; r.resid = g.resid; r.ldr = g.ldr; r.out_f32 = g.out_f32;
}

template <bool AT, int RB, int U, bool GLU, bool DUAL>
static int launch_rows16(const Rows16Args& a, hipStream_t st) {
  const dim3 grid(a.n_units * a.n_split), blk(ROWS16_NW * 64);
  const size_t lds = (size_t)ROWS16_NW * (GLU ? 2 : RB) * 1024;   // times the blocks of 16 tokens
  if (a.M <= 16) hipLaunchKernelGGL((rows16_kernel<AT, 1, RB, ROWS16_NW, U, GLU, DUAL>), grid, blk, lds, st, a);
  else if (a.M <= 32) hipLaunchKernelGGL((rows16_kernel<AT, 2, RB, ROWS16_NW, U, GLU, DUAL>), grid, blk, 2 * lds, st, a);
  else hipLaunchKernelGGL((rows16_kernel<AT, 4, RB, ROWS16_NW, 4, GLU, DUAL>), grid, blk, 4 * lds, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// g as for the large-batch launcher (destinations tiled or row-major).
int launch_skinny_bf16(const GemmArgs& g, int act, float* part, unsigned* counters, int n_clear, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0) return 0;
  if (g.M > SKINNY_MAX_M || (g.N & 31) || g.partial) return -1;
  const bool glu = act == ACT_GLU && g.act_cols > 0, dual = g.A1 != nullptr, at = g.a_tiled != 0;
  // (a gated product reads the caller's row-major tokens, or two tiled left operands)
  if ((dual && (!at || !glu || g.act_cols != g.N)) || (glu && ((g.act_cols & 63) || at != dual))) return -1;
  Rows16Args a = {};
  a.A = g.A; a.A1 = g.A1; a.Bt = g.Bt; a.lda = g.lda; a.ldb = g.ldb;
  a.M = g.M; a.K = g.K; a.steps = (g.K + 31) / 32;
  fill_reduce_args(a.e, g, act);
  a.part = part; a.counters = counters;
  a.clear = counters; a.n_clear = n_clear;
  a.pair_units = glu ? g.act_cols / 32 : 0;
  const int blocks = (g.N - (glu ? g.act_cols : 0)) / 32;
  // Units of 16 rows while all their workgroups find a CU of their own, else of 32 (which share the
  // activation loads): with 16 rows throughout the OPT-13B-sized layers take 2 % more, with 32 from
  // half as many units on the Llama-sized one 4 % more.  What is left of the machine is filled by
  // cutting the reduction, at least 32 steps a range; one and a quarter rounds of workgroups instead
  // of one take 2 % (Llama-sized) to 12 % (OPT-13B-sized) more.
  const bool one = a.pair_units + 2 * blocks <= ROWS16_WGS;
  a.n_units = a.pair_units + blocks * (one ? 2 : 1);
  a.n_split = 1;
  if (one && !glu && n_clear == 0 && counters != nullptr) {
    int S = ROWS16_WGS / a.n_units;
    if (S > a.steps / 32) S = a.steps / 32;
    if (S > ROWS16_MAX_SPLIT) S = ROWS16_MAX_SPLIT;
    a.n_split = S < 1 ? 1 : S;
  }
  if (dual) return launch_rows16<true, 2, 4, true, true>(a, st);
  if (at) {
    return one ? launch_rows16<true, 1, 6, false, false>(a, st) : launch_rows16<true, 2, 6, false, false>(a, st);
  }
  if (glu) return one ? launch_rows16<false, 1, 4, true, false>(a, st) : launch_rows16<false, 2, 6, true, false>(a, st);
  return one ? launch_rows16<false, 1, 8, false, false>(a, st) : launch_rows16<false, 2, 6, false, false>(a, st);
}

int launch_skinny_reduce(const GemmArgs& g, int act, const float* part, int n_split, int f16_out, hipStream_t st) {
  return launch_skinny_reduce2(g, act, part, n_split, g.N / 32, n_split, f16_out, st);
}

int launch_skinny_reduce2(const GemmArgs& g, int act, const float* part, int n_split, int rb_split, int n_split_b,
                          int f16_out, hipStream_t st) {
  SkinnyReduceArgs r = {};
  r.f16_out = f16_out; r.rb_split = rb_split; r.n_split_b = n_split_b;
  r.part = part; r.n_rb = g.N / 32; r.n_split = n_split; r.M = g.M; r.N = g.N;
  r.act = act; r.act_cols = g.act_cols; r.split_col = g.split_col;
  r.C0 = g.C0; r.C1 = g.C1; r.ldc0 = g.ldc0; r.ldc1 = g.ldc1;
  r.c0_tiled = g.c0_tiled; r.c1_tiled = g.c1_tiled; r.n_store = g.n_store;
  r.bias = g.bias; r.bias_cols = g.bias_cols; r.resid = g.resid; r.ldr = g.ldr; r.out_f32 = g.out_f32;
  hipLaunchKernelGGL(skinny_reduce_kernel, dim3(r.n_rb), dim3(256), 0, st, r);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Four groups a wavefront (d_model 4096) and with them one piece of outputs a CU; five and up to 320 pieces only for
// gated layers.  Both sides (us, four layers of 16 tokens, the kernels for 32 / these): 5120 x 13824 gated 241 /
// 203, 4608 x 12000 gated 203 / 185, 5120 x 20480 not gated 231 / 234.
// Long reductions are left to them too where few outputs make few workgroups of DOWN (their ranges fill the machine): both sides, 8
// tokens, not gated 128 x 13824 16.5 / 15.6, x 24576 19.9 / 22.8; 512 x 16384 18.7 / 17.5, x 32768 26.7 / 28.4; 1024 x 24576 27.9 /
// 24.5, x 49152 36.8 / 41.7; 2048 x 32768 37.6 / 35.6, x 49152 48.0 / 48.6; gated 128 x 16384 19.7 / 18.4, x 32768 28.2 / 30; 512 x
// 24576 28.4 / 24.9, x 49152 37.1 / 42.6; 1024 x 32768 36.9 / 33, x 49152 46.0 / 45.
bool quant16_fits(int M, int d_model, int neurons, bool gated) {
  if (M > 16 || d_model > 128 * Q16_NW * (gated ? Q16_MAX_GPW : Q16_MAX_GPW - 1)) return false;
  return neurons <= (gated ? 20480 + 24 * d_model : 14336 + 16 * d_model);
}

template <bool GLU>
static void launch_q16_up(const Q16UpArgs& a, hipStream_t st) {
  const dim3 grid(a.units8 + a.wgs3), blk(Q16_NW * 64);
  switch ((a.G + Q16_NW - 1) / Q16_NW) {
    case 1: hipLaunchKernelGGL((quant16_up_kernel<1, GLU>), grid, blk, 0, st, a); break;
    case 2: hipLaunchKernelGGL((quant16_up_kernel<2, GLU>), grid, blk, 0, st, a); break;
    case 3: hipLaunchKernelGGL((quant16_up_kernel<3, GLU>), grid, blk, 0, st, a); break;
    case 4: hipLaunchKernelGGL((quant16_up_kernel<4, GLU>), grid, blk, 0, st, a); break;
    default: hipLaunchKernelGGL((quant16_up_kernel<5, GLU>), grid, blk, 0, st, a); break;
  }
}

int launch_quant16_up(const GemmArgs& g, int act, const SkinnyQ& q8, int n8, const SkinnyQ& q3, int n3, hipStream_t st) {
  if (n8 + n3 <= 0) return 0;
  const bool glu = act == ACT_GLU;
  if (g.M <= 0 || !quant16_fits(g.M, g.K, (n8 + n3) / (glu ? 2 : 1), glu) || (g.K & 127) || (n8 & 63) || (n3 & 63)) return -1;
  Q16UpArgs a = {};
  a.X = g.A; a.lda = g.lda; a.M = g.M; a.G = g.K / 128;
  a.codes[0] = (const char*)q8.codes; a.codes[1] = (const char*)q3.codes;
  a.scales[0] = (const uint16_t*)q8.scales; a.scales[1] = (const uint16_t*)q3.scales;
  a.units8 = n8 / 32; a.units3 = n3 / 32; a.rb3 = n8 / 32;
  // One pair of 8-bit pieces a workgroup (2.7 times as long as a 3-bit one).  The 3-bit ones share what is left of one round of the
  // machine, unless a whole round for them behind the 8-bit ones is shorter: 16 tokens, left / whole round, gated 4096 x 24576 with a
  // tenth of 8 bits 56.7 / 44.3, not gated 4096 x 32768 49.0 / 45.4, 4096 x 24576 35.0 / 37.7.  Two workgroups of one group a
  // wavefront are resident a CU (110 registers; 512 x 8192: 12.6 -> 11.8), and more of equal length gain nothing there.
  const int round = a.G <= Q16_NW ? 512 : 256, left = round - a.units8;
  const int whole = (a.units3 + round - 1) / round, shared = left > 0 ? (a.units3 + left - 1) / left : a.units3;
  const bool behind = left <= 0 || shared > whole + 2.7;
  const int wgs = behind ? round : left, each = behind ? whole : shared;
  a.wgs3 = a.units3 < 1 ? 0 : round == 512 ? (a.units3 + each - 1) / each : a.units3 < wgs ? a.units3 : wgs;
  fill_reduce_args(a.e, g, act);
  a.e.f16_out = 1;
  if (glu) launch_q16_up<true>(a, st);
  else launch_q16_up<false>(a, st);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_quant16_down(const GemmArgs& g, const SkinnyQ& q8, const SkinnyQ& q3, hipStream_t st) {
  if (g.M <= 0 || g.M > 16 || (g.N & 127) || !g.a_tiled || (q8.Kp & 63) || (q3.Kp & 63)) return -1;
  Q16DownArgs a = {};
  a.H = g.A;
  a.codes[0] = (const char*)q8.codes; a.codes[1] = (const char*)q3.codes;
  a.scales[0] = (const uint16_t*)q8.scales; a.scales[1] = (const uint16_t*)q3.scales;
  a.Kp[0] = q8.Kp; a.Kp[1] = q3.Kp;
  fill_reduce_args(a.e, g, ACT_NONE);
  hipLaunchKernelGGL(quant16_down_kernel, dim3(g.N / 16), dim3(Q16_DOWN_NW * 64), 0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

constexpr int SKQ_MAX_SPLIT = 32;
size_t skinny_q_part_bytes(int n_max) {
  // two streamed segments per product, each at most SKQ_MAX_SPLIT ranges of one 4 KiB tile per row block
  return (size_t)2 * SKQ_MAX_SPLIT * ((n_max + 31) / 32) * 4096;
}

// kernel arguments and workgroup count of one part (0 workgroups if it is empty)
static int q_part_args(const GemmArgs& g, const SkinnyQ& q, float* part, int slot0, int rb_out0, int n_rb_part,
                       int max_wgs, SkinnyQArgs* out, int* wgs) {
  *wgs = 0;
  SkinnyQArgs a = {};
  *out = a;
  if (g.N <= 0 || g.K <= 0) return 0;
  if (g.M <= 0 || g.M > 32 || (g.K & 63) || (q.bits != 3 && q.bits != 8)) return -1;
  if ((q.down != 0) != (g.a_tiled != 0) || (!q.down && (g.K & 127))) return -1;
  const int rbs = skq_rb(q.bits, q.down != 0);
  if (g.N % (32 * rbs)) return -1;
  a.A = g.A; a.lda = g.lda; a.M = g.M;
  a.n_rb = g.N / 32;
  const int n_rbg = a.n_rb / rbs;
  const int ub = q.down ? 1 : 2;
  a.nu_total = g.K / (64 * ub);
  // ranges: about 512 workgroups, at least two units per wavefront, and partial tiles (4 KiB
  // per row block and range) of at most half of the packed weights' bytes
  const size_t wbytes = (size_t)a.n_rb * (g.K / 64) * qblock_bytes(q.bits);
  int S = (512 + n_rbg - 1) / n_rbg;
  if (S > a.nu_total / 8) S = a.nu_total / 8;
  const int cap = (int)(wbytes / ((size_t)8192 * a.n_rb));
  if (S > cap) S = cap;
  if (S > SKQ_MAX_SPLIT) S = SKQ_MAX_SPLIT;
  if (S > max_wgs / n_rbg) S = max_wgs / n_rbg;
  if (S < 1) S = 1;
  a.nu_per = (a.nu_total + S - 1) / S;
  a.n_split = (a.nu_total + a.nu_per - 1) / a.nu_per;
  a.slot0 = slot0; a.rb_out0 = rb_out0; a.n_rb_part = n_rb_part;
  a.codes = (const char*)q.codes; a.scales = (const uint16_t*)q.scales; a.G = q.G; a.Kp = q.Kp;
  a.part = part;
  *out = a;
  *wgs = n_rbg * a.n_split;
  return 0;
}

int launch_skinny_q_pair(const GemmArgs& g8, const SkinnyQ& q8, const GemmArgs& g3, const SkinnyQ& q3, float* part,
                         int n_split[2], hipStream_t st) {
  n_split[0] = n_split[1] = 0;
  const bool down = (g8.N > 0 && g8.K > 0) ? q8.down != 0 : q3.down != 0;
  SkinnyQ2Args a = {};
  int w8 = 0, w3 = 0;
  // The kernels hold three workgroups per CU: the 3-bit part takes its ranges first, the 8-bit
  // part what is left of one full round (768 workgroups), so that no second round starts for a
  // few workgroups.
  constexpr int ROUND = 768;
  if (down) {
    // same rows, two segments of the reduction: the 3-bit ranges follow the 8-bit ones
    const int n_rb = (g8.N > 0 ? g8.N : g3.N) / 32;
    if (q_part_args(g3, q3, part, 0, 0, n_rb, ROUND, &a.s3, &w3)) return -1;
    if (q_part_args(g8, q8, part, 0, 0, n_rb, ROUND - w3, &a.s8, &w8)) return -1;
    a.s3.slot0 = a.s8.n_split;
  } else {
    // two row ranges of one output: the 3-bit rows follow the 8-bit rows
    const int n_rb = (g8.N > 0 ? g8.N / 32 : 0) + (g3.N > 0 ? g3.N / 32 : 0);
    if (q_part_args(g3, q3, part, 0, g8.N > 0 ? g8.N / 32 : 0, n_rb, ROUND, &a.s3, &w3)) return -1;
    if (q_part_args(g8, q8, part, 0, 0, n_rb, ROUND - w3, &a.s8, &w8)) return -1;
  }
  if (w8 + w3 == 0) return 0;
  a.wg8 = w8;
  // LDS: the four wavefronts' accumulators of the row blocks, [4][RB][16][64] floats
  constexpr int rb_dn = skq_rb(3, true) > skq_rb(8, true) ? skq_rb(3, true) : skq_rb(8, true);
  constexpr int rb_up = skq_rb(3, false) > skq_rb(8, false) ? skq_rb(3, false) : skq_rb(8, false);
  if (down) hipLaunchKernelGGL(skinny_stream_q2_kernel<true>, dim3(w8 + w3), dim3(256), 4 * rb_dn * 4096, st, a);
  else hipLaunchKernelGGL(skinny_stream_q2_kernel<false>, dim3(w8 + w3), dim3(256), 4 * rb_up * 4096, st, a);
  if (hipGetLastError() != hipSuccess) return -1;
  n_split[0] = a.s8.n_split; n_split[1] = a.s3.n_split;
  return 0;
}

}  // namespace ffsplit
