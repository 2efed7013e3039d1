// bf16 GEMM for the backbone projections on gfx950 matrix cores.
//
//   C[M][N] (+)= epi( X[M][K] * W[N][K]^T )     X = activations, W = weights
//
// MFMA: v_mfma_f32_16x16x32_bf16.  The weight tile is the MFMA "A" operand
// and the token tile the "B" operand: lane l holds 8 consecutive K values of
// weight row l & 15 and of token row l & 15, K block 8 * (l >> 4), and ends
// with 4 consecutive output columns 4 * (l >> 4) .. +3 of token row l & 15,
// so the epilogue writes 8-byte (bf16) / 16-byte (fp32) vectors along the
// row-major output.  Measured on the 2048-wide shapes the 16x16x32 form runs
// 3-10% faster than 32x32x16 with the same operand traffic (the chip is
// power-limited and this form needs less energy per flop); a K=64 slab is two
// K=32 steps.  Every loop below issues, per output element, the same MFMA
// sequence (slab order, K=32 steps in order, the same lane layout), so all
// tile shapes and loops give identical bits.
//
// Operand staging: global_load_lds_dwordx4 moves 16-byte chunks straight from
// global memory into LDS (no register staging).  K advances 64 per slab (one
// 128-byte segment of every operand row).  Chunk c of LDS row r sits at
// position c ^ swz(r), swz(r) = (r >> 1) & 7: two 128-byte rows share a
// 256-byte bank row, and every 16-lane phase of a fragment read (16
// consecutive rows, one chunk) covers all 64 banks.  Each DMA instruction
// fills 1 KB = 8 rows; the lane -> source-chunk assignment applies the
// swizzle.
//
// Loops: the 256x256 tile (4 wavefronts, one per SIMD) runs a ring-buffered
// loop (ring_run); smaller tiles, of short launches, last partly filled waves
// and small grouped problems, run flex_tile.  gemm_plan picks shapes and K
// splits by an estimated time.
//
// Launch order of the ring launches: tiles are walked in groups of 32
// token-tiles (token tile fastest).  Workgroups are dealt round-robin to the 8 XCDs, so the 32 tiles
// an XCD holds at a time form a block of 4 token tiles x 8 weight tiles, and
// every weight slab is requested by all XCDs at about the same time.
// Measured in the step on the 2048-wide workload: groups of 32 give 290.1 ms
// per step against 292.9 (16), 298.7 (8), 292.0 (64) and 300.6 (128); an
// explicit XCD remap giving each XCD a contiguous block of tiles was no
// faster with 4x8 blocks and 13% slower with 16x2 (32x32x16 loop).
//
// Epilogues: bf16 store, GELU -> bf16, fp32 residual add (in place), fp32
// store, GELU with fp32 pre-activation save, GELU' product, and GeGLU, whose
// gate and up weight rows are interleaved in 16-row blocks as they are
// loaded, so the gate and up accumulators of an output column land in the
// same lane.
#include <algorithm>
#include <type_traits>

#include "jn_device.h"
#include "jn_internal.h"

namespace jnx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

#define JN_GPTR(p) ((__attribute__((address_space(1))) void*)(p))
#define JN_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int kBK = 64;       // K per slab (128-byte rows)
constexpr int kGroupM = 32;   // token tiles per L2 group

__device__ __forceinline__ int lds_swz(int r) { return (r >> 1) & 7; }

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// s_waitcnt with only the LDS / scalar-memory counter constrained.
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  static_assert(N >= 0 && N < 16, "lgkmcnt range");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (N << 8));
}

// T fragments of 16 rows each (rows row0, row0 + 16, ...), chunk position pos.
template <int T>
__device__ __forceinline__ void gemm_frags(bf16x8 (&f)[T], const uint16_t* stage, int row0, int pos) {
#pragma unroll
  for (int i = 0; i < T; ++i) f[i] = *reinterpret_cast<const bf16x8*>(stage + (row0 + i * 16) * kBK + pos * 8);
}

// Source row of weight-tile row r: plain, or for GeGLU the gate / up rows
// interleaved in 16-row blocks (block 2b = gate columns 16b.., 2b+1 = up).
template <bool GLU>
__device__ __forceinline__ const uint16_t* weight_row(const uint16_t* W, const uint16_t* W2, int64_t ldw, int32_t tn,
                                                      int BN, int r, int32_t N) {
  if constexpr (GLU) {
    const int32_t col = min(tn * (BN / 2) + (r >> 5) * 16 + (r & 15), N - 1);
    return (((r >> 4) & 1) ? W2 : W) + (int64_t)col * ldw;
  } else {
    return W + (int64_t)min(tn * BN + r, N - 1) * ldw;
  }
}

// Two floats -> two bf16 (round to nearest even) by one v_cvt_pk_bf16_f32;
// pack_bf2 converts each value alone and merges them with a shift and an
// OR.  Same bits.  Used in the GeGLU epilogue only: in the QKV kernel's staged
// epilogue the packed form changed the register allocation of the main loop
// (operand fragments moved through the accumulation registers, 16% slower).
typedef float gemm_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 gemm_bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf2_cvt(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(gemm_f32x2{lo, hi}, gemm_bf16x2));
}

// Largest divisor of `rows` that is at most `most`.
constexpr int row_batch(int rows, int most) {
  int b = most < rows ? most : rows;
  while (rows % b != 0) --b;
  return b;
}

// Position of tile pid in the grouped walk (kGroupM token tiles per group).
__device__ __forceinline__ void tile_of(int32_t pid, int32_t tiles_m, int32_t tiles_n, int32_t& tm, int32_t& tn) {
  const int32_t per_group = kGroupM * tiles_n;
  const int32_t first_m = (pid / per_group) * kGroupM;
  const int32_t gsize = min(tiles_m - first_m, kGroupM);
  tm = first_m + (pid % per_group) % gsize;
  tn = (pid % per_group) / gsize;
}

// Sum of the split-K partials in range order, then the epilogue.  Thread =
// 4 consecutive output columns of one row.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int32_t S,
                                                            int64_t stride, int32_t M, int32_t N,
                                                            void* __restrict__ C, int64_t ldc) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int32_t q = N / 4;
  if (e >= (int64_t)M * q) return;
  const int32_t m = (int32_t)(e / q), n = (int32_t)(e % q) * 4;
  float4 acc = *reinterpret_cast<const float4*>(part + (int64_t)m * N + n);
  for (int32_t s = 1; s < S; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(part + s * stride + (int64_t)m * N + n);
    acc.x += v.x;
    acc.y += v.y;
    acc.z += v.z;
    acc.w += v.w;
  }
  if constexpr (EPI == EPI_RESID_F32) {
    float4* p = reinterpret_cast<float4*>(reinterpret_cast<float*>(C) + (int64_t)m * ldc + n);
    float4 o = *p;
    o.x += acc.x;
    o.y += acc.y;
    o.z += acc.z;
    o.w += acc.w;
    *p = o;
  } else {
    if constexpr (EPI == EPI_GELU_BF16) {
      acc.x = gelu_fast_f(acc.x);
      acc.y = gelu_fast_f(acc.y);
      acc.z = gelu_fast_f(acc.z);
      acc.w = gelu_fast_f(acc.w);
    }
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(C) + (int64_t)m * ldc + n) =
        make_uint2(pack_bf2(acc.x, acc.y), pack_bf2(acc.z, acc.w));
  }
}

// Epilogues of both loops.  acc[i][j] covers weight rows 16 i .. and tokens
// 16 j .. of the wave's part (first token m0, first output column n0); lane l
// owns columns 16 i + 4 (l >> 4) .. +3 of token 16 j + (l & 15).  Each wave
// turns its part around in LDS of its own (`stage`, no barriers), 16-byte
// chunks at position chunk ^ f(row) so that writes and reads cover all banks,
// and then touches global memory in whole row segments (128 to 512 contiguous
// bytes per row and instruction; straight from the MFMA layout an instruction
// touches 64 bytes, or in bf16 32, of 16 rows).  A wave whose part lies inside
// the output takes a path without lane masks: a mask per store is a branch, and
// each then waits for its own LDS read.
//
// Results of 16 bits (bf16, GELU, GeGLU): converted by v_cvt_pk_bf16_f32 on the
// way into LDS; batches of 16-token blocks that fit 8 KB.  The others pass
// through as fp32, one 16-token block at a time, and the fp32 rows they read
// (residual, saved pre-activation) are requested AHEAD blocks in advance.
// 256x256 tiles of 65,536 tokens x 3,072 columns, K = 768, before (direct
// stores, masks; bf16 staged behind barriers) and now: bf16 311 -> 264 us, GELU
// 356 -> 320, GeGLU 281 -> 262, residual add 523 -> 461; 72 tiles (the chip
// mostly idle): 21.1 -> 19.8, 25.3 -> 23.9, 21.4 -> 20.4 and 33.7 -> 24.0 us.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr bool epi_bf16(int epi) { return epi == EPI_BF16 || epi == EPI_GELU_BF16 || epi == EPI_GEGLU_BF16; }
constexpr bool epi_reads(int epi) { return epi == EPI_RESID_F32 || epi == EPI_GELUGRAD_BF16; }

// Sizes of the 16-bit epilogue of a wave's part.
template <int EPI, int TN, int TM>
struct Epi16 {
  static constexpr bool GLU = EPI == EPI_GEGLU_BF16;
  static constexpr int WC = GLU ? 8 * TN : 16 * TN;           // output columns per wave
  static constexpr int CH = WC / 8, RI = 64 / CH;             // 16-byte chunks per row, rows per instruction
  static constexpr int NB = row_batch(TM, 4096 / (16 * WC));  // 16-token blocks per batch
  static constexpr int NI = (NB * 16 + RI - 1) / RI;          // instructions per batch (the last of 16-column parts half used)
  static constexpr int STORES = TM / NB * NI;                 // of a whole part, one per instruction
  static_assert((CH & (CH - 1)) == 0 && CH <= 16 && TM % NB == 0, "row segments");
};

template <int EPI, int TN, int TM, bool WHOLE>
__device__ __forceinline__ void epilogue_bf16(const GemmArgs& g, const f32x4 (&acc)[TN][TM], uint16_t* stage,
                                              int32_t m0, int32_t n0, int lane) {
  using E = Epi16<EPI, TN, TM>;
  constexpr bool GLU = E::GLU;
  constexpr int WC = E::WC, CH = E::CH, RI = E::RI, NB = E::NB, NI = E::NI;
  const int quad = lane >> 4, row = lane & 15, c = lane & (CH - 1), rr = lane / CH;
  const int32_t m = m0 + rr, n = n0 + c * 8;
  uint16_t* C = reinterpret_cast<uint16_t*>(g.C) + (int64_t)m * g.ldc + n;
  const int64_t step = RI * g.ldc;
  auto swz = [](int r) { return CH == 16 ? r & 15 : (r / (16 / CH)) & (CH - 1); };
  auto put = [&](int j) __attribute__((always_inline)) {  // blocks j .. j + NB - 1
#pragma unroll
    for (int jj = 0; jj < NB; ++jj) {
#pragma unroll
      for (int i = 0; i < TN; i += GLU ? 2 : 1) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = acc[i][j + jj][e];
          v[e] = GLU ? gelu_fast_f(a) * acc[i + (GLU ? 1 : 0)][j + jj][e] : EPI == EPI_GELU_BF16 ? gelu_fast_f(a) : a;
        }
        const int chunk = 2 * (GLU ? i / 2 : i) + (quad >> 1);
        *reinterpret_cast<u32x2*>(stage + (16 * jj + row) * WC + (chunk ^ swz(row)) * 8 + (quad & 1) * 4) =
            u32x2{pack_bf2_cvt(v[0], v[1]), pack_bf2_cvt(v[2], v[3])};
      }
    }
  };
  u32x4 v[NI];
  put(0);
#pragma unroll
  for (int j = 0; j < TM; j += NB) {
#pragma unroll
    for (int it = 0; it < NI; ++it)
      v[it] = *reinterpret_cast<const u32x4*>(stage + (RI * it + rr) * WC + (c ^ swz((RI * it + rr) & 15)) * 8);
    if (j + NB < TM) put(j + NB);  // (a wave's LDS operations stay in order)
#pragma unroll
    for (int it = 0; it < NI; ++it)
      if ((NB * 16 % RI == 0 || RI * it + rr < NB * 16) && (WHOLE || (m + 16 * j + RI * it < g.M && n < g.N)))
        *reinterpret_cast<u32x4*>(C + it * step) = v[it];
    C += NB * 16 * g.ldc;
  }
}

template <int EPI, int TN, int TM, bool WHOLE, bool ONCE>
__device__ __forceinline__ void epilogue_f32(const GemmArgs& g, const f32x4 (&acc)[TN][TM], float* stage, int32_t m0,
                                             int32_t n0, int lane) {
  constexpr int WC = 16 * TN, CH = 4 * TN, RI = 64 / CH, NI = TN;  // as above; NI per block
  constexpr bool READS = epi_reads(EPI);
  constexpr int AHEAD = TM < 3 ? TM : 3;
  static_assert((CH & (CH - 1)) == 0 && RI >= 2, "row segments");
  const int quad = lane >> 4, row = lane & 15, c = lane & (CH - 1), rr = lane / CH;
  const int32_t m = m0 + rr, n = n0 + c * 4;
  const float* src = g.aux;  // a residual add without aux is in place
  int64_t ldr = g.ldaux;
  if (EPI == EPI_RESID_F32 && !src) {
    src = reinterpret_cast<const float*>(g.C);
    ldr = g.ldc;
  }
  const float* R = READS ? src + (int64_t)m * ldr + n : nullptr;
  f32x4 r[READS ? AHEAD : 1][NI];
  auto fetch = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      if constexpr (WHOLE)
        r[j % AHEAD][it] = *reinterpret_cast<const f32x4*>(R + it * RI * ldr);
      else  // lanes outside the output read its last row or column block
        r[j % AHEAD][it] = *reinterpret_cast<const f32x4*>(src + (int64_t)min(m + 16 * j + RI * it, g.M - 1) * ldr +
                                                           min(n, g.N - 4));
    }
    R += 16 * ldr;
  };
  if constexpr (READS) {
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) fetch(j);
  }
  const int64_t base = (int64_t)m * g.ldc + n, step = RI * g.ldc;
#pragma unroll
  for (int j = 0; j < TM; ++j) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
      *reinterpret_cast<f32x4*>(stage + row * WC + ((4 * i + quad) ^ (row & (CH - 1))) * 4) = acc[i][j];
    f32x4 v[NI];
#pragma unroll
    for (int it = 0; it < NI; ++it)
      v[it] = *reinterpret_cast<const f32x4*>(stage + (RI * it + rr) * WC + (c ^ ((RI * it + rr) & (CH - 1))) * 4);
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      if (!WHOLE && !(m + 16 * j + RI * it < g.M && n < g.N)) continue;
      const int64_t at = base + 16 * j * g.ldc + it * step;
      const f32x4 a = v[it];
      if constexpr (EPI == EPI_F32 || EPI == EPI_RESID_F32) {
        f32x4* const p = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + at);
        if constexpr (ONCE)
          __builtin_nontemporal_store(a, p);
        else
          *p = READS ? r[j % AHEAD][it] + a : a;
      } else {
        float y[4];
        if constexpr (EPI == EPI_GELU_SAVE) {
          *reinterpret_cast<f32x4*>(g.aux + (int64_t)(m + 16 * j + RI * it) * g.ldaux + n) = a;
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = gelu_exact_f(a[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = a[e] * gelu_grad_fast_f(r[j % AHEAD][it][e]);
        }
        *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(g.C) + at) =
            u32x2{pack_bf2_cvt(y[0], y[1]), pack_bf2_cvt(y[2], y[3])};
      }
    }
    if constexpr (READS)
      if (j + AHEAD < TM) fetch(j + AHEAD);
  }
}

// stage: 8 KB of the wave's own.  Returns whether the part lay inside the
// output.  ONCE: fp32 results that no kernel reads next (weight gradients), stored
// non-temporally so that the caches keep what the next launches read (16
// tenants' GELU' data gradient after them 216 -> 202 us).
template <int EPI, int TN, int TM, bool ONCE = false>
__device__ __forceinline__ bool gemm_epilogue(const GemmArgs& g, const f32x4 (&acc)[TN][TM], uint16_t* stage,
                                              int32_t m0, int32_t n0, int lane) {
  const bool whole = m0 + 16 * TM <= g.M && n0 + (EPI == EPI_GEGLU_BF16 ? 8 : 16) * TN <= g.N;
  asm volatile("" : "+v"(lane));  // lane offsets are formed here, not held in registers through a loop over tiles
  if constexpr (epi_bf16(EPI)) {
    if (whole)
      epilogue_bf16<EPI, TN, TM, true>(g, acc, stage, m0, n0, lane);
    else
      epilogue_bf16<EPI, TN, TM, false>(g, acc, stage, m0, n0, lane);
  } else {
    if (whole)
      epilogue_f32<EPI, TN, TM, true, ONCE>(g, acc, reinterpret_cast<float*>(stage), m0, n0, lane);
    else
      epilogue_f32<EPI, TN, TM, false, ONCE>(g, acc, reinterpret_cast<float*>(stage), m0, n0, lane);
  }
  wait_lgkmcnt<0>();  // the stage is read before anything else is written there
  __builtin_amdgcn_sched_barrier(0);
  return whole;
}

// Buffer resource of a row-major bf16 panel starting at `base`, `bytes` long
// (loads past the end return zero).  Word 3 is the CDNA raw-buffer format.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel_rsrc(const uint16_t* base, int64_t bytes) {
  const int32_t n = (int32_t)min(bytes, (int64_t)0x7fffffff);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), (short)0, n, 0x00020000);
}

// Chunk position swizzle of k-line k of a transposed operand's half-slab
// (32 chunks of 16 bytes per line): the 16 k-lines one ds_read_b64_tr_b16
// touches (8 per half-wave, 2 chunks each) cover every LDS bank once per
// half-wave (checked with a bank model on the CPU).
__device__ __forceinline__ int tswz(int k) { return 2 * ((k & 3) | ((k & 8) >> 1)); }

// Tiles of short, ragged and grouped launches: BN weight rows x BM tokens on
// 4 wavefronts (2 x 2), LDS stages of one K=64 slab each: NS for the tokens,
// NSW (NS or NS - 1) for the weights.  Between two barriers every wave issues
// 2 TN TM MFMAs (the second K=32 half of slab kt, then the first half of slab
// kt+1), the next half's fragment reads under them, and the DMA of one slab
// spread evenly over the window, the weights under the first half and the
// tokens under the second: a DMA instruction occupies the CU's load path for
// ~16 cycles per KB, so a burst of them after the barrier stalls the wave's
// MFMA issue.  With all operands in the L2 the
// 256x160 tile takes 0.67 us per slab (2.0 PFLOP/s over 256 CUs), 128x128
// 0.32 us, 64x96 0.20 us; the interleaved 128x128 loop it replaced issued a
// slab's DMA in one burst and took 0.77 us per slab of the one-sample QKV
// projection.  300 tokens, 2048-wide, before and after: QKV 24.3 -> 17.1 us
// (128x96), O 15.7 -> 13.3 (64x96), GeGLU 57.5 -> 43.5 (256x160: 256 tiles, 320
// instead of 512 padded rows), down 51.2 -> 33.8 (128x160, K split 8 ways).
// More stages measured no faster.  Rows past M and N are fetched as
// zeros without touching memory (lane offsets past the buffer range).
//
// TR as in ring_run below; a transposed operand's tile side is a multiple of
// 128 (its 64 k-lines hold BN or BM elements, swizzled by tswz).
// [kt0, kt1): the K slabs summed.  WIDE: the row offsets inside a panel may
// exceed 32 bits (leading dimensions beyond 4M elements), so every DMA
// instruction's 8 rows get a buffer base of their own.
template <int BN, int BM, int NS, int NSW, int EPI, int TR, bool WIDE = false>
__device__ __forceinline__ void flex_tile(const GemmArgs& g, int32_t tm, int32_t tn, int32_t kt0, int32_t kt1,
                                          uint16_t* __restrict__ lds) {
  constexpr bool TX = (TR & GEMM_TRANS_X) != 0, TW = (TR & GEMM_TRANS_W) != 0;
  constexpr bool GLU = EPI == EPI_GEGLU_BF16;
  constexpr int WGN = 2, WGM = 2, NWV = WGN * WGM;
  constexpr int WN = BN / WGN, WM = BM / WGM;
  constexpr int TN = WN / 16, TM = WM / 16;
  constexpr int NW = BN / (8 * NWV), NX = BM / (8 * NWV);  // 1 KB DMA instructions per wave per slab
  constexpr int SLW = BN * kBK, SLX = BM * kBK;            // elements per stage
  static_assert(BN % 32 == 0 && BM % 32 == 0 && NS >= 3 && (NSW == NS || NSW == NS - 1), "tile shape");
  static_assert(!WIDE || (TR == 0 && !GLU), "wide rows");
  static_assert((!TX || BM % 128 == 0) && (!TW || BN % 128 == 0) && !(GLU && (TR || TN % 2)), "operand layout");
  const int32_t M = g.M, N = g.N;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave / WGM, wm = wave % WGM;
  const int32_t m0 = tm * BM, c0 = GLU ? tn * (BN / 2) : tn * BN;
  const int KT = kt1 - kt0;
  // operand panels from slab kt0 on; a row-major panel's lanes past the last
  // row carry an offset past its range, a transposed one's range ends with K
  constexpr uint32_t kPast = 0x80000000u;
  const int64_t k0 = (int64_t)kt0 * kBK;
  const uint16_t* const xb = TX ? g.X + k0 * g.ldx + m0 : g.X + (int64_t)m0 * g.ldx + k0;
  const uint16_t* const wb = TW ? g.W + k0 * g.ldw + c0 : g.W + (int64_t)c0 * g.ldw + k0;
  const uint16_t* const wb2 = GLU ? g.W2 + (int64_t)c0 * g.ldw + k0 : wb;
  const __amdgpu_buffer_rsrc_t xr = panel_rsrc(xb, TX ? ((g.K - k0) * g.ldx - m0) * 2 : (int64_t)0x7fffffff);
  const __amdgpu_buffer_rsrc_t wr = panel_rsrc(wb, TW ? ((g.K - k0) * g.ldw - c0) * 2 : (int64_t)0x7fffffff);
  const __amdgpu_buffer_rsrc_t wr2 = panel_rsrc(wb2, (int64_t)0x7fffffff);
  uint32_t xo[NX], wo[NW];
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    if constexpr (TX) {
      constexpr int LPL = BM / 8;  // lanes per k-line
      const int kl = (wave * NX + i) * (64 / LPL) + lane / LPL;
      xo[i] = (uint32_t)(((int64_t)kl * g.ldx + ((lane % LPL) ^ tswz(kl)) * 8) * 2);
    } else {
      const int r = (BM / NWV) * wave + 8 * i + (lane >> 3);
      const int64_t row = WIDE ? lane >> 3 : r;
      xo[i] = m0 + r < M ? (uint32_t)((row * g.ldx + ((lane & 7) ^ lds_swz(r)) * 8) * 2) : kPast;
    }
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if constexpr (TW) {
      constexpr int LPL = BN / 8;
      const int kl = (wave * NW + i) * (64 / LPL) + lane / LPL;
      wo[i] = (uint32_t)(((int64_t)kl * g.ldw + ((lane % LPL) ^ tswz(kl)) * 8) * 2);
    } else {
      const int r = (BN / NWV) * wave + 8 * i + (lane >> 3);
      const int32_t col = GLU ? c0 + (r >> 5) * 16 + (r & 15) : c0 + r;
      const int64_t row = WIDE ? lane >> 3 : col - c0;
      wo[i] = col < N ? (uint32_t)((row * g.ldw + ((lane & 7) ^ lds_swz(r)) * 8) * 2) : kPast;
    }
  }
  const int32_t xso = TX ? (int32_t)(kBK * 2 * g.ldx) : kBK * 2;  // byte step between slabs
  const int32_t wso = TW ? (int32_t)(kBK * 2 * g.ldw) : kBK * 2;
  uint16_t* const wl = lds;
  uint16_t* const xl = lds + NSW * SLW;
  const int dw = wave * NW * 512, dx = wave * NX * 512;
  // DMA d of slab `slab` into stage `st` (16-byte DMA to LDS does not exist
  // for the host pass)
#ifndef __HIP_DEVICE_COMPILE__
#define JN_FLEX_DMA_X(d, slab, st) (void)(d)
#define JN_FLEX_DMA_W(d, slab, st) (void)(d)
#else
#define JN_FLEX_DMA_X(d, slab, st)                                                                                    \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                                           \
      WIDE ? panel_rsrc(xb + (int64_t)((BM / NWV) * wave + 8 * (d)) * g.ldx, 0x7fffffff) : xr,                        \
      JN_LPTR(xl + (st) * SLX + dx + (d) * 512), 16, TX ? xo[d] + (uint32_t)((slab) * xso) : xo[d],                   \
      TX ? 0 : (slab) * xso, 0, 0)
#define JN_FLEX_DMA_W(d, slab, st)                                                                                    \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                                           \
      WIDE ? panel_rsrc(wb + (int64_t)((BN / NWV) * wave + 8 * (d)) * g.ldw, 0x7fffffff)                              \
           : (GLU && ((((BN / NWV) * wave + 8 * (d)) >> 4) & 1)) ? wr2 : wr,                                          \
      JN_LPTR(wl + (st) * SLW + dw + (d) * 512), 16, TW ? wo[d] + (uint32_t)((slab) * wso) : wo[d],                   \
      TW ? 0 : (slab) * wso, 0, 0)
#endif

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int sw = lds_swz(lane & 15), quad = lane >> 4;
  const int wrow = wn * WN + (lane & 15), xrow = wm * WM + (lane & 15);
  // transposed reads as in ring_run, for k-lines of BN / BM elements
  const int te = (lane & 15) >> 2, tc = lane & 3;
  const int tsub = 8 * (tc >> 1) + 4 * (tc & 1) + 16 * ((te & 3) | ((quad & 1) << 2));
  auto frag_w = [&](const uint16_t* slot, int f, int h) -> bf16x8 {
    if constexpr (TW) {
      const uint16_t* p = slot + (32 * h + 8 * quad + te) * BN + (tsub ^ (16 * (wn * TN + f)));
      const bf16x4 lo = __builtin_bit_cast(bf16x4, lds_read_tr_b16<0>(p));
      const bf16x4 hi = __builtin_bit_cast(bf16x4, lds_read_tr_b16<8 * BN>(p));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      return *reinterpret_cast<const bf16x8*>(slot + (wrow + 16 * f) * kBK + ((4 * h + quad) ^ sw) * 8);
    }
  };
  auto frag_x = [&](const uint16_t* slot, int f, int h) -> bf16x8 {
    if constexpr (TX) {
      const uint16_t* p = slot + (32 * h + 8 * quad + te) * BM + (tsub ^ (16 * (wm * TM + f)));
      const bf16x4 lo = __builtin_bit_cast(bf16x4, lds_read_tr_b16<0>(p));
      const bf16x4 hi = __builtin_bit_cast(bf16x4, lds_read_tr_b16<8 * BM>(p));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      return *reinterpret_cast<const bf16x8*>(slot + (xrow + 16 * f) * kBK + ((4 * h + quad) ^ sw) * 8);
    }
  };

  constexpr int Q = TN * TM, F = TN + TM, D = NW + NX;
  constexpr int FP = (F + Q - 1) / Q, FS = Q / F > 0 ? Q / F : 1;  // fragment reads per MFMA, MFMAs per read
  // Weight slab kt+NSW is requested in phase 1 of iteration kt and token slab
  // kt+NS-1 in its phase 0; the first slabs in the same order, so that the
  // counted waits below hold from the first iteration on.
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int sl = min(s, KT - 1);
    if (NSW < NS && s < NS - 1) {
#pragma unroll
      for (int d = 0; d < NX; ++d) JN_FLEX_DMA_X(d, sl, s);
    }
    if (s < NSW) {
#pragma unroll
      for (int d = 0; d < NW; ++d) JN_FLEX_DMA_W(d, sl, s);
    }
    if (NSW == NS && s < NS - 1) {
#pragma unroll
      for (int d = 0; d < NX; ++d) JN_FLEX_DMA_X(d, sl, s);
    }
  }
  wait_vmcnt<(NS - 2) * D + (NSW == NS ? NW : 0)>();  // slab 0 landed
  __builtin_amdgcn_s_barrier();
  bf16x8 fa[F], fb[F];  // first-half / second-half fragments: weights, then tokens
#pragma unroll
  for (int i = 0; i < TN; ++i) fa[i] = frag_w(wl, i, 0);
#pragma unroll
  for (int j = 0; j < TM; ++j) fa[TN + j] = frag_x(xl, j, 0);
  wait_lgkmcnt<0>();
  int sx = 0, sv = 0;  // kt % NS, kt % NSW
  for (int kt = 0; kt < KT; ++kt) {
    const int nxt = sx + 1 == NS ? 0 : sx + 1, prv = sx == 0 ? NS - 1 : sx - 1, nxv = sv + 1 == NSW ? 0 : sv + 1;
    // past the last slab the DMAs repeat it into a free stage (no branches)
    const int f0 = min(kt - 1 + NS, KT - 1), f1 = min(kt + NSW, KT - 1);
    {
      const uint16_t *cw = wl + sv * SLW, *cx = xl + sx * SLX;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int i = q / TM, j = q % TM;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fa[TN + j], acc[i][j], 0, 0, 0);
        if (q % FS == 0) {
#pragma unroll
          for (int e = 0; e < FP; ++e) {
            const int f = (q / FS) * FP + e;
            if (f < TN)
              fb[f] = frag_w(cw, f, 1);
            else if (f < F)
              fb[f] = frag_x(cx, f - TN, 1);
          }
        }
#pragma unroll
        for (int d = 0; d < NX; ++d)
          if ((2 * d + 1) * Q / (2 * NX) == q) JN_FLEX_DMA_X(d, f0, prv);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wait_lgkmcnt<0>();
    wait_vmcnt<(NS - 2) * NX + (NSW - 2) * NW>();  // slab kt+1 landed
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    {
      const uint16_t *nw = wl + nxv * SLW, *nx = xl + nxt * SLX;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int i = q / TM, j = q % TM;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[i], fb[TN + j], acc[i][j], 0, 0, 0);
        if (q % FS == 0) {
#pragma unroll
          for (int e = 0; e < FP; ++e) {
            const int f = (q / FS) * FP + e;
            if (f < TN)
              fa[f] = frag_w(nw, f, 0);
            else if (f < F)
              fa[f] = frag_x(nx, f - TN, 0);
          }
        }
#pragma unroll
        for (int d = 0; d < NW; ++d)
          if ((2 * d + 1) * Q / (2 * NW) == q) JN_FLEX_DMA_W(d, f1, sv);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wait_lgkmcnt<0>();
    sx = nxt;
    sv = nxv;
  }
#undef JN_FLEX_DMA_X
#undef JN_FLEX_DMA_W
  wait_vmcnt<0>();  // the repeated slabs' DMAs land before the LDS is used again
  __builtin_amdgcn_s_barrier();
  // accumulators pinned to the accumulation registers (as in ring_run)
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) asm volatile("" : "+a"(acc[i][j]));
  static_assert(4 * 4096 <= NSW * SLW + NS * SLX, "epilogue stages");
  gemm_epilogue<EPI, TN, TM, TR == (GEMM_TRANS_X | GEMM_TRANS_W)>(g, acc, lds + wave * 4096, m0 + wm * WM, (tn * BN + wn * WN) / (GLU ? 2 : 1), lane);
}

// Tile idx of an XCD-contiguous walk over `total` work items: the hardware
// deals workgroups round-robin to the 8 XCDs, and every XCD takes one run of
// consecutive items (the padded grid's workgroups past the end do nothing).
// A short launch's token tiles are the fast index, so one XCD holds all token
// tiles of its weight tiles: a weight row is fetched from memory by one L2
// instead of by all eight.
__device__ __forceinline__ int32_t xcd_item(int32_t b, int32_t grid) { return (b & 7) * (grid >> 3) + (b >> 3); }

// Tile t of the walk inside a launch or problem: token tiles fastest, all of
// them for up to 16 (each weight row is then wanted by one XCD at one time),
// else in groups of 8, so that an XCD's 32 tiles in flight form an 8 x 4 block.
__device__ __forceinline__ void flex_walk(int32_t t, int32_t tiles_m, int32_t tiles_n, int32_t& tm, int32_t& tn) {
  const int32_t gm = tiles_m <= 16 ? tiles_m : 8, per = gm * tiles_n;
  const int32_t grp = t / per, r = t - grp * per, size = min(tiles_m - grp * gm, gm);
  tm = grp * gm + r % size;
  tn = r / size;
}

// One launch over g: K ranges (slabs KT s / S ..), then tiles.
template <int BN, int BM, int NS, int NSW, int EPI, int OCC, bool WIDE>
__global__ __launch_bounds__(256, OCC) void gemm_flex_kernel(GemmArgs g, int32_t S) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[(NSW * BN + NS * BM) * kBK];
  const int32_t tiles = g.tiles_m * g.tiles_n, idx = xcd_item(blockIdx.x, gridDim.x);
  if (idx >= tiles * S) return;
  const int32_t s = idx / tiles, t = idx - s * tiles;
  const int64_t KT = g.K / kBK;
  if (s) g.C = reinterpret_cast<float*>(g.C) + (int64_t)s * g.split_c;
  int32_t tm, tn;
  flex_walk(t, g.tiles_m, g.tiles_n, tm, tn);
  flex_tile<BN, BM, NS, NSW, EPI, 0, WIDE>(g, tm, tn, (int32_t)(KT * s / S), (int32_t)(KT * (s + 1) / S), lds);
}

// One launch over several independent problems (one per tenant): work item i
// is tile i - tile_start of the problem whose tile range holds it.
template <int BN, int BM, int NS, int NSW, int EPI, int TR, int OCC, bool WIDE>
__global__ __launch_bounds__(256, OCC) void gemm_grouped_flex_kernel(const GemmArgs* __restrict__ probs, int32_t nprob,
                                                                     int32_t total, bool uneven) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[(NSW * BN + NS * BM) * kBK];
  const int32_t idx = uneven ? (int32_t)blockIdx.x : xcd_item(blockIdx.x, gridDim.x);
  if (idx >= total) return;
  int32_t p = 0;
  while (p + 1 < nprob && probs[p + 1].tile_start <= idx) ++p;
  const GemmArgs g = probs[p];
  int32_t tm, tn;
  flex_walk(idx - g.tile_start, g.tiles_m, g.tiles_n, tm, tn);
  flex_tile<BN, BM, NS, NSW, EPI, TR, WIDE>(g, tm, tn, 0, (g.K + kBK - 1) / kBK, lds);
}

// Ring-buffered loop of the 256x256 tile on 4 wavefronts, one per SIMD, each
// 128 weight rows x 128 tokens (64 accumulator blocks, kept in the
// accumulation registers).  Per K=64 slab kt, phase 0 runs the first k-half's
// 64 MFMAs while reading the second half's fragments and fetching the token
// half of slab kt+2; every wave then waits for its own DMA of slab kt+1 and a
// workgroup barrier; phase 1 runs the second half's MFMAs while reading slab
// kt+1's first-half fragments and fetching the weight half of slab kt+2.  The
// LDS holds two weight slots and three token slots (5 x 32 KB = 160 KB): a
// slot is refilled only after the barrier that follows its last fragment
// read.  The stream has no branches: past a tile's last slab the DMAs fetch the
// next tile's first two slabs (behind the workgroup's last tile, or where either
// tile has fewer than three slabs, they repeat slab KT-1 into free slots), so
// every phase issues the same instructions; each DMA is one buffer load to LDS
// with a per-lane 32-bit offset and the slab offset in a scalar register.  The
// epilogue runs between the last slab and the next tile's first, whose MFMAs
// take zero accumulators and whose wait counts the epilogue's stores (memory
// operations finish in order) instead of waiting for them.
// Measured on the 2048-wide shapes against the 8-wave ping-pong loop it
// replaces (two waves per SIMD alternating memory and compute phases): GeGLU
// 8.27 -> 7.36 ms, QKV 1.63 -> 1.50 ms.  Per-phase cycle stamps showed what
// the 8-wave loop and the first 4-wave versions lost: each conditional branch
// in the MFMA stream cost 30-50 cycles of issue, and global_load_lds with a
// 64-bit address computed per instruction cost more than the buffer form.
// Cycle stamps of the one-tile form on 65,536 x 3,072, K = 768: 2.5 to 3.5 us
// until the first fragments, 1.25 to 1.6 us per slab (2,330 cycles, 2,048 of
// MFMA; the clock falls to 1.5 to 1.9 GHz with the whole chip busy, so this is
// power), then the epilogue; with kRingChain tiles in a row the first part goes
// (bf16 291 -> 262 us).
// next(r, q, tm, tn): problem and tile of the workgroup's r-th turn, or false,
// and then nothing of them is set or read; lds holds 5 x 32 KB.
//
// TR: operands stored transposed (GEMM_TRANS_X: X is [K][M], element (m, k)
// at X[k * ldx + m]; GEMM_TRANS_W: W is [K][N]).  A transposed operand's
// half-slab is 64 k-lines of 256 rows (512 B per line, 2 lines per DMA
// instruction), its 16-byte chunks at position chunk ^ tswz(k); a fragment
// is two ds_read_b64_tr_b16 (k-slots 0..3 and 4..7 of the lane's k block), so
// the MFMA sequence per output element is the one of the row-major layout.
// Loads past line K of a transposed operand return zero (buffer range), so
// with both operands transposed K need not be a multiple of 64.
template <int EPI, int TR, class Next>
__device__ __forceinline__ void ring_run(const Next& next, uint16_t* __restrict__ lds) {
  constexpr bool TX = (TR & GEMM_TRANS_X) != 0, TW = (TR & GEMM_TRANS_W) != 0;
  constexpr int BN = 256, BM = 256, WGN = 2, WGM = 2;
  constexpr int WN = BN / WGN, WM = BM / WGM;
  constexpr int TN = WN / 16, TM = WM / 16;
  constexpr int NI = 8;            // 1 KB DMA instructions per wave per half-slab
  constexpr int SLOT = 256 * kBK;  // elements per half-slab slot
  constexpr bool GLU = EPI == EPI_GEGLU_BF16;
  // Stores of a whole tile's 16-bit epilogue per wave, counted by the first
  // slab's wait: one fewer and the wait would pass before slab 1 has landed.
  using E16 = Epi16<EPI, TN, TM>;
  static_assert(E16::NB * 16 % E16::RI == 0, "every instruction of a whole part stores");
  static_assert(!(GLU && TW), "GeGLU weights are row-major");

  GemmArgs g;
  int32_t tm, tn;
  if (!next(0, g, tm, tn)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave / WGM, wm = wave % WGM;

  // DMA sources of the tile being fetched: token rows tm*256.., weight rows
  // (GeGLU: gate and up columns tn*128..) -- rows past the end are clamped to
  // the last one.  row-major operand: wave w fetches rows 64w .. 64w+63 of the
  // half-slab, 8 rows per instruction; transposed: k-lines 16w .. 16w+15, 2 per
  // instruction.  Byte step between slabs: one 128-byte row segment (in the
  // scalar offset), or 64 k-lines of a transposed operand (in the lane offset,
  // which the buffer range check covers, so lines past K read zero).
  __amdgpu_buffer_rsrc_t xr, wr, wr2;
  uint32_t xo[NI], wo[NI];
  int32_t xso, wso;
  auto source = [&](const GemmArgs& q, int32_t qm, int32_t qn) {
    const int32_t m0 = qm * BM;
    const int32_t c0 = GLU ? qn * (BN / 2) : qn * BN;
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // (as in gemm_epilogue)
    xr = panel_rsrc(TX ? q.X + m0 : q.X + (int64_t)m0 * q.ldx,
                    TX ? ((int64_t)q.K * q.ldx - m0) * 2 : (int64_t)(q.M - m0) * q.ldx * 2);
    wr = panel_rsrc(TW ? q.W + c0 : q.W + (int64_t)c0 * q.ldw,
                    TW ? ((int64_t)q.K * q.ldw - c0) * 2 : (int64_t)(q.N - c0) * q.ldw * 2);
    if constexpr (GLU) wr2 = panel_rsrc(q.W2 + (int64_t)c0 * q.ldw, (int64_t)(q.N - c0) * q.ldw * 2);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = 64 * wave + 8 * i + (lane >> 3);
      const int chunk = (lane & 7) ^ lds_swz(r);
      const int kl = 16 * wave + 2 * i + (lane >> 5);
      const int tchunk = (lane & 31) ^ tswz(kl);
      if constexpr (TX)
        xo[i] = (uint32_t)(((int64_t)kl * q.ldx + tchunk * 8) * 2);
      else
        xo[i] = (uint32_t)min(r, q.M - 1 - m0) * (uint32_t)(q.ldx * 2) + chunk * 16;
      if constexpr (TW) {
        wo[i] = (uint32_t)(((int64_t)kl * q.ldw + tchunk * 8) * 2);
      } else {
        const int32_t col = GLU ? (r >> 5) * 16 + (r & 15) : r;
        wo[i] = (uint32_t)min(col, q.N - 1 - c0) * (uint32_t)(q.ldw * 2) + chunk * 16;
      }
    }
    xso = TX ? (int32_t)(kBK * 2 * q.ldx) : kBK * 2;
    wso = TW ? (int32_t)(kBK * 2 * q.ldw) : kBK * 2;
  };
  const int dro = wave * NI * 512;         // this wave's 1 KB blocks inside a slot
  uint16_t* const ring2 = lds;             // weight slabs, two slots
  uint16_t* const ring3 = lds + 2 * SLOT;  // token slabs, three slots
  // DMA i of slab `slab` into a slot; in GeGLU tiles, instruction i covers
  // weight rows of one 16-row block, all gate (W) or all up (W2)
#ifndef __HIP_DEVICE_COMPILE__
#define JN_DMA_W(i, slab, slot) (void)(slab)
#define JN_DMA_X(i, slab, slot) (void)(slab)
#else
#define JN_DMA_W(i, slab, slot)                                                                                  \
  __builtin_amdgcn_raw_ptr_buffer_load_lds((GLU && (((i) >> 1) & 1)) ? wr2 : wr,                                \
                                           JN_LPTR(ring2 + (slot) * SLOT + dro + (i) * 512), 16,                \
                                           TW ? wo[i] + (uint32_t)((slab) * wso) : wo[i], TW ? 0 : (slab) * wso, 0, 0)
#define JN_DMA_X(i, slab, slot)                                                                                  \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, JN_LPTR(ring3 + (slot) * SLOT + dro + (i) * 512), 16,            \
                                           TX ? xo[i] + (uint32_t)((slab) * xso) : xo[i], TX ? 0 : (slab) * xso, 0, \
                                           0)
#endif

  f32x4 acc[TN][TM];
  const int sw = lds_swz(lane & 15), quad = lane >> 4;
  const int wrow = wn * WN + (lane & 15), xrow = wm * WM + (lane & 15);
  // transposed reads (inline assembly, covered by the loop's LDS waits at
  // every phase boundary): lane (quad, e = (lane & 15) / 4, c = lane & 3) reads k-line
  // 8 quad + e (+4) at rows rbase + 4c; tr_base(part) | 16 ts, XORed with 16 f
  // per fragment f, addresses the swizzled chunk (bits 4-6 are free below)
  const int te = (lane & 15) >> 2, tc = lane & 3;
  const int tlane = (8 * quad + te) * 256 + 8 * (tc >> 1) + 4 * (tc & 1) + 16 * ((te & 3) | ((quad & 1) << 2));
  const int twl = tlane + 128 * wn, txl = tlane + 128 * wm;
  // fragment f (16 rows) of k-half h of a half-slab slot
  auto frag_w = [&](const uint16_t* slot, int f, int h) -> bf16x8 {
    if constexpr (TW) {
      const uint16_t* p = slot + 8192 * h + (twl ^ (16 * f));
      const bf16x4 lo = __builtin_bit_cast(bf16x4, lds_read_tr_b16<0>(p));
      const bf16x4 hi = __builtin_bit_cast(bf16x4, lds_read_tr_b16<2048>(p));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      return *reinterpret_cast<const bf16x8*>(slot + (wrow + 16 * f) * kBK + ((4 * h + quad) ^ sw) * 8);
    }
  };
  auto frag_x = [&](const uint16_t* slot, int f, int h) -> bf16x8 {
    if constexpr (TX) {
      const uint16_t* p = slot + 8192 * h + (txl ^ (16 * f));
      const bf16x4 lo = __builtin_bit_cast(bf16x4, lds_read_tr_b16<0>(p));
      const bf16x4 hi = __builtin_bit_cast(bf16x4, lds_read_tr_b16<2048>(p));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      return *reinterpret_cast<const bf16x8*>(slot + (xrow + 16 * f) * kBK + ((4 * h + quad) ^ sw) * 8);
    }
  };
  bf16x8 fa[TN + TM], fb[TN + TM];  // first-half / second-half fragments: weights, then tokens
  int slot2 = 0, slot3 = 0;         // slots of the current slab

  // slabs 0 and 1 of a tile (both halves)
  auto prologue = [&](int KT) {
    const int s1 = min(1, KT - 1);
#pragma unroll
    for (int i = 0; i < NI; ++i) JN_DMA_W(i, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) JN_DMA_X(i, 0, 0);
#pragma unroll
    for (int i = 0; i < NI; ++i) JN_DMA_X(i, s1, 1);
#pragma unroll
    for (int i = 0; i < NI; ++i) JN_DMA_W(i, s1, 1);
    wait_vmcnt<2 * NI>();
    __builtin_amdgcn_s_barrier();
    slot2 = slot3 = 0;
  };
  auto first_frags = [&]() {
#pragma unroll
    for (int i = 0; i < TN; ++i) fa[i] = frag_w(ring2 + slot2 * SLOT, i, 0);
#pragma unroll
    for (int j = 0; j < TM; ++j) fa[TN + j] = frag_x(ring3 + slot3 * SLOT, j, 0);
    wait_lgkmcnt<0>();
  };
  // One slab; sf: slab fetched; stored: the last STORES memory operations
  // before this slab's were stores.
  auto slab = [&](auto first, int sf, bool stored) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first)::value;
    const int next3 = slot3 == 2 ? 0 : slot3 + 1;
    const int prev3 = slot3 == 0 ? 2 : slot3 - 1;
    // ---- phase 0: first k-half MFMAs; second-half fragments; token DMA of the slab after next
    {
      const uint16_t* cw = ring2 + slot2 * SLOT;
      const uint16_t* cx = ring3 + slot3 * SLOT;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < TN * TM; ++q) {
        const int i = q / TM, j = q % TM;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fa[TN + j],
                                                            FIRST ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i][j], 0, 0, 0);
        if ((q & 3) == 0) {
          const int f = q >> 2;
          if (f < TN)
            fb[f] = frag_w(cw, f, 1);
          else
            fb[f] = frag_x(cx, f - TN, 1);
        }
        if ((q & 7) == 6) JN_DMA_X(q >> 3, sf, prev3);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the next slab landed (the token DMA just issued may stay in flight)
    wait_lgkmcnt<0>();
    if (FIRST && epi_bf16(EPI) && stored)
      wait_vmcnt<NI + E16::STORES>();
    else
      wait_vmcnt<NI>();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // ---- phase 1: second k-half MFMAs; the next slab's first-half fragments; weight DMA of the slab after next
    {
      const uint16_t* nw = ring2 + (slot2 ^ 1) * SLOT;
      const uint16_t* nx = ring3 + next3 * SLOT;
#pragma unroll
      for (int q = 0; q < TN * TM; ++q) {
        const int i = q / TM, j = q % TM;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[i], fb[TN + j], acc[i][j], 0, 0, 0);
        if ((q & 3) == 0) {
          const int f = q >> 2;
          if (f < TN)
            fa[f] = frag_w(nw, f, 0);
          else
            fa[f] = frag_x(nx, f - TN, 0);
        }
        if ((q & 7) == 6) JN_DMA_W(q >> 3, sf, slot2);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wait_lgkmcnt<0>();
    slot2 ^= 1;
    slot3 = next3;
  };

  source(g, tm, tn);
  int KT = (g.K + kBK - 1) / kBK;
  prologue(KT);
  bool stored = false;
  for (int r = 1;; ++r) {
    // the last two slabs fetch the next tile's first two, where both tiles
    // have three slabs; else (and behind the last tile) they repeat a slab
    GemmArgs gn;
    int32_t tmn, tnn;
    const bool more = next(r, gn, tmn, tnn);
    const int KTn = more ? (gn.K + kBK - 1) / kBK : 0;
    const bool joined = KT >= 3 && KTn >= 3;
    first_frags();  // (read again behind an epilogue, which needs the registers)
    slab(std::true_type{}, min(2, KT - 1), stored);
    for (int kt = 1; kt < KT - 2; ++kt) slab(std::false_type{}, kt + 2, false);
    if (joined) source(gn, tmn, tnn);
    for (int kt = max(1, KT - 2); kt < KT; ++kt) slab(std::false_type{}, joined ? kt + 2 - KT : KT - 1, false);
    // Pin the accumulators to the accumulation registers where the loop ends.
    // Left to itself, the register allocator placed some accumulators of the
    // epilogues that can store straight from either register file (fp32 store,
    // fp32 pre-activation save) in vector registers and copied them into
    // accumulation registers before every MFMA of the loop (with spills to
    // scratch in the grouped variants).
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) asm volatile("" : "+a"(acc[i][j]));
    // the free token slot; a wave uses the part that only its own DMAs fill
    const bool whole =
        gemm_epilogue<EPI, TN, TM, TR == (GEMM_TRANS_X | GEMM_TRANS_W)>(g, acc, ring3 + (slot3 == 0 ? 2 : slot3 - 1) * SLOT + dro, tm * BM + wm * WM,
                                   (tn * BN + wn * WN) / (GLU ? 2 : 1), lane);
    if (!more) break;
    stored = joined && whole;
    g = gn;
    tm = tmn;
    tn = tnn;
    KT = KTn;
    if (!joined) {
      wait_vmcnt<0>();  // the repeated slabs' DMAs land before their slots are filled
      __builtin_amdgcn_s_barrier();
      source(g, tm, tn);
      prologue(KT);
    }
  }
#undef JN_DMA_W
#undef JN_DMA_X
  wait_vmcnt<0>();  // ... or before the LDS is released
}

// Position of a workgroup's r-th tile: groups of 256 workgroups, `chain` tiles
// each, walk chain x 256 consecutive tiles in rounds of 256.
__device__ __forceinline__ int64_t chain_tile(int32_t b, int32_t chain, int32_t r) {
  return (int64_t)(b >> 8) * 256 * chain + 256 * r + (b & 255);
}

// One launch of ring tiles over g.
template <int EPI>
__global__ __launch_bounds__(256, 1) void gemm_ring_kernel(GemmArgs g, int32_t chain) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[5 * 256 * kBK];
  auto next = [&](int32_t r, GemmArgs& q, int32_t& tm, int32_t& tn) __attribute__((always_inline)) {
    const int64_t t = chain_tile(blockIdx.x, chain, r);
    if (r >= chain || t >= (int64_t)g.tiles_m * g.tiles_n) return false;
    q = g;
    tile_of((int32_t)t, g.tiles_m, g.tiles_n, tm, tn);
    return true;
  };
  ring_run<EPI, 0>(next, lds);
}

// The same over S K ranges, fp32 partials, in gemm_flex_kernel's walk.
__global__ __launch_bounds__(256, 1) void gemm_ring_split_kernel(GemmArgs g, int32_t S) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[5 * 256 * kBK];
  auto next = [&](int32_t r, GemmArgs& q, int32_t& tm, int32_t& tn) __attribute__((always_inline)) {
    const int32_t tiles = g.tiles_m * g.tiles_n, idx = xcd_item(blockIdx.x, gridDim.x);
    if (r > 0 || idx >= tiles * S) return false;
    const int32_t s = idx / tiles;
    const int64_t KT = g.K / kBK, k0 = KT * s / S, k1 = KT * (s + 1) / S;
    q = g;
    q.X += k0 * kBK;
    q.W += k0 * kBK;
    q.K = (int32_t)(k1 - k0) * kBK;
    q.C = reinterpret_cast<float*>(g.C) + (int64_t)s * g.split_c;
    flex_walk(idx - s * tiles, g.tiles_m, g.tiles_n, tm, tn);
    return true;
  };
  ring_run<EPI_F32, 0>(next, lds);
}

// Grouped ring tiles: problem p owns tiles [tile_start, tile_start + tiles).
template <int EPI, int TR>
__global__ __launch_bounds__(256, 1) void gemm_grouped_ring_kernel(const GemmArgs* __restrict__ probs, int32_t nprob,
                                                                   int32_t total, int32_t chain) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[5 * 256 * kBK];
  int32_t p = 0;
  auto next = [&](int32_t r, GemmArgs& q, int32_t& tm, int32_t& tn) __attribute__((always_inline)) {
    const int64_t t = chain_tile(blockIdx.x, chain, r);
    if (r >= chain || t >= total) return false;
    while (p + 1 < nprob && probs[p + 1].tile_start <= t) ++p;
    q = probs[p];
    tile_of((int32_t)t - q.tile_start, q.tiles_m, q.tiles_n, tm, tn);
    return true;
  };
  ring_run<EPI, TR>(next, lds);
}

// Data and weight gradients of one layer in one launch: both read dY, neither
// the other's output.  Workgroups [0, gd) run the data gradient's 128x96 tiles
// (contractions over the layer's width, the longer ones, so they start first),
// the rest the weight gradient's 128x128 tiles (contractions over the tenant's
// rows).  gd and the rest are multiples of 8, so both keep their XCD walk.
// Alone, a single tenant's launches fill few CUs (400 rows, 1,024 wide: 40
// data-gradient tiles of 10 to 26 us, 64 to 256 weight-gradient tiles of 9 to
// 12 us); a pair takes about the longer of the two (24.7 -> 12, 37 -> 26 us,
// with the key/value weight gradient 45 -> 26), one tenant's step 792 -> 696 us.
template <int EPI>
__global__ __launch_bounds__(256, 1) void gemm_grad_pair_kernel(const GemmArgs* __restrict__ dprobs, int32_t nd,
                                                                int32_t td, int32_t gd,
                                                                const GemmArgs* __restrict__ wprobs, int32_t nw,
                                                                int32_t tw) {
  constexpr int BN = 128, BM = 96, NS = 4, LDS = NS * (BN + BM) * kBK;
  static_assert(LDS >= 5 * 128 * kBK, "stages of both loops");
  __shared__ __attribute__((aligned(1024))) uint16_t lds[LDS];
  const bool data = (int32_t)blockIdx.x < gd;
  const GemmArgs* const probs = data ? dprobs : wprobs;
  const int32_t n = data ? nd : nw;
  const int32_t idx = data ? xcd_item(blockIdx.x, gd) : xcd_item(blockIdx.x - gd, gridDim.x - gd);
  if (idx >= (data ? td : tw)) return;
  int32_t p = 0;
  while (p + 1 < n && probs[p + 1].tile_start <= idx) ++p;
  const GemmArgs g = probs[p];
  int32_t tm, tn;
  flex_walk(idx - g.tile_start, g.tiles_m, g.tiles_n, tm, tn);
  const int32_t KT = (g.K + kBK - 1) / kBK;
  if (data)
    flex_tile<BN, BM, NS, NS, EPI, GEMM_TRANS_W>(g, tm, tn, 0, KT, lds);
  else
    flex_tile<128, 128, 3, 2, EPI_F32, GEMM_TRANS_X | GEMM_TRANS_W>(g, tm, tn, 0, KT, lds);
}

// Tile shapes: the 256x256 ring loop, then shapes of the flexible loop.  occ:
// workgroups per CU.  slab: microseconds per K=64 slab with all 256 CUs busy,
// measured on the 2048-wide projections at 2,469 tokens (the chip is then
// power-limited; a few busy CUs run 1.1 / 0.8 / 0.6 / 0.4 / 0.27); slab1: with
// one workgroup on the CU.  fix: per tile, fetching the first slabs and the
// launch's share.
struct TileShape {
  int bn, bm, occ;
  double slab, slab1, fix;
};
constexpr TileShape kShapes[] = {
    {256, 256, 1, 1.45, 1.45, 5.0}, {256, 160, 1, 1.10, 1.10, 4.5}, {256, 128, 1, 0.90, 0.90, 4.5},
    {128, 160, 1, 0.62, 0.62, 4.0}, {128, 96, 1, 0.46, 0.46, 4.0},  {64, 96, 2, 0.26, 0.28, 4.0},
    {128, 128, 2, 0.54, 0.62, 2.3},
};
constexpr int kNumShapes = 6;   // of every launch
constexpr int k128Shape = 6;    // and of unsplit residual adds and grouped weight gradients

// 32-bit lane offsets span the 256 rows of a panel; beyond (leading dimensions
// past 4M elements), the small shape runs with one buffer base per DMA
// instruction (kWideShape of the grouped launches).
constexpr int kWideShape = 7;
static bool wide_rows(const GemmArgs& g) { return 512 * std::max(g.ldx, g.ldw) > (int64_t)0x7fffffff; }

// Tiles per workgroup of a ring launch, and its workgroups.  Eight: 1, 4, 8 and
// 64 tiles in a row take 289, 277, 275 and 273 us on 65,536 x 3,072, K = 768,
// and workgroups that are replaced every few tiles keep sharing the chip with
// other streams' launches.
constexpr int32_t kRingChain = 8;
static int32_t ring_chain(int32_t tiles) { return std::min(kRingChain, (tiles + 255) / 256); }
static unsigned ring_groups(int32_t tiles, int32_t chain) {
  const int64_t whole = tiles / (256 * (int64_t)chain), rest = tiles - whole * 256 * chain;
  return (unsigned)(whole * 256 + std::min<int64_t>(rest, 256));
}

// The 256x256 ring loop over all tiles of g (and S K ranges).
static hipError_t launch_ring(hipStream_t s, int epi, GemmArgs g, int32_t S) {
  const int32_t NL = epi == EPI_GEGLU_BF16 ? 2 * g.N : g.N;
  g.tiles_m = (g.M + 255) / 256;
  g.tiles_n = (NL + 255) / 256;
  const int32_t tiles = g.tiles_m * g.tiles_n, chain = ring_chain(tiles);
  const dim3 grid(ring_groups(tiles, chain)), block(256);
  if (S > 1) {
    if (epi != EPI_F32) return hipErrorInvalidValue;
    gemm_ring_split_kernel<<<dim3((tiles * S + 7) / 8 * 8), block, 0, s>>>(g, S);
    return hipGetLastError();
  }
  switch (epi) {
    case EPI_BF16: gemm_ring_kernel<EPI_BF16><<<grid, block, 0, s>>>(g, chain); break;
    case EPI_GELU_BF16: gemm_ring_kernel<EPI_GELU_BF16><<<grid, block, 0, s>>>(g, chain); break;
    case EPI_RESID_F32: gemm_ring_kernel<EPI_RESID_F32><<<grid, block, 0, s>>>(g, chain); break;
    case EPI_GEGLU_BF16: gemm_ring_kernel<EPI_GEGLU_BF16><<<grid, block, 0, s>>>(g, chain); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int BN, int BM, int NS, int OCC, bool WIDE = false>
static hipError_t launch_flex(hipStream_t s, int epi, GemmArgs g, int32_t S) {
  const int32_t NL = epi == EPI_GEGLU_BF16 ? 2 * g.N : g.N;
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = (NL + BN - 1) / BN;
  const dim3 grid((unsigned)(((int64_t)g.tiles_m * g.tiles_n * S + 7) / 8 * 8)), block(256);
#define JN_GEMM_CASE(E) \
  case E: gemm_flex_kernel<BN, BM, NS, NS, E, OCC, WIDE><<<grid, block, 0, s>>>(g, S); break;
  if constexpr (WIDE) {
    switch (epi) {
      JN_GEMM_CASE(EPI_RESID_F32)
      JN_GEMM_CASE(EPI_F32)
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (epi) {
      JN_GEMM_CASE(EPI_BF16)
      JN_GEMM_CASE(EPI_GELU_BF16)
      JN_GEMM_CASE(EPI_RESID_F32)
      JN_GEMM_CASE(EPI_GEGLU_BF16)
      JN_GEMM_CASE(EPI_F32)
      default: return hipErrorInvalidValue;
    }
  }
#undef JN_GEMM_CASE
  return hipGetLastError();
}

// 128x128 residual tiles, two workgroups per CU (three token and two weight
// stages each).
static hipError_t launch_resid128(hipStream_t s, GemmArgs g) {
  g.tiles_m = (g.M + 127) / 128;
  g.tiles_n = (g.N + 127) / 128;
  const dim3 grid((unsigned)(((int64_t)g.tiles_m * g.tiles_n + 7) / 8 * 8));
  gemm_flex_kernel<128, 128, 3, 2, EPI_RESID_F32, 2, false><<<grid, 256, 0, s>>>(g, 1);
  return hipGetLastError();
}

// One launch over all rows of g with tile shape t and S K ranges.
static hipError_t launch_rows(hipStream_t s, int epi, const GemmArgs& g, int t, int32_t S = 1) {
  if (wide_rows(g)) return launch_flex<64, 96, 4, 2, true>(s, epi, g, S);
  switch (t) {
    case 0: return launch_ring(s, epi, g, S);
    case 1: return launch_flex<256, 160, 3, 1>(s, epi, g, S);
    case 2: return launch_flex<256, 128, 3, 1>(s, epi, g, S);
    case 3: return launch_flex<128, 160, 4, 1>(s, epi, g, S);
    case 4: return launch_flex<128, 96, 4, 1>(s, epi, g, S);
    case 5: return launch_flex<64, 96, 4, 2>(s, epi, g, S);
    default: return epi == EPI_RESID_F32 && S == 1 ? launch_resid128(s, g) : hipErrorInvalidValue;
  }
}

static hipError_t launch_grouped_ring(hipStream_t s, int epi, const GemmArgs* dprobs, int32_t nprob,
                                      int32_t total_tiles, int trans, bool uneven) {
  const int32_t chain = uneven ? 1 : ring_chain(total_tiles);
  dim3 grid(ring_groups(total_tiles, chain)), block(256);
#define JN_GEMM_CASE(E, T) \
  case E * 4 + T: gemm_grouped_ring_kernel<E, T><<<grid, block, 0, s>>>(dprobs, nprob, total_tiles, chain); break;
  switch (epi * 4 + trans) {
    JN_GEMM_CASE(EPI_BF16, 0)
    JN_GEMM_CASE(EPI_RESID_F32, 0)
    JN_GEMM_CASE(EPI_F32, 0)
    JN_GEMM_CASE(EPI_GELU_SAVE, 0)
    JN_GEMM_CASE(EPI_GELUGRAD_BF16, 0)
    JN_GEMM_CASE(EPI_F32, GEMM_TRANS_W)
    JN_GEMM_CASE(EPI_GELUGRAD_BF16, GEMM_TRANS_W)
    JN_GEMM_CASE(EPI_F32, GEMM_TRANS_X | GEMM_TRANS_W)
    default:
      return hipErrorInvalidValue;
  }
#undef JN_GEMM_CASE
  return hipGetLastError();
}

template <int BN, int BM, int NS, int NSW, int OCC, bool WIDE = false>
static hipError_t launch_grouped_flex(hipStream_t s, int epi, const GemmArgs* dprobs, int32_t nprob, int32_t total,
                                      int trans, bool uneven) {
  const dim3 grid((unsigned)((total + 7) / 8 * 8)), block(256);
#define JN_GEMM_CASE(E, T)                                                                                       \
  case E * 4 + T:                                                                                                \
    gemm_grouped_flex_kernel<BN, BM, NS, NSW, E, T, OCC, WIDE><<<grid, block, 0, s>>>(dprobs, nprob, total, uneven); break;
  if constexpr (WIDE) {
    switch (epi * 4 + trans) {
      JN_GEMM_CASE(EPI_RESID_F32, 0)
      JN_GEMM_CASE(EPI_F32, 0)
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  if constexpr (BN % 128 == 0 && BM % 128 == 0) {
    if (trans == (GEMM_TRANS_X | GEMM_TRANS_W)) {
      switch (epi * 4 + trans) {
        JN_GEMM_CASE(EPI_F32, GEMM_TRANS_X | GEMM_TRANS_W)
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    }
  }
  if constexpr (BN % 128 == 0 && NSW == NS) {
    if (trans == GEMM_TRANS_W) {
      switch (epi * 4 + trans) {
        JN_GEMM_CASE(EPI_F32, GEMM_TRANS_W)
        JN_GEMM_CASE(EPI_GELUGRAD_BF16, GEMM_TRANS_W)
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    }
  }
  if constexpr (NSW == NS) {
    switch (epi * 4 + trans) {
      JN_GEMM_CASE(EPI_BF16, 0)
      JN_GEMM_CASE(EPI_RESID_F32, 0)
      JN_GEMM_CASE(EPI_F32, 0)
      JN_GEMM_CASE(EPI_GELU_SAVE, 0)
      JN_GEMM_CASE(EPI_GELUGRAD_BF16, 0)
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
#undef JN_GEMM_CASE
}

// Bytes an epilogue reads and writes per tile element (GeGLU: per gate or up
// element), and the microseconds of its GELU per element and CU.
static double epi_bytes(int epi) {
  switch (epi) {
    case EPI_RESID_F32: return 8.0;
    case EPI_F32: return 4.0;
    case EPI_GELU_SAVE: case EPI_GELUGRAD_BF16: return 6.0;
    case EPI_GEGLU_BF16: return 1.0;
    default: return 2.0;
  }
}
static double epi_alu(int epi) {
  switch (epi) {
    case EPI_GELU_BF16: return 7.5e-5;
    case EPI_GEGLU_BF16: return 4e-5;
    case EPI_GELU_SAVE: case EPI_GELUGRAD_BF16: return 8e-5;
    default: return 0.0;
  }
}

// Time of `tiles` tiles of shape t with `slabs` slabs each, in microseconds:
// rounds of 256 tiles, each its slabs, fixed cost and GELU, plus the epilogue's
// bytes at the copy rate (4.8 TB/s).  One workgroup per CU runs its epilogue
// while its matrix cores idle, and all tiles of a round reach it together (the
// 768-wide O projection spends 33 of a round's 55 us there); with two per CU
// about half of it runs under the other's main loop, and over many rounds the
// tiles drift apart and the weights stay in the caches (13%).  Against measurements
// (300 to 28,812 tokens, 768- and 2048-wide projections) within ~15%.
static double tiles_time(int epi, int64_t tiles, double slabs, int t) {
  const TileShape& T = kShapes[t];
  const double elems = (double)T.bn * T.bm, rounds = (double)((tiles + 255) / 256);
  const double once = rounds * (T.fix + elems * epi_alu(epi)) + tiles * elems * epi_bytes(epi) / 4.8e6;
  if (T.occ == 2) return rounds * slabs * (rounds > 1 ? T.slab : T.slab1) + 0.5 * (once + T.fix);
  return (rounds * slabs * T.slab + once) * (1.0 - 0.013 * std::min(rounds - 1.0, 10.0));
}

// K may be split (fp32 partials of S ranges added in range order by a second
// launch, which applies the epilogue) where the launch has at most 128 tiles
// of 256x256 and K >= 2048: with fewer, longer tiles most CUs would idle.  Two
// launches that split a GEMM differently sum its K ranges differently, so the
// limits also bound which batches can differ in their last bits.
static bool may_split(int epi, int32_t rows, int32_t N, int32_t K) {
  if (epi != EPI_BF16 && epi != EPI_RESID_F32 && epi != EPI_GELU_BF16) return false;
  return K >= 2048 && N % 4 == 0 && (int64_t)((rows + 255) / 256) * ((N + 255) / 256) <= 128;
}

// One launch over `rows` rows and S K ranges; a split adds the launch of its
// reduction and the second half of the fp32 partials' round trip.  stream: the time
// its weights take from memory at least.
static double tile_time(int epi, int32_t rows, int32_t N, int32_t K, int t, int32_t S, double stream) {
  const TileShape& T = kShapes[t];
  const int64_t NL = epi == EPI_GEGLU_BF16 ? 2 * (int64_t)N : N;
  const int64_t tiles = (rows + T.bm - 1) / T.bm * ((NL + T.bn - 1) / T.bn) * S;
  const double us = std::max(stream, tiles_time(S > 1 ? EPI_F32 : epi, tiles, (double)((K / kBK + S - 1) / S), t));
  return S > 1 ? us + 4.0 + 4e-6 * S * (double)rows * N / 4.8 : us;
}

// Where a split is a choice, no launch is faster than its weights come from memory
// (33 MB 8.6 us, 100 MB 20 to 23, 134 MB 28 to 31), and ranges that start whole
// multiples of 4 KB apart, all workgroups then asking the same channels, take a fifth
// longer (one row, 4,096 x 16,384 in 3, 5, 6 and 12 ranges 32, 30, 30 and 28 us, in 4
// and 8 34 and 37; 2,048 x 16,384 in 8 19, in 6 and 16 16 and 15).  Of two as fast,
// the one of fewer ranges.
static double stream_time(int32_t N, int32_t K, int32_t S) {
  const double us = 2.5 + 2.0 * (double)N * K / 5.4e6;
  return (S > 1 && K % (2048 * S) == 0 ? 1.2 * us : us) + 0.05 * S;
}

// Shape and K split of one launch over `rows` rows; ranges of >= 8 slabs.
static double plan_launch(int epi, int32_t rows, int32_t N, int32_t K, bool split, int* shape, int32_t* S) {
  const int32_t smax = split && may_split(epi, rows, N, K) ? std::min(16, K / (8 * kBK)) : 1;
  double stream[17] = {};  // of k ranges
  for (int32_t k = 1; smax > 1 && k <= smax; ++k) stream[k] = stream_time(N, K, k);
  double best = 1e300;
  for (int t = 0; t <= k128Shape; ++t) {
    if (t == k128Shape && epi != EPI_RESID_F32) break;
    for (int32_t k = 1; k <= (t == k128Shape ? 1 : smax); ++k) {
      const double us = tile_time(epi, rows, N, K, t, k, stream[k]);
      if (us < best * 0.999) {
        best = us;
        *shape = t;
        *S = k;
      }
    }
  }
  return best;
}

// Launches of one GEMM: rows [0, m1) as whole waves of 256x256 ring tiles and
// the rest with the shape (and, for K >= kTailSplitK, the K split) that the
// estimate gives the shortest time, or one launch over all rows.  The cut lies
// where the leading tiles fill the last or the last but one wave.  The split
// tail of a long contraction is summed in K ranges, so a row of such a launch
// can differ in its last bits from the same row in another batch (every shape
// runs the same MFMA sequence per output element, so nothing else can).
constexpr int32_t kTailSplitK = 8192;
constexpr double kLaunchGap = 3.0;  // microseconds between two launches on one stream

GemmPlan gemm_plan(int epi, int32_t M, int32_t N, int32_t K) {
  GemmPlan P;
  if (M <= 0 || N <= 0 || K <= 0) return P;
  double best = plan_launch(epi, M, N, K, true, &P.shape, &P.S);
  const int64_t tn = ((epi == EPI_GEGLU_BF16 ? 2 * (int64_t)N : N) + 255) / 256, tm = (M + 255) / 256;
  const int64_t waves = (tm * tn + 255) / 256;
  int64_t last = -1;
  for (int64_t w = waves - 1; w >= 1 && w >= waves - 2; --w) {
    const int64_t r = std::min(tm - 1, 256 * w / tn);
    if (r < 1 || r == last) continue;
    last = r;
    const int32_t m1 = (int32_t)(r * 256);
    int t = 0;
    int32_t S = 1;
    double us = tile_time(epi, m1, N, K, 0, 1, 0.0) + kLaunchGap;
    us += plan_launch(epi, M - m1, N, K, K >= kTailSplitK, &t, &S);
    if (us < best * 0.99) {
      best = us;
      P.m1 = m1;
      P.shape = t;
      P.S = S;
    }
  }
  return P;
}

int32_t gemm_split(int epi, int32_t M, int32_t N, int32_t K) {
  const GemmPlan P = gemm_plan(epi, M, N, K);
  return P.m1 == 0 ? P.S : 1;
}

size_t gemm_split_bytes(int epi, int32_t M, int32_t N, int32_t K) {
  const GemmPlan P = gemm_plan(epi, M, N, K);
  return P.S > 1 ? (size_t)P.S * (M - P.m1) * N * sizeof(float) : 0;
}

static hipError_t launch_splitk_reduce(hipStream_t s, int epi, const float* part, int32_t S, int32_t M, int32_t N,
                                       void* C, int64_t ldc) {
  const int64_t work = (int64_t)M * (N / 4), stride = (int64_t)M * N;
  const dim3 grid((unsigned)((work + 255) / 256));
  switch (epi) {
    case EPI_BF16: splitk_reduce_kernel<EPI_BF16><<<grid, 256, 0, s>>>(part, S, stride, M, N, C, ldc); break;
    case EPI_RESID_F32: splitk_reduce_kernel<EPI_RESID_F32><<<grid, 256, 0, s>>>(part, S, stride, M, N, C, ldc); break;
    case EPI_GELU_BF16: splitk_reduce_kernel<EPI_GELU_BF16><<<grid, 256, 0, s>>>(part, S, stride, M, N, C, ldc); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gemm(hipStream_t s, int epi, const void* A, int64_t lda, const void* B, const void* B2, int64_t ldb,
                       void* C, int64_t ldc, int32_t M, int32_t N, int32_t K, void* split_ws, size_t split_bytes,
                       bool partials_only) {
  if (M <= 0 || N <= 0 || K <= 0 || K % kBK != 0 || N % 32 != 0) return hipErrorInvalidValue;
  const GemmPlan P = gemm_plan(epi, M, N, K);
  GemmArgs g{};
  g.X = reinterpret_cast<const uint16_t*>(A);
  g.W = reinterpret_cast<const uint16_t*>(B);
  g.W2 = reinterpret_cast<const uint16_t*>(B2);
  g.C = C;
  g.ldx = lda;
  g.ldw = ldb;
  g.ldc = ldc;
  g.N = N;
  g.K = K;
  if (P.m1 > 0) {
    g.M = P.m1;
    const hipError_t e = launch_rows(s, epi, g, 0);
    if (e != hipSuccess) return e;
    const size_t esize = epi == EPI_RESID_F32 ? 4 : 2;
    g.X += (int64_t)P.m1 * lda;
    g.C = static_cast<char*>(C) + (size_t)P.m1 * ldc * esize;
  }
  g.M = M - P.m1;
  if (P.S == 1) return launch_rows(s, epi, g, P.shape);
  if (!split_ws || split_bytes < (size_t)P.S * g.M * N * sizeof(float)) return hipErrorInvalidValue;
  void* const out = g.C;
  g.C = split_ws;
  g.ldc = N;
  g.split_c = (int64_t)g.M * N;
  const hipError_t e = launch_rows(s, EPI_F32, g, P.shape, P.S);
  if (e != hipSuccess || (partials_only && P.m1 == 0)) return e;
  return launch_splitk_reduce(s, epi, reinterpret_cast<const float*>(split_ws), P.S, g.M, N, out, ldc);
}

// Shapes a grouped launch may take: a transposed operand's tile side is a
// multiple of 128 elements.
static bool grouped_shape_ok(int trans, int t) {
  if (t == k128Shape) return trans == (GEMM_TRANS_X | GEMM_TRANS_W);
  const TileShape& T = kShapes[t];
  return (!(trans & GEMM_TRANS_W) || T.bn % 128 == 0) && (!(trans & GEMM_TRANS_X) || T.bm % 128 == 0);
}

// Weight gradients of tenants of unequal sizes contract over unequal row
// counts: a tile takes as long as its tenant's share.  Where the longest is a
// quarter over the mean the tiles are launched longest first, one per workgroup
// in launch order (no runs of tiles per workgroup or XCD, which would leave the
// large tenants' runs for last), so that the short ones fill the gaps, and the
// shape's estimate counts the longest tile.  16 tenants of 250 to 2,150 rows:
// 1,024 x 1,024 69 -> 58 us (256 ring tiles before, 128x128 tiles now), 3,072 x
// 1,024 142 -> 118, and over their 3K to 25K prefix rows 2,048 x 768 525 -> 454.
bool gemm_grouped_uneven(const GemmArgs* probs, int32_t nprob) {
  int64_t longest = 0, sum = 0;
  for (int32_t p = 0; p < nprob; ++p) {
    if (probs[p].trans != (GEMM_TRANS_X | GEMM_TRANS_W)) return false;
    longest = std::max<int64_t>(longest, probs[p].K);
    sum += probs[p].K;
  }
  return 4 * longest * nprob > 5 * sum;
}

// Shape of a grouped launch: the estimate over all problems' tiles, where every
// offset fits 32 bits.
int gemm_grouped_tile_shape(int epi, const GemmArgs* probs, int32_t nprob) {
  bool narrow = true, trans = false;
  constexpr int64_t kMax = 0x7fffffff;
  for (int32_t p = 0; p < nprob; ++p) {
    const GemmArgs& g = probs[p];
    // per-lane panel offsets: 256 rows of a row-major operand, or its whole
    // K lines (plus one slab) for a transposed one
    const int64_t kx = (int64_t)g.K + kBK, span_x = (g.trans & GEMM_TRANS_X) ? kx * g.ldx : 256 * g.ldx;
    const int64_t span_w = (g.trans & GEMM_TRANS_W) ? kx * g.ldw : 256 * g.ldw;
    if (2 * std::max(span_x, span_w) > kMax) narrow = false;
    trans = trans || g.trans != 0;
  }
  if (!narrow) return trans ? -1 : kWideShape;
  const bool uneven = gemm_grouped_uneven(probs, nprob);
  int64_t longest = 0;
  for (int32_t p = 0; p < nprob; ++p) longest = std::max<int64_t>(longest, (probs[p].K + kBK - 1) / kBK);
  int best = 0;
  double best_us = 1e300;
  for (int t = 0; t <= k128Shape; ++t) {
    const TileShape& T = kShapes[t];
    if (!grouped_shape_ok(trans ? probs[0].trans : 0, t)) continue;
    int64_t tiles = 0, work = 0;  // tiles, and slabs of all tiles
    for (int32_t p = 0; p < nprob; ++p) {
      const int64_t n = (int64_t)((probs[p].M + T.bm - 1) / T.bm) * ((probs[p].N + T.bn - 1) / T.bn);
      tiles += n;
      work += n * ((probs[p].K + kBK - 1) / kBK);
    }
    double us = tiles_time(epi, tiles, (double)work / tiles, t);
    if (uneven) us = std::max(us, longest * std::max(T.slab, T.slab1) + tiles_time(epi, tiles, 0.0, t));
    if (us < best_us * 0.999) {
      best_us = us;
      best = t;
    }
  }
  return best;
}

int32_t gemm_grouped_prepare(GemmArgs* probs, int32_t nprob, int shape) {
  if (shape < 0 || shape > kWideShape || nprob <= 0) return -1;
  const TileShape& T = kShapes[shape == kWideShape ? kNumShapes - 1 : shape];
  const int BN = T.bn, BM = T.bm;
  if (gemm_grouped_uneven(probs, nprob))
    std::stable_sort(probs, probs + nprob, [](const GemmArgs& a, const GemmArgs& b) { return a.K > b.K; });
  int32_t total = 0;
  for (int32_t p = 0; p < nprob; ++p) {
    const GemmArgs& g = probs[p];
    const bool ragged_ok = g.trans == (GEMM_TRANS_X | GEMM_TRANS_W);
    if (g.trans != probs[0].trans || g.trans < 0 || g.trans > 3) return -1;
    if (shape == kWideShape ? g.trans != 0 : !grouped_shape_ok(g.trans, shape)) return -1;
    if (g.M <= 0 || g.N <= 0 || g.K <= 0 || (!ragged_ok && g.K % kBK != 0) || g.N % 32 != 0) return -1;
    probs[p].tiles_m = (probs[p].M + BM - 1) / BM;
    probs[p].tiles_n = (probs[p].N + BN - 1) / BN;
    probs[p].tile_start = total;
    total += probs[p].tiles_m * probs[p].tiles_n;
  }
  return total;
}

hipError_t launch_gemm_grouped(hipStream_t s, int epi, const GemmArgs* dprobs, int32_t nprob, int32_t total_tiles,
                               int shape, int trans, bool uneven) {
  if (nprob <= 0 || total_tiles <= 0) return hipErrorInvalidValue;
  switch (shape) {
    case 0: return launch_grouped_ring(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    case 1: return launch_grouped_flex<256, 160, 3, 3, 1>(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    case 2: return launch_grouped_flex<256, 128, 3, 3, 1>(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    case 3: return launch_grouped_flex<128, 160, 4, 4, 1>(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    case 4: return launch_grouped_flex<128, 96, 4, 4, 1>(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    case 5: return launch_grouped_flex<64, 96, 4, 4, 2>(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    case k128Shape: return launch_grouped_flex<128, 128, 3, 2, 2>(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    case kWideShape: return launch_grouped_flex<64, 96, 4, 4, 2, true>(s, epi, dprobs, nprob, total_tiles, trans, uneven);
    default: return hipErrorInvalidValue;
  }
}

// Which data and weight gradients run as a pair: those whose estimates pick the
// tile shapes of few rows.  Two 128x128 tiles share a CU in their own launch
// but not in a pair, so up to two rounds of them.  Many tenants' gradients fill
// the chip by themselves: 256x128 and ring tiles as a pair were slower (16
// tenants' MLP layer 362 -> 436 us, query and key/value 612 -> 701).
bool gemm_grad_pair_ok(int epi, int dshape, int wshape, int32_t wtiles) {
  return (epi == EPI_F32 || epi == EPI_GELUGRAD_BF16) && dshape == 4 && wshape == k128Shape && wtiles <= 512;
}

hipError_t launch_gemm_grad_pair(hipStream_t s, int epi, const GemmArgs* dprobs, int32_t nd, int32_t td,
                                 const GemmArgs* wprobs, int32_t nw, int32_t tw) {
  if (nd <= 0 || nw <= 0 || td <= 0 || tw <= 0) return hipErrorInvalidValue;
  const int32_t gd = (td + 7) / 8 * 8, gw = (tw + 7) / 8 * 8;
  const dim3 grid(gd + gw), block(256);
  switch (epi) {
    case EPI_F32: gemm_grad_pair_kernel<EPI_F32><<<grid, block, 0, s>>>(dprobs, nd, td, gd, wprobs, nw, tw); break;
    case EPI_GELUGRAD_BF16:
      gemm_grad_pair_kernel<EPI_GELUGRAD_BF16><<<grid, block, 0, s>>>(dprobs, nd, td, gd, wprobs, nw, tw);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace jnx
