// Tenant split and tenant-private action heads (fp32):
//   pool       mean of each sample's valid rows of the shared feature, written
//              in tenant order (the split of the shared features by slices)
//   head_gemm  one launch per head layer and direction for all tenants, fp32
//              matrix-core tiles: forward (bias, GELU or the squared-error loss
//              and its gradient fused), weight gradient (bias gradient fused)
//              and data gradient (GELU derivative fused); tenant row ranges are
//              read from the device maps, so the host needs no per-tenant counts
// Every reduction runs in a fixed order: results are bitwise reproducible.
#include <algorithm>

#include "jn_device.h"
#include "jn_internal.h"

namespace jnx {

// ------------------------------------------------------------------ pool ---

// Block = (sample, 512-column chunk); 256 threads = 4 wavefronts, lane l
// owning columns 8 l .. 8 l + 7 (one 16-byte load covers 1 KB of a row per
// wave).  Wave w sums rows w, w+4, w+8, ... of the sample in that order, eight
// loads in flight per lane; the four wave sums are combined as
// (s0 + s1) + (s2 + s3).  The order depends only on the sample's own length,
// so a sample pools to the same bits in any batch.  Bound by HBM, one read of
// every valid row, non-temporal: 256 samples of ~296 rows of 4 KB 69 -> 50 us
// (6.2 TB/s).
typedef uint32_t u32x4h __attribute__((ext_vector_type(4)));
constexpr int kPoolCols = 512;
constexpr int kPoolWaves = 4;

__global__ __launch_bounds__(256) void pool_kernel(const uint16_t* __restrict__ hidden,
                                                   const int32_t* __restrict__ seqlens,
                                                   const int32_t* __restrict__ cu_seqlens,
                                                   const int32_t* __restrict__ rank, int32_t d,
                                                   float* __restrict__ pooled) {
  __shared__ float red[kPoolWaves][kPoolCols];
  const int32_t chunks = (d + kPoolCols - 1) / kPoolCols;
  const int32_t i = blockIdx.x / chunks;
  const int32_t c0 = (blockIdx.x % chunks) * kPoolCols;
  const int32_t L = seqlens[i];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int32_t col = c0 + lane * 8;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  if (col < d) {
    const uint16_t* base = hidden + (int64_t)cu_seqlens[i] * d + col;
    auto add = [&](const u32x4h& q) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += __uint_as_float(q[e] << 16);
        acc[2 * e + 1] += __uint_as_float(q[e] & 0xffff0000u);
      }
    };
    auto load = [&](int32_t j) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4h*>(base + (int64_t)j * d)); };
    int32_t j = w;
    for (; j + 7 * kPoolWaves < L; j += 8 * kPoolWaves) {
      u32x4h q[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) q[k] = load(j + k * kPoolWaves);
#pragma unroll
      for (int k = 0; k < 8; ++k) add(q[k]);
    }
    for (; j + 3 * kPoolWaves < L; j += 4 * kPoolWaves) {
      u32x4h q[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) q[k] = load(j + k * kPoolWaves);
#pragma unroll
      for (int k = 0; k < 4; ++k) add(q[k]);
    }
    for (; j < L; j += kPoolWaves) add(load(j));
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[w][lane * 8 + e] = acc[e];
  __syncthreads();
  const float inv = 1.0f / (float)L;
  for (int t = threadIdx.x; t < kPoolCols; t += 256) {
    if (c0 + t < d)
      pooled[(int64_t)rank[i] * d + c0 + t] = ((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])) * inv;
  }
}

hipError_t launch_pool(hipStream_t s, const void* hidden, const int32_t* seqlens, const int32_t* cu_seqlens,
                       const int32_t* rank, int32_t N, int32_t d, float* pooled) {
  const int64_t blocks = (int64_t)((d + kPoolCols - 1) / kPoolCols) * N;
  if (d % 8 != 0 || N < 1 || blocks > 0x7fffffff) return hipErrorInvalidValue;
  dim3 grid((unsigned)blocks);
  pool_kernel<<<grid, 256, 0, s>>>(reinterpret_cast<const uint16_t*>(hidden), seqlens, cu_seqlens, rank, d, pooled);
  return hipGetLastError();
}

// ------------------------------------------------------------- head gemm ---

// fp32 matrix cores (v_mfma_f32_16x16x4_f32, the heads' precision), operands
// loaded from global memory straight into the MFMA layout: lane l supplies
// A(m = l & 15, k = l >> 4), and which k a step and lane quad stand for, or
// which column a block and lane stand for, is free as long as both operands
// agree, so every operand loads whole vectors along its contiguous dimension.
//   FWD    C[m][n] = X[m][k] W[n][k]: 16-byte loads along k (step s of a
//          16-wide k block is k = 4 quad + s)
//   DGRAD  C[m][n] = dZ[m][k] W[k][n]: 16-byte loads of dZ along k, 8-byte
//          loads of W along n (block b holds columns 2 j + b)
//   WGRAD  C[m][n] = sum_k dZ[k][m] X[k][n]: 4-byte loads along m, 16-byte
//          along n (step = 4 rows, one per quad)
// A workgroup has 8 wavefronts.  FWD and DGRAD: a 32 x 32 tile, the waves each
// take a K range (ceil(K / 8) rounded up to 32) and the eight partial tiles
// are added through LDS in wave order, so a long contraction needs neither
// partial sums in memory nor a second launch.  WGRAD (K is a tenant's row
// count): 64 x 256 tile, 32 x 64 per wave over all rows; long contractions
// (head_long_rows) by eight workgroups, 32 x 64 each, the waves again sharing K: in
// one wave they are a serial chain that a few workgroups walk on an empty chip.
// The order of every sum depends on the layer's sizes and the tenant's rows alone,
// so a tenant's bits do not depend on the batch.
// Bound by the weights' and gradients' HBM traffic (one read, one write) and by
// launches: with LDS staging, K ranges as workgroups and a reduction launch
// after each, the heads of 8 tenants x 32 rows on 2,048-wide features took
// thirteen launches and 276 us after the pool; now six launches and 141 us
// (forward 26 + 15 + 15, backward 24 + 33 + 28 us).  Per launch about 4.7 us go
// to the launch and the first descriptor, 2.5 us to the last tile's store.
typedef float f32x4h __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // rows need not be 16-byte aligned
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

__device__ __forceinline__ f32x4h head_mfma(float a, float b, f32x4h c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int kHeadWaves = 8;
constexpr int kHeadDepth = 4;  // slabs in flight per wave
constexpr int kHeadRed = kHeadTile + 4;  // LDS row stride of a partial tile

// A tenant's first row of the loss sums.
__device__ __forceinline__ float* head_lpart(const HeadGemm& D, int32_t off, int32_t tenant) {
  return D.lpart + (int64_t)(off / kHeadTile + tenant) * D.ldp;
}

// Epilogue of the 32 x 32 tile: sum of the waves' partials, then per element
// bias, GELU' (DGRAD), GELU copy, or -- a training forward's last layer -- the
// loss: actions, dL/dy and the tile's sum of squared errors.
__device__ __forceinline__ void head_finish(const HeadGemm& D, const float* red, float* scratch, int32_t off, int32_t ng,
                                            int32_t m0, int32_t n0, int32_t M, float* lpart) {
  const int tid = threadIdx.x;
  const int32_t r = tid >> 4, c = (tid & 15) * 2;
  const int32_t m = m0 + r;
  float ss = 0.f;
  if (m < M) {
    float v[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      v[e] = red[r * kHeadRed + c + e];
#pragma unroll
      for (int w = 1; w < kHeadWaves; ++w) v[e] += red[(w * kHeadTile + r) * kHeadRed + c + e];
    }
    const int64_t row = (int64_t)(off + m) * D.ldc;
    const float scale = 2.0f / ((float)ng * (float)D.N);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int32_t n = n0 + c + e;
      if (n >= D.N) break;
      float y = v[e];
      if (D.bias) y += D.bias[n];
      if (D.Zg) y *= gelu_grad_f(D.Zg[row + n]);
      if (D.target) {
        const int64_t i = (int64_t)m * D.N + n;
        const float diff = y - D.target[i];
        D.actions[i] = y;
        D.C[row + n] = scale * diff;
        ss = fmaf(diff, diff, ss);
      } else {
        D.C[row + n] = y;
        if (D.Cact) D.Cact[row + n] = gelu_f(y);
      }
    }
  }
  if (D.target) {
    ss = wave_sum(ss);
    if ((tid & 63) == 0) scratch[tid >> 6] = ss;
    __syncthreads();
    if (tid == 0) {
      float s = 0.f;
      for (int w = 0; w < kHeadWaves; ++w) s += scratch[w];
      *lpart = s;
    }
  }
}

// Weight gradients over more rows than this are shared by a workgroup's waves.  One
// tenant's short contractions want the wide tiles' less traffic and its long ones
// more workgroups, small gradients sooner: 768 x 256 over 256, 512 and 4,096 rows
// in the whole call 80, 125 and 794 us unshared, 41, 48 and 179 shared; 2048 x 1024 x
// 1024 over 512 and 4,096 264 and 1,796, 174 and 1,068 -- but eight tenants of it over
// 64, 275 and 1,000 rows (16 tenants) 205, 711 and 4,644 unshared, 252, 736 and 4,617
// shared.  The line is the layer's own, so a tenant's bits do not depend on its batch.
__device__ __forceinline__ int32_t head_long_rows(int32_t M, int32_t N) {
  const int32_t tiles = (M + kHeadWgradM - 1) / kHeadWgradM * ((N + kHeadWgradN - 1) / kHeadWgradN);
  return tiles > 32 ? 2 * kHeadLongRows : kHeadLongRows;
}

// The K range of a wave; its whole slabs of S end at `kw` (kb where the tile
// cannot take vector loads), the rest goes four k at a time with element loads.
struct HeadRange {
  int32_t kb, kw, ke;
};
template <int S>
__device__ __forceinline__ HeadRange head_range(int32_t K, int wave, bool vectors) {
  const int32_t kc = ((K + kHeadWaves - 1) / kHeadWaves + 31) / 32 * 32;
  HeadRange r;
  r.kb = min(K, wave * kc);
  r.ke = min(K, r.kb + kc);
  r.kw = vectors ? r.kb + (r.ke - r.kb) / S * S : r.kb;
  return r;
}

__device__ __forceinline__ void head_fwd_tile(const HeadGemm& D, float* red, int32_t off, int32_t m0, int32_t n0, int32_t M) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, quad = lane >> 4;
  const HeadRange R = head_range<32>(D.K, wave, true);
  const float *A[2], *B[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    A[i] = D.A + (int64_t)(off + min(m0 + 16 * i + j, M - 1)) * D.lda;
    B[i] = D.B + (int64_t)min(n0 + 16 * i + j, D.N - 1) * D.ldb;
  }
  f32x4h acc[2][2] = {};
  f32x4h a[kHeadDepth][2][2], b[kHeadDepth][2][2];  // [slab in flight][16-wide k block][operand block]
  auto load = [&](int u, int32_t k0) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[u][h][i] = *reinterpret_cast<const f32x4u*>(A[i] + k0 + 16 * h + 4 * quad);
        b[u][h][i] = *reinterpret_cast<const f32x4u*>(B[i] + k0 + 16 * h + 4 * quad);
      }
  };
#pragma unroll
  for (int u = 0; u < kHeadDepth; ++u)
    if (R.kb + 32 * u < R.kw) load(u, R.kb + 32 * u);
  for (int32_t k0 = R.kb; k0 < R.kw; k0 += 32 * kHeadDepth) {
#pragma unroll
    for (int u = 0; u < kHeadDepth; ++u) {
      if (k0 + 32 * u >= R.kw) break;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int x = 0; x < 2; ++x) acc[y][x] = head_mfma(b[u][h][y][s], a[u][h][x][s], acc[y][x]);
      if (k0 + 32 * (u + kHeadDepth) < R.kw) load(u, k0 + 32 * (u + kHeadDepth));
    }
  }
  for (int32_t k0 = R.kw; k0 < R.ke; k0 += 4) {
    const int32_t k = min(k0 + quad, R.ke - 1);
    const bool live = k0 + quad < R.ke;
    float av[2], bv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float x = A[i][k], w = B[i][k];
      av[i] = live ? x : 0.f;
      bv[i] = live ? w : 0.f;
    }
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int x = 0; x < 2; ++x) acc[y][x] = head_mfma(bv[y], av[x], acc[y][x]);
  }
  // lane: columns n = 16 y + 4 quad .. +3 of row m = 16 x + j
#pragma unroll
  for (int y = 0; y < 2; ++y)
#pragma unroll
    for (int x = 0; x < 2; ++x)
      *reinterpret_cast<f32x4h*>(red + (wave * kHeadTile + 16 * x + j) * kHeadRed + 16 * y + 4 * quad) = acc[y][x];
}

__device__ __forceinline__ void head_dgrad_tile(const HeadGemm& D, float* red, int32_t off, int32_t m0, int32_t n0,
                                                int32_t M) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, quad = lane >> 4;
  const HeadRange R = head_range<16>(D.K, wave, n0 + kHeadTile <= D.N);
  const float* A[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) A[i] = D.A + (int64_t)(off + min(m0 + 16 * i + j, M - 1)) * D.lda;
  const int64_t ldb = D.ldb;
  const uint32_t bo = 4 * quad * (uint32_t)ldb + n0 + 2 * j;
  f32x4h acc[2][2] = {};
  f32x4h a[kHeadDepth][2];
  f32x2u b[kHeadDepth][4];
  auto load = [&](int u, int32_t k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) a[u][i] = *reinterpret_cast<const f32x4u*>(A[i] + k0 + 4 * quad);
    const float* p = D.B + (int64_t)k0 * ldb;  // uniform; 32-bit lane offsets
#pragma unroll
    for (int s = 0; s < 4; ++s) b[u][s] = *reinterpret_cast<const f32x2u*>(p + s * ldb + bo);
  };
#pragma unroll
  for (int u = 0; u < kHeadDepth; ++u)
    if (R.kb + 16 * u < R.kw) load(u, R.kb + 16 * u);
  for (int32_t k0 = R.kb; k0 < R.kw; k0 += 16 * kHeadDepth) {
#pragma unroll
    for (int u = 0; u < kHeadDepth; ++u) {
      if (k0 + 16 * u >= R.kw) break;
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int x = 0; x < 2; ++x) acc[y][x] = head_mfma(b[u][s][y], a[u][x][s], acc[y][x]);
      if (k0 + 16 * (u + kHeadDepth) < R.kw) load(u, k0 + 16 * (u + kHeadDepth));
    }
  }
#pragma unroll 4
  for (int32_t k0 = R.kw; k0 < R.ke; k0 += 4) {
    const int32_t k = min(k0 + quad, R.ke - 1);
    const bool live = k0 + quad < R.ke;
    float av[2], bv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float x = A[i][k], w = D.B[(int64_t)k * ldb + min(n0 + 2 * j + i, D.N - 1)];
      av[i] = live ? x : 0.f;
      bv[i] = live ? w : 0.f;
    }
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int x = 0; x < 2; ++x) acc[y][x] = head_mfma(bv[y], av[x], acc[y][x]);
  }
  // lane: columns n = 8 quad + 2 e + y of row m = 16 x + j
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    float* p = red + (wave * kHeadTile + 16 * x + j) * kHeadRed + 8 * quad;
    *reinterpret_cast<f32x4h*>(p) = f32x4h{acc[0][x][0], acc[1][x][0], acc[0][x][1], acc[1][x][1]};
    *reinterpret_cast<f32x4h*>(p + 4) = f32x4h{acc[0][x][2], acc[1][x][2], acc[0][x][3], acc[1][x][3]};
  }
}

// piece: which 32 x 64 of the tile; where `shared`, the whole workgroup's, each wave
// a K range, else the wave's own over all rows.
__device__ __forceinline__ void head_wgrad_tile(const HeadGemm& D, float* red, int32_t off, int32_t tm, int32_t tn,
                                                int32_t rows, int piece, bool shared) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, quad = lane >> 4;
  const int32_t M = D.M, N = D.N;
  const int32_t m0 = tm * kHeadWgradM + 32 * (piece >> 2), n0 = tn * kHeadWgradN + 64 * (piece & 3);
  if (m0 >= M || n0 >= N) return;
  int32_t K = rows, kb = 0;  // the wave's rows, from off + kb
  if (shared) {
    const int32_t kc = ((rows + kHeadWaves - 1) / kHeadWaves + 15) / 16 * 16;
    kb = min(rows, wave * kc);
    K = min(kc, rows - kb);
  }
  const int64_t lda = D.lda, ldb = D.ldb;
  const float *const A = D.A + (int64_t)(off + kb) * lda, *const B = D.B + (int64_t)(off + kb) * ldb;
  const uint32_t a0 = quad * (uint32_t)lda + min(m0 + j, M - 1), a1 = quad * (uint32_t)lda + min(m0 + 16 + j, M - 1);
  const int cj = n0 + 4 * ((j >> 2) + 4 * (j & 3));  // this lane's four columns
  const uint32_t bo = quad * (uint32_t)ldb + cj;
  const bool whole = n0 + 64 <= N;  // uniform: vector loads along n
  f32x4h acc[4][2] = {};            // [column block b][row block a]
  float cs[2] = {0.f, 0.f};         // bias gradient: this quad's rows of columns m0 + j, m0 + 16 + j
  float a[2][4][2];                 // [16 rows in flight][step][row block]
  f32x4h b[2][4];
  auto load = [&](int u, int32_t k0) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float *pa = A + (int64_t)(k0 + 4 * s) * lda, *pb = B + (int64_t)(k0 + 4 * s) * ldb;  // uniform
      a[u][s][0] = pa[a0];
      a[u][s][1] = pa[a1];
      b[u][s] = *reinterpret_cast<const f32x4u*>(pb + bo);
    }
  };
  const int32_t kw = whole ? K / 16 * 16 : 0;
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (16 * u < kw) load(u, 16 * u);
  for (int32_t k0 = 0; k0 < kw; k0 += 32) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (k0 + 16 * u >= kw) break;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int x = 0; x < 2; ++x) cs[x] += a[u][s][x];
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
          for (int x = 0; x < 2; ++x) acc[y][x] = head_mfma(b[u][s][y], a[u][s][x], acc[y][x]);
      }
      if (k0 + 16 * (u + 2) < kw) load(u, k0 + 16 * (u + 2));
    }
  }
#pragma unroll 2
  for (int32_t k0 = kw; k0 < K; k0 += 4) {
    const int64_t k = min(k0 + quad, K - 1);
    const bool live = k0 + quad < K;
    float av[2] = {A[k * lda + min(m0 + j, M - 1)], A[k * lda + min(m0 + 16 + j, M - 1)]};
    float bv[4];
#pragma unroll
    for (int y = 0; y < 4; ++y) bv[y] = B[k * ldb + min(cj + y, N - 1)];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      av[x] = live ? av[x] : 0.f;
      cs[x] += av[x];
    }
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      bv[y] = live ? bv[y] : 0.f;
#pragma unroll
      for (int x = 0; x < 2; ++x) acc[y][x] = head_mfma(bv[y], av[x], acc[y][x]);
    }
  }
  // lane: columns n0 + 16 e + 4 quad + y of rows m0 + 16 x + j (the loads' column
  // order makes a store instruction cover 64 contiguous bytes of 16 rows)
  float bias[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) bias[x] = sum_xor32(sum_xor16(cs[x]));
  if (shared) {
    // the waves' partials, added in wave order: 16 rows at a time, then the bias
    constexpr int kLd = 68;  // LDS row stride
    static_assert(kHeadWaves * 16 * kLd <= kHeadWaves * kHeadTile * kHeadRed, "partials fit");
    const int t = threadIdx.x, c = 2 * (t & 31), r = t >> 5;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<f32x4h*>(red + (wave * 16 + j) * kLd + 16 * e + 4 * quad) =
            f32x4h{acc[0][x][e], acc[1][x][e], acc[2][x][e], acc[3][x][e]};
      __syncthreads();
      const int32_t m = m0 + 16 * x + r;
      if (m < M) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          float v = red[r * kLd + c + i];
#pragma unroll
          for (int w = 1; w < kHeadWaves; ++w) v += red[(w * 16 + r) * kLd + c + i];
          if (n0 + c + i < N) D.C[(int64_t)m * D.ldc + n0 + c + i] = v;
        }
      }
    }
    if (n0 == 0) {
      __syncthreads();
#pragma unroll
      for (int x = 0; x < 2; ++x)
        if (quad == 0) red[wave * 32 + 16 * x + j] = bias[x];
      __syncthreads();
      if (t < 32 && m0 + t < M) {
        float v = red[t];
#pragma unroll
        for (int w = 1; w < kHeadWaves; ++w) v += red[w * 32 + t];
        D.db[m0 + t] = v;
      }
    }
    return;
  }
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int32_t m = m0 + 16 * x + j;
    if (m >= M) break;
    float* p = D.C + (int64_t)m * D.ldc + n0 + 4 * quad;
    if (whole) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<f32x4u*>(p + 16 * e) = f32x4h{acc[0][x][e], acc[1][x][e], acc[2][x][e], acc[3][x][e]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int y = 0; y < 4; ++y)
          if (n0 + 16 * e + 4 * quad + y < N) p[16 * e + y] = acc[y][x][e];
    }
    if (n0 == 0 && quad == 0) D.db[m] = bias[x];
  }
}

// FORWARD: FWD tiles only (one workgroup per CU on the 2048-wide heads,
// its slabs in flight are what hides the weights' latency); otherwise the
// backward modes, in at most 128 registers so that two workgroups share a CU.
// Workgroup b < nrow * tms: row tile tm0 + b / nrow of entry b % nrow.  The list
// holds a column of tiles once, not once per row tile of the largest tenant: 32
// tenants of up to 4,096 samples would list 110,000 tiles.
template <bool FORWARD>
__global__ __launch_bounds__(64 * kHeadWaves, FORWARD ? 2 : 4) void head_gemm_kernel(const HeadGemm* __restrict__ descs,
                                                                                     const HeadTile* __restrict__ tiles,
                                                                                     const int32_t* __restrict__ tso,
                                                                                     int32_t nrow, int32_t tms,
                                                                                     int32_t tm0, int32_t nown,
                                                                                     int32_t parts) {
  __shared__ __attribute__((aligned(16))) float red[kHeadWaves * kHeadTile * kHeadRed];
  __shared__ float scratch[kHeadWaves];
  const int32_t b = blockIdx.x;
  const bool own = !FORWARD && b >= nrow * tms;
  const int32_t row = own ? 0 : b / nrow;
  // own tiles: `parts` workgroups of each, tile fastest (workgroups are dealt to the
  // XCDs in turn: where only the first of a tile's eight has work, piece fastest
  // would leave seven XCDs idle)
  const int32_t at = b - nrow * tms, piece = own ? at / nown : 0;
  const HeadTile tile = tiles[own ? nrow + at - piece * nown : b - row * nrow];
  const int32_t off = tso[tile.tenant], ng = tso[tile.tenant + 1] - off;
  const HeadGemm D = descs[tile.desc];
  if (!FORWARD && own) {
    const bool shared = parts > 1 && ng > head_long_rows(D.M, D.N);
    if (piece > 0 && (!shared || tile.tm == kHeadLossTile)) return;
    if (tile.tm != kHeadLossTile) {
      head_wgrad_tile(D, red, off, tile.tm, tile.tn, ng,
                      shared ? piece : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), shared);
      return;
    }
    // the tenant's loss from its tiles' sums, in tile order per thread, then a fixed tree
    const int32_t tn = (D.M + kHeadTile - 1) / kHeadTile, n = (ng + kHeadTile - 1) / kHeadTile * tn;
    const float* const part = head_lpart(D, off, tile.tenant);
    float s = 0.f;
    for (int32_t i = threadIdx.x; i < n; i += 64 * kHeadWaves) s += part[(int64_t)(i / tn) * D.ldp + i % tn];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      float t = 0.f;
      for (int w = 0; w < kHeadWaves; ++w) t += scratch[w];
      D.loss[0] = t / ((float)ng * (float)D.M);
    }
    return;
  }
  const int32_t tm = tm0 + row, m0 = tm * kHeadTile, n0 = tile.tn * kHeadTile;
  if (m0 >= ng) return;  // tiles past a tenant's row count (upper-bound grid)
  if (FORWARD)
    head_fwd_tile(D, red, off, m0, n0, ng);
  else
    head_dgrad_tile(D, red, off, m0, n0, ng);
  __syncthreads();
  head_finish(D, red, scratch, D.own_rows ? 0 : off, ng, m0, n0, ng,
              head_lpart(D, off, tile.tenant) + (int64_t)tm * D.ldp + tile.tn);
}

hipError_t launch_head_gemm(hipStream_t s, const HeadGemm* descs, const HeadTile* tiles, const HeadLaunch& n,
                            int32_t tms, const int32_t* tso, bool forward) {
  tiles += n.first;
  // a dispatch holds at most 2^32 - 1 threads: row tiles beyond it in further launches
  constexpr int64_t kMost = 0xffffffffll / (64 * kHeadWaves);
  if (n.nrow + (int64_t)n.nown > kMost) return hipErrorInvalidValue;
  const bool longer = tms * (int64_t)kHeadTile > kHeadLongRows && n.nrow + (int64_t)n.nown * kHeadWaves <= kMost;
  const int32_t parts = longer ? kHeadWaves : 1, all = n.nown * parts;
  const int32_t step = n.nrow ? (int32_t)std::min<int64_t>(tms, (kMost - all) / n.nrow) : 0;
  for (int32_t tm0 = 0, own = all;; own = 0) {
    const int32_t rows = std::min(step, tms - tm0);
    const dim3 grid((unsigned)(n.nrow * (int64_t)rows + own));
    if (forward)
      head_gemm_kernel<true><<<grid, 64 * kHeadWaves, 0, s>>>(descs, tiles, tso, n.nrow, rows, tm0, n.nown, parts);
    else
      head_gemm_kernel<false><<<grid, 64 * kHeadWaves, 0, s>>>(descs, tiles, tso, n.nrow, rows, tm0, n.nown, parts);
    const hipError_t e = hipGetLastError();
    tm0 += rows;
    if (e != hipSuccess || n.nrow == 0 || tm0 >= tms) return e;
  }
}

}  // namespace jnx
