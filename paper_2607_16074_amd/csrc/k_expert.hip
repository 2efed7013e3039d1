// Kernels of the tenant-private action expert (forward, loss, weight
// gradients).  GEMMs go through the grouped bf16 GEMM (k_gemm.hip); this file
// holds the rest:
//   copy2d       grouped strided 2-D copy with zero padding and fp32 <-> bf16
//                conversion (operand padding, bf16 rounding points, saves)
//   ksum         ordered sum of the K-range partials of a split weight gradient
//   transpose    grouped bf16 transpose with zero-padded columns (operands of
//                the data- and weight-gradient GEMMs where they cannot be read
//                transposed in place)
//   prefix       tenant-ordered copy of every sample's valid backbone rows
//   rmsnorm      per-tenant-gain RMSNorm forward (fp32 -> bf16) and backward
//                (fp32 and its bf16 copy), gain gradients by fixed-order sums
//   attention    self- / cross-attention forward and backward on the bf16
//                matrix cores, per (sample, head); a sample's queries never
//                see another sample's keys
//   loss         per-tenant mean squared error and its gradient
#include <algorithm>

#include "jn_device.h"
#include "jn_internal.h"

namespace jnx {

// ---------------------------------------------------------------- copy2d ---
// Each block covers 2048 elements of one descriptor (row-major over rows x
// cols).  Descriptors whose columns, leading dimensions and source width are
// multiples of 4 move 4 elements per thread step (16-byte fp32 / 8-byte bf16
// accesses); the rest go element by element.

__device__ __forceinline__ void copy4_load(const CopyDesc& D, int64_t r, int64_t c, float (&v)[4]) {
  if (r < D.src_rows && c < D.src_cols) {
    const int64_t si = r * D.src_ld + c;
    if (D.src_bf16) {
      const uint2 u = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(D.src) + si);
      v[0] = __uint_as_float(u.x << 16);
      v[1] = __uint_as_float(u.x & 0xffff0000u);
      v[2] = __uint_as_float(u.y << 16);
      v[3] = __uint_as_float(u.y & 0xffff0000u);
    } else {
      const float4 f = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(D.src) + si);
      v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
    }
  } else {
    v[0] = v[1] = v[2] = v[3] = 0.f;
  }
}

__global__ __launch_bounds__(256) void copy2d_kernel(const CopyDesc* __restrict__ descs, int32_t ndesc) {
  int32_t p = 0;
  const int32_t b = blockIdx.x;
  while (p + 1 < ndesc && descs[p + 1].block_start <= b) ++p;
  const CopyDesc D = descs[p];
  const int64_t total = (int64_t)D.rows * D.cols;
  const int64_t base = (int64_t)(b - D.block_start) * 256 * 8;
  const bool vec = D.vec != 0;
  if (vec) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int64_t e = base + ((int64_t)k * 256 + threadIdx.x) * 4;
      if (e >= total) break;
      const int64_t r = e / D.cols, c = e % D.cols;
      float v[4];
      copy4_load(D, r, c, v);
      const int64_t di = r * D.dst_ld + c;
      if (D.dst_bf16)
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(D.dst) + di) =
            make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
      else
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(D.dst) + di) = make_float4(v[0], v[1], v[2], v[3]);
    }
    return;
  }
  for (int k = 0; k < 8; ++k) {
    const int64_t e = base + (int64_t)k * 256 + threadIdx.x;
    if (e >= total) break;
    const int64_t r = e / D.cols, c = e % D.cols;
    float v = 0.f;
    if (r < D.src_rows && c < D.src_cols) {
      const int64_t si = r * D.src_ld + c;
      v = D.src_bf16 ? bf2f(reinterpret_cast<const uint16_t*>(D.src)[si]) : reinterpret_cast<const float*>(D.src)[si];
    }
    const int64_t di = r * D.dst_ld + c;
    if (D.dst_bf16)
      reinterpret_cast<uint16_t*>(D.dst)[di] = f2bf(v);
    else
      reinterpret_cast<float*>(D.dst)[di] = v;
  }
}

int32_t copy2d_prepare(CopyDesc* d, int32_t n) {
  int32_t total = 0;
  for (int32_t i = 0; i < n; ++i) {
    const CopyDesc& D = d[i];
    const bool vec = D.cols % 4 == 0 && D.src_ld % 4 == 0 && D.dst_ld % 4 == 0 &&
                     (D.src_cols % 4 == 0 || D.src_cols >= D.cols) &&
                     (D.src == nullptr || reinterpret_cast<uintptr_t>(D.src) % 16 == 0) &&
                     reinterpret_cast<uintptr_t>(D.dst) % 16 == 0;
    d[i].vec = vec ? 1 : 0;
    d[i].block_start = total;
    // vector descriptors: 2048 elements per block as 512 threads-steps of 4
    total += (int32_t)(((int64_t)D.rows * D.cols + 2047) / 2048);
  }
  return total;
}

hipError_t launch_copy2d(hipStream_t s, const CopyDesc* d, int32_t n, int32_t blocks) {
  if (blocks <= 0) return hipSuccess;
  copy2d_kernel<<<blocks, 256, 0, s>>>(d, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------ ksum ---
// One block per 4096 elements of a descriptor (a thread sums 4 x 4 columns).
__global__ __launch_bounds__(256) void ksum_kernel(const KSumDesc* __restrict__ descs, int32_t ndesc) {
  const int32_t b = blockIdx.x;
  int32_t i = 0;
  while (i + 1 < ndesc && descs[i + 1].block_start <= b) ++i;
  const KSumDesc D = descs[i];
  const int64_t base = (int64_t)(b - D.block_start) * 4096;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t e = base + ((int64_t)k * 256 + threadIdx.x) * 4;
    if (e >= D.n) break;
    float4 acc = *reinterpret_cast<const float4*>(D.src + e);
    for (int32_t r = 1; r < D.S; ++r) {
      const float4 v = *reinterpret_cast<const float4*>(D.src + r * D.n + e);
      acc.x += v.x;
      acc.y += v.y;
      acc.z += v.z;
      acc.w += v.w;
    }
    *reinterpret_cast<float4*>(D.dst + e) = acc;
  }
}

int32_t ksum_prepare(KSumDesc* d, int32_t n) {
  int32_t total = 0;
  for (int32_t i = 0; i < n; ++i) {
    if (d[i].n <= 0 || d[i].n % 4 != 0 || d[i].S < 1 || reinterpret_cast<uintptr_t>(d[i].src) % 16 != 0 ||
        reinterpret_cast<uintptr_t>(d[i].dst) % 16 != 0)
      return -1;
    d[i].block_start = total;
    total += (int32_t)((d[i].n + 4095) / 4096);
  }
  return total;
}

hipError_t launch_ksum(hipStream_t s, const KSumDesc* d, int32_t n, int32_t blocks) {
  if (blocks <= 0 || n <= 0) return hipSuccess;
  ksum_kernel<<<blocks, 256, 0, s>>>(d, n);
  return hipGetLastError();
}

// ------------------------------------------------------------- transpose ---
// dst[c][r] = src[r][c] for r < rows, 0 for rows <= r < rows_pad; 64x64 tiles.
// Tiles that lie wholly inside the source (and whose leading dimensions are
// multiples of 8) move 16 bytes per thread access; edge tiles go element by
// element.

__global__ __launch_bounds__(256) void transpose_kernel(const TransDesc* __restrict__ descs, int32_t ndesc) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[64][72];
  int32_t p = 0;
  const int32_t b = blockIdx.x;
  while (p + 1 < ndesc && descs[p + 1].block_start <= b) ++p;
  const TransDesc D = descs[p];
  const int32_t tcols = (D.cols + 63) / 64;
  const int32_t local = b - D.block_start;
  const int32_t r0 = (local / tcols) * 64, c0 = (local % tcols) * 64;
  const bool full = r0 + 64 <= D.rows && c0 + 64 <= D.cols && D.src_ld % 8 == 0 && D.dst_ld % 8 == 0 &&
                    r0 + 64 <= D.rows_pad && reinterpret_cast<uintptr_t>(D.src) % 16 == 0 &&
                    reinterpret_cast<uintptr_t>(D.dst) % 16 == 0;
  if (full) {
    // load: thread t takes row t >> 2, columns 16*(t & 3) .. +15
    const int rr = threadIdx.x >> 2, cc = 16 * (threadIdx.x & 3);
    const uint4* sp = reinterpret_cast<const uint4*>(D.src + (int64_t)(r0 + rr) * D.src_ld + c0 + cc);
    *reinterpret_cast<uint4*>(&tile[rr][cc]) = sp[0];
    *reinterpret_cast<uint4*>(&tile[rr][cc + 8]) = sp[1];
    __syncthreads();
    // store: thread t writes output row (input column) t >> 2, outputs 16*(t & 3) .. +15
    uint32_t o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (uint32_t)tile[cc + 2 * i][rr] | ((uint32_t)tile[cc + 2 * i + 1][rr] << 16);
    uint4* dp = reinterpret_cast<uint4*>(D.dst + (int64_t)(c0 + rr) * D.dst_ld + r0 + cc);
    dp[0] = make_uint4(o[0], o[1], o[2], o[3]);
    dp[1] = make_uint4(o[4], o[5], o[6], o[7]);
    return;
  }
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int32_t r = r0 + i, c = c0 + tx;
    uint16_t v = 0;
    if (r < D.rows && c < D.cols) v = D.src[(int64_t)r * D.src_ld + c];
    tile[i][tx] = v;
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int32_t c = c0 + i, r = r0 + tx;
    if (c < D.cols && r < D.rows_pad) D.dst[(int64_t)c * D.dst_ld + r] = tile[tx][i];
  }
}

int32_t transpose_prepare(TransDesc* d, int32_t n) {
  int32_t total = 0;
  for (int32_t i = 0; i < n; ++i) {
    d[i].block_start = total;
    total += ((d[i].rows_pad + 63) / 64) * ((d[i].cols + 63) / 64);
  }
  return total;
}

hipError_t launch_transpose(hipStream_t s, const TransDesc* d, int32_t n, int32_t blocks) {
  if (blocks <= 0) return hipSuccess;
  transpose_kernel<<<blocks, 256, 0, s>>>(d, n);
  return hipGetLastError();
}

// ----------------------------------------------------------------- prefix ---
// zoff[k] (k in tenant order) = row of the tenant-ordered prefix buffer where
// sample tenant_perm[k]'s valid backbone rows start; zoff[N] = total rows.

__global__ __launch_bounds__(256) void prefix_offsets_kernel(const int32_t* __restrict__ tenant_perm,
                                                            const int32_t* __restrict__ seqlens, int32_t N,
                                                            int32_t* __restrict__ zoff) {
  __shared__ int32_t part[256];
  const int per = (N + 255) / 256;
  const int k0 = threadIdx.x * per;
  int32_t s = 0;
  for (int k = k0; k < min(N, k0 + per); ++k) s += seqlens[tenant_perm[k]];
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t run = 0;
    for (int t = 0; t < 256; ++t) {
      const int32_t v = part[t];
      part[t] = run;
      run += v;
    }
  }
  __syncthreads();
  int32_t run = part[threadIdx.x];
  for (int k = k0; k < min(N, k0 + per); ++k) {
    zoff[k] = run;
    run += seqlens[tenant_perm[k]];
  }
  if (threadIdx.x == 255) zoff[N] = run;
}

// Copy each sample's rows, one contiguous run on both sides: a block moves 512
// consecutive 16-byte chunks at a time, `per` blocks per sample (consecutive
// ones, and the reads non-temporal, as measured for the pack kernel: 288 samples
// of ~600 rows of 1.5 KB 94 -> 80 us).  Rows past `cap` are dropped so an
// inconsistent caller row count cannot overflow.
constexpr int kPrefixRun = 512;
typedef uint32_t u32x4x __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void prefix_gather_kernel(const uint16_t* __restrict__ hidden,
                                                           const int32_t* __restrict__ tenant_perm,
                                                           const int32_t* __restrict__ seqlens,
                                                           const int32_t* __restrict__ cu_seqlens,
                                                           const int32_t* __restrict__ zoff, int32_t d, int64_t cap,
                                                           uint16_t* __restrict__ z, int32_t per) {
  const int32_t k = blockIdx.x / per, part = blockIdx.x % per;
  const int32_t i = tenant_perm[k];
  const int64_t chunks = d / 8, at = zoff[k];
  const int64_t n = min((int64_t)seqlens[i], cap - at) * chunks;
  const u32x4x* src = reinterpret_cast<const u32x4x*>(hidden) + cu_seqlens[i] * chunks;
  u32x4x* dst = reinterpret_cast<u32x4x*>(z) + at * chunks;
  for (int64_t e = (int64_t)part * kPrefixRun + threadIdx.x; e < n; e += (int64_t)per * kPrefixRun) {
    const bool two = e + 256 < n;
    const u32x4x a = __builtin_nontemporal_load(src + e);
    if (two) {
      const u32x4x b = __builtin_nontemporal_load(src + e + 256);
      dst[e + 256] = b;
    }
    dst[e] = a;
  }
}

// The same over consecutive chunks of the prefix buffer, whichever samples they
// belong to (as the ragged walk of the pack kernel).
__global__ __launch_bounds__(256) void prefix_ragged_kernel(const uint16_t* __restrict__ hidden,
                                                           const int32_t* __restrict__ tenant_perm,
                                                           const int32_t* __restrict__ cu_seqlens,
                                                           const int32_t* __restrict__ zoff, int32_t N, int32_t d,
                                                           int64_t cap, uint16_t* __restrict__ z) {
  const int64_t chunks = d / 8, all = min((int64_t)zoff[N], cap) * chunks;
  for (int64_t at = (int64_t)blockIdx.x * kPrefixRun; at < all; at += (int64_t)gridDim.x * kPrefixRun) {
    const int64_t n = min((int64_t)kPrefixRun, all - at);
    const int32_t ra = (int32_t)(at / chunks), rb = (int32_t)((at + n - 1) / chunks);
    const int32_t ka = last_at(zoff, N, ra), kb = ka + last_at(zoff + ka, min(N - ka, rb - ra + 1), rb);
    const uint32_t c0 = (uint32_t)(at - ra * chunks);
    for (int64_t e = threadIdx.x; e < n; e += 256) {
      const uint32_t r = (c0 + (uint32_t)e) / (uint32_t)chunks, c = c0 + (uint32_t)e - r * (uint32_t)chunks;
      const int32_t row = ra + (int32_t)r, k = ka + last_at(zoff + ka, kb - ka + 1, row);
      const int64_t src = cu_seqlens[tenant_perm[k]] + (row - zoff[k]);
      reinterpret_cast<u32x4x*>(z)[at + e] =
          __builtin_nontemporal_load(reinterpret_cast<const u32x4x*>(hidden) + src * chunks + c);
    }
  }
}

hipError_t launch_prefix(hipStream_t s, const void* hidden, const int32_t* tenant_perm, const int32_t* seqlens,
                         const int32_t* cu_seqlens, int32_t N, int32_t max_seqlen, int32_t d, int64_t cap,
                         int32_t* zoff, void* z) {
  prefix_offsets_kernel<<<1, 256, 0, s>>>(tenant_perm, seqlens, N, zoff);
  const int64_t chunks = d / 8;
  const int32_t per = spread_blocks(max_seqlen * chunks, cap * chunks, N, kPrefixRun);
  if (per == 0) {
    const unsigned blocks = (unsigned)std::min<int64_t>((cap * chunks + kPrefixRun - 1) / kPrefixRun, kMostBlocks);
    prefix_ragged_kernel<<<blocks, 256, 0, s>>>(reinterpret_cast<const uint16_t*>(hidden), tenant_perm, cu_seqlens, zoff,
                                                N, d, cap, reinterpret_cast<uint16_t*>(z));
    return hipGetLastError();
  }
  prefix_gather_kernel<<<dim3((unsigned)N * per), 256, 0, s>>>(reinterpret_cast<const uint16_t*>(hidden), tenant_perm,
                                                               seqlens, cu_seqlens, zoff, d, cap,
                                                               reinterpret_cast<uint16_t*>(z), per);
  return hipGetLastError();
}

// ---------------------------------------------------------------- rmsnorm ---
// Rows are tenant-contiguous: tenant t owns rows [roff[t], roff[t+1]) and its
// gain is gains[t] (bf16 [d]).  One wavefront per row, d = 64 * 4 * NC.

__device__ __forceinline__ int32_t row_tenant(const int32_t* roff, int32_t G, int32_t row) {
  int32_t t = 0;
  while (t + 1 < G && roff[t + 1] <= row) ++t;
  return t;
}

template <int NC>
__global__ __launch_bounds__(256) void xrms_fwd_kernel(const float* __restrict__ x, const uint16_t* const* __restrict__ gains,
                                                      const int32_t* __restrict__ roff, int32_t G, int32_t rows,
                                                      int32_t d, float eps, uint16_t* __restrict__ h) {
  const int lane = threadIdx.x & 63;
  const int32_t row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const uint16_t* g = gains[row_tenant(roff, G, row)];
  float v[NC][4];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const float4 q = *reinterpret_cast<const float4*>(x + (int64_t)row * d + (c * 64 + lane) * 4);
    v[c][0] = q.x; v[c][1] = q.y; v[c][2] = q.z; v[c][3] = q.w;
#pragma unroll
    for (int k = 0; k < 4; ++k) ss += v[c][k] * v[c][k];
  }
  ss = wave_sum(ss);
  const float r = rsqrtf(ss / (float)d + eps);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int e = (c * 64 + lane) * 4;
    const uint2 gq = *reinterpret_cast<const uint2*>(g + e);
    const float g0 = __uint_as_float(gq.x << 16), g1 = __uint_as_float(gq.x & 0xffff0000u);
    const float g2 = __uint_as_float(gq.y << 16), g3 = __uint_as_float(gq.y & 0xffff0000u);
    *reinterpret_cast<uint2*>(h + (int64_t)row * d + e) =
        make_uint2(pack_bf2(v[c][0] * r * g0, v[c][1] * r * g1), pack_bf2(v[c][2] * r * g2, v[c][3] * r * g3));
  }
}

// dx (+)= r g dh - x r^3 (sum_j g_j dh_j x_j) / d, its bf16 copy (the operand
// of the next block's gradient GEMMs), and the gain gradient's column sums of
// dh_j x_j r.  Workgroup = one segment of kXrmsSeg rows of one tenant, wave w
// rows w, w + 4 of it; the four waves' column sums are added in order and
// written as the segment's partial row.  HBM-bound (22 B per element): the sums
// used to go through a [rows][d] buffer (8 B per element more, and a summing
// launch of 64 workgroups): 14,400 x 1024 46 + 38 + 15 us (with the separate
// bf16 copy) -> 46 + 6 us.
template <int NC>
__global__ __launch_bounds__(256) void xrms_bwd_kernel(const float* __restrict__ x, const uint16_t* const* __restrict__ gains,
                                                      const int32_t* __restrict__ roff, const int32_t* __restrict__ soff,
                                                      int32_t G, int32_t d, float eps, const float* __restrict__ dh,
                                                      bool first, float* __restrict__ dx, uint16_t* __restrict__ dxb,
                                                      float* __restrict__ part) {
  __shared__ float red[4][NC * 256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int32_t b = blockIdx.x, t = row_tenant(soff, G, b);
  const int32_t r0 = roff[t] + (b - soff[t]) * kXrmsSeg, r1 = min(r0 + kXrmsSeg, roff[t + 1]);
  const uint16_t* g = gains[t];
  float gg[NC][4], cs[NC][4];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const uint2 gq = *reinterpret_cast<const uint2*>(g + (c * 64 + lane) * 4);
    gg[c][0] = __uint_as_float(gq.x << 16);
    gg[c][1] = __uint_as_float(gq.x & 0xffff0000u);
    gg[c][2] = __uint_as_float(gq.y << 16);
    gg[c][3] = __uint_as_float(gq.y & 0xffff0000u);
#pragma unroll
    for (int k = 0; k < 4; ++k) cs[c][k] = 0.f;
  }
  for (int32_t row = r0 + w; row < r1; row += 4) {
    float xv[NC][4], dv[NC][4], ov[NC][4];
    float ss = 0.f, dot = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int64_t e = (int64_t)row * d + (c * 64 + lane) * 4;
      const float4 q = *reinterpret_cast<const float4*>(x + e);
      const float4 u = *reinterpret_cast<const float4*>(dh + e);
      const float4 o = first ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<const float4*>(dx + e);
      xv[c][0] = q.x; xv[c][1] = q.y; xv[c][2] = q.z; xv[c][3] = q.w;
      dv[c][0] = u.x; dv[c][1] = u.y; dv[c][2] = u.z; dv[c][3] = u.w;
      ov[c][0] = o.x; ov[c][1] = o.y; ov[c][2] = o.z; ov[c][3] = o.w;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        ss += xv[c][k] * xv[c][k];
        dot += gg[c][k] * dv[c][k] * xv[c][k];
      }
    ss = wave_sum(ss);
    dot = wave_sum(dot);
    const float r = rsqrtf(ss / (float)d + eps);
    const float coef = r * r * r * dot / (float)d;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int64_t e = (int64_t)row * d + (c * 64 + lane) * 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        ov[c][k] += r * (gg[c][k] * dv[c][k]) - xv[c][k] * coef;
        cs[c][k] += dv[c][k] * xv[c][k] * r;
      }
      *reinterpret_cast<float4*>(dx + e) = make_float4(ov[c][0], ov[c][1], ov[c][2], ov[c][3]);
      *reinterpret_cast<uint2*>(dxb + e) = make_uint2(pack_bf2(ov[c][0], ov[c][1]), pack_bf2(ov[c][2], ov[c][3]));
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    *reinterpret_cast<float4*>(&red[w][(c * 64 + lane) * 4]) = make_float4(cs[c][0], cs[c][1], cs[c][2], cs[c][3]);
  __syncthreads();
  for (int j = threadIdx.x; j < NC * 256; j += 256)
    part[(int64_t)b * d + j] = (red[0][j] + red[1][j]) + (red[2][j] + red[3][j]);
}

// dg_t[j] = sum of tenant t's segment partials, of every norm of the step in
// one launch (z: norm n's partials at n * stride, its pointers at out + n G;
// one launch per norm cost 4.5 us each): block = (tenant, 64 columns), wave w
// adds segments w, w + 4, .. in order, then the four sums in order.
__global__ __launch_bounds__(256) void colsum_final_kernel(const float* __restrict__ part, const int32_t* __restrict__ soff,
                                                           float* const* __restrict__ out, int32_t d) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int32_t t = blockIdx.x, j = blockIdx.y * 64 + lane, G = gridDim.x;
  part += (int64_t)blockIdx.z * soff[G] * d;
  out += (int64_t)blockIdx.z * G;
  float s = 0.f;
#pragma unroll 8
  for (int32_t b = soff[t] + w; b < soff[t + 1]; b += 4) s += part[(int64_t)b * d + j];
  red[w][lane] = s;
  __syncthreads();
  if (w == 0) out[t][j] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

hipError_t launch_xrms_fwd(hipStream_t s, const float* x, const void* const* gains, const int32_t* roff, int32_t G,
                           int32_t rows, int32_t d, float eps, void* h) {
  dim3 grid((rows + 3) / 4);
  auto gp = reinterpret_cast<const uint16_t* const*>(gains);
  auto hp = reinterpret_cast<uint16_t*>(h);
  switch (d) {
    case 256: xrms_fwd_kernel<1><<<grid, 256, 0, s>>>(x, gp, roff, G, rows, d, eps, hp); break;
    case 512: xrms_fwd_kernel<2><<<grid, 256, 0, s>>>(x, gp, roff, G, rows, d, eps, hp); break;
    case 1024: xrms_fwd_kernel<4><<<grid, 256, 0, s>>>(x, gp, roff, G, rows, d, eps, hp); break;
    case 2048: xrms_fwd_kernel<8><<<grid, 256, 0, s>>>(x, gp, roff, G, rows, d, eps, hp); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_xrms_bwd(hipStream_t s, const float* x, const void* const* gains, const int32_t* roff,
                           const int32_t* soff, int32_t G, int32_t segs, int32_t d, float eps, const float* dh,
                           bool first, float* dx, uint16_t* dxb, float* part) {
  auto gp = reinterpret_cast<const uint16_t* const*>(gains);
#define JN_XRMS(NC) \
  case 256 * NC:    \
    xrms_bwd_kernel<NC><<<segs, 256, 0, s>>>(x, gp, roff, soff, G, d, eps, dh, first, dx, dxb, part); break;
  switch (d) {
    JN_XRMS(1)
    JN_XRMS(2)
    JN_XRMS(4)
    JN_XRMS(8)
    default: return hipErrorInvalidValue;
  }
#undef JN_XRMS
  return hipGetLastError();
}

hipError_t launch_gain_sums(hipStream_t s, const float* part, const int32_t* soff, int32_t G, int32_t segs, int32_t d,
                            int32_t norms, float* const* dg) {
  for (int32_t n = 0; n < norms; n += 65535) {  // (the grid's z limit)
    colsum_final_kernel<<<dim3(G, d / 64, std::min(norms - n, 65535)), 256, 0, s>>>(part + (int64_t)n * segs * d, soff,
                                                                                   dg + (int64_t)n * G, d);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// -------------------------------------------------------------- attention ---
// Self- / cross-attention of the expert on the bf16 matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation and softmax statistics).
// Queries: rows q_row0 + 0..Lq-1 of Q (Lq <= 64: four 16-row blocks, one per
// wave); keys / values: rows kv_row0 .. + Lk - 1 of K / V.  Self attention:
// the sample's own action rows; cross attention: the sample's rows of the
// tenant-ordered prefix (zoff), so a query never sees another sample's keys.
// Q, K, V are bf16 (their projections store them so); the probabilities are
// rounded to bf16 before they meet V, and in the backward the incoming output
// gradient, the recomputed probabilities and the score gradient before they
// meet their products.  The softmax runs in the log2 domain: lse holds
// m + log2(l) of the scaled scores.
//
// MFMA layouts (16x16x32): A (16 x 32) -- lane l supplies row l & 15,
// k-slots 8 (l >> 4) .. +7; B (32 x 16) -- column l & 15, the same k-slots;
// D -- lane l holds rows 4 (l >> 4) .. +3 of column l & 15.  Scores are
// formed transposed where the lane should own a query (S^T = K Q^T: lane =
// query, registers = 4 keys of each 16-key block), so a query's row
// statistics need only exchanges with lanes l ^ 16 and l ^ 32.  Products
// whose contraction runs over the rows of a row-major LDS tile (V^T P^T,
// K^T dS^T, dO^T P, Q^T dS) read their A operand with ds_read_b64_tr_b16:
// lane (g, j) of 16-lane group g addresses row 32 c + 4 g + j / 4 (and +16)
// at column 16 t + 4 (j % 4) and receives column 16 t + j of rows
// 32 c + 4 g .. +3 and 32 c + 16 + 4 g .. +3, so k-slot s of lane (g, j)
// is row 32 c + 4 g + (s & 3) + 16 (s >> 2) -- the order in which the lane
// already holds the matching B values (register e of blocks 2c and 2c+1).
// Every LDS tile row is a permutation of its 16-byte chunks (chunk c at
// c ^ swz(row)) so that both the 16-byte fragment reads and the transposed
// reads touch each bank once per 256 bytes.

typedef __bf16 xbf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 xbf16x4 __attribute__((ext_vector_type(4)));
typedef float xf32x4 __attribute__((ext_vector_type(4)));

#define XA_GPTR(p) ((__attribute__((address_space(1))) void*)(p))
#define XA_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

template <int HD>
__device__ __forceinline__ int xa_swz(int r) {
  if constexpr (HD == 64) {
    const int x = (r >> 1) & 7;  // 2 rows per 256-byte bank row: bit-reversed row pair
    return ((x & 1) << 2) | (x & 2) | (x >> 2);
  } else {
    // one row per bank row; rows r and r ^ 8 share a bank slot pair, so the
    // transposed reads of 16-lane groups q and q ^ 1, which the hardware
    // serves together, stay on 16 distinct slots (a fragment read's 16 rows
    // as well).  The backbone attention's head-width-256 rule, which also
    // avoids the q / q ^ 2 pairing, measured 1% slower here.
    return ((r & 7) << 1) | ((r >> 3) & 1);
  }
}

// 16-byte fragment: logical chunk c (8 elements) of row r of an LDS tile
template <int HD>
__device__ __forceinline__ xbf16x8 xa_frag(const uint16_t* t, int r, int c) {
  return *reinterpret_cast<const xbf16x8*>(t + r * HD + ((c ^ xa_swz<HD>(r)) * 8));
}

// transposed A operand: rows 32 c + 4 g + {0..3, 16..19} of column 16 t + j
// (lane (g, j)); swz = xa_swz(4 g + j / 4), shared by those rows
template <int HD>
__device__ __forceinline__ xbf16x8 xa_tr(const uint16_t* t, int c, int ct, int quad, int j16, int swz) {
  const int col = ct * 16 + 4 * (j16 & 3);
  const int pos = (((col >> 3) ^ swz) * 8) + (col & 7);
  const int r0 = c * 32 + 4 * quad + (j16 >> 2);
  const xbf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) xbf16x4*)(t + r0 * HD + pos));
  const xbf16x4 hi =
      __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) xbf16x4*)(t + (r0 + 16) * HD + pos));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// The same without the compiler's vmcnt(0) in front of it, which would wait for
// the K/V tile being fetched; the caller waits (lgkmcnt).
template <int HD>
__device__ __forceinline__ xbf16x8 xa_tr_async(const uint16_t* t, int c, int ct, int quad, int j16, int swz) {
  const int col = ct * 16 + 4 * (j16 & 3);
  const int pos = (((col >> 3) ^ swz) * 8) + (col & 7);
  const uint16_t* p = t + (c * 32 + 4 * quad + (j16 >> 2)) * HD + pos;
  const xbf16x4 lo = __builtin_bit_cast(xbf16x4, lds_read_tr_b16<0>(p));
  const xbf16x4 hi = __builtin_bit_cast(xbf16x4, lds_read_tr_b16<16 * HD * 2>(p));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ xf32x4 xa_mfma(xbf16x8 a, xbf16x8 b, xf32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 8 fp32 values -> bf16 operand (round to nearest even)
__device__ __forceinline__ xbf16x8 xa_pack8(const float* v) {
  xbf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (__bf16)v[e];
  return r;
}

// Lanes of quads 2u and 2u + 1 hold 8-byte pieces a (row block t) and b (t + 1)
// of the same two 32-byte runs; afterwards the even quad has both pieces of
// block t, the odd one both of block t + 1, in order.
__device__ __forceinline__ uint4 xa_pair16(uint2 a, uint2 b) {
  const auto x = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
  const auto y = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
  return make_uint4(x[0], y[0], x[1], y[1]);
}

__device__ __forceinline__ void attn_rows(const AttnArgs& A, int32_t k, int32_t& q0, int32_t& Lq, int64_t& kv0,
                                          int32_t& Lk) {
  q0 = k * A.Lq;
  Lq = A.Lq;
  if (A.zoff) {
    kv0 = A.zoff[k];
    const int64_t kv1 = min((int64_t)A.zoff[k + 1], A.kv_cap);
    Lk = (int32_t)max((int64_t)0, kv1 - kv0);
  } else {
    kv0 = (int64_t)k * A.Lq;
    Lk = A.Lq;
  }
}

// K and V tiles of 64 keys ([64][HD] bf16 each, swizzled), double buffered,
// moved by direct DMA: 1 KB instructions, lane -> (row RPI v + lane / CPR,
// chunk (lane % CPR) ^ swz(row)); rows past the sample repeat its last row.
template <int HD>
struct XaTiles {
  static constexpr int CPR = HD / 8, RPI = 512 / HD, TILE = 64 * HD, NDMA = 2 * TILE / 512, DPW = NDMA / 4;
  __device__ __forceinline__ static void issue(uint16_t* stage, const uint16_t* Kb, const uint16_t* Vb, int64_t ld,
                                               int64_t kv0, int32_t Lk, int32_t j0, int wave, int lane) {
#pragma unroll
    for (int k = 0; k < DPW; ++k) {
      const int u = wave * DPW + k;
      const bool isv = u >= NDMA / 2;
      const int v = isv ? u - NDMA / 2 : u;
      const int r = v * RPI + lane / CPR;
      const int c = (lane % CPR) ^ xa_swz<HD>(r);
      const int64_t key = kv0 + min(j0 + r, Lk - 1);
      const uint16_t* src = (isv ? Vb : Kb) + key * ld + c * 8;
      __builtin_amdgcn_global_load_lds(XA_GPTR(src), XA_LPTR(stage + u * 512), 16, 0, 0);
    }
  }
};

// Forward: one workgroup per (sample, head), wave w = queries 16 w ..;
// O = softmax(Q K^T scale) V in fp32 (and a bf16 copy), lse per query.
// K and V are read once (16 tenants, 288 samples of ~600 keys: 0.68 GB, 110 us
// at the copy rate of 6.2 TB/s, 194 measured).  A sample's heads are consecutive
// workgroups, so that the 256-byte head slices of a K / V row are read at about
// the same time (backward 343 -> 325 us, forward unchanged).
template <int HD>
__global__ __launch_bounds__(256, 2) void xattn_fwd_kernel(AttnArgs A) {
  using T = XaTiles<HD>;
  constexpr int NQC = HD / 32, NOT = HD / 16;
  __shared__ __attribute__((aligned(1024))) uint16_t lds[2][2 * T::TILE];
  const int k = blockIdx.x / A.nheads, h = blockIdx.x % A.nheads;
  int32_t q0, Lq, Lk;
  int64_t kv0;
  attn_rows(A, k, q0, Lq, kv0, Lk);
  if (Lk <= 0) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j16 = lane & 15, quad = lane >> 4;
  const int qi = wave * 16 + j16;  // this lane's query
  const int64_t qrow = q0 + min(qi, Lq - 1);
  const float sl2 = A.scale * 1.4426950408889634f;
  xbf16x8 qf[NQC];
#pragma unroll
  for (int c = 0; c < NQC; ++c) qf[c] = *reinterpret_cast<const xbf16x8*>(A.Q + qrow * A.ldq + h * HD + c * 32 + quad * 8);
  const uint16_t* Kb = A.K + A.kcol + h * HD;
  const uint16_t* Vb = A.V + A.vcol + h * HD;
  const int vswz = xa_swz<HD>(4 * quad + (j16 >> 2));

  xf32x4 o[NOT];
#pragma unroll
  for (int t = 0; t < NOT; ++t) o[t] = xf32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const int32_t ntiles = (Lk + 63) / 64;
  T::issue(&lds[0][0], Kb, Vb, A.ldkv, kv0, Lk, 0, wave, lane);
  for (int32_t jt = 0; jt < ntiles; ++jt) {
    const int32_t j0 = jt * 64;
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_s_barrier();  // tile jt landed; tile jt-1's buffer is free
    T::issue(&lds[(jt + 1) & 1][0], Kb, Vb, A.ldkv, kv0, Lk, min(j0 + 64, (ntiles - 1) * 64), wave, lane);
    const uint16_t* Ks = &lds[jt & 1][0];
    const uint16_t* Vs = Ks + T::TILE;
    xf32x4 s[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) s[kb] = xf32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NQC; ++c)
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) s[kb] = xa_mfma(xa_frag<HD>(Ks, kb * 16 + j16, 4 * c + quad), qf[c], s[kb]);
    if (j0 + 64 > Lk) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j0 + kb * 16 + quad * 4 + e >= Lk) s[kb][e] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[kb][e]);
    const float m_new = fmaxf(m, max_xor32(max_xor16(mx)) * sl2);
    if (__any(m_new > m)) {  // (else alpha is 1 for every lane)
      const float alpha = __builtin_amdgcn_exp2f(m - m_new);
      l *= alpha;
#pragma unroll
      for (int t = 0; t < NOT; ++t) o[t] *= alpha;
      m = m_new;
    }
    float lsum = 0.f;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[kb][e] = __builtin_amdgcn_exp2f(fmaf(s[kb][e], sl2, -m));  // (below 2^-126: zero)
        lsum += s[kb][e];
      }
    l += sum_xor32(sum_xor16(lsum));
    xbf16x8 pf[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pf[c][e] = (__bf16)s[2 * c][e];
        pf[c][4 + e] = (__bf16)s[2 * c + 1][e];
      }
    // V^T of head-dim block t + 1 is read under the products of block t
    xbf16x8 vb[2][2];
#pragma unroll
    for (int c = 0; c < 2; ++c) vb[0][c] = xa_tr_async<HD>(Vs, c, 0, quad, j16, vswz);
#pragma unroll
    for (int t = 0; t < NOT; ++t) {
      if (t + 1 < NOT) {
#pragma unroll
        for (int c = 0; c < 2; ++c) vb[(t + 1) & 1][c] = xa_tr_async<HD>(Vs, c, t + 1, quad, j16, vswz);
        __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (4 << 8));  // lgkmcnt(4): block t's reads
      } else {
        __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));  // lgkmcnt(0)
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < 2; ++c) o[t] = xa_mfma(vb[t & 1][c], pf[c], o[t]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);  // the repeated last tile's DMA lands before the LDS is released
  if (qi >= Lq) return;
  const float inv = 1.f / l;
  const int64_t row = q0 + qi;
  float* orow = A.O + row * A.ldo + h * HD + quad * 4;
  uint16_t* brow = A.Ob + row * A.ldo + h * HD + quad * 4;
#pragma unroll
  for (int t = 0; t < NOT; ++t) {
    const float v0 = o[t][0] * inv, v1 = o[t][1] * inv, v2 = o[t][2] * inv, v3 = o[t][3] * inv;
    *reinterpret_cast<float4*>(orow + t * 16) = make_float4(v0, v1, v2, v3);
    *reinterpret_cast<uint2*>(brow + t * 16) = make_uint2(pack_bf2(v0, v1), pack_bf2(v2, v3));
  }
  if (quad == 0) A.lse[row * A.nheads + h] = m + __log2f(l);
}

// Backward: one workgroup per (sample, head) walks the sample's 64-key tiles;
// its queries (<= 64, zero rows past Lq) and their bf16-rounded output
// gradients stay in LDS.  Wave w owns keys 16 w .. of a tile: scores
// untransposed, S = Q K^T (lane = key, registers = 4 queries of each 16-query
// block), P from the saved lse, dP = dO V^T, dS = P (dP - D) with
// D = sum(dO * O) per query, so P and dS are already the B operands of
// dV^T = dO^T P and dK^T = Q^T dS.  dS then goes through LDS ([key][query]),
// and the wave owning queries 16 w .. adds K^T dS^T to its dQ^T.
// Memory-bound: K and V are read once and dK and dV written once (16 tenants,
// 288 samples of ~600 keys: 1.4 GB, 226 us at the copy rate of 6.2 TB/s).  As two kernels,
// a query side and a key side of one workgroup per key tile, K, V, the queries
// and the output gradients were read again for every tile and S and dP formed
// twice: 199 + 455 us, now 325 (self attention 55 + 46 -> 72).  One K/V buffer, so that two workgroups
// share a CU (72 KB of LDS each) and one's products hide the other's loads.
template <int HD>
__global__ __launch_bounds__(256, 2) void xattn_bwd_kernel(AttnArgs A) {
  using T = XaTiles<HD>;
  constexpr int NQC = HD / 32, NOT = HD / 16, CPR = HD / 8;
  __shared__ __attribute__((aligned(1024))) uint16_t kv[2 * T::TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t qt[64 * HD];
  __shared__ __attribute__((aligned(1024))) uint16_t dt[64 * HD];
  __shared__ __attribute__((aligned(1024))) uint16_t ds[64 * 64];
  __shared__ float lse_s[64], d_s[64];
  const int k = blockIdx.x / A.nheads, h = blockIdx.x % A.nheads;
  int32_t q0, Lq, Lk;
  int64_t kv0;
  attn_rows(A, k, q0, Lq, kv0, Lk);
  if (Lk <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j16 = lane & 15, quad = lane >> 4;
  const float sl2 = A.scale * 1.4426950408889634f;
  const uint16_t* Kb = A.K + A.kcol + h * HD;
  const uint16_t* Vb = A.V + A.vcol + h * HD;
  const uint16_t *Ks = kv, *Vs = kv + T::TILE;
  // Q and bf16(dO): 64 rows x CPR chunks of 8 elements; D by CPR lanes per row
  for (int e = tid; e < 64 * CPR; e += 256) {
    const int r = e / CPR, c = e % CPR;
    const int pos = r * HD + ((c ^ xa_swz<HD>(r)) * 8);
    uint4 qv = make_uint4(0, 0, 0, 0), dv = make_uint4(0, 0, 0, 0);
    float D = 0.f;
    if (r < Lq) {
      const int64_t row = q0 + r;
      const float* dp = A.dO + row * A.ldo + h * HD + c * 8;
      const float* op = A.O + row * A.ldo + h * HD + c * 8;
      qv = *reinterpret_cast<const uint4*>(A.Q + row * A.ldq + h * HD + c * 8);
      const float4 a = *reinterpret_cast<const float4*>(dp), b = *reinterpret_cast<const float4*>(dp + 4);
      const float4 u = *reinterpret_cast<const float4*>(op), v = *reinterpret_cast<const float4*>(op + 4);
      dv = make_uint4(pack_bf2(a.x, a.y), pack_bf2(a.z, a.w), pack_bf2(b.x, b.y), pack_bf2(b.z, b.w));
      D = fmaf(a.x, u.x, fmaf(a.y, u.y, fmaf(a.z, u.z, a.w * u.w))) +
          fmaf(b.x, v.x, fmaf(b.y, v.y, fmaf(b.z, v.z, b.w * v.w)));
    }
#pragma unroll
    for (int o = CPR / 2; o > 0; o >>= 1) D += __shfl_xor(D, o, kWave);
    if (c == 0) d_s[r] = D;
    *reinterpret_cast<uint4*>(qt + pos) = qv;
    *reinterpret_cast<uint4*>(dt + pos) = dv;
  }
  if (tid < 64) lse_s[tid] = tid < Lq ? A.lse[(q0 + tid) * A.nheads + h] : INFINITY;  // P = 0 past Lq
  T::issue(kv, Kb, Vb, A.ldkv, kv0, Lk, 0, wave, lane);

  const int tswz = xa_swz<HD>(4 * quad + (j16 >> 2)), sswz = xa_swz<64>(4 * quad + (j16 >> 2));
  const int krow = wave * 16 + j16;  // this lane's key in the tile
  xf32x4 dq[NOT];
#pragma unroll
  for (int t = 0; t < NOT; ++t) dq[t] = xf32x4{0.f, 0.f, 0.f, 0.f};
  const int32_t ntiles = (Lk + 63) / 64;
  for (int32_t jt = 0; jt < ntiles; ++jt) {
    const int32_t key = jt * 64 + krow;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's part of tile jt landed: a barrier alone waits for no DMA
    __syncthreads();                // every wave's did (first: the staged rows too)
    xf32x4 s[4], dp[4];
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) s[qb] = dp[qb] = xf32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NQC; ++c) {
      const xbf16x8 kf = xa_frag<HD>(Ks, krow, 4 * c + quad), vf = xa_frag<HD>(Vs, krow, 4 * c + quad);
#pragma unroll
      for (int qb = 0; qb < 4; ++qb) {
        s[qb] = xa_mfma(xa_frag<HD>(qt, qb * 16 + j16, 4 * c + quad), kf, s[qb]);
        dp[qb] = xa_mfma(xa_frag<HD>(dt, qb * 16 + j16, 4 * c + quad), vf, dp[qb]);
      }
    }
    // P and dS as B operands: k-slot s of chunk c is query 32 c + 4 quad + (s & 3) + 16 (s >> 2)
    xbf16x8 pb[2], db[2];
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) {
      xbf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int q = qb * 16 + quad * 4 + e;
        const float pv = key < Lk ? exp2f(fmaf(s[qb][e], sl2, -lse_s[q])) : 0.f;
        pb[qb >> 1][(qb & 1) * 4 + e] = (__bf16)pv;
        w[e] = (__bf16)(pv * (dp[qb][e] - d_s[q]));
        db[qb >> 1][(qb & 1) * 4 + e] = w[e];
      }
      *reinterpret_cast<xbf16x4*>(ds + krow * 64 + (((2 * qb + (quad >> 1)) ^ xa_swz<64>(krow)) * 8) + 4 * (quad & 1)) = w;
    }
    uint16_t* const vrow = A.dV + (kv0 + key) * A.lddkv + A.dvcol + h * HD;
    uint16_t* const krw = A.dK + (kv0 + key) * A.lddkv + A.dkcol + h * HD;
    // lane holds dV^T / dK^T rows (head dims) 16 t + 4 quad .. +3 of its key;
    // quads 2u and 2u + 1 swap halves of a pair of t, so a lane stores 16 bytes
#pragma unroll
    for (int t = 0; t < NOT; t += 2) {
      xf32x4 dv[2], dk[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        dv[i] = dk[i] = xf32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          dv[i] = xa_mfma(xa_tr<HD>(dt, c, t + i, quad, j16, tswz), pb[c], dv[i]);
          dk[i] = xa_mfma(xa_tr<HD>(qt, c, t + i, quad, j16, tswz), db[c], dk[i]);
        }
      }
      const uint4 vo = xa_pair16(make_uint2(pack_bf2(dv[0][0], dv[0][1]), pack_bf2(dv[0][2], dv[0][3])),
                                 make_uint2(pack_bf2(dv[1][0], dv[1][1]), pack_bf2(dv[1][2], dv[1][3])));
      const uint4 ko = xa_pair16(make_uint2(pack_bf2(dk[0][0] * A.scale, dk[0][1] * A.scale),
                                            pack_bf2(dk[0][2] * A.scale, dk[0][3] * A.scale)),
                                 make_uint2(pack_bf2(dk[1][0] * A.scale, dk[1][1] * A.scale),
                                            pack_bf2(dk[1][2] * A.scale, dk[1][3] * A.scale)));
      const int col = (t + (quad & 1)) * 16 + 8 * (quad >> 1);
      if (key < Lk) {
        *reinterpret_cast<uint4*>(vrow + col) = vo;
        *reinterpret_cast<uint4*>(krw + col) = ko;
      }
    }
    __syncthreads();  // dS of every key
    xbf16x8 sb[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) sb[c] = xa_tr<64>(ds, c, wave, quad, j16, sswz);
#pragma unroll
    for (int t = 0; t < NOT; ++t)
#pragma unroll
      for (int c = 0; c < 2; ++c) dq[t] = xa_mfma(xa_tr<HD>(Ks, c, t, quad, j16, tswz), sb[c], dq[t]);
    if (jt + 1 < ntiles) {
      __syncthreads();  // K and V free
      T::issue(kv, Kb, Vb, A.ldkv, kv0, Lk, (jt + 1) * 64, wave, lane);
    }
  }
  const int qi = wave * 16 + j16;
  if (qi >= Lq) return;
  uint16_t* out = A.dQ + (q0 + qi) * A.lddq + h * HD + quad * 4;
#pragma unroll
  for (int t = 0; t < NOT; ++t)
    *reinterpret_cast<uint2*>(out + t * 16) = make_uint2(pack_bf2(dq[t][0] * A.scale, dq[t][1] * A.scale),
                                                         pack_bf2(dq[t][2] * A.scale, dq[t][3] * A.scale));
}

hipError_t launch_xattn(hipStream_t s, const AttnArgs& A, int32_t nsamples, bool backward) {
  if (A.Lq > 64 || A.Lq < 1 || A.max_lk < 1) return hipErrorInvalidValue;
  const int64_t wgs = (int64_t)nsamples * A.nheads;  // heads fastest: they share the rows of K and V
  if (wgs > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs);
  switch (A.hd) {
    case 64:
      if (backward) {
        xattn_bwd_kernel<64><<<grid, 256, 0, s>>>(A);
      } else {
        xattn_fwd_kernel<64><<<grid, 256, 0, s>>>(A);
      }
      break;
    case 128:
      if (backward) {
        xattn_bwd_kernel<128><<<grid, 256, 0, s>>>(A);
      } else {
        xattn_fwd_kernel<128><<<grid, 256, 0, s>>>(A);
      }
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------- loss ---
// Tenant t: rows [roff[t], roff[t+1]) of pred_pad [rows][ldp]; first `a`
// columns valid.  pred / target: the caller's [rows_t][a] buffers.  Block
// (tenant, part) takes rows part, part + kXLossParts, ..: a thread per padded
// column of 256 / ldp rows; the part's sum of squares (fixed-order tree) goes
// to `part`, and a second launch adds a tenant's parts in order.  One block per
// tenant took 307 us on 16 tenants of 14,400 rows in all, 8.7 + 3.3 us now.

__global__ __launch_bounds__(256) void xloss_kernel(const XLossDesc* __restrict__ descs, const int32_t* __restrict__ roff,
                                                   const float* __restrict__ pred_pad, int32_t ldp,
                                                   uint16_t* __restrict__ dpred_pad, float* __restrict__ part) {
  __shared__ float red[256];
  const int32_t t = blockIdx.x, p = blockIdx.y;
  const XLossDesc D = descs[t];
  const int32_t r0 = roff[t], rows = roff[t + 1] - r0;
  const int32_t rpb = 256 / ldp, c = threadIdx.x % ldp;
  const float scale = 2.0f / (float)((int64_t)rows * D.a);
  float ss = 0.f;
  if ((int32_t)threadIdx.x < rpb * ldp) {
#pragma unroll 4
    for (int32_t rr = p * rpb + threadIdx.x / ldp; rr < rows; rr += kXLossParts * rpb) {
      const int64_t gi = (int64_t)(r0 + rr) * ldp + c;
      float g = 0.f;
      if (c < D.a) {
        const float y = pred_pad[gi];
        const float diff = y - D.target[(int64_t)rr * D.a + c];
        D.pred[(int64_t)rr * D.a + c] = y;
        g = scale * diff;
        ss += diff * diff;
      }
      dpred_pad[gi] = f2bf(g);
    }
  }
  red[threadIdx.x] = ss;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[t * kXLossParts + p] = red[0];
}

__global__ __launch_bounds__(64) void xloss_final_kernel(const XLossDesc* __restrict__ descs, const int32_t* __restrict__ roff,
                                                        int32_t G, const float* __restrict__ part) {
  const int32_t t = blockIdx.x * 64 + threadIdx.x;
  if (t >= G) return;
  float s = 0.f;
#pragma unroll 8
  for (int p = 0; p < kXLossParts; ++p) s += part[t * kXLossParts + p];
  descs[t].loss[0] = s / (float)((int64_t)(roff[t + 1] - roff[t]) * descs[t].a);
}

hipError_t launch_xloss(hipStream_t s, const XLossDesc* d, const int32_t* roff, int32_t G, const float* pred_pad,
                        int32_t ldp, uint16_t* dpred_pad, float* part) {
  if (ldp < 1 || ldp > 256) return hipErrorInvalidValue;
  xloss_kernel<<<dim3(G, kXLossParts), 256, 0, s>>>(d, roff, pred_pad, ldp, dpred_pad, part);
  xloss_final_kernel<<<(G + 63) / 64, 64, 0, s>>>(d, roff, G, part);
  return hipGetLastError();
}

// ------------------------------------------------------------- flow prep ---
// One block per expert row: the tenant is found from the descriptors' row
// ranges, the sample from row / chunk.  Columns [0, a): bf16(t e + (1-t) A)
// and vel = e - A; [a, kap): 0; [kap, kap + d_time): bf16 of sin / cos of
// 1000 t w_j with w_j = 10000^(-j / (d_time/2)) (fp32 math).
__global__ __launch_bounds__(256) void flow_prep_kernel(const FlowDesc* __restrict__ d, int32_t G, int32_t chunk,
                                                        int32_t kap, int32_t d_time, uint16_t* __restrict__ in_rows,
                                                        int32_t ld) {
  const int64_t row = blockIdx.x;
  int32_t g = 0;
  while (g + 1 < G && row >= d[g + 1].roff) ++g;
  const FlowDesc D = d[g];
  const int64_t r = row - D.roff;
  if (r < 0 || r >= D.rows) return;
  const float tau = D.t[r / chunk];
  uint16_t* out = in_rows + row * ld;
  const int32_t half = d_time >> 1;
  const float l2 = 13.287712379549449f;  // log2(10000)
  for (int32_t c = threadIdx.x; c < kap + d_time; c += 256) {
    float v = 0.f;
    if (c < D.a) {
      const float e = D.noise[r * D.a + c], A = D.act[r * D.a + c];
      v = tau * e + (1.0f - tau) * A;
      D.vel[r * D.a + c] = e - A;
    } else if (c >= kap) {
      const int32_t j = c - kap;
      const int32_t jj = j < half ? j : j - half;
      const float ang = 1000.0f * tau * exp2f(-(float)jj / (float)half * l2);
      v = j < half ? sinf(ang) : cosf(ang);
    }
    out[c] = f2bf(v);
  }
}

hipError_t launch_flow_prep(hipStream_t s, const FlowDesc* d, int32_t G, int64_t total_rows, int32_t chunk,
                            int32_t kap, int32_t d_time, uint16_t* in_rows, int32_t ld) {
  if (G < 1 || total_rows < 1 || total_rows > 0x7fffffff || chunk < 1 || ld < kap + d_time) return hipErrorInvalidValue;
  flow_prep_kernel<<<(unsigned)total_rows, 256, 0, s>>>(d, G, chunk, kap, d_time, in_rows, ld);
  return hipGetLastError();
}

}  // namespace jnx
