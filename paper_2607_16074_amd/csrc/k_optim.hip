// Per-tenant AdamW step over every tensor of every tenant in one launch.
// Block b updates elements [2048 (b - block_start), +2048) of the tensor whose
// block range holds b; each thread handles 8 elements as two 16-byte accesses
// per operand (the tail of a tensor element by element).  HBM-bound: 16 bytes
// read and 12 written per element (+2 for a bf16 copy).  ONCE, more than the last-
// level cache holds: all but p's read non-temporal, since nothing of it is used
// again before it has left the caches (28.5M parameters: 151 -> 135 us of the launch
// alone, 5.9 TB/s; the call over 336 MB 145 -> 113, but over 33 MB 14.5 -> 16.6 and over
// 168 58 -> 60, so up to there plain).
#include "jn_device.h"
#include "jn_internal.h"

namespace jnx {

typedef float f32x4o __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void adamw_elem(const AdamwTenant& h, float& p, float g, float& m, float& v) {
  m = h.b1 * m + (1.f - h.b1) * g;
  v = h.b2 * v + (1.f - h.b2) * g * g;
  const float den = sqrtf(v) * h.inv_sqrt_bc2 + h.eps;
  p = p * h.decay - h.step_size * (m / den);
}

template <bool ONCE>
__device__ __forceinline__ f32x4o get(const f32x4o* p) {
  if constexpr (ONCE)
    return __builtin_nontemporal_load(p);
  else
    return *p;
}
template <bool ONCE>
__device__ __forceinline__ void put(f32x4o v, f32x4o* p) {
  if constexpr (ONCE)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <bool ONCE>
__global__ __launch_bounds__(256) void adamw_kernel(const AdamwTensor* __restrict__ ts, int32_t n,
                                                    const AdamwTenant* __restrict__ tens) {
  // the last tensor whose block range starts at or before this block (binary search)
  const int32_t b = blockIdx.x;
  int32_t lo = 0, hi = n - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (ts[mid].block_start <= b) lo = mid; else hi = mid - 1;
  }
  const int32_t i = lo;
  const AdamwTensor T = ts[i];
  const AdamwTenant H = tens[T.tenant];
  const int64_t e0 = (int64_t)(b - T.block_start) * kAdamwBlockElems;
#pragma unroll
  for (int k = 0; k < kAdamwBlockElems / 1024; ++k) {
    const int64_t e = e0 + ((int64_t)k * 256 + threadIdx.x) * 4;
    if (e >= T.numel) break;
    if (e + 4 <= T.numel) {
      f32x4o *const pp = reinterpret_cast<f32x4o*>(T.p + e), *const pm = reinterpret_cast<f32x4o*>(T.m + e),
             *const pv = reinterpret_cast<f32x4o*>(T.v + e);
      f32x4o p = *pp, m = get<ONCE>(pm), v = get<ONCE>(pv);
      const f32x4o g = get<ONCE>(reinterpret_cast<const f32x4o*>(T.g + e));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float pj = p[j], mj = m[j], vj = v[j];
        adamw_elem(H, pj, g[j], mj, vj);
        p[j] = pj;
        m[j] = mj;
        v[j] = vj;
      }
      put<ONCE>(p, pp);
      put<ONCE>(m, pm);
      put<ONCE>(v, pv);
      if (T.b16) *reinterpret_cast<uint2*>(T.b16 + e) = make_uint2(pack_bf2(p[0], p[1]), pack_bf2(p[2], p[3]));
    } else {
      for (int64_t j = e; j < T.numel; ++j) {
        float p = T.p[j], m = T.m[j], v = T.v[j];
        adamw_elem(H, p, T.g[j], m, v);
        T.p[j] = p;
        T.m[j] = m;
        T.v[j] = v;
        if (T.b16) T.b16[j] = f2bf(p);
      }
    }
  }
}

int32_t adamw_prepare(AdamwTensor* t, int32_t n) {
  int32_t total = 0;
  for (int32_t i = 0; i < n; ++i) {
    t[i].block_start = total;
    total += (int32_t)((t[i].numel + kAdamwBlockElems - 1) / kAdamwBlockElems);
  }
  return total;
}

hipError_t launch_adamw(hipStream_t s, const AdamwTensor* t, int32_t n, const AdamwTenant* ten, int32_t blocks) {
  if (blocks <= 0) return hipSuccess;
  if (blocks * kAdamwBlockElems * 16 > kStreamBytes)
    adamw_kernel<true><<<blocks, 256, 0, s>>>(t, n, ten);
  else
    adamw_kernel<false><<<blocks, 256, 0, s>>>(t, n, ten);
  return hipGetLastError();
}

}  // namespace jnx
