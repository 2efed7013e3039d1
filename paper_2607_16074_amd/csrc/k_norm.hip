// RMSNorm over rows of the packed batch: one wavefront per row, the row held
// in registers between the sum-of-squares pass and the scaling pass, a
// butterfly wave reduction (deterministic order), fp32 math, bf16 output.
#include <type_traits>

#include "jn_device.h"
#include "jn_internal.h"

namespace jnx {

constexpr int kNormRowsPerBlock = 4;  // 4 waves, one row each

// Vectors of the non-temporal loads.
template <int W>
struct NormVec {
  typedef float f __attribute__((ext_vector_type(W)));
};

// Load VEC bf16 values starting at element `e` of a bf16 row.
template <int VEC>
__device__ __forceinline__ void load_bf(const uint16_t* row, int e, float* v) {
  if constexpr (VEC == 8) {
    uint4 q = *reinterpret_cast<const uint4*>(row + e);
    uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[2 * k] = __uint_as_float(w[k] << 16);
      v[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
    }
  } else if constexpr (VEC == 4) {
    uint2 q = *reinterpret_cast<const uint2*>(row + e);
    v[0] = __uint_as_float(q.x << 16);
    v[1] = __uint_as_float(q.x & 0xffff0000u);
    v[2] = __uint_as_float(q.y << 16);
    v[3] = __uint_as_float(q.y & 0xffff0000u);
  } else {
    uint32_t q = *reinterpret_cast<const uint32_t*>(row + e);
    v[0] = __uint_as_float(q << 16);
    v[1] = __uint_as_float(q & 0xffff0000u);
  }
}

template <int VEC, bool STREAM = false>
__device__ __forceinline__ void load_f32(const float* row, int e, float* v) {
  constexpr int W = VEC % 4 == 0 ? 4 : 2;
  typedef typename NormVec<W>::f V;
#pragma unroll
  for (int k = 0; k < VEC; k += W) {
    const V* p = reinterpret_cast<const V*>(row + e + k);
    V q;
    if constexpr (STREAM)
      q = __builtin_nontemporal_load(p);
    else
      q = *p;
#pragma unroll
    for (int i = 0; i < W; ++i) v[k + i] = q[i];
  }
}

template <int VEC>
__device__ __forceinline__ void store_f32(float* row, int e, const float* v) {
#pragma unroll
  for (int k = 0; k < VEC; k += 2) *reinterpret_cast<float2*>(row + e + k) = make_float2(v[k], v[k + 1]);
}

template <int VEC>
__device__ __forceinline__ void store_bf(uint16_t* row, int e, const float* v) {
  if constexpr (VEC == 8) {
    *reinterpret_cast<uint4*>(row + e) =
        make_uint4(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7]));
  } else if constexpr (VEC == 4) {
    *reinterpret_cast<uint2*>(row + e) = make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
  } else {
    *reinterpret_cast<uint32_t*>(row + e) = pack_bf2(v[0], v[1]);
  }
}

// IN_BF16: x is bf16 (the packed tokens); its fp32 widening is also written to
// x_out (the residual stream).  Otherwise x is the fp32 residual stream.
// Each lane owns elements (c*64 + lane)*VEC .. +VEC for c < NC.  HBM-bound; the
// fp32 rows are read non-temporal, so that h, which the next GEMM reads, is what
// the caches keep: 295,606 x 768 236 -> 212 us (6.4 TB/s), 75,776 x 2048 159 ->
// 153.  (A non-temporal store of x_out: 239 -> 255 us on the latter.)
template <int VEC, int NC, bool IN_BF16>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const void* __restrict__ xin, float* __restrict__ x_out,
                                                      const uint16_t* __restrict__ g, uint16_t* __restrict__ h,
                                                      int32_t rows, int32_t d, float eps) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * kNormRowsPerBlock + (threadIdx.x >> 6);
  if (row >= rows) return;
  float v[NC][VEC];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int e = (c * 64 + lane) * VEC;
    if constexpr (IN_BF16)
      load_bf<VEC>(reinterpret_cast<const uint16_t*>(xin) + row * d, e, v[c]);
    else
      load_f32<VEC, true>(reinterpret_cast<const float*>(xin) + row * d, e, v[c]);
#pragma unroll
    for (int k = 0; k < VEC; ++k) ss += v[c][k] * v[c][k];
  }
  ss = wave_sum(ss);
  const float r = rsqrtf(ss / (float)d + eps);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int e = (c * 64 + lane) * VEC;
    if constexpr (IN_BF16) store_f32<VEC>(x_out + row * d, e, v[c]);
    float gv[VEC], o[VEC];
    load_bf<VEC>(g, e, gv);
#pragma unroll
    for (int k = 0; k < VEC; ++k) o[k] = v[c][k] * r * gv[k];
    store_bf<VEC>(h + row * d, e, o);
  }
}

// Reduction of a split residual projection and the norm after it in one pass:
// v = x + ((part[0] + part[1]) + ...), written back to x, then the norm of v in
// rmsnorm_kernel's order (which every wave forms for itself from the row in LDS).
// One workgroup per row, its column blocks dealt to up to four wavefronts: these
// batches have few rows, and the S + 1 reads of a row are what it waits for.  As two
// launches, in one wavefront per row, and now: 1 row of 4096, S = 8, 10.3, 17.3 and
// 5.8 us; 100 rows 9.7, 17.0 and 6.5; 300 rows of 2048, S = 8, 9.8, 6.6 and 6.4;
// 2,468 rows 39 (S = 8), 19.9 and 19.8 (S = 3).
constexpr int split_waves(int nc) { return nc < 4 ? nc : 4; }
template <int VEC, int NC>
__global__ __launch_bounds__(64 * split_waves(NC)) void rmsnorm_split_kernel(
    float* __restrict__ x, const float* __restrict__ part, int32_t S, int64_t stride, const uint16_t* __restrict__ g,
    uint16_t* __restrict__ h, int32_t d, float eps) {
  constexpr int W = split_waves(NC), CW = (NC + W - 1) / W;
  __shared__ __attribute__((aligned(16))) float line[NC * 64 * VEC];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = blockIdx.x;
  auto at = [&](int i) { return ((w + W * i) * 64 + lane) * VEC; };  // the wave's column block i
  auto mine = [&](int i) { return NC % W == 0 || w + W * i < NC; };
  float v[CW][VEC], a[CW][VEC];
#pragma unroll
  for (int i = 0; i < CW; ++i)
    if (mine(i)) {
      load_f32<VEC>(x + row * d, at(i), v[i]);
      load_f32<VEC>(part + row * d, at(i), a[i]);
    }
#pragma unroll 4
  for (int32_t s = 1; s < S; ++s) {
#pragma unroll
    for (int i = 0; i < CW; ++i)
      if (mine(i)) {
        float q[VEC];
        load_f32<VEC>(part + s * stride + row * d, at(i), q);
#pragma unroll
        for (int k = 0; k < VEC; ++k) a[i][k] += q[k];
      }
  }
#pragma unroll
  for (int i = 0; i < CW; ++i)
    if (mine(i)) {
#pragma unroll
      for (int k = 0; k < VEC; ++k) v[i][k] += a[i][k];
      store_f32<VEC>(x + row * d, at(i), v[i]);
      store_f32<VEC>(line, at(i), v[i]);
    }
  __syncthreads();
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    float q[VEC];
    load_f32<VEC>(line, (c * 64 + lane) * VEC, q);
#pragma unroll
    for (int k = 0; k < VEC; ++k) ss += q[k] * q[k];
  }
  ss = wave_sum(ss);
  const float r = rsqrtf(ss / (float)d + eps);
#pragma unroll
  for (int i = 0; i < CW; ++i)
    if (mine(i)) {
      float gv[VEC], o[VEC];
      load_bf<VEC>(g, at(i), gv);
#pragma unroll
      for (int k = 0; k < VEC; ++k) o[k] = v[i][k] * r * gv[k];
      store_bf<VEC>(h + row * d, at(i), o);
    }
}

// Calls f<VEC, NC>() with the lane layout of row width d: a multiple of 128 up
// to 4096; widths without a layout of their own take two elements per lane.
template <typename F>
static hipError_t with_width(int32_t d, F&& f) {
#define JN_RMS(VEC, NC) \
  if (d == 64 * (VEC) * (NC)) return f(std::integral_constant<int, VEC>(), std::integral_constant<int, NC>());
  JN_RMS(2, 1)   // 128
  JN_RMS(4, 1)   // 256
  JN_RMS(4, 2)   // 512
  JN_RMS(4, 3)   // 768
  JN_RMS(8, 2)   // 1024
  JN_RMS(8, 3)   // 1536
  JN_RMS(8, 4)   // 2048
  JN_RMS(8, 5)   // 2560
  JN_RMS(8, 6)   // 3072
  JN_RMS(8, 8)   // 4096
#define JN_RMS2(NC) JN_RMS(2, NC)
  JN_RMS2(3) JN_RMS2(5) JN_RMS2(7) JN_RMS2(9) JN_RMS2(10) JN_RMS2(11) JN_RMS2(13) JN_RMS2(14) JN_RMS2(15)
  JN_RMS2(17) JN_RMS2(18) JN_RMS2(19) JN_RMS2(20) JN_RMS2(21) JN_RMS2(22) JN_RMS2(23) JN_RMS2(25)
  JN_RMS2(26) JN_RMS2(27) JN_RMS2(28) JN_RMS2(29) JN_RMS2(30) JN_RMS2(31)
#undef JN_RMS2
#undef JN_RMS
  return hipErrorInvalidValue;
}

template <bool IN_BF16>
static hipError_t launch_rms(hipStream_t s, const void* x, float* x_out, const void* g, void* h, int32_t rows,
                             int32_t d, float eps) {
  const dim3 grid((rows + kNormRowsPerBlock - 1) / kNormRowsPerBlock);
  return with_width(d, [&](auto vec, auto nc) {
    rmsnorm_kernel<vec(), nc(), IN_BF16><<<grid, 256, 0, s>>>(x, x_out, reinterpret_cast<const uint16_t*>(g),
                                                              reinterpret_cast<uint16_t*>(h), rows, d, eps);
    return hipGetLastError();
  });
}

hipError_t launch_rmsnorm_split(hipStream_t s, float* x, const float* part, int32_t S, const void* g, void* h,
                                int32_t rows, int32_t d, float eps) {
  return with_width(d, [&](auto vec, auto nc) {
    rmsnorm_split_kernel<vec(), nc()><<<dim3(rows), 64 * split_waves(nc()), 0, s>>>(
        x, part, S, (int64_t)rows * d, reinterpret_cast<const uint16_t*>(g), reinterpret_cast<uint16_t*>(h), d, eps);
    return hipGetLastError();
  });
}

hipError_t launch_rmsnorm_bf16in(hipStream_t s, const void* x_bf16, float* x_out, const void* g, void* h,
                                 int32_t rows, int32_t d, float eps) {
  return launch_rms<true>(s, x_bf16, x_out, g, h, rows, d, eps);
}

hipError_t launch_rmsnorm_f32in(hipStream_t s, const float* x, const void* g, void* h, int32_t rows, int32_t d,
                                float eps) {
  return launch_rms<false>(s, x, nullptr, g, h, rows, d, eps);
}

}  // namespace jnx
