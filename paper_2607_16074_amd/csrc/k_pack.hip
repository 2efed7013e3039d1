// Pack (canonicalize + pad into one physical batch) and unpack (split back by
// the recorded slices).  Both are plain HBM copies.
#include <algorithm>
#include <type_traits>

#include "jn_device.h"
#include "jn_internal.h"

namespace jnx {

typedef uint32_t u32x4p __attribute__((ext_vector_type(4)));
constexpr int kFlat = 512;  // elements (16 or 4 bytes) a block moves at a time

// A small host table to device memory by a kernel that reads the (coherent)
// pinned staging buffer: a launch costs the host about 3 us less than an
// asynchronous copy and the copy's own kernel, and the stream waits for no copy
// in between (two tenants' smallest step 115.6 -> 106.9 us, 8 x 32 heads 231 ->
// 217, one tenant's expert step 816 -> 792).  Above 64 KB the copy's bandwidth
// counts.
// System-scope loads: a staging buffer is rewritten by the host between calls.
__global__ __launch_bounds__(256) void upload_kernel(uint32_t* __restrict__ dst, const uint32_t* src, int32_t words,
                                                     uint32_t* __restrict__ tail_dst, int32_t all) {
  const int32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= all) return;
  const uint32_t v = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (i < words)
    dst[i] = v;
  else
    tail_dst[i - words] = v;
}

hipError_t launch_upload(hipStream_t s, void* dst, const void* src, size_t bytes, void* tail_dst, size_t tail) {
  if (bytes + tail > kUploadBytes || (bytes | tail) % 4 != 0 || ((uintptr_t)dst | (uintptr_t)tail_dst) % 4 != 0) {
    const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess || tail == 0) return e;
    return hipMemcpyAsync(tail_dst, static_cast<const char*>(src) + bytes, tail, hipMemcpyHostToDevice, s);
  }
  const int32_t words = (int32_t)(bytes / 4), all = (int32_t)((bytes + tail) / 4);
  upload_kernel<<<(all + 255) / 256, 256, 0, s>>>(static_cast<uint32_t*>(dst), static_cast<const uint32_t*>(src), words,
                                                  static_cast<uint32_t*>(tail_dst), all);
  return hipGetLastError();
}

// A sample's rows are one contiguous run in the request and in the packed
// buffer, so a block moves kFlat consecutive elements of it (a row boundary
// means nothing; live: elements that exist in the source, the rest are zeros),
// all of a thread's loads issued before its first store.  Every byte is touched
// once, so the loads are non-temporal, and ONCE, the stores too (kStreamBytes).
// Bound by HBM, and by which of its
// pieces are in flight together: with consecutive blocks on consecutive 8 KB of
// a sample 256 samples of ~296 rows of 4 KB take 100 us (6.1 TB/s), with 16 KB
// per block 109, 32 KB 112 (119 without the non-temporal hint), 32 KB with
// consecutive blocks on different samples 125; 16 rows per block, samples
// fastest, one load in flight: 130.
template <bool ONCE, typename V>
__device__ __forceinline__ void put(V v, V* p) {
  if constexpr (ONCE)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <bool ONCE, typename V>
__device__ __forceinline__ void move_run(const V* __restrict__ src, V* __restrict__ dst, int64_t at, int64_t live,
                                         int64_t n) {
  const int64_t e0 = at + threadIdx.x;
  V v[kFlat / 256];
  if (at + kFlat <= live) {
#pragma unroll
    for (int u = 0; u < kFlat / 256; ++u) v[u] = __builtin_nontemporal_load(src + e0 + u * 256);
#pragma unroll
    for (int u = 0; u < kFlat / 256; ++u) put<ONCE>(v[u], dst + e0 + u * 256);
    return;
  }
#pragma unroll
  for (int u = 0; u < kFlat / 256; ++u) {
    v[u] = V{};
    if (e0 + u * 256 < live) v[u] = __builtin_nontemporal_load(src + e0 + u * 256);
  }
#pragma unroll
  for (int u = 0; u < kFlat / 256; ++u)
    if (e0 + u * 256 < n) put<ONCE>(v[u], dst + e0 + u * 256);
}

template <bool ONCE>
__global__ __launch_bounds__(256) void pack_kernel(const ReqEntry* __restrict__ req_table,
                                                   const int32_t* __restrict__ sample_request,
                                                   const int32_t* __restrict__ sample_local,
                                                   const int32_t* __restrict__ seqlens,
                                                   const int32_t* __restrict__ cu_seqlens, int32_t d,
                                                   u32x4p* __restrict__ tokens, int32_t* __restrict__ token_sample,
                                                   int32_t* __restrict__ token_pos, int32_t per) {
  const int32_t i = blockIdx.x / per, part = blockIdx.x % per;
  const int32_t base = cu_seqlens[i];
  const int32_t rows = cu_seqlens[i + 1] - base;  // aligned rows of this sample
  const int32_t L = seqlens[i];
  const ReqEntry e = req_table[sample_request[i]];
  const int64_t chunks = d / 8;  // 16-byte chunks per row
  const u32x4p* src = reinterpret_cast<const u32x4p*>(e.in) + (int64_t)sample_local[i] * e.max_len * chunks;
  for (int64_t at = (int64_t)part * kFlat; at < rows * chunks; at += (int64_t)per * kFlat)
    move_run<ONCE>(src, tokens + base * chunks, at, L * chunks, rows * chunks);
  for (int64_t j = (int64_t)part * 256 + threadIdx.x; j < rows; j += (int64_t)per * 256) {
    token_sample[base + j] = j < L ? i : -1;
    token_pos[base + j] = j < L ? (int32_t)j : -1;
  }
}

// The same over consecutive elements of the packed buffer, whichever samples they
// belong to: for batches of a few long samples among many short ones (spread_blocks).
constexpr int kRaggedRuns = 4;  // most kFlat runs of a workgroup, between two searches
__global__ __launch_bounds__(256) void pack_ragged_kernel(const ReqEntry* __restrict__ req_table,
                                                          const int32_t* __restrict__ sample_request,
                                                          const int32_t* __restrict__ sample_local,
                                                          const int32_t* __restrict__ seqlens,
                                                          const int32_t* __restrict__ cu_seqlens, int32_t N, int32_t T,
                                                          int32_t d, int32_t run, u32x4p* __restrict__ tokens,
                                                          int32_t* __restrict__ token_sample,
                                                          int32_t* __restrict__ token_pos) {
  const uint32_t chunks = d / 8;
  const int64_t all = (int64_t)T * chunks;
  for (int64_t at = (int64_t)blockIdx.x * run; at < all; at += (int64_t)gridDim.x * run) {
    // rows ra .. rb, of samples ia .. ib (a sample has a row or more)
    const int64_t n = min((int64_t)run, all - at);
    const int32_t ra = (int32_t)(at / chunks), rb = (int32_t)((at + n - 1) / chunks);
    const int32_t ia = last_at(cu_seqlens, N, ra), ib = ia + last_at(cu_seqlens + ia, min(N - ia, rb - ra + 1), rb);
    const uint32_t c0 = (uint32_t)(at - ra * (int64_t)chunks);
    if (ia == ib) {
      const ReqEntry q = req_table[sample_request[ia]];
      const int64_t from = at - cu_seqlens[ia] * (int64_t)chunks;
      const u32x4p* src = reinterpret_cast<const u32x4p*>(q.in) + (int64_t)sample_local[ia] * q.max_len * chunks + from;
      const int64_t live = seqlens[ia] * (int64_t)chunks - from;
      for (int64_t e = 0; e < n; e += kFlat) move_run<false>(src, tokens + at, e, live, n);
    } else {
      for (int64_t e = threadIdx.x; e < n; e += 256) {
        const uint32_t r = (c0 + (uint32_t)e) / chunks, c = c0 + (uint32_t)e - r * chunks;
        const int32_t row = ra + (int32_t)r, i = ia + last_at(cu_seqlens + ia, ib - ia + 1, row);
        const int32_t j = row - cu_seqlens[i];
        u32x4p v{};
        if (j < seqlens[i]) {
          const ReqEntry q = req_table[sample_request[i]];
          v = __builtin_nontemporal_load(reinterpret_cast<const u32x4p*>(q.in) +
                                         ((int64_t)sample_local[i] * q.max_len + j) * chunks + c);
        }
        tokens[at + e] = v;
      }
    }
    for (int32_t row = ra + (c0 != 0) + (int32_t)threadIdx.x; row <= rb; row += 256) {  // rows that start here
      const int32_t i = ia + last_at(cu_seqlens + ia, ib - ia + 1, row), j = row - cu_seqlens[i];
      const bool live = j < seqlens[i];
      token_sample[row] = live ? i : -1;
      token_pos[row] = live ? j : -1;
    }
  }
}

// RAGGED: the workgroups of a sample are those of its own request (as above, for
// requests of unlike padded lengths), found in the request table.
template <typename V, bool RAGGED, bool ONCE>
__global__ __launch_bounds__(256) void unpack_kernel(const ReqEntry* __restrict__ req_table, int32_t R,
                                                     const int32_t* __restrict__ sample_request,
                                                     const int32_t* __restrict__ sample_local,
                                                     const int32_t* __restrict__ seqlens,
                                                     const int32_t* __restrict__ cu_seqlens, const V* __restrict__ rows,
                                                     int64_t row_vecs, int32_t per, int32_t N) {
  int32_t i, part;
  if constexpr (RAGGED) {
    const int32_t b = blockIdx.x;
    int32_t lo = 0, hi = R - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (req_table[mid].block <= b) lo = mid; else hi = mid - 1;
    }
    const ReqEntry q = req_table[lo];
    per = (int32_t)min((q.max_len * row_vecs + kFlat - 1) / kFlat, (int64_t)per);
    i = q.first + (b - q.block) / per;
    part = (b - q.block) % per;
    if (i >= N) return;
  } else {
    i = blockIdx.x / per;
    part = blockIdx.x % per;
  }
  const ReqEntry e = req_table[sample_request[i]];
  const int32_t s = sample_local[i];
  // the host checks that the requests match the packed batch; a sample
  // beyond its request's buffer is still never written
  if (s >= e.n) return;
  const int64_t n = e.max_len * row_vecs, live = min((int64_t)seqlens[i] * row_vecs, n);
  const V* src = rows + cu_seqlens[i] * row_vecs;
  for (int64_t at = (int64_t)part * kFlat; at < n; at += (int64_t)per * kFlat)
    move_run<ONCE>(src, reinterpret_cast<V*>(e.out) + s * n, at, live, n);
}

// Results beyond the last-level cache are stored non-temporally: packed and unpacked
// again, 300 rows of 4 KB, 225 MB take 158 us with plain and 167 with non-temporal
// stores, 300 MB 228 and 217.
hipError_t launch_pack(hipStream_t s, const ReqEntry* req_table, const int32_t* sample_request,
                       const int32_t* sample_local, const int32_t* seqlens, const int32_t* cu_seqlens, int32_t N,
                       int32_t T, int32_t d, int32_t max_rows, void* tokens, int32_t* token_sample,
                       int32_t* token_pos) {
  const int64_t chunks = d / 8;
  const int32_t per = spread_blocks(max_rows * chunks, T * chunks, N, kFlat);
  if (per == 0) {
    // (4096: two workgroups' worth of every place on the chip)
    const int64_t pieces = (T * chunks + kFlat - 1) / kFlat;
    const int32_t run = kFlat * (int32_t)std::min<int64_t>(kRaggedRuns, std::max<int64_t>(1, pieces / 4096));
    const int64_t blocks = (T * chunks + run - 1) / run;
    pack_ragged_kernel<<<(unsigned)std::min<int64_t>(blocks, kMostBlocks), 256, 0, s>>>(
        req_table, sample_request, sample_local, seqlens, cu_seqlens, N, T, d, run,
        reinterpret_cast<u32x4p*>(tokens), token_sample, token_pos);
    return hipGetLastError();
  }
  auto go = [&](auto once) {
    pack_kernel<once()><<<(unsigned)N * per, 256, 0, s>>>(
        req_table, sample_request, sample_local, seqlens, cu_seqlens, d, reinterpret_cast<u32x4p*>(tokens), token_sample,
        token_pos, per);
    return hipGetLastError();
  };
  return T * chunks * 16 > kStreamBytes ? go(std::true_type()) : go(std::false_type());
}

int32_t unpack_blocks(ReqEntry* table, int32_t R, int32_t N, int64_t row_bytes, bool vec16, int32_t* per) {
  const int64_t vecs = row_bytes / (vec16 ? 16 : 4);
  int64_t most = 0, all = 0, blocks = 0;
  for (int32_t r = 0; r < R; ++r) {
    most = std::max(most, table[r].max_len * vecs);
    all += table[r].n * (table[r].max_len * vecs);
  }
  *per = spread_blocks(most, all, N, kFlat);
  if (*per > 0) return N * *per;
  for (int32_t r = 0; r < R; ++r) {
    table[r].block = (int32_t)blocks;
    blocks += table[r].n * std::min<int64_t>((table[r].max_len * vecs + kFlat - 1) / kFlat, most_per(N));
  }
  return (int32_t)blocks;
}

hipError_t launch_unpack(hipStream_t s, const ReqEntry* req_table, int32_t R, const int32_t* sample_request,
                         const int32_t* sample_local, const int32_t* seqlens, const int32_t* cu_seqlens, int32_t N,
                         int32_t blocks, int32_t per, const void* rows, int64_t row_bytes, bool vec16,
                         int64_t out_bytes) {
  // vec16: the caller checked that the source, every destination and the row
  // pitch are 16-byte aligned
  const int64_t vecs = row_bytes / (vec16 ? 16 : 4);
  auto go = [&](auto v, auto ragged, auto once) {
    typedef decltype(v) V;
    unpack_kernel<V, ragged(), once()><<<(unsigned)blocks, 256, 0, s>>>(
        req_table, R, sample_request, sample_local, seqlens, cu_seqlens, reinterpret_cast<const V*>(rows), vecs,
        ragged() ? most_per(N) : per, N);
    return hipGetLastError();
  };
  auto form = [&](auto v) {
    if (per == 0) return go(v, std::true_type(), std::false_type());
    return out_bytes > kStreamBytes ? go(v, std::false_type(), std::true_type())
                                    : go(v, std::false_type(), std::false_type());
  };
  return vec16 ? form(u32x4p()) : form(uint32_t());
}

}  // namespace jnx
