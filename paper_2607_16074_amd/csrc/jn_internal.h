// Internal declarations shared by the host library and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "joynexus.h"

namespace jnx {

// Device request table entry (one per request), written by jn_pack_group and
// patched by jn_unpack with the output pointer.
struct ReqEntry {
  const void* in;      // bf16 [n][max_len][d]
  void* out;           // unpack destination [n][max_len][row_bytes]
  int32_t max_len;
  int32_t n;
  int32_t first;       // packed index of the request's first sample
  int32_t block;       // ragged unpack: the request's first workgroup
};
static_assert(sizeof(ReqEntry) == 32, "ReqEntry layout");

// Size of the last-level cache: kernels that touch every byte once do so non-
// temporally only where they touch more than this.
constexpr int64_t kStreamBytes = 256 << 20;

// ------------------------------------------------------------ launchers ---
// All launchers enqueue on `s`; shapes were validated by the caller.

// Table of `bytes` at `src` (pinned, coherent) to device memory, and the `tail`
// bytes behind it to `tail_dst`.
constexpr size_t kUploadBytes = 64 << 10;
hipError_t launch_upload(hipStream_t s, void* dst, const void* src, size_t bytes, void* tail_dst, size_t tail);

// Copies of N samples' runs, `all` elements together, the longest `most`: blocks
// for every sample, of `piece` elements at a time, or 0 for a walk over the samples'
// common order.  A workgroup that finds nothing costs a ninth of one that moves 8
// KB (0.3 ns, 2.7), so a sample gets the blocks of twice the mean at most and longer
// ones go round again, up to four times; beyond that the walk, whose searches
// cost about as much as the copy of short runs.
constexpr int32_t kMostBlocks = 0xffffff;  // of 256 threads: a dispatch holds 2^32 - 1 threads
inline int32_t most_per(int32_t N) { return kMostBlocks / N > 1 ? kMostBlocks / N : 1; }
inline int32_t spread_blocks(int64_t most, int64_t all, int32_t N, int64_t piece) {
  const int64_t pieces = (most + piece - 1) / piece, mean = all > 0 ? (all + N * piece - 1) / (N * piece) : 1;
  if (pieces > 8 * mean) return 0;
  const int64_t per = pieces < 4 * mean ? pieces : 2 * mean;
  return (int32_t)(per < most_per(N) ? per : most_per(N));
}

hipError_t launch_pack(hipStream_t s, const ReqEntry* req_table, const int32_t* sample_request,
                       const int32_t* sample_local, const int32_t* seqlens, const int32_t* cu_seqlens,
                       int32_t N, int32_t T, int32_t d, int32_t max_rows, void* tokens,
                       int32_t* token_sample, int32_t* token_pos);

// Workgroups of an unpack and blocks per sample (0: those of each request's own
// padded length, from the `block`s that this fills in).
int32_t unpack_blocks(ReqEntry* table, int32_t R, int32_t N, int64_t row_bytes, bool vec16, int32_t* per);
hipError_t launch_unpack(hipStream_t s, const ReqEntry* req_table, int32_t R, const int32_t* sample_request,
                         const int32_t* sample_local, const int32_t* seqlens, const int32_t* cu_seqlens, int32_t N,
                         int32_t blocks, int32_t per, const void* rows, int64_t row_bytes, bool vec16,
                         int64_t out_bytes);

// x_out (fp32, optional) = widened x_bf16; h = RMS(x) * g  (bf16)
hipError_t launch_rmsnorm_bf16in(hipStream_t s, const void* x_bf16, float* x_out, const void* g,
                                 void* h, int32_t rows, int32_t d, float eps);
// h = RMS(x) * g (bf16) from the fp32 residual stream
hipError_t launch_rmsnorm_f32in(hipStream_t s, const float* x, const void* g, void* h, int32_t rows,
                                int32_t d, float eps);

// x += (part[0] + part[1]) + ... (S fp32 planes of rows x d, added in order),
// then h = RMS(x) * g (bf16): the reduction of a split residual projection
// together with the norm that reads its result.
hipError_t launch_rmsnorm_split(hipStream_t s, float* x, const float* part, int32_t S, const void* g, void* h,
                                int32_t rows, int32_t d, float eps);

enum GemmEpi : int32_t {
  EPI_BF16 = 0,          // C bf16 = acc
  EPI_GELU_BF16 = 1,     // C bf16 = gelu(acc)
  EPI_RESID_F32 = 2,     // C fp32 = (aux, or C itself) + acc
  EPI_GEGLU_BF16 = 3,    // weights gate|up interleaved at load; C bf16 = gelu(gate) * up
  EPI_F32 = 4,           // C fp32 = acc
  EPI_GELU_SAVE = 5,     // aux fp32 = acc; C bf16 = gelu(acc)
  EPI_GELUGRAD_BF16 = 6  // C bf16 = acc * gelu'(aux fp32)
};

// Operand layouts of a grouped problem (GemmArgs::trans): X stored [K][M]
// (element (m, k) at X[k * ldx + m]), W stored [K][N].
constexpr int GEMM_TRANS_X = 1, GEMM_TRANS_W = 2;

// One GEMM problem: C[M][N] (+)= epi(X[M][K] W[N][K]^T); bf16 X, W row-major
// unless `trans` says otherwise.
struct GemmArgs {
  const uint16_t* X;
  const uint16_t* W;
  const uint16_t* W2;   // GeGLU up weights
  void* C;
  float* aux;           // GELU pre-activation (saved or read); residual source (null: C)
  int64_t ldx, ldw, ldc, ldaux;
  int32_t M, N, K;
  int32_t tiles_m, tiles_n, tile_start;  // filled by the launchers
  int32_t trans;        // GEMM_TRANS_* bits (grouped launches only)
  int64_t split_c;      // split-K: elements between the fp32 partial outputs of
                        // consecutive K ranges; 0 when unsplit
};

// Grouped launch over nprob problems sharing one epilogue: the host fills
// the problems, calls gemm_grouped_prepare (tile ranges, returns the tile
// total, or -1 if a problem is not M, N, K > 0 with K % 64 == 0 and
// N % 32 == 0), uploads them and launches.  shape from gemm_grouped_tile_shape.
// Problems with transposed operands (all of one launch alike) have no shape
// (-1) where their offsets do not fit 32 bits; with both operands transposed K
// need not be a multiple of 64.  Combinations launched: EPI_F32 with
// GEMM_TRANS_W or both, EPI_GELUGRAD_BF16 with GEMM_TRANS_W.
// uneven: gemm_grouped_uneven of the problems; gemm_grouped_prepare then sorts
// them, longest contraction first.
int gemm_grouped_tile_shape(int epi, const GemmArgs* probs, int32_t nprob);
bool gemm_grouped_uneven(const GemmArgs* probs, int32_t nprob);
int32_t gemm_grouped_prepare(GemmArgs* probs, int32_t nprob, int shape);
hipError_t launch_gemm_grouped(hipStream_t s, int epi, const GemmArgs* dprobs, int32_t nprob, int32_t total_tiles,
                               int shape, int trans, bool uneven);

// A data gradient (GEMM_TRANS_W) and a weight gradient (EPI_F32, both operands
// transposed), prepared as above with the shapes that gemm_grad_pair_ok takes,
// in one launch; neither reads what the other writes.
bool gemm_grad_pair_ok(int epi, int dshape, int wshape, int32_t wtiles);
hipError_t launch_gemm_grad_pair(hipStream_t s, int epi, const GemmArgs* dprobs, int32_t nd, int32_t td,
                                 const GemmArgs* wprobs, int32_t nw, int32_t tw);

// C[M][N] (+)= epi(A[M][K] * B[N][K]^T); A, B bf16 row-major with leading
// dims lda, ldb (elements); for EPI_GEGLU_BF16, B is w_gate and B2 is w_up,
// each [N][K], and C has N columns.
//
// Launches with few tiles for the GPU and a long K (epilogues EPI_BF16,
// EPI_RESID_F32, EPI_GELU_BF16) split K: each of S ranges writes fp32 partials
// [S][rows][N] into `split_ws` (gemm_split_bytes(), 0 where nothing is split)
// and a reduction adds them in range order, then applies the epilogue.  The
// split depends only on (epi, M, N, K).  gemm_split(): S of a launch that is
// split over all its rows, else 1; with partials_only such a launch leaves the
// reduction to the caller (launch_rmsnorm_split).
hipError_t launch_gemm(hipStream_t s, int epi, const void* A, int64_t lda, const void* B,
                       const void* B2, int64_t ldb, void* C, int64_t ldc, int32_t M, int32_t N,
                       int32_t K, void* split_ws = nullptr, size_t split_bytes = 0, bool partials_only = false);
int32_t gemm_split(int epi, int32_t M, int32_t N, int32_t K);
struct GemmPlan {
  int32_t m1 = 0;      // rows of the leading ring launch (0: none)
  int32_t shape = 0;   // the other rows: 256x256, 256x160, 256x128, 128x160, 128x96, 64x96, 128x128
  int32_t S = 1;
};
GemmPlan gemm_plan(int epi, int32_t M, int32_t N, int32_t K);
size_t gemm_split_bytes(int epi, int32_t M, int32_t N, int32_t K);

// Varlen attention over the packed batch (bidirectional or causal inside each
// sample).  qkv: bf16 [T][(H + 2 Hkv) hd] (q | k | v); out: bf16 [T][d],
// d = H hd.  Query head h reads key/value head h / (H / Hkv).  Alignment rows
// of `out` are zeroed.
hipError_t launch_attention(hipStream_t s, const void* qkv, void* out, const int32_t* seqlens,
                            const int32_t* cu_seqlens, int32_t N, int32_t d, int32_t n_heads, int32_t n_kv_heads,
                            bool causal, int32_t max_seqlen, int32_t align);
// In-place rotary embedding of the first `heads` head slices (hd wide) of
// every row of qkv [T][ld] whose token_pos >= 0: pair (i, i + hd/2) rotated
// by token_pos * theta^(-2i/hd).
hipError_t launch_rope(hipStream_t s, void* qkv, int32_t ld, const int32_t* token_pos, int32_t T, int32_t heads,
                       int32_t hd, float theta);

// ---- heads ----
// pooled[sample_tenant_rank[i]][:] = mean over valid rows of hidden for sample i
hipError_t launch_pool(hipStream_t s, const void* hidden, const int32_t* seqlens,
                       const int32_t* cu_seqlens, const int32_t* rank, int32_t N, int32_t d,
                       float* pooled);

// One fp32 GEMM of a tenant head, C(m, n) = sum_k A B, of one of three kinds:
//   FWD    A = X [row][k], B = W [n][k], C [row][n]
//   DGRAD  A = dZ [row][k], B = W [k][n], C [row][n]
//   WGRAD  A = dZ [row][m], B = X [row][n], C = dW [m][n], contracted over
//          the tenant's rows
// Row operands are tenant-ordered buffers: the kernel starts at the tenant's
// first row (tenant_sample_off, read on the device), and its row count stands
// for M (FWD, DGRAD) or K (WGRAD).
struct HeadGemm {
  const float* A;
  const float* B;
  float* C;
  const float* bias;    // FWD: C += bias[n]
  float* Cact;          // FWD: also store gelu(C) (same layout as C; may be null)
  const float* Zg;      // DGRAD: C *= gelu'(Zg) (same layout as C)
  float* db;            // WGRAD: db[m] = sum of A over the rows
  // FWD of a training head's last layer (target set): actions = y, C = dL/dy of
  // L = mean((y - target)^2), and the tile's sum of squared errors in lpart;
  // target and actions are the tenant's own [n_g][N] buffers.  The last layer's
  // WGRAD: lpart, and loss for the tenant's loss tile
  const float* target;
  union {
    float* actions;
    float* loss;
  };
  float* lpart;         // [row tile of all tenants][ldp]: tenant t starts at off_t / 32 + t
  int64_t lda, ldb, ldc;
  int32_t M, N, K;      // M: WGRAD only; K: FWD and DGRAD only
  int32_t own_rows;     // FWD: C is the tenant's own buffer (rows from 0)
  int32_t ldp;
  int32_t reserved;
};
struct HeadTile {
  int32_t desc;
  int32_t tenant;
  int32_t tm;  // WGRAD (FWD and DGRAD: 0); kHeadLossTile: sum the tenant's lpart
  int32_t tn;
};
constexpr int kHeadTile = 32;                        // FWD and DGRAD tiles are 32 x 32
constexpr int kHeadWgradM = 64, kHeadWgradN = 256;   // WGRAD tiles
constexpr int32_t kHeadLossTile = -1;
constexpr int32_t kHeadLongRows = 256;               // up to here no WGRAD is cut into K ranges
// The first nrow of the list are column tiles of FWD or DGRAD, each run for row
// tiles 0 .. tms - 1; the nown behind them (WGRAD and loss tiles) run once.
// forward: every tile is FWD; otherwise none is.
struct HeadLaunch {
  int32_t first = 0, nrow = 0, nown = 0;
};
hipError_t launch_head_gemm(hipStream_t s, const HeadGemm* descs, const HeadTile* tiles, const HeadLaunch& n,
                            int32_t tms, const int32_t* tenant_sample_off, bool forward);

// ---- action expert (k_expert.hip) ----
// dst[r][c] = cvt(src[r][c]) for r < src_rows, c < src_cols, else 0; r < rows, c < cols.
struct CopyDesc {
  const void* src;
  void* dst;
  int64_t src_ld, dst_ld;
  int32_t rows, cols, src_rows, src_cols;
  int32_t src_bf16, dst_bf16;
  int32_t block_start, vec;  // filled by copy2d_prepare
};
int32_t copy2d_prepare(CopyDesc* d, int32_t n);

// dst[i] = ((src[0][i] + src[1][i]) + ...) + src[S-1][i], i < n (parts
// n elements apart, fp32; n % 4 == 0, 16-byte aligned): the K ranges of a
// split weight gradient added in range order.
struct KSumDesc {
  const float* src;
  float* dst;
  int64_t n;
  int32_t S;
  int32_t block_start;  // filled by ksum_prepare
};
int32_t ksum_prepare(KSumDesc* d, int32_t n);
hipError_t launch_ksum(hipStream_t s, const KSumDesc* d, int32_t n, int32_t blocks);
hipError_t launch_copy2d(hipStream_t s, const CopyDesc* d, int32_t n, int32_t blocks);

// bf16 dst[c][r] = src[r][c] (r < rows), 0 for rows <= r < rows_pad; c < cols.
struct TransDesc {
  const uint16_t* src;
  uint16_t* dst;
  int64_t src_ld, dst_ld;
  int32_t rows, cols, rows_pad, block_start;
};
int32_t transpose_prepare(TransDesc* d, int32_t n);
hipError_t launch_transpose(hipStream_t s, const TransDesc* d, int32_t n, int32_t blocks);

// zoff[k] for tenant-order samples k (prefix sums of their valid lengths) and
// the tenant-ordered copy z of their backbone rows (rows >= cap dropped).
hipError_t launch_prefix(hipStream_t s, const void* hidden, const int32_t* tenant_perm, const int32_t* seqlens,
                         const int32_t* cu_seqlens, int32_t N, int32_t max_seqlen, int32_t d, int64_t cap,
                         int32_t* zoff, void* z);

// RMSNorm with per-tenant gains (rows tenant-contiguous, roff [G+1] device).
hipError_t launch_xrms_fwd(hipStream_t s, const float* x, const void* const* gains, const int32_t* roff, int32_t G,
                           int32_t rows, int32_t d, float eps, void* h);
// dx (+)= dRMS(x, g) . dh (set instead of added to where `first`), dxb = its
// bf16 copy; part [segs][d]: column sums of dh x r over each segment.  Tenant
// t's rows are cut into segments of kXrmsSeg, numbered from soff[t] (soff [G+1]
// device, `segs` in all).
constexpr int kXrmsSeg = 8;
hipError_t launch_xrms_bwd(hipStream_t s, const float* x, const void* const* gains, const int32_t* roff,
                           const int32_t* soff, int32_t G, int32_t segs, int32_t d, float eps, const float* dh,
                           bool first, float* dx, uint16_t* dxb, float* part);
// dg[n G + t] = sum over tenant t's segments of part [norms][segs][d].
hipError_t launch_gain_sums(hipStream_t s, const float* part, const int32_t* soff, int32_t G, int32_t segs, int32_t d,
                            int32_t norms, float* const* dg);

// fp32 attention of each tenant-order sample k over its own keys: queries
// rows [k*Lq, (k+1)*Lq) of Q; keys / values rows [kv0, kv0 + Lk) with
// kv0 = zoff[k], Lk = zoff[k+1] - zoff[k] (cross, clamped to kv_cap) or the
// sample's own query rows (self, zoff null).
struct AttnArgs {
  const uint16_t* Q;  // bf16
  const uint16_t* K;
  const uint16_t* V;
  float* O;        // forward output / backward input (fp32)
  uint16_t* Ob;    // forward output, bf16 copy of O (leading dimension ldo)
  float* lse;      // forward output / backward input, [rows][nheads], log2 domain
  const float* dO;
  uint16_t* dQ;    // bf16 gradients
  uint16_t* dK;
  uint16_t* dV;
  const int32_t* zoff;
  int64_t ldq, ldkv, ldo, lddq, lddkv, kv_cap;
  int32_t kcol, vcol, dkcol, dvcol;
  int32_t Lq, hd, nheads, max_lk;    // max_lk: largest key count of any sample
  float scale;
};
hipError_t launch_xattn(hipStream_t s, const AttnArgs& A, int32_t nsamples, bool backward);

// Flow-matching inputs of one tenant's expert rows (rows = n * chunk, tenant
// arrival order): input row [x | 0 | phi(t)] (bf16, ld columns: x = t*noise +
// (1-t)*act in the first a, zeros up to kap, the d_time flow-time features
// after) and vel = noise - act (fp32 [rows][a]).
struct FlowDesc {
  const float* t;       // [n]
  const float* noise;   // [rows][a]
  const float* act;     // [rows][a]
  float* vel;           // [rows][a]
  int64_t roff;         // first row of the tenant in the expert's row space
  int32_t rows, a;
};
hipError_t launch_flow_prep(hipStream_t s, const FlowDesc* d, int32_t G, int64_t total_rows, int32_t chunk,
                            int32_t kap, int32_t d_time, uint16_t* in_rows, int32_t ld);

struct XLossDesc {
  const float* target;  // [rows_t][a]
  float* pred;          // [rows_t][a]
  float* loss;          // [1]
  int32_t a, reserved;
};
// dpred_pad: bf16 [rows][ldp], zero past the tenant's a columns; part: scratch
// of kXLossParts floats per tenant.
constexpr int kXLossParts = 64;
hipError_t launch_xloss(hipStream_t s, const XLossDesc* d, const int32_t* roff, int32_t G, const float* pred_pad,
                        int32_t ldp, uint16_t* dpred_pad, float* part);

// ------------------------------------------------------------ optimizer ---

struct AdamwTensor {
  float* p;
  const float* g;
  float* m;
  float* v;
  uint16_t* b16;        // optional bf16 copy of the new parameters
  int64_t numel;
  int32_t tenant, block_start;
};
// per tenant: p = p * decay - step_size * m / (sqrt(v) * inv_sqrt_bc2 + eps)
struct AdamwTenant {
  float decay, step_size, inv_sqrt_bc2, eps, b1, b2, reserved0, reserved1;
};
constexpr int64_t kAdamwBlockElems = 2048;
int32_t adamw_prepare(AdamwTensor* t, int32_t n);  // fills block_start, returns the block count
hipError_t launch_adamw(hipStream_t s, const AdamwTensor* t, int32_t n, const AdamwTenant* ten, int32_t blocks);

}  // namespace jnx
