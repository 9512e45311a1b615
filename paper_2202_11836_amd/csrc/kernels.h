// Host-side launchers of the encoder-stage kernels (gfx950).  Every launcher
// enqueues on the given stream and returns the launch status; none of them
// synchronises.  Shapes are validated by the caller (the stage engine).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

// ---------------------------------------------------------------------------
// GEMM:  C[m, n] = sum_k A(m, k) * B(k, n), then an epilogue.
//   A(m, k) = A[m * lda + k]  if a_kmajor  else  A[k * lda + m]
//   B(k, n) = B[n * ldb + k]  if b_kmajor  else  B[k * ldb + n]
// fp32, batched over grid z: batch index zb splits into (zb / zdiv, zb % zdiv),
// and each operand is offset by (zb / zdiv) * s*1 + (zb % zdiv) * s*2.
// With ksplit > 1 the K range is cut into ksplit chunks of kchunk elements
// and each chunk writes an fp32 partial to C + split * M * ldc (EPI_PARTIAL).
// ---------------------------------------------------------------------------
enum GemmEpi {
  EPI_STORE = 0,    // C = alpha * acc (+ bias[n] when bias != nullptr)
  EPI_GELU = 1,     // u = acc + bias[n]:  GELU(u) -> C;  GELU'(u) -> C2
  EPI_MUL = 2,      // C = acc * aux[m, n]  (the FFN backward: dU = dG * GELU'(u))
  EPI_RESID = 3,    // C = acc + aux[m, n]  (fp32)
  EPI_PARTIAL = 4,  // fp32 C[split][m][n] = acc over this split's K range
  EPI_DSUM = 5,     // C = acc (dO), and per row and head (64 columns) of C as stored
                    // the sum over its columns of C * (aux + aux2): rowsum(dO * O)
};

struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  void* C2;
  const float* bias;
  const void* aux;
  const void* aux2;  // EPI_DSUM: the rounding residual of aux (same layout)
  // EPI_DSUM: receives the sums, row m = b S + s of head j at dsum[(b * (N / 64)
  // + j) * S + s]
  float* dsum;
  int dsum_S;
  int M, N, K;
  int64_t lda, ldb, ldc, ldaux;
  int zdiv;
  int64_t sA1, sA2, sB1, sB2, sC1, sC2;
  int ksplit;
  int kchunk;
  float alpha;
  int tile;  // bf16: a GemmTile, 0 = gemm_bf16_plan's choice
  // EPI_MUL on bf16: column sums of the stored output per block of
  // gemm_colpart_rows(tile) rows, colpart[m / rows][n].
  // fp32: column sums of the stored output per block of 32 rows of each batch
  // entry, colpart[(zb / zdiv) * cp_batch + (m / 32) * cp_ld + (zb % zdiv) *
  // sC2 + n].
  float* colpart;
  int64_t cp_batch, cp_ld;
};

inline GemmArgs gemm_args(const void* A, int64_t lda, const void* B, int64_t ldb, void* C,
                          int64_t ldc, int M, int N, int K) {
  GemmArgs g{};
  g.A = A; g.B = B; g.C = C; g.lda = lda; g.ldb = ldb; g.ldc = ldc;
  g.M = M; g.N = N; g.K = K; g.zdiv = 1; g.ksplit = 1; g.kchunk = K; g.alpha = 1.0f;
  return g;
}

// Compute units of the device (256 without one), asked once.
int device_cus();

// Tile shapes of the bf16 GEMMs: the first in gemm.hip (persistent work-
// groups), the others in gemm_mid.hip.
enum GemmTile {
  GEMM_TILE_256x256 = 1,
  GEMM_TILE_256x128 = 2,
  GEMM_TILE_128x128 = 3,
  GEMM_TILE_128x64 = 4,
  GEMM_TILE_64x64 = 5
};
struct GemmPlan {
  int tile;
  int ks;  // splits of K (1 unless `split`)
};
// Tile (and, with split, the number of K splits) for a bf16 GEMM.  split: the
// consumer sums fp32 partials, so the output may be GEMM_SPLIT_MAX or fewer
// partials, of at most max(M * N, GEMM_SPLIT_ELEMS) elements in all.
constexpr int GEMM_SPLIT_MAX = 6;
constexpr int64_t GEMM_SPLIT_ELEMS = (int64_t)4 << 20;
GemmPlan gemm_bf16_plan(int M, int N, int K, bool b_kmajor, GemmEpi epi, bool split);
// Rows per column partial sum of EPI_MUL with this tile, and the most partial
// rows any token count up to M needs.
inline int gemm_colpart_rows(int tile) {
  return tile == GEMM_TILE_64x64 ? 64 : tile == GEMM_TILE_256x128 ? 256 : 128;
}
int64_t gemm_colpart_max(int64_t M);
// bf16 operands on MFMA (fp32 accumulation), A k-major, batch 1.  b k-major:
// EPI_STORE, EPI_GELU, EPI_PARTIAL; n-major: EPI_STORE, EPI_MUL, EPI_PARTIAL,
// and EPI_DSUM with the tiles of gemm_mid.hip.
// EPI_PARTIAL writes fp32 (C[split][M][ldc], ksplit splits of kchunk), the
// others bf16.
hipError_t gemm_bf16(const GemmArgs& g, bool b_kmajor, GemmEpi epi, hipStream_t st);
// g with its K range cut into ks chunks of whole k-tiles.
inline GemmArgs gemm_split(GemmArgs g, int ks) {
  g.kchunk = ((g.K + ks - 1) / ks + 63) / 64 * 64;
  g.ksplit = (g.K + g.kchunk - 1) / g.kchunk;
  return g;
}
// fp32 operands on fp32 MFMA, same conventions: A k-major, ksplit 1; B
// k-major with EPI_STORE or EPI_GELU, n-major with EPI_STORE, EPI_MUL or
// EPI_RESID.
hipError_t gemm_f32(const GemmArgs& g, bool a_kmajor, bool b_kmajor, GemmEpi epi, int batch,
                    hipStream_t st);
// The attention backward's dV = P^T dC, dK = dS^T Q and, unless null, dQ = dS K
// of every (batch, head) in one launch (equal M and N, EPI_STORE).
hipError_t gemm_f32_attn_bwd(const GemmArgs& dv, const GemmArgs& dk, const GemmArgs* dq, int batch,
                             hipStream_t st);

// Up to GEMM_GROUP_MAX weight-gradient GEMMs in one launch, stream-K: each
// problem p[q] is a GEMM with both operands m/n-major (A(m, k) = A[k * lda +
// m], B(k, n) = B[k * ldb + n]: token-major activations and output
// gradients), batch 1, and all share one K.  The k-tiles (of 64) of their
// 256 x 256 tiles are laid end to end in two phases, the first kf k-tiles
// of every tile, then the rest of every tile, and the sequence is cut into
// one contiguous range per work-group (one work-group per CU); kf is the
// average range length when a tile holds more than that, so that the
// work-groups of the first phase each own one tile's first kf k-tiles and
// all run over the same k at the same time.  The part of a range inside one
// tile's phase (a piece) writes an fp32 partial to slot j of its problem's C
// (C + j * M * ldc), j = its rank among that tile's pieces in k order;
// wgrad_group_reduce then sums each tile's pieces in k order.  ksplit /
// kchunk of p[q] are ignored.
constexpr int GEMM_GROUP_MAX = 4;
struct GemmGroup {
  GemmArgs g[GEMM_GROUP_MAX];
  int n;
  int tile0[GEMM_GROUP_MAX + 1];  // first (global) tile of each problem; tile0[n] = all tiles
  int kt;                         // k-tiles per tile, ceil(K / 64)
  int kf;                         // k-tiles of each tile in the first phase
  int64_t work;                   // k-tiles over all tiles, tile0[n] * kt
};
// Slots of M x N fp32 partials each problem's C must hold for the plan of
// such a group (the most pieces of one tile) on this device: 0 when the plan
// needs none, -1 for invalid sizes.
int wgrad_group_slots(const int* M, const int* N, int n, int K);
hipError_t gemm_bf16_wgrad_group(const GemmArgs* p, int n, hipStream_t st);
// A gradient on the backward residual stream of a bf16 stage: one bf16 tensor
// bf, or the fp32 sum (hi + lo) + product of a residual branch carried as its
// bf16 rounding and rounding residual and a data-gradient GEMM's product, in
// bf16 (b) or as np fp32 partials pf, n elements apart (n: the tensor's size).
struct GradIn {
  const bf16_t* bf;
  const bf16_t* hi;
  const bf16_t* lo;
  const bf16_t* b;
  const float* pf;
  int np;  // 2, 4 or 6 with pf
};
// Column reductions, and the rounding of a gradient, run with a layer's weight
// gradients (tail.h): out[v][c] = the sum over the nblk partial rows b of
// part[(b * nvec + v) * n + c], v < nvec <= 4, in a fixed order (null outputs
// are skipped);  gout (may be null) = gin (a sum, not bf) rounded to bf16, gn
// elements (a multiple of 8).  units, unit0: set by the launchers.
struct ColJob {
  const float* part;
  int nblk, nvec, n;
  float* out[4];
};
constexpr int COLJOB_MAX = 4;
struct TailJobs {
  ColJob col[COLJOB_MAX];
  int ncol;
  int unit0[COLJOB_MAX + 1];
  int units;
  GradIn gin;
  bf16_t* gout;
  int64_t gn;
};
// out[q][m][n] = the sum over the pieces of (m, n)'s tile of slot j of
// p[q].C, in k order (same p as the GEMM launch), and the jobs of tail, in one
// launch.
hipError_t wgrad_group_reduce(const GemmArgs* p, float* const* out, int n, const TailJobs& tail,
                              hipStream_t st);

// Whether the bf16 GEMMs take g's shapes and strides.
bool gemm_bf16_ok(const GemmArgs& g, bool b_kmajor);
// gemm_bf16 with one of the tiles of gemm_mid.hip.
hipError_t gemm_mid(const GemmArgs& g, bool b_kmajor, GemmEpi epi, int tile, hipStream_t st);
// Whether the weight-gradient launches take n problems (both operands m/n-major,
// one K) of these shapes and strides.
bool wgrad_args_ok(const GemmArgs* p, int n);
// n weight gradients (operands m/n-major, ldc = N), each written whole, and
// the jobs of tail, in one launch.
hipError_t gemm_mid_wgrad(const GemmArgs* p, float* const* out, int n, int tile,
                          const TailJobs& tail, hipStream_t st);
// How a layer's weight gradients are computed: 0 = the stream-K group above
// with its reduction, else a tile of gemm_mid_wgrad (no partials).
int wgrad_plan(const int* M, const int* N, int n, int K);

// Weight gradients of one fp32 layer (both operands m/n-major, equal K) and the
// jobs of tail, in one launch; with ks > 1 splits over K (p[q].C holds ks slots
// of M x N partials) a second one has the splits' fixed-order sums and the tail.
// plan: gemm_f32_wgrad_plan of the whole layer (width h, feed-forward width f),
// also when only one half of it is computed: splits and tiles set the order of
// the sums, and a half-layer stage sums in the same order as a whole one.
struct F32WgradPlan {
  int ks;      // splits over K
  bool small;  // 32 x 32 tiles (else 64 x 64)
};
F32WgradPlan gemm_f32_wgrad_plan(int h, int f, int K);
hipError_t gemm_f32_wgrad_group(const GemmArgs* p, float* const* out, int n, F32WgradPlan plan,
                                const TailJobs& tail, hipStream_t st);

// ---------------------------------------------------------------------------
// Row kernels (one wavefront per row), T = float or bf16_t.
// ---------------------------------------------------------------------------
// z = a + bias + resid (+ resid_lo);  y = gamma * xhat + beta with
// xhat = (z - mean) * rstd.  a is the fp32 output of the preceding GEMM, the
// sum of np partials rows * h apart (np = 1, 2, 4 or 6);
// resid_lo (optional, may be null) is the rounding residual of resid; ylo
// (optional, may be null) receives y - y as stored, in T.
template <typename T, typename TA>
hipError_t add_ln_fwd(const TA* a, int np, const float* bias, const T* resid, const T* resid_lo,
                      const float* gamma, const float* beta, T* y, T* ylo, T* xhat, float* rstd,
                      int rows, int h, hipStream_t st);

// dz = rstd * (g - mean(g) - xhat * mean(g * xhat)), g = dy * gamma.
// Column partial sums per block of ln_bwd_rpb(rows) rows (ln_bwd_blocks(rows)
// blocks): part[blk][0][:] = sum dy*xhat, part[blk][1][:] = sum dy,
// part[blk][2][:] = sum dz.
int ln_bwd_rpb(int rows);
int ln_bwd_blocks(int rows);
int ln_bwd_blocks_max(int rows);  // the most any number of rows up to this one needs
hipError_t ln_bwd_f32(const float* dy, const float* xhat, const float* rstd, const float* gamma,
                      float* dz, float* part, int rows, int h, hipStream_t st);

// bf16 stages: ln_bwd_f32 for such a gradient.  dz in bf16 and, when dzlo is
// not null, dz's bf16 rounding residual.
hipError_t ln_bwd_bf16(const GradIn& dy, const bf16_t* xhat, const float* rstd, const float* gamma,
                       bf16_t* dz, bf16_t* dzlo, float* part, int rows, int h, hipStream_t st);
// out = the gradient (any form of it) in fp32, n elements (a multiple of 8).
hipError_t grad_f32(const GradIn& in, float* out, int64_t n, hipStream_t st);

// Start of a forward pass: X = x (nx bytes, a multiple of 16; both 16-byte
// aligned); mask = key_mask, or all ones when that is null; when kext is not
// null, kext[b] = 1 + last s with mask[b][s] != 0 (0 if none).
struct PrepArgs {
  const void* x;
  void* X;
  int64_t nx;
  const uint8_t* key_mask;
  uint8_t* mask;
  int B, S;
  int* kext;
};
hipError_t stage_prep(const PrepArgs& p, hipStream_t st);
// The same beside gemm_bf16(g, true, epi, st) in its launch (EPI_STORE or
// EPI_GELU with a tile of gemm_mid.hip; g may read x, not X).
hipError_t gemm_mid_prep(const GemmArgs& g, GemmEpi epi, const PrepArgs& p, hipStream_t st);

// part[blk][n] = sum over the block's rows of x[row][n].
template <typename T>
hipError_t col_partial(const T* x, int rows, int n, float* part, int nblk, hipStream_t st);

// ---------------------------------------------------------------------------
// Attention row kernels on a materialised score matrix.
// scores/dP: fp32 [B*H][S][ld]; P, dS: T [B*H][S][ld]; mask: uint8 [B][S].
// ---------------------------------------------------------------------------
template <typename T>
hipError_t softmax_fwd(const float* scores, const uint8_t* mask, T* P, int BH, int H, int S,
                       int ld, float scale, hipStream_t st);
template <typename T>
hipError_t softmax_bwd(const float* dP, const T* P, T* dS, int BH, int S, int ld, float scale,
                       hipStream_t st);

// ---------------------------------------------------------------------------
// Fused attention (bf16 stages, head dim 64).
//   qkv:  [B*S, 3h] (Q | K | V, head j = columns 64 j .. 64 j + 63 of each)
//   mask: [B, S] uint8 key mask; kext: [B] ints, 1 + last valid key
//   out:  forward: context [B*S, h]; backward: dQKV [B*S, 3h]
//   lse:  [B*H, S] fp32 log2-sum-exp of the scaled scores (forward output)
//   o, dout: forward context and its gradient [B*S, h] (backward inputs)
//   out_lo / o_lo: the context's bf16 rounding residual [B*S, h]
//   dsum: [B*H, S] fp32 rowsum(dO * O) (written by attn_backward_dq, or by the
//   EPI_DSUM product that makes dO)
// ---------------------------------------------------------------------------
struct AttnArgs {
  // backward, optional: column sums of dQKV per 32-row block of each
  // sequence, colpart[b * ceil(S / 32) + s / 32][3h]
  float* colpart;
  const bf16_t* qkv;
  const uint8_t* mask;
  const int* kext;
  bf16_t* out;
  float* lse;
  const bf16_t* o;
  const bf16_t* dout;
  // forward, optional: the bf16 rounding residual of the context, out_lo =
  // bf16(C - bf16(C)) with C the fp32 context; backward, optional: the same
  // tensor, added to o where D = rowsum(dO * O) is formed
  bf16_t* out_lo;
  const bf16_t* o_lo;
  float* dsum;
  int B, S, H, h;
  float scale_log2;  // softmax scale * log2(e)
  float scale;       // softmax scale
};
// Forward pass (needs kext).
hipError_t attn_forward(const AttnArgs& a, hipStream_t st);
// Backward, into out's Q, K and V blocks: dsum and dQ, then dK and dV; or all in
// one launch, given dsum (EPI_DSUM of the product that makes dout).
hipError_t attn_backward_dq(const AttnArgs& a, hipStream_t st);
hipError_t attn_backward_dkdv(const AttnArgs& a, hipStream_t st);
hipError_t attn_backward(const AttnArgs& a, hipStream_t st);

// ---------------------------------------------------------------------------
// Attention of fp32 stages with S <= ATTN_F32_MAX_S (attn_f32.hip).
//   qkv [B*S, 3h], mask [B, S] as above; P, dS: [B*H, S, S]
//   forward: P = masked softmax(scale Q K^T), out = P V (row stride ldo)
//   backward_rows: dS = scale P (dC V^T - rowsum(P dC V^T)), out = dQ = dS K,
//   and its column sums per 32-row block of each sequence,
//   colpart[b * ceil(S / 32) + s / 32][3h] (the first h columns)
// ---------------------------------------------------------------------------
constexpr int ATTN_F32_MAX_S = 512;
struct AttnF32Args {
  const float* qkv;
  const uint8_t* mask;
  float* P;
  const float* dC;
  float* dS;
  float* out;
  int64_t ldo;
  float* colpart;
  int S, H, h;
  float scale;
};
hipError_t attn_f32_forward(const AttnF32Args& a, int B, hipStream_t st);
hipError_t attn_f32_backward_rows(const AttnF32Args& a, int B, hipStream_t st);
