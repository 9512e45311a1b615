// Masked self-attention of fp32 stages (head dim 64, sequences of up to
// ATTN_F32_MAX_S tokens), forward and the row half of the backward, on
// v_mfma_f32_16x16x4_f32.
//
// A work-group has 32 query rows of one (batch, head).  Its 32 x S scores (or
// dP) stay in LDS from the product that makes them through the softmax (or
// its derivative) to the product that uses them; the probabilities P (or dS)
// also go to memory, where the backward (or its dV and dK) reads them.  As
// three launches (scores, softmax, context) each read and wrote the score
// matrix, and the smallest stages' time is their launches: BERT-base 16 x 128
// 43 -> 23 us forward, the attention backward 52 -> 49 us; two
// layers of width 128 at 2 x 32 take 8 launches fewer, 164 -> 156 us a step.
//
// Four wavefronts, 16 x 16 output blocks: in the first product each takes one
// half of the rows and every other block of 16 keys, operands straight from
// memory (K = 64: one read of each row, 16 bytes a lane), in the second 16 of
// the 64 columns.  With 32 x 32 blocks a 32-token sequence left three
// wavefronts idle for 2048 cycles, and no launch was saved that this did not
// cost.  What the second product (and the softmax derivative) reads first is
// requested at the start.
#include "kernels.h"

namespace {

constexpr int HD = 64;

// One 16 x 16 block: lane l has A row, B column l % 16 at k = l / 16, and C rows
// 4 (l / 16) .. + 3 of column l % 16.
__device__ __forceinline__ f32x4_t mfma4(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// LD: row length of the LDS matrix, 8 more than a multiple of 64 (the 8 rows
// x 8 columns of a softmax access, and the rows of a fragment read, then fall
// on distinct banks); S <= LD - 8.
template <bool BWD, int LD>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnF32Args a) {
  __shared__ __attribute__((aligned(16))) float sc[32 * LD];
  __shared__ uint8_t msk[BWD ? 1 : LD];
  const int S = a.S, h = a.h, nq = (S + 31) / 32;
  int w = blockIdx.x;  // each XCD takes a contiguous range: row blocks share keys
  const int n = gridDim.x;
  if ((n & 7) == 0) w = (w & 7) * (n >> 3) + (w >> 3);
  const int qb = w % nq, bh = w / nq, b = bh / a.H, j = bh % a.H, q0 = qb * 32;
  const int tid = threadIdx.x, lane = tid & 63, kq = lane >> 4, rr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t ld = 3 * (int64_t)h;
  const float* Q = a.qkv + (int64_t)b * S * ld + j * HD;
  const float* K = Q + h;
  const float* V = Q + 2 * h;
  const int ng = (S + 15) / 16;  // groups of 16 keys

  // sc = Q K^T, or dC V^T (rows and keys past the last: repeats of it, not
  // used).  Lanes hold k = 16 g + 4 kq + i of their row.
  const int rh = 16 * (wave & 1);
  f32x4_t fa[4], fb[2][4];
  {
    const int q = min(q0 + rh + rr, S - 1);
    const float* A = BWD ? a.dC + ((int64_t)b * S + q) * h + j * HD : Q + q * ld;
#pragma unroll
    for (int g = 0; g < 4; ++g) fa[g] = *(const f32x4_t*)(A + 16 * g + 4 * kq);
  }
  auto keys = [&](f32x4_t (&f)[4], int kb) {
    const float* B = (BWD ? V : K) + min(16 * kb + rr, S - 1) * ld;
#pragma unroll
    for (int g = 0; g < 4; ++g) f[g] = *(const f32x4_t*)(B + 16 * g + 4 * kq);
  };
  keys(fb[0], wave >> 1);
  // (first reads of the later phases)
  constexpr int PRE = 4;
  const float* B2 = (BWD ? K : V) + 16 * wave + rr;
  float vb[PRE][4];
#pragma unroll
  for (int g = 0; g < PRE; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) vb[g][i] = B2[min(16 * g + 4 * kq + i, S - 1) * ld];
  const float* Pg = a.P + ((int64_t)bh * S + q0 + 8 * wave) * S;
  const int live = min(8, S - q0 - 8 * wave);  // rows 8 wave .. that exist (may be < 0)
  float p0[8];
  if constexpr (BWD) {
#pragma unroll
    for (int r = 0; r < 8; ++r) p0[r] = (r < live && lane < S) ? Pg[(int64_t)r * S + lane] : 0.0f;
  }
  auto scores = [&](const f32x4_t (&f)[4], int kb) {
    f32x4_t acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i & 1] = mfma4(fa[g][i], f[g][i], acc[i & 1]);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      sc[(rh + 4 * kq + r) * LD + 16 * kb + rr] = acc[0][r] + acc[1][r];
  };
  for (int kb = wave >> 1; kb < ng; kb += 4) {
    if (kb + 2 < ng) keys(fb[1], kb + 2);
    scores(fb[0], kb);
    if (kb + 4 < ng) keys(fb[0], kb + 4);
    if (kb + 2 < ng) scores(fb[1], kb + 2);
  }
  if constexpr (!BWD)
    for (int c = tid; c < 16 * ng; c += 256) msk[c] = c < S ? a.mask[(int64_t)b * S + c] : 0;
  __syncthreads();

  // Rows 8 wave .. + 7: P = softmax(scale * sc) over the valid keys (none, or a
  // sum that is not a positive number: a row of zeros, as in softmax_fwd),
  // or dS = scale * P * (sc - rowsum(sc * P)); columns S .. 16 ng - 1 get 0.
  float* rows = sc + 8 * wave * LD;
  if constexpr (!BWD) {
    // eight lanes per row
    float* row = rows + (lane >> 3) * LD;
    const int c0 = lane & 7;
    float mx = -INFINITY;
#pragma unroll 4
    for (int c = c0; c < S; c += 8) mx = fmaxf(mx, msk[c] ? a.scale * row[c] : -INFINITY);
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    float sum = 0.0f;
#pragma unroll 4
    for (int c = c0; c < 16 * ng; c += 8) {  // (msk is 0 from S on)
      const float s = row[c];
      const float e = msk[c] ? expf(a.scale * s - mx) : 0.0f;
      row[c] = e;
      sum += e;
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) sum += __shfl_xor(sum, o, 64);
    const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
    __syncthreads();
    float f[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) f[r] = __shfl(inv, 8 * r, 64);
    float* Pw = a.P + ((int64_t)bh * S + q0 + 8 * wave) * S;
    for (int c = lane; c < S; c += 64) {
      float p[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) p[r] = f[r] > 0.0f ? rows[r * LD + c] * f[r] : 0.0f;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        rows[r * LD + c] = p[r];
        if (r < live) Pw[(int64_t)r * S + c] = p[r];
      }
    }
  } else {
    float dot[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) dot[r] = lane < S ? p0[r] * rows[r * LD + lane] : 0.0f;
    for (int c = lane + 64; c < S; c += 64)
#pragma unroll
      for (int r = 0; r < 8; ++r)
        if (r < live) dot[r] += rows[r * LD + c] * Pg[(int64_t)r * S + c];
#pragma unroll
    for (int r = 0; r < 8; ++r) dot[r] = wave_sum(dot[r]);
    float* dSg = a.dS + ((int64_t)bh * S + q0 + 8 * wave) * S;
    for (int c = lane; c < 16 * ng; c += 64)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        float d = 0.0f;
        if (c < S && r < live) {
          d = a.scale * (c < 64 ? p0[r] : Pg[(int64_t)r * S + c]) * (rows[r * LD + c] - dot[r]);
          dSg[(int64_t)r * S + c] = d;
        }
        rows[r * LD + c] = d;
      }
  }
  __syncthreads();

  // C = P V, or dQ = dS K: 16 columns, both halves of the rows.
  f32x4_t acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  auto group = [&](int g, const float (&f)[4]) {
    const float* p = sc + rr * LD + 16 * g + 4 * kq;
    const f32x4_t a0 = *(const f32x4_t*)p, a1 = *(const f32x4_t*)(p + 16 * LD);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[0] = mfma4(a0[i], f[i], acc[0]);
      acc[1] = mfma4(a1[i], f[i], acc[1]);
    }
  };
#pragma unroll
  for (int g = 0; g < PRE; ++g)
    if (g < ng) group(g, vb[g]);
#pragma unroll 4
  for (int g = PRE; g < ng; ++g) {
    float f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = B2[min(16 * g + 4 * kq + i, S - 1) * ld];
    group(g, f);
  }
  float* out = a.out + (int64_t)b * S * a.ldo + j * HD + 16 * wave + rr;
  float sum = 0.0f;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = q0 + 16 * t + 4 * kq + r;
      if (q < S) {
        out[(int64_t)q * a.ldo] = acc[t][r];
        sum += acc[t][r];
      }
    }
  if constexpr (BWD) {  // column sums of the 32 rows
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (kq == 0) a.colpart[((int64_t)b * nq + qb) * ld + j * HD + 16 * wave + rr] = sum;
  }
}

template <bool BWD>
hipError_t launch(const AttnF32Args& a, int B, hipStream_t st) {
  if (B <= 0 || a.S <= 0) return hipSuccess;
  const int64_t n = (int64_t)((a.S + 31) / 32) * B * a.H;
  if (a.S > ATTN_F32_MAX_S || n >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)n), blk(256);
  if (a.S <= 64) hipLaunchKernelGGL((attn_f32_kernel<BWD, 72>), grid, blk, 0, st, a);
  else if (a.S <= 128) hipLaunchKernelGGL((attn_f32_kernel<BWD, 136>), grid, blk, 0, st, a);
  else if (a.S <= 256) hipLaunchKernelGGL((attn_f32_kernel<BWD, 264>), grid, blk, 0, st, a);
  else hipLaunchKernelGGL((attn_f32_kernel<BWD, 520>), grid, blk, 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t attn_f32_forward(const AttnF32Args& a, int B, hipStream_t st) {
  return launch<false>(a, B, st);
}
hipError_t attn_f32_backward_rows(const AttnF32Args& a, int B, hipStream_t st) {
  return launch<true>(a, B, st);
}
