// HBM-bound row kernels of the encoder layer: residual + bias + LayerNorm
// (forward and backward), the column partial sums of the gamma / beta / bias
// gradients (reduced by the units of tail.h), and the masked row softmax of long
// fp32 sequences (forward and backward).
// One wavefront owns one row; reductions across the row are wavefront
// shuffles.  No MFMA here.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "tail.h"

namespace {

constexpr float LN_EPS = 1e-12f;

// 8 consecutive elements <-> 8 floats (16-byte bf16 / 32-byte fp32 accesses).
__device__ __forceinline__ void load8(const bf16_t* p, float v[8]) {
  u32x4_t r = *(const u32x4_t*)p;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(r[i] << 16);
    v[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void load8(const float* p, float v[8]) {
  f32x4_t a = *(const f32x4_t*)p, b = *(const f32x4_t*)(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = a[i];
    v[4 + i] = b[i];
  }
}
__device__ __forceinline__ void store8(bf16_t* p, const float v[8]) {
  u32x4_t r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
  *(u32x4_t*)p = r;
}
__device__ __forceinline__ void store8(float* p, const float v[8]) {
  f32x4_t a, b;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = v[i];
    b[i] = v[4 + i];
  }
  *(f32x4_t*)p = a;
  *(f32x4_t*)(p + 4) = b;
}
// Round to the storage type and back (what a store followed by a load gives).
__device__ __forceinline__ float as_stored(float v, const bf16_t*) { return bf2f(f2bf(v)); }
__device__ __forceinline__ float as_stored(float v, const float*) { return v; }

// One wavefront per row.  Lane `lane` owns the 8-column chunks
// c = lane + 64 i (i < NC, c < h / 8).  The residual is resid, plus
// resid_lo when not null (a value carried as its bf16 rounding and the
// rounding residual); ylo, when not null, receives y's rounding residual
// y - bf16(y) in bf16, so that y + ylo carries y to about 16 significant
// bits.  a is the sum of NP partials (rows * h apart), all loads issued
// before the sum.
template <typename T, typename TA, int NC, int NP>
__global__ __launch_bounds__(256) void add_ln_fwd_kernel(const TA* __restrict__ a,
                                                         const float* __restrict__ bias,
                                                         const T* __restrict__ resid,
                                                         const T* __restrict__ resid_lo,
                                                         const float* __restrict__ gamma,
                                                         const float* __restrict__ beta,
                                                         T* __restrict__ y, T* __restrict__ ylo,
                                                         T* __restrict__ xhat,
                                                         float* __restrict__ rstd, int rows, int h) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int nchunk = h >> 3;
  const int64_t base = (int64_t)row * h;
  float z[NC][8];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < nchunk) {
      float av[8], rv[8], bv[8], lv[8];
      float ap[NP][8];
#pragma unroll
      for (int q = 0; q < NP; ++q) load8(a + q * (int64_t)rows * h + base + 8 * c, ap[q]);
      load8(resid + base + 8 * c, rv);
      load8(bias + 8 * c, bv);
      if (resid_lo) {
        load8(resid_lo + base + 8 * c, lv);
#pragma unroll
        for (int k = 0; k < 8; ++k) rv[k] += lv[k];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        av[k] = ap[0][k];
#pragma unroll
        for (int q = 1; q < NP; ++q) av[k] += ap[q][k];
        z[i][k] = av[k] + bv[k] + rv[k];
        s += z[i][k];
      }
    }
  }
  const float mean = wave_sum(s) / (float)h;
  float s2 = 0.0f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    if (lane + 64 * i < nchunk) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        float d = z[i][k] - mean;
        s2 += d * d;
      }
    }
  }
  const float var = wave_sum(s2) / (float)h;
  const float r = 1.0f / sqrtf(var + LN_EPS);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < nchunk) {
      float gv[8], btv[8], xh[8], yv[8];
      load8(gamma + 8 * c, gv);
      load8(beta + 8 * c, btv);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        xh[k] = (z[i][k] - mean) * r;
        yv[k] = gv[k] * xh[k] + btv[k];
      }
      store8(xhat + base + 8 * c, xh);
      store8(y + base + 8 * c, yv);
      if (ylo) {
#pragma unroll
        for (int k = 0; k < 8; ++k) yv[k] -= as_stored(yv[k], y);
        store8(ylo + base + 8 * c, yv);
      }
    }
  }
  if (lane == 0) rstd[row] = r;
}

// LayerNorm backward.  A block of 4 wavefronts handles `rpb` consecutive
// rows (one row per wavefront at a time); per-column partial sums of
// dy*xhat, dy and dz are kept per lane, combined across the 4 wavefronts in
// LDS in a fixed order and written as one partial row per block.
template <typename T, int NC>
__global__ __launch_bounds__(256) void ln_bwd_kernel(const T* __restrict__ dy,
                                                     const T* __restrict__ xhat,
                                                     const float* __restrict__ rstd,
                                                     const float* __restrict__ gamma,
                                                     T* __restrict__ dz, float* __restrict__ part,
                                                     int rows, int h, int rpb) {
  extern __shared__ float red[];  // [4 wavefronts][3][h]
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int nchunk = h >> 3;
  float pg[NC][8], pb[NC][8], pz[NC][8], gm[NC][8];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
#pragma unroll
    for (int k = 0; k < 8; ++k) pg[i][k] = pb[i][k] = pz[i][k] = gm[i][k] = 0.0f;
    if (c < nchunk) load8(gamma + 8 * c, gm[i]);
  }
  const int r0 = blockIdx.x * rpb;
  const int r1 = min(rows, r0 + rpb);
  const float inv_h = 1.0f / (float)h;
  // Two rows per wavefront at a time (rows row and row + 4), so that the
  // loads of both are in flight together.
  for (int row0 = r0 + wave; row0 < r1; row0 += 8) {
    float dv[2][NC][8], xv[2][NC][8];
    float sg[2] = {0.0f, 0.0f}, sgx[2] = {0.0f, 0.0f};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = row0 + 4 * u;
      const int64_t base = (int64_t)row * h;
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int c = lane + 64 * i;
        if (c < nchunk && row < r1) {
          load8(dy + base + 8 * c, dv[u][i]);
          load8(xhat + base + 8 * c, xv[u][i]);
        } else {
#pragma unroll
          for (int k = 0; k < 8; ++k) dv[u][i][k] = xv[u][i][k] = 0.0f;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float g = dv[u][i][k] * gm[i][k];
          sg[u] += g;
          sgx[u] += g * xv[u][i][k];
          pg[i][k] += dv[u][i][k] * xv[u][i][k];
          pb[i][k] += dv[u][i][k];
        }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      sg[u] = wave_sum(sg[u]) * inv_h;
      sgx[u] = wave_sum(sgx[u]) * inv_h;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = row0 + 4 * u;
      if (row >= r1) continue;
      const int64_t base = (int64_t)row * h;
      const float rs = rstd[row];
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int c = lane + 64 * i;
        if (c < nchunk) {
          float d[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            d[k] = rs * (dv[u][i][k] * gm[i][k] - sg[u] - xv[u][i][k] * sgx[u]);
            // The column sum uses the value as stored, so that the bias
            // gradient of the preceding linear layer matches the gradient
            // that flows on.
            pz[i][k] += as_stored(d[k], dz);
          }
          store8(dz + base + 8 * c, d);
        }
      }
    }
  }
  // Each wavefront parks its partials in LDS; after one barrier every
  // thread sums the 4 wavefronts' values of its columns in a fixed order.
  float* mine = red + wave * 3 * h;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < nchunk) {
      const int col = 8 * c;
      *(f32x4_t*)(mine + col) = f32x4_t{pg[i][0], pg[i][1], pg[i][2], pg[i][3]};
      *(f32x4_t*)(mine + col + 4) = f32x4_t{pg[i][4], pg[i][5], pg[i][6], pg[i][7]};
      *(f32x4_t*)(mine + h + col) = f32x4_t{pb[i][0], pb[i][1], pb[i][2], pb[i][3]};
      *(f32x4_t*)(mine + h + col + 4) = f32x4_t{pb[i][4], pb[i][5], pb[i][6], pb[i][7]};
      *(f32x4_t*)(mine + 2 * h + col) = f32x4_t{pz[i][0], pz[i][1], pz[i][2], pz[i][3]};
      *(f32x4_t*)(mine + 2 * h + col + 4) = f32x4_t{pz[i][4], pz[i][5], pz[i][6], pz[i][7]};
    }
  }
  __syncthreads();
  float* P = part + (int64_t)blockIdx.x * 3 * h;
  for (int e = threadIdx.x; e < 3 * h; e += 256)
    P[e] = ((red[e] + red[3 * h + e]) + red[6 * h + e]) + red[9 * h + e];
}

// bf16 LayerNorm backward with the rows kept as packed bf16 (unpacked where
// used) and gamma in registers: the same arithmetic and partial rows as
// ln_bwd_kernel, twice the loads in flight.  Register budget: two
// work-groups per CU (16384 rows of 32 per work-group are 512 work-groups,
// two per CU), which keeps every per-column partial in registers.
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf_at(const u32x4_t& r, int k) {
  return (k & 1) ? bf_hi(r[k >> 1]) : bf_lo(r[k >> 1]);
}

// Product of a data-gradient GEMM at 8 elements: NP fp32 partials, n apart.
template <int NP>
__device__ __forceinline__ void load_parts(const float* pf, int64_t n, float v[8]) {
  float p[NP][8];
#pragma unroll
  for (int q = 0; q < NP; ++q) load8(pf + q * n, p[q]);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    v[k] = p[0][k];
#pragma unroll
    for (int q = 1; q < NP; ++q) v[k] += p[q][k];
  }
}

// The incoming gradient is one bf16 tensor (NP = -1), or the backward
// residual stream of a bf16 stage, never itself rounded to bf16: the fp32 sum
// (hi + lo) + product of the residual branch, carried as its bf16 rounding
// plus the rounding residual (about 16 significant bits), and the
// data-gradient GEMM's product in bf16 (NP = 0) or as NP fp32 partials.
// dz goes out in bf16 (the operand of the following GEMMs) and, when dzlo
// is not null, its rounding residual dz - bf16(dz) in bf16 as well (the
// residual branch of the next addition).
template <int NC, int NP>
__global__ __launch_bounds__(256, (NC <= 2 ? 2 : 1)) void ln_bwd_bf16_kernel(
    GradIn in, const bf16_t* __restrict__ xhat, const float* __restrict__ rstd,
    const float* __restrict__ gamma, bf16_t* __restrict__ dz, bf16_t* __restrict__ dzlo,
    float* __restrict__ part, int rows, int h, int rpb) {
  extern __shared__ float red[];  // [4 wavefronts][3][h]
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int nchunk = h >> 3;
  // gamma of the lane's columns, in registers for all rows
  float pg[NC][8], pb[NC][8], pz[NC][8], gm[NC][8];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
#pragma unroll
    for (int k = 0; k < 8; ++k) pg[i][k] = pb[i][k] = pz[i][k] = gm[i][k] = 0.0f;
    if (c < nchunk) load8(gamma + 8 * c, gm[i]);
  }
  const int r0 = blockIdx.x * rpb;
  const int r1 = min(rows, r0 + rpb);
  const float inv_h = 1.0f / (float)h;
  for (int row0 = r0 + wave; row0 < r1; row0 += 8) {
    // packed bf16: the gradient or the product, with hi and lo beside it
    u32x4_t dr[2][NC], xr[2][NC], hr[2][NC], lr[2][NC];
    float pr[NP > 0 ? 2 : 1][NC][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = row0 + 4 * u;
      const int64_t base = (int64_t)row * h;
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int c = lane + 64 * i;
        if (c < nchunk && row < r1) {
          if constexpr (NP >= 0) {
            hr[u][i] = *(const u32x4_t*)(in.hi + base + 8 * c);
            lr[u][i] = *(const u32x4_t*)(in.lo + base + 8 * c);
          }
          if constexpr (NP > 0) load_parts<NP>(in.pf + base + 8 * c, (int64_t)rows * h, pr[u][i]);
          else dr[u][i] = *(const u32x4_t*)((NP == 0 ? in.b : in.bf) + base + 8 * c);
          xr[u][i] = *(const u32x4_t*)(xhat + base + 8 * c);
        } else {
          hr[u][i] = lr[u][i] = dr[u][i] = u32x4_t{0, 0, 0, 0};
          xr[u][i] = u32x4_t{0, 0, 0, 0};
          if constexpr (NP > 0) {
#pragma unroll
            for (int k = 0; k < 8; ++k) pr[u][i][k] = 0.0f;
          }
        }
      }
    }
    // the incoming gradient at (u, i, k)
    auto dyv = [&](int u, int i, int k) -> float {
      if constexpr (NP > 0) return (bf_at(hr[u][i], k) + bf_at(lr[u][i], k)) + pr[u][i][k];
      else if constexpr (NP == 0) return (bf_at(hr[u][i], k) + bf_at(lr[u][i], k)) + bf_at(dr[u][i], k);
      else return bf_at(dr[u][i], k);
    };
    float sg[2] = {0.0f, 0.0f}, sgx[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < NC; ++i) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float d = dyv(u, i, k), x = bf_at(xr[u][i], k);
          const float g = d * gm[i][k];
          sg[u] += g;
          sgx[u] += g * x;
          pg[i][k] += d * x;
          pb[i][k] += d;
        }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      sg[u] = wave_sum(sg[u]) * inv_h;
      sgx[u] = wave_sum(sgx[u]) * inv_h;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = row0 + 4 * u;
      if (row >= r1) continue;
      const int64_t base = (int64_t)row * h;
      const float rs = rstd[row];
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int c = lane + 64 * i;
        if (c < nchunk) {
          float dd[8];
#pragma unroll
          for (int k = 0; k < 8; ++k)
            dd[k] = rs * (dyv(u, i, k) * gm[i][k] - sg[u] - bf_at(xr[u][i], k) * sgx[u]);
          u32x4_t o;
#pragma unroll
          for (int k2 = 0; k2 < 4; ++k2) {
            o[k2] = pack_bf16x2(dd[2 * k2], dd[2 * k2 + 1]);
            // The column sum uses the value as stored, so that the bias
            // gradient of the preceding linear layer matches the gradient
            // its weight gradient is formed from.
            pz[i][2 * k2] += bf_lo(o[k2]);
            pz[i][2 * k2 + 1] += bf_hi(o[k2]);
          }
          *(u32x4_t*)(dz + base + 8 * c) = o;
          if (dzlo) {
            u32x4_t lo;
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2)
              lo[k2] = pack_bf16x2(dd[2 * k2] - bf_lo(o[k2]), dd[2 * k2 + 1] - bf_hi(o[k2]));
            *(u32x4_t*)(dzlo + base + 8 * c) = lo;
          }
        }
      }
    }
  }
  float* mine = red + wave * 3 * h;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < nchunk) {
      const int col = 8 * c;
      *(f32x4_t*)(mine + col) = f32x4_t{pg[i][0], pg[i][1], pg[i][2], pg[i][3]};
      *(f32x4_t*)(mine + col + 4) = f32x4_t{pg[i][4], pg[i][5], pg[i][6], pg[i][7]};
      *(f32x4_t*)(mine + h + col) = f32x4_t{pb[i][0], pb[i][1], pb[i][2], pb[i][3]};
      *(f32x4_t*)(mine + h + col + 4) = f32x4_t{pb[i][4], pb[i][5], pb[i][6], pb[i][7]};
      *(f32x4_t*)(mine + 2 * h + col) = f32x4_t{pz[i][0], pz[i][1], pz[i][2], pz[i][3]};
      *(f32x4_t*)(mine + 2 * h + col + 4) = f32x4_t{pz[i][4], pz[i][5], pz[i][6], pz[i][7]};
    }
  }
  __syncthreads();
  float* P = part + (int64_t)blockIdx.x * 3 * h;
  for (int e = threadIdx.x; e < 3 * h; e += 256)
    P[e] = ((red[e] + red[3 * h + e]) + red[6 * h + e]) + red[9 * h + e];
}

// The gradient `in` at 8 elements per thread (n % 8 == 0).
template <int NP>
__global__ __launch_bounds__(256) void grad_kernel(GradIn in, float* __restrict__ out, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  float v[8];
  if constexpr (NP < 0) {
    load8(in.bf + i, v);
  } else {
    float l[8], b[8];
    load8(in.hi + i, v);
    load8(in.lo + i, l);
    if constexpr (NP > 0) load_parts<NP>(in.pf + i, n, b);
    else load8(in.b + i, b);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = (v[k] + l[k]) + b[k];
  }
  store8(out + i, v);
}

// Four units per work-group.
__global__ __launch_bounds__(256) void stage_prep_kernel(PrepArgs p) {
  prep_unit(p, blockIdx.x * 4 + (threadIdx.x >> 6), threadIdx.x & 63);
}

template <typename T>
__global__ __launch_bounds__(256) void col_partial_kernel(const T* __restrict__ x, int rows, int n,
                                                          int rows_per_blk,
                                                          float* __restrict__ part) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  const int blk = blockIdx.y;
  if (c >= n) return;
  const int r0 = blk * rows_per_blk, r1 = min(rows, r0 + rows_per_blk);
  float s = 0.0f;
  for (int r = r0; r < r1; ++r) s += ld_f(x + (int64_t)r * n + c);
  part[(int64_t)blk * n + c] = s;
}

// P = softmax over keys of scale * scores, masked keys -> 0, empty rows -> 0.
template <typename T>
__global__ __launch_bounds__(256) void softmax_fwd_kernel(const float* __restrict__ scores,
                                                          const uint8_t* __restrict__ mask,
                                                          T* __restrict__ P, int BH, int H, int S,
                                                          int ld, float scale) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= (int64_t)BH * S) return;
  const int b = (int)(row / S) / H;
  const float* srow = scores + row * ld;
  const uint8_t* mrow = mask + (int64_t)b * S;
  T* prow = P + row * ld;
  float mx = -INFINITY;
  for (int c = lane; c < S; c += 64)
    if (mrow[c]) mx = fmaxf(mx, scale * srow[c]);
  mx = wave_max(mx);
  float sum = 0.0f;
  if (mx != -INFINITY) {
    for (int c = lane; c < S; c += 64)
      if (mrow[c]) sum += expf(scale * srow[c] - mx);
  }
  sum = wave_sum(sum);
  const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
  for (int c = lane; c < ld; c += 64) {
    float p = 0.0f;
    if (c < S && mrow[c] && sum > 0.0f) p = expf(scale * srow[c] - mx) * inv;
    st_f(prow + c, p);
  }
}

// dS = scale * P * (dP - sum_j dP_j P_j).
template <typename T>
__global__ __launch_bounds__(256) void softmax_bwd_kernel(const float* __restrict__ dP,
                                                          const T* __restrict__ P,
                                                          T* __restrict__ dS, int BH, int S,
                                                          int ld, float scale) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= (int64_t)BH * S) return;
  const float* drow = dP + row * ld;
  const T* prow = P + row * ld;
  T* orow = dS + row * ld;
  float dot = 0.0f;
  for (int c = lane; c < S; c += 64) dot += drow[c] * ld_f(prow + c);
  dot = wave_sum(dot);
  for (int c = lane; c < ld; c += 64) {
    float v = 0.0f;
    if (c < S) v = scale * ld_f(prow + c) * (drow[c] - dot);
    st_f(orow + c, v);
  }
}

}  // namespace

template <typename T, typename TA>
hipError_t add_ln_fwd(const TA* a, int np, const float* bias, const T* resid, const T* resid_lo,
                      const float* gamma, const float* beta, T* y, T* ylo, T* xhat, float* rstd,
                      int rows, int h, hipStream_t st) {
  if (h % 64 != 0 || h > 2048) return hipErrorInvalidValue;
  if (rows <= 0) return hipSuccess;
  const int nc = (h / 8 + 63) / 64;
  dim3 grid((rows + 3) / 4), blk(256);
#define LAUNCH_LN(NCV, NPV)                                                                   \
  hipLaunchKernelGGL((add_ln_fwd_kernel<T, TA, NCV, NPV>), grid, blk, 0, st, a, bias, resid,  \
                     resid_lo, gamma, beta, y, ylo, xhat, rstd, rows, h)
#define LAUNCH_LN_NC(NPV)               \
  switch (nc) {                         \
    case 1: LAUNCH_LN(1, NPV); break;   \
    case 2: LAUNCH_LN(2, NPV); break;   \
    case 3: LAUNCH_LN(3, NPV); break;   \
    default: LAUNCH_LN(4, NPV); break;  \
  }
  if (np == 1) {
    LAUNCH_LN_NC(1)
  } else if constexpr (std::is_same<T, bf16_t>::value) {
    if (np == 2) LAUNCH_LN_NC(2)
    else if (np == 4) LAUNCH_LN_NC(4)
    else if (np == 6) LAUNCH_LN_NC(6)
    else return hipErrorInvalidValue;
  } else {
    return hipErrorInvalidValue;
  }
#undef LAUNCH_LN_NC
#undef LAUNCH_LN
  return hipGetLastError();
}

// 32 rows per work-group (two row pairs per wavefront and eight loads of them
// in flight hide HBM latency) above 4096 rows, then half as many at each power of
// two, so that 1024, 2048 and 4096 rows are 256 work-groups, one per CU (2048 rows
// of 768 took 15.5 us in 64 work-groups), and between them there are 129 to 256.
// Not more: rows wider than 1024 leave room for one work-group per CU, and with
// the lines at 2040, 4080 and 8160 rows (129 to 510 work-groups) width 2048 went
// from 17.7 to 22.7 us at 1536 rows, 23.4 to 28.9 at 2064 and 38.8 to 43.7 at
// 5040.  Widths up to 1024 have room for two and are faster that way (768: 20.9
// -> 17.9 us at 5040 rows, 12.8 -> 11.4 at 2064, unchanged up to 2040); a line per
// width is not drawn.
int ln_bwd_rpb(int rows) { return rows > 4096 ? 32 : rows > 2048 ? 16 : rows > 1024 ? 8 : 4; }
int ln_bwd_blocks(int rows) { return (rows + ln_bwd_rpb(rows) - 1) / ln_bwd_rpb(rows); }
int ln_bwd_blocks_max(int rows) {
  // 1024, 2048 and 4096 rows make 256 work-groups each
  return rows <= 1024 ? ln_bwd_blocks(rows) : std::max(256, ln_bwd_blocks(rows));
}

hipError_t ln_bwd_bf16(const GradIn& in, const bf16_t* xhat, const float* rstd, const float* gamma,
                       bf16_t* dz, bf16_t* dzlo, float* part, int rows, int h, hipStream_t st) {
  if (h % 64 != 0 || h > 2048) return hipErrorInvalidValue;
  if (!in.bf && (!in.hi || !in.lo || (!in.b && !in.pf))) return hipErrorInvalidValue;
  if (rows <= 0) return hipSuccess;
  const int nc = (h / 8 + 63) / 64;
  dim3 grid(ln_bwd_blocks(rows)), blk(256);
  size_t sh = (size_t)4 * 3 * h * sizeof(float);
  const int rpb = ln_bwd_rpb(rows);
#define LAUNCH_LNB(NCV, NPV)                                                                   \
  hipLaunchKernelGGL((ln_bwd_bf16_kernel<NCV, NPV>), grid, blk, sh, st, in, xhat, rstd, gamma, \
                     dz, dzlo, part, rows, h, rpb)
#define LAUNCH_LNB_NC(NPV)               \
  switch (nc) {                          \
    case 1: LAUNCH_LNB(1, NPV); break;   \
    case 2: LAUNCH_LNB(2, NPV); break;   \
    case 3: LAUNCH_LNB(3, NPV); break;   \
    default: LAUNCH_LNB(4, NPV); break;  \
  }
  if (in.bf) LAUNCH_LNB_NC(-1)
  else if (in.b) LAUNCH_LNB_NC(0)
  else if (in.np == 2) LAUNCH_LNB_NC(2)
  else if (in.np == 4) LAUNCH_LNB_NC(4)
  else if (in.np == 6) LAUNCH_LNB_NC(6)
  else return hipErrorInvalidValue;
#undef LAUNCH_LNB_NC
#undef LAUNCH_LNB
  return hipGetLastError();
}

hipError_t grad_f32(const GradIn& in, float* out, int64_t n, hipStream_t st) {
  if (n % 8 != 0) return hipErrorInvalidValue;
  if (n == 0) return hipSuccess;
  const dim3 grid((unsigned)((n / 8 + 255) / 256)), blk(256);
  if (in.bf) hipLaunchKernelGGL(grad_kernel<-1>, grid, blk, 0, st, in, out, n);
  else if (in.b) hipLaunchKernelGGL(grad_kernel<0>, grid, blk, 0, st, in, out, n);
  else if (in.np == 2) hipLaunchKernelGGL(grad_kernel<2>, grid, blk, 0, st, in, out, n);
  else if (in.np == 4) hipLaunchKernelGGL(grad_kernel<4>, grid, blk, 0, st, in, out, n);
  else if (in.np == 6) hipLaunchKernelGGL(grad_kernel<6>, grid, blk, 0, st, in, out, n);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t stage_prep(const PrepArgs& p, hipStream_t st) {
  const int64_t blocks = (prep_units(p) + 3) / 4;
  if (p.nx % 16 != 0 || blocks >= ((int64_t)1 << 29)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(stage_prep_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p);
  return hipGetLastError();
}

hipError_t ln_bwd_f32(const float* dy, const float* xhat, const float* rstd, const float* gamma,
                      float* dz, float* part, int rows, int h, hipStream_t st) {
  if (h % 64 != 0 || h > 2048) return hipErrorInvalidValue;
  if (rows <= 0) return hipSuccess;
  const int nc = (h / 8 + 63) / 64;
  dim3 grid(ln_bwd_blocks(rows)), blk(256);
  size_t sh = (size_t)4 * 3 * h * sizeof(float);
  const int rpb = ln_bwd_rpb(rows);
#define LAUNCH_LNB(NCV)                                                                        \
  hipLaunchKernelGGL((ln_bwd_kernel<float, NCV>), grid, blk, sh, st, dy, xhat, rstd, gamma, dz, \
                     part, rows, h, rpb)
  switch (nc) {
    case 1: LAUNCH_LNB(1); break;
    case 2: LAUNCH_LNB(2); break;
    case 3: LAUNCH_LNB(3); break;
    default: LAUNCH_LNB(4); break;
  }
#undef LAUNCH_LNB
  return hipGetLastError();
}

template <typename T>
hipError_t col_partial(const T* x, int rows, int n, float* part, int nblk, hipStream_t st) {
  int rpb = (rows + nblk - 1) / nblk;
  if (rpb < 1) rpb = 1;
  hipLaunchKernelGGL(col_partial_kernel<T>, dim3((n + 255) / 256, nblk), dim3(256), 0, st, x, rows,
                     n, rpb, part);
  return hipGetLastError();
}

template <typename T>
hipError_t softmax_fwd(const float* scores, const uint8_t* mask, T* P, int BH, int H, int S,
                       int ld, float scale, hipStream_t st) {
  int64_t rows = (int64_t)BH * S;
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(softmax_fwd_kernel<T>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st,
                     scores, mask, P, BH, H, S, ld, scale);
  return hipGetLastError();
}

template <typename T>
hipError_t softmax_bwd(const float* dP, const T* P, T* dS, int BH, int S, int ld, float scale,
                       hipStream_t st) {
  int64_t rows = (int64_t)BH * S;
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(softmax_bwd_kernel<T>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, dP,
                     P, dS, BH, S, ld, scale);
  return hipGetLastError();
}

template hipError_t add_ln_fwd<float, float>(const float*, int, const float*, const float*, const float*,
                                             const float*, const float*, float*, float*, float*,
                                             float*, int, int, hipStream_t);
template hipError_t add_ln_fwd<bf16_t, float>(const float*, int, const float*, const bf16_t*,
                                              const bf16_t*, const float*, const float*, bf16_t*,
                                              bf16_t*, bf16_t*, float*, int, int, hipStream_t);
template hipError_t col_partial<float>(const float*, int, int, float*, int, hipStream_t);
template hipError_t softmax_fwd<float>(const float*, const uint8_t*, float*, int, int, int, int,
                                       float, hipStream_t);
template hipError_t softmax_bwd<float>(const float*, const float*, float*, int, int, int, float,
                                       hipStream_t);
