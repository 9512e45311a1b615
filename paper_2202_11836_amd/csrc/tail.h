// Small work around a stage's GEMMs, as units of one wavefront that the GEMM
// kernels take on in extra work-groups: the reductions and conversions at the
// end of a layer's backward, and the copies at the start of a forward pass.
//
// On their own they are launches of 3 to 5 us whose work is 1 to 2 us.  Behind
// the tiles of a GEMM launch they run on CUs that its last round leaves idle.
// The units use no LDS, but their work-groups are the GEMM kernel's and hold its
// 64 to 144 KB: beside one of the larger tiles they wait for a free CU.
#pragma once
#include <cstddef>

#include "kernels.h"

namespace {

constexpr int TAIL_GRAD_UNIT = 2048;  // elements of the gradient per wavefront

// 16 columns of a column reduction: out[c] = the sum over partial rows b of
// part[(b * nvec + v) * n + c].  4 lanes x 4 columns per row; 64 stripes of
// rows (a lane sums stripes lane / 4 + 16 j), combined by a fixed-order tree.
// D rows of loads in flight.
template <int D>
__device__ __forceinline__ void colred_unit(const float* __restrict__ part, int nblk, int nvec,
                                            int n, int v, int bx, float* out, int lane) {
  const int c = bx * 16 + 4 * (lane & 3);
  if (!out) return;  // (uniform)
  f32x4_t s[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) s[j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  if (c < n) {
    const float* p = part + (int64_t)v * n + c;
    const int64_t row = (int64_t)nvec * n;
    int b = lane >> 2;
    for (; b + 16 * (D - 1) < nblk; b += 16 * D) {
      f32x4_t x[D];
#pragma unroll
      for (int j = 0; j < D; ++j) x[j] = *(const f32x4_t*)(p + (b + 16 * j) * row);
#pragma unroll
      for (int j = 0; j < D; ++j) s[j & 3] += x[j];
    }
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
      if (b + 16 * j < nblk) s[j & 3] += *(const f32x4_t*)(p + (b + 16 * j) * row);
  }
  f32x4_t t = (s[0] + s[2]) + (s[1] + s[3]);
#pragma unroll
  for (int o = 32; o >= 4; o >>= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] += __shfl_xor(t[e], o, 64);
  if (lane < 4 && c < n) *(f32x4_t*)(out + c) = t;
}

__device__ __forceinline__ void unpack8(u32x4_t r, float v[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(r[i] << 16);
    v[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u);
  }
}

// TAIL_GRAD_UNIT elements from i0 of the gradient (hi + lo) + product, rounded
// to bf16; D / 4 steps of loads in flight.
template <int D>
__device__ __forceinline__ void grad_unit(const GradIn& in, bf16_t* out, int64_t n, int64_t i0,
                                          int lane) {
#pragma unroll(D / 4)
  for (int j = 0; j < TAIL_GRAD_UNIT / 512; ++j) {
    const int64_t i = i0 + 512 * j + 8 * lane;
    if (i >= n) continue;
    float h[8], l[8], b[8];
    unpack8(*(const u32x4_t*)(in.hi + i), h);
    unpack8(*(const u32x4_t*)(in.lo + i), l);
    if (in.pf) {
      f32x4_t x = *(const f32x4_t*)(in.pf + i), y = *(const f32x4_t*)(in.pf + i + 4);
      for (int q = 1; q < in.np; ++q) {
        x += *(const f32x4_t*)(in.pf + q * n + i);
        y += *(const f32x4_t*)(in.pf + q * n + i + 4);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = x[e], b[4 + e] = y[e];
    } else {
      unpack8(*(const u32x4_t*)(in.b + i), b);
    }
    u32x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = pack_bf16x2((h[2 * e] + l[2 * e]) + b[2 * e], (h[2 * e + 1] + l[2 * e + 1]) + b[2 * e + 1]);
    *(u32x4_t*)(out + i) = o;
  }
}

// Unit u of t (nothing past the last).  t is read in place, in the
// kernel-argument segment (a by-value argument indexed by a run-time job
// number would be copied to scratch memory first).  D = 8; 4 in kernels that
// live on many resident wavefronts (64 registers).
typedef const __attribute__((address_space(4))) TailJobs ktail_t;
__device__ __forceinline__ ktail_t* tail_arg(int offset) {
  return (ktail_t*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                    offset);
}
template <int D>
__device__ __forceinline__ void tail_unit(ktail_t* t, int u, int lane) {
  u = __builtin_amdgcn_readfirstlane(u);
  if (u >= t->units) return;
  const int cols = t->unit0[COLJOB_MAX];
  if (u >= cols) {
    const GradIn in = {nullptr, t->gin.hi, t->gin.lo, t->gin.b, t->gin.pf, t->gin.np};
    grad_unit<D>(in, t->gout, t->gn, (int64_t)(u - cols) * TAIL_GRAD_UNIT, lane);
    return;
  }
  int j = 0;
#pragma unroll
  for (int k = 1; k < COLJOB_MAX; ++k)
    if (k < t->ncol && u >= t->unit0[k]) j = k;
  const auto* c = &t->col[j];
  const int n = c->n, nx = (n + 15) / 16, r = u - t->unit0[j], v = r / nx;
  colred_unit<D>(c->part, c->nblk, c->nvec, n, v, r - v * nx, c->out[v], lane);
}

// Unit u of a forward pass's start: one sequence's mask and key extent, or
// PREP_CHUNKS 16-byte chunks of x.  Eight loads in flight per lane: as a launch of
// its own the copy takes 17.6 us for 16384 x 1024 bf16 and 15.2 for 16384 x 768,
// against 20.5 and 16.6 with four (events around the launch, 1% apart from run to
// run); 8192 x 1024 takes 11.3 either way.
constexpr int PREP_CHUNKS = 512;
__device__ __forceinline__ void prep_unit(const PrepArgs& p, int u, int lane) {
  if (u < p.B) {
    const int64_t b0 = (int64_t)u * p.S;
    int last = 0;
    for (int s0 = 0; s0 < p.S; s0 += 512) {
      int v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = 1;
      if (p.key_mask) {  // (positions clamped: no load waits for another)
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = p.key_mask[b0 + min(s0 + 64 * k + lane, p.S - 1)];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int s = s0 + 64 * k + lane;
        if (s < p.S) p.mask[b0 + s] = (uint8_t)v[k];
        if (s < p.S && v[k]) last = s + 1;
      }
    }
    if (!p.kext) return;
    for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
    if (lane == 0) p.kext[u] = last;
    return;
  }
  const int64_t n16 = p.nx / 16, i0 = (int64_t)(u - p.B) * PREP_CHUNKS + lane;
  const u32x4_t* x = (const u32x4_t*)p.x;
  u32x4_t v[PREP_CHUNKS / 64];
#pragma unroll
  for (int k = 0; k < PREP_CHUNKS / 64; ++k)
    if (i0 + 64 * k < n16) v[k] = x[i0 + 64 * k];
#pragma unroll
  for (int k = 0; k < PREP_CHUNKS / 64; ++k)
    if (i0 + 64 * k < n16) ((u32x4_t*)p.X)[i0 + 64 * k] = v[k];
}

}  // namespace

inline int64_t prep_units(const PrepArgs& p) {
  return p.B + (p.nx / 16 + PREP_CHUNKS - 1) / PREP_CHUNKS;
}

// Checks t's jobs and numbers their units; false for invalid ones.
inline bool tail_prepare(TailJobs& t) {
  if (t.ncol < 0 || t.ncol > COLJOB_MAX) return false;
  int64_t units = 0;
  for (int j = 0; j < t.ncol; ++j) {
    const ColJob& c = t.col[j];
    if (c.nvec < 1 || c.nvec > 4 || c.n < 0 || c.n % 4 != 0 || c.nblk < 0 || !c.part) return false;
    t.unit0[j] = (int)units;
    units += (int64_t)((c.n + 15) / 16) * c.nvec;
    if (units >= ((int64_t)1 << 30)) return false;
  }
  for (int j = t.ncol; j <= COLJOB_MAX; ++j) t.unit0[j] = (int)units;
  if (t.gout) {
    const GradIn& g = t.gin;
    if (t.gn < 0 || t.gn % 8 != 0 || !g.hi || !g.lo || (!g.b && !g.pf)) return false;
    units += (t.gn + TAIL_GRAD_UNIT - 1) / TAIL_GRAD_UNIT;
    if (units >= ((int64_t)1 << 30)) return false;
  }
  t.units = (int)units;
  return true;
}
