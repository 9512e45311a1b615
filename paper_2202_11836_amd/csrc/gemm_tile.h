// Device pieces shared by the bf16 GEMM kernels: buffer resources, k-tile
// loads into LDS, MFMA operand fragments, 8-column epilogues.
#pragma once
#include <type_traits>

#include "kernels.h"

namespace {

// Buffer resource over [base, base + bytes): loads past the end return 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
  const int nrec = (int)(bytes < 0 ? 0 : (bytes > 0x7fffffff ? 0x7fffffff : bytes));
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, nrec, 0x00020000);
}

typedef __attribute__((address_space(3))) void lds_void_t;

// LDS tile layouts (no padding; 16-byte chunks XOR-swizzled so that the
// fragment reads of each 16-lane group hit distinct banks):
//   k-major  [R][BK]: row r, logical chunk c (8 k values) at physical chunk
//            c ^ kswz(r) of the row's 2 BK bytes, kswz(r) = (r >> 1) & 7 for
//            BK = 64 and (r >> 2) & 3 for BK = 32;
//   m/n-major [BK][R]: k-row k, logical chunk c (8 rows/columns) at physical
//            chunk c ^ nswz(k) of the row's 2R bytes, nswz(k) = 4 (k & 3) for
//            R >= 128 and 4 ((k >> 1) & 1) for R = 64, so the 4 k-rows x 2
//            chunks of each 16-lane transposing read, and the two groups of a
//            32-lane pass, cover 16 distinct chunks.
//
// dma_tile issues the direct-to-LDS loads (buffer_load ... lds, 16 bytes per
// lane; lane l of a load lands at LDS base + 16 l) that fill one operand tile
// of k-tile k0 (k relative to the resource, see the kernel), so the tile
// never passes through VGPRs.  Each 1 KB block is one instruction; the W
// wavefronts of the work-group split the blocks.
template <int BK>
__device__ __forceinline__ int kswz(int r) {
  return BK == 64 ? ((r >> 1) & 7) : ((r >> 2) & 3);
}

template <int R>
__device__ __forceinline__ int nswz(int k) {
  return R >= 128 ? 4 * (k & 3) : 4 * ((k >> 1) & 1);
}

// Load i of the NB / W that one wavefront makes for an operand tile.
template <int R, bool KMAJ, int BK, int W>
__device__ __forceinline__ void dma_load(__amdgpu_buffer_rsrc_t rs, int64_t ld, int k0, char* dst,
                                         int wave, int lane, int i) {
  constexpr int NB = R * BK * 2 / 1024;  // 1 KB blocks in the tile
  const int q = wave * (NB / W) + i;
  int64_t elem;
  if constexpr (KMAJ) {
    constexpr int CPR = BK / 8;   // chunks per row
    constexpr int RPB = 64 / CPR; // rows per block
    const int row = RPB * q + lane / CPR;
    const int c = (lane % CPR) ^ kswz<BK>(row);
    elem = (int64_t)row * ld + k0 + 8 * c;
  } else {
    constexpr int CPR = R / 8;           // chunks per k-row
    constexpr int KPB = 64 / CPR;        // k-rows per block
    const int kr = KPB * q + lane / CPR;
    const int c = (lane % CPR) ^ nswz<R>(kr);
    elem = (int64_t)(k0 + kr) * ld + 8 * c;
  }
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + q * 1024), 16, (int)(elem * 2),
                                           0, 0, 0);
}
template <int R, bool KMAJ, int BK, int W>
__device__ __forceinline__ void dma_tile(__amdgpu_buffer_rsrc_t rs, int64_t ld, int k0, char* dst,
                                         int wave, int lane) {
#pragma unroll
  for (int i = 0; i < R * BK * 2 / 1024 / W; ++i)
    dma_load<R, KMAJ, BK, W>(rs, ld, k0, dst, wave, lane, i);
}

// MFMA operand fragments: 8 consecutive k (offset ks * 16 + 8 * (lane / 32))
// of row r0 + lane % 32.  k-major: one 16-byte read.  m/n-major: two
// ds_read_b64_tr_b16.  That instruction works on groups of 16 lanes: lane j
// supplies the address of 4 consecutive 16-bit values V[j][0..3], and lane i
// receives V[4e + i / 4][i % 4] for e = 0..3.  Lane j of a group points at
// k-row k0 + j / 4, columns mb + 4 (j % 4), so lane i receives column mb + i
// at k-rows k0 .. k0 + 3 (the second read: k0 + 4 .. k0 + 7).
typedef __attribute__((address_space(3))) char lds_char_t;

// An m/n-major fragment as read: the two halves of the transposing reads
// (ds_read_tr16_b64), combined only after lds_wait() / frag_hold().
struct TrFrag {
  u32x2_t lo, hi;
};
__device__ __forceinline__ bf16x8_t frag_val(const bf16x8_t& v) { return v; }
__device__ __forceinline__ bf16x8_t frag_val(const TrFrag& v) {
  return __builtin_bit_cast(bf16x8_t, u32x4_t{v.lo[0], v.lo[1], v.hi[0], v.hi[1]});
}
__device__ __forceinline__ void frag_hold(bf16x8_t&) {}
__device__ __forceinline__ void frag_hold(TrFrag& v) {
  lds_hold(v.lo);
  lds_hold(v.hi);
}

// Per-lane LDS addresses of one operand's fragments in ring slot 0, so that
// every fragment read in the main loop is one instruction with an immediate
// offset (no per-read address arithmetic).  k-major: one address per
// k-step, fragment f (32 rows further) at +f * 32 * 2 BK.  m/n-major: one
// address per fragment, k-step ks at +ks * 16 * 2R, the second transposing
// read at +4 * 2R.  (The swizzle terms depend only on the lane because the
// wavefront's first row is a multiple of 32.)
template <int R, bool KMAJ, int BK, int NF>
struct FragPtrs {
  static constexpr int KS = BK / 16;
  static constexpr int N = KMAJ ? KS : NF;
  using Frag = typename std::conditional<KMAJ, bf16x8_t, TrFrag>::type;
  uint32_t p[N];
  __device__ __forceinline__ void init(uint32_t base, int r0, int lane) {
    if constexpr (KMAJ) {
      const int r = r0 + (lane & 31);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        p[ks] = base + r * (2 * BK) + 16 * ((2 * ks + (lane >> 5)) ^ kswz<BK>(r));
    } else {
      const int grp = lane >> 4, j = lane & 15;
      const int kr = 8 * (grp >> 1) + (j >> 2);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const int col = r0 + f * 32 + 16 * (grp & 1) + 4 * (j & 3);
        p[f] = base + kr * (2 * R) + 16 * ((col >> 3) ^ nswz<R>(kr)) + 2 * (col & 7);
      }
    }
  }
  __device__ __forceinline__ void advance(int delta) {
#pragma unroll
    for (int n = 0; n < N; ++n) p[n] += delta;
  }
  // fragment f of k-step KSI
  template <int KSI>
  __device__ __forceinline__ Frag get(int f) const {
    if constexpr (KMAJ) {
      return *(const __attribute__((address_space(3))) bf16x8_t*)(
          (const lds_char_t*)(uintptr_t)p[KSI] + f * 32 * (2 * BK));
    } else {
      return TrFrag{ds_read_tr16_b64<KSI * 16 * (2 * R)>(p[f]),
                    ds_read_tr16_b64<KSI * 16 * (2 * R) + 4 * (2 * R)>(p[f])};
    }
  }
};


// Epilogue for 8 consecutive columns n..n+7 of row m (n % 8 == 0, n < N):
// EPI_STORE, EPI_GELU, EPI_PARTIAL (slot zs).
// b0, b1: bias[n .. n + 7], loaded once per tile by the caller.
template <int EPI>
__device__ __forceinline__ void epi8(const GemmArgs& g, int zs, int m, int n, float v[8], f32x4_t b0,
                                     f32x4_t b1) {
  static_assert(EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_PARTIAL, "");
  const int64_t idx = (int64_t)m * g.ldc + n;
  if constexpr (EPI == EPI_PARTIAL) {
    float* C = (float*)g.C + (int64_t)zs * g.M * g.ldc + idx;
    *(f32x4_t*)C = f32x4_t{v[0], v[1], v[2], v[3]};
    *(f32x4_t*)(C + 4) = f32x4_t{v[4], v[5], v[6], v[7]};
    return;
  }
  if (EPI == EPI_STORE) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] *= g.alpha;
  }
  if (g.bias) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] += b0[i];
      v[4 + i] += b1[i];
    }
  }
  if (EPI == EPI_GELU) {
    // v holds u = acc + bias: store GELU(u) and GELU'(u)
    u32x4_t o, q;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float gv[2], dv[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float u = v[2 * i + e];
        const GeluParts p = gelu_parts(u);
        gv[e] = u * p.cdf;
        dv[e] = fmaf(u * 0.39894228040143268f, p.e, p.cdf);
      }
      o[i] = pack_bf16x2(gv[0], gv[1]);
      q[i] = pack_bf16x2(dv[0], dv[1]);
    }
    *(u32x4_t*)((bf16_t*)g.C + idx) = o;
    *(u32x4_t*)((bf16_t*)g.C2 + idx) = q;
    return;
  }
  u32x4_t o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
  *(u32x4_t*)((bf16_t*)g.C + idx) = o;
}

// EPI_MUL on 8 values: v * aux (aux: 8 packed bf16), rounded to bf16 and packed;
// v returns the rounded values.
__device__ __forceinline__ u32x4_t mul8(float v[8], u32x4_t x) {
  u32x4_t o;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] *= __uint_as_float(x[i] << 16);
    v[2 * i + 1] *= __uint_as_float(x[i] & 0xffff0000u);
    o[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    v[2 * i] = __uint_as_float(o[i] << 16);
    v[2 * i + 1] = __uint_as_float(o[i] & 0xffff0000u);
  }
  return o;
}

// s_waitcnt immediate (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] |
// lgkmcnt[11:8] | vmcnt[5:4] << 14) for "lgkmcnt = 0 and at most N vector
// memory operations outstanding".
template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | 0x70 | (((N >> 4) & 3) << 14));
}

}  // namespace
