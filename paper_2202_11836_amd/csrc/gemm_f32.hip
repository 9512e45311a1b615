// Dense contractions of fp32 stages on v_mfma_f32_32x32x2_f32 (fp32 operands,
// fp32 fused multiply-adds), with the epilogues of gemm.hip.
//
// What bounds it: the fp32 matrix rate (64 FLOP per cycle and SIMD, 157
// TFLOP/s), so a wavefront's MFMAs take 64 cycles each and everything else
// fits underneath if the loads are requested early enough.  k-tiles go from
// HBM straight into a ring of LDS slots with direct-to-LDS buffer loads, up
// to NS of them in flight, one barrier per k-tile; each wavefront owns
// one 32 x 32 output block.  Three work-group shapes (and one more for the
// smallest outputs, gemm_f32_16_kernel):
//   64 x 64, 2 x 2 wavefronts, k-tiles of 32, four slots (64 KB, two
//     work-groups per CU);
//   64 x 32, 2 x 1 wavefronts times two that split every k-tile by k, four
//     slots (48 KB, three work-groups per CU), where 64 x 64 tiles leave the
//     last round of CUs part idle;
//   32 x 32, four wavefronts splitting every k-tile of 64 by k (their sums
//     are added in wavefront order at the end), eight slots: for outputs with
//     few 64 x 64 tiles, where the chain of MFMAs of one wavefront and the
//     memory latency are the time.
// Measured against a vector-ALU kernel (64 x 64 tiles, 4 x 4 outputs per
// thread, one global load -> LDS -> barrier per 16 k): a BERT-base layer at 16 x
// 128 tokens, forward and backward, 3689 -> 910 us; two layers of width 128 at
// 64 tokens 1086 -> 128 us.  Largest relative error against 64 bits 1.2e-6 ->
// 7e-7 and 3.2e-7 -> 2.3e-7.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "tail.h"

namespace {

typedef __attribute__((address_space(3))) void lds_void_t;

// 32 x 32 work-groups are used below one 64 x 64 tile per CU: the chip is part
// idle then and a tile's latency is the kernel's time.
inline bool few_tiles(int64_t t64) { return t64 < device_cus(); }

enum F32Tile { T64x64, T64x32, T32x32 };
template <F32Tile T>
struct Cfg {
  static constexpr int BM = T == T32x32 ? 32 : 64, BN = T == T64x64 ? 64 : 32;
  static constexpr int MB = BM / 32, NB = BN / 32;  // wavefronts along m and n
  static constexpr int KG = 4 / (MB * NB);          // and along k
  static constexpr int BK = T == T32x32 ? 64 : 32;  // k-tile depth
  static constexpr int A_BYTES = BM * BK * 4, STAGE = (BM + BN) * BK * 4;
};

// Buffer resource from base on; lanes that must read 0 use offset OOB.
constexpr int OOB = 0x7fffff00;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const float* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, OOB, 0x00020000);
}

// 16 or 4 bytes per lane to LDS (lane l's at dst + l * 16 or 4).
template <bool VEC>
__device__ __forceinline__ void load_lds(__amdgpu_buffer_rsrc_t rs, char* dst, int off) {
  if constexpr (VEC)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)dst, 16, off, 0, 0, 0);
  else
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)dst, 4, off, 0, 0, 0);
}

// "lgkmcnt = 0 and at most N vector memory operations outstanding" (gfx9
// s_waitcnt encoding).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | 0x70 | (((N >> 4) & 3) << 14));
}
// Wait until at most `after` (0 .. MAX) of the latest k-tiles' loads, PER
// each, are outstanding: loads complete in order.
template <int PER, int MAX>
__device__ __forceinline__ void wait_after(int after) {
  if constexpr (MAX == 0) {
    wait_vm<0>();
  } else {
    if (after >= MAX) wait_vm<PER * MAX>();
    else wait_after<PER, MAX - 1>(after);
  }
}

// Direct-to-LDS loads of one operand's k-tile (rows or columns 0 .. R - 1 of
// `nr`, k values k0 .. k0 + BK - 1 below kend; everything outside reads 0:
// the lane's offset is moved past the resource).  Each load has a resource of
// its own, from its first element on, so that the 32-bit offsets span a few
// rows only.  LDS layouts:
//   k-major: BK / 32 sub-tiles [R][32], rows of 128 bytes with 16-byte chunk
//     c at c ^ ((row >> 1) & 7), so that the 16 rows of a fragment read fall
//     on distinct banks;
//   m/n-major: [BK][R], as in memory.
// VEC: 16 bytes per lane (operand 16-byte aligned, its contiguous extent a
// multiple of 4); else 4 bytes per lane.
// What does not change from k-tile to k-tile is worked out once: per
// instruction i of the wavefront's N, its first element's address p, the
// lane's byte offset vo from there and its k in the tile, kx (too large for
// any range where the row or column is outside).
template <int R, int BK, bool KMAJ, bool VEC>
struct DmaOp {
  static constexpr int BYTES = VEC ? 16 : 4, PERI = 64 * BYTES;
  static constexpr int N = R * BK * 4 / PERI / 4;
  const float* p[N];
  int vo[N], kx[N];
  __device__ __forceinline__ void init(const float* base, int64_t ld, int nr, int wave, int lane) {
    const int el = lane * (BYTES / 4);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int e0 = (wave * N + i) * (PERI / 4);  // the instruction's first element
      bool in;
      if constexpr (KMAJ) {
        const int sub = e0 / (R * 32), row0 = (e0 % (R * 32)) / 32;  // whole rows of 32
        const int dr = el >> 5, row = row0 + dr;
        kx[i] = 32 * sub + 4 * (((el & 31) >> 2) ^ ((row >> 1) & 7)) + (el & 3);
        p[i] = base + row0 * ld;
        vo[i] = (dr * (int)ld + kx[i]) * 4;
        in = row < nr;
      } else {
        const int kr0 = e0 / R, c0 = e0 % R;  // c0 != 0: a part of one k-row
        const int dk = (c0 + el) / R, col = (c0 + el) % R;
        kx[i] = kr0 + dk;
        p[i] = base + kr0 * ld;
        vo[i] = (dk * (int)ld + col) * 4;
        in = col < nr;
      }
      if (!in) kx[i] = 1 << 30;
    }
  }
  // Instruction i of the k-tile at k0.
  __device__ __forceinline__ void issue(int i, int64_t ld, int k0, int kend, char* dst, int wave) const {
    const bool in = k0 + kx[i] < kend;
    char* to = dst + (wave * N + i) * PERI;
    if constexpr (KMAJ) load_lds<VEC>(rsrc_of(p[i]), to, in ? vo[i] + k0 * 4 : OOB);
    else load_lds<VEC>(rsrc_of(p[i] + k0 * ld), to, in ? vo[i] : OOB);
  }
};

// Four consecutive k's of the lane's row (k-major) or column: k = 8 g + 4 hf
// + j of the k range starting at kk (a multiple of 8) of the tile.  Both
// operands use this k order, so MFMA step j multiplies k = 8 g + j (lanes
// 0-31) and 8 g + 4 + j (lanes 32-63).
// (LDS addresses are plain integers: read through the shared array's pointer,
// the compiler made every k-tile's first read wait for all loads in flight.)
typedef const __attribute__((address_space(3))) float lds_cfloat_t;
typedef const __attribute__((address_space(3))) f32x4_t lds_cf32x4_t;
template <int R, bool KMAJ>
__device__ __forceinline__ f32x4_t frag4(uint32_t tile, int r, int kk, int hf) {
  if constexpr (KMAJ) {
    const int c = ((kk & 31) >> 2) + hf;
    return *(lds_cf32x4_t*)(uintptr_t)(tile + (kk >> 5) * (R * 128) + r * 128 +
                                       16 * (c ^ ((r >> 1) & 7)));
  } else {
    lds_cfloat_t* p = (lds_cfloat_t*)(uintptr_t)(tile + ((kk + 4 * hf) * R + r) * 4);
    return f32x4_t{p[0], p[R], p[2 * R], p[3 * R]};
  }
}

// Work-group barrier that leaves direct-to-LDS loads in flight (a plain
// __syncthreads() waits for all of them); the caller has waited for those
// that matter and for its own LDS operations.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// N output elements of column n, rows m(0) .. m(N - 1) (v: the accumulators):
// every operand is loaded before the first store (loads and stores share one
// counter, so a load behind a store waits for it).  Returns their sum as
// stored.
template <int EPI, int N, typename F>
__device__ __forceinline__ float epilogue(const GemmArgs& g, int64_t offC, int zs, F row, int n,
                                          const float* v) {
  if (n >= g.N) return 0.0f;
  float x[N];
  float bias = 0.0f;
  if (EPI == EPI_GELU || (EPI == EPI_STORE && g.bias)) bias = g.bias[n];
  if (EPI == EPI_MUL || EPI == EPI_RESID) {
    const float* aux = (const float*)g.aux + offC + n;
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = row(i) < g.M ? aux[(int64_t)row(i) * g.ldaux] : 0.0f;
  }
  float* C = (float*)g.C + (EPI == EPI_PARTIAL ? (int64_t)zs * g.M * g.ldc : offC) + n;
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (row(i) >= g.M) continue;
    const int64_t at = (int64_t)row(i) * g.ldc;
    float o = v[i];
    if (EPI == EPI_STORE) o = o * g.alpha + bias;
    if (EPI == EPI_MUL) o *= x[i];
    if (EPI == EPI_RESID) o += x[i];
    if (EPI == EPI_GELU) {
      const float u = o + bias;
      o = gelu_f(u);
      ((float*)g.C2 + offC + n)[at] = gelu_grad_f(u);
    }
    C[at] = o;
    sum += o;
  }
  return sum;
}

// One output tile (tm, tn) of batch entry zb over split zs of K.
template <F32Tile TILE, int NS, bool AK, bool BKM, bool VEC, int EPI>
__device__ __forceinline__ void tile_f32(const GemmArgs& g, int tm, int tn, int zb, int zs, char* smem) {
  using C = Cfg<TILE>;
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, KG = C::KG, BLK = C::MB * C::NB;
  using DA = DmaOp<BM, BK, AK, VEC>;
  using DB = DmaOp<BN, BK, BKM, VEC>;
  constexpr int PA = DA::N, PER = PA + DB::N;
  constexpr int FIRST = TILE == T32x32 ? NS - 1 : NS;  // k-tiles requested ahead
  static_assert(PER * (FIRST - 1) <= 63, "vmcnt range");
  const int lane = threadIdx.x & 63, hf = lane >> 5, rr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = tm * BM, n0 = tn * BN;
  const int kbeg = zs * g.kchunk, kend = min(g.K, kbeg + g.kchunk);
  const int64_t za = zb / g.zdiv, zr = zb % g.zdiv;
  const int nt = (kend - kbeg + BK - 1) / BK;
  const float* A = (const float*)g.A + za * g.sA1 + zr * g.sA2 + (AK ? (int64_t)kbeg : kbeg * g.lda);
  const float* B = (const float*)g.B + za * g.sB1 + zr * g.sB2 + (BKM ? (int64_t)kbeg : kbeg * g.ldb);
  if constexpr (AK) A += (int64_t)m0 * g.lda; else A += m0;
  if constexpr (BKM) B += (int64_t)n0 * g.ldb; else B += n0;
  const int nk = kend - kbeg, nm = g.M - m0, nn = g.N - n0;
  DA da;
  DB db;
  da.init(A, g.lda, nm, wave, lane);
  db.init(B, g.ldb, nn, wave, lane);
  // Load d (0 .. PER - 1) of k-tile t: A's, then B's.
  auto load = [&](int t, int d, char* slot) {
    if (d < PA) da.issue(d, g.lda, t * BK, nk, slot, wave);
    else db.issue(d - PA, g.ldb, t * BK, nk, slot + C::A_BYTES, wave);
  };
#pragma unroll
  for (int t = 0; t < FIRST; ++t)
    if (t < nt) {
#pragma unroll
      for (int d = 0; d < PER; ++d) load(t, d, smem + t * C::STAGE);
    }
  const int kg = wave / BLK, blk = wave % BLK;
  const int wm = (blk / C::NB) * 32, wn = (blk % C::NB) * 32;
  const int kw = kg * (BK / KG);  // the wavefront's k's of a k-tile
  // One accumulator per group of 8 k's in a k-tile, added at the end: a chain
  // of K / 8 additions per value instead of K / 2 (and, with one wavefront per
  // SIMD, MFMAs that do not wait for one another).
  constexpr int NF = BK / KG / 8, NM = 4 * NF;
  f32x16_t accs[NF];
#pragma unroll
  for (int s = 0; s < NF; ++s)
#pragma unroll
    for (int r = 0; r < 16; ++r) accs[s][r] = 0.0f;
  // Few k-tiles and one wavefront per SIMD: each k-tile's MFMAs start as soon
  // as it has landed.  (The loop below took 0.3 us more per product of two
  // layers of width 128 at 64 tokens, 164 -> 175 us.)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  if constexpr (TILE == T32x32) {
    for (int t = 0; t < nt; ++t) {
      // k-tile t has landed for everyone, and nobody reads k-tile t - 1 any
      // more.
      wait_after<PER, NS - 2>(min(nt - 1, t + NS - 2) - t);
      ring_barrier();
      if (t + NS - 1 < nt) {
#pragma unroll
        for (int d = 0; d < PER; ++d) load(t + NS - 1, d, smem + ((t + NS - 1) % NS) * C::STAGE);
      }
      // All of the k-tile's fragments first, so that the wavefront waits for
      // LDS once per k-tile and not once per four MFMAs.
      const uint32_t slot = lds0 + (t % NS) * C::STAGE;
      f32x4_t a[NF], b[NF];
#pragma unroll
      for (int s = 0; s < NF; ++s) {
        a[s] = frag4<BM, AK>(slot, wm + rr, kw + 8 * s, hf);
        b[s] = frag4<BN, BKM>(slot + C::A_BYTES, wn + rr, kw + 8 * s, hf);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int s = 0; s < NF; ++s)
          accs[s] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s][j], b[s][j], accs[s], 0, 0, 0);
    }
  } else {
    // While the MFMAs of k-tile t run, the fragments of k-tile t + 1 are read
    // (two register sets) and k-tile t + NS is requested, each between two
    // MFMAs, so that a wavefront alone on its SIMD keeps the matrix core busy.
    // (With reads and requests ahead of the MFMAs a BERT-base layer at 16 x 128
    // took 967 us instead of 910.)
    // At the barrier of step t everyone holds k-tile t's fragments, so its slot
    // takes k-tile t + NS, and k-tile t + 1 has landed.
    f32x4_t fa[2][NF], fb[2][NF];
    auto read = [&](auto set, auto fc, uint32_t slot) {
      constexpr int S = decltype(set)::value, F = decltype(fc)::value, s = F / 2;
      if constexpr (F % 2 == 0) fa[S][s] = frag4<BM, AK>(lds0 + slot, wm + rr, kw + 8 * s, hf);
      else fb[S][s] = frag4<BN, BKM>(lds0 + slot + C::A_BYTES, wn + rr, kw + 8 * s, hf);
    };
    wait_after<PER, NS - 1>(min(nt - 1, NS - 1));
    ring_barrier();
    static_for<0, 2 * NF>([&](auto f) { read(std::integral_constant<int, 0>(), f, 0); });
    uint32_t slot = 0;
    // ISSUE: 1 = request k-tile t + NS between the MFMAs, 0 = nothing left to
    // request, 2 = request it if there is one.
    auto step = [&](auto par, auto issue_c, int t) {
      constexpr int cur = decltype(par)::value;
      constexpr int ISSUE = decltype(issue_c)::value;
      using Next = std::integral_constant<int, cur ^ 1>;
      if constexpr (ISSUE == 1) wait_vm<PER * (NS - 2)>();
      else wait_after<PER, NS - 2>(max(0, min(nt - 1, t + NS - 1) - (t + 1)));
      ring_barrier();
      char* const free_slot = smem + slot;
      // (after the last k-tile these reads fetch a stale slot, never used)
      slot = slot == (NS - 1) * C::STAGE ? 0 : slot + C::STAGE;
      if (ISSUE == 2 && t + NS < nt) {
#pragma unroll
        for (int d = 0; d < PER; ++d) load(t + NS, d, free_slot);
      }
      static_for<0, NM>([&](auto mc) {
        constexpr int m = decltype(mc)::value, s = m % NF, j = m / NF;
        accs[s] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[cur][s][j], fb[cur][s][j], accs[s], 0, 0, 0);
        if constexpr (m % 2 == 0) read(Next(), std::integral_constant<int, m / 2>(), slot);
        if constexpr (ISSUE == 1) {
#pragma unroll
          for (int d = 0; d < PER; ++d)
            if (d * NM / PER == m) load(t + NS, d, free_slot);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    int t = 0;
    for (; t + 1 + NS < nt; t += 2) {
      step(I0(), I1(), t);
      step(I1(), I1(), t + 1);
    }
    for (; t < nt; t += 2) {
      step(I0(), I2(), t);
      if (t + 1 < nt) step(I1(), I0(), t + 1);
    }
  }
  f32x16_t acc = accs[0];
#pragma unroll
  for (int s = 1; s < NF; ++s) acc += accs[s];
  const int64_t offC = za * g.sC1 + zr * g.sC2;
  const int n = n0 + wn + rr;
  // The k groups' sums, added in their order; each of a block's wavefronts
  // then owns NR accumulator registers (register r: row 8 (r / 4) + 4 hf +
  // r % 4 of the block).
  constexpr int NR = 16 / KG;
  float v[NR];
  if constexpr (KG > 1) {
    __syncthreads();  // the ring becomes the exchange area: [wave][16][64]
    float* ex = (float*)smem;
#pragma unroll
    for (int r = 0; r < 16; ++r) ex[(wave * 16 + r) * 64 + lane] = acc[r];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const float* p = ex + (blk * 16 + NR * kg + j) * 64 + lane;
      v[j] = p[0];
#pragma unroll
      for (int k = 1; k < KG; ++k) v[j] += p[k * BLK * 1024];
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = acc[r];
  }
  const int mb = m0 + wm + 4 * hf;
  const float cs = epilogue<EPI, NR>(
      g, offC, zs, [&](int j) { return mb + 8 * ((NR * kg + j) >> 2) + (j & 3); }, n, v);
  if (g.colpart) {  // column sums per block of 32 rows, in a fixed order
    float* P = g.colpart + (zb / g.zdiv) * g.cp_batch + (zb % g.zdiv) * g.sC2;
    if constexpr (KG > 1) {
      float* ex = (float*)smem;
      __syncthreads();
      ex[((blk * KG + kg) * 2 + hf) * 32 + rr] = cs;
      __syncthreads();
      if (kg == 0 && hf == 0 && n < g.N && m0 + wm < g.M) {
        const float* p = ex + blk * KG * 64 + rr;
        float sum = p[0];
#pragma unroll
        for (int i = 1; i < 2 * KG; ++i) sum += p[i * 32];
        P[(int64_t)((m0 + wm) / 32) * g.cp_ld + n] = sum;
      }
    } else {
      const float sum = cs + __shfl_xor(cs, 32, 64);
      if (hf == 0 && n < g.N && m0 + wm < g.M) P[(int64_t)((m0 + wm) / 32) * g.cp_ld + n] = sum;
    }
  }
}

// Consecutive work-groups go round robin over the 8 XCDs: each XCD takes a
// contiguous range of tiles, walked in groups of 8 tile-rows that share B.
__device__ __forceinline__ void tile_of(int bid, int nbm, int nbn, int& tm, int& tn) {
  const int total = nbm * nbn;
  if ((total & 7) == 0) bid = (bid & 7) * (total >> 3) + (bid >> 3);
  constexpr int GM = 8;
  const int group = bid / (GM * nbn), first = group * GM, size = min(nbm - first, GM);
  const int r = bid - group * GM * nbn;
  tm = first + r % size;
  tn = r / size;
}

// One 16 x 16 output tile (v_mfma_f32_16x16x4_f32, four wavefronts splitting
// each k-tile of 64 by k), for outputs so small that even 32 x 32 tiles leave
// most CUs idle: a wavefront's chain of MFMAs is a quarter as long (K = 512: 1024
// cycles against 4096).  64 x 128 x 512 7.4 -> 4.6 us, two layers of width 128
// at 64 tokens 156 -> 128 us a step.  Operands 16-byte aligned, batch 1, no
// column sums.
constexpr int T16_NS = 8;
constexpr int T16_STAGE = 2 * 16 * 64 * 4;
template <bool AK, bool BKM, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_16_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) char smem[T16_NS * T16_STAGE];
  constexpr int NS = T16_NS, BK = 64, OP = T16_STAGE / 2;
  const int lane = threadIdx.x & 63, kq = lane >> 4, rr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tm, tn;
  tile_of(blockIdx.x, (g.M + 15) / 16, (g.N + 15) / 16, tm, tn);
  const int m0 = tm * 16, n0 = tn * 16, nt = (g.K + BK - 1) / BK;
  DmaOp<16, BK, AK, true> da;
  DmaOp<16, BK, BKM, true> db;
  static_assert(decltype(da)::N == 1 && decltype(db)::N == 1, "one load each");
  da.init((const float*)g.A + (AK ? m0 * g.lda : m0), g.lda, g.M - m0, wave, lane);
  db.init((const float*)g.B + (BKM ? n0 * g.ldb : n0), g.ldb, g.N - n0, wave, lane);
  auto issue = [&](int t) {
    char* slot = smem + (t % NS) * T16_STAGE;
    da.issue(0, g.lda, t * BK, g.K, slot, wave);
    db.issue(0, g.ldb, t * BK, g.K, slot + OP, wave);
  };
#pragma unroll
  for (int t = 0; t < NS - 1; ++t)
    if (t < nt) issue(t);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  // Lane's operand values: k = 16 wave + 4 kq + i of its row or column.
  auto frag = [&](auto kmaj, uint32_t tile) {
    const int k = 16 * wave + 4 * kq;
    if constexpr (decltype(kmaj)::value) {
      return *(lds_cf32x4_t*)(uintptr_t)(tile + (k >> 5) * (16 * 128) + rr * 128 +
                                         16 * (((k & 31) >> 2) ^ ((rr >> 1) & 7)));
    } else {
      lds_cfloat_t* p = (lds_cfloat_t*)(uintptr_t)(tile + (k * 16 + rr) * 4);
      return f32x4_t{p[0], p[16], p[32], p[48]};
    }
  };
  f32x4_t acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  for (int t = 0; t < nt; ++t) {
    // k-tile t has landed for everyone, and nobody reads k-tile t - 1 any more.
    wait_after<2, NS - 2>(min(nt - 1, t + NS - 2) - t);
    ring_barrier();
    if (t + NS - 1 < nt) issue(t + NS - 1);
    const uint32_t slot = lds0 + (t % NS) * T16_STAGE;
    const f32x4_t a = frag(std::integral_constant<bool, AK>(), slot);
    const f32x4_t b = frag(std::integral_constant<bool, BKM>(), slot + OP);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      acc[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], acc[i & 1], 0, 0, 0);
  }
  // Sums over the wavefronts, in their order; wavefront w owns register w (row
  // 4 kq + w).
  __syncthreads();
  float* ex = (float*)smem;
#pragma unroll
  for (int r = 0; r < 4; ++r) ex[(wave * 4 + r) * 64 + lane] = acc[0][r] + acc[1][r];
  __syncthreads();
  const float* p = ex + wave * 64 + lane;
  const float v[1] = {((p[0] + p[256]) + p[512]) + p[768]};
  epilogue<EPI, 1>(g, 0, 0, [&](int) { return m0 + 4 * kq + wave; }, n0 + rr, v);
}

template <F32Tile T, bool VEC>
struct Ring {
  // 4-byte loads: as many slots as keep the outstanding count within vmcnt's
  // range
  static constexpr int NS = T == T32x32 && VEC ? 8 : 4;
  static constexpr int LDS = NS * Cfg<T>::STAGE;
};

template <F32Tile T, bool AK, bool BKM, bool VEC, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  using Rg = Ring<T, VEC>;
  __shared__ __attribute__((aligned(1024))) char smem[Rg::LDS];
  constexpr int BM = Cfg<T>::BM, BN = Cfg<T>::BN;
  int tm, tn;
  tile_of(blockIdx.x, (g.M + BM - 1) / BM, (g.N + BN - 1) / BN, tm, tn);
  tile_f32<T, Rg::NS, AK, BKM, VEC, EPI>(g, tm, tn, blockIdx.z / g.ksplit, blockIdx.z % g.ksplit,
                                             smem);
}

// Contractions of the attention backward in one launch (grid y), per (batch,
// head): p[0] dV = P^T dC, p[1] dK = dS^T Q, and p[2] dQ = dS K.
struct Attn3 {
  GemmArgs p[3];
};
template <F32Tile T, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_attn_bwd_kernel(Attn3 a) {
  using Rg = Ring<T, VEC>;
  __shared__ __attribute__((aligned(1024))) char smem[Rg::LDS];
  constexpr int R = Cfg<T>::BM;
  static_assert(R == Cfg<T>::BN, "square tiles");
  const int nbn = (a.p[0].N + R - 1) / R;
  const int tm = blockIdx.x / nbn, tn = blockIdx.x % nbn;
  if (blockIdx.y == 2)
    tile_f32<T, Rg::NS, true, false, VEC, EPI_STORE>(a.p[2], tm, tn, blockIdx.z, 0, smem);
  else if (blockIdx.y == 0)
    tile_f32<T, Rg::NS, false, false, VEC, EPI_STORE>(a.p[0], tm, tn, blockIdx.z, 0, smem);
  else
    tile_f32<T, Rg::NS, false, false, VEC, EPI_STORE>(a.p[1], tm, tn, blockIdx.z, 0, smem);
}

// A layer's weight gradients in one launch: work-group b serves problem q
// with blk0[q] <= b < blk0[q + 1]; a problem's work-groups are its tiles times
// its splits.  The tail's units (one split only) follow, four per work-group.
struct WgradGroup {
  GemmArgs p[GEMM_GROUP_MAX];
  int blk0[GEMM_GROUP_MAX + 1];
  int n;
  TailJobs tail;
};
template <F32Tile T>
__global__ __launch_bounds__(256) void gemm_f32_wgrad_kernel(WgradGroup w) {
  using Rg = Ring<T, true>;
  __shared__ __attribute__((aligned(1024))) char smem[Rg::LDS];
  constexpr int R = Cfg<T>::BM;
  static_assert(R == Cfg<T>::BN, "square tiles");
  const int b = blockIdx.x;
  if (b >= w.blk0[GEMM_GROUP_MAX]) {
    tail_unit<8>(tail_arg(offsetof(WgradGroup, tail)), (b - w.blk0[GEMM_GROUP_MAX]) * 4 + (int)(threadIdx.x >> 6), threadIdx.x & 63);
    return;
  }
  int q = 0;
#pragma unroll
  for (int k = 1; k < GEMM_GROUP_MAX; ++k)
    if (k < w.n && b >= w.blk0[k]) q = k;
  // (a copy per problem: a run-time index into the argument would put it in
  // scratch memory)
  GemmArgs g;
  switch (q) {
    case 0: g = w.p[0]; break;
    case 1: g = w.p[1]; break;
    case 2: g = w.p[2]; break;
    default: g = w.p[3]; break;
  }
  const int nbm = (g.M + R - 1) / R, nbn = (g.N + R - 1) / R;
  const int lb = b - w.blk0[q], zs = lb / (nbm * nbn);
  int tm, tn;
  tile_of(lb - zs * nbm * nbn, nbm, nbn, tm, tn);
  tile_f32<T, Rg::NS, false, false, true, EPI_PARTIAL>(g, tm, tn, 0, zs, smem);
}

// out[q] = the fixed-order sum of problem q's splits; then the tail, four
// units per work-group.
struct F32Reduce {
  const float* part[GEMM_GROUP_MAX];
  float* out[GEMM_GROUP_MAX];
  int64_t mn[GEMM_GROUP_MAX];
  int ks[GEMM_GROUP_MAX];
  int blk0[GEMM_GROUP_MAX + 1];
  int n;
  TailJobs tail;
};
__global__ __launch_bounds__(256, 8) void gemm_f32_group_reduce_kernel(F32Reduce rd) {
  const int b = blockIdx.x;
  if (b >= rd.blk0[GEMM_GROUP_MAX]) {
    tail_unit<4>(tail_arg(offsetof(F32Reduce, tail)), (b - rd.blk0[GEMM_GROUP_MAX]) * 4 + (int)(threadIdx.x >> 6), threadIdx.x & 63);
    return;
  }
  int q = 0;
#pragma unroll
  for (int k = 1; k < GEMM_GROUP_MAX; ++k)
    if (k < rd.n && b >= rd.blk0[k]) q = k;
  const float* part;
  float* out;
  int64_t mn;
  int ks, b0;
  switch (q) {
    case 0: part = rd.part[0]; out = rd.out[0]; mn = rd.mn[0]; ks = rd.ks[0]; b0 = rd.blk0[0]; break;
    case 1: part = rd.part[1]; out = rd.out[1]; mn = rd.mn[1]; ks = rd.ks[1]; b0 = rd.blk0[1]; break;
    case 2: part = rd.part[2]; out = rd.out[2]; mn = rd.mn[2]; ks = rd.ks[2]; b0 = rd.blk0[2]; break;
    default: part = rd.part[3]; out = rd.out[3]; mn = rd.mn[3]; ks = rd.ks[3]; b0 = rd.blk0[3]; break;
  }
  const int64_t i = ((int64_t)(b - b0) * 256 + threadIdx.x) * 4;
  if (i >= mn) return;
  f32x4_t s = *(const f32x4_t*)(part + i);
  for (int z = 1; z < ks; ++z) s += *(const f32x4_t*)(part + (int64_t)z * mn + i);
  *(f32x4_t*)(out + i) = s;
}

// 16-byte loads: the operand's contiguous extent, row stride and every batch
// offset are multiples of 4 (all allocations are 256-byte aligned).
bool vec_ok(const GemmArgs& g, bool ak, bool bk) {
  const int64_t any = g.lda | g.ldb | g.sA1 | g.sA2 | g.sB1 | g.sB2 | (ak ? g.K : g.M) |
                      (bk ? g.K : g.N);
  return (any & 3) == 0 && (((uintptr_t)g.A | (uintptr_t)g.B) & 15) == 0;
}
// A load's offsets are 32-bit bytes below OOB.  k-major: 7 rows and the k extent,
// less than 7 x 2^27 + 2^30; m/n-major: up to 15 k-rows (16 x 16 tiles), less than
// 15 x 2^27.
bool fits(const GemmArgs& g) {
  const int64_t k = g.K;
  return std::max(g.lda, g.ldb) < ((int64_t)1 << 25) && k * 4 < ((int64_t)1 << 30);
}
int64_t tiles_of(const GemmArgs& g, int bm, int bn) {
  return (int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn);
}
// 32 x 32 tiles below one 64 x 64 tile per CU.  Otherwise a CU works through its
// share of the tiles two or three at a time, and the fullest CU is the time: 64 x
// 32 tiles (5% slower for their size) where they divide more evenly.
F32Tile f32_tile(const GemmArgs& g, int64_t batch) {
  const int64_t cus = device_cus();
  const int64_t t64 = tiles_of(g, 64, 64) * batch, t32 = tiles_of(g, 64, 32) * batch;
  if (few_tiles(t64)) return T32x32;
  return ((t32 + cus - 1) / cus) * 21 < ((t64 + cus - 1) / cus) * 40 ? T64x32 : T64x64;
}

template <bool AK, bool BKM, int EPI>
hipError_t launch(const GemmArgs& g, int batch, hipStream_t st) {
  const bool vec = vec_ok(g, AK, BKM);
  const F32Tile t = f32_tile(g, (int64_t)batch * g.ksplit);
  auto grid = [&](int bm, int bn) {
    return dim3((unsigned)tiles_of(g, bm, bn), 1, (unsigned)(batch * g.ksplit));
  };
  if (vec) {
    // 16 x 16 tiles while they are one per CU (the line 32 x 32 tiles have too)
    if (tiles_of(g, 16, 16) <= device_cus() && batch * g.ksplit == 1 && !g.colpart)
      hipLaunchKernelGGL((gemm_f32_16_kernel<AK, BKM, EPI>), grid(16, 16), dim3(256), 0, st, g);
    else if (t == T32x32)
      hipLaunchKernelGGL((gemm_f32_kernel<T32x32, AK, BKM, true, EPI>), grid(32, 32), dim3(256), 0, st, g);
    else if (t == T64x32)
      hipLaunchKernelGGL((gemm_f32_kernel<T64x32, AK, BKM, true, EPI>), grid(64, 32), dim3(256), 0, st, g);
    else
      hipLaunchKernelGGL((gemm_f32_kernel<T64x64, AK, BKM, true, EPI>), grid(64, 64), dim3(256), 0, st, g);
    return hipGetLastError();
  }
  // Operands with rows that are not 16-byte aligned: the score matrix of a
  // sequence length that is not a multiple of 4 (EPI_STORE, P V).
  if constexpr (EPI == EPI_STORE && AK && !BKM) {
    if (t == T32x32)
      hipLaunchKernelGGL((gemm_f32_kernel<T32x32, AK, BKM, false, EPI>), grid(32, 32), dim3(256), 0, st, g);
    else
      hipLaunchKernelGGL((gemm_f32_kernel<T64x64, AK, BKM, false, EPI>), grid(64, 64), dim3(256), 0, st, g);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t gemm_f32(const GemmArgs& g, bool a_kmajor, bool b_kmajor, GemmEpi epi, int batch,
                    hipStream_t st) {
  if (g.M <= 0 || g.N <= 0 || batch <= 0) return hipSuccess;
  if (!a_kmajor || g.ksplit != 1 || !fits(g)) return hipErrorInvalidValue;
  if (b_kmajor) {
    if (epi == EPI_STORE) return launch<true, true, EPI_STORE>(g, batch, st);
    if (epi == EPI_GELU) return launch<true, true, EPI_GELU>(g, batch, st);
  } else {
    if (epi == EPI_STORE) return launch<true, false, EPI_STORE>(g, batch, st);
    if (epi == EPI_MUL) return launch<true, false, EPI_MUL>(g, batch, st);
    if (epi == EPI_RESID) return launch<true, false, EPI_RESID>(g, batch, st);
  }
  return hipErrorInvalidValue;
}

hipError_t gemm_f32_attn_bwd(const GemmArgs& dv, const GemmArgs& dk, const GemmArgs* dq, int batch,
                             hipStream_t st) {
  if (dv.M <= 0 || batch <= 0) return hipSuccess;
  const unsigned n = dq ? 3 : 2;
  Attn3 a = {{dv, dk, dq ? *dq : dk}};
  bool vec = true;
  for (unsigned i = 0; i < n; ++i) {
    const GemmArgs& g = a.p[i];
    if (g.M != dv.M || g.N != dv.N || g.ksplit != 1 || !fits(g)) return hipErrorInvalidValue;
    vec = vec && vec_ok(g, i == 2, false);
  }
  const bool small = few_tiles(tiles_of(dv, 64, 64) * batch * n);
  const int r = small ? 32 : 64;
  const dim3 grid((unsigned)tiles_of(dv, r, r), n, (unsigned)batch);
  if (small && vec)
    hipLaunchKernelGGL((gemm_f32_attn_bwd_kernel<T32x32, true>), grid, dim3(256), 0, st, a);
  else if (small)
    hipLaunchKernelGGL((gemm_f32_attn_bwd_kernel<T32x32, false>), grid, dim3(256), 0, st, a);
  else if (vec)
    hipLaunchKernelGGL((gemm_f32_attn_bwd_kernel<T64x64, true>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((gemm_f32_attn_bwd_kernel<T64x64, false>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

F32WgradPlan gemm_f32_wgrad_plan(int h, int f, int K) {
  // Two work-groups of 64 x 64 per CU over the layer's four gradients (h and f
  // are multiples of 64); k ranges of at least 256.
  const int64_t hb = h / 64, fb = f / 64, tiles = 4 * hb * hb + 2 * hb * fb;
  int ks = (int)std::max<int64_t>(1, std::min<int64_t>(2 * device_cus() / tiles, K / 256));
  // Width 64 over so many tokens that the column partials of one-token sequences
  // fill the no-alloc backward's scratch: 6.3 MB of partials, what the scratch
  // has left for them (h = f = 64: 64 splits, not 85).
  if (h == 64 && K > 262144)
    ks = (int)std::max<int64_t>(1, std::min<int64_t>(ks, 128 * 3 * 64 * 64 / (tiles * 4096)));
  const int chunk = ((K + ks - 1) / ks + 63) / 64 * 64;
  ks = (K + chunk - 1) / chunk;
  return {ks, few_tiles(tiles * ks)};
}

hipError_t gemm_f32_wgrad_group(const GemmArgs* p, float* const* out, int n, F32WgradPlan plan,
                                const TailJobs& tail, hipStream_t st) {
  const int ks = plan.ks;
  const bool small = plan.small;
  if (ks < 1 || n < 1 || n > GEMM_GROUP_MAX) return hipErrorInvalidValue;
  WgradGroup w{};
  F32Reduce rd{};
  for (int q = 0; q < n; ++q) {
    GemmArgs g = p[q];
    if (g.M < 1 || g.N < 1 || g.K < 1 || g.ldc != g.N || !vec_ok(g, false, false))
      return hipErrorInvalidValue;
    g = gemm_split(g, ks);
    if (g.ksplit != ks) return hipErrorInvalidValue;
    if (!fits(g)) return hipErrorInvalidValue;
    // one split writes the gradient itself
    if (g.ksplit == 1) g.C = out[q];
    w.p[q] = g;
  }
  int64_t blocks = 0, rblocks = 0;
  for (int q = 0; q < n; ++q) {
    const GemmArgs& g = w.p[q];
    w.blk0[q] = (int)blocks;
    blocks += tiles_of(g, small ? 32 : 64, small ? 32 : 64) * g.ksplit;
    if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    if (g.ksplit > 1) {
      const int j = rd.n++;
      rd.part[j] = (const float*)g.C;
      rd.out[j] = out[q];
      rd.mn[j] = (int64_t)g.M * g.N;
      rd.ks[j] = g.ksplit;
      rd.blk0[j] = (int)rblocks;
      rblocks += (rd.mn[j] / 4 + 255) / 256;
    }
  }
  for (int q = n; q <= GEMM_GROUP_MAX; ++q) w.blk0[q] = (int)blocks;
  w.n = n;
  for (int j = rd.n; j <= GEMM_GROUP_MAX; ++j) rd.blk0[j] = (int)rblocks;
  TailJobs& t = ks > 1 ? rd.tail : w.tail;
  t = tail;
  if (!tail_prepare(t)) return hipErrorInvalidValue;
  (ks > 1 ? rblocks : blocks) += (t.units + 3) / 4;
  if (blocks >= ((int64_t)1 << 31) || rblocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  if (small)
    hipLaunchKernelGGL((gemm_f32_wgrad_kernel<T32x32>), dim3((unsigned)blocks), dim3(256), 0, st, w);
  else
    hipLaunchKernelGGL((gemm_f32_wgrad_kernel<T64x64>), dim3((unsigned)blocks), dim3(256), 0, st, w);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || ks == 1) return e;
  hipLaunchKernelGGL(gemm_f32_group_reduce_kernel, dim3((unsigned)rblocks), dim3(256), 0, st, rd);
  return hipGetLastError();
}
