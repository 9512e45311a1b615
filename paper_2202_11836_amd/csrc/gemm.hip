// Dense contractions of bf16 stages with many output tiles: MFMA GEMM (fp32
// accumulate) with fused epilogues, and the tile rules of all bf16 GEMMs.
//
// A persistent work-group per CU walks 256 x 256 output tiles; its 8 wavefronts
// (two per SIMD) form a 2 x 4 grid, each owning a 128 x 64 sub-tile computed with
// v_mfma_f32_32x32x16_bf16.  k-tiles of 64 go straight from HBM into a ring
// of LDS slots with direct-to-LDS buffer loads, issued ahead of use, so no
// staging registers and no LDS store instructions sit in the main loop, and
// the one barrier per k-tile overlaps the MFMAs of the last k-step.  Operands stored m/n-contiguous in
// HBM keep that layout in LDS and their MFMA fragments are read with gfx950's
// transposing LDS read.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "gemm_tile.h"
#include "tail.h"

namespace {

// Tile order inside a z slice: groups of TILE_GM tile-rows, column by column
// within a group (tiles that share A rows / B columns run close together).
// (4 rather than 8: 1-3% faster for the 12- and 16-tile-wide encoder GEMMs,
// -1.2% per stage step.)
constexpr int TILE_GM = 4;

// Linear tile index -> (m tile, n tile) for a persistent grid.  Work-group
// w starts on XCD w % 8 and keeps it (the grid is a multiple of 8), so the
// tile ranges are dealt out per XCD as above.
__device__ __forceinline__ void decode_tile(int vt, int total, int nbm, int nbn, int& tm, int& tn,
                                            bool xcd_remap = true) {
  int bid = vt;
  if (xcd_remap && (total & 7) == 0) bid = (vt & 7) * (total >> 3) + (vt >> 3);
  constexpr int GM = TILE_GM;
  const int per_group = GM * nbn;
  const int group = bid / per_group;
  const int first_m = group * GM;
  const int gsize = min(nbm - first_m, GM);
  const int r = bid - group * per_group;
  tm = first_m + r % gsize;
  tn = r / gsize;
}

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM
//
// Block = 2 x (waves / 2) wavefronts over a BM x BN tile; each wavefront
// owns a (BM/2) x (BN/(waves/2)) sub-tile = TM x TN accumulators of 32 x 32.
// k-tiles of 64 sit in a ring of two LDS slots (with the epilogue staging
// area, the full 160 KB of a gfx950 CU), one barrier per k-tile.  The
// epilogue stages each 16-row half of a wavefront's 32-row slab through LDS
// (fp32) so that bias / activation operands are read and the results written
// as 16-byte row segments.
// ---------------------------------------------------------------------------
// (A deeper ring of k-tiles of 32 was measured slower: twice the barriers per
// k, and the loads are not the limit at this depth.)
template <int BM, int BN>
struct TileCfg {
  static constexpr int BK = 64;
  static constexpr int NS = 2;
  // 8 wavefronts, two per SIMD: while one waits on loads, a barrier or its
  // epilogue, the other's MFMAs keep the matrix core busy.
  static constexpr int WAVES = 8;
  static constexpr int WGN = WAVES / 2;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int WM = BM / 2, WN = BN / WGN;
  static constexpr int TM = WM / 32, TN = WN / 32;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  // Epilogue staging, beside the ring: 16 rows x WN fp32 per wavefront.
  static constexpr int EPI_BYTES = WAVES * 16 * WN * 4;
  static constexpr int LDS_BYTES = NS * STAGE_BYTES + EPI_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
  static_assert(A_BYTES % (1024 * WAVES) == 0 && B_BYTES % (1024 * WAVES) == 0,
                "whole 1 KB blocks per wavefront");
};

// One output tile's operands: buffer resources and k-tile range.
struct TileOps {
  __amdgpu_buffer_rsrc_t rsA, rsB;
  int kA0, kB0;     // first k of the range, relative to each resource
  int ntiles;       // k-tiles
  int m0, n0, zs;
};

// Operands of output tile (tm, tn) over k in [kbeg, kend), partial slot zs.
template <int BM, int BN, bool AK, bool BKM>
__device__ __forceinline__ TileOps tile_ops_at(const GemmArgs& g, int zs, int tm, int tn,
                                               int kbeg, int kend) {
  TileOps o;
  o.zs = zs;
  o.m0 = tm * BM;
  o.n0 = tn * BN;
  const bf16_t* A = (const bf16_t*)g.A;
  const bf16_t* B = (const bf16_t*)g.B;
  constexpr int BK = TileCfg<BM, BN>::BK;
  o.ntiles = (kend - kbeg + BK - 1) / BK;
  // k-major: from the tile's first row to the operand's last row (rows past
  // it read 0; K is a multiple of 64).  m/n-major: from the range's first
  // k-row and the tile's first column to the end of the operand (k-rows past
  // K read 0; reads past the valid columns of a row only feed output rows /
  // columns that are never stored).
  if constexpr (AK) {
    o.rsA = make_rsrc(A + (int64_t)o.m0 * g.lda, (int64_t)(g.M - o.m0) * g.lda * 2);
    o.kA0 = kbeg;
  } else {
    o.rsA = make_rsrc(A + (int64_t)kbeg * g.lda + o.m0, ((int64_t)(g.K - kbeg) * g.lda - o.m0) * 2);
    o.kA0 = 0;
  }
  if constexpr (BKM) {
    o.rsB = make_rsrc(B + (int64_t)o.n0 * g.ldb, (int64_t)(g.N - o.n0) * g.ldb * 2);
    o.kB0 = kbeg;
  } else {
    o.rsB = make_rsrc(B + (int64_t)kbeg * g.ldb + o.n0, ((int64_t)(g.K - kbeg) * g.ldb - o.n0) * 2);
    o.kB0 = 0;
  }
  return o;
}

template <int BM, int BN, bool AK, bool BKM>
__device__ __forceinline__ TileOps tile_ops(const GemmArgs& g, int vt, int total, int nbm, int nbn) {
  int tm, tn;
  decode_tile(vt, total, nbm, nbn, tm, tn);
  return tile_ops_at<BM, BN, AK, BKM>(g, 0, tm, tn, 0, g.K);
}

// k-tile t of an output tile -> ring slot t % NS.
template <int BM, int BN, bool AK, bool BKM>
__device__ __forceinline__ void issue_ktile(const GemmArgs& g, const TileOps& T, int t, char* smem,
                                            int wave, int lane) {
  using C = TileCfg<BM, BN>;
  char* b = smem + (t % C::NS) * C::STAGE_BYTES;
  dma_tile<BM, AK, C::BK, C::WAVES>(T.rsA, g.lda, T.kA0 + t * C::BK, b, wave, lane);
  dma_tile<BN, BKM, C::BK, C::WAVES>(T.rsB, g.ldb, T.kB0 + t * C::BK, b + C::A_BYTES, wave, lane);
}

// Group launch (stream-K).  Range r of the G work-groups covers k-tiles
// [sk_begin(r), sk_begin(r + 1)) of the group's W k-tiles (tiles end to end,
// each tile's K in k-tiles); work-group w takes range (w % 8) G / 8 + w / 8,
// so each XCD (work-groups are dealt round robin over the 8 XCDs; the grid
// is a multiple of 8) works on a contiguous eighth of the tiles.
__host__ __device__ __forceinline__ int64_t sk_begin(int64_t r, int64_t work, int G) {
  return r * work / G;
}
// The range that holds k-tile x: the largest r with sk_begin(r) <= x (never
// an empty range).
__host__ __device__ __forceinline__ int sk_range(int64_t x, int64_t work, int G) {
  return (int)(((x + 1) * G + work - 1) / work - 1);
}
// The two-phase sequence: tile t's first-phase segment (kf k-tiles) starts
// at t kf, its second-phase segment (kt - kf) at nt kf + t (kt - kf).
struct SkSeq {
  int64_t work;
  int nt, kt, kf, G;
};
// Sequence position x -> tile t, k-tile k0 within the tile, k-tiles left in
// the segment.
__host__ __device__ __forceinline__ void sk_locate(const SkSeq& q, int64_t x, int& t, int& k0,
                                                   int& left) {
  const int64_t p1 = (int64_t)q.nt * q.kf;
  if (x < p1) {
    t = (int)(x / q.kf);
    k0 = (int)(x - (int64_t)t * q.kf);
    left = q.kf - k0;
  } else {
    const int k2 = q.kt - q.kf;
    const int64_t y = x - p1;
    t = (int)(y / k2);
    const int o = (int)(y - (int64_t)t * k2);
    k0 = q.kf + o;
    left = k2 - o;
  }
}
// Ranges over tile t's segments: the first phase's [a1, a1 + n1) and the
// second's [a2, a2 + n2) (n2 = 0 without a second phase); the slot of the
// piece of range r is r - a1, or n1 + r - a2.
__host__ __device__ __forceinline__ void sk_tile_ranges(const SkSeq& q, int t, int& a1, int& n1,
                                                        int& a2, int& n2) {
  const int64_t s1 = (int64_t)t * q.kf;
  a1 = sk_range(s1, q.work, q.G);
  n1 = sk_range(s1 + q.kf - 1, q.work, q.G) - a1 + 1;
  if (q.kf < q.kt) {
    const int64_t s2 = (int64_t)q.nt * q.kf + (int64_t)t * (q.kt - q.kf);
    a2 = sk_range(s2, q.work, q.G);
    n2 = sk_range(s2 + (q.kt - q.kf) - 1, q.work, q.G) - a2 + 1;
  } else {
    a2 = n2 = 0;
  }
}

// Position of tile (tm, tn) in a problem's tile order (the inverse of
// decode_tile, without the XCD remap).
__host__ __device__ __forceinline__ int tile_pos(int tm, int tn, int nbm, int nbn) {
  const int group = tm / TILE_GM, first_m = group * TILE_GM;
  const int gsize = min(nbm - first_m, TILE_GM);
  return group * TILE_GM * nbn + tn * gsize + (tm - first_m);
}

// The group table is read in place from the kernel-argument segment (a
// by-value argument indexed by a run-time problem number would be copied
// to scratch memory first).
typedef const __attribute__((address_space(4))) GemmGroup kgroup_t;
__device__ __forceinline__ kgroup_t* group_table() {
  return (kgroup_t*)__builtin_amdgcn_kernarg_segment_ptr();
}

// What a weight gradient uses of problem p's arguments.
__device__ __forceinline__ void group_args(kgroup_t* gg, int p, GemmArgs& g) {
  const __attribute__((address_space(4))) GemmArgs* a = &gg->g[p];
  g.A = a->A;
  g.B = a->B;
  g.C = a->C;
  g.M = a->M;
  g.N = a->N;
  g.K = a->K;
  g.lda = a->lda;
  g.ldb = a->ldb;
  g.ldc = a->ldc;
}

// Persistent kernel: each work-group walks output tiles vt = blockIdx.x,
// + gridDim.x, ... (GROUP: the pieces of its stream-K range, see sk_begin).
// The first NS k-tiles of the next output tile are loaded while the current
// tile's epilogue runs.
template <int BM, int BN, bool AK, bool BKM, int EPI, bool GROUP = false>
__global__ __launch_bounds__((TileCfg<BM, BN>::THREADS), 1) void gemm_bf16_kernel(
    typename std::conditional<GROUP, GemmGroup, GemmArgs>::type ka) {
  using C = TileCfg<BM, BN>;
  constexpr int TM = C::TM, TN = C::TN, NS = C::NS;
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS_BYTES];

  GemmArgs g;
  int nbm, nbn, total, vt;
  TileOps T;
  // GROUP: this work-group's stream-K range [kb, ke) and the length of the
  // piece being computed.
  int64_t kb = 0, ke = 0;
  int plen = 0;
  const int G = gridDim.x;
  const int rg = (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3);
  // The piece of the range that starts at k-tile kb: its problem, tile,
  // k range and partial slot.
  auto piece = [&]() {
    kgroup_t* gt = group_table();
    const SkSeq sq = {gt->work, gt->tile0[GEMM_GROUP_MAX], gt->kt, gt->kf, G};
    int t, k0, left;
    sk_locate(sq, kb, t, k0, left);
    plen = (int)min<int64_t>(ke - kb, left);
    int q = 0;
#pragma unroll
    for (int qq = 1; qq < GEMM_GROUP_MAX; ++qq)
      if (qq < gt->n && t >= gt->tile0[qq]) q = qq;
    group_args(gt, q, g);
    nbm = (g.M + BM - 1) / BM;
    nbn = (g.N + BN - 1) / BN;
    int tm, tn;
    decode_tile(t - gt->tile0[q], nbm * nbn, nbm, nbn, tm, tn, false);
    int a1, n1, a2, n2;
    sk_tile_ranges(sq, t, a1, n1, a2, n2);
    const int slot = k0 < gt->kf ? rg - a1 : n1 + rg - a2;
    T = tile_ops_at<BM, BN, AK, BKM>(g, slot, tm, tn, k0 * C::BK,
                                     min(g.K, (k0 + plen) * C::BK));
  };
  if constexpr (GROUP) {
    kgroup_t* gt = group_table();
    kb = sk_begin(rg, gt->work, G);
    ke = sk_begin(rg + 1, gt->work, G);
    if (kb >= ke) return;
    piece();
    vt = 0;
    total = 0;
  } else {
    g = ka;
    vt = blockIdx.x;
    nbm = (g.M + BM - 1) / BM;
    nbn = (g.N + BN - 1) / BN;
    total = nbm * nbn;
    if (vt >= total) return;
    T = tile_ops<BM, BN, AK, BKM>(g, vt, total, nbm, nbn);
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: LDS DMA targets in SGPRs
  const int wm = wave / C::WGN, wn = wave % C::WGN;
  const int hf = lane >> 5, rr = lane & 31;
  constexpr int KS = C::BK / 16;
  // Transposing fragment reads (an m/n-major operand): issued as inline
  // assembly, waited for explicitly.
  constexpr bool TR = !AK || !BKM;

  // First k-tiles of the first output tile.
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < T.ntiles) issue_ktile<BM, BN, AK, BKM>(g, T, t, smem, wave, lane);

  for (;;) {
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    const int ntiles = T.ntiles;

    // The first k-tiles are in flight (issued before the previous epilogue
    // or above); wait for everything outstanding, then read k-tile 0.
    using PA = FragPtrs<BM, AK, C::BK, TM>;
    using PB = FragPtrs<BN, BKM, C::BK, TN>;
    typename PA::Frag af[2][TM];
    typename PB::Frag bfr[2][TN];
    PA pa;
    PB pb;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char_t*)smem;
    pa.init(lds0, wm * C::WM, lane);
    pb.init(lds0 + C::A_BYTES, wn * C::WN, lane);
    // Bias of the lane's 8 epilogue columns (the same for all its chunks),
    // loaded once per tile ahead of the wait below: a load in the epilogue
    // would be waited for behind every store issued before it (loads and
    // stores share one counter, so the wait has to drain both).
    constexpr int ECH = C::WN / 8;  // 8-column chunks per staged row
    static_assert(64 % ECH == 0, "a lane's chunks share their columns");
    constexpr bool BIAS = EPI == EPI_STORE || EPI == EPI_GELU;
    f32x4_t bias0 = {0, 0, 0, 0}, bias1 = {0, 0, 0, 0};
    if (BIAS && g.bias) {
      const int bn = T.n0 + wn * C::WN + (lane % ECH) * 8;
      if (bn < g.N) {
        bias0 = *(const f32x4_t*)(g.bias + bn);
        bias1 = *(const f32x4_t*)(g.bias + bn + 4);
      }
    }
    wait_vm_lgkm0<0>();
    __syncthreads();
    if (ntiles > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[0][i] = pa.template get<0>(i);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[0][j] = pb.template get<0>(j);
    }
    // Main loop.  While the MFMAs of k-step ks run, the fragments of ks + 1
    // are read; in the last k-step of a k-tile they come from the next
    // k-tile instead: wait for this wavefront's loads of k-tile t + 1 and
    // its reads of k-tile t, barrier (every wavefront's k-tile t + 1 has
    // landed and nobody reads k-tile t's slot any more), refill that slot
    // with k-tile t + NS, then read.
    //
    // Only the first half of the wavefronts (0 .. WAVES/2 - 1)
    // request their part of k-tile t + NS right after that barrier; the
    // other half request theirs at the start of k-tile t + 1.  Issuing the
    // direct-to-LDS loads stalls a wavefront until the CU's address unit
    // takes them (64 KB per k-tile), and wavefronts w and
    // w + 4 share a SIMD: split this way, one of each pair issues MFMAs
    // while the other issues its loads, instead of both stalling at once.
    // The slot is free for both halves: its last reads (k-tile t) completed
    // before the barrier.  Before the wait at the end of any k-tile both
    // halves have requested the same k-tiles, so that wait is unchanged.
    // Measured (same box): encoder GEMM set -3.9%, weight-gradient group -5%,
    // 8192^3 -3%; splitting the pairs the other way (even / odd wavefronts) or
    // each wavefront's own loads in two gave -0.3% to -1.6%; requesting the
    // second half one or two k-steps later was slower than not splitting.
    for (int t = 0; t < ntiles; ++t) {
      static_for<0, KS>([&](auto ksc) {
        constexpr int ks = decltype(ksc)::value;
        constexpr int cur = ks & 1, nxt = cur ^ 1;
        if constexpr (ks == 0) {
          if (wave >= C::WAVES / 2 && t >= 1 && t - 1 + NS < ntiles)
            issue_ktile<BM, BN, AK, BKM>(g, T, t - 1 + NS, smem, wave, lane);
        }
        if constexpr (TR) {
          // This k-step's fragments (read during the previous one) have
          // landed; the transposing reads are not tracked by the compiler.
          lds_wait();
#pragma unroll
          for (int i = 0; i < TM; ++i) frag_hold(af[cur][i]);
#pragma unroll
          for (int j = 0; j < TN; ++j) frag_hold(bfr[cur][j]);
        }
        if (ks + 1 < KS) {
          if constexpr (TR) {
            // Interleaved below, with the MFMAs.
          } else {
#pragma unroll
          for (int i = 0; i < TM; ++i) af[nxt][i] = pa.template get<(ks + 1) % KS>(i);
#pragma unroll
          for (int j = 0; j < TN; ++j) bfr[nxt][j] = pb.template get<(ks + 1) % KS>(j);
          }
        } else {
          // Unconditional (also for the last k-tile, whose "next" fragments
          // are never used): a branch here would make the compiler wait for
          // these reads before the last k-step's MFMAs.
          wait_vm_lgkm0<0>();
          __syncthreads();
          if (t + NS < ntiles && wave < C::WAVES / 2)
            issue_ktile<BM, BN, AK, BKM>(g, T, t + NS, smem, wave, lane);
          // move the fragment pointers to the next ring slot
          const int delta = ((t + 1) % NS == 0) ? -(NS - 1) * C::STAGE_BYTES : C::STAGE_BYTES;
          pa.advance(delta);
          pb.advance(delta);
          if constexpr (!TR) {
#pragma unroll
            for (int i = 0; i < TM; ++i) af[nxt][i] = pa.template get<0>(i);
#pragma unroll
            for (int j = 0; j < TN; ++j) bfr[nxt][j] = pb.template get<0>(j);
          }
        }
        if constexpr (TR) {
          // One MFMA, then its share of the next k-step's fragment reads
          // (from the next k-tile after the last k-step), in this order:
          // each read issues while the matrix core works on the MFMA
          // before it.
          constexpr int NM = TM * TN, NF = TM + TN;
          constexpr int kn = ks + 1 < KS ? ks + 1 : 0;
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            acc[m / TN][m % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                frag_val(af[cur][m / TN]), frag_val(bfr[cur][m % TN]), acc[m / TN][m % TN], 0, 0, 0);
#pragma unroll
            for (int f = 0; f < NF; ++f)
              if ((f * NM) / NF == m) {
                if (f < TM) af[nxt][f] = pa.template get<kn>(f);
                else bfr[nxt][f - TM] = pb.template get<kn>(f - TM);
              }
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[cur][i], bfr[cur][j],
                                                                acc[i][j], 0, 0, 0);
        // Issue order: one MFMA, then the next k-step's fragment reads
        // spread evenly behind the MFMAs (each read issues while the
        // matrix core works on the MFMA before it) instead of all reads
        // ahead of the MFMAs.  Measured: -3% over the encoder GEMMs, -6%
        // for the weight gradients (two reads per fragment).
        {
          constexpr int NM = TM * TN;
          constexpr int NR = TM * (AK ? 1 : 2) + TN * (BKM ? 1 : 2);
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, (NR + NM - 1) / NM, 0);  // LDS read
          }
        }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    if constexpr (TR) {
      // The last k-step's reads of the "next" fragments (never used) must
      // land before their registers are reused.
      lds_wait();
#pragma unroll
      for (int i = 0; i < TM; ++i) frag_hold(af[0][i]), frag_hold(af[1][i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) frag_hold(bfr[0][j]), frag_hold(bfr[1][j]);
    }

    // Every wavefront has read its last fragments: the whole ring is free.
    // Start the next output tile's first NS k-tiles, then run this tile's
    // epilogue (its staging area is separate from the ring).
    __syncthreads();
    const int m0 = T.m0, n0 = T.n0, zs = T.zs;
    const GemmArgs ge = g;  // this tile's problem (g moves on to the next tile's)
    const int mw = m0 + wm * C::WM, nw = n0 + wn * C::WN;
    constexpr int CH = C::WN / 8;  // 8-column chunks per staged row
    constexpr int QN = 16 * CH / 64;  // chunks per lane per staged 16-row half
    // EPI_MUL reads one bf16 operand chunk per output chunk; the
    // chunks of the next staged half are loaded while this one is processed
    // (the first ones before the next tile's k-tiles are requested).
    constexpr bool AUX = EPI == EPI_MUL;
    u32x4_t axv[2][QN];
    auto aux_load = [&](int it, u32x4_t* dst) {
#pragma unroll
      for (int q = 0; q < QN; ++q) {
        const int c = lane + 64 * q;
        const int row = c / CH, col = (c % CH) * 8;
        const int m = mw + (it >> 1) * 32 + 16 * (it & 1) + row, n = nw + col;
        dst[q] = (m < ge.M && n < ge.N)
                     ? *(const u32x4_t*)((const bf16_t*)ge.aux + (int64_t)m * ge.ldaux + n)
                     : u32x4_t{0, 0, 0, 0};
      }
    };
    if constexpr (AUX) aux_load(0, axv[0]);
    bool more;
    if constexpr (GROUP) {
      kb += plen;
      more = kb < ke;
      if (more) piece();
    } else {
      vt += gridDim.x;
      more = vt < total;
      if (more) T = tile_ops<BM, BN, AK, BKM>(g, vt, total, nbm, nbn);
    }
    auto issue_next = [&]() {
      if (more) {
#pragma unroll
        for (int t = 0; t < NS; ++t)
          if (t < T.ntiles) issue_ktile<BM, BN, AK, BKM>(g, T, t, smem, wave, lane);
      }
    };
    // EPI_MUL reads an operand per output chunk.  Loads and stores share one
    // counter, so a load waited for after stores drains the stores too: this
    // epilogue computes every chunk first (results packed into the registers
    // the consumed accumulators free), then requests the next tile's k-tiles
    // and stores.  The others request the
    // k-tiles first and store as they go.
    if constexpr (!AUX) issue_next();
    u32x4_t res[AUX ? 2 * TM : 1][QN];

    // Epilogue.  32x32 accumulator layout: lane holds column (lane % 32);
    // register r holds row 8 * (r / 4) + 4 * (lane / 32) + (r % 4).  Each
    // 16-row half (registers 0-7, 8-15) of a 32-row slab is staged through
    // the wavefront's LDS area as fp32; columns are XOR-swizzled by 32 on
    // rows 4-7 / 12-15 so the two lane halves' stores hit different banks.
    float* stg = (float*)(smem + NS * C::STAGE_BYTES) + wave * 16 * C::WN;
    // Column sums (EPI_MUL): every lane keeps one 8-column chunk (CH divides
    // 64) over the rows it writes.
    static_assert(64 % CH == 0 && C::WM == 128, "column sums per 128 rows");
    float csum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (EPI == EPI_PARTIAL) {
      // fp32 results straight from the accumulators, no LDS round trip: for
      // each register, lanes 0-31 and 32-63 write 32 consecutive columns of
      // two rows, whole 128-byte lines.
      float* Cp = (float*)ge.C + (int64_t)zs * ge.M * ge.ldc;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int n = nw + j * 32 + rr;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m = mw + i * 32 + 8 * (r >> 2) + 4 * hf + (r & 3);
            if (m < ge.M && n < ge.N) Cp[(int64_t)m * ge.ldc + n] = acc[i][j][r];
          }
        }
    } else {
  #pragma unroll
      for (int i = 0; i < TM; ++i) {
  #pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int it = 2 * i + half;
          if constexpr (AUX) {
            if (it + 1 < 2 * TM) aux_load(it + 1, axv[(it + 1) & 1]);
          }
  #pragma unroll
          for (int j = 0; j < TN; ++j)
  #pragma unroll
            for (int r = 8 * half; r < 8 * half + 8; ++r) {
              const int row = 8 * ((r >> 2) & 1) + 4 * hf + (r & 3);  // 0..15
              const int col = (j * 32 + rr) ^ (hf * 32);
              stg[row * C::WN + col] = acc[i][j][r];
            }
          __builtin_amdgcn_wave_barrier();
  #pragma unroll
          for (int q = 0; q < QN; ++q) {
            const int c = lane + 64 * q;
            const int row = c / CH, col = (c % CH) * 8;
            const int pcol = col ^ (((row >> 2) & 1) * 32);
            const int m = mw + i * 32 + 16 * half + row, n = nw + col;
            float v[8];
            const f32x4_t x0 = *(const f32x4_t*)(stg + row * C::WN + pcol);
            const f32x4_t x1 = *(const f32x4_t*)(stg + row * C::WN + pcol + 4);
  #pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] = x0[e];
              v[4 + e] = x1[e];
            }
            if constexpr (AUX) {
              res[it][q] = mul8(v, axv[it & 1][q]);
              // keep the packed result here (not recomputed from fp32 values
              // held until the stores)
              asm volatile("" : "+v"(res[it][q]));
              if (m < ge.M && n < ge.N) {
  #pragma unroll
                for (int e = 0; e < 8; ++e) csum[e] += v[e];
              }
            } else if (m < ge.M && n < ge.N) {
              epi8<EPI>(ge, zs, m, n, v, bias0, bias1);
            }
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
    if constexpr (AUX) {
      issue_next();
#pragma unroll
      for (int it = 0; it < 2 * TM; ++it)
#pragma unroll
        for (int q = 0; q < QN; ++q) {
          const int c = lane + 64 * q;
          const int row = c / CH, col = (c % CH) * 8;
          const int m = mw + (it >> 1) * 32 + 16 * (it & 1) + row, n = nw + col;
          if (m < ge.M && n < ge.N)
            *(u32x4_t*)((bf16_t*)ge.C + (int64_t)m * ge.ldc + n) = res[it][q];
        }
    }
    if (AUX && ge.colpart) {
      // lanes l, l ^ 16, l ^ 32, l ^ 48 hold the same columns: fixed-order sum
#pragma unroll
      for (int e = 0; e < 8; ++e) {
#pragma unroll
        for (int o = CH; o < 64; o <<= 1) csum[e] += __shfl_xor(csum[e], o, 64);
      }
      const int n = nw + (lane % CH) * 8;
      // colpart has ceil(M / 128) rows: the last tile's second 128-row slab
      // lies past them when their number is odd
      if (lane < CH && n < ge.N && mw < ge.M) {
        float* P = ge.colpart + (int64_t)(mw / C::WM) * ge.N + n;
        *(f32x4_t*)P = f32x4_t{csum[0], csum[1], csum[2], csum[3]};
        *(f32x4_t*)(P + 4) = f32x4_t{csum[4], csum[5], csum[6], csum[7]};
      }
    }
    if (!more) break;
  }
}

// wgrad_group_reduce: block b serves problem q with blk0[q] <= b <
// blk0[q + 1]; each thread sums 4 consecutive elements of one tile over the
// tile's pieces (slots) in k order.
struct SkReduce {
  const float* part[GEMM_GROUP_MAX];
  float* out[GEMM_GROUP_MAX];
  int M[GEMM_GROUP_MAX], N[GEMM_GROUP_MAX];
  int blk0[GEMM_GROUP_MAX + 1];
  int tile0[GEMM_GROUP_MAX];
  int n;
  SkSeq seq;
  TailJobs tail;  // four units per work-group, after the split-K blocks
};

__global__ __launch_bounds__(256, 8) void wgrad_group_reduce_kernel(SkReduce rd) {
  const int b = blockIdx.x;
  if (b >= rd.blk0[GEMM_GROUP_MAX]) {
    tail_unit<4>(tail_arg(offsetof(SkReduce, tail)), (b - rd.blk0[GEMM_GROUP_MAX]) * 4 + (int)(threadIdx.x >> 6), threadIdx.x & 63);
    return;
  }
  int q = 0;
#pragma unroll
  for (int k = 1; k < GEMM_GROUP_MAX; ++k)
    if (k < rd.n && b >= rd.blk0[k]) q = k;
  const float* part;
  float* out;
  int M, N, b0, t0;
  switch (q) {
    case 0: part = rd.part[0]; out = rd.out[0]; M = rd.M[0]; N = rd.N[0]; b0 = rd.blk0[0]; t0 = rd.tile0[0]; break;
    case 1: part = rd.part[1]; out = rd.out[1]; M = rd.M[1]; N = rd.N[1]; b0 = rd.blk0[1]; t0 = rd.tile0[1]; break;
    case 2: part = rd.part[2]; out = rd.out[2]; M = rd.M[2]; N = rd.N[2]; b0 = rd.blk0[2]; t0 = rd.tile0[2]; break;
    default: part = rd.part[3]; out = rd.out[3]; M = rd.M[3]; N = rd.N[3]; b0 = rd.blk0[3]; t0 = rd.tile0[3]; break;
  }
  const int64_t mn = (int64_t)M * N;
  const int64_t i = ((int64_t)(b - b0) * blockDim.x + threadIdx.x) * 4;
  if (i >= mn) return;
  const int m = (int)(i / N), n = (int)(i - (int64_t)m * N);  // N % 4 == 0: one tile
  const int nbm = (M + 255) / 256, nbn = (N + 255) / 256;
  const int t = t0 + tile_pos(m / 256, n / 256, nbm, nbn);
  const SkSeq sq = rd.seq;
  int a1, n1, a2, n2;
  sk_tile_ranges(sq, t, a1, n1, a2, n2);
  // slot 0 (range a1 holds the tile's first k-tile) is always written; an
  // empty range wrote no slot
  f32x4_t s = *(const f32x4_t*)(part + i);
  for (int j = 1; j < n1 + n2; ++j) {
    const int r = j < n1 ? a1 + j : a2 + j - n1;
    if (sk_begin(r, sq.work, sq.G) < sk_begin(r + 1, sq.work, sq.G))
      s += *(const f32x4_t*)(part + (int64_t)j * mn + i);
  }
  *(f32x4_t*)(out + i) = s;
}

}  // namespace

int device_cus() {
  static const int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    return n;
  }();
  return cus;
}

namespace {

template <bool AK, bool BKM, int EPI>
hipError_t launch_256(const GemmArgs& g, hipStream_t st) {
  const int64_t total = (int64_t)((g.M + 255) / 256) * ((g.N + 255) / 256);
  // One work-group per CU (LDS and registers allow no more); a multiple of
  // 8 so that each work-group stays on one XCD's share of the tiles.
  int64_t grid = std::min<int64_t>(total, device_cus());
  if (grid >= 8) grid -= grid % 8;
  hipLaunchKernelGGL((gemm_bf16_kernel<256, 256, AK, BKM, EPI>), dim3((unsigned)grid),
                     dim3(TileCfg<256, 256>::THREADS), 0, st, g);
  return hipGetLastError();
}

}  // namespace

bool gemm_bf16_ok(const GemmArgs& g, bool b_kmajor) {
  // Vector epilogue and n-major staging work in 8-column units; k-tiles of
  // 64 never straddle a split boundary, and k-major operands are read
  // without a k bound.
  if (g.N % 8 != 0 || g.ldc % 8 != 0 || g.K % 64 != 0 || g.lda % 8 != 0 || g.ldb % 8 != 0)
    return false;
  // Operands are read through buffer resources with 32-bit byte extents and
  // offsets: each operand must span less than 2 GiB.
  return (int64_t)g.M * g.lda * 2 < ((int64_t)1 << 31) &&
         (int64_t)(b_kmajor ? g.N : g.K) * g.ldb * 2 < ((int64_t)1 << 31);
}

hipError_t gemm_bf16(const GemmArgs& g0, bool b_kmajor, GemmEpi epi, hipStream_t st) {
  GemmArgs g = g0;
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (!gemm_bf16_ok(g, b_kmajor)) return hipErrorInvalidValue;
  if (g.ksplit > 1 && (g.kchunk % 64 != 0 || epi != EPI_PARTIAL)) return hipErrorInvalidValue;
  if (epi == EPI_MUL && !g.colpart) return hipErrorInvalidValue;
  if (epi == EPI_DSUM && (!g.aux || !g.aux2 || !g.dsum || g.dsum_S < 1 || g.M % g.dsum_S != 0 ||
                          g.N % 64 != 0))
    return hipErrorInvalidValue;
  if (g.tile == 0) g.tile = gemm_bf16_plan(g.M, g.N, g.K, b_kmajor, epi, false).tile;
  if (g.tile == GEMM_TILE_256x256 && g.ksplit == 1) {
    if (b_kmajor) {
      if (epi == EPI_STORE) return launch_256<true, true, EPI_STORE>(g, st);
      if (epi == EPI_GELU) return launch_256<true, true, EPI_GELU>(g, st);
      if (epi == EPI_PARTIAL) return launch_256<true, true, EPI_PARTIAL>(g, st);
    } else {
      if (epi == EPI_STORE) return launch_256<true, false, EPI_STORE>(g, st);
      if (epi == EPI_MUL) return launch_256<true, false, EPI_MUL>(g, st);
    }
    return hipErrorInvalidValue;
  }
  return gemm_mid(g, b_kmajor, epi, g.tile, st);
}

namespace {

// Time model of a tile shape, in microseconds: a launch (a), per round of
// work-groups over the CUs its k-tiles (c each) and epilogue (e per 128 x 128
// outputs; twice that for the GELU and GELU' ones), but no less than its
// operand traffic out of L2 (bw, TB/s) plus its output (wb, TB/s).  64 x 64
// work-groups share a CU in pairs, so their rounds are not whole.  Fitted to
// 7700 timed launches (M 40 .. 16384, the products of layers of width 192 ..
// 2048); the tile it picks is on average 1.8% slower than the best one
// measured, and 2.1 times faster than the rule it replaces (tiles of 128 x 128
// and more, no splits, four wavefronts).
struct TileModel {
  int bm, bn;
  double a, c, e, bw, wb;
};
constexpr TileModel TILE_MODEL[] = {
    {256, 256, 5.0, 1.30, 0.94, 9.8, 4.15}, {256, 128, 5.0, 0.75, 0.2, 13.0, 3.65},
    {128, 128, 4.0, 0.327, 0.87, 13.7, 2.9}, {128, 64, 3.0, 0.242, 2.7, 16.6, 1.96},
    {64, 64, 3.1, 0.167, 1.2, 18.7, 3.53}};

double tile_time(int tile, int64_t M, int64_t N, int64_t K, int ks, GemmEpi epi) {
  const TileModel& m = TILE_MODEL[tile - 1];
  const double cus = device_cus();
  const double wg = (double)((M + m.bm - 1) / m.bm) * ((N + m.bn - 1) / m.bn) * ks;
  const double nk = (double)((K / 64 + ks - 1) / ks);
  const double rounds = tile == GEMM_TILE_64x64 ? std::max(1.0, wg / cus) : std::ceil(wg / cus);
  const bool act = epi == EPI_GELU || epi == EPI_MUL;
  const double epil = m.e * (m.bm * m.bn / 16384.0) * (act ? 2.0 : 1.0);
  const double out = (double)M * N * (act || epi == EPI_PARTIAL ? 4 : 2) * ks;
  const double mem = wg * nk * (m.bm + m.bn) * 128.0 / (m.bw * 1e6) + out / (m.wb * 1e6);
  // a consumer that sums partials reads them at about 5 TB/s
  const double extra = (ks - 1) * (double)M * N * 4 / 5e6;
  return m.a + std::max(rounds * (nk * m.c + epil), mem) + extra;
}

}  // namespace

bool wgrad_args_ok(const GemmArgs* p, int n) {
  if (n < 1 || n > GEMM_GROUP_MAX || !p) return false;
  for (int q = 0; q < n; ++q) {
    const GemmArgs& g = p[q];
    // the checks gemm_bf16 makes, for two m/n-major operands; one K for all
    if (g.M < 0 || g.N < 0 || g.K < 1 || g.K != p[0].K) return false;
    if (g.N % 8 != 0 || g.ldc % 8 != 0 || g.M % 8 != 0 || g.lda % 8 != 0 || g.ldb % 8 != 0)
      return false;
    if ((int64_t)g.K * g.lda * 2 >= ((int64_t)1 << 31) ||
        (int64_t)g.K * g.ldb * 2 >= ((int64_t)1 << 31))
      return false;
  }
  return true;
}

GemmPlan gemm_bf16_plan(int M, int N, int K, bool b_kmajor, GemmEpi epi, bool split) {
  const int64_t cus = device_cus();
  const int64_t t1 = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
  const bool act = epi == EPI_GELU || epi == EPI_MUL;
  GemmPlan best = {GEMM_TILE_128x128, 1};
  double tb = 0.0;
  auto consider = [&](int tile, int ks) {
    const double t = tile_time(tile, M, N, K, ks, epi);
    if (tb == 0.0 || t < tb) {
      tb = t;
      best = {tile, ks};
    }
  };
  // 256 x 256 tiles read a quarter as much per product as 64 x 64 ones, but
  // below three quarters of a tile per CU (55% with the long epilogues) the
  // model, fitted over several rounds, does not describe them: idle CUs cost
  // more.
  if (M >= 256 && N >= 256 && (epi != EPI_PARTIAL || b_kmajor) &&
      t1 >= (act ? cus * 11 / 20 : cus * 3 / 4))
    consider(GEMM_TILE_256x256, 1);
  consider(GEMM_TILE_256x128, 1);
  consider(GEMM_TILE_128x128, 1);
  consider(GEMM_TILE_128x64, 1);
  // (column sums of 64-row tiles are only provided for up to 8192 rows)
  if (epi != EPI_MUL || M <= 8192) consider(GEMM_TILE_64x64, 1);
  if (split) {
    for (int ks = 2; ks <= GEMM_SPLIT_MAX; ks += 2) {
      const int chunk = ((K + ks - 1) / ks + 63) / 64 * 64;
      if ((K + chunk - 1) / chunk != ks || (int64_t)ks * M * N > GEMM_SPLIT_ELEMS) continue;
      for (int tile = GEMM_TILE_256x128; tile <= GEMM_TILE_64x64; ++tile) consider(tile, ks);
    }
  }
  return best;
}

int64_t gemm_colpart_max(int64_t M) {
  return std::max((M + 127) / 128, (std::min<int64_t>(M, 8192) + 63) / 64);
}

namespace {

// Grid of a group launch: one work-group per CU, a multiple of 8.
int group_grid() {
  const int cus = device_cus();
  return std::max(8, cus - cus % 8);
}

// First-phase k-tiles per tile: the average range, when shorter than a tile.
int first_phase(int64_t tiles, int kt) {
  const int64_t w = tiles * kt / group_grid();
  return (int)std::max<int64_t>(1, std::min<int64_t>(kt, w));
}

// The k-tile sequence of a group launch of `tiles` tiles.
SkSeq group_seq(int64_t tiles, int K) {
  const int kt = (K + 63) / 64;
  return {tiles * kt, (int)tiles, kt, first_phase(tiles, kt), group_grid()};
}

// The stream-K table of a group; false for invalid problems.
bool group_table_of(const GemmArgs* p, int n, GemmGroup& gg) {
  if (!wgrad_args_ok(p, n)) return false;
  gg = GemmGroup{};
  gg.n = n;
  int64_t tiles = 0;
  for (int q = 0; q < n; ++q) {
    const GemmArgs& g = p[q];
    gg.g[q] = g;
    gg.tile0[q] = (int)tiles;
    tiles += (int64_t)((g.M + 255) / 256) * ((g.N + 255) / 256);
    if (tiles >= ((int64_t)1 << 24)) return false;
  }
  gg.tile0[n] = (int)tiles;
  for (int q = n + 1; q <= GEMM_GROUP_MAX; ++q) gg.tile0[q] = (int)tiles;
  gg.kt = (p[0].K + 63) / 64;
  gg.work = tiles * gg.kt;
  gg.kf = first_phase(tiles, gg.kt);
  return true;
}

}  // namespace

// The stream-K group against whole gradients per work-group (gemm_mid.hip).
// The group's k-tiles of 256 x 256 run at twice the rate per byte read, but it
// writes about 256 + tiles partials of 256 KB and reads them back (50-60 us at
// width 1024, whatever the token count), and with few tokens most of its
// work-groups have almost no k-tiles.  The model's figures are fitted to timed
// groups of width 192 .. 2048 and 40 .. 16384 tokens; on average its choice is
// 0.8% slower than the best one.  Width 768: 2048 tokens 84 -> 37 us, 16384
// tokens 276 -> 237 us; width 1024 (1.5 rounds of 256 x 128 tiles): 4096 tokens
// 132 -> 117 us, 16384 tokens 382 us against 428 us (the group stays).
int wgrad_plan(const int* M, const int* N, int n, int K) {
  const double cus = device_cus(), kt = (K + 63) / 64;
  double area = 0, t256 = 0, t2 = 0, t128 = 0, t64 = 0;
  auto cd = [](int a, int b) { return (double)((a + b - 1) / b); };
  for (int q = 0; q < n; ++q) {
    area += (double)M[q] * N[q];
    t256 += cd(M[q], 256) * cd(N[q], 256);
    t2 += cd(M[q], 256) * cd(N[q], 128);
    t128 += cd(M[q], 128) * cd(N[q], 128);
    t64 += cd(M[q], 64) * cd(N[q], 64);
  }
  const bool whole = t256 / cus == std::floor(t256 / cus);
  const double pieces = whole ? t256 : std::max(t256, cus) + t256;
  const double group = 25 + t256 * kt / cus * 1.8 + (pieces * 262144 * 2 + area * 4) / 8e6;
  auto mid = [&](double wg, double rounds, double a, double c, double e, double kbytes, double bw,
                 double wb) {
    return a + std::max(rounds * (kt * c + e), wg * kt * kbytes / (bw * 1e6) + area * 4 / (wb * 1e6));
  };
  const double m2 = mid(t2, std::ceil(t2 / cus), 5.9, 0.59, 0.14, 49152, 12.9, 4.3);
  const double m128 = mid(t128, std::ceil(t128 / cus), 4.6, 0.36, 0.48, 32768, 14.5, 3.6);
  const double m64 = mid(t64, std::max(1.0, t64 / cus), 3.3, 0.24, 0.0, 16384, 25.0, 3.1);
  // (beyond 8192 tokens the operands of tiles that are far apart no longer
  // meet in the caches and the models of whole gradients are too fast, unless
  // the 256 x 128 tiles are one round: width 512, 16384 tokens 145 us with the
  // group against 159 us)
  if (K > 8192 && !(t2 <= cus && m2 < group && t2 > 0.75 * cus)) return 0;
  if (group < m2 && group < m128 && group < m64) return 0;
  return m2 <= m128 && m2 <= m64 ? GEMM_TILE_256x128 : m128 <= m64 ? GEMM_TILE_128x128 : GEMM_TILE_64x64;
}

int wgrad_group_slots(const int* M, const int* N, int n, int K) {
  if (n < 1 || n > GEMM_GROUP_MAX || K < 1) return -1;
  int64_t tiles = 0;
  for (int q = 0; q < n; ++q) {
    if (M[q] < 0 || N[q] < 0) return -1;
    tiles += (int64_t)((M[q] + 255) / 256) * ((N[q] + 255) / 256);
  }
  if (tiles == 0 || wgrad_plan(M, N, n, K) != 0) return 0;
  const SkSeq sq = group_seq(tiles, K);
  int slots = 1;
  for (int t = 0; t < (int)tiles; ++t) {
    int a1, n1, a2, n2;
    sk_tile_ranges(sq, t, a1, n1, a2, n2);
    slots = std::max(slots, n1 + n2);
  }
  return slots;
}

hipError_t gemm_bf16_wgrad_group(const GemmArgs* p, int n, hipStream_t st) {
  GemmGroup gg;
  if (!group_table_of(p, n, gg)) return hipErrorInvalidValue;
  if (gg.work == 0) return hipSuccess;
  hipLaunchKernelGGL((gemm_bf16_kernel<256, 256, false, false, EPI_PARTIAL, true>),
                     dim3((unsigned)group_grid()), dim3(TileCfg<256, 256>::THREADS),
                     0, st, gg);
  return hipGetLastError();
}

hipError_t wgrad_group_reduce(const GemmArgs* p, float* const* out, int n, const TailJobs& tail,
                              hipStream_t st) {
  GemmGroup gg{};
  SkReduce rd{};
  rd.tail = tail;
  if (!group_table_of(p, n, gg) || !out || !tail_prepare(rd.tail)) return hipErrorInvalidValue;
  rd.n = n;
  rd.seq = {gg.work, gg.tile0[n], gg.kt, gg.kf, group_grid()};
  int64_t blocks = 0;
  for (int q = 0; q < n; ++q) {
    if (p[q].ldc != p[q].N) return hipErrorInvalidValue;  // partial slots are dense M x N
    rd.part[q] = (const float*)p[q].C;
    rd.out[q] = out[q];
    rd.M[q] = p[q].M;
    rd.N[q] = p[q].N;
    rd.tile0[q] = gg.tile0[q];
    rd.blk0[q] = (int)blocks;
    blocks += ((int64_t)p[q].M * p[q].N / 4 + 255) / 256;
    if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  }
  for (int q = n; q <= GEMM_GROUP_MAX; ++q) rd.blk0[q] = (int)blocks;
  blocks += (rd.tail.units + 3) / 4;
  if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(wgrad_group_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, st, rd);
  return hipGetLastError();
}
