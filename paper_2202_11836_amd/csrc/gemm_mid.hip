// bf16 MFMA GEMM for outputs that have too few 256 x 256 tiles to fill the
// chip: all but the largest token counts.  Same operands, LDS layouts and
// epilogues as gemm.hip.
//
// What bounds it.  A CU takes 1 KB of operands per 17 cycles into LDS and
// about 30 bytes per cycle from L2 when all CUs read, and with few tiles most
// CUs idle.  So: small tiles where there are few of them, every load requested
// early, and nothing in the loop that waits for something the loop itself has
// just started.  Every wavefront owns a 64 x 64 block (4 accumulators of
// v_mfma_f32_32x32x16_bf16: each fragment read from LDS feeds two MFMAs), and
// the KG wavefronts that share a block split each k-tile of 64 by k; their
// sums are added through LDS in k order at the end, where the epilogue reads
// rows of 8 columns.  k-tiles come straight from HBM into a ring of NS LDS
// slots; while the MFMAs of k-tile t run, the fragments of k-tile t + 1 are
// read and k-tile t + NS is requested, one read or load between two MFMAs (a
// load stalls its wavefront until the CU's address unit takes it: ahead of the
// MFMAs those stalls took as long as the MFMAs, 0.46 -> 0.38 us per k-tile of
// 128 x 128).  One barrier per k-tile that leaves the later ones in flight.
// Outputs that the next kernel sums anyway (fp32, EPI_PARTIAL) are also split
// over work-groups (ksplit).  Measured against the 4-wavefront kernels this
// replaced, at the products of a BERT-base layer: 231 tokens, FFN2 54 -> 6 us,
// its data gradient 56 -> 6 us, QKV 19 -> 5.5 us; 2048 tokens, FFN1 + GELU 25
// -> 21 us, FFN2 29 -> 17 us.
#include <algorithm>

#include "gemm_tile.h"
#include "tail.h"

namespace {

// KG wavefronts per 64 x 64 block, two resident wavefronts per SIMD (8 per
// work-group, or two work-groups of 4).
template <int BM, int BN>
struct MidCfg {
  static constexpr int BK = 64;
  static constexpr int BLK = (BM / 64) * (BN / 64);
  static constexpr int W = BLK == 1 ? 4 : 8;
  static constexpr int KG = W / BLK;
  static constexpr int KSW = 4 / KG;  // k-steps of 16 per wavefront and k-tile
  static constexpr int THREADS = 64 * W;
  static constexpr int A_BYTES = BM * BK * 2, STAGE = (BM + BN) * BK * 2;
  static constexpr int NS = BLK == 2 ? 5 : BLK == 8 ? 3 : 4;
  static constexpr int EX = KG * BM * BN * 4;  // exchange area of the k sums
  static constexpr int LDS = NS * STAGE > EX ? NS * STAGE : EX;
  static constexpr int PER = STAGE / 1024 / W;  // loads per k-tile and wavefront
  static_assert(PER * (NS - 1) <= 63 && LDS <= 160 * 1024, "");
};

// Wait until at most `after` (0 .. MAX) of the latest k-tiles' loads are
// outstanding (and this wavefront's LDS operations are done).
template <int PER, int MAX>
__device__ __forceinline__ void wait_after(int after) {
  if constexpr (MAX == 0) {
    wait_vm_lgkm0<0>();
  } else {
    if (after >= MAX) wait_vm_lgkm0<PER * MAX>();
    else wait_after<PER, MAX - 1>(after);
  }
}

// Work-group barrier that leaves direct-to-LDS loads in flight.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Work-group -> (split, m tile, n tile).  Consecutive work-groups go round
// robin over the 8 XCDs; each XCD takes a contiguous range, walked in groups
// of 4 tile-rows (tiles that share A rows / B columns meet in one L2).
__device__ __forceinline__ void mid_tile(int bid, int total, int nbm, int nbn, int& zs, int& tm,
                                         int& tn) {
  if ((total & 7) == 0) bid = (bid & 7) * (total >> 3) + (bid >> 3);
  zs = bid / (nbm * nbn);
  const int r0 = bid - zs * nbm * nbn;
  constexpr int GM = 4;
  const int group = r0 / (GM * nbn), first = group * GM, size = min(nbm - first, GM);
  const int r = r0 - group * GM * nbn;
  tm = first + r % size;
  tn = r / size;
}

template <int BM, int BN, bool AK, bool BKM, int EPI>
__device__ __forceinline__ void mid_body(const GemmArgs& g, int zs, int tm, int tn, char* smem) {
  using C = MidCfg<BM, BN>;
  constexpr int NS = C::NS, KG = C::KG, KSW = C::KSW;
  constexpr bool TR = !AK || !BKM;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, rr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / C::BLK, blk = wave % C::BLK;
  const int wm = (blk / (BN / 64)) * 64, wn = (blk % (BN / 64)) * 64;
  const int m0 = tm * BM, n0 = tn * BN;
  const int kbeg = zs * g.kchunk, kend = min(g.K, kbeg + g.kchunk);
  const int nt = (kend - kbeg + C::BK - 1) / C::BK;
  const bf16_t* A = (const bf16_t*)g.A;
  const bf16_t* B = (const bf16_t*)g.B;
  // Resources as in gemm.hip: k-major operands end at their last row,
  // m/n-major ones at k-row kend (a k range that is not the operand's last
  // one ends there too: k ranges are whole k-tiles).
  __amdgpu_buffer_rsrc_t rsA, rsB;
  if constexpr (AK) rsA = make_rsrc(A + (int64_t)m0 * g.lda, (int64_t)(g.M - m0) * g.lda * 2);
  else rsA = make_rsrc(A + (int64_t)kbeg * g.lda + m0, ((int64_t)(kend - kbeg) * g.lda - m0) * 2);
  if constexpr (BKM) rsB = make_rsrc(B + (int64_t)n0 * g.ldb, (int64_t)(g.N - n0) * g.ldb * 2);
  else rsB = make_rsrc(B + (int64_t)kbeg * g.ldb + n0, ((int64_t)(kend - kbeg) * g.ldb - n0) * 2);
  auto issue = [&](int t) {
    char* d = smem + (t % NS) * C::STAGE;
    dma_tile<BM, AK, C::BK, C::W>(rsA, g.lda, (AK ? kbeg : 0) + t * C::BK, d, wave, lane);
    dma_tile<BN, BKM, C::BK, C::W>(rsB, g.ldb, (BKM ? kbeg : 0) + t * C::BK, d + C::A_BYTES, wave, lane);
  };
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < nt) issue(t);

  // Fragment addresses in ring slot 0 of the wavefront's first k-step.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char_t*)smem;
  using PA = FragPtrs<BM, AK, C::BK, 2>;
  using PB = FragPtrs<BN, BKM, C::BK, 2>;
  PA pa;
  PB pb;
  pa.init(lds0, wm, lane);
  pb.init(lds0 + C::A_BYTES, wn, lane);
  // (k-major: one address per k-step, fragment f 32 rows on; m/n-major: one
  // per fragment, k-step s 16 k-rows on)
  uint32_t ua[AK ? KSW : 2], ub[BKM ? KSW : 2];
#pragma unroll
  for (int s = 0; s < KSW; ++s) {
    auto at = [&](uint32_t base, int r) {  // k-major: chunk 2 ks + hf of row r
      return base + r * (2 * C::BK) + 16 * ((2 * (kg * KSW + s) + hf) ^ kswz<C::BK>(r));
    };
    if constexpr (AK) ua[s] = at(lds0, wm + rr);
    if constexpr (BKM) ub[s] = at(lds0 + C::A_BYTES, wn + rr);
  }
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    if constexpr (!AK) ua[f] = pa.p[f] + kg * KSW * 16 * (2 * BM);
    if constexpr (!BKM) ub[f] = pb.p[f] + kg * KSW * 16 * (2 * BN);
  }
  // Fragment f of the wavefront's k-step s; u: an operand's addresses, R its
  // tile's rows.
  auto frag = [&](auto kmaj, auto rows, auto sc, auto fc, const uint32_t* u, uint32_t slot) {
    constexpr int s = decltype(sc)::value, f = decltype(fc)::value, R = decltype(rows)::value;
    if constexpr (decltype(kmaj)::value) {
      return *(const __attribute__((address_space(3))) bf16x8_t*)((lds_char_t*)(uintptr_t)(u[s] + slot) +
                                                                 f * 32 * (2 * C::BK));
    } else {
      const uint32_t at = u[f] + slot;
      return TrFrag{ds_read_tr16_b64<s * 16 * (2 * R)>(at), ds_read_tr16_b64<s * 16 * (2 * R) + 4 * 2 * R>(at)};
    }
  };
  using KA = std::integral_constant<bool, AK>;
  using KB = std::integral_constant<bool, BKM>;
  using RA = std::integral_constant<int, BM>;
  using RB = std::integral_constant<int, BN>;

  // The epilogue's operands, requested ahead of the main loop's waits: a
  // thread's chunks of 8 columns share their columns.
  constexpr int CPR = BN / 8, RPP = C::THREADS / CPR, NCH = BM / RPP;
  const int ec = (tid % CPR) * 8, er = tid / CPR;
  const int n = n0 + ec;
  f32x4_t b0 = {0, 0, 0, 0}, b1 = {0, 0, 0, 0};
  if ((EPI == EPI_STORE || EPI == EPI_GELU) && g.bias && n < g.N) {
    b0 = *(const f32x4_t*)(g.bias + n);
    b1 = *(const f32x4_t*)(g.bias + n + 4);
  }
  constexpr bool AUX = EPI == EPI_MUL, DSUM = EPI == EPI_DSUM;

  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // While the MFMAs of k-tile t run, the fragments of k-tile t + 1 are read
  // (two register sets).  At the barrier of step t everyone holds k-tile t's
  // fragments, so its slot takes k-tile t + NS, and k-tile t + 1 has landed.
  typename PA::Frag af[2][KSW][2];
  typename PB::Frag bf[2][KSW][2];
  constexpr int NM = KSW * 4;  // MFMAs, and as many fragments, per k-tile
  auto read = [&](auto set, auto f, uint32_t slot) {
    constexpr int S = decltype(set)::value, F = decltype(f)::value, s = F / 4, q = F % 4;
    using Sc = std::integral_constant<int, s>;
    if constexpr (q < 2) af[S][s][q] = frag(KA(), RA(), Sc(), std::integral_constant<int, q>(), ua, slot);
    else bf[S][s][q - 2] = frag(KB(), RB(), Sc(), std::integral_constant<int, q - 2>(), ub, slot);
  };
  wait_after<C::PER, NS - 1>(min(nt - 1, NS - 1));
  ring_barrier();
  static_for<0, NM>([&](auto f) { read(std::integral_constant<int, 0>(), f, 0); });
  uint32_t slot = 0;
  // One k-tile.  ISSUE: 1 = request k-tile t + NS between the MFMAs (a load
  // stalls its wavefront until the CU's address unit takes it, 17 cycles per
  // 1 KB; ahead of the MFMAs those stalls add up to as much time as the MFMAs
  // themselves), 0 = nothing left to request, 2 = request it if there is one.
  auto step = [&](auto par, auto issue_c, int t) {
    constexpr int cur = decltype(par)::value, ISSUE = decltype(issue_c)::value;
    using Next = std::integral_constant<int, cur ^ 1>;
    if constexpr (ISSUE == 1) wait_vm_lgkm0<C::PER * (NS - 2)>();
    else wait_after<C::PER, NS - 2>(max(0, min(nt - 1, t + NS - 1) - (t + 1)));
    if constexpr (TR) lds_wait();  // (on every path: the waits above branch)
    ring_barrier();
    if constexpr (TR) {
#pragma unroll
      for (int s = 0; s < KSW; ++s)
#pragma unroll
        for (int f = 0; f < 2; ++f) frag_hold(af[cur][s][f]), frag_hold(bf[cur][s][f]);
    }
    const uint32_t free_slot = slot;
    // (after the last k-tile these reads fetch a stale slot, never used)
    slot = slot == (NS - 1) * C::STAGE ? 0 : slot + C::STAGE;
    if (ISSUE == 2 && t + NS < nt) issue(t + NS);
    static_for<0, NM>([&](auto mc) {
      constexpr int m = decltype(mc)::value, s = m / 4, i = (m % 4) / 2, j = m % 2;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          frag_val(af[cur][s][i]), frag_val(bf[cur][s][j]), acc[i][j], 0, 0, 0);
      read(Next(), mc, slot);
      if constexpr (ISSUE == 1) {
        constexpr int PA_N = BM * C::BK * 2 / 1024 / C::W;  // A loads, then B loads
#pragma unroll
        for (int d = 0; d < C::PER; ++d)
          if (d * NM / C::PER == m) {
            char* dst = smem + free_slot;
            if (d < PA_N)
              dma_load<BM, AK, C::BK, C::W>(rsA, g.lda, (AK ? kbeg : 0) + (t + NS) * C::BK, dst, wave,
                                            lane, d);
            else
              dma_load<BN, BKM, C::BK, C::W>(rsB, g.ldb, (BKM ? kbeg : 0) + (t + NS) * C::BK,
                                             dst + C::A_BYTES, wave, lane, d - PA_N);
          }
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
  if constexpr (TR) {  // the unused last reads land before their registers are reused
    lds_wait();
#pragma unroll
    for (int s = 0; s < KSW; ++s)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        frag_hold(af[0][s][f]), frag_hold(bf[0][s][f]);
        frag_hold(af[1][s][f]), frag_hold(bf[1][s][f]);
      }
  }

  u32x4_t ax[AUX || DSUM ? NCH : 1], ax2[DSUM ? NCH : 1];
  if constexpr (AUX || DSUM) {
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int m = m0 + er + q * RPP;
      const int64_t at = (int64_t)m * g.ldaux + n;
      const bool in = m < g.M && n < g.N;
      ax[q] = in ? *(const u32x4_t*)((const bf16_t*)g.aux + at) : u32x4_t{0, 0, 0, 0};
      if constexpr (DSUM)
        ax2[q] = in ? *(const u32x4_t*)((const bf16_t*)g.aux2 + at) : u32x4_t{0, 0, 0, 0};
    }
  }
  // DSUM: sequence and position of the thread's row, advanced with it.
  int sb = 0, ss = 0;
  if constexpr (DSUM) {
    sb = (m0 + er) / g.dsum_S;
    ss = m0 + er - sb * g.dsum_S;
  }
  // The k sums: [k group][row][column] fp32 over the ring.
  __syncthreads();
  float* ex = (float*)smem;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        ex[(kg * BM + wm + 32 * i + 8 * (r >> 2) + 4 * hf + (r & 3)) * BN + wn + 32 * j + rr] =
            acc[i][j][r];
  __syncthreads();
  float cs[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < NCH; ++q) {
    const int row = er + q * RPP, m = m0 + row;
    float v[8];
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      const float* p = ex + (k * BM + row) * BN + ec;
      const f32x4_t x0 = *(const f32x4_t*)p, x1 = *(const f32x4_t*)(p + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = k ? v[e] + x0[e] : x0[e];
        v[4 + e] = k ? v[4 + e] + x1[e] : x1[e];
      }
    }
    if (m < g.M && n < g.N) {
      if constexpr (AUX) {
        const u32x4_t o = mul8(v, ax[q]);
        *(u32x4_t*)((bf16_t*)g.C + (int64_t)m * g.ldc + n) = o;
#pragma unroll
        for (int e = 0; e < 8; ++e) cs[e] += v[e];
      } else if constexpr (DSUM) {
        u32x4_t o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
        *(u32x4_t*)((bf16_t*)g.C + (int64_t)m * g.ldc + n) = o;
        // the head's 64 columns: 8 neighbouring lanes (rows of one head are
        // all inside or all outside, N being a multiple of 64)
        float d = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          d += __uint_as_float(o[i] << 16) *
               (__uint_as_float(ax[q][i] << 16) + __uint_as_float(ax2[q][i] << 16));
          d += __uint_as_float(o[i] & 0xffff0000u) *
               (__uint_as_float(ax[q][i] & 0xffff0000u) + __uint_as_float(ax2[q][i] & 0xffff0000u));
        }
#pragma unroll
        for (int x = 1; x < 8; x <<= 1) d += __shfl_xor(d, x, 64);
        if ((tid & 7) == 0) g.dsum[((int64_t)sb * (g.N >> 6) + (n >> 6)) * g.dsum_S + ss] = d;
      } else {
        epi8<EPI>(g, zs, m, n, v, b0, b1);
      }
    }
    if constexpr (DSUM)
      for (ss += RPP; ss >= g.dsum_S; ss -= g.dsum_S) ++sb;
  }
  if constexpr (AUX) {
    // Column sums of the tile's stored values: one partial row per tile.
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) ex[er * BN + ec + e] = cs[e];
    __syncthreads();
    if (tid < BN && n0 + tid < g.N) {
      float s = 0.0f;
#pragma unroll
      for (int k = 0; k < RPP; ++k) s += ex[k * BN + tid];
      g.colpart[(int64_t)tm * g.N + n0 + tid] = s;
    }
  }
}

template <int BM, int BN, bool AK, bool BKM, int EPI>
__global__ __launch_bounds__((MidCfg<BM, BN>::THREADS), 2) void gemm_mid_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) char smem[MidCfg<BM, BN>::LDS];
  const int nbm = (g.M + BM - 1) / BM, nbn = (g.N + BN - 1) / BN;
  int zs, tm, tn;
  mid_tile(blockIdx.x, nbm * nbn * g.ksplit, nbm, nbn, zs, tm, tn);
  mid_body<BM, BN, AK, BKM, EPI>(g, zs, tm, tn, smem);
}

// The same beside the start of a forward pass, in the work-groups after the
// tiles.
template <int BM, int BN, int EPI>
__global__ __launch_bounds__((MidCfg<BM, BN>::THREADS), 2) void gemm_mid_prep_kernel(GemmArgs g,
                                                                                   PrepArgs p) {
  __shared__ __attribute__((aligned(1024))) char smem[MidCfg<BM, BN>::LDS];
  const int nbm = (g.M + BM - 1) / BM, nbn = (g.N + BN - 1) / BN, total = nbm * nbn;
  if ((int)blockIdx.x >= total) {
    prep_unit(p, ((int)blockIdx.x - total) * MidCfg<BM, BN>::W + (int)(threadIdx.x >> 6),
              threadIdx.x & 63);
    return;
  }
  int zs, tm, tn;
  mid_tile(blockIdx.x, total, nbm, nbn, zs, tm, tn);
  mid_body<BM, BN, true, true, EPI>(g, 0, tm, tn, smem);
}

// Weight gradients of one layer in one launch, each written whole; the tail's
// units, one per wavefront, in the work-groups after the tiles.
struct MidGroup {
  GemmArgs g[GEMM_GROUP_MAX];
  int blk0[GEMM_GROUP_MAX + 1];
  int n;
  TailJobs tail;
};
template <int BM, int BN>
__global__ __launch_bounds__((MidCfg<BM, BN>::THREADS), 2) void gemm_mid_wgrad_kernel(MidGroup w) {
  __shared__ __attribute__((aligned(1024))) char smem[MidCfg<BM, BN>::LDS];
  const int b = blockIdx.x;
  if (b >= w.blk0[GEMM_GROUP_MAX]) {
    constexpr int W = MidCfg<BM, BN>::W;
    tail_unit<8>(tail_arg(offsetof(MidGroup, tail)), (b - w.blk0[GEMM_GROUP_MAX]) * W + (int)(threadIdx.x >> 6), threadIdx.x & 63);
    return;
  }
  int q = 0;
#pragma unroll
  for (int k = 1; k < GEMM_GROUP_MAX; ++k)
    if (k < w.n && b >= w.blk0[k]) q = k;
  GemmArgs g;
  int base, cnt;
  switch (q) {
    case 0: g = w.g[0]; base = w.blk0[0]; cnt = w.blk0[1]; break;
    case 1: g = w.g[1]; base = w.blk0[1]; cnt = w.blk0[2]; break;
    case 2: g = w.g[2]; base = w.blk0[2]; cnt = w.blk0[3]; break;
    default: g = w.g[3]; base = w.blk0[3]; cnt = w.blk0[4]; break;
  }
  int zs, tm, tn;
  mid_tile(b - base, cnt - base, (g.M + BM - 1) / BM, (g.N + BN - 1) / BN, zs, tm, tn);
  mid_body<BM, BN, false, false, EPI_PARTIAL>(g, 0, tm, tn, smem);
}

template <int BM, int BN, bool AK, bool BKM, int EPI>
hipError_t launch(const GemmArgs& g, hipStream_t st) {
  const int64_t total = (int64_t)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) * g.ksplit;
  hipLaunchKernelGGL((gemm_mid_kernel<BM, BN, AK, BKM, EPI>), dim3((unsigned)total),
                     dim3(MidCfg<BM, BN>::THREADS), 0, st, g);
  return hipGetLastError();
}

template <int BM, int BN>
hipError_t dispatch(const GemmArgs& g, bool b_kmajor, GemmEpi epi, hipStream_t st) {
  if (b_kmajor) {
    if (epi == EPI_STORE) return launch<BM, BN, true, true, EPI_STORE>(g, st);
    if (epi == EPI_GELU) return launch<BM, BN, true, true, EPI_GELU>(g, st);
    if (epi == EPI_PARTIAL) return launch<BM, BN, true, true, EPI_PARTIAL>(g, st);
  } else {
    if (epi == EPI_STORE) return launch<BM, BN, true, false, EPI_STORE>(g, st);
    if (epi == EPI_MUL) return launch<BM, BN, true, false, EPI_MUL>(g, st);
    if (epi == EPI_PARTIAL) return launch<BM, BN, true, false, EPI_PARTIAL>(g, st);
    if (epi == EPI_DSUM) return launch<BM, BN, true, false, EPI_DSUM>(g, st);
  }
  return hipErrorInvalidValue;
}

template <int BM, int BN>
hipError_t dispatch_prep(const GemmArgs& g, GemmEpi epi, const PrepArgs& p, hipStream_t st) {
  constexpr int W = MidCfg<BM, BN>::W;
  const int64_t total =
      (int64_t)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) + (prep_units(p) + W - 1) / W;
  if (total >= ((int64_t)1 << 28)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)total), blk(MidCfg<BM, BN>::THREADS);
  if (epi == EPI_STORE)
    hipLaunchKernelGGL((gemm_mid_prep_kernel<BM, BN, EPI_STORE>), grid, blk, 0, st, g, p);
  else
    hipLaunchKernelGGL((gemm_mid_prep_kernel<BM, BN, EPI_GELU>), grid, blk, 0, st, g, p);
  return hipGetLastError();
}

}  // namespace

hipError_t gemm_mid_prep(const GemmArgs& g, GemmEpi epi, const PrepArgs& p, hipStream_t st) {
  if ((epi != EPI_STORE && epi != EPI_GELU) || g.ksplit != 1 || p.nx % 16 != 0 || !gemm_bf16_ok(g, true))
    return hipErrorInvalidValue;
  switch (g.tile) {
    case GEMM_TILE_256x128: return dispatch_prep<256, 128>(g, epi, p, st);
    case GEMM_TILE_128x128: return dispatch_prep<128, 128>(g, epi, p, st);
    case GEMM_TILE_128x64: return dispatch_prep<128, 64>(g, epi, p, st);
    case GEMM_TILE_64x64: return dispatch_prep<64, 64>(g, epi, p, st);
  }
  return hipErrorInvalidValue;
}

hipError_t gemm_mid(const GemmArgs& g, bool b_kmajor, GemmEpi epi, int tile, hipStream_t st) {
  switch (tile) {
    case GEMM_TILE_256x128: return dispatch<256, 128>(g, b_kmajor, epi, st);
    case GEMM_TILE_128x128: return dispatch<128, 128>(g, b_kmajor, epi, st);
    case GEMM_TILE_128x64: return dispatch<128, 64>(g, b_kmajor, epi, st);
    case GEMM_TILE_64x64: return dispatch<64, 64>(g, b_kmajor, epi, st);
  }
  return hipErrorInvalidValue;
}

hipError_t gemm_mid_wgrad(const GemmArgs* p, float* const* out, int n, int tile,
                          const TailJobs& tail, hipStream_t st) {
  if (!wgrad_args_ok(p, n) || !out) return hipErrorInvalidValue;
  MidGroup w{};
  w.n = n;
  w.tail = tail;
  if (!tail_prepare(w.tail)) return hipErrorInvalidValue;
  const int bm = tile == GEMM_TILE_64x64 ? 64 : tile == GEMM_TILE_256x128 ? 256 : 128;
  const int bn = tile == GEMM_TILE_64x64 ? 64 : 128;
  int64_t blocks = 0;
  for (int q = 0; q < n; ++q) {
    if (p[q].ldc != p[q].N) return hipErrorInvalidValue;
    w.g[q] = p[q];
    w.g[q].C = out[q];
    w.g[q].ksplit = 1;
    w.g[q].kchunk = p[q].K;
    w.blk0[q] = (int)blocks;
    blocks += (int64_t)((p[q].M + bm - 1) / bm) * ((p[q].N + bn - 1) / bn);
    if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  }
  for (int q = n; q <= GEMM_GROUP_MAX; ++q) w.blk0[q] = (int)blocks;
  const int waves = tile == GEMM_TILE_64x64 ? MidCfg<64, 64>::W : MidCfg<128, 128>::W;
  blocks += (w.tail.units + waves - 1) / waves;
  if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks);
  switch (tile) {
    case GEMM_TILE_256x128:
      hipLaunchKernelGGL((gemm_mid_wgrad_kernel<256, 128>), grid, dim3(MidCfg<256, 128>::THREADS), 0, st, w);
      break;
    case GEMM_TILE_128x128:
      hipLaunchKernelGGL((gemm_mid_wgrad_kernel<128, 128>), grid, dim3(MidCfg<128, 128>::THREADS), 0, st, w);
      break;
    case GEMM_TILE_64x64:
      hipLaunchKernelGGL((gemm_mid_wgrad_kernel<64, 64>), grid, dim3(MidCfg<64, 64>::THREADS), 0, st, w);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
