// The layer's projections of at most 512 rows (Q|K|V: 384; gate|up also 961 to 1024).  Up to 256 rows one workgroup per column
// slice takes ALL rows (Q|K|V from 81 rows on: half of them), its four waves a quarter of the reduction each; above, see the second
// kernel.
//
// What bounds these launches is the number of 128-byte lines a CU has under way: about 256 of them, whatever the depth of
// the rings, so a line that misses L2 (625 ns) moves at 52 GB/s per CU, one that hits at 125, a mixture at 45 to 68.  A tile
// of R rows and C columns pulls (R + C) k elements; the 128 x 256 tiles of the ring kernel on 192 CUs pull 3.1 MB for the
// gate|up projection of 224 rows (70 us), 224 x 96 on 256 CUs 2.6 MB, of which only 0.8 come from HBM.
//
//  * With the waves along k a wave wants every activation fragment of its k-tiles and nobody else does: fragments go
//    global -> LDS -> registers inside the wave, with no barrier on their way, each read from LDS once.
//  * Weights go global -> registers, each fragment wanted by one wave per row tile (non-temporal).  They are asked for
//    in one go at the end of a k-step, together with nothing else: hits queue behind misses, so misses in bursts cost one
//    latency per 256 lines (8 misses and 20 hits a burst 68 GB/s per CU, 2 and 4: 55).  A barrier ahead of them keeps the four
//    waves' bursts one: without it the waves drift apart and the lines of one hold up the hits of the others (a block at N = 512,
//    us: 64 rows 117.7 -> 115.9, 96 133.6 -> 128.6, 128 147.1 -> 136.9, 160 166.0 -> 150.6, 224 185.1 -> 168.5, 256 190.8 ->
//    177.4; with one to three row blocks nearly all lines are misses, 40 rows 107.3 -> 107.7, and there is none).  Four to eight
//    row blocks ask for two steps' weights together (80 rows 125.2 -> 123.9, 128 139.9 -> 137.5); with more the rings hold no more
//    than two steps of activations (224 rows equal, 256 179.0 -> 184.1).
//  * At the end the four waves' sums meet in LDS, 64 rows at a time; row block 4 p + w is added up and finished by
//    wave w.
#include "mfma_tile.h"

constexpr int WK_WAVES = 4;
constexpr int WK_K = 32;                              // k per MFMA step
constexpr int WK_STEP = WK_K * WK_WAVES;              // k per step of the workgroup

// NA 16-row blocks, NBK 16-column blocks; RD steps of a wave in its rings.
template <int OUT, int NA, int NBK> struct WkCfg {
  static constexpr int RD = NA <= 8 ? 4 : 2;
  static constexpr int BURST = NA >= 4 && NA <= 8 ? 2 : 1;                  // steps whose weights are asked for together
  static constexpr int P = NA + NBK;                  // loads per wave and step
  // loads younger than those of an even, an odd step when it begins, in the order in which the loop issues them
  static constexpr int EVEN = BURST == 2 ? 3 * NBK + 2 * NA : (RD - 1) * P, ODD = BURST == 2 ? 2 * NBK + 3 * NA : (RD - 1) * P;
  static constexpr int R = NA < 4 ? NA : 4;           // activation fragments read ahead
  static constexpr int RING = WK_WAVES * RD * NA * 1024;
  static constexpr int PASS = WK_WAVES * (WK_WAVES - 1) * NBK * 1024;       // sums that change waves in one pass of 64 rows
  static constexpr int BUFS = NA > 4 ? 2 : 1;
  static constexpr int EPI = BUFS * PASS + (OUT == 3 ? WK_WAVES * 16 * VUNIT * 2 : 0);
  static constexpr int LDS = RING > EPI ? RING : EPI;
  static_assert(EVEN <= 63 && ODD <= 63 && (BURST == 1 || RD == 4) && LDS <= 160 * 1024, "wait counts, LDS");
};

template <int V> struct WkInt { static constexpr int value = V; };

template <int N, int NBK>
__device__ __forceinline__ void wk_landed(Frag (&b)[NBK]) {
  static_assert(N >= 0 && N <= 63 && (NBK == 4 || NBK == 6), "vmcnt range");
  if constexpr (NBK == 4)
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]) : "n"(N) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(%6)" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5]) : "n"(N) : "memory");
}

// OUT 0: fp32 plane of the k-split (Cf [splits][m_upper][n]); 2: gate|up with SwiGLU (Cb, fragment-tiled, ldc = d_ff);
// 3: Q|K|V with RoPE and the cache scatter.
template <int OUT, int NA, int NBK>
__global__ __launch_bounds__(256, 1) void gemm_wavek_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wp, int n, int k, int splits, const int32_t* __restrict__ m_dev,
    int m_upper, float* __restrict__ Cf, bf16_t* __restrict__ Cb, size_t ldc, int tiles_m, int tiles_n, RopeScatter rs) {
  typedef WkCfg<OUT, NA, NBK> WC;
  constexpr int RD = WC::RD, P = WC::P, R = WC::R, HB = NBK / 2, BURST = WC::BURST;
  extern __shared__ Frag lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g4 = lane >> 4, row_in = lane & 15;
  // consecutive workgroups go to consecutive XCDs: with the split in the low bits an XCD sees one split's activations
  // and the row tiles of one column tile stay on one XCD
  const int split = blockIdx.x % splits, wg = blockIdx.x / splits;
  const int tm = (wg >> 3) % tiles_m, tn = (wg >> 3) / tiles_m * 8 + (wg & 7), m0 = tm * NA * 16;
  if (tn >= tiles_n || (tm > 0 && m0 >= *m_dev)) return;
  if (OUT == 3 && rs.kc == nullptr && tn * HB >= 4 * rs.H) return;        // queries only: a slice of keys or values
  const int k_split = k / splits, steps = k_split / WK_STEP;
  const int K16 = k / 16, NF = n / 16;

  // packed 16-column block of this tile's block b
  auto col_block = [&](int b) {
    if constexpr (OUT == 2) {                         // gate blocks, then the up blocks of the same columns
      const int t = tn * HB + b % HB;
      return (t >> 1) * 4 + (t & 1) + (b / HB) * 2;
    } else if constexpr (OUT == 3) {                  // dims j .., then the dims 64 further on, of one head
      const int u = tn * HB + b % HB;
      return (u >> 2) * 8 + (u & 3) + (b / HB) * 4;
    } else {
      return tn * NBK + b;
    }
  };
  // a 16 x 32 operand lies in two neighbouring 32 x 16 blocks: lane l takes row l % 16 and the 8 k of group l / 16, 256
  // contiguous bytes per group
  const uint32_t lane_off = ((uint32_t)(g4 >> 1) * 64u + (uint32_t)((g4 & 1) * 32 + row_in)) * 16u;
  uint32_t b_voff[NBK];
#pragma unroll
  for (int b = 0; b < NBK; ++b) {
    const int f = min(col_block(b), NF - 1);          // columns past the end: valid ones, not stored
    b_voff[b] = (uint32_t)(f >> 1) * (uint32_t)K16 * 1024u + (uint32_t)(f & 1) * 256u + lane_off;
  }
  const int n_mb = (m_upper + 31) / 32;
  uint32_t a_voff[NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const int ab = m0 / 16 + a;                       // rows past the end: valid ones, not stored
    a_voff[a] = (uint32_t)min(ab >> 1, n_mb - 1) * (uint32_t)K16 * 1024u + (uint32_t)(ab & 1) * 256u + lane_off;
  }
  // wave w takes the k-tiles w, w + 4, ..: a workgroup reads its column blocks in contiguous 8 KiB
  const uint32_t k_off = ((uint32_t)(split * k_split) / 16u + (uint32_t)wave * 2u) * 1024u;
  uint64_t pa = (uint64_t)(uintptr_t)A + k_off, pb = (uint64_t)(uintptr_t)Wp + k_off;
  constexpr uint32_t K_STEP = WK_STEP / 16 * 1024;
  // Loads are inline assembly: the compiler would make every LDS read wait for all direct-to-LDS loads.  The register-ring
  // contract: fb is a read-write operand of every load and of the wait that covers it, every fetched slot is consumed, and
  // the kernel holds no spill (the build fails on scratch).
  const uint32_t ring = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) Frag*)lds + (uint32_t)wave * (RD * NA * 1024u));
  typedef const __attribute__((address_space(3))) Frag LFrag;
  LFrag* ring_l = (LFrag*)lds + wave * (RD * NA * 64) + lane;
  asm volatile("" : "+v"(ring_l));
  auto fetch_a = [&](int slot, int a) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(ring + (uint32_t)((slot * NA + a) * 1024)),
                 "v"(a_voff[a]), "s"(pa) : "memory", "m0");
  };
  Frag fb[RD][NBK];
#pragma unroll
  for (int u = 0; u < RD; ++u)
#pragma unroll
    for (int b = 0; b < NBK; ++b) fb[u][b] = Frag{};
  auto fetch_b = [&](int slot) {
#pragma unroll
    for (int b = 0; b < NBK; ++b)
      asm volatile("global_load_dwordx4 %0, %1, %2 nt" : "+v"(fb[slot][b]) : "v"(b_voff[b]), "s"(pb) : "memory");
    pb += K_STEP;
  };
  f32x4 acc[NA][NBK];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NBK; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the first 64 accumulator blocks live in the AGPR half, the rest beside the operands
  auto mma = [&](const Frag& w, const Frag& x, int a, int b) {
    if (a * NBK + b < 64) asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[a][b]) : "v"(w), "v"(x));
    else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[a][b]) : "v"(w), "v"(x));
  };
  auto pin = [&](int a, int b) {
    if (a * NBK + b < 64) asm volatile("" : "+a"(acc[a][b]));
    else asm volatile("" : "+v"(acc[a][b]));
  };

  const int count = *m_dev;                           // asked for ahead of the loads, waited for behind them
#pragma unroll
  for (int u = 0; u < RD; ++u) {
    if (BURST == 1) fetch_b(u);
#pragma unroll
    for (int a = 0; a < NA; ++a) fetch_a(u, a);
    pa += K_STEP;
    if (BURST == 2 && u % 2 == 1) { fetch_b(u - 1); fetch_b(u); }
  }
  const int M = min(count, m_upper);
  if (M <= 0) {                                       // uniform; nothing of the prologue's may still be on its way
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return;
  }
  // 16-row blocks past the count: from here on the tile's first block in their place (lines that are on their way anyway), so
  // that a bound above the count costs no more reads (one block at N = 512, bound 160: 1 row 136 -> 115 us, 33 rows 141 -> 124; bound
  // 256: no row 141 -> 32, 33 rows 161 -> 143; tight bounds the same within 0.5 %).  Not in a second row tile, which would run ahead of
  // the first and leave it without the weight lines both want (200 rows bounded by 384 212 -> 216)
#pragma unroll
  for (int a = 1; a < NA; ++a)
    if (tm == 0 && a * 16 >= M) a_voff[a] = a_voff[0];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NBK; ++b) pin(a, b);          // zeroed before the wait states
  asm volatile("s_nop 7" ::: "memory");

  // one step out of slot u; FETCH: each fragment's slot is asked for again as soon as its MFMAs are issued
  Frag af[R];
  auto step = [&](auto fetch, int u, int v) {         // activations out of slot u, weights out of slot v
#pragma unroll
    for (int a = 0; a < R; ++a) af[a] = ring_l[(u * NA + a) * 64];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
#pragma unroll
      for (int b = 0; b < NBK; ++b) mma(fb[v][b], af[a % R], a, b);
      if (a + R < NA) af[a % R] = ring_l[(u * NA + a + R) * 64];
      if constexpr (decltype(fetch)::value) fetch_a(u, a);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (decltype(fetch)::value) pa += K_STEP;
    __builtin_amdgcn_sched_barrier(0);
  };
  auto landed = [&](auto younger, int v) {
    wk_landed<decltype(younger)::value>(fb[v]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto weights = [&](int v) {                         // a burst, of slot v and those before it
    if constexpr (NA >= 4) asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int b = BURST - 1; b >= 0; --b) fetch_b(v - b);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int s = 0; s + RD < steps; s += RD) {
#pragma unroll
    for (int u = 0; u < RD; ++u) {
      if (u % 2 == 0) landed(WkInt<WC::EVEN>{}, u);
      else landed(WkInt<WC::ODD>{}, u);
      step(WkInt<1>{}, u, u);
      if (u % BURST == BURST - 1) weights(u);
    }
  }
  // the flat ids of the rows this lane will finish (none past the row count: the array may end there), behind the last
  // fragments, which are waited for first; younger loads make those waits no looser
  constexpr int PASSES = (NA + 3) / 4;
  int gid[PASSES];
  if constexpr (OUT == 3) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int row = m0 + (p * 4 + wave) * 16 + row_in;
      gid[p] = p * 4 + wave < NA && row < M ? rs.active_idx[row] : -1;
    }
  }
  // the last RD steps fetch nothing; after the last wait no load is in flight
  landed(WkInt<WC::EVEN>{}, 0);
  step(WkInt<0>{}, 0, 0);
  landed(WkInt<BURST == 2 ? 2 * P : (RD - 2) * P>{}, 1);
  step(WkInt<0>{}, 1, 1);
  if constexpr (RD == 4) {
    landed(WkInt<BURST == 2 ? NBK : P>{}, 2);
    step(WkInt<0>{}, 2, 2);
    landed(WkInt<0>{}, 3);
    step(WkInt<0>{}, 3, 3);
  }
  static_assert(RD == 2 || RD == 4, "last steps are written out");
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NBK; ++b) pin(a, b);

  // the waves' sums meet in LDS: of the row blocks 4 p .. 4 p + 3 wave w keeps block 4 p + w and hands the others over
  int seq[PASSES];
  constexpr bool EARLY = NA <= 8;                     // all of a lane's table rows at once, where registers are free
  float4 tab[EARLY ? PASSES : 1][HB][2];
  if constexpr (OUT == 3) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      seq[p] = max(gid[p], 0) / rs.N;
      gid[p] -= seq[p] * rs.N;                        // the slot, -1 past the row count
      if constexpr (EARLY) {
#pragma unroll
        for (int b = 0; b < HB; ++b) rope_load_unit(tab[p][b], max(gid[p], 0), (tn * HB + b & 3) * 16, rs);
      }
    }
  }
  __syncthreads();                                    // every wave is done with its ring
  bf16_t* stage = reinterpret_cast<bf16_t*>(reinterpret_cast<char*>(lds) + WC::BUFS * WC::PASS) + wave * 16 * VUNIT;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    f32x4* exch = reinterpret_cast<f32x4*>(lds) + (p % WC::BUFS) * (WC::PASS / 16);   // [to][from, less the wave itself][NBK][64]
    f32x4 c[NBK];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a = p * 4 + j;
      if (a >= NA) continue;
#pragma unroll
      for (int b = 0; b < NBK; ++b) pin(a, b);        // read here, not all at once ahead
      if (j == wave) {
#pragma unroll
        for (int b = 0; b < NBK; ++b) c[b] = acc[a][b];
      } else {
        f32x4* e = exch + ((j * 3 + wave - (wave > j)) * NBK) * 64 + lane;
#pragma unroll
        for (int b = 0; b < NBK; ++b) e[b * 64] = acc[a][b];
      }
    }
    __syncthreads();                                  // also: the pass before the last has been read
    const int a = p * 4 + wave, row = m0 + a * 16 + row_in;
    if (a >= NA || m0 + a * 16 >= M) continue;
    // in wave order whichever wave adds: a row's sums do not depend on where in the launch it stands
    const f32x4* e = exch + wave * 3 * NBK * 64 + lane;
    auto add = [&](auto own) {
#pragma unroll
      for (int b = 0; b < NBK; ++b) {
        const f32x4 x = e[b * 64], y = e[(NBK + b) * 64], z = e[(2 * NBK + b) * 64];
        if constexpr (decltype(own)::value == 0) c[b] = c[b] + x + y + z;             // wave 0 or 1
        else if constexpr (decltype(own)::value == 2) c[b] = x + y + c[b] + z;
        else c[b] = x + y + z + c[b];
      }
    };
    if (wave < 2) add(WkInt<0>{});
    else if (wave == 2) add(WkInt<2>{});
    else add(WkInt<3>{});
    if constexpr (OUT == 0) {
#pragma unroll
      for (int b = 0; b < NBK; ++b) {
        const int col = (tn * NBK + b) * 16 + 4 * g4;
        if (row < M && col < n) *reinterpret_cast<f32x4*>(Cf + ((size_t)split * m_upper + row) * ldc + col) = c[b];
      }
    } else if constexpr (OUT == 2) {
      float gs[4 * HB], us[4 * HB], y[4 * HB];
#pragma unroll
      for (int e = 0; e < 4 * HB; ++e) {
        gs[e] = c[e >> 2][e & 3];
        us[e] = c[(e >> 2) + HB][e & 3];
      }
      silu_mul(gs, us, y);
#pragma unroll
      for (int b = 0; b < HB; ++b) {
        const int col = (tn * HB + b) * 16 + 4 * g4;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16_t)y[b * 4 + e];
        if (row < M && col < (n >> 1)) *reinterpret_cast<bf16x4*>(Cb + afrag_index(row, col, (int)ldc)) = v;
      }
    } else {
      if constexpr (!EARLY) {
#pragma unroll
        for (int b = 0; b < HB; ++b) rope_load_unit(tab[0][b], max(gid[p], 0), (tn * HB + b & 3) * 16, rs);
      }
#pragma unroll
      for (int b = 0; b < HB; ++b) {
        const int u = tn * HB + b, hsec = u >> 2, sec = hsec / rs.H, head = hsec - sec * rs.H, j0 = (u & 3) * 16;
        if (sec > 2 || (sec > 0 && rs.kc == nullptr)) continue;
        if (sec < 2) {
          if (gid[p] >= 0) rope_store_unit(c[b], c[b + HB], tab[EARLY ? p : 0][b], sec, head, j0, row, seq[p], gid[p], rs);
        } else {
          v_store_unit(stage, c[b], c[b + HB], head, j0, seq[p], gid[p], rs);
        }
      }
    }
  }
}

template <int OUT, int NA, int NBK>
static int launch_wavek(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int n, int k, int splits,
                        float* Cf, void* Cb, size_t ldc, const RopeScatter& rs) {
  const size_t sh = WkCfg<OUT, NA, NBK>::LDS;
  auto kern = gemm_wavek_kernel<OUT, NA, NBK>;
  static unsigned long long lds_ok = 0;
  SL_ALLOW_DYNAMIC_LDS(lds_ok, kern, sh);
  const int tiles_m = sl_cdiv(mu, NA * 16), tiles_n = sl_cdiv(n, NBK * 16);
  hipLaunchKernelGGL(kern, dim3(8 * sl_cdiv(tiles_n, 8) * tiles_m * splits), dim3(256), sh, s, (const bf16_t*)A, (const bf16_t*)Wp, n, k,
                     splits, m_dev, mu, Cf, (bf16_t*)Cb, ldc, tiles_m, tiles_n, rs);
  SL_LAUNCH_CHECK();
  return SL_OK;
}

// A launch of `blocks` 16-row blocks per workgroup; compiled for the heights LO .. HI that its form takes (wavek_blocks).
template <int OUT, int NBK, int LO, int HI>
static int launch_blocks(hipStream_t s, int blocks, const void* A, const void* Wp, const int32_t* m_dev, int mu, int n, int k, int splits,
                         float* Cf, void* Cb, size_t ldc, const RopeScatter& rs = RopeScatter{}) {
#define GO(NA) \
  if constexpr (NA >= LO && NA <= HI) \
    if (blocks == NA) return launch_wavek<OUT, NA, NBK>(s, A, Wp, m_dev, mu, n, k, splits, Cf, Cb, ldc, rs)
  GO(1); GO(2); GO(3); GO(4); GO(5); GO(6); GO(7); GO(8); GO(10); GO(12); GO(14); GO(16);
#undef GO
  return SL_EINVAL;
}

// ---- 2 x 2 waves ------------------------------------------------------------------------------------------------
// 257 to 512 rows: two row tiles, and with them twice as wide column slices, are too many sums for one wave.  TM = 16 NA rows x
// 32 NBK columns per workgroup: wave w takes the k-tiles 2 s + w / 2 and the half w % 2 of the columns.  The two waves of a
// k-tile share its activations, each fetching half of the fragments, so a step ends in a barrier; it stands R row blocks before
// the last MFMAs, which cover it and the first LDS reads of the next step.  256 x 192 tiles of the gate|up projection fill 256
// CUs where 256 x 256 left 64 idle: 512 rows 92 -> 82 us (loop 1970 cycles a step of 1536 MFMA cycles with weights from HBM, 1770
// from the memory-side cache: the lines under way again, 28 bytes per cycle).
template <int OUT, int NA, int NBK> struct W22Cfg {
  static_assert(NA % 2 == 0, "the waves of a k-tile fetch half of its activation fragments each");
  static constexpr int RD = 3;                        // steps in the rings: one in use, two under way
  static constexpr int P = NBK + NA / 2;              // loads per wave and step, weights first
  static constexpr int R = NA % 4 == 0 ? 4 : NA % 5 == 0 ? 5 : 7;       // activation fragments read ahead
  static constexpr int BAR = NA - R;                  // row block before which the next step is published
  static constexpr int LATE = BAR * P / NA;           // loads of a step issued before that
  static constexpr int RING = 2 * RD * NA * 1024;
  static constexpr int PASS = 4 * 2 * NBK * 1024;     // exchange: 2 row blocks per wave and pass
  static constexpr int LDS = RING > 2 * PASS ? RING : 2 * PASS;
  static_assert(NA % R == 0 && P <= 63 && LDS <= 160 * 1024, "schedule");
};

// XCD x owns the column tiles 8 c + x; the row tiles and splits of one column tile follow each other.  Only row tiles that hold
// rows are counted, so the workgroups without work are the last ones: an XCD's workgroups go to its four shader engines in turn,
// and with every fourth one working they all went to one engine's eight CUs, two to a CU (gate|up of 16 rows bounded by 1024 116 us,
// of 300 rows 128; now 62 and 76).  Three count as four: 600 rows 131 us, in threes 138.  One to four row tiles and a power of two of
// splits: every workgroup waits for the count before its first load, so no divisions behind it.
struct W22Tile { int tm, tn, split; };
__host__ __device__ inline W22Tile w22_tile(int wg, int row_tiles, int splits) {
  const int sh = row_tiles > 2 ? 2 : row_tiles - 1, xcd = wg & 7, j = wg >> 3, group = j >> sh;
  return W22Tile{j & ((1 << sh) - 1), (group >> __builtin_ctz(splits)) * 8 + xcd, group & (splits - 1)};
}
void slk_wave22_tile(int wg, int row_tiles, int splits, int* out) {     // for tests
  const W22Tile t = w22_tile(wg, row_tiles, splits);
  out[0] = t.tm; out[1] = t.tn; out[2] = t.split;
}

template <int OUT, int NA, int NBK>
__global__ __launch_bounds__(256, 1) void gemm_wave22_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ Wp, int n, int k, int splits, const int32_t* __restrict__ m_dev,
    int m_upper, float* __restrict__ Cf, bf16_t* __restrict__ Cb, size_t ldc, int tiles_n) {
  typedef W22Cfg<OUT, NA, NBK> WC;
  constexpr int RD = WC::RD, P = WC::P, R = WC::R, HB = NBK / 2, TM = NA * 16;
  extern __shared__ Frag lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int kg = wave >> 1, cg = wave & 1;
  const int g4 = lane >> 4, row_in = lane & 15;
  const int M = min(*m_dev, m_upper);
  if (M <= 0) return;
  const W22Tile tile = w22_tile(blockIdx.x, (M + TM - 1) / TM, splits);
  const int tm = tile.tm, tn = tile.tn, split = tile.split, m0 = tm * TM;
  if (tn >= tiles_n || m0 >= M) return;
  const int k_split = k / splits, steps = k_split / 64;
  const int K16 = k / 16, NF = n / 16;
  auto col_block = [&](int b) {
    const int t = (tn * 2 + cg) * HB + b % HB;
    if constexpr (OUT == 2) return (t >> 1) * 4 + (t & 1) + (b / HB) * 2;
    else return (tn * 2 + cg) * NBK + b;
  };
  const uint32_t lane_off = ((uint32_t)(g4 >> 1) * 64u + (uint32_t)((g4 & 1) * 32 + row_in)) * 16u;
  uint32_t b_voff[NBK];
#pragma unroll
  for (int b = 0; b < NBK; ++b) {
    const int f = min(col_block(b), NF - 1);
    b_voff[b] = (uint32_t)(f >> 1) * (uint32_t)K16 * 1024u + (uint32_t)(f & 1) * 256u + lane_off;
  }
  const int n_mb = (m_upper + 31) / 32;
  uint32_t a_voff[NA / 2];                            // row blocks 2 i + cg
#pragma unroll
  for (int i = 0; i < NA / 2; ++i) a_voff[i] = (uint32_t)min(m0 / 32 + i, n_mb - 1) * (uint32_t)K16 * 1024u + (uint32_t)cg * 256u + lane_off;
  const uint32_t k_off = ((uint32_t)(split * k_split) / 16u + (uint32_t)kg * 2u) * 1024u;
  uint64_t pa = (uint64_t)(uintptr_t)A + k_off, pb = (uint64_t)(uintptr_t)Wp + k_off;

  const uint32_t ring = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) Frag*)lds + (uint32_t)(kg * (RD * NA) + cg) * 1024u);
  typedef const __attribute__((address_space(3))) Frag LFrag;
  LFrag* ring_l = (LFrag*)lds + kg * (RD * NA * 64) + lane;
  asm volatile("" : "+v"(ring_l));
  auto a_frag = [&](int slot, int a) -> Frag { return ring_l[(slot * NA + a) * 64]; };
  Frag fb[RD][NBK];
#pragma unroll
  for (int u = 0; u < RD; ++u)
#pragma unroll
    for (int b = 0; b < NBK; ++b) fb[u][b] = Frag{};
  // load i of a step into slot `slot`: the weights, then this wave's half of the activations
  auto fetch = [&](int slot, int i) {
    if (i < NBK) {
      asm volatile("global_load_dwordx4 %0, %1, %2 nt" : "+v"(fb[slot][i]) : "v"(b_voff[i]), "s"(pb) : "memory");
    } else {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(ring + (uint32_t)((slot * NA + 2 * (i - NBK)) * 1024)),
                   "v"(a_voff[i - NBK]), "s"(pa) : "memory", "m0");
    }
  };
  int fetched = 0;
  auto next = [&] {                                   // past the end the last step again (never used)
    const uint32_t d = fetched < steps - 1 ? 4096u : 0u;
    pa += d;
    pb += d;
    ++fetched;
  };
  f32x4 acc[NA][NBK];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NBK; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mma = [&](const Frag& w, const Frag& x, int a, int b) {
    if (a * NBK + b < 64) asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[a][b]) : "v"(w), "v"(x));
    else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[a][b]) : "v"(w), "v"(x));
  };
  auto pin = [&](int a, int b) {
    if (a * NBK + b < 64) asm volatile("" : "+a"(acc[a][b]));
    else asm volatile("" : "+v"(acc[a][b]));
  };
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int i = 0; i < P; ++i) fetch(u, i);
    next();
  }
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NBK; ++b) pin(a, b);
  Frag af[R];
  wk_landed<P>(fb[0]);
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int a = 0; a < R; ++a) af[a] = a_frag(0, a);
  asm volatile("s_nop 7" ::: "memory");

  for (int s = 0; s < steps; s += RD) {
#pragma unroll
    for (int u = 0; u < RD; ++u) {
      if (u > 0 && s + u >= steps) break;
      const int nu = (u + 1) % RD, fu = (u + 2) % RD;
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        if (a == WC::BAR) {
          // every wave has read the last of this step, and its own loads of the next one have landed
          wk_landed<WC::LATE>(fb[nu]);
          asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int b = 0; b < NBK; ++b) mma(fb[u][b], af[a % R], a, b);
        af[a % R] = a + R < NA ? a_frag(u, a + R) : a_frag(nu, a + R - NA);
#pragma unroll
        for (int i = a * P / NA; i < (a + 1) * P / NA; ++i) fetch(fu, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      next();
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < RD; ++u) wk_landed<0>(fb[u]);
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NBK; ++b) pin(a, b);

  // the two k-tiles' sums meet in LDS: of the row blocks 4 p .. 4 p + 3 the wave keeps those with a / 2 % 2 == kg
  __syncthreads();
  constexpr int PASSES = (NA + 3) / 4;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    f32x4* exch = reinterpret_cast<f32x4*>(lds) + (p & 1) * (WC::PASS / 16);          // [cg][to kg][2][NBK][64]
    f32x4 c[2][NBK];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a = p * 4 + j;
      if (a >= NA) continue;
#pragma unroll
      for (int b = 0; b < NBK; ++b) pin(a, b);
      if (j >> 1 == kg) {
#pragma unroll
        for (int b = 0; b < NBK; ++b) c[j & 1][b] = acc[a][b];
      } else {
        f32x4* e = exch + ((cg * 2 + (j >> 1)) * 2 + (j & 1)) * NBK * 64 + lane;
#pragma unroll
        for (int b = 0; b < NBK; ++b) e[b * 64] = acc[a][b];
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int a = p * 4 + kg * 2 + h, row = m0 + a * 16 + row_in;
      if (a >= NA || m0 + a * 16 >= M) continue;
#pragma unroll
      for (int b = 0; b < NBK; ++b) c[h][b] += exch[(((cg * 2 + kg) * 2 + h) * NBK + b) * 64 + lane];
      if constexpr (OUT == 0) {
#pragma unroll
        for (int b = 0; b < NBK; ++b) {
          const int col = ((tn * 2 + cg) * NBK + b) * 16 + 4 * g4;
          if (row < M && col < n) *reinterpret_cast<f32x4*>(Cf + ((size_t)split * m_upper + row) * ldc + col) = c[h][b];
        }
      } else if constexpr (OUT == 2) {
        float gs[4 * HB], us[4 * HB], y[4 * HB];
#pragma unroll
        for (int e = 0; e < 4 * HB; ++e) {
          gs[e] = c[h][e >> 2][e & 3];
          us[e] = c[h][(e >> 2) + HB][e & 3];
        }
        silu_mul(gs, us, y);
#pragma unroll
        for (int b = 0; b < HB; ++b) {
          const int col = ((tn * 2 + cg) * HB + b) * 16 + 4 * g4;
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (bf16_t)y[b * 4 + e];
          if (row < M && col < (n >> 1)) *reinterpret_cast<bf16x4*>(Cb + afrag_index(row, col, (int)ldc)) = v;
        }
      }
    }
  }
}

template <int OUT, int NA, int NBK>
static int launch_wave22(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int n, int k, int splits,
                         float* Cf, void* Cb, size_t ldc) {
  const size_t sh = W22Cfg<OUT, NA, NBK>::LDS;
  auto kern = gemm_wave22_kernel<OUT, NA, NBK>;
  static unsigned long long lds_ok = 0;
  SL_ALLOW_DYNAMIC_LDS(lds_ok, kern, sh);
  const int tiles_m = sl_cdiv(mu, NA * 16), tiles_n = sl_cdiv(n, 32 * NBK);
  if (tiles_m > 4 || splits < 1 || (splits & (splits - 1))) return SL_EINVAL;         // what w22_tile numbers
  hipLaunchKernelGGL(kern, dim3(8 * sl_cdiv(tiles_n, 8) * (tiles_m == 3 ? 4 : tiles_m) * splits), dim3(256), sh, s, (const bf16_t*)A, (const bf16_t*)Wp, n, k,
                     splits, m_dev, mu, Cf, (bf16_t*)Cb, ldc, tiles_n);
  SL_LAUNCH_CHECK();
  return SL_OK;
}
template <int OUT, int NBK>
static int launch22_blocks(hipStream_t s, int blocks, const void* A, const void* Wp, const int32_t* m_dev, int mu, int n, int k, int splits,
                           float* Cf, void* Cb, size_t ldc) {
  switch (blocks) {
    case 10: return launch_wave22<OUT, 10, NBK>(s, A, Wp, m_dev, mu, n, k, splits, Cf, Cb, ldc);
    case 12: return launch_wave22<OUT, 12, NBK>(s, A, Wp, m_dev, mu, n, k, splits, Cf, Cb, ldc);
    case 14: return launch_wave22<OUT, 14, NBK>(s, A, Wp, m_dev, mu, n, k, splits, Cf, Cb, ldc);
    case 16: return launch_wave22<OUT, 16, NBK>(s, A, Wp, m_dev, mu, n, k, splits, Cf, Cb, ldc);
  }
  return SL_EINVAL;
}

// ---- which launches ---------------------------------------------------------------------------------------------
// Whole trips of the rings, 32-bit offsets; and a single round of workgroups that fills most of the chip: the slices are as
// narrow as the epilogues allow, so fewer than 160 of them leave too many CUs idle (the other kernels then choose their own
// tiles), and a second round would read the activations again.  Measured at the LLaDA-8B shapes, one block at N = 512, us
// before -> with these launches (before: the weight-stream kernel up to 32 rows, the ring kernel, and the RoPE and SwiGLU
// kernels behind them): 16 rows 110 -> 99, 48 rows 134 -> 109, 64 rows 143 -> 120, 128 rows 163 -> 149, 224 rows 204 -> 187,
// 256 rows 210 -> 195, 320 rows 240 -> 217, 400 rows 265 -> 239, 512 rows 280 -> 258.
static bool fits(int mu, int n, int k, int k_unit, int workgroups) {
  return mu > 0 && n > 0 && n % 32 == 0 && k % k_unit == 0 && (size_t)n * k * 2 < ((size_t)1 << 32) &&
         sl_align_up(mu, 32) * k * 2 < ((size_t)1 << 32) && workgroups >= 160 && workgroups <= 256;
}
constexpr int kWavekTrip = 4 * WK_STEP;               // k of a whole trip of the deepest ring
constexpr int kPlanes = 4;

// A launch's form: waves along k (1) or 2 x 2 waves (2), 16-row and 16-column blocks per workgroup, row tiles; kernel 0: not
// taken.  Waves along k: the smallest compiled height that covers the rows, from `lowest` on.
struct WkForm { int kernel, blocks, cols, tiles_m; };
static WkForm wavek_form(int mu, int tiles_m, int cols, int lowest) {
  int b = sl_cdiv(mu, 16 * tiles_m);
  if (b < lowest) b = lowest;
  if (b > 8) b = (b + 1) / 2 * 2;
  return WkForm{1, b, cols, tiles_m};
}
// 2 x 2 waves: whole pairs of blocks, evenly over tiles of at most 256 rows
static WkForm wave22_form(int mu, int cols) {
  const int tiles_m = sl_cdiv(mu, 256);
  return WkForm{2, (int)sl_align_up(sl_cdiv(mu, tiles_m), 32) / 16, cols, tiles_m};
}

// Q|K|V: up to 80 rows 64 columns (two units of 16 + 16 that RoPE pairs) for all rows; from 81 rows on 96 columns for half of the
// rows each, where (rows / 2 + 96) is less to read than (rows + 64) and 256 CUs share the work instead of 192 (96 rows 37.7 ->
// 35.4 us, 256 rows 56 -> 47; 80 rows 34.8 -> 34.6, 64 rows 29.5 -> 32.5).  Up to 384 rows: there 55 us against 62 of the
// ring kernel's k-split with RoPE behind it, at 400 rows 60 against 59 of its fused form.
constexpr int kWavekQkvRows = 384, kWavekQkvOneTile = 80;
static WkForm qkv_form(int mu, int H, int k) {
  if (mu > kWavekQkvRows || H <= 0 || !fits(mu, 3 * H * 128, k, kWavekTrip, mu > kWavekQkvOneTile ? 8 * H : 6 * H)) return WkForm{};
  return mu > kWavekQkvOneTile ? wavek_form(mu, 2, 6, 4) : wavek_form(mu, 1, 4, 1);
}
int slk_wavek_qkv_ok(int mu, int H, int k) { return qkv_form(mu, H, k).kernel != 0; }
int slk_wavek_qkv_rope(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int H, int k,
                       const int32_t* active_idx, int N, int n_pad, const void* rope_tab, void* q, void* kc, void* vc) {
  const int n = 3 * H * 128;
  const WkForm f = qkv_form(mu, H, k);
  if (!f.kernel || !active_idx || !rope_tab || !q || (kc == nullptr) != (vc == nullptr)) return SL_EINVAL;
  if ((uintptr_t)q % 16 || (uintptr_t)kc % 16 || (uintptr_t)vc % 16 || (uintptr_t)rope_tab % 16) return SL_EINVAL;
  const RopeScatter rs{active_idx, (const float2*)rope_tab, (bf16_t*)q, (bf16_t*)kc, (bf16_t*)vc, N, n_pad, H};
  if (f.tiles_m == 2) return launch_blocks<3, 6, 4, 12>(s, f.blocks, A, Wp, m_dev, mu, n, k, 1, nullptr, nullptr, (size_t)n, rs);
  return launch_blocks<3, 4, 1, 5>(s, f.blocks, A, Wp, m_dev, mu, n, k, 1, nullptr, nullptr, (size_t)n, rs);
}

// gate|up: up to 256 rows 48 gate columns and their 48 up columns per workgroup, up to 512 rows 96 + 96 with two row tiles.
// Four row tiles where the ring kernel's best tiles, 192 rows on five row tiles, no longer cover the rows (992 rows 166 -> 153 us;
// 960 rows 145 against 153, 857 rows 143.5 / 143, 800 rows 124 / 143), and the column slices fill the second round of workgroups
// too; three are a round and a half (700 rows 119 against 146).
constexpr int kRingRows5 = 5 * 192;
static WkForm swiglu_form(int mu, int dff, int k) {
  if (mu <= 256) return fits(mu, 2 * dff, k, kWavekTrip, sl_cdiv(dff, 48)) ? wavek_form(mu, 1, 6, 1) : WkForm{};
  const int slices = sl_cdiv(dff, 96);
  const bool two_tiles = mu <= 512, four_tiles = mu > kRingRows5 && mu <= 1024 && 2 * slices > 224;
  return (two_tiles || four_tiles) && fits(mu, 2 * dff, k, 64, 2 * slices) ? wave22_form(mu, 6) : WkForm{};
}
int slk_wavek_swiglu_ok(int mu, int dff, int k) { return swiglu_form(mu, dff, k).kernel != 0; }
int slk_wavek_swiglu(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int dff, int k, void* a) {
  const WkForm f = swiglu_form(mu, dff, k);
  if (!f.kernel) return SL_EINVAL;
  if (f.kernel == 1) return launch_blocks<2, 6, 1, 16>(s, f.blocks, A, Wp, m_dev, mu, 2 * dff, k, 1, nullptr, a, (size_t)dff);
  return launch22_blocks<2, 6>(s, f.blocks, A, Wp, m_dev, mu, 2 * dff, k, 1, nullptr, a, (size_t)dff);
}

// Out and down, k in four splits: up to 256 rows 64 columns for all rows, up to 512 rows 128 columns and two row tiles (512 rows
// down 56.5 -> 50 us, 264 rows 46.5 -> 41).  The number of planes, 0 if these launches do not take the shape.  (Two row tiles of
// 128 columns with the waves along k: the same from 128 rows on, slower below.)
static WkForm planes_form(int mu, int n, int k) {
  if (mu <= 256) return fits(mu, n, k, kPlanes * kWavekTrip, kPlanes * sl_cdiv(n, 64)) ? wavek_form(mu, 1, 4, 1) : WkForm{};
  return mu <= 512 && fits(mu, n, k, kPlanes * 64, 2 * kPlanes * sl_cdiv(n, 128)) ? wave22_form(mu, 4) : WkForm{};
}
int slk_wavek_splits(int mu, int n, int k) { return planes_form(mu, n, k).kernel ? kPlanes : 0; }
int slk_wavek_planes(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int n, int k, float* Cf) {
  const WkForm f = planes_form(mu, n, k);
  if (!f.kernel || !Cf || (uintptr_t)Cf % 16) return SL_EINVAL;
  if (f.kernel == 1) return launch_blocks<0, 4, 1, 16>(s, f.blocks, A, Wp, m_dev, mu, n, k, kPlanes, Cf, nullptr, (size_t)n);
  return launch22_blocks<0, 4>(s, f.blocks, A, Wp, m_dev, mu, n, k, kPlanes, Cf, nullptr, (size_t)n);
}

// for tests: the form of a layer's launch; projection 0: Q|K|V (width = heads), 1: gate|up (d_ff), 2: Out and down (columns)
void slk_wavek_form(int projection, int mu, int width, int k, int* out) {
  const WkForm f = projection == 0 ? qkv_form(mu, width, k) : projection == 1 ? swiglu_form(mu, width, k) : planes_form(mu, width, k);
  out[0] = f.kernel; out[1] = f.blocks; out[2] = f.cols; out[3] = f.tiles_m;
}
