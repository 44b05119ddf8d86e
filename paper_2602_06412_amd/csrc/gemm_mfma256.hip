// The projection GEMM of launches bounded by more than 32 rows (where gemm_wavek.hip takes a layer's shape: Q|K|V of more than
// 384 rows, the other projections of more than 512, gate|up not of 961 to 1024): one TM x 256 output tile per workgroup and CU, TM
// any multiple of 32 from 64 to 256.  Four waves, one per SIMD; each owns all TM rows of 64 columns (up to 256 accumulator
// registers), so a weight fragment is wanted by exactly one wave.
//
//  * Weights go global -> registers: a ring of DB k-tiles (32 deep) of B fragments per wave.  They never touch LDS,
//    which the four waves need for the activations: with both operands in LDS and eight (TM/2) x 64 waves (the form
//    this kernel replaces) LDS moved 128 KiB per k-tile of 1024 MFMA cycles, its peak rate; here it moves 80 KiB.
//  * Activations go global -> LDS by direct loads (no registers tied up) into a ring of RING k-tiles, KT per
//    barrier; every wave reads all of them, fragments LA row blocks ahead of the MFMAs that use them.
//  * One wave per SIMD has nobody to cover for it, so the loop body is laid out by hand and unrolled over the whole
//    ring: one LDS read per row block, one global load every GAP MFMAs, never two together (loads bunched at the
//    ends of a k-tile: 1402 cycles per k-tile; spread: 1220), and no vector-ALU instruction at all: an address
//    addition between two MFMAs costs a whole MFMA slot (with one per LDS read: 1261 cycles, none: 1132; the
//    floor is 1024).  LDS addresses are two base registers plus immediates, global ones scalar bases.
//  * The epilogues work on registers: two lane-group swaps give a lane eight consecutive columns, i.e. 16-byte
//    pieces (8-byte pieces: 19000 cycles per tile; 16-byte: 10000).
// Inside a step of 8192 rows (us; eight-wave form -> this): 24576 x 4096 1188 -> 1130, 4096 x 12288 578 -> 539, the LM head
// 6142 -> 5696.
//
// A short tile is bound by the rate at which one CU pulls lines that miss its L2 (about 20 B per clock, whatever
// the depth of the ring: four or eight k-tiles in flight measure the same), so a launch wants many CUs before it
// wants tall tiles; the launch plan prices that.
//
// The products are v_mfma_f32_16x16x32_bf16, not 32x32x16: same flops per cycle, but measured
// on this chip with random operands a loop of 16x16x32 sustains ~1.93 PFLOP/s at ~1.95 GHz where
// 32x32x16 sustains ~1.65 at ~1.65 GHz (the clock is managed by power, and the deeper dot
// product moves a quarter of the accumulator data per flop).  A 16 x 32 operand of that
// instruction (lane l: row l % 16, k = 8 * (l / 16) .. +7) is gathered from two neighbouring
// 32 x 16 blocks by giving every lane its own slot address; each group of 16 lanes still reads
// 256 contiguous bytes.  The weight fragment is passed as the first operand, so a lane ends up
// with four consecutive columns of one output row.
#include "mfma_tile.h"

constexpr int BK2 = 32;                   // k per k-tile: one 16x16x32 MFMA k-step
constexpr int TILE = 256;                 // columns per tile, and rows of the full-height tile
constexpr int NB = 4;                     // 16-column blocks per wave
// Rows per tile TM: any multiple of 32 from 64 to 256, so that a launch can fit its row tiles to the
// number of active rows (320 rows = two tiles of 160, not two of 256) and latency follows M.
template <int TM> struct TileCfg {
  static_assert(TM % 32 == 0 && TM >= 64 && TM <= 256, "tile height");
  static constexpr int NA = TM / 16;                // 16-row blocks
  static constexpr int A_FR = TM / 16;              // 1 KiB fragments (32 rows x 16 k) of A per k-tile
  static constexpr int NAD = (A_FR + 3) / 4;        // direct-to-LDS loads per wave and k-tile
  static constexpr int P = NAD + NB;                // global loads per wave and k-tile
  static constexpr int KTB = TM * BK2 * 2;          // LDS bytes per k-tile
  static constexpr int DB = 4;                      // B ring: DB - 1 k-tiles in flight beyond the one in use
  static constexpr int KT = 2;                      // k-tiles per barrier
  static constexpr int RING = 8;                    // A ring, in k-tiles; also the unroll of the loop
  static constexpr int KA = RING - KT;              // A k-tiles fetched ahead
  static constexpr int LDS = RING * KTB;
  static constexpr int TOUCH = 256;                 // behind the ring, where a kernel touches: a wave's touches land here, never read
  // fragment registers: R row blocks, read LA ahead (R divides NA: static indices)
  static constexpr int R = NA % 8 == 0 ? 8 : NA % 7 == 0 ? 7 : NA % 6 == 0 ? 6 : NA % 5 == 0 ? 5 : 4;
  static constexpr int LA = R > 6 ? 6 : R - 1;
  static constexpr int BARG = NA - LA + 1;          // row block before which a stage's barrier stands
  static constexpr int GAP = NA * NB / P;           // MFMAs between two global loads
  static_assert(NA % R == 0 && RING % DB == 0 && RING % KT == 0 && GAP >= 2 && NAD * GAP < NA * NB, "schedule");
  // at the start of k-tile kt everything issued in k-tiles <= kt - (DB - 1) has landed (the B wait); the A tiles of
  // the stage published by that k-tile's barrier were issued RING - 2 KT k-tiles earlier
  static_assert(RING - 2 * KT >= DB - 1 && KA >= DB - 1 && (DB - 2) * P <= 63, "waits");
};

// PROBE: one workgroup in the middle of the grid also records shader-clock cycles and 100 MHz
// wall ticks of its prologue, k loop and epilogue into probe[0..7] (a measurement aid: the
// clock under this kernel is set by the chip's power management, not by the nominal 2.4 GHz).

// Wait until at most N younger loads are outstanding; names the registers it releases, which keeps the MFMAs that
// read them behind it.
template <int N>
__device__ __forceinline__ void b_landed(Frag (&b)[NB]) {
  static_assert(N >= 0 && N <= 63 && NB == 4, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%4)" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]) : "n"(N) : "memory");
}

// One TM x 256 output tile (rows m0 .., column tile tn) by the whole 256-thread workgroup.
// NT: weight loads carry the non-temporal hint (see stream_weights).
template <int OUT, int TM, bool NT, bool PROBE, bool TCH>
__device__ __forceinline__ void ring_tile(
    const bf16_t* __restrict__ A, int a_tiled, const bf16_t* __restrict__ Wp, int n, int k, int k_per_split,
    const int M, int m_upper, float* __restrict__ Cf, bf16_t* __restrict__ Cb,
    const int32_t* __restrict__ row_map, size_t ldc, const int m0, const int tn, long long* __restrict__ probe,
    const RopeScatter& rs, const int share, const int tm) {
  typedef TileCfg<TM> TC;
  constexpr int NA = TC::NA, NAD = TC::NAD, P = TC::P, DB = TC::DB, KT = TC::KT, RING = TC::RING, KA = TC::KA, KTB = TC::KTB,
                R = TC::R, LA = TC::LA, BARG = TC::BARG, GAP = TC::GAP;
  extern __shared__ Frag lds[];           // [RING k-tiles][TM/32 row blocks x 2 k halves][64 lanes]

  const int n0 = tn * TILE;
  const int kbeg = blockIdx.y * k_per_split;
  const int ktiles = k_per_split / BK2;             // even, at least RING (k_tiles_ok)
  const int last = ktiles - 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int K16 = k / 16, NF = n / 16;
  const int g4 = lane >> 4;

  // A: wave w moves fragments w, w + 4, .. of a k-tile (fragment f = row block f / 2, k half f % 2), modulo A_FR (a
  // wave without a fragment of its own repeats another wave's load, same bytes to the same place, so that every
  // wave issues the same number of loads and one wait count serves all).  A is row-major [m_upper, k] (a 32 x 16
  // fragment is gathered from 32 rows) or already fragment-tiled (one contiguous 1 KiB block per fragment, rows
  // padded to 32).  Rows past the end read valid ones; their products are never stored.
  // Addresses: 64-bit scalar base of the tile + 32-bit per-lane byte offset.
  uint32_t a_voff[NAD], a_lds[NAD];
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) Frag*)lds);
#pragma unroll
  for (int i = 0; i < NAD; ++i) {
    const int f = (wave + 4 * i) % TC::A_FR;
    if (a_tiled) {
      const int n_mb = (m_upper + 31) / 32, mb0 = m0 / 32;
      const int mb = min(f >> 1, n_mb - 1 - mb0);
      a_voff[i] = (((uint32_t)mb * (uint32_t)K16 + (uint32_t)(f & 1)) * 64u + (uint32_t)lane) * 16u;
    } else {
      const int row = min((f >> 1) * 32 + (lane & 31), m_upper - 1 - m0);
      a_voff[i] = ((uint32_t)row * (uint32_t)k + (uint32_t)((lane >> 5) * 8 + (f & 1) * 16)) * 2u;
    }
    a_lds[i] = lds_base + __builtin_amdgcn_readfirstlane((uint32_t)f * 1024u);
  }
  const uint32_t a_step = a_tiled ? 2048u : BK2 * 2u;                          // bytes per k-tile
  uint64_t pa = (uint64_t)(uintptr_t)A + (a_tiled ? ((uint64_t)(m0 / 32) * (uint32_t)K16 + (uint32_t)(kbeg / 16)) * 1024u
                                                  : ((uint64_t)m0 * (uint32_t)k + (uint32_t)kbeg) * 2u);
  // B: 16-column block b of this wave.  For the Q|K|V launch a wave takes the blocks whose columns RoPE pairs (dims
  // j and j + 64 of a head), otherwise 64 consecutive columns; columns past the end read the last block.
  auto col_block = [&](int b) {                                                // inside the tile
    return OUT == 3 ? (wave >> 1) * 8 + (wave & 1) * 2 + (b & 1) + (b >> 1) * 4 : wave * NB + b;
  };
  uint32_t b_voff[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int f = min(col_block(b), NF - 1 - n0 / 16);
    b_voff[b] = (((uint32_t)(f >> 1) * (uint32_t)K16 + (uint32_t)(g4 >> 1)) * 64u +
                 (uint32_t)((g4 & 1) * 32 + (f & 1) * 16 + (lane & 15))) * 16u;
  }
  uint64_t pb = (uint64_t)(uintptr_t)Wp + ((uint64_t)(n0 / 32) * (uint32_t)K16 + (uint32_t)(kbeg / 16)) * 1024u;

  // Direct-to-LDS loads are issued as inline assembly on purpose: when the compiler sees an LDS-DMA instruction it
  // makes every later LDS read wait for ALL of them (vmcnt(0)), which would collapse the ring to a depth of one.
  // Here the code itself guarantees, with explicit vmcnt waits and the barriers, that a k-tile is read only after
  // its loads have landed.  The hardware writes lane L's 16 bytes at M0 + 16 L; at least one instruction stands
  // between the write of M0 and the load.
  auto set_m0 = [&](int slot, int i) { asm volatile("s_mov_b32 m0, %0" ::"s"(a_lds[i] + (uint32_t)(slot * KTB)) : "m0"); };
  auto issue_a = [&](int i) { asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(a_voff[i]), "s"(pa) : "memory", "m0"); };
  // Register-ring contract.  The compiler cannot see that a register is still being written after the load has
  // issued, so nothing may give it a reason to touch fb between a load and the b_landed that waits for it:
  //  * the ring registers are read-write operands of both the load and the wait, i.e. one live value from the first
  //    load to the wait that follows it, and the loads past the last k-tile (re-fetches of it) are waited for by
  //    name after the loop;
  //  * the loop must hold no register copy or spill: the build fails if the compiler reports scratch for this kernel.
  Frag fb[DB][NB];
#pragma unroll
  for (int u = 0; u < DB; ++u)
#pragma unroll
    for (int b = 0; b < NB; ++b) fb[u][b] = Frag{};
  auto issue_b = [&](int slot, int b) {
    if constexpr (NT) asm volatile("global_load_dwordx4 %0, %1, %2 nt" : "+v"(fb[slot][b]) : "v"(b_voff[b]), "s"(pb) : "memory");
    else asm volatile("global_load_dwordx4 %0, %1, %2" : "+v"(fb[slot][b]) : "v"(b_voff[b]), "s"(pb) : "memory");
  };
  // next k-tile to fetch; past the end the last one again (never used)
  int kt_a = 0, kt_b = 0;
  auto next_a = [&] { pa += kt_a < last ? a_step : 0u; ++kt_a; };
  auto next_b = [&] { pb += kt_b < last ? 2048u : 0u; ++kt_b; };

  // acc[a][b]: rows 16a .., block b; lane l holds row l % 16, columns 4 * (l / 16) .. +3
  f32x4 acc[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  // From intrinsics the compiler shuffles accumulators through register copies in this loop (hundreds per trip); as
  // assembly with a read-write accumulator it cannot.  It then does not know the result latency either: the wait
  // states before the first use and after the last are written out.
  auto mma = [&](const Frag& bf, const Frag& af, f32x4& c) {
    asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(bf), "v"(af));
  };

  // 16 x 32 operand out of the 32 x 16 blocks in LDS: lane l wants row l % 16 and the 8 k of group g = l / 16, i.e.
  // slot (l % 16) + 32 * (g % 2) of k-block g / 2; a second 16-row half of a block is 16 slots further on
  typedef const __attribute__((address_space(3))) Frag LFrag;
  constexpr int HALF = 64 * 1024 / KTB < RING ? 64 * 1024 / KTB : RING;      // k-tiles one 16-bit offset reaches
  LFrag* sa_lo = (LFrag*)lds + (lane >> 5) * 64 + (g4 & 1) * 32 + (lane & 15);
  LFrag* sa_hi = sa_lo + HALF * (KTB / 16);
  asm volatile("" : "+v"(sa_lo), "+v"(sa_hi));      // two base registers, not one address addition per read
  auto a_frag = [&](int slot, int a) -> Frag {
    static_assert(2 * HALF >= RING, "two bases reach the ring");
    const int o = (slot % HALF) * (KTB / 16) + (a >> 1) * 128 + (a & 1) * 16;
    return slot < HALF ? sa_lo[o] : sa_hi[o];
  };
  Frag af[R];

  // Touches (TCH; share > 2 row tiles that hold rows run side by side on one XCD and want the same weights): a lane reads four
  // bytes of a 128-byte line, a wave the 64 lines of 32 columns and four k-tiles, two such chunks ahead of the loads of the k-tile
  // it is issued in.  Chunk p's 8 column blocks are dealt over the 4 share waves; t_x counts down to this wave's next one.
  // They count in vmcnt like any load and make its waits, which ignore them, no looser.  Kernels of their own: in the others the
  // few scalar instructions cost (gate|up of 700 rows, 160-row tiles that never touch, 124 -> 130 us).
  const uint32_t t_voff = (uint32_t)lane * 128u;
  const uint32_t t_lds = lds_base + (uint32_t)(RING * KTB) + (uint32_t)__builtin_amdgcn_readfirstlane(wave) * TC::TOUCH;
  const int t_blocks = min(8, NF / 2 - n0 / 32);
  int t_x = __builtin_amdgcn_readfirstlane(wave * share + tm);
  // Two under a larger bound lose by it (a block with cold weights: 140 and 224 rows bounded by 896 + 1 %, by 2048 + 2 %), three do not
  // (300 rows bounded by 2048 - 3 %).
  int t_left = share > 2 ? ktiles / 4 - 1 : 0;      // whole chunks after the first, which the prologue fetches
  uint64_t pt = pb + 8192u;
  auto touch = [&] {
    if constexpr (TCH) {
      if (t_left <= 0) return;
      if (t_x < t_blocks)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(t_lds), "v"(t_voff),
                     "s"(pt + (uint64_t)((uint32_t)t_x * (uint32_t)K16) * 1024u) : "memory", "m0");
      t_x -= 8;
      if (t_x < 0) t_x += 4 * share;
      pt += 8192u;
      --t_left;
    }
  };

  long long pc0 = 0, pw0 = 0, pc1 = 0, pw1 = 0, pc2 = 0, pw2 = 0;
  if (PROBE) { pc0 = clock64(); pw0 = wall_clock64(); }
  touch();
  // prologue: loads in the order in which the loop would have issued them
#pragma unroll
  for (int j = 0; j < KA; ++j) {
#pragma unroll
    for (int i = 0; i < NAD; ++i) {
      set_m0(j, i);
      asm volatile("s_nop 0");
      issue_a(i);
    }
    next_a();
    if (j >= KA - (DB - 1)) {
#pragma unroll
      for (int b = 0; b < NB; ++b) issue_b(j - (KA - (DB - 1)), b);
      next_b();
    }
  }
  b_landed<(DB - 2) * P>(fb[0]);
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int a = 0; a < LA; ++a) af[a] = a_frag(0, a);
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) asm volatile("" : "+a"(acc[a][b]));          // zeroed before the wait states
  asm volatile("s_nop 7" ::: "memory");
  if (PROBE) { pc1 = clock64(); pw1 = wall_clock64(); }

  // One k-tile per step u: A tile kt + KA into the LDS slot whose readers passed the previous barrier, B tile
  // kt + DB - 1 into the registers of tile kt - 1.  sched_barrier(0) keeps the order written here.
  for (int kt = 0; kt < ktiles; kt += RING) {
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      if (u > 0 && u % 2 == 0 && kt + u >= ktiles) break;
      const int slot_b = u % DB, fetch_b = (u + DB - 1) % DB, fetch_a = (u + KA) % RING, next = (u + 1) % RING;
      const bool publish = u % KT == KT - 1;
      if (u % 4 == 0) touch();
      b_landed<(DB - 2) * P>(fb[slot_b]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < NA * NB; ++q) {
        const int a = q / NB, o = q / GAP;
        if (publish && q == BARG * NB) {
          // every wave has read the last of this stage, and its own loads of the next one have landed
          asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        mma(fb[slot_b][q % NB], af[a % R], acc[a][q % NB]);
        if (q % NB == NB - 1) {                     // after the last use of af[a % R]
          if (a + LA < NA) af[(a + LA) % R] = a_frag(u, a + LA);
          else if (!publish || a > BARG) af[(a + LA) % R] = a_frag(next, a + LA - NA);
          else if (a == BARG) {
#pragma unroll
            for (int x = NA - LA; x <= BARG; ++x) af[(x + LA) % R] = a_frag(next, x + LA - NA);
          }
        }
        if (o < P && q % GAP == GAP - 1) {
          if (o < NAD) issue_a(o);
          else issue_b(fetch_b, o - NAD);
        }
        if (o < NAD && q % GAP == GAP - 2) set_m0(fetch_a, o);
        if (q == NAD * GAP) next_a();
        __builtin_amdgcn_sched_barrier(0);
      }
      next_b();
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (PROBE) { pc2 = clock64(); pw2 = wall_clock64(); }
#pragma unroll
  for (int u = 0; u < DB; ++u) b_landed<0>(fb[u]);  // drain the (unused) tail re-fetches, registers named
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) asm volatile("" : "+a"(acc[a][b]));

  const int row_in = lane & 15;
  if constexpr (OUT == 0) {
    // fp32 partial plane of this k-split: 16 bytes per lane, 64 contiguous bytes per row and block
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const int row = m0 + a * 16 + row_in;
      if (row >= M) continue;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int col = n0 + (wave * NB + b) * 16 + 4 * g4;
        if (col < n) *reinterpret_cast<f32x4*>(Cf + ((size_t)blockIdx.y * m_upper + row) * ldc + col) = acc[a][b];
      }
    }
    return;
  }
  if constexpr (OUT == 1) {
    // bf16 rows.  Streaming stores: these rows (the step's logits, 259 MB at M = 1024) are read once by the next
    // kernel and would otherwise sit dirty in the memory-side cache and be written back under that kernel's reads
    // (scoring 111 -> 99 us)
    // The rows leave through LDS (a wave's own corner of the drained ring), eight rows of a whole 128-byte line each per
    // instruction: stored from the accumulators' layout, half lines at a time, the launch wrote 1.45 times its bytes.
    // One map entry per thread, all at once.  LM head, both forms of the stores on one box (weights still hinted): 8192 rows
    // 6164 -> 5878 us, 1024 rows 800 -> 781, 512 rows 489 -> 466.
    __syncthreads();
    int* row_sh = reinterpret_cast<int*>(lds);        // [TM] output row, -1 past M
    {
      const int r = threadIdx.x, row = m0 + r;
      if (r < TM) row_sh[r] = row < M ? (row_map ? row_map[row] : row) : -1;
    }
    __syncthreads();
    constexpr int RS = 9;                             // 16-byte pieces per staged row: eight and one of padding
    static_assert(TM * 4 + 4 * 2 * 16 * RS * 16 <= TC::LDS, "staging fits the ring");
    uint4* stage = reinterpret_cast<uint4*>(row_sh + TM) + wave * 2 * 16 * RS;
    const int wp = row_in * RS + (g4 & 1) * 2 + (g4 >> 1), rl = lane >> 3, c0 = n0 + wave * 64 + (lane & 7) * 8;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
#pragma unroll
      for (int b = 0; b < NB; ++b) asm volatile("" : "+a"(acc[a][b]));     // read here, not all at once ahead (spills)
      uint4* st = stage + (a & 1) * 16 * RS;
      st[wp] = pack_swap(acc[a][0], acc[a][1]);
      st[wp + 4] = pack_swap(acc[a][2], acc[a][3]);
      asm volatile("" ::: "memory");                  // written by other lanes of the wave: LDS keeps a wave's order
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint4 v = st[(rl + 8 * h) * RS + (lane & 7)];
        const int orow = row_sh[a * 16 + rl + 8 * h];
        if (orow >= 0 && c0 < n) __builtin_nontemporal_store(__builtin_bit_cast(Frag, v), reinterpret_cast<Frag*>(Cb + (size_t)orow * ldc + c0));
      }
      asm volatile("" ::: "memory");
    }
    if (PROBE) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // the stores have left
      const long long pc3 = clock64(), pw3 = wall_clock64();
      if (blockIdx.x == ((gridDim.x >> 1) & ~7u) && threadIdx.x == 0) {
        probe[0] = pc1 - pc0; probe[1] = pc2 - pc1; probe[2] = pc3 - pc2;
        probe[3] = pw1 - pw0; probe[4] = pw2 - pw1; probe[5] = pw3 - pw2;
        probe[6] = gridDim.x; probe[7] = ktiles;
      }
    }
    return;
  }
  if constexpr (OUT == 4) {
    // residual add in the epilogue: Cb [m, n] row-major <- rnd(Cb + sums) in place (each element belongs to exactly
    // one workgroup, which reads it before it writes it).  All of a wave's rows are requested before the first is
    // needed (rows and columns past the end: valid ones, not stored).
    const int c0 = n0 + wave * 64 + (g4 & 1) * 16 + (g4 >> 1) * 8;
    Frag x[NA][2];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const bf16_t* p = Cb + (size_t)min(m0 + a * 16 + row_in, M - 1) * ldc;
#pragma unroll
      for (int h = 0; h < 2; ++h) x[a][h] = *reinterpret_cast<const Frag*>(p + min(c0 + 32 * h, n - 8));
    }
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const int row = m0 + a * 16 + row_in;
      bf16_t* p = Cb + (size_t)row * ldc + c0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        Frag v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[a][2 * h][e]), __float_as_uint(acc[a][2 * h + 1][e]), false, false);
          v[e] = (bf16_t)((float)x[a][h][e] + __uint_as_float(w[0]));
          v[4 + e] = (bf16_t)((float)x[a][h][4 + e] + __uint_as_float(w[1]));
        }
        if (row < M && c0 + 32 * h < n) *reinterpret_cast<Frag*>(p + 32 * h) = v;      // read again by the norm kernel
      }
    }
    return;
  }
  if constexpr (OUT == 2) {
    // columns are gate/up interleaved by 32-column blocks: of a wave's 64 columns the first 32 are gate columns
    // c .. c+31 and the last 32 the up columns of the same c (n = 2 d_ff, ldc = d_ff), so accumulators b and b+2 of
    // a lane pair up; eight consecutive columns of a row are one 16-byte unit of the fragment-tiled layout.
    const int c = (n0 / 64 + wave) * 32 + (g4 & 1) * 16 + (g4 >> 1) * 8;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const int row = m0 + a * 16 + row_in;
      float gs[8], us[8], y[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        gs[e] = acc[a][e >> 2][e & 3];
        us[e] = acc[a][(e >> 2) + 2][e & 3];
      }
      silu_mul(gs, us, y);
      const uint4 o = pack_swap(f32x4{y[0], y[1], y[2], y[3]}, f32x4{y[4], y[5], y[6], y[7]});
      if (row < M && c < (n >> 1)) *reinterpret_cast<uint4*>(Cb + afrag_index(row, c, (int)ldc)) = o;
    }
    return;
  }
  if constexpr (OUT == 3) {
    // n = 3 H 128 columns = [q | k | v], each a whole number of 256-column tiles: this tile holds two heads of one of
    // the three, a wave 32 dims j of one of them (blocks 0, 1) and dims j + 64 (blocks 2, 3), so RoPE, which pairs
    // them, stays inside a lane.  It is applied to the unrounded sums, like the stand-alone kernel does.
    const int hd = rs.H * 128;
    const int sec = n0 / hd;                          // 0 q, 1 k, 2 v
    if (sec > 0 && rs.kc == nullptr) return;          // queries only (uniform over the workgroup)
    const int head = ((n0 - sec * hd) >> 7) + (wave >> 1), j0 = (wave & 1) * 32;
    // the ring is drained: its space holds each row's flat id, sequence and slot (-1 past M)
    __syncthreads();
    int* row_sh = reinterpret_cast<int*>(lds);        // [TM] flat id, [TM] sequence, [TM] slot
    scatter_rows_of_tile(row_sh, TM, m0, M, rs);
    __syncthreads();
    if (sec < 2) {
#pragma unroll
      for (int a = 0; a < NA; ++a) {
#pragma unroll
        for (int b = 0; b < NB; ++b) asm volatile("" : "+a"(acc[a][b]));     // read here, not all at once ahead (spills)
        const int r = a * 16 + row_in;
        if (row_sh[r] < 0) continue;
        float4 tab[4];
        rope_load_row(tab, row_sh[2 * TM + r], j0, rs);
        rope_store_row(acc[a], tab, sec, head, j0, m0 + r, row_sh[TM + r], row_sh[2 * TM + r], rs);
      }
    } else {
      // half of the tile's rows at a time
      constexpr int GR = (NA + 1) / 2;                // 16-row groups per pass
      static_assert(3 * TM * 4 + 4 * GR * 16 * VSTAGE * 2 <= TC::LDS, "staging fits the ring");
      bf16_t* stage = reinterpret_cast<bf16_t*>(row_sh + 3 * TM) + wave * GR * 16 * VSTAGE;
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
        constexpr int G0 = GR;
        const int groups = pass == 0 ? G0 : NA - G0;
#pragma unroll
        for (int a = 0; a < GR; ++a) {
          if (pass * GR + a >= NA) continue;
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            f32x4& c = acc[pass * GR + a < NA ? pass * GR + a : 0][b];
            asm volatile("" : "+a"(c));
            v_stage_block(stage, a * 16 + row_in, b, c);
          }
        }
#pragma unroll 1
        for (int a = 0; a < groups; ++a) {
          const int r = (pass * GR + a) * 16 + row_in;
          v_store_rows(stage + a * 16 * VSTAGE, row_sh[TM + r], row_sh[2 * TM + r], head, j0, rs);
        }
      }
    }
  }
}

// Workgroup -> tile.  Consecutive workgroups go to consecutive XCDs (blockIdx.x = 8 * j + xcd), each with an
// L2 of its own that holds a few k-steps of the ~32 tiles its CUs work on at a time; XCD x owns the column
// tiles 8 c + x.  Operand bytes that leave an L2 are about (distinct row tiles + distinct column tiles) among
// those 32, per k-step: 33 when an XCD walks down one column tile after the other, 12 for 8 x 4 tiles.  An
// XCD therefore walks bands of gn of its column tiles, column fastest, so that the tiles in flight form a
// block of about (32 / gn) x gn.  Measured at 8192 rows: L2 fetch bytes of the layer projections halve from
// gn = 1 to gn = 4 and the launches get 2 to 5 % faster; wider bands and splitting the rows over XCDs
// (which fetches every weight tile into several L2s) are slower at few row tiles.
struct TileMap {
  int gn, cn;        // band width; column tiles per XCD
};
__device__ inline bool tile_of_workgroup(const TileMap& tmap, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int full = tmap.cn / tmap.gn * tmap.gn;     // column tiles in whole bands
  int c;
  if (j < tiles_m * full) {
    const int band = j / (tiles_m * tmap.gn), q = j - band * tiles_m * tmap.gn;
    tm = q / tmap.gn;
    c = band * tmap.gn + q % tmap.gn;
  } else {
    const int q = j - tiles_m * full, w = tmap.cn - full;
    tm = q / w;
    c = full + q % w;
  }
  tn = c * 8 + xcd;
  return tm < tiles_m && tn < tiles_n;
}
static TileMap pick_tile_map(int tiles_m, int tiles_n) {
  const int cn = sl_cdiv(tiles_n, 8), gn = tiles_m >= 16 ? 4 : 2;
  return TileMap{gn < cn ? gn : cn, cn};
}

template <int OUT, int TM, bool NT, bool PROBE = false, bool TCH = false>
__global__ __launch_bounds__(256, 1) void gemm_mfma256_kernel(
    const bf16_t* __restrict__ A, int a_tiled, const bf16_t* __restrict__ Wp, int n, int k, int k_per_split,
    const int32_t* __restrict__ m_dev, int m_upper, float* __restrict__ Cf, bf16_t* __restrict__ Cb,
    const int32_t* __restrict__ row_map, size_t ldc, int tiles_m, int tiles_n, TileMap tmap,
    long long* __restrict__ probe, RopeScatter rs) {
  const int M = min(*m_dev, m_upper);
  int tm, tn;
  if (!tile_of_workgroup(tmap, tiles_m, tiles_n, tm, tn) || tm * TM >= M) return;
  ring_tile<OUT, TM, NT, PROBE, TCH>(A, a_tiled, Wp, n, k, k_per_split, M, m_upper, Cf, Cb, row_map, ldc, tm * TM, tn, probe, rs,
                                 TCH ? (M + TM - 1) / TM : 0, tm);
}

// Workgroup slots a launch takes on the chip's 256 CUs.  Column tiles go to the XCDs in turn, so the XCD with the most of
// them (32 CUs) decides how many rounds there are, and the slots it leaves empty elsewhere count.
static int ring_slots(int tiles_m, int tiles_n, int splits) { return 8 * tiles_m * sl_cdiv(tiles_n, 8) * splits; }

// Whether a launch's weight loads carry the non-temporal hint.  With one row tile a weight line is wanted once, and in one
// round of workgroups the row tiles of a column want it at about the same time: the hint keeps the weights from pushing
// activations and planes out of the caches (one row tile, LM head of 64 rows: 168 us with it, 194 without; one round, Q|K|V
// of 576 rows: 65 and 68).  From the second round on the workgroups of a column have drifted apart and a line marked for
// eviction is gone before the next one asks.  Short tiles live on those lines: gate|up of 576 rows 131 us with, 105 without,
// 700 rows 143 / 117; LM head of 288 rows 329 / 275, Q|K|V of 2600 rows 293 / 226.  Taller tiles have the arithmetic to hide
// it until more than 3072 rows share the lines: LM head of 4654 rows 3714 / 3217, of 8192 rows 5882 / 5659, gate|up 654 / 637
// and 1111 / 1090; at 2304 rows gate|up gains 3 us and the down projection behind it loses 13, its activations evicted.
static bool stream_weights(int tiles_m, int tiles_n, int splits, int tm) {
  if (tiles_m == 1 || ring_slots(tiles_m, tiles_n, splits) <= 256) return true;
  return tm > 160 && tiles_m * tm <= 3072;
}

// Whether the row tiles of a launch touch each other's weights ahead of their loads.  A CU keeps about 256 lines under way, a
// line that misses its L2 for 625 ns, one that hits for 250.  In one round of workgroups the R row tiles of a column run side by
// side on one XCD, ask for a weight line together and all wait for it; with each touching 1/R of the lines a few k-tiles ahead
// (four bytes a line) all but one find them in L2.  It pays where short tiles wait for lines and many share them.  Weights out of
// HBM, us without -> with: down of 1024 rows (128 x 8, two splits) 95 -> 86, 2048 rows (128 x 16) 164 -> 149, Out of 768 rows
// (128 x 6) 34.2 -> 32.0, 1536 rows (128 x 12) 55 -> 48; 202 launches of six and more row tiles (n = 1024 .. 8192, k = 512 .. 12288,
// 576 .. 2048 rows) gain 6 % on average, up to 23 %.  Four tiles of 128 rows gain as well (n = 3072 .. 16384, k = 2048 .. 12288: 4 % on
// average, Q|K|V of 512 rows 58 -> 51), other heights and fewer sharers do not: Q|K|V of 544 rows (128 x 5) 63.5 -> 66, 704 rows
// (160 x 5) 73 -> 75, 960 rows (192 x 5) 83.5 -> 86, gate|up of 512 rows (256 x 2) 84 -> 92; 96-row tiles of four or five gain 2 to 4 us in
// Q|K|V of 390 to 430 rows and the launches behind them lose it.  Tall tiles have fewer lines to wait for per MFMA and lose over
// short reductions (160 x 8, n = 8192, k = 512 and 1024 14.3 -> 14.9 and 21.4 -> 22.9); over longer ones they gain or are equal within the
// runs of one size (down of 1280 rows 103 -> 101; Out of 1280 rows alone 40.4 -> 41.3, but six layers of 600 rows bounded by 1280 2655 ->
// 2642).
// 128-row tiles over a short reduction, split so that they fill the chip, lose too: n = 4096, k = 2048 in two of 1024 rows 22.7 -> 23.9,
// n = 7168 of 416 rows 21.1 -> 22.4, n = 3072 in four 15.8 -> 16.7; with fewer workgroups they gain (n = 5120 in two, 512 rows 21.5 ->
// 20.7), and so do shorter tiles (n = 2048 in two, 64 x 14 16.7 -> 15.0).
// The touches carry no non-temporal hint: with it the lines are gone before they are read (Q|K|V of 512 rows 69).
static bool touches_weights(int tiles_m, int tiles_n, int splits, int tm, int k) {
  if (ring_slots(tiles_m, tiles_n, splits) > 256) return false;
  if (tm == 128 && splits > 1 && k / splits <= 1024 && tiles_m * tiles_n * splits >= 192) return false;
  if (tm == 160) return tiles_m >= 6 && k / splits >= 2048;
  return tm < 160 && (tiles_m >= 6 || (tm == 128 && tiles_m == 4));
}

template <int OUT, int TM, bool NT, bool TCH = false>
static int launch_ring_hint(hipStream_t s, const void* A, int a_tiled, const void* Wp, const int32_t* m_dev, int mu, int n, int k,
                       int splits, float* Cf, void* Cb, const int32_t* row_map, size_t ldc, const RopeScatter& rs) {
  const int tiles_m = sl_cdiv(mu, TM), tiles_n = sl_cdiv(n, TILE);
  const size_t sh = TileCfg<TM>::LDS + (TCH ? 4 * TileCfg<TM>::TOUCH : 0);
  auto kern = gemm_mfma256_kernel<OUT, TM, NT, false, TCH>;
  static unsigned long long lds_ok = 0;              // one per kernel instantiation
  SL_ALLOW_DYNAMIC_LDS(lds_ok, kern, sh);
  const TileMap tmap = pick_tile_map(tiles_m, tiles_n);
  dim3 grid(8 * tiles_m * tmap.cn, splits), block(256);
  hipLaunchKernelGGL(kern, grid, block, sh, s, (const bf16_t*)A, a_tiled, (const bf16_t*)Wp, n, k, k / splits, m_dev, mu, Cf,
                     (bf16_t*)Cb, row_map, ldc, tiles_m, tiles_n, tmap, (long long*)nullptr, rs);
  SL_LAUNCH_CHECK();
  return SL_OK;
}
template <int OUT, int TM>
static int launch_ring(hipStream_t s, const void* A, int a_tiled, const void* Wp, const int32_t* m_dev, int mu, int n, int k,
                       int splits, float* Cf, void* Cb, const int32_t* row_map, size_t ldc, const RopeScatter& rs) {
  if constexpr (TM <= 160) {                          // one round of workgroups: hinted
    if (touches_weights(sl_cdiv(mu, TM), sl_cdiv(n, TILE), splits, TM, k))
      return launch_ring_hint<OUT, TM, true, true>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
  }
  return stream_weights(sl_cdiv(mu, TM), sl_cdiv(n, TILE), splits, TM)
             ? launch_ring_hint<OUT, TM, true>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs)
             : launch_ring_hint<OUT, TM, false>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
}

// ---- tile heights of a launch ------------------------------------------------------------------
// Cost model in units of one full-height tile's time on 256 CUs: a full round of workgroups costs 1, a last partial
// round nearly the same whatever its fill (measured: the busy CUs of a partial round run at a higher clock), a tile
// of TM rows kTileCost[TM / 32] of a full one.  The constants are those for which the choices of height and split come
// nearest to the fastest launch of each size in a sweep of 88 sizes (n = 4096 .. 126464, k = 4096 and 12288, 40 .. 2048
// rows, weights out of HBM, every height and split): 1.7 % above it on average.  The narrow matrices take shorter tiles
// than when a partial round cost the same at any fill: n = k = 4096, 128 rows 128 x 8 splits 20.3 us -> 64 x 8 17.6,
// 224 rows 128 x 4 24.7 -> 64 x 4 21.4; n = 4096, k = 12288, 128 rows 36.8 -> 31.5, 1280 rows 192 x 2 118 -> 160 x 2 111.
// A launch runs uniform tiles of one height (any multiple of 32 from 64 to 256): the smallest number of
// row tiles that covers the rows, or more and shorter ones where that saves a round of workgroups.
// Fewer, taller tiles win near-ties (less operand traffic per flop).
static double ring_rounds_cost(int slots) {
  const int rest = slots % 256;
  return slots / 256 + (rest ? 0.9 + 0.025 * rest / 256.0 : 0.0);
}
static const double kTileCost[9] = {0, 0, 0.485, 0.55, 0.56, 0.70, 0.795, 0.86, 1.0};   // by TM / 32

struct RingChoice {
  int tm;          // rows per tile
  double cost;     // in full-tile rounds
};
static RingChoice ring_choice(int mu, int n, int splits) {
  RingChoice best{256, 1e30};
  const int t_min = sl_cdiv(mu, 256), t_max = sl_cdiv(mu, 64);
  for (int t = t_min; t <= t_max; ++t) {
    int tm = (int)sl_align_up((size_t)sl_cdiv(mu, t), 32);
    if (tm < 64) tm = 64;
    if (sl_cdiv(mu, tm) != t) continue;              // the same height with fewer tiles was already priced
    const double c = ring_rounds_cost(ring_slots(t, sl_cdiv(n, TILE), splits)) * kTileCost[tm / 32];
    if (c < 0.99 * best.cost) best = RingChoice{tm, c};
  }
  return best;
}

// cost of the cheapest ring launch for (mu rows, n columns, `splits` k-splits), in full-tile rounds
double slk_ring_cost(int mu, int n, int splits) { return ring_choice(mu, n, splits).cost; }
int slk_ring_tile_rows(int mu, int n, int splits) { return ring_choice(mu, n, splits).tm; }

template <int OUT>
static int launch256(hipStream_t s, const void* A, int a_tiled, const void* Wp, const int32_t* m_dev, int mu, int n, int k,
                     int splits, float* Cf, void* Cb, const int32_t* row_map, size_t ldc,
                     const RopeScatter& rs = RopeScatter{}) {
  const RingChoice c = ring_choice(mu, n, splits);
  switch (c.tm) {
    case 64: return launch_ring<OUT, 64>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
    case 96: return launch_ring<OUT, 96>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
    case 128: return launch_ring<OUT, 128>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
    case 160: return launch_ring<OUT, 160>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
    case 192: return launch_ring<OUT, 192>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
    case 224: return launch_ring<OUT, 224>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
    default: return launch_ring<OUT, 256>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, Cb, row_map, ldc, rs);
  }
}

// The k loop takes k-tiles in pairs (an odd last one would be added twice) and its prologue wants a ring of them.
static bool k_tiles_ok(int k, int splits) { return k % (2 * BK2 * splits) == 0 && k / (BK2 * splits) >= 8; }

int slk_gemm_mfma256(hipStream_t s, const void* A, int a_tiled, const void* Wp, const int32_t* m_dev, int mu, int n,
                     int k, int splits, float* Cf, void* Cb, const int32_t* row_map, size_t ldc) {
  if (mu <= 0) return SL_OK;
  if (splits < 1 || n % 32 || !k_tiles_ok(k, splits)) return SL_EINVAL;
  if (!Cf && splits != 1) return SL_EINVAL;
  if (Cf && ((uintptr_t)Cf % 16 || ldc % 4)) return SL_EINVAL;       // 16-byte fp32 stores
  if ((size_t)n * k >= ((size_t)1 << 31) * 8 || (size_t)mu * k >= ((size_t)1 << 32)) return SL_EINVAL;
  return Cf ? launch256<0>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, Cf, nullptr, nullptr, ldc)
            : launch256<1>(s, A, a_tiled, Wp, m_dev, mu, n, k, splits, nullptr, Cb, row_map, ldc);
}

// The LM-head launch (bf16 rows, no split) with the cycle probe switched on; probe = 8 int64 on the device.
template <bool NT>
static int launch_probe(hipStream_t s, const void* A, int a_tiled, const void* Wp, const int32_t* m_dev, int mu, int n, int k,
                        void* Cb, const int32_t* row_map, size_t ldc, long long* probe) {
  const int tiles_m = sl_cdiv(mu, TILE), tiles_n = sl_cdiv(n, TILE);
  const size_t sh = TileCfg<256>::LDS;
  auto kern = gemm_mfma256_kernel<1, 256, NT, true>;
  static unsigned long long lds_ok = 0;
  SL_ALLOW_DYNAMIC_LDS(lds_ok, kern, sh);
  const TileMap tmap = pick_tile_map(tiles_m, tiles_n);
  dim3 grid(8 * tiles_m * tmap.cn, 1), block(256);
  hipLaunchKernelGGL(kern, grid, block, sh, s, (const bf16_t*)A, a_tiled, (const bf16_t*)Wp, n, k, k, m_dev, mu,
                     (float*)nullptr, (bf16_t*)Cb, row_map, ldc, tiles_m, tiles_n, tmap, probe, RopeScatter{});
  SL_LAUNCH_CHECK();
  return SL_OK;
}
int slk_gemm_mfma256_probe(hipStream_t s, const void* A, int a_tiled, const void* Wp, const int32_t* m_dev, int mu, int n,
                           int k, void* Cb, const int32_t* row_map, size_t ldc, long long* probe) {
  if (mu <= 0 || !probe || !Cb) return SL_EINVAL;
  if (n % 32 || !k_tiles_ok(k, 1)) return SL_EINVAL;
  if ((size_t)n * k >= ((size_t)1 << 31) * 8 || (size_t)mu * k >= ((size_t)1 << 32)) return SL_EINVAL;
  return stream_weights(sl_cdiv(mu, TILE), sl_cdiv(n, TILE), 1, TILE)
             ? launch_probe<true>(s, A, a_tiled, Wp, m_dev, mu, n, k, Cb, row_map, ldc, probe)
             : launch_probe<false>(s, A, a_tiled, Wp, m_dev, mu, n, k, Cb, row_map, ldc, probe);
}

int slk_gemm_mfma256_swiglu(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int dff, int k,
                            void* a) {
  if (mu <= 0) return SL_OK;
  const int n = 2 * dff;
  if (dff % 32 || !k_tiles_ok(k, 1)) return SL_EINVAL;
  if ((size_t)n * k >= ((size_t)1 << 31) * 8 || (size_t)mu * k >= ((size_t)1 << 32)) return SL_EINVAL;
  return launch256<2>(s, A, 1, Wp, m_dev, mu, n, k, 1, nullptr, a, nullptr, (size_t)dff);
}

// Q|K|V projection + RoPE + scatter in one launch: q [mu, H*128] packed bf16, K / V into the layer's
// cache at the rows' own slots (kc = vc = null: queries only).  Unsplit only; H even, so
// that a 256-column tile is two whole heads of q, k or v.
int slk_gemm_mfma256_qkv_rope(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int H, int k,
                              const int32_t* active_idx, int N, int n_pad, const void* rope_tab, void* q, void* kc,
                              void* vc) {
  if (mu <= 0) return SL_OK;
  const int n = 3 * H * 128;
  if (H < 2 || H % 2 || !k_tiles_ok(k, 1) || !active_idx || !rope_tab || !q) return SL_EINVAL;
  if ((kc == nullptr) != (vc == nullptr)) return SL_EINVAL;
  if ((uintptr_t)q % 16 || (uintptr_t)kc % 16 || (uintptr_t)vc % 16 || (uintptr_t)rope_tab % 16) return SL_EINVAL;
  if ((size_t)n * k >= ((size_t)1 << 31) * 8 || (size_t)mu * k >= ((size_t)1 << 32)) return SL_EINVAL;
  const RopeScatter rs{active_idx, (const float2*)rope_tab, (bf16_t*)q, (bf16_t*)kc, (bf16_t*)vc, N, n_pad, H};
  return launch256<3>(s, A, 1, Wp, m_dev, mu, n, k, 1, nullptr, nullptr, nullptr, (size_t)n, rs);
}

// x [mu, n] bf16 row-major <- rnd(x + A W^T) in place: a projection with the residual add in its
// epilogue (unsplit only; n % 8 == 0 for the 16-byte row pieces).
int slk_gemm_mfma256_residual(hipStream_t s, const void* A, const void* Wp, const int32_t* m_dev, int mu, int n, int k,
                              void* x) {
  if (mu <= 0) return SL_OK;
  if (n % 32 || !k_tiles_ok(k, 1) || !x || (uintptr_t)x % 16) return SL_EINVAL;
  if ((size_t)n * k >= ((size_t)1 << 31) * 8 || (size_t)mu * k >= ((size_t)1 << 32)) return SL_EINVAL;
  return launch256<4>(s, A, 1, Wp, m_dev, mu, n, k, 1, nullptr, x, nullptr, (size_t)n);
}
