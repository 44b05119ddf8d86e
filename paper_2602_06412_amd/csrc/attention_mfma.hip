// Bidirectional M x N attention of the active rows on the MFMA units (bf16, d_h = 128):
//   o[r, h] = softmax(q[r, h] . K[b, h, 0..N)^T / sqrt(d_h)) V[b, h, 0..N)
// for the packed active rows r of each sequence b against ALL N cached slots of that
// sequence, no mask (Alg. 1 'attention' line; Sec. 2.1: locked slots are served from the
// cache, live slots were just overwritten by this step's K/V write).
//
// Flash-style, computed transposed so that softmax statistics live in one lane:
//   S^T[key, q] = K Q^T   (MFMA A = K fragment from LDS, B = Q^T fragment kept in registers)
//   lane l of the accumulator owns query q = l%32 and 16 keys per 32-key block, so the row
//   max / sum of the online softmax need one cross-lane exchange (lanes l, l^32) only;
//   O^T[dim, q] += V^T P^T  (A = V^T fragment from LDS, B = P^T = the accumulator registers
//   of the first product rounded to half precision, used in place: no LDS round trip, no
//   transpose).
// The K/V cache layouts (kc_index / vc_index) make every fragment of a 64-slot tile a
// contiguous block, so a tile is a straight 16 KiB + 16 KiB copy into LDS.
//
// Precision of P.  The second product runs on half-precision operands: V is cached as the half
// image of its bf16 values (vcache_half_bits: exact in the range activations live in), P is
// rounded to half precision (11 significant bits, round to nearest even) by the two thick-launch
// kernels and carried as a pair of halves (22 bits) by the thin one, where the second half costs
// nothing.  One bf16 value per probability (8 bits, what a plain bf16 attention does) is not
// enough against an fp64 softmax: measured on one full-size layer, the rms error of the logits
// grows by 17 % with bf16 probabilities, by 5-8 % with one half, by nothing with two; the largest
// error and the share of logits beyond 2e-2 stay where the bf16 roundings of the activations put
// them with one half or two.
//
// One workgroup = 4 waves x 32 queries of ONE sequence and one head; packed rows of
// different sequences never share a tile (the varlen case of a ragged batch).
#include "sl_common.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

typedef bf16x8 FragA;       // one lane's 16-byte share of an MFMA operand fragment

constexpr int QT = 128;          // queries per workgroup
constexpr int KT = 64;           // slots per K/V tile
constexpr int DH = 128;
constexpr int kMaxBatch = SL_MAX_BATCH;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
constexpr float kMaxLag = 8.0f;   // probabilities may exceed 1 by up to 2^8 before the reference moves
typedef uint32_t PFrag __attribute__((ext_vector_type(4)));   // eight half-precision probabilities, packed in pairs

// O^T += V^T P^T on one fragment pair: V is cached as half-precision images of its bf16 values, P is
// rounded to half precision (see the kernels), the product accumulates in fp32.
__device__ inline f32x16 mfma_pv(const FragA& v, const PFrag& p, const f32x16& acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, v), __builtin_bit_cast(f16x8, p), acc, 0, 0, 0);
}
// Two probabilities as a packed pair of halves, round to nearest even.
__device__ inline uint32_t pack_half2(float a, float b) {
  const f32x2 pp = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, f16x2));
}
// What the halves of such a pair leave of (a, b), again as a packed pair: P = hi + lo carries 22 bits.
__device__ inline uint32_t pack_half2_rest(float a, float b, uint32_t hi) {
  const f16x2 h = __builtin_bit_cast(f16x2, hi);
  return pack_half2(a - (float)h[0], b - (float)h[1]);
}

// SPLIT: the key tiles are divided over gridDim.z workgroups (thin launches would otherwise
// leave most CUs idle and walk all N slots serially); each writes its unnormalised O, running
// max and sum, and attention_merge_kernel combines them.
//
// Software pipeline.  With one wave per SIMD nothing else can hide the softmax arithmetic, so
// each wave overlaps its own work: iteration t issues the MFMAs of O += V(t-1)^T P(t-1)^T and of
// S(t+1) = K(t+1) Q^T while the vector ALU turns S(t) into P(t) (MFMAs run asynchronously once
// issued).  O is kept relative to the running max of the tiles already ADDED, so the rescale by
// alpha(t) follows the accumulation of tile t-1 and happens only when some lane's max moved.
// K and V tiles arrive by direct-to-LDS loads into three-slot rings (K(t+3) and V(t+1) are issued
// in iteration t, two iterations ahead of their use); one barrier per tile.
template <bool SPLIT>
__global__ __launch_bounds__(256, 1) void attention_mfma_kernel(const bf16_t* __restrict__ q,
                                                                const bf16_t* __restrict__ kc,
                                                                const bf16_t* __restrict__ vc,
                                                                const int32_t* __restrict__ active_idx,
                                                                const int32_t* __restrict__ m_dev, int m_upper, int B,
                                                                int H, int N, int n_pad, bf16_t* __restrict__ o,
                                                                int tiles_per_split, float* __restrict__ part_o,
                                                                float* __restrict__ part_ml) {
  extern __shared__ FragA lds[];             // K ring [R][16 KiB] | V ring [R][16 KiB]
  __shared__ int cu[kMaxBatch + 2];
  constexpr int TILE_F = KT * DH / 8;        // FragA elements per tile
  FragA* const ldsK = lds;
  constexpr int R = 3;                       // ring depth: tiles are requested R-1 iterations ahead
  FragA* const ldsV = lds + R * TILE_F;
  const int M = min(*m_dev, m_upper);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // blockIdx.x = head: consecutive workgroup ids go to different XCDs, so the query tiles of
  // one head (same K/V) land on one XCD and share its L2
  const int hh = blockIdx.x;
  // per-sequence row ranges: cu[b] = first packed row whose flat id >= b*N
  if (B == 1) {
    if (tid <= 1) cu[tid] = tid ? M : 0;
  } else if (tid <= B) {
    int lo = 0, hi = M;
    const long long key = (long long)tid * N;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((long long)active_idx[mid] < key) lo = mid + 1; else hi = mid;
    }
    cu[tid] = lo;
  }
  __syncthreads();
  int b = 0, tile = blockIdx.y, row0 = -1, row_end = 0;
  for (; b < B; ++b) {
    const int cnt = cu[b + 1] - cu[b];
    const int nt = (cnt + QT - 1) / QT;
    if (tile < nt) { row0 = cu[b] + tile * QT; row_end = cu[b + 1]; break; }
    tile -= nt;
  }
  if (row0 < 0) return;                       // uniform across the workgroup

  const size_t head_base = ((size_t)b * H + hh) * n_pad * DH;
  const FragA* kg = reinterpret_cast<const FragA*>(kc + head_base);
  const FragA* vg = reinterpret_cast<const FragA*>(vc + head_base);
  const int kt_lo = SPLIT ? blockIdx.z * tiles_per_split : 0;
  const int kt_hi = SPLIT ? min(n_pad / KT, kt_lo + tiles_per_split) : n_pad / KT;
  const int T = kt_hi - kt_lo;               // >= 1 tiles for this workgroup

  // a 16 KiB tile is a straight copy: 16 chunks of 1 KiB, four per wave, lane L's 16 bytes land at
  // chunk base + 16 L
  // Addressing is scalar except for one per-lane byte offset: the tile pointer g is uniform
  // (instruction form "vgpr offset + sgpr base"), and the LDS destination is a scalar sum on the
  // wave's LDS base, read once.  l is a slot of the K or V ring, given as its index into lds.
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) FragA*)(lds + wave * 4 * 64));
  const uint32_t lane_voff = (uint32_t)((wave * 4 * 64 + lane) * 16);
  auto load_chunk = [&](const FragA* g, const FragA* l, int c) {
    const uint32_t laddr = lds_wave + (uint32_t)((l - lds) + c * 64) * 16u;
    const uint64_t gbase = (uint64_t)(uintptr_t)g + (uint64_t)(c * 1024);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_voff), "s"(gbase), "s"(laddr)
                 : "memory", "m0");
  };
  auto load_tile = [&](const FragA* g, FragA* l) {
#pragma unroll
    for (int c = 0; c < 4; ++c) load_chunk(g, l, c);
  };
  // prologue loads: K(0..R-1), V(0..R-3); V(0) also into the slot iteration 0 multiplies by P = 0
#pragma unroll
  for (int j = 0; j < R; ++j) load_tile(kg + (size_t)min(kt_lo + j, kt_hi - 1) * TILE_F, ldsK + j * TILE_F);
#pragma unroll
  for (int j = 0; j < R - 2; ++j) load_tile(vg + (size_t)min(kt_lo + j, kt_hi - 1) * TILE_F, ldsV + j * TILE_F);
  load_tile(vg + (size_t)kt_lo * TILE_F, ldsV + (R - 1) * TILE_F);

  // Q^T fragments: lane holds query (lane&31), dims ks*16 + (lane>>5)*8 .. +7
  const int my_row = row0 + wave * 32 + (lane & 31);
  const int ld_row = my_row < row_end ? my_row : row_end - 1;
  FragA qf[8];
  {
    const bf16_t* qp = q + ((size_t)ld_row * H + hh) * DH + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = *reinterpret_cast<const FragA*>(qp + ks * 16);
  }

  f32x16 acc_o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_o[i][v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float sc = 1.4426950408889634f / sqrtf((float)DH);   // log2(e) / sqrt(d_h)

  // S^T = K Q^T for one tile: two 32-key blocks
  auto scores = [&](const FragA* kt_lds, f32x16 (&sv)[2]) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sv[kb][v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const FragA a = kt_lds[(kb * 8 + ks) * 64 + lane];
        sv[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], sv[kb], 0, 0, 0);
      }
    }
  };
  // accumulator register v of block kb is key 32*kb + 8*(v/4) + 4*(lane>>5) + v%4
  auto mask_tail = [&](int kt, f32x16 (&sv)[2]) {
    const int kbase = kt * KT + 4 * (lane >> 5);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (kbase + 32 * kb + 8 * (v / 4) + (v % 4) >= N) sv[kb][v] = -INFINITY;
  };
  // O^T += V^T P^T
  auto pv = [&](const FragA* vt_lds, const PFrag (&ph)[4]) {
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      FragA a[4];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) a[mb] = vt_lds[(2 * st + (lane >> 5)) * DH + mb * 32 + (lane & 31)];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) acc_o[mb] = mfma_pv(a[mb], ph[st], acc_o[mb]);
    }
  };
  // One pipeline step for tile t: scores sc_cur -> probabilities p_new, while the MFMAs add tile t-1
  // (p_old) and compute the scores of tile t+1 (sc_next).
  auto step = [&](int t, f32x16 (&sc_cur)[2], f32x16 (&sc_next)[2], const PFrag (&p_old)[4], PFrag (&p_new)[4]) {
    // loads complete in order, eight chunks per wave per iteration: all but those of the last
    // R-2 iterations have landed, which covers K(t+1) and V(t-1)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 * (R - 2)) : "memory");
    __syncthreads();      // ... for everyone; the slots of K(t) and V(t-2) are free
    // K(t+R) and V(t+R-2) go into the two slots the barrier just freed, one 1 KiB chunk every second
    // MFMA slot below (a burst of eight would fill the load queue and stall the wave at issue).
    // Past the last tile K re-fetches the last one; nothing reads it.
    const FragA* k_src = kg + (size_t)min(kt_lo + t + R, kt_hi - 1) * TILE_F;
    const FragA* v_src = vg + (size_t)min(kt_lo + t + R - 2, kt_hi - 1) * TILE_F;
    FragA* const k_dst = ldsK + (t % R) * TILE_F;
    FragA* const v_dst = ldsV + ((t + R - 2) % R) * TILE_F;
    const FragA* vt_lds = ldsV + ((t + R - 1) % R) * TILE_F + (lane >> 5) * DH + (lane & 31);
    const FragA* kt_lds = ldsK + ((t + 1) % R) * TILE_F + lane;
    // The block below is laid out by hand as 32 slots, one MFMA each, fenced so that the compiler
    // keeps the order: slots 0..15 add tile t-1 (V fragment groups of four), slots 16..31 compute the
    // scores of tile t+1; LDS fragments are read 8..12 slots ahead of their MFMA; the softmax of tile
    // t rides along, one pair of probabilities every second slot (an MFMA occupies the matrix pipe
    // for 32 cycles and leaves the vector ALU about 20 of them).
    FragA va[3][4], kf[16];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) va[0][mb] = vt_lds[mb * 32];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) va[1][mb] = vt_lds[2 * DH + mb * 32];
    // The reference point of the exponentials follows the running max only in jumps of more than
    // kMaxLag (in the exp2 domain): a stale reference is exact mathematics (numerator and
    // denominator carry the same factor, at most 2^kMaxLag), and O is then rescaled on a tile only
    // when some query of the wave really jumped.  With near-uniform scores the max of 32 queries
    // creeps up on almost every tile, and rescaling 64 accumulators each time cost a quarter of
    // the kernel.  First tile: m_run = -inf, so every query jumps (alpha = 0 on a zero O).
    float mx = sc_cur[0][0], m_new = 0.f, alpha = 1.f, mb_ = 0.f;
    float psum = 0.f, pa = 0.f, pb = 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      if (i < 16 && i % 2 == 0) {
        if (i < 8) load_chunk(k_src, k_dst, i / 2);
        else load_chunk(v_src, v_dst, i / 2 - 4);
      }
      if (i < 8) {                                   // V fragments of group st + 2, eight slots ahead
        const int st = i >> 2, r = i & 3;
        va[(st + 2) % 3][r] = vt_lds[(2 * (st + 2)) * DH + r * 32];
      }
      if (i >= 4 && i < 20) {                        // K fragments of tile t+1, twelve slots ahead
        const int q = i - 4, jr = (q & 1) * 8 + (q >> 1);
        kf[jr] = kt_lds[jr * 64];
      }
      if (i < 16) {
        const int st = i >> 2, mb = i & 3;
        acc_o[mb] = mfma_pv(va[st % 3][mb], p_old[st], acc_o[mb]);
      } else {
        const int jj = i - 16, kb = jj & 1, ks = jj >> 1, j = kb * 8 + ks;   // the two score blocks alternate
        if (ks == 0) {
          f32x16 z;
#pragma unroll
          for (int v = 0; v < 16; ++v) z[v] = 0.f;
          sc_next[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j], qf[ks], z, 0, 0, 0);
        } else {
          sc_next[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j], qf[ks], sc_next[kb], 0, 0, 0);
        }
      }
      // Vector work of tile t, tied to its slot by the empty asm statements (without them the compiler
      // sinks all of it below the last MFMA).  Slots 0..3: the tile's row max, a dependent chain that
      // would otherwise hold the first MFMA back (the MFMAs of these slots add tile t-1 and do not need
      // it); the two lanes of a query exchange their halves with a lane-half swap, a vector-ALU
      // instruction.  Slots 4..31: the softmax, one pair of probabilities (2pr, 2pr+1 of this lane:
      // register v of block kb, for P^T step 2*kb + v/8) at a time, exponentials in one slot, sum and
      // rounding to a pair of halves in the next; the last four slots carry two such pieces each.
      if (i < 4) {
        const int kb = i >> 1, v0 = (i & 1) * 8;
#pragma unroll
        for (int v = 0; v < 8; ++v) mx = fmaxf(mx, sc_cur[kb][v0 + v]);
        if (i == 3) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
          mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
          const float m_cand = fmaxf(m_run, mx);    // finite: every tile holds at least one real key
          m_new = (m_cand - m_run) * sc > kMaxLag ? m_cand : m_run;
          alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sc);
          mb_ = m_new * sc;
          asm volatile("" : "+v"(m_new), "+v"(alpha), "+v"(mb_));
        } else {
          asm volatile("" : "+v"(mx));
        }
      } else {
#pragma unroll
        for (int u = 0; u < (i < 28 ? 1 : 2); ++u) {
          const int piece = i < 28 ? i - 4 : 24 + 2 * (i - 28) + u;      // 32 pieces: (pair, half of its work)
          const int pr = piece >> 1;
          const int x = 2 * pr, kb = x >> 4, v = x & 15, stp = 2 * kb + (v >> 3), e = v & 7;
          if ((piece & 1) == 0) {
            pa = __builtin_amdgcn_exp2f(fmaf(sc_cur[kb][v], sc, -mb_));
            pb = __builtin_amdgcn_exp2f(fmaf(sc_cur[kb][v + 1], sc, -mb_));
            asm volatile("" : "+v"(pa), "+v"(pb));
          } else {
            psum += pa + pb;
            uint32_t hw = pack_half2(pa, pb);
            asm volatile("" : "+v"(hw), "+v"(psum));
            p_new[stp][e >> 1] = hw;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run = l_run * alpha + psum;
    m_run = m_new;
    if (__any(alpha != 1.0f)) {                // the running max rarely moves after the first tiles
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[i][v] *= alpha;
    }
    if ((kt_lo + t + 2) * KT > N) mask_tail(kt_lo + t + 1, sc_next);
  };

  f32x16 s0[2], s1[2];
  PFrag p0[4], p1[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) p0[i][e] = 0u;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  scores(ldsK, s0);
  if ((kt_lo + 1) * KT > N) mask_tail(kt_lo, s0);
  for (int t = 0; t < T; t += 2) {
    step(t, s0, s1, p0, p1);
    if (t + 1 < T) step(t + 1, s1, s0, p1, p0);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();                            // V(T-1) landed
  if (T & 1) pv(ldsV + ((T - 1) % R) * TILE_F, p1);
  else pv(ldsV + ((T - 1) % R) * TILE_F, p0);

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (SPLIT) {
    if (my_row < row_end) {
      const size_t slot = ((size_t)blockIdx.z * m_upper + my_row) * H + hh;
      float* po = part_o + slot * DH + 4 * (lane >> 5);
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4*>(po + mb * 32 + 8 * g) =
              make_float4(acc_o[mb][4 * g], acc_o[mb][4 * g + 1], acc_o[mb][4 * g + 2], acc_o[mb][4 * g + 3]);
      if (lane < 32) {
        part_ml[slot * 2] = m_run * sc;          // running max in the exp2 domain
        part_ml[slot * 2 + 1] = l_tot;
      }
    }
    return;
  }
  const float inv = 1.0f / l_tot;
  if (my_row < row_end) {
    // o is written in the fragment-tiled activation layout the Out-projection GEMM reads
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc_o[mb][4 * g + e] * inv);
        *reinterpret_cast<bf16x4*>(o + afrag_index(my_row, hh * DH + mb * 32 + 8 * g + 4 * (lane >> 5), H * DH)) = w;
      }
  }
}

// Second form of the same product for launches with more workgroups than CUs: the wave does not
// pipeline its own tile steps (scores, softmax, P.V in sequence) and THREE workgroups share a CU, so
// that one's softmax runs under the others' MFMAs and barrier waits.  What lets three fit: P is one
// half-precision value per probability (no lo half: 32 MFMAs per tile instead of 48, no vector work to
// form it; 151 registers), and V has ONE 16 KiB slot next to K's two (48 KiB per workgroup): V(t) is
// requested at the top of step t, when the barrier has shown that everyone is done with V(t-1), and
// arrives under the scores and the softmax of the step; a second barrier per step makes it visible.
// Measured at sum M = 8192 rows of N = 1024: 220 us (two workgroups per CU, P as two halves) ->
// 206 us (three per CU) -> 157 us (one half).  Same fragment layouts as above.
template <bool SPLIT>
__global__ __launch_bounds__(256, 3) void attention_trio_kernel(const bf16_t* __restrict__ q,
                                                                const bf16_t* __restrict__ kc,
                                                                const bf16_t* __restrict__ vc,
                                                                const int32_t* __restrict__ active_idx,
                                                                const int32_t* __restrict__ m_dev, int m_upper, int B,
                                                                int H, int N, int n_pad, bf16_t* __restrict__ o,
                                                                int tiles_per_split, float* __restrict__ part_o,
                                                                float* __restrict__ part_ml) {
  extern __shared__ FragA lds[];             // K ring [2][16 KiB] | V slot [16 KiB]
  __shared__ int cu[kMaxBatch + 2];
  constexpr int TILE_F = KT * DH / 8;
  FragA* const ldsK = lds;
  FragA* const ldsV = lds + 2 * TILE_F;
  const int M = min(*m_dev, m_upper);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int hh = blockIdx.x;
  if (B == 1) {
    if (tid <= 1) cu[tid] = tid ? M : 0;
  } else if (tid <= B) {
    int lo = 0, hi = M;
    const long long key = (long long)tid * N;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((long long)active_idx[mid] < key) lo = mid + 1; else hi = mid;
    }
    cu[tid] = lo;
  }
  __syncthreads();
  int b = 0, tile = blockIdx.y, row0 = -1, row_end = 0;
  for (; b < B; ++b) {
    const int cnt = cu[b + 1] - cu[b];
    const int nt = (cnt + QT - 1) / QT;
    if (tile < nt) { row0 = cu[b] + tile * QT; row_end = cu[b + 1]; break; }
    tile -= nt;
  }
  if (row0 < 0) return;                       // uniform across the workgroup

  const size_t head_base = ((size_t)b * H + hh) * n_pad * DH;
  const FragA* kg = reinterpret_cast<const FragA*>(kc + head_base);
  const FragA* vg = reinterpret_cast<const FragA*>(vc + head_base);
  const int kt_lo = SPLIT ? blockIdx.z * tiles_per_split : 0;
  const int kt_hi = SPLIT ? min(n_pad / KT, kt_lo + tiles_per_split) : n_pad / KT;
  const int T = kt_hi - kt_lo;               // >= 1 tiles for this workgroup

  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) FragA*)(lds + wave * 4 * 64));
  const uint32_t lane_voff = (uint32_t)((wave * 4 * 64 + lane) * 16);
  auto load_tile = [&](const FragA* g, const FragA* l) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t laddr = lds_wave + (uint32_t)((l - lds) + c * 64) * 16u;
      const uint64_t gbase = (uint64_t)(uintptr_t)g + (uint64_t)(c * 1024);
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                   :
                   : "v"(lane_voff), "s"(gbase), "s"(laddr)
                   : "memory", "m0");
    }
  };
  load_tile(kg + (size_t)kt_lo * TILE_F, ldsK);

  const int my_row = row0 + wave * 32 + (lane & 31);
  const int ld_row = my_row < row_end ? my_row : row_end - 1;
  FragA qf[8];
  {
    const bf16_t* qp = q + ((size_t)ld_row * H + hh) * DH + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = *reinterpret_cast<const FragA*>(qp + ks * 16);
  }
  f32x16 acc_o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_o[i][v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float sc = 1.4426950408889634f / sqrtf((float)DH);   // log2(e) / sqrt(d_h)

  for (int t = 0; t < T; ++t) {
    const int slot = t & 1;
    // K(t) has landed (it was requested one iteration ago) ...
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();       // ... for everyone, and everyone is done with tile t-1: V's slot and K(t-1)'s are free
    // V(t) first, then K(t+1): loads complete in order, so "all but the last four" below means V(t)
    load_tile(vg + (size_t)(kt_lo + t) * TILE_F, ldsV);
    if (t + 1 < T) load_tile(kg + (size_t)(kt_lo + t + 1) * TILE_F, ldsK + (slot ^ 1) * TILE_F);
    // S^T = K Q^T: two 32-key blocks; register v of block kb is key 32*kb + 8*(v/4) + 4*(lane>>5) + v%4
    f32x16 sv[2];
    const FragA* kt_lds = ldsK + slot * TILE_F + lane;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sv[kb][v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
        sv[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt_lds[(kb * 8 + ks) * 64], qf[ks], sv[kb], 0, 0, 0);
    }
    if ((kt_lo + t + 1) * KT > N) {
      const int kbase = (kt_lo + t) * KT + 4 * (lane >> 5);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kbase + 32 * kb + 8 * (v / 4) + (v % 4) >= N) sv[kb][v] = -INFINITY;
    }
    float mx = sv[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sv[kb][v]);
    {   // the two lanes of a query exchange their halves' maxima (a lane-half swap: vector ALU, no LDS trip)
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    // the reference of the exponentials follows the running max only in jumps (see kMaxLag)
    const float m_cand = fmaxf(m_run, mx);
    const float m_new = (m_cand - m_run) * sc > kMaxLag ? m_cand : m_run;
    const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sc);
    const float mb_ = m_new * sc;
    if (__any(alpha != 1.0f)) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[i][v] *= alpha;
    }
    // P in half precision, round to nearest even; pair (v, v+1) of block kb belongs to P^T step 2*kb + v/8
    PFrag ph[4];
    float psum = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const float pa = __builtin_amdgcn_exp2f(fmaf(sv[kb][v], sc, -mb_));
        const float pb = __builtin_amdgcn_exp2f(fmaf(sv[kb][v + 1], sc, -mb_));
        psum += pa + pb;
        ph[2 * kb + (v >> 3)][(v & 7) >> 1] = pack_half2(pa, pb);
      }
    l_run = l_run * alpha + psum;
    m_run = m_new;
    // V(t) has landed (K(t+1)'s four chunks may still be in flight) ...
    if (t + 1 < T) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();       // ... for everyone
    // O^T += V^T P^T
    const FragA* vt_lds = ldsV + (lane >> 5) * DH + (lane & 31);
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      FragA a[4];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) a[mb] = vt_lds[(2 * st) * DH + mb * 32];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) acc_o[mb] = mfma_pv(a[mb], ph[st], acc_o[mb]);
    }
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (SPLIT) {
    if (my_row < row_end) {
      const size_t slot = ((size_t)blockIdx.z * m_upper + my_row) * H + hh;
      float* po = part_o + slot * DH + 4 * (lane >> 5);
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4*>(po + mb * 32 + 8 * g) =
              make_float4(acc_o[mb][4 * g], acc_o[mb][4 * g + 1], acc_o[mb][4 * g + 2], acc_o[mb][4 * g + 3]);
      if (lane < 32) {
        part_ml[slot * 2] = m_run * sc;
        part_ml[slot * 2 + 1] = l_tot;
      }
    }
    return;
  }
  const float inv = 1.0f / l_tot;
  if (my_row < row_end) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc_o[mb][4 * g + e] * inv);
        *reinterpret_cast<bf16x4*>(o + afrag_index(my_row, hh * DH + mb * 32 + 8 * g + 4 * (lane >> 5), H * DH)) = w;
      }
  }
}

// Third form, for launches of few rows (late steps of a schedule, where the whole product is a few
// MFLOP and its time is launches and memory latency): one workgroup = ONE head and 32 queries of one
// sequence; its four waves split the key tiles (wave w takes tiles w, w + 4, ..), each with the full
// flash recurrence on its own tiles, and merge their (O, max, sum) through LDS, so there is no
// partial-result buffer and no merge launch.  K and V fragments go global -> registers directly (the
// cache layouts make every MFMA fragment of a tile one contiguous 1 KiB block: no LDS staging, no
// barrier in the loop).  The next tile is asked for fragment by fragment while this one is computed, each into the registers
// of a fragment that has been read for the last time: 32 loads in a row fill the CU's load queue and the wave stands at
// their issue (a tile's compute takes 1.65 us and its loads 1.1; in a row 2.1 us, so 1.75).  One block, 32 queries a
// workgroup: 16 rows of N = 512 96.0 -> 95.4 us, 64 rows of N = 2048 121.7 -> 120.7.
// Same fragment layouts as the kernels above; P is carried as two halves (hi + lo, 22 bits: the
// matrix pipe idles here anyway).
// SPLIT: as above, for sequences whose tiles are too many for four waves; each workgroup leaves its merged sums to
// attention_merge_kernel.
// PAIRS: 32 queries per workgroup or 64, two waves for each 32 of them: one round of workgroups where 32 queries make two (the
// two waves that want a tile ask for it together).  One block, 32 -> 64 queries, medians of seven runs: 300 rows of N = 512 201.2 -> 198.1
// us, of N = 1024 210.7 -> 207.5, of 4 x 800 214.6 -> 207.3, 288 rows of 8 x 1024 218.5 -> 215.3, 457 rows of N = 1024 253.3 -> 251.7, 512
// rows of N = 512 238.6 -> 237.0.  A wave then makes two states of every fourth tile, one behind the other, where it could make one of
// every second: so a row's sums are made of the same four states in both forms, and its result is the same bit by bit (against one
// state: 457 rows 258.7 -> 258.6, 300 rows of N = 512 200.9 -> 201.8, 512 rows 243.3 -> 243.8).
// Which of the two is decided on the device, by the tiles that hold rows (thin_pairs): the host knows a bound only, which counts a
// part-filled tile for every sequence but one.  One block, 64 queries wherever the bound exceeds a round -> decided here: 16 rows of
// N = 512 bounded by 512 206.4 -> 203.4 us, 2 x 1024 with 96 and 160 rows 189.7 -> 186.7, 4 x 1024 with 50 rows each 179.2 -> 176.2, 6 x 20
// and 150 rows of 7 x 1024 228.9 -> 222.2, 4 x 2048 with 50 each 190.8 -> 183.4, 200 rows of N = 2048 bounded by 512 244.6 -> 234.1; where
// the keys and values of a batch are what is waited for (8 x 512, 160 rows) the forms are equal, 159.9 and 159.6.
template <int V> struct AtInt { static constexpr int value = V; };
// sum over the lanes up to this one
__device__ inline int wave_prefix_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);      // row_shr:1, :2, :4, :8 within 16 lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);      // lane 15 of a row to the odd rows behind it,
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);      // lane 31 to the upper half
  return v;
}
constexpr int QTT = 32;          // queries per workgroup of the thin kernel; PAIRS: or 64
constexpr int kThinOneRound = 256, kThinPairs = 512;          // workgroups of 32 queries
// Whether the rows' tiles of 64 (t64 per head) are taken instead of those of 32 (t32), in a grid of `rows` workgroups per head: where
// 32 make more than one round and 64 do not (12 x 512 with ten rows each, two rounds of either: 154.7 us with 64, 152.1 with 32),
// or where the grid has no place for all tiles of 32.
__host__ __device__ inline bool thin_pairs(int t32, int t64, int H, int rows) {
  return t32 * H > kThinOneRound && (t64 * H <= kThinOneRound || t32 > rows);
}
template <bool SPLIT, bool PAIRS>
__global__ __launch_bounds__(256, 1) void attention_thin_kernel(const bf16_t* __restrict__ q,
                                                                const bf16_t* __restrict__ kc,
                                                                const bf16_t* __restrict__ vc,
                                                                const int32_t* __restrict__ active_idx,
                                                                const int32_t* __restrict__ m_dev, int m_upper, int B,
                                                                int H, int N, int n_pad, bf16_t* __restrict__ o,
                                                                int tiles_per_split, float* __restrict__ part_o,
                                                                float* __restrict__ part_ml) {
  extern __shared__ FragA lds[];             // the merge: partial O [4 states, PAIRS 8][16][64 lanes] float4 | (m, l) [4, 8][64]
  __shared__ int cu[kMaxBatch + 2];
  constexpr int TILE_F = KT * DH / 8;
  const int M = min(*m_dev, m_upper);
  static_assert(!(PAIRS && SPLIT), "forms");
  const int tid = threadIdx.x, wave = PAIRS ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6, lane = tid & 63;
  const int hh = blockIdx.x;
  const int t_lo = SPLIT ? blockIdx.z * tiles_per_split : 0;
  const int t_hi = SPLIT ? min(n_pad / KT, t_lo + tiles_per_split) : n_pad / KT;
  const FragA *kg, *vg;
  auto head_of = [&](int b) {
    const size_t head_base = ((size_t)b * H + hh) * n_pad * DH;
    kg = reinterpret_cast<const FragA*>(kc + head_base) + lane;
    vg = reinterpret_cast<const FragA*>(vc + head_base) + (lane >> 5) * DH + (lane & 31);
  };
  FragA kf[16], vf[16];
  // fragments of tile t: K block (kb, ks) at (kb*8 + ks)*64 + lane, V^T block (st, mb) at (2*st + lane>>5)*DH + mb*32 + lane&31
  auto load_kv = [&](int t) {
    const FragA* kt = kg + (size_t)t * TILE_F;
    const FragA* vt = vg + (size_t)t * TILE_F;
#pragma unroll
    for (int j = 0; j < 16; ++j) kf[j] = kt[j * 64];
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) vf[st * 4 + mb] = vt[(2 * st) * DH + mb * 32];
  };
  int t = t_lo + wave;                        // this wave's first tile
  int row0 = -1, row_end = 0;
  int qw = QTT;                               // queries per workgroup
  bool two = false;                           // 64: two states per wave, waves 2 z + g for queries 32 g ..
  auto start = [&]() {
    if constexpr (PAIRS) {
      two = qw != QTT;
      if (two) t = wave >> 1;
    }
    if (t < t_hi) load_kv(t);
  };
  // workgroups past the rows leave (uniformly) before their first load: under a bound far above the row count most do (200 rows of
  // N = 512 bounded by 512: 12.3 us with a key tile asked for ahead of the test, 11.4 behind it)
  if (B == 1) {
    // one sequence: its row range is known without a search, LDS and a barrier (16 rows, N = 512 10.3 -> 9.9 us; 457 rows,
    // N = 1024 29.8 -> 28.5).  The loads in each branch: behind both, the address of a sequence that is not a constant costs 0.2 us
    // (24 rows of N = 512 7.9 -> 8.1; two sequences of 2048, split 15.7 -> 16.2).
    if constexpr (PAIRS)
      if (thin_pairs(sl_cdiv_dev(M, QTT), sl_cdiv_dev(M, 2 * QTT), H, gridDim.y)) qw = 2 * QTT;
    if ((int)blockIdx.y * qw >= M) return;
    row0 = blockIdx.y * qw;
    row_end = M;
    head_of(0);
    start();
  } else {
    if (tid <= B) {
      int lo = 0, hi = M;
      const long long key = (long long)tid * N;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((long long)active_idx[mid] < key) lo = mid + 1; else hi = mid;
      }
      cu[tid] = lo;
    }
    __syncthreads();
    int b = 0;
    if constexpr (PAIRS) {                    // lane = sequence, 64 at a time: the tiles of all of them, and this workgroup's
      auto locate = [&](int queries) {
        int tiles = 0;
        qw = queries;
        row0 = -1;
        for (int b0 = 0; b0 < B; b0 += 64) {
          const int c0 = cu[min(b0 + lane, B)], c1 = cu[min(b0 + lane + 1, B)], nt = (c1 - c0 + qw - 1) / qw;
          const int up_to = wave_prefix_sum(nt), tile = (int)blockIdx.y - tiles;
          const unsigned long long here = __ballot(tile < up_to);
          if (here != 0 && row0 < 0) {
            const int l = __ffsll(here) - 1;
            b = b0 + l;
            row0 = __builtin_amdgcn_readlane(c0, l) + (tile - __builtin_amdgcn_readlane(up_to - nt, l)) * qw;
            row_end = __builtin_amdgcn_readlane(c1, l);
          }
          tiles += __builtin_amdgcn_readlane(up_to, 63);
        }
        return tiles;
      };
      const int t32 = locate(QTT);
      if (t32 * H > kThinOneRound && !thin_pairs(t32, locate(2 * QTT), H, gridDim.y)) locate(QTT);
    } else {
      int tile = blockIdx.y;
      for (; b < B; ++b) {
        const int cnt = cu[b + 1] - cu[b];
        const int nt = (cnt + QTT - 1) / QTT;
        if (tile < nt) { row0 = cu[b] + tile * QTT; row_end = cu[b + 1]; break; }
        tile -= nt;
      }
    }
    if (row0 < 0) return;
    head_of(b);
    start();
  }

  // a wave holds 32 queries: lane = query (lane & 31), dims ks*16 + (lane>>5)*8 .. +7
  const int qg_w = two ? wave & 1 : 0;
  const int my_row = row0 + qg_w * QTT + (lane & 31);
  const int ld_row = my_row < row_end ? my_row : row_end - 1;
  FragA qf[8];
  {
    const bf16_t* qp = q + ((size_t)ld_row * H + hh) * DH + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = *reinterpret_cast<const FragA*>(qp + ks * 16);
  }
  f32x16 acc_o[4];
  float m_run, l_run;
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc_o[i][v] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
  };
  clear();
  const float sc = 1.4426950408889634f / sqrtf((float)DH);   // log2(e) / sqrt(d_h)

  // One tile; `more`: this wave's next one is asked for on the way, K's fragments behind the scores that read them, V's behind the
  // products.
  auto tile_step = [&](auto more, int t, int t_next) {
    constexpr bool MORE = decltype(more)::value;
    const FragA* kt_n = kg + (size_t)t_next * TILE_F;
    const FragA* vt_n = vg + (size_t)t_next * TILE_F;
    f32x16 sv[2], zero;
#pragma unroll
    for (int v = 0; v < 16; ++v) zero[v] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int kb = i & 1, ks = i >> 1;
      sv[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb * 8 + ks], qf[ks], ks ? sv[kb] : zero, 0, 0, 0);
    }
    if ((t + 1) * KT > N) {                  // register v of block kb is key 32*kb + 8*(v/4) + 4*(lane>>5) + v%4
      const int kbase = t * KT + 4 * (lane >> 5);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kbase + 32 * kb + 8 * (v / 4) + (v % 4) >= N) sv[kb][v] = -INFINITY;
    }
    float mx = sv[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sv[kb][v]);
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    // the reference follows the running max only in jumps (see kMaxLag); finite: every tile holds a real key
    const float m_cand = fmaxf(m_run, mx);
    const float m_new = (m_cand - m_run) * sc > kMaxLag ? m_cand : m_run;
    const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sc);
    const float mb_ = m_new * sc;
    if (__any(alpha != 1.0f)) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[i][v] *= alpha;
    }
    // the second half's probabilities are made between the MFMAs of the first half's product: one wave per SIMD has nobody
    // else to keep the matrix pipe busy under its vector work (one block, medians of seven runs, ahead of them -> between: 16 rows
    // 95.1 -> 94.9 us, 300 rows of N = 512 200.7 -> 200.0; 457 rows and 256 rows of N = 2048 equal)
    PFrag ph[4], pl[4];
    float psum = 0.f;
    auto pair = [&](int kb, int v) {
      const float pa = __builtin_amdgcn_exp2f(fmaf(sv[kb][v], sc, -mb_));
      const float pb = __builtin_amdgcn_exp2f(fmaf(sv[kb][v + 1], sc, -mb_));
      psum += pa + pb;
      const uint32_t hw = pack_half2(pa, pb);
      const uint32_t lw = pack_half2_rest(pa, pb, hw);
      ph[2 * kb + (v >> 3)][(v & 7) >> 1] = hw;
      pl[2 * kb + (v >> 3)][(v & 7) >> 1] = lw;
    };
    auto product = [&](int i) {              // MFMA i of the tile's 32
      const int st = i >> 3, mb = i & 3;
      acc_o[mb] = mfma_pv(vf[st * 4 + mb], (i >> 2) & 1 ? pl[st] : ph[st], acc_o[mb]);
    };
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      if constexpr (MORE) { kf[v] = kt_n[v * 64]; kf[v + 1] = kt_n[(v + 1) * 64]; }
      pair(0, v);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      product(v);
      pair(1, v);
      product(v + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int i = 16; i < 32; ++i) {
      product(i);
      if constexpr (MORE) {                  // fragment i - 16 has been read for the last time
        vf[i - 16] = vt_n[2 * ((i - 16) >> 2) * DH + (i & 3) * 32];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // a state (O, max, sum) covers every fourth tile.  The merge: lanes stand side by side in LDS, as a lane's 64 sums in a row put
  // all lanes on the same banks, 2 us of the launch (16 rows, N = 512: 10.1 -> 8.3 us).
  constexpr int STATES = PAIRS ? 8 : 4;
  float4* sh_o = reinterpret_cast<float4*>(lds);                           // [STATES][16 pieces][64 lanes]
  float2* sh_ml = reinterpret_cast<float2*>(sh_o + STATES * 16 * 64);      // [STATES][64]
  auto leave = [&](int z) {
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    float4* po = sh_o + z * 16 * 64 + lane;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        po[(mb * 4 + g) * 64] =
            make_float4(acc_o[mb][4 * g], acc_o[mb][4 * g + 1], acc_o[mb][4 * g + 2], acc_o[mb][4 * g + 3]);
    sh_ml[z * 64 + lane] = make_float2(m_run * sc, l_tot);         // reference in the exp2 domain (-inf: no tile)
  };
  if constexpr (!PAIRS) {
    for (; t + 4 < t_hi; t += 4) tile_step(AtInt<1>{}, t, t + 4);
    if (t < t_hi) tile_step(AtInt<0>{}, t, 0);
    leave(wave);
  } else {
    int z = t;                                // the wave's first state (t_lo is 0); of two, the second is z + 2
    bool follows = two && z + 2 < t_hi;       // a state with tiles comes behind this one
    for (;;) {
      const int t_next = t + 4 < t_hi ? t + 4 : follows ? z + 2 : t_hi;
      if (t_next >= t_hi) break;
      tile_step(AtInt<1>{}, t, t_next);
      if (t + 4 >= t_hi) {
        leave(qg_w * 4 + z);
        clear();
        z += 2;
        follows = false;
      }
      t = t_next;
    }
    if (t < t_hi) tile_step(AtInt<0>{}, t, 0);
    leave(qg_w * 4 + z);
    if (two && z < 2) {                       // the second state has no tile
      clear();
      leave(qg_w * 4 + z + 2);
    }
  }
  __syncthreads();
  // a wave finishes 4 NG dims of its 32 queries, from piece g0 on; the four states are added in the same order whoever made them
  float num[16 * (PAIRS ? 2 : 1)], den = 0.f, mx = -INFINITY;
  auto merge = [&](auto pieces, int g0) {
    constexpr int NG = decltype(pieces)::value;
    const int s0 = qg_w * 4;
    float2 ml[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) { ml[z] = sh_ml[(s0 + z) * 64 + lane]; mx = fmaxf(mx, ml[z].x); }
#pragma unroll
    for (int v = 0; v < 4 * NG; ++v) num[v] = 0.f;
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const float w = __builtin_amdgcn_exp2f(ml[z].x - mx);
      den = fmaf(w, ml[z].y, den);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const float4 pz = sh_o[((s0 + z) * 16 + g0 + g) * 64 + lane];
        num[4 * g] = fmaf(w, pz.x, num[4 * g]);
        num[4 * g + 1] = fmaf(w, pz.y, num[4 * g + 1]);
        num[4 * g + 2] = fmaf(w, pz.z, num[4 * g + 2]);
        num[4 * g + 3] = fmaf(w, pz.w, num[4 * g + 3]);
      }
    }
  };
  auto finish = [&](auto pieces, int g0) {
    constexpr int NG = decltype(pieces)::value;
    merge(pieces, g0);
    const float inv = 1.0f / den;
    if (my_row < row_end) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        bf16x4 w4;
#pragma unroll
        for (int e = 0; e < 4; ++e) w4[e] = (__bf16)(num[4 * g + e] * inv);
        *reinterpret_cast<bf16x4*>(o + afrag_index(my_row, hh * DH + (g0 + g) * 8 + 4 * (lane >> 5), H * DH)) = w4;
      }
    }
  };
  if constexpr (SPLIT) {
    merge(AtInt<4>{}, wave * 4);
    if (my_row < row_end) {
      const size_t slot = ((size_t)blockIdx.z * m_upper + my_row) * H + hh;
      float* po = part_o + slot * DH + wave * 32 + 4 * (lane >> 5);
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(po + 8 * g) = make_float4(num[4 * g], num[4 * g + 1], num[4 * g + 2], num[4 * g + 3]);
      if (wave == 0 && lane < 32) {
        part_ml[slot * 2] = mx;
        part_ml[slot * 2 + 1] = den;
      }
    }
  } else if (PAIRS && two) {
    finish(AtInt<8>{}, (wave >> 1) * 8);
  } else {
    finish(AtInt<4>{}, wave * 4);
  }
}

// o[row, h, :] = sum_z 2^(m_z - m) O_z / sum_z 2^(m_z - m) l_z over the key splits z.  Four dims per thread, 32 threads
// per (row, head); a launch of few rows is one chain of memory latencies, so four splits are read at a time, sums and
// weights together (64 rows, one dim per thread and a maximum pass first: 6.7 us; so: 4.6 us).
constexpr int kMergeHeads = 8;      // (row, head) pairs per workgroup
__global__ __launch_bounds__(32 * kMergeHeads) void attention_merge_kernel(const float* __restrict__ part_o,
                                                                           const float* __restrict__ part_ml,
                                                                           const int32_t* __restrict__ m_dev,
                                                                           int m_upper, int H, int Z,
                                                                           bf16_t* __restrict__ o) {
  const int M = min(*m_dev, m_upper);
  const int row = blockIdx.x, hh = blockIdx.y * kMergeHeads + (threadIdx.x >> 5), dd = (threadIdx.x & 31) * 4;
  if (row >= M || hh >= H) return;
  const size_t zs = (size_t)m_upper * H, slot = (size_t)row * H + hh;
  float mx = -INFINITY, den = 0.f, num[4] = {0.f, 0.f, 0.f, 0.f};
  for (int z0 = 0; z0 < Z; z0 += 4) {
    float2 ml[4];
    float4 po[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t sl = slot + (size_t)min(z0 + i, Z - 1) * zs;
      ml[i] = *reinterpret_cast<const float2*>(part_ml + sl * 2);
      po[i] = *reinterpret_cast<const float4*>(part_o + sl * DH + dd);
    }
    float m_new = mx;
#pragma unroll
    for (int i = 0; i < 4; ++i) m_new = fmaxf(m_new, ml[i].x);           // finite: every split holds a real key
    const float old = exp2f(mx - m_new);
    den *= old;
#pragma unroll
    for (int e = 0; e < 4; ++e) num[e] *= old;
    mx = m_new;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (z0 + i < Z) {
        const float w = exp2f(ml[i].x - mx);
        den = fmaf(w, ml[i].y, den);
        num[0] = fmaf(w, po[i].x, num[0]);
        num[1] = fmaf(w, po[i].y, num[1]);
        num[2] = fmaf(w, po[i].z, num[2]);
        num[3] = fmaf(w, po[i].w, num[3]);
      }
  }
  bf16x4 w4;
#pragma unroll
  for (int e = 0; e < 4; ++e) w4[e] = (__bf16)(num[e] / den);
  *reinterpret_cast<bf16x4*>(o + afrag_index(row, hh * DH + dd, H * DH)) = w4;
}

// Which kernel a launch of `blocks` (row tile, head) workgroups takes: the three-per-CU kernel as
// soon as there are more workgroups than CUs, the pipelined one otherwise (at N = 2048 and 857 rows,
// 224 workgroups: 46 us against 62 us for the three-per-CU kernel with the keys split three ways).
static bool attention_use_trio(int blocks) { return blocks > 256; }

// The thin kernel (32 queries and one head per workgroup, key tiles split over its waves): key splits Z of a launch,
// 0 = another kernel.  Unsplit while its workgroups fit the chip in one round and a wave's share of the keys stays
// short (16 tiles).  Longer sequences: up to one workgroup per CU, with as many splits as that leaves room for (a wave
// keeps one tile at least) and at most 32 tiles per split.  Measured as one block of the layer, B = 1, the pipelined
// kernel with its splits against this one, N = 2048: 32 rows 124.6 against 119.6 us (Z = 8), 64 rows 153.0 / 145.8 (4),
// 128 rows 180.7 / 171.6 (2), 256 rows 228.7 / 225.4 (1); N = 4096, 64 rows 157.9 / 151.3 (4), 256 rows (64 tiles per split)
// 237.5 / 237.7.  Up to two workgroups per CU by the bound it takes 32 or 64 queries each, where 32 tiles or fewer are to be walked: N = 2048,
// 320 rows 226.1 / 224.1, 384 rows 237.7 / 234.9, 480 rows 276.2 / 273.4, N = 1100, 300 rows 218.0 / 212.4; batches of even sequences:
// 2 x 1100, 300 rows 220.2 / 214.7, 2 x 2048, 300 rows 230.2 / 227.9, 450 rows 283.1 / 279.0, 4 x 1600, 200 rows 193.8 / 183.0, 4 x 2048,
// 300 rows 236.1 / 230.0, 8 x 2048, 64 rows 151.6 / 150.4, 288 rows 257.3 / 254.0, 12 x 1500, 60 rows 165.6 / 166.1; bounds far above the
// rows, N = 2048: 16 rows bounded by 384 184.8 / 176.9, 64 by 512 226.7 / 216.7.  Beyond that it loses to the
// three-per-CU kernel: N = 1024, 600 rows 317.5 / 326.6, 800 rows 369.5 / 377.8.
static int attention_thin_splits(int m_upper, int B, int H, int n_pad, int* tiles_per_split) {
  const int n_tiles = n_pad / KT, blocks = (sl_cdiv(m_upper, QTT) + B - 1) * H;
  *tiles_per_split = n_tiles;
  if (n_tiles <= 16) return blocks <= kThinPairs ? 1 : 0;
  if (blocks > kThinOneRound) return blocks <= kThinPairs && n_tiles <= 32 ? 1 : 0;
  const int Z = 256 / blocks < sl_cdiv(n_tiles, 4) ? 256 / blocks : sl_cdiv(n_tiles, 4);
  *tiles_per_split = sl_cdiv(n_tiles, Z);
  return *tiles_per_split <= 32 ? sl_cdiv(n_tiles, *tiles_per_split) : 0;
}

// Workgroups per head of an unsplit thin launch that may take 64 queries each, 0 where the bound is one round of 32 anyway: room
// for every row within the bound at 64, and at 32 for every distribution that then makes one round.
static int attention_thin_pair_tiles(int m_upper, int B, int H) {
  const int tiles32 = sl_cdiv(m_upper, QTT) + B - 1, tiles64 = sl_cdiv(m_upper, 2 * QTT) + B - 1;
  if (tiles32 * H <= kThinOneRound) return 0;
  const int round = tiles32 < kThinOneRound / H ? tiles32 : kThinOneRound / H;
  return tiles64 > round ? tiles64 : round;
}
// for tests: key splits of the thin kernel (0: another kernel's launch), workgroups per head, whether they may take 64 queries; and
// whether they do
void slk_attention_thin_form(int m_upper, int B, int H, int n_pad, int* out) {
  int tps;
  out[0] = attention_thin_splits(m_upper, B, H, n_pad, &tps);
  out[1] = out[0] == 1 ? attention_thin_pair_tiles(m_upper, B, H) : 0;
  out[2] = out[1] != 0;
  if (!out[2]) out[1] = sl_cdiv(m_upper, QTT) + B - 1;
}
int slk_attention_thin_pairs(int t32, int t64, int H, int rows) { return thin_pairs(t32, t64, H, rows); }

// Key-split plan for a launch bounded by m_upper rows: the keys are split just far enough to
// give every CU one workgroup of the pipelined kernel (LDS rings, 370 registers per lane: one per
// CU) or three of the other; splitting further only adds partial-result traffic and more
// rounds of workgroups.  Returns Z (1 = no split) and the tiles per split.
int slk_attention_splits(int m_upper, int B, int H, int n_pad, int* tiles_per_split) {
  const int n_tiles = n_pad / KT;
  const int blocks = (sl_cdiv(m_upper, QT) + B - 1) * H;
  int Z = (attention_use_trio(blocks) ? 768 : 256) / blocks;
  if (Z < 1) Z = 1;
  if (Z > n_tiles) Z = n_tiles;
  const int tps = sl_cdiv(n_tiles, Z);
  *tiles_per_split = tps;
  return sl_cdiv(n_tiles, tps);
}

// fp32 scratch floats the split path may need for any launch of at most m_upper rows
size_t slk_attention_scratch_elems(int m_upper, int B, int H, int n_pad) {
  size_t splits_rows = 0;                    // the splits of both kernels depend on a launch's row tiles only
  int tps;
  for (int t = 1; (t - 1) * QT < m_upper; ++t) {
    const int mu = t * QT < m_upper ? t * QT : m_upper;
    const int Z = slk_attention_splits(mu, B, H, n_pad, &tps);
    if (Z > 1 && (size_t)Z * mu > splits_rows) splits_rows = (size_t)Z * mu;
  }
  for (int t = 1; (t - 1) * QTT < m_upper; ++t) {
    const int mu = t * QTT < m_upper ? t * QTT : m_upper;
    const int Z = attention_thin_splits(mu, B, H, n_pad, &tps);
    if (Z > 1 && (size_t)Z * mu > splits_rows) splits_rows = (size_t)Z * mu;
  }
  return splits_rows * H * (DH + 2);
}

int slk_attention_mfma(hipStream_t s, const void* q, const void* kc, const void* vc, const int32_t* active_idx,
                       const int32_t* m_dev, int m_upper, int B, int H, int N, int n_pad, void* o, float* scratch) {
  if (m_upper <= 0) return SL_OK;
  if (B > kMaxBatch || n_pad % KT) return SL_EINVAL;
  int tps;
  const auto merge = [&](const float* po, const float* pml, int Z) {
    hipLaunchKernelGGL(attention_merge_kernel, dim3(m_upper, sl_cdiv(H, kMergeHeads)), dim3(32 * kMergeHeads), 0, s, po, pml,
                       m_dev, m_upper, H, Z, (bf16_t*)o);
    SL_LAUNCH_CHECK();
    return SL_OK;
  };
  const int Zt = attention_thin_splits(m_upper, B, H, n_pad, &tps);
  if (Zt == 1 || (Zt > 1 && scratch)) {
    const size_t sh_thin = (size_t)(4 * 64 * 64 + 4 * 64 * 2) * sizeof(float);
    static unsigned long long lds_thin[3] = {0, 0, 0};
    SL_ALLOW_DYNAMIC_LDS(lds_thin[0], (attention_thin_kernel<false, false>), sh_thin);
    SL_ALLOW_DYNAMIC_LDS(lds_thin[1], (attention_thin_kernel<true, false>), sh_thin);
    SL_ALLOW_DYNAMIC_LDS(lds_thin[2], (attention_thin_kernel<false, true>), 2 * sh_thin);
    if (const int tiles = Zt == 1 ? attention_thin_pair_tiles(m_upper, B, H) : 0) {
      hipLaunchKernelGGL((attention_thin_kernel<false, true>), dim3(H, tiles, 1), dim3(256), 2 * sh_thin, s,
                         (const bf16_t*)q, (const bf16_t*)kc, (const bf16_t*)vc, active_idx, m_dev, m_upper, B, H, N, n_pad, (bf16_t*)o, tps,
                         (float*)nullptr, (float*)nullptr);
      SL_LAUNCH_CHECK();
      return SL_OK;
    }
    float* po = Zt > 1 ? scratch : nullptr;
    float* pml = Zt > 1 ? scratch + (size_t)Zt * m_upper * H * DH : nullptr;
    hipLaunchKernelGGL((Zt > 1 ? attention_thin_kernel<true, false> : attention_thin_kernel<false, false>),
                       dim3(H, sl_cdiv(m_upper, QTT) + B - 1, Zt), dim3(256), sh_thin, s, (const bf16_t*)q, (const bf16_t*)kc,
                       (const bf16_t*)vc, active_idx, m_dev, m_upper, B, H, N, n_pad, (bf16_t*)o, tps, po, pml);
    SL_LAUNCH_CHECK();
    return Zt > 1 ? merge(po, pml, Zt) : SL_OK;
  }
  const int Z = scratch ? slk_attention_splits(m_upper, B, H, n_pad, &tps) : 1;
  dim3 grid(H, sl_cdiv(m_upper, QT) + B - 1, Z), block(256);
  const bool trio = attention_use_trio((int)(grid.x * grid.y));
  const size_t sh = (trio ? 3 : 6) * (size_t)KT * DH * 2;   // 16 KiB slots: K 2 + V 1, or three each
  static unsigned long long lds_ok[4] = {0, 0, 0, 0};
  SL_ALLOW_DYNAMIC_LDS(lds_ok[0], attention_mfma_kernel<false>, 6 * (size_t)KT * DH * 2);
  SL_ALLOW_DYNAMIC_LDS(lds_ok[1], attention_mfma_kernel<true>, 6 * (size_t)KT * DH * 2);
  SL_ALLOW_DYNAMIC_LDS(lds_ok[2], attention_trio_kernel<false>, 3 * (size_t)KT * DH * 2);
  SL_ALLOW_DYNAMIC_LDS(lds_ok[3], attention_trio_kernel<true>, 3 * (size_t)KT * DH * 2);
  if (Z == 1) {
    hipLaunchKernelGGL(trio ? attention_trio_kernel<false> : attention_mfma_kernel<false>, grid, block, sh, s,
                       (const bf16_t*)q, (const bf16_t*)kc, (const bf16_t*)vc, active_idx, m_dev, m_upper, B, H, N, n_pad,
                       (bf16_t*)o, 0, nullptr, nullptr);
    SL_LAUNCH_CHECK();
    return SL_OK;
  }
  float* part_o = scratch;
  float* part_ml = scratch + (size_t)Z * m_upper * H * DH;
  hipLaunchKernelGGL(trio ? attention_trio_kernel<true> : attention_mfma_kernel<true>, grid, block, sh, s,
                     (const bf16_t*)q, (const bf16_t*)kc, (const bf16_t*)vc, active_idx, m_dev, m_upper, B, H, N, n_pad,
                     (bf16_t*)o, tps, part_o, part_ml);
  SL_LAUNCH_CHECK();
  return merge(part_o, part_ml, Z);
}
