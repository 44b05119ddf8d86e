// Pieces shared by the projection kernels whose accumulators are 16 x 16 blocks: lane l of a wave holds row l % 16,
// columns 4 (l / 16) .. + 3 of a block.
#pragma once
#include "sl_common.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef bf16x8 Frag;                      // one lane's 16-byte share of an operand
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// The Q|K|V projection with RoPE and the scatter into q / the K and V caches in its epilogue (the launch then replaces
// the projection's fp32 output and the separate RoPE + cache-write kernel).
struct RopeScatter {
  const int32_t* active_idx;   // [M] flat row ids
  const float2* rope_tab;      // [n_pad][64] (cos, sin)
  bf16_t* q;                   // [M, H*128] packed
  bf16_t* kc;                  // this layer's K cache, or null (queries only)
  bf16_t* vc;                  // this layer's V cache, or null
  int N, n_pad, H;
};

// 8 consecutive columns per lane out of two 16 x 16 blocks: lane group g = l / 16 holds columns 4 g .. 4 g + 3 of
// each; after swapping the odd groups of the first with the even groups of the second it holds columns
// 8 (g / 2) .. + 7 of block g % 2.
__device__ __forceinline__ uint4 pack_swap(const f32x4& x, const f32x4& y) {
  bf16x4 vx, vy;
#pragma unroll
  for (int e = 0; e < 4; ++e) { vx[e] = (bf16_t)x[e]; vy[e] = (bf16_t)y[e]; }
  const uint2 ux = __builtin_bit_cast(uint2, vx), uy = __builtin_bit_cast(uint2, vy);
  const auto p = __builtin_amdgcn_permlane16_swap(ux.x, uy.x, false, false);
  const auto q = __builtin_amdgcn_permlane16_swap(ux.y, uy.y, false, false);
  return make_uint4(p[0], q[0], p[1], q[1]);
}

// Each row's flat id (-1 past M), sequence and slot into row_sh [3][rows], by the whole workgroup.
__device__ __forceinline__ void scatter_rows_of_tile(int* row_sh, int rows, int m0, int M, const RopeScatter& rs) {
  for (int r = threadIdx.x; r < rows; r += blockDim.x) {
    const int row = m0 + r;
    const int g = row < M ? rs.active_idx[row] : -1;
    const int bb = g < 0 ? 0 : g / rs.N;
    row_sh[r] = g;
    row_sh[rows + r] = bb;
    row_sh[2 * rows + r] = g < 0 ? -1 : g - bb * rs.N;
  }
}

// Packed row `row` (slot i of sequence bb): blocks 0, 1 of c are dims j0 .. j0 + 31 of a head, blocks 2, 3 the dims 64
// further on.  RoPE, which pairs them, is applied to the unrounded sums, like the stand-alone kernel does.  sec 0: q, 1: k.
__device__ __forceinline__ void rope_load_row(float4 (&t)[4], int i, int j0, const RopeScatter& rs) {
  const int g4 = (threadIdx.x & 63) >> 4;
  const float4* tab = reinterpret_cast<const float4*>(rs.rope_tab + (size_t)i * 64 + j0);
#pragma unroll
  for (int b = 0; b < 2; ++b) { t[2 * b] = tab[b * 8 + 2 * g4]; t[2 * b + 1] = tab[b * 8 + 2 * g4 + 1]; }   // (cos, sin) of 4 dims
}
__device__ __forceinline__ void rope_store_row(const f32x4 (&c)[4], const float4 (&t)[4], int sec, int head, int j0, int row,
                                               int bb, int i, const RopeScatter& rs) {
  const int g4 = (threadIdx.x & 63) >> 4, hd = rs.H * 128;
  f32x4 lo[2], hi[2];                                 // dims j and j + 64
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const float4 t0 = t[2 * b], t1 = t[2 * b + 1];
    const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = c[b][e], y = c[b + 2][e];
      lo[b][e] = x * cs[e] - y * sn[e];
      hi[b][e] = y * cs[e] + x * sn[e];
    }
  }
  const uint4 o1 = pack_swap(lo[0], lo[1]), o2 = pack_swap(hi[0], hi[1]);
  const int dim = j0 + (g4 & 1) * 16 + (g4 >> 1) * 8;
  if (sec == 0) {
    bf16_t* qr = rs.q + (size_t)row * hd + head * 128 + dim;
    *reinterpret_cast<uint4*>(qr) = o1;
    *reinterpret_cast<uint4*>(qr + 64) = o2;
  } else {
    bf16_t* kb = rs.kc + ((size_t)bb * rs.H + head) * rs.n_pad * 128;
    *reinterpret_cast<uint4*>(kb + kc_index(i, dim, 128)) = o1;
    *reinterpret_cast<uint4*>(kb + kc_index(i, 64 + dim, 128)) = o2;
  }
}

// V: the cache keeps eight slots of a dim together, so the rows pass through LDS as cache elements (a wave's own corner, no
// barrier): rows of VSTAGE elements, columns 0 .. 31 the dims j0 .., 32 .. 63 the dims 64 further on.
constexpr int VSTAGE = 72;
__device__ __forceinline__ void v_stage_block(bf16_t* stage, int row, int block, const f32x4& c) {
  const int g4 = (threadIdx.x & 63) >> 4;
  bf16x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = vcache_half_bits(c[e]);
  *reinterpret_cast<bf16x4*>(stage + row * VSTAGE + block * 16 + 4 * g4) = v;
}
// 16 staged rows, row l % 16 being slot i of sequence bb (i = -1: no row): if they are the 16 slots of one aligned block they
// leave as 16-byte groups of eight slots per dim, otherwise as 2-byte stores, a row per instruction.
__device__ __forceinline__ void v_store_rows(const bf16_t* stage, int bb, int i, int head, int j0, const RopeScatter& rs) {
  const int lane = threadIdx.x & 63, row_in = lane & 15;
  const int dim = j0 + (lane & 31) + (lane >> 5) * 64;
  bf16_t* vb = rs.vc + (size_t)head * rs.n_pad * 128;
  const size_t seq = (size_t)rs.H * rs.n_pad * 128;
  const bf16_t* col = stage + lane;
  const int i0 = __builtin_amdgcn_readfirstlane(i), bb0 = __builtin_amdgcn_readfirstlane(bb);
  if (i0 >= 0 && i0 % 16 == 0 && i0 + 16 <= rs.N && __all(i == i0 + row_in && bb == bb0)) {
    bf16_t* vr = vb + bb0 * seq;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = col[((e >> 2) * 8 + 4 * h + (e & 3)) * VSTAGE];
      *reinterpret_cast<bf16x8*>(vr + vc_index(i0 + 4 * h, dim, 128)) = o;
    }
  } else {
    // lane r of the first 16 holds row r's offset; it is read across as a scalar
    const uint64_t off = i < 0 ? 0 : (uint64_t)bb * seq + vc_index(i, 0, 128);
    const uint32_t off_lo = (uint32_t)off, off_hi = (uint32_t)(off >> 32);
    bf16_t v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = col[r * VSTAGE];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint64_t o = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(off_hi, r) << 32 | (uint32_t)__builtin_amdgcn_readlane(off_lo, r);
      if (__builtin_amdgcn_readlane(i, r) >= 0) vb[o + (uint32_t)dim * 8] = v[r];
    }
  }
}

// The same for a unit of 16 + 16 columns by one wave: lo the dims j0 .. j0 + 15 of a head, hi those 64 further on; a lane's
// four dims are 8-byte pieces.
__device__ __forceinline__ void rope_load_unit(float4 (&t)[2], int i, int j0, const RopeScatter& rs) {
  const float4* tab = reinterpret_cast<const float4*>(rs.rope_tab + (size_t)i * 64 + j0 + 4 * ((threadIdx.x & 63) >> 4));
  t[0] = tab[0];                                      // (cos, sin) pairs of 4 dims
  t[1] = tab[1];
}
__device__ __forceinline__ void rope_store_unit(const f32x4& lo, const f32x4& hi, const float4 (&t)[2], int sec, int head, int j0,
                                                int row, int bb, int i, const RopeScatter& rs) {
  const int g4 = (threadIdx.x & 63) >> 4, dim = j0 + 4 * g4;
  const float4 t0 = t[0], t1 = t[1];
  const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
  bf16x4 o1, o2;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    o1[e] = (bf16_t)(lo[e] * cs[e] - hi[e] * sn[e]);
    o2[e] = (bf16_t)(hi[e] * cs[e] + lo[e] * sn[e]);
  }
  bf16_t *p1, *p2;
  if (sec == 0) {
    p1 = rs.q + (size_t)row * rs.H * 128 + head * 128 + dim;
    p2 = p1 + 64;
  } else {
    bf16_t* kb = rs.kc + ((size_t)bb * rs.H + head) * rs.n_pad * 128;
    p1 = kb + kc_index(i, dim, 128);
    p2 = kb + kc_index(i, dim + 64, 128);
  }
  *reinterpret_cast<bf16x4*>(p1) = o1;
  *reinterpret_cast<bf16x4*>(p2) = o2;
}
constexpr int VUNIT = 36;                 // elements per staged row: 16 + 16 and padding
__device__ __forceinline__ void v_store_unit(bf16_t* stage, const f32x4& lo, const f32x4& hi, int head, int j0, int bb, int i,
                                             const RopeScatter& rs) {
  const int lane = threadIdx.x & 63, g4 = lane >> 4, row_in = lane & 15, half = lane >> 5;
  asm volatile("" ::: "memory");                      // the rows of the unit before have been read: LDS keeps a wave's order
  bf16x4 v0, v1;
#pragma unroll
  for (int e = 0; e < 4; ++e) { v0[e] = vcache_half_bits(lo[e]); v1[e] = vcache_half_bits(hi[e]); }
  *reinterpret_cast<bf16x4*>(stage + row_in * VUNIT + 4 * g4) = v0;
  *reinterpret_cast<bf16x4*>(stage + row_in * VUNIT + 16 + 4 * g4) = v1;
  asm volatile("" ::: "memory");
  const int dim = j0 + (lane & 15) + ((lane >> 4) & 1) * 64;
  bf16_t* vb = rs.vc + (size_t)head * rs.n_pad * 128;
  const size_t seq = (size_t)rs.H * rs.n_pad * 128;
  const bf16_t* col = stage + (lane & 31);
  const int i0 = __builtin_amdgcn_readfirstlane(i), bb0 = __builtin_amdgcn_readfirstlane(bb);
  if (i0 >= 0 && i0 % 16 == 0 && i0 + 16 <= rs.N && __all(i == i0 + row_in && bb == bb0)) {
    bf16x8 o;                                         // lanes 0 .. 31 the first eight slots of a dim, 32 .. 63 the others
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = col[((e >> 2) * 8 + 4 * half + (e & 3)) * VUNIT];
    *reinterpret_cast<bf16x8*>(vb + bb0 * seq + vc_index(i0 + 4 * half, dim, 128)) = o;
  } else {
    // four neighbouring dims of the 16 rows per instruction: a lane keeps its row, whose address it has, and rows that share
    // a group of eight slots share the 64-byte segment they write (two rows per instruction and their addresses read across
    // the lanes: Q|K|V of 224 rows, last workgroup 40.7 us after the first one's start, now 34.9; one block 169.4 -> 167.5)
    const bf16_t* mine = stage + row_in * VUNIT + g4;
    bf16_t v[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) v[d] = mine[4 * d];
    if (i >= 0) {
      bf16_t* p = vb + bb * seq + vc_index(i, j0 + g4, 128);
#pragma unroll
      for (int d = 0; d < 8; ++d) p[((d & 3) * 4 + (d >> 2) * 64) * 8] = v[d];
    }
  }
}
