// Shape-generic projection kernels: C[m, n] = sum_k A[m, k] * W[n, k]  (y = x W^T), any m / n / k, storage type
// fp32 or bf16, on the fp32 matrix instructions (fp32 products and sums).  The path of the fp32 configuration and
// of shapes the bf16 MFMA kernels do not tile.
//
// These shapes are small (72 x 256 x 256 and the like), so a launch is bound by how many waves it puts on the chip
// and by one chain of load latencies, not by arithmetic: operands go global -> registers without LDS, 16 bytes per
// lane, several k-chunks in flight.  A lane of the 16 x 16 x 4 instruction holds one k of one row; giving lane group
// g the four consecutive k = 4 g .. 4 g + 3 of a 16-deep chunk (and feeding element e of all groups to the e-th
// instruction) turns that into 16-byte loads: a sum over k may take its terms in any order.  W is the first
// operand, so a lane ends up with four consecutive columns of one output row.
//  * few tiles: one 16 x 16 output tile per workgroup, the k-chunks dealt to its four waves, partial sums added
//    through LDS in wave order (72 x 256 x 256: 55 -> 4.4 us, 8 workgroups before, 80 now);
//  * many tiles: 64 x 64 per workgroup, 32 x 32 per wave, which reads each operand element four times less often.
// Up to three matrices of one shape (Q, K, V) share a launch; gate and up share one that applies SwiGLU.
//
// What is left of such a step is the number of dependent launches, 3 to 5 us each.  fp32 layers whose launches all take
// the 16 x 16 form (slk_generic_fused) therefore have none but their projections and attention: a workgroup sees whole
// rows of A on its way through k, so it sums their squares and scales its results by the norm it would have waited for
// (NORM; the gain goes into the operand); Q|K|V rotates and scatters its own columns (MODE 2); Out and down add to the
// residual in place (RES).  The tiny model's step (2 blocks, 72 rows): 21 launches -> 15,
// 88.5 -> 77.2 us; 300 rows of 4 x 256 slots 118.1 -> 103.5, 600 rows 157.6 -> 139.8.
#include "sl_common.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KC = 16;    // k per chunk: four instructions

// four consecutive elements; zeros past the row's end (k % 4 == 0 on the vector path, so a piece is whole or absent)
template <typename T, bool VEC>
__device__ inline f32x4 load4(const T* row, int kk, int k) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (kk < k) {
      if constexpr (sizeof(T) == 4) v = *reinterpret_cast<const f32x4*>(row + kk);
      else {
        const bf16x4_t u = *reinterpret_cast<const bf16x4_t*>(row + kk);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (float)u[e];
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (kk + e < k) v[e] = st<T>::ld(row + kk + e);
  }
  return v;
}

struct GenericMats { const void* w[3]; };

struct GenericNorm { const float* gain; float eps; };          // NORM: A holds the rows before RMSNorm

struct GenericRope {          // MODE 2: where Q|K|V goes (as slk_rope_kv_write)
  const int32_t* active_idx;
  const float2* tab;          // [n_pad][dh / 2]
  float *q, *kc, *vc;         // kc = vc = null: queries only
  int H, dh, N, n_pad;
};

// MODE 0: matrix z of the launch -> columns z * n .. of C_f32 / C_T.  MODE 1: w[0] = gate, w[1] = up: C_T =
// silu(gate) * up.  MODE 2: matrix z is q, k or v: 16 columns of a head's first half and those they rotate with, RoPE and
// the scatter.  RES: C_T += the product.  MB x MB blocks of 16 x 16 per wave; KS waves share a tile's k-chunks (MB == 1: 4,
// else 1), UC chunks of each in flight.
template <typename T, int MODE, int MB, bool VEC, bool NORM, bool RES, int UC>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const T* __restrict__ A, GenericMats mats,
                                                           const int32_t* __restrict__ m_dev, int m_upper, int n,
                                                           int k, float* __restrict__ C_f32, T* __restrict__ C_T,
                                                           const int32_t* __restrict__ out_row_map, size_t ldc,
                                                           GenericNorm norm, GenericRope rope) {
  constexpr int KS = MB == 1 ? 4 : 1, NW = MODE >= 1 ? 2 : 1;
  static_assert((!NORM && !RES && MODE != 2) || (MB == 1 && VEC && sizeof(T) == 4), "forms of the fused launches");
  __shared__ f32x4 part[KS > 1 ? (KS - 1) * NW * 64 : 1];
  __shared__ float part_sq[NORM ? (KS - 1) * 16 : 1];
  const int M = min(*m_dev, m_upper);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, l16 = lane & 15;
  const int m0 = blockIdx.y * (MB == 1 ? 16 : 64) + (MB == 1 ? 0 : (wave >> 1) * 32);
  int n0 = blockIdx.x * (MB == 1 ? 16 : 64) + (MB == 1 ? 0 : (wave & 1) * 32);
  if constexpr (MODE == 2) n0 = (int)blockIdx.x / (rope.dh >> 5) * rope.dh + (int)blockIdx.x % (rope.dh >> 5) * 16;
  if ((int)blockIdx.y * (MB == 1 ? 16 : 64) >= M) return;
  const T* W[NW];
  W[0] = (const T*)mats.w[MODE == 1 ? 0 : blockIdx.z];
  if (MODE == 1) W[NW - 1] = (const T*)mats.w[1];
  if (MODE == 2) W[NW - 1] = W[0] + (size_t)(rope.dh >> 1) * k;
  // rows past the end read the last one; their products are not stored
  const T *ar[MB], *wr[NW][MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    ar[i] = A + (size_t)min(m0 + i * 16 + l16, M - 1) * k;
#pragma unroll
    for (int w = 0; w < NW; ++w) wr[w][i] = W[w] + (size_t)min(n0 + i * 16 + l16, n - 1) * k;
  }
  f32x4 acc[NW][MB][MB];
#pragma unroll
  for (int w = 0; w < NW; ++w)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < MB; ++j) acc[w][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int chunks = sl_cdiv_dev(k, KC);
  float sq = 0.f;
  for (int c0 = KS > 1 ? wave : 0; c0 < chunks; c0 += KS * UC) {
    f32x4 a[UC][MB], b[UC][NW][MB], gain[NORM ? UC : 1];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int kk = (c0 + u * KS) * KC + 4 * g;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        a[u][i] = load4<T, VEC>(ar[i], kk, k);
#pragma unroll
        for (int w = 0; w < NW; ++w) b[u][w][i] = load4<T, VEC>(wr[w][i], kk, k);
      }
      if constexpr (NORM) gain[u] = load4<float, true>(norm.gain, kk, k);
    }
    if constexpr (NORM) {
#pragma unroll
      for (int u = 0; u < UC; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sq = fmaf(a[u][0][e], a[u][0][e], sq);
          a[u][0][e] *= gain[u][e];
        }
    }
#pragma unroll
    for (int u = 0; u < UC; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
              acc[w][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[u][w][j][e], a[u][i][e], acc[w][i][j], 0, 0, 0);
  }
  if constexpr (NORM) {        // lane group g holds its k of row l16
    sq += __shfl_xor(sq, 16, 64);
    sq += __shfl_xor(sq, 32, 64);
    if (wave > 0 && g == 0) part_sq[(wave - 1) * 16 + l16] = sq;
  }
  if constexpr (KS > 1) {
    if (wave > 0) {
#pragma unroll
      for (int w = 0; w < NW; ++w) part[((wave - 1) * NW + w) * 64 + lane] = acc[w][0][0];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int s = 0; s < KS - 1; ++s)
#pragma unroll
      for (int w = 0; w < NW; ++w) acc[w][0][0] += part[(s * NW + w) * 64 + lane];
    if constexpr (NORM) {
#pragma unroll
      for (int s = 0; s < KS - 1; ++s) sq += part_sq[s * 16 + l16];
      const float rstd = 1.0f / sqrtf(sq / (float)k + norm.eps);
#pragma unroll
      for (int w = 0; w < NW; ++w) acc[w][0][0] *= rstd;
    }
  }
  if constexpr (MODE == 2) {
    const int row = m0 + l16;
    if (row >= M) return;
    const int flat = rope.active_idx[row], seq = flat / rope.N, slot = flat - seq * rope.N, half = rope.dh >> 1;
    const int head = n0 / rope.dh, j = n0 - head * rope.dh + 4 * g;
    f32x4 lo = acc[0][0][0], hi = acc[1][0][0];
    if (blockIdx.z < 2) {
      const float* tab = reinterpret_cast<const float*>(rope.tab + (size_t)slot * half + j);
      const f32x4 t0 = *reinterpret_cast<const f32x4*>(tab), t1 = *reinterpret_cast<const f32x4*>(tab + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float c = e < 2 ? t0[2 * e] : t1[2 * (e - 2)], sn = e < 2 ? t0[2 * e + 1] : t1[2 * (e - 2) + 1];
        const float x = lo[e], y = hi[e];
        lo[e] = x * c - y * sn;
        hi[e] = y * c + x * sn;
      }
    }
    const size_t head_base = ((size_t)seq * rope.H + head) * rope.n_pad * rope.dh;
    if (blockIdx.z == 0) {
      float* p = rope.q + ((size_t)row * rope.H + head) * rope.dh + j;
      *reinterpret_cast<f32x4*>(p) = lo;
      *reinterpret_cast<f32x4*>(p + half) = hi;
    } else if (blockIdx.z == 1) {
      *reinterpret_cast<f32x4*>(rope.kc + head_base + kc_index(slot, j, rope.dh)) = lo;
      *reinterpret_cast<f32x4*>(rope.kc + head_base + kc_index(slot, j + half, rope.dh)) = hi;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        rope.vc[head_base + vc_index(slot, j + e, rope.dh)] = lo[e];
        rope.vc[head_base + vc_index(slot, j + half + e, rope.dh)] = hi[e];
      }
    }
    return;
  }
  const size_t coff = MODE == 0 ? (size_t)blockIdx.z * n : 0;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int row = m0 + i * 16 + l16;
    if (row >= M) continue;
    const size_t orow = out_row_map ? (size_t)out_row_map[row] : (size_t)row;
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      const int col = n0 + j * 16 + 4 * g;
      f32x4 v = acc[0][i][j];
      if constexpr (MODE == 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = v[e] / (1.0f + expf(-v[e])) * acc[NW - 1][i][j][e];
      }
      if (C_f32) {
        float* p = C_f32 + orow * ldc + coff + col;
        if (VEC && col + 4 <= n) *reinterpret_cast<f32x4*>(p) = v;
        else
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < n) p[e] = v[e];
      } else {
        T* p = C_T + orow * ldc + coff + col;
        if (VEC && col + 4 <= n) {
          if constexpr (sizeof(T) == 4) {
            if constexpr (RES) v += *reinterpret_cast<const f32x4*>(p);
            *reinterpret_cast<f32x4*>(p) = v;
          } else {
            bf16x4_t u;
#pragma unroll
            for (int e = 0; e < 4; ++e) u[e] = (bf16_t)v[e];
            *reinterpret_cast<bf16x4_t*>(p) = u;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < n) st<T>::stv(p + e, RES ? st<T>::ld(p + e) + v[e] : v[e]);
        }
      }
    }
  }
}

// a 16 x 16 tile per workgroup until that alone puts four workgroups on every CU; then the 64 x 64 form, if it
// still fills the chip (at 24 tiles of 64 x 64 the chip idles: that was the form before, 55 us against 4.4)
static bool small_tiles(int m_upper, int n, int nm) {
  const long small = (long)sl_cdiv(n, 16) * sl_cdiv(m_upper, 16) * nm, big = (long)sl_cdiv(n, 64) * sl_cdiv(m_upper, 64) * nm;
  return small <= 1024 || big < 192;
}

template <typename T, int MODE>
static int launch_generic(hipStream_t s, const void* A, const GenericMats& mats, int nm, const int32_t* m_dev, int m_upper,
                          int n, int k, float* C_f32, void* C_T, const int32_t* out_row_map, size_t ldc) {
  // 16-byte pieces need aligned rows (the model's dimensions are multiples of 8; plain weights are the caller's)
  uintptr_t bits = (uintptr_t)A | (uintptr_t)C_f32 | (uintptr_t)C_T;
  for (int i = 0; i < (MODE == 1 ? 2 : nm); ++i) bits |= (uintptr_t)mats.w[i];
  const bool vec = bits % 16 == 0 && k % 8 == 0 && n % 8 == 0 && ldc % 8 == 0;
#define GO(MB, VEC)                                                                                                   \
  hipLaunchKernelGGL((gemm_generic_kernel<T, MODE, MB, VEC, false, false, 4>),                                        \
                     dim3(sl_cdiv(n, MB == 1 ? 16 : 64), sl_cdiv(m_upper, MB == 1 ? 16 : 64), nm), dim3(256), 0, s,   \
                     (const T*)A, mats, m_dev, m_upper, n, k, C_f32, (T*)C_T, out_row_map, ldc, GenericNorm{}, GenericRope{})
  if (small_tiles(m_upper, n, nm)) { if (vec) GO(1, true); else GO(1, false); }
  else { if (vec) GO(2, true); else GO(2, false); }
#undef GO
  SL_LAUNCH_CHECK();
  return SL_OK;
}

int slk_gemm_generic(hipStream_t s, int dtype, const void* A, const void* const* W, int nm, const int32_t* m_dev,
                     int m_upper, int n, int k, float* C_f32, void* C_T, const int32_t* out_row_map, size_t ldc) {
  if (m_upper <= 0) return SL_OK;
  if (nm < 1 || nm > 3) return SL_EINVAL;
  GenericMats mats{};
  for (int i = 0; i < nm; ++i) mats.w[i] = W[i];
  return dtype == SL_BF16 ? launch_generic<bf16_t, 0>(s, A, mats, nm, m_dev, m_upper, n, k, C_f32, C_T, out_row_map, ldc)
                          : launch_generic<float, 0>(s, A, mats, nm, m_dev, m_upper, n, k, C_f32, C_T, out_row_map, ldc);
}

int slk_gemm_generic_swiglu(hipStream_t s, int dtype, const void* A, const void* w_gate, const void* w_up,
                            const int32_t* m_dev, int m_upper, int dff, int k, void* a) {
  if (m_upper <= 0) return SL_OK;
  const GenericMats mats{{w_gate, w_up, nullptr}};
  return dtype == SL_BF16 ? launch_generic<bf16_t, 1>(s, A, mats, 1, m_dev, m_upper, dff, k, nullptr, a, nullptr, dff)
                          : launch_generic<float, 1>(s, A, mats, 1, m_dev, m_upper, dff, k, nullptr, a, nullptr, dff);
}

// ---- fp32 layers without row-wise launches -----------------------------------------------------------------------
// Whether a launch of `nm` matrices of n columns can take its part of that: its 16 x 16 form only (the 64 x 64 form reads
// a row of A in many more workgroups than it saves launches for), and 16-byte pieces throughout.
int slk_generic_fused(int m_upper, int n, int k, int nm, uintptr_t bits) {
  return small_tiles(m_upper, n, nm) && bits % 16 == 0 && k % 8 == 0 && n % 8 == 0;
}

// The chunks that each of the four waves has in flight: all of them, where that is nine to twelve (reductions of 513 to 768) and no CU
// gets a second workgroup.  Three load latencies are then one, and the registers that takes (109 to 212, room for 2 to 4 workgroups
// where four chunks leave it for 5 to 8) cost nothing: launches of 33 to 256 workgroups 0.3 to 0.6 us less of 5 to 10 (80 workgroups,
// k = 688 5.2 -> 4.8, k = 768, Q|K|V 9.6 -> 9.1); up to 512 two latencies are fewer registers' worth (Q|K|V, k = 512 7.6 -> 8.0, k = 264
// 5.3 -> 6.0), and launches of more workgroups lose a round (steps of 300 rows, d = 512 198.6 -> 214.9 us, 600 rows, d = 264 137.4 -> 179.8).
static bool deep(long workgroups, int k) { return workgroups <= 256 && k > 2 * 4 * 4 * KC && k <= 12 * 4 * KC; }

template <int MODE, bool NORM, bool RES>
static int launch_fused(hipStream_t s, const float* A, const GenericMats& mats, int tiles, int nm, const int32_t* m_dev, int m_upper,
                        int n, int k, float* C, const int32_t* out_row_map, const GenericNorm& norm, const GenericRope& rope) {
  const dim3 grid(tiles, sl_cdiv(m_upper, 16), nm);
  const auto kernel = deep((long)tiles * grid.y * nm, k) ? gemm_generic_kernel<float, MODE, 1, true, NORM, RES, 12>
                                                         : gemm_generic_kernel<float, MODE, 1, true, NORM, RES, 4>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, A, mats, m_dev, m_upper, n, k, (float*)nullptr, C, out_row_map, (size_t)n, norm, rope);
  SL_LAUNCH_CHECK();
  return SL_OK;
}

int slk_generic_norm_qkv_rope(hipStream_t s, const void* x, const void* gain, float eps, const void* const* w, const int32_t* m_dev,
                              int m_upper, int H, int dh, int k, const int32_t* active_idx, int N, int n_pad, const void* rope_tab,
                              void* q, void* kc, void* vc) {
  if (m_upper <= 0) return SL_OK;
  if ((kc == nullptr) != (vc == nullptr) || dh % 32) return SL_EINVAL;
  return launch_fused<2, true, false>(s, (const float*)x, GenericMats{{w[0], w[1], w[2]}}, H * dh / 32, kc == nullptr ? 1 : 3, m_dev,
                                      m_upper, H * dh, k, nullptr, nullptr, GenericNorm{(const float*)gain, eps},
                                      GenericRope{active_idx, (const float2*)rope_tab, (float*)q, (float*)kc, (float*)vc, H, dh, N, n_pad});
}
int slk_generic_residual(hipStream_t s, const void* A, const void* w, const int32_t* m_dev, int m_upper, int n, int k, void* x) {
  if (m_upper <= 0) return SL_OK;
  return launch_fused<0, false, true>(s, (const float*)A, GenericMats{{w, nullptr, nullptr}}, sl_cdiv(n, 16), 1, m_dev, m_upper, n, k,
                                      (float*)x, nullptr, GenericNorm{}, GenericRope{});
}
int slk_generic_norm_swiglu(hipStream_t s, const void* x, const void* gain, float eps, const void* w_gate, const void* w_up,
                            const int32_t* m_dev, int m_upper, int dff, int k, void* a) {
  if (m_upper <= 0) return SL_OK;
  return launch_fused<1, true, false>(s, (const float*)x, GenericMats{{w_gate, w_up, nullptr}}, sl_cdiv(dff, 16), 1, m_dev, m_upper, dff,
                                      k, (float*)a, nullptr, GenericNorm{(const float*)gain, eps}, GenericRope{});
}
int slk_generic_norm_linear(hipStream_t s, const void* x, const void* gain, float eps, const void* w, const int32_t* m_dev, int m_upper,
                            int n, int k, void* y, const int32_t* out_row_map) {
  if (m_upper <= 0) return SL_OK;
  return launch_fused<0, true, false>(s, (const float*)x, GenericMats{{w, nullptr, nullptr}}, sl_cdiv(n, 16), 1, m_dev, m_upper, n, k,
                                      (float*)y, out_row_map, GenericNorm{(const float*)gain, eps}, GenericRope{});
}
