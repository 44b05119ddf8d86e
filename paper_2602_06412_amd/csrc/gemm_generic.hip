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
#include "sl_common.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KC = 16;    // k per chunk: four instructions
constexpr int UC = 4;     // chunks in flight per wave

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

// MODE 0: matrix z of the launch -> columns z * n .. of C_f32 / C_T.  MODE 1: w[0] = gate, w[1] = up: C_T =
// silu(gate) * up.  MB x MB blocks of 16 x 16 per wave; KS waves share a tile's k-chunks (MB == 1: 4, else 1).
template <typename T, int MODE, int MB, bool VEC>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const T* __restrict__ A, GenericMats mats,
                                                           const int32_t* __restrict__ m_dev, int m_upper, int n,
                                                           int k, float* __restrict__ C_f32, T* __restrict__ C_T,
                                                           const int32_t* __restrict__ out_row_map, size_t ldc) {
  constexpr int KS = MB == 1 ? 4 : 1, NW = MODE == 1 ? 2 : 1;
  __shared__ f32x4 part[KS > 1 ? (KS - 1) * NW * 64 : 1];
  const int M = min(*m_dev, m_upper);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, l16 = lane & 15;
  const int m0 = blockIdx.y * (MB == 1 ? 16 : 64) + (MB == 1 ? 0 : (wave >> 1) * 32);
  const int n0 = blockIdx.x * (MB == 1 ? 16 : 64) + (MB == 1 ? 0 : (wave & 1) * 32);
  if ((int)blockIdx.y * (MB == 1 ? 16 : 64) >= M) return;
  const T* W[NW];
  W[0] = (const T*)mats.w[MODE == 1 ? 0 : blockIdx.z];
  if (NW == 2) W[NW - 1] = (const T*)mats.w[1];
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
  for (int c0 = KS > 1 ? wave : 0; c0 < chunks; c0 += KS * UC) {
    f32x4 a[UC][MB], b[UC][NW][MB];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int kk = (c0 + u * KS) * KC + 4 * g;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        a[u][i] = load4<T, VEC>(ar[i], kk, k);
#pragma unroll
        for (int w = 0; w < NW; ++w) b[u][w][i] = load4<T, VEC>(wr[w][i], kk, k);
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
          if constexpr (sizeof(T) == 4) *reinterpret_cast<f32x4*>(p) = v;
          else {
            bf16x4_t u;
#pragma unroll
            for (int e = 0; e < 4; ++e) u[e] = (bf16_t)v[e];
            *reinterpret_cast<bf16x4_t*>(p) = u;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < n) st<T>::stv(p + e, v[e]);
        }
      }
    }
  }
}

template <typename T, int MODE>
static int launch_generic(hipStream_t s, const void* A, const GenericMats& mats, int nm, const int32_t* m_dev, int m_upper,
                          int n, int k, float* C_f32, void* C_T, const int32_t* out_row_map, size_t ldc) {
  // 16-byte pieces need aligned rows (the model's dimensions are multiples of 8; plain weights are the caller's)
  uintptr_t bits = (uintptr_t)A | (uintptr_t)C_f32 | (uintptr_t)C_T;
  for (int i = 0; i < (MODE == 1 ? 2 : nm); ++i) bits |= (uintptr_t)mats.w[i];
  const bool vec = bits % 16 == 0 && k % 8 == 0 && n % 8 == 0 && ldc % 8 == 0;
  // a 16 x 16 tile per workgroup until that alone puts four workgroups on every CU; then the 64 x 64 form, if it
  // still fills the chip (at 24 tiles of 64 x 64 the chip idles: that was the form before, 55 us against 4.4)
  const long small = (long)sl_cdiv(n, 16) * sl_cdiv(m_upper, 16) * nm, big = (long)sl_cdiv(n, 64) * sl_cdiv(m_upper, 64) * nm;
  const bool tiny = small <= 1024 || big < 192;
#define GO(MB, VEC)                                                                                                   \
  hipLaunchKernelGGL((gemm_generic_kernel<T, MODE, MB, VEC>),                                                         \
                     dim3(sl_cdiv(n, MB == 1 ? 16 : 64), sl_cdiv(m_upper, MB == 1 ? 16 : 64), nm), dim3(256), 0, s,   \
                     (const T*)A, mats, m_dev, m_upper, n, k, C_f32, (T*)C_T, out_row_map, ldc)
  if (tiny) { if (vec) GO(1, true); else GO(1, false); }
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
