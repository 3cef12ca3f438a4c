// GEMM for fp32 storage: Y[m][n] = sum_k X[m][k] * W[n][k], fp32 operands and accumulation (v_mfma_f32_16x16x4_f32), W
// row-major (the fp32 packed layout).  fp32 is the reference mode: small models, few rows, one launch after the other, so
// a launch is a latency chain and the kernel is built to keep that chain short:
//   * a workgroup owns 16 MT rows x 16 NT columns and its eight waves split K, so a contraction of 256 is two trips of
//     loads per wave, and the waves' sums meet once in LDS (added in wave order: deterministic);
//   * operands go from memory to registers as they are used: lane l loads 16 bytes (features 4 (l / 16) .. +3 of a 16-feature
//     chunk) of row l % 16 of X and of W, and MFMA j of a chunk takes component j of both.  That visits the chunk's
//     features in another order than they are numbered, the same for both operands;
//   * up to four chunks of loads are requested before the first is multiplied.
// Measured per launch, portable kernel / this one: at 15 rows (N x K) 768 x 256 and 256 x 256 22 / 3.4 us, 256 x 688 64 / 4.5
// us; at 64 rows 4096 x 4096 565 / 53 us, the four products of a 4096-wide layer together 3457 / 587 us.
// SWIGLU (gate/up matrix, whose gate and up tiles alternate): a workgroup's two column tiles are a pair, and SiLU(gate) * up leaves
// the kernel instead of the sums (a launch of its own took 2.7 us beside 3.6 for the product at 15 rows, 1376 x 256; 3.6 together).
// HEADS: blockIdx.z = Medusa head, each with its own X, matrix and output (three heads of 1024 columns from one row: 9.9 us in
// three launches, 3.4 in one).
#include <type_traits>

#include "kernels.h"

namespace mdz {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Waves = 8;
constexpr int kF32Ahead = 4;  // chunks of 16 features requested together

struct HeadMatrices {
  const void* w[MDZ_MAX_HEADS];
  int64_t x_stride, y_stride;  // elements from head to head
};

__device__ inline float silu_f32(float v) { return v / (1.0f + expf(-v)); }

template <int MT, int NT, bool SWIGLU, typename Heads>
__global__ void __launch_bounds__(kF32Waves * 64)
    gemm_f32_kernel(const float* __restrict__ X, const float* __restrict__ W, float* __restrict__ Y, int M, int N, int K,
                    int64_t ldy, int vec_store, Heads heads) {
  static_assert(!SWIGLU || NT == 2, "gate and up tiles of a pair in one workgroup");
  if constexpr (std::is_same_v<Heads, HeadMatrices>) {
    W = static_cast<const float*>(heads.w[blockIdx.z]);
    X += blockIdx.z * heads.x_stride, Y += blockIdx.z * heads.y_stride;
  }
  __shared__ f32x4 sums[kF32Waves][MT * NT][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.y * 16 * MT, n0 = blockIdx.x * 16 * NT;
  const int chunks = K / 16, c_lo = wave * chunks / kF32Waves, c_hi = (wave + 1) * chunks / kF32Waves;
  const int r = lane & 15, kq = (lane >> 4) * 4;
  // rows beyond M (columns beyond N) repeat the last one and are not stored
  const float* xp[MT];
  const float* wp[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) xp[i] = X + (int64_t)min(m0 + 16 * i + r, M - 1) * K + kq;
#pragma unroll
  for (int j = 0; j < NT; ++j) wp[j] = W + (int64_t)min(n0 + 16 * j + r, N - 1) * K + kq;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c = c_lo; c < c_hi; c += kF32Ahead) {
    f32x4 x[kF32Ahead][MT], w[kF32Ahead][NT];
#pragma unroll
    for (int u = 0; u < kF32Ahead; ++u)
      if (c + u < c_hi) {
#pragma unroll
        for (int j = 0; j < NT; ++j) w[u][j] = *reinterpret_cast<const f32x4*>(wp[j] + (c + u) * 16);
#pragma unroll
        for (int i = 0; i < MT; ++i) x[u][i] = *reinterpret_cast<const f32x4*>(xp[i] + (c + u) * 16);
      }
#pragma unroll
    for (int u = 0; u < kF32Ahead; ++u)
      if (c + u < c_hi) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)  // W x X^T: a lane then holds four consecutive columns of one row
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][j][e], x[u][i][e], acc[i][j], 0, 0, 0);
      }
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) sums[wave][i * NT + j][lane] = acc[i][j];
  __syncthreads();
  // D layout of the 16x16 MFMA: lane holds row m = lane % 16, columns 4 (lane / 16) .. +3
  if constexpr (SWIGLU) {
    if (wave < MT) {
      f32x4 gate = sums[0][2 * wave][lane], up = sums[0][2 * wave + 1][lane];
#pragma unroll
      for (int w = 1; w < kF32Waves; ++w) gate += sums[w][2 * wave][lane], up += sums[w][2 * wave + 1][lane];
      const int m = m0 + 16 * wave + r;
      if (m < M) {
        f32x4 u;
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = silu_f32(gate[e]) * up[e];
        *reinterpret_cast<f32x4*>(Y + (int64_t)m * ldy + n0 / 2 + kq) = u;
      }
    }
    return;
  }
  for (int t = wave; t < MT * NT; t += kF32Waves) {
    f32x4 v = sums[0][t][lane];
#pragma unroll
    for (int w = 1; w < kF32Waves; ++w) v += sums[w][t][lane];
    const int m = m0 + 16 * (t / NT) + r, n = n0 + 16 * (t % NT) + kq;
    if (m >= M) continue;
    float* y = Y + (int64_t)m * ldy + n;
    if (vec_store && n + 4 <= N) {
      *reinterpret_cast<f32x4*>(y) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < N) y[e] = v[e];
    }
  }
}

bool gemm_f32_supported(int dtype, int K) { return dtype == MDZ_FP32 && K % 16 == 0; }

template <typename Heads>
static int launch_gemm_f32_t(const void* X, const void* Wp, float* Y, int M, int N, int K, int64_t ldy, int n_heads, const Heads& heads,
                             hipStream_t st) {
  if (M == 0 || N == 0) return MDZ_OK;
  const int vec = ldy % 4 == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
  // Two column tiles per workgroup halve the X requests; they are taken once one per workgroup would not fill the chip
  // twice over.  Row blocks of 64.
  const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4, nb_m = (M + 16 * mt - 1) / (16 * mt);
  const int nt = (int64_t)((N + 31) / 32) * nb_m * n_heads >= 2 * num_cus() ? 2 : 1;
#define MDZ_F32_CASE(MT, NT)                                                                                           \
  if (mt == MT && nt == NT) {                                                                                           \
    launch_timed(PROF_GEMM, gemm_f32_kernel<MT, NT, false, Heads>, dim3((N + 16 * NT - 1) / (16 * NT), nb_m, n_heads), kF32Waves * 64, 0, st, \
                 (const float*)X, (const float*)Wp, Y, M, N, K, ldy, vec, heads);                                        \
    MDZ_LAUNCH_CHECK();                                                                                                 \
    return MDZ_OK;                                                                                                      \
  }
  MDZ_F32_CASE(1, 1)
  MDZ_F32_CASE(2, 1)
  MDZ_F32_CASE(4, 1)
  MDZ_F32_CASE(1, 2)
  MDZ_F32_CASE(2, 2)
  MDZ_F32_CASE(4, 2)
#undef MDZ_F32_CASE
  MDZ_FAIL(MDZ_EUNSUPPORTED, "gemm: no fp32 kernel for %d rows", M);
}

struct OneMatrix {};
int launch_gemm_f32(const void* X, const void* Wp, float* Y, int M, int N, int K, int64_t ldy, hipStream_t st) {
  return launch_gemm_f32_t(X, Wp, Y, M, N, K, ldy, 1, OneMatrix{}, st);
}

// one product per Medusa head: head k's X starts k * x_stride elements after the first, its output k * y_stride (multiples of four)
int launch_gemm_f32_heads(const void* X, int64_t x_stride, const void* const* Wp, int n_heads, float* Y, int64_t y_stride, int M, int N,
                          int K, int64_t ldy, hipStream_t st) {
  HeadMatrices heads{};
  for (int k = 0; k < n_heads; ++k) heads.w[k] = Wp[k];
  heads.x_stride = x_stride, heads.y_stride = y_stride;
  return launch_gemm_f32_t(X, nullptr, Y, M, N, K, ldy, n_heads, heads, st);
}

// the gate/up product with the SwiGLU in its epilogue: U [M][N / 2], starting on 16 bytes
bool gemm_f32_swiglu_supported(int dtype, int N, int K) { return gemm_f32_supported(dtype, K) && N % 32 == 0; }
int launch_gemm_f32_swiglu(const void* X, const void* Wp, float* U, int M, int N, int K, hipStream_t st) {
  if (M == 0 || N == 0) return MDZ_OK;
  const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4, nb_m = (M + 16 * mt - 1) / (16 * mt);
  auto kernel = mt == 1 ? gemm_f32_kernel<1, 2, true, OneMatrix> : mt == 2 ? gemm_f32_kernel<2, 2, true, OneMatrix> : gemm_f32_kernel<4, 2, true, OneMatrix>;
  launch_timed(PROF_GEMM, kernel, dim3(N / 32, nb_m), kF32Waves * 64, 0, st, (const float*)X, (const float*)Wp, U, M, N, K, (int64_t)(N / 2), 1, OneMatrix{});
  MDZ_LAUNCH_CHECK();
  return MDZ_OK;
}

}  // namespace mdz
