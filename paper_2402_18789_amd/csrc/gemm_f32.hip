// fp32 projections on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 sums).
//
//   TRANS = false:  C[M, N] = A[M, K] W[N, K]^T (+ bias[N]) (+ residual[M, N])
//   TRANS = true :  C[M, N] = A[M, K] W[K, N]   (+ bias[N]) (+ residual[M, N])
//
// The fp32 configuration's products are small (M <= a few hundred rows, N and K <= 1400): what bounds them is neither
// arithmetic nor bytes but the chain load -> product -> load of a block that walks K alone.  So a block owns a small
// tile (16 TM x 16 TN) and its wavefronts cut K among themselves, 16 columns at a time in turn, with the operands of
// U such steps in flight straight from global memory (16 bytes per lane; no LDS on the way in, nothing to wait for but
// the data); the wavefronts' sums meet in LDS and are added in wavefront order.  Against the element-wise kernel (one block
// per 64 x 64 outputs, operands staged in LDS 16 k at a time): 16 x 768 x 256 34 -> 8.5 us with the launch, 272 x 1376 x 256
// 43 -> 8.3, 256 x 4096 x 4096 717 -> 144 (60 TFLOP/s), 1024 x 4096 x 4096 837 -> 558; transposed 846 -> 159 and 988 -> 666.
#include "flexco_internal.h"

namespace flexco {
namespace {

template <bool TRANS, int TM, int TN, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_f32_mfma_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                                float* __restrict__ C, const float* __restrict__ bias,
                                                                const float* __restrict__ res, int M, int N, int K,
                                                                size_t lda, size_t ldw, size_t ldc, size_t ldr) {
  constexpr int U = TM * TN == 1 ? 6 : 2;     // steps of 16 k in flight per wavefront
  __shared__ f32x4 red[NW][TM * TN][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15, kq = 4 * (lane >> 4);
  const int m0 = blockIdx.y * 16 * TM, n0 = blockIdx.x * 16 * TN;
  // rows / columns past the end repeat the last one: read in bounds, never stored
  const float* ar[TM];
  const float* wr[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) ar[i] = A + (size_t)min(m0 + 16 * i + l16, M - 1) * lda;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = min(n0 + 16 * j + l16, N - 1);
    wr[j] = TRANS ? W + n : W + (size_t)n * ldw;
  }
  f32x4 acc[TM][TN] = {};
  const int steps = (K + 15) / 16;
  for (int c0 = wave; c0 < steps; c0 += NW * U) {
    f32x4 a[U][TM], w[U][TN];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c0 + u * NW) * 16 + kq;
      const bool ok = k < K;                   // K % 4 == 0: a lane's four k are inside or outside together
#pragma unroll
      for (int i = 0; i < TM; ++i) a[u][i] = ok ? *reinterpret_cast<const f32x4*>(ar[i] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (TRANS) {
#pragma unroll
          for (int e = 0; e < 4; ++e) w[u][j][e] = ok ? wr[j][(size_t)(k + e) * ldw] : 0.f;
        } else {
          w[u][j] = ok ? *reinterpret_cast<const f32x4*>(wr[j] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][e], w[u][j][e], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) red[wave][i * TN + j][lane] = acc[i][j];
  __syncthreads();
  // element p of the tile: register e of lane l of fragment f = row 4 (l / 16) + e, column l % 16
  for (int p = threadIdx.x; p < TM * TN * 256; p += 64 * NW) {
    const int f = p >> 8, e = (p >> 6) & 3, l = p & 63;
    float v = red[0][f][l][e];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][f][l][e];
    const int row = m0 + 16 * (f / TN) + 4 * (l >> 4) + e, col = n0 + 16 * (f % TN) + (l & 15);
    if (row < M && col < N) {
      if (bias) v += bias[col];
      if (res) v += res[(size_t)row * ldr + col];
      C[(size_t)row * ldc + col] = v;
    }
  }
}

template <int TM, int TN, int NW>
void launch_tiles(bool trans_w, const float* A, const float* W, float* C, const float* bias, const float* res, int M, int N,
                  int K, size_t lda, size_t ldw, size_t ldc, size_t ldr, hipStream_t s) {
  const dim3 grid((N + 16 * TN - 1) / (16 * TN), (M + 16 * TM - 1) / (16 * TM));
  if (trans_w)
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<true, TM, TN, NW>), grid, dim3(64 * NW), 0, s, A, W, C, bias, res, M, N, K, lda, ldw,
                       ldc, ldr);
  else
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<false, TM, TN, NW>), grid, dim3(64 * NW), 0, s, A, W, C, bias, res, M, N, K, lda,
                       ldw, ldc, ldr);
}

}  // namespace

int32_t launch_gemm_f32_mfma(const void* A, const void* W, void* C, const void* bias, const void* residual, int M, int N, int K,
                             size_t lda, size_t ldw, size_t ldc, size_t ldr, bool trans_w, hipStream_t s) {
  // 16-byte operand loads: whole groups of four k, rows 16-byte aligned (the transposed form reads W element by element)
  if (K % 4 != 0 || lda % 4 != 0 || !aligned16(A) || (!trans_w && (ldw % 4 != 0 || !aligned16(W)))) return FLEXCO_EUNSUPPORTED;
  // 16 x 16 tiles until they fill the chip's block slots (eight wavefronts each, four blocks per CU), then 32 x 32 ones, which
  // read half as many operand bytes per product
  const long tiles16 = (long)((M + 15) / 16) * ((N + 15) / 16);
  if (tiles16 <= 1024)
    launch_tiles<1, 1, 8>(trans_w, (const float*)A, (const float*)W, (float*)C, (const float*)bias, (const float*)residual, M, N, K,
                          lda, ldw, ldc, ldr, s);
  else
    launch_tiles<2, 2, 4>(trans_w, (const float*)A, (const float*)W, (float*)C, (const float*)bias, (const float*)residual, M, N, K,
                          lda, ldw, ldc, ldr, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of gemm_f32_mfma failed: %s", hipGetErrorString(e));
  return FLEXCO_OK;
}

}  // namespace flexco
