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
//
// Where the tiles leave the chip's slots empty, a launch costs more than what it does: the norm of the rows and the gate of
// [gate | up] are then part of the product (layer of the fp32 configuration, 68 tokens 53 -> 49 us, one token 36 -> 31; hidden 4096,
// ffn 4096 8 tokens 97 -> 90, 68 tokens 245 -> 243).
#include "flexco_internal.h"

namespace flexco {
namespace {

// NORM: A holds the rows before their RMSNorm; a lane multiplies its pieces by the gain and adds their squares, and the sums are
// scaled by the row's 1 / rms at the end.  The normed rows (norm.h, for who reads them besides) and the copy of the input rows
// (norm.save) are written by the blocks of a row tile together, once they know it.
// GLU (TN = 2): the second fragment's columns are those of `up`, N further on; C = silu(gate) * up, and the rows the caller keeps of
// gate and up go to glu.save_gate / save_up.
template <bool TRANS, int TM, int TN, int NW, bool NORM, bool GLU>
__global__ __launch_bounds__(64 * NW) void gemm_f32_mfma_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                                float* __restrict__ C, const float* __restrict__ bias,
                                                                const float* __restrict__ res, int M, int N, int K,
                                                                size_t lda, size_t ldw, size_t ldc, size_t ldr, F32Norm norm,
                                                                F32Glu glu) {
  static_assert(!NORM || TM == 1, "one row tile per block");
  static_assert(!GLU || (TM == 1 && TN == 2), "a column tile of gate and one of up");
  constexpr int U = TM * TN == 1 ? 6 : TM * TN == 2 ? 3 : 2;     // steps of 16 k in flight per wavefront
  __shared__ f32x4 red[NW][TM * TN][64];
  __shared__ float squares[NORM ? NW : 1][16];
  f32x4 squared = {0.f, 0.f, 0.f, 0.f};      // (four short chains: no more rounding than the norm's own launch)
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15, kq = 4 * (lane >> 4);
  const int m0 = blockIdx.y * 16 * TM, n0 = blockIdx.x * 16 * (GLU ? 1 : TN);
  // rows / columns past the end repeat the last one: read in bounds, never stored
  const float* ar[TM];
  const float* wr[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) ar[i] = A + (size_t)min(m0 + 16 * i + l16, M - 1) * lda;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = GLU ? min(n0 + l16, N - 1) + j * N : min(n0 + 16 * j + l16, N - 1);
    wr[j] = TRANS ? W + n : W + (size_t)n * ldw;
  }
  f32x4 acc[TM][TN] = {};
  const int steps = (K + 15) / 16;
  for (int c0 = wave; c0 < steps; c0 += NW * U) {
    f32x4 a[U][TM], w[U][TN], g[NORM ? U : 1];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c0 + u * NW) * 16 + kq;
      const bool ok = k < K;                   // K % 4 == 0: a lane's four k are inside or outside together
      if constexpr (NORM) g[u] = *reinterpret_cast<const f32x4*>(norm.g + (ok ? k : 0));
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
    if constexpr (NORM) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          squared[e] += a[u][0][e] * a[u][0][e];
          a[u][0][e] *= g[u][e];
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
  if constexpr (NORM) {
    const float ss = sum_xor32(sum_xor16((squared[0] + squared[1]) + (squared[2] + squared[3])));
    if (lane < 16) squares[wave][l16] = ss;
  }
  __syncthreads();
  auto row_scale = [&](int r) {          // 1 / rms of row m0 + r
    float t = squares[0][r];
#pragma unroll
    for (int w = 1; w < (NORM ? NW : 1); ++w) t += squares[w][r];
    return 1.0f / sqrtf(t / K + norm.eps);
  };
  // element p of the tile: register e of lane l of fragment f = row 4 (l / 16) + e, column l % 16
  auto sum_of = [&](int f, int e, int l) {
    float v = red[0][f][l][e];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][f][l][e];
    return v;
  };
  if constexpr (GLU) {
    for (int p = threadIdx.x; p < 256; p += 64 * NW) {
      const int e = (p >> 6) & 3, l = p & 63, r = 4 * (l >> 4) + e, row = m0 + r, col = n0 + (l & 15);
      if (row >= M || col >= N) continue;
      float gate = sum_of(0, e, l), up = sum_of(1, e, l);
      if constexpr (NORM) { const float sc = row_scale(r); gate *= sc; up *= sc; }
      if (glu.save_gate && row >= glu.save_row0 && row < glu.save_row0 + glu.save_rows) {
        const size_t o = (size_t)(row - glu.save_row0) * N + col;
        glu.save_gate[o] = gate;
        glu.save_up[o] = up;
      }
      C[(size_t)row * ldc + col] = gate / (1.0f + __expf(-gate)) * up;
    }
  } else {
    for (int p = threadIdx.x; p < TM * TN * 256; p += 64 * NW) {
      const int f = p >> 8, e = (p >> 6) & 3, l = p & 63, r = 16 * (f / TN) + 4 * (l >> 4) + e;
      const int row = m0 + r, col = n0 + 16 * (f % TN) + (l & 15);
      float v = sum_of(f, e, l);
      if (row < M && col < N) {
        if constexpr (NORM) v *= row_scale(r);
        if (bias) v += bias[col];
        if (res) v += res[(size_t)row * ldr + col];
        C[(size_t)row * ldc + col] = v;
      }
    }
  }
  if constexpr (NORM) {
    if (norm.h || norm.save) {
      const int pieces = K / 4;
      for (int p = blockIdx.x * 64 * NW + threadIdx.x; p < 16 * pieces; p += gridDim.x * 64 * NW) {
        const int r = p / pieces, row = m0 + r, k = 4 * (p % pieces);
        if (row >= M) break;                      // (rows rise with p)
        f32x4 v = *reinterpret_cast<const f32x4*>(A + (size_t)row * lda + k);
        if (norm.save && row >= norm.save_row0 && row < norm.save_row0 + norm.save_rows)
          *reinterpret_cast<f32x4*>(norm.save + (size_t)(row - norm.save_row0) * K + k) = v;
        if (norm.h) {
          const f32x4 gv = *reinterpret_cast<const f32x4*>(norm.g + k);
          const float sc = row_scale(r);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = v[e] * sc * gv[e];
          *reinterpret_cast<f32x4*>(norm.h + (size_t)row * K + k) = v;
        }
      }
    }
  }
}

template <int TM, int TN, int NW>
void launch_tiles(bool trans_w, const float* A, const float* W, float* C, const float* bias, const float* res, int M, int N,
                  int K, size_t lda, size_t ldw, size_t ldc, size_t ldr, hipStream_t s) {
  const dim3 grid((N + 16 * TN - 1) / (16 * TN), (M + 16 * TM - 1) / (16 * TM));
  if (trans_w)
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<true, TM, TN, NW, false, false>), grid, dim3(64 * NW), 0, s, A, W, C, bias, res, M, N,
                       K, lda, ldw, ldc, ldr, F32Norm{}, F32Glu{});
  else
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<false, TM, TN, NW, false, false>), grid, dim3(64 * NW), 0, s, A, W, C, bias, res, M, N,
                       K, lda, ldw, ldc, ldr, F32Norm{}, F32Glu{});
}

// 16 x 16 tiles until they fill the chip's block slots (eight wavefronts each, four blocks per CU), then 32 x 32 ones, which
// read half as many operand bytes per product
bool small_tiles(int M, int N) { return (long)((M + 15) / 16) * ((N + 15) / 16) <= 1024; }

}  // namespace

bool gemm_f32_takes_norm(int M, int N, int K, const void* x, const void* W, const F32Norm& norm) {
  return K % 4 == 0 && small_tiles(M, N) && aligned16(x) && aligned16(W) && aligned16(norm.g) && aligned16(norm.h) && aligned16(norm.save);
}

// The gate within the product gives a block two fragments, half as many blocks and half as many steps in flight: it takes less where the
// plain product has more than a block of 16 x 16 per CU, or few steps.  Measured over layers of hidden 512 to 8192 (us, gate and up as
// one product and SwiGLU -> the gate within): 288 to 1024 tiles -1 to -40 (one token, 768 tiles, from K = 3072 on: +5 to +13), up to
// 256 tiles K = 512 to 1024 -0.5, 1536 +0.4, 2048 +1.7, 4096 +3.8, 8192 +12.
bool gemm_f32_takes_gate(int M, int F, int K) {
  return K <= 1024 || (long)((M + 15) / 16) * ((2 * F + 15) / 16) > 256;
}

int32_t launch_gemm_f32_norm_glu(const void* A, const void* W, void* C, const void* bias, int M, int N, int K, size_t ldc, const F32Norm* norm,
                                 const F32Glu* glu, hipStream_t s) {
  // (N: columns of C; the gated form's W has 2 N rows)
  if (K % 4 != 0 || !aligned16(A) || !aligned16(W) || !small_tiles(M, glu ? 2 * N : N)) return FLEXCO_EUNSUPPORTED;
  const dim3 grid((N + 15) / 16, (M + 15) / 16), block(512);
#define FLEXCO_F32_NG(TN_, NORM_, GLU_)                                                                                       \
  hipLaunchKernelGGL((gemm_f32_mfma_kernel<false, 1, TN_, 8, NORM_, GLU_>), grid, block, 0, s, (const float*)A, (const float*)W, \
                     (float*)C, (const float*)bias, (const float*)nullptr, M, N, K, (size_t)K, (size_t)K, ldc, (size_t)0,          \
                     norm ? *norm : F32Norm{}, glu ? *glu : F32Glu{})
  if (norm && glu) FLEXCO_F32_NG(2, true, true);
  else if (norm) FLEXCO_F32_NG(1, true, false);
  else FLEXCO_F32_NG(2, false, true);
#undef FLEXCO_F32_NG
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of gemm_f32_mfma failed: %s", hipGetErrorString(e));
  return FLEXCO_OK;
}

int32_t launch_gemm_f32_mfma(const void* A, const void* W, void* C, const void* bias, const void* residual, int M, int N, int K,
                             size_t lda, size_t ldw, size_t ldc, size_t ldr, bool trans_w, hipStream_t s) {
  // 16-byte operand loads: whole groups of four k, rows 16-byte aligned (the transposed form reads W element by element)
  if (K % 4 != 0 || lda % 4 != 0 || !aligned16(A) || (!trans_w && (ldw % 4 != 0 || !aligned16(W)))) return FLEXCO_EUNSUPPORTED;
  if (small_tiles(M, N))
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
