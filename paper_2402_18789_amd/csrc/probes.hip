// Machine-ceiling probes for the benchmark: what this GPU delivers for the two resources the
// rooflines are quoted against, measured with the simplest possible kernels.  They compute
// nothing of the method; bench.py times them with events on the stream they are launched on.
#include "flexco_internal.h"
#include "device_types.h"

namespace flexco {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// The products in assembly and the fences around them as in the projection kernels, for the reasons given there.
#define FLEXCO_P_MFMA(c_, b_, a_) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c_) : "v"(b_), "v"(a_));
#define FLEXCO_P_FENCE(MT_, NT_)                                                                             \
  {                                                                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");                                                       \
    _Pragma("unroll") for (int i = 0; i < MT_; ++i)                                                          \
      _Pragma("unroll") for (int j = 0; j < NT_; ++j) asm volatile("" : "+a"(acc[i][j]));                    \
    __builtin_amdgcn_sched_barrier(0);                                                                       \
  }
typedef unsigned int frag_t __attribute__((ext_vector_type(4), may_alias));

// back-to-back v_mfma_f32_16x16x32_bf16, the projection kernels' product, on register operands: 32 independent
// accumulators per wavefront, one wavefront per SIMD
__global__ __launch_bounds__(256) void probe_mfma_kernel(int iters, float* sink) {
#ifdef __HIP_DEVICE_COMPILE__      // (the host pass knows no such assembly)
  const int lane = threadIdx.x & 63;
  bf16x8 a[8], b[4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // operand values spread over [-1, 1) like activations and weights, not zeros: the clock the
      // chip sustains depends on how many bits toggle
      const unsigned h = (unsigned)(lane * 8 + j + 64 * i) * 2654435761u;
      a[i][j] = (bf16_t)((float)(h >> 8 & 0xffff) / 32768.f - 1.f);
      if (i < 4) b[i][j] = (bf16_t)((float)(h >> 4 & 0xffff) / 32768.f - 1.f);
    }
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  frag_t af[8], bf[4];
#pragma unroll
  for (int i = 0; i < 8; ++i) af[i] = __builtin_bit_cast(frag_t, a[i]);
#pragma unroll
  for (int i = 0; i < 4; ++i) bf[i] = __builtin_bit_cast(frag_t, b[i]);
  FLEXCO_P_FENCE(8, 4)
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) FLEXCO_P_MFMA(acc[i][j], bf[j], af[i])
  }
  FLEXCO_P_FENCE(8, 4)
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) s += acc[i][j][0];
  if (s == 12345.678f) sink[0] = s;   // keeps the loop; never true in practice
#endif
}

// The same products with their operands fetched from LDS the way the projection kernels fetch them: a block of
// 4 wavefronts (2 x 2) owns a (32 MT) x (32 NT) tile, LDS holds one 64-column stage of both operand tiles (128-byte
// rows, 16-byte chunks XOR-swizzled by row), every 32-column slice costs a wavefront MT + NT ds_read_b128 for
// MT x NT products, and the fragments of a slice are fetched while the slice before it is multiplied.
// LOADS: per stage the block also brings a whole stage of tile bytes from global memory straight into a second
// LDS buffer (global_load_lds, 1 KB per wavefront instruction, from a few hundred KB that stay in cache) and ends
// the stage with a barrier - everything the projection kernels' k-loop does except wait for memory.
// What the matrix cores sustain when LDS feeds them (MT = NT = 4: the 128 x 128 tile, 8: the 256 x 256 tile).
#define FLEXCO_GP(p) ((const __attribute__((address_space(1))) void*)(p))
#define FLEXCO_LP(p) ((__attribute__((address_space(3))) void*)(p))
template <int MT, int NT, bool LOADS>
__global__ __launch_bounds__(256) void probe_mfma_lds_kernel(const bf16_t* __restrict__ src, int iters, float* sink) {
#ifdef __HIP_DEVICE_COMPILE__      // (the host pass knows no such assembly)
  constexpr int BM = 32 * MT, BN = 32 * NT, ST = (BM + BN) * 64;
  __shared__ __attribute__((aligned(1024))) bf16_t tile[ST];
  __shared__ __attribute__((aligned(1024))) bf16_t land[LOADS ? ST : 8];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int i = tid; i < ST; i += 256) {
    const unsigned h = (unsigned)i * 2654435761u;
    tile[i] = (bf16_t)((float)(h >> 8 & 0xffff) / 32768.f - 1.f);
  }
  __syncthreads();
  const int wm0 = (wave >> 1) * 16 * MT, wn0 = (wave & 1) * 16 * NT;
  const int l16 = lane & 15, q4 = lane >> 4;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int NLD = (BM + BN) / 32;                       // 1 KB load instructions per wavefront and stage
  const bf16_t* g = src + (size_t)(blockIdx.x & 7) * ST + lane * 8;
  frag_t a0[MT], b0[NT], a1[MT], b1[NT];
  // fragment q of a slice's MT + NT: rows of the first tile, then of the second
#define FLEXCO_P_FRAG(kk_, af_, bf_, q_)                                                                     \
  {                                                                                                          \
    const int r = (q_) < MT ? wm0 + (q_) * 16 + l16 : wn0 + ((q_) - MT) * 16 + l16;                          \
    const frag_t f = *reinterpret_cast<const frag_t*>(tile + ((q_) < MT ? r : BM + r) * 64 + ((((kk_) * 4 + q4) ^ ((r >> 1) & 7)) * 8)); \
    if ((q_) < MT) af_[(q_) < MT ? (q_) : 0] = f; else bf_[(q_) < MT ? 0 : (q_) - MT] = f;                   \
  }
  // a slice's products, a read of the next slice behind each until they are used up
#define FLEXCO_P_SLICE(af_, bf_, kk_, raf_, rbf_)                                                            \
  {                                                                                                          \
    _Pragma("unroll") for (int n = 0; n < MT * NT; ++n) {                                                    \
      FLEXCO_P_MFMA(acc[n / NT][n % NT], bf_[n % NT], af_[n / NT])                                           \
      if (n < MT + NT) FLEXCO_P_FRAG(kk_, raf_, rbf_, n)                                                     \
      __builtin_amdgcn_sched_barrier(0);                                                                     \
    }                                                                                                        \
  }
#pragma unroll
  for (int q = 0; q < MT + NT; ++q) FLEXCO_P_FRAG(0, a0, b0, q)
  FLEXCO_P_FENCE(MT, NT)
  for (int it = 0; it < iters; ++it) {
    if (LOADS) {
#pragma unroll
      for (int p = 0; p < NLD; ++p)
        __builtin_amdgcn_global_load_lds(FLEXCO_GP(g + (p * 4 + wave) * 512), FLEXCO_LP(land + (p * 4 + wave) * 512), 16, 0, 0);
    }
    FLEXCO_P_SLICE(a0, b0, 1, a1, b1)
    FLEXCO_P_SLICE(a1, b1, 0, a0, b0)
    if (LOADS) {
      __builtin_amdgcn_s_waitcnt(0x0F70 | (NLD & 15) | ((NLD >> 4) << 14));   // the stage before this one has landed
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
    }
    asm volatile("" ::: "memory");      // the fragments are read again in every iteration
  }
  if (LOADS) __builtin_amdgcn_s_waitcnt(0x0F70);   // nothing may land in LDS after the block ends
  FLEXCO_P_FENCE(MT, NT)
#undef FLEXCO_P_FRAG
#undef FLEXCO_P_SLICE
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) s += acc[i][j][0];
  if (LOADS) s += (float)land[tid];
  if (s == 12345.678f) sink[0] = s;
#endif
}

// every block streams its own contiguous piece with 16-byte loads, 8 in flight per lane
__global__ __launch_bounds__(256) void probe_read_kernel(const u32x4* __restrict__ src, size_t vec_per_block,
                                                         unsigned* sink) {
  const u32x4* p = src + (size_t)blockIdx.x * vec_per_block;
  u32x4 acc = {0, 0, 0, 0};
  for (size_t i = threadIdx.x; i + 7 * 256 < vec_per_block; i += 8 * 256) {
    u32x4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p[i + j * 256];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc ^= v[j];
  }
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) sink[0] = acc.x;   // keeps the loads
}

}  // namespace

}  // namespace flexco

using namespace flexco;

extern "C" int32_t flexco_probe_mfma(int32_t blocks, int32_t iters, void* sink, double* flops, void* stream) {
  clear_error();
  FLEXCO_CHECK(blocks > 0 && iters > 0 && sink && flops, FLEXCO_EINVAL, "probe_mfma: bad argument");
  hipLaunchKernelGGL(probe_mfma_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, iters, (float*)sink);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of probe_mfma failed: %s", hipGetErrorString(e));
  *flops = (double)blocks * 4.0 * iters * 32.0 * (2.0 * 16 * 16 * 32);
  return FLEXCO_OK;
}

extern "C" int32_t flexco_probe_mfma_lds(int32_t blocks, int32_t iters, int32_t tile, const void* src, size_t src_bytes,
                                         void* sink, double* flops, void* stream) {
  clear_error();
  FLEXCO_CHECK(blocks > 0 && iters > 0 && sink && flops, FLEXCO_EINVAL, "probe_mfma_lds: bad argument");
  FLEXCO_CHECK(tile == 128 || tile == 256, FLEXCO_EINVAL, "probe_mfma_lds: tile must be 128 or 256");
  const size_t need = (size_t)8 * 2 * tile * 64 * sizeof(bf16_t);       // 8 regions of one stage of both tiles
  FLEXCO_CHECK(!src || (aligned16(src) && src_bytes >= need), FLEXCO_EINVAL,
               "probe_mfma_lds: src must be 16-byte aligned and hold %zu bytes", need);
  hipStream_t s = (hipStream_t)stream;
  const bf16_t* p = (const bf16_t*)src;
  if (tile == 128 && src) hipLaunchKernelGGL((probe_mfma_lds_kernel<4, 4, true>), dim3(blocks), dim3(256), 0, s, p, iters, (float*)sink);
  else if (tile == 128) hipLaunchKernelGGL((probe_mfma_lds_kernel<4, 4, false>), dim3(blocks), dim3(256), 0, s, p, iters, (float*)sink);
  else if (src) hipLaunchKernelGGL((probe_mfma_lds_kernel<8, 8, true>), dim3(blocks), dim3(256), 0, s, p, iters, (float*)sink);
  else hipLaunchKernelGGL((probe_mfma_lds_kernel<8, 8, false>), dim3(blocks), dim3(256), 0, s, p, iters, (float*)sink);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of probe_mfma_lds failed: %s", hipGetErrorString(e));
  const double per_slice = (tile == 128 ? 16.0 : 64.0) * (2.0 * 16 * 16 * 32);
  *flops = (double)blocks * 4.0 * iters * 2.0 * per_slice;
  return FLEXCO_OK;
}

extern "C" int32_t flexco_probe_read(const void* src, size_t bytes, int32_t blocks, void* sink, double* bytes_read,
                                     void* stream) {
  clear_error();
  FLEXCO_CHECK(src && sink && bytes_read && blocks > 0, FLEXCO_EINVAL, "probe_read: bad argument");
  FLEXCO_CHECK(aligned16(src), FLEXCO_EINVAL, "probe_read: misaligned pointer");
  const size_t vec_per_block = bytes / 16 / (size_t)blocks / 2048 * 2048;   // whole rounds of 8 loads x 256 lanes
  FLEXCO_CHECK(vec_per_block > 0, FLEXCO_ESHAPE, "probe_read: %zu bytes are too few for %d blocks", bytes, blocks);
  hipLaunchKernelGGL(probe_read_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, (const u32x4*)src, vec_per_block,
                     (unsigned*)sink);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of probe_read failed: %s", hipGetErrorString(e));
  *bytes_read = (double)vec_per_block * 16.0 * blocks;
  return FLEXCO_OK;
}
