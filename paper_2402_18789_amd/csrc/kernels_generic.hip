// Element-wise, normalisation, RoPE/cache-append, LoRA and type-generic fallback kernels.
//
// Everything here computes in fp32 whatever the storage type, one thread block per row or
// per small tile.  These kernels carry the fp32 configuration end to end and the parts of
// the bf16 configurations that are bound by HBM traffic or are tiny (norms, RoPE, SwiGLU,
// rank-r LoRA products).  The dense bf16 contractions live in gemm_mfma.hip /
// attn_mfma.hip.
#include <algorithm>
#include <cmath>
#include <initializer_list>
#include <mutex>
#include <vector>
#include "flexco_internal.h"
#include "device_types.h"

namespace flexco {

// --------------------------------------------------------------------------------------
// reductions
// --------------------------------------------------------------------------------------
// Every lane gets the result.  Within a row of 16 lanes the partner's value comes through the data-parallel
// primitives, as an operand modifier of the addition itself (lane ^ 1, lane ^ 2, then the other quad of eight lanes
// and the other half of the row by mirrored reads - the quads, then the halves, are uniform by then); only the two
// exchanges between rows go through the LDS crossbar (row swaps for the last two steps as well, as the attention kernels use
// them in their softmax chain, were 3 - 5 % slower in a kernel of sixteen independent sums, which overlap their crossbar round trips).
template <int CTRL>
__device__ inline float dpp_read(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;
__device__ inline float wave_sum(float v) {
  v += dpp_read<DPP_XOR1>(v);
  v += dpp_read<DPP_XOR2>(v);
  v += dpp_read<DPP_HALF_MIRROR>(v);
  v += dpp_read<DPP_MIRROR>(v);
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}
__device__ inline float wave_max(float v) {
  v = fmaxf(v, dpp_read<DPP_XOR1>(v));
  v = fmaxf(v, dpp_read<DPP_XOR2>(v));
  v = fmaxf(v, dpp_read<DPP_HALF_MIRROR>(v));
  v = fmaxf(v, dpp_read<DPP_MIRROR>(v));
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  v = fmaxf(v, __shfl_xor(v, 32, 64));
  return v;
}
// sum over a block of 256 threads; every thread gets the result
__device__ inline float block_sum256(float v, float* red /* >= 4 floats of LDS */) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// --------------------------------------------------------------------------------------
// RMSNorm forward / backward (one block of 256 threads per row)
// --------------------------------------------------------------------------------------
// VEC: rows are read and written in 16-byte pieces (the host picks it when H is a multiple of the
// vector width and every pointer and row pitch is 16-byte aligned).
template <typename T, bool VEC>
__device__ inline void norm_row(const size_t row, const T* __restrict__ x, const T* __restrict__ g, T* __restrict__ h, int H, float eps,
                                T* __restrict__ save, int save_row0, int save_rows, float* red) {
  constexpr int N = Vec<T>::N;
  const T* xr = x + row * H;
  // rows [save_row0, save_row0 + save_rows) also leave a copy of the INPUT row in `save` (the finetune
  // window's rows of an activation graph pruning keeps, written by the kernel that reads them anyway)
  T* sv = (save && (int)row >= save_row0 && (int)row < save_row0 + save_rows) ? save + (row - save_row0) * H : nullptr;
  float ss = 0.f;
  if (VEC) {
    for (int i = threadIdx.x * N; i < H; i += 256 * N) {
      float v[N];
      Vec<T>::load(xr + i, v);
      if (sv) Vec<T>::store(sv + i, v);
#pragma unroll
      for (int j = 0; j < N; ++j) ss += v[j] * v[j];
    }
  } else {
    for (int i = threadIdx.x; i < H; i += 256) {
      const float v = ld(xr + i);
      if (sv) st(sv + i, v);
      ss += v * v;
    }
  }
  ss = block_sum256(ss, red);
  const float rstd = 1.0f / sqrtf(ss / H + eps);
  if (VEC) {
    for (int i = threadIdx.x * N; i < H; i += 256 * N) {
      float v[N], gv[N];
      Vec<T>::load(xr + i, v);
      Vec<T>::load(g + i, gv);
#pragma unroll
      for (int j = 0; j < N; ++j) v[j] = v[j] * rstd * gv[j];
      Vec<T>::store(h + row * H + i, v);
    }
  } else {
    for (int i = threadIdx.x; i < H; i += 256) st(h + row * H + i, ld(xr + i) * rstd * ld(g + i));
  }
}

template <typename T, bool VEC>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const T* __restrict__ x, const T* __restrict__ g,
                                                      T* __restrict__ h, int H, float eps, T* __restrict__ save,
                                                      int save_row0, int save_rows) {
  __shared__ float red[4];
  norm_row<T, VEC>(blockIdx.x, x, g, h, H, eps, save, save_row0, save_rows, red);
}

// x = sums + res, h = rmsnorm(x), bf16: the output projection's partial sums added by the norm that reads the product next
// (a launch of its own cost 4.7 us, as much as this kernel).  Eight wavefronts per row, everything a thread needs - the
// partial sums, the residual, the gain - on its way at once, the row in registers between the two passes.
constexpr int NORM_SUMS_VECS = 4;                 // 16-byte pieces per thread: rows of up to 512 x 8 x 4 elements
__global__ __launch_bounds__(512) void rmsnorm_sums_kernel(SplitSums sums, const bf16_t* __restrict__ res, bf16_t* __restrict__ x,
                                                           const bf16_t* __restrict__ g, bf16_t* __restrict__ h, int H, float eps,
                                                           bf16_t* __restrict__ save, int save_row0, int save_rows) {
  __shared__ float red[8];
  const size_t row = blockIdx.x, stride = (size_t)gridDim.x * H;
  bf16_t* sv = (save && (int)row >= save_row0 && (int)row < save_row0 + save_rows) ? save + (row - save_row0) * H : nullptr;
  bf16x8 v[NORM_SUMS_VECS];
  float ss = 0.f;
#pragma unroll
  for (int q = 0; q < NORM_SUMS_VECS; ++q) {
    const int i = (q * 512 + threadIdx.x) * 8;
    if (i < H) {
      const float* p = sums.part + row * H + i;
      const bf16x8 r8 = *reinterpret_cast<const bf16x8*>(res + row * H + i);
      float t[8];
      {
        const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) { t[j] = a[j]; t[4 + j] = b[j]; }
      }
      int sp = 1;
      for (; sp + 3 <= sums.splits; sp += 3) {      // three splits in flight, added in split order
        f32x4 a[3], b[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          a[u] = *reinterpret_cast<const f32x4*>(p + (sp + u) * stride);
          b[u] = *reinterpret_cast<const f32x4*>(p + (sp + u) * stride + 4);
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j) { t[j] += a[u][j]; t[4 + j] += b[u][j]; }
      }
      for (; sp < sums.splits; ++sp) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(p + sp * stride), b = *reinterpret_cast<const f32x4*>(p + sp * stride + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) { t[j] += a[j]; t[4 + j] += b[j]; }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[q][j] = (bf16_t)(t[j] + (float)r8[j]);
        ss += (float)v[q][j] * (float)v[q][j];
      }
      *reinterpret_cast<bf16x8*>(x + row * H + i) = v[q];
      if (sv) *reinterpret_cast<bf16x8*>(sv + i) = v[q];
    }
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) ss += red[w];
  const float rstd = 1.0f / sqrtf(ss / H + eps);
#pragma unroll
  for (int q = 0; q < NORM_SUMS_VECS; ++q) {
    const int i = (q * 512 + threadIdx.x) * 8;
    if (i < H) {
      const bf16x8 g8 = *reinterpret_cast<const bf16x8*>(g + i);
      bf16x8 o;
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = (bf16_t)((float)v[q][j] * rstd * (float)g8[j]);
      *reinterpret_cast<bf16x8*>(h + row * H + i) = o;
    }
  }
}

// v[0..N) = the N consecutive elements at `idx` of a product whose split-K partial sums still lie in
// part[split][stride]: added in split order and rounded to the storage type, exactly as the reduction
// kernel would have written them.
template <typename T, int N>
__device__ inline void load_split_sum(const float* __restrict__ part, int splits, size_t stride, size_t idx, float* v) {
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] = 0.f;
  for (int sp = 0; sp < splits; ++sp) {
    const float* p = part + (size_t)sp * stride + idx;
    if (N % 4 == 0) {
#pragma unroll
      for (int q = 0; q < N / 4; ++q) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(p + 4 * q);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 * q + j] += t[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < N; ++j) v[j] += p[j];
    }
  }
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] = (float)(T)v[j];
}

// dx = rstd * (g * dh) - x * rstd^3 * mean(x * g * dh)  (+ add);  hn (optional) = x rstd g, the row
// the forward norm produced (same arithmetic, same bits), for callers that need it again
//
// loss.accum (optional): one block more than rows adds the rows' losses, which are there since an earlier launch:
// *accum += scale * sum_i row[i], rows added in index order by strided partial sums of 256 threads.  (A launch of its own took
// 2.5 us of every head: fp32, hidden 256, 32 rows of 1000 logits 21.2 -> 19.5 us, 128 of 32000 178.7 -> 175.0.)
__device__ inline void loss_sum(const LossSum& l) {
  __shared__ float part[256];
  const int t = threadIdx.x;
  if (t < 256) {
    float s = 0.f;
    for (int i = t; i < l.n; i += 256) s += l.row[i];
    part[t] = s;
  }
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) part[t] += part[t + o];
    __syncthreads();
  }
  if (t == 0) l.accum[0] += l.scale * part[0];
}

template <typename T, bool VEC>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const T* __restrict__ x, const T* __restrict__ g,
                                                          const T* __restrict__ dh, const T* __restrict__ add,
                                                          T* __restrict__ dx, T* __restrict__ hn, int H, float eps,
                                                          const float* __restrict__ dh_part, int splits, size_t stride,
                                                          LossSum loss) {
  if (loss.accum && blockIdx.x == gridDim.x - 1) return loss_sum(loss);
  // dh_part: dh still lies as split-K partial sums (see load_split_sum); the row's sums are kept in LDS
  // between the two passes (dynamic shared memory of H floats, only then)
  extern __shared__ float dh_row[];
  __shared__ float red[4];
  constexpr int N = Vec<T>::N;
  const size_t row = blockIdx.x;
  const T* xr = x + row * H;
  const T* dr = dh + row * H;
  float ss = 0.f, sd = 0.f;
  if (VEC) {
    for (int i = threadIdx.x * N; i < H; i += 256 * N) {
      float v[N], gv[N], dv[N];
      Vec<T>::load(xr + i, v);
      Vec<T>::load(g + i, gv);
      if (dh_part) {
        load_split_sum<T, N>(dh_part, splits, stride, row * H + i, dv);
#pragma unroll
        for (int j = 0; j < N; ++j) dh_row[i + j] = dv[j];
      } else {
        Vec<T>::load(dr + i, dv);
      }
#pragma unroll
      for (int j = 0; j < N; ++j) { ss += v[j] * v[j]; sd += v[j] * gv[j] * dv[j]; }
    }
  } else {
    for (int i = threadIdx.x; i < H; i += 256) {
      float v = ld(xr + i);
      float d1;
      if (dh_part) { load_split_sum<T, 1>(dh_part, splits, stride, row * H + i, &d1); dh_row[i] = d1; }
      else d1 = ld(dr + i);
      ss += v * v;
      sd += v * ld(g + i) * d1;
    }
  }
  ss = block_sum256(ss, red);
  sd = block_sum256(sd, red);
  const float rstd = 1.0f / sqrtf(ss / H + eps);
  const float coef = rstd * rstd * rstd * sd / H;
  if (VEC) {
    for (int i = threadIdx.x * N; i < H; i += 256 * N) {
      float v[N], gv[N], dv[N], av[N];
      Vec<T>::load(xr + i, v);
      Vec<T>::load(g + i, gv);
      if (dh_part) {           // (each thread reads back what it wrote itself)
#pragma unroll
        for (int j = 0; j < N; ++j) dv[j] = dh_row[i + j];
      } else {
        Vec<T>::load(dr + i, dv);
      }
      if (add) Vec<T>::load(add + row * H + i, av);
      if (hn) {
        float hv[N];
#pragma unroll
        for (int j = 0; j < N; ++j) hv[j] = v[j] * rstd * gv[j];
        Vec<T>::store(hn + row * H + i, hv);
      }
#pragma unroll
      for (int j = 0; j < N; ++j) {
        v[j] = rstd * gv[j] * dv[j] - v[j] * coef;
        if (add) v[j] += av[j];
      }
      Vec<T>::store(dx + row * H + i, v);
    }
  } else {
    for (int i = threadIdx.x; i < H; i += 256) {
      if (hn) st(hn + row * H + i, ld(xr + i) * rstd * ld(g + i));
      float v = rstd * ld(g + i) * (dh_part ? dh_row[i] : ld(dr + i)) - ld(xr + i) * coef;
      if (add) v += ld(add + row * H + i);
      st(dx + row * H + i, v);
    }
  }
}

// The same backward for bf16 rows of up to 8192 elements, sixteen wavefronts per row: a thread owns four elements of
// each 4096-element stretch and keeps them in registers between the two passes, and every load of a row (x, g, the
// residual gradient, all split-K partial sums) is in flight at once.  A window of a few hundred rows gives the
// one-block-per-row kernel above one block of four wavefronts per CU, which waits out the latency of each of its
// loads in turn; here the chip holds four times as many wavefronts and each waits once.
// The sums over the row are taken in another order than above: hn may differ from the forward norm's row in the last
// bit of an element.
template <int IT>
__global__ __launch_bounds__(1024) void rmsnorm_bwd_wide_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ g,
                                                                const bf16_t* __restrict__ dh,
                                                                const bf16_t* __restrict__ add, bf16_t* __restrict__ dx,
                                                                bf16_t* __restrict__ hn, int H, float eps,
                                                                const float* __restrict__ dh_part, int splits,
                                                                size_t stride, LossSum loss) {
  if (loss.accum && blockIdx.x == gridDim.x - 1) return loss_sum(loss);
  __shared__ float red[2][16];
  const size_t row = blockIdx.x;
  const int wave = threadIdx.x >> 6;
  float v[IT][4], gv[IT][4], dv[IT][4], av[IT][4];
  auto ld4 = [](const bf16_t* p, float (&o)[4]) {
    const bf16x4 t = *reinterpret_cast<const bf16x4*>(p);
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (float)t[j];
  };
  auto st4 = [](bf16_t* p, const float (&o)[4]) {
    bf16x4 t;
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = (bf16_t)o[j];
    *reinterpret_cast<bf16x4*>(p) = t;
  };
  float ss = 0.f, sd = 0.f;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int i = (it * 1024 + (int)threadIdx.x) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[it][j] = gv[it][j] = dv[it][j] = av[it][j] = 0.f;
    if (i < H) {
      ld4(x + row * H + i, v[it]);
      ld4(g + i, gv[it]);
      if (add) ld4(add + row * H + i, av[it]);
      if (dh_part) {   // split-K partial sums, added in split order and rounded to the storage type (see load_split_sum)
        const float* p = dh_part + row * H + i;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        int sp = 0;
        for (; sp + 4 <= splits; sp += 4) {
          const f32x4 t0 = *reinterpret_cast<const f32x4*>(p + (size_t)sp * stride);
          const f32x4 t1 = *reinterpret_cast<const f32x4*>(p + (size_t)(sp + 1) * stride);
          const f32x4 t2 = *reinterpret_cast<const f32x4*>(p + (size_t)(sp + 2) * stride);
          const f32x4 t3 = *reinterpret_cast<const f32x4*>(p + (size_t)(sp + 3) * stride);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = (((acc[j] + t0[j]) + t1[j]) + t2[j]) + t3[j];
        }
        for (; sp < splits; ++sp) {
          const f32x4 t0 = *reinterpret_cast<const f32x4*>(p + (size_t)sp * stride);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] += t0[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) dv[it][j] = (float)(bf16_t)acc[j];
      } else {
        ld4(dh + row * H + i, dv[it]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) { ss += v[it][j] * v[it][j]; sd += v[it][j] * gv[it][j] * dv[it][j]; }
    }
  }
  ss = wave_sum(ss);
  sd = wave_sum(sd);
  if ((threadIdx.x & 63) == 0) { red[0][wave] = ss; red[1][wave] = sd; }
  __syncthreads();
  ss = sd = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) { ss += red[0][w]; sd += red[1][w]; }
  const float rstd = 1.0f / sqrtf(ss / H + eps);
  const float coef = rstd * rstd * rstd * sd / H;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int i = (it * 1024 + (int)threadIdx.x) * 4;
    if (i < H) {
      if (hn) {
        float hv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) hv[j] = v[it][j] * rstd * gv[it][j];
        st4(hn + row * H + i, hv);
      }
      float o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        o[j] = rstd * gv[it][j] * dv[it][j] - v[it][j] * coef;
        if (add) o[j] += av[it][j];
      }
      st4(dx + row * H + i, o);
    }
  }
}

// Rotation angles.  Pair i of a head turns by pos * theta^(-2 i / d).  The host hands over the frequencies in
// revolutions, theta^(-2 i / d) / (2 pi), as doubles (a kernel argument: pow and a double-precision sincos per
// (token, i) on the device were a third of these kernels' run time).  The device takes the fractional part of
// pos * rev in double precision (exact to 1e-10 of a turn at any position) and the sine and cosine of that
// fraction of a turn in single precision (angle in [0, 2 pi): about 5e-7 absolute).
constexpr int ROPE_MAX_HALF = 128;   // head_dim <= 256
struct RopeFreq {
  double rev[ROPE_MAX_HALF];
};
__device__ inline void rope_cos_sin(const RopeFreq& f, int i, int pos, float* c, float* sn) {
  const double r = (double)pos * f.rev[i];
  const float turn = (float)(r - floor(r));
  sincosf(turn * 6.283185307179586f, sn, c);
}

// --------------------------------------------------------------------------------------
// RoPE + cache append (Alg. 2: Forward then Append of Q, K, V).  One block per token.
//   qkv row = [q heads | k heads | v heads]; q is rotated in place, k is rotated and
//   written to the K pages, v is written to the (position-minor) V pages, and rows of
//   the finetune window also store the rotated q in the sequence's Q cache.
// --------------------------------------------------------------------------------------
// VEC: a thread rotates Vec<T>::N neighbouring pairs of one head with 16-byte accesses (head_dim / 2 a
// multiple of the vector width, every pointer 16-byte aligned); same arithmetic, same results.
// SUMS (with VEC): the rows lie as the projection's partial sums; q is written to qkv, k and v go to the pool only.
template <typename T, bool VEC, bool SUMS = false>
__global__ __launch_bounds__(SUMS ? 512 : 256) void rope_append_kernel(T* __restrict__ qkv, const int32_t* __restrict__ tok_pos,
                                                          const int32_t* __restrict__ slot, T* __restrict__ kp,
                                                          T* __restrict__ vp, int nq, int nkv, int d, int ps,
                                                          RopeFreq freq, int ft_tok0, int n_ft, int ft_pos0,
                                                          T* __restrict__ q_cache, SplitSums sums, const T* __restrict__ bias) {
  extern __shared__ float cs[];   // cos[d/2], sin[d/2]
  constexpr int THREADS = SUMS ? 512 : 256;
  const int t = blockIdx.x;
  const int pos = tok_pos[t];
  const int half = d >> 1;
  for (int i = threadIdx.x; i < half; i += THREADS) rope_cos_sin(freq, i, pos, &cs[i], &cs[half + i]);
  // the run of tokens this token's v row is written with (below): its first token and its length.  One lane per
  // neighbouring token looks at that token's slot and its predecessor's, all at once (a chain of dependent loads
  // along the run would cost more than the kernel's whole run time)
  constexpr int RUN = 16;
  __shared__ int run_info[2];
  if constexpr (VEC) {
    if (threadIdx.x < 64) {
      const int k = threadIdx.x, tt = t - (RUN - 1) + k;     // lanes 0 .. 31: tokens t - 15 .. t + 16
      bool first = false;                                     // tt begins a run (or lies past the batch)
      if (k < 2 * RUN) {
        if (tt >= (int)gridDim.x) first = true;
        else if (tt >= 0) {
          const int s1 = slot[tt];
          first = tt == 0 || slot[tt - 1] + 1 != s1 || (s1 % ps) % RUN == 0;
        }
      }
      const unsigned long long m = __ballot(first);
      if (k == 0) {
        const int k0 = 31 - __clz((unsigned)(m & 0xFFFFu));              // the last beginning at or before t
        const unsigned after = (unsigned)((m >> RUN) & 0xFFFFu);
        const int k1 = after ? RUN + __ffs(after) - 1 : 2 * RUN;         // the first beginning after t
        run_info[0] = t - (RUN - 1) + k0;
        run_info[1] = k1 - k0;
      }
    }
  }
  __syncthreads();
  const int qkv_dim = (nq + 2 * nkv) * d;
  T* row = qkv + (size_t)t * qkv_dim;
  const int sl = slot[t];
  const size_t page = sl / ps;
  const int pip = sl % ps;
  const bool is_ft = (t >= ft_tok0 && t < ft_tok0 + n_ft);
  // rotate q and k heads
  const T* vrow = row + (nq + nkv) * d;
  if constexpr (VEC) {
    constexpr int N = Vec<T>::N;
    const int hv = half / N;
    // P pieces of N elements of a token's row, `gap` elements apart.  Partial sums: those of four splits at a time are on
    // their way together (past the last split it is read again and left out), added in split order.
    auto load = [&](int token, int col, auto& v, int gap) {
      constexpr int P = sizeof(v) / (N * sizeof(float));
      if constexpr (SUMS) {
        constexpr int U = 4;
        const size_t stride = (size_t)gridDim.x * qkv_dim;
        const float* p = sums.part + (size_t)token * qkv_dim + col;
        float b[P][N] = {};
        if (bias)
#pragma unroll
          for (int q = 0; q < P; ++q) Vec<T>::load(bias + col + q * gap, b[q]);
#pragma unroll
        for (int q = 0; q < P; ++q)
#pragma unroll
          for (int e = 0; e < N; ++e) v[q][e] = 0.f;
        for (int sp = 0; sp < sums.splits; sp += U) {
          f32x4 t4[U][P][N / 4];
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < P; ++q)
#pragma unroll
              for (int e4 = 0; e4 < N / 4; ++e4)
                t4[u][q][e4] = *reinterpret_cast<const f32x4*>(p + min(sp + u, sums.splits - 1) * stride + q * gap + 4 * e4);
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (sp + u < sums.splits)
#pragma unroll
              for (int q = 0; q < P; ++q)
#pragma unroll
                for (int e = 0; e < N; ++e) v[q][e] += t4[u][q][e / 4][e % 4];
        }
#pragma unroll
        for (int q = 0; q < P; ++q)
#pragma unroll
          for (int e = 0; e < N; ++e) v[q][e] = (float)(T)(v[q][e] + b[q][e]);
      } else {
#pragma unroll
        for (int q = 0; q < P; ++q) Vec<T>::load(qkv + (size_t)token * qkv_dim + col + q * gap, v[q]);
      }
    };
    for (int idx = threadIdx.x; idx < (nq + nkv) * hv; idx += THREADS) {
      const int head = idx / hv, i = (idx % hv) * N;
      T* hp = row + head * d;
      float x[2][N], rlo[N], rhi[N];
      load(t, head * d + i, x, half);
      const float (&lo)[N] = x[0], (&hi)[N] = x[1];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float c = cs[i + j], sn = cs[half + i + j];
        rlo[j] = lo[j] * c - hi[j] * sn;
        rhi[j] = hi[j] * c + lo[j] * sn;
      }
      if (head < nq) {
        Vec<T>::store(hp + i, rlo);
        Vec<T>::store(hp + half + i, rhi);
        if (is_ft) {
          T* qc = q_cache + (size_t)(ft_pos0 + (t - ft_tok0)) * nq * d + head * d;
          Vec<T>::store(qc + i, rlo);
          Vec<T>::store(qc + half + i, rhi);
        }
      } else {
        const int kh = head - nq;
        T* dst = kp + ((page * nkv + kh) * ps + pip) * (size_t)d;
        Vec<T>::store(dst + i, rlo);
        Vec<T>::store(dst + half + i, rhi);
      }
    }
    // v: a channel's positions are the contiguous index of a V page, so one token's row is nkv d scattered elements
    // (these stores were half of the kernel's time).  Tokens whose slots follow each other inside a page (a chunk's
    // rows) form a run; a run begins at a page's first position, at a multiple of 16 positions, and where the slot
    // is not the one after the previous token's.  The blocks of a run's tokens share its v rows out by channels:
    // each reads its channels of every row of the run (no block ever writes them) and stores, per channel, the
    // run's positions side by side - 16-byte pieces for a run of 16, a contiguous stretch of the page per block.
    const int t0 = run_info[0], len = run_info[1];
    const int j = t - t0;
    const int pip0 = pip - j;
    const int nv = nkv * d / N;                       // 16-byte pieces of a v row
    const int v_lo = (int)((long)nv * j / len), v_hi = (int)((long)nv * (j + 1) / len);
    const bool whole = len == RUN && ps % N == 0;
    const int v0 = (nq + nkv) * d;
    // Partial sums: a piece of a row is a round trip per four splits, so a run's rows are not one thread's, one after the other:
    // each (row, piece) has a thread of its own, and a channel's positions meet in LDS (a chunk's tokens, this kernel: 8B shape
    // 128 tokens in four ranges 36 -> 10 us, 32B 300 tokens 67 -> 17, 600 tokens 99 -> 23; rows that lie whole take 11 to 14).
    if constexpr (SUMS) {
      if (len > 1) {
        __shared__ __attribute__((aligned(16))) T tile[THREADS * N];      // [channel][position in the run]
        const int at_once = THREADS / len;                                // pieces
        for (int p0 = v_lo; p0 < v_hi; p0 += at_once) {
          const int np = min(at_once, v_hi - p0), k = THREADS - 1 - threadIdx.x;      // (the threads with the least to rotate first)
          if (p0 > v_lo) __syncthreads();                                 // the tile's readers of the round before are done
          if (k < np * len) {
            const int jj = k / np, p = k % np;
            float v[1][N];
            load(t0 + jj, v0 + (p0 + p) * N, v, 0);
#pragma unroll
            for (int c = 0; c < N; ++c) tile[(p * N + c) * len + jj] = (T)v[0][c];
          }
          __syncthreads();
          const int per = whole ? RUN / N : len, n_out = np * N * per;    // stores per channel: 16 bytes, or one position
          for (int o = threadIdx.x; o < n_out; o += THREADS) {
            const int ch = p0 * N + o / per, at = o % per, kh = ch / d, i = ch % d;
            T* dst = vp + ((page * nkv + kh) * (size_t)d + i) * ps + pip0;
            if (whole) *reinterpret_cast<f32x4*>(dst + at * N) = *reinterpret_cast<const f32x4*>(tile + o * N);
            else dst[at] = tile[o];
          }
        }
        return;
      }
    }
    for (int vi = v_lo + THREADS - 1 - threadIdx.x; vi < v_hi; vi += THREADS) {      // (the threads with the least to rotate first)
      const int idx = vi * N, kh = idx / d, i = idx % d;
      T* dst = vp + ((page * nkv + kh) * (size_t)d + i) * ps + pip0;
      if (whole) {        // (all sixteen loads in flight before the first store)
        float rows[RUN][N];
#pragma unroll
        for (int jj = 0; jj < RUN; ++jj) {
          float v[1][N];
          load(t0 + jj, v0 + idx, v, 0);
#pragma unroll
          for (int c = 0; c < N; ++c) rows[jj][c] = v[0][c];
        }
#pragma unroll
        for (int c = 0; c < N; ++c) {
          float col[RUN];
#pragma unroll
          for (int jj = 0; jj < RUN; ++jj) col[jj] = rows[jj][c];
#pragma unroll
          for (int piece = 0; piece < RUN / N; ++piece) Vec<T>::store(dst + (size_t)c * ps + piece * N, &col[piece * N]);
        }
      } else {
        for (int jj = 0; jj < len; ++jj) {
          float v[1][N];
          load(t0 + jj, v0 + idx, v, 0);
#pragma unroll
          for (int c = 0; c < N; ++c) dst[(size_t)c * ps + jj] = (T)v[0][c];
        }
      }
    }
  } else {
    for (int idx = threadIdx.x; idx < (nq + nkv) * half; idx += 256) {
      const int head = idx / half, i = idx % half;
      T* hp = row + head * d;
      const float lo = ld(hp + i), hi = ld(hp + half + i);
      const float c = cs[i], sn = cs[half + i];
      const float rlo = lo * c - hi * sn, rhi = hi * c + lo * sn;
      if (head < nq) {
        st(hp + i, rlo);
        st(hp + half + i, rhi);
        if (is_ft) {
          T* qc = q_cache + (size_t)(ft_pos0 + (t - ft_tok0)) * nq * d + head * d;
          st(qc + i, rlo);
          st(qc + half + i, rhi);
        }
      } else {
        const int kh = head - nq;
        T* dst = kp + ((page * nkv + kh) * ps + pip) * (size_t)d;
        st(dst + i, rlo);
        st(dst + half + i, rhi);
      }
    }
    for (int idx = threadIdx.x; idx < nkv * d; idx += 256) {
      const int kh = idx / d, i = idx % d;
      vp[((page * nkv + kh) * (size_t)d + i) * ps + pip] = vrow[idx];
    }
  }
}

// Backward of the q/k/v rotation for a window: dqkv[n, (nq+2nkv)d] = [rope^T(dq) | rope^T(dk) | dv]
// dq rows are in the storage type, dk/dv rows are the (float) accumulator rows of the window.
// N consecutive floats with 16-byte loads
template <int N>
__device__ inline void load_f32_run(const float* p, float (&v)[N]) {
#pragma unroll
  for (int q4 = 0; q4 < N / 4; ++q4) {
    const f32x4 t = *reinterpret_cast<const f32x4*>(p + 4 * q4);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[4 * q4 + q] = t[q];
  }
}

// VEC as in rope_append_kernel
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void rope_bwd_pack_kernel(const T* __restrict__ dq, const float* __restrict__ dk,
                                                            const float* __restrict__ dv, T* __restrict__ dqkv,
                                                            int nq, int nkv, int d, RopeFreq freq, int win_start) {
  extern __shared__ float cs[];
  const int r = blockIdx.x;
  const int pos = win_start + r;
  const int half = d >> 1;
  // a grid of two blocks per row (short windows: the row's chain of loads is the whole run time) gives the
  // query heads to block 0 and the key heads and v to block 1
  const int part = gridDim.y == 2 ? (int)blockIdx.y : -1;
  const int h_lo = part == 1 ? nq : 0, h_hi = part == 0 ? nq : nq + nkv;
  for (int i = threadIdx.x; i < half; i += 256) rope_cos_sin(freq, i, pos, &cs[i], &cs[half + i]);
  __syncthreads();
  T* out = dqkv + (size_t)r * (nq + 2 * nkv) * d;
  if constexpr (VEC) {
    constexpr int N = Vec<T>::N;
    const int hv = half / N;
    for (int idx = h_lo * hv + threadIdx.x; idx < h_hi * hv; idx += 256) {
      const int head = idx / hv, i = (idx % hv) * N;
      float lo[N], hi[N], rlo[N], rhi[N];
      if (head < nq) {
        const T* p = dq + (size_t)r * nq * d + head * d;
        Vec<T>::load(p + i, lo);
        Vec<T>::load(p + half + i, hi);
      } else {
        const float* p = dk + (size_t)r * nkv * d + (head - nq) * d;
        load_f32_run<N>(p + i, lo);
        load_f32_run<N>(p + half + i, hi);
      }
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float c = cs[i + j], sn = cs[half + i + j];
        // transpose of the rotation: turn by the negative angle
        rlo[j] = lo[j] * c + hi[j] * sn;
        rhi[j] = hi[j] * c - lo[j] * sn;
      }
      Vec<T>::store(out + head * d + i, rlo);
      Vec<T>::store(out + head * d + half + i, rhi);
    }
    for (int idx = threadIdx.x * N; part != 0 && idx < nkv * d; idx += 256 * N) {
      float v[N];
      load_f32_run<N>(dv + (size_t)r * nkv * d + idx, v);
      Vec<T>::store(out + (nq + nkv) * d + idx, v);
    }
  } else {
  for (int idx = h_lo * half + threadIdx.x; idx < h_hi * half; idx += 256) {
    const int head = idx / half, i = idx % half;
    float lo, hi;
    if (head < nq) {
      const T* p = dq + (size_t)r * nq * d + head * d;
      lo = ld(p + i); hi = ld(p + half + i);
    } else {
      const float* p = dk + (size_t)r * nkv * d + (head - nq) * d;
      lo = p[i]; hi = p[half + i];
    }
    const float c = cs[i], sn = cs[half + i];
    // transpose of the rotation: turn by the negative angle
    const float rlo = lo * c + hi * sn, rhi = hi * c - lo * sn;
    st(out + head * d + i, rlo);
    st(out + head * d + half + i, rhi);
  }
  for (int idx = threadIdx.x; part != 0 && idx < nkv * d; idx += 256) {
    const float v = dv[(size_t)r * nkv * d + idx];
    st(out + (nq + nkv) * d + idx, v);
  }
  }
}

// --------------------------------------------------------------------------------------
// (IA)^3 bypass network (Sec. 4.1: Y = X + X (.) (l - 1) = X (.) l on the adapter's rows).
// Forward: one block per listed token; up to two column ranges of the row, each with its own vector;
// rows of the finetune window first keep the unscaled values (the other operand of the product, which
// the vector's gradient needs).
// --------------------------------------------------------------------------------------
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void ia3_scale_rows_kernel(T* __restrict__ buf, size_t ldb,
                                                             const int32_t* __restrict__ tok, Ia3ScaleArgs a) {
  constexpr int N = VEC ? Vec<T>::N : 1;
  const int t = tok[blockIdx.x];
  T* row = buf + (size_t)t * ldb;
  const bool is_ft = t >= a.ft_tok0 && t < a.ft_tok0 + a.n_ft;
  for (int sg = 0; sg < a.n_seg; ++sg) {
    const T* l = (const T*)a.l[sg];
    T* sv = (is_ft && a.save[sg]) ? (T*)a.save[sg] + (size_t)(a.ft_pos0 + (t - a.ft_tok0)) * a.ld_save[sg] : nullptr;
    T* p = row + a.col0[sg];
    for (int c = threadIdx.x * N; c < a.width[sg]; c += 256 * N) {
      float v[N], lv[N];
      if (VEC) {
        Vec<T>::load(p + c, v);
        Vec<T>::load(l + c, lv);
        if (sv) Vec<T>::store(sv + c, v);          // (a value of type T passes through float unchanged)
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] *= lv[j];
        Vec<T>::store(p + c, v);
      } else {
        v[0] = ld(p + c);
        if (sv) st(sv + c, v[0]);
        st(p + c, v[0] * ld(l + c));
      }
    }
  }
}

// Backward of the product Y = X (.) l over a window of n rows: G holds dY.  Per chunk of IA3_CHUNK rows and
// per column, part[chunk][c] = sum_r G[r, c] X[r, c] (the chunk's share of dl[c]), and G[r, c] <- G[r, c] l[c]
// (= dX) in place.  The second kernel adds the chunks in order into dl: no atomics, a fixed order.
constexpr int IA3_CHUNK = 8;
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void ia3_colgrad_kernel(Ia3ColgradArgs a, float* __restrict__ part, int n, int C) {
  constexpr int N = VEC ? Vec<T>::N : 1;
  T* __restrict__ const G = (T*)a.G[blockIdx.z];
  const T* __restrict__ const X = (const T*)a.X[blockIdx.z];
  const T* __restrict__ const l = (const T*)a.l[blockIdx.z];
  const size_t ldg = a.ldg, ldx = a.ldx;
  const int c = (blockIdx.x * 256 + threadIdx.x) * N;
  if (c >= C) return;
  const int r0 = blockIdx.y * IA3_CHUNK;
  float lv[N], acc[N], g[IA3_CHUNK][N], x[IA3_CHUNK][N];
  if (VEC) Vec<T>::load(l + c, lv); else lv[0] = ld(l + c);
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] = 0.f;
#pragma unroll
  for (int i = 0; i < IA3_CHUNK; ++i) {            // every load of the chunk in flight before the first use
    const int r = min(r0 + i, n - 1);
    if (VEC) { Vec<T>::load(G + (size_t)r * ldg + c, g[i]); Vec<T>::load(X + (size_t)r * ldx + c, x[i]); }
    else { g[i][0] = ld(G + (size_t)r * ldg + c); x[i][0] = ld(X + (size_t)r * ldx + c); }
  }
#pragma unroll
  for (int i = 0; i < IA3_CHUNK; ++i) {
    if (r0 + i >= n) break;
#pragma unroll
    for (int j = 0; j < N; ++j) { acc[j] += g[i][j] * x[i][j]; g[i][j] *= lv[j]; }
    if (VEC) Vec<T>::store(G + (size_t)(r0 + i) * ldg + c, g[i]); else st(G + (size_t)(r0 + i) * ldg + c, g[i][0]);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) part[((size_t)blockIdx.z * gridDim.y + blockIdx.y) * C + c + j] = acc[j];
}

__global__ __launch_bounds__(256) void ia3_colgrad_finalize_kernel(const float* __restrict__ part, int chunks, int C,
                                                                   float* __restrict__ dl0, float* __restrict__ dl1) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= C) return;
  float* const dl = blockIdx.y ? dl1 : dl0;
  part += (size_t)blockIdx.y * chunks * C;
  float acc = 0.f;
  for (int k0 = 0; k0 < chunks; k0 += 8) {   // eight loads in flight, added in chunk order
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = k0 + i < chunks ? part[(size_t)(k0 + i) * C + c] : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc += v[i];
  }
  dl[c] += acc;
}

// --------------------------------------------------------------------------------------
// SwiGLU forward / backward
// --------------------------------------------------------------------------------------
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void swiglu_kernel(const T* __restrict__ gu, T* __restrict__ act, int F,
                                                     T* __restrict__ save_gate, T* __restrict__ save_up, int save_row0, int save_rows) {
  constexpr int N = VEC ? Vec<T>::N : 1;
  const size_t row = blockIdx.y;
  const int i = (blockIdx.x * 256 + threadIdx.x) * N;
  if (i >= F) return;
  float g[N], u[N];
  if (VEC) { Vec<T>::load(gu + row * 2 * F + i, g); Vec<T>::load(gu + row * 2 * F + F + i, u); }
  else { g[0] = ld(gu + row * 2 * F + i); u[0] = ld(gu + row * 2 * F + F + i); }
  if (save_gate && (int)row >= save_row0 && (int)row < save_row0 + save_rows) {      // (values of T: stored as they are)
    const size_t o = (row - save_row0) * F + i;
    if (VEC) { Vec<T>::store(save_gate + o, g); Vec<T>::store(save_up + o, u); }
    else { st(save_gate + o, g[0]); st(save_up + o, u[0]); }
  }
#pragma unroll
  for (int j = 0; j < N; ++j) g[j] = g[j] / (1.0f + __expf(-g[j])) * u[j];
  if (VEC) Vec<T>::store(act + row * F + i, g); else st(act + row * F + i, g[0]);
}

// from saved gate, up and dact: dgu = [dgate | dup]
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const T* __restrict__ gate, const T* __restrict__ up,
                                                         const T* __restrict__ dact, T* __restrict__ dgu,
                                                         T* __restrict__ act, int F, const float* __restrict__ dact_part,
                                                         int splits, size_t stride) {
  constexpr int N = VEC ? Vec<T>::N : 1;
  const size_t row = blockIdx.y;
  const int i = (blockIdx.x * 256 + threadIdx.x) * N;
  if (i >= F) return;
  float g[N], u[N], da[N];
  if (VEC) { Vec<T>::load(gate + row * F + i, g); Vec<T>::load(up + row * F + i, u); }
  else { g[0] = ld(gate + row * F + i); u[0] = ld(up + row * F + i); }
  if (dact_part) load_split_sum<T, N>(dact_part, splits, stride, row * F + i, da);   // dact still lies as split-K partial sums
  else if (VEC) Vec<T>::load(dact + row * F + i, da);
  else da[0] = ld(dact + row * F + i);
  float dg[N], du[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const float sg = 1.0f / (1.0f + __expf(-g[j]));
    dg[j] = da[j] * u[j] * (sg + g[j] * sg * (1.0f - sg));
    du[j] = da[j] * g[j] * sg;
  }
  if (VEC) { Vec<T>::store(dgu + row * 2 * F + i, dg); Vec<T>::store(dgu + row * 2 * F + F + i, du); }
  else { st(dgu + row * 2 * F + i, dg[0]); st(dgu + row * 2 * F + F + i, du[0]); }
  if (act) {   // the rematerialised SwiGLU output (as remat_kernel computes it), for callers that need it again
#pragma unroll
    for (int j = 0; j < N; ++j) g[j] = g[j] / (1.0f + __expf(-g[j])) * u[j];
    if (VEC) Vec<T>::store(act + row * F + i, g); else st(act + row * F + i, g[0]);
  }
}

// The inputs of a window's adapted projections again (rematerialisation, Alg. 1): act = silu(gate) * up from the saved gate and
// up in the first n * act_blocks blocks, then the rows of up to two norms.  One launch, as none reads another (fp32
// configuration: two launches of 2.6 and 2.8 us and the gap between them).
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void remat_kernel(RematArgs a, int act_blocks) {
  __shared__ float red[4];
  constexpr int N = VEC ? Vec<T>::N : 1;
  int b = blockIdx.x;
  if (b >= a.n * act_blocks) {
    b -= a.n * act_blocks;
    const int z = b / a.n;
    norm_row<T, VEC>(b % a.n, (const T*)a.x[z], (const T*)a.g[z], (T*)a.h[z], a.H, a.eps, (T*)nullptr, 0, 0, red);
    return;
  }
  const T *gate = (const T*)a.gate, *up = (const T*)a.up;
  T* act = (T*)a.act;
  const int F = a.F;
  const size_t row = b / act_blocks;
  const int i = ((b % act_blocks) * 256 + threadIdx.x) * N;
  if (i >= F) return;
  float g[N], u[N];
  if (VEC) { Vec<T>::load(gate + row * F + i, g); Vec<T>::load(up + row * F + i, u); }
  else { g[0] = ld(gate + row * F + i); u[0] = ld(up + row * F + i); }
#pragma unroll
  for (int j = 0; j < N; ++j) g[j] = g[j] / (1.0f + __expf(-g[j])) * u[j];
  if (VEC) Vec<T>::store(act + row * F + i, g); else st(act + row * F + i, g[0]);
}

// N = 4 consecutive elements with one access, or one element
template <int N>
__device__ inline void load_run(const float* p, float (&v)[N]) {
  if constexpr (N == 4) { const f32x4 t = *reinterpret_cast<const f32x4*>(p); v[0] = t[0]; v[1] = t[1]; v[2] = t[2]; v[3] = t[3]; }
  else v[0] = *p;
}
template <int N>
__device__ inline void load_run(const bf16_t* p, float (&v)[N]) {
  if constexpr (N == 4) { const bf16x4 t = *reinterpret_cast<const bf16x4*>(p); v[0] = (float)t[0]; v[1] = (float)t[1]; v[2] = (float)t[2]; v[3] = (float)t[3]; }
  else v[0] = (float)*p;
}
template <int N, typename T>
__device__ inline void store_run(T* p, const float (&v)[N]) {
  typedef T run_t __attribute__((ext_vector_type(4)));
  if constexpr (N == 4) *reinterpret_cast<run_t*>(p) = run_t{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
  else *p = (T)v[0];
}

// The SwiGLU backward of a window with an (IA)^3 vector on the product, in one pass over gate, up and dact: per chunk of IA3_CHUNK
// rows and per column, part[chunk][c] = sum_r dact[r, c] act[r, c] with the rematerialised act, then dact <- dact (.) l and dgu as
// swiglu_bwd_kernel writes it; act and dact are rounded to the storage type where the separate kernels stored them, so the results
// are the same bits.  Bound by its bytes; four
// elements per thread, so that few rows give blocks enough, and four rows' loads in flight together.  205 x 14336 in an (IA)^3 layer: the sum of the
// product's partial sums, the rematerialisation, the column sums and the backward 9.0 + 5.6 + 6.2 + 6.2 us -> 16.5.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void ia3_swiglu_bwd_kernel(const T* __restrict__ gate, const T* __restrict__ up,
                                                             const T* __restrict__ dact, const T* __restrict__ l,
                                                             T* __restrict__ dgu, float* __restrict__ part, int n, int F,
                                                             const float* __restrict__ dact_part, int splits, size_t stride) {
  constexpr int N = VEC ? 4 : 1, R = 4, U = 4;
  static_assert(IA3_CHUNK % R == 0, "whole groups of rows");
  const int c = (blockIdx.x * 256 + threadIdx.x) * N;
  if (c >= F) return;
  const int r0 = blockIdx.y * IA3_CHUNK;
  float lv[N], acc[N];
  load_run<N>(l + c, lv);
#pragma unroll
  for (int j = 0; j < N; ++j) acc[j] = 0.f;
  for (int i0 = 0; i0 < IA3_CHUNK && r0 + i0 < n; i0 += R) {
    float g[R][N], u[R][N], da[R][N];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const size_t o = (size_t)min(r0 + i0 + i, n - 1) * F + c;
      load_run<N>(gate + o, g[i]);
      load_run<N>(up + o, u[i]);
      if (!dact_part) load_run<N>(dact + o, da[i]);
    }
    if (dact_part) {             // added in split order and rounded as load_split_sum does, U splits of all rows on their way at once
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) da[i][j] = 0.f;
      for (int sp = 0; sp < splits; sp += U) {
        float t[U][R][N];
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
          for (int i = 0; i < R; ++i)
            load_run<N>(dact_part + min(sp + q, splits - 1) * stride + (size_t)min(r0 + i0 + i, n - 1) * F + c, t[q][i]);
#pragma unroll
        for (int q = 0; q < U; ++q)
          if (sp + q < splits)
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
              for (int j = 0; j < N; ++j) da[i][j] += t[q][i][j];
      }
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) da[i][j] = (float)(T)da[i][j];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const size_t row = r0 + i0 + i;
      if ((int)row >= n) break;
      float dg[N], du[N];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const float gj = g[i][j], uj = u[i][j];
        acc[j] += da[i][j] * (float)(T)(gj / (1.0f + __expf(-gj)) * uj);
        const float d = (float)(T)(da[i][j] * lv[j]);
        const float sg = 1.0f / (1.0f + __expf(-gj));
        dg[j] = d * uj * (sg + gj * sg * (1.0f - sg));
        du[j] = d * gj * sg;
      }
      store_run<N>(dgu + row * 2 * F + c, dg);
      store_run<N>(dgu + row * 2 * F + F + c, du);
    }
  }
#pragma unroll
  for (int j = 0; j < N; ++j) part[(size_t)blockIdx.y * F + c + j] = acc[j];
}

// --------------------------------------------------------------------------------------
// strided row copy: dst row i = src row i, `width` units of V (uint4 = 16 bytes, or 4-byte words)
// --------------------------------------------------------------------------------------
template <typename V>
__global__ __launch_bounds__(256) void copy_rows_kernel(const char* __restrict__ src, size_t ld_src,
                                                        char* __restrict__ dst, size_t ld_dst, int width) {
  const size_t row = blockIdx.y;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= width) return;
  reinterpret_cast<V*>(dst + row * ld_dst)[i] = reinterpret_cast<const V*>(src + row * ld_src)[i];
}

// --------------------------------------------------------------------------------------
// LoRA building blocks on a row range.  S(i, j) denotes element (long index i, rank index j)
// of a LoRA matrix, addressed as S[i * s_i + j * s_j], so that the same kernels serve
// A [r, in] (s_i = 1, s_j = in) and B [out, r] (s_i = r, s_j = 1).
// A launch takes a batch of products (the targets of one projection, u and t, dA and dB): they are small, and a launch
// costs 4 - 6 us whatever it does (the fp32 configuration's co-served iteration: 51 -> 41 launches, 311 -> 255 us; 28 now).
// --------------------------------------------------------------------------------------
// acc[j] += sum over this thread's i of X[i] * S(i, j); low ranks: the loads of four passes at once (past the end they repeat
// the last element, unused)
template <typename T, int R>
__device__ inline void lora_row_sums(float (&acc)[R], const T* __restrict__ X, const T* __restrict__ S, size_t s_i, size_t s_j, int n_long,
                                     int r) {
  constexpr int P = R <= 8 ? 4 : R <= 16 ? 2 : 1;
  for (int i0 = threadIdx.x; i0 < n_long; i0 += 256 * P) {
    float xv[P], sv[P][R];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int i = min(i0 + 256 * p, n_long - 1);
      xv[p] = ld(X + i);
#pragma unroll
      for (int j = 0; j < R; ++j) sv[p][j] = j < r ? ld(S + (size_t)i * s_i + (size_t)j * s_j) : 0.f;
    }
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (i0 + 256 * p < n_long) {
#pragma unroll
        for (int j = 0; j < R; ++j) acc[j] += xv[p] * sv[p][j];
      }
  }
}

// out[m, j] = sum_i X[m, i] * S(i, j)        one block per row m; R = rank bound
template <typename T, int R>
__global__ __launch_bounds__(256) void lora_reduce_long_kernel(LoraBatch b, int r, const int32_t* __restrict__ row_idx) {
  __shared__ float red[4][R];
  const LoraProduct& p = b.p[blockIdx.y];
  const T* __restrict__ X = (const T*)p.X;
  const T* __restrict__ S = (const T*)p.S;
  float* __restrict__ out = p.U;
  const size_t ldx = p.ldx, s_i = p.s_i, s_j = p.s_j;
  const int n_long = p.n_long;
  const size_t mo = blockIdx.x;
  const size_t m = row_idx ? (size_t)row_idx[mo] : mo;
  float acc[R];
#pragma unroll
  for (int j = 0; j < R; ++j) acc[j] = 0.f;
  lora_row_sums<T, R>(acc, X + m * ldx, S, s_i, s_j, n_long, r);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const float v = wave_sum(acc[j]);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][j] = v;
  }
  __syncthreads();
  if (threadIdx.x < r) out[mo * r + threadIdx.x] = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

// Y[m, i] += scale * sum_j U[m, j] * S(i, j) for 16 rows from m0 on and 256 columns from i0 on; products z0 .. z1 - 1, which
// share their Y, one after the other.  The rows' elements are asked for together, ROWS = 16 or 4 of them: a launch of a few rows
// waits for its code, and one row of rank 64 takes 11.6 us in the form of sixteen.
template <typename T, int R, int ROWS>
__device__ inline void lora_expand_rows(float (&us)[64][R], const LoraBatch& b, int z0, int z1, int i0, int m0, int n, int r, float scale,
                                        const int32_t* __restrict__ row_idx) {
  const int i = i0 + threadIdx.x;
  const LoraProduct& y0 = b.p[z0];
  T* yp[ROWS];
  float yv[ROWS];
#pragma unroll
  for (int mm = 0; mm < ROWS; ++mm) {
    const int row = min(m0 + mm, n - 1);
    yp[mm] = (T*)y0.Y + (row_idx ? (size_t)row_idx[row] : (size_t)row) * y0.ldy + min(i, y0.n_long - 1);
  }
#pragma unroll
  for (int mm = 0; mm < ROWS; ++mm) yv[mm] = ld(yp[mm]);
  for (int z = z0; z < z1; ++z) {
    const LoraProduct& p = b.p[z];
    const T* __restrict__ S = (const T*)p.S;
    float sv[R];
#pragma unroll
    for (int j = 0; j < R; ++j) sv[j] = (j < r) ? ld(S + (size_t)min(i, p.n_long - 1) * p.s_i + (size_t)j * p.s_j) : 0.f;
    __syncthreads();
    for (int idx = threadIdx.x; idx < ROWS * R; idx += 256) {
      const int mm = idx / R, j = idx % R;
      us[mm][j] = (m0 + mm < n && j < r) ? p.U[(size_t)(m0 + mm) * r + j] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int mm = 0; mm < ROWS; ++mm) {
      float a = 0.f;
#pragma unroll
      for (int j = 0; j < R; ++j) a += us[mm][j] * sv[j];
      yv[mm] = (float)(T)(yv[mm] + scale * a);        // (each product is rounded to the storage type by itself)
    }
  }
  if (i < y0.n_long) {
#pragma unroll
    for (int mm = 0; mm < ROWS; ++mm)
      if (m0 + mm < n) st(yp[mm], yv[mm]);
  }
}
template <typename T, int R>
__device__ inline void lora_expand_block(float (&us)[64][R], const LoraBatch& b, int z0, int z1, int i0, int m0, int n, int r, float scale,
                                         const int32_t* __restrict__ row_idx) {
  if (n - m0 > 4) lora_expand_rows<T, R, 16>(us, b, z0, z1, i0, m0, n, r, scale, row_idx);
  else lora_expand_rows<T, R, 4>(us, b, z0, z1, i0, m0, n, r, scale, row_idx);
}

// grid (ceil(n_long/256), ceil(n/16), products), or, for products that share their Y, one z block that adds them one after the other
template <typename T, int R>
__global__ __launch_bounds__(256) void lora_expand_kernel(LoraBatch b, int n, int r, float scale,
                                                          const int32_t* __restrict__ row_idx) {
  __shared__ float us[64][R];
  const bool shared_y = gridDim.z == 1;
  lora_expand_block<T, R>(us, b, blockIdx.z, shared_y ? b.count : (int)blockIdx.z + 1, blockIdx.x * 256, blockIdx.y * 16, n, r, scale,
                          row_idx);
}

// Both of a few rows in one launch: u = x A^T, then y += scale u B^T, a block per row and product (down.p[z]: x, A, u;
// up.p[z]: B, y) that keeps u between them.
template <typename T, int R>
__global__ __launch_bounds__(256) void lora_rows_kernel(LoraBatch down, LoraBatch up, int r, float scale,
                                                        const int32_t* __restrict__ row_idx) {
  __shared__ float red[4][R], us[R];
  const size_t mo = blockIdx.x;
  const size_t m = row_idx ? (size_t)row_idx[mo] : mo;
  const LoraProduct& p = down.p[blockIdx.y];
  const T* __restrict__ X = (const T*)p.X + m * p.ldx;
  const T* __restrict__ S = (const T*)p.S;
  float acc[R];
#pragma unroll
  for (int j = 0; j < R; ++j) acc[j] = 0.f;
  lora_row_sums<T, R>(acc, X, S, p.s_i, p.s_j, p.n_long, r);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const float v = wave_sum(acc[j]);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][j] = v;
  }
  __syncthreads();
  if (threadIdx.x < R) {
    const float v = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
    us[threadIdx.x] = v;                          // (ranks past r: zero)
    if ((int)threadIdx.x < r) p.U[mo * r + threadIdx.x] = v;
  }
  __syncthreads();
  const LoraProduct& o = up.p[blockIdx.y];
  const T* __restrict__ B = (const T*)o.S;
  for (int i = threadIdx.x; i < o.n_long; i += 256) {
    float a = 0.f;
#pragma unroll
    for (int j = 0; j < R; ++j)
      if (j < r) a += us[j] * ld(B + (size_t)i * o.s_i + (size_t)j * o.s_j);
    T* y = (T*)o.Y + m * o.ldy + i;
    st(y, ld(y) + scale * a);
  }
}

// G(i, j) += scale * sum_m X[m, i] * U[m, j]      one thread per long index i, all ranks j
template <typename T, int R>
__device__ inline void lora_outer_block(float (&us)[64][R], const LoraProduct& p, int i, int n, int r, float scale) {
  const T* __restrict__ X = (const T*)p.X;
  const float* __restrict__ U = p.U;
  float* __restrict__ G = p.G;
  const size_t ldx = p.ldx, g_i = p.g_i, g_j = p.g_j;
  const int ic = min(i, p.n_long - 1);
  float acc[R];
#pragma unroll
  for (int j = 0; j < R; ++j) acc[j] = 0.f;
  for (int m0 = 0; m0 < n; m0 += 64) {
    __syncthreads();
    for (int idx = threadIdx.x; idx < 64 * R; idx += 256) {
      const int mm = idx / R, j = idx % R;
      us[mm][j] = (m0 + mm < n && j < r) ? U[(size_t)(m0 + mm) * r + j] : 0.f;
    }
    __syncthreads();
    const int mend = min(64, n - m0);
#pragma unroll 16
    for (int mm = 0; mm < mend; ++mm) {
      const float xv = ld(X + (size_t)(m0 + mm) * ldx + ic);
#pragma unroll
      for (int j = 0; j < R; ++j) acc[j] += xv * us[mm][j];
    }
  }
  if (i < p.n_long) {        // all loads of the accumulated gradient first (one round trip, not R in a row)
    float gv[R];
#pragma unroll
    for (int j = 0; j < R; ++j) gv[j] = j < r ? G[(size_t)i * g_i + (size_t)j * g_j] : 0.f;
#pragma unroll
    for (int j = 0; j < R; ++j)
      if (j < r) G[(size_t)i * g_i + (size_t)j * g_j] = gv[j] + scale * acc[j];
  }
}

// The outer products of a backward window (z = blockIdx.y) and, behind them, dx += scale sum_z t_z A_z by blocks of 16 rows: they
// read the same t and write nothing the other reads.
template <typename T, int R>
__global__ __launch_bounds__(256) void lora_outer_kernel(LoraBatch b, LoraBatch back, int n, int r, float scale) {
  __shared__ float us[64][R];
  if ((int)blockIdx.y < b.count) {
    const LoraProduct& p = b.p[blockIdx.y];
    if ((int)blockIdx.x * 256 < p.n_long) lora_outer_block<T, R>(us, p, blockIdx.x * 256 + threadIdx.x, n, r, scale);
  } else if ((int)blockIdx.x * 256 < back.p[0].n_long) {
    lora_expand_block<T, R>(us, back, 0, back.count, blockIdx.x * 256, (blockIdx.y - b.count) * 16, n, r, scale, nullptr);
  }
}

// --------------------------------------------------------------------------------------
// type-generic dense projection (fallback and the fp32 configuration)
//   TRANS_W = false: C[m, n] = sum_k A[m, k] W[n, k]      TRANS_W = true: ... W[k, n]
// 64 x 64 tile, BK = 16, 256 threads, 4 x 4 outputs per thread, fp32 accumulation.
// --------------------------------------------------------------------------------------
template <typename T, bool TRANS_W>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const T* __restrict__ A, const T* __restrict__ W,
                                                           T* __restrict__ C, const T* __restrict__ bias,
                                                           const T* __restrict__ residual, int M, int N, int K,
                                                           size_t lda, size_t ldw, size_t ldc, size_t ldr) {
  __shared__ float As[16][64 + 1];
  __shared__ float Ws[16][64 + 1];
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int idx = threadIdx.x; idx < 64 * 16; idx += 256) {
      const int mm = idx / 16, kk = idx % 16;
      As[kk][mm] = (m0 + mm < M && k0 + kk < K) ? ld(A + (size_t)(m0 + mm) * lda + k0 + kk) : 0.f;
      if (!TRANS_W) {
        Ws[kk][mm] = (n0 + mm < N && k0 + kk < K) ? ld(W + (size_t)(n0 + mm) * ldw + k0 + kk) : 0.f;
      }
    }
    if (TRANS_W) {
      for (int idx = threadIdx.x; idx < 64 * 16; idx += 256) {
        const int kk = idx / 64, nn = idx % 64;
        Ws[kk][nn] = (n0 + nn < N && k0 + kk < K) ? ld(W + (size_t)(k0 + kk) * ldw + n0 + nn) : 0.f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; b[i] = Ws[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      float v = acc[i][j];
      if (bias) v += ld(bias + n);
      if (residual) v += ld(residual + (size_t)m * ldr + n);
      st(C + (size_t)m * ldc + n, v);
    }
  }
}

// --------------------------------------------------------------------------------------
// host launchers
// --------------------------------------------------------------------------------------
#define DISPATCH_T(dtype, ...)                                   \
  do {                                                           \
    if ((dtype) == FLEXCO_BF16) { using T = bf16_t; __VA_ARGS__; } \
    else { using T = float; __VA_ARGS__; }                       \
  } while (0)

static int32_t post_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of %s failed: %s", what, hipGetErrorString(e));
  return FLEXCO_OK;
}

int32_t launch_gemm_generic(const void* A, const void* W, void* C, const void* bias, const void* residual, int M,
                            int N, int K, size_t lda, size_t ldw, size_t ldc, size_t ldr, bool trans_w, int dtype,
                            hipStream_t s) {
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  DISPATCH_T(dtype, {
    if (trans_w)
      hipLaunchKernelGGL((gemm_generic_kernel<T, true>), grid, dim3(256), 0, s, (const T*)A, (const T*)W, (T*)C,
                         (const T*)bias, (const T*)residual, M, N, K, lda, ldw, ldc, ldr);
    else
      hipLaunchKernelGGL((gemm_generic_kernel<T, false>), grid, dim3(256), 0, s, (const T*)A, (const T*)W, (T*)C,
                         (const T*)bias, (const T*)residual, M, N, K, lda, ldw, ldc, ldr);
  });
  return post_launch("gemm_generic");
}

// 16-byte row accesses are possible when the width is a multiple of 16 bytes and everything is aligned
static bool vec_ok(int dtype, int width, std::initializer_list<const void*> ptrs) {
  const int nvec = dtype == FLEXCO_BF16 ? 8 : 4;
  if (width % nvec != 0) return false;
  for (const void* p : ptrs)
    if (p && !aligned16(p)) return false;
  return true;
}
#define DISPATCH_TV(dtype, vec, ...)                                  \
  do {                                                               \
    if (vec) { constexpr bool VEC = true; DISPATCH_T(dtype, __VA_ARGS__); }  \
    else { constexpr bool VEC = false; DISPATCH_T(dtype, __VA_ARGS__); }     \
  } while (0)

int32_t launch_rmsnorm(const void* x, const void* g, void* h, int T_, int H, float eps, int dtype, hipStream_t s,
                       void* save, int save_row0, int save_rows) {
  if (T_ == 0) return FLEXCO_OK;
  const bool vec = vec_ok(dtype, H, {x, g, h, save});
  DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((rmsnorm_kernel<T, VEC>), dim3(T_), dim3(256), 0, s, (const T*)x,
                                             (const T*)g, (T*)h, H, eps, (T*)save, save_row0, save ? save_rows : 0));
  return post_launch("rmsnorm");
}

int32_t launch_rmsnorm_sums(const SplitSums& sums, const void* res, void* x, const void* g, void* h, int T_, int H, float eps,
                            hipStream_t s, void* save, int save_row0, int save_rows) {
  if (T_ == 0) return FLEXCO_OK;
  if (H > 512 * 8 * NORM_SUMS_VECS || !vec_ok(FLEXCO_BF16, H, {sums.part, res, x, g, h, save}))
    return fail(FLEXCO_EUNSUPPORTED, "rmsnorm_sums: not covered");
  hipLaunchKernelGGL(rmsnorm_sums_kernel, dim3(T_), dim3(512), 0, s, sums, (const bf16_t*)res, (bf16_t*)x, (const bf16_t*)g, (bf16_t*)h,
                     H, eps, (bf16_t*)save, save_row0, save ? save_rows : 0);
  return post_launch("rmsnorm_sums");
}

int32_t launch_rmsnorm_bwd(const void* x, const void* g, const void* dh, const void* add, void* dx, int T_, int H,
                           float eps, int dtype, hipStream_t s, void* hn, const float* dh_part, int splits, const LossSum* loss) {
  if (T_ == 0) return FLEXCO_OK;
  const bool vec = vec_ok(dtype, H, {x, g, dh, add, dx, hn, dh_part});
  const size_t shm = dh_part ? sizeof(float) * (size_t)H : 0;
  const LossSum ls = loss ? *loss : LossSum{nullptr, 0, 0.f, nullptr};
  const dim3 grid(T_ + (ls.accum ? 1 : 0));
  // bf16 rows of up to 8192 elements: sixteen wavefronts per row
  if (dtype == FLEXCO_BF16 && vec && H <= 8192) {
#define FLEXCO_NORM_BWD_WIDE(IT_)                                                                                  \
    hipLaunchKernelGGL((rmsnorm_bwd_wide_kernel<IT_>), grid, dim3(1024), 0, s, (const bf16_t*)x,                \
                       (const bf16_t*)g, (const bf16_t*)dh, (const bf16_t*)add, (bf16_t*)dx, (bf16_t*)hn, H, eps,   \
                       dh_part, splits, (size_t)T_ * H, ls)
    if (H <= 4096) FLEXCO_NORM_BWD_WIDE(1); else FLEXCO_NORM_BWD_WIDE(2);
#undef FLEXCO_NORM_BWD_WIDE
    return post_launch("rmsnorm_bwd");
  }
  DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((rmsnorm_bwd_kernel<T, VEC>), grid, dim3(256), shm, s, (const T*)x,
                                             (const T*)g, (const T*)dh, (const T*)add, (T*)dx, (T*)hn, H, eps, dh_part,
                                             splits, (size_t)T_ * H, ls));
  return post_launch("rmsnorm_bwd");
}

// The frequencies of a (theta, head_dim) pair, computed once (a model has one pair; a lock guards the few cached ones).
static int32_t rope_freq(const flexco_layer_cfg& c, RopeFreq* out) {
  const int half = c.head_dim / 2;
  if (half > ROPE_MAX_HALF) return fail(FLEXCO_EUNSUPPORTED, "rotary embedding: head_dim %d above %d", c.head_dim, 2 * ROPE_MAX_HALF);
  struct Entry { float theta; int d; RopeFreq f; };
  static std::mutex mu;
  static std::vector<Entry> cache;
  std::lock_guard<std::mutex> lock(mu);
  for (const Entry& e : cache)
    if (e.theta == c.rope_theta && e.d == c.head_dim) { *out = e.f; return FLEXCO_OK; }
  Entry e;
  e.theta = c.rope_theta; e.d = c.head_dim;
  for (int i = 0; i < ROPE_MAX_HALF; ++i)
    e.f.rev[i] = i < half ? std::pow((double)c.rope_theta, -2.0 * (double)i / (double)c.head_dim) / 6.283185307179586476925 : 0.0;
  if (cache.size() >= 16) cache.clear();
  cache.push_back(e);
  *out = e.f;
  return FLEXCO_OK;
}

bool rope_append_vec(const flexco_layer_cfg& c, const void* qkv, const flexco_kv_pool& pool, const void* q_cache) {
  return c.head_dim % 2 == 0 && vec_ok(c.dtype, c.head_dim / 2, {qkv, pool.k_pages, pool.v_pages, q_cache});
}

int32_t launch_rope_append(const flexco_layer_cfg& c, void* qkv, const int32_t* tok_pos, const int32_t* slot,
                           const flexco_kv_pool& pool, int T_, int ft_tok0, int n_ft, int ft_pos0, void* q_cache,
                           hipStream_t s, const SplitSums* sums, const void* bias) {
  if (T_ == 0) return FLEXCO_OK;
  const size_t shm = sizeof(float) * c.head_dim;
  RopeFreq freq;
  FLEXCO_TRY(rope_freq(c, &freq));
  const bool vec = rope_append_vec(c, qkv, pool, q_cache);
  if (sums && sums->splits > 1) {
    if (!vec || c.dtype != FLEXCO_BF16 || !aligned16(bias)) return fail(FLEXCO_EUNSUPPORTED, "rope_append: partial sums not covered");
    hipLaunchKernelGGL((rope_append_kernel<bf16_t, true, true>), dim3(T_), dim3(512), shm, s, (bf16_t*)qkv, tok_pos, slot,
                       (bf16_t*)pool.k_pages, (bf16_t*)pool.v_pages, c.n_q_heads, c.n_kv_heads, c.head_dim, c.page_size, freq,
                       ft_tok0, n_ft, ft_pos0, (bf16_t*)q_cache, *sums, (const bf16_t*)bias);
    return post_launch("rope_append");
  }
  DISPATCH_TV(c.dtype, vec, hipLaunchKernelGGL((rope_append_kernel<T, VEC>), dim3(T_), dim3(256), shm, s, (T*)qkv, tok_pos,
                                               slot, (T*)pool.k_pages, (T*)pool.v_pages, c.n_q_heads, c.n_kv_heads,
                                               c.head_dim, c.page_size, freq, ft_tok0, n_ft, ft_pos0,
                                               (T*)q_cache, SplitSums{}, (const T*)nullptr));
  return post_launch("rope_append");
}

int32_t launch_rope_bwd_pack(const flexco_layer_cfg& c, const void* dq, const float* dk_rows, const float* dv_rows,
                             void* dqkv, int win_start, int n, hipStream_t s) {
  const size_t shm = sizeof(float) * c.head_dim;
  if (n == 0) return FLEXCO_OK;
  RopeFreq freq;
  FLEXCO_TRY(rope_freq(c, &freq));
  const dim3 grid(n, n <= 512 ? 2 : 1);   // few rows: two blocks per row
  // 16-byte accesses: also the float rows of dk / dv (their row pitch nkv d floats is a multiple of 16 bytes then)
  const bool vec = c.head_dim % 2 == 0 && vec_ok(c.dtype, c.head_dim / 2, {dq, dk_rows, dv_rows, dqkv});
  DISPATCH_TV(c.dtype, vec, hipLaunchKernelGGL((rope_bwd_pack_kernel<T, VEC>), grid, dim3(256), shm, s, (const T*)dq,
                                               dk_rows, dv_rows, (T*)dqkv, c.n_q_heads, c.n_kv_heads, c.head_dim,
                                               freq, win_start));
  return post_launch("rope_bwd_pack");
}

int32_t launch_ia3_scale_rows(void* buf, size_t ld, const int32_t* tok, int n_tok, const Ia3ScaleArgs& a, int dtype,
                              hipStream_t s) {
  if (n_tok == 0 || a.n_seg == 0) return FLEXCO_OK;
  const int vn = dtype == FLEXCO_BF16 ? 8 : 4;
  bool vec = ld % vn == 0 && aligned16(buf);
  for (int sg = 0; sg < a.n_seg; ++sg)
    vec = vec && a.col0[sg] % vn == 0 && a.width[sg] % vn == 0 && aligned16(a.l[sg]) && aligned16(a.save[sg]) &&
          a.ld_save[sg] % vn == 0;
  DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((ia3_scale_rows_kernel<T, VEC>), dim3(n_tok), dim3(256), 0, s, (T*)buf, ld,
                                             tok, a));
  return post_launch("ia3_scale_rows");
}

int32_t launch_ia3_colgrad(const Ia3ColgradArgs& a, int n_seg, float* part, int n, int C, int dtype, hipStream_t s) {
  if (n == 0 || C == 0) return FLEXCO_OK;
  const int chunks = (n + IA3_CHUNK - 1) / IA3_CHUNK;
  const int vn = dtype == FLEXCO_BF16 ? 8 : 4;
  bool vec = C % vn == 0 && a.ldg % vn == 0 && a.ldx % vn == 0;
  for (int i = 0; i < n_seg; ++i) vec = vec && aligned16(a.G[i]) && aligned16(a.X[i]) && aligned16(a.l[i]);
  const int per = 256 * (vec ? vn : 1);
  DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((ia3_colgrad_kernel<T, VEC>), dim3((C + per - 1) / per, chunks, n_seg), dim3(256), 0,
                                             s, a, part, n, C));
  hipLaunchKernelGGL(ia3_colgrad_finalize_kernel, dim3((C + 255) / 256, n_seg), dim3(256), 0, s, part, chunks, C, a.dl[0], a.dl[1]);
  return post_launch("ia3_colgrad");
}

int32_t launch_ia3_swiglu_bwd(const void* gate, const void* up, const void* dact, const void* l, void* dgu, float* part, float* dl,
                              int n, int F, int dtype, hipStream_t s, const float* dact_part, int splits) {
  if (n == 0) return FLEXCO_OK;
  const bool vec = vec_ok(dtype, F, {gate, up, dact, l, dgu, dact_part});
  const int per = 256 * (vec ? 4 : 1), chunks = (n + IA3_CHUNK - 1) / IA3_CHUNK;
  DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((ia3_swiglu_bwd_kernel<T, VEC>), dim3((F + per - 1) / per, chunks), dim3(256), 0, s,
                                             (const T*)gate, (const T*)up, (const T*)dact, (const T*)l, (T*)dgu, part, n, F, dact_part,
                                             splits, (size_t)n * F));
  hipLaunchKernelGGL(ia3_colgrad_finalize_kernel, dim3((F + 255) / 256), dim3(256), 0, s, part, chunks, F, dl, (float*)nullptr);
  return post_launch("ia3_swiglu_bwd");
}

int32_t launch_swiglu(const void* gu, void* act, int T_, int F, int dtype, hipStream_t s, void* save_gate, void* save_up,
                      int save_row0, int save_rows) {
  if (T_ == 0) return FLEXCO_OK;
  const bool vec = vec_ok(dtype, F, {gu, act, save_gate, save_up});
  const int per = 256 * (vec ? (dtype == FLEXCO_BF16 ? 8 : 4) : 1);
  DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((swiglu_kernel<T, VEC>), dim3((F + per - 1) / per, T_), dim3(256), 0, s,
                                             (const T*)gu, (T*)act, F, (T*)save_gate, (T*)save_up, save_row0, save_rows));
  return post_launch("swiglu");
}

int32_t launch_swiglu_bwd(const void* gate, const void* up, const void* dact, void* dgu, int n, int F, int dtype,
                          hipStream_t s, void* act, const float* dact_part, int splits) {
  if (n == 0) return FLEXCO_OK;
  const bool vec = vec_ok(dtype, F, {gate, up, dact, dgu, act, dact_part});
  const int per = 256 * (vec ? (dtype == FLEXCO_BF16 ? 8 : 4) : 1);
  DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((swiglu_bwd_kernel<T, VEC>), dim3((F + per - 1) / per, n), dim3(256), 0,
                                             s, (const T*)gate, (const T*)up, (const T*)dact, (T*)dgu, (T*)act, F, dact_part,
                                             splits, (size_t)n * F));
  return post_launch("swiglu_bwd");
}

int32_t launch_remat(const RematArgs& a, int dtype, hipStream_t s) {
  if (a.n == 0) return FLEXCO_OK;
  // each in the form that its own rows allow: one launch, or two where some are not 16-byte aligned
  for (const bool vec : {true, false}) {
    RematArgs p = a;
    p.norms = 0;
    if (a.act && vec_ok(dtype, a.F, {a.gate, a.up, a.act}) != vec) p.act = nullptr;
    for (int z = 0; z < a.norms; ++z)
      if (vec_ok(dtype, a.H, {a.x[z], a.g[z], a.h[z]}) == vec) {
        p.x[p.norms] = a.x[z];
        p.g[p.norms] = a.g[z];
        p.h[p.norms++] = a.h[z];
      }
    if (!p.act && p.norms == 0) continue;
    const int per = 256 * (vec ? (dtype == FLEXCO_BF16 ? 8 : 4) : 1), act_blocks = p.act ? (p.F + per - 1) / per : 0;
    DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((remat_kernel<T, VEC>), dim3(p.n * (act_blocks + p.norms)), dim3(256), 0, s, p, act_blocks));
  }
  return post_launch("remat");
}

int32_t launch_copy_rows(const void* src, size_t ld_src_bytes, void* dst, size_t ld_dst_bytes, int n_rows,
                         size_t width_bytes, hipStream_t s) {
  if (n_rows == 0 || width_bytes == 0) return FLEXCO_OK;
  if (width_bytes % 4) return fail(FLEXCO_ESHAPE, "row copy of %zu bytes is not a multiple of 4", width_bytes);
  const bool v16 = width_bytes % 16 == 0 && ld_src_bytes % 16 == 0 && ld_dst_bytes % 16 == 0 && aligned16(src) &&
                   aligned16(dst);
  if (v16) {
    const int w = (int)(width_bytes / 16);
    hipLaunchKernelGGL((copy_rows_kernel<uint4>), dim3((w + 255) / 256, n_rows), dim3(256), 0, s, (const char*)src,
                       ld_src_bytes, (char*)dst, ld_dst_bytes, w);
  } else {
    const int w = (int)(width_bytes / 4);
    hipLaunchKernelGGL((copy_rows_kernel<uint32_t>), dim3((w + 255) / 256, n_rows), dim3(256), 0, s, (const char*)src,
                       ld_src_bytes, (char*)dst, ld_dst_bytes, w);
  }
  return post_launch("copy_rows");
}

template <int R>
static int32_t lora_ops(int op, const LoraBatch& b, bool shared_y, int n, int r, float scale, int dtype, const int32_t* row_idx,
                        hipStream_t s, const LoraBatch& back) {
  int wide = 0;
  for (int z = 0; z < b.count; ++z) wide = std::max(wide, (b.p[z].n_long + 255) / 256);
  for (int z = 0; z < back.count; ++z) wide = std::max(wide, (back.p[z].n_long + 255) / 256);
  DISPATCH_T(dtype, {
    if (op == 0)
      hipLaunchKernelGGL((lora_reduce_long_kernel<T, R>), dim3(n, b.count), dim3(256), 0, s, b, r, row_idx);
    else if (op == 1)
      hipLaunchKernelGGL((lora_expand_kernel<T, R>), dim3(wide, (n + 15) / 16, shared_y ? 1 : b.count), dim3(256), 0, s, b, n, r,
                         scale, row_idx);
    else
      hipLaunchKernelGGL((lora_outer_kernel<T, R>), dim3(wide, b.count + (back.count ? (n + 15) / 16 : 0)), dim3(256), 0, s, b, back, n, r,
                         scale);
  });
  return post_launch("lora kernel");
}

// Up to this many rows the two launches' cost is that they are two (4 - 5 us of host and queue each), and the matrices are
// read once per row from L2; beyond, the row blocks of the separate expand kernel read them a sixteenth as often.
constexpr int LORA_ROWS_MAX = 256;
// A row's block walks both products alone, and wide or high-rank ones take longer that way than the launch they save: up
// to this many passes of 256 elements x ranks (rounded up as the kernels do).  Layer forward of 4 / 32 / 128 / 250 rows,
// one launch against two, us: width 256, rank 8 (32) 73 / 105 / 122 / 140 against 85 / 122 / 143 / 158; width 512, ffn 1376,
// rank 8 (64) 88 / 130 / 175 / 194 against 83 / 135 / 185 / 199; the same, rank 64 (512) 302 / 450 / 509 / 677 against
// 211 / 373 / 426 / 446; 8 rows at the 8B shape, rank 8 (576) 643 against 471.
constexpr int LORA_ROWS_WORK = 64;
static int lora_rows_work(int in, int out, int r) {
  return ((in + 255) / 256 + (out + 255) / 256) * (r <= 8 ? 8 : r <= 16 ? 16 : r <= 32 ? 32 : 64);
}
static int32_t lora_rows(const LoraBatch& down, const LoraBatch& up, int n, int r, float scale, int dtype, const int32_t* row_idx,
                         hipStream_t s) {
  const dim3 grid(n, down.count);
#define FLEXCO_LORA_ROWS(R_) \
  DISPATCH_T(dtype, hipLaunchKernelGGL((lora_rows_kernel<T, R_>), grid, dim3(256), 0, s, down, up, r, scale, row_idx))
  if (r <= 8) FLEXCO_LORA_ROWS(8);
  else if (r <= 16) FLEXCO_LORA_ROWS(16);
  else FLEXCO_LORA_ROWS(32);                     // (ranks past 32 have too much work at any width)
#undef FLEXCO_LORA_ROWS
  return post_launch("lora_rows");
}

static int32_t lora_dispatch(int op, const LoraBatch& b, bool shared_y, int n, int r, float scale, int dtype, hipStream_t s,
                             const int32_t* row_idx = nullptr, const LoraBatch* back_in = nullptr) {
  if (n == 0 || b.count == 0) return FLEXCO_OK;
  LoraBatch back = {};
  if (back_in) back = *back_in;
  if (r <= 8) return lora_ops<8>(op, b, shared_y, n, r, scale, dtype, row_idx, s, back);
  if (r <= 16) return lora_ops<16>(op, b, shared_y, n, r, scale, dtype, row_idx, s, back);
  if (r <= 32) return lora_ops<32>(op, b, shared_y, n, r, scale, dtype, row_idx, s, back);
  return lora_ops<64>(op, b, shared_y, n, r, scale, dtype, row_idx, s, back);
}

// u <- relu(u); where u <= 0 the matching element of t (if given) is zeroed: the ReLU's backward mask
__global__ __launch_bounds__(256) void relu_mask_kernel(float* __restrict__ u, float* __restrict__ t, size_t count) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  if (!(u[i] > 0.f)) {
    u[i] = 0.f;
    if (t) t[i] = 0.f;
  }
}

int32_t launch_relu_mask(float* u, float* t, size_t count, hipStream_t s) {
  if (count == 0) return FLEXCO_OK;
  hipLaunchKernelGGL(relu_mask_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, u, t, count);
  return post_launch("relu_mask");
}

// u_z[n, r] = x_z[rows, in] A_z^T,  A_z [r, in]; rows = row_idx[0..n) or 0..n.  Then y_z[rows, out] += scale * u_z B_z^T,
// B_z [out, r], the y_z being different columns.
int32_t launch_lora_apply(const LoraTarget* tg, int count, int n, int r, float scale, int dtype, const int32_t* row_idx, hipStream_t s) {
  LoraBatch down, up;
  down.count = up.count = count;
  for (int z = 0; z < count; ++z) {
    const LoraTarget& t = tg[z];
    down.p[z] = {t.x, t.ldx, t.A, 1, (size_t)t.in, t.u, nullptr, 0, nullptr, 0, 0, t.in};
    up.p[z] = {nullptr, 0, t.B, (size_t)r, 1, t.u, t.y, t.ldy, nullptr, 0, 0, t.out};
  }
  if (n == 0 || count == 0) return FLEXCO_OK;
  int work = 0;      // (the targets' blocks run side by side)
  for (int z = 0; z < count; ++z) work = std::max(work, lora_rows_work(tg[z].in, tg[z].out, r));
  if (n <= LORA_ROWS_MAX && work <= LORA_ROWS_WORK) return lora_rows(down, up, n, r, scale, dtype, row_idx, s);
  const int32_t rc = lora_dispatch(0, down, false, n, r, 0.f, dtype, s, row_idx);
  return rc ? rc : lora_dispatch(1, up, count == 1, n, r, scale, dtype, s, row_idx);
}

int32_t launch_lora_shrink(const void* x, size_t ldx, const void* A, float* u, int n, int in, int r, int dtype,
                           const int32_t* row_idx, hipStream_t s) {
  LoraBatch b;
  b.count = 1;
  b.p[0] = {x, ldx, A, 1, (size_t)in, u, nullptr, 0, nullptr, 0, 0, in};
  return lora_dispatch(0, b, false, n, r, 0.f, dtype, s, row_idx);
}
// y[rows, out] += scale * u B^T,  B [out, r]
int32_t launch_lora_expand(const float* u, const void* B, void* y, size_t ldy, int n, int out, int r, float scale,
                           int dtype, const int32_t* row_idx, hipStream_t s) {
  LoraBatch b;
  b.count = 1;
  b.p[0] = {nullptr, 0, B, (size_t)r, 1, const_cast<float*>(u), y, ldy, nullptr, 0, 0, out};
  return lora_dispatch(1, b, true, n, r, scale, dtype, s, row_idx);
}

// Gradients of the LoRA bypasses of up to three targets on n rows (Sec. 4.1 form y = scale (x A^T) B^T):
//   u = x A^T; t = dy B; dB += scale dy^T u; dA += scale t^T x; dx += scale t A   (one dx, or none, for all of them)
// With relu (a bottleneck adapter: y = relu(x A^T) B^T, one target) u becomes relu(u) and t is zeroed where u <= 0.
int32_t launch_lora_bwd(const LoraTarget* tg, int count, void* dx, size_t lddx, int n, int r, float scale, int dtype, hipStream_t s,
                        bool relu) {
  LoraBatch long_sums, outer, back;
  long_sums.count = outer.count = 2 * count;
  back.count = count;
  for (int z = 0; z < count; ++z) {
    const LoraTarget& t = tg[z];
    long_sums.p[2 * z] = {t.x, t.ldx, t.A, 1, (size_t)t.in, t.u, nullptr, 0, nullptr, 0, 0, t.in};
    long_sums.p[2 * z + 1] = {t.y, t.ldy, t.B, (size_t)r, 1, t.t, nullptr, 0, nullptr, 0, 0, t.out};
    outer.p[2 * z] = {t.y, t.ldy, nullptr, 0, 0, t.u, nullptr, 0, t.dB, (size_t)r, 1, t.out};
    outer.p[2 * z + 1] = {t.x, t.ldx, nullptr, 0, 0, t.t, nullptr, 0, t.dA, 1, (size_t)t.in, t.in};
    back.p[z] = {nullptr, 0, t.A, 1, (size_t)t.in, t.t, dx, lddx, nullptr, 0, 0, t.in};
  }
  int32_t rc;
  // (u, t and dx of a row in one launch, as the forward pass does: no faster at width 256, rank 8, and everywhere else
  // slower, a window of 64 rows at the 8B shape, rank 8, 895 us against 549.  The outer products read dy and x, which may be dx
  // itself - the adapter's in-place call: only where dx is neither do they share a launch with it, 15 -> 6.7 us for the fp32
  // configuration's down projection.)
  if ((rc = lora_dispatch(0, long_sums, false, n, r, 0.f, dtype, s))) return rc;
  if (relu && (rc = launch_relu_mask(tg[0].u, tg[0].t, (size_t)n * r, s))) return rc;
  const bool with_dx = dx && !relu && (n + 15) / 16 < 60000;
  if ((rc = lora_dispatch(2, outer, false, n, r, scale, dtype, s, nullptr, with_dx ? &back : nullptr))) return rc;
  return dx && !with_dx ? lora_dispatch(1, back, true, n, r, scale, dtype, s) : FLEXCO_OK;
}

}  // namespace flexco
