// Type-generic mixed attention (forward partials + merge) and window backward.
//
// These kernels serve the fp32 configuration and any shape the MFMA kernels do not cover.
// They share the work list and the partial-result format with the MFMA path:
//   work item (tile, split) x kv head  ->  for each column c of the tile (token c / group,
//   query head kvh * group + c % group): running max m, sum l and un-normalised
//   accumulator acc[d] over the keys of the split that the column may see.
//   part_ml [n_parts, nkv, cols_per_tile, 2], part_acc [n_parts, nkv, cols_per_tile, d]
// The merge kernel combines the splits of a tile (log-sum-exp weighting).
#include <algorithm>
#include "flexco_internal.h"
#include "device_types.h"

namespace flexco {

__device__ inline float wsum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline float wmax(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

struct AttnArgs {
  const int32_t *tok_pos, *block_table, *tile_req, *tile_tok0, *tile_ntok, *tile_nsplit, *tile_part0, *item_tile,
      *item_split, *item_ntiles;
  int max_pages, nq, nkv, d, ps, split_keys, cols_per_tile, col_blocks;
  float scale;
  // rows of a tile with a single key split go straight to the output, as the merge kernel would write them
  void* out;
  size_t ldo;
  float* lse;         // or NULL
  AttnKeep keep;
};

__device__ inline int lane_int(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ inline float lane_float(float v, int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); }

// One wavefront per column, four of a tile's sixteen per block (sixteen kept other CUs idle while they shared one's issue
// slots: the fp32 configuration's 68-token batch 19 us against 12.6; 40 decode tokens of 500 - 1000 keys 163 against 121).  The kernel is a chain of loads (the fp32 configuration's grids do not
// fill the chip): K rows and V page rows are read 16 bytes at a time with several loads in flight - a lane per key for the
// scores, a lane per channel for the output - and a page id is looked up once per page (one element and one
// lookup at a time: 78 us for the fp32 configuration's 68-token batch).  SHORT: the form for batches whose columns are all of at
// most 64 keys and channels: such a column has its V on the way beside its K, before the softmax, and takes page ids from the lanes
// that looked them up (16.2 -> 12.6 us there); a longer one is still right.  In the kernel of all batches the extra code,
// which such launches wait for, cost the others 8 - 25 %.  The tables are read in as few dependent steps as there are.
constexpr int FWD_NW = 4;
template <typename T, bool SHORT>
__global__ __launch_bounds__(64 * FWD_NW) void attn_fwd_generic_kernel(AttnArgs a, const T* __restrict__ q, size_t ldq,
                                                                   const T* __restrict__ kp, const T* __restrict__ vp,
                                                                   float* __restrict__ part_ml,
                                                                   float* __restrict__ part_acc) {
  extern __shared__ float smem[];   // per wave: q[d] + scores[split_keys]
  constexpr int N = Vec<T>::N;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float* qs = smem + wave * (a.d + a.split_keys);
  float* sc = qs + a.d;
  // col_blocks blocks per tile of the work item that has this split (blockIdx.z = tile within the item, run of columns)
  const int item = blockIdx.x, kvh = blockIdx.y, tile_in = blockIdx.z / a.col_blocks, run = blockIdx.z % a.col_blocks;
  const int ntl = a.item_ntiles[item], tile0 = a.item_tile[item], split = a.item_split[item];
  if (tile_in >= ntl) return;
  const int tile = tile0 + tile_in;
  const int r = a.tile_req[tile], t0 = a.tile_tok0[tile], ntok = a.tile_ntok[tile], nsplit = a.tile_nsplit[tile], part0 = a.tile_part0[tile];
  if (split >= nsplit) return;
  const int group = a.nq / a.nkv;
  const int part = part0 + split;
  const int k0 = split * a.split_keys, pg0 = k0 / a.ps;       // the first key of a page
  const int32_t* bt = a.block_table + (size_t)r * a.max_pages + pg0;
  const int my_pg = lane / a.ps, my_off = lane % a.ps;        // where the lane's key is in a run of 64
  const bool whole = nsplit == 1;                             // the whole key range: normalised rows, straight to the output
  for (int c = run * FWD_NW + wave; c < ntok * group; c += FWD_NW * a.col_blocks) {
    const int t = t0 + c / group, h = kvh * group + c % group;
    const int pos = a.tok_pos[t];
    int first_page = 0;
    if (SHORT) first_page = bt[min(my_pg, a.max_pages - 1 - pg0)];     // (past the last key: not used)
    for (int dd = lane; dd < a.d; dd += 64) qs[dd] = ld(q + (size_t)t * ldq + h * a.d + dd);
    const int nk = max(0, min(k0 + a.split_keys, pos + 1) - k0);
    // a column of one run: V of the lane's first channel, 64 keys
    const bool short_run = SHORT && nk <= 64 && a.ps % N == 0;         // (uniform)
    float v1[SHORT ? 64 / N : 1][N];
    if (short_run) {
#pragma unroll
      for (int u = 0; u < (SHORT ? 64 / N : 0); ++u) {
        const int un = min(u * N, max(nk - 1, 0) / N * N);    // past the last key: the last unit again, not used
        const T* vr = vp + (((size_t)lane_int(first_page, un) * a.nkv + kvh) * (size_t)a.d + min(lane, a.d - 1)) * a.ps + lane_int(my_off, un);
        Vec<T>::load(vr, v1[u]);
      }
    }
    __builtin_amdgcn_wave_barrier();
    float m = -INFINITY;
    for (int jj = lane; jj < nk; jj += 64) {
      const size_t page = SHORT && jj < 64 ? first_page : bt[jj / a.ps];
      const T* kr = kp + ((page * a.nkv + kvh) * a.ps + (SHORT && jj < 64 ? my_off : jj % a.ps)) * (size_t)a.d;   // rows are whole 16-byte units
      float s = 0.f;
#pragma unroll 8
      for (int dd = 0; dd < a.d; dd += N) {
        float kv[N];
        Vec<T>::load(kr + dd, kv);
#pragma unroll
        for (int e = 0; e < N; ++e) s += qs[dd + e] * kv[e];
      }
      s *= a.scale;
      sc[jj] = s;
      m = fmaxf(m, s);
    }
    m = wmax(m);
    float l = 0.f;
    for (int jj = lane; jj < nk; jj += 64) {
      const float p = __expf(sc[jj] - m);
      sc[jj] = p;
      l += p;
    }
    l = wsum(l);
    __builtin_amdgcn_wave_barrier();
    const size_t idx = ((size_t)part * a.nkv + kvh) * a.cols_per_tile + c;
    const bool kept = whole && a.keep.lse2 && t >= a.keep.tok0 && t < a.keep.tok0 + a.keep.n;
    const float inv = 1.0f / l;
    for (int dd = lane; dd < a.d; dd += 64) {
      float acc = 0.f;
      if (short_run && dd < 64) {
#pragma unroll
        for (int u = 0; u < (SHORT ? 64 / N : 0); ++u)
#pragma unroll
          for (int e = 0; e < N; ++e)
            if (u * N + e < nk) acc += sc[u * N + e] * v1[u][e];
      } else {
        for (int j0 = 0; j0 < nk; j0 += a.ps) {
          const T* vr = vp + (((size_t)bt[j0 / a.ps] * a.nkv + kvh) * (size_t)a.d + dd) * a.ps;
          const int n = min(a.ps, nk - j0);
          if (a.ps % N == 0) {               // (a page row is whole 16-byte units; slots past the last key may hold anything)
#pragma unroll 4
            for (int p0 = 0; p0 < n; p0 += N) {
              float v[N];
              Vec<T>::load(vr + p0, v);
#pragma unroll
              for (int e = 0; e < N; ++e)
                if (p0 + e < n) acc += sc[j0 + p0 + e] * v[e];
            }
          } else {
            for (int p = 0; p < n; ++p) acc += sc[j0 + p] * ld(vr + p);
          }
        }
      }
      if (!whole) {
        part_acc[idx * a.d + dd] = acc;
        continue;
      }
      st((T*)a.out + (size_t)t * a.ldo + h * a.d + dd, acc * inv);
      if (kept) st((T*)a.keep.out2 + ((size_t)(t - a.keep.tok0) * a.nq + h) * a.d + dd, acc * inv);
    }
    if (lane == 0) {
      if (!whole) { part_ml[idx * 2] = m; part_ml[idx * 2 + 1] = l; }
      else if (a.lse) a.lse[(size_t)t * a.nq + h] = m + __logf(l);
      if (kept) a.keep.lse2[(size_t)(t - a.keep.tok0) * a.nq + h] = m + __logf(l);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// key splits that share a partial row: fold for a request of one token, else 1
__device__ inline int token_fold(int t, int fold, const int32_t* tok_req, const int32_t* req_tok_off) {
  if (fold == 1) return 1;
  const int r = tok_req[t];
  return req_tok_off[r + 1] - req_tok_off[r] == 1 ? fold : 1;
}

// One wave per (token, query head): combine the tile's splits (every fold-th has a partial row).
template <typename T>
__global__ __launch_bounds__(64) void attn_merge_kernel(const int32_t* __restrict__ tok_tile,
                                                        const int32_t* __restrict__ tile_tok0,
                                                        const int32_t* __restrict__ tile_nsplit,
                                                        const int32_t* __restrict__ tile_part0,
                                                        const float* __restrict__ part_ml,
                                                        const float* __restrict__ part_acc, T* __restrict__ out,
                                                        size_t ldo, float* __restrict__ lse, int nq, int nkv, int d,
                                                        int cols_per_tile, int fold_in, const int32_t* __restrict__ req_tok_off,
                                                        const int32_t* __restrict__ tok_req, AttnKeep keep) {
  const int t = blockIdx.x, h = blockIdx.y;
  const int group = nq / nkv, kvh = h / group;
  const int tile = tok_tile[t];
  const int c = (t - tile_tok0[tile]) * group + h % group;
  const int nsplit = tile_nsplit[tile], part0 = tile_part0[tile];
  const int fold = token_fold(t, fold_in, tok_req, req_tok_off);
  if (nsplit <= fold) return;   // the attention kernel has written these rows itself
  float M = -INFINITY;
  for (int s = 0; s < nsplit; s += fold) {
    const size_t idx = ((size_t)(part0 + s) * nkv + kvh) * cols_per_tile + c;
    M = fmaxf(M, part_ml[idx * 2]);
  }
  float L = 0.f;
  for (int s = 0; s < nsplit; s += fold) {
    const size_t idx = ((size_t)(part0 + s) * nkv + kvh) * cols_per_tile + c;
    const float ms = part_ml[idx * 2];
    if (ms > -INFINITY) L += part_ml[idx * 2 + 1] * __expf(ms - M);
  }
  const float inv = 1.0f / L;
  const bool kept = keep.lse2 && t >= keep.tok0 && t < keep.tok0 + keep.n;
  for (int dd = threadIdx.x; dd < d; dd += 64) {
    float acc = 0.f;
    for (int s = 0; s < nsplit; s += fold) {
      const size_t idx = ((size_t)(part0 + s) * nkv + kvh) * cols_per_tile + c;
      const float ms = part_ml[idx * 2];
      if (ms > -INFINITY) acc += part_acc[idx * d + dd] * __expf(ms - M);
    }
    st(out + (size_t)t * ldo + h * d + dd, acc * inv);
    if (kept) st((T*)keep.out2 + ((size_t)(t - keep.tok0) * nq + h) * d + dd, acc * inv);
  }
  if (threadIdx.x == 0) {
    if (lse) lse[(size_t)t * nq + h] = M + __logf(L);
    if (kept) keep.lse2[(size_t)(t - keep.tok0) * nq + h] = M + __logf(L);
  }
}

__device__ inline void store4(float* p, const float (&v)[4]) { *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]}; }
__device__ inline void store4(bf16_t* p, const float (&v)[4]) {
  bf16x4 t;
#pragma unroll
  for (int j = 0; j < 4; ++j) t[j] = (bf16_t)v[j];
  *reinterpret_cast<bf16x4*>(p) = t;
}

// The same for head_dim 128 with 16-byte accesses: 32 lanes per (token, query head), eight of them per block (the
// one-wavefront form above is a grid of T x nq blocks of which most leave at once - tiles with a single split - and
// the others read four bytes per lane).
template <typename T>
__global__ __launch_bounds__(256) void attn_merge128_kernel(const int32_t* __restrict__ tok_tile,
                                                            const int32_t* __restrict__ tile_tok0,
                                                            const int32_t* __restrict__ tile_nsplit,
                                                            const int32_t* __restrict__ tile_part0,
                                                            const float* __restrict__ part_ml,
                                                            const float* __restrict__ part_acc, T* __restrict__ out,
                                                            size_t ldo, float* __restrict__ lse, int nq, int nkv,
                                                            int cols_per_tile, int fold_in, const int32_t* __restrict__ req_tok_off,
                                                        const int32_t* __restrict__ tok_req, AttnKeep keep) {
  constexpr int d = 128;
  const int t = blockIdx.x, h = blockIdx.y * 8 + (threadIdx.x >> 5), ln = threadIdx.x & 31;
  if (h >= nq) return;
  const int group = nq / nkv, kvh = h / group;
  const int tile = tok_tile[t];
  const int fold = token_fold(t, fold_in, tok_req, req_tok_off);
  const int nsplit = (tile_nsplit[tile] + fold - 1) / fold;     // partial rows
  if (nsplit == 1) return;   // the attention kernel has written these rows itself
  const int c = (t - tile_tok0[tile]) * group + h % group;
  const size_t idx0 = ((size_t)tile_part0[tile] * nkv + kvh) * cols_per_tile + c;
  const size_t step = (size_t)fold * nkv * cols_per_tile;         // from one partial row to the next
  // The chain of loads is what this kernel's time is: U splits' at once (past the last one they repeat it), added in
  // split order.  The first U splits' maxima are kept for the second pass.
  constexpr int U = 8;
  float M = -INFINITY;
  float2 first[U];
#pragma unroll
  for (int u = 0; u < U; ++u) first[u] = *reinterpret_cast<const float2*>(part_ml + (idx0 + min(u, nsplit - 1) * step) * 2);
#pragma unroll
  for (int u = 0; u < U; ++u) M = fmaxf(M, first[u].x);
  for (int s = U; s < nsplit; ++s) M = fmaxf(M, part_ml[(idx0 + s * step) * 2]);
  float L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < nsplit; s += U) {
    float2 ml[U];
    f32x4 a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t idx = idx0 + min(s + u, nsplit - 1) * step;
      ml[u] = s == 0 ? first[u] : *reinterpret_cast<const float2*>(part_ml + idx * 2);
      a[u] = *reinterpret_cast<const f32x4*>(part_acc + idx * d + 4 * ln);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u < nsplit && ml[u].x > -INFINITY) {        // (the sums of a split without a visible key are not written)
        const float w = __expf(ml[u].x - M);
        L += ml[u].y * w;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += a[u][j] * w;
      }
    }
  }
  const float inv = 1.0f / L;
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = acc[j] * inv;
  const bool kept = keep.lse2 && t >= keep.tok0 && t < keep.tok0 + keep.n;
  store4(out + (size_t)t * ldo + h * d + 4 * ln, v);
  if (kept) store4((T*)keep.out2 + ((size_t)(t - keep.tok0) * nq + h) * d + 4 * ln, v);
  if (ln == 0) {
    if (lse) lse[(size_t)t * nq + h] = M + __logf(L);
    if (kept) keep.lse2[(size_t)(t - keep.tok0) * nq + h] = M + __logf(L);
  }
}

// ------------------------------------------------------------------------------------------
// window backward (Sec. 6.1): queries = window rows at positions win_start + i, keys/values
// = cached rows [0, l).  P is recomputed from Q, K and the stored log-sum-exp.
// ------------------------------------------------------------------------------------------
// (delta = rowsum(dO (.) O) of a row is computed here and left for the dK / dV kernel)
//
// Few of the lane groups' guards and LDS lookups of a 64-key run are needed: a lane owns channels lane + 64 u, u < DU = the least of
// 1, 2, 4 that covers head_dim, and a key's (row's) factor and address come from the lane that holds them (lane_float,
// lane_int) instead of from LDS (most of a run's instructions were guards of channels past head_dim), rows of several keys or pairs
// at a time.  fp32 configuration 15.1 -> 10.3 us for dQ, 9.7 -> 6.0 for dK / dV; layer's backward of a window of 256 rows in 2048, bf16 of
// head_dim 256 2610 -> 1990 us, 64 2390 -> 1880, fp32 of head_dim 64 2140 -> 1465.
template <typename T, int DU>
__device__ inline void bwd_dq_row(const size_t i, const int h, const T* __restrict__ q, const T* __restrict__ dout,
                                  const T* __restrict__ out, const float* __restrict__ lse, float* __restrict__ delta,
                                  const T* __restrict__ kp, const T* __restrict__ vp, const int32_t* __restrict__ pages,
                                  T* __restrict__ dq, int win_start, int nq, int nkv, int d, int ps, float scale,
                                  float* smem) {
  constexpr int N = Vec<T>::N;
  float* qs = smem;                 // smem: q[d], do[d]
  float* dos = smem + d;
  const int lane = threadIdx.x;
  const int group = nq / nkv, kvh = h / group;
  const int p = win_start + (int)i;
  const float row_lse = lse[i * nq + h];
  float row_delta = 0.f;
#pragma unroll
  for (int u = 0; u < DU; ++u) {
    const int dd = lane + 64 * u;
    if (dd >= d) break;
    qs[dd] = ld(q + (i * nq + h) * d + dd);
    const float o = ld(dout + (i * nq + h) * d + dd);
    dos[dd] = o;
    row_delta += ld(out + (i * nq + h) * d + dd) * o;
  }
  row_delta = wsum(row_delta);
  if (lane == 0) delta[i * nq + h] = row_delta;
  float acc[DU];
#pragma unroll
  for (int u = 0; u < DU; ++u) acc[u] = 0.f;
  __builtin_amdgcn_wave_barrier();
  for (int kc = 0; kc <= p; kc += 64) {
    const int j = min(kc + lane, p);
    const int my_page = pages[j / ps], my_off = j % ps;
    const size_t page = my_page;
    const T* kr = kp + ((page * nkv + kvh) * ps + my_off) * (size_t)d;
    const T* vr = vp + ((page * nkv + kvh) * (size_t)d) * ps + my_off;
    float s = 0.f, dp = 0.f;
    // eight rows of V on their way per lane (a V element is a load of its own): 32 for bf16 and 16 for fp32 had too few wavefronts
    // on a CU; and where a grid leaves slots empty code that runs once is fetched once, and fetching it is what such a launch waits
    // for (fp32 configuration, 32 rows 13.8 us, 8 rows 11.2 before the keys' rows came in groups)
    constexpr int U = 8 / N;
#pragma unroll U
    for (int dd = 0; dd < d; dd += N) {
      float kv[N], vv[N];
      Vec<T>::load(kr + dd, kv);
#pragma unroll
      for (int e = 0; e < N; ++e, vr += ps) vv[e] = ld(vr);
#pragma unroll
      for (int e = 0; e < N; ++e) {
        s += qs[dd + e] * kv[e];
        dp += dos[dd + e] * vv[e];
      }
    }
    const float pj = __expf(s * scale - row_lse);
    const float ds = kc + lane <= p ? pj * (dp - row_delta) * scale : 0.f;
    // (eight keys' rows on their way; past the last key its row again, times zero.  The lane reads are no loop a compiler unrolls.)
    const int nk = min(64, p + 1 - kc);
    for (int j0 = 0; j0 < nk; j0 += 8) {
#pragma unroll
      for (int jj = j0; jj < j0 + 8; ++jj) {
        const T* kj = kp + (((size_t)lane_int(my_page, jj) * nkv + kvh) * ps + lane_int(my_off, jj)) * (size_t)d;
        const float w = lane_float(ds, jj);
#pragma unroll
        for (int u = 0; u < DU; ++u)
          acc[u] += w * ld(kj + min(lane + 64 * u, d - 1));    // (channels past head_dim: not stored)
      }
    }
  }
#pragma unroll
  for (int u = 0; u < DU; ++u)
    if (lane + 64 * u < d) st(dq + (i * nq + h) * d + lane + 64 * u, acc[u]);
}

// one wave per (key j, kv head): sums over every window row that sees key j and every
// query head of the group; adds into the KV-gradient accumulator rows (Sec. 7).
// VEC: rows of q and dout are read 16 bytes at a time (their alignment is the caller's).  FEW: for launches that leave slots empty
// (more rows at a time per lane).  DELTA: delta computed here from the rows of out.
template <typename T, int DU, bool VEC, bool FEW, bool DELTA>
__device__ inline void bwd_dkv_key(const int j, const int kvh, const T* __restrict__ q, const T* __restrict__ dout,
                                   const T* __restrict__ out, const float* __restrict__ lse, const float* __restrict__ delta,
                                   const T* __restrict__ kp, const T* __restrict__ vp, const int32_t* __restrict__ pages,
                                   float* __restrict__ dk_accum, float* __restrict__ dv_accum, int win_start, int win_len,
                                   int nq, int nkv, int d, int ps, float scale, float* smem) {
  constexpr int N = VEC ? Vec<T>::N : 1;
  float* ks = smem;                 // smem: k[d], v[d]
  float* vs = smem + d;
  const int lane = threadIdx.x;
  const int group = nq / nkv;
  const size_t page = pages[j / ps];
  for (int dd = lane; dd < d; dd += 64) {
    ks[dd] = ld(kp + ((page * nkv + kvh) * ps + j % ps) * (size_t)d + dd);
    vs[dd] = ld(vp + ((page * nkv + kvh) * (size_t)d + dd) * ps + j % ps);
  }
  const int i_first = max(0, j - win_start);          // first window row that sees key j
  const int n_pairs = (win_len - i_first) * group;
  float dk[DU], dv[DU];
#pragma unroll
  for (int u = 0; u < DU; ++u) dk[u] = dv[u] = 0.f;
  __builtin_amdgcn_wave_barrier();
  for (int pc = 0; pc < n_pairs; pc += 64) {
    const int pr = min(pc + lane, n_pairs - 1);
    const int my_i = i_first + pr / group, my_h = kvh * group + pr % group;
    const size_t row = (size_t)my_i * nq + my_h;                // of q and dout
    const T* qr = q + row * d;
    const T* dor = dout + row * d;
    const float row_lse = lse[row];
    float row_delta = DELTA ? 0.f : delta[row];
    float s = 0.f, dp = 0.f;
#pragma unroll VEC ? (FEW ? 8 : 4) : 2
    for (int dd = 0; dd < d; dd += N) {
      float qv[N], ov[N];
      if constexpr (VEC) {
        Vec<T>::load(qr + dd, qv);
        Vec<T>::load(dor + dd, ov);
      } else {
        qv[0] = ld(qr + dd);
        ov[0] = ld(dor + dd);
      }
#pragma unroll
      for (int e = 0; e < N; ++e) {
        s += qv[e] * ks[dd + e];
        dp += ov[e] * vs[dd + e];
      }
      if constexpr (DELTA) {
        float av[N];
        Vec<T>::load(out + row * d + dd, av);
#pragma unroll
        for (int e = 0; e < N; ++e) row_delta += av[e] * ov[e];
      }
    }
    const float pj = pc + lane < n_pairs ? __expf(s * scale - row_lse) : 0.f;
    const float ds = pj * (dp - row_delta) * scale;
    constexpr int G = FEW ? 16 / DU : 4;      // pairs' rows on their way; past the last pair its rows again, times zero
    const int np = min(64, n_pairs - pc);
    for (int p0 = 0; p0 < np; p0 += G) {
#pragma unroll
      for (int pp = p0; pp < p0 + G; ++pp) {
        const size_t at = ((size_t)lane_int(my_i, pp) * nq + lane_int(my_h, pp)) * d;
        const float wp = lane_float(pj, pp), wd = lane_float(ds, pp);
#pragma unroll
        for (int u = 0; u < DU; ++u) {
          const int dd = min(lane + 64 * u, d - 1);
          dv[u] += wp * ld(dout + at + dd);
          dk[u] += wd * ld(q + at + dd);
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < DU; ++u) {
    const int dd = lane + 64 * u;
    if (dd < d) {
      dk_accum[((size_t)j * nkv + kvh) * d + dd] += dk[u];
      dv_accum[((size_t)j * nkv + kvh) * d + dd] += dv[u];
    }
  }
}

// dQ of a (window row, query head) per block, delta left for the kernel below
template <typename T, int DU>
__global__ __launch_bounds__(64) void attn_bwd_dq_generic_kernel(const T* __restrict__ q, const T* __restrict__ dout,
                                                                 const T* __restrict__ out, const float* __restrict__ lse,
                                                                 float* __restrict__ delta, const T* __restrict__ kp,
                                                                 const T* __restrict__ vp, const int32_t* __restrict__ pages,
                                                                 T* __restrict__ dq, int win_start, int nq, int nkv, int d,
                                                                 int ps, float scale) {
  extern __shared__ float smem[];
  bwd_dq_row<T, DU>(blockIdx.x, blockIdx.y, q, dout, out, lse, delta, kp, vp, pages, dq, win_start, nq, nkv, d, ps, scale, smem);
}

template <typename T, int DU, bool VEC, bool FEW>
__global__ __launch_bounds__(64) void attn_bwd_dkv_generic_kernel(const T* __restrict__ q, const T* __restrict__ dout,
                                                                  const float* __restrict__ lse, const float* __restrict__ delta,
                                                                  const T* __restrict__ kp, const T* __restrict__ vp,
                                                                  const int32_t* __restrict__ pages, float* __restrict__ dk_accum,
                                                                  float* __restrict__ dv_accum, int win_start, int win_len, int nq,
                                                                  int nkv, int d, int ps, float scale) {
  extern __shared__ float smem[];
  bwd_dkv_key<T, DU, VEC, FEW, false>(blockIdx.x, blockIdx.y, q, dout, (const T*)nullptr, lse, delta, kp, vp, pages, dk_accum, dv_accum,
                                      win_start, win_len, nq, nkv, d, ps, scale, smem);
}

// Both in one launch, the rows of dQ first (their blocks walk longer): nothing of one is read by the other, as a key's block
// computes delta itself.
template <typename T, int DU>
__global__ __launch_bounds__(64) void attn_bwd_few_generic_kernel(const T* __restrict__ q, const T* __restrict__ dout,
                                                                  const T* __restrict__ out, const float* __restrict__ lse,
                                                                  float* __restrict__ delta, const T* __restrict__ kp,
                                                                  const T* __restrict__ vp, const int32_t* __restrict__ pages,
                                                                  T* __restrict__ dq, float* __restrict__ dk_accum,
                                                                  float* __restrict__ dv_accum, int win_start, int win_len, int nq,
                                                                  int nkv, int d, int ps, float scale) {
  extern __shared__ float smem[];
  const int n_dq = win_len * nq, b = blockIdx.x;
  if (b < n_dq)
    bwd_dq_row<T, DU>(b / nq, b % nq, q, dout, out, lse, delta, kp, vp, pages, dq, win_start, nq, nkv, d, ps, scale, smem);
  else
    bwd_dkv_key<T, DU, true, true, true>((b - n_dq) / nkv, (b - n_dq) % nkv, q, dout, out, lse, delta, kp, vp, pages, dk_accum, dv_accum,
                                         win_start, win_len, nq, nkv, d, ps, scale, smem);
}

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

int32_t launch_attention_generic(const flexco_layer_cfg& c, const flexco_maps& m, const void* q, size_t ldq,
                                 const flexco_kv_pool& pool, float* part_ml, float* part_acc, void* out, size_t ldo, float* lse,
                                 hipStream_t s, const AttnKeep* keep) {
  AttnArgs a;
  a.out = out; a.ldo = ldo; a.lse = lse;
  a.keep = keep ? *keep : AttnKeep{nullptr, nullptr, 0, 0};
  a.tok_pos = m.tok_pos; a.block_table = m.block_table; a.tile_req = m.tile_req; a.tile_tok0 = m.tile_tok0;
  a.tile_ntok = m.tile_ntok; a.tile_nsplit = m.tile_nsplit; a.tile_part0 = m.tile_part0; a.item_tile = m.item_tile;
  a.item_split = m.item_split; a.item_ntiles = m.item_ntiles;
  a.max_pages = m.max_pages; a.nq = c.n_q_heads; a.nkv = c.n_kv_heads; a.d = c.head_dim; a.ps = c.page_size;
  a.split_keys = m.kv_split_pages * c.page_size;
  a.cols_per_tile = m.tile_tokens * (c.n_q_heads / c.n_kv_heads);
  a.scale = 1.0f / sqrtf((float)c.head_dim);
  const size_t shm = 4 * sizeof(float) * (size_t)(a.d + a.split_keys);
  if (shm > 64 * 1024) return fail(FLEXCO_EUNSUPPORTED, "kv_split_pages * page_size = %d keys is too large for the generic attention kernel", a.split_keys);
  // a list of nothing but single tokens has one tile per item and a group of columns per tile (8 of them, 10 - 500 keys, with the blocks
  // of whole items as well 1 - 3 % more)
  const bool singles = m.n_single == m.n_items;
  a.col_blocks = singles ? (c.n_q_heads / c.n_kv_heads + FWD_NW - 1) / FWD_NW : 4;
  const dim3 grid(m.n_items, c.n_kv_heads, (singles ? 1 : FLEXCO_ATTN_ITEM_TILES) * a.col_blocks);
  DISPATCH_T(c.dtype, {
    const bool one_run = m.max_kv_len <= 64 && a.d <= 64;
    const auto kern = one_run ? attn_fwd_generic_kernel<T, true> : attn_fwd_generic_kernel<T, false>;
    hipLaunchKernelGGL(kern, grid, dim3(64 * FWD_NW), shm, s, a, (const T*)q, ldq, (const T*)pool.k_pages, (const T*)pool.v_pages, part_ml,
                       part_acc);
  });
  return post_launch("attn_fwd_generic");
}

int32_t launch_attention_merge(const flexco_layer_cfg& c, const flexco_maps& m, const float* part_ml,
                               const float* part_acc, void* out, size_t ldo, float* lse, hipStream_t s,
                               int fold, const AttnKeep* keep_in) {
  AttnKeep keep{nullptr, nullptr, 0, 0};
  if (keep_in) keep = *keep_in;
  const int cpt = m.tile_tokens * (c.n_q_heads / c.n_kv_heads);
  if (c.head_dim == 128 && ((uintptr_t)part_acc & 15) == 0 && ldo % 4 == 0 && ((uintptr_t)out & 15) == 0 &&
      ((uintptr_t)keep.out2 & 15) == 0) {
    DISPATCH_T(c.dtype, hipLaunchKernelGGL((attn_merge128_kernel<T>), dim3(m.T, (c.n_q_heads + 7) / 8), dim3(256), 0, s,
                                           m.tok_tile, m.tile_tok0, m.tile_nsplit, m.tile_part0, part_ml, part_acc, (T*)out,
                                           ldo, lse, c.n_q_heads, c.n_kv_heads, cpt, fold, m.req_tok_off, m.tok_req, keep));
    return post_launch("attn_merge");
  }
  DISPATCH_T(c.dtype, hipLaunchKernelGGL((attn_merge_kernel<T>), dim3(m.T, c.n_q_heads), dim3(64), 0, s, m.tok_tile,
                                         m.tile_tok0, m.tile_nsplit, m.tile_part0, part_ml, part_acc, (T*)out, ldo,
                                         lse, c.n_q_heads, c.n_kv_heads, c.head_dim, cpt, fold, m.req_tok_off, m.tok_req, keep));
  return post_launch("attn_merge");
}

int32_t launch_attention_bwd_generic(const flexco_layer_cfg& c, const flexco_kv_pool& pool, const int32_t* seq_pages,
                                     int win_start, int win_len, const void* q, const void* out, const float* lse, float* delta,
                                     const void* dout, void* dq, float* dk_accum, float* dv_accum, hipStream_t s) {
  const float scale = 1.0f / sqrtf((float)c.head_dim);
  const int l = win_start + win_len;
  const size_t shm = sizeof(float) * 2 * (size_t)c.head_dim;
  const bool vec = aligned16(q) && aligned16(dout);      // (head_dim rows are whole 16-byte units)
#define FLEXCO_BWD_GENERIC(DU_, VEC_, FEW_)                                                                            \
  DISPATCH_T(c.dtype, {                                                                                               \
    hipLaunchKernelGGL((attn_bwd_dq_generic_kernel<T, DU_>), dim3(win_len, c.n_q_heads), dim3(64), shm, s, (const T*)q, (const T*)dout, \
                       (const T*)out, lse, delta, (const T*)pool.k_pages, (const T*)pool.v_pages, seq_pages, (T*)dq, win_start,         \
                       c.n_q_heads, c.n_kv_heads, c.head_dim, c.page_size, scale);                                    \
    hipLaunchKernelGGL((attn_bwd_dkv_generic_kernel<T, DU_, VEC_, FEW_>), dim3(l, c.n_kv_heads), dim3(64), shm, s, (const T*)q, (const T*)dout, \
                       lse, delta, (const T*)pool.k_pages, (const T*)pool.v_pages, seq_pages, dk_accum, dv_accum, win_start, win_len,   \
                       c.n_q_heads, c.n_kv_heads, c.head_dim, c.page_size, scale);                                    \
  })
#define FLEXCO_BWD_FEW(DU_)                                                                                            \
  DISPATCH_T(c.dtype, hipLaunchKernelGGL((attn_bwd_few_generic_kernel<T, DU_>), dim3(win_len * c.n_q_heads + l * c.n_kv_heads), dim3(64), \
                                         shm, s, (const T*)q, (const T*)dout, (const T*)out, lse, delta, (const T*)pool.k_pages, \
                                         (const T*)pool.v_pages, seq_pages, (T*)dq, dk_accum, dv_accum, win_start, win_len, \
                                         c.n_q_heads, c.n_kv_heads, c.head_dim, c.page_size, scale))
#define FLEXCO_BWD_D(MACRO_, ...)                            \
  if (c.head_dim <= 64) MACRO_(1, ##__VA_ARGS__);            \
  else if (c.head_dim <= 128) MACRO_(2, ##__VA_ARGS__);      \
  else MACRO_(4, ##__VA_ARGS__);
  // Keys' blocks of at most one wavefront per SIMD: both halves in one launch, side by side, more rows at a time per lane (two launches,
  // the second with as many rows at a time / one; fp32, windows [start, +rows): 4 heads of 64, [0, +8) 9.1 / 4.6 us, [32, +32)
  // 14.2 / 8.9, [0, +256) 65 / 41, [216, +40) 35 / 30; 16 heads over 2 of 64, [0, +512) 573 / 515; bf16 67 / 35 and 693 / 513).  As every
  // key's block reads out as well, only while an operand's rows fit an XCD's L2 (16 heads over 2 of 256, [0, +512), bf16 of 4 MB
  // 1888 / 1630, fp32 of 8 MB 1981 / 2143), and in fp32 only while the key blocks that see the whole window are few or the rows
  // short: it is the third operand that bounds them then.  Rows in MB x those blocks, measured over 202 windows (two launches / one):
  // up to 571 0.48 - 1.02 of the time, 720 to 960 (64 heads over 2 of 64, [448, +64)) 324 / 357, 1024 (32 over 1 of 64, [512, +256))
  // 1059 / 1264, 2048 (16 over 1 of 256) 1700 / 2285; bf16 0.44 - 0.96 at any.
  // Two launches also where dQ is written over the rows of out (a row's block reads its own before).  Their second is then the form
  // with more rows at a time all the same (fp32, one row at a time / more: 32 heads over 1 of 64, [0, +1024) 5088 / 4092 us, 16 over 2 of
  // 64, [100, +156), dQ over out 183 / 161; head_dim 256 and bf16 level).
  const size_t row_bytes = esize(c.dtype) * (size_t)win_len * c.n_q_heads * c.head_dim;
  const char *o0 = (const char*)out, *q0 = (const char*)dq;
  const bool over_out = q0 < o0 + row_bytes && o0 < q0 + row_bytes;
  const bool few = (long)l * c.n_kv_heads <= 1024;
  const bool third_ok = row_bytes <= (4u << 20) && (c.dtype == FLEXCO_BF16 || row_bytes * win_start * c.n_kv_heads <= (640u << 20));
  if (vec && few && aligned16(out) && !over_out && third_ok) { FLEXCO_BWD_D(FLEXCO_BWD_FEW) }
  else if (vec && few) { FLEXCO_BWD_D(FLEXCO_BWD_GENERIC, true, true) }
  else if (vec) { FLEXCO_BWD_D(FLEXCO_BWD_GENERIC, true, false) }
  else { FLEXCO_BWD_D(FLEXCO_BWD_GENERIC, false, false) }
#undef FLEXCO_BWD_D
#undef FLEXCO_BWD_FEW
#undef FLEXCO_BWD_GENERIC
  return post_launch("attn_bwd_generic");
}

}  // namespace flexco
