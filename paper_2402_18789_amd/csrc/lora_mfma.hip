// bf16 LoRA kernels around the projection GEMMs.
//
// The bypass network of Sec. 4.1, y = f_B(x) + scale (x A^T) B^T with rank r << in, out, is
// split so that the large dimension is touched once:
//   shrink   u = x A^T  (or t = dy B)   skinny product [n, K] x [K, r] on the matrix cores:
//            one wavefront multiplies 16 rows by up to 64 ranks with v_mfma_f32_16x16x32_bf16,
//            both operands fetched in rows of 256 bytes and turned in LDS,
//            K is cut across the 8 wavefronts of a block, whose partial sums are added
//            in wavefront order through LDS, so results do not depend on scheduling; the block
//            writes the fp32 result and/or the scaled bf16 operand of the GEMM extension.
//   expand   is not a kernel: the projection GEMM appends the rank-r product as extra
//            k-steps (gemm_mfma.hip), reading the bf16 matrix the shrink kernel writes.
//   outer    dB += scale dy^T u,  dA += scale t^T x : every output element is a sum over
//            the window's rows only; on the matrix cores (u, t as bf16, the rows of x / dy through
//            transposing LDS reads), 128 output columns per block, rows shared out over 4
//            wavefronts, fixed-order LDS reduction; a plain FMA kernel covers unaligned shapes.
#include <algorithm>
#include <cstring>
#include "flexco_internal.h"
#include "device_types.h"

namespace flexco {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
#define FLEXCO_GP(p) ((const __attribute__((address_space(1))) void*)(p))
#define FLEXCO_LP(p) ((__attribute__((address_space(3))) void*)(p))
#define FLEXCO_LDS __attribute__((address_space(3)))
__device__ inline bf16x8 tr_pair(const bf16_t* a, const bf16_t* b) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)a);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)b);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// One block per RB rows and matrix; K is cut, in whole groups of 128 columns, across the block's wavefronts (and over gridDim.z
// blocks), whose partial sums are added in wavefront order through LDS.
//
// What bounds it: one block's round trip and, for long contractions, the rate at which a CU takes its operands in.  The matrix
// instruction wants 16 different rows in 16 neighbouring lanes; loads in that order keep the address unit busy for 62
// cycles per KB.  So a load takes four rows of 256 bytes, 16 lanes side by side (16 cycles per KB), and the operands are turned
// in 4 KB of LDS per wavefront, piece c of row r at c ^ r (no bank met twice by the 16 lanes that read or write together).
// Loads of U groups are in flight together; a wavefront waits for no other before the sums.
// RB = 8 (half of an operand's rows are then read past, their results dropped) where that still leaves a block its own CU: fewer rows
// behind each other.  Wavefronts: 8; two blocks fit a CU up to rank 32.
// Measured, us, operands in fragment order -> turned (same products): 1024 x 4096, three products of rank 16 11.0 -> 6.3, one
// 10.6 -> 5.6; 2048 x 5120, three 21.0 -> 10.6; 48 x 5120, twelve 12.8 -> 6.5; 1405 x 5120, three of rank 32 31.0 -> 12.9; 1024 x
// 14336 in one launch 27.6 -> 10.9 (in eight ranges 9.9 -> 7.8, each with a launch of 5 us that adds them).
// KM: S lies [K][r] (a B_t as it is, r a multiple of 16): a load takes 32 of its rows, 16 ranks each, and the operand comes from
// transposing LDS reads, four k of 16 ranks each.  (Before, a launch of 6 us turned the B_t of a backward window first.)
template <int RT, int RB, bool KM>   // rank tiles of 16, rows of a block (8 or 16), the low-rank operand's layout
__global__ __launch_bounds__(512) void lora_shrink_kernel(LoraShrinkArgs a) {
  constexpr int U = RT == 1 ? 2 : 1, NW = 8, XP = RB / 4;
  __shared__ __attribute__((aligned(16))) bf16_t turn[NW][16 * 128];
  __shared__ __attribute__((aligned(16))) float red[NW][RT][64][4];
  const int z = blockIdx.y, row0 = blockIdx.x * RB;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 15, g = lane >> 4;
  const int row = row0 + m;
  const int want = a.want[z];
  const bool in_block = m < RB && row < a.rows;
  const int row_ad = (in_block && a.row_adapter) ? a.row_adapter[row] : 0;
  // bit m: row m takes part.  Every wavefront looks at the same rows, so this is the same for the whole block
  const unsigned rows_ok = (unsigned)__ballot(in_block && row_ad >= 0 && (want < 0 || row_ad == want)) & 0xffffu;
  if (!rows_ok) {   // a tile without adapter rows: only its zero rows of the GEMM operand are due
    if (a.out_ext[z] && blockIdx.z == 0)
      for (int idx = threadIdx.x; idx < RB * a.r; idx += 64 * NW)
        if (row0 + idx / a.r < a.rows) a.out_ext[z][(size_t)row0 * a.r + idx] = (bf16_t)0.f;
    return;
  }
  const int slices = NW * gridDim.z, slice = blockIdx.z * NW + wave, groups = a.K[z] / 128;
  int k = (int)((long)groups * slice / slices) * 128;
  const int k1 = (int)((long)groups * (slice + 1) / slices) * 128;
  const int lr = lane >> 4, lc = lane & 15;       // load p of a group: 16-byte piece lc of row 4 p + lr
  const bf16_t* xp[XP];
  const bf16_t* sp[RT][4];
#pragma unroll
  for (int p = 0; p < XP; ++p) {                  // rows that take no part read row 0; their results are dropped
    const int mm = 4 * p + lr;
    xp[p] = a.X[z] + (rows_ok >> mm & 1 ? (size_t)(row0 + mm) : 0) * a.ldx[z] + lc * 8;
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int j = rt * 16 + 4 * p + lr;
      if (KM) sp[rt][p] = a.S[z] + (size_t)(32 * p + (lane >> 1)) * a.r + rt * 16 + (lane & 1) * 8;
      else sp[rt][p] = a.S[z] + (size_t)(j < a.r ? j : 0) * a.lds[z] + lc * 8;
    }
  const size_t s_step = KM ? a.r : 1;             // elements of S per step of k
  f32x4 acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
  bf16_t* const buf = turn[wave];
  if (RB < 16) {                                  // rows that no load fills
#pragma unroll
    for (int p = XP; p < 4; ++p) *reinterpret_cast<bf16x8*>(buf + (4 * p + lr) * 128 + lc * 8) = zero;
  }
  // (LDS instructions of a wavefront run in order; the fences keep the compiler from moving them past each other)
#define FLEXCO_TURN(v_, n_, f_)                                                                       \
  {                                                                                                   \
    asm volatile("" ::: "memory");                                                                    \
    _Pragma("unroll") for (int p = 0; p < n_; ++p)                                                    \
      *reinterpret_cast<bf16x8*>(buf + (4 * p + lr) * 128 + ((lc ^ (4 * p + lr)) & 15) * 8) = v_[p];  \
    asm volatile("" ::: "memory");                                                                    \
    _Pragma("unroll") for (int s = 0; s < 4; ++s)                                                     \
      f_[s] = *reinterpret_cast<const bf16x8*>(buf + m * 128 + (((4 * s + g) ^ m) & 15) * 8);         \
  }
#define FLEXCO_TURN_KM(v_, f_)                                                                        \
  {                                                                                                   \
    asm volatile("" ::: "memory");                                                                    \
    _Pragma("unroll") for (int p = 0; p < 4; ++p) *reinterpret_cast<bf16x8*>(buf + p * 512 + lane * 8) = v_[p]; \
    asm volatile("" ::: "memory");                                                                    \
    _Pragma("unroll") for (int s = 0; s < 4; ++s) {                                                   \
      const bf16_t* t_ = buf + (32 * s + 8 * g + (m >> 2)) * 16 + 4 * (m & 3);                        \
      f_[s] = tr_pair(t_, t_ + 4 * 16);                                                               \
    }                                                                                                 \
  }
#define FLEXCO_SHRINK_GROUPS(U_)                                                                      \
  {                                                                                                   \
    bf16x8 x_[U_][XP], s_[U_][RT][4];                                                                 \
    _Pragma("unroll") for (int u = 0; u < U_; ++u) {                                                  \
      _Pragma("unroll") for (int p = 0; p < XP; ++p)                                                  \
        x_[u][p] = *reinterpret_cast<const bf16x8*>(xp[p] + k + 128 * u);                             \
      _Pragma("unroll") for (int rt = 0; rt < RT; ++rt)                                               \
        _Pragma("unroll") for (int p = 0; p < 4; ++p)                                                 \
          s_[u][rt][p] = *reinterpret_cast<const bf16x8*>(sp[rt][p] + (k + 128 * u) * s_step);          \
    }                                                                                                 \
    _Pragma("unroll") for (int u = 0; u < U_; ++u) {                                                  \
      bf16x8 fx_[4], fs_[4];                                                                          \
      FLEXCO_TURN(x_[u], XP, fx_)                                                                     \
      _Pragma("unroll") for (int rt = 0; rt < RT; ++rt) {                                             \
        if (KM) FLEXCO_TURN_KM(s_[u][rt], fs_) else FLEXCO_TURN(s_[u][rt], 4, fs_)                    \
        _Pragma("unroll") for (int s = 0; s < 4; ++s)                                                 \
          acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx_[s], KM || rt * 16 + m < a.r ? fs_[s] : zero, acc[rt], 0, 0, 0); \
      }                                                                                               \
    }                                                                                                 \
    k += 128 * U_;                                                                                    \
  }
  if (U > 1)
    while (k + 128 * U <= k1) FLEXCO_SHRINK_GROUPS(U)
  while (k < k1) FLEXCO_SHRINK_GROUPS(1)
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) *reinterpret_cast<f32x4*>(red[wave][rt][lane]) = acc[rt];
  __syncthreads();
  // D[row = 4 (lane / 16) + e][rank = lane % 16]: one thread per (lane, e) pair of a rank tile
  if (threadIdx.x >= 16 * RB) return;
  const int ln = threadIdx.x >> 2, e = threadIdx.x & 3;
  const int mm = 4 * (ln >> 4) + e, orow = row0 + mm;
  if (orow >= a.rows) return;
  const bool out_ok = rows_ok >> mm & 1;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int rank = rt * 16 + (ln & 15);
    if (rank >= a.r) continue;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += red[w][rt][ln][e];
    const size_t o = (size_t)orow * a.r + rank;
    if (a.ksplit > 1) {   // partial product of this block's k range; the finalize kernel adds them up
      a.part[((size_t)(z * a.ksplit + blockIdx.z) * a.rows) * a.r + o] = v;
      continue;
    }
    if (a.relu >> z & 1) v = fmaxf(v, 0.f);
    if (a.out_f32[z] && out_ok && orow >= a.f32_lo && orow < a.f32_hi)
      a.out_f32[z][(size_t)(orow - a.f32_lo) * a.r + rank] = v;
    if (a.out_ext[z]) a.out_ext[z][o] = (bf16_t)(out_ok ? v * a.scale : 0.f);
  }
}

// Second step of a shrink whose contraction was cut over several blocks: out = sum of the partial
// products in block order, written like the one-step kernel writes it.
__global__ __launch_bounds__(256) void lora_shrink_finalize_kernel(LoraShrinkArgs a) {
  const int z = blockIdx.y;
  const size_t o = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (o >= (size_t)a.rows * a.r) return;
  const int orow = (int)(o / a.r), rank = (int)(o % a.r);
  const int o_ad = a.row_adapter ? a.row_adapter[orow] : 0;
  const bool out_ok = o_ad >= 0 && (a.want[z] < 0 || o_ad == a.want[z]);
  float v = 0.f;
  if (out_ok)   // (a tile without any adapter row wrote no partial products)
    for (int ks = 0; ks < a.ksplit; ++ks) v += a.part[((size_t)(z * a.ksplit + ks) * a.rows) * a.r + o];
  if (a.relu >> z & 1) v = fmaxf(v, 0.f);
  if (a.out_f32[z] && out_ok && orow >= a.f32_lo && orow < a.f32_hi)
    a.out_f32[z][(size_t)(orow - a.f32_lo) * a.r + rank] = v;
  if (a.out_ext[z]) a.out_ext[z][o] = (bf16_t)(out_ok ? v * a.scale : 0.f);
}

__global__ __launch_bounds__(256) void relu_bwd_mask_kernel(const float* __restrict__ u, float* __restrict__ t,
                                                            bf16_t* __restrict__ t_ext, size_t count) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const float v = u[i] > 0.f ? t[i] : 0.f;
  t[i] = v;
  if (t_ext) t_ext[i] = (bf16_t)v;
}

// G(i, j) += scale * sum_m X[m, i] U[m, j],  G element (i, j) at G[i * g_i + j * g_j]
// Rows are taken in chunks of 256: the chunk's U rows are staged in LDS (broadcast reads), each
// wavefront owns 64 rows of the chunk and issues their 64 loads of X together (a 256-row window is one
// chunk: one wait for U, one for X).
template <int R>
__global__ __launch_bounds__(256) void lora_outer_mfma_path_kernel(LoraOuterArgs a) {
  const int e = blockIdx.y;
  const int n = a.n, r = a.r, n_long = a.n_long[e];
  if ((int)blockIdx.x * 64 >= n_long) return;   // entries of one launch differ in width
  const bf16_t* __restrict__ X = a.X[e];
  const float* __restrict__ U = a.U[e];
  float* __restrict__ G = a.G[e];
  const size_t ldx = a.ldx[e], g_i = a.g_i[e], g_j = a.g_j[e];
  const float scale = a.scale;
  extern __shared__ float smem[];   // us[256][R], later reused as red[3][64][R]
  constexpr int CH = 256, RB = 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const int ic = i < n_long ? i : n_long - 1;
  float acc[R];
#pragma unroll
  for (int j = 0; j < R; ++j) acc[j] = 0.f;
  for (int mb = 0; mb < n; mb += CH) {
    __syncthreads();
    for (int idx = threadIdx.x; idx < CH * R; idx += 256) {
      const int mm = idx / R, j = idx % R;
      smem[idx] = (mb + mm < n && j < r) ? U[(size_t)(mb + mm) * r + j] : 0.f;
    }
    __syncthreads();
    float xv[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int m = mb + wave * RB + q;
      xv[q] = (float)X[(size_t)(m < n ? m : n - 1) * ldx + ic];   // rows past n meet zero U rows
    }
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const float* u = smem + (wave * RB + q) * R;
#pragma unroll
      for (int j = 0; j < R; ++j) acc[j] += xv[q] * u[j];
    }
  }
  __syncthreads();
  if (wave > 0) {
#pragma unroll
    for (int j = 0; j < R; ++j) smem[((wave - 1) * 64 + lane) * R + j] = acc[j];
  }
  __syncthreads();
  if (wave == 0 && i < n_long) {
    // all loads of the accumulated gradient first, then the stores (one round trip, not R in a row)
    float gv[R];
#pragma unroll
    for (int j = 0; j < R; ++j) gv[j] = j < r ? G[(size_t)i * g_i + (size_t)j * g_j] : 0.f;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j < r) {
        const float v = acc[j] + smem[(0 * 64 + lane) * R + j] + smem[(1 * 64 + lane) * R + j] + smem[(2 * 64 + lane) * R + j];
        G[(size_t)i * g_i + (size_t)j * g_j] = gv[j] + scale * v;
      }
    }
  }
}

// The same products on the matrix cores: G^T[j, i] += scale sum_m U[m, j] X[m, i] with
// v_mfma_f32_16x16x32_bf16, D rows = 16 ranks, D columns = 16 of the block's 128 columns i, k = 32 rows m.
// Eight wavefronts: four for each half of the columns.
//   * U^T (bf16) is staged in LDS once per 256-row chunk, 16-byte pieces XOR-swizzled with the rank; a lane reads its 8
//     consecutive m of one rank with one ds_read_b128.
//   * X: wavefront w owns rows 64 (w % 4) .. + 64 of the chunk and the columns of its half, two [32 rows][64 columns] tiles that go from
//     global memory straight into its own LDS buffers; the operand (8 consecutive rows of one column)
//     comes from two transposing reads (ds_read_b64_tr_b16).  32-byte column pairs are XOR-swizzled
//     with row % 4 so that the four rows of a read sit on different banks.
//   * a half's four sums are added in wavefront order through LDS, a quarter of its columns by each wavefront.
// What bounds it: the rows' way in, tile after tile (single buffers; two blocks share a CU up to rank 32), and U, which every block
// reads whole: hence columns by the 128 (with blocks of 64 columns and four wavefronts, whose sums one wavefront added and wrote, us
// with nothing cached: a 14B window of 1024 rows, 14 products of rank 16 72 -> 65, of 300 rows 36 -> 29; 32B, rank 32, 1024 rows
// 139 -> 109, 300 rows 78 -> 48; 8B, 10 products, 256 rows 18.6 -> 16.1; 257 rows x 1000 - 1864, rank 48, 44 -> 18).  Same sums.
template <int RT>   // rank tiles of 16
__global__ __launch_bounds__(512) void lora_outer_mfma_kernel(LoraOuterArgs a) {
  // element (rank, row) of U^T
  auto ut_at = [](int j, int m) { return j * 256 + (((m >> 3) ^ (j & 15)) << 3) + (m & 7); };
  __shared__ __attribute__((aligned(1024))) bf16_t xt[8][2][32 * 64];       // per wavefront: two X tiles; at the end the sums
  __shared__ __attribute__((aligned(16))) bf16_t ut[RT * 16 * 256];         // U^T of the chunk, [rank][row]
  const int e = blockIdx.y;
  const int n = a.n, r = a.r, n_long = a.n_long[e];
  if ((int)blockIdx.x * 128 >= n_long) return;   // entries of one launch differ in width
  const bf16_t* __restrict__ X = a.X[e];
  const float* __restrict__ U = a.U[e];
  float* __restrict__ G = a.G[e];
  const size_t ldx = a.ldx[e], g_i = a.g_i[e], g_j = a.g_j[e];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rows_of = wave & 3;                   // quarter of a chunk's rows
  const int i0 = blockIdx.x * 128 + 64 * (wave >> 2);
  const int c = lane & 15, g = lane >> 4;

  f32x4 acc[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) acc[rt][cg] = f32x4{0.f, 0.f, 0.f, 0.f};

  // tile loads: instruction q fills rows 8 q .. + 8 of a tile; lane -> row 8 q + lane / 8, physical chunk
  // lane % 8; it fetches the logical chunk that belongs there (pair = physical pair ^ row % 4)
  const int d_row = lane >> 3, d_pc = lane & 7;
  const int d_lch = ((((d_pc >> 1) ^ (d_row & 3)) << 1) | (d_pc & 1));
  const int d_col = min(i0 + d_lch * 8, n_long - 8);
  // transposing reads: source lane c of group g -> row 8 g + c / 4 (+ 4), columns 16 cg + 4 (c % 4) ..
  const int t_row = 8 * g + (c >> 2);
  const int t_k = (c >> 2) & 3;

  // a wavefront's two tiles of the chunk that starts at row mb0 (its own LDS buffers: nobody else reads them)
  auto load_tiles = [&](int mb0) {
    const int mw0 = mb0 + 64 * rows_of;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = min(mw0 + 32 * st + 8 * q + d_row, n - 1);   // rows past n meet zero U
        __builtin_amdgcn_global_load_lds(FLEXCO_GP(X + (size_t)row * ldx + d_col), FLEXCO_LP(&xt[wave][st][q * 512]), 16, 0, 0);
      }
  };
  load_tiles(0);
  // what the sums are added to (nobody else writes it)
  float gv[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = min(i0 + 16 * rows_of + c, n_long - 1), j = min(rt * 16 + 4 * g + q, r - 1);
      gv[rt][q] = G[(size_t)col * g_i + (size_t)j * g_j];
    }
  for (int mb = 0; mb < n; mb += 256) {
    __syncthreads();   // the previous chunk's reads of ut are done
    if (r == RT * 16) {
      // full rank tiles: the chunk of U is one contiguous run of floats; 2 RT 16-byte loads per thread,
      // all in flight before the first is converted
      f32x4 uv[2 * RT];
#pragma unroll
      for (int k = 0; k < 2 * RT; ++k) {
        const int idx4 = tid + 512 * k, m = idx4 / (4 * RT);
        uv[k] = mb + m < n ? *reinterpret_cast<const f32x4*>(U + ((size_t)mb * r + (size_t)idx4 * 4)) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int k = 0; k < 2 * RT; ++k) {
        const int idx4 = tid + 512 * k, m = idx4 / (4 * RT), j = 4 * (idx4 % (4 * RT));
#pragma unroll
        for (int q = 0; q < 4; ++q) ut[ut_at(j + q, m)] = (bf16_t)uv[k][q];
      }
    } else {
      for (int idx = tid; idx < 256 * RT * 16; idx += 512) {
        const int m = idx / (RT * 16), j = idx % (RT * 16);
        ut[ut_at(j, m)] = (bf16_t)((mb + m < n && j < r) ? U[(size_t)(mb + m) * r + j] : 0.f);
      }
    }
    const int mw = mb + 64 * rows_of;
    __syncthreads();   // ut is complete; the barrier's wait also covers this wavefront's tile loads
    if (mw < n) {
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        bf16x8 af[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          af[rt] = *reinterpret_cast<const bf16x8*>(&ut[ut_at(rt * 16 + c, 64 * rows_of + 32 * st + 8 * g)]);
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) {
          const bf16_t* p = &xt[wave][st][t_row * 64 + ((cg ^ t_k) << 4) + 4 * (c & 3)];
          const bf16x8 xf = tr_pair(p, p + 4 * 64);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) acc[rt][cg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[rt], xf, acc[rt][cg], 0, 0, 0);
        }
      }
    }
    // the next chunk's tiles travel while the other wavefronts finish and U is staged: this wavefront's reads
    // of its buffers have returned (the products above consumed them)
    if (mb + 256 < n) {
      asm volatile("" ::: "memory");
      load_tiles(mb + 256);
    }
  }
  // lane (column c of group cg, g) holds ranks 16 rt + 4 g .. + 4; this wavefront adds up group rows_of of its half
  const int i = i0 + 16 * rows_of + c;
  float* const red = reinterpret_cast<float*>(&xt[0][0][0]);      // [wave][cg][lane][4]
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    __syncthreads();                                 // every wavefront's reads of the tiles (of the sums before) are done
#pragma unroll
    for (int cg = 0; cg < 4; ++cg) *reinterpret_cast<f32x4*>(red + ((wave * 4 + cg) * 64 + lane) * 4) = acc[rt][cg];
    __syncthreads();
    f32x4 v = *reinterpret_cast<const f32x4*>(red + (((wave & 4) * 4 + rows_of) * 64 + lane) * 4);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const f32x4 o = *reinterpret_cast<const f32x4*>(red + ((((wave & 4) + w) * 4 + rows_of) * 64 + lane) * 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += o[q];
    }
    if (i < n_long)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = rt * 16 + 4 * g + q;
        if (j < r) G[(size_t)i * g_i + (size_t)j * g_j] = gv[rt][q] + a.scale * v[q];
      }
  }
}

int32_t post(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of %s failed: %s", what, hipGetErrorString(e));
  return FLEXCO_OK;
}

}  // namespace

int32_t launch_lora_shrink_mfma(const LoraShrinkArgs& a_in, int n_mats, hipStream_t s) {
  LoraShrinkArgs a = a_in;
  if (a.rows == 0 || n_mats == 0) return FLEXCO_OK;
  for (int z = 0; z < n_mats; ++z)
    if (a.K[z] % 128 != 0) return fail(FLEXCO_ESHAPE, "LoRA shrink: K = %d is not a multiple of 128", a.K[z]);
  if (a.s_kmajor && a.r % 16 != 0) return fail(FLEXCO_ESHAPE, "LoRA shrink: rank %d is not a multiple of 16", a.r);
  // Long contractions of one width, with scratch at hand, are cut over several blocks per row tile where the low-rank operand is
  // over half a MB (rank tiles x K > 16384; a block takes in 64 bytes a cycle): 256 KB to a block, in whole groups of 128 columns.  The
  // launch that adds the partial products costs 5 us.  (48 x 13824, four products of rank 16 10.3 in one launch, 7.2 + 4.7 in two
  // ranges; 205 x 27648, two of rank 32 27.2 against 16.3 + 5.4.)
  int kmin = a.K[0], kmax = a.K[0];
  for (int z = 1; z < n_mats; ++z) { kmin = a.K[z] < kmin ? a.K[z] : kmin; kmax = a.K[z] > kmax ? a.K[z] : kmax; }
  const int rt = (a.r + 15) / 16;
  a.ksplit = 1;
  if (a.part && n_mats <= a.part_slots && kmin == kmax && (long)rt * kmax > 16384)
    a.ksplit = (int)std::min<long>(LORA_SHRINK_SPLITS, ((long)rt * kmax + 8191) / 8192);
  // blocks of 8 rows while those that have work are no more than the CUs (1024 x 4096, rank 16, one product 5.6 against 6.0 us; three
  // products 8.1 against 6.3)
  const long on = a.rows_on ? a.rows_on : a.rows;
  const int rb = (on + 7) / 8 * n_mats * a.ksplit <= 256 ? 8 : 16;
  const dim3 grid((a.rows + rb - 1) / rb, n_mats, a.ksplit), block(512);
#define FLEXCO_SHRINK(RT_)                                                                            \
  {                                                                                                   \
    if (a.s_kmajor) {                                                                                 \
      if (rb == 8) hipLaunchKernelGGL((lora_shrink_kernel<RT_, 8, true>), grid, block, 0, s, a);      \
      else hipLaunchKernelGGL((lora_shrink_kernel<RT_, 16, true>), grid, block, 0, s, a);             \
    } else {                                                                                          \
      if (rb == 8) hipLaunchKernelGGL((lora_shrink_kernel<RT_, 8, false>), grid, block, 0, s, a);     \
      else hipLaunchKernelGGL((lora_shrink_kernel<RT_, 16, false>), grid, block, 0, s, a);            \
    }                                                                                                 \
  }
  switch (rt) {
    case 1: FLEXCO_SHRINK(1) break;
    case 2: FLEXCO_SHRINK(2) break;
    case 3: FLEXCO_SHRINK(3) break;
    default: FLEXCO_SHRINK(4) break;
  }
#undef FLEXCO_SHRINK
  if (a.ksplit > 1)
    hipLaunchKernelGGL(lora_shrink_finalize_kernel, dim3((unsigned)(((size_t)a.rows * a.r + 255) / 256), n_mats), dim3(256),
                       0, s, a);
  return post("lora_shrink");
}

int32_t launch_relu_bwd_mask(const float* u, float* t, void* t_ext, size_t count, hipStream_t s) {
  if (count == 0) return FLEXCO_OK;
  hipLaunchKernelGGL(relu_bwd_mask_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, u, t, (bf16_t*)t_ext, count);
  return post("relu_bwd_mask");
}

int32_t launch_lora_outer_batch(const LoraOuterArgs& a, hipStream_t s) {
  if (a.n == 0 || a.count == 0) return FLEXCO_OK;
  int mx = 0;
  bool tiles_ok = a.r <= 64;     // whole 16-byte column chunks, rows and base pointers 16-byte aligned
  for (int e = 0; e < a.count; ++e) {
    mx = a.n_long[e] > mx ? a.n_long[e] : mx;
    tiles_ok = tiles_ok && a.n_long[e] % 8 == 0 && a.n_long[e] >= 8 && a.ldx[e] % 8 == 0 && aligned16(a.X[e]) && aligned16(a.U[e]);
  }
  if (tiles_ok) {
    const dim3 grid((mx + 127) / 128, a.count);
    switch ((a.r + 15) / 16) {
      case 1: hipLaunchKernelGGL(lora_outer_mfma_kernel<1>, grid, dim3(512), 0, s, a); break;
      case 2: hipLaunchKernelGGL(lora_outer_mfma_kernel<2>, grid, dim3(512), 0, s, a); break;
      case 3: hipLaunchKernelGGL(lora_outer_mfma_kernel<3>, grid, dim3(512), 0, s, a); break;
      default: hipLaunchKernelGGL(lora_outer_mfma_kernel<4>, grid, dim3(512), 0, s, a); break;
    }
    return post("lora_outer");
  }
  const dim3 grid((mx + 63) / 64, a.count);
  if (a.r <= 16)
    hipLaunchKernelGGL(lora_outer_mfma_path_kernel<16>, grid, dim3(256), 256 * 16 * sizeof(float), s, a);
  else if (a.r <= 32)
    hipLaunchKernelGGL(lora_outer_mfma_path_kernel<32>, grid, dim3(256), 256 * 32 * sizeof(float), s, a);
  else
    hipLaunchKernelGGL(lora_outer_mfma_path_kernel<64>, grid, dim3(256), 256 * 64 * sizeof(float), s, a);
  return post("lora_outer");
}

int32_t launch_lora_outer_bf16(const void* X, size_t ldx, const float* U, float* G, size_t g_i, size_t g_j, int n,
                               int n_long, int r, float scale, hipStream_t s) {
  LoraOuterArgs a;
  memset(&a, 0, sizeof(a));
  a.X[0] = (const bf16_t*)X; a.ldx[0] = ldx; a.U[0] = U; a.G[0] = G; a.g_i[0] = g_i; a.g_j[0] = g_j; a.n_long[0] = n_long;
  a.count = 1; a.n = n; a.r = r; a.scale = scale;
  return launch_lora_outer_batch(a, s);
}

}  // namespace flexco
