// bf16 projections on the matrix cores (v_mfma_f32_16x16x32_bf16), LDS-staged.
//
//   TRANS = false:  C[M, N] = A[M, K] W[N, K]^T (+ bias[N]) (+ residual[M, N])   forward form
//   TRANS = true :  C[M, N] = A[M, K] W[K, N]                                      input-gradient form
//
// The frozen base projections run over ALL tokens of the mixed batch in one launch, so a
// weight is read from HBM once per iteration whatever the mix of inference and finetuning
// tokens (the paper's fused forward, Sec. 6.2).  The input-gradient form serves the
// token-window backward, where weight gradients are pruned away (Alg. 1) and only
// dX = dY W remains.
//
// Tiling: block tile BM x BN, 256 threads = 4 wavefronts in a 2 x 2 grid, each owning
// (BM/2) x (BN/2) as 16 x 16 MFMA tiles with fp32 accumulators.  Tiles of 160 to 256 rows have a kernel of their own
// (gemm_bf16_quad_kernel), and so have input gradients of few row tiles (gemm_bf16_pair_kernel: eight wavefronts, 128 x 128).
//   * Forward form: operand tiles go from global memory straight into LDS
//     (buffer_load_dwordx4 ... lds: one wavefront instruction fills 1 KB; lane l lands at
//     base + 16 l), no staging registers and no LDS write instructions.  LDS is a ring of stages
//     (four of 32 or 40 KB for the 128-row tiles, two of 32 KB where two blocks share a CU, six of 24 KB for the
//     64-row tile) whose loads are in flight while another stage is multiplied; the per-stage barrier carries no
//     memory fence, the wait in front of it names exactly the loads that must have landed.  Rows are XOR-swizzled in 16-byte chunks (applied to the
//     global address a lane fetches) so that the ds_read_b128 operand fetches of 16 consecutive
//     rows hit 64 distinct banks.
//   * Input-gradient form: the same ring; the W tile is [64][BN] (k-major as in memory), loaded
//     the same way, and an MFMA operand (8 consecutive k of one column) comes from two
//     transposing LDS reads (ds_read_b64_tr_b16).
// Work-group ids are remapped so that ids that land on the same XCD (id mod 8) work on
// neighbouring tiles of the same range of K, M fastest: the W tile they share stays in that XCD's L2.
#include <algorithm>
#include <cstring>
#include "flexco_internal.h"
#include "device_types.h"

namespace flexco {

namespace {

constexpr int BK = 64;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int frag_t __attribute__((ext_vector_type(4), may_alias));   // 8 bf16 of one row or column: an operand of a product
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define FLEXCO_LDS __attribute__((address_space(3)))

#define FLEXCO_GP(p) ((const __attribute__((address_space(1))) void*)(p))
#define FLEXCO_LP(p) ((__attribute__((address_space(3))) void*)(p))


// c += w a^T on a 16 x 16 block over 32 of K.  The W fragment is the first operand: a lane then holds, for ONE output
// row (lane % 16), 4 consecutive output columns.
// 16 x 16 x 32 products rather than 32 x 32 x 16: both have the same peak, but on real data the chip's power limit sets
// the rate, and the larger form moves every accumulator through the register file twice as often (back to back from
// registers, N(0, 1) operands: 2.04 against 1.78 PFLOP/s; on zeros 2.43 and 2.45).
// In assembly: accumulators of four registers left to the compiler wander between the two register files (64 - 330 moves
// per pass of the loop below; 0 this way).  The compiler does not see a product in it, hence FLEXCO_ACC_FENCE before
// anything else touches the accumulators (32 wait states, the products need 18) and the order of a loop's instructions
// is the one they are written in.
// Operands come from LDS reads, whose waits the compiler places for any use.  A vector instruction that writes one
// would have to be two wait states ahead of the product, which the compiler does not see to here either: fragments are
// held as whole registers (as 16-bit elements the stages behind a main loop had them reassembled, right in front
// of 11 products of the 128 x 192 tile), those stages, where paths join and copies may arise,
// carry the wait states themselves (FLEXCO_PAD), and a test reads the built code of all of them.  (Wait states in front of
// every product: 2048 x 24576 x 5120 362 -> 378 us, 1024 x 28672 x 4096 179 -> 192; behind the main loops alone: no difference.)
#define FLEXCO_PAD "s_nop 1\n\t"
#define FLEXCO_MFMA(c_, w_, a_, pad_) asm volatile(pad_ "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c_) : "v"(w_), "v"(a_));
#define FLEXCO_ACC_FENCE                                                                              \
  {                                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                \
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");                                                \
    _Pragma("unroll") for (int i = 0; i < MT; ++i)                                                    \
      _Pragma("unroll") for (int j = 0; j < NT; ++j) asm volatile("" : "+a"(acc[i][j]));              \
    __builtin_amdgcn_sched_barrier(0);                                                                \
  }

// ---- epilogue: register e of acc[i][j] is row lane % 16, column 4 (lane / 16) + e of
// the 16 x 16 block.  Stored as they lie, an instruction would touch 16 rows with 32 (bf16) or 64 (fp32)
// bytes each; measured (with 32 x 32 blocks), such stores run at about 1 TB/s where whole 128-byte lines reach 3.5.  So every
// wavefront turns its rows through a piece of the (now free) ring that only it touches (stg): accumulators in,
// 16 bytes per lane along a row out, 128 contiguous bytes or more per row and instruction.
// row0, col0 / ac_w: first row and column (act column) of this wavefront's tile. ------------
template <int MT, int NT>
__device__ __forceinline__ void store_tile_glu(const f32x4 (&acc)[MT][NT], bf16_t* stg, bf16_t* __restrict__ C, size_t ldc,
                                               const GemmGlu& glu, int M, int N, int row0, int ac_w, int lane) {
  // acc[i][2 f] (gate) and acc[i][2 f + 1] (up) belong to act columns 16 f .. + 16
  constexpr int AW = NT * 8;                       // act columns of a wavefront's tile
  constexpr int PITCH = AW + 8;                    // staged row in elements (16 bytes of padding)
  constexpr int LPR = AW / 8;                      // lanes that cover a row, 16 bytes each
  constexpr int LPRP = LPR <= 4 ? 4 : 8;           // ... rounded up to a power of two (the others idle)
  constexpr int RPI = 64 / LPRP;                   // rows per instruction
  const int l16 = lane & 15, q4 = lane >> 4;
  const int ac_end = min(glu.col0 + N / 2, glu.F);
  const int rl = lane / LPRP, cl = (lane % LPRP) * 8;
  const bool lane_on = (lane % LPRP) < LPR && ac_w + cl < ac_end;   // F % 8 == 0: a run of 8 is in or out as a whole
#pragma unroll
  for (int i = 0; i < MT; i += 2) {
    const int ni = i + 1 < MT ? 2 : 1;             // fragments of 16 rows in this group (compile-time after unrolling)
    const int rb = row0 + i * 16;
    const bool band_saves = glu.save_gate && rb + 32 > glu.save_row0 && rb < glu.save_row0 + glu.save_rows;   // uniform
#pragma unroll
    for (int what = 0; what < 3; ++what) {         // 0: act, 1: gate, 2: up (the last two for finetune rows only)
      if (what > 0 && !band_saves) break;
#pragma unroll
      for (int ii = 0; ii < ni; ++ii)
#pragma unroll
        for (int f = 0; f < NT / 2; ++f) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            // gate and up pass through the storage type first (they are what the backward pass reads back)
            const bf16_t gs = (bf16_t)acc[i + ii][2 * f][e], us = (bf16_t)acc[i + ii][2 * f + 1][e];
            const float gv = (float)gs, uv = (float)us;
            // (reciprocal instruction, 1 ulp, instead of the ten-instruction IEEE division: the tile's 64 K sigmoids are on
            // the critical path of a launch whose blocks all end together)
            o[e] = what == 0 ? (bf16_t)(gv * __builtin_amdgcn_rcpf(1.0f + __expf(-gv)) * uv) : (what == 1 ? gs : us);
          }
          *reinterpret_cast<bf16x4*>(stg + (ii * 16 + l16) * PITCH + f * 16 + 4 * q4) = o;
        }
      bf16_t* dst = what == 0 ? C : (what == 1 ? glu.save_gate : glu.save_up);
      const size_t ldd = what == 0 ? ldc : glu.ld_save;
#pragma unroll
      for (int p = 0; p < ni * 16 / RPI; ++p) {
        const int r = p * RPI + rl, row = rb + r;
        const int drow = what == 0 ? row : row - glu.save_row0;
        const bool ok = lane_on && row < M && (what == 0 || (drow >= 0 && drow < glu.save_rows));
        if (ok) *reinterpret_cast<bf16x8*>(dst + (size_t)drow * ldd + ac_w + cl) = *reinterpret_cast<const bf16x8*>(stg + r * PITCH + cl);
      }
      if (MT * NT > 16) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// fp32 staging (what is added to the accumulators - bias, residual - is added in fp32 before the one rounding):
// 32 rows x 64 columns at a time (32 columns where the wavefront's tile has that many left), rows 272 bytes apart.
// P: this K split's partial sums, else NULL.  PRE: bias and residual were fetched ahead (bpre, rpre).
constexpr int STORE_PITCH32 = 64 + 4;
template <int MT, int NT, bool PRE, int PM, int PG>
__device__ __forceinline__ void store_tile(const f32x4 (&acc)[MT][NT], float* stg, float* __restrict__ P, bf16_t* __restrict__ C,
                                           size_t ldc, const bf16_t* __restrict__ bias, const bf16_t* __restrict__ res, size_t ldr,
                                           const bf16x8 (&bpre)[PG], const bf16x8 (&rpre)[PM][PG][4], int M, int N, int row0,
                                           int col0, int lane) {
  const int l16 = lane & 15, q4 = lane >> 4;
#pragma unroll
  for (int i = 0; i < MT; i += 2) {
    const int ni = i + 1 < MT ? 2 : 1;               // fragments of 16 rows in this group (compile-time after unrolling)
    const int rb = row0 + i * 16;
#pragma unroll
    for (int j0 = 0; j0 < NT; j0 += 4) {
      const int nj = (j0 + 2 < NT) ? 2 : 1;          // 32-column halves in this group (compile-time after unrolling)
#pragma unroll
      for (int ii = 0; ii < ni; ++ii)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          if (jj >= 2 * nj) break;
          *reinterpret_cast<f32x4*>(stg + (ii * 16 + l16) * STORE_PITCH32 + jj * 16 + 4 * q4) = acc[i + ii][j0 + jj];
        }
      const int cb = col0 + j0 * 16;                 // first column of the group
      if (P) {
        // 16 lanes x 4 columns per row, 4 rows per instruction
        const int rl = lane >> 4, cl = (lane & 15) * 4;
#pragma unroll
        for (int p = 0; p < 4 * ni; ++p) {
          const int r = p * 4 + rl, row = rb + r, col = cb + cl;
          if (cl < nj * 32 && row < M && col < N)    // N % 8 == 0: a run of 4 is inside or outside as a whole
            *reinterpret_cast<f32x4*>(P + (size_t)row * N + col) = *reinterpret_cast<const f32x4*>(stg + r * STORE_PITCH32 + cl);
        }
      } else {
        // 8 lanes x 8 columns per row, 8 rows per instruction
        const int rl = lane >> 3, cl = (lane & 7) * 8;
#pragma unroll
        for (int p = 0; p < 2 * ni; ++p) {
          const int r = p * 8 + rl, row = rb + r, col = cb + cl;
          if (cl < nj * 32 && row < M && col < N) {  // N % 8 == 0: a run of 8 is inside or outside as a whole
            const f32x4 lo = *reinterpret_cast<const f32x4*>(stg + r * STORE_PITCH32 + cl);
            const f32x4 hi = *reinterpret_cast<const f32x4*>(stg + r * STORE_PITCH32 + cl + 4);
            float v[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
            if (bias) {
              bf16x8 b8;
              if constexpr (PRE) b8 = bpre[j0 / 4]; else b8 = *reinterpret_cast<const bf16x8*>(bias + col);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] += (float)b8[e];
            }
            if (res) {
              bf16x8 r8;
              if constexpr (PRE) r8 = rpre[i / 2][j0 / 4][p]; else r8 = *reinterpret_cast<const bf16x8*>(res + (size_t)row * ldr + col);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] += (float)r8[e];
            }
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (bf16_t)v[e];
            *reinterpret_cast<bf16x8*>(C + (size_t)row * ldc + col) = o;
          }
        }
      }
      // (keeps the scheduler from gathering the stores of the whole tile up front, which costs more
      // registers than the large tile has left)
      if (MT * NT > 16) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Tile (of gridDim.x) and range of K (of gridDim.y) of this block.  Blocks go to the eight XCDs in turn, so the n-th block of an
// XCD takes the n-th place of its eighth of all places, tile after tile within a range: an XCD works on one range or two, on
// neighbouring columns, and reads their part of A only (with every range in every XCD, and no order at all for tiles that are no
// multiple of eight: 1024 x 5120 x 13824 in 3 ranges 115 -> 106 us, input gradient 800 x 5120 x 27648 198 -> 170 (4)).  One row
// tile shares no weights and keeps an XCD to columns of its own, over all ranges: rows of A a multiple of 4 KB apart put a range's
// stage on one channel of the L2 (input gradient 256 x 4096 x 28672 82 us the other way, 78 this); so do the two row tiles of a
// forward product cut over 128-row tiles (200 x 5120 x 5120 35.4 us the other way, 34.6 this).  apart: this second form.
__device__ __forceinline__ void place_of_block(bool apart, int* lid, int* range) {
  if (apart && (gridDim.x & 7) == 0) {
    *range = blockIdx.y;
    *lid = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    return;
  }
  const int at = blockIdx.y * gridDim.x + blockIdx.x, total = gridDim.x * gridDim.y;
  const int xcd = at & 7, rest = total & 7;
  const int place = xcd * (total >> 3) + min(xcd, rest) + (at >> 3);      // (the first `rest` XCDs have one more)
  *range = place / (int)gridDim.x;
  *lid = place - *range * (int)gridDim.x;
}

template <int BM, int BN, bool TRANS, bool GLU = false, int NSTAGES = 0, bool SPREAD = false>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                        bf16_t* __restrict__ C, const bf16_t* __restrict__ bias,
                                                        const bf16_t* __restrict__ res, int M, int N, int K,
                                                        size_t lda, size_t ldw, size_t ldc, size_t ldr, int tiles_m,
                                                        int tiles_n, GemmExt ext, float* __restrict__ part,
                                                        GemmGlu glu) {
#ifdef __HIP_DEVICE_COMPILE__      // (the host pass knows no such assembly)
  constexpr int WM = BM / 2, WN = BN / 2, MT = WM / 16, NT = WN / 16;

  // ---- work-group id -> tile, XCD-aware ------------------------------------------------
  int lid, range;
  place_of_block(!TRANS || tiles_m == 1, &lid, &range);
  const int tm = lid % tiles_m, tn = lid / tiles_m;
  const int m0 = tm * BM, n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront-uniform: LDS bases of the tile loads stay scalar
  const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN;

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // split-K: `range` owns whole stages of K, in ranges that differ by one at most, and writes fp32 partial sums to `part`
  const int st_all = K / BK;
  const int st_beg = (int)((long)st_all * range / gridDim.y);
  const int ns = (int)((long)st_all * (range + 1) / gridDim.y) - st_beg;      // stages of this block (at least one)
  const int kbeg = st_beg * BK;
  const int l16 = lane & 15, q4 = lane >> 4;

  // ===================== operand tiles: global memory -> LDS directly ==========================
  // A ring of stages of 64 k-columns; a stage holds the A tile [BM][64] and the W tile ([BN][64]
  // in the forward form, [64][BN] in the input-gradient form), A first.  The 128-row forward
  // tiles use four stages (32 KB each at 128 columns, 40 KB - all of the LDS - at 192): up to
  // three in flight or waiting while one is multiplied.
  // The input-gradient form uses two stages of 32 KB, so that two blocks share a CU (its grids are
  // K-split into more blocks than CUs); a stage's buffer is handed to the loads of the stage after next as
  // soon as its last fragments are in registers.  The stages are separate arrays, not one indexed
  // buffer: the compiler then sees that loads in flight target an array no ds_read of that
  // moment touches, and inserts no wait of its own.
  // NSTAGES = 6 for the 64-row tile (24 KB a stage, 144 KB): batches of few tokens, whose time is the weights' way out of
  // HBM.  A block has 80 KB of weights on their way (128-row tiles, half of whose loads repeat the last row: 48 KB).  With
  // a 48-token batch at the 14B shape, reduction launches included: qkv 36 -> 21 us, down 40 -> 32 us; 8 tokens, 8B shape: o
  // 16.7 -> 12.3, down 27.7 -> 26, gate/up 4.5 TB/s either way.  (Fragments of W straight from global memory into
  // registers, a block's wavefronts cutting K, no partial sums: 5.3 TB/s for one row, but the blocks' reads of A
  // compete: 16 rows 3.8, 64 rows 1.7 TB/s.)
  // NSTAGES = 2 for a 128-row forward tile: two such blocks share a CU.  With more tiles than CUs that is 15-30 %
  // faster than one four-stage block per CU in two rounds (one block's waits are the other's products); with one
  // tile per CU the four stages win.
  constexpr int NST = NSTAGES ? NSTAGES : TRANS ? 2 : 4;            // stages in the ring
  static_assert((BM + BN) * BK * 2 * NST <= 160 * 1024, "the ring fits the LDS of a CU");
  constexpr int SL = BK / 32;                                       // MFMA k-slices per stage
  constexpr int PA = BM / 32, PB = BN / 32;                         // 1 KB load instructions per wavefront and stage
  constexpr int ST_ELEMS = (BM + BN) * BK;
  static_assert(!TRANS || BN == 128, "the input-gradient form's W tile swizzle assumes 256-byte rows");
  __shared__ __attribute__((aligned(1024))) bf16_t ring0[ST_ELEMS];
  __shared__ __attribute__((aligned(1024))) bf16_t ring1[ST_ELEMS];
  __shared__ __attribute__((aligned(1024))) bf16_t ring2[NST >= 4 ? ST_ELEMS : 8];
  __shared__ __attribute__((aligned(1024))) bf16_t ring3[NST >= 4 ? ST_ELEMS : 8];
  __shared__ __attribute__((aligned(1024))) bf16_t ring4[NST == 6 ? ST_ELEMS : 8];
  __shared__ __attribute__((aligned(1024))) bf16_t ring5[NST == 6 ? ST_ELEMS : 8];
  // [rows][64] tiles (128-byte rows): chunk c of row r is stored at chunk c ^ ((r >> 1) & 7) (the
  // variant measured fastest for the ds_read_b128 operand fetches: 85 % of the LDS peak).
  // [64][BN] W tile of the input-gradient form (256- or 512-byte rows, read by transposing LDS reads of
  // 4 consecutive rows x 32 bytes, two such blocks 8 rows apart per pass): chunk c of row r is stored at
  // chunk c ^ (4 (r & 3)) ^ (2 (r / 8 & 1)), which puts the four rows on the four 64-byte quarters of the banks
  // and the two blocks on the halves of a quarter.
#define FLEXCO_KEY(r_) (((r_) >> 1) & 7)
  // Load instruction p of wavefront w fills 1 KB = rows 8 (4 p + w) .. + 8 of a [rows][64] tile (rows
  // TR (4 p + w) .. + TR of the [64][BN] tile, TR = 512 / BN); lane l lands at base + 16 l, so it fetches from
  // global memory the logical chunk that belongs at its physical chunk.  The keys do not depend on p.
  const int d_row = lane >> 3;
  const int d_c = (lane & 7) ^ FLEXCO_KEY(wave * 8 + d_row);
  constexpr int TCH = BN / 8, TR = 64 / TCH;      // 16-byte chunks of a W-tile row, rows per load instruction
  const int t_row = lane / TCH;
  const int t_k = wave * TR + t_row;              // its row, up to a multiple of 16
  const int t_c = (lane % TCH) ^ ((t_k & 3) << 2) ^ (((t_k >> 3) & 1) << 1);
  // byte offsets from the tile's own corner - gated form: from its first gate row, the up rows F further on - in 32 bits
  // (the launcher refuses what would not fit)
  const int ac0 = GLU ? glu.col0 + tn * (BN / 2) : 0;
  unsigned oa[PA], ow[PB];
#pragma unroll
  for (int p = 0; p < PA; ++p) oa[p] = (unsigned)((size_t)min((p * 4 + wave) * 8 + d_row, M - 1 - m0) * lda * 2 + d_c * 16);
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    if (GLU) {
      // W-tile rows alternate between the two halves of W in runs of 16: rows 32 f .. + 16 are gate rows
      // (act columns tile + 16 f .. + 16), rows 32 f + 16 .. + 16 the up rows of the same columns, so that
      // a lane holds gate and up of the same 4 act columns in neighbouring accumulators
      const int rr = (p * 4 + wave) * 8 + d_row;
      const int ac = ac0 + (rr >> 5) * 16 + (rr & 15);
      ow[p] = (unsigned)(((size_t)((rr >> 4) & 1) * glu.F + (min(ac, glu.F - 1) - ac0)) * ldw * 2 + d_c * 16);
    } else if (!TRANS) {
      ow[p] = (unsigned)((size_t)min((p * 4 + wave) * 8 + d_row, N - 1 - n0) * ldw * 2 + d_c * 16);
    } else {
      int col = t_c * 8;
      if (n0 + col >= N) col = 0;   // masked at the store
      ow[p] = (unsigned)((size_t)((p * 4 + wave) * TR + t_row) * ldw * 2 + col * 2);
    }
  }
  const char* const pa = (const char*)(A + (size_t)m0 * lda + kbeg);
  const char* const pw = (const char*)(GLU ? W + (size_t)ac0 * ldw + kbeg : (TRANS ? W + (size_t)kbeg * ldw + n0 : W + (size_t)n0 * ldw + kbeg));
  const size_t wstep = TRANS ? (size_t)BK * ldw * 2 : (size_t)BK * 2;

  // stage index past the end: clamped, the loads repeat the last stage into a free buffer
  // SPREAD: a block walks its stages from one of its own on, round to the one before.  Where rows of W lie a multiple of 4 KB apart, the
  // 128 bytes that all rows' stage s takes sit on the same few memory channels, and blocks that start together stay together; column
  // tiles spread over the stages use all of them.  (Products of one row tile only: others' weights are shared
  // between row tiles.)
  const int first = SPREAD ? (int)((long)tn * ns / tiles_n) : 0;
  auto stage_at = [&](int s) {
    const int t = min(s, ns - 1) + first;
    return (size_t)(SPREAD && t >= ns ? t - ns : t);
  };
#define GEMM_SRC_A(s_) __builtin_amdgcn_make_buffer_rsrc((void*)(pa + stage_at(s_) * (BK * 2)), 0, -1, 0x00027000)
#define GEMM_SRC_W(s_) __builtin_amdgcn_make_buffer_rsrc((void*)(pw + stage_at(s_) * wstep), 0, -1, 0x00027000)
  // The 64-row tile's weights are read by one block and once: non-temporal loads (cache policy bit 1), which leave the
  // caches to what is read again.  8 x 28672 x 4096 with weights in no cache 50.6 -> 47.2 us (5.0 TB/s), calls back to
  // back, a layer of 48 tokens at the 14B shape 253 -> 229, of 8 at the 8B shape 135 -> 128 (among other work 257 -> 252 and 131 -> 122).  Tiles whose weights meet several row tiles lose
  // up to 5 % with it.
  constexpr int W_AUX = BM == 64 ? 2 : 0;
  // load instruction q of a stage's PA + PB
#define FLEXCO_LOAD(ring_, q_)                                                                        \
  {                                                                                                   \
    if ((q_) < PA)                                                                                    \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sa_, FLEXCO_LP(ring_ + ((q_) * 4 + wave) * 512), 16, oa[(q_) < PA ? (q_) : 0], 0, 0, 0); \
    else                                                                                              \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sw_, FLEXCO_LP(ring_ + BM * BK + (((q_) - PA) * 4 + wave) * 512), 16, ow[(q_) < PA ? 0 : (q_) - PA], 0, 0, W_AUX); \
  }
#define FLEXCO_DMA(ring_, s_)                                                                         \
  {                                                                                                   \
    const __amdgpu_buffer_rsrc_t sa_ = GEMM_SRC_A(s_), sw_ = GEMM_SRC_W(s_);                      \
    _Pragma("unroll") for (int q = 0; q < PA + PB; ++q) FLEXCO_LOAD(ring_, q)                         \
  }
  // Operand fragments of W in the input-gradient form come from transposing LDS reads
  // (ds_read_b64_tr_b16): within a group of 16 lanes, lane s hands in the address of 4 consecutive
  // columns, 4 (s % 4) .., of row s / 4, and lane i receives column i of those 4 rows - i.e. 4
  // consecutive k for one column, the MFMA operand order.  Group g of the wavefront covers k rows
  // 8 g .. + 8 of a slice's 32; two reads (rows 0..3 and 4..7) make the 8 k of a fragment.
  // (element offset of a read inside the W tile; one index expression from the array on: behind a longer chain of pointer
  // steps the compiler loses which array a read is from and waits for every load in flight, and did: the input-gradient
  // products took 1.2 - 1.4 times as long)
  int tr_off[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int col = wn0 + j * 16 + 4 * (lane & 3);
    tr_off[j] = (8 * q4 + (l16 >> 2)) * BN + (((col >> 3) ^ ((l16 >> 2) << 2) ^ ((q4 & 1) << 1)) * 8) + (col & 7);
  }
  // fragment q of a slice's MT + NT: rows of A first, then columns of W
#define FLEXCO_FRAG(ring_, kk_, af_, bf_, q_)                                                         \
  {                                                                                                   \
    if ((q_) < MT) {                                                                                  \
      const int r_ = wm0 + (q_) * 16 + l16;                                                           \
      af_[(q_) < MT ? (q_) : 0] = *reinterpret_cast<const frag_t*>(ring_ + r_ * BK + (((kk_) * 4 + q4) ^ FLEXCO_KEY(r_)) * 8); \
    } else {                                                                                          \
      const int j_ = (q_) < MT ? 0 : (q_) - MT;                                                       \
      if (!TRANS) {                                                                                   \
        const int r_ = wn0 + j_ * 16 + l16;                                                           \
        bf_[j_] = *reinterpret_cast<const frag_t*>(ring_ + (BM + r_) * BK + (((kk_) * 4 + q4) ^ FLEXCO_KEY(r_)) * 8); \
      } else {                                                                                        \
        const s16x4 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)(ring_ + (tr_off[j_] + (BM * BK + (kk_) * 32 * BN)))); \
        const s16x4 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)(ring_ + (tr_off[j_] + (BM * BK + ((kk_) * 32 + 4) * BN)))); \
        bf_[j_] = __builtin_shufflevector(__builtin_bit_cast(u32x2, lo_), __builtin_bit_cast(u32x2, hi_), 0, 1, 2, 3); \
      }                                                                                               \
    }                                                                                                 \
  }
  // Barrier without the memory fences of __syncthreads (those would drain every load in
  // flight): the wait before it covers exactly the stage that has to be complete, and the
  // empty asm statements keep the compiler from moving LDS accesses across it.
#define FLEXCO_WAIT_BARRIER(imm_)                                                                     \
  {                                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                \
    __builtin_amdgcn_s_waitcnt(imm_);                                                                 \
    asm volatile("" ::: "memory");                                                                    \
    __builtin_amdgcn_s_barrier();                                                                     \
    asm volatile("" ::: "memory");                                                                    \
    __builtin_amdgcn_sched_barrier(0);                                                                \
  }
  // Stage s (ring buffer cur_) enters with its slice-0 fragments in set 0.  Slices alternate
  // between the two fragment sets, each fetched one slice ahead.  In the last slice:
  //   wait until this wavefront's loads of stage s + 1 have landed (with four stages those of
  //   stage s + 2 may stay in flight), barrier -> stage s + 1 is complete for everyone, and
  //   nobody reads the freed buffer any more; start the loads of the stage that takes it over;
  //   fetch slice 0 of stage s + 1; then the last slice's MFMAs cover those latencies.
  // Why nobody does: with four or six stages it held stage s - 1, whose last fragments the products before this barrier
  // have used.  With two it held stage s itself, whose last fragments were asked for in the slice before and are used
  // behind the barrier only: there the wait in front of it names the LDS reads too (lgkmcnt(0)).
  // A read (and, in the stage's last slice, a load) goes behind each product until they are used up.
#define FLEXCO_SLICE(af_, bf_, ring_, kk_, raf_, rbf_, load_, pad_)                                   \
  {                                                                                                   \
    _Pragma("unroll") for (int n = 0; n < MT * NT; ++n) {                                             \
      FLEXCO_MFMA(acc[n / NT][n % NT], bf_[n % NT], af_[n / NT], pad_)                                \
      load_                                                                                           \
      if (n < MT + NT) FLEXCO_FRAG(ring_, kk_, raf_, rbf_, n)                                         \
      __builtin_amdgcn_sched_barrier(0);                                                              \
    }                                                                                                 \
  }
#define FLEXCO_STAGE_PAD(cur_, nxt_, free_, s_, pad_)                                                 \
  {                                                                                                   \
    FLEXCO_SLICE(af0, bf0, cur_, 1, af1, bf1, , pad_)                                                 \
    FLEXCO_WAIT_BARRIER(WAIT_NEXT_STAGE)                                                              \
    const __amdgpu_buffer_rsrc_t sa_ = GEMM_SRC_A((s_) + AHEAD), sw_ = GEMM_SRC_W((s_) + AHEAD);  \
    FLEXCO_SLICE(af1, bf1, nxt_, 0, af0, bf0, if (n < NLD) FLEXCO_LOAD(free_, n), pad_)               \
  }
#define FLEXCO_STAGE(cur_, nxt_, free_, s_) FLEXCO_STAGE_PAD(cur_, nxt_, free_, s_, "")
  static_assert(SL == 2 && MT * NT >= MT + NT && MT * NT >= PA + PB, "a slice's products outnumber its reads and a stage's loads");
  constexpr int NLD = PA + PB;                                     // loads of one stage
  // s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at
  // their maxima (no wait)
#define FLEXCO_VMCNT(n_) (0x0F70 | ((n_) & 15) | (((n_) >> 4) << 14))
  // before a stage's barrier: the next stage has landed, the ones after it (up to s + 2 of four, s + 4 of six) may stay in flight
  // (two stages: and this wavefront's LDS reads have returned, see above)
  constexpr int WAIT_NEXT_STAGE = NST > 2 ? FLEXCO_VMCNT((NST - 3) * NLD) : 0x0070;
  // the buffer freed at stage s's barrier held stage s - 1 (four stages, six) or stage s itself (two)
  constexpr int AHEAD = NST > 2 ? NST - 1 : 2;
  // ---- operands of the rank-r extension's first step and the residual / bias of the epilogue, fetched ahead of the
  // main loop (128-row tiles: the registers are there; their round trips - one or two per block, all blocks
  // ending together - otherwise lie open at the end of the launch) --------------------------------------------
  // forward form: an entry covers a column range whose ends are multiples of 32, so each 16-column
  // fragment of the tile belongs to at most one entry; fragments outside this entry multiply zeros
  // (16 x 16 x 16 products: lane l holds k = 4 (l / 16) .. + 4 of row or column l % 16)
#define FLEXCO_EXT_SKIPS(e_) (!TRANS && !GLU && (n0 + BN <= ext.col0[e_] || n0 >= ext.col1[e_]))
#define FLEXCO_EXT_LOAD(e_, k2_, af_, bfr_)                                                           \
  {                                                                                                   \
    const bf16_t* A2_ = ext.A2[e_];                                                                   \
    const bf16_t* W2_ = ext.W2[e_];                                                                   \
    _Pragma("unroll") for (int i = 0; i < MT; ++i) {                                                  \
      const int r_ = min(m0 + wm0 + i * 16 + l16, M - 1);                                             \
      af_[i] = *reinterpret_cast<const bf16x4*>(A2_ + (size_t)r_ * ext.r + (k2_) + q4 * 4);           \
    }                                                                                                 \
    _Pragma("unroll") for (int j = 0; j < NT; ++j) {                                                  \
      if (GLU) {                                                                                      \
        /* even fragments are gate, odd ones up rows: column of the [gate | up] range the entries address */ \
        const int ac_ = glu.col0 + tn * (BN / 2) + ((wn0 + (j & ~1) * 16) >> 1) + l16;                \
        const int lc_ = (j & 1) * glu.F + ac_;                                                        \
        if (ac_ < glu.F && lc_ >= ext.col0[e_] && lc_ < ext.col1[e_]) {                               \
          bfr_[j] = *reinterpret_cast<const bf16x4*>(W2_ + (size_t)(lc_ - ext.col0[e_]) * ext.ldw2[e_] + (k2_) + q4 * 4); \
        } else {                                                                                      \
          _Pragma("unroll") for (int q = 0; q < 4; ++q) bfr_[j][q] = (bf16_t)0.f;                     \
        }                                                                                             \
      } else if (!TRANS) {                                                                            \
        const int cj_ = n0 + wn0 + j * 16;                                                            \
        if (cj_ >= ext.col0[e_] && cj_ < ext.col1[e_]) {                                              \
          const int c_ = min(cj_ + l16, ext.col1[e_] - 1) - ext.col0[e_];                             \
          bfr_[j] = *reinterpret_cast<const bf16x4*>(W2_ + (size_t)c_ * ext.ldw2[e_] + (k2_) + q4 * 4); \
        } else {                                                                                      \
          _Pragma("unroll") for (int q = 0; q < 4; ++q) bfr_[j][q] = (bf16_t)0.f;                     \
        }                                                                                             \
      } else {                                                                                        \
        const int c_ = min(n0 + wn0 + j * 16 + l16, N - 1);                                           \
        _Pragma("unroll") for (int q = 0; q < 4; ++q) bfr_[j][q] = W2_[(size_t)((k2_) + q4 * 4 + q) * ext.ldw2[e_] + c_]; \
      }                                                                                               \
    }                                                                                                 \
  }
#define FLEXCO_EXT_MFMAS(af_, bfr_)                                                                   \
  {                                                                                                   \
    _Pragma("unroll") for (int i = 0; i < MT; ++i)                                                    \
      _Pragma("unroll") for (int j = 0; j < NT; ++j)                                                  \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, bfr_[j]), __builtin_bit_cast(s16x4, af_[i]), acc[i][j], 0, 0, 0); \
  }
  // The 64-row tile has registers for the operands of eight steps: a decode batch of several adapters has one step per
  // adapter and target, each a round trip of its own otherwise (48 tokens with four adapters at the 14B shape: gate/up 64.6 -> 60.0
  // us, down 33.0 -> 31.0, the layer 252 -> 245).
  constexpr int PF = MT * NT > 16 ? 0 : BM == 64 ? 8 : 1;
#define FLEXCO_EXT_NEXT(e_, k2_)                                                                      \
  {                                                                                                   \
    k2_ += 16;                                                                                        \
    if (k2_ >= ext.r) {                                                                               \
      k2_ = 0;                                                                                        \
      do ++e_; while (e_ < ext.n && FLEXCO_EXT_SKIPS(e_));                                            \
    }                                                                                                 \
  }
  const int ext_n = range == 0 ? ext.n : 0;
  int ext_e = -1, ext_k = ext.r;                    // the first step that was not fetched ahead
  if (ext_n > 0) FLEXCO_EXT_NEXT(ext_e, ext_k) else ext_e = 0;
  int n_pf = 0;
  bf16x4 paf[PF ? PF : 1][MT], pbf[PF ? PF : 1][NT];
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (ext_e < ext_n) {
      FLEXCO_EXT_LOAD(ext_e, ext_k, paf[u], pbf[u])
      ++n_pf;
      FLEXCO_EXT_NEXT(ext_e, ext_k)
    }
  // residual and bias in the layout the epilogue stores in: 8 lanes x 8 columns per row, 8 rows per instruction,
  // 32 rows x 64 columns per group of 2 x 4 fragments
  constexpr int NG = (NT + 3) / 4;
  constexpr bool PF_RES = !GLU && MT * NT <= 24;
  bf16x8 rpre[PF_RES ? MT / 2 : 1][PF_RES ? NG : 1][4];
  bf16x8 bpre[PF_RES ? NG : 1];
  if constexpr (PF_RES) if (!part) {
#pragma unroll
    for (int j0 = 0; j0 < NT; j0 += 4) {
      const int col = n0 + wn0 + j0 * 16 + (lane & 7) * 8;
      const bool col_ok = (lane & 7) * 8 < ((j0 + 2 < NT) ? 64 : 32) && col < N;
      if (bias && col_ok) bpre[j0 / 4] = *reinterpret_cast<const bf16x8*>(bias + col);
      if (res) {
#pragma unroll
        for (int i = 0; i < MT / 2; ++i)
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const int row = m0 + wm0 + i * 32 + p * 8 + (lane >> 3);
            if (col_ok && row < M) rpre[i][j0 / 4][p] = *reinterpret_cast<const bf16x8*>(res + (size_t)row * ldr + col);
          }
      }
    }
  }
  frag_t af0[MT], bf0[NT], af1[MT], bf1[NT];
  FLEXCO_ACC_FENCE
#define FLEXCO_FIRST_FRAGS                                                                            \
  { _Pragma("unroll") for (int q = 0; q < MT + NT; ++q) FLEXCO_FRAG(ring0, 0, af0, bf0, q) }
  if constexpr (NST == 6) {
    FLEXCO_DMA(ring0, 0)
    FLEXCO_DMA(ring1, 1)
    FLEXCO_DMA(ring2, 2)
    FLEXCO_DMA(ring3, 3)
    FLEXCO_DMA(ring4, 4)
    FLEXCO_WAIT_BARRIER(FLEXCO_VMCNT(4 * NLD))
    FLEXCO_FIRST_FRAGS
    int st = 0;
    for (; st + 5 < ns; st += 6) {
      FLEXCO_STAGE(ring0, ring1, ring5, st)
      FLEXCO_STAGE(ring1, ring2, ring0, st + 1)
      FLEXCO_STAGE(ring2, ring3, ring1, st + 2)
      FLEXCO_STAGE(ring3, ring4, ring2, st + 3)
      FLEXCO_STAGE(ring4, ring5, ring3, st + 4)
      FLEXCO_STAGE(ring5, ring0, ring4, st + 5)
    }
    if (st < ns) FLEXCO_STAGE_PAD(ring0, ring1, ring5, st, FLEXCO_PAD)
    if (st + 1 < ns) FLEXCO_STAGE_PAD(ring1, ring2, ring0, st + 1, FLEXCO_PAD)
    if (st + 2 < ns) FLEXCO_STAGE_PAD(ring2, ring3, ring1, st + 2, FLEXCO_PAD)
    if (st + 3 < ns) FLEXCO_STAGE_PAD(ring3, ring4, ring2, st + 3, FLEXCO_PAD)
    if (st + 4 < ns) FLEXCO_STAGE_PAD(ring4, ring5, ring3, st + 4, FLEXCO_PAD)
  } else if constexpr (NST == 4) {
    FLEXCO_DMA(ring0, 0)
    FLEXCO_DMA(ring1, 1)
    FLEXCO_DMA(ring2, 2)
    FLEXCO_WAIT_BARRIER(FLEXCO_VMCNT(2 * NLD))
    FLEXCO_FIRST_FRAGS
    int st = 0;
    for (; st + 3 < ns; st += 4) {
      FLEXCO_STAGE(ring0, ring1, ring3, st)
      FLEXCO_STAGE(ring1, ring2, ring0, st + 1)
      FLEXCO_STAGE(ring2, ring3, ring1, st + 2)
      FLEXCO_STAGE(ring3, ring0, ring2, st + 3)
    }
    if (st < ns) FLEXCO_STAGE_PAD(ring0, ring1, ring3, st, FLEXCO_PAD)
    if (st + 1 < ns) FLEXCO_STAGE_PAD(ring1, ring2, ring0, st + 1, FLEXCO_PAD)
    if (st + 2 < ns) FLEXCO_STAGE_PAD(ring2, ring3, ring1, st + 2, FLEXCO_PAD)
  } else {
    FLEXCO_DMA(ring0, 0)
    FLEXCO_DMA(ring1, 1)
    FLEXCO_WAIT_BARRIER(FLEXCO_VMCNT(NLD))
    FLEXCO_FIRST_FRAGS
    int st = 0;
    for (; st + 1 < ns; st += 2) {
      FLEXCO_STAGE(ring0, ring1, ring0, st)
      FLEXCO_STAGE(ring1, ring0, ring1, st + 1)
    }
    if (st < ns) FLEXCO_STAGE_PAD(ring0, ring1, ring0, st, FLEXCO_PAD)
  }
  __builtin_amdgcn_s_waitcnt(FLEXCO_VMCNT(0));   // nothing may land in LDS after the block ends
  FLEXCO_ACC_FENCE

  // ---- rank-r extension: C += A2 W2^T (forward form; the entry whose column range holds this
  // block) or C += sum_e A2_e W2_e (input-gradient form; every entry).  This is the LoRA bypass
  // network (Sec. 4.1) folded into the base projection as extra k-steps of 16, operands read
  // straight from global memory (they are [rows, r] / [r, cols] matrices of a few KB per tile).
  // The first PF steps' operands were fetched before the main loop where the tile leaves registers for them.
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (u < n_pf) FLEXCO_EXT_MFMAS(paf[u], pbf[u])
  while (ext_e < ext_n) {
    bf16x4 af[MT], bfr[NT];
    FLEXCO_EXT_LOAD(ext_e, ext_k, af, bfr)
    FLEXCO_EXT_MFMAS(af, bfr)
    FLEXCO_EXT_NEXT(ext_e, ext_k)
  }
  __syncthreads();   // every wavefront is done with the ring, and (after its own wait above) its loads have landed
  if constexpr (GLU) {
    static_assert(4 * 32 * (WN / 2 + 8) <= ST_ELEMS, "the staged act rows of four wavefronts fit a stage");
    store_tile_glu<MT, NT>(acc, ring0 + wave * 32 * (WN / 2 + 8), C, ldc, glu, M, N, m0 + wm0, glu.col0 + tn * (BN / 2) + (wn0 >> 1), lane);
  } else {
    static_assert(2 * 32 * STORE_PITCH32 * 4 <= ST_ELEMS * 2, "the staged rows of two wavefronts fit a stage");
    store_tile<MT, NT, PF_RES>(acc, reinterpret_cast<float*>(wave < 2 ? ring0 : ring1) + (wave & 1) * 32 * STORE_PITCH32,
                               part ? part + (size_t)range * M * N : nullptr, C, ldc, bias, res, ldr, bpre, rpre, M, N, m0 + wm0, n0 + wn0, lane);
  }
#endif
}

// The 256-row tiles (256 x 256, and 256 x 192 and 256 x 128 in the forward form): four wavefronts, one per SIMD, 2 x 2 of 128 x 128
// (96, 64) each.  (Written below for 256 columns; at 192 (128) a W half-tile has 96 (64) columns and a phase 64 x 48 (32) of the
// wavefront's tile.)
//
// What bounds it: the matrix pipes, if the loads keep up; a block of 64 KB per 64 columns of K needs about 3000 cycles of
// cover for a load under load, and two whole 64 KB stages give 2048.  So LDS is eight half-tiles of 16 KB (two stages x
// {A0, A1, W0, W1}; A0 / A1 hold the first / second 64 rows of each wavefront's 128, W0 / W1 the same of its columns), and
// a stage is four phases of 32 products (64 x 64 of the wavefront's tile).  While a phase multiplies what is in
// registers, the half-tile the next phase needs is read from LDS, and the buffer that the phase before has read takes the
// load that will be read seven phases on (about 3500 cycles).  Every half-tile is read exactly once:
//     even stage s:  A0 x W0 (reads W1(s)),  A0 x W1 (reads A1(s)),  A1 x W1 (reads A0(s + 1)),  A1 x W0 (reads W1(s + 1))
//     odd stage s:   A0 x W1 (reads W0(s)),  A0 x W0 (reads A1(s)),  A1 x W0 (reads A0(s + 1)),  A1 x W1 (reads W0(s + 1))
// The vmcnt before a phase's barrier: all but the six youngest half-tiles (NA = 4 or NW = 4 (3, 2) instructions each) have landed.
// K is cut over gridDim.y blocks in whole stages, in ranges that differ by a stage at most.
// Measured against two 64 KB stages of 32 x 32 x 16 products (M x N x K, N(0, 1) x N(0, 0.02) operands): forward
// 2048 x 24576 x 5120 442 -> 383 us (1.35 PFLOP/s), 512 x 128256 x 4096 535 -> 435, 4096^3 114 -> 97; input gradient
// 1024 x 13824 x 5120 173 -> 115 us (1.26 PFLOP/s), 1536 x 8192 x 28672 895 -> 551.  What is left is the power limit (4096^3
// on zeros: 76 us) and, at K = 4096, the 10 us a tile's first loads and its epilogue take.  Eight wavefronts in two sets
// that take turns at the matrix pipes and at LDS (64 x 128 each, half as many products per barrier) were as fast with
// 32 x 32 x 16 products and read half as much again from LDS.
template <int BM, int BN, bool TRANS, bool GLU>
__global__ __launch_bounds__(256) void gemm_bf16_quad_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                             bf16_t* __restrict__ C, const bf16_t* __restrict__ bias,
                                                             const bf16_t* __restrict__ res, int M, int N, int K,
                                                             size_t lda, size_t ldw, size_t ldc, size_t ldr, int tiles_m,
                                                             int tiles_n, GemmExt ext, float* __restrict__ part,
                                                             GemmGlu glu) {
#ifdef __HIP_DEVICE_COMPILE__
  // HM0, HM1, HN: 16-row fragments of A0 and A1 (one more in A0 where the tile has an odd number), 16-column fragments of a phase
  constexpr int MT = BM / 32, NT = BN / 32, HM1 = MT / 2, HM0 = MT - HM1, HN = NT / 2;
  constexpr int NA0 = HM0, NA1 = HM1, NW = HN;                    // load instructions of a half-tile
  static_assert(BM % 32 == 0 && BM >= 160 && BM <= 256 && 2 * HM0 + NA1 <= 2 * HM1 * HN && 2 * HN + NA0 <= 2 * HM1 * HN,
                "a half-tile is read and another's loads go out within a phase's products");
  static_assert(BN == 256 || ((BN == 192 || BN == 128) && !TRANS), "the input-gradient form's W tile swizzle assumes 256-byte rows");
  int lid, range;
  place_of_block(tiles_m == 1, &lid, &range);
  const int tm = lid % tiles_m, tn = lid / tiles_m;
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int wm0 = wm * (BM / 2), wn0 = wn * (BN / 2);
  const int l16 = lane & 15, q4 = lane >> 4;
  const int st_all = K / BK;
  const int st_beg = (int)((long)st_all * range / gridDim.y);
  const int ns = (int)((long)st_all * (range + 1) / gridDim.y) - st_beg;      // stages of this block (at least one)
  const int kbeg = st_beg * BK;

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // (separate arrays: the compiler then sees that loads in flight target an array no ds_read of that moment touches)
  __shared__ __attribute__((aligned(1024))) bf16_t a0e[HM0 * 32 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t a0o[HM0 * 32 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t a1e[HM1 * 32 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t a1o[HM1 * 32 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t w0e[HN * 32 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t w0o[HN * 32 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t w1e[HN * 32 * BK];
  __shared__ __attribute__((aligned(1024))) bf16_t w1o[HN * 32 * BK];

  // ---- loads: instruction p of wavefront w fills 1 KB of a half-tile: rows 8 (4 p + w) .. + 8 of [128][64], or
  // rows 4 (4 p + w) .. + 4 of [64][128].  16-byte chunk c of a 128-byte row r is stored at c ^ ((r / 2) % 8), of a
  // 256-byte row at c ^ 4 (r % 4) ^ 2 (r / 8 % 2) (as in the kernel above).  Byte offsets from the tile's own corner fit 32 bits. ----
  const int ac0 = GLU ? glu.col0 + tn * (BN / 2) : 0;
  unsigned oa0[NA0], oa1[NA1], ow[2][NW];
  {
    const int d_row = lane >> 3;
    const int d_c = (lane & 7) ^ (((wave * 8 + d_row) >> 1) & 7);
    const int t_row = lane >> 4;
    const int t_c = (lane & 15) ^ ((t_row & 3) << 2) ^ (((wave >> 1) & 1) << 1);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int r = (p * 4 + wave) * 8 + d_row;
      const int ra0 = (BM / 2) * (r / (16 * HM0)) + r % (16 * HM0), ra1 = (BM / 2) * (r / (16 * HM1)) + 16 * HM0 + r % (16 * HM1);
      if (p < NA0) oa0[p < NA0 ? p : 0] = (unsigned)((size_t)min(ra0, M - 1 - m0) * lda * 2 + d_c * 16);     // tile row of a half-tile's row r
      if (p < NA1) oa1[p < NA1 ? p : 0] = (unsigned)((size_t)min(ra1, M - 1 - m0) * lda * 2 + d_c * 16);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (p >= NW) continue;
        const int rt = (BN / 2) * (r / (BN / 4)) + (BN / 4) * h + r % (BN / 4);      // the same for rows of W
        if (GLU) {
          const int ac = ac0 + (rt >> 5) * 16 + (rt & 15);
          ow[h][p] = (unsigned)(((size_t)((rt >> 4) & 1) * glu.F + (min(ac, glu.F - 1) - ac0)) * ldw * 2 + d_c * 16);
        } else if (!TRANS) {
          ow[h][p] = (unsigned)((size_t)min(rt, N - 1 - n0) * ldw * 2 + d_c * 16);
        } else {
          const int cl = t_c * 8;
          int col = 128 * (cl >> 6) + 64 * h + (cl & 63);
          if (n0 + col >= N) col = 0;                                // masked at the store
          ow[h][p] = (unsigned)((size_t)((p * 4 + wave) * 4 + t_row) * ldw * 2 + col * 2);
        }
      }
    }
  }
  const char* const pa = (const char*)(A + (size_t)m0 * lda + kbeg);
  const char* const pw = (const char*)(GLU ? W + (size_t)ac0 * ldw + kbeg : (TRANS ? W + (size_t)kbeg * ldw + n0 : W + (size_t)n0 * ldw + kbeg));
  const size_t wstep = TRANS ? (size_t)BK * ldw * 2 : (size_t)BK * 2;
  // (a stage past the end: clamped, the loads repeat the last stage into a free buffer)
  // (one row tile, which the 128-column form is for, and rows of W a multiple of 4 KB apart: column tiles start at stages of
  // their own, see the kernel above; gated 256 x 28672 x 4096 69 -> 63 us.  The other forms were 1 % slower for these three instructions a phase)
  constexpr bool SPREAD = BN == 128;
  const int first = SPREAD && tiles_m == 1 && (ldw & 2047) == 0 ? (int)((long)tn * ns / tiles_n) : 0;
  auto stage_at = [&](int s) {
    const int t = min(s, ns - 1) + first;
    return (size_t)(SPREAD && t >= ns ? t - ns : t);
  };
#define Q_LOAD(buf_, src_, off_, p_) \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(src_, FLEXCO_LP(buf_ + ((p_) * 4 + wave) * 512), 16, off_[p_], 0, 0, 0);
#define Q_LOAD_A(buf_, h_, s_) \
  { const __amdgpu_buffer_rsrc_t b_ = GEMM_SRC_A(s_); _Pragma("unroll") for (int p = 0; p < NA##h_; ++p) Q_LOAD(buf_, b_, oa##h_, p) }
#define Q_LOAD_W(buf_, g_, s_) \
  { const __amdgpu_buffer_rsrc_t b_ = GEMM_SRC_W(s_); _Pragma("unroll") for (int p = 0; p < NW; ++p) Q_LOAD(buf_, b_, ow[g_], p) }
  const int key = l16 >> 1;
  int tr_off[HN];       // (one index expression from the array on, see the kernel above)
#pragma unroll
  for (int jj = 0; jj < HN; ++jj) {
    const int col = wn * 64 + jj * 16 + 4 * (lane & 3);
    tr_off[jj] = (8 * q4 + (l16 >> 2)) * 128 + (((col >> 3) ^ ((l16 >> 2) << 2) ^ ((q4 & 1) << 1)) * 8) + (col & 7);
  }
  // fragment q_ (16 rows or columns x 32 of K) of the eight (six) a wavefront reads of a half-tile
#define Q_READ_ROWS(dst_, buf_, rows_, n_, q_)                                                        \
  dst_[(q_) % n_][(q_) / n_] = *reinterpret_cast<const frag_t*>(buf_ + (rows_ + ((q_) % n_) * 16 + l16) * BK + ((((q_) / n_) * 4 + q4) ^ key) * 8);
#define Q_READ_A0(dst_, buf_, q_) if ((q_) < 2 * HM0) Q_READ_ROWS(dst_, buf_, wm * (16 * HM0), HM0, (q_) % (2 * HM0))
#define Q_READ_A1(dst_, buf_, q_) if ((q_) < 2 * HM1) Q_READ_ROWS(dst_, buf_, wm * (16 * HM1), HM1, (q_) % (2 * HM1))
#define Q_READ_W(dst_, buf_, q_)                                                                      \
  if ((q_) < 2 * HN) {                                                                                \
    if (!TRANS) {                                                                                     \
      Q_READ_ROWS(dst_, buf_, wn * (BN / 4), HN, (q_) % (2 * HN))                                     \
    } else {                                                                                          \
      const s16x4 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)(buf_ + (tr_off[(q_) % HN] + (((q_) / HN) & 1) * 32 * 128)));       \
      const s16x4 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)(buf_ + (tr_off[(q_) % HN] + ((((q_) / HN) & 1) * 32 + 4) * 128))); \
      dst_[(q_) % HN][((q_) / HN) & 1] = __builtin_shufflevector(__builtin_bit_cast(u32x2, lo_), __builtin_bit_cast(u32x2, hi_), 0, 1, 2, 3); \
    }                                                                                                 \
  }
#define Q_WAIT(n_) (0x0070 | ((n_) & 15) | (((n_) >> 4) << 14))      /* vmcnt(n), lgkmcnt(0) */
  // a phase: 32 (24, 16) products; behind each second one (each of 16) goes a read for the next phase, then the loads into the
  // buffer the last phase has read.  At its end this wavefront's reads are in registers and its loads of the half-tile that is read
  // next have landed (vm_: instructions of the six younger ones)
#define Q_PHASE(READ_, nr_, rdst_, rbuf_, lbuf_, lsrc_, loff_, nl_, i0_, hm_, j0_, a_, w_, vm_, pad_)  \
  {                                                                                                   \
    constexpr int PH = 2 * hm_ * HN;                               /* products of the phase */        \
    const __amdgpu_buffer_rsrc_t src_ = lsrc_;                                                        \
    _Pragma("unroll") for (int n = 0; n < PH; ++n) {                                                  \
      FLEXCO_MFMA(acc[i0_ + (n / HN) % hm_][j0_ + n % HN], w_[n % HN][n / (hm_ * HN)], a_[(n / HN) % hm_][n / (hm_ * HN)], pad_) \
      if (PH >= 24) {                                                                                 \
        if ((n & 1) && n < 16) READ_(rdst_, rbuf_, n >> 1)                                            \
        if ((n & 1) && n >= 16 && n < 16 + 2 * nl_) Q_LOAD(lbuf_, src_, loff_, ((n - 16) >> 1) % nl_) \
        if (n & 1) __builtin_amdgcn_sched_barrier(0);                                                 \
      } else {                                                                                        \
        if (n < nr_) READ_(rdst_, rbuf_, n)                                                           \
        if (n >= nr_ && n < nr_ + nl_) Q_LOAD(lbuf_, src_, loff_, (n - nr_) % nl_)                    \
        __builtin_amdgcn_sched_barrier(0);                                                            \
      }                                                                                               \
    }                                                                                                 \
    Q_END(vm_)                                                                                        \
  }
#define Q_END(vm_)                                                                                    \
  {                                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                \
    __builtin_amdgcn_s_waitcnt(Q_WAIT(vm_));                                                          \
    asm volatile("" ::: "memory");                                                                    \
    __builtin_amdgcn_s_barrier();                                                                     \
    asm volatile("" ::: "memory");                                                                    \
    __builtin_amdgcn_sched_barrier(0);                                                                \
  }
  // (a stage's loads go out in the order W, W, A1, A0)
  constexpr int VM0 = 2 * NA0 + NA1 + 3 * NW, VM1 = NA0 + NA1 + 4 * NW, VM2 = NA0 + 2 * NA1 + 3 * NW, VM3 = 2 * NA0 + 2 * NA1 + 2 * NW;
#define Q_EVEN(s_, pad_)                                                                              \
  {                                                                                                   \
    Q_PHASE(Q_READ_W, 2 * HN, fw1, w1e, w0e, GEMM_SRC_W((s_) + 2), ow[0], NW, 0, HM0, 0, fa0, fw0, VM0, pad_)        \
    Q_PHASE(Q_READ_A1, 2 * HM1, fa1, a1e, w1e, GEMM_SRC_W((s_) + 2), ow[1], NW, 0, HM0, HN, fa0, fw1, VM1, pad_)     \
    Q_PHASE(Q_READ_A0, 2 * HM0, fa0, a0o, a1e, GEMM_SRC_A((s_) + 2), oa1, NA1, HM0, HM1, HN, fa1, fw1, VM2, pad_)    \
    Q_PHASE(Q_READ_W, 2 * HN, fw1, w1o, a0o, GEMM_SRC_A((s_) + 3), oa0, NA0, HM0, HM1, 0, fa1, fw0, VM3, pad_)       \
  }
#define Q_ODD(s_, pad_)                                                                               \
  {                                                                                                   \
    Q_PHASE(Q_READ_W, 2 * HN, fw0, w0o, w1o, GEMM_SRC_W((s_) + 2), ow[1], NW, 0, HM0, HN, fa0, fw1, VM0, pad_)       \
    Q_PHASE(Q_READ_A1, 2 * HM1, fa1, a1o, w0o, GEMM_SRC_W((s_) + 2), ow[0], NW, 0, HM0, 0, fa0, fw0, VM1, pad_)      \
    Q_PHASE(Q_READ_A0, 2 * HM0, fa0, a0e, a1o, GEMM_SRC_A((s_) + 2), oa1, NA1, HM0, HM1, 0, fa1, fw0, VM2, pad_)     \
    Q_PHASE(Q_READ_W, 2 * HN, fw0, w0e, a0e, GEMM_SRC_A((s_) + 3), oa0, NA0, HM0, HM1, HN, fa1, fw1, VM3, pad_)      \
  }
  // The rank-r extension's steps (entry, 16 of its rank) in turn, entries that miss the tile left out.  The operands of the
  // first step are fetched here: their round trip lies open behind the main loop otherwise, every tile (1 % of a 1024-row
  // window's backward; two steps' operands, where there are registers for them, were no faster).
  const int ext_n = range == 0 ? ext.n : 0;
  int ext_e = -1, ext_k = ext.r;
  bf16x4 xa[MT], xw[NT];
  if (ext_n > 0) FLEXCO_EXT_NEXT(ext_e, ext_k)
  const bool ext_on = ext_n > 0 && ext_e < ext_n;
  if (ext_on) FLEXCO_EXT_LOAD(ext_e, ext_k, xa, xw)
  frag_t fa0[HM0][2], fa1[HM1][2], fw0[HN][2], fw1[HN][2];
  Q_LOAD_A(a0e, 0, 0) Q_LOAD_W(w0e, 0, 0) Q_LOAD_W(w1e, 1, 0) Q_LOAD_A(a1e, 1, 0)
  Q_LOAD_A(a0o, 0, 1) Q_LOAD_W(w1o, 1, 1) Q_LOAD_W(w0o, 0, 1) Q_LOAD_A(a1o, 1, 1)
  Q_END(VM2)                                     // A0(0), W0(0) have landed
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    Q_READ_A0(fa0, a0e, q)
    Q_READ_W(fw0, w0e, q)
  }
  Q_END(VM2)
  Q_LOAD_A(a0e, 0, 2)
  FLEXCO_ACC_FENCE
  Q_END(VM3)                                     // W1(0)
  int st = 0;
  for (; st + 1 < ns; st += 2) {
    Q_EVEN(st, "")
    Q_ODD(st + 1, "")
  }
  if (st < ns) Q_EVEN(st, FLEXCO_PAD)
  __builtin_amdgcn_s_waitcnt(Q_WAIT(0));         // nothing may land in LDS after the block ends
  FLEXCO_ACC_FENCE

  // ---- rank-r extension (see the kernel above) ----
  if (ext_on) {
    FLEXCO_EXT_MFMAS(xa, xw)
    FLEXCO_EXT_NEXT(ext_e, ext_k)
    while (ext_e < ext_n) {
      bf16x4 af[MT], bfr[NT];
      FLEXCO_EXT_LOAD(ext_e, ext_k, af, bfr)
      FLEXCO_EXT_MFMAS(af, bfr)
      FLEXCO_EXT_NEXT(ext_e, ext_k)
    }
  }
  __syncthreads();   // every wavefront is done with the half-tiles, and (after its own wait above) its loads have landed
  // (a half-tile per wavefront to turn its rows in)
  bf16_t* const stg = wave == 0 ? a0e : wave == 1 ? a0o : wave == 2 ? (HM1 > 2 ? a1e : w0e) : (HM1 > 2 ? a1o : w0o);
  constexpr int STG = (HM1 > 2 || HN > HM1 ? 3 : 2) * 32 * BK;     // elements of the smallest of them
  static_assert(32 * STORE_PITCH32 * 4 <= STG * 2 && 32 * (NT * 8 + 8) <= STG, "the staged rows of a wavefront fit a half-tile");
  if constexpr (GLU) {
    store_tile_glu<MT, NT>(acc, stg, C, ldc, glu, M, N, m0 + wm0, glu.col0 + tn * (BN / 2) + (wn0 >> 1), lane);
  } else {
    bf16x8 bpre[1], rpre[1][1][4];
    store_tile<MT, NT, false>(acc, reinterpret_cast<float*>(stg), part ? part + (size_t)range * M * N : nullptr, C, ldc,
                              bias, res, ldr, bpre, rpre, M, N, m0 + wm0, n0 + wn0, lane);
  }
#endif
}

// Input-gradient products of few row tiles: 128 x 128 tiles by eight wavefronts in two groups of four (2 x 2 of 64 x 64 each, two
// wavefronts per SIMD).  A group multiplies its half of every stage's 64 of K, and the groups' sums are added through LDS at
// the end.
// What bounds these products is the weights' way in (256 x 14336 and 16384, K 1024 to 4096: about 53 GB/s per CU of operand tiles,
// whatever the ring's depth; 0.60 to 0.63 us per stage with weights from HBM, 0.41 from the memory-side cache), and what they pay on top is partial sums: to
// fill the chip with two blocks of four wavefronts per CU takes twice the ranges of K.  One block of eight has the second
// wavefront per SIMD without them, and a ring of four stages instead of two.  Products and the launch that adds the ranges, us, M x N x K,
// two blocks per CU -> this kernel (ranges): 256 x 14336 x 4096 57 -> 47 (2 -> 1), 256 x 4096 x 4096 26.7 -> 22.6 (8 -> 4),
// 256 x 4096 x 6144 32.4 -> 27.7 (8 -> 4), 128 x 4096 x 28672 65 -> 58, 1024 x 4096 x 4096 54 -> 42 (4 -> 1).  A ring of five
// stages and rows of A and W 128 or 256 bytes off the multiples of 4 KB: the same to 2 %; the forward form built this way: the
// same as its four wavefronts.
__global__ __launch_bounds__(512) void gemm_bf16_pair_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                             bf16_t* __restrict__ C, const bf16_t* __restrict__ bias,
                                                             const bf16_t* __restrict__ res, int M, int N, int K,
                                                             size_t lda, size_t ldw, size_t ldc, size_t ldr, int tiles_m,
                                                             int tiles_n, GemmExt ext, float* __restrict__ part,
                                                             GemmGlu glu) {
#ifdef __HIP_DEVICE_COMPILE__
  constexpr bool TRANS = true, GLU = false;
  constexpr int BM = 128, BN = 128, NST = 4, NT = 4, NA = 2, NW = 2;       // NA, NW: load instructions of a wavefront and stage
  constexpr int ST_ELEMS = (BM + BN) * BK;
  int lid, range;
  place_of_block(tiles_m == 1, &lid, &range);
  const int tm = lid % tiles_m, tn = lid / tiles_m;
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2;
  const int fm0 = ((wave >> 1) & 1) * 64, wn0 = (wave & 1) * 64;  // corner of the wavefront's 64 x 64
  const int wm0 = fm0 + grp * 32;                                 // ... of the 32 x 64 it finishes
  const int l16 = lane & 15, q4 = lane >> 4;
  const int st_all = K / BK;
  const int st_beg = (int)((long)st_all * range / gridDim.y);
  const int ns = (int)((long)st_all * (range + 1) / gridDim.y) - st_beg;      // stages of this block (at least one)
  const int kbeg = st_beg * BK;

  __shared__ __attribute__((aligned(1024))) bf16_t ring0[ST_ELEMS];
  __shared__ __attribute__((aligned(1024))) bf16_t ring1[ST_ELEMS];
  __shared__ __attribute__((aligned(1024))) bf16_t ring2[ST_ELEMS];
  __shared__ __attribute__((aligned(1024))) bf16_t ring3[ST_ELEMS];
  const int d_row = lane >> 3;
  const int d_c = (lane & 7) ^ FLEXCO_KEY(wave * 8 + d_row);
  const int t_row = lane >> 4;
  const int t_k = wave * 4 + t_row;
  const int t_c = (lane & 15) ^ ((t_k & 3) << 2) ^ (((t_k >> 3) & 1) << 1);
  unsigned oa[NA], ow[NW];
#pragma unroll
  for (int p = 0; p < NA; ++p) oa[p] = (unsigned)((size_t)min((p * 8 + wave) * 8 + d_row, M - 1 - m0) * lda * 2 + d_c * 16);
#pragma unroll
  for (int p = 0; p < NW; ++p) {
    int col = t_c * 8;
    if (n0 + col >= N) col = 0;   // masked at the store
    ow[p] = (unsigned)((size_t)(p * 32 + t_k) * ldw * 2 + col * 2);
  }
  const char* const pa = (const char*)(A + (size_t)m0 * lda + kbeg);
  const char* const pw = (const char*)(W + (size_t)kbeg * ldw + n0);
  const size_t wstep = (size_t)BK * ldw * 2;
  auto stage_at = [&](int s) { return (size_t)min(s, ns - 1); };
  // load instruction q of a stage's NA + NW
#define P_LOAD(ring_, q_)                                                                             \
  {                                                                                                   \
    if ((q_) < NA)                                                                                    \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sa_, FLEXCO_LP(ring_ + ((q_) * 8 + wave) * 512), 16, oa[(q_) < NA ? (q_) : 0], 0, 0, 0); \
    else                                                                                              \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(sw_, FLEXCO_LP(ring_ + BM * BK + (((q_) - NA) * 8 + wave) * 512), 16, ow[(q_) < NA ? 0 : (q_) - NA], 0, 0, 0); \
  }
#define P_DMA(ring_, s_)                                                                              \
  {                                                                                                   \
    const __amdgpu_buffer_rsrc_t sa_ = GEMM_SRC_A(s_), sw_ = GEMM_SRC_W(s_);                      \
    _Pragma("unroll") for (int q = 0; q < NA + NW; ++q) P_LOAD(ring_, q)                              \
  }
  // element offsets of the wavefront's fragments in a stage, its half of K
  int a_off[4], w_off[NT];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = fm0 + i * 16 + l16;
    a_off[i] = r * BK + ((grp * 4 + q4) ^ FLEXCO_KEY(r)) * 8;
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int col = wn0 + j * 16 + 4 * (lane & 3);
    w_off[j] = BM * BK + grp * 32 * BN + (8 * q4 + (l16 >> 2)) * BN + (((col >> 3) ^ ((l16 >> 2) << 2) ^ ((q4 & 1) << 1)) * 8) + (col & 7);
  }
#define P_FRAG(ring_, af_, bf_, q_)                                                                   \
  {                                                                                                   \
    if ((q_) < 4) {                                                                                   \
      af_[(q_) & 3] = *reinterpret_cast<const frag_t*>(ring_ + a_off[(q_) & 3]);                      \
    } else {                                                                                          \
      const s16x4 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)(ring_ + w_off[(q_) & 3]));            \
      const s16x4 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FLEXCO_LDS s16x4*)(ring_ + (w_off[(q_) & 3] + 4 * BN))); \
      bf_[(q_) & 3] = __builtin_shufflevector(__builtin_bit_cast(u32x2, lo_), __builtin_bit_cast(u32x2, hi_), 0, 1, 2, 3); \
    }                                                                                                 \
  }
  // Before stage s's products: this wavefront's fragments of stage s are in registers and its loads of stage s + 1 have
  // landed; behind the barrier that holds for all, so stage s's buffer takes the loads of stage s + NST.
#define P_STAGE(cur_, nxt_, s_, af_, bf_, raf_, rbf_, pad_)                                           \
  {                                                                                                   \
    P_BARRIER((NST - 2) * (NA + NW))                                                                  \
    const __amdgpu_buffer_rsrc_t sa_ = GEMM_SRC_A((s_) + NST), sw_ = GEMM_SRC_W((s_) + NST);      \
    _Pragma("unroll") for (int n = 0; n < 16; ++n) {                                                  \
      FLEXCO_MFMA(acc[n / NT][n % NT], bf_[n % NT], af_[n / NT], pad_)                                \
      if (n < 8) P_FRAG(nxt_, raf_, rbf_, n)                                                          \
      if (n >= 8 && n < 8 + NA + NW) P_LOAD(cur_, n - 8)                                              \
      __builtin_amdgcn_sched_barrier(0);                                                              \
    }                                                                                                 \
  }
#define P_BARRIER(vm_)                                                                                \
  {                                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                \
    __builtin_amdgcn_s_waitcnt(Q_WAIT(vm_));                                                          \
    asm volatile("" ::: "memory");                                                                    \
    __builtin_amdgcn_s_barrier();                                                                     \
    asm volatile("" ::: "memory");                                                                    \
    __builtin_amdgcn_sched_barrier(0);                                                                \
  }
  const int ext_n = range == 0 ? ext.n : 0;
  int ext_e = -1, ext_k = ext.r;
  bf16x4 xa[2], xw[NT];
  if (ext_n > 0) FLEXCO_EXT_NEXT(ext_e, ext_k)
  const bool ext_on = ext_n > 0 && ext_e < ext_n;
  if (ext_on) {
    constexpr int MT = 2;
    FLEXCO_EXT_LOAD(ext_e, ext_k, xa, xw)
  }
  f32x4 sum[2][NT];
  // (a wavefront's piece of the free ring: 9216 bytes, three to a stage)
  auto piece = [&](int w) { return reinterpret_cast<float*>((w < 3 ? ring0 : w < 6 ? ring1 : ring2) + (w % 3) * 4608); };
  {
    constexpr int MT = 4;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
    frag_t af0[4], bf0[NT], af1[4], bf1[NT];
    P_DMA(ring0, 0)
    P_DMA(ring1, 1)
    P_DMA(ring2, 2)
    P_DMA(ring3, 3)
    FLEXCO_ACC_FENCE
    P_BARRIER((NST - 1) * (NA + NW))
#pragma unroll
    for (int q = 0; q < 8; ++q) P_FRAG(ring0, af0, bf0, q)
    int st = 0;
    for (; st + 3 < ns; st += 4) {
      P_STAGE(ring0, ring1, st, af0, bf0, af1, bf1, "")
      P_STAGE(ring1, ring2, st + 1, af1, bf1, af0, bf0, "")
      P_STAGE(ring2, ring3, st + 2, af0, bf0, af1, bf1, "")
      P_STAGE(ring3, ring0, st + 3, af1, bf1, af0, bf0, "")
    }
    if (st < ns) P_STAGE(ring0, ring1, st, af0, bf0, af1, bf1, FLEXCO_PAD)
    if (st + 1 < ns) P_STAGE(ring1, ring2, st + 1, af1, bf1, af0, bf0, FLEXCO_PAD)
    if (st + 2 < ns) P_STAGE(ring2, ring3, st + 2, af0, bf0, af1, bf1, FLEXCO_PAD)
    __builtin_amdgcn_s_waitcnt(Q_WAIT(0));         // nothing may land in LDS after this
    FLEXCO_ACC_FENCE
    __syncthreads();                               // every wavefront is done with the ring
    // each group hands the other the half of its sums that the other finishes
    float* const out = piece(wave);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) *reinterpret_cast<f32x4*>(out + (i * NT + j) * 256 + lane * 4) = grp ? acc[i][j] : acc[i + 2][j];
    __syncthreads();
    const float* const in = piece(wave ^ 4);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const f32x4 o = *reinterpret_cast<const f32x4*>(in + (i * NT + j) * 256 + lane * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[i][j][r] = (grp ? acc[i + 2][j][r] : acc[i][j][r]) + o[r];
      }
  }
  constexpr int MT = 2;
  f32x4 (&acc)[MT][NT] = sum;
  if (ext_on) {
    FLEXCO_EXT_MFMAS(xa, xw)
    FLEXCO_EXT_NEXT(ext_e, ext_k)
    while (ext_e < ext_n) {
      bf16x4 af[MT], bfr[NT];
      FLEXCO_EXT_LOAD(ext_e, ext_k, af, bfr)
      FLEXCO_EXT_MFMAS(af, bfr)
      FLEXCO_EXT_NEXT(ext_e, ext_k)
    }
  }
  // (turned in the piece that only this wavefront has read)
  float* const stg = piece(wave ^ 4);
  static_assert(32 * STORE_PITCH32 * 4 <= 9216, "the staged rows of a wavefront fit its piece");
  const bf16x8 bpre[1] = {}, rpre[1][1][4] = {};
  store_tile<MT, NT, false>(acc, stg, part ? part + (size_t)range * M * N : nullptr, C, ldc, bias, res, ldr, bpre, rpre, M, N,
                            m0 + wm0, n0 + wn0, lane);
#endif
}

// C[row, col] = sum over splits of part[split][row][col] (+ bias) (+ residual), fixed order
__global__ __launch_bounds__(256) void gemm_splitk_reduce_kernel(const float* __restrict__ part, int splits,
                                                                 bf16_t* __restrict__ C, const bf16_t* __restrict__ bias,
                                                                 const bf16_t* __restrict__ res, int M, int N,
                                                                 size_t ldc, size_t ldr) {
  const size_t idx = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= (size_t)M * N) return;
  const int row = (int)(idx / N), col = (int)(idx % N);     // N % 8 == 0: the 4 elements share a row
  const size_t mn = (size_t)M * N;
  f32x4 v = *reinterpret_cast<const f32x4*>(part + idx);
  int sp = 1;
  for (; sp + 3 <= splits; sp += 3) {        // three loads in flight, added in split order
    f32x4 w[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) w[q] = *reinterpret_cast<const f32x4*>(part + (sp + q) * mn + idx);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] += w[q][j];
  }
  for (; sp < splits; ++sp) {
    const f32x4 w = *reinterpret_cast<const f32x4*>(part + sp * mn + idx);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += w[j];
  }
  bf16x4 o;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float x = v[j];
    if (bias) x += (float)bias[col + j];
    if (res) x += (float)res[(size_t)row * ldr + col + j];
    o[j] = (bf16_t)x;
  }
  *reinterpret_cast<bf16x4*>(C + (size_t)row * ldc + col) = o;
}

template <int BN, bool TRANS, bool GLU>
auto quad_kernel(int rows) {
  if constexpr (BN == 256) if (rows == 160) return gemm_bf16_quad_kernel<160, BN, TRANS, GLU>;
  return rows == 256 ? gemm_bf16_quad_kernel<256, BN, TRANS, GLU> : rows == 224 ? gemm_bf16_quad_kernel<224, BN, TRANS, GLU> : gemm_bf16_quad_kernel<192, BN, TRANS, GLU>;
}

// PAIR: the input-gradient kernel of eight wavefronts (128 x 128); BM = 256: the kernel of 160 to 256 rows, `rows` of them
template <int BM, int BN, bool TRANS, bool GLU = false, int NSTAGES = 0, bool SPREAD = false, bool PAIR = false>
int32_t launch_cfg(const void* A, const void* W, void* C, const void* bias, const void* res, int M, int N, int K,
                   size_t lda, size_t ldw, size_t ldc, size_t ldr, const GemmExt& ext, hipStream_t s,
                   int timer_id, float* part = nullptr, int splits = 1, bool first_of_call = true,
                   const GemmGlu* glu_in = nullptr, bool skip_reduce = false, int rows = BM) {
  // all LDS is static; the 256-row tiles have a kernel of their own
  constexpr bool QUAD = BM == 256;
  constexpr int THREADS = PAIR ? 512 : 256;
  static_assert(!PAIR || (TRANS && BM == 128 && BN == 128), "the kernel of eight wavefronts has one form");
  void (*kern)(const bf16_t*, const bf16_t*, bf16_t*, const bf16_t*, const bf16_t*, int, int, int, size_t, size_t, size_t, size_t,
               int, int, GemmExt, float*, GemmGlu);
  if constexpr (QUAD) kern = quad_kernel<BN, TRANS, GLU>(rows);
  else if constexpr (PAIR) kern = gemm_bf16_pair_kernel;
  else kern = gemm_bf16_kernel<BM, BN, TRANS, GLU, NSTAGES, SPREAD>;
  GemmGlu glu;
  if (glu_in) glu = *glu_in; else memset(&glu, 0, sizeof(glu));
  const int tiles_m = (M + rows - 1) / rows, tiles_n = (N + BN - 1) / BN;
  // while the class's timer runs, the kernels carry an event pair of their own (start and end stamps of
  // the dispatch itself)
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (timer_id >= 0) (void)kernel_timer_pair(timer_id, &e0, &e1, first_of_call);
  // (the plain launch when no pair is due: it is the form a stream capture records)
#define FLEXCO_LAUNCH_TIMED(kern_, grid_, threads_, ...)                                              \
  {                                                                                                   \
    if (e0) hipExtLaunchKernelGGL(kern_, grid_, dim3(threads_), 0, s, e0, e1, 0, __VA_ARGS__);        \
    else hipLaunchKernelGGL(kern_, grid_, dim3(threads_), 0, s, __VA_ARGS__);                         \
  }
  FLEXCO_LAUNCH_TIMED(kern, dim3(tiles_m * tiles_n, splits), THREADS, (const bf16_t*)A, (const bf16_t*)W, (bf16_t*)C,
                      (const bf16_t*)bias, (const bf16_t*)res, M, N, K, lda, ldw, ldc, ldr, tiles_m, tiles_n, ext,
                      splits > 1 ? part : nullptr, glu)
  if (splits > 1 && !skip_reduce) {
    const size_t quads = ((size_t)M * N + 3) / 4;
    e0 = e1 = nullptr;
    if (timer_id >= 0) (void)kernel_timer_pair(timer_id, &e0, &e1, false);
    FLEXCO_LAUNCH_TIMED(gemm_splitk_reduce_kernel, dim3((unsigned)((quads + 255) / 256)), 256, part, splits, (bf16_t*)C,
                        (const bf16_t*)bias, (const bf16_t*)res, M, N, ldc, ldr)
  }
#undef FLEXCO_LAUNCH_TIMED
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FLEXCO_EHIP, "launch of gemm_bf16 failed: %s", hipGetErrorString(e));
  return FLEXCO_OK;
}

}  // namespace

static bool ext_fits(const GemmExt& ext, bool trans_w, int N) {
  if (ext.n == 0) return true;
  if (ext.r % 16 != 0) return false;
  if (trans_w) return true;
  for (int e = 0; e < ext.n; ++e)      // whole 32-column fragments per entry
    if (ext.col0[e] % 32 != 0 || (ext.col1[e] % 32 != 0 && ext.col1[e] != N)) return false;
  return true;
}

// The entries of `ext` restricted to output columns [c0, c1), in the coordinates of a GEMM over those
// columns only.
static GemmExt sub_ext(const GemmExt& ext, int c0, int c1) {
  GemmExt o;
  o.n = 0;
  o.r = ext.r;
  for (int e = 0; e < ext.n; ++e) {
    const int lo = std::max(ext.col0[e], c0), hi = std::min(ext.col1[e], c1);
    if (lo >= hi) continue;
    o.col0[o.n] = lo - c0;
    o.col1[o.n] = hi - c0;
    o.A2[o.n] = ext.A2[e];
    o.W2[o.n] = ext.W2[e] + (size_t)(lo - ext.col0[e]) * ext.ldw2[e];
    o.ldw2[o.n] = ext.ldw2[e];
    ++o.n;
  }
  return o;
}

// Largest split count <= want that cuts K into whole 64-wide steps and fits the partial buffer.
// Split count for a grid of `tiles` output tiles: the one with the least estimated time,
// rounds of `want` resident blocks (resident blocks per CU x 256) times the k-range of a block, plus a
// small charge per split for the partial sums it writes and the reduction reads back.  Splits cut K
// into whole 64-wide stages, at least four per block, and must fit the partial buffer.
static int pick_splits(int M, int N, int K, int tiles, size_t part_elems, int want) {
  if (part_elems == 0) return 1;
  int best = 1;
  double best_cost = 1e30;
  for (int sp = 1; sp <= 16; ++sp) {
    if (K % (sp * BK) != 0 || (sp > 1 && K / sp < 4 * BK)) continue;
    if (sp > 1 && (size_t)sp * M * N > part_elems) break;
    const int rounds = (tiles * sp + want - 1) / want;
    const double cost = (double)rounds / sp + 0.015 * (sp - 1);   // (0.02 took 7 splits where 8 fill the last CU slots: 3 % slower)
    if (cost < best_cost - 1e-12) { best_cost = cost; best = sp; }
  }
  return best;
}

// Rates of the input-gradient form's two tile shapes with every block slot taken, PFLOP/s: fitted to twelve products of
// 512 to 1536 rows at the 8B, 14B and 32B shapes with the 32 x 32 x 16 kernels (the 256 x 256 tile reaches 1.26 now).  What they
// decide is a first tile and equal cut; k_ranges prices that choice with the present kernels' times and takes the
// 256 x 256 tile, at the number of ranges that suits it, where that is estimated 7 % better; pair_ranges then puts
// the eight-wavefront kernel in the place of 128 x 128 tiles where a window has few row tiles.
constexpr double TRANS_RATE_128 = 0.94, TRANS_RATE_256 = 1.05;

// ---- estimated times, us, of launches of `blocks` blocks over `stages` 64-wide stages of K each.  Fitted to products of
// 256 to 2048 rows at the 8B, 14B and 32B shapes with N(0, 1) x N(0, 0.02) operands, weights not in a cache; within 10 % of
// each of some 150 measurements but for windows of 256 rows, which wait for HBM (up to 20 % above the estimate, all shapes
// alike).  A launch runs in rounds over the CUs; a stage of the 256-row tiles takes longer the more CUs multiply at the
// same time (the chip's power limit: 256 x 256 tiles 1.03 us at up to 128 blocks, 1.31 at 256).
// The rows of a "256-row" tile are M's own: tiles of M / n rows in 32s for the fewest row tiles n, or for one more, so that the last
// tile is not left half empty (gated 300 x 28672 x 4096 95 -> 74 us, 600 rows 161 -> 122, 800 rows 164 -> 151; input gradient
// 300 x 4096 x 28672 96 -> 86).  cols: column tiles times ranges of K.  Narrow tiles of 160 rows were no faster than of 192.
// (A class: what M alone decides is taken out of the planner's loops over columns and ranges.)
class Tile256 {
 public:
  Tile256(int M, int bn) : few_((M + 255) / 256), bn_(bn == 256 ? 0 : bn == 192 ? 1 : 2) {
    // a stage of fewer rows against one of 256, measured: 256, 192 and 128 columns wide, 160, 192 and 224 rows; in one round
    // the weights' way in weighs more, and with one row tile it is all there is
    static const double PART[2][3][3] = {{{0.82, 0.85, 0.90}, {1, 0.90, 0.96}, {1, 0.85, 0.95}}, {{0.72, 0.80, 0.90}, {1, 0.84, 0.95}, {1, 0.74, 0.92}}};
    for (int i = 0; i < 2; ++i) {
      const int n = few_ + i;
      rows_[i] = std::max(((M + n - 1) / n + 31) / 32 * 32, bn == 256 ? 160 : 192);
      for (int more = 0; more < 2; ++more) part_[i][more] = rows_[i] == 256 || few_ == 1 ? 1.0 : PART[more][bn_][(rows_[i] - 160) / 32];
    }
  }
  // cols: column tiles times ranges of K; rows: those of the tiles that take this long
  double us(long cols, double stages, int* rows = nullptr) const {
    const double t0 = us_of(0, cols, stages);
    // (in one round a tile more was as often slower where it is one of few: input gradient 512 x 14336 x 4096 66 -> 72 us)
    const double t1 = few_ >= 4 || (few_ + 1) * cols > 256 ? us_of(1, cols, stages) : 1e300;
    const bool more = t1 < t0 * 0.98;
    if (rows) *rows = rows_[more];
    return more ? t1 : t0;
  }
  // no product of these or of more columns takes less
  double at_least(long cols, double stages) const { return cols ? std::min(us_of(0, cols, stages), us_of(1, cols, stages)) : 0.0; }

 private:
  double us_of(int i, long cols, double stages) const {
    static const double STAGE[3] = {1.03, 0.85, 0.70}, OVER[3] = {0.0022, 0.0013, 0.0009};
    const long blocks = (few_ + i) * cols, rounds = (blocks + 255) / 256;
    // (blocks above 128, over the rounds; all rounds but the last are full)
    const long over = (rounds - 1) * 128 + std::max(0L, blocks - (rounds - 1) * 256 - 128);
    return rounds * (bn_ == 2 ? 5 : 9) + stages * part_[i][rounds > 1] * (STAGE[bn_] * rounds + OVER[bn_] * over);
  }
  int few_, bn_, rows_[2];       // fewest row tiles; rows of a tile with that many, and with one more
  double part_[2][2];
};
static double us_tile128x192(long blocks, double stages) { return ((blocks + 255) / 256) * (4 + 0.76 * stages); }
// 128 x 128: one four-stage block per CU, or with more blocks than CUs two two-stage blocks
static double us_tile128(long blocks, double stages) {
  if (blocks <= 256) return 3 + 0.6 * stages;
  const long rounds = (blocks + 511) / 512;
  return rounds * (3 + (blocks < 461 * rounds ? 0.95 : 1.1) * stages);
}
static double at_least_tile128(long blocks, double stages) {      // no more blocks take less
  return blocks <= 256 ? (blocks ? 3 + 0.6 * stages : 0.0) : ((blocks + 511) / 512) * (3 + 0.95 * stages);
}
// partial sums out and back in, and the launch that adds them (also where the next kernel will add them: who comes next is not
// known here)
static double us_partial_sums(int splits, int M, int N) { return splits > 1 ? 4 + (double)splits * M * N * 1e-6 : 0.0; }

// Tile shapes of a forward-form product by estimated time: columns [0, 256 a) in 256-wide tiles and the rest in ONE of
// the three narrower shapes, as two launches (a partial last round of wide tiles is what the narrower ones avoid);
// a = 0 is a single shape for the whole matrix.
struct GemmPlan {
  int a256;    // number of 256-wide column tiles
  int rest;    // shape of the remaining columns: 0 = 128 x 128, 1 = 128 x 192, 2 = 256 x 192
  double us;
};
static GemmPlan plan_forward(int M, int N, int K) {
  const double ns = K / BK;
  const long tm128 = (M + 127) / 128;
  const Tile256 wide(M, 256), narrow(M, 192);
  GemmPlan best{0, 0, 1e300};
  const int n256 = (N + 255) / 256;
  // (runs of eight a that cannot win, by the run's fewest wide and fewest other columns, are passed over: 512 x 128256 x 4096
  // 8.3 us on the host without this, 1.0 with; gated 512 x 28672 x 4096 1.6 and 0.35)
  constexpr int RUN = 8;
  for (int top = n256; top >= 0; top -= RUN) {
    const int low = std::max(top - RUN + 1, 0), least = std::max(N - 256 * top, 0);
    const long c128 = tm128 * ((least + 127) / 128), c192 = (least + 191) / 192;
    if (wide.at_least(low, ns) + std::min({at_least_tile128(c128, ns), us_tile128x192(tm128 * c192, ns), narrow.at_least(c192, ns)}) >= best.us) continue;
    for (int a = top; a >= low; --a) {
      const int rest = N - 256 * a;                 // columns left for the narrower tiles
      const double t_a = a ? wide.us(a, ns) : 0.0;
      if (rest <= 0) {
        if (t_a < best.us - 1e-9) best = GemmPlan{a, 0, t_a};
        continue;
      }
      const long c192 = (rest + 191) / 192;
      const double t_rest[3] = {us_tile128(tm128 * ((rest + 127) / 128), ns), us_tile128x192(tm128 * c192, ns), narrow.us(c192, ns)};
      for (int sh = 2; sh >= 0; --sh)
        if (t_a + t_rest[sh] < best.us - 1e-9) best = GemmPlan{a, sh, t_a + t_rest[sh]};
    }
  }
  return best;
}

// Forward products of at most THIN_ROWS rows run on 64 x 128 tiles, K cut until the tiles cover the chip, ten stages or
// more to a block (4096 columns, K = 4096: 11.8 - 12.6 us with 4 to 8 ranges, 15.9 with 12; K = 14336: 35, 29, 26 us with 4, 5, 8).
constexpr int THIN_ROWS = 64;
static int thin_splits(int M, int N, int K, size_t part_elems) {
  int sp = std::min(256 / ((N + 127) / 128), K / BK / 10);
  if (sp > 1) sp = (int)std::min<size_t>(sp, part_elems / ((size_t)M * N));
  return std::max(sp, 1);
}
// Whether the column tiles of a product of one row tile start at stages of their own: rows of W a multiple of 4 KB apart.  Asked for the
// 64-row tiles, 128 x 128 tiles cut over K and the gated 128 x 128 form on its deep ring; the whole 128 x 128 and 128 x 192 forms of up to
// 128 rows (the loss head of a short window among them) walk K in order and were not measured with it.  A layer at the
// 8B shape (8 and 28 KB), us: 1 token 116 -> 106, 8 tokens 123 -> 114, 30 tokens 143 -> 130, 70 tokens 185 -> 177, 128 tokens
// 220 -> 210, 160 and 250 tokens (two row tiles) level; at the 14B and 32B shapes (10, 27 and 54 KB) 0.4 % slower with it.
static bool spread_stages(int M, size_t ldw) { return M <= 128 && ldw % 2048 == 0; }

// Ranges of K in whole stages, equal to within one, to run a product on 256 x 256 tiles with, or 0: the choice so far, of *us, is as
// good.  For products whose 256 x 256 tiles leave CUs idle (or whose last round does), at the price of partial
// sums.  1: the tiles as they are, input-gradient form only (the forward plan has that choice).
// Measured (us, the choice so far -> ranges): forward 1024 x 4096 x 14336 135 -> 99 (4), 2048 x 4096 x 14336 210 -> 172 (2),
// 1405 x 5120 x 27648 400 -> 312 (2); input gradient 512 x 4096 x 128256 625 -> 419 (8), 512 x 4096 x 28672 152 -> 103 (8),
// 1024 x 5120 x 7168 126 -> 74 (3), 1024 x 5120 x 5120 100 -> 60 (3), 256 x 4096 x 28672 91 -> 77 (12).
static int k_ranges(int M, int N, int K, bool trans_w, size_t part_elems, double* us) {
  const int ns = K / BK;
  const long cols = (N + 255) / 256;
  const Tile256 tile(M, 256);
  int best = 0;
  double least = (trans_w ? 0.93 : 0.95) * *us;     // (the large tiles have to win clearly)
  for (int r = trans_w ? 1 : 2; r <= 16 && ns / r >= 4; ++r) {
    if (r > 1 && (size_t)r * M * N > part_elems) break;
    const double t = tile.us(cols * r, (double)((ns + r - 1) / r)) + us_partial_sums(r, M, N);
    if (t < least) { least = t; best = r; }
  }
  if (best) *us = least;
  return best;
}

// Ranges of K (1: whole) to run an input-gradient product in on the 128 x 128 kernel of eight wavefronts, or 0: by the choice so
// far (large: on 256-row tiles, in an estimated us).  One round of blocks only: more tiles than CUs are shared out better two blocks of
// four to a CU
// (512 x 14336 x 4096 83 us on this kernel, 62 on 256 x 256 tiles).  Measured on 130 products of 33 to 1024 rows at the three models'
// shapes, weights from HBM.  Against the plan's 128 x 128 tiles, two blocks to a CU: 81 to 256 rows 0.82 - 0.95 of their time, with more
// and with fewer rows 0.79 - 0.95 where the blocks fill the chip and 0.95 - 1.27 where they do not (640 x 4096 x 6144, 160
// blocks: 59 against 46 us; 33 x 14336 x 4096, 224 blocks: 36 against 31).  What it gains is at a block's ends: over hundreds of
// stages idle CUs cost more (84 to 128 rows x 5120, 240 blocks: K 55296, 144 stages, 0.96 - 1.00; K 152064, 396 stages, 1.02 - 1.08;
// 256 blocks of 250 stages, 4096 x 128256, 0.98 - 1.01).  Against 256 x 256 tiles by the estimates (this one's within 12 %), which see
// those at few rows too low: 150 x 14336 x 4096 39 us against 44 where they say 46 and 42.
static int pair_ranges(int M, int N, int K, size_t part_elems, bool large, double us) {
  const int ns = K / BK;
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
  us = large ? (M <= 192 ? 1.12 : 1.03) * us : 1e30;
  int best = 0;
  for (int r = 1; r <= 16 && tiles * r <= 256 && ns / r >= (r > 1 ? 4 : 1); ++r) {
    if (r > 1 && (size_t)r * M * N > part_elems) break;
    const double t = 6 + 0.62 * ((ns + r - 1) / r) + us_partial_sums(r, M, N);
    if (t < us) { us = t; best = r; }
  }
  const bool idle = tiles * best < 250, long_runs = best && ns / best > 200;
  return idle && (long_runs || (!large && (M > 256 || M <= 80))) ? 0 : best;
}

// Whether a forward product runs on 256 x 128 tiles, one launch over all columns, instead of by the choice so far (of other_us).
// They fill the chip where the others need a second round or leave CUs idle: measured against them, us,
// 1200 x 6144 x 4096 64 -> 52, 2048 x 4096 x 4096 63 -> 52, 1024 x 7168 x 5120 98 -> 71, 1405 x 5120 x 5120 81 -> 65,
// gated 256 x 28672 x 4096 83 -> 63.  Time: fitted to 150 products of 129 to 2048 rows.  A round of fewer than 164 blocks
// has to win by a tenth (1024 x 5120 x 5120, 160 blocks: 68 us where 128 x 192 tiles take 65).
static bool takes_256x128(int M, int N, int K, double other_us) {
  const long cols = (N + 127) / 128;
  int rows;
  const double us = Tile256(M, 128).us(cols, K / BK, &rows);
  const long blocks = (M + rows - 1) / rows * cols;
  return M > 128 && us < (blocks >= 164 && blocks <= 256 ? 0.99 : 0.90) * other_us;
}

// What the launchers below launch for a shape, and flexco_gemm_plan returns: one or two launches, each a tile shape over a range
// of output columns, possibly with K cut across blocks.  A pure function of the arguments (host arithmetic only).  The gated
// form is a forward product of 2F columns without scratch.
GemmLaunchPlan plan_gemm_mfma(int M, int N, int K, bool trans_w, size_t part_elems) {
  GemmLaunchPlan pl;
  pl.n = 0;
  const int ns = K / BK;
  auto add = [&](int bm, int bn, int cols, int splits, int stages) {
    if (bm == 256) Tile256(M, bn).us((long)((cols + bn - 1) / bn) * splits, (double)((ns + splits - 1) / splits), &bm);     // M's own rows
    pl.step[pl.n++] = GemmLaunchStep{bm, bn, cols, splits, stages};
  };
  if (trans_w) {
    // few row tiles (a finetune window) and a long contraction: cut K across blocks so that the
    // weight stream is spread over the whole chip; partial sums are reduced in split order
    // (256 x 128 tiles, one block per CU, were measured slower than two co-resident 128 x 128 blocks)
    const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
    const int sp = part_elems ? pick_splits(M, N, K, tiles, part_elems, 512) : 1;
    // A window of 512 rows or more has the rows for 256 x 256 tiles, one block per CU, which sustain more per CU
    // than two 128 x 128 blocks; few of them cover the output, so the choice goes by estimated time: whole rounds of
    // the grid over the block slots x the k-range of a block x the area a CU holds at a time over the rate of the
    // shape, plus the partial sums' way out and back in (1 us per million of them).
    int sp256 = 0;
    if (M >= 512) {
      auto est_us = [&](long blocks, int slots, int splits, double area, double pflops) {
        const double rounds = (double)((blocks * splits + slots - 1) / slots);
        return rounds * (K / splits) * area * 2.0 * 256 / (pflops * 1e9) + (splits > 1 ? (double)splits * M * N * 1e-6 : 0.0);
      };
      double best = 0.97 * est_us(tiles, 512, sp, 2.0 * 128 * 128, TRANS_RATE_128);   // (the large tile has to win clearly)
      const long tiles256 = (long)((M + 255) / 256) * ((N + 255) / 256);
      for (int c = 1; c <= 16; ++c) {
        if (K % (c * BK) != 0 || (c > 1 && (K / c < 8 * BK || (size_t)c * M * N > part_elems))) continue;
        const double t = est_us(tiles256, 256, c, 256.0 * 256, TRANS_RATE_256);
        if (t < best - 1e-9) { best = t; sp256 = c; }
      }
    }
    const int cut = sp256 ? sp256 : sp;
    const double s = (double)ns / cut;
    // (this form's 128 x 128 blocks of four wavefronts have two stages whatever their number)
    const long blocks = (long)tiles * cut;
    double us = (sp256 ? Tile256(M, 256).us((long)((N + 255) / 256) * cut, s)
                       : blocks <= 256 ? 3 + 0.85 * s : ((blocks + 511) / 512) * (3 + 1.1 * s)) + us_partial_sums(cut, M, N);
    const int ranges = k_ranges(M, N, K, true, part_elems, &us);
    if (const int pair = pair_ranges(M, N, K, part_elems, ranges || sp256, us)) add(128, 128, N, pair, 4);
    else if (ranges) add(256, 256, N, ranges, 2);
    else if (sp256) add(256, 256, N, sp256, 2);
    else add(128, 128, N, sp, 2);
    return pl;
  }
  if (M <= THIN_ROWS) {
    add(THIN_ROWS, 128, N, thin_splits(M, N, K, part_elems), 6);
    return pl;
  }
  // A batch of few tokens (decode-only iterations) has one or two row tiles and far fewer output tiles
  // than CUs, and its time is the weight stream's: cut K across blocks so that the whole chip pulls on it.
  int cut = 1;
  const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
  if (part_elems && M <= 256 && tiles < 192) cut = pick_splits(M, N, K, tiles, part_elems, 256);
  GemmPlan fp{0, 0, us_tile128((long)tiles * cut, (double)ns / cut) + us_partial_sums(cut, M, N)};
  if (cut == 1) fp = plan_forward(M, N, K);
  double us = fp.us;
  const int ranges = k_ranges(M, N, K, false, part_elems, &us);
  if (takes_256x128(M, N, K, us)) {
    add(256, 128, N, 1, 2);
    return pl;
  }
  if (ranges || cut > 1) {
    if (ranges) add(256, 256, N, ranges, 2);
    else add(128, 128, N, cut, 4);
    return pl;
  }
  const int n1 = std::min(N, 256 * fp.a256);
  if (n1 > 0) add(256, 256, n1, 1, 2);
  if (n1 < N) {
    // more 128 x 128 tiles than CUs: two-stage blocks, two per CU (the planner takes 128 x 192 tiles for single
    // rounds only)
    const long t128 = (long)((M + 127) / 128) * ((N - n1 + 127) / 128);
    if (fp.rest == 0) add(128, 128, N - n1, 1, t128 > 256 ? 2 : 4);
    else if (fp.rest == 1) add(128, 192, N - n1, 1, 4);
    else add(256, 192, N - n1, 1, 2);
  }
  return pl;
}

// The kernels address a tile's rows by 32-bit byte offsets from its first.
static bool offsets_fit(size_t ld, size_t rows) { return ld <= 0xffff0000u / 2 / rows; }

// Whether the tiled kernels take a product: K in whole 64-wide steps, 16-byte aligned rows (and 8-byte aligned runs of 4
// output columns in C, bias and residual), tile rows in reach, a rank-r extension of whole steps.
static bool takes_product(const void* C, const void* bias, const void* residual, int N, int K, size_t lda, size_t ldw,
                          size_t ldc, size_t ldr, bool trans_w, const GemmExt* ext) {
  if (K % BK != 0 || lda % 8 != 0 || ldw % 8 != 0 || N % 8 != 0 || ldc % 4 != 0 || (residual && ldr % 4 != 0) ||
      ((uintptr_t)C & 7) || ((uintptr_t)bias & 7) || ((uintptr_t)residual & 7))
    return false;
  return offsets_fit(lda, 256) && offsets_fit(ldw, 256) && (!ext || ext_fits(*ext, trans_w, N));
}

// The kernel of a launch of the plan.  spread: the column tiles may start at stages of their own.
template <bool GLU>
static auto forward_form(const GemmLaunchStep& st, bool spread) {
  if (st.bm == THIN_ROWS) return spread ? launch_cfg<THIN_ROWS, 128, false, GLU, 6, true> : launch_cfg<THIN_ROWS, 128, false, GLU, 6>;
  if (st.bm > 128) return st.bn == 256 ? launch_cfg<256, 256, false, GLU> : st.bn == 192 ? launch_cfg<256, 192, false, GLU> : launch_cfg<256, 128, false, GLU>;
  if (st.bn == 192) return launch_cfg<128, 192, false, GLU>;
  if (st.stages == 2) return launch_cfg<128, 128, false, GLU, 2>;
  return spread && (GLU || st.splits > 1) ? launch_cfg<128, 128, false, GLU, 0, true> : launch_cfg<128, 128, false, GLU>;
}
static auto input_gradient_form(const GemmLaunchStep& st) {
  if (st.bm > 128) return launch_cfg<256, 256, true>;
  return st.stages == 4 ? launch_cfg<128, 128, true, false, 0, false, true> : launch_cfg<128, 128, true>;
}

int32_t launch_gemm_mfma(const void* A, const void* W, void* C, const void* bias, const void* residual, int M, int N,
                         int K, size_t lda, size_t ldw, size_t ldc, size_t ldr, bool trans_w, const GemmExt* ext_in,
                         hipStream_t s, float* part, size_t part_elems, int timer_id, int* splits_out) {
  if (splits_out) *splits_out = 1;
  if (K % BK != 0) return FLEXCO_EUNSUPPORTED;
  const GemmLaunchPlan pl = plan_gemm_mfma(M, N, K, trans_w, part ? part_elems : 0);
  // splits_out: the caller's next kernel adds the partial sums itself (part[split][M][N], in split order), and bias and residual
  // with them; the reduction launch is left out
  const bool leave = splits_out && pl.step[0].splits > 1;
  if (leave) bias = residual = nullptr;
  if (!takes_product(C, bias, residual, N, K, lda, ldw, ldc, ldr, trans_w, ext_in)) return FLEXCO_EUNSUPPORTED;
  if (leave) *splits_out = pl.step[0].splits;
  GemmExt ext;
  if (ext_in) ext = *ext_in; else ext.n = 0;
  int c0 = 0;
  for (int i = 0; i < pl.n; ++i) {
    const GemmLaunchStep& st = pl.step[i];
    const auto form = trans_w ? input_gradient_form(st) : forward_form<false>(st, spread_stages(M, ldw));
    const bool all = st.cols == N;
    const int32_t rc = form(A, (const bf16_t*)W + (size_t)c0 * ldw, (bf16_t*)C + c0, bias ? (const bf16_t*)bias + c0 : nullptr,
                            residual ? (const bf16_t*)residual + c0 : nullptr, M, st.cols, K, lda, ldw, ldc, ldr,
                            all ? ext : sub_ext(ext, c0, c0 + st.cols), s, timer_id, part, st.splits, i == 0, nullptr, leave, st.bm);
    if (rc) return rc;
    c0 += st.cols;
  }
  return FLEXCO_OK;
}

// Gated form: the plan of a forward product of the 2F interleaved columns; a tile of BN W-rows covers
// BN / 2 act columns.
int32_t launch_gemm_glu_mfma(const void* A, const void* W, void* act, int M, int F, int K, size_t lda, size_t ldw,
                             size_t ld_act, const GemmExt* ext_in, void* save_gate, void* save_up, int save_row0,
                             int save_rows, size_t ld_save, hipStream_t s, int timer_id) {
  if (K % BK != 0 || lda % 8 != 0 || ldw % 8 != 0 || F % 8 != 0 || ld_act % 4 != 0 || ld_save % 4 != 0 ||
      ((uintptr_t)act & 7) || ((uintptr_t)save_gate & 7) || ((uintptr_t)save_up & 7))
    return FLEXCO_EUNSUPPORTED;
  if (!offsets_fit(lda, 256) || !offsets_fit(ldw, (size_t)F + 256)) return FLEXCO_EUNSUPPORTED;   // (gate and up rows of W in one tile)
  GemmExt ext;
  if (ext_in) ext = *ext_in; else ext.n = 0;
  if (ext.n > 0 && ext.r % 16 != 0) return FLEXCO_EUNSUPPORTED;
  GemmGlu glu;
  glu.F = F; glu.col0 = 0; glu.save_gate = (bf16_t*)save_gate; glu.save_up = (bf16_t*)save_up;
  glu.save_row0 = save_row0; glu.save_rows = save_gate ? save_rows : 0; glu.ld_save = ld_save;
  const int N = 2 * F;
  const GemmLaunchPlan pl = plan_gemm_mfma(M, N, K, false, 0);
  int c0 = 0;                                       // interleaved columns done = 2 x the act columns done
  for (int i = 0; i < pl.n; ++i) {
    const GemmLaunchStep& st = pl.step[i];
    glu.col0 = c0 / 2;
    const int32_t rc = forward_form<true>(st, spread_stages(M, ldw))(A, W, act, nullptr, nullptr, M, st.cols, K, lda, ldw, ld_act, 0, ext, s,
                                                                     timer_id, nullptr, 1, i == 0, &glu, false, st.bm);
    if (rc) return rc;
    c0 += st.cols;
  }
  return FLEXCO_OK;
}

}  // namespace flexco
