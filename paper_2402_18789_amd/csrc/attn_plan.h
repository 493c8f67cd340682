#pragma once
// Which attention kernel a batch's work list takes, how many of its key splits as one, and in which order.  Host arithmetic on the
// maps' sums alone.
#include <algorithm>
#include <cstdint>
#include "flexco.h"

#ifdef __HIPCC__
#define FLEXCO_HOST_DEVICE __host__ __device__
#else
#define FLEXCO_HOST_DEVICE
#endif

namespace flexco {

// The item of the work list that turn `turn` takes where the block of a request of one token takes fold neighbouring key splits as one (turns
// are dealt to the chip's parts one after the other; turns run to turns_of(n_items, fold), those past the last item have none).
// Within runs of 32 fold items, at a stride of fold: the items that are left with work are every fold-th of a request, so in the list's own
// order requests of a multiple of fold splits left all of it to every fold-th part of the chip.  Us, 8 kv heads: 24 requests of 1024
// keys in eights 49.9 -> 23.9, 4 of 3072 in fours 33.6 -> 19.2, 24 of 4096 in fours 140 -> 80; odd numbers of splits within 5 %.  Runs, so
// that the list's order - the longest first, chunks early - stays what it is (at a stride through the whole list a batch whose chunks are
// half the work 96 -> 106).
constexpr int FOLD_RUN = 32;
FLEXCO_HOST_DEVICE inline int turns_of(int n_items, int fold) { return (n_items + fold - 1) / fold * fold; }
FLEXCO_HOST_DEVICE inline int item_of_turn(int turn, int n_items, int fold) {
  const int base = turn / (FOLD_RUN * fold) * (FOLD_RUN * fold), left = n_items - base;
  const int run = left < FOLD_RUN * fold ? (left + fold - 1) / fold : FOLD_RUN;
  return base + (turn - base) % run * fold + (turn - base) / run;
}

// alone: the four-wavefront kernel takes the whole work list in one launch: its blocks, two or three per CU, keep as many
// bytes on their way as the one-wavefront kernel's items did, and share a CU between streaming and multiplying blocks.  Measured
// against what was done before (one kernel for everything, or the two beside each other on two streams; us): the 14B shape's 512 decode
// tokens with 512 + 1024 chunk rows 612 -> 568, the 8B shape's 96 decode tokens beside 211 + 205 rows 122 -> 99, 217 decode
// tokens beside 279 + 40 rows 294 -> 108, 105 beside 74 + 73 166 -> 112, chunks of 713 + 487 + 205 rows without a decode token
// 144 -> 67 (a last tile of one token had sent them to the pair of kernels).
//
// fold: the work list is cut for one wavefront per item and head, i.e. into more pieces than blocks of four need; the block of a
// request of one token takes that many neighbouring key splits as one, up to the 256 pages of its table.
//
// Where the lines lie: measured with 1 - 768 requests of fifteen length laws (16 to 8192 keys, equal and unequal), 8, 4, 2 and 32 kv heads,
// decode tokens alone and beside eight kinds of chunks, in the default cut and in nine others (4259 lists, every kernel and fold).  What decides is how the pieces fill the rounds: the chip
// holds 1024 wavefronts of the one kernel and 512 blocks of the other, and a round that is nearly empty costs as much as a full one.
// Times below: the four-wavefront kernel over the one-wavefront kernel, mean / worst of the lists between the lines.  In all, of the attention
// before the four-wavefront kernel took decode tokens: lists of nothing else 0.90 (worst 1.04), others 0.79 (1.06).
struct AttnPlan { bool alone; int fold; bool lag; };

// Lists of nothing but decode tokens.  0: the one-wavefront kernel, else the fold.
inline int plan_decode(const flexco_maps& m, int nkv) {
  const int64_t blocks = (int64_t)m.n_items * nkv, whole = (int64_t)m.n_tiles * nkv;
  const int sp = m.kv_split_pages;
  const double pages = (double)m.stream_pages / m.n_single;
  if (m.n_parts == m.n_tiles) {          // no request is cut
    if (blocks <= 512) return 1;         // 0.77 / 0.82 (one list of one request 1.1)
    // a block's fixed chain (tables, first stages) outweighs few pages: 4 pages 1.04 - 1.29, 22 pages 1.02 - 1.07 (at 1024 blocks 0.89)
    if (pages < 8 || (pages < 24 && blocks > 1024)) return 0;
    // equal ones in one round of the one kernel 1.04 - 1.06; else up to 1024 blocks 0.90 / 1.02, 1280 0.89 / 0.93, 1536 0.96 / 0.98, 2560
    // 0.97 / 0.98; 1792, 2048 and from 3072 on 1.00 - 1.04
    if (blocks <= 1024 && pages > 0.9 * m.max_pages) return 0;
    return blocks <= 1536 || (blocks > 2048 && blocks <= 2560) ? 1 : 0;
  }
  // about the blocks that are left with f splits taken as one
  auto left = [&](int f) { return (blocks + whole * (f - 1) / 2) / f; };
  const bool full = blocks > 900 && blocks <= 1100;      // one full round of the one-wavefront kernel
  int fold = 1;                          // the fold that leaves no request cut, i.e. no sums to merge
  while (fold * sp < m.max_pages && 2 * fold * sp <= 256) fold *= 2;
  // up to 40 pages from 160 requests x heads on 0.84 - 0.93 (against a full round 1.34), up to 64 from 384 on 0.71 - 0.92, up to 128 by
  // one fold from 768 on 0.92 / 1.00; fewer or longer ones leave CUs idle (up to 64 pages, 128 - 256 of them up to 1.5)
  if (fold * sp >= m.max_pages) {
    if ((m.max_pages <= 64 && whole >= 384) || (fold == 2 && m.max_pages <= 128 && whole >= 768)) return fold;
    if (m.max_pages <= 40 && whole >= 160 && blocks > 512) return full ? 0 : fold;
  }
  if (sp > 128) return blocks <= 3072 ? 1 : 0;        // 0.68 - 1.00; above 1.00 - 1.03
  // Fine cuts of many blocks (asked for; the default cut leaves 1024 to 2048, or as few as pieces of 8 pages make): down to that first.
  int f = 1;
  while (2 * f * sp <= 8 || (2 * f * sp <= 256 && left(f) >= 2048)) f *= 2;
  const int64_t n = left(f);
  const int p = f * sp;                  // pages of a piece
  if (n <= 512 && p >= 12) return f;
  if (p >= 24) {
    // 1100 - 1700 blocks 0.89 - 0.97; around one full round, or nearly two, 1.00 - 1.06 - there pieces of 32 in pairs 0.95
    if (n > 1700) return p < 64 ? 2 * f : f > 1 ? f : 0;
    return n > 1100 || f > 1 ? f : 0;
  }
  if (p >= 12) {
    // by fours where these are 448 to 540 0.90 - 0.94, by pairs from 620 on 0.90 - 0.97; else 0.96 - 1.27
    if (left(4 * f) >= 448 && left(4 * f) <= 540) return 4 * f;
    return left(2 * f) >= 620 ? 2 * f : f > 1 ? f : 0;
  }
  // pieces of 8 pages.  One round of blocks: as they are 0.76 - 0.93 where a request has up to eight of them, else by pairs 0.65 - 0.87 (as they
  // are 0.80 - 0.99).
  if (n <= 512) return m.max_pages <= 8 * p ? f : 2 * f;
  // A request of twenty or more: the merge of their sums is what takes the time, by fours 0.58 - 0.90.
  if (m.max_pages >= 20 * p) return 4 * f;
  if (left(4 * f) >= 320) return 4 * f;                    // 0.73 - 0.88 / 1.03
  return left(2 * f) <= 352 ? 2 * f : f > 1 ? f : 0;       // 0.89 - 1.00; one or two hundred pairs more 0.94 - 1.01 / 1.24
}

// Lists with chunks.  (Against what was done before them - above - 0.78 on average.)
inline int plan_mixed(const flexco_maps& m, int nkv) {
  const int64_t blocks = (int64_t)m.n_items * nkv;
  const int sp = m.kv_split_pages;
  // a long stream beside few chunk products, whose wavefronts it outlasts (about 1.5 ns per page and head against 1 us per page of a
  // chunk's): as if alone
  if (4 * (int64_t)m.chunk_tile_pages < m.stream_pages && 0.0015 * m.stream_pages * nkv > 2.0 * std::min(256, m.max_pages))
    return plan_decode(m, nkv);
  // else pieces of 24 pages or more as they are (32 in pairs 1.05 of that, 64 1.05), of 16 in pairs (0.95 of whole) unless the chunks are the
  // work (1.05); of 8 likewise (0.92 and 1.02), by fours where merging a stream of long contexts is the work (0.85 of
  // whole), few of them as they are; finer ones as if cut into 8
  if (sp >= 24) return 1;
  const int64_t stream = m.stream_pages, chunks = m.chunk_tile_pages;
  if (sp >= 12) return 5 * stream < 2 * chunks ? 1 : 2;
  int f = 1;
  while (2 * f * sp <= 8) f *= 2;
  const bool merges = m.max_pages >= 20 * f * sp;
  if (merges && chunks < stream) return 4 * f;
  return blocks <= 300 * f || (!merges && 5 * stream < chunks) ? f : 2 * f;
}

// Rows of chunks keep their key ranges, and the reference point of their exponentials lags its maximum exactly where
// the four-wavefront kernel took them before (no single token, or products that outweigh the stream): the probabilities'
// rounding to bf16 depends on both, and the window's saved rows and gradients with it.
inline AttnPlan plan_attention(const flexco_maps& m, int nkv) {
  const bool lag = m.n_single == 0 || m.chunk_tile_pages >= m.stream_pages;
  if (m.n_single == 0) return {true, 1, lag};
  if (!m.req_tok_off || m.kv_split_pages <= 0 || m.n_items <= 0) return {false, 1, lag};
  int fold = m.n_single == m.n_items ? plan_decode(m, nkv) : plan_mixed(m, nkv);
  if (fold == 0) return {false, 1, lag};
  while (fold > 1 && fold * m.kv_split_pages > 256) fold /= 2;
  return {true, fold, lag};
}

}  // namespace flexco
