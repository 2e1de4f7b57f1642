// C-ABI layer of libflashblock.so: argument validation (host only, no GPU touched), split
// heuristics, workspace carving and kernel dispatch.  Contract: include/flashblock.h.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <string>

#include "../../include/flashblock_prof.h"
#include "fb_kernels.h"

namespace {

thread_local std::string g_last_hip_error;

constexpr long long kFoldKernelMaxRows = 4096;   // largest row count the one-kernel split fold + internal attention is used for
constexpr int kMaxKeyBlocks = 16384;   // LDS-resident per-KV-group block tables in the sparse helpers
constexpr float kLog2e = 1.4426950408889634f;

fb_status hip_fail(hipError_t e) {
  g_last_hip_error = hipGetErrorString(e);
  return FB_ERR_HIP;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

fb_status check_shape(const fb_shape* s) {
  if (s == nullptr) return FB_ERR_NULL;
  if (s->struct_size != sizeof(fb_shape)) return FB_ERR_SHAPE;
  if (s->dtype != FB_F32 && s->dtype != FB_BF16) return FB_ERR_DTYPE;
  if (s->batch < 1 || s->n_q_heads < 1 || s->n_kv_heads < 1 || s->block_len < 1 || s->prefix_len < 0)
    return FB_ERR_SHAPE;
  if (s->n_q_heads % s->n_kv_heads != 0) return FB_ERR_SHAPE;
  if (s->n_q_heads / s->n_kv_heads > 32) return FB_ERR_SHAPE;
  if (!(s->scale >= 0.f) || isinf(s->scale)) return FB_ERR_SHAPE;   // rejects NaN and negatives
  if (s->head_dim < 1) return FB_ERR_SHAPE;
  if (s->head_dim != 64 && s->head_dim != 128) return FB_ERR_UNSUPPORTED;
  if ((long long)s->batch * s->n_q_heads > 65535) return FB_ERR_UNSUPPORTED;   // grid.y of the fp32 mass kernel
  const long long rows = (long long)s->batch * s->n_q_heads * s->block_len;
  if (rows > (1ll << 28)) return FB_ERR_UNSUPPORTED;
  return FB_OK;
}

float eff_scale(const fb_shape* s) { return s->scale > 0.f ? s->scale : 1.0f / sqrtf((float)s->head_dim); }

long long rows_of(const fb_shape* s) { return (long long)s->batch * s->n_q_heads * s->block_len; }

// Scratch memory of fb_external_partial_builtin_ws: the split partials of one call.  One copy per GPU the
// library runs on, held until the process ends.
constexpr size_t kBuiltinWsBytes = (size_t)20 * 1024 * 1024;

// Splits of the fp32 passes: workgroups of f32_row_tile rows, one per CU (their K/V stages take most of the LDS), so as
// many splits as keep the workgroup count within 256 (one round); a split is at least one tile.  256 partials of at most 64
// rows are 8.5 MB: two or more splits and the block-internal set (as much as half of them) always fit the built-in scratch
// array.  per_head: the passes whose workgroups belong to one query head.
int f32_splits(const fb_shape* s, bool per_head) {
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  const long long nrows = per_head ? s->block_len : (long long)(s->n_q_heads / s->n_kv_heads) * s->block_len;
  const long long rt = fb::f32_row_tile(nrows);
  const long long groups = (long long)s->batch * (per_head ? s->n_q_heads : s->n_kv_heads) * ((nrows + rt - 1) / rt);
  long long ns = 256 / groups;
  if (ns > tiles) ns = tiles;
  if (ns > FB_MAX_SPLITS) ns = FB_MAX_SPLITS;
  if (ns < 1) ns = 1;
  return (int)ns;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int auto_splits(const fb_shape* s, int active_heads = 0) {
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  if (s->dtype == FB_BF16 && active_heads > 0 && active_heads < s->n_q_heads) {
    // Per-head refresh with a hint: only the KV groups of flagged heads do work (at most
    // min(Hkv, active) of them per batch element).  8-wavefront workgroups, one per CU; among the two
    // split counts around 256 / groups take the one with the shorter critical path
    // (rounds of 256 workgroups x tiles per split), never fewer than 8 tiles per split.
    const int G = s->n_q_heads / s->n_kv_heads;
    const long long kvg = active_heads < s->n_kv_heads ? active_heads : s->n_kv_heads;
    const long long groups = (long long)s->batch * kvg * ((G * s->block_len + fb::kRowsPerWgBf16 - 1) / fb::kRowsPerWgBf16);
    long long best = 1, best_cost = -1;
    const long long lo = 256 / groups > 1 ? 256 / groups : 1;
    for (long long ns = lo; ns <= lo + 1; ++ns) {
      if (ns > 1 && tiles < 8 * ns) continue;
      if (ns > FB_MAX_SPLITS) continue;
      const long long cost = ((groups * ns + 255) / 256) * ((tiles + ns - 1) / ns);
      if (best_cost < 0 || cost < best_cost) { best = ns; best_cost = cost; }
    }
    return (int)best;
  }
  if (s->dtype == FB_BF16) {
    // Every split costs a 128-row fp32 partial written and read back, so splits are as few as
    // still fill the GPU.
    const int G = s->n_q_heads / s->n_kv_heads;
    const long long groups =
        (long long)s->batch * s->n_kv_heads * ((G * s->block_len + fb::kRowsPerWgBf16 - 1) / fb::kRowsPerWgBf16);
    // Long prefixes: one 8-wavefront workgroup per CU (256 CUs), each streaming >= 8 tiles.
    // Shorter ones: 4-wavefront workgroups, up to two per CU, never fewer than 4 tiles per split.
    const long long per_cu = (256 + groups - 1) / groups;
    long long ns;
    if (tiles >= 8 * per_cu) {
      ns = per_cu;
    } else {
      ns = tiles / 4;
      const long long hi = (512 + groups - 1) / groups;
      if (ns > hi) ns = hi;
    }
    if (ns > FB_MAX_SPLITS) ns = FB_MAX_SPLITS;
    if (ns < 1) ns = 1;
    return (int)ns;
  }
  return f32_splits(s, false);
}

// Pieces that the streaming kernel cuts the prefix of up to 128 rows per KV head into, where the nseg splits of auto_splits, one
// more than fit 256 workgroups, would leave a second round with a few of them: one round, and the splits stay as the reference
// segments of the walk (fb_stream_bf16.hip), so that results do not change with the cut.  (A refresh step, 11 splits -> 10 pieces, batch 3,
// 8 heads of 9 rows, head_dim 128 / 64, 8 / 12 / 24 tiles a split 30.1 / 38.1 / 73.2 -> 24.8 / 29.1 / 49.2 us and 22.7 / 27.9 / 43.7 -> 20.8 /
// 24.1 / 33.7; 3 -> 2 pieces, batch 15, 50 rows of 2 heads a group, 8 / 16 tiles 44.1 / 68.3 -> 36.9 / 57.7; never slower.)
int dense_parts(const fb_shape* s, int nseg) {
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  const long long groups = (long long)s->batch * s->n_kv_heads;
  const long long nrows = (long long)(s->n_q_heads / s->n_kv_heads) * s->block_len;
  if (s->dtype != FB_BF16 || nrows > fb::kRowsPerWgBf16 || tiles < 8 * nseg || groups * nseg <= 256 || 256 / groups < 2) return nseg;
  return (int)(256 / groups);
}

// Splits of the plain dense external pass.  KV groups above 128 rows run 256-row workgroups, one per
// CU: as many splits as keep the workgroup count within the 256 CUs (one round), each with at least 8 tiles.
int dense_splits(const fb_shape* s) {
  const int G = s->n_q_heads / s->n_kv_heads;
  const long long nrows = (long long)G * s->block_len;
  if (s->dtype != FB_BF16 || !fb::dense_row_pairs((int)std::min<long long>(nrows, 1 << 30), s->head_dim)) return dense_parts(s, auto_splits(s));
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  const long long groups = (long long)s->batch * s->n_kv_heads * ((nrows + 2 * fb::kRowsPerWgBf16 - 1) / (2 * fb::kRowsPerWgBf16));
  long long ns = 256 / groups;
  if (ns > tiles / 8) ns = tiles / 8;
  if (ns > FB_MAX_SPLITS) ns = FB_MAX_SPLITS;
  if (ns < 1) ns = 1;
  return (int)ns;
}

// Reference segments of the plain dense pass.
int dense_segments(const fb_shape* s) {
  const long long nrows = (long long)(s->n_q_heads / s->n_kv_heads) * s->block_len;
  return s->dtype == FB_BF16 && nrows <= fb::kRowsPerWgBf16 ? auto_splits(s) : dense_splits(s);
}

// Splits of the per-head refresh.  fp32: one query head per workgroup.
// bf16 with a hint: auto_splits, whose two candidates around 256 / groups both drop out where the stream is too short for 8
// tiles per split of them, which leaves 1.  There, splits of 8 tiles, up to 7 (from 8 on the combine takes a workgroup for
// every row, flagged or not: 1 of 10 heads of 1500 rows, head_dim 64, 6000 keys, 34.4 us with 11 and 20.1 with 7), and no
// fewer than without a hint; from 16 tiles on, below which the combine costs what the splits save (15 of 16 heads of 319
// rows, batch 2, 9 tiles, 18.5 us with 1 and 19.9 with 2).  One split left a handful of CUs with the whole stream (hinted with 1, unhinted, now: 1 of 8
// heads of 1000 rows, 3000 keys, 54.1, 23.1, 21.9 us; 1 of 12, 16000 keys, 210, 93.8, 48.5; 2 of 32 / 8 heads of 64 rows, 8000
// keys, 84.2, 17.1, 16.6).
int heads_splits(const fb_shape* s, int active_heads) {
  if (s->dtype != FB_BF16) return f32_splits(s, true);
  const int ns = auto_splits(s, active_heads), tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  const long long groups = (long long)s->batch * std::min(active_heads, s->n_kv_heads) *
                           (((long long)(s->n_q_heads / s->n_kv_heads) * s->block_len + fb::kRowsPerWgBf16 - 1) / fb::kRowsPerWgBf16);
  if (active_heads <= 0 || active_heads >= s->n_q_heads || tiles < 16 || tiles >= 8 * (256 / groups)) return ns;
  return std::max({ns, auto_splits(s), std::min(tiles / 8, 7)});
}

// Split counts of the sparse passes (bf16): one workgroup per CU in both modes - 8 wavefronts in
// the reuse pass, 4 wavefronts with two accumulator sets in the refresh pass.
int sparse_splits(const fb_shape* s, bool refresh) {
  (void)refresh;
  if (s->dtype != FB_BF16) return f32_splits(s, true);
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  const int G = s->n_q_heads / s->n_kv_heads;
  const long long groups =
      (long long)s->batch * s->n_kv_heads * ((G * s->block_len + fb::kRowsPerWgBf16 - 1) / fb::kRowsPerWgBf16);
  long long ns = (256 + groups - 1) / groups;
  const long long cap = tiles / 4;
  if (ns > cap) ns = cap;
  if (ns > FB_MAX_SPLITS) ns = FB_MAX_SPLITS;
  if (ns < 1) ns = 1;
  return (int)ns;
}

// Paged pass: sequences differ in length, so equal split counts give unequal workgroups.  Aim at
// ~2 eight-wavefront workgroups per CU (dispatched longest sequence first, the hardware dispatcher
// evens them out), each with at least 16 tiles on the longest sequence.
int paged_splits(const fb_shape* s) {
  if (s->dtype != FB_BF16) return auto_splits(s);
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  const int G = s->n_q_heads / s->n_kv_heads;
  const long long groups =
      (long long)s->batch * s->n_kv_heads * ((G * s->block_len + fb::kRowsPerWgBf16 - 1) / fb::kRowsPerWgBf16);
  long long ns = (512 + groups - 1) / groups;
  const long long cap = tiles / 16;
  if (ns > cap) ns = cap;
  if (ns > FB_MAX_SPLITS) ns = FB_MAX_SPLITS;
  if (ns < 1) ns = 1;
  return (int)ns;
}

struct WsLayout {
  size_t o[2], m[2], l[2], mask, ulist, umask, ucnt, order, total;
};

WsLayout ws_layout(const fb_shape* s, int nsplit, int nsets, int nblk, int nsplit2 = -1) {
  WsLayout w;
  const size_t rows = (size_t)rows_of(s);
  size_t off = 0;
  for (int i = 0; i < 2; ++i) {
    const size_t n = (i < nsets) ? (size_t)((i == 1 && nsplit2 >= 0) ? nsplit2 : nsplit) * rows : 0;
    w.o[i] = off; off = align256(off + n * s->head_dim * sizeof(float));
    w.m[i] = off; off = align256(off + n * sizeof(float));
    w.l[i] = off; off = align256(off + n * sizeof(float));
  }
  const size_t nb = (size_t)s->batch * s->n_kv_heads * nblk;
  w.mask = off;  off = align256(off + nb * sizeof(uint32_t));
  w.ulist = off; off = align256(off + nb * sizeof(int32_t));
  w.umask = off; off = align256(off + nb * sizeof(uint32_t));
  w.ucnt = off;  off = align256(off + (nblk > 0 ? (size_t)s->batch * s->n_kv_heads * sizeof(int32_t) : 0));
  w.order = off; off = align256(off + (size_t)s->batch * sizeof(int32_t));   // paged pass: sequences by length
  w.total = off;
  return w;
}

// Per-head refresh over KV groups of more than 128 rows (bf16) with a hint: 256-row workgroups, each of the ns
// splits as two, its even and its odd tiles, so that the flagged groups fill the CUs that 128-row workgroups with two
// tile streams each would.  The split partials are stored densely by rank among the flagged KV groups (cap groups per batch
// element; groups beyond it are streamed unsplit).  ns = 0: the hint says nothing, or the shape is another kernel's.
struct HeadsPlan {
  int ns, cap;
  size_t o, m, l, total;      // workspace offsets
};

HeadsPlan heads_plan(const fb_shape* s, int active_heads, int ns) {
  HeadsPlan h = {0, 0, 0, 0, 0, 0};
  const long long nrows = (long long)(s->n_q_heads / s->n_kv_heads) * s->block_len;
  if (s->dtype != FB_BF16 || active_heads <= 0 || active_heads >= s->n_q_heads) return h;
  if (!fb::dense_row_pairs((int)std::min<long long>(nrows, 1 << 30), s->head_dim)) return h;
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  // Twice the split partials have to be earned: from 12 tiles per stream on where the split count is 2 or more, from 24 unsplit, and from 40
  // where the 128-row workgroups fill half the chip unsplit and would write the final partial themselves.  Us there and here: 9
  // heads of 1140 rows, 5 flagged, 207 tiles, 5 splits 58.6 and 55.6; 11 of 3014, 5 flagged, 74 tiles, 2 splits 57.9 and 54.9; 8 of
  // 3828, 7 flagged, 116 tiles 126 and 108; 8 of 4392, 4 flagged, 113 tiles 119 and 96; 9 of 4226, 7 flagged, 50 tiles 61.6 and 66.7.
  // And not where twice the splits of half the row tiles spill into one round of workgroups more (tiles of 256 rows; a start and an
  // end 5 of them, 4 there): of 5 splits and more always (4 of 1093, 3 flagged, 550 tiles, 9 splits 84 and 109; 5 of 3178, 2 flagged, 374
  // tiles, 5 splits 98 and 131), of fewer on short streams (long ones gain all the same: 7 of 2608, 331 tiles, 3 splits 178 and 150).  With
  // several heads to a KV group the row tiles hold the flagged heads' rows only, but workgroups are launched for all, and a grid of more
  // than a round costs a second one all the same: on short streams not then (12 groups of 2 x 407 rows, 22 flagged, 73 tiles, 3 splits 43.8 and
  // 69.1; 4 of 2 x 430, 2 flagged, 467 tiles, 18 splits 46.3 and 69.2; of 28 random such calls 12 lost, to 1.57, 14 won, to 0.63).
  const long long kvg = (long long)s->batch * std::min(active_heads, s->n_kv_heads);
  const long long wgs = kvg * ((nrows + fb::kRowsPerWgBf16 - 1) / fb::kRowsPerWgBf16), wgs256 = kvg * ((nrows + 2 * fb::kRowsPerWgBf16 - 1) / (2 * fb::kRowsPerWgBf16));
  const bool spills = (wgs256 * 2 * ns + 255) / 256 * (tiles / ns / 2 + 5) > (wgs * ns + 255) / 256 * (tiles / ns + 4);
  const bool is_long = tiles >= 48 * ns && !(ns == 1 && wgs >= 128 && tiles < 128);
  if (tiles < (ns > 1 ? 24 * ns : wgs >= 128 ? 80 : 48) || (spills && ((ns >= 5 && s->n_q_heads == s->n_kv_heads) || !is_long)) || 2 * ns > FB_MAX_SPLITS) return h;
  if (nrows * s->head_dim * 2 >= (1ll << 32)) return h;      // 32-bit query offsets between the heads of a group
  h.ns = 2 * ns;
  h.cap = std::min(active_heads, s->n_kv_heads);
  const size_t n = (size_t)h.ns * s->batch * h.cap * nrows;
  h.m = align256(n * s->head_dim * sizeof(float));
  h.l = h.m + align256(n * sizeof(float));
  h.total = h.l + align256(n * sizeof(float));
  return h;
}

// The split count that callers size the workspace of the per-head refresh with: that of the pass, or more where the plan's
// 2 ns cap group partials would not fit the (ns + 1) Hkv of it (7 of 8 heads of 2080 rows against 37440 keys: 28 and 24,
// 343 us by the register-staged kernel and 302 by the plan).  The route of a caller who follows the header depends on
// shape and hint alone.
int heads_ws_splits(const fb_shape* s, int active_heads) {
  int n = heads_splits(s, active_heads);
  const HeadsPlan h = heads_plan(s, active_heads, n);
  while (h.ns > 0 && ws_layout(s, n, 2, 0, 1).total < h.total) ++n;
  return n;
}

// Refresh step of more than 128 rows per KV head in ns >= 2 splits (bf16) by the row-pair kernel: every split as two streams, the even
// and the odd tiles, which are the tile groups of the register-staged pass, so that weights round alike; the block's own keys as two more
// (from 640 tokens on), or by the fold kernel or the internal pass (one tile).  0: not this route.  By tiles per split, against the
// register-staged pass and the combine (us a refresh step, head_dim 128): blocks of many tokens always (5 heads of 4300 rows, 3 splits, 12 /
// 24 / 60 tiles 201 / 257 / 351 and 104 / 145 / 249; 12 heads of 1023, 5 splits, 75 / 108 / 156 and 57 / 77 / 112; head_dim 64, 4 heads of
// 2728 rows, 5 splits, 65 / 86 / 115 and 54 / 63 / 87).  One tile: twice the partials have to be earned where the fold kernel reads them
// (up to 4096 rows: batch 3, 168 rows of 8 heads, 6 splits, 24 / 36 / 60 tiles 72 / 104 / 159 and 77 / 96 / 131; head_dim 64 48 / 64 / 97
// and 51 / 62 / 87), not where combine and internal pass do (batch 7, 152 rows, 3 splits, 12 / 24 tiles 50 / 78 and 47 / 66;
// batch 3, 212 rows, 6 splits, 14 tiles, blocks of 53, 55 and 63), and one tile never where the streams' 256-row workgroups are a
// round more than the 128-row ones (an odd number of those to a head: 80 heads of 344 rows, 2 splits of 15 tiles, head_dim 64, 480 and 640 workgroups,
// 44.1 and 55.8; 84 of 360, 130 tiles 209 and 240; of 47 random such calls 37 lost, to 1.27), unless at head_dim 128 the streams are long
// (540 rows, 26 tiles 1.07, 368 rows, 65 tiles 1.01, 344 rows, 143 tiles 0.93 times).  One round of combine and internal pass at head_dim 64:
// from 32 tiles on (16 heads of 992 rows, 2 splits of 14 26.2 and 31.9; 928 rows, 18 1.15, 228 rows, 24 1.04, 420 rows, 35 0.98 times).
int step_streams(const fb_shape* s, int ns) {
  const long long nrows = (long long)(s->n_q_heads / s->n_kv_heads) * s->block_len;
  const int tiles = (s->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
  if (s->dtype != FB_BF16 || ns < 2 || nrows <= fb::kRowsPerWgBf16 || 2 * ns > FB_MAX_SPLITS) return 0;
  if (s->block_len > fb::kKeyTile && s->block_len < 640) return 0;
  const long long heads = (long long)s->batch * s->n_kv_heads, wgs = heads * ((nrows + 127) / 128) * ns, rows256 = (nrows + 255) / 256;
  if (s->block_len <= fb::kKeyTile) {
    if ((heads * rows256 * 2 * ns + 255) / 256 > (wgs + 255) / 256 && !(s->head_dim == 128 && tiles >= 80 * ns)) return 0;
    int least = 6 + 4 * ns;
    // The fold kernel's line is later where one round there is a few heads of many rows each (8 splits, head_dim 128, means of random calls at
    // 32 / 40 / 48 / 56 / 64 tiles: 16 heads of up to 256 rows 1.00 / 0.95 / 0.92 / 0.90 / 0.84 times, 8 of up to 512 1.10 / 1.02 / 0.99 / 0.95 /
    // 0.91, 4 of up to 1024 1.17 / 1.12 / 1.08 / 1.04 / 0.96).
    if (rows_of(s) <= kFoldKernelMaxRows) least = s->head_dim == 64 || wgs > 256 || ns > 8 || nrows <= 384 ? 36 : nrows <= 768 ? 48 : 64;
    else if (s->head_dim == 64 && wgs <= 256) least = std::max(32, least);
    return tiles >= least * ns ? 2 * ns : 0;
  }
  if (tiles < 10 * ns) return 0;
  // Both ways by their rounds of 256 workgroups, in tiles of 256 rows: a tile of 128 rows takes the register-staged kernel as long as one of 256
  // the row-pair kernel, a start and an end 4 and 5 tiles; the last split's workgroup runs the block too, here the block's streams
  // fill what the prefix's leave; and ns + 1 more partials are written and read.  (4 heads of 2026 rows, 11933 keys, one full round
  // there and a second one of the block's streams here: 75 us there, 80 here.)
  const int btiles = (s->block_len + fb::kKeyTile - 1) / fb::kKeyTile, per = tiles / ns;
  const long long there = (wgs + 255) / 256 * (std::max(per, per - std::min(2 + btiles, per / 2) + btiles) + 4);
  const long long a = per / 2 + 5, b = btiles / 2 + 5, na = heads * rows256 * 2 * ns, nb = heads * rows256 * 2, busy = na % 256;
  const long long fit = busy ? (256 - busy) * (a / b) : 0;
  const long long here = (na + 255) / 256 * a + (std::max(nb - fit, 0ll) + 255) / 256 * b + heads * nrows * (ns + 1) / (s->head_dim == 128 ? 6700 : 13400) ;
  if (here + here / 5 >= there) return 0;
  if (s->head_dim == 64) {
    // What the model leaves out there, with both sides measured (us, there and here).  Few heads in many splits, whose second round there
    // is a few workgroups: one head of 640 rows, 52 splits of 10 / 14 / 20 tiles 28.9 / 35.1 / 42.8 and 31.5 / 36.3 / 41.4, two of 640, 26
    // splits 27.9 / 34.6 / 42.1 and 30.7 / 34.8 / 40.2; from 22 splits down never slower here.
    if (ns > 22 && per < 16) return 0;
    // Just one round there, of fewer than 8 heads: only where the block is long beside the splits, or the splits long beside the block.  1
    // head of 1024 rows, 64 / 80 / 96 / 128 tiles a split 55.3 / 66.2 / 78.0 / 99.3 and 59.8 / 69.3 / 76.9 / 95.0; 4 of 1024, 64 / 80 59.8 / 71.2 and
    // 59.9 / 68.4; 1 of 2048, 10 / 16 / 96 / 128 / 200 38.8 / 40.8 / 79.5 / 102 / 152 and 41.6 / 44.1 / 88.2 / 105 / 142; 2 of 4096 (two query heads of
    // 2048), 160 126 and 120; 2 of 4096, 16 / 32 / 96 62.8 / 69.5 / 96.5 and 61.4 / 70.0 / 105; 1 of 8192, 64 / 128 / 200 127 / 154 / 190 and 120 / 157 /
    // 198.  (8 heads of 2048, 80 tiles: 79.7 and 70.1.)
    if (wgs <= 256 && heads < 8 && per * 128 > btiles * btiles && per < 5 * btiles) return 0;
  }
  return 2 * ns;
}

fb_status check_key_block(const fb_shape* s, int32_t key_block, int32_t topk, int* nblk) {
  if (key_block <= 0 || topk < 0) return FB_ERR_SHAPE;
  if (key_block % fb::kKeyTile != 0) return FB_ERR_UNSUPPORTED;
  const long long nb = ((long long)s->prefix_len + key_block - 1) / key_block;
  if (nb > kMaxKeyBlocks) return FB_ERR_UNSUPPORTED;
  *nblk = (int)nb;
  return FB_OK;
}

fb::PassParams base_pass(const fb_shape* s, const void* q, const void* k, const void* v, int nkeys, int nsplit) {
  fb::PassParams p;
  memset(&p, 0, sizeof(p));
  p.q = q; p.k = k; p.v = v;
  p.B = s->batch; p.Hq = s->n_q_heads; p.Hkv = s->n_kv_heads; p.G = s->n_q_heads / s->n_kv_heads;
  p.Bq = s->block_len; p.nkeys = nkeys; p.nsplit = nsplit;
  p.scale_log2 = eff_scale(s) * kLog2e;
  p.key_block = fb::kKeyTile;
  return p;
}

// Split partials of the dense passes, and one block-internal partial for fb_refresh_step.  The split count of fb_external_splits sizes for
// the library's own dense passes too, which ask for a partial per reference segment (as many as there were splits before there were pieces).
size_t pass_workspace(const fb_shape* s, int n_splits) {
  int ns = n_splits > 0 ? n_splits : std::max({auto_splits(s), dense_splits(s), heads_splits(s, 0)});
  if (n_splits > 0 && n_splits == dense_splits(s)) ns = std::max(ns, dense_segments(s));
  return ws_layout(s, ns, 2, 0, 1).total;
}

hipError_t launch_attn(const fb_shape* s, const fb::PassParams& p, fb::PassMode mode, hipStream_t st) {
  return s->dtype == FB_BF16 ? fb::launch_attn_bf16(p, s->head_dim, mode, st)
                             : fb::launch_attn_f32(p, s->head_dim, mode, st);
}

// Attention launch with optional measurement events.  bf16 kernels take them as their own start / stop events
// (the kernel's dispatch timestamps); where the launch does not (fp32 kernel), they are recorded around it.
hipError_t timed_attn(const fb_shape* s, const fb::PassParams& p, fb::PassMode mode, hipStream_t st, void* ev_begin,
                      void* ev_end) {
  hipError_t e = hipSuccess;
  const bool in_launch = s->dtype == FB_BF16 && (ev_begin || ev_end);
  if (in_launch) {
    fb::tl_kernel_events.start = (hipEvent_t)ev_begin;
    fb::tl_kernel_events.stop = (hipEvent_t)ev_end;
  } else if (ev_begin && (e = hipEventRecord((hipEvent_t)ev_begin, st)) != hipSuccess) {
    return e;
  }
  e = launch_attn(s, p, mode, st);
  fb::tl_kernel_events = fb::KernelEvents{};      // never left behind for an unrelated launch
  if (e != hipSuccess) return e;
  if (!in_launch && ev_end) e = hipEventRecord((hipEvent_t)ev_end, st);
  return e;
}

}  // namespace

extern "C" {

int fb_version(void) { return FB_VERSION; }

const char* fb_status_string(int status) {
  switch (status) {
    case FB_OK: return "FB_OK";
    case FB_ERR_NULL: return "FB_ERR_NULL: required pointer is NULL";
    case FB_ERR_SHAPE: return "FB_ERR_SHAPE: dimension, head grouping, scale or mode out of range";
    case FB_ERR_DTYPE: return "FB_ERR_DTYPE: dtype is not FB_F32 / FB_BF16";
    case FB_ERR_ALIGN: return "FB_ERR_ALIGN: tensor pointer not 16-byte aligned";
    case FB_ERR_WORKSPACE: return "FB_ERR_WORKSPACE: workspace NULL or too small";
    case FB_ERR_UNSUPPORTED: return "FB_ERR_UNSUPPORTED: request outside what the kernels cover";
    case FB_ERR_HIP: return "FB_ERR_HIP: HIP launch failed";
    default: return "unknown fb_status";
  }
}

const char* fb_last_hip_error(void) { return g_last_hip_error.c_str(); }

fb_status fb_check_shape(const fb_shape* shape) { return check_shape(shape); }

int32_t fb_external_splits(const fb_shape* shape) {
  if (check_shape(shape) != FB_OK) return 0;
  return dense_splits(shape);
}

const char* fb_external_kernel_name(const fb_shape* shape) {
  thread_local char name[96];
  name[0] = 0;
  if (check_shape(shape) != FB_OK) return name;
  if (shape->dtype != FB_BF16) {
    const bool few = dense_splits(shape) == 1 &&
                     fb::f32_few_keys(rows_of(shape), (long long)(shape->n_q_heads / shape->n_kv_heads) * shape->block_len, shape->prefix_len);
    snprintf(name, sizeof(name), "attn_f32_%skernel<%d, %d>", few ? "few_" : "", shape->head_dim, (int)fb::kPassDense);
    return name;
  }
  fb::PassParams p = base_pass(shape, nullptr, nullptr, nullptr, shape->prefix_len, dense_splits(shape));
  p.nseg = dense_segments(shape);
  fb::attn_bf16_dense_name(p, shape->head_dim, name, sizeof(name));
  return name;
}

int32_t fb_paged_splits(const fb_shape* shape) {
  if (check_shape(shape) != FB_OK) return 0;
  return paged_splits(shape);
}

size_t fb_workspace_bytes(const fb_shape* shape, int32_t key_block, int32_t topk, int32_t n_splits) {
  if (check_shape(shape) != FB_OK) return 0;
  if (n_splits < 0 || n_splits > FB_MAX_SPLITS) return 0;
  size_t t = pass_workspace(shape, n_splits);
  if (n_splits == 0) {
    if (const int streams = step_streams(shape, auto_splits(shape))) t = std::max(t, ws_layout(shape, streams, 2, 0, 2).total);
  }
  if (key_block != 0) {
    int nblk = 0;
    if (check_key_block(shape, key_block, topk, &nblk) != FB_OK) return 0;
    const size_t ts = ws_layout(shape, sparse_splits(shape, false), 2, nblk).total;
    if (ts > t) t = ts;
  }
  return t > 0 ? t : 256;
}

}  // extern "C"

namespace {

fb_status external_partial_impl(const fb_shape* shape, const void* q, const void* k_prefix,
                                const void* v_prefix, const fb_paged_kv* paged, const uint8_t* head_mask,
                                bool use_head_mask, int n_active_heads, float* o_part, float* m_part, float* lse_part,
                                int32_t n_splits, void* workspace, size_t workspace_bytes,
                                void* ev_begin, void* ev_attn_end, void* ev_end, void* hip_stream,
                                fb::CombineParams* fold_out = nullptr) {
  // fold_out: the caller folds the split partials itself (with a kernel that does more than the plain combine); it
  // gets the combine's parameters instead of the combine launch.  Left with nsplit = 0 when there was one split
  // and the attention kernel wrote the final partial itself.
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  if (!q || !o_part || !m_part || !lse_part) return FB_ERR_NULL;
  if (use_head_mask && !head_mask) return FB_ERR_NULL;
  if (paged) {
    if (paged->struct_size != sizeof(fb_paged_kv)) return FB_ERR_SHAPE;
    if (!paged->block_table || !paged->prefix_lens) return FB_ERR_NULL;
    if (paged->num_pages <= 0 || paged->page_size <= 0 || paged->max_pages <= 0) return FB_ERR_SHAPE;
    if (paged->page_size % fb::kKeyTile != 0) return FB_ERR_UNSUPPORTED;
    if ((long long)paged->max_pages * paged->page_size < shape->prefix_len) return FB_ERR_SHAPE;
    k_prefix = paged->k_pool;
    v_prefix = paged->v_pool;
  }
  if (shape->prefix_len > 0 && (!k_prefix || !v_prefix)) return FB_ERR_NULL;
  if (n_splits < 0 || n_splits > FB_MAX_SPLITS) return FB_ERR_SHAPE;
  if (!aligned16(q) || !aligned16(k_prefix) || !aligned16(v_prefix) || !aligned16(o_part) ||
      !aligned16(m_part) || !aligned16(lse_part) || !aligned16(workspace))
    return FB_ERR_ALIGN;
  if (n_active_heads < 0) return FB_ERR_SHAPE;
  int ns = n_splits > 0 ? n_splits
                        : (paged ? paged_splits(shape)
                                 : use_head_mask ? heads_splits(shape, n_active_heads) : dense_splits(shape));
  // per-head refresh, bf16: a buffer below the documented size that holds the splits of auto_splits is taken with those
  if (use_head_mask && shape->dtype == FB_BF16 && workspace_bytes < ws_layout(shape, ns, 1, 0).total)
    ns = auto_splits(shape, n_active_heads);
  const int nseg = (n_splits > 0 || paged || use_head_mask) ? ns : dense_segments(shape);
  if (!workspace || workspace_bytes < ws_layout(shape, nseg, 1, 0).total) return FB_ERR_WORKSPACE;
  const WsLayout w = ws_layout(shape, ns, 1, 0);

  hipStream_t stream = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;
  fb::PassParams p = base_pass(shape, q, k_prefix, v_prefix, shape->prefix_len, ns);
  p.ws_o = (float*)(ws + w.o[0]); p.ws_m = (float*)(ws + w.m[0]); p.ws_l = (float*)(ws + w.l[0]);
  p.nseg = nseg;
  p.head_on = use_head_mask ? head_mask : nullptr;
  fb::PassMode mode = use_head_mask ? fb::kPassDenseHeads : fb::kPassDense;
  if (use_head_mask) {
    const HeadsPlan h = heads_plan(shape, n_active_heads, ns);
    if (h.ns > 0 && h.total <= workspace_bytes) {        // (always, unless the buffer is below fb_workspace_bytes of heads_ws_splits)
      ns = p.nsplit = h.ns;
      p.heads_cap = h.cap;
      p.ws_o = (float*)ws; p.ws_m = (float*)(ws + h.m); p.ws_l = (float*)(ws + h.l);
      p.o_final = o_part; p.m_final = m_part; p.l_final = lse_part;
    }
  }
  if (paged) {
    mode = fb::kPassDensePaged;
    p.block_table = paged->block_table; p.prefix_lens = paged->prefix_lens;
    p.page_size = paged->page_size; p.max_pages = paged->max_pages; p.num_pages = paged->num_pages;
    if (shape->batch > 1 && shape->batch <= 128 && shape->dtype == FB_BF16) {
      p.order_inline = 1;       // the bf16 kernel ranks up to 128 sequences in its prologue
    } else if (shape->batch > 1) {
      p.seq_order = (int32_t*)(ws + w.order);
      hipError_t eo = fb::launch_seq_order(paged->prefix_lens, (int32_t*)(ws + w.order), shape->batch, stream);
      if (eo != hipSuccess) return hip_fail(eo);
    }
  }
  if (ns == 1) {   // the attention kernel writes the final partial itself
    p.direct = 1;
    p.ws_o = o_part; p.ws_m = m_part; p.ws_l = lse_part;
  }
  hipError_t e = timed_attn(shape, p, mode, stream, ev_begin, ev_attn_end);
  if (e != hipSuccess) return hip_fail(e);

  if (fold_out) memset(fold_out, 0, sizeof(*fold_out));
  if (!p.direct) {
    fb::CombineParams c;
    memset(&c, 0, sizeof(c));
    c.rows = (int)rows_of(shape); c.D = shape->head_dim; c.nsplit = ns;
    c.ws_o = p.ws_o; c.ws_m = p.ws_m; c.ws_l = p.ws_l;
    c.o = o_part; c.m = m_part; c.lse = lse_part;
    c.head_on = p.head_on; c.Bq = shape->block_len;
    c.heads_cap = p.heads_cap;
    c.Hq = shape->n_q_heads; c.Hkv = shape->n_kv_heads; c.G = shape->n_q_heads / shape->n_kv_heads;
    if (fold_out) {
      *fold_out = c;
    } else {
      e = fb::launch_combine(c, stream);
      if (e != hipSuccess) return hip_fail(e);
    }
  }
  if (ev_end && (e = hipEventRecord((hipEvent_t)ev_end, stream)) != hipSuccess) return hip_fail(e);
  return FB_OK;
}

}  // namespace

extern "C" {

fb_status fb_external_partial_prof(const fb_shape* shape, const void* q, const void* k_prefix,
                                   const void* v_prefix, float* o_part, float* m_part, float* lse_part,
                                   int32_t n_splits, void* workspace, size_t workspace_bytes,
                                   void* ev_begin, void* ev_attn_end, void* ev_end, void* hip_stream) {
  return external_partial_impl(shape, q, k_prefix, v_prefix, nullptr, nullptr, false, 0, o_part, m_part, lse_part, n_splits,
                               workspace, workspace_bytes, ev_begin, ev_attn_end, ev_end, hip_stream);
}

int32_t fb_external_heads_splits(const fb_shape* shape, int32_t n_active_heads) {
  if (check_shape(shape) != FB_OK || n_active_heads < 0) return 0;
  return heads_ws_splits(shape, n_active_heads);
}

fb_status fb_external_partial_heads(const fb_shape* shape, const void* q, const void* k_prefix,
                                    const void* v_prefix, const uint8_t* head_mask, int32_t n_active_heads,
                                    float* o_part, float* m_part, float* lse_part, void* workspace,
                                    size_t workspace_bytes, void* hip_stream) {
  return external_partial_impl(shape, q, k_prefix, v_prefix, nullptr, head_mask, true, n_active_heads, o_part, m_part, lse_part, 0,
                               workspace, workspace_bytes, nullptr, nullptr, nullptr, hip_stream);
}

fb_status fb_external_partial_paged(const fb_shape* shape, const void* q, const fb_paged_kv* kv, float* o_part,
                                    float* m_part, float* lse_part, int32_t n_splits, void* workspace,
                                    size_t workspace_bytes, void* hip_stream) {
  if (!kv) return FB_ERR_NULL;
  return external_partial_impl(shape, q, nullptr, nullptr, kv, nullptr, false, 0, o_part, m_part, lse_part, n_splits,
                               workspace, workspace_bytes, nullptr, nullptr, nullptr, hip_stream);
}

fb_status fb_external_partial_ex(const fb_shape* shape, const void* q, const void* k_prefix,
                                 const void* v_prefix, float* o_part, float* m_part, float* lse_part,
                                 int32_t n_splits, void* workspace, size_t workspace_bytes,
                                 void* hip_stream) {
  return fb_external_partial_prof(shape, q, k_prefix, v_prefix, o_part, m_part, lse_part, n_splits,
                                  workspace, workspace_bytes, nullptr, nullptr, nullptr, hip_stream);
}

fb_status fb_external_partial(const fb_shape* shape, const void* q, const void* k_prefix,
                              const void* v_prefix, float* o_part, float* m_part, float* lse_part,
                              void* workspace, size_t workspace_bytes, void* hip_stream) {
  return fb_external_partial_ex(shape, q, k_prefix, v_prefix, o_part, m_part, lse_part, 0, workspace,
                                workspace_bytes, hip_stream);
}

}  // extern "C"

namespace {

static __device__ __align__(256) unsigned char scratch[kBuiltinWsBytes];

constexpr int kMaxDevices = 16;
std::atomic<void*> g_scratch_ptr[kMaxDevices];   // device address of `scratch` per device, looked up on first use

// The array's name is only a host-side handle: its device address comes from hipGetSymbolAddress, asked once
// per device with that device current, and that address is what kernels and copies get.
fb_status builtin_ws(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  if (dev < 0 || dev >= kMaxDevices) return FB_ERR_UNSUPPORTED;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e);
    if (ptr == nullptr) return FB_ERR_HIP;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // racing first calls store the same address
  }
  *out = ptr;
  return FB_OK;
}

}  // namespace

extern "C" {

size_t fb_builtin_workspace_bytes(void) { return kBuiltinWsBytes; }

fb_status fb_external_partial_builtin_ws(const fb_shape* shape, const void* q, const void* k_prefix,
                                         const void* v_prefix, float* o_part, float* m_part, float* lse_part,
                                         void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  if (pass_workspace(shape, 0) > kBuiltinWsBytes) return FB_ERR_WORKSPACE;   // too large for the built-in scratch
  if (!q || !o_part || !m_part || !lse_part) return FB_ERR_NULL;      // host-side checks before any HIP call
  if (shape->prefix_len > 0 && (!k_prefix || !v_prefix)) return FB_ERR_NULL;
  void* ws = nullptr;
  st = builtin_ws(&ws);
  if (st != FB_OK) return st;
  return external_partial_impl(shape, q, k_prefix, v_prefix, nullptr, nullptr, false, 0, o_part, m_part, lse_part, 0,
                               ws, kBuiltinWsBytes, nullptr, nullptr, nullptr, hip_stream);
}

fb_status fb_head_similarity(const fb_shape* shape, const float* o_a, const float* o_b, float* sim,
                             void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  if (!o_a || !o_b || !sim) return FB_ERR_NULL;
  if (!aligned16(o_a) || !aligned16(o_b) || !aligned16(sim)) return FB_ERR_ALIGN;
  hipError_t e = fb::launch_head_similarity(o_a, o_b, sim, shape->batch * shape->n_q_heads, shape->block_len,
                                            shape->head_dim, (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_fail(e);
  return FB_OK;
}

fb_status fb_internal_merge(const fb_shape* shape, const void* q, const void* k_block,
                            const void* v_block, const float* o_part, const float* m_part,
                            const float* lse_part, void* out, float* lse_out, void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  if (!q || !k_block || !v_block || !out) return FB_ERR_NULL;
  const int n_ext = (o_part != nullptr) + (m_part != nullptr) + (lse_part != nullptr);
  if (n_ext != 0 && n_ext != 3) return FB_ERR_NULL;   // all three or none
  if (!aligned16(q) || !aligned16(k_block) || !aligned16(v_block) || !aligned16(o_part) ||
      !aligned16(m_part) || !aligned16(lse_part) || !aligned16(out) || !aligned16(lse_out))
    return FB_ERR_ALIGN;
  fb::PassParams p = base_pass(shape, q, k_block, v_block, shape->block_len, 1);
  p.ext_o = o_part; p.ext_m = m_part; p.ext_lse = lse_part;
  p.out = out; p.lse_out = lse_out;
  hipError_t e = launch_attn(shape, p, fb::kPassInternal, (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_fail(e);
  return FB_OK;
}

fb_status fb_refresh_step_prof(const fb_shape* shape, const void* q, const void* k_prefix, const void* v_prefix,
                               const void* k_block, const void* v_block, float* o_part, float* m_part,
                               float* lse_part, void* out, float* lse_out, void* workspace,
                               size_t workspace_bytes, void* ev_begin, void* ev_attn_end, void* ev_end,
                               void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  if (!q || !k_block || !v_block || !o_part || !m_part || !lse_part || !out) return FB_ERR_NULL;
  if (shape->prefix_len > 0 && (!k_prefix || !v_prefix)) return FB_ERR_NULL;
  if (!aligned16(q) || !aligned16(k_prefix) || !aligned16(v_prefix) || !aligned16(k_block) ||
      !aligned16(v_block) || !aligned16(o_part) || !aligned16(m_part) || !aligned16(lse_part) ||
      !aligned16(out) || !aligned16(lse_out) || !aligned16(workspace))
    return FB_ERR_ALIGN;
  // Small block and many splits (the LLM shapes): the prefix splits already fill every CU, so the
  // block's own keys are not streamed by the attention kernel at all (plain dense pass, with its split
  // count); one fold kernel (4 rows per workgroup) folds the splits, computes the rows' block-internal
  // attention and merges.
  // (fp32: the block's own keys are one more workgroup of the pass, which then needs a place in the single round)
  const int segs = dense_segments(shape);
  const bool few_rows = (long long)(shape->n_q_heads / shape->n_kv_heads) * shape->block_len <= fb::kRowsPerWgBf16;
  // (blocks that are no multiple of the fold kernel's rows used to be the register-staged pass and the combine only, and still are
  // where these are the faster end: by tiles per split, 8 / 16 / 24 / 48 of them, batch 2 and 4, 56 rows of 8 KV heads, head_dim 128 22.6 /
  // 32.9 / 49.6 / 87.0 and 23.9 / 33.5 / 49.1 / 83.7 us; head_dim 64, 16 / 24 / 32 / 48 22.1 / 27.5 / 33.9 / 51.6 and 22.3 / 26.4 / 31.3 /
  // 46.7, 108 rows level at 32.  Where one round in pieces replaces two, it always wins)
  const bool fours = shape->block_len % fb::kFoldRows == 0;
  const int odd_tiles = dense_parts(shape, segs) < segs ? 8 : shape->head_dim == 128 ? 24 : 32;
  const bool small_block = shape->dtype == FB_BF16 && shape->block_len <= fb::kMaxInlineBlock && segs >= 8 &&
                           (fours || (few_rows && (shape->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile >= odd_tiles * segs));
  const int ns = small_block ? segs : std::max(1, auto_splits(shape) - (shape->dtype == FB_F32 ? 1 : 0));
  const WsLayout w = ws_layout(shape, ns, 2, 0, 1);
  const size_t need = shape->dtype == FB_F32 ? pass_workspace(shape, 0) : w.total;
  if (!workspace || workspace_bytes < need) return FB_ERR_WORKSPACE;
  if (shape->dtype == FB_BF16 && !small_block && ns == 1) {
    // Many rows per KV head, unsplit: the row-pair streaming kernel, once over the prefix (it writes the partial itself) and
    // once over the block, against the register-staged pass over both and the combine (video shape, a refresh and a reuse
    // step: 1380 -> 1320 us)
    const fb::PassParams d = base_pass(shape, q, k_prefix, v_prefix, shape->prefix_len, 1);
    fb::PassParams in = base_pass(shape, q, k_block, v_block, shape->block_len, 1);
    if (fb::dense_row_pairs(d.G * d.Bq, shape->head_dim) && fb::stream_bf16_covers(d, shape->head_dim, fb::kPassDense) &&
        fb::internal_many_rows(in) && shape->block_len > 7 * fb::kKeyTile) {
      st = external_partial_impl(shape, q, k_prefix, v_prefix, nullptr, nullptr, false, 0, o_part, m_part, lse_part, 1, workspace,
                                 workspace_bytes, ev_begin, ev_attn_end, nullptr, hip_stream);
      if (st != FB_OK) return st;
      in.ext_o = o_part; in.ext_m = m_part; in.ext_lse = lse_part;
      in.out = out; in.lse_out = lse_out;
      in.rotate = 1;
      hipError_t e = launch_attn(shape, in, fb::kPassInternal, (hipStream_t)hip_stream);
      if (e == hipSuccess && ev_end) e = hipEventRecord((hipEvent_t)ev_end, (hipStream_t)hip_stream);
      return e == hipSuccess ? FB_OK : hip_fail(e);
    }
  }

  hipStream_t stream = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;
  fb::PassParams p = base_pass(shape, q, k_prefix, v_prefix, shape->prefix_len, ns);
  p.k2 = k_block; p.v2 = v_block;
  if (shape->dtype == FB_F32 && fb::f32_refresh_one((long long)p.B * p.Hkv * ((p.G * p.Bq + 15) / 16), shape->head_dim, shape->prefix_len, p.Bq)) {
    // one launch, no split partials (the workspace stays unused)
    p.nsplit = 1;
    p.ws_o = o_part; p.ws_m = m_part; p.ws_l = lse_part;
    p.out = out; p.lse_out = lse_out;
    hipError_t e = timed_attn(shape, p, fb::kPassRefreshOne, stream, ev_begin, ev_attn_end);
    if (e == hipSuccess && ev_end) e = hipEventRecord((hipEvent_t)ev_end, stream);
    return e == hipSuccess ? FB_OK : hip_fail(e);
  }
  {
    // prefix tiles the block phase is worth (its cold load, LDS hand-over and epilogue), capped at half a split
    const int tiles = (shape->prefix_len + fb::kKeyTile - 1) / fb::kKeyTile;
    const int btiles = (shape->block_len + fb::kKeyTile - 1) / fb::kKeyTile;
    p.blk_cost = ns > 1 ? std::min(2 + btiles, tiles / ns / 2) : 0;
  }
  // Few splits, up to 128 rows per KV head and a block of one tile: the streaming kernel over the prefix, then the internal
  // pass folds the splits, against the register-staged pass over both and the combine (a refresh and a reuse step, head_dim
  // 128: batch 6, 31 rows, 9000 keys 90.8 -> 83.3 us; batch 8, 32 rows, 20000 keys 146 -> 138).  head_dim 64 by tiles per split
  // (a refresh step): more than one round of workgroups from 32 on (36 tiles, 288 workgroups, blocks of 9 62.5 -> 58.5); one
  // round from 44 on (64 KV heads, blocks of 24, 36 tiles 36.4 -> 37.4, 48 44.2 -> 44.2, 64 57.2 -> 53.7), blocks of more than
  // one 32-key tile from 64 on (blocks of 61, 36 tiles 39.5 -> 41.7, 56 54.1 -> 54.6, 64 63.7 -> 60.6
  // us); always where one round in pieces replaces two (3 splits -> 2, 8 / 16 tiles a split 28.4 / 39.0 -> 25.6 / 35.0)
  const int d64_tiles = dense_parts(shape, ns) < ns ? 8 : (long long)p.B * p.Hkv * ns > 256 ? 32 : p.Bq <= 32 ? 44 : 64;
  fb::PassParams in = base_pass(shape, q, k_block, v_block, shape->block_len, 1);
  in.fold_ns = ns;
  const bool fold_internal = shape->dtype == FB_BF16 && !small_block && ns > 1 && p.G * p.Bq <= 128 &&
                             p.Bq <= fb::kKeyTile && fb::stream_bf16_covers(p, shape->head_dim, fb::kPassDense) &&
                             (shape->head_dim == 128 || shape->prefix_len >= (long long)d64_tiles * fb::kKeyTile * ns) &&
                             fb::internal_fold_covers(in, shape->head_dim);
  p.whole_tiles = fold_internal || (small_block && !fours) ? 1 : 0;
  if (small_block || fold_internal) {
    p.nseg = ns;
    p.nsplit = in.fold_ns = dense_parts(shape, ns);
  }
  p.ws_o = (float*)(ws + w.o[0]); p.ws_m = (float*)(ws + w.m[0]); p.ws_l = (float*)(ws + w.l[0]);
  p.ws_o2 = (float*)(ws + w.o[1]); p.ws_m2 = (float*)(ws + w.m[1]); p.ws_l2 = (float*)(ws + w.l[1]);
  const int streams = small_block || fold_internal ? 0 : step_streams(shape, ns);
  const WsLayout w2 = ws_layout(shape, streams, 2, 0, 2);
  const bool by_parity = streams > 0 && workspace_bytes >= w2.total;     // (below: a buffer of before, with the route of before)
  if (by_parity) {
    p.by_parity = 1;
    p.nsplit = streams;
    if (p.Bq <= fb::kKeyTile) p.k2 = p.v2 = nullptr;
    p.ws_o = (float*)(ws + w2.o[0]); p.ws_m = (float*)(ws + w2.m[0]); p.ws_l = (float*)(ws + w2.l[0]);
    p.ws_o2 = (float*)(ws + w2.o[1]); p.ws_m2 = (float*)(ws + w2.m[1]); p.ws_l2 = (float*)(ws + w2.l[1]);
  }
  hipError_t e = timed_attn(shape, p, small_block || fold_internal ? fb::kPassDense : fb::kPassRefreshFused, stream, ev_begin, ev_attn_end);
  if (e != hipSuccess) return hip_fail(e);

  fb::CombineParams c;
  memset(&c, 0, sizeof(c));
  c.rows = (int)rows_of(shape); c.D = shape->head_dim; c.nsplit = p.nsplit;
  c.ws_o = p.ws_o; c.ws_m = p.ws_m; c.ws_l = p.ws_l;
  c.o = o_part; c.m = m_part; c.lse = lse_part;
  c.Bq = shape->block_len;
  c.fin_out = out; c.fin_lse = lse_out; c.fin_bf16 = shape->dtype == FB_BF16;
  if (fold_internal) {
    in.ws_o = p.ws_o; in.ws_m = p.ws_m; in.ws_l = p.ws_l;
    in.o_final = o_part; in.m_final = m_part; in.l_final = lse_part;
    in.out = out; in.lse_out = lse_out;
    e = launch_attn(shape, in, fb::kPassInternal, stream);
  } else if (by_parity && p.k2 == nullptr && rows_of(shape) > kFoldKernelMaxRows) {
    c.fin_out = nullptr;
    e = fb::launch_combine(c, stream, by_parity);
    if (e != hipSuccess) return hip_fail(e);
    in.fold_ns = 0;
    in.ext_o = o_part; in.ext_m = m_part; in.ext_lse = lse_part;
    in.out = out; in.lse_out = lse_out;
    e = launch_attn(shape, in, fb::kPassInternal, stream);
  } else if (small_block || (by_parity && p.k2 == nullptr)) {
    c.blk_q = q; c.blk_k = k_block; c.blk_v = v_block;
    c.Hq = shape->n_q_heads; c.Hkv = shape->n_kv_heads; c.G = shape->n_q_heads / shape->n_kv_heads;
    c.scale_log2 = p.scale_log2;
    e = fb::launch_refresh_fold(c, stream);
  } else {
    c.blk_o = p.ws_o2; c.blk_m = p.ws_m2; c.blk_l = p.ws_l2;
    c.blk_ns = by_parity ? 2 : 1;
    e = fb::launch_combine(c, stream, by_parity);
  }
  if (e != hipSuccess) return hip_fail(e);
  if (ev_end && (e = hipEventRecord((hipEvent_t)ev_end, stream)) != hipSuccess) return hip_fail(e);
  return FB_OK;
}

fb_status fb_refresh_step_paged(const fb_shape* shape, const void* q, const fb_paged_kv* kv, const void* k_block,
                                const void* v_block, float* o_part, float* m_part, float* lse_part, void* out,
                                float* lse_out, int32_t n_splits, void* workspace, size_t workspace_bytes,
                                void* hip_stream) {
  if (!kv) return FB_ERR_NULL;
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  if (!k_block || !v_block || !out) return FB_ERR_NULL;
  if (!aligned16(k_block) || !aligned16(v_block) || !aligned16(out) || !aligned16(lse_out)) return FB_ERR_ALIGN;
  // One split: the paged pass writes the partial itself and the internal pass follows.  Several splits and a small block of
  // few rows: one kernel of 4 rows per workgroup folds, computes the rows' block-internal attention and merges (as in
  // fb_refresh_step; beyond a few thousand rows that latency chain loses: 219 vs ~165 us per step at batch 32, block 32).
  // Few splits otherwise (bf16): the internal pass folds them (batch 8,
  // 32 rows, up to 8000 keys 61.2 -> 58.5 us a refresh and a reuse step; batch 32 162.2 -> 159.7); at head_dim 128 blocks of more
  // than one 32-key tile only in one round of its 32-row workgroups (blocks of 64, 256 of them, 45.4 -> 43.9 a refresh step;
  // blocks of 40, 640 of them, 96.7 -> 102).  Else combine + internal pass.
  fb::PassParams in = base_pass(shape, q, k_block, v_block, shape->block_len, 1);
  in.out = out; in.lse_out = lse_out;
  in.fold_ns = n_splits > 0 ? n_splits : paged_splits(shape);
  // Blocks that are no multiple of that kernel's rows: only from 5 splits on and up to 896 rows, fp32 1408 (batch 11, 4026 rows, blocks of 61, 2
  // splits 37.3 us the other way and 61.3 by it; 1008 rows, 5 splits 34.0 and 38.2; 504 rows, 10 splits 25.6 and 23.5.  Random calls, by it against
  // the other way: inside these lines 0.97 on average and 1.01 in 95 of 100, fp32 0.93 and 1.02; outside up to 1.64, fp32 1.41).
  const bool fours = shape->block_len % fb::kFoldRows == 0;
  const long long fold_rows = fours ? kFoldKernelMaxRows : shape->dtype == FB_BF16 ? 896 : 1408;
  const bool fold_kernel = shape->block_len <= fb::kMaxInlineBlock && rows_of(shape) <= fold_rows && (fours || in.fold_ns >= 5);
  const bool one_round = (long long)in.B * in.Hkv * ((in.G * in.Bq + 31) / 32) <= 256;
  const bool fold_internal = !fold_kernel && shape->dtype == FB_BF16 && in.fold_ns > 1 &&
                             (shape->head_dim == 64 || in.Bq <= 32 || one_round) &&
                             fb::internal_fold_covers(in, shape->head_dim);
  fb::CombineParams c;
  st = external_partial_impl(shape, q, nullptr, nullptr, kv, nullptr, false, 0, o_part, m_part, lse_part, n_splits,
                             workspace, workspace_bytes, nullptr, nullptr, nullptr, hip_stream,
                             fold_kernel || fold_internal ? &c : nullptr);
  if (st != FB_OK) return st;
  hipError_t e = hipSuccess;
  if (fold_kernel && c.nsplit > 0) {
    c.fin_out = out; c.fin_lse = lse_out; c.fin_bf16 = shape->dtype == FB_BF16;
    c.blk_q = q; c.blk_k = k_block; c.blk_v = v_block;
    c.scale_log2 = eff_scale(shape) * kLog2e;
    e = fb::launch_refresh_fold(c, (hipStream_t)hip_stream);
  } else {
    if (fold_internal) {
      in.ws_o = (float*)c.ws_o; in.ws_m = (float*)c.ws_m; in.ws_l = (float*)c.ws_l;
      in.o_final = o_part; in.m_final = m_part; in.l_final = lse_part;
    } else {
      in.fold_ns = 0;
      in.ext_o = o_part; in.ext_m = m_part; in.ext_lse = lse_part;
    }
    e = launch_attn(shape, in, fb::kPassInternal, (hipStream_t)hip_stream);
  }
  return e == hipSuccess ? FB_OK : hip_fail(e);
}

fb_status fb_refresh_step(const fb_shape* shape, const void* q, const void* k_prefix, const void* v_prefix,
                          const void* k_block, const void* v_block, float* o_part, float* m_part,
                          float* lse_part, void* out, float* lse_out, void* workspace, size_t workspace_bytes,
                          void* hip_stream) {
  return fb_refresh_step_prof(shape, q, k_prefix, v_prefix, k_block, v_block, o_part, m_part, lse_part, out,
                              lse_out, workspace, workspace_bytes, nullptr, nullptr, nullptr, hip_stream);
}

fb_status fb_pool_keys(const fb_shape* shape, const void* k_prefix, int32_t key_block, float* k_pooled,
                       void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  int nblk = 0;
  st = check_key_block(shape, key_block, 0, &nblk);
  if (st != FB_OK) return st;
  if (shape->prefix_len > 0 && (!k_prefix || !k_pooled)) return FB_ERR_NULL;
  if (!aligned16(k_prefix) || !aligned16(k_pooled)) return FB_ERR_ALIGN;
  fb::PoolParams p;
  p.k = k_prefix; p.k_pooled = k_pooled;
  p.BH = shape->batch * shape->n_kv_heads; p.nkeys = shape->prefix_len; p.D = shape->head_dim;
  p.key_block = key_block; p.nblk = nblk; p.is_bf16 = shape->dtype == FB_BF16;
  hipError_t e = fb::launch_pool_keys(p, (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_fail(e);
  return FB_OK;
}

size_t fb_select_workspace_bytes(const fb_shape* shape, int32_t key_block) {
  if (check_shape(shape) != FB_OK) return 0;
  int nblk = 0;
  if (check_key_block(shape, key_block, 0, &nblk) != FB_OK) return 0;
  const size_t heads = (size_t)shape->batch * shape->n_q_heads;
  return align256(heads * shape->head_dim * sizeof(float)) + align256(heads * nblk * sizeof(float)) + 256;
}

fb_status fb_select_topk(const fb_shape* shape, const void* q, const float* k_pooled, int32_t key_block,
                         int32_t topk, int32_t* sel_idx, void* workspace, size_t workspace_bytes,
                         void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  int nblk = 0;
  st = check_key_block(shape, key_block, topk, &nblk);
  if (st != FB_OK) return st;
  if (topk == 0) return FB_OK;
  if (!q || !sel_idx || (nblk > 0 && !k_pooled)) return FB_ERR_NULL;
  if (!aligned16(q) || !aligned16(k_pooled) || !aligned16(sel_idx) || !aligned16(workspace)) return FB_ERR_ALIGN;
  if (workspace && workspace_bytes < fb_select_workspace_bytes(shape, key_block)) return FB_ERR_WORKSPACE;
  fb::SelectParams p;
  memset(&p, 0, sizeof(p));
  p.q = q; p.k_pooled = k_pooled; p.sel_idx = sel_idx;
  if (workspace) {
    p.qbar_ws = (float*)workspace;
    p.scores_ws = (float*)((char*)workspace +
                           align256((size_t)shape->batch * shape->n_q_heads * shape->head_dim * sizeof(float)));
  }
  p.B = shape->batch; p.Hq = shape->n_q_heads; p.Hkv = shape->n_kv_heads;
  p.G = shape->n_q_heads / shape->n_kv_heads; p.Bq = shape->block_len; p.D = shape->head_dim;
  p.nblk = nblk; p.topk = topk; p.is_bf16 = shape->dtype == FB_BF16;
  hipError_t e = fb::launch_select_topk(p, (hipStream_t)hip_stream);
  if (e != hipSuccess) return hip_fail(e);
  return FB_OK;
}

size_t fb_select_mass_workspace_bytes(const fb_shape* shape, int32_t key_block) {
  if (check_shape(shape) != FB_OK) return 0;
  int nblk = 0;
  if (check_key_block(shape, key_block, 0, &nblk) != FB_OK) return 0;
  return align256((size_t)rows_of(shape) * nblk * sizeof(float)) + 256;
}

fb_status fb_select_topk_mass(const fb_shape* shape, const void* q, const void* k_prefix, const float* lse_part,
                              int32_t key_block, int32_t topk, int32_t* sel_idx, float* mass_out,
                              void* workspace, size_t workspace_bytes, void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  int nblk = 0;
  st = check_key_block(shape, key_block, topk, &nblk);
  if (st != FB_OK) return st;
  if (topk == 0 || nblk == 0) return FB_OK;
  if (!q || !k_prefix || !lse_part || !sel_idx) return FB_ERR_NULL;
  if (!aligned16(q) || !aligned16(k_prefix) || !aligned16(lse_part) || !aligned16(sel_idx) ||
      !aligned16(mass_out) || !aligned16(workspace))
    return FB_ERR_ALIGN;
  if (!workspace || workspace_bytes < fb_select_mass_workspace_bytes(shape, key_block)) return FB_ERR_WORKSPACE;
  hipStream_t stream = (hipStream_t)hip_stream;
  const bool bf16 = shape->dtype == FB_BF16;

  fb::MassParams m;
  memset(&m, 0, sizeof(m));
  m.q = q; m.k = k_prefix; m.lse = lse_part; m.rowmass = (float*)workspace;
  m.B = shape->batch; m.Hq = shape->n_q_heads; m.Hkv = shape->n_kv_heads;
  m.G = shape->n_q_heads / shape->n_kv_heads; m.Bq = shape->block_len;
  m.nkeys = shape->prefix_len; m.key_block = key_block; m.nblk = nblk;
  m.scale_log2 = eff_scale(shape) * kLog2e;
  {
    // key-block ranges per row tile: enough workgroups for ~2 per CU, never more than key blocks
    const long long groups = bf16
        ? (long long)m.B * m.Hkv * ((m.G * m.Bq + fb::kRowsPerWgBf16 - 1) / fb::kRowsPerWgBf16)
        : (long long)m.B * m.Hq * ((m.Bq + fb::kRowsPerWgF32 - 1) / fb::kRowsPerWgF32);
    long long ns = ((bf16 ? 512 : 1024) + groups - 1) / groups;
    if (ns > nblk) ns = nblk;
    if (ns > 65535) ns = 65535;
    m.nsplit = (int)ns;
  }
  hipError_t e = bf16 ? fb::launch_block_mass_bf16(m, shape->head_dim, stream)
                      : fb::launch_block_mass_f32(m, shape->head_dim, stream);
  if (e != hipSuccess) return hip_fail(e);

  fb::SelectParams p;
  memset(&p, 0, sizeof(p));
  p.sel_idx = sel_idx; p.rowmass = m.rowmass; p.score_out = mass_out;
  p.B = m.B; p.Hq = m.Hq; p.Hkv = m.Hkv; p.G = m.G; p.Bq = m.Bq; p.D = shape->head_dim;
  p.nblk = nblk; p.topk = topk; p.is_bf16 = bf16;
  e = fb::launch_select_topk(p, stream);
  if (e != hipSuccess) return hip_fail(e);
  return FB_OK;
}

fb_status fb_sparse_external_residual(const fb_shape* shape, int32_t mode, const void* q,
                                      const void* k_prefix, const void* v_prefix, int32_t key_block,
                                      int32_t topk, const int32_t* sel_idx, float* res_o, float* res_m,
                                      float* res_lse, float* o_part, float* m_part, float* lse_part,
                                      void* workspace, size_t workspace_bytes, void* hip_stream) {
  fb_status st = check_shape(shape);
  if (st != FB_OK) return st;
  if (mode != FB_SPARSE_REFRESH && mode != FB_SPARSE_REUSE && mode != FB_SPARSE_REUSE_SAME_SELECTION)
    return FB_ERR_SHAPE;
  const bool keep_masks = mode == FB_SPARSE_REUSE_SAME_SELECTION;
  if (keep_masks) mode = FB_SPARSE_REUSE;
  int nblk = 0;
  st = check_key_block(shape, key_block, topk, &nblk);
  if (st != FB_OK) return st;
  if (!q || !res_o || !res_m || !res_lse || !o_part || !m_part || !lse_part) return FB_ERR_NULL;
  if (shape->prefix_len > 0 && (!k_prefix || !v_prefix)) return FB_ERR_NULL;
  if (topk > 0 && !sel_idx && !keep_masks) return FB_ERR_NULL;
  if (!aligned16(q) || !aligned16(k_prefix) || !aligned16(v_prefix) || !aligned16(sel_idx) ||
      !aligned16(res_o) || !aligned16(res_m) || !aligned16(res_lse) || !aligned16(o_part) ||
      !aligned16(m_part) || !aligned16(lse_part) || !aligned16(workspace))
    return FB_ERR_ALIGN;
  const int ns = sparse_splits(shape, mode == FB_SPARSE_REFRESH);
  const WsLayout w = ws_layout(shape, ns, 2, nblk);
  if (!workspace || workspace_bytes < ws_layout(shape, sparse_splits(shape, false), 2, nblk).total)
    return FB_ERR_WORKSPACE;

  hipStream_t stream = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;

  fb::MaskParams mp;
  mp.sel_idx = topk > 0 ? sel_idx : nullptr;
  mp.blk_mask = (uint32_t*)(ws + w.mask); mp.union_list = (int32_t*)(ws + w.ulist);
  mp.union_mask = (uint32_t*)(ws + w.umask);
  mp.union_cnt = (int32_t*)(ws + w.ucnt);
  mp.B = shape->batch; mp.Hq = shape->n_q_heads; mp.Hkv = shape->n_kv_heads;
  mp.G = shape->n_q_heads / shape->n_kv_heads; mp.topk = topk; mp.nblk = nblk;
  hipError_t e = hipSuccess;
  if (nblk > 0 && !keep_masks) {
    e = fb::launch_build_masks(mp, stream);
    if (e != hipSuccess) return hip_fail(e);
  }

  fb::PassParams p = base_pass(shape, q, k_prefix, v_prefix, shape->prefix_len, ns);
  p.ws_o = (float*)(ws + w.o[0]); p.ws_m = (float*)(ws + w.m[0]); p.ws_l = (float*)(ws + w.l[0]);
  p.ws_o2 = (float*)(ws + w.o[1]); p.ws_m2 = (float*)(ws + w.m[1]); p.ws_l2 = (float*)(ws + w.l[1]);
  p.blk_mask = mp.blk_mask; p.union_list = mp.union_list; p.union_mask = mp.union_mask; p.union_cnt = mp.union_cnt;
  p.key_block = key_block; p.nblk = nblk;

  fb::CombineParams c;
  memset(&c, 0, sizeof(c));
  c.rows = (int)rows_of(shape); c.D = shape->head_dim; c.nsplit = ns;
  c.o = o_part; c.m = m_part; c.lse = lse_part;
  if (nblk > 0) {
    c.ws_o = p.ws_o; c.ws_m = p.ws_m; c.ws_l = p.ws_l;
    e = launch_attn(shape, p, mode == FB_SPARSE_REFRESH ? fb::kPassSparseRefresh : fb::kPassSparseReuse, stream);
    if (e != hipSuccess) return hip_fail(e);
  } else {
    c.nsplit = 0;   // empty prefix: nothing selected, nothing residual
  }
  if (mode == FB_SPARSE_REFRESH) {
    if (nblk > 0) { c.ws_o2 = p.ws_o2; c.ws_m2 = p.ws_m2; c.ws_l2 = p.ws_l2; }
    c.res_out_o = res_o; c.res_out_m = res_m; c.res_out_lse = res_lse;
  } else {
    c.res_in_o = res_o; c.res_in_m = res_m; c.res_in_lse = res_lse;
  }
  e = fb::launch_combine(c, stream);
  if (e != hipSuccess) return hip_fail(e);
  return FB_OK;
}

}  // extern "C"
