// bf16 streaming attention pass for gfx950 (MI355X): K/V tiles travel from global memory straight into a ring
// of LDS stages (direct-to-LDS 16-byte loads, no register staging), K operands are read back with
// ds_read_b128 from a rotation-swizzled row-major layout, V operands with the transposing LDS read
// (ds_read_b64_tr_b16) from row-major V, so nothing is transposed or re-stored on the way.
//
// Computes the per-row statistics of Eq. 3-4/6 (arxiv 2602.05305, Section 4.2) of a block of query rows
// against a stream of keys and either stores split partials / the final partial (external passes) or finishes
// with the log-space composition of Eq. 8-9 against a cached partial (internal pass).
//
// Work decomposition: one workgroup streams one list of 64-key tiles through NS ring stages.
//   kKeySplit  NRG = 4, 2 or 1 groups of 32 group-flattened rows (8, 4 or 2 wavefronts); wavefront w owns row group
//              w % NRG and the key half w / NRG of every tile; the two halves exchange accumulator halves through LDS
//              after the last tile and each finishes and stores half of the output columns.  (LLM-shaped blocks:
//              the whole KV group is one workgroup, every K/V byte is fetched once; NRG = 2 / 1 for KV groups of
//              at most 64 / 32 rows, the 4- and 8-token blocks, where more row groups would compute padding.)
//              Sparse refresh pass: the same layout with two accumulator sets per wavefront (selected /
//              residual key blocks); a tile's scores are computed once and go to the set the row's head routes
//              the tile's key block to, so the eight wavefronts stay evenly loaded whatever the selection.
//              At head_dim 64 two tiles per barrier.
//   kTileSplit the same with whole tiles: half h takes every other tile, two tiles per barrier.  (Refresh step with few splits; internal
//              pass of one round of workgroups.)
//   kRowPair   256 rows, 4 wavefronts of 64 rows and whole tiles (many rows per KV head): fb_rows_bf16.h.
//   kRowPairShort  256 rows, wavefront w owns rows [32 w, +32) and whole tiles, two tiles per barrier: dense streams too short for
//              kRowPair, whose ends cost more (its first scores stand alone, it scores a tile past the last one, and four
//              wavefronts store what eight do here).
//   Per tile and wavefront: S^T = K Q^T on v_mfma_f32_32x32x16_bf16 (A = K rows from LDS, B = Q^T in
//   registers), in-lane online softmax with a lazily moved reference, O^T += V^T P^T with the lane's own
//   probabilities as the B operand (register layout reasoning: fb_attn_bf16.hip, which is the same).
// LDS layout of a stage: [K: 64 rows x D*2 bytes][V: 64 rows x D*2 bytes], rows unpadded, the 16-byte chunks
//   of a row rotated by a row-dependent amount (K: by row, V: by 4*row at head_dim 128; by row/2 and
//   4*(row/2) at head_dim 64) so that both read patterns are bank-conflict-free.  A direct-to-LDS load puts
//   the 64 lanes' chunks at consecutive LDS addresses, so the rotation is applied on the global-address side.
// Synchronisation: the direct-to-LDS loads are issued from inline assembly, invisible to the compiler's
//   wait-count insertion (which would otherwise drain every outstanding load before any LDS read); each
//   wavefront waits for its own loads of a tile with an explicit s_waitcnt vmcnt(n), then the workgroup
//   barrier makes the tile visible to all.  The stage refilled after barrier t is the one last read in
//   iteration t-1, which every wavefront has left by then.
#include <stdio.h>

#include "fb_kernels.h"
#include "fb_rows_bf16.h"

namespace fb {
namespace {

// (kKeySplitSingle: the key split with one tile per barrier at head_dim 64 as well)
// kKeySplitParts, kTileSplitParts: the first two where the workgroups' ranges are not the reference segments (PassParams::nseg)
enum StreamLayout : int { kKeySplit = 0, kTileSplit = 1, kRowPair = 2, kKeySplitSingle = 3, kRowPairShort = 4, kKeySplitParts = 5, kTileSplitParts = 6 };
constexpr bool in_parts(int layout) { return layout == kKeySplitParts || layout == kTileSplitParts; }
constexpr int whole_layout(int layout) { return layout == kKeySplitParts ? kKeySplit : layout == kTileSplitParts ? kTileSplit : layout; }
constexpr bool key_split(int layout) { return layout == kKeySplit || layout == kKeySplitSingle; }

// Key split at head_dim 64: two tiles per barrier, their scores and weights computed together, because a tile's fixed cost
// (barrier, refill, the softmax's cross-lane step) is large against its 16 KB: batch 4, 64K keys, 32 rows
// per KV head 118 -> 101 us a refresh and a reuse step, 128K keys 64.6 -> 60.7, a sparse block at 64K 209 -> 201.  Not at
// head_dim 128, where pairs of tiles leave 64 KB in flight instead of 96 (128K keys: 1 % slower).  Dense and paged passes: at every
// length the kernel takes (one tile -> two; 8, 16, 40 tiles per split: 128 rows of 8 KV heads 19.05 -> 18.95, 26.0 -> 25.3,
// 46.8 -> 45.1 us; 64 rows 17.4 -> 17.7, 23.9 -> 23.4, 42.8 -> 40.0; 64 paged sequences of 16 rows 13.8 -> 12.6, 21.6 ->
// 20.2, 42.9 -> 37.5).
constexpr bool paired_halves(int D, int layout) { return D == 64 && layout == kKeySplit; }

// NRG: 32-row groups of a key-split workgroup (4: 128 rows, 8 wavefronts; 2: 64 rows, 4 wavefronts; 1: 32 rows, 2
// wavefronts: the small blocks of 4- and 8-token diffusion steps, where more row groups would compute padding rows)
template <int D, int LAYOUT, int NSETS = 1, int NRG = 4>
struct SCfg {
  static constexpr bool RP = LAYOUT == kRowPairShort;
  static constexpr int NW = RP ? 8 : 2 * NRG;         // wavefronts per workgroup
  static constexpr int THREADS = 64 * NW;
  static constexpr int KT = 64;                       // keys per tile
  static constexpr int ROWB = D * 2;                  // bytes per key row
  static constexpr int CPR = ROWB / 16;               // 16-byte chunks per row
  static constexpr int OPB = KT * ROWB;               // bytes per operand (K or V) per tile
  static constexpr int STAGE = 2 * OPB;
  static constexpr int NLOAD = OPB / (THREADS * 16);  // direct-to-LDS loads per lane, operand and tile
  static constexpr int LSTEP = NW * 1024;             // LDS bytes one load of every wavefront covers
  static constexpr int LPT = 2 * NLOAD;               // loads per lane and tile
  static constexpr int NS = (D == 128) ? 4 : (RP || LAYOUT == kKeySplitSingle) ? 6 : 8;       // ring stages
  static constexpr int NKS = D / 16;                  // MFMA k-steps of the score product
  static constexpr int NDB = D / 32;                  // 32-wide output column blocks
  static constexpr int ROWS = RP ? 256 : 32 * NRG;
  static constexpr int NKB = key_split(LAYOUT) ? 1 : 2;    // 32-key blocks of a tile one wavefront computes
  static constexpr int QPARTS = (ROWS + 63) / 64;             // the query rows are loaded 64 at a time, like a K operand
  static constexpr int QSTAGES = (QPARTS * OPB + STAGE - 1) / STAGE;   // ring stages they pass through at start
  static constexpr int MERGE = RP ? 0 : NSETS * NRG * 2 * (NDB / 2 * 16 + 2) * 64 * 4;   // key-half exchange
  static constexpr int RING = NS * STAGE;
  static constexpr int FIFO = RING > MERGE ? RING : MERGE;
  static constexpr int LDS = FIFO;
  static_assert(QSTAGES >= 1 && QSTAGES < NS && NLOAD >= 1, "ring geometry");
  static_assert((NS - 1) * LPT <= 63, "the loads of NS - 1 tiles in flight must fit the 6-bit load counter");
  // rotation (in chunks) of row `row`
  __device__ static __forceinline__ int rot_k(int row) { return D == 128 ? row : (row >> 1); }
  __device__ static __forceinline__ int rot_v(int row) { return D == 128 ? 4 * row : 4 * (row >> 1); }
};

// wait until at most `tiles` tiles' worth of this lane's direct-to-LDS loads are outstanding
// (the counter has 6 bits: counts above 63 cannot be asked for, and no ring here keeps that many loads in flight)
template <int LPT>
__device__ __forceinline__ void wait_tiles(int tiles) {
  constexpr int kMax = 63 / LPT;       // largest tile count the counter can express
  if (kMax >= 5 && tiles >= 5) wait_vm<(kMax >= 5 ? 5 : 0) * LPT>();
  else if (kMax >= 4 && tiles >= 4) wait_vm<(kMax >= 4 ? 4 : 0) * LPT>();
  else if (kMax >= 3 && tiles >= 3) wait_vm<(kMax >= 3 ? 3 : 0) * LPT>();
  else if (kMax >= 2 && tiles >= 2) wait_vm<(kMax >= 2 ? 2 : 0) * LPT>();
  else if (kMax >= 1 && tiles >= 1) wait_vm<(kMax >= 1 ? 1 : 0) * LPT>();
  else wait_vm<0>();
}

// Running softmax state of the 32 rows a wavefront owns (one row per lane pair l, l^32).
template <int NDB>
struct WaveAcc {
  float m, l;          // log2-domain running reference; per-lane partial row sum
  f32x16 o[NDB];       // O^T: lane (row = lane%32, h = lane/32) holds d = 32db + 8(r/4) + 4h + r%4
  __device__ __forceinline__ void init() {
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int i = 0; i < NDB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
  }
};

// Scores of this wavefront's 32 rows against key blocks [kb0, kb0 + NKB) of the tile in `stage`.
// kaddr[ks] = per-lane byte address (within a stage, key block 0) of the K chunk of k-step ks.
template <int D, int NKB>
__device__ __forceinline__ void tile_scores(f32x16 (&s)[NKB], const bf16x8 (&qreg)[D / 16],
                                            const unsigned char* __restrict__ stage, const uint32_t (&kaddr)[D / 16],
                                            int kb0) {
  constexpr int NKS = D / 16, ROWB = D * 2;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
  for (int ks0 = 0; ks0 < NKS; ks0 += 2) {
    bf16x8 a[2][NKB];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
        a[u][kb] = *(const bf16x8*)(stage + kaddr[ks0 + u] + (kb0 + kb) * 32 * ROWB);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u][kb], qreg[ks0 + u], s[kb], 0, 0, 0);
  }
  if constexpr (D == 128 && NKB == 1) {
    // one accumulator chain: every operand is requested one MFMA ahead.  Left to itself the compiler does so in some
    // instantiations and waits for each read in front of its MFMA in others (per-head refresh, up to 32 rows per KV head: 190
    // cycles a tile; 4 x 8 KV groups, 16752 keys, 59.5 -> 56.8 us; a sparse block at 64K keys 261.3 -> 258.7)
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);         // LDS reads
#pragma unroll
    for (int ks = 2; ks < NKS; ++ks) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
  }
}

// A reference that moves down scales what is accumulated up, by at most this many powers of two.  All that a segment farther below
// adds to a row, 2^17 keys of it, is below 2^-15 of the row's sum and its rounding to bf16 below 2^-24 of it, so where its reference
// lies no longer shows.  And 2^17 keys of weight 2^8 leave less than 2^57 times a value, the squares of 128 such sums fp32 can add (the
// similarity of two partials does).
constexpr float kMostDown = 32.f;

// Online softmax update with the tile's scores: moves the running reference if needed (rescaling the accumulators),
// adds the row sums, and leaves the tile's probabilities, rounded to bf16, in pb (B operands of the value product).
//   s[kb][r] = raw dot product of query row lane%32 with key 32 (kb0 + kb) + 8 (r/4) + 4 h + r%4
template <int D, int NKB>
__device__ __forceinline__ void tile_softmax(WaveAcc<D / 32>& st, f32x16 (&s)[NKB], bf16x8 (&pb)[2 * NKB], int kb0,
                                             float scale_log2, bool lane_on, int nvalid, int h, bool fresh = false) {
  constexpr int NDB = D / 32;
  if (nvalid < 64) {
    // the empty asm keeps this a real (wavefront-uniform) branch instead of per-score selects on every tile
    asm volatile("" ::: "memory");
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = (kb0 + kb) * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        if (key >= nvalid) s[kb][r] = -INFINITY;
      }
  }
  float tmax = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[kb][r]);
  tmax = lane_on ? tmax * scale_log2 : -INFINITY;
  tmax = max_halves(tmax);
  // Lazy reference: m moves only when the tile maximum exceeds it by more than kLazy (log2 units); weights
  // stay below 2^kLazy, (o, l, m) remain exactly paired, and the accumulators are rescaled on few tiles only.
  constexpr float kLazy = 8.f;
  // fresh: the first tile of a reference segment moves it always (down as well, by up to kMostDown)
  const float m_new = (tmax > st.m + kLazy || (fresh && tmax > st.m - kMostDown)) ? tmax : st.m;
  const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(st.m - m_use);
  float lsum = 0.f;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float pf = __builtin_amdgcn_exp2f(fmaf(s[kb][r], scale_log2, -m_use));
      if (!lane_on) pf = 0.f;
      lsum += pf;
      pb[2 * kb + r / 8][r % 8] = (__bf16)pf;
    }
  st.l = st.l * alpha + lsum;
  st.m = m_new;
  if (__any(alpha != 1.f)) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
  }
}

// Value accumulation O^T[db] += V^T P^T over 16-key steps: A operand element e of lane half h is key
// 16u + 8(e/4) + 4h + e%4 of the key block, i.e. two transposing reads of 4 consecutive keys each.
//   vaddr[db] = per-lane byte address (within a stage) of the lane's share of the transposing V read of column block
//               db, key offset 0 (the lane's own 4h + i/4 row offset is inside); the 4-key groups are reached
//               through immediate offsets
template <int D, int NKB>
__device__ __forceinline__ void tile_pv(WaveAcc<D / 32>& st, const bf16x8 (&pb)[2 * NKB],
                                        const unsigned char* __restrict__ stage, const uint32_t (&vaddr)[D / 32], int kb0) {
  constexpr int NDB = D / 32, ROWB = D * 2, OPB = 64 * ROWB;
#pragma unroll
  for (int t = 0; t < 2 * NKB; ++t) {
    const int krow = (kb0 + t / 2) * 32 + 16 * (t % 2);
    bf16x8 a[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const unsigned char* base = stage + OPB + vaddr[db] + krow * ROWB;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(base));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(base + 8 * ROWB));
      const s16x8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      a[db] = __builtin_bit_cast(bf16x8, both);
    }
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[db], pb[t], st.o[db], 0, 0, 0);
  }
}

template <int D, int NKB>
__device__ __forceinline__ void tile_softmax_pv(WaveAcc<D / 32>& st, f32x16 (&s)[NKB],
                                                const unsigned char* __restrict__ stage,
                                                const uint32_t (&vaddr)[D / 32], int kb0, float scale_log2,
                                                bool lane_on, int nvalid, int h, bool fresh = false) {
  bf16x8 pb[2 * NKB];
  tile_softmax<D, NKB>(st, s, pb, kb0, scale_log2, lane_on, nvalid, h, fresh);
  tile_pv<D, NKB>(st, pb, stage, vaddr, kb0);
}

// The reference a stream would have after this tile as its first one; nothing is accumulated yet.
template <int NDB, int NKB>
__device__ __forceinline__ void tile_reference(WaveAcc<NDB>& st, const f32x16 (&s)[NKB], int kb0, float scale_log2, int nvalid, int h) {
  float tmax = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if ((kb0 + kb) * 32 + 8 * (r / 4) + 4 * h + (r % 4) < nvalid) tmax = fmaxf(tmax, s[kb][r]);
  st.m = max_halves(tmax * scale_log2);
}

// One tile of a wavefront for every accumulator set that any of its rows feeds (on).
template <int D, int NSETS, int NKB>
__device__ __forceinline__ void sets_tile(WaveAcc<D / 32> (&accs)[NSETS], const bool (&on)[NSETS], const bf16x8 (&qreg)[D / 16],
                                          const unsigned char* __restrict__ stage, const uint32_t (&kaddr)[D / 16],
                                          const uint32_t (&vaddr)[D / 32], int kb0, float scale_log2, int nvalid, int h) {
  f32x16 s[NKB];
  tile_scores<D, NKB>(s, qreg, stage, kaddr, kb0);
#pragma unroll
  for (int i = 0; i < NSETS; ++i) {
    if (NSETS > 1 && !__any(on[i])) continue;
    tile_softmax_pv<D, NKB>(accs[i], s, stage, vaddr, kb0, scale_log2, on[i], nvalid, h);
  }
}

// Scores for one 32-key block of each of two tiles, whose accumulator chains alternate.
template <int D>
__device__ __forceinline__ void two_scores(f32x16 (&s)[2], const bf16x8 (&qreg)[D / 16], const unsigned char* __restrict__ stage_a,
                                           const unsigned char* __restrict__ stage_b, const uint32_t (&kaddr)[D / 16], int kb0) {
  constexpr int NKS = D / 16, ROWB = D * 2;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) s[i][r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    const bf16x8 a = *(const bf16x8*)(stage_a + kaddr[ks] + kb0 * 32 * ROWB);
    const bf16x8 b = *(const bf16x8*)(stage_b + kaddr[ks] + kb0 * 32 * ROWB);
    s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], s[0], 0, 0, 0);
    s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, qreg[ks], s[1], 0, 0, 0);
  }
}

// Softmax update and value product of the two blocks.  Each tile moves the reference by the rule of tile_softmax, one
// after the other; unless the second moves it (rare), both tiles' weights are taken against the same reference and
// computed together, else one after the other.
template <int D>
__device__ __forceinline__ void two_softmax_pv(WaveAcc<D / 32>& st, f32x16 (&s)[2], const unsigned char* __restrict__ stage_a,
                                               const unsigned char* __restrict__ stage_b, const uint32_t (&vaddr)[D / 32],
                                               int kb0, float scale_log2, bool on_a, bool on_b, int nva, int nvb, int h) {
  constexpr int NDB = D / 32;
  constexpr float kLazy = 8.f;
  const bool on[2] = {on_a, on_b};
  const int nv[2] = {nva, nvb};
  float tmax[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (nv[i] < 64) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = kb0 * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        if (key >= nv[i]) s[i][r] = -INFINITY;
      }
    }
    tmax[i] = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) tmax[i] = fmaxf(tmax[i], s[i][r]);
    tmax[i] = on[i] ? tmax[i] * scale_log2 : -INFINITY;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) tmax[i] = max_halves(tmax[i]);
  const float m_a = (tmax[0] > st.m + kLazy) ? tmax[0] : st.m;
  const float m_b = (tmax[1] > m_a + kLazy) ? tmax[1] : m_a;
  if (__any(m_b != m_a)) {
    f32x16 one[1] = {s[0]};
    tile_softmax_pv<D, 1>(st, one, stage_a, vaddr, kb0, scale_log2, on_a, nva, h);
    one[0] = s[1];
    tile_softmax_pv<D, 1>(st, one, stage_b, vaddr, kb0, scale_log2, on_b, nvb, h);
    return;
  }
  const float m_use = (m_a == -INFINITY) ? 0.f : m_a;
  const float alpha = __builtin_amdgcn_exp2f(st.m - m_use);
  bf16x8 pa[2], pb[2];
  float lsum[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float pf = __builtin_amdgcn_exp2f(fmaf(s[i][r], scale_log2, -m_use));
      if (!on[i]) pf = 0.f;
      lsum[i] += pf;
      if (i == 0) pa[r / 8][r % 8] = (__bf16)pf;
      else pb[r / 8][r % 8] = (__bf16)pf;
    }
  st.l = (st.l * alpha + lsum[0]) + lsum[1];
  st.m = m_a;
  if (__any(alpha != 1.f)) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
  }
  tile_pv<D, 1>(st, pa, stage_a, vaddr, kb0);
  tile_pv<D, 1>(st, pb, stage_b, vaddr, kb0);
}

// A tile of the stream (all wavefront-uniform).  TileRaw is what the table lookups deliver (fetched one iteration
// before the tile is issued, with no arithmetic on the loaded words, so that the wait for them falls into the
// next iteration); TileDesc adds the addresses.
struct TileRaw {
  int e;            // entry of the pass's tile list
  int word;         // sparse reuse: key block; paged: page id; else unused
  uint32_t mask;    // selection mask of the tile's key block (sparse passes), else all ones
};
struct TileDesc {
  int k0;
  uint32_t mask;
  const unsigned char* kt;
  const unsigned char* vt;
};

// What a workgroup does with an entry of its stream (TileRaw::mask) where its range is not a reference segment.
constexpr uint32_t kSegFirst = 1u, kSegReference = 2u, kSegPad = 4u;

// Every layout but kRowPair: two wavefronts per row group, or one (kRowPairShort).  PARTS: the stream of a (batch element, KV head) is
// p.nseg reference segments, each visited in an order of its own, and the workgroups take p.nsplit even pieces of that walk.
template <int D, int MODE, int LAYOUT, int NRG, bool PARTS>
__device__ __forceinline__ void halves_pass(const PassParams& p, unsigned char* ring) {
  static_assert(!PARTS || (MODE == kPassDense && (LAYOUT == kKeySplit || LAYOUT == kTileSplit)), "reference segments: dense pass");
  constexpr int NSETS = (MODE == kPassSparseRefresh) ? 2 : 1;
  using C = SCfg<D, LAYOUT, NSETS, NRG>;
  static_assert(MODE == kPassDense || MODE == kPassDenseHeads || MODE == kPassDensePaged || MODE == kPassSparseReuse ||
                    MODE == kPassSparseRefresh || (MODE == kPassInternal && LAYOUT == kTileSplit), "modes of this form");
  constexpr bool kHalves = LAYOUT != kRowPairShort;
  static_assert(kHalves || MODE == kPassDense, "one wavefront per row group: dense pass");
  // Whole tiles and head_dim 64: two tiles per barrier (tiles t, t+1 are computed while t+2, t+3 are in flight); key split at 128:
  // one tile per barrier, NS - 1 in flight.
  constexpr bool kPairs = !key_split(LAYOUT) || paired_halves(D, LAYOUT);
  constexpr int AHEAD = kPairs ? C::NS - 2 : C::NS - 1;
  static_assert(!kPairs || C::NS % 2 == 0, "pairs of tiles: an even number of stages");
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));     // wavefront-uniform (scalar)
  const int rg = kHalves ? wave % NRG : wave;                  // 32-row group
  const int half = kHalves ? wave / NRG : 0;                   // keys of this wavefront: half of every tile, or every other tile
  const int kb0 = key_split(LAYOUT) ? half : 0;              // first 32-key block of a tile

  // ---- workgroup -> (row tile, batch, KV head, split).  Hardware deals consecutive workgroup ids round-robin
  // to the 8 XCDs; each XCD gets a contiguous range of units so that row tiles sharing K/V share an L2.
  const int nwg = gridDim.x;
  const int nrows = p.G * p.Bq;
  int rt;
  uint32_t rest;
  if constexpr (MODE == kPassDensePaged) {
    // ragged sequences: contiguous ranges would give the XCDs unequal work; deal the units round-robin
    const uint32_t j = blockIdx.x >> 3, xcd = blockIdx.x & 7;
    const uint32_t jq = fastdiv(j, p.div_rowtiles);
    rt = (int)(j - jq * p.div_rowtiles.d);
    rest = jq * 8 + xcd;
    if (rest >= (uint32_t)(p.B * p.Hkv * p.nsplit)) return;   // workgroup-uniform
  } else {
    const int bid = blockIdx.x, q8 = nwg / 8, r8 = nwg % 8;
    const int xcd = bid % 8, j = bid / 8;
    int w = (xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8) + j;
    // biased cut (the host sets it only for one row tile, an even split count and a grid that is a multiple of 8):
    // the two XCDs of a pair take alternate work items of the pair's contiguous range, so that even-numbered splits
    // run on even XCDs and odd-numbered ones on odd XCDs
    if (p.xcd_bias) w = (xcd >> 1) * (2 * q8) + 2 * j + (xcd & 1);
    if constexpr (MODE == kPassDenseHeads) {
      if (p.div_rowtiles.d > 1) w = bid;     // whole heads drop out: deal a head's row tiles over the XCDs
    }
    rest = fastdiv((uint32_t)w, p.div_rowtiles);
    rt = w - (int)(rest * p.div_rowtiles.d);
  }
  const uint32_t unit = rest;
  const uint32_t r2 = fastdiv(rest, p.div_nsplit);
  const int split = (int)(rest - r2 * p.div_nsplit.d);
  rest = r2;
  int b = (int)fastdiv(rest, p.div_hkv);
  const int kvh = (int)(rest - (uint32_t)b * p.div_hkv.d);
  if constexpr (MODE == kPassDensePaged) {
    if (p.seq_order != nullptr) {
      b = sload(p.seq_order, b);
    } else if (p.order_inline) {
      // small batch: this workgroup finds the sequence with the b-th longest prefix itself (ties: lower index
      // first): lengths to LDS, one rank per thread, the thread whose sequence has rank b publishes it
      int* lens_s = (int*)ring;
      __shared__ int chosen;
      for (int i = threadIdx.x; i < p.B; i += C::THREADS) lens_s[i] = p.prefix_lens[i];
      __syncthreads();
      for (int i = threadIdx.x; i < p.B; i += C::THREADS) {
        const int li = lens_s[i];
        int rank = 0;
        for (int j = 0; j < p.B; ++j) {
          const int lj = lens_s[j];
          rank += (lj > li || (lj == li && j < i)) ? 1 : 0;
        }
        if (rank == b) chosen = i;
      }
      __syncthreads();
      b = __builtin_amdgcn_readfirstlane(chosen);
      __syncthreads();                       // the ring is free again before the first direct-to-LDS load
    }
  }
  const int bk = b * p.Hkv + kvh;
  int nkeys = p.nkeys;
  if constexpr (MODE == kPassDensePaged) nkeys = min(p.nkeys, max(0, sload(p.prefix_lens, b)));   // this sequence's prefix

  const int row0 = rt * C::ROWS;                               // first group-flattened row of the workgroup
  const int row = row0 + rg * 32 + l32;
  const bool row_ok = row < nrows;
  const size_t grow_base = (size_t)(b * p.Hq + kvh * p.G) * p.Bq;
  const size_t grow = grow_base + row;
  bool head_active = true;
  if constexpr (MODE == kPassDenseHeads) {
    head_active = row_ok && p.head_on[b * p.Hq + kvh * p.G + row / p.Bq] != 0;
    if (!__syncthreads_or(head_active ? 1 : 0)) return;
  }
  // contiguous cache: this KV head's [nkeys, D] slab; paged cache: the pool (tiles add their page offset)
  const unsigned char* __restrict__ Kg =
      (const unsigned char*)p.k + ((MODE == kPassDensePaged) ? (size_t)0 : (size_t)bk * nkeys * C::ROWB);
  const unsigned char* __restrict__ Vg =
      (const unsigned char*)p.v + ((MODE == kPassDensePaged) ? (size_t)0 : (size_t)bk * nkeys * C::ROWB);

  // ---- tile list of this workgroup: a contiguous range of the pass's tile list, visited in rotated order
  // (workgroups that run in lockstep would otherwise read the same offset of their chunks, i.e. the same
  // channels, at once; row tiles of one unit share the offset so that one L2 serves them)
  int tpb = 1, total;
  if constexpr (MODE == kPassSparseReuse) {
    tpb = p.key_block / C::KT;
    total = sload(p.union_cnt, bk) * tpb;
  } else {
    total = (nkeys + C::KT - 1) / C::KT;
  }
  TileRange tr = p.xcd_bias ? biased_range(total, p.div_bias, split) : split_range(total, p.div_nsplit, split);
  const uint32_t rsrc = (p.div_rowtiles.d == 1) ? blockIdx.x : unit;
  if constexpr (LAYOUT == kTileSplit) {
    // as the register-staged refresh pass cuts them, so that the running references start from the same tiles and results
    // stay the same up to fp32 sums: the last split is blk_cost tiles (at most half a split, 3 for a block of one tile) shorter
    tr = split_range(total + p.blk_cost, p.div_nsplit, split);
    tr.begin = min(tr.begin, total);
    tr.end = min(tr.end, total);
  }
  int ntiles = tr.end - tr.begin;
  // PARTS.  A weight is rounded to bf16 against the running reference, so the tile a reference starts from decides single roundings.
  // Segments fix those tiles whatever the number of workgroups: each has its tiles, its order and its first tile; a workgroup that
  // starts inside one takes its reference from that first tile (streamed once more, nothing accumulated), one that
  // walks into the next starts a new reference there.  Segments are cut and rotated as nsplit = nseg would cut them.
  int seg = 0, seg_begin = 0, seg_len = 1, seg_rot = 0, seg_pos = 0, part_left = 0, ref_at = 0, nref = 0, last_e = 0;
  bool pad_next = false;
  constexpr int kFirst = LAYOUT == kTileSplit ? 2 : 1;          // tiles that start a reference: one for each wavefront half
  int seg_base = 0, seg_rem = 0, seg_q8 = 0;                     // the cut of split_range, and of the grid of nseg splits over the XCDs
  if constexpr (PARTS) {
    const int all = total + (LAYOUT == kTileSplit ? p.blk_cost : 0);
    seg_base = all / p.nseg;
    seg_rem = all - seg_base * p.nseg;
    seg_q8 = (p.B * p.Hkv * p.nseg) >> 3;
  }
  auto seg_range = [&](int i) -> TileRange {
    if (LAYOUT == kKeySplit && p.seg_bias) return biased_range(total, p.div_bias, i);
    const int begin = i * seg_base + min(i, seg_rem);
    return {min(begin, total), min(begin + seg_base + (i < seg_rem ? 1 : 0), total)};
  };
  auto seg_open = [&](int i) {
    const TileRange r = seg_range(i);
    seg = i;
    seg_begin = r.begin;
    seg_len = max(r.end - r.begin, 1);
    // the workgroup that nsplit = nseg would give it, whose number rotates the order
    const uint32_t w = r2 * (uint32_t)p.nseg + (uint32_t)i;
    uint32_t bid;
    if (p.seg_bias) {
      const uint32_t q2 = 2u * (uint32_t)seg_q8, pair = w / q2, r1 = w - pair * q2;
      bid = (r1 >> 1) * 8 + 2 * pair + (r1 & 1);
    } else {
      const uint32_t r8 = (uint32_t)(p.B * p.Hkv * p.nseg) & 7u, lim = r8 * (uint32_t)(seg_q8 + 1);
      const uint32_t from = w < lim ? w : w - lim, q = (uint32_t)seg_q8 + (w < lim ? 1u : 0u), x = from / q;
      bid = (from - x * q) * 8 + (w < lim ? 0u : r8) + x;
    }
    seg_rot = (int)((bid * 13u + (bid >> 5) * 7u) % (uint32_t)seg_len);
  };
  if constexpr (PARTS) {
    auto seg_of = [&](int x) -> int {
      int i = min((int)((float)x * (float)p.nseg / (float)total), p.nseg - 1);
      while (i > 0 && seg_range(i).begin > x) --i;
      while (i + 1 < p.nseg && seg_range(i).end <= x) ++i;
      return i;
    };
    auto cut = [&](int i) -> int {                               // where piece i of the walk begins
      if (i >= p.nsplit) return total;
      const int x = split_range(total, p.div_nsplit, i).begin;
      if (LAYOUT == kKeySplit) return x;
      const int b0 = seg_range(seg_of(x)).begin;                 // pairs of tiles stay together
      return b0 + ((x - b0) & ~1);
    };
    const int begin = cut(split), end = cut(split + 1);
    part_left = end - begin;
    const int first = seg_of(begin);
    seg_open(first);
    seg_pos = begin - seg_begin;
    nref = seg_pos > 0 ? kFirst : 0;
    ntiles = nref + part_left;
    if (LAYOUT == kTileSplit) {
      // a segment's last tile alone: the next one starts with a new pair
      for (int i = first; i + 1 < p.nseg; ++i) {
        const TileRange r = seg_range(i);
        if (r.end >= end) break;
        ntiles += (r.end - r.begin) & 1;
      }
    }
  }
  auto next_entry = [&]() -> TileRaw {
    TileRaw r;
    r.word = 0;
    if (ref_at < nref) {
      int j = ref_at++ + seg_rot;
      if (j >= seg_len) j -= seg_len;
      r.e = seg_begin + j;
      r.mask = kSegReference;
    } else if (pad_next) {
      pad_next = false;
      r.e = last_e;
      r.mask = kSegPad;
    } else {
      int j = seg_pos + seg_rot;
      if (j >= seg_len) j -= seg_len;
      r.e = last_e = seg_begin + j;
      r.mask = seg_pos < kFirst ? kSegFirst : 0u;
      ++seg_pos;
      --part_left;
      if (seg_pos >= seg_len && part_left > 0) {
        pad_next = LAYOUT == kTileSplit && (seg_len & 1) != 0;
        seg_open(seg + 1);
        seg_pos = 0;
      }
    }
    return r;
  };
  const int rot = PARTS || MODE == kPassInternal || ntiles <= 0 ? 0 : (int)((rsrc * 13u + (rsrc >> 5) * 7u) % (unsigned)ntiles);
  const uint32_t* __restrict__ bmask = p.blk_mask ? p.blk_mask + (size_t)bk * p.nblk : nullptr;
  const int32_t* __restrict__ ulist = p.union_list ? p.union_list + (size_t)bk * p.nblk : nullptr;
  const uint32_t* __restrict__ umask = p.union_mask ? p.union_mask + (size_t)bk * p.nblk : nullptr;
  auto tile_raw = [&](int i) -> TileRaw {        // i-th tile of this workgroup (asked for in order): table lookups only
    if constexpr (PARTS) return next_entry();
    int j = i + rot;
    if (j >= ntiles) j -= ntiles;
    TileRaw r;
    r.e = tr.begin + j;
    r.word = 0;
    r.mask = 0xffffffffu;
    if constexpr (MODE == kPassSparseReuse) {
      const int blk_i = (int)fastdiv((uint32_t)r.e, p.div_tpb);     // entry of the union list
      r.word = sload(ulist, blk_i);
      r.mask = (uint32_t)sload(umask, blk_i);
    } else if constexpr (MODE == kPassSparseRefresh) {
      r.mask = (uint32_t)sload(bmask, (int)fastdiv((uint32_t)r.e, p.div_tpb));
    } else if constexpr (MODE == kPassDensePaged) {
      r.word = sload(p.block_table + (size_t)b * p.max_pages, (int)fastdiv((uint32_t)(r.e * C::KT), p.div_page));
    }
    return r;
  };
  auto tile_desc = [&](const TileRaw& r) -> TileDesc {
    TileDesc d;
    d.mask = r.mask;
    d.k0 = (MODE == kPassSparseReuse)
               ? r.word * p.key_block + C::KT * (r.e - (int)(fastdiv((uint32_t)r.e, p.div_tpb) * p.div_tpb.d))
               : r.e * C::KT;
    if constexpr (MODE == kPassDensePaged) {
      const uint32_t slot = fastdiv((uint32_t)d.k0, p.div_page);
      const int page = min(max(r.word, 0), p.num_pages - 1);       // clamped into the pool
      const int in_page = d.k0 - (int)(slot * p.div_page.d);
      const size_t off = (((size_t)page * p.Hkv + kvh) * p.page_size + in_page) * C::ROWB;
      d.kt = Kg + off;
      d.vt = Vg + off;
    } else {
      // a list entry past the end of the keys (reuse pass, short last key block) is skipped by the compute; its
      // loads, issued all the same so that every tile counts the same number of loads, read the head's first keys
      const int kload = (MODE == kPassSparseReuse && d.k0 >= nkeys) ? 0 : d.k0;
      d.kt = Kg + (size_t)kload * C::ROWB;
      d.vt = Vg + (size_t)kload * C::ROWB;
    }
    return d;
  };

  // ---- direct-to-LDS load slots of this lane: operand chunk pidx = (j*8 + wave)*64 + lane lives at LDS row
  // pidx / CPR, chunk position pidx % CPR, and holds logical chunk (position - rotation(row)) of that row.
  const uint32_t ring_base = (uint32_t)(uintptr_t)ring;
  int ld_row[C::NLOAD];
  uint32_t off_k[C::NLOAD], off_v[C::NLOAD];     // byte offsets inside a full tile
  int ck[C::NLOAD], cv[C::NLOAD];
#pragma unroll
  for (int j = 0; j < C::NLOAD; ++j) {
    const int pidx = (j * C::NW + wave) * 64 + lane;
    const int r = pidx / C::CPR, pc = pidx % C::CPR;
    ld_row[j] = r;
    ck[j] = (pc - C::rot_k(r)) & (C::CPR - 1);
    cv[j] = (pc - C::rot_v(r)) & (C::CPR - 1);
    off_k[j] = (uint32_t)(r * C::ROWB + ck[j] * 16);
    off_v[j] = (uint32_t)(r * C::ROWB + cv[j] * 16);
  }
  // (first key, mask) of the tiles in the ring, oldest first: [0] is the tile computed in this iteration
  int qk0[C::NS];
  uint32_t qmask[C::NS];
#pragma unroll
  for (int i = 0; i < C::NS; ++i) { qk0[i] = 0; qmask[i] = 0u; }
  auto issue_tile = [&](int i, const TileDesc& d) {
    const uint32_t sbase = ring_base + (uint32_t)(i % C::NS) * C::STAGE + wave * 1024;
    const int nvalid = nkeys - d.k0;
    if (nvalid >= C::KT) {
#pragma unroll
      for (int j = 0; j < C::NLOAD; ++j) dma16(d.kt, off_k[j], sbase + j * C::LSTEP);
#pragma unroll
      for (int j = 0; j < C::NLOAD; ++j) dma16(d.vt, off_v[j], sbase + C::OPB + j * C::LSTEP);
    } else {
      // ragged tile: rows past the end read the last key (in bounds; their scores are masked); an entry past the
      // end of the keys reads one row of the address tile_desc gave it
      const int last = max(nvalid, 1) - 1;
#pragma unroll
      for (int j = 0; j < C::NLOAD; ++j)
        dma16(d.kt, (uint32_t)(min(ld_row[j], last) * C::ROWB + ck[j] * 16), sbase + j * C::LSTEP);
#pragma unroll
      for (int j = 0; j < C::NLOAD; ++j)
        dma16(d.vt, (uint32_t)(min(ld_row[j], last) * C::ROWB + cv[j] * 16), sbase + C::OPB + j * C::LSTEP);
    }
  };

  // ---- prologue: the query rows go through the last ring stage(s), then the first tiles; everything is in
  // flight before the first wait.
  {
    const unsigned char* qg = (const unsigned char*)p.q + (grow_base + row0) * C::ROWB;
    const int qvalid = nrows - row0;                     // >= 1
    const uint32_t qbase = ring_base + (uint32_t)(C::NS - C::QSTAGES) * C::STAGE + wave * 1024;
#pragma unroll
    for (int part = 0; part < C::QPARTS; ++part)         // 64 rows at a time, each laid out like a K operand
#pragma unroll
      for (int j = 0; j < C::NLOAD; ++j) {
        const int r = min(64 * part + ld_row[j], qvalid - 1);
        dma16(qg, (uint32_t)(r * C::ROWB + ck[j] * 16), qbase + part * C::OPB + j * C::LSTEP);
      }
  }
  constexpr int kPre = (AHEAD < C::NS - C::QSTAGES) ? AHEAD : C::NS - C::QSTAGES;   // tiles issued while the queries sit in the ring
  {
    int pre = 0;
#pragma unroll
    for (int i = 0; i < kPre; ++i)
      if (i < ntiles) {
        const TileDesc d = tile_desc(tile_raw(i));
        issue_tile(i, d);
        qk0[i] = d.k0;
        qmask[i] = d.mask;
        ++pre;
      }
    wait_tiles<C::LPT>(pre);                             // the query loads were issued first
  }
  __syncthreads();
  bf16x8 qreg[C::NKS];
  {
    const int r = rg * 32 + l32;
    const unsigned char* qs = ring + (C::NS - C::QSTAGES) * C::STAGE + (r / 64) * C::OPB + (r % 64) * C::ROWB;
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks)
      qreg[ks] = *(const bf16x8*)(qs + ((2 * ks + h + C::rot_k(r % 64)) & (C::CPR - 1)) * 16);
  }
  if constexpr (kPre < AHEAD) {
    // the queries took more than the last stage: the remaining start-up tiles go out once everyone has read them
    __syncthreads();
#pragma unroll
    for (int i = kPre; i < AHEAD; ++i)
      if (i < ntiles) {
        const TileDesc d = tile_desc(tile_raw(i));
        issue_tile(i, d);
        qk0[i] = d.k0;
        qmask[i] = d.mask;
      }
  }
  // table words of the next tile to be issued, fetched one iteration ahead (lookups off the critical path; one wavefront per row
  // group: no table, and computing the tile ahead only lengthens the loop)
  constexpr int NNEXT = kPairs ? 2 : 1;
  TileRaw rnext[NNEXT];
#pragma unroll
  for (int u = 0; u < NNEXT; ++u) {
    rnext[u].e = 0; rnext[u].word = 0; rnext[u].mask = 0u;
    if (kHalves && AHEAD + u < ntiles) rnext[u] = tile_raw(AHEAD + u);
  }

  // per-lane LDS read addresses inside a stage
  uint32_t kaddr[C::NKS], vaddr[C::NDB];
#pragma unroll
  for (int ks = 0; ks < C::NKS; ++ks)
    kaddr[ks] = (uint32_t)(l32 * C::ROWB + ((2 * ks + h + C::rot_k(l32)) & (C::CPR - 1)) * 16);
  {
    const int i16 = lane & 15, blk1 = (lane >> 4) & 1;
    const int rrow = 4 * h + (i16 >> 2);                 // row of this lane inside an 8-key group
#pragma unroll
    for (int db = 0; db < C::NDB; ++db) {
      const int c = 4 * db + 2 * blk1 + ((i16 & 3) >> 1);
      const int pc = (c + C::rot_v(rrow)) & (C::CPR - 1);   // 8-key groups start at multiples of 8: same rotation
      vaddr[db] = (uint32_t)(rrow * C::ROWB + pc * 16 + (i16 & 1) * 8);
    }
  }

  WaveAcc<C::NDB> accs[NSETS];
#pragma unroll
  for (int i = 0; i < NSETS; ++i) accs[i].init();
  WaveAcc<C::NDB>& acc = accs[0];
  const uint32_t my_bit = 1u << ((row_ok ? row : 0) / p.Bq);

  auto lane_on_of = [&](uint32_t mask, int set) -> bool {
    if constexpr (MODE == kPassDenseHeads) return head_active;
    else if constexpr (MODE == kPassSparseReuse) return row_ok && (mask & my_bit) != 0u;
    else if constexpr (MODE == kPassSparseRefresh) return row_ok && (((mask & my_bit) != 0u) == (set == 0));
    else return true;
  };
  constexpr bool kMasked = (MODE == kPassDenseHeads || MODE == kPassSparseReuse || MODE == kPassSparseRefresh);
  // issue of tile t + AHEAD + u (into a stage every wavefront has left for good), then the lookups of the tile that
  // follows in this slot; the queue then holds tiles t .. t + AHEAD + u
  auto refill = [&](int t, int u) {
    if (t + AHEAD + u < ntiles) {
      const TileDesc d = tile_desc(kHalves ? rnext[u] : tile_raw(t + AHEAD + u));
      issue_tile(t + AHEAD + u, d);
      qk0[AHEAD + u] = d.k0;
      qmask[AHEAD + u] = d.mask;
      if (kHalves && t + AHEAD + u + NNEXT < ntiles) rnext[u] = tile_raw(t + AHEAD + u + NNEXT);
    }
  };
  auto advance = [&]() {
#pragma unroll
    for (int i = 0; i + NNEXT < C::NS; ++i) {
      qk0[i] = qk0[i + NNEXT];
      qmask[i] = qmask[i + NNEXT];
    }
  };
  // one tile of a wavefront whose row group is shared by two (key halves)
  bool seg_waits = false;          // PARTS: the segment's first tile has no key for this half (the ragged last tile): the next one counts
  auto half_tile = [&](const unsigned char* stage, int k0, uint32_t mask) __attribute__((always_inline)) {
    if constexpr (PARTS) {
      if (mask & kSegPad) return;
    }
    const int nvalid = min(C::KT, nkeys - k0);
    const bool fresh = PARTS && ((mask & kSegFirst) != 0u || seg_waits);
    if constexpr (PARTS) seg_waits = fresh && nvalid <= 32 * kb0;
    if constexpr (MODE == kPassSparseReuse) {
      if (nvalid <= 0) return;                               // a list entry past the end of the keys
    }
    bool on[NSETS];
    bool any_on = false;
#pragma unroll
    for (int i = 0; i < NSETS; ++i) {
      on[i] = lane_on_of(mask, i);
      any_on = any_on || on[i];
    }
    if (kMasked && !__any(any_on)) return;
    if constexpr (D == 128 && NSETS > 1 && NRG == 4) {
      // the one form with 256 registers and two accumulator sets: written out here, four of them spill.  With fewer row
      // groups, which have registers to spare, the call is 4 to 7 % slower (16 rows per KV head, batch 4, 16752 keys, refresh
      // 76 against 79 us)
      sets_tile<D, NSETS, C::NKB>(accs, on, qreg, stage, kaddr, vaddr, kb0, p.scale_log2, nvalid, h);
    } else {
      f32x16 s[C::NKB];
      tile_scores<D, C::NKB>(s, qreg, stage, kaddr, kb0);
      if constexpr (PARTS) {
        if (mask & kSegReference) {
          tile_reference<C::NDB, C::NKB>(acc, s, kb0, p.scale_log2, nvalid, h);
          return;
        }
      }
#pragma unroll
      for (int i = 0; i < NSETS; ++i) {
        if (NSETS > 1 && !__any(on[i])) continue;
        tile_softmax_pv<D, C::NKB>(accs[i], s, stage, vaddr, kb0, p.scale_log2, on[i], nvalid, h, fresh);
      }
    }
  };

  // two tiles whose key halves this wavefront owns: as half_tile for one and then the other, with the same results bit for
  // bit, but the scores, the cross-lane maxima and the weights of both in one go
  auto two_tiles = [&](const unsigned char* stage_a, int k0a, uint32_t mask_a, const unsigned char* stage_b, int k0b,
                       uint32_t mask_b) __attribute__((always_inline)) {
    if constexpr (PARTS) {
      if ((mask_a | mask_b) != 0u || seg_waits) {
        half_tile(stage_a, k0a, mask_a);
        half_tile(stage_b, k0b, mask_b);
        return;
      }
    }
    const int nva = min(C::KT, nkeys - k0a), nvb = min(C::KT, nkeys - k0b);
    bool ona[NSETS], onb[NSETS];
    bool any_a = false, any_b = false;
#pragma unroll
    for (int i = 0; i < NSETS; ++i) {
      ona[i] = lane_on_of(mask_a, i);
      onb[i] = lane_on_of(mask_b, i);
      any_a = any_a || ona[i];
      any_b = any_b || onb[i];
    }
    const bool need_a = (!kMasked || __any(any_a)) && (MODE != kPassSparseReuse || nva > 0);
    const bool need_b = (!kMasked || __any(any_b)) && (MODE != kPassSparseReuse || nvb > 0);
    if (!(need_a && need_b)) {
      if (need_a) half_tile(stage_a, k0a, mask_a);
      if (need_b) half_tile(stage_b, k0b, mask_b);
      return;
    }
    f32x16 s[2];
    two_scores<D>(s, qreg, stage_a, stage_b, kaddr, kb0);
#pragma unroll
    for (int i = 0; i < NSETS; ++i) {
      const bool set_a = NSETS == 1 || __any(ona[i]), set_b = NSETS == 1 || __any(onb[i]);
      if (set_a && set_b) {
        two_softmax_pv<D>(accs[i], s, stage_a, stage_b, vaddr, kb0, p.scale_log2, ona[i], onb[i], nva, nvb, h);
      } else if (set_a || set_b) {
        f32x16 s1[1] = {set_a ? s[0] : s[1]};
        tile_softmax_pv<D, 1>(accs[i], s1, set_a ? stage_a : stage_b, vaddr, kb0, p.scale_log2, set_a ? ona[i] : onb[i],
                              set_a ? nva : nvb, h);
      }
    }
  };

  if constexpr (!kHalves) {
    for (int t = 0; t < ntiles; t += 2) {
      wait_tiles<C::LPT>(min(AHEAD - 2, max(ntiles - 2 - t, 0)));   // tiles issued after tile t+1 so far
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u) refill(t, u);
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (t + u < ntiles) {
          const unsigned char* stage = ring + ((t + u) % C::NS) * C::STAGE;
          f32x16 s[C::NKB];
          tile_scores<D, C::NKB>(s, qreg, stage, kaddr, kb0);
          tile_softmax_pv<D, C::NKB>(acc, s, stage, vaddr, kb0, p.scale_log2, true, min(C::KT, nkeys - qk0[u]), h);
        }
      advance();
    }
  } else if constexpr (LAYOUT == kTileSplit) {
    for (int t = 0; t < ntiles; t += 2) {
      wait_tiles<C::LPT>(min(AHEAD - 2, max(ntiles - 2 - t, 0)));   // tiles issued after tile t+1 so far
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u) refill(t, u);
      const int k0 = half ? qk0[1] : qk0[0];
      const uint32_t mask = half ? qmask[1] : qmask[0];
      if constexpr (MODE == kPassInternal) {
        if (t == 0 && half) {                                        // one reference for both streams, that of the first tile
          f32x16 s[C::NKB];
          tile_scores<D, C::NKB>(s, qreg, ring, kaddr, kb0);
          tile_reference<C::NDB, C::NKB>(acc, s, kb0, p.scale_log2, min(C::KT, nkeys - qk0[0]), h);
        }
      }
      advance();
      if (t + half < ntiles) half_tile(ring + ((t + half) % C::NS) * C::STAGE, k0, mask);
    }
  } else if constexpr (kPairs) {
    for (int t = 0; t < ntiles; t += 2) {
      wait_tiles<C::LPT>(min(AHEAD - 2, max(ntiles - 2 - t, 0)));
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u) refill(t, u);
      const int k0a = qk0[0], k0b = qk0[1];
      const uint32_t mask_a = qmask[0], mask_b = qmask[1];
      advance();
      const unsigned char* stage_a = ring + (t % C::NS) * C::STAGE;
      const unsigned char* stage_b = ring + ((t + 1) % C::NS) * C::STAGE;
      if (t + 1 < ntiles) two_tiles(stage_a, k0a, mask_a, stage_b, k0b, mask_b);
      else half_tile(stage_a, k0a, mask_a);
    }
  } else {
    for (int t = 0; t < ntiles; ++t) {
      wait_tiles<C::LPT>(min(AHEAD - 1, ntiles - 1 - t));      // tiles issued after tile t so far
      __syncthreads();
      refill(t, 0);
      const int k0 = qk0[0];
      const uint32_t mask = qmask[0];
      advance();
      half_tile(ring + (t % C::NS) * C::STAGE, k0, mask);
    }
  }

  // Output column blocks this wavefront finishes and stores: all of them, or, where two wavefronts share a row group, half: they
  // exchange halves, so that both take part in the merge and in the stores (the wavefront of key half 0 keeps the lower column
  // blocks, the other one the upper ones).
  constexpr int NDBK = kHalves ? C::NDB / 2 : C::NDB;
  const int db_keep = half * NDBK;
  if constexpr (kHalves) {
    // ---- merge the two key halves through LDS.  Record per (set, row group, key half): the NDBK column blocks the
    // wavefront gives away, then its m and l; [register][lane] so that neighbouring lanes hit neighbouring banks.
    constexpr int REC = NDBK * 16 + 2;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NSETS; ++i) {
      float* mine = (float*)ring + (((size_t)i * NRG + rg) * 2 + half) * REC * 64 + lane;
#pragma unroll
      for (int db = 0; db < NDBK; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          // static register indices: select between the two halves instead of indexing by half
          mine[(db * 16 + r) * 64] = half ? accs[i].o[db][r] : accs[i].o[NDBK + db][r];
        }
      mine[(NDBK * 16) * 64] = accs[i].m;
      mine[(NDBK * 16 + 1) * 64] = accs[i].l;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NSETS; ++i) {
      const float* other = (const float*)ring + (((size_t)i * NRG + rg) * 2 + (half ^ 1)) * REC * 64 + lane;
      WaveAcc<C::NDB>& a = accs[i];
      const float mo = other[(NDBK * 16) * 64], lo = other[(NDBK * 16 + 1) * 64];
      // both wavefronts of the pair evaluate the same expressions on (key half 0, key half 1) in that order
      const float m0 = half ? mo : a.m, m1 = half ? a.m : mo;
      const float l0 = half ? lo : a.l, l1 = half ? a.l : lo;
      const float M = fmaxf(m0, m1);
      const float Mu = (M == -INFINITY) ? 0.f : M;
      const float w0 = __builtin_amdgcn_exp2f(m0 - Mu), w1 = __builtin_amdgcn_exp2f(m1 - Mu);
      const float ws = half ? w1 : w0, wo = half ? w0 : w1;
#pragma unroll
      for (int db = 0; db < NDBK; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float x = other[(db * 16 + r) * 64];
          // kept block = lower ones for key half 0, upper ones for key half 1; result parked in o[db]
          const float own = half ? a.o[NDBK + db][r] : a.o[db][r];
          a.o[db][r] = half ? (x * wo + own * ws) : (own * ws + x * wo);
        }
      a.l = l0 * w0 + l1 * w1;
      a.m = M;
    }
  }

  // ---- epilogue
  const float l_row = sum_halves(acc.l);
  if constexpr (MODE == kPassInternal) {
    // Eq. 8-9 with the cached pair expressed through (o, m, lse): A_out e^{L_out-M} = o e^{m-M}
    if (!row_ok) return;
    const bool has_ext = p.ext_o != nullptr;
    float me2 = -INFINITY, le = 0.f;
    f32x4 e[NDBK * 4];
    if (has_ext) {
#pragma unroll
      for (int i = 0; i < NDBK * 4; ++i) e[i] = *(const f32x4*)(p.ext_o + grow * D + 32 * (db_keep + i / 4) + 8 * (i % 4) + 4 * h);
      const float em = p.ext_m[grow], el = p.ext_lse[grow];
      if (el != -INFINITY) {
        me2 = em * kLog2e;
        le = exp2f((el - em) * kLog2e);
      }
    }
    const float M2 = fmaxf(me2, acc.m);
    const float Mu = (M2 == -INFINITY) ? 0.f : M2;
    const float we = exp2f(me2 - Mu), wi = exp2f(acc.m - Mu);
    const float den = le * we + l_row * wi;
    const float inv = den > 0.f ? 1.f / den : 0.f;
    __bf16* out = (__bf16*)p.out + grow * D;
#pragma unroll
    for (int db = 0; db < NDBK; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4 x = has_ext ? e[db * 4 + q4] : f32x4{0.f, 0.f, 0.f, 0.f};
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (acc.o[db][4 * q4 + i] * wi + x[i] * we) * inv;
        u32x2 pk;
        pk.x = pack_bf16x2(r[0], r[1]);
        pk.y = pack_bf16x2(r[2], r[3]);
        *(u32x2*)(out + 32 * (db_keep + db) + 8 * q4 + 4 * h) = pk;
      }
    if (p.lse_out != nullptr && h == 0 && half == 0) p.lse_out[grow] = den > 0.f ? (M2 + log2f(den)) * kLn2 : -INFINITY;
  } else {
    if (p.direct) {
      // single split: this is the final partial.  Same conversion as the split combine: m is rounded when
      // converted to natural-log units, o is rescaled to the reference consumers recover from it.
      if (!(row_ok && head_active)) return;
      float m_nat = -INFINITY, L = -INFINITY, adj = 0.f;
      if (l_row > 0.f) {
        m_nat = acc.m * kLn2;
        adj = exp2f(acc.m - m_nat * kLog2e);
        L = (acc.m + log2f(l_row)) * kLn2;
      }
#pragma unroll
      for (int db = 0; db < NDBK; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int d0 = 32 * (db_keep + db) + 8 * q4 + 4 * h;
          f32x4 o4 = {acc.o[db][4 * q4] * adj, acc.o[db][4 * q4 + 1] * adj, acc.o[db][4 * q4 + 2] * adj,
                      acc.o[db][4 * q4 + 3] * adj};
          *(f32x4*)(p.ws_o + grow * D + d0) = o4;
        }
      if (h == 0 && half == 0) {
        p.ws_m[grow] = m_nat;
        p.ws_l[grow] = L;
      }
      return;
    }
    if (!row_ok) return;
    const size_t wrow = ((size_t)(split * p.B + b) * p.Hkv + kvh) * nrows + row;
#pragma unroll
    for (int i = 0; i < NSETS; ++i) {
      float* __restrict__ w_o = i ? p.ws_o2 : p.ws_o;
      float* __restrict__ w_m = i ? p.ws_m2 : p.ws_m;
      float* __restrict__ w_l = i ? p.ws_l2 : p.ws_l;
      const WaveAcc<C::NDB>& a = accs[i];
      const float l_i = (i == 0) ? l_row : sum_halves(a.l);
#pragma unroll
      for (int db = 0; db < NDBK; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int d0 = 32 * (db_keep + db) + 8 * q4 + 4 * h;
          f32x4 o4 = {a.o[db][4 * q4], a.o[db][4 * q4 + 1], a.o[db][4 * q4 + 2], a.o[db][4 * q4 + 3]};
          // streaming store: read next by another kernel, never again by this one (measured: faster than staging
          // the rows through LDS for whole-row stores, and faster than write-back stores)
          __builtin_nontemporal_store(o4, (f32x4*)(w_o + wrow * D + d0));
        }
      if (h == 0 && half == 0) {
        w_m[wrow] = a.m;
        w_l[wrow] = l_i;
      }
    }
  }
}

template <int D, int MODE, int LAYOUT, int NRG>
__global__ __launch_bounds__(LAYOUT == kRowPair ? RCfg<D>::THREADS : LAYOUT == kRowPairShort ? 512 : 2 * NRG * 64, 1) void attn_stream_kernel(const PassParams p) {
  extern __shared__ __align__(16) unsigned char ring[];
  if constexpr (LAYOUT == kRowPair) rows_pass<D, MODE>(p, ring);
  else halves_pass<D, MODE, whole_layout(LAYOUT), NRG, in_parts(LAYOUT)>(p, ring);
}

template <int D, int MODE, int LAYOUT, int NRG = 4>
hipError_t launch_stream(const PassParams& p, hipStream_t s) {
  using C = std::conditional_t<LAYOUT == kRowPair, RCfg<D>, SCfg<D, whole_layout(LAYOUT), (MODE == kPassSparseRefresh) ? 2 : 1, NRG>>;
  // row pairs: the shortest range has to hold what is loaded ahead (the routes here ask for more); per-head refresh: two splits
  // share a range
  if (LAYOUT == kRowPair && (p.nkeys + C::KT - 1) / C::KT < kRowsTiles * (MODE == kPassDenseHeads || MODE == kPassRefreshFused ? (p.nsplit + 1) / 2 : p.nsplit))
    return hipErrorInvalidValue;
  if (MODE == kPassRefreshFused) {
    // the last range, blk_cost tiles shorter, and the block's own
    const int pairs = p.nsplit / 2, tiles = (p.nkeys + C::KT - 1) / C::KT, all = tiles + p.blk_cost;
    if (p.nsplit % 2 != 0 || pairs < 1 || all / pairs - p.blk_cost < kRowsTiles || (p.k2 != nullptr && (p.Bq + C::KT - 1) / C::KT < kRowsTiles)) return hipErrorInvalidValue;
  }
  auto kern = attn_stream_kernel<D, MODE, LAYOUT, NRG>;
  static LdsLimit lim;
  hipError_t e = raise_lds_limit(kern, C::LDS, lim, C::LDS);
  if (e != hipSuccess) return e;
  const int nrows = p.G * p.Bq;
  const int ntile_rows = (nrows + C::ROWS - 1) / C::ROWS;
  long long nwg = (long long)p.B * p.Hkv * ntile_rows * p.nsplit;
  if (MODE == kPassDensePaged) nwg = (((long long)p.B * p.Hkv * p.nsplit + 7) / 8) * 8 * ntile_rows;
  if (MODE == kPassDenseHeads && LAYOUT == kRowPair) nwg = (long long)p.B * (p.heads_cap * p.nsplit + p.Hkv) * ntile_rows;
  if (MODE == kPassRefreshFused && p.k2 != nullptr) nwg += (long long)p.B * p.Hkv * ntile_rows * 2;
  if (nwg >= (1ll << 31)) return hipErrorInvalidValue;
  PassParams q = p;
  if (MODE == kPassDensePaged) q.div_page = make_fastdiv((uint32_t)p.page_size);
  q.div_tpb = make_fastdiv((uint32_t)((MODE == kPassDenseHeads && LAYOUT == kRowPair) ? p.Bq : p.key_block > 0 ? p.key_block / kKeyTile : 1));
  {
    // long streams only: below 64 tiles per split a 1/64 bias rounds away
    const int tiles = (p.nkeys + kKeyTile - 1) / kKeyTile;
    auto biased = [&](int n, long long wgs) {
      return key_split(whole_layout(LAYOUT)) && (MODE == kPassDense || MODE == kPassSparseRefresh) && ntile_rows == 1 && n % 2 == 0 &&
             wgs % 8 == 0 && tiles >= 64 * n && (long long)tiles * 64 * n < (1ll << 31);
    };
    if constexpr (in_parts(LAYOUT)) {
      const long long segs = (long long)p.B * p.Hkv * p.nseg;
      if (ntile_rows != 1 || p.nseg < 1 || tiles < 8 * p.nseg || tiles < 8 * p.nsplit || segs < 8 || segs >= (1ll << 31)) return hipErrorInvalidValue;
      q.seg_bias = biased(p.nseg, segs) ? 1 : 0;
      q.xcd_bias = 0;
      q.div_bias = make_fastdiv(64u * (uint32_t)p.nseg);
    } else {
      q.xcd_bias = biased(p.nsplit, nwg) ? 1 : 0;
      q.div_bias = make_fastdiv(64u * (uint32_t)p.nsplit);
    }
  }
  q.div_rowtiles = make_fastdiv((uint32_t)ntile_rows);
  q.div_nsplit = make_fastdiv((uint32_t)p.nsplit);
  q.div_hkv = make_fastdiv((uint32_t)p.Hkv);
  launch_attn_kernel(kern, dim3((unsigned)nwg), dim3(C::THREADS), C::LDS, s, q);
  return hipGetLastError();
}

// key-split layout with as many 32-row groups per workgroup as the KV group has rows for
template <int D, int MODE>
hipError_t launch_key_split(const PassParams& p, hipStream_t s) {
  const int nrows = p.G * p.Bq;
  if constexpr (D == 64 && (MODE == kPassSparseRefresh || MODE == kPassSparseReuse)) {
    // sparse passes with short streams: waiting for pairs of tiles costs more than it saves (32 / 8 heads, 32 rows, a
    // block at 32K keys, 16 tiles per split, 143.8 us single and 146.5 paired; at 48K, 24 tiles, 177.4 and 174.2)
    if (p.nkeys < 24 * kKeyTile * p.nsplit) {
      if (nrows <= 32) return launch_stream<D, MODE, kKeySplitSingle, 1>(p, s);
      if (nrows <= 64) return launch_stream<D, MODE, kKeySplitSingle, 2>(p, s);
      return launch_stream<D, MODE, kKeySplitSingle, 4>(p, s);
    }
  }
  if (nrows <= 32) return launch_stream<D, MODE, kKeySplit, 1>(p, s);
  if (nrows <= 64) return launch_stream<D, MODE, kKeySplit, 2>(p, s);
  return launch_stream<D, MODE, kKeySplit, 4>(p, s);
}

template <int D, int LAYOUT>
hipError_t launch_parts(const PassParams& p, hipStream_t s) {
  const int nrows = p.G * p.Bq;
  if (nrows <= 32) return launch_stream<D, kPassDense, LAYOUT, 1>(p, s);
  if (nrows <= 64) return launch_stream<D, kPassDense, LAYOUT, 2>(p, s);
  return launch_stream<D, kPassDense, LAYOUT, 4>(p, s);
}

// Dense row pairs: 32 rows per wavefront (kRowPairShort) below 14 tiles per split, 64 (kRowPair) from there on.  External pass, us, 32 against
// 64 rows per wavefront, a ragged last tile: 8 / 64 heads of 32 rows, one split, 8 / 10 / 12 / 14 / 16 / 32 tiles 19.2 / 22.1 / 25.0 / 28.0 /
// 30.9 / 54.1 and 21.0 / 23.3 / 25.3 / 28.2 / 30.1 / 49.5; 16 splits, 8 / 12 / 14 / 24 tiles 26.3 / 32.8 / 35.7 / 50.7 and 27.7 / 32.6 / 35.3 / 47.2;
// batch 16 in 2 splits, all CUs, 8 / 16 tiles 32.9 / 47.7 and 32.5 / 45.1; head_dim 64, 8 heads of 1500 rows, 8 / 12 / 16 / 32 tiles 14.7 / 19.3 /
// 23.8 / 41.5 and 15.8 / 19.7 / 23.5 / 39.2.
constexpr int kShortRowTiles = 14;
inline bool short_row_pairs(const PassParams& p) {
  return (p.nkeys + kKeyTile - 1) / kKeyTile < kShortRowTiles * p.nsplit;
}

// Internal pass in two streams of tiles per row group (kTileSplit, both with the reference of the first tile): the most workgroups that
// are one round, of 1, 2 or 4 row groups; 0: another kernel.  Without splits a pass of this kind leaves most of the chip idle or, by
// the register-staged kernel's column split, computes every score four times (us, there and here, head_dim 64 / 128: one row group, 4
// heads of 700 / 1300 rows 14.1 / 23.9 and 11.2 / 16.9, 16.5 / 27.4 and 14.8 / 22.7; two, 4 heads of 2332 39 and 26, 65 and 36; four, 5 heads of
// 4300 69 and 47, 84 and 67, 16 of 2048 (row pairs there) 40 and 27, 56 and 42).  Short blocks are over before the second stream
// pays: one row group 4 / 5 tiles (3 tiles 7.6 and 8.4), two 6 / 3 (5 tiles at head_dim 64 8.5 and 8.6), four 6 (5 tiles 9.2 and 9.7).
inline int internal_streams(const PassParams& p, int D) {
  if (p.fold_ns > 0 || p.rotate) return 0;      // (rotated: another first tile)
  const long long heads = (long long)p.B * p.Hkv, nrows = (long long)p.G * p.Bq;
  const int tiles = (p.nkeys + kKeyTile - 1) / kKeyTile;
  const int nrg = heads * ((nrows + 31) / 32) <= 256 ? 1 : heads * ((nrows + 63) / 64) <= 256 ? 2 : heads * ((nrows + 127) / 128) <= 256 ? 4 : 0;
  const int least = nrg == 1 ? (D == 64 ? 4 : 5) : nrg == 2 ? (D == 64 ? 6 : 3) : 6;
  return tiles >= least ? nrg : 0;
}

template <int D>
hipError_t launch_stream_d(const PassParams& p, PassMode mode, hipStream_t s) {
  const int nrows = p.G * p.Bq;
  switch (mode) {
    case kPassDense:
      if (dense_row_pairs(nrows, D)) return short_row_pairs(p) ? launch_stream<D, kPassDense, kRowPairShort>(p, s) : launch_stream<D, kPassDense, kRowPair>(p, s);
      if (p.nseg > 0 && p.nseg != p.nsplit) {
        if (p.whole_tiles) return launch_parts<D, kTileSplitParts>(p, s);
        return launch_parts<D, kKeySplitParts>(p, s);
      }
      if (p.whole_tiles) {
        if (nrows <= 32) return launch_stream<D, kPassDense, kTileSplit, 1>(p, s);
        if (nrows <= 64) return launch_stream<D, kPassDense, kTileSplit, 2>(p, s);
        return launch_stream<D, kPassDense, kTileSplit, 4>(p, s);
      }
      return launch_key_split<D, kPassDense>(p, s);
    case kPassDenseHeads:
      // many rows per KV head, with a hint: 3 of 12 heads of 4680 rows against 37440 keys 354 us by the register-staged
      // kernel in 2 splits, 284 us here in 4
      if (p.heads_cap > 0) return launch_stream<D, kPassDenseHeads, kRowPair>(p, s);
      return launch_key_split<D, kPassDenseHeads>(p, s);
    case kPassDensePaged: return launch_key_split<D, kPassDensePaged>(p, s);
    case kPassSparseReuse: return launch_key_split<D, kPassSparseReuse>(p, s);
    case kPassSparseRefresh: return launch_key_split<D, kPassSparseRefresh>(p, s);
    case kPassInternal:
      switch (internal_streams(p, D)) {
        case 1: return launch_stream<D, kPassInternal, kTileSplit, 1>(p, s);
        case 2: return launch_stream<D, kPassInternal, kTileSplit, 2>(p, s);
        case 4: return launch_stream<D, kPassInternal, kTileSplit, 4>(p, s);
        default: return launch_stream<D, kPassInternal, kRowPair>(p, s);
      }
    case kPassRefreshFused: return launch_stream<D, kPassRefreshFused, kRowPair>(p, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Shapes the streaming kernel takes over from the register-staged one: KV groups of up to 128 rows (and the many-row
// shapes of the row-pair layout) whose workgroups stream at least 8 tiles each.
bool stream_bf16_covers(const PassParams& p, int D, PassMode mode) {
  const int nrows = p.G * p.Bq;
  const int tiles = (p.nkeys + kKeyTile - 1) / kKeyTile;
  switch (mode) {
    case kPassDense:
      return (nrows <= 128 || dense_row_pairs(nrows, D)) && tiles >= 8 * p.nsplit;
    case kPassDenseHeads:
      if (p.heads_cap > 0) return true;
      return nrows <= 128 && tiles >= 8 * p.nsplit;
    case kPassDensePaged:
    case kPassSparseReuse:
    case kPassSparseRefresh:
      return nrows <= 128 && tiles >= 8 * p.nsplit;
    case kPassInternal:
      // From 16 tiles on: shorter streams of several rounds of workgroups are the register-staged kernel's, whose start and end cost
      // less (us, there and here: 128 KV heads of 2048 rows, blocks of 512 / 520 / 704 / 900 / 1100 / 1280 117 / 143 / 202 / 322 /
      // 423 / 520 and 134 / 163 / 219 / 330 / 427 / 513; head_dim 64, two rows a key, 512 / 704 / 1100 / 1280 36.4 / 61.5 / 140 /
      // 158 and 39.9 / 65.1 / 141 / 155; one round, 32 heads of 1024 / 1536 rows 40.7 / 53.7 and 38.9 / 52.0).
      return internal_streams(p, D) > 0 || (internal_many_rows(p) && tiles >= 16);
    case kPassRefreshFused: return p.by_parity != 0;
    default: return false;
  }
}

// Name of the instantiation launch_stream_bf16 picks, as a kernel trace prints it (without the namespaces).
int stream_bf16_name(const PassParams& p, int D, PassMode mode, char* buf, size_t n) {
  const bool rp = (mode == kPassDense && dense_row_pairs(p.G * p.Bq, D)) || mode == kPassInternal;
  const int nrows = p.G * p.Bq;
  return snprintf(buf, n, "attn_stream_kernel<%d, %d, %d, %d>", D, (int)mode,
                  !rp ? (int)(mode == kPassDense && p.nseg > 0 && p.nseg != p.nsplit ? kKeySplitParts : kKeySplit) : mode == kPassDense && short_row_pairs(p) ? (int)kRowPairShort : (int)kRowPair,
                  (rp || nrows > 64) ? 4 : nrows > 32 ? 2 : 1);
}

hipError_t launch_stream_bf16(const PassParams& p, int D, PassMode mode, hipStream_t s) {
  return D == 64 ? launch_stream_d<64>(p, mode, s) : launch_stream_d<128>(p, mode, s);
}

}  // namespace fb
