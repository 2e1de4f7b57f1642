// Internal interface between the C-ABI layer (fb_api.hip) and the gfx950 kernels.
// Not installed; the public contract is include/flashblock.h.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <atomic>

namespace fb {

constexpr int kKeyTile = 64;  // keys per main-loop iteration in every attention kernel

// Division of a non-negative 31-bit integer by a launch-time constant, without the ~25
// instruction integer-division sequence in the (cold, run-once) kernel prologue:
// q = (mulhi(n, magic) + n) >> shift with magic = floor(2^32 (2^shift - d) / d) + 1, shift = ceil(log2 d).
struct FastDiv {
  uint32_t magic, shift, d;
};

inline FastDiv make_fastdiv(uint32_t d) {
  FastDiv f;
  f.d = d;
  uint32_t s = 0;
  while ((1ull << s) < d) ++s;
  f.shift = s;
  f.magic = (uint32_t)((((1ull << s) - d) << 32) / d + 1);
  return f;
}

__host__ __device__ __forceinline__ uint32_t fastdiv(uint32_t n, const FastDiv& f) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint64_t t = (uint64_t)__umulhi(n, f.magic) + n;
#else
  const uint64_t t = (((uint64_t)n * f.magic) >> 32) + n;
#endif
  return (uint32_t)(t >> f.shift);
}

// Kernels with more than 64 KiB of dynamic LDS need their per-kernel limit raised before the first launch on a
// device.  One flag word per kernel remembers the devices on which that was done (bit d = device d): the only
// state the library keeps between calls.  It is an atomic, so concurrent first calls from several host threads are
// safe (the attribute call is idempotent), and it is per device, so a second GPU gets its own call.
struct LdsLimit {
  std::atomic<uint32_t> devices{0};
};

// bytes: what this launch needs; limit: what to ask for (the kernel's fixed size, or, for kernels whose size
// varies from call to call, kLdsLimitMax, which leaves room for their small static arrays).
constexpr size_t kLdsLimitMax = 160 * 1024 - 2048;

template <typename K>
hipError_t raise_lds_limit(K kern, size_t bytes, LdsLimit& st, size_t limit) {
  if (bytes <= 48 * 1024) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint32_t bit = (dev >= 0 && dev < 32) ? (1u << dev) : 0u;
  if (bit != 0u && (st.devices.load(std::memory_order_acquire) & bit) != 0u) return hipSuccess;
  e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)limit);
  if (e == hipSuccess && bit != 0u) st.devices.fetch_or(bit, std::memory_order_release);
  return e;
}

// Measurement hook (include/flashblock_prof.h): events that the NEXT bf16 attention launch of this host thread is to
// carry as its own start / stop events (hipExtLaunchKernelGGL: the timestamps of the kernel's dispatch, what a
// profiler's kernel trace reports, instead of markers recorded around it).  Cleared by the launch that takes them.
struct KernelEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
inline thread_local KernelEvents tl_kernel_events;

template <typename K, typename P>
void launch_attn_kernel(K kern, dim3 grid, dim3 block, size_t lds, hipStream_t s, const P& params) {
  KernelEvents& ev = tl_kernel_events;
  if (ev.start != nullptr || ev.stop != nullptr) {
    hipExtLaunchKernelGGL(kern, grid, block, lds, s, ev.start, ev.stop, 0, params);
    ev = KernelEvents{};
  } else {
    hipLaunchKernelGGL(kern, grid, block, lds, s, params);
  }
}

// What a pass iterates over and what it emits.
enum PassMode : int {
  kPassDense = 0,          // keys [0, nkeys) cut into nsplit tile ranges -> split partials
  kPassInternal = 1,       // keys [0, nkeys), no split; epilogue = Eq. 8-9 merge with cached partial
  kPassSparseRefresh = 2,  // like dense, but every key block is routed to the selected or the residual set
  kPassSparseReuse = 3,    // only key blocks of the per-KV-group union list; selected set only
  kPassDenseHeads = 4,     // dense, but only query heads flagged in head_on take part (others keep their cache)
  kPassDensePaged = 5,     // dense over a paged KV pool with a block table and per-sequence prefix lengths
  kPassRefreshFused = 6,   // dense over the prefix, and the block's own keys into partial set 1: in the last split's workgroup
                           // (register-staged), as an extra split (fp32), as two streams or not at all (by_parity)
  kPassRefreshOne = 7      // fp32: a whole refresh step in one kernel (prefix unsplit, final partial, then the block and the merge)
};

// One attention pass.  Rows of one KV group are addressed "group-flattened": query head
// kvh*G+g, block row i  <->  flat row g*Bq+i, which is contiguous in Q / partial / out memory.
struct PassParams {
  const void* q;        // [B,Hq,Bq,D]
  const void* k;        // [B,Hkv,nkeys,D]
  const void* v;        // [B,Hkv,nkeys,D]
  int B, Hq, Hkv, G, Bq, nkeys;
  int nsplit;
  float scale_log2;     // scale * log2(e): scores are kept in the log2 domain inside the kernels
  // split partial sets in the workspace, layout [set][split][B*Hq*Bq] rows:
  //   o [.., D] sum exp2(s2 - m2) v ; m2 (log2 domain reference) ; l = sum exp2(s2 - m2)
  float* ws_o;  float* ws_m;  float* ws_l;      // set 0: dense / selected
  float* ws_o2; float* ws_m2; float* ws_l2;     // set 1: residual (sparse refresh only)
  // internal pass epilogue
  const float* ext_o; const float* ext_m; const float* ext_lse;   // cached partial (natural log), may be null
  void* out; float* lse_out;
  // sparse passes
  const uint32_t* blk_mask;   // [B,Hkv,nblk] bit g set: head g of the group selected the block
  const int32_t* union_list;  // [B,Hkv,nblk] ascending blocks with mask != 0
  const uint32_t* union_mask; // [B,Hkv,nblk] mask of the i-th listed block (no dependent lookup in the reuse pass)
  const int32_t* union_cnt;   // [B,Hkv]
  int key_block, nblk;
  const uint8_t* head_on;     // [B,Hq] per-head refresh flags (kPassDenseHeads), else null
  // per-head refresh, heads_cap > 0 (row-pair kernel): an even number of splits, 2i and 2i + 1 with the even and the odd
  // tiles of the i-th range; their partials are stored by rank among the flagged KV groups, [split][B][heads_cap][G*Bq] rows;
  // groups of a higher rank run unsplit and write the final partial
  int heads_cap;
  // dense pass of up to 128 rows, nseg > 0 and != nsplit: reference segments (halves_pass), cut and ordered as nseg splits would
  // be, with their bias (seg_bias).  (These and by_parity stand where the pointers' alignment leaves room: eight bytes more of
  // arguments cost 0.1 us between two kernels, 0.5 % of a sparse block.)
  int nseg;
  float* o_final; float* m_final; float* l_final;
  // internal pass, fold_ns > 0: the external statistics are fold_ns split partials in ws_o / ws_m / ws_l, which the pass
  // folds, writes to o_final / m_final / l_final (natural-log units) and merges
  int fold_ns;
  // streaming kernel, refresh step: whole tiles for the two wavefronts of a row group, splits cut with blk_cost; and the
  // many-row internal pass visits its tiles in rotated order
  int whole_tiles, rotate, seg_bias;
  // paged pass: k/v point at the pools [num_pages, Hkv, page_size, D]
  const int32_t* block_table; // [B, max_pages] page ids
  const int32_t* prefix_lens; // [B] keys per sequence (<= nkeys)
  int page_size, max_pages, num_pages;
  // fused refresh pass by the row-pair kernel (many rows per KV head): an even nsplit, splits 2i and 2i + 1 with the even and the odd
  // tiles of the i-th range, and with k2 != null two partials of the block's own keys, likewise, in set 1
  int by_parity;
  const int32_t* seq_order;   // [B] sequences by descending prefix length (longest work is dispatched first), or null
  int order_inline;           // seq_order == null and 1: each workgroup ranks the (few) sequences itself
  // fused refresh pass: the block's own K/V [B,Hkv,Bq,D] go into partial set 1 (bf16: second phase of the last
  // split's workgroup, which gets blk_cost prefix tiles fewer; fp32: one extra split index; by_parity: two streams, or null)
  const void* k2; const void* v2; int blk_cost;
  // dense / heads / paged pass with nsplit == 1: ws_o / ws_m / ws_l are the caller's final (o, m, lse)
  // arrays and the kernel emits natural-log units itself (no combine pass)
  int direct;
  // streaming bf16 pass: 1 = splits alternate between the even and the odd XCD of a pair and the odd XCDs' splits are a
  // little shorter (see biased_range)
  int xcd_bias;
  FastDiv div_rowtiles, div_nsplit, div_hkv;   // bf16 pass: decomposition of the linear workgroup index
  FastDiv div_page;                            // bf16 paged pass: key index -> page slot
  FastDiv div_bias;                            // streaming bf16 pass, xcd_bias: by 64 * nsplit
  FastDiv div_tpb;                             // streaming sparse passes: tile index -> key block (tiles per key block); per-head
                                               // refresh by rank: row -> head (block_len)
};

// Fold split partials (and optionally a cached residual) into final (o, m, lse) partials.
struct CombineParams {
  int rows, D, nsplit;
  int blk_ns;                       // partials at blk_o / blk_m / blk_l, `rows` rows each
  const float* ws_o;  const float* ws_m;  const float* ws_l;    // selected / dense set, may be null when nsplit==0
  const float* ws_o2; const float* ws_m2; const float* ws_l2;   // residual set (refresh) or null
  const float* res_in_o; const float* res_in_m; const float* res_in_lse;   // cached residual (reuse) or null
  float* res_out_o; float* res_out_m; float* res_out_lse;                  // residual out (refresh) or null
  float* o; float* m; float* lse;                                          // total out
  const uint8_t* head_on; int Bq;   // if head_on != null: rows of heads with a zero flag are left untouched
  int heads_cap;                    // > 0: split partials stored by rank among the flagged KV groups (PassParams)
  // fused refresh step: block-internal partial (one split, log2 domain) merged with the total by Eq. 8-9 into
  // the normalised output (storage type) and its log-normaliser; null = no final output
  const float* blk_o; const float* blk_m; const float* blk_l;
  void* fin_out; float* fin_lse; int fin_bf16;
  // ... or, for a block of at most kMaxInlineBlock keys, the block's q / k / v themselves (storage type
  // fin_bf16): the fold kernel computes the block-internal attention of its rows itself
  const void* blk_q; const void* blk_k; const void* blk_v;
  int Hq, Hkv, G; float scale_log2;
};

struct SelectParams {
  const void* q; const float* k_pooled; int32_t* sel_idx;
  int B, Hq, Hkv, G, Bq, D, nblk, topk, is_bf16;
  // score source "attention mass": per-row masses [B][nblk][Hq*Bq] (then q / k_pooled are unused), and an
  // optional copy of the block scores [B,Hq,nblk]
  const float* rowmass; float* score_out;
  // optional scratch: mean queries [B,Hq,D] and block scores [B,Hq,nblk]; both set = scoring runs as kernels of
  // its own over the whole chip instead of inside the (one workgroup per head) selection kernel
  float* qbar_ws; float* scores_ws;
};

// Attention mass of every (query row, key block): sum over the block's keys of exp(s - lse).
struct MassParams {
  const void* q; const void* k; const float* lse; float* rowmass;   // rowmass [B][nblk][Hq*Bq]
  int B, Hq, Hkv, G, Bq, nkeys, key_block, nblk, nsplit;            // nsplit: key-block ranges per row tile
  float scale_log2;
};

struct PoolParams {
  const void* k; float* k_pooled;
  int BH, nkeys, D, key_block, nblk, is_bf16;
};

struct MaskParams {
  const int32_t* sel_idx; uint32_t* blk_mask; int32_t* union_list; uint32_t* union_mask; int32_t* union_cnt;
  int B, Hq, Hkv, G, topk, nblk;
};

// Host-side launchers; each returns the hipError_t of its launch(es).
hipError_t launch_attn_f32(const PassParams& p, int D, PassMode mode, hipStream_t s);
hipError_t launch_attn_bf16(const PassParams& p, int D, PassMode mode, hipStream_t s);
// Streaming form of the bf16 pass (direct-to-LDS tile ring); covers a subset of (shape, mode) combinations.
bool stream_bf16_covers(const PassParams& p, int D, PassMode mode);
hipError_t launch_stream_bf16(const PassParams& p, int D, PassMode mode, hipStream_t s);
int stream_bf16_name(const PassParams& p, int D, PassMode mode, char* buf, size_t n);
// Whether the internal pass of p can fold p.fold_ns split partials itself (few splits; not the row-pair kernels).
bool internal_fold_covers(const PassParams& p, int D);
// Name of the kernel launch_attn_bf16 runs for the dense external pass of p (profiler spelling, no namespace).
int attn_bf16_dense_name(const PassParams& p, int D, char* buf, size_t n);
// streams: of a refresh step whose splits are streams (PassParams::by_parity).
hipError_t launch_combine(const CombineParams& p, hipStream_t s, bool streams = false);
// Fold + block-internal attention + merge in one kernel; needs blk_q/k/v, Bq <= kMaxInlineBlock.
hipError_t launch_refresh_fold(const CombineParams& p, hipStream_t s);
constexpr int kMaxInlineBlock = 64;
constexpr int kFoldRows = 4;
hipError_t launch_pool_keys(const PoolParams& p, hipStream_t s);
hipError_t launch_select_topk(const SelectParams& p, hipStream_t s);
hipError_t launch_build_masks(const MaskParams& p, hipStream_t s);
hipError_t launch_block_mass_f32(const MassParams& p, int D, hipStream_t s);
hipError_t launch_block_mass_bf16(const MassParams& p, int D, hipStream_t s);
hipError_t launch_seq_order(const int32_t* prefix_lens, int32_t* seq_order, int B, hipStream_t s);
hipError_t launch_head_similarity(const float* o_a, const float* o_b, float* sim, int BH, int Bq, int D, hipStream_t s);

// Row tiles (workgroups along the group-flattened row axis) per KV group, per kernel family.
constexpr int kRowsPerWgBf16 = 128;  // 4 waves x 32 rows
constexpr int kRowsPerWgF32 = 4;     // fp32 mass kernel: 4 waves x 1 row
// fp32 attention pass: rows of a workgroup, by the rows that share a K/V stream.  Shared by the split heuristic and the
// launcher.  Above 32 rows 64 against 32, each with its own splits: 128 rows of 8 KV heads against 4111 keys 39.4 -> 37.6 us, at
// batch 4 115 -> 93, 12 heads of 1000 rows 399 -> 297.  17 to 32 rows in one workgroup, which reads K and V once, though two
// of 16 rows take less at 24 rows of 8 heads (4111 keys 20.6 and 18.1 us).
inline int f32_row_tile(long long nrows) { return nrows <= 16 ? 16 : nrows <= 32 ? 32 : 64; }
// fp32 internal and unsplit dense passes over at most 16 keys: one wavefront per row (attn_f32_few_kernel).  Up to 4096 rows, or
// 32 to a KV head, which a 16-row workgroup pads or a 64-row one does (head_dim 128, 4 / 16 keys: 128 rows 6.9 -> 3.7 / 6.9 -> 3.8
// us, 4096 rows 7.2 -> 6.8 / 7.2 -> 6.9; 16 rows of 1024 KV heads 23.9 -> 18.8; but 128 rows of 128 KV heads, 16 keys, 15.1 ->
// 18.8).
constexpr int kFewKeysF32 = 16;
inline bool f32_few_keys(long long rows, long long group_rows, int nkeys) {
  return nkeys >= 1 && nkeys <= kFewKeysF32 && (rows <= 4096 || group_rows <= 32);
}
// fp32 refresh step in one launch (kPassRefreshOne): 16-row workgroups, one round of them, that run prefix and block tiles
// themselves (head_dim 64: two tiles side by side, every tile with a stage of its own; 128: one after the other), against splits, a
// combine and its launch.  What it saves everybody is that launch's host time; what it costs or saves on the device depends on the
// tiles (all of the prefix and the block) and on the workgroups, of which the splits need several rounds where they are many.
// A refresh step replayed from a graph, us, splits -> one launch:
//   head_dim 64, 16 workgroups: 2 tiles 7.3 -> 6.6, 3 8.3 -> 7.4, 4 8.2 -> 8.2, 5 8.1 -> 9.0; 64: 5 8.8 -> 9.2; 80: 5 11.1 -> 9.2;
//     256: 2 9.9 -> 7.0, 5 15.4 -> 9.5
//   head_dim 128, 8 workgroups: 2 tiles 9.1 -> 9.3, 3 10.7 -> 11.4; 96: 3 11.5 -> 11.7; 112: 3 11.7 -> 11.5; 144: 3 15.9 -> 11.8
// and issued call by call with a reuse step behind it: head_dim 64, 2 to 64 workgroups, 3 / 5 tiles 11-14 -> 10 / 12.6-14.5 -> 10.9-12;
// head_dim 128, 2 / 3 tiles 14.3 -> 12 / 14.2-14.8 -> 14.2-14.9.  So the fifth tile of head_dim 64 trades up to 1 us on the device for
// 2 us of host time at up to 64 workgroups, and the third of 128 is taken only where the device gains.  One tile more: head_dim 64,
// 512 keys, 8.8 -> 13.8; 128, 256 keys 11.7 -> 15.
constexpr int kOneTiles = 5;         // at head_dim 64: one LDS stage each
inline bool f32_refresh_one(long long wgs16, int head_dim, int prefix_len, int block_len) {
  const int tiles = (prefix_len + kKeyTile - 1) / kKeyTile + (block_len + kKeyTile - 1) / kKeyTile;
  return wgs16 <= 256 && tiles <= (head_dim == 64 ? kOneTiles : wgs16 > 100 ? 3 : 2);
}

// Whether the internal pass writes over any of its inputs: rows' bytes of storage type and of fp32.
inline bool internal_in_place(const PassParams& p, int D, size_t esize) {
  const size_t rows = (size_t)p.B * p.Hq * p.Bq, kv = (size_t)p.B * p.Hkv * p.nkeys * D * esize;
  const struct { const void* at; size_t n; } outs[] = {{p.out, rows * D * esize}, {p.lse_out, rows * 4}},
      ins[] = {{p.q, rows * D * esize}, {p.k, kv}, {p.v, kv}, {p.ext_o, rows * D * 4}, {p.ext_m, rows * 4}, {p.ext_lse, rows * 4}};
  for (const auto& o : outs)
    for (const auto& i : ins)
      if (o.at && i.at && (uintptr_t)o.at < (uintptr_t)i.at + i.n && (uintptr_t)i.at < (uintptr_t)o.at + o.n) return true;
  return false;
}

// bf16 dense external pass: KV groups of more than 128 rows run 256-row workgroups (row pairs, one shared tile stream), so every
// K/V tile is staged once per 256 rows.  At head_dim 64 only from 1024 rows on: below, on streams of up to some 16000 keys, they
// are slower with the splits they get (us, 128-row workgroups and row pairs: 64 / 8 heads of 32 rows, 1000 / 4111 / 16384 keys 12.7 / 15.3 / 24.1
// and 18.4 / 21.5 / 25.3), though faster on long ones (32768 / 100000 keys 35.5 / 82.2 and 34.9 / 68.8; 8 heads of 300 rows 76 / 203 and
// 48 / 116), which a rule by length does not tell apart yet.  Shared by the split heuristic and the launcher.
inline bool dense_row_pairs(int nrows, int head_dim) {
  return nrows >= 1024 || (head_dim >= 128 && nrows > kRowsPerWgBf16);
}

// Compute-bound internal pass: many rows per KV head, a 256-row workgroup for (almost) every CU.
inline bool internal_many_rows(const PassParams& p) {
  const int nrows = p.G * p.Bq;
  return nrows >= 1024 && (long long)p.B * p.Hkv * ((nrows + 255) / 256) >= 128;
}

// ---- device helpers shared by the attention kernels -------------------------------------
// One 16-byte direct-to-LDS load per lane: lane l's chunk lands at LDS byte lds_base + 16 l.  Global address =
// base (wavefront-uniform) + off (per lane, unsigned 32-bit).  A direct-to-LDS load needs one wait state after a scalar write of
// M0, which nothing puts between two instructions of one asm block: hence the s_nop, here and wherever M0 is written by hand.
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds_base) {
  // base and lds_base are wavefront-uniform by construction; readfirstlane says so to the compiler, which
  // otherwise may hand the "s" operands over in vector registers (not encodable here)
  // (the builtin returns int: each half goes through uint32_t so that nothing is sign-extended)
  const uint64_t b = (uint64_t)(uintptr_t)base;
  const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  const uint64_t bu = ((uint64_t)b_hi << 32) | (uint64_t)b_lo;
  const uint32_t lu = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_base);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(bu), "s"(lu)
               : "memory", "m0");
}

// Maximum / sum of lanes l and l ^ 32, by exchanging the halves of the wavefront in registers (a shuffle goes through the LDS:
// some 130 cycles in a tile's chain from scores to weights).
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Lane l's value combined with lane l ^ 16's.
__device__ __forceinline__ float max_rows(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_rows(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The value of the lane N below, around the 16 lanes of a row (DPP row_ror).  Where a value repeats every 2 N lanes, that is
// lane l ^ N's.
template <int N>
__device__ __forceinline__ float turn16(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xf, 0xf, false));
}
// Lane l ^ 4's value where the four lanes of every quad hold the same one (DPP row_half_mirror: lane 7 - l within eight lanes).  A
// turn by 4 would not do before a turn by 8: lanes of even and of odd quads would add up in different orders.
__device__ __forceinline__ float swap_quads(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, false));
}
// Sum / maximum over the 16 lanes of a row, over the wavefront: the order of the butterfly over lanes 32, 16, 8, 4, 2, 1.
__device__ __forceinline__ float sum16(float x) {
  x += turn16<8>(x);
  x += turn16<4>(x);
  x += turn16<2>(x);
  return x + turn16<1>(x);
}
__device__ __forceinline__ float max16(float x) {
  x = fmaxf(x, turn16<8>(x));
  x = fmaxf(x, turn16<4>(x));
  x = fmaxf(x, turn16<2>(x));
  return fmaxf(x, turn16<1>(x));
}
__device__ __forceinline__ float wave_sum(float x) { return sum16(sum_rows(sum_halves(x))); }
__device__ __forceinline__ float wave_max(float x) { return max16(max_rows(max_halves(x))); }

// Per-head refresh: whether any query head of KV group `kvh` of batch element b is flagged.
__device__ __forceinline__ bool group_flagged(const uint8_t* head_on, int b, int Hq, int G, int kvh) {
  uint32_t any = 0;
  for (int g = 0; g < G; ++g) any |= head_on[b * Hq + kvh * G + g];
  return any != 0;
}

// Wavefront-uniform table lookup as a scalar load (constant address space).  The tables were written by earlier
// kernels, so they are constant here; without this the compiler, which sees the inline assembly's memory
// clobber, falls back to vector loads, and its wait for them (vmcnt(0)) would also drain every direct-to-LDS
// load in flight.
__device__ __forceinline__ int32_t sload(const void* table, int idx) {
  typedef const __attribute__((address_space(4))) int32_t* cptr;
  return ((cptr)(uintptr_t)table)[__builtin_amdgcn_readfirstlane(idx)];
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Tile schedule of one workgroup: which 64-key tiles it visits.
struct TileRange {
  int begin, end;   // entries [begin, end) of the pass's tile list
};

__device__ __forceinline__ TileRange split_range(int total, int nsplit, int split) {
  // balanced contiguous cut of `total` entries into nsplit pieces: the first total % nsplit
  // pieces get one entry more (one 32-bit division, no 64-bit arithmetic)
  const int base = total / nsplit, rem = total - base * nsplit;
  TileRange r;
  r.begin = split * base + min(split, rem);
  r.end = r.begin + base + (split < rem ? 1 : 0);
  return r;
}

// Cut of `total` tiles into an even number of pieces in which the even-numbered pieces are 1/64 longer and the
// odd-numbered ones 1/64 shorter than the mean (weights 65 : 63).  Used with a workgroup mapping that puts the
// odd-numbered splits on the odd-numbered XCDs: on the MI355X boards measured, the odd XCD of each pair streams
// about 4 % slower than the even one whichever KV head it reads (finish times of 128K passes per XCD, in-kernel
// clocks, with the head-to-XCD assignment rotated), and the pass ends with its slowest XCD.  A fixed, deterministic
// cut, deliberately a little weaker than the measured asymmetry: 128K pass 99.4 -> 97.4 us, batch 4 neutral; on a
// board without the asymmetry it would cost under 2 %.
// by_weights: division by 64 * nsplit (a 64-bit division here is some 250 cold instructions in front of the first load:
// a refresh and a reuse step at 32K keys 44.9 -> 44.7 us, 128K 110.8 -> 110.4); the host keeps total * 64 * nsplit below 2^31.
__device__ __forceinline__ TileRange biased_range(int total, const FastDiv& by_weights, int split) {
  auto cum = [](int s) -> uint32_t { return 64u * (uint32_t)s + (uint32_t)(s & 1); };
  TileRange r;
  r.begin = (int)fastdiv((uint32_t)total * cum(split), by_weights);
  r.end = (64u * (uint32_t)(split + 1) == by_weights.d) ? total : (int)fastdiv((uint32_t)total * cum(split + 1), by_weights);
  return r;
}

// The same cut with the division by nsplit done through its precomputed magic number.
__device__ __forceinline__ TileRange split_range(int total, const FastDiv& by_nsplit, int split) {
  const int base = (int)fastdiv((uint32_t)total, by_nsplit), rem = total - base * (int)by_nsplit.d;
  TileRange r;
  r.begin = split * base + min(split, rem);
  r.end = r.begin + base + (split < rem ? 1 : 0);
  return r;
}

}  // namespace fb
