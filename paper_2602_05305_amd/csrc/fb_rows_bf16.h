// bf16 attention pass over many rows per KV head (gfx950): 256 rows per workgroup, 64 per wavefront, one wavefront per SIMD.
// The device code behind the row-pair layout of attn_stream_kernel (fb_stream_bf16.hip), which describes tiles, rotation and
// register layouts; what is different here:
//
// What bounds it: with 32 rows per wavefront every product takes one 1 KB operand from LDS, 256 KB per 256 x 64 tile, which
// holds the LDS as long as the products hold the matrix cores, and two wavefronts per SIMD did not hide that in one another
// (3900 cycles a tile against 2048 of products).  Here an operand serves two products (rows l, l + 32 of the wavefront), and the
// wavefront has the SIMD to itself: 512 registers, 128 accumulators and 64 query registers of them in the accumulator half.
//   * One wavefront issues in order, and the matrix core runs beside the vector unit only while other instructions follow a
//     product: two products in a row idle the vector unit for one of them (4 x (2 products, 2 exp, 5 fma) 338 cycles, 8 x (product,
//     exp, 3 fma) 286).  So the loop is written in slots of one product each, with the softmax of tile t spread over the products
//     Q K(t+1) and P V(t), and the slots are pinned (sched_barrier).
//   * The products are inline assembly, because the register halves have to be stated: left to itself the compiler keeps the
//     scores in the accumulator half and moves 64 to 320 registers per tile.  Waits that the hardware does not do by
//     itself: a vector instruction may read a product's result 12 wait states after it (settle), a product may read what a
//     vector instruction wrote 2 wait states after it (weights are packed a slot ahead of their product).
//   * Every tile costs the same loads, one per three slots (eight in a row: 5 to 9 % of the pass, all four wavefronts wait for
//     the address unit), the ring's stages are compile-time constants (four tiles written out), and a tile's rare work (reference
//     moved, ragged tile) is one branch at its top.
// Measured (12 heads of 4680 rows, 37440 keys, against 32 rows per wavefront, alternating): 1015 -> 886 us, 2.26 M cycles at 2.23
// GHz -> 1.78 M at 2.02 (the part lowers its clock as the matrix cores get busier, so time falls less than cycles); reuse step
// of 4680 keys 147 -> 131 us.  Same tiles, order and references per row: results are the same up to the contraction of the row
// sum in the epilogue.  Its ends cost more, so short streams keep the 32 rows (short_row_pairs in fb_stream_bf16.hip).
#pragma once

#include <type_traits>

#include "fb_kernels.h"

namespace fb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}

// Shortest range of tiles.  Loads run ahead, five tiles of them before the loop, which looks out for the ragged tile from its own first
// requests on: a range that ends with one must not come round to it before.
constexpr int kRowsTiles = 5;

template <int D>
struct RCfg {
  static constexpr int THREADS = 256, ROWS = 256, KT = 64;
  static constexpr int ROWB = D * 2, CPR = ROWB / 16, OPB = KT * ROWB;
  static constexpr int NLOAD = OPB / (THREADS * 16);
  static constexpr int NS = 4;                       // stages of each ring (K, V)
  static constexpr int QOFF = (2 * NS - 2) * OPB;    // the queries start in the last two V stages
  static constexpr int LDS = QOFF + 4 * OPB;
  static constexpr int NKS = D / 16, NDB = D / 32;
  static constexpr int NQK = 2 * NKS, NPV = 4 * NDB, NCH = NQK + NPV;
  __device__ static __forceinline__ int rot_k(int row) { return D == 128 ? row : (row >> 1); }
  __device__ static __forceinline__ int rot_v(int row) { return D == 128 ? 4 * row : 4 * (row >> 1); }
};

__device__ __forceinline__ void mfma_first(f32x16& d, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_score(f32x16& d, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_value(f32x16& d, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
template <int N>
__device__ __forceinline__ void settle(f32x16 (&s)[2][2]) {
  if constexpr (N > 0) asm volatile("s_nop %4\n\ts_nop %4" : "+v"(s[0][0]), "+v"(s[0][1]), "+v"(s[1][0]), "+v"(s[1][1]) : "n"(N));
  else asm volatile("" : "+v"(s[0][0]), "+v"(s[0][1]), "+v"(s[1][0]), "+v"(s[1][1]));
}
template <int NDB>
__device__ __forceinline__ void settle_o(f32x16 (&o)[2][NDB]) {
  if constexpr (NDB == 4)
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(o[0][0]), "+a"(o[0][1]), "+a"(o[0][2]), "+a"(o[0][3]), "+a"(o[1][0]), "+a"(o[1][1]), "+a"(o[1][2]), "+a"(o[1][3]));
  else
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(o[0][0]), "+a"(o[0][1]), "+a"(o[1][0]), "+a"(o[1][1]));
}

constexpr int cmin(int a, int b) { return a < b ? a : b; }

// f(integral constants B .. E - 1): a loop whose counter is a constant in every trip
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

template <int N> using Int = std::integral_constant<int, N>;

// dma16 to LDS byte lds_base + AT
template <int AT>
__device__ __forceinline__ void dma16_at(const void* base, uint32_t off, uint32_t lds_base) {
  const uint64_t b = (uint64_t)(uintptr_t)base;
  const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  const uint64_t bu = ((uint64_t)b_hi << 32) | (uint64_t)b_lo;
  const uint32_t lu = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_base);
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(bu), "s"(lu), "i"(AT)
               : "memory", "m0", "scc");
}

template <int D, int MODE>
__device__ __forceinline__ void rows_pass(const PassParams& p, unsigned char* ring) {
  using C = RCfg<D>;
  constexpr bool kHeads = MODE == kPassDenseHeads;
  // refresh step in several splits: every split as two streams (below), and two more over the block's own keys
  constexpr bool kFused = MODE == kPassRefreshFused;
  constexpr bool kParity = kHeads || kFused;
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));

  // ---- workgroup -> (row tile, batch, KV head, split): a contiguous range of units per XCD (fb_stream_bf16.hip); per-head
  // refresh: whole heads drop out, so a head's row tiles are dealt over the XCDs
  const int nwg = gridDim.x;
  const int nrows = p.G * p.Bq;
  int w = blockIdx.x;
  bool own_block = false;                                    // (the prefix's workgroups are the first of the grid)
  if constexpr (!kHeads) {
    const int npre = kFused ? p.B * p.Hkv * p.nsplit * (int)p.div_rowtiles.d : nwg;
    own_block = kFused && w >= npre;
    const int bid = own_block ? w - npre : w, n = own_block ? nwg - npre : npre, q8 = n / 8, r8 = n % 8;
    const int xcd = bid % 8, j = bid / 8;
    w = (xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8) + j;
  }
  uint32_t rest = fastdiv((uint32_t)w, p.div_rowtiles);
  const int rt = w - (int)(rest * p.div_rowtiles.d);
  const uint32_t unit = rest;
  int split = 0;
  if (kFused && own_block) {
    split = (int)(rest & 1);
    rest >>= 1;
  } else if constexpr (MODE != kPassInternal) {
    const uint32_t r2 = fastdiv(rest, p.div_nsplit);
    split = (int)(rest - r2 * p.div_nsplit.d);
    rest = r2;
  }
  int b, kvh, rank = 0;
  bool direct = p.direct != 0;                               // this workgroup writes the final partial
  if constexpr (kHeads) {
    // The first B * heads_cap * nsplit units belong to the flagged KV groups by rank (the workgroups that have work are then
    // the first of the grid and spread evenly over the chip whatever the mask; dealt out by head, some masks left a
    // shader engine with two rounds of workgroups: 569 or 1010 us for 6 of 12 heads); B * Hkv units at the end, one split
    // each, are for groups beyond the hint.
    const uint32_t ranked = (uint32_t)(p.B * p.heads_cap);
    const uint32_t units = ranked * p.div_nsplit.d;
    const bool extra = unit >= units;
    const uint32_t bu = extra ? unit - units : rest;
    const uint32_t per = extra ? (uint32_t)p.Hkv : (uint32_t)p.heads_cap;
    b = (int)(bu / per);
    const int want = (int)(bu - (uint32_t)b * per);          // rank, or KV group
    int seen = 0, hit = -1;
    for (int g0 = 0; g0 < p.Hkv && hit < 0; g0 += 64) {
      unsigned long long mask = __ballot(g0 + lane < p.Hkv && group_flagged(p.head_on, b, p.Hq, p.G, g0 + lane));
      if (extra) {
        if (want < g0 + 64) {
          const unsigned long long below = (1ull << (want - g0)) - 1;
          if (((mask >> (want - g0)) & 1) && seen + __popcll(mask & below) >= p.heads_cap) hit = want;
          break;
        }
      } else if (want < seen + __popcll(mask)) {
        for (int k = want - seen; k > 0; --k) mask &= mask - 1;
        hit = g0 + __ffsll(mask) - 1;
      }
      seen += __popcll(mask);
    }
    if (hit < 0) return;                                     // workgroup-uniform
    kvh = __builtin_amdgcn_readfirstlane(hit);
    rank = want;
    if (extra) direct = true;
  } else {
    b = (int)fastdiv(rest, p.div_hkv);
    kvh = (int)(rest - (uint32_t)b * p.div_hkv.d);
  }
  const int bk = b * p.Hkv + kvh;
  const int nkeys = own_block ? p.Bq : p.nkeys;              // at least kRowsTiles tiles to a range (launch_stream sees to it)
  const int row0 = rt * C::ROWS;
  const size_t grow_base = (size_t)(b * p.Hq + kvh * p.G) * p.Bq;
  // Per-head refresh: row tiles are cut from the rows of the group's flagged heads, one head after the other; workgroups past the last
  // one leave, and wavefronts past it only load.  (Cut from all rows, a tile computed those of other heads along: 1 of 4 heads of
  // 64 rows flagged in each of 8 KV groups, batch 2, 40000 keys, 99.5 us, where wavefronts of 32 rows that skip theirs take 82.3;
  // so 73.5.  Every other of 8 heads of 373 rows, 4 KV groups, batch 3, 6877 keys 171, 149, 117.5.)
  int nflagged = nrows, head_of = 0;                         // rows of flagged heads; lane k: the k-th flagged head of the group
  bool gaps = false;
  if constexpr (kHeads) {
    const unsigned long long on = __ballot(lane < p.G && p.head_on[b * p.Hq + kvh * p.G + min(lane, p.G - 1)] != 0);
    int k = 0;
    for (int g = 0; g < p.G; ++g)
      if ((on >> g) & 1) {
        head_of = lane == k ? g : head_of;
        ++k;
      }
    nflagged = k * p.Bq;
    gaps = k < p.G;
    if (row0 >= nflagged) return;                            // workgroup-uniform
  }
  // the r-th of the rows that are computed, r < nflagged, as a row of the group (every lane takes part)
  auto group_row = [&](int r) __attribute__((always_inline)) {
    if (!kHeads || !gaps) return r;
    const int k = (int)fastdiv((uint32_t)r, p.div_tpb);      // (divisor here: block_len)
    return r + (__shfl(head_of, k, 64) - k) * p.Bq;
  };

  const unsigned char* __restrict__ Kg = (const unsigned char*)(own_block ? p.k2 : p.k) + (size_t)bk * nkeys * C::ROWB;
  const unsigned char* __restrict__ Vg = (const unsigned char*)(own_block ? p.v2 : p.v) + (size_t)bk * nkeys * C::ROWB;

  // ---- tiles of this workgroup: positions first, first + stride, ... of a range, rotated (per-head refresh, partials by rank, and refresh
  // step: splits 2i and 2i + 1 take the even and the odd tiles of the i-th range, the two tile groups of the register-staged kernel,
  // whose references these are)
  const int total = (nkeys + C::KT - 1) / C::KT;
  TileRange tr = (MODE == kPassInternal) ? TileRange{0, total} : split_range(total, p.div_nsplit, split);
  uint32_t rsrc = (p.div_rowtiles.d == 1) ? blockIdx.x : unit;
  int stride = 1, first = 0;
  if constexpr (kFused) {
    const int pairs = p.nsplit / 2, range_i = own_block ? pairs - 1 : split >> 1;
    tr = own_block ? TileRange{0, total} : split_range(total + p.blk_cost, pairs, range_i);
    tr.begin = min(tr.begin, total);
    tr.end = min(tr.end, total);
    stride = 2;
    first = split & 1;
    rsrc = (uint32_t)(bk * pairs + range_i);
  }
  if constexpr (kHeads) {
    if (direct) {
      tr = TileRange{0, total};
    } else {
      const int pairs = p.nsplit / 2;
      tr = split_range(total, pairs, split >> 1);
      stride = 2;
      first = split & 1;
      rsrc = (uint32_t)((b * p.Hkv + kvh) * pairs + (split >> 1));
    }
  }
  const int range = tr.end - tr.begin;
  const int ntiles = kParity ? (range - first + stride - 1) / stride : range;
  const int rot = ((MODE == kPassInternal && !p.rotate) || range <= 0) ? 0 : (int)((rsrc * 13u + (rsrc >> 5) * 7u) % (unsigned)range);
  // the ragged tile: its keys, and which of this workgroup's tiles it is (far from every one if none)
  const int nvalid = nkeys - (total - 1) * C::KT;
  int t_ragged = -(1 << 30), again = 1 << 30;                // ... again among the loads past the last tile
  if (nvalid < C::KT && tr.end == total) {
    const int x = range - 1 - rot - first;
    if (x >= 0 && x % stride == 0) t_ragged = x / stride;
    if (!kParity) again = t_ragged + range;
  }

  const uint32_t ring_base = (uint32_t)(uintptr_t)ring;
  constexpr uint32_t VOFF = C::NS * C::OPB;
  // direct-to-LDS load slots of this lane: LDS row, logical chunk of K and of V, and the byte offset inside a tile
  uint32_t off_k[C::NLOAD], off_v[C::NLOAD];
  int ld_row[C::NLOAD], ck[C::NLOAD], cv[C::NLOAD];
#pragma unroll
  for (int j = 0; j < C::NLOAD; ++j) {
    const int pidx = (j * 4 + wave) * 64 + lane;
    const int r = pidx / C::CPR, pc = pidx % C::CPR;
    ld_row[j] = r;
    ck[j] = (pc - C::rot_k(r)) & (C::CPR - 1);
    cv[j] = (pc - C::rot_v(r)) & (C::CPR - 1);
  }
  // ragged tile: rows past the end read the last key (in bounds; their scores are masked)
  auto aim = [&](uint32_t (&off)[C::NLOAD], const int (&chunk)[C::NLOAD], bool ragged) __attribute__((always_inline)) {
    const int last = ragged ? nvalid - 1 : C::KT - 1;
#pragma unroll
    for (int j = 0; j < C::NLOAD; ++j) off[j] = (uint32_t)(min(ld_row[j], last) * C::ROWB + chunk[j] * 16);
  };
  // One stream of tiles per operand: the address of the next tile, in rotated order.  Past the last tile it goes on, through the
  // first ones again (two streams to a range: with the first tile of the range, which is whole): every iteration requests the same
  // number of loads, and what these bring is never read.
  struct Stream {
    const unsigned char *next, *first, *src;
    int at, left;
  };
  auto open_stream = [&](const unsigned char* base) {
    Stream st;
    st.at = first + rot;
    if (st.at >= range) st.at -= range;
    st.first = base + (size_t)tr.begin * C::OPB;
    st.next = st.first + (size_t)st.at * C::OPB;
    st.left = ntiles;
    return st;
  };
  Stream kst = open_stream(Kg), vst = open_stream(Vg);
  auto step_stream = [&](Stream& st) __attribute__((always_inline)) {
    if constexpr (kParity) {
      st.src = st.left > 0 ? st.next : st.first;
      --st.left;
      st.at += stride;
      if (st.at >= range) st.at -= range;
      st.next = st.first + (size_t)st.at * C::OPB;
    } else {
      st.src = st.next;
      const bool wrap = ++st.at == range;
      st.next = wrap ? st.first : st.next + C::OPB;
      st.at = wrap ? 0 : st.at;
    }
  };
  const uint32_t dst_base = ring_base + wave * 1024;
  auto load_k1 = [&](auto i_, auto j_) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value, j = decltype(j_)::value;
    dma16_at<(i % C::NS) * C::OPB + j * 4096>(kst.src, off_k[j], dst_base);
  };
  auto load_v1 = [&](auto i_, auto j_) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value, j = decltype(j_)::value;
    dma16_at<(int)VOFF + (i % C::NS) * C::OPB + j * 4096>(vst.src, off_v[j], dst_base);
  };
  auto issue_k = [&](auto i_) __attribute__((always_inline)) { step_stream(kst); aim(off_k, ck, decltype(i_)::value == t_ragged); static_for<0, C::NLOAD>([&](auto j_) __attribute__((always_inline)) { load_k1(i_, j_); }); };
  auto issue_v = [&](auto i_) __attribute__((always_inline)) { step_stream(vst); aim(off_v, cv, decltype(i_)::value == t_ragged); static_for<0, C::NLOAD>([&](auto j_) __attribute__((always_inline)) { load_v1(i_, j_); }); };

  // prologue
  {
    const int at = kHeads ? __builtin_amdgcn_readfirstlane(group_row(row0)) : row0;
    const unsigned char* qg = (const unsigned char*)p.q + (grow_base + at) * C::ROWB;
    const int qvalid = nflagged - row0;
#pragma unroll
    for (int part = 0; part < 4; ++part)
#pragma unroll
      for (int j = 0; j < C::NLOAD; ++j) {
        int r = min(64 * part + ld_row[j], qvalid - 1);
        if constexpr (kHeads) r = group_row(row0 + r) - at;
        dma16(qg, (uint32_t)(r * C::ROWB + ck[j] * 16), ring_base + C::QOFF + part * C::OPB + wave * 1024 + j * 4096);
      }
  }
  if (ntiles > 0) {
    issue_k(Int<0>{}); issue_k(Int<1>{}); issue_v(Int<0>{}); issue_k(Int<2>{}); issue_v(Int<1>{}); issue_k(Int<3>{});
    wait_vm<5 * C::NLOAD>();
  } else {
    wait_vm<0>();
  }
  __syncthreads();
  if constexpr (kParity) {
    if (row0 + wave * 64 >= nflagged) {
      // no rows for this wavefront: its share of the loads, at the barriers of the loop below, and nothing else
      if (ntiles > 0) {
        wait_vm<3 * C::NLOAD>();
        __syncthreads();
        issue_v(Int<2>{});
        issue_k(Int<4>{});
        for (int t = 0; t < ntiles; ++t) {
          wait_vm<3 * C::NLOAD>();
          __syncthreads();
          step_stream(vst);
          aim(off_v, cv, t + 3 == t_ragged);
#pragma unroll
          for (int j = 0; j < C::NLOAD; ++j) dma16(vst.src, off_v[j], dst_base + VOFF + (t + 3) % C::NS * C::OPB + j * 4096);
          step_stream(kst);
          aim(off_k, ck, t + 5 == t_ragged);
#pragma unroll
          for (int j = 0; j < C::NLOAD; ++j) dma16(kst.src, off_k[j], dst_base + (t + 5) % C::NS * C::OPB + j * 4096);
        }
      }
      wait_vm<0>();
      return;
    }
  }
  bf16x8 qreg[2][C::NKS];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int r = 32 * g + l32;
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks)
      qreg[g][ks] = *(const bf16x8*)(ring + C::QOFF + wave * C::OPB + r * C::ROWB + ((2 * ks + h + C::rot_k(r)) & (C::CPR - 1)) * 16);
  }
  uint32_t kaddr[C::NKS], vaddr[C::NDB];
#pragma unroll
  for (int ks = 0; ks < C::NKS; ++ks) kaddr[ks] = (uint32_t)(l32 * C::ROWB + ((2 * ks + h + C::rot_k(l32)) & (C::CPR - 1)) * 16);
  {
    const int i16 = lane & 15, blk1 = (lane >> 4) & 1;
    const int rrow = 4 * h + (i16 >> 2);
#pragma unroll
    for (int db = 0; db < C::NDB; ++db) {
      const int c = 4 * db + 2 * blk1 + ((i16 & 3) >> 1);
      const int pc = (c + C::rot_v(rrow)) & (C::CPR - 1);
      vaddr[db] = (uint32_t)(VOFF + rrow * C::ROWB + pc * 16 + (i16 & 1) * 8);
    }
  }
  f32x16 o[2][C::NDB];
  float m[2], mold[2], l[2], mu[2], alpha[2], mx[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    m[g] = mold[g] = -INFINITY; l[g] = 0.f; mu[g] = 0.f; alpha[g] = 1.f; mx[g] = -INFINITY;
#pragma unroll
    for (int i = 0; i < C::NDB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[g][i][r] = 0.f;
  }
  constexpr float kLazy = 8.f;
  const float scale_log2 = p.scale_log2;

  // operand of QK chunk c of tile i / PV chunk c of tile i
  auto load_kop = [&](auto i_, auto c_) __attribute__((always_inline)) -> bf16x8 {
    constexpr int i = decltype(i_)::value, c = decltype(c_)::value, ks = c / 2, kb = c % 2;
    return *(const bf16x8*)(ring + kaddr[ks] + (i % C::NS) * C::OPB + kb * 32 * C::ROWB);
  };
  auto load_vop = [&](auto i_, auto c_) __attribute__((always_inline)) -> bf16x8 {
    constexpr int i = decltype(i_)::value, c = decltype(c_)::value, step = c / C::NDB, db = c % C::NDB;
    const unsigned char* base = ring + vaddr[db] + (i % C::NS) * C::OPB + step * 16 * C::ROWB;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(base));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(base + 8 * C::ROWB));
    const s16x8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, both);
  };
  // reference update from the tile's maxima, in five steps
  auto ref_step = [&](auto i_) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value;
    static_for<0, 2>([&](auto g_) __attribute__((always_inline)) {
      constexpr int g = decltype(g_)::value;
      if constexpr (i == 0) mx[g] *= scale_log2;
      if constexpr (i == 1) mx[g] = max_halves(mx[g]);
      if constexpr (i == 2) {
        mold[g] = m[g];
        m[g] = (mx[g] > m[g] + kLazy) ? mx[g] : m[g];
      }
      if constexpr (i == 3) mu[g] = (m[g] == -INFINITY) ? 0.f : m[g];
      if constexpr (i == 4) {
        alpha[g] = __builtin_amdgcn_exp2f(mold[g] - mu[g]);
        mx[g] = -INFINITY;
      }
    });
  };
  auto mask_tile = [&](f32x16 (&s)[2][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kb * 32 + 8 * (r / 4) + 4 * h + (r % 4);
          if (key >= nvalid) s[g][kb][r] = -INFINITY;
        }
  };
  constexpr int AHEAD = 4, NOP = 8;      // operands are requested two at a time, AHEAD and AHEAD + 1 chunks early
  bf16x8 op[NOP];
  // s: scores of tile t (maxima known), sn: scores of tile t + 1
  auto body = [&](f32x16 (&s)[2][2], f32x16 (&sn)[2][2], int t, auto tt_) __attribute__((always_inline)) {
    constexpr int tt = decltype(tt_)::value;          // t modulo the stages
    const bool moved = __any(alpha[0] != 1.f || alpha[1] != 1.f);
    if (moved || (unsigned)(t - t_ragged + 5) <= 5u || t + 5 >= again) {
      // rare: the reference moved, or the ragged tile is near: requested in this iteration or the last one, or computed now
      if (t == t_ragged) {
        mask_tile(s);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          m[g] = mold[g];
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx[g] = fmaxf(mx[g], s[g][kb][r]);
        }
        static_for<0, 5>(ref_step);
      }
      aim(off_k, ck, t + 5 == t_ragged || t + 5 == again);
      aim(off_v, cv, t + 3 == t_ragged || t + 3 == again);
      if (__any(alpha[0] != 1.f || alpha[1] != 1.f)) {
        settle_o<C::NDB>(o);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          l[g] *= alpha[g];
#pragma unroll
          for (int db = 0; db < C::NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[g][db][r] *= alpha[g];
        }
        settle_o<C::NDB>(o);
      }
    }
    // Weights, three stages a slot or more apart: x = score * scale - reference, e = exp2(x), then sum and packing of a pair.
    float ls[2] = {0.f, 0.f};
    uint32_t pk[2][4][4];
    float xs[64];
    auto stage1 = [&](auto u_) __attribute__((always_inline)) {
      constexpr int u = decltype(u_)::value, q = u / 2, kb = q / 16, r = 2 * ((q % 16) / 2) + u % 2, g = q % 2;
      xs[u] = fmaf(s[g][kb][r], scale_log2, -mu[g]);
    };
    auto stage2 = [&](auto u_) __attribute__((always_inline)) {
      constexpr int u = decltype(u_)::value;
      xs[u] = __builtin_amdgcn_exp2f(xs[u]);
      asm volatile("" : "+v"(xs[u]));                    // here, not where it is used
    };
    auto stage3 = [&](auto u_) __attribute__((always_inline)) {
      constexpr int u = decltype(u_)::value, q = u / 2, kb = q / 16, r = 2 * ((q % 16) / 2), g = q % 2;
      ls[g] += xs[u];
      if constexpr (u % 2 == 1) {
        uint32_t w = pack_bf16x2(xs[u - 1], xs[u]);
        asm volatile("" : "+v"(w), "+v"(ls[g]));
        pk[g][2 * kb + r / 8][(r % 8) / 2] = w;
      }
    };
    constexpr int NSLOT = 2 * C::NCH, SB = 2 * C::NQK;     // slots: one product each
    constexpr int S1 = NSLOT - 2 * C::NDB - 4;             // stage 1 ends here, so that the last weights are packed in time
    auto stage1_upto = [](int j) constexpr { return j <= 0 ? 0 : cmin(64, 64 * j / S1); };
    constexpr int M0 = SB + 3, M1 = NSLOT - 5;             // maxima of tile t + 1 in slots [M0, M1)
    static_for<0, NSLOT>([&](auto j_) __attribute__((always_inline)) {
      constexpr int j = decltype(j_)::value, c = j / 2, g = j % 2;
      if constexpr (j == SB) {
        // every wavefront has left K(t+1) and V(t-1); V(t+1) and K(t+2) have landed
        wait_vm<3 * C::NLOAD>();
        __syncthreads();
      }
      if constexpr (g == 0 && c % 2 == 0) asm volatile("" ::"v"(op[c % NOP]), "v"(op[(c + 1) % NOP]));      // one wait for two
      if constexpr (c < C::NQK) {
        constexpr int ks = c / 2, kb = c % 2;
        if constexpr (ks == 0) mfma_first(sn[g][kb], op[c % NOP], qreg[g][ks]);
        else mfma_score(sn[g][kb], op[c % NOP], qreg[g][ks]);
      } else {
        constexpr int step = (c - C::NQK) / C::NDB, db = (c - C::NQK) % C::NDB;
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 w = {pk[g][step][0], pk[g][step][1], pk[g][step][2], pk[g][step][3]};
        mfma_value(o[g][db], op[c % NOP], __builtin_bit_cast(bf16x8, w));
        if constexpr (c == C::NQK && g == 1) settle<0>(sn);
      }
      __builtin_amdgcn_sched_barrier(0);        // the product first: two in a row leave the vector unit idle for one of them
      if constexpr (g == 0 && c % 2 == 0) {
        static_for<c + AHEAD, c + AHEAD + 2>([&](auto ca_) __attribute__((always_inline)) {
          constexpr int ca = decltype(ca_)::value;
          if constexpr (ca < C::NQK) op[ca % NOP] = load_kop(Int<tt + 1>{}, Int<ca>{});
          else if constexpr (ca < C::NCH) op[ca % NOP] = load_vop(Int<tt>{}, Int<ca - C::NQK>{});
          else op[ca % NOP] = load_kop(Int<tt + 2>{}, Int<ca - C::NCH>{});
        });
      }
      // loads of V(t+3) and K(t+5), one at a time: eight in a row keep the four wavefronts waiting for the address unit
      if constexpr (j == SB + 1) step_stream(vst);
      if constexpr (j == SB + 1 + 3 * C::NLOAD) step_stream(kst);
      if constexpr (j > SB + 1 && (j - SB - 2) % 3 == 0) {
        constexpr int i = (j - SB - 2) / 3;
        if constexpr (i < C::NLOAD) load_v1(Int<tt + 3>{}, Int<i>{});
        else if constexpr (i < 2 * C::NLOAD) load_k1(Int<tt + 5>{}, Int<i - C::NLOAD>{});
      }
      static_for<stage1_upto(j - 2), stage1_upto(j - 1)>(stage3);
      static_for<stage1_upto(j - 1), stage1_upto(j)>(stage2);
      static_for<stage1_upto(j), stage1_upto(j + 1)>(stage1);
      // 32 steps of two values
      constexpr int u0 = j <= M0 ? 0 : cmin(32, 32 * (j - M0) / (M1 - M0)), u1 = j < M0 ? 0 : cmin(32, 32 * (j + 1 - M0) / (M1 - M0));
      static_for<u0, u1>([&](auto u_) __attribute__((always_inline)) {
        constexpr int u = decltype(u_)::value, mg = u % 2, i = u / 2, kb = i / 8, r = 2 * (i % 8);
        mx[mg] = fmaxf(fmaxf(mx[mg], sn[mg][kb][r]), sn[mg][kb][r + 1]);
      });
      if constexpr (j >= M1) ref_step(std::integral_constant<int, j - M1>{});
      if constexpr (j != SB - 1) __builtin_amdgcn_sched_barrier(0);
    });
    l[0] += ls[0];
    l[1] += ls[1];
  };

  f32x16 sa[2][2], sb[2][2];
  if (ntiles > 0) {
    static_for<0, C::NQK>([&](auto c_) __attribute__((always_inline)) {
      constexpr int c = decltype(c_)::value, ks = c / 2, kb = c % 2;
      const bf16x8 a = load_kop(Int<0>{}, c_);
      if constexpr (ks == 0) {
        mfma_first(sa[0][kb], a, qreg[0][ks]);
        mfma_first(sa[1][kb], a, qreg[1][ks]);
      } else {
        mfma_score(sa[0][kb], a, qreg[0][ks]);
        mfma_score(sa[1][kb], a, qreg[1][ks]);
      }
    });
    settle<15>(sa);
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx[g] = fmaxf(mx[g], sa[g][kb][r]);
    static_for<0, 5>(ref_step);
    alpha[0] = alpha[1] = 1.f;         // the first reference: nothing to rescale (the branch of a moved one costs 3600 cycles)
    // the queries and K(0) have been read by everyone; K(1) and V(0) have landed
    wait_vm<3 * C::NLOAD>();
    __syncthreads();
    issue_v(Int<2>{});
    issue_k(Int<4>{});
    static_for<0, AHEAD>([&](auto c_) __attribute__((always_inline)) { op[decltype(c_)::value] = load_kop(Int<1>{}, c_); });
    aim(off_k, ck, false);
    aim(off_v, cv, false);
    for (int t = 0;;) {
      body(sa, sb, t, Int<0>{});
      if (++t >= ntiles) break;
      body(sb, sa, t, Int<1>{});
      if (++t >= ntiles) break;
      body(sa, sb, t, Int<2>{});
      if (++t >= ntiles) break;
      body(sb, sa, t, Int<3>{});
      if (++t >= ntiles) break;
    }
  }

  settle_o<C::NDB>(o);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int r = row0 + wave * 64 + g * 32 + l32;
    const bool row_ok = r < nflagged;                        // the others repeat the last one
    const int row = kHeads ? group_row(min(r, nflagged - 1)) : r;
    const size_t grow = grow_base + row;
    const float l_row = sum_halves(l[g]);
    if constexpr (MODE == kPassInternal) {
      if (row_ok) {
        const bool has_ext = p.ext_o != nullptr;
        float me2 = -INFINITY, le = 0.f;
        if (has_ext) {
          const float em = p.ext_m[grow], el = p.ext_lse[grow];
          if (el != -INFINITY) {
            me2 = em * kLog2e;
            le = exp2f((el - em) * kLog2e);
          }
        }
        const float M2 = fmaxf(me2, mold[g]);
        const float Mu = (M2 == -INFINITY) ? 0.f : M2;
        const float we = exp2f(me2 - Mu), wi = exp2f(mold[g] - Mu);
        const float den = le * we + l_row * wi;
        const float inv = den > 0.f ? 1.f / den : 0.f;
        __bf16* out = (__bf16*)p.out + grow * D;
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const int d0 = 32 * db + 8 * q4 + 4 * h;
            f32x4 e = {0.f, 0.f, 0.f, 0.f};
            if (has_ext) e = *(const f32x4*)(p.ext_o + grow * D + d0);
            float r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = (o[g][db][4 * q4 + i] * wi + e[i] * we) * inv;
            u32x2 pk;
            pk.x = pack_bf16x2(r[0], r[1]);
            pk.y = pack_bf16x2(r[2], r[3]);
            *(u32x2*)(out + d0) = pk;
          }
        if (p.lse_out != nullptr && h == 0) p.lse_out[grow] = den > 0.f ? (M2 + log2f(den)) * kLn2 : -INFINITY;
      }
    } else if (direct) {
      // the final partial: natural-log units, o rescaled to the reference that consumers recover from the rounded m
      if (row_ok) {
        float mo = -INFINITY, lo = -INFINITY, adj = 0.f;
        if (l_row > 0.f) {
          mo = mold[g] * kLn2;
          adj = exp2f(mold[g] - mo * kLog2e);
          lo = (mold[g] + log2f(l_row)) * kLn2;
        }
        float* __restrict__ fin_o = kHeads ? p.o_final : p.ws_o;
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4 o4 = {o[g][db][4 * q4] * adj, o[g][db][4 * q4 + 1] * adj, o[g][db][4 * q4 + 2] * adj, o[g][db][4 * q4 + 3] * adj};
            *(f32x4*)(fin_o + grow * D + 32 * db + 8 * q4 + 4 * h) = o4;
          }
        if (h == 0) {
          (kHeads ? p.m_final : p.ws_m)[grow] = mo;
          (kHeads ? p.l_final : p.ws_l)[grow] = lo;
        }
      }
    } else if (row_ok) {
      // (a branch of its own down to the stores: sharing them with the final partial's costs them their non-temporal hint, and these
      // partials, read once by the combine, then displace K and V in L2)
      const size_t wrow = ((size_t)(split * p.B + b) * (kHeads ? p.heads_cap : p.Hkv) + (kHeads ? rank : kvh)) * nrows + row;
      float* __restrict__ w_o = own_block ? p.ws_o2 : p.ws_o;
#pragma unroll
      for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x4 o4 = {o[g][db][4 * q4], o[g][db][4 * q4 + 1], o[g][db][4 * q4 + 2], o[g][db][4 * q4 + 3]};
          __builtin_nontemporal_store(o4, (f32x4*)(w_o + wrow * D + 32 * db + 8 * q4 + 4 * h));
        }
      if (h == 0) {
        (own_block ? p.ws_m2 : p.ws_m)[wrow] = mold[g];
        (own_block ? p.ws_l2 : p.ws_l)[wrow] = l_row;
      }
    }
  }
  wait_vm<0>();      // the loads past the last tile write to this workgroup's LDS
}

}  // namespace
}  // namespace fb
