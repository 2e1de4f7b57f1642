// fp32 attention pass for gfx950: matrix instructions on fp32 values or on their bf16 parts, softmax statistics exchanged between lanes in
// registers.
//
// Computes the per-row statistics of Eq. 3-4/6 (arxiv 2602.05305, Section 4.2) over a key range, for storage
// type float.  This is the exactness path (max-abs 1e-5 against a float64 reference): sums are fp32, products are fp32
// (v_mfma_f32_16x16x4_f32) or, in 64-row workgroups, made of exact bf16 parts (v_mfma_f32_16x16x32_bf16, off by no more than half an fp32
// step: split_pair; not on short streams at head_dim 64), the running maximum is exact, and every reduction has a fixed order, so results are bit-reproducible.
//
// What bounds it: in 16- and 32-row workgroups the fp32 matrix rate (64 flop per clock and SIMD; 2 x 64 x 16 x D x 2 flop per 16 rows and
// tile), in 64-row ones the vector work of splitting K and V (f32_tile_parts), at the smallest shapes the launch and one memory round trip.  Before this form the pass gave every query row a
// wavefront and accumulated values by shuffle broadcasts: 32 x 128 rows against 4111 keys, head_dim 128, took 353 us.
//
// Work decomposition: one workgroup = WR x 4 wavefronts = WR*RB*16 rows x one range of 64-key tiles.  Wavefront
// (wr, wk) owns rows [16 RB wr, +16 RB) and keys [16 wk, +16) of every tile; the four key quarters meet through LDS
// after the last tile, each wavefront finishing a quarter of the output columns.  Four wavefronts along the keys keep
// the smallest shapes (16 rows) as short as a tile of 64 keys allows; RB = 2 lets every K / V operand feed two MFMAs.
// Rows are group-flattened (all query heads of a KV head share the K/V stream), except in the passes that select per
// query head (per-head refresh, sparse), where a workgroup belongs to one query head and skips what the head skips:
// an unselected key block is then never touched, whatever values it holds.
// Per tile: S^T = K Q^T (A = K rows from LDS, B = Q^T in registers; lane l holds row l%16 and keys 4(l/16)..+3),
//   O^T += V^T P^T with the lane's own probabilities as the B operand: the contraction index of a k-step is the key
//   4(l/16) + r, so nothing moves between lanes.
// Tiles go straight from global memory into two LDS stages (direct-to-LDS loads); the 16-byte chunks of a row are
//   rotated on the global-address side (K: by the row, V: by the row rounded down to 4) so that both read patterns hit
//   all 64 banks.
#include "fb_kernels.h"

namespace fb {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Over the lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float max_quarters(float x) { return max_halves(max_rows(x)); }
__device__ __forceinline__ float sum_quarters(float x) { return sum_halves(sum_rows(x)); }

constexpr bool f32_per_head(int mode) {
  return mode == kPassDenseHeads || mode == kPassSparseRefresh || mode == kPassSparseReuse;
}

// TG > 1: tiles side by side, one per group of 4 WR wavefronts, and a stage for every tile of the stream, kOneTiles at most
// (one-launch refresh step at head_dim 64)
template <int D, int RB, int WR, int TG = 1>
struct FCfg {
  static constexpr int GW = 4 * WR, NW = GW * TG, THREADS = 64 * NW;   // wavefronts of a group, of the workgroup
  static constexpr int ROWS = 16 * RB * WR;             // query rows of a workgroup
  static constexpr int ROWB = D * 4, CPR = ROWB / 16;   // bytes and 16-byte chunks of a key row
  static constexpr int OPB = kKeyTile * ROWB, STAGE = 2 * OPB;
  static constexpr int NLOAD = OPB / (GW * 1024);       // direct-to-LDS loads per lane, operand and tile
  static constexpr int NQ = D / 16;                     // float4 query registers per row block
  static constexpr int NDB = D / 16, NDBK = NDB / 4;    // 16-wide output column blocks; per finishing wavefront
  static constexpr int RING = (TG > 1 ? kOneTiles : 2) * STAGE;
  static constexpr int MERGE = NW * RB * (NDB * 1024 + 512);
  static constexpr int FLAGS = RING > MERGE ? RING : MERGE;
  static constexpr bool kParts = RB == 2 && WR == 2;    // products from bf16 parts (f32_tile_parts)
  static constexpr int LDS = FLAGS + (kParts ? NW * 4 : 0);
  static_assert(LDS <= 160 * 1024 && 2 * NLOAD <= 63, "LDS size and load counter");
  __device__ static __forceinline__ int rot_k(int row) { return row; }
  __device__ static __forceinline__ int rot_v(int row) { return row & ~3; }
};

// Running softmax state of a wavefront: RB blocks of 16 rows (row = lane%16; m is shared by the row's four lanes, l is
// the lane's own share of the row sum), O^T with lane (row, g = lane/16) holding columns 16 db + 4 g .. +3.
template <int RB, int NDB>
struct FState {
  float m[RB], l[RB];
  f32x4 o[RB][NDB];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      m[rb] = -INFINITY;
      l[rb] = 0.f;
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[rb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
};

// Online softmax with an exact running maximum; s becomes the weights.
template <int RB, int NDB>
__device__ __forceinline__ void f32_softmax(FState<RB, NDB>& st, f32x4 (&s)[RB], float scale_log2, int key0, int nvalid) {
  // s[rb][r] = raw dot product of row lane%16 with key key0 + r of the tile (key0 includes the lane's 4 (lane/16))
  if (nvalid < kKeyTile) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (key0 + r >= nvalid) s[rb][r] = -INFINITY;
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    float tmax = fmaxf(fmaxf(s[rb][0], s[rb][1]), fmaxf(s[rb][2], s[rb][3])) * scale_log2;
    tmax = max_quarters(tmax);
    const float m_new = fmaxf(st.m[rb], tmax);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(st.m[rb] - m_use);
    float lsum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[rb][r] = __builtin_amdgcn_exp2f(fmaf(s[rb][r], scale_log2, -m_use));
      lsum += s[rb][r];
    }
    st.l[rb] = st.l[rb] * alpha + lsum;
    st.m[rb] = m_new;
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) st.o[rb][db][r] *= alpha;
    }
  }
}

// An fp32 value as the sum of three bf16 values: the value rounded to bf16, what that left rounded again, the rest.  Exactly, from 2^-110
// (below, the lowest part is a subnormal number and ends at 2^-133: values of 2^-116 come out with a relative error of 2.7e-6) up to the largest
// value that rounds to a finite one; beyond and for infinities a part is NaN (f32_pass).  Of the nine products of two such sums the six largest are kept.  The middle part is at most 2^-8 of the value, the
// lowest 2^-17, so what is left out is below 2^-24 of the product, half an fp32 step, as its own rounding is (2^-24.2 the largest of
// 20 million random pairs; with the upper part cut off instead of rounded 2^-22).  Rounding it costs as many instructions: refresh step, 128 rows of
// 8 KV heads, 4111 keys 32.7 -> 32.9 us, batch 4, 8192 keys 169.9 -> 170.4, head_dim 64, 192 rows, 6000 keys 55.3 -> 56.6.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct Parts {
  u32x4 h, m, l;       // pairs of bf16
};
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  // (a conversion the compiler knows: a product that reads it needs two wait states, which inline assembly does not get)
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  auto round_pair = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2)); };
  h = round_pair(a, b);
  const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
  m = round_pair(ra, rb);
  l = __builtin_amdgcn_perm(__float_as_uint(rb - __uint_as_float(m & 0xffff0000u)), __float_as_uint(ra - __uint_as_float(m << 16)), 0x07060302u);
}
__device__ __forceinline__ Parts split_parts(const f32x4& a, const f32x4& b) {
  Parts p;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    uint32_t h, m, l;
    split_pair(a[2 * i], a[2 * i + 1], h, m, l);
    p.h[i] = h; p.m[i] = m; p.l[i] = l;
    split_pair(b[2 * i], b[2 * i + 1], h, m, l);
    p.h[2 + i] = h; p.m[2 + i] = m; p.l[2 + i] = l;
  }
  return p;
}
__device__ __forceinline__ f32x4 mfma_parts(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 64-row workgroups, but short streams at head_dim 64: products on the bf16 matrix cores.  The fp32 ones take 32 cycles for 16 x 16 x 4, the bf16 ones 16 for 16 x 16 x
// 32, so that six of them take 3072 of 8192 cycles a tile and SIMD; what bounds the tile now is the vector work of splitting K and V
// (11 instructions a pair of values, once for both row blocks).  128 rows of 8 KV heads, 256 workgroups, 8 / 32 tiles each, head_dim
// 128 92 / 172 -> 72 / 132 us, 64 50 -> 41; a refresh step over 4111 keys 33 -> 28.  With one row block, or in the 32-row workgroups,
// whose short streams lose up to 3 % (32 rows, 4096 keys 17.8 -> 18.3), the splitting costs what it saves.  Tried: four row blocks to a
// wavefront, one wavefront per SIMD (half the splitting, but its latencies show: 172 -> 174), operands in five slots, four under way
// (level).
// Sums: the products of the upper parts in one chain, the small ones in another; its error against 64 bits is no larger (4111 keys
// 6.8e-7 -> 5.5e-7, relative).
template <int D>
struct QParts {
  Parts q[2][D / 32];
};
template <int D, int WR>
__device__ __forceinline__ void f32_tile_parts(FState<2, D / 16>& st, const QParts<D>& q, const unsigned char* __restrict__ stage,
                                               const uint32_t (&kaddr)[D / 16], const uint32_t (&vaddr)[D / 16], float scale_log2,
                                               int key0, int nvalid) {
  using C = FCfg<D, 2, WR>;
  f32x4 s[2], small[2];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) s[rb] = small[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < D / 32; ++j) {
    // the lane's eight contraction elements of a step: columns 16 (2 j) + 4 g .. + 3 and 16 (2 j + 1) + 4 g .. + 3, as the queries have them
    const Parts k = split_parts(*(const f32x4*)(stage + kaddr[2 * j]), *(const f32x4*)(stage + kaddr[2 * j + 1]));
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) s[rb] = mfma_parts(k.h, q.q[rb][j].h, s[rb]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) small[rb] = mfma_parts(k.h, q.q[rb][j].l, small[rb]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) small[rb] = mfma_parts(k.h, q.q[rb][j].m, small[rb]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) small[rb] = mfma_parts(k.m, q.q[rb][j].m, small[rb]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) small[rb] = mfma_parts(k.m, q.q[rb][j].h, small[rb]);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) small[rb] = mfma_parts(k.l, q.q[rb][j].h, small[rb]);
  }
  if constexpr (D == 128) {
    // the next step's splitting between this one's products (head_dim 64: level or slower)
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);         // LDS reads
    __builtin_amdgcn_sched_group_barrier(0x002, 44, 0);        // vector instructions
#pragma unroll
    for (int j = 0; j + 1 < D / 32; ++j) {
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // product
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
      }
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 12, 0);
  }
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) s[rb] += small[rb];
  f32_softmax<2, C::NDB>(st, s, scale_log2, key0, nvalid);
  // contraction elements 0 .. 3 of a lane: its four keys in one part, 4 .. 7: the same keys in another, so that a product of 32 takes
  // two of the six: (h, m) x (h, h), (h, m) x (m, m), (l, h) x (h, l)
  u32x4 p_hh[2], p_mm[2], p_hl[2];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    uint32_t h0, m0, l0, h1, m1, l1;
    split_pair(s[rb][0], s[rb][1], h0, m0, l0);
    split_pair(s[rb][2], s[rb][3], h1, m1, l1);
    p_hh[rb] = u32x4{h0, h1, h0, h1};
    p_mm[rb] = u32x4{m0, m1, m0, m1};
    p_hl[rb] = u32x4{h0, h1, l0, l1};
  }
  // at head_dim 128 two column blocks at a time: four chains of products instead of two that wait for themselves
  constexpr int NB = D == 128 ? 2 : 1;
#pragma unroll
  for (int d0 = 0; d0 < C::NDB; d0 += NB) {
    u32x4 hm[NB], lh[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = *(const float*)(stage + C::OPB + vaddr[d0 + i] + r * C::ROWB);
      uint32_t h0, m0, l0, h1, m1, l1;
      split_pair(v[0], v[1], h0, m0, l0);
      split_pair(v[2], v[3], h1, m1, l1);
      hm[i] = u32x4{h0, h1, m0, m1};
      lh[i] = u32x4{l0, l1, h0, h1};
    }
#pragma unroll
    for (int x = 0; x < 2 * NB; ++x) st.o[x % 2][d0 + x / 2] = mfma_parts(lh[x / 2], p_hl[x % 2], st.o[x % 2][d0 + x / 2]);
#pragma unroll
    for (int x = 0; x < 2 * NB; ++x) st.o[x % 2][d0 + x / 2] = mfma_parts(hm[x / 2], p_mm[x % 2], st.o[x % 2][d0 + x / 2]);
#pragma unroll
    for (int x = 0; x < 2 * NB; ++x) st.o[x % 2][d0 + x / 2] = mfma_parts(hm[x / 2], p_hh[x % 2], st.o[x % 2][d0 + x / 2]);
  }
  if constexpr (D == 128) {
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 88, 0);
#pragma unroll
    for (int d0 = NB; d0 < C::NDB; d0 += NB) {
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
      }
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 12, 0);
  }
}

template <int D, int RB, int WR>
__device__ __forceinline__ void f32_tile(FState<RB, D / 16>& st, const f32x4 (&q)[RB][D / 16],
                                         const unsigned char* __restrict__ stage, const uint32_t (&kaddr)[D / 16],
                                         const uint32_t (&vaddr)[D / 16], float scale_log2, int key0, int nvalid) {
  using C = FCfg<D, RB, WR>;
  // two accumulator chains at least: a chain's product waits for the one before it
  constexpr int NC = RB == 1 ? 2 : 1;
  f32x4 s[RB], part[NC][RB];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) part[c][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < C::NQ; ++j) {
    const f32x4 a = *(const f32x4*)(stage + kaddr[j]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        part[i % NC][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], q[rb][j][i], part[i % NC][rb], 0, 0, 0);
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) s[rb] = NC == 1 ? part[0][rb] : part[0][rb] + part[NC - 1][rb];
  f32_softmax<RB, C::NDB>(st, s, scale_log2, key0, nvalid);
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int db = 0; db < C::NDB; ++db) {
      const float a = *(const float*)(stage + C::OPB + vaddr[db] + r * C::ROWB);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        st.o[rb][db] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, s[rb][r], st.o[rb][db], 0, 0, 0);
    }
}

// Products of a pass: fp32; of bf16 parts; fp32 again, half of the rows at a time, where those of parts gave a NaN.
enum F32Products : int { kProductsF32, kProductsParts, kProductsAgain };

// The pass of one workgroup.  kProductsParts: false, and nothing stored, where a NaN came out.  half: of the rows, kProductsAgain.
template <int D, int MODE, int RB, int WR, int TG, int PRODUCTS>
__device__ __forceinline__ bool f32_pass(const PassParams& p, unsigned char* ring, int half = 0) {
  constexpr bool PARTS = PRODUCTS == kProductsParts;
  using C = FCfg<D, RB, WR, TG>;
  constexpr bool kPerHead = f32_per_head(MODE);
  // kPassRefreshOne, a whole refresh step in one launch: the prefix's tiles and then the block's own are one stream with two sets
  // of statistics; the first one is written as the final partial, then the second is merged in (Eq. 8-9)
  constexpr bool kOne = (MODE == kPassRefreshOne);
  constexpr int NSETS = (MODE == kPassSparseRefresh || kOne) ? 2 : 1;
  constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
  // the lane's number anew, so that nothing made of it is kept in a register meanwhile
  auto lane_again = [](int& x) __attribute__((always_inline)) {
    x = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(x));
  };
  int lane = threadIdx.x & 63, wg = blockIdx.x;
  if constexpr (PRODUCTS == kProductsAgain) {
    lane_again(lane);
    asm volatile("" : "+s"(wg));
  }
  int l16 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wk = wave & 3, wr = (wave >> 2) % WR, tg = TG == 1 ? 0 : wave / C::GW, gwave = TG == 1 ? wave : wave % C::GW;
  static_assert(TG == 1 || MODE == kPassRefreshOne, "tile groups");

  // ---- workgroup -> (row tile, split, head, batch); each XCD gets a contiguous range so that row tiles and heads that
  // share K/V share an L2 (ragged paged sequences are dealt round-robin instead)
  int rt;
  uint32_t rest;
  if constexpr (MODE == kPassDensePaged) {
    const uint32_t j = (uint32_t)wg >> 3, xcd = wg & 7;
    const uint32_t jq = fastdiv(j, p.div_rowtiles);
    rt = (int)(j - jq * p.div_rowtiles.d);
    rest = jq * 8 + xcd;
    if (rest >= (uint32_t)(p.B * p.Hkv * p.nsplit)) return true;   // workgroup-uniform
  } else {
    const int bid = wg, q8 = gridDim.x / 8, r8 = gridDim.x % 8, xcd = bid % 8;
    const int w = (xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8) + bid / 8;
    rest = fastdiv((uint32_t)w, p.div_rowtiles);
    rt = w - (int)(rest * p.div_rowtiles.d);
  }
  const uint32_t r2 = fastdiv(rest, p.div_nsplit);            // divisor: splits (+ 1 in the fused pass: the block's keys)
  const int split = (int)(rest - r2 * p.div_nsplit.d);
  int b = (int)fastdiv(r2, p.div_hkv);                        // divisor: query heads (per-head passes) or KV heads
  const int unit_h = (int)(r2 - (uint32_t)b * p.div_hkv.d);
  if constexpr (MODE == kPassDensePaged) {
    if (p.seq_order != nullptr) b = sload(p.seq_order, b);
  }
  const int kvh = kPerHead ? unit_h / p.G : unit_h;
  const int nrows = kPerHead ? p.Bq : p.G * p.Bq;
  const size_t grow_base = (size_t)(b * p.Hq + (kPerHead ? unit_h : unit_h * p.G)) * p.Bq;
  if constexpr (MODE == kPassDenseHeads) {
    if (p.head_on[b * p.Hq + unit_h] == 0) return true;       // this head keeps its cached partial
  }
  const int bk = b * p.Hkv + kvh;
  const bool own_block = (MODE == kPassRefreshFused) && (split == p.nsplit);
  int nkeys = own_block ? p.Bq : p.nkeys;
  if constexpr (MODE == kPassDensePaged) nkeys = min(p.nkeys, max(0, sload(p.prefix_lens, b)));   // this sequence's prefix

  // contiguous cache: this KV head's [nkeys, D] slab; paged cache: the pool (tiles add their page offset)
  const size_t slab = (MODE == kPassDensePaged) ? (size_t)0 : (size_t)bk * nkeys * C::ROWB;
  const unsigned char* __restrict__ Kg = (const unsigned char*)(own_block ? p.k2 : p.k) + slab;
  const unsigned char* __restrict__ Vg = (const unsigned char*)(own_block ? p.v2 : p.v) + slab;

  // ---- tile list; tiles that this workgroup's head sits out are never fetched
  int tpb = 1, total;
  if constexpr (MODE == kPassSparseReuse) {
    tpb = p.key_block / kKeyTile;
    total = sload(p.union_cnt, bk) * tpb;
  } else {
    total = (nkeys + kKeyTile - 1) / kKeyTile;
  }
  const int prefix_tiles = total;
  if constexpr (kOne) total += (p.Bq + kKeyTile - 1) / kKeyTile;
  TileRange tr = {0, total};
  if (MODE != kPassInternal && !kOne && !own_block) tr = split_range(total, p.nsplit, split);
  struct Tile {
    int k0;
    bool is_sel;
    size_t off;      // bytes from Kg / Vg
  };
  int e_next = tr.begin + tg;
  auto next_tile = [&](Tile& t) -> bool {
    for (; e_next < tr.end; e_next += TG) {
      t.is_sel = true;
      if constexpr (MODE == kPassSparseReuse) {
        const int blk = sload(p.union_list + (size_t)bk * p.nblk, e_next / tpb);
        t.k0 = blk * p.key_block + kKeyTile * (e_next % tpb);
        const uint32_t mask = (uint32_t)sload(p.blk_mask + (size_t)bk * p.nblk, blk);
        if (!((mask >> (unit_h - kvh * p.G)) & 1u) || t.k0 >= nkeys) continue;
      } else {
        t.k0 = e_next * kKeyTile;
        if constexpr (kOne) {
          t.is_sel = e_next < prefix_tiles;
          if (!t.is_sel) t.k0 -= prefix_tiles * kKeyTile;
        }
        if constexpr (MODE == kPassSparseRefresh) {
          const uint32_t mask = (uint32_t)sload(p.blk_mask + (size_t)bk * p.nblk, t.k0 / p.key_block);
          t.is_sel = ((mask >> (unit_h - kvh * p.G)) & 1u) != 0u;
        }
      }
      if constexpr (MODE == kPassDensePaged) {
        const int slot = (int)fastdiv((uint32_t)t.k0, p.div_page);
        const int page = min(max(sload(p.block_table + (size_t)b * p.max_pages, slot), 0), p.num_pages - 1);
        t.off = (((size_t)page * p.Hkv + kvh) * p.page_size + (t.k0 - slot * (int)p.div_page.d)) * C::ROWB;
      } else {
        t.off = (size_t)t.k0 * C::ROWB;
      }
      e_next += TG;
      return true;
    }
    return false;
  };

  auto keys_of = [&](const Tile& t) -> int { return kOne && !t.is_sel ? p.Bq : nkeys; };

  // ---- direct-to-LDS load slots: operand chunk (j*NW + wave)*64 + lane lives at LDS row chunk / CPR, position chunk % CPR
  const uint32_t ring_base = (uint32_t)(uintptr_t)ring;
  auto issue = [&](const Tile& t, int stage_i) {
    const uint32_t base = ring_base + (uint32_t)stage_i * C::STAGE + gwave * 1024;
    const int last = min(kKeyTile, keys_of(t) - t.k0) - 1;    // rows past the end read the last key (masked below)
    const unsigned char* kt = Kg + t.off;
    const unsigned char* vt = Vg + t.off;
    if constexpr (kOne) {
      if (!t.is_sel) {
        kt = (const unsigned char*)p.k2 + (size_t)bk * p.Bq * C::ROWB + t.off;
        vt = (const unsigned char*)p.v2 + (size_t)bk * p.Bq * C::ROWB + t.off;
      }
    }
#pragma unroll
    for (int j = 0; j < C::NLOAD; ++j) {
      const int chunk = (j * C::GW + gwave) * 64 + lane, r = chunk / C::CPR, pc = chunk % C::CPR;
      dma16(kt, (uint32_t)(min(r, last) * C::ROWB + ((pc - C::rot_k(r)) & (C::CPR - 1)) * 16),
            base + j * C::GW * 1024);
    }
#pragma unroll
    for (int j = 0; j < C::NLOAD; ++j) {
      const int chunk = (j * C::GW + gwave) * 64 + lane, r = chunk / C::CPR, pc = chunk % C::CPR;
      dma16(vt, (uint32_t)(min(r, last) * C::ROWB + ((pc - C::rot_v(r)) & (C::CPR - 1)) * 16),
            base + C::OPB + j * C::GW * 1024);
    }
  };

  Tile t0 = {0, true, 0}, t1 = {0, true, 0}, t2 = {0, true, 0};
  bool have0 = next_tile(t0);
  if (have0) issue(t0, tg);
  // queries: rows past the end read the group's last row; what they compute is never stored
  const int row0 = (PRODUCTS == kProductsAgain ? 2 * rt + half : rt) * C::ROWS + wr * 16 * RB;
  f32x4 q[RB][C::NQ];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float* qr = (const float*)p.q + (grow_base + min(row0 + 16 * rb + l16, nrows - 1)) * D + 4 * g4;
#pragma unroll
    for (int j = 0; j < C::NQ; ++j) q[rb][j] = *(const f32x4*)(qr + 16 * j);
  }
  QParts<D> qp;
  if constexpr (PARTS) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < D / 32; ++j) qp.q[rb][j] = split_parts(q[rb][2 * j], q[rb][2 * j + 1]);
  }
  // the wait for the queries belongs here: in the loop it would also wait for the tiles in flight
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int j = 0; j < C::NQ; ++j) {
      if constexpr (PARTS) asm volatile("" ::"v"(qp.q[rb][j / 2].h));
      else asm volatile("" ::"v"(q[rb][j]));
    }
  bool have1 = have0 && next_tile(t1);
  if (have1) issue(t1, tg + TG);

  // per-lane LDS read addresses inside a stage
  uint32_t kaddr[C::NQ], vaddr[C::NDB];
  {
    const int krow = 16 * wk + l16, vrow = 16 * wk + 4 * g4;
#pragma unroll
    for (int j = 0; j < C::NQ; ++j) kaddr[j] = (uint32_t)(krow * C::ROWB + ((4 * j + g4 + C::rot_k(krow)) & (C::CPR - 1)) * 16);
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
      vaddr[db] = (uint32_t)(vrow * C::ROWB + ((4 * db + (l16 >> 2) + C::rot_v(vrow)) & (C::CPR - 1)) * 16 + (l16 & 3) * 4);
  }

  FState<RB, C::NDB> sets[NSETS];
#pragma unroll
  for (int i = 0; i < NSETS; ++i) sets[i].init();

  bool have3 = false;
  Tile t3 = {0, true, 0};
  if constexpr (TG > 1) {                                       // everything is requested here; no stage is used twice
    static_assert(3 * TG >= kOneTiles, "three tiles a group");
    have3 = have1 && next_tile(t3);
    if (have3) issue(t3, tg + 2 * TG);
    wait_vm<0>();
    __syncthreads();
  }
  for (int t = 0; have0; ++t) {
    if constexpr (TG == 1) {
      if (have1) wait_vm<2 * C::NLOAD>();
      else wait_vm<0>();
      __syncthreads();
    }
    unsigned char* stage = ring + (TG > 1 ? tg + t * TG : t & 1) * C::STAGE;
    const int nvalid = min(kKeyTile, keys_of(t0) - t0.k0);
    if (nvalid < kKeyTile) {
      // value rows past the end: a weight of 0 must not meet an infinity or NaN of the duplicated last key.  A wavefront reads
      // the rows of its own 16 keys and clears them itself.
      for (int c = max(nvalid, 16 * wk) * C::CPR + lane; c < (16 * wk + 16) * C::CPR; c += 64)
        *(f32x4*)(stage + C::OPB + c * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
      // other lanes of the wavefront read them: LDS keeps the order by itself, the compiler is told (no instruction)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    const int key0 = 16 * wk + 4 * g4;
    auto tile = [&](FState<RB, C::NDB>& st) __attribute__((always_inline)) {
      if constexpr (PARTS) f32_tile_parts<D, WR>(st, qp, stage, kaddr, vaddr, p.scale_log2, key0, nvalid);
      else f32_tile<D, RB, WR>(st, q, stage, kaddr, vaddr, p.scale_log2, key0, nvalid);
    };
    if (NSETS > 1 && !t0.is_sel) tile(sets[NSETS - 1]);
    else tile(sets[0]);
    const bool have2 = TG > 1 ? have3 : have1 && next_tile(t2);      // workgroup-uniform (several groups: group-uniform)
    if constexpr (TG > 1) {
      t2 = t3;
      have3 = false;
    } else if (have2) {
      __syncthreads();                                        // every wavefront has left this stage
      issue(t2, t & 1);
    }
    t0 = t1;
    t1 = t2;
    have0 = have1;
    have1 = have2;
  }

  [[maybe_unused]] int* flags = (int*)(ring + C::FLAGS);
  if constexpr (PARTS) {
    lane_again(lane);
    l16 = lane & 15;
    g4 = lane >> 4;
    // a NaN in the row sums: a score was one; in the accumulators: a value had no parts, and that shows in every row of the wavefront
    float x = 0.f;
#pragma unroll
    for (int i = 0; i < NSETS; ++i) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) x = __builtin_elementwise_maximum(x, sets[i].l[rb]);
#pragma unroll
      for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) x = __builtin_elementwise_maximum(x, sets[i].o[0][db][r]);
    }
    const int nan = __any(x != x);
    if (lane == 0) flags[wave] = nan;
  }

  // ---- the four key quarters of a row block meet in LDS: records [wavefront][row block][column block][lane], then
  // (m, l) per lane; wavefront wk finishes column blocks [wk*NDBK, +NDBK), folding the quarters in order
  float pm[kOne ? RB : 1], pl[kOne ? RB : 1];                   // kPassRefreshOne: the prefix's statistics
  f32x4 po[kOne ? RB : 1][C::NDBK];
#pragma unroll
  for (int i = 0; i < NSETS; ++i) {
    __syncthreads();
    f32x4* rec_o = (f32x4*)ring;
    float2* rec_ml = (float2*)(ring + C::NW * RB * C::NDB * 1024);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float l = sets[i].l[rb];
      l = sum_quarters(l);
#pragma unroll
      for (int db = 0; db < C::NDB; ++db) rec_o[((wave * RB + rb) * C::NDB + db) * 64 + lane] = sets[i].o[rb][db];
      rec_ml[(wave * RB + rb) * 64 + lane] = make_float2(sets[i].m[rb], l);
    }
    __syncthreads();
    if constexpr (PARTS) {
      if (i == 0 && __any(flags[lane & (C::NW - 1)])) return false;        // workgroup-uniform
    }
    if (TG > 1 && tg != 0) continue;                          // the first group finishes
    constexpr int NR = 4 * TG;                                // records of a row block: key quarter by quarter, group by group
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int row = row0 + 16 * rb + l16;
      const bool row_ok = row < nrows;
      const size_t grow = grow_base + row;
      float mq[NR], lq[NR], M = -INFINITY;
#pragma unroll
      for (int w = 0; w < NR; ++w) {
        const float2 ml = rec_ml[(((w / 4 * WR + wr) * 4 + w % 4) * RB + rb) * 64 + lane];
        mq[w] = ml.x;
        lq[w] = ml.y;
        M = fmaxf(M, ml.x);
      }
      const float Mu = (M == -INFINITY) ? 0.f : M;
      float l = 0.f;
      f32x4 o[C::NDBK];
#pragma unroll
      for (int d = 0; d < C::NDBK; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NR; ++w) {
        const float wgt = __builtin_amdgcn_exp2f(mq[w] - Mu);
        l = fmaf(lq[w], wgt, l);
#pragma unroll
        for (int d = 0; d < C::NDBK; ++d) {
          const f32x4 x = rec_o[((((w / 4 * WR + wr) * 4 + w % 4) * RB + rb) * C::NDB + wk * C::NDBK + d) * 64 + lane];
#pragma unroll
          for (int r = 0; r < 4; ++r) o[d][r] = fmaf(x[r], wgt, o[d][r]);
        }
      }
      if (!row_ok) continue;
      const int d0 = wk * C::NDBK * 16 + 4 * g4;              // first column of o[0]; o[d] is 16 d further
      const bool writes_ml = (wk == 0 && g4 == 0);
      if constexpr (kOne) {
        if (i == 0) {
          pm[rb] = M;
          pl[rb] = l;
#pragma unroll
          for (int d = 0; d < C::NDBK; ++d) po[rb][d] = o[d];
        }
      }
      if (MODE == kPassInternal || (kOne && i == 1)) {
        // Eq. 8-9 with the cached pair expressed through (o, m, lse): A_out e^{L_out-M} = o e^{m-M}.
        float me2 = -INFINITY, le = 0.f;
        if constexpr (kOne) {
          me2 = pm[rb];
          le = pl[rb];
        } else if (p.ext_o != nullptr) {
          const float me = p.ext_m[grow], lse = p.ext_lse[grow];
          if (lse != -INFINITY) {
            me2 = me * kLog2e;
            le = exp2f((lse - me) * kLog2e);
          }
        }
        const float M2 = fmaxf(me2, M);
        const float M2u = (M2 == -INFINITY) ? 0.f : M2;
        const float we = exp2f(me2 - M2u), wi = exp2f(M - M2u);
        const float den = le * we + l * wi;
        const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
        for (int d = 0; d < C::NDBK; ++d) {
          f32x4 num = o[d] * wi;
          if (le > 0.f) {
            const f32x4 x = kOne ? po[kOne ? rb : 0][d] : *(const f32x4*)(p.ext_o + grow * D + d0 + 16 * d);
#pragma unroll
            for (int r = 0; r < 4; ++r) num[r] = fmaf(x[r], we, num[r]);
          }
          *(f32x4*)((float*)p.out + grow * D + d0 + 16 * d) = num * inv;
        }
        if (p.lse_out != nullptr && writes_ml) p.lse_out[grow] = den > 0.f ? (M2 + log2f(den)) * kLn2 : -INFINITY;
      } else {
        if (kOne || p.direct) {
          // single split: this is the final partial; same unit conversion as the split combine
          float m_nat = -INFINITY, L = -INFINITY, adj = 0.f;
          if (l > 0.f) {
            m_nat = M * kLn2;
            adj = exp2f(M - m_nat * kLog2e);
            L = (M + log2f(l)) * kLn2;
          }
#pragma unroll
          for (int d = 0; d < C::NDBK; ++d) *(f32x4*)(p.ws_o + grow * D + d0 + 16 * d) = o[d] * adj;
          if (writes_ml) {
            p.ws_m[grow] = m_nat;
            p.ws_l[grow] = L;
          }
        } else {
          const bool set1 = own_block || i == 1;              // residual keys, or the block's own keys
          const size_t rows_total = (size_t)p.B * p.Hq * p.Bq;
          const size_t wrow = (own_block ? (size_t)0 : (size_t)split * rows_total) + grow;
          float* __restrict__ w_o = set1 ? p.ws_o2 : p.ws_o;
          float* __restrict__ w_m = set1 ? p.ws_m2 : p.ws_m;
          float* __restrict__ w_l = set1 ? p.ws_l2 : p.ws_l;
#pragma unroll
          for (int d = 0; d < C::NDBK; ++d) *(f32x4*)(w_o + wrow * D + d0 + 16 * d) = o[d];
          if (writes_ml) {
            w_m[wrow] = M;
            w_l[wrow] = l;
          }
        }
      }
    }
  }
  return true;
}

// 64-row workgroups: an infinity has no parts (its remainder is NaN), a part of 0 must not meet one, and parts of opposite signs may
// overflow where their sum does not.  All of it leaves a NaN in the row sums or the accumulators of the pass by parts; such a
// workgroup does its pass over again with the fp32 products, so that a value counts for what it does in the other workgroups.
template <int D, int MODE, int RB, int WR, int TG = 1, bool PARTS = FCfg<D, RB, WR, TG>::kParts>
__global__ __launch_bounds__(256 * WR * TG, 1) void attn_f32_kernel(const PassParams p) {
  extern __shared__ __align__(16) unsigned char ring[];
  if constexpr (PARTS) {
    if (f32_pass<D, MODE, RB, WR, TG, kProductsParts>(p, ring)) return;
    // (p is the only argument: read again from where the arguments are, instead of kept in registers throughout the first pass)
    typedef const __attribute__((address_space(4))) PassParams* Args;
    Args args = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      __syncthreads();                                          // the flags, and the first half's records, have been read
      f32_pass<D, MODE, RB / 2, WR, TG, kProductsAgain>(*(const PassParams*)args, ring, half);
    }
  } else {
    f32_pass<D, MODE, RB, WR, TG, kProductsF32>(p, ring);
  }
}

// Attention mass per (query row, key block): sum over the block's keys of exp(s - lse), fp32 storage.
// One wavefront per query row, 4 rows of one query head per workgroup, lane j scores key j of a tile staged in LDS.
template <int D>
__global__ __launch_bounds__(256) void block_mass_f32_kernel(const MassParams p) {
  constexpr int KSTR = D + 4;
  constexpr float kLog2e = 1.4426950408889634f;
  __shared__ __align__(16) float Ks[kKeyTile * KSTR];
  __shared__ __align__(16) float Qs[4 * D];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int chunk = blockIdx.x, bh = blockIdx.y, split = blockIdx.z;
  const int b = bh / p.Hq, h = bh % p.Hq, kvh = h / p.G;
  const int row = chunk * 4 + wave, nkeys = p.nkeys;
  const bool valid = row < p.Bq;
  const float* __restrict__ Q = (const float*)p.q + (size_t)bh * p.Bq * D;
  const float* __restrict__ K = (const float*)p.k + (size_t)(b * p.Hkv + kvh) * nkeys * D;
  for (int i = tid; i < 4 * D; i += 256) {
    const int r = chunk * 4 + i / D;
    Qs[i] = (r < p.Bq) ? Q[(size_t)r * D + (i % D)] : 0.f;
  }
  const float lse = valid ? p.lse[(size_t)bh * p.Bq + row] : 0.f;
  const bool live = lse != -INFINITY;
  const float lse2 = live ? lse * kLog2e : 0.f;
  const int tpb = p.key_block / kKeyTile;
  const TileRange br = split_range(p.nblk, p.nsplit, split);
  const int t0 = br.begin * tpb, t1 = min(br.end * tpb, (nkeys + kKeyTile - 1) / kKeyTile);
  float acc = 0.f;
  for (int t = t0; t < t1; ++t) {
    const int k0 = t * kKeyTile;
    __syncthreads();
    for (int c = tid; c < kKeyTile * (D / 4); c += 256) {
      const int r = c / (D / 4), c4 = c % (D / 4);
      float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k0 + r < nkeys) val = *(const float4*)(K + (size_t)(k0 + r) * D + c4 * 4);
      *(float4*)(Ks + r * KSTR + c4 * 4) = val;
    }
    __syncthreads();
    const float4* kr = (const float4*)(Ks + lane * KSTR);
    const float4* qr = (const float4*)(Qs + wave * D);
    float s = 0.f;
#pragma unroll 8
    for (int i = 0; i < D / 4; ++i) {
      const float4 a = kr[i], c = qr[i];
      s = fmaf(a.x, c.x, s);
      s = fmaf(a.y, c.y, s);
      s = fmaf(a.z, c.z, s);
      s = fmaf(a.w, c.w, s);
    }
    acc += (k0 + lane < nkeys) ? exp2f(s * p.scale_log2 - lse2) : 0.f;
    if ((t + 1) % tpb == 0 || t + 1 == t1) {
      const float tot = wave_sum(acc);
      if (valid && lane == 0)
        p.rowmass[((size_t)b * p.nblk + t / tpb) * ((size_t)p.Hq * p.Bq) + (size_t)h * p.Bq + row] = live ? tot : 0.f;
      acc = 0.f;
    }
  }
}

// At most 16 keys (the small blocks' internal pass, a prefix that short): one wavefront per query row, no LDS, no barrier.  A
// tile of 64 keys costs the same loads and matrix products however few of its keys exist; here everything is requested at once
// (lane = key x quarter of the score product; 64 lanes across the columns of V and of the cached partial).
// What bounds it is launch and one memory round trip.  (128 rows of 8 KV heads, head_dim 128, blocks of 4: 6.9 us with 16-row
// workgroups, 5.2 with the earlier form that staged K in LDS, 3.7 so.)
template <int D, int MODE>
__global__ __launch_bounds__(256) void attn_f32_few_kernel(const PassParams p) {
  static_assert(MODE == kPassInternal || MODE == kPassDense, "unsplit passes");
  constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
  constexpr int NC = D / 64, NQ4 = D / 16;
  typedef float colv __attribute__((ext_vector_type(NC)));
  const int lane = threadIdx.x & 63, key = lane >> 2, part = lane & 3;
  const uint32_t row = blockIdx.x * 4 + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // batch, head, block row
  if (row >= (uint32_t)(p.B * p.Hq * p.Bq)) return;           // wavefront-uniform
  const int nkeys = p.nkeys;
  const size_t bk = fastdiv(row, p.div_rowtiles);             // divisor: rows of a KV group
  const float* __restrict__ Q = (const float*)p.q + (size_t)row * D;
  const float* __restrict__ K = (const float*)p.k + bk * nkeys * D;
  const float* __restrict__ V = (const float*)p.v + bk * nkeys * D + lane * NC;
  f32x4 k4[NQ4], q4[NQ4];
#pragma unroll
  for (int i = 0; i < NQ4; ++i) {
    k4[i] = *(const f32x4*)(K + (size_t)min(key, nkeys - 1) * D + (part + 4 * i) * 4);
    q4[i] = *(const f32x4*)(Q + (part + 4 * i) * 4);
  }
  colv v[kFewKeysF32];
#pragma unroll
  for (int j = 0; j < kFewKeysF32; ++j) v[j] = *(const colv*)(V + (size_t)min(j, nkeys - 1) * D);
  const bool has_ext = MODE == kPassInternal && p.ext_o != nullptr;      // uniform
  float em = -INFINITY, el = -INFINITY;
  colv eo = 0.f;
  if (has_ext) {
    em = p.ext_m[row];
    el = p.ext_lse[row];
    eo = *(const colv*)(p.ext_o + (size_t)row * D + lane * NC);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NQ4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) s = fmaf(k4[i][r], q4[i][r], s);
  // the four lanes of a key (DPP quad_perm: l ^ 1, l ^ 2)
  s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0xb1, 0xf, 0xf, false));
  s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x4e, 0xf, 0xf, false));
  if (key >= nkeys) s = -INFINITY;
  float m = s * p.scale_log2;
  m = fmaxf(m, swap_quads(m));
  m = max_quarters(fmaxf(m, turn16<8>(m)));
  const float m_use = (m == -INFINITY) ? 0.f : m;
  const float w = __builtin_amdgcn_exp2f(fmaf(s, p.scale_log2, -m_use));
  // in the same order on every lane: all columns of a row are divided by the same denominator
  float l = w + swap_quads(w);
  l = sum_quarters(l + turn16<8>(l));
  colv o = 0.f;
#pragma unroll
  for (int j = 0; j < kFewKeysF32; ++j)
    if (j < nkeys) {                                          // uniform: a weight of 0 must not meet the duplicated last key
      const float wj = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(w), 4 * j));
#pragma unroll
      for (int c = 0; c < NC; ++c) o[c] = fmaf(wj, v[j][c], o[c]);
    }
  if constexpr (MODE == kPassInternal) {
    // Eq. 8-9 with the cached pair expressed through (o, m, lse): A_out e^{L_out-M} = o e^{m-M}.
    float me2 = -INFINITY, le = 0.f;
    if (el != -INFINITY) {
      me2 = em * kLog2e;
      le = exp2f((el - em) * kLog2e);
    }
    const float M2 = fmaxf(me2, m);
    const float M2u = (M2 == -INFINITY) ? 0.f : M2;
    const float we = exp2f(me2 - M2u), wi = exp2f(m - M2u);
    const float den = le * we + l * wi;
    const float inv = den > 0.f ? 1.f / den : 0.f;
    colv num = o * wi;
    if (le > 0.f) {
#pragma unroll
      for (int c = 0; c < NC; ++c) num[c] = fmaf(eo[c], we, num[c]);
    }
    *(colv*)((float*)p.out + (size_t)row * D + lane * NC) = num * inv;
    if (p.lse_out != nullptr && lane == 0) p.lse_out[row] = den > 0.f ? (M2 + log2f(den)) * kLn2 : -INFINITY;
  } else {
    // the final partial; same unit conversion as the split combine
    float m_nat = -INFINITY, L = -INFINITY, adj = 0.f;
    if (l > 0.f) {
      m_nat = m * kLn2;
      adj = exp2f(m - m_nat * kLog2e);
      L = (m + log2f(l)) * kLn2;
    }
    *(colv*)(p.ws_o + (size_t)row * D + lane * NC) = o * adj;
    if (lane == 0) {
      p.ws_m[row] = m_nat;
      p.ws_l[row] = L;
    }
  }
}

// Internal pass over 17 to 64 keys, few rows: every wavefront is a workgroup of its own and finishes 16 rows x 32 output
// columns without LDS and without a barrier (the fp32 form of internal_wave_kernel in fb_attn_bf16.hip).  What bounds it is
// launch, one memory round trip and one wavefront's products: K and Q rows in matrix operand order and V's single elements are
// requested at once, with the cached partial; the D / 32 wavefronts of a row block repeat its scores.  (Against 16-row workgroups of
// 4 wavefronts that stage a tile of 64 keys in LDS: 128 rows of 8 KV heads, blocks of 32, 6.7 -> 4.8 us.)
template <int D, int NKQ>
__global__ __launch_bounds__(64) void internal_f32_wave_kernel(const PassParams p) {
  constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
  constexpr int NQ = D / 16, NW = D / 32;
  const int lane = threadIdx.x, l16 = lane & 15, g4 = lane >> 4;
  // one KV head's workgroups on one XCD: they share K, V and Q rows
  const int bid = blockIdx.x, q8 = gridDim.x / 8, r8 = gridDim.x % 8, xcd = bid % 8;
  const uint32_t w = (uint32_t)((xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8) + bid / 8);
  const int cw = (int)(w % NW);                                  // 32-column group
  const uint32_t rg = w / NW;
  const uint32_t bk = fastdiv(rg, p.div_rowtiles);               // batch * Hkv + KV head
  const int rt = (int)(rg - bk * p.div_rowtiles.d);
  const int nrows = p.G * p.Bq, nkeys = p.nkeys;
  const int row = rt * 16 + l16;
  const bool row_ok = row < nrows;
  const size_t grow = (size_t)bk * nrows + min(row, nrows - 1);   // rows past the end read the last row; never stored
  const float* __restrict__ Q = (const float*)p.q + grow * D + 4 * g4;
  const float* __restrict__ K = (const float*)p.k + (size_t)bk * nkeys * D;
  const float* __restrict__ V = (const float*)p.v + (size_t)bk * nkeys * D + 32 * cw;
  f32x4 kr[NKQ][NQ], qr[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) qr[j] = *(const f32x4*)(Q + 16 * j);
#pragma unroll
  for (int u = 0; u < NKQ; ++u)
#pragma unroll
    for (int j = 0; j < NQ; ++j) kr[u][j] = *(const f32x4*)(K + (size_t)min(16 * u + l16, nkeys - 1) * D + 16 * j + 4 * g4);
  float vr[NKQ][4][2];                                            // key 16 u + 4 g4 + r, column 16 db + l16
#pragma unroll
  for (int u = 0; u < NKQ; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int db = 0; db < 2; ++db) vr[u][r][db] = V[(size_t)min(16 * u + 4 * g4 + r, nkeys - 1) * D + 16 * db + l16];
  const bool has_ext = p.ext_o != nullptr;                        // uniform
  f32x4 eo[2];
  float em = -INFINITY, el = -INFINITY;
  if (has_ext) {
    em = p.ext_m[grow];
    el = p.ext_lse[grow];
#pragma unroll
    for (int db = 0; db < 2; ++db) eo[db] = *(const f32x4*)(p.ext_o + grow * D + 32 * cw + 16 * db + 4 * g4);
  }
  f32x4 s[NKQ];
#pragma unroll
  for (int u = 0; u < NKQ; ++u) s[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int u = 0; u < NKQ; ++u) s[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[u][j][i], qr[j][i], s[u], 0, 0, 0);
  float m = -INFINITY;
#pragma unroll
  for (int u = 0; u < NKQ; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (16 * u + 4 * g4 + r >= nkeys) s[u][r] = -INFINITY;
      m = fmaxf(m, s[u][r]);
    }
  m *= p.scale_log2;
  m = max_quarters(m);
  const float m_use = (m == -INFINITY) ? 0.f : m;
  float l = 0.f;
#pragma unroll
  for (int u = 0; u < NKQ; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[u][r] = __builtin_amdgcn_exp2f(fmaf(s[u][r], p.scale_log2, -m_use));
      l += s[u][r];
    }
  l = sum_quarters(l);
  f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int u = 0; u < NKQ; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool there = 16 * u + 4 * g4 + r < nkeys;             // a weight of 0 must not meet the duplicated last key
#pragma unroll
      for (int db = 0; db < 2; ++db) o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(there ? vr[u][r][db] : 0.f, s[u][r], o[db], 0, 0, 0);
    }
  // Eq. 8-9 with the cached pair expressed through (o, m, lse): A_out e^{L_out-M} = o e^{m-M}.
  float me2 = -INFINITY, le = 0.f;
  if (el != -INFINITY) {
    me2 = em * kLog2e;
    le = exp2f((el - em) * kLog2e);
  }
  const float M2 = fmaxf(me2, m);
  const float M2u = (M2 == -INFINITY) ? 0.f : M2;
  const float we = exp2f(me2 - M2u), wi = exp2f(m - M2u);
  const float den = le * we + l * wi;
  const float inv = den > 0.f ? 1.f / den : 0.f;
  if (!row_ok) return;
#pragma unroll
  for (int db = 0; db < 2; ++db) {
    f32x4 num = o[db] * wi;
    if (le > 0.f) {
#pragma unroll
      for (int r = 0; r < 4; ++r) num[r] = fmaf(eo[db][r], we, num[r]);
    }
    *(f32x4*)((float*)p.out + grow * D + 32 * cw + 16 * db + 4 * g4) = num * inv;
  }
  if (p.lse_out != nullptr && g4 == 0 && cw == 0) p.lse_out[grow] = den > 0.f ? (M2 + log2f(den)) * kLn2 : -INFINITY;
}

template <int D>
hipError_t launch_internal_f32_wave(const PassParams& p, hipStream_t s) {
  PassParams q = p;
  const int rowtiles = (p.G * p.Bq + 15) / 16;
  q.div_rowtiles = make_fastdiv((uint32_t)rowtiles);
  const dim3 grid((unsigned)((long long)p.B * p.Hkv * rowtiles * (D / 32)));
  if (p.nkeys <= 32) hipLaunchKernelGGL((internal_f32_wave_kernel<D, 2>), grid, dim3(64), 0, s, q);
  else if (p.nkeys <= 48) hipLaunchKernelGGL((internal_f32_wave_kernel<D, 3>), grid, dim3(64), 0, s, q);
  else hipLaunchKernelGGL((internal_f32_wave_kernel<D, 4>), grid, dim3(64), 0, s, q);
  return hipGetLastError();
}

template <int D, int MODE>
hipError_t launch_f32_few(const PassParams& p, hipStream_t s) {
  PassParams q = p;
  q.div_rowtiles = make_fastdiv((uint32_t)(p.G * p.Bq));
  const long long rows = (long long)p.B * p.Hq * p.Bq;
  hipLaunchKernelGGL((attn_f32_few_kernel<D, MODE>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, q);
  return hipGetLastError();
}

// head_dim 64, 64-row workgroups: tiles each up to which they keep the fp32 products.  Splitting the queries and looking for a NaN cost 3 us a
// round of workgroups, which the tiles have not earned by then (a refresh step, fp32 products and parts: 12 heads of 464 rows, batch 6, 55 keys
// 36.1 and 44.6 us; random calls by tiles a workgroup, parts 1 / 2 / 3 / 4 / 5: 1.18 / 1.11 / 1.08 / 0.98 / 0.92 times.  head_dim 128: 0.98 at one).
// In many rounds it shows longer, as two workgroups of the fp32 products share a CU and hide each other's start and end (external pass, 720
// workgroups, 4 tiles 1.06 times; 1040, 6 1.05, 960, 8 0.98; 2856, 4 1.16, 2340, 6 1.09, 2336, 9 1.03; internal pass, 4 tiles 27.4 and 28.9 us, 5 31.9 and 33.0; 576 workgroups, 6 52.7 and 56.0, 648, 9
// 117 and 122).
inline int few_tiles_f32(long long workgroups, bool internal) {
  if (internal) return workgroups > 512 ? 9 : 5;
  return workgroups > 768 ? 8 : workgroups > 512 ? 4 : 3;
}

template <int D, int MODE, int RB, int WR, int TG = 1, bool PARTS = FCfg<D, RB, WR, TG>::kParts>
hipError_t launch_f32(const PassParams& p, hipStream_t s) {
  using C = FCfg<D, RB, WR, TG>;
  auto kern = attn_f32_kernel<D, MODE, RB, WR, TG, PARTS>;
  static LdsLimit lim;
  hipError_t e = raise_lds_limit(kern, C::LDS, lim, C::LDS);
  if (e != hipSuccess) return e;
  constexpr bool per_head = f32_per_head(MODE);
  const int heads = per_head ? p.Hq : p.Hkv, nrows = per_head ? p.Bq : p.G * p.Bq;
  const int rowtiles = (nrows + C::ROWS - 1) / C::ROWS;
  const int nsplit = p.nsplit + (MODE == kPassRefreshFused ? 1 : 0);
  long long units = (long long)p.B * heads * nsplit;
  if (MODE == kPassDensePaged) units = (units + 7) / 8 * 8;
  if (units * rowtiles >= (1ll << 31)) return hipErrorInvalidValue;
  PassParams q = p;
  if (MODE == kPassDensePaged) q.div_page = make_fastdiv((uint32_t)p.page_size);
  q.div_rowtiles = make_fastdiv((uint32_t)rowtiles);
  q.div_nsplit = make_fastdiv((uint32_t)nsplit);
  q.div_hkv = make_fastdiv((uint32_t)heads);
  hipLaunchKernelGGL(kern, dim3((unsigned)(units * rowtiles)), dim3(C::THREADS), C::LDS, s, q);
  return hipGetLastError();
}

template <int D, int MODE>
hipError_t launch_f32_rows(const PassParams& p, hipStream_t s) {
  if constexpr (MODE == kPassInternal || MODE == kPassDense) {
    if ((MODE == kPassInternal || p.direct) && f32_few_keys((long long)p.B * p.Hq * p.Bq, p.G * p.Bq, p.nkeys))
      return launch_f32_few<D, MODE>(p, s);
  }
  const int nrows = f32_per_head(MODE) ? p.Bq : p.G * p.Bq;
  if constexpr (MODE == kPassInternal) {
    // One wavefront per 16 rows x 32 columns while repeating the scores per column group costs less than a staged tile of 64
    // keys.  Before -> so, us (32 / 8 heads, head_dim 128 unless noted): 32 keys, 256 wavefronts 6.7 -> 4.8, 2048 13.5 -> 10.2
    // (head_dim 64, 2048 10.1 -> 7.0); 48 keys, 384 6.7 -> 6.0, 640 level (head_dim 64, 1536 9.2 -> 7.2); 64 keys, 256 6.5 -> 5.8,
    // 512 6.5 -> 7.0 (head_dim 64, 512 5.2 -> 5.3).  Not in place: several workgroups read a row's queries.
    const long long waves = (long long)p.B * p.Hkv * ((nrows + 15) / 16) * (D / 32);
    const long long most = p.nkeys <= 32 ? 2048 : p.nkeys <= 48 ? (D == 64 ? 1536 : 512) : 256;
    if (p.nkeys > kFewKeysF32 && p.nkeys <= 64 && waves <= most && !internal_in_place(p, D, 4)) return launch_internal_f32_wave<D>(p, s);
  }
  int tile = f32_row_tile(nrows);
  if (MODE == kPassInternal) {
    // the internal pass has no splits to fill the chip with: 16-row workgroups until 64-row ones do (blocks of 32, 64-row
    // workgroups: 16 of them 14.2 us, 7.2 with 16 rows; 128 14.8 and 13.2; 256 15.5 and 23.8; blocks of 1000, 192 of them, 85
    // and 105)
    if ((long long)p.B * p.Hkv * ((nrows + 63) / 64) < 256) tile = 16;
  } else {
    // too few tiles for the splits that would fill the chip: smaller workgroups as long as they are one round (128 rows of 8
    // KV heads, head_dim 128, 32 / 64 / 192 keys: 64-row workgroups 12.9 / 12.7 / 15.5 us, 16-row ones 6.4 / 6.2 / 9.2)
    const long long units = (long long)p.B * (f32_per_head(MODE) ? p.Hq : p.Hkv) * (p.nsplit + (MODE == kPassRefreshFused ? 1 : 0));
    if (units * ((nrows + 15) / 16) <= 256) tile = 16;
    else if (tile > 32 && units * ((nrows + 31) / 32) <= 256) tile = 32;
  }
  if (tile == 16) return launch_f32<D, MODE, 1, 1>(p, s);
  // two accumulator sets at head_dim 128: 64-row workgroups have half the registers a wavefront and spill in the tile loop
  // (32 / 8 heads of 40 rows, 4111 keys, refresh 138 us with 64 rows and 82 with 32)
  constexpr bool fits64 = !(D == 128 && MODE == kPassSparseRefresh);
  if constexpr (fits64) {
    // (sparse reuse: how many tiles a head has is not known here, and it always takes the parts)
    if constexpr (D == 64 && MODE != kPassSparseReuse) {
      const int splits = MODE == kPassInternal ? 1 : p.nsplit;
      const long long workgroups = (long long)p.B * (f32_per_head(MODE) ? p.Hq : p.Hkv) * splits * ((nrows + 63) / 64);
      if (tile > 32 && (p.nkeys + kKeyTile - 1) / kKeyTile <= few_tiles_f32(workgroups, MODE == kPassInternal) * splits) return launch_f32<D, MODE, 2, 2, 1, false>(p, s);
    }
    if (tile > 32) return launch_f32<D, MODE, 2, 2>(p, s);
  }
  return launch_f32<D, MODE, 2, 1>(p, s);
}

template <int D>
hipError_t launch_d(const PassParams& p, PassMode mode, hipStream_t s) {
  switch (mode) {
    case kPassDense: return launch_f32_rows<D, kPassDense>(p, s);
    case kPassInternal: return launch_f32_rows<D, kPassInternal>(p, s);
    case kPassSparseRefresh: return launch_f32_rows<D, kPassSparseRefresh>(p, s);
    case kPassSparseReuse: return launch_f32_rows<D, kPassSparseReuse>(p, s);
    case kPassDenseHeads: return launch_f32_rows<D, kPassDenseHeads>(p, s);
    case kPassDensePaged: return launch_f32_rows<D, kPassDensePaged>(p, s);
    case kPassRefreshFused: return launch_f32_rows<D, kPassRefreshFused>(p, s);
    case kPassRefreshOne: return launch_f32<D, kPassRefreshOne, 1, 1, D == 64 ? 2 : 1>(p, s);      // (the caller has checked f32_refresh_one)
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_block_mass_f32(const MassParams& p, int D, hipStream_t s) {
  const dim3 grid((p.Bq + kRowsPerWgF32 - 1) / kRowsPerWgF32, p.B * p.Hq, p.nsplit);
  if (D == 64) hipLaunchKernelGGL(block_mass_f32_kernel<64>, grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL(block_mass_f32_kernel<128>, grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_attn_f32(const PassParams& p, int D, PassMode mode, hipStream_t s) {
  if (D == 64) return launch_d<64>(p, mode, s);
  return launch_d<128>(p, mode, s);
}

}  // namespace fb
