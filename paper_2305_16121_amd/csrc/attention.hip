// Flash-style attention for the local heads of one TMP rank (gfx950, bf16 MFMA, fp32 softmax).
//
// Work decomposition.  A workgroup owns one or two groups of 32 rows of one (sequence, head): queries (forward, dQ) or keys
// (dK/dV); its four waves are (row group) x (part of the reduction range).  The workgroup stages the tiles of the reduction
// range -- keys a query block sees, or queries that see a key block -- for all its waves, and the partial results of a
// row group meet once, through LDS, at the end.  Calls with few blocks keep a form in which each wave
// stages tiles of its own (see below).
//
// Forward and dQ compute the TRANSPOSED score tile S^T = K*Q^T with v_mfma_f32_32x32x16_bf16, so that a lane owns
// one query (accumulator column l%32) and 16 keys of the tile: the online softmax is lane-local except for one
// exchange between the two lane halves, and the exponentials are already in B-operand position for
// O^T = V^T * P^T (the k index of that product is permuted the same way for both operands: rows 4*(l/32)+{0..3}
// and +8 of each 16-key step; the V^T operand comes from the LDS transpose read ds_read_b64_tr_b16).
// dK/dV keeps S = Q*K^T un-transposed so a lane owns one key and P^T / dS^T are in A-operand position.
// No atomics: dQ and dK/dV are separate passes, results are deterministic.
#include <type_traits>

#include "common.h"

namespace oases {

namespace {

constexpr int NT = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct AttnArgs {
  const uint16_t* qkv;   // [batch*seq, ld]
  const uint16_t* out;   // [batch*seq, hp]
  const uint16_t* dout;  // [batch*seq, hp]
  uint16_t* out_w;       // forward output
  uint16_t* dqkv;        // [batch*seq, ld]
  float* lse;            // [batch, heads, seq]
  float* delta;          // [batch, heads, seq]
  int seq, heads, ld, hp;
  int seq0;    // first sequence of the row range
  int first;   // first position (within each sequence) of the row range
  int pos0;    // the same rounded down to a whole block, where the blocks start: a row is then in the same block, and its sums run over the same tiles
               // in the same order, whatever range it is called with (and a 4 x 4 block of the dropout mask belongs to one quad of lanes)
  int npos;    // positions per sequence from pos0 to the end of the row range
  int blocks;  // 32-row blocks per sequence
  int nseq;    // sequences in the row range
  float scale, scale_log2;
  // dropout on the probabilities (DROP kernels): Philox key, counter word 3 (layer | 2^31), byte threshold, 1/(1 - T/256),
  // global index of local head 0 and heads of the unsharded layer
  uint32_t dk0, dk1, dc3, dthresh;
  float dscale;
  int head0, heads_total;
};

// Dropout mask of the probabilities: the 4 x 4 block (q div 4, k div 4) of (sequence b, global head) draws one
// Philox4x32-10 output with counter (k div 4, q div 4, b * heads_total + head, layer | 2^31); element (q, k) keeps its
// value iff byte (k mod 4) of word (q mod 4) is >= the threshold.
__device__ __forceinline__ Philox4 attn_drop_block(const AttnArgs& a, uint32_t k4, uint32_t q4, uint32_t bh) {
  return philox4x32_10(k4, q4, bh, a.dc3, a.dk0, a.dk1);
}

// A 32-row tile of a [*, D] bf16 slice in LDS, rows padded so that BOTH access patterns are conflict-free on 64
// banks: ds_read_b128 of 16 consecutive rows at one column (row stride = 4 resp. 12 banks mod 64) and the
// transpose read of 4 consecutive rows x 32 bytes.
template <int D>
struct AT {
  static constexpr int pad = D == 128 ? 48 : 16;
  static constexpr int row = D * 2 + pad;
  static constexpr int bytes = 32 * row;
  static constexpr int cpr = D / 8;            // 16-byte chunks per row
  static constexpr int per_lane = 32 * cpr / 64;  // chunks per lane when one wave moves the tile
};

// Workgroup id -> ((sequence, head) pair, 32-row block).  Workgroup ids go round-robin over the 8 XCDs, so pair p
// of every group of 8 pairs is given the ids congruent to p mod 8: all blocks of one (sequence, head) then run on
// one XCD and its K/V (about 1 MB) stays in that XCD's L2 instead of every L2 streaming every head.
__device__ __forceinline__ void decode_block(int wg, int pairs, int blocks, int& pair, int& blk) {
  const int per_group = 8 * blocks;
  const int gi = wg / per_group, w = wg - gi * per_group;
  const int pg = min(8, pairs - 8 * gi);
  pair = 8 * gi + w % pg;
  blk = w / pg;
}

// one wave: rows [r0, r0+32) of a [*, D] slice (row stride ld elements) -> registers; rows outside [rmin, rmax) read
// as ZERO: such rows may hold anything (rows of a sub-batch that has not been computed yet), and a masked
// probability of 0 would still turn an inf/NaN there into NaN inside the MFMA.  Tiles inside the range take the
// path without clamps and selects (uniform branch).
template <int D>
__device__ __forceinline__ void wave_load(u32x4* regs, const uint16_t* __restrict__ base, int ld, int r0, int rmin, int rmax, int lane) {
  constexpr int cpr = AT<D>::cpr, rows_per_pass = 64 / cpr;
  if (r0 >= rmin && r0 + 32 <= rmax) {
    const char* sb = reinterpret_cast<const char*>(base) + (size_t)r0 * ld * 2;
    const uint32_t voff = (uint32_t)(((lane / cpr) * ld + (lane % cpr) * 8) * 2);
#pragma unroll
    for (int i = 0; i < AT<D>::per_lane; i++)
      regs[i] = *reinterpret_cast<const u32x4*>(sb + (size_t)i * rows_per_pass * ld * 2 + voff);
  } else {
#pragma unroll
    for (int i = 0; i < AT<D>::per_lane; i++) {
      int c = lane + 64 * i;
      int row = c / cpr, cc = c % cpr;
      int r = max(min(r0 + row, rmax - 1), rmin);
      u32x4 v = *reinterpret_cast<const u32x4*>(base + (size_t)r * ld + cc * 8);
      regs[i] = (r0 + row >= rmin && r0 + row < rmax) ? v : u32x4{0u, 0u, 0u, 0u};
    }
  }
}
template <int D>
__device__ __forceinline__ void wave_store(const u32x4* regs, char* lds, int lane) {
#pragma unroll
  for (int i = 0; i < AT<D>::per_lane; i++) {
    int c = lane + 64 * i;
    int row = c / AT<D>::cpr, cc = c % AT<D>::cpr;
    *reinterpret_cast<u32x4*>(lds + row * AT<D>::row + (cc << 4)) = regs[i];
  }
}
// operand fragment (32 tile rows x 16 contraction), contraction along D (16-wide step ks)
template <int D>
__device__ __forceinline__ bf16x8 kc_frag(const char* lds, int ks, int lane) {
  return *reinterpret_cast<const bf16x8*>(lds + (lane & 31) * AT<D>::row + ((ks * 2 + (lane >> 5)) << 4));
}
// operand fragment whose contraction index is the tile ROW (16-row step j) and whose free index is the column
// c0 + l%32; element e of lane half g is row 16j + 8*(e/4) + 4g + e%4 (matches an accumulator column)
template <int D>
__device__ __forceinline__ bf16x8 mc_frag(const char* lds, int j, int c0, int lane) {
  constexpr int rowb = AT<D>::row;
  int krow = j * 16 + 4 * (lane >> 5) + ((lane & 15) >> 2);
  int col = c0 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const char* p = lds + krow * rowb + col * 2;
  short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(p));
  short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(p + 8 * rowb));
  typedef short short8v __attribute__((ext_vector_type(8)));
  short8v v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int o) {
  u32x4 r = {pack_bf16x2(v[o], v[o + 1]), pack_bf16x2(v[o + 2], v[o + 3]), pack_bf16x2(v[o + 4], v[o + 5]),
             pack_bf16x2(v[o + 6], v[o + 7])};
  return __builtin_bit_cast(bf16x8, r);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; i++) z[i] = 0.f;
  return z;
}
// What stands before it is issued before what stands behind it.
#define OASES_ISSUED() __builtin_amdgcn_sched_barrier(0)
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)

// 32 x D bf16 rows of one operand straight from global memory into B/A-operand registers: lane l holds row l%32,
// columns 16 ks + 8 (l/32) .. +7
template <int D>
__device__ __forceinline__ void load_row_frags(bf16x8* f, const uint16_t* __restrict__ rowp, bool ok, int g) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (ok) v = *reinterpret_cast<const u32x4*>(rowp + ks * 16 + 8 * g);
    f[ks] = __builtin_bit_cast(bf16x8, v);
  }
}

// the inverse rotation of columns d and d + D/2
__device__ __forceinline__ void turn_back(float& x1, float& x2, const float2& t) {
  const float cs = t.x, sn = -t.y, a = x1, b = x2;
  x1 = a * cs - b * sn;
  x2 = b * cs + a * sn;
}

// sum of the four waves' partial accumulators through LDS: wave w ends up with elements [w*E/4, (w+1)*E/4) of the flattened (tile, element)
// index, or (HALVES) with [w*E/8, (w+1)*E/8) of each half of it -- columns d and d + D/2, which a rotation takes together -- summed over
// the four partials with the weights sc[0..3]
template <int E, bool HALVES>
__device__ __forceinline__ int part_element(int wave, int k) {
  return HALVES ? wave * (E / 8) + k % (E / 8) + (k >= E / 8 ? E / 2 : 0) : wave * (E / 4) + k;
}
template <int E, bool HALVES>
__device__ __forceinline__ void combine4(const f32x16* acc, float* lds_part, int wave, int lane, const float* sc, float* out) {
  __syncthreads();  // every wave is done with its tiles: the staging area is free
#pragma unroll
  for (int e = 0; e < E; e++) lds_part[(wave * E + e) * 64 + lane] = acc[e / 16][e % 16];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < E / 4; k++) {
    const int e = part_element<E, HALVES>(wave, k);
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 4; w++) v += lds_part[(w * E + e) * 64 + lane] * sc[w];
    out[k] = v;
  }
}

// ---- tiles shared by the workgroup ----------------------------------------------------------------
// A tile of R rows x D bf16 in LDS without padding: 16-byte chunk c of row r sits at slot c ^ f(r).  f is a bijection over
// the rows that fill the 64 banks once (16 rows of 256 bytes, 8 pairs of rows of 128 bytes), so 16 consecutive rows read at one
// chunk (ds_read_b128) fall on 16 places; its two high bits come from the low bits of the row, so the 4 rows x 4 chunks of a
// transpose read do too.
template <int D>
__device__ __forceinline__ int tile_f(int r) {
  if (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  const int u = (r >> 1) & 7;
  return ((u & 1) << 2) | (u >> 1);
}
template <int D>
__device__ __forceinline__ int tile_chunk(int r, int c) { return r * (2 * D) + ((c ^ tile_f<D>(r)) << 4); }

// all 256 threads: R rows from row r0 of a [*, D] slice (row stride ld elements) -> registers; rows outside [rmin, rmax) read as zero (their
// probabilities are masked to 0, but 0 times what memory holds there may be NaN)
template <int D, int R>
struct SharedTile {
  static constexpr int bytes = R * 2 * D;
  static constexpr int cpr = D / 8, per = R * cpr / NT, rows_per_pass = NT / cpr;
  u32x4 v[per];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ base, int ld, int r0, int rmin, int rmax, int tid) {
    const int row = tid / cpr, cc = tid % cpr;
    if (r0 >= rmin && r0 + R <= rmax) {
      const char* sb = reinterpret_cast<const char*>(base) + (size_t)r0 * ld * 2;
      const uint32_t voff = (uint32_t)((row * ld + cc * 8) * 2);
#pragma unroll
      for (int i = 0; i < per; i++) v[i] = *reinterpret_cast<const u32x4*>(sb + (size_t)i * rows_per_pass * ld * 2 + voff);
    } else {
#pragma unroll
      for (int i = 0; i < per; i++) {
        const int r = r0 + row + i * rows_per_pass;
        const u32x4 x = *reinterpret_cast<const u32x4*>(base + (size_t)max(min(r, rmax - 1), rmin) * ld + cc * 8);
        v[i] = r >= rmin && r < rmax ? x : u32x4{0u, 0u, 0u, 0u};
      }
    }
  }
  __device__ __forceinline__ void store(char* lds, int tid) const {
    const int row = tid / cpr, cc = tid % cpr;
#pragma unroll
    for (int i = 0; i < per; i++) *reinterpret_cast<u32x4*>(lds + tile_chunk<D>(row + i * rows_per_pass, cc)) = v[i];
  }
};
// operand fragments of 32 tile rows from row r0 (a multiple of 32), as kc_frag and mc_frag above
template <int D>
__device__ __forceinline__ bf16x8 tile_kc(const char* lds, int r0, int ks, int lane) {
  return *reinterpret_cast<const bf16x8*>(lds + r0 * (2 * D) + tile_chunk<D>(lane & 31, ks * 2 + (lane >> 5)));
}
template <int D>
__device__ __forceinline__ bf16x8 tile_mc(const char* lds, int r0, int j, int dt, int lane) {
  const int kr = 4 * (lane >> 5) + ((lane & 15) >> 2), c = 4 * dt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  const char* p = lds + (r0 + 16 * j) * (2 * D) + 8 * (lane & 1);
  short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(p + tile_chunk<D>(kr, c)));
  short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(p + tile_chunk<D>(kr + 8, c)));
  typedef short short8v __attribute__((ext_vector_type(8)));
  short8v v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}
// the same from one address for all fragments of a tile.  off: tile_mc_offset of the lane plus the tile's offset in lds, a multiple of its row (2 D
// bytes): the columns of a fragment (bits 6, 7) and the swizzle eight rows on (bit 5) are bits of it
template <int D>
__device__ __forceinline__ int tile_mc_offset(int lane) {
  return tile_chunk<D>(4 * (lane >> 5) + ((lane & 15) >> 2), 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) + 8 * (lane & 1);
}
template <int D>
__device__ __forceinline__ bf16x8 tile_mc_at(const char* lds, uint32_t off, int j, int dt) {
  const uint32_t o = off ^ (dt << 6);
  short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(lds + o + 16 * j * 2 * D));
  short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(lds + (o ^ 32) + (16 * j + 8) * 2 * D));
  typedef short short8v __attribute__((ext_vector_type(8)));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// barrier behind LDS accesses only: global loads into registers stay in flight (__syncthreads would wait for them)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Workgroup id -> ((sequence, head) pair, block), as decode_block, with the long blocks first in even groups of eight pairs and
// last in odd ones: of two workgroups that share a CU from the start one is long and one short.
__device__ __forceinline__ void decode_block_serpentine(int wg, int pairs, int blocks, int& pair, int& blk) {
  const int per_group = 8 * blocks, gi = wg / per_group;
  decode_block(wg, pairs, blocks, pair, blk);
  if (gi & 1) blk = blocks - 1 - blk;
}
// The same where a CU holds four workgroups.  An XCD deals its workgroups to 32 CUs layer by layer; with 16, 8, 4.. blocks an even number of
// groups fills a layer, so every layer would be dealt alike and a CU would get four long workgroups: odd layers are turned round.  us, causal,
// turned or not (D = 64): 8x1024x8 28.2 -> 21.3, 8x512x16 17.7 -> 14.2, 16x512x16 27.3 -> 27.6, 8x960x8 (15 blocks: not turned) 23.7.
__device__ __forceinline__ void decode_block_layers(int wg, int pairs, int blocks, int& pair, int& blk) {
  decode_block_serpentine(wg, pairs, blocks, pair, blk);
  if (16 % blocks == 0 && ((wg >> 8) & 1)) blk = blocks - 1 - blk;
}

// A value of the wave's lower half (lanes 0..31) and of its upper half, in every lane l of either: those of lanes l % 32 and
// l % 32 + 32.  (The two operands are made distinct: given one value twice, the compiler takes both results for the same.)
__device__ __forceinline__ void wave_halves(float v, float& lo, float& hi) {
  uint32_t u = __builtin_bit_cast(uint32_t, v), w = u;
  asm volatile("" : "+v"(w));
  const auto r = __builtin_amdgcn_permlane32_swap(u, w, false, false);
  lo = __builtin_bit_cast(float, (uint32_t)r[0]);
  hi = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float half_max(float v) { float a, b; wave_halves(v, a, b); return fmaxf(a, b); }
__device__ __forceinline__ float half_sum(float v) { float a, b; wave_halves(v, a, b); return a + b; }
// at the head of a rarely taken branch: keeps the compiler from running its body every time and selecting
#define OASES_RARE() asm volatile("")

// value of lane i of every four lanes
template <int I>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, I * 0x55, 0xf, 0xf, true); }

// Dropout words of four 4-key groups (keys k0 + 8 i, i = 0..3) for this lane's query q.  The four lanes of a quad hold the four
// queries of one 4 x 4 block row, so each computes the block of one group and they trade words (a Philox call is some 40
// multiplications at a quarter of the rate; one instead of four).
__device__ __forceinline__ void drop_words_of_query(const AttnArgs& a, uint32_t (&w)[4], int k0, int q, uint32_t bh, int lane) {
  const int j = lane & 3;
  const Philox4 m = attn_drop_block(a, (uint32_t)(k0 + 8 * j) >> 2, (uint32_t)q >> 2, bh);
#define OASES_QUAD(i)                                                                                              \
  {                                                                                                                \
    const uint32_t x0 = quad_lane<i>(m.v[0]), x1 = quad_lane<i>(m.v[1]), x2 = quad_lane<i>(m.v[2]), x3 = quad_lane<i>(m.v[3]); \
    w[i] = j == 0 ? x0 : j == 1 ? x1 : j == 2 ? x2 : x3;                                                           \
  }
  OASES_QUAD(0) OASES_QUAD(1) OASES_QUAD(2) OASES_QUAD(3)
#undef OASES_QUAD
}

// =================================================================================================
// forward: QG groups of 32 queries x KG key parts, one wave each (QG * KG = 4).  What bounds it: the chain of a tile (LDS reads,
// eight dependent MFMAs, the softmax, eight more) with two waves on a SIMD to cover for each other, and LDS bandwidth, 96 KB per
// 64 x 64 scores at D = 128.  Measured, tiles private to a wave -> this, us: 8x1024x8x64 (batch x seq x heads x columns, causal)
// 35.3 -> 31.5, 4x2048x4x128 45.9 -> 40.5, 2x2048x4x128 32.2 -> 30.4, 4x1024x12x128 not causal 65.6 -> 47.0.  The workgroup stages 32 KG keys of K and V at
// a time for all its waves, two stages: the next tile goes from registers to LDS while this one is multiplied, and the tile
// behind it is on its way from memory.  A wave keeps (m, l, O) of its queries over its part of the keys; the KG partial
// results of a query group meet once, through LDS, at the end.
// =================================================================================================
template <int D, int QG, int KG>
struct FwdLds {
  static constexpr int E = D / 2;  // accumulator elements of a lane
  static constexpr int NS = D == 128 && KG == 4 ? 1 : 2;  // stages; 128 keys of 128 columns take 64 KB: one, so that two workgroups fit a CU
  static constexpr int kTile = SharedTile<D, 32 * KG>::bytes, kStages = 2 * NS * kTile, kPart = 4 * E * 64 * 4;
  static constexpr int bytes = (kStages > kPart ? kStages : kPart) + 1024;  // + m[4][32], l[4][32]
};
// FOUR: 64 columns, two query groups and no dropout fit four workgroups on a CU (33 KB of LDS each) as long as a wave has 128 registers.
template <int D, int QG, bool DROP>
constexpr bool kFwdFour = D == 64 && QG == 2 && !DROP;
template <int D, int QG, int KG, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(NT, (kFwdFour<D, QG, DROP> ? 4 : 2)) void attn_fwd_kernel(AttnArgs a) {
  constexpr int KS = D / 16, DT = D / 32, E = DT * 16, BK = 32 * KG;
  constexpr bool FOUR = kFwdFour<D, QG, DROP>;
  using L = FwdLds<D, QG, KG>;
  __shared__ __attribute__((aligned(16))) char lds[L::bytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  const int qg = wave % QG, kg = wave / QG;
  int pair, blk;
  if constexpr (FOUR && CAUSAL) decode_block_layers(blockIdx.x, a.nseq * a.heads, a.blocks, pair, blk);
  else decode_block_serpentine(blockIdx.x, a.nseq * a.heads, a.blocks, pair, blk);
  const int sq = pair / a.heads, head = pair % a.heads, qb = a.blocks - 1 - blk;  // long rows first
  const int seq_idx = a.seq0 + sq;
  const int wg_end = min(a.pos0 + a.npos, a.pos0 + (qb + 1) * 32 * QG);   // end of the workgroup's queries
  const int q_begin = a.pos0 + (qb * QG + qg) * 32;
  const int q_end = min(wg_end, q_begin + 32);
  const size_t rowbase = (size_t)seq_idx * a.seq;
  const uint16_t* Qp = a.qkv + rowbase * a.ld + head * D;
  const uint16_t* Kp = Qp + a.hp;
  const uint16_t* Vp = Qp + 2 * a.hp;
  const int qpos = q_begin + (lane & 31);
  const bool qok = qpos < q_end && qpos >= a.first;

  const int kv_end = CAUSAL ? wg_end : a.seq;
  const int nt = (kv_end + BK - 1) / BK;
  SharedTile<D, BK> rk, rv;
  rk.load(Kp, a.ld, 0, 0, kv_end, tid);
  rv.load(Vp, a.ld, 0, 0, kv_end, tid);
  bf16x8 qf[KS];
  load_row_frags<D>(qf, Qp + (size_t)qpos * a.ld, qok, g);
  f32x16 o[DT];
#pragma unroll
  for (int i = 0; i < DT; i++) o[i] = zero16();
  float m = -1e30f, l = 0.f;
  rk.store(lds, tid);
  rv.store(lds + L::kTile, tid);
  if (nt > 1) {
    rk.load(Kp, a.ld, BK, 0, kv_end, tid);
    rv.load(Vp, a.ld, BK, 0, kv_end, tid);
  }
  lds_barrier();
  for (int t = 0; t < nt; t++) {
    const char* lk = lds + (L::NS == 2 ? (t & 1) * 2 * L::kTile : 0);
    const char* lv = lk + L::kTile;
    auto park_next = [&]() {  // tile t + 1, into a stage that every wave has read for the last time before the last barrier
      if (t + 1 >= nt) return;
      char* nk = lds + (L::NS == 2 ? ((t & 1) ^ 1) * 2 * L::kTile : 0);
      rk.store(nk, tid);
      rv.store(nk + L::kTile, tid);
      if (t + 2 < nt) {
        rk.load(Kp, a.ld, (t + 2) * BK, 0, kv_end, tid);
        rv.load(Vp, a.ld, (t + 2) * BK, 0, kv_end, tid);
      }
    };
    if constexpr (L::NS == 2) park_next();
    const int kv0 = t * BK + 32 * kg;
    if (kv0 < a.seq && !(CAUSAL && kv0 >= q_end)) {  // uniform over the wave: some key is visible to some query
      // The fragments of K are requested together, and those of V ahead of the softmax that covers their latency; left to itself the compiler
      // requests one or two at a time and every product waits for one.  us: 4x2048x4x128 43.4 -> 42.2, not causal 58 -> 54.  FOUR: eight addresses
      // would take the registers past 128, and with them the fourth workgroup of a CU (8x1896x4x64 36.4 -> 42.2 us); the fragments of an operand
      // lie where two or three bits of one offset differ, which is formed here and again for every tile: 34.1 us.
      // Not V ahead with dropout, 128 columns and one query group, where the registers spill (4x1032x3 24.2 -> 25.5 us).
      constexpr bool V_AHEAD = !(D == 128 && QG == 1 && DROP);
      f32x16 s = zero16();
      bf16x8 kf[KS], vf[2][DT];
      uint32_t ko = (uint32_t)(lk - lds) + 32 * kg * 2 * D + tile_chunk<D>(lane & 31, g);
      uint32_t vo = (uint32_t)(lv - lds) + 32 * kg * 2 * D + tile_mc_offset<D>(lane);
      if constexpr (FOUR) asm volatile("" : "+v"(ko), "+v"(vo));
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        if constexpr (FOUR) kf[ks] = *reinterpret_cast<const bf16x8*>(lds + (ko ^ (ks << 5)));
        else kf[ks] = tile_kc<D>(lk, 32 * kg, ks, lane);
      }
      OASES_ISSUED();
#pragma unroll
      for (int ks = 0; ks < KS; ks++) s = MFMA(kf[ks], qf[ks], s);
      if constexpr (V_AHEAD) {
        OASES_ISSUED();
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
          for (int dt = 0; dt < DT; dt++) {
            if constexpr (FOUR) vf[j][dt] = tile_mc_at<D>(lds, vo, j, dt);
            else vf[j][dt] = tile_mc<D>(lv, 32 * kg, j, dt, lane);
          }
        OASES_ISSUED();
      }
      if ((kv0 + 32 > a.seq) || (CAUSAL && kv0 + 31 > q_begin)) {
        OASES_RARE();
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const int kvpos = kv0 + 8 * (i >> 2) + 4 * g + (i & 3);
          if (kvpos >= a.seq || (CAUSAL && kvpos > qpos)) s[i] = -INFINITY;
        }
      }
      float mloc = s[0];
#pragma unroll
      for (int i = 1; i < 16; i++) mloc = fmaxf(mloc, s[i]);
      mloc = half_max(mloc);
      // The reference m of the exponentials is the largest score so far, exactly: the largest probability of a row is then 1, which bf16
      // holds without error, and those next to it lie at the upper end of a binade, where its relative error is least.  A
      // reference that lags behind the maximum (by up to 2^6, so that fewer tiles rescale O) costs 3 to 14 % of the output's accuracy
      // and gives 0.3 to 4 us: error against 64 bits, 4x2048x4x128 causal 2.07e-3 -> 1.99e-3 and 36.5 -> 40.5 us, with scores four
      // times as wide 1.94e-3 -> 1.70e-3; 8x512x4x64 8.8 -> 9.1 us.  Each query moves by its own scores alone (alpha = 1 for the others of the wave).  m
      // starts at a finite value: a part may begin on tiles that are masked for some of its queries, and exp2 must not see inf - inf.
      if (__any(mloc > m)) {
        OASES_RARE();
        const float mnew = fmaxf(m, mloc);
        const float alpha = __builtin_amdgcn_exp2f((m - mnew) * a.scale_log2);
        m = mnew;
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; dt++)
#pragma unroll
          for (int i = 0; i < 16; i++) o[dt][i] *= alpha;
      }
      const float nm = -m * a.scale_log2;
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.scale_log2, nm));
        s[i] = p;
        l += p;
      }
      if (DROP) {  // the row sum keeps every probability; what goes on to V is dropped and rescaled
        uint32_t w[4];
        drop_words_of_query(a, w, kv0 + 4 * g, qpos, (uint32_t)(seq_idx * a.heads_total + a.head0 + head), lane);
#pragma unroll
        for (int grp = 0; grp < 4; grp++)
#pragma unroll
          for (int e = 0; e < 4; e++) s[4 * grp + e] = ((w[grp] >> (8 * e)) & 0xffu) >= a.dthresh ? s[4 * grp + e] * a.dscale : 0.f;
      }
#pragma unroll
      for (int j = 0; j < 2; j++) {
        bf16x8 pb = pack8(s, 8 * j);
#pragma unroll
        for (int dt = 0; dt < DT; dt++) o[dt] = MFMA(V_AHEAD ? vf[j][dt] : tile_mc<D>(lv, 32 * kg, j, dt, lane), pb, o[dt]);
      }
    }
    lds_barrier();
    if constexpr (L::NS == 1) {
      park_next();
      lds_barrier();
    }
  }
  l = half_sum(l);

  // merge the KG partial (m, l, O) of a query group: weights 2^(m_k - m); wave (qg, kg) finishes elements [kg E/KG, (kg+1) E/KG)
  static_assert(KG == 2 || KG == 4, "one or two row groups");
  float* part = reinterpret_cast<float*>(lds);
  float* stat = reinterpret_cast<float*>(lds + L::bytes - 1024);
  if (g == 0) { stat[wave * 32 + lane] = m; stat[128 + wave * 32 + lane] = l; }
#pragma unroll
  for (int e = 0; e < E; e++)
    if (e / (E / KG) != kg) part[(wave * E + e) * 64 + lane] = o[e / 16][e % 16];
  lds_barrier();
  float sc[KG], mt = -INFINITY, lt = 0.f;
#pragma unroll
  for (int k = 0; k < KG; k++) mt = fmaxf(mt, stat[(k * QG + qg) * 32 + (lane & 31)]);
#pragma unroll
  for (int k = 0; k < KG; k++) {
    sc[k] = __builtin_amdgcn_exp2f((stat[(k * QG + qg) * 32 + (lane & 31)] - mt) * a.scale_log2);
    lt += stat[128 + (k * QG + qg) * 32 + (lane & 31)] * sc[k];
  }
  auto finish = [&](auto kg_c) {
    constexpr int MY = decltype(kg_c)::value;
    const float inv = 1.0f / lt;
    uint16_t* op = a.out_w + (rowbase + qpos) * a.hp + head * D;
#pragma unroll
    for (int k = 0; k < E / KG; k += 4) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const int e = MY * (E / KG) + k + u;
        v[u] = 0.f;
#pragma unroll
        for (int w = 0; w < KG; w++) v[u] += (w == MY ? o[e / 16][e % 16] : part[((w * QG + qg) * E + e) * 64 + lane]) * sc[w];
      }
      const int e = MY * (E / KG) + k, d = (e / 16) * 32 + 8 * ((e % 16) >> 2) + 4 * g;
      if (qok) *reinterpret_cast<u32x2*>(op + d) = u32x2{pack_bf16x2(v[0] * inv, v[1] * inv), pack_bf16x2(v[2] * inv, v[3] * inv)};
    }
  };
  if constexpr (KG == 2) { if (kg == 0) finish(std::integral_constant<int, 0>{}); else finish(std::integral_constant<int, 1>{}); }
  if constexpr (KG == 4) {
    if (kg == 0) finish(std::integral_constant<int, 0>{});
    else if (kg == 1) finish(std::integral_constant<int, 1>{});
    else if (kg == 2) finish(std::integral_constant<int, 2>{});
    else finish(std::integral_constant<int, 3>{});
  }
  if (qok && kg == 0 && g == 0) a.lse[((size_t)seq_idx * a.heads + head) * a.seq + qpos] = (mt * a.scale_log2 + __builtin_amdgcn_logf(lt)) * kLn2;
}

// =================================================================================================
// backward: delta = rowsum(dO * O)
// =================================================================================================
template <int D>
__global__ __launch_bounds__(NT) void attn_delta_kernel(AttnArgs a, int first_row, int n_rows) {
  constexpr int LPR = D / 8;  // lanes per (row, head)
  const int gid = blockIdx.x * NT + threadIdx.x;
  const int pair = gid / LPR, c = gid % LPR;
  const int r = pair / a.heads, head = pair % a.heads;
  float s = 0.f;
  const bool ok = r < n_rows;
  const size_t row = (size_t)first_row + r;
  if (ok) {
    u32x4 x = *reinterpret_cast<const u32x4*>(a.out + row * a.hp + head * D + c * 8);
    u32x4 y = *reinterpret_cast<const u32x4*>(a.dout + row * a.hp + head * D + c * 8);
#pragma unroll
    for (int j = 0; j < 4; j++) {
      s += bf16_bits_to_f32(x[j] & 0xffffu) * bf16_bits_to_f32(y[j] & 0xffffu);
      s += bf16_bits_to_f32(x[j] >> 16) * bf16_bits_to_f32(y[j] >> 16);
    }
  }
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (ok && c == 0) {
    int b = (int)(row / a.seq), pos = (int)(row % a.seq);
    a.delta[((size_t)b * a.heads + head) * a.seq + pos] = s;
  }
}

// =================================================================================================
// backward: dQ.  QG groups of 32 queries x KG key parts, tiles and waves as in the forward kernel (measured, wave-private tiles
// -> this, us: 4x2048x4x128 69 -> 49, 8x1024x8x64 42.8 -> 33.5).  OWN_DELTA: the workgroup
// forms delta of its queries itself and leaves it for the dK/dV kernel behind it; otherwise it is there already.
// =================================================================================================
template <int D, int QG, int KG>
struct BwdLds {
  static constexpr int E = D / 2, kTile = SharedTile<D, 32 * KG>::bytes, kStat = KG * 256;
  static constexpr int kStage = 2 * kTile + kStat;  // two operand tiles and, dK/dV only, lse and delta of the tile's queries
  static constexpr int kPart = 4 * E * 64 * 4;
  static constexpr int bytes = 2 * kStage > kPart ? 2 * kStage : kPart;
};
// the KG partial sums of a group meet through LDS: wave (qg, kg) ends up with elements [kg E/KG, (kg+1) E/KG) of the flattened
// (tile, element) index, handed to emit(first element, four values)
template <int E, int QG, int KG, int MY, typename Emit>
__device__ __forceinline__ void finish_part(const f32x16* acc, const float* part, int qg, int lane, Emit emit) {
#pragma unroll
  for (int k = 0; k < E / KG; k += 4) {
    f32x4 v;
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int e = MY * (E / KG) + k + u;
      v[u] = 0.f;
#pragma unroll
      for (int w = 0; w < KG; w++) v[u] += w == MY ? acc[e / 16][e % 16] : part[((w * QG + qg) * E + e) * 64 + lane];
    }
    emit(MY * (E / KG) + k, v);
  }
}
template <int E, int QG, int KG, typename Emit>
__device__ __forceinline__ void combine_parts(const f32x16* acc, char* lds, int qg, int kg, int lane, Emit emit) {
  float* part = reinterpret_cast<float*>(lds);
  lds_barrier();  // every wave is done with the tiles, or with the exchange before this one
#pragma unroll
  for (int e = 0; e < E; e++)
    if (e / (E / KG) != kg) part[((kg * QG + qg) * E + e) * 64 + lane] = acc[e / 16][e % 16];
  lds_barrier();
  if constexpr (KG == 2) {
    if (kg == 0) finish_part<E, QG, 2, 0>(acc, part, qg, lane, emit); else finish_part<E, QG, 2, 1>(acc, part, qg, lane, emit);
  } else {
    if (kg == 0) finish_part<E, QG, 4, 0>(acc, part, qg, lane, emit);
    else if (kg == 1) finish_part<E, QG, 4, 1>(acc, part, qg, lane, emit);
    else if (kg == 2) finish_part<E, QG, 4, 2>(acc, part, qg, lane, emit);
    else finish_part<E, QG, 4, 3>(acc, part, qg, lane, emit);
  }
}

template <int D, int QG, int KG, bool CAUSAL, bool DROP, bool OWN_DELTA>
__device__ __forceinline__ void attn_dq_block(const AttnArgs& a, int wg, char* lds) {
  constexpr int KS = D / 16, DT = D / 32, E = DT * 16, BK = 32 * KG;
  using L = BwdLds<D, QG, KG>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  const int qg = wave % QG, kg = wave / QG;
  int pair, blk;
  decode_block_serpentine(wg, a.nseq * a.heads, a.blocks, pair, blk);
  const int sq = pair / a.heads, head = pair % a.heads, qb = a.blocks - 1 - blk;
  const int seq_idx = a.seq0 + sq;
  const int wg_end = min(a.pos0 + a.npos, a.pos0 + (qb + 1) * 32 * QG);
  const int q_begin = a.pos0 + (qb * QG + qg) * 32;
  const int q_end = min(wg_end, q_begin + 32);
  const size_t rowbase = (size_t)seq_idx * a.seq;
  const uint16_t* Qp = a.qkv + rowbase * a.ld + head * D;
  const uint16_t* Kp = Qp + a.hp;
  const uint16_t* Vp = Qp + 2 * a.hp;
  const uint16_t* dOp = a.dout + rowbase * a.hp + head * D;
  const int qpos = q_begin + (lane & 31);
  const bool qok = qpos < q_end && qpos >= a.first;

  const int kv_end = CAUSAL ? wg_end : a.seq;
  const int nt = (kv_end + BK - 1) / BK;
  SharedTile<D, BK> rk, rv;
  rk.load(Kp, a.ld, 0, 0, kv_end, tid);
  rv.load(Vp, a.ld, 0, 0, kv_end, tid);
  bf16x8 qf[KS], dof[KS];
  load_row_frags<D>(qf, Qp + (size_t)qpos * a.ld, qok, g);
  load_row_frags<D>(dof, dOp + (size_t)qpos * a.hp, qok, g);
  const size_t si = ((size_t)seq_idx * a.heads + head) * a.seq + qpos;
  const float lse2 = qok ? a.lse[si] * kLog2e : 0.f;
  float dl = 0.f;
  if constexpr (OWN_DELTA) {
    // eight columns at a time, then a tree over the eights: the order of attn_delta_kernel, so that a row's delta does not depend
    // on which of the two kernels it comes from
    const uint16_t* op = a.out + (rowbase + qpos) * a.hp + head * D;
    float part[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      u32x4 x = {0u, 0u, 0u, 0u};
      if (qok) x = *reinterpret_cast<const u32x4*>(op + ks * 16 + 8 * g);
      const u32x4 y = __builtin_bit_cast(u32x4, dof[ks]);
      part[ks] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        part[ks] += bf16_bits_to_f32(x[j] & 0xffffu) * bf16_bits_to_f32(y[j] & 0xffffu);
        part[ks] += bf16_bits_to_f32(x[j] >> 16) * bf16_bits_to_f32(y[j] >> 16);
      }
    }
#pragma unroll
    for (int o = KS / 2; o > 0; o >>= 1)
#pragma unroll
      for (int ks = 0; ks < o; ks++) part[ks] += part[ks + o];
    dl = half_sum(part[0]);
    if (qok && kg == 0 && g == 0) a.delta[si] = dl;
  } else if (qok) {
    dl = a.delta[si];
  }
  f32x16 acc[DT];
#pragma unroll
  for (int i = 0; i < DT; i++) acc[i] = zero16();
  rk.store(lds, tid);
  rv.store(lds + L::kTile, tid);
  if (nt > 1) {
    rk.load(Kp, a.ld, BK, 0, kv_end, tid);
    rv.load(Vp, a.ld, BK, 0, kv_end, tid);
  }
  lds_barrier();
  for (int t = 0; t < nt; t++) {
    const char* lk = lds + (t & 1) * L::kStage;
    const char* lv = lk + L::kTile;
    if (t + 1 < nt) {
      char* nk = lds + ((t & 1) ^ 1) * L::kStage;
      rk.store(nk, tid);
      rv.store(nk + L::kTile, tid);
      if (t + 2 < nt) {
        rk.load(Kp, a.ld, (t + 2) * BK, 0, kv_end, tid);
        rv.load(Vp, a.ld, (t + 2) * BK, 0, kv_end, tid);
      }
    }
    const int kv0 = t * BK + 32 * kg;
    if (kv0 < a.seq && !(CAUSAL && kv0 >= q_end)) {
      f32x16 s = zero16(), dp = zero16();
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        s = MFMA(tile_kc<D>(lk, 32 * kg, ks, lane), qf[ks], s);
        dp = MFMA(tile_kc<D>(lv, 32 * kg, ks, lane), dof[ks], dp);
      }
      if (DROP) {  // dP = dropout factor * (dO V^T)
        uint32_t w[4];
        drop_words_of_query(a, w, kv0 + 4 * g, qpos, (uint32_t)(seq_idx * a.heads_total + a.head0 + head), lane);
#pragma unroll
        for (int grp = 0; grp < 4; grp++)
#pragma unroll
          for (int e = 0; e < 4; e++) dp[4 * grp + e] = ((w[grp] >> (8 * e)) & 0xffu) >= a.dthresh ? dp[4 * grp + e] * a.dscale : 0.f;
      }
      // only tiles on the diagonal or at the end of the sequence pay for the mask (a wave-uniform branch)
      auto scores = [&](auto mask_c) {
#pragma unroll
        for (int i = 0; i < 16; i++) {
          float ds = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.scale_log2, -lse2)) * (dp[i] - dl);
          if (decltype(mask_c)::value) {
            const int kvpos = kv0 + 8 * (i >> 2) + 4 * g + (i & 3);
            if (kvpos >= a.seq || (CAUSAL && kvpos > qpos)) ds = 0.f;
          }
          s[i] = ds;
        }
      };
      if ((kv0 + 32 > a.seq) || (CAUSAL && kv0 + 31 > q_begin)) scores(std::true_type{}); else scores(std::false_type{});
#pragma unroll
      for (int j = 0; j < 2; j++) {
        bf16x8 db = pack8(s, 8 * j);
#pragma unroll
        for (int dt = 0; dt < DT; dt++) acc[dt] = MFMA(tile_mc<D>(lk, 32 * kg, j, dt, lane), db, acc[dt]);
      }
    }
    lds_barrier();
  }
  uint16_t* op = a.dqkv + (rowbase + qpos) * a.ld + head * D;
  combine_parts<E, QG, KG>(acc, lds, qg, kg, lane, [&](int e, const f32x4& v) {
    const int d = (e / 16) * 32 + 8 * ((e % 16) >> 2) + 4 * g;
    if (qok) *reinterpret_cast<u32x2*>(op + d) = u32x2{pack_bf16x2(v[0] * a.scale, v[1] * a.scale), pack_bf16x2(v[2] * a.scale, v[3] * a.scale)};
  });
}

// =================================================================================================
// backward: dK, dV.  JG groups of 32 keys x RG query parts (D = 64; 8x1024x8x64 78 -> 45 us); the tiles are 32 RG queries of Q and dO with their lse and delta.
// S = Q K^T puts a key on a lane and P, dS into operand position; dV^T = dO^T P and dK^T = Q^T dS then leave four consecutive
// columns of a key on a lane.
// =================================================================================================
template <int D, int JG, int RG, bool CAUSAL, bool DROP>
__device__ __forceinline__ void attn_dkv_block(const AttnArgs& a, int wg, char* lds) {
  constexpr int KS = D / 16, DT = D / 32, E = DT * 16, BQ = 32 * RG;
  using L = BwdLds<D, JG, RG>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  const int jg = wave % JG, rg = wave / JG;
  int pair, kb;
  decode_block_serpentine(wg, a.nseq * a.heads, a.blocks, pair, kb);  // early key blocks are the long ones
  const int sq = pair / a.heads, head = pair % a.heads;
  const int seq_idx = a.seq0 + sq;
  const int wg_begin = a.pos0 + kb * 32 * JG;
  const int k_begin = wg_begin + 32 * jg;
  const int k_end = min(a.pos0 + a.npos, k_begin + 32);
  const size_t rowbase = (size_t)seq_idx * a.seq;
  const uint16_t* Qp = a.qkv + rowbase * a.ld + head * D;
  const uint16_t* Kp = Qp + a.hp;
  const uint16_t* Vp = Qp + 2 * a.hp;
  const uint16_t* dOp = a.dout + rowbase * a.hp + head * D;
  const float* lsep = a.lse + ((size_t)seq_idx * a.heads + head) * a.seq;
  const float* dlp = a.delta + ((size_t)seq_idx * a.heads + head) * a.seq;
  const int kpos = k_begin + (lane & 31);
  const bool kok = kpos < k_end && kpos >= a.first;

  const int q_first = CAUSAL ? wg_begin : 0;  // earlier queries never see a key of this block
  const int qmin = CAUSAL ? a.first : 0;
  const int nt = (a.seq - q_first + BQ - 1) / BQ;
  SharedTile<D, BQ> rq, rdo;
  float rstat = 0.f;
  auto fetch = [&](int t) {
    const int q0 = q_first + t * BQ;
    rq.load(Qp, a.ld, q0, qmin, a.seq, tid);
    rdo.load(dOp, a.hp, q0, qmin, a.seq, tid);
    if (tid < 2 * BQ) {
      const int qp = min(q0 + (tid % BQ), a.seq - 1);
      rstat = tid < BQ ? lsep[qp] * kLog2e : dlp[qp];
    }
  };
  auto park = [&](char* st) {
    rq.store(st, tid);
    rdo.store(st + L::kTile, tid);
    if (tid < 2 * BQ) reinterpret_cast<float*>(st + 2 * L::kTile)[tid] = rstat;
  };
  fetch(0);
  bf16x8 kf[KS], vf[KS];
  load_row_frags<D>(kf, Kp + (size_t)kpos * a.ld, kok, g);
  load_row_frags<D>(vf, Vp + (size_t)kpos * a.ld, kok, g);
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int i = 0; i < DT; i++) { dk[i] = zero16(); dv[i] = zero16(); }
  park(lds);
  if (nt > 1) fetch(1);
  lds_barrier();
  for (int t = 0; t < nt; t++) {
    const char* lq = lds + (t & 1) * L::kStage;
    const char* ldo = lq + L::kTile;
    const float* lstat = reinterpret_cast<const float*>(lq + 2 * L::kTile) + 32 * rg;  // [BQ] lse * log2(e), [BQ] delta
    if (t + 1 < nt) {
      park(lds + ((t & 1) ^ 1) * L::kStage);
      if (t + 2 < nt) fetch(t + 2);
    }
    const int q0 = q_first + t * BQ + 32 * rg;
    if (q0 < a.seq && !(CAUSAL && q0 + 31 < k_begin)) {  // uniform over the wave: some query sees some key
      f32x16 s = zero16(), dp = zero16();
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        s = MFMA(tile_kc<D>(lq, 32 * rg, ks, lane), kf[ks], s);
        dp = MFMA(tile_kc<D>(ldo, 32 * rg, ks, lane), vf[ks], dp);
      }
      Philox4 dw;  // the four lanes of a quad share the keys of a 4 x 4 block: each draws the block of one group of queries
      if (DROP) dw = attn_drop_block(a, (uint32_t)kpos >> 2, (uint32_t)(q0 + 8 * (lane & 3) + 4 * g) >> 2, (uint32_t)(seq_idx * a.heads_total + a.head0 + head));
      // only tiles on the diagonal or at the end of the sequence pay for the mask (a wave-uniform branch)
      auto scores = [&](auto mask_c) {
        auto group = [&](auto i4_c) {
          constexpr int I4 = decltype(i4_c)::value;
          const int ql = 8 * I4 + 4 * g;  // 4 consecutive queries
          const f32x4 l4 = *reinterpret_cast<const f32x4*>(lstat + ql);
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(lstat + BQ + ql);
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const int i = 4 * I4 + e;
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.scale_log2, -l4[e]));
            float dpe = dp[i], pv = p;  // pv: what multiplied V in forward
            if (DROP) {  // this lane's key is byte (kpos mod 4) of the word of query e of the group
              const bool keep = ((quad_lane<I4>(dw.v[e]) >> (8 * (kpos & 3))) & 0xffu) >= a.dthresh;
              dpe = keep ? dpe * a.dscale : 0.f;
              pv = keep ? p * a.dscale : 0.f;
            }
            float ds = p * (dpe - d4[e]);
            if (decltype(mask_c)::value) {
              const int qp = q0 + ql + e;
              if (qp >= a.seq || (CAUSAL && kpos > qp)) { pv = 0.f; ds = 0.f; }   // select, never multiply: the rest may be NaN
            }
            s[i] = pv;
            dp[i] = ds;
          }
        };
        group(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 1>{});
        group(std::integral_constant<int, 2>{});
        group(std::integral_constant<int, 3>{});
      };
      if ((q0 + 32 > a.seq) || (CAUSAL && q0 < k_begin + 31)) scores(std::true_type{}); else scores(std::false_type{});
#pragma unroll
      for (int j = 0; j < 2; j++) {
        bf16x8 pa = pack8(s, 8 * j);
        bf16x8 da = pack8(dp, 8 * j);
#pragma unroll
        for (int dt = 0; dt < DT; dt++) {
          dv[dt] = MFMA(tile_mc<D>(ldo, 32 * rg, j, dt, lane), pa, dv[dt]);
          dk[dt] = MFMA(tile_mc<D>(lq, 32 * rg, j, dt, lane), da, dk[dt]);
        }
      }
    }
    lds_barrier();
  }
  uint16_t* dKp = a.dqkv + (rowbase + kpos) * a.ld + a.hp + head * D;
  uint16_t* dVp = dKp + a.hp;
  combine_parts<E, JG, RG>(dk, lds, jg, rg, lane, [&](int e, const f32x4& v) {
    const int d = (e / 16) * 32 + 8 * ((e % 16) >> 2) + 4 * g;
    if (kok) *reinterpret_cast<u32x2*>(dKp + d) = u32x2{pack_bf16x2(v[0] * a.scale, v[1] * a.scale), pack_bf16x2(v[2] * a.scale, v[3] * a.scale)};
  });
  combine_parts<E, JG, RG>(dv, lds, jg, rg, lane, [&](int e, const f32x4& v) {
    const int d = (e / 16) * 32 + 8 * ((e % 16) >> 2) + 4 * g;
    if (kok) *reinterpret_cast<u32x2*>(dVp + d) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  });
}

// =================================================================================================
// backward: dK, dV with 128 columns.  64 keys x 64 queries at a time: two groups of 32 keys x two halves of a query tile, one wave each,
// which is alone on its SIMD (keys, values and accumulators take 192 registers).  What bounded the wave-private form below on
// large calls is the path from L2 to the registers: 16 KB of Q and dO for 32 x 32 scores, some 1850 of the 4600 cycles of a
// tile just to issue; here the four waves share them (half the bytes a score), and a wave's chain is covered by its own
// next tile: the products S and dP of tile t+1 stand between the exponentials of tile t.  Three stages: tile t+1 is read for these
// products, tile t for dV and dK, and tile t+2 written over tile t-1, whose last reads lie before the barrier that ended
// iteration t-1.  Measured (both backward
// passes by themselves, us; inside a step of h 4096 the first 151 -> 132): 4x2048x4x128 causal 148 -> 122, not causal 222 -> 173, 8x1024x8x128 174 -> 152, 8x512x4x128 42 -> 35.
// =================================================================================================
struct Dkv128Lds {
  static constexpr int kTile = SharedTile<128, 64>::bytes, kStage = 2 * kTile + 512;  // Q, dO, lse * log2(e) [64], delta [64]
  static constexpr int kStages = 3 * kStage, kPart = 4 * 64 * 64 * 4;
  static constexpr int bytes = kStages > kPart ? kStages : kPart;
};
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(NT, 1) void attn_dkv128_kernel(AttnArgs a) {
  constexpr int D = 128, KS = D / 16, DT = D / 32, E = DT * 16;
  using L = Dkv128Lds;
  __shared__ __attribute__((aligned(16))) char lds[L::bytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  const int jg = wave & 1, rg = wave >> 1;
  int pair, kb;
  decode_block(blockIdx.x, a.nseq * a.heads, a.blocks, pair, kb);  // early key blocks are the long ones
  const int sq = pair / a.heads, head = pair % a.heads;
  const int seq_idx = a.seq0 + sq;
  const int wg_begin = a.pos0 + kb * 64;
  const int k_begin = wg_begin + 32 * jg;
  const int k_end = min(a.pos0 + a.npos, k_begin + 32);
  const size_t rowbase = (size_t)seq_idx * a.seq;
  const uint16_t* Qp = a.qkv + rowbase * a.ld + head * D;
  const uint16_t* Kp = Qp + a.hp;
  const uint16_t* Vp = Qp + 2 * a.hp;
  const uint16_t* dOp = a.dout + rowbase * a.hp + head * D;
  const float* lsep = a.lse + ((size_t)seq_idx * a.heads + head) * a.seq;
  const float* dlp = a.delta + ((size_t)seq_idx * a.heads + head) * a.seq;
  const int kpos = k_begin + (lane & 31);
  const bool kok = kpos < k_end && kpos >= a.first;

  const int q_first = CAUSAL ? wg_begin : 0;  // earlier queries never see a key of this block
  const int qmin = CAUSAL ? a.first : 0;
  const int nt = (a.seq - q_first + 63) / 64;
  SharedTile<D, 64> rq, rdo;
  float rstat = 0.f;
  auto fetch = [&](int t) {
    const int q0 = q_first + t * 64;
    rq.load(Qp, a.ld, q0, qmin, a.seq, tid);
    rdo.load(dOp, a.hp, q0, qmin, a.seq, tid);
    if (tid < 128) {
      const int qp = min(q0 + (tid & 63), a.seq - 1);
      rstat = (tid < 64 ? lsep : dlp)[qp];
    }
  };
  auto park = [&](int t) {
    char* st = lds + (t % 3) * L::kStage;
    rq.store(st, tid);
    rdo.store(st + L::kTile, tid);
    if (tid < 128) reinterpret_cast<float*>(st + 2 * L::kTile)[tid] = tid < 64 ? rstat * kLog2e : rstat;
  };
  bf16x8 kf[KS], vf[KS];
  {
    SharedTile<D, 64> rk, rv;
    rk.load(Kp, a.ld, wg_begin, a.first, a.pos0 + a.npos, tid);
    rv.load(Vp, a.ld, wg_begin, a.first, a.pos0 + a.npos, tid);
    fetch(0);
    char* st = lds + 2 * L::kStage;
    rk.store(st, tid);
    rv.store(st + L::kTile, tid);
    park(0);
    if (nt > 1) fetch(1);
    lds_barrier();
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      kf[ks] = tile_kc<D>(st, 32 * jg, ks, lane);
      vf[ks] = tile_kc<D>(st + L::kTile, 32 * jg, ks, lane);
    }
  }
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int i = 0; i < DT; i++) { dk[i] = zero16(); dv[i] = zero16(); }
  f32x16 s, dp;
  auto products = [&](const char* st, f32x16& s1, f32x16& dp1) {  // S and dP of this wave's half of the tile in st
    s1 = zero16();
    dp1 = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      s1 = MFMA(tile_kc<D>(st, 32 * rg, ks, lane), kf[ks], s1);
      dp1 = MFMA(tile_kc<D>(st + L::kTile, 32 * rg, ks, lane), vf[ks], dp1);
    }
  };
  products(lds, s, dp);
  if (nt > 1) park(1);
  if (nt > 2) fetch(2);
  lds_barrier();  // also: every wave has its keys, so stage 2 may take tile 2
  auto tile = [&](auto mask_c, auto next_c, int t) {
    constexpr bool MASK = decltype(mask_c)::value, NEXT = decltype(next_c)::value;
    const char* cur = lds + (t % 3) * L::kStage;
    const float* lstat = reinterpret_cast<const float*>(cur + 2 * L::kTile) + 32 * rg;  // [64] lse * log2(e), [64] delta
    const int q0 = q_first + t * 64 + 32 * rg;
    if (NEXT && t + 2 < nt) {
      park(t + 2);
      if (t + 3 < nt) fetch(t + 3);
    }
    Philox4 dw;  // the four lanes of a quad share the keys of a 4 x 4 block: each draws the block of one group of queries
    if (DROP) dw = attn_drop_block(a, (uint32_t)kpos >> 2, (uint32_t)(q0 + 8 * (lane & 3) + 4 * g) >> 2, (uint32_t)(seq_idx * a.heads_total + a.head0 + head));
    f32x16 sn, dpn;
    if constexpr (NEXT) products(lds + ((t + 1) % 3) * L::kStage, sn, dpn);
    auto group = [&](auto i4_c) {
      constexpr int I4 = decltype(i4_c)::value;
      const int ql = 8 * I4 + 4 * g;  // 4 consecutive queries
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(lstat + ql);
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(lstat + 64 + ql);
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int i = 4 * I4 + e;
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.scale_log2, -l4[e]));
        float dpe = dp[i], pv = p;  // pv: what multiplied V in forward
        if (DROP) {  // this lane's key is byte (kpos mod 4) of the word of query e of the group
          const bool keep = ((quad_lane<I4>(dw.v[e]) >> (8 * (kpos & 3))) & 0xffu) >= a.dthresh;
          dpe = keep ? dpe * a.dscale : 0.f;
          pv = keep ? p * a.dscale : 0.f;
        }
        float ds = p * (dpe - d4[e]);
        if (MASK) {
          const int qp = q0 + ql + e;
          if (qp >= a.seq || (CAUSAL && kpos > qp)) { pv = 0.f; ds = 0.f; }   // select, never multiply: the rest may be NaN
        }
        s[i] = pv;
        dp[i] = ds;
      }
    };
    group(std::integral_constant<int, 0>{});
    group(std::integral_constant<int, 1>{});
    group(std::integral_constant<int, 2>{});
    group(std::integral_constant<int, 3>{});
#pragma unroll
    for (int j = 0; j < 2; j++) {
      bf16x8 pa = pack8(s, 8 * j);
      bf16x8 da = pack8(dp, 8 * j);
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        dv[dt] = MFMA(tile_mc<D>(cur + L::kTile, 32 * rg, j, dt, lane), pa, dv[dt]);
        dk[dt] = MFMA(tile_mc<D>(cur, 32 * rg, j, dt, lane), da, dk[dt]);
      }
    }
    if constexpr (NEXT) {
      s = sn;
      dp = dpn;
      lds_barrier();
    }
  };
  // The mask matters to the first tile (diagonal) and to the last (end of the sequence); in between there is one form of a tile, so that the
  // accumulators stay where they are.
  using T_ = std::true_type;
  using F_ = std::false_type;
  int t = 0;
  if (nt > 1) {
    tile(T_{}, T_{}, 0);
    for (t = 1; t + 1 < nt; t++) tile(F_{}, T_{}, t);
  }
  tile(T_{}, F_{}, t);
  uint16_t* dKp = a.dqkv + (rowbase + kpos) * a.ld + a.hp + head * D;
  uint16_t* dVp = dKp + a.hp;
  combine_parts<E, 2, 2>(dk, lds, jg, rg, lane, [&](int e, const f32x4& v) {
    const int d = (e / 16) * 32 + 8 * ((e % 16) >> 2) + 4 * g;
    if (kok) *reinterpret_cast<u32x2*>(dKp + d) = u32x2{pack_bf16x2(v[0] * a.scale, v[1] * a.scale), pack_bf16x2(v[2] * a.scale, v[3] * a.scale)};
  });
  combine_parts<E, 2, 2>(dv, lds, jg, rg, lane, [&](int e, const f32x4& v) {
    const int d = (e / 16) * 32 + 8 * ((e % 16) >> 2) + 4 * g;
    if (kok) *reinterpret_cast<u32x2*>(dVp + d) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  });
}

// =================================================================================================
// backward over blocks of 32 rows, a wave by itself.  The four waves of a workgroup split the reduction range -- the 32-row key tiles
// a query block sees, or the 32-row query tiles that see a key block -- round-robin, each staging its own tiles in a private
// slice of LDS, so the loops need no barrier; the four partial results meet once, through LDS, at the end.  Rows are padded
// instead of swizzled.  This form stays where the shared tiles above do not pay: calls with few blocks, whose time is the
// chain of the longest one (a quarter of it per wave here).  With rotary embeddings dQ and dK can leave it as gradients of what was
// rotated -- the values that a launch over dqkv would read, rounded like them -- which saves that launch and its gap: two
// recomputed layers of h 1024, 512 tokens, 538 -> 534 us a step.
// =================================================================================================
template <int D>
struct WaveLds {  // LDS of a backward workgroup: the larger of the two passes' staging areas and of the partial-sum exchange
  static constexpr int E = (D / 32) * 16;
  static constexpr int kStageDq = 4 * 2 * AT<D>::bytes, kStageDkv = 4 * (2 * AT<D>::bytes + 256), kPart = 4 * E * 64 * 4;
  static constexpr int bytes = kStageDkv > kPart ? kStageDkv : kPart;
  static_assert(kStageDkv >= kStageDq, "the dK/dV staging area is the larger one");
};

template <int D, bool CAUSAL, bool DROP, bool ROPE = false>
__device__ __forceinline__ void wave_dq_block(const AttnArgs& a, int wg, char* lds, const float2* rope = nullptr) {
  constexpr int KS = D / 16, DT = D / 32, E = DT * 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5;
  int pair, blk;
  decode_block(wg, a.nseq * a.heads, a.blocks, pair, blk);
  const int sq = pair / a.heads, head = pair % a.heads, qb = a.blocks - 1 - blk;
  const int seq_idx = a.seq0 + sq;
  const int q_begin = a.pos0 + qb * 32;
  const int q_end = min(a.pos0 + a.npos, q_begin + 32);
  const size_t rowbase = (size_t)seq_idx * a.seq;
  const uint16_t* Qp = a.qkv + rowbase * a.ld + head * D;
  const uint16_t* Kp = Qp + a.hp;
  const uint16_t* Vp = Qp + 2 * a.hp;
  const uint16_t* dOp = a.dout + rowbase * a.hp + head * D;
  const int qpos = q_begin + (lane & 31);
  const bool qok = qpos < q_end && qpos >= a.first;

  bf16x8 qf[KS], dof[KS];
  load_row_frags<D>(qf, Qp + (size_t)qpos * a.ld, qok, g);
  load_row_frags<D>(dof, dOp + (size_t)qpos * a.hp, qok, g);
  float lse2 = 0.f, dl = 0.f;
  if (qok) {
    size_t si = ((size_t)seq_idx * a.heads + head) * a.seq + qpos;
    lse2 = a.lse[si] * kLog2e;
    dl = a.delta[si];
  }
  f32x16 acc[DT];
#pragma unroll
  for (int i = 0; i < DT; i++) acc[i] = zero16();

  const int kv_end = CAUSAL ? q_end : a.seq;
  const int nt = (kv_end + 31) / 32;
  char* lk = lds + wave * 2 * AT<D>::bytes;
  char* lv = lk + AT<D>::bytes;
  u32x4 rk[AT<D>::per_lane], rv[AT<D>::per_lane];
  if (wave < nt) {
    wave_load<D>(rk, Kp, a.ld, wave * 32, 0, kv_end, lane);
    wave_load<D>(rv, Vp, a.ld, wave * 32, 0, kv_end, lane);
  }
  for (int t = wave; t < nt; t += 4) {
    const int kv0 = t * 32;
    wave_store<D>(rk, lk, lane);
    wave_store<D>(rv, lv, lane);
    if (t + 4 < nt) {
      wave_load<D>(rk, Kp, a.ld, kv0 + 128, 0, kv_end, lane);
      wave_load<D>(rv, Vp, a.ld, kv0 + 128, 0, kv_end, lane);
    }
    f32x16 s = zero16(), dp = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      s = MFMA(kc_frag<D>(lk, ks, lane), qf[ks], s);
      dp = MFMA(kc_frag<D>(lv, ks, lane), dof[ks], dp);
    }
    const bool need_mask = (kv0 + 32 > a.seq) || (CAUSAL && kv0 + 31 > q_begin);
    if (DROP) {  // dP = dropout factor * (dO V^T)
      uint32_t w[4];
      drop_words_of_query(a, w, kv0 + 4 * g, qpos, (uint32_t)(seq_idx * a.heads_total + a.head0 + head), lane);
#pragma unroll
      for (int grp = 0; grp < 4; grp++)
#pragma unroll
        for (int e = 0; e < 4; e++) dp[4 * grp + e] = ((w[grp] >> (8 * e)) & 0xffu) >= a.dthresh ? dp[4 * grp + e] * a.dscale : 0.f;
    }
    // only tiles on the diagonal or at the end of the sequence pay for the mask (a wave-uniform branch)
    auto scores = [&](auto mask_c) {
#pragma unroll
      for (int i = 0; i < 16; i++) {
        float ds = __builtin_amdgcn_exp2f(s[i] * a.scale_log2 - lse2) * (dp[i] - dl);
        if (decltype(mask_c)::value) {
          int kvpos = kv0 + 8 * (i >> 2) + 4 * g + (i & 3);
          if (kvpos >= a.seq || (CAUSAL && kvpos > qpos)) ds = 0.f;
        }
        s[i] = ds;
      }
    };
    if (need_mask) scores(std::true_type{}); else scores(std::false_type{});
#pragma unroll
    for (int j = 0; j < 2; j++) {
      bf16x8 db = pack8(s, 8 * j);
#pragma unroll
      for (int dt = 0; dt < DT; dt++) acc[dt] = MFMA(mc_frag<D>(lk, j, 32 * dt, lane), db, acc[dt]);
    }
  }
  const float one[4] = {1.f, 1.f, 1.f, 1.f};
  float res[E / 4];
  combine4<E, ROPE>(acc, reinterpret_cast<float*>(lds), wave, lane, one, res);
  if (qok) {
    uint16_t* op = a.dqkv + (rowbase + qpos) * a.ld + head * D;
#pragma unroll
    for (int k = 0; k < (ROPE ? E / 8 : E / 4); k += 4) {
      const int e = part_element<E, ROPE>(wave, k), dt = e / 16, i = e % 16;
      const int d = dt * 32 + 8 * (i >> 2) + 4 * g;
      u32x2 v = {pack_bf16x2(res[k] * a.scale, res[k + 1] * a.scale), pack_bf16x2(res[k + 2] * a.scale, res[k + 3] * a.scale)};
      if constexpr (ROPE) {
        const float* hi = res + E / 8 + k;
        u32x2 w = {pack_bf16x2(hi[0] * a.scale, hi[1] * a.scale), pack_bf16x2(hi[2] * a.scale, hi[3] * a.scale)};
        float lo_[4], hi_[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
          lo_[j] = bf16_bits_to_f32((j & 1) ? v[j >> 1] >> 16 : v[j >> 1] & 0xffffu);
          hi_[j] = bf16_bits_to_f32((j & 1) ? w[j >> 1] >> 16 : w[j >> 1] & 0xffffu);
          turn_back(lo_[j], hi_[j], rope[(size_t)qpos * (D / 2) + d + j]);
        }
        v = u32x2{pack_bf16x2(lo_[0], lo_[1]), pack_bf16x2(lo_[2], lo_[3])};
        *reinterpret_cast<u32x2*>(op + d + D / 2) = u32x2{pack_bf16x2(hi_[0], hi_[1]), pack_bf16x2(hi_[2], hi_[3])};
      }
      *reinterpret_cast<u32x2*>(op + d) = v;
    }
  }
}

// dK, dV of a 32-key block; the four waves split the 32-query tiles that see it
template <int D, bool CAUSAL, bool DROP, bool ROPE = false>
__device__ __forceinline__ void wave_dkv_block(const AttnArgs& a, int wg, char* lds, const float2* rope = nullptr) {
  constexpr int KS = D / 16, DT = D / 32, E = DT * 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5;
  int pair, kb;
  decode_block(wg, a.nseq * a.heads, a.blocks, pair, kb);  // early key blocks are the long ones
  const int sq = pair / a.heads, head = pair % a.heads;
  const int seq_idx = a.seq0 + sq;
  const int k_begin = a.pos0 + kb * 32;
  const int k_end = min(a.pos0 + a.npos, k_begin + 32);
  const size_t rowbase = (size_t)seq_idx * a.seq;
  const uint16_t* Qp = a.qkv + rowbase * a.ld + head * D;
  const uint16_t* Kp = Qp + a.hp;
  const uint16_t* Vp = Qp + 2 * a.hp;
  const uint16_t* dOp = a.dout + rowbase * a.hp + head * D;
  const float* lsep = a.lse + ((size_t)seq_idx * a.heads + head) * a.seq;
  const float* dlp = a.delta + ((size_t)seq_idx * a.heads + head) * a.seq;
  const int kpos = k_begin + (lane & 31);
  const bool kok = kpos < k_end && kpos >= a.first;

  bf16x8 kf[KS], vf[KS];
  load_row_frags<D>(kf, Kp + (size_t)kpos * a.ld, kok, g);
  load_row_frags<D>(vf, Vp + (size_t)kpos * a.ld, kok, g);
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int i = 0; i < DT; i++) { dk[i] = zero16(); dv[i] = zero16(); }

  const int qt0 = CAUSAL ? k_begin / 32 : 0;   // first query tile that sees this key block
  const int qmin = CAUSAL ? a.first : 0;       // earlier queries never see a key of this row range
  const int nqt = (a.seq + 31) / 32;
  char* lq = lds + wave * (2 * AT<D>::bytes + 256);
  char* ldo = lq + AT<D>::bytes;
  float* lstat = reinterpret_cast<float*>(ldo + AT<D>::bytes);  // [32] lse * log2(e), [32] delta
  u32x4 rq[AT<D>::per_lane], rdo[AT<D>::per_lane];
  float rstat = 0.f;
  auto fetch = [&](int t) {
    wave_load<D>(rq, Qp, a.ld, t * 32, qmin, a.seq, lane);
    wave_load<D>(rdo, dOp, a.hp, t * 32, qmin, a.seq, lane);
    const int qp = min(t * 32 + (lane & 31), a.seq - 1);
    rstat = g == 0 ? lsep[qp] * kLog2e : dlp[qp];
  };
  if (qt0 + wave < nqt) fetch(qt0 + wave);
  for (int t = qt0 + wave; t < nqt; t += 4) {
    const int q0 = t * 32;
    wave_store<D>(rq, lq, lane);
    wave_store<D>(rdo, ldo, lane);
    lstat[lane] = rstat;
    if (t + 4 < nqt) fetch(t + 4);
    f32x16 s = zero16(), dp = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      s = MFMA(kc_frag<D>(lq, ks, lane), kf[ks], s);
      dp = MFMA(kc_frag<D>(ldo, ks, lane), vf[ks], dp);
    }
    const bool need_mask = (q0 + 32 > a.seq) || (CAUSAL && q0 < k_begin + 31);
    Philox4 dw;  // the four lanes of a quad share the keys of a 4 x 4 block: each draws the block of one group of queries
    if (DROP) dw = attn_drop_block(a, (uint32_t)kpos >> 2, (uint32_t)(q0 + 8 * (lane & 3) + 4 * g) >> 2, (uint32_t)(seq_idx * a.heads_total + a.head0 + head));
    // only tiles on the diagonal or at the end of the sequence pay for the mask (a wave-uniform branch)
    auto scores = [&](auto mask_c) {
      auto group = [&](auto i4_c) {
        constexpr int I4 = decltype(i4_c)::value;
        const int ql = 8 * I4 + 4 * g;  // 4 consecutive queries
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(lstat + ql);
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(lstat + 32 + ql);
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int i = 4 * I4 + e;
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.scale_log2, -l4[e]));
          float dpe = dp[i], pv = p;  // pv: what multiplied V in forward
          if (DROP) {  // this lane's key is byte (kpos mod 4) of the word of query e of the group
            const bool keep = ((quad_lane<I4>(dw.v[e]) >> (8 * (kpos & 3))) & 0xffu) >= a.dthresh;
            dpe = keep ? dpe * a.dscale : 0.f;
            pv = keep ? p * a.dscale : 0.f;
          }
          float ds = p * (dpe - d4[e]);
          if (decltype(mask_c)::value) {
            const int qp = q0 + ql + e;
            if (qp >= a.seq || (CAUSAL && kpos > qp)) { pv = 0.f; ds = 0.f; }   // select, never multiply: the rest may be NaN
          }
          s[i] = pv;
          dp[i] = ds;
        }
      };
      group(std::integral_constant<int, 0>{});
      group(std::integral_constant<int, 1>{});
      group(std::integral_constant<int, 2>{});
      group(std::integral_constant<int, 3>{});
    };
    if (need_mask) scores(std::true_type{}); else scores(std::false_type{});
#pragma unroll
    for (int j = 0; j < 2; j++) {
      bf16x8 pa = pack8(s, 8 * j);
      bf16x8 da = pack8(dp, 8 * j);
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        dv[dt] = MFMA(pa, mc_frag<D>(ldo, j, 32 * dt, lane), dv[dt]);
        dk[dt] = MFMA(da, mc_frag<D>(lq, j, 32 * dt, lane), dk[dt]);
      }
    }
  }
  // accumulator row = key 8*(i/4) + 4g + i%4 of the block, column = d = 32*dt + l%32
  const float one[4] = {1.f, 1.f, 1.f, 1.f};
  float rk_[E / 4], rv_[E / 4];
  combine4<E, ROPE>(dk, reinterpret_cast<float*>(lds), wave, lane, one, rk_);
  combine4<E, ROPE>(dv, reinterpret_cast<float*>(lds), wave, lane, one, rv_);
  uint16_t* dKp = a.dqkv + rowbase * a.ld + a.hp + head * D;
  uint16_t* dVp = dKp + a.hp;
#pragma unroll
  for (int k = 0; k < (ROPE ? E / 8 : E / 4); k++) {
    const int e = part_element<E, ROPE>(wave, k), dt = e / 16, i = e % 16;
    const int kp = k_begin + 8 * (i >> 2) + 4 * g + (i & 3), d = dt * 32 + (lane & 31);
    if (kp < k_end && kp >= a.first) {
      const size_t o = (size_t)kp * a.ld + d;
      uint16_t lo = (uint16_t)f32_to_bf16_bits(rk_[k] * a.scale);
      if constexpr (ROPE) {
        constexpr int H = E / 8;
        uint16_t hi = (uint16_t)f32_to_bf16_bits(rk_[H + k] * a.scale);
        float x1 = bf16_bits_to_f32(lo), x2 = bf16_bits_to_f32(hi);
        turn_back(x1, x2, rope[(size_t)kp * (D / 2) + d]);
        lo = (uint16_t)f32_to_bf16_bits(x1);
        dKp[o + D / 2] = (uint16_t)f32_to_bf16_bits(x2);
        dVp[o + D / 2] = (uint16_t)f32_to_bf16_bits(rv_[H + k]);
      }
      dKp[o] = lo;
      dVp[o] = (uint16_t)f32_to_bf16_bits(rv_[k]);
    }
  }
}

// dQ as a launch of its own, which leaves delta behind if it covers every query that dK/dV reads
template <int D, int QG, bool CAUSAL, bool DROP, bool OWN_DELTA>
__global__ __launch_bounds__(NT, 2) void attn_dq_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) char lds[BwdLds<D, QG, 4 / QG>::bytes];
  attn_dq_block<D, QG, 4 / QG, CAUSAL, DROP, OWN_DELTA>(a, blockIdx.x, lds);
}
template <int JG, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(NT, 2) void attn_dkv_kernel(AttnArgs a) {  // D = 64
  __shared__ __attribute__((aligned(16))) char lds[BwdLds<64, JG, 4 / JG>::bytes];
  attn_dkv_block<64, JG, 4 / JG, CAUSAL, DROP>(a, blockIdx.x, lds);
}
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(NT, 1) void wave_dq_kernel(AttnArgs a) {  // D = 128
  __shared__ __attribute__((aligned(16))) char lds[WaveLds<128>::bytes];
  wave_dq_block<128, CAUSAL, DROP>(a, blockIdx.x, lds);
}
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(NT, 1) void wave_dkv_kernel(AttnArgs a) {  // D = 128
  __shared__ __attribute__((aligned(16))) char lds[WaveLds<128>::bytes];
  wave_dkv_block<128, CAUSAL, DROP>(a, blockIdx.x, lds);
}
// Both passes in ONE launch, for calls with few blocks (at most one workgroup per CU and pass): the passes are independent (dK/dV
// per key block, dQ per query block) and each alone leaves the chip waiting for its longest workgroups, so their workgroups
// are dealt out together -- groups of eight ids (one per XCD) alternate between a dK/dV block and a dQ block, long blocks of
// both kinds first.  Measured (256 blocks of 2048-token sequences, D = 128): 40 -> 32 us; with 512 blocks and more the single
// launch is about 10 % slower than two.
template <int D, bool CAUSAL, bool DROP, bool ROPE>
__device__ __forceinline__ void both_passes_block(const AttnArgs& a, int n_blocks, const float2* rope, char* lds) {
  const int w = blockIdx.x, idx = (w >> 4) * 8 + (w & 7);
  if (idx >= n_blocks) return;  // the last group of eight may be ragged (whole workgroup leaves: no barrier is skipped by part of it)
  if ((w >> 3) & 1) wave_dq_block<D, CAUSAL, DROP, ROPE>(a, idx, lds, rope);
  else wave_dkv_block<D, CAUSAL, DROP, ROPE>(a, idx, lds, rope);
}
template <int D, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(NT, 1) void attn_bwd_kernel(AttnArgs a, int n_blocks) {
  __shared__ __attribute__((aligned(16))) char lds[WaveLds<D>::bytes];
  both_passes_block<D, CAUSAL, DROP, false>(a, n_blocks, nullptr, lds);
}
// the same for a pass with rotary embeddings: dQ and dK stored turned back by rope, (cos, sin) [seq, D / 2].  A kernel of its own: with the table
// among its arguments and the other order of stores the one above took, D = 128, 10.0 -> 10.4 us for 4 x 16 x 8 and 17.6 -> 18.1 for 5 x 80 x 10.
template <int D, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(NT, 1) void attn_bwd_rope_kernel(AttnArgs a, int n_blocks, const float2* rope) {
  __shared__ __attribute__((aligned(16))) char lds[WaveLds<D>::bytes];
  both_passes_block<D, CAUSAL, DROP, true>(a, n_blocks, rope, lds);
}

// blocks of `groups` x 32 rows over the positions of the row range
void set_blocks(AttnArgs& a, int groups) {
  const int end = a.pos0 + a.npos;
  a.pos0 = a.first & ~(32 * groups - 1);
  a.npos = end - a.pos0;
  a.blocks = (a.npos + 32 * groups - 1) / (32 * groups);
}

int fill_args(AttnArgs& a, int batch, int seq, int heads, int head_dim, int causal, int row0, int rows, const char* who) {
  if (batch <= 0 || seq <= 0 || heads <= 0 || (head_dim != 64 && head_dim != 128) || row0 < 0 || rows <= 0 ||
      (long)row0 + rows > (long)batch * seq) {
    set_error("%s: bad shape (batch=%d seq=%d heads=%d head_dim=%d row0=%d rows=%d)", who, batch, seq, heads, head_dim, row0, rows);
    return OASES_EINVAL;
  }
  a.seq = seq;
  a.heads = heads;
  a.hp = heads * head_dim;
  a.ld = 3 * a.hp;
  a.seq0 = row0 / seq;
  if (row0 % seq == 0 && rows % seq == 0) {
    a.first = a.pos0 = 0;
    a.npos = seq;
    a.blocks = (seq + 31) / 32;
    return rows / seq;  // number of sequences
  }
  if (row0 / seq != (row0 + rows - 1) / seq) {
    set_error("%s: rows [%d,%d) are neither whole sequences nor part of one sequence", who, row0, row0 + rows);
    return OASES_EINVAL;
  }
  if (!causal) {
    set_error("%s: a row range inside one sequence needs causal attention", who);
    return OASES_EINVAL;
  }
  a.first = row0 % seq;
  a.npos = rows;
  a.pos0 = a.first;
  set_blocks(a, 1);
  return 1;
}

}  // namespace

// fills the dropout fields; false (after set_error) on a bad rate or head range
static bool fill_dropout(AttnArgs& a, uint64_t seed, int layer, float p_attn, int head0, int heads_total, int heads, const char* who) {
  if (!(p_attn >= 0.f && p_attn < 1.f)) { set_error("%s: attention dropout rate %g outside [0,1)", who, (double)p_attn); return false; }
  int T = (int)__builtin_rint((double)p_attn * 256.0);
  if (T > 255) T = 255;
  a.dthresh = (uint32_t)T;
  if (T == 0) return true;
  if (heads_total <= 0 || head0 < 0 || head0 + heads > heads_total) { set_error("%s: heads [%d,%d) outside the %d heads of the layer", who, head0, head0 + heads, heads_total); return false; }
  a.dk0 = (uint32_t)seed;
  a.dk1 = (uint32_t)(seed >> 32);
  a.dc3 = ((uint32_t)layer & 0x7fffffffu) | 0x80000000u;
  a.dscale = (float)(256.0 / (256.0 - T));
  a.head0 = head0;
  a.heads_total = heads_total;
  return true;
}

// 32-row groups of a workgroup that shares its tiles: two halve the tiles read from L2, one has half as long a chain of tiles.
// Two once they fill the chip twice, or once and the chains are short.  Both sides measured, forward / backward, us, one group
// -> two (causal, batch x seq x heads x columns): 8x1024x8x64 40.6 / 104.9 -> 31.4 / 77.2, 4x2048x4x128 57.5 / 155 -> 40.5 / 132,
// 8x512x4x64 9.6 / 24.7 -> 9.1 / 23.7, 8x256x8x128 10.8 / 40.9 -> 9.1 / 33.3, but 1x2048x8x64 18.9 / 47.8 -> 25.7 / 62.9 and 2x2048x4x128
// 30.3 / 79.9 -> 38.2 / 86.0.
// nseq, npos: sequences and positions of the row range, or of the whole batch for a choice that does not depend on the range (pin)
static int attn_query_groups(const AttnArgs& a, int nseq, int npos) {
  const long blocks = (long)nseq * a.heads * ((npos + 63) / 64);
  return blocks >= 512 || (blocks >= 256 && a.seq <= 512) ? 2 : 1;
}

int launch_attention_fwd(const void* qkv, void* out, float* lse, int batch, int seq, int heads, int head_dim, int causal,
                         int row0, int rows, hipStream_t s, uint64_t seed, int layer, float p_attn, int head0, int heads_total,
                         bool pin) {
  if (!qkv || !out || !lse) { set_error("attention_fwd: NULL argument"); return OASES_ENULL; }
  if (!aligned16(qkv) || !aligned16(out)) { set_error("attention_fwd: pointer not 16-byte aligned"); return OASES_EALIGN; }
  AttnArgs a{};
  int nseq = fill_args(a, batch, seq, heads, head_dim, causal, row0, rows, "attention_fwd");
  if (nseq < 0) return nseq;
  a.qkv = (const uint16_t*)qkv;
  a.out_w = (uint16_t*)out;
  a.lse = lse;
  a.scale = 1.0f / sqrtf((float)head_dim);
  a.scale_log2 = a.scale * kLog2e;
  a.nseq = nseq;
  if (!fill_dropout(a, seed, layer, p_attn, head0, heads_total, heads, "attention_fwd")) return OASES_EINVAL;
  const int qg = attn_query_groups(a, pin ? batch : nseq, pin ? seq : a.npos);
  set_blocks(a, qg);
  dim3 grid(nseq * a.blocks * heads), block(NT);
#define OASES_ATTN_FWD_Q(DD, QQ, CC)                                                                        \
  do {                                                                                                      \
    if (a.dthresh) hipLaunchKernelGGL((attn_fwd_kernel<DD, QQ, 4 / QQ, CC, true>), grid, block, 0, s, a);   \
    else hipLaunchKernelGGL((attn_fwd_kernel<DD, QQ, 4 / QQ, CC, false>), grid, block, 0, s, a);            \
  } while (0)
#define OASES_ATTN_FWD(DD, CC) do { if (qg == 2) OASES_ATTN_FWD_Q(DD, 2, CC); else OASES_ATTN_FWD_Q(DD, 1, CC); } while (0)
  if (head_dim == 64) { if (causal) OASES_ATTN_FWD(64, true); else OASES_ATTN_FWD(64, false); }
  else { if (causal) OASES_ATTN_FWD(128, true); else OASES_ATTN_FWD(128, false); }
#undef OASES_ATTN_FWD
#undef OASES_ATTN_FWD_Q
  OASES_LAUNCH_CHECK("attn_fwd_kernel");
  return 0;
}

// How the backward of a call is launched.
struct BwdPlan {
  bool one_launch;  // both passes together
  int qg;           // 32-row groups of a workgroup that shares its tiles
  bool own_delta;   // dQ covers every query that dK/dV reads, and forms delta on the way
};
static BwdPlan bwd_plan(const AttnArgs& a, int nseq, int batch, int head_dim, bool pin) {
  BwdPlan p;
  const int choice_blocks = (pin ? batch * ((a.seq + 31) / 32) : nseq * a.blocks) * a.heads;
  // (dropout makes a tile several times the work: there the launch pays up to half as many; 256 blocks of 512-token sequences, D = 64,
  // in one launch against two: 17.5 -> 18.4 us without dropout, 24.0 -> 19.6 with)
  p.one_launch = choice_blocks <= (a.dthresh && head_dim == 64 ? 128 : 256);
  p.qg = attn_query_groups(a, pin ? batch : nseq, pin ? a.seq : a.npos);
  const bool wave_dq = head_dim == 128 && p.qg == 1;
  p.own_delta = !p.one_launch && !wave_dq && a.npos == a.seq;
  return p;
}
bool attention_bwd_turns_back(int batch, int seq, int heads, int head_dim, int causal, float p_attn) {
  AttnArgs a{};
  const int nseq = fill_args(a, batch, seq, heads, head_dim, causal, 0, batch * seq, "attention_bwd");
  return nseq > 0 && fill_dropout(a, 0, 0, p_attn, 0, heads, heads, "attention_bwd") && bwd_plan(a, nseq, batch, head_dim, false).one_launch;
}
bool attention_bwd_forms_delta(int batch, int seq, int heads, int head_dim, int causal, float p_attn) {
  AttnArgs a{};
  const int nseq = fill_args(a, batch, seq, heads, head_dim, causal, 0, batch * seq, "attention_bwd");
  return nseq > 0 && fill_dropout(a, 0, 0, p_attn, 0, heads, heads, "attention_bwd") && bwd_plan(a, nseq, batch, head_dim, false).own_delta;
}

int launch_attention_bwd(const void* qkv, const void* out, const void* dout, const float* lse, float* delta, void* dqkv,
                         int batch, int seq, int heads, int head_dim, int causal, int row0, int rows, hipStream_t s, uint64_t seed,
                         int layer, float p_attn, int head0, int heads_total, bool pin, bool delta_ready,
                         const float* rope) {
  if (!qkv || !out || !dout || !lse || !delta || !dqkv) { set_error("attention_bwd: NULL argument"); return OASES_ENULL; }
  if (!aligned16(qkv) || !aligned16(out) || !aligned16(dout) || !aligned16(dqkv)) {
    set_error("attention_bwd: pointer not 16-byte aligned");
    return OASES_EALIGN;
  }
  AttnArgs a{};
  int nseq = fill_args(a, batch, seq, heads, head_dim, causal, row0, rows, "attention_bwd");
  if (nseq < 0) return nseq;
  a.qkv = (const uint16_t*)qkv;
  a.out = (const uint16_t*)out;
  a.dout = (const uint16_t*)dout;
  a.lse = const_cast<float*>(lse);
  a.delta = delta;
  a.dqkv = (uint16_t*)dqkv;
  a.scale = 1.0f / sqrtf((float)head_dim);
  a.scale_log2 = a.scale * kLog2e;
  // delta for every query that sees a key of the range: from the first row to the end of the last sequence
  const int first_row = row0;
  const int n_rows = (a.seq0 + nseq) * seq - row0;
  const long pairs = (long)n_rows * heads * (head_dim / 8);
  a.nseq = nseq;
  if (!fill_dropout(a, seed, layer, p_attn, head0, heads_total, heads, "attention_bwd")) return OASES_EINVAL;
  dim3 dgrid((unsigned)((pairs + NT - 1) / NT)), block(NT);
  const int n_blocks = nseq * a.blocks * heads;  // of 32 rows
  const BwdPlan plan = bwd_plan(a, nseq, batch, head_dim, pin);
  if (rope && !plan.one_launch) { set_error("attention_bwd: dQ and dK are turned back by the kernel of both passes only"); return OASES_EINVAL; }
  const float2* const table = reinterpret_cast<const float2*>(rope);
  const bool one_launch = plan.one_launch, own_delta = plan.own_delta;
  const int qg = plan.qg;
  if (!own_delta && !delta_ready) {
    if (head_dim == 64) hipLaunchKernelGGL((attn_delta_kernel<64>), dgrid, block, 0, s, a, first_row, n_rows);
    else hipLaunchKernelGGL((attn_delta_kernel<128>), dgrid, block, 0, s, a, first_row, n_rows);
    OASES_LAUNCH_CHECK("attn_delta_kernel");
  }
  AttnArgs q = a;
  set_blocks(q, qg);
  const dim3 bgrid(2 * ((n_blocks + 7) / 8) * 8), grid(n_blocks), qgrid(nseq * q.blocks * heads);
#define OASES_ATTN_DQ(DD, QQ, CC, DR)                                                                               \
  do {                                                                                                              \
    if (own_delta) hipLaunchKernelGGL((attn_dq_kernel<DD, QQ, CC, DR, true>), qgrid, block, 0, s, q);               \
    else if constexpr (CC) hipLaunchKernelGGL((attn_dq_kernel<DD, QQ, CC, DR, false>), qgrid, block, 0, s, q);      \
  } while (0)
#define OASES_ATTN_BWD(DD, CC, DR)                                                                                  \
  do {                                                                                                              \
    if (one_launch) {                                                                                               \
      if (table) hipLaunchKernelGGL((attn_bwd_rope_kernel<DD, CC, DR>), bgrid, block, 0, s, a, n_blocks, table);    \
      else hipLaunchKernelGGL((attn_bwd_kernel<DD, CC, DR>), bgrid, block, 0, s, a, n_blocks);                      \
    } else {                                                                                                        \
      if (qg == 2) OASES_ATTN_DQ(DD, 2, CC, DR);                                                                    \
      else if constexpr (DD == 64) OASES_ATTN_DQ(DD, 1, CC, DR);                                                    \
      else hipLaunchKernelGGL((wave_dq_kernel<CC, DR>), grid, block, 0, s, a);                                      \
      if (DD == 128 && qg == 2) hipLaunchKernelGGL((attn_dkv128_kernel<CC, DR>), qgrid, block, 0, s, q);               \
      else if constexpr (DD == 128) hipLaunchKernelGGL((wave_dkv_kernel<CC, DR>), grid, block, 0, s, a);                 \
      else if (qg == 2) hipLaunchKernelGGL((attn_dkv_kernel<2, CC, DR>), qgrid, block, 0, s, q);                    \
      else hipLaunchKernelGGL((attn_dkv_kernel<1, CC, DR>), qgrid, block, 0, s, q);                                 \
    }                                                                                                               \
  } while (0)
#define OASES_ATTN_BWD_D(DD, CC) do { if (a.dthresh) OASES_ATTN_BWD(DD, CC, true); else OASES_ATTN_BWD(DD, CC, false); } while (0)
  if (head_dim == 64) { if (causal) OASES_ATTN_BWD_D(64, true); else OASES_ATTN_BWD_D(64, false); }
  else { if (causal) OASES_ATTN_BWD_D(128, true); else OASES_ATTN_BWD_D(128, false); }
#undef OASES_ATTN_BWD_D
#undef OASES_ATTN_BWD
#undef OASES_ATTN_DQ
  OASES_LAUNCH_CHECK("attn_bwd kernels");
  return 0;
}

}  // namespace oases
