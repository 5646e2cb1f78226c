// bf16 MFMA GEMM family for gfx950: C = A*B with fp32 accumulation, LDS-staged tiles.
//
// One kernel template covers the three contractions of a linear map under Megatron's partition
// (paper Sec. II): forward (A k-contiguous, B n-contiguous), input gradient (both k-contiguous) and
// weight gradient (both stored with the contraction index as the row).  A k-contiguous operand tile
// is kept in LDS as [rows][64 k] with a 16-byte-chunk XOR swizzle (chunk ^ (row/2)%8: 16 consecutive rows of
// 128 bytes then cover all 64 banks once) and read with ds_read_b128; an
// operand stored with the contraction index as row is kept as [64 k][rows] (padded rows) and read
// with the LDS transpose read ds_read_b64_tr_b16, which hands each lane 4 consecutive k of one row.
// v_mfma_f32_32x32x16_bf16 (the register-staged and the four-wave kernels; the others: see the epilogues of 16x16x32): A lane l holds row l%32, k = 8*(l/32)..+7; B the same with columns;
// accumulator element i of lane l is C[8*(i/4) + 4*(l/32) + i%4][l%32].
#include <algorithm>
#include <type_traits>
#ifdef OASES_GEMM_TUNE_HOOK
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#endif

#include "common.h"

// This file is compiled once per contraction form (OASES_GEMM_PART = 0: NN and the host entry points, 1: NT, 2: TN), so
// that the three sets of kernel instantiations build in parallel; without the macro one object holds everything.
#ifndef OASES_GEMM_PART
#define OASES_GEMM_PART -1
#endif
#define OASES_GEMM_HAS(part) (OASES_GEMM_PART < 0 || OASES_GEMM_PART == (part))

namespace oases {

struct GemmArgs {
  const uint16_t* A;
  const uint16_t* B;
  void* C;
  const float* bias;
  uint16_t* aux;
  int M, N, K;
  int lda, ldb, ldc, ldaux;
  int tiles_m, tiles_n;
  int ksplit, k_per;  // split-K: slice s covers k in [s*k_per, min(K, (s+1)*k_per)) and writes partial s
};
// What only some kernels read, apart so that the others are not given it (copying a kernel's arguments is a part of the host time of a launch:
// 88 -> 136 bytes 0.1 us)
struct GemmCall : GemmArgs {
  float* part = nullptr;         // slices that the launch adds up itself (SliceSum): partial sums, and a counter per tile
  uint32_t* counters = nullptr;  // nullptr: slices write planes that a second launch adds up
  // weight gradients of a group: [N], += the column sums of B (a bias gradient), or nullptr; EPI_BF16_DELTA: [M / seq, N / head_dim, seq], the row
  // sums of C * aux over the head_dim columns of a head
  float* sums = nullptr;
  int seq = 0, head_dim = 0;
};

// one launcher per contraction form, each defined in its own part
// choice_rows > 0: the kernel is chosen as if the launch had that many rows (see launch_gemm)
int launch_gemm_nn(const GemmCall& g, int epi, float* ws, size_t ws_bytes, int forced_variant, int choice_rows, hipStream_t s);
int launch_gemm_nt(const GemmCall& g, int epi, float* ws, size_t ws_bytes, int forced_variant, int choice_rows, hipStream_t s);
int launch_gemm_tn(const GemmCall& g, float* ws, size_t ws_bytes, int forced_variant, hipStream_t s);

namespace {

constexpr int BK = 64;          // k extent of one LDS stage
constexpr int kMcPadBytes = 64; // row padding of a "contraction-major" tile (keeps transpose reads off the same banks)


template <int R, bool KC>
struct TileLayout {
  static constexpr int row_bytes = KC ? BK * 2 : R * 2 + kMcPadBytes;
  static constexpr int rows = KC ? R : BK;
  static constexpr int bytes = rows * row_bytes;
  static constexpr int chunks_per_row = KC ? BK / 8 : R / 8;
  static constexpr int chunks = rows * chunks_per_row;
};

// global -> registers for one operand tile.  FULL: the tile lies inside the matrix and the k range inside K,
// so no predicate is needed; otherwise addresses are clamped into the matrix and out-of-range chunks zeroed
// (no divergent branches either way).
template <int R, bool KC, int NT, bool FULL>
__device__ __forceinline__ void load_tile_global(u32x4* regs, const uint16_t* __restrict__ base, int ld, int r0, int k0,
                                                 int rmax, int kmax, int tid) {
  using L = TileLayout<R, KC>;
#pragma unroll
  for (int i = 0; i < L::chunks / NT; i++) {
    int c = tid + i * NT;
    int row = c / L::chunks_per_row, cc = c % L::chunks_per_row;
    int gr, gk;
    if (KC) { gr = r0 + row; gk = k0 + cc * 8; } else { gk = k0 + row; gr = r0 + cc * 8; }
    if (FULL) {
      // uniform base (scalar registers, advanced per k iteration) + one loop-invariant 32-bit lane offset
      static_assert(NT % L::chunks_per_row == 0, "row of a chunk must not depend on the pass");
      constexpr int rows_per_pass = NT / L::chunks_per_row;
      const char* sb = reinterpret_cast<const char*>(base) +
                       ((size_t)(KC ? r0 : k0) * ld + (KC ? k0 : r0) + (size_t)i * rows_per_pass * ld) * 2;
      const uint32_t voff = (uint32_t)(((tid / L::chunks_per_row) * ld + (tid % L::chunks_per_row) * 8) * 2);
      regs[i] = *reinterpret_cast<const u32x4*>(sb + voff);
    } else {
      const bool ok = (gr < rmax) && (gk < kmax);
      const int cr = min(gr, KC ? rmax - 1 : rmax - 8), ck = min(gk, KC ? kmax - 8 : kmax - 1);
      const uint16_t* p = KC ? base + (size_t)cr * ld + ck : base + (size_t)ck * ld + cr;
      u32x4 v = *reinterpret_cast<const u32x4*>(p);
      regs[i] = ok ? v : u32x4{0u, 0u, 0u, 0u};
    }
  }
}

template <int R, bool KC, int NT>
__device__ __forceinline__ void store_tile_lds(const u32x4* regs, char* lds, int tid) {
  using L = TileLayout<R, KC>;
#pragma unroll
  for (int i = 0; i < L::chunks / NT; i++) {
    int c = tid + i * NT;
    int row = c / L::chunks_per_row, cc = c % L::chunks_per_row;
    int off = KC ? row * L::row_bytes + ((cc ^ ((row >> 1) & 7)) << 4) : row * L::row_bytes + (cc << 4);
    *reinterpret_cast<u32x4*>(lds + off) = regs[i];
  }
}

// One 32(row) x 16(k) MFMA operand fragment out of an LDS tile.  r0: first row of the fragment in the
// tile (multiple of 32); kk: which 16-wide k step of the stage.
template <int R, bool KC>
__device__ __forceinline__ bf16x8 read_frag(const char* lds, int r0, int kk, int lane) {
  using L = TileLayout<R, KC>;
  if (KC) {
    int row = r0 + (lane & 31);
    int chunk = kk * 2 + (lane >> 5);
    const char* p = lds + row * L::row_bytes + ((chunk ^ ((lane >> 1) & 7)) << 4);
    return *reinterpret_cast<const bf16x8*>(p);
  } else {
    int krow = kk * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2);
    int col = r0 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const char* p = lds + krow * L::row_bytes + col * 2;
    short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(p));
    short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((OASES_LDS short4v*)(p + 4 * L::row_bytes));
    typedef short short8v __attribute__((ext_vector_type(8)));
    short8v v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
}

enum { EPI_F32 = 0, EPI_BF16 = 1, EPI_BIAS_BF16 = 2, EPI_BIAS_GELU = 3, EPI_DGELU = 4, EPI_ACC_F32 = 5, EPI_SWIGLU = 6, EPI_DSWIGLU = 7,
       EPI_BF16_DELTA = 8 };  // EPI_BF16, and delta (small-tile kernels of the NT form: launch_gemm_delta)

// silu(z) = z * sigmoid(z) and its derivative, on the fast exp2 / rcp units
__device__ __forceinline__ float fast_sigmoid(float z) { return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z)); }
__device__ __forceinline__ float silu_f(float z) { return z * fast_sigmoid(z); }
__device__ __forceinline__ float silu_grad_f(float z) { const float sg = fast_sigmoid(z); return sg * (1.0f + z * (1.0f - sg)); }

// instruction-group hints for the machine scheduler (kinds: 0x8 MFMA, 0x20 VMEM read, 0x100 LDS read, 0x200 LDS write)
#define SGB(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)

// What the epilogue of four consecutive elements C[row][col .. col+3] reads besides the accumulator: bias (f), the old value
// of C (f), pre-activations (a; SwiGLU gradient: gate a, up b).
struct EpiOperands {
  f32x4 f;
  u32x2 a, b;
};
template <int EPI>
__device__ __forceinline__ EpiOperands epi_load(const GemmArgs& g, int row, int col) {
  EpiOperands o;
  if constexpr (EPI == EPI_BIAS_BF16 || EPI == EPI_BIAS_GELU) o.f = *reinterpret_cast<const f32x4*>(g.bias + col);
  if constexpr (EPI == EPI_ACC_F32) o.f = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.C) + (size_t)row * g.ldc + col);
  if constexpr (EPI == EPI_DGELU || EPI == EPI_BF16_DELTA) o.a = *reinterpret_cast<const u32x2*>(g.aux + (size_t)row * g.ldaux + col);
  if constexpr (EPI == EPI_DSWIGLU) {
    // gate and up pre-activations of 32 columns sit in blocks side by side in aux ([gate 32 | up 32] per block)
    const uint16_t* p = g.aux + (size_t)row * g.ldaux + (size_t)col + (col & ~31);
    o.a = *reinterpret_cast<const u32x2*>(p);
    o.b = *reinterpret_cast<const u32x2*>(p + 32);
  }
  return o;
}
// bf16 results of four columns: out goes to C; also: the second array an epilogue writes (bias+GeLU: pre-activations;
// SwiGLU gradient: out = dgate, also = dup)
template <int EPI>
__device__ __forceinline__ void epi_bf16(f32x4 v, const EpiOperands& o, u32x2& out, u32x2& also) {
  if constexpr (EPI == EPI_DSWIGLU) {
    float dg[4], du[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const float ge = bf16_bits_to_f32((e & 1) ? o.a[e >> 1] >> 16 : o.a[e >> 1] & 0xffffu);
      const float ue = bf16_bits_to_f32((e & 1) ? o.b[e >> 1] >> 16 : o.b[e >> 1] & 0xffffu);
      dg[e] = v[e] * ue * silu_grad_f(ge);
      du[e] = v[e] * silu_f(ge);
    }
    out = u32x2{pack_bf16x2(dg[0], dg[1]), pack_bf16x2(dg[2], dg[3])};
    also = u32x2{pack_bf16x2(du[0], du[1]), pack_bf16x2(du[2], du[3])};
    return;
  }
  if constexpr (EPI == EPI_BIAS_BF16 || EPI == EPI_BIAS_GELU) v += o.f;
  if constexpr (EPI == EPI_BIAS_GELU) {
    also = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = gelu_tanh(v[e]);
  }
  if constexpr (EPI == EPI_DGELU) {
    v[0] *= gelu_tanh_grad(bf16_bits_to_f32(o.a[0] & 0xffffu));
    v[1] *= gelu_tanh_grad(bf16_bits_to_f32(o.a[0] >> 16));
    v[2] *= gelu_tanh_grad(bf16_bits_to_f32(o.a[1] & 0xffffu));
    v[3] *= gelu_tanh_grad(bf16_bits_to_f32(o.a[1] >> 16));
  }
  out = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}
template <int EPI>
__device__ __forceinline__ void epi_apply(const GemmArgs& g, int row, int col, f32x4 v, const EpiOperands& o) {
  const size_t at = (size_t)row * g.ldc + col;
  if constexpr (EPI == EPI_F32 || EPI == EPI_ACC_F32) {
    if constexpr (EPI == EPI_ACC_F32) v = o.f + v;
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + at) = v;
  } else {
    u32x2 out, also;
    epi_bf16<EPI>(v, o, out, also);
    // the gradients of gate and up go to C in the block layout of aux
    uint16_t* cp = reinterpret_cast<uint16_t*>(g.C) + at + (EPI == EPI_DSWIGLU ? (col & ~31) : 0);
    *reinterpret_cast<u32x2*>(cp) = out;
    if constexpr (EPI == EPI_DSWIGLU) *reinterpret_cast<u32x2*>(cp + 32) = also;
    if constexpr (EPI == EPI_BIAS_GELU) *reinterpret_cast<u32x2*>(g.aux + (size_t)row * g.ldaux + col) = also;
  }
}

// Two neighbouring quarters of a tile row (eight columns each, a lane holds columns 0..3, lane + 32 columns 4..7) <-> all
// eight columns of quarter lane / 32 in one lane: bf16 arrays are read and written 16 bytes at a time.  Its own inverse.
// A row of C or aux starts at a multiple of 8 bytes only, hence the type.  (Half the memory instructions; against 8 bytes a
// lane: 8192 x 2048 x 4096 bias+GeLU 128 -> 120 us, dGeLU 147 -> 144, 8192 x 2752 x 4096 SwiGLU 197 -> 186.)
typedef u32x4 u32x4_align8 __attribute__((aligned(8)));
__device__ __forceinline__ void swap_halves(u32x2& x, u32x2& y) {
#pragma unroll
  for (int k = 0; k < 2; k++) {
    const auto r = __builtin_amdgcn_permlane32_swap(x[k], y[k], false, false);
    x[k] = r[0];
    y[k] = r[1];
  }
}
__device__ __forceinline__ void load_quarters(const uint16_t* p, u32x2& x, u32x2& y) {  // still to be swapped
  const u32x4 v = *reinterpret_cast<const u32x4_align8*>(p);
  x = u32x2{v[0], v[1]};
  y = u32x2{v[2], v[3]};
}

// A tile's part of a lane: row lane % 32, quarters q of four columns from 8 q + 4 (lane / 32).  All that the epilogue reads is
// requested before the first store: C may be what aux or the bias is as far as the compiler knows, so it keeps a load behind
// every store written before it, and a tile finished quarter by quarter pays four memory latencies.  Measured in the
// eight-wave kernels, which also run a tile row ahead, 8192 x 2048 x 4096 dGeLU 192 -> 147 us, bias+GeLU 161 -> 128, 2048 x 4096 x
// 8192 accumulating 133 -> 129.  Beyond the edge the operands come from the last row / columns and are not used.
template <int EPI, bool FULL>
__device__ __forceinline__ void epi_request(const GemmArgs& g, int row0, int col0, int lane, EpiOperands (&o)[4]) {
  int row = row0 + (lane & 31);
  if (!FULL) row = min(row, g.M - 1);
  if constexpr (EPI == EPI_DGELU || EPI == EPI_DSWIGLU) {
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      int col = col0 + 8 * (q + (lane >> 5));
      if (!FULL) col = min(col, g.N - 8);
      const uint16_t* p = g.aux + (size_t)row * g.ldaux + col + (EPI == EPI_DSWIGLU ? (col & ~31) : 0);
      load_quarters(p, o[q].a, o[q + 1].a);
      if constexpr (EPI == EPI_DSWIGLU) load_quarters(p + 32, o[q].b, o[q + 1].b);
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < 4; q++) {
    int col = col0 + 8 * q + 4 * (lane >> 5);
    if (!FULL) col = min(col, g.N - 4);
    o[q] = epi_load<EPI>(g, row, col);
  }
}
template <int EPI, bool FULL>
__device__ __forceinline__ void epi_finish(const GemmArgs& g, int row0, int col0, int lane, const f32x16& a, const EpiOperands (&o)[4]) {
  const int row = row0 + (lane & 31);
  if (!FULL && row >= g.M) return;
  if constexpr (EPI != EPI_ACC_F32) {
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      EpiOperands x = o[q], y = o[q + 1];
      if constexpr (EPI == EPI_DGELU || EPI == EPI_DSWIGLU) swap_halves(x.a, y.a);
      if constexpr (EPI == EPI_DSWIGLU) swap_halves(x.b, y.b);
      u32x2 out[2], also[2];
      epi_bf16<EPI>(f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]}, x, out[0], also[0]);
      epi_bf16<EPI>(f32x4{a[4 * q + 4], a[4 * q + 5], a[4 * q + 6], a[4 * q + 7]}, y, out[1], also[1]);
      swap_halves(out[0], out[1]);
      if constexpr (EPI == EPI_DSWIGLU || EPI == EPI_BIAS_GELU) swap_halves(also[0], also[1]);
      const int col = col0 + 8 * (q + (lane >> 5));
      if (!FULL && col >= g.N) continue;
      uint16_t* cp = reinterpret_cast<uint16_t*>(g.C) + (size_t)row * g.ldc + col + (EPI == EPI_DSWIGLU ? (col & ~31) : 0);
      *reinterpret_cast<u32x4_align8*>(cp) = u32x4{out[0][0], out[0][1], out[1][0], out[1][1]};
      if constexpr (EPI == EPI_DSWIGLU) *reinterpret_cast<u32x4_align8*>(cp + 32) = u32x4{also[0][0], also[0][1], also[1][0], also[1][1]};
      if constexpr (EPI == EPI_BIAS_GELU)
        *reinterpret_cast<u32x4_align8*>(g.aux + (size_t)row * g.ldaux + col) = u32x4{also[0][0], also[0][1], also[1][0], also[1][1]};
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int col = col0 + 8 * q + 4 * (lane >> 5);
    if (!FULL && col >= g.N) continue;
    epi_apply<EPI>(g, row, col, f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]}, o[q]);
  }
}

// Epilogue of one 32 x 32 accumulator tile whose first element is C[row0][col0].  Transposed accumulator (every epilogue
// but the plain fp32 store): element e is C[row][col + (e&3)] with row = row0 + (lane & 31), col = col0 + 8 (e>>2) +
// 4 (lane>>5), so a lane owns 4 consecutive columns.
template <int EPI, bool FULL>
__device__ __forceinline__ void epilogue_tile(const GemmArgs& g, int row0, int col0, int lane, const f32x16& a) {
  if constexpr (EPI == EPI_F32) {
    // element e is C[row0 + 8 (e>>2) + 4 (lane>>5) + (e&3)][col], col = lane & 31 of the tile
    const int col = col0 + (lane & 31);
    if (!FULL && col >= g.N) return;
    float* cbase = reinterpret_cast<float*>(g.C) + col;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int row = row0 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      if (!FULL && row >= g.M) continue;
      float* p = cbase + (size_t)row * g.ldc;
      *p = a[e];
    }
    return;
  }
  EpiOperands o[4];
  epi_request<EPI, FULL>(g, row0, col0, lane, o);
  epi_finish<EPI, FULL>(g, row0, col0, lane, a, o);
}

// SwiGLU: two neighbouring accumulator tiles, gate (first column col0 of the interleaved [gate 32 | up 32] layout) and up,
// hold the same 32 columns of f, element for element
template <bool FULL>
__device__ __forceinline__ void epilogue_tile_swiglu(const GemmArgs& g, int row0, int col0, int lane, const f32x16& ag, const f32x16& au) {
  const int row = row0 + (lane & 31);
  if (!FULL && row >= g.M) return;
#pragma unroll
  for (int q = 0; q < 4; q += 2) {
    u32x2 pg[2], pu[2], pf[2];
#pragma unroll
    for (int t = 0; t < 2; t++) {
      float f[4];
      const int b = 4 * (q + t);
#pragma unroll
      for (int e = 0; e < 4; e++) f[e] = silu_f(ag[b + e]) * au[b + e];
      pg[t] = u32x2{pack_bf16x2(ag[b], ag[b + 1]), pack_bf16x2(ag[b + 2], ag[b + 3])};
      pu[t] = u32x2{pack_bf16x2(au[b], au[b + 1]), pack_bf16x2(au[b + 2], au[b + 3])};
      pf[t] = u32x2{pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3])};
    }
    swap_halves(pg[0], pg[1]);
    swap_halves(pu[0], pu[1]);
    swap_halves(pf[0], pf[1]);
    const int c = 8 * (q + (lane >> 5));
    if (!FULL && col0 + c >= g.N) continue;
    uint16_t* ap = g.aux + (size_t)row * g.ldaux + col0 + c;
    *reinterpret_cast<u32x4_align8*>(ap) = u32x4{pg[0][0], pg[0][1], pg[1][0], pg[1][1]};
    *reinterpret_cast<u32x4_align8*>(ap + 32) = u32x4{pu[0][0], pu[0][1], pu[1][0], pu[1][1]};
    *reinterpret_cast<u32x4_align8*>(reinterpret_cast<uint16_t*>(g.C) + (size_t)row * g.ldc + col0 / 2 + c) = u32x4{pf[0][0], pf[0][1], pf[1][0], pf[1][1]};
  }
}

// ---- accumulators of v_mfma_f32_16x16x32_bf16 (the eight-wave and small-tile kernels) -------------------------------------------------
// A lane l holds row l%16, k = 8*(l/16)..+7; B the same with columns.  The B fragment comes first, so that element e of lane l is
// C[l%16][4*(l/16) + e]: a lane owns four consecutive columns.  Two tiles of 16 columns side by side make 32 columns of a row: between them
// v_permlane16_swap turns "columns 4 (l/16)..+3 of either tile" into eight columns of one tile (its own inverse), so that bf16 arrays are read
// and written 16 bytes at a time.
__device__ __forceinline__ void swap_rows16(u32x2& x, u32x2& y) {
#pragma unroll
  for (int k = 0; k < 2; k++) {
    const auto r = __builtin_amdgcn_permlane16_swap(x[k], y[k], false, false);
    x[k] = r[0];
    y[k] = r[1];
  }
}
__device__ __forceinline__ int col16(int lane) { return 16 * ((lane >> 4) & 1) + 8 * (lane >> 5); }  // the lane's eight columns behind the swap
// fp32 outputs (EPI_F32, EPI_ACC_F32): the A fragment first, element e of lane l is C[4*(l/16) + e][l%16]; the same swap between the two tiles makes x the
// rows 8*(l/32) + e, columns l%32, and y the rows 4 further on: half a wave writes and reads whole lines of 128 bytes in the order of its lanes.
constexpr bool epi_rows(int epi) { return epi == EPI_F32 || epi == EPI_ACC_F32; }
__device__ __forceinline__ void swap_lines(f32x4& x, f32x4& y) {
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const float xe = x[e], ye = y[e];
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, xe), __builtin_bit_cast(uint32_t, ye), false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    x[e] = __builtin_bit_cast(float, r0);
    y[e] = __builtin_bit_cast(float, r1);
  }
}
// the 16 rows x 32 columns of C from (row0, col0), in that order of the lanes: address arithmetic in scalar registers.  (Stores that go past the caches
// shorten a launch of few rows, 4096 x 1024 x 1024 17.1 -> 16.0 us, whose L2s have less to write back at its end, but the kernel that reads the result then pays
// for it: steps of h 4096 1767 -> 1795 us, h 2048 forward 309 -> 316, h 12288 with 128 rows 971 -> 983, h 1024 606 -> 601.)
// 32-bit offsets within the 16 rows: leading dimensions up to kLdcOfLines; the forms that check their bounds (FULL false) take any.
constexpr int kLdcOfLines = 32 << 20;
static_assert(15ll * kLdcOfLines * 4 + 32 * 4 <= 0x7fffffff, "offsets of the 16 rows");
struct LinesOfC {
  __amdgpu_buffer_rsrc_t rs;
  int at, pitch;
  __device__ __forceinline__ LinesOfC(const GemmArgs& g, int row0, int col0, int lane)
      : rs(__builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float*>(g.C) + (size_t)row0 * g.ldc + col0, 0, 0x7fffffff, 0x00020000)),
        at((8 * (lane >> 5) * g.ldc + (lane & 31)) * 4), pitch(g.ldc * 4) {}
  template <bool AROUND>
  __device__ __forceinline__ float load(int row) const { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, at, row * pitch, AROUND ? 2 : 0)); }
  template <bool AROUND>
  __device__ __forceinline__ void store(int row, float v) const { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rs, at, row * pitch, AROUND ? 2 : 0); }
};
template <bool AROUND>
__device__ __forceinline__ void store16(uint16_t* p, const u32x2& x, const u32x2& y) {
  const u32x4_align8 v = u32x4{x[0], x[1], y[0], y[1]};
  if constexpr (AROUND) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_align8*>(p));
  else *reinterpret_cast<u32x4_align8*>(p) = v;
}
// requests ahead of the first store, as epi_request: 16 rows x 32 columns from (row0, col0)
// AROUND (eight-wave kernels): a gradient that is added to and the pre-activations that are kept for the backward pass go past the caches, where they would only
// drive out what the next kernels read.  us a step: h 4096 1769 -> 1759, h 8192 2765 -> 2752, llama h 4096 1856 -> 1847.  Not on small tiles (h 12288 with 128 rows 968 -> 979).
template <int EPI, bool FULL, bool AROUND = false>
__device__ __forceinline__ void epi_request16(const GemmArgs& g, int row0, int col0, int lane, EpiOperands (&o)[2]) {
  if constexpr (EPI == EPI_ACC_F32) {
    if constexpr (FULL) {
      const LinesOfC c(g, row0, col0, lane);
#pragma unroll
      for (int t = 0; t < 2; t++)
#pragma unroll
        for (int e = 0; e < 4; e++) o[t].f[e] = c.template load<AROUND>(4 * t + e);
      return;
    }
    const int col = min(col0 + (lane & 31), g.N - 1);
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int row = min(row0 + 8 * (lane >> 5) + 4 * t + e, g.M - 1);
        o[t].f[e] = reinterpret_cast<const float*>(g.C)[(size_t)row * g.ldc + col];
      }
    return;
  }
  int row = row0 + (lane & 15);
  if (!FULL) row = min(row, g.M - 1);
  if constexpr (EPI == EPI_DGELU || EPI == EPI_DSWIGLU) {
    int col = col0 + col16(lane);
    if (!FULL) col = min(col, g.N - 8);
    const uint16_t* p = g.aux + (size_t)row * g.ldaux + col + (EPI == EPI_DSWIGLU ? (col & ~31) : 0);
    load_quarters(p, o[0].a, o[1].a);
    if constexpr (EPI == EPI_DSWIGLU) load_quarters(p + 32, o[0].b, o[1].b);
  } else {
#pragma unroll
    for (int t = 0; t < 2; t++) {
      int col = col0 + 16 * t + 4 * (lane >> 4);
      if (!FULL) col = min(col, g.N - 4);
      o[t] = epi_load<EPI>(g, row, col);
    }
  }
}
template <int EPI, bool FULL, bool AROUND = false>
__device__ __forceinline__ void epi_finish16(const GemmArgs& g, int row0, int col0, int lane, const f32x4& a0, const f32x4& a1, const EpiOperands (&o)[2]) {
  if constexpr (EPI == EPI_F32 || EPI == EPI_ACC_F32) {
    f32x4 v[2] = {a0, a1};
    swap_lines(v[0], v[1]);
    if constexpr (FULL) {
      const LinesOfC c(g, row0, col0, lane);
#pragma unroll
      for (int t = 0; t < 2; t++)
#pragma unroll
        for (int e = 0; e < 4; e++) c.template store<AROUND && EPI == EPI_ACC_F32>(4 * t + e, EPI == EPI_ACC_F32 ? o[t].f[e] + v[t][e] : v[t][e]);
      return;
    }
    const int col = col0 + (lane & 31);
    if (col >= g.N) return;
    float* cp = reinterpret_cast<float*>(g.C) + col;
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int row = row0 + 8 * (lane >> 5) + 4 * t + e;
        if (row >= g.M) continue;
        cp[(size_t)row * g.ldc] = EPI == EPI_ACC_F32 ? o[t].f[e] + v[t][e] : v[t][e];
      }
  } else {
    const int row = row0 + (lane & 15);
    if (!FULL && row >= g.M) return;
    EpiOperands x = o[0], y = o[1];
    if constexpr (EPI == EPI_DGELU || EPI == EPI_DSWIGLU) swap_rows16(x.a, y.a);
    if constexpr (EPI == EPI_DSWIGLU) swap_rows16(x.b, y.b);
    u32x2 out[2], also[2];
    epi_bf16<EPI>(a0, x, out[0], also[0]);
    epi_bf16<EPI>(a1, y, out[1], also[1]);
    swap_rows16(out[0], out[1]);
    if constexpr (EPI == EPI_DSWIGLU || EPI == EPI_BIAS_GELU) swap_rows16(also[0], also[1]);
    const int col = col0 + col16(lane);
    if (!FULL && col >= g.N) return;
    uint16_t* cp = reinterpret_cast<uint16_t*>(g.C) + (size_t)row * g.ldc + col + (EPI == EPI_DSWIGLU ? (col & ~31) : 0);
    *reinterpret_cast<u32x4_align8*>(cp) = u32x4{out[0][0], out[0][1], out[1][0], out[1][1]};
    if constexpr (EPI == EPI_DSWIGLU) *reinterpret_cast<u32x4_align8*>(cp + 32) = u32x4{also[0][0], also[0][1], also[1][0], also[1][1]};
    if constexpr (EPI == EPI_BIAS_GELU) store16<AROUND>(g.aux + (size_t)row * g.ldaux + col, also[0], also[1]);
  }
}
// SwiGLU: gate columns col0 .. col0+31 of the interleaved layout in g0, g1, the up columns behind them in u0, u1
template <bool FULL, bool AROUND = false>
__device__ __forceinline__ void epi_swiglu16(const GemmArgs& g, int row0, int col0, int lane, const f32x4& g0, const f32x4& g1, const f32x4& u0, const f32x4& u1) {
  const int row = row0 + (lane & 15);
  if (!FULL && row >= g.M) return;
  u32x2 pg[2], pu[2], pf[2];
#pragma unroll
  for (int t = 0; t < 2; t++) {
    const f32x4& ag = t ? g1 : g0;
    const f32x4& au = t ? u1 : u0;
    float f[4];
#pragma unroll
    for (int e = 0; e < 4; e++) f[e] = silu_f(ag[e]) * au[e];
    pg[t] = u32x2{pack_bf16x2(ag[0], ag[1]), pack_bf16x2(ag[2], ag[3])};
    pu[t] = u32x2{pack_bf16x2(au[0], au[1]), pack_bf16x2(au[2], au[3])};
    pf[t] = u32x2{pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3])};
  }
  swap_rows16(pg[0], pg[1]);
  swap_rows16(pu[0], pu[1]);
  swap_rows16(pf[0], pf[1]);
  const int c = col16(lane);
  if (!FULL && col0 + c >= g.N) return;
  uint16_t* ap = g.aux + (size_t)row * g.ldaux + col0 + c;
  store16<AROUND>(ap, pg[0], pg[1]);
  store16<AROUND>(ap + 32, pu[0], pu[1]);
  store16<false>(reinterpret_cast<uint16_t*>(g.C) + (size_t)row * g.ldc + col0 / 2 + c, pf[0], pf[1]);
}
// Waves of a workgroup form a WGM x WGN x WGK grid: a wave owns a (BM/WGM) x (BN/WGN) part of the block tile and,
// when WGK > 1, every WGK-th pair of the 16-wide k steps of each stage; the WGK partial accumulators of a part are
// added through LDS after the k loop, in a fixed order.  Splitting k inside the workgroup instead of the tile keeps
// the wave tile at 128 x 128 for the rectangular block tiles, which is what bounds the LDS bytes read per MFMA.
template <int BM, int BN, int WGM, int WGN, int WGK, bool A_KC, bool B_KC, int EPI, bool FULL>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, char* lds, int m0, int n0) {
  constexpr int NT = 64 * WGM * WGN * WGK;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int KS = (BK / 16) / WGK;  // k steps of one stage that a wave multiplies
  static_assert(WGK == 1 || (KS == 2 && TM * TN >= 16), "k split inside the workgroup: two steps per wave, deep pipeline");
  using LA = TileLayout<BM, A_KC>;
  using LB = TileLayout<BN, B_KC>;
  constexpr int NA = LA::chunks / NT, NB = LB::chunks / NT;
  constexpr int kStage = LA::bytes + LB::bytes;  // stage s: A at lds + s*kStage, B behind it
  constexpr int NREAD = TM * (A_KC ? 1 : 2) + TN * (B_KC ? 1 : 2);  // LDS reads of one 16-wide k step
  constexpr int NMFMA = TM * TN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave / (WGM * WGN), wm = (wave / WGN) % WGM, wn = wave % WGN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  u32x4 ra[NA], rb[NB];
  bf16x8 fa[2][TM], fb[2][TN];
  const int nk = (g.K + BK - 1) / BK;

  auto fetch_a = [&](int kt) { load_tile_global<BM, A_KC, NT, FULL>(ra, g.A, g.lda, m0, kt * BK, g.M, g.K, tid); };
  auto fetch_b = [&](int kt) { load_tile_global<BN, B_KC, NT, FULL>(rb, g.B, g.ldb, n0, kt * BK, g.N, g.K, tid); };
  auto park_a = [&](int stage) { store_tile_lds<BM, A_KC, NT>(ra, lds + stage * kStage, tid); };
  auto park_b = [&](int stage) { store_tile_lds<BN, B_KC, NT>(rb, lds + stage * kStage + LA::bytes, tid); };
  auto frags = [&](int stage, int kk, int buf) {
    const char* la = lds + stage * kStage;
    const char* lb = la + LA::bytes;
#pragma unroll
    for (int i = 0; i < TM; i++) fa[buf][i] = read_frag<BM, A_KC>(la, wm * WTM + i * 32, wk * KS + kk, lane);
#pragma unroll
    for (int j = 0; j < TN; j++) fb[buf][j] = read_frag<BN, B_KC>(lb, wn * WTN + j * 32, wk * KS + kk, lane);
  };
  // the B fragment is the first MFMA operand: the accumulator then holds C^T, i.e. a lane owns 4 consecutive
  // columns of one row of C per group of four accumulator elements (16-byte stores in the epilogue)
  // ROWMAJ (plain fp32 output): the A fragment goes first instead and the accumulator holds C itself -- a lane owns
  // one column, 32 lanes one 128-byte row segment, so that every epilogue store writes whole cache lines (measured:
  // up to 18 % on short-k launches whose time is mostly the fp32 output).  Not for the accumulating epilogue, whose
  // read-modify-write wants the 16-byte accesses.
  constexpr bool ROWMAJ = EPI == EPI_F32;
  auto mma = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        if constexpr (ROWMAJ) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][i], fb[buf][j], acc[i][j], 0, 0, 0);
        else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[buf][j], fa[buf][i], acc[i][j], 0, 0, 0);
      }
  };
  // one 16-wide k step: LDS reads of the next step interleaved one-for-one with this step's MFMAs
  auto hint_step = [&]() {
    constexpr int PER = (NREAD + NMFMA - 1) / NMFMA;
#pragma unroll
    for (int i = 0; i < NMFMA; i++) {
      SGB(0x008, 1);
      SGB(0x100, PER);
    }
  };

  if constexpr (TM * TN >= 16) {
    // Pipeline.  While tile kt is multiplied out of stage kt&1, tile kt+1 sits in the other stage.  One operand's half
    // of tile kt+2 is written into stage kt&1 right behind the barrier of iteration kt (which releases that stage),
    // the other's during the first k step of iteration kt+1; each half's registers are refilled from global memory
    // right behind its LDS store, a whole iteration ahead of the next store.  LDS stores and global loads are thus
    // spread over two k steps and never wait at the top of the loop.
    // "early" half: stored during the first k step, "late" half: stored behind the barrier, where it competes with the
    // first fragment reads of the next stage -- the smaller operand tile goes there.
    constexpr bool LATE_A = BM <= BN;
    constexpr int N_EARLY = LATE_A ? NB : NA, N_LATE = LATE_A ? NA : NB;
    auto fetch_early = [&](int kt) { if constexpr (LATE_A) fetch_b(kt); else fetch_a(kt); };
    auto fetch_late = [&](int kt) { if constexpr (LATE_A) fetch_a(kt); else fetch_b(kt); };
    auto park_early = [&](int stage) { if constexpr (LATE_A) park_b(stage); else park_a(stage); };
    auto park_late = [&](int stage) { if constexpr (LATE_A) park_a(stage); else park_b(stage); };
    fetch_a(0);
    fetch_b(0);
    park_a(0);
    park_b(0);
    if (nk > 1) { fetch_late(1); park_late(1); fetch_early(1); }
    if (nk > 2) fetch_late(2);
    __syncthreads();
    frags(0, 0, 0);

    // one 64-wide k iteration; M1/M2/M3: tile kt+1 / kt+2 / kt+3 exists.  The steady state (all true) is branch-free
    // so that the scheduler sees one block per iteration.
    auto iteration = [&](auto m1_c, auto m2_c, auto m3_c, int kt) {
      constexpr bool M1 = decltype(m1_c)::value, M2 = decltype(m2_c)::value, M3 = decltype(m3_c)::value;
      const int cur = kt & 1;
      if (M1) park_early(cur ^ 1);  // early half of tile kt+1 (the stage was released by the previous barrier)
      if (M2) fetch_early(kt + 2);
      frags(cur, 1, 1);
      mma(0);
  #pragma unroll
      for (int i = 0; i < NMFMA; i++) {
        SGB(0x008, 1);
        SGB(0x100, (NREAD + NMFMA - 1) / NMFMA);
        if (M1) SGB(0x200, (N_EARLY + NMFMA - 1) / NMFMA);
        if (M2) SGB(0x020, (N_EARLY + NMFMA - 1) / NMFMA);
      }
      if (KS == 4) {
        frags(cur, 2, 0);
        mma(1);
        hint_step();
        frags(cur, 3, 1);
        mma(0);
        hint_step();
      }
      // every wave has its last fragments of stage `cur` in registers, and stage cur^1 (tile kt+1) is complete
      __syncthreads();
      if (M1) frags(cur ^ 1, 0, 0);
      if (M2) park_late(cur);       // late half of tile kt+2 -> the stage just released
      if (M3) fetch_late(kt + 3);
      mma(1);
  #pragma unroll
      for (int i = 0; i < NMFMA; i++) {
        SGB(0x008, 1);
        if (M1) SGB(0x100, (NREAD + NMFMA - 1) / NMFMA);
        if (M2) SGB(0x200, (N_LATE + NMFMA - 1) / NMFMA);
        if (M3) SGB(0x020, (N_LATE + NMFMA - 1) / NMFMA);
      }
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    int kt = 0;
    for (; kt + 3 < nk; kt++) iteration(T_{}, T_{}, T_{}, kt);
    if (kt + 2 < nk) { iteration(T_{}, T_{}, F_{}, kt); kt++; }
    if (kt + 1 < nk) { iteration(T_{}, F_{}, F_{}, kt); kt++; }
    iteration(F_{}, F_{}, F_{}, kt);
  } else {
    // Pipeline for the smaller tiles (their LDS traffic per MFMA is higher; a single burst of LDS stores at the top of
    // the iteration disturbs the fragment reads least): tile kt+1 waits in registers, is stored into the other stage
    // at the top of iteration kt, and the registers are refilled with tile kt+2 right behind.
    fetch_a(0);
    fetch_b(0);
    park_a(0);
    park_b(0);
    if (nk > 1) { fetch_a(1); fetch_b(1); }
    __syncthreads();
    frags(0, 0, 0);
    auto iteration = [&](auto m1_c, auto m2_c, int kt) {
      constexpr bool M1 = decltype(m1_c)::value, M2 = decltype(m2_c)::value;
      const int cur = kt & 1;
      if (M1) { park_a(cur ^ 1); park_b(cur ^ 1); }
      if (M2) { fetch_a(kt + 2); fetch_b(kt + 2); }
      frags(cur, 1, 1);
      mma(0);
      if (M1) SGB(0x200, NA + NB);
  #pragma unroll
      for (int i = 0; i < NMFMA; i++) {
        SGB(0x008, 1);
        if (M2) SGB(0x020, (NA + NB + NMFMA - 1) / NMFMA);
        SGB(0x100, (NREAD + NMFMA - 1) / NMFMA);
      }
      frags(cur, 2, 0);
      mma(1);
      hint_step();
      frags(cur, 3, 1);
      mma(0);
      hint_step();
      __syncthreads();
      if (M1) frags(cur ^ 1, 0, 0);
      mma(1);
      hint_step();
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    int kt = 0;
    for (; kt + 2 < nk; kt++) iteration(T_{}, T_{}, kt);
    if (kt + 1 < nk) { iteration(T_{}, F_{}, kt); kt++; }
    iteration(F_{}, F_{}, kt);
  }

  auto emit = [&](int i, int j, const f32x16& a) { epilogue_tile<EPI, FULL>(g, m0 + wm * WTM + i * 32, n0 + wn * WTN + j * 32, lane, a); };
  auto emit_pair = [&](int i, int jj, const f32x16& ag, const f32x16& au) {
    epilogue_tile_swiglu<FULL>(g, m0 + wm * WTM + i * 32, n0 + wn * WTN + jj * 64, lane, ag, au);
  };

  static_assert(TN % 2 == 0, "tiles of a wave are finished in pairs");
  if constexpr (WGK == 1) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j += 2) {
        if constexpr (EPI == EPI_SWIGLU) {
          emit_pair(i, j / 2, acc[i][j], acc[i][j + 1]);
        } else {
          emit(i, j, acc[i][j]);
          emit(i, j + 1, acc[i][j + 1]);
        }
      }
  } else {
    // The two waves that hold the k halves of one part each finish one half of its rows: a wave hands the
    // accumulator tiles of the other half over through LDS (lane-for-lane, 16 bytes per lane and store) and adds what
    // it receives to its own; the sum of two terms does not depend on which of them is "own".
    static_assert(WGK == 2 && TM % 2 == 0, "pairwise exchange");
    constexpr int HM = TM / 2;
    f32x4* xch = reinterpret_cast<f32x4*>(lds);
    const int mine = wave * (HM * TN * 4), theirs = (wave ^ (WGM * WGN)) * (HM * TN * 4);
    __syncthreads();  // every wave is done with the operand stages
    auto hand_over = [&](auto half_c) {  // half_c: which half of the tile rows leaves this wave
      constexpr int H = decltype(half_c)::value;
#pragma unroll
      for (int i = 0; i < HM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const f32x16& a = acc[H * HM + i][j];
            xch[(mine + (i * TN + j) * 4 + q) * 64 + lane] = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
          }
    };
    auto finish = [&](auto half_c) {  // half_c: which half of the tile rows this wave keeps
      constexpr int H = decltype(half_c)::value;
#pragma unroll
      for (int i = 0; i < HM; i++)
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
          f32x16 a[2] = {acc[H * HM + i][j], acc[H * HM + i][j + 1]};
#pragma unroll
          for (int t = 0; t < 2; t++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
              const f32x4 o = xch[(theirs + (i * TN + j + t) * 4 + q) * 64 + lane];
#pragma unroll
              for (int e = 0; e < 4; e++) a[t][4 * q + e] += o[e];
            }
          if constexpr (EPI == EPI_SWIGLU) {
            emit_pair(H * HM + i, j / 2, a[0], a[1]);
          } else {
            emit(H * HM + i, j, a[0]);
            emit(H * HM + i, j + 1, a[1]);
          }
        }
    };
    if (wk == 0) hand_over(std::integral_constant<int, 1>{}); else hand_over(std::integral_constant<int, 0>{});
    __syncthreads();
    if (wk == 0) finish(std::integral_constant<int, 0>{}); else finish(std::integral_constant<int, 1>{});
  }
}

// workgroup id within a launch of tiles_m x tiles_n tiles -> tile: undo the round-robin of workgroup ids over the 8 XCDs so
// that each XCD's L2 sees a contiguous range of tiles, then walk that range in groups of 8 tile rows
__device__ __forceinline__ void tile_of_workgroup(int pid, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
  const int T = tiles_m * tiles_n;
  const int per = (T + 7) / 8, tall = (T % 8 == 0) ? 8 : T % 8;
  const int xcd = pid & 7, local = pid >> 3;
  const int logical = xcd < tall ? xcd * per + local : tall * per + (xcd - tall) * (per - 1) + local;
  constexpr int GM = 8;
  const int width = GM * tiles_n;
  const int group = logical / width, first_m = group * GM;
  const int gsz = min(tiles_m - first_m, GM);
  tile_m = first_m + (logical % width) % gsz;
  tile_n = (logical % width) / gsz;
}

template <int BM, int BN, int WGM, int WGN, int WGK, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(64 * WGM * WGN * WGK) void gemm_kernel(GemmArgs g) {  // g: by value, adjusted per k slice
  using LA = TileLayout<BM, A_KC>;
  using LB = TileLayout<BN, B_KC>;
  constexpr int kStages = 2 * (LA::bytes + LB::bytes);
  constexpr int kExchange = WGK > 1 ? BM * BN * 4 : 0;  // half of every wave's accumulator
  __shared__ __attribute__((aligned(16))) char lds[kStages > kExchange ? kStages : kExchange];

  // workgroup -> (k slice, tile)
  int tile_m, tile_n;
  const int T = g.tiles_m * g.tiles_n;
  const int slice = blockIdx.x / T;
  tile_of_workgroup(blockIdx.x - slice * T, g.tiles_m, g.tiles_n, tile_m, tile_n);
  if (g.ksplit > 1) {  // this workgroup's k range and partial-result plane
    const int k0 = slice * g.k_per;
    g.A += A_KC ? (size_t)k0 : (size_t)k0 * g.lda;
    g.B += B_KC ? (size_t)k0 : (size_t)k0 * g.ldb;
    g.K = min(g.K - k0, g.k_per);
    g.C = reinterpret_cast<float*>(g.C) + (size_t)slice * g.M * g.ldc;
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const bool full = (m0 + BM <= g.M) && (n0 + BN <= g.N) && (g.K % BK == 0);
  if (full) gemm_tile<BM, BN, WGM, WGN, WGK, A_KC, B_KC, EPI, true>(g, lds, m0, n0);
  else gemm_tile<BM, BN, WGM, WGN, WGK, A_KC, B_KC, EPI, false>(g, lds, m0, n0);
}

// =================================================================================================
// 256 x 256 tiles fed by direct-to-LDS loads (global_load_lds_dwordx4): no staging registers, four LDS stages of 32 k,
// three tiles (96 KB per CU) in flight.  The compiler would put s_waitcnt vmcnt(0) in front of every LDS read that
// might alias a pending LDS DMA, so the fragment reads are inline assembly and every wait is placed by hand:
//   vmcnt  -- DMA instructions complete in order, 8 per wave and tile: "tile t has landed" = at most 8 x (younger tiles
//             in flight) outstanding, then the workgroup barrier makes all four waves' parts visible;
//   lgkmcnt -- LDS reads return in order: fragments of the first k step are waited for with the second step's reads
//             still outstanding; the second step's are waited for before the barrier, so that a stage is never
//             refilled while a wave still reads it.
// K must be a whole number of 32-wide stages and there are no k slices; M and N may end inside a tile where the operand
// is row-indexed (see dtl_src); everything else runs on the kernels above.
// =================================================================================================
#ifndef OASES_DTL_STAGES
#define OASES_DTL_STAGES 4
#endif
constexpr int BKD = 32, NSD = OASES_DTL_STAGES;
constexpr int kDtlOperand = 256 * BKD * 2;  // bytes of one operand tile
constexpr int kDtlStage = 2 * kDtlOperand;

template <int OFF>
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
template <int OFF>
__device__ __forceinline__ u32x2 lds_read_tr16_b64(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
// the eight fragments of one k step become valid: at most N younger LDS reads may still be outstanding
template <int N>
__device__ __forceinline__ void lds_wait(u32x4 (&a)[4], u32x4 (&b)[4]) {
  asm volatile("s_waitcnt lgkmcnt(%8)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3])
               : "n"(N));
}

// Operand tile in LDS.  KC (k contiguous in memory): [256 rows][32 k] = 64-byte rows, 16-byte chunk c of row r at slot
// c ^ ((r/4)%4) (16 consecutive rows at one chunk then cover all 64 banks).  MC (row index contiguous in memory):
// [32 k][256 rows] = 512-byte k rows, chunk c of k row kr at slot c ^ 4*(kr%4) (the 4 k rows x 64 bytes that 32 lanes of
// a transpose read touch in one LDS cycle then fall on 16 different chunk positions mod 16).  One DMA instruction of a wave writes 1 KB
// of the tile, lane i the 16 bytes at i*16: the swizzle is applied to the global address the lane fetches.
// `extent`: rows of the operand's free dimension (M of A, N of B).  A row-indexed operand may end inside the tile
// (extent a multiple of 8, so whole 16-byte chunks): chunks beyond it are fetched from column 0 instead -- valid memory,
// and the rows / columns of C they feed are never stored.  A k-major operand must fill its tiles.
//
// The eight-wave kernels fetch the tiles with buffer loads (resource in SGPRs + 32-bit lane offset + SGPR tile offset)
// straight into LDS: no address arithmetic in the vector ALU and half the address registers; measured 5-10 % faster
// there than global_load_lds with 64-bit lane addresses (TN 2048 x 4096 x 8192: 1029 -> 1120 TFLOP/s, 4096 x 4096 x
// 8192: 1111 -> 1228).  An operand must span less than 2 GiB (gemm_span_fits, checked by the launcher).
typedef void OASES_LDS* lds_ptr_t;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ uint32_t lane_offset(const char* p, const void* base) { return (uint32_t)(p - reinterpret_cast<const char*>(base)); }
// 16 bytes per lane: lane i's go to dst + 16 i (dst is uniform over the wave)
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t tile_off, char* dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)dst, 16, (int)lane_off, (int)tile_off, 0, 0);
}

// the same through global_load_lds (64-bit lane address): what the four-wave kernels use -- they issue a tile's loads between
// MFMAs of the same wave, where the buffer form measured 5-10 % slower
__device__ __forceinline__ void dma16_global(const void* base, uint32_t lane_off, uint32_t tile_off, char* dst) {
  typedef const void __attribute__((address_space(1))) * gptr_t;
  __builtin_amdgcn_global_load_lds((gptr_t)(reinterpret_cast<const char*>(base) + lane_off + (size_t)tile_off), (lds_ptr_t)dst, 16, 0, 0);
}

template <bool KC>
__device__ __forceinline__ const char* dtl_src(const uint16_t* base, int ld, int r0, int q, int lane, int extent) {
  if (KC) {
    const int row = 16 * q + (lane >> 2), chunk = (lane & 3) ^ ((row >> 2) & 3);
    return reinterpret_cast<const char*>(base + (size_t)(r0 + row) * ld + chunk * 8);
  }
  const int kr = 2 * q + (lane >> 5), cc = (lane & 31) ^ (4 * (kr & 3));
  int col = r0 + cc * 8;
  if (col >= extent) col = 0;
  return reinterpret_cast<const char*>(base + (size_t)kr * ld + col);
}
// per-lane LDS offsets of the fragment reads of a wave's 128-row part starting at tile row R0
template <bool KC>
__device__ __forceinline__ void dtl_frag_offsets(uint32_t* off, int R0, int lane) {
  if (KC) {  // off[kk]: fragment i adds 32 rows = 2048 bytes
#pragma unroll
    for (int kk = 0; kk < 2; kk++) {
      const int row = R0 + (lane & 31), chunk = kk * 2 + (lane >> 5);
      off[kk] = (uint32_t)(row * 64 + 16 * (chunk ^ ((row >> 2) & 3)));
    }
  } else {  // off[i]: k step kk adds 16 k rows = 8192 bytes, the second half of the fragment 4 k rows = 2048 bytes
    const int krow = 8 * (lane >> 5) + ((lane & 15) >> 2);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int col = R0 + 32 * i + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      off[i] = (uint32_t)(krow * 512 + (((col >> 3) ^ (4 * (krow & 3))) << 4) + (col & 7) * 2);
    }
  }
}
template <bool KC, int KK>
__device__ __forceinline__ void dtl_read_frags(u32x4 (&f)[4], uint32_t base, const uint32_t* off) {
  if constexpr (KC) {
    const uint32_t a = base + off[KK];
    f[0] = lds_read_b128<0>(a);
    f[1] = lds_read_b128<2048>(a);
    f[2] = lds_read_b128<4096>(a);
    f[3] = lds_read_b128<6144>(a);
  } else {
#define OASES_TR(i)                                                         \
  {                                                                         \
    const u32x2 lo = lds_read_tr16_b64<KK * 8192>(base + off[i]);           \
    const u32x2 hi = lds_read_tr16_b64<KK * 8192 + 2048>(base + off[i]);    \
    f[i] = u32x4{lo[0], lo[1], hi[0], hi[1]};                               \
  }
    OASES_TR(0) OASES_TR(1) OASES_TR(2) OASES_TR(3)
#undef OASES_TR
  }
}

template <bool A_KC, bool B_KC, int EPI, bool FULL>
__global__ __launch_bounds__(256) void gemm_dtl_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) char lds[NSD * kDtlStage];
  int tile_m, tile_n;
  tile_of_workgroup(blockIdx.x, g.tiles_m, g.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * 256, n0 = tile_n * 256;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  constexpr int WGM = 2, WGN = 2, WTM = 128, WTN = 128, TM = 4, TN = 4;
  const int nk = g.K / BKD;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  // DMA sources of this lane: instruction j of this wave is instruction q = 4*wave + j of the operand tile
  // (the swizzle of an MC tile depends on the parity of q: one source pointer for even, one for odd instructions)
  const uint32_t srcA[2] = {lane_offset(dtl_src<A_KC>(g.A, g.lda, m0, 4 * wave, lane, g.M), g.A), lane_offset(dtl_src<A_KC>(g.A, g.lda, m0, 4 * wave + 1, lane, g.M), g.A)};
  const uint32_t srcB[2] = {lane_offset(dtl_src<B_KC>(g.B, g.ldb, n0, 4 * wave, lane, g.N), g.B), lane_offset(dtl_src<B_KC>(g.B, g.ldb, n0, 4 * wave + 1, lane, g.N), g.B)};
  const uint32_t stepA_q = A_KC ? 32u * g.lda * 2 : 4u * g.lda * 2;   // two instructions on: 32 rows resp. 4 k rows
  const uint32_t stepB_q = B_KC ? 32u * g.ldb * 2 : 4u * g.ldb * 2;
  const uint32_t stepA_k = A_KC ? (uint32_t)BKD * 2 : (uint32_t)BKD * g.lda * 2;          // next k tile
  const uint32_t stepB_k = B_KC ? (uint32_t)BKD * 2 : (uint32_t)BKD * g.ldb * 2;
  auto issue = [&](int t) {
    char* st = lds + (t % NSD) * kDtlStage + wave * 4096;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      dma16_global(g.A, srcA[j & 1], (uint32_t)t * stepA_k + (j >> 1) * stepA_q, st + j * 1024);
      dma16_global(g.B, srcB[j & 1], (uint32_t)t * stepB_k + (j >> 1) * stepB_q, st + kDtlOperand + j * 1024);
    }
  };

  uint32_t offA[4], offB[4];
  dtl_frag_offsets<A_KC>(offA, wm * WTM, lane);
  dtl_frag_offsets<B_KC>(offB, wn * WTN, lane);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(OASES_LDS char*)lds;
  u32x4 fa[2][4], fb[2][4];
  constexpr int NRA = A_KC ? 4 : 8, NRB = B_KC ? 4 : 8, NR = NRA + NRB > 15 ? 15 : NRA + NRB;  // reads of one k step (lgkmcnt saturates at 15)
  auto mma = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, fa[buf][i]), b = __builtin_bit_cast(bf16x8, fb[buf][j]);
        if constexpr (EPI == EPI_F32) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i][j], 0, 0, 0);
        else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc[i][j], 0, 0, 0);
      }
  };
  // s_waitcnt vmcnt(n) only.  Steady state: NSD-2 younger tiles of 8 DMA instructions each may still be in flight
  constexpr int kYoung = 8 * (NSD - 2);
  constexpr int kVm16 = ((kYoung >> 4) << 14) | (kYoung & 15) | (7 << 4) | (15 << 8), kVm0 = (7 << 4) | (15 << 8);

#pragma unroll
  for (int t = 0; t < NSD - 1; t++)
    if (t < nk) issue(t);
  if (nk > NSD - 2) __builtin_amdgcn_s_waitcnt(kVm16); else __builtin_amdgcn_s_waitcnt(kVm0);
  __builtin_amdgcn_s_barrier();
  dtl_read_frags<A_KC, 0>(fa[0], lds0, offA);
  dtl_read_frags<B_KC, 0>(fb[0], lds0 + kDtlOperand, offB);

  // one 32-wide k tile.  STEADY: tile kt+NSD-1 exists and is requested now (its stage held tile kt-1; a wave passes the
  // barrier of an iteration only after all its reads of that iteration's tile have returned), so NSD-2 younger tiles
  // are in flight when tile kt+1 must have landed; NEXT: tile kt+1 exists.
  uint32_t cur = lds0;
  auto iteration = [&](auto steady_c, auto next_c, int kt) {
    constexpr bool STEADY = decltype(steady_c)::value, NEXT = decltype(next_c)::value;
    const uint32_t nxt = cur + kDtlStage == lds0 + NSD * kDtlStage ? lds0 : cur + kDtlStage;
    dtl_read_frags<A_KC, 1>(fa[1], cur, offA);
    dtl_read_frags<B_KC, 1>(fb[1], cur + kDtlOperand, offB);
    lds_wait<NR>(fa[0], fb[0]);
    if (STEADY) issue(kt + NSD - 1);
    mma(0);
    lds_wait<0>(fa[1], fb[1]);  // requested before the MFMAs above; with it every read this wave makes of tile kt is complete
    if (NEXT) {
      if (STEADY) __builtin_amdgcn_s_waitcnt(kVm16); else __builtin_amdgcn_s_waitcnt(kVm0);  // own part of tile kt+1 has landed
      __builtin_amdgcn_s_barrier();  // tile kt+1 is visible to every wave, and no wave reads tile kt any more
      dtl_read_frags<A_KC, 0>(fa[0], nxt, offA);
      dtl_read_frags<B_KC, 0>(fb[0], nxt + kDtlOperand, offB);
    }
    mma(1);
    cur = nxt;
  };
  {
    using T_ = std::true_type;
    using F_ = std::false_type;
    int kt = 0;
    for (; kt + NSD - 1 < nk; kt++) iteration(T_{}, T_{}, kt);
    for (; kt + 1 < nk; kt++) iteration(F_{}, T_{}, kt);
    iteration(F_{}, F_{}, kt);
  }
  auto emit = [&](int i, int j, const f32x16& a) { epilogue_tile<EPI, FULL>(g, m0 + wm * WTM + i * 32, n0 + wn * WTN + j * 32, lane, a); };
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j += 2) {
      if constexpr (EPI == EPI_SWIGLU) {  // tiles j (gate) and j+1 (up) of the interleaved 64-column blocks
        epilogue_tile_swiglu<FULL>(g, m0 + wm * WTM + i * 32, n0 + wn * WTN + j * 32, lane, acc[i][j], acc[i][j + 1]);
      } else {
        emit(i, j, acc[i][j]);
        emit(i, j + 1, acc[i][j + 1]);
      }
    }
}

// =================================================================================================
// 128 x 256 tiles fed by direct-to-LDS loads.  Three LDS stages of 64 k (48 KB each); the two wave pairs split the four
// 16-wide k steps of a stage between them, so a wave keeps the 128 x 128 accumulator of the square kernel (same LDS
// bytes read per MFMA) while the launch has twice as many workgroups; the two partial sums of a part meet once,
// through LDS, after the k loop.  Waits as in the kernel above; a wave issues 12 DMA instructions per tile (4 of A,
// 8 of B).  K % 64 == 0; M and N may end inside a tile (see rect_src).
// Operand tile in LDS.  KC: [R rows][64 k] = 128-byte rows, chunk c of row r at slot c ^ ((r/2)%8) (16 consecutive
// rows at one chunk cover all 64 banks); one DMA instruction covers 8 rows.  MC: [64 k][R rows], k row = 2R bytes,
// chunk c of k row kr at slot c ^ 4*(kr%4); one DMA instruction covers 512/R k rows.  In both the swizzle of
// instruction q depends on the parity of q only.
// =================================================================================================
constexpr int BKR = 64, NSR = 3;
constexpr int kRectA = BKR * 128 * 2, kRectB = BKR * 256 * 2, kRectStage = kRectA + kRectB;

template <bool KC, int R>
__device__ __forceinline__ const char* rect_src(const uint16_t* base, int ld, int r0, int q, int lane, int extent) {
  if (KC) {  // rows beyond the operand's extent: the last row again (valid memory; what they feed is never stored)
    const int row = 8 * q + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    return reinterpret_cast<const char*>(base + (size_t)min(r0 + row, extent - 1) * ld + chunk * 8);
  }
  constexpr int CPR = R / 8, KPI = 64 / CPR;
  const int kr = KPI * q + lane / CPR, cc = (lane % CPR) ^ (4 * (kr & 3));
  int col = r0 + cc * 8;
  if (col >= extent) col = 0;  // beyond a row-indexed operand's extent: see dtl_src
  return reinterpret_cast<const char*>(base + (size_t)kr * ld + col);
}
// per-lane LDS offsets of the fragment reads of a wave's 128-row part starting at tile row R0, for the k half wk of a
// tile.  KC: off[kk], k step kk of the half (fragment i adds 32 rows = 4096 bytes); MC: off[i], fragment i (k step kk
// adds 16 k rows, the second half of a fragment 4 k rows).
template <bool KC, int R>
__device__ __forceinline__ void rect_frag_offsets(uint32_t* off, int R0, int wk, int lane) {
  if (KC) {
#pragma unroll
    for (int kk = 0; kk < 2; kk++) {
      const int row = R0 + (lane & 31), chunk = 4 * wk + 2 * kk + (lane >> 5);
      off[kk] = (uint32_t)(row * 128 + 16 * (chunk ^ ((row >> 1) & 7)));
    }
  } else {
    const int krow = 32 * wk + 8 * (lane >> 5) + ((lane & 15) >> 2);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int col = R0 + 32 * i + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      off[i] = (uint32_t)(krow * (2 * R) + (((col >> 3) ^ (4 * (krow & 3))) << 4) + (col & 7) * 2);
    }
  }
}
template <bool KC, int R, int KK>
__device__ __forceinline__ void rect_read_frags(u32x4 (&f)[4], uint32_t base, const uint32_t* off) {
  if constexpr (KC) {
    const uint32_t a = base + off[KK];
    f[0] = lds_read_b128<0>(a);
    f[1] = lds_read_b128<4096>(a);
    f[2] = lds_read_b128<8192>(a);
    f[3] = lds_read_b128<12288>(a);
  } else {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const u32x2 lo = lds_read_tr16_b64<KK * 16 * 2 * R>(base + off[i]);
      const u32x2 hi = lds_read_tr16_b64<KK * 16 * 2 * R + 4 * 2 * R>(base + off[i]);
      f[i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
  }
}

constexpr int kRectExchange = 128 * 256 * 4;
constexpr int kRectLds = NSR * kRectStage > kRectExchange ? NSR * kRectStage : kRectExchange;

// one 128 x 256 tile: workgroup `pid` of the tiles_m x tiles_n tiles of problem g; lds: kRectLds bytes, 1024-byte aligned
template <bool A_KC, bool B_KC, int EPI, bool FULL>
__device__ __forceinline__ void dtl_rect_tile(const GemmArgs& g, int pid, char* lds) {
  int tile_m, tile_n;
  tile_of_workgroup(pid, g.tiles_m, g.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * 128, n0 = tile_n * 256;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave & 1, wk = wave >> 1;
  constexpr int TM = 4, TN = 4;
  const int nk = g.K / BKR;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  // this wave's DMA instructions of a tile: A instructions 4*wave .. 4*wave+3, B instructions 8*wave .. 8*wave+7, one
  // source pointer each (rows or chunks beyond an operand's extent are redirected per instruction)
  uint32_t srcA[4], srcB[8];
#pragma unroll
  for (int j = 0; j < 4; j++) srcA[j] = lane_offset(rect_src<A_KC, 128>(g.A, g.lda, m0, 4 * wave + j, lane, g.M), g.A);
#pragma unroll
  for (int j = 0; j < 8; j++) srcB[j] = lane_offset(rect_src<B_KC, 256>(g.B, g.ldb, n0, 8 * wave + j, lane, g.N), g.B);
  const uint32_t stepA_k = A_KC ? (uint32_t)BKR * 2 : (uint32_t)BKR * g.lda * 2, stepB_k = B_KC ? (uint32_t)BKR * 2 : (uint32_t)BKR * g.ldb * 2;  // next k tile
  auto issue = [&](int t) {
    char* st = lds + (t % NSR) * kRectStage;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      dma16_global(g.A, srcA[j], (uint32_t)t * stepA_k, st + (4 * wave + j) * 1024);
      dma16_global(g.B, srcB[2 * j], (uint32_t)t * stepB_k, st + kRectA + (8 * wave + 2 * j) * 1024);
      dma16_global(g.B, srcB[2 * j + 1], (uint32_t)t * stepB_k, st + kRectA + (8 * wave + 2 * j + 1) * 1024);
    }
  };

  uint32_t offA[4], offB[4];
  rect_frag_offsets<A_KC, 128>(offA, 0, wk, lane);
  rect_frag_offsets<B_KC, 256>(offB, wn * 128, wk, lane);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(OASES_LDS char*)lds;
  u32x4 fa[2][4], fb[2][4];
  auto mma = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, fa[buf][i]), b = __builtin_bit_cast(bf16x8, fb[buf][j]);
        if constexpr (EPI == EPI_F32) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i][j], 0, 0, 0);
        else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc[i][j], 0, 0, 0);
      }
  };
  constexpr int kYoung = 12 * (NSR - 2);  // DMA instructions of the younger tiles that may still be in flight
  constexpr int kVmSteady = ((kYoung >> 4) << 14) | (kYoung & 15) | (7 << 4) | (15 << 8), kVm0 = (7 << 4) | (15 << 8);
  constexpr int NRA = A_KC ? 4 : 8, NRB = B_KC ? 4 : 8, NR = NRA + NRB > 15 ? 15 : NRA + NRB;  // reads of one k step (the counter saturates at 15)

#pragma unroll
  for (int t = 0; t < NSR - 1; t++)
    if (t < nk) issue(t);
  if (nk > NSR - 2) __builtin_amdgcn_s_waitcnt(kVmSteady); else __builtin_amdgcn_s_waitcnt(kVm0);
  __builtin_amdgcn_s_barrier();
  rect_read_frags<A_KC, 128, 0>(fa[0], lds0, offA);
  rect_read_frags<B_KC, 256, 0>(fb[0], lds0 + kRectA, offB);

  uint32_t cur = lds0;
  auto iteration = [&](auto steady_c, auto next_c, int kt) {
    constexpr bool STEADY = decltype(steady_c)::value, NEXT = decltype(next_c)::value;
    const uint32_t nxt = cur + kRectStage == lds0 + NSR * kRectStage ? lds0 : cur + kRectStage;
    rect_read_frags<A_KC, 128, 1>(fa[1], cur, offA);
    rect_read_frags<B_KC, 256, 1>(fb[1], cur + kRectA, offB);
    lds_wait<NR>(fa[0], fb[0]);
    if (STEADY) issue(kt + NSR - 1);  // into the stage of tile kt-1: its reads had returned before any wave passed the last barrier
    mma(0);
    lds_wait<0>(fa[1], fb[1]);  // requested before the MFMAs above; with it every read this wave makes of tile kt is complete
    if (NEXT) {
      if (STEADY) __builtin_amdgcn_s_waitcnt(kVmSteady); else __builtin_amdgcn_s_waitcnt(kVm0);  // own part of tile kt+1 has landed
      __builtin_amdgcn_s_barrier();  // tile kt+1 is visible to every wave, and no wave reads tile kt any more
      rect_read_frags<A_KC, 128, 0>(fa[0], nxt, offA);
      rect_read_frags<B_KC, 256, 0>(fb[0], nxt + kRectA, offB);
    }
    mma(1);
    cur = nxt;
  };
  {
    using T_ = std::true_type;
    using F_ = std::false_type;
    int kt = 0;
    for (; kt + NSR - 1 < nk; kt++) iteration(T_{}, T_{}, kt);
    for (; kt + 1 < nk; kt++) iteration(F_{}, T_{}, kt);
    iteration(F_{}, F_{}, kt);
  }

  // The two waves that hold the k halves of one 128 x 128 part each finish 64 of its rows: a wave hands the accumulator
  // tiles of the other 64 rows over through LDS (lane for lane) and adds what it receives to its own.
  constexpr int HM = TM / 2;
  f32x4* xch = reinterpret_cast<f32x4*>(lds);
  const int mine = wave * (HM * TN * 4), theirs = (wave ^ 2) * (HM * TN * 4);
  __syncthreads();  // every wave is done with the operand stages (all DMA has landed: the last tile was waited for)
  auto hand_over = [&](auto half_c) {
    constexpr int H = decltype(half_c)::value;
#pragma unroll
    for (int i = 0; i < HM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const f32x16& a = acc[H * HM + i][j];
          xch[(mine + (i * TN + j) * 4 + q) * 64 + lane] = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
        }
  };
  auto finish = [&](auto half_c) {
    constexpr int H = decltype(half_c)::value;
#pragma unroll
    for (int i = 0; i < HM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        f32x16 a = acc[H * HM + i][j];
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const f32x4 o = xch[(theirs + (i * TN + j) * 4 + q) * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; e++) a[4 * q + e] += o[e];
        }
        epilogue_tile<EPI, FULL>(g, m0 + (H * HM + i) * 32, n0 + wn * 128 + j * 32, lane, a);
      }
  };
  if (wk == 0) hand_over(std::integral_constant<int, 1>{}); else hand_over(std::integral_constant<int, 0>{});
  __syncthreads();
  if (wk == 0) finish(std::integral_constant<int, 0>{}); else finish(std::integral_constant<int, 1>{});
}

template <bool A_KC, bool B_KC, int EPI, bool FULL>
__global__ __launch_bounds__(256) void gemm_dtl_rect_kernel(GemmArgs g) {  // g: by value, adjusted per k slice
  __shared__ __attribute__((aligned(1024))) char lds[kRectLds];
  int pid = blockIdx.x;
  if (g.ksplit > 1) {  // this workgroup's k range (k_per: a whole number of stages) and fp32 partial-result plane
    const int T = g.tiles_m * g.tiles_n, slice = pid / T, k0 = slice * g.k_per;
    pid -= slice * T;
    g.A += A_KC ? (size_t)k0 : (size_t)k0 * g.lda;
    g.B += B_KC ? (size_t)k0 : (size_t)k0 * g.ldb;
    g.K = g.k_per;
    g.C = reinterpret_cast<float*>(g.C) + (size_t)slice * g.M * g.ldc;
  }
  dtl_rect_tile<A_KC, B_KC, EPI, FULL>(g, pid, lds);
}

// =================================================================================================
// Eight-wave kernels: two waves on every SIMD, alternating between a memory phase and an MFMA phase.
// A wave's part of the block tile is 128 x 64 (128 accumulator registers), so two waves fit the register file of a SIMD.
// Waves 0-3 (group 0, one per SIMD) and waves 4-7 (group 1) run the same loop one phase apart: group 1 passes one extra barrier before the
// loop and group 0 one behind it, so that every workgroup barrier ends a memory phase of one group and an MFMA phase of
// the other.  Memory phase of iteration k: the 12 operand fragments (32 k) are read from LDS into registers, and the wave waits until its
// own direct-to-LDS loads of what is read next have landed.  MFMA phase: 32 v_mfma_f32_16x16x32_bf16, and between them the loads that refill LDS.
//   Why 16x16x32 and not 32x32x16: the chip lowers its clock under MFMA load, and the smaller shape moves half the accumulator registers per
// flop (registers only, random-normal operands 1865 -> 2115 TFLOP/s, zeros 2425 with either).  Its sums are those of the larger shape bit for bit.
//   Why the loads stand between the MFMAs: a memory phase issues 24 reads at most, and an instruction that loads 1 KB holds its wave up for 16 cycles and
// more; behind the reads they made the memory phase the longer of the two (TN 4096 x 2048 x 8192 with the MFMAs left out 115 of 131 us).
//   Numbering: barriers B0 (before the loop, all waves), B(2k+1) = {group 0 ends its memory phase k, group 1 ends its MFMA phase k-1 (k = 0: the
// extra barrier)}, B(2k+2) = {group 0 ends MFMA phase k, group 1 ends memory phase k}.  Group 0 reads for iteration k between B(2k) and
// B(2k+1), group 1 between B(2k+1) and B(2k+2); every wave's reads have returned (lgkmcnt(0)) before it reaches the barrier that ends the phase.
// So (a) what group 0 loads is there for both groups' iteration k+1 if its waves have waited before B(2k+1) (memory phase k), what group 1 loads if its
// waves have waited before B(2k+2) (memory phase k); (b) in its MFMA phase k group 0 may refill what was read last in iteration k-1, group 1 what
// was read last in iteration k.
//   256 x 256 tiles (variant 301256256): waves 2 x 4, both groups read the same 32 k.  Group 0 loads A, group 1 B, each into a ring of its own; 160 KB in
// all.  A k-major operand comes in units of 64 k, rows of 128 bytes: rows of 64 bytes take the L2 twice the requests and the loop was bound by them
// (NT 4096 x 4096 x 8192 without MFMAs 196 -> 154 us).  us on cold operands, four stages of 32 k that both groups load in their memory phases with 32x32x16 ->
// now: 8192 rows x 4096 NN 1536 bias 102 -> 95, NN 2048 x 4096 bias+GeLU 125 -> 107, NT 2048 x 4096 dGeLU 135 -> 115, NT 4096 x 2048 138 -> 122, NN
// 4096 x 2048 130 -> 117, NN 4096 x 512 60 -> 54.5; TN 4096 x 4096 x 8192 224 -> 213.
//   128 x 256 tiles (301128256, over k slices 302128256 / 304128256): waves 1 x 4 x 2 -- the two groups take the k halves of 64 k and add their
// accumulators through LDS after the loop.  TN: the halves are stages of their own (six), group 0 loads those of group 1 and the other way round, so
// that a load has two iterations to arrive (4096 x 2048 x 8192 129 -> 122 us).  With a k-major operand, whose 128-byte rows hold both halves: three stages of 64 k that
// all waves load in their memory phases (NT 4096 x 2048 x 8192 121 -> 116).
// A row-indexed operand may end inside its tile, and on 128 x 256 tiles so may a k-major one (pp_src).  K: whole multiples of 32 resp. 64, TN on 128 x 256 tiles any.
// =================================================================================================
// Chunk swizzles of the operand tiles that 16-row fragments are read from: 16-byte chunk c of a row lies at slot c ^ swizzle(row).
//   Row-indexed, k rows of 256 bytes and more: one LDS cycle of the transpose read serves 32 lanes, 8 bytes each, here the k rows 0..3 and 8..11 of
//   an eight-row pitch x 32 bytes, which then fall on 16 different chunk positions mod 16.
//   k-major, rows of 128 bytes: one cycle of ds_read_b128 serves the lanes 0-3, 12-15, 20-27 (or 4-11, 16-19, 28-31) of a half wave, and lanes
//   16-31 hold the next chunk of the rows of lanes 0-15.  (Rows of 64 bytes would do for a stage of 32 k, with 2 ((row/8)%2), but a load of half
//   lines takes the L2 twice the requests: TCP_TCC_READ_REQ of NT 4096 x 4096 x 8192 33.5 against 16.8 million.)
// SQ_LDS_BANK_CONFLICT is 0 with both.
__device__ __forceinline__ int mc_swizzle(int kr) { return 4 * (kr & 3) ^ 2 * ((kr >> 3) & 1); }
__device__ __forceinline__ int kc_swizzle(int row) { return (row >> 1) & 7; }
// byte offset from the operand of the 16 bytes that a lane fetches in DMA instruction q of the first k tile (k-major: 64 k) of R rows (columns)
// from r0.  Rows / columns beyond the operand's extent are fetched from its last row / first column: valid memory, and what they feed is never stored.
template <bool KC, int R>
__device__ __forceinline__ uint32_t pp_src(int ld, int r0, int q, int lane, int extent) {
  if (KC) {
    const int row = 8 * q + (lane >> 3), chunk = (lane & 7) ^ kc_swizzle(row);
    return ((uint32_t)min(r0 + row, extent - 1) * ld + chunk * 8) * 2u;
  }
  constexpr int CPR = R / 8, KPI = 64 / CPR;
  const int kr = KPI * q + lane / CPR, cc = (lane % CPR) ^ mc_swizzle(kr);
  int col = r0 + cc * 8;
  if (col >= extent) col = 0;
  return ((uint32_t)kr * ld + col) * 2u;
}
// Fragments of 16 rows (columns) x 32 k from an operand tile in LDS.  k-major, PITCH bytes a row: one offset, fragment i adds 16 rows; row-indexed,
// PITCH bytes a k row: an offset per fragment (the swizzle falls on the column), its second half lies four k rows on.
template <bool KC, int N>
struct FragOffsets {
  uint32_t off[KC ? 1 : N];
};
template <bool KC, int PITCH, int N>
__device__ __forceinline__ void read_frags16(u32x4 (&f)[N], uint32_t base, const FragOffsets<KC, N>& o) {
  static_assert(N == 2 || N == 4 || N == 8, "fragments of a wave");
  if constexpr (KC) {
    const uint32_t a = base + o.off[0];
    f[0] = lds_read_b128<0>(a);
    f[1] = lds_read_b128<16 * PITCH>(a);
    if constexpr (N > 2) {
      f[2] = lds_read_b128<32 * PITCH>(a);
      f[3] = lds_read_b128<48 * PITCH>(a);
    }
    if constexpr (N > 4) {
      f[4] = lds_read_b128<64 * PITCH>(a);
      f[5] = lds_read_b128<80 * PITCH>(a);
      f[6] = lds_read_b128<96 * PITCH>(a);
      f[7] = lds_read_b128<112 * PITCH>(a);
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; i++) {
      const u32x2 lo = lds_read_tr16_b64<0>(base + o.off[i]);
      const u32x2 hi = lds_read_tr16_b64<4 * PITCH>(base + o.off[i]);
      f[i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
  }
}

// SWZ(row or k row): the chunk swizzle of the layout; R0: first row (column) of the wave's part; chunk0 / krow0: its k range in the tile
template <int PITCH, int N, class SWZ>
__device__ __forceinline__ FragOffsets<true, N> frag_offsets_kc(int R0, int chunk0, int lane, SWZ swz) {
  const int row = R0 + (lane & 15);
  FragOffsets<true, N> o;
  o.off[0] = (uint32_t)(row * PITCH + (((chunk0 + (lane >> 4)) ^ swz(row)) << 4));
  return o;
}
template <int PITCH, int N, class SWZ>
__device__ __forceinline__ FragOffsets<false, N> frag_offsets_mc(int R0, int krow0, int lane, SWZ swz) {
  const int krow = krow0 + 8 * (lane >> 4) + ((lane & 15) >> 2);
  FragOffsets<false, N> o;
#pragma unroll
  for (int i = 0; i < N; i++) {
    const int col = R0 + 16 * i + 4 * (lane & 3);
    o.off[i] = (uint32_t)(krow * PITCH + (((col >> 3) ^ swz(krow)) << 4) + (col & 7) * 2);
  }
  return o;
}
// the fragments of a k step of 32 against each other, every second row of tiles backwards: neighbouring MFMAs share an operand
// between(i): what goes behind row i
template <bool ROWS, int NA, int NB, class F>
__device__ __forceinline__ void mma16(f32x4 (&acc)[NA][NB], const u32x4 (&fa)[NA], const u32x4 (&fb)[NB], F between) {
#pragma unroll
  for (int i = 0; i < NA; i++) {
#pragma unroll
    for (int jj = 0; jj < NB; jj++) {
      const int j = (i & 1) ? NB - 1 - jj : jj;
      const bf16x8 a = __builtin_bit_cast(bf16x8, fa[i]), b = __builtin_bit_cast(bf16x8, fb[j]);
      if constexpr (ROWS) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[i][j], 0, 0, 0);
      else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, acc[i][j], 0, 0, 0);
    }
    between(i);
  }
}
__device__ __forceinline__ void wait_frags16(u32x4 (&a)[8], u32x4 (&b)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]),
                 "+v"(b[3]));
}
__device__ __forceinline__ void wait_frags16(u32x4 (&a)[2], u32x4 (&b)[2]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]));
}
__device__ __forceinline__ void wait_frags16(u32x4 (&a)[2], u32x4 (&b)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
}
__device__ __forceinline__ void wait_frags16(u32x4 (&a)[4], u32x4 (&b)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
}

constexpr int kPpLds256 = 5 * (256 + 256) * 64;                             // 160 KB
constexpr int kPpExchange = 8 * 2 * 2 * 4 * 64 * 16;                        // 128 x 256 tiles: half of every wave's accumulator
constexpr int kPpLds128 = 6 * (128 + 256) * 64;                  // 144 KB
static_assert(kPpExchange + 16 <= kPpLds128, "exchange and flag");

// k slices that are added up by the launch itself: every workgroup of a tile leaves its partial sums in `part`
// ([tile][slice][wave][group of four][half][lane] x 2 floats, so that each access of a wave is whole lines) and counts itself in; whoever counts last
// has all of them, adds them in slice order (its own from registers, at its place) and runs the epilogue.  Nobody waits for
// anybody, so it does not matter how many workgroups are resident.  The counter is 0 before the launch and again behind it.
// Partial sums and counters cross XCDs, whose L2s do not see each other's lines: they are stored and loaded as relaxed atomics of
// agent scope, i.e. past the L2, and a wave has waited for its stores when its workgroup counts itself in.  (Plain stores between
// release and acquire fences, which write back and drop whole L2s, took 15 us and more per launch.)
struct SliceSum {
  float* part;
  uint32_t* counter;
  int slice, slices;
};
// true in every thread of the workgroup that came last.  lds: four bytes that no wave uses any more
__device__ __forceinline__ bool last_slice(const SliceSum& ss, char* lds) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();  // the whole workgroup's partial sums are written
  uint32_t* flag = reinterpret_cast<uint32_t*>(lds);
  if (threadIdx.x == 0) {
    const uint32_t before = __hip_atomic_fetch_add(ss.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = before == (uint32_t)ss.slices - 1;
    if (last) __hip_atomic_store(ss.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = last;
  }
  __syncthreads();
  return *flag != 0;
}
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void slice_store(uint64_t* p, const f32x4& v) {
  const u64x2 w = __builtin_bit_cast(u64x2, v);
  __hip_atomic_store(p, w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(p + 64, w[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x4 slice_load(uint64_t* p) {
  const u64x2 w = {__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), __hip_atomic_load(p + 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
  return __builtin_bit_cast(f32x4, w);
}

// v: this lane's N groups of four partial sums, replaced by the sums over the slices where the function returns true (the workgroup that came last)
template <int N>
__device__ __forceinline__ bool sum_slices(const SliceSum& ss, f32x4 (&v)[N], char* flag) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr size_t plane = 8 * N * 128;  // in pairs of floats; eight waves
  uint64_t* p = reinterpret_cast<uint64_t*>(ss.part) + (size_t)wave * N * 128 + lane;
#pragma unroll
  for (int q = 0; q < N; q++) slice_store(p + ss.slice * plane + q * 128, v[q]);
  if (!last_slice(ss, flag)) return false;
  f32x4 sum[N];
#pragma unroll
  for (int q = 0; q < N; q++) sum[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int sl = 0; sl < ss.slices; sl++) {
    f32x4 x[N];
#pragma unroll
    for (int q = 0; q < N; q++) x[q] = sl == ss.slice ? v[q] : slice_load(p + sl * plane + q * 128);
#pragma unroll
    for (int q = 0; q < N; q++) sum[q] = sl == 0 ? x[q] : sum[q] + x[q];
  }
#pragma unroll
  for (int q = 0; q < N; q++) v[q] = sum[q];
  return true;
}

template <int N>
__device__ __forceinline__ void vm_wait() {  // vmcnt(N)
  __builtin_amdgcn_s_waitcnt(((N >> 4) << 14) | (N & 15) | (7 << 4) | (15 << 8));
}
template <int BM, bool A_KC, bool B_KC, int EPI, bool FULL, bool SLICED = false>
__device__ __forceinline__ void pp_tile(const GemmArgs& g, int pid, char* lds, const SliceSum& ss = SliceSum{}) {
  static_assert(BM == 256 || BM == 128, "block tiles 256 x 256 and 128 x 256");
  static_assert(!SLICED || BM == 128, "slices: 128 x 256 tiles");
  constexpr bool SQ = BM == 256;
  constexpr bool HALVES = !SQ && !A_KC && !B_KC;     // 128 x 256, each group's k half a stage of its own
  // k extent of what an instruction fetches of a row, and with it of a stage: the row-indexed operands 32 (64 where both groups read one stage), the
  // k-major ones 64, whole lines of 128 bytes
  constexpr int TK_A = A_KC || (!SQ && !HALVES) ? 64 : 32, TK_B = B_KC || (!SQ && !HALVES) ? 64 : 32;
  int tile_m, tile_n;
  tile_of_workgroup(pid, g.tiles_m, g.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * 256;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, wn = wave & 3;          // grp: phase group; 256 x 256: also the row half, 128 x 256: the k half

  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const __amdgpu_buffer_rsrc_t rsA = operand_rsrc(g.A), rsB = operand_rsrc(g.B);
  const uint32_t stepA_k = 2u * TK_A * (A_KC ? 1u : g.lda), stepB_k = 2u * TK_B * (B_KC ? 1u : g.ldb);  // next k tile

  constexpr int PITCH_A = A_KC ? 2 * TK_A : 2 * BM, PITCH_B = B_KC ? 2 * TK_B : 2 * 256;  // row pitches of the two layouts
  const int k32 = !SQ && !HALVES ? grp : 0;
  FragOffsets<A_KC, 8> offA;
  FragOffsets<B_KC, 4> offB;
  const int ra = SQ ? grp * 128 : 0;
  if constexpr (A_KC) offA = frag_offsets_kc<PITCH_A, 8>(ra, 4 * k32, lane, kc_swizzle);
  else offA = frag_offsets_mc<PITCH_A, 8>(ra, 32 * k32, lane, mc_swizzle);
  if constexpr (B_KC) offB = frag_offsets_kc<PITCH_B, 4>(wn * 64, 4 * k32, lane, kc_swizzle);
  else offB = frag_offsets_mc<PITCH_B, 4>(wn * 64, 32 * k32, lane, mc_swizzle);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(OASES_LDS char*)lds;
  u32x4 fa[8], fb[4];
  // the end of a memory phase and the MFMA phase, with the loads that go between its MFMAs.  left: k from the first of the fragments on (HALVES:
  // weight gradients over a number of rows that is no whole number of k tiles; k beyond K counts as zero in both operands)
  auto multiply = [&](auto between, int left = 32) {
    wait_frags16(fa, fb);
    __builtin_amdgcn_sched_barrier(0);
    if (HALVES && left < 32 && 8 * (lane >> 4) >= left) {
#pragma unroll
      for (int i = 0; i < 8; i++) fa[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < 4; j++) fb[j] = u32x4{0u, 0u, 0u, 0u};
    }
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    mma16<epi_rows(EPI)>(acc, fa, fb, between);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto begin = [&]() {
    __builtin_amdgcn_s_barrier();                 // B0
    if (grp == 1) __builtin_amdgcn_s_barrier();   // group 1 runs one phase behind
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (SQ) {
    const int S = g.K / 32;  // iterations
    // the two groups run code of their own: a branch between MFMAs, taken or not, costs the MFMA pipe more than what it jumps over
    auto run = [&](auto grp_c) {
      constexpr int GRP = decltype(grp_c)::value;
      // a unit of a ring: 64 k (k-major: two k tiles, an instruction fetches 8 rows x 128 bytes) or one k tile of 32 (row-indexed)
      constexpr int RING_A = A_KC ? 3 : 5, RING_B = B_KC ? 2 : A_KC ? 4 : 5;       // units
      constexpr int UNIT_A = 256 * TK_A * 2, UNIT_B = 256 * TK_B * 2, kB = RING_A * UNIT_A;  // bytes; where the ring of B begins
      static_assert(kB + RING_B * UNIT_B == kPpLds256, "rings");
      // what this group loads
      constexpr bool KC = GRP ? B_KC : A_KC;
      constexpr int PER = KC ? 8 : 4, RING = GRP ? RING_B : RING_A, UNIT = GRP ? UNIT_B : UNIT_A;
      const __amdgpu_buffer_rsrc_t rs = GRP ? rsB : rsA;
      const uint32_t step = GRP ? stepB_k : stepA_k;
      uint32_t src[PER];
#pragma unroll
      for (int j = 0; j < PER; j++) src[j] = pp_src<KC, 256>(GRP ? g.ldb : g.lda, GRP ? n0 : m0, PER * wn + j, lane, GRP ? g.N : g.M);
      char* const dst = lds + (GRP ? kB : 0) + PER * wn * 1024;
      auto issue1 = [&](int j, int u, uint32_t at) { dma16(rs, src[j], (uint32_t)u * step, dst + at + j * 1024); };
      // all of unit u; K an odd number of k tiles: the second half of the last unit of a k-major operand lies beyond K and is fetched from the first half (not used)
      auto issue_all = [&](int u, uint32_t at) {
        const uint32_t back = KC && 2 * u + 1 == S ? 64 : 0;
#pragma unroll
        for (int j = 0; j < PER; j++) {
          const int chunk = (lane & 7) ^ ((4 * j + (lane >> 4)) & 7);  // of eight: instruction j of a k-major unit
          dma16(rs, chunk >= 4 ? src[j] - back : src[j], (uint32_t)u * step, dst + at + j * 1024);
        }
      };
      // before the loop: as many units as are there when the loop is in MFMA phase 0
      constexpr int FIRST = GRP ? RING : KC ? 2 : 4, TILES = KC ? 2 : 1;
#pragma unroll
      for (int u = 0; u < FIRST; u++)
        if (u * TILES < S) issue_all(u, u * UNIT);
      if (S < 5) vm_wait<0>(); else vm_wait<PER * (FIRST - 1)>();  // unit 0
      begin();
      uint32_t curA = 0, curB = kB, into = FIRST % RING * UNIT;
      constexpr int YOUNG = KC ? (GRP ? 0 : 8) : 4 * ((GRP ? RING : 4) - 2);  // instructions behind those of what is read next
      auto read = [&](uint32_t odd) {
        FragOffsets<A_KC, 8> oa = offA;
        FragOffsets<B_KC, 4> ob = offB;
        if constexpr (A_KC) oa.off[0] ^= odd * 64;  // the other four chunks of a row
        if constexpr (B_KC) ob.off[0] ^= odd * 64;
        read_frags16<A_KC, PITCH_A>(fa, lds0 + curA, oa);
        read_frags16<B_KC, PITCH_B>(fb, lds0 + curB, ob);
      };
      auto advance = [&](bool odd) {
        if (!A_KC || odd) curA = curA + UNIT_A == RING_A * UNIT_A ? 0 : curA + UNIT_A;
        if (!B_KC || odd) curB = curB + UNIT_B == kPpLds256 ? kB : curB + UNIT_B;
      };
      auto advance_into = [&]() { into = into + UNIT == RING * UNIT ? 0 : into + UNIT; };
      auto unit_of = [&](int kt) { return KC ? (kt >> 1) + 2 : kt + (GRP ? RING : 4); };
      // MFMA phase kt loads, if k-major, unit kt / 2 + 2 (A: even kt, B: odd), else unit kt + 4 (A) or kt + RING_B
      auto iteration = [&](auto odd_c, int kt) {
        constexpr bool ODD = decltype(odd_c)::value;
        read(ODD);
        constexpr bool ON = !KC || ODD == (GRP == 1);
        if (!KC || ODD) vm_wait<YOUNG>();
        multiply([&](int i) {
          if (ON && i < PER) {
            __builtin_amdgcn_sched_barrier(0);
            issue1(i, unit_of(kt), into);
            __builtin_amdgcn_sched_barrier(0);
          }
        });
        advance(ODD);
        if (ON) advance_into();
      };
      int kt = 0;
      for (; kt + 1 + 5 < S; kt += 2) {
        iteration(std::false_type{}, kt);
        iteration(std::true_type{}, kt + 1);
      }
      for (; kt < S; kt++) {  // few k tiles left behind this one: what is still to be loaded goes behind the MFMA phase
        const bool odd = kt & 1;
        read(odd);
        int young;  // as above, as far as it exists
        if (KC) young = GRP ? (odd ? 0 : 8) : 2 * (kt >> 1) + 4 < S ? 8 : 0;
        else young = 4 * (min(S, unit_of(kt)) - (kt + 2));
        if (young >= 12) vm_wait<12>();
        else if (young >= 8) vm_wait<8>();
        else if (young >= 4) vm_wait<4>();
        else vm_wait<0>();
        multiply([](int) {});
        const int u = unit_of(kt);
        if ((!KC || odd == (GRP == 1)) && u * TILES < S) {
          issue_all(u, into);
          advance_into();
        }
        advance(odd);
      }
    };
    if (grp == 0) run(std::integral_constant<int, 0>{}); else run(std::integral_constant<int, 1>{});
  } else {
    constexpr int TK = TK_A, NS = HALVES ? 6 : 3;                            // k of a stage, stages
    constexpr int kOpA = BM * TK * 2, kStage = (BM + 256) * TK * 2;          // bytes of the A part of a stage (B behind it), of a stage
    constexpr int PER_A = 2, PER_B = 4, PER = PER_A + PER_B;                 // direct-to-LDS instructions of a wave per k tile that it loads
    const int nk = HALVES ? (g.K + 63) / 64 : g.K / TK, S = HALVES ? 2 * nk : nk;  // iterations of a wave, k tiles
    uint32_t srcA[PER_A], srcB[PER_B];
    const int lw = HALVES ? wn : wave;  // which of the waves that load a k tile
#pragma unroll
    for (int j = 0; j < PER_A; j++) srcA[j] = pp_src<A_KC, BM>(g.lda, m0, PER_A * lw + j, lane, g.M);
#pragma unroll
    for (int j = 0; j < PER_B; j++) srcB[j] = pp_src<B_KC, 256>(g.ldb, n0, PER_B * lw + j, lane, g.N);
    auto issue1 = [&](int j, int t, uint32_t at) {  // instruction j of k tile t into the stage at byte `at`
      if (j < PER_A) dma16(rsA, srcA[j], (uint32_t)t * stepA_k, lds + at + (PER_A * lw + j) * 1024);
      else dma16(rsB, srcB[j - PER_A], (uint32_t)t * stepB_k, lds + at + kOpA + (PER_B * lw + j - PER_A) * 1024);
    };
    auto issue_all = [&](int t, uint32_t at) {  // k rows beyond K from k = 0
#pragma unroll
      for (int j = 0; j < PER; j++) {
        if (!HALVES || 32 * t + 32 <= g.K) {
          issue1(j, t, at);
        } else if (j < PER_A) {
          const int kr = 4 * (PER_A * lw + j) + (lane >> 4);
          dma16(rsA, 32 * t + kr < g.K ? srcA[j] + (uint32_t)t * stepA_k : srcA[j] - kr * (stepA_k / 32), 0, lds + at + (PER_A * lw + j) * 1024);
        } else {
          const int q = PER_B * lw + j - PER_A, kr = 2 * q + (lane >> 5);
          dma16(rsB, 32 * t + kr < g.K ? srcB[j - PER_A] + (uint32_t)t * stepB_k : srcB[j - PER_A] - kr * (stepB_k / 32), 0, lds + at + kOpA + q * 1024);
        }
      }
    };
    auto next = [](uint32_t at, int n) { return at + n * kStage >= NS * kStage ? at + (n - NS) * kStage : at + n * kStage; };
    auto read = [&](uint32_t at) {
      read_frags16<A_KC, PITCH_A>(fa, lds0 + at, offA);
      read_frags16<B_KC, PITCH_B>(fb, lds0 + at + kOpA, offB);
    };
    if constexpr (HALVES) {
      // before the loop: group 0 k tiles 1 and 3, group 1 k tiles 0, 2 and 4
#pragma unroll
      for (int q = 0; q < 3; q++) {
        const int t = 1 - grp + 2 * q;
        if (t < min(S, NS - 1)) issue_all(t, t * kStage);
      }
      if (grp == 1) {  // own part of tile 0
        if (S >= NS - 1) vm_wait<2 * PER>(); else vm_wait<0>();
      }
      begin();
      uint32_t cur = grp * kStage, into = grp ? 0 : (NS - 1) * kStage;  // stages that the iteration reads and refills,
      const int ahead = grp ? NS : NS - 1;                              // the latter with k tile 2 kt + ahead
      auto iteration = [&](auto steady_c, int kt) {
        constexpr bool STEADY = decltype(steady_c)::value;  // that k tile exists and is whole
        read(cur);
        if (STEADY || nk - 1 - kt > grp) vm_wait<PER>(); else vm_wait<0>();  // the k tile of this wave's loads that is read next, and one behind it
        multiply([&](int i) {
          if (STEADY && i < PER) {
            __builtin_amdgcn_sched_barrier(0);
            issue1(i, 2 * kt + ahead, into);
            __builtin_amdgcn_sched_barrier(0);
          }
        }, STEADY ? 32 : g.K - 32 * (2 * kt + grp));
        if (!STEADY && 2 * kt + ahead < S) issue_all(2 * kt + ahead, into);
        cur = next(cur, 2);
        into = next(into, 2);
      };
      int kt = 0;
      for (; 2 * kt + ahead < g.K / 32; kt++) iteration(std::true_type{}, kt);
      for (; kt < nk; kt++) iteration(std::false_type{}, kt);
    } else {
#pragma unroll
      for (int t = 0; t < NS - 1; t++)
        if (t < S)
#pragma unroll
          for (int j = 0; j < PER; j++) issue1(j, t, t * kStage);
      if (S > 1) vm_wait<PER>(); else vm_wait<0>();  // own part of tile 0
      begin();
      uint32_t cur = 0, into = (NS - 1) * kStage;
      auto iteration = [&](auto steady_c, int kt) {
        constexpr bool STEADY = decltype(steady_c)::value;  // k tile kt + 2 exists
        read(cur);
        if (STEADY) {
#pragma unroll
          for (int j = 0; j < PER; j++) issue1(j, kt + NS - 1, into);
          vm_wait<PER>();
        } else {
          vm_wait<0>();
        }
        multiply([](int) {});
        cur = next(cur, 1);
        into = next(into, 1);
      };
      int kt = 0;
      for (; kt + NS - 1 < S; kt++) iteration(std::true_type{}, kt);
      for (; kt < S; kt++) iteration(std::false_type{}, kt);
    }
  }
  if (grp == 0) __builtin_amdgcn_s_barrier();   // group 0 catches up: both groups have passed the same number of barriers
  __builtin_amdgcn_sched_barrier(0);

  // What the epilogue reads besides the accumulators is under way a tile row ahead (see epi_request; a bias once for all rows).
  constexpr bool BIAS = EPI == EPI_BIAS_BF16 || EPI == EPI_BIAS_GELU, READS = BIAS || EPI == EPI_ACC_F32 || EPI == EPI_DGELU || EPI == EPI_DSWIGLU;
  EpiOperands eo[2][2][2][2];  // [buffer][16 rows][32 columns][16 columns]
  auto request = [&](EpiOperands (&o)[2][2][2], int row0) {
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int j = 0; j < 2; j++) {
        if (!BIAS || h == 0) epi_request16<EPI, FULL, true>(g, row0 + 16 * h, n0 + wn * 64 + 32 * j, lane, o[h][j]);
      }
  };
  // 16 rows of the wave's 64 columns
  auto finish_rows = [&](int row, const f32x4& a0, const f32x4& a1, const f32x4& a2, const f32x4& a3, const EpiOperands (&o)[2][2]) {
    if constexpr (EPI == EPI_SWIGLU) {  // the wave's 64 columns are one [gate 32 | up 32] block
      epi_swiglu16<FULL, true>(g, row, n0 + wn * 64, lane, a0, a1, a2, a3);
    } else {
      epi_finish16<EPI, FULL, true>(g, row, n0 + wn * 64, lane, a0, a1, o[0]);
      epi_finish16<EPI, FULL, true>(g, row, n0 + wn * 64 + 32, lane, a2, a3, o[1]);
    }
  };
  if constexpr (SQ) {
    const int r0 = m0 + grp * 128;
    if constexpr (READS) request(eo[0], r0);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if (READS && !BIAS && i < 3) request(eo[(i + 1) & 1], r0 + 32 * (i + 1));
#pragma unroll
      for (int h = 0; h < 2; h++)
        finish_rows(r0 + 32 * i + 16 * h, acc[2 * i + h][0], acc[2 * i + h][1], acc[2 * i + h][2], acc[2 * i + h][3], eo[BIAS ? 0 : i & 1][BIAS ? 0 : h]);
    }
  } else {
    // The two waves that hold the k halves of one 128 x 64 part each finish 64 of its rows: a wave hands the accumulator
    // tiles of the other 64 rows over through LDS (lane for lane) and adds what it receives to its own (two terms: the
    // order of the addition does not matter).
    f32x4* xch = reinterpret_cast<f32x4*>(lds);
    const int mine = wave * 16, theirs = (wave ^ 4) * 16;  // 4 x 4 tiles per wave
    __syncthreads();  // every wave has its last fragments in registers, and all direct-to-LDS loads have landed
    auto hand_over = [&](auto half_c) {
      constexpr int H = decltype(half_c)::value;
#pragma unroll
      for (int q = 0; q < 16; q++) xch[(mine + q) * 64 + lane] = acc[H * 4 + (q >> 2)][q & 3];
    };
    if (grp == 0) hand_over(std::integral_constant<int, 1>{}); else hand_over(std::integral_constant<int, 0>{});
    __syncthreads();
    f32x4 v[16];  // this wave's 64 x 64 part of the tile, both k halves
    auto gather = [&](auto half_c) {
      constexpr int H = decltype(half_c)::value;
#pragma unroll
      for (int q = 0; q < 16; q++) v[q] = acc[H * 4 + (q >> 2)][q & 3] + xch[(theirs + q) * 64 + lane];
    };
    if (grp == 0) gather(std::integral_constant<int, 0>{}); else gather(std::integral_constant<int, 1>{});
    if constexpr (SLICED) {
      if (!sum_slices<16>(ss, v, lds + kPpLds128 - 16)) return;
    }
    if constexpr (READS) {
      request(eo[0], m0 + grp * 64);
      if (!BIAS) request(eo[1], m0 + grp * 64 + 32);
    }
#pragma unroll
    for (int i = 0; i < 4; i++)
      finish_rows(m0 + grp * 64 + 16 * i, v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3], eo[BIAS ? 0 : i >> 1][BIAS ? 0 : i & 1]);
  }
}

// this workgroup's k range (k_per: a whole number of stages) and, unless the launch adds its slices up itself (OWN), its fp32 plane; floats: partial
// sums of a workgroup
template <bool A_KC, bool B_KC, bool OWN, class G>
__device__ __forceinline__ SliceSum take_slice(G& g, int& pid, int floats) {
  const int T = g.tiles_m * g.tiles_n, slice = pid / T, k0 = slice * g.k_per;
  pid -= slice * T;
  g.A += A_KC ? (size_t)k0 : (size_t)k0 * g.lda;
  g.B += B_KC ? (size_t)k0 : (size_t)k0 * g.ldb;
  g.K = min(g.K - k0, g.k_per);
  if constexpr (OWN) {
    return SliceSum{g.part + (size_t)pid * g.ksplit * floats, g.counters + pid, slice, g.ksplit};
  } else {
    g.C = reinterpret_cast<float*>(g.C) + (size_t)slice * g.M * g.ldc;
    return SliceSum{};
  }
}

// SLICED: k slices that the launch adds up itself.  G: GemmArgs or GemmCall, written out where a kernel is launched (a type formed from an unnamed
// enumeration would have another name on the host)
template <int BM, bool A_KC, bool B_KC, int EPI, bool FULL, bool SLICED, class G>
__global__ __launch_bounds__(512) void gemm_pp_kernel(G g) {  // by value, adjusted per k slice
  __shared__ __attribute__((aligned(1024))) char lds[BM == 256 ? kPpLds256 : kPpLds128];
  int pid = blockIdx.x;
  SliceSum ss{};
  if (BM == 128 && g.ksplit > 1) ss = take_slice<A_KC, B_KC, SLICED>(g, pid, 128 * 256);
  pp_tile<BM, A_KC, B_KC, EPI, FULL, SLICED>(g, pid, lds, ss);
}

// Two weight-gradient contractions over the same K rows in one launch: the tiles of the second problem follow those of
// the first, so that two launches that would each leave CUs idle (or need k slices to fill them) share one round.  SLICED: slice
// after slice of all tiles, added up as above.
template <bool FULL, bool SLICED>
__global__ __launch_bounds__(512) void gemm_pp_group_kernel(GemmArgs g0, GemmArgs g1, float* part, uint32_t* counters) {
  __shared__ __attribute__((aligned(1024))) char lds[kPpLds128];
  const int first = g0.tiles_m * g0.tiles_n, T = first + g1.tiles_m * g1.tiles_n;
  int pid = blockIdx.x;
  SliceSum ss{};
  if constexpr (SLICED) {
    const int slice = pid / T;
    pid -= slice * T;
    ss = SliceSum{part + (size_t)pid * g0.ksplit * 128 * 256, counters + pid, slice, g0.ksplit};
  }
  const bool second = pid >= first;
  GemmArgs g = second ? g1 : g0;
  if constexpr (SLICED) {
    const int k0 = ss.slice * g.k_per;
    g.A += (size_t)k0 * g.lda;
    g.B += (size_t)k0 * g.ldb;
    g.K = min(g.K - k0, g.k_per);
  }
  pp_tile<128, false, false, EPI_ACC_F32, FULL, SLICED>(g, second ? pid - first : pid, lds, ss);
}

// =================================================================================================
// Small tiles: 64 x 64 (TN = 1) and 64 x 128 (TN = 2), for launches that the large tiles would leave short of workgroups or
// that are a chain of memory latencies rather than MFMA work.  Eight waves: 2 x 2 parts of 32 x 32 TN elements, times two
// k halves -- a wave multiplies one of the two 32-wide k steps of a 64-wide stage (v_mfma_f32_16x16x32_bf16), and the two partial sums of a part
// meet once, through LDS, after the loop (a k half has its own accumulator, so the order of the additions is the same for
// every shape).  Tiles come by direct-to-LDS buffer loads into NS stages, so NS-1 tiles are in flight: with K of a few
// hundred the whole k extent is requested before the first MFMA, and the launch pays one memory latency instead of one
// per tile.  The stages take 80 KB (64 x 64, five) and 72 KB (64 x 128, three): two workgroups share a CU.  What the epilogue reads (bias, old C, pre-activations) is
// requested first of all and has arrived by the time it is needed.  One barrier per tile:
//   tile kt has landed when at most PER x (younger tiles in flight) of the wave's loads are outstanding; the barrier makes
//   all waves' parts of it visible and also says that every wave is done with tile kt-1 (its fragments were waited for
//   before its MFMAs), whose stage then takes tile kt+NS-1.
// Any M, N, K that are multiples of 8: rows and columns beyond an operand are fetched from valid memory and never stored;
// k beyond K in the last tile is fetched from k = 0 and replaced by zeros in the fragments.
// Layouts of the operand tiles: k-major [R][64] as in the eight-wave kernels; row-indexed [64][R] with chunk c of k row kr at
// slot c ^ st_swizzle(kr): for R = 128 (256-byte k rows share all banks) the swizzle of the eight-wave kernels, for R = 64 (every second 128-byte k row
// does) the same of the k rows that meet, 4 ((kr/2)%2) ^ 2 ((kr/8)%2).
//   What bounds it: LDS bandwidth when the chip is full (48 KB resp. 72 KB read and written per stage, 0.16 / 0.24 us at 128
// bytes per clock; measured 0.22 / 0.33 us per stage and workgroup), one memory latency plus some 3 us of launch and drain
// otherwise.  Measured in microseconds, register-staged kernels before -> this one: NN bias 256 x 768 x 512 9.5 -> 4.4,
// NT dGeLU 256 x 1024 x 512 12.5 -> 4.8, NN bias+GeLU 200 x 2048 x 1024 18.6 -> 6.8, NT dSwiGLU 1024 x 704 x 1024 21.4 -> 8.1,
// NN bias+GeLU 2048 x 1024 x 1024 18.0 -> 11.2, TN 1024 x 512 x 512 10.0 -> 4.8, NT bf16 4096 x 512 x 2048 22.9 -> 13.9, NN fp32
// 64 x 12288 x 1536 23.1 -> 9.2.  Five stages against three or nine for 64 x 64 and three against six for 64 x 128: within
// 5 % of each other or better; 128 x 128 tiles on the same scheme (four stages): slower on every shape that these two win.
// 16x16x32 MFMAs and a wave's half of the rows (whole lines of C, bf16 sixteen bytes a lane) against 32x32x16 and a half of the columns of every row, us:
// 4096 x 1024 x 1024 NN bias+GeLU 20.8 -> 18.1, NT dGeLU 18.7 -> 17.6, fp32 16.5 -> 16.9; TN 12288 x 6144 x 128 150 -> 137; 512 x 768 x 512 bias 6.8 -> 6.6.  Steps:
// h 1024 619 -> 608, h 12288 with 128 rows 998 -> 969, two recomputed layers of h 1024 536 -> 524, three of 600 rows 533 -> 526.  The fragments of a k step
// requested ahead of the MFMAs of the one before it: within 1 % (the loop waits for its loads, not for LDS).
// =================================================================================================
constexpr int BKS = 64;
template <int R>
__device__ __forceinline__ int st_swizzle(int kr) { return R == 64 ? 4 * ((kr >> 1) & 1) ^ 2 * ((kr >> 3) & 1) : mc_swizzle(kr); }
// byte offset from the operand of the 16 bytes that a lane fetches in DMA instruction q of a tile that starts at row r0
// (k tile 0), and the lane's k within the tile
template <bool KC, int R>
__device__ __forceinline__ uint32_t st_src(int ld, int r0, int q, int lane, int extent, int* k) {
  if (KC) {
    const int row = 8 * q + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    *k = chunk * 8;
    return ((uint32_t)min(r0 + row, extent - 1) * ld + chunk * 8) * 2u;
  }
  constexpr int CPR = R / 8, KPI = 64 / CPR;
  const int kr = KPI * q + lane / CPR, cc = (lane % CPR) ^ st_swizzle<R>(kr);
  int col = r0 + cc * 8;
  if (col >= extent) col = 0;
  *k = kr;
  return ((uint32_t)kr * ld + col) * 2u;
}
template <int TM, int TN, int NS>
struct StLds {
  static constexpr int kStage = 64 * (TM + TN) * BKS * 2, kExchange = 8 * TM * TN * 2 * 64 * 16;  // exchange: half of every wave's accumulator
  static constexpr int bytes = NS * kStage > kExchange ? NS * kStage : kExchange;
};
// sum of the eight bf16 values of a fragment, in fp32
__device__ __forceinline__ float frag_sum(const u32x4& f) {
  const bf16x2_ one = {(__bf16)1.0f, (__bf16)1.0f};
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; i++) s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_, (uint32_t)f[i]), one, s, false);
  return s;
}
// the sums of two fragments of 16 columns each, of the k rows of lanes l and l + 32: lane l has column l%16 of the first, lane 32 + l of the second one
__device__ __forceinline__ float frag_sum_pair(const u32x4& f0, const u32x4& f1) {
  const float x = frag_sum(f0), y = frag_sum(f1);
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
  const uint32_t lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}
// EPI_BF16_DELTA (dO = dZ1 Wo^T): the tile holds whole heads of dO, so the row sums of dO * O come from the registers that store it, for one
// more operand of the epilogue; the launch that read both arrays again is saved (a step of two recomputed layers, h 1024, 512 tokens:
// 544.7 -> 538.2 us; three layers of h 1024, 600 tokens, 128 columns a head: 534.9 -> 533.0, on 64x128 instead of 64x64 tiles).
// COLSUM (weight gradients): the waves of the first row of tiles that hold the first 32 rows also add up B's columns, whose fragments they
// have in registers (eight k of a column to a lane): the vector ALU has time, LDS is what the kernel waits for.  Eight tiles to a partial sum.
// SLICED: k slices that the launch adds up itself; in a kernel of its own, since the code of the sum, even where it is passed over, costs
// every launch 0.1 us (216x1024x256 NN 3.31 -> 3.40, 64x64x64 2.50 -> 2.60).
template <int TM, int TN, int NS, bool A_KC, bool B_KC, int EPI, bool COLSUM = false, bool SLICED = false, class G>
__device__ __forceinline__ void st_tile(const G& g, int pid, char* lds, const SliceSum& ss = SliceSum{}) {
  constexpr int BM = 64 * TM, BN = 64 * TN;
  constexpr int kOpA = BM * BKS * 2, kStage = StLds<TM, TN, NS>::kStage;
  constexpr int PER_A = TM, PER_B = TN, PER = PER_A + PER_B;  // direct-to-LDS instructions of a wave per stage
  static_assert(EPI != EPI_SWIGLU || TN == 2, "gate and up columns of a block must belong to one wave");
  int tile_m, tile_n;
  tile_of_workgroup(pid, g.tiles_m, g.tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
  const int row0 = m0 + wm * 32 * TM, col0 = n0 + wn * 32 * TN;
  const int nk = (g.K + BKS - 1) / BKS, ktail = g.K % BKS;

  // operands of the epilogue.  A wave finishes half wk of its rows
  EpiOperands pre[TM][TN][2];
  if constexpr (EPI != EPI_F32 && EPI != EPI_SWIGLU) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) epi_request16<EPI, false>(g, row0 + 16 * (TM * wk + i), col0 + 32 * j, lane, pre[i][j]);
  }

  const __amdgpu_buffer_rsrc_t rsA = operand_rsrc(g.A), rsB = operand_rsrc(g.B);
  uint32_t srcA[PER_A], srcB[PER_B];
  int kA[PER_A], kB[PER_B];
#pragma unroll
  for (int j = 0; j < PER_A; j++) srcA[j] = st_src<A_KC, BM>(g.lda, m0, PER_A * wave + j, lane, g.M, &kA[j]);
#pragma unroll
  for (int j = 0; j < PER_B; j++) srcB[j] = st_src<B_KC, BN>(g.ldb, n0, PER_B * wave + j, lane, g.N, &kB[j]);
  const uint32_t unitA = A_KC ? 2u : 2u * g.lda, unitB = B_KC ? 2u : 2u * g.ldb;  // one k further
  auto issue = [&](int t, int stage) {
    char* st = lds + stage * kStage;
    const uint32_t tA = (uint32_t)t * BKS * unitA, tB = (uint32_t)t * BKS * unitB;
    if (ktail && t == nk - 1) {  // k >= K: fetched from k = 0 of the same row / column (valid memory, zeroed later)
#pragma unroll
      for (int j = 0; j < PER_A; j++) dma16(rsA, kA[j] < ktail ? srcA[j] + tA : srcA[j] - kA[j] * unitA, 0, st + (PER_A * wave + j) * 1024);
#pragma unroll
      for (int j = 0; j < PER_B; j++) dma16(rsB, kB[j] < ktail ? srcB[j] + tB : srcB[j] - kB[j] * unitB, 0, st + kOpA + (PER_B * wave + j) * 1024);
    } else {
#pragma unroll
      for (int j = 0; j < PER_A; j++) dma16(rsA, srcA[j], tA, st + (PER_A * wave + j) * 1024);
#pragma unroll
      for (int j = 0; j < PER_B; j++) dma16(rsB, srcB[j], tB, st + kOpA + (PER_B * wave + j) * 1024);
    }
  };
  constexpr int PITCH_A = A_KC ? 2 * BKS : 2 * BM, PITCH_B = B_KC ? 2 * BKS : 2 * BN, RA = 2 * TM, CB = 2 * TN;
  auto swz_kc = [](int row) { return (row >> 1) & 7; };
  FragOffsets<A_KC, RA> offA;
  FragOffsets<B_KC, CB> offB;
  if constexpr (A_KC) offA = frag_offsets_kc<PITCH_A, RA>(wm * 32 * TM, 4 * wk, lane, swz_kc);
  else offA = frag_offsets_mc<PITCH_A, RA>(wm * 32 * TM, 32 * wk, lane, st_swizzle<BM>);
  if constexpr (B_KC) offB = frag_offsets_kc<PITCH_B, CB>(wn * 32 * TN, 4 * wk, lane, swz_kc);
  else offB = frag_offsets_mc<PITCH_B, CB>(wn * 32 * TN, 32 * wk, lane, st_swizzle<BN>);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(OASES_LDS char*)lds;

  f32x4 acc[RA][CB];
#pragma unroll
  for (int i = 0; i < RA; i++)
#pragma unroll
    for (int j = 0; j < CB; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int t = 0; t < NS - 1; t++)
    if (t < nk) issue(t, t);

  u32x4 fa[RA], fb[CB];
  int stage = 0;
  bool sums = false;
  if constexpr (COLSUM) sums = g.sums && tile_m == 0 && wm == 0;
  float csum[TN], part[TN];  // lane l: column 32 j + 16 (l/32) + l%16, k = 8 ((l/16)%2)..+7 and the same 16 further on
#pragma unroll
  for (int j = 0; j < TN; j++) csum[j] = part[j] = 0.f;
  // one tile; YOUNG: tiles behind it that may still be in flight (compile-time, for the wait); steady: tile kt+NS-1 exists
  auto iteration = [&](auto young_c, auto steady_c, int kt) {
    constexpr int Y = PER * decltype(young_c)::value;
    constexpr bool STEADY = decltype(steady_c)::value;
    __builtin_amdgcn_s_waitcnt(((Y >> 4) << 14) | (Y & 15) | (7 << 4) | (15 << 8));  // vmcnt(Y)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (STEADY) issue(kt + NS - 1, stage == 0 ? NS - 1 : stage - 1);
    const uint32_t st = lds0 + (uint32_t)stage * kStage;
    read_frags16<A_KC, PITCH_A>(fa, st, offA);
    read_frags16<B_KC, PITCH_B>(fb, st + kOpA, offB);
    wait_frags16(fa, fb);
    __builtin_amdgcn_sched_barrier(0);
    if (!STEADY && decltype(young_c)::value == 0 && ktail) {  // last tile: k beyond K counts as zero in both operands
      if (32 * wk + 8 * (lane >> 4) >= ktail) {
#pragma unroll
        for (int i = 0; i < RA; i++) fa[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int j = 0; j < CB; j++) fb[j] = u32x4{0u, 0u, 0u, 0u};
      }
    }
    if (COLSUM && sums) {
#pragma unroll
      for (int j = 0; j < TN; j++) {
        part[j] += frag_sum_pair(fb[2 * j], fb[2 * j + 1]);
        if ((kt & 7) == 7) {
          csum[j] += part[j];
          part[j] = 0.f;
        }
      }
    }
    mma16<epi_rows(EPI)>(acc, fa, fb, [](int) {});
    stage = stage == NS - 1 ? 0 : stage + 1;
  };
  int kt = 0;
  for (; kt + NS - 1 < nk; kt++) iteration(std::integral_constant<int, NS - 2>{}, std::true_type{}, kt);
  // drain: the tile with r tiles behind it, r = NS-2 .. 0
  auto drain = [&](auto self, auto r_c) {
    constexpr int R = decltype(r_c)::value;
    if (nk > R) iteration(r_c, std::false_type{}, nk - 1 - R);
    if constexpr (R > 0) self(self, std::integral_constant<int, R - 1>{});
  };
  drain(drain, std::integral_constant<int, NS - 2>{});

  // The two k halves of a part: each wave hands the rows that the other one finishes over through LDS and adds what it
  // receives to its own (two terms: the order of the addition does not matter)
  f32x4* xch = reinterpret_cast<f32x4*>(lds);
  constexpr int NV = TM * CB;  // tiles of a wave's half
  __syncthreads();  // every wave has its last fragments in registers, and all direct-to-LDS loads have landed
  auto hand_over = [&](auto half_c) {
    constexpr int I = TM * decltype(half_c)::value;
#pragma unroll
    for (int q = 0; q < NV; q++) xch[(wave * NV + q) * 64 + lane] = acc[I + q / CB][q % CB];
  };
  if (wk == 0) hand_over(std::integral_constant<int, 1>{}); else hand_over(std::integral_constant<int, 0>{});
  float* xsum = reinterpret_cast<float*>(lds + StLds<TM, TN, NS>::kExchange) + 64 * TN * wn;
  if (COLSUM && sums) {
#pragma unroll
    for (int j = 0; j < TN; j++) {
      csum[j] += part[j];
      if (wk == 1) xsum[64 * j + lane] = csum[j];
    }
  }
  __syncthreads();
  if constexpr (COLSUM) if (sums && wk == 0) {
    static_assert(StLds<TM, TN, NS>::kExchange + 512 * TN <= StLds<TM, TN, NS>::bytes, "column sums behind the exchange");
#pragma unroll
    for (int j = 0; j < TN; j++) {
      float t = csum[j] + xsum[64 * j + lane];
      t += __shfl_xor(t, 16, 64);  // the other k of a step
      const int col = col0 + 32 * j + 16 * (lane >> 5) + (lane & 15);
      if (!(lane & 16) && col < g.N) g.sums[col] += t;
    }
  }
  f32x4 v[NV];  // [row part][column part]
  auto gather = [&](auto half_c) {
    constexpr int I = TM * decltype(half_c)::value;
#pragma unroll
    for (int q = 0; q < NV; q++) v[q] = acc[I + q / CB][q % CB] + xch[((wave ^ 4) * NV + q) * 64 + lane];
  };
  u32x2 w[EPI == EPI_BF16_DELTA ? NV : 1] = {};  // EPI_BF16_DELTA: dO as it is stored
  auto finish = [&](auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
#pragma unroll
    for (int i = 0; i < TM; i++) {
      const int row = row0 + 16 * (TM * wk + i);
      if constexpr (EPI == EPI_SWIGLU) {
        epi_swiglu16<FULL>(g, row, col0, lane, v[i * CB], v[i * CB + 1], v[i * CB + 2], v[i * CB + 3]);
      } else if constexpr (EPI == EPI_BF16_DELTA) {
        const int r = row + (lane & 15);
        if (!FULL && r >= g.M) continue;
#pragma unroll
        for (int j = 0; j < CB; j++) {
          const int col = col0 + 16 * j + 4 * (lane >> 4);
          if (!FULL && col >= g.N) continue;
          const f32x4& x = v[i * CB + j];
          w[i * CB + j] = u32x2{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])};
          *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(g.C) + (size_t)r * g.ldc + col) = w[i * CB + j];
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; j++) epi_finish16<EPI, FULL>(g, row, col0 + 32 * j, lane, v[i * CB + 2 * j], v[i * CB + 2 * j + 1], pre[i][j]);
      }
    }
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  if constexpr (SLICED) {
    static_assert(StLds<TM, TN, NS>::kExchange < StLds<TM, TN, NS>::bytes, "four bytes behind the exchange");
    if (wk == 0) gather(H0{}); else gather(H1{});
    if (!sum_slices<NV>(ss, v, lds + StLds<TM, TN, NS>::kExchange)) return;
  } else {
    if (wk == 0) gather(H0{}); else gather(H1{});
  }
  if (m0 + BM <= g.M && n0 + BN <= g.N && (!epi_rows(EPI) || g.ldc <= kLdcOfLines)) finish(std::true_type{}); else finish(std::false_type{});
  // The sums of a row, in the order of 32x32 accumulators: in each of 32 columns the four chains of columns 16 H + 4 b ..+3, +8 (H, b = 0, 1), which run on
  // through the wave's parts of 32; then both b, both H and both waves of a head (which hold its column parts, one each where a head is 64 columns of a
  // 128-wide tile), these by way of LDS.  A lane of the upper half holds the +8 of the lane 32 below it, whose chain it goes on with.
  if constexpr (EPI == EPI_BF16_DELTA) {
    constexpr int at = StLds<TM, TN, NS>::kExchange + 1024;
    static_assert(at + BM * 16 <= StLds<TM, TN, NS>::bytes, "row sums behind the exchange");
    float* red = reinterpret_cast<float*>(lds + at);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int H = 0; H < 2; H++) {
        auto chain = [&](float s) {
#pragma unroll
          for (int j = 0; j < TN; j++)
#pragma unroll
            for (int k = 0; k < 2; k++) {
              const uint32_t x = w[i * CB + 2 * j + H][k], o = pre[i][j][H].a[k];
              s += bf16_bits_to_f32(x & 0xffffu) * bf16_bits_to_f32(o & 0xffffu);
              s += bf16_bits_to_f32(x >> 16) * bf16_bits_to_f32(o >> 16);
            }
          return s;
        };
        const float below = __shfl_xor(chain(0.f), 32, 64);
        float s = chain(lane < 32 ? 0.f : below);
        s += __shfl_xor(s, 16, 64);
        if ((lane & 48) == 32) red[4 * (wm * 32 * TM + 16 * (TM * wk + i) + (lane & 15)) + 2 * wn + H] = s;
      }
    __syncthreads();
    const int r = tid % BM, part = tid / BM;  // a head is 64 columns (one column part of a 128-wide tile) or all columns of the tile
    const bool one = g.head_dim == BN;
    const int row = m0 + r, head = n0 / g.head_dim + part, heads = g.N / g.head_dim;
    if (part < (one ? 1 : 2) && row < g.M && head < heads) {
      const float* p = red + 4 * r + 2 * part;
      g.sums[((size_t)(row / g.seq) * heads + head) * g.seq + row % g.seq] = one ? (p[0] + p[1]) + (p[2] + p[3]) : p[0] + p[1];
    }
  }
}

template <int TM, int TN, int NS, bool A_KC, bool B_KC, int EPI, bool SLICED, class G>
__global__ __launch_bounds__(512) void gemm_st_kernel(G g) {  // by value, adjusted per k slice
  __shared__ __attribute__((aligned(1024))) char lds[StLds<TM, TN, NS>::bytes];
  int pid = blockIdx.x;
  SliceSum ss{};
  if (SLICED || g.ksplit > 1) ss = take_slice<A_KC, B_KC, SLICED>(g, pid, 64 * TM * 64 * TN);
  st_tile<TM, TN, NS, A_KC, B_KC, EPI, false, SLICED>(g, pid, lds, ss);
}

// two weight gradients over the same K rows, tiles of the second behind those of the first
template <int TN, int NS>
__global__ __launch_bounds__(512) void gemm_st_group_kernel(GemmCall g0, GemmCall g1) {
  __shared__ __attribute__((aligned(1024))) char lds[StLds<1, TN, NS>::bytes];
  const int first = g0.tiles_m * g0.tiles_n;
  const bool second = (int)blockIdx.x >= first;
  const GemmCall g = second ? g1 : g0;
  st_tile<1, TN, NS, false, false, EPI_ACC_F32, true>(g, second ? blockIdx.x - first : blockIdx.x, lds);
}

// split-K second pass: C = epilogue(sum over slices of the fp32 partial planes), slices added in index order
template <int EPI>
__global__ __launch_bounds__(256) void splitk_fixup_kernel(const float* __restrict__ part, int S, GemmArgs g) {
  const int nc4 = g.N >> 2;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)g.M * nc4) return;
  const int row = (int)(idx / nc4), col = (int)(idx % nc4) * 4;
  const size_t plane = (size_t)g.M * g.N;
  f32x4 v = *reinterpret_cast<const f32x4*>(part + (size_t)row * g.N + col);
  for (int s2 = 1; s2 < S; s2++) v += *reinterpret_cast<const f32x4*>(part + s2 * plane + (size_t)row * g.N + col);
  epi_apply<EPI>(g, row, col, v, epi_load<EPI>(g, row, col));
}

template <int BM, int BN, int WGM, int WGN, int WGK, bool A_KC, bool B_KC, int EPI>
int launch_one(const GemmArgs& g0, int ksplit, float* ws, hipStream_t s) {
  GemmArgs g = g0;
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = (g.N + BN - 1) / BN;
  g.ksplit = 1;
  g.k_per = g.K;
  dim3 block(64 * WGM * WGN * WGK);
  if (ksplit <= 1) {
    hipLaunchKernelGGL((gemm_kernel<BM, BN, WGM, WGN, WGK, A_KC, B_KC, EPI>), dim3(g.tiles_m * g.tiles_n), block, 0, s, g);
    OASES_LAUNCH_CHECK("gemm_kernel");
    return 0;
  }
  // first pass: fp32 partial planes [ksplit][M][N] in the workspace; second pass: sum + the real epilogue
  if (!ws) { set_error("gemm: split-K chosen without a workspace"); return OASES_ENULL; }
  if (EPI == EPI_SWIGLU || EPI == EPI_DSWIGLU) { set_error("gemm: the SwiGLU epilogues do not run over k slices"); return OASES_EINVAL; }
  GemmArgs p = g;
  p.ksplit = ksplit;
  p.k_per = ((g.K + ksplit - 1) / ksplit + BK - 1) / BK * BK;
  p.C = ws;
  p.ldc = g.N;
  hipLaunchKernelGGL((gemm_kernel<BM, BN, WGM, WGN, WGK, A_KC, B_KC, EPI_F32>), dim3(g.tiles_m * g.tiles_n * ksplit), block, 0, s, p);
  OASES_LAUNCH_CHECK("gemm_kernel (split-K)");
  const long n4 = (long)g.M * (g.N / 4);
  hipLaunchKernelGGL((splitk_fixup_kernel<EPI>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, ws, ksplit, g);
  OASES_LAUNCH_CHECK("splitk_fixup_kernel");
  return 0;
}

// Whether a launch of a pass adds up its own k slices, or a second launch does: the last workgroup of a tile reads the other slices' sums at some
// 47 GB/s; a second launch costs 6 to 9 us inside a step.  us, own -> two launches: inside a step 400 x 2560 x 5120 over three of 128x128 25.3 -> 30,
// 256 x 256 x 12600 TN over eight of 64x64 14 -> 17; four of 128x128 128 x 6144 x 12288 56 -> 46 + 5.4, NT 75 -> 66 + 6.1 (19 steps 0 to 2 % shorter); over four
// of 128x256 forward pass of three layers with 400 x 4096 x 8192 519 -> 508, of two with 304 x 3840 x 10240 and 304 x 5120 x 10240 468 -> 449, of
// one with 160 x 5632 x 11264 207 -> 198; over two of 128x256 the two are within 1 % of a step (24 of them).
inline bool own_slices(int slices, int bm, int bn) { return (slices - 1) * bm * bn * 4 <= 128 << 10; }
inline int st_k_per(int K, int slices) { return ((K + slices - 1) / slices + BKS - 1) / BKS * BKS; }  // k of one slice

template <int TM, int TN, int NS, bool A_KC, bool B_KC, int EPI>
int launch_small(const GemmCall& g0, int ksplit, float* ws, size_t ws_bytes, hipStream_t s) {
  GemmCall g = g0;
  g.tiles_m = (g.M + 64 * TM - 1) / (64 * TM);
  g.tiles_n = (g.N + 64 * TN - 1) / (64 * TN);
  using G = std::conditional_t<EPI == EPI_BF16_DELTA, GemmCall, GemmArgs>;
  if (ksplit <= 1) {
    hipLaunchKernelGGL((gemm_st_kernel<TM, TN, NS, A_KC, B_KC, EPI, false, G>), dim3(g.tiles_m * g.tiles_n), dim3(512), 0, s, g);
    OASES_LAUNCH_CHECK("gemm_st_kernel");
    return 0;
  }
  const size_t T = (size_t)g.tiles_m * g.tiles_n;
  if constexpr (EPI != EPI_SWIGLU && EPI != EPI_DSWIGLU)
    if (g.counters && ws && (EPI == EPI_BF16_DELTA || own_slices(ksplit, 64 * TM, 64 * TN)) && T <= kSliceCounters && T * ksplit * (64 * TM * 64 * TN * 4) <= ws_bytes) {
      g.ksplit = ksplit;
      g.k_per = st_k_per(g.K, ksplit);
      g.part = ws;
      hipLaunchKernelGGL((gemm_st_kernel<TM, TN, NS, A_KC, B_KC, EPI, true, GemmCall>), dim3(g.tiles_m * g.tiles_n * ksplit), dim3(512), 0, s, g);
      OASES_LAUNCH_CHECK("gemm_st_kernel (slices)");
      return 0;
    }
  if constexpr (EPI == EPI_SWIGLU || EPI == EPI_DSWIGLU || EPI == EPI_BF16_DELTA) {
    set_error("gemm: an epilogue that pairs columns does not run over k slices of two launches");
    return OASES_EINVAL;
  } else {
    if (!ws) { set_error("gemm: split-K chosen without a workspace"); return OASES_ENULL; }
    GemmArgs p = g;
    p.ksplit = ksplit;
    p.k_per = st_k_per(g.K, ksplit);
    p.C = ws;
    p.ldc = g.N;
    hipLaunchKernelGGL((gemm_st_kernel<TM, TN, NS, A_KC, B_KC, EPI_F32, false, GemmArgs>), dim3(g.tiles_m * g.tiles_n * ksplit), dim3(512), 0, s, p);
    OASES_LAUNCH_CHECK("gemm_st_kernel (split-K)");
    const long n4 = (long)g.M * (g.N / 4);
    hipLaunchKernelGGL((splitk_fixup_kernel<EPI>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, ws, ksplit, g);
    OASES_LAUNCH_CHECK("splitk_fixup_kernel");
    return 0;
  }
}

// Tile and split-K choice by a small time model.  What it chooses settles the order in which the fp32 terms of an output element are added: a 256x256 tile
// and the square register-staged one run through k in one chain, the others (the k halves of 64) in two, every k slice in one or two of its own, and fewer chains round worse
// (rms against 64 bits over 8192 rows 5.7e-7 with one, 4.0e-7 with two).  So its rates stay the ones that the results were fixed with: another kernel for
// a shape is taken where it adds in the same order (same_sums).  Bigger tiles run closer to the MFMA rate (fewer LDS bytes per flop)
// but a launch only uses the chip well if its workgroup count is near a multiple of the 256 CUs; splitting K multiplies
// the workgroup count at the price of a second pass over fp32 partial planes.  Rates measured on this part.
struct TileChoice { int bm, bn, ksplit; bool wave_ksplit; bool dtl = false; bool pp = false; bool st = false; };  // st: the small-tile kernel; pp: the eight-wave kernel of a direct-to-LDS tile shape
// per kind of contraction (0: NN, 1: NT, 2: TN, 3: NN with the bias+GeLU epilogue): whether the rectangular tiles
// split k between waves, and the sustained rates of the four block tiles
// Shapes the direct-to-LDS kernels cover, per kind of contraction (0, 3: NN, 1: NT, 2: TN): whole k tiles; in the
// 256 x 256 kernel a k-major operand must fill its tiles and a row-indexed one (A of TN; B of NN and TN) may end inside
// its last tile; in the 128 x 256 kernel both may.
bool dtl_fits(int kind, int M, int N, int K) {
  return (kind == 2 || M % 256 == 0) && (kind != 1 || N % 256 == 0) && M % 8 == 0 && N % 8 == 0 && K % BKD == 0 && K >= BKD;
}
bool dtl_rect_fits(int kind, int M, int N, int K) {  // the 128 x 256 kernel redirects rows of a k-major operand too
  (void)kind;
  return M % 8 == 0 && N % 8 == 0 && K % BKR == 0 && K >= BKR;
}
// The eight-wave kernel also takes weight gradients over any number of rows from 1024 on, which have a name of their own (W = 6): the others keep to the
// bounds above and refuse what lies outside.  Fewer than 1024 rows stay on small tiles: 2560 x 5120 x 808 60 us.
bool pp128_fits(int kind, int M, int N, int K) { return dtl_rect_fits(kind, M, N, K) || (kind == 2 && M % 8 == 0 && N % 8 == 0 && K % 8 == 0 && K >= 1024); }
bool dtl_rect_whole(int M, int N, int K) { return M % 128 == 0 && N % 256 == 0 && K % BKR == 0 && K >= BKR; }
bool rect_slices_whole(int kind, int M, int N, int K, int S) { return K % (S * BKR) == 0 && dtl_rect_fits(kind, M, N, K / S); }
bool pp_slices_fit(int kind, int M, int N, int K, int S) {  // S k slices of whole stages; a weight gradient's last one may be shorter
  if (S == 1) return pp128_fits(kind, M, N, K);
  return (kind == 2 && K >= 1024 * S && dtl_rect_fits(kind, M, N, K)) || rect_slices_whole(kind, M, N, K, S);
}
struct KindTable { bool wave_ksplit; float r256x256, r128x256, r256x128, r128x128; };
const KindTable g_kinds[4] = {{true, 1200.f, 1080.f, 960.f, 740.f}, {true, 1200.f, 1080.f, 960.f, 740.f},
                        {true, 1200.f, 1080.f, 960.f, 740.f}, {false, 1200.f, 1080.f, 900.f, 740.f}};
TileChoice pick_large_tile(int kind, int epi, int M, int N, int K, size_t ws_bytes) {
  const KindTable& kt = g_kinds[kind];
  // Tiles that the direct-to-LDS kernels do not cover run on the register-staged kernels.  256x256: at three quarters of their rate (NT dSwiGLU 8192 x
  // 1376 x 4096: 138 us against 133 on 128x256 tiles, which may be ragged, 9984 x 2624 x 1600 153 against 138, NT 8656 x 1984 x 1344 76 against 60).  128x256
  // where k is no whole number of stages: at half (NN 9576 x 1536 x 1376: 81 us, 62 on 256x256); TN at 700 and 740 (2560 x 5120 x 808: 256x256 75 us,
  // 128x256 75, 64x128 60).
  const bool rect = dtl_rect_fits(kind, M, N, K);
  const float r128 = rect ? kt.r128x256 : kind == 2 ? 740.f : 650.f, r256x128 = rect ? kt.r256x128 : kind == 2 ? 740.f : 600.f;
  const struct { int bm, bn; float tflops; } cand[] = {{256, 256, kt.r256x256}, {128, 256, r128}, {256, 128, r256x128}, {128, 128, kt.r128x128}};
  TileChoice best{128, 128, 1, kt.wave_ksplit};
  double best_t = 1e30;
  for (auto& c : cand) {
    const long tm = (M + c.bm - 1) / c.bm, tn = (N + c.bn - 1) / c.bn;
    for (int S = 1; S <= 8; S *= 2) {
      if (S > 1 && ((size_t)S * M * N * 4 > ws_bytes || K / S < 512)) break;
      const long wgs = tm * tn * S, rounds = (wgs + 255) / 256;
      // time of one workgroup's tile slice at the tile's rate (one workgroup per CU), times the number of rounds
      const double tflops = c.bm == 256 && c.bn == 256 && !(S == 1 && dtl_fits(kind, M, N, K)) ? (kind == 2 ? 700.f : 900.f) : c.tflops;
      double t = (double)rounds * (2.0 * c.bm * c.bn * ((double)K / S) + 3.0e6) / (tflops * 1e12 / 256.0);
      if (S > 1) t += ((double)(2 * S + 1) * M * N * 4.0) / 3.0e12 + 4e-6;
      if (t < best_t) { best_t = t; best = TileChoice{c.bm, c.bn, S, kt.wave_ksplit}; }
    }
  }
  // Whole tiles without k slices: the eight-wave direct-to-LDS kernels, which measure faster than the four-wave and the
  // register-staged kernels of the same tile on every shape of the two full-size workloads (cold operands, 3-15 %).
  if (best.ksplit == 1) {
    if (best.bm == 256 && best.bn == 256 && dtl_fits(kind, M, N, K)) best.dtl = best.pp = true;
    if (best.bm == 128 && best.bn == 256 && dtl_rect_fits(kind, M, N, K)) best = TileChoice{128, 256, 1, true, true, true};
    // Few rows, long k (a sub-batch of 1024 rows against K = 8192): 128 x 128 tiles fill the chip but run at the small
    // tile's rate; the 128 x 256 direct-to-LDS kernel over two k slices fills it too, and is faster even with its second
    // pass (measured on cold operands: 87-93 us against 108-116 us).
    const long rtiles = (long)((M + 127) / 128) * ((N + 255) / 256);
    if (best.bm == 128 && best.bn == 128 && epi != EPI_SWIGLU && epi != EPI_DSWIGLU && 2 * rtiles >= 192 && 2 * rtiles <= 256 && K >= 4096 &&
        K % (2 * BKR) == 0 && dtl_rect_fits(kind, M, N, K / 2) && (size_t)2 * M * N * 4 <= ws_bytes)
      best = TileChoice{128, 256, 2, true, true, true};
  } else if (best.bm == 128 && best.bn == 256 && (best.ksplit == 2 || best.ksplit == 4) && epi != EPI_SWIGLU && epi != EPI_DSWIGLU &&
             rect_slices_whole(kind, M, N, K, best.ksplit)) {
    best = TileChoice{128, 256, best.ksplit, true, true, true};  // k slices of whole stages: the eight-wave kernel
  }
  return best;
}

// Time of an eight-wave launch over wgs workgroups, seconds.  What the MFMA loops are bound by is the power they draw together, so a
// round that leaves CUs idle runs its stages faster, down to three quarters of the time of a full one (128x256 tiles, a 64-wide
// stage: 256 workgroups 0.9 us, 144 or fewer 0.68); the output, read and written, moves at 4 TB/s.
double pp_seconds(long wgs, int k_per, double out_bytes, double stage) {
  double t = out_bytes / 4.0e12;
  for (; wgs > 0; wgs -= 256) t += 4.0e-6 + k_per / 64 * stage * std::max(0.75, (double)std::min(wgs, 256L) / 256.0);
  return t;
}
constexpr double kStage256 = 1.75e-6, kStage128 = 0.9e-6;  // of the model
double pp_seconds(int bm, long wgs, int k_per, double out_bytes) { return pp_seconds(wgs, k_per, out_bytes, bm == 256 ? kStage256 : kStage128); }
// today's time of a weight gradient on 128x256 tiles without k slices
double pp128_seconds(long tiles, int K, double out_bytes) { return pp_seconds(tiles, K, out_bytes, 0.83e-6); }

// Small tiles against the choice above, by the same kind of model (measured on this part): a launch costs 2.9 us, a
// workgroup 0.225 us (64 x 64) or 0.335 us (64 x 128) per 64-wide stage of its slice, two workgroups on a CU take turns at the
// LDS, so the busiest CU's workgroups add up; the output moves at 4 TB/s (3.1 TB/s with the large tiles, one workgroup per
// CU: nothing covers the latency of its read-modify-write); k slices cost a second launch and their planes.  The
// eight-wave kernels run better than the model on long k, so they give way only to a tenth less; the register-staged ones
// wait out two more memory latencies, 2 us, before the first product.  Both sides measured,
// us, large tile -> small: 4096 x 1536 x 2048 NN bias 31.6 -> 34.8 (stays large), 1024 x 3072 x 8192 56.2 -> 71.6 (stays
// large), 4096 x 512 x 4096 NT 29.8 -> 22.9, 1024 x 1024 x 4096 TN 21.4 -> 16.9, 64 x 4608 x 12288 NN 53.5 -> 34.8,
// 6144 x 12288 x 128 TN 195 -> 152.  Slices of 8192 k and more stay with the large tiles.
// own_sum: a call of a pass, whose launches add up a few slices by themselves (SliceSum, own_slices): the last workgroup of a tile then reads the other
// slices' sums, one after the other at some 47 GB/s, instead of a second launch; 128x128 tiles on the same scheme are candidates, with any
// number of slices (0.6 us a stage, 0.85 of that where 218 and fewer workgroups leave CUs idle and the others more of the power; what TN reads and writes moves at
// 3.4 TB/s from the second round on, since a CU holds one workgroup: 10240 x 3840 x 208 92 us on 64x128, 118 on 128x128).  Measured, us, the choice without -> with, second launches
// included: inside a step 128 x 4608 x 12288 NN 52 -> 45 (register-staged kernel over eight slices -> 128x128 over six), NT 128 x 6144 x 12288 79 -> 71 (over five); 512 x 8192 x 3072 NT 47 -> 36, 8192 x 512 x
// 2048 NT 31 -> 26, 200 x 3072 x 8192 36 -> 27; 1488 x 3072 x 3072 NN stays on 144 tiles of 128x256 (40; 64x128 over two slices 72).
TileChoice pick_tile(int kind, int epi, int M, int N, int K, size_t ws_bytes, double* seconds = nullptr, bool own_sum = false, int bn_min = 0) {
  const TileChoice large = pick_large_tile(kind, epi, M, N, K, ws_bytes);
  const KindTable& kt = g_kinds[kind];
  const double out = (double)M * N * (epi == EPI_F32 ? 4.0 : kind == 2 ? 8.0 : epi == EPI_SWIGLU ? 3.0 : epi == EPI_DSWIGLU ? 8.0 : epi == EPI_BIAS_GELU || epi == EPI_DGELU ? 4.0 : 2.0);
  auto tiles = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  // a second launch: 3.2 us by itself; in a pass (see own_slices) 6.2, behind 128x256 tiles 9.  At 6.5 there 400 x 4096 x 8192 goes to four slices of
  // 128x256, 508 us for that pass, 490 on two of 128x128; at 9 behind 128x128 tiles, too, six of 18 passes take 2 to 4 % more.
  auto slices = [&](int S, int bm, int bn) {
    const bool own = own_sum && (bn_min || own_slices(S, bm, bn));
    return S <= 1 ? 0.0 : 2.0 * S * M * N * 4.0 / 6.0e12 + (own ? 2.0e-6 + (S - 1) * bm * bn * 4.0 / 47.0e9 : own_sum ? (bm * bn > 128 * 128 ? 9.0e-6 : 6.2e-6) : 3.2e-6);
  };
  auto room = [&](int S, int bm, int bn) {  // partial sums and counters of slices that the launch adds up
    return S <= 1 || (tiles(bm, bn) <= kSliceCounters && (size_t)tiles(bm, bn) * S * bm * bn * 4 <= ws_bytes);
  };
  // (in a pass the register-staged 128x256 kernel, over slices that are no whole stages, runs at its own rate: 208 x 7168 x 4800 over four 43 us, not 36)
  const double rate = large.bm == 256 && large.bn == 256 ? kt.r256x256 : large.bm == 256 ? kt.r256x128 : large.bn == 256 ? (own_sum && !large.pp ? 650.f : kt.r128x256) : kt.r128x128;
  const long wgs = (long)((M + large.bm - 1) / large.bm) * ((N + large.bn - 1) / large.bn) * large.ksplit;
  double best_t = (double)((wgs + 255) / 256) * (2.0 * large.bm * large.bn * ((double)K / large.ksplit) + 3.0e6) / (rate * 1e12 / 256.0) +
                  out / 3.1e12 + slices(large.ksplit, 128, 256);
  if (large.pp) best_t *= 0.9; else best_t += 2.0e-6;
  if (own_sum && large.pp) best_t = pp_seconds(large.bm, wgs, K / large.ksplit, out) + slices(large.ksplit, 128, 256);
  if (bn_min) best_t = 1e30;  // the small-tile kernels alone
  TileChoice best = large;
  // Weights that no cache keeps are read once per row of tiles: not on 64-row tiles when there are more rows and k can be sliced, which 128-row tiles
  // need to fill the chip.  The model has no term for weight bytes.  us, 64 -> 128 rows: 128 x 4608 x 12288 (113 MB) NN 51 -> 39, NT 48 -> 42, 128 x 4800 x
  // 7168 (69 MB) 32 -> 27, 208 x 7168 x 4800 38 -> 34; below, 128 x 3072 x 8192 (50 MB) 25 -> 27.  The SwiGLU epilogues, which take no slices: 128 x
  // 4800 x 7168 53 -> 67, its gradient 38 -> 77.
  const bool streams = own_sum && kind != 2 && M > 64 && 2.0 * N * K > 64.0e6 && epi != EPI_SWIGLU && epi != EPI_DSWIGLU;
  for (int bn = epi == EPI_SWIGLU || bn_min == 128 ? 128 : 64; bn <= 128; bn += 64)
    for (int S = 1; S <= 16; S *= 2) {
      const int k_per = st_k_per(K, S);
      if (S > 1 && ((size_t)S * M * N * 4 > ws_bytes || k_per < 2 * BKS || (long)(S - 1) * k_per >= K)) break;
      if (k_per >= 8192 || streams || (own_sum && !room(S, 64, bn))) continue;
      const long wgs = tiles(64, bn) * S, per_cu = (wgs + 255) / 256;
      const double t = 2.9e-6 + (double)per_cu * ((k_per + BKS - 1) / BKS) * (bn == 64 ? 0.225e-6 : 0.335e-6) + out / 4.0e12 + slices(S, 64, bn);
      if (t < best_t) {
        best_t = t;
        best = TileChoice{64, bn, S, true};
        best.st = true;
      }
    }
  if (own_sum)
    for (int S = 1; S <= 16; S++) {
      const int k_per = st_k_per(K, S);
      if (S > 1 && (!room(S, 128, 128) || k_per < 2 * BKS || (long)(S - 1) * k_per >= K)) break;
      const long wgs = tiles(128, 128) * S;
      const double t = 4.0e-6 + (double)((wgs + 255) / 256) * ((k_per + BKS - 1) / BKS) * 0.6e-6 * (wgs < 218 ? 0.85 : 1.0) + out / (kind == 2 && wgs > 256 ? 3.4e12 : 4.0e12) + slices(S, 128, 128);
      if (t < best_t) {
        best_t = t;
        best = TileChoice{128, 128, S, true};
        best.st = true;
      }
    }
  if (seconds) *seconds = best_t;
  return best;
}

// The kernel for the sums that the model has chosen: the 128x256 eight-wave kernel adds as the register-staged ones of 128x256 and (waves that split k) 256x128
// tiles and the small tiles do, and takes shapes that the model does not price it for.  seconds: the model's, of its choice.
//   Weight gradients over any number of rows, us, cold operands: register-staged -> this one 12336 x 472 x 1064 54 -> 40, over two slices 11544 x 144 x 4928 88 -> 58,
// four 5728 x 168 x 6720 65 -> 46; the better small tiles -> this one 6144 x 3072 x 7240 357 -> 309, 4096 x 4096 x 1992 108 -> 93, 3072 x 3072 x 2920 98 -> 87, 2560 x
// 2560 x 2056 57 -> 47, with 184 tiles 11736 x 288 x 1112 38 -> 35; with fewer the chip is left too empty: 122 (15544 x 136 x 1248) 26 -> 32, 110 (6928 x 408 x 1240) 26 -> 36.
//   256x128 tiles, which fill their last round better, at long k: NT 7040 x 3456 x 3456 251 -> 191, dGeLU 14544 x 2176 x 5120 435 -> 354, NN 8648 x 4736 x 4096 377 -> 313, TN
// 14280 x 1600 x 5568 374 -> 328; TN 12984 x 576 x 1280 56 -> 56, NT dGeLU 8232 x 832 x 768 36 -> 43, NN bias 9056 x 896 x 384 21 -> 24.
constexpr long kPpLeastTiles = 160;
TileChoice same_sums(const TileChoice& t, double seconds, int kind, int M, int N, int K) {
  if (t.pp) return t;
  const TileChoice pp{128, 256, t.ksplit, true, true, true};
  const long tiles = (long)((M + 127) / 128) * ((N + 255) / 256);
  bool takes;
  if (t.st) takes = kind == 2 && t.ksplit == 1 && K % BKR && pp128_fits(kind, M, N, K) && tiles >= kPpLeastTiles && pp128_seconds(tiles, K, 8.0 * M * N) < seconds;
  else if (t.bm == 128 && t.bn == 256) takes = kind == 2 && (t.ksplit == 1 || t.ksplit == 2 || t.ksplit == 4) && pp_slices_fit(kind, M, N, K, t.ksplit);
  else takes = t.bm == 256 && t.bn == 128 && t.wave_ksplit && t.ksplit == 1 && K >= 2048 && pp128_fits(kind, M, N, K);
  return takes ? pp : t;
}

int encode_variant(const TileChoice& t, int kind, int M, int N, int K) {
  const bool rect = t.bm != t.bn, any_rows = t.pp && t.bm == 128 && !rect_slices_whole(kind, M, N, K, t.ksplit);
  return (t.st ? (t.bm == 128 ? 500000000 : 400000000) : t.dtl ? (any_rows ? 600000000 : t.pp ? 300000000 : 200000000) : rect && t.wave_ksplit ? 100000000 : 0) +
         t.ksplit * 1000000 + t.bm * 1000 + t.bn;
}
// variant -> TileChoice; false if no such instantiation exists or the k slices do not fit the problem / workspace
bool decode_variant(int variant, int kind, int M, int N, int K, size_t ws_bytes, TileChoice* t) {
  if (variant <= 0) return false;
  const int wk = variant / 100000000, S = variant / 1000000 % 100, bm = variant / 1000 % 1000, bn = variant % 1000;
  const bool square = (bm == 256 && bn == 256) || (bm == 128 && bn == 128), rect = (bm == 256 && bn == 128) || (bm == 128 && bn == 256);
  if ((wk == 2 || wk == 3) && S == 1) {  // direct-to-LDS kernels (3: eight waves), one k slice
    if (bm == 256 && bn == 256 && dtl_fits(kind, M, N, K)) { *t = TileChoice{256, 256, 1, false, true, wk == 3}; return true; }
    if (bm == 128 && bn == 256 && dtl_rect_fits(kind, M, N, K)) { *t = TileChoice{128, 256, 1, true, true, wk == 3}; return true; }
    return false;
  }
  if ((wk == 2 || wk == 3) && bm == 128 && bn == 256 && (S == 2 || S == 4)) {  // the 128 x 256 kernels over k slices of whole stages
    if (!rect_slices_whole(kind, M, N, K, S) || (size_t)S * M * N * 4 > ws_bytes) return false;
    *t = TileChoice{128, 256, S, true, true, wk == 3};
    return true;
  }
  if (wk == 6) {  // the eight-wave 128 x 256 kernel on weight gradients over any number of rows
    if (kind != 2 || bm != 128 || bn != 256 || (S != 1 && S != 2 && S != 4) || !pp_slices_fit(kind, M, N, K, S) || (S > 1 && (size_t)S * M * N * 4 > ws_bytes)) return false;
    *t = TileChoice{128, 256, S, true, true, true};
    return true;
  }
  if (wk >= 4) {  // small tiles; k slices of whole stages that all start inside K
    const bool tile = (wk == 4 && bm == 64 && (bn == 64 || bn == 128)) || (wk == 5 && bm == 128 && bn == 128);
    if (!tile || S < 1 || S > 16) return false;
    if (S > 1 && ((size_t)S * M * N * 4 > ws_bytes || (long)(S - 1) * st_k_per(K, S) >= K)) return false;
    *t = TileChoice{bm, bn, S, true};
    t->st = true;
    return true;
  }
  if (wk > 1 || !(square || rect) || (wk == 1 && !rect) || S < 1 || S > 8) return false;
  if (S > 1) {
    const int k_per = ((K + S - 1) / S + BK - 1) / BK * BK;
    if ((size_t)S * M * N * 4 > ws_bytes || (long)(S - 1) * k_per >= K) return false;
  }
  *t = TileChoice{bm, bn, S, wk == 1};
  return true;
}

template <bool A_KC, bool B_KC, int EPI>
int launch_shape(const GemmCall& g, float* ws, size_t ws_bytes, int forced_variant, int choice_rows, hipStream_t s) {
  constexpr int kind = !A_KC ? 2 : B_KC ? 1 : (EPI == EPI_BIAS_GELU || EPI == EPI_SWIGLU) ? 3 : 0;
  if (EPI == EPI_SWIGLU || EPI == EPI_DSWIGLU) ws_bytes = 0;  // their epilogues pair columns: no second pass over partial planes
  TileChoice t;
  if (forced_variant == 0) {
    // Pinned choice: the number of k slices and whether waves split k -- the two things that set the order in which the
    // fp32 terms of an output element are added -- come from (choice_rows, N, K, epilogue), so every launch over a part of
    // those rows adds in the same order.  The 256 x 256 direct-to-LDS kernels need whole row tiles; a part that has none
    // runs the staged kernel of the same tile, which adds in the same order.
    const bool pinned = kind != 2 && choice_rows > g.M;
    const int rows = pinned ? choice_rows : g.M;
    double seconds;
    t = pick_tile(kind, EPI, rows, g.N, g.K, ws ? ws_bytes : 0, &seconds, g.counters != nullptr);
    if (gemm_span_fits(A_KC ? rows : g.K, g.lda) && gemm_span_fits(B_KC ? g.N : g.K, g.ldb)) t = same_sums(t, seconds, kind, rows, g.N, g.K);
    if (pinned && t.dtl && t.bm == 256 && !dtl_fits(kind, g.M, g.N, g.K)) t.dtl = t.pp = false;
    if ((t.dtl || t.st) && !(gemm_span_fits(A_KC ? rows : g.K, g.lda) && gemm_span_fits(B_KC ? g.N : g.K, g.ldb))) {
      if (t.st) t = pick_large_tile(kind, EPI, rows, g.N, g.K, ws ? ws_bytes : 0);
      t.dtl = t.pp = false;
    }
#ifdef OASES_GEMM_TUNE_HOOK
    {  // tuning aid (not compiled into the library): OASES_GEMM_TUNE="kind:epi:M:N:K=variant;..." overrides the choice
      static const char* tune = getenv("OASES_GEMM_TUNE");
      if (tune) {
        char key[96];
        snprintf(key, sizeof key, "%d:%d:%d:%d:%d=", kind, (int)EPI, g.M, g.N, g.K);
        const char* hit = strstr(tune, key);
        TileChoice tt;
        if (hit && decode_variant(atoi(hit + strlen(key)), kind, g.M, g.N, g.K, ws ? ws_bytes : 0, &tt)) t = tt;
      }
    }
#endif
  } else if (!decode_variant(forced_variant, kind, g.M, g.N, g.K, ws ? ws_bytes : 0, &t)) {
    set_error("gemm: variant %d does not exist or does not fit M=%d N=%d K=%d with %zu workspace bytes", forced_variant, g.M, g.N, g.K, ws ? ws_bytes : (size_t)0);
    return OASES_EINVAL;
  } else if ((t.dtl || t.st) && !(gemm_span_fits(A_KC ? g.M : g.K, g.lda) && gemm_span_fits(B_KC ? g.N : g.K, g.ldb))) {
    set_error("gemm: variant %d (direct-to-LDS) needs operands that span less than 2 GiB (lda=%d ldb=%d)", forced_variant, g.lda, g.ldb);
    return OASES_EINVAL;
  }
  if (t.st) {
    if (t.bm == 128) return launch_small<2, 2, 4, A_KC, B_KC, EPI>(g, t.ksplit, ws, ws_bytes, s);
    if (t.bn == 128) return launch_small<1, 2, 3, A_KC, B_KC, EPI>(g, t.ksplit, ws, ws_bytes, s);
    if constexpr (EPI != EPI_SWIGLU) return launch_small<1, 1, 5, A_KC, B_KC, EPI>(g, t.ksplit, ws, ws_bytes, s);
    set_error("gemm: the 64x64 kernel has no SwiGLU epilogue");
    return OASES_EINVAL;
  }
  constexpr bool kLines = epi_rows(EPI);
  if (kLines && t.pp && t.bm == 256 && A_KC && B_KC && g.ldc > kLdcOfLines) t.dtl = t.pp = false;  // no form that checks its bounds: the staged kernel of the same tile
  if (t.dtl && t.pp) {
    constexpr bool kCanBeRagged = !A_KC || !B_KC;
    const int bm = t.bm;
    GemmCall d = g;
    d.tiles_m = (g.M + bm - 1) / bm;
    d.tiles_n = (g.N + 255) / 256;
    const bool tiles = g.M % bm == 0 && g.N % 256 == 0, whole = tiles && (!kLines || g.ldc <= kLdcOfLines);
    if (!tiles && bm == 256 && !kCanBeRagged) { set_error("gemm: direct-to-LDS kernel on a shape it does not cover"); return OASES_EINVAL; }
    if (bm == 128 && t.ksplit > 1) {
      if constexpr (EPI == EPI_SWIGLU || EPI == EPI_DSWIGLU) {
        set_error("gemm: the SwiGLU epilogues do not run over k slices");
        return OASES_EINVAL;
      } else {
        if (!ws) { set_error("gemm: split-K chosen without a workspace"); return OASES_ENULL; }
        GemmCall p = d;
        p.ksplit = t.ksplit;
        p.k_per = st_k_per(g.K, t.ksplit);
        const dim3 sgrid(d.tiles_m * d.tiles_n * t.ksplit);
        if (g.counters && own_slices(t.ksplit, 128, 256) && d.tiles_m * d.tiles_n <= kSliceCounters && (size_t)d.tiles_m * d.tiles_n * t.ksplit * 128 * 256 * 4 <= ws_bytes) {
          p.part = ws;
          if (whole) hipLaunchKernelGGL((gemm_pp_kernel<128, A_KC, B_KC, EPI, true, true, GemmCall>), sgrid, dim3(512), 0, s, p);
          else hipLaunchKernelGGL((gemm_pp_kernel<128, A_KC, B_KC, EPI, false, true, GemmCall>), sgrid, dim3(512), 0, s, p);
          OASES_LAUNCH_CHECK("gemm_pp_kernel (slices)");
          return 0;
        }
        p.counters = nullptr;
        p.C = ws;
        p.ldc = g.N;
        if (tiles && p.ldc <= kLdcOfLines) hipLaunchKernelGGL((gemm_pp_kernel<128, A_KC, B_KC, EPI_F32, true, false, GemmArgs>), sgrid, dim3(512), 0, s, p);
        else hipLaunchKernelGGL((gemm_pp_kernel<128, A_KC, B_KC, EPI_F32, false, false, GemmArgs>), sgrid, dim3(512), 0, s, p);
        OASES_LAUNCH_CHECK("gemm_pp_kernel (split-K)");
        const long n4 = (long)g.M * (g.N / 4);
        hipLaunchKernelGGL((splitk_fixup_kernel<EPI>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, ws, t.ksplit, d);
        OASES_LAUNCH_CHECK("splitk_fixup_kernel");
        return 0;
      }
    }
    const dim3 grid(d.tiles_m * d.tiles_n);
    if (bm == 128) {
      if (whole) hipLaunchKernelGGL((gemm_pp_kernel<128, A_KC, B_KC, EPI, true, false, GemmArgs>), grid, dim3(512), 0, s, d);
      else hipLaunchKernelGGL((gemm_pp_kernel<128, A_KC, B_KC, EPI, false, false, GemmArgs>), grid, dim3(512), 0, s, d);
    } else {
      if (whole) hipLaunchKernelGGL((gemm_pp_kernel<256, A_KC, B_KC, EPI, true, false, GemmArgs>), grid, dim3(512), 0, s, d);
      else if constexpr (kCanBeRagged) hipLaunchKernelGGL((gemm_pp_kernel<256, A_KC, B_KC, EPI, false, false, GemmArgs>), grid, dim3(512), 0, s, d);
    }
    OASES_LAUNCH_CHECK("gemm_pp_kernel");
    return 0;
  }
  if (t.dtl) {
    if (EPI == EPI_SWIGLU && t.bm == 128) {
      set_error("gemm: the 128x256 direct-to-LDS kernel has no SwiGLU epilogue");
      return OASES_EINVAL;
    } else {
      // the 256 x 256 instantiation with bounds checks in the epilogue exists only where a tile can be ragged
      constexpr bool kCanBeRagged = !A_KC || !B_KC;
      const int bm = t.bm;  // 128 or 256; both kernels have 256-column tiles
      GemmArgs d = g;
      d.tiles_m = (g.M + bm - 1) / bm;
      d.tiles_n = (g.N + 255) / 256;
      const dim3 grid(d.tiles_m * d.tiles_n);
      const bool whole = g.M % bm == 0 && g.N % 256 == 0;
      if (!whole && bm == 256 && !kCanBeRagged) { set_error("gemm: direct-to-LDS kernel on a shape it does not cover"); return OASES_EINVAL; }
      if (bm == 128 && t.ksplit > 1) {
        // k slices: fp32 partial planes [slices][M][N] in the workspace, then the sum and the real epilogue
        if constexpr (EPI == EPI_SWIGLU || EPI == EPI_DSWIGLU) {
          set_error("gemm: the SwiGLU epilogues do not run over k slices");
          return OASES_EINVAL;
        } else {
          if (!ws) { set_error("gemm: split-K chosen without a workspace"); return OASES_ENULL; }
          GemmArgs p = d;
          p.ksplit = t.ksplit;
          p.k_per = g.K / t.ksplit;
          p.C = ws;
          p.ldc = g.N;
          const dim3 sgrid(d.tiles_m * d.tiles_n * t.ksplit);
          if (whole) hipLaunchKernelGGL((gemm_dtl_rect_kernel<A_KC, B_KC, EPI_F32, true>), sgrid, dim3(256), 0, s, p);
          else hipLaunchKernelGGL((gemm_dtl_rect_kernel<A_KC, B_KC, EPI_F32, false>), sgrid, dim3(256), 0, s, p);
          OASES_LAUNCH_CHECK("gemm_dtl_rect_kernel (split-K)");
          const long n4 = (long)g.M * (g.N / 4);
          hipLaunchKernelGGL((splitk_fixup_kernel<EPI>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, ws, t.ksplit, d);
          OASES_LAUNCH_CHECK("splitk_fixup_kernel");
          return 0;
        }
      } else if (bm == 128) {
        if constexpr (EPI != EPI_SWIGLU) {
          if (whole) hipLaunchKernelGGL((gemm_dtl_rect_kernel<A_KC, B_KC, EPI, true>), grid, dim3(256), 0, s, d);
          else hipLaunchKernelGGL((gemm_dtl_rect_kernel<A_KC, B_KC, EPI, false>), grid, dim3(256), 0, s, d);
        }
      } else {
        if (whole) hipLaunchKernelGGL((gemm_dtl_kernel<A_KC, B_KC, EPI, true>), grid, dim3(256), 0, s, d);
        else if constexpr (kCanBeRagged) hipLaunchKernelGGL((gemm_dtl_kernel<A_KC, B_KC, EPI, false>), grid, dim3(256), 0, s, d);
      }
      OASES_LAUNCH_CHECK("gemm direct-to-LDS kernel");
      return 0;
    }
  }
  if (t.bm == 256 && t.bn == 256) return launch_one<256, 256, 2, 2, 1, A_KC, B_KC, EPI>(g, t.ksplit, ws, s);
  if (!t.wave_ksplit) {
    if (t.bm == 256 && t.bn == 128) return launch_one<256, 128, 2, 2, 1, A_KC, B_KC, EPI>(g, t.ksplit, ws, s);
    if (t.bm == 128 && t.bn == 256) return launch_one<128, 256, 2, 2, 1, A_KC, B_KC, EPI>(g, t.ksplit, ws, s);
  }
  if (t.bm == 256 && t.bn == 128) return launch_one<256, 128, 2, 1, 2, A_KC, B_KC, EPI>(g, t.ksplit, ws, s);
  if (t.bm == 128 && t.bn == 256) return launch_one<128, 256, 1, 2, 2, A_KC, B_KC, EPI>(g, t.ksplit, ws, s);
  return launch_one<128, 128, 2, 2, 1, A_KC, B_KC, EPI>(g, t.ksplit, ws, s);
}

}  // namespace

#if OASES_GEMM_HAS(0)
int launch_gemm_nn(const GemmCall& g, int epi, float* ws, size_t ws_bytes, int forced_variant, int choice_rows, hipStream_t s) {
  switch (epi) {
    case EPI_F32: return launch_shape<true, false, EPI_F32>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_BF16: return launch_shape<true, false, EPI_BF16>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_BIAS_BF16: return launch_shape<true, false, EPI_BIAS_BF16>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_BIAS_GELU: return launch_shape<true, false, EPI_BIAS_GELU>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_DGELU: return launch_shape<true, false, EPI_DGELU>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_SWIGLU: return launch_shape<true, false, EPI_SWIGLU>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    default: set_error("gemm: unknown epilogue %d", epi); return OASES_EINVAL;
  }
}
#endif
#if OASES_GEMM_HAS(1)
int launch_gemm_nt(const GemmCall& g, int epi, float* ws, size_t ws_bytes, int forced_variant, int choice_rows, hipStream_t s) {
  switch (epi) {
    case EPI_F32: return launch_shape<true, true, EPI_F32>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_BF16: return launch_shape<true, true, EPI_BF16>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_BIAS_BF16: return launch_shape<true, true, EPI_BIAS_BF16>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_BIAS_GELU: return launch_shape<true, true, EPI_BIAS_GELU>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_DGELU: return launch_shape<true, true, EPI_DGELU>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    case EPI_DSWIGLU: return launch_shape<true, true, EPI_DSWIGLU>(g, ws, ws_bytes, forced_variant, choice_rows, s);
    default: set_error("gemm: unknown epilogue %d", epi); return OASES_EINVAL;
  }
}
#endif
#if OASES_GEMM_HAS(1)
// The small-tile kernel for launch_gemm_delta, whose tiles hold whole heads, or 0 where it is expected to take more than 3 us longer than the
// kernel that the product alone would get: attn_delta_kernel, which is saved, takes 3.5 us and the launch gap ahead of it 1 to 2.
int gemm_delta_variant(int M, int N, int K, int head_dim, size_t ws_bytes) {
  double alone, t;
  pick_tile(1, EPI_BF16, M, N, K, ws_bytes, &alone, true);
  const TileChoice c = pick_tile(1, EPI_BF16, M, N, K, ws_bytes, &t, true, head_dim);
  return c.st && t < alone + 3.0e-6 ? encode_variant(c, 1, M, N, K) : 0;
}
int launch_gemm_delta(int variant, int M, int N, int K, const void* A, const void* B, void* C, const void* out, float* delta, int seq, int head_dim,
                      float* ws, size_t ws_bytes, uint32_t* counters, hipStream_t s) {
  TileChoice t;
  if (!A || !B || !C || !out || !delta || !ws || !counters) { set_error("gemm_delta: NULL argument"); return OASES_ENULL; }
  if (head_dim <= 0 || seq <= 0 || M % 8 || K % 8 || N % head_dim || M % seq || variant < 400000000 ||
      (variant % 1000 != head_dim && variant % 1000 != 2 * head_dim) || !decode_variant(variant, 1, M, N, K, ws_bytes, &t) || !gemm_span_fits(M, K) || !gemm_span_fits(N, K)) {
    set_error("gemm_delta: variant %d does not fit M=%d N=%d K=%d seq=%d head_dim=%d", variant, M, N, K, seq, head_dim);
    return OASES_EINVAL;
  }
  GemmCall g{{(const uint16_t*)A, (const uint16_t*)B, C, nullptr, (uint16_t*)const_cast<void*>(out), M, N, K, K, K, N, N, 0, 0, 1, K}};
  g.counters = counters;
  g.sums = delta;
  g.seq = seq;
  g.head_dim = head_dim;
  if (t.bm == 128) return launch_small<2, 2, 4, true, true, EPI_BF16_DELTA>(g, t.ksplit, ws, ws_bytes, s);
  if (t.bn == 128) return launch_small<1, 2, 3, true, true, EPI_BF16_DELTA>(g, t.ksplit, ws, ws_bytes, s);
  return launch_small<1, 1, 5, true, true, EPI_BF16_DELTA>(g, t.ksplit, ws, ws_bytes, s);
}
#endif  // NT part
#if OASES_GEMM_HAS(2)
int launch_gemm_tn(const GemmCall& g, float* ws, size_t ws_bytes, int forced_variant, hipStream_t s) {
  return launch_shape<false, false, EPI_ACC_F32>(g, ws, ws_bytes, forced_variant, 0, s);
}

bool gemm_tn_pair_wins(int K, int M0, int N0, int M1, int N1) {
  if (M0 <= 0 || N0 <= 0 || M1 <= 0 || N1 <= 0 || !dtl_rect_whole(M0, N0, K) || !dtl_rect_whole(M1, N1, K)) return false;
  // few rows: what counts is the traffic of the gradients, which small tiles move faster (see pick_tile)
  if (pick_tile(2, EPI_ACC_F32, M0, N0, K, 0).st && pick_tile(2, EPI_ACC_F32, M1, N1, K, 0).st) return false;
  const long t0 = (long)(M0 / 128) * (N0 / 256), t1 = (long)(M1 / 128) * (N1 / 256);
  // enough tiles to be worth whole 128 x 256 tiles at all, and fewer rounds of 256 workgroups together than apart
  return t0 + t1 > 128 && (t0 + t1 + 255) / 256 < (t0 + 255) / 256 + (t1 + 255) / 256;
}

int launch_gemm_tn_pair(int K, int M0, int N0, const void* A0, int lda0, const void* B0, int ldb0, void* C0, int ldc0, int M1, int N1,
                        const void* A1, int lda1, const void* B1, int ldb1, void* C1, int ldc1, hipStream_t s) {
  if (K <= 0 || M0 <= 0 || N0 <= 0 || M1 <= 0 || N1 <= 0 || !dtl_rect_whole(M0, N0, K) || !dtl_rect_whole(M1, N1, K)) {
    set_error("gemm_tn_pair: needs M %% 128 == 0, N %% 256 == 0, K %% 64 == 0 for both problems (got K=%d, %dx%d and %dx%d)", K, M0, N0, M1, N1);
    return OASES_EINVAL;
  }
  if ((lda0 % 8) || (ldb0 % 8) || (ldc0 % 4) || (lda1 % 8) || (ldb1 % 8) || (ldc1 % 4) || lda0 < M0 || ldb0 < N0 || ldc0 < N0 || lda1 < M1 ||
      ldb1 < N1 || ldc1 < N1) {
    set_error("gemm_tn_pair: leading dimension too small or not a multiple of 8 (A, B) / 4 (C)");
    return OASES_EINVAL;
  }
  if (!gemm_span_fits(K, lda0) || !gemm_span_fits(K, ldb0) || !gemm_span_fits(K, lda1) || !gemm_span_fits(K, ldb1)) {
    set_error("gemm_tn_pair: an operand spans 2 GiB or more (K=%d rows)", K);
    return OASES_EINVAL;
  }
  if (!A0 || !B0 || !C0 || !A1 || !B1 || !C1) { set_error("gemm_tn_pair: NULL operand"); return OASES_ENULL; }
  if (!aligned16(A0) || !aligned16(B0) || !aligned16(C0) || !aligned16(A1) || !aligned16(B1) || !aligned16(C1)) {
    set_error("gemm_tn_pair: operand not 16-byte aligned");
    return OASES_EALIGN;
  }
  GemmArgs g0{(const uint16_t*)A0, (const uint16_t*)B0, C0, nullptr, nullptr, M0, N0, K, lda0, ldb0, ldc0, 0, M0 / 128, N0 / 256, 1, K};
  GemmArgs g1{(const uint16_t*)A1, (const uint16_t*)B1, C1, nullptr, nullptr, M1, N1, K, lda1, ldb1, ldc1, 0, M1 / 128, N1 / 256, 1, K};
  const dim3 grid(g0.tiles_m * g0.tiles_n + g1.tiles_m * g1.tiles_n);
  if (std::max(ldc0, ldc1) <= kLdcOfLines) hipLaunchKernelGGL((gemm_pp_group_kernel<true, false>), grid, dim3(512), 0, s, g0, g1, nullptr, nullptr);
  else hipLaunchKernelGGL((gemm_pp_group_kernel<false, false>), grid, dim3(512), 0, s, g0, g1, nullptr, nullptr);
  OASES_LAUNCH_CHECK("gemm_pp_group_kernel");
  return 0;
}

// Two weight gradients of a block in one launch.  Variants as those of a single GEMM: 30S128256 (here S = 1, 2, 4 or 8 slices, summed by the launch
// itself), 601128256, 401064064, 401064128.
static bool tn_group_fits(int variant, int K, int M0, int N0, int M1, int N1, size_t ws_bytes) {
  if (variant == 401064064 || variant == 401064128) return true;
  if (variant == 601128256) return K >= 1024;
  const int S = variant / 1000000 % 100;
  if (variant != 300128256 + S * 1000000 || (S != 1 && S != 2 && S != 4 && S != 8) || K % BKR) return false;
  const long T = (long)((M0 + 127) / 128) * ((N0 + 255) / 256) + (long)((M1 + 127) / 128) * ((N1 + 255) / 256);
  return S == 1 || (T <= kSliceCounters && (long)(S - 1) * st_k_per(K, S) < K && (size_t)T * S * 128 * 256 * 4 <= ws_bytes);  // every slice has stages of its own
}
static double tn_single_seconds(int M, int N, int K, size_t ws_bytes) {
  double t;
  const TileChoice c = pick_tile(2, EPI_ACC_F32, M, N, K, ws_bytes, &t, true);
  if (c.st || !c.pp) return t;
  t = pp_seconds(c.bm, (long)((M + c.bm - 1) / c.bm) * ((N + 255) / 256) * c.ksplit, K / c.ksplit, 8.0 * M * N);
  return c.ksplit > 1 ? t + 2.0e-6 + 2.7e-6 * (c.ksplit - 1) : t;
}
// Which kernel, how many slices, and whether one launch takes less time than two.  k slices cost 2 us and 2.7 us each: the last workgroup of a tile
// reads the others' sums one after the other.  Inside a step, us, two launches -> one (small tiles bring the bias gradient along, which is a launch of
// its own beside two: + its time): 8192 rows, 2048x2048 twice 170 -> 125 (one round instead of two with slices), 512x2048 and 2048x1536 119 -> 85
// (two slices); 4096 rows, 1024x1024 twice 34 to 48 + 5 -> 34 (64x128; four slices of 128x256 38 + 5, 64x64 36), 256x1024 and 1024x768 32 + 5 -> 23 (64x64; 64x128 33); 2048
// rows, the same 21 + 4 -> 20 and 19 + 4 -> 13.5; 512 rows, 1024x512 twice 11.4 + 2.4 -> 7.3 (64x64; 64x128 9.4); 128 rows, 12288x6144 and 6144x12288
// 282 + 5 -> 272.  8192 rows, 1376x4096 and 4096x2752 stay two (118 and 173; by themselves 268 together, one launch 290).
// Those were taken with 32x32x16 MFMAs.  On the kernels as they are, by themselves on cold operands (with the launch that clears the counters), two launches -> one, the choice
// first: 8192 rows, 2048x2048 twice 175 -> 149 (two slices 162, 64x128 227), 512x2048 and 2048x1536 130 -> 97 (one slice 133); 4096 rows, 1024x1024 twice 51 -> 42 (four slices
// 42, 64x64 48), 256x1024 and 1024x768 38 -> 32 (four slices 37, 64x128 41); 2048 rows 29 -> 25 (64x64 28) and 24 -> 19 (64x128 24), 704x1024 and 1024x1408 35 -> 36 (64x128
// 32, which adds up in half as many chains); 512 rows 10.8 -> 9.8 (64x128 11.6); 128 rows 288 -> 291 (128x256 257).  1376x4096 and 4096x2752 stay two: 332, one launch 324.
int gemm_tn_group_variant(int K, int M0, int N0, int M1, int N1, size_t ws_bytes, bool bias, bool* wins) {
  const double out = ((double)M0 * N0 + (double)M1 * N1) * 8.0;
  double best_t = 1e30;
  int best = 0;
  const long T = (long)((M0 + 127) / 128) * ((N0 + 255) / 256) + (long)((M1 + 127) / 128) * ((N1 + 255) / 256);
  for (int S = 1; S <= 8; S *= 2) {
    const int v = 300128256 + S * 1000000;
    if (!tn_group_fits(v, K, M0, N0, M1, N1, ws_bytes)) continue;
    const double t = pp_seconds(128, T * S, st_k_per(K, S), out) + (S > 1 ? 2.0e-6 + 2.7e-6 * S : 0.0);
    if (t < best_t) { best_t = t; best = v; }
  }
  for (int bn = 64; bn <= 128; bn += 64) {
    const long per_cu = ((long)((M0 + 63) / 64) * ((N0 + bn - 1) / bn) + (long)((M1 + 63) / 64) * ((N1 + bn - 1) / bn) + 255) / 256;
    const double t = 2.9e-6 + (double)per_cu * ((K + BKS - 1) / BKS) * (bn == 64 ? 0.225e-6 : 0.335e-6) + out / 4.0e12;
    if (t < best_t) { best_t = t; best = 401064000 + bn; }
  }
  if (wins) *wins = gemm_span_fits(K, std::max({M0, N0, M1, N1})) && best_t < tn_single_seconds(M0, N0, K, ws_bytes) + tn_single_seconds(M1, N1, K, ws_bytes);
  // rows that are no whole number of stages: the same sums on the eight-wave kernel (same_sums).  Not where the small tiles bring a bias gradient: the launch that
  // it would need instead rounds a fifth more (rms against 64 bits, 3960 rows 3.8e-8 and 4.6e-8)
  if (!bias && best / 100000000 == 4 && K % BKR && T >= kPpLeastTiles && tn_group_fits(601128256, K, M0, N0, M1, N1, ws_bytes) && pp128_seconds(T, K, out) < best_t) best = 601128256;
  return best;
}

int launch_gemm_tn_group(int variant, int K, const TnProblem& a, const TnProblem& b, float* ws, size_t ws_bytes, uint32_t* counters, hipStream_t s) {
  for (const TnProblem* p : {&a, &b}) {
    if (K <= 0 || p->M <= 0 || p->N <= 0 || K % 8 || p->M % 8 || p->N % 8 || p->lda % 8 || p->ldb % 8 || p->ldc % 4 || p->lda < p->M || p->ldb < p->N ||
        p->ldc < p->N) {
      set_error("gemm_tn_group: K, M, N, lda, ldb must be positive multiples of 8, ldc of 4, no leading dimension below its width (K=%d M=%d N=%d)", K, p->M, p->N);
      return OASES_EINVAL;
    }
    if (!gemm_span_fits(K, p->lda) || !gemm_span_fits(K, p->ldb)) { set_error("gemm_tn_group: an operand spans 2 GiB or more (K=%d rows)", K); return OASES_EINVAL; }
    if (!p->A || !p->B || !p->C) { set_error("gemm_tn_group: NULL operand"); return OASES_ENULL; }
    if (!aligned16(p->A) || !aligned16(p->B) || !aligned16(p->C)) { set_error("gemm_tn_group: operand not 16-byte aligned"); return OASES_EALIGN; }
  }
  if (!variant) variant = gemm_tn_group_variant(K, a.M, a.N, b.M, b.N, ws && counters ? ws_bytes : 0, a.colsum || b.colsum);
  if (!tn_group_fits(variant, K, a.M, a.N, b.M, b.N, ws && counters ? ws_bytes : 0)) {
    set_error("gemm_tn_group: variant %d does not exist or does not fit K=%d, %dx%d and %dx%d with %zu workspace bytes", variant, K, a.M, a.N, b.M, b.N, ws_bytes);
    return OASES_EINVAL;
  }
  const int bm = variant / 1000 % 1000, bn = variant % 1000, S = variant / 1000000 % 100;
  if (bm != 64 && (a.colsum || b.colsum)) { set_error("gemm_tn_group: column sums come with the small tiles only"); return OASES_EINVAL; }
  auto args = [&](const TnProblem& p) {
    return GemmCall{{(const uint16_t*)p.A, (const uint16_t*)p.B, p.C, nullptr, nullptr, p.M, p.N, K, p.lda, p.ldb, p.ldc, 0,
                     (p.M + bm - 1) / bm, (p.N + bn - 1) / bn, S, st_k_per(K, S)}, ws, counters, p.colsum};
  };
  const GemmCall g0 = args(a), g1 = args(b);
  const dim3 grid((unsigned)((g0.tiles_m * g0.tiles_n + g1.tiles_m * g1.tiles_n) * S));
  if (bm == 64) {
    if (bn == 64) hipLaunchKernelGGL((gemm_st_group_kernel<1, 5>), grid, dim3(512), 0, s, g0, g1);
    else hipLaunchKernelGGL((gemm_st_group_kernel<2, 3>), grid, dim3(512), 0, s, g0, g1);
    OASES_LAUNCH_CHECK("gemm_st_group_kernel");
    return 0;
  }
  const bool whole = a.M % 128 == 0 && a.N % 256 == 0 && b.M % 128 == 0 && b.N % 256 == 0 && std::max(a.ldc, b.ldc) <= kLdcOfLines;
  if (S > 1) {
    if (whole) hipLaunchKernelGGL((gemm_pp_group_kernel<true, true>), grid, dim3(512), 0, s, g0, g1, ws, counters);
    else hipLaunchKernelGGL((gemm_pp_group_kernel<false, true>), grid, dim3(512), 0, s, g0, g1, ws, counters);
  } else {
    if (whole) hipLaunchKernelGGL((gemm_pp_group_kernel<true, false>), grid, dim3(512), 0, s, g0, g1, nullptr, nullptr);
    else hipLaunchKernelGGL((gemm_pp_group_kernel<false, false>), grid, dim3(512), 0, s, g0, g1, nullptr, nullptr);
  }
  OASES_LAUNCH_CHECK("gemm_pp_group_kernel");
  return 0;
}

#endif  // TN part
#if OASES_GEMM_HAS(0)
int gemm_variant(int op, int epi, int M, int N, int K, size_t ws_bytes, bool pass) {
  const int kind = op == OASES_GEMM_TN ? 2 : op == OASES_GEMM_NT ? 1 : (epi == EPI_BIAS_GELU || epi == EPI_SWIGLU) ? 3 : 0;
  if (epi == EPI_SWIGLU || epi == EPI_DSWIGLU) ws_bytes = 0;
  if (op == OASES_GEMM_TN) epi = EPI_ACC_F32;
  double seconds;
  const TileChoice t = pick_tile(kind, epi, M, N, K, ws_bytes, &seconds, pass);
  return encode_variant(same_sums(t, seconds, kind, M, N, K), kind, M, N, K);
}

int launch_gemm(int op, int epi, int M, int N, int K, const void* A, int lda, const void* B, int ldb, void* C,
                int ldc, const float* bias, void* aux, int ldaux, void* splitk_ws, size_t splitk_ws_bytes, int forced_variant,
                hipStream_t s, int choice_rows, uint32_t* counters) {
  float* ws = reinterpret_cast<float*>(splitk_ws);
  const size_t wsb = splitk_ws_bytes;
  if (M <= 0 || N <= 0 || K <= 0 || (M % 8) || (N % 8) || (K % 8) || (lda % 8) || (ldb % 8) || (ldc % 4) || (aux && ldaux % 4)) {
    set_error("gemm: M,N,K,lda,ldb must be positive multiples of 8, ldc/ldaux of 4 (got M=%d N=%d K=%d lda=%d ldb=%d ldc=%d)", M, N, K, lda, ldb, ldc);
    return OASES_EINVAL;
  }
  if (!A || !B || !C) { set_error("gemm: NULL operand"); return OASES_ENULL; }
  if (!aligned16(A) || !aligned16(B) || !aligned16(C) || !aligned16(bias) || !aligned16(aux)) { set_error("gemm: operand not 16-byte aligned"); return OASES_EALIGN; }
  GemmCall g{{(const uint16_t*)A, (const uint16_t*)B, C, bias, (uint16_t*)aux, M, N, K, lda, ldb, ldc, ldaux, 0, 0, 1, K}};
  g.counters = ws ? counters : nullptr;
  if (op == OASES_GEMM_TN) {
    if (lda < M || ldb < N || ldc < N) { set_error("gemm TN: leading dimension too small"); return OASES_EINVAL; }
    return launch_gemm_tn(g, ws, wsb, forced_variant, s);
  }
  const bool nn = op == OASES_GEMM_NN;
  if (!nn && op != OASES_GEMM_NT) { set_error("gemm: unknown op %d", op); return OASES_EINVAL; }
  const int c_cols = epi == EPI_SWIGLU ? N / 2 : epi == EPI_DSWIGLU ? 2 * N : N;  // SwiGLU: C is [M, N/2]; its gradient: [M, 2N]
  if (lda < K || (nn ? ldb < N : ldb < K) || ldc < c_cols) { set_error("gemm: leading dimension too small"); return OASES_EINVAL; }
  if (epi == EPI_SWIGLU && (!nn || N % 64 || !aux || ldaux < N)) { set_error("gemm: SwiGLU epilogue needs the NN form, N %% 64 == 0 and aux [M,N]"); return OASES_EINVAL; }
  if (epi == EPI_DSWIGLU && (nn || N % 32 || !aux || ldaux < 2 * N)) { set_error("gemm: SwiGLU-gradient epilogue needs the NT form, N %% 32 == 0 and aux [M,2N]"); return OASES_EINVAL; }
  if ((epi == OASES_EPI_BIAS_BF16 || epi == OASES_EPI_BIAS_GELU) && !bias) { set_error("gemm: bias epilogue without bias"); return OASES_ENULL; }
  if ((epi == OASES_EPI_BIAS_GELU || epi == OASES_EPI_DGELU) && (!aux || ldaux < N)) { set_error("gemm: GeLU epilogue without aux"); return OASES_ENULL; }
  if ((nn && epi == EPI_DSWIGLU) || (!nn && epi == EPI_SWIGLU) || epi < 0 || epi > EPI_DSWIGLU || epi == EPI_ACC_F32) {
    set_error("gemm: unknown epilogue %d", epi);
    return OASES_EINVAL;
  }
  return nn ? launch_gemm_nn(g, epi, ws, wsb, forced_variant, choice_rows, s) : launch_gemm_nt(g, epi, ws, wsb, forced_variant, choice_rows, s);
}
#endif  // NN part and host entry points

}  // namespace oases
