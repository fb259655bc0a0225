// Flash-style causal grouped-query attention for gfx950, head_dim 128 or 64, bf16 storage, fp32 softmax and
// accumulation, v_mfma_f32_32x32x16_bf16 throughout.  Three kernels: forward, dQ, and dK/dV.  The
// [S,S] score matrix never exists; only the per-row log-sum-exp is kept for the backward pass.
//
// Orientation.  An MFMA 32x32 result leaves each lane with ONE column (lane % 32) and 16 of the 32 rows.
// Every product is therefore arranged so that the index a lane needs a scalar for is the column:
//   forward / dQ : S^T = K Q^T (rows = keys, columns = queries) -> the running max / sum, lse and delta
//                  of a query are per-lane scalars, and a row reduction is 16 in-lane steps plus one
//                  exchange with lane ^ 32;
//   dK/dV        : S = Q K^T (rows = queries, columns = keys)   -> the dK/dV columns of a key stay in
//                  one lane.
// In both cases the probabilities come out of the MFMA exactly in the register layout that the next
// MFMA wants for its B operand (8 contraction values per lane), provided the A operand enumerates the
// contraction index in the same order {4g..4g+3, 8+4g..8+4g+3} (g = lane / 32).  That A operand (V^T,
// K^T, dO^T, Q^T) is read from the row-major LDS tile with the transposing LDS read
// ds_read_b64_tr_b16, so nothing is ever transposed through registers or HBM.
//
// Tiles.  Forward and dQ: one block = 128 queries of one head (4 waves x 32 queries, Q in registers; capped
// at 256 VGPRs so that two blocks share a CU and one block's softmax overlaps the other's MFMAs; the forward of head size 128
// also makes the next tile's scores beside a tile's exponentials), K/V streamed in 64-key tiles, double buffered in LDS.  dK/dV: one block = 128 keys of one kv
// head (4 waves x 32 keys, K [and V] in registers), Q/dO streamed in tiles of 32 (dV pass) or 64 (dK pass)
// queries for each of the G query heads of the group, so dK/dV are summed over the group in registers: no
// atomics, deterministic.  dV and dK are two launches of one template: a fused pass needs 350 registers (K, V
// fragments and two 32x128 accumulators), i.e. one block per CU with nothing to hide the exponentials behind;
// the two halves need 168 and 212, run 3 and 2 blocks per CU, and together take 0.7x the fused time although
// S = Q K^T is computed twice.
// Where blocks are few, a block is 64 keys and eight waves in four sets that share the query tiles (kFewKW, kFewNS).
// Every streamed tile reaches LDS by LDS-DMA loads (no staging registers); operand fragments are read from LDS
// through small register rings, a few MFMAs ahead of their use.
// Causality: tiles entirely above the diagonal are never loaded; heavy blocks are scheduled first; the
// per-element causal test is made only by the (wave-uniformly chosen) tiles that touch the diagonal.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "prof.h"
#include "tide_common.h"

namespace tide {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

namespace {

// LDS row pitch in elements, D = head_dim (128 or 64): 272 B = 4 banks past a multiple of 64, resp. 144 B = 36 banks.
// The rows of a 16-row read then start on 16 different groups of 4 banks, and rows 4 apart 16 banks apart.
constexpr int pitch(int D) { return D + 8; }
// Streamed tiles (K, V, Q, dO) keep row r of the tile in LDS row perm(r): inside every group of 16 rows the two
// 2-bit fields of the row number are exchanged.  A row read (16 lanes = 16 consecutive tile rows, 16 bytes each)
// still meets 16 different LDS rows, 4 banks apart: all 64 banks once.  A transposing read (32 lanes = 4
// consecutive tile rows x 64 contiguous bytes) now meets LDS rows that are 4 apart, i.e. 16 banks apart: four
// disjoint windows.  With the rows in natural order those four windows overlapped (4 banks apart), and half of all
// LDS cycles of the three kernels were bank-conflict cycles (by counter).  Every address stays base + constant.
__device__ __forceinline__ int perm(int r) { return (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3); }
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ f32x16_t mfma(u32x4_t a, u32x4_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// A/B operand whose contraction index is contiguous in the LDS tile: tile row row0 + r with row0 a multiple of 16
// and prow = perm(r) (computed once per lane)
template <int D>
__device__ __forceinline__ u32x4_t frag(const bf16_t* tile, int row0, int prow, int kofs) {
  return *reinterpret_cast<const u32x4_t*>(tile + (row0 + prow) * pitch(D) + kofs);
}

// A operand taken from the tile TRANSPOSED: tile is [k][pitch] (k = contraction index, 16 rows starting
// at kbase), the operand row is the tile column nbase + lane % 32, and the 8 contraction values of the
// lane are k = kbase + {4g..4g+3, 8+4g..8+4g+3}.
template <int D>
__device__ __forceinline__ u32x4_t frag_tr(const bf16_t* tile, int kbase, int nbase, int lane) {
  const int g = lane >> 5;
  const int l16 = lane & 15;
  const int col = nbase + ((lane >> 4) & 1) * 16 + (l16 & 3) * 4;
  const int row = kbase + ((l16 >> 2) << 2) + g;   // perm(kbase + 4 g + (l16 >> 2)); kbase is a multiple of 16
  typedef __attribute__((address_space(3))) s16x4_t* lds_ptr_t;
  const bf16_t* p0 = tile + row * pitch(D) + col;
  const bf16_t* p1 = p0 + 2 * pitch(D);                // perm of the tile row 8 further on
  s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p0));
  s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p1));
  u32x2_t a = __builtin_bit_cast(u32x2_t, lo), b = __builtin_bit_cast(u32x2_t, hi);
  u32x4_t r;
  r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
  return r;
}

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return f2bf2(lo, hi);
}

// registers q0..q0+7 of a 32x32 accumulator -> the 8-value B operand of the next MFMA
__device__ __forceinline__ u32x4_t pack_half(const f32x16_t& v, int half) {
  u32x4_t r;
#pragma unroll
  for (int w = 0; w < 4; ++w)
    r[w] = pack2(v[half * 8 + 2 * w], v[half * 8 + 2 * w + 1]);
  return r;
}

// Probabilities and score gradients enter their products as bf16.  At head size 128 that is one value, rounded.  At
// head size 64, which was served in fp32 arithmetic, each is the sum of two (the rounded value and the rounded rest, 16
// bits of mantissa together): with one the results were 1.25 to 1.4 times as far from fp64 as in fp32 arithmetic, with
// two they are as close (0.155 to 0.20 %, their own rounding, over six shapes and four seeds); 16 x 2048, 32 / 8 heads: 0.38 + 1.53 ms with
// one, 0.50 + 1.82 with two.
constexpr int parts(int D) { return D == 64 ? 2 : 1; }
template <int NP>
__device__ __forceinline__ void pack_parts(const f32x16_t& v, int half, u32x4_t (&r)[NP]) {
  r[0] = pack_half(v, half);
  if constexpr (NP == 2) {
#pragma unroll
    for (int w = 0; w < 4; ++w)
      r[1][w] = pack2(v[half * 8 + 2 * w] - __uint_as_float(r[0][w] << 16), v[half * 8 + 2 * w + 1] - __uint_as_float(r[0][w] & 0xFFFF0000u));
  }
}
// acc + a * (sum of the parts of b), the small part first
template <int NP>
__device__ __forceinline__ f32x16_t mfma_parts(u32x4_t a, const u32x4_t (&b)[NP], f32x16_t acc) {
#pragma unroll
  for (int i = NP - 1; i >= 0; --i) acc = mfma(a, b[i], acc);
  return acc;
}

// row index (0..31) that accumulator register q of this lane holds
__device__ __forceinline__ int acc_row(int q, int g) { return 8 * (q >> 2) + 4 * g + (q & 3); }

// Staging of a tile of 64 or 32 rows x D columns (bf16) of a row-major global matrix in LDS, without registers:
// LDS-DMA loads (16 bytes per lane straight into LDS, written as instructions so that the waits are this file's
// own: the compiler does not see that they write LDS).  A 64-row tile with its 272-byte (D = 64: 144-byte)
// pitch is 17 (9) chunks of 1 KiB of consecutive LDS bytes; wave w of NW issues the chunks w, w + NW, ... and lane l of chunk c
// fills the bytes c * 1024 + 16 l .. + 16, i.e. LDS row (c * 1024 + 16 l) / 272 = tile row perm(LDS row), 16-byte
// piece ((c * 1024 + 16 l) % 272) / 16; the last piece of a row is its padding and loads from beyond the buffer
// (zeros).  Rows past the end of the sequence lie beyond the buffer as well.
__device__ __forceinline__ i32x4_t rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)base;
  i32x4_t r;
  r[0] = (int)(uint32_t)a; r[1] = (int)((uint32_t)(a >> 32) & 0xffffu); r[2] = (int)bytes; r[3] = 0x00020000;
  return r;
}
__device__ __forceinline__ void dma16(i32x4_t rs, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rs) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const bf16_t* p) {
  typedef __attribute__((address_space(3))) const bf16_t* lds_p;
  return (uint32_t)(uintptr_t)(lds_p)p;
}
template <int ROWS, int D, int NW = 4>   // NW: waves that share the loads; rows of the tile (64, or 32: 8.5 or 4.5 chunks, the second half of the last is not part of the tile)
struct TileDma {
  static constexpr int PITCH = pitch(D);
  static constexpr int BYTES = ROWS * PITCH * 2;
  static constexpr int CHUNKS = (BYTES + 1023) / 1024;   // D = 128: 17 / 9, D = 64: 9 / 5
  static constexpr int PER_WAVE = (CHUNKS + NW - 1) / NW;   // the last not in every wave
  uint32_t voff[PER_WAVE];   // byte offset of the lane's piece from the tile's first element (beyond any buffer: padding)
  __device__ __forceinline__ void init(int ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int o = (wave + NW * i) * 1024 + lane * 16;
      const int R = o / (PITCH * 2), piece = (o % (PITCH * 2)) / 16;
      // (2^31 is beyond any sequence, see attn_mfma_supported)
      voff[i] = (piece < D / 8 && o < BYTES) ? (uint32_t)(perm(R) * ld + piece * 8) * 2u : 0x80000000u;
    }
  }
  // tile_bytes: byte offset of the tile's first element from src, whose `bytes` bytes may be read; wave_s: the wave index as a
  // scalar.  The tile's place goes into the descriptor (scalar operations), so that the lane offsets are loop constants.
  __device__ __forceinline__ void issue(const bf16_t* src, uint32_t bytes, const bf16_t* tile, uint32_t tile_bytes, int wave_s) const {
    const i32x4_t rs = rsrc_words((const char*)src + tile_bytes, bytes - tile_bytes);
    const uint32_t base = lds_address(tile);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i)   // (the test is for the last round of chunks alone)
      if (NW * (i + 1) <= CHUNKS || wave_s + NW * i < CHUNKS) dma16(rs, base + (uint32_t)(wave_s + NW * i) * 1024u, voff[i]);
  }
};
#define TIDE_ATTN_WAIT_DMA() __builtin_amdgcn_s_waitcnt(0x0F70)   /* vmcnt(0) */

// Write a wave's 32 x D result, held transposed in D / 32 accumulators (acc[ct] = rows ct*32.., column =
// lane % 32 = the wave-local output row), into an LDS tile [rows][pitch] at rows wave*32.. as bf16.
template <int D>
__device__ __forceinline__ void stage_out(bf16_t* tile, const f32x16_t (&acc)[D / 32], float mul, int wave, int lane) {
  const int g = lane >> 5, r = wave * 32 + (lane & 31);
#pragma unroll
  for (int ct = 0; ct < D / 32; ++ct)
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
      const int c = ct * 32 + 8 * qq + 4 * g;
      uint2 v;
      v.x = pack2(acc[ct][qq * 4 + 0] * mul, acc[ct][qq * 4 + 1] * mul);
      v.y = pack2(acc[ct][qq * 4 + 2] * mul, acc[ct][qq * 4 + 3] * mul);
      *reinterpret_cast<uint2*>(tile + r * pitch(D) + c) = v;
    }
}

// Copy the staged [ROWS][D] tile to global rows row0.. (< row_end) of a matrix with leading dim ld; NT threads.
template <int D, int ROWS = 128, int NT = 256>
__device__ __forceinline__ void copy_out(const bf16_t* tile, bf16_t* dst, int64_t row0, int64_t row_end, int ld,
                                         int col0, int tid) {
#pragma unroll
  for (int i = 0; i < (ROWS * D / 8 + NT - 1) / NT; ++i) {
    const int p = tid + i * NT;
    const int row = p / (D / 8), piece = p % (D / 8);
    if (row < ROWS && row0 + row < row_end)
      *reinterpret_cast<i32x4_t*>(dst + (size_t)(row0 + row) * ld + col0 + piece * 8) =
          *reinterpret_cast<const i32x4_t*>(tile + row * pitch(D) + piece * 8);
  }
}

// which of the wave's 32 output rows (held as for stage_out) hold something that is not finite; `ask`: this lane's row counts
template <int NC>
__device__ __forceinline__ uint32_t not_finite(const f32x16_t (&acc)[NC], bool ask) {
  float z[4] = {0.f, 0.f, 0.f, 0.f};   // four chains: the sum is on the way to the store
#pragma unroll
  for (int ct = 0; ct < NC; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) z[q & 3] = fmaf(acc[ct][q], 0.f, z[q & 3]);
  const uint64_t rows = __builtin_amdgcn_ballot_w64((z[0] + z[1]) + (z[2] + z[3]) != 0.f && ask);
  return (uint32_t)rows | (uint32_t)(rows >> 32);
}

constexpr int BQ = 128, BKV = 64;
// By how much (log2) the reference that a row's sums are kept relative to may fall behind the running maximum; see the forward kernel.
constexpr float lag(int D) { return D == 64 ? 8.0f : 0.0f; }

// The waves of a SIMD belong to two blocks: the one in a phase of MFMAs alone goes before the other's vector instructions, which
// then run under them (head size 128: forward 2 to 4 %, backward 1 to 2 %; head size 64, three or four blocks: backward 1 % slower).
template <int D>
__device__ __forceinline__ void matrix_phase(bool on) {
  if constexpr (D == 128) {
    if (on) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
  }
}

// the value of lane ^ 32, and the larger of it and this lane's, without the LDS round trip of a shuffle
__device__ __forceinline__ float swap_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);   // {lower half twice, upper half twice}
  return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}
__device__ __forceinline__ float row_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
constexpr int kv_tile(int D) { return BKV * pitch(D); }  // elements

// Head size 64 halves the operand and accumulator registers and the LDS tiles: 114 / 167 / 125 / 147 registers for the
// forward, dQ, dV and dK kernels, i.e. 4, 3, 4 and 3 blocks per CU (held to 4, 4, 5 and 3 the dQ and dV kernels spill:
// backward 1.53 -> 2.73 ms at 16 x 2048, 32 / 8 heads, with one bf16 value per probability).  Against the one-wave-per-row kernels (attention_simple.hip) that
// served this head size: 6 x 777, 16 / 4 heads, forward + backward 17.55 -> 0.144 ms.
constexpr int blocks_per_cu(int D, int at64, int at128) { return D == 64 ? at64 : at128; }
// Depth of the operand-fragment rings of the three kernels (0 in the dQ kernel: the plain loop).  Measured when the tiles
// were still staged through registers, backward at 16 x 2048 / 2 x 16384: dQ 0 / dK-dV 4: 3.56 / 21.4 ms; 2 / 4: 3.48 /
// 21.0; 4 / 4: 3.79 / 22.7 (the dQ kernel, then at 256 registers, spilled with a ring of four); 0 / 2: 3.60 / 21.2;
// before the rings 3.65 / 21.6.  With LDS-DMA tile loads (dQ at 233 registers) depths of 2 to 6 measure the same.
#ifndef TIDE_ATTN_DQ_RING
#define TIDE_ATTN_DQ_RING 2
#endif
#ifndef TIDE_ATTN_DKV_RING
#define TIDE_ATTN_DKV_RING 4
#endif
// Work item (x, y, z) of an nx * ny * nz problem from the block's place in the 1-D dispatch order.
// Work-groups go to the 8 XCDs round-robin and every XCD has its own L2.  The blocks of a "group" (all x of gy
// consecutive y of one z: the query blocks of the heads that share a kv head, or the key blocks of one kv
// head) stream the same K/V resp. Q/dO rows, so a whole group is given to ONE XCD, group after group, x
// fastest.  With the plain (x, y, z) order the 16 key blocks of a kv head were spread over all XCDs and the
// dK / dV passes hit L2 on 2 % of their requests.  Falls back to the plain order when the number of
// groups is not a multiple of 8.
struct Work3 { int x, y, z; };
__device__ __forceinline__ Work3 xcd_group_work(int nx, int ny, int nz, int gy) {
  const int n = blockIdx.x;
  const int per_group = nx * gy, groups_per_z = ny / gy, ngroups = groups_per_z * nz;
  int grp, in_g;
  if ((ngroups & 7) == 0) {
    const int xcd = n & 7, slot = n >> 3;
    grp = (slot / per_group) * 8 + xcd;
    in_g = slot % per_group;
  } else {
    grp = n / per_group;
    in_g = n % per_group;
  }
  Work3 w;
  w.x = in_g % nx;
  w.y = (grp % groups_per_z) * gy + in_g / nx;
  w.z = grp / groups_per_z;
  return w;
}

}  // namespace

// ------------------------------------------------------------------------------------------------
// forward
// ------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256, blocks_per_cu(D, 4, 2)) void attn_fwd_mfma_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out,
                                                            float* __restrict__ lse, int Smax, int nh, int nkv,
                                                            const int* __restrict__ cu, int64_t T, int nseq) {
  constexpr int NK = D / 16, NC = D / 32;   // k16 steps of a score product, 32-column tiles of a result
  constexpr int KV_TILE = kv_tile(D);
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  bf16_t* sK = smem;                 // [2][KV_TILE]
  bf16_t* sV = smem + 2 * KV_TILE;   // [2][KV_TILE]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, g = lane >> 5, plr = perm(lr);
  const int nqb = (Smax + BQ - 1) / BQ;
  const Work3 wk = xcd_group_work(nqb, nh, nseq, nh / nkv);
  const int qb = nqb - 1 - wk.x;  // heavy (late) query blocks first
  const int h = wk.y, b = wk.z;
  const SeqView sv = seq_view(cu, b, Smax, T);
  const int S = sv.len;
  const int G = nh / nkv, kh = h / G;
  const int ld = (nh + 2 * nkv) * D;
  const int q0 = qb * BQ, qw = q0 + wave * 32, iq = qw + lr;
  if (q0 >= S) return;   // the whole block, before any barrier: this sequence is shorter
  const bf16_t* base = qkv + (size_t)sv.row0 * ld;
  const __amdgpu_buffer_rsrc_t rs = rsrc(base, (uint32_t)((size_t)S * ld * 2));
  const int kcol = (nh + kh) * D, vcol = (nh + nkv + kh) * D;
  const float c = kLog2e / sqrtf((float)D);

  u32x4_t qf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)
    qf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)iq * (uint32_t)ld + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));

  f32x16_t o[NC];
#pragma unroll
  for (int ct = 0; ct < NC; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) o[ct][q] = 0.f;
  float m = -INFINITY, l = 0.f;   // l: this lane's share of the row's sum (its partner, lane ^ 32, has the rest)

  const int kv_end = min(S, q0 + BQ);
  const int nt = (kv_end + BKV - 1) / BKV;
  const uint32_t seq_bytes = (uint32_t)((size_t)S * ld * 2);
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  TileDma<64, D> dma;
  dma.init(ld, wave, lane);
  auto fetch_k = [&](int t) {
    if (t < nt) dma.issue(base, seq_bytes, sK + (t & 1) * KV_TILE, ((uint32_t)(t * BKV) * (uint32_t)ld + (uint32_t)kcol) * 2u, wave_s);
  };
  auto fetch_v = [&](int t) {
    if (t < nt) dma.issue(base, seq_bytes, sV + (t & 1) * KV_TILE, ((uint32_t)(t * BKV) * (uint32_t)ld + (uint32_t)vcol) * 2u, wave_s);
  };
  // The sums are kept relative to m, which follows the running maximum of the row.  At head size 64 it may fall behind by 2^8: the
  // accumulators are then rescaled once or twice per row, not in nearly every tile (one of 32 rows nearly always finds a new
  // maximum; 6 x 777 30.4 -> 29.0 us).  At head size 128, where a probability is one bf16 value, that of the largest score has to
  // stay the exact 1 it is relative to the maximum itself: with a lag the results were 2 % (flat scores) to 17 % (peaked ones) further from
  // 64 bits (and 16 x 2048 took 700 us, 745 without).
  auto follow = [&](float tm) {
    const bool moved = (tm - m) * c > lag(D);   // the first tile: m = -inf, and key 0 is visible to every query
    if (__builtin_amdgcn_ballot_w64(moved) != 0) {   // wave-uniform
      const float mn = moved ? tm : m, alpha = __builtin_amdgcn_exp2f((m - mn) * c);
      l *= alpha;
      m = mn;
#pragma unroll
      for (int ct = 0; ct < NC; ++ct)
#pragma unroll
        for (int q = 0; q < 16; ++q) o[ct][q] *= alpha;
    }
  };
  constexpr int RING = 4, NP = parts(D);
  auto k_frag = [&](const bf16_t* K, int i) { return frag<D>(K, (i / NK) * 32, plr, (i % NK) * 16 + g * 8); };
  fetch_k(0);
  if constexpr (D == 64) fetch_v(0);
  // vmcnt(0): nothing of the prologue is in flight inside the loop.  The Q (and dO) fragments are first used there, so
  // the compiler issues their loads last and, at the loop's head, still counts them as outstanding; inside the loop
  // the next tile's eight loads are then younger than they are, and the waits it puts in front of the first MFMAs
  // ("all but 7, 6, ... 0 loads done") make every tile wait for the tile after it to arrive from memory.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();
  if constexpr (D == 64) {
    // Four blocks share a CU (the pipelined form below needs 197 registers, two blocks: 16 x 2048, 32 / 8 heads 541 -> 574 us).
    for (int t = 0; t < nt; ++t) {
      const int j0 = t * BKV;
      fetch_k(t + 1);   // into the stage whose last readers passed the barrier at the end of the step before
      fetch_v(t + 1);
      if (j0 <= qw + 31) {  // wave-uniform: the tile has at least one unmasked key for this wave
        const bf16_t* K = sK + (t & 1) * KV_TILE;
        const bf16_t* V = sV + (t & 1) * KV_TILE;
        f32x16_t s[2];
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)
#pragma unroll
          for (int q = 0; q < 16; ++q) s[jt][q] = 0.f;
        {
          // the K fragments through a ring: a fragment is requested RING MFMAs before its own (read, wait, MFMA one after
          // the other leaves the LDS latency, three MFMA times, exposed at every step)
          u32x4_t kb[RING];
#pragma unroll
          for (int i = 0; i < RING; ++i) kb[i] = k_frag(K, i);
#pragma unroll
          for (int i = 0; i < 2 * NK; ++i) {
            s[i / NK] = mfma(kb[i % RING], qf[i % NK], s[i / NK]);
            if (i + RING < 2 * NK) kb[i % RING] = k_frag(K, i + RING);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (j0 + BKV - 1 > qw) {  // the tile touches the diagonal of this wave
#pragma unroll
          for (int jt = 0; jt < 2; ++jt)
#pragma unroll
            for (int q = 0; q < 16; ++q)
              if (j0 + jt * 32 + acc_row(q, g) > iq) s[jt][q] = -INFINITY;
        }
        float tm = -INFINITY;
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)
#pragma unroll
          for (int q = 0; q < 16; ++q) tm = fmaxf(tm, s[jt][q]);
        follow(row_max(tm));
        const float mc = m * c;
        float ps[2] = {0.f, 0.f};
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            const float p = __builtin_amdgcn_exp2f(s[jt][q] * c - mc);
            s[jt][q] = p;
            ps[q & 1] += p;
          }
        l += ps[0] + ps[1];
        u32x4_t pf[4][NP];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) pack_parts(s[ks >> 1], ks & 1, pf[ks]);
#pragma unroll
        for (int ct = 0; ct < NC; ++ct)
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) o[ct] = mfma_parts(frag_tr<D>(V, ks * 16, ct * 32, lane), pf[ks], o[ct]);
      }
      TIDE_ATTN_WAIT_DMA();
      __syncthreads();
    }
  } else {
    fetch_k(1);
    fetch_v(0);

    // One tile is two MFMA phases: the scores of tile t + 1 (2 NK MFMAs) beside the exponentials of tile t, then its P V beside
    // the row maxima of the scores just made.  The order of MFMAs, operand reads (a ring of four fragments) and vector
    // instructions is written out and pinned: left to two waves of a SIMD that took turns by chance, the matrix pipes were 40 % and
    // the vector units 50 % busy, one after the other.  us before / now: 16 x 2048, 32 / 8 heads 770 / 745, 4 x 1024 68.6 / 65.1
    // (the larger one sits at the power limit: without exponentials it takes 7 % less, without operand reads 11).
    // A ring of six: the same; of eight: spills.  The same order in the dQ kernel (halves of a tile) gave nothing.
    constexpr int NS = 2 * NK, EPM = 32 / NS;   // MFMAs of a score tile, exponentials beside each
    f32x16_t sa[2], sb[2];
    float tma = -INFINITY, tmb = -INFINITY;   // this lane's maximum of sa, sb
    auto v_frag = [&](const bf16_t* V, int i) { return frag_tr<D>(V, (i / NC) * 16, (i % NC) * 32, lane); };   // k16 step i / NC, columns i % NC
    {
      const bf16_t* K = sK;   // tile 0: every wave sees key 0
      u32x4_t kb[RING];
#pragma unroll
      for (int i = 0; i < RING; ++i) kb[i] = k_frag(K, i);
#pragma unroll
      for (int jt = 0; jt < 2; ++jt)
#pragma unroll
        for (int q = 0; q < 16; ++q) sa[jt][q] = 0.f;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        sa[i / NK] = mfma(kb[i % RING], qf[i % NK], sa[i / NK]);
        if (i + RING < NS) kb[i % RING] = k_frag(K, i + RING);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < 32; ++q) tma = fmaxf(tma, sa[q / 16][q % 16]);
    }
    TIDE_ATTN_WAIT_DMA();
    __syncthreads();

    auto step = [&](f32x16_t (&s)[2], float tm, f32x16_t (&sn)[2], float& tmn, int t) {
      const int j0 = t * BKV;
      // (K(t) was last read in the step before, V(t - 1) as well: the barrier at its end has passed)
      auto fetch = [&] { fetch_k(t + 2); fetch_v(t + 1); };
      if (j0 > qw + 31) {
        fetch();
      } else {   // wave-uniform: the tile has at least one unmasked key for this wave
        const bf16_t* K = sK + ((t + 1) & 1) * KV_TILE;
        const bf16_t* V = sV + (t & 1) * KV_TILE;
        const bool more = t + 1 < nt && j0 + BKV <= qw + 31;   // the next tile has one, too
        u32x4_t ring[RING];
        if (more) {
#pragma unroll
          for (int i = 0; i < RING; ++i) ring[i] = k_frag(K, i);
        }
        __builtin_amdgcn_sched_barrier(0);
        fetch();   // behind the first operand reads, which arrive meanwhile
        if (j0 + BKV - 1 > qw) {  // the tile touches the diagonal of this wave
          tm = -INFINITY;
#pragma unroll
          for (int jt = 0; jt < 2; ++jt)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
              if (j0 + jt * 32 + acc_row(q, g) > iq) s[jt][q] = -INFINITY;
              tm = fmaxf(tm, s[jt][q]);
            }
        }
        tm = row_max(tm);
        follow(tm);
        const float mc = m * c;
        u32x4_t pf[4][NP];
        float ps[2] = {0.f, 0.f};
        float mcx = mc;
        auto prob = [&](int e) {   // element e = 0 .. 31 of the lane; every eighth completes an operand of P V
          const float p = __builtin_amdgcn_exp2f(fmaf(s[e / 16][e % 16], c, -mcx));
          s[e / 16][e % 16] = p;
          ps[e & 1] += p;
        };
        if (more) {
          asm volatile("" : "+v"(mcx));   // (or the multiply-adds, which both branches have, move out of them and ahead of the MFMAs)
#pragma unroll
          for (int jt = 0; jt < 2; ++jt)
#pragma unroll
            for (int q = 0; q < 16; ++q) sn[jt][q] = 0.f;
#pragma unroll
          for (int i = 0; i < NS; ++i) {
            sn[i / NK] = mfma(ring[i % RING], qf[i % NK], sn[i / NK]);
            ring[i % RING] = i + RING < NS ? k_frag(K, i + RING) : v_frag(V, i + RING - NS);
#pragma unroll
            for (int u = 0; u < EPM; ++u) prob(i * EPM + u);
            if ((i + 1) * EPM % 8 == 0) pack_parts(s[i * EPM / 16], i * EPM % 16 / 8, pf[i * EPM / 8]);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
          for (int i = 0; i < RING; ++i) ring[i] = v_frag(V, i);
#pragma unroll
          for (int e = 0; e < 32; ++e) prob(e);
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) pack_parts(s[ks >> 1], ks & 1, pf[ks]);
        }
        l += ps[0] + ps[1];
        matrix_phase<D>(true);
        constexpr int NV = 4 * NC, MPM = (32 + NV - 1) / NV;   // fragments of V, maxima beside each
        float mx[2] = {-INFINITY, -INFINITY};
        auto pv = [&](auto MORE) {
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            o[i % NC] = mfma_parts(ring[i % RING], pf[i / NC], o[i % NC]);
            if (i + RING < NV) ring[i % RING] = v_frag(V, i + RING);
            if constexpr (decltype(MORE)::value) {
#pragma unroll
              for (int u = 0; u < MPM; ++u) {
                const int e = i * MPM + u;
                if (e < 32) mx[u & 1] = fmaxf(mx[u & 1], sn[e / 16][e % 16]);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        if (more) pv(std::true_type{});
        else pv(std::false_type{});
        matrix_phase<D>(false);
        tmn = fmaxf(mx[0], mx[1]);
      }
      TIDE_ATTN_WAIT_DMA();
      __syncthreads();
    };
    for (int t = 0; t < nt; t += 2) {
      step(sa, tma, sb, tmb, t);
      if (t + 1 < nt) step(sb, tmb, sa, tma, t + 1);
    }
  }
  l += swap_halves(l);

  const float inv = 1.0f / l;
  stage_out<D>(smem, o, inv, wave, lane);
  if constexpr (D == 64) {
    // A masked key has probability zero, but zero times a NaN or an infinity of its V row is a NaN that reaches the earlier
    // queries of its tile.  Rows that are not finite although their sum is are made again from the keys they see alone,
    // a channel per lane.  No row of finite inputs is, and 32 multiply-adds per lane and block find out.
    for (uint32_t rows = not_finite(o, l - l == 0.f && iq < S); rows != 0; rows &= rows - 1) {   // wave-uniform
      const int r = __builtin_ctz(rows);
      const float mr = __shfl(m, r, 64), ir = __shfl(inv, r, 64);
      const float qv = bf2f(base[(size_t)(qw + r) * ld + h * D + lane]);
      float acc = 0.f;
#pragma unroll 1
      for (int j = 0; j <= qw + r; ++j) {   // below S
        const bf16_t* row = base + (size_t)j * ld;
        acc += __builtin_amdgcn_exp2f((wave_sum(qv * bf2f(row[kcol + lane])) - mr) * c) * bf2f(row[vcol + lane]);
      }
      asm volatile("" ::: "memory");   // after the wave's own wider stores of the row
      smem[(wave * 32 + r) * pitch(D) + lane] = f2bf(acc * ir);
    }
  }
  if (g == 0 && iq < S) lse[stat_index(cu, T, sv, b, h, nh, Smax, iq)] = m * (1.0f / sqrtf((float)D)) + logf(l);
  __syncthreads();
  copy_out<D>(smem, out, sv.row0 + q0, sv.row0 + min(S, q0 + BQ), nh * D, h * D, tid);
}

// ------------------------------------------------------------------------------------------------
// backward, dQ: same streaming structure as the forward pass.  It also makes delta = rowsum(dO * O), which the dK / dV
// passes read: the dO fragments are in registers anyway, so O is all that is loaded for it (a pass of its own
// read dO again: 100 us at 16 x 2048, 32 heads, against 45 us more in this kernel).
// ------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256, blocks_per_cu(D, 3, 2)) void attn_dq_mfma_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ out, const bf16_t* __restrict__ dout,
                                                           const float* __restrict__ lse, float* __restrict__ delta,
                                                           bf16_t* __restrict__ dqkv, int Smax, int nh, int nkv,
                                                           const int* __restrict__ cu, int64_t T, int nseq) {
  constexpr int NK = D / 16, NC = D / 32;   // k16 steps of a score product, 32-column tiles of a result
  constexpr int KV_TILE = kv_tile(D);
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  bf16_t* sK = smem;
  bf16_t* sV = smem + 2 * KV_TILE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, g = lane >> 5, plr = perm(lr);
  const int nqb = (Smax + BQ - 1) / BQ;
  const Work3 wk = xcd_group_work(nqb, nh, nseq, nh / nkv);
  const int qb = nqb - 1 - wk.x;
  const int h = wk.y, b = wk.z;
  const SeqView sv = seq_view(cu, b, Smax, T);
  const int S = sv.len;
  const int G = nh / nkv, kh = h / G;
  const int ld = (nh + 2 * nkv) * D, ldo = nh * D;
  const int q0 = qb * BQ, qw = q0 + wave * 32, iq = qw + lr;
  if (q0 >= S) return;   // the whole block, before any barrier
  const __amdgpu_buffer_rsrc_t rs = rsrc(qkv + (size_t)sv.row0 * ld, (uint32_t)((size_t)S * ld * 2));
  const __amdgpu_buffer_rsrc_t rso = rsrc(dout + (size_t)sv.row0 * ldo, (uint32_t)((size_t)S * ldo * 2));
  const int kcol = (nh + kh) * D, vcol = (nh + nkv + kh) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const float c = kLog2e * scale;

  u32x4_t qf[NK], dof[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    qf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)iq * (uint32_t)ld + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));
    dof[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rso, ((uint32_t)iq * (uint32_t)ldo + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));
  }
  const bool valid = iq < S;
  const bool edge_q = qw + 32 > S;   // wave-uniform: some query row of this wave lies past the sequence
  const float lse_i = valid ? lse[stat_index(cu, T, sv, b, h, nh, Smax, iq)] * kLog2e : 0.f;
  float del_i = 0.f;   // a row past the end loads zeros
  {
    const __amdgpu_buffer_rsrc_t rsout = rsrc(out + (size_t)sv.row0 * ldo, (uint32_t)((size_t)S * ldo * 2));
    u32x4_t of[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
      of[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsout, ((uint32_t)iq * (uint32_t)ldo + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        del_i = fmaf(__uint_as_float(of[kk][w] << 16), __uint_as_float(dof[kk][w] << 16), del_i);
        del_i = fmaf(__uint_as_float(of[kk][w] & 0xFFFF0000u), __uint_as_float(dof[kk][w] & 0xFFFF0000u), del_i);
      }
    del_i += __shfl_xor(del_i, 32, 64);
    if (valid && g == 0) delta[stat_index(cu, T, sv, b, h, nh, Smax, iq)] = del_i;
  }

  f32x16_t dq[NC];
#pragma unroll
  for (int ct = 0; ct < NC; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) dq[ct][q] = 0.f;

  const int kv_end = min(S, q0 + BQ);
  const int nt = (kv_end + BKV - 1) / BKV;
  const bf16_t* seq = qkv + (size_t)sv.row0 * ld;
  const uint32_t seq_bytes = (uint32_t)((size_t)S * ld * 2);
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  TileDma<64, D> dma;
  dma.init(ld, wave, lane);
  dma.issue(seq, seq_bytes, sK, (uint32_t)kcol * 2u, wave_s);
  dma.issue(seq, seq_bytes, sV, (uint32_t)vcol * 2u, wave_s);
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): nothing of the prologue is in flight inside the loop (see the forward kernel)
  __syncthreads();

  for (int t = 0; t < nt; ++t) {
    const int st = t & 1;
    const int j0 = t * BKV;
    if (t + 1 < nt) {
      const uint32_t row_bytes = (uint32_t)(j0 + BKV) * (uint32_t)ld * 2u;
      dma.issue(seq, seq_bytes, sK + (st ^ 1) * KV_TILE, row_bytes + (uint32_t)kcol * 2u, wave_s);
      dma.issue(seq, seq_bytes, sV + (st ^ 1) * KV_TILE, row_bytes + (uint32_t)vcol * 2u, wave_s);
    }
    if (j0 <= qw + 31) {
      const bf16_t* K = sK + st * KV_TILE;
      const bf16_t* V = sV + st * KV_TILE;
      const bool diag = j0 + BKV - 1 > qw;
      u32x4_t dsf[4][parts(D)];
#pragma unroll
      for (int jt = 0; jt < 2; ++jt) {
        f32x16_t s, dp;
#pragma unroll
        for (int q = 0; q < 16; ++q) { s[q] = 0.f; dp[q] = 0.f; }
#if TIDE_ATTN_DQ_RING == 0
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
          s = mfma(frag<D>(K, jt * 32, plr, kk * 16 + g * 8), qf[kk], s);
          dp = mfma(frag<D>(V, jt * 32, plr, kk * 16 + g * 8), dof[kk], dp);
        }
#else
        {
          // K and V fragments alternately through a ring, each requested TIDE_ATTN_DQ_RING MFMAs ahead (see the forward kernel)
          constexpr int RING = TIDE_ATTN_DQ_RING;
          u32x4_t fb[RING];
          auto fetch = [&](int i) { return frag<D>((i & 1) ? V : K, jt * 32, plr, (i >> 1) * 16 + g * 8); };
#pragma unroll
          for (int i = 0; i < RING; ++i) fb[i] = fetch(i);
#pragma unroll
          for (int i = 0; i < 2 * NK; ++i) {
            if (i & 1) dp = mfma(fb[i % RING], dof[i >> 1], dp);
            else s = mfma(fb[i % RING], qf[i >> 1], s);
            if (i + RING < 2 * NK) fb[i % RING] = fetch(i + RING);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#endif
        if (diag || edge_q) {   // wave-uniform: only a tile on the diagonal or the last query block needs per-element tests (-4.5 %)
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            float p = __builtin_amdgcn_exp2f(s[q] * c - lse_i);
            if (!valid || (diag && (j0 + jt * 32 + acc_row(q, g) > iq))) p = 0.f;
            s[q] = p * (dp[q] - del_i);
          }
        } else {
#pragma unroll
          for (int q = 0; q < 16; ++q) s[q] = __builtin_amdgcn_exp2f(s[q] * c - lse_i) * (dp[q] - del_i);
        }
        pack_parts(s, 0, dsf[2 * jt]);
        pack_parts(s, 1, dsf[2 * jt + 1]);
      }
      matrix_phase<D>(true);
#pragma unroll
      for (int ct = 0; ct < NC; ++ct)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dq[ct] = mfma_parts(frag_tr<D>(K, ks * 16, ct * 32, lane), dsf[ks], dq[ct]);
      matrix_phase<D>(false);
    }
    TIDE_ATTN_WAIT_DMA();
    __syncthreads();
  }
  stage_out<D>(smem, dq, scale, wave, lane);
  if constexpr (D == 64) {
    // as in the forward kernel: a later key of the tile that is not finite
    const uint32_t again = not_finite(dq, valid && lse_i - lse_i == 0.f && del_i - del_i == 0.f);
    for (uint32_t rows = again; rows != 0; rows &= rows - 1) {   // wave-uniform
      const int r = __builtin_ctz(rows);
      const float L = __shfl(lse_i, r, 64), De = __shfl(del_i, r, 64);
      const bf16_t* base = qkv + (size_t)sv.row0 * ld;
      const float qv = bf2f(base[(size_t)(qw + r) * ld + h * D + lane]), dov = bf2f(dout[((size_t)sv.row0 + qw + r) * ldo + h * D + lane]);
      float acc = 0.f;
#pragma unroll 1
      for (int j = 0; j <= qw + r; ++j) {   // below S
        const bf16_t* row = base + (size_t)j * ld;
        const float kv = bf2f(row[kcol + lane]), p = __builtin_amdgcn_exp2f(wave_sum(qv * kv) * c - L);
        acc += p * (wave_sum(dov * bf2f(row[vcol + lane])) - De) * kv;
        if (__builtin_amdgcn_ballot_w64(acc - acc == 0.f) == 0) break;
      }
      asm volatile("" ::: "memory");   // after the wave's own wider stores of the row
      smem[(wave * 32 + r) * pitch(D) + lane] = f2bf(acc * scale);
    }
  }
  __syncthreads();
  copy_out<D>(smem, dqkv, sv.row0 + q0, sv.row0 + min(S, q0 + BQ), ld, h * D, tid);
}

// ------------------------------------------------------------------------------------------------
// backward, dK and dV
// ------------------------------------------------------------------------------------------------
namespace {
// Query rows per streamed tile (32 or 64: two halves of 32 between two barriers) of the dV and of the dK pass.
// Measured, backward at 16 x 2048 / 2 x 16384 (dV rows / dK rows): 32 / 32: 3.18 / 18.2 ms; 32 / 64: 3.08 / 18.0;
// 64 / 32: 3.14 / 18.7; 64 / 64: 3.09 / 18.5 (with 64 rows the dV pass loses its third block per CU to the LDS).
#ifndef TIDE_ATTN_DV_ROWS
#define TIDE_ATTN_DV_ROWS 32
#endif
#ifndef TIDE_ATTN_DK_ROWS
#define TIDE_ATTN_DK_ROWS 64
#endif
// (with several sets of waves per block, 32 in both passes: the sets' stages have to fit the LDS)
template <int WHICH, int NS>
constexpr int dkv_rows() { return WHICH == 1 && NS == 1 ? TIDE_ATTN_DK_ROWS : TIDE_ATTN_DV_ROWS; }
template <int BI, int D> struct DkvStage {
  static constexpr int Q_TILE = TileDma<BI, D>::CHUNKS * 512;   // elements: the tile rounded up to whole 1 KiB chunks of the LDS-DMA loads
  static constexpr int STAGE = 2 * Q_TILE + 4 * BI;          // Q tile, dO tile, then lse[BI] and delta[BI] as floats
};
}  // namespace

// Two forms of a block.  KW = 4, NS = 1: 128 keys on four waves, every wave walks all query tiles; two or three blocks
// share a CU and hide each other's waits.  With few blocks (a handful of sequences) there is nobody to share with, and the
// pass takes as long as the longest chain of query tiles, G heads times the sequence: KW = 2, NS = 4 has 64 keys on two
// waves, four such sets, each with LDS stages of its own, take every fourth query tile, and the sets' sums are added through
// LDS at the end, in a fixed order.
constexpr int kFewKW = 2, kFewNS = 4;
// One gradient per pass (WHICH = 0: dV, 1: dK).  Half the accumulators and, for dV, half the operand
// registers of the fused kernel: the pass fits 256 VGPRs, two blocks share a CU, and one block's
// exponentials overlap the other's MFMAs.  The price is that S = Q K^T is computed in both passes.
template <int WHICH, int D, int KW, int NS>
__global__ __launch_bounds__(KW * NS * 64, NS > 1 ? 1 : WHICH == 0 ? blocks_per_cu(D, 4, 3) : blocks_per_cu(D, 3, 2)) void attn_dkv_mfma_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dout,
                                                            const float* __restrict__ lse, const float* __restrict__ delta,
                                                            bf16_t* __restrict__ dqkv, int Smax, int nh, int nkv,
                                                            const int* __restrict__ cu, int64_t T, int nseq) {
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  constexpr int KB = KW * 32, SET = KW * 64;   // keys of the block, threads of a set
  const int set = NS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / SET) : 0;
  const int tid = threadIdx.x - set * SET, lane = tid & 63, wave = tid >> 6;   // inside the set
  const int lr = lane & 31, g = lane >> 5, plr = perm(lr);
  const Work3 wk = xcd_group_work((Smax + KB - 1) / KB, nkv, nseq, 1);
  const int jb = wk.x, kh = wk.y, b = wk.z;  // early key blocks are the heavy ones
  const SeqView sv = seq_view(cu, b, Smax, T);
  const int S = sv.len;
  const int G = nh / nkv;
  const int ld = (nh + 2 * nkv) * D, ldo = nh * D;
  const int j0 = jb * KB, jw = j0 + wave * 32, jk = jw + lr;
  if (j0 >= S) return;   // the whole block, before any barrier
  const __amdgpu_buffer_rsrc_t rs = rsrc(qkv + (size_t)sv.row0 * ld, (uint32_t)((size_t)S * ld * 2));
  const int kcol = (nh + kh) * D, vcol = (nh + nkv + kh) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const float c = kLog2e * scale;

  constexpr bool DK = WHICH == 1;
  constexpr int BI = dkv_rows<WHICH, NS>();
  constexpr int NK = D / 16, NC = D / 32;
  constexpr int Q_TILE = DkvStage<BI, D>::Q_TILE, DKV_STAGE = DkvStage<BI, D>::STAGE;
  u32x4_t kf[NK], vf[DK ? NK : 1];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    kf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)jk * (uint32_t)ld + (uint32_t)(kcol + kk * 16 + g * 8)) * 2u, 0, 0));
    if constexpr (DK) vf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)jk * (uint32_t)ld + (uint32_t)(vcol + kk * 16 + g * 8)) * 2u, 0, 0));
  }
  f32x16_t dacc[NC];   // dK or dV of this wave's 32 keys
#pragma unroll
  for (int ct = 0; ct < NC; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) dacc[ct][q] = 0.f;

  const int i_begin = (j0 / BI) * BI;                  // first query tile that can see a key of this block
  const int nit = (S - i_begin + BI - 1) / BI;         // query tiles per head
  const int ntiles = G * nit;

  const bf16_t *seq = qkv + (size_t)sv.row0 * ld, *seq_do = dout + (size_t)sv.row0 * ldo;
  const uint32_t seq_bytes = (uint32_t)((size_t)S * ld * 2), seq_do_bytes = (uint32_t)((size_t)S * ldo * 2);
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  TileDma<BI, D, KW> dmq, dmo;   // LDS-DMA loads of the Q and the dO tile (their row pitches in memory differ)
  dmq.init(ld, wave, lane);
  dmo.init(ldo, wave, lane);
  bf16_t* stages = smem + set * 2 * DKV_STAGE;
  float stat = 0.f;  // threads 0..BI-1 carry lse, BI..2BI-1 carry delta of the staged tile
  // Query tiles are walked from the END of the sequence down to the first one that sees this block's keys: the key
  // blocks of a kv head run side by side on one XCD, and this way all of them want the same Q / dO tile at about
  // the same time (walking up from each block's own first tile, they were spread over the whole sequence and the
  // passes fetched nearly every tile through the fabric: 3.8 GB per launch at the 8B shape, L2 hits 21 %).
  // (and tile by tile over the G query heads, not head by head: blocks with fewer tiles would otherwise move on
  // to the next head early)
  auto tile_i0 = [&](int u) { return i_begin + (nit - 1 - u / G) * BI; };
  auto gload = [&](int u, int st) {   // tile u into stage st (whose last readers have passed a barrier)
    const int hh = kh * G + u % G;
    const int i0 = tile_i0(u);
    bf16_t* base = stages + st * DKV_STAGE;
    dmq.issue(seq, seq_bytes, base, ((uint32_t)i0 * (uint32_t)ld + (uint32_t)(hh * D)) * 2u, wave_s);
    dmo.issue(seq_do, seq_do_bytes, base + Q_TILE, ((uint32_t)i0 * (uint32_t)ldo + (uint32_t)(hh * D)) * 2u, wave_s);
    if (tid < 2 * BI) {
      const int i = i0 + (tid & (BI - 1));
      const float* src = (tid < BI) ? lse : delta;
      // (used in sstore only: the load stays in flight; a row past the sequence gets lse = +inf there, delta = 0)
      stat = (i < S) ? src[stat_index(cu, T, sv, b, hh, nh, Smax, i)] : ((tid < BI) ? INFINITY : 0.f);
    }
  };
  auto sstore = [&](int st) {
    bf16_t* base = stages + st * DKV_STAGE;
    if (tid < 2 * BI) reinterpret_cast<float*>(base + 2 * Q_TILE)[tid] = stat * ((tid < BI) ? kLog2e : 1.f);   // lse * log2(e), delta
  };

  if (NS == 1 || set < ntiles) {   // (one set: there is always a tile)
    gload(set, 0);
    sstore(0);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the tile and the K / V fragments have arrived before the loop
  __syncthreads();
  // (the sets' trip counts differ by one at most: every set passes every barrier)
  for (int r = 0; r * NS < ntiles; ++r) {
    const int st = r & 1, u = r * NS + set;
    if (u + NS < ntiles) gload(u + NS, st ^ 1);
    const int it0 = NS == 1 || u < ntiles ? tile_i0(u) : S;   // past the end: no half of the tile is entered
#pragma unroll
    for (int hf = 0; hf < BI / 32; ++hf) {
    const int i0 = it0 + hf * 32;   // this half's first query
    if (i0 + 31 >= jw && i0 < S) {  // wave-uniform: some query of the half sees some key of this wave
      const bf16_t* Qt = stages + st * DKV_STAGE;
      const bf16_t* dOt = Qt + Q_TILE;
      const float* stats = reinterpret_cast<const float*>(Qt + 2 * Q_TILE) + hf * 32;
      f32x16_t s, dp;
#pragma unroll
      for (int q = 0; q < 16; ++q) { s[q] = 0.f; dp[q] = 0.f; }
      {
        // Q (and, in the dK pass, dO) fragments through a ring, each requested TIDE_ATTN_DKV_RING MFMAs ahead
        constexpr int RING = TIDE_ATTN_DKV_RING, NF = DK ? 2 * NK : NK;
        u32x4_t fb[RING];
        auto fetch = [&](int i) {
          if constexpr (DK) return frag<D>((i & 1) ? dOt : Qt, hf * 32, plr, (i >> 1) * 16 + g * 8);
          else return frag<D>(Qt, hf * 32, plr, i * 16 + g * 8);
        };
#pragma unroll
        for (int i = 0; i < RING; ++i) fb[i] = fetch(i);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          if constexpr (DK) {
            if (i & 1) dp = mfma(fb[i % RING], vf[i >> 1], dp);
            else s = mfma(fb[i % RING], kf[i >> 1], s);
          } else {
            s = mfma(fb[i % RING], kf[i], s);
          }
          if (i + RING < NF) fb[i % RING] = fetch(i + RING);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // Rows past the end of the sequence carry lse = +inf (see sstore), i.e. p = 0 without a test; the causal test is
      // per element, and only a half that touches the diagonal makes it (wave-uniform branch).
      const bool diag = i0 < jw + 32;  // some (query, key) pair of the half is above the diagonal
      auto probs = [&](auto MASK) {
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          const float4 l4 = *reinterpret_cast<const float4*>(stats + 8 * qq + 4 * g);   // lse * log2(e), see sstore
          const float4 d4 = *reinterpret_cast<const float4*>(stats + BI + 8 * qq + 4 * g);
          const float lv4[4] = {l4.x, l4.y, l4.z, l4.w}, dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int q = qq * 4 + e;
            float p = __builtin_amdgcn_exp2f(s[q] * c - lv4[e]);
            if constexpr (decltype(MASK)::value) {
              if (i0 + 8 * qq + 4 * g + e < jk) p = 0.f;
            }
            s[q] = DK ? p * (dp[q] - dv4[e]) : p;   // dS for the dK pass, P for the dV pass
          }
        }
      };
      if (diag) probs(std::true_type{});
      else probs(std::false_type{});
      u32x4_t pf[2][parts(D)];
      pack_parts(s, 0, pf[0]);
      pack_parts(s, 1, pf[1]);
      const bf16_t* Xt = DK ? Qt : dOt;   // dK += dS^T Q, dV += P^T dO
      matrix_phase<D>(true);
#pragma unroll
      for (int ct = 0; ct < NC; ++ct)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) dacc[ct] = mfma_parts(frag_tr<D>(Xt, hf * 32 + ks * 16, ct * 32, lane), pf[ks], dacc[ct]);
      matrix_phase<D>(false);
    }
    }
    if (u + NS < ntiles) sstore(st ^ 1);
    TIDE_ATTN_WAIT_DMA();
    __syncthreads();
  }
  if constexpr (NS > 1) {
    // sets n .. 2n - 1 hand their sums to sets 0 .. n - 1, for n = NS / 2, NS / 4, ... (every stage is free by now)
    float* sums = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int n = NS / 2; n >= 1; n /= 2) {
      float* mine = sums + ((size_t)((set % n) * KW + wave) * NC * 16) * 64 + lane;
      if (set >= n && set < 2 * n) {
#pragma unroll
        for (int ct = 0; ct < NC; ++ct)
#pragma unroll
          for (int q = 0; q < 16; ++q) mine[(ct * 16 + q) * 64] = dacc[ct][q];
      }
      __syncthreads();
      if (set < n) {
#pragma unroll
        for (int ct = 0; ct < NC; ++ct)
#pragma unroll
          for (int q = 0; q < 16; ++q) dacc[ct][q] += mine[(ct * 16 + q) * 64];
      }
      __syncthreads();
    }
  }
  const int64_t r0 = sv.row0 + j0, r1 = sv.row0 + min(S, j0 + KB);
  if (set == 0) {
    stage_out<D>(smem, dacc, DK ? scale : 1.0f, wave, lane);
    if constexpr (D == 64) {
      // As in the forward kernel, from the other side: the queries jw .. j - 1 meet key j with weight zero.  Keys after the
      // first of them that is not finite are made again from the queries that see them alone (a later query takes every
      // key before it with it, rightly).
      uint32_t rows = not_finite(dacc, jk < S);
      const bf16_t *base = qkv + (size_t)sv.row0 * ld, *dob = dout + (size_t)sv.row0 * ldo;
      if (rows != 0) {   // wave-uniform
        int first = 31;
#pragma unroll 1
        for (int i = 0; i < first && jw + i < S; ++i) {
          float odd = 0.f;
          for (int hh = kh * G; hh < (kh + 1) * G; ++hh)
            odd += 0.f * (bf2f(base[(size_t)(jw + i) * ld + hh * D + lane]) + bf2f(dob[(size_t)(jw + i) * ldo + hh * D + lane]) +
                          delta[stat_index(cu, T, sv, b, hh, nh, Smax, jw + i)]);
          if (__builtin_amdgcn_ballot_w64(odd != 0.f) != 0) first = i;
        }
        rows &= first == 31 ? 0u : ~((2u << first) - 1u);
      }
      for (; rows != 0; rows &= rows - 1) {
        const int r = __builtin_ctz(rows), j = jw + r;
        const float kv = bf2f(base[(size_t)j * ld + kcol + lane]), vv = bf2f(base[(size_t)j * ld + vcol + lane]);
        float acc = 0.f;
        for (int hh = kh * G; hh < (kh + 1) * G && __builtin_amdgcn_ballot_w64(acc - acc == 0.f) != 0; ++hh)
#pragma unroll 1
          for (int i = j; i < S; ++i) {
            const float qv = bf2f(base[(size_t)i * ld + hh * D + lane]), dov = bf2f(dob[(size_t)i * ldo + hh * D + lane]);
            const size_t at = stat_index(cu, T, sv, b, hh, nh, Smax, i);
            const float p = __builtin_amdgcn_exp2f(wave_sum(qv * kv) * c - lse[at] * kLog2e);
            acc += DK ? p * (wave_sum(dov * vv) - delta[at]) * qv : p * dov;
            if (__builtin_amdgcn_ballot_w64(acc - acc == 0.f) == 0) break;
          }
        asm volatile("" ::: "memory");   // after the wave's own wider stores of the row
        smem[(wave * 32 + r) * pitch(D) + lane] = f2bf(DK ? acc * scale : acc);
      }
    }
  }
  __syncthreads();
  copy_out<D, KB, SET * NS>(smem, dqkv, r0, r1, ld, DK ? kcol : vcol, threadIdx.x);
}


// ------------------------------------------------------------------------------------------------
bool attn_mfma_supported(const AttnArgs& a) {
  if (a.dtype != kBF16 || (a.dh != 128 && a.dh != 64)) return false;
  if (a.B <= 0 || a.S <= 0 || a.B > 65535 || a.nh > 65535) return false;
  const int64_t ld = (int64_t)(a.nh + 2 * a.nkv) * a.dh;
  if ((int64_t)a.S * ld * 2 >= ((int64_t)1 << 31)) return false;   // 32-bit offsets inside one sequence
  if (((uintptr_t)a.qkv | (uintptr_t)a.out | (uintptr_t)a.dout | (uintptr_t)a.dqkv) & 15) return false;
  if ((int64_t)((a.S + BQ - 1) / BQ) * a.nh * a.B >= ((int64_t)1 << 31)) return false;   // 1-D grids
  return true;
}

namespace {
constexpr size_t fwd_smem(int D) { return (size_t)4 * kv_tile(D) * sizeof(bf16_t); }   // 69632 / 36864 B (>= the 128 x pitch output tile)
template <int WHICH, int D, int KW, int NS>
constexpr size_t dkv_smem() {
  const size_t st = (size_t)NS * 2 * DkvStage<dkv_rows<WHICH, NS>(), D>::STAGE * sizeof(bf16_t), out = (size_t)KW * 32 * pitch(D) * sizeof(bf16_t);
  const size_t sums = NS > 1 ? (size_t)(NS / 2) * KW * (D / 32) * 16 * 64 * sizeof(float) : 0;
  const size_t m = st > out ? st : out;
  return m > sums ? m : sums;
}

hipError_t set_smem(const void* f, size_t bytes, bool& done) {
  if (done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) done = true;
  return e;
}

template <int D>
hipError_t launch_fwd(const AttnArgs& a, hipStream_t s) {
  static bool done = false;
  hipError_t e = set_smem((const void*)attn_fwd_mfma_kernel<D>, fwd_smem(D), done);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((int64_t)((a.S + BQ - 1) / BQ) * a.nh * a.B));   // 1-D: the kernel maps blocks to work itself
  ProfScope ps("attn_fwd_mfma", 2.0 * a.B * a.nh * D * (double)a.S * (a.S + 1), 0, s);
  hipLaunchKernelGGL(attn_fwd_mfma_kernel<D>, grid, dim3(256), fwd_smem(D), s, (const bf16_t*)a.qkv, (bf16_t*)a.out, a.lse, a.S, a.nh, a.nkv, a.cu_seqlens, a.total_rows, a.B);
  return hipGetLastError();
}

template <int WHICH, int D, int KW, int NS>
hipError_t launch_dkv(const AttnArgs& a, hipStream_t s) {
  constexpr size_t smem = dkv_smem<WHICH, D, KW, NS>();
  static_assert(smem <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  const hipError_t e = set_smem((const void*)attn_dkv_mfma_kernel<WHICH, D, KW, NS>, smem, done);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((int64_t)((a.S + KW * 32 - 1) / (KW * 32)) * a.nkv * a.B));
  hipLaunchKernelGGL((attn_dkv_mfma_kernel<WHICH, D, KW, NS>), grid, dim3(KW * NS * 64), smem, s, (const bf16_t*)a.qkv, (const bf16_t*)a.dout, a.lse, a.delta, (bf16_t*)a.dqkv, a.S, a.nh, a.nkv, a.cu_seqlens, a.total_rows, a.B);
  return hipGetLastError();
}

template <int D>
hipError_t launch_bwd(const AttnArgs& a, hipStream_t s) {
  static bool done_q = false;
  hipError_t e = set_smem((const void*)attn_dq_mfma_kernel<D>, fwd_smem(D), done_q);
  if (e != hipSuccess) return e;
  const dim3 gq((unsigned)((int64_t)((a.S + BQ - 1) / BQ) * a.nh * a.B));
  const double pairs = (double)a.B * a.nh * D * (double)a.S * (a.S + 1) / 2.0;  // (query, key, channel) triples
  {
    ProfScope ps("attn_dq_mfma", 6.0 * pairs, 0, s);   // S, dP and dQ products
    hipLaunchKernelGGL(attn_dq_mfma_kernel<D>, gq, dim3(256), fwd_smem(D), s, (const bf16_t*)a.qkv, (const bf16_t*)a.out, (const bf16_t*)a.dout, a.lse, a.delta, (bf16_t*)a.dqkv, a.S, a.nh, a.nkv, a.cu_seqlens, a.total_rows, a.B);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  ProfScope ps("attn_dkv_mfma", 10.0 * pairs, 0, s);   // dV pass: S, dV; dK pass: S, dP, dK
  // blocks of 128 keys that have rows: a packed batch holds at most one partly filled block per sequence
  const int64_t blocks = a.nkv * (a.cu_seqlens ? std::min<int64_t>(a.total_rows / 128 + a.B, (int64_t)((a.S + 127) / 128) * a.B)
                                               : (int64_t)((a.S + 127) / 128) * a.B);
  const int64_t chain = (int64_t)(a.nh / a.nkv) * ((a.S + 31) / 32);
  // Which form of the dK / dV passes: blocks of 128 keys, and the longest chain of 32-query tiles (heads of the group times
  // sequence).  Whole backward, us, four-wave blocks / four sets, 32 / 8 heads: 2 x 1024 (128 blocks, chain 128) 294 / 158,
  // 4 x 512 (128, 64) 162 / 97, 4 x 1024 (256, 128) 336 / 279, 8 x 512 (256, 64) 191 / 183, 1 x 8192 (512, 1024) 2706 / 2365,
  // 8 x 1024 (512, 128) 460 / 476, 16 x 512 (512, 64) 280 / 333, 8 x 2048 (1024, 256) 1408 / 1540; 64 x 117 with 16 / 4
  // heads of 64 (256, 16) 62 / 66.
  const bool few = blocks <= 128 || (blocks <= 256 && chain >= 32) || (blocks <= 512 && chain >= 256);
  if (few) {
    e = launch_dkv<0, D, kFewKW, kFewNS>(a, s);
    return e == hipSuccess ? launch_dkv<1, D, kFewKW, kFewNS>(a, s) : e;
  }
  e = launch_dkv<0, D, 4, 1>(a, s);
  return e == hipSuccess ? launch_dkv<1, D, 4, 1>(a, s) : e;
}
}  // namespace

hipError_t launch_attn_fwd_mfma(const AttnArgs& a, hipStream_t s) { return a.dh == 64 ? launch_fwd<64>(a, s) : launch_fwd<128>(a, s); }
hipError_t launch_attn_bwd_mfma(const AttnArgs& a, hipStream_t s) { return a.dh == 64 ? launch_bwd<64>(a, s) : launch_bwd<128>(a, s); }

}  // namespace tide
