// Flash-style causal grouped-query attention for gfx950, head_dim 128 or 64, bf16 storage, fp32 softmax and
// accumulation, v_mfma_f32_32x32x16_bf16 throughout.  Four kernels: forward, dQ, and dK/dV of either head size.  The
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
// Tiles.  Forward and dQ: one block = four items of 32 queries of one head (a wave each, Q in registers) that read the same keys
// (see row_item); K/V streamed in steps of 32 keys, double buffered in LDS.  What bounds a full chip is the sum of the matrix and
// vector work of a SIMD's two or three waves (16 x 2048, 32 / 8 heads: the forward's matrix pipes are busy 53 % of the cycles, at 1.8 GHz under the power limit), so registers are
// kept for three waves in the forward: with steps of 64 keys and two waves, whose MFMAs and exponentials were interleaved by hand, it took 727 us, so 620.
// dK/dV: the keys of a block stay in registers, Q/dO are streamed in tiles of 32 queries for each of the G query heads of the group, so
// dK/dV are summed over the group in registers: no atomics, deterministic.  At head size 64 (199 registers) a wave makes both.  At head size 128
// that takes 350 registers, so two waves share 32 keys, one for S, P and dV, one for dP, dS and dK, and P goes through LDS (168 registers, three
// waves per SIMD); the two passes that this replaces, one per gradient, made S and its exponentials twice.
// Where blocks are few, sets of waves share the keys (forward, dQ) or the query tiles (dK / dV): see launch_fwd_form, launch_bwd.
// Every streamed tile reaches LDS by LDS-DMA loads (no staging registers); operand fragments are read from LDS
// through small register rings, a few MFMAs ahead of their use.
// Causality: tiles entirely above the diagonal are never loaded; heavy blocks are scheduled first (see WorkMap); the
// per-element causal test is made only by the (wave-uniformly chosen) tiles that touch the diagonal.
#include <algorithm>
#include <cfloat>
#include <numeric>
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
// a barrier between reads of LDS and what other waves' loads write there next: every operand read has returned (its MFMA has been
// issued), and loads in flight stay in flight (__syncthreads() would wait for them)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
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

// Head size 64 halves the operand and accumulator registers and the LDS tiles: 111 registers in the forward and 154 in the dQ
// kernel, i.e. 4 and 3 blocks per CU.  Against the one-wave-per-row kernels (attention_simple.hip) that
// served this head size: 6 x 777, 16 / 4 heads, forward + backward 17.55 -> 0.097 ms.
constexpr int blocks_per_cu(int D, int at64, int at128) { return D == 64 ? at64 : at128; }
// Waves that a SIMD has to hold at least, and depth of the operand rings, in the forward and dQ kernels (NS: sets of waves per block).
constexpr int row_waves(int D, int NS) { return blocks_per_cu(D, 4, NS == 1 ? 3 : 2); }
constexpr int dq_waves(int D, int NS) { return NS == 1 ? blocks_per_cu(D, 3, 2) : 2; }
constexpr int kRowRing = 4;
constexpr int dq_ring(int D) { return D == 64 ? 8 : 4; }
// Work item (x, y, z) of an nx * ny * nz problem from the block's place in the 1-D dispatch order.
// Work-groups go to the 8 XCDs round-robin and every XCD has its own L2.  The nx blocks of a group (y, z: a kv head of a sequence)
// stream the same K/V resp. Q/dO rows, so a whole group is given to one XCD; groups that are few and no multiple of 8 are left to the
// plain order.  x counts from the heaviest block of a group down.  An XCD takes its groups in chunks, and of a chunk all
// heaviest blocks first, so that what ends last is light blocks of many groups: group after group, the last groups'
// heaviest blocks began when the others had nothing left to do.  us, a group / a chunk at a time: backward of 16 x 2048, 32 / 8 heads of 128 2430 / 2180, of 16 x 1024
// 725 / 634, of 7 x 979, 32 heads of 64 277 / 183; forward of 13 x 759, 16 / 4 heads of 128 60 / 48.
// Sequences of a packed batch differ, and some may be empty.  There a group is given to one XCD only where the heads of ONE sequence keep all eight busy (their number is a
// multiple of 8).  Otherwise all go in the plain order, with the groups counted up to a number that has as many factors of 2 as the heads have: block x of
// group g is on XCD (x times that number + g) % 8, so that a group comes to no more XCDs than it takes for a sequence's heads to reach all.
// (Dealt like a fixed batch, forward of one sequence of 5693 positions and 16 empty ones, 10 / 2 heads of 64, 416 us on two XCDs, so 117; backward 1037 / 449.)
struct Work3 { int x, y, z; bool on; };
struct WorkMap { int nx, ny, groups, per_xcd, chunk, stride; };   // per_xcd 0: groups are not dealt to XCDs; stride: the groups that the plain order counts
inline WorkMap work_map(int nx, int ny, int nz, bool packed) {
  const int groups = ny * nz;
  const bool dealt = packed ? ny % 8 == 0 : groups % 8 == 0 || groups >= 32;
  int stride = groups;
  if (packed && !dealt)
    while (std::gcd(stride, 8) != std::gcd(ny, 8)) ++stride;
  return WorkMap{nx, ny, groups, dealt ? (groups + 7) / 8 : 0, 1, stride};
}
inline int64_t work_blocks(const WorkMap& w) { return (int64_t)w.nx * (w.per_xcd ? 8 * w.per_xcd : w.stride); }
__device__ __forceinline__ Work3 work_item(const WorkMap& w) {
  const int n = blockIdx.x;
  int x, grp;
  if (w.per_xcd) {
    const int slot = n >> 3, first = slot / (w.chunk * w.nx) * w.chunk, in = slot - first * w.nx, size = min(w.chunk, w.per_xcd - first);
    x = in / size;
    grp = (first + in - x * size) * 8 + (n & 7);
  } else {
    x = n / w.stride;
    grp = n - x * w.stride;
  }
  const int z = grp / w.ny;
  return Work3{x, grp - z * w.ny, z, grp < w.groups};
}

}  // namespace

// The rows that a wave of the forward and dQ kernels owns: 32 queries of one head.  The query heads of a kv head read the same
// keys, so its items are counted block of 32 queries by block, the heads of the group fastest, and a block's KW waves take KW
// consecutive ones, from the end of the sequence down: with four heads per group all four waves stop at the same key (with 128
// queries of one head per block, two of them sat out the last tile).
struct RowItem { int h, qw; bool on; int kv_end; };   // head, first query, whether there is one; end of the keys that the block's waves see
template <int KW>
__device__ __forceinline__ RowItem row_item(int x, int wave_s, int kh, int G, int S) {
  const int first = (S + 31) / 32 * G - 1 - x * KW, i = first - wave_s, qb = i / G;
  return RowItem{kh * G + (i - qb * G), i >= 0 ? qb * 32 : -32, i >= 0, min(S, first / G * 32 + 32)};
}
template <int KW>
__host__ __device__ constexpr int row_blocks(int S, int G) { return ((S + 31) / 32 * G + KW - 1) / KW; }
// The keys and values that a step of the forward and dQ kernels takes: 32 of each, side by side in LDS (rows 0 .. 31 the keys, 32 .. 63
// the values), i.e. one 64-row tile of 17 (9) whole chunks, double buffered.  (Three stages, with the loads two steps ahead: no gain with a
// full chip, 1 x 526 positions of head size 64 13.4 -> 14.6 us.)
template <int D, int KW>
struct KvDma {
  static constexpr int STAGE = 64 * pitch(D);   // elements
  TileDma<64, D, KW> dma;
  __device__ __forceinline__ void init(int ld, int v_off, int wave, int lane) {   // v_off: bytes from a row's key to its value
    using Dma = TileDma<64, D, KW>;
#pragma unroll
    for (int i = 0; i < Dma::PER_WAVE; ++i) {
      const int o = (wave + KW * i) * 1024 + lane * 16, R = o / (pitch(D) * 2), piece = o % (pitch(D) * 2) / 16;
      dma.voff[i] = piece < D / 8 && o < Dma::BYTES ? (uint32_t)(perm(R & 31) * ld + piece * 8) * 2u + (R >= 32 ? (uint32_t)v_off : 0u) : 0x80000000u;
    }
  }
};

// a wave's own 32 staged rows (stage_out) to global memory, rows past the sequence left out
template <int D>
__device__ __forceinline__ void copy_rows(const bf16_t* tile, bf16_t* dst, int64_t row0, int rows, int ld, int col0, int wave, int lane) {
  asm volatile("" ::: "memory");   // behind the wave's narrower writes of the rows (LDS operations of a wave stay in order)
#pragma unroll
  for (int i = 0; i < 32 * (D / 8) / 64; ++i) {
    const int p = lane + 64 * i, row = p / (D / 8), piece = p % (D / 8);
    if (row < rows)
      *reinterpret_cast<i32x4_t*>(dst + (size_t)(row0 + row) * ld + col0 + piece * 8) =
          *reinterpret_cast<const i32x4_t*>(tile + (wave * 32 + row) * pitch(D) + piece * 8);
  }
}

// The sums of the sets of a block: sets n .. 2n - 1 hand theirs to sets 0 .. n - 1, for n = NS / 2, NS / 4, ..., and set 0 has the whole.  In
// a fixed order; every LDS stage is free by then.
template <int KW, int NS, int N>
__device__ __forceinline__ void merge_sets(bf16_t* smem, f32x16_t (&acc)[N], int set, int wave, int lane) {
  float* sums = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int n = NS / 2; n >= 1; n /= 2) {
    float* mine = sums + ((set % n) * KW + wave) * N * 16 * 64 + lane;
    if (set >= n && set < 2 * n) {
#pragma unroll
      for (int ct = 0; ct < N; ++ct)
#pragma unroll
        for (int q = 0; q < 16; ++q) mine[(ct * 16 + q) * 64] = acc[ct][q];
    }
    __syncthreads();
    if (set < n) {
#pragma unroll
      for (int ct = 0; ct < N; ++ct)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[ct][q] += mine[(ct * 16 + q) * 64];
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------------
// forward
// ------------------------------------------------------------------------------------------------
template <int D, int KW, int NS>
__global__ __launch_bounds__(KW * NS * 64, row_waves(D, NS)) void attn_fwd_mfma_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out,
                                                            float* __restrict__ lse, int Smax, int nh, int nkv,
                                                            const int* __restrict__ cu, int64_t T, WorkMap map) {
  constexpr int NK = D / 16, NC = D / 32, BK = 32;   // k16 steps of a score product, 32-column tiles of a result, keys per step
  using Kv = KvDma<D, KW>;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), set = NS > 1 ? wave_all / KW : 0, wave_s = wave_all - set * KW;
  const int lane = threadIdx.x & 63, wave = wave_s;
  bf16_t* stages = smem + set * 2 * Kv::STAGE;
  const int lr = lane & 31, g = lane >> 5, plr = perm(lr);
  const int G = nh / nkv;
  const Work3 wk = work_item(map);
  if (!wk.on) return;
  const int kh = wk.y, b = wk.z;
  const SeqView sv = seq_view(cu, b, Smax, T);
  const int S = sv.len;
  const int ld = (nh + 2 * nkv) * D;
  if (wk.x >= row_blocks<KW>(S, G)) return;   // the whole block, before any barrier: this sequence is shorter
  const RowItem item = row_item<KW>(wk.x, wave_s, kh, G, S);
  const int h = item.h, qw = item.qw, iq = qw + lr;
  const bool valid = item.on && iq < S;
  const bf16_t* base = qkv + (size_t)sv.row0 * ld;
  const __amdgpu_buffer_rsrc_t rs = rsrc(base, (uint32_t)((size_t)S * ld * 2));
  const int kcol = (nh + kh) * D, vcol = (nh + nkv + kh) * D;
  const float c = kLog2e / sqrtf((float)D);

  const int nt = (item.kv_end + BK - 1) / BK, nr = (nt + NS - 1) / NS;   // tiles, and rounds of them: set s takes tiles s, s + NS, ...
  const uint32_t seq_bytes = (uint32_t)((size_t)S * ld * 2);
  Kv kv;
  kv.init(ld, (vcol - kcol) * 2, wave, lane);
  auto fetch = [&](int t) {   // the set's t-th tile
    const int tile = set + NS * t;
    if (tile < nt) kv.dma.issue(base, seq_bytes, stages + (t & 1) * Kv::STAGE, ((uint32_t)(tile * BK) * (uint32_t)ld + (uint32_t)kcol) * 2u, wave_s);
  };
  fetch(0);

  u32x4_t qf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)   // (a row past the sequence is beyond the buffer: zeros)
    qf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)(item.on ? iq : S) * (uint32_t)ld + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));

  f32x16_t o[NC];
#pragma unroll
  for (int ct = 0; ct < NC; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) o[ct][q] = 0.f;
  // The reference begins below every score that is a number: where all keys of the first steps score -inf (a product of finite inputs can
  // overflow to it), or a set's first step shows a query no key at all, the scores are then relative to that and weigh nothing.  (From -inf it was -inf less
  // -inf, a NaN that stayed in the row.)
  float m = -FLT_MAX, l = 0.f;   // l: this lane's share of the row's sum (its partner, lane ^ 32, has the rest)

  // The sums are kept relative to m, which follows the running maximum of the row.  At head size 64 it may fall behind by 2^8: the
  // accumulators are then rescaled once or twice per row, not in nearly every tile (one of 32 rows nearly always finds a new
  // maximum; 6 x 777 30.4 -> 29.0 us).  At head size 128, where a probability is one bf16 value, that of the largest score has to
  // stay the exact 1 it is relative to the maximum itself: with a lag the results were 2 % (flat scores) to 17 % (peaked ones) further from
  // 64 bits (and 16 x 2048 took 700 us, 745 without).
  auto follow = [&](float tm) {
    const bool moved = (tm - m) * c > lag(D);
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
  // vmcnt(0): nothing of the prologue is in flight inside the loop.  The Q (and dO) fragments are first used there, so
  // the compiler issues their loads last and, at the loop's head, still counts them as outstanding; inside the loop
  // the next tiles' loads are then younger than they are, and the waits it puts in front of the first MFMAs
  // make every tile wait for the tile after it to arrive from memory.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  lds_barrier();
  constexpr int NP = parts(D), NV = 2 * NC, RK = kRowRing, RV = 4;
  for (int t = 0; t < nr; ++t) {
    const int j0 = (set + NS * t) * BK;
    fetch(t + 1);   // into the stage whose last readers passed the barrier at the end of the step before
    if (j0 <= qw + 31) {  // wave-uniform: the tile has at least one unmasked key for this wave
      const bf16_t *K = stages + (t & 1) * Kv::STAGE, *V = K + 32 * pitch(D);
      auto k_frag = [&](int i) { return frag<D>(K, 0, plr, i * 16 + g * 8); };
      auto v_frag = [&](int i) { return frag_tr<D>(V, (i / NC) * 16, (i % NC) * 32, lane); };   // k16 step i / NC, columns i % NC
      f32x16_t s;
#pragma unroll
      for (int q = 0; q < 16; ++q) s[q] = 0.f;
      u32x4_t kb[RK], vb[RV];
      // the K fragments through a ring: a fragment is requested RK MFMAs before its own (read, wait, MFMA one after
      // the other leaves the LDS latency, three MFMA times, exposed at every step)
#pragma unroll
      for (int i = 0; i < RK; ++i) kb[i] = k_frag(i);
      matrix_phase<D>(true);
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        s = mfma(kb[i % RK], qf[i], s);
        if (i + RK < NK) kb[i % RK] = k_frag(i + RK);
        __builtin_amdgcn_sched_barrier(0);
      }
      matrix_phase<D>(false);
#pragma unroll
      for (int i = 0; i < RV; ++i) vb[i] = v_frag(i);   // arrive beside the exponentials
      __builtin_amdgcn_sched_barrier(0);
      if (j0 + BK - 1 > qw) {  // the tile touches the diagonal of this wave
#pragma unroll
        for (int q = 0; q < 16; ++q)
          if (j0 + acc_row(q, g) > iq) s[q] = -INFINITY;
      }
      float tm[2] = {-INFINITY, -INFINITY};
#pragma unroll
      for (int q = 0; q < 16; ++q) tm[q & 1] = fmaxf(tm[q & 1], s[q]);
      follow(row_max(fmaxf(tm[0], tm[1])));
      const float mc = m * c;
      float ps[2] = {0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float p = __builtin_amdgcn_exp2f(s[q] * c - mc);
        s[q] = p;
        ps[q & 1] += p;
      }
      l += ps[0] + ps[1];
      u32x4_t pf[2][NP];
      pack_parts(s, 0, pf[0]);
      pack_parts(s, 1, pf[1]);
      matrix_phase<D>(true);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        o[i % NC] = mfma_parts(vb[i % RV], pf[i / NC], o[i % NC]);
        if (i + RV < NV) vb[i % RV] = v_frag(i + RV);
        __builtin_amdgcn_sched_barrier(0);
      }
      matrix_phase<D>(false);
    }
    TIDE_ATTN_WAIT_DMA();
    lds_barrier();
  }
  if constexpr (NS > 1) {
    // sets n .. 2n - 1 hand their maxima and sums to sets 0 .. n - 1, for n = NS / 2, NS / 4, ... (every stage is free by now)
    float* sums = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int n = NS / 2; n >= 1; n /= 2) {
      float* mine = sums + ((set % n) * KW + wave) * (NC * 16 + 2) * 64 + lane;
      if (set >= n && set < 2 * n) {
#pragma unroll
        for (int ct = 0; ct < NC; ++ct)
#pragma unroll
          for (int q = 0; q < 16; ++q) mine[(ct * 16 + q) * 64] = o[ct][q];
        mine[NC * 16 * 64] = m;
        mine[(NC * 16 + 1) * 64] = l;
      }
      __syncthreads();
      if (set < n) {
        const float mo = mine[NC * 16 * 64], lo = mine[(NC * 16 + 1) * 64], mn = fmaxf(m, mo);
        const float wa = __builtin_amdgcn_exp2f((m - mn) * c), wb = __builtin_amdgcn_exp2f((mo - mn) * c);
        m = mn;
        l = l * wa + lo * wb;
#pragma unroll
        for (int ct = 0; ct < NC; ++ct)
#pragma unroll
          for (int q = 0; q < 16; ++q) o[ct][q] = o[ct][q] * wa + mine[(ct * 16 + q) * 64] * wb;
      }
      __syncthreads();
    }
    if (set != 0) return;
  }
  l += swap_halves(l);

  const float inv = 1.0f / l;
  stage_out<D>(smem, o, inv, wave, lane);
  if constexpr (D == 64) {
    // A masked key has probability zero, but zero times a NaN or an infinity of its V row is a NaN that reaches the earlier
    // queries of its tile.  Rows that are not finite although their sum is are made again from the keys they see alone,
    // a channel per lane.  No row of finite inputs is, and 32 multiply-adds per lane and block find out.
    for (uint32_t rows = not_finite(o, l - l == 0.f && valid); rows != 0; rows &= rows - 1) {   // wave-uniform
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
  if (g == 0 && valid) lse[stat_index(cu, T, sv, b, h, nh, Smax, iq)] = m * (1.0f / sqrtf((float)D)) + logf(l);
  if (item.on) copy_rows<D>(smem, out, sv.row0 + qw, S - qw, nh * D, h * D, wave, lane);
}

// ------------------------------------------------------------------------------------------------
// backward, dQ: same streaming structure as the forward pass.  It also makes delta = rowsum(dO * O), which the dK / dV
// passes read: the dO fragments are in registers anyway, so O is all that is loaded for it (a pass of its own
// read dO again: 100 us at 16 x 2048, 32 heads, against 45 us more in this kernel).
// ------------------------------------------------------------------------------------------------
template <int D, int KW, int NS>
__global__ __launch_bounds__(KW * NS * 64, dq_waves(D, NS)) void attn_dq_mfma_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ out, const bf16_t* __restrict__ dout,
                                                           const float* __restrict__ lse, float* __restrict__ delta,
                                                           bf16_t* __restrict__ dqkv, int Smax, int nh, int nkv,
                                                           const int* __restrict__ cu, int64_t T, WorkMap map) {
  constexpr int NK = D / 16, NC = D / 32, BK = 32;   // as in the forward kernel
  using Kv = KvDma<D, KW>;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), set = NS > 1 ? wave_all / KW : 0, wave_s = wave_all - set * KW;
  const int lane = threadIdx.x & 63, wave = wave_s;
  bf16_t* stages = smem + set * 2 * Kv::STAGE;
  const int lr = lane & 31, g = lane >> 5, plr = perm(lr);
  const int G = nh / nkv;
  const Work3 wk = work_item(map);
  if (!wk.on) return;
  const int kh = wk.y, b = wk.z;
  const SeqView sv = seq_view(cu, b, Smax, T);
  const int S = sv.len;
  const int ld = (nh + 2 * nkv) * D, ldo = nh * D;
  if (wk.x >= row_blocks<KW>(S, G)) return;   // the whole block, before any barrier
  const RowItem item = row_item<KW>(wk.x, wave_s, kh, G, S);
  const int h = item.h, qw = item.qw, iq = qw + lr, row = item.on ? iq : S;
  const __amdgpu_buffer_rsrc_t rs = rsrc(qkv + (size_t)sv.row0 * ld, (uint32_t)((size_t)S * ld * 2));
  const __amdgpu_buffer_rsrc_t rso = rsrc(dout + (size_t)sv.row0 * ldo, (uint32_t)((size_t)S * ldo * 2));
  const int kcol = (nh + kh) * D, vcol = (nh + nkv + kh) * D;
  const float scale = 1.0f / sqrtf((float)D);
  const float c = kLog2e * scale;

  u32x4_t qf[NK], dof[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    qf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)row * (uint32_t)ld + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));
    dof[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rso, ((uint32_t)row * (uint32_t)ldo + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));
  }
  const bool valid = item.on && iq < S;
  const bool edge_q = qw + 32 > S;   // wave-uniform: some query row of this wave lies past the sequence
  const float lse_i = valid ? lse[stat_index(cu, T, sv, b, h, nh, Smax, iq)] * kLog2e : 0.f;
  float del_i = 0.f;   // a row past the end loads zeros
  {
    const __amdgpu_buffer_rsrc_t rsout = rsrc(out + (size_t)sv.row0 * ldo, (uint32_t)((size_t)S * ldo * 2));
    u32x4_t of[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
      of[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsout, ((uint32_t)row * (uint32_t)ldo + (uint32_t)(h * D + kk * 16 + g * 8)) * 2u, 0, 0));
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        del_i = fmaf(__uint_as_float(of[kk][w] << 16), __uint_as_float(dof[kk][w] << 16), del_i);
        del_i = fmaf(__uint_as_float(of[kk][w] & 0xFFFF0000u), __uint_as_float(dof[kk][w] & 0xFFFF0000u), del_i);
      }
    del_i += __shfl_xor(del_i, 32, 64);
    if (valid && g == 0 && set == 0) delta[stat_index(cu, T, sv, b, h, nh, Smax, iq)] = del_i;
  }

  f32x16_t dq[NC];
#pragma unroll
  for (int ct = 0; ct < NC; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) dq[ct][q] = 0.f;

  const int nt = (item.kv_end + BK - 1) / BK, nr = (nt + NS - 1) / NS;   // set s takes tiles s, s + NS, ...
  const bf16_t* seq = qkv + (size_t)sv.row0 * ld;
  const uint32_t seq_bytes = (uint32_t)((size_t)S * ld * 2);
  Kv kv;
  kv.init(ld, (vcol - kcol) * 2, wave, lane);
  auto fetch = [&](int t) {
    const int tile = set + NS * t;
    if (tile < nt) kv.dma.issue(seq, seq_bytes, stages + (t & 1) * Kv::STAGE, ((uint32_t)(tile * BK) * (uint32_t)ld + (uint32_t)kcol) * 2u, wave_s);
  };
  fetch(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): nothing of the prologue is in flight inside the loop (see the forward kernel)
  lds_barrier();

  constexpr int NP = parts(D), NX = 2 * NC, RING = dq_ring(D), RX = 4;
  for (int t = 0; t < nr; ++t) {
    const int j0 = (set + NS * t) * BK;
    fetch(t + 1);
    if (j0 <= qw + 31) {
      const bf16_t *K = stages + (t & 1) * Kv::STAGE, *V = K + 32 * pitch(D);
      const bool diag = j0 + BK - 1 > qw;
      auto x_frag = [&](int i) { return frag_tr<D>(K, (i / NC) * 16, (i % NC) * 32, lane); };   // of K^T
      u32x4_t fb[RING], xb[RX];
      f32x16_t s, dp;
#pragma unroll
      for (int q = 0; q < 16; ++q) { s[q] = 0.f; dp[q] = 0.f; }
      // K and V fragments alternately through a ring, each requested RING MFMAs ahead (see the forward kernel)
      auto fetch_frag = [&](int i) { return frag<D>((i & 1) ? V : K, 0, plr, (i >> 1) * 16 + g * 8); };
#pragma unroll
      for (int i = 0; i < RING; ++i) fb[i] = fetch_frag(i);
      matrix_phase<D>(true);
#pragma unroll
      for (int i = 0; i < 2 * NK; ++i) {
        if (i & 1) dp = mfma(fb[i % RING], dof[i >> 1], dp);
        else s = mfma(fb[i % RING], qf[i >> 1], s);
        if (i + RING < 2 * NK) fb[i % RING] = fetch_frag(i + RING);
        __builtin_amdgcn_sched_barrier(0);
      }
      matrix_phase<D>(false);
#pragma unroll
      for (int i = 0; i < RX; ++i) xb[i] = x_frag(i);   // arrive beside the exponentials
      __builtin_amdgcn_sched_barrier(0);
      if (diag || edge_q) {   // wave-uniform: only a tile on the diagonal or the last query block needs per-element tests (-4.5 %)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          float p = __builtin_amdgcn_exp2f(s[q] * c - lse_i);
          if (!valid || (diag && (j0 + acc_row(q, g) > iq))) p = 0.f;
          s[q] = p * (dp[q] - del_i);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 16; ++q) s[q] = __builtin_amdgcn_exp2f(s[q] * c - lse_i) * (dp[q] - del_i);
      }
      u32x4_t dsf[2][NP];
      pack_parts(s, 0, dsf[0]);
      pack_parts(s, 1, dsf[1]);
      matrix_phase<D>(true);
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        dq[i % NC] = mfma_parts(xb[i % RX], dsf[i / NC], dq[i % NC]);
        if (i + RX < NX) xb[i % RX] = x_frag(i + RX);
        __builtin_amdgcn_sched_barrier(0);
      }
      matrix_phase<D>(false);
    }
    TIDE_ATTN_WAIT_DMA();
    lds_barrier();
  }
  if constexpr (NS > 1) {
    merge_sets<KW, NS, NC>(smem, dq, set, wave, lane);
    if (set != 0) return;
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
  if (item.on) copy_rows<D>(smem, dqkv, sv.row0 + qw, S - qw, ld, h * D, wave, lane);
}

// ------------------------------------------------------------------------------------------------
// backward, dK and dV
// ------------------------------------------------------------------------------------------------
namespace {
template <int D> struct DkvStage {
  static constexpr int BI = 32;                              // queries per streamed tile
  static constexpr int Q_TILE = TileDma<BI, D>::CHUNKS * 512;   // elements: the tile rounded up to whole 1 KiB chunks of the LDS-DMA loads
  static constexpr int STAGE = 2 * Q_TILE + 4 * BI;          // Q tile, dO tile, then BI floats from lse and BI from delta, see sstore
};
// LDS of a set of the pair kernel, elements: two stages, then 4 KB of probabilities per pair
template <int KW> constexpr int pair_set() { return 2 * DkvStage<128>::STAGE + KW * 2048; }
}  // namespace

// Head size 64.  KW waves of 32 keys; NS sets of them, each with LDS stages of its own, take every NS-th query tile, and the sets' sums are added
// through LDS at the end, in a fixed order: with few blocks there is nobody to share a CU with, and the kernel takes as long as the longest
// chain of query tiles, G heads times the sequence.  dK and dV in two launches: 6 x 777, 34 + 41 us, in one 46.  The score products begin from - lse and
// - delta, which their rows' accumulators read from LDS (16 to 32 vector instructions fewer per 32 x 32 scores than zeros and two
// subtractions), and the walk over tiles and heads is a counter (a division by G per tile was 100 scalar instructions).
template <int KW, int NS>
__global__ __launch_bounds__(KW * NS * 64, NS > 1 ? 1 : 2) void attn_dkv_mfma_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dout,
                                                            const float* __restrict__ lse, const float* __restrict__ delta,
                                                            bf16_t* __restrict__ dqkv, int Smax, int nh, int nkv,
                                                            const int* __restrict__ cu, int64_t T, WorkMap map) {
  constexpr int D = 64;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  constexpr int KB = KW * 32, SET = KW * 64;   // keys of the block, threads of a set
  const int set = NS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / SET) : 0;
  const int tid = threadIdx.x - set * SET, lane = tid & 63, wave = tid >> 6;   // inside the set
  const int lr = lane & 31, g = lane >> 5, plr = perm(lr);
  const Work3 wk = work_item(map);
  if (!wk.on) return;
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

  constexpr int BI = DkvStage<D>::BI, NK = D / 16, NC = D / 32;
  constexpr int Q_TILE = DkvStage<D>::Q_TILE, DKV_STAGE = DkvStage<D>::STAGE;
  u32x4_t kf[NK], vf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    kf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)jk * (uint32_t)ld + (uint32_t)(kcol + kk * 16 + g * 8)) * 2u, 0, 0));
    vf[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)jk * (uint32_t)ld + (uint32_t)(vcol + kk * 16 + g * 8)) * 2u, 0, 0));
  }
  constexpr int NA = 2 * NC;
  f32x16_t dacc[NA];   // dV and dK of this wave's 32 keys
#pragma unroll
  for (int ct = 0; ct < NA; ++ct)
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
  struct Place { int hg, i0; };   // head of the group and first query of a tile
  Place at = {0, i_begin + (nit - 1) * BI};
  auto advance = [&](Place& p, int n) {   // n tiles further on
    p.hg += n;
    while (p.hg >= G) { p.hg -= G; p.i0 -= BI; }
  };
  const float to_scores = -sqrtf((float)D);
  auto gload = [&](const Place& p, int st) {   // a tile into stage st (whose last readers have passed a barrier)
    const int hh = kh * G + p.hg, i0 = p.i0;
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
  // What the score products begin from, in place of zeros: - lse sqrt(D), so that S comes out as (q k / sqrt(D) - lse) sqrt(D) and the
  // probability is exp2 of it times one constant, and - delta.
  auto sstore = [&](int st) {
    bf16_t* base = stages + st * DKV_STAGE;
    if (tid < 2 * BI) reinterpret_cast<float*>(base + 2 * Q_TILE)[tid] = stat * ((tid < BI) ? to_scores : -1.f);
  };

  if (NS == 1 || set < ntiles) {   // (one set: there is always a tile)
    advance(at, set);
    gload(at, 0);
    sstore(0);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the tile and the K / V fragments have arrived before the loop
  __syncthreads();
  // (the sets' trip counts differ by one at most: every set passes every barrier)
  for (int r = 0; r * NS < ntiles; ++r) {
    const int st = r & 1, u = r * NS + set;
    const int i0 = NS == 1 || u < ntiles ? at.i0 : S;   // past the end: not entered
    if (u + NS < ntiles) {
      advance(at, NS);
      gload(at, st ^ 1);
    }
    if (i0 + 31 >= jw && i0 < S) {  // wave-uniform: some query of the tile sees some key of this wave
      const bf16_t* Qt = stages + st * DKV_STAGE;
      const bf16_t* dOt = Qt + Q_TILE;
      const float* stats = reinterpret_cast<const float*>(Qt + 2 * Q_TILE);
      f32x16_t s, dp;
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {   // row 8 qq + 4 g + e is register 4 qq + e
        const float4 l4 = *reinterpret_cast<const float4*>(stats + 8 * qq + 4 * g), d4 = *reinterpret_cast<const float4*>(stats + BI + 8 * qq + 4 * g);
        s[4 * qq] = l4.x; s[4 * qq + 1] = l4.y; s[4 * qq + 2] = l4.z; s[4 * qq + 3] = l4.w;
        dp[4 * qq] = d4.x; dp[4 * qq + 1] = d4.y; dp[4 * qq + 2] = d4.z; dp[4 * qq + 3] = d4.w;
      }
      {
        // Q and dO fragments alternately through a ring, each requested RING MFMAs ahead (depths of 2 to 6 measure the same)
        constexpr int RING = 4, NF = 2 * NK;
        u32x4_t fb[RING];
        auto fetch = [&](int i) { return frag<D>((i & 1) ? dOt : Qt, 0, plr, (i >> 1) * 16 + g * 8); };
#pragma unroll
        for (int i = 0; i < RING; ++i) fb[i] = fetch(i);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          if (i & 1) dp = mfma(fb[i % RING], vf[i >> 1], dp);
          else s = mfma(fb[i % RING], kf[i >> 1], s);
          if (i + RING < NF) fb[i % RING] = fetch(i + RING);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // Rows past the end of the sequence carry lse = +inf (see sstore), i.e. p = 0 without a test; the causal test is
      // per element, and only a tile that touches the diagonal makes it (wave-uniform branch).
      auto probs = [&](auto MASK) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          float p = __builtin_amdgcn_exp2f(s[q] * c);
          if constexpr (decltype(MASK)::value) {
            if (i0 + acc_row(q, g) < jk) p = 0.f;
          }
          s[q] = p;            // P for dV
          dp[q] = p * dp[q];   // dS for dK
        }
      };
      if (i0 < jw + 32) probs(std::true_type{});   // some (query, key) pair of the tile is above the diagonal
      else probs(std::false_type{});
      // dV += P^T dO, dK += dS^T Q
      auto product = [&](const f32x16_t& x, const bf16_t* Xt, int c0) {
        u32x4_t pf[2][parts(D)];
        pack_parts(x, 0, pf[0]);
        pack_parts(x, 1, pf[1]);
#pragma unroll
        for (int ct = 0; ct < NC; ++ct)
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) dacc[c0 + ct] = mfma_parts(frag_tr<D>(Xt, ks * 16, ct * 32, lane), pf[ks], dacc[c0 + ct]);
      };
      product(s, dOt, 0);
      product(dp, Qt, NC);
    }
    if (u + NS < ntiles) sstore(st ^ 1);
    TIDE_ATTN_WAIT_DMA();
    __syncthreads();
  }
  if constexpr (NS > 1) {
    merge_sets<KW, NS, NA>(smem, dacc, set, wave, lane);
    if (set != 0) return;
  }
  // one result after the other through the wave's own 32 rows of LDS
  auto store = [&](auto C0, auto ISK) {
    constexpr int c0 = decltype(C0)::value;
    constexpr bool is_k = decltype(ISK)::value;
    f32x16_t (&acc)[NC] = *reinterpret_cast<f32x16_t (*)[NC]>(&dacc[c0]);
    stage_out<D>(smem, acc, is_k ? scale : 1.0f, wave, lane);
    {
      // As in the forward kernel, from the other side: the queries jw .. j - 1 meet key j with weight zero.  Keys after the
      // first of them that is not finite are made again from the queries that see them alone (a later query takes every
      // key before it with it, rightly).
      uint32_t rows = not_finite(acc, jk < S);
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
        float sum = 0.f;
        for (int hh = kh * G; hh < (kh + 1) * G && __builtin_amdgcn_ballot_w64(sum - sum == 0.f) != 0; ++hh)
#pragma unroll 1
          for (int i = j; i < S; ++i) {
            const float qv = bf2f(base[(size_t)i * ld + hh * D + lane]), dov = bf2f(dob[(size_t)i * ldo + hh * D + lane]);
            const size_t at = stat_index(cu, T, sv, b, hh, nh, Smax, i);
            const float p = __builtin_amdgcn_exp2f(wave_sum(qv * kv) * c - lse[at] * kLog2e);
            sum += is_k ? p * (wave_sum(dov * vv) - delta[at]) * qv : p * dov;
            if (__builtin_amdgcn_ballot_w64(sum - sum == 0.f) == 0) break;
          }
        asm volatile("" ::: "memory");   // after the wave's own wider stores of the row
        smem[(wave * 32 + r) * pitch(D) + lane] = f2bf(is_k ? sum * scale : sum);
      }
    }
    copy_rows<D>(smem, dqkv, sv.row0 + jw, S - jw, ld, is_k ? kcol : vcol, wave, lane);
    asm volatile("" ::: "memory");
  };
  store(std::integral_constant<int, 0>{}, std::false_type{});
  store(std::integral_constant<int, NC>{}, std::true_type{});
}


// Head size 128.  Two waves share 32 keys: the value wave makes S = Q K^T, the probabilities and dV += P^T dO, the key wave dP = dO V^T, dS = P (dP - delta)
// and dK += dS^T Q.  P goes from one to the other through LDS in fp32, 16 registers per lane in the layout that both products have.  KW pairs
// and NS sets as above.  Against a launch per gradient (16 and 24 MFMAs per 32 x 32 scores, S and its exponentials in both), forward and
// backward, us: 16 x 2048, 32 / 8 heads 2818 -> 2573; 5 x 1601, 40 / 8 832 -> 663; 42 x 190, 16 / 8 113 -> 92; 1 x 500, 32 / 8 88 -> 65; eighteen shapes 1.22 times as fast in the mean.
// What bounds it at 16 x 2048 (matrix pipes 54 % busy, L2 hits 47 %, at 1.9 GHz): 2561 us are 2246 without its tile loads, 2522 without the exponentials, 2483
// without the exchange of P.  128 keys per block (8 waves, one block per CU) halve the loads, but nobody is there at its two barriers: 2674 for 2582.
template <int KW, int NS>
__global__ __launch_bounds__(KW * NS * 128, NS == 1 ? 3 : 2) void attn_dkv_pair_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dout,
                                                            const float* __restrict__ lse, const float* __restrict__ delta,
                                                            bf16_t* __restrict__ dqkv, int Smax, int nh, int nkv,
                                                            const int* __restrict__ cu, int64_t T, WorkMap map) {
  constexpr int D = 128, BI = DkvStage<D>::BI, NW = 2 * KW, NK = D / 16, NC = D / 32;   // NW: waves of a set
  constexpr int TILE = DkvStage<D>::Q_TILE, STAGE = DkvStage<D>::STAGE;
  static_assert(KW == 1 || KW == 2, "one or two key waves share the loads");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), set = NS > 1 ? wave_all / NW : 0, wave_s = wave_all - set * NW;
  const int lane = threadIdx.x & 63, lr = lane & 31, g = lane >> 5, plr = perm(lr);
  const bool is_k = wave_s >= KW;   // which wave of its pair
  const int pair = is_k ? wave_s - KW : wave_s;
  const Work3 wk = work_item(map);
  if (!wk.on) return;
  const int kh = wk.y, b = wk.z, j0 = wk.x * KW * 32, jw = j0 + pair * 32, jk = jw + lr;   // early key blocks are the heavy ones
  const SeqView sv = seq_view(cu, b, Smax, T);
  const int S = sv.len, G = nh / nkv;
  const int ld = (nh + 2 * nkv) * D, ldo = nh * D;
  if (j0 >= S) return;   // the whole block, before any barrier
  const bf16_t *seq = qkv + (size_t)sv.row0 * ld, *seq_do = dout + (size_t)sv.row0 * ldo;
  const uint32_t seq_bytes = (uint32_t)((size_t)S * ld * 2), seq_do_bytes = (uint32_t)((size_t)S * ldo * 2);
  const __amdgpu_buffer_rsrc_t rs = rsrc(seq, seq_bytes);
  const int col = (is_k ? nh + nkv + kh : nh + kh) * D;   // of what the wave holds: the key wave V, the value wave K
  const float scale = 1.0f / sqrtf((float)D);
  const float c = kLog2e * scale;

  u32x4_t f[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)
    f[kk] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, ((uint32_t)jk * (uint32_t)ld + (uint32_t)(col + kk * 16 + g * 8)) * 2u, 0, 0));
  f32x16_t dacc[NC];   // dV or dK of the pair's 32 keys
#pragma unroll
  for (int ct = 0; ct < NC; ++ct)
#pragma unroll
    for (int q = 0; q < 16; ++q) dacc[ct][q] = 0.f;

  // tiles from the end of the sequence down, over the G heads, as at head size 64
  const int nit = (S - j0 + BI - 1) / BI, ntiles = G * nit;   // (j0 is a multiple of BI)
  bf16_t* stages = smem + set * pair_set<KW>();
  float4* probs = reinterpret_cast<float4*>(stages + 2 * STAGE) + pair * 256 + lane;
  struct Place { int hg, i0; };
  Place at = {0, j0 + (nit - 1) * BI};
  auto advance = [&](int n) {
    at.hg += n;
    while (at.hg >= G) { at.hg -= G; at.i0 -= BI; }
  };
  // The key waves load: they have nothing to do while the value waves make the probabilities.  Of two, the first the Q tile, the second the dO tile.
  const bool load_q = KW == 1 || pair == 0, load_do = KW == 1 || pair == 1;
  TileDma<BI, D, 1> dma[3 - KW];
  if constexpr (KW == 1) {
    dma[0].init(ld, 0, lane);
    dma[1].init(ldo, 0, lane);
  } else {
    dma[0].init(load_q ? ld : ldo, 0, lane);
  }
  const float to_scores = -sqrtf((float)D);
  float stat = 0.f;   // of the key wave that loads Q: lanes below BI carry lse, the others delta
  auto gload = [&](int st) {   // the tile at `at` into stage st, whose last readers have passed a barrier
    if (!is_k) return;
    const int hh = kh * G + at.hg;
    bf16_t* base = stages + st * STAGE;
    if (load_q) {
      dma[0].issue(seq, seq_bytes, base, ((uint32_t)at.i0 * (uint32_t)ld + (uint32_t)(hh * D)) * 2u, 0);
      const int i = at.i0 + (lane & (BI - 1));
      const float* src = lane < BI ? lse : delta;   // (used in sstore only; a row past the sequence gets lse = +inf, delta = 0)
      stat = i < S ? src[stat_index(cu, T, sv, b, hh, nh, Smax, i)] : lane < BI ? INFINITY : 0.f;
    }
    if (load_do) dma[2 - KW].issue(seq_do, seq_do_bytes, base + TILE, ((uint32_t)at.i0 * (uint32_t)ldo + (uint32_t)(hh * D)) * 2u, 0);
  };
  auto sstore = [&](int st) {   // what the score products begin from, as at head size 64
    if (is_k && load_q) reinterpret_cast<float*>(stages + st * STAGE + 2 * TILE)[lane] = stat * (lane < BI ? to_scores : -1.f);
  };
  if (NS == 1 || set < ntiles) {   // (one set: there is always a tile)
    advance(set);
    gload(0);
    sstore(0);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the tile and the fragments have arrived before the loop
  __syncthreads();
  constexpr int RING = 4, NX = 2 * NC;
  // (the sets' trip counts differ by one at most: every wave passes every barrier)
  for (int r = 0; r * NS < ntiles; ++r) {
    const int st = r & 1, u = r * NS + set;
    const int i0 = NS == 1 || u < ntiles ? at.i0 : S;
    const bool live = i0 + 31 >= jw && i0 < S;   // wave-uniform, the same for both waves of a pair: some query of the tile sees some key of theirs
    const bf16_t *Qt = stages + st * STAGE, *dOt = Qt + TILE;
    const bf16_t *Xt = is_k ? dOt : Qt, *Yt = is_k ? Qt : dOt;   // rows of the first product, columns of the second
    f32x16_t s;
    u32x4_t xb[RING];
    auto y_frag = [&](int i) { return frag_tr<D>(Yt, (i / NC) * 16, (i % NC) * 32, lane); };   // k16 step i / NC, columns i % NC
    if (live) {
      const float* stats = reinterpret_cast<const float*>(Qt + 2 * TILE) + (is_k ? BI : 0);
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {   // row 8 qq + 4 g + e is register 4 qq + e
        const float4 l4 = *reinterpret_cast<const float4*>(stats + 8 * qq + 4 * g);
        s[4 * qq] = l4.x; s[4 * qq + 1] = l4.y; s[4 * qq + 2] = l4.z; s[4 * qq + 3] = l4.w;
      }
      u32x4_t fb[RING];
      auto x_frag = [&](int i) { return frag<D>(Xt, 0, plr, i * 16 + g * 8); };
#pragma unroll
      for (int i = 0; i < RING; ++i) fb[i] = x_frag(i);
      matrix_phase<D>(true);
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        s = mfma(fb[i % RING], f[i], s);
        if (i + RING < NK) fb[i % RING] = x_frag(i + RING);
        __builtin_amdgcn_sched_barrier(0);
      }
      matrix_phase<D>(false);
#pragma unroll
      for (int i = 0; i < RING; ++i) xb[i] = y_frag(i);   // arrive beside the exponentials
      __builtin_amdgcn_sched_barrier(0);
      if (!is_k) {
        if (i0 < jw + 32) {   // some (query, key) pair of the tile is above the diagonal
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            const float p = __builtin_amdgcn_exp2f(s[q] * c);
            s[q] = i0 + acc_row(q, g) < jk ? 0.f : p;
          }
        } else {
#pragma unroll
          for (int q = 0; q < 16; ++q) s[q] = __builtin_amdgcn_exp2f(s[q] * c);
        }
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) probs[64 * qq] = make_float4(s[4 * qq], s[4 * qq + 1], s[4 * qq + 2], s[4 * qq + 3]);
      }
    }
    if (u + NS < ntiles) {
      advance(NS);
      gload(st ^ 1);
    }
    lds_barrier();   // P is there
    if (live) {
      if (is_k) {
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          const float4 p4 = probs[64 * qq];
          s[4 * qq] *= p4.x; s[4 * qq + 1] *= p4.y; s[4 * qq + 2] *= p4.z; s[4 * qq + 3] *= p4.w;
        }
      }
      u32x4_t pf[2][parts(D)];
      pack_parts(s, 0, pf[0]);
      pack_parts(s, 1, pf[1]);
      matrix_phase<D>(true);
#pragma unroll
      for (int i = 0; i < NX; ++i) {
        dacc[i % NC] = mfma_parts(xb[i % RING], pf[i / NC], dacc[i % NC]);
        if (i + RING < NX) xb[i % RING] = y_frag(i + RING);
        __builtin_amdgcn_sched_barrier(0);
      }
      matrix_phase<D>(false);
    }
    if (u + NS < ntiles) sstore(st ^ 1);
    TIDE_ATTN_WAIT_DMA();
    __syncthreads();   // the stage and the probabilities are read, the next tile is there
  }
  if constexpr (NS > 1) {
    merge_sets<NW, NS, NC>(smem, dacc, set, wave_s, lane);
    if (set != 0) return;
  }
  stage_out<D>(smem, dacc, is_k ? scale : 1.0f, wave_s, lane);
  copy_rows<D>(smem, dqkv, sv.row0 + jw, S - jw, ld, (is_k ? nh + kh : nh + nkv + kh) * D, wave_s, lane);
}

// ------------------------------------------------------------------------------------------------
bool attn_mfma_supported(const AttnArgs& a) {
  if (a.dtype != kBF16 || (a.dh != 128 && a.dh != 64)) return false;
  if (a.B <= 0 || a.S <= 0 || a.B > 65535 || a.nh > 65535) return false;
  const int64_t ld = (int64_t)(a.nh + 2 * a.nkv) * a.dh;
  if ((int64_t)a.S * ld * 2 >= ((int64_t)1 << 31)) return false;   // 32-bit offsets inside one sequence
  if (((uintptr_t)a.qkv | (uintptr_t)a.out | (uintptr_t)a.dout | (uintptr_t)a.dqkv) & 15) return false;
  if ((int64_t)((a.S + 127) / 128) * a.nh * a.B >= ((int64_t)1 << 31)) return false;   // 1-D grids
  return true;
}

namespace {
template <int D, int KW, int NS>
constexpr size_t row_smem() {   // of the forward and dQ kernels
  const size_t st = (size_t)NS * 2 * KvDma<D, KW>::STAGE * sizeof(bf16_t), out = (size_t)KW * 32 * pitch(D) * sizeof(bf16_t);
  const size_t sums = NS > 1 ? (size_t)(NS / 2) * KW * (D / 32 * 16 + 2) * 64 * sizeof(float) : 0;
  return std::max({st, out, sums});
}
// of the dK / dV kernels: waves of a set, a set's LDS, and the accumulators that sets merge
template <int D>
constexpr size_t dkv_smem(int waves, int NS, int set_elems, int accumulators) {
  const size_t st = (size_t)NS * set_elems * sizeof(bf16_t), out = (size_t)waves * 32 * pitch(D) * sizeof(bf16_t);
  return std::max({st, out, (size_t)(NS / 2) * waves * accumulators * 16 * 64 * sizeof(float)});
}

hipError_t set_smem(const void* f, size_t bytes, bool& done) {
  if (done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) done = true;
  return e;
}

// Groups in a chunk (see WorkMap), equal chunks.  Forward and dQ: all of an XCD's where they are three rounds of blocks or fewer; of more, as many as
// have 4 MB of keys and values, the L2 of an XCD, two to eight (64 x 199, 32 / 8 heads, forward, 4 / 8 / 16 / 64 of 64 groups: 57 / 56 / 65 / 71 us; 16 x 2048, 1 / 4 / 16 of
// 16: 659 / 620 / 651).  dK / dV, which read more per block: sixteen at head size 64 (backward of
// 32 x 512, 4 / 8 / 16 / 32 of 32: 453 / 448 / 425 / 433); at 128 all where they are three rounds of blocks or fewer, otherwise eight (forward and backward of 16 x 2048,
// 2 / 4 / 8 / 16 of 16: 2581 / 2529 / 2522 / 2582; of 11 x 815, 16 / 8 heads, 4 / 6 / 11 of 11: 206 / 194 / 191).  (Rounds of 32 CUs times the three
// blocks that one holds of the form with one set; the forms with two sets are for fewer blocks than that in any case.)
int row_chunk(int per_xcd, int nx, int slots, int64_t kv_bytes) {
  if (per_xcd * (int64_t)nx <= 3 * slots) return std::max(1, per_xcd);
  const int most = (int)std::min<int64_t>(8, std::max<int64_t>(2, (4 << 20) / kv_bytes)), n = (per_xcd + most - 1) / most;
  return (per_xcd + n - 1) / n;
}
int key_chunk(int per_xcd, int nx, int D) {
  const int most = D == 64 ? 16 : per_xcd * (int64_t)nx <= 3 * 32 * 3 ? std::max(1, per_xcd) : 8;
  const int n = std::max(1, (per_xcd + most - 1) / most);
  return std::max(1, (per_xcd + n - 1) / n);
}
// Of a packed batch chunks of an odd number of groups: behind a sequence's last block its turns go to blocks that end at once, and an XCD's
// four shader engines take the blocks in turn as well: 880 and 5707 positions, 64 / 8 heads of 64, chunks of two / three, forward 604 / 424 us, backward
// 2163 / 1408 (dK / dV in two sets there, too).
void set_chunk(WorkMap& map, int chunk, const AttnArgs& a) {
  map.chunk = chunk;
  if (!a.cu_seqlens || !map.per_xcd) return;
  map.chunk |= 1;
  map.per_xcd = (map.per_xcd + map.chunk - 1) / map.chunk * map.chunk;
}
template <int D, int KW, int NS>
WorkMap row_map(const AttnArgs& a, int waves) {
  WorkMap map = work_map(row_blocks<KW>(a.S, a.nh / a.nkv), a.nkv, a.B, a.cu_seqlens != nullptr);
  set_chunk(map, row_chunk(map.per_xcd, map.nx, 32 * 4 * waves / (KW * NS), (int64_t)a.S * D * 4), a);
  return map;
}
template <int KW, int D>
WorkMap key_map(const AttnArgs& a) {
  WorkMap map = work_map((a.S + KW * 32 - 1) / (KW * 32), a.nkv, a.B, a.cu_seqlens != nullptr);
  set_chunk(map, key_chunk(map.per_xcd, map.nx, D), a);
  return map;
}
// A launch has fewer than 2^32 threads, and in a packed batch the number of sequences and the longest length are bounds that can ask for more blocks
// than that, nearly all of them without rows: such a batch is launched as two.  (A fixed batch of so many blocks does not fit the memory.)
bool splits_batch(const AttnArgs& a, const WorkMap& map, int threads) {
  return a.cu_seqlens && a.B > 1 && work_blocks(map) * threads > (int64_t)UINT32_MAX;
}
template <typename Launch>
hipError_t launch_halves(const AttnArgs& a, const Launch& launch) {
  AttnArgs half = a;
  half.B = a.B / 2;
  const hipError_t e = launch(half);
  if (e != hipSuccess) return e;
  half.cu_seqlens = a.cu_seqlens + half.B;
  half.B = a.B - half.B;
  return launch(half);
}
template <int D, int KW, int NS>
hipError_t launch_fwd(const AttnArgs& a, hipStream_t s) {
  constexpr size_t smem = row_smem<D, KW, NS>();
  static_assert(smem <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  const hipError_t e = set_smem((const void*)attn_fwd_mfma_kernel<D, KW, NS>, smem, done);
  if (e != hipSuccess) return e;
  const WorkMap map = row_map<D, KW, NS>(a, row_waves(D, NS));
  if (splits_batch(a, map, KW * NS * 64)) return launch_halves(a, [&](const AttnArgs& half) { return launch_fwd<D, KW, NS>(half, s); });
  const dim3 grid((unsigned)work_blocks(map));   // 1-D: the kernel maps blocks to work itself
  ProfScope ps("attn_fwd_mfma", 2.0 * a.B * a.nh * D * (double)a.S * (a.S + 1), 0, s);
  hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, KW, NS>), grid, dim3(KW * NS * 64), smem, s, (const bf16_t*)a.qkv, (bf16_t*)a.out, a.lse, a.S, a.nh, a.nkv, a.cu_seqlens, a.total_rows, map);
  return hipGetLastError();
}

template <int D, int KW, int NS>
hipError_t launch_dq(const AttnArgs& a, hipStream_t s) {
  constexpr size_t smem = row_smem<D, KW, NS>();
  static_assert(smem <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  const hipError_t e = set_smem((const void*)attn_dq_mfma_kernel<D, KW, NS>, smem, done);
  if (e != hipSuccess) return e;
  const WorkMap map = row_map<D, KW, NS>(a, dq_waves(D, NS));
  if (splits_batch(a, map, KW * NS * 64)) return launch_halves(a, [&](const AttnArgs& half) { return launch_dq<D, KW, NS>(half, s); });
  const dim3 grid((unsigned)work_blocks(map));
  ProfScope ps("attn_dq_mfma", 3.0 * a.B * a.nh * D * (double)a.S * (a.S + 1), 0, s);   // S, dP and dQ products
  hipLaunchKernelGGL((attn_dq_mfma_kernel<D, KW, NS>), grid, dim3(KW * NS * 64), smem, s, (const bf16_t*)a.qkv, (const bf16_t*)a.out, (const bf16_t*)a.dout, a.lse, a.delta, (bf16_t*)a.dqkv, a.S, a.nh, a.nkv, a.cu_seqlens, a.total_rows, map);
  return hipGetLastError();
}

template <int KW, int NS>
hipError_t launch_dkv(const AttnArgs& a, hipStream_t s) {   // head size 64
  constexpr size_t smem = dkv_smem<64>(KW, NS, 2 * DkvStage<64>::STAGE, 4);
  static_assert(smem <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  const hipError_t e = set_smem((const void*)attn_dkv_mfma_kernel<KW, NS>, smem, done);
  if (e != hipSuccess) return e;
  const WorkMap map = key_map<KW, 64>(a);
  if (splits_batch(a, map, KW * NS * 64)) return launch_halves(a, [&](const AttnArgs& half) { return launch_dkv<KW, NS>(half, s); });
  const dim3 grid((unsigned)work_blocks(map));
  hipLaunchKernelGGL((attn_dkv_mfma_kernel<KW, NS>), grid, dim3(KW * NS * 64), smem, s, (const bf16_t*)a.qkv, (const bf16_t*)a.dout, a.lse, a.delta, (bf16_t*)a.dqkv, a.S, a.nh, a.nkv, a.cu_seqlens, a.total_rows, map);
  return hipGetLastError();
}
template <int KW, int NS>
hipError_t launch_dkv_pair(const AttnArgs& a, hipStream_t s) {   // head size 128
  constexpr size_t smem = dkv_smem<128>(2 * KW, NS, pair_set<KW>(), 4);
  static_assert(smem <= 160 * 1024, "LDS of a CU");
  static bool done = false;
  const hipError_t e = set_smem((const void*)attn_dkv_pair_kernel<KW, NS>, smem, done);
  if (e != hipSuccess) return e;
  const WorkMap map = key_map<KW, 128>(a);
  if (splits_batch(a, map, KW * NS * 128)) return launch_halves(a, [&](const AttnArgs& half) { return launch_dkv_pair<KW, NS>(half, s); });
  const dim3 grid((unsigned)work_blocks(map));
  hipLaunchKernelGGL((attn_dkv_pair_kernel<KW, NS>), grid, dim3(KW * NS * 128), smem, s, (const bf16_t*)a.qkv, (const bf16_t*)a.dout, a.lse, a.delta, (bf16_t*)a.dqkv, a.S, a.nh, a.nkv, a.cu_seqlens, a.total_rows, map);
  return hipGetLastError();
}

// Blocks of four items that have rows, the steps of the longest, and the blocks that are launched.  A packed batch holds at most one partly filled item of
// every head per sequence; its launch is made for sequences that are all as long as the longest.
struct RowWork { int64_t blocks; int steps; int64_t launched; };
RowWork row_work(const AttnArgs& a) {
  const int64_t per_seq = (a.S + 31) / 32, items = a.cu_seqlens ? std::min<int64_t>(a.total_rows / 32 + a.B, per_seq * a.B) : per_seq * a.B;
  return RowWork{(items * a.nh + 3) / 4, (int)per_seq, (int64_t)row_blocks<4>(a.S, a.nh / a.nkv) * a.nkv * a.B};
}
struct Form { int kw, ns; };   // waves (dK / dV at head size 128: pairs of them) and sets
// Which form of the forward and dQ kernels: four waves that walk all keys; or, where a block's steps are a longer chain than the blocks of a CU are many,
// sets of waves that share the steps.  The lines run where the two take equally long over 1200 fixed batches (1 .. 96 sequences of 16 .. 4000 positions, twelve head counts).
// A packed batch can launch many times the blocks that have rows; those end at once, but the more waves they have the longer that takes: sets only up to 4096
// (forward; 8192 where they are at most 16 times those that have rows) and 8192 (dQ) launched blocks of four items, over 750 packed batches (up to 9000 rows, up to 200 empty sequences).  us, four waves / two sets of two / two
// sets of four: forward of head size 128, 16 / 4 heads 1 x 2665 (336 blocks of 84 steps) 65.9 / 47.5 / 51.8, 16 / 8 heads 5 x 1021 (640, 32) 35.6 / 42.5 / 42.5, 32 / 8 heads 7 x 98 (224, 4)
// 7.4 / 8.7 / 8.8, 6 / 6 heads, 7748 rows of 36 sequences (13176 launched) 22.2 / 45.2 / 47.9; of 64, 16 / 8 heads 1 x 526 (68, 17) 13.5 / 9.4 / 12.1, 8 / 1 heads 48 x 165 (576, 6)
// 8.9 / 11.7 / 11.9, 16 / 8 heads, 2439 rows of 41 sequences (12792 launched) 18.4 / 31.5 / 34.3.  Backward, four waves / two sets of two / four sets of two (head size 64): 1 x 727 with
// 32 / 8 heads (184, 23) 95.2 / 80.9 / 76.6, 6 x 777 with 16 / 4 (600, 25) 104 / 90 / 109, 5 x 103 with 40 / 8 (200, 4) 23.6 / 22.0 / 27.9; of 128, 5 x 132 with 64 / 8 (400, 5) 37.8 / 45.2.
Form fwd_form(const AttnArgs& a) {
  const RowWork w = row_work(a);
  if (w.launched > std::max<int64_t>(4096, std::min<int64_t>(8192, 16 * w.blocks))) return Form{4, 1};
  if (a.dh == 64) return w.steps >= 5 && w.blocks <= std::min(960, 32 * w.steps) ? Form{2, 2} : Form{4, 1};
  if (w.blocks <= std::min(256, 32 * w.steps) && w.steps >= 4) return Form{2, 2};
  if (w.blocks <= 384 && w.steps >= 24) return Form{2, 2};
  return w.blocks <= 512 && w.steps >= 28 ? Form{4, 2} : Form{4, 1};
}
Form dq_form(const AttnArgs& a) {
  const RowWork w = row_work(a);
  if (w.launched > 8192) return Form{4, 1};
  if (a.dh == 128) return w.steps >= 4 && w.blocks <= std::min(832, 32 * w.steps) ? Form{2, 2} : Form{4, 1};
  if (w.steps >= 8 && w.blocks <= std::min(352, 12 * w.steps)) return Form{2, 4};
  return w.steps >= 3 && w.blocks <= std::min(1280, 48 * w.steps) ? Form{2, 2} : Form{4, 1};
}
// dK / dV, likewise by the blocks of 64 keys and the chain of query tiles of the first of them, over the same shapes.  (A packed batch has fewer
// blocks than its bound, and its longest sequence is a longer chain beside them.)
Form dkv_form(const AttnArgs& a) {
  // a packed batch holds at most one partly filled block per sequence
  const int64_t all = (int64_t)((a.S + 63) / 64) * a.B, blocks = a.nkv * (a.cu_seqlens ? std::min<int64_t>(a.total_rows / 64 + a.B, all) : all);
  const int64_t chain = (int64_t)(a.nh / a.nkv) * ((a.S + 31) / 32);   // the longest: 32-query tiles, heads of the group times sequence
  if (a.dh == 64) {
    // Whole backward, us, blocks of 64 keys with four, two sets and one: 1 x 727 with 32 / 8 heads (96 blocks, chain 92) 74.7 / 92.8 / 128,
    // 5 x 787 (520, 100) 103 / 113 / 150, 12 x 486 with 40 / 8 (768, 80) 118 / 114 / 138, 4 sequences of 8874 rows with 32 / 8 (1136, 436) 546 / 539 / 700; where the
    // chain is short, 96 x 32 with 4 / 4 (384, 1) 18.2 / 13.1 / 11.7, 51 x 62 with 6 / 6 (306, 2) 22.1 / 16.9 / 15.7, 61 x 156 (1464, 25) 125 / 105 / 101.
    if (chain >= 6 && (blocks <= 256 || blocks <= std::min<int64_t>(512, 16 * chain) || blocks <= std::min<int64_t>(1024, 5 * chain))) return Form{2, 4};
    return chain >= 4 && blocks <= std::min<int64_t>(a.cu_seqlens ? 2560 : 1280, std::max<int64_t>(512, 40 * chain)) ? Form{2, 2} : Form{2, 1};
  }
  // Forward and backward, us, one set of two pairs / two sets / two sets of one pair, blocks of 64 keys and chain: 1 x 500 with 32 / 8 heads (64, 64) 89 / 73 / 67,
  // 2 x 905 (240, 116) 162 / 138 / 129, 7 x 405 with 40 / 8 (392, 65) 139 / 125 / 143, 1 x 6341 with 16 / 4 (400, 796) 1110 / 902 / 1124, 3 x 1333 (504, 168) 302 / 270 / 332,
  // 16 x 181 (384, 24) 70 / 69 / 76, 18 x 209 with 16 / 8 (576, 14) 55 / 58 / 66, 4 x 2208 with 16 / 4 (560, 276; backward) 367 / 313 / 415, 5 x 1601 with 40 / 8 (1040, 255) 656 / 709 / 907.
  if (blocks <= 256 && chain >= 4 && blocks <= std::max<int64_t>(96, 24 * chain)) return Form{1, 2};
  return blocks <= std::min<int64_t>(512, 16 * chain) || blocks <= std::min<int64_t>(832, 8 * chain) ? Form{2, 2} : Form{2, 1};
}

template <int D>
hipError_t launch_fwd_form(const AttnArgs& a, hipStream_t s) {
  const Form f = fwd_form(a);
  if (f.ns == 1) return launch_fwd<D, 4, 1>(a, s);
  if constexpr (D == 128)
    if (f.kw == 4) return launch_fwd<D, 4, 2>(a, s);
  return launch_fwd<D, 2, 2>(a, s);
}
template <int D>
hipError_t launch_bwd(const AttnArgs& a, hipStream_t s) {
  const Form q = dq_form(a), kv = dkv_form(a);
  hipError_t e;
  if (q.ns == 1) e = launch_dq<D, 4, 1>(a, s);
  else if (D == 128 || q.ns == 2) e = launch_dq<D, 2, 2>(a, s);
  else e = launch_dq<64, 2, 4>(a, s);
  if (e != hipSuccess) return e;
  // S, dP, dV and dK products of every (query, key, channel) triple
  ProfScope ps("attn_dkv_mfma", 4.0 * a.B * a.nh * D * (double)a.S * (a.S + 1), 0, s);
  if constexpr (D == 64) return kv.ns == 4 ? launch_dkv<2, 4>(a, s) : kv.ns == 2 ? launch_dkv<2, 2>(a, s) : launch_dkv<2, 1>(a, s);
  else return kv.ns == 1 ? launch_dkv_pair<2, 1>(a, s) : kv.kw == 1 ? launch_dkv_pair<1, 2>(a, s) : launch_dkv_pair<2, 2>(a, s);
}
}  // namespace

int attn_mfma_form(const AttnArgs& a, int pass) {
  if (!attn_mfma_supported(a)) return 0;
  const Form f = pass == 0 ? fwd_form(a) : pass == 1 ? dq_form(a) : dkv_form(a);
  return f.kw * 10 + f.ns;
}
hipError_t launch_attn_fwd_mfma(const AttnArgs& a, hipStream_t s) { return a.dh == 64 ? launch_fwd_form<64>(a, s) : launch_fwd_form<128>(a, s); }
hipError_t launch_attn_bwd_mfma(const AttnArgs& a, hipStream_t s) { return a.dh == 64 ? launch_bwd<64>(a, s) : launch_bwd<128>(a, s); }

}  // namespace tide
