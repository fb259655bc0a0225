// bf16 MFMA GEMM for gfx950 (CDNA4), fp32 accumulation, for the three layouts of the training step:
//   NT  C = A[M,K] B[N,K]^T   forward projections           (both operands K-contiguous)
//   NN  C = A[M,K] B[K,N]     input gradients dX = dY W     (B is N-contiguous)
//   TN  C = A[K,M]^T B[K,N]   weight gradients dW = dY^T X  (both operands contracted over rows)
//
// Design
//   * A block computes a tile of 128, 160, 192, 224 or 256 x 256 (8 wavefronts, the block owns its CU) or of 128 x 128 (4
//     wavefronts, two blocks share a CU) with v_mfma_f32_16x16x32_bf16; a wave owns half the rows x 64 of it.  Two waves per
//     SIMD either way: one alone cannot issue MFMAs back to back (measured ~83 % of the multi-wave MFMA rate).
//   * K is walked in slabs of 64 through five LDS units (see the kernel), filled by LDS-DMA buffer loads (global -> LDS
//     without passing through registers, hardware zero-fill outside the valid extent, so ragged M / N / K need no special
//     code).  What bounds the large tile is the memory side next to the matrix pipes: with every operand row aliased to
//     one line (all loads hit) the same code runs 25-40 % faster; the small tile needs twice the operand bytes per flop and is
//     bound by their delivery from L2 (1.16 PFLOP/s at 17-19 TB/s).
//   * Synchronisation is manual: one `s_waitcnt vmcnt(n)` (own DMA of the next slab has landed, younger loads stay in
//     flight) and one `s_barrier` per slab, before its last quarter.  Each unit is its own __shared__ array and every read
//     address is "array + per-lane offset + constant": the compiler can then tell that the operand reads do not alias the
//     DMA writes in flight and does not drain vmcnt before them.  Slabs past K are dummies (their loads fall outside the
//     buffer and zero-fill the free unit).  The instruction order is pinned: MFMA / LDS read (or DMA issue) alternate, so
//     LDS and address traffic hides in the MFMA shadow.
//   * LDS layout.  A "K-major" operand (contraction index contiguous in memory) is stored [row][64] with the 16-byte
//     pieces of a row XOR-swizzled by (row >> 1) & 7: DMA can only write 1 KiB contiguous per instruction, so padding is
//     impossible, and the swizzle makes the 16-byte operand reads of 16 consecutive rows hit 16 different bank groups.  An
//     operand whose contraction index is the slow one (B of NN, both operands of TN) is stored as in memory, [k][row], and
//     transposed on the way to the MFMA by ds_read_b64_tr_b16 (two per MFMA operand: four k each), swizzled by
//     TIDE_RSWZ.  No transposed copy of an operand ever exists in HBM.
//   * The contraction may run over two operand pairs back to back (d b = dGate W_gate + dUp W_up), and
//     the epilogue fuses alpha (host and device scalar), a residual add, accumulation into C and the cast.
//     bf16 results without residual/accumulate go through a wave-private LDS patch to leave as 16-byte
//     row segments; everything else is stored straight from the accumulators.
//   * Tiles that do not fill the chip are split over K (two forms, see MfmaParams), and the tile is chosen with that
//     in mind (tile_edge); in between, the tile's height is (tall_height).
//   * Work-groups are renumbered so that each of the 8 XCDs (round-robin dispatch) gets a contiguous
//     range of tiles, walked in groups of 4 tile-rows: neighbouring tiles share A/B panels in that
//     XCD's L2.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "kernels.h"
#include "prof.h"
#include "tide_common.h"

namespace tide {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

namespace {

struct MfmaParams {
  const bf16_t* A; const bf16_t* B; const bf16_t* A2; const bf16_t* B2;
  void* C; const void* R; const float* alpha_dev;
  int M, N, K, K2;
  int lda, ldb, ldc, ldr;
  float alpha;
  int accumulate;
  int tiles_m, tiles_n;
  const int* m_dev; int m_off;   // optional device-side M: effective M = clamp(*m_dev - m_off, 0, M)
  const int* k_dev; int k_off;   // optional device-side K (pair 0 only)
  // Split over K.  kSplitTail (256 x 256 tiles, fp32 results): tiles [0, split_full) are whole; each later tile is
  // worked on by split_s blocks, each over 1/split_s of the slabs; part 0 writes C, part j > 0 writes its 256 x 256
  // partial sum to split_scratch[(j - 1) * (tiles - split_full) + tile - split_full], and splitk_fixup_kernel adds the
  // partial sums to C in a fixed order afterwards.  kSplitAll: the tiles from split_all().full on are worked on by
  // split_all().parts blocks each, every one of which writes its partial sum to split_scratch[part * tail + tile - full];
  // splitk_reduce_kernel adds them in the order of the parts and does what the epilogue would.  Both kernels take the
  // number of parts from the sizes they find on the device; with one part the epilogue has written C.
  int split, split_s, split_full;
  float* split_scratch;
};
struct MfmaAdamParams : MfmaParams { AdamTarget adam; };
enum : int { kSplitNone = 0, kSplitTail = 1, kSplitAll = 2 };

// How a launch whose tiles do not fill the chip is split over K.  ns, measured on 256 x 256 and on 128 x 128 tiles:
//   slab       a slab of 64: 1410, or 550 (750 once blocks share a CU, 870 at two per CU: 1.16 PFLOP/s, the rate
//              at which L2 delivers the operands of 128 x 128 tiles)
//   traffic    one tile's partial sum, written and read back at about 8 TB/s: 65 / 16
//   fixed      the second launch, and what storing an fp32 partial sum takes longer than storing a bf16 result: 12000 / 5000
// With nk slabs and t tiles to split, n parts save slab nk (1 - 1 / n) - traffic t n, most at n = sqrt(slab nk / (traffic t));
// that has to exceed the fixed costs, and a part keeps a few slabs.
struct SplitCost { int slots, min_slabs, slab, traffic, fixed; };
__host__ __device__ inline constexpr SplitCost split_cost(int BT) {
  return BT == 256 ? SplitCost{256, 8, 1410, 65, 12000} : SplitCost{512, 4, 550, 16, 5000};
}
__host__ __device__ inline int split_parts(int BT, int tiles, int slabs) {
  const SplitCost c = split_cost(BT);
  if (tiles <= 0) return 1;
  const int by_slots = c.slots / tiles, by_k = slabs / c.min_slabs;
  int lo = 1, hi = by_slots < by_k ? by_slots : by_k;
  if (hi < 2) return 1;
  while (lo < hi) {   // largest n with traffic t n^2 <= slab nk
    const int n = (lo + hi + 1) / 2;
    if ((int64_t)c.traffic * tiles * n * n <= (int64_t)c.slab * slabs) lo = n; else hi = n - 1;
  }
  if (lo < 2) return 1;
  const int64_t part = (slabs + lo - 1) / lo;
  const int64_t cost = c.fixed + (int64_t)c.traffic * tiles * lo + (BT == 128 && tiles * lo > 256 ? 250 * part : 0);
  return c.slab * (slabs - part) > cost ? lo : 1;
}
struct SplitAll { int full, parts; };   // tiles that are not split, and the parts of each of the others
template <int BT>
__host__ __device__ inline SplitAll split_all(int tiles, int slabs) {
  // whole rounds of 256 large tiles stay whole (more than 256 small ones are never split)
  const int full = BT == 256 ? tiles / 256 * 256 : 0;
  const int n = split_parts(BT, tiles - full, slabs);
  return n > 1 ? SplitAll{full, n} : SplitAll{tiles, 1};
}
// 64-deep slabs of a contraction over one or two operand pairs
__host__ __device__ inline int split_slabs(int K, int K2) { return (K + 63) / 64 + (K2 + 63) / 64; }

// tile index (XCD-contiguous order, groups of 4 tile rows) -> tile coordinates
#ifndef TIDE_TILE_GROUP
#define TIDE_TILE_GROUP 4
#endif
__device__ __forceinline__ void tile_coords(int v, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
  constexpr int GROUP = TIDE_TILE_GROUP;
  const int per_group = GROUP * tiles_n;
  const int gid = v / per_group;
  const int first_m = gid * GROUP;
  const int gsz = min(tiles_m - first_m, GROUP);
  const int in_g = v - gid * per_group;
  tile_m = first_m + in_g % gsz;
  tile_n = in_g / gsz;
}

// wait until at most n of this wave's vector-memory operations are outstanding (vmcnt only)
#define TIDE_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8))

// swizzle of a row-major stage: 16-byte piece index ^= (k-row & 3) << 2, i.e. the four k-rows that one transposing read
// touches sit in four different 64-byte bank groups; and bit 1 of the piece index is flipped with bit 3 of the k-row: the
// 16-lane groups of a read differ in k by 8 rows, and the flip keeps two neighbouring groups on different banks.
#define TIDE_RSWZ(krow) ((((krow) & 3) << 2) ^ ((((krow) >> 3) & 1) << 1))
constexpr uint32_t kOobOffset = 0x7FFFFFF0u;  // beyond any buffer extent used here: the load returns zeros

// One LDS-DMA load of 16 bytes per lane, written as an instruction: the 64 lanes' data go to 1 KiB of LDS at
// `lds_addr` (a scalar), each lane fetches from byte `voff` of the buffer `rsrc` (zeros outside its extent).
// The compiler does not see that this writes LDS, so it never orders an LDS read after it by waiting for every
// load in flight (which it does for the builtin form as soon as it cannot prove that the read and the loads in
// flight touch different arrays, e.g. where paths of the loop merge); all waits on these loads are explicit.
typedef int i32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4_t make_rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)base;
  i32x4_t r;
  r[0] = (int)(uint32_t)a; r[1] = (int)((uint32_t)(a >> 32) & 0xffffu); r[2] = (int)bytes; r[3] = 0x00020000;
  return r;
}
__device__ __forceinline__ void dma16(i32x4_t rsrc, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rsrc));
}

// One operand (A or B) of one block: R rows (BM or BN) of the tile, either K-major or row-major over K.
template <int R, int NW, bool RMAJ, int T16, int BK>   // T16 = 16-row MFMA fragments per wave along this dimension; BK = slab depth
struct Operand {
  // Rows that a stage has room for: every wave issues the same number of 1 KiB DMA instructions, and a row-major k-row is a
  // power of two long.  The rows from R on are beyond the loads' extent and hold zeros that no read touches.
  static constexpr int RL = RMAJ ? (R > 128 ? 256 : 128) : (R * BK * 2 + NW * 1024 - 1) / (NW * 1024) * (NW * 1024) / (BK * 2);
  static_assert(R % 16 == 0 && R <= RL, "rows of a tile");
  static constexpr int STAGE = RL * BK;                                  // elements per stage
  static constexpr int CHUNKS = STAGE * 2 / 1024;                        // 1 KiB DMA instructions per stage
  static constexpr int PER_WAVE = CHUNKS / NW;
  static_assert(CHUNKS % NW == 0 && PER_WAVE >= 1, "DMA chunks must split evenly over the waves");
  static constexpr int PPR = RL / 8;                                     // 16-byte pieces per k-row (row-major)
  static constexpr int RPC = 64 / PPR;                                   // k-rows per DMA chunk (row-major)
  static constexpr int KPIECES = BK / 8;                                 // 16-byte pieces per K-major row (4 or 8)
  static constexpr int KROWS = 64 / KPIECES;                             // K-major rows per DMA chunk (16 or 8)
  static constexpr int SWZ_SHIFT = (BK == 32) ? 2 : 1;                   // swizzle: piece ^= (row >> shift) & (KPIECES-1)

  // Stateless on purpose: the tile pointers and extents stay plain kernel locals (SGPRs).  Bundling them
  // in a struct with the per-lane offsets made the compiler keep that struct in scratch memory, the
  // buffer descriptors then lived in VGPRs and every DMA load became a waterfall loop.

  // per-lane byte offsets of this wave's DMA chunks, without the k0 term; K-major also yields the 16-byte
  // piece of a row that this lane fetches (swizzled)
  static __device__ __forceinline__ void lane_offsets(int ld, int wave, int lane, uint32_t (&off)[PER_WAVE],
                                                      int (&piece)[PER_WAVE]) {
    if (RMAJ) {
      // chunk = RPC k-rows x (R*2) bytes; LDS slot (krow, s) holds piece s ^ TIDE_RSWZ(krow) of that k-row
      const int kr = lane / PPR, pc = lane % PPR;
#pragma unroll
      for (int i = 0; i < PER_WAVE; ++i) {
        const int krow = (wave * PER_WAVE + i) * RPC + kr;
        const int p = pc ^ TIDE_RSWZ(krow);
        off[i] = R == RL || p < R / 8 ? (uint32_t)((krow * ld + p * 8) * 2) : kOobOffset;
        piece[i] = 0;
      }
    } else {
      // chunk = KROWS rows x (BK*2) bytes; LDS slot (row, s) holds piece s ^ swizzle(row) of that row
      const int rl = lane / KPIECES, slot = lane % KPIECES;
#pragma unroll
      for (int i = 0; i < PER_WAVE; ++i) {
        const int row = (wave * PER_WAVE + i) * KROWS + rl;
        piece[i] = slot ^ ((row >> SWZ_SHIFT) & (KPIECES - 1));
        off[i] = (uint32_t)((row * ld + piece[i] * 8) * 2);
      }
    }
  }

  // The scalar part of the slab [k0, k0+BK) of a K-major operand whose last slab is ragged.  tile = operand pointer already
  // offset to the tile's first row; rows_valid = tile rows inside the matrix; Kc = contraction length.  A slab with k0 >= Kc is
  // a dummy: every load is out of range and writes zeros.
  // The loads are issued one by one as instructions (dma16): chunk<I> issues the wave's I-th chunk into the LDS unit at byte address `unit` (scalar); wave_s is the wave index as a scalar.
  struct SlabDesc { i32x4_t rs; int k0, Kc; };
  static __device__ __forceinline__ SlabDesc slab_desc(const bf16_t* tile, int ld, int rows_valid, int k0, int Kc) {
    SlabDesc d;
    d.k0 = k0; d.Kc = Kc;
    d.rs = make_rsrc_words(tile, (uint32_t)(((int64_t)(rows_valid - 1) * ld + Kc) * 2));
    return d;
  }
  // A load whose lane offset is a loop constant: a row-major operand always, a K-major one when every slab is
  // whole (K a multiple of BK), where neither the per-lane test "is this piece still inside K" nor a per-lane k
  // offset is needed: the slab's k0 sits in the descriptor's base (and its extent ends k0 earlier, so the row
  // bound stays where it was), and a dummy slab has an empty extent.
  template <int I>
  static __device__ __forceinline__ void chunk_whole(const SlabDesc& d, uint32_t unit, const uint32_t (&off)[PER_WAVE], int wave_s) {
    dma16(d.rs, unit + (uint32_t)((wave_s * PER_WAVE + I) * 1024), off[I]);
  }
  template <int I>
  static __device__ __forceinline__ void chunk(const SlabDesc& d, uint32_t unit, const uint32_t (&off)[PER_WAVE],
                                               const int (&piece)[PER_WAVE], int wave_s) {
    const bool kin = (d.k0 + piece[I] * 8) < d.Kc;
    dma16(d.rs, unit + (uint32_t)((wave_s * PER_WAVE + I) * 1024), kin ? off[I] + (uint32_t)(d.k0 * 2) : kOobOffset);
  }

  // Per-lane element offsets of the operand reads inside a stage, computed once.  K-major: one per k32 step (the swizzle
  // is an XOR, not additive in the step); row-major: one per fragment.  The values are made opaque to the optimiser:
  // every read address is then "stage array + offset + constant", a short chain that keeps the no-alias information
  // of the stage arrays (longer chains lose it, and a read without it waits for all DMA writes in flight).
  // ---- 16x16x32 MFMA: a fragment is 16 tile rows x 32 k; lane l holds row l & 15, k = 8 * (l >> 4) .. + 7 ----
  static constexpr int NRO16 = RMAJ ? T16 : BK / 32;
  static __device__ __forceinline__ void read_offsets16(int wbase, int lane, uint32_t (&ro)[NRO16]) {
    const int r16 = lane & 15, g = lane >> 4;
    if (RMAJ) {
      // transposing reads: lane j of a 16-lane group addresses k-row j / 4, tile rows 4 * (j % 4) .. + 3 and
      // receives tile row j for those 4 k; the group's k-rows start at 8 * g
      const int kq = (lane >> 2) & 3, rq = lane & 3;
#pragma unroll
      for (int i = 0; i < T16; ++i) {
        const int col = wbase + 16 * i + 4 * rq;
        const int krow = g * 8 + kq;
        ro[i] = (uint32_t)(krow * RL + ((((col >> 3) ^ TIDE_RSWZ(krow)) << 3) | (col & 7)));
      }
    } else {
      const int sw = (r16 >> SWZ_SHIFT) & (KPIECES - 1);
#pragma unroll
      for (int h = 0; h < NRO16; ++h) ro[h] = (uint32_t)((wbase + r16) * BK + (((h * 4 + g) ^ sw) * 8));
    }
#pragma unroll
    for (int i = 0; i < NRO16; ++i) asm("" : "+v"(ro[i]));
  }
  // NF fragments starting at fragment index F0, of the k32 step `h` (< BK/32) of a stage
  template <int F0, int NF, typename StagePtr>
  static __device__ __forceinline__ void frags16(StagePtr stage, int h, const uint32_t (&ro)[NRO16], u32x4_t (&f)[NF]) {
    if (RMAJ) {
      typedef short s16x4_t __attribute__((ext_vector_type(4)));
      typedef __attribute__((address_space(3))) s16x4_t* lds_tr_t;
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_t)(stage + ro[F0 + i] + (h * 32) * RL));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_t)(stage + ro[F0 + i] + (h * 32 + 4) * RL));
        const uint2 a = __builtin_bit_cast(uint2, lo), b2 = __builtin_bit_cast(uint2, hi);
        f[i][0] = a.x; f[i][1] = a.y; f[i][2] = b2.x; f[i][3] = b2.y;
      }
    } else {
      typedef __attribute__((address_space(3))) const u32x4_t* lds_v4_t;
#pragma unroll
      for (int i = 0; i < NF; ++i) f[i] = *(lds_v4_t)(stage + ro[h] + (F0 + i) * 16 * BK);
    }
  }

};

template <int N>
struct Int : std::integral_constant<int, N> {};

// A weight's state passes through once per step, and past the caches: kept in L2 it drove out the operand panels that the
// blocks still multiplying read there (us with plain / non-temporal loads and stores, neither alone does it: 128256 x 4096 over 1700
// rows 3910 / 3516, over 300 3262 / 3032, 32000 x 2048 over 2560 589 / 575).
typedef float f32x4_nt __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 load_once(const float* q) {
  const f32x4_nt x = __builtin_nontemporal_load(reinterpret_cast<const f32x4_nt*>(q));
  return make_float4(x.x, x.y, x.z, x.w);
}
__device__ __forceinline__ void store_once(float* q, float4 v) {
  const f32x4_nt x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<f32x4_nt*>(q));
}
// four weights' update: g their gradient, m / v / th as loaded, at their offset
__device__ __forceinline__ void adam_store(const AdamTarget& t, const AdamRate& rate, float* C, size_t at, float4 g, float4 m, float4 v, float4 th) {
  adam_update(rate, g.x, m.x, v.x, th.x);
  adam_update(rate, g.y, m.y, v.y, th.y);
  adam_update(rate, g.z, m.z, v.z, th.z);
  adam_update(rate, g.w, m.w, v.w, th.w);
  store_once(C + at, g);
  store_once(t.m + at, m);
  store_once(t.v + at, v);
  store_once(t.master + at, th);
  *reinterpret_cast<uint2*>((bf16_t*)t.w + at) = make_uint2(f2bf2(th.x, th.y), f2bf2(th.z, th.w));
}

}  // namespace

// ------------------------------------------------------------------------------------------------
// Tiles of BM x BN with v_mfma_f32_16x16x32_bf16: BN = 256 on eight waves of BM / 2 x 64, BN = 128 on four waves of 64 x 64
// (whose five LDS units of 16 KiB let two blocks share a CU).  On this chip the matrix pipes sustain a higher rate under
// the package power limit with this form than with 32x32x16 (a pure-MFMA loop on random operands: 2.10 against 1.88
// PFLOP/s), while the LDS operand traffic per flop is the same (a 16-row x 32-k fragment is one 16-byte read per lane, like
// a 32-row x 16-k one).  A wave owns (BM / 32) x 4 tiles of 16 x 16; a "quarter" of the schedule is one k32 step of four of
// its A fragments against its four B fragments: 16 MFMAs (256 clocks), with the A fragments double-buffered per quarter
// and the B fragments per k32 step.  A slab is four quarters at BM = 256; below, two of all its A fragments.  The MFMAs take the B fragment
// first, so accumulator element q of lane l in tile (i, j) is row 16 i + (l & 15), column 16 j + 4 (l >> 4) + q (see the
// epilogue).  (Four waves of 128 x 128 at BM = 256, a third less LDS traffic, measured 2.5 to 10 % slower: one wave per SIMD
// leaves every wait of that wave exposed.)
// KWHOLE: every slab of the launch is whole (K, and K2 of a second operand pair, multiples of 64 known on the
// host).  A K-major operand's loads then need neither the per-lane test "is this piece still inside K" nor a
// per-lane k offset: k0 moves into the buffer descriptor and the lane offsets are loop constants, which takes
// three vector instructions per load out of the loop (they compete with the MFMAs for the vector issue port;
// NT 33.2 -> 32.2 ms and NN 30.1 -> 29.5 ms per training step at the 8B shape).
// ------------------------------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int BM, int BN, bool AMM, bool BNM, typename TO, bool KWHOLE, bool ADAM, bool LONG = false>
__device__ __forceinline__ void gemm_block(std::conditional_t<ADAM, MfmaAdamParams, MfmaParams> p, int pid) {   // pid: which of the launch's blocks
  static_assert(BN == 256 ? BM % 32 == 0 && BM >= 128 && BM <= 256 : BN == 128 && BM == 128, "tile edges");
  constexpr int BK = 64, WAVES_M = 2, WAVES_N = BN / 64, NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;   // BM / 2 x 64
  constexpr int TM = WM / 16, TN = WN / 16;             // 4 to 8 x 4 tiles of 16 x 16
  constexpr int GA = TM == 8 ? 4 : TM;                  // A fragments per quarter
  constexpr int TM2 = (TM + 1) / 2;                     // pairs of tile rows, the last of an odd TM half empty
  using OpA = Operand<BM, NW, AMM, TM, BK>;
  using OpB = Operand<BN, NW, BNM, TN, BK>;
  constexpr int A_STAGE = OpA::STAGE, B_STAGE = OpB::STAGE;
  constexpr int NVA = OpA::PER_WAVE, NVB = OpB::PER_WAVE;
  constexpr int NMF = GA * TN;                          // MFMAs per quarter
  typedef __attribute__((address_space(3))) const bf16_t* lds_bf_t;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  const int lc = lane & 15, lg = lane >> 4;

  if (p.m_dev) p.M = max(0, min(p.M, *p.m_dev - p.m_off));
  if (p.k_dev) p.K = max(0, min(p.K, *p.k_dev - p.k_off));
  if (p.K == 0 && p.K2 == 0 && p.accumulate && p.split != kSplitTail && !ADAM) return;   // nothing to add

  int tile_m, tile_n;
  int part = 0, nparts = 1, tail_index = 0, ntail = 0;   // split over K (see MfmaParams)
  {
    const int tiles_m = (p.M + BM - 1) / BM;
    const int nb = tiles_m * p.tiles_n;
    int full = nb;                           // tiles that are not split
    if (p.split == kSplitTail) { full = p.split_full; nparts = p.split_s; }   // (never with a device-side M)
    else if (p.split == kSplitAll) {
      const SplitAll sa = split_all<BN>(nb, split_slabs(p.K, p.A2 ? p.K2 : 0));
      full = sa.full; nparts = sa.parts;
    }
    ntail = nb - full;
    const int items = full + ntail * nparts;
    if (pid >= items) return;
    // Work-groups go to the XCDs round-robin in the order of their index: the whole tiles (a multiple of 256)
    // come first and each XCD gets a contiguous range of them; the parts of the split tiles come last, again
    // spread over all XCDs, so that they fill the last round everywhere.
    int count = full, base = 0;
    if (pid >= full) { base = full; pid -= full; count = items - full; }
    const int xcd = pid & 7, idx = pid >> 3;
    const int q = count >> 3, r = count & 7;
    int v = base + xcd * q + min(xcd, r) + idx;
    if (v >= full) {
      const int u = v - full;
      if (p.split == kSplitAll) {            // part by part: the tiles an XCD works on share the panels of one K range
        part = u / ntail;
        tail_index = u - part * ntail;
      } else {
        tail_index = u / nparts;
        part = u - tail_index * nparts;
      }
      v = full + tail_index;
    } else {
      nparts = 1;
    }
    tile_coords(v, tiles_m, p.tiles_n, tile_m, tile_n);
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const bf16_t* a_tile0 = AMM ? p.A + m0 : p.A + (size_t)m0 * p.lda;
  const bf16_t* b_tile0 = BNM ? p.B + n0 : p.B + (size_t)n0 * p.ldb;
  const bf16_t* a_tile1 = p.A2 ? (AMM ? p.A2 + m0 : p.A2 + (size_t)m0 * p.lda) : a_tile0;
  const bf16_t* b_tile1 = p.B2 ? (BNM ? p.B2 + n0 : p.B2 + (size_t)n0 * p.ldb) : b_tile0;
  const int a_rows = min(BM, p.M - m0), b_rows = min(BN, p.N - n0);
  uint32_t a_off[NVA], b_off[NVB];
  int a_piece[NVA], b_piece[NVB];
  OpA::lane_offsets(p.lda, wave, lane, a_off, a_piece);
  OpB::lane_offsets(p.ldb, wave, lane, b_off, b_piece);

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[i][j][q] = 0.f;

  const int nk1 = (p.K + BK - 1) / BK;
  const int nkp2 = p.A2 ? (p.K2 + BK - 1) / BK : 0;
  // this block's slabs: all of them, or its part of a split tile (slab numbers below are relative to kt_lo)
  const int nk_all = nk1 + nkp2;
  const int per_part = (nk_all + nparts - 1) / nparts;
  const int kt_lo = min(nk_all, part * per_part);
  const int nk = min(nk_all, kt_lo + per_part) - kt_lo;

  // which operand pair and k offset slab kt stands for (slabs past nk are dummies: every load out of range)
  auto slab = [&](int kt, int& pr, int& k0, int& Kc) {
    const int g = kt_lo + kt;
    pr = 0; k0 = g * BK; Kc = p.K;
    if (kt >= nk) { k0 = p.K + BK; }
    else if (g >= nk1) { pr = 1; k0 = (g - nk1) * BK; Kc = p.K2; }
  };
  uint32_t a_ro[OpA::NRO16], b_ro[OpB::NRO16];
  OpA::read_offsets16(wave_m * WM, lane, a_ro);
  OpB::read_offsets16(wave_n * WN, lane, b_ro);
  // A fragments of group G (0, 1) / the B fragments of the k32 step h of an LDS unit
  auto frags_a = [&](const bf16_t* unit, int h, auto G, u32x4_t (&fa)[GA]) {
    OpA::template frags16<decltype(G)::value * GA, GA>((lds_bf_t)unit, h, a_ro, fa);
  };
  auto frags_b = [&](const bf16_t* unit, int h, u32x4_t (&fb)[TN]) {
    OpB::template frags16<0, TN>((lds_bf_t)unit, h, b_ro, fb);
  };
  // ---- epilogue: needs, per wave, an LDS patch of 32 x (WN + 4) floats that no DMA is writing any more ----
  // The MFMAs are issued with their operands swapped (B fragment first), so an accumulator tile holds the
  // TRANSPOSE of its 16 x 16 block: element q of lane l in tile (i, j) is row m = 16 i + (l & 15), columns
  // n = 16 j + 4 (l >> 4) + q.  A lane thus owns four CONSECUTIVE columns of one row: 16 bytes of an fp32 result
  // (one store instead of four), 8 bytes of a bf16 one (one LDS write per tile into the staging patch).
  constexpr int kPatchElems = 32 * (WN + 4) * 2;   // in bf16 elements
  auto epilogue = [&](bf16_t* patch_mem) {
    float alpha = p.alpha;
    if (p.alpha_dev) alpha *= *p.alpha_dev;
    TO* C = (TO*)p.C;
    const TO* R = (const TO*)p.R;
    const int wm0 = m0 + wave_m * WM, wn0 = n0 + wave_n * WN;
    if (!ADAM && p.split == kSplitAll && nparts > 1) {
      // the partial sum as it is, tile-local; rows and columns past the matrix are not read back
      float* out = p.split_scratch + ((size_t)part * ntail + tail_index) * (size_t)(BM * BN);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int row = wave_m * WM + 16 * i + lc, col = wave_n * WN + 16 * j + 4 * lg;
          if (m0 + row < p.M && n0 + col < p.N) *reinterpret_cast<f32x4_t*>(out + row * BN + col) = acc[i][j];
        }
      return;
    }
    if constexpr (ADAM) {
      if (nparts == 1) {
        // The weight's update with the gradient still in the accumulators.  Sixteen rows of the wave at a time go through its
        // LDS patch, so that every access of the five float arrays is a 256-byte row segment; the old values of those rows are
        // requested before the patch is written.  Bound by memory, like the separate pass, which reads the gradient again: 34
        // bytes per weight in two kernels, 30 here (128256 x 4096 over 1400 rows 1.41 + 2.89 ms, 3.21 so; 5632 x 2048 over 2500 53 + 66 us,
        // 112).  Two rows of four loads instead of four in flight, or the CUs started in 2 to 16 phases: no gain.
        __builtin_amdgcn_s_barrier();
        constexpr int PF = WN + 4, PIECES = WN / 4, NT = 16 * PIECES / 64;
        float* patch = reinterpret_cast<float*>(patch_mem);
        float* Cf = reinterpret_cast<float*>(C);
        const AdamRate rate = adam_rate(p.adam);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          float4 m[NT], v[NT], th[NT], old[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const int pc = lane + 64 * t, gm = wm0 + 16 * i + pc / PIECES, gn = wn0 + pc % PIECES * 4;
            const size_t at = (size_t)gm * p.ldc + gn;
            m[t] = v[t] = th[t] = old[t] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (gm < p.M && gn < p.N) {
              m[t] = load_once(p.adam.m + at);
              v[t] = load_once(p.adam.v + at);
              th[t] = load_once(p.adam.master + at);
              if (p.accumulate) old[t] = *reinterpret_cast<const float4*>(Cf + at);
            }
          }
#pragma unroll
          for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4_t*>(patch + lc * PF + 16 * j + 4 * lg) = acc[i][j];
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const int pc = lane + 64 * t, row = pc / PIECES, gm = wm0 + 16 * i + row, gn = wn0 + pc % PIECES * 4;
            if (gm < p.M && gn < p.N) {
              const size_t at = (size_t)gm * p.ldc + gn;
              const float4 a = *reinterpret_cast<const float4*>(patch + row * PF + pc % PIECES * 4);
              float4 g = make_float4(alpha * a.x, alpha * a.y, alpha * a.z, alpha * a.w);
              if (p.accumulate) { g.x += old[t].x; g.y += old[t].y; g.z += old[t].z; g.w += old[t].w; }
              adam_store(p.adam, rate, Cf, at, g, m[t], v[t], th[t]);
            }
          }
        }
        return;
      }
    }
    bool staged = false;
    if constexpr (sizeof(TO) == 2) {
      constexpr int PIECES = WN / 8;
      if (!R && !p.accumulate && (p.ldc % 8) == 0 && (p.N % 8) == 0) {
        staged = true;
        // bf16 result through the wave's LDS patch (32 rows = two tile rows at a time) so that it leaves as
        // 16-byte row segments.  Every wave waited for its own DMA; the barrier orders the last operand reads
        // of the other waves before the patch writes.
        __builtin_amdgcn_s_barrier();
        constexpr int PP = WN + 8;
        bf16_t* patch = patch_mem;
#pragma unroll
        for (int i2 = 0; i2 < TM2; ++i2) {
#pragma unroll
          for (int ih = 0; ih < min(2, TM - 2 * i2); ++ih)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              const f32x4_t v = acc[2 * i2 + ih][j];
              *reinterpret_cast<uint2*>(patch + (16 * ih + lc) * PP + 16 * j + 4 * lg) =
                  make_uint2(f2bf2(alpha * v[0], alpha * v[1]), f2bf2(alpha * v[2], alpha * v[3]));
            }
#pragma unroll
          for (int t = 0; t < 16 * min(2, TM - 2 * i2) * PIECES / 64; ++t) {
            const int pc = lane + 64 * t;
            const int row = pc / PIECES, piece = pc % PIECES;
            const int gm = wm0 + 32 * i2 + row, gn = wn0 + piece * 8;
            const u32x4_t val = *reinterpret_cast<const u32x4_t*>(patch + row * PP + piece * 8);
            if (gm < p.M && gn < p.N)
              *reinterpret_cast<u32x4_t*>(reinterpret_cast<bf16_t*>(C) + (size_t)gm * p.ldc + gn) = val;
          }
        }
      } else if (R && !p.accumulate && (p.ldc % 8) == 0 && (p.ldr % 8) == 0 && (p.N % 8) == 0) {
        staged = true;
        // bf16 result plus residual: the patch keeps fp32 so that alpha * acc + residual is rounded once
        __builtin_amdgcn_s_barrier();
        constexpr int PF = WN + 4;
        float* patch = reinterpret_cast<float*>(patch_mem);
        const bf16_t* Rb = reinterpret_cast<const bf16_t*>(R);
#pragma unroll
        for (int i2 = 0; i2 < TM2; ++i2) {
#pragma unroll
          for (int ih = 0; ih < min(2, TM - 2 * i2); ++ih)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              const f32x4_t v = acc[2 * i2 + ih][j];
              *reinterpret_cast<float4*>(patch + (16 * ih + lc) * PF + 16 * j + 4 * lg) =
                  make_float4(alpha * v[0], alpha * v[1], alpha * v[2], alpha * v[3]);
            }
#pragma unroll
          for (int t = 0; t < 16 * min(2, TM - 2 * i2) * PIECES / 64; ++t) {
            const int pc = lane + 64 * t;
            const int row = pc / PIECES, piece = pc % PIECES;
            const int gm = wm0 + 32 * i2 + row, gn = wn0 + piece * 8;
            if (gm < p.M && gn < p.N) {
              float v[8], r[8];
              const float4 a0 = *reinterpret_cast<const float4*>(patch + row * PF + piece * 8);
              const float4 a1 = *reinterpret_cast<const float4*>(patch + row * PF + piece * 8 + 4);
              v[0] = a0.x; v[1] = a0.y; v[2] = a0.z; v[3] = a0.w; v[4] = a1.x; v[5] = a1.y; v[6] = a1.z; v[7] = a1.w;
              ld8(Rb, (size_t)gm * p.ldr + gn, r);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] += r[e];
              st8(reinterpret_cast<bf16_t*>(C), (size_t)gm * p.ldc + gn, v);
            }
          }
        }
      }
    }
    if (staged) return;
    if constexpr (sizeof(TO) == 4) {
      if (!R && (p.ldc % 4) == 0 && (p.N % 4) == 0 && (((uintptr_t)C) & 15) == 0) {
        // fp32 result: a lane's four columns are one 16-byte access.  With accumulate, the old values of two tile
        // rows are all requested before the first of them is used.  A later part of a split tile stores its
        // partial sum to its scratch tile instead (pitch 256, tile-local coordinates, never accumulating).
        float* Cf = reinterpret_cast<float*>(C);
        size_t pitch = (size_t)p.ldc;
        int mo = 0, no = 0;
        bool add = p.accumulate != 0;
        if (part > 0) {
          Cf = p.split_scratch + ((size_t)(part - 1) * ntail + tail_index) * (size_t)(BM * BN);
          pitch = BN; mo = m0; no = n0; add = false;
        }
#pragma unroll
        for (int i2 = 0; i2 < TM2; ++i2) {
          float4 old[2][TN];
          if (add) {
#pragma unroll
            for (int ih = 0; ih < min(2, TM - 2 * i2); ++ih)
#pragma unroll
              for (int j = 0; j < TN; ++j) {
                const int gm = wm0 + 16 * (2 * i2 + ih) + lc, gn = wn0 + 16 * j + 4 * lg;
                old[ih][j] = (gm < p.M && gn < p.N) ? *reinterpret_cast<const float4*>(Cf + (size_t)gm * pitch + gn)
                                                    : make_float4(0.f, 0.f, 0.f, 0.f);
              }
          }
#pragma unroll
          for (int ih = 0; ih < min(2, TM - 2 * i2); ++ih)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              const int gm = wm0 + 16 * (2 * i2 + ih) + lc, gn = wn0 + 16 * j + 4 * lg;
              const f32x4_t v = acc[2 * i2 + ih][j];
              float4 o = make_float4(alpha * v[0], alpha * v[1], alpha * v[2], alpha * v[3]);
              if (add) { o.x += old[ih][j].x; o.y += old[ih][j].y; o.z += old[ih][j].z; o.w += old[ih][j].w; }
              if (gm < p.M && gn < p.N) *reinterpret_cast<float4*>(Cf + (size_t)(gm - mo) * pitch + (gn - no)) = o;
            }
        }
        return;
      }
    }
    // everything else, element by element
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int gm = wm0 + 16 * i + lc;
      if (gm >= p.M) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int gn = wn0 + 16 * j + 4 * lg + q;
          if (gn >= p.N) continue;
          float v = alpha * acc[i][j][q];
          if (R) v += ldf(R, (size_t)gm * p.ldr + gn);
          if (p.accumulate) v += ldf(C, (size_t)gm * p.ldc + gn);
          stf(C, (size_t)gm * p.ldc + gn, v);
        }
    }
  };

  u32x4_t fa0[GA], fa1[GA], fb0[TN], fb1[TN];
  {
    // ---- slabs of 64: THREE LDS units for one operand and TWO for the other (5 x 32 KiB = all of the 160 KiB) ----
    // The operand DMA of a slab has to land within one slab time when the ring is two deep on both sides, and
    // a burst of 64 KiB per CU takes about that long to deliver: the matrix pipes then wait for it every slab.
    // With a third unit, the "deep" operand is fetched one slab further ahead and only the other one's half of
    // the bytes is on the one-slab clock.  Slab kt lives in deep unit kt % 3 and shallow unit kt % 2; the barrier
    // of a slab sits before its last quarter.  Loads complete in order, so waiting for "all but the youngest
    // NDEEP" means everything older than the deep operand's youngest slab has landed.
    constexpr bool DEEPB = BM < BN;   // which operand owns the three units: the larger
    constexpr int D_STAGE = DEEPB ? B_STAGE : A_STAGE, S_STAGE = DEEPB ? A_STAGE : B_STAGE;
    __shared__ __attribute__((aligned(1024))) bf16_t ld0[D_STAGE];
    __shared__ __attribute__((aligned(1024))) bf16_t ld1[D_STAGE];
    __shared__ __attribute__((aligned(1024))) bf16_t ld2[D_STAGE];
    __shared__ __attribute__((aligned(1024))) bf16_t ls0[S_STAGE];
    __shared__ __attribute__((aligned(1024))) bf16_t ls1[S_STAGE];
    // the units that only the long rings have (A: ld0 .. ld4, B: ls0 .. ls4)
    __shared__ __attribute__((aligned(1024))) bf16_t ld3[LONG ? D_STAGE : 1];
    __shared__ __attribute__((aligned(1024))) bf16_t ld4[LONG ? D_STAGE : 1];
    __shared__ __attribute__((aligned(1024))) bf16_t ls2[LONG ? S_STAGE : 1];
    __shared__ __attribute__((aligned(1024))) bf16_t ls3[LONG ? S_STAGE : 1];
    __shared__ __attribute__((aligned(1024))) bf16_t ls4[LONG ? S_STAGE : 1];
    static_assert(!LONG || (!DEEPB && TM == GA), "long rings: squares of 128");
    auto deep = [&](auto U) -> bf16_t* {
      if constexpr (decltype(U)::value == 0) return ld0;
      else if constexpr (decltype(U)::value == 1) return ld1;
      else if constexpr (decltype(U)::value == 2) return ld2;
      else if constexpr (decltype(U)::value == 3) return ld3;
      else return ld4;
    };
    auto shal = [&](auto U) -> bf16_t* {
      if constexpr (decltype(U)::value == 0) return ls0;
      else if constexpr (decltype(U)::value == 1) return ls1;
      else if constexpr (decltype(U)::value == 2) return ls2;
      else if constexpr (decltype(U)::value == 3) return ls3;
      else return ls4;
    };
    auto unit_a = [&](auto D, auto S) -> bf16_t* { if constexpr (DEEPB) return shal(S); else return deep(D); };
    auto unit_b = [&](auto D, auto S) -> bf16_t* { if constexpr (DEEPB) return deep(D); else return shal(S); };
    typedef __attribute__((address_space(3))) bf16_t* lds_wp;
    auto lds_addr = [](bf16_t* q) -> uint32_t { return (uint32_t)(uintptr_t)(lds_wp)q; };
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    // The descriptor of an operand's next slab.  The loop asks for every slab of an operand once and in order, so
    // a running base address and a count of the k still to come are enough: a handful of scalar operations per
    // slab and no branch (computing pair, offset and extent from the slab number took twice as many, with
    // branches, in one burst between two quarters that the matrix pipes spent waiting).  When the count runs out
    // the walk moves on to the second operand pair, if there is one, and then to empty extents (the dummy slabs).
    // A K-major operand can be walked when every slab is whole; one with ragged K keeps the per-slab form
    // because its loads need k0 and K for their per-lane test.
    constexpr bool WALK_A = KWHOLE || AMM, WALK_B = KWHOLE || BNM;
    // the block's slabs start in the first operand pair, or (a later part of a split tile) in the second
    const bool in2 = kt_lo >= nk1 && nkp2 > 0;
    const int k_first = (in2 ? kt_lo - nk1 : kt_lo) * BK, k_last = kt_lo + nk;
    const int rem0 = in2 ? min(p.K2, (k_last - nk1) * BK) - k_first : min(p.K, k_last * BK) - k_first;
    const bf16_t* a_first = in2 ? a_tile1 : a_tile0;
    const bf16_t* b_first = in2 ? b_tile1 : b_tile0;
    uint64_t a_base = (uint64_t)(a_first + (AMM ? (size_t)k_first * p.lda : (size_t)k_first));
    uint64_t b_base = (uint64_t)(b_first + (BNM ? (size_t)k_first * p.ldb : (size_t)k_first));
    uint64_t a_next = (uint64_t)a_tile1, b_next = (uint64_t)b_tile1;
    int a_rem = rem0, b_rem = rem0;
    int a_nrem = !in2 && k_last > nk1 ? min(p.K2, (k_last - nk1) * BK) : 0, b_nrem = a_nrem;
    const uint32_t a_step = AMM ? (uint32_t)(2 * BK) * (uint32_t)p.lda : (uint32_t)(2 * BK);
    const uint32_t b_step = BNM ? (uint32_t)(2 * BK) * (uint32_t)p.ldb : (uint32_t)(2 * BK);
    // extent of a live slab: row-major over K: (rows of the slab - 1) * ld + columns left; K-major: (tile rows - 1) * ld + k left
    const uint32_t a_ext0 = AMM ? (uint32_t)(2 * (p.M - m0)) : (uint32_t)(2 * (a_rows - 1)) * (uint32_t)p.lda;
    const uint32_t b_ext0 = BNM ? (uint32_t)(2 * (p.N - n0)) : (uint32_t)(2 * (b_rows - 1)) * (uint32_t)p.ldb;
    auto walk = [&](auto RM, uint64_t& base, uint64_t& next, int& rem, int& nrem, uint32_t step, uint32_t ext0, int ld) {
      i32x4_t rs;
      const uint32_t bytes = decltype(RM)::value ? ext0 + (uint32_t)(min(rem, BK) - 1) * (uint32_t)(2 * ld) : ext0 + (uint32_t)(2 * rem);
      rs[0] = (int)(uint32_t)base; rs[1] = (int)((uint32_t)(base >> 32) & 0xffffu); rs[2] = rem > 0 ? (int)bytes : 0; rs[3] = 0x00020000;
      base += step;
      rem -= BK;
      const bool over = rem <= 0;
      base = over ? next : base;
      rem = over ? nrem : rem;
      nrem = over ? 0 : nrem;
      return rs;
    };
    auto desc_a = [&](int kt) {
      typename OpA::SlabDesc d;
      if constexpr (WALK_A) {
        d.k0 = 0; d.Kc = 0;
        d.rs = walk(std::bool_constant<AMM>{}, a_base, a_next, a_rem, a_nrem, a_step, a_ext0, p.lda);
      } else {
        int pr, k0, Kc;
        slab(kt, pr, k0, Kc);
        d = OpA::slab_desc(pr ? a_tile1 : a_tile0, p.lda, a_rows, k0, Kc);
      }
      return d;
    };
    auto desc_b = [&](int kt) {
      typename OpB::SlabDesc d;
      if constexpr (WALK_B) {
        d.k0 = 0; d.Kc = 0;
        d.rs = walk(std::bool_constant<BNM>{}, b_base, b_next, b_rem, b_nrem, b_step, b_ext0, p.ldb);
      } else {
        int pr, k0, Kc;
        slab(kt, pr, k0, Kc);
        d = OpB::slab_desc(pr ? b_tile1 : b_tile0, p.ldb, b_rows, k0, Kc);
      }
      return d;
    };
    auto dma_a = [&](auto I, const typename OpA::SlabDesc& d, bf16_t* unit) {
      if constexpr (WALK_A) OpA::template chunk_whole<decltype(I)::value>(d, lds_addr(unit), a_off, wave_s);
      else OpA::template chunk<decltype(I)::value>(d, lds_addr(unit), a_off, a_piece, wave_s);
    };
    auto dma_b = [&](auto I, const typename OpB::SlabDesc& d, bf16_t* unit) {
      if constexpr (WALK_B) OpB::template chunk_whole<decltype(I)::value>(d, lds_addr(unit), b_off, wave_s);
      else OpB::template chunk<decltype(I)::value>(d, lds_addr(unit), b_off, b_piece, wave_s);
    };
    constexpr int NDEEP = DEEPB ? NVB : NVA, NSHAL = DEEPB ? NVA : NVB;
    static_assert(GA + TN + NDEEP <= GA * TN && GA + TN + NSHAL <= GA * TN, "a quarter has a slot for every read and load it carries");
    auto desc_deep = [&](int kt) { if constexpr (DEEPB) return desc_b(kt); else return desc_a(kt); };
    auto desc_shal = [&](int kt) { if constexpr (DEEPB) return desc_a(kt); else return desc_b(kt); };
    auto dma_deep = [&](auto I, const auto& d, bf16_t* unit) { if constexpr (DEEPB) dma_b(I, d, unit); else dma_a(I, d, unit); };
    auto dma_shal = [&](auto I, const auto& d, bf16_t* unit) { if constexpr (DEEPB) dma_a(I, d, unit); else dma_b(I, d, unit); };
    auto all_deep = [&](bf16_t* unit, int kt) {
      const auto d = desc_deep(kt);
      [&]<int... I>(std::integer_sequence<int, I...>) { (dma_deep(Int<I>{}, d, unit), ...); }(std::make_integer_sequence<int, NDEEP>{});
    };
    auto all_shal = [&](bf16_t* unit, int kt) {
      const auto d = desc_shal(kt);
      [&]<int... I>(std::integer_sequence<int, I...>) { (dma_shal(Int<I>{}, d, unit), ...); }(std::make_integer_sequence<int, NSHAL>{});
    };
    // one fragment of A (index F of group G) / of B (index F) of the k32 step h of a unit
    auto frag_a = [&](const bf16_t* unit, int h, auto G, auto F, u32x4_t (&fa)[GA]) {
      u32x4_t t[1];
      OpA::template frags16<decltype(G)::value * GA + decltype(F)::value, 1>((lds_bf_t)unit, h, a_ro, t);
      fa[decltype(F)::value] = t[0];
    };
    auto frag_b = [&](const bf16_t* unit, int h, auto F, u32x4_t (&fb)[TN]) {
      u32x4_t t[1];
      OpB::template frags16<decltype(F)::value, 1>((lds_bf_t)unit, h, b_ro, t);
      fb[decltype(F)::value] = t[0];
    };
    // One quarter, instruction by instruction: MFMA X of A group G, then whatever `after(Int<X>)` issues (operand
    // reads of a later quarter, DMA loads); the order is pinned.
    auto quarter = [&](auto G, u32x4_t (&fa)[GA], u32x4_t (&fb)[TN], auto&& after) {
      constexpr int g0 = decltype(G)::value * GA;
      [&]<int... X>(std::integer_sequence<int, X...>) {
        ([&] {
          constexpr int i = X / TN, j = X % TN;
          acc[g0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[j]),
                                                                   __builtin_bit_cast(bf16x8_t, fa[i]), acc[g0 + i][j], 0, 0, 0);
          after(Int<X>{});
          __builtin_amdgcn_sched_barrier(0);
        }(), ...);
      }(std::make_integer_sequence<int, NMF>{});
    };

    if constexpr (LONG) {
      // ---- five units for either operand: slab kt lives in unit kt % 5.  A's next slab (kt + 4) is requested in the first part of
      // slab kt, B's (kt + 5) in the second, into the units that slabs kt - 1 and kt have left at their barriers: four slabs ahead.
      constexpr int NL = NVA + NVB;
      all_shal(ls0, 0); all_deep(ld0, 0);
      all_shal(ls1, 1); all_deep(ld1, 1);
      all_shal(ls2, 2); all_deep(ld2, 2);
      all_shal(ls3, 3); all_deep(ld3, 3);
      all_shal(ls4, 4);
      TIDE_WAIT_VMCNT(3 * NL + NVB);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      frags_a(ld0, 0, Int<0>{}, fa0);
      frags_b(ls0, 0, fb0);
      __builtin_amdgcn_sched_barrier(0);
      auto step = [&](auto U, int kt) {
        constexpr int u = decltype(U)::value;
        const auto da = desc_deep(kt + 4);
        quarter(Int<0>{}, fa0, fb0, [&](auto X) {
          constexpr int x = decltype(X)::value;
          if constexpr (x < GA) frag_a(deep(U), 1, Int<0>{}, X, fa1);
          else if constexpr (x < GA + TN) frag_b(shal(U), 1, Int<x - GA>{}, fb1);
          else if constexpr (x < GA + TN + NVA) dma_deep(Int<x - GA - TN>{}, da, deep(Int<(u + 4) % 5>{}));
        });
        // the wave's operand reads have returned, and its loads of the next slab have landed: those of the three after it may be in flight
        __builtin_amdgcn_s_waitcnt(((3 * NL) & 15) | (((3 * NL) >> 4) << 14));   // vmcnt, lgkmcnt(0), expcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const auto db = desc_shal(kt + 5);
        quarter(Int<0>{}, fa1, fb1, [&](auto X) {
          constexpr int x = decltype(X)::value;
          if constexpr (x < GA) frag_a(deep(Int<(u + 1) % 5>{}), 0, Int<0>{}, X, fa0);
          else if constexpr (x < GA + TN) frag_b(shal(Int<(u + 1) % 5>{}), 0, Int<x - GA>{}, fb0);
          else if constexpr (x < GA + TN + NVB) dma_shal(Int<x - GA - TN>{}, db, shal(U));
        });
      };
      for (int kt = 0; kt < nk; kt += 5) {
        step(Int<0>{}, kt);
        if (__builtin_expect(kt + 1 < nk, 1)) step(Int<1>{}, kt + 1);
        if (__builtin_expect(kt + 2 < nk, 1)) step(Int<2>{}, kt + 2);
        if (__builtin_expect(kt + 3 < nk, 1)) step(Int<3>{}, kt + 3);
        if (__builtin_expect(kt + 4 < nk, 1)) step(Int<4>{}, kt + 4);
      }
    } else {
    all_deep(ld0, 0);
    all_shal(ls0, 0);
    TIDE_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    frags_a(unit_a(Int<0>{}, Int<0>{}), 0, Int<0>{}, fa0);
    frags_b(unit_b(Int<0>{}, Int<0>{}), 0, fb0);
    all_deep(ld1, 1);
    all_shal(ls1, 1);
    __builtin_amdgcn_sched_barrier(0);
    // (below eight tile rows per wave a slab is two parts, one per k32 step, with the barrier between them, and each part
    // begins with its loads: they have to land within a slab, which is short here.  With the loads after the operand reads and
    // the larger operand in the two units, a slab of 160 x 256 took 1.04 us where it takes 0.92 so, one of 128 x 256 0.85 / 0.74 at
    // 256 busy CUs, and NT 8193 x 1024 x 32000 620 / 454 us on 192 / 160 rows.  Loads that test every lane against a ragged K would
    // hold up the reads: they go behind the reads of A.  Us, loads last / first / so, at most 128 blocks of 128 x 128: NT 2165 x 256 x 688
    // 8.8 / 9.1 / 8.8, NN 176 x 4096 x 688 8.4 / 8.7 / 8.5; 200 blocks: NN 36 x 25600 x 688 10.2 / 9.7 / 9.9.)
    // One slab: deep unit D, shallow unit S (fa0 / fb0 hold its first quarter's operands); the next slab's units
    // are DN, SN; DP is the deep unit the slab before vacated.
    auto step = [&](auto D, auto S, auto DN, auto SN, auto DP, int kt) {
      const bf16_t* ua = unit_a(D, S);
      const bf16_t* ubb = unit_b(D, S);
      if constexpr (TM == GA) {
        constexpr int READS_AHEAD = WALK_A && WALK_B ? 0 : GA;
        const auto dd1 = desc_deep(kt + 2);
        quarter(Int<0>{}, fa0, fb0, [&](auto X) {
          constexpr int x = decltype(X)::value;
          constexpr int z = x - READS_AHEAD, y = z < 0 ? x : x - NDEEP;
          if constexpr (z >= 0 && z < NDEEP) dma_deep(Int<z>{}, dd1, deep(DP));
          else if constexpr (y < GA) frag_a(ua, 1, Int<0>{}, Int<y>{}, fa1);
          else if constexpr (y < GA + TN) frag_b(ubb, 1, Int<y - GA>{}, fb1);
        });
        __builtin_amdgcn_s_waitcnt((NDEEP & 15) | ((NDEEP >> 4) << 14));   // as below
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const bf16_t* uan = unit_a(DN, SN);
        const bf16_t* ubn = unit_b(DN, SN);
        const auto ds = desc_shal(kt + 2);
        quarter(Int<0>{}, fa1, fb1, [&](auto X) {
          constexpr int x = decltype(X)::value;
          constexpr int z = x - READS_AHEAD, y = z < 0 ? x : x - NSHAL;
          if constexpr (z >= 0 && z < NSHAL) dma_shal(Int<z>{}, ds, shal(S));
          else if constexpr (y < GA) frag_a(uan, 0, Int<0>{}, Int<y>{}, fa0);
          else if constexpr (y < GA + TN) frag_b(ubn, 0, Int<y - GA>{}, fb0);
        });
        return;
      } else {
      quarter(Int<0>{}, fa0, fb0, [&](auto X) {
        if constexpr (decltype(X)::value < GA) frag_a(ua, 0, Int<1>{}, X, fa1);
      });
      const auto dd1 = desc_deep(kt + 2);
      quarter(Int<1>{}, fa1, fb0, [&](auto X) {
        constexpr int x = decltype(X)::value;
        if constexpr (x < GA) frag_a(ua, 1, Int<0>{}, X, fa0);
        else if constexpr (x < GA + TN) frag_b(ubb, 1, Int<x - GA>{}, fb1);
        else if constexpr (x < GA + TN + NDEEP) dma_deep(Int<x - GA - TN>{}, dd1, deep(DP));
      });
      quarter(Int<0>{}, fa0, fb1, [&](auto X) {
        if constexpr (decltype(X)::value < GA) frag_a(ua, 1, Int<1>{}, X, fa1);
      });
      // every operand read of this wave from the slab's units has returned; its share of the next slab (and of
      // everything older) has landed; only its youngest deep-operand loads may still be in flight
      __builtin_amdgcn_s_waitcnt((NDEEP & 15) | ((NDEEP >> 4) << 14));   // vmcnt(NDEEP), lgkmcnt(0), expcnt(0)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      const bf16_t* uan = unit_a(DN, SN);
      const bf16_t* ubn = unit_b(DN, SN);
      const auto ds = desc_shal(kt + 2);
      quarter(Int<1>{}, fa1, fb1, [&](auto X) {
        constexpr int x = decltype(X)::value;
        if constexpr (x < GA) frag_a(uan, 0, Int<0>{}, X, fa0);
        else if constexpr (x < GA + TN) frag_b(ubn, 0, Int<x - GA>{}, fb0);
        // the shallow operand's loads follow the A reads (K-major B) or all eight reads (row-major B): measured,
        // 0.2-0.9 % per layout against issuing them beside the first reads
        constexpr int s0 = BNM ? GA + TN : GA;
        if constexpr (x >= s0 && x < s0 + NSHAL) dma_shal(Int<x - s0>{}, ds, shal(S));
      });
      }
    };
    // The unit numbers repeat every six slabs.  The last round skips the slabs past nk one by one (a chain of
    // uniform branches with the single loop exit at the bottom: early exits out of the middle made the compiler
    // spill the accumulators).
    for (int kt = 0; kt < nk; kt += 6) {
      step(Int<0>{}, Int<0>{}, Int<1>{}, Int<1>{}, Int<2>{}, kt);
      if (__builtin_expect(kt + 1 < nk, 1)) step(Int<1>{}, Int<1>{}, Int<2>{}, Int<0>{}, Int<0>{}, kt + 1);
      if (__builtin_expect(kt + 2 < nk, 1)) step(Int<2>{}, Int<0>{}, Int<0>{}, Int<1>{}, Int<1>{}, kt + 2);
      if (__builtin_expect(kt + 3 < nk, 1)) step(Int<0>{}, Int<1>{}, Int<1>{}, Int<0>{}, Int<2>{}, kt + 3);
      if (__builtin_expect(kt + 4 < nk, 1)) step(Int<1>{}, Int<0>{}, Int<2>{}, Int<1>{}, Int<0>{}, kt + 4);
      if (__builtin_expect(kt + 5 < nk, 1)) step(Int<2>{}, Int<1>{}, Int<0>{}, Int<0>{}, Int<1>{}, kt + 5);
    }
    }
    TIDE_WAIT_VMCNT(0);   // dummy slabs still in flight write LDS: let them land before the patches are written
    constexpr int PPU = D_STAGE / kPatchElems;   // epilogue patches per deep unit; a wave left over takes the first shallow one
    static_assert(PPU >= 1 && S_STAGE >= kPatchElems && NW <= 3 * PPU + 1, "the epilogue patches fit four units");
    const int pu = wave / PPU;
    bf16_t* unit = pu == 0 ? ld0 : (pu == 1 ? ld1 : (pu == 2 ? ld2 : ls0));
    epilogue(unit + (wave % PPU) * kPatchElems);
  }
}

template <int BM, int BN, bool AMM, bool BNM, typename TO, bool KWHOLE, bool ADAM = false>
__global__ __launch_bounds__(2 * BN) void gemm_mfma_kernel(std::conditional_t<ADAM, MfmaAdamParams, MfmaParams> p) {
  gemm_block<BM, BN, AMM, BNM, TO, KWHOLE, ADAM>(p, blockIdx.x);
}
// squares of 128, one block on a CU (see few_blocks)
template <bool AMM, bool BNM, typename TO, bool KWHOLE>
__global__ __launch_bounds__(256) void gemm_mfma_few_kernel(MfmaParams p) {
  gemm_block<128, 128, AMM, BNM, TO, KWHOLE, false, true>(p, blockIdx.x);
}

// The weight gradients of a layer with their updates, product after product over the blocks of one launch.  A product of few rows is
// bound by its weight's 30 bytes per element, and with a launch each its first tiles all multiply while the memory waits, its last ones update
// while the matrix pipes wait, and partly filled rounds come on top.  Six weights of 0.06 G elements together, us, a launch each / one: over 132
// rows 429 / 341 (5.3 TB/s of state), over 4096 681 / 612; of 0.27 G elements over 1999 rows 2115 / 1864.
struct MfmaAdamGroup { MfmaAdamParams p[kMaxGemmGroup]; int first[kMaxGemmGroup + 1]; int n; };   // first block of each, a multiple of 8 (XCDs)
template <int BM, int BN>
__global__ __launch_bounds__(2 * BN) void gemm_mfma_adam_group_kernel(MfmaAdamGroup g) {
  int i = 0;
#pragma unroll
  for (int k = 1; k < kMaxGemmGroup; ++k)
    if (k < g.n && (int)blockIdx.x >= g.first[k]) i = k;
  gemm_block<BM, BN, true, true, float, false, true>(g.p[i], blockIdx.x - g.first[i]);
}

// C[tile] += the partial sums of the later parts of every split tile, in the order of the parts (deterministic).
// Eight blocks per split tile (32 rows each); 256 threads, a thread adds 4 consecutive columns of 4 rows at a
// time, with the old values and every part's addends of those rows requested before the first sum.
template <bool ADAM>
__global__ __launch_bounds__(256) void splitk_fixup_kernel(AdamTarget adam, float* __restrict__ C, int ldc, int M, int N, int tiles_n,
                                                           int split_full, int split_s, const float* __restrict__ scratch) {
  const int tiles_m = (M + 255) / 256;
  const int ntail = tiles_m * tiles_n - split_full;
  const int tile = blockIdx.x >> 3, rblk = blockIdx.x & 7;
  int tile_m, tile_n;
  tile_coords(split_full + tile, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * 256, n0 = tile_n * 256;
  const int c4 = (threadIdx.x & 63) * 4, r0 = rblk * 32 + (threadIdx.x >> 6);
  const int gn = n0 + c4;
  if (gn >= N) return;
  AdamRate rate;
  if constexpr (ADAM) rate = adam_rate(adam);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    float4 v[4], am[4], av[4], ath[4];
    bool ok[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + (half * 4 + i) * 4;
      ok[i] = m0 + r < M;
      v[i] = ok[i] ? *reinterpret_cast<const float4*>(C + (size_t)(m0 + r) * ldc + gn) : make_float4(0.f, 0.f, 0.f, 0.f);
      if constexpr (ADAM) {
        if (ok[i]) {
          const size_t at = (size_t)(m0 + r) * ldc + gn;
          am[i] = load_once(adam.m + at);
          av[i] = load_once(adam.v + at);
          ath[i] = load_once(adam.master + at);
        }
      }
    }
    for (int j = 1; j < split_s; ++j) {
      float4 x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = r0 + (half * 4 + i) * 4;
        x[i] = *reinterpret_cast<const float4*>(scratch + ((size_t)(j - 1) * ntail + tile) * 65536 + (size_t)r * 256 + c4);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) { v[i].x += x[i].x; v[i].y += x[i].y; v[i].z += x[i].z; v[i].w += x[i].w; }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + (half * 4 + i) * 4;
      if (!ok[i]) continue;
      if constexpr (ADAM) adam_store(adam, rate, C, (size_t)(m0 + r) * ldc + gn, v[i], am[i], av[i], ath[i]);
      else *reinterpret_cast<float4*>(C + (size_t)(m0 + r) * ldc + gn) = v[i];
    }
  }
}

// C[tile] = alpha * (the partial sums of a tile's parts, in their order) + residual + old value.  A launch that came out
// as one part per tile has written C itself.  A block covers 2048 elements of a tile; a thread owns 8 consecutive columns.
template <typename TO, int BT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(MfmaParams p) {
  constexpr int PER_ROW = BT / 8, ROWS = 256 / PER_ROW, BLOCKS = BT / ROWS;
  if (p.m_dev) p.M = max(0, min(p.M, *p.m_dev - p.m_off));
  if (p.k_dev) p.K = max(0, min(p.K, *p.k_dev - p.k_off));
  const int tiles_m = (p.M + BT - 1) / BT, tiles = tiles_m * p.tiles_n;
  const SplitAll sa = split_all<BT>(tiles, split_slabs(p.K, p.A2 ? p.K2 : 0));
  const int tail = blockIdx.x / BLOCKS, ntail = tiles - sa.full;
  if (tail >= ntail) return;
  int tile_m, tile_n;
  tile_coords(sa.full + tail, tiles_m, p.tiles_n, tile_m, tile_n);
  const int row = (blockIdx.x % BLOCKS) * ROWS + threadIdx.x / PER_ROW, col = (threadIdx.x % PER_ROW) * 8;
  const int gm = tile_m * BT + row, gn = tile_n * BT + col;
  if (gm >= p.M || gn >= p.N) return;
  const float* src = p.split_scratch + (size_t)tail * (BT * BT) + row * BT + col;
  const size_t stride = (size_t)ntail * (BT * BT);
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < sa.parts; j += 4) {        // four parts' loads in flight at a time
    Raw8<float> x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u].zero();
      if (j + u < sa.parts) x[u].load(src, (size_t)(j + u) * stride);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float y[8];
      x[u].get(y);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += y[e];
    }
  }
  float alpha = p.alpha;
  if (p.alpha_dev) alpha *= *p.alpha_dev;
  TO* C = (TO*)p.C + (size_t)gm * p.ldc + gn;
  float r[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, old[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (p.R) ld8((const TO*)p.R, (size_t)gm * p.ldr + gn, r);
  if (p.accumulate) ld8(C, 0, old);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = alpha * v[e] + r[e] + old[e];
  st8(C, 0, v);
}

namespace {
// How the last round of a 256 x 256-tile launch is split over K: fp32 results without residual on tiles that do
// not fill the last round of the 256 CUs (at most half of it: otherwise two parts per tile would not fit the round).
struct SplitPlan { int s, full; size_t bytes; };
SplitPlan plan_split(const GemmArgs& a) {
  SplitPlan sp{1, 0, 0};
#ifdef TIDE_NO_SPLITK
  return sp;
#endif
  if (a.out_dtype != kF32 || a.residual || a.A2 || a.m_dev) return sp;
  if ((a.ldc % 4) || (a.N % 4) || (((uintptr_t)a.C) & 15)) return sp;
  const int64_t tiles = ((a.M + 255) / 256) * ((a.N + 255) / 256);
  if (tiles < 200) return sp;
  const int rem = (int)(tiles % 256);
  if (rem == 0 || rem > 128) return sp;
  const int64_t slabs = (a.K + 31) / 32;
  int s = 256 / rem;
  if (s > 8) s = 8;
  while (s > 1 && slabs / s < 32) --s;       // a part keeps at least 32 slabs (1024 k): below that its fixed cost dominates
  if (s <= 1) return sp;
  sp.s = s; sp.full = (int)(tiles - rem);
  sp.bytes = (size_t)(s - 1) * (size_t)rem * 65536 * sizeof(float);
  return sp;
}
}  // namespace

namespace {

// the reduction moves 8 columns at a time
bool split_possible(const GemmArgs& a) {
  return a.N % 8 == 0 && a.ldc % 8 == 0 && !((uintptr_t)a.C & 15) && !(a.residual && (a.ldr % 8 || ((uintptr_t)a.residual & 15)));
}

// Rows a launch whose number of rows is on the device alone is planned for: 85 % of the upper bound, the share of a batch
// that carries loss when prompts are 15 % of it (60 % in padded batches, 90 to 100 % in packed ones).  The kernels take
// the true number.  With 1 to 100 % of the rows no step or evaluation was slower than unsplit (8 x 512 and 2 x 200 bf16 steps,
// 1.08 to 1.5 times as fast; 3 x 1333 and 8 x 1024 evaluations, 0.99 to 1.08).
int64_t planned_rows(const GemmArgs& a) { return a.m_dev ? (a.M * 17 + 19) / 20 : a.M; }
int64_t tile_count(int64_t M, int64_t N, int e) { return ((M + e - 1) / e) * ((N + e - 1) / e); }

// Which tile a launch takes: 256 x 256 from 200 of them on; below that the cheaper one by the costs above, with or
// without a split, the small one in doubt.  With t tiles of 128 x 128 the chip runs rounds of 512 at the rate of two per
// CU (950 ns per slab) and the rest at that of one (580) up to 256, in between (800) up to 400.  Both operands row-major
// over K (TN) cost two LDS reads per fragment: 1050 / 700 ns, and 1470 on a large tile.  us, small / large tile: NN 2560 x
// 2048 x 32000: 400 / 258 (80 tiles in three parts), NT 1999 x 4096 x 12288: 191 / 160 (two), NN 2560 x 2048 x 11264: 136 / 102 (three).
// These costs decide between the squares and their splits, and the sizes of scratch that callers keep follow from them; tall_height, with
// costs of its own, measured at the number of CUs that are busy, then weighs the outcome against whole tiles of every height.
int tile_edge(const GemmArgs& a) {
  if (tile_count(a.M, a.N, 256) >= 200) return 256;
  const int64_t rows = planned_rows(a), t256 = tile_count(rows, a.N, 256), t128 = tile_count(rows, a.N, 128);
  const int slabs = split_slabs((int)a.K, a.A2 ? (int)a.K2 : 0);
  const bool can = split_possible(a), tn = a.layout == kTN;
  const SplitCost c2 = split_cost(256), c1 = split_cost(128);   // time in ns
  const int n256 = can ? split_parts(256, (int)t256, slabs) : 1, n128 = can ? split_parts(128, (int)t128, slabs) : 1;
  const int64_t p256 = (slabs + n256 - 1) / n256, p128 = (slabs + n128 - 1) / n128, blocks = t128 * n128, rest = blocks % 512;
  const int64_t time256 = (tn ? 1470 : c2.slab) * p256 + (n256 > 1 ? c2.fixed + c2.traffic * t256 * n256 : a.out_dtype == kF32 ? 14000 : 7000);
  const int64_t alone = tn ? 700 : 580, shared = tn ? 1050 : 950;
  const int64_t time128 = p128 * (blocks / 512 * shared + (rest == 0 ? 0 : rest <= 256 ? alone : rest <= 400 ? (alone + shared) / 2 : shared)) +
                          (n128 > 1 ? c1.fixed + c1.traffic * blocks : 0) + 4000;
  return time256 * 20 < time128 * 19 ? 256 : 128;
}

// Grid and scratch of a kSplitAll launch on tiles of BT x BT (blocks 0: it is not split).  With sizes known on the device
// alone they are the most that any size up to the given ones asks for.
struct SplitGrid { int64_t blocks, tail; size_t bytes; };
SplitGrid plan_split_all(const GemmArgs& a, int BT) {
  SplitGrid sp{0, 0, 0};
  if (!split_possible(a)) return sp;
  const int64_t tm = (a.M + BT - 1) / BT, tn = (a.N + BT - 1) / BT;
  // (a launch of many rounds has little to gain from its last one)
  if (BT == 256 && tm * tn > 4 * 256) return sp;
  const int slabs = split_slabs((int)a.K, a.A2 ? (int)a.K2 : 0);
  // with fewer slabs (a K known on the device alone) there are never more parts
  auto at = [&](int tiles) { return BT == 256 ? split_all<256>(tiles, slabs) : split_all<128>(tiles, slabs); };
  const int planned = (int)((planned_rows(a) + BT - 1) / BT * tn);
  const SplitAll sp0 = at(planned);
  if (sp0.parts < 2) return sp;
  if (a.m_dev) {
    // The number of rows may turn out to need no split, and the second launch then costs 5 us for nothing: only where the
    // split is planned to save twice what it costs (8 x 512 bf16 step, times as fast as one fixed older build: 1.101
    // where it was to save its cost once, 1.115 and 1.118 so; 3 x 1333 evaluation of the 8B-shaped draft 1.018, 1.020).
    const SplitCost c = split_cost(BT);
    const int64_t saved = (int64_t)c.slab * (slabs - (slabs + sp0.parts - 1) / sp0.parts);
    if (saved < 2 * (c.fixed + (int64_t)c.traffic * (planned - sp0.full) * sp0.parts)) return sp;
  }
  int64_t parts = 0, most = tm * tn;
  for (int64_t t = a.m_dev ? 1 : tm; t <= tm; ++t) {
    const int tiles = (int)(t * tn);
    if (BT == 128 && tiles > split_cost(128).slots / 2) break;   // no room for a second part from here on
    const SplitAll sa = at(tiles);
    if (sa.parts < 2) continue;
    const int64_t tail = tiles - sa.full, n = tail * sa.parts;
    if (n > parts) parts = n;
    if (tail > sp.tail) sp.tail = tail;
    if (sa.full + n > most) most = sa.full + n;
  }
  if (parts == 0) return sp;
  sp.bytes = (size_t)parts * BT * BT * sizeof(float);
  sp.blocks = most;
  return sp;
}
}  // namespace

// Tiles of edge BT that hold partial sums (a tile's parts times the tiles), at most, of a launch of up to `tiles` tiles and
// `slabs` slabs: split_parts gives n parts to t tiles only with t n <= slots, n <= slabs / min_slabs, traffic t n^2 <= slab
// slabs (so that t n <= sqrt(slab slabs t / traffic)) and where the slabs saved are worth the fixed costs.
static int64_t split_tiles_bound(int BT, int64_t tiles, int slabs) {
  const SplitCost c = split_cost(BT);
  const int64_t by_k = slabs / c.min_slabs, t = std::min<int64_t>(tiles, c.slots / 2), work = (int64_t)c.slab * slabs;
  if (by_k < 2 || work <= c.fixed) return 0;
  int64_t root = (int64_t)std::sqrt((double)(work * t / c.traffic));
  while ((root + 1) * (root + 1) <= work * t / c.traffic) ++root;
  while (root * root > work * t / c.traffic) --root;
  return std::min(std::min<int64_t>(c.slots, t * by_k), root);
}

size_t gemm_splitk_scratch_bound(const GemmArgs& a) {
  if (!gemm_mfma_supported(a)) return 0;
  size_t bytes = 0;
  const int slabs = split_slabs((int)a.K, a.A2 ? (int)a.K2 : 0);
  if (split_possible(a))
    for (const int BT : {128, 256})
      bytes = std::max(bytes, (size_t)split_tiles_bound(BT, tile_count(a.M, a.N, BT), slabs) * BT * BT * sizeof(float));
  if (a.layout == kTN) return std::max(bytes, plan_split(a).bytes);   // (the number of parts grows with K)
  if (a.out_dtype != kF32 || tile_count(a.M, a.N, 256) < 200) return bytes;
  const int s = (int)std::min<int64_t>(8, (a.K + 31) / 32 / 32);      // plan_split's parts: s - 1 sums of each of up to 256 / s tiles
  return s < 2 ? bytes : std::max(bytes, (size_t)(256 - 256 / s) * 65536 * sizeof(float));
}

namespace {
// What a launch does with the scratch it is given: the tile edge, and which split.
struct LaunchPlan { int BM, BN, split; SplitPlan tail; SplitGrid all; };

// Time (ns) of a launch of whole tiles, and of a planned split.  The chip's power is shared: a slab takes a tile longer the
// more CUs are busy.  Measured on r x c tiles, 64 to 288 of them, K = 1024 and 4096 (ns per slab with 256 CUs busy, change
// per CU in tenths, least, and what a tile takes beside its slabs; both operands row-major over K / others).
struct TileCost { int full, slope, least, fixed; };
TileCost tile_cost(int BM, bool tn) {
  switch (BM) {
    case 256: return tn ? TileCost{1391, 28, 1035, 13700} : TileCost{1344, 31, 945, 8500};
    case 224: return tn ? TileCost{1224, 24, 915, 14400} : TileCost{1213, 27, 860, 7800};
    case 192: return tn ? TileCost{1070, 22, 790, 12500} : TileCost{1074, 26, 740, 7200};
    case 160: return tn ? TileCost{951, 21, 675, 10600} : TileCost{902, 21, 635, 6900};
    default: return tn ? TileCost{770, 18, 535, 9500} : TileCost{736, 15, 540, 6500};
  }
}
int64_t rounds_time(int BM, bool tn, int64_t tiles, int64_t slabs, int64_t fed = 0) {   // fed: the least that a slab's operands take to arrive
  const TileCost c = tile_cost(BM, tn);
  const int64_t rounds = tiles / 256, rest = tiles % 256, last = std::max({(int64_t)c.least, c.full - c.slope * (256 - rest) / 10, fed});
  // behind full rounds a partly filled one has the memory for its float results nearly to itself (TN 14336 x 4096 x 915, 3.5 rounds: 131 us,
  // in four full ones of 224 rows 136)
  const int64_t fixed = tn && rounds ? c.fixed * (90 + rest * 166 / 256) / 256 : c.fixed;
  return rounds * (slabs * c.full + c.fixed) + (rest ? slabs * last + fixed : 0);
}
// 128 x 128: one block on a CU takes 465 to 550, two 870, and what a partly filled round adds to full ones is less
int64_t small_rounds_time(bool tn, int64_t blocks, int64_t slabs) {
  const int64_t rounds = blocks / 512, rest = blocks % 512;
  if (rounds == 0) {
    if (rest <= 256) return slabs * (465 + std::max<int64_t>(0, rest - 128) * 13 / 20) + (tn ? 5000 : 2500);
    return slabs * (700 + (rest - 320) * 9 / 10) + (tn ? 10000 : 7000);
  }
  return slabs * (rounds * 870 + (rest == 0 ? 0 : rest <= 128 ? 330 : rest <= 256 ? 430 : rest <= 384 ? 680 : 820)) + (tn ? 12000 : 8500);
}
int64_t launch_time(const GemmArgs& a, const LaunchPlan& lp, int64_t rows) {
  const bool tn = a.layout == kTN;
  const int64_t slabs = split_slabs((int)a.K, a.A2 ? (int)a.K2 : 0), tiles = ((rows + lp.BM - 1) / lp.BM) * ((a.N + lp.BN - 1) / lp.BN);
  if (lp.split == kSplitTail) {
    const int64_t tail = tiles - lp.tail.full, part = (slabs + lp.tail.s - 1) / lp.tail.s;
    return rounds_time(256, tn, lp.tail.full, slabs) + rounds_time(256, tn, tail * lp.tail.s, part) + 5000 + 40 * tail * lp.tail.s;
  }
  if (lp.BN == 256) {
    const SplitAll sa = lp.split == kSplitAll ? split_all<256>((int)tiles, (int)slabs) : SplitAll{(int)tiles, 1};
    const int64_t tail = tiles - sa.full, part = (slabs + sa.parts - 1) / sa.parts;
    // One row of tiles reads B once, from memory where it is larger than the 256 MB of the last cache.  A CU receives about 28 GB/s of
    // that, so that fewer than 168 do not reach the 4.7 TB/s of the chip (us, small tiles, split / 125 large ones: NT 39 x 32000 x 6144
    // 83 / 111, NN 157 x 32000 x 25600 355 / 438; small ones / 197 large ones: NT 127 x 50304 x 14336 334 / 308)
    const int64_t fed = rows <= lp.BM && tiles < 168 && 2 * a.N * slabs * 64 > 256000000 ? 1170 : 0;
    return rounds_time(lp.BM, tn, sa.full, slabs, fed) + (tail ? rounds_time(256, tn, tail * sa.parts, part) + 4000 + 40 * tail * sa.parts : 0);
  }
  const SplitAll sa = lp.split == kSplitAll ? split_all<128>((int)tiles, (int)slabs) : SplitAll{(int)tiles, 1};
  const int64_t blocks = sa.full + (tiles - sa.full) * sa.parts, part = (slabs + sa.parts - 1) / sa.parts;
  return small_rounds_time(tn, blocks, part) + (sa.parts > 1 ? 5000 + 16 * blocks : 0);
}

// Tiles of 128 to 224 x 256 where they fill the rounds of the 256 CUs better than the squares, and large tiles where the
// costs above, which allow for the power that idle CUs leave to the others, like them better than tile_edge did.  us, by
// tile_edge / so: NN 1665 x 5632 x 2048 47.8 / 35.0 (160 rows), NT 3400 x 14336 x 4096 332 / 290 (192), NT 4096 x 2048 x 6144 89 / 78
// (128), TN 5632 x 2048 x 2560 64.9 / 55.0 (192), NN 3125 x 5120 x 12288 445 / 302 (128); over 618 random products (200 to
// 12000 rows, 5 to 600 GFLOP) 6 % in the mean; of 44 TN products of 256 to 32000 columns whose split gave way the slowest takes 1.02 times
// as long.  With a row count known on the device alone a height has to pay over the
// range that batches have: the sum over 50, 55 .. 100 % of the bound (at 60, 85 and 100 % alone, a height can miss the round that
// the rows between just fill: evaluation of 8 x 512 rows, 2048 / 5632 wide, us before heights / so chosen / now, 62 % of the rows 731 / 771 /
// 718, 85 % 927 / 906 / 904, 100 % 1031 / 984 / 1000).
// (bf16 results added to old ones, which leave the kernel element by element, are as tile_edge has them)
bool tall_possible(const GemmArgs& a) {
  if (a.layout == kTN) return a.out_dtype == kF32;
  return a.out_dtype == kBF16 && !a.accumulate && a.K % 64 == 0 && (!a.A2 || a.K2 % 64 == 0) && !a.k_dev;
}
int tall_height(const GemmArgs& a, const LaunchPlan& lp) {
  if (!tall_possible(a)) return 0;
  auto total = [&](const LaunchPlan& l) {
    if (!a.m_dev) return launch_time(a, l, a.M);
    int64_t t = 0;
    for (int share = 10; share <= 20; ++share) t += launch_time(a, l, std::max<int64_t>(1, a.M * share / 20));
    return t;
  };
  // Only for a gain beyond the model's error, which is larger beside a split of the last round (us, split / so: TN 4096 x 5120 x
  // 4929 169 / 177 and 4096 x 5632 x 6231 226 / 229 on 192 rows, both 4 % cheaper by the model) and beside small tiles that are split (NT
  // 688 x 5120 x 5632 50.5 / 54.9 and 3887 x 1024 x 5632 53.2 / 55.4, 5 and 7 % cheaper).
  const int percent = lp.split == kSplitTail ? 85 : lp.split == kSplitAll && lp.BN == 128 ? 92 : 96;
  int64_t best = total(lp) * percent / 100;
  int height = 0;
  for (const int BM : {256, 224, 192, 160, 128}) {
    const int64_t t = total(LaunchPlan{BM, 256, kSplitNone, {1, 0, 0}, {0, 0, 0}});
    if (t < best) { best = t; height = BM; }
  }
  return height;
}

// With the weight's update behind it a product of few rows is bound by the weight's 30 bytes per element, and two small blocks on
// a CU overlap one's update with the other's products: us as planned otherwise / so, 128256 x 4096 over 300 rows 3090 / 2815, over
// 1400 3318 / 3212, over 2500 3898 / 4115; 14336 x 4096 over 1400 398 / 364; 4096 x 4096 over 700 116 / 111; 5632 x 2048 (704 blocks)
// over 700 83 / 86.  Otherwise tiles and split are those of the product alone: its costs have no term for the update.
bool update_bound(const GemmArgs& a) {
  const int64_t rows = a.k_dev ? (a.K * 17 + 19) / 20 : a.K;   // see planned_rows
  return rows <= 2048 && tile_count(a.M, a.N, 128) >= 1024;
}

LaunchPlan plan_launch(const GemmArgs& a, bool adam = false) {
  if (adam && update_bound(a)) return LaunchPlan{128, 128, kSplitNone, {1, 0, 0}, {0, 0, 0}};
  const int e = tile_edge(a);
  LaunchPlan lp{e, e, kSplitNone, plan_split(a), {0, 0, 0}};
  const bool scratch_ok = a.scratch && (((uintptr_t)a.scratch) & 15) == 0;
  if (lp.tail.s > 1) {
    if (scratch_ok && a.scratch_bytes >= lp.tail.bytes) lp.split = kSplitTail;
  } else {
    lp.all = plan_split_all(a, e);
    if (lp.all.blocks > 0 && scratch_ok && a.scratch_bytes >= lp.all.bytes) lp.split = kSplitAll;
    else if (lp.all.blocks > 0 && tile_count(a.M, a.N, 256) < 200) lp.BM = lp.BN = 128;   // chosen for its split: without scratch, too few large tiles to run them whole
  }
  if (const int BM = tall_height(a, lp)) { lp.BM = BM; lp.BN = 256; lp.split = kSplitNone; }
  return lp;
}
}  // namespace

size_t gemm_split_tail_bytes(const GemmArgs& a) { return gemm_mfma_supported(a) ? plan_split(a).bytes : 0; }
size_t gemm_splitk_scratch_bytes(const GemmArgs& a) {
  if (!gemm_mfma_supported(a)) return 0;
  const SplitPlan tail = plan_split(a);
  return tail.s > 1 ? tail.bytes : plan_split_all(a, tile_edge(a)).bytes;
}

bool gemm_mfma_supported(const GemmArgs& a) {
  if (a.in_dtype != kBF16) return false;
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return false;
  if (a.lda % 8 || a.ldb % 8) return false;
  // A K-major operand is read in 16-byte pieces along K.  With both operands row-major over K (TN) a k-row is either
  // loaded or, past K, lies outside the buffer and loads zeros, so any K will do: it is the number of rows of a batch
  // there, which need not be a multiple of anything (a packed batch, an odd sequence length).  On the shape-agnostic
  // kernel 4096 x 12288 x 3999 took 6.36 ms, on this one 0.33 ms (and 28 instead of 1.3 ms for a 128256-entry dW_lm).
  const bool any_k = a.layout == kTN;
  if (!any_k && a.K % 8) return false;
  if (a.A2 && (a.K2 <= 0 || (!any_k && a.K2 % 8) || !a.B2 || a.k_dev)) return false;
  if (((uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.A2 | (uintptr_t)a.B2) & 15) return false;
  // 32-bit byte offsets inside one tile
  const int64_t lim = (int64_t)1 << 21;
  if (a.lda >= lim || a.ldb >= lim || a.ldc >= lim) return false;
  if (a.M >= ((int64_t)1 << 24) || a.N >= ((int64_t)1 << 24) || a.K >= ((int64_t)1 << 24) || a.K2 >= ((int64_t)1 << 24)) return false;
  if (a.layout == kNN || a.layout == kTN) {
    if (a.N % 8) return false;  // B rows are read in 16-byte pieces along N
  }
  if (a.layout == kTN && a.M % 8) return false;
  return true;
}

namespace {

// every slab whole (and K known on the host): the DMA loads of a K-major operand take loop-constant lane offsets
bool whole_slabs(const MfmaParams& p) { return !p.k_dev && p.K % 64 == 0 && (!p.A2 || p.K2 % 64 == 0); }

// Squares of 128 that leave CUs idle have a CU's whole LDS to themselves: rings of five units per operand, four slabs ahead.  The weights
// of a step come from memory, and with the three and two units that fit twice into a CU a slab waits for them: us in a step, 3 + 2 units / 5 + 5,
// 132 blocks of 32 slabs 27.3 / 19.5, 96 27.5 / 18.7, 48 30.2 / 21.6; 192 blocks of 64 slabs, alone and repeated, 34.4 / 28.6.  Evaluation of 2 x 144
// rows, 2048 / 5632 wide, 247 / 214; steps of 132 to 1000 rows 0.6 to 2.3 % less.  Weights from memory / one product over and over in the caches: 258 x 1024 x 1024 15.3 -> 10.8
// / 9.0 -> 9.4, 384 x 4096 x 1536 21.4 -> 18.6 / 12.5 -> 12.9, 132 x 2048 x 2048 26.8 -> 16.9 / 14.0 -> 14.3, 96 x 1024 x 5632 67.9 -> 49.6 / 30.7 -> 30.4: what up to 24 slabs lose in the
// caches are the nine units of slabs past the last (last steps that request nothing, in a loop of their own, cost 1 us more at any depth, tests in the one loop 0.13 us per slab).  Not below 16 slabs, where filling the rings shows (8 slabs and fewer, 8.1 / 8.4 to
// 13.1 / 13.7), nor with nearly every CU busy (250 blocks of 32 slabs 23.3 / 24.1).  Nor split over K: the costs of a split give no part 16 slabs as long as its
// blocks are 224 or fewer, and one over a number of rows known on the device can have less than at the bound.
bool few_blocks(int split, int64_t tiles, int slabs) { return split == kSplitNone && tiles <= 224 && slabs >= 16; }

template <int BM, int BN, bool AMM, bool BNM, typename TO, typename P>
hipError_t launch_tiles(const P& p, const SplitGrid& all, hipStream_t s) {   // all: of a kSplitAll launch
  constexpr bool ADAM = std::is_same_v<P, MfmaAdamParams>;
  P q = p;
  q.tiles_m = (p.M + BM - 1) / BM;
  q.tiles_n = (p.N + BN - 1) / BN;
  const int tiles = q.tiles_m * q.tiles_n;
  const int64_t items = q.split == kSplitAll ? all.blocks
                      : q.split == kSplitTail ? q.split_full + (int64_t)(tiles - q.split_full) * q.split_s : tiles;
  if constexpr (BM == BN && !ADAM) {
    // (with both operands row-major over K the two forms are the same code: one instantiation)
    auto* kernel = gemm_mfma_kernel<BM, BN, AMM, BNM, TO, false>;
    if constexpr (!(AMM && BNM)) {
      if (whole_slabs(p)) kernel = gemm_mfma_kernel<BM, BN, AMM, BNM, TO, true>;
    }
    if constexpr (BM == 128) {
      if (few_blocks(q.split, tiles, split_slabs(p.K, p.A2 ? p.K2 : 0))) {
        kernel = gemm_mfma_few_kernel<AMM, BNM, TO, false>;
        if constexpr (!(AMM && BNM)) {
          if (whole_slabs(p)) kernel = gemm_mfma_few_kernel<AMM, BNM, TO, true>;
        }
      }
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)items), dim3(2 * BN), 0, s, q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || q.split != kSplitAll) return e;
    hipLaunchKernelGGL((splitk_reduce_kernel<TO, BM>), dim3((unsigned)(all.tail * (BM * BM / 2048))), dim3(256), 0, s, q);
  } else {
    hipLaunchKernelGGL((gemm_mfma_kernel<BM, BN, AMM, BNM, TO, !(AMM && BNM), ADAM>), dim3((unsigned)items), dim3(2 * BN), 0, s, q);
  }
  return hipGetLastError();
}

template <bool AMM, bool BNM, typename TO, typename P>
hipError_t launch_layout(const P& p, const LaunchPlan& lp, hipStream_t s) {
  if constexpr (sizeof(TO) == (AMM && BNM ? 4 : 2)) {
    if (lp.BN == 256) switch (lp.BM) {
      case 224: return launch_tiles<224, 256, AMM, BNM, TO>(p, lp.all, s);
      case 192: return launch_tiles<192, 256, AMM, BNM, TO>(p, lp.all, s);
      case 160: return launch_tiles<160, 256, AMM, BNM, TO>(p, lp.all, s);
      case 128: return launch_tiles<128, 256, AMM, BNM, TO>(p, lp.all, s);
    }
  }
  if (lp.BN == 256) return launch_tiles<256, 256, AMM, BNM, TO>(p, lp.all, s);
  return launch_tiles<128, 128, AMM, BNM, TO>(p, lp.all, s);
}

}  // namespace

const char* gemm_kernel_name(const GemmArgs& a) {
  if (!gemm_mfma_supported(a)) return a.in_dtype == kF32 && a.out_dtype == kF32 ? "gemm_fp32" : "gemm_simple";
  static const char* const square[3][2][2] = {{{"gemm_mfma_nt_128_bf16out", "gemm_mfma_nt_256_bf16out"}, {"gemm_mfma_nt_128_f32out", "gemm_mfma_nt_256_f32out"}},
                                              {{"gemm_mfma_nn_128_bf16out", "gemm_mfma_nn_256_bf16out"}, {"gemm_mfma_nn_128_f32out", "gemm_mfma_nn_256_f32out"}},
                                              {{"gemm_mfma_tn_128_bf16out", "gemm_mfma_tn_256_bf16out"}, {"gemm_mfma_tn_128_f32out", "gemm_mfma_tn_256_f32out"}}};
  static const char* const tall[3][4] = {{"gemm_mfma_nt_128x256_bf16out", "gemm_mfma_nt_160x256_bf16out", "gemm_mfma_nt_192x256_bf16out", "gemm_mfma_nt_224x256_bf16out"},
                                         {"gemm_mfma_nn_128x256_bf16out", "gemm_mfma_nn_160x256_bf16out", "gemm_mfma_nn_192x256_bf16out", "gemm_mfma_nn_224x256_bf16out"},
                                         {"gemm_mfma_tn_128x256_f32out", "gemm_mfma_tn_160x256_f32out", "gemm_mfma_tn_192x256_f32out", "gemm_mfma_tn_224x256_f32out"}};
  const LaunchPlan lp = plan_launch(a);
  return lp.BM == lp.BN ? square[a.layout][a.out_dtype == kF32][lp.BN == 256] : tall[a.layout][(lp.BM - 128) / 32];
}

bool gemm_long_rings(const GemmArgs& a) {
  if (!gemm_mfma_supported(a)) return false;
  const LaunchPlan lp = plan_launch(a);
  return lp.BN == 128 && few_blocks(lp.split, tile_count(a.M, a.N, 128), split_slabs((int)a.K, a.A2 ? (int)a.K2 : 0));
}

const char* gemm_adam_kernel_name(const GemmArgs& a) {
  static const char* const updating[6] = {"gemm_mfma_tn_128x256_adamw", "gemm_mfma_tn_160x256_adamw", "gemm_mfma_tn_192x256_adamw", "gemm_mfma_tn_224x256_adamw",
                                          "gemm_mfma_tn_256_adamw", "gemm_mfma_tn_128_adamw"};
  const LaunchPlan lp = plan_launch(a, true);
  return updating[lp.BN == 128 ? 5 : (lp.BM - 128) / 32];
}


namespace {
// algorithmic work of the call, for the optional profiler; fixed: the bytes of a weight's update, which do not depend on the rows that ran
struct GemmProf {
  ProfScope ps;
  GemmProf(const GemmArgs& a, double fixed, hipStream_t s) : ps(prof_enabled() ? (fixed > 0 ? gemm_adam_kernel_name(a) : gemm_kernel_name(a)) : "", flops(a), bytes(a) + fixed, s) {
    if (a.m_dev) prof_dynamic(a.m_dev, a.m_off, a.M, 0, fixed);
    else if (a.k_dev) prof_dynamic(a.k_dev, a.k_off, a.K, 0, fixed);
  }
  static double k_all(const GemmArgs& a) { return (double)a.K + (a.A2 ? (double)a.K2 : 0.0); }
  static double flops(const GemmArgs& a) { return 2.0 * (double)a.M * (double)a.N * k_all(a); }
  static double bytes(const GemmArgs& a) {
    return (double)dtype_size(a.in_dtype) * k_all(a) * ((double)a.M + (double)a.N) +
           (double)dtype_size(a.out_dtype) * (double)a.M * (double)a.N * (1.0 + (a.accumulate ? 1.0 : 0.0) + (a.residual ? 1.0 : 0.0));
  }
};
void fill_params(MfmaParams& p, const GemmArgs& a, const LaunchPlan& lp) {
  p.A = (const bf16_t*)a.A; p.B = (const bf16_t*)a.B;
  p.A2 = (const bf16_t*)a.A2; p.B2 = (const bf16_t*)a.B2;
  p.C = a.C; p.R = a.residual; p.alpha_dev = a.alpha_dev;
  p.M = (int)a.M; p.N = (int)a.N; p.K = (int)a.K; p.K2 = a.A2 ? (int)a.K2 : 0;
  p.lda = (int)a.lda; p.ldb = (int)a.ldb; p.ldc = (int)a.ldc; p.ldr = (int)a.ldr;
  p.alpha = a.alpha; p.accumulate = a.accumulate; p.tiles_m = p.tiles_n = 0;
  p.m_dev = a.m_dev; p.m_off = (int)a.m_off; p.k_dev = a.k_dev; p.k_off = (int)a.k_off;
  p.split = lp.split; p.split_s = lp.split == kSplitTail ? lp.tail.s : 1; p.split_full = lp.split == kSplitTail ? lp.tail.full : 0;
  p.split_scratch = lp.split != kSplitNone ? (float*)a.scratch : nullptr;
}
template <bool ADAM>
hipError_t launch_fixup(const MfmaParams& p, const AdamTarget& t, hipStream_t s) {
  const int tiles_n = (p.N + 255) / 256, ntail = ((p.M + 255) / 256) * tiles_n - p.split_full;
  hipLaunchKernelGGL(splitk_fixup_kernel<ADAM>, dim3((unsigned)ntail * 8u), dim3(256), 0, s, t, (float*)p.C, p.ldc, p.M, p.N, tiles_n,
                     p.split_full, p.split_s, p.split_scratch);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_gemm_mfma(const GemmArgs& a, hipStream_t s) {
  MfmaParams p;
  const LaunchPlan lp = plan_launch(a);
  fill_params(p, a, lp);
  const bool f32out = a.out_dtype == kF32;
  hipError_t e = hipErrorInvalidValue;
  switch (a.layout) {
    case kNT: e = f32out ? launch_layout<false, false, float>(p, lp, s) : launch_layout<false, false, bf16_t>(p, lp, s); break;
    case kNN: e = f32out ? launch_layout<false, true, float>(p, lp, s) : launch_layout<false, true, bf16_t>(p, lp, s); break;
    case kTN: e = f32out ? launch_layout<true, true, float>(p, lp, s) : launch_layout<true, true, bf16_t>(p, lp, s); break;
  }
  return e != hipSuccess || p.split != kSplitTail ? e : launch_fixup<false>(p, AdamTarget{}, s);
}

// (a product whose tiles are all split, which only one with scratch is, is left as it is: the update in the kernel that adds the parts took longer than
// the pass over the weight, 8000 rows of a 1280 / 3440 wide step 3736 us so, 3613 with the pass)
bool gemm_adam_supported(const GemmArgs& a, const AdamTarget& t) {
  return a.layout == kTN && a.out_dtype == kF32 && !a.residual && !a.A2 && gemm_mfma_supported(a) && a.N % 8 == 0 && a.ldc % 8 == 0 &&
         !(((uintptr_t)a.C | (uintptr_t)t.m | (uintptr_t)t.v | (uintptr_t)t.master | (uintptr_t)t.w) & 15) && plan_launch(a, true).split != kSplitAll;
}

// A tile's update takes its CU 8 to 12 us (128 x 128) with the rest of the chip idle or not; one pass over the weights left takes 5 us and
// 34 bytes per element.  Whole steps (us; no update in a product / in all / from half the CUs' worth of tiles on): width 256, 64 rows 228 /
// 289 / 227; width 512, 1000 rows 628 / 630 / 582; 768, 300 rows 631 / 598 / 555; 1024, 1000 rows 1011 / 911 / 907; 1536, 300 rows
// 1089 / 931 / 935.  With a bound of 4 M elements the last takes 965, with 1 M the one of width 768 takes 578.
bool gemm_adam_pays(const GemmArgs& a) { return tile_count(a.M, a.N, 128) > 128; }

hipError_t launch_gemm_adam(const GemmArgs& a, const AdamTarget& t, hipStream_t s) {
  if (!gemm_adam_supported(a, t)) return hipErrorInvalidValue;
  MfmaAdamParams p;
  const LaunchPlan lp = plan_launch(a, true);
  fill_params(p, a, lp);
  p.adam = t;
  // beside the product's own: the two moments and the master copy read and written, the weight written
  const GemmProf ps(a, 26.0 * (double)a.M * (double)a.N, s);
  const hipError_t e = launch_layout<true, true, float>(p, lp, s);
  return e != hipSuccess || p.split != kSplitTail ? e : launch_fixup<true>(p, t, s);
}

namespace {
template <int BM, int BN>
hipError_t launch_adam_group(MfmaAdamGroup& g, hipStream_t s) {
  g.first[0] = 0;
  for (int i = 0; i < g.n; ++i) {
    MfmaAdamParams& p = g.p[i];
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    g.first[i + 1] = g.first[i] + (p.tiles_m * p.tiles_n + 7) / 8 * 8;
  }
  hipLaunchKernelGGL((gemm_mfma_adam_group_kernel<BM, BN>), dim3((unsigned)g.first[g.n]), dim3(2 * BN), 0, s, g);
  return hipGetLastError();
}
}  // namespace

// Whole steps, us, a launch each / one on 160 x 256 / on 256 x 256 tiles (on 128 x 128 and 192 x 256 nowhere better than the best of these by more than
// the spread): 2048 / 5632 wide, 132 rows 1125 / 1070 / 1085, 700 1455 / 1380 / 1395, 1900 2087 / 1980 / 2010, 3000 2320 / 2249 / 2267, 6000 4320 /
// 4210 / 4165; 4096 / 14336 wide, 300 rows 5516 / 5451 / 5580, 1000 7466 / 7300 / 7395, 1999 10470 / 10226 / 10355, 3000 13517 / 13212 / 13180,
// 4200 20020 / 19900 / 19790, 8000 31130 / 31385 / 30970, 32768 102950 / 105100 / 103240: there a launch each finds an operand of the product
// before still in a cache.
bool gemm_adam_group_pays(int64_t rows) { return rows <= 8192; }

hipError_t launch_gemm_adam_group(const GemmArgs* a, const AdamTarget* t, int n, hipStream_t s) {
  if (n < 1 || n > kMaxGemmGroup) return hipErrorInvalidValue;
  MfmaAdamGroup g;
  g.n = n;
  int64_t rows = 0;
  double flops = 0, bytes = 0, fixed_flops = 0, fixed_bytes = 0;   // fixed: of products whose sizes are all known here, and of the updates
  const GemmArgs* dyn = nullptr;                                   // (the others of a step share one size on the device)
  for (int i = 0; i < n; ++i) {
    if (!gemm_adam_supported(a[i], t[i])) return hipErrorInvalidValue;
    fill_params(g.p[i], a[i], LaunchPlan{128, 128, kSplitNone, {1, 0, 0}, {0, 0, 0}});
    g.p[i].adam = t[i];
    rows = std::max(rows, a[i].K);
    const double update = 26.0 * (double)a[i].M * (double)a[i].N, f = GemmProf::flops(a[i]), b = GemmProf::bytes(a[i]);
    flops += f;
    bytes += b + update;
    fixed_bytes += update;
    if (a[i].k_dev) dyn = &a[i];
    else { fixed_flops += f; fixed_bytes += b; }
  }
  ProfScope ps("gemm_mfma_tn_group_adamw", flops, bytes, s);
  if (dyn) prof_dynamic(dyn->k_dev, dyn->k_off, dyn->K, fixed_flops, fixed_bytes);
  return rows <= 4096 ? launch_adam_group<160, 256>(g, s) : launch_adam_group<256, 256>(g, s);
}

hipError_t launch_gemm(const GemmArgs& a, hipStream_t s) {
  const GemmProf ps(a, 0, s);
  if (gemm_mfma_supported(a)) return launch_gemm_mfma(a, s);
  return a.in_dtype == kF32 && a.out_dtype == kF32 ? launch_gemm_fp32(a, s) : launch_gemm_simple(a, s);
}

// ------------------------------------------------------------------------------------------------
// Pure-MFMA probe: what the matrix pipes deliver with nothing else going on (operands in registers, no
// LDS, no memory).  8 waves per block, 8 independent accumulators per wave.  The operands are random bf16 values
// (random sign and mantissa, magnitude in [0.5, 2)), a different pair for each of the 8 MFMAs: what the pipes draw
// depends on how many operand bits change from one instruction to the next, and under its package power limit the
// chip sustains 1.84 PFLOP/s on such operands against 2.45 PFLOP/s on constant ones.  Timed over a few hundred
// milliseconds, the rate is the practical ceiling for the GEMM above.
// ------------------------------------------------------------------------------------------------
namespace {
__device__ __forceinline__ uint32_t probe_hash(uint32_t x) {
  x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
  return x;
}
__device__ __forceinline__ uint32_t probe_pair(uint32_t seed) {   // two bf16 values with |x| in [0.5, 2)
  const uint32_t h = probe_hash(seed);
  const uint32_t lo = 0x3F00u | (h & 0x80FFu) | ((h >> 9) & 0x0080u);
  const uint32_t hi = 0x3F00u | ((h >> 16) & 0x80FFu) | ((h >> 3) & 0x0080u);
  return lo | (hi << 16);
}
}  // namespace

__global__ __launch_bounds__(512) void mfma_probe_kernel(float* __restrict__ sink, int iters) {
  const uint32_t tid = blockIdx.x * 512u + threadIdx.x;
  u32x4_t a[8], b[8];
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      a[j][w] = probe_pair(tid * 64u + j * 4 + w);
      b[j][w] = probe_pair(tid * 64u + 32 + j * 4 + w);
    }
  f32x16_t acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a[j]), __builtin_bit_cast(bf16x8_t, b[(j + 3) & 7]), acc[j], 0, 0, 0);
  }
  float v = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int q = 0; q < 16; ++q) v += acc[j][q];
  sink[(size_t)blockIdx.x * 512 + threadIdx.x] = v;
}

hipError_t launch_mfma_probe(int blocks, int iters, float* sink, hipStream_t s) {
  hipLaunchKernelGGL(mfma_probe_kernel, dim3((unsigned)blocks), dim3(512), 0, s, sink, iters);
  return hipGetLastError();
}

}  // namespace tide
