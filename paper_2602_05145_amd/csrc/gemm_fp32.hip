// fp32 GEMM for gfx950 on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: fp32 products, fp32 accumulation),
// any sizes, strides and layout.  It is the whole GEMM path of fp32 mode.
//
// What bounds it.  The fp32 matrix rate (157 TFLOP/s) is a sixteenth of the bf16 one, so a 128 x 128 tile needs only
// 8 bytes per clock and CU from L2 and 16 from LDS: plain double-buffered LDS staging through registers keeps the
// pipes busy, and neither LDS-DMA loads nor deeper rings have anything to win.  What matters is how many CUs work:
//   * tile kernel, 128 x 128 (four waves of 64 x 64), or 64 x 64 (four waves of 32 x 32) where the larger tile
//     leaves most of the 256 CUs without one;
//   * a result of less than about 200 tiles of 64 x 64 (the fp32 configuration's 128 rows) is bound by latency: walking
//     K = 4096 in 16-deep LDS slabs on 8 blocks took 769 us of barriers and load latency.  There one block computes
//     a 32 x 32 or 16 x 16 tile, its 4 or 16 waves split the contraction, load their fragments straight from L2 into
//     registers (no LDS, no barrier in the loop, 8 to 32 loads in flight per lane) and add their sums through LDS at
//     the end, in the order of the waves.
//
// Contraction order.  A 32x32x2 instruction takes k values {a, b} from the lower and the upper half of the wave
// (16x16x4: four, from its quarters).  The kernels feed it {8 s + i, 8 s + 4 + i} for i = 0..3: a lane's four values of a group of 8 k are consecutive,
// one 16-byte read of an operand whose contraction index is contiguous.
#include <type_traits>

#include "kernels.h"
#include "prof.h"
#include "tide_common.h"

namespace tide {

namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

struct Fp32GemmParams {
  const float* A; const float* B; const float* A2; const float* B2;
  float* C; const float* R; const float* alpha_dev;
  int64_t lda, ldb, ldc, ldr;
  int M, N, K, K2;
  float alpha;
  int accumulate;
  const int* m_dev; int64_t m_off;
  const int* k_dev; int64_t k_off;
  // SwiGLU's backward behind the product of dh (EXT instantiations): gt and u share C's layout and become dgate and dup
  float *gt, *u;
};

// sizes that are only known on the device (block-uniform)
__device__ __forceinline__ void device_sizes(Fp32GemmParams& p) {
  if (p.m_dev) p.M = (int)max((int64_t)0, min((int64_t)p.M, (int64_t)*p.m_dev - p.m_off));
  if (p.k_dev) p.K = (int)max((int64_t)0, min((int64_t)p.K, (int64_t)*p.k_dev - p.k_off));
}

// Four consecutive elements p[i .. i+3] of which `left` exist (the rest are zeros); VEC: p + i is 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ f32x4_t load4(const float* p, int64_t i, int left) {
  if (VEC && left >= 4) return *reinterpret_cast<const f32x4_t*>(p + i);
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
  if (left > 0) v.x = p[i];
  if (left > 1) v.y = p[i + 1];
  if (left > 2) v.z = p[i + 2];
  if (left > 3) v.w = p[i + 3];
  return v;
}

// gate and up of an element of dh, requested ahead of it: behind it they are one more latency at the end of the launch
__device__ __forceinline__ float2 load_behind(const Fp32GemmParams& p, int gm, int gn) {
  const size_t at = (size_t)gm * p.ldc + gn;
  return gm < p.M && gn < p.N ? make_float2(p.gt[at], p.u[at]) : make_float2(0.f, 0.f);
}

template <bool EXT>
__device__ __forceinline__ void store_c(const Fp32GemmParams& p, float alpha, int gm, int gn, float acc, float2 x = make_float2(0.f, 0.f)) {
  float v = alpha * acc;
  if (p.R) v += p.R[(size_t)gm * p.ldr + gn];
  const size_t at = (size_t)gm * p.ldc + gn;
  float* c = p.C + at;
  if (p.accumulate) v += *c;
  *c = v;
  if constexpr (EXT) {
    const float sg = sigmoidf_(x.x);
    p.gt[at] = v * x.y * sg * (1.f + x.x * (1.f - sg));
    p.u[at] = v * x.x * sg;
  }
}

}  // namespace

// ---- tiles of 128 x 128 (T = 2) or 64 x 64 (T = 1): four waves, each T x T instruction tiles of 32 x 32 ----
template <int T, bool AKM, bool BKM, bool VEC>
__global__ __launch_bounds__(256, 2) void gemm_fp32_tile_kernel(Fp32GemmParams p) {
  constexpr int BT = 64 * T, BK = 32;
  // K-major operand: [row][k], pitch 36: the 16 rows of a 16-byte read start 4 banks * 9 apart, i.e. on 16 different
  // bank groups.  Row-major operand: [k][row], pitch BT + 8: the two k-rows of a read, 4 apart, lie on opposite
  // halves of the 64 banks.
  constexpr int KP = BK + 4, RP = BT + 8;
  constexpr int ASZ = AKM ? BT * KP : BK * RP, BSZ = BKM ? BT * KP : BK * RP;
  constexpr int PIECES = BT * BK / 4 / 256;   // 16-byte pieces per thread, operand and slab
  __shared__ __attribute__((aligned(16))) float sA[2][ASZ];
  __shared__ __attribute__((aligned(16))) float sB[2][BSZ];
  device_sizes(p);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, g = lane >> 5;
  const int m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
  if (m0 >= p.M) return;                                        // whole block, before any barrier
  if (p.K == 0 && p.K2 == 0 && p.accumulate) return;            // nothing to add
  const int wm = (wave >> 1) * 32 * T, wn = (wave & 1) * 32 * T;
  f32x16_t acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  const int nk1 = (p.K + BK - 1) / BK, nk = nk1 + (p.K2 + BK - 1) / BK;

  // slab t passes through register set t & 1 and LDS stage t & 1: it is requested two slabs before its turn (one slab
  // of a 64 x 64 tile is 1024 clocks of MFMAs, less than a load takes to arrive)
  f32x4_t ra0[PIECES], rb0[PIECES], ra1[PIECES], rb1[PIECES];
  auto fetch = [&](auto KM, const float* base, int64_t ld, int r0, int rows, int k0, int K, f32x4_t (&r)[PIECES]) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int pc = tid + i * 256;
      if constexpr (decltype(KM)::value) {
        const int row = pc / (BK / 4), k = k0 + (pc % (BK / 4)) * 4;
        r[i] = load4<VEC>(base, (int64_t)(r0 + row) * ld + k, r0 + row < rows ? K - k : 0);
      } else {
        const int k = k0 + pc / (BT / 4), col = r0 + (pc % (BT / 4)) * 4;
        r[i] = load4<VEC>(base, (int64_t)k * ld + col, k < K ? rows - col : 0);
      }
    }
  };
  auto put = [&](auto KM, float* s, const f32x4_t (&r)[PIECES]) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int pc = tid + i * 256;
      if constexpr (decltype(KM)::value) *reinterpret_cast<f32x4_t*>(s + (pc / (BK / 4)) * KP + (pc % (BK / 4)) * 4) = r[i];
      else *reinterpret_cast<f32x4_t*>(s + (pc / (BT / 4)) * RP + (pc % (BT / 4)) * 4) = r[i];
    }
  };
  auto fetch_slab = [&](int t, f32x4_t (&ra)[PIECES], f32x4_t (&rb)[PIECES]) {
    const bool second = t >= nk1;
    const int k0 = (second ? t - nk1 : t) * BK, K = second ? p.K2 : p.K;
    fetch(std::bool_constant<AKM>{}, second ? p.A2 : p.A, p.lda, m0, p.M, k0, K, ra);
    fetch(std::bool_constant<BKM>{}, second ? p.B2 : p.B, p.ldb, n0, p.N, k0, K, rb);
  };
  auto put_slab = [&](int st, const f32x4_t (&ra)[PIECES], const f32x4_t (&rb)[PIECES]) {
    put(std::bool_constant<AKM>{}, sA[st], ra);
    put(std::bool_constant<BKM>{}, sB[st], rb);
  };
  // the lane's four values of k group s (8 k) for the 32 rows that start at `row`
  auto frag = [&](auto KM, const float* s, int row, int grp) {
    if constexpr (decltype(KM)::value) return *reinterpret_cast<const f32x4_t*>(s + (row + lr) * KP + grp * 8 + 4 * g);
    else {
      const float* q = s + (grp * 8 + 4 * g) * RP + row + lr;
      return f32x4_t{q[0], q[RP], q[2 * RP], q[3 * RP]};
    }
  };
  auto multiply = [&](int st) {
#pragma unroll
    for (int grp = 0; grp < BK / 8; ++grp) {
      f32x4_t fa[T], fb[T];
#pragma unroll
      for (int i = 0; i < T; ++i) fa[i] = frag(std::bool_constant<AKM>{}, sA[st], wm + 32 * i, grp);
#pragma unroll
      for (int j = 0; j < T; ++j) fb[j] = frag(std::bool_constant<BKM>{}, sB[st], wn + 32 * j, grp);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
    }
  };
  if (nk > 0) {
    fetch_slab(0, ra0, rb0);
    if (nk > 1) fetch_slab(1, ra1, rb1);
    put_slab(0, ra0, rb0);
  }
  __syncthreads();
  // (a stage is written after the barrier that its last readers passed, at the end of the slab before)
  for (int t = 0; t < nk; t += 2) {
    if (t + 2 < nk) fetch_slab(t + 2, ra0, rb0);
    multiply(0);
    if (t + 1 < nk) put_slab(1, ra1, rb1);
    __syncthreads();
    if (t + 1 >= nk) break;
    if (t + 3 < nk) fetch_slab(t + 3, ra1, rb1);
    multiply(1);
    if (t + 2 < nk) put_slab(0, ra0, rb0);
    __syncthreads();
  }
  float alpha = p.alpha;
  if (p.alpha_dev) alpha *= *p.alpha_dev;
  // register q of lane (lr, g) is row 8 (q / 4) + 4 g + q % 4, column lr
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int gm = m0 + wm + 32 * i + 8 * (q >> 2) + 4 * g + (q & 3);
#pragma unroll
      for (int j = 0; j < T; ++j) {
        const int gn = n0 + wn + 32 * j + lr;
        if (gm < p.M && gn < p.N) store_c<false>(p, alpha, gm, gn, acc[i][j][q]);
      }
    }
}

// ---- one E x E tile per block (E = 32, or 16 with v_mfma_f32_16x16x4_f32), the contraction split over NW waves ----
// wave `wave`'s share of the tile at (m0, n0), left in its part
template <int E, int NW, bool AKM, bool BKM, bool VEC>
__device__ __forceinline__ void wavek_share(const Fp32GemmParams& p, int m0, int n0, int wave, int lane, float* part) {
  constexpr int NG = 64 / E;     // lane groups, each with four consecutive k of a group of KG
  constexpr int KG = 4 * NG;     // 8 (E = 32) or 16
  constexpr int NACC = E * E / 64;
  typedef float acc_t __attribute__((ext_vector_type(NACC)));
  constexpr int U = 4;   // groups whose loads are issued together
  const int lr = lane % E, g = lane / E;
  acc_t acc;
#pragma unroll
  for (int q = 0; q < NACC; ++q) acc[q] = 0.f;
  // rows past the end repeat the last one: they are never stored
  const int am = min(m0 + lr, p.M - 1), bn = min(n0 + lr, p.N - 1);
  auto fetch = [&](auto KM, const float* base, int64_t ld, int row, int k, int K) {
    if constexpr (decltype(KM)::value) return load4<VEC>(base, (int64_t)row * ld + k, K - k);
    else {
      f32x4_t v = {0.f, 0.f, 0.f, 0.f};
      const float* q = base + (int64_t)k * ld + row;
      if (k < K) v.x = q[0];
      if (k + 1 < K) v.y = q[ld];
      if (k + 2 < K) v.z = q[2 * ld];
      if (k + 3 < K) v.w = q[3 * ld];
      return v;
    }
  };
  for (int pair = 0; pair < 2; ++pair) {
    const float* A = pair ? p.A2 : p.A;
    const float* B = pair ? p.B2 : p.B;
    const int K = pair ? p.K2 : p.K;
    const int ng = (K + KG - 1) / KG;
    // neighbouring waves take neighbouring groups: together they read whole lines
    for (int g0 = wave; g0 < ng; g0 += NW * U) {
      f32x4_t fa[U], fb[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = (g0 + u * NW) * KG + 4 * g;   // groups past the end are zeros
        fa[u] = fetch(std::bool_constant<AKM>{}, A, p.lda, am, k, K);
        fb[u] = fetch(std::bool_constant<BKM>{}, B, p.ldb, bn, k, K);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (E == 32) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u][e], fb[u][e], acc, 0, 0, 0);
          else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][e], fb[u][e], acc, 0, 0, 0);
        }
    }
  }
  // register q of lane (lr, g) is row 4 g + q (E = 16) or 8 (q / 4) + 4 g + q % 4 (E = 32), column lr
#pragma unroll
  for (int q = 0; q < NACC; ++q) part[(8 * (q >> 2) + 4 * g + (q & 3)) * E + lr] = acc[q];
}

template <int E, int NW, bool AKM, bool BKM, bool VEC, bool EXT>
__device__ __forceinline__ void wavek_tile(Fp32GemmParams p, int tile_m, int tile_n) {
  __shared__ __attribute__((aligned(16))) float part[NW][E * E];
  device_sizes(p);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = tile_m * E, n0 = tile_n * E;
  if (m0 >= p.M) return;                                        // whole block, before any barrier
  if (p.K == 0 && p.K2 == 0 && p.accumulate) return;            // nothing to add
  constexpr int PE = (E * E + NW * 64 - 1) / (NW * 64);   // elements of C per thread
  float2 behind[PE];
  if constexpr (EXT) {
#pragma unroll
    for (int i = 0; i < PE; ++i) {
      const int e = threadIdx.x + i * NW * 64;
      behind[i] = load_behind(p, e < E * E ? m0 + e / E : p.M, n0 + e % E);
    }
  }
  wavek_share<E, NW, AKM, BKM, VEC>(p, m0, n0, wave, lane, part[wave]);
  __syncthreads();
  float alpha = p.alpha;
  if (p.alpha_dev) alpha *= *p.alpha_dev;
#pragma unroll
  for (int i = 0; i < PE; ++i) {
    const int e = threadIdx.x + i * NW * 64;
    if (e >= E * E) break;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += part[w][e];
    const int gm = m0 + e / E, gn = n0 + e % E;
    if (gm < p.M && gn < p.N) store_c<EXT>(p, alpha, gm, gn, v, behind[i]);
  }
}

template <int E, int NW, bool AKM, bool BKM, bool VEC, bool EXT = false>
__global__ __launch_bounds__(NW * 64) void gemm_fp32_wavek_kernel(Fp32GemmParams p) {
  wavek_tile<E, NW, AKM, BKM, VEC, EXT>(p, blockIdx.y, blockIdx.x);
}

// Gate and up products (NT, same sizes and left operand) and h = silu(gate) up: tiles of 16 x 16, four waves for either.
template <bool VEC>
__global__ __launch_bounds__(512) void gemm_fp32_swiglu_kernel(Fp32GemmParams p, const float* B_up, float* C_up, float* h) {
  __shared__ __attribute__((aligned(16))) float part[8][256];
  __shared__ float gate[256];
  device_sizes(p);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), e = threadIdx.x & 255;
  const bool up = wave >= 4;
  const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
  if (m0 >= p.M) return;   // whole block, before any barrier
  if (up) { p.B = B_up; p.C = C_up; }
  wavek_share<16, 4, true, true, VEC>(p, m0, n0, wave & 3, lane, part[wave]);
  __syncthreads();
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) v += part[(up ? 4 : 0) + w][e];
  v *= p.alpha;
  if (!up) gate[e] = v;
  __syncthreads();
  const int gm = m0 + e / 16, gn = n0 + e % 16;
  if (gm >= p.M || gn >= p.N) return;
  const size_t at = (size_t)gm * p.ldc + gn;
  p.C[at] = v;
  if (up) h[at] = gate[e] * sigmoidf_(gate[e]) * v;
}

// Several independent products of one layout in one launch: a product of the fp32 configuration is 4 us of launch and
// latency, whatever its size.
namespace {
struct Fp32Group { Fp32GemmParams p[kMaxGemmGroup]; int first[kMaxGemmGroup + 1]; int n; };   // first tile of each
}
template <bool AKM, bool BKM, bool VEC>
__global__ __launch_bounds__(256) void gemm_fp32_group_kernel(Fp32Group g) {
  int i = 0;
#pragma unroll
  for (int k = 1; k < kMaxGemmGroup; ++k)
    if (k < g.n && (int)blockIdx.x >= g.first[k]) i = k;
  const int tile = blockIdx.x - g.first[i], tiles_n = (g.p[i].N + 15) / 16;
  wavek_tile<16, 4, AKM, BKM, VEC, false>(g.p[i], tile / tiles_n, tile % tiles_n);
}

namespace {

// Which kernel.  The large tile when it gives every CU one; the small one, or the 32-row tile of the split over waves,
// when it gives three CUs in four one (300 x 2048 x 2048: 54 us with 160 tiles of 64 refused, 79 us with them; 512 x 256 x
// 4096: 30 us with 128 tiles of 32 refused, 40 with them); else tiles of 16.  Sixteen waves from K = 1024 on
// (TN 688 x 256 x 512: 8 us with four, 55 with sixteen, whose blocks then have two loads each; NN 128 x 256 x 4096 needs
// them: 16 us).  Against the fp32-FMA kernel (64 x 64 tiles, gemm_simple.hip) that this file replaces, us before and now:
// 128 x 256 x 768 106 / 6, NN 128 x 256 x 4096 769 / 16, TN 4096 x 256 x 1024 192 / 36, NT 214 x 5632 x 5120 855 / 255, NN 3000 x
// 2048 x 2048 421 / 309, NT 32768 x 256 x 2048 805 / 295 (117 TFLOP/s).
constexpr int64_t kBigTiles = 256, kSmallTiles = 192;
constexpr int64_t kWideK = 1024;

template <int E, bool AKM, bool BKM, bool VEC, bool EXT>
void launch_wavek(const Fp32GemmParams& p, dim3 grid, hipStream_t s) {
  if constexpr (!EXT) {   // (see gemm_swiglu_supported)
    if ((int64_t)p.K + p.K2 >= kWideK) {
      hipLaunchKernelGGL((gemm_fp32_wavek_kernel<E, 16, AKM, BKM, VEC>), grid, dim3(1024), 0, s, p);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_fp32_wavek_kernel<E, 4, AKM, BKM, VEC, EXT>), grid, dim3(256), 0, s, p);
}

template <bool AKM, bool BKM, bool VEC, bool EXT>
hipError_t launch_fp32_layout(const Fp32GemmParams& p, hipStream_t s) {
  auto tiles = [&](int64_t e) { return ((p.M + e - 1) / e) * ((p.N + e - 1) / e); };
  auto grid = [&](int e) { return dim3((unsigned)((p.N + e - 1) / e), (unsigned)((p.M + e - 1) / e)); };
  if constexpr (!EXT) {   // (see gemm_swiglu_supported)
    if (tiles(128) >= kBigTiles) {
      hipLaunchKernelGGL((gemm_fp32_tile_kernel<2, AKM, BKM, VEC>), grid(128), dim3(256), 0, s, p);
      return hipGetLastError();
    }
    if (tiles(64) >= kSmallTiles) {
      hipLaunchKernelGGL((gemm_fp32_tile_kernel<1, AKM, BKM, VEC>), grid(64), dim3(256), 0, s, p);
      return hipGetLastError();
    }
  }
  if (tiles(32) >= kSmallTiles) launch_wavek<32, AKM, BKM, VEC, EXT>(p, grid(32), s);
  else launch_wavek<16, AKM, BKM, VEC, EXT>(p, grid(16), s);
  return hipGetLastError();
}

template <bool AKM, bool BKM, bool EXT = false>
hipError_t launch_fp32_vec(const Fp32GemmParams& p, bool vec, hipStream_t s) {
  return vec ? launch_fp32_layout<AKM, BKM, true, EXT>(p, s) : launch_fp32_layout<AKM, BKM, false, EXT>(p, s);
}

}  // namespace

namespace {
bool fp32_params(const GemmArgs& a, Fp32GemmParams& p, bool& vec) {   // false: sizes beyond 32-bit counting
  const int64_t lim = (int64_t)1 << 30;
  if (a.M >= lim || a.N >= lim || a.K >= lim || a.K2 >= lim) return false;
  p.A = (const float*)a.A; p.B = (const float*)a.B; p.A2 = (const float*)a.A2; p.B2 = (const float*)a.B2;
  p.C = (float*)a.C; p.R = (const float*)a.residual; p.alpha_dev = a.alpha_dev;
  p.lda = a.lda; p.ldb = a.ldb; p.ldc = a.ldc; p.ldr = a.ldr;
  p.M = (int)a.M; p.N = (int)a.N; p.K = (int)a.K; p.K2 = a.A2 ? (int)a.K2 : 0;
  p.alpha = a.alpha; p.accumulate = a.accumulate;
  p.m_dev = a.m_dev; p.m_off = a.m_off; p.k_dev = a.k_dev; p.k_off = a.k_off;
  p.gt = p.u = nullptr;
  // 16-byte loads where every row of every operand starts on a 16-byte boundary
  vec = a.lda % 4 == 0 && a.ldb % 4 == 0 && (((uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.A2 | (uintptr_t)a.B2) & 15) == 0;
  return true;
}

template <bool AKM, bool BKM>
hipError_t launch_fp32_group(const Fp32Group& g, bool vec, hipStream_t s) {
  if (vec) hipLaunchKernelGGL((gemm_fp32_group_kernel<AKM, BKM, true>), dim3((unsigned)g.first[g.n]), dim3(256), 0, s, g);
  else hipLaunchKernelGGL((gemm_fp32_group_kernel<AKM, BKM, false>), dim3((unsigned)g.first[g.n]), dim3(256), 0, s, g);
  return hipGetLastError();
}
}  // namespace

// The sizes whose products run on tiles of 16 or 32: there a launch of its own is what the pass over the activations costs, and it
// waits for the products' last block (a step of 128 rows: 181.0 us with the two passes of SwiGLU as launches, 178.0 without).
// AdamW behind the weight gradients in the same way was slower (179.9): it is bound by memory, and these kernels have few loads in flight.
bool gemm_swiglu_supported(const GemmArgs& a) {
  Fp32GemmParams p;
  bool vec;
  return a.in_dtype == kF32 && a.out_dtype == kF32 && a.M > 0 && a.N > 0 && !a.residual && !a.A2 && !a.accumulate && !a.alpha_dev &&
         fp32_params(a, p, vec) && a.K < kWideK && ((a.M + 63) / 64) * ((a.N + 63) / 64) < kSmallTiles;
}

hipError_t launch_gemm_swiglu_fwd(const GemmArgs& a, const GemmArgs& up, float* h, hipStream_t s) {
  Fp32GemmParams p, q;
  bool vec, vec_up;
  if (!gemm_swiglu_supported(a) || !gemm_swiglu_supported(up) || a.layout != kNT || up.layout != kNT || up.A != a.A || up.M != a.M || up.N != a.N ||
      up.K != a.K || up.lda != a.lda || up.ldb != a.ldb || up.ldc != a.ldc || up.m_dev != a.m_dev || up.m_off != a.m_off ||
      !fp32_params(a, p, vec) || !fp32_params(up, q, vec_up)) return hipErrorInvalidValue;
  ProfScope ps("gemm_fp32_swiglu", 4.0 * a.M * a.N * (double)a.K, 4.0 * (a.K * (a.M + 2.0 * a.N) + 3.0 * a.M * a.N), s);
  if (a.m_dev) prof_dynamic(a.m_dev, a.m_off, a.M);
  const dim3 grid((unsigned)((a.N + 15) / 16), (unsigned)((a.M + 15) / 16));
  if (vec && vec_up) hipLaunchKernelGGL(gemm_fp32_swiglu_kernel<true>, grid, dim3(512), 0, s, p, q.B, q.C, h);
  else hipLaunchKernelGGL(gemm_fp32_swiglu_kernel<false>, grid, dim3(512), 0, s, p, q.B, q.C, h);
  return hipGetLastError();
}

hipError_t launch_gemm_swiglu_bwd(const GemmArgs& a, float* gt, float* u, hipStream_t s) {
  Fp32GemmParams p;
  bool vec;
  if (!gemm_swiglu_supported(a) || a.layout != kNN || !fp32_params(a, p, vec)) return hipErrorInvalidValue;
  ProfScope ps("gemm_fp32_swiglu_bwd", 2.0 * a.M * a.N * (double)a.K, 4.0 * (a.K * (a.M + (double)a.N) + 5.0 * a.M * a.N), s);
  if (a.m_dev) prof_dynamic(a.m_dev, a.m_off, a.M);
  p.gt = gt; p.u = u;
  return launch_fp32_vec<true, false, true>(p, vec, s);
}

hipError_t launch_gemm_fp32(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  Fp32GemmParams p;
  bool vec;
  if (!fp32_params(a, p, vec)) return launch_gemm_simple(a, s);   // the kernel that counts in 64 bits
  if ((a.M + 63) / 64 > 65535) return hipErrorInvalidValue;
  switch (a.layout) {
    case kNT: return launch_fp32_vec<true, true>(p, vec, s);
    case kNN: return launch_fp32_vec<true, false>(p, vec, s);
    case kTN: return launch_fp32_vec<false, false>(p, vec, s);
    default: return hipErrorInvalidValue;
  }
}

// n independent products, one launch when all of them are fp32, of one layout and of the size that the split over four
// waves serves alone; one by one otherwise
hipError_t launch_gemm_group(const GemmArgs* a, int n, hipStream_t s) {
  Fp32Group g;
  g.n = n;
  g.first[0] = 0;
  bool vec = true, together = n > 1 && n <= kMaxGemmGroup;
  double flops = 0, bytes = 0, fixed_flops = 0, fixed_bytes = 0;   // fixed: of products whose sizes are all known here
  const int* dyn = nullptr;                                        // (the others of a step share one size on the device)
  int64_t dyn_off = 0, dyn_max = 0;
  for (int i = 0; together && i < n; ++i) {
    bool v = false;
    together = a[i].in_dtype == kF32 && a[i].out_dtype == kF32 && a[i].layout == a[0].layout && a[i].M > 0 && a[i].N > 0 &&
               fp32_params(a[i], g.p[i], v) && (int64_t)g.p[i].K + g.p[i].K2 < kWideK &&
               ((a[i].M + 63) / 64) * ((a[i].N + 63) / 64) < kSmallTiles;
    if (!together) break;
    vec = vec && v;
    g.first[i + 1] = g.first[i] + (int)(((a[i].M + 15) / 16) * ((a[i].N + 15) / 16));
    const double k = (double)g.p[i].K + g.p[i].K2, f = 2.0 * a[i].M * a[i].N * k, b = 4.0 * (k * (a[i].M + a[i].N) + a[i].M * (double)a[i].N);
    flops += f;
    bytes += b;
    if (a[i].m_dev) { dyn = a[i].m_dev; dyn_off = a[i].m_off; dyn_max = a[i].M; }
    else if (a[i].k_dev) { dyn = a[i].k_dev; dyn_off = a[i].k_off; dyn_max = a[i].K; }
    else { fixed_flops += f; fixed_bytes += b; }
  }
  if (!together) {
    for (int i = 0; i < n; ++i) {
      const hipError_t e = launch_gemm(a[i], s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  ProfScope ps("gemm_fp32_group", flops, bytes, s);
  if (dyn) prof_dynamic(dyn, dyn_off, dyn_max, fixed_flops, fixed_bytes);
  switch (a[0].layout) {
    case kNT: return launch_fp32_group<true, true>(g, vec, s);
    case kNN: return launch_fp32_group<true, false>(g, vec, s);
    case kTN: return launch_fp32_group<false, false>(g, vec, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tide
