// Shape-agnostic causal grouped-query attention for gfx950 in fp32 arithmetic: any head_dim <= 256, any sequence length,
// fp32 or bf16 storage.  It is the attention path of fp32 mode and the bf16 path for head sizes the flash kernels do not
// take.  Deterministic: no atomics; every output element is produced by one block in a fixed order.
//
// Activation layout: qkv [B*S, (nh + 2 nkv) dh] with q heads first, then k heads, then v heads; query
// head h reads kv head h / (nh / nkv).  lse[b, h, i] is the log-sum-exp of the scaled scores of row i.
// Packed batches (cu_seqlens given): sequence b owns rows [cu[b], cu[b+1]) and lse / delta are [nh, T].
//
// All products run on v_mfma_f32_16x16x4_f32 (fp32 products and sums).  A block is four waves and 16 rows: 16 queries of a
// head (forward, dQ) or 16 keys of a kv head (dK, dV).  It walks the other side in tiles of 64, 16 rows per wave for the
// score products (their contraction runs over the head, 16 channels at a time, fragments straight from L2 into
// registers), passes the 16 x 64 probabilities or score gradients through LDS, and the waves share the columns of the
// second product.  What bounds it at the sizes it serves (the fp32 configuration has 64 to 1024 positions and 4 heads)
// is latency, so there are one or two barriers per tile and no staging of operands.  fp32, forward + backward, us, one
// wavefront per row on the vector units before / now: 2 x 64, 4 / 2 heads of 64: 6 + 37 / 6 + 17; 1 x 1024: 101 + 1382 / 39 + 155;
// 2 x 1024, 16 / 8 heads of 128: 1287 + 24316 / 233 + 1071.
#include <type_traits>

#include "kernels.h"
#include "prof.h"
#include "tide_common.h"

namespace tide {

namespace {

constexpr int kMaxDh = 256;
constexpr int BR = 16, BT = 64;      // rows of a block, rows of a tile of the other side
constexpr int PP = BT + 4;           // LDS pitch of the 16 x 64 exchange (the 16-byte reads of 16 rows hit 16 bank groups)
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// four consecutive channels c .. c+3 of a row, zeros past dh; VEC: they are aligned to 16 (fp32) or 8 (bf16) bytes
template <bool VEC>
__device__ __forceinline__ f32x4_t row4(const float* p, int c, int dh) {
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
  if (VEC) {
    if (c < dh) v = *reinterpret_cast<const f32x4_t*>(p + c);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < dh) v[e] = p[c + e];
  }
  return v;
}
template <bool VEC>
__device__ __forceinline__ f32x4_t row4(const bf16_t* p, int c, int dh) {
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
  if (VEC) {
    if (c < dh) {
      const uint2 w = *reinterpret_cast<const uint2*>(p + c);
      v = f32x4_t{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u)};
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < dh) v[e] = bf2f(p[c + e]);
  }
  return v;
}

// acc += A B^T over the 16 channels of one group: both fragments hold, for row l % 16, channels 4 (l / 16) .. + 3
__device__ __forceinline__ f32x4_t mma16(f32x4_t a, f32x4_t b, f32x4_t acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
  return acc;
}

// Register q of a 16 x 16 result in lane l is row 4 (l / 16) + q, column l % 16.
struct Geo {
  int lane, wave, lr, g;
  __device__ Geo() : lane(threadIdx.x & 63), wave(threadIdx.x >> 6), lr(lane & 15), g(lane >> 4) {}
};

// the wave's columns of the second product: acc[t] += X[16 x 64] Y[64 x 16 columns], X from the exchange in LDS, Y's rows
// r0 .. r0 + 63 from memory (zeros from row `rows` on).  Loads past the end are of the last row or column instead, so that
// none is behind a branch, between which the compiler waits (bf16, 1 x 700, 8 / 2 heads of 80: 77 + 565 / 49 + 321 us); BRANCH:
// behind branches, which take fewer registers (fp32, same, heads of 256, backward: 1053 / 794; of 18, forward 49 / 36).
template <bool BRANCH, int NCT, typename T>
__device__ __forceinline__ void second_product(const Geo& z, const float* x, const T* y, size_t ld, int r0, int rows, int dh, f32x4_t (&acc)[NCT]) {
#pragma unroll
  for (int t = 0; t < NCT; ++t) {
    const int col = (z.wave + 4 * t) * 16 + z.lr;
    f32x4_t v[4];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = r0 + grp * 16 + 4 * z.g + e;
        if constexpr (BRANCH) v[grp][e] = (r < rows && col < dh) ? ldf(y, (size_t)r * ld + col) : 0.f;
        else {
          const float f = ldf(y, (size_t)min(r, rows - 1) * ld + min(col, dh - 1));
          v[grp][e] = (r < rows && col < dh) ? f : 0.f;
        }
      }
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) acc[t] = mma16(*reinterpret_cast<const f32x4_t*>(x + z.lr * PP + grp * 16 + 4 * z.g), v[grp], acc[t]);
  }
}

template <typename T, int NG, bool VEC>
constexpr bool kBranchBwd = sizeof(T) == 4 && (NG == 16 || !VEC);

// Causality where values are not finite.  X is zero where a position sees nothing of another, but zero times the other's NaN
// or infinity is not: it reaches all 16 x 64 results of a tile on the diagonal.  Rows of a result that are not finite, and
// where that can be such a tile's doing, are therefore made again at the end from the positions they see alone, by the
// wave whose columns they are, a channel per lane.  No row of finite inputs is.
// Bits of the block's rows (4 (l / 16) + q) in which a wave's columns hold something that is not finite; ask[q]: the row counts.
template <int NCT>
__device__ __forceinline__ uint32_t not_finite(const Geo& z, const f32x4_t (&acc)[NCT], const bool (&ask)[4]) {
  uint32_t rows = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float odd = 0.f;
#pragma unroll
    for (int t = 0; t < NCT; ++t) odd = fmaf(acc[t][q], 0.f, odd);
    const uint64_t b = __builtin_amdgcn_ballot_w64(odd != 0.f && ask[q]);
#pragma unroll
    for (int g = 0; g < 4; ++g) rows |= ((b >> (16 * g)) & 0xFFFFu) != 0 ? 1u << (4 * g + q) : 0u;
  }
  return rows;
}
// what the lanes of row r hold in v
__device__ __forceinline__ float of_row(const f32x4_t& v, int r) {
  const int q = r & 3;
  return __shfl(q == 0 ? v[0] : q == 1 ? v[1] : q == 2 ? v[2] : v[3], 4 * (r & 12), 64);
}
// channels lane, lane + 64, ... of a row
constexpr int NU = kMaxDh / 64;
template <typename T>
__device__ __forceinline__ void channels(const T* row, int lane, int dh, float (&v)[NU]) {
#pragma unroll
  for (int u = 0; u < NU; ++u) v[u] = lane + 64 * u < dh ? ldf(row, lane + 64 * u) : 0.f;
}
__device__ __forceinline__ float dot(const float (&a)[NU], const float (&b)[NU]) {
  float s = 0.f;
#pragma unroll
  for (int u = 0; u < NU; ++u) s = fmaf(a[u], b[u], s);
  return wave_sum(s);
}
// channel lane + 64 u is one of the wave's columns: (wave + 4 t) 16 .. + 15
__device__ __forceinline__ bool own_channel(const Geo& z, int u, int dh) { return z.g == z.wave && z.lane + 64 * u < dh; }
// the stores of the rows as they came out are done before a row is stored again, by other lanes of the wave
__device__ __forceinline__ void wait_stores() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
}
__device__ __forceinline__ float times_zero(const float (&a)[NU]) {   // not zero where something is not finite
  return fmaf(a[0], 0.f, a[1] * 0.f) + fmaf(a[2], 0.f, a[3] * 0.f);
}

// Over the 16 lanes of a group, by rotations inside the group on the vector unit (DPP row_ror), about 10 clocks a step; through
// the LDS crossbar the four rows' chains of four steps were 0.8 us, most of what a sequence of a few positions takes.
template <int N>
__device__ __forceinline__ float rotate16(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x120 + N, 0xF, 0xF, false));
}
__device__ __forceinline__ float max16(float v) {
  v = fmaxf(v, rotate16<8>(v));
  v = fmaxf(v, rotate16<4>(v));
  v = fmaxf(v, rotate16<2>(v));
  return fmaxf(v, rotate16<1>(v));
}
__device__ __forceinline__ float sum16(float v) {
  v += rotate16<8>(v);
  v += rotate16<4>(v);
  v += rotate16<2>(v);
  return v + rotate16<1>(v);
}

}  // namespace

// NG groups of 16 channels (dh <= 16 NG), NCT = NG / 4 column tiles per wave
template <typename T, int NG, bool VEC>
__global__ __launch_bounds__(256) void attn_fwd_simple_kernel(const T* __restrict__ qkv, T* __restrict__ out, float* __restrict__ lse,
                                                              int Smax, int nh, int nkv, int dh, const int* __restrict__ cu, int64_t Trows) {
  constexpr int NCT = NG / 4;
  __shared__ __attribute__((aligned(16))) float ps[2][BR * PP];
  __shared__ float red[2][4][BR];
  const int i0 = blockIdx.x * BR, h = blockIdx.y, b = blockIdx.z;
  const SeqView sv = seq_view(cu, b, Smax, Trows);
  const int S = sv.len;
  if (i0 >= S) return;   // whole block: the sequence is shorter than the grid
  const Geo z;
  const int kh = h / (nh / nkv);
  const size_t ld = (size_t)(nh + 2 * nkv) * dh;
  const float scale = 1.0f / sqrtf((float)dh);
  const T* base = qkv + (size_t)sv.row0 * ld;
  const T* K = base + (size_t)(nh + kh) * dh;
  const T* V = base + (size_t)(nh + nkv + kh) * dh;
  f32x4_t qf[NG];
#pragma unroll
  for (int c = 0; c < NG; ++c) qf[c] = row4<VEC>(base + (size_t)min(i0 + z.lr, S - 1) * ld + (size_t)h * dh, c * 16 + 4 * z.g, dh) * scale;
  f32x4_t o[NCT], m, l;
#pragma unroll
  for (int q = 0; q < 4; ++q) { m[q] = -INFINITY; l[q] = 0.f; }
#pragma unroll
  for (int t = 0; t < NCT; ++t) o[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int last = min(i0 + BR, S) - 1;   // last query of the block
  for (int j0 = 0, st = 0; j0 <= last; j0 += BT, st ^= 1) {
    const int j = j0 + z.wave * 16 + z.lr;
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
    const T* kr = K + (size_t)min(j, S - 1) * ld;
#pragma unroll
    for (int c = 0; c < NG; ++c) s = mma16(qf[c], row4<VEC>(kr, c * 16 + 4 * z.g, dh), s);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (j > i0 + 4 * z.g + q || j >= S) s[q] = -INFINITY;
      const float v = max16(s[q]);
      if (z.lr == 0) red[st][z.wave][4 * z.g + q] = v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 4 * z.g + q;
      const float tm = fmaxf(fmaxf(red[st][0][r], red[st][1][r]), fmaxf(red[st][2][r], red[st][3][r]));
      const float nm = fmaxf(m[q], tm);        // finite: key 0 is visible to every query
      const float corr = __expf(m[q] - nm);    // first tile: exp(-inf) = 0
      const float p = __expf(s[q] - nm);
      l[q] = l[q] * corr + p;                  // this lane's keys only
      m[q] = nm;
#pragma unroll
      for (int t = 0; t < NCT; ++t) o[t][q] *= corr;
      ps[st][r * PP + z.wave * 16 + z.lr] = p;
    }
    __syncthreads();   // (the other buffer is written next: its readers pass this barrier first)
    second_product<sizeof(T) == 4 && !VEC, NCT>(z, ps[st], V, ld, j0, S, dh, o);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float v = sum16(l[q]);
    if (z.lr == 0) red[0][z.wave][4 * z.g + q] = v;
  }
  __syncthreads();
  f32x4_t sum, inv;
  bool ask[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = 4 * z.g + q, i = i0 + r;
    sum[q] = (red[0][0][r] + red[0][1][r]) + (red[0][2][r] + red[0][3][r]);
    inv[q] = 1.0f / sum[q];
    ask[q] = i < S && sum[q] - sum[q] == 0.f;
    if (i >= S) continue;
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
      const int col = (z.wave + 4 * t) * 16 + z.lr;
      if (col < dh) stf(out, ((size_t)sv.row0 + i) * ((size_t)nh * dh) + (size_t)h * dh + col, o[t][q] * inv[q]);
    }
    if (z.wave == 0 && z.lr == 0) lse[stat_index(cu, Trows, sv, b, h, nh, Smax, i)] = m[q] + logf(sum[q]);
  }
  for (uint32_t again = not_finite(z, o, ask); again != 0; again &= again - 1) {   // wave-uniform
    const int r = __builtin_ctz(again), i = i0 + r;
    const float mr = of_row(m, r), ir = of_row(inv, r);
    float qv[NU], kv[NU], vv[NU], acc[NU] = {0.f, 0.f, 0.f, 0.f};
    channels(base + (size_t)i * ld + (size_t)h * dh, z.lane, dh, qv);
#pragma unroll
    for (int u = 0; u < NU; ++u) qv[u] *= scale;
#pragma unroll 1
    for (int j = 0; j <= i; ++j) {
      channels(K + (size_t)j * ld, z.lane, dh, kv);
      channels(V + (size_t)j * ld, z.lane, dh, vv);
      const float p = __expf(dot(qv, kv) - mr);
#pragma unroll
      for (int u = 0; u < NU; ++u) acc[u] = fmaf(p, vv[u], acc[u]);
    }
    wait_stores();
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (own_channel(z, u, dh)) stf(out, ((size_t)sv.row0 + i) * ((size_t)nh * dh) + (size_t)h * dh + z.lane + 64 * u, acc[u] * ir);
  }
}

// dQ, and delta[b,h,i] = sum_c dO[i,h,c] * O[i,h,c] for the dK / dV kernel
template <typename T, int NG, bool VEC>
__global__ __launch_bounds__(256) void attn_dq_simple_kernel(const T* __restrict__ qkv, const T* __restrict__ out, const T* __restrict__ dout,
                                                             const float* __restrict__ lse, float* __restrict__ delta, T* __restrict__ dqkv,
                                                             int Smax, int nh, int nkv, int dh, const int* __restrict__ cu, int64_t Trows) {
  constexpr int NCT = NG / 4;
  __shared__ __attribute__((aligned(16))) float ps[2][BR * PP];
  const int i0 = blockIdx.x * BR, h = blockIdx.y, b = blockIdx.z;
  const SeqView sv = seq_view(cu, b, Smax, Trows);
  const int S = sv.len;
  if (i0 >= S) return;
  const Geo z;
  const int kh = h / (nh / nkv);
  const size_t ld = (size_t)(nh + 2 * nkv) * dh;
  const float scale = 1.0f / sqrtf((float)dh);
  const T* base = qkv + (size_t)sv.row0 * ld;
  const T* K = base + (size_t)(nh + kh) * dh;
  const T* V = base + (size_t)(nh + nkv + kh) * dh;
  f32x4_t qf[NG], df[NG];
  float dsum = 0.f;
  {
    const int i = min(i0 + z.lr, S - 1);
    const size_t ro = ((size_t)sv.row0 + i) * ((size_t)nh * dh) + (size_t)h * dh;
#pragma unroll
    for (int c = 0; c < NG; ++c) {
      qf[c] = row4<VEC>(base + (size_t)i * ld + (size_t)h * dh, c * 16 + 4 * z.g, dh) * scale;
      df[c] = row4<VEC>(dout + ro, c * 16 + 4 * z.g, dh);
      const f32x4_t of = row4<VEC>(out + ro, c * 16 + 4 * z.g, dh);
#pragma unroll
      for (int e = 0; e < 4; ++e) dsum = fmaf(of[e], df[c][e], dsum);
    }
  }
  dsum += __shfl_xor(dsum, 16, 64);
  dsum += __shfl_xor(dsum, 32, 64);     // every lane: the row l % 16
  f32x4_t L, D, dq[NCT];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = i0 + 4 * z.g + q;
    D[q] = __shfl(dsum, 4 * z.g + q, 64);
    L[q] = i < S ? lse[stat_index(cu, Trows, sv, b, h, nh, Smax, i)] : 0.f;
    if (z.wave == 0 && z.lr == 0 && i < S) delta[stat_index(cu, Trows, sv, b, h, nh, Smax, i)] = D[q];
  }
#pragma unroll
  for (int t = 0; t < NCT; ++t) dq[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int last = min(i0 + BR, S) - 1;
  for (int j0 = 0, st = 0; j0 <= last; j0 += BT, st ^= 1) {
    const int j = j0 + z.wave * 16 + z.lr;
    f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = s;
    const size_t jr = (size_t)min(j, S - 1) * ld;
#pragma unroll
    for (int c = 0; c < NG; ++c) {
      s = mma16(qf[c], row4<VEC>(K + jr, c * 16 + 4 * z.g, dh), s);
      dp = mma16(df[c], row4<VEC>(V + jr, c * 16 + 4 * z.g, dh), dp);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + 4 * z.g + q;
      ps[st][(4 * z.g + q) * PP + z.wave * 16 + z.lr] = (j <= i && i < S) ? __expf(s[q] - L[q]) * (dp[q] - D[q]) : 0.f;
    }
    __syncthreads();   // (a buffer is written again two tiles on: its readers pass the barrier in between first)
    second_product<kBranchBwd<T, NG, VEC>, NCT>(z, ps[st], K, ld, j0, S, dh, dq);
  }
  bool ask[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = i0 + 4 * z.g + q;
    ask[q] = i < S && L[q] - L[q] == 0.f && D[q] - D[q] == 0.f;
    if (i >= S) continue;
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
      const int col = (z.wave + 4 * t) * 16 + z.lr;
      if (col < dh) stf(dqkv, ((size_t)sv.row0 + i) * ld + (size_t)h * dh + col, dq[t][q] * scale);
    }
  }
  for (uint32_t again = not_finite(z, dq, ask); again != 0; again &= again - 1) {   // wave-uniform
    const int r = __builtin_ctz(again), i = i0 + r;
    const float Lr = of_row(L, r), Dr = of_row(D, r);
    float qv[NU], dov[NU], kv[NU], vv[NU], acc[NU] = {0.f, 0.f, 0.f, 0.f};
    channels(base + (size_t)i * ld + (size_t)h * dh, z.lane, dh, qv);
    channels(dout + ((size_t)sv.row0 + i) * ((size_t)nh * dh) + (size_t)h * dh, z.lane, dh, dov);
#pragma unroll
    for (int u = 0; u < NU; ++u) qv[u] *= scale;
#pragma unroll 1
    for (int j = 0; j <= i; ++j) {
      channels(K + (size_t)j * ld, z.lane, dh, kv);
      channels(V + (size_t)j * ld, z.lane, dh, vv);
      const float d = __expf(dot(qv, kv) - Lr) * (dot(dov, vv) - Dr);
#pragma unroll
      for (int u = 0; u < NU; ++u) acc[u] = fmaf(d, kv[u], acc[u]);
    }
    wait_stores();
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (own_channel(z, u, dh)) stf(dqkv, ((size_t)sv.row0 + i) * ld + (size_t)h * dh + z.lane + 64 * u, acc[u] * scale);
  }
}

template <typename T, int NG, bool VEC>
__global__ __launch_bounds__(256) void attn_dkv_simple_kernel(const T* __restrict__ qkv, const T* __restrict__ dout, const float* __restrict__ lse,
                                                              const float* __restrict__ delta, T* __restrict__ dqkv, int Smax, int nh, int nkv,
                                                              int dh, const int* __restrict__ cu, int64_t Trows) {
  constexpr int NCT = NG / 4;
  __shared__ __attribute__((aligned(16))) float ps[2][BR * PP];   // probabilities, transposed: [key][query]
  __shared__ __attribute__((aligned(16))) float ds[2][BR * PP];   // score gradients
  const int j0 = blockIdx.x * BR, kh = blockIdx.y, b = blockIdx.z;
  const SeqView sv = seq_view(cu, b, Smax, Trows);
  const int S = sv.len;
  if (j0 >= S) return;
  const Geo z;
  const int G = nh / nkv;
  const size_t ld = (size_t)(nh + 2 * nkv) * dh, ldo = (size_t)nh * dh;
  const float scale = 1.0f / sqrtf((float)dh);
  const T* base = qkv + (size_t)sv.row0 * ld;
  const int j = j0 + z.lr;              // this lane's key
  f32x4_t kf[NG], vf[NG], dk[NCT], dv[NCT];
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    const T* r = base + (size_t)min(j, S - 1) * ld;
    kf[c] = row4<VEC>(r + (size_t)(nh + kh) * dh, c * 16 + 4 * z.g, dh) * scale;
    vf[c] = row4<VEC>(r + (size_t)(nh + nkv + kh) * dh, c * 16 + 4 * z.g, dh);
  }
#pragma unroll
  for (int t = 0; t < NCT; ++t) dk[t] = dv[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int st = 0;
  for (int hh = kh * G; hh < (kh + 1) * G; ++hh) {
    const T* Q = base + (size_t)hh * dh;
    const T* dO = dout + (size_t)sv.row0 * ldo + (size_t)hh * dh;
    for (int i0 = j0; i0 < S; i0 += BT, st ^= 1) {
      const int iw = i0 + z.wave * 16;
      const size_t ir = (size_t)min(iw + z.lr, S - 1);
      f32x4_t s = {0.f, 0.f, 0.f, 0.f}, dp = s, p, d;
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        s = mma16(row4<VEC>(Q + ir * ld, c * 16 + 4 * z.g, dh), kf[c], s);
        dp = mma16(row4<VEC>(dO + ir * ldo, c * 16 + 4 * z.g, dh), vf[c], dp);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = iw + 4 * z.g + q;
        p[q] = d[q] = 0.f;
        if (i < S && j <= i) {
          const size_t at = stat_index(cu, Trows, sv, b, hh, nh, Smax, i);
          p[q] = __expf(s[q] - lse[at]);
          d[q] = p[q] * (dp[q] - delta[at]);
        }
      }
      *reinterpret_cast<f32x4_t*>(&ps[st][z.lr * PP + z.wave * 16 + 4 * z.g]) = p;
      *reinterpret_cast<f32x4_t*>(&ds[st][z.lr * PP + z.wave * 16 + 4 * z.g]) = d;
      __syncthreads();   // (as in the dQ kernel)
      second_product<kBranchBwd<T, NG, VEC>, NCT>(z, ps[st], dO, ldo, i0, S, dh, dv);
      second_product<kBranchBwd<T, NG, VEC>, NCT>(z, ds[st], Q, ld, i0, S, dh, dk);
    }
  }
  bool ask[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = j0 + 4 * z.g + q;
    ask[q] = r < S;
    if (r >= S) continue;
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
      const int col = (z.wave + 4 * t) * 16 + z.lr;
      if (col >= dh) continue;
      T* row = dqkv + ((size_t)sv.row0 + r) * ld;
      stf(row, (size_t)(nh + kh) * dh + col, dk[t][q] * scale);
      stf(row, (size_t)(nh + nkv + kh) * dh + col, dv[t][q]);
    }
  }
  uint32_t again = not_finite(z, dk, ask) | not_finite(z, dv, ask);
  if (again != 0) {   // wave-uniform
    // the queries j0 .. j - 1 meet key j with weight zero: only keys after the first of them that is not finite (a later
    // query takes every key before it with it, rightly)
    int first = BR - 1;
#pragma unroll 1
    for (int i = 0; i < first && j0 + i < S; ++i) {
      float odd = 0.f, qv[NU], dov[NU];
      for (int hh = kh * G; hh < (kh + 1) * G; ++hh) {
        channels(base + (size_t)(j0 + i) * ld + (size_t)hh * dh, z.lane, dh, qv);
        channels(dout + ((size_t)sv.row0 + j0 + i) * ldo + (size_t)hh * dh, z.lane, dh, dov);
        odd += times_zero(qv) + times_zero(dov);
      }
      if (__builtin_amdgcn_ballot_w64(odd != 0.f) != 0) first = i;
    }
    again &= ~((2u << first) - 1u);
  }
  for (; again != 0; again &= again - 1) {
    const int jr = j0 + __builtin_ctz(again);
    float kv[NU], vv[NU], qv[NU], dov[NU], ak[NU] = {0.f, 0.f, 0.f, 0.f}, av[NU] = {0.f, 0.f, 0.f, 0.f};
    channels(base + (size_t)jr * ld + (size_t)(nh + kh) * dh, z.lane, dh, kv);
    channels(base + (size_t)jr * ld + (size_t)(nh + nkv + kh) * dh, z.lane, dh, vv);
#pragma unroll
    for (int u = 0; u < NU; ++u) kv[u] *= scale;
    for (int hh = kh * G; hh < (kh + 1) * G; ++hh)
#pragma unroll 1
      for (int i = jr; i < S; ++i) {
        channels(base + (size_t)i * ld + (size_t)hh * dh, z.lane, dh, qv);
        channels(dout + ((size_t)sv.row0 + i) * ldo + (size_t)hh * dh, z.lane, dh, dov);
        const size_t at = stat_index(cu, Trows, sv, b, hh, nh, Smax, i);
        const float p = __expf(dot(qv, kv) - lse[at]), d = p * (dot(dov, vv) - delta[at]);
#pragma unroll
        for (int u = 0; u < NU; ++u) { ak[u] = fmaf(d, qv[u], ak[u]); av[u] = fmaf(p, dov[u], av[u]); }
        bool live = false;   // a sum that is not finite stays so
#pragma unroll
        for (int u = 0; u < NU; ++u) live |= own_channel(z, u, dh) && (ak[u] - ak[u] == 0.f || av[u] - av[u] == 0.f);
        if (__builtin_amdgcn_ballot_w64(live) == 0) break;
      }
    T* row = dqkv + ((size_t)sv.row0 + jr) * ld;
    wait_stores();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int col = z.lane + 64 * u;
      if (!own_channel(z, u, dh)) continue;
      stf(row, (size_t)(nh + kh) * dh + col, ak[u] * scale);
      stf(row, (size_t)(nh + nkv + kh) * dh + col, av[u]);
    }
  }
}

namespace {

bool simple_ok(const AttnArgs& a) {
  return a.dh <= kMaxDh && a.B <= 65535 && a.nh <= 65535 && a.S > 0 && a.B > 0;
}

template <typename T, int NG, bool VEC>
hipError_t fwd_simple(const AttnArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((attn_fwd_simple_kernel<T, NG, VEC>), dim3((unsigned)((a.S + BR - 1) / BR), a.nh, a.B), dim3(256), 0, s, (const T*)a.qkv, (T*)a.out,
                     a.lse, a.S, a.nh, a.nkv, a.dh, a.cu_seqlens, a.total_rows);
  return hipGetLastError();
}

template <typename T, int NG, bool VEC>
hipError_t bwd_simple(const AttnArgs& a, hipStream_t s) {
  const unsigned nb = (unsigned)((a.S + BR - 1) / BR);
  hipLaunchKernelGGL((attn_dq_simple_kernel<T, NG, VEC>), dim3(nb, a.nh, a.B), dim3(256), 0, s, (const T*)a.qkv, (const T*)a.out, (const T*)a.dout, a.lse,
                     a.delta, (T*)a.dqkv, a.S, a.nh, a.nkv, a.dh, a.cu_seqlens, a.total_rows);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_dkv_simple_kernel<T, NG, VEC>), dim3(nb, a.nkv, a.B), dim3(256), 0, s, (const T*)a.qkv, (const T*)a.dout, a.lse, a.delta,
                     (T*)a.dqkv, a.S, a.nh, a.nkv, a.dh, a.cu_seqlens, a.total_rows);
  return hipGetLastError();
}

template <typename T, int NG>
hipError_t run_simple(const AttnArgs& a, bool bwd, hipStream_t s) {
  // every row of every head starts at a multiple of dh elements: four of them are one load when dh and the bases allow it
  const bool vec = a.dh % 4 == 0 && (((uintptr_t)a.qkv | (uintptr_t)a.out | (uintptr_t)a.dout | (uintptr_t)a.dqkv) & 15) == 0;
  if (bwd) return vec ? bwd_simple<T, NG, true>(a, s) : bwd_simple<T, NG, false>(a, s);
  return vec ? fwd_simple<T, NG, true>(a, s) : fwd_simple<T, NG, false>(a, s);
}

template <typename T>
hipError_t run_simple(const AttnArgs& a, bool bwd, hipStream_t s) {
  if (a.dh <= 64) return run_simple<T, 4>(a, bwd, s);
  if (a.dh <= 128) return run_simple<T, 8>(a, bwd, s);
  return run_simple<T, 16>(a, bwd, s);
}

}  // namespace

hipError_t launch_attn_fwd_simple(const AttnArgs& a, hipStream_t s) {
  if (!simple_ok(a)) return hipErrorInvalidValue;
  ProfScope ps("attn_fwd_simple", 2.0 * a.B * a.nh * a.dh * (double)a.S * (a.S + 1), 0, s);
  return a.dtype == kBF16 ? run_simple<bf16_t>(a, false, s) : run_simple<float>(a, false, s);
}

hipError_t launch_attn_bwd_simple(const AttnArgs& a, hipStream_t s) {
  if (!simple_ok(a)) return hipErrorInvalidValue;
  ProfScope ps("attn_bwd_simple", 7.0 * a.B * a.nh * a.dh * (double)a.S * (a.S + 1), 0, s);
  return a.dtype == kBF16 ? run_simple<bf16_t>(a, true, s) : run_simple<float>(a, true, s);
}

}  // namespace tide
