// fp32 GEMM on the matrix cores: C[M,N] = epilogue(op(A) op(B)) with v_mfma_f32_32x32x2_f32, whose products and sums are fp32.  It serves the
// fp32 precision mode, any shape and alignment (large outputs of operands that cannot be read 16 bytes at a time go to the general kernel, see
// gemm_f32_pays).
//
// The products of the small fp32 configurations (128 rows, widths of 64 to 1000) are bound by latency: few tiles, short contractions.  So a
// block owns one 32x32 tile, its 4 or 8 wavefronts take the contraction in turns of 8 k, and every wavefront loads straight into
// the operand registers of the MFMAs, four turns (8 loads) in flight while the four before are multiplied; LDS only adds the wavefronts'
// partial tiles up, in a fixed order.  MFMA only needs both operands to agree on the order of k: lanes 0-31 hold k 0-3 of a
// turn, lanes 32-63 k 4-7, which is one 16-byte load where the contraction is contiguous and four loads of whole 128-byte lines where
// it is not.  Large outputs take blocks of 64x64 whose 4 wavefronts own a tile each (all of K): operands are then shared through L1.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace tfm {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct F32Params {
  int M, N, K;
  const float* A; int lda;
  const float* B; int ldb;
  float* C; int ldc;
  const float* bias; int relu; const float* mask; const float* residual;
  uint64_t drop_key; uint32_t drop_thr; float inv_keep, mask_scale;
  float* colsum;                                         // [M] sums of A's columns over K (TN only), or null
};

// Rows r0 .. r0 + 31 of an operand, 8 k at a time.  TR: the contraction is the slow index.  VEC: 16-byte loads (K, ld and base allow it).
// Rows beyond the end are the last one again (their results are not stored), k beyond the end reads zero.
template <bool TR, bool VEC>
struct F32Operand {
  const float* at;
  int ld, K, k0;
  __device__ __forceinline__ void init(const float* p, int ld_, int r0, int rows, int K_, int lane) {
    const int row = min(r0 + (lane & 31), rows - 1);
    ld = ld_; K = K_; k0 = (lane >> 5) * 4;
    at = TR ? p + row : p + (size_t)row * ld;
  }
  __device__ __forceinline__ void load(int turn, float (&v)[4]) const {
    const int k = turn * 8 + k0;
    if constexpr (!TR && VEC) {
      float4 x = {0.f, 0.f, 0.f, 0.f};
      if (k < K) x = *reinterpret_cast<const float4*>(at + k);
      v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = k + e < K ? (TR ? at[(size_t)(k + e) * ld] : at[k + e]) : 0.f;
    }
  }
};

// Tile (tm, tn) of 32 WM x 32 WN outputs; WK wavefronts share the contraction of each 32x32 part.
template <bool ATR, bool BTR, bool VEC, int WM, int WN, int WK, bool QUADS>
__device__ __forceinline__ void gemm_f32_tile(const F32Params& p, int tm, int tn) {
  constexpr int NW = WM * WN * WK, U = 4, PITCH = 36;     // (16-byte rows of the box, no bank conflicts in either pass)
  __shared__ __attribute__((aligned(16))) float box[NW][32 * PITCH];
  __shared__ float sums[NW][32];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
  const int m0 = (tm * WM + wm) * 32, n0 = (tn * WN + wn) * 32;
  F32Operand<ATR, VEC> oa;
  F32Operand<BTR, VEC> ob;
  oa.init(p.A, p.lda, m0, p.M, p.K, lane);
  ob.init(p.B, p.ldb, n0, p.N, p.K, lane);
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  float cs = 0.f;
  float a[U][4], b[U][4], a2[U][4], b2[U][4];
  auto fetch = [&](int t, float (&x)[U][4], float (&y)[U][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      oa.load((t * U + u) * WK + wk, x[u]);
      ob.load((t * U + u) * WK + wk, y[u]);
    }
  };
  auto multiply = [&](const float (&x)[U][4], const float (&y)[U][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(y[u][e], x[u][e], acc, 0, 0, 0);      // transposed product: a lane holds 4 consecutive columns
        if (ATR) cs += x[u][e];
      }
  };
  const int trips = (p.K + 8 * U * WK - 1) / (8 * U * WK);
  fetch(0, a, b);
  // QUADS (4 wavefronts or more share a tile, whole aligned quadruples of columns): a thread finishes at most one, and what the epilogue adds to it is on its
  // way with the operands.  In a trip of its own behind the sums, element by element, it was 0.5 us of a launch: X W^T with a bias 128 x 192 x 64 3.9 us, now
  // 3.3, 128 x 64 x 256 5.3 and 4.6, 512^3 8.6 and 8.0; dY W with a residual 128 x 64 x 256 4.9 and 4.4 (out of a graph, over 24 sets of operands).
  // An instance of its own: with the other epilogue in it as well, which lanes beyond N went through, 82 x 132 x 64 3.6, now 3.4.
  const int er = (wk * 64 + lane) >> 3, ec = ((wk * 64 + lane) & 7) * 4;
  float4 bias4 = {0.f, 0.f, 0.f, 0.f}, mask4 = {1.f, 1.f, 1.f, 1.f}, res4 = {0.f, 0.f, 0.f, 0.f};
  const bool mine = wk * 64 + lane < 256 && m0 + er < p.M && n0 + ec < p.N;
  if (QUADS && mine) {
    const size_t o = (size_t)(m0 + er) * p.ldc + n0 + ec;
    if (p.bias) bias4 = *reinterpret_cast<const float4*>(p.bias + n0 + ec);
    if (p.mask) mask4 = *reinterpret_cast<const float4*>(p.mask + o);
    if (p.residual) res4 = *reinterpret_cast<const float4*>(p.residual + o);
  }
  for (int t = 0; t < trips; t += 2) {                    // (turns beyond K multiply zeros)
    fetch(t + 1, a2, b2);
    multiply(a, b);
    if (t + 2 < trips) fetch(t + 2, a, b);
    if (t + 1 < trips) multiply(a2, b2);
  }
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<float4*>(&box[wave][(lane & 31) * PITCH + g * 8 + (lane >> 5) * 4]) = float4{acc[g * 4], acc[g * 4 + 1], acc[g * 4 + 2], acc[g * 4 + 3]};
  if (ATR && p.colsum && tn == 0 && wn == 0) {
    cs += __shfl_xor(cs, 32);
    if (lane < 32) sums[wave][lane] = cs;
  }
  __syncthreads();
  if (ATR && p.colsum && tn == 0 && wn == 0 && wk == 0 && lane < 32 && m0 + lane < p.M) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < WK; ++w) t += sums[wave + w][lane];
    p.colsum[m0 + lane] = t;
  }
  // 4 consecutive columns a lane
  if constexpr (QUADS) {
    if (!mine) return;
    const int m = m0 + er, n = n0 + ec;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const float4 x = *reinterpret_cast<const float4*>(&box[wave - wk + w][er * PITCH + ec]);
      v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
    }
    const float bv[4] = {bias4.x, bias4.y, bias4.z, bias4.w}, mv[4] = {mask4.x, mask4.y, mask4.z, mask4.w}, rv[4] = {res4.x, res4.y, res4.z, res4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (p.bias) v[e] += bv[e];
      if (p.relu) v[e] = fmaxf(v[e], 0.f);
    }
    if (p.drop_thr) {                                    // (a multiple of 4 columns: the four bits are of one word)
      const uint64_t word = drop_word(p.drop_key, ((uint64_t)m * p.N + n) >> 2);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = drop_keep(word, e, p.drop_thr) ? v[e] * p.inv_keep : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (p.mask) v[e] = mv[e] > 0.f ? v[e] * p.mask_scale : 0.f;
      if (p.residual) v[e] += rv[e];
    }
    *reinterpret_cast<float4*>(p.C + (size_t)m * p.ldc + n) = float4{v[0], v[1], v[2], v[3]};
    return;
  }
  for (int idx = wk * 64 + lane; idx < 256; idx += 64 * WK) {
    const int r = idx >> 3, c = (idx & 7) * 4, m = m0 + r, n = n0 + c;
    if (m >= p.M) continue;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const float4 x = *reinterpret_cast<const float4*>(&box[wave - wk + w][r * PITCH + c]);
      v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (n + e >= p.N) continue;
      const size_t o = (size_t)m * p.ldc + n + e;
      if (p.bias) v[e] += p.bias[n + e];
      if (p.relu) v[e] = fmaxf(v[e], 0.f);
      if (p.drop_thr) {
        const uint64_t i = (uint64_t)m * p.N + n + e;
        v[e] = drop_keep(drop_word(p.drop_key, i >> 2), (int)(i & 3), p.drop_thr) ? v[e] * p.inv_keep : 0.f;
      }
      if (p.mask) v[e] = p.mask[o] > 0.f ? v[e] * p.mask_scale : 0.f;
      if (p.residual) v[e] += p.residual[o];
      p.C[o] = v[e];
    }
  }
}

// (QUADS takes 12 registers.  X W^T with 4 wavefronts is held to the 128 with which 4 blocks share a compute unit: with 132 there were 3, 2000 x 512 x 64 with
// a bias 8.3 us, now 6.6.  dY W with 8 has 142 and would spill with 128: 1000 x 512 x 300 14.6 us, now 10.2.)
template <int FORM, bool VEC, int WM, int WN, int WK, bool QUADS>
__global__ __launch_bounds__(64 * WM * WN * WK, QUADS && FORM == 0 && WK == 4 ? 4 : 1) void gemm_f32_kernel(F32Params p) {
  gemm_f32_tile<FORM == 2, FORM != 0, VEC, WM, WN, WK, QUADS>(p, blockIdx.y, blockIdx.x);
}

// Weight gradients C_i = A_i^T B_i with the column sums of A_i, the tiles of many products end to end (see launch_wgrad_grouped)
struct F32Job { const float *A, *B; float *C, *colsum; int M, N, K, lda, ldb, ldc, tile_begin, tiles_n; };
struct F32Table { int n; F32Job job[WGRAD_GROUP_MAX]; };
static_assert(sizeof(F32Table) <= 4096, "kernel argument space");

template <int WM, int WN, int WK, bool QUADS>
__global__ __launch_bounds__(64 * WM * WN * WK) void gemm_f32_grouped_kernel(F32Table tab) {
  int i = 0;
  for (int j = 1; j < tab.n; ++j) i = (int)blockIdx.x >= tab.job[j].tile_begin ? j : i;
  const F32Job& g = tab.job[i];
  F32Params p{g.M, g.N, g.K, g.A, g.lda, g.B, g.ldb, g.C, g.ldc, nullptr, 0, nullptr, nullptr, 0, 0, 1.f, 1.f, g.colsum};
  const int tile = blockIdx.x - g.tile_begin;
  gemm_f32_tile<true, true, false, WM, WN, WK, QUADS>(p, tile / g.tiles_n, tile % g.tiles_n);
}

static long tiles32(int M, int N) { return (long)((M + 31) / 32) * ((N + 31) / 32); }

// us a launch out of a graph, with 64x64 LDS tiles on the vector ALUs (the general kernel) and now, X W^T / dY W / A^T B: 128 x 64 x 256 37 and 4.5 / 32 and
// 4.3 / 38 and 4.8; 128 x 64 x 1000 224 and 9.7 / 194 and 10.5 / 206 and 9.9; 512^3 93 and 7.9 / 89 and 6.9 / 107 and 7.1; with 64x64 blocks here 4096 x
// 1024 x 1024 247 and 161 (53 TFLOP/s) / 241 and 154 / 285 and 142; 2000 x 8192 x 512 365 and 323 / 377 and 269 / 368 and 282.  The error against 64 bits
// is 0.4-0.6 of the former where wavefronts share K, equal elsewhere.  Up to 1024 tiles of 32 (4 a compute unit) the small blocks keep more of the chip
// busy, small and large (before the epilogue's operands came early): 512^3 7.9 and 20.8 / 6.9 and 22.6 / 7.1 and 26.5, 1024 x 1024 x 512 25.0 and 21.0 / 22.4 and 22.8 / 22.5 and 26.8, 2000 x
// 1024 x 1024 (2016 tiles) 87 and 74 / 78 and 69 / 75 and 74; 8 wavefronts take K = 1000 in 4 trips to memory where 4 take 8, and
// below K = 256 have no second turn to take.  (16 wavefronts beyond K = 512 spill: 128 x 64 x 1000 dY W 10.6 and 14.8.)
template <int FORM, bool VEC>
static void gemm_f32_launch(hipStream_t s, const F32Params& p, bool quads) {
  const dim3 small((p.N + 31) / 32, (p.M + 31) / 32), large((p.N + 63) / 64, (p.M + 63) / 64);
#define F32_SMALL(WK) \
  do { if (quads) hipLaunchKernelGGL((gemm_f32_kernel<FORM, VEC, 1, 1, WK, true>), small, dim3(64 * WK), 0, s, p); \
       else hipLaunchKernelGGL((gemm_f32_kernel<FORM, VEC, 1, 1, WK, false>), small, dim3(64 * WK), 0, s, p); } while (0)
  if (tiles32(p.M, p.N) > 1024) hipLaunchKernelGGL((gemm_f32_kernel<FORM, VEC, 2, 2, 1, false>), large, dim3(256), 0, s, p);
  else if (p.K > 256) F32_SMALL(8);
  else F32_SMALL(4);
#undef F32_SMALL
}

static bool f32_vec(const GemmArgs& a) {
  const auto rows16 = [&](const void* q, int ld) { return ((uintptr_t)q & 15) == 0 && ld % 4 == 0; };
  return a.form != 2 && a.K % 4 == 0 && rows16(a.A, a.lda) && (a.form != 0 || rows16(a.B, a.ldb));
}

// Whether it is faster than the general kernel, which goes through LDS.  An operand with contiguous K that is read 4 bytes at a time takes four loads of
// 32 rows each where one of 16 bytes does otherwise; with blocks of 64x64, which have all of K to themselves, that is what bounds them.  us, the general
// kernel and this one, X W^T: 1642 x 7588 x 645 406 and 823, 2311 x 2623 x 2018 611 and 1196, 391 x 5104 x 191 (2080 tiles of 32) 39 and
// 48, 1119 x 1760 x 2708 (1925) 627 and 477; dY W (one such operand): 762 x 5624 x 4383 (4224) 1010 and 1512, 1785 x 1811 x 2093 (3192) 514 and 577,
// 749 x 3996 x 193 (3000) 48.0 and 44.8, 2246 x 952 x 2718 (2130) 613 and 553.
bool gemm_f32_pays(const GemmArgs& a) {
  return a.form == 2 || f32_vec(a) || tiles32(a.M, a.N) <= (a.form == 0 ? 2000 : 3100);
}

void launch_gemm_f32(hipStream_t s, const GemmArgs& a) {
  if (a.M <= 0 || a.N <= 0) return;
  const auto whole = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
  const bool quads = a.N % 4 == 0 && a.ldc % 4 == 0 && whole(a.C) && whole(a.bias) && whole(a.mask) && whole(a.residual);
  const F32Params p{a.M, a.N, a.K, (const float*)a.A, a.lda, (const float*)a.B, a.ldb, (float*)a.C, a.ldc, (const float*)a.bias, a.relu,
                    (const float*)a.mask, (const float*)a.residual, a.drop_key, a.drop_p > 0.f ? drop_threshold(a.drop_p) : 0u, 1.f / (1.f - a.drop_p),
                    a.mask_scale, nullptr};
  const bool vec = f32_vec(a);
  if (a.form == 0) { if (vec) gemm_f32_launch<0, true>(s, p, quads); else gemm_f32_launch<0, false>(s, p, quads); }
  else if (a.form == 1) { if (vec) gemm_f32_launch<1, true>(s, p, quads); else gemm_f32_launch<1, false>(s, p, quads); }
  else gemm_f32_launch<2, false>(s, p, quads);
}

void launch_wgrad_grouped_f32(hipStream_t s, const WgradJob* jobs, int n) {
  if (n <= 0) return;
  F32Table tab;
  long t32 = 0;
  int K = 0;
  for (int i = 0; i < n; ++i) { t32 += tiles32(jobs[i].M, jobs[i].N); K = std::max(K, jobs[i].K); }
  // (small and large blocks, us: 1024 tiles, K = 128 9.9 and 9.0, 512 23 and 26, 2000 72 and 93; 2048 tiles 19 and 13, 46 and 39, 139 and
  // 141; 4096 tiles 38 and 26, 91 and 76, 280 and 278)
  const bool large = t32 >= 2048;
  const int edge = large ? 64 : 32;
  int tiles = 0;
  bool quads = true;
  for (int i = 0; i < n; ++i) {
    const WgradJob& j = jobs[i];
    quads = quads && j.N % 4 == 0 && j.ldc % 4 == 0 && ((uintptr_t)j.C & 15) == 0;
    tab.job[i] = {(const float*)j.A, (const float*)j.B, (float*)j.C, (float*)j.colsum, j.M, j.N, j.K, j.lda, j.ldb, j.ldc, tiles, (j.N + edge - 1) / edge};
    tiles += tab.job[i].tiles_n * ((j.M + edge - 1) / edge);
  }
  tab.n = n;
#define F32_GROUPED(WK) \
  do { if (quads) hipLaunchKernelGGL((gemm_f32_grouped_kernel<1, 1, WK, true>), dim3(tiles), dim3(64 * WK), 0, s, tab); \
       else hipLaunchKernelGGL((gemm_f32_grouped_kernel<1, 1, WK, false>), dim3(tiles), dim3(64 * WK), 0, s, tab); } while (0)
  if (large) hipLaunchKernelGGL((gemm_f32_grouped_kernel<2, 2, 1, false>), dim3(tiles), dim3(256), 0, s, tab);
  else if (K > 256) F32_GROUPED(8);
  else F32_GROUPED(4);
#undef F32_GROUPED
}

}  // namespace tfm
