// X W^T for few rows (a decoding step, a handful of sentences): C[R,N] = epilogue(X[R,K] W[N,K]^T), R <= 64, fp16/bf16, where
// that is faster than the tiled kernel (gemm_thin_pays).
//
// Such a product is one pass over the weights, and on this chip a dependent chain: launch, one trip to memory, reduction,
// store.  The tiled kernel walks K step by step through an LDS ring (5.7 us for 4 rows of a 1024 x 1024 layer); here every load of a
// block is in flight at once (3.5 us).  A block owns 16 * NT output columns;
// its 8 wavefronts split K, fetch their weights and rows straight into the registers of 16x16x32 MFMAs (weights as the left
// operand, so that a lane ends up with 4 consecutive columns of one row), and LDS adds up the 8 partial tiles.  The contraction
// index is dealt so that a lane reads 32 and four lanes 128 contiguous bytes of a weight row: lanes of group g take
// k = 16 g .. 16 g + 15 of every 64-wide unit.  MFMA only needs both operands to agree on the order.
//
// With LN the rows are not read but made: s = x + bias + y (y in the compute dtype or as fp32 split-K slices), LayerNorm, into
// LDS, one wavefront per row.  Every block repeats that, for at most 8 rows, while its weights are on their way: 5.1 us for a
// 3072 x 1024 layer and 4 rows, against 4.3 + 4.4 us for a LayerNorm kernel and the product after it.  (16 rows a block, for
// products of more rows, cost 13.4 us against 5.0 + 5.9: a block then reads 130-260 KB of slices.)
#include <algorithm>
#include <cmath>

#include "common.h"
#include "kernels.h"

namespace tfm {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

static __device__ __forceinline__ f32x4 mfma16(half_t, u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
static __device__ __forceinline__ f32x4 mfma16(bf16_t, u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int THIN_WAVES = 8, THIN_UNIT = 64;            // wavefronts per block; K elements of a unit
constexpr int THIN_NORM_SPLITS = 4;                      // LN: slices a row's y may come in
constexpr int THIN_UNITS = 4, THIN_UNITS_4 = 3;          // units a wavefront holds, and with four tiles of rows (more never
                                                         // pays there); beside a row that it makes (LN):
constexpr int THIN_NORM_UNITS = 3, THIN_NORM_WIDE_UNITS = 2;                   // with one and with four column tiles

struct ThinParams {
  int R, N, K, kblock;                                   // kblock: K elements per blockIdx.y slice
  const uint16_t* X; int ldx;
  const uint16_t* W; int ldw;
  uint16_t* C; int ldc;
  const uint16_t* bias;
  int relu;
  float* partial;                                        // fp32 slices [gridDim.y][R][N] instead of C, or null
  ThinNorm ln;
};

template <typename T> __device__ __forceinline__ void unpack8(u32x4 r, float (&v)[8]) {
  Pack<T, 8> k;
  __builtin_memcpy(&k, &r, 16);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = to_f<T>(k.v[e]);
}

// A row of LayerNorm in the making: everything a wavefront needs for it, loaded first and looked at later.
template <typename T, int NCH> struct NormRow {
  u32x4 x[NCH], y[NCH], bias[NCH], gamma[NCH], beta[NCH];
  f32x4 part[NCH][THIN_NORM_SPLITS][2];

  __device__ __forceinline__ void load(const ThinNorm& q, int R, int d, int lane, int row) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = min((lane + 64 * c) * 8, d - 8);
      const size_t at = (size_t)row * d + col;
      x[c] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(q.x) + at);
      if (q.splits > 0) {
#pragma unroll
        for (int k = 0; k < THIN_NORM_SPLITS; ++k)
          if (k < q.splits) {
            const f32x4* src = reinterpret_cast<const f32x4*>(q.partial + (size_t)k * R * d + at);
            part[c][k][0] = src[0];
            part[c][k][1] = src[1];
          }
        if (q.bias) bias[c] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(q.bias) + col);
      } else if (q.y) y[c] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(q.y) + at);
      gamma[c] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(q.gamma) + col);
      beta[c] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(q.beta) + col);
    }
  }

  // to: the row in LDS; keeps: this block also stores the finished row
  __device__ __forceinline__ void finish(const ThinNorm& q, int d, int lane, int row, bool keeps, T* to) const {
    float v[NCH][8], sum = 0.f, sq = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      unpack8<T>(x[c], v[c]);
      if (q.splits > 0) {
        float t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = part[c][0][e >> 2][e & 3];
#pragma unroll
        for (int k = 1; k < THIN_NORM_SPLITS; ++k)
          if (k < q.splits) {
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] += part[c][k][e >> 2][e & 3];
          }
        if (q.bias) {
          float b[8];
          unpack8<T>(bias[c], b);
#pragma unroll
          for (int e = 0; e < 8; ++e) t[e] += b[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[c][e] += t[e];
      } else if (q.y) {
        float t[8];
        unpack8<T>(y[c], t);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[c][e] += t[e];
      }
      const bool in = (lane + 64 * c) * 8 < d;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (q.s_out) v[c][e] = to_f<T>(from_f<T>(v[c][e]));                    // normalise exactly what is stored
        if (in) sum += v[c][e];
      }
    }
    const float mu = wave_sum(sum) / (float)d;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      if ((lane + 64 * c) * 8 < d) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float t = v[c][e] - mu; sq += t * t; }
      }
    const float rs = rsqrtf(wave_sum(sq) / (float)d + LN_EPS);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (lane + 64 * c) * 8;
      if (col >= d) continue;
      float ga[8], be[8], o[8];
      unpack8<T>(gamma[c], ga);
      unpack8<T>(beta[c], be);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = ga[e] * ((v[c][e] - mu) * rs) + be[e];
      store_f<T, 8>(to + col, o);
      if (keeps) {
        store_f<T, 8>(reinterpret_cast<T*>(q.n_out) + (size_t)row * d + col, o);
        if (q.s_out) store_f<T, 8>(reinterpret_cast<T*>(q.s_out) + (size_t)row * d + col, v[c]);
      }
    }
  }
};

// U: units per wavefront (8 * U * 64 >= kblock).  RT: 16-row tiles.
template <typename T, int RT, int NT, int U, bool LN>
__global__ __launch_bounds__(64 * THIN_WAVES) void gemm_thin_kernel(ThinParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 16 * NT;
  const int k0 = blockIdx.y * p.kblock, kend = min(p.K, k0 + p.kblock);
  u32x4 w[U][NT][2];
  auto load_w = [&]() {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k = k0 + (wave * U + u) * THIN_UNIT + g * 16 + h * 8;
          const int n = min(n0 + j * 16 + l16, p.N - 1);
          w[u][j][h] = k < kend ? *reinterpret_cast<const u32x4*>(p.W + (size_t)n * p.ldw + k) : u32x4{0, 0, 0, 0};
        }
  };
  u32x4 x[U][RT][2];
  if constexpr (!LN) {
    load_w();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k = k0 + (wave * U + u) * THIN_UNIT + g * 16 + h * 8;
          const int r = min(i * 16 + l16, p.R - 1);
          x[u][i][h] = k < kend ? *reinterpret_cast<const u32x4*>(p.X + (size_t)r * p.ldx + k) : u32x4{0, 0, 0, 0};
        }
  } else {
    static_assert(RT == 1, "one tile of rows");
    // Loads return in order: the row's are issued ahead of the weights', which then arrive while the row is being made.
    const int d = p.K, pitch = d + 8;
    T* rows = reinterpret_cast<T*>(smem);
    NormRow<T, U> q;
    q.load(p.ln, p.R, d, lane, min(wave, p.R - 1));
    __builtin_amdgcn_sched_barrier(0);
    load_w();
    __builtin_amdgcn_sched_barrier(0);
    if (wave < p.R) q.finish(p.ln, d, lane, wave, blockIdx.x == (unsigned)wave % gridDim.x, rows + wave * pitch);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = (wave * U + u) * THIN_UNIT + g * 16 + h * 8;
        const int r = min(l16, p.R - 1);
        x[u][0][h] = k < kend ? *reinterpret_cast<const u32x4*>(rows + r * pitch + k) : u32x4{0, 0, 0, 0};
      }
    __syncthreads();                                     // (the partial tiles below re-use the LDS)
  }
  f32x4 acc[RT][NT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = mfma16(T{}, w[u][j][h], x[u][i][h], acc[i][j]);
  f32x4* red = reinterpret_cast<f32x4*>(smem);           // [wavefront][tile][lane]
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) red[(wave * RT * NT + i * NT + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  for (int q = tid; q < RT * NT * 64; q += 64 * THIN_WAVES) {
    f32x4 s = red[q];
#pragma unroll
    for (int k = 1; k < THIN_WAVES; ++k) {
      const f32x4 t = red[k * RT * NT * 64 + q];
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += t[e];
    }
    const int tile = q >> 6, ql = q & 63;
    const int r = tile / NT * 16 + (ql & 15), n = n0 + tile % NT * 16 + (ql >> 4) * 4;
    if (r >= p.R || n >= p.N) continue;
    float o[4] = {s[0], s[1], s[2], s[3]};
    if (p.partial) {
      store_f<float, 4>(p.partial + ((size_t)blockIdx.y * p.R + r) * p.N + n, o);
      continue;
    }
    if (p.bias) {
      float b[4];
      load_f<T, 4>(reinterpret_cast<const T*>(p.bias) + n, b);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] += b[e];
    }
    if (p.relu) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaxf(o[e], 0.f);
    }
    store_f<T, 4>(reinterpret_cast<T*>(p.C) + (size_t)r * p.ldc + n, o);
  }
}

// U: the most units a wavefront may hold, which the callers' limits on K keep to
template <typename T, int RT, int NT, bool LN, int U>
static void thin_launch(hipStream_t s, const ThinParams& p, int splits) {
  if constexpr (U > 1) {
    if (p.kblock <= (U - 1) * THIN_WAVES * THIN_UNIT) { thin_launch<T, RT, NT, LN, U - 1>(s, p, splits); return; }
  }
  const dim3 grid((p.N + 16 * NT - 1) / (16 * NT), splits), block(64 * THIN_WAVES);
  size_t sh = (size_t)THIN_WAVES * RT * NT * 1024;
  if (LN) sh = std::max(sh, (size_t)p.R * (p.K + 8) * 2);
  hipLaunchKernelGGL((gemm_thin_kernel<T, RT, NT, U, LN>), grid, block, sh, s, p);
}
// How a product is cut: 16-row tiles rt and 16-column tiles nt of a block, blocks along N, slices of K and their length.
struct ThinPlan { int rt, nt, blocks, splits, kblock; bool defer; };
static int thin_least_splits(int K) {
  constexpr int most = THIN_UNITS * THIN_WAVES * THIN_UNIT;
  return (K + most - 1) / most;
}
// Enough columns for a block to own several tiles of them, us with several / with one, K = 512: 16 rows N = 4096 5.0 / 3.8, 8192
// 5.3 / 4.9, 16384 6.7 / 7.3, 65536 12.9 / 17.5; 64 rows N = 4096 5.9 / 5.4, 8192 6.4 / 7.9, 65536 26 / 39.  K = 768 and 1024 alike.
static bool thin_wide(int N) { return N >= 8192; }
static ThinPlan thin_plan(const GemmArgs& a) {
  ThinPlan q;
  const bool wide = thin_wide(a.N);
  q.rt = a.M <= 16 ? 1 : a.M <= 32 ? 2 : 4;
  q.nt = !wide ? 1 : q.rt < 4 ? 4 : 2;
  q.blocks = (a.N + 16 * q.nt - 1) / (16 * q.nt);
  // Deferred (the next kernel adds the slices up, with the residual): the result stays in fp32 even as a single slice, so that no
  // contraction is too short for the sum to be taken in 32 bits.  A narrow output has few blocks, and slices of K of at least one
  // unit per wavefront then fill the chip.  Otherwise only a contraction of more than 4 units per wavefront is cut.  (No ReLU in a
  // deferred reduction.)
  const int least = 64 * THIN_WAVES, need = thin_least_splits(a.K);
  const size_t slice = (size_t)a.M * a.N * 4;
  q.defer = a.deferred_splits && !a.relu && a.splitk_ws && need * slice <= a.splitk_ws_bytes;
  int splits = need;
  if (q.defer) {
    splits = std::max(splits, std::min(std::min(256 / ((a.N + 15) / 16), a.K / least), 4));
    while (splits > need && splits * slice > a.splitk_ws_bytes) --splits;
  }
  q.kblock = ((a.K + splits - 1) / splits + least - 1) / least * least;
  q.splits = (a.K + q.kblock - 1) / q.kblock;
  return q;
}

template <typename T>
static void thin_dispatch(hipStream_t s, const ThinParams& p, const ThinPlan& q) {
#define THIN(RT, NT) thin_launch<T, RT, NT, false, RT == 4 ? THIN_UNITS_4 : THIN_UNITS>(s, p, q.splits)
  if (q.rt == 1) { if (q.nt == 4) THIN(1, 4); else THIN(1, 1); }
  else if (q.rt == 2) { if (q.nt == 4) THIN(2, 4); else THIN(2, 1); }
  else { if (q.nt == 2) THIN(4, 2); else THIN(4, 1); }
#undef THIN
}
// LN with 4 column tiles: up to 2 units a wavefront (K = 1024); beyond, the row in the making and the weights no longer fit
// 256 registers (100-430 spilled).  A decoder-only model of 6 blocks, width 1536, inner size 8192, 32 steps: 1 row 10.7 -> 10.1 ms,
// 8 rows 12.5 -> 11.7 with a column tile each; inner size 6144, where only the vocabulary is that wide: equal within the spread.
template <typename T>
static void thin_norm_dispatch(hipStream_t s, const ThinParams& p, bool wide) {
  if (wide && p.K <= THIN_NORM_WIDE_UNITS * THIN_WAVES * THIN_UNIT) thin_launch<T, 1, 4, true, THIN_NORM_WIDE_UNITS>(s, p, 1);
  else thin_launch<T, 1, 1, true, THIN_NORM_UNITS>(s, p, 1);
}

// What the kernel takes: X W^T, at most THIN_ROWS rows, no epilogue but bias and ReLU.  Slices are at most 4 units per
// wavefront, so a longer contraction needs the split-K workspace.  (Alignment and strides as gemm_mfma_supported.)
bool gemm_thin_supported(const GemmArgs& a) {
  if (a.form != 0 || a.M > THIN_ROWS || a.mask || a.residual || a.drop_p != 0.f) return false;
  const int least = thin_least_splits(a.K);
  return least == 1 || (least <= DEFERRED_SPLITS_MAX && a.splitk_ws && (size_t)least * a.M * a.N * 4 <= a.splitk_ws_bytes);
}
// Whether it is faster than the tiled kernel.  Both wait for what a compute unit has to fetch, some 33 KiB per us: here 256 blocks
// at a time, each its weights and all the rows again, and 1 KiB a row more for the sums of the wavefronts (20 for the reduction of slices);
// there 512 tiles at a time, whose 64 rows are no more than that.  The tiled kernel pays 60 KiB more for its start, and with few tiles 100 for
// the walk through a longer K in a ring, or for the reduction of its slices; where the slices are added up by somebody else it has more and
// shorter ones, and 60 KiB are all that is left.  Measured alone, us here / there: 4 rows of 1024 x 1024 3.5 / 5.7; of 3072 x 1024 32 rows 5.3 / 6.0, 64
// 7.2 / 6.1; of 1536 x 512 48 rows 4.5 / 4.6; of 5120 x 1280 12 rows 7.3 / 8.6, 20 8.9 / 8.8; of 6144 x 1536 16 8.9 / 10.2; of 32768 x 1024 6 13.2 / 13.3,
// 16 14.5 / 13.6, 48 23.6 / 15.2; of 207744 x 64 16 10.5 / 19.0, 32 16.6 / 19.6, 48 27.3 / 20.7; deferred, of 1024 x 1024 32 3.7 / 3.6, 64 4.7 / 3.8, of
// 1024 x 4096 16 4.3 / 4.4, 32 5.3 / 4.5.  Over 930 products of 1 to 64 rows, N 64 to 207744 and K 64 to 8192, it loses 0.5 % to the better of
// both and is more than 5 % behind it in 33 (always this kernel: 7 % and 279, never: 16 % and 505); deferred, 603 products, 1.2 % and 53 (12 % and
// 298, 5 % and 176).  In decoder-only models of width 512 to 2048, 9 to 64 rows, where the weights come from memory if there are more than 256 MB of
// them and the slices' reduction is in the next kernel, each kind of product on either kernel: 0.35 % of the step (5.8 and 6.2 %).
bool gemm_thin_pays(const GemmArgs& a) {
  const ThinPlan q = thin_plan(a);
  if (q.rt == 4 && q.kblock > THIN_UNITS_4 * THIN_WAVES * THIN_UNIT) return false;
  if (q.defer && !gemm_mfma_slices(a)) return true;      // (a sum that the next kernel is to take in 32 bits: there it would leave 2-byte values)
  const double kib = 1024.0, tiles = (a.N + 63) / 64, rounds = std::ceil(q.blocks * q.splits / 256.0);
  const double per_row = rounds * std::min(q.kblock, a.K) * 2.0;
  const double there = (tiles <= 512 ? tiles / 512 : std::ceil(tiles / 512)) * 256.0 * a.K;
  if (q.defer) return per_row * (16 * q.nt + 16 * q.rt) <= 1.15 * there + 60 * kib;
  return per_row * (16 * q.nt + a.M) + (a.M + (q.splits > 1 ? 20 : 0)) * kib <= there + (tiles <= 96 && a.K >= 512 ? 160 : 60) * kib;
}
// ... and with the rows made by the product itself: a wavefront each (8 rows of at most 1536 values: 25 KB of LDS), the contraction
// in one slice.  32 steps of a decoder-only model of 6 blocks (inner size 4 times the width, vocabulary 32768), ms with the rows made
// inside / by a LayerNorm kernel, for 1, 4 and 8 rows: width 512 5.0 / 6.1, 5.3 / 6.4, 5.8 / 6.6; 768 5.7 / 7.0, 6.0 / 7.5, 6.6 / 7.9;
// 1024 6.0 / 7.4, 6.4 / 7.8, 6.9 / 7.9; 1536 9.5 / 9.8, 9.8 / 10.4, 11.1 / 10.6.  At 2048, 4 units a wavefront, 60-100 registers were
// spilled (inner size 8192: 15.2 / 12.7 and 18.9 / 13.6 for 1 and 8 rows).
bool gemm_thin_norm_supported(const GemmArgs& a, const ThinNorm& q) {
  return gemm_mfma_supported(a) && gemm_thin_supported(a) && a.M <= THIN_WAVES && a.K <= THIN_NORM_UNITS * THIN_WAVES * THIN_UNIT &&
         q.splits <= THIN_NORM_SPLITS;
}

static ThinParams thin_params(const GemmArgs& a) {
  ThinParams p{};
  p.R = a.M; p.N = a.N; p.K = a.K;
  p.X = (const uint16_t*)a.A; p.ldx = a.lda; p.W = (const uint16_t*)a.B; p.ldw = a.ldb; p.C = (uint16_t*)a.C; p.ldc = a.ldc;
  p.bias = (const uint16_t*)a.bias; p.relu = a.relu;
  return p;
}

// (C complete, one slice: the split-K workspace may hold the slices that the rows are made from)
void launch_gemm_thin_norm(hipStream_t s, const GemmArgs& a, const ThinNorm& q) {
  ThinParams p = thin_params(a);
  p.ln = q;
  p.kblock = (a.K + 64 * THIN_WAVES - 1) / (64 * THIN_WAVES) * (64 * THIN_WAVES);
  if (a.dt == F16) thin_norm_dispatch<half_t>(s, p, thin_wide(a.N));
  else thin_norm_dispatch<bf16_t>(s, p, thin_wide(a.N));
}

void launch_gemm_thin(hipStream_t s, const GemmArgs& a) {
  ThinParams p = thin_params(a);
  const ThinPlan q = thin_plan(a);
  p.kblock = q.kblock;
  p.partial = q.splits > 1 || q.defer ? (float*)a.splitk_ws : nullptr;
  if (a.dt == F16) thin_dispatch<half_t>(s, p, q); else thin_dispatch<bf16_t>(s, p, q);
  if (a.deferred_splits) *a.deferred_splits = q.defer ? q.splits : 0;
  if (q.splits > 1 && !q.defer) launch_splitk_reduce(s, a.dt, p.partial, q.splits, a.M, a.N, a.C, a.ldc, a.bias, a.relu);
}

}  // namespace tfm
