// Residual + dropout + LayerNorm forward and backward, and column sums (bias gradients).  All HBM-bound: one
// wavefront owns one row, each lane moves 8 contiguous elements per access (16 bytes in half precision), the row
// stays in registers between the statistics and the normalisation, statistics are fp32.
#include "common.h"
#include "kernels.h"

namespace tfm {

constexpr int LN_VEC = 8;

// s = x + drop(y); n = gamma * (s - mean) * rstd + beta.  NCH = chunks of 8 elements per lane (d <= NCH * 512), WAVES rows per block.
// Bound by memory, a few hundred rows by one trip to it: everything a row needs is asked for before the first of it is looked at.  (gamma and beta
// only after the statistics, and a chunk at a time: 280 x 1024 3.4 us against 3.0, 1020 x 1024 5.0 and 4.2, 900 x 1536 6.2 and 5.0, 3000 x 1536 11.1 and
// 10.6; more rows: see ln_fwd_by_chunks.  1, 2 or 8 rows a block: 1020 x 1024 4.4, 4.7 and 4.6.)
// y comes in the compute dtype (MAXS = 0; or null), or as bias + the sum of fp32 slices, at most MAXS of them (the last one is asked for again where
// there are fewer: with a branch around every slice the second 512 columns waited for the first, 24 rows x 1024, 4 slices 4.8 us against 3.2).  mean,
// rstd: null in a decoding step, which has an instance without them and without dropout (TRAIN = false), and a wavefront a block, whose row is then in
// scalar registers and needs no test: 5-12 % together, 268 rows x 1024, 3 slices 3.9 us, now 3.5.
template <typename T, int NCH, int MAXS, int WAVES, bool TRAIN>
__global__ __launch_bounds__(64 * WAVES) void layernorm_fwd_row_kernel(
    const T* __restrict__ x, const T* __restrict__ y, const float* __restrict__ partial, int splits, const T* __restrict__ bias,
    const T* __restrict__ gamma, const T* __restrict__ beta, T* __restrict__ s_out, T* __restrict__ n_out, float* __restrict__ mean,
    float* __restrict__ rstd, int rows, int d, uint64_t key, uint32_t thr, float inv_keep) {
  const int lane = threadIdx.x & 63, row = WAVES == 1 ? (int)blockIdx.x : (int)(blockIdx.x * WAVES + (threadIdx.x >> 6));
  if (WAVES > 1 && row >= rows) return;
  const size_t base = (size_t)row * d, slice = (size_t)rows * d;
  Pack<T, LN_VEC> xr[NCH], yr[NCH], gr[NCH], br[NCH], hr[NCH];
  float4 t[NCH][MAXS > 0 ? MAXS : 1][2];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = min((lane + 64 * c) * LN_VEC, d - LN_VEC);
    xr[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>(x + base + col);
    if constexpr (MAXS > 0) {
#pragma unroll
      for (int k = 0; k < MAXS; ++k) {
        const float4* p = reinterpret_cast<const float4*>(partial + min(k, splits - 1) * slice + base + col);
        t[c][k][0] = p[0];
        t[c][k][1] = p[1];
      }
      hr[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>((bias ? bias : gamma) + col);
    } else {
      yr[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>((y ? y : x) + base + col);
    }
    gr[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>(gamma + col);
    br[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>(beta + col);
  }
  __builtin_amdgcn_sched_barrier(0);
  float v[NCH][LN_VEC];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (lane + 64 * c) * LN_VEC;
    if (col < d) {
      float u[LN_VEC];
      if constexpr (MAXS > 0) {
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) u[i] = (&t[c][0][i >> 2].x)[i & 3];
#pragma unroll
        for (int k = 1; k < MAXS; ++k)                    // in order
          if (k < splits) {
#pragma unroll
            for (int i = 0; i < LN_VEC; ++i) u[i] += (&t[c][k][i >> 2].x)[i & 3];
          }
        if (bias) {
#pragma unroll
          for (int i = 0; i < LN_VEC; ++i) u[i] += to_f<T>(hr[c].v[i]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) u[i] = to_f<T>(yr[c].v[i]);
      }
      if (TRAIN && thr) drop_apply<LN_VEC>(u, key, base + col, thr, inv_keep);
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) v[c][i] = MAXS > 0 || y ? to_f<T>(xr[c].v[i]) + u[i] : to_f<T>(xr[c].v[i]);
      if (s_out) {
        store_f<T, LN_VEC>(s_out + base + col, v[c]);
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) v[c][i] = to_f<T>(from_f<T>(v[c][i]));     // the backward pass reads the stored sum: normalise exactly that
      }
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) sum += v[c][i];
    }
  }
  const float mu = wave_sum(sum) / (float)d;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (lane + 64 * c) * LN_VEC;
    if (col < d) {
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) { const float u = v[c][i] - mu; sq += u * u; }
    }
  }
  const float rs = rsqrtf(wave_sum(sq) / (float)d + LN_EPS);
  if (TRAIN && mean && lane == 0) { mean[row] = mu; rstd[row] = rs; }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (lane + 64 * c) * LN_VEC;
    if (col < d) {
      float o[LN_VEC];
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) o[i] = to_f<T>(gr[c].v[i]) * ((v[c][i] - mu) * rs) + to_f<T>(br[c].v[i]);
      store_f<T, LN_VEC>(n_out + base + col, o);
    }
  }
}

// The same with y in the compute dtype, a chunk at a time and gamma and beta behind the statistics: faster for the rows of ln_fwd_by_chunks.
template <typename T, int NCH>
__global__ __launch_bounds__(256) void layernorm_fwd_chunks_kernel(
    const T* __restrict__ x, const T* __restrict__ y, const T* __restrict__ gamma, const T* __restrict__ beta,
    T* __restrict__ s_out, T* __restrict__ n_out, float* __restrict__ mean, float* __restrict__ rstd, int rows, int d,
    uint64_t key, uint32_t thr, float inv_keep) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const size_t base = (size_t)row * d;
  float v[NCH][LN_VEC];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (lane + 64 * c) * LN_VEC;
    if (col < d) {
      load_f<T, LN_VEC>(x + base + col, v[c]);
      if (y) {
        float t[LN_VEC];
        load_f<T, LN_VEC>(y + base + col, t);
        if (thr) drop_apply<LN_VEC>(t, key, base + col, thr, inv_keep);
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) v[c][i] += t[i];
      }
      if (s_out) {
        store_f<T, LN_VEC>(s_out + base + col, v[c]);
        // the backward pass reads the stored (rounded) sum, so normalise exactly that
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) v[c][i] = to_f<T>(from_f<T>(v[c][i]));
      }
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) sum += v[c][i];
    }
  }
  const float mu = wave_sum(sum) / (float)d;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (lane + 64 * c) * LN_VEC;
    if (col < d) {
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) { const float t = v[c][i] - mu; sq += t * t; }
    }
  }
  const float rs = rsqrtf(wave_sum(sq) / (float)d + LN_EPS);
  if (mean && lane == 0) { mean[row] = mu; rstd[row] = rs; }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (lane + 64 * c) * LN_VEC;
    if (col < d) {
      float g[LN_VEC], b[LN_VEC], o[LN_VEC];
      load_f<T, LN_VEC>(gamma + col, g);
      load_f<T, LN_VEC>(beta + col, b);
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) o[i] = g[i] * ((v[c][i] - mu) * rs) + b[i];
      store_f<T, LN_VEC>(n_out + base + col, o);
    }
  }
}

template <typename T, int MAXS>
static void splitk_ln_dispatch(hipStream_t s, const SplitkNorm& q, int rows, int d, uint64_t key, float p) {
  const uint32_t thr = p > 0.f ? drop_threshold(p) : 0u;
  const float inv_keep = 1.f / (1.f - p);
  const int nch = (d + 511) / 512;
#define SLN_EITHER(N, TRAIN)                                                                                                                \
  hipLaunchKernelGGL((layernorm_fwd_row_kernel<T, N, MAXS, 1, TRAIN>), dim3(rows), dim3(64), 0, s, (const T*)q.x, (const T*)nullptr, q.partial, q.splits, \
                     (const T*)q.bias, (const T*)q.gamma, (const T*)q.beta, (T*)q.s_out, (T*)q.n_out, q.mean, q.rstd, rows, d, key, thr, inv_keep)
#define SLN(N) do { if (q.mean || thr) SLN_EITHER(N, true); else SLN_EITHER(N, false); } while (0)
  if (nch <= 1) SLN(1); else if (nch == 2) SLN(2); else if (nch == 3) SLN(3); else SLN(4);
#undef SLN_EITHER
#undef SLN
}
template <typename T>
static void splitk_ln_splits(hipStream_t s, const SplitkNorm& q, int rows, int d, uint64_t key, float p) {
  static_assert(DEFERRED_SPLITS_MAX == 8, "the widest instance");
  if (q.splits <= 2) splitk_ln_dispatch<T, 2>(s, q, rows, d, key, p);
  else if (q.splits <= 4) splitk_ln_dispatch<T, 4>(s, q, rows, d, key, p);
  else splitk_ln_dispatch<T, 8>(s, q, rows, d, key, p);
}
void launch_splitk_layernorm_fwd(hipStream_t s, int dt, const SplitkNorm& q, int rows, int d, uint64_t key, float p) {
  if (rows <= 0) return;
  if (dt == F16) splitk_ln_splits<half_t>(s, q, rows, d, key, p);
  else if (dt == BF16) splitk_ln_splits<bf16_t>(s, q, rows, d, key, p);
  // (split-K launches exist for the 2-byte types only)
}

// Some 3 to 4 blocks of 4 rows a compute unit are all there at once, ask for everything at once and then store at once: reads and writes overlap less
// than where a wavefront works chunk by chunk.  Fewer blocks are bound by the trips to memory, of more the later ones overlap the earlier.  us in one trip /
// by chunks:
//   fp16 3000 x 1024  8.4/ 8.5  3264  9.3/ 8.9  4224 10.4/10.3  6000 12.8/12.7  8000 15.0/15.0      bf16 4224 10.4/10.1  6000 12.9/12.7
//        3000 x 1536 10.7/11.3  3264 12.2/12.0  4224 14.8/13.8  5000 15.2/15.2  6000 17.7/18.3
//        3000 x 2048 12.9/13.9  3264 15.6/14.8  4224 17.7/17.3  5000 18.7/20.1          up to 768 columns one trip throughout
//   fp32 2000 x 1024 10.1/10.3  2600 13.4/12.6  3600 16.2/15.6  4000 15.8/15.9  4224 18.1/19.8
//        1020 x 1536  8.9/ 9.5  2000 13.9/13.7  2600 18.1/16.3  3600 22.9/22.2  4000 23.4/24.0          up to 512 columns equal
//        1020 x 2048 11.1/12.1  1200 14.6/14.1  2600 23.0/20.9  3600 29.9/28.4  4000 29.2/30.3
// and without y, where the one trip asks for x twice: 512 columns, 2000 / 4000 rows fp16 3.7/3.6 and 5.1/4.8, fp32 5.0/5.0 and 9.6/9.2; wider rows within 2 %.
static bool ln_fwd_by_chunks(int dt, int rows, int d, bool y) {
  if (!y && d <= 512) return true;
  if (dt == F32) return d > 512 && rows > (d > 1024 ? 1024 : 2048) && rows <= 3840;
  return d > 768 && rows > 3072 && rows <= (d <= 1024 ? 6144 : 4352);
}
template <typename T>
static void ln_fwd_dispatch(hipStream_t s, int dt, const void* x, const void* y, const void* gamma, const void* beta, void* s_out,
                            void* n_out, float* mean, float* rstd, int rows, int d, uint64_t key, float p) {
  constexpr int WAVES = 4;
  const uint32_t thr = (p > 0.f && y) ? drop_threshold(p) : 0u;
  const float inv_keep = 1.f / (1.f - p);
  const int nch = (d + 511) / 512;
#define LN_FWD(N)                                                                                                                              \
  hipLaunchKernelGGL((layernorm_fwd_row_kernel<T, N, 0, WAVES, true>), dim3((rows + WAVES - 1) / WAVES), dim3(64 * WAVES), 0, s, (const T*)x, (const T*)y, \
                     (const float*)nullptr, 0, (const T*)nullptr, (const T*)gamma, (const T*)beta, (T*)s_out, (T*)n_out, mean, rstd, rows, d, key, \
                     thr, inv_keep)
#define LN_FWD_CHUNKS(N)                                                                                                                        \
  hipLaunchKernelGGL((layernorm_fwd_chunks_kernel<T, N>), dim3((rows + WAVES - 1) / WAVES), dim3(64 * WAVES), 0, s, (const T*)x, (const T*)y, \
                     (const T*)gamma, (const T*)beta, (T*)s_out, (T*)n_out, mean, rstd, rows, d, key, thr, inv_keep)
  if (ln_fwd_by_chunks(dt, rows, d, y != nullptr)) { if (nch <= 1) LN_FWD_CHUNKS(1); else if (nch == 2) LN_FWD_CHUNKS(2); else if (nch == 3) LN_FWD_CHUNKS(3); else LN_FWD_CHUNKS(4); }
  else if (nch <= 1) LN_FWD(1); else if (nch == 2) LN_FWD(2); else if (nch == 3) LN_FWD(3); else LN_FWD(4);
#undef LN_FWD
#undef LN_FWD_CHUNKS
}

void launch_residual_layernorm_fwd(hipStream_t s, int dt, const void* x, const void* y, const void* gamma,
                                   const void* beta, void* s_out, void* n_out, float* mean, float* rstd, int rows,
                                   int d, uint64_t key, float p) {
  if (rows <= 0) return;
  if (dt == F32) ln_fwd_dispatch<float>(s, dt, x, y, gamma, beta, s_out, n_out, mean, rstd, rows, d, key, p);
  else if (dt == F16) ln_fwd_dispatch<half_t>(s, dt, x, y, gamma, beta, s_out, n_out, mean, rstd, rows, d, key, p);
  else ln_fwd_dispatch<bf16_t>(s, dt, x, y, gamma, beta, s_out, n_out, mean, rstd, rows, d, key, p);
}

// ---- backward -----------------------------------------------------------------------------------------------------------
// Per row: xhat = (s - mean) rstd; dxhat = dn * gamma; ds = rstd (dxhat - mean(dxhat) - xhat mean(dxhat xhat)) + add.
// Column partial sums (dgamma = sum dn xhat, dbeta = sum dn, dbias = sum dropout-backward(ds)) are kept in registers
// while a wavefront walks its rows, combined across the block's 8 wavefronts in LDS (one quantity at a time, so the
// LDS footprint stays at 8 rows), and written once per block to partial[block][3][d]; a second kernel adds the
// partials in a fixed order.  One block per CU, 8 wavefronts each, keeps enough rows in flight to cover HBM latency.
constexpr int LNB_MAX_BLOCKS = 256;
constexpr int LNB_WAVES = 8;

template <typename T, int NCH>
__global__ __launch_bounds__(64 * LNB_WAVES) void layernorm_bwd_kernel(
    const T* __restrict__ dn, const T* __restrict__ add, const T* __restrict__ sres, const float* __restrict__ mean,
    const float* __restrict__ rstd, const T* __restrict__ gamma, T* __restrict__ ds, T* __restrict__ ds_drop,
    float* __restrict__ partial, int rows, int d, uint64_t key, uint32_t thr, float inv_keep, int nk) {
  extern __shared__ float lds[];     // [LNB_WAVES][d]
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float g[NCH][LN_VEC], ag[NCH][LN_VEC], ab[NCH][LN_VEC], ac[NCH][LN_VEC];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (lane + 64 * c) * LN_VEC;
    if (col < d) load_f<T, LN_VEC>(gamma + col, g[c]);
#pragma unroll
    for (int i = 0; i < LN_VEC; ++i) ag[c][i] = ab[c][i] = ac[c][i] = 0.f;
  }
  // The next row's operands are fetched into registers before the current row's reductions, so a wavefront always has
  // a full row of loads in flight.
  float a[NCH][LN_VEC], b[NCH][LN_VEC], t[NCH][LN_VEC];
  const int rstep = gridDim.x * LNB_WAVES;
  int row = blockIdx.x * LNB_WAVES + w;
  auto fetch = [&](int r, float (&fa)[NCH][LN_VEC], float (&fb)[NCH][LN_VEC], float (&ft)[NCH][LN_VEC]) {
    const size_t base = (size_t)r * d;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (lane + 64 * c) * LN_VEC;
      if (col < d) {
        load_f<T, LN_VEC>(dn + base + col, fa[c]);
        load_f<T, LN_VEC>(sres + base + col, fb[c]);
        if (add) load_f<T, LN_VEC>(add + base + col, ft[c]);
      }
    }
  };
  if (row < rows) fetch(row, a, b, t);
  for (; row < rows; row += rstep) {
    const size_t base = (size_t)row * d;
    const float mu = mean[row], rs = rstd[row];
    float xh[NCH][LN_VEC], dxh[NCH][LN_VEC], tt[NCH][LN_VEC];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (lane + 64 * c) * LN_VEC;
      if (col < d) {
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) {
          xh[c][i] = (b[c][i] - mu) * rs;
          dxh[c][i] = a[c][i] * g[c][i];
          s1 += dxh[c][i];
          s2 += dxh[c][i] * xh[c][i];
          ag[c][i] += a[c][i] * xh[c][i];
          ab[c][i] += a[c][i];
          tt[c][i] = t[c][i];
        }
      }
    }
    if (row + rstep < rows) fetch(row + rstep, a, b, t);
    const float c1 = wave_sum(s1) / (float)d, c2 = wave_sum(s2) / (float)d;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (lane + 64 * c) * LN_VEC;
      if (col < d) {
        float o[LN_VEC];
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) o[i] = rs * (dxh[c][i] - c1 - xh[c][i] * c2);
        if (add) {
#pragma unroll
          for (int i = 0; i < LN_VEC; ++i) o[i] += tt[c][i];
        }
        store_f<T, LN_VEC>(ds + base + col, o);
        if (thr) {
          drop_apply<LN_VEC>(o, key, base + col, thr, inv_keep);
          store_f<T, LN_VEC>(ds_drop + base + col, o);
        }
        // the consumers read the rounded value; sum exactly what they will see
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) ac[c][i] += to_f<T>(from_f<T>(o[i]));
      }
    }
  }
  for (int k = 0; k < nk; ++k) {                        // nk = 2: the bias sum is not wanted
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (lane + 64 * c) * LN_VEC;
      if (col < d) {
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) lds[w * d + col + i] = k == 0 ? ag[c][i] : (k == 1 ? ab[c][i] : ac[c][i]);
      }
    }
    __syncthreads();
    for (int col = threadIdx.x; col < d; col += 64 * LNB_WAVES) {
      float t = 0.f;
#pragma unroll
      for (int ww = 0; ww < LNB_WAVES; ++ww) t += lds[ww * d + col];
      partial[((size_t)blockIdx.x * 3 + k) * d + col] = t;
    }
  }
}

// Column held by slot p of the row kernel's LDS / partial layout: lane l keeps elements i = 0..7 of 8-vector
// l + 64 c in slot c * 512 + i * 64 + l, so that a wavefront's stores of one element hit 64 different banks
// (storing a lane's 8 values side by side would be an 8-way conflict, 16 wavefronts deep).  d must be a multiple of 512.
__host__ __device__ __forceinline__ int ln_slot_column(int p) { return ((p & 63) + 64 * (p >> 9)) * 8 + ((p >> 6) & 7); }

// What is done with a value stays behind this place, and so do the loads of everything made opaque ahead of it.  (A barrier for the scheduler comes late: the
// additions of bf16 rows, made of integer shifts, had moved up between the loads by then, see layernorm_bwd_row_kernel.)
template <typename P> __device__ __forceinline__ void opaque(P& x) {
  typedef uint32_t words __attribute__((ext_vector_type(4)));
  words w[sizeof(P) / 16];
  __builtin_memcpy(w, &x, sizeof(P));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(P) / 16); ++i) asm volatile("" : "+v"(w[i]));
  __builtin_memcpy(&x, w, sizeof(P));
}

// The same computation when every row can have a wavefront of its own: WAVES of them per block (see lnr_waves), one row each, no loop.  Nothing is
// accumulated across rows, so the three per-column
// quantities go from the row's registers straight into the block's LDS reduction, the register footprint stays below
// 128 (without slices) and a row's two dependent passes are the whole critical path.  (d = 512 NCH: every lane has all its columns.)
// MAXS > 0: the incoming gradient is dn (or nothing, if null) + the sum of at most MAXS fp32 slices (launch_layernorm_bwd).
template <typename T, int NCH, int WAVES, int MAXS>
__global__ __launch_bounds__(64 * WAVES) void layernorm_bwd_row_kernel(
    const T* __restrict__ dn, const float* __restrict__ slices, int splits, const T* __restrict__ add, const T* __restrict__ sres, const float* __restrict__ mean,
    const float* __restrict__ rstd, const T* __restrict__ gamma, T* __restrict__ ds, T* __restrict__ ds_drop,
    float* __restrict__ partial, int rows, int d, uint64_t key, uint32_t thr, float inv_keep, int nk) {
  __shared__ float lds[2][WAVES][512];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = blockIdx.x * WAVES + w;
  const bool live = row < rows;
  const size_t base = (size_t)(live ? row : 0) * d;
  float a[NCH][LN_VEC], xh[NCH][LN_VEC], o[NCH][LN_VEC];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int i = 0; i < LN_VEC; ++i) a[c][i] = xh[c][i] = o[c][i] = 0.f;
  if (live) {
    // The row's operands in one trip to memory.  (A part of `add`, or all of it, the compiler asks for behind the sums, in the branch that reads it, but in
    // the instances with opaque operands.)
    const float mu = mean[row], rs = rstd[row];
    Pack<T, LN_VEC> ar[NCH], br[NCH], gr[NCH], tr[NCH];
    float4 sl[NCH][MAXS > 0 ? MAXS : 1][2];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (lane + 64 * c) * LN_VEC;
      ar[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>((MAXS == 0 || dn ? dn : sres) + base + col);
      br[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>(sres + base + col);
      tr[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>((add ? add : sres) + base + col);
#pragma unroll
      for (int k = 0; k < MAXS; ++k) {                    // (past the end: the last one again)
        const float4* p = reinterpret_cast<const float4*>(slices + (size_t)min(k, splits - 1) * rows * d + base + col);
        sl[c][k][0] = p[0];
        sl[c][k][1] = p[1];
      }
      gr[c] = *reinterpret_cast<const Pack<T, LN_VEC>*>(gamma + col);
    }
    __builtin_amdgcn_sched_barrier(0);
    // bf16 rows with slices otherwise come in up to 20 groups of loads, each waited for before the next.  us without / with, and with an `add` (128 x
    // 1024, 8 slices 6.3/5.8 and 6.6/5.9; 256 x 1024, 4 slices 5.2/5.0 and 5.5/5.2; 290 x 1024, 3 slices 5.2/5.0 and 5.5/5.1; 512 columns equal).  At 1536
    // columns the groups are the better order: 64 rows, 8 slices 7.3/7.7 and 7.7/7.9, 192 rows, 3 slices 6.2/6.4 and 6.6/6.6.
    if constexpr (MAXS > 0 && NCH <= 2 && std::is_same<T, bf16_t>::value) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        opaque(ar[c]); opaque(br[c]); opaque(gr[c]); opaque(tr[c]);
#pragma unroll
        for (int k = 0; k < MAXS; ++k) { opaque(sl[c][k][0]); opaque(sl[c][k][1]); }
      }
    }
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) {
        a[c][i] = MAXS == 0 || dn ? to_f<T>(ar[c].v[i]) : 0.f;
        if constexpr (MAXS > 0) {
          float sum = (&sl[c][0][i >> 2].x)[i & 3];
#pragma unroll
          for (int k = 1; k < MAXS; ++k)
            if (k < splits) sum += (&sl[c][k][i >> 2].x)[i & 3];
          a[c][i] += sum;
        }
        xh[c][i] = (to_f<T>(br[c].v[i]) - mu) * rs;
        o[c][i] = a[c][i] * to_f<T>(gr[c].v[i]);         // dxhat, turned into ds below
        s1 += o[c][i];
        s2 += o[c][i] * xh[c][i];
      }
    }
    const float c1 = wave_sum(s1) / (float)d, c2 = wave_sum(s2) / (float)d;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (lane + 64 * c) * LN_VEC;
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) o[c][i] = rs * (o[c][i] - c1 - xh[c][i] * c2);
      if (add) {
#pragma unroll
        for (int i = 0; i < LN_VEC; ++i) o[c][i] += to_f<T>(tr[c].v[i]);
      }
      store_f<T, LN_VEC>(ds + base + col, o[c]);
      if (thr) {
        drop_apply<LN_VEC>(o[c], key, base + col, thr, inv_keep);
        store_f<T, LN_VEC>(ds_drop + base + col, o[c]);
      }
      // the consumers read the rounded value; sum exactly what they will see
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) o[c][i] = to_f<T>(from_f<T>(o[c][i]));
    }
  }
  // 512 columns of one quantity at a time, in two LDS stages by turns: a stage is written again only after the barrier behind which every
  // wavefront has read it, so that a stage costs one barrier.
  int u = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (k == nk) break;                                   // nk = 2: the bias sum is not wanted
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i)                    // slot (c, i, lane): consecutive lanes, consecutive banks
        lds[u][w][i * 64 + lane] = k == 0 ? a[c][i] * xh[c][i] : (k == 1 ? a[c][i] : o[c][i]);
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 512; j += 64 * WAVES) {         // partials stay in slot order (see ln_slot_column)
        const int at = j + threadIdx.x;
        if (64 * WAVES > 512 && at >= 512) break;
        float t = 0.f;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) t += lds[u][ww][at];
        partial[((size_t)blockIdx.x * 3 + k) * d + c * 512 + at] = t;
      }
      u ^= 1;
    }
  }
}

// out_k[j] = sum_p partial[p][k][j], p in a fixed order; k < nk <= 3.  One block owns 32 columns of one k: 32 row
// lanes stride over the partials (coalesced 128-byte reads, all of a lane's loads in flight at once for up to 256
// partials), then LDS combines the 32 lanes in a fixed order.
constexpr int RP_LANES = 32;
template <typename T>
__device__ __forceinline__ void reduce_partials_body(const float* __restrict__ partial, int np, int nk, int n, T* o0, T* o1, T* o2, int slots) {
  __shared__ float sh[RP_LANES][33];
  const int cx = threadIdx.x & 31, py = threadIdx.x >> 5;
  const int k = blockIdx.y;
  const int j = blockIdx.x * 32 + cx;
  float acc = 0.f;
  if (j < n) {
    int p = py;
    for (; p + 7 * RP_LANES < np; p += 8 * RP_LANES) {  // 8 loads in flight per thread; the order of the adds is fixed
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = partial[((size_t)(p + RP_LANES * u) * nk + k) * n + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += v[u];
    }
    // The last ones too, where they are more than 3 (past the end: the last one again).  One after the other they made blocks of 4 rows lose what they gain:
    // LayerNorm backward with its reduction, 1000 x 512 fp16, 250 partials 8.6 us against 7.9 with 63 of them, now 7.0; 1000 x 1024 10.3 and 10.4, now 8.8.
    // (32 partials 5.2 us, in this form 5.6.)
    if (np - (p - py) > 3 * RP_LANES) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = partial[((size_t)min(p + RP_LANES * u, np - 1) * nk + k) * n + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = p + RP_LANES * u < np ? acc + v[u] : acc;
    } else {
      for (; p < np; p += RP_LANES) acc += partial[((size_t)p * nk + k) * n + j];
    }
  }
  sh[py][cx] = acc;
  __syncthreads();
  if (py == 0 && j < n) {
    T* o = k == 0 ? o0 : (k == 1 ? o1 : o2);
    if (o) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < RP_LANES; ++i) t += sh[i][cx];
      o[slots ? ln_slot_column(j) : j] = from_f<T>(t);    // slots: index j is a slot of the row kernel's layout
    }
  }
}
template <typename T>
__global__ __launch_bounds__(32 * RP_LANES) void reduce_partials_kernel(const float* __restrict__ partial, int np, int nk, int n, T* o0,
                                                                        T* o1, T* o2, int slots) {
  reduce_partials_body<T>(partial, np, nk, n, o0, o1, o2, slots);
}
// The reductions of many LayerNorm backward launches in one: blockIdx.z picks the job (the table travels in the kernel
// arguments).  Every job has the [np][3][d] layout; an output that is null is skipped.
struct LnReduceTable { LnReduceJob job[LN_REDUCE_MAX]; };
template <typename T>
__global__ __launch_bounds__(32 * RP_LANES) void reduce_partials_batched_kernel(LnReduceTable tab, int d) {
  const LnReduceJob& j = tab.job[blockIdx.z];
  reduce_partials_body<T>(j.partial, j.np, 3, d, (T*)j.dgamma, (T*)j.dbeta, (T*)j.dbias, j.slots);
}

static int lnb_blocks(int rows) {
  int b = (rows + LNB_WAVES - 1) / LNB_WAVES;
  return b > LNB_MAX_BLOCKS ? LNB_MAX_BLOCKS : (b < 1 ? 1 : b);
}
// Wavefronts per block of the row kernel, 0: the looping one.  A column sum takes a block through LDS row by row, so small blocks are done
// sooner, and on more compute units, as long as there are not more than LNB_MAX_BLOCKS partials for the reduction behind it (whose share is
// counted here, as it was before the last partials came in one trip).  us with 4 / 8 / 16 wavefronts: 280 x 1024 3.8/4.4/6.0, 1020 x 1024 5.9/5.9/7.2, 1500 x 1024 6.9/6.6/7.7, 2000 x 1024 7.9/7.4/8.2, 900 x
// 512 3.4/3.5/4.4, 1800 x 512 5.0/4.6/5.3, 900 x 1536 7.1/7.5/9.5, 1800 x 1536 10.2/9.8/11.7; 3264 x 1024 -/11.4/11.2, 3700 x 512 -/6.6/6.2.
constexpr int LNR_FEWEST = 4;
static int lnr_waves(int rows, int d) {
  if (d % 512 || d > 1536) return 0;                     // (three 512-column parts of a row are what the registers of 16 wavefronts hold)
  for (int w = LNR_FEWEST; w <= 16; w *= 2)
    if (rows <= LNB_MAX_BLOCKS * w) return w;
  return 0;
}
// (enough for any smaller number of rows as well)
size_t layernorm_bwd_scratch_bytes(int rows, int d) {
  const int most = (rows + LNR_FEWEST - 1) / LNR_FEWEST;
  return (size_t)(most > LNB_MAX_BLOCKS ? LNB_MAX_BLOCKS : (most < 1 ? 1 : most)) * 3 * d * sizeof(float);
}

template <typename T>
static void ln_bwd_dispatch(hipStream_t s, const void* dn, const void* add, const void* sres, const float* mean,
                            const float* rstd, const void* gamma, void* ds, void* ds_drop, void* dgamma, void* dbeta,
                            void* dbias, int rows, int d, uint64_t key, float p, void* scratch, LnReduceJob* defer, const float* slices, int splits) {
  const int nk = dbias ? 3 : 2;
  const uint32_t thr = (p > 0.f && ds_drop) ? drop_threshold(p) : 0u;
  const float inv_keep = 1.f / (1.f - p);
  const int nch = (d + 511) / 512;
  // A wavefront per row where that can be: 3000 rows of 1536 34.0 us in the looping kernel, now 14.2.  (3264 rows of
  // 1024 11.5 us before the LDS stages took turns and the added gradient came with the row, now 10.2.)
  const int waves = lnr_waves(rows, d);
  if (waves) {
    const int nbr = (rows + waves - 1) / waves;
#define LN_BWD_ROW(N, W, S)                                                                                             \
  hipLaunchKernelGGL((layernorm_bwd_row_kernel<T, N, W, S>), dim3(nbr), dim3(64 * W), 0, s, (const T*)dn, slices, splits, (const T*)add,  \
                     (const T*)sres, mean, rstd, (const T*)gamma, (T*)ds, (T*)ds_drop, (float*)scratch, rows, d, key, thr, \
                     inv_keep, nk)
#define LN_BWD_SLICES(N) do { if (splits <= 2) LN_BWD_ROW(N, LNR_FEWEST, 2); else if (splits <= 4) LN_BWD_ROW(N, LNR_FEWEST, 4); else LN_BWD_ROW(N, LNR_FEWEST, 8); } while (0)
#define LN_BWD_WAVES(N) do { if (waves == 4) LN_BWD_ROW(N, 4, 0); else if (waves == 8) LN_BWD_ROW(N, 8, 0); else LN_BWD_ROW(N, 16, 0); } while (0)
    if (splits > 0) {
      if constexpr (sizeof(T) == 2) { if (nch == 1) LN_BWD_SLICES(1); else if (nch == 2) LN_BWD_SLICES(2); else LN_BWD_SLICES(3); }
    } else if (nch == 1) LN_BWD_WAVES(1); else if (nch == 2) LN_BWD_WAVES(2); else LN_BWD_WAVES(3);
#undef LN_BWD_SLICES
#undef LN_BWD_WAVES
#undef LN_BWD_ROW
    if (defer) { *defer = LnReduceJob{(const float*)scratch, nbr, 1, dgamma, dbeta, dbias}; return; }
    hipLaunchKernelGGL((reduce_partials_kernel<T>), dim3((d + 31) / 32, 3), dim3(32 * RP_LANES), 0, s, (const float*)scratch, nbr, 3, d,
                       (T*)dgamma, (T*)dbeta, (T*)dbias, 1);
    return;
  }
  const int nb = lnb_blocks(rows);
  const size_t shm = (size_t)LNB_WAVES * d * sizeof(float);
#define LN_BWD(N)                                                                                                       \
  hipLaunchKernelGGL((layernorm_bwd_kernel<T, N>), dim3(nb), dim3(64 * LNB_WAVES), shm, s, (const T*)dn, (const T*)add,             \
                     (const T*)sres, mean, rstd, (const T*)gamma, (T*)ds, (T*)ds_drop, (float*)scratch, rows, d, key, thr, \
                     inv_keep, nk)
  if (nch <= 1) LN_BWD(1); else if (nch == 2) LN_BWD(2); else if (nch == 3) LN_BWD(3); else LN_BWD(4);
#undef LN_BWD
  if (defer) { *defer = LnReduceJob{(const float*)scratch, nb, 0, dgamma, dbeta, dbias}; return; }
  hipLaunchKernelGGL((reduce_partials_kernel<T>), dim3((d + 31) / 32, 3), dim3(32 * RP_LANES), 0, s, (const float*)scratch, nb, 3, d,
                     (T*)dgamma, (T*)dbeta, (T*)dbias, 0);
}

bool layernorm_bwd_takes_slices(int dt, int rows, int d) { return dt != F32 && lnr_waves(rows, d) == LNR_FEWEST; }
void launch_layernorm_bwd(hipStream_t s, int dt, const void* dn, const void* add, const void* sres, const float* mean,
                          const float* rstd, const void* gamma, void* ds, void* ds_drop, void* dgamma, void* dbeta,
                          void* dbias, int rows, int d, uint64_t key, float p, void* scratch, LnReduceJob* defer, const float* slices, int splits) {
#define LN_BWD_T(T) ln_bwd_dispatch<T>(s, dn, add, sres, mean, rstd, gamma, ds, ds_drop, dgamma, dbeta, dbias, rows, d, key, p, scratch, defer, slices, splits)
  if (dt == F32) LN_BWD_T(float); else if (dt == F16) LN_BWD_T(half_t); else LN_BWD_T(bf16_t);
#undef LN_BWD_T
}

void launch_ln_reduce_batched(hipStream_t s, int dt, const LnReduceJob* jobs, int n, int d) {
  for (int i0 = 0; i0 < n; i0 += LN_REDUCE_MAX) {
    const int m = n - i0 < LN_REDUCE_MAX ? n - i0 : LN_REDUCE_MAX;
    LnReduceTable tab;
    for (int i = 0; i < m; ++i) tab.job[i] = jobs[i0 + i];
    const dim3 grid((d + 31) / 32, 3, m), block(32 * RP_LANES);
    if (dt == F32) hipLaunchKernelGGL((reduce_partials_batched_kernel<float>), grid, block, 0, s, tab, d);
    else if (dt == F16) hipLaunchKernelGGL((reduce_partials_batched_kernel<half_t>), grid, block, 0, s, tab, d);
    else hipLaunchKernelGGL((reduce_partials_batched_kernel<bf16_t>), grid, block, 0, s, tab, d);
  }
}

// ---- column sums --------------------------------------------------------------------------------------------------------
// out[j] = sum_r x[r, j].  Block = 64 column chunks (8 columns each) x 4 row lanes; grid.y row slabs write partials.
constexpr int CS_ROWS_PER_BLOCK = 64;

template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const T* __restrict__ x, int ld, int rows, int n, float* __restrict__ partial) {
  __shared__ float lds[4][64 * LN_VEC];
  const int cx = threadIdx.x & 63, ry = threadIdx.x >> 6;
  const int col = (blockIdx.x * 64 + cx) * LN_VEC;
  float acc[LN_VEC];
#pragma unroll
  for (int i = 0; i < LN_VEC; ++i) acc[i] = 0.f;
  const int r0 = blockIdx.y * CS_ROWS_PER_BLOCK;
  const int r1 = min(rows, r0 + CS_ROWS_PER_BLOCK);
  if (col < n) {
    for (int r = r0 + ry; r < r1; r += 4) {
      float t[LN_VEC];
      load_f<T, LN_VEC>(x + (size_t)r * ld + col, t);
#pragma unroll
      for (int i = 0; i < LN_VEC; ++i) acc[i] += t[i];
    }
  }
#pragma unroll
  for (int i = 0; i < LN_VEC; ++i) lds[ry][cx * LN_VEC + i] = acc[i];
  __syncthreads();
  for (int j = threadIdx.x; j < 64 * LN_VEC; j += 256) {
    const int c = blockIdx.x * 64 * LN_VEC + j;
    if (c < n) partial[(size_t)blockIdx.y * n + c] = (lds[0][j] + lds[1][j]) + (lds[2][j] + lds[3][j]);
  }
}

size_t colsum_scratch_bytes(int rows, int n) {
  return (size_t)((rows + CS_ROWS_PER_BLOCK - 1) / CS_ROWS_PER_BLOCK + 1) * n * sizeof(float);
}

template <typename T>
static void colsum_dispatch(hipStream_t s, const void* x, int ld, int rows, int n, void* out, void* scratch) {
  const int ny = (rows + CS_ROWS_PER_BLOCK - 1) / CS_ROWS_PER_BLOCK;
  dim3 grid((n + 64 * LN_VEC - 1) / (64 * LN_VEC), ny);
  hipLaunchKernelGGL((colsum_kernel<T>), grid, dim3(256), 0, s, (const T*)x, ld, rows, n, (float*)scratch);
  hipLaunchKernelGGL((reduce_partials_kernel<T>), dim3((n + 31) / 32, 1), dim3(32 * RP_LANES), 0, s, (const float*)scratch, ny, 1, n,
                     (T*)out, (T*)nullptr, (T*)nullptr, 0);
}

void launch_colsum(hipStream_t s, int dt, const void* x, int ld, int rows, int n, void* out, void* scratch) {
  if (dt == F32) colsum_dispatch<float>(s, x, ld, rows, n, out, scratch);
  else if (dt == F16) colsum_dispatch<half_t>(s, x, ld, rows, n, out, scratch);
  else colsum_dispatch<bf16_t>(s, x, ld, rows, n, out, scratch);
}

}  // namespace tfm
