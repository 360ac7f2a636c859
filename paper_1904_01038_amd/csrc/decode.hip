// Kernels of the incremental decoding step (Implementation, Inference): a per-row key/value cache indexed through an
// ancestry table, so a step computes exactly one new position per row.
//
// Cache layout.  Self-attention keys and values of decoder layer l live in K_l, V_l [rows][max_steps][d]: row r writes
// position t of ITS OWN row at step t and never moves anything.  When the search re-orders the beams, only an
// ancestry table changes: anc[r][s] is the physical row that holds position s of the hypothesis now living in row r
// (anc_new[r][s] = anc_old[parent[r]][s] for s < t, anc_new[r][t] = r).  Beams that share a prefix therefore read the
// same cache lines (L2 hits) and a re-ordering costs rows * t integers instead of a copy of every layer's cache.
// Cross-attention keys and values are projected once per source sentence and shared by its beams.
#include "common.h"
#include "kernels.h"

namespace tfm {

// The start of a step, one block per row: the row's ancestry table and its input vector sqrt(d) * E[prev] + PE(t), or, for
// prev = -1 - k (adaptive inputs), sqrt(d) * alt[k] + PE(t).  prev and parent are read where the host left them, in its pinned
// memory: two words per row in one trip, where a copy to the device first was a launch of its own (3.3 us and the host's time
// for it; the ancestry table another 1.7 us).
template <typename T>
__global__ __launch_bounds__(128) void decode_begin_kernel(const int* __restrict__ prev, const int* __restrict__ parent,
                                                           const int* __restrict__ anc_old, int* __restrict__ anc_new, int max_steps,
                                                           int t, const T* __restrict__ E, const T* __restrict__ alt,
                                                           const float* __restrict__ pe, T* __restrict__ out, int d, float scale) {
  const int r = blockIdx.x;
  const int id = prev[r], from = parent[r];
  for (int s = threadIdx.x; s <= t; s += 128) anc_new[(size_t)r * max_steps + s] = s < t ? anc_old[(size_t)from * max_steps + s] : r;
  const T* e = id >= 0 ? E + (size_t)id * d : alt + (size_t)(-1 - id) * d;
  const float* p = pe + (size_t)t * d;
  for (int col = threadIdx.x * 8; col < d; col += 128 * 8) {
    float v[8], q[8];
    load_f<T, 8>(e + col, v);
    load_f<float, 8>(p + col, q);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = scale * v[i] + q[i];
    store_f<T, 8>(out + (size_t)r * d + col, v);
  }
}
void launch_decode_begin(hipStream_t s, int dt, const int* prev, const int* parent, const int* anc_old, int* anc_new, int rows,
                         int max_steps, int t, const void* E, const void* alt, const float* pe, void* out, int d) {
  const float scale = sqrtf((float)d);
#define DB(T)                                                                                                                     \
  hipLaunchKernelGGL(decode_begin_kernel<T>, dim3(rows), dim3(128), 0, s, prev, parent, anc_old, anc_new, max_steps, t, (const T*)E, \
                     (const T*)alt, pe, (T*)out, d, scale)
  if (dt == F32) DB(float); else if (dt == F16) DB(half_t); else DB(bf16_t);
#undef DB
}

// K[r][t][:] = qkv[r][d .. 2d), V[r][t][:] = qkv[r][2d .. 3d)
template <typename T>
__global__ __launch_bounds__(256) void cache_append_kernel(const T* __restrict__ qkv, T* __restrict__ Kc, T* __restrict__ Vc,
                                                           int rows, int d, int max_steps, int t) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= rows * d) return;
  const int r = i / d, e = i - r * d;
  const size_t dst = ((size_t)r * max_steps + t) * d + e;
  Kc[dst] = qkv[(size_t)r * 3 * d + d + e];
  Vc[dst] = qkv[(size_t)r * 3 * d + 2 * d + e];
}
void launch_cache_append(hipStream_t s, int dt, const void* qkv, void* Kc, void* Vc, int rows, int d, int max_steps, int t) {
  const int n = rows * d;
  dim3 grid((n + 255) / 256), block(256);
  if (dt == F32) hipLaunchKernelGGL(cache_append_kernel<float>, grid, block, 0, s, (const float*)qkv, (float*)Kc, (float*)Vc, rows, d, max_steps, t);
  else if (dt == F16) hipLaunchKernelGGL(cache_append_kernel<half_t>, grid, block, 0, s, (const half_t*)qkv, (half_t*)Kc, (half_t*)Vc, rows, d, max_steps, t);
  else hipLaunchKernelGGL(cache_append_kernel<bf16_t>, grid, block, 0, s, (const bf16_t*)qkv, (bf16_t*)Kc, (bf16_t*)Vc, rows, d, max_steps, t);
}

// One wavefront per (row, head): a single query against n positions.
//   phase 1  lane = position: score = q . K[pos] / sqrt(dh), kept in LDS together with the row's address
//   phase 2  softmax over the positions (fp32)
//   phase 3  lane = feature: out[e] = sum_pos p[pos] V[pos][e]; a V row of one head is one 128-byte line at dh = 64
template <typename T, int VEC>
__global__ __launch_bounds__(64) void decode_attention_kernel(DecodeAttnArgs p) {
  extern __shared__ float smem[];
  const int r = blockIdx.x, h = blockIdx.y, lane = threadIdx.x, dh = p.dh;
  int n, base = 0;
  if (p.anc) n = p.t + 1;
  else { const int s = r / p.beam; base = p.src_off[s]; n = p.src_off[s + 1] - base; }
  float* sc = smem;                                    // [n_max] scores, then probabilities
  int* rowi = reinterpret_cast<int*>(smem + p.n_max);  // [n_max] element offset of the position's K row / V row
  float* qs = smem + 2 * p.n_max;                      // [dh]
  const T* q = reinterpret_cast<const T*>(p.q) + (size_t)r * p.ldq + h * dh;
  for (int e = lane; e < dh; e += 64) qs[e] = to_f<T>(q[e]);
  const T* K = reinterpret_cast<const T*>(p.k);
  const T* V = reinterpret_cast<const T*>(p.v);
  __syncthreads();
  const float scale = rsqrtf((float)dh);
  float lmax = -INFINITY;
  for (int s = lane; s < n; s += 64) {
    // element offset of (position s, head h) from the K and V bases (both have the same strides)
    const long long off = p.anc ? ((long long)p.anc[(size_t)r * p.max_steps + s] * p.max_steps + s) * p.row_stride + h * dh
                                : (long long)(base + s) * p.row_stride + h * dh;
    const T* kr = K + off;
    float acc = 0.f;
    for (int e = 0; e < dh; e += VEC) {
      float kv[VEC];
      load_f<T, VEC>(kr + e, kv);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc += qs[e + i] * kv[i];
    }
    acc *= scale;
    sc[s] = acc;
    // offsets fit in 32 bits: the host checks that every cache and projection holds fewer than 2^31 elements
    rowi[s] = (int)off;
    lmax = fmaxf(lmax, acc);
  }
  const float m = wave_max(lmax);
  float lsum = 0.f;
  for (int s = lane; s < n; s += 64) {
    const float e = __expf(sc[s] - m);
    sc[s] = e;
    lsum += e;
  }
  const float inv = 1.f / wave_sum(lsum);
  __syncthreads();
  T* out = reinterpret_cast<T*>(p.o) + (size_t)r * p.ldo + h * dh;
  for (int e = lane; e < dh; e += 64) {
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    int s = 0;
    for (; s + 4 <= n; s += 4) {
      a0 += sc[s] * to_f<T>(V[rowi[s] + e]);
      a1 += sc[s + 1] * to_f<T>(V[rowi[s + 1] + e]);
      a2 += sc[s + 2] * to_f<T>(V[rowi[s + 2] + e]);
      a3 += sc[s + 3] * to_f<T>(V[rowi[s + 3] + e]);
    }
    for (; s < n; ++s) a0 += sc[s] * to_f<T>(V[rowi[s] + e]);
    out[e] = from_f<T>((a0 + a1 + a2 + a3) * inv);
  }
}

// The same for head width 64 and 2-byte elements, one wavefront and two trips to memory: the position table and the query,
// then the keys AND the values of a chunk of positions together, so that the values travel while the scores are formed.  Longer histories go
// on in chunks with a running maximum.  Bound by that chain (a launch that loads and stores a little takes 1.6-2.5 us) up to some 1000 wavefronts, then
// by instructions and by the keys and values.  So the instructions are few: the scores of 16 positions are two MFMAs, keys as the left operand
// (lane = position, group of 8 features), the query in all 16 columns of the right one, and come out 4 positions to a group of 16 lanes,
// in all of its lanes; a lane then asks for 16 bytes of the values of two of its group's positions, 8 whole rows of 128 bytes a load, and
// the final sum over lanes halves what a lane holds with every exchange.  (Scores by 8 FMAs and 3 lane exchanges for every 16 bytes of a
// key, and every lane with the whole sum: 381 -> 560 vector instructions for 32 positions; 64 wavefronts and 21 positions 3.3 us against 2.7,
// 384 3.1 against 2.7, 1024 and 16 positions 2.9 against 2.7, 4096 5.2 and 5.2.  Relative error of the result against 64 bits, keys from 3e-6 to 8 in size,
// the same five digits.)
// The beams of a sentence are the wavefronts of one block: they read the same source positions (and mostly the same history),
// which then come into one L1 and one L2 once, where blocks of one row each were dealt out to different XCDs.
//
// Chunks of 64 positions hold 132 registers over the history (3072 wavefronts on the chip at once) and 116-123 over the source (4096), chunks of 32
// 92 (5120) and 70-78 (6144): a trip less for 33-64 and 97-128 positions, against half the work for the others.  us with chunks of 64 / of 32, fp16, 16 heads, 4 beams, for
// histories of 16, 32, 48, 64, 80 and 112 positions
//     64 wavefronts  2.9/2.5  3.0/2.7  3.2/3.4  3.4/3.6   4.5/ 4.3   4.8/ 5.2
//   1024             3.0/2.7  3.2/2.8  3.7/4.1  4.0/4.4   5.5/ 5.4   5.9/ 6.6
//   2048             3.8/3.3  4.5/3.9  4.8/5.1  5.2/5.5   7.3/ 6.4   8.0/ 7.6
//   3072             5.0/4.0  5.4/4.6  5.8/6.4  6.4/6.6   9.3/ 8.2  10.7/10.9
//   4096             6.2/4.5  7.0/5.2  7.8/7.2  9.3/8.0  14.4/10.6  16.8/14.0
// and for sources, whose operands change from launch to launch (at least 4.2 us a launch from this host), of up to 32, 40, 48, 64, 80 and 112 positions
//   1024             4.2/4.1  4.2/4.0  4.1/4.2  4.2/4.2   4.8/ 4.7   5.1/ 5.3
//   2048             4.4/4.2  4.6/4.7  4.7/4.8  5.2/5.1   6.5/ 5.8   7.1/ 6.9
//   3072             5.1/4.5  5.4/5.5  5.7/5.7  6.2/6.2   8.1/ 7.3   9.7/ 9.3
//   4096             5.9/5.0  6.3/6.5  6.6/6.8  7.2/7.4  10.4/ 9.6  13.1/12.9
//   4288                      7.5/7.2  7.9/7.4  8.6/8.2
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
static __device__ __forceinline__ f32x4 mfma16(half_t, uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
static __device__ __forceinline__ f32x4 mfma16(bf16_t, uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int DEC_ATT_WAVES = 8;                         // rows per block at most

template <typename T, int U, bool SELF>                  // chunks of 16 * U positions; SELF: in the caches, at rows from the ancestry table
static __device__ __forceinline__ void decode_attention64(const DecodeAttnArgs& p) {
  __shared__ __attribute__((aligned(16))) T sq[DEC_ATT_WAVES][64];
  constexpr int dh = 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4, odd = (lane >> 3) & 1, f = lane & 7;
  const int r = blockIdx.x * (blockDim.x >> 6) + wave, h = blockIdx.y;
  int n, base = 0;
  if (SELF) n = p.t + 1;
  else { const int s = r / p.beam; base = p.src_off[s]; n = p.src_off[s + 1] - base; }
  const T* K = reinterpret_cast<const T*>(p.k) + h * dh;
  const T* V = reinterpret_cast<const T*>(p.v) + h * dh;
  // position t of a self-attention step may still be outside the caches: it is read from the new rows, and 16 lanes copy
  // this head's 128 + 128 bytes into the row's own cache lines for the steps to come (nobody reads them during this launch)
  const bool fresh = SELF && p.k_new;
  const T* knew = reinterpret_cast<const T*>(p.k_new) + (size_t)r * p.ld_new + h * dh;
  const T* vnew = reinterpret_cast<const T*>(p.v_new) + (size_t)r * p.ld_new + h * dh;
  // Position s is row first * per + s of the caches (past the end: the last one, with weight 0).  The lane asks for position c of a
  // tile's keys and for positions 4 g + 2 j + odd of its values, j = 0, 1.
  const int per = SELF ? p.max_steps : 1;
  const int* anc = p.anc + (size_t)r * p.max_steps;
  int kfirst[U], vfirst[U][2];
  auto k_pos = [&](int s0, int u) { return min(s0 + 16 * u + c, n - 1); };
  auto v_pos = [&](int s0, int u, int j) { return min(s0 + 16 * u + 4 * g + 2 * j + odd, n - 1); };
  auto look_up = [&](int s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) kfirst[u] = SELF ? anc[k_pos(s0, u)] : base;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < 2; ++j) vfirst[u][j] = SELF ? anc[v_pos(s0, u, j)] : base;
  };
  look_up(0);
  uint4 q[2];                                            // the query's features 32 i + 8 g .. + 7
  if (p.q_partial) {                                     // it arrives as the slices of a split-K product (at most 8)
    const size_t at = (size_t)r * p.H * dh + h * dh + lane, slice = (size_t)p.rows * p.H * dh;
    float part[8];                                       // (asked for together: the last slice again where there are fewer)
#pragma unroll
    for (int k = 0; k < 8; ++k) part[k] = p.q_partial[min(k, p.q_splits - 1) * slice + at];
    float qv = part[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) qv = k < p.q_splits ? qv + part[k] : qv;
    if (p.q_bias) qv += to_f<T>(reinterpret_cast<const T*>(p.q_bias)[h * dh + lane]);
    T* qs = sq[wave];
    qs[lane] = from_f<T>(qv);                            // rounded as the stored projection would be
    __syncthreads();                                     // (every row of the launch comes this way, or none does)
#pragma unroll
    for (int i = 0; i < 2; ++i) q[i] = reinterpret_cast<const uint4*>(qs)[4 * i + g];
  } else {
    const uint4* from = reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(p.q) + (size_t)r * p.ldq + h * dh);
#pragma unroll
    for (int i = 0; i < 2; ++i) q[i] = from[4 * i + g];
  }
  auto larger = [](uint32_t a, uint32_t b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); };
  auto sum = [](uint32_t a, uint32_t b) { return __float_as_uint(__uint_as_float(a) + __uint_as_float(b)); };
  const float scale = 0.125f * 1.44269504088896340736f;  // (exponentials to base 2)
  float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  // 16 bytes of position s, `piece` bytes into its row (byte offsets are below 2^32, which the host checks)
  auto fetch = [&](const T* cache, const T* row_new, int first, int s, uint32_t piece) {
    const uint32_t at = (uint32_t)(first * per + s) * (uint32_t)p.row_stride * 2u + piece;
    const char* from = reinterpret_cast<const char*>(cache) + at;
    if (SELF) from = fresh && s >= p.t ? reinterpret_cast<const char*>(row_new) + piece : from;
    return reinterpret_cast<const uint4*>(from);
  };
  for (int s0 = 0; s0 < n; s0 += 16 * U) {
    uint4 kv[U][2], vv[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint4* from = fetch(K, knew, kfirst[u], k_pos(s0, u), 16 * g);
      kv[u][0] = from[0];
      kv[u][1] = from[4];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < 2; ++j) vv[u][j] = *fetch(V, vnew, vfirst[u][j], v_pos(s0, u, j), 16 * f);
    if (s0 + 16 * U < n) look_up(s0 + 16 * U);           // the next chunk's rows
    asm volatile("" ::: "memory");                      // (all loads of a chunk are on their way before the first is looked at)
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sc[U];                                         // of positions 4 g .. 4 g + 3 of a tile, in all lanes of a group; past the end the last one's
    float mn = m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sc[u] = mfma16(T{}, kv[u][1], q[1], mfma16(T{}, kv[u][0], q[0], f32x4{0.f, 0.f, 0.f, 0.f}));
#pragma unroll
      for (int e = 0; e < 4; ++e) mn = fmaxf(mn, sc[u][e]);
    }
    mn = __uint_as_float(with_lane_32(with_lane_16(__float_as_uint(mn), larger), larger));
    const float top = mn > -INFINITY ? mn : 0.f;         // scores of -infinity alone, so far: weight 0, as beside others
    const float keep = __builtin_amdgcn_exp2f((m - top) * scale);
    m = mn;
    l *= keep;                                           // (l: this lane's share, as of acc; the lanes are added up at the end)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= keep;
    const int left = n - s0 - 4 * g - odd;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float w = __builtin_amdgcn_exp2f(((odd ? sc[u][2 * j + 1] : sc[u][2 * j]) - top) * scale);
        w = left > 16 * u + 2 * j ? w : 0.f;
        l += w;
        Pack<T, 8> x;
        __builtin_memcpy(&x, &vv[u][j], 16);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += w * to_f<T>(x.v[i]);
      }
  }
  // Features 8 f .. 8 f + 7 over the lanes that differ in bits 3, 4 and 5 of their number.  Each exchange halves what a lane is left with: one feature,
  // 4 odd + 2 (bit 4) + (bit 5).
  float y[4], z[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[2 * i]), __float_as_uint(acc[2 * i + 1]), false, false);
    y[i] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(y[2 * i]), __float_as_uint(y[2 * i + 1]), false, false);
    z[i] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  }
  const float sent = odd ? z[0] : z[1];
  const float o = (odd ? z[1] : z[0]) + __int_as_float(dpp_move<0x128, 0xf>(0, __float_as_int(sent)));       // row_ror:8
  l = __uint_as_float(with_lane_8(with_lane_16(with_lane_32(__float_as_uint(l), sum), sum), sum));
  reinterpret_cast<T*>(p.o)[(size_t)r * p.ldo + h * dh + 8 * f + 4 * odd + 2 * (g & 1) + (g >> 1)] = from_f<T>(o * (1.f / l));
  if (fresh && lane < 16) {
    T* cache = const_cast<T*>(odd ? V : K) + ((size_t)r * p.max_steps + p.t) * p.row_stride + f * 8;
    *reinterpret_cast<uint4*>(cache) = *reinterpret_cast<const uint4*>((odd ? vnew : knew) + f * 8);
  }
}

template <typename T, int U>                             // over the history
__global__ __launch_bounds__(64 * DEC_ATT_WAVES) void decode_attention64_kernel(DecodeAttnArgs p) { decode_attention64<T, U, true>(p); }
template <typename T, int U>                             // over the source sentence: no table, positions one behind the other
__global__ __launch_bounds__(64 * DEC_ATT_WAVES) void decode_source_attention64_kernel(DecodeAttnArgs p) { decode_attention64<T, U, false>(p); }

// 8 elements of a key against 8 of the query, in 32-bit FMAs.  (v_dot2_f32_f16 truncates what lies far below the larger term and
// below a fixed floor: 1.6e-5 of the result with subnormal keys, where FMAs are off by 6e-8.)
template <typename T> __device__ __forceinline__ float dot8_acc(const float (&q)[8], uint4 k, float c) {
  Pack<T, 8> x;
  __builtin_memcpy(&x, &k, 16);
#pragma unroll
  for (int i = 0; i < 8; ++i) c = fmaf(q[i], to_f<T>(x.v[i]), c);
  return c;
}
// op over the lanes that differ in bits 0, 1 and 2 of their number (a group of 8), and in bits 3, 4 and 5 (across the groups)
template <typename Op> __device__ __forceinline__ float over_lanes(float v, Op op) {
  v = op(v, __int_as_float(dpp_move<0xB1, 0xf>(0, __float_as_int(v))));        // quad_perm 1,0,3,2
  v = op(v, __int_as_float(dpp_move<0x4E, 0xf>(0, __float_as_int(v))));        // quad_perm 2,3,0,1
  return op(v, __int_as_float(dpp_move<0x141, 0xf>(0, __float_as_int(v))));    // row_half_mirror
}
template <typename Op> __device__ __forceinline__ float over_groups(float v, Op op) {
  auto bits = [&](uint32_t a, uint32_t b) { return __float_as_uint(op(__uint_as_float(a), __uint_as_float(b))); };
  return __uint_as_float(with_lane_32(with_lane_16(with_lane_8(__float_as_uint(v), bits), bits), bits));
}

// The same for many wavefronts and many positions, which are bound by keys and values on their way from L2 where the beams of a sentence share them: a
// load fetches 8 whole rows of 128 bytes, of the keys too, where the kernels above touch the halves of 16.  Lane = (group g = lane / 8, 16-byte piece
// f = lane % 8): a score is 8 FMAs and 3 lane exchanges.  Chunks of 32 positions, 81 registers.  us above / here, histories of 66, 96 and 128 positions:
//   104 x 16 heads, 4 beams  6.6/ 6.6   6.9/ 6.8   9.0/ 8.2      110 x 24, 5 beams  9.6/ 9.2  10.7/ 9.5  13.6/11.6
//   136                      8.3/ 8.0   9.2/ 8.2  11.3/10.1      300 x 24          20.1/19.0  22.4/19.9  27.1/24.1
//   268                     12.1/11.8  14.1/12.9  17.8/16.0      one beam: 130 x 16 10.6/11.3  12.2/12.9  15.3/15.8
// and sources of up to 66, 80, 96 and 128:  200 x 16, 4 beams 8.2/7.9  9.2/8.6  10.0/8.8  13.3/11.8;  170 x 24, 5 beams 9.3/9.7  10.5/10.8  11.3/10.8  15.0/14.7.
// The line is at two chunks and not at 44 positions, where the times cross (200 x 16, history of 40 7.5/7.5, of 64 8.6/7.8): the kernels add in another order, and
// up to there a sentence has one of them.
template <typename T>
__global__ __launch_bounds__(64 * DEC_ATT_WAVES) void decode_long_attention_kernel(DecodeAttnArgs p) {
  constexpr int U = 4;                                   // chunks of 8 * U positions
  __shared__ __attribute__((aligned(16))) T sq[DEC_ATT_WAVES][64];
  constexpr int dh = 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 3, f = lane & 7;
  const int r = blockIdx.x * (blockDim.x >> 6) + wave, h = blockIdx.y;
  T* qs = sq[wave];
  int n, base = 0;
  if (p.anc) n = p.t + 1;
  else { const int s = r / p.beam; base = p.src_off[s]; n = p.src_off[s + 1] - base; }
  const T* K = reinterpret_cast<const T*>(p.k) + h * dh;
  const T* V = reinterpret_cast<const T*>(p.v) + h * dh;
  // position t of a self-attention step may still be outside the caches: it is read from the new rows, and 16 lanes copy
  // this head's 128 + 128 bytes into the row's own cache lines for the steps to come (nobody reads them during this launch)
  const T* knew = nullptr;
  const T* vnew = nullptr;
  if (p.anc && p.k_new) {
    knew = reinterpret_cast<const T*>(p.k_new) + (size_t)r * p.ld_new + h * dh;
    vnew = reinterpret_cast<const T*>(p.v_new) + (size_t)r * p.ld_new + h * dh;
  }
  // Position s is row first[u] * per + s of the caches, s = g, g + 8, ... of the chunk (past the end: the last one, with weight 0).
  // The choice between the two tables is made once for all U of them: made for each, it put a wait behind every single load.
  const int per = p.anc ? p.max_steps : 1;
  int first[U];
  auto look_up = [&](int s0) {
    if (p.anc) {
#pragma unroll
      for (int u = 0; u < U; ++u) first[u] = p.anc[(size_t)r * p.max_steps + min(s0 + 8 * u + g, n - 1)];
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) first[u] = base;
    }
  };
  look_up(0);
  uint4 qh;                                              // this lane's piece of the query
  if (p.q_partial) {                                     // the query arrives as the slices of a split-K product (at most 8)
    const size_t at = (size_t)r * p.H * dh + h * dh + lane, slice = (size_t)p.rows * p.H * dh;
    float part[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) part[k] = k < p.q_splits ? p.q_partial[k * slice + at] : 0.f;
    float qv = part[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) qv += part[k];
    if (p.q_bias) qv += to_f<T>(reinterpret_cast<const T*>(p.q_bias)[h * dh + lane]);
    qs[lane] = from_f<T>(qv);                            // rounded as the stored projection would be
    __syncthreads();                                     // (every row of the launch comes this way, or none does)
    qh = reinterpret_cast<const uint4*>(qs)[f];
  } else {
    qh = reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(p.q) + (size_t)r * p.ldq + h * dh)[f];
  }
  auto add = [](float x, float y) { return x + y; };
  auto larger = [](float x, float y) { return fmaxf(x, y); };
  float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  for (int s0 = 0; s0 < n; s0 += 8 * U) {
    uint4 kv[U], vv[U];
    int off[U];                                          // (the host checks that they fit)
#pragma unroll
    for (int u = 0; u < U; ++u) off[u] = (first[u] * per + min(s0 + 8 * u + g, n - 1)) * p.row_stride;
#pragma unroll
    for (int u = 0; u < U; ++u) kv[u] = *reinterpret_cast<const uint4*>(((knew && s0 + 8 * u + g >= p.t) ? knew : K + off[u]) + f * 8);
#pragma unroll
    for (int u = 0; u < U; ++u) vv[u] = *reinterpret_cast<const uint4*>(((vnew && s0 + 8 * u + g >= p.t) ? vnew : V + off[u]) + f * 8);
    if (s0 + 8 * U < n) look_up(s0 + 8 * U);             // the next chunk's rows
    // The query is looked at only now, when the chunk's loads are on their way (its conversion ahead of the loop would wait for it
    // first: 0.35 us of 4.7), and its values are opaque: seen as halves, the FMAs would be paired into v_dot2_f32_f16.
    asm volatile("" : "+v"(qh.x), "+v"(qh.y), "+v"(qh.z), "+v"(qh.w));
    float q[8], sc[U], mn = m;
    {
      Pack<T, 8> x;
      __builtin_memcpy(&x, &qh, 16);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        q[i] = to_f<T>(x.v[i]);
        asm("" : "+v"(q[i]));
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sc[u] = over_lanes(dot8_acc<T>(q, kv[u], 0.f), add);
      sc[u] = s0 + 8 * u + g < n ? sc[u] * 0.125f : -INFINITY;
      mn = fmaxf(mn, sc[u]);
    }
    mn = over_groups(mn, larger);
    const float top = mn > -INFINITY ? mn : 0.f;         // scores of -infinity alone, so far: weight 0, as beside others
    const float keep = __expf(m - top);
    m = mn;
    l *= keep;                                           // (l: this group's share; the groups are added up at the end)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= keep;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float w = __expf(sc[u] - top);
      l += w;
      Pack<T, 8> x;
      __builtin_memcpy(&x, &vv[u], 16);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += w * to_f<T>(x.v[i]);
    }
  }
  const float inv = 1.f / over_groups(l, add);
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = over_groups(acc[i], add) * inv;
  if (g == 0) store_f<T, 8>(reinterpret_cast<T*>(p.o) + (size_t)r * p.ldo + h * dh + f * 8, acc);
  if (knew && g < 2) {
    T* cache = const_cast<T*>(g == 0 ? K : V) + ((size_t)r * p.max_steps + p.t) * p.row_stride + f * 8;
    *reinterpret_cast<uint4*>(cache) = *reinterpret_cast<const uint4*>((g == 0 ? knew : vnew) + f * 8);
  }
}

// (16-byte accesses: the host side lays q, the caches and the output out with head slices at multiples of 128 bytes)
static bool decode_attention_fast(const DecodeAttnArgs& a) {
  return a.dh == 64 && a.dt != F32 && a.ldq % 8 == 0 && a.row_stride % 8 == 0 && a.ldo % 8 == 0 && (!a.k_new || a.ld_new % 8 == 0);
}
bool decode_attention_appends(const DecodeAttnArgs& a) { return a.anc && a.k_new && a.v_new && decode_attention_fast(a); }

void launch_decode_attention(hipStream_t s, const DecodeAttnArgs& a) {
  if (a.rows <= 0) return;
  dim3 grid(a.rows, a.H), block(64);
  const size_t smem = (size_t)(2 * a.n_max + a.dh) * sizeof(float);
  if (decode_attention_fast(a) && a.q_splits <= 8) {
    const int w = a.beam <= DEC_ATT_WAVES ? a.beam : 1;  // (rows = sentences * beam)
    grid = dim3(a.rows / w, a.H);
    block = dim3(64 * w);
    // (the lines: see the table above.  33-64 positions of the history are faster in one chunk up to 3072 wavefronts, of the source up to 4096)
    const int halves = (a.n_max + 31) / 32, waves = a.rows * a.H;
    const bool all = halves == 2 ? waves <= (a.anc ? 3072 : 4096) : halves > 3 && waves < 2048;
    if (w > 1 && waves >= 2048 && a.n_max > (a.anc ? 64 : 80)) {               // (the lines: see decode_long_attention_kernel)
      if (a.dt == F16) hipLaunchKernelGGL((decode_long_attention_kernel<half_t>), grid, block, 0, s, a);
      else hipLaunchKernelGGL((decode_long_attention_kernel<bf16_t>), grid, block, 0, s, a);
      return;
    }
#define DA64(KERNEL, T)                                                                                                      \
  do { if (all) hipLaunchKernelGGL((KERNEL<T, 4>), grid, block, 0, s, a); else hipLaunchKernelGGL((KERNEL<T, 2>), grid, block, 0, s, a); } while (0)
    if (a.dt == F16) { if (a.anc) DA64(decode_attention64_kernel, half_t); else DA64(decode_source_attention64_kernel, half_t); }
    else if (a.anc) DA64(decode_attention64_kernel, bf16_t); else DA64(decode_source_attention64_kernel, bf16_t);
#undef DA64
    return;
  }
  if (a.q_partial)                                     // the general kernel reads a finished query: finish it into q first
    launch_splitk_reduce(s, a.dt, a.q_partial, a.q_splits, a.rows, a.H * a.dh, const_cast<void*>(a.q), a.ldq, a.q_bias, 0);
  const bool vec = a.dh % 8 == 0;
#define DA(T, VEC) hipLaunchKernelGGL((decode_attention_kernel<T, VEC>), grid, block, smem, s, a)
  if (a.dt == F32) { if (vec) DA(float, 8); else DA(float, 1); }
  else if (a.dt == F16) { if (vec) DA(half_t, 8); else DA(half_t, 1); }
  else { if (vec) DA(bf16_t, 8); else DA(bf16_t, 1); }
#undef DA
}

__device__ __forceinline__ bool better(float v, int i, float w, int j) { return v > w || (v == w && i < j); }

// Per row: log-sum-exp of the logits and the k best tokens (larger value first, equal values by ascending id).
//
// One block looks at 4096 values of a row (16 per thread) and leaves the k best of them with their (maximum, sum of
// exponentials); further launches of the same kernel reduce those lists, 4096 candidates per block, until one block per row
// is left, which writes the result.  A row never has to fit one compute unit, so a step with few rows and a large vocabulary
// still fills the chip (24 rows of the adaptive language model, 40000 + 207744 + 267742 columns: with one block per row these
// three passes took 1.28 ms of a step of 1.66 ms; 4 rows x 32768 with 1024 threads a row and no second launch: 17 us against
// 8.0 + 6.1 us).
//
// Selection costs little because almost no value takes part in it.  Every wavefront splits its lanes into at least k groups;
// the smallest of the groups' maxima is a value that at least k others reach, so no value among the block's k best lies below
// it.  The largest such bound of the block filters the registers, and every survivor counts how many others are better than
// itself: that is its place.  Should more than TOPK_LIST survive (many equal values), or too few (values of -infinity, or NaN),
// the block falls back to k rounds over all of its values.  -infinity is a value like any other, after the finite ones; NaN is
// never a candidate and makes the row's log-sum-exp NaN.
//
// An adaptive softmax has its scores in several segments, the head's tokens and each tail cluster's, whose blocks share the first launch; the second one
// knows every block's (maximum, sum) pair, so it adds log p(cluster), the head's score of the cluster less the cluster's own log-sum-exp, to a
// tail's candidates, in 32 bits.  24 rows of 267742 scores: 11.2 + 10.6 us, where a pass for each tail's log-sum-exp, a copy of all
// the scores into one row and the passes over that row were 9 launches and 60 us.
constexpr int TOPK_THREADS = 256, TOPK_PER = 16, TOPK_TILE = TOPK_THREADS * TOPK_PER, TOPK_LIST = 256;

struct TopkList { float* v; int* id; float *m, *s; };    // per row: n * k candidates, n (maximum, sum of exp(value - maximum)) pairs

// VEC > 0: values of the segments, VEC per load; VEC == 0: candidates of the `n_in` lists of `in`, TOPK_TILE / k lists per block, with CLUSTERS those
// of the launch over several segments (a flag of both: over one segment the search for a block's cost a step of one sentence 1 %)
template <typename T, int VEC, bool CLUSTERS>
__global__ __launch_bounds__(TOPK_THREADS) void row_topk_kernel(TopkSegments sg, TopkList in, int n_in, int k, TopkList out,
                                                      float* __restrict__ top_logp, int* __restrict__ top_id, float* __restrict__ lse_out) {
  constexpr int NT = TOPK_THREADS, PER = TOPK_PER, NW = NT / 64;
  static_assert(NT >= TOPK_LIST, "one survivor per thread");
  __shared__ float sh[16], sh_bound[NW];
  __shared__ __attribute__((aligned(16))) float list_v[TOPK_LIST];
  __shared__ __attribute__((aligned(16))) int list_i[TOPK_LIST];
  __shared__ int list_n;
  __shared__ float sh_off[TOPK_SEGMENTS], sh_m[TOPK_SEGMENTS], sh_s;
  static_assert(TOPK_SEGMENTS <= NW, "a wavefront per segment");
  const int row = blockIdx.x, blk = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float c[PER];
  int id0 = 0;                                           // VEC > 0: id of this thread's first value (the others follow from it)
  int ids[VEC == 0 ? PER : 1];
  int l0 = 0, l1 = 0;                                    // VEC == 0: the lists of this block
  int V = 0, base = 0;                                   // VEC > 0: values of this block's segment from the block's first on; that one's id
  if constexpr (VEC > 0) {
    int g = 0;
    if constexpr (CLUSTERS) {
      for (int i = 1; i < sg.n; ++i) g = blk >= sg.blk0[i] ? i : g;
    }
    const int at = (blk - sg.blk0[g]) * NT * PER, width = sg.ld[g] - at;
    V = sg.V[g] - at;
    base = sg.lo[g] + at;
    const T* zr = reinterpret_cast<const T*>(sg.z[g]) + (size_t)row * sg.ld[g] + at;
    id0 = (wave * 64 * (PER / VEC) + lane) * VEC;
#pragma unroll
    for (int i = 0; i < PER / VEC; ++i) {
      const int col = id0 + i * 64 * VEC;
      float t[VEC];
#pragma unroll
      for (int j = 0; j < VEC; ++j) t[j] = -INFINITY;
      if (col + VEC <= width) load_f<T, VEC>(zr + col, t);
#pragma unroll
      for (int j = 0; j < VEC; ++j) c[i * VEC + j] = !CLUSTERS || col + j < V ? t[j] : -INFINITY;       // (one segment: V == ld)
    }
  } else {
    const int per = TOPK_TILE / k;
    l0 = blk * per;
    l1 = min(n_in, l0 + per);
    const size_t at = (size_t)row * n_in * k;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int q = l0 * k + e * NT + tid;
      const bool ok = q < l1 * k;
      c[e] = ok ? in.v[at + q] : -INFINITY;
      ids[e] = ok ? in.id[at + q] : 0x7fffffff;
    }
    if constexpr (CLUSTERS) {
      if (wave < sg.n) {                                 // a segment's log-sum-exp, in one trip to memory
        const float entry = wave == 0 ? 0.f : to_f<T>(reinterpret_cast<const T*>(sg.z[0])[(size_t)row * sg.ld[0] + sg.V[0] + wave - 1]);
        const size_t first = (size_t)row * n_in;
        auto scaled = [](float s, float m, float to) { return s * (m > -INFINITY ? __expf(m - to) : 1.f); };         // (0 or NaN times 1)
        float m = -INFINITY, se = 0.f;
        for (int l = sg.blk0[wave] + lane; l < sg.blk0[wave + 1]; l += 64) {
          const float lm = in.m[first + l], ls = in.s[first + l], mn = fmaxf(m, lm);
          se = scaled(se, m, mn) + scaled(ls, lm, mn);
          m = mn;
        }
        const float top = wave_max(m);
        se = wave_sum(scaled(se, m, top));
        if (lane == 0) {
          const float off = wave == 0 ? 0.f : entry - (top + logf(se));
          sh_off[wave] = off;
          sh_m[wave] = wave == 0 ? top : entry;
          if (wave == 0) sh_s = se;
          if (blk == 0) sg.off[(size_t)row * TOPK_SEGMENTS + wave] = off;
        }
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        float off = 0.f;
        for (int i = 1; i < sg.n; ++i) off = ids[e] >= sg.lo[i] ? sh_off[i] : off;
        c[e] = ids[e] == 0x7fffffff ? c[e] : c[e] + off;
      }
    }
  }
  auto id_of = [&](int e) { return VEC > 0 ? id0 + (e / (VEC > 0 ? VEC : 1)) * 64 * VEC + e % (VEC > 0 ? VEC : 1) : ids[VEC > 0 ? 0 : e]; };
  float lmax = -INFINITY;
#pragma unroll
  for (int e = 0; e < PER; ++e) lmax = fmaxf(lmax, c[e]);
  {
    auto with = [](float v, int moved) { return fmaxf(v, __int_as_float(moved)); };
    float x = lmax;                                      // groups of 4 lanes, of 8 for k <= 8, of 16 for k <= 4
    x = with(x, dpp_move<0xB1, 0xf>(0, __float_as_int(x)));                    // quad_perm 1,0,3,2
    x = with(x, dpp_move<0x4E, 0xf>(0, __float_as_int(x)));                    // quad_perm 2,3,0,1
    if (k <= 8) x = with(x, dpp_move<0x141, 0xf>(0, __float_as_int(x)));       // row_half_mirror
    if (k <= 4) x = with(x, dpp_move<0x140, 0xf>(0, __float_as_int(x)));       // row_mirror
    const float bound = k == 1 ? wave_max(x) : -wave_max(-x);
    if (lane == 0) sh_bound[wave] = bound;
  }
  if (tid == 0) list_n = 0;
  float gm, gs;
  if constexpr (VEC > 0) {
    gm = block_max(lmax, sh);                            // (its barriers also publish sh_bound and list_n)
    float se = 0.f;
    if (gm > -INFINITY) {
#pragma unroll
      for (int e = 0; e < PER; ++e) se += __expf(c[e] - gm);
    } else {
#pragma unroll
      for (int e = 0; e < PER; ++e) se += c[e] != c[e] ? c[e] : 0.f;
    }
    gs = block_sum(se, sh);
  } else if constexpr (CLUSTERS) {                       // the head's tokens and clusters share its distribution
    gm = sh_m[0];
    for (int i = 1; i < sg.n; ++i) gm = fmaxf(gm, sh_m[i]);
    gs = sh_s * (sh_m[0] > -INFINITY ? __expf(sh_m[0] - gm) : 1.f);
    for (int i = 1; i < sg.n; ++i) {
      gs += gm > -INFINITY ? __expf(sh_m[i] - gm) : sh_m[i] != sh_m[i] ? sh_m[i] : 0.f;
      if (!(sh_off[i] < INFINITY)) gs = __uint_as_float(0x7fc00000u);           // NaN in a tail, or a tail of -infinity alone
    }
    if (blk > 0) { gm = -INFINITY; gs = 0.f; }           // (the next launch adds the blocks' sums up)
    __syncthreads();                                     // publishes sh_bound and list_n
  } else {
    float m = -INFINITY;
    for (int l = l0 + tid; l < l1; l += NT) m = fmaxf(m, in.m[(size_t)row * n_in + l]);
    gm = block_max(m, sh);
    float se = 0.f;
    for (int l = l0 + tid; l < l1; l += NT) {
      const float lm = in.m[(size_t)row * n_in + l];
      se += in.s[(size_t)row * n_in + l] * (lm > -INFINITY ? __expf(lm - gm) : 1.f);       // (0 or NaN times 1)
    }
    gs = block_sum(se, sh);
  }
  float bound = sh_bound[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) bound = fmaxf(bound, sh_bound[w]);
  if (lmax >= bound && lmax > -INFINITY) {                // few lanes; the order of the list does not matter
    auto kept = [&](int e) { return c[e] >= bound && c[e] > -INFINITY; };
    int mine = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) mine += kept(e) ? 1 : 0;
    int at = atomicAdd(&list_n, mine);
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (kept(e)) {
        if (at < TOPK_LIST) { list_v[at] = c[e]; list_i[at] = id_of(e); }
        ++at;
      }
  }
  __syncthreads();
  const int lists = gridDim.y;
  const bool last = lists == 1;
  const float lse = gm + logf(gs);
  if (tid == 0) {
    if (last) { if (lse_out) lse_out[row] = lse; }
    else { out.m[(size_t)row * lists + blk] = gm; out.s[(size_t)row * lists + blk] = gs; }
  }
  auto emit = [&](int r, float v, int id) {
    id = id == 0x7fffffff ? id : id + base;
    if (last) {
      top_logp[(size_t)row * k + r] = v - lse;
      top_id[(size_t)row * k + r] = id;
    } else {
      out.v[((size_t)row * lists + blk) * k + r] = v;
      out.id[((size_t)row * lists + blk) * k + r] = id;
    }
  };
  const int n = list_n, least = VEC > 0 ? min(k, V) : k;
  if (n <= TOPK_LIST && n >= least) {
    if (tid < 16 && n + tid < TOPK_LIST) { list_v[n + tid] = -INFINITY; list_i[n + tid] = 0x7fffffff; }     // whole groups of 16 below
    __syncthreads();
    if (tid < n) {
      const float v = list_v[tid];
      const int id = list_i[tid];
      int rank = 0;
      for (int j = 0; j < n; j += 16) {                  // 16 at a time: their LDS reads are in flight together
        float4 o[4];
        int4 oi[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          o[q] = *reinterpret_cast<const float4*>(list_v + j + 4 * q);
          oi[q] = *reinterpret_cast<const int4*>(list_i + j + 4 * q);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          rank += (int)better(o[q].x, oi[q].x, v, id) + (int)better(o[q].y, oi[q].y, v, id) + (int)better(o[q].z, oi[q].z, v, id) +
                  (int)better(o[q].w, oi[q].w, v, id);
      }
      if (rank < k) emit(rank, v, id);
    } else if (tid < k) emit(tid, -INFINITY, 0x7fffffff);                       // fewer than k columns
    return;
  }
  unsigned left = 0;                                     // the values that have not been taken yet
#pragma unroll
  for (int e = 0; e < PER; ++e) left |= c[e] == c[e] && id_of(e) < (VEC > 0 ? V : 0x7fffffff) ? 1u << e : 0u;
  for (int r = 0; r < k; ++r) {
    float v = -INFINITY;
    int id = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if ((left >> e & 1) && better(c[e], id_of(e), v, id)) { v = c[e]; id = id_of(e); }
    const float top = block_max(v, sh);
    id = wave_min_i32(v == top ? id : 0x7fffffff);
    if (lane == 0) list_i[wave] = id;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) id = min(id, list_i[w]);
    if (tid == 0) emit(r, top, id);
#pragma unroll
    for (int e = 0; e < PER; ++e) left &= id_of(e) == id ? ~(1u << e) : ~0u;
    __syncthreads();
  }
}

static int topk_blocks(int n, int per) { return (n + per - 1) / per; }
static size_t topk_list_bytes(int rows, int n, int k) { return (size_t)rows * n * (k + 1) * 8; }
size_t row_topk_scratch_bytes(int rows, const TopkSegments& sg, int k) {
  int n0 = 0;
  for (int i = 0; i < sg.n; ++i) n0 += topk_blocks(sg.V[i], TOPK_TILE);
  if (n0 == 1) return 0;
  return topk_list_bytes(rows, n0, k) + topk_list_bytes(rows, topk_blocks(n0, TOPK_TILE / k), k);
}

template <typename T>
static void row_topk_typed(hipStream_t s, TopkSegments sg, int rows, int k, float* top_logp, int* top_id, float* lse, void* scratch) {
  auto list_at = [&](char* p, int n) {
    TopkList l;
    const size_t c = (size_t)rows * n * k, h = (size_t)rows * n;
    l.v = (float*)p; l.id = (int*)(p + c * 4); l.m = (float*)(p + c * 8); l.s = (float*)(p + c * 8 + h * 4);
    return l;
  };
  int n = 0, n_in = 0;
  const uintptr_t al = (uintptr_t)sg.z[0] | (uintptr_t)sg.ld[0] * sizeof(T);       // what every load's address is a multiple of
  for (int i = 0; i < sg.n; ++i) {
    sg.blk0[i] = n;
    n += topk_blocks(sg.V[i], TOPK_TILE);
  }
  sg.blk0[sg.n] = n;
  char* bufs[2] = {(char*)scratch, (char*)scratch + (n > 1 ? topk_list_bytes(rows, n, k) : 0)};
  TopkList out = list_at(bufs[0], n), in{};
  // (rows along x: y and z of a grid end at 65536)
#define TK(VEC, CLUSTERS) \
  hipLaunchKernelGGL((row_topk_kernel<T, VEC, CLUSTERS>), dim3(rows, n), dim3(TOPK_THREADS), 0, s, sg, in, n_in, k, out, top_logp, top_id, lse)
  const bool clusters = sg.n > 1;                        // (whose loads are always of 8 values)
  if (clusters) TK(8, true); else if (al % (8 * sizeof(T)) == 0) TK(8, false); else if (al % (2 * sizeof(T)) == 0) TK(2, false); else TK(1, false);
  for (int which = 1; n > 1; which ^= 1) {
    const bool first = n_in == 0;
    n_in = n;
    in = out;
    n = topk_blocks(n, TOPK_TILE / k);
    out = list_at(bufs[which], n);
    if (clusters && first) TK(0, true); else TK(0, false);
  }
#undef TK
}

void launch_row_topk(hipStream_t s, int dt, const TopkSegments& sg, int rows, int k, float* top_logp, int* top_id, float* lse, void* scratch) {
  if (rows <= 0) return;
  if (dt == F32) row_topk_typed<float>(s, sg, rows, k, top_logp, top_id, lse, scratch);
  else if (dt == F16) row_topk_typed<half_t>(s, sg, rows, k, top_logp, top_id, lse, scratch);
  else row_topk_typed<bf16_t>(s, sg, rows, k, top_logp, top_id, lse, scratch);
}

// out[r][col0 + v] = z[r][v] + off[r] - lse[r] in fp32 (test access to the full distribution); off: of row r at r * TOPK_SEGMENTS, or null
template <typename T>
__global__ __launch_bounds__(256) void logprob_rows_kernel(const T* __restrict__ z, int ldz, const float* __restrict__ off,
                                                           const float* __restrict__ lse, float* __restrict__ out, int ldo, int V) {
  const int row = blockIdx.y;
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= V) return;
  float v = to_f<T>(z[(size_t)row * ldz + col]);
  if (off) v += off[(size_t)row * TOPK_SEGMENTS];
  out[(size_t)row * ldo + col] = v - lse[row];
}
// rows r0 .. r0 + rows - 1 of the segments
void launch_logprob_rows(hipStream_t s, int dt, const TopkSegments& sg, const float* lse, float* out, int r0, int rows) {
  if (rows <= 0) return;
  const int ldo = sg.lo[sg.n - 1] + sg.V[sg.n - 1];
  for (int i = 0; i < sg.n; ++i) {
    dim3 grid((sg.V[i] + 255) / 256, rows), block(256);
    const float* off = i ? sg.off + (size_t)r0 * TOPK_SEGMENTS + i : nullptr;
#define LP(T) hipLaunchKernelGGL(logprob_rows_kernel<T>, grid, block, 0, s, (const T*)sg.z[i] + (size_t)r0 * sg.ld[i], sg.ld[i], off, lse + r0, out + sg.lo[i], ldo, sg.V[i])
    if (dt == F32) LP(float); else if (dt == F16) LP(half_t); else LP(bf16_t);
#undef LP
  }
}

}  // namespace tfm
