// MFMA GEMM for gfx950: C[M,N] = epilogue(op(A) op(B)), fp16 or bf16 operands, fp32 accumulation in the matrix
// cores (v_mfma_f32_32x32x16_{f16,bf16}).
//
// What bounds them on MI355X: a long one the power that the chip may draw (with normally distributed operands an MFMA loop alone stops at 1.64
// PFLOP/s and 1.65 GHz, one that also reads its fragments from LDS at 1.42; a K-step costs the same whether its tiles come from L2 or from
// beyond), a short one the 4-7 us around the K loop.  So the design moves few bytes per flop, spreads what it moves evenly and keeps
// the instructions that run once per launch few.
//
//  * Tiles: BM x BN output tile per block, K walked in steps of 32 or 64.  4 wavefronts up to 128x128 and for 192x128, 8 for larger ones, so
//    that a wavefront has 64x64 or more, and reads (1/64 + 1/64) fragment bytes per flop, half of what one of 32x32 reads.  (The two smallest tilings are for
//    launches that leave compute units idle: 64x128 has wavefronts of 32x64, 64x64 of 32x32.)  Which tiling: see plan_gemm.
//  * Fetch: CDNA4 direct-to-LDS buffer loads (buffer_load_dwordx4 ... lds): no staging registers and no ds_write on
//    the load path; range-checked, so ragged M and N read zeros without branches, and a ragged K is taken care of in the first K-step.  A
//    ring of 3 to 5 stages keeps two to four K-steps in flight; one barrier per K-step.  A lane's offsets never change (the K-step is the
//    scalar offset), and the loads are issued a few behind every MFMA: in one burst after the barrier they held up the wavefront
//    that issued them (256x256: 2550 clocks per 64 of K, spread 2300, the MFMAs alone 2048).  They are issued as assembly and tracked
//    with s_waitcnt vmcnt by hand, because the compiler would otherwise drain every outstanding direct-to-LDS load before each LDS read.
//  * LDS layout: unpadded tiles (the direct-to-LDS path writes 1 KB per wavefront contiguously), XOR-swizzled on the
//    global-address side so that fragment reads are bank-conflict free.  An operand whose contraction index is
//    contiguous in memory (A of "NT"/"NN", B of "NT") is staged [row][k] and read with ds_read_b128; an operand
//    whose contraction index is the slow one (B of "NN", both of "TN") is staged as it lies, [k][row], and read with
//    the LDS transpose read ds_read_b64_tr_b16 (a 16-lane group reads a 4(k) x 16(row) patch, each lane receives
//    the 4 k-values of one row).
//  * Math: fragments of a later sub-step of 16 k are read while the MFMAs of the current one execute (software pipeline
//    across the barrier, pinned with scheduling fences).  Accumulators are produced transposed (B fragment first), so
//    a lane holds 4 consecutive columns of one output row; the epilogue turns the tile around in LDS so that the
//    bias / ReLU / ReLU-mask / residual reads and the stores are whole 128-byte lines.
//  * Block ids are re-mapped so that each XCD (blocks are dealt round-robin to the 8 XCDs, each with its own L2) works
//    on a contiguous run of tiles.
//  * Weight gradients: a single projection's dY^T X has 16-256 output tiles, too few for 256 compute units.  The training
//    step therefore queues them and launches the tiles of up to 48 products end to end as ONE grouped launch
//    (gemm_mfma_grouped_kernel; problem table in the kernel arguments; the first tile column of each product also sums
//    the rows of dY^T it already holds as fragments, which is the bias gradient).
//  * Outputs with few tiles and a long contraction (input gradients of few rows, scores of a tail cluster, a weight gradient launched on
//    its own) split K across blockIdx.y; fp32 partial tiles are then added in a fixed order by a second kernel (no atomics, reproducible).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace tfm {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr uint32_t OOB = 0x80000000u;                   // beyond any buffer this kernel accepts: reads as zero

template <typename T> struct Mfma;
template <> struct Mfma<half_t> {
  static __device__ __forceinline__ f32x16 run(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mfma<bf16_t> {
  static __device__ __forceinline__ f32x16 run(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};

// x / d by one multiplication for x < limit: with m = ceil(2^32 / d), x * m / 2^32 exceeds x / d by less than x / 2^32, which does
// not reach the next whole number while x * d < 2^32.  (Beyond: m = 0, a division.)
struct Divisor {
  uint32_t d, m;
  __host__ void set(uint32_t by, uint32_t limit) { d = by; m = by > 1 && (uint64_t)by * limit < 0x100000000ull ? (uint32_t)((0x100000000ull + by - 1) / by) : 0u; }
  __device__ __forceinline__ uint32_t quotient(uint32_t x) const { return m ? __umulhi(x, m) : x / d; }
};
constexpr int GROUP_M = 8;

struct MfmaGemmParams {
  int M, N, K;
  const uint16_t* A; int lda;
  const uint16_t* B; int ldb;
  uint16_t* C; int ldc;
  const uint16_t* bias;
  int relu;
  const uint16_t* mask;
  const uint16_t* residual;
  int tiles_m, tiles_total;
  Divisor per_band, last_band;                           // tiles of a full band; tile rows of the last one if it is not full
  int ksteps_per_split;                                  // split-K: K-steps per blockIdx.y slice
  float* partial;                                        // split-K: fp32 partial tiles [split][M][N], else null
  uint32_t a_bytes, b_bytes;                             // extents for the range-checked loads
  uint64_t drop_key; uint32_t drop_thr; float inv_keep;  // dropout on the result (thr = 0: off), see GemmArgs
  float mask_scale;
  uint16_t* colsum;                                      // grouped weight gradients: [M] sums of A's rows over K (a bias gradient), or null
};

// Sum of the 8 values of a fragment register quadruple, added to c in fp32 (fixed order).
template <typename T> struct FragSum;
template <> struct FragSum<half_t> {
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ float run(u32x4 a, float c) {
    const f16x2 one = {(_Float16)1.f, (_Float16)1.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t word = a[w];                          // (a copy: bit-casting the vector element in place read element 0 every time)
      c = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, word), one, c, false);
    }
    return c;
  }
};
template <> struct FragSum<bf16_t> {
  static __device__ __forceinline__ float run(u32x4 a, float c) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t word = a[w];
      c += __uint_as_float(word << 16);
      c += __uint_as_float(word & 0xffff0000u);
    }
    return c;
  }
};

template <int I, int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) { f(std::integral_constant<int, I>{}); static_for<I + 1, N>(f); }
}

// One operand's path from global memory into the LDS ring.
//   ROWS: tile rows (M or N extent of the block tile);  NW: wavefronts in the block;  TR: see the file comment.
// A direct-to-LDS load writes the wavefront's 64 x 16 bytes contiguously, so piece g of a stage fills bytes
// [g*1024, (g+1)*1024) of the tile; each lane chooses WHICH global vector it fetches so that the tile ends up swizzled:
//   [row][k] tile, 2*BK-byte rows:   16-byte slot s of row r holds k-vector    s ^ swz(r)
//   [k][row] tile, ROWS*2-byte rows: 16-byte slot s of k-row k holds row-vector s ^ tswz(k)
// Every wavefront issues LOADS loads a stage, so that one vmcnt serves all of them; where the pieces do not divide by the wavefronts
// (192 rows on 8 of them), the last load of some fetches nothing and lands beside the ring.
template <int ROWS, int BK, int NW, bool TR>
struct Operand {
  static constexpr int TILE_BYTES = ROWS * BK * 2;
  static constexpr int PIECES = TILE_BYTES / 1024;
  static constexpr int LOADS = (PIECES + NW - 1) / NW;
  static constexpr bool EVEN = PIECES % NW == 0;
  static_assert(PIECES * 1024 == TILE_BYTES, "whole 1 KB pieces");
  static constexpr int ROW_BYTES = ROWS * 2;             // [k][row] layout only
  static constexpr int KROW_BYTES = BK * 2;              // [row][k] layout only: 64 or 128
  static constexpr int VPR = BK / 8;                     // 16-byte vectors per [row][k] row: 4 or 8
  // swizzle of the [row][k] layout: slot ^= f(row) with f chosen so that 16 consecutive rows cover 16 distinct
  // 16-byte bank groups: 64-byte rows: (row >> 2) & 3;  128-byte rows: (row >> 1) & 7
  static __device__ __forceinline__ int swz(int row) { return BK == 32 ? ((row >> 2) & 3) : ((row >> 1) & 7); }
  // of the [k][row] layout: the 4 k-rows of a transposing read lie in distinct 32-byte bank groups; rows of 256 bytes and more
  // start at the same bank, rows of 128 bytes at two
  static __device__ __forceinline__ int tswz(int k) { return ROWS == 64 ? (k & 3) << 1 : (k & 3) << 2; }
  static_assert(NW % 2 == 0 || NW == 1, "the swizzle repeats after one or two pieces, so that a lane's loads differ by a constant only");
  static constexpr int KPP = TR ? 1024 / ROW_BYTES : 0, RPPC = TR ? 0 : 64 / VPR;          // k-rows or rows of a piece
  uint32_t off[LOADS];                                   // byte offset of this lane's vector in K-step 0
  int kfirst;                                            // load 0's k index inside the K-step (for a ragged last K-step)
  uint32_t step;                                         // byte stride between K-steps

  // Bounds: the hardware compares these offsets, without the scalar one, with the operand's extent.  Rows beyond the matrix lie beyond
  // it; columns beyond the width of a [k][row] operand would not, so they get an offset that does; k beyond the end, see issue_ragged.
  __device__ __forceinline__ void init(int ld, int row0, int width, int wave, int lane) {
    if (!TR) {
      const int row = wave * RPPC + lane / VPR;
      kfirst = ((lane % VPR) ^ swz(row)) * 8;
      off[0] = ((uint32_t)(row0 + row) * (uint32_t)ld + (uint32_t)kfirst) * 2u;
    } else {
      const int slot = lane % (ROW_BYTES / 16);
      kfirst = wave * KPP + lane / (ROW_BYTES / 16);
      const int col = row0 + (slot ^ tswz(kfirst)) * 8;
      off[0] = col < width ? ((uint32_t)kfirst * (uint32_t)ld + (uint32_t)col) * 2u : OOB;
    }
    const uint32_t by = (uint32_t)(NW * (TR ? KPP : RPPC)) * (uint32_t)ld * 2u;
#pragma unroll
    for (int i = 1; i < LOADS; ++i) off[i] = off[i - 1] + by;                              // (OOB + less than 2^31 stays out of range)
    if (!EVEN && (LOADS - 1) * NW + wave >= PIECES) off[LOADS - 1] = OOB;
    step = TR ? (uint32_t)BK * (uint32_t)ld * 2u : (uint32_t)BK * 2u;
  }
  // Load i of a stage: `soff` = byte offset of the K-step, `dst` = LDS address of the stage's tile plus wave * 1024, `dump` = 1 KB of
  // LDS for a load without a piece.  Issued as assembly on purpose (see the file comment); the instruction between the write of m0
  // and the load that reads it is a required wait state.
  template <int i> __device__ __forceinline__ void issue(const u32x4& rsrc, uint32_t soff, uint32_t dst, uint32_t dump, int wave, uint32_t o) const {
    uint32_t to = dst + i * NW * 1024;
    if (!EVEN && i == LOADS - 1) to = i * NW + wave < PIECES ? to : dump;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(__builtin_amdgcn_readfirstlane(to)), "v"(o),
                 "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane(soff))
                 : "memory", "m0");
  }
  template <int i> __device__ __forceinline__ void issue(const u32x4& rsrc, uint32_t soff, uint32_t dst, uint32_t dump, int wave) const {
    issue<i>(rsrc, soff, dst, dump, wave, off[i]);
  }
  // the same for K-step kt, of which only the k below kend are read
  template <int i> __device__ __forceinline__ void issue_ragged(const u32x4& rsrc, int kt, int kend, uint32_t dst, uint32_t dump, int wave) const {
    const bool in = kt * BK + kfirst + i * NW * KPP < kend && off[i] < OOB;
    issue<i>(rsrc, 0u, dst, dump, wave, in ? off[i] + (uint32_t)kt * step : OOB);
  }
};

// The fragments a wavefront reads of one operand: TILES row tiles of 32, KKW sub-steps of 16 k.  The addresses follow the ring (one
// addition each per K-step); the row tile or the sub-step, whichever the swizzle does not depend on, is an immediate offset.
template <int ROWS, int BK, bool TR, int TILES, int KKW>
struct Frags {
  static constexpr int NA = TR ? TILES : KKW;
  typedef Operand<ROWS, BK, 1, TR> O;
  uint32_t at[NA];
  // rows r0 .. r0 + 32 * TILES - 1 of the tile at LDS address `base`
  __device__ __forceinline__ void init(uint32_t base, int r0, int lane) {
    if constexpr (!TR) {
      const int row = r0 + (lane & 31);
#pragma unroll
      for (int k = 0; k < KKW; ++k) at[k] = base + row * O::KROW_BYTES + ((k * 2 + (lane >> 5)) ^ O::swz(row)) * 16;
    } else {
      const int s = lane & 15, ibase = lane & 16;
      const int k = (lane >> 5) * 8 + (s >> 2);
#pragma unroll
      for (int i = 0; i < TILES; ++i)                    // (32-byte segments)
        at[i] = base + k * O::ROW_BYTES + (((r0 + i * 32 + ibase) >> 4) ^ (O::tswz(k) >> 1)) * 32 + (s & 3) * 8;
    }
  }
  __device__ __forceinline__ void move(uint32_t by) {
#pragma unroll
    for (int i = 0; i < NA; ++i) at[i] += by;
  }
  // Row tile i, sub-step kk: lane l gets row 32 i + l % 32, k-group l / 32 (8 k-values).
  __device__ __forceinline__ u32x4 get(int i, int kk) const {
    if constexpr (!TR) {
      typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
      return *(lds_u32x4*)(uintptr_t)(at[kk] + i * 32 * O::KROW_BYTES);
    } else {
      typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
      const uint32_t p = at[i] + kk * 16 * O::ROW_BYTES;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)p);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(p + 4 * O::ROW_BYTES));
      const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
      return u32x4{l2[0], l2[1], h2[0], h2[1]};
    }
  }
};

// One output tile (or one K-slice of it).  `tile` is the tile id inside this problem after the XCD re-mapping, `slice`
// the split-K slice.  AHEAD: sub-steps between a fragment's read and its use.  CS: the block column tn == 0 also sums A's rows
// over K (see MfmaGemmParams::colsum).
template <typename T, int BM, int BN, int WM, int WN, int BK, int STAGES, int AHEAD, bool ATR, bool BTR, bool CS>
__device__ __forceinline__ void gemm_mfma_tile(const MfmaGemmParams& p, int tile, int slice) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;    // MFMA tiles per wavefront
  constexpr int KK = BK / 16;                            // MFMA sub-steps per K-step
  constexpr int D = STAGES - 1;                          // K-steps in flight ahead of the one being consumed
  constexpr int SETS = AHEAD == 1 ? 2 : KK;              // register sets of fragments
  static_assert(KK % SETS == 0 && AHEAD < SETS, "a sub-step uses the same registers in every K-step, and never those that are being filled");
  static_assert(STAGES >= 3, "the loads of a K-step are spread over the one before the last that needs the slot");
  typedef Operand<BM, BK, NW, ATR> OA;
  typedef Operand<BN, BK, NW, BTR> OB;
  // One LDS block: the ring (a slot holds a stage of A and of B), and (re-using it once the K loop is over) the epilogue's
  // staging area.
  constexpr int SW = TN * 32;                             // epilogue strip width in columns
  constexpr int SP = SW + 4;                              // its padded pitch in floats: conflict-free for both passes
  constexpr uint32_t SLOT = OA::TILE_BYTES + OB::TILE_BYTES;
  constexpr int RING_BYTES = STAGES * SLOT + (OA::EVEN && OB::EVEN ? 0 : 1024);
  constexpr int STRIP_BYTES = NW * 32 * SP * 4;
  constexpr int HP = SW + 8;                              // pitch in elements of the tile turned around in the output type
  constexpr int BOX_BYTES = NW * TM * 32 * HP * 2;
  constexpr int EPI_BYTES = BOX_BYTES > STRIP_BYTES ? BOX_BYTES : STRIP_BYTES;
  constexpr int LDS_BYTES = RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS per CU");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS_BYTES];
  // Tile ids run column-major inside bands of GROUP_M tile rows, so the run of ids an XCD works on at one time
  // covers a compact patch of the output and shares its A and B panels in that XCD's L2.
  const uint32_t band = p.per_band.quotient(tile), in_band = tile - band * p.per_band.d;
  const bool full = (band + 1) * GROUP_M <= (uint32_t)p.tiles_m;
  const int tn = full ? in_band / GROUP_M : p.last_band.quotient(in_band);
  const int tm = band * GROUP_M + (full ? in_band % GROUP_M : in_band - tn * p.last_band.d);
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // raw buffer descriptors: base, stride 0, byte extent, format word
  u32x4 ra = {(uint32_t)(uintptr_t)p.A, (uint32_t)((uintptr_t)p.A >> 32) & 0xffffu, p.a_bytes, 0x00020000u};
  u32x4 rb = {(uint32_t)(uintptr_t)p.B, (uint32_t)((uintptr_t)p.B >> 32) & 0xffffu, p.b_bytes, 0x00020000u};
  // split-K: this block covers K-steps kt0 .. kt0 + nk - 1 (nk may be 0).  A ragged last K-step is taken first: only the first one's loads test k.
  const int kt0 = slice * p.ksteps_per_split;
  const int nk = max(0, min(p.ksteps_per_split, (p.K + BK - 1) / BK - kt0));
  const bool ragged = nk > 0 && (kt0 + nk) * BK > p.K;
  OA oa;
  OB ob;
  oa.init(p.lda, m0, p.M, wave, lane);
  ob.init(p.ldb, n0, p.N, wave, lane);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)(&smem[0]), dump = lds0 + STAGES * SLOT;
  const uint32_t lds_a = lds0 + wave * 1024, lds_b = lds0 + OA::TILE_BYTES + wave * 1024;
  constexpr int LT = OA::LOADS + OB::LOADS;
  uint32_t sa = (uint32_t)kt0 * oa.step, sb = (uint32_t)kt0 * ob.step;                     // byte offsets of the K-step that is fetched next
  int fetched = 0;                                        // K-steps asked for
  auto issue = [&](auto l, uint32_t slot) __attribute__((always_inline)) {
    constexpr int L = decltype(l)::value;
    if constexpr (L < OA::LOADS) oa.template issue<L>(ra, sa, lds_a + slot, dump, wave);
    else ob.template issue<L - OA::LOADS>(rb, sb, lds_b + slot, dump, wave);
  };
  // K-steps beyond the last fetch nothing: no bytes in range, and no scalar offset either
  auto next_step = [&]() __attribute__((always_inline)) {
    sa += oa.step;
    sb += ob.step;
    if (++fetched >= nk) { sa = sb = 0u; ra[2] = rb[2] = 0u; }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  u32x4 fa[SETS][TM], fb[SETS][TN];
  Frags<BM, BK, ATR, TM, KK> ga;
  Frags<BN, BK, BTR, TN, KK> gb;
  ga.init(lds0, wm * (BM / WM), lane);
  gb.init(lds0 + OA::TILE_BYTES, wn * (BN / WN), lane);
  // fragment r of a sub-step, in the order in which its MFMAs need them
  auto read = [&](int set, int kk, int r) __attribute__((always_inline)) {
    if (r == 0) fa[set][0] = ga.get(0, kk);
    else if (r <= TN) fb[set][r - 1] = gb.get(r - 1, kk);
    else fa[set][r - TN] = ga.get(r - TN, kk);
  };
  constexpr int R = TM + TN, NM = TM * TN;
  // Row sums of A: the wavefronts of the first tile column that hold the first column strip see every A fragment of
  // their rows exactly once (K-steps beyond the slice read zeros), so they add them up on the vector ALU beside the MFMAs.
  const bool do_cs = CS && p.colsum != nullptr && tn == 0 && wn == 0;
  float cs[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) cs[i] = 0.f;

  constexpr int WAIT = LT * (D - 1);                      // loads that may still be in flight when a K-step must have landed
  static_assert(WAIT <= 63, "vmcnt is a 6-bit count");
  // s_waitcnt immediate: vmcnt[3:0] in bits 3:0 and vmcnt[5:4] in bits 15:14, expcnt (6:4) at its maximum, lgkmcnt (11:8) 0: this
  // wavefront's reads of the slot that is given up have returned as well
  constexpr int WAITCNT = 0x0070 | (WAIT & 15) | ((WAIT >> 4) << 14);
  if (ragged || nk == 0) {
    const int kt = kt0 + nk - 1, kend = nk > 0 ? p.K : 0;
    static_for<0, OA::LOADS>([&](auto l) { oa.template issue_ragged<decltype(l)::value>(ra, kt, kend, lds_a, dump, wave); });
    static_for<0, OB::LOADS>([&](auto l) { ob.template issue_ragged<decltype(l)::value>(rb, kt, kend, lds_b, dump, wave); });
    sa -= oa.step;
    sb -= ob.step;
  } else {
    static_for<0, LT>([&](auto l) { issue(l, 0u); });
  }
  next_step();
  static_for<1, D>([&](auto t) {
    static_for<0, LT>([&](auto l) { issue(l, decltype(t)::value * SLOT); });
    next_step();
  });
  __builtin_amdgcn_s_waitcnt(WAITCNT);                    // K-step 0 has landed
  asm volatile("s_barrier" ::: "memory");
  static_for<0, AHEAD>([&](auto j) { static_for<0, R>([&](auto r) { read(decltype(j)::value, decltype(j)::value, decltype(r)::value); }); });
  // Software pipeline: while the MFMAs of one sub-step run, the fragments of the sub-step AHEAD of it are read from LDS and a few
  // of the loads of K-step kt + D are issued, one behind every MFMA (the scheduling fences keep that order), so that neither LDS
  // nor the loads' path sees a burst.  In sub-step KK - AHEAD the next K-step must have landed: wait, barrier, and the slot of this
  // one is free; its successor D K-steps on is asked for during the next K-step.
  uint32_t slot = 0, freed = (STAGES - 1) * SLOT;
  for (int kt = 0; kt < nk; ++kt) {
    const uint32_t next = slot == (STAGES - 1) * SLOT ? 0u : slot + SLOT, by = next - slot;
    static_for<0, KK>([&](auto jc) {
      constexpr int j = decltype(jc)::value, to = j + AHEAD, set = j % SETS;
      constexpr int Q = NM / 2;                           // the barrier stands before this MFMA of its sub-step
      static_for<0, NM>([&](auto qc) {
        constexpr int q = decltype(qc)::value, i = q / TN, jj = q % TN;
        if constexpr (to == KK && q == Q) {
          ga.move(by);
          gb.move(by);
          __builtin_amdgcn_s_waitcnt(WAITCNT);
          asm volatile("s_barrier" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        acc[i][jj] = Mfma<T>::run(fb[set][jj], fa[set][i], acc[i][jj]);                   // transposed product: D'[n][m]
        if constexpr (to != KK) {
          static_for<q * R / NM, (q + 1) * R / NM>([&](auto r) { read(to % SETS, to % KK, decltype(r)::value); });
        } else if constexpr (q >= Q) {
          static_for<(q - Q) * R / (NM - Q), (q - Q + 1) * R / (NM - Q)>([&](auto r) { read(to % SETS, 0, decltype(r)::value); });
        }
        constexpr int g = j * NM + q, G = (KK - AHEAD) * NM + Q;                           // G MFMAs stand before the barrier
        if constexpr (g < G) static_for<g * LT / G, (g + 1) * LT / G>([&](auto l) { issue(l, freed); });
        __builtin_amdgcn_sched_barrier(0);
      });
      if (CS && do_cs) {
#pragma unroll
        for (int i = 0; i < TM; ++i) cs[i] = FragSum<T>::run(fa[set][i], cs[i]);
      }
    });
    freed = slot;
    slot = next;
    next_step();
  }
  __builtin_amdgcn_s_waitcnt(0x0070);                    // drain the trailing (empty) loads before the ring is re-used
  __syncthreads();
  // Epilogue.  The accumulators hold, per lane, 4 consecutive columns of one row, which would make every store an
  // 8-byte fragment of a different cache line.  Each wavefront therefore turns its tile around in its own slice of LDS (free
  // now: every wavefront is past its last fragment read), so that 8 lanes store one whole 128-byte line of the output.
  // The steps that few products have (dropout, a factor behind the mask) are compiled apart: the instructions of an epilogue are
  // fetched as it runs, once per launch and compute unit, and jumping over unrolled steps took 3 us of a launch (128x128 of
  // X W^T, K = 1024: 13.7 us against 10.7 us; 256x256 34.1 against 30.8).
  const int mw = m0 + wm * (BM / WM) ;   // first row of this wavefront's tile
  const T* bias = reinterpret_cast<const T*>(p.bias);
  const T* mask = reinterpret_cast<const T*>(p.mask);
  const T* res = reinterpret_cast<const T*>(p.residual);
  T* C = reinterpret_cast<T*>(p.C);
  float* P = p.partial ? p.partial + (size_t)slice * p.M * p.N : nullptr;
  if (CS && do_cs) {                                      // lanes l and l + 32 hold the two k-groups of row l
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const float t = cs[i] + __shfl_xor(cs[i], 32);
      const int m = m0 + wm * (BM / WM) + i * 32 + (lane & 31);
      if (lane < 32 && m < p.M) reinterpret_cast<T*>(p.colsum)[m] = from_f<T>(t);
    }
  }
  constexpr int LPR = SW / 8, RPP = 64 / LPR;             // lanes per row and rows per pass when re-reading: 8 columns a lane
  const int cr = (lane % LPR) * 8, nr = n0 + wn * (BN / WN) + cr, mr = mw + lane / LPR;    // (8 columns entirely inside or outside N)
  if (!res && !P) {
    // Bias, ReLU, dropout and the mask's factor are applied to the accumulators and the finished values go through LDS in the
    // output type, the whole tile before the first of it is read back.  (Against fp32 strips with the epilogue's steps on the far
    // side, averages inside a step: 192x256 tiles of X W^T 37.9 -> 35.5 us, 128x128 of a 1536-wide dY W 159 -> 145.)
    T* box = reinterpret_cast<T*>(smem) + wave * (TM * 32 * HP);
    const int nw = n0 + wn * (BN / WN) + (lane >> 5) * 4;
    auto fill = [&](auto relu, auto general) __attribute__((always_inline)) {
      Pack<T, 4> braw[TN][4];
      if (bias) {                                         // all of a lane's pieces in one trip to memory
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) braw[j][rg] = *reinterpret_cast<const Pack<T, 4>*>(bias + min(nw + j * 32 + rg * 8, p.N - 4));
      } else {
        __builtin_memset(braw, 0, sizeof(braw));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const int c = j * 32 + rg * 8 + (lane >> 5) * 4, n = nw + j * 32 + rg * 8;
          float bb[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) bb[e] = to_f<T>(braw[j][rg].v[e]);
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const int r = i * 32 + (lane & 31);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[i][j][rg * 4 + e] + bb[e];
            if (decltype(relu)::value || (decltype(general)::value && p.relu)) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
            }
            if constexpr (decltype(general)::value) {
              if (p.drop_thr) drop_apply<4>(v, p.drop_key, (uint64_t)(mw + r) * p.N + n, p.drop_thr, p.inv_keep);
              if (mask) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] *= p.mask_scale;
              }
            }
            store_f<T, 4>(box + r * HP + c, v);
          }
        }
    };
    if (p.drop_thr || (mask && p.mask_scale != 1.f)) fill(std::false_type{}, std::true_type{});
    else if (p.relu) fill(std::true_type{}, std::false_type{});
    else fill(std::false_type{}, std::false_type{});
    asm volatile("" ::: "memory");                        // (LDS operations of one wavefront complete in order)
    constexpr int PASSES = TM * 32 / RPP;
    if (nr >= p.N) return;
    if (mask) {
      // The masks are asked for all at once: between the stores, which may alias them, each pass would wait for its own.  (Here and
      // not further up: beside the accumulators they would not fit.)
      u32x4 keep[PASSES];
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps)
        keep[ps] = *reinterpret_cast<const u32x4*>(mask + (size_t)min(mr + ps * RPP, p.M - 1) * p.ldc + nr);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) {
        u32x4 v = *reinterpret_cast<const u32x4*>(box + (ps * RPP + lane / LPR) * HP + cr);
        if (mr + ps * RPP >= p.M) continue;
        Pack<T, 8> k;
        __builtin_memcpy(&k, &keep[ps], 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] &= (to_f<T>(k.v[2 * e]) > 0.f ? 0x0000ffffu : 0u) | (to_f<T>(k.v[2 * e + 1]) > 0.f ? 0xffff0000u : 0u);
        *reinterpret_cast<u32x4*>(C + (size_t)(mr + ps * RPP) * p.ldc + nr) = v;
      }
    } else {
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(box + (ps * RPP + lane / LPR) * HP + cr);
        if (mr + ps * RPP < p.M) *reinterpret_cast<u32x4*>(C + (size_t)(mr + ps * RPP) * p.ldc + nr) = v;
      }
    }
    return;
  }
  // With a residual to add before the one rounding, or as a split-K slice: in fp32, one 32 x (TN*32) strip at a time.
  // out(i, ps, m, w): the 8 values from column nr of row m, pass ps of row tile i
  constexpr int PASSES = 32 / RPP;
  auto strips = [&](auto out) __attribute__((always_inline)) {
    float* strip = reinterpret_cast<float*>(smem) + wave * (32 * SP);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          float4 v = {acc[i][j][rg * 4], acc[i][j][rg * 4 + 1], acc[i][j][rg * 4 + 2], acc[i][j][rg * 4 + 3]};
          *reinterpret_cast<float4*>(strip + (lane & 31) * SP + j * 32 + rg * 8 + (lane >> 5) * 4) = v;
        }
      // (LDS operations of one wavefront complete in order: the reads below see the writes above)
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) {
        const int m = mr + i * 32 + ps * RPP;
        const float* at = strip + (ps * RPP + lane / LPR) * SP + cr;
        const float4 lo = *reinterpret_cast<const float4*>(at), hi = *reinterpret_cast<const float4*>(at + 4);
        float w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        if (m < p.M && nr < p.N) out(i, ps, m, w);
      }
    }
  };
  if (P) {                                                // split-K: raw fp32 tile, summed by splitk_reduce_kernel
    strips([&](int, int, int m, float (&w)[8]) __attribute__((always_inline)) { store_f<float, 8>(P + (size_t)m * p.N + nr, w); });
  } else if (!bias && !p.relu && !p.drop_thr && !mask) {  // an input gradient
    u32x4 add[TM][PASSES];                               // the whole tile's in one trip to memory: behind a store each strip's would be waited for
    if (nr < p.N) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps)
          add[i][ps] = *reinterpret_cast<const u32x4*>(res + (size_t)min(mr + i * 32 + ps * RPP, p.M - 1) * p.ldc + nr);
    }
    strips([&](int i, int ps, int m, float (&w)[8]) __attribute__((always_inline)) {
      Pack<T, 8> k;
      __builtin_memcpy(&k, &add[i][ps], 16);
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] += to_f<T>(k.v[e]);
      store_f<T, 8>(C + (size_t)m * p.ldc + nr, w);
    });
  } else {
    strips([&](int, int, int m, float (&w)[8]) __attribute__((always_inline)) {
      float k[8];
      if (bias) {
        load_f<T, 8>(bias + nr, k);
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] += k[e];
      }
      if (p.relu) {
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = fmaxf(w[e], 0.f);
      }
      if (p.drop_thr) drop_apply<8>(w, p.drop_key, (uint64_t)m * p.N + nr, p.drop_thr, p.inv_keep);
      const size_t o = (size_t)m * p.ldc + nr;
      if (mask) {
        load_f<T, 8>(mask + o, k);
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = k[e] > 0.f ? w[e] * p.mask_scale : 0.f;
      }
      load_f<T, 8>(res + o, k);
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] += k[e];
      store_f<T, 8>(C + o, w);
    });
  }
}

// XCD-aware block order: hardware deals block b to XCD b % 8; give each XCD a contiguous run of tile ids
__device__ __forceinline__ int xcd_tile(int b, int nb) {
  const int q = nb >> 3, r = nb & 7, x = b & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}

template <typename T, int BM, int BN, int WM, int WN, int BK, int STAGES, int AHEAD, bool ATR, bool BTR>
__global__ __launch_bounds__(64 * WM * WN) void gemm_mfma_kernel(MfmaGemmParams p) {
  gemm_mfma_tile<T, BM, BN, WM, WN, BK, STAGES, AHEAD, ATR, BTR, false>(p, xcd_tile(blockIdx.x, p.tiles_total), blockIdx.y);
}

// Grouped weight gradients: one launch covers the tiles of up to GROUP_MAX independent products C_i = A_i^T B_i (each
// with its own shapes and, optionally, the row sums of A_i^T as a bias gradient).  A single projection's weight gradient
// has 16-256 tiles, too few to fill 256 compute units for more than a fraction of a round; the tiles of many of them
// laid end to end do.  The table travels in the kernel arguments.
constexpr int GROUP_MAX = 48;
struct GroupedProblem {
  const uint16_t* A; const uint16_t* B; uint16_t* C; uint16_t* colsum;
  int M, N, K, lda, ldb, ldc, tile_begin, tiles_m, tiles_n;
  uint32_t band_m, last_m;                               // multipliers of the two Divisors
};
struct GroupedTable {
  int n, tiles_total;
  GroupedProblem pr[GROUP_MAX];
};
static_assert(sizeof(GroupedTable) <= 4096, "kernel argument space");

template <typename T, int BM, int BN, int WM, int WN, int BK, int STAGES>
__global__ __launch_bounds__(64 * WM * WN) void gemm_mfma_grouped_kernel(GroupedTable tab) {
  const int tile = xcd_tile(blockIdx.x, tab.tiles_total);
  int pi = 0;
  for (int i = 1; i < tab.n; ++i) pi = tile >= tab.pr[i].tile_begin ? i : pi;
  const GroupedProblem& g = tab.pr[pi];
  MfmaGemmParams p;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.A = g.A; p.lda = g.lda; p.B = g.B; p.ldb = g.ldb; p.C = g.C; p.ldc = g.ldc;
  p.bias = nullptr; p.relu = 0; p.mask = nullptr; p.residual = nullptr;
  p.tiles_m = g.tiles_m; p.tiles_total = 0; p.per_band = {(uint32_t)(GROUP_M * g.tiles_n), g.band_m}; p.last_band = {(uint32_t)g.tiles_m % GROUP_M, g.last_m};
  p.ksteps_per_split = (g.K + BK - 1) / BK;
  p.partial = nullptr;
  p.a_bytes = (uint32_t)(((g.K - 1) * g.lda + g.M) * 2); p.b_bytes = (uint32_t)(((g.K - 1) * g.ldb + g.N) * 2);   // (below 2^31: wgrad_group_supported)
  p.colsum = g.colsum;
  p.drop_key = 0; p.drop_thr = 0; p.inv_keep = 1.f; p.mask_scale = 1.f;
  gemm_mfma_tile<T, BM, BN, WM, WN, BK, STAGES, 1, true, true, true>(p, tile - g.tile_begin, 0);
}

// C[m, n] = epilogue(sum over splits (fixed order) of partial[s][m][n]); epilogue = optional bias[n], ReLU, residual [M, N] of stride ldc
template <typename T>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, int splits, int M, int N, T* __restrict__ C, int ldc,
                                                            const T* __restrict__ bias, int relu, const T* __restrict__ residual) {
  const size_t idx = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  const size_t total = (size_t)M * N;
  if (idx >= total) return;
  float4 a = *reinterpret_cast<const float4*>(partial + idx);
  for (int s = 1; s < splits; ++s) {
    const float4 b = *reinterpret_cast<const float4*>(partial + (size_t)s * total + idx);
    a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
  }
  const int m = (int)(idx / N), n = (int)(idx % N);
  float v[4] = {a.x, a.y, a.z, a.w};
  if (bias) {
    float bb[4];
    load_f<T, 4>(bias + n, bb);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += bb[e];
  }
  if (relu) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
  }
  if (residual) {
    float k[4];
    load_f<T, 4>(residual + (size_t)m * ldc + n, k);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += k[e];
  }
  store_f<T, 4>(C + (size_t)m * ldc + n, v);
}

void launch_splitk_reduce(hipStream_t s, int dt, const float* partial, int splits, int M, int N, void* C, int ldc, const void* bias, int relu,
                          const void* residual) {
  const size_t quads = ((size_t)M * N + 3) / 4;
  dim3 grid((unsigned)((quads + 255) / 256)), block(256);
  if (dt == F16) hipLaunchKernelGGL((splitk_reduce_kernel<half_t>), grid, block, 0, s, partial, splits, M, N, (half_t*)C, ldc, (const half_t*)bias, relu, (const half_t*)residual);
  else if (dt == BF16) hipLaunchKernelGGL((splitk_reduce_kernel<bf16_t>), grid, block, 0, s, partial, splits, M, N, (bf16_t*)C, ldc, (const bf16_t*)bias, relu, (const bf16_t*)residual);
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// bytes spanned by a [rows, width] view with row stride ld (elements of 2 bytes)
static uint64_t extent_bytes(int rows, int width, int ld) { return ((uint64_t)(rows - 1) * ld + width) * 2ull; }

bool gemm_mfma_supported(const GemmArgs& a) {
  if (a.dt != F16 && a.dt != BF16) return false;
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return false;
  // every 16-byte vector must lie entirely inside or outside the matrix and be aligned
  const bool a_tr = a.form == 2, b_tr = a.form != 0;
  if ((a_tr ? a.M : a.K) % 8 || (b_tr ? a.N : a.K) % 8 || a.N % 8) return false;
  if (a.lda % 8 || a.ldb % 8 || a.ldc % 8) return false;
  if (!aligned16(a.A) || !aligned16(a.B) || !aligned16(a.C)) return false;
  if (a.bias && !aligned16(a.bias)) return false;
  if (a.mask && !aligned16(a.mask)) return false;
  if (a.residual && !aligned16(a.residual)) return false;
  // 32-bit byte offsets in the range-checked loads, including the rows of a ragged last tile
  const uint64_t lim = 0x7f000000ull;
  const uint64_t ea = a_tr ? extent_bytes(a.K + 256, a.M + 256, a.lda) : extent_bytes(a.M + 256, a.K + 256, a.lda);
  const uint64_t eb = b_tr ? extent_bytes(a.K + 256, a.N + 256, a.ldb) : extent_bytes(a.N + 256, a.K + 256, a.ldb);
  if (ea >= lim || eb >= lim) return false;
  return true;
}

// The tilings, and what a launch of each costs.  In a round (one tile on every compute unit, two of 64x64) a K-step of 64 takes `few` us when
// hardly a tile runs and `one` when every compute unit has one: the clock follows the power that is drawn (2.4 GHz on zeros, 1.5-1.7 on
// normally distributed operands with all matrix cores busy), and the memory system is shared.  Two tiles on a compute unit take `two` where
// all of them have two and `some` where hardly any has.  `first` us is launch, fetch of the instructions, first trip to memory
// and epilogue; later rounds overlap some of that.  Fitted to 830 products (X W^T with bias and ReLU, dY W with residual or mask; fp16 and
// bf16), each on every tiling, launches back to back out of a graph over 12 sets of operands, or 600 MB of them: 350 of the models' (widths 512-2048,
// 250-4200 rows) and 480 of 65-4100 rows with 64-32768 columns and K = 64-32768.  The tiling with the least cost is 1.2 % slower than the
// best of the seven on average, up to 11 % in 95 of 100 products and 28 % at most (3064 x 20000, K = 256).  Most of that is `some` of 64x64, which is not
// from these but from training steps of 12 blocks, whose operands come from memory and whose clock is higher; by the products alone 0.424 it
// would be (0.4 %, 2 %).  ms a step, with 0.424 and 0.3: 264 tiles (2100 x 512) 2.25 and 2.19, 272 (1060 x 1024) 3.70 and 3.58, 288 (720 x 1536) 5.77 and
// 5.61, 312 (800 x 1536) 5.81 and 5.70, 328 (2600 x 512) 2.33 and 2.34, 336 (1300 x 1024) 3.82 and 3.92, 360 (900 x 1536) 5.89 and 5.93; with 0.28 the last
// one 6.18.  (Of 4 blocks, whose operands stay in the cache, 0.424 is the better one from 300 tiles on.)
//   tiling     wavefronts  K-step  ring      measured: rows x columns x K (us; in brackets 128x128 on 16 wavefronts, 64x128 on 8 of
//                                            32x32, 192x256 and 256x256 with a ring of two, loads issued in one burst after the barrier)
//   256x256      2 x 4       32     4        4096 x 4096 x 1024 NN 36.5 (39.8); 3264 x 4096 x 1024 33.1 (34.5), NN with a mask 37.9 (43.1)
//   256x128      4 x 2       64     3        3000 x 8192 x 1536 77.9 (81.9)
//   192x256      2 x 4       32     4        3264 x 3072 x 1024 28.8 (29.8)
//   192x128      2 x 2       64     3        3000 x 1536 x 4608 NN 55.3, 3000 x 1536 x 8192 89.3 (288 tiles of 128x128 in two rounds: 76.1, 122)
//   128x128      2 x 2       64     4        4096 x 1024 x 4096 NN 42.7 (44.3), 3264 x 1024 x 1024 11.2 (11.8)
//    64x128      2 x 2       64     4        3520 x 512 x 1536 NN 11.0 (11.8)
//    64x64       2 x 2       64     5, 4     280 x 1024 x 3072 NN, K in 3 slices, 10.4 (24 tiles of 128x128: 22.0).  5 slots for X W^T where a compute unit has one tile:
//                                            few rows find their weights in memory, and a fourth K-step in flight covers more of that trip.  Two tiles
//                                            cover each other's.  5 / 4 slots: 290 x 3072 x 1024 (240 tiles) 7.1/7.2, 900 x 512 x 2048 9.3/9.6, 500 x 1024 x
//                                            1024 6.3/6.6; 290 x 4096 x 1024 (320 tiles) 11.1/10.8, NN 10.0/9.5, 900 x 1536 x 512 7.0/6.7, 3300 x 512 x 512 7.3/7.0;
//                                            the kernels of a decoder block for 268 rows 71.0 / 73.8 (6 slots 71.0, 7 71.6).  Of 119 such products with K = 512-8192
//                                            4.1 % on average, at most 1.2 % slower; of 101 dY W, which read the weights along their rows, 0.2 % slower, up to
//                                            2.5: those keep 4
//   128x128      2 x 2       32     3        A^T B alone, up to 512 tiles, two on a compute unit: 6144 x 1024 x 190 7.6 (one: 10.1), 3072 x 1536 x 2902
//                                            41.2 (48.2)
// Wavefronts of 64x64 or more read half of the LDS bytes per flop of 32x32 ones.  Measured and dropped: 256x256 on 4 wavefronts of 128x128 (one per
// SIMD: 8 % slower), rings of five slots elsewhere (equal; 64x128 up to 4 % slower), two groups of wavefronts with half of the K-steps each (2 us more per launch for
// the exchange, 3 % less per K-step); over the 480 products also 128x128 on 16 wavefronts, 128x128 with K-steps of 32 and
// 64x128 on 8 wavefronts: with them to choose from the best is 0.4-0.8 % faster.
enum Tiling { T256x256, T256x128, T192x256, T192x128, T128x128, T64x128, T64x64, T128x128_PAIRS, TILINGS };
struct TilingCost { int bm, bn; float first, later, few, one, some, two; };
static const TilingCost TILING[TILINGS] = {{256, 256, 8.1f, 6.5f, 0.878f, 1.73f, 0.f, 0.f}, {256, 128, 5.85f, 3.75f, 0.438f, 0.925f, 0.f, 0.f},
    {192, 256, 6.85f, 4.45f, 0.711f, 1.48f, 0.f, 0.f}, {192, 128, 5.25f, 2.8f, 0.37f, 0.77f, 0.f, 0.f}, {128, 128, 4.2f, 2.4f, 0.327f, 0.58f, 0.f, 0.f},
    {64, 128, 3.1f, 1.95f, 0.257f, 0.38f, 0.f, 0.f}, {64, 64, 2.9f, 1.85f, 0.18f, 0.247f, 0.3f, 0.424f}, {128, 128, 3.5f, 2.5f, 0.4f, 0.877f, 1.144f, 1.144f}};
static long tiles_of(Tiling t, int M, int N) { return (long)((M + TILING[t].bm - 1) / TILING[t].bm) * ((N + TILING[t].bn - 1) / TILING[t].bn); }
static float launch_cost(Tiling t, long tiles, int ksteps) {
  const TilingCost& c = TILING[t];
  const bool pairs = c.two > 0.f;
  const long full = tiles >> (pairs ? 9 : 8), rest = tiles & (pairs ? 511 : 255);
  float step = (float)full * (pairs ? c.two : c.one);
  if (rest) step += rest > 256 ? c.some + (c.two - c.some) * (1.f / 256.f) * (float)(rest - 256) : c.few + (c.one - c.few) * (1.f / 256.f) * (float)rest;
  return c.first + (float)(full + (rest ? 1 : 0) - 1) * c.later + step * (float)ksteps;
}

// X W^T and dY W with too few tiles of 64x64 for the chip (few rows, or a narrow output): K in slices, so that the other operand streams through
// more compute units; bias, ReLU and residual move into the reduction.  That is a kernel of its own unless the caller's next one
// does it: 1.2 us, 0.26 for every slice, whose additions wait for one another, and 0.56 for a million bytes of partial sums (fitted with the costs above
// to 250 products in 1 to 64 slices: the count chosen here is 0.1 % slower than the best on average, 5 % at most).  90 x 1056, K = 3072: 11.8
// in one piece, 8.6 in 4; 255 x 1024, K = 2048: 9.0 and 8.9 in 3; 204 x 512, K = 8192: 25.4, 11.3 in 6, 27.9 in 48; 400 x 256, K = 40000 32.7.
// More tiles than compute units gain nothing, and where the other operand comes from beyond the caches they lose: 9 x 8192, K = 2048 12.7 us in
// one piece, 10.4 in 2 (256 tiles), 12.3 in 4.
struct GemmPlan { Tiling tiling; int slices; float cost; };
static GemmPlan plan_slices(const GemmArgs& a) {
  const long tiles = tiles_of(T64x64, a.M, a.N);
  const int nk = (a.K + 63) / 64;
  GemmPlan best{T64x64, 1, launch_cost(T64x64, tiles, nk)};
  if (a.form == 2 || !a.splitk_ws || a.mask || a.drop_p > 0.f || nk < 8) return best;
  const size_t slice = (size_t)a.M * a.N * sizeof(float);
  if (a.deferred_splits) {                               // (the next kernel takes at most so many slices, without ReLU or residual, and all at once)
    if (a.relu || a.residual || tiles > 128) return best;
    long n = std::min(std::min(256 / tiles, (long)nk / 4), (long)DEFERRED_SPLITS_MAX);
    while (n > 1 && n * slice > a.splitk_ws_bytes) --n;
    if (n > 1) best = {T64x64, (int)n, launch_cost(T64x64, n * tiles, (nk + (int)n - 1) / (int)n)};
    return best;
  }
  const float per_slice = 0.26f + 0.56e-6f * (float)slice;
  for (int n = 2; n <= 16 && n <= nk / 4 && n * tiles <= 256 && n * slice <= a.splitk_ws_bytes; ++n) {
    const float c = launch_cost(T64x64, n * tiles, (nk + n - 1) / n) + 1.2f + per_slice * (float)n;
    if (c < best.cost) best = {T64x64, n, c};
  }
  return best;
}

static GemmPlan plan_gemm(const GemmArgs& a) {
  const int nk = (a.K + 63) / 64;
  GemmPlan best = a.form == 2 ? GemmPlan{T128x128, 1, launch_cost(T128x128, tiles_of(T128x128, a.M, a.N), nk)} : plan_slices(a);
  const auto look = [&](Tiling t) {
    const float c = launch_cost(t, tiles_of(t, a.M, a.N), nk);
    if (c < best.cost) best = {t, 1, c};
  };
  if (a.form != 2) for (const Tiling t : {T256x256, T256x128, T192x256, T192x128, T128x128, T64x128}) look(t);
  else {                                                 // (a [k][row] tile of A has 128 or 256 rows)
    look(T256x256);
    if (tiles_of(T128x128_PAIRS, a.M, a.N) <= 512) look(T128x128_PAIRS);
  }
  return best;
}

bool gemm_mfma_slices(const GemmArgs& a) { return plan_gemm(a).slices > 1; }

template <typename T, int BM, int BN, int WM, int WN, int BK, int STAGES, int AHEAD>
static void gemm_mfma_launch(hipStream_t s, const GemmArgs& a, int splits) {
  MfmaGemmParams p;
  p.M = a.M; p.N = a.N; p.K = a.K;
  p.A = (const uint16_t*)a.A; p.lda = a.lda; p.B = (const uint16_t*)a.B; p.ldb = a.ldb; p.C = (uint16_t*)a.C; p.ldc = a.ldc;
  p.bias = (const uint16_t*)a.bias; p.relu = a.relu; p.mask = (const uint16_t*)a.mask; p.residual = (const uint16_t*)a.residual;
  p.colsum = nullptr;
  p.drop_key = a.drop_key; p.drop_thr = a.drop_p > 0.f ? drop_threshold(a.drop_p) : 0u; p.inv_keep = 1.f / (1.f - a.drop_p);
  p.mask_scale = a.mask_scale;
  const int tiles_n = (a.N + BN - 1) / BN;
  p.tiles_m = (a.M + BM - 1) / BM;
  p.tiles_total = tiles_n * p.tiles_m;
  p.per_band.set(GROUP_M * tiles_n, p.tiles_total);
  p.last_band.set(p.tiles_m % GROUP_M, GROUP_M * tiles_n);
  p.a_bytes = (uint32_t)(a.form == 2 ? extent_bytes(a.K, a.M, a.lda) : extent_bytes(a.M, a.K, a.lda));
  p.b_bytes = (uint32_t)(a.form == 0 ? extent_bytes(a.N, a.K, a.ldb) : extent_bytes(a.K, a.N, a.ldb));
  // Split-K: slices of K go to blockIdx.y, fp32 partial tiles go to the caller's workspace and are added in a fixed order.
  const int nk = (a.K + BK - 1) / BK;
  if (a.form == 2 && a.splitk_ws && !a.bias && !a.relu && !a.mask && !a.residual && !p.drop_thr && p.tiles_total <= 128 && nk * BK >= 2048) {
    splits = std::min(256 / p.tiles_total, 8);            // a weight gradient on its own, whose output has too few tiles to fill the chip
    while (splits > 1 && (size_t)splits * a.M * a.N * sizeof(float) > a.splitk_ws_bytes) --splits;
  }
  p.ksteps_per_split = (nk + splits - 1) / splits;
  p.partial = splits > 1 ? (float*)a.splitk_ws : nullptr;
  dim3 grid(p.tiles_total, splits), block(64 * WM * WN);
  constexpr bool TN_ONLY = BK == 32 && BM == 128, NT_ONLY = STAGES == 5;
  if constexpr (TN_ONLY) hipLaunchKernelGGL((gemm_mfma_kernel<T, BM, BN, WM, WN, BK, STAGES, AHEAD, true, true>), grid, block, 0, s, p);
  else if (a.form == 0) hipLaunchKernelGGL((gemm_mfma_kernel<T, BM, BN, WM, WN, BK, STAGES, AHEAD, false, false>), grid, block, 0, s, p);
  else if constexpr (BN == BM && BM >= 128) {
    if (a.form == 1) hipLaunchKernelGGL((gemm_mfma_kernel<T, BM, BN, WM, WN, BK, STAGES, AHEAD, false, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_mfma_kernel<T, BM, BN, WM, WN, BK, STAGES, AHEAD, true, true>), grid, block, 0, s, p);
  } else if constexpr (!NT_ONLY) {
    if (a.form == 1) hipLaunchKernelGGL((gemm_mfma_kernel<T, BM, BN, WM, WN, BK, STAGES, AHEAD, false, true>), grid, block, 0, s, p);
  }
  if (a.deferred_splits) *a.deferred_splits = splits > 1 ? splits : 0;
  if (splits > 1 && !a.deferred_splits) launch_splitk_reduce(s, a.dt, (const float*)a.splitk_ws, splits, a.M, a.N, a.C, a.ldc, a.bias, a.relu, a.residual);
}

// ---- grouped weight gradients ---------------------------------------------------------------------------------------------
bool wgrad_group_supported(int dt, const WgradJob& j) {
  if (dt == F32) return true;
  GemmArgs a{dt, 2, j.M, j.N, j.K, j.A, j.lda, j.B, j.ldb, j.C, j.ldc, nullptr, 0, nullptr, nullptr};
  if (!gemm_mfma_supported(a)) return false;
  return j.colsum == nullptr || ((uintptr_t)j.colsum & 1) == 0;
}

template <typename T, int BM, int BN, int WM, int WN, int BK, int STAGES>
static void wgrad_grouped_launch(hipStream_t s, const WgradJob* jobs, int n) {
  GroupedTable tab;
  int tiles = 0;
  for (int i = 0; i < n; ++i) {
    const WgradJob& j = jobs[i];
    GroupedProblem& g = tab.pr[i];
    g.A = (const uint16_t*)j.A; g.B = (const uint16_t*)j.B; g.C = (uint16_t*)j.C; g.colsum = (uint16_t*)j.colsum;
    g.M = j.M; g.N = j.N; g.K = j.K; g.lda = j.lda; g.ldb = j.ldb; g.ldc = j.ldc;
    const int tiles_n = (j.N + BN - 1) / BN;
    g.tiles_m = (j.M + BM - 1) / BM;
    Divisor per_band, last_band;
    per_band.set(GROUP_M * tiles_n, g.tiles_m * tiles_n);
    last_band.set(g.tiles_m % GROUP_M, GROUP_M * tiles_n);
    g.tiles_n = tiles_n; g.band_m = per_band.m; g.last_m = last_band.m;
    g.tile_begin = tiles;
    tiles += g.tiles_m * tiles_n;
  }
  tab.n = n; tab.tiles_total = tiles;
  hipLaunchKernelGGL((gemm_mfma_grouped_kernel<T, BM, BN, WM, WN, BK, STAGES>), dim3(tiles), dim3(64 * WM * WN), 0, s, tab);
}

// (the cost of the launch with either tiling, see launch_cost; K of the longest product)
void launch_wgrad_grouped(hipStream_t s, int dt, const WgradJob* jobs, int n) {
  if (dt == F32) return launch_wgrad_grouped_f32(s, jobs, n);
  if (n <= 0) return;
  long t256 = 0, t128 = 0;
  int K = 0;
  for (int i = 0; i < n; ++i) {
    t256 += tiles_of(T256x256, jobs[i].M, jobs[i].N);
    t128 += tiles_of(T128x128, jobs[i].M, jobs[i].N);
    K = std::max(K, jobs[i].K);
  }
  const int ks = (K + 63) / 64;
  const bool big = launch_cost(T256x256, t256, ks) <= launch_cost(T128x128, t128, ks);
  if (dt == F16) {
    if (big) wgrad_grouped_launch<half_t, 256, 256, 2, 4, 32, 4>(s, jobs, n);
    else wgrad_grouped_launch<half_t, 128, 128, 2, 2, 64, 4>(s, jobs, n);
  } else {
    if (big) wgrad_grouped_launch<bf16_t, 256, 256, 2, 4, 32, 4>(s, jobs, n);
    else wgrad_grouped_launch<bf16_t, 128, 128, 2, 2, 64, 4>(s, jobs, n);
  }
}

template <typename T>
static void gemm_mfma_dispatch(hipStream_t s, const GemmArgs& a) {
  const GemmPlan q = plan_gemm(a);
  switch (q.tiling) {
    case T256x256: gemm_mfma_launch<T, 256, 256, 2, 4, 32, 4, 1>(s, a, q.slices); break;
    case T256x128: gemm_mfma_launch<T, 256, 128, 4, 2, 64, 3, 1>(s, a, q.slices); break;
    case T192x256: gemm_mfma_launch<T, 192, 256, 2, 4, 32, 4, 1>(s, a, q.slices); break;
    case T192x128: gemm_mfma_launch<T, 192, 128, 2, 2, 64, 3, 1>(s, a, q.slices); break;
    case T64x128: gemm_mfma_launch<T, 64, 128, 2, 2, 64, 4, 1>(s, a, q.slices); break;
    case T64x64:
      if (a.form == 0 && tiles_of(T64x64, a.M, a.N) * q.slices <= 256) gemm_mfma_launch<T, 64, 64, 2, 2, 64, 5, 2>(s, a, q.slices);
      else gemm_mfma_launch<T, 64, 64, 2, 2, 64, 4, 2>(s, a, q.slices);
      break;
    case T128x128_PAIRS: gemm_mfma_launch<T, 128, 128, 2, 2, 32, 3, 1>(s, a, q.slices); break;
    default: gemm_mfma_launch<T, 128, 128, 2, 2, 64, 4, 1>(s, a, q.slices); break;
  }
}

void launch_gemm_mfma(hipStream_t s, const GemmArgs& a) {
  if (a.dt == F16) gemm_mfma_dispatch<half_t>(s, a);
  else gemm_mfma_dispatch<bf16_t>(s, a);
}

}  // namespace tfm
