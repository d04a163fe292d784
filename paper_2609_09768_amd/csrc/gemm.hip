// Projections of the decoder layer on the selected tokens (gfx950).
//
// Paper: under selective recompute only the selected tokens pass through a
// layer (Section 3.4; Section 4 setup), so every projection of the layer
// (fused Q/K/V, O, gate/up, down) multiplies the selected rows' activations
// by a weight matrix:
//   c[i, j] = sum_e a[r_i, e] * w[j, e]  (+ residual[i, j]),
// with r_i = a_rows[i] (a gather of the selected rows) or i, and w in the
// [out, in] layout of the model's linear layers.  The residual addition of
// the O and down projections is fused into the store.
//
// A dense contraction, so it runs on the matrix cores:
// v_mfma_f32_16x16x32_bf16, float32 accumulation, rounded once to bf16 after
// the residual is added in float32.  (The 16x16 shape moves half the
// accumulator bytes per FLOP of the 32x32 one; on this power-limited chip
// it ran 8-13 % faster on the layer's shapes, with identical results.)
//
// One workgroup of 8 waves (two per SIMD) computes one tile of c over the
// whole K.  The tile is 256 x 256, 256 x 192, 128 x 128 or 64 x 64, and a
// launch mixes a large and a small one (gemm_plan.h): the tiles of a
// selection rarely fill 256 CUs a whole number of times, and a last round of
// a few large tiles would cost as much as a full one.  Common to all tiles:
// - Activation and weight rows go from memory straight into LDS in 128-byte
//   pieces of K (global loads with an LDS destination: per-lane 64-bit
//   addresses, so the row gather costs nothing; no registers, no VALU).
// - LDS rows are 128 bytes (64 bf16 of K); the 16-byte piece p of row r is
//   stored at p ^ ((r >> 1) & 7), so the operand reads (16 lanes: 16
//   consecutive rows, one piece) fall in 16 distinct bank groups.
// - The MFMA computes each 16 x 16 block transposed (weight rows as the
//   first operand), so a lane ends with one output row and four consecutive
//   columns per block: 8-byte stores (16 for the large tiles, see store_wave)
//   and residual loads, issued together before the first store.
// - LDS is eight arrays of 16 KB, four for each operand, so that the
//   compiler's wait-count pass can tell loads in flight into one from the
//   reads of another; every wait for a load is explicit.
// - Workgroup ids are dispatched round-robin over the 8 XCDs; they are
//   renumbered so that each XCD gets a contiguous range of tiles, walked in
//   groups of 8 row tiles, so workgroups that share activation or weight
//   rows tend to share an L2 (5,056 x 28,672 x 4,096 836 us, 864 with groups of
//   4).  Where K is short, an XCD's tiles that are stored together matter more
//   than those rows, and groups of 4 make them twice as wide: 17,339 x 29,064 x
//   320 472 us instead of 560, x 1,024 902 and 987, 14,227 x 17,720 x 128 158
//   and 171, 18,856 x 28,672 x 1,024 969 and 968; up to 6 % slower for a few
//   (40,000 x 8,192 x 320 313 and 294), and groups of 16 are worse.
#include "kvc_internal.h"
#include "gemm_plan.h"

#include <type_traits>

namespace kvc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

constexpr int kBK = kGemmSlice;     // K elements of an LDS row (128 bytes)
constexpr int kXcds = 8;

// s_waitcnt immediate (gfx9 encoding: vmcnt bits 3:0 and 15:14, expcnt 6:4,
// lgkmcnt 11:8): at most vm vector-memory operations in flight, and lgkm
// (15: not waited for) LDS operations.
constexpr int wait_imm(int vm, int lgkm) { return (vm & 15) | (7 << 4) | (lgkm << 8) | ((vm >> 4) << 14); }

template <int I>
using Int = std::integral_constant<int, I>;

constexpr int kThreads = kGemmThreads;
constexpr int kWaves = 8;
constexpr int kArray = 128 * kBK;   // bf16 of one LDS array: 128 rows (16 KB)

struct GemmParams {
  const uint16_t* a;
  const int32_t* a_rows;
  long long n_a_rows;
  const uint16_t* w;
  const uint16_t* res;
  uint16_t* c;
  long long m, n, k;
  // the first big_wgs workgroups take large tiles (big_rows rows of tiles),
  // the others small ones, from row small_row0 on
  int big_wgs, big_tiles_m, big_tiles_n;
  int small_tiles_m, small_tiles_n;
  long long small_row0;
  int group_m;  // row tiles per group of the tile walk
};

// The eight LDS arrays of a workgroup.
struct Lds {
  uint16_t *a0, *a1, *a2, *a3, *w0, *w1, *w2, *w3;
};

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& u) { return __builtin_bit_cast(bf16x8, u); }

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Barrier that orders LDS accesses without waiting for loads in flight (the
// waits are explicit): nothing moves across it in the compiler.
__device__ __forceinline__ void barrier_only() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// Workgroup id -> (row tile, column tile).  Ids go round-robin over the
// XCDs; v renumbers them so each XCD holds a contiguous range of v (a
// bijection on [0, T)), and v walks groups of group_m row tiles column by
// column.
__device__ __forceinline__ void tile_of(int bid, int tiles_m, int tiles_n, int group_m, int& tm, int& tn) {
  const int total = tiles_m * tiles_n;
  const int per = total / kXcds, rem = total % kXcds;
  const int x = bid % kXcds, slot = bid / kXcds;
  const int v = x * per + min(x, rem) + slot;
  const int group = v / (group_m * tiles_n);
  const int first = group * group_m;
  const int gm = min(group_m, tiles_m - first);
  const int in_group = v - group * group_m * tiles_n;
  tm = first + in_group % gm;
  tn = in_group / gm;
}

// This lane's source of the 16-byte piece it loads for row `row` of a tile's
// activation rows (m0 + row) or weight rows (n0 + row): rows past m or n read
// the last valid row (their results are not stored), an invalid gather entry
// reads row 0 (its result is zeroed at the store).
__device__ __forceinline__ const uint16_t* a_source(const GemmParams& P, long long am) {
  if (am >= P.m) am = P.m - 1;
  long long ar = P.a_rows ? (long long)P.a_rows[am] : am;
  if (ar < 0 || ar >= P.n_a_rows) ar = 0;
  return P.a + ar * P.k;
}
__device__ __forceinline__ const uint16_t* w_source(const GemmParams& P, long long wr) {
  if (wr >= P.n) wr = P.n - 1;
  return P.w + wr * P.k;
}

__device__ __forceinline__ void load_lds16(const uint16_t* src, uint16_t* dst) {
  __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)dst, 16, 0, 0);
}

// LDS address of an array as a number the compiler does not see through.
__device__ __forceinline__ uint32_t lds_address(uint16_t* p) {
  uint32_t a = (uint32_t)reinterpret_cast<uintptr_t>((lds_void*)p);
  asm volatile("" : "+s"(a));
  return a;
}

// b0 .. b7 by index, as values (a choice between variables of a closure would
// go through memory).
__device__ __forceinline__ uint32_t pick8(int w, uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3, uint32_t b4,
                                          uint32_t b5, uint32_t b6, uint32_t b7) {
  uint32_t r = b0;
  r = w == 1 ? b1 : r;
  r = w == 2 ? b2 : r;
  r = w == 3 ? b3 : r;
  r = w == 4 ? b4 : r;
  r = w == 5 ? b5 : r;
  r = w == 6 ? b6 : r;
  r = w == 7 ? b7 : r;
  return r;
}

// Output row m is a gather of an invalid entry: its product is zero.
__device__ __forceinline__ bool zero_row(const GemmParams& P, long long m) {
  if (!P.a_rows) return false;
  const long long ar = P.a_rows[min(m, P.m - 1)];
  return ar < 0 || ar >= P.n_a_rows;
}

// Residual at four consecutive columns of row m from column n, zero without
// one.  Past the edges it reads inside the matrix (n is a multiple of 8) and
// the value is not used, so the loads of a tile need no branches and are in
// flight together.
__device__ __forceinline__ uint2 residual4(const GemmParams& P, long long m, long long n) {
  if (!P.res) return make_uint2(0, 0);
  return *reinterpret_cast<const uint2*>(P.res + min(m, P.m - 1) * P.n + min(n, P.n - 4));
}

__device__ __forceinline__ f32x4 residual_f32(const uint2& r2) {
  return f32x4{__uint_as_float(r2.x << 16), __uint_as_float(r2.x & 0xFFFF0000u), __uint_as_float(r2.y << 16),
               __uint_as_float(r2.y & 0xFFFF0000u)};
}

// Four consecutive outputs of row m from column n.
__device__ __forceinline__ void store4(const GemmParams& P, long long m, long long n, bool zero, const f32x4& acc,
                                       const uint2& r2) {
  if (m >= P.m || n >= P.n) return;
  f32x4 v = zero ? f32x4{0.f, 0.f, 0.f, 0.f} : acc;
  if (P.res) v += residual_f32(r2);
  *reinterpret_cast<uint2*>(P.c + m * P.n + n) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}

// Two adjacent 16-column blocks of 16 output rows, four columns of each in a
// lane, to 16 bytes of one block in a lane and back: lanes of even q = lane / 16
// get columns 4 q .. 4 q + 7 of the first block, those of odd q columns
// 4 (q - 1) .. of the second.
__device__ __forceinline__ void swap_blocks(uint2& a, uint2& b) {
  const auto x = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
  const auto y = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
  a = make_uint2(x[0], y[0]);
  b = make_uint2(x[1], y[1]);
}

// The outputs of a wave of tile_256: 16 rows each at m and m + 128, + 16, + 32
// and + 48, 16 NT columns from n on.  ZERO: some row is a gather of an invalid
// entry.  Two blocks are stored together, 64 bytes of a row in one instruction,
// and an address is a scalar per 16 rows, the lane's offset from it and a
// constant.  The L2 takes about one piece of a line per store instruction and
// row, and every CU stores its tile at once, so stores of 32 bytes of a row (8
// a lane, 37 instructions each) cost more than the K loop where K is short:
// 8,192 x 8,192 x 64 46.2 -> 36.7 us, x 512 94 -> 83, 30,000 x 4,096 x 64 86 ->
// 61, 18,856 x 28,672 x 4,096 3,280 -> 3,185.  (Non-temporal stores, which the
// L2 does not gather into lines, took four times as long.)
template <int NT, bool RES, bool ZERO>
__device__ __forceinline__ void store_wave(const GemmParams& P, long long m, long long n, int lane,
                                           const f32x4 (&acc)[NT][2][4]) {
  const int rl = lane & 15, q = lane >> 4;
  // first column of this lane's piece of a pair of blocks (n is a multiple of
  // 8, so it lies in c as a whole or not at all), and of a single block
  const int pair_col = 16 * (q & 1) + 4 * (q & 2), one_col = 4 * q;
  // bytes, below 2^30
  const uint32_t pair_off = (uint32_t)(rl * (int)P.n + pair_col) * 2, one_off = (uint32_t)(rl * (int)P.n + one_col) * 2;
  bool in[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) in[nt] = n + 16 * nt + (nt + 1 < NT || !(NT & 1) ? pair_col : one_col) < P.n;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const long long mh = m + 128 * h;
    uint2 r[4][NT];
    if (RES) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const bool row = mh + 16 * mt + rl < P.m;
        const char* src = reinterpret_cast<const char*>(P.res + (mh + 16 * mt) * P.n + n);
#pragma unroll
        for (int nt = 0; nt + 1 < NT; nt += 2) {
          uint4 u = make_uint4(0, 0, 0, 0);
          if (row && in[nt]) u = *reinterpret_cast<const uint4*>(src + pair_off + 32 * nt);
          r[mt][nt] = make_uint2(u.x, u.y);
          r[mt][nt + 1] = make_uint2(u.z, u.w);
        }
        if (NT & 1) {
          r[mt][NT - 1] = make_uint2(0, 0);
          if (row && in[NT - 1]) r[mt][NT - 1] = *reinterpret_cast<const uint2*>(src + one_off + 32 * (NT - 1));
        }
      }
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bool row = mh + 16 * mt + rl < P.m;
      const bool zero = ZERO && zero_row(P, mh + 16 * mt + rl);
      char* dst = reinterpret_cast<char*>(P.c + (mh + 16 * mt) * P.n + n);
      uint2 o[NT];
      if (RES) {
#pragma unroll
        for (int nt = 0; nt + 1 < NT; nt += 2) swap_blocks(r[mt][nt], r[mt][nt + 1]);
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        f32x4 v = zero ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[nt][h][mt];
        if (RES) v += residual_f32(r[mt][nt]);
        o[nt] = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
      }
#pragma unroll
      for (int nt = 0; nt + 1 < NT; nt += 2) {
        swap_blocks(o[nt], o[nt + 1]);
        if (row && in[nt])
          *reinterpret_cast<uint4*>(dst + pair_off + 32 * nt) = make_uint4(o[nt].x, o[nt].y, o[nt + 1].x, o[nt + 1].y);
      }
      if ((NT & 1) && row && in[NT - 1]) *reinterpret_cast<uint2*>(dst + one_off + 32 * (NT - 1)) = o[NT - 1];
    }
  }
}

// A tile of 256 rows and 64 NT columns (NT = 4 or 3) in K slices of 64, two of
// them in LDS.  Each wave owns 64 rows of each half of the tile's rows and NT
// adjacent blocks of 16 columns.  A slice is two phases (figures for NT = 4):
// the tile's upper rows (16 fragments read, 32 MFMAs), then the lower ones (8
// read, 32 MFMAs).  The two waves of a SIMD run half a phase apart (waves 4..7
// pass one barrier more at the start): while one reads its fragments and
// issues the loads, the other keeps the matrix cores busy.  A half tile
// is refilled as soon as both have read it, one phase later, so a load has
// a whole slice (about 0.9 us) to arrive.  Alone on the chip a tile takes
// 0.93 us per slice (2 x 1031 MFMA cycles are 0.86 us at 2.4 GHz); with all
// CUs busy 1.40 us, held by the power limit (1.8 GHz) and the shared caches.
// Against all waves in step with one barrier per slice: 5,056 x 28,672 x
// 4,096 990 -> 850 us (1.40 PFLOP/s), 4,096 x 4,096 x 16,384 415 -> 357 (1.54).
// NT = 3 takes 1.10 us per slice, 5 % more per column, and is chosen where its
// tiles fill the CUs better: 696 x 28,672 x 4,096 (450 tiles in two rounds for
// 336 in one and a third) 146 us, 203 with 256 x 256 tiles alone, 217 x 37,888
// x 3,584 69 and 95.
// Measured and not taken: four phases per slice of 16 MFMAs (3 % slower),
// raised wave priority in the MFMA phases (no gain), a third slot for the
// weights (3 % slower), a K start that differs from workgroup to workgroup
// (no gain).
template <int NT>
__device__ __forceinline__ void tile_256(const GemmParams& P, const Lds& S, int tm, int tn) {
  uint16_t* const As[2][2] = {{S.a0, S.a1}, {S.a2, S.a3}};  // [slice % 2][half tile]
  uint16_t* const Ws[2][2] = {{S.w0, S.w1}, {S.w2, S.w3}};  // [slice % 2][rows 0..127, 128..]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long m0 = (long long)tm * 256, n0 = (long long)tn * (64 * NT);
  const int wn = wave & 3;
  // The LDS rows of this wave's block nt begin at 128 (nt / 2) + strip(nt), and
  // LDS row `row` holds weight row column(row) of the tile: each wave's blocks
  // lie in both of the operand's arrays, and are adjacent columns of c.
  auto strip = [&](int nt) __attribute__((always_inline)) { return nt < 2 || NT == 4 ? 32 * wn + 16 * (nt & 1) : 16 * wn; };
  auto column = [&](int row) __attribute__((always_inline)) {
    return row < 128 ? 16 * NT * (row >> 5) + (row & 31)
                     : NT == 4 ? 64 * ((row - 128) >> 5) + 32 + (row & 31) : 48 * ((row - 128) >> 4) + 32 + (row & 15);
  };
  const int wm = wave >> 2;  // rows 64 wm .. +63 of each half

  const uint16_t* a_src[2][2];
  const uint16_t* w_src[NT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = 16 * wave + 8 * j + (lane >> 3);
      a_src[h][j] = a_source(P, m0 + 128 * h + row) + 8 * ((lane & 7) ^ ((row >> 1) & 7));
    }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int row = 64 * j + 8 * wave + (lane >> 3);
    w_src[j] = w_source(P, n0 + column(row)) + 8 * ((lane & 7) ^ ((row >> 1) & 7));
  }
  auto load_half = [&](const uint16_t* const (&src)[2], int t, uint16_t* dst) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2; ++j) load_lds16(src[j] + (long long)t * kBK, dst + (16 * wave + 8 * j) * kBK);
  };
  auto load_w = [&](int t, auto bufc) __attribute__((always_inline)) {
    constexpr int B = decltype(bufc)::value;
#pragma unroll
    for (int j = 0; j < NT; ++j)
      load_lds16(w_src[j] + (long long)t * kBK, Ws[B][j >> 1] + (64 * (j & 1) + 8 * wave) * kBK);
  };

  const int rl = lane & 15, q = lane >> 4, sw = (rl >> 1) & 7;
  int rd[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) rd[ks] = rl * kBK + 8 * ((4 * ks + q) ^ sw);
  f32x4 acc[NT][2][4];  // [nt][A half][mt]
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[nt][h][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[2][4], fw[2][NT];  // [ks][mt], [ks][nt]
  auto read_a = [&](const uint16_t* base) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
        fa[ks][mt] = as_bf16x8(*reinterpret_cast<const uint4*>(base + (64 * wm + 16 * mt) * kBK + rd[ks]));
  };
  auto read_w = [&](auto bufc, int nt) __attribute__((always_inline)) {
    constexpr int B = decltype(bufc)::value;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      fw[ks][nt] = as_bf16x8(*reinterpret_cast<const uint4*>(Ws[B][nt >> 1] + strip(nt) * kBK + rd[ks]));
  };
  auto multiply = [&](int h) __attribute__((always_inline)) {
    barrier_only();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          acc[nt][h][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[ks][nt], fa[ks][mt], acc[nt][h][mt], 0, 0, 0);
    barrier_only();
  };

  const int nk = (int)(P.k / kBK);
  // Slice t, in buffer B, of which MORE (up to 2) slices follow.  (The last
  // slices are separate code: with the loads behind branches in the loop, the
  // compiler's wait-count pass waits for all of them in every second slice.)
  auto slice = [&](int t, auto bufc, auto morec) __attribute__((always_inline)) {
    constexpr int B = decltype(bufc)::value;
    constexpr int MORE = decltype(morec)::value;
    // upper rows.  The waits leave the loads issued after the half tiles of
    // the next phase in flight, and finish this wave's reads before the
    // barrier, after which others may refill what it read.
    read_w(bufc, 0);
    read_w(bufc, 1);
    read_a(As[B][0]);
#pragma unroll
    for (int nt = 2; nt < NT; ++nt) read_w(bufc, nt);
    if constexpr (MORE >= 1) load_half(a_src[1], t + 1, As[1 - B][1]);
    __builtin_amdgcn_s_waitcnt(wait_imm(MORE >= 1 ? 4 + NT : 0, 0));
    multiply(0);
    // lower rows
    read_a(As[B][1]);
    if constexpr (MORE >= 2) {
      load_half(a_src[0], t + 2, As[B][0]);
      load_w(t + 2, bufc);
    }
    __builtin_amdgcn_s_waitcnt(wait_imm(MORE >= 2 ? 4 + NT : MORE == 1 ? 2 : 0, 0));
    multiply(1);
  };

  // Slice 0 goes to buffer nk % 2, so that the last two are in buffers 0, 1.
  auto start = [&](auto bufc) __attribute__((always_inline)) {
    constexpr int B = decltype(bufc)::value;
    const int second = min(1, nk - 1);  // a single slice is loaded twice
    load_half(a_src[0], 0, As[B][0]);
    load_w(0, bufc);
    load_half(a_src[1], 0, As[B][1]);
    load_half(a_src[0], second, As[1 - B][0]);
    load_w(second, Int<1 - B>{});
    __builtin_amdgcn_s_waitcnt(wait_imm(4 + NT, 15));
    barrier_only();
    if (wm == 1) barrier_only();
  };
  if (nk == 1) {
    start(Int<1>{});
    slice(0, Int<1>{}, Int<0>{});
  } else {
    int t = 0;
    if (nk & 1) {
      start(Int<1>{});
      slice(t++, Int<1>{}, Int<2>{});
    } else {
      start(Int<0>{});
    }
    for (; t + 2 < nk; t += 2) {
      slice(t, Int<0>{}, Int<2>{});
      slice(t + 1, Int<1>{}, Int<2>{});
    }
    slice(t, Int<0>{}, Int<1>{});
    slice(t + 1, Int<1>{}, Int<0>{});
  }
  if (wm == 0) barrier_only();

  bool zero = false;
  if (P.a_rows) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) zero |= zero_row(P, m0 + 128 * h + 64 * wm + 16 * mt + rl);
  }
  const long long mw = m0 + 64 * wm, nw = n0 + 16 * NT * wn;
  if (__any(zero)) {
    if (P.res) store_wave<NT, true, true>(P, mw, nw, lane, acc);
    else store_wave<NT, false, true>(P, mw, nw, lane, acc);
  } else {
    if (P.res) store_wave<NT, true, false>(P, mw, nw, lane, acc);
    else store_wave<NT, false, false>(P, mw, nw, lane, acc);
  }
}

// A BT x BT tile, BT = 128 or 64, with the K of each slice shared by
// WK = 2 or 4 groups of waves (WM x WN waves each, 64 x 64 or 32 x 64 of the
// tile per wave): the small tiles still get eight waves, and 32 KB slices
// four deep (K slices of 64 or 128) keep up to 96 KB of loads in flight per
// CU.  One barrier per slice; each wave reads the fragments of the next slice
// between the MFMAs of this one.  At the end the groups' float32 sums are
// added through LDS in a fixed order.  With all CUs busy 64 of K take
// 0.48 us (128) or 0.23 us (64): a 128 tile runs at 73 % and a 64 tile at
// 38 % of the rate of a 256 tile, bound by the loads (64 and 128 bytes per
// CU and MFMA cycle).  Against 256 x 256 tiles only: 217 x 3,584 x 18,944
// 362 -> 56 us, 696 x 4,096 x 4,096 94 -> 30 us, 696 x 4,096 x 14,336 281 ->
// 88 us, and with both sizes in one launch 5,056 x 4,096 x 14,336 675 ->
// 441 us.  (128 x 256 tiles, 128 x 64 tiles and four waves with two
// workgroups per CU were slower on most shapes.)
template <int BT, int WM, int WN, int WK>
__device__ __forceinline__ void tile_ring(const GemmParams& P, const Lds& L, long long m0, int tn) {
  constexpr int BM = BT, BN = BT;
  constexpr int NS = 4;                       // slices in LDS
  constexpr int SUB = WK / 2;                 // 64-wide pieces of K per slice
  constexpr int UPW = 4;                      // load instructions per wave and slice, two for each operand
  constexpr int MT = BM / WM / 16, NT = BN / WN / 16;
  static_assert(WM * WN * WK == kWaves && SUB * BT == 128, "eight waves, 16 KB of each operand per slice");
  uint16_t* const SA[NS] = {L.a0, L.a1, L.a2, L.a3};
  uint16_t* const SW[NS] = {L.w0, L.w1, L.w2, L.w3};

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long n0 = (long long)tn * BN;
  const int kg = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;

  const int nk = (int)(P.k / kBK);
  const int ns = (nk + SUB - 1) / SUB;  // slices
  // wave w fills rows 16 w .. 16 w + 15 of both arrays of a slot (row r holds
  // row r % BT of the tile, piece r / BT of the slice's K)
  const uint16_t* a_src[2];
  const uint16_t* w_src[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = (16 * wave + 8 * j) % BT + (lane >> 3);
    const int piece = (lane & 7) ^ ((row >> 1) & 7);
    a_src[j] = a_source(P, m0 + row) + 8 * piece;
    w_src[j] = w_source(P, n0 + row) + 8 * piece;
  }
  // load j of slice t: rows 8 (j % 2) .. of this wave's 16, of A (j < 2) or W
  auto load_unit = [&](int t, int slot, auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    // a piece of the last slice past K is loaded from inside it and not used
    const int kb = SUB == 1 ? t : min(t * SUB + 16 * wave / BT, nk - 1);
    load_lds16((j < 2 ? a_src[j & 1] : w_src[j & 1]) + (long long)kb * kBK,
               (j < 2 ? SA[slot] : SW[slot]) + (16 * wave + 8 * (j & 1)) * kBK);
  };
  auto load_slot = [&](int t, auto slotc) __attribute__((always_inline)) {
    constexpr int slot = decltype(slotc)::value;
    load_unit(t, slot, Int<0>{});
    load_unit(t, slot, Int<1>{});
    load_unit(t, slot, Int<2>{});
    load_unit(t, slot, Int<3>{});
  };
  const int rl = lane & 15, q = lane >> 4, sw = (rl >> 1) & 7;
  // this wave's 32-wide K step of a slice is step kg
  const int rd = (kg >> 1) * BT * kBK + rl * kBK + 8 * ((4 * (kg & 1) + q) ^ sw);
  const int rda = rd + wm * (BM / WM) * kBK, rdw = rd + wn * (BN / WN) * kBK;
  f32x4 acc[NT][MT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 f[2][NT + MT];
  auto read_frag = [&](int slot, int set, int i) __attribute__((always_inline)) {
    const uint16_t* p = i < NT ? SW[slot] + rdw + i * 16 * kBK : SA[slot] + rda + (i - NT) * 16 * kBK;
    f[set][i] = as_bf16x8(*reinterpret_cast<const uint4*>(p));
  };
  auto multiply = [&](int set, auto&& between) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NT * MT; ++i) {
      const int nt = i / MT, mt = i % MT;
      acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[set][nt], f[set][NT + mt], acc[nt][mt], 0, 0, 0);
      between(i);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr int NM = NT * MT, NF = NT + MT;
  // Slice t, in slot B, whose fragments are in set B % 2.  MAIN: the slot is
  // refilled with slice t + NS; otherwise no slices follow those in the ring.
  auto slice = [&](int t, auto slotc, auto mainc) __attribute__((always_inline)) {
    constexpr int B = decltype(slotc)::value;
    constexpr bool MAIN = decltype(mainc)::value;
    constexpr int NX = (B + 1) % NS, set = B & 1;
    constexpr bool HAS_NEXT = MAIN || B + 1 < NS;
    if (HAS_NEXT) {
      // slice t + 1 has arrived (every wave's part, after the barrier) and
      // every wave holds its fragments of slice t
      constexpr int behind = MAIN ? NS - 2 : (NS - 2 - B > 0 ? NS - 2 - B : 0);
      __builtin_amdgcn_s_waitcnt(wait_imm(UPW * behind, 0));
      barrier_only();
    }
    if (SUB > 1 && !MAIN && B == NS - 1 && t * SUB + (kg >> 1) >= nk) {
      // the piece lies past K: both operands are zeroed, since what was loaded
      // in its place may hold an infinity
#pragma unroll
      for (int i = 0; i < NF; ++i) f[set][i] = as_bf16x8(make_uint4(0, 0, 0, 0));
    }
    multiply(set, [&](int i) __attribute__((always_inline)) {
      constexpr int RPM = (NF + NM - 1) / NM;  // reads after an MFMA
      if (HAS_NEXT) {
#pragma unroll
        for (int r = i * RPM; r < (i + 1) * RPM && r < NF; ++r) read_frag(NX, set ^ 1, r);
      }
      if (MAIN) {
        constexpr int every = NM / UPW < 2 ? 1 : 2;  // a load after every (second) MFMA
        if (i == every - 1) load_unit(t + NS, B, Int<0>{});
        if (i == 2 * every - 1) load_unit(t + NS, B, Int<1>{});
        if (i == 3 * every - 1) load_unit(t + NS, B, Int<2>{});
        if (i == 4 * every - 1) load_unit(t + NS, B, Int<3>{});
      }
    });
  };
  // The ring ends with its last slot, so the number of slices fixes the slot
  // it starts with.
  const int s0 = (NS - ns % NS) % NS;
  auto start = [&](auto s0c) __attribute__((always_inline)) {
    constexpr int Z = decltype(s0c)::value;
    if constexpr (Z <= 0) load_slot(0 - Z, Int<0>{});
    if constexpr (Z <= 1) load_slot(1 - Z, Int<1>{});
    if constexpr (Z <= 2) load_slot(2 - Z, Int<2>{});
    load_slot(3 - Z, Int<3>{});
    // (the first reads stand in both branches: the wait-count pass merges
    // them into a wait for every load otherwise)
    auto first = [&]() __attribute__((always_inline)) {
      barrier_only();
#pragma unroll
      for (int r = 0; r < NF; ++r) read_frag(Z, Z & 1, r);
    };
    if (ns >= NS) {
      if constexpr (Z > 0) load_slot(NS - Z, Int<0>{});
      if constexpr (Z > 1) load_slot(NS - Z + 1, Int<1>{});
      if constexpr (Z > 2) load_slot(NS - Z + 2, Int<2>{});
      __builtin_amdgcn_s_waitcnt(wait_imm(UPW * (NS - 1), 15));
      first();
    } else {
      __builtin_amdgcn_s_waitcnt(wait_imm(UPW * (NS - 1 - Z), 15));
      first();
    }
  };
  if (s0 == 0) start(Int<0>{});
  else if (s0 == 1) start(Int<1>{});
  else if (s0 == 2) start(Int<2>{});
  else start(Int<3>{});
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;
  int t = 0;
  if (ns >= NS && s0 != 0) {
    if (s0 <= 1) slice(t++, Int<1>{}, Yes{});
    if (s0 <= 2) slice(t++, Int<2>{}, Yes{});
    slice(t++, Int<3>{}, Yes{});
  }
  for (; t + NS < ns; t += NS) {
    slice(t, Int<0>{}, Yes{});
    slice(t + 1, Int<1>{}, Yes{});
    slice(t + 2, Int<2>{}, Yes{});
    slice(t + 3, Int<3>{}, Yes{});
  }
  const bool all = ns >= NS;
  if (all || s0 == 0) slice(t++, Int<0>{}, No{});
  if (all || s0 <= 1) slice(t++, Int<1>{}, No{});
  if (all || s0 <= 2) slice(t++, Int<2>{}, No{});
  slice(t++, Int<3>{}, No{});

  // Sum the WK groups' shares in LDS (the ring is no longer read): wave kg of
  // a tile part finishes its column blocks kg NT / WK .., taking the shares
  // in the order of the groups.
  constexpr int NTO = NT / WK;               // column blocks a wave stores
  constexpr int kShare = NTO * MT * 64 * 4;  // floats one wave hands another
  static_assert(NTO * WK == NT, "column blocks divide over the K groups");
  static_assert((WK - 1) * kShare * 4 <= kArray * 2, "a wave's shares fit one array");
  // wave w's shares lie in its own array; the LDS addresses are opaque
  // numbers, since the compiler cannot make a table of them
  const uint32_t b0 = lds_address(L.a0), b1 = lds_address(L.a1), b2 = lds_address(L.a2), b3 = lds_address(L.a3);
  const uint32_t b4 = lds_address(L.w0), b5 = lds_address(L.w1), b6 = lds_address(L.w2), b7 = lds_address(L.w3);
  auto base_of = [=](int w) __attribute__((always_inline)) { return pick8(w, b0, b1, b2, b3, b4, b5, b6, b7); };
  auto share = [=](uint32_t base, int d, int i) __attribute__((always_inline)) {
    return reinterpret_cast<lds_f32x4*>(base + (uint32_t)(((d - 1) * kShare + i * 256) * 4 + lane * 16));
  };
  __builtin_amdgcn_s_waitcnt(wait_imm(0, 0));
  barrier_only();
#pragma unroll
  for (int o = 0; o < WK; ++o) {
    if (o == kg) continue;
    const uint32_t to = base_of(wave - kg + o);
#pragma unroll
    for (int i = 0; i < NTO; ++i)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) *share(to, kg ^ o, i * MT + mt) = acc[o * NTO + i][mt];
  }
  __builtin_amdgcn_s_waitcnt(wait_imm(0, 0));
  barrier_only();
  const uint32_t mine = base_of(wave);
#pragma unroll
  for (int o = 0; o < WK; ++o) {
    if (o != kg) continue;
    const long long m = m0 + wm * (BM / WM) + rl;
    const long long n = n0 + wn * (BN / WN) + 16 * o * NTO + 4 * q;
    uint2 r[MT][NTO];
    bool zero[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      zero[mt] = zero_row(P, m + 16 * mt);
#pragma unroll
      for (int i = 0; i < NTO; ++i) r[mt][i] = residual4(P, m + 16 * mt, n + 16 * i);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < NTO; ++i) {
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < WK; ++g)
          v += g == o ? acc[o * NTO + i][mt] : *share(mine, g ^ o, i * MT + mt);
        store4(P, m + 16 * mt, n + 16 * i, zero[mt], v, r[mt][i]);
      }
  }
}

// One tile of the launch: a large one for the first big_wgs workgroups, a
// small one for the others.  MODE 0: 256 x 256 and 128 x 128, 1: 256 x 192
// and 128 x 128, 2: 128 x 128 and 64 x 64.
template <int MODE>
__global__ __launch_bounds__(kThreads) void gemm_kernel(const GemmParams P) {
  __shared__ __attribute__((aligned(16))) uint16_t A0[kArray], A1[kArray], A2[kArray], A3[kArray];
  __shared__ __attribute__((aligned(16))) uint16_t W0[kArray], W1[kArray], W2[kArray], W3[kArray];
  const Lds S = {A0, A1, A2, A3, W0, W1, W2, W3};
  int tm, tn;
  if ((int)blockIdx.x < P.big_wgs) {
    tile_of((int)blockIdx.x, P.big_tiles_m, P.big_tiles_n, P.group_m, tm, tn);
    if constexpr (MODE == 0) tile_256<4>(P, S, tm, tn);
    else if constexpr (MODE == 1) tile_256<3>(P, S, tm, tn);
    else tile_ring<128, 2, 2, 2>(P, S, (long long)tm * 128, tn);
  } else {
    tile_of((int)blockIdx.x - P.big_wgs, P.small_tiles_m, P.small_tiles_n, P.group_m, tm, tn);
    if constexpr (MODE < 2) tile_ring<128, 2, 2, 2>(P, S, P.small_row0 + (long long)tm * 128, tn);
    else tile_ring<64, 2, 1, 4>(P, S, P.small_row0 + (long long)tm * 64, tn);
  }
}

}  // namespace

int64_t gemm_work_items(int64_t m, int64_t n) {
  if (m <= 0 || n <= 0) return 0;
  return gemm_div_up<int64_t>(m, 256) * gemm_div_up<int64_t>(n, 256) * kThreads;
}

hipError_t launch_gemm(int64_t m, int64_t n, int64_t k, const uint16_t* a, int64_t n_a_rows,
                       const int32_t* a_rows, const uint16_t* w, const uint16_t* res, uint16_t* c,
                       hipStream_t s) {
  if (m <= 0 || n <= 0) return hipSuccess;
  GemmParams P;
  P.a = a;
  P.a_rows = a_rows;
  P.n_a_rows = n_a_rows;
  P.w = w;
  P.res = res;
  P.c = c;
  P.m = m;
  P.n = n;
  P.k = k;
  const GemmPlan plan = gemm_plan(m, n, k);
  const GemmTile& B = kGemmBig[plan.mode];
  const GemmTile& S = kGemmSmall[plan.mode];
  P.big_tiles_m = (int)plan.big_rows;
  P.big_tiles_n = (int)gemm_div_up<int64_t>(n, B.cols);
  P.big_wgs = P.big_tiles_m * P.big_tiles_n;
  P.small_row0 = plan.big_rows * B.rows;
  P.small_tiles_m = P.small_row0 < m ? (int)gemm_div_up<int64_t>(m - P.small_row0, S.rows) : 0;
  P.small_tiles_n = (int)gemm_div_up<int64_t>(n, S.cols);
  P.group_m = k < 2048 ? 4 : 8;
  const unsigned wgs = (unsigned)P.big_wgs + (unsigned)P.small_tiles_m * (unsigned)P.small_tiles_n;
  if (plan.mode == 0) hipLaunchKernelGGL(gemm_kernel<0>, dim3(wgs), dim3(kThreads), 0, s, P);
  else if (plan.mode == 1) hipLaunchKernelGGL(gemm_kernel<1>, dim3(wgs), dim3(kThreads), 0, s, P);
  else hipLaunchKernelGGL(gemm_kernel<2>, dim3(wgs), dim3(kThreads), 0, s, P);
  return hipGetLastError();
}

}  // namespace kvc
