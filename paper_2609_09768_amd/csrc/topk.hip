// Step a3: top-k row selection by deviation (gfx950).
//
// Paper: the tokens with the largest key deviation are recomputed, a fixed
// fraction of them (Section 3.2).  The selection here: the k largest d,
// ties to the lower row, returned in ascending row order.
//
// No sort.  Each float64 d maps to a 64-bit key whose unsigned order is the
// order of d, and the k-th largest key is closed in on by histograms.  n and k
// are known on the host, so nothing is read back, and the output is written
// in row order directly (per-block or per-thread counts and a scan).
//
// Up to 262,144 candidates the histograms follow the keys: the first covers
// [smallest key, largest key] (bins of a power of two in width), the next the
// bin the threshold fell into, until that bin holds few keys, which are then
// ranked against each other (by key, then row), or exactly as many as are
// still to be taken, or only equal keys, which are taken by row.  Deviations
// of one layer lie within a few octaves, so one histogram (of 2,048 bins) or
// two (of 256) are enough where digits of the raw key take eight passes; keys
// from the whole float64 range take up to six or eight.
// - Up to 16,384 candidates (contexts to about 16k tokens): one workgroup of
//   1,024 threads, keys in registers, bins in LDS.
// - Up to 262,144: one launch of a workgroup per 2,048 rows with grid barriers
//   between the histograms (below).
// - Above: a radix select one byte at a time (8 passes over the keys, most
//   significant byte first): every workgroup histograms the byte of the keys
//   that still match the prefix found so far, and the last workgroup to
//   finish (atomic ticket) picks the byte, updates the prefix and the
//   remaining rank, and clears the histogram for the next pass; then a count
//   and an ordered write, 11 launches.
#include "kvc_internal.h"

namespace kvc {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = kTopkRowsPerBlock / kThreads;  // 8 consecutive rows per thread

__device__ __forceinline__ unsigned long long order_key(double x) {
  unsigned long long b = (unsigned long long)__double_as_longlong(x);
  if ((b << 1) == 0ull) b = 0ull;  // -0.0 == +0.0
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// Exclusive scan over the 256 threads of a block; returns the block total.
__device__ __forceinline__ unsigned int block_excl_scan(unsigned int v, unsigned int* sh,
                                                        unsigned int& total) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
#pragma unroll
  for (int off = 1; off < kThreads; off <<= 1) {
    const unsigned int add = (t >= off) ? sh[t - off] : 0u;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  total = sh[kThreads - 1];
  const unsigned int incl = sh[t];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(kThreads) void topk_init(TopkState* st, long long k) {
  const int t = threadIdx.x;
  st->hist[t] = 0u;
  if (t == 0) {
    st->prefix = 0ull;
    st->mask = 0ull;
    st->rem = k;
    st->done = 0u;
  }
}

__global__ __launch_bounds__(kThreads) void topk_radix_pass(const double* __restrict__ dev,
                                                            long long n, TopkState* st,
                                                            int shift) {
  __shared__ unsigned int h[kThreads];
  __shared__ unsigned int suf[kThreads];
  __shared__ int is_last;
  const int t = threadIdx.x;
  const unsigned long long prefix = st->prefix;
  const unsigned long long mask = st->mask;
  const long long rem = st->rem;
  h[t] = 0u;
  __syncthreads();
  for (long long i = (long long)blockIdx.x * kThreads + t; i < n; i += (long long)gridDim.x * kThreads) {
    const unsigned long long key = order_key(dev[i]);
    if ((key & mask) == prefix) atomicAdd(&h[(key >> shift) & 255ull], 1u);
  }
  __syncthreads();
  if (h[t]) atomicAdd(&st->hist[t], h[t]);
  __threadfence();
  __syncthreads();
  if (t == 0) is_last = (atomicAdd(&st->done, 1u) == gridDim.x - 1);
  __syncthreads();
  if (!is_last) return;
  __threadfence();
  const unsigned int cnt = __hip_atomic_load(&st->hist[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // suf[b] = number of matching keys whose byte is >= b
  suf[t] = cnt;
  __syncthreads();
#pragma unroll
  for (int off = 1; off < kThreads; off <<= 1) {
    const unsigned int add = (t + off < kThreads) ? suf[t + off] : 0u;
    __syncthreads();
    suf[t] += add;
    __syncthreads();
  }
  const long long above = (long long)(suf[t] - cnt);
  if (above < rem && rem <= (long long)suf[t]) {  // exactly one byte value qualifies
    st->prefix = prefix | ((unsigned long long)t << shift);
    st->mask = mask | (255ull << shift);
    st->rem = rem - above;
  }
  st->hist[t] = 0u;
  if (t == 0) st->done = 0u;
}

// Per block of 2048 rows: how many keys are above T and equal to T.
__global__ __launch_bounds__(kThreads) void topk_count(const double* __restrict__ dev, long long n,
                                                       const TopkState* st,
                                                       unsigned int* __restrict__ bc) {
  __shared__ unsigned int sh[kThreads];
  const unsigned long long T = st->prefix;
  const long long base = (long long)blockIdx.x * kTopkRowsPerBlock + (long long)threadIdx.x * kItems;
  unsigned int gt = 0u, eq = 0u;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const long long r = base + i;
    if (r < n) {
      const unsigned long long key = order_key(dev[r]);
      gt += key > T;
      eq += key == T;
    }
  }
  unsigned int tot_gt, tot_eq;
  block_excl_scan(gt, sh, tot_gt);
  block_excl_scan(eq, sh, tot_eq);
  if (threadIdx.x == 0) {
    bc[2 * blockIdx.x] = tot_gt;
    bc[2 * blockIdx.x + 1] = tot_eq;
  }
}

__global__ __launch_bounds__(kThreads) void topk_write(const double* __restrict__ dev, long long n,
                                                       const TopkState* st,
                                                       const unsigned int* __restrict__ bc,
                                                       long long k, long long n_append,
                                                       int32_t* __restrict__ out) {
  __shared__ unsigned int sh[kThreads];
  __shared__ unsigned long long red[2];
  const int t = threadIdx.x;
  // the appended rows n .. n + n_append - 1 after the selection (no launch of their own)
  for (long long i = (long long)blockIdx.x * kThreads + t; i < n_append; i += (long long)gridDim.x * kThreads)
    out[k + i] = (int32_t)(n + i);
  const unsigned long long T = st->prefix;
  const long long need_eq = st->rem;  // rows equal to T still to take, in row order

  // counts of all earlier blocks
  unsigned long long gtb = 0ull, eqb = 0ull;
  for (int b = t; b < (int)blockIdx.x; b += kThreads) {
    gtb += bc[2 * b];
    eqb += bc[2 * b + 1];
  }
  if (t == 0) { red[0] = 0ull; red[1] = 0ull; }
  __syncthreads();
  if (gtb) atomicAdd(&red[0], gtb);
  if (eqb) atomicAdd(&red[1], eqb);
  __syncthreads();
  const long long gt_before = (long long)red[0];
  const long long eq_before = (long long)red[1];
  const long long sel_before = gt_before + (eq_before < need_eq ? eq_before : need_eq);

  const long long base = (long long)blockIdx.x * kTopkRowsPerBlock + (long long)t * kItems;
  unsigned long long keys[kItems];
  unsigned int eq_t = 0u;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const long long r = base + i;
    keys[i] = (r < n) ? order_key(dev[r]) : 0ull;
    eq_t += (r < n) && keys[i] == T;
  }
  unsigned int tot;
  const unsigned int eq_excl = block_excl_scan(eq_t, sh, tot);
  bool take[kItems];
  unsigned int sel_t = 0u;
  long long rank = eq_before + eq_excl;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const long long r = base + i;
    const bool valid = r < n;
    const bool is_eq = valid && keys[i] == T;
    take[i] = valid && (keys[i] > T || (is_eq && rank < need_eq));
    rank += is_eq;
    sel_t += take[i];
  }
  const unsigned int sel_excl = block_excl_scan(sel_t, sh, tot);
  long long o = sel_before + sel_excl;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    if (take[i] && o < k) out[o++] = (int32_t)(base + i);  // o < k always; the guard keeps writes in bounds
  }
}

// ---- single-workgroup path -------------------------------------------------
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallItems = 16;  // consecutive rows per thread at most, keys in registers
constexpr long long kSmallMax = (long long)kSmallThreads * kSmallItems;
constexpr int kSmallBins = 2048;
constexpr int kMaxCand = 128;    // keys left in the threshold's bin that are ranked one against another

// The keys that may still be selected: [lo, lo + 2^bits), and what is known
// of them.  Uniform over the workgroup (and the grid).
struct Bracket {
  unsigned long long lo;
  int bits;            // 64: everything from lo on
  long long rem;       // rows of the bracket to take; every key above it is taken
  unsigned int count;  // keys in the bracket
  __device__ bool in(unsigned long long key) const { return key >= lo && (bits >= 64 || ((key - lo) >> bits) == 0); }
  __device__ bool above(unsigned long long key) const { return bits < 64 && key >= lo && ((key - lo) >> bits) != 0; }
  // how the rest is decided
  __device__ bool all() const { return (long long)count == rem; }
  __device__ bool few() const { return count <= kMaxCand; }
  __device__ bool equal() const { return bits == 0; }
  __device__ bool done() const { return all() || few() || equal(); }
};

// Bits of a bracket that spans [lo, hi].
__device__ __forceinline__ int span_bits(unsigned long long lo, unsigned long long hi) { return 64 - __clzll((long long)(hi - lo)); }

// Largest of two values over a wave.
__device__ __forceinline__ void wave_max2(unsigned long long& a, unsigned long long& b) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const unsigned long long x = __shfl_xor(a, m, 64), y = __shfl_xor(b, m, 64);
    a = x > a ? x : a;
    b = y > b ? y : b;
  }
}

// Exclusive scan over the block's WAVES x 64 threads (wave scans + wave totals).
template <int WAVES>
__device__ __forceinline__ unsigned int block_scan(unsigned int v, unsigned int* wsum, unsigned int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int u = __shfl_up(incl, off, 64);
    if (lane >= off) incl += u;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  unsigned int before = 0u, tot = 0u;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const unsigned int x = wsum[w];
    before += (w < wave) ? x : 0u;
    tot += x;
  }
  __syncthreads();  // wsum is reused by the next scan
  total = tot;
  return before + incl - v;
}

// Sum over 2 or 8 consecutive lanes, in all of them, without the LDS round
// trips of a shuffle (0.3 us in a chain of 8): lanes 1 and 2 apart by
// quad_perm, 4 apart by row_half_mirror once the sums of four are equal.
template <int CTRL>
__device__ __forceinline__ int add_dpp(int r) {
  return r + __builtin_amdgcn_update_dpp(0, r, CTRL, 0xF, 0xF, false);
}
template <int LANES>
__device__ __forceinline__ int sum_lanes(int r) {
  static_assert(LANES == 2 || LANES == 8, "");
  r = add_dpp<0xB1>(r);
  if (LANES == 2) return r;
  return add_dpp<0x141>(add_dpp<0x4E>(r));
}

// Whether candidate c is among the first `rem` of the n candidates (larger key
// first, then lower row), for LANES consecutive lanes that share it, each
// comparing every LANES-th.  (Each candidate ranked by the thread that holds
// its row, one after the other, cost up to 45 us where a hundred candidates
// lay in few waves: 16,385 keys from the whole float64 range 57 -> 21 us,
// 16,384 deviations 32 -> 19.)
template <int LANES>
__device__ __forceinline__ bool among_first(int c, long long rem, const unsigned long long* ck, const int* cr, int n) {
  int r = 0;
  if (c < n) {
    const unsigned long long key = ck[c];
    const int row = cr[c];
#pragma unroll 8
    for (int j = (int)(threadIdx.x % LANES); j < n; j += LANES) r += (ck[j] > key) || (ck[j] == key && cr[j] < row);
  }
  return (sum_lanes<LANES>(r) < rem) & (c < n);
}

// One workgroup: 1,024 candidates 18.2 -> 6.6 us, 4,000 22.0 -> 8.3, 16,384 39.4
// -> 18.2 against eight byte passes; bound by the chain of its steps (loads, reduction, histogram,
// scan, rank, scan, store), 1 to 2 us each.
template <int ITEMS>
__global__ __launch_bounds__(kSmallThreads) void topk_small(const double* __restrict__ dev, long long n,
                                                            long long k, long long n_append,
                                                            int32_t* __restrict__ out) {
  __shared__ unsigned int hist[kSmallBins];
  __shared__ unsigned int wsum[kSmallWaves];
  __shared__ unsigned long long smax[kSmallWaves], sneg[kSmallWaves];
  __shared__ unsigned long long ck[kMaxCand];
  __shared__ int cr[kMaxCand];
  __shared__ Bracket s_next;
  __shared__ unsigned int s_cand;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (long long i = t; i < n_append; i += kSmallThreads) out[k + i] = (int32_t)(n + i);
  const int base = t * ITEMS, nv = (int)n;
  unsigned long long key[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) key[i] = (base + i < nv) ? order_key(dev[base + i]) : 0ull;
#pragma unroll
  for (int b = t; b < kSmallBins; b += kSmallThreads) hist[b] = 0u;
  if (t == 0) s_cand = 0u;
  unsigned long long hi = 0ull, neg = 0ull;  // largest key, largest ~key
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (base + i < nv) {
      hi = key[i] > hi ? key[i] : hi;
      neg = ~key[i] > neg ? ~key[i] : neg;
    }
  wave_max2(hi, neg);
  if (lane == 0) {
    smax[wave] = hi;
    sneg[wave] = neg;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSmallWaves; ++w) {
    hi = smax[w] > hi ? smax[w] : hi;
    neg = sneg[w] > neg ? sneg[w] : neg;
  }
  Bracket b = {~neg, span_bits(~neg, hi), k, (unsigned int)n};
  while (!b.done()) {
    const int shift = b.bits > 11 ? b.bits - 11 : 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (base + i < nv && b.in(key[i])) atomicAdd(&hist[(key[i] - b.lo) >> shift], 1u);
    __syncthreads();
    // thread t holds bins 2 t and 2 t + 1; keys in higher bins = all - those up to here
    const unsigned int c0 = hist[2 * t], c1 = hist[2 * t + 1];
    unsigned int tot;
    const unsigned int before = block_scan<kSmallWaves>(c0 + c1, wsum, tot);
    hist[2 * t] = 0u;
    hist[2 * t + 1] = 0u;
    const long long above1 = (long long)(tot - before - c0 - c1), above0 = above1 + c1;
    if (above1 < b.rem && b.rem <= above0)
      s_next = {b.lo + ((unsigned long long)(2 * t + 1) << shift), shift, b.rem - above1, c1};
    else if (above0 < b.rem && b.rem <= above0 + c0)
      s_next = {b.lo + ((unsigned long long)(2 * t) << shift), shift, b.rem - above0, c0};
    __syncthreads();  // exactly one bin qualifies
    b = s_next;
    __syncthreads();
  }
  unsigned int take = 0u, in = 0u;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (base + i < nv) {
      take |= (unsigned int)b.above(key[i]) << i;
      in |= (unsigned int)b.in(key[i]) << i;
    }
  unsigned int tot;
  if (b.all()) {
    take |= in;
  } else if (b.few()) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (in >> i & 1u) {
        const unsigned int j = atomicAdd(&s_cand, 1u);
        ck[j] = key[i];
        cr[j] = base + i;
      }
    __syncthreads();
    // eight lanes a candidate; the rows taken come back through the bins,
    // which are zero, as a mask for each thread
    constexpr int kLanes = kSmallThreads / kMaxCand;
    const int c = t / kLanes;
    if (among_first<kLanes>(c, b.rem, ck, cr, (int)s_cand) && t % kLanes == 0)
      atomicOr(&hist[cr[c] / ITEMS], 1u << (cr[c] % ITEMS));
    __syncthreads();
    take |= hist[t];
  } else {  // equal keys: by row
    long long rank = block_scan<kSmallWaves>((unsigned int)__popc(in), wsum, tot);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (in >> i & 1u) take |= (unsigned int)(rank++ < b.rem) << i;
  }
  long long o = block_scan<kSmallWaves>((unsigned int)__popc(take), wsum, tot);
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if ((take >> i & 1u) && o < k) out[o++] = (int32_t)(base + i);  // o < k always; kept in bounds
}

template <int ITEMS>
hipError_t launch_small(const double* dev, int64_t n, int64_t k, int64_t n_append, int32_t* out, hipStream_t s) {
  hipLaunchKernelGGL(topk_small<ITEMS>, dim3(1), dim3(kSmallThreads), 0, s, dev, (long long)n, (long long)k,
                     (long long)n_append, out);
  return hipGetLastError();
}

// ---- fused path: all steps in one launch -------------------------------------
// From 16,385 to kFusedMaxRows candidates: one workgroup per 2,048 rows (at
// most 128, so every workgroup is resident at once on the 256 CUs), each
// thread keeping its 8 consecutive rows' keys in registers.  The steps are
// separated by grid barriers (an arrival counter in the workspace); after
// each histogram every workgroup reads it and picks the same bin, so no
// workgroup has to publish it.  Histogram h adds into array h % 3; after its
// barrier, workgroup 0 clears array (h + 2) % 3, which every workgroup
// finished reading before it arrived there and which nobody adds into before
// the next barrier.  Once the rest is decided the other two arrays hold the
// candidates.  Four barriers (range, two histograms, counts and candidates)
// where eight byte passes took nine: 32,000 candidates 30.6 -> 15.3 us,
// 124,000 36.8 -> 22.0, and in a layer the deviation's launch zeroes the state
// (4 us for a launch of its own).
constexpr int kFusedMaxBlocks = 128;
constexpr long long kFusedMaxRows = (long long)kFusedMaxBlocks * kTopkRowsPerBlock;
constexpr int kFusedWaves = kThreads / 64;
// Every barrier wait is bounded (spin_limit looks at the counter, seconds in
// all), and a workgroup whose wait runs out leaves the kernel: it reads no
// exchanged value, and since it does not arrive again, no later barrier lets
// any other workgroup pass.  So whoever goes on has seen every arrival and
// holds the same bracket as the others, and the launch ends after one
// exhausted wait per workgroup at most, with the rows of the workgroups that
// left not written.  It happens only if some workgroup of the grid cannot run
// at all, which at most 128 workgroups of 256 threads on 256 CUs does not
// (the other kernels that may share the GPU, on other streams, all finish on
// their own).
// The search needs at most eight histograms of 256 bins for 64-bit keys.
// That, and the number of candidates, is checked all the same, so that a
// workspace which another stream writes meanwhile (not allowed) makes the
// selection wrong and nothing else.
static_assert(sizeof(TopkFused::hist[0]) == kThreads * 4 && kMaxCand * 8 <= kThreads * 4, "candidates fit a histogram");

__global__ __launch_bounds__(kThreads) void topk_fused_init(TopkFused* st) {
  unsigned int* w = reinterpret_cast<unsigned int*>(st);
  for (int i = threadIdx.x; i < (int)(sizeof(TopkFused) / 4); i += kThreads) w[i] = 0u;
}

__device__ __forceinline__ unsigned int load_dev(const unsigned int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_dev(unsigned int* p, unsigned int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every workgroup of the grid arrives once per barrier id, then waits until
// all have; the workgroup's *gave_up (0 before) is set if the spin bound is
// reached first.  The caller looks at it beside its first reads of exchanged
// values and uses none of them if it is set: 0.5 us of 15 at 20,000
// candidates, 0.3 to 0.7 from 64,000 on, and 0.2 more with a result written
// and read at every barrier.  Everything the workgroups exchange (histogram
// adds and clears, ranges, block counts, candidates, the arrival counter) is
// a device-scope atomic, performed where all XCDs see it, so the barrier
// needs no cache writeback: each wave waits until its own atomics are done
// before the workgroup arrives, and a workgroup uses the exchanged values
// only after it has seen every arrival.
__device__ __forceinline__ void grid_barrier(TopkFused* st, unsigned int id, int spin_limit, int* gave_up) {
  __builtin_amdgcn_s_waitcnt(0);  // this wave's adds and stores are done
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(&st->arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned int target = (id + 1u) * gridDim.x;
    int left = spin_limit;
#pragma unroll 8
    for (; left > 0; --left) {
      if (load_dev(&st->arrive) >= target) break;
      __builtin_amdgcn_s_sleep(1);
    }
    if (left == 0) *gave_up = 1;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kThreads) void topk_fused(const double* __restrict__ dev, long long n, long long k,
                                                       long long n_append, TopkFused* st,
                                                       unsigned int* __restrict__ bc, int32_t* __restrict__ out,
                                                       int spin_limit) {
  __shared__ unsigned int h[kThreads];
  __shared__ unsigned int wsum[kFusedWaves];
  __shared__ unsigned long long smax[kFusedWaves], sneg[kFusedWaves];
  __shared__ unsigned long long ck[kMaxCand];
  __shared__ int cr[kMaxCand];
  __shared__ Bracket s_next;
  __shared__ unsigned int red[2];
  __shared__ int gave_up;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const long long base = (long long)blockIdx.x * kTopkRowsPerBlock + (long long)t * kItems;
  for (long long i = (long long)blockIdx.x * kThreads + t; i < n_append; i += (long long)gridDim.x * kThreads)
    out[k + i] = (int32_t)(n + i);
  unsigned long long key[kItems];
  unsigned int valid = 0u;
  unsigned long long hi = 0ull, neg = 0ull;  // largest key, largest ~key
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const bool v = base + i < n;
    key[i] = v ? order_key(dev[base + i]) : 0ull;
    valid |= (unsigned int)v << i;
    hi = key[i] > hi ? key[i] : hi;
    const unsigned long long c = v ? ~key[i] : 0ull;
    neg = c > neg ? c : neg;
  }
  h[t] = 0u;
  if (t == 0) gave_up = 0;
  unsigned int bar = 0u;
  // largest hi and neg of the grid, through range[i] of the workspace
  auto grid_max2 = [&](int i) {
    wave_max2(hi, neg);
    if (lane == 0) {
      smax[wave] = hi;
      sneg[wave] = neg;
    }
    __syncthreads();
    unsigned long long* range = st->range[i];
    if (t == 0) {
#pragma unroll
      for (int w = 1; w < kFusedWaves; ++w) {
        hi = smax[w] > hi ? smax[w] : hi;
        neg = sneg[w] > neg ? sneg[w] : neg;
      }
      __hip_atomic_fetch_max(&range[0], hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_max(&range[1], neg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    grid_barrier(st, bar++, spin_limit, &gave_up);
    hi = __hip_atomic_load(&range[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    neg = __hip_atomic_load(&range[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return gave_up == 0;
  };
  if (!grid_max2(0)) return;
  Bracket b = {~neg, span_bits(~neg, hi), k, (unsigned int)n};
  if (t == 0) s_next = b;
  int level = 0;
  while (level < kTopkMaxLevels && !b.done()) {
    const int shift = b.bits > 8 ? b.bits - 8 : 0;
    unsigned int* gh = st->hist[level % 3];
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if ((valid >> i & 1u) && b.in(key[i])) atomicAdd(&h[(key[i] - b.lo) >> shift], 1u);
    __syncthreads();
    if (h[t]) atomicAdd(&gh[t], h[t]);
    h[t] = 0u;
    grid_barrier(st, bar++, spin_limit, &gave_up);
    const unsigned int c = load_dev(&gh[t]);
    unsigned int tot;
    const unsigned int before = block_scan<kFusedWaves>(c, wsum, tot);
    const long long above = (long long)(tot - before - c);
    if (above < b.rem && b.rem <= above + c)  // exactly one bin qualifies
      s_next = {b.lo + ((unsigned long long)t << shift), shift, b.rem - above, c};
    __syncthreads();
    const unsigned int count = b.count;
    b = s_next;
    if (gave_up) return;
    __syncthreads();  // s_next is rewritten by the next level
    if (blockIdx.x == 0 && !b.done()) store_dev(&st->hist[(level + 2) % 3][t], 0u);
    ++level;
    if (b.count == count && !b.done()) {
      // a histogram that told no keys apart: they lie close together (equal,
      // most often), so the bracket shrinks to their range: three distinct
      // values in 262,144 rows 60 -> 38 us, 56 with byte passes
      hi = neg = 0ull;
#pragma unroll
      for (int i = 0; i < kItems; ++i)
        if ((valid >> i & 1u) && b.in(key[i])) {
          hi = key[i] > hi ? key[i] : hi;
          neg = ~key[i] > neg ? ~key[i] : neg;
        }
      if (!grid_max2(level)) return;
      b.lo = ~neg;
      b.bits = span_bits(~neg, hi);
    }
  }
  // Per workgroup: rows above the bracket and (equal keys) in it, and the
  // candidates, then the ordered write.
  unsigned int take = 0u, in = 0u;
#pragma unroll
  for (int i = 0; i < kItems; ++i)
    if (valid >> i & 1u) {
      take |= (unsigned int)b.above(key[i]) << i;
      in |= (unsigned int)b.in(key[i]) << i;
    }
  const bool few = !b.all() && b.few(), ties = !b.all() && !b.few();
  if (b.all()) take |= in;
  unsigned int tot_take, tot_in = 0u, in_before = 0u;
  block_scan<kFusedWaves>((unsigned int)__popc(take), wsum, tot_take);
  if (ties) in_before = block_scan<kFusedWaves>((unsigned int)__popc(in), wsum, tot_in);
  // array level % 3 was last read (or never used), the one after it is clean
  unsigned long long* gk = reinterpret_cast<unsigned long long*>(st->hist[level % 3]);
  unsigned int* gr = st->hist[(level + 1) % 3];
  if (few) {
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if (in >> i & 1u) {
        const unsigned int j = atomicAdd(&st->cand, 1u);
        if (j >= kMaxCand) continue;
        __hip_atomic_store(&gk[j], key[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        store_dev(&gr[j], (unsigned int)(base + i));
      }
  }
  if (t == 0) {
    store_dev(&bc[2 * blockIdx.x], tot_take);
    store_dev(&bc[2 * blockIdx.x + 1], tot_in);
    red[0] = 0u;
    red[1] = 0u;
  }
  grid_barrier(st, bar++, spin_limit, &gave_up);
  if (t < (int)blockIdx.x) {  // at most 128 workgroups
    atomicAdd(&red[0], load_dev(&bc[2 * t]));
    if (ties) atomicAdd(&red[1], load_dev(&bc[2 * t + 1]));
  }
  const int nc = few ? (int)b.count : 0;
  if (t < nc) {
    ck[t] = __hip_atomic_load(&gk[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    cr[t] = (int)load_dev(&gr[t]);
  }
  __syncthreads();
  long long sel_before = red[0];
  if (gave_up) return;
  if (few) {
    // two lanes a candidate; this workgroup's rows come back through the bins,
    // which are zero, and those taken in earlier workgroups are counted
    constexpr int kLanes = kThreads / kMaxCand;
    const int c = t / kLanes;
    const bool first = among_first<kLanes>(c, b.rem, ck, cr, nc) && t % kLanes == 0;
    const int at = first ? cr[c] - (int)(blockIdx.x * kTopkRowsPerBlock) : 0;  // place in this workgroup's rows
    if (first && at >= 0 && at < kTopkRowsPerBlock) atomicOr(&h[at / kItems], 1u << (at % kItems));
    sel_before += __syncthreads_count(first && at < 0);
    take |= h[t];
  } else if (ties) {
    const long long eq_before = red[1];
    sel_before += eq_before < b.rem ? eq_before : b.rem;
    long long rank = eq_before + in_before;
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if (in >> i & 1u) take |= (unsigned int)(rank++ < b.rem) << i;
  }
  unsigned int tot;
  long long o = sel_before + block_scan<kFusedWaves>((unsigned int)__popc(take), wsum, tot);
#pragma unroll
  for (int i = 0; i < kItems; ++i)
    if ((take >> i & 1u) && o < k) out[o++] = (int32_t)(base + i);  // o < k always; kept in bounds
}

// out[i] = start + i for i < count
__global__ __launch_bounds__(kThreads) void iota_kernel(int32_t* __restrict__ out, long long count,
                                                        long long start) {
  for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < count;
       i += (long long)gridDim.x * kThreads)
    out[i] = (int32_t)(start + i);
}

hipError_t launch_iota(int32_t* out, long long count, long long start, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  long long blocks = (count + kThreads - 1) / kThreads;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(iota_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, out, count, start);
  return hipGetLastError();
}

}  // namespace

size_t topk_clear_bytes(int64_t n) { return n > kSmallMax && n <= kFusedMaxRows ? sizeof(TopkFused) : 0; }

hipError_t launch_select_topk(const double* dev, int64_t n, int64_t k, int64_t n_append,
                              int32_t* idx_out, void* ws, bool cleared, hipStream_t s, int spin_limit) {
  if (k == 0) return launch_iota(idx_out, n_append, n, s);
  if (k == n) return launch_iota(idx_out, n + n_append, 0, s);
  if (n <= kSmallMax) {
    if (n <= kSmallThreads) return launch_small<1>(dev, n, k, n_append, idx_out, s);
    if (n <= 2 * kSmallThreads) return launch_small<2>(dev, n, k, n_append, idx_out, s);
    if (n <= 4 * kSmallThreads) return launch_small<4>(dev, n, k, n_append, idx_out, s);
    if (n <= 8 * kSmallThreads) return launch_small<8>(dev, n, k, n_append, idx_out, s);
    return launch_small<16>(dev, n, k, n_append, idx_out, s);
  }
  const size_t state = sizeof(TopkState) > sizeof(TopkFused) ? sizeof(TopkState) : sizeof(TopkFused);
  unsigned int* bc = reinterpret_cast<unsigned int*>(static_cast<char*>(ws) + align256(state));
  const long long nblk = topk_blocks(n);
  if (n <= kFusedMaxRows) {
    TopkFused* fs = static_cast<TopkFused*>(ws);
    if (!cleared) hipLaunchKernelGGL(topk_fused_init, dim3(1), dim3(kThreads), 0, s, fs);
    hipLaunchKernelGGL(topk_fused, dim3((unsigned)nblk), dim3(kThreads), 0, s, dev, (long long)n, (long long)k,
                       (long long)n_append, fs, bc, idx_out, spin_limit);
    return hipGetLastError();
  }
  TopkState* st = static_cast<TopkState*>(ws);
  long long pass_blocks = (n + kThreads * 8 - 1) / (kThreads * 8);
  if (pass_blocks > 1024) pass_blocks = 1024;
  hipLaunchKernelGGL(topk_init, dim3(1), dim3(kThreads), 0, s, st, (long long)k);
  for (int shift = 56; shift >= 0; shift -= 8)
    hipLaunchKernelGGL(topk_radix_pass, dim3((unsigned)pass_blocks), dim3(kThreads), 0, s, dev,
                       (long long)n, st, shift);
  hipLaunchKernelGGL(topk_count, dim3((unsigned)nblk), dim3(kThreads), 0, s, dev, (long long)n, st, bc);
  hipLaunchKernelGGL(topk_write, dim3((unsigned)nblk), dim3(kThreads), 0, s, dev, (long long)n, st,
                     bc, (long long)k, (long long)n_append, idx_out);
  return hipGetLastError();
}

}  // namespace kvc
