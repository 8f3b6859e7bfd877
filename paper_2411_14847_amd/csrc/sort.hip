// Prefix scan and the two sorts for wave64 (gfx950): the views' depth order (below), and a radix sort
// of one list of 32-bit keys, the densification's ranking of all members.
//
// The radix sort is reduce-then-scan with a fixed grid, so that the element count can stay on the
// device (no host round trip; the launch sequence is graph-capturable).  Each of three passes over
// an 11-bit digit is
//   (1) upsweep: every block histograms its contiguous chunk into LDS (per-wave
//       sub-histograms to spread LDS atomics), written digit-major to global memory;
//   (2) scan: one workgroup per digit turns the [radix][blocks] counts into global offsets;
//   (3) scatter: every block re-reads its chunk in batches of 4,096 pairs, ranks them stably
//       with wave ballots (11 ballots give each lane the mask of lanes holding the same
//       digit; each wave ranks its own quarter of the batch), orders the batch by digit in
//       LDS and writes each digit's run contiguously.
// A pass never depends on forward progress between workgroups.
#include <algorithm>

#include "dass_internal.h"

namespace dass {
namespace {

constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;                      // items per thread per batch
constexpr int kBatch = kSortThreads * kSortItems;  // 2048
constexpr int kRadixBits = 11, kRadix = 1 << kRadixBits;
constexpr int kMaxSortBlocks = 512;

__device__ __forceinline__ uint64_t lanemask_lt() {
  const int lane = threadIdx.x & 63;
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Inclusive scan within a wave of 64 lanes (shuffle-up steps).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

__device__ __forceinline__ uint64_t wave_incl_scan64(uint64_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint64_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

// Exclusive scan across a 256-thread block; returns the exclusive prefix, *total the sum.
__device__ __forceinline__ uint32_t block_excl_scan256(uint32_t x, uint32_t* s_wave, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = wave_incl_scan(x);
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < 4; w++) {
    uint32_t s = s_wave[w];
    if (w < wave) base += s;
    tot += s;
  }
  __syncthreads();
  if (total) *total = tot;
  return base + inc - x;
}

__device__ __forceinline__ uint32_t digit_of(uint32_t k, int shift) { return (k >> shift) & (kRadix - 1u); }

__device__ __forceinline__ void chunk_of(uint32_t count, int blocks, uint32_t& lo, uint32_t& hi) {
  const uint32_t chunk = (uint32_t)(((uint64_t)count + blocks - 1) / blocks);
  const uint64_t l = (uint64_t)blockIdx.x * chunk;
  lo = (uint32_t)(l < count ? l : count);
  const uint64_t h = l + chunk;
  hi = (uint32_t)(h < count ? h : count);
}

__global__ __launch_bounds__(kSortThreads) void k_upsweep(const uint32_t* __restrict__ keys,
                                                          const uint32_t* __restrict__ d_count, int shift, int blocks,
                                                          uint32_t* __restrict__ hist) {
  constexpr int R = kRadix;
  __shared__ uint32_t s_h[4][R];
  const int tid = threadIdx.x, wave = tid >> 6;
  for (int i = tid; i < 4 * R; i += kSortThreads) (&s_h[0][0])[i] = 0;
  __syncthreads();
  uint32_t lo, hi;
  chunk_of(*d_count, blocks, lo, hi);
  uint32_t i = lo + tid;
  // eight independent loads in flight per thread, then their LDS increments
  for (; i + (kSortItems - 1) * kSortThreads < hi; i += kSortItems * kSortThreads) {
    uint32_t k[kSortItems];
#pragma unroll
    for (int u = 0; u < kSortItems; u++) k[u] = keys[i + u * kSortThreads];
#pragma unroll
    for (int u = 0; u < kSortItems; u++) atomicAdd(&s_h[wave][digit_of(k[u], shift)], 1u);
  }
  for (; i < hi; i += kSortThreads) atomicAdd(&s_h[wave][digit_of(keys[i], shift)], 1u);
  __syncthreads();
  for (int d = tid; d < R; d += kSortThreads)
    hist[(int64_t)d * blocks + blockIdx.x] = s_h[0][d] + s_h[1][d] + s_h[2][d] + s_h[3][d];
}

// Exclusive scan of each digit's row of block counts (one workgroup per digit); the row total
// goes to totals[digit].  The scatter adds the exclusive scan of the totals.
__global__ __launch_bounds__(kSortThreads) void k_scan_rows(uint32_t* __restrict__ hist, int blocks,
                                                            uint32_t* __restrict__ totals) {
  __shared__ uint32_t s_w[4];
  uint32_t* row = hist + (int64_t)blockIdx.x * blocks;
  const int per = (blocks + kSortThreads - 1) / kSortThreads;
  const int b = threadIdx.x * per, e = min(b + per, blocks);
  uint32_t sum = 0;
  for (int i = b; i < e; i++) sum += row[i];
  uint32_t tot;
  uint32_t run = block_excl_scan256(sum, s_w, &tot);
  for (int i = b; i < e; i++) {
    const uint32_t c = row[i];
    row[i] = run;
    run += c;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

// Exclusive scan over R digits held D = R/256 per thread (consecutive); returns per-thread
// prefix base (the thread's first digit's offset); *total is the sum of all.
template <int D>
__device__ __forceinline__ uint32_t block_excl_scan_digits(const uint32_t* c, uint32_t* s_tmp, uint32_t* total) {
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < D; i++) sum += c[i];
  return block_excl_scan256(sum, s_tmp, total);
}

// Orders LDS accesses of the lanes of one wave (a wave's LDS instructions complete in order;
// this only keeps the compiler from moving them across the point).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Each batch of 256 IT pairs is split into four runs of 64 IT consecutive pairs, one per wave; a
// wave ranks its run slot by slot (64 pairs at a time) against its own running digit counts,
// with no workgroup barrier, so the ranks follow the input order.  Waves are then combined by
// an exclusive prefix of their counts per digit, the batch is ordered by digit in LDS, and each
// digit's run is written to its global position.
__global__ __launch_bounds__(kSortThreads) void k_scatter(const uint32_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                          uint32_t* __restrict__ vout,
                                                          const uint32_t* __restrict__ d_count, int shift, int blocks,
                                                          const uint32_t* __restrict__ hist,
                                                          const uint32_t* __restrict__ totals) {
  constexpr int R = kRadix, IT = 16;         // pairs per thread and batch
  constexpr int D = R / kSortThreads;        // digits owned per thread
  constexpr int kWaveRun = IT * 64;          // consecutive pairs ranked by one wave per batch
  constexpr int kBatchP = kSortThreads * IT;  // pairs per batch
  __shared__ uint32_t s_base[R];             // global write position of the next item of each digit
  __shared__ uint32_t s_boff[R];             // exclusive digit offsets within the batch
  __shared__ uint32_t s_wc[4][R];            // per-wave digit counts, then their prefix over waves
  __shared__ uint32_t s_tmp[4];
  __shared__ uint32_t s_k[kBatchP];
  __shared__ uint32_t s_v[kBatchP];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const uint32_t count = *d_count;
  uint32_t lo, hi;
  chunk_of(count, blocks, lo, hi);
  {  // global base of each digit for this block: row prefix + exclusive scan of the digit totals
    uint32_t tv[D];
#pragma unroll
    for (int i = 0; i < D; i++) tv[i] = totals[tid * D + i];
    uint32_t run = block_excl_scan_digits<D>(tv, s_tmp, nullptr);
#pragma unroll
    for (int i = 0; i < D; i++) {
      const int d = tid * D + i;
      s_base[d] = hist[(int64_t)d * blocks + blockIdx.x] + run;
      run += tv[i];
    }
  }
  const uint64_t lt = lanemask_lt();

  for (uint32_t batch = lo; batch < hi; batch += kBatchP) {
    const uint32_t nb = min((uint32_t)kBatchP, hi - batch);
    const uint32_t wbase = batch + (uint32_t)(wave * kWaveRun);
    for (int d = lane; d < R; d += 64) s_wc[wave][d] = 0;
    uint32_t key[IT], val[IT], rank[IT], dig[IT];
#pragma unroll
    for (int s = 0; s < IT; s++) {
      const uint32_t idx = wbase + (uint32_t)(s * 64 + lane);
      if (idx < hi) {
        key[s] = kin[idx];
        val[s] = vin[idx];
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int s = 0; s < IT; s++) {
      const bool valid = wbase + (uint32_t)(s * 64 + lane) < hi;
      const uint32_t d = valid ? digit_of(key[s], shift) : 0u;
      dig[s] = d;
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int b = 0; b < kRadixBits; b++) {
        const uint64_t m = __ballot((d >> b) & 1);
        peers &= ((d >> b) & 1) ? m : ~m;
      }
      const uint32_t rw = __popcll(peers & lt);
      const uint32_t base = s_wc[wave][d];  // every lane of the digit reads before the leader adds
      wave_lds_sync();
      if (valid && rw == 0) s_wc[wave][d] = base + __popcll(peers);
      wave_lds_sync();
      rank[s] = base + rw;
    }
    __syncthreads();
    uint32_t c[D];
#pragma unroll
    for (int i = 0; i < D; i++) {  // thread owns digits tid*D..: prefix over waves, batch count
      const int dd = tid * D + i;
      uint32_t run = 0;
#pragma unroll
      for (int w = 0; w < 4; w++) {
        const uint32_t x = s_wc[w][dd];
        s_wc[w][dd] = run;
        run += x;
      }
      c[i] = run;
    }
    {
      uint32_t run = block_excl_scan_digits<D>(c, s_tmp, nullptr);
#pragma unroll
      for (int i = 0; i < D; i++) {
        s_boff[tid * D + i] = run;
        run += c[i];
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++) {
      if (wbase + (uint32_t)(s * 64 + lane) < hi) {
        const uint32_t pos = s_boff[dig[s]] + s_wc[wave][dig[s]] + rank[s];
        s_k[pos] = key[s];
        s_v[pos] = val[s];
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++) {
      const uint32_t j = s * kSortThreads + tid;
      if (j < nb) {
        const uint32_t k = s_k[j];
        const uint32_t d = digit_of(k, shift);
        const uint32_t o = s_base[d] + (j - s_boff[d]);
        if (o < count) {  // always true for a consistent histogram; keeps stores in bounds
          kout[o] = k;
          vout[o] = s_v[j];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < D; i++) s_base[tid * D + i] += c[i];
    __syncthreads();
  }
}

// ---- per-view depth order --------------------------------------------------------------------
// The depth keys of a view are the float32 bits of its Gaussians' depths less those of the near
// plane (positive floats order as their bits), so below 2^27 - 1 for depths up to about 13,000,
// and kDepthInvisible for a Gaussian that is not drawn.  The sort is stable: equal depths keep
// index order.
// Bound: a pass reads and writes 8 bytes per Gaussian-view (4 in the upsweep); with 4M of them the
// scatter moves 64 MB in 33 us, short of the copy rate by the latency of its chain (digit counts, keys, 16 ranks,
// two reorderings in LDS).  Against four 9-bit passes over 64-bit (view, depth) keys: 20 views of
// 200k 0.209 -> 0.127 ms, 4 of 1M 0.214 -> 0.178, one of 200k 65 -> 65 us in 7 instead of 13
// launches; small views (12 launches before) 20 x 12k 0.084 -> 0.032 ms, 1 x 2k 50 -> 12 us.
constexpr int kDepthBits = 9;  // digit
constexpr int kDepthR = 1 << kDepthBits;

// Rank of a lane's digit among the lanes of the wave, and the count of the digits before: the lanes
// of a digit meet in the digit's mask (zero between calls), its last lane advances the count.
__device__ __forceinline__ uint32_t wave_rank(uint64_t* mask, uint16_t* count, uint32_t d, bool valid, int lane,
                                              uint64_t lt) {
  if (valid) atomicOr(reinterpret_cast<unsigned long long*>(&mask[d]), 1ull << lane);
  wave_lds_sync();
  const uint64_t m = mask[d];
  const uint32_t base = count[d];
  wave_lds_sync();
  if (valid && (m >> lane) == 1ull) {
    count[d] = (uint16_t)(base + __popcll(m));
    mask[d] = 0ull;
  }
  wave_lds_sync();
  return base + __popcll(m & lt);
}

// Views of few Gaussians: the whole view in LDS, one workgroup per view.  Thread t of wave w
// holds elements 64 (IT w + s) + t, s < IT, in registers between passes; the passes cover the
// range of the view's own visible keys, 9 bits each.
constexpr int kDepthLdsThreads = 1024, kDepthLdsWaves = 16;
template <int IT>
__global__ __launch_bounds__(kDepthLdsThreads) void k_depth_lds(int n, const uint32_t* __restrict__ keys,
                                                                uint32_t* __restrict__ out,
                                                                uint32_t* __restrict__ far) {
  __shared__ uint32_t s_x[IT * kDepthLdsThreads];  // in digit order: the keys, then the values
  __shared__ uint64_t s_mask[kDepthLdsWaves][kDepthR];
  __shared__ uint16_t s_wc[kDepthLdsWaves][kDepthR];
  __shared__ uint32_t s_off[kDepthR];
  __shared__ uint32_t s_red[2][kDepthLdsWaves];
  const int v = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = (int64_t)v * n;
  const int first = wave * 64 * IT + lane;  // element of slot 0
  uint32_t key[IT], val[IT];
  uint32_t lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
  for (int s = 0; s < IT; s++) {
    const int i = first + s * 64;
    key[s] = i < n ? keys[row + i] : kDepthInvisible;
    val[s] = (uint32_t)i;
    if (key[s] != kDepthInvisible) {
      lo = min(lo, key[s]);
      hi = max(hi, key[s]);
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
  }
  if (lane == 0) {
    s_red[0][wave] = lo;
    s_red[1][wave] = hi;
  }
  if (tid == 0) far[v] = 0;  // the other path's flag: not needed here
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kDepthLdsWaves; w++) {
    lo = min(lo, s_red[0][w]);
    hi = max(hi, s_red[1][w]);
  }
  const uint32_t top = hi >= lo ? hi - lo + 1 : 0u;  // the key of what is not drawn
  const int bits = 32 - __builtin_clz(top | 1u);
#pragma unroll
  for (int s = 0; s < IT; s++) key[s] = key[s] == kDepthInvisible ? top : key[s] - lo;
  const uint64_t lt = lanemask_lt();
  for (int d = lane; d < kDepthR; d += 64) s_mask[wave][d] = 0;
  for (int shift = 0; shift < bits; shift += kDepthBits) {
    for (int d = lane; d < kDepthR; d += 64) s_wc[wave][d] = 0;
    wave_lds_sync();
    uint32_t rank[IT];
#pragma unroll
    for (int s = 0; s < IT; s++)  // (elements past n stay out: their order is the last)
      rank[s] = wave_rank(s_mask[wave], s_wc[wave], (key[s] >> shift) & (kDepthR - 1), first + s * 64 < n, lane, lt);
    __syncthreads();
    if (tid < kDepthR) {  // digit tid: prefix over the waves, its count in s_off
      uint32_t run = 0;
#pragma unroll
      for (int w = 0; w < kDepthLdsWaves; w++) {
        const uint32_t x = s_wc[w][tid];
        s_wc[w][tid] = (uint16_t)run;
        run += x;
      }
      const uint32_t inc = wave_incl_scan(run);
      s_off[tid] = inc - run;
      if (lane == 63) s_red[0][wave] = inc;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++)
      if (first + s * 64 < n) {
        const uint32_t d = (key[s] >> shift) & (kDepthR - 1);
        rank[s] += s_off[d] + s_wc[wave][d];
#pragma unroll
        for (int w = 0; w < kDepthR / 64; w++) rank[s] += (uint32_t)w < d / 64 ? s_red[0][w] : 0u;
        s_x[rank[s]] = key[s];
      }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++)
      if (first + s * 64 < n) key[s] = s_x[first + s * 64];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++)
      if (first + s * 64 < n) s_x[rank[s]] = val[s];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++)
      if (first + s * 64 < n) val[s] = s_x[first + s * 64];
  }
#pragma unroll
  for (int s = 0; s < IT; s++)
    if (first + s * 64 < n) out[row + first + s * 64] = val[s];
}

// Larger views: least-significant-digit radix sort of every view by itself, three
// 9-bit digits of the keys' low 27 bits.  A pass is an upsweep (each block's digit counts) and a
// scatter, whose blocks add up the counts of the blocks before them by themselves.
constexpr int kDepthIt = 16;  // keys per thread of the upsweep's loads
constexpr int kDepthBatch = kSortThreads * kDepthIt;  // 4,096 pairs
constexpr int kDepthBlocks = 64;                       // blocks per view at most

// View v and block b of it that a workgroup takes, and the block's part [lo, hi) of the view.  Each
// XCD gets a contiguous part of the (view, block) order (workgroups are dealt to the XCDs
// round-robin), so the short runs that neighbouring blocks write to a digit merge in one L2.
__device__ __forceinline__ bool depth_piece(int n, int nv, int blocks, int& v, int& b, int& lo, int& hi) {
  const int total = nv * blocks, per = (total + kNumXcd - 1) / kNumXcd;
  const int i = (int)(blockIdx.x % kNumXcd) * per + (int)(blockIdx.x / kNumXcd);
  if (i >= total) return false;
  v = i / blocks;
  b = i % blocks;
  const int chunk = (n + blocks - 1) / blocks;
  lo = min(b * chunk, n);
  hi = min(lo + chunk, n);
  return true;
}

__global__ __launch_bounds__(kSortThreads) void k_depth_upsweep(int n, int nv, int blocks, int shift,
                                                                const uint32_t* __restrict__ keys,
                                                                uint32_t* __restrict__ hist,
                                                                uint32_t* __restrict__ far) {
  __shared__ uint32_t s_h[4][kDepthR];
  const int tid = threadIdx.x, wave = tid >> 6;
  for (int i = tid; i < 4 * kDepthR; i += kSortThreads) (&s_h[0][0])[i] = 0;
  __syncthreads();
  int v, b, lo, hi;
  if (!depth_piece(n, nv, blocks, v, b, lo, hi)) return;
  if (shift == 0 && b == 0 && tid == 0) {  // the projection's flag, for the passes of this call
    far[DASS_MAX_VIEWS + v] = far[v];
    far[v] = 0;
  }
  const uint32_t* __restrict__ k = keys + (int64_t)v * n;
  int i = lo + tid;
  for (; i + (kDepthIt - 1) * kSortThreads < hi; i += kDepthIt * kSortThreads) {
    uint32_t x[kDepthIt];
#pragma unroll
    for (int u = 0; u < kDepthIt; u++) x[u] = k[i + u * kSortThreads];
#pragma unroll
    for (int u = 0; u < kDepthIt; u++) atomicAdd(&s_h[wave][(x[u] >> shift) & (kDepthR - 1)], 1u);
  }
  for (; i < hi; i += kSortThreads) atomicAdd(&s_h[wave][(k[i] >> shift) & (kDepthR - 1)], 1u);
  __syncthreads();
  for (int d = tid; d < kDepthR; d += kSortThreads)
    hist[((int64_t)v * blocks + b) * kDepthR + d] = s_h[0][d] + s_h[1][d] + s_h[2][d] + s_h[3][d];
}

// NT threads.  FIRST: the values are the positions themselves.  LAST: the keys are written only if the view has
// far depths (a fourth digit follows), and its values then go to vspare.
template <bool FIRST, bool LAST, int NT>
__global__ __launch_bounds__(NT) void k_depth_scatter(int n, int nv, int blocks, int shift,
                                                                const uint32_t* __restrict__ kin,
                                                                const uint32_t* __restrict__ vin,
                                                                uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                                const uint32_t* __restrict__ hist,
                                                                const uint32_t* __restrict__ far,
                                                                uint32_t* __restrict__ vspare) {
  constexpr int NW = NT / 64, IT = kDepthBatch / NT;  // waves, pairs per thread and batch
  constexpr int OWN = NT < kDepthR ? NT : kDepthR;    // threads that own digits
  constexpr int D = kDepthR / OWN;                    // digits owned per thread
  constexpr int kRun = IT * 64;                       // consecutive pairs ranked by one wave per batch
  __shared__ uint32_t s_base[kDepthR], s_boff[kDepthR], s_tmp[OWN / 64];
  __shared__ uint16_t s_wc[NW][kDepthR];
  __shared__ uint64_t s_mask[NW][kDepthR];
  for (int i = threadIdx.x; i < NW * kDepthR; i += NT) (&s_mask[0][0])[i] = 0;
  __shared__ uint32_t s_x[kDepthBatch];  // the batch in digit order: its keys, then its values
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int v, blk, lo, hi;
  if (!depth_piece(n, nv, blocks, v, blk, lo, hi) || lo >= hi) return;  // uniform over the workgroup
  const int64_t row = (int64_t)v * n;
  const bool write_keys = !LAST || far[DASS_MAX_VIEWS + v] != 0;
  if (LAST && write_keys) vout = vspare;
  // exclusive scan over the digits, thread t < OWN with the digits t D, t D + 1, ...; whole workgroup
  auto digit_scan = [&](const uint32_t (&x)[D]) {
    uint32_t own = 0;
#pragma unroll
    for (int i = 0; i < D; i++) own += x[i];
    const uint32_t inc = wave_incl_scan(own);
    if (lane == 63 && tid < OWN) s_tmp[wave] = inc;
    __syncthreads();
    uint32_t run = inc - own;
#pragma unroll
    for (int w = 0; w < OWN / 64; w++) run += w < wave ? s_tmp[w] : 0u;
    __syncthreads();
    return run;
  };
  {  // first position of each digit: the digit's counts in the blocks before, after all smaller digits;
     // where threads outnumber the digits, they read the blocks' counts in turn
    constexpr int G = NT / OWN, kAhead = D == 2 ? 8 : 16;
    const int o = tid % OWN, gr = tid / OWN;
    const uint32_t* __restrict__ h = hist + (int64_t)v * blocks * kDepthR + o * D;
    uint32_t before[D], total[D];
#pragma unroll
    for (int i = 0; i < D; i++) before[i] = total[i] = 0u;
    for (int b = gr; b < blocks; b += G * kAhead) {
      typedef uint32_t Digits __attribute__((ext_vector_type(D)));  // a thread's digits, one load
      Digits x[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; u++)
        x[u] = b + u * G < blocks ? *reinterpret_cast<const Digits*>(h + (int64_t)(b + u * G) * kDepthR) : Digits(0u);
#pragma unroll
      for (int u = 0; u < kAhead; u++)
#pragma unroll
        for (int i = 0; i < D; i++) {
          total[i] += x[u][i];
          before[i] += b + u * G < blk ? x[u][i] : 0u;
        }
    }
    if (G > 1) {
      static_assert(G <= 2, "one other group's sums");
      if (gr == 1) s_base[o] = total[0], s_boff[o] = before[0];
      __syncthreads();
      if (gr == 0) total[0] += s_base[o], before[0] += s_boff[o];
      __syncthreads();
    }
    uint32_t run = digit_scan(total);
    if (gr == 0) {
#pragma unroll
      for (int i = 0; i < D; i++) {
        s_base[o * D + i] = run + before[i];
        run += total[i];
      }
    }
  }
  const uint64_t lt = lanemask_lt();
  for (int batch = lo; batch < hi; batch += kDepthBatch) {
    const int nb = min(kDepthBatch, hi - batch);
    const int wbase = batch + wave * kRun;
    for (int d = lane; d < kDepthR; d += 64) s_wc[wave][d] = 0;
    uint32_t key[IT], val[IT], rank[IT];
#pragma unroll
    for (int s = 0; s < IT; s++) {
      const int i = wbase + s * 64 + lane;
      if (i < hi) {
        key[s] = kin[row + i];
        val[s] = FIRST ? (uint32_t)i : vin[row + i];
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int s = 0; s < IT; s++) {
      const bool valid = wbase + s * 64 + lane < hi;
      const uint32_t d = valid ? (key[s] >> shift) & (kDepthR - 1) : 0u;
      rank[s] = wave_rank(s_mask[wave], s_wc[wave], d, valid, lane, lt);
    }
    __syncthreads();
    uint32_t c[D];
#pragma unroll
    for (int i = 0; i < D; i++) c[i] = 0u;
    if (tid < OWN) {
#pragma unroll
      for (int i = 0; i < D; i++) {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < NW; w++) {
          const uint32_t x = s_wc[w][tid * D + i];
          s_wc[w][tid * D + i] = (uint16_t)run;
          run += x;
        }
        c[i] = run;
      }
    }
    {
      uint32_t run = digit_scan(c);
      if (tid < OWN) {
#pragma unroll
        for (int i = 0; i < D; i++) {
          s_boff[tid * D + i] = run;
          run += c[i];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++)
      if (wbase + s * 64 + lane < hi) {
        const uint32_t d = (key[s] >> shift) & (kDepthR - 1);
        rank[s] += s_boff[d] + s_wc[wave][d];  // position in the ordered batch
        s_x[rank[s]] = key[s];
      }
    __syncthreads();
    uint32_t to[IT];  // where the batch's elements tid, tid + NT, ... go
#pragma unroll
    for (int s = 0; s < IT; s++) {
      const int j = s * NT + tid;
      if (j < nb) {
        const uint32_t k = s_x[j];
        const uint32_t d = (k >> shift) & (kDepthR - 1);
        to[s] = s_base[d] + ((uint32_t)j - s_boff[d]);  // below n for a consistent histogram
        if (write_keys && to[s] < (uint32_t)n) kout[row + to[s]] = k;
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++)
      if (wbase + s * 64 + lane < hi) s_x[rank[s]] = val[s];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < IT; s++) {
      const int j = s * NT + tid;
      if (j < nb && to[s] < (uint32_t)n) vout[row + to[s]] = s_x[j];
    }
    if (batch + kDepthBatch >= hi) break;
    __syncthreads();
    if (tid < OWN) {
#pragma unroll
      for (int i = 0; i < D; i++) s_base[tid * D + i] += c[i];
    }
    __syncthreads();
  }
}

// The fourth digit (bits 27 to 30) of the views that have depths beyond the low 27 bits (float
// depths from 13,107 on: distant Gaussians of an unbounded scene); the workgroups of other views return at
// once.  One launch: each of a view's workgroups counts the digits of the whole view by itself (a column of
// counters per thread), those before its own part first, and then places its part, 1,024 at a time.
// us of a whole render without / with far depths (one or nine in ten alike): a view of 200k 148 / 175, of 1M
// 347 / 467, 20 of 200k 825 / 870; 580, 2650 and 1280 with one workgroup per view.
constexpr int kFarThreads = 1024, kFarDigits = 16;
__global__ __launch_bounds__(kFarThreads) void k_depth_far(int n, int blocks, const uint32_t* __restrict__ keys,
                                                           const uint32_t* __restrict__ vin,
                                                           uint32_t* __restrict__ vout,
                                                           const uint32_t* __restrict__ far) {
  __shared__ uint32_t s_cnt[kFarDigits][kFarThreads];
  __shared__ uint32_t s_before[kFarDigits], s_base[kFarDigits], s_wc[kFarThreads / 64][kFarDigits];
  const int v = blockIdx.x / blocks, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (far[DASS_MAX_VIEWS + v] == 0) return;  // uniform over the workgroup
  const int64_t row = (int64_t)v * n;
  const int chunk = (n + blocks - 1) / blocks;
  const int lo = min((int)(blockIdx.x % blocks) * chunk, n), hi = min(lo + chunk, n);
  const auto digit = [&](uint32_t k) { return (k >> 27) & (kFarDigits - 1u); };
  const auto count = [&](int b, int e) {  // into the thread's own column
    constexpr int kAhead = 8;
    int i = b + tid;
    for (; i + (kAhead - 1) * kFarThreads < e; i += kAhead * kFarThreads) {
      uint32_t k[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; u++) k[u] = keys[row + i + u * kFarThreads];
#pragma unroll
      for (int u = 0; u < kAhead; u++) atomicAdd(&s_cnt[digit(k[u])][tid], 1u);
    }
    for (; i < e; i += kFarThreads) atomicAdd(&s_cnt[digit(keys[row + i])][tid], 1u);
  };
  static_assert(kFarThreads / 64 == kFarDigits, "a wave adds up a digit's columns");
  const auto total = [&] {  // of the wave's digit
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < kFarThreads; i += 64) x += s_cnt[wave][i + lane];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
  };
#pragma unroll
  for (int d = 0; d < kFarDigits; d++) s_cnt[d][tid] = 0u;
  count(0, lo);
  __syncthreads();
  const uint32_t before = total();
  if (lane == 0) s_before[wave] = before;
  __syncthreads();
  count(lo, n);
  __syncthreads();
  const uint32_t all = total();
  if (lane == 0) s_base[wave] = all;
  __syncthreads();
  if (tid == 0) {
    uint32_t run = 0;
    for (int d = 0; d < kFarDigits; d++) {
      const uint32_t x = s_base[d];
      s_base[d] = run + s_before[d];
      run += x;
    }
  }
  __syncthreads();
  const uint64_t lt = lanemask_lt();
  for (int b = lo; b < hi; b += kFarThreads) {
    const int i = b + tid;
    const bool valid = i < hi;
    const uint32_t d = valid ? digit(keys[row + i]) : 0u;
    const uint32_t val = valid ? vin[row + i] : 0u;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const uint64_t m = __ballot((d >> k) & 1);
      peers &= ((d >> k) & 1) ? m : ~m;
    }
    if (lane < kFarDigits) s_wc[wave][lane] = 0;
    wave_lds_sync();
    const uint32_t rw = __popcll(peers & lt);
    if (valid && rw == 0) s_wc[wave][d] = __popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t o = s_base[d] + rw;
      for (int w = 0; w < wave; w++) o += s_wc[w][d];
      vout[row + o] = val;
    }
    __syncthreads();
    if (tid < kFarDigits)
      for (int w = 0; w < kFarThreads / 64; w++) s_base[tid] += s_wc[w][tid];
    __syncthreads();
  }
}

// ---- scan of uint32 -> uint64 (exclusive), 3 phases ----------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;  // 4096

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint32_t* __restrict__ in, int64_t n,
                                                              uint64_t* __restrict__ sums) {
  __shared__ uint64_t s_w[4];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  uint64_t acc = 0;
  for (int i = threadIdx.x; i < kScanTile; i += kScanThreads) {
    const int64_t j = base + i;
    if (j < n) acc += in[j];
  }
  // wave reduce
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) sums[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

// exclusive scan of nb block sums in place (single workgroup of 1024), nb <= 1024 * 64
__global__ __launch_bounds__(1024) void k_scan_sums(uint64_t* __restrict__ sums, int nb) {
  __shared__ uint64_t s_w[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (nb + 1023) / 1024;
  const int b = tid * per, e = min(b + per, nb);
  uint64_t sum = 0;
  for (int i = b; i < e; i++) sum += sums[i];
  uint64_t inc = wave_incl_scan64(sum);
  if (lane == 63) s_w[wave] = inc;
  __syncthreads();
  uint64_t base = 0;
  for (int w = 0; w < wave; w++) base += s_w[w];
  uint64_t run = base + inc - sum;
  for (int i = b; i < e; i++) {
    uint64_t c = sums[i];
    sums[i] = run;
    run += c;
  }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_final(const uint32_t* __restrict__ in, int64_t n,
                                                             const uint64_t* __restrict__ sums,
                                                             uint64_t* __restrict__ out) {
  __shared__ uint64_t s_w[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)tid * kScanItems;  // blocked layout
  uint32_t x[kScanItems];
  uint64_t local = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; i++) {
    const int64_t j = base + i;
    x[i] = j < n ? in[j] : 0u;
    local += x[i];
  }
  uint64_t inc = wave_incl_scan64(local);
  if (lane == 63) s_w[wave] = inc;
  __syncthreads();
  uint64_t run = sums[blockIdx.x] + inc - local;
  for (int w = 0; w < wave; w++) run += s_w[w];
#pragma unroll
  for (int i = 0; i < kScanItems; i++) {
    const int64_t j = base + i;
    if (j < n) out[j] = run;
    run += x[i];
  }
  if (base <= n - 1 && n - 1 < base + kScanItems) out[n] = run;  // holder of the last element
}

__global__ void k_set_u64(uint64_t* p, uint64_t v) { *p = v; }

}  // namespace

int sort_blocks_for(int64_t max_count) {
  int64_t b = (max_count + 4 * kBatch - 1) / (4 * kBatch);
  const int64_t one = (max_count + kBatch - 1) / kBatch;
  if (b < 256) b = one < 256 ? one : 256;
  if (b < 1) b = 1;
  if (b > kMaxSortBlocks) b = kMaxSortBlocks;
  return (int)b;
}

int radix_sort_u32(uint32_t* keys[2], uint32_t* vals[2], const uint32_t* d_count, int64_t max_count, uint32_t* hist,
                   int blocks, hipStream_t st) {
  int cur = 0;
  if (max_count == 0) return cur;
  uint32_t* totals = hist + (int64_t)kRadix * kMaxSortBlocks;
  for (int shift = 0; shift < 32; shift += kRadixBits, cur ^= 1) {
    k_upsweep<<<blocks, kSortThreads, 0, st>>>(keys[cur], d_count, shift, blocks, hist);
    k_scan_rows<<<kRadix, kSortThreads, 0, st>>>(hist, blocks, totals);
    k_scatter<<<blocks, kSortThreads, 0, st>>>(keys[cur], vals[cur], keys[cur ^ 1], vals[cur ^ 1], d_count, shift, blocks,
                                               hist, totals);
  }
  return cur;
}

size_t depth_hist_elems(int max_views) { return (size_t)max_views * kDepthBlocks * kDepthR; }

template <int NT>
static void depth_passes(int n, int nv, int blocks, unsigned grid, uint32_t* const keys[2], uint32_t* const vals[2],
                         uint32_t* spare, uint32_t* hist, uint32_t* far, hipStream_t st) {
  k_depth_upsweep<<<grid, kSortThreads, 0, st>>>(n, nv, blocks, 0, keys[0], hist, far);
  k_depth_scatter<true, false, NT><<<grid, NT, 0, st>>>(n, nv, blocks, 0, keys[0], nullptr, keys[1], vals[1], hist, far,
                                                        spare);
  k_depth_upsweep<<<grid, kSortThreads, 0, st>>>(n, nv, blocks, 9, keys[1], hist, far);
  k_depth_scatter<false, false, NT><<<grid, NT, 0, st>>>(n, nv, blocks, 9, keys[1], vals[1], keys[0], vals[0], hist, far,
                                                         spare);
  k_depth_upsweep<<<grid, kSortThreads, 0, st>>>(n, nv, blocks, 18, keys[0], hist, far);
  k_depth_scatter<false, true, NT><<<grid, NT, 0, st>>>(n, nv, blocks, 18, keys[0], vals[0], keys[1], vals[1], hist, far,
                                                        spare);
}

void launch_depth_sort(int n, int nv, uint32_t* const keys[2], uint32_t* const vals[2], uint32_t* spare, uint32_t* hist,
                       uint32_t* far, hipStream_t st) {
  if (n <= 0) return;
  // a view in LDS as long as one workgroup's registers hold it: 16,384 Gaussians in 43 us, against
  // 47 (1 view) to 49 us (20) for the radix passes at 20,000; 12,000 in 32, 4,000 in 16 us
  if (n <= 2 * kDepthLdsThreads)
    k_depth_lds<2><<<nv, kDepthLdsThreads, 0, st>>>(n, keys[0], vals[1], far);
  else if (n <= 4 * kDepthLdsThreads)
    k_depth_lds<4><<<nv, kDepthLdsThreads, 0, st>>>(n, keys[0], vals[1], far);
  else if (n <= 8 * kDepthLdsThreads)
    k_depth_lds<8><<<nv, kDepthLdsThreads, 0, st>>>(n, keys[0], vals[1], far);
  else if (n <= 12 * kDepthLdsThreads)
    k_depth_lds<12><<<nv, kDepthLdsThreads, 0, st>>>(n, keys[0], vals[1], far);
  else if (n <= 16 * kDepthLdsThreads)
    k_depth_lds<16><<<nv, kDepthLdsThreads, 0, st>>>(n, keys[0], vals[1], far);
  else {
    const int blocks = std::min(kDepthBlocks, (n + kDepthBatch - 1) / kDepthBatch);
    const unsigned grid = (unsigned)((blocks * nv + kNumXcd - 1) / kNumXcd * kNumXcd);
    // blocks of 1,024 threads, four pairs each, while every block has a CU to itself: the ranks are a chain
    // per wave, sixteen pairs long with 256 threads.  us of the sort, 256 -> 1,024 threads: one view of
    // 200k 65 -> 51, four (196 blocks) 66 -> 54, of 1M (256) 155 -> 129; eight of 200k (392) 71, 80
    if (blocks * nv <= 256)
      depth_passes<1024>(n, nv, blocks, grid, keys, vals, spare, hist, far, st);
    else
      depth_passes<256>(n, nv, blocks, grid, keys, vals, spare, hist, far, st);
    // a workgroup per CU at most, so that without far depths the launch is over at once
    const int far_blocks = std::max(8, std::min(32, 256 / nv));
    k_depth_far<<<nv * far_blocks, kFarThreads, 0, st>>>(n, far_blocks, keys[1], spare, vals[1], far);
  }
}

size_t scan_tmp_elems(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile) + 1; }

void scan_u32_to_u64(const uint32_t* in, uint64_t* out, int64_t n, uint64_t* tmp, hipStream_t st) {
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  if (n == 0) {
    k_set_u64<<<1, 1, 0, st>>>(out, 0);
    return;
  }
  k_scan_reduce<<<(unsigned)nb, kScanThreads, 0, st>>>(in, n, tmp);
  k_scan_sums<<<1, 1024, 0, st>>>(tmp, (int)nb);
  k_scan_final<<<(unsigned)nb, kScanThreads, 0, st>>>(in, n, tmp, out);
}

}  // namespace dass
