// Tile binning: from the per-view depth order of the Gaussians and their tile rectangles to one
// list per tile, in depth order, without materialising or sorting (tile, Gaussian) keys.
//
// The tile lists are a stable counting sort of the Gaussians' keys by tile, and the keys of a
// Gaussian follow from its rectangle, so both passes over them walk the rectangles:
//   (1) count: a wave takes a run of consecutive depth positions (a chunk) of one view and counts
//       its keys per tile into a row of the histogram [view][chunk][tile];
//   (2) rows / tiles: an exclusive scan over the chunks of each tile, then over the tiles, which
//       gives every tile's range (and the key count, checked against the key budget);
//   (3) scatter: the wave walks its chunk again, 64 Gaussians (one per lane) at a time, and stores
//       each key's record index at its tile's next position.
// Every wave works alone (no workgroup barriers, no dependence between workgroups).  A key's rank
// among the 64 Gaussians comes from a 64-bit lane mask per tile: the bits below the lane's own.
//
// Bound: the record indices are written once (4 bytes per key), the rectangles read twice; the
// scatter waits on LDS and on its stores.  The keys-and-radix-sort form it replaces wrote 8 bytes per
// key, read them twice and wrote them again per 8- to 11-bit pass, then read them for the ranges:
// 1.5e7 keys of 20 views (64x32 tiles) 0.30 -> 0.17 ms, 2.2e7 keys of 8 mixed views (16x16 tiles)
// 0.43 -> 0.32 ms, 2e8 keys of wide Gaussians 2.56 -> 0.60 ms, 8e5 keys of one view 62 -> 35 us.
#include <algorithm>

#include "dass_internal.h"

namespace dass {
namespace {

// Tiles a wave counts or scatters at once; a view's tiles beyond this are taken window by window.
// The count's windows only have to fit its array.  The scatter is bound by latency, so by the waves
// per CU, also where small tiles give many windows and the rectangles are read once for each: whole
// renders with 256, 512 and 1,024 tiles, in us: 8 views of 200k Gaussians at 1920x1080 in 16x16 tiles (32
// windows of 256 each) 944, 1051, 1076; one at 3840x2160 (127) 473, 510, 511; one of 1M there 1619, 1652,
// 1668; 20 of 200k at 1352x1014 in 32x32 tiles (6) 1312, 1316, 1318.
constexpr int kWinTiles = 1024;
constexpr int kScatterTiles = 256;
// ((bx + 1) | 1)(by + 1) for bx by <= kWinTiles: at most bx by + bx + 2 by + 2
constexpr int kDiffCells = 3 * kWinTiles + 8;

__device__ __forceinline__ uint64_t lane_lt(int lane) { return lane == 0 ? 0ull : (~0ull >> (64 - lane)); }

// Orders the LDS accesses of one wave's lanes (its LDS instructions complete in order; this keeps
// the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int wave_max(int x) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) x = max(x, __shfl_xor(x, d, 64));
  return __builtin_amdgcn_readfirstlane(x);
}
__device__ __forceinline__ int wave_min(int x) { return -wave_max(-x); }

// Inclusive scans over the lanes: steps of 1, 2, 4, 8 within rows of 16, then rows 0 and 2 into 1
// and 3, then the lower half into the upper (DPP; a lane without a source takes 0).
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp0(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ int wave_scan_add(int x) {
  x += dpp0<0x111, 0xF>(x);
  x += dpp0<0x112, 0xF>(x);
  x += dpp0<0x114, 0xF>(x);
  x += dpp0<0x118, 0xF>(x);
  x += dpp0<0x142, 0xA>(x);
  x += dpp0<0x143, 0xC>(x);
  return x;
}
__device__ __forceinline__ int wave_scan_max(int x) {  // x >= 0
  x = max(x, dpp0<0x111, 0xF>(x));
  x = max(x, dpp0<0x112, 0xF>(x));
  x = max(x, dpp0<0x114, 0xF>(x));
  x = max(x, dpp0<0x118, 0xF>(x));
  x = max(x, dpp0<0x142, 0xA>(x));
  x = max(x, dpp0<0x143, 0xC>(x));
  return x;
}

// Window w of a view's tile grid, in tiles.
struct Window {
  int x0, y0, bx, by;  // bx by <= the window's tile limit; empty (bx = 0) past the view's last window
};
__device__ __forceinline__ Window window_of(int TX, int TY, int w, int most) {
  const int wx = min(TX, most), rows = most / wx;  // window size limits
  const int nx = (TX + wx - 1) / wx, ny = (TY + rows - 1) / rows;
  const int wy = (TY + ny - 1) / ny;  // rows spread evenly over the windows
  Window o{0, 0, 0, 0};
  if (w >= nx * ny) return o;
  o.x0 = (w % nx) * wx;
  o.y0 = (w / nx) * wy;
  o.bx = min(wx, TX - o.x0);
  o.by = min(wy, TY - o.y0);
  if (o.by <= 0) o.bx = 0;
  return o;
}

// A Gaussian's rectangle clipped to the window, relative to it.
struct Clip {
  int x0, y0, w, h;
};
__device__ __forceinline__ Clip clip_rect(uint2 r, const Window& W) {
  Clip c;
  const int x0 = max((int)(r.x & 0xFFFFu) - W.x0, 0), y0 = max((int)(r.x >> 16) - W.y0, 0);
  const int x1 = min((int)(r.y & 0xFFFFu) - W.x0, W.bx), y1 = min((int)(r.y >> 16) - W.y0, W.by);
  const bool any = x1 > x0 && y1 > y0;
  c.x0 = x0;
  c.y0 = y0;
  c.w = any ? x1 - x0 : 0;
  c.h = any ? y1 - y0 : 0;
  return c;
}

// Which (view, window, chunk) a workgroup takes: chunks innermost, and each XCD a contiguous part
// of that order (workgroups are dealt to the XCDs round-robin), so the lists of a window are
// written through one L2, where the short runs of neighbouring chunks merge into whole lines.
struct Piece {
  int v, win, chunk;
};
__device__ __forceinline__ bool piece_of(int chunks, int nv, int wins, Piece& o) {
  const int64_t total = (int64_t)chunks * nv * wins, per = (total + kNumXcd - 1) / kNumXcd;
  const int64_t i = (int64_t)(blockIdx.x % kNumXcd) * per + blockIdx.x / kNumXcd;
  if (i >= total || (int64_t)(blockIdx.x / kNumXcd) >= per) return false;
  o.chunk = (int)(i % chunks);
  o.win = (int)(i / chunks % wins);
  o.v = (int)(i / chunks / wins);
  return true;
}

// Keys per tile of a chunk: every rectangle adds its four corners to a two-dimensional difference
// array (four LDS atomics whatever its area), summed along both axes at the end.  Window 0 also
// leaves the rectangles in depth order for the scatter.
__global__ __launch_bounds__(64) void k_bin_count(int n, int nv, int wins, int chunk, int chunks, BinViews bv,
                                                  const uint32_t* __restrict__ gid, const uint2* __restrict__ rect_u,
                                                  uint2* __restrict__ rect_s, uint32_t* __restrict__ hist) {
  __shared__ int s_diff[kDiffCells];
  Piece pc;
  if (!piece_of(chunks, nv, wins, pc)) return;
  const int v = pc.v, lane = threadIdx.x;
  const int TX = bv.TX[v], TY = bv.TY[v];
  const Window W = window_of(TX, TY, pc.win, kWinTiles);
  if (W.bx == 0) return;
  const int dw = (W.bx + 1) | 1;  // odd: a column's rows fall in different banks
  for (int t = lane; t < dw * (W.by + 1); t += 64) s_diff[t] = 0;
  wave_sync();
  const int p0 = pc.chunk * chunk, p1 = min(p0 + chunk, n);
  const int64_t row = (int64_t)v * n;
  // indices two steps ahead, rectangles one step ahead
  uint32_t g1 = p0 + lane < p1 ? gid[row + p0 + lane] : 0u;
  uint2 r1 = rect_u[row + g1];
  g1 = p0 + 64 + lane < p1 ? gid[row + p0 + 64 + lane] : 0u;
  for (int b = p0; b < p1; b += 64) {
    const int p = b + lane;
    const uint2 r = p < p1 ? r1 : make_uint2(0u, 0u);
    r1 = rect_u[row + g1];
    g1 = p + 128 < p1 ? gid[row + p + 128] : 0u;
    if (pc.win == 0 && p < p1) rect_s[row + p] = r;
    const Clip c = clip_rect(r, W);
    if (c.w > 0) {
      const int a = c.y0 * dw + c.x0;
      atomicAdd(&s_diff[a], 1);
      atomicAdd(&s_diff[a + c.w], -1);
      atomicAdd(&s_diff[a + c.h * dw], -1);
      atomicAdd(&s_diff[a + c.h * dw + c.w], 1);
    }
  }
  wave_sync();
  for (int y = lane; y < W.by; y += 64) {
    int run = 0;
    for (int x = 0; x < W.bx; x++) {
      run += s_diff[y * dw + x];
      s_diff[y * dw + x] = run;
    }
  }
  wave_sync();
  uint32_t* __restrict__ out = hist + (int64_t)bv.tile_base[v] * chunks + (int64_t)pc.chunk * TX * TY;
  for (int x = lane; x < W.bx; x += 64) {
    int run = 0;
    for (int y = 0; y < W.by; y++) {
      run += s_diff[y * dw + x];
      out[(W.y0 + y) * TX + W.x0 + x] = (uint32_t)run;
    }
  }
}

// Exclusive scan over the chunks of every tile, in place; the tile's total to tile_tot.  A
// workgroup takes 16 tiles of one view (blockIdx.y) and splits the chunks over 64 groups of 16
// threads: few dependent loads per thread, 64-byte lines per group.
constexpr int kRowTiles = 16, kRowGroups = 64;
__global__ __launch_bounds__(kRowTiles * kRowGroups) void k_bin_rows(int chunks, BinViews bv,
                                                                     uint32_t* __restrict__ hist,
                                                                     uint32_t* __restrict__ tile_tot) {
  __shared__ uint32_t s_sum[kRowGroups][kRowTiles];
  const int v = blockIdx.y, tl = threadIdx.x % kRowTiles, grp = threadIdx.x / kRowTiles;
  const int nt = bv.TX[v] * bv.TY[v];
  if (blockIdx.x * kRowTiles >= nt) return;  // uniform over the workgroup
  const int t = blockIdx.x * kRowTiles + tl;
  const int per = (chunks + kRowGroups - 1) / kRowGroups;
  const int c0 = min(grp * per, chunks), c1 = t < nt ? min(c0 + per, chunks) : c0;
  uint32_t* __restrict__ col = hist + (int64_t)bv.tile_base[v] * chunks + t;
  constexpr int kAhead = 8;  // loads in flight
  uint32_t sum = 0;
  for (int c = c0; c < c1; c += kAhead) {
    uint32_t x[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; u++) x[u] = c + u < c1 ? col[(int64_t)(c + u) * nt] : 0u;
#pragma unroll
    for (int u = 0; u < kAhead; u++) sum += x[u];
  }
  s_sum[grp][tl] = sum;
  __syncthreads();
  uint32_t run = 0;
  for (int w = 0; w < grp; w++) run += s_sum[w][tl];
  if (grp == kRowGroups - 1 && t < nt) tile_tot[bv.tile_base[v] + t] = run + sum;
  for (int c = c0; c < c1; c += kAhead) {
    uint32_t x[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; u++) x[u] = c + u < c1 ? col[(int64_t)(c + u) * nt] : 0u;
#pragma unroll
    for (int u = 0; u < kAhead; u++) {
      if (c + u < c1) col[(int64_t)(c + u) * nt] = run;
      run += x[u];
    }
  }
}

// Ranges of all tiles: exclusive scan of the totals, clamped to the key budget, whose overflow is
// recorded.  A workgroup takes 4,096 tiles and sums the totals before them by itself (a few
// coalesced loads per thread), so the workgroups do not wait for each other.  tile_tot is padded
// to a multiple of 4 tiles.
constexpr int kTilesPer = 4;
__global__ __launch_bounds__(1024) void k_bin_tiles(int tiles, const uint32_t* __restrict__ tile_tot, int64_t cap,
                                                    uint2* __restrict__ ranges, uint64_t* __restrict__ n_keys,
                                                    uint32_t* __restrict__ err) {
  __shared__ uint64_t s_before[16], s_w[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int first = blockIdx.x * 1024 * kTilesPer, t0 = first + tid * kTilesPer;
  const uint4* __restrict__ tot4 = reinterpret_cast<const uint4*>(tile_tot);
  uint4 own = make_uint4(0u, 0u, 0u, 0u);
  if (t0 < tiles) own = tot4[t0 / 4];
  uint64_t before = 0;
  for (int i = tid; i < first / 4; i += 1024) {
    const uint4 q = tot4[i];
    before += (uint64_t)q.x + q.y + q.z + q.w;
  }
  const uint32_t x[kTilesPer] = {own.x, t0 + 1 < tiles ? own.y : 0u, t0 + 2 < tiles ? own.z : 0u,
                                 t0 + 3 < tiles ? own.w : 0u};
  const uint64_t sum = (uint64_t)x[0] + x[1] + x[2] + x[3];
  uint64_t inc = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(inc, d, 64);
    before += __shfl_xor(before, d, 64);
    if (lane >= d) inc += y;
  }
  if (lane == 63) {
    s_before[wave] = before;
    s_w[wave] = inc;
  }
  __syncthreads();
  uint64_t run = inc - sum;
#pragma unroll
  for (int w = 0; w < 16; w++) {
    run += s_before[w];
    if (w < wave) run += s_w[w];
  }
#pragma unroll
  for (int i = 0; i < kTilesPer; i++) {
    const uint64_t end = run + x[i];
    if (t0 + i < tiles)
      ranges[t0 + i] = make_uint2((uint32_t)(run < (uint64_t)cap ? run : (uint64_t)cap),
                                  (uint32_t)(end < (uint64_t)cap ? end : (uint64_t)cap));
    run = end;
  }
  if (t0 < tiles && t0 + kTilesPer >= tiles) {  // the thread with the last tile
    *n_keys = run;
    if (run > (uint64_t)cap) atomicOr(err, kErrKeyOverflow);
  }
}

// The keys of 64 rectangles (area, start: the lane's keys and those before them, total: of all).
__device__ __forceinline__ void place_by_key(const Clip& c, int area, int start, int total, uint32_t val, const Window& W,
                                             int lane, uint64_t bit, uint64_t lt, uint32_t cap, int* s_own,
                                             uint64_t* s_mask, uint32_t* s_pos, uint32_t* __restrict__ vals) {
  const int where = (c.y0 * W.bx + c.x0) | (c.w << 16);
  int carry = 0;  // 1 + the lane that owns the last key of the keys before
  for (int k0 = 0; k0 < total; k0 += 64) {
    // 1 + lane at the first key of every Gaussian that starts among these 64, then a max-scan
    const int at = start - k0;
    const bool here = area > 0 && at >= 0 && at < 64;
    s_own[lane] = 0;
    wave_sync();
    if (here) s_own[at] = lane + 1;
    wave_sync();
    int own = s_own[lane];
    own = max(wave_scan_max(own), carry);
    carry = __builtin_amdgcn_readlane(own, 63);
    const int k = k0 + lane, src = own - 1;
    const int wh = __shfl(where, src, 64);
    const int i = k - __shfl(start, src, 64);
    const uint32_t vv = (uint32_t)__shfl((int)val, src, 64);
    const bool live = k < total;
    const int w = wh >> 16;
    // i / w by a float reciprocal, corrected to the exact quotient (i < 2^20)
    int q = (int)((float)i * __builtin_amdgcn_rcpf((float)w));
    int x = i - q * w;
    if (x < 0) {
      q--;
      x += w;
    } else if (x >= w) {
      q++;
      x -= w;
    }
    const int t = live ? (wh & 0xFFFF) + q * W.bx + x : 0;
    if (live) atomicOr(reinterpret_cast<unsigned long long*>(&s_mask[t]), (unsigned long long)bit);
    wave_sync();
    const uint64_t m = s_mask[t];
    const uint32_t pos = s_pos[t];
    const uint32_t o = pos + (uint32_t)__popcll(m & lt);
    if (live && o < cap) vals[o] = vv;
    wave_sync();
    if (live && (m >> lane) == 1ull) {  // the tile's last key among the 64
      s_pos[t] = min(pos + (uint32_t)__popcll(m), cap);
      s_mask[t] = 0ull;
    }
    wave_sync();
  }
}

// A (view, window, chunk) per wave, 64 Gaussians at a time, either
//   by key: the group's keys spread evenly over the lanes, 64 at a time in Gaussian order (lane l
//     finds the Gaussian of its key by a max-scan over the lanes where a Gaussian's keys start); a
//     lane mask per tile in LDS ranks the keys that meet in a tile;
//   by tile (more than kDenseKeys keys per tile of the group's common box), with the next seven groups:
//     the wave walks the box, its lanes holding eight rectangles each, collects a tile's run in LDS and
//     stores it in one piece; a row's positions stay in registers.  By key, 64 neighbouring keys of a
//     wide Gaussian are stored to 64 lines, and a store of the few lanes of one group costs what a
//     full one does: 2e8 keys of Gaussians over about 50 tiles each took 2.34 ms by key alone, 0.77 ms
//     by tile with one group at a time, 0.51 so.
//     At 2 keys the call gains 8 us, but groups just past the line that are followed by sparse ones cost
//     20 views of 200k small Gaussians 154 us instead of 98.
constexpr int kDenseKeys = 3;
constexpr int kGroups = 8;  // of 64 Gaussians
__global__ __launch_bounds__(64) void k_bin_scatter(int n, int nv, int wins, int chunk, int chunks,
                                                    BinViews bv, const uint32_t* __restrict__ gid,
                                                    const uint2* __restrict__ rect_s, const uint32_t* __restrict__ hist,
                                                    const uint2* __restrict__ ranges, const uint64_t* __restrict__ n_keys,
                                                    uint32_t* __restrict__ vals) {
  __shared__ uint64_t s_mask[kScatterTiles];
  __shared__ int s_own[64];
  __shared__ uint32_t s_run[64 * kGroups];   // a tile's run
  __shared__ uint32_t s_pos[kScatterTiles];  // next position of each tile's list (the key budget at most)
  Piece pc;
  if (!piece_of(chunks, nv, wins, pc)) return;
  const int v = pc.v, lane = threadIdx.x;
  const int TX = bv.TX[v], TY = bv.TY[v];
  const Window W = window_of(TX, TY, pc.win, kScatterTiles);
  if (W.bx == 0) return;
  const uint32_t cap = bv.cap;
  const bool fits = *n_keys <= (uint64_t)cap;
  {
    const uint32_t* __restrict__ h = hist + (int64_t)bv.tile_base[v] * chunks + (int64_t)pc.chunk * TX * TY;
    const uint2* __restrict__ rg = ranges + bv.tile_base[v];
    for (int y = 0; y < W.by; y++)
      for (int x = lane; x < W.bx; x += 64) {
        const int g = (W.y0 + y) * TX + W.x0 + x;
        const uint32_t first = rg[g].x, before = h[g];
        s_mask[y * W.bx + x] = 0ull;
        s_pos[y * W.bx + x] = before < cap - first ? first + before : cap;  // past the key budget: nothing is stored
      }
  }
  wave_sync();
  const uint64_t lt = lane_lt(lane), bit = 1ull << lane;
  const int p0 = pc.chunk * chunk, p1 = min(p0 + chunk, n);
  const int64_t row = (int64_t)v * n;
  uint2 r_next = make_uint2(0u, 0u);
  uint32_t g_next = 0;
  if (p0 + lane < p1) {
    r_next = rect_s[row + p0 + lane];
    g_next = gid[row + p0 + lane];
  }
  for (int b = p0; b < p1; b += 64) {
    const uint2 r = b + lane < p1 ? r_next : make_uint2(0u, 0u);
    const uint32_t val = (uint32_t)row + g_next;
    if (b + 64 + lane < p1) {  // the next 64 while these are placed
      r_next = rect_s[row + b + 64 + lane];
      g_next = gid[row + b + 64 + lane];
    }
    const Clip c = clip_rect(r, W);
    const int area = c.w * c.h;
    const int incl = wave_scan_add(area), start = incl - area;
    const int total = __builtin_amdgcn_readlane(incl, 63);
    if (total == 0) continue;
    if (total > 4 * 64 && fits) {
      int x0 = area ? c.x0 : kScatterTiles, x1 = area ? c.x0 + c.w : 0;
      int y0 = area ? c.y0 : kScatterTiles, y1 = area ? c.y0 + c.h : 0;
      if (total > kDenseKeys * (wave_max(x1) - wave_min(x0)) * (wave_max(y1) - wave_min(y0))) {
        // these 64 and the next 64 (kGroups - 1), whatever they are
        Clip cs[kGroups];
        uint32_t vs[kGroups];
        cs[0] = c;
        vs[0] = val;
#pragma unroll
        for (int i = 1; i < kGroups; i++) {
          const int e = b + 64 * i + lane;
          cs[i] = clip_rect(e < p1 ? rect_s[row + e] : make_uint2(0u, 0u), W);
          vs[i] = e < p1 ? (uint32_t)row + gid[row + e] : 0u;
          if (cs[i].w > 0) {
            x0 = min(x0, cs[i].x0);
            x1 = max(x1, cs[i].x0 + cs[i].w);
            y0 = min(y0, cs[i].y0);
            y1 = max(y1, cs[i].y0 + cs[i].h);
          }
        }
        x0 = wave_min(x0);
        x1 = wave_max(x1);
        y0 = wave_min(y0);
        y1 = wave_max(y1);
        for (int y = y0; y < y1; y++) {
          uint32_t width[kGroups];  // of the lane's rectangles in this row
#pragma unroll
          for (int i = 0; i < kGroups; i++) {
            width[i] = (uint32_t)(y - cs[i].y0) < (uint32_t)cs[i].h ? (uint32_t)cs[i].w : 0u;
            __asm__ volatile("" : "+v"(width[i]));  // one compare per tile below, not two
          }
          for (int xb = x0; xb < x1; xb += 64) {
            const int nx = min(64, x1 - xb);
            uint32_t* prow = &s_pos[y * W.bx + xb];
            int posv = lane < nx ? (int)prow[lane] : 0;  // lane i: the position of tile xb + i
            for (int x = 0; x < nx; x++) {
              int cnt = 0;
#pragma unroll
              for (int i = 0; i < kGroups; i++) {
                const bool in = (uint32_t)(xb + x - cs[i].x0) < width[i];
                const uint64_t m = __ballot(in);
                if (m != 0) {
                  if (in)
                    s_run[__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)cnt))] = vs[i];
                  cnt += (int)__popcll(m);
                }
              }
              if (cnt == 0) continue;
              wave_sync();
              const int pos = __builtin_amdgcn_readlane(posv, x);
              for (int k = lane; k < cnt; k += 64) vals[(uint32_t)pos + (uint32_t)k] = s_run[k];
              wave_sync();
              if (lane == x) posv = pos + cnt;
            }
            if (lane < nx) prow[lane] = (uint32_t)posv;
          }
        }
        wave_sync();
        b += 64 * (kGroups - 1);
        if (b + 64 + lane < p1) {
          r_next = rect_s[row + b + 64 + lane];
          g_next = gid[row + b + 64 + lane];
        }
        continue;
      }
    }
    place_by_key(c, area, start, total, val, W, lane, bit, lt, cap, s_own, s_mask, s_pos, vals);
  }
}

int windows_of(int TX, int TY, int most) {
  const int wx = TX < most ? TX : most, rows = most / wx;
  return ((TX + wx - 1) / wx) * ((TY + rows - 1) / rows);
}

}  // namespace

// 128 chunks per tile, within 1 GB as far as one chunk is (contexts for more than 2M tiles have fewer per
// tile), and up to 16 MB more, as far as chunks of 64 Gaussians need it.
int64_t bin_hist_elems(int64_t max_tiles, int64_t max_gaussians) {
  return std::max(max_tiles, std::min(128 * max_tiles, int64_t(1) << 28)) +
         std::min(int64_t(1) << 22, max_tiles * (max_gaussians / 64 + 1));
}

void launch_binning(int n, int nv, const CamsK& cams, int64_t total_tiles, Workspace& ws, hipStream_t st) {
  if (total_tiles == 0) return;
  uint64_t* n_keys = reinterpret_cast<uint64_t*>(ws.counters + 4);
  BinViews bv{};
  bv.cap = (uint32_t)ws.cap_keys;
  int nt_max = 1, wins = 1, wins_s = 1;
  for (int v = 0; v < nv; v++) {
    const int TX = cams.c[v].TX, TY = cams.c[v].TY;
    bv.TX[v] = TX;
    bv.TY[v] = TY;
    bv.tile_base[v] = cams.c[v].tile_base;
    nt_max = std::max(nt_max, TX * TY);
    wins = std::max(wins, windows_of(TX, TY, kWinTiles));
    wins_s = std::max(wins_s, windows_of(TX, TY, kScatterTiles));
  }
  // Gaussians per chunk: about 2,048 chunks over the call, at most 512 Gaussians each, and a
  // histogram (tiles x chunks) within its buffer.  More chunks balance the scatter but lengthen the
  // row scan: one view of 200k Gaussians takes 35 us in all with 1,563 chunks and 47 with 3,125;
  // 20 views 0.166 ms with chunks of 512, 0.183 with 256, 0.23 with 1,024.  And no more than about 64
  // counts per Gaussian where it has many tiles: 32 views of 3840x2160 in 16x16 tiles with 2k Gaussians took
  // 2.28 ms in chunks of 64, 1,000 counts each (2.09 with sorted keys), 2.13 in chunks of 512; 20k 3.70,
  // 3.50; one view with 20k 197 us, 181.
  int64_t chunk = ((int64_t)nv * n / 2048 + 63) / 64 * 64;
  chunk = std::max(chunk, (total_tiles / nv / 64 + 63) / 64 * 64);
  chunk = std::min<int64_t>(std::max<int64_t>(chunk, 64), 512);
  const int64_t max_chunks = ws.cap_bin / total_tiles;  // >= 1
  chunk = std::max(chunk, ((n + max_chunks - 1) / max_chunks + 63) / 64 * 64);
  const int chunks = (int)((n + chunk - 1) / chunk);
  const auto grid = [&](int w) { return (unsigned)(((int64_t)chunks * nv * w + kNumXcd - 1) / kNumXcd * kNumXcd); };
  if (chunks > 0)
    k_bin_count<<<grid(wins), 64, 0, st>>>(n, nv, wins, (int)chunk, chunks, bv, ws.gid_s, ws.rect_u, ws.rect_s,
                                           ws.bin_hist);
  k_bin_rows<<<dim3((nt_max + kRowTiles - 1) / kRowTiles, nv), kRowTiles * kRowGroups, 0, st>>>(chunks, bv, ws.bin_hist,
                                                                                             ws.tile_tot);
  k_bin_tiles<<<(unsigned)((total_tiles + 4095) / 4096), 1024, 0, st>>>((int)total_tiles, ws.tile_tot, ws.cap_keys, ws.ranges, n_keys, ws.err);
  if (chunks > 0)
    k_bin_scatter<<<grid(wins_s), 64, 0, st>>>(n, nv, wins_s, (int)chunk, chunks, bv, ws.gid_s, ws.rect_s,
                                               ws.bin_hist, ws.ranges, n_keys, ws.vals);
}

}  // namespace dass
