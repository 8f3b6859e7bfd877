// D-SSIM term of the fidelity loss, Eq. (3): L = (1/V) sum_v [(1 - lambda) L1_v + lambda (1 -
// SSIM_v)], with SSIM_v the mean over the three channels and all pixels of the SSIM map (11x11
// Gaussian window, sigma 1.5, zero padding, C1 = 0.01^2, C2 = 0.03^2 for images in [0, 1]).
//
// Large calls take one pass.  A wave takes a strip of one channel of one view, kCols (128) columns of which the
// inner 108 are output, two neighbouring columns per lane, and marches down the rows of its
// segment.  Per row it
//   - writes the row's pixels to LDS, takes the horizontal window sums of t, t^2, d and d^2 (t = x + y,
//     d = y - x: all the SSIM map needs) and adds them to the eleven output rows they reach, kept as
//     partial sums in registers (a shift per row that costs nothing: each multiply-add writes its
//     neighbour's register);
//   - the row five above is then complete: its SSIM value and three derivative maps go through a second LDS
//     row (its window scaled by dL/dSSIM) and a second set of partial sums in the same way (the window is
//     symmetric, so the adjoint of a window sum is the same sum), which completes dL/dx ten rows above,
//     to which the L1 term is added.
// The waves share nothing, so there are no barriers, and the maps never leave the chip.
//
// Differences that cancel are avoided, so that no range of values loses digits (dark images and a black
// background that both images share least of all, whose gradient is exactly 0):
//   - with V = var(d), D = (var(t) + V) / 2 + C2 the structure's denominator and e = V / D, the structure
//     is 1 - e and the luminance 1 - l, l = mu_d^2 / C: both errors are small where the images are alike;
//   - with K = (1 - l) / D, the gradient is 2 W*[(1 - e) (mu_d + mu_x l) / C + K ((d - mu_d) + e (x - mu_x))],
//     d and x at the pixel, the rest at the window's centre.  The first form's sum of W*P1, 2 x W*P2 and y W*P3
//     is the same with terms of the size of x K where these are of the size of d K;
//   - t enters var(t) less a shift that every lane takes from the pixels themselves: every kAhead rows
//     the horizontal mean of its newest row, the partial sums moved to it.
//
// Bound: vector ALU, about 470 instructions per row and lane (two pixels) at two waves per SIMD (the
// 140 partial sums); the halo costs a quarter of the work.  20 views at 1352x1014: 1.30 ms in the two
// passes (whose maps moved 2.2 GB) -> 0.775 ms, the relative error against 64 bits 8.6e-6 -> 3.5e-7.  (0.76 ms
// and 1.3e-6 with x, y less a fixed 0.5 in the first form; but then the gradient of a dark image, [0, 0.02],
// was off by 1.5e-4 of the pixel's share where the two passes are by 2.8e-6, now 1.5e-7, and that of a
// shared black background by 1.2e-4 where it is 0.)
#include <algorithm>

#include "dass_internal.h"

namespace dass {
namespace {

constexpr int kR = 5;            // window radius
constexpr int kTaps = 2 * kR + 1;
constexpr int kLanes = 64;
constexpr int kCols = 2 * kLanes;           // columns a wave reads
constexpr int kOut = kCols - 4 * kR;        // columns it writes (108)
constexpr int kRowW = kCols + 2 * kR;       // an LDS row: the columns and what the outer lanes read beyond them
// The shift of t stays within this (t lies in [0, 2]), and where it is no number.
constexpr float kMaxShift = 4.f;
constexpr int kBehind = 2 * kR + 1;         // rows between the one read and the one that completes
constexpr int kRing = kBehind + 1;
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

// Orders the LDS accesses of one wave's lanes (its LDS instructions complete in order; this keeps
// the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1 / x: the hardware reciprocal and one Newton step (about one unit in the last place).
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, r, 1.f), r, r);
}

// Window sums of a new row h (per column) into the eleven partial rows, the oldest first; returns
// the oldest, which h completes.
// (Written as three-address multiply-adds: left to itself the compiler takes the two-address form
// and a register move for each.)
__device__ __forceinline__ float fma3(float w, float h, float c) {
  float o;
  __asm__("v_fma_f32 %0, %1, %2, %3" : "=v"(o) : "s"(w), "v"(h), "v"(c));
  return o;
}
__device__ __forceinline__ float push(float (&acc)[kTaps - 1], const float* w, float h) {
  const float done = fma3(w[kTaps - 1], h, acc[0]);
#pragma unroll
  for (int i = 0; i < kTaps - 2; i++) acc[i] = fma3(w[kTaps - 2 - i], h, acc[i + 1]);
  acc[kTaps - 2] = w[0] * h;
  return done;
}

__global__ __launch_bounds__(kLanes, 2) void k_ssim(SsimArgs a, int per, float* __restrict__ loss_slots) {
  // the pixels (t, d) of the last twelve rows and a row's derivative maps; a lane's window starts on an
  // even column, so it is read in aligned pairs
  __shared__ __align__(16) float2 s_td[kRing][kRowW];
  __shared__ __align__(16) float s_p[3][kRowW];
  const int lane = threadIdx.x;
  const int64_t wave = (int64_t)(blockIdx.x % kNumXcd) * per + blockIdx.x / kNumXcd;
  const int64_t first = wave * a.rows, end = min(first + a.rows, a.total_rows);
  // the margins that only the outermost lanes read: their sums are not used, but must be numbers
  if (lane < kR) {
#pragma unroll
    for (int i = 0; i < kRing; i++) s_td[i][lane] = s_td[i][kRowW - 1 - lane] = make_float2(0.f, 0.f);
#pragma unroll
    for (int m = 0; m < 3; m++) s_p[m][lane] = s_p[m][kRowW - 1 - lane] = 0.f;
  }
  float part = 0.f;  // this wave's share of the loss
  int vi = 0;
  for (int64_t at = first; at < end;) {
  while (vi + 1 < a.nv && at >= a.v[vi + 1].row_begin) vi++;
  const SsimView& V = a.v[vi];
  const int W = V.W, H = V.H;
  // rows innermost, then strips, then channels
  const int64_t t = at - V.row_begin;
  const int y_lo = (int)(t % H), y_hi = (int)min((int64_t)H, y_lo + (end - at));
  const int strip = (int)(t / H) % V.strips, c = (int)(t / H) / V.strips;
  at += y_hi - y_lo;
  const int64_t hw = (int64_t)W * H;
  const int x_lo = (int)((int64_t)W * strip / V.strips), x_hi = (int)((int64_t)W * (strip + 1) / V.strips);
  const float* __restrict__ X = V.render + c * hw;
  const float* __restrict__ Y = V.target + c * hw;
  float w[kTaps];
#pragma unroll
  for (int i = 0; i < kTaps; i++) w[i] = a.w[i];
  const float gS = a.gS[vi], sl1 = a.l1_scale[vi];
  float wg[kTaps];  // the window scaled by 2 dL/dSSIM, for the derivative maps
#pragma unroll
  for (int i = 0; i < kTaps; i++) wg[i] = 2.f * gS * w[i];
  const int x0 = x_lo - 2 * kR + 2 * lane;  // this lane's columns x0, x0 + 1
  int xc[2];            // the columns kept inside the image, for the loads
  bool in[2], owns[2];  // column inside the image; written by this wave
#pragma unroll
  for (int j = 0; j < 2; j++) {
    in[j] = x0 + j >= 0 && x0 + j < W;
    xc[j] = min(max(x0 + j, 0), W - 1);
    owns[j] = x0 + j >= x_lo && x0 + j < x_hi;
  }
  // partial sums: moments (t and t^2 less the shift, d, d^2), derivative maps
  float am[4][2][kTaps - 1], ap[3][2][kTaps - 1];
#pragma unroll
  for (int i = 0; i < kTaps - 1; i++) {
#pragma unroll
    for (int j = 0; j < 2; j++) {
#pragma unroll
      for (int m = 0; m < 4; m++) am[m][j][i] = 0.f;
#pragma unroll
      for (int m = 0; m < 3; m++) ap[m][j][i] = 0.f;
    }
  }
  float ssum = 0.f, l1sum = 0.f;
  // the pixels of row r as they lie in memory (any pixel where the row or column is outside)
  auto fetch = [&](int r, float* px, float* py) {
    const int64_t p = (int64_t)min(max(r, 0), H - 1) * W;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      px[j] = X[p + xc[j]];
      py[j] = Y[p + xc[j]];
    }
  };
  // In step r the moments' row is r and the derivatives' row r - 6 (formed in the step before from the
  // moments of rows up to r - 1), so both sets of horizontal sums are independent; the row that
  // completes is r - 11.  Pixels are loaded kAhead steps ahead into registers of their own (the steps
  // are unrolled kAhead times): the waves are few (two per SIMD, for their partial sums), so the
  // loads' latency has to be hidden by the wave itself.
  constexpr int kAhead = 4;
  float qx[kAhead][2], qy[kAhead][2], P[3][2];
  float shift = 0.f, mean = 0.f;  // of the lane's two columns; the newest row's horizontal mean less the shift
#pragma unroll
  for (int i = 0; i < kAhead; i++) fetch(y_lo - 2 * kR + i, qx[i], qy[i]);
#pragma unroll
  for (int m = 0; m < 3; m++) P[m][0] = P[m][1] = 0.f;
  // the last channel's waves also form the error map, from all channels' pixels a step ahead
  const bool errs = c == 2 && V.err != nullptr;
  float en[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  int slot = 0;  // of row r in the ring; row r - 11 is in the next one
  const int r_end = y_hi + kBehind;
  for (int r0 = y_lo - 2 * kR; r0 < r_end; r0 += kAhead) {
    {  // the shift to the newest row's mean.  (Rows that still entered with a shift from beyond an edge
       // weigh at most 0.16 together in the first windows that lie on this side of it altogether.)
      const float to = shift + mean, by = fabsf(to) <= kMaxShift ? to - shift : 0.f;
      shift += by;
#pragma unroll
      for (int i = 0; i < kTaps - 1; i++) {
        const float wi = a.w_before[kTaps - 1 - i];  // the weights this partial sum has taken
#pragma unroll
        for (int j = 0; j < 2; j++) {
          const float was = am[0][j][i];
          am[0][j][i] = fmaf(-by, wi, was);
          am[1][j][i] = fmaf(-by, was + am[0][j][i], am[1][j][i]);
        }
      }
    }
#pragma unroll
  for (int u0 = 0; u0 < kAhead; u0++) {
    const int r = r0 + u0;
    if (r >= r_end) break;  // uniform
    float2* __restrict__ row = s_td[slot];
    slot = slot + 1 == kRing ? 0 : slot + 1;
    const bool in_r = r >= 0 && r < H;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const float x = in[j] && in_r ? qx[u0][j] : 0.f, y = in[j] && in_r ? qy[u0][j] : 0.f;
      row[kR + 2 * lane + j] = make_float2(x + y, y - x);
    }
#pragma unroll
    for (int m = 0; m < 3; m++) {
      s_p[m][kR + 2 * lane] = P[m][0];
      s_p[m][kR + 1 + 2 * lane] = P[m][1];
    }
    const int ro = r - kBehind;
    const float2 o0 = s_td[slot][kR + 2 * lane], o1 = s_td[slot][kR + 1 + 2 * lane];
    const float ot[2] = {o0.x, o1.x}, od[2] = {o0.y, o1.y};
    fetch(r + kAhead, qx[u0], qy[u0]);
    float er[2];  // |error| of channels 0 and 1 summed, row ro
    if (errs) {
      const int64_t p = (int64_t)min(max(ro + 1, 0), H - 1) * W;
#pragma unroll
      for (int j = 0; j < 2; j++) {
        er[j] = fabsf(en[j][0] - en[j][1]) + fabsf(en[j][2] - en[j][3]);
        en[j][0] = V.render[p + xc[j]];
        en[j][1] = V.target[p + xc[j]];
        en[j][2] = V.render[hw + p + xc[j]];
        en[j][3] = V.target[hw + p + xc[j]];
      }
    }
    wave_sync();
    // horizontal sums over the columns x0 - 5 .. x0 + 6
    float h[4][2], g[3][2];
#pragma unroll
    for (int m = 0; m < 4; m++) h[m][0] = h[m][1] = 0.f;
#pragma unroll
    for (int m = 0; m < 3; m++) g[m][0] = g[m][1] = 0.f;
#pragma unroll
    for (int i2 = 0; i2 < (kTaps + 1) / 2; i2++) {
      const float4 q2 = *reinterpret_cast<const float4*>(&row[2 * lane + 2 * i2]);
      float2 d2[3];
#pragma unroll
      for (int m = 0; m < 3; m++) d2[m] = *reinterpret_cast<const float2*>(&s_p[m][2 * lane + 2 * i2]);
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const float vt = (u ? q2.z : q2.x) - shift, vd = u ? q2.w : q2.y;
        const float vtt = vt * vt, vdd = vd * vd;
#pragma unroll
        for (int j = 0; j < 2; j++) {
          const int k = 2 * i2 + u - j;
          if (k < 0 || k >= kTaps) continue;
          h[0][j] = fmaf(w[k], vt, h[0][j]);
          h[1][j] = fmaf(w[k], vtt, h[1][j]);
          h[2][j] = fmaf(w[k], vd, h[2][j]);
          h[3][j] = fmaf(w[k], vdd, h[3][j]);
#pragma unroll
          for (int m = 0; m < 3; m++) g[m][j] = fmaf(wg[k], u ? d2[m].y : d2[m].x, g[m][j]);
        }
      }
    }
    wave_sync();
    mean = h[0][0];
    float out[2];
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const float q0 = push(ap[0][j], w, g[0][j]), q1 = push(ap[1][j], w, g[1][j]), q2 = push(ap[2][j], w, g[2][j]);
      const float l1 = od[j] < 0.f ? sl1 : (od[j] > 0.f ? -sl1 : 0.f);
      out[j] = l1 + fmaf(od[j], q1, fmaf(0.5f * (ot[j] - od[j]), q2, q0));
    }
    const int rs = r - kR;  // the row whose moments are complete
    const bool in_y = rs >= 0 && rs < H, counts = rs >= y_lo && rs < y_hi;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const float ut = push(am[0][j], w, h[0][j]), e2 = push(am[1][j], w, h[1][j]);
      const float md = push(am[2][j], w, h[2][j]), d2 = push(am[3][j], w, h[3][j]);
      const float mt = ut + shift, mx = 0.5f * (mt - md), my = 0.5f * (mt + md);
      const float Vd = fmaf(-md, md, d2), Vt = fmaf(-ut, ut, e2);
      const float iC = recip(fmaf(mx, mx, fmaf(my, my, kC1)));  // 1 / luminance denominator
      const float iD = recip(fmaf(0.5f, Vt + Vd, kC2));         // 1 / (sigma_x^2 + sigma_y^2 + C2)
      const float e = Vd * iD, l = md * md * iC;                // 1 - structure, 1 - luminance
      const float K = (1.f - l) * iD, Ke = K * e;
      const float S = (1.f - l) * (1.f - e);
      const bool on = in[j] && in_y;  // outside the image the map and its derivatives are 0
      P[0][j] = on ? (1.f - e) * iC * fmaf(mx, l, md) - fmaf(Ke, mx, K * md) : 0.f;
      P[1][j] = on ? K : 0.f;
      P[2][j] = on ? Ke : 0.f;
      ssum += owns[j] && counts ? S : 0.f;
    }
    if (ro >= y_lo) {  // uniform (ro < y_hi)
      float* __restrict__ o = V.dl + c * hw + (int64_t)ro * W + x0;
#pragma unroll
      for (int j = 0; j < 2; j++) {
        if (!owns[j]) continue;
        o[j] = out[j];
        const float e = fabsf(od[j]);
        l1sum += e;
        if (errs) V.err[(int64_t)ro * W + x0 + j] = (er[j] + e) * (1.0f / 3.0f);  // in channel order
      }
    }
  }
  }
  part += ssum * gS + l1sum * sl1;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) part += __shfl_xor(part, d, 64);
  if (lane == 0 && first < end) atomicAdd(&loss_slots[blockIdx.x % kLossSlots], part);
}

// ---- two passes over tiles (small calls) ---------------------------------------------------------
// One workgroup per 32x32 pixel tile (channels in turn), each staging the tile plus its 5-pixel
// halo in LDS and applying the separable window as a horizontal then a vertical 11-tap sum; every
// thread slides the window over 4 consecutive outputs, so each staged value is read from LDS
// about once per 4 outputs instead of 11 times:
//   forward: the five window moments (mu_x, mu_y, E[x^2], E[y^2], E[xy]) of every pixel, the
//     SSIM map and its derivatives with respect to mu_x, E[x^2] and E[xy], scaled by
//     dL/dSSIM; these three maps go to the caller's scratch;
//   backward: the window sums of the three maps give dL/dx as above, to which the L1 term and the error
//     map of Sec. 3.4 are added.
constexpr int kT = 32;           // output tile edge
constexpr int kE = kT + 2 * kR;  // staged edge (42)
constexpr int kEP = kE + 1;      // padded staged row
constexpr int kHP = kT + 1;      // padded row of horizontal sums
constexpr int kRun = 4;          // consecutive outputs per thread and pass
constexpr int kThreads = 256;

// Workgroups are dealt to the XCDs round-robin; remapping gives each XCD a contiguous range of
// tiles, so the halos a tile shares with its neighbours are read through the same L2.
__device__ __forceinline__ int64_t tile_of_block(int64_t bid, int64_t per) {
  return (bid % kNumXcd) * per + bid / kNumXcd;
}

__device__ __forceinline__ int view_of_block(const SsimArgs& a, int64_t blk) {
  int v = 0;
  while (v + 1 < a.nv && blk >= a.v[v + 1].block_begin) v++;
  return v;
}

// Sum over the workgroup of x, added times `scale` into one loss slot.
__device__ __forceinline__ void add_to_slot(float x, float scale, float* s_w, float* loss_slots) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicAdd(&loss_slots[blockIdx.x % kLossSlots], ((s_w[0] + s_w[1]) + (s_w[2] + s_w[3])) * scale);
}

// Stages rows [oy - 5, oy + 37) x cols [ox - 5, ox + 37) of the NS planes src[k] into dst[k]
// (zero outside the image).  All loads are issued before the first LDS store, so their
// latencies overlap.
constexpr int kStageIters = (kE * kE + kThreads - 1) / kThreads;
template <int NS>
__device__ __forceinline__ void stage(float (*dst)[kE][kEP], const float* const (&src)[NS], int ox, int oy, int W,
                                      int H) {
  float v[NS][kStageIters];
#pragma unroll
  for (int u = 0; u < kStageIters; u++) {
    const int e = threadIdx.x + u * kThreads;
    const int r = e / kE, q = e % kE;
    const int gx = ox - kR + q, gy = oy - kR + r;
    const bool in = e < kE * kE && gx >= 0 && gy >= 0 && gx < W && gy < H;
    const int64_t p = in ? (int64_t)gy * W + gx : 0;
#pragma unroll
    for (int k = 0; k < NS; k++) v[k][u] = in ? src[k][p] : 0.f;
  }
#pragma unroll
  for (int u = 0; u < kStageIters; u++) {
    const int e = threadIdx.x + u * kThreads;
    if (e < kE * kE) {
#pragma unroll
      for (int k = 0; k < NS; k++) dst[k][e / kE][e % kE] = v[k][u];
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_ssim_fwd(SsimArgs a, int64_t total, int64_t per,
                                                           float* __restrict__ loss_slots) {
  __shared__ float s_xy[2][kE][kEP];  // render, target
  __shared__ float s_h[5][kE][kHP];    // horizontal sums of x, y, x^2, y^2, xy
  __shared__ float s_w[4];
  const int tid = threadIdx.x;
  const int64_t blk = tile_of_block(blockIdx.x, per);
  if (blk >= total) return;  // uniform over the workgroup
  const int vi = view_of_block(a, blk);
  const SsimView& V = a.v[vi];
  const int t = (int)(blk - V.block_begin);
  const int ox = (t % V.TX) * kT, oy = (t / V.TX) * kT;
  const int64_t hw = (int64_t)V.W * V.H;
  const int col = tid % kT, i0 = (tid / kT) * kRun;  // vertical pass: pixels (col, i0 .. i0 + 3)
  const float gS = a.gS[vi];                          // dL/dSSIM(pixel, channel)
  float ssum = 0.f;
  for (int c = 0; c < 3; c++) {
    const float* const planes[2] = {V.render + c * hw, V.target + c * hw};
    stage<2>(s_xy, planes, ox, oy, V.W, V.H);
    __syncthreads();
    // horizontal: row r, outputs q0 .. q0 + 3
    for (int task = tid; task < kE * (kT / kRun); task += kThreads) {
      const int r = task / (kT / kRun), q0 = (task % (kT / kRun)) * kRun;
      float h[5][kRun];
#pragma unroll
      for (int m = 0; m < 5; m++)
#pragma unroll
        for (int o = 0; o < kRun; o++) h[m][o] = 0.f;
#pragma unroll
      for (int n = 0; n < kTaps + kRun - 1; n++) {
        const float xv = s_xy[0][r][q0 + n], yv = s_xy[1][r][q0 + n];
        const float xx = xv * xv, yy = yv * yv, xy = xv * yv;
#pragma unroll
        for (int o = 0; o < kRun; o++) {
          const int k = n - o;
          if (k < 0 || k >= kTaps) continue;
          const float w = a.w[k];
          h[0][o] += w * xv;
          h[1][o] += w * yv;
          h[2][o] += w * xx;
          h[3][o] += w * yy;
          h[4][o] += w * xy;
        }
      }
#pragma unroll
      for (int m = 0; m < 5; m++)
#pragma unroll
        for (int o = 0; o < kRun; o++) s_h[m][r][q0 + o] = h[m][o];
    }
    __syncthreads();
    // vertical: column col, rows i0 .. i0 + 3
    float mo[5][kRun];
#pragma unroll
    for (int m = 0; m < 5; m++) {
#pragma unroll
      for (int o = 0; o < kRun; o++) mo[m][o] = 0.f;
#pragma unroll
      for (int n = 0; n < kTaps + kRun - 1; n++) {
        const float hv = s_h[m][i0 + n][col];
#pragma unroll
        for (int o = 0; o < kRun; o++) {
          const int k = n - o;
          if (k >= 0 && k < kTaps) mo[m][o] += a.w[k] * hv;
        }
      }
    }
    float* P = V.scratch + (int64_t)(3 * c) * hw;
#pragma unroll
    for (int o = 0; o < kRun; o++) {
      const int px = ox + col, py = oy + i0 + o;
      if (px >= V.W || py >= V.H) continue;
      const float mx = mo[0][o], my = mo[1][o];
      const float A = 2.f * mx * my + kC1;                                // luminance numerator
      const float B = 2.f * (mo[4][o] - mx * my) + kC2;                   // 2 sigma_xy + C2
      const float Cc = mx * mx + my * my + kC1;                           // luminance denominator
      const float D = (mo[2][o] - mx * mx) + (mo[3][o] - my * my) + kC2;  // sigma_x^2 + sigma_y^2 + C2
      const float iCD = 1.f / (Cc * D);
      const float S = A * B * iCD;
      const float dmx = (2.f * my * B - 2.f * my * A) * iCD - S * (2.f * mx / Cc - 2.f * mx / D);
      const float dxx = -S / D;
      const float dxy = 2.f * A * iCD;
      const int64_t p = (int64_t)py * V.W + px;
      P[p] = gS * dmx;
      P[hw + p] = gS * dxx;
      P[2 * hw + p] = gS * dxy;
      ssum += S;
    }
    __syncthreads();  // the next channel restages
  }
  add_to_slot(ssum, gS, s_w, loss_slots);
}

__global__ __launch_bounds__(kThreads) void k_ssim_bwd(SsimArgs a, int64_t total, int64_t per,
                                                           float* __restrict__ loss_slots) {
  __shared__ float s_p[3][kE][kEP];
  __shared__ float s_h[3][kE][kHP];
  __shared__ float s_w[4];
  const int tid = threadIdx.x;
  const int64_t blk = tile_of_block(blockIdx.x, per);
  if (blk >= total) return;  // uniform over the workgroup
  const int vi = view_of_block(a, blk);
  const SsimView& V = a.v[vi];
  const int t = (int)(blk - V.block_begin);
  const int ox = (t % V.TX) * kT, oy = (t / V.TX) * kT;
  const int64_t hw = (int64_t)V.W * V.H;
  const int col = tid % kT, i0 = (tid / kT) * kRun;
  const float sl1 = a.l1_scale[vi];  // (1 - lambda) / (3 H W V)
  float e[kRun] = {0.f, 0.f, 0.f, 0.f};
  for (int c = 0; c < 3; c++) {
    const float* P = V.scratch + (int64_t)(3 * c) * hw;
    const float* const planes[3] = {P, P + hw, P + 2 * hw};
    stage<3>(s_p, planes, ox, oy, V.W, V.H);
    __syncthreads();
    for (int task = tid; task < kE * (kT / kRun); task += kThreads) {
      const int r = task / (kT / kRun), q0 = (task % (kT / kRun)) * kRun;
#pragma unroll
      for (int m = 0; m < 3; m++) {
        float h[kRun] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < kTaps + kRun - 1; n++) {
          const float pv = s_p[m][r][q0 + n];
#pragma unroll
          for (int o = 0; o < kRun; o++) {
            const int k = n - o;
            if (k >= 0 && k < kTaps) h[o] += a.w[k] * pv;
          }
        }
#pragma unroll
        for (int o = 0; o < kRun; o++) s_h[m][r][q0 + o] = h[o];
      }
    }
    __syncthreads();
    float Q[3][kRun];
#pragma unroll
    for (int m = 0; m < 3; m++) {
#pragma unroll
      for (int o = 0; o < kRun; o++) Q[m][o] = 0.f;
#pragma unroll
      for (int n = 0; n < kTaps + kRun - 1; n++) {
        const float hv = s_h[m][i0 + n][col];
#pragma unroll
        for (int o = 0; o < kRun; o++) {
          const int k = n - o;
          if (k >= 0 && k < kTaps) Q[m][o] += a.w[k] * hv;
        }
      }
    }
#pragma unroll
    for (int o = 0; o < kRun; o++) {
      const int px = ox + col, py = oy + i0 + o;
      if (px >= V.W || py >= V.H) continue;
      const int64_t pix = (int64_t)py * V.W + px;
      const float x = V.render[c * hw + pix], y = V.target[c * hw + pix];
      const float d = x - y;
      const float l1 = d > 0.f ? sl1 : (d < 0.f ? -sl1 : 0.f);
      V.dl[c * hw + pix] = l1 + (Q[0][o] + 2.f * x * Q[1][o] + y * Q[2][o]);
      e[o] += fabsf(d);  // summed over channels in channel order
    }
    __syncthreads();  // the next channel restages
  }
  float l1sum = 0.f;
#pragma unroll
  for (int o = 0; o < kRun; o++) {
    const int px = ox + col, py = oy + i0 + o;
    if (px >= V.W || py >= V.H) continue;
    if (V.err) V.err[(int64_t)py * V.W + px] = e[o] * (1.0f / 3.0f);
    l1sum += e[o];
  }
  add_to_slot(l1sum, sl1, s_w, loss_slots);
}

// Whether a view's outputs lie in its inputs, or its error map in its gradient.  The two passes read the windows'
// pixels before the first output and only the own pixel's afterwards, so that the gradient may take
// the place of the images; the waves of the one pass read pixels that others write.
bool in_place(const SsimView& V) {
  const int64_t hw = (int64_t)V.W * V.H;
  const auto meet = [](const float* a, int64_t na, const float* b, int64_t nb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + (uintptr_t)nb * 4 && y < x + (uintptr_t)na * 4;
  };
  if (meet(V.dl, 3 * hw, V.render, 3 * hw) || meet(V.dl, 3 * hw, V.target, 3 * hw)) return true;
  return V.err && (meet(V.err, hw, V.render, 3 * hw) || meet(V.err, hw, V.target, 3 * hw) || meet(V.err, hw, V.dl, 3 * hw));
}

}  // namespace

void launch_ssim(SsimArgs& a, float* loss_slots, hipStream_t st) {
  // One pass: every (channel, strip) of every view is H rows long; all rows are dealt to the waves in
  // equal runs, so that the waves the chip holds (two per SIMD) end together.  A run of rows costs 21
  // more (its halo), and once more where it passes into the next strip.
  int64_t total = 0;
  double pixels = 0.0;
  bool two = false;  // in place: the two passes
  for (int v = 0; v < a.nv; v++) {
    a.v[v].strips = (a.v[v].W + kOut - 1) / kOut;
    a.v[v].row_begin = total;
    total += 3ll * a.v[v].strips * a.v[v].H;
    pixels += (double)a.v[v].W * a.v[v].H;
    two = two || in_place(a.v[v]);
  }
  if (total == 0) return;
  constexpr int kSlots = 2048;
  // A row takes a wave about 1.8 us, and the two passes 47 us per million pixels, so few or narrow
  // strips go through the passes: measured in us, passes / one pass, 1 view of 1352x1014 80 / 104, 2
  // views 129 / 112, 3 198 / 168, 6 406 / 270, 20 1300 / 775; 1 of 1920x1080 100 / 120, 2 197 / 168; 9 of
  // 640x480 132 / 134, 20 324 / 221; 10 of 500x500 123 / 134, 20 267 / 207; 20 of 333x477 161 / 176
  // (four strips of 84 columns each), 20 of 109x1014 130 / 175.
  if (two || 1.8 * ((double)total / kSlots + 29.0) >= 47e-6 * pixels) {
    int64_t blocks = 0;
    for (int v = 0; v < a.nv; v++) {
      a.v[v].TX = (a.v[v].W + kT - 1) / kT;
      a.v[v].block_begin = blocks;
      blocks += (int64_t)a.v[v].TX * ((a.v[v].H + kT - 1) / kT);
    }
    const int64_t per = (blocks + kNumXcd - 1) / kNumXcd;
    k_ssim_fwd<<<(unsigned)(per * kNumXcd), kThreads, 0, st>>>(a, blocks, per, loss_slots);
    k_ssim_bwd<<<(unsigned)(per * kNumXcd), kThreads, 0, st>>>(a, blocks, per, loss_slots);
    return;
  }
  a.total_rows = total;
  a.rows = std::max<int64_t>(8, (total + kSlots - 1) / kSlots);
  const int64_t waves = (total + a.rows - 1) / a.rows;
  const int64_t per = (waves + kNumXcd - 1) / kNumXcd;
  k_ssim<<<(unsigned)(per * kNumXcd), kLanes, 0, st>>>(a, (int)per, loss_slots);
}

}  // namespace dass
