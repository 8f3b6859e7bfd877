// The front-to-back blend with its adjoint (App. A.1), over each tile's list of record indices
// (view * n + Gaussian) in depth order.
//
// Blend.  One wave per sub-tile of a tile (16x16 with four pixels per lane, one in each 8x8
// quadrant, or 8x8 with one pixel per lane, for small images where the lists are walked by few
// waves).  The tile's list is consumed in batches of 64, 128 or 256 entries (a per-call option),
// each culled against the quadrants of the wave's sub-tile and compacted into LDS; every lane walks its pixels front
// to back, skipping the quadrants an entry misses, and the wave stops as soon as every pixel
// has hit the transmittance stop.
// The backward recomputes each entry's alpha per batch, recovers the transmittance by dividing
// out (1 - alpha) from T_final while walking backwards, sums each Gaussian's 9 gradient terms
// over the wave and issues one vector atomic per (Gaussian, wave).
#include "dass_internal.h"

namespace dass {
namespace {

// B: list entries staged in LDS per batch (64, 128 or 256; a per-call option)
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ int xcd_logical(int bid, int per) {
  // consecutive workgroups land on different XCDs; give each XCD a contiguous tile range
  return (bid % kNumXcd) * per + bid / kNumXcd;
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = i; j < n; j += stride) p[j] = v;
}

__device__ __forceinline__ int view_of(const ViewsIO& io, int nv, int b) {
  int v = 0;
  while (v + 1 < nv && b >= io.v[v + 1].tile_base) v++;
  return v;
}

// ---- blend ------------------------------------------------------------------------------------
// One wave per sub-tile (16x16 or 8x8 pixels).  The sub-tile is cut into 8x8 quadrants and
// lane (qx, qy) of the 8x8 lane grid owns pixel (qx, qy) of every quadrant.  Batches of up to
// 128 list entries are loaded by the wave, culled per quadrant and compacted into LDS in list
// order; an entry leaves a quadrant only if the minimum of its quadratic form over the
// quadrant's pixel rectangle exceeds the alpha >= 1/255 level by a margin, i.e. when every pixel
// of that quadrant would skip it anyway, and leaves the list when no quadrant keeps it.  The list
// position of every kept entry is carried along (low 27 bits, the quadrant mask in the top four),
// so n_contrib still counts positions in the full list; the walk skips a quadrant an entry misses
// with a uniform branch.
// An entry's alpha never exceeds its opacity, so only an entry with opacity >= 0.99 can meet the
// alpha clamp; the backward marks those (kClampBit) and tests the clamp for its zero derivative
// on them alone.  For any other entry the clamp is inactive in the definition's arithmetic (the
// opacity times a falloff <= 1 is below 0.99), and an alpha that float32 rounds to 0.99 there
// keeps its derivative.
constexpr int kLanes = 64;
constexpr int kPosBits = 27;  // list positions carried with the clamp bit and the quadrant mask
constexpr int kPosMask = (1 << kPosBits) - 1;
constexpr uint32_t kClampBit = 1u << kPosBits;
constexpr int kQmShift = 28;
constexpr uint32_t kInfBit = 1u;  // (backward by quadrant) the colour is not finite
constexpr float kNever = 2.0f;  // alpha threshold of a stopped pixel: above every alpha (<= 0.99)

__device__ __forceinline__ uint64_t lane_lt_mask(int lane) { return lane == 0 ? 0ull : (~0ull >> (64 - lane)); }

// Minimum of q(d) = A dx^2 + 2B dx dy + C dy^2, d = pixel - mean, over the pixel-centre
// rectangle [x0, x1] x [y0, y1] (mean at (mx, my)); ia, ic = 1/A, 1/C (0 if not positive).  For
// a convex q the minimiser is the mean when it lies inside; otherwise it lies on the edge that
// faces the mean in x (when mx is outside [x0, x1]) or on the one that faces it in y: the
// vertical segment at the rectangle's x nearest mx and the horizontal segment at its y nearest my
// hold it in every case, and on each segment the line minimiser is clamped to the segment.
__device__ __forceinline__ float rect_min_q(float mx, float my, float A, float B, float C, float ia, float ic,
                                            float x0, float x1, float y0, float y1) {
  // (med3 of a value and an ordered pair clamps it to the pair's interval)
  float dx = __builtin_amdgcn_fmed3f(mx, x0, x1) - mx;
  float dy = __builtin_amdgcn_fmed3f(-B * dx * ic, y0 - my, y1 - my);
  const float qv = A * dx * dx + 2.f * B * dx * dy + C * dy * dy;
  dy = __builtin_amdgcn_fmed3f(my, y0, y1) - my;
  dx = __builtin_amdgcn_fmed3f(-B * dy * ia, x0 - mx, x1 - mx);
  const float qh = A * dx * dx + 2.f * B * dx * dy + C * dy * dy;
  return fminf(qv, qh);
}

// Bit k set if the entry (mean (mx, my) relative to the sub-tile origin, conic A B C, opacity o)
// may reach alpha >= 1/255 at a pixel centre of 8x8 quadrant k = (k % PW, k / PW).
template <int PW>
__device__ __forceinline__ uint32_t quad_mask(float mx, float my, float A, float B, float C, float o) {
  if (!(o * 255.0f > 0.999f)) return 0u;  // alpha <= o < 1/255 everywhere (with margin)
  // q <= 2 ln(255 o)  <=>  o exp(-q/2) >= 1/255; the margin keeps every kept decision
  // (hardware log2: 255 o > 1 here, and the margin covers its rounding)
  const float thr = (2.0f * 0.6931471805599453f) * __builtin_amdgcn_logf(255.0f * o) * 1.001f + 1e-3f;
  const float ia = A > 0.f ? __builtin_amdgcn_rcpf(A) : 0.f, ic = C > 0.f ? __builtin_amdgcn_rcpf(C) : 0.f;
  uint32_t m = 0;
  if constexpr (PW == 2) {
    // rect_min_q for the 2x2 grid of quadrants, sharing the work of each column and row: the
    // vertical segment of column cx sits at the same x (and the line minimiser there at the
    // same y) for both rows, and likewise for the horizontal segment of row cy; relative to the
    // mean, clamp(mx, x0, x1) - mx = clamp(0, x0 - mx, x1 - mx).
    const float xl[2] = {-mx, 8.f - mx}, xh[2] = {7.f - mx, 15.f - mx};
    const float yl[2] = {-my, 8.f - my}, yh[2] = {7.f - my, 15.f - my};
    const float nbc = -B * ic, nba = -B * ia, b2 = 2.f * B;
    float qv[4];
#pragma unroll
    for (int cx = 0; cx < 2; cx++) {
      const float dx = __builtin_amdgcn_fmed3f(0.f, xl[cx], xh[cx]);
      const float ys = dx * nbc, ax = A * dx * dx, bx = b2 * dx;
#pragma unroll
      for (int cy = 0; cy < 2; cy++) {
        const float dy = __builtin_amdgcn_fmed3f(ys, yl[cy], yh[cy]);
        qv[cx + 2 * cy] = fmaf(dy, fmaf(C, dy, bx), ax);  // A dx^2 + 2B dx dy + C dy^2
      }
    }
#pragma unroll
    for (int cy = 0; cy < 2; cy++) {
      const float dy = __builtin_amdgcn_fmed3f(0.f, yl[cy], yh[cy]);
      const float xs = dy * nba, cy2 = C * dy * dy, by = b2 * dy;
#pragma unroll
      for (int cx = 0; cx < 2; cx++) {
        const float dx = __builtin_amdgcn_fmed3f(xs, xl[cx], xh[cx]);
        const float qh = fmaf(dx, fmaf(A, dx, by), cy2);
        if (fminf(qv[cx + 2 * cy], qh) <= thr) m |= 1u << (cx + 2 * cy);
      }
    }
    return m;
  }
#pragma unroll 1  // rolled: unrolled, the four rectangles cost the forward an occupancy step
  for (int k = 0; k < PW * PW; k++) {
    const float x0 = (float)(8 * (k % PW)), y0 = (float)(8 * (k / PW));
    if (rect_min_q(mx, my, A, B, C, ia, ic, x0, x0 + 7.f, y0, y0 + 7.f) <= thr) m |= 1u << k;
  }
  return m;
}

template <int CTRL>
__device__ __forceinline__ float dppf(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Transposing reduction of nine per-lane values of two list entries over the wave: each step pairs values (x, y) and
// adds every value to its copy on the partner lane across one lane bit, keeping x's pair total
// on the lanes with that bit clear and y's on the lanes with it set, so the number of values
// per lane halves at each step without selects.
// Lane bits 5 and 4 (partners 32 or 16 lanes apart): gfx950's permlane swaps exchange the upper
// half of x with the lower half of y (the odd 16-lane rows of x with the even rows of y), after
// which x + y holds x's total on one side and y's on the other.
__device__ __forceinline__ float swap32_sum(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_sum(float x, float y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Lane bits 3 and 2 (partners 8 or 4 lanes apart in a 16-lane row): two DPP adds whose bank
// masks (a bank is 4 consecutive lanes of a row) write complementary halves of the lanes.  The
// leading s_nop gives the DPP reads of x and y the two wait states they need after a VALU write.
__device__ __forceinline__ float dpp_pair8(float x, float y) {
  float o;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"  // lanes with bit 3 clear
      "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc"       // lanes with bit 3 set
      : "=&v"(o)
      : "v"(x), "v"(y));
  return o;
}
__device__ __forceinline__ float dpp_pair4(float x, float y) {
  float o;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %1, %1 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"  // bit 2 clear: lane + 4
      "v_add_f32_dpp %0, %2, %2 row_shr:4 row_mask:0xf bank_mask:0xa"       // bit 2 set: lane - 4
      : "=&v"(o)
      : "v"(x), "v"(y));
  return o;
}

// Sums two entries' nine values v0, v1 over the wave.  Afterwards lane bit 5 is the entry and bits 4..1
// = m the value kRedSlot[m] (-1: a duplicate of another lane's total); `odd` = lane bit 1.  41
// instructions for the two (one entry at a time: 26 each, for a full wave that carries one).
__device__ __forceinline__ float wave_reduce18(const float* v0, const float* v1, bool odd) {
  float c[9];
#pragma unroll
  for (int i = 0; i < 9; i++) c[i] = swap32_sum(v0[i], v1[i]);
  // bit 4 -> 0 1 2 3 4 or 5 6 7 8 4
  const float b0 = swap16_sum(c[0], c[5]), b1 = swap16_sum(c[1], c[6]), b2 = swap16_sum(c[2], c[7]);
  const float b3 = swap16_sum(c[3], c[8]), b4 = swap16_sum(c[4], c[4]);
  // bit 3 -> (bits 4, 3) = 00: 0 1 2, 01: 3 4 2, 10: 5 6 7, 11: 8 4 7
  const float d0 = dpp_pair8(b0, b3), d1 = dpp_pair8(b1, b4), d2 = b2 + dppf<0x128>(b2);
  // bit 2 -> the first or the second of these, and the third
  float e0 = dpp_pair4(d0, d1), e1 = dpp_pair4(d2, d2);
  e0 += dppf<0x4E>(e0);  // quad_perm 2, 3, 0, 1
  e1 += dppf<0x4E>(e1);
  const float f = odd ? e1 : e0;
  return f + dppf<0xB1>(f);  // quad_perm 1, 0, 3, 2
}
__constant__ int kRedSlot[16] = {0, 2, 1, -1, 3, -1, 4, -1, 5, 7, 6, -1, 8, -1, -1, -1};

// A staged list entry in LDS: one 48-byte row, so a wave reads an entry's fields from one address.
struct FwdStage {
  float4 co;   // log2-scaled conic, log2 opacity
  float4 rgb;  // colour, (list position + 1) | quadrant mask << 28 (int bits)
  float2 xy;   // mean relative to the sub-tile origin
  float2 pad;
};
struct BwdStage {
  float4 co;   // as the forward's
  float4 rgb;  // colour, list position | clamp bit | quadrant mask << 28 (int bits)
  float2 xy;
  uint32_t p;  // record index = gradient row (view * n + Gaussian)
  float io;    // 1 / opacity
};

// L1: the epilogue also forms the L1 term against the view's target (dL/drgb, error map and
// this sub-tile's share of the loss, added into one of kLossSlots partial sums).
template <bool COUNT, bool L1, int SUB, int B>
__global__ __launch_bounds__(kLanes) void k_blend_fwd(ViewsIO io, int nv, int total_blocks, int per, float bg0,
                                                      float bg1, float bg2, const uint2* __restrict__ ranges,
                                                      const uint32_t* __restrict__ vals, const Rec* __restrict__ rec,
                                                      unsigned long long* __restrict__ pairs,
                                                      float* __restrict__ loss_slots) {
  constexpr int PW = SUB / 8, NP = PW * PW;  // quadrants per edge, pixels per lane
  __shared__ FwdStage s_st[B];
  const int lb = xcd_logical(blockIdx.x, per);
  if (lb >= total_blocks) return;
  const int b = lb / io.sn, sub = lb - b * io.sn;  // tile, SUB x SUB sub-tile of it
  const int v = view_of(io, nv, b);
  const ViewIO& V = io.v[v];
  const int t = b - V.tile_base;
  const int tx = t % V.TX, ty = t / V.TX;
  const int ox = tx * io.tw + (sub % io.sx) * SUB, oy = ty * io.th + (sub / io.sx) * SUB;
  if (ox >= V.W || oy >= V.H) return;  // sub-tile entirely outside the image
  const int lane = threadIdx.x;
  const int qx = lane & 7, qy = lane >> 3;
  const float fx0 = (float)ox, fy0 = (float)oy;
  const uint64_t lt = lane_lt_mask(lane);
  const uint2 r = ranges[b];
  if (r.y - r.x > (uint32_t)kPosMask) {  // positions would not fit their bits: reported, not drawn
    if (lane == 0) atomicOr(io.err, kErrListTooLong);
    return;
  }
  // thr[k]: the alpha a pixel's entries must reach to blend; 1/255 while it walks its list,
  // kNever once it has stopped (or for a pixel outside the image), so it never blends again and
  // keeps its transmittance
  float T[NP], thr[NP], c0[NP], c1[NP], c2[NP];
  uint32_t last[NP];  // (list position + 1) of the last blended entry, quadrant mask above it
#pragma unroll
  for (int k = 0; k < NP; k++) {
    const int px = ox + qx + 8 * (k % PW), py = oy + qy + 8 * (k / PW);
    T[k] = 1.f;
    thr[k] = (px < V.W && py < V.H) ? kAlphaMin : kNever;
    c0[k] = c1[k] = c2[k] = 0.f;
    last[k] = 0;
  }
  uint32_t n_eval = 0, n_blend = 0;
  for (uint32_t start = r.x; start < r.y; start += B) {
    const int n_in = (int)min((uint32_t)B, r.y - start);
    int n_kept = 0;
#pragma unroll
    for (int k = 0; k < B / kLanes; k++) {
      const int e = k * kLanes + lane;
      uint32_t qm = 0;
      float2 xy;
      float4 co, rgb;
      if (e < n_in) {
        const Rec R = rec[vals[start + e]];
        xy = make_float2((R.r0.x - fx0) + R.r0.z, (R.r0.y - fy0) + R.r0.w);
        qm = quad_mask<PW>(xy.x, xy.y, R.r1.x, R.r1.y, R.r1.z, R.r1.w);
        // exponent in base 2 with the opacity folded in: alpha = 2^(q' + log2 o)
        co = make_float4(-0.5f * kLog2e * R.r1.x, -kLog2e * R.r1.y, -0.5f * kLog2e * R.r1.z, __log2f(R.r1.w));
        rgb = make_float4(R.r2.x, R.r2.y, R.r2.z,
                          __uint_as_float(((uint32_t)(start - r.x) + e + 1) | (qm << kQmShift)));
      }
      const bool keep = qm != 0;
      const uint64_t m = __ballot(keep);
      if (keep) {
        const int pos = n_kept + __popcll(m & lt);
        s_st[pos].co = co;
        s_st[pos].rgb = rgb;
        s_st[pos].xy = xy;
      }
      n_kept += __popcll(m);
    }
    // quadrants with a pixel still walking (a stopped pixel stays stopped); a quadrant leaves the
    // mask as soon as its last pixel stops, and the wave leaves the batch when none is left
    uint32_t qalive = 0;
#pragma unroll
    for (int k = 0; k < NP; k++) qalive |= __ballot(thr[k] < 1.f) != 0 ? 1u << k : 0u;
    __syncthreads();
    for (int j = 0; j < n_kept && qalive != 0; j++) {
      const float2 xy = s_st[j].xy;
      const float4 co = s_st[j].co;
      const float4 c = s_st[j].rgb;
      const uint32_t wv = __float_as_uint(c.w);  // (position + 1) | quadrant mask << 28
      const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)wv);  // same for all lanes
      const uint32_t qm = (w >> kQmShift) & qalive;
      const float dxb = xy.x - (float)qx, dyb = xy.y - (float)qy;
#pragma unroll
      for (int k = 0; k < NP; k++) {
        if (NP > 1 && !((qm >> k) & 1u)) continue;  // uniform: no pixel of quadrant k can take it
        const float dx = dxb - (float)(8 * (k % PW)), dy = dyb - (float)(8 * (k / PW));
        // the conic is positive definite, so the exponent (before log2 o) is never above 0
        const float pw = fmaf(dx, fmaf(co.x, dx, co.y * dy), fmaf(co.z * dy, dy, co.w));
        const float a = fminf(kAlphaMax, __builtin_amdgcn_exp2f(pw));
        const bool ok = a >= thr[k];
        float wgt = ok ? a * T[k] : 0.f;
        T[k] -= wgt;  // updated in place: a pixel that stops here gets its transmittance back below
        bool take = ok;
        // only a pixel that passed the test can cross the stop: the others keep a transmittance at
        // or above it (a stopped pixel's is restored below, to within one rounding of the value
        // before its stop; were that under the stop, this branch would only repeat the restore)
        const bool stop = T[k] < kTStop;
        if (__builtin_expect(__ballot(stop) != 0, 0)) {  // uniform: a pixel of the quadrant stops here
          // T - w + w: the transmittance before this entry up to one rounding
          T[k] = stop ? T[k] + wgt : T[k];
          wgt = stop ? 0.f : wgt;
          take = ok && !stop;
          if (COUNT) n_eval += thr[k] < 1.f ? 1u : 0u;
          thr[k] = stop ? kNever : thr[k];
          if (__ballot(thr[k] < 1.f) == 0) qalive &= ~(1u << k);
        } else if (COUNT) {
          n_eval += thr[k] < 1.f ? 1u : 0u;
        }
        if (COUNT) n_blend += take ? 1u : 0u;
        c0[k] = fmaf(c.x, wgt, c0[k]);
        c1[k] = fmaf(c.y, wgt, c1[k]);
        c2[k] = fmaf(c.z, wgt, c2[k]);
        last[k] = take ? wv : last[k];
      }
    }
    bool alive = false;
#pragma unroll
    for (int k = 0; k < NP; k++) alive = alive || thr[k] < 1.f;
    if (__ballot(alive) == 0) break;
    __syncthreads();
  }
  float l1sum = 0.f;
#pragma unroll
  for (int k = 0; k < NP; k++) {
    const int px = ox + qx + 8 * (k % PW), py = oy + qy + 8 * (k / PW);
    if (px < V.W && py < V.H) {
      const int64_t hw = (int64_t)V.W * V.H;
      const int64_t pix = (int64_t)py * V.W + px;
      const float col[3] = {c0[k] + T[k] * bg0, c1[k] + T[k] * bg1, c2[k] + T[k] * bg2};
      if (!L1 || V.rgb) {
#pragma unroll
        for (int c = 0; c < 3; c++) V.rgb[c * hw + pix] = col[c];
      }
      V.t_final[pix] = T[k];
      V.n_contrib[pix] = (int)(last[k] & kPosMask);
      if (L1) {
        const float sc = V.l1_scale;
        float e = 0.f;
#pragma unroll
        for (int c = 0; c < 3; c++) {
          const float d = col[c] - V.target[c * hw + pix];
          V.dl_out[c * hw + pix] = d > 0.f ? sc : (d < 0.f ? -sc : 0.f);
          e += fabsf(d);
        }
        if (V.err) V.err[pix] = e * (1.0f / 3.0f);
        l1sum += e;
      }
    }
  }
  if (L1) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) l1sum += __shfl_xor(l1sum, d, 64);
    if (lane == 0) atomicAdd(&loss_slots[lb % kLossSlots], l1sum * V.l1_scale);
  }
  if (COUNT) {
    atomicAdd(&pairs[0], (unsigned long long)n_eval);
    atomicAdd(&pairs[1], (unsigned long long)n_blend);
  }
}

template <int SUB, int B>
__global__ __launch_bounds__(kLanes) void k_blend_bwd(ViewsIO io, int nv, int total_blocks, int per, float bg0,
                                                      float bg1, float bg2, const uint2* __restrict__ ranges,
                                                      const uint32_t* __restrict__ vals, const Rec* __restrict__ rec,
                                                      float* __restrict__ g2d) {
  constexpr int PW = SUB / 8, NP = PW * PW;  // quadrants per edge, pixels per lane
  __shared__ BwdStage s_st[B];
  const int lb = xcd_logical(blockIdx.x, per);
  if (lb >= total_blocks) return;
  const int b = lb / io.sn, sub = lb - b * io.sn;  // tile, SUB x SUB sub-tile of it
  const int v = view_of(io, nv, b);
  const ViewIO& V = io.v[v];
  const int t = b - V.tile_base;
  const int tx = t % V.TX, ty = t / V.TX;
  const int ox = tx * io.tw + (sub % io.sx) * SUB, oy = ty * io.th + (sub / io.sx) * SUB;
  if (ox >= V.W || oy >= V.H) return;  // sub-tile entirely outside the image
  const int lane = threadIdx.x;
  const int qx = lane & 7, qy = lane >> 3;
  const float fx0 = (float)ox, fy0 = (float)oy;
  const uint64_t lt = lane_lt_mask(lane);
  const uint2 r = ranges[b];
  if (r.y - r.x > (uint32_t)kPosMask) return;  // the forward reported it
  const int64_t hw = (int64_t)V.W * V.H;
  // per pixel: transmittance, dL/d(pixel colour), nS = -dL/dC . (colour blended behind the
  // current entry, background included)
  float T[NP], dC0[NP], dC1[NP], dC2[NP], nS[NP];
  int last[NP];
  int qlast[NP];  // per quadrant: the largest n_contrib of its pixels (uniform)
  int max_all = 0;
#pragma unroll
  for (int k = 0; k < NP; k++) {
    const int px = ox + qx + 8 * (k % PW), py = oy + qy + 8 * (k / PW);
    T[k] = 1.f;
    dC0[k] = dC1[k] = dC2[k] = 0.f;
    last[k] = 0;
    if (px < V.W && py < V.H) {
      const int64_t pix = (int64_t)py * V.W + px;
      T[k] = V.t_final[pix];
      last[k] = V.n_contrib[pix];
      dC0[k] = V.dl[pix];
      dC1[k] = V.dl[hw + pix];
      dC2[k] = V.dl[2 * hw + pix];
    }
    nS[k] = -(bg0 * dC0[k] + bg1 * dC1[k] + bg2 * dC2[k]);
    int mx = last[k];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) mx = max(mx, __shfl_xor(mx, d, 64));
    qlast[k] = __builtin_amdgcn_readfirstlane(mx);
    max_all = max(max_all, qlast[k]);
  }
  const int max_last = min(max_all, (int)(r.y - r.x));  // n_contrib never exceeds the list length
  if (max_last <= 0) return;
  const int slot = kRedSlot[(lane >> 1) & 15];
  const bool writes = (lane & 1) == 0 && slot >= 0, odd = (lane & 2) != 0;
  const int nbatch = (max_last + B - 1) / B;
  for (int bi = nbatch - 1; bi >= 0; bi--) {
    const uint32_t start = r.x + (uint32_t)bi * B;
    const int n_in = min(B, max_last - bi * B);
    __syncthreads();
    int n_kept = 0;
#pragma unroll
    for (int k = 0; k < B / kLanes; k++) {
      const int e = k * kLanes + lane;
      uint32_t qm = 0;
      float2 xy;
      float4 cn, rgb;
      uint32_t p = 0;
      if (e < n_in) {
        p = vals[start + e];
        const Rec R = rec[p];
        xy = make_float2((R.r0.x - fx0) + R.r0.z, (R.r0.y - fy0) + R.r0.w);
        cn = R.r1;
        qm = quad_mask<PW>(xy.x, xy.y, cn.x, cn.y, cn.z, cn.w);
        // and only the quadrants where some pixel's last contribution is at or after the entry
        // (a compare per lane and quadrant here instead of a scalar test per entry and quadrant
        // in the walk; an entry left with none is not staged)
#pragma unroll
        for (int k = 0; k < NP; k++)
          if (bi * B + e >= qlast[k]) qm &= ~(1u << k);
        const uint32_t cb = cn.w >= kAlphaMax ? kClampBit : 0u;  // as the forward's
        rgb = make_float4(R.r2.x, R.r2.y, R.r2.z, __uint_as_float((uint32_t)(bi * B + e) | cb | (qm << kQmShift)));
      }
      const bool keep = qm != 0;
      const uint64_t m = __ballot(keep);
      if (keep) {
        const int pos = n_kept + __popcll(m & lt);
        s_st[pos].co = make_float4(-0.5f * kLog2e * cn.x, -kLog2e * cn.y, -0.5f * kLog2e * cn.z, __log2f(cn.w));
        s_st[pos].rgb = rgb;
        s_st[pos].xy = xy;
        s_st[pos].p = p;
        s_st[pos].io = 1.0f / cn.w;
      }
      n_kept += __popcll(m);
    }
    __syncthreads();
    // one entry over the sub-tile's quadrants: whether any pixel blended it
    auto entry = [&](int j, float* __restrict__ m) {
      const float2 xy = s_st[j].xy;
      const float4 co = s_st[j].co;
      const float4 c = s_st[j].rgb;
      const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(__float_as_int(c.w));  // same for all lanes
      const int idx = (int)(w & kPosMask);
      const uint32_t qm = w >> kQmShift;
      const float dxb = xy.x - (float)qx, dyb = xy.y - (float)qy;
      // per-lane sums over its pixels: m = (sum dP dx, sum dP dy, sum dP dx^2, sum dP dx dy,
      // sum dP dy^2, d opacity (times the opacity until the reduction), d rgb),
      // dP = dL/d(exponent), (dx, dy) = mean - pixel
#pragma unroll
      for (int q = 0; q < 9; q++) m[q] = 0.f;
      bool any = false;
      const bool clampable = (w & kClampBit) != 0;  // uniform
#pragma unroll
      for (int k = 0; k < NP; k++) {
        // uniform: the entry misses quadrant k, or lies behind the last contribution of every
        // pixel there (both folded into the staged mask)
        if (NP > 1 && !((qm >> k) & 1u)) continue;
        const float dx = dxb - (float)(8 * (k % PW)), dy = dyb - (float)(8 * (k / PW));
        const float pw = fmaf(dx, fmaf(co.x, dx, co.y * dy), fmaf(co.z * dy, dy, co.w));  // + log2 o
        const float araw = __builtin_amdgcn_exp2f(pw);
        const float a = fminf(kAlphaMax, araw);
        const bool take = (idx < last[k]) && (a >= kAlphaMin);  // the forward blended this entry here
        if (__ballot(take) == 0) continue;  // uniform
        any = true;
        // branch-free over the lanes: a pixel that did not blend the entry sees alpha 0, which
        // leaves its transmittance and colour-behind unchanged and adds nothing
        const float ae = take ? a : 0.f;
        T[k] = T[k] * __builtin_amdgcn_rcpf(1.f - ae);  // transmittance before this entry
        const float wgt = ae * T[k];
        m[6] = fmaf(wgt, dC0[k], m[6]);
        m[7] = fmaf(wgt, dC1[k], m[7]);
        m[8] = fmaf(wgt, dC2[k], m[8]);
        // dL/d alpha = T (dL/dC . (colour - colour behind)); the colour behind moves by alpha of that
        const float ed = fmaf(c.x, dC0[k], fmaf(c.y, dC1[k], fmaf(c.z, dC2[k], nS[k])));
        nS[k] = fmaf(-ae, ed, nS[k]);
        // dP = alpha dL/d alpha = alpha T ed: dL/d(exponent), and the opacity times dL/d(opacity)
        float dP = wgt * ed;
        if (__builtin_expect(clampable, 0)) {
          __asm__ volatile("");  // keeps this rarely taken uniform branch a branch
          dP = araw < kAlphaMax ? dP : 0.f;  // no derivative through an active clamp
        }
        m[5] += dP;  // d alpha / d o = alpha / o, the 1 / o applied once per entry
        const float pdx = dP * dx, pdy = dP * dy;
        m[0] += pdx;
        m[1] += pdy;
        m[2] = fmaf(pdx, dx, m[2]);
        m[3] = fmaf(pdx, dy, m[3]);
        m[4] = fmaf(pdy, dy, m[4]);
      }
      return any;
    };
    // two entries at a time, for their sums over the lanes to be taken together (one at a time, us:
    // 13 views of 1280x720 1012, 4 of 1920x1080 1005; now 990, 980)
    for (int j = n_kept - 1; j >= 0; j -= 2) {
      float m0[9], m1[9];
      const bool any0 = entry(j, m0);
      const bool any1 = j > 0 && entry(j - 1, m1);
      if (j == 0) {
#pragma unroll
        for (int q = 0; q < 9; q++) m1[q] = 0.f;
      }
      if (any0 || any1) {  // uniform
        // the sums are linear in the entry's conic, so the conic is applied once per
        // (view, Gaussian) by the projection adjoint, not here
        const float tot = wave_reduce18(m0, m1, odd);
        const int e = lane < 32 ? j : max(j - 1, 0);
        const float o = slot == 5 ? s_st[e].io : 1.f;
        if (writes && (lane < 32 ? any0 : any1)) atomicAdd(&g2d[(int64_t)s_st[e].p * 9 + slot], tot * o);
      }
    }
  }
}

// ---- one wave per quadrant ------------------------------------------------------------------
// The same blend with a workgroup of four waves per 16x16 sub-tile, wave k taking quadrant k (one
// pixel per lane), for calls of few sub-tiles: there the time is that of one wave walking its list,
// entry after entry, and here a list is walked by four waves, each over the entries that reach
// its own quadrant only.  The four stage a batch together (one entry per thread, not compacted:
// a 64-bit mask per quadrant and 64 entries says which to walk).  A wave blends two entries at a
// time, whose alphas (and, in the adjoint, whose sums over the lanes) do not wait for each other, and
// reads the next two from LDS meanwhile.  Pixels see the operations of the kernels above in the same
// order, so the images, n_contrib and, up to the order of the sums, the gradients are the same.
// Entries one by one -> two at a time, us forward / backward: one view of 2k Gaussians at 128x128 21 -> 17
// / 40 -> 34; 20 views of 12k (7k and 5k appended) at 128x128 116 -> 90 / 179 -> 168.
constexpr int kQB = 256;  // threads per workgroup = entries per batch
constexpr float kLogNone = -1000.f;  // log2 of no opacity (alpha 0)

// The sub-tile of a workgroup.  All workgroups of such a call are on the CUs at once, so how long lists
// are spread over them counts: by_view views of one size are taken in turn for each sub-tile, since the
// crowded ones, mostly in the middle of each view, otherwise come in a stride that lands on the same CUs
// (20 views of 64 sub-tiles: 124 -> 116 us forward, 235 -> 179 backward).  One view, or views of several
// sizes: neighbours on the same XCD.
__device__ __forceinline__ int q_block(int w, int total, int per, int by_view) {
  if (by_view == 0) return xcd_logical(w, per);
  return w < total ? (w % by_view) * (total / by_view) + w / by_view : total;
}

// The next two of the 64 staged entries that mask m holds, in list order or against it, 64 (the entry
// of opacity 0) when there is none; taken from m.  The scalar find of a zero mask gives -1.
__device__ __forceinline__ int q_first(uint64_t& m) {
  int j;
  asm("s_ff1_i32_b64 %0, %1" : "=s"(j) : "s"(m));
  m &= ~(1ull << (j & 63));
  return (int)min((uint32_t)j, 64u);
}
__device__ __forceinline__ int q_last(uint64_t& m) {
  int j;
  asm("s_flbit_i32_b64 %0, %1" : "=s"(j) : "s"(m));
  j ^= 63;
  m &= ~(1ull << (j & 63));
  return (int)min((uint32_t)j, 64u);
}

template <bool L1>
__global__ __launch_bounds__(kQB) void k_blend_fwd_q(ViewsIO io, int nv, int total_blocks, int per, int by_view,
                                                     float bg0, float bg1, float bg2, const uint2* __restrict__ ranges,
                                                     const uint32_t* __restrict__ vals, const Rec* __restrict__ rec,
                                                     float* __restrict__ loss_slots) {
  __shared__ FwdStage s_st[4][65];  // [64]: an entry of opacity 0
  __shared__ uint64_t s_q[4][4];  // [quadrant][64 entries]
  const int lb = q_block(blockIdx.x, total_blocks, per, by_view);
  if (lb >= total_blocks) return;
  const int b = lb / io.sn, sub = lb - b * io.sn;
  const int v = view_of(io, nv, b);
  const ViewIO& V = io.v[v];
  const int t = b - V.tile_base;
  const int tx = t % V.TX, ty = t / V.TX;
  const int ox = tx * io.tw + (sub % io.sx) * 16, oy = ty * io.th + (sub / io.sx) * 16;
  if (ox >= V.W || oy >= V.H) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int k = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qx = lane & 7, qy = lane >> 3;
  const int px = ox + qx + 8 * (k & 1), py = oy + qy + 8 * (k >> 1);
  const float kx = (float)(8 * (k & 1)), ky = (float)(8 * (k >> 1));
  const float fx0 = (float)ox, fy0 = (float)oy;
  const uint2 r = ranges[b];
  if (r.y - r.x > (uint32_t)kPosMask) {
    if (tid == 0) atomicOr(io.err, kErrListTooLong);
    return;
  }
  if (lane == 0) {
    s_st[k][64].xy = make_float2(0.f, 0.f);
    s_st[k][64].co = make_float4(0.f, 0.f, 0.f, kLogNone);
    s_st[k][64].rgb = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  float T = 1.f, thr = (px < V.W && py < V.H) ? kAlphaMin : kNever, c0 = 0.f, c1 = 0.f, c2 = 0.f;
  uint32_t last = 0;
  bool alive = __ballot(thr < 1.f) != 0;  // uniform over the wave
  for (uint32_t start = r.x; start < r.y; start += kQB) {
    if (!__syncthreads_or(alive)) break;  // also: the batch before has been walked
    uint32_t qm = 0;
    if (start + tid < r.y) {
      const Rec R = rec[vals[start + tid]];
      const float2 xy = make_float2((R.r0.x - fx0) + R.r0.z, (R.r0.y - fy0) + R.r0.w);
      qm = quad_mask<2>(xy.x, xy.y, R.r1.x, R.r1.y, R.r1.z, R.r1.w);
      if (qm) {
        s_st[k][lane].xy = xy;
        s_st[k][lane].co = make_float4(-0.5f * kLog2e * R.r1.x, -kLog2e * R.r1.y, -0.5f * kLog2e * R.r1.z, __log2f(R.r1.w));
        s_st[k][lane].rgb = make_float4(R.r2.x, R.r2.y, R.r2.z, __uint_as_float((uint32_t)(start - r.x) + tid + 1));
      }
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const uint64_t m = __ballot((qm >> i) & 1u);
      if (lane == 0) s_q[i][k] = m;
    }
    __syncthreads();
    for (int g = 0; g < 4 && alive; g++) {
      const uint64_t mv = s_q[k][g];
      uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mv) |
                   ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(mv >> 32)) << 32);
      if (m == 0) continue;
      const FwdStage* st = s_st[g];
      int ja = q_first(m), jb = q_first(m);
      FwdStage A = st[ja], B = st[jb];
      auto blend2 = [&](const FwdStage& A, FwdStage& B) {
        // the operations of k_blend_fwd, the two alphas side by side
        float aa, ab;
        {
          const float dx = (A.xy.x - (float)qx) - kx, dy = (A.xy.y - (float)qy) - ky;
          const float pw = fmaf(dx, fmaf(A.co.x, dx, A.co.y * dy), fmaf(A.co.z * dy, dy, A.co.w));
          aa = fminf(kAlphaMax, __builtin_amdgcn_exp2f(pw));
        }
        {
          const float dx = (B.xy.x - (float)qx) - kx, dy = (B.xy.y - (float)qy) - ky;
          const float pw = fmaf(dx, fmaf(B.co.x, dx, B.co.y * dy), fmaf(B.co.z * dy, dy, B.co.w));
          ab = fminf(kAlphaMax, __builtin_amdgcn_exp2f(pw));
        }
        bool ta = aa >= thr, tb = ab >= thr;
        float wa = ta ? aa * T : 0.f;
        const float T1 = T - wa;
        float wb = tb ? ab * T1 : 0.f;
        const float T2 = T1 - wb;
        if (__builtin_expect(__ballot(T2 < kTStop) != 0, 0)) {  // T1 >= T2: some pixel stops at one of them
          const bool stop_a = T1 < kTStop;
          T = stop_a ? T1 + wa : T1;
          wa = stop_a ? 0.f : wa;
          ta = ta && !stop_a;
          thr = stop_a ? kNever : thr;
          // the quadrant's last pixel stopped at A: it does not see B, whose colour may be infinite
          if (__ballot(thr < 1.f) == 0) B.rgb.x = B.rgb.y = B.rgb.z = 0.f;
          tb = ab >= thr;
          wb = tb ? ab * T : 0.f;
          T -= wb;
          const bool stop_b = T < kTStop;
          T = stop_b ? T + wb : T;
          wb = stop_b ? 0.f : wb;
          tb = tb && !stop_b;
          thr = stop_b ? kNever : thr;
          alive = __ballot(thr < 1.f) != 0;
        } else {
          T = T2;
        }
        c0 = fmaf(B.rgb.x, wb, fmaf(A.rgb.x, wa, c0));
        c1 = fmaf(B.rgb.y, wb, fmaf(A.rgb.y, wa, c1));
        c2 = fmaf(B.rgb.z, wb, fmaf(A.rgb.z, wa, c2));
        last = ta ? __float_as_uint(A.rgb.w) : last;
        last = tb ? __float_as_uint(B.rgb.w) : last;
      };
      for (;;) {  // two pairs in turn: the next is read while one is blended
        bool more = m != 0;
        ja = q_first(m), jb = q_first(m);
        FwdStage An = st[ja], Bn = st[jb];
        blend2(A, B);
        if (!more || !alive) break;
        more = m != 0;
        ja = q_first(m), jb = q_first(m);
        A = st[ja];
        B = st[jb];
        blend2(An, Bn);
        if (!more || !alive) break;
      }
    }
  }
  float l1sum = 0.f;
  if (px < V.W && py < V.H) {
    const int64_t hw = (int64_t)V.W * V.H;
    const int64_t pix = (int64_t)py * V.W + px;
    const float col[3] = {c0 + T * bg0, c1 + T * bg1, c2 + T * bg2};
    if (!L1 || V.rgb) {
#pragma unroll
      for (int c = 0; c < 3; c++) V.rgb[c * hw + pix] = col[c];
    }
    V.t_final[pix] = T;
    V.n_contrib[pix] = (int)last;
    if (L1) {
      const float sc = V.l1_scale;
      float e = 0.f;
#pragma unroll
      for (int c = 0; c < 3; c++) {
        const float d = col[c] - V.target[c * hw + pix];
        V.dl_out[c * hw + pix] = d > 0.f ? sc : (d < 0.f ? -sc : 0.f);
        e += fabsf(d);
      }
      if (V.err) V.err[pix] = e * (1.0f / 3.0f);
      l1sum = e;
    }
  }
  if (L1) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) l1sum += __shfl_xor(l1sum, d, 64);
    if (lane == 0) atomicAdd(&loss_slots[(lb * 4 + k) % kLossSlots], l1sum * V.l1_scale);
  }
}

// The adjoint: an entry's nine sums over a quadrant are added to the batch's rows in LDS, and the
// batch's rows go to global memory once for the four quadrants.
__global__ __launch_bounds__(kQB) void k_blend_bwd_q(ViewsIO io, int nv, int total_blocks, int per, int by_view,
                                                     float bg0, float bg1, float bg2, const uint2* __restrict__ ranges,
                                                     const uint32_t* __restrict__ vals, const Rec* __restrict__ rec,
                                                     float* __restrict__ g2d) {
  __shared__ BwdStage s_st[4][65];  // [64]: an entry of opacity 0
  __shared__ float s_acc[kQB * 9];
  __shared__ uint64_t s_q[4][4];
  __shared__ int s_last[4];
  const int lb = q_block(blockIdx.x, total_blocks, per, by_view);
  if (lb >= total_blocks) return;
  const int b = lb / io.sn, sub = lb - b * io.sn;
  const int v = view_of(io, nv, b);
  const ViewIO& V = io.v[v];
  const int t = b - V.tile_base;
  const int tx = t % V.TX, ty = t / V.TX;
  const int ox = tx * io.tw + (sub % io.sx) * 16, oy = ty * io.th + (sub / io.sx) * 16;
  if (ox >= V.W || oy >= V.H) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int k = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qx = lane & 7, qy = lane >> 3;
  const int px = ox + qx + 8 * (k & 1), py = oy + qy + 8 * (k >> 1);
  const float kx = (float)(8 * (k & 1)), ky = (float)(8 * (k >> 1));
  const float fx0 = (float)ox, fy0 = (float)oy;
  const uint2 r = ranges[b];
  if (r.y - r.x > (uint32_t)kPosMask) return;
  const int64_t hw = (int64_t)V.W * V.H;
  if (lane == 0) {
    s_st[k][64].xy = make_float2(0.f, 0.f);
    s_st[k][64].co = make_float4(0.f, 0.f, 0.f, kLogNone);
    s_st[k][64].rgb = make_float4(0.f, 0.f, 0.f, 0.f);
    s_st[k][64].io = 0.f;
  }
  float T = 1.f, dC0 = 0.f, dC1 = 0.f, dC2 = 0.f;
  int last = 0;
  if (px < V.W && py < V.H) {
    const int64_t pix = (int64_t)py * V.W + px;
    T = V.t_final[pix];
    last = V.n_contrib[pix];
    dC0 = V.dl[pix];
    dC1 = V.dl[hw + pix];
    dC2 = V.dl[2 * hw + pix];
  }
  float nS = -(bg0 * dC0 + bg1 * dC1 + bg2 * dC2);
  int mx = last;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) mx = max(mx, __shfl_xor(mx, d, 64));
  if (lane == 0) s_last[k] = mx;
  __syncthreads();
  int qlast[4], max_all = 0;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    qlast[i] = s_last[i];
    max_all = max(max_all, qlast[i]);
  }
  const int max_last = __builtin_amdgcn_readfirstlane(min(max_all, (int)(r.y - r.x)));
  if (max_last <= 0) return;  // uniform over the workgroup
  const int slot = kRedSlot[(lane >> 1) & 15];
  const bool writes = (lane & 1) == 0 && slot >= 0, odd = (lane & 2) != 0;
  for (int bi = (max_last + kQB - 1) / kQB - 1; bi >= 0; bi--) {
    const int idx0 = bi * kQB;
    uint32_t qm = 0;
    if (idx0 + tid < max_last) {
      const uint32_t p = vals[r.x + (uint32_t)(idx0 + tid)];
      const Rec R = rec[p];
      const float2 xy = make_float2((R.r0.x - fx0) + R.r0.z, (R.r0.y - fy0) + R.r0.w);
      const float4 cn = R.r1;
      qm = quad_mask<2>(xy.x, xy.y, cn.x, cn.y, cn.z, cn.w);
#pragma unroll
      for (int i = 0; i < 4; i++)
        if (idx0 + tid >= qlast[i]) qm &= ~(1u << i);
      if (qm) {
        s_st[k][lane].xy = xy;
        s_st[k][lane].co = make_float4(-0.5f * kLog2e * cn.x, -kLog2e * cn.y, -0.5f * kLog2e * cn.z, __log2f(cn.w));
        const bool inf = !(fabsf(R.r2.x) + fabsf(R.r2.y) + fabsf(R.r2.z) < INFINITY);
        s_st[k][lane].rgb = make_float4(R.r2.x, R.r2.y, R.r2.z,
                                        __uint_as_float((cn.w >= kAlphaMax ? kClampBit : 0u) | (inf ? kInfBit : 0u)));
        s_st[k][lane].p = p;
        s_st[k][lane].io = 1.0f / cn.w;
      }
    }
#pragma unroll
    for (int i = 0; i < 9; i++) s_acc[i * kQB + tid] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const uint64_t m = __ballot((qm >> i) & 1u);
      if (lane == 0) s_q[i][k] = m;
    }
    __syncthreads();
    for (int g = 3; g >= 0; g--) {
      const uint64_t mv = s_q[k][g];
      uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mv) |
                   ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(mv >> 32)) << 32);
      if (m == 0) continue;
      const BwdStage* st = s_st[g];
      int ja = q_last(m), jb = q_last(m);
      BwdStage A = st[ja], B = st[jb];
      auto blend2 = [&](BwdStage& A, BwdStage& B, int pa, int pb) {
        // the operations of k_blend_bwd, the two alphas side by side
        const float dxa = (A.xy.x - (float)qx) - kx, dya = (A.xy.y - (float)qy) - ky;
        const float dxb = (B.xy.x - (float)qx) - kx, dyb = (B.xy.y - (float)qy) - ky;
        const float ra = __builtin_amdgcn_exp2f(
            fmaf(dxa, fmaf(A.co.x, dxa, A.co.y * dya), fmaf(A.co.z * dya, dya, A.co.w)));
        const float rb = __builtin_amdgcn_exp2f(
            fmaf(dxb, fmaf(B.co.x, dxb, B.co.y * dyb), fmaf(B.co.z * dyb, dyb, B.co.w)));
        const float aa = fminf(kAlphaMax, ra), ab = fminf(kAlphaMax, rb);
        const bool ta = (idx0 + g * 64 + pa < last) && (aa >= kAlphaMin);
        const bool tb = (idx0 + g * 64 + pb < last) && (ab >= kAlphaMin);
        const uint64_t ma = __ballot(ta), mb = __ballot(tb);
        if ((ma | mb) != 0) {
          const uint32_t wab = (uint32_t)__builtin_amdgcn_readfirstlane(
              (int)(__float_as_uint(A.rgb.w) | __float_as_uint(B.rgb.w)));
          // an entry that no pixel takes adds nothing, also where a product with its 0 is no number
          if (__builtin_expect((wab & kInfBit) != 0, 0)) {  // uniform, rare
            __asm__ volatile("");
            if (ma == 0) A.rgb.x = A.rgb.y = A.rgb.z = 0.f;
            if (mb == 0) B.rgb.x = B.rgb.y = B.rgb.z = 0.f;
          }
          const float ea = ta ? aa : 0.f, eb = tb ? ab : 0.f;
          const float ia = __builtin_amdgcn_rcpf(1.f - ea), ib = __builtin_amdgcn_rcpf(1.f - eb);
          const float Ta = T * ia;
          T = Ta * ib;
          const float wa = ea * Ta, wb = eb * T;
          const float da = fmaf(A.rgb.x, dC0, fmaf(A.rgb.y, dC1, fmaf(A.rgb.z, dC2, nS)));
          nS = fmaf(-ea, da, nS);
          const float db = fmaf(B.rgb.x, dC0, fmaf(B.rgb.y, dC1, fmaf(B.rgb.z, dC2, nS)));
          nS = fmaf(-eb, db, nS);
          float Pa = wa * da, Pb = wb * db;
          if (__builtin_expect((wab & kClampBit) != 0, 0)) {  // uniform, rare
            __asm__ volatile("");
            if (__float_as_uint(A.rgb.w) & kClampBit) Pa = ra < kAlphaMax ? Pa : 0.f;
            if (__float_as_uint(B.rgb.w) & kClampBit) Pb = rb < kAlphaMax ? Pb : 0.f;
          }
          const float xa = Pa * dxa, ya = Pa * dya, xb = Pb * dxb, yb = Pb * dyb;
          const float sa[9] = {xa, ya, xa * dxa, xa * dya, ya * dya, Pa * A.io, wa * dC0, wa * dC1, wa * dC2};
          const float sb[9] = {xb, yb, xb * dxb, xb * dyb, yb * dyb, Pb * B.io, wb * dC0, wb * dC1, wb * dC2};
          const float tot = wave_reduce18(sa, sb, odd);
          const int pos = lane < 32 ? (ma != 0 ? pa : 64) : (mb != 0 ? pb : 64);
          if (writes && pos < 64) atomicAdd(&s_acc[(g * 64 + pos) * 9 + slot], tot);
        }
      };
      for (;;) {
        bool more = m != 0;
        int pa = ja, pb = jb;
        ja = q_last(m), jb = q_last(m);
        BwdStage An = st[ja], Bn = st[jb];
        blend2(A, B, pa, pb);
        if (!more) break;
        more = m != 0;
        pa = ja, pb = jb;
        ja = q_last(m), jb = q_last(m);
        A = st[ja];
        B = st[jb];
        blend2(An, Bn, pa, pb);
        if (!more) break;
      }
    }
    __syncthreads();
    // nine consecutive threads per entry: one 36-byte row
#pragma unroll 1
    for (int i = 0; i < 9; i++) {
      const int x = i * kQB + tid;
      const float val = s_acc[x];
      if (val != 0.f) atomicAdd(&g2d[(int64_t)s_st[x / 9 / 64][x / 9 % 64].p * 9 + x % 9], val);
    }
    __syncthreads();
  }
}

// Identity-feature render of 16x16 sub-tiles: the forward's walk (same lists, culling, alpha,
// transmittance and stop, so the weights alpha_i T_i are the colour render's) accumulating up to
// kFeatMaxC per-Gaussian features instead of colours, with no background.
//
// The accumulation is an outer product of a quadrant's 64 weights and the entry's 16 features and runs on
// the matrix cores in fp32: v_mfma_f32_16x16x1 in four blocks of 16 pixels x 16 channels takes the weights
// as the walk leaves them, one pixel per lane, and one feature of the entry per lane, in place of 16
// multiply-adds per (entry, quadrant) with the same rounding.  A workgroup is two waves of two
// quadrants each, staging 128 entries together: six waves to a SIMD, four with all quadrants in one wave
// (their 64 sums).  The bound of six also keeps the sums in place: without it the compiler moves them
// between two register files around each product.  20 views of 200k Gaussians at 1352x1014, 16 channels:
// 1805 us with multiply-adds, 1700 with four quadrants to a wave, 1710 with four 4x4x1 products of 4
// channels, 1655 so.  Of the SIMDs' quad-cycles 52 % issue vector instructions (6.3e8 beside the products,
// the colour forward 6.8e8, in 79 % of its own), the matrix cores are busy in 28 %, and at least a fifth
// has neither: the waves, 5.4 to a SIMD where the forward has 6.9, wait 44 % of their time for the
// staging's loads and the barriers of the two.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kFeatThreads = 128;  // = entries per batch
static_assert(kFeatMaxC == 16, "a product takes 16 channels");

__global__ __launch_bounds__(kFeatThreads, 6) void k_blend_feat_h(ViewsIO io, int nv, int total_blocks, int per, FeatIO fo,
                                                               const uint2* __restrict__ ranges,
                                                               const uint32_t* __restrict__ vals,
                                                               const Rec* __restrict__ rec) {
  __shared__ float2 s_xy[kFeatThreads];
  __shared__ float4 s_co[kFeatThreads];
  __shared__ uint32_t s_g[kFeatThreads];  // Gaussian, ~0: not kept
  __shared__ float4 s_f[kFeatThreads][kFeatMaxC / 4];
  __shared__ uint64_t s_q[4][2];  // [quadrant][64 entries]
  const int lb = xcd_logical(blockIdx.x, per);
  if (lb >= total_blocks) return;
  const int b = lb / io.sn, sub = lb - b * io.sn;
  const int v = view_of(io, nv, b);
  const ViewIO& V = io.v[v];
  const int t = b - V.tile_base;
  const int tx = t % V.TX, ty = t / V.TX;
  const int ox = tx * io.tw + (sub % io.sx) * 16, oy = ty * io.th + (sub / io.sx) * 16;
  if (ox >= V.W || oy >= V.H) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // quadrants 2 w and 2 w + 1
  const int qx = lane & 7, qy = lane >> 3;
  const float ky = (float)(8 * w);
  const float fx0 = (float)ox, fy0 = (float)oy;
  const uint2 r = ranges[b];
  if (r.y - r.x > (uint32_t)kPosMask) return;  // the colour forward reported it
  const uint32_t gbase = (uint32_t)v * (uint32_t)fo.n;  // record index = view * n + Gaussian
  float T[2], thr[2];  // thr: as the colour forward's
  f32x16 acc[2];       // [quadrant]: lane l, element 4 b + i = channel l % 16 of the quadrant's pixel 16 b + 4 (l / 16) + i
  bool alive[2];       // uniform over the wave
#pragma unroll
  for (int k = 0; k < 2; k++) {
    T[k] = 1.f;
    thr[k] = (ox + qx + 8 * k < V.W && oy + qy + 8 * w < V.H) ? kAlphaMin : kNever;
    alive[k] = __ballot(thr[k] < 1.f) != 0;
#pragma unroll
    for (int c = 0; c < 16; c++) acc[k][c] = 0.f;
  }
  for (uint32_t start = r.x; start < r.y; start += kFeatThreads) {
    if (!__syncthreads_or(alive[0] || alive[1])) break;  // also: the batch before has been walked
    uint32_t qm = 0, rid = 0;
    if (start + tid < r.y) {
      rid = vals[start + tid];
      const Rec R = rec[rid];
      const float2 xy = make_float2((R.r0.x - fx0) + R.r0.z, (R.r0.y - fy0) + R.r0.w);
      qm = quad_mask<2>(xy.x, xy.y, R.r1.x, R.r1.y, R.r1.z, R.r1.w);
      if (qm) {
        s_xy[tid] = xy;
        s_co[tid] = make_float4(-0.5f * kLog2e * R.r1.x, -kLog2e * R.r1.y, -0.5f * kLog2e * R.r1.z, __log2f(R.r1.w));
      }
    }
    s_g[tid] = qm ? rid - gbase : ~0u;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const uint64_t m = __ballot((qm >> i) & 1u);
      if (lane == 0) s_q[i][w] = m;
    }
    __syncthreads();
    // the kept entries' features (Gaussian-major copy: one 64-byte row each), four lanes per row
#pragma unroll
    for (int i = 0; i < kFeatMaxC / 4; i++) {
      const int e = i * (kFeatThreads / 4) + (tid >> 2);
      const uint32_t g = s_g[e];
      if (g != ~0u) s_f[e][tid & 3] = reinterpret_cast<const float4*>(fo.feat16)[(size_t)g * (kFeatMaxC / 4) + (tid & 3)];
    }
    __syncthreads();
    for (int g = 0; g < 2; g++) {
      uint64_t m[2];
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const uint64_t mv = s_q[2 * w + k][g];
        m[k] = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mv) |
               ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(mv >> 32)) << 32);
        if (!alive[k]) m[k] = 0;
      }
      while ((m[0] | m[1]) != 0) {
        const int j = (int)__builtin_ctzll(m[0] | m[1]);
        const int e = g * 64 + j;
        const float2 xy = s_xy[e];
        const float4 co = s_co[e];
        const float fe = reinterpret_cast<const float*>(s_f[e])[lane & 15];
        const float dxb = xy.x - (float)qx, dy = (xy.y - (float)qy) - ky;
#pragma unroll
        for (int k = 0; k < 2; k++) {
          if (!((m[k] >> j) & 1ull)) continue;  // uniform
          m[k] &= ~(1ull << j);
          const float dx = dxb - (float)(8 * k);
          // the colour forward's alpha, weight and stop, operation for operation
          const float pw = fmaf(dx, fmaf(co.x, dx, co.y * dy), fmaf(co.z * dy, dy, co.w));
          const float a = fminf(kAlphaMax, __builtin_amdgcn_exp2f(pw));
          const bool ok = a >= thr[k];
          float wgt = ok ? a * T[k] : 0.f;
          T[k] -= wgt;
          const bool stop = T[k] < kTStop;
          if (__builtin_expect(__ballot(stop) != 0, 0)) {  // uniform: a pixel of the quadrant stops here
            T[k] = stop ? T[k] + wgt : T[k];
            wgt = stop ? 0.f : wgt;
            thr[k] = stop ? kNever : thr[k];
            alive[k] = __ballot(thr[k] < 1.f) != 0;
            if (!alive[k]) m[k] = 0;
          }
          acc[k] = __builtin_amdgcn_mfma_f32_16x16x1f32(wgt, fe, acc[k], 0, 0, 0);
        }
      }
    }
  }
  float* __restrict__ out = fo.out[v];
  const int64_t hw = (int64_t)V.W * V.H;
  // four pixels of a row at once where every row of every plane starts on 16 bytes
  const bool wide = (V.W & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  const int ch = lane & 15;
  if (ch >= fo.C) return;
#pragma unroll
  for (int k = 0; k < 2; k++) {
#pragma unroll
    for (int b4 = 0; b4 < 4; b4++) {
      const int q = 16 * b4 + 4 * (lane >> 4);  // pixel of the quadrant (row-major, 8 wide)
      const int px = ox + 8 * k + (q & 7), py = oy + 8 * w + (q >> 3);
      if (py >= V.H || px >= V.W) continue;
      float* __restrict__ o = out + ch * hw + (int64_t)py * V.W + px;
      if (wide) {
        *reinterpret_cast<f32x4*>(o) = f32x4{acc[k][4 * b4], acc[k][4 * b4 + 1], acc[k][4 * b4 + 2], acc[k][4 * b4 + 3]};
      } else {
#pragma unroll
        for (int i = 0; i < 4; i++)
          if (px + i < V.W) o[i] = acc[k][4 * b4 + i];
      }
    }
  }
}

// The same for 8x8 sub-tiles, one wave each, by multiply-adds.
template <int SUB, int B>
__global__ __launch_bounds__(kLanes) void k_blend_feat(ViewsIO io, int nv, int total_blocks, int per, FeatIO fo,
                                                       const uint2* __restrict__ ranges,
                                                       const uint32_t* __restrict__ vals, const Rec* __restrict__ rec) {
  constexpr int PW = SUB / 8, NP = PW * PW;
  __shared__ float2 s_xy[B];
  __shared__ float4 s_co[B];
  __shared__ uint32_t s_qm[B];
  __shared__ float4 s_f[B][kFeatMaxC / 4];
  const int lb = xcd_logical(blockIdx.x, per);
  if (lb >= total_blocks) return;
  const int b = lb / io.sn, sub = lb - b * io.sn;
  const int v = view_of(io, nv, b);
  const ViewIO& V = io.v[v];
  const int t = b - V.tile_base;
  const int tx = t % V.TX, ty = t / V.TX;
  const int ox = tx * io.tw + (sub % io.sx) * SUB, oy = ty * io.th + (sub / io.sx) * SUB;
  if (ox >= V.W || oy >= V.H) return;
  const int lane = threadIdx.x;
  const int qx = lane & 7, qy = lane >> 3;
  const float fx0 = (float)ox, fy0 = (float)oy;
  const uint64_t lt = lane_lt_mask(lane);
  const uint2 r = ranges[b];
  if (r.y - r.x > (uint32_t)kPosMask) return;  // the colour forward reported it
  const uint32_t gbase = (uint32_t)v * (uint32_t)fo.n;  // record index = view * n + Gaussian
  float T[NP], thr[NP], acc[NP][kFeatMaxC];  // thr: as the colour forward's
#pragma unroll
  for (int k = 0; k < NP; k++) {
    const int px = ox + qx + 8 * (k % PW), py = oy + qy + 8 * (k / PW);
    T[k] = 1.f;
    thr[k] = (px < V.W && py < V.H) ? kAlphaMin : kNever;
#pragma unroll
    for (int c = 0; c < kFeatMaxC; c++) acc[k][c] = 0.f;
  }
  for (uint32_t start = r.x; start < r.y; start += B) {
    const int n_in = (int)min((uint32_t)B, r.y - start);
    int n_kept = 0;
#pragma unroll
    for (int k = 0; k < B / kLanes; k++) {
      const int e = k * kLanes + lane;
      uint32_t qm = 0, rid = 0;
      float2 xy;
      float4 co;
      if (e < n_in) {
        rid = vals[start + e];
        const Rec R = rec[rid];
        xy = make_float2((R.r0.x - fx0) + R.r0.z, (R.r0.y - fy0) + R.r0.w);
        qm = quad_mask<PW>(xy.x, xy.y, R.r1.x, R.r1.y, R.r1.z, R.r1.w);
        co = make_float4(-0.5f * kLog2e * R.r1.x, -kLog2e * R.r1.y, -0.5f * kLog2e * R.r1.z, __log2f(R.r1.w));
      }
      const bool keep = qm != 0;
      const uint64_t m = __ballot(keep);
      if (keep) {
        const int pos = n_kept + __popcll(m & lt);
        s_xy[pos] = xy;
        s_co[pos] = co;
        s_qm[pos] = qm;
        // Gaussian-major copy: one 64-byte row per entry
        const float4* __restrict__ f = reinterpret_cast<const float4*>(fo.feat16) + (size_t)(rid - gbase) * (kFeatMaxC / 4);
#pragma unroll
        for (int c = 0; c < kFeatMaxC / 4; c++) s_f[pos][c] = f[c];
      }
      n_kept += __popcll(m);
    }
    uint32_t qalive = 0;
#pragma unroll
    for (int k = 0; k < NP; k++) qalive |= __ballot(thr[k] < 1.f) != 0 ? 1u << k : 0u;
    __syncthreads();
    for (int j = 0; j < n_kept && qalive != 0; j++) {
      const float2 xy = s_xy[j];
      const float4 co = s_co[j];
      const uint32_t qm = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_qm[j]) & qalive;
      const float dxb = xy.x - (float)qx, dyb = xy.y - (float)qy;
      float4 fe[kFeatMaxC / 4];
#pragma unroll
      for (int c = 0; c < kFeatMaxC / 4; c++) fe[c] = s_f[j][c];
#pragma unroll
      for (int k = 0; k < NP; k++) {
        if (NP > 1 && !((qm >> k) & 1u)) continue;
        const float dx = dxb - (float)(8 * (k % PW)), dy = dyb - (float)(8 * (k / PW));
        // the colour forward's alpha, weight and stop, operation for operation
        const float pw = fmaf(dx, fmaf(co.x, dx, co.y * dy), fmaf(co.z * dy, dy, co.w));
        const float a = fminf(kAlphaMax, __builtin_amdgcn_exp2f(pw));
        const bool ok = a >= thr[k];
        float wgt = ok ? a * T[k] : 0.f;
        T[k] -= wgt;
        const bool stop = T[k] < kTStop;  // as the colour forward's: only a passing pixel can cross it
        if (__builtin_expect(__ballot(stop) != 0, 0)) {  // uniform: a pixel of the quadrant stops here
          T[k] = stop ? T[k] + wgt : T[k];
          wgt = stop ? 0.f : wgt;
          thr[k] = stop ? kNever : thr[k];
          if (__ballot(thr[k] < 1.f) == 0) qalive &= ~(1u << k);
        }
#pragma unroll
        for (int c = 0; c < kFeatMaxC / 4; c++) {
          acc[k][4 * c] += fe[c].x * wgt;
          acc[k][4 * c + 1] += fe[c].y * wgt;
          acc[k][4 * c + 2] += fe[c].z * wgt;
          acc[k][4 * c + 3] += fe[c].w * wgt;
        }
      }
    }
    bool alive = false;
#pragma unroll
    for (int k = 0; k < NP; k++) alive = alive || thr[k] < 1.f;
    if (__ballot(alive) == 0) break;
    __syncthreads();
  }
  float* __restrict__ out = fo.out[v];
#pragma unroll
  for (int k = 0; k < NP; k++) {
    const int px = ox + qx + 8 * (k % PW), py = oy + qy + 8 * (k / PW);
    if (px < V.W && py < V.H) {
      const int64_t hw = (int64_t)V.W * V.H;
      const int64_t pix = (int64_t)py * V.W + px;
#pragma unroll
      for (int c = 0; c < kFeatMaxC; c++)
        if (c < fo.C) out[c * hw + pix] = acc[k][c];
    }
  }
}

__global__ void k_debug_keys(uint32_t tile, uint32_t row0, const uint32_t* __restrict__ vals,
                             const Rec* __restrict__ rec, uint32_t lo, uint32_t cnt, uint64_t* __restrict__ kout,
                             uint32_t* __restrict__ vout) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cnt) return;
  const uint32_t p = vals[lo + i];  // record index of the view's Gaussian
  kout[i] = ((uint64_t)tile << 32) | (uint64_t)__float_as_uint(rec[p].r2.w);
  vout[i] = p - row0;
}

}  // namespace

void launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  k_fill_u32<<<(unsigned)blocks, 256, 0, st>>>(p, v, n);
}

// The number of views if there are several and all have as many tiles, else 0.
static inline int views_alike(const ViewsIO& io, int nv, int64_t total_tiles) {
  if (nv < 2 || total_tiles % nv) return 0;
  for (int v = 1; v < nv; v++)
    if (io.v[v].tile_base != v * (total_tiles / nv)) return 0;
  return nv;
}

// Whether a call's 16x16 sub-tiles are walked by one wave per quadrant: up to where the chip's 1,024 SIMDs
// hold about ten (forward) or four (backward) of the four-quadrant waves each, so the longest list sets the
// time.  The backward's line lies lower for one view (or views of several sizes), whose crowded middle is on
// few XCDs, and wide footprints, whose lists are alike.  Times of the call in us, one quadrant per wave /
// four: forward (one view; frustum scene of narrow footprints, or wide ones of about 200 pixels, 100k
// Gaussians), 5,632 sub-tiles 174 / 188, 249 / 295 wide; 8,160 200 / 208, 280 / 325; 10,240 213 / 218, 319 /
// 365 (20k narrow ones 119 / 114); forward and backward, 1,024 narrow 322 / 419, wide 437 / 522; 3,072 352 /
// 359, 490 / 554; 3,584 386 / 397, 632 / 595 (500k: 545 / 642, 784 / 796); 4,032 392 / 391, 553 / 557 (20k
// wide 456 / 416); 4,096 412 / 414, 773 / 641; 4,800 420 / 394, 544 / 535; 16 views of 256 sub-tiles
// each 904 / 1040, 842 / 923.
constexpr int64_t kByQuadrantFwd = 10240, kByQuadrantBwd = 4096, kByQuadrantBwdOne = 3600;
static inline bool by_quadrant(const ViewsIO& io, int64_t sub_tiles, int64_t most) {
  return io.sub == 16 && sub_tiles <= most;
}

static inline int per_xcd(int64_t total_tiles) { return (int)((total_tiles + kNumXcd - 1) / kNumXcd); }

// One wave per (tile, sub-tile); the sub-tiles of a tile are consecutive logical blocks, so they
// run on the same XCD and share its L2 for the tile's list and records.
template <bool COUNT, bool L1, int B>
void blend_fwd_batch(const ViewsIO& io, int nv, int total, int per, const float bg[3], const Workspace& ws,
                     hipStream_t st) {
  const dim3 grid(per * kNumXcd), block(kLanes);
  if (io.sub == 8)
    k_blend_fwd<COUNT, L1, 8, B><<<grid, block, 0, st>>>(io, nv, total, per, bg[0], bg[1], bg[2], ws.ranges, ws.vals,
                                                        ws.rec_u, ws.pairs, ws.loss_slots);
  else
    k_blend_fwd<COUNT, L1, 16, B><<<grid, block, 0, st>>>(io, nv, total, per, bg[0], bg[1], bg[2], ws.ranges, ws.vals,
                                                         ws.rec_u, ws.pairs, ws.loss_slots);
}

template <bool COUNT, bool L1>
void blend_fwd_variant(const ViewsIO& io, int nv, int total, int per, const float bg[3], const Workspace& ws,
                       hipStream_t st) {
  if (io.batch == 64)
    blend_fwd_batch<COUNT, L1, 64>(io, nv, total, per, bg, ws, st);
  else if (io.batch == 256)
    blend_fwd_batch<COUNT, L1, 256>(io, nv, total, per, bg, ws, st);
  else
    blend_fwd_batch<COUNT, L1, 128>(io, nv, total, per, bg, ws, st);
}

void launch_blend_fwd(const ViewsIO& io, int nv, int64_t total_tiles, const float bg[3], const Workspace& ws,
                      bool count_pairs, bool l1, hipStream_t st) {
  const int64_t total = total_tiles * io.sn;
  if (total == 0) return;
  const int per = per_xcd(total);
  ViewsIO iov = io;
  iov.err = ws.err;
  if (by_quadrant(io, total, kByQuadrantFwd) && !count_pairs) {
    const dim3 grid(per * kNumXcd);
    const int alike = views_alike(io, nv, total_tiles);
    if (l1)
      k_blend_fwd_q<true><<<grid, kQB, 0, st>>>(iov, nv, (int)total, per, alike, bg[0], bg[1], bg[2], ws.ranges, ws.vals,
                                                ws.rec_u, ws.loss_slots);
    else
      k_blend_fwd_q<false><<<grid, kQB, 0, st>>>(iov, nv, (int)total, per, alike, bg[0], bg[1], bg[2], ws.ranges,
                                                 ws.vals, ws.rec_u, ws.loss_slots);
    return;
  }
  if (count_pairs) {
    if (l1)
      blend_fwd_variant<true, true>(iov, nv, (int)total, per, bg, ws, st);
    else
      blend_fwd_variant<true, false>(iov, nv, (int)total, per, bg, ws, st);
  } else {
    if (l1)
      blend_fwd_variant<false, true>(iov, nv, (int)total, per, bg, ws, st);
    else
      blend_fwd_variant<false, false>(iov, nv, (int)total, per, bg, ws, st);
  }
}

// features [C][stride] -> Gaussian-major rows of kFeatMaxC floats (zeros beyond C)
__global__ __launch_bounds__(256) void k_feat_rows(const float* __restrict__ feat, int64_t stride, int C, int n,
                                                   float4* __restrict__ rows) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g >= n) return;
  float v[kFeatMaxC];
#pragma unroll
  for (int c = 0; c < kFeatMaxC; c++) v[c] = c < C ? feat[c * stride + g] : 0.f;
#pragma unroll
  for (int c = 0; c < kFeatMaxC / 4; c++)
    rows[(size_t)g * (kFeatMaxC / 4) + c] = make_float4(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
}

void launch_blend_feat(const ViewsIO& io, int nv, int64_t total_tiles, const FeatIO& fo, const Workspace& ws,
                       hipStream_t st) {
  if (fo.n > 0)
    k_feat_rows<<<(fo.n + 255) / 256, 256, 0, st>>>(fo.feat, fo.stride, fo.C, fo.n, reinterpret_cast<float4*>(fo.feat16));
  const int64_t total = total_tiles * io.sn;
  if (total == 0) return;
  const int per = per_xcd(total);
  const dim3 grid(per * kNumXcd), block(kLanes);
#define DASS_FEAT(SUBT, BT) k_blend_feat<SUBT, BT><<<grid, block, 0, st>>>(io, nv, (int)total, per, fo, ws.ranges, ws.vals, ws.rec_u)
  if (io.sub == 8) {
    if (io.batch == 64) DASS_FEAT(8, 64);
    else if (io.batch == 256) DASS_FEAT(8, 256);
    else DASS_FEAT(8, 128);
  } else {
    k_blend_feat_h<<<grid, kFeatThreads, 0, st>>>(io, nv, (int)total, per, fo, ws.ranges, ws.vals, ws.rec_u);
  }
#undef DASS_FEAT
}

__global__ __launch_bounds__(256) void k_loss_finish(float* __restrict__ slots, float* __restrict__ loss, float add) {
  __shared__ float s_w[4];
  float acc = 0.f;
  for (int i = threadIdx.x; i < kLossSlots; i += 256) {
    acc += slots[i];
    slots[i] = 0.f;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0 && loss) *loss += ((s_w[0] + s_w[1]) + (s_w[2] + s_w[3])) + add;
}

void launch_loss_finish(float* slots, float* loss, float add, hipStream_t st) {
  k_loss_finish<<<1, 256, 0, st>>>(slots, loss, add);
}

void launch_blend_bwd(const ViewsIO& io, int nv, int64_t total_tiles, const float bg[3], const Workspace& ws,
                      hipStream_t st) {
  const int64_t total = total_tiles * io.sn;
  if (total == 0) return;
  const int per = per_xcd(total);
  const dim3 grid(per * kNumXcd), block(kLanes);
  const int alike = views_alike(io, nv, total_tiles);
  if (by_quadrant(io, total, alike ? kByQuadrantBwd : kByQuadrantBwdOne)) {
    k_blend_bwd_q<<<grid, kQB, 0, st>>>(io, nv, (int)total, per, alike, bg[0], bg[1], bg[2], ws.ranges, ws.vals, ws.rec_u,
                                        ws.g2d);
    return;
  }
#define DASS_BWD(SUBT, BT)                                                                                     \
  k_blend_bwd<SUBT, BT><<<grid, block, 0, st>>>(io, nv, (int)total, per, bg[0], bg[1], bg[2], ws.ranges, ws.vals, \
                                                ws.rec_u, ws.g2d)
  if (io.sub == 8) {
    if (io.batch == 64) DASS_BWD(8, 64);
    else if (io.batch == 256) DASS_BWD(8, 256);
    else DASS_BWD(8, 128);
  } else {
    if (io.batch == 64) DASS_BWD(16, 64);
    else if (io.batch == 256) DASS_BWD(16, 256);
    else DASS_BWD(16, 128);
  }
#undef DASS_BWD
}

void launch_debug_keys(int view, int n, const Workspace& ws, uint32_t tile, uint32_t lo, uint32_t cnt, uint64_t* kout,
                       uint32_t* vout, hipStream_t st) {
  if (cnt > 0)
    k_debug_keys<<<(cnt + 255) / 256, 256, 0, st>>>(tile, (uint32_t)((int64_t)view * n), ws.vals, ws.rec_u, lo, cnt,
                                                     kout, vout);
}

}  // namespace dass
