// Per-iteration updates around the rasterizer: dynamics-aware shift (Sec. 3.3) and its
// adjoint, a multi-tensor Adam step, the L1 fidelity gradient with the error map (Sec. 3.4),
// and error-guided densification (Sec. 3.4, Alg. 1, Eq. 4).  All are memory-bound
// elementwise passes; each is one launch over all of its groups / views.
#include <algorithm>

#include "dass_internal.h"

namespace dass {
namespace {

// Hamilton product (w, x, y, z).
__device__ __forceinline__ void qmul(const double* a, const double* b, double* o) {
  o[0] = a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3];
  o[1] = a[0] * b[1] + a[1] * b[0] + a[2] * b[3] - a[3] * b[2];
  o[2] = a[0] * b[2] - a[1] * b[3] + a[2] * b[0] + a[3] * b[1];
  o[3] = a[0] * b[3] + a[1] * b[2] - a[2] * b[1] + a[3] * b[0];
}

__global__ __launch_bounds__(256) void k_copy_mq(const float* __restrict__ mean, const float* __restrict__ quat,
                                                 float* __restrict__ om, float* __restrict__ oq, int n, int stride) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  for (int i = 0; i < 3; i++) om[(int64_t)i * stride + g] = mean[(int64_t)i * stride + g];
  for (int i = 0; i < 4; i++) oq[(int64_t)i * stride + g] = quat[(int64_t)i * stride + g];
}

__global__ __launch_bounds__(256) void k_shift_fwd(const float* __restrict__ mean, const float* __restrict__ quat,
                                                   float* __restrict__ om, float* __restrict__ oq, int stride, int n,
                                                   const int32_t* __restrict__ idx, int n_dyn,
                                                   const float* __restrict__ dpos, const float* __restrict__ drot) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_dyn) return;
  const int64_t g = idx[j];
  if (g < 0 || g >= n) return;  // out-of-range index: ignored
  double q[4], s[4], o[4], qn = 0.0, sn = 0.0;
  for (int i = 0; i < 4; i++) {
    q[i] = quat[i * (int64_t)stride + g];
    s[i] = drot[(int64_t)i * n_dyn + j];
    qn += q[i] * q[i];
    sn += s[i] * s[i];
  }
  const double iq = 1.0 / sqrt(qn), is = 1.0 / sqrt(sn);
  for (int i = 0; i < 4; i++) { q[i] *= iq; s[i] *= is; }
  qmul(q, s, o);
  for (int i = 0; i < 3; i++)
    om[i * (int64_t)stride + g] = (float)((double)mean[i * (int64_t)stride + g] + (double)dpos[(int64_t)i * n_dyn + j]);
  for (int i = 0; i < 4; i++) oq[i * (int64_t)stride + g] = (float)o[i];
}

// d sigma_hat = L(q_hat)^T dq' = conj(q_hat) (x) dq'; then back through sigma_hat = sigma/|sigma|.
__global__ __launch_bounds__(256) void k_shift_adj(const float* __restrict__ quat, const float* __restrict__ dmean,
                                                   const float* __restrict__ dquat, int stride, int n,
                                                   const int32_t* __restrict__ idx, int n_dyn,
                                                   const float* __restrict__ drot, float* __restrict__ d_dpos,
                                                   float* __restrict__ d_drot) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_dyn) return;
  const int64_t g = idx[j];
  if (g < 0 || g >= n) return;  // out-of-range index: ignored
  if (dmean)
    for (int i = 0; i < 3; i++) d_dpos[(int64_t)i * n_dyn + j] += dmean[i * (int64_t)stride + g];
  if (!dquat) return;
  double qc[4], s[4], d[4], e[4], qn = 0.0, sn = 0.0;
  for (int i = 0; i < 4; i++) {
    qc[i] = quat[i * (int64_t)stride + g];
    s[i] = drot[(int64_t)i * n_dyn + j];
    d[i] = dquat[i * (int64_t)stride + g];
    qn += qc[i] * qc[i];
    sn += s[i] * s[i];
  }
  qn = sqrt(qn);
  sn = sqrt(sn);
  qc[0] /= qn;
  for (int i = 1; i < 4; i++) qc[i] = -qc[i] / qn;  // conjugate of the unit quaternion
  qmul(qc, d, e);
  double dot = 0.0;
  for (int i = 0; i < 4; i++) { s[i] /= sn; dot += s[i] * e[i]; }
  for (int i = 0; i < 4; i++) d_drot[(int64_t)i * n_dyn + j] += (float)((e[i] - s[i] * dot) / sn);
}

// ---- Adam ------------------------------------------------------------------------------------
constexpr int kAdamPerBlock = 1024;  // elements per block

__global__ __launch_bounds__(256) void k_adam(AdamArgs a) {
  const int64_t blk = blockIdx.x;
  int gi = 0;
  while (gi + 1 < a.n_groups && blk >= a.g[gi + 1].block_begin) gi++;
  const AdamGroupK& G = a.g[gi];
  const int64_t base = (blk - G.block_begin) * kAdamPerBlock;
  const float omb1 = 1.f - a.b1, omb2 = 1.f - a.b2;
  float bc1 = a.bc1, bc2 = a.bc2;
  if (a.d_step) {
    const double st = (double)*a.d_step;
    bc1 = (float)(1.0 - pow((double)a.b1, st));
    bc2 = (float)(1.0 - pow((double)a.b2, st));
  }
  for (int k = threadIdx.x; k < kAdamPerBlock; k += blockDim.x) {
    const int64_t i = base + k;
    if (i >= G.n) break;
    const float g = G.g[i];
    const float m = a.b1 * G.m[i] + omb1 * g;
    const float v = a.b2 * G.v[i] + omb2 * g * g;
    G.m[i] = m;
    G.v[i] = v;
    const float mh = m / bc1, vh = v / bc2;
    G.p[i] -= G.lr * mh / (sqrtf(vh) + a.eps);
  }
}

// ---- L1 + error map ---------------------------------------------------------------------------
constexpr int kL1PerBlock = 2048;

__global__ __launch_bounds__(256) void k_l1(L1Args a, float* __restrict__ loss) {
  __shared__ float s_w[4];
  const int64_t blk = blockIdx.x;
  int vi = 0;
  while (vi + 1 < a.nv && blk >= a.v[vi + 1].block_begin) vi++;
  const L1View& V = a.v[vi];
  const float sc = a.scale / (3.0f * (float)V.hw);
  const int64_t base = (blk - V.block_begin) * kL1PerBlock;
  float acc = 0.f;
  for (int k = threadIdx.x; k < kL1PerBlock; k += blockDim.x) {
    const int64_t p = base + k;
    if (p >= V.hw) break;
    float e = 0.f;
#pragma unroll
    for (int c = 0; c < 3; c++) {
      const float d = V.render[c * V.hw + p] - V.target[c * V.hw + p];
      V.dl[c * V.hw + p] = d > 0.f ? sc : (d < 0.f ? -sc : 0.f);
      e += fabsf(d);
    }
    if (V.err) V.err[p] = e * (1.0f / 3.0f);
    acc += e;
  }
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0 && loss) atomicAdd(loss, (s_w[0] + s_w[1] + s_w[2] + s_w[3]) * sc);
}

// ---- densification ----------------------------------------------------------------------------
// Alg. 1: [P, 1] T with T the full (row-vector) projection built from the intrinsics; pixel
// x = Round(0.5((x_norm + 1) W - 1)), y likewise with y_norm and H, Round(z) = floor(z + 0.5).
// Columns 0 (x), 1 (y) and 3 (homogeneous) of T, rows P0, P1, P2, 1, for one camera:
__device__ void alg1_columns(const CamK& c, double* T /* [3][4] */) {
#pragma clang fp contract(off)
  const double W = (double)c.W, H = (double)c.H;
  const double sx = (2.0 * (double)c.fx) / W, sy = (2.0 * (double)c.fy) / H;
  const double kx = (2.0 * (double)c.cx + 1.0) / W - 1.0;
  const double ky = (2.0 * (double)c.cy + 1.0) / H - 1.0;
  for (int i = 0; i < 3; i++) {
    T[i] = sx * (double)c.R[i] + kx * (double)c.R[6 + i];
    T[4 + i] = sy * (double)c.R[3 + i] + ky * (double)c.R[6 + i];
    T[8 + i] = (double)c.R[6 + i];
  }
  T[3] = sx * (double)c.t[0] + kx * (double)c.t[2];
  T[7] = sy * (double)c.t[1] + ky * (double)c.t[2];
  T[11] = (double)c.t[2];
}

__device__ bool alg1_pixel(const double* T, int Wi, int Hi, double X, double Y, double Z, int& xn, int& yn) {
#pragma clang fp contract(off)
  const double W = (double)Wi, H = (double)Hi;
  const double hx = ((X * T[0] + Y * T[1]) + Z * T[2]) + T[3];
  const double hy = ((X * T[4] + Y * T[5]) + Z * T[6]) + T[7];
  const double hw = ((X * T[8] + Y * T[9]) + Z * T[10]) + T[11];
  if (!(hw > 0.0)) return false;
  const double xnorm = hx / hw, ynorm = hy / hw;
  const double xf = floor(0.5 * ((xnorm + 1.0) * W - 1.0) + 0.5);
  const double yf = floor(0.5 * ((ynorm + 1.0) * H - 1.0) + 0.5);
  if (xf < 0.0 || yf < 0.0 || xf >= W || yf >= H) return false;
  xn = (int)xf;
  yn = (int)yf;
  return true;
}

// Selection (Alg. 1), two kernels.  The score is the largest error at the Gaussian's pixel over the
// views that see it; the member test needs it, whether any of these errors passes gamma, and the mean
// gradient norm.
//
// k_densify_scores reads the error maps at random pixels, a line per read, and is bound by these lines:
// an XCD takes the (view, Gaussians) blocks of one view after the other, so that the lines of one map
// (5.5 MB at 1352x1014) are read again from its 4 MB L2 and not all views' maps at once.  Each of up to
// `planes` groups of views leaves its largest error in a row of codes.  200k Gaussians, 20 views of
// 1352x1014: 65 us with a workgroup over all views, 34 now.
constexpr int kScoreThreads = 256, kScorePer = 4;  // Gaussians of a workgroup: 1,024
__global__ __launch_bounds__(kScoreThreads) void k_densify_scores(SceneK s, DensifyArgs a, int n_base, int group,
                                                                 int chunks, int total, int per,
                                                                 uint32_t* __restrict__ codes) {
  __shared__ double s_T[DASS_MAX_VIEWS][12];
  const int b = (int)(blockIdx.x % kNumXcd) * per + (int)(blockIdx.x / kNumXcd);
  if (b >= total) return;
  const int row = b / chunks, g0 = (b - row * chunks) * (kScoreThreads * kScorePer) + (int)threadIdx.x;
  const int v0 = row * group, v1 = min(v0 + group, a.nv);
  if (v0 + (int)threadIdx.x < v1) alg1_columns(a.cams[v0 + threadIdx.x], s_T[threadIdx.x]);
  __syncthreads();
  double X[kScorePer], Y[kScorePer], Z[kScorePer];
  uint32_t code[kScorePer];
#pragma unroll
  for (int i = 0; i < kScorePer; i++) {
    const int g = min(g0 + i * kScoreThreads, n_base - 1);
    X[i] = s.mean[g];
    Y[i] = s.mean[(int64_t)s.stride + g];
    Z[i] = s.mean[2 * (int64_t)s.stride + g];
    code[i] = 0u;
  }
  for (int v = v0; v < v1; v++) {
    const int W = a.cams[v].W, H = a.cams[v].H;
    bool in[kScorePer];
    float e[kScorePer];
#pragma unroll
    for (int i = 0; i < kScorePer; i++) {
      int x, y;
      in[i] = alg1_pixel(s_T[v - v0], W, H, X[i], Y[i], Z[i], x, y);
      e[i] = in[i] ? a.err[v][(int64_t)y * W + x] : 0.f;
    }
    // the error, at least 0, and below it whether the error passes gamma: the largest code of the
    // views has both for all of them
#pragma unroll
    for (int i = 0; i < kScorePer; i++)
      if (in[i]) code[i] = max(code[i], __float_as_uint(fmaxf(0.f, e[i])) << 1 | (e[i] > a.gamma_err ? 1u : 0u));
  }
#pragma unroll
  for (int i = 0; i < kScorePer; i++)
    if (g0 + i * kScoreThreads < n_base) codes[(int64_t)row * n_base + g0 + i * kScoreThreads] = code[i];
}

// The k_max best members are all that a call uses of the ranking, so that they are selected, not sorted:
// three histogram passes over 11, 11 and 10 bits of the rank key (the complemented score bits: ascending
// key = descending score, ties by index) find the key of the last one, two more collect the members
// before it and as many of that key as still fit, in index order, and each one's rank among them is
// counted.  Every pass takes the Gaussians in at most kSelBlocks equal runs.  200k Gaussians, 20 views,
// 5,000 children: pack, scan and a stable sort of all members in 13 launches 109 us, now 6 and 41 us; up to
// kSelMost children (the count of ranks grows with their square; the call with 16,384 126 us, sorted
// 151), else they are sorted.
constexpr int kSelThreads = 1024, kSelBlocks = 256, kSelBits[3] = {11, 11, 10}, kSelShift[3] = {21, 10, 0};
constexpr int kSelBins = 2048, kSelMost = 16384;
// uint32 workspace: histograms [3][kSelBins], state, counts [kSelBlocks][2]
constexpr int kSelState = 3 * kSelBins, kSelCounts = kSelState + 16;
struct SelRun {
  int n, run, want;  // Gaussians, of a workgroup, best members that are used (at most)
};

// The digit of the want-th smallest key among those of the histogram (want >= 1, at most their number),
// and the keys with a smaller one: to *state.  Whole workgroup.
__device__ __forceinline__ uint32_t sel_digit(const uint32_t* __restrict__ hist, uint32_t want, uint32_t* s_w,
                                              uint32_t* s_res, uint32_t& before) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
  uint32_t inc = h0 + h1;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(inc, d, 64);
    if (lane >= d) inc += y;
  }
  if (lane == 63) s_w[w] = inc;
  __syncthreads();
  uint32_t base = 0;
  for (int i = 0; i < w; i++) base += s_w[i];
  const uint32_t e0 = base + inc - h0 - h1, e1 = e0 + h0;
  if (e0 < want && want <= e1) s_res[0] = 2 * tid, s_res[1] = e0;
  if (e1 < want && want <= e1 + h1) s_res[0] = 2 * tid + 1, s_res[1] = e1;
  __syncthreads();
  before = s_res[1];
  return s_res[0];
}

// Adds the workgroup's histogram to the call's.
__device__ __forceinline__ void sel_add(const uint32_t* __restrict__ s_h, uint32_t* __restrict__ hist) {
  __syncthreads();
  for (int i = threadIdx.x; i < kSelBins; i += kSelThreads)
    if (s_h[i]) atomicAdd(&hist[i], s_h[i]);
}

// Members and their rank keys from the rows of codes; the first digit's histogram (sel != 0).
__global__ __launch_bounds__(kSelThreads) void k_densify_members(SelRun r, const uint32_t* __restrict__ codes, int rows,
                                                                 float tau_pos, float tau_err,
                                                                 const float* __restrict__ gsum,
                                                                 const int32_t* __restrict__ gcnt,
                                                                 uint32_t* __restrict__ keep,
                                                                 uint32_t* __restrict__ score_key,
                                                                 uint32_t* __restrict__ sel) {
  __shared__ uint32_t s_h[kSelBins];
  for (int i = threadIdx.x; i < kSelBins; i += kSelThreads) s_h[i] = 0u;
  __syncthreads();
  const int g1 = min((int)(blockIdx.x + 1) * r.run, r.n);
  for (int g = blockIdx.x * r.run + threadIdx.x; g < g1; g += kSelThreads) {
    uint32_t code = 0u;
#pragma unroll 4
    for (int k = 0; k < rows; k++) code = max(code, codes[(int64_t)k * r.n + g]);
    const int32_t c = gcnt[g];
    const float gbar = c > 0 ? gsum[g] / (float)c : 0.f;
    const bool in_s = (gbar > tau_pos) || ((code & 1u) != 0 && gbar > tau_err);
    const uint32_t key = ~(code >> 1);
    keep[g] = in_s ? 1u : 0u;
    score_key[g] = key;
    if (sel && in_s) atomicAdd(&s_h[key >> kSelShift[0]], 1u);
  }
  if (sel) sel_add(s_h, sel);
}

// The digit of pass P - 1 (to the state, with what is still wanted beyond it), and the histogram of
// pass P over the keys that agree in the digits before.  state: [0] key prefix, [1] still wanted.
template <int P>
__global__ __launch_bounds__(kSelThreads) void k_densify_digit(SelRun r, const uint32_t* __restrict__ keep,
                                                               const uint32_t* __restrict__ score_key,
                                                               uint32_t* __restrict__ sel,
                                                               uint32_t* __restrict__ d_count) {
  __shared__ uint32_t s_h[kSelBins], s_w[kSelThreads / 64], s_res[2], s_n;
  uint32_t* __restrict__ state = sel + kSelState + 4 * P;  // of this pass (the one before: 4 words earlier)
  for (int i = threadIdx.x; i < kSelBins; i += kSelThreads) s_h[i] = 0u;
  uint32_t want, prefix = 0u;
  if (P == 1) {  // the first digit's histogram also gives the number of members
    if (threadIdx.x == 0) s_n = 0u;
    __syncthreads();
    uint32_t m = sel[2 * threadIdx.x] + sel[2 * threadIdx.x + 1];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m += __shfl_xor(m, d, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(&s_n, m);
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) *d_count = s_n;
    want = min(s_n, (uint32_t)r.want);
  } else {
    prefix = state[-4];
    want = state[-3];
  }
  if (want == 0u) {  // no members: nothing is collected
    if (blockIdx.x == 0 && threadIdx.x == 0) state[0] = 0u, state[1] = 0u;
    return;
  }
  uint32_t before;
  const uint32_t digit = sel_digit(sel + (P - 1) * kSelBins, want, s_w, s_res, before);
  prefix |= digit << kSelShift[P - 1];
  want -= before;
  if (blockIdx.x == 0 && threadIdx.x == 0) state[0] = prefix, state[1] = want;
  const int g1 = min((int)(blockIdx.x + 1) * r.run, r.n);
  for (int g = blockIdx.x * r.run + threadIdx.x; g < g1; g += kSelThreads) {
    const uint32_t key = score_key[g];
    if (keep[g] && (key >> kSelShift[P - 1]) == (prefix >> kSelShift[P - 1]))
      atomicAdd(&s_h[(key >> kSelShift[P]) & ((1u << kSelBits[P]) - 1u)], 1u);
  }
  sel_add(s_h, sel + P * kSelBins);
}

// The last digit, and how many members of each run lie before the key and at it.
__global__ __launch_bounds__(kSelThreads) void k_densify_count(SelRun r, const uint32_t* __restrict__ keep,
                                                               const uint32_t* __restrict__ score_key,
                                                               uint32_t* __restrict__ sel) {
  __shared__ uint32_t s_w[kSelThreads / 64], s_res[2], s_c[2];
  uint32_t* __restrict__ state = sel + kSelState + 12;
  uint32_t prefix = state[-4], want = state[-3];
  if (want == 0u) {
    if (blockIdx.x == 0 && threadIdx.x == 0) state[0] = 0u, state[1] = 0u;
    return;
  }
  if (threadIdx.x < 2) s_c[threadIdx.x] = 0u;
  uint32_t before;
  prefix |= sel_digit(sel + 2 * kSelBins, want, s_w, s_res, before);
  want -= before;
  if (blockIdx.x == 0 && threadIdx.x == 0) state[0] = prefix, state[1] = want;
  uint32_t less = 0, same = 0;
  const int g1 = min((int)(blockIdx.x + 1) * r.run, r.n);
  for (int g = blockIdx.x * r.run + threadIdx.x; g < g1; g += kSelThreads) {
    const uint32_t key = score_key[g];
    if (keep[g]) less += key < prefix ? 1u : 0u, same += key == prefix ? 1u : 0u;
  }
  if (less) atomicAdd(&s_c[0], less);
  if (same) atomicAdd(&s_c[1], same);
  __syncthreads();
  if (threadIdx.x < 2) sel[kSelCounts + 2 * blockIdx.x + threadIdx.x] = s_c[threadIdx.x];
}

// (key, index) of the members before the key of the last one, and of the first `want` at it, in index
// order per kind: those before first.
__global__ __launch_bounds__(kSelThreads) void k_densify_collect(SelRun r, const uint32_t* __restrict__ keep,
                                                                 const uint32_t* __restrict__ score_key,
                                                                 const uint32_t* __restrict__ sel,
                                                                 uint64_t* __restrict__ out) {
  __shared__ uint32_t s_w[2][kSelThreads / 64], s_at[2], s_less;
  const uint32_t last = sel[kSelState + 12], want = sel[kSelState + 13];
  if (want == 0u) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid < 2) s_at[tid] = 0u;
  if (tid == 2) s_less = 0u;
  __syncthreads();
  if (tid < (int)gridDim.x) {
    const uint32_t l = sel[kSelCounts + 2 * tid], e = sel[kSelCounts + 2 * tid + 1];
    if (l) atomicAdd(&s_less, l);
    if (tid < (int)blockIdx.x) {
      if (l) atomicAdd(&s_at[0], l);
      if (e) atomicAdd(&s_at[1], e);
    }
  }
  __syncthreads();
  uint32_t at_l = s_at[0], at_e = s_at[1];
  const uint32_t all_less = s_less;
  const uint64_t lt = (1ull << lane) - 1ull;
  const int g0 = blockIdx.x * r.run, g1 = min(g0 + r.run, r.n);
  for (int base = g0; base < g1; base += kSelThreads) {  // uniform
    const int g = base + tid;
    const uint32_t key = g < g1 ? score_key[g] : 0u;
    const bool in = g < g1 && keep[g] != 0u;
    const uint64_t bl = __ballot(in && key < last), be = __ballot(in && key == last);
    if (lane == 0) {
      s_w[0][w] = (uint32_t)__popcll(bl);
      s_w[1][w] = (uint32_t)__popcll(be);
    }
    __syncthreads();
    uint32_t ol = at_l, oe = at_e, tl = 0, te = 0;
    for (int i = 0; i < kSelThreads / 64; i++) {
      if (i < w) ol += s_w[0][i], oe += s_w[1][i];
      tl += s_w[0][i];
      te += s_w[1][i];
    }
    const uint64_t kv = (uint64_t)key << 32 | (uint32_t)g;
    if (in && key < last) out[ol + (uint32_t)__popcll(bl & lt)] = kv;
    if (in && key == last) {
      const uint32_t e = oe + (uint32_t)__popcll(be & lt);
      if (e < want) out[all_less + e] = kv;
    }
    at_l += tl;
    at_e += te;
    __syncthreads();
  }
}

// Ranks of the collected members by counting: a wave takes a member, its lanes every 64th of the others,
// tile after tile of LDS, which sixteen waves share (5,000 members 9.3 us; 13.3 with sixteen lanes to a
// member and four waves).
constexpr int kRankThreads = 1024, kRankLanes = 64, kRankTile = 4096;
__global__ __launch_bounds__(kRankThreads) void k_densify_rank(int want, const uint32_t* __restrict__ d_count,
                                                               const uint64_t* __restrict__ in,
                                                               uint32_t* __restrict__ sel_idx) {
  __shared__ uint64_t s_k[kRankTile];
  const int m = (int)min(*d_count, (uint32_t)want);
  const int i0 = blockIdx.x * (kRankThreads / kRankLanes);
  if (i0 >= m) return;
  const int i = i0 + (int)threadIdx.x / kRankLanes, sub = threadIdx.x % kRankLanes;
  const uint64_t mine = in[min(i, m - 1)];
  int rank = 0;
  for (int base = 0; base < m; base += kRankTile) {
    const int cnt = min(kRankTile, m - base);
    __syncthreads();
    for (int j = threadIdx.x; j < cnt; j += kRankThreads) s_k[j] = in[base + j];
    __syncthreads();
#pragma unroll 8
    for (int j = sub; j < cnt; j += kRankLanes) rank += s_k[j] < mine ? 1 : 0;
  }
#pragma unroll
  for (int d = 1; d < kRankLanes; d <<= 1) rank += __shfl_xor(rank, d, 64);
  if (sub == 0 && i < m) sel_idx[rank] = (uint32_t)mine;
}

// members packed in index order: key and Gaussian index at the member's rank in the scan
__global__ __launch_bounds__(256) void k_densify_pack(int n_base, const uint32_t* __restrict__ keep,
                                                      const uint64_t* __restrict__ pos,
                                                      const uint32_t* __restrict__ score_key,
                                                      uint32_t* __restrict__ sel_keys, uint32_t* __restrict__ sel_vals,
                                                      uint32_t* __restrict__ d_count) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g == 0) *d_count = (uint32_t)pos[n_base];
  if (g >= n_base || !keep[g]) return;
  sel_keys[pos[g]] = score_key[g];
  sel_vals[pos[g]] = (uint32_t)g;
}

__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t i) {
  uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ double u01(uint64_t x) { return (double)(x >> 11) * 0x1.0p-53; }

// A quad of lanes per child, so the float64 chains run side by side: lane i < 3 forms the
// child's i-th normal draw and scale, lane 3 copies the quaternion and the opacity logit; every
// lane then forms its mean component from the quad's draws (the same products and sums as
// written for one thread) and copies a quarter of the SH planes.
__global__ __launch_bounds__(256) void k_densify_spawn(float* __restrict__ mean, float* __restrict__ quat,
                                                       float* __restrict__ log_scale, float* __restrict__ logit,
                                                       float* __restrict__ sh, int n_sh, int stride, int n, int capacity,
                                                       const uint32_t* __restrict__ sel_idx,
                                                       const uint32_t* __restrict__ d_count, int k_max, uint64_t seed,
                                                       int32_t* __restrict__ n_appended) {
  const uint32_t ns = *d_count;
  const int room = capacity - n;
  const int n_app = ns == 0 ? 0 : (k_max < room ? k_max : room);
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = tid >> 2, l = tid & 3;
  if (tid == 0 && n_appended) *n_appended = n_app < 0 ? 0 : n_app;
  if (j >= n_app) return;  // uniform over a quad (n_app whole children)
  const int64_t p = (int64_t)sel_idx[j % ns];  // parents in rank order
  const int64_t c = (int64_t)n + j;
  const int64_t st = stride;
  // lane l < 3: scale l and normal draw l (Box-Muller on draws 4j .. 4j+3: z0, z1 from the
  // first pair, z2 from the second)
  double scl = 0.0, zl = 0.0;
  if (l < 3) {
    const double TWO_PI = 6.283185307179586476925;
    const uint64_t d0 = 4ull * (uint64_t)j + (l == 2 ? 2u : 0u);
    const double ua = 1.0 - u01(splitmix64(seed, d0)), ub = u01(splitmix64(seed, d0 + 1));
    const double r = sqrt(-2.0 * log(ua));
    zl = l == 1 ? r * sin(TWO_PI * ub) : r * cos(TWO_PI * ub);
    scl = exp((double)log_scale[l * st + p]);
  }
  const int q0 = (int)(threadIdx.x & 63) & ~3;  // the quad's first lane in the wave
  double sc[3], z[3];
#pragma unroll
  for (int k = 0; k < 3; k++) {
    sc[k] = __shfl(scl, q0 + k, 64);
    z[k] = __shfl(zl, q0 + k, 64);
  }
  if (l < 3) {
    double q[4], qn = 0.0;
    for (int i = 0; i < 4; i++) {
      q[i] = quat[i * st + p];
      qn += q[i] * q[i];
    }
    qn = sqrt(qn);
    for (int i = 0; i < 4; i++) q[i] /= qn;
    const double w = q[0], x = q[1], y = q[2], zq = q[3];
    const double R[9] = {1.0 - 2.0 * (y * y + zq * zq), 2.0 * (x * y - w * zq), 2.0 * (x * zq + w * y),
                         2.0 * (x * y + w * zq), 1.0 - 2.0 * (x * x + zq * zq), 2.0 * (y * zq - w * x),
                         2.0 * (x * zq - w * y), 2.0 * (y * zq + w * x), 1.0 - 2.0 * (x * x + y * y)};
    const int i = l;
    const double off = R[i * 3 + 0] * sc[0] * z[0] + R[i * 3 + 1] * sc[1] * z[1] + R[i * 3 + 2] * sc[2] * z[2];
    mean[i * st + c] = (float)((double)mean[i * st + p] + off);
    const double ln16 = 0.47000362924573558;  // ln 1.6
    log_scale[i * st + c] = (float)((double)log_scale[i * st + p] - ln16);
  } else {
    for (int i = 0; i < 4; i++) quat[i * st + c] = quat[i * st + p];
    logit[c] = logit[p];
  }
  // the child row c >= n never overlaps a parent row p < n: a quarter of the planes per lane,
  // loaded together, then stored
  float shv[12];
#pragma unroll
  for (int k = 0; k < 12; k++) shv[k] = 4 * k + l < n_sh ? sh[(int64_t)(4 * k + l) * st + p] : 0.f;
#pragma unroll
  for (int k = 0; k < 12; k++)
    if (4 * k + l < n_sh) sh[(int64_t)(4 * k + l) * st + c] = shv[k];
}

}  // namespace

void launch_shift_fwd(const SceneK& in, float* out_mean, float* out_quat, const int32_t* dyn_idx, int n_dyn,
                      const float* dpos, const float* drot, hipStream_t st) {
  if (in.n > 0)
    k_copy_mq<<<(in.n + 255) / 256, 256, 0, st>>>(in.mean, in.quat, out_mean, out_quat, in.n, in.stride);
  if (n_dyn > 0)
    k_shift_fwd<<<(n_dyn + 255) / 256, 256, 0, st>>>(in.mean, in.quat, out_mean, out_quat, in.stride, in.n, dyn_idx,
                                                      n_dyn, dpos, drot);
}

void launch_shift_adj(const SceneK& in, const float* dmean, const float* dquat, const int32_t* dyn_idx, int n_dyn,
                      const float* drot, float* d_dpos, float* d_drot, hipStream_t st) {
  if (n_dyn > 0)
    k_shift_adj<<<(n_dyn + 255) / 256, 256, 0, st>>>(in.quat, dmean, dquat, in.stride, in.n, dyn_idx, n_dyn, drot,
                                                      d_dpos, d_drot);
}

__global__ void k_step_increment(int32_t* s) { *s += 1; }

void launch_step_increment(int32_t* d_step, hipStream_t st) { k_step_increment<<<1, 1, 0, st>>>(d_step); }

void launch_adam(const AdamArgs& a, int64_t total_blocks, hipStream_t st) {
  if (total_blocks > 0) k_adam<<<(unsigned)total_blocks, 256, 0, st>>>(a);
}

void launch_l1(const L1Args& a, int64_t total_blocks, float* loss, hipStream_t st) {
  if (total_blocks > 0) k_l1<<<(unsigned)total_blocks, 256, 0, st>>>(a, loss);
}

static void densify_members(const SceneK& s, const DensifyArgs& a, const DensifyWs& w, const SelRun& r,
                            const float* gsum, const int32_t* gcnt, uint32_t* sel, hipStream_t st) {
  // a row of codes per group of views, as many as the buffer holds: one view each unless a call has
  // more views than the context was made for
  const int rows_max = (int)std::min<int64_t>(a.nv, w.cap_codes / r.n);
  const int group = (a.nv + rows_max - 1) / rows_max, rows = (a.nv + group - 1) / group;
  const int chunk = kScoreThreads * kScorePer, chunks = (r.n + chunk - 1) / chunk;
  const int64_t total = (int64_t)rows * chunks, per = (total + kNumXcd - 1) / kNumXcd;
  k_densify_scores<<<(unsigned)(per * kNumXcd), kScoreThreads, 0, st>>>(s, a, r.n, group, chunks, (int)total, (int)per,
                                                                       w.codes);
  k_densify_members<<<(r.n + r.run - 1) / r.run, kSelThreads, 0, st>>>(r, w.codes, rows, a.tau_pos, a.tau_err, gsum, gcnt,
                                                                      w.keep, w.score_key, sel);
}

static SelRun sel_run(int n, int want) {
  const int per = (n + kSelBlocks - 1) / kSelBlocks;
  return SelRun{n, (per + kSelThreads - 1) / kSelThreads * kSelThreads, want};
}

bool densify_selects(int want) { return want <= kSelMost; }

void launch_densify_select(const SceneK& s, const DensifyArgs& a, const float* gsum, const int32_t* gcnt, int n_base,
                           int want, const DensifyWs& w, uint32_t* sel_idx, uint32_t* d_count, hipStream_t st) {
  if (n_base <= 0 || want <= 0) {
    launch_fill_u32(d_count, 0u, 1, st);
    return;
  }
  const SelRun r = sel_run(n_base, std::min(want, n_base));
  const unsigned blocks = (unsigned)((n_base + r.run - 1) / r.run);
  launch_fill_u32(w.sel, 0u, kSelState, st);
  densify_members(s, a, w, r, gsum, gcnt, w.sel, st);
  k_densify_digit<1><<<blocks, kSelThreads, 0, st>>>(r, w.keep, w.score_key, w.sel, d_count);
  k_densify_digit<2><<<blocks, kSelThreads, 0, st>>>(r, w.keep, w.score_key, w.sel, d_count);
  k_densify_count<<<blocks, kSelThreads, 0, st>>>(r, w.keep, w.score_key, w.sel);
  k_densify_collect<<<blocks, kSelThreads, 0, st>>>(r, w.keep, w.score_key, w.sel, w.pos);
  const int per = kRankThreads / kRankLanes;
  k_densify_rank<<<(r.want + per - 1) / per, kRankThreads, 0, st>>>(r.want, d_count, w.pos, sel_idx);
}

void launch_densify_pack(const SceneK& s, const DensifyArgs& a, const float* gsum, const int32_t* gcnt, int n_base,
                         const DensifyWs& w, uint64_t* scan_tmp, uint32_t* sel_keys, uint32_t* sel_vals,
                         uint32_t* d_count, hipStream_t st) {
  launch_fill_u32(d_count, 0u, 1, st);
  if (n_base <= 0) return;
  densify_members(s, a, w, sel_run(n_base, 0), gsum, gcnt, nullptr, st);
  scan_u32_to_u64(w.keep, w.pos, n_base, scan_tmp, st);
  k_densify_pack<<<(n_base + 255) / 256, 256, 0, st>>>(n_base, w.keep, w.pos, w.score_key, sel_keys, sel_vals, d_count);
}

void launch_densify_spawn(float* mean, float* quat, float* log_scale, float* logit, float* sh, int n_planes_sh,
                          int stride, int n, int capacity, const uint32_t* sel_idx, const uint32_t* d_count, int k_max,
                          uint64_t seed, int32_t* n_appended, hipStream_t st) {
  const int blocks = k_max > 0 ? (int)(((int64_t)k_max * 4 + 255) / 256) : 1;
  k_densify_spawn<<<blocks, 256, 0, st>>>(mean, quat, log_scale, logit, sh, n_planes_sh, stride, n, capacity, sel_idx,
                                           d_count, k_max, seed, n_appended);
}

int adam_per_block() { return kAdamPerBlock; }
int l1_per_block() { return kL1PerBlock; }

}  // namespace dass
