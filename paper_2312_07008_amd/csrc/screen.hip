// Learned pair screening (row a12; not part of the paper's method): pair
// features, a 5-64-64-1 tanh network trained in FP32 with mean squared error
// and Adam, and the mask that drops core pairs whose predicted ||t_ij||_F is
// below a threshold.
//
// Pair quantities for unordered core pairs i <= j (row-major order, the order
// of the pass's pair list):
//   q_iQ = ||B^Q_i.||_2,  U_ij = sum_Q q_iQ q_jQ >= ||V_ij||_F,
//   W_ij = (sum_Q q_iQ^2 q_jQ^2)^(1/2)  (||V_ij||_F for mutually orthogonal rank-one terms),
//   g_ij = max |1 - e^{-s D^2}| / |D| over the pair's range of denominators D (Eq. A7),
// so ||t_ij||_F <= g_ij U_ij is a rigorous screen and log(g_ij W_ij) is the scale
// the network corrects.  Features
//   x = (e_i, e_j, log(U/W), 0.1 (log W_ij - (log W_ii + log W_jj)/2), 0.1 log(g W)).
// Parameters (FP32) are packed [W1 64x5, b1, W2 64x64, b2, w3, b3] = 4609 values.
#include <algorithm>
#include <cmath>
#include <cfloat>

#include "../../include/dfpt2.h"
#include "common.h"
#include "host.h"

namespace dfpt2 {

namespace {
constexpr int H = 64;
constexpr int NIN = 5;
constexpr int NP = H * NIN + H + H * H + H + H + 1;  // 4609
constexpr int OFF_W1 = 0, OFF_B1 = H * NIN, OFF_W2 = OFF_B1 + H, OFF_B2 = OFF_W2 + H * H, OFF_W3 = OFF_B2 + H,
              OFF_B3 = OFF_W3 + H;
constexpr int BW_SAMPLES = 128;  // samples that the sizes of the workspaces count one row of gradients for

// q2[i][Q] = sum_a B[i][a][Q]^2 for core holes
// Bound by the latency of its loads (60 virtuals: 11 us with one thread per column, all rows
// one after the other): a workgroup takes 64 columns, its 16 waves the rows w, w + 16, ...
__global__ __launch_bounds__(1024) void colnorm2_kernel(const double* B, int n_v, int n_aux, double* q2) {
  __shared__ double sh[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int Q = blockIdx.x * 64 + lane;
  const int i = blockIdx.y;
  const double* Bi = B + (size_t)i * n_v * n_aux + min(Q, n_aux - 1);
  double acc = 0.0;
#pragma unroll 4
  for (int a = w; a < n_v; a += 16) {
    const double x = Bi[(size_t)a * n_aux];
    acc += x * x;
  }
  sh[w][lane] = acc;
  __syncthreads();
  if (w > 0 || Q >= n_aux) return;
  for (int g = 1; g < 16; ++g) acc += sh[g][lane];
  q2[(size_t)i * n_aux + Q] = acc;
}

__device__ double reg_fun(double s, double x) { return x > 0.0 ? -expm1(-s * x * x) / x : 0.0; }

// one wave per pair; W_ii^2 = sum_Q q2_iQ^2 and W_jj^2 come along with the pair's own sums, and
// lanes 0 to 4 take one regularizer value and one logarithm each.  The virtual energies are
// ascending: the denominator range uses the first and last.
__global__ void pair_features_kernel(const double* q2, const double* eps_h, const double* eps_v, int n_v, int n_core,
                                     int n_aux, double s, double x_star, float* feats, double* log_scale,
                                     int n_pairs) {
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (p >= n_pairs) return;
  int i = 0, rem = p;
  while (rem >= n_core - i) {
    rem -= n_core - i;
    ++i;
  }
  const int j = i + rem;
  double u = 0.0, w2 = 0.0, wi = 0.0, wj = 0.0;
  for (int Q = lane; Q < n_aux; Q += 64) {
    const double a = q2[(size_t)i * n_aux + Q], b = q2[(size_t)j * n_aux + Q];
    u += sqrt(a) * sqrt(b);
    w2 += a * b;
    wi += a * a;
    wj += b * b;
  }
  u = wave_sum(u);
  w2 = wave_sum(w2);
  wi = wave_sum(wi);
  wj = wave_sum(wj);
  const double ei = eps_h[i], ej = eps_h[j];
  double lo = fabs(ei + ej - 2.0 * eps_v[0]), hi = fabs(ei + ej - 2.0 * eps_v[n_v - 1]);
  if (lo > hi) {
    const double t = lo;
    lo = hi;
    hi = t;
  }
  const double r = reg_fun(s, lane == 0 ? x_star : lane == 1 ? lo : hi);
  const double r0 = __shfl(r, 0, 64), r1 = __shfl(r, 1, 64), r2 = __shfl(r, 2, 64);
  const double g = (lo <= x_star && x_star <= hi) ? r0 : fmax(r1, r2);
  const double w = sqrt(w2);
  const double l = log(lane == 0 ? w : lane == 1 ? u : lane == 2 ? g : lane == 3 ? wi : wj);
  const double lw = __shfl(l, 0, 64), lu = __shfl(l, 1, 64), lg = __shfl(l, 2, 64);
  const double li = __shfl(l, 3, 64), lj = __shfl(l, 4, 64);
  if (lane != 0) return;
  float* f = feats + (size_t)p * NIN;
  f[0] = (float)ei;
  f[1] = (float)ej;
  f[2] = (float)(lu - lw);
  f[3] = (float)(0.1 * (lw - 0.25 * (li + lj)));
  f[4] = (float)(0.1 * (lg + lw));
  log_scale[2 * (size_t)p] = lg + lw;
  log_scale[2 * (size_t)p + 1] = lg + lu;
}

// ------------------------------------------------------------------ network
// One workgroup of eight waves takes tiles of 64, 32 or 16 samples (net_plan); the products of a tile (z2 = h1 W2^T,
// dz2 W2, dz2^T h1, dz1^T inputs) run on the FP32 matrix pipe (16x16x4, 32 rows and 16 columns
// per wave), everything between them in registers and LDS:
//   kForward   pred, and the activations where the caller wants them
//   kBackward  parameter gradients from activations and d pred
//   kTrain     both, with d pred = 2 (pred - y) / n and the loss formed on the way: the
//              activations and d pred of a training step never reach memory
// The gradients of a workgroup's tiles add up in its registers and leave as one row of
// `partial` (NP parameter gradients, then the sum of squared residuals); at most
// kMaxGroups rows are summed afterwards in a fixed order.  What bounds a step at ten
// thousand samples is latency, hence two waves per SIMD, conflict-free LDS rows and every
// read of memory in flight before the first barrier.  A step of 11000 samples: 179 us as
// five launches (one thread per sample forward, 128 samples per workgroup backward, one
// thread per reduced parameter), 27 us with four waves and 32x32x2 products (mlp_kernel 19.7),
// 19 us so (mlp_kernel 12.7, sum_partials_kernel 4.1).  A tanh without branches: no faster.
enum NetMode { kForward, kBackward, kTrain };
constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int LD = H + 20;          // LDS row of a 64-wide matrix: 16 rows of 4 columns hit distinct banks, 4 rows of 16 nearly
constexpr int kMaxGroups = 256;
constexpr int PROW = (NP + 1 + 3) / 4 * 4;  // floats per row of partial sums

typedef float f4r __attribute__((ext_vector_type(4)));

template <int MODE, int TS>
__global__ __launch_bounds__(kThreads, 1) void mlp_kernel(const float* Wp, const float* X, const float* y, int n, float* out,
                                                          float* cache, const float* dout, float* partial) {
  __shared__ float w2[H * LD], sh1[TS * LD], sh2[TS * LD], sdz[TS * LD];
  __shared__ float w1[H * NIN], b1[H], b2[H], w3[H], sx[TS * 8], sdo[TS], red[2][kWaves][H], lred[2][kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l16 = lane & 15, q4 = lane >> 4;
  // this wave's 16 x 16 blocks: columns cq, rows rh and, where there are more than 32, rh + 32
  // (two waves of a SIMD share the blocks of its columns evenly)
  constexpr int NI = TS > 32 ? 2 : 1;
  static_assert(TS == 64 || TS == 32 || TS == 16, "whole blocks per wave, or one for half of them");
  const int rh = __builtin_amdgcn_readfirstlane(wv >> 2) * 16, cq = (wv & 3) * 16;
  // everything that the first tile reads from memory is in flight at once
  const int ntile = (n + TS - 1) / TS, xr = tid >> 3, xc = tid & 7;  // row and input of this thread
  auto input = [&](int tile) {  // column 5 is 1: its gradient is b1's
    const int s = tile * TS + xr;
    return xc < NIN && xr < TS && s < n ? X[(size_t)s * NIN + xc] : xc == NIN ? 1.f : 0.f;
  };
  auto target = [&](int tile) {
    const int s = tile * TS + xr;
    return MODE == kTrain && xr < TS && s < n ? y[s] : 0.f;
  };
  static_assert(TS * 8 <= kThreads, "an input and an eighth of an output per thread");
  float wr[H * H / kThreads], xn = input(blockIdx.x), yn = target(blockIdx.x);
#pragma unroll
  for (int k = 0; k < H * H / kThreads; ++k) wr[k] = Wp[OFF_W2 + kThreads * k + tid];
  const float b3 = Wp[OFF_B3];
  for (int k = tid; k < H * NIN; k += kThreads) w1[k] = Wp[OFF_W1 + k];
  if (tid < H) {
    b1[tid] = Wp[OFF_B1 + tid];
    b2[tid] = Wp[OFF_B2 + tid];
    w3[tid] = Wp[OFF_W3 + tid];
  }
#pragma unroll
  for (int k = 0; k < H * H / kThreads; ++k) w2[(kWaves * k + wv) * LD + lane] = wr[k];
  f4r g2[2], gx;  // gradients of W2 (rows k, columns m) and of W1 and b1 (rows m, columns inputs)
#pragma unroll
  for (int r = 0; r < 4; ++r) g2[0][r] = g2[1][r] = gx[r] = 0.f;
  float gb2 = 0.f, gw3 = 0.f, gb3 = 0.f, loss = 0.f;
  for (int tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
    const int s0 = tile * TS, ns = min(TS, n - s0);
    __syncthreads();  // the previous tile's readers are done
    if (xr < TS) sx[tid] = xn;
    const float yr = yn;
    if (tile + (int)gridDim.x < ntile) {
      xn = input(tile + gridDim.x);
      yn = target(tile + gridDim.x);
    }
    if (MODE == kBackward)
      for (int k = tid; k < TS * H; k += kThreads) {
        const int r = k >> 6, c = k & 63;
        const float* a = cache + (size_t)(s0 + r) * 2 * H;
        sh1[r * LD + c] = r < ns ? a[c] : 0.f;
        sh2[r * LD + c] = r < ns ? a[H + c] : 0.f;
      }
    if (MODE == kBackward && tid < TS) sdo[tid] = tid < ns ? dout[s0 + tid] : 0.f;
    __syncthreads();
    if (MODE != kBackward) {
      {  // h1: thread (k, 8 samples)
        const int k = lane;
        float wk[NIN];
#pragma unroll
        for (int c = 0; c < NIN; ++c) wk[c] = w1[k * NIN + c];
        const float bk = b1[k];
#pragma unroll 4
        for (int r = wv; r < TS; r += kWaves) {
          float z = bk;
#pragma unroll
          for (int c = 0; c < NIN; ++c) z = fmaf(wk[c], sx[r * 8 + c], z);
          const float h = tanhf(z);
          sh1[r * LD + k] = h;
          if (MODE == kForward && cache && r < ns) cache[(size_t)(s0 + r) * 2 * H + k] = h;
        }
      }
      __syncthreads();
      f4r z2[NI];  // rows s, columns k
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) z2[i][r] = 0.f;
#pragma unroll
      for (int m = 0; m < H; m += 4) {
        const float bw = w2[(cq + l16) * LD + m + q4];
#pragma unroll
        for (int i = 0; i < NI; ++i)
          if (TS > 16 || rh == 0)
            z2[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(sh1[(rh + 32 * i + l16) * LD + m + q4], bw, z2[i], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (TS > 16 || rh == 0)
#pragma unroll
          for (int r = 0; r < 4; ++r) {  // register r: row 4 (lane / 16) + r
            const int row = rh + 32 * i + 4 * q4 + r, k = cq + l16;
            const float h = tanhf(z2[i][r] + b2[k]);
            sh2[row * LD + k] = h;
            if (MODE == kForward && cache && row < ns) cache[(size_t)(s0 + row) * 2 * H + H + k] = h;
          }
      __syncthreads();
      if (xr < TS) {  // output: eight threads per sample, whole waves
        const int r = xr, q = xc;
        float o = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) o = fmaf(w3[8 * k + q], sh2[r * LD + 8 * k + q], o);
        o += __shfl_xor(o, 1, 64);
        o += __shfl_xor(o, 2, 64);
        o += __shfl_xor(o, 4, 64);
        o += b3;
        if (q == 0) {
          if (MODE == kForward && r < ns) out[s0 + r] = o;
          if (MODE == kTrain) {
            const float e = r < ns ? o - yr : 0.f;
            sdo[r] = 2.f * e / (float)n;  // (a product with a rounded 2 / n would scale all gradients by its error)
            loss = fmaf(e, e, loss);
          }
        }
      }
      if (MODE == kTrain) __syncthreads();
    }
    if (MODE == kForward) continue;
    // dz2 = dout w3 (1 - h2^2), the gradients of b2 and w3: thread (k, 8 samples)
    {
      const int k = lane;
      const float wk = w3[k];
#pragma unroll
      for (int r = wv; r < TS; r += kWaves) {
        const float h = sh2[r * LD + k], d = sdo[r], z = d * wk * (1.f - h * h);
        sdz[r * LD + k] = z;
        gb2 += z;
        gw3 = fmaf(d, h, gw3);
      }
    }
    if (tid < TS) gb3 += sdo[tid];
    __syncthreads();
    f4r z1[NI];  // dz2 W2: rows s, columns m
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) z1[i][r] = 0.f;
#pragma unroll
    for (int k = 0; k < H; k += 4) {
      const float bw = w2[(k + q4) * LD + cq + l16];
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (TS > 16 || rh == 0)
          z1[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(sdz[(rh + 32 * i + l16) * LD + k + q4], bw, z1[i], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < TS; r += 4) {
      const float bh = sh1[(r + q4) * LD + cq + l16];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        g2[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(sdz[(r + q4) * LD + rh + 32 * i + l16], bh, g2[i], 0, 0, 0);
    }
    // dz1 (over h2, which is no longer needed), then the gradients of W1 and b1: dz1^T times
    // the inputs, four waves with 16 rows m each (columns 8 to 15 repeat 0 to 7)
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (TS > 16 || rh == 0)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = rh + 32 * i + 4 * q4 + r, m = cq + l16;
          const float h = sh1[row * LD + m];
          sh2[row * LD + m] = z1[i][r] * (1.f - h * h);
        }
    __syncthreads();
    if (wv < 4) {
#pragma unroll
      for (int r = 0; r < TS; r += 4)
        gx = __builtin_amdgcn_mfma_f32_16x16x4f32(sh2[(r + q4) * LD + cq + l16], sx[(r + q4) * 8 + (l16 & 7)], gx, 0, 0, 0);
    }
  }
  if (MODE == kForward) return;
  float* part = partial + (size_t)blockIdx.x * PROW;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[OFF_W2 + (rh + 32 * i + 4 * q4 + r) * H + cq + l16] = g2[i][r];
  if (wv < 4) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = cq + 4 * q4 + r;
      if (l16 < NIN) part[OFF_W1 + m * NIN + l16] = gx[r];
      else if (l16 == NIN) part[OFF_B1 + m] = gx[r];
    }
  }
  red[0][wv][lane] = gb2;
  red[1][wv][lane] = gw3;
  for (int o = 32; o > 0; o >>= 1) {
    gb3 += __shfl_xor(gb3, o, 64);
    loss += __shfl_xor(loss, o, 64);
  }
  if (lane == 0) {
    lred[0][wv] = gb3;
    lred[1][wv] = loss;
  }
  __syncthreads();
  if (tid < 2 * H + 2) {
    const int which = tid < 2 * H ? tid >> 6 : tid & 1;
    const float* v = tid < 2 * H ? &red[which][0][lane] : lred[which];
    const int step = tid < 2 * H ? H : 1;
    float s[kWaves];
#pragma unroll
    for (int k = 0; k < kWaves; ++k) s[k] = v[k * step];
#pragma unroll
    for (int w = kWaves / 2; w > 0; w >>= 1)
#pragma unroll
      for (int k = 0; k < w; ++k) s[k] += s[k + w];
    part[tid >= 2 * H ? (which ? NP : OFF_B3) : (which ? OFF_W3 : OFF_B2) + lane] = s[0];
  }
}

// Sums the rows of partial (32 parameters x 16 threads a workgroup), then dW or, training,
// Adam on the parameter and the loss
struct AdamArgs {
  float *W, *m, *v, *loss;
  float lr, b1, b2, eps, c1, c2, n;
};

__device__ inline void adam_update(float& W, float& m, float& v, float g, const AdamArgs& a) {
  const float mk = a.b1 * m + (1.f - a.b1) * g;
  const float vk = a.b2 * v + (1.f - a.b2) * g * g;
  m = mk;
  v = vk;
  W -= a.lr * (mk / a.c1) / (sqrtf(vk / a.c2) + a.eps);
}

template <bool kAdam>
__global__ __launch_bounds__(512) void sum_partials_kernel(const float* partial, int nblk, float* dW, AdamArgs a) {
  __shared__ float sh[16][32];
  const int c = threadIdx.x & 31, q = threadIdx.x >> 5, k = blockIdx.x * 32 + c;
  float acc = 0.f;
  if (k <= NP) {
#pragma unroll 4
    for (int b = q; b < nblk; b += 16) acc += partial[(size_t)b * PROW + k];
  }
  sh[q][c] = acc;
  __syncthreads();
  if (q != 0 || k > NP) return;
  float s[16];  // in pairs
#pragma unroll
  for (int b = 0; b < 16; ++b) s[b] = sh[b][c];
#pragma unroll
  for (int w = 8; w > 0; w >>= 1)
#pragma unroll
    for (int b = 0; b < w; ++b) s[b] += s[b + w];
  acc = s[0];
  if (kAdam) {
    if (k < NP) adam_update(a.W[k], a.m[k], a.v[k], acc, a);
    else *a.loss = acc / a.n;
  } else if (k < NP) {
    dW[k] = acc;
  }
}

__global__ void adam_kernel(const float* g, int n, AdamArgs a) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) adam_update(a.W[k], a.m[k], a.v[k], g[k], a);
}

// y[p] = log ||t_ij||_F - log(g W) for the core pairs, from the pass's pair_tnorm
__global__ void targets_kernel(const float* pair_tnorm, const double* log_scale, int n_core, int n_h, float* y,
                               int n_pairs) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n_pairs) return;
  int i = 0, rem = p;
  while (rem >= n_core - i) {
    rem -= n_core - i;
    ++i;
  }
  const int j = i + rem;
  y[p] = (float)(log((double)pair_tnorm[(size_t)i * n_h + j]) - log_scale[2 * (size_t)p]);
}

// mask: all ones, then core pairs whose predicted log-norm is below log(thr) set to 0.
//   mode 0: log(g W) + pred + margin;  mode 1: rigorous bound log(g U).
__global__ void mask_kernel(const float* pred, const double* log_scale, int n_core, int n_h, double log_thr,
                            double margin, int mode, uint8_t* mask, int* n_dropped, int n_pairs) {
  // phase 1 (all threads of the single workgroup): fill ones
  for (int k = threadIdx.x; k < n_h * n_h; k += blockDim.x) mask[k] = 1;
  __syncthreads();
  int dropped = 0;
  for (int p = threadIdx.x; p < n_pairs; p += blockDim.x) {
    const double ln = (mode == 0) ? log_scale[2 * (size_t)p] + (double)pred[p] + margin : log_scale[2 * (size_t)p + 1];
    if (ln < log_thr) {
      int i = 0, rem = p;
      while (rem >= n_core - i) {
        rem -= n_core - i;
        ++i;
      }
      const int j = i + rem;
      mask[(size_t)i * n_h + j] = 0;
      mask[(size_t)j * n_h + i] = 0;
      ++dropped;
    }
  }
  for (int off = 32; off > 0; off >>= 1) dropped += __shfl_xor(dropped, off, 64);
  __shared__ int sh[16];
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = dropped;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
    *n_dropped = t;
  }
}

// u* solving 2 u^2 e^{-u^2} = 1 - e^{-u^2} (maximum of (1 - e^{-u^2}) / u), by bisection
double regularizer_peak() {
  double lo = 0.5, hi = 2.0;
  for (int it = 0; it < 200; ++it) {
    const double mid = 0.5 * (lo + hi);
    if (2.0 * mid * mid * std::exp(-mid * mid) > -std::expm1(-mid * mid)) lo = mid;
    else hi = mid;
  }
  return 0.5 * (lo + hi);
}

int train_nblk(int64_t n) { return (int)((n + BW_SAMPLES - 1) / BW_SAMPLES); }

// Samples per tile and workgroups over n samples, with room for `rows` rows of partial sums:
// the tile with the least work on the busiest unit, a tile costing its samples and about 32
// more in fixed latency.  Twelve training steps, us: 200 samples 159, 194 with tiles of 64; 4096
// samples 182 and 208; 8192 samples 211 and 217.  (Tiles of 48, whose blocks do not fill the
// eight waves: 272 instead of 234 at 11000.)
struct NetPlan {
  int ts, groups;
};
NetPlan net_plan(int64_t n, int64_t rows) {
  NetPlan best{64, 1};
  int64_t least = INT64_MAX;
  for (int ts : {64, 32, 16}) {
    const int64_t tiles = (n + ts - 1) / ts, g = std::max<int64_t>(1, std::min<int64_t>({tiles, kMaxGroups, rows}));
    const int64_t cost = (tiles + g - 1) / g * (ts + 32);
    if (cost < least) {
      least = cost;
      best = NetPlan{ts, (int)g};
    }
  }
  return best;
}

template <int MODE>
void launch_mlp(const NetPlan& p, hipStream_t s, const float* W, const float* X, const float* y, int n, float* out,
                float* cache, const float* dout, float* partial) {
  const dim3 grid(p.groups), block(kThreads);
  if (p.ts == 64) hipLaunchKernelGGL((mlp_kernel<MODE, 64>), grid, block, 0, s, W, X, y, n, out, cache, dout, partial);
  else if (p.ts == 32) hipLaunchKernelGGL((mlp_kernel<MODE, 32>), grid, block, 0, s, W, X, y, n, out, cache, dout, partial);
  else hipLaunchKernelGGL((mlp_kernel<MODE, 16>), grid, block, 0, s, W, X, y, n, out, cache, dout, partial);
}

AdamArgs adam_args(float* W, float* m, float* v, float lr, float b1, float b2, float eps, int64_t step) {
  AdamArgs a{};
  a.W = W;
  a.m = m;
  a.v = v;
  a.lr = lr;
  a.b1 = b1;
  a.b2 = b2;
  a.eps = eps;
  a.c1 = (float)(1.0 - std::pow((double)b1, (double)step));
  a.c2 = (float)(1.0 - std::pow((double)b2, (double)step));
  return a;
}

}  // namespace

}  // namespace dfpt2

using namespace dfpt2;

extern "C" {

int pairscreen_num_params(void) { return NP; }

int pairscreen_workspace_size(const dfpt2_opts* opts, size_t* bytes) {
  g_last_error.clear();
  if (!bytes) return fail(DFPT2_ERR_INVALID_ARG, "bytes is null");
  PassPlan pl;
  int st = plan_pass(opts, &pl);
  if (st != DFPT2_OK) return st;
  // the second term is not used: each wave of pair_features_kernel forms the diagonal values itself
  *bytes = align_up(sizeof(double) * (size_t)(pl.n_core > 0 ? pl.n_core : 1) * pl.n_aux, 256) +
           align_up(sizeof(double) * (size_t)(pl.n_core > 0 ? pl.n_core : 1), 256) + 256;
  return DFPT2_OK;
}

int pairscreen_features(const dfpt2_opts* opts, const double* eps_hole, const double* eps_vir, const double* B,
                        float* feats, double* log_scale, void* workspace, size_t ws_bytes, dfpt2_stream_t stream) {
  g_last_error.clear();
  PassPlan pl;
  int st = plan_pass(opts, &pl);
  if (st != DFPT2_OK) return st;
  if (!eps_hole || !eps_vir || !B || !feats || !log_scale || !workspace)
    return fail(DFPT2_ERR_INVALID_ARG, "null pointer argument");
  size_t need = 0;
  pairscreen_workspace_size(opts, &need);
  if (ws_bytes < need) return fail(DFPT2_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, need);
  if (pl.n_core == 0) return DFPT2_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  double* q2 = reinterpret_cast<double*>(ws);
  ProfScope ps(DFPT2_STAGE_SCREEN, s);
  hipLaunchKernelGGL(colnorm2_kernel, dim3((pl.n_aux + 63) / 64, pl.n_core), dim3(1024), 0, s, B, pl.n_v, pl.n_aux,
                     q2);
  const double x_star = regularizer_peak() / std::sqrt(opts->s);
  hipLaunchKernelGGL(pair_features_kernel, dim3((pl.n_up + 3) / 4), dim3(256), 0, s, q2, eps_hole, eps_vir, pl.n_v,
                     pl.n_core, pl.n_aux, opts->s, x_star, feats, log_scale, pl.n_up);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DFPT2_OK : hip_fail(e, "features");
}

int pairscreen_mlp_forward(const float* W, const float* feats, int64_t n, float* pred, float* act_cache,
                           dfpt2_stream_t stream) {
  g_last_error.clear();
  if (!W || !feats || !pred) return fail(DFPT2_ERR_INVALID_ARG, "null pointer argument");
  if (n < 0 || n > (1ll << 30)) return fail(DFPT2_ERR_INVALID_ARG, "bad sample count");
  if (n == 0) return DFPT2_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope ps(DFPT2_STAGE_SCREEN, s);
  NetPlan p = net_plan(n, kMaxGroups);
  p.groups = (int)std::min<int64_t>((n + p.ts - 1) / p.ts, 2048);
  launch_mlp<kForward>(p, s, W, feats, nullptr, (int)n, pred, act_cache, nullptr, nullptr);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DFPT2_OK : hip_fail(e, "mlp forward");
}

int pairscreen_backward_workspace_size(int64_t n, size_t* bytes) {
  g_last_error.clear();
  if (!bytes || n < 0) return fail(DFPT2_ERR_INVALID_ARG, "bad argument");
  *bytes = sizeof(float) * (size_t)(train_nblk(n) > 0 ? train_nblk(n) : 1) * NP + 256;
  return DFPT2_OK;
}

int pairscreen_mlp_backward(const float* W, const float* feats, const float* act_cache, const float* dpred, int64_t n,
                            float* dW, void* workspace, size_t ws_bytes, dfpt2_stream_t stream) {
  g_last_error.clear();
  if (!W || !feats || !act_cache || !dpred || !dW || !workspace)
    return fail(DFPT2_ERR_INVALID_ARG, "null pointer argument");
  if (n <= 0 || n > (1ll << 30)) return fail(DFPT2_ERR_INVALID_ARG, "bad sample count");
  size_t need = 0;
  pairscreen_backward_workspace_size(n, &need);
  if (ws_bytes < need) return fail(DFPT2_ERR_WORKSPACE, "workspace too small");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope ps(DFPT2_STAGE_SCREEN, s);
  float* partial = static_cast<float*>(workspace);
  const NetPlan p = net_plan(n, (int64_t)(need / sizeof(float) / PROW));
  launch_mlp<kBackward>(p, s, W, feats, nullptr, (int)n, nullptr, const_cast<float*>(act_cache), dpred, partial);
  hipLaunchKernelGGL(sum_partials_kernel<false>, dim3((NP + 32) / 32), dim3(512), 0, s, partial, p.groups, dW, AdamArgs{});
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DFPT2_OK : hip_fail(e, "mlp backward");
}

int pairscreen_adam_step(float* W, const float* dW, float* m, float* v, int64_t n_params, float lr, float b1, float b2,
                         float eps, int64_t step, dfpt2_stream_t stream) {
  g_last_error.clear();
  if (!W || !dW || !m || !v) return fail(DFPT2_ERR_INVALID_ARG, "null pointer argument");
  if (n_params <= 0 || step < 1 || !(lr > 0.f) || !(b1 >= 0.f && b1 < 1.f) || !(b2 >= 0.f && b2 < 1.f) || !(eps > 0.f))
    return fail(DFPT2_ERR_INVALID_ARG, "bad Adam hyper-parameters");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope ps(DFPT2_STAGE_SCREEN, s);
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n_params + 255) / 256)), dim3(256), 0, s, dW, (int)n_params,
                     adam_args(W, m, v, lr, b1, b2, eps, step));
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DFPT2_OK : hip_fail(e, "adam");
}

int pairscreen_train_workspace_size(int64_t n, size_t* bytes) {
  g_last_error.clear();
  if (!bytes || n <= 0) return fail(DFPT2_ERR_INVALID_ARG, "bad argument");
  // Room for predictions, their gradients, activations and dW, none of which a step writes any more:
  // rows of partial sums take it (net_plan), and the size that callers are told stays.
  size_t b = 0;
  b += align_up(sizeof(float) * n, 256);
  b += align_up(sizeof(float) * n, 256);
  b += align_up(sizeof(float) * n * 2 * H, 256);
  b += align_up(sizeof(float) * NP, 256);
  size_t bw = 0;
  pairscreen_backward_workspace_size(n, &bw);
  b += align_up(bw, 256);
  *bytes = b;
  return DFPT2_OK;
}

int pairscreen_train(float* W, float* m, float* v, const float* feats, const float* y, int64_t n, int64_t steps,
                     int64_t step0, float lr, float* losses, void* workspace, size_t ws_bytes, dfpt2_stream_t stream) {
  g_last_error.clear();
  if (!W || !m || !v || !feats || !y || !losses || !workspace) return fail(DFPT2_ERR_INVALID_ARG, "null pointer");
  if (n <= 0 || steps <= 0 || step0 < 0 || !(lr > 0.f)) return fail(DFPT2_ERR_INVALID_ARG, "bad argument");
  size_t need = 0;
  pairscreen_train_workspace_size(n, &need);
  if (ws_bytes < need) return fail(DFPT2_ERR_WORKSPACE, "workspace too small");
  float* partial = static_cast<float*>(workspace);
  const NetPlan p = net_plan(n, (int64_t)(need / sizeof(float) / PROW));
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  for (int64_t t = 1; t <= steps; ++t) {
    ProfScope ps(DFPT2_STAGE_SCREEN, s);
    launch_mlp<kTrain>(p, s, W, feats, y, (int)n, nullptr, nullptr, nullptr, partial);
    AdamArgs a = adam_args(W, m, v, lr, 0.9f, 0.999f, 1e-8f, step0 + t);
    a.loss = losses + (t - 1);
    a.n = (float)n;
    hipLaunchKernelGGL(sum_partials_kernel<true>, dim3((NP + 32) / 32), dim3(512), 0, s, partial, p.groups, nullptr, a);
    const hipError_t le = hipGetLastError();
    if (le != hipSuccess) return hip_fail(le, "train");
  }
  hipError_t e = hipStreamSynchronize(s);
  prof_flush();
  return e == hipSuccess ? DFPT2_OK : hip_fail(e, "train sync");
}

int pairscreen_targets(const float* pair_tnorm, const double* log_scale, int64_t n_core, int64_t n_h, float* y,
                       dfpt2_stream_t stream) {
  g_last_error.clear();
  if (!pair_tnorm || !log_scale || !y) return fail(DFPT2_ERR_INVALID_ARG, "null pointer");
  if (n_core < 0 || n_h < n_core || n_core > 1024) return fail(DFPT2_ERR_INVALID_ARG, "bad hole counts");
  const int np = (int)(n_core * (n_core + 1) / 2);
  if (np == 0) return DFPT2_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(targets_kernel, dim3((np + 255) / 256), dim3(256), 0, s, pair_tnorm, log_scale, (int)n_core,
                     (int)n_h, y, np);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? DFPT2_OK : hip_fail(e, "targets");
}

int pairscreen_build_mask(const float* pred, const double* log_scale, int64_t n_core, int64_t n_h, double threshold,
                          double margin, int mode, uint8_t* mask, int64_t* n_dropped, void* workspace,
                          size_t ws_bytes, dfpt2_stream_t stream) {
  g_last_error.clear();
  if (!log_scale || !mask || !workspace || ws_bytes < 64) return fail(DFPT2_ERR_INVALID_ARG, "null pointer");
  if (mode != 0 && mode != 1) return fail(DFPT2_ERR_INVALID_ARG, "mode must be 0 (network) or 1 (bound)");
  if (mode == 0 && !pred) return fail(DFPT2_ERR_INVALID_ARG, "pred is null in network mode");
  if (!(threshold > 0.0) || !std::isfinite(margin)) return fail(DFPT2_ERR_INVALID_ARG, "threshold must be > 0");
  if (n_core < 0 || n_h < n_core || n_core > 1024 || n_h > 1088) return fail(DFPT2_ERR_INVALID_ARG, "bad hole counts");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope ps(DFPT2_STAGE_SCREEN, s);
  int* d_drop = static_cast<int*>(workspace);
  const int np = (int)(n_core * (n_core + 1) / 2);
  hipLaunchKernelGGL(mask_kernel, dim3(1), dim3(1024), 0, s, pred, log_scale, (int)n_core, (int)n_h,
                     std::log(threshold), margin, mode, mask, d_drop, np);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "mask");
  ps.close();
  if (n_dropped) {
    int h = 0;
    if ((e = hipMemcpyAsync(&h, d_drop, sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess) return hip_fail(e, "copy");
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "sync");
    prof_flush();
    *n_dropped = h;
  }
  return DFPT2_OK;
}

}  // extern "C"
