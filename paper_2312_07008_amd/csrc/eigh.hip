// FP64 symmetric eigensolver on the GPU, for the natural-orbital problem of
// Eq. 8 (Gamma V = n V) and for the recanonicalization of the kept space.
//
//   1. Householder reduction to tridiagonal form, one column per step on the full
//      symmetric matrix: the reflector, p = tau A v and the rank-2 update
//      A -= v w^T + w v^T with w = p - (tau/2)(p.v) v, applied lazily with the next
//      column's product.  Up to n = 2048 in one launch, the matrix in registers (one
//      workgroup up to n = 128, cooperating workgroups above); then one launch per column,
//      two above n = 2731.
//   2. Splitting at negligible off-diagonal entries, then every eigenvalue by
//      multisection on Sturm counts (one, two or four waves per eigenvalue, a point per lane).
//   3. Eigenvectors of the tridiagonal matrix: isolated eigenvalues by twisted
//      factorizations of T - lambda I, two solves each; the others by inverse iteration with a partially
//      pivoted LU.  Eigenvalues closer than a small multiple of ||T|| form a group that
//      one thread handles in order, orthogonalizing every iterate against the group's
//      earlier vectors.
//   4. Back-transformation Z <- H_0 H_1 ... H_{n-3} Z in compact-WY blocks of 16
//      reflectors on the matrix pipe, 16 columns of Z in a workgroup's registers (above
//      n = 2048 blocks of 8, one workgroup per 2 or 1 columns held in LDS).
//   5. One first-order orthonormalization of all columns (two FP64 GEMMs): it
//      restores orthogonality between vectors of close eigenvalues that were formed apart.
//   6. Columns sorted by eigenvalue and oriented so that the largest-magnitude
//      component is positive.
// n = 1200, ms before and after the resident reduction, the product-form counts, the
// twisted factorizations and the matrix-pipe back-transformation: reduction 11.6 -> 5.0,
// eigenvalues 1.8 -> 0.46, vectors 5.9 -> 0.44, back-transformation 2.0 -> 0.48, the whole
// call 22.5 -> 6.7.
#include <algorithm>
#include <cmath>
#include <cfloat>
#include <type_traits>

#include "common.h"
#include "eigh.h"

namespace dfpt2 {

namespace {

__device__ inline double block_sum(double v, double* sh) {
  // 256-thread workgroup sum; sh holds >= 4 doubles; ends with a barrier
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  const int nw = blockDim.x >> 6;
  for (int k = 0; k < nw; ++k) t += sh[k];
  __syncthreads();
  return t;
}

// ---------------------------------------------------------------- step a
// Reflector of column k and p = tau A22 v, rows split over the grid.
__global__ __launch_bounds__(256) void tridiag_step_a(const double* A, int n, int k, double* Vs,
                                                      double* tau, double* d, double* e, double* p) {
  extern __shared__ double vsh[];  // m doubles
  __shared__ double red[8];
  const int m = n - k - 1;
  const double* rowk = A + (size_t)k * n + (k + 1);  // x_i = A[k][k+1+i] (symmetric)
  double s2 = 0.0;
  for (int i = 1 + threadIdx.x; i < m; i += blockDim.x) s2 += rowk[i] * rowk[i];
  s2 = block_sum(s2, red);
  const double alpha = rowk[0];
  double t = 0.0, beta = alpha, scale = 0.0;
  if (s2 > 0.0) {
    const double mu = sqrt(alpha * alpha + s2);
    beta = (alpha > 0.0) ? -mu : mu;
    t = (beta - alpha) / beta;
    scale = 1.0 / (alpha - beta);
  }
  for (int i = threadIdx.x; i < m; i += blockDim.x) vsh[i] = (i == 0) ? 1.0 : rowk[i] * scale;
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < m; i += blockDim.x) Vs[(size_t)k * n + i] = vsh[i];
    if (threadIdx.x == 0) {
      tau[k] = t;
      e[k] = beta;
      d[k] = A[(size_t)k * n + k];
    }
  }
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int nwaves = gridDim.x * (blockDim.x >> 6);
  for (int r = gw; r < m; r += nwaves) {
    const double* row = A + (size_t)(k + 1 + r) * n + (k + 1);
    double acc = 0.0;
    for (int c = lane; c < m; c += 64) acc += row[c] * vsh[c];
    acc = wave_sum(acc);
    if (lane == 0) p[r] = t * acc;
  }
}

// ---------------------------------------------------------------- step b
// A22 -= v w^T + w v^T, w = p - (tau/2)(p.v) v.  grid.x over columns, grid.y over row bands.
__global__ __launch_bounds__(256) void tridiag_step_b(double* A, int n, int k, const double* Vs,
                                                      const double* tau, const double* p) {
  __shared__ double red[8];
  const int m = n - k - 1;
  const double t = tau[k];
  if (t == 0.0) return;
  const double* v = Vs + (size_t)k * n;
  double dot = 0.0;
  for (int i = threadIdx.x; i < m; i += blockDim.x) dot += p[i] * v[i];
  dot = block_sum(dot, red);
  const double K = 0.5 * t * dot;
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= m) return;
  const double vc = v[c];
  const double wc = p[c] - K * vc;
  const int rows_per = (m + gridDim.y - 1) / gridDim.y;
  const int r0 = blockIdx.y * rows_per;
  const int r1 = min(m, r0 + rows_per);
  for (int r = r0; r < r1; ++r) {
    const double vr = v[r];
    const double wr = p[r] - K * vr;
    double* a = A + (size_t)(k + 1 + r) * n + (k + 1 + c);
    *a -= vr * wc + wr * vc;
  }
}

// ---------------------------------------------------------------- fused step
// Column k with the rank-2 update of column k - 1 applied lazily: the update
// A -= v' w'^T + w' v'^T of column k - 1 (over indices k .. n - 1; w' = p' -
// (tau'/2)(p'.v') v' rebuilt here from p' = p of column k - 1) is applied to row k
// on the fly (it gives the reflector and d[k]) and, row by row, to the trailing
// block k + 1 .. n - 1, which is stored back and multiplied by v_k in the same
// pass: one launch per column instead of two, and each trailing row read and
// written once.  v', w' and v_k are staged in LDS ((3 m + 2) doubles, m = n - k - 1).
__global__ __launch_bounds__(256) void tridiag_step_lazy(double* A, int n, int k, double* Vs, double* tau,
                                                         double* d, double* e, const double* p_prev,
                                                         double* p_out) {
  extern __shared__ double sh[];
  const int m = n - k - 1;
  double* vsh = sh;           // v_k: m
  double* vpr = sh + m;       // v': m + 1 (index k + i)
  double* wpr = vpr + m + 1;  // w': m + 1
  __shared__ double red[8];
  if (k > 0) {  // workgroup-uniform
    const double* vp = Vs + (size_t)(k - 1) * n;
    double dot = 0.0;
    for (int i = threadIdx.x; i <= m; i += blockDim.x) dot += p_prev[i] * vp[i];
    dot = block_sum(dot, red);
    const double K = 0.5 * tau[k - 1] * dot;
    for (int i = threadIdx.x; i <= m; i += blockDim.x) {
      vpr[i] = vp[i];
      wpr[i] = p_prev[i] - K * vp[i];
    }
  } else {
    for (int i = threadIdx.x; i <= m; i += blockDim.x) vpr[i] = wpr[i] = 0.0;
  }
  __syncthreads();
  const double v0 = vpr[0], w0 = wpr[0];
  const double* rowk = A + (size_t)k * n + (k + 1);
  double s2 = 0.0;
  for (int i = 1 + threadIdx.x; i < m; i += blockDim.x) {
    const double x = rowk[i] - (v0 * wpr[1 + i] + w0 * vpr[1 + i]);
    s2 += x * x;
  }
  s2 = block_sum(s2, red);
  const double alpha = rowk[0] - (v0 * wpr[1] + w0 * vpr[1]);
  double t = 0.0, beta = alpha, scale = 0.0;
  if (s2 > 0.0) {
    const double mu = sqrt(alpha * alpha + s2);
    beta = (alpha > 0.0) ? -mu : mu;
    t = (beta - alpha) / beta;
    scale = 1.0 / (alpha - beta);
  }
  for (int i = threadIdx.x; i < m; i += blockDim.x)
    vsh[i] = (i == 0) ? 1.0 : (rowk[i] - (v0 * wpr[1 + i] + w0 * vpr[1 + i])) * scale;
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < m; i += blockDim.x) Vs[(size_t)k * n + i] = vsh[i];
    if (threadIdx.x == 0) {
      tau[k] = t;
      e[k] = beta;
      d[k] = A[(size_t)k * n + k] - 2.0 * v0 * w0;
    }
  }
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int nwaves = gridDim.x * (blockDim.x >> 6);
  for (int r = gw; r < m; r += nwaves) {
    double* row = A + (size_t)(k + 1 + r) * n + (k + 1);
    const double vr = vpr[1 + r], wr = wpr[1 + r];
    double acc = 0.0;
    for (int c = lane; c < m; c += 64) {
      const double a = row[c] - (vr * wpr[1 + c] + wr * vpr[1 + c]);
      row[c] = a;
      acc += a * vsh[c];
    }
    acc = wave_sum(acc);
    if (lane == 0) p_out[r] = t * acc;
  }
}

// ---------------------------------------------------------------- resident form
// The whole reduction in one launch, the matrix in registers (n <= kResidentMax).  The
// launch-per-column form above pays ~10 us a column at n = 1200 for a launch, two passes
// of vectors through memory and the row's way to and from L2; the arithmetic is 1 us.
// Per column, every workgroup needs two vectors: p of the previous column and the row k
// as its update by the column before left it (its owner hands it out).  It forms w and the
// reflector for itself (each thread a few entries, two workgroup sums), and every wave
// updates its row and multiplies it by the reflector in the same pass.  All workgroups run
// the same operations on the same numbers, so that they agree to the bit.
//
// kResRows rows per wave (lane l holds columns l, l + 64, ...), 4 waves per workgroup, row
// r on workgroup r mod G.  The two vectors go through memory, one slot per column and entry that
// starts as kEmpty (a NaN pattern that no arithmetic here produces) and is written once, by
// a 64-bit atomic store at device scope; readers poll the entry itself, so that a column
// costs one trip through memory and no grid barrier.  All workgroups have to be resident:
// the launch is cooperative, and every wait is bounded (kWaitTicks, or as soon as another
// workgroup has given up): then *status = 2 and the caller starts again with the
// launch-per-column form.  A column takes 2.5 us at n = 130 (the trip through memory, two
// workgroup sums, a square root and a division) and 4.2 us at n = 1200.
constexpr int kResidentMax = 2048;
constexpr int kSmallMax = 128;
constexpr unsigned long long kEmpty = ~0ull;
constexpr unsigned long long kWaitTicks = 100000000ull;  // of the 100 MHz counter: 1 s

template <int CTRL, int ROWS>
__device__ inline double dpp_add(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, false);
  return x + __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

__device__ inline double read_lane(double x, int lane) {  // lane uniform
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// sum over the wave by DPP (rows of 16, then across rows), on every lane
__device__ inline double wave_sum_dpp(double v) {
  v = dpp_add<0x111, 0xf>(v);  // row_shr:1
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return read_lane(v, 63);
}

// 1 / q to within an ulp or two (finite, normal q): the hardware's estimate and two
// Newton steps, a third of the latency of a correctly rounded division
__device__ inline double fast_rcp(double q) {
  double r = __builtin_amdgcn_rcp(q);
  r = fma(fma(-q, r, 1.0), r, r);
  return fma(fma(-q, r, 1.0), r, r);
}

// sqrt(a) to within an ulp or two (a well inside the normal range): the hardware's estimate
// of 1 / sqrt(a), two Newton steps and one of the root itself
__device__ inline double fast_sqrt(double a) {
  double r = __builtin_amdgcn_rsq(a);
  r = fma(0.5 * r, fma(-a * r, r, 1.0), r);
  r = fma(0.5 * r, fma(-a * r, r, 1.0), r);
  const double g = a * r;
  return fma(fma(-g, g, a), 0.5 * r, g);
}

// reflector of a column from alpha = x_0 and s2 = sum of the other x_i^2: v = (1, scale x_i).
// Every column's chain goes through it: with rounded roots and divisions, and
// with every column of a row updated to the end, the reduction of a 60 x 60 matrix took 102 us, 81 so.
// t is a quotient, not a product with a reciprocal: its remainder corrects it.  The eigenpairs of
// 60 to 1200 rows are then off by the same as with rounded roots and divisions.
__device__ inline void reflector(double alpha, double s2, double& beta, double& t, double& scale) {
  t = scale = 0.0;
  beta = alpha;
  if (s2 > 0.0) {
    const double a = fma(alpha, alpha, s2);
    if (a > 1e-200 && a < 1e200) {
      const double mu = fast_sqrt(a);
      beta = (alpha > 0.0) ? -mu : mu;
      const double rb = fast_rcp(beta), num = beta - alpha;
      t = num * rb;
      t = fma(fma(-beta, t, num), rb, t);
      scale = fast_rcp(alpha - beta);
    } else {
      const double mu = sqrt(a);
      beta = (alpha > 0.0) ? -mu : mu;
      t = (beta - alpha) / beta;
      scale = 1.0 / (alpha - beta);
    }
  }
}

__device__ inline void publish(unsigned long long* p, double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  __hip_atomic_store(p, u == kEmpty ? 0x7ff8000000000000ull : u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kResThreads = 256;
constexpr int kResRows = 2;  // rows per wave: 1200 rows 7.9, 6.8, 7.7, 10.3 ms in all with 1, 2, 4, 8

// J 64-wide column groups (n <= 64 J), RW rows per wave
template <int J, int RW>
__global__ __launch_bounds__(kResThreads) void tridiag_resident(const double* A_in, int n, double* A_out, double* Vs,
                                                        double* tau, double* d, double* e, unsigned long long* P,
                                                        unsigned long long* R, double* p_last, int* status, int G,
                                                        unsigned long long wait) {
  constexpr int NC = 64 * J, NT = kResThreads, NW = NT / 64, Q = (NC + NT - 1) / NT;
  __shared__ double ws[NC], vs[NC], xs[NC];  // w, v of the previous column, x of this one (0 up to k + 1)
  __shared__ double part1[NW], part2[NW], sc[3];
  __shared__ int dead;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wg = blockIdx.x;  // of G
  int row[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) row[r] = wg + G * (wv + NW * r);
  const bool writer = wg == (n - 1) % G;            // owns row n - 1, runs to the end
  const int last = wg + (n - 1 - wg) / G * G;       // largest row of the workgroup
  double a[RW][J], vo[Q], v_row[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    v_row[r] = 0.0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = lane + 64 * j;
      a[r][j] = (row[r] < n && c < n) ? A_in[(size_t)row[r] * n + c] : 0.0;
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) vo[q] = 0.0;
  for (int c = tid; c < NC; c += NT) ws[c] = vs[c] = xs[c] = 0.0;
  if (tid == 0) dead = 0;
  double t_prev = 0.0;
  __syncthreads();
  for (int k = 0; k + 2 < n; ++k) {
    if (k >= last) break;  // workgroup-uniform: nothing left to update
    // p of column k - 1 and row k, entries c = tid + NT q
    double p[Q], x[Q];
    if (k == 0) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int c = tid + NT * q;
        p[q] = 0.0;
        x[q] = c < n ? A_in[c] : 0.0;
      }
    } else {
      unsigned long long pv[Q], rv[Q];
      unsigned long long t0 = 0;
      for (int spin = 0;; ++spin) {
        bool ok = true;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int c = tid + NT * q;
          pv[q] = rv[q] = 0;
          if (c >= k && c < n) {
            pv[q] = __hip_atomic_load(P + (size_t)(k - 1) * n + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            rv[q] = __hip_atomic_load(R + (size_t)k * n + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) ok = ok && pv[q] != kEmpty && rv[q] != kEmpty;
        if (ok) break;
        if ((spin & 255) == 255) {
          const unsigned long long now = wall_clock64();
          if (spin == 255) t0 = now;
          if (now - t0 > wait || __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            dead = 1;
            break;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        p[q] = __builtin_bit_cast(double, pv[q]);
        x[q] = __builtin_bit_cast(double, rv[q]);
      }
    }
    // K = tau / 2 p . v of the previous column (p and v are zero at c < k and c >= n)
    double dot = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      dot = fma(p[q], vo[q], dot);
      if (tid + NT * q == k) {
        sc[0] = p[q];
        sc[1] = x[q];
      }
    }
    dot = wave_sum_dpp(dot);
    if (lane == 0) part1[wv] = dot;
    __syncthreads();
    if (dead) {  // workgroup-uniform
      if (tid == 0) __hip_atomic_store(status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    dot = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) dot += part1[q];
    const double K = 0.5 * t_prev * dot;
    const double v0 = k > 0 ? 1.0 : 0.0, w0 = k > 0 ? sc[0] - K : 0.0, dk = sc[1] - 2.0 * v0 * w0;
    // w, and x = row k with the update of column k - 1 (kept beyond k + 1; alpha = x_{k+1})
    double s2 = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int c = tid + NT * q;
      const double w = fma(-K, vo[q], p[q]);
      x[q] -= fma(v0, w, w0 * vo[q]);
      if (c == k + 1) sc[2] = x[q];
      if (c <= k + 1 || c >= n) x[q] = 0.0;
      s2 = fma(x[q], x[q], s2);
      if (c < NC) {
        ws[c] = w;
        vs[c] = vo[q];
        xs[c] = x[q];
      }
    }
    s2 = wave_sum_dpp(s2);
    if (lane == 0) part2[wv] = s2;
    __syncthreads();
    s2 = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) s2 += part2[q];
    const double alpha = sc[2];
    double beta, t, scale;
    reflector(alpha, s2, beta, t, scale);
    // the wave's rows: update by column k - 1, then their products with (1, scale x)
    const int j0 = k >> 6, j1 = (k + 1) >> 6, l1 = (k + 1) & 63;
    double acc[RW], ak[RW], w_row[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      acc[r] = ak[r] = 0.0;
      w_row[r] = row[r] < n ? ws[row[r]] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (j >= j0) {
        const int c = lane + 64 * j;
        const double wc = ws[c], vc = vs[c], xc = xs[c];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
          a[r][j] -= fma(v_row[r], wc, w_row[r] * vc);
          acc[r] = fma(a[r][j], xc, acc[r]);
          if (j == j1) ak[r] = read_lane(a[r][j], l1);
        }
      }
#pragma unroll
    for (int r = 0; r < RW; ++r) acc[r] = wave_sum_dpp(acc[r]);
#pragma unroll
    for (int r = 0; r < RW; ++r)
      if (row[r] > k && row[r] < n) {  // wave-uniform
        const double pr = t * fma(scale, acc[r], ak[r]);
        if (lane == 0) {
          publish(P + (size_t)k * n + row[r], pr);
          if (k + 3 == n) p_last[row[r] - (k + 1)] = pr;
        }
        if (row[r] == k + 1) {
#pragma unroll
          for (int j = 0; j < J; ++j) {
            const int c = lane + 64 * j;
            if (c > k && c < n) publish(R + (size_t)(k + 1) * n + c, a[r][j]);
          }
        }
        if (k + 3 == n) {  // the last 2 x 2 block, with the update of column n - 3 pending
#pragma unroll
          for (int j = 0; j < J; ++j) {
            const int c = lane + 64 * j;
            if (c >= n - 2 && c < n) A_out[(size_t)row[r] * n + c] = a[r][j];
          }
        }
        v_row[r] = row[r] == k + 1 ? 1.0 : xs[row[r]] * scale;
      }
    t_prev = t;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int c = tid + NT * q;
      vo[q] = c == k + 1 ? 1.0 : x[q] * scale;
      if (writer && c > k && c < n) Vs[(size_t)k * n + (c - k - 1)] = vo[q];
    }
    if (writer && tid == 0) {
      tau[k] = t;
      e[k] = beta;
      d[k] = dk;
    }
  }
}

// The same for n <= 4 N4 <= kSmallMax in one workgroup: four lanes per row (N4 columns
// each, c = 4 i + lane), the two vectors in LDS, three barriers a column.  n = 60: 4.9 us
// a column with a launch each, 1.5 us so.  A row's product goes to four sums: with one, and the
// reciprocal in the reflector, the eigenvalues' rms error over 120 matrices of 100 and 128 rows was
// 1.00 to 1.04 times that of the form with a launch each, 0.93 to 0.99 so, in the same time.
template <int N4>
__global__ __launch_bounds__(16 * N4) void tridiag_small(const double* A_in, int n, double* A_out, double* Vs,
                                                         double* tau, double* d, double* e, double* p_last, int* status) {
  constexpr int NC = 4 * N4, NW = N4 / 4;
  __shared__ double ps[NC], rs[NC];          // p of the previous column, row k
  __shared__ double ws[NC], vs[NC], xs[NC];  // w, v of the previous column, x of this one (0 up to k + 1)
  __shared__ double part1[NW], part2[NW], sc[1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = tid >> 2, q4 = tid & 3;
  double a[N4], vo = 0.0, v_row = 0.0, t_prev = 0.0;
  if (tid == 0) *status = 0;
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    const int c = 4 * i + q4;
    a[i] = (row < n && c < n) ? A_in[(size_t)row * n + c] : 0.0;
  }
  if (tid < NC) {
    ps[tid] = 0.0;
    rs[tid] = tid < n ? A_in[tid] : 0.0;
  }
  // columns k .. k1 - 1, whose rows have nothing left in the first I0 of a lane's columns
  auto columns = [&](auto I0, int k, const int k1) __attribute__((always_inline)) {
    for (; k < k1 && k + 2 < n; ++k) {
      __syncthreads();
      double p = 0.0, x = 0.0;  // thread c < NC: entry c (threads beyond hold zeros)
      if (tid >= k && tid < n) {
        p = ps[tid];
        x = rs[tid];
      }
      double s = wave_sum_dpp(p * vo);
      if (lane == 0) part1[wv] = s;
      const double pk = ps[k], rk = rs[k];
      __syncthreads();
      double dot = 0.0;
  #pragma unroll
      for (int q = 0; q < NW; ++q) dot += part1[q];
      const double K = 0.5 * t_prev * dot, v0 = k > 0 ? 1.0 : 0.0, w0 = k > 0 ? pk - K : 0.0;
      const double w = fma(-K, vo, p);
      x -= fma(v0, w, w0 * vo);
      if (tid == k + 1) sc[0] = x;
      if (tid <= k + 1 || tid >= n) x = 0.0;
      if (tid < NC) {
        ws[tid] = w;
        vs[tid] = vo;
        xs[tid] = x;
      }
      s = wave_sum_dpp(x * x);
      if (lane == 0) part2[wv] = s;
      __syncthreads();
      double s2 = 0.0;
  #pragma unroll
      for (int q = 0; q < NW; ++q) s2 += part2[q];
      double beta, t, scale;
      reflector(sc[0], s2, beta, t, scale);
      double ac[4] = {}, ak = 0.0;
      const double w_row = ws[row];
  #pragma unroll
      for (int i = I0(); i < N4; ++i) {
        const int c = 4 * i + q4;
        a[i] -= fma(v_row, ws[c], w_row * vs[c]);
        ac[i & 3] = fma(a[i], xs[c], ac[i & 3]);
        if (c == k + 1) ak = a[i];
      }
      double acc = fma(scale, (ac[0] + ac[1]) + (ac[2] + ac[3]), ak);  // ak: on one of the row's lanes
      acc += __shfl_xor(acc, 1, 64);
      acc += __shfl_xor(acc, 2, 64);
      if (row > k && row < n) {
        if (q4 == 0) {
          ps[row] = t * acc;
          if (k + 3 == n) p_last[row - (k + 1)] = t * acc;
        }
        if (row == k + 1) {
  #pragma unroll
          for (int i = I0(); i < N4; ++i) {
            const int c = 4 * i + q4;
            if (c > k) rs[c] = a[i];
          }
        }
        if (k + 3 == n) {  // the last 2 x 2 block, with the update of column n - 3 pending
  #pragma unroll
          for (int i = I0(); i < N4; ++i) {
            const int c = 4 * i + q4;
            if (c >= n - 2 && c < n) A_out[(size_t)row * n + c] = a[i];
          }
        }
        v_row = row == k + 1 ? 1.0 : xs[row] * scale;
      }
      vo = tid == k + 1 ? 1.0 : x * scale;
      if (tid > k && tid < n) Vs[(size_t)k * n + (tid - k - 1)] = vo;
      if (tid == 0) {
        tau[k] = t;
        e[k] = beta;
        d[k] = rk - 2.0 * v0 * w0;
      }
      t_prev = t;
    }
  };
  columns(std::integral_constant<int, 0>{}, 0, N4);
  columns(std::integral_constant<int, N4 / 4>{}, N4, 2 * N4);
  columns(std::integral_constant<int, N4 / 2>{}, 2 * N4, 3 * N4);
  columns(std::integral_constant<int, 3 * N4 / 4>{}, 3 * N4, 4 * N4);
}

// slots of the resident form
__global__ void fill_empty(unsigned long long* p, size_t n, int* status) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *status = 0;
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) p[k] = kEmpty;
}

template <int J, int RW>
hipError_t launch_resident_multi(const double* A_in, int n, double* A_out, double* Vs, double* tau, double* d, double* e,
                                 unsigned long long* P, unsigned long long* R, double* p_last, int* status,
                                 hipStream_t st, EighPath path) {
  int G = (n + 4 * RW - 1) / (4 * RW);
  unsigned long long wait = path == EighPath::kMissed ? kWaitTicks / 1000 : kWaitTicks;
  void* args[] = {&A_in, &n, &A_out, &Vs, &tau, &d, &e, &P, &R, &p_last, &status, &G, &wait};
  return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&tridiag_resident<J, RW>),
                                    dim3(path == EighPath::kMissed ? G - 1 : G), dim3(kResThreads), args, 0, st);
}

// false: not launched (the caller takes the launch-per-column form)
bool launch_resident(const double* A_in, int n, double* A_out, double* Vs, double* tau, double* d, double* e,
                     unsigned long long* P, unsigned long long* R, double* p_last, int* status, hipStream_t st,
                     EighPath path) {
  if (path == EighPath::kRefused) return false;
  if (n <= kSmallMax) {
    if (n <= 64) hipLaunchKernelGGL(tridiag_small<16>, dim3(1), dim3(256), 0, st, A_in, n, A_out, Vs, tau, d, e, p_last, status);
    else hipLaunchKernelGGL(tridiag_small<32>, dim3(1), dim3(512), 0, st, A_in, n, A_out, Vs, tau, d, e, p_last, status);
    return true;
  }
  const size_t slots = 2 * (size_t)n * n;
  hipLaunchKernelGGL(fill_empty, dim3((unsigned)std::min<size_t>(2048, (slots + 255) / 256)), dim3(256), 0, st, P, slots, status);
  hipError_t err = hipErrorInvalidValue;
#define DFPT2_RESIDENT(J) err = launch_resident_multi<J, kResRows>(A_in, n, A_out, Vs, tau, d, e, P, R, p_last, status, st, path)
  if (n <= 256) DFPT2_RESIDENT(4);
  else if (n <= 512) DFPT2_RESIDENT(8);
  else if (n <= 768) DFPT2_RESIDENT(12);
  else if (n <= 1024) DFPT2_RESIDENT(16);
  else if (n <= 1280) DFPT2_RESIDENT(20);
  else if (n <= 1664) DFPT2_RESIDENT(26);
  else DFPT2_RESIDENT(32);
#undef DFPT2_RESIDENT
  if (err != hipSuccess) (void)hipGetLastError();
  return err == hipSuccess;
}

// d[n-2], d[n-1], e[n-2] from the last 2 x 2 block of the reduced matrix, with the update of column
// n - 3 still pending unless p_last (p of that column) is null; one thread
__device__ inline void tridiag_tail(const double* A, int n, const double* Vs, const double* tau, const double* p_last,
                                    double* d, double* e) {
  if (p_last) {  // with the update of column n - 3 pending
    const double* v = Vs + (size_t)(n - 3) * n;  // entries 0, 1 <-> indices n - 2, n - 1
    const double K = 0.5 * tau[n - 3] * (p_last[0] * v[0] + p_last[1] * v[1]);
    const double w0 = p_last[0] - K * v[0], w1 = p_last[1] - K * v[1];
    d[n - 2] = A[(size_t)(n - 2) * n + (n - 2)] - 2.0 * v[0] * w0;
    d[n - 1] = A[(size_t)(n - 1) * n + (n - 1)] - 2.0 * v[1] * w1;
    e[n - 2] = A[(size_t)(n - 1) * n + (n - 2)] - (v[1] * w0 + w1 * v[0]);
  } else if (n >= 2) {
    d[n - 2] = A[(size_t)(n - 2) * n + (n - 2)];
    d[n - 1] = A[(size_t)(n - 1) * n + (n - 1)];
    e[n - 2] = A[(size_t)(n - 1) * n + (n - 2)];
  } else {
    d[0] = A[0];
  }
}

// ---------------------------------------------------------------- splitting
// Zero negligible off-diagonals, record unreduced blocks: blk_start[pos], blk_end[pos]
// = first and one past the last position of the block containing pos.  Also the norm.
// One workgroup; every thread owns a run of positions, the starts are a prefix maximum
// and the ends a suffix minimum over the runs (a single thread took 450 us at n = 1200).
// First the reduction's last 2 x 2 block (p_last: see tridiag_tail).
__global__ __launch_bounds__(1024) void tridiag_split(int n, double* d, double* e, int* blk_start, int* blk_end,
                                                      double* tnorm, const double* A, const double* Vs, const double* tau,
                                                      const double* p_last) {
  __shared__ double shn[1024];
  __shared__ int last[1024], first[1024];
  const int tid = threadIdx.x, per = (n + 1023) / 1024;
  const int i0 = min(n, tid * per), i1 = min(n, i0 + per);
  if (tid == 0) tridiag_tail(A, n, Vs, tau, p_last, d, e);
  __syncthreads();
  double nrm = 0.0;
  for (int i = i0; i < i1; ++i)
    nrm = fmax(nrm, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0));
  shn[tid] = nrm;
  __syncthreads();  // the neighbours have read e before it changes
  auto breaks = [&](int i) {
    if (i == n - 1) return true;
    const double ee = fabs(e[i]);
    return ee <= DBL_EPSILON * sqrt(fabs(d[i])) * sqrt(fabs(d[i + 1])) || ee <= DBL_MIN * 1e6 || ee <= 1e-300;
  };
  int lb = -1, fb = n;  // last and first break of the run
  for (int i = i0; i < i1; ++i)
    if (breaks(i)) {
      if (i + 1 < n) e[i] = 0.0;
      lb = i;
      if (fb == n) fb = i;
    }
  last[tid] = lb;
  first[tid] = fb;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int l = tid >= o ? last[tid - o] : -1, f = tid + o < 1024 ? first[tid + o] : n;
    const double q = tid >= o ? shn[tid - o] : 0.0;
    __syncthreads();
    last[tid] = max(last[tid], l);
    first[tid] = min(first[tid], f);
    shn[tid] = fmax(shn[tid], q);
    __syncthreads();
  }
  if (tid == 1023) *tnorm = shn[1023];
  int st = (tid > 0 ? last[tid - 1] : -1) + 1;
  for (int i = i0; i < i1; ++i) {
    blk_start[i] = st;
    if (i + 1 < n ? e[i] == 0.0 : true) st = i + 1;
  }
  int en = tid + 1 < 1024 ? first[tid + 1] : n;
  for (int i = i1 - 1; i >= i0; --i) {
    if (i + 1 < n ? e[i] == 0.0 : true) en = i;
    blk_end[i] = en + 1;
  }
}

// Sturm counts (eigenvalues of the block smaller than x) at a point.  In the scaled form below (kProduct) T is scaled by a
// power of two to ||T|| <= 1 and the count is the number of sign changes of
//     p_{i+1} = (d_i - x) p_i - e_{i-1}^2 p_{i-1},
// rescaled by a power of two every 8 steps: three FP64 operations a step instead of the
// dozen of q_{i+1} = d_i - x - e_{i-1}^2 / q_i, and the same backward error (p_{i+1} / p_i
// is q_i with d - x and e off by a few relative roundings).  A zero p_i takes either sign
// for exactly one change between its neighbours, as it should.  It needs e^2 >= 1e-60 in
// the scaled block, so that 8 steps cannot underflow; otherwise the q form runs.
template <bool kProduct>
__device__ inline int sturm(const double* d, const double* e, int s, int t, double x, double pivmin) {
  double q = d[s] - x, q0 = 1.0;
  if (!kProduct && fabs(q) < pivmin) q = -pivmin;
  int c = q < 0.0;
  if (kProduct) {
    auto hi = [](double v) { return (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32); };
    for (int i0 = s + 1; i0 < t; i0 += 8) {
      const int m = min(8, t - i0);
      auto step = [&](int i) {  // LDS holds e^2
        const double q2 = fma(d[i] - x, q, -e[i - 1] * q0);
        c += (hi(q2) ^ hi(q)) >> 31;
        q0 = q;
        q = q2;
      };
      if (m == 8) {
#pragma unroll
        for (int r = 0; r < 8; ++r) step(i0 + r);
      } else {
        for (int r = 0; r < m; ++r) step(i0 + r);
      }
      const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(q0), fabs(q)));
      q0 = __builtin_amdgcn_ldexp(q0, -ex);
      q = __builtin_amdgcn_ldexp(q, -ex);
    }
  } else {
    for (int i = s + 1; i < t; ++i) {
      q = fma(-e[i - 1] * e[i - 1], fast_rcp(q), d[i] - x);
      if (fabs(q) < pivmin) q = -pivmin;
      c += q < 0.0;
    }
  }
  return c;
}

// Bracket [lo, hi] of the j-th eigenvalue of the block [s, t) shrunk by W waves of a point per
// lane: the bracket becomes the interval between the highest point whose count is <= j and
// the next one (64 W + 1 times smaller per round, 7 to 9 rounds).  The invariant count(lo) <=
// j < count(hi) holds whatever the rounding.
template <bool kProduct, int W>
__device__ double multisect(const double* d, const double* e, int s, int t, int j, double lo, double hi,
                            double pivmin, int wv, int lane, unsigned long long (*masks)[W]) {
  constexpr int N = 64 * W;
  for (int it = 0; it < 64; ++it) {
    if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi)) + pivmin) break;
    const double h = (hi - lo) / (N + 1.0);
    auto point = [&](int k) { return fmin(fmax(fma((double)(k + 1), h, lo), lo), hi); };
    const double x = point(wv * 64 + lane);
    const int c = sturm<kProduct>(d, e, s, t, x, pivmin);
    unsigned long long m = __ballot((x <= lo) ? true : (x >= hi) ? false : c <= j);
    int klo = -1;
    if (W == 1) {
      if (m) klo = 63 - __clzll((long long)m);
    } else {  // the same rounds in every wave: one barrier each, masks of two rounds
      if (lane == 0) masks[it & 1][wv] = m;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < W; ++w) {
        m = masks[it & 1][w];
        if (m) klo = 64 * w + 63 - __clzll((long long)m);
      }
    }
    const double nlo = klo >= 0 ? point(klo) : lo, nhi = klo + 1 < N ? point(klo + 1) : hi;
    if (!(nlo > lo || nhi < hi)) break;  // the points no longer split the bracket
    lo = nlo;
    hi = nhi;
  }
  return 0.5 * (lo + hi);
}

// The (g - start)-th eigenvalue of the block containing position g: one wave, four of them a
// workgroup (W = 1), or a workgroup of W waves.  What
// bounds it is the issue of the counts' FP64 operations, and up to 512 positions, which leave
// SIMDs idle, the chain of one count.  d and e^2 (or e) come from LDS up to n = kSturmLds.
// n = 1200: 1.8 ms with full divisions and global reads, 1.3 ms with fast reciprocals (and two
// points per lane, to fill their latency); in the product form 0.66 ms with two points and
// 0.46 with one.  n = 60: 33 us with W = 1, 21 us
// with W = 4.  The last blocks form the factors of the back-transformation (wy16_t), which
// takes no time of its own here.
constexpr int kSturmLds = 4096;

__device__ void wy16_t(int blk, int n, const double* Vs, const double* tau, double* Tout, double* sh);
constexpr int kWySh = 4 * 256 + 16 * 17;  // doubles of LDS

template <bool kLds, int W>
__global__ __launch_bounds__(256) void tridiag_multisect(int n, const double* dg, const double* eg,
                                                         const int* blk_start, const int* blk_end,
                                                         const double* tnorm, double* lam, int nblk,
                                                         const double* Vs, const double* tau, double* Tout) {
  constexpr int G = W == 1 ? 4 : 1;  // eigenvalues per workgroup
  extern __shared__ double msh[];
  __shared__ int small;
  __shared__ unsigned long long masks[2][W];
  const int first = (n + G - 1) / G;
  if ((int)blockIdx.x >= first) {
    if ((int)blockIdx.x - first < nblk) wy16_t(blockIdx.x - first, n, Vs, tau, Tout, msh);
    return;
  }
  const int wv = W == 1 ? 0 : threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = W == 1 ? blockIdx.x * 4 + (threadIdx.x >> 6) : blockIdx.x;
  const double nrm = fmax(*tnorm, DBL_MIN);
  int ex = 0;
  bool product = false;
  if (kLds) {
    ex = nrm < 1e300 ? __builtin_amdgcn_frexp_exp(nrm) : 0;
    if (threadIdx.x == 0) small = nrm < 1e300 ? 0 : 1;
    __syncthreads();
    int sm = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const double ei = i + 1 < n ? ldexp(eg[i], -ex) : 0.0;
      msh[i] = ldexp(dg[i], -ex);
      msh[n + i] = ei;
      sm |= ei != 0.0 && !(ei * ei >= 1e-60);
    }
    if (sm) small = 1;
    __syncthreads();
    product = !small;
    if (product)
      for (int i = threadIdx.x; i < n; i += blockDim.x) msh[n + i] *= msh[n + i];  // e^2
    __syncthreads();
  }
  if (g >= n) return;  // wave-uniform; only where W == 1
  const int s = blk_start[g], t = blk_end[g], j = g - s;
  double lo = DBL_MAX, hi = -DBL_MAX;
  for (int i = s + lane; i < t; i += 64) {
    const double r = (i > s ? fabs(eg[i - 1]) : 0.0) + (i + 1 < t ? fabs(eg[i]) : 0.0);
    lo = fmin(lo, dg[i] - r);
    hi = fmax(hi, dg[i] + r);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, 64));
    hi = fmax(hi, __shfl_xor(hi, o, 64));
  }
  const double pivmin = DBL_MIN * fmax(1.0, nrm * nrm) * 4.0;
  const double pad = 2.0 * DBL_EPSILON * nrm * (t - s) + 2.0 * pivmin;
  lo -= pad;
  hi += pad;
  double x;
  if (product)  // in units of 2^ex (exact)
    x = ldexp(multisect<true, W>(msh, msh + n, s, t, j, ldexp(lo, -ex), ldexp(hi, -ex), 8.0 * DBL_MIN, wv, lane, masks), ex);
  else
    x = multisect<false, W>(dg, eg, s, t, j, lo, hi, pivmin, wv, lane, masks);
  if (lane == 0 && wv == 0) lam[g] = x;
}

// ------------------------------------------------------------ twisted factorization
// Eigenvector of an eigenvalue that is isolated in its block (both gaps above
// kIsolated ||T||): T - lam = L D L^T from the top and U D U^T from the
// bottom, z = 1 at the row r where they leave the smallest pivot, and z_i = -l_i z_{i+1}
// above, z_{i+1} = -u_i z_i below.  Either factorization is exact for off-diagonals off
// by a few ulps (as in the Sturm counts), so the residual is the twist pivot over ||z||
// plus a few ulps of ||T||.  That is a single solve, of the start vector e_r, and leaves
// (lam's error) / gap of its neighbours in z; a second one with the same factors squares it
// away, as inverse iteration's do.  Relative error of the vectors of random symmetric matrices of
// 600 and 1200 rows, in units of inverse iteration's: 0.95 and 1.02, with one solve 1.55 and 2.31.
// A residual of z above 50 eps ||T|| or a value that is not finite leaves done[g] = 0, and the
// vector to inverse iteration.  What bounds it is the chain of a factorization (one reciprocal and
// three operations a position).  A wave takes VW vectors, 64 / VW lanes each: lane 0 of a
// group runs down the block and lane 1 up, each writing its multipliers to LDS, all lanes
// search for the twist, lanes 0 and 1 run the recurrences of the two solves, and all lanes
// scale and store.  n = 1200: 5.9 ms for inverse iteration (its LU
// arrays stream through memory nine times), 1.4 ms with one thread per vector and l, u in
// memory, 0.44 ms so (0.28 with one solve).
constexpr double kIsolated = 1e-8;
// LDS of a wave of VW vectors: d, e and the multipliers l, u
constexpr size_t twisted_bytes(int n, int vw) { return (size_t)n * 8 * (2 + 2 * vw); }
constexpr size_t kTwistedLds = 160 * 1024 - 256;

// x <- b_k - c_k x (kAdd; else -c_k x) for k < n, each x stored over b_k; eight reads in flight
template <bool kAdd>
__device__ inline double recur(const double* c, double* b, int stride, int n, double x) {
  for (; n >= 8; n -= 8, c += 8 * stride, b += 8 * stride) {
    double cv[8], bv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      cv[k] = c[k * stride];
      bv[k] = kAdd ? b[k * stride] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) b[k * stride] = x = kAdd ? fma(-cv[k], x, bv[k]) : -cv[k] * x;
  }
  for (; n > 0; --n, c += stride, b += stride) *b = x = kAdd ? fma(-*c, x, *b) : -*c * x;
  return x;
}

template <int VW>
__global__ __launch_bounds__(64) void tridiag_twisted(int n, const double* dg, const double* eg, const int* blk_start,
                                                      const int* blk_end, const double* tnorm, const double* lam,
                                                      double* __restrict__ X, int* done, const double* vec_floor) {
  extern __shared__ double msh[];
  constexpr int G = 64 / VW;
  double *d = msh, *e = msh + n, *Lm = msh + 2 * n, *Um = Lm + (size_t)VW * n;
  const int lane = threadIdx.x, v = lane / G, q = lane - v * G, g = blockIdx.x * VW + v;
  for (int i = lane; i < n; i += 64) {
    d[i] = dg[i];
    e[i] = i + 1 < n ? eg[i] : 0.0;
  }
  __syncthreads();
  const double nrm = fmax(*tnorm, DBL_MIN), pivmin = DBL_MIN * fmax(1.0, nrm * nrm) * 4.0;
  int s = 0, t = 0;
  double x = 0.0;
  bool go = g < n;
  if (go) {
    s = blk_start[g];
    t = blk_end[g];
    x = lam[g];
    go = t - s > 1 && !(vec_floor && !(x > *vec_floor)) && !(g > s && !(fabs(x - lam[g - 1]) > kIsolated * nrm)) &&
         !(g + 1 < t && !(fabs(lam[g + 1] - x) > kIsolated * nrm));
    if (!go && q == 0) done[g] = 0;
  }
  if (!go) s = t = 0;  // the group's lanes stay for the barriers
  // factorizations: lane 0 downwards (l at v + VW i), lane 1 upwards (u)
  if (q < 2 && t > s) {
    const int st = q == 0 ? 1 : -1;
    int i = q == 0 ? s : t - 1, o = q == 0 ? s : t - 2;  // position, off-diagonal towards the next one
    double* M = (q == 0 ? Lm : Um) + v;
    double piv = d[i] - x;
#pragma unroll 4
    for (int k = t - 1 - s; k > 0; --k, i += st, o += st) {
      if (fabs(piv) < pivmin) piv = -pivmin;
      const double eo = e[o], m = eo * fast_rcp(piv);
      M[(size_t)o * VW] = m;
      piv = fma(-eo, m, d[i + st] - x);
    }
  }
  __syncthreads();
  // twist where the pivot, with its rounding, is smallest
  int r = 0x7fffffff;
  double best = DBL_MAX, gam = 0.0;
  for (int i = s + q; i < t; i += G) {
    const double el = i > s ? e[i - 1] * Lm[(size_t)(i - 1) * VW + v] : 0.0;
    const double eu = i + 1 < t ? e[i] * Um[(size_t)i * VW + v] : 0.0;
    const double dx = d[i] - x, ga = (dx - el) - eu;
    const double c = fabs(ga) + DBL_EPSILON * (fabs(dx) + fabs(el) + fabs(eu));
    if (c < best) {
      best = c;
      r = i;
      gam = ga;
    }
  }
#pragma unroll
  for (int o = G / 2; o >= 1; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64), og = __shfl_xor(gam, o, 64);
    const int orr = __shfl_xor(r, o, 64);
    if (ob < best || (ob == best && orr < r)) {
      best = ob;
      gam = og;
      r = orr;
    }
  }
  if (r < s || r >= t) r = s;  // no finite pivot (the residual test below fails)
  __syncthreads();
  // From here on l_i counts for i < r only and u_i for i >= r; the vectors lie in the other
  // halves: entry i < r over u_i, entry i + 1 > r over l_i.
  const int cnt = q > 1 || t <= s ? 0 : q == 0 ? r - s : t - 1 - r, dir = q == 0 ? VW : -VW;
  double* C = (q == 0 ? Lm : Um) + v;  // multipliers and vector of the lane's half
  double* B = (q == 0 ? Um : Lm) + v;
  // z_i (lane 0), z_{i+1} (lane 1), away from the twist
  const int near = (q == 0 ? r - 1 : r) * VW, far = (q == 0 ? s : t - 2) * VW;
  if (cnt > 0) recur<false>(C + near, B + near, -dir, cnt, 1.0);
  __syncthreads();
  auto entry = [&](int i) {
    return i < r ? Um[(size_t)i * VW + v] : i > r ? Lm[(size_t)(i - 1) * VW + v] : 1.0;
  };
  auto norm = [&] {
    double nz = 0.0;
    for (int i = s + q; i < t; i += G) {
      const double z = entry(i);
      nz = fma(z, z, nz);
    }
#pragma unroll
    for (int o = G / 2; o >= 1; o >>= 1) nz += __shfl_xor(nz, o, 64);
    return sqrt(nz);
  };
  double nn = norm();
  if (go && (!(nn < 1e150) || !(best < DBL_MAX) || !(fabs(gam) <= 50.0 * DBL_EPSILON * nrm * nn))) {
    if (q == 0) done[g] = 0;
    go = false;
    s = t = 0;
  }
  __syncthreads();
  // The second solve, (T - lam I) y = z, in place.  N D N^T with N's columns l, u: first N w = z,
  // w_{i+1} = z_{i+1} - l_i w_i above the twist (lane 0), w_i = z_i - u_i w_{i+1} below (lane 1)
  double a = 0.0;
  if (cnt > 0 && t > s) a = C[near] * recur<true>(C + far, B + far + dir, dir, cnt - 1, B[far]);
  a += __shfl_xor(a, 1, 64);
  const double sc = gam / (1.0 - __shfl(a, lane - q, 64));  // scales y to y_r = 1
  __syncthreads();
  // w_i / D_i, with 1 / D_i = l_i / e_i above the twist and u_{i-1} / e_{i-1} below
  for (int i = s + q; i < t; i += G) {
    if (i < r) Um[(size_t)i * VW + v] = sc * Um[(size_t)i * VW + v] * Lm[(size_t)i * VW + v] / e[i];
    if (i > r) Lm[(size_t)(i - 1) * VW + v] = sc * Lm[(size_t)(i - 1) * VW + v] * Um[(size_t)(i - 1) * VW + v] / e[i - 1];
  }
  __syncthreads();
  // N^T y: y_i = w_i / D_i - l_i y_{i+1}, y_{i+1} = w_{i+1} / D_{i+1} - u_i y_i
  if (cnt > 0 && t > s) recur<true>(C + near, B + near, -dir, cnt, 1.0);
  __syncthreads();
  nn = norm();
  if (!go) return;
  if (!(nn < 1e150)) {
    if (q == 0) done[g] = 0;
    return;
  }
  const double inv = 1.0 / nn;
  for (int i = q; i < n; i += G) X[(size_t)i * n + g] = (i >= s && i < t) ? entry(i) * inv : 0.0;
  if (q == 0) done[g] = 1;
}

// no vector is formed by a twisted factorization (n beyond its LDS)
__global__ void zero_done(int n, int* done) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) done[g] = 0;
}

// ------------------------------------------------------------ inverse iteration
struct LuCols {
  double *u1, *u2, *u3, *l, *piv;  // [pos][n] layout, column g owned by thread g
};

__device__ inline double hash_unit(unsigned a, unsigned b) {
  unsigned h = a * 2654435761u ^ (b + 0x9e3779b9u + (a << 6) + (a >> 2));
  h ^= h >> 16;
  h *= 0x7feb352du;
  h ^= h >> 15;
  h *= 0x846ca68bu;
  h ^= h >> 16;
  return ((double)(h & 0xffffff) / 16777216.0) - 0.5;
}

// Factor T_b - lam I (block [s, t)) into column g of the LU arrays.
__device__ void lu_factor(const double* d, const double* e, int s, int t, double lam, double tiny,
                          const LuCols& L, int n, int g) {
  double alpha = d[s] - lam;
  double beta = (s + 1 < t) ? e[s] : 0.0;
  for (int i = s; i < t - 1; ++i) {
    const double c = e[i];
    const double an = d[i + 1] - lam;
    const double bn = (i + 2 < t) ? e[i + 1] : 0.0;
    const size_t o = (size_t)i * n + g;
    if (fabs(alpha) >= fabs(c)) {
      double a_ = alpha;
      if (a_ == 0.0) a_ = tiny;
      const double mlt = c / a_;
      L.u1[o] = a_;
      L.u2[o] = beta;
      L.u3[o] = 0.0;
      L.l[o] = mlt;
      L.piv[o] = 0.0;
      alpha = an - mlt * beta;
      beta = bn;
    } else {
      const double mlt = alpha / c;
      L.u1[o] = c;
      L.u2[o] = an;
      L.u3[o] = bn;
      L.l[o] = mlt;
      L.piv[o] = 1.0;
      alpha = beta - mlt * an;
      beta = -mlt * bn;
    }
  }
  const size_t o = (size_t)(t - 1) * n + g;
  L.u1[o] = (alpha == 0.0) ? tiny : alpha;
  L.u2[o] = 0.0;
  L.u3[o] = 0.0;
}

// Solve in place: x (column g of X over positions [s, t)) <- (T - lam I)^{-1} (scl x);
// returns max |x| of the result.  The values each step produces for the next are
// carried in registers, so the loads of a step depend on nothing written by the
// one before.
__device__ double lu_solve(int s, int t, const LuCols& L, int n, int g, double* __restrict__ X, int xcol,
                           double scl) {
  const double* __restrict__ u1 = L.u1;
  const double* __restrict__ u2 = L.u2;
  const double* __restrict__ u3 = L.u3;
  const double* __restrict__ lm = L.l;
  const double* __restrict__ pv = L.piv;
  double yi = X[(size_t)s * n + xcol] * scl;
#pragma unroll 4
  for (int i = s; i < t - 1; ++i) {
    const size_t o = (size_t)i * n + g;
    double yn = X[(size_t)(i + 1) * n + xcol] * scl;
    if (pv[o] != 0.0) {
      const double tmp = yi;
      yi = yn;
      yn = tmp;
    }
    yn -= lm[o] * yi;
    X[(size_t)i * n + xcol] = yi;
    yi = yn;
  }
  X[(size_t)(t - 1) * n + xcol] = yi;
  double x1 = 0.0, x2 = 0.0;  // the solved X[i + 1], X[i + 2]
  double mx = 0.0;
#pragma unroll 4
  for (int i = t - 1; i >= s; --i) {
    const size_t o = (size_t)i * n + g;
    double v = X[(size_t)i * n + xcol];
    if (i + 1 < t) v -= u2[o] * x1;
    if (i + 2 < t) v -= u3[o] * x2;
    v = v / u1[o];
    X[(size_t)i * n + xcol] = v;
    mx = fmax(mx, fabs(v));
    x2 = x1;
    x1 = v;
  }
  return mx;
}

// Group leaders (first eigenvalue of a near-degenerate run inside a block) compute
// the vectors of their whole group; X is row-major n x n, column g = vector g.
// vec_floor: if non-null, eigenvectors are formed only for eigenvalues above
// *vec_floor; the other columns of X are zero (callers that drop those
// eigenpairs, such as the NAF compression, skip the cost of large clusters).
__global__ void tridiag_inverse_iteration(int n, const double* d, const double* e, const int* blk_start,
                                          const int* blk_end, const double* tnorm, const double* lam,
                                          LuCols L, double* X, int* status, const double* vec_floor,
                                          const int* done) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  // done: the twisted factorization formed this vector; 2: there is no tridiagonal matrix
  if (g >= n || done[g] || *status == 2) return;
  const int s = blk_start[g], t = blk_end[g];
  if (vec_floor && !(lam[g] > *vec_floor)) {
    for (int i = 0; i < n; ++i) X[(size_t)i * n + g] = 0.0;
    return;
  }
  const double nrm = (*tnorm > 0.0) ? *tnorm : 1.0;
  const double grp_tol = 1e-10 * nrm;
  if (t - s == 1) {  // a 1 x 1 block: the unit vector
    for (int i = 0; i < n; ++i) X[(size_t)i * n + g] = (i == s) ? 1.0 : 0.0;
    return;
  }
  // a leader above the floor starts its group; earlier members below the floor were zeroed
  if (vec_floor && g > s && fabs(lam[g] - lam[g - 1]) <= grp_tol && !(lam[g - 1] > *vec_floor)) {
    // lam[g - 1] was skipped: g leads what remains of the group
  } else if (g > s && fabs(lam[g] - lam[g - 1]) <= grp_tol) {
    return;
  }
  int g1 = g + 1;
  while (g1 < t && fabs(lam[g1] - lam[g1 - 1]) <= grp_tol) ++g1;
  const double tiny = DBL_EPSILON * nrm;
  double lq = 0.0;
  for (int q = g; q < g1; ++q) {
    // zero the column outside the block, random start inside
    for (int i = 0; i < n; ++i) X[(size_t)i * n + q] = (i >= s && i < t) ? hash_unit(q, i) : 0.0;
    // shifts of a group are kept a few ulps apart so that the factors differ; no further,
    // so that a shift stays with its own eigenvalue wherever the gaps are wider
    lq = q == g ? lam[q] : fmax(lam[q], lq + 4.0 * DBL_EPSILON * nrm);
    lu_factor(d, e, s, t, lq, tiny, L, n, g);
    // the solves and the orthogonalization are linear, so between iterations the
    // vector is only rescaled against overflow (by 1 / max |x|, applied as the
    // next solve loads it); it is normalized once at the end
    double scl = 1.0;
    for (int it = 0; it < 4; ++it) {
      double mx = lu_solve(s, t, L, n, g, X, q, scl);
      if (q > g) {
        // orthogonalize against earlier (unit) vectors of the group, twice for stability
        mx = 0.0;
        for (int pass = 0; pass < 2; ++pass) {
          for (int r = g; r < q; ++r) {
            double dp = 0.0;
            for (int i = s; i < t; ++i) dp += X[(size_t)i * n + r] * X[(size_t)i * n + q];
            for (int i = s; i < t; ++i) {
              const double y = X[(size_t)i * n + q] - dp * X[(size_t)i * n + r];
              X[(size_t)i * n + q] = y;
              if (pass == 1 && r == q - 1) mx = fmax(mx, fabs(y));
            }
          }
        }
      }
      if (!(mx > 0.0) || !isfinite(mx)) {
        atomicMax(status, 1);
        return;
      }
      scl = 1.0 / mx;
    }
    double nx = 0.0;
    for (int i = s; i < t; ++i) {
      const double y = X[(size_t)i * n + q] * scl;
      nx += y * y;
    }
    const double inv = scl / sqrt(nx);
    for (int i = s; i < t; ++i) X[(size_t)i * n + q] *= inv;
  }
}

// ------------------------------------------------------------ back-transform
// Z <- H_0 H_1 ... H_{n-3} Z with H_k = I - tau_k v_k v_k^T (v_k: 1 at row k + 1,
// Vs[k][.] below it), applied in compact-WY blocks of WY_NB reflectors: for the
// block k0 .. k0 + WY_NB - 1, H_k0 ... H_{k0+WY_NB-1} = I - V T V^T with T upper
// triangular (T_cc = tau_c, T[0:c, c] = -tau_c T[0:c, 0:c] V[:, 0:c]^T v_c), and the
// blocks go from the last to the first: Z <- Z - V (T (V^T Z)).
constexpr int WY_NB = 8;

// V[i][j] of block k0 (row i of the full vector of reflector k0 + j), 0 outside
__device__ inline double wy_v(const double* Vs, int n, int k0, int nr, int i, int j) {
  const int k = k0 + j;
  return (j < nr && i > k) ? Vs[(size_t)k * n + (i - k - 1)] : 0.0;
}

// One workgroup per block: S = V^T V (upper triangle) by a pass over the rows,
// then T by the forward recurrence (one thread).  T: [nblk][WY_NB][WY_NB].
__global__ __launch_bounds__(256) void wy_build_t(int n, const double* Vs, const double* tau, double* Tout) {
  constexpr int NS = WY_NB * (WY_NB + 1) / 2;
  __shared__ double part[4][NS];
  __shared__ double S[WY_NB][WY_NB];
  const int b = blockIdx.x, k0 = b * WY_NB;
  const int nr = min(WY_NB, n - 2 - k0);  // reflectors 0 .. n - 3
  double acc[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) acc[q] = 0.0;
  for (int i = k0 + 1 + threadIdx.x; i < n; i += blockDim.x) {
    double v[WY_NB];
#pragma unroll
    for (int j = 0; j < WY_NB; ++j) v[j] = wy_v(Vs, n, k0, nr, i, j);
    int q = 0;
#pragma unroll
    for (int l = 0; l < WY_NB; ++l)
#pragma unroll
      for (int c = l; c < WY_NB; ++c) acc[q++] += v[l] * v[c];
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    const double t = wave_sum(acc[q]);
    if (lane == 0) part[w][q] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int q = 0;
    for (int l = 0; l < WY_NB; ++l)
      for (int c = l; c < WY_NB; ++c, ++q) S[l][c] = (part[0][q] + part[1][q]) + (part[2][q] + part[3][q]);
    double T[WY_NB][WY_NB];
    for (int c = 0; c < WY_NB; ++c) {
      const double tc = c < nr ? tau[k0 + c] : 0.0;
      for (int i = 0; i < WY_NB; ++i) T[i][c] = 0.0;
      T[c][c] = tc;
      for (int i = 0; i < c; ++i) {
        double sum = 0.0;
        for (int l = i; l < c; ++l) sum += T[i][l] * S[l][c];
        T[i][c] = -tc * sum;
      }
    }
    double* To = Tout + (size_t)b * WY_NB * WY_NB;
    for (int i = 0; i < WY_NB; ++i)
      for (int c = 0; c < WY_NB; ++c) To[i * WY_NB + c] = T[i][c];
  }
}

// One workgroup per WY_CW columns of Z, held in LDS; the blocks of reflectors in
// reverse order, two barriers per block.
template <int WY_CW>
__global__ __launch_bounds__(256) void tridiag_backtransform(int n, const double* Vs, const double* Tall,
                                                             double* Z) {
  extern __shared__ double zs[];  // [n][WY_CW]
  __shared__ double part[4][WY_NB * WY_CW];
  __shared__ double Wsh[WY_NB][WY_CW];
  const int c0 = blockIdx.x * WY_CW;
  const int ncol = min(WY_CW, n - c0);
  for (int idx = threadIdx.x; idx < n * WY_CW; idx += blockDim.x) {
    const int r = idx / WY_CW, c = idx % WY_CW;
    zs[idx] = (c < ncol) ? Z[(size_t)r * n + c0 + c] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int nblk = (n - 2 + WY_NB - 1) / WY_NB;
  for (int b = nblk - 1; b >= 0; --b) {
    const int k0 = b * WY_NB, nr = min(WY_NB, n - 2 - k0);
    // P = V^T Z over the rows below k0
    double acc[WY_NB][WY_CW];
#pragma unroll
    for (int j = 0; j < WY_NB; ++j)
#pragma unroll
      for (int c = 0; c < WY_CW; ++c) acc[j][c] = 0.0;
    for (int i = k0 + 1 + threadIdx.x; i < n; i += blockDim.x) {
      const double* zr = zs + (size_t)i * WY_CW;
#pragma unroll
      for (int j = 0; j < WY_NB; ++j) {
        const double v = wy_v(Vs, n, k0, nr, i, j);
#pragma unroll
        for (int c = 0; c < WY_CW; ++c) acc[j][c] += v * zr[c];
      }
    }
#pragma unroll
    for (int j = 0; j < WY_NB; ++j)
#pragma unroll
      for (int c = 0; c < WY_CW; ++c) {
        const double t = wave_sum(acc[j][c]);
        if (lane == 0) part[w][j * WY_CW + c] = t;
      }
    __syncthreads();
    // W = T P (T upper triangular)
    if (threadIdx.x < WY_NB * WY_CW) {
      const int j = threadIdx.x / WY_CW, c = threadIdx.x % WY_CW;
      const double* T = Tall + (size_t)b * WY_NB * WY_NB;
      double sum = 0.0;
      for (int l = j; l < WY_NB; ++l) {
        const int q = l * WY_CW + c;
        sum += T[j * WY_NB + l] * ((part[0][q] + part[1][q]) + (part[2][q] + part[3][q]));
      }
      Wsh[j][c] = sum;
    }
    __syncthreads();
    // Z -= V W
    for (int i = k0 + 1 + threadIdx.x; i < n; i += blockDim.x) {
      double* zr = zs + (size_t)i * WY_CW;
      double u[WY_CW];
#pragma unroll
      for (int c = 0; c < WY_CW; ++c) u[c] = 0.0;
#pragma unroll
      for (int j = 0; j < WY_NB; ++j) {
        const double v = wy_v(Vs, n, k0, nr, i, j);
#pragma unroll
        for (int c = 0; c < WY_CW; ++c) u[c] += v * Wsh[j][c];
      }
#pragma unroll
      for (int c = 0; c < WY_CW; ++c) zr[c] -= u[c];
    }
    __syncthreads();
  }
  for (int idx = threadIdx.x; idx < n * WY_CW; idx += blockDim.x) {
    const int r = idx / WY_CW, c = idx % WY_CW;
    if (c < ncol) Z[(size_t)r * n + c0 + c] = zs[idx];
  }
}

// The same back-transformation on the FP64 matrix pipe, in blocks of 16 reflectors, for
// 8 <= n <= 2048.  A workgroup keeps 16 columns of Z in registers: the register r of a 16 x 16
// block in the products' output layout (row 4 r + lane / 16) is the second operand of the
// contraction step r, so Z is the operand of P = V^T Z, takes V (T P) and never moves.  Row
// blocks are dealt round-robin to the 8 waves (the
// reflectors act below k0 only); the waves' partial P meet in LDS, one barrier per block.
// Every sum is formed in pairs from products of four terms, and V (T P) apart from Z: with a
// sum of hundreds of terms on one accumulator, and Z as the accumulator of its update, the
// largest residual of 600 and 1200 random rows was 2.0 and 2.5 times that of sums over a
// workgroup's threads, 1.0 so.
// What bounds it: two passes over V per block from L2 and the chain P -> T P -> Z.
// n = 1200: 2.0 ms with blocks of 8 on vector instructions, Z in LDS and three barriers;
// 0.48 ms so (0.44 with one accumulator per sum).
constexpr int WY16 = 16;

// V[i][j] of block k0, 0 outside
__device__ inline double wy16_v(const double* Vs, int n, int k0, int nr, int i, int j) {
  const int k = k0 + j;
  return (j < nr && i > k && i < n) ? Vs[(size_t)k * n + (i - k - 1)] : 0.0;
}

// T of block blk ([16][16], upper triangular): S = V^T V, then each row by itself; 256 threads
__device__ void wy16_t(int blk, int n, const double* Vs, const double* tau, double* Tout, double* sh) {
  double(*part)[256] = reinterpret_cast<double(*)[256]>(sh);
  double(*S)[17] = reinterpret_cast<double(*)[17]>(sh + 4 * 256);
  const int k0 = blk * WY16, nr = min(WY16, n - 2 - k0);  // reflectors 0 .. n - 3
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  d4 acc = (d4){0.0, 0.0, 0.0, 0.0};
  for (int rb = k0 / 16 * 16 + 16 * w; rb < n; rb += 16 * (blockDim.x >> 6)) {
    d4 m[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double v = wy16_v(Vs, n, k0, nr, rb + 4 * r + kq, r16);
      m[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, (d4){0.0, 0.0, 0.0, 0.0}, 0, 0, 0);
    }
    acc += (m[0] + m[1]) + (m[2] + m[3]);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) part[w][(kq + 4 * r) * 16 + r16] = acc[r];
  __syncthreads();
  for (int k = tid; k < 256; k += blockDim.x) {
    double v = part[0][k];
    for (int q = 1; q < (int)(blockDim.x >> 6); ++q) v += part[q][k];
    S[k >> 4][k & 15] = v;
  }
  __syncthreads();
  if (tid < 16) {  // T_cc = tau_c, T[i][c] = -tau_c sum_l T[i][l] S[l][c]
    double T[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const double tc = c < nr ? tau[k0 + c] : 0.0;
      double sum = 0.0;
#pragma unroll
      for (int l = 0; l < c; ++l) sum += (l >= tid ? T[l] : 0.0) * S[l][c];
      T[c] = c < tid ? 0.0 : c == tid ? tc : -tc * sum;
      Tout[(size_t)blk * 256 + tid * 16 + c] = T[c];
    }
  }
}

__global__ __launch_bounds__(256) void wy16_build_t(int n, const double* Vs, const double* tau, double* Tout) {
  __shared__ double sh[kWySh];
  wy16_t(blockIdx.x, n, Vs, tau, Tout, sh);
}

template <int NB>
__global__ __launch_bounds__(512) void backtransform16(int n, const double* Vs, const double* Tall, double* Z) {
  __shared__ double part[2][8][256];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r16 = lane & 15, kq = lane >> 4;
  const int c = blockIdx.x * 16 + r16;
  const d4 zero = (d4){0.0, 0.0, 0.0, 0.0};
  d4 z[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * (w + 8 * b) + 4 * r + kq;
      z[b][r] = (i < n && c < n) ? Z[(size_t)i * n + c] : 0.0;
    }
  const int nblk = (n - 2 + WY16 - 1) / WY16;
  for (int blk = nblk - 1; blk >= 0; --blk) {
    const int k0 = blk * WY16, nr = min(WY16, n - 2 - k0), buf = blk & 1;
    // V[i][j] = Vs[(k0 + j) n + i - (k0 + j) - 1] for j < nr and k0 + j < i < n: a buffer
    // load from row k0, at an offset out of range (which reads zero) elsewhere: no branch
    auto desc = __builtin_amdgcn_make_buffer_rsrc((void*)(Vs + (size_t)k0 * n), 0, 0x7fffffff, 0x00020000);
    auto vload = [&](int i, int j) {
      const int o = (j * (n - 1) + i - k0 - 1) * 8;
      const bool in = j < nr && i > k0 + j && i < n;
      typedef uint32_t u2 __attribute__((ext_vector_type(2)));
      return __builtin_bit_cast(double, (u2)__builtin_amdgcn_raw_buffer_load_b64(desc, in ? o : (int)0x80000000, 0, 0));
    };
    d4 ps[2] = {zero, zero};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int rb = 16 * (w + 8 * b);
      if (rb + 15 > k0 && rb < n) {  // wave-uniform
        double v[4];
        d4 m[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = vload(rb + 4 * r + kq, r16);
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r], z[b][r], zero, 0, 0, 0);
        ps[b & 1] += (m[0] + m[1]) + (m[2] + m[3]);
      }
    }
    const d4 p = ps[0] + ps[1];
    double t[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) t[r] = Tall[(size_t)blk * 256 + r16 * 16 + 4 * r + kq];
#pragma unroll
    for (int r = 0; r < 4; ++r) part[buf][w][r * 64 + lane] = p[r];
    __syncthreads();
    d4 wm[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double q[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) q[k] = part[buf][k][r * 64 + lane];
      const double sum = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
      wm[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[r], -sum, zero, 0, 0, 0);
    }
    const d4 wv = (wm[0] + wm[1]) + (wm[2] + wm[3]);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int rb = 16 * (w + 8 * b);
      if (rb + 15 > k0 && rb < n) {
        double v[4];
        d4 u = zero;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = vload(rb + r16, 4 * r + kq);
#pragma unroll
        for (int r = 0; r < 4; ++r) u = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r], wv[r], u, 0, 0, 0);
        z[b] += u;
      }
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * (w + 8 * b) + 4 * r + kq;
      if (i < n && c < n) Z[(size_t)i * n + c] = z[b][r];
    }
}

// ------------------------------------------------------------ sort + orient
// M = I - U with U = strictly upper part of E + diag(E) / 2, where E = Z^T Z - I
// arrives as G = Z^T Z in M (in place)
__global__ void orth_correction(int n, double* M) {
  const size_t nn = (size_t)n * n;
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < nn; k += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(k / n), j = (int)(k - (size_t)i * n);
    const double g = M[k];
    M[k] = i < j ? -g : i == j ? 1.0 - 0.5 * (g - 1.0) : 0.0;
  }
}

// Out column dst(g) = sign-oriented column g; descending: dst = n - 1 - rank.  One workgroup per
// 16 columns (whole 128-byte lines), 64 rows at a time; wave w finds the rank of column w among
// all eigenvalues (ascending, ties by index).
// Nothing is written after a reduction that was given up: the next attempt reads the matrix
// again, and a caller may have named one buffer for the matrix and the vectors.
__global__ __launch_bounds__(1024) void eig_permute(int n, const double* lam, const double* Zin, double* w_out,
                                                    double* Z_out, int descending, const int* status) {
  if (*status == 2) return;
  __shared__ int rank[16];
  {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = min((int)blockIdx.x * 16 + w, n - 1);
    const double x = lam[g];
    int r = 0;
    for (int q = lane; q < n; q += 64) {
      const double y = lam[q];
      r += (y < x || (y == x && q < g)) ? 1 : 0;
    }
    for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
    if (lane == 0) rank[w] = r;
  }
  __shared__ double bestv[64][17];
  __shared__ int besti[64][17];
  const int c = threadIdx.x & 15, q = threadIdx.x >> 4, g = blockIdx.x * 16 + c;
  double bv = -1.0;
  int bi = 0x7fffffff;
  if (g < n)
    for (int i = q; i < n; i += 64) {
      const double a = fabs(Zin[(size_t)i * n + g]);
      if (a > bv) {  // the lowest row of the largest magnitude
        bv = a;
        bi = i;
      }
    }
  bestv[q][c] = bv;
  besti[q][c] = bi;
  __syncthreads();
  for (int o = 32; o > 0; o >>= 1) {
    if (q < o) {
      const double ov = bestv[q + o][c];
      const int oi = besti[q + o][c];
      if (ov > bestv[q][c] || (ov == bestv[q][c] && oi < besti[q][c])) {
        bestv[q][c] = ov;
        besti[q][c] = oi;
      }
    }
    __syncthreads();
  }
  if (g >= n) return;
  bi = besti[0][c];
  const double sgn = (bi < n && Zin[(size_t)bi * n + g] < 0.0) ? -1.0 : 1.0;
  const int dst = descending ? (n - 1 - rank[c]) : rank[c];
  if (q == 0) w_out[dst] = lam[g];
  for (int i = q; i < n; i += 64) Z_out[(size_t)i * n + dst] = sgn * Zin[(size_t)i * n + g];
}

// *floor = rel * (largest eigenvalue magnitude)
__global__ void lam_floor(int n, const double* lam, double rel, double* floor) {
  __shared__ double m[64];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 64) v = fmax(v, fabs(lam[i]));
  m[threadIdx.x] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 64; ++i) v = fmax(v, m[i]);
    *floor = rel * fmax(v, m[0]);
  }
}

__global__ void zero_int(int* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

}  // namespace

size_t eigh_workspace_bytes(int n) {
  const size_t nn = (size_t)n * n;
  size_t b = 0;
  auto add = [&](size_t x) { b += align_up(x, 256); };
  add(nn * 8);      // A work copy
  add(nn * 8);      // reflectors
  add(nn * 8);      // X (tridiagonal eigenvectors, then back-transformed)
  add(5 * nn * 8);  // LU columns
  add((size_t)n * 8 * 5);  // tau d e p lam
  add((size_t)n * 4 * 3 + 64);  // blk_start blk_end done status
  add(64);          // tnorm
  add((size_t)((n + WY_NB - 1) / WY_NB + 1) * WY_NB * WY_NB * 8);  // compact-WY T factors
  return b;
}

// resident: try the one-launch tridiagonalization
static int eigh_attempt(const double* A_in, int n, double* w_out, double* Z_out, char* ws, size_t ws_bytes,
                        hipStream_t st, int descending, double vec_floor_rel, bool resident, EighPath path, int* hs) {
  if (n < 1 || n > kEighMaxN) return fail(DFPT2_ERR_INVALID_ARG, "eigh: n=%d outside [1, %d]", n, kEighMaxN);
  if (ws_bytes < eigh_workspace_bytes(n)) return fail(DFPT2_ERR_WORKSPACE, "eigh workspace too small");
  const size_t nn = (size_t)n * n;
  size_t off = 0;
  auto take = [&](size_t x) {
    char* p = ws + off;
    off += align_up(x, 256);
    return p;
  };
  double* A = (double*)take(nn * 8);
  double* Vs = (double*)take(nn * 8);
  double* X = (double*)take(nn * 8);
  double* lu = (double*)take(5 * nn * 8);
  double* tau = (double*)take((size_t)n * 8 * 5);
  double* d = tau + n;
  double* e = d + n;
  double* p = e + n;
  double* lam = p + n;
  int* blk_start = (int*)take((size_t)n * 4 * 3 + 64);
  int* blk_end = blk_start + n;
  int* done = blk_end + n;
  int* status = done + n;
  double* tnorm = (double*)take(64);
  double* Tall = (double*)take((size_t)((n + WY_NB - 1) / WY_NB + 1) * WY_NB * WY_NB * 8);
  hipError_t err;
  ProfScope prof_all(DFPT2_STAGE_EIGH, st);
  // 1. tridiagonalization: in one launch up to kResidentMax (the slots of its vectors lie
  //    in the LU columns); else one lazy-update launch per column where its LDS staging
  //    fits in 64 KB; else the two-launch form
  double* pb[2] = {p, lam};  // p of consecutive columns alternate (lam is free until step 2)
  unsigned long long* slots = reinterpret_cast<unsigned long long*>(lu);
  resident = resident && n >= 3 && n <= kResidentMax &&
             launch_resident(A_in, n, A, Vs, tau, d, e, slots, slots + nn, pb[(n - 3) & 1], status, st,
                             path);
  if (!resident) hipLaunchKernelGGL(zero_int, dim3(1), dim3(64), 0, st, status, 1);
  if (!resident && (err = hipMemcpyAsync(A, A_in, nn * 8, hipMemcpyDeviceToDevice, st)) != hipSuccess)
    return hip_fail(err, "eigh copy");
  const double* p_last = nullptr;
  if (resident) {
    p_last = pb[(n - 3) & 1];
  } else if (n >= 3 && (size_t)(3 * (n - 1) + 2) * 8 <= 64 * 1024) {
    for (int k = 0; k + 2 < n; ++k) {
      const int m = n - k - 1;
      int ga = (m + 3) / 4;
      if (ga > 512) ga = 512;
      hipLaunchKernelGGL(tridiag_step_lazy, dim3(ga), dim3(256), (size_t)(3 * m + 2) * 8, st, A, n, k, Vs, tau, d,
                         e, pb[(k + 1) & 1], pb[k & 1]);
    }
    p_last = pb[(n - 3) & 1];
  } else {
    for (int k = 0; k + 2 < n; ++k) {
      const int m = n - k - 1;
      int ga = (m + 3) / 4;
      if (ga > 512) ga = 512;
      hipLaunchKernelGGL(tridiag_step_a, dim3(ga), dim3(256), (size_t)m * 8, st, A, n, k, Vs, tau, d, e, p);
      int gx = (m + 255) / 256;
      int gy = (m + 15) / 16;
      if (gy > 256) gy = 256;
      hipLaunchKernelGGL(tridiag_step_b, dim3(gx, gy), dim3(256), 0, st, A, n, k, Vs, tau, p);
    }
  }
  // 2. split + multisection
  hipLaunchKernelGGL(tridiag_split, dim3(1), dim3(1024), 0, st, n, d, e, blk_start, blk_end, tnorm, A, Vs, tau, p_last);
  // (the factors T of the back-transformation's 16-blocks go to A, free by now, where it holds
  // them: from n = 23 on; else later to the LU columns)
  const bool wy16 = n >= 8 && n <= 2048, early = wy16 && n >= 23;
  const int nblk16 = (n - 2 + WY16 - 1) / WY16, nb = early ? nblk16 : 0;
  const size_t de_bytes = std::max((size_t)n * 16, early ? kWySh * sizeof(double) : 0);
  if (n <= 256)
    hipLaunchKernelGGL((tridiag_multisect<true, 4>), dim3(n + nb), dim3(256), de_bytes, st, n, d, e, blk_start, blk_end,
                       tnorm, lam, nb, Vs, tau, A);
  else if (n <= 512)
    hipLaunchKernelGGL((tridiag_multisect<true, 2>), dim3(n + nb), dim3(128), de_bytes, st, n, d, e, blk_start, blk_end,
                       tnorm, lam, nb, Vs, tau, A);
  else if (n <= kSturmLds)
    hipLaunchKernelGGL((tridiag_multisect<true, 1>), dim3((n + 3) / 4 + nb), dim3(256), de_bytes, st, n, d, e, blk_start,
                       blk_end, tnorm, lam, nb, Vs, tau, A);
  else
    hipLaunchKernelGGL((tridiag_multisect<false, 1>), dim3((n + 3) / 4), dim3(256), 0, st, n, d, e, blk_start, blk_end,
                       tnorm, lam, 0, Vs, tau, A);
  const dim3 tw_grid((n + 63) / 64);
  // 3. eigenvectors of isolated eigenvalues by twisted factorizations, the others by
  //    inverse iteration
  LuCols L{lu, lu + nn, lu + 2 * nn, lu + 3 * nn, lu + 4 * nn};
  const double* floor_ptr = nullptr;
  if (vec_floor_rel > 0.0) {
    hipLaunchKernelGGL(lam_floor, dim3(1), dim3(64), 0, st, n, lam, vec_floor_rel, tnorm + 1);
    floor_ptr = tnorm + 1;
  }
  if (twisted_bytes(n, 4) <= kTwistedLds)
    hipLaunchKernelGGL(tridiag_twisted<4>, dim3((n + 3) / 4), dim3(64), twisted_bytes(n, 4), st, n, d, e, blk_start,
                       blk_end, tnorm, lam, X, done, floor_ptr);
  else if (twisted_bytes(n, 1) <= kTwistedLds)
    hipLaunchKernelGGL(tridiag_twisted<1>, dim3(n), dim3(64), twisted_bytes(n, 1), st, n, d, e, blk_start, blk_end,
                       tnorm, lam, X, done, floor_ptr);
  else
    hipLaunchKernelGGL(zero_done, dim3((n + 255) / 256), dim3(256), 0, st, n, done);
  hipLaunchKernelGGL(tridiag_inverse_iteration, tw_grid, dim3(64), 0, st, n, d, e, blk_start, blk_end, tnorm, lam, L, X,
                     status, floor_ptr, done);
  // 4. back-transformation (compact-WY blocks): on the matrix pipe while a workgroup's
  //    16 columns fit its registers
  if (wy16) {
    double* Tall = early ? A : lu;
    if (!early) hipLaunchKernelGGL(wy16_build_t, dim3(nblk16), dim3(256), 0, st, n, Vs, tau, Tall);
    const dim3 grid((n + 15) / 16), block(512);
    if (n <= 128) hipLaunchKernelGGL(backtransform16<1>, grid, block, 0, st, n, Vs, Tall, X);
    else if (n <= 512) hipLaunchKernelGGL(backtransform16<4>, grid, block, 0, st, n, Vs, Tall, X);
    else if (n <= 1280) hipLaunchKernelGGL(backtransform16<10>, grid, block, 0, st, n, Vs, Tall, X);
    else hipLaunchKernelGGL(backtransform16<16>, grid, block, 0, st, n, Vs, Tall, X);
  } else if (n > 2) {
    const int cw = (size_t)n * 2 * 8 <= 150 * 1024 ? 2 : 1;  // columns per workgroup that the LDS holds
    if ((size_t)n * cw * 8 > 150 * 1024) return fail(DFPT2_ERR_UNSUPPORTED, "eigh: n=%d too large", n);
    const int nblk = (n - 2 + WY_NB - 1) / WY_NB;
    hipLaunchKernelGGL(wy_build_t, dim3(nblk), dim3(256), 0, st, n, Vs, tau, Tall);
    const dim3 grid((n + cw - 1) / cw), block(256);
    const size_t bytes = (size_t)n * cw * 8;
    if (cw == 2) hipLaunchKernelGGL(tridiag_backtransform<2>, grid, block, bytes, st, n, Vs, Tall, X);
    else hipLaunchKernelGGL(tridiag_backtransform<1>, grid, block, bytes, st, n, Vs, Tall, X);
  }
  // 5. one first-order orthonormalization of all columns: with G = Z^T Z = I + E
  //    and E small, Z <- Z (I - U), U = strict upper part of E + diag(E) / 2, leaves
  //    Z^T Z = I + O(E^2).  E is non-negligible only between vectors of close
  //    eigenvalues whose gap inverse iteration left unresolved (relative gaps
  //    just above the grouping tolerance), and mixing those moves the residuals
  //    by no more than their gap times E.  The LU columns are free by now.
  double* G = lu;
  double* Zo = lu + nn;
  double* Part = lu + 2 * nn;  // partial products, 3 nn; only the upper triangle of G is read
  if (n <= 512) {  // the whole of M at once: a launch less, few flops more
    if ((err = gemm_f64_orth(X, n, G, Part, 3 * nn, st)) != hipSuccess) return hip_fail(err, "eigh orthonormalization");
  } else {
    if ((err = gemm_f64(X, n, 0, 1, X, n, 0, 0, G, n, 0, n, n, n, 1, 1.0, 0.0, st, Part, 3 * nn, true)) != hipSuccess)
      return hip_fail(err, "eigh orthonormalization");
    hipLaunchKernelGGL(orth_correction, dim3((unsigned)((nn + 255) / 256 < 65535 ? (nn + 255) / 256 : 65535)),
                       dim3(256), 0, st, n, G);
  }
  if ((err = gemm_f64(X, n, 0, 0, G, n, 0, 0, Zo, n, 0, n, n, n, 1, 1.0, 0.0, st, Part, 3 * nn)) != hipSuccess)
    return hip_fail(err, "eigh orthonormalization");
  // 6. sort + orient
  hipLaunchKernelGGL(eig_permute, dim3((n + 15) / 16), dim3(1024), 0, st, n, lam, Zo, w_out, Z_out, descending,
                     status);
  if ((err = hipGetLastError()) != hipSuccess) return hip_fail(err, "eigh launch");
  prof_all.close();
  if ((err = hipMemcpyAsync(hs, status, sizeof(int), hipMemcpyDeviceToHost, st)) != hipSuccess)
    return hip_fail(err, "eigh status copy");
  if ((err = hipStreamSynchronize(st)) != hipSuccess) return hip_fail(err, "eigh sync");
  prof_flush();
  return DFPT2_OK;
}

int eigh_run(const double* A_in, int n, double* w_out, double* Z_out, char* ws, size_t ws_bytes, hipStream_t st,
             int descending, double vec_floor_rel, EighPath path, int* attempts) {
  int hs = 0;
  int rc = eigh_attempt(A_in, n, w_out, Z_out, ws, ws_bytes, st, descending, vec_floor_rel, true, path, &hs);
  if (attempts) *attempts = 1;
  // 2: the workgroups of the resident form did not meet in time (held off the GPU by
  // other work); the launch-per-column form waits for nothing
  if (rc == DFPT2_OK && hs == 2) {
    rc = eigh_attempt(A_in, n, w_out, Z_out, ws, ws_bytes, st, descending, vec_floor_rel, false, path, &hs);
    if (attempts) *attempts = 2;
  }
  if (rc != DFPT2_OK) return rc;
  if (hs != 0) return fail(DFPT2_ERR_NOT_CONVERGED, "inverse iteration produced a zero or non-finite vector");
  return DFPT2_OK;
}

}  // namespace dfpt2

extern "C" int dfpt2_eigh_sym_path(const double* A, int64_t n, double* w, double* Z, void* workspace, size_t ws_bytes,
                                   dfpt2_stream_t stream, int path, int* attempts) {
  using namespace dfpt2;
  g_last_error.clear();
  if (!A || !w || !Z || !workspace) return fail(DFPT2_ERR_INVALID_ARG, "null pointer argument");
  if (n < 1 || n > kEighMaxN || path < 0 || path > 2) return fail(DFPT2_ERR_INVALID_ARG, "bad argument");
  return eigh_run(A, (int)n, w, Z, static_cast<char*>(workspace), ws_bytes, reinterpret_cast<hipStream_t>(stream), 0,
                  -1.0, static_cast<EighPath>(path), attempts);
}
