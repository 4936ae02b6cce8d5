// Small kernels: fills, pair-list compaction and the compensated energy reductions.
#include <cmath>
#include "common.h"
#include "kernels.h"

namespace dfpt2 {

__global__ void fill_kernel(double* p, size_t n, double v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

hipError_t launch_fill(double* p, size_t n, double v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

// Start of a pass, one launch (five before, 2 us and a gap of as much each: a tenth of a
// small molecule's pass).  Workgroup 0 lists the pairs; the others clear the per-pair
// results (core-core entries start at 0 and masked pairs stay 0), the density's partial
// slices and its diagonal.
//
// The list: unordered core-core pairs (i <= j) whose mask entry is set, in row-major
// order.  One wave per row i: each lane scans a strip of j, a wave prefix sum
// places the survivors, and rows are laid out by a serial scan of row counts
// done by the first wave (n_core is at most a few hundred).
// count[0]: their number; count[1] = 0, set later by the BF16 split when a row of B lies
// below the range its slices need.
__global__ __launch_bounds__(1024) void pass_begin_kernel(const uint8_t* mask, int n_core, int n_h, int2* pairs,
                                                          int* count, double* pair_energy, float* pair_tnorm,
                                                          double* Dpart, size_t n_Dpart, double* diag, int n_diag) {
  __shared__ int row_start[1025];
  if (blockIdx.x > 0) {
    const size_t i0 = (size_t)(blockIdx.x - 1) * blockDim.x + threadIdx.x, step = (size_t)(gridDim.x - 1) * blockDim.x;
    const size_t nn = (size_t)n_h * n_h;
    for (size_t i = i0; i < n_Dpart; i += step) Dpart[i] = 0.0;
    if (pair_energy)
      for (size_t i = i0; i < nn; i += step) pair_energy[i] = 0.0;
    if (pair_tnorm)
      for (size_t i = i0; i < nn; i += step) pair_tnorm[i] = 0.0f;
    for (size_t i = i0; i < (size_t)n_diag; i += step) diag[i] = 0.0;
    return;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  // row counts
  for (int i = w; i < n_core; i += nw) {
    int c = 0;
    for (int j = i + lane; j < n_core; j += 64) c += (mask == nullptr || mask[(size_t)i * n_h + j]) ? 1 : 0;
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (lane == 0) row_start[i + 1] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    row_start[0] = 0;
    for (int i = 0; i < n_core; ++i) row_start[i + 1] += row_start[i];
    count[0] = row_start[n_core];
    count[1] = 0;
  }
  __syncthreads();
  for (int i = w; i < n_core; i += nw) {
    int base = row_start[i];
    for (int j0 = i; j0 < n_core; j0 += 64) {
      const int j = j0 + lane;
      const int keep = (j < n_core) && (mask == nullptr || mask[(size_t)i * n_h + j]) ? 1 : 0;
      // exclusive prefix within the wave
      unsigned long long bal = __ballot(keep);
      const int before = __popcll(bal & ((1ull << lane) - 1ull));
      if (keep) pairs[base + before] = make_int2(i, j);
      base += __popcll(bal);
    }
  }
}

hipError_t launch_pass_begin(const uint8_t* mask, int n_core, int n_h, int2* pairs, int* count, double* pair_energy,
                             float* pair_tnorm, double* Dpart, size_t n_Dpart, double* diag, int n_diag,
                             hipStream_t st) {
  if (n_core > 1024) return hipErrorInvalidValue;
  size_t most = n_Dpart > (size_t)n_diag ? n_Dpart : (size_t)n_diag;
  if ((pair_energy || pair_tnorm) && (size_t)n_h * n_h > most) most = (size_t)n_h * n_h;
  const size_t blocks = most == 0 ? 0 : (most + 1023) / 1024;
  hipLaunchKernelGGL(pass_begin_kernel, dim3((unsigned)(1 + (blocks < 1024 ? blocks : 1024))), dim3(1024), 0, st, mask,
                     n_core, n_h, pairs, count, pair_energy, pair_tnorm, Dpart, n_Dpart, diag, n_diag);
  return hipGetLastError();
}

// one wave per pair: double-double sum of the tile partials
__global__ void pair_reduce_kernel(const double* epart, const double* tpart, int nTP, int n_pairs,
                                   double* pe, double* tn2) {
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (p >= n_pairs) return;
  double hi = 0.0, lo = 0.0, t = 0.0;
  for (int k = lane; k < nTP; k += 64) {
    if (epart) dd_add(hi, lo, epart[(size_t)p * nTP + k]);
    if (tpart) t += tpart[(size_t)p * nTP + k];
  }
  wave_sum_dd(hi, lo);
  t = wave_sum(t);
  if (lane == 0) {
    if (pe) {
      pe[2 * (size_t)p] = hi;
      pe[2 * (size_t)p + 1] = lo;
    }
    if (tn2) tn2[p] = t;
  }
}

hipError_t launch_pair_reduce(const double* epart, const double* tpart, int nTP, int n_pairs,
                              double* pe, double* tn2, hipStream_t st) {
  if (n_pairs <= 0) return hipSuccess;
  const int wpb = 4;
  hipLaunchKernelGGL(pair_reduce_kernel, dim3((n_pairs + wpb - 1) / wpb), dim3(64 * wpb), 0, st,
                     epart, tpart, nTP, n_pairs, pe, tn2);
  return hipGetLastError();
}

// single workgroup: E = sum of pair energies in double-double; scatter of the
// per-pair values into n_h x n_h matrices.
__global__ __launch_bounds__(1024) void energy_finalize_kernel(EnergyFinalizeArgs a) {
  __shared__ double sh[2][1024 / 64];
  const int n = *a.count;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const double* pe = a.pe;
  if (a.nTP > 0) {  // few tile partials: a thread per pair, which reads its own results below
    for (int p = threadIdx.x; p < n; p += blockDim.x) {
      double hi = 0.0, lo = 0.0, t = 0.0;
      for (int k = 0; k < a.nTP; ++k) {
        dd_add(hi, lo, a.epart[(size_t)p * a.nTP + k]);
        t += a.tpart[(size_t)p * a.nTP + k];
      }
      a.pe[2 * p] = hi;
      a.pe[2 * p + 1] = lo;
      a.tn2[p] = t;
    }
  }
  double hi = 0.0, lo = 0.0;
  for (int p = threadIdx.x; p < n; p += blockDim.x) dd_add_dd(hi, lo, pe[2 * p], pe[2 * p + 1]);
  for (int p = threadIdx.x; p < a.n_act_pairs; p += blockDim.x) dd_add_dd(hi, lo, a.pe_act[2 * p], a.pe_act[2 * p + 1]);
  wave_sum_dd(hi, lo);
  if (lane == 0) {
    sh[0][w] = hi;
    sh[1][w] = lo;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double h = 0.0, l = 0.0;
    for (int k = 0; k < nw; ++k) dd_add_dd(h, l, sh[0][k], sh[1][k]);
    a.e_out[0] = h;
    a.e_out[1] = l;
    if (a.correction) {
      double ch = a.e_full[0], cl = a.e_full[1];
      dd_add_dd(ch, cl, -h, -l);
      a.correction[0] = ch;
      a.correction[1] = cl;
    }
  }
  if (!a.pair_energy && !a.pair_tnorm) return;
  for (int p = threadIdx.x; p < n; p += blockDim.x) {
    const int2 pr = a.pairs[p];
    const double e = pe[2 * p] + pe[2 * p + 1];
    const double half = (pr.x == pr.y) ? e : 0.5 * e;
    if (a.pair_energy) {
      a.pair_energy[(size_t)pr.x * a.n_h + pr.y] = half;
      a.pair_energy[(size_t)pr.y * a.n_h + pr.x] = half;
    }
    if (a.pair_tnorm) {
      const float tn = (float)sqrt(a.tn2[p]);
      a.pair_tnorm[(size_t)pr.x * a.n_h + pr.y] = tn;
      a.pair_tnorm[(size_t)pr.y * a.n_h + pr.x] = tn;
    }
  }
}

hipError_t launch_energy_finalize(const EnergyFinalizeArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(energy_finalize_kernel, dim3(1), dim3(1024), 0, st, a);
  return hipGetLastError();
}

}  // namespace dfpt2
