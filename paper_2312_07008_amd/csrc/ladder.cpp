// Density-fitted particle-particle ladder (the N_C^2 N_V^4 part of the two-body
// contraction C2 = [O2, T2]_2 of the high-level step, Eq. 6), in the full or in
// the truncated virtual space, whose cost the FNO truncation cuts by
// (N_V'/N_V)^4 (Sec. 2):
//     (ac|bd) = sum_Q B^Q_ac B^Q_bd,     R^p_ab = sum_cd (ac|bd) T^p_cd.
//
// Integral-direct over blocks of the pairs (a, b), b <= a, whose matrices
// V^{ab}_cd = (ac|bd) serve both orders, V^{ba}_cd = V^{ab}_dc:
//     R^p_ab, R^p_ba = 1/2 sum_{c>=d} S^{ab}_cd T+^p_cd +- 1/2 sum_{c>d} A^{ab}_cd T-^p_cd
// with S, A = V_cd +- V_dc and T+, T- = T_cd +- T_dc (T+_cc = T_cc).  Half the integrals
// and half the contraction of R^p_ab = sum_cd (ac|bd) T^p_cd over all (a, b): N^4 n_aux +
// N^4 n_amp operations.  Per block
//   V[(a,b)][c][d] = sum_Q B[(a,c)][Q] B[(b,d)][Q]     (tiles with b <= a)
//   S, A           packed triangles of each V[(a,b)]
//   R              two GEMMs [p][triangle] x [triangle][(a,b)], stored to both (a,b), (b,a)
// What bounds it is the FP64 matrix pipe in the three GEMMs.  V and S, A hold some pairs
// at a time, ~16 GB in all (more only where 1024 pairs are).  N' = 133, 800 auxiliary functions, 400
// amplitude matrices, ms: integrals 4.8, split 0.7, contraction 2.7; over all (a, b) and
// (c, d) integrals 9.3, contraction 5.0.
//
// Truncated space: with the kept NOs X [N_V][ldx] (first N' columns) the inputs are transformed
// first, B'^Q = X^T B^Q X (over both virtual indices of B[a][c][Q]) and
// T'^p = X^T T^p X, by four more GEMMs.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/dfpt2.h"
#include "common.h"
#include "host.h"

namespace dfpt2 {
namespace {

struct LadderPlan {
  int n, nk, na, np, vcols, scols, tp;
  bool transform;
  size_t off_Y, off_Bk, off_Z, off_Tk, off_Tp, off_V, off_S, bytes;
};

constexpr double kVBytes = 2.0e9;    // V of the pairs whose integrals are formed at a time
constexpr double kSBytes = 14.0e9;   // S and A of the pairs that are contracted at a time
constexpr int kBlockPairs = 16384;   // pairs of either, where the bytes allow: enough to fill the GPU
constexpr int kMinPairs = 1024;      // pairs contracted at a time, whatever the bytes
constexpr double kTBytes = 2.0e9;    // T+ and T- of the amplitudes that are contracted at a time in the full space

int plan_ladder(int64_t n_vir, int64_t n_aux, int64_t n_amp, int64_t n_kept, bool transform, LadderPlan* pl) {
  if (n_vir < 1 || n_vir > 2048) return fail(DFPT2_ERR_INVALID_ARG, "n_vir must lie in [1, 2048]");
  if (n_aux < 1 || n_aux > (1 << 20)) return fail(DFPT2_ERR_INVALID_ARG, "n_aux must lie in [1, 2^20]");
  if (n_amp < 1 || n_amp > 65535) return fail(DFPT2_ERR_INVALID_ARG, "n_amp must lie in [1, 65535]");
  if (transform) {
    if (n_kept < 1 || n_kept > n_vir) return fail(DFPT2_ERR_INVALID_ARG, "n_kept must lie in [1, n_vir]");
  } else if (n_kept != 0 && n_kept != n_vir) {
    return fail(DFPT2_ERR_INVALID_ARG, "without X, n_kept must be 0 or n_vir");
  }
  LadderPlan& p = *pl;
  p = LadderPlan{};
  p.n = (int)n_vir;
  p.nk = transform ? (int)n_kept : (int)n_vir;
  p.na = (int)n_aux;
  p.np = (int)n_amp;
  p.transform = transform;
  const double pair = (double)p.nk * p.nk * sizeof(double), all = 0.5 * p.nk * (p.nk + 1.0);
  p.vcols = (int)std::max(1.0, std::min({all, (double)kBlockPairs, kVBytes / pair}));
  p.scols = (int)std::min(all, std::max((double)kMinPairs, std::min((double)kBlockPairs, kSBytes / pair)));
  if ((double)p.nk * p.na > 2.0e9 || (double)p.nk * p.nk > 2.0e9)
    return fail(DFPT2_ERR_INVALID_ARG, "ladder operands exceed the GEMM index range");
  size_t off = 0;
  auto take = [&](size_t b) {
    const size_t o = off;
    off = align_up(off + b, 256);
    return o;
  };
  const size_t d = sizeof(double);
  p.off_Y = take(transform ? d * p.n * p.nk * p.na : 0);
  p.off_Bk = take(transform ? d * p.nk * p.nk * p.na : 0);
  p.off_Z = take(transform ? d * p.np * p.n * p.nk : 0);
  p.off_Tk = take(transform ? d * p.np * p.nk * p.nk : 0);
  // T+ and T-: of all amplitudes where T' was formed, over the half-transformed Z (n >= nk);
  // in the full space of kTBytes at a time, split again for every block of pairs (a few percent of its
  // contraction at worst), so that the workspace does not grow with the amplitudes
  p.tp = transform ? p.np : (int)std::max(1.0, std::min((double)p.np, kTBytes / pair));
  p.off_Tp = transform ? p.off_Z : take(d * p.tp * p.nk * p.nk);
  p.off_V = take(d * p.vcols * p.nk * p.nk);
  p.off_S = take(d * p.scols * p.nk * p.nk);
  p.bytes = off;
  return DFPT2_OK;
}

// plus[m][c (c + 1) / 2 + d] = in[m][c][d] + in[m][d][c] (d < c), diag in[m][c][c] (d = c);
// minus[m][c (c - 1) / 2 + d] = in[m][c][d] - in[m][d][c] (d < c).  One workgroup per matrix
// and pair of 32 x 32 tiles, the transposed one through LDS; bound by memory.
__global__ __launch_bounds__(256) void sym_split_kernel(const double* in, int n, double diag, double* plus, double* minus) {
  __shared__ double tr[32][33];
  int J, I;
  tile_pair(blockIdx.x, (n + 31) / 32, J, I);  // J <= I
  const size_t m = blockIdx.y;
  const double* M = in + m * n * n;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
#pragma unroll
  for (int r = y; r < 32; r += 8) {
    const int c = J * 32 + r, d = I * 32 + x;
    tr[r][x] = c < n && d < n ? M[(size_t)c * n + d] : 0.0;
  }
  __syncthreads();
  double* P = plus + m * ((size_t)n * (n + 1) / 2);
  double* Q = minus + m * ((size_t)n * (n - 1) / 2);
#pragma unroll
  for (int r = y; r < 32; r += 8) {
    const int c = I * 32 + r, d = J * 32 + x;
    if (c >= n || d > c) continue;
    const double v = M[(size_t)c * n + d], w = tr[x][r];
    P[(size_t)c * (c + 1) / 2 + d] = c == d ? diag * v : v + w;
    if (d < c) Q[(size_t)c * (c - 1) / 2 + d] = v - w;
  }
}

void sym_split(const double* in, int n, int count, double diag, double* plus, double* minus, hipStream_t st) {
  const int nt = (n + 31) / 32;
  for (int m0 = 0; m0 < count; m0 += 65535) {
    const int k = std::min(65535, count - m0);
    hipLaunchKernelGGL(sym_split_kernel, dim3(nt * (nt + 1) / 2, k), dim3(256), 0, st, in + (size_t)m0 * n * n, n, diag,
                       plus + (size_t)m0 * n * (n + 1) / 2, minus + (size_t)m0 * n * (n - 1) / 2);
  }
}

}  // namespace
}  // namespace dfpt2

using namespace dfpt2;

extern "C" {

int pp_ladder_workspace_size(int64_t n_vir, int64_t n_aux, int64_t n_amp, int64_t n_kept, size_t* bytes) {
  g_last_error.clear();
  if (!bytes) return fail(DFPT2_ERR_INVALID_ARG, "bytes is null");
  LadderPlan p;
  const int st = plan_ladder(n_vir, n_aux, n_amp, n_kept, n_kept != 0, &p);
  if (st != DFPT2_OK) return st;
  *bytes = p.bytes;
  return DFPT2_OK;
}

int pp_ladder(int64_t n_vir, int64_t n_aux, int64_t n_amp, const double* B_vv, const double* T, const double* X,
              int64_t ldx, int64_t n_kept, double* R, void* workspace, size_t ws_bytes, dfpt2_stream_t stream) {
  g_last_error.clear();
  if (!B_vv || !T || !R || !workspace) return fail(DFPT2_ERR_INVALID_ARG, "null pointer argument");
  LadderPlan p;
  if (!X && n_kept != 0 && n_kept != n_vir) return fail(DFPT2_ERR_INVALID_ARG, "without X, n_kept must be 0 or n_vir");
  int st = plan_ladder(n_vir, n_aux, n_amp, X ? n_kept : 0, X != nullptr, &p);
  if (st != DFPT2_OK) return st;
  if (X && (ldx < n_kept || ldx > n_vir)) return fail(DFPT2_ERR_INVALID_ARG, "ldx must lie in [n_kept, n_vir]");
  if (ws_bytes < p.bytes) return fail(DFPT2_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, p.bytes);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  hipError_t e;
  const int n = p.n, nk = p.nk, na = p.na, np = p.np, lx = X ? (int)ldx : 0;
  const double* Bk = B_vv;
  const double* Tk = T;
  if (p.transform) {
    ProfScope ps(DFPT2_STAGE_LADDER_TRANSFORM, s);
    double* Y = reinterpret_cast<double*>(ws + p.off_Y);
    double* Bt = reinterpret_cast<double*>(ws + p.off_Bk);
    double* Z = reinterpret_cast<double*>(ws + p.off_Z);
    double* Tt = reinterpret_cast<double*>(ws + p.off_Tk);
    // Y[a] = X^T B[a]  (nk x na per a)
    if ((e = gemm_f64(X, lx, 0, 1, B_vv, na, (long long)n * na, 0, Y, na, (long long)nk * na, nk, na, n, n, 1.0, 0.0,
                      s)) != hipSuccess)
      return hip_fail(e, "ladder transform (B, first index)");
    // B'[a'][(c', Q)] = sum_a X[a][a'] Y[a][(c', Q)]
    if ((e = gemm_f64(X, lx, 0, 1, Y, nk * na, 0, 0, Bt, nk * na, 0, nk, nk * na, n, 1, 1.0, 0.0, s)) != hipSuccess)
      return hip_fail(e, "ladder transform (B, second index)");
    // Z[p] = T[p] X, T'[p] = X^T Z[p]
    if ((e = gemm_f64(T, n, (long long)n * n, 0, X, lx, 0, 0, Z, nk, (long long)n * nk, n, nk, n, np, 1.0, 0.0, s)) !=
        hipSuccess)
      return hip_fail(e, "ladder transform (T)");
    if ((e = gemm_f64(X, lx, 0, 1, Z, nk, (long long)n * nk, 0, Tt, nk, (long long)nk * nk, nk, nk, n, np, 1.0, 0.0,
                      s)) != hipSuccess)
      return hip_fail(e, "ladder transform (T)");
    Bk = Bt;
    Tk = Tt;
  }
  {
    ProfScope ps(DFPT2_STAGE_LADDER, s);
    double* V = reinterpret_cast<double*>(ws + p.off_V);
    const int kp = nk * (nk + 1) / 2, km = nk * (nk - 1) / 2;
    double* Tp = reinterpret_cast<double*>(ws + p.off_Tp);
    double* Tm = Tp + (size_t)p.tp * kp;
    if (p.tp == np) sym_split(Tk, nk, np, 1.0, Tp, Tm, s);
    double* S = reinterpret_cast<double*>(ws + p.off_S);
    double* A = S + (size_t)p.scols * kp;
    const int all = nk * (nk + 1) / 2;
    const size_t nv = (size_t)p.vcols * nk * nk;  // V is free while the pairs are contracted
    LadderBlock q{nk, 0, 0, 0, 0};
    for (int t = 0; t < all;) {
      const int t0 = t;
      while (t < all) {
        // the next rows a that fit, or the next part of a row
        const int room = p.scols - (t - t0), row = q.a0 + 1 - q.b0;
        if (t > t0 && room < std::min(row, p.vcols)) break;
        const int most = std::min(room, p.vcols);
        q.a1 = q.a0 + 1;
        if (q.b0 == 0 && row <= most) {
          while (q.a1 < nk && q.first(q.a1 + 1) <= most) ++q.a1;
          q.b1 = q.a1;
        } else {
          q.b1 = std::min(q.b0 + most, q.a1);
        }
        const int cols = q.columns();
        if ((e = ladder_integrals(Bk, na, q, V, s)) != hipSuccess) return hip_fail(e, "ladder integrals");
        sym_split(V, nk, cols, 2.0, S + (size_t)(t - t0) * kp, A + (size_t)(t - t0) * km, s);
        t += cols;
        if (q.b1 < q.a1) {
          q.b0 = q.b1;
        } else {
          q.a0 = q.a1;
          q.b0 = 0;
        }
      }
      for (int p0 = 0; p0 < np; p0 += p.tp) {
        const int m = std::min(p.tp, np - p0);
        double* Rp = R + (size_t)p0 * nk * nk;
        if (p.tp < np) sym_split(Tk + (size_t)p0 * nk * nk, nk, m, 1.0, Tp, Tm, s);
        if ((e = ladder_contract(Tp, S, m, kp, nk, t0, t - t0, true, Rp, V, nv, s)) != hipSuccess ||
            (km > 0 && (e = ladder_contract(Tm, A, m, km, nk, t0, t - t0, false, Rp, V, nv, s)) != hipSuccess))
          return hip_fail(e, "ladder contraction");
      }
    }
  }
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "ladder launch");
  return DFPT2_OK;
}

}  // extern "C"
