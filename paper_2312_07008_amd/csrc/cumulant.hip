// The first-order singles (Eq. A6) and the Eq. A9 terms that carry them or the
// two-body density cumulant lambda_uv^xy of the reference:
//     D1  2 t_e^m t_f^m + t_e^u t_f^v gamma_u^v
//     D2  (t_e^u t_fv^xy + t_ey^uv t_f^x) lambda_uv^xy
//     D3  t_ee'^uv t_fe'^xy lambda_uv^xy
//     D4  P( t_ey^mv t_fu^mx ) lambda_uv^xy
//     D5  1/2 t_ez^uv t_fw^xy eta_w^z lambda_uv^xy
//     D6  1/2 P( t_ey^wv t_fu^zx ) gamma_w^z lambda_uv^xy
// (t_ab^ij: particles a, b created, holes i, j annihilated; m core, u..z active,
// e, f, e' virtual; eta = 2 - gamma; P(t_ap^ij t_cd^kq) = 2 t_ap^ij t_cd^kq -
// t_ap^ij t_cd^qk - t_ap^ji t_cd^kq - t_aq^ji t_cd^pk) with the singles
//     t_e^i = 1/2 sum_ux (eps_x - eps_u) gamma_x^u tc_ex^iu (1 - e^{-s D^2}) / D,
//     D = eps_i - eps_e,  tc_ab^ij = 2 t_ab^ij - t_ab^ji          (Eq. A6, f = 0).
//
// Every term but D3 is a rank-K product D += L R^T over a few small index
// ranges, with L a gather of the amplitudes X[e][i][j][x] = t_ex^ij (one virtual
// and one active particle, the same array as active_particle.hip) or of the
// singles, and R a contraction of amplitudes with lambda, gamma or eta.  D4 and
// D6 are one form over every hole h with the hole weight w (1 on core holes,
// gamma / 2 on active ones, as the 1/2 and gamma_w^z of D6 and the shared core
// index of D4 make them):
//     sum_{h v y} X[e][h][v][y] (w (2 Q1 - Q2))[f][h v y]
//   - sum_{h v y} X[e][v][h][y] (w (Q1 + Q4))[f][h v y],
//     Q1[f][h v y] = sum_{u x} X[f][h][x][u] lambda_uv^xy,
//     Q2[f][h v y] = sum_{u x} X[f][x][h][u] lambda_uv^xy,
//     Q4[f][h v y] = sum_{u x} X[f][x][h][u] lambda_uv^yx.
// The K columns are [D4+D6 first half | second half | D5 | D1 | D2]; one FP64
// MFMA GEMM forms E = L R^T.  D3 needs the virtual-virtual amplitudes of the
// active hole pairs, T[e][uv][e'] (one GEMM), mixed with lambda
// over the hole pair (a GEMM batched over e) and contracted over (uv, e') into
// the same E.  Each term is symmetric in (e, f); D += (E + E^T) / 2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "../../include/dfpt2.h"
#include "common.h"
#include "host.h"

namespace dfpt2 {
namespace {

__device__ inline size_t xidx(int e, int i, int j, int x, int n_h, int n_a) {
  return (((size_t)e * n_h + i) * n_h + j) * n_a + x;
}

// The kernels over X take one e (or f) per grid row and index within it in 32 bits: the
// 64-bit divisions by run-time sizes of one flat index cost more than the memory they go
// through.  Measured below at 400 virtuals and 48 holes, 8 of them active.

// X[e][i][j][x] *= (1 - exp(-s D^2)) / D,  D = eps_i + eps_j - eps_e - eps_(n_core + x)
// (42 us with one flat index, 31 so)
__global__ void cs_regularize_x(double* X, const double* eps_h, const double* eps_v, int n_h, int n_a, int n_core,
                                double s) {
  const unsigned per = (unsigned)n_h * n_h * n_a;
  const double ee = eps_v[blockIdx.y];
  double* Xe = X + (size_t)blockIdx.y * per;
  for (unsigned k = blockIdx.x * blockDim.x + threadIdx.x; k < per; k += gridDim.x * blockDim.x) {
    const unsigned ij = k / n_a, x = k - ij * n_a, i = ij / n_h, j = ij - i * n_h;
    const double dl = eps_h[i] + eps_h[j] - ee - eps_h[n_core + x];
    Xe[k] = (dl != 0.0) ? Xe[k] * (1.0 - exp(-s * dl * dl)) / dl : 0.0;
  }
}

// T[e][u v][e'] *= (1 - exp(-s D^2)) / D,  D = eps_u + eps_v - eps_e - eps_e'.  As a matrix
// of rows r = (u, e) and columns c = (v, e') T is symmetric and only r <= c is read; a
// workgroup takes a 32 x 32 tile (I <= J) and writes it and, through LDS, its transpose.
__global__ __launch_bounds__(256) void cs_regularize_t(double* T, const double* eps_h, const double* eps_v, int n_v,
                                                       int n_a, int n_core, double s) {
  __shared__ double tr[32][33];
  const unsigned m = (unsigned)n_a * n_v;
  int I, J;
  tile_pair(blockIdx.x, (int)((m + 31) / 32), I, J);
  const size_t K3 = (size_t)n_a * m;
  const unsigned x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const unsigned c = J * 32 + x, v = c / n_v;
  const double ec = c < m ? eps_h[n_core + v] - eps_v[c - v * n_v] : 0.0;
  for (unsigned q = y; q < 32; q += 8) {
    const unsigned r = I * 32 + q, u = r / n_v, e = r - u * n_v;
    if (r > c || c >= m) continue;
    double* t = T + e * K3 + (size_t)u * m + c;
    const double dl = (eps_h[n_core + u] - eps_v[e]) + ec;
    const double z = (dl != 0.0) ? *t * (1.0 - exp(-s * dl * dl)) / dl : 0.0;
    *t = z;
    tr[q][x] = z;
  }
  __syncthreads();
  for (unsigned q = y; q < 32; q += 8) {
    const unsigned r = J * 32 + q, u = r / n_v, e = r - u * n_v, c2 = I * 32 + x;
    if (r < m && c2 < r) T[e * K3 + (size_t)u * m + c2] = tr[x][q];
  }
}

// singles t1[i][e] (Eq. A6 with f = 0): one wave per (e, i), lanes over (u, x)
__global__ void cs_singles(const double* X, const double* eps_h, const double* eps_v, const double* gamma, int n_v,
                           int n_h, int n_a, int n_core, double s, double* t1) {
  const int e = blockIdx.y, i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n_h) return;
  double src = 0.0;
  for (int k = lane; k < n_a * n_a; k += 64) {
    const int u = k / n_a, x = k - u * n_a;
    const double w = (eps_h[n_core + x] - eps_h[n_core + u]) * gamma[x * n_a + u];
    if (w == 0.0) continue;
    src += w * (2.0 * X[xidx(e, i, n_core + u, x, n_h, n_a)] - X[xidx(e, n_core + u, i, x, n_h, n_a)]);
  }
  src = wave_sum(src);
  const double dl = eps_h[i] - eps_v[e];
  if (lane == 0) t1[(size_t)i * n_v + e] = (dl != 0.0) ? 0.5 * src * (1.0 - exp(-s * dl * dl)) / dl : 0.0;
}

// Qa = 2 Q1 - Q2 and Qb = -(Q1 + Q4), [f][h][v][y].  A workgroup takes one f and 24 holes:
// the amplitudes go through LDS (a few x at a time), a lane has one (v, y) of six holes, so
// that each element of lambda read serves six sums (180 us with one output a thread and all
// reads from memory, 36 so).
constexpr int kQHoles = 6;
__global__ __launch_bounds__(256) void cs_q(const double* X, const double* lam, int n_h, int n_a, int n_core, double* Qa,
                                            double* Qb) {
  constexpr int H = 4 * kQHoles;
  __shared__ double a1[H][64], a2[H][64];
  const int f = blockIdx.y, h0 = blockIdx.x * H, tid = threadIdx.x, lane = tid & 63, g = tid >> 6;
  const int xc = n_a < 8 ? n_a : 64 / n_a, n2 = n_a * n_a;  // x at a time: xc n_a <= 64
  for (int vy0 = 0; vy0 < n2; vy0 += 64) {
    const int vy = min(vy0 + lane, n2 - 1), v = vy / n_a, y = vy - v * n_a;
    double q1[kQHoles] = {}, q2[kQHoles] = {}, q4[kQHoles] = {};
    for (int x0 = 0; x0 < n_a; x0 += xc) {
      const int nx = min(xc, n_a - x0) * n_a;
      __syncthreads();
      for (int k = tid; k < H * 64; k += 256) {
        const int h = min(h0 + (k >> 6), n_h - 1), q = k & 63, dx = q / n_a, u = q - dx * n_a;
        if (q < nx) {
          a1[k >> 6][q] = X[xidx(f, h, n_core + x0 + dx, u, n_h, n_a)];
          a2[k >> 6][q] = X[xidx(f, n_core + x0 + dx, h, u, n_h, n_a)];
        }
      }
      __syncthreads();
      for (int q = 0; q < nx; ++q) {
        const int dx = q / n_a, u = q - dx * n_a, x = x0 + dx;
        const size_t uv = ((size_t)u * n_a + v) * n2;
        const double l = lam[uv + x * n_a + y], lt = lam[uv + y * n_a + x];
#pragma unroll
        for (int k = 0; k < kQHoles; ++k) {
          const double b1 = a1[g * kQHoles + k][q], b2 = a2[g * kQHoles + k][q];
          q1[k] += b1 * l;
          q2[k] += b2 * l;
          q4[k] += b2 * lt;
        }
      }
    }
    if (vy0 + lane >= n2) continue;
#pragma unroll
    for (int k = 0; k < kQHoles; ++k) {
      const int h = h0 + g * kQHoles + k;
      if (h >= n_h) continue;
      const size_t o = ((size_t)f * n_h + h) * n2 + vy;
      Qa[o] = 2.0 * q1[k] - q2[k];
      Qb[o] = -(q1[k] + q4[k]);
    }
  }
}

// W1[f][u] = sum_{v x y} t_fv^xy lambda_uv^xy and
// R5[f][u v z] = 1/2 sum_{x y w} t_fw^xy eta_w^z lambda_uv^xy, one workgroup per f: a wave per
// u, and t eta for a few z at a time in LDS (82 and 133 us with a thread per output, 17 so)
__global__ __launch_bounds__(512) void cs_w1_r5(const double* X, const double* lam, const double* gamma, int n_h, int n_a,
                                                int n_core, double* W1, double* R5) {
  __shared__ double xe[4096];
  const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63, n2 = n_a * n_a;
  for (int u = tid >> 6; u < n_a; u += 8) {
    double acc = 0.0;
    for (int k = lane; k < n2 * n_a; k += 64) {
      const int v = k / n2, xy = k - v * n2, x = xy / n_a, y = xy - x * n_a;
      acc += X[xidx(f, n_core + x, n_core + y, v, n_h, n_a)] * lam[(size_t)u * n2 * n_a + k];
    }
    acc = wave_sum(acc);
    if (lane == 0) W1[(size_t)f * n_a + u] = acc;
  }
  const int zc = min(n_a, 4096 / n2);
  for (int z0 = 0; z0 < n_a; z0 += zc) {
    const int nz = min(zc, n_a - z0);
    __syncthreads();
    for (int k = tid; k < n2 * nz; k += 512) {
      const int xy = k / nz, z = z0 + k - xy * nz, x = xy / n_a, y = xy - x * n_a;
      double acc = 0.0;
      for (int w = 0; w < n_a; ++w)
        acc += X[xidx(f, n_core + x, n_core + y, w, n_h, n_a)] * ((w == z ? 2.0 : 0.0) - gamma[w * n_a + z]);
      xe[k] = acc;
    }
    __syncthreads();
    for (int k = tid; k < n2 * nz; k += 512) {
      const int uv = k / nz, dz = k - uv * nz;
      double acc = 0.0;
#pragma unroll 4
      for (int xy = 0; xy < n2; ++xy) {
        const double l = lam[(size_t)uv * n2 + xy];
        acc += l == 0.0 ? 0.0 : xe[xy * nz + dz] * l;
      }
      R5[((size_t)f * n2 + uv) * n_a + z0 + dz] = 0.5 * acc;
    }
  }
}

struct CsDims {
  int n_v, n_h, n_a, n_core;
  int kA, kC, kD, kE, K;  // column ranges: A (and B) = n_h n_a^2, C = n_a^3, D = n_h, E = 2 n_a
  bool lam;
};

// L[e][k] (gathers) and R[f][k] (contractions, hole weight w on segments A/B)
__global__ void cs_build_lr(const double* X, const double* t1, const double* Qa, const double* Qb, const double* R5,
                            const double* W1, const double* gamma, CsDims d, double* L, double* R) {
  const size_t n = (size_t)d.n_v * d.K;
  const int n_h = d.n_h, n_a = d.n_a, nc = d.n_core, n_v = d.n_v;
  for (size_t q = blockIdx.x * (size_t)blockDim.x + threadIdx.x; q < n; q += (size_t)gridDim.x * blockDim.x) {
    const int row = (int)(q / d.K);
    int k = (int)(q - (size_t)row * d.K);
    double lv = 0.0, rv = 0.0;
    if (d.lam && k < 2 * d.kA) {  // D4 + D6
      const bool second = k >= d.kA;
      if (second) k -= d.kA;
      const int y = k % n_a, v = (k / n_a) % n_a, h = k / (n_a * n_a);
      lv = second ? X[xidx(row, nc + v, h, y, n_h, n_a)] : X[xidx(row, h, nc + v, y, n_h, n_a)];
      const double* Q = second ? Qb : Qa;
      if (h < nc) {
        rv = Q[(((size_t)row * n_h + h) * n_a + v) * n_a + y];
      } else {
        const int w = h - nc;
        double acc = 0.0;
        for (int z = 0; z < n_a; ++z) acc += gamma[w * n_a + z] * Q[(((size_t)row * n_h + nc + z) * n_a + v) * n_a + y];
        rv = 0.5 * acc;
      }
    } else {
      if (d.lam) k -= 2 * d.kA;
      if (d.lam && k < d.kC) {  // D5
        const int z = k % n_a, v = (k / n_a) % n_a, u = k / (n_a * n_a);
        lv = X[xidx(row, nc + u, nc + v, z, n_h, n_a)];
        rv = R5[(size_t)row * d.kC + k];
      } else {
        if (d.lam) k -= d.kC;
        if (k < d.kD) {  // D1: k = hole i
          lv = t1[(size_t)k * n_v + row];
          if (k < nc) {
            rv = 2.0 * t1[(size_t)k * n_v + row];
          } else {
            double acc = 0.0;
            for (int v = 0; v < n_a; ++v) acc += gamma[(k - nc) * n_a + v] * t1[(size_t)(nc + v) * n_v + row];
            rv = acc;
          }
        } else {  // D2 (only with lambda): t_e^u W1[f][u], then W1[e][x] t_f^x
          k -= d.kD;
          if (k < n_a) {
            lv = t1[(size_t)(nc + k) * n_v + row];
            rv = W1[(size_t)row * n_a + k];
          } else {
            k -= n_a;
            lv = W1[(size_t)row * n_a + k];
            rv = t1[(size_t)(nc + k) * n_v + row];
          }
        }
      }
    }
    L[q] = lv;
    R[q] = rv;
  }
}

// D += scale (E + E^T) / 2
__global__ void cs_sym_add(const double* E, double* D, int n_v, double scale) {
  const size_t n = (size_t)n_v * n_v;
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const size_t a = k / n_v, b = k - a * n_v;
    D[k] += 0.5 * scale * (E[k] + E[b * n_v + a]);
  }
}

struct CsPlan {
  CsDims d;
  int n_aux;
  size_t off_X, off_t1, off_Qa, off_Qb, off_W1, off_R5, off_L, off_R, off_E, off_T, off_M, bytes;
};

int plan_cs(const dfpt2_opts* o, bool with_lambda, CsPlan* p) {
  if (!o) return fail(DFPT2_ERR_INVALID_ARG, "opts is null");
  PassPlan pp;
  const int st = plan_pass(o, &pp);  // the same size checks as the pass
  if (st != DFPT2_OK) return st;
  *p = CsPlan{};
  CsDims& d = p->d;
  d.n_core = (int)o->n_core;
  d.n_a = (int)o->n_act;
  d.n_h = d.n_core + d.n_a;
  d.n_v = (int)o->n_vir;
  d.lam = with_lambda;
  p->n_aux = (int)o->n_aux;
  const size_t n_v = d.n_v, n_h = d.n_h, n_a = d.n_a;
  d.kA = (int)(n_h * n_a * n_a);
  d.kC = (int)(n_a * n_a * n_a);
  d.kD = (int)n_h;
  d.kE = (int)(2 * n_a);
  d.K = with_lambda ? 2 * d.kA + d.kC + d.kD + d.kE : d.kD;
  const double k3 = (double)n_a * n_a * n_v;
  if ((double)n_h * n_h * n_a > 2.0e9 || k3 > 2.0e9)
    return fail(DFPT2_ERR_INVALID_ARG, "too many hole pairs x active orbitals");
  size_t off = 0;
  auto take = [&](size_t b) {
    const size_t o_ = off;
    off = align_up(off + b, 256);
    return o_;
  };
  p->off_X = take(sizeof(double) * n_v * n_h * n_h * n_a);
  p->off_t1 = take(sizeof(double) * n_h * n_v);
  p->off_Qa = take(with_lambda ? sizeof(double) * n_v * n_h * n_a * n_a : 0);
  p->off_Qb = take(with_lambda ? sizeof(double) * n_v * n_h * n_a * n_a : 0);
  p->off_W1 = take(with_lambda ? sizeof(double) * n_v * n_a : 0);
  p->off_R5 = take(with_lambda ? sizeof(double) * n_v * n_a * n_a * n_a : 0);
  p->off_L = take(sizeof(double) * n_v * (size_t)d.K);
  p->off_R = take(sizeof(double) * n_v * (size_t)d.K);
  p->off_E = take(sizeof(double) * n_v * n_v);
  p->off_T = take(with_lambda ? sizeof(double) * n_v * n_a * n_a * n_v : 0);
  p->off_M = take(with_lambda ? sizeof(double) * n_v * n_a * n_a * n_v : 0);
  p->bytes = off;
  return DFPT2_OK;
}

int grid_cs(size_t n) {
  const size_t g = (n + 255) / 256;
  return (int)(g < 65535 ? (g > 0 ? g : 1) : 65535);
}

}  // namespace
}  // namespace dfpt2

using namespace dfpt2;

extern "C" {

int dfpt2_cumulant_singles_workspace_size(const dfpt2_opts* opts, int with_lambda, size_t* bytes) {
  g_last_error.clear();
  if (!bytes) return fail(DFPT2_ERR_INVALID_ARG, "bytes is null");
  CsPlan p;
  const int st = plan_cs(opts, with_lambda != 0, &p);
  if (st != DFPT2_OK) return st;
  *bytes = p.bytes;
  return DFPT2_OK;
}

int dfpt2_add_cumulant_singles_density(const dfpt2_opts* opts, const double* eps_hole, const double* eps_vir,
                                       const double* gamma_act, const double* lambda_act, const double* B,
                                       const double* B_act, double* D_vv, double* t1_out, void* workspace,
                                       size_t ws_bytes, dfpt2_stream_t stream) {
  g_last_error.clear();
  CsPlan p;
  int st = plan_cs(opts, lambda_act != nullptr, &p);
  if (st != DFPT2_OK) return st;
  const CsDims& d = p.d;
  if (d.n_a == 0) return DFPT2_OK;  // no active orbitals: no singles source, no cumulant
  if (!eps_hole || !eps_vir || !gamma_act || !B || !B_act || !D_vv || !workspace)
    return fail(DFPT2_ERR_INVALID_ARG, "null pointer argument");
  if (ws_bytes < p.bytes) return fail(DFPT2_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, p.bytes);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  double* X = reinterpret_cast<double*>(ws + p.off_X);
  double* t1 = reinterpret_cast<double*>(ws + p.off_t1);
  double* Qa = reinterpret_cast<double*>(ws + p.off_Qa);
  double* Qb = reinterpret_cast<double*>(ws + p.off_Qb);
  double* W1 = reinterpret_cast<double*>(ws + p.off_W1);
  double* R5 = reinterpret_cast<double*>(ws + p.off_R5);
  double* L = reinterpret_cast<double*>(ws + p.off_L);
  double* R = reinterpret_cast<double*>(ws + p.off_R);
  double* E = reinterpret_cast<double*>(ws + p.off_E);
  double* T = reinterpret_cast<double*>(ws + p.off_T);
  double* M = reinterpret_cast<double*>(ws + p.off_M);
  const int n_v = d.n_v, n_h = d.n_h, n_a = d.n_a, nc = d.n_core, na = p.n_aux;
  const int KX = n_h * n_h * n_a, NA = n_h * n_a;
  const double sflow = opts->s;
  hipError_t e;
  ProfScope ps(DFPT2_STAGE_ACTIVE, s);
  // amplitudes with one active particle, X[e][(i, j, x)] (as active_particle.hip)
  if ((e = gemm_f64(B, na, 0, 0, B_act, na, 0, 1, X, KX, 0, n_h * n_v, NA, na, 1, 1.0, 0.0, s, nullptr, 0, false, n_v,
                    NA)) != hipSuccess)
    return hip_fail(e, "active-particle integrals");
  const size_t nx = (size_t)n_v * KX;
  hipLaunchKernelGGL(cs_regularize_x, dim3((unsigned)std::min((KX + 255) / 256, 4096), n_v), dim3(256), 0, s, X,
                     eps_hole, eps_vir, n_h, n_a, nc, sflow);
  hipLaunchKernelGGL(cs_singles, dim3((n_h + 3) / 4, n_v), dim3(256), 0, s, X, eps_hole, eps_vir, gamma_act,
                     n_v, n_h, n_a, nc, sflow, t1);
  if (d.lam) {
    hipLaunchKernelGGL(cs_q, dim3((n_h + 4 * kQHoles - 1) / (4 * kQHoles), n_v), dim3(256), 0, s, X, lambda_act, n_h, n_a,
                       nc, Qa, Qb);
    hipLaunchKernelGGL(cs_w1_r5, dim3(n_v), dim3(512), 0, s, X, lambda_act, gamma_act, n_h, n_a, nc, W1, R5);
  }
  hipLaunchKernelGGL(cs_build_lr, dim3(grid_cs((size_t)n_v * d.K)), dim3(256), 0, s, X, t1, Qa, Qb, R5, W1,
                     gamma_act, d, L, R);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "cumulant/singles kernels");
  // E = L R^T (X is free from here on: partial products of the split contractions)
  if ((e = gemm_f64(L, d.K, 0, 0, R, d.K, 0, 1, E, n_v, 0, n_v, n_v, d.K, 1, 1.0, 0.0, s, X, nx)) != hipSuccess)
    return hip_fail(e, "cumulant/singles density");
  if (d.lam) {
    // T[e][(u, v)][e'] = sum_Q B_ue^Q B_ve'^Q: rows (u, e) times themselves, the tiles from
    // the diagonal on (0.38 ms; 1.10 as a product per u batched over v)
    const int K3 = n_a * n_a * n_v, NAV = n_a * n_v;
    const double* Ba = B + (size_t)nc * n_v * na;
    if ((e = gemm_f64(Ba, na, 0, 0, Ba, na, 0, 1, T, K3, 0, NAV, NAV, na, 1, 1.0, 0.0, s, nullptr, 0, true, n_v, NAV)) !=
        hipSuccess)
      return hip_fail(e, "active-active integrals");
    const int nt = (NAV + 31) / 32;
    hipLaunchKernelGGL(cs_regularize_t, dim3((unsigned)nt * (nt + 1) / 2), dim3(256), 0, s, T, eps_hole, eps_vir, n_v,
                       n_a, nc, sflow);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "active-active amplitudes");
    // M[f][(u, v)][e'] = sum_(x, y) lambda_uv^xy T[f][(x, y)][e'], batched over f
    if ((e = gemm_f64(lambda_act, n_a * n_a, 0, 0, T, n_v, (long long)K3, 0, M, n_v, (long long)K3, n_a * n_a, n_v,
                      n_a * n_a, n_v, 1.0, 0.0, s)) != hipSuccess)
      return hip_fail(e, "cumulant mixing");
    // E += T M^T over (u v, e')
    if ((e = gemm_f64(T, K3, 0, 0, M, K3, 0, 1, E, n_v, 0, n_v, n_v, K3, 1, 1.0, 1.0, s, X, nx)) != hipSuccess)
      return hip_fail(e, "cumulant active-active term");
  }
  const double scale = opts->density_convention == 1 ? 0.5 : 1.0;
  hipLaunchKernelGGL(cs_sym_add, dim3(grid_cs((size_t)n_v * n_v)), dim3(256), 0, s, E, D_vv, n_v, scale);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "cumulant/singles add");
  if (t1_out && (e = hipMemcpyAsync(t1_out, t1, sizeof(double) * n_h * n_v, hipMemcpyDeviceToDevice, s)) != hipSuccess)
    return hip_fail(e, "singles copy");
  return DFPT2_OK;
}

}  // extern "C"
