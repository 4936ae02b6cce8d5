// Batched FP64 GEMM on the 16x16x4 FP64 MFMA, used by the eigensolver, the NO
// transform and recanonicalization (Sec. 2), the natural auxiliary functions, the
// particle-particle ladder and the density terms with active particles:
//     C[b] = alpha op(A[b]) op(B[b]) + beta C[b],   op(A) M x K, op(B) K x N.
//
// What bounds it: the FP64 matrix pipe, 64 cycles per 16x16x4 product (78 TFLOP/s
// sustained by a loop of products alone).  A 16-deep chunk of a 64 x 64 tile is 16
// products per wave against 16 KB of operands, so LDS and L2 have slack; what costs
// time is whatever keeps a SIMD's waves from issuing products.  Hence:
//  * two chunks are fetched ahead into registers (8 bytes per lane: any leading dimension
//    and alignment) by buffer loads whose descriptor base moves with the chunk (scalar
//    arithmetic) at byte offsets that never change: no vector instruction and no branch
//    but the loads (8192 x 8192 x 2048: 60.3 TFLOP/s with 64-bit addresses per load,
//    62.6 so).  Rows beyond the matrix read a clamped row, whose products reach no stored
//    element; the last, partial chunk of the contraction runs on its own behind the loop
//    and selects zeros for both operands, so that an infinity or NaN behind the end of a
//    row cannot enter.
//  * LDS holds both operands k-major ([k][m], [k][n]) with rows of 18 (mod 32) doubles:
//    the 16 lanes along k that store a row of a k-contiguous operand and the 16 + 16
//    lanes that read a fragment hit distinct banks.
//  * three workgroups fit a unit and fill each other's waits at the barriers; a contraction
//    that is long for its number of tiles is split over workgroups whose partial tiles are
//    summed in a fixed order (choose_split).  128 x 128 tiles, two per unit: no faster at any
//    size tried (ladder of 133 virtuals 8.34 ms with them where they looked better, 8.10
//    without; 894 x 4000 x 1200 of 80 stacks the same).
// Measured against the kernel before (128 x 128 tiles, predicated loads, no split), TFLOP/s:
// A B^T 4256 x 17689 x 800 37 -> 56, A^T B 894 x 4000 x 1200 of 80 stacks 50 -> 61,
// A B 1200^3 14 -> 41, A B^T 400 x 400 x 18432 1.5 -> 33.  The second chunk in flight took the
// density terms of 40 + 8 holes and 400 virtuals from 1.96 to 1.90 ms.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "host.h"

namespace dfpt2 {

namespace {

struct GemmArgs {
  const double* A;
  const double* B;
  double* C;
  int M, N, K;
  int lda, ldb, ldc;
  long long sA, sB, sC;
  int row_n;          // row m of C lies at (m % row_n) ldc + (m / row_n) row_s (no groups: row_n = M)
  long long row_s;
  double alpha, beta;
  int batch, tm, tn;  // tiles along M and N
  int per;            // tiles of a product
  int nsplit, kper;   // splits of the contraction, chunks per split
  double* part;       // [nsplit][batch][M][N] partial products, or null (nsplit == 1)
  int upper;          // only the tiles that reach the diagonal or lie above it
  int orth;           // the product P is written as I - (strict upper part of P - I) - diag(P - I) / 2
  int mode;           // 0, or a form of the ladder (LadderBlock in host.h):
                      // kIntegrals: row (a, c), column (b, d) -> C[packed (a, b)][c][d], b <= a only
                      // kPlus:  column j = (a, b): v/2 to C[row][a][b] and C[row][b][a]
                      // kMinus: column j = (a, b): v/2 added to C[row][a][b], subtracted from C[row][b][a]
  LadderBlock lad;    // kIntegrals; else n, and the triangle's index of column 0 in a0
};
enum { kIntegrals = 1, kPlus, kMinus };

constexpr int GK = 16;     // contraction chunk
constexpr int kTile = 64;  // tile edge

// pair (a, b), b <= a, of index t of the triangle
__device__ inline void ladder_pair(int t, int& a, int& b) {
  a = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);  // off by at most one
  if ((long long)a * (a + 1) / 2 > t) --a;
  if ((long long)(a + 1) * (a + 2) / 2 <= t) ++a;
  b = (int)(t - (long long)a * (a + 1) / 2);
}

__device__ inline void ladder_store(double* R, int n, int a, int b, double v, bool plus) {
  double *ab = R + (size_t)a * n + b, *ba = R + (size_t)b * n + a;
  if (plus) {
    *ab = *ba = 0.5 * v;
  } else if (a != b) {
    *ab += 0.5 * v;
    *ba -= 0.5 * v;
  }
}

__device__ inline double* c_row(const GemmArgs& g, int b, int m) {
  const int q = m / g.row_n;
  return g.C + b * g.sC + (size_t)(m - q * g.row_n) * g.ldc + q * g.row_s;
}

__device__ inline double orth_value(double v, int m, int n) { return m < n ? -v : m == n ? 1.0 - 0.5 * (v - 1.0) : 0.0; }

constexpr int BAND = 8;  // tile rows of a band

// first tile column and number of tile columns that a band of tile rows has:
// all; of an integral block those with a b <= a; of an upper triangle those from the diagonal on
__host__ __device__ inline int band_columns(const GemmArgs& g, int band, int& first) {
  first = g.upper ? band * BAND : 0;
  if (g.mode != kIntegrals) return g.tn - first;
  const int m1 = (band + 1) * BAND * kTile, last = (m1 < g.M ? m1 : g.M) - 1;
  const long long cols = (long long)(g.lad.a0 + last / g.lad.n + 1 - g.lad.b0) * g.lad.n;  // b0 <= a0
  const long long t = (cols + kTile - 1) / kTile;
  return t < g.tn ? (int)t : g.tn;
}


// LDS row of a T-wide operand tile: T + pad = 18 (mod 32) doubles
constexpr int lds_row(int t) { return t + (18 - t % 32 + 32) % 32; }

// operand element r of thread tid: (row of the tile, k of the chunk).  KCONTIG: the
// operand's k runs contiguously in memory, lanes along k; else lanes along the rows.
template <bool KCONTIG, int T>
__device__ inline void stage_index(int e, int& row, int& k) {
  if (KCONTIG) {
    row = e / GK;
    k = e - row * GK;
  } else {
    k = e / T;
    row = e - k * T;
  }
}

typedef uint32_t u2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kRange = 0x80000000u;  // bytes a buffer load may reach past its chunk's base

// Four waves, 2 x 2; each owns BM x BN blocks of 16 x 16.  WIDE: the operands' rows are
// so far apart that a chunk spans more than the 2 GB of a buffer load's offsets.
template <bool TA, bool TB, bool WIDE>
__global__ __launch_bounds__(256, 2) void gemm_f64_kernel(GemmArgs g) {
  constexpr int BM = 2, BN = 2, TM = kTile, TN = kTile;
  constexpr int LA = lds_row(TM), LB = lds_row(TN);
  constexpr int PA = TM * GK / 256, PB = TN * GK / 256;
  __shared__ double As[2][GK][LA];
  __shared__ double Bs[2][GK][LB];
  // XCD-aware order: consecutive workgroups go round-robin to the 8 XCDs; remapped so
  // that each walks a contiguous range of (batch, split, tile), tiles in bands of 8
  // tile rows, and its resident workgroups share panels through its L2
  const int nblk = gridDim.x;
  int L = blockIdx.x;
  {
    const int x = L & 7, k = L >> 3, q = nblk >> 3, rem = nblk & 7;
    L = (x < rem) ? x * (q + 1) + k : rem * (q + 1) + (x - rem) * q + k;
  }
  const int per = g.per;
  const int outer = L / per, t = L - outer * per;
  const int b = outer / g.nsplit, split = outer - b * g.nsplit;
  int band = 0, tr = t, jt0 = 0;
  if (g.mode == kIntegrals || g.upper)
    for (int c; tr >= (c = BAND * band_columns(g, band, jt0)); ++band) tr -= c;
  else {
    band = t / (BAND * g.tn);
    tr = t - band * BAND * g.tn;
  }
  const int h = min(BAND, g.tm - band * BAND);
  const int jt = jt0 + tr / h, it = band * BAND + tr % h;
  const int m0 = it * TM, n0 = jt * TN;
  if (g.upper && m0 >= n0 + TN) return;  // workgroup-uniform, before any barrier
  if (g.mode == kIntegrals && g.lad.b0 + n0 / g.lad.n > g.lad.a0 + (min(m0 + TM, g.M) - 1) / g.lad.n) return;
  const double* A = g.A + b * g.sA;
  const double* Bm = g.B + b * g.sB;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wr = w >> 1, wc = w & 1, r16 = lane & 15, kq = lane >> 4;
  const int kbeg = split * g.kper * GK, kend = min(g.K, kbeg + g.kper * GK);

  // A: op(A)[m][k] is A[m][k] (k contiguous) or, transposed, A[k][m] (m contiguous)
  // B: op(B)[k][n] is B[k][n] (n contiguous) or, transposed, B[n][k] (k contiguous)
  double ra[2][PA], rb[2][PB];  // two chunks in flight
  // Loads go through buffer descriptors whose base is the chunk's (scalar arithmetic),
  // at byte offsets that stay the same from chunk to chunk: no vector instruction but the
  // load itself, which matters because the FP64 products hold the vector pipe.
  const double* At = TA ? A : A + (size_t)m0 * g.lda;
  const double* Bt = TB ? Bm + (size_t)n0 * g.ldb : Bm;
  constexpr int SA = 256 / TM, SB = 256 / TN;  // k step between a thread's elements (row-contiguous operands)
  int rowa, rowb, ka, kb;
  stage_index<!TA, TM>(tid, rowa, ka);
  stage_index<TB, TN>(tid, rowb, kb);
  uint32_t oa[TA ? 1 : PA], ob[TB ? PB : 1];
  if constexpr (!WIDE) {
#pragma unroll
    for (int r = 0; r < (TA ? 1 : PA); ++r)
      oa[r] = TA ? ((uint32_t)ka * g.lda + min(m0 + rowa, g.M - 1)) * 8u
                 : ((uint32_t)min(rowa + 16 * r, g.M - 1 - m0) * g.lda + ka) * 8u;
#pragma unroll
    for (int r = 0; r < (TB ? PB : 1); ++r)
      ob[r] = TB ? ((uint32_t)min(rowb + 16 * r, g.N - 1 - n0) * g.ldb + kb) * 8u
                 : ((uint32_t)kb * g.ldb + min(n0 + rowb, g.N - 1)) * 8u;
  }
  // whole chunk at k0
  auto load = [&](auto S, int k0) __attribute__((always_inline)) {
    if constexpr (WIDE) {
#pragma unroll
      for (int r = 0; r < PA; ++r)
        ra[S()][r] = TA ? At[(size_t)(k0 + ka + SA * r) * g.lda + min(m0 + rowa, g.M - 1)]
                   : At[(size_t)min(rowa + 16 * r, g.M - 1 - m0) * g.lda + k0 + ka];
#pragma unroll
      for (int r = 0; r < PB; ++r)
        rb[S()][r] = TB ? Bt[(size_t)min(rowb + 16 * r, g.N - 1 - n0) * g.ldb + k0 + kb]
                   : Bt[(size_t)(k0 + kb + SB * r) * g.ldb + min(n0 + rowb, g.N - 1)];
    } else {
      auto da = __builtin_amdgcn_make_buffer_rsrc((void*)(At + (TA ? (size_t)k0 * g.lda : (size_t)k0)), 0, kRange, 0x00020000);
      auto db = __builtin_amdgcn_make_buffer_rsrc((void*)(Bt + (TB ? (size_t)k0 : (size_t)k0 * g.ldb)), 0, kRange, 0x00020000);
#pragma unroll
      for (int r = 0; r < PA; ++r)
        ra[S()][r] = __builtin_bit_cast(double, (u2)__builtin_amdgcn_raw_buffer_load_b64(da, oa[TA ? 0 : r], TA ? SA * r * g.lda * 8 : 0, 0));
#pragma unroll
      for (int r = 0; r < PB; ++r)
        rb[S()][r] = __builtin_bit_cast(double, (u2)__builtin_amdgcn_raw_buffer_load_b64(db, ob[TB ? r : 0], TB ? 0 : SB * r * g.ldb * 8, 0));
    }
  };
  // the last `left` < GK steps of the contraction at k0; the others are zero
  auto load_tail = [&](int k0, int left) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < PA; ++r) {
      const int k = ka + (TA ? SA * r : 0), kk = k0 + min(k, left - 1);
      const double v = TA ? At[(size_t)kk * g.lda + min(m0 + rowa, g.M - 1)]
                          : At[(size_t)min(rowa + 16 * r, g.M - 1 - m0) * g.lda + kk];
      ra[0][r] = k < left ? v : 0.0;
    }
#pragma unroll
    for (int r = 0; r < PB; ++r) {
      const int k = kb + (TB ? 0 : SB * r), kk = k0 + min(k, left - 1);
      const double v = TB ? Bt[(size_t)min(rowb + 16 * r, g.N - 1 - n0) * g.ldb + kk]
                          : Bt[(size_t)kk * g.ldb + min(n0 + rowb, g.N - 1)];
      rb[0][r] = k < left ? v : 0.0;
    }
  };
  auto store = [&](auto S, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < PA; ++r) {
      int row, k;
      stage_index<!TA, TM>(tid + 256 * r, row, k);
      As[buf][k][row] = ra[S()][r];
    }
#pragma unroll
    for (int r = 0; r < PB; ++r) {
      int col, k;
      stage_index<TB, TN>(tid + 256 * r, col, k);
      Bs[buf][k][col] = rb[S()][r];
    }
  };

  d4 acc[BM][BN];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j) acc[i][j] = (d4){0.0, 0.0, 0.0, 0.0};

  auto products = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int k4 = 0; k4 < GK / 4; ++k4) {
      const int k = k4 * 4 + kq;
      double a[BM], bb[BN];
#pragma unroll
      for (int i = 0; i < BM; ++i) a[i] = As[buf][k][(wr * BM + i) * 16 + r16];
#pragma unroll
      for (int j = 0; j < BN; ++j) bb[j] = Bs[buf][k][(wc * BN + j) * 16 + r16];
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], bb[j], acc[i][j], 0, 0, 0);
    }
  };
  const int kfull = kbeg + (kend - kbeg) / GK * GK;
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  int buf = 0;
  if (kbeg < kfull) {  // loads two chunks ahead; past the end the last chunk again, not read
    const int last = kfull - GK;
    load(S0{}, kbeg);
    load(S1{}, min(kbeg + GK, last));
    store(S0{}, 0);
    __syncthreads();
    int k0 = kbeg;
    for (; k0 + GK < kfull; k0 += 2 * GK) {
      load(S0{}, min(k0 + 2 * GK, last));
      products(0);
      store(S1{}, 1);
      __syncthreads();
      load(S1{}, min(k0 + 3 * GK, last));
      products(1);
      store(S0{}, 0);
      __syncthreads();
    }
    if (k0 < kfull) {
      products(0);
      buf = 1;
    }
  }
  if (kfull < kend) {  // workgroup-uniform
    load_tail(kfull, kend - kfull);
    store(S0{}, buf);
    __syncthreads();
    products(buf);
  }
  // register r of lane l holds row l / 16 + 4 r and column l % 16 of a 16 x 16 block
  if (g.mode && !g.part) {
    const LadderBlock q = g.lad;
    int x[BN], y[BN];  // kIntegrals: b and d of the column; else a and b
#pragma unroll
    for (int j = 0; j < BN; ++j) {
      const int gn = n0 + (wc * BN + j) * 16 + r16;
      if (g.mode == kIntegrals) {
        const int bl = gn / q.n;
        y[j] = gn - bl * q.n;
        x[j] = gn < g.N ? q.b0 + bl : 0x7fffffff;
      } else {
        ladder_pair(q.a0 + min(gn, g.N - 1), x[j], y[j]);
      }
    }
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gm = m0 + (wr * BM + i) * 16 + kq + 4 * r;
        if (gm >= g.M) continue;
        const int a = q.a0 + gm / q.n, c = gm % q.n;
        double* row = g.mode == kIntegrals ? g.C + (q.first(a) * q.n + c) * q.n : g.C + (size_t)gm * q.n * q.n;
#pragma unroll
        for (int j = 0; j < BN; ++j) {
          const double v = acc[i][j][r];
          if (g.mode == kIntegrals) {
            if (x[j] <= a) row[(size_t)x[j] * q.n * q.n + y[j]] = v;
          } else if (n0 + (wc * BN + j) * 16 + r16 < g.N) {
            ladder_store(row, q.n, x[j], y[j], v, g.mode == kPlus);
          }
        }
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int gm = m0 + (wr * BM + i) * 16 + kq + 4 * r;
      if (gm >= g.M) continue;
      double* row = g.part ? g.part + (((size_t)split * g.batch + b) * g.M + gm) * g.N : c_row(g, b, gm);
#pragma unroll
      for (int j = 0; j < BN; ++j) {
        const int gn = n0 + (wc * BN + j) * 16 + r16;
        if (gn >= g.N) continue;
        double* dst = row + gn;
        double v = acc[i][j][r];
        if (!g.part) {
          v *= g.alpha;
          if (g.beta != 0.0) v += g.beta * *dst;
          if (g.orth) v = orth_value(v, gm, gn);
        }
        *dst = v;
      }
    }
}


// C = alpha sum over the splits of their partial products + beta C, in the order of
// the splits; with `upper`, the tiles wholly below the diagonal were not formed
__global__ __launch_bounds__(256) void gemm_f64_sum(GemmArgs g) {
  const size_t mn = (size_t)g.M * g.N, all = mn * g.batch;
  for (size_t q = blockIdx.x * (size_t)blockDim.x + threadIdx.x; q < all; q += (size_t)gridDim.x * blockDim.x) {
    const int b = (int)(q / mn);
    const size_t o = q - b * mn;
    const int m = (int)(o / g.N), n = (int)(o - (size_t)m * g.N);
    if (g.upper && m / kTile > n / kTile) continue;
    double v = 0.0;
    for (int k = 0; k < g.nsplit; ++k) v += g.part[((size_t)k * g.batch) * mn + q];
    if (g.mode) {
      int x, y;
      ladder_pair(g.lad.a0 + n, x, y);
      ladder_store(g.C + (size_t)m * g.lad.n * g.lad.n, g.lad.n, x, y, v, g.mode == kPlus);
      continue;
    }
    double* dst = c_row(g, b, m) + n;
    v *= g.alpha;
    if (g.beta != 0.0) v += g.beta * *dst;
    *dst = g.orth ? orth_value(v, m, n) : v;
  }
}

// Splits of the contraction by the estimated time on 256 compute units: the products done
// (padding included) by the busiest unit, at the share of the matrix rate that 1, 2, 3
// workgroups on a unit reach (LDS holds three; one alone has nothing to fill the waits at its
// barriers), plus the partial products' way through memory.  Measured shares 0.42, 0.61 and
// 0.78 (34 TFLOP/s at 361 workgroups, 62 at 16384): 1200^3 goes from 34 to 41 TFLOP/s split in
// two.  What is left after whole rounds runs at the lower shares: A B^T 400 x 8911 x 8911 (980
// tiles, three rounds of 256 and one alone on a unit) 43 TFLOP/s whole, 48 split in two.
int choose_split(int M, int N, int K, int batch, bool upper, size_t part_doubles) {
  constexpr int kFit = 3;
  constexpr double kRate[kFit] = {0.42, 0.61, 0.78};
  const double flop_us = 305e3;  // per unit at 78 TFLOP/s
  int best = 1;
  double best_t = 1e300;
  const int nchunk = (K + GK - 1) / GK;
  const double tm = (M + kTile - 1) / kTile, tn = (N + kTile - 1) / kTile;
  const double n = tm * tn * batch * (upper ? 0.5 * (1.0 + 1.0 / tn) : 1.0);
  for (int s = 1; s <= 64; ++s) {
    if (s > 1 && ((size_t)s * batch * M * N > part_doubles || nchunk < 8 * s)) break;
    const int per_unit = (int)std::min(std::ceil(n * s / 256.0), 1e8), rest = per_unit % kFit;
    // rounds of as many as fit, then the rest at the rate that fewer reach
    const double eff = (per_unit - rest) / kRate[kFit - 1] + (rest ? rest / kRate[rest - 1] : 0.0);
    const double us = eff * 2.0 * kTile * kTile * GK * std::ceil((double)nchunk / s) / flop_us +
                      (s > 1 ? 5.0 + (double)s * batch * M * N * 16.0 / 4e6 : 0.0);
    if (us < best_t * 0.999) {
      best_t = us;
      best = s;
    }
  }
  return best;
}

template <bool WIDE>
void launch_kernel(const GemmArgs& g, int transA, int transB, unsigned blocks, hipStream_t st) {
  if (transA) {
    if (transB) hipLaunchKernelGGL((gemm_f64_kernel<true, true, WIDE>), dim3(blocks), dim3(256), 0, st, g);
    else hipLaunchKernelGGL((gemm_f64_kernel<true, false, WIDE>), dim3(blocks), dim3(256), 0, st, g);
  } else {
    if (transB) hipLaunchKernelGGL((gemm_f64_kernel<false, true, WIDE>), dim3(blocks), dim3(256), 0, st, g);
    else hipLaunchKernelGGL((gemm_f64_kernel<false, false, WIDE>), dim3(blocks), dim3(256), 0, st, g);
  }
}

hipError_t launch_gemm(GemmArgs& g, int transA, int transB, double* part, size_t part_doubles, hipStream_t st) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
  const int nsplit = choose_split(g.M, g.N, g.K, g.batch, g.upper != 0, part ? part_doubles : 0);
  // byte span of a chunk: 16 rows of an operand whose tile rows run contiguously, up to
  // 64 rows of a k-contiguous one
  const bool wide = ((transA ? 16.0 : 64.0) * g.lda + 64.0) * 8.0 >= kRange ||
                    ((transB ? 64.0 : 16.0) * g.ldb + 64.0) * 8.0 >= kRange;
  g.tm = (g.M + kTile - 1) / kTile;
  g.tn = (g.N + kTile - 1) / kTile;
  const int nchunk = g.K > 0 ? (g.K + GK - 1) / GK : 0;  // K <= 0 leaves C = beta C
  g.kper = (nchunk + nsplit - 1) / nsplit;
  g.nsplit = g.kper > 0 ? (nchunk + g.kper - 1) / g.kper : 1;
  g.part = g.nsplit > 1 ? part : nullptr;
  double per = 0.0;
  if (g.mode == kIntegrals || g.upper)
    for (int band = 0, first; band * BAND < g.tm; ++band)
      per += (double)std::min(BAND, g.tm - band * BAND) * band_columns(g, band, first);
  else per = (double)g.tm * g.tn;
  const double blocks = per * g.batch * g.nsplit;
  if (blocks > 2147483647.0) return hipErrorInvalidValue;
  const unsigned nb = (unsigned)blocks;
  g.per = (int)per;
  if (wide) launch_kernel<true>(g, transA, transB, nb, st);
  else launch_kernel<false>(g, transA, transB, nb, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || g.nsplit <= 1) return e;
  const size_t all = ((size_t)g.M * g.N * g.batch + 255) / 256;
  hipLaunchKernelGGL(gemm_f64_sum, dim3((unsigned)(all < 16384 ? all : 16384)), dim3(256), 0, st, g);
  return hipGetLastError();
}

}  // namespace

hipError_t gemm_f64(const double* A, int lda, long long sA, int transA, const double* B, int ldb, long long sB,
                    int transB, double* C, int ldc, long long sC, int M, int N, int K, int batch, double alpha,
                    double beta, hipStream_t st, double* part, size_t part_doubles, bool upper,
                    int row_n, long long row_s) {
  GemmArgs g{};
  g.A = A;
  g.B = B;
  g.C = C;
  g.M = M;
  g.N = N;
  g.K = K;
  g.lda = lda;
  g.ldb = ldb;
  g.ldc = ldc;
  g.sA = sA;
  g.sB = sB;
  g.sC = sC;
  g.alpha = alpha;
  g.beta = beta;
  g.batch = batch;
  g.upper = upper ? 1 : 0;
  g.row_n = row_n > 0 ? row_n : (M > 0 ? M : 1);
  g.row_s = row_s;
  return launch_gemm(g, transA, transB, part, part_doubles, st);
}

hipError_t gemm_f64_orth(const double* X, int n, double* M, double* part, size_t part_doubles, hipStream_t st) {
  GemmArgs g{};
  g.A = g.B = X;
  g.C = M;
  g.M = g.N = g.K = g.lda = g.ldb = g.ldc = g.row_n = n;
  g.alpha = 1.0;
  g.batch = 1;
  g.orth = 1;
  return launch_gemm(g, 1, 0, part, part_doubles, st);
}

hipError_t ladder_integrals(const double* Bk, int n_aux, const LadderBlock& q, double* V, hipStream_t st) {
  GemmArgs g{};
  g.A = Bk + (size_t)q.a0 * q.n * n_aux;
  g.B = Bk + (size_t)q.b0 * q.n * n_aux;
  g.C = V;
  g.M = (q.a1 - q.a0) * q.n;
  g.N = (q.b1 - q.b0) * q.n;
  g.K = n_aux;
  g.lda = g.ldb = n_aux;
  g.alpha = 1.0;
  g.batch = 1;
  g.mode = kIntegrals;
  g.lad = q;
  return launch_gemm(g, 0, 1, nullptr, 0, st);
}

hipError_t ladder_contract(const double* T, const double* G, int n_amp, int K, int n, int t0, int count, bool plus,
                           double* R, double* part, size_t part_doubles, hipStream_t st) {
  GemmArgs g{};
  g.A = T;
  g.B = G;
  g.C = R;
  g.M = n_amp;
  g.N = count;
  g.K = K;
  g.lda = g.ldb = K;
  g.alpha = 1.0;
  g.batch = 1;
  g.mode = plus ? kPlus : kMinus;
  g.lad.n = n;
  g.lad.a0 = t0;
  return launch_gemm(g, 0, 1, part, part_doubles, st);
}

}  // namespace dfpt2
