// FP64 density kernel: the virtual block of the second-order 1-RDM (Eq. A9)
// accumulated over hole pairs on FP64 MFMA.
//
// For an unordered pair {i < j} with amplitude matrix T = T^{ij} the two
// ordered pairs contribute T (2T - T^T)^T + T^T (2T - T^T).  With the symmetric and
// antisymmetric parts T = S + A this is 2 S S^T + 6 A A^T: two products of one operand
// each with itself.  With a virtual c running along the contraction and
//     s[a][c] = T[a][c] + T[c][a],   d[a][c] = T[a][c] - T[c][a]
// it is 1/2 s s^T + 3/2 d d^T.  For i == j (T symmetric, d = 0) the same expression gets
// half the weight and the second product is skipped.  The result is symmetric, so only
// tiles (A <= B) of D are formed.
//
// Workgroup = (tile pair (A, B), split s).  Split s owns a contiguous range of
// pairs and accumulates into its own slice Dpart[s]; slices are summed in a
// fixed order afterwards, so results are bitwise reproducible.  Per 16-deep chunk the four
// operand panels (rows A and B of T, and of T^T, i.e. columns A and B) are staged through
// LDS; s and d are formed from two fragments as they are read, the first ones times the
// pair's weight, so that one set of accumulators takes all pairs.
// As in the FP64 pair kernel: buffer loads one chunk ahead at constant offsets, XOR-swizzled
// LDS panels, the 16 x 16 blocks beyond n_v skipped, no branch in the loop over the chunks
// of a pair; each XCD walks a contiguous range of (split, tile pair).
//
// What bounds it: the matrix pipe at the clock that it leaves (about 2 GHz), with 20% of
// the products' time lost where the last tile row is narrow and in the last round.
// 40 cores + 8 active, 400 virtuals, ms per pass: 4.5, 4.8 with the narrow tile pairs among the
// others, 5.1 before (the operands 2T - T^T
// formed with weights in the loop, whole tiles, predicated loads).  Without any load in
// the loop 4.2; chunks of 8 with three or four workgroups per unit, and 27 or 54 splits
// (whole rounds) instead of 64: no faster.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace dfpt2 {

namespace {
constexpr int TM = 64;
constexpr int KC = 16;
constexpr int PANEL = KC * TM;
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// place of (k, row) in a panel (pair_f64.hip)
__device__ inline int slot(int k, int row) { return k * TM + (row ^ (((k & 1) << 4) | ((k >> 1) << 1))); }
}  // namespace

__global__ __launch_bounds__(256, 2) void density_f64_kernel(DensityKernelArgs a) {
  __shared__ double lds[2][4][PANEL];  // T[A, c..], T[B, c..], T[c.., A], T[c.., B]
  // Each XCD walks a contiguous range of (split, tile pair); tile pairs with at most 16 columns,
  // which take half as long, come after the others of all splits (pair_f64.hip)
  int split, A, Bt;
  {
    const int edge = a.n_v - (a.nt - 1) * TM, nf = edge <= 16 ? a.nt - 1 : a.nt;
    const uint32_t full = nf * (nf + 1) / 2, rest = a.nTP - full, all = full * gridDim.y;
    const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x;
    auto xcd = [](uint32_t h, uint32_t nblk) {
      const uint32_t x = h & 7, k = h >> 3, q = nblk >> 3, rem = nblk & 7;
      return (x < rem) ? x * (q + 1) + k : rem * (q + 1) + (x - rem) * q + k;
    };
    if (id < all) {
      const uint32_t L = xcd(id, all);
      split = (int)(L / full);
      tile_pair((int)(L - split * full), nf, A, Bt);
    } else {
      const uint32_t L = xcd(id - all, rest * gridDim.y);
      split = (int)(L / rest);
      A = (int)(L - split * rest);
      Bt = a.nt - 1;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 1, wc = w & 1, r16 = lane & 15, kq = lane >> 4;
  const int n_v = a.n_v;
  const int p0 = (int)((int64_t)split * a.n_pairs / a.nsplit);
  const int p1 = (int)((int64_t)(split + 1) * a.n_pairs / a.nsplit);
  const int ncc = (n_v + KC - 1) / KC, tail = n_v - (ncc - 1) * KC;  // columns of the last chunk
  const int blk[2] = {A, Bt};

  // row panels: column ka of the chunk, rows lr + 16 h; column panels: row kc + 4 h of the
  // chunk, column cc of the block
  const int ka = tid & 15, lr = tid >> 4, cc = lane, kc = tid >> 6;
  uint32_t orow[2][4], ocol[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
#pragma unroll
    for (int h = 0; h < 4; ++h) orow[q][h] = ((uint32_t)min(lr + 16 * h, n_v - 1 - blk[q] * TM) * n_v + ka) * 8u;
    ocol[q] = ((uint32_t)kc * n_v + min(blk[q] * TM + cc, n_v - 1)) * 8u;
  }
  auto matrix = [&](int p) { return a.T + (size_t)(a.slot ? a.slot[p] : p) * n_v * n_v; };
  const uint32_t out = ka >= tail ? 0x80000000u : 0u;  // of range in the last chunk: reads zero
  auto load = [&](double (&st)[4][4], const double* Tp, int ci) __attribute__((always_inline)) {
    const uint32_t mask = ci == ncc - 1 ? out : 0u;
    // the rows left below the chunk's first bound the column panels
    const uint64_t left = (uint64_t)(n_v - ci * KC) * n_v * 8;
    auto dc = __builtin_amdgcn_make_buffer_rsrc((void*)(Tp + (size_t)ci * KC * n_v), 0,
                                                (uint32_t)(left < 0x7fffffff ? left : 0x7fffffff), 0x00020000);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      auto dr = __builtin_amdgcn_make_buffer_rsrc((void*)(Tp + (size_t)blk[q] * TM * n_v + ci * KC), 0, 0x7fffffff, 0x00020000);
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        st[q][h] = __builtin_bit_cast(double, (u2)__builtin_amdgcn_raw_buffer_load_b64(dr, orow[q][h] | mask, 0, 0));
        st[2 + q][h] =
            __builtin_bit_cast(double, (u2)__builtin_amdgcn_raw_buffer_load_b64(dc, ocol[q], 4 * h * n_v * 8, 0));
      }
    }
  };
  auto store = [&](double (&st)[4][4], int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        lds[buf][q][slot(ka, lr + 16 * h)] = st[q][h];
        lds[buf][2 + q][slot(kc + 4 * h, cc)] = st[2 + q][h];
      }
  };

  const int nbi = min(2, max(0, (n_v - A * TM - wr * 32 + 15) / 16)), nbj = min(2, max(0, (n_v - Bt * TM - wc * 32 + 15) / 16));
  d4 D[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) D[x][y] = (d4){0.0, 0.0, 0.0, 0.0};

  auto run = [&](auto NI, auto NJ) __attribute__((always_inline)) {
    double st[4][4];
    // chunk `ci` of pair `p`, its products from buffer BUF; ANTI: also d d^T
    auto products = [&](int buf, auto ANTI, double ws, double wx) __attribute__((always_inline)) {
#pragma unroll
      for (int k4 = 0; k4 < KC / 4; ++k4) {
        const int k = k4 * 4 + kq;
        double sa[2], da[2], sb[2], db[2];
#pragma unroll
        for (int b = 0; b < NI(); ++b) {
          const int o = slot(k, wr * 32 + b * 16 + r16);
          const double x1 = lds[buf][0][o], x2 = lds[buf][2][o];
          sa[b] = (x1 + x2) * ws;
          da[b] = (x1 - x2) * wx;
        }
#pragma unroll
        for (int b = 0; b < NJ(); ++b) {
          const int o = slot(k, wc * 32 + b * 16 + r16);
          const double x1 = lds[buf][1][o], x2 = lds[buf][3][o];
          sb[b] = x1 + x2;
          db[b] = x1 - x2;
        }
#pragma unroll
        for (int bi = 0; bi < NI(); ++bi)
#pragma unroll
          for (int bj = 0; bj < NJ(); ++bj) {
            D[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[bi], sb[bj], D[bi][bj], 0, 0, 0);
          }
        if (ANTI()) {
#pragma unroll
          for (int bi = 0; bi < NI(); ++bi)
#pragma unroll
            for (int bj = 0; bj < NJ(); ++bj)
              D[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(da[bi], db[bj], D[bi][bj], 0, 0, 0);
        }
      }
    };
    // the chunks of all pairs are one sequence whose loads run one ahead of the products
    // (at the end the last pair's first chunk is loaded once more, and not read)
    const double *Tp = matrix(p0), *Tn;
    int buf = 0;
    load(st, Tp, 0);
    store(st, 0);
    __syncthreads();
    for (int p = p0; p < p1; ++p, Tp = Tn) {
      const int2 pr = a.pairs[p];
      Tn = matrix(min(p + 1, p1 - 1));
      const double wp = a.w * (pr.x == pr.y ? 0.5 : 1.0) * (a.pw ? a.pw[p] : 1.0);
      const double ws = 0.5 * wp, wx = 1.5 * wp;
      auto chunks = [&](auto ANTI) __attribute__((always_inline)) {
        for (int c = 1; c <= ncc; ++c) {
          const bool last = c == ncc;
          load(st, last ? Tn : Tp, last ? 0 : c);
          products(buf, ANTI, ws, wx);
          store(st, buf ^= 1);
          __syncthreads();
        }
      };
      if (pr.x == pr.y) chunks(std::false_type{});
      else chunks(std::true_type{});
    }
  };
  using N0 = std::integral_constant<int, 0>;
  using N1 = std::integral_constant<int, 1>;
  using N2 = std::integral_constant<int, 2>;
  if (p0 < p1) {  // workgroup-uniform; the instances have the same loads and barriers
    if (nbi == 0 || nbj == 0) run(N0{}, N0{});
    else if (nbi == 1) nbj == 1 ? run(N1{}, N1{}) : run(N1{}, N2{});
    else nbj == 1 ? run(N2{}, N1{}) : run(N2{}, N2{});
  }

  double* Dp = a.Dpart + (size_t)split * n_v * n_v;
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ga = A * TM + wr * 32 + bi * 16 + kq + 4 * r;
      if (ga >= n_v) continue;
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const int gb = Bt * TM + wc * 32 + bj * 16 + r16;
        if (gb >= n_v) continue;
        double* dst = Dp + (size_t)ga * n_v + gb;
        *dst = a.accumulate ? *dst + D[bi][bj][r] : D[bi][bj][r];
      }
    }
}

// Sum of the slices: 64 columns of a row and 4 shares of the slices per workgroup, so that a
// thread's chain of dependent additions is a quarter of them (60 virtuals, 55 slices: 14 us
// with one thread per element, its loads one after the other).
__global__ __launch_bounds__(256) void density_reduce_kernel(const double* Dpart, int nsplit, int n_v, const double* diag,
                                                             double* D) {
  __shared__ double sh[3][64];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int b = blockIdx.x * 64 + lane, a = blockIdx.y;
  if (a > (int)blockIdx.x * 64 + 63) return;  // below the diagonal
  const size_t off = (size_t)a * n_v + min(b, n_v - 1), stride = (size_t)n_v * n_v;
  double v = 0.0;
#pragma unroll 8
  for (int s = g; s < nsplit; s += 4) v += Dpart[off + s * stride];
  if (g > 0) sh[g - 1][lane] = v;
  __syncthreads();
  if (g > 0 || b >= n_v || a > b) return;
  v = (v + sh[0][lane]) + (sh[1][lane] + sh[2][lane]);
  if (diag && a == b) v += diag[a];
  D[off] = v;
  D[(size_t)b * n_v + a] = v;
}

hipError_t launch_density_f64(const DensityKernelArgs& a, hipStream_t st) {
  if (a.n_pairs <= 0) return hipSuccess;
  dim3 grid(a.nTP, a.nsplit), block(256);
  hipLaunchKernelGGL(density_f64_kernel, grid, block, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_density_reduce(const double* Dpart, int nsplit, int n_v, const double* diag, double* D,
                                 hipStream_t st) {
  dim3 block(256), grid((n_v + 63) / 64, n_v);
  hipLaunchKernelGGL(density_reduce_kernel, grid, block, 0, st, Dpart, nsplit, n_v, diag, D);
  return hipGetLastError();
}

}  // namespace dfpt2
