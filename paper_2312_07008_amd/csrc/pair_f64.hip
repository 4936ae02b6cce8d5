// FP64 pair kernel: V = B_i B_j^T on FP64 MFMA with the DSRG regularizer and
// the PT2 energy fused into the epilogue (paper App. A, Eq. A7).
//
// One workgroup owns an unordered hole pair {i <= j} and a 64 x 64 tile pair
// (I <= J) of virtual row/column blocks.  It computes, in the same register
// layout,
//     P = V^{ij}[I, J] = B_i[I] B_j[J]^T      and     Q = V^{ji}[I, J] = B_j[I] B_i[J]^T,
// so that element (a, b) of Q is V^{ij}_{ba}: the exchange partner needed by
// 2 t^{ij}_{ab} - t^{ij}_{ba} sits in the same lane and register as P_ab.
// For i == j the integrals are symmetric, Q = P and the second product is skipped.
//
// Epilogue, per element (a in I, b in J):
//   Delta = eps_i + eps_j - eps_a - eps_b,  x = exp(-s Delta^2)
//   T_P = P (1 - x)/Delta,  T_Q = Q (1 - x)/Delta             (Eq. A7)
//   energy  += w (1 - x^2)/Delta (2 P^2 + 2 Q^2 - 2 P Q)       (both ordered pairs)
//   ||T||^2 += T_P^2 (+ T_Q^2 off the diagonal tile)
// and the amplitudes of the unordered pair are stored as the full matrix
// T^{ij}: T_P at [a][b] and, for I < J, T_Q at the mirrored position [b][a]
// (T^{ij}_{ba} = T^{ji}_{ab}).  Optionally the renormalized integrals
// Vr = V (1 + x) are stored the same way (used when active holes are rotated).
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace dfpt2 {

namespace {
constexpr int TM = 64;        // tile edge
constexpr int KC = 16;        // aux chunk per pipeline stage
constexpr int PANEL = KC * TM;
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// place of (k, row) in a panel, k-major: the row is XOR-swizzled by the bits of k so that
// the 16 lanes along k of a store (times two rows) and the 16 + 16 lanes of a fragment
// read (rows of one block, k and k + 1) hit distinct banks without padding
__device__ inline int slot(int k, int row) { return k * TM + (row ^ (((k & 1) << 4) | ((k >> 1) << 1))); }
}  // namespace

// What bounds it: the FP64 matrix pipe (64 cycles a product, 78 TFLOP/s), as long as
// nothing else holds the SIMD.  Per 16-deep chunk a wave has 16 products of a 32 x 32
// quadrant, 16 fragment reads, 8 loads and 8 LDS stores:
//  * P and Q are formed one after the other, so that two panels in two LDS buffers are
//    32 KB and three workgroups share a unit: the others fill one's waits at its barriers
//    (both at once, four panels, two workgroups: 14.1 instead of 12.4 ms).
//  * loads are 8-byte buffer loads (any n_aux) at byte offsets that never change, from
//    descriptors whose base moves with the chunk; they run two chunks ahead in two register
//    stages, so that a launch with one workgroup per unit (a small molecule) is not paced
//    by the memory's latency.  Rows beyond n_v read a clamped row and reach no stored
//    element; the partial chunk of the contraction comes first, outside the loop, with its
//    missing columns read out of the descriptor's range, as zeros.
//  * the products of 16 x 16 blocks that lie wholly beyond n_v are skipped (wave-uniform).
//  * on a diagonal tile Q is P^T, exchanged through LDS instead of computed again.
// 40 cores + 8 active, 400 virtuals, 1600 auxiliary functions, ms per pass: 11.6, 18.0 before
// (predicated 16-byte loads one chunk ahead, padded LDS rows, whole tiles computed).
//
// STORE = false: energy-only variant (kept-space pass) that writes no amplitudes.
// WIDE: rows so long that a panel spans more than the 2 GB of a buffer load's offsets.
template <bool STORE, bool WIDE>
__global__ __launch_bounds__(256, 3) void pair_gemm_f64_kernel(PairKernelArgs a) {
  __shared__ double lds[2][2][PANEL];
  __shared__ double red[2][4];
  // Each XCD walks a contiguous range of (pair, tile pair); the tile pairs I < J, which take
  // two products, of all pairs first, then those of half their length (on the diagonal, or with
  // at most 16 columns): workgroups that keep step find the panels that they share in the L2
  // (size above: 72 -> 50% of the requests miss, 12.5 -> 11.6 ms per pass).
  int p, I, J;
  {
    const int edge = a.n_v - (a.nt - 1) * TM, nf = edge <= 16 ? a.nt - 1 : a.nt;
    const int full = nf * (nf - 1) / 2, rest = a.nTP - full;
    const uint64_t np = gridDim.y, all = np * full, id = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    auto xcd = [](uint64_t h, uint64_t nblk) {
      const uint64_t x = h & 7, k = h >> 3, q = nblk >> 3, rem = nblk & 7;
      return (x < rem) ? x * (q + 1) + k : rem * (q + 1) + (x - rem) * q + k;
    };
    if (id < all) {
      const uint64_t L = xcd(id, all);
      p = (int)(L / full);
      tile_pair((int)(L - (uint64_t)p * full), nf - 1, I, J);
      ++J;
    } else {
      const uint64_t L = xcd(id - all, np * rest);
      p = (int)(L / rest);
      const int t = (int)(L - (uint64_t)p * rest);
      I = t < a.nt ? t : t - a.nt;
      J = t < a.nt ? t : a.nt - 1;
    }
  }
  const int tp = I * a.nt - I * (I - 1) / 2 + J - I;  // place of the tile pair's partial sums
  const int2 pr = a.pairs[p];
  const int hi_i = pr.x, hi_j = pr.y;
  const bool same = (hi_i == hi_j), two = !same && I != J;  // two: Q is a product of its own
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 1, wc = w & 1;
  const int n_v = a.n_v, n_aux = a.n_aux;
  const int r16 = lane & 15, kq = lane >> 4;

  // thread: column ka of the chunk, rows lr + 16 h of a panel
  const int ka = tid & 15, lr = tid >> 4;
  typename std::conditional<WIDE, uint64_t, uint32_t>::type off[2][4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    off[0][h] = ((decltype(off[0][0] + 0))min(lr + 16 * h, n_v - 1 - I * TM) * n_aux + ka) * 8u;
    off[1][h] = ((decltype(off[0][0] + 0))min(lr + 16 * h, n_v - 1 - J * TM) * n_aux + ka) * 8u;
  }
  // 16 x 16 blocks of this wave that reach into n_v
  const int nbi = min(2, max(0, (n_v - I * TM - wr * 32 + 15) / 16)), nbj = min(2, max(0, (n_v - J * TM - wc * 32 + 15) / 16));
  const int nfull = n_aux / KC, tail = n_aux - nfull * KC, n = nfull + (tail ? 1 : 0);
  auto chunk_at = [&](int i) { return (tail ? i - 1 : i) * KC; };  // i > 0, or no tail

  // acc = rows I of hole x times rows J of hole y, over all auxiliary functions, for the
  // first NI x NJ blocks of the wave: no branch in the loop, whose merges would copy the
  // accumulators and wait for the products in flight (the whole pass of the size above 17.9 ms, 19.8 with a branch).
  // Waves of a workgroup may run different instances: the same loads, stores and barriers.
  auto contract = [&](auto NI, auto NJ, d4 (&acc)[2][2], int x, int y) __attribute__((always_inline)) {
    const double* base[2] = {a.B + ((size_t)x * n_v + (size_t)I * TM) * n_aux,
                             a.B + ((size_t)y * n_v + (size_t)J * TM) * n_aux};
    // chunk at k0 into a register stage; `mask` is or'ed into the offsets (out of range: zero)
    auto load = [&](double (&st)[2][4], int k0, uint32_t mask) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if constexpr (WIDE) {
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            const char* src = reinterpret_cast<const char*>(base[q] + k0) + off[q][h];
            st[q][h] = mask ? 0.0 : *reinterpret_cast<const double*>(src);
          }
        } else {
          auto desc = __builtin_amdgcn_make_buffer_rsrc((void*)(base[q] + k0), 0, 0x7fffffff, 0x00020000);
#pragma unroll
          for (int h = 0; h < 4; ++h)
            st[q][h] = __builtin_bit_cast(
                double, (u2)__builtin_amdgcn_raw_buffer_load_b64(desc, (uint32_t)off[q][h] | mask, 0, 0));
        }
      }
    };
    auto store = [&](double (&st)[2][4], int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int h = 0; h < 4; ++h) lds[buf][q][slot(ka, lr + 16 * h)] = st[q][h];
    };
    auto products = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int k4 = 0; k4 < KC / 4; ++k4) {
        const int k = k4 * 4 + kq;
        double u[2], v[2];
#pragma unroll
        for (int b = 0; b < NI(); ++b) u[b] = lds[buf][0][slot(k, wr * 32 + b * 16 + r16)];
#pragma unroll
        for (int b = 0; b < NJ(); ++b) v[b] = lds[buf][1][slot(k, wc * 32 + b * 16 + r16)];
#pragma unroll
        for (int bi = 0; bi < NI(); ++bi)
#pragma unroll
          for (int bj = 0; bj < NJ(); ++bj)
            acc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[bi], v[bj], acc[bi][bj], 0, 0, 0);
      }
    };
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) acc[bi][bj] = (d4){0.0, 0.0, 0.0, 0.0};
    double s0[2][4], s1[2][4];
    if (tail) load(s0, nfull * KC, ka < tail ? 0u : 0x80000000u);
    else load(s0, 0, 0u);
    if (n > 1) load(s1, chunk_at(1), 0u);
    __syncthreads();  // the readers of an earlier contraction are done
    store(s0, 0);
    __syncthreads();
    for (int i = 0; i + 1 < n; i += 2) {
      load(s0, chunk_at(min(i + 2, n - 1)), 0u);
      products(0);
      store(s1, 1);
      __syncthreads();
      load(s1, chunk_at(min(i + 3, n - 1)), 0u);
      products(1);
      store(s0, 0);
      __syncthreads();
    }
    if (n & 1) products(0);
  };
  d4 P[2][2], Q[2][2];
  auto both = [&](auto NI, auto NJ) __attribute__((always_inline)) {
    contract(NI, NJ, P, hi_i, hi_j);
    if (two) contract(NI, NJ, Q, hi_j, hi_i);
  };
  using N0 = std::integral_constant<int, 0>;
  using N1 = std::integral_constant<int, 1>;
  using N2 = std::integral_constant<int, 2>;
  if (nbi == 0 || nbj == 0) both(N0{}, N0{});
  else if (nbi == 1) nbj == 1 ? both(N1{}, N1{}) : both(N1{}, N2{});
  else nbj == 1 ? both(N2{}, N1{}) : both(N2{}, N2{});
  if (same) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) Q[x][y] = P[x][y];
  } else if (!two) {  // diagonal tile: Q = P^T through LDS (columns XOR-swizzled by the row)
    __syncthreads();
    double* ex = &lds[0][0][0];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = wr * 32 + bi * 16 + kq + 4 * r;
          ex[row * TM + ((wc * 32 + bj * 16 + r16) ^ (row & 31))] = P[bi][bj][r];
        }
    __syncthreads();
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = wc * 32 + bj * 16 + r16;
          Q[bi][bj][r] = ex[row * TM + ((wr * 32 + bi * 16 + kq + 4 * r) ^ (row & 31))];
        }
  }

  // ---- epilogue
  const double ei = a.eps_h[hi_i], ej = a.eps_h[hi_j];
  const double eij = ei + ej;
  const double s = a.s;
  const bool offdiag = (I < J);
  const double blk_w = (offdiag ? 2.0 : 1.0) * (same ? 0.5 : 1.0) * a.e_weight;
  double* Tp = (STORE && a.T) ? a.T + (size_t)p * n_v * n_v : nullptr;
  double* Vp = (STORE && a.Vr) ? a.Vr + (size_t)p * n_v * n_v : nullptr;
  double esum = 0.0, tsum = 0.0;
#pragma unroll
  for (int bi = 0; bi < 2; ++bi) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ga = I * TM + wr * 32 + bi * 16 + kq + 4 * r;
      const bool va = ga < n_v;
      const double ea = va ? a.eps_v[ga] : 0.0;
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const int gb = J * TM + wc * 32 + bj * 16 + r16;
        const bool vb = gb < n_v;
        if (!(va && vb)) continue;
        const double eb = a.eps_v[gb];
        const double dl = eij - ea - eb;
        const double x = exp(-s * dl * dl);
        const double g1 = (dl != 0.0) ? (1.0 - x) / dl : 0.0;
        const double vp = P[bi][bj][r], vq = Q[bi][bj][r];
        const double tp_ = vp * g1, tq_ = vq * g1;
        esum += (1.0 + x) * g1 * (2.0 * vp * vp + 2.0 * vq * vq - 2.0 * vp * vq);
        tsum += tp_ * tp_ + (offdiag ? tq_ * tq_ : 0.0);
        if (STORE && Tp) {
          Tp[(size_t)ga * n_v + gb] = tp_;
          if (offdiag) Tp[(size_t)gb * n_v + ga] = tq_;
        }
        if (STORE && Vp) {
          Vp[(size_t)ga * n_v + gb] = vp * (1.0 + x);
          if (offdiag) Vp[(size_t)gb * n_v + ga] = vq * (1.0 + x);
        }
      }
    }
  }
  esum = wave_sum(esum);
  tsum = wave_sum(tsum);
  if (lane == 0) {
    red[0][w] = esum;
    red[1][w] = tsum;
  }
  __syncthreads();
  if (tid == 0) {
    const size_t o = (size_t)p * a.nTP + tp;
    if (a.epart) a.epart[o] = blk_w * ((red[0][0] + red[0][1]) + (red[0][2] + red[0][3]));
    if (a.tpart) a.tpart[o] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

hipError_t launch_pair_gemm_f64(const PairKernelArgs& a, int n_pairs, hipStream_t st) {
  if (n_pairs <= 0) return hipSuccess;
  const dim3 grid(a.nTP, n_pairs), block(256);
  const bool store = a.T != nullptr || a.Vr != nullptr;
  if ((double)TM * a.n_aux * 8.0 >= 2147483647.0) {
    if (store) hipLaunchKernelGGL((pair_gemm_f64_kernel<true, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((pair_gemm_f64_kernel<false, true>), grid, block, 0, st, a);
  } else {
    if (store) hipLaunchKernelGGL((pair_gemm_f64_kernel<true, false>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((pair_gemm_f64_kernel<false, false>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace dfpt2
