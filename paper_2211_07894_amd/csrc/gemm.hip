// Matrix-core contractions of the hot path (FP64 form: v_mfma_f64_16x16x4f64).
//
//  tn_sym   H[b] = A^T diag(w_b) A over the grid index (K = M, long), for the
//           projected perturbation Hbreve' = Psi^T H' Psi of Eq. (21) and for Gram
//           matrices in Rayleigh-Ritz.  Only upper 128x128 tiles are computed;
//           split-K partials go to workspace and are summed in a fixed order.
//  backproj out[p] = scale sum_ij A_ip G_ij A_jp, the density of a symmetric
//           subspace matrix (Eqs. (16), (20)); Z = G A never leaves the chip:
//           each block owns 128 grid points and walks the upper block triangle.
//  nn       Out = Wt^T B (K = N, short), the rotations Psi_o = L^{-1} Y and
//           Psi_R = Q^T Psi_o of Rayleigh-Ritz.
//
// Blocks are "state-major" [N][M] arrays, so every operand streams contiguous
// grid points.  Lane layout of v_mfma_f64_16x16x4f64 (measured on gfx950):
//   A operand: lane l supplies A[l%16][l/16]   (row, k)
//   B operand: lane l supplies B[l/16][l%16]   (k, col)
//   D: lane l, register v holds D[4v + l/16][l%16].
#include <algorithm>
#include <type_traits>

#include "blocks.h"
#include "lrdm_internal.h"
#include "xcd.h"

namespace lrdm {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int BT = 128;   // output tile (rows and columns)
constexpr int KT = 32;    // k extent staged in LDS per step
constexpr int LDP = BT + 1;  // LDS row pitch in doubles

__device__ inline d4 mfma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// V consecutive elements of storage type S from a 16-byte aligned address.
template <int V>
__device__ inline void load_run(const double* src, double (&v)[V]) {
  const double2* s2 = reinterpret_cast<const double2*>(src);
#pragma unroll
  for (int q = 0; q < V / 2; ++q) {
    const double2 x = s2[q];
    v[2 * q] = x.x;
    v[2 * q + 1] = x.y;
  }
}
template <int V>
__device__ inline void load_run(const float* src, float (&v)[V]) {
  const float4* s4 = reinterpret_cast<const float4*>(src);
#pragma unroll
  for (int q = 0; q < V / 4; ++q) {
    const float4 x = s4[q];
    v[4 * q] = x.x;
    v[4 * q + 1] = x.y;
    v[4 * q + 2] = x.z;
    v[4 * q + 3] = x.w;
  }
}

// Stage rows [r0, r0+T) x cols [k0, k0+KT) of a row-major [nrows][ld] array of
// storage type S (double or float; the arithmetic is FP64 either way) into
// S[k][row] (transposed).  Each of 256 threads loads T / 8 consecutive k of one row.
// Out-of-range elements are zero.  load() only issues the reads, so they stay in
// flight during the current K-tile's matrix-core work.
template <typename S, int T>
struct TileLoad {
  static constexpr int V = T / 8, PER = KT / V;   // PER threads a row
  S v[V];
  __device__ inline void load(const S* __restrict__ X, int64_t ld, int nrows, int r0,
                              int64_t k0, int64_t kend) {
    const int t = threadIdx.x;
    const int row = t / PER;
    const int64_t kb = k0 + t % PER * V;
    const int gr = r0 + row;
    const bool aligned = (reinterpret_cast<uintptr_t>(X + (int64_t)gr * ld + kb) & 15) == 0;
    if (gr < nrows && kb + V <= kend && aligned) {
      load_run<V>(X + (int64_t)gr * ld + kb, v);
    } else {
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const int64_t k = kb + q;
        v[q] = (gr < nrows && k < kend) ? X[(int64_t)gr * ld + k] : (S)0;
      }
    }
  }
  __device__ inline void store(double* Sm) const {
    const int t = threadIdx.x;
    const int row = t / PER;
    const int kb = t % PER * V;
#pragma unroll
    for (int q = 0; q < V; ++q) Sm[(kb + q) * (T + 1) + row] = (double)v[q];
  }
};

// ------------------------------------------------------------------ tn_sym
// 1-D grid over (split, batch) groups of upper tiles (xcd_map).  part layout:
// [batch][split][tile][T][T].  An element's chain of sums does not depend on the tile edge T
// (32, 64 or 128).
template <typename SA, typename SB, int T>
__global__ __launch_bounds__(256, 2) void tn_sym_f64_kernel(
    const SA* __restrict__ A, const SB* __restrict__ B, const double* __restrict__ w,
    int64_t w_stride, int N, int64_t M, int nspin, int nt, int64_t kchunk, int nsplit, int batch,
    const unsigned char* __restrict__ active, double* __restrict__ part) {
  constexpr int R = T / 32, LD = T + 1;   // 16-row strips of a wave, LDS pitch
  __shared__ double As[KT * LD];
  __shared__ double Bs[KT * LD];
  __shared__ double Ws[KT];   // w over the current K-tile (1 when w is absent)
  const int ntiles = nt * (nt + 1) / 2;
  int group, tile;
  xcd_map(blockIdx.x, nsplit * batch, ntiles, group, tile);
  const int split = group % nsplit, b = group / nsplit;
  // upper-triangle tile index -> (ti, tj), ti <= tj
  int ti = 0, rem = tile;
  while (rem >= nt - ti) { rem -= nt - ti; ++ti; }
  const int tj = ti + rem;
  const int c = b % nspin;
  const SA* Ac = A + (int64_t)c * N * M;
  const SB* Bc = B + (int64_t)c * N * M;
  const double* wb = w ? w + (int64_t)b * w_stride : nullptr;
  const int64_t kbeg = (int64_t)split * kchunk;
  // an inactive block (blocks.h) keeps a zero partial tile
  const bool on = block_active(active, c, (N + BT - 1) / BT, ti * T / BT, tj * T / BT);
  const int64_t kend = on ? min(M, kbeg + kchunk) : kbeg;

  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wr = wid >> 1, wc = wid & 1;
  d4 acc[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  // the weight of B's column k is applied as B is read from LDS (the FP64 product
  // w[k] * B[j][k], as if B had been scaled in memory)
  auto wload = [&](int64_t k0) {
    const int64_t k = k0 + threadIdx.x;
    return (threadIdx.x < KT && k < kend) ? (wb ? wb[k] : 1.0) : 0.0;
  };
  TileLoad<SA, T> la;
  TileLoad<SB, T> lb;
  double wn = 0.0;
  if (kbeg < kend) {
    la.load(Ac, M, N, ti * T, kbeg, kend);
    lb.load(Bc, M, N, tj * T, kbeg, kend);
    wn = wload(kbeg);
  }
  for (int64_t k0 = kbeg; k0 < kend; k0 += KT) {
    __syncthreads();
    la.store(As);
    lb.store(Bs);
    if (threadIdx.x < KT) Ws[threadIdx.x] = wn;
    __syncthreads();
    if (k0 + KT < kend) {
      la.load(Ac, M, N, ti * T, k0 + KT, kend);
      lb.load(Bc, M, N, tj * T, k0 + KT, kend);
      wn = wload(k0 + KT);
    }
#pragma unroll
    for (int kk = 0; kk < KT; kk += 4) {
      const int kr = (kk + (lane >> 4)) * LD;
      const double wk = Ws[kk + (lane >> 4)];
      double a[R], bb[R];
#pragma unroll
      for (int i = 0; i < R; ++i) a[i] = As[kr + wr * (T / 2) + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < R; ++j) bb[j] = Bs[kr + wc * (T / 2) + j * 16 + (lane & 15)] * wk;
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j) acc[i][j] = mfma64(a[i], bb[j], acc[i][j]);
    }
  }
  double* out = part + (((int64_t)b * nsplit + split) * ntiles + tile) * (T * T);
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = wr * (T / 2) + i * 16 + 4 * v + (lane >> 4);
        const int col = wc * (T / 2) + j * 16 + (lane & 15);
        out[row * T + col] = acc[i][j][v];
      }
}

// H[b][i][j] = H[b][j][i] = the sum over the splits of the partial tile (edge T) holding
// (i, j), i <= j.  Many splits: eight groups of them in parallel (threadIdx.y), added in
// a fixed order; few: eight rows per block.
__global__ __launch_bounds__(256) void tn_reduce_wide_kernel(const double* __restrict__ part,
                                                             int N, int nt, int T, int nsplit,
                                                             double* __restrict__ H) {
  __shared__ double red[8][32];
  const int b = blockIdx.z, i = blockIdx.y, j = blockIdx.x * 32 + threadIdx.x;
  if ((int)(blockIdx.x * 32 + 31) < i) return;   // whole block below the diagonal
  const int ntiles = nt * (nt + 1) / 2;
  const bool on = j < N && i <= j;
  double s = 0.0;
  if (on) {
    const int ti = i / T, tj = j / T;
    const int tile = ti * nt - ti * (ti - 1) / 2 + (tj - ti);
    const double* p = part + ((int64_t)b * nsplit * ntiles + tile) * (T * T) +
                      (i - ti * T) * T + (j - tj * T);
    for (int q = threadIdx.y; q < nsplit; q += 8) s += p[(int64_t)q * ntiles * (T * T)];
  }
  red[threadIdx.y][threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.y == 0 && on) {
#pragma unroll
    for (int q = 1; q < 8; ++q) s += red[q][threadIdx.x];
    H[((int64_t)b * N + i) * N + j] = s;
    H[((int64_t)b * N + j) * N + i] = s;
  }
}

__global__ void tn_reduce_kernel(const double* __restrict__ part, int N, int nt, int T, int nsplit,
                                 double* __restrict__ H) {
  const int b = blockIdx.z;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = blockIdx.y * blockDim.y + threadIdx.y;
  if (i >= N || j >= N) return;
  const int ii = min(i, j), jj = max(i, j);
  const int ti = ii / T, tj = jj / T;
  // tile index of (ti, tj) in the upper-triangle enumeration
  const int tile = ti * nt - ti * (ti - 1) / 2 + (tj - ti);
  const int ntiles = nt * (nt + 1) / 2;
  const double* p = part + ((int64_t)b * nsplit * ntiles + tile) * (T * T) + (ii - ti * T) * T +
                    (jj - tj * T);
  double s = 0.0;
  for (int q = 0; q < nsplit; ++q) s += p[(int64_t)q * ntiles * (T * T)];
  H[((int64_t)b * N + i) * N + j] = s;
}

// ------------------------------------------------------------------ backproj
// Stage G rows [j0, j0+KT) x cols [i0, i0+BT) (G symmetric: G[j][i] = G[i][j]) or
// A rows [j0, j0+KT) x cols [p0, p0+BT) straight (no transpose) into S[k][col].
template <typename S>
struct RowLoad {
  S v[16];
  double fac;
  // thread t: row (t >> 3) of KT, 16 consecutive columns starting (t & 7) * 16
  __device__ inline void load(const S* __restrict__ X, int64_t ld, int nrows, int64_t ncols,
                              int j0, int64_t c0, double factor) {
    const int t = threadIdx.x;
    const int row = t >> 3;
    const int64_t cb = c0 + (t & 7) * 16;
    const int gr = j0 + row;
    const bool aligned = (reinterpret_cast<uintptr_t>(X + (int64_t)gr * ld + cb) & 15) == 0;
    fac = factor;
    if (gr < nrows && cb + 16 <= ncols && aligned) {
      load_run<16>(X + (int64_t)gr * ld + cb, v);
    } else {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int64_t cc = cb + q;
        v[q] = (gr < nrows && cc < ncols) ? X[(int64_t)gr * ld + cc] : (S)0;
      }
    }
  }
  // the factor is applied here, after the current K-tile's work, so that the
  // reads issued by load() stay in flight meanwhile
  __device__ inline void store(double* Sm) const {
    const int t = threadIdx.x;
    const int row = t >> 3;
    const int cb = (t & 7) * 16;
#pragma unroll
    for (int q = 0; q < 16; ++q) Sm[row * LDP + cb + q] = (double)v[q] * fac;
  }
};

// 1-D grid over (point block of BT points, batch b = direction * nspin + channel);
// the directions of one point block run together on one XCD (xcd_map).
__global__ __launch_bounds__(256, 2) void backproj_f64_kernel(
    const double* __restrict__ A, const double* __restrict__ G, int N, int64_t M, int nspin,
    int batch, double scale, const double* __restrict__ sub,
    const unsigned char* __restrict__ active, double* __restrict__ out) {
  __shared__ double Gs[KT * LDP];
  __shared__ double Ps[KT * LDP];
  __shared__ double red[4][64];
  int pblk, b;
  xcd_map(blockIdx.x, (int)((M + BT - 1) / BT), batch, pblk, b);
  const int c = b % nspin;
  const double* Ac = A + (int64_t)c * N * M;
  const double* Gb = G + (int64_t)b * N * N;
  const int64_t p0 = (int64_t)pblk * BT;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wr = wid >> 1, wc = wid & 1;
  double dsum[4] = {0.0, 0.0, 0.0, 0.0};   // per lane: columns wc*64 + j*16 + lane%16
  const int nib = (N + BT - 1) / BT;
  for (int ib = 0; ib < nib; ++ib) {
    const int i0 = ib * BT;
    // K runs over j in [i0, N): the diagonal block once, blocks right of it twice
    // (G symmetric), so only the upper block triangle is touched; inactive blocks
    // (blocks.h) are skipped, and a row block with none active contributes nothing
    const uint64_t bits = active_row_bits(active, c, nib, ib);
    const int nk = active_ktiles(bits, N, KT);
    if (nk == 0) continue;
    d4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    RowLoad<double> lg, lp;
    {
      int J;
      const int j0 = active_ktile(bits, 0, KT, J);
      lg.load(Gb, N, N, N, j0, i0, J > ib ? 2.0 : 1.0);
      lp.load(Ac, M, N, M, j0, p0, 1.0);
    }
    for (int t = 0; t < nk; ++t) {
      __syncthreads();
      lg.store(Gs);
      lp.store(Ps);
      __syncthreads();
      if (t + 1 < nk) {
        int J;
        const int jn = active_ktile(bits, t + 1, KT, J);
        lg.load(Gb, N, N, N, jn, i0, J > ib ? 2.0 : 1.0);
        lp.load(Ac, M, N, M, jn, p0, 1.0);
      }
#pragma unroll
      for (int kk = 0; kk < KT; kk += 4) {
        const int kr = (kk + (lane >> 4)) * LDP;
        double a[4], bb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = Gs[kr + wr * 64 + i * 16 + (lane & 15)];
#pragma unroll
        for (int j = 0; j < 4; ++j) bb[j] = Ps[kr + wc * 64 + j * 16 + (lane & 15)];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = mfma64(a[i], bb[j], acc[i][j]);
      }
    }
    // row-dot with A[i][p] for the rows of this block
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int gi = i0 + wr * 64 + i * 16 + 4 * v + (lane >> 4);
        if (gi < N) {
          const double* arow = Ac + (int64_t)gi * M;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int64_t p = p0 + wc * 64 + j * 16 + (lane & 15);
            if (p < M) dsum[j] += acc[i][j][v] * arow[p];
          }
        }
      }
  }
  // reduce over the 4 lane groups of a wave, then over the two row-waves
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    double v = dsum[j];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    dsum[j] = v;
  }
  if (lane < 16) {
#pragma unroll
    for (int j = 0; j < 4; ++j) red[wid][j * 16 + lane] = dsum[j];
  }
  __syncthreads();
  if (threadIdx.x < BT) {
    const int col = threadIdx.x;             // 0..127
    const int wcc = col >> 6, cl = col & 63;
    const double v = red[wcc][cl] + red[2 + wcc][cl];
    const int64_t p = p0 + col;
    if (p < M) {
      double r = scale * v;
      if (sub) r -= sub[(int64_t)b * M + p];
      out[(int64_t)b * M + p] = r;
    }
  }
}

// ------------------------------------------------------------------ nn
// Out[i][p] = sum_j Wt[j][i] B[j][p]; 1-D grid over (point block, row block), the
// row blocks of one point block together on one XCD (they read the same slice of B).
template <typename T>
// upper: Wt is upper triangular (Wt[j][i] = 0 for j > i), so row block i0 needs
// only k < i0 + BT.
__global__ __launch_bounds__(256, 2) void nn_f64_kernel(const double* __restrict__ Wt,
                                                        const T* __restrict__ B,
                                                        T* __restrict__ Out, int N, int64_t M,
                                                        int upper) {
  __shared__ double Ws[KT * LDP];
  __shared__ double Bs[KT * LDP];
  int pblk, rblk;
  const int nrb = (N + BT - 1) / BT;
  xcd_map(blockIdx.x, (int)((M + BT - 1) / BT), nrb, pblk, rblk);
  if (upper) rblk = nrb - 1 - rblk;   // the longest row blocks first
  const int64_t p0 = (int64_t)pblk * BT;
  const int i0 = rblk * BT;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wr = wid >> 1, wc = wid & 1;
  d4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  RowLoad<double> lw;
  RowLoad<T> lb;
  const int kmax = upper ? min(N, i0 + BT) : N;
  lw.load(Wt, N, N, N, 0, i0, 1.0);
  lb.load(B, M, N, M, 0, p0, 1.0);
  for (int j0 = 0; j0 < kmax; j0 += KT) {
    __syncthreads();
    lw.store(Ws);
    lb.store(Bs);
    __syncthreads();
    if (j0 + KT < kmax) {
      lw.load(Wt, N, N, N, j0 + KT, i0, 1.0);
      lb.load(B, M, N, M, j0 + KT, p0, 1.0);
    }
#pragma unroll
    for (int kk = 0; kk < KT; kk += 4) {
      const int kr = (kk + (lane >> 4)) * LDP;
      double a[4], bb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = Ws[kr + wr * 64 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 4; ++j) bb[j] = Bs[kr + wc * 64 + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma64(a[i], bb[j], acc[i][j]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int gi = i0 + wr * 64 + i * 16 + 4 * v + (lane >> 4);
      if (gi >= N) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t p = p0 + wc * 64 + j * 16 + (lane & 15);
        if (p < M) Out[(int64_t)gi * M + p] = (T)acc[i][j][v];
      }
    }
}

// ------------------------------------------------------------------ adjoint rotation
// Out_c[i][p] = scale * sum_m w_m[p] sum_j X_m[i][j] Psi_c[j][p] over the nmat
// symmetric matrices X_m of channel c (m = 0 .. nmat-1 at X + ((m * nspin) + c) N^2,
// weights at w + ((m * nspin) + c) M; two lists, the second starting at m = nx).
// FP64 arithmetic for either storage type.  grid x = point block, y = row block,
// z = channel.  The column weights travel with each staged K-tile.
template <typename T>
__global__ __launch_bounds__(256, 2) void adj_psi_f64_kernel(
    const double* __restrict__ X1, const double* __restrict__ w1, const double* __restrict__ X2,
    const double* __restrict__ w2, int nx, const T* __restrict__ Psi, int N, int64_t M, int nspin,
    double scale, T* __restrict__ Out) {
  __shared__ double Xs[KT * LDP];
  __shared__ double Bs[KT * LDP];
  __shared__ double Wc[BT];
  const int64_t p0 = (int64_t)blockIdx.x * BT;
  const int i0 = blockIdx.y * BT;
  const int c = blockIdx.z;
  const T* Pc = Psi + (int64_t)c * N * M;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wr = wid >> 1, wc = wid & 1;
  const int nkt = (N + KT - 1) / KT;
  const int nstep = 2 * nx * nkt;              // (matrix, K-tile) steps
  d4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  RowLoad<double> lx;
  RowLoad<T> lb;
  double wn = 0.0;
  auto load = [&](int step) {
    const int m = step / nkt, j0 = (step % nkt) * KT;
    const int64_t b = (int64_t)(m % nx) * nspin + c;
    const double* X = (m < nx ? X1 : X2) + b * N * N;
    const double* w = (m < nx ? w1 : w2) + b * M;
    lx.load(X, N, N, N, j0, i0, 1.0);
    lb.load(Pc, M, N, M, j0, p0, 1.0);
    if (threadIdx.x < BT) {
      const int64_t p = p0 + threadIdx.x;
      wn = p < M ? w[p] : 0.0;
    }
  };
  if (nstep > 0) load(0);
  for (int step = 0; step < nstep; ++step) {
    __syncthreads();
    lx.store(Xs);
    lb.store(Bs);
    if (threadIdx.x < BT) Wc[threadIdx.x] = wn;
    __syncthreads();
    if (step + 1 < nstep) load(step + 1);
    double wcol[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) wcol[j] = Wc[wc * 64 + j * 16 + (lane & 15)];
#pragma unroll
    for (int kk = 0; kk < KT; kk += 4) {
      const int kr = (kk + (lane >> 4)) * LDP;
      double a[4], bb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = Xs[kr + wr * 64 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 4; ++j) bb[j] = Bs[kr + wc * 64 + j * 16 + (lane & 15)] * wcol[j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma64(a[i], bb[j], acc[i][j]);
    }
  }
  T* Oc = Out + (int64_t)c * N * M;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int gi = i0 + wr * 64 + i * 16 + 4 * v + (lane >> 4);
      if (gi >= N) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t p = p0 + wc * 64 + j * 16 + (lane & 15);
        if (p < M) Oc[(int64_t)gi * M + p] = (T)(scale * acc[i][j][v]);
      }
    }
}

}  // namespace

hipError_t launch_tn_reduce(lrdm_ctx* ctx, const double* part, int N, int T, int nsplit, int batch,
                            double* H, bool in_order) {
  const int nt = (N + T - 1) / T;
  if (nsplit >= 16 && !in_order)
    tn_reduce_wide_kernel<<<dim3((N + 31) / 32, N, batch), dim3(32, 8), 0, ctx->stream>>>(
        part, N, nt, T, nsplit, H);
  else
    tn_reduce_kernel<<<dim3((N + 31) / 32, (N + 7) / 8, batch), dim3(32, 8), 0, ctx->stream>>>(
        part, N, nt, T, nsplit, H);
  return hipGetLastError();
}

// Partial tiles of 128 x 128 a range of points takes, in bytes.
static size_t tn_range_bytes(int N, int batch) {
  const int ntb = (N + BT - 1) / BT;
  return (size_t)batch * (ntb * (ntb + 1) / 2) * BT * BT * sizeof(double);
}

// Ranges the partial sums have room for: tn_split_cap, or for the forms that use more
// (FP32 and BF16X3) with a workspace of the preferred size (split_limit 0) as many as
// fill 96 MiB, each at least 512 points.
int tn_range_cap(int N, int64_t M, int batch, int order, int split_limit) {
  const int ntb = (N + BT - 1) / BT;
  const int cap = tn_split_cap(ntb * (ntb + 1) / 2 * batch, M);
  if (split_limit > 0) return std::min(cap, split_limit);
  if (order == TN_ARITH_F64 || order == TN_ORDERED_F64) return cap;
  const int64_t room = (int64_t)(((size_t)96 << 20) / tn_range_bytes(N, batch));
  return (int)std::max<int64_t>(cap, std::min<int64_t>(room, M / 512));
}

size_t tn_part_bytes(int N, int64_t M, int batch, int order, int split_limit) {
  const size_t tiles = tn_range_cap(N, M, batch, order, split_limit) * tn_range_bytes(N, batch);
  return split_limit > 0 || order != TN_ARITH_F64 ? tiles
                                                  : std::max(tiles, tn_direct_bytes(N, M, batch));
}

// FP32 arithmetic (whose partial sums are grouped by K-tile, so that any count gives the
// same sums up to the FP64 additions): the count within the workspace whose workgroups,
// two per tile and two per CU, finish first, each with a fixed cost of twelve K-tiles and
// all of them one range late: workgroups do not start together, so that one or two
// rounds of long ranges leave a tail, and from about six rounds on it no longer matters.
// 64^3, 300 states, 3 directions: 18 ranges (1 round) 1839 us, 37 1750, 56 1538, 113 1550;
// 64^3, 700, 2: 7 ranges 5069, 14 3904, 42 3564; 48^3, 256, 8: 21 888, 64 872; 24^3, 32,
// 4: 33 us (512-point ranges), 566 with ranges of at least 2048 points on 128-row tiles.
// The other forms: tn_splits.
int tn_default_splits(int N, int64_t M, int batch, int order, int split_limit) {
  const int ntb = (N + BT - 1) / BT;
  const int items = ntb * (ntb + 1) / 2 * batch;
  if (order == TN_STAGED_LP || order == TN_SPLIT_LP) {
    // Staged through registers (rows at any address), or BF16X3 splitting both operands: a
    // workgroup per tile and CU, so that the long ranges of tn_splits can fill a round that
    // the count above overfills: 27 x 33 x 35, 800 states, 2 channels, 4 ranges (224
    // workgroups) 1390 us, 10 1645; 129 states, 1 channel, 4 ranges 1394, 60 108 (FP32).
    // Groups of tiles that divide among the XCDs stay on one each (xcd.h).
    auto cost = [&](int s) {
      const int64_t groups = (int64_t)s * batch;
      const int64_t rounds = groups % 8 == 0 ? (groups / 8 * (items / batch) + 31) / 32
                                             : (groups * (items / batch) + 255) / 256;
      return rounds * (double)((M + KT * s - 1) / (KT * s) + 6);
    };
    const int ring = tn_default_splits(N, M, batch, TN_ARITH_F32, split_limit);
    const int lengthy = std::min(tn_splits(items, M),
                                 tn_range_cap(N, M, batch, order, split_limit));
    return cost(lengthy) <= (order == TN_SPLIT_LP ? 1.0 : 0.95) * cost(ring) ? lengthy : ring;
  }
  if (order != TN_ARITH_F32) return tn_splits(items, M);
  const int cap = tn_range_cap(N, M, batch, order, split_limit);
  const int halves = 2 * items - (N - (ntb - 1) * BT <= BT / 2 ? ntb * batch : 0);
  int best = 1;
  double least = 1e300;
  for (int s = 1; s <= cap; ++s) {
    const double rounds = (double)(((int64_t)halves * s + 511) / 512);
    const double cost = (rounds + 1.0) * ((double)((M + KT * s - 1) / (KT * s)) + 12.0);
    if (cost < least) {
      least = cost;
      best = s;
    }
  }
  return best;
}

// Parts each range of a BF16X3 projection with pre-split pieces is cut into: its FP32
// sums run over groups of 128 points from the range's start, so that a cut between
// groups leaves them as they are.  One workgroup per tile, part and CU; the cost as above.
// Cut only for a tenth or more: the kernel with parts is 1 % slower and writes that many
// more partial tiles (2700 workgroups a direction set, cut for a predicted 3 %: 0.987x).
int tn_range_parts(int N, int64_t M, int batch, int nsplit, int64_t kchunk, int split_limit) {
  const int ntb = (N + BT - 1) / BT;
  const int64_t wgs = (int64_t)(ntb * (ntb + 1) / 2) * batch * nsplit;
  const int64_t groups = (kchunk + BT - 1) / BT;
  const int most = (int)std::min<int64_t>(
      groups, tn_range_cap(N, M, batch, TN_ARITH_BF16X3, split_limit) / nsplit);
  auto cost_of = [&](int q) {
    const double rounds = (double)((wgs * q + 255) / 256);
    return rounds * ((double)((groups + q - 1) / q * (BT / KT)) + 12.0);
  };
  int best = 1;
  double least = 0.9 * cost_of(1);
  for (int q = 2; q <= most; ++q) {
    const double cost = cost_of(q);
    if (cost < least) {
      least = cost;
      best = q;
    }
  }
  return best;
}

int tn_split_count(const lrdm_ctx* ctx, int N, int64_t M, int batch, int arith, bool weighted,
                   int order) {
  const int ntb = (N + BT - 1) / BT;
  const int ntiles = ntb * (ntb + 1) / 2;
  const auto it = ctx->tn_tuned.find({N, M, batch, arith, weighted ? 1 : 0});
  int s = tn_default_splits(N, M, batch, order, ctx->split_limit);
  if (it != ctx->tn_tuned.end() && it->second >= 1 &&
      it->second <= tn_range_cap(N, M, batch, order, ctx->split_limit))
    s = it->second;
  if (ctx->split_limit > 0) s = std::min(s, std::min(ctx->split_limit, tn_split_cap(ntiles * batch, M)));
  return s;
}

int tn_variant(const lrdm_ctx* ctx, int N, int64_t M, int batch, int arith, bool weighted) {
  const auto it = ctx->tn_variant.find({N, M, batch, arith, weighted ? 1 : 0});
  return it == ctx->tn_variant.end() ? TN_VAR_DEFAULT : it->second;
}

size_t tn_workspace_bytes(int N, int64_t M, int batch, lrdm_prec prec, int split_limit) {
  const int order = prec == LRDM_FP64 ? TN_ARITH_F64 : TN_ARITH_F32;
  return ws_align(tn_part_bytes(N, M, batch, order, split_limit)) + tn_split_bytes(N, M, prec);
}

template <typename SA, typename SB>
hipError_t launch_tn_sym_f64(lrdm_ctx* ctx, const SA* A, const SB* B, const double* w,
                             int64_t w_stride, int N, int64_t M, int nspin, int batch,
                             double* H, const unsigned char* active) {
  const int ntb = (N + BT - 1) / BT;
  const int ntiles = ntb * (ntb + 1) / 2;
  constexpr bool fp32 = sizeof(SA) == sizeof(float);
  constexpr int order = fp32 ? TN_ORDERED_F64 : TN_ARITH_F64;
  const int ns = tn_split_count(ctx, N, M, batch, TN_ARITH_F64, w != nullptr, order);
  int64_t kchunk = (M + ns - 1) / ns;
  kchunk = (kchunk + KT - 1) / KT * KT;
  const size_t room = tn_part_bytes(N, M, batch, order, ctx->split_limit);
  double* part = static_cast<double*>(ws_take(ctx, room));
  // A block held in FP32 keeps one order of its sums (that of this kernel, at any tile edge):
  // the basis an ill-conditioned filtered block is orthonormalised to is rounded to FP32, so
  // that a Gram matrix off by one rounding moves its Ritz pairs by far more.
  if constexpr (!fp32) {
    if (tn_direct_ok(N, M, batch)) {
      // the autotuned count, relative to the default one, scales the number of ranges
      const TnDirectPlan p = tn_direct_plan(N, M, batch, room,
                                            (double)ns / tn_splits(ntiles * batch, M));
      if (B)
        return launch_tn_direct<SA, SB>(ctx, p, A, B, w, w_stride, N, M, nspin, batch, part, H, active,
                                        static_cast<const void*>(A) == static_cast<const void*>(B));
      return launch_tn_direct<SA, SA>(ctx, p, A, A, w, w_stride, N, M, nspin, batch, part, H, active,
                                      true);
    }
  }
  auto run = [&](auto edge) -> hipError_t {
    constexpr int T = decltype(edge)::value;
    const int nt = (N + T - 1) / T;
    const unsigned grd = (unsigned)(nt * (nt + 1) / 2 * ns * batch);
    {
      ProfScope prof(ctx, w ? "proj" : "gram");
      if (B)
        tn_sym_f64_kernel<SA, SB, T><<<grd, 256, 0, ctx->stream>>>(
            A, B, w, w_stride, N, M, nspin, nt, kchunk, ns, batch, active, part);
      else
        tn_sym_f64_kernel<SA, SA, T><<<grd, 256, 0, ctx->stream>>>(
            A, A, w, w_stride, N, M, nspin, nt, kchunk, ns, batch, active, part);
      LRDM_HIP(hipGetLastError());
    }
    return launch_tn_reduce(ctx, part, N, T, ns, batch, H, fp32);
  };
  // The largest edge that leaves enough workgroups (eight to a CU; of 64 rows four).
  // Gram product, edge 128 / 64 / 32: 24^3, 32 states (4 ranges) 1116 / 419 / 155 us;
  // 48^3, 256 (48 workgroups of 128) 1001 / 352 / 310; 64^3, 200 (640 of 64)
  // 705 / 534 / 394; 64^3, 512 (640 of 128, 2304 of 64) 1803 / 1395 / 1661; 64^3, 1024
  // (2304 of 128) 5007 / 4981 / 6517.
  if constexpr (fp32) {
    const int64_t each = (int64_t)ns * batch;
    const int nt = (N + 63) / 64;
    if (ntiles * each < 2048) {
      if (nt * (nt + 1) / 2 * each < 1024) return run(std::integral_constant<int, 32>{});
      return run(std::integral_constant<int, 64>{});
    }
  }
  return run(std::integral_constant<int, BT>{});
}
template hipError_t launch_tn_sym_f64<double, double>(lrdm_ctx*, const double*, const double*,
                                                      const double*, int64_t, int, int64_t, int,
                                                      int, double*, const unsigned char*);
template hipError_t launch_tn_sym_f64<float, float>(lrdm_ctx*, const float*, const float*,
                                                    const double*, int64_t, int, int64_t, int, int,
                                                    double*, const unsigned char*);
template hipError_t launch_tn_sym_f64<float, double>(lrdm_ctx*, const float*, const double*,
                                                     const double*, int64_t, int, int64_t, int,
                                                     int, double*, const unsigned char*);

template <>
hipError_t launch_tn_sym<double>(lrdm_ctx* ctx, const double* A, const double* B,
                                 const double* w, int64_t w_stride, int N, int64_t M, int nspin,
                                 int batch, lrdm_prec, double* H, const unsigned char* active) {
  return launch_tn_sym_f64<double, double>(ctx, A, B, w, w_stride, N, M, nspin, batch, H, active);
}

template <>
hipError_t launch_backproj<double>(lrdm_ctx* ctx, const double* A, const double* G, int N,
                                   int64_t M, int nspin, int batch, lrdm_prec, double scale,
                                   const double* sub, double* out, const unsigned char* active) {
  if (backproj_direct_ok(N))
    return launch_backproj_direct(ctx, A, G, N, M, nspin, batch, scale, sub, out, active);
  const unsigned grd = (unsigned)((M + BT - 1) / BT * batch);
  ProfScope prof(ctx, "backproj");
  backproj_f64_kernel<<<grd, 256, 0, ctx->stream>>>(A, G, N, M, nspin, batch, scale, sub, active,
                                                    out);
  return hipGetLastError();
}

template <typename S>
hipError_t launch_nn_f64(lrdm_ctx* ctx, const double* Wt, const S* B, S* Out, int N, int64_t M,
                         bool upper) {
  const unsigned grd = (unsigned)((M + BT - 1) / BT) * (unsigned)((N + BT - 1) / BT);
  ProfScope prof(ctx, "nn");
  nn_f64_kernel<S><<<grd, 256, 0, ctx->stream>>>(Wt, B, Out, N, M, upper ? 1 : 0);
  return hipGetLastError();
}
template hipError_t launch_nn_f64<double>(lrdm_ctx*, const double*, const double*, double*, int,
                                          int64_t, bool);
template hipError_t launch_nn_f64<float>(lrdm_ctx*, const double*, const float*, float*, int,
                                         int64_t, bool);

template <>
hipError_t launch_adj_psi<double>(lrdm_ctx* ctx, const double* X1, const double* w1,
                                  const double* X2, const double* w2, int nx, const double* Psi,
                                  int N, int64_t M, int nspin, double scale, double* Out,
                                  const unsigned char*) {
  dim3 grd((unsigned)((M + BT - 1) / BT), (N + BT - 1) / BT, nspin);
  ProfScope prof(ctx, "adj_psi");
  adj_psi_f64_kernel<double><<<grd, 256, 0, ctx->stream>>>(X1, w1, X2, w2, nx, Psi, N, M, nspin,
                                                           scale, Out);
  return hipGetLastError();
}

}  // namespace lrdm
