// Hartree kernel K_c of Eq. (3) on the periodic grid:
//     dV = 4 pi (-Lap_h)^{-1} u,  q = 0 component removed,
// with the same 7-point Laplacian as the Hamiltonian.  -Lap_h is a sum of
// per-axis circulant second differences, diagonalised by a real orthonormal
// basis of each axis: column 0 = 1/sqrt(n); columns 2m-1, 2m = sqrt(2/n) cos, sin
// of 2 pi m j / n (m < n/2); for even n the last column (-1)^j / sqrt(n).  The
// eigenvalue of a column with frequency m is (2 - 2 cos(2 pi m / n)) / h^2.
// The transform is three passes of a dense n x n matrix along x, y and z.
#include <algorithm>

#include "lrdm_internal.h"

namespace lrdm {
namespace {

__device__ inline int freq_of(int col, int n) {
  // column index -> frequency m
  if (col == 0) return 0;
  if ((n % 2 == 0) && col == n - 1) return n / 2;
  return (col + 1) / 2;
}

struct Axes {
  int n[3];
  double h[3];
  double* U[3];     // [n][n]
  double* lam[3];   // [n]
};

// U[j][col] and lam[col] of axis blockIdx.z.
__global__ void basis_kernel(Axes ax) {
  const int d = blockIdx.z, n = ax.n[d];
  const double h = ax.h[d];
  double* __restrict__ U = ax.U[d];
  double* __restrict__ lam = ax.lam[d];
  const int col = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (col >= n || j >= n) return;
  const int m = freq_of(col, n);
  double v;
  if (col == 0) {
    v = 1.0 / sqrt((double)n);
  } else if ((n % 2 == 0) && col == n - 1) {
    v = ((j & 1) ? -1.0 : 1.0) / sqrt((double)n);
  } else {
    // angle 2 pi m j / n reduced exactly modulo n before the trigonometric call
    const double frac = 2.0 * (double)((int64_t)m * j % n) / (double)n;
    double s, c;
    sincospi(frac, &s, &c);
    v = sqrt(2.0 / n) * ((col & 1) ? c : s);
  }
  U[(int64_t)j * n + col] = v;
  if (j == 0) {
    double s, c;
    sincospi(2.0 * (double)m / (double)n, &s, &c);
    lam[col] = (2.0 - 2.0 * c) / (h * h);
  }
}

// out[.., k, ..] = sum_j B(j, k) in[.., j, ..] along one axis, B = U (forward
// uses U^T: coefficient k = sum_j U[j][k] x_j; inverse: x_j = sum_k U[j][k] c_k).
__global__ void axis_kernel(const double* __restrict__ in, double* __restrict__ out, int nx,
                            int ny, int nz, int axis, const double* __restrict__ U, int inverse,
                            int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int64_t M = (int64_t)nx * ny * nz;
  const int64_t b = e / M;
  const int64_t p = e - b * M;
  const int x = (int)(p % nx);
  const int y = (int)((p / nx) % ny);
  const int z = (int)(p / ((int64_t)nx * ny));
  int n, k;
  int64_t stride, base;
  if (axis == 0) { n = nx; k = x; stride = 1; base = p - x; }
  else if (axis == 1) { n = ny; k = y; stride = nx; base = p - (int64_t)y * nx; }
  else { n = nz; k = z; stride = (int64_t)nx * ny; base = p - (int64_t)z * nx * ny; }
  const double* src = in + b * M + base;
  double s = 0.0;
  if (!inverse) {
    for (int j = 0; j < n; ++j) s += U[(int64_t)j * n + k] * src[j * stride];
  } else {
    for (int j = 0; j < n; ++j) s += U[(int64_t)k * n + j] * src[j * stride];
  }
  out[e] = s;
}

// The same transform for axes of at most kLdsAxis points, staged through LDS: the
// axis basis U (n x n) and a tile of the data, so that every value is read from
// HBM once per pass.
//  * axis 0 (x, contiguous lines): a block takes 64 lines of n points;
//  * axes 1 and 2: a block takes, for one index of the slower dimensions, the n
//    planes of a run of up to 64 consecutive points of the faster ones
//    (in[j][i] with j along the axis, i contiguous).
// out[.., k, ..] = sum_j coef(j, k) in[.., j, ..], coef = U[j][k] (forward) or
// U[k][j] (inverse).
constexpr int kLdsAxis = 64;

__global__ __launch_bounds__(256) void axis_lds_kernel(const double* __restrict__ in,
                                                       double* __restrict__ out, int n,
                                                       int64_t inner, int64_t lines,
                                                       const double* __restrict__ U,
                                                       int inverse) {
  __shared__ double Us[kLdsAxis * kLdsAxis];
  __shared__ double T[kLdsAxis * (kLdsAxis + 1)];
  for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
    const int j = e / n, k = e - j * n;
    Us[j * kLdsAxis + k] = inverse ? U[(int64_t)k * n + j] : U[(int64_t)j * n + k];
  }
  if (inner == 1) {
    // 64 contiguous lines of n points: T[line][j]
    const int64_t l0 = (int64_t)blockIdx.x * 64;
    const int nl = (int)min((int64_t)64, lines - l0);
    const double* src = in + l0 * n;
    for (int e = threadIdx.x; e < nl * n; e += blockDim.x) {
      const int l = e / n, j = e - l * n;
      T[l * (kLdsAxis + 1) + j] = src[e];
    }
    __syncthreads();
    double* dst = out + l0 * n;
    for (int e = threadIdx.x; e < nl * n; e += blockDim.x) {
      const int l = e / n, k = e - l * n;
      double acc = 0.0;
      for (int j = 0; j < n; ++j) acc += Us[j * kLdsAxis + k] * T[l * (kLdsAxis + 1) + j];
      dst[e] = acc;
    }
    return;
  }
  // a block: one outer index o and a run of up to 64 points i0 .. i0 + w
  const int64_t chunks = (inner + 63) / 64;
  const int64_t o = (int64_t)blockIdx.x / chunks;
  const int64_t i0 = ((int64_t)blockIdx.x - o * chunks) * 64;
  const int w = (int)min((int64_t)64, inner - i0);
  const double* src = in + o * n * inner + i0;
  for (int e = threadIdx.x; e < n * 64; e += blockDim.x) {
    const int j = e >> 6, i = e & 63;
    if (i < w) T[j * (kLdsAxis + 1) + i] = src[(int64_t)j * inner + i];
  }
  __syncthreads();
  double* dst = out + o * n * inner + i0;
  for (int e = threadIdx.x; e < n * 64; e += blockDim.x) {
    const int k = e >> 6, i = e & 63;
    if (i >= w) continue;
    double acc = 0.0;
    for (int j = 0; j < n; ++j) acc += Us[j * kLdsAxis + k] * T[j * (kLdsAxis + 1) + i];
    dst[(int64_t)k * inner + i] = acc;
  }
}

// Grids of at most kLdsAxis points an axis take three passes over memory instead of eight:
// x and y forward on whole planes, z forward, the symbol and z back on runs of
// columns, y and x back on planes.  A pass is a product of the axis basis and the tile,
// both in LDS, on the FP64 matrix cores (the vector units have the same rate, but a wave
// reads 8 bytes of LDS per 32 products for them, where an outer product held in registers
// needs four times that); sizes are padded to 16 with zeros.
// 64^3, 16 directions: 131 us against 510 with an LDS pass per axis; 48^3, 8 directions
// 50 against 186; 24^3, 4 directions 20 against 57, most of it the launches (4 for 11).
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int kHartreeThreads = 512;
constexpr int kTiles = 2;   // of a wave: 16 of a plane's or a run's 64 x 64 at most

__host__ __device__ constexpr int pad16(int n) { return (n + 15) & ~15; }
// Row strides in LDS: sixteen rows at one column lie in different banks.
__host__ __device__ constexpr int lds_stride(int n) { return pad16(n) + 2; }

// U into LDS, zero past n.
__device__ inline void stage_basis(const double* __restrict__ U, int n, double* Us) {
  const int m = pad16(n), st = lds_stride(n);
  const int k = threadIdx.x & 63;
  if (k < m)
    for (int j = threadIdx.x >> 6; j < m; j += kHartreeThreads / 64)
      Us[j * st + k] = j < n && k < n ? U[(int64_t)j * n + k] : 0.0;
}

// Along the rows of T (ROWS: out[l][k] = sum_j coef(j, k) T[l][j]) or its columns
// (out[k][l] = sum_j coef(j, k) T[j][l]), in place; coef = U[j][k], INV: U[k][j].
// n along the axis, m16 lines (padded); every thread of the workgroup calls it.
template <bool ROWS, bool INV>
__device__ inline void axis_pass(double* T, int st, const double* Us, int n, int m16) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int col = lane & 15, g = lane >> 4;
  const int us = lds_stride(n), nk = pad16(n) / 16, tiles = nk * (m16 / 16);
  d4 acc[kTiles];
  int tk[kTiles], tl[kTiles];
#pragma unroll
  for (int u = 0; u < kTiles; ++u) {
    const int tile = wid + u * (kHartreeThreads / 64);
    tl[u] = tile / nk;
    tk[u] = tile - tl[u] * nk;
    acc[u] = d4{0.0, 0.0, 0.0, 0.0};
    if (tile >= tiles) continue;
    const double* c = INV ? Us + (16 * tk[u] + col) * us + g : Us + g * us + 16 * tk[u] + col;
    const double* t = ROWS ? T + (16 * tl[u] + col) * st + g : T + g * st + 16 * tl[u] + col;
    const int cs = INV ? 1 : us, ts = ROWS ? 1 : st;
#pragma unroll 4
    for (int j = 0; j < n; j += 4) {
      const double a = c[j * cs], b = t[j * ts];
      acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(ROWS ? b : a, ROWS ? a : b, acc[u], 0, 0, 0);
    }
  }
  __syncthreads();   // every read of T is done
#pragma unroll
  for (int u = 0; u < kTiles; ++u) {
    if (wid + u * (kHartreeThreads / 64) >= tiles) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (ROWS)
        T[(16 * tl[u] + 4 * v + g) * st + 16 * tk[u] + col] = acc[u][v];
      else
        T[(16 * tk[u] + 4 * v + g) * st + 16 * tl[u] + col] = acc[u][v];
    }
  }
  __syncthreads();
}

// Plane blockIdx.x of direction blockIdx.y: forward, the sum of in's channels to out
// [r][M]; INV, in [r][M] to every channel of out.
template <bool INV>
__global__ __launch_bounds__(kHartreeThreads) void hartree_plane_kernel(
    const double* __restrict__ in, int nspin, double* __restrict__ out, int nx, int ny, int64_t M,
    const double* __restrict__ Ux, const double* __restrict__ Uy) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_hartree[];
  double* T = reinterpret_cast<double*>(smem_hartree);   // [ny16][st]
  const int st = lds_stride(nx), ny16 = pad16(ny);
  double* Us = T + ny16 * st;
  const int64_t plane = (int64_t)blockIdx.x * nx * ny;
  const int x = threadIdx.x & 63, y0 = threadIdx.x >> 6;
  constexpr int DY = kHartreeThreads / 64;
  stage_basis(INV ? Uy : Ux, INV ? ny : nx, Us);
  const int nin = INV ? 1 : nspin;
  const double* src = in + (int64_t)blockIdx.y * nin * M + plane;
  if (x < pad16(nx))
    for (int y = y0; y < ny16; y += DY) {
      double s = 0.0;
      if (x < nx && y < ny)
        for (int c = 0; c < nin; ++c) s += src[(int64_t)c * M + y * nx + x];
      T[y * st + x] = s;
    }
  __syncthreads();
  if (INV) axis_pass<false, true>(T, st, Us, ny, pad16(nx));
  else axis_pass<true, false>(T, st, Us, nx, ny16);
  stage_basis(INV ? Ux : Uy, INV ? nx : ny, Us);
  __syncthreads();
  if (INV) axis_pass<true, true>(T, st, Us, nx, ny16);
  else axis_pass<false, false>(T, st, Us, ny, pad16(nx));
  const int nout = INV ? nspin : 1;
  double* dst = out + (int64_t)blockIdx.y * nout * M + plane;
  if (x < nx)
    for (int y = y0; y < ny; y += DY) {
      const double v = T[y * st + x];
      for (int c = 0; c < nout; ++c) dst[(int64_t)c * M + y * nx + x] = v;
    }
}

// W columns (points of the plane from blockIdx.x W on) of direction blockIdx.y, in
// place: z forward, the symbol, z back.
__global__ __launch_bounds__(kHartreeThreads) void hartree_column_kernel(
    double* __restrict__ c, int nx, int ny, int nz, int W, const double* __restrict__ Uz,
    const double* __restrict__ lx, const double* __restrict__ ly, const double* __restrict__ lz) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_hartree[];
  double* T = reinterpret_cast<double*>(smem_hartree);   // [nz16][st]
  const int st = lds_stride(W), nz16 = pad16(nz);
  double* Us = T + nz16 * st;
  const int P = nx * ny;
  const int i = threadIdx.x % W, z0 = threadIdx.x / W, dz = kHartreeThreads / W;
  const int p = blockIdx.x * W + i;
  double* col = c + (int64_t)blockIdx.y * P * nz + p;
  stage_basis(Uz, nz, Us);
  for (int z = z0; z < nz16; z += dz)
    T[z * st + i] = z < nz && p < P ? col[(int64_t)z * P] : 0.0;
  __syncthreads();
  axis_pass<false, false>(T, st, Us, nz, W);
  if (p < P) {
    const int y = p / nx, x = p - y * nx;
    for (int z = z0; z < nz; z += dz) {
      const double lam = lx[x] + ly[y] + lz[z];
      const double four_pi = 12.566370614359172953850573533118;
      const double v = T[z * st + i];
      T[z * st + i] = (p == 0 && z == 0) ? 0.0 : v * (four_pi / lam);
    }
  }
  __syncthreads();
  axis_pass<false, true>(T, st, Us, nz, W);
  if (p < P)
    for (int z = z0; z < nz; z += dz) col[(int64_t)z * P] = T[z * st + i];
}

__global__ void sum_channels_kernel(const double* __restrict__ u, int nspin, int64_t M, int r,
                                    double* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)r * M) return;
  const int64_t k = e / M, p = e - k * M;
  double s = 0.0;
  for (int c = 0; c < nspin; ++c) s += u[(k * nspin + c) * M + p];
  out[e] = s;
}

__global__ void symbol_kernel(double* __restrict__ c, int nx, int ny, int nz,
                              const double* __restrict__ lx, const double* __restrict__ ly,
                              const double* __restrict__ lz, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int64_t M = (int64_t)nx * ny * nz;
  const int64_t p = e % M;
  const int x = (int)(p % nx);
  const int y = (int)((p / nx) % ny);
  const int z = (int)(p / ((int64_t)nx * ny));
  const double lam = lx[x] + ly[y] + lz[z];
  const double four_pi = 12.566370614359172953850573533118;
  c[e] = (x == 0 && y == 0 && z == 0) ? 0.0 : c[e] * (four_pi / lam);
}

__global__ void scatter_channels_kernel(const double* __restrict__ src, int64_t M, int r,
                                        int nspin, double* __restrict__ dV) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)r * nspin * M) return;
  const int64_t p = e % M;
  const int64_t k = e / (M * nspin);
  dV[e] = src[k * M + p];
}

}  // namespace

size_t hartree_workspace_bytes(const Grid3& g) {
  return ws_align((size_t)(g.nx * g.nx + g.ny * g.ny + g.nz * g.nz + g.nx + g.ny + g.nz) * 8);
}

// scratch: 2 * r * M doubles
hipError_t launch_hartree(lrdm_ctx* ctx, const Grid3& g, const double* u, int u_nspin, double* dV,
                          int dv_nspin, int r, double* scratch) {
  ProfScope prof(ctx, "hartree");
  double* tabs = static_cast<double*>(ws_take(ctx, hartree_workspace_bytes(g)));
  double* Ux = tabs;
  double* Uy = Ux + (int64_t)g.nx * g.nx;
  double* Uz = Uy + (int64_t)g.ny * g.ny;
  double* lx = Uz + (int64_t)g.nz * g.nz;
  double* ly = lx + g.nx;
  double* lz = ly + g.ny;
  const Axes ax{{g.nx, g.ny, g.nz}, {g.hx, g.hy, g.hz}, {Ux, Uy, Uz}, {lx, ly, lz}};
  const int most = std::max(g.nx, std::max(g.ny, g.nz));
  basis_kernel<<<dim3((most + 63) / 64, most, 3), 64, 0, ctx->stream>>>(ax);
  LRDM_HIP(hipGetLastError());
  const int64_t total = (int64_t)r * g.M;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  double* a = scratch;
  double* b = scratch + total;
  if (most <= kLdsAxis && r <= 65535) {
    const int u16 = std::max(pad16(g.nx) * lds_stride(g.nx), pad16(g.ny) * lds_stride(g.ny));
    const size_t plane = (size_t)(pad16(g.ny) * lds_stride(g.nx) + u16) * sizeof(double);
    // runs of 64 columns, or of 16 where those leave CUs without a workgroup
    const int64_t P = (int64_t)g.nx * g.ny;
    const int W = (P + 63) / 64 * r >= 256 ? 64 : 16;
    const size_t run = (size_t)pad16(g.nz) * (lds_stride(W) + lds_stride(g.nz)) * sizeof(double);
    auto room = [&](auto kernel, size_t bytes) -> hipError_t {
      return bytes <= 65536 ? hipSuccess
                            : hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                                  (int)bytes);
    };
    LRDM_HIP(room(&hartree_plane_kernel<false>, plane));
    LRDM_HIP(room(&hartree_plane_kernel<true>, plane));
    LRDM_HIP(room(&hartree_column_kernel, run));
    const dim3 planes(g.nz, r);
    hartree_plane_kernel<false><<<planes, kHartreeThreads, plane, ctx->stream>>>(
        u, u_nspin, a, g.nx, g.ny, g.M, Ux, Uy);
    hartree_column_kernel<<<dim3((unsigned)((P + W - 1) / W), r), kHartreeThreads, run,
                            ctx->stream>>>(a, g.nx, g.ny, g.nz, W, Uz, lx, ly, lz);
    hartree_plane_kernel<true><<<planes, kHartreeThreads, plane, ctx->stream>>>(
        a, dv_nspin, dV, g.nx, g.ny, g.M, Ux, Uy);
    return hipGetLastError();
  }
  // one pass along `axis`: LDS-staged for axes of at most kLdsAxis points
  auto pass = [&](const double* in, double* out, int axis, const double* Ud, int inverse) {
    const int n = axis == 0 ? g.nx : (axis == 1 ? g.ny : g.nz);
    if (n > kLdsAxis) {
      axis_kernel<<<blocks, 256, 0, ctx->stream>>>(in, out, g.nx, g.ny, g.nz, axis, Ud, inverse,
                                                   total);
      return;
    }
    const int64_t inner = axis == 0 ? 1 : (axis == 1 ? g.nx : (int64_t)g.nx * g.ny);
    const int64_t lines = total / n;                 // lines of n points along the axis
    const int64_t nblk = axis == 0 ? (lines + 63) / 64 : (lines / inner) * ((inner + 63) / 64);
    axis_lds_kernel<<<(unsigned)nblk, 256, 0, ctx->stream>>>(in, out, n, inner, lines, Ud,
                                                             inverse);
  };
  sum_channels_kernel<<<blocks, 256, 0, ctx->stream>>>(u, u_nspin, g.M, r, a);
  pass(a, b, 0, Ux, 0);
  pass(b, a, 1, Uy, 0);
  pass(a, b, 2, Uz, 0);
  symbol_kernel<<<blocks, 256, 0, ctx->stream>>>(b, g.nx, g.ny, g.nz, lx, ly, lz, total);
  pass(b, a, 2, Uz, 1);
  pass(a, b, 1, Uy, 1);
  if (dv_nspin == 1) {
    pass(b, dV, 0, Ux, 1);
  } else {
    pass(b, a, 0, Ux, 1);
    const int64_t tot2 = total * dv_nspin;
    scatter_channels_kernel<<<(unsigned)((tot2 + 255) / 256), 256, 0, ctx->stream>>>(a, g.M, r,
                                                                                    dv_nspin, dV);
  }
  return hipGetLastError();
}

}  // namespace lrdm
