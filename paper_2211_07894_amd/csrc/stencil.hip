// Stencil Hamiltonian applied to a block of vectors, fused with one step of the
// Chebyshev three-term recurrence (Sec. II C):
//     Yout = alpha (H - c0) Yin + beta Yold,   H = -1/2 Lap_h + diag(V)
// with the 7-point periodic Laplacian.  alpha = 1, c0 = 0, beta = 0 gives H Y.
// Yin and Yold have storage type TI, Yout type TO; the arithmetic is done in TO
// (H Y of an FP32 block can be formed and kept in FP64).
//
// Layout: vectors are [N][nz][ny][nx], x fastest.  A block owns one vector and a
// run of z planes; it marches in z keeping the planes z-1, z, z+1 of its points
// in registers and the whole current plane in LDS (double-buffered) for the x
// and y neighbours.  Every element of Yin is read from HBM about once (plus two
// halo planes per z run), Yold once, Yout written once: 3 M N s bytes per step,
// the bound of this HBM-limited kernel.
//
// The recurrence step of the filter takes a vectorised form of the same sweep
// when nx is a multiple of the 16-byte group (4 FP32 or 2 FP64 points): each
// thread owns groups of consecutive x points and moves each of Yin, Yold and V
// (V in the storage type) with one 16-byte load per plane, two planes ahead of
// the plane it computes, so that about twice the bytes are in flight per CU with
// fewer registers than the scalar form.  Yout may be the same buffer as Yold
// (each element is read, then written, by the same thread).
//
// A filter seldom takes single steps: a state that fits in LDS takes the whole filter
// in one workgroup (cheb_lds_kernel), and else up to five consecutive steps run in
// one sweep (cheb_sweep_kernel): each intermediate block is formed plane by plane and
// used by the next step while its planes are in registers and LDS, and only the last
// two blocks are written, so S steps move 4 M N s bytes instead of 3 S M N s.
#include <algorithm>

#include "lrdm_internal.h"

namespace lrdm {
namespace {

template <typename TI, typename T, int PPT>
__global__ __launch_bounds__(1024) void cheb_plane_kernel(
    const TI* __restrict__ Yin, const TI* Yold, T* Yout,
    const double* __restrict__ V, int nx, int ny, int nz, int zrun, T wx, T wy, T wz, T dshift,
    T alpha, T beta) {
  extern __shared__ unsigned char smem_raw[];
  T* plane = reinterpret_cast<T*>(smem_raw);
  const int P = nx * ny;
  const int64_t M = (int64_t)P * nz;
  const int vec = blockIdx.x;
  const int z0 = blockIdx.y * zrun;
  const int z1 = min(nz, z0 + zrun);
  const TI* yin = Yin + (int64_t)vec * M;
  const TI* yold = Yold ? Yold + (int64_t)vec * M : nullptr;
  T* yout = Yout + (int64_t)vec * M;

  int xy[PPT];   // (y << 16) | x of each point owned by this thread, -1 if none
  T prev[PPT], cur[PPT], next[PPT];
  T vcur[PPT], ocur[PPT];   // V and Yold at the current plane, loaded one plane ahead
  {
    const int zm = (z0 == 0) ? nz - 1 : z0 - 1;
    const int zp = (z0 + 1 == nz) ? 0 : z0 + 1;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      const int qq = threadIdx.x + j * blockDim.x;
      if (qq < P) {
        const int y = qq / nx, x = qq - y * nx;
        xy[j] = (y << 16) | x;
        prev[j] = (T)yin[(int64_t)zm * P + qq];
        cur[j] = (T)yin[(int64_t)z0 * P + qq];
        next[j] = (T)yin[(int64_t)zp * P + qq];
        vcur[j] = (T)V[(int64_t)z0 * P + qq];
        ocur[j] = yold ? (T)yold[(int64_t)z0 * P + qq] : T(0);
      } else {
        xy[j] = -1;
        prev[j] = cur[j] = next[j] = vcur[j] = ocur[j] = T(0);
      }
    }
  }
  int buf = 0;
  for (int z = z0; z < z1; ++z) {
    T* pl = plane + buf * P;
#pragma unroll
    for (int j = 0; j < PPT; ++j)
      if (xy[j] >= 0) pl[threadIdx.x + j * blockDim.x] = cur[j];
    __syncthreads();
    // loads for the next planes, issued before this plane's arithmetic
    const bool more = z + 1 < z1;
    const int zn = (z + 2 >= nz) ? z + 2 - nz : z + 2;
    T nn[PPT], vn[PPT], on[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      const int qq = threadIdx.x + j * blockDim.x;
      nn[j] = vn[j] = on[j] = T(0);
      if (xy[j] >= 0 && more) {
        nn[j] = (T)yin[(int64_t)zn * P + qq];
        vn[j] = (T)V[(int64_t)(z + 1) * P + qq];
        if (yold) on[j] = (T)yold[(int64_t)(z + 1) * P + qq];
      }
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      if (xy[j] < 0) continue;
      const int x = xy[j] & 0xffff, y = xy[j] >> 16;
      const int q = y * nx + x;
      const int xm = (x == 0) ? q + nx - 1 : q - 1;
      const int xp = (x == nx - 1) ? q - nx + 1 : q + 1;
      const int ym = (y == 0) ? q + P - nx : q - nx;
      const int yp = (y == ny - 1) ? q - P + nx : q + nx;
      const int64_t off = (int64_t)z * P + q;
      const T c = cur[j];
      const T hy = wx * (pl[xm] + pl[xp]) + wy * (pl[ym] + pl[yp]) +
                   wz * (prev[j] + next[j]) + (vcur[j] + dshift) * c;
      T out = alpha * hy;
      if (yold) out += beta * ocur[j];
      yout[off] = out;
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      prev[j] = cur[j];
      cur[j] = next[j];
      next[j] = nn[j];
      vcur[j] = vn[j];
      ocur[j] = on[j];
    }
    buf ^= 1;
  }
}

template <typename TI, typename T, int PPT>
hipError_t launch_plane(lrdm_ctx* ctx, const Grid3& g, const double* V, const TI* Yin,
                        const TI* Yold, T* Yout, int N, int threads, int zrun, double alpha,
                        double c0, double beta) {
  const int P = g.nx * g.ny;
  const size_t smem = 2 * (size_t)P * sizeof(T);
  const T wx = T(-0.5 / (g.hx * g.hx)), wy = T(-0.5 / (g.hy * g.hy)), wz = T(-0.5 / (g.hz * g.hz));
  const T dshift = T(1.0 / (g.hx * g.hx) + 1.0 / (g.hy * g.hy) + 1.0 / (g.hz * g.hz) - c0);
  dim3 grd(N, (g.nz + zrun - 1) / zrun);
  if (smem > 65536)
    LRDM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&cheb_plane_kernel<TI, T, PPT>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  ProfScope prof(ctx, beta != 0.0 ? "cheb_step" : "hpsi");
  cheb_plane_kernel<TI, T, PPT><<<grd, threads, smem, ctx->stream>>>(
      Yin, beta != 0.0 ? Yold : nullptr, Yout, V, g.nx, g.ny, g.nz, zrun, wx, wy, wz, dshift,
      T(alpha), T(beta));
  return hipGetLastError();
}

template <typename TI, typename T>
hipError_t launch_stencil(lrdm_ctx* ctx, const Grid3& g, const double* V, const TI* Yin,
                          const TI* Yold, T* Yout, int N, double alpha, double c0, double beta) {
  const int P = g.nx * g.ny;
  // whole plane per block: up to 1024 threads, PPT points per thread
  int threads = P <= 1024 ? ((P + 63) / 64) * 64 : 1024;
  const int ppt = (P + threads - 1) / threads;
  // z runs: enough blocks for the chip (N * runs >= ~2048) but runs of >= 8 planes
  int runs = 1;
  while ((int64_t)N * runs < 2048 && g.nz / (runs * 2) >= 8) runs *= 2;
  const int zrun = (g.nz + runs - 1) / runs;
  if (ppt <= 1)
    return launch_plane<TI, T, 1>(ctx, g, V, Yin, Yold, Yout, N, threads, zrun, alpha, c0, beta);
  if (ppt <= 2)
    return launch_plane<TI, T, 2>(ctx, g, V, Yin, Yold, Yout, N, threads, zrun, alpha, c0, beta);
  if (ppt <= 4)
    return launch_plane<TI, T, 4>(ctx, g, V, Yin, Yold, Yout, N, threads, zrun, alpha, c0, beta);
  if (ppt <= 8)
    return launch_plane<TI, T, 8>(ctx, g, V, Yin, Yold, Yout, N, threads, zrun, alpha, c0, beta);
  return hipErrorInvalidValue;  // planes above 8192 points are rejected by validation
}


template <typename T, int W>
using vec_t = T __attribute__((ext_vector_type(W)));
// The same at any address of an element: V in double is the caller's.
template <typename T, int W>
struct Unaligned {
  typedef vec_t<T, W> type __attribute__((aligned(sizeof(T))));
};

// Vectorised step; W points per 16-byte group of the input type TI, Q groups per
// thread; arithmetic, V and Yout in T (T = TI for the recurrence, T = double for
// H Y of an FP32 block).
template <typename TI, typename T, int Q>
__global__ __launch_bounds__(1024) void cheb_vec_kernel(const TI* __restrict__ Yin, const TI* Yold,
                                                       T* Yout, const T* __restrict__ Vt, int nx,
                                                       int ny, int nz, int zrun, T wx, T wy, T wz,
                                                       T dshift, T alpha, T beta) {
  constexpr int W = 16 / sizeof(TI);
  using V = vec_t<T, W>;
  using VI = vec_t<TI, W>;
  extern __shared__ unsigned char smem_raw[];
  V* plane = reinterpret_cast<V*>(smem_raw);
  const int P = nx * ny, G = P / W, nxg = nx / W;
  const int64_t MG = (int64_t)G * nz;
  const int z0 = blockIdx.y * zrun;
  const int z1 = min(nz, z0 + zrun);
  const VI* yin = reinterpret_cast<const VI*>(Yin) + (int64_t)blockIdx.x * MG;
  const VI* yold = Yold ? reinterpret_cast<const VI*>(Yold) + (int64_t)blockIdx.x * MG : nullptr;
  V* yout = reinterpret_cast<V*>(Yout) + (int64_t)blockIdx.x * MG;
  using VU = typename Unaligned<T, W>::type;
  const VU* vg = reinterpret_cast<const VU*>(Vt);
  const V zero = V(T(0));
  // Yin planes z-1 .. z+2, Yold and V planes z, z+1 of each owned group
  V prev[Q], cur[Q], next[Q], ahead[Q], o0[Q], o1[Q], v0[Q], v1[Q];
  {
    const int zm = (z0 == 0) ? nz - 1 : z0 - 1;
    const int zp = (z0 + 1 == nz) ? 0 : z0 + 1;
    const int zpp = (zp + 1 == nz) ? 0 : zp + 1;
    const bool m1 = z0 + 1 < z1;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int gi = threadIdx.x + j * blockDim.x;
      prev[j] = cur[j] = next[j] = ahead[j] = o0[j] = o1[j] = v0[j] = v1[j] = zero;
      if (gi < G) {
        prev[j] = __builtin_convertvector(yin[(int64_t)zm * G + gi], V);
        cur[j] = __builtin_convertvector(yin[(int64_t)z0 * G + gi], V);
        next[j] = __builtin_convertvector(yin[(int64_t)zp * G + gi], V);
        v0[j] = vg[(int64_t)z0 * G + gi];
        if (yold) o0[j] = __builtin_convertvector(yold[(int64_t)z0 * G + gi], V);
        if (m1) {
          ahead[j] = __builtin_convertvector(yin[(int64_t)zpp * G + gi], V);
          v1[j] = vg[(int64_t)(z0 + 1) * G + gi];
          if (yold) o1[j] = __builtin_convertvector(yold[(int64_t)(z0 + 1) * G + gi], V);
        }
      }
    }
  }
  int buf = 0;
  for (int z = z0; z < z1; ++z) {
    V* pl = plane + buf * G;
    const T* pls = reinterpret_cast<const T*>(pl);
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int gi = threadIdx.x + j * blockDim.x;
      if (gi < G) pl[gi] = cur[j];
    }
    __syncthreads();
    // loads two planes ahead, issued before this plane's arithmetic
    const bool more2 = z + 2 < z1;
    const int zy = (z + 3 >= nz) ? z + 3 - nz : z + 3;
    VI ny_[Q], no[Q];
    V nv[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int gi = threadIdx.x + j * blockDim.x;
      ny_[j] = no[j] = VI(TI(0));
      nv[j] = zero;
      if (gi < G && more2) {
        ny_[j] = yin[(int64_t)zy * G + gi];
        nv[j] = vg[(int64_t)(z + 2) * G + gi];
        if (yold) no[j] = yold[(int64_t)(z + 2) * G + gi];
      }
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int gi = threadIdx.x + j * blockDim.x;
      if (gi >= G) continue;
      const int y = gi / nxg, x0 = (gi - y * nxg) * W;
      const int q = W * gi;
      const V ym = pl[y == 0 ? gi + G - nxg : gi - nxg];
      const V yp = pl[y == ny - 1 ? gi - G + nxg : gi + nxg];
      const T left = pls[x0 == 0 ? q + nx - 1 : q - 1];
      const T right = pls[x0 + W == nx ? q + W - nx : q + W];
      const V c = cur[j], pz = prev[j], nzv = next[j], vv = v0[j], o = o0[j];
      V out;
#pragma unroll
      for (int e = 0; e < W; ++e) {
        const T xl = e == 0 ? left : c[e == 0 ? 0 : e - 1];
        const T xr = e == W - 1 ? right : c[e == W - 1 ? 0 : e + 1];
        const T hy = wx * (xl + xr) + wy * (ym[e] + yp[e]) + wz * (pz[e] + nzv[e]) +
                     (vv[e] + dshift) * c[e];
        out[e] = alpha * hy + beta * o[e];
      }
      yout[(int64_t)z * G + gi] = out;
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      prev[j] = cur[j];
      cur[j] = next[j];
      next[j] = ahead[j];
      ahead[j] = __builtin_convertvector(ny_[j], V);
      o0[j] = o1[j];
      o1[j] = __builtin_convertvector(no[j], V);
      v0[j] = v1[j];
      v1[j] = nv[j];
    }
    buf ^= 1;
  }
}

template <typename TI, typename T, int Q>
hipError_t launch_vec(lrdm_ctx* ctx, const char* scope, const Grid3& g, const T* Vt, const TI* Yin,
                      const TI* Yold, T* Yout, int N, int threads, int zrun, double alpha,
                      double c0, double beta) {
  const int P = g.nx * g.ny;
  const size_t smem = 2 * (size_t)P * sizeof(T);
  const T wx = T(-0.5 / (g.hx * g.hx)), wy = T(-0.5 / (g.hy * g.hy)), wz = T(-0.5 / (g.hz * g.hz));
  const T dshift = T(1.0 / (g.hx * g.hx) + 1.0 / (g.hy * g.hy) + 1.0 / (g.hz * g.hz) - c0);
  dim3 grd(N, (g.nz + zrun - 1) / zrun);
  if (smem > 65536)
    LRDM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&cheb_vec_kernel<TI, T, Q>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  ProfScope prof(ctx, scope);
  cheb_vec_kernel<TI, T, Q><<<grd, threads, smem, ctx->stream>>>(
      Yin, beta != 0.0 ? Yold : nullptr, Yout, Vt, g.nx, g.ny, g.nz, zrun, wx, wy, wz, dshift,
      T(alpha), T(beta));
  return hipGetLastError();
}

template <typename T, int S>
struct ChebCoef {
  T a[S], b[S];
};

// The whole filter of one state in one workgroup, for states that fit in LDS: Y_k
// of every point in LDS for the x and y neighbours, Y_k and Y_{k-1} of the
// thread's own points in registers, so that a state is read once and written once.
// Thread t owns group t % G of the plane on the ZP planes from (t / G) ZP (ZP divides nz; the z
// neighbours come from its own registers, across its ends from LDS).  Each element is
// formed as the single step forms it.  A step of 24^3 in FP64 takes a workgroup 9100 cycles:
// 3700 for the 34 bytes a point it moves through LDS, 2500 of FP64 instructions, the
// rest latency between its two barriers (3.5 waves a SIMD).  Degree 20: 32 states 147 -> 76 us,
// 256 states 295 -> 89 us (single steps before; one workgroup a state, so 32 states leave
// most of the chip idle).
constexpr int kLdsDegree = 64;     // steps one launch takes (coefficients by value)
template <typename T>
struct ChebCoefs {
  T a[kLdsDegree], b[kLdsDegree];
};

template <typename T, int ZP>
__global__ __launch_bounds__(1024) void cheb_lds_kernel(const T* __restrict__ X,
                                                       T* __restrict__ Y,
                                                       const T* __restrict__ Vt, int nx, int ny,
                                                       int nz, int degree, T wx, T wy,
                                                       T wz, T dshift, ChebCoefs<T> cf) {
  constexpr int W = 16 / sizeof(T);
  using V = vec_t<T, W>;
  extern __shared__ unsigned char smem_raw[];
  V* lds = reinterpret_cast<V*>(smem_raw);
  const int P = nx * ny, G = P / W, nxg = nx / W;
  const int gi = threadIdx.x % G, z0 = (int)(threadIdx.x / G) * ZP;
  const bool on = z0 < nz;
  const int y = gi / nxg, x0 = (gi - y * nxg) * W;
  const int gm = y == 0 ? gi + G - nxg : gi - nxg, gp = y == ny - 1 ? gi - G + nxg : gi + nxg;
  const int el = x0 == 0 ? W * gi + nx - 1 : W * gi - 1;
  const int er = x0 + W == nx ? W * gi + W - nx : W * gi + W;
  const int64_t base = (int64_t)blockIdx.x * G * nz;
  const V* in = reinterpret_cast<const V*>(X) + base;
  V* out = reinterpret_cast<V*>(Y) + base;
  using VU = typename Unaligned<T, W>::type;
  const VU* vg = reinterpret_cast<const VU*>(Vt);
  V cur[ZP], old[ZP];
#pragma unroll
  for (int j = 0; j < ZP; ++j) {
    cur[j] = old[j] = V(T(0));
    if (on) {
      cur[j] = in[(z0 + j) * G + gi];
      lds[(z0 + j) * G + gi] = cur[j];
    }
  }
  V vnext = on ? vg[z0 * G + gi] : V(T(0));   // V one plane ahead
  __syncthreads();
  for (int k = 0; k < degree; ++k) {
    const T alpha = cf.a[k], beta = cf.b[k];
    // an offset of zero the compiler does not know: the planes' addresses and V are
    // formed again in each step instead of being kept in (and spilled from) registers
    int again = 0;
    asm volatile("" : "+r"(again));
    const int p0 = (z0 + again) * G;
    if (on) {
      const V below = lds[(z0 == 0 ? nz - 1 : z0 - 1) * G + gi];
      const V above = lds[(z0 + ZP == nz ? 0 : z0 + ZP) * G + gi];
#pragma unroll
      for (int j = 0; j < ZP; ++j) {
        const V* pl = lds + p0 + j * G;
        const T* pls = reinterpret_cast<const T*>(pl);
        const V vv = vnext;
        vnext = vg[p0 + (j + 1 < ZP ? j + 1 : 0) * G + gi];
        const V ym = pl[gm], yp = pl[gp];
        const T left = pls[el], right = pls[er];
        const V c = cur[j], pz = j == 0 ? below : cur[j == 0 ? 0 : j - 1];
        const V nzv = j + 1 < ZP ? cur[j + 1 < ZP ? j + 1 : j] : above;
        const V o = old[j];
        V r;
#pragma unroll
        for (int e = 0; e < W; ++e) {
          const T xl = e == 0 ? left : c[e == 0 ? 0 : e - 1];
          const T xr = e == W - 1 ? right : c[e == W - 1 ? 0 : e + 1];
          const T hy = wx * (xl + xr) + wy * (ym[e] + yp[e]) + wz * (pz[e] + nzv[e]) +
                       (vv[e] + dshift) * c[e];
          r[e] = alpha * hy + beta * o[e];
        }
        old[j] = r;
        // one plane's neighbour values live at a time
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (k + 1 < degree) __syncthreads();     // every read of Y_k is done
#pragma unroll
    for (int j = 0; j < ZP; ++j) {
      const V r = old[j];
      old[j] = cur[j];
      cur[j] = r;
      if (on && k + 1 < degree) lds[p0 + j * G + gi] = r;
    }
    if (k + 1 < degree) __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < ZP; ++j)
    if (on) out[(z0 + j) * G + gi] = cur[j];
}

// S recurrence steps in one sweep over a run of z planes of one state, out of place:
// stage 0 is Y_k (Yb), stage -1 Y_{k-1} (Ya, NULL for k = 0: the first step has no
// Y_{k-1}), stage s = 1 .. S is Y_{k+s}, each element formed by the single step's
// operations (the compiler fuses the last sum the other way round, beta o rounded first, so
// that the outputs agree to rounding, not to the bit: held to one order the two-group form
// spills more and 24^3 through LDS takes 3 % longer).  Only the last two stages are written (stage S-1 to Yp, stage S to Yq; the next
// sweep's inputs), so S steps move 4 M N s bytes, plus 2 S halo planes a run.
// At iteration h stage s is formed on plane h - s: the plane above is stage s-1's
// newest value (formed in this iteration), its own plane and the one below are
// stage s-1's newest values of the last two iterations (registers, and LDS for the x
// and y neighbours), and Y of two steps before is stage s-2's value of two
// iterations ago.  LDS: [2 buffers][S stages][G groups]; a thread owns Q groups.
// HBM-bound up to S = 5 at 64 x 64 FP32 planes (the copy rate), so the stages are as
// many as registers and LDS allow.  The planes that close the period, or a run, are
// formed again at its other end instead of being kept, and the outputs go to buffers of
// their own: the registers hold more stages instead.  Measured (single steps, or three
// steps a sweep in place at 1024 states, before): 64^3, 1024 states, degree 40 FP32 11.9
// -> 7.2 ms (S = 5; S = 4 8.9, 3 12.2), FP64 49.3 -> 33.6 ms (S = 2); 48^3, 256 states,
// degree 30 FP64 4.20 -> 1.89 ms (S = 3), FP32 1.62 -> 0.64 ms; 40^3, 300 states FP64
// 2.91 -> 1.13 ms.
template <typename T, int S, int Q, int MAXT>
__global__ __launch_bounds__(MAXT) void cheb_sweep_kernel(const T* __restrict__ Ya,
                                                         const T* __restrict__ Yb,
                                                         T* __restrict__ Yp, T* __restrict__ Yq,
                                                         const T* __restrict__ Vt, int nx, int ny,
                                                         int nz, int zrun, T wx, T wy, T wz,
                                                         T dshift, ChebCoef<T, S> cf) {
  constexpr int W = 16 / sizeof(T);
  using V = vec_t<T, W>;
  extern __shared__ unsigned char smem_raw[];
  V* lds = reinterpret_cast<V*>(smem_raw);
  const int P = nx * ny, G = P / W, nxg = nx / W;
  const int z0 = blockIdx.y * zrun, z1 = min(nz, z0 + zrun);
  const int64_t base = (int64_t)blockIdx.x * G * nz;
  const V* A = Ya ? reinterpret_cast<const V*>(Ya) + base : nullptr;
  const V* B = reinterpret_cast<const V*>(Yb) + base;
  V* Op = reinterpret_cast<V*>(Yp) + base;
  V* Oq = reinterpret_cast<V*>(Yq) + base;
  using VU = typename Unaligned<T, W>::type;
  const VU* vg = reinterpret_cast<const VU*>(Vt);
  const V zero = V(T(0));
  auto wrap = [&](int z) { return z < 0 ? z + nz : (z >= nz ? z - nz : z); };
  bool on[Q];
  int gi[Q], gm[Q], gp[Q], el[Q], er[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    gi[q] = threadIdx.x + q * blockDim.x;
    on[q] = gi[q] < G;
    const int g = on[q] ? gi[q] : 0, y = g / nxg, x0 = (g - y * nxg) * W;
    gm[q] = y == 0 ? g + G - nxg : g - nxg;
    gp[q] = y == ny - 1 ? g - G + nxg : g + nxg;
    el[q] = x0 == 0 ? W * g + nx - 1 : W * g - 1;
    er[q] = x0 + W == nx ? W * g + W - nx : W * g + W;
  }
  // n1, n2[s]: stage s formed one and two iterations ago; vw[s]: V on plane h - s
  V n1[S][Q], n2[S][Q], vw[S + 1][Q], bn[Q], an[Q], vn[Q];
  const int h0 = z0 - S, h1 = z1 + S;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
#pragma unroll
    for (int s = 0; s < S; ++s) n1[s][q] = n2[s][q] = zero;
#pragma unroll
    for (int s = 0; s <= S; ++s) vw[s][q] = zero;
    an[q] = zero;
    bn[q] = on[q] ? B[(int64_t)wrap(h0) * G + gi[q]] : zero;
    vn[q] = on[q] ? vg[(int64_t)wrap(h0) * G + gi[q]] : zero;
  }
  for (int h = h0; h < h1; ++h) {
    const V* buf = lds + (h & 1) * S * G;
    V* nxt = lds + ((h + 1) & 1) * S * G;
    V b[Q], a[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
#pragma unroll
      for (int s = S; s > 0; --s) vw[s][q] = vw[s - 1][q];
      b[q] = bn[q];
      a[q] = an[q];
      vw[0][q] = vn[q];
      // operands of the next iteration, issued before this one's arithmetic
      if (on[q] && h + 1 < h1) {
        const int64_t zn = (int64_t)wrap(h + 1) * G + gi[q];
        bn[q] = B[zn];
        vn[q] = vg[zn];
        if (A) an[q] = A[(int64_t)wrap(h) * G + gi[q]];
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      V up = b[q], upup = zero;        // stages s-1 and s-2 formed in this iteration
#pragma unroll
      for (int s = 1; s <= S; ++s) {
        const int p = h - s;
        V val = zero;
        if (p >= z0 - (S - s) && p < z1 + (S - s) && on[q]) {
          const V* pl = buf + (s - 1) * G;
          const T* pls = reinterpret_cast<const T*>(pl);
          const V ym = pl[gm[q]], yp = pl[gp[q]];
          const T left = pls[el[q]], right = pls[er[q]];
          const V c = n1[s - 1][q], pz = n2[s - 1][q], vv = vw[s][q];
          const V o = s == 1 ? a[q] : n2[s >= 2 ? s - 2 : 0][q];
#pragma unroll
          for (int e = 0; e < W; ++e) {
            const T xl = e == 0 ? left : c[e == 0 ? 0 : e - 1];
            const T xr = e == W - 1 ? right : c[e == W - 1 ? 0 : e + 1];
            const T hy = wx * (xl + xr) + wy * (ym[e] + yp[e]) + wz * (pz[e] + up[e]) +
                         (vv[e] + dshift) * c[e];
            val[e] = cf.a[s - 1] * hy + cf.b[s - 1] * o[e];
          }
          if (p >= z0 && p < z1) {
            if (s == S - 1) Op[(int64_t)p * G + gi[q]] = val;
            if (s == S) Oq[(int64_t)p * G + gi[q]] = val;
          }
        }
        // stage s-2 is not needed any more as it stood
        if (s >= 2) {
          n2[s >= 2 ? s - 2 : 0][q] = n1[s >= 2 ? s - 2 : 0][q];
          n1[s >= 2 ? s - 2 : 0][q] = upup;
        }
        upup = up;
        up = val;
      }
      n2[S - 1][q] = n1[S - 1][q];
      n1[S - 1][q] = upup;
      if (on[q]) {
#pragma unroll
        for (int s = 0; s < S; ++s) nxt[s * G + gi[q]] = n1[s][q];
      }
    }
    __syncthreads();
  }
}

__global__ void convert_kernel(const double* __restrict__ a, int64_t n, float* __restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

}  // namespace

template <typename T>
bool cheb_vec_ok(const Grid3& g) {
  constexpr int W = 16 / sizeof(T);
  const int P = g.nx * g.ny;
  return g.nx % W == 0 && P / W <= 2 * 1024;
}

hipError_t launch_to_float(lrdm_ctx* ctx, const double* a, int64_t n, float* b) {
  convert_kernel<<<(unsigned)((n + 255) / 256), 256, 0, ctx->stream>>>(a, n, b);
  return hipGetLastError();
}

// ------------------------------------------------------------------ the filter
namespace {

constexpr int kLdsBytes = 160 * 1024;
constexpr int kCus = 256;

// z runs of a single step: enough blocks for the chip (N * runs >= ~1024) but runs of
// >= 8 planes.
int cheb_step_runs(const Grid3& g, int N) {
  int runs = 1;
  while ((int64_t)N * runs < 1024 && g.nz / (runs * 2) >= 8) runs *= 2;
  return runs;
}

// Planes a thread of cheb_lds_kernel owns (0: the state does not fit): nz over the
// largest divisor of nz that leaves at most 1024 threads, at most 8.
template <typename T>
int cheb_lds_planes(const Grid3& g, int degree) {
  constexpr int W = 16 / sizeof(T);
  if (degree > kLdsDegree || g.M * (int64_t)sizeof(T) > kLdsBytes) return 0;
  const int G = g.nx * g.ny / W;
  for (int zp = 1; zp <= 8; ++zp)
    if (g.nz % zp == 0 && (int64_t)G * (g.nz / zp) <= 1024) return zp;
  return 0;
}

// Groups per thread and stages of cheb_sweep_kernel: within the registers (one group:
// five stages at 1024 threads; two: three at 640, two at 1024, where more spill) and
// the LDS of two planes a stage.
template <typename T>
int cheb_sweep_stages(const Grid3& g) {
  constexpr int W = 16 / sizeof(T);
  const int P = g.nx * g.ny, G = P / W;
  if (G > 2048) return 0;
  const int regs = G <= 1024 ? 5 : (G <= 1280 ? 3 : 2);
  return std::min(regs, (int)(kLdsBytes / (2 * (int64_t)P * sizeof(T))));
}

}  // namespace

// The form of a filter: whole states in LDS; sweeps of up to S steps over batches of
// states; or one step at a time.  The sweeps keep three blocks of a batch beside Y,
// the single steps one block of N states; room: how many states of workspace there are
// (0: as many as wanted).  Times in microseconds from the rates measured on the sweep
// and the single step (19.5 bytes a nanosecond and CU, or 45 where the last-level cache
// holds a batch's four blocks; 0.11 ns a point and stage, half a microsecond a plane):
// the sweeps lose where halo planes outweigh the saved passes.  Against forced choices of
// stages and run at seventeen sizes of 7 to 20 planes and more, degree 20, the plan is within
// 8 % of the best from 128 states on; with few states up to 25 % off (64 x 64 x 12 in FP32, one
// state: 92 us against 74).  Whole states in LDS are taken wherever they fit.  From 128 states
// on they beat the best sweeps at every size (24^3 in FP64 81 us against 95, 256 states 89
// against 135; 32^3 in FP32 93 against 100), and small ones at any count (16^3 24 against 40,
// 24^3 in FP32 43 against 56); of the largest, up to some 60 states would go faster in sweeps
// (24^3 in FP64, 32 states, 78 against 58; 32^3 in FP32 87 against 66), which the rule leaves.
template <typename T>
ChebPlan cheb_plan(const Grid3& g, int N, int degree, int64_t room) {
  constexpr int W = 16 / sizeof(T);
  ChebPlan p{};
  if (!cheb_vec_ok<T>(g)) return p;
  // one step gains nothing from LDS: 24^3, 600 states in FP64 37 us against 22
  if (degree > 1 && cheb_lds_planes<T>(g, degree) > 0) {
    p.kind = ChebPlan::kLds;
    return p;
  }
  const double P = (double)g.nx * g.ny, block = (double)g.M * N * sizeof(T);
  // a single step takes as long as its longest run of planes however few the states
  const int step_planes = (g.nz + cheb_step_runs(g, N) - 1) / cheb_step_runs(g, N);
  double best = degree * std::max(3.0 * block / 4.9e6,
                                  2.0 + step_planes * (0.3 + 27e-6 * P * sizeof(T)));
  const int smax = std::min(degree, cheb_sweep_stages<T>(g));
  const int G = (int)(P / W), threads = G <= 1024 ? (G + 63) / 64 * 64 : ((G + 1) / 2 + 63) / 64 * 64;
  for (int S = 2; S <= smax; ++S) {
    if (g.nz < 2 * S) break;
    const int per_cu = std::max(1, std::min(1024 / threads, (int)(kLdsBytes / (2 * S * P * sizeof(T)))));
    const int slots = kCus * per_cu;
    int nb = std::min(N, slots);
    if (room > 0) nb = (int)std::min<int64_t>(nb, room / 3);
    if (nb < 1) continue;
    const int batches = (N + nb - 1) / nb;
    nb = (N + batches - 1) / batches;
    const int sweeps = (degree + S - 1) / S;
    for (int runs = 1; runs <= std::max(1, g.nz / 4); ++runs) {
      const int zrun = (g.nz + runs - 1) / runs;
      if ((g.nz + zrun - 1) / zrun != runs) continue;
      const int rounds = (nb * runs + slots - 1) / slots;
      const int share = std::min(per_cu, (nb * runs + kCus - 1) / kCus);
      const double rate = 4.0 * g.M * nb * sizeof(T) < 200e6 ? 45e3 : 19.5e3;
      const double plane = share * std::max(4.0 * P * sizeof(T) / rate, S * P * 0.11e-3) + 0.5;
      const double t = batches * sweeps * (rounds * (zrun + 2 * S) * plane + 4.0);
      if (t < best) {
        best = t;
        p.kind = ChebPlan::kSweeps;
        p.stages = S;
        p.batch = nb;
        p.zrun = zrun;
      }
    }
  }
  return p;
}
template ChebPlan cheb_plan<double>(const Grid3&, int, int, int64_t);
template ChebPlan cheb_plan<float>(const Grid3&, int, int, int64_t);

namespace {

template <typename T>
struct StencilCoef {
  T wx, wy, wz, dshift;
  StencilCoef(const Grid3& g, double c0)
      : wx(T(-0.5 / (g.hx * g.hx))), wy(T(-0.5 / (g.hy * g.hy))), wz(T(-0.5 / (g.hz * g.hz))),
        dshift(T(1.0 / (g.hx * g.hx) + 1.0 / (g.hy * g.hy) + 1.0 / (g.hz * g.hz) - c0)) {}
};

template <typename T, int ZP>
hipError_t launch_lds(lrdm_ctx* ctx, const Grid3& g, const T* Vt, const T* X, T* Y, int N,
                      int degree, double c0, const ChebCoefs<T>& cf) {
  const int G = g.nx * g.ny / (int)(16 / sizeof(T));
  const int threads = (G * (g.nz / ZP) + 63) / 64 * 64;
  const int smem = (int)(g.M * sizeof(T));
  const StencilCoef<T> k(g, c0);
  if (smem > 65536)
    LRDM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&cheb_lds_kernel<T, ZP>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, smem));
  ProfScope prof(ctx, "cheb_lds");
  cheb_lds_kernel<T, ZP><<<N, threads, smem, ctx->stream>>>(X, Y, Vt, g.nx, g.ny, g.nz, degree,
                                                            k.wx, k.wy, k.wz, k.dshift, cf);
  return hipGetLastError();
}

template <typename T, int S, int Q, int MAXT>
hipError_t launch_sweep_q(lrdm_ctx* ctx, const Grid3& g, const T* Vt, const T* Ya, const T* Yb,
                          T* Yp, T* Yq, int N, int zrun, double c0, const double* a,
                          const double* b) {
  const int P = g.nx * g.ny, G = P / (int)(16 / sizeof(T));
  const int threads = ((G + Q - 1) / Q + 63) / 64 * 64;
  const int smem = 2 * S * P * (int)sizeof(T);
  const StencilCoef<T> k(g, c0);
  ChebCoef<T, S> cf;
  for (int s = 0; s < S; ++s) {
    cf.a[s] = T(a[s]);
    cf.b[s] = T(b[s]);
  }
  if (smem > 65536)
    LRDM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&cheb_sweep_kernel<T, S, Q, MAXT>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, smem));
  ProfScope prof(ctx, "cheb_sweep");
  cheb_sweep_kernel<T, S, Q, MAXT><<<dim3(N, (g.nz + zrun - 1) / zrun), threads, smem,
                                     ctx->stream>>>(Ya, Yb, Yp, Yq, Vt, g.nx, g.ny, g.nz, zrun,
                                                    k.wx, k.wy, k.wz, k.dshift, cf);
  return hipGetLastError();
}

template <typename T, int S>
hipError_t launch_sweep_s(lrdm_ctx* ctx, const Grid3& g, const T* Vt, const T* Ya, const T* Yb,
                          T* Yp, T* Yq, int N, int zrun, double c0, const double* a,
                          const double* b) {
  const int G = g.nx * g.ny / (int)(16 / sizeof(T));
  if (G <= 1024)
    return launch_sweep_q<T, S, 1, 1024>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
  if constexpr (S <= 3)
    if (G <= 1280)
      return launch_sweep_q<T, S, 2, 640>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
  if constexpr (S <= 2)
    return launch_sweep_q<T, S, 2, 1024>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_sweep(lrdm_ctx* ctx, int S, const Grid3& g, const T* Vt, const T* Ya,
                        const T* Yb, T* Yp, T* Yq, int N, int zrun, double c0, const double* a,
                        const double* b) {
  switch (S) {
    case 1: return launch_sweep_s<T, 1>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
    case 2: return launch_sweep_s<T, 2>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
    case 3: return launch_sweep_s<T, 3>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
    case 4: return launch_sweep_s<T, 4>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
    case 5: return launch_sweep_s<T, 5>(ctx, g, Vt, Ya, Yb, Yp, Yq, N, zrun, c0, a, b);
  }
  return hipErrorInvalidValue;
}

}  // namespace

template <typename T>
hipError_t launch_cheb_lds(lrdm_ctx* ctx, const Grid3& g, const T* Vt, const T* X, T* Y, int N,
                           double c0, const std::vector<double>& a, const std::vector<double>& b) {
  const int degree = (int)a.size();
  ChebCoefs<T> cf{};
  for (int k = 0; k < degree; ++k) {
    cf.a[k] = T(a[k]);
    cf.b[k] = T(b[k]);
  }
  switch (cheb_lds_planes<T>(g, degree)) {
    case 1: return launch_lds<T, 1>(ctx, g, Vt, X, Y, N, degree, c0, cf);
    case 2: return launch_lds<T, 2>(ctx, g, Vt, X, Y, N, degree, c0, cf);
    case 3: return launch_lds<T, 3>(ctx, g, Vt, X, Y, N, degree, c0, cf);
    case 4: return launch_lds<T, 4>(ctx, g, Vt, X, Y, N, degree, c0, cf);
    case 5: return launch_lds<T, 5>(ctx, g, Vt, X, Y, N, degree, c0, cf);
    case 6: return launch_lds<T, 6>(ctx, g, Vt, X, Y, N, degree, c0, cf);
    case 7: return launch_lds<T, 7>(ctx, g, Vt, X, Y, N, degree, c0, cf);
    case 8: return launch_lds<T, 8>(ctx, g, Vt, X, Y, N, degree, c0, cf);
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_cheb_lds<double>(lrdm_ctx*, const Grid3&, const double*, const double*,
                                            double*, int, double, const std::vector<double>&,
                                            const std::vector<double>&);
template hipError_t launch_cheb_lds<float>(lrdm_ctx*, const Grid3&, const float*, const float*,
                                           float*, int, double, const std::vector<double>&,
                                           const std::vector<double>&);

template <typename T>
hipError_t launch_cheb_sweeps(lrdm_ctx* ctx, const ChebPlan& p, const Grid3& g, const T* Vt,
                              const T* X, T* Y, T* W, int N, double c0,
                              const std::vector<double>& a, const std::vector<double>& b) {
  const int degree = (int)a.size();
  // sweeps of even length; a sweep of one step (it writes no Y_{k+S-1}) comes last
  const int n = (degree + p.stages - 1) / p.stages, least = degree / n, more = degree % n;
  const int64_t blk = g.M * p.batch;
  for (int i0 = 0; i0 < N; i0 += p.batch) {
    const int nb = std::min(p.batch, N - i0);
    const T* x = X + g.M * i0;
    // sweeps write the pairs {W0, Y} and {W1, W2} in turn, the last one the pair of Y
    T* pair[2][2] = {{W, Y + g.M * i0}, {W + blk, W + 2 * blk}};
    int to = n % 2 ? 0 : 1, k = 0;
    const T *ya = nullptr, *yb = x;
    for (int s = 0; s < n; ++s) {
      const int S = least + (s < more ? 1 : 0);
      LRDM_HIP(launch_sweep<T>(ctx, S, g, Vt, ya, yb, pair[to][0], pair[to][1], nb, p.zrun, c0,
                               &a[k], &b[k]));
      ya = pair[to][0];
      yb = pair[to][1];
      to ^= 1;
      k += S;
    }
  }
  return hipSuccess;
}
template hipError_t launch_cheb_sweeps<double>(lrdm_ctx*, const ChebPlan&, const Grid3&,
                                               const double*, const double*, double*, double*, int,
                                               double, const std::vector<double>&,
                                               const std::vector<double>&);
template hipError_t launch_cheb_sweeps<float>(lrdm_ctx*, const ChebPlan&, const Grid3&,
                                              const float*, const float*, float*, float*, int,
                                              double, const std::vector<double>&,
                                              const std::vector<double>&);

template <typename T>
hipError_t launch_cheb_step_vec(lrdm_ctx* ctx, const Grid3& g, const T* Vt, const T* Yin,
                                const T* Yold, T* Yout, int N, double alpha, double c0,
                                double beta) {
  constexpr int W = 16 / sizeof(T);
  const int G = g.nx * g.ny / W;
  if (!cheb_vec_ok<T>(g)) return hipErrorInvalidValue;
  const int threads = G <= 1024 ? ((G + 63) / 64) * 64 : 1024;
  const int runs = cheb_step_runs(g, N);
  const int zrun = (g.nz + runs - 1) / runs;
  if (G <= threads)
    return launch_vec<T, T, 1>(ctx, "cheb_step", g, Vt, Yin, Yold, Yout, N, threads, zrun, alpha,
                               c0, beta);
  return launch_vec<T, T, 2>(ctx, "cheb_step", g, Vt, Yin, Yold, Yout, N, threads, zrun, alpha,
                             c0, beta);
}

template bool cheb_vec_ok<double>(const Grid3&);
template bool cheb_vec_ok<float>(const Grid3&);
template hipError_t launch_cheb_step_vec<double>(lrdm_ctx*, const Grid3&, const double*,
                                                 const double*, const double*, double*, int,
                                                 double, double, double);
template hipError_t launch_cheb_step_vec<float>(lrdm_ctx*, const Grid3&, const float*,
                                                const float*, const float*, float*, int, double,
                                                double, double);


template <typename T>
hipError_t launch_cheb_step(lrdm_ctx* ctx, const Grid3& g, const double* V, const T* Yin,
                            const T* Yold, T* Yout, int N, double alpha, double c0, double beta) {
  return launch_stencil<T, T>(ctx, g, V, Yin, Yold, Yout, N, alpha, c0, beta);
}

template <typename T>
hipError_t launch_hpsi_f64(lrdm_ctx* ctx, const Grid3& g, const double* V, const T* Y, double* HY,
                           int N) {
  constexpr int W = 16 / sizeof(T);
  auto aligned = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  const int G = g.nx * g.ny / W;
  if (cheb_vec_ok<T>(g) && G <= 1024 && aligned(Y) && aligned(HY) && aligned(V)) {
    const int threads = ((G + 63) / 64) * 64;
    int runs = 1;
    while ((int64_t)N * runs < 1024 && g.nz / (runs * 2) >= 8) runs *= 2;
    const int zrun = (g.nz + runs - 1) / runs;
    return launch_vec<T, double, 1>(ctx, "hpsi", g, V, Y, nullptr, HY, N, threads, zrun, 1.0, 0.0,
                                    0.0);
  }
  return launch_stencil<T, double>(ctx, g, V, Y, nullptr, HY, N, 1.0, 0.0, 0.0);
}

template hipError_t launch_cheb_step<double>(lrdm_ctx*, const Grid3&, const double*, const double*,
                                             const double*, double*, int, double, double, double);
template hipError_t launch_cheb_step<float>(lrdm_ctx*, const Grid3&, const double*, const float*,
                                            const float*, float*, int, double, double, double);
template hipError_t launch_hpsi_f64<double>(lrdm_ctx*, const Grid3&, const double*, const double*,
                                            double*, int);
template hipError_t launch_hpsi_f64<float>(lrdm_ctx*, const Grid3&, const double*, const float*,
                                           double*, int);

}  // namespace lrdm
