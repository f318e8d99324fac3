// The FP64 back-projection out[b][p] = scale sum_ij G_b[i][j] A_i[p] A_j[p] - sub
// for few states, on strips of 16 rows (the meaning of backproj_f64_kernel in
// gemm.hip, which takes 128-row blocks: 96 states cost it 128 x 96 products a point
// where the triangle of strips holds 96 x 112 / 2).
//
// A workgroup owns 32 points and holds every state at them in LDS, so that a state
// is read once per group of directions, as the right operand of the matrix cores and
// again as the rows that the products (G A)[i][p] are dotted with.  Its waves
// share the strips; G comes 16 x 16 at a time from the caches, two blocks ahead, and
// each such block serves 32 points.  What holds it is the latency of those reads and
// the waves a CU has room for: 64 points a workgroup halve the reads and were slower on
// every shape but one (48^3, 256 states, 8 directions: 1539 us against 1374), one block
// ahead and addresses per lane took 1.45x as long.
//
// Measured against backproj_f64_kernel: 24^3, 32 states, 4 directions 22 -> 11 us;
// 36 x 40 x 32, 96 states, 8 matrices 255 -> 117; 48^3, 256 states, 8 directions
// 2004 -> 1370 (42 TFLOP/s of the triangle's products); 40^3, 384 states, 20 directions
// 5825 -> 4631; 48^3, 512 states, 4 directions 2986 -> 2673.  Past 512 states the points
// of a workgroup no longer fit LDS.
#include <algorithm>

#include "blocks.h"
#include "lrdm_internal.h"

namespace lrdm {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kStrip = 16;

constexpr int NP = 2;            // 16-point groups of a workgroup
constexpr int P = kStrip * NP;

// 1-D grid over (group of directions, channel, P points).
__global__ __launch_bounds__(1024, 4) void backproj_direct_kernel(
    const double* __restrict__ A, const double* __restrict__ G, int N, int64_t M, int nspin,
    int dirs, int per_group, int pblocks, double scale, const double* __restrict__ sub,
    const unsigned char* __restrict__ active, double* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_direct[];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int col = lane & 15, g = lane >> 4;
  const int grp = blockIdx.x / pblocks;
  const int c = grp % nspin, d0 = grp / nspin * per_group;
  const int d1 = min(dirs, d0 + per_group);
  const int64_t p0 = (int64_t)(blockIdx.x % pblocks) * P;
  const int ntb = (N + kBlockEdge - 1) / kBlockEdge;
  const int nst = (N + kStrip - 1) / kStrip;
  // [16 nst][P], zero past N and M; odd rows with neighbouring 16 points exchanged, so
  // that the rows a half-wave reads lie in different banks
  double* const As = reinterpret_cast<double*>(smem_direct);
  double* const red = As + nst * kStrip * P;    // [2][waves][P]
  const double* Ac = A + (int64_t)c * N * M;
  for (int e = threadIdx.x; e < nst * kStrip * P; e += blockDim.x) {
    const int row = e / P;
    const int64_t p = p0 + e % P;
    As[e ^ (row & 1) * kStrip] = row < N && p < M ? Ac[(int64_t)row * M + p] : 0.0;
  }
  __syncthreads();
  const double* const even = As + g * P + col + (g & 1) * kStrip;
  const double* const odd = As + g * P + col + kStrip - (g & 1) * kStrip;
  // row 4 t + g of strip jb at the lane's points of 16-point group q
  auto at = [&](int jb, int t, int q) {
    return (q & 1 ? odd : even)[(kStrip * jb + 4 * t) * P + (q & ~1) * kStrip];
  };
  const uint32_t off = g * N + col;
  const int full = N / kStrip;   // strips before the short one
  for (int d = d0; d < d1; ++d) {
    const int b = d * nspin + c;
    const double* Gb = G + (int64_t)b * N * N;
    // entries (j, i) of G, j = 16 jb + 4 t + g and i = 16 ib + col; zero past N
    auto load = [&](int ib, int jb, double (&x)[4]) {
      if (max(ib, jb) < full) {
        const double* blk = Gb + (int64_t)kStrip * jb * N + kStrip * ib;
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = (blk + (int64_t)4 * t * N)[off];
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int j = kStrip * jb + 4 * t + g, i = kStrip * ib + col;
          const double v = Gb[(int64_t)min(j, N - 1) * N + min(i, N - 1)];
          x[t] = j < N && i < N ? v : 0.0;
        }
      }
    };
    double sum[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) sum[q] = 0.0;
    // the strips in turn to and fro over the waves, so that long and short ones mix;
    // another wave begins in each direction
    const int first = __builtin_amdgcn_readfirstlane((wid + d) % waves);
    for (int k = 0;; ++k) {
      const int ib = k * waves + (k & 1 ? waves - 1 - first : first);
      if (k * waves >= nst) break;
      if (ib >= nst) continue;
      const int I = ib * kStrip / kBlockEdge;
      d4 acc[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) acc[q] = d4{0.0, 0.0, 0.0, 0.0};
      // strips right of the diagonal count twice (G symmetric): they come first and are
      // doubled with the accumulator; inactive blocks (blocks.h) are left out
      for (int J = ntb - 1; J >= I; --J) {
        const bool on = block_active(active, c, ntb, I, J);
        const int lo = J == I ? ib : J * (kBlockEdge / kStrip);
        const int hi = min(nst, (J + 1) * (kBlockEdge / kStrip));
        double x[4], nx[4], ny[4];
        if (on) {
          load(ib, hi - 1, x);
          load(ib, max(hi - 2, lo), nx);
        }
        for (int jb = hi - 1; on && jb >= lo; --jb) {
          load(ib, max(jb - 2, lo), ny);
          if (jb == ib) {
#pragma unroll
            for (int q = 0; q < NP; ++q) acc[q] *= 2.0;
          }
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < NP; ++q)
              acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t], at(jb, t, q), acc[q], 0, 0, 0);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            x[t] = nx[t];
            nx[t] = ny[t];
          }
        }
        if (J == I && !on) {   // no strip on the diagonal came to double the others
#pragma unroll
          for (int q = 0; q < NP; ++q) acc[q] *= 2.0;
        }
      }
#pragma unroll
      for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          sum[q] = fma(acc[q][v], at(ib, v, q), sum[q]);
    }
    double* const r = red + ((d - d0) & 1) * (waves * P);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      sum[q] += __shfl_xor(sum[q], 16, 64);
      sum[q] += __shfl_xor(sum[q], 32, 64);
      if (g == 0) r[wid * P + kStrip * q + col] = sum[q];
    }
    // the buffer of direction d is written again after the barrier of d + 1 only
    __syncthreads();
    const int64_t p = p0 + threadIdx.x;
    if (threadIdx.x < P && p < M) {
      double v = 0.0;
      for (int k = 0; k < waves; ++k) v += r[k * P + threadIdx.x];
      v *= scale;
      if (sub) v -= sub[(int64_t)b * M + p];
      out[(int64_t)b * M + p] = v;
    }
  }
}

}  // namespace

bool backproj_direct_ok(int N) { return N <= 512; }

hipError_t launch_backproj_direct(lrdm_ctx* ctx, const double* A, const double* G, int N,
                                  int64_t M, int nspin, int batch, double scale,
                                  const double* sub, double* out, const unsigned char* active) {
  const int dirs = batch / nspin;
  // as many waves as there are pairs of strips, while the states of several workgroups fit
  // a CU's LDS; 96 states with 4 or 8 waves take 117 and 154 us, 256 states with 4, 8
  // or 16 take 1630, 1375 and 1792, 384 with 8 or 16 take 5280 and 4631
  const int waves = N <= 32 ? 2 : N <= 160 ? 4 : N <= 256 ? 8 : 16;
  const int pblocks = (int)((M + P - 1) / P);
  // directions that share the states in LDS, as many as leave four workgroups a CU
  const int per = (int)std::min<int64_t>(
      dirs, std::max<int64_t>(1, (int64_t)pblocks * batch / 1024));
  const int groups = (dirs + per - 1) / per;
  const size_t lds =
      (size_t)((N + kStrip - 1) / kStrip * kStrip + 2 * waves) * P * sizeof(double);
  if (lds > 65536)
    LRDM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&backproj_direct_kernel),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  ProfScope prof(ctx, "backproj");
  backproj_direct_kernel<<<(unsigned)(groups * nspin * pblocks), 64 * waves, lds, ctx->stream>>>(
      A, G, N, M, nspin, dirs, per, pblocks, scale, sub, active, out);
  return hipGetLastError();
}

}  // namespace lrdm
