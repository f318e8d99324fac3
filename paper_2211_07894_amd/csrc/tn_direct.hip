// The FP64 projection H[b] = A diag(w_b) B^T over the grid index on tiles of 32
// and 64 rows (the meaning, split-K partials and determinism of tn_sym_f64_kernel in
// gemm.hip).
//
// A contraction over K = M points has few output tiles when N is small or the
// directions are few, so the chip is filled along K: a workgroup owns one tile and
// one range of points, and its four waves interleave over the range, each holding the
// whole tile in registers; the four partial tiles meet in LDS at the end.  The
// operands go from global memory straight into the registers the matrix cores read:
// lane l supplies row l % 16 of each 16-row strip at E consecutive points of the
// step (any order of the points is allowed as long as A and B use the same one), so
// there is no LDS traffic and no barrier inside the loop, and the next step's reads
// are in flight during the current step's products.  On a tile of the diagonal A
// and B are the same rows: they are read once, and only the strips i <= j are formed.
//
// Measured against tn_sym_f64_kernel (128-row tiles, at least 4096 points a range):
// 24^3, 32 states, 4 directions 1127 -> 16 us; 27 x 33 x 35, 90 states, 2 channels
// 1356 -> 46 us; 48^3, 256 states, Gram product 1170 -> 207 us (35 TFLOP/s), 8
// directions 1790 -> 1234 us (47 TFLOP/s); 40^3, 384 states, 20 directions 4070 -> 3980 us;
// 48^3, 512 states, 8 matrices 4740 -> 5520 us.  What holds it there is the loads: a
// 64-row tile needs twice the bytes of a 128-row one per product, and the reads of 16 rows
// of different pages per instruction arrive at about 10 bytes a clock and CU (48^3, 256
// states, 8 directions: 7.2 GB asked for, 2.9 GB of it past L2, in 1234 us).
#include <algorithm>

#include "blocks.h"
#include "lrdm_internal.h"
#include "xcd.h"

namespace lrdm {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int KW = 4;        // waves of a workgroup, interleaved over the steps

// E points of one row, at any address a row element can have.
template <typename S, int E>
struct __attribute__((packed, aligned(sizeof(S)))) Pack {
  S v[E];
};

// Points a lane takes per row and step: two on 64-row tiles (with four, both buffers and
// the accumulators pass 256 registers, and with them the second wave of each SIMD),
// four on 32-row ones.
constexpr int lane_points(int T) { return T == 64 ? 2 : 4; }

// One step's operands of a lane.
template <typename SA, typename SB, int R, int E>
struct StepRegs {
  Pack<SA, E> a[R];
  Pack<SB, E> b[R];
  Pack<double, E> w;
};

// acc += the step's products; DIAG: the tile lies on the diagonal (B = A, strips i <= j).
template <typename SA, typename SB, int R, int E, bool W, bool DIAG>
__device__ inline void step_products(const StepRegs<SA, SB, R, E>& s, d4 (&acc)[R][R]) {
#pragma unroll
  for (int e = 0; e < E; ++e) {
    double a[R], b[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      a[i] = (double)s.a[i].v[e];
      b[i] = DIAG ? a[i] : (double)s.b[i].v[e];
      if (W) b[i] *= s.w.v[e];
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = DIAG ? i : 0; j < R; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
  }
}

// The wave's steps of [kbeg, kend): full ones with the next step's reads in flight,
// then the range's last, partial step (zeros past its end).
template <typename SA, typename SB, int R, int E, bool W, bool DIAG>
__device__ inline void wave_range(const SA* const (&ra)[R], const SB* const (&rb)[R],
                                  const double* wb, int64_t kbeg, int64_t kend, int wid, int g,
                                  d4 (&acc)[R][R]) {
  constexpr int KS = 4 * E, STRIDE = KS * KW;
  StepRegs<SA, SB, R, E> cur, nxt;
  auto load = [&](int64_t k, StepRegs<SA, SB, R, E>& s) {
#pragma unroll
    for (int i = 0; i < R; ++i) s.a[i] = *reinterpret_cast<const Pack<SA, E>*>(ra[i] + k);
    if (!DIAG) {
#pragma unroll
      for (int i = 0; i < R; ++i) s.b[i] = *reinterpret_cast<const Pack<SB, E>*>(rb[i] + k);
    }
    if (W) s.w = *reinterpret_cast<const Pack<double, E>*>(wb + k);
  };
  int64_t k = kbeg + KS * wid;
  if (k + KS <= kend) load(k, cur);
  for (; k + KS <= kend; k += STRIDE) {
    if (k + STRIDE + KS <= kend) load(k + STRIDE, nxt);
    step_products<SA, SB, R, E, W, DIAG>(cur, acc);
    cur = nxt;
  }
  if (k < kend) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool in = k + E * g + e < kend;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        cur.a[i].v[e] = in ? ra[i][k + e] : SA(0);
        if (!DIAG) cur.b[i].v[e] = in ? rb[i][k + e] : SB(0);
      }
      if (W) cur.w.v[e] = in ? wb[k + e] : 0.0;
    }
    step_products<SA, SB, R, E, W, DIAG>(cur, acc);
  }
}

template <typename SA, typename SB, int T, bool W>
__global__ __launch_bounds__(64 * KW, 2) void tn_direct_kernel(
    const SA* __restrict__ A, const SB* __restrict__ B, const double* __restrict__ w,
    int64_t w_stride, int N, int64_t M, int nspin, int nt, int64_t kchunk, int nsplit, int batch,
    const unsigned char* __restrict__ active, int same, double* __restrict__ part) {
  constexpr int R = T / 16;
  constexpr int E = lane_points(T);
  __shared__ double red[2][T * T];
  const int ntiles = nt * (nt + 1) / 2;
  // every tile and direction of one range of points on one XCD: they read the
  // same points of Psi
  int sp, item;
  xcd_map(blockIdx.x, nsplit, ntiles * batch, sp, item);
  const int tile = item % ntiles, b = item / ntiles;
  int ti = 0, rem = tile;
  while (rem >= nt - ti) { rem -= nt - ti; ++ti; }
  const int tj = ti + rem;
  const int c = b % nspin;
  const int64_t kbeg = (int64_t)sp * kchunk;
  // an inactive block (blocks.h) keeps a zero partial tile
  const int nb = (N + kBlockEdge - 1) / kBlockEdge;
  const bool on = block_active(active, c, nb, ti * T / kBlockEdge, tj * T / kBlockEdge);
  const int64_t kend = on ? min(M, kbeg + kchunk) : kbeg;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  // rows past N read row N - 1: their products are never read
  const SA* ra[R];
  const SB* rb[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    ra[i] = A + ((int64_t)c * N + min(ti * T + 16 * i + li, N - 1)) * M + E * g;
    rb[i] = B + ((int64_t)c * N + min(tj * T + 16 * i + li, N - 1)) * M + E * g;
  }
  const double* wb = W ? w + (int64_t)b * w_stride + E * g : nullptr;
  d4 acc[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  if (same && ti == tj)
    wave_range<SA, SB, R, E, W, true>(ra, rb, wb, kbeg, kend, wid, g, acc);
  else
    wave_range<SA, SB, R, E, W, false>(ra, rb, wb, kbeg, kend, wid, g, acc);
  // the four waves' tiles in a fixed order: (0 + 2) + (1 + 3)
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) f((16 * i + 4 * v + g) * T + 16 * j + li, i, j, v);
  };
  if (wid >= 2) each([&](int o, int i, int j, int v) { red[wid - 2][o] = acc[i][j][v]; });
  __syncthreads();
  if (wid < 2) each([&](int o, int i, int j, int v) { acc[i][j][v] += red[wid][o]; });
  __syncthreads();
  if (wid == 1) each([&](int o, int i, int j, int v) { red[0][o] = acc[i][j][v]; });
  __syncthreads();
  if (wid == 0) {
    double* out = part + (((int64_t)b * nsplit + sp) * ntiles + tile) * (T * T);
    each([&](int o, int i, int j, int v) { out[o] = acc[i][j][v] + red[0][o]; });
  }
}

}  // namespace

int tn_direct_tile(int N) { return N <= 32 ? 32 : 64; }

// Up to 384 states the 64-row tiles win at any size (no padding to 128 rows), but for the
// last 16, which 128-row tiles pad little, where rows are a multiple of 2 MB apart and the
// 16 that a load reads fall together (384 states, 64^3: 1 direction 1028 us against 1228, 2
// 1961 against 2001, 4 3747 against 3616, 16 14516 against 13750; 60^3, 16 directions 9886
// against 10511; 368 states, 64^3, 16 directions 13823 against 13835); beyond, only where
// 128-row tiles and ranges of 4096 points leave workgroup slots of the chip (two per CU)
// empty.
bool tn_direct_ok(int N, int64_t M, int batch) {
  if (N <= 368) return true;
  const int nt = (N + kBlockEdge - 1) / kBlockEdge;
  const int items = nt * (nt + 1) / 2 * batch;
  const int64_t wgs = (int64_t)items * tn_splits(items, M);
  return N <= 384 ? wgs < 1024 || M % (1 << 18) != 0 : wgs < 384;
}

// 64 ranges of points (of at least 192 points): at 48^3 and 256 states 32, 64 and 128
// ranges take 280, 207 and 204 us, with 8 directions 1234, 1250 and 1236 us, at 27 x 33
// x 35 and 90 states 53, 46 and 52 us.
static int tn_direct_ranges(int64_t M) { return (int)std::max<int64_t>(1, std::min<int64_t>(64, M / 192)); }

size_t tn_direct_bytes(int N, int64_t M, int batch) {
  if (!tn_direct_ok(N, M, batch)) return 0;
  const int T = tn_direct_tile(N), nt = (N + T - 1) / T;
  const size_t range = (size_t)nt * (nt + 1) / 2 * batch * T * T * sizeof(double);
  return std::min<size_t>(range * tn_direct_ranges(M), (size_t)96 << 20);
}

TnDirectPlan tn_direct_plan(int N, int64_t M, int batch, size_t budget, double scale) {
  TnDirectPlan p;
  p.tile = tn_direct_tile(N);
  const int nt = (N + p.tile - 1) / p.tile;
  const size_t range = (size_t)nt * (nt + 1) / 2 * batch * p.tile * p.tile * sizeof(double);
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>(budget / range, (M + 63) / 64));
  p.nsplit = (int)std::min<int64_t>(
      most, std::max<int64_t>(1, (int64_t)(tn_direct_ranges(M) * scale + 0.5)));
  // whole groups of ranges per XCD where there are enough (xcd.h)
  if (p.nsplit > kXcds) p.nsplit = p.nsplit / kXcds * kXcds;
  const int64_t step = 16 * KW;
  p.kchunk = ((M + p.nsplit - 1) / p.nsplit + step - 1) / step * step;
  return p;
}

template <typename SA, typename SB>
hipError_t launch_tn_direct(lrdm_ctx* ctx, const TnDirectPlan& p, const SA* A, const SB* B,
                            const double* w, int64_t w_stride, int N, int64_t M, int nspin,
                            int batch, double* part, double* H, const unsigned char* active,
                            bool same) {
  const int nt = (N + p.tile - 1) / p.tile;
  const unsigned grd = (unsigned)(nt * (nt + 1) / 2 * p.nsplit * batch);
  auto go = [&](auto kernel) {
    kernel<<<grd, 64 * KW, 0, ctx->stream>>>(A, B, w, w_stride, N, M, nspin, nt, p.kchunk,
                                             p.nsplit, batch, active, same ? 1 : 0, part);
  };
  {
    ProfScope prof(ctx, w ? "proj" : "gram");
    if (p.tile == 32) {
      if (w) go(tn_direct_kernel<SA, SB, 32, true>);
      else go(tn_direct_kernel<SA, SB, 32, false>);
    } else {
      if (w) go(tn_direct_kernel<SA, SB, 64, true>);
      else go(tn_direct_kernel<SA, SB, 64, false>);
    }
    LRDM_HIP(hipGetLastError());
  }
  return launch_tn_reduce(ctx, part, N, p.tile, p.nsplit, batch, H);
}
template hipError_t launch_tn_direct<double, double>(lrdm_ctx*, const TnDirectPlan&,
                                                     const double*, const double*, const double*,
                                                     int64_t, int, int64_t, int, int, double*,
                                                     double*, const unsigned char*, bool);

}  // namespace lrdm
