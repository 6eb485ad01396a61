// usp_moments.hip -- per-cell moments and the per-cell USP-FPM state.
#include "usp_cell.h"

namespace usp {

constexpr int CELL_BLOCK = 256;

// 16 lanes per cell, four cells per wave (every lane stays active for the
// row permutes; lanes of cells past M carry zeros).
template <typename S, bool G>
__global__ __launch_bounds__(CELL_BLOCK) void k_moments(GridP g, PartP<S> p, const int64_t* offsets,
                                                        double* mom, const uint32_t* perm) {
  const int64_t M = g.M;
  const int64_t c = ((int64_t)blockIdx.x * CELL_BLOCK + threadIdx.x) / MOM_LANES;
  const int sub = threadIdx.x & (MOM_LANES - 1);
  const bool valid = c < M;
  const int64_t o0 = valid ? offsets[c] : 0, o1 = valid ? offsets[c + 1] : 0;
  double v[NMOM];
  row_moments<S, G>(p.cx, p.cy, p.cz, p.erot, p.vib, o0, o1, sub, v, perm);
  if (valid) store_moments(mom, M, c, sub, v);
}

// On grids of few cells 16 lanes a cell leave the chip idle: a workgroup of
// WAVES waves takes a cell (lane i of it the particles i, i + 64 WAVES, ...),
// the waves' sums are added in wave order, and with `state` one lane goes on
// to the cell state (a serial chain of some 8 us, for all cells at once),
// which saves its launch.  200 cells of 1000 particles: 22 + 10 us for the
// two kernels before, 12 together; 0.7M FP64 particles in 1800 cells: the
// moments 38 -> 18 us.
template <typename S, bool G, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_moments_wide(GridP g, GasP gas, PartP<S> p,
                                                             const int64_t* __restrict__ offsets,
                                                             double* mom,
                                                             const uint32_t* __restrict__ perm,
                                                             double dt, const double* dt_cell,
                                                             double* cs, int64_t* counters,
                                                             int state) {
  __shared__ double part[WAVES][20];
  const int64_t M = g.M, c = blockIdx.x;
  const int64_t o0 = offsets[c], o1 = offsets[c + 1], N = o1 - o0;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  auto at = [&](int64_t i) -> int64_t {
    if constexpr (G) return (int64_t)perm[i];
    else return i;
  };
  double r0 = 0.0, r1 = 0.0, r2 = 0.0;
  if (N > 0) {
    const int64_t j = at(o0);
    r0 = (double)p.cx[j]; r1 = (double)p.cy[j]; r2 = (double)p.cz[j];
  }
  double s[20];
#pragma unroll
  for (int k = 0; k < 20; ++k) s[k] = 0.0;
  constexpr int STEP = 64 * WAVES;
  for (int64_t b = o0 + threadIdx.x; b < o1; b += 4 * STEP) {
    // four slots' loads in flight (a slot past the cell reads the first)
    int64_t j[4];
    MomIn<S> a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) j[u] = at(b + u * STEP < o1 ? b + u * STEP : o0);
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = mom_load<S>(p.cx, p.cy, p.cz, p.erot, p.vib, j[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (b + u * STEP < o1) mom_add(a[u], r0, r1, r2, s);
  }
#pragma unroll
  for (int k = 0; k < 20; ++k) s[k] = wave_sum(s[k]);
  if constexpr (WAVES > 1) {
    if (lane < 20) {
      double w = 0.0;
#pragma unroll
      for (int k = 0; k < 20; ++k)
        if (k == lane) w = s[k];
      part[wid][lane] = w;
    }
    __syncthreads();
    if (wid != 0) return;
#pragma unroll
    for (int k = 0; k < 20; ++k) {
      double t = part[0][k];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) t += part[w][k];
      s[k] = t;
    }
  }
  double v[NMOM];
  moments_from_sums(s, N, r0, r1, r2, v);
  if (lane < MOM_LANES) store_moments(mom, M, c, lane, v);
  if (state && lane == 0) {
    double w[NCS];
    cell_state(g, gas, v, c, dt_cell ? dt_cell[c] : dt, w, counters);
    store_cell_state(cs, M, c, w);
  }
}

// Waves a cell: 0 the 16-lane kernel, which also keeps the 0D grids (the
// batched solve sums its cells in that order).  The rule looks at the grid
// alone, so that a state gives the same bits from buffers of any capacity.
static int moment_waves(const GridP& g) {
  return g.dim == 0 || g.M > 4096 ? 0 : g.M <= 512 ? 4 : 1;
}

template <typename S, int WAVES>
static hipError_t moments_wide(const GridP& g, const GasP& gas, const PartP<S>& p,
                               const int64_t* offsets, double* mom, double dt,
                               const double* dt_cell, double* cs, int64_t* counters,
                               hipStream_t st, const uint32_t* perm, int state) {
  const int nb = (int)g.M;
  if (perm)
    k_moments_wide<S, true, WAVES><<<nb, 64 * WAVES, 0, st>>>(g, gas, p, offsets, mom, perm, dt,
                                                              dt_cell, cs, counters, state);
  else
    k_moments_wide<S, false, WAVES><<<nb, 64 * WAVES, 0, st>>>(g, gas, p, offsets, mom, perm, dt,
                                                               dt_cell, cs, counters, state);
  return hipGetLastError();
}

// Per-cell state of cell c.
__device__ __forceinline__ void reconstruct_cell(const GridP& g, const GasP& gas, const double* mom,
                                                 double dt, const double* dt_cell, double* cs,
                                                 int64_t* counters, int64_t c) {
  const int64_t M = g.M;
  double m[NMOM], v[NCS];
#pragma unroll
  for (int k = 0; k < NMOM; ++k) m[k] = mom[k * M + c];
  cell_state(g, gas, m, c, dt_cell ? dt_cell[c] : dt, v, counters);
  store_cell_state(cs, M, c, v);
}

// Per-cell state, one thread per cell.
__global__ void k_reconstruct(GridP g, GasP gas, const double* mom, double dt,
                              const double* dt_cell, double* cs, int64_t* counters) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c < g.M) reconstruct_cell(g, gas, mom, dt, dt_cell, cs, counters, c);
}

__global__ void k_stencil(GridP g, double* cs) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c < g.M && g.dim != 0) stencil_cell(g, cs, c);
}

// Grids of at most CELL_SMALL cells (launch-bound steps): the cell state and
// then the stencils in one block, the barrier between them standing in for
// the launch boundary (the stencils read the neighbours' usability).
constexpr int64_t CELL_SMALL = 256;
__global__ __launch_bounds__(256) void k_cell_state_small(GridP g, GasP gas, const double* mom,
                                                          double dt, const double* dt_cell,
                                                          double* cs, int64_t* counters) {
  for (int64_t c = threadIdx.x; c < g.M; c += blockDim.x)
    reconstruct_cell(g, gas, mom, dt, dt_cell, cs, counters, c);
  if (g.dim == 0) return;
  __syncthreads();
  for (int64_t c = threadIdx.x; c < g.M; c += blockDim.x) stencil_cell(g, cs, c);
}

// Field sampling: the raw particle sums of each cell, N <f(c)>, formed
// from the central moment planes (c = U + C) and added to the running sums.
// Thread per cell, plain read-modify-write: deterministic.
__global__ void k_sample_fields(int64_t M, const double* __restrict__ mom,
                                double* __restrict__ acc) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= M) return;
  const double N = mom[M_N * M + c];
  if (N == 0.0) return;
  double U[3], P[6], qt[3], qr[3], qi[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    U[k] = mom[(M_UX + k) * M + c];
    qt[k] = mom[(M_QTRX + k) * M + c];
    qr[k] = mom[(M_QROTX + k) * M + c];
    qi[k] = mom[(M_QIX + k) * M + c];
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) P[k] = mom[(M_PXX + k) * M + c];
  const double er = mom[M_EROT * M + c], Ib = mom[M_IBAR * M + c];
  // Pi as a full matrix: xx yy zz xy xz yz
  const double PU[3] = {P[0] * U[0] + P[3] * U[1] + P[4] * U[2],
                        P[3] * U[0] + P[1] * U[1] + P[5] * U[2],
                        P[4] * U[0] + P[5] * U[1] + P[2] * U[2]};
  const double hU2 = 0.5 * (U[0] * U[0] + U[1] * U[1] + U[2] * U[2]);
  const double htr = 0.5 * (P[0] + P[1] + P[2]);
  double v[USP_NSAMP];
  v[0] = 1.0;
  v[1] = U[0]; v[2] = U[1]; v[3] = U[2];
  v[4] = P[0] + U[0] * U[0]; v[5] = P[1] + U[1] * U[1]; v[6] = P[2] + U[2] * U[2];
  v[7] = P[3] + U[0] * U[1]; v[8] = P[4] + U[0] * U[2]; v[9] = P[5] + U[1] * U[2];
  v[10] = er; v[11] = Ib;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    v[12 + k] = (hU2 + htr) * U[k] + PU[k] + qt[k];
    v[15 + k] = U[k] * er + qr[k];
    v[18 + k] = U[k] * Ib + qi[k];
  }
#pragma unroll
  for (int k = 0; k < USP_NSAMP; ++k) acc[k * M + c] += N * v[k];
}

hipError_t launch_sample_fields(const GridP& g, const double* mom, double* acc, hipStream_t st) {
  k_sample_fields<<<cdiv(g.M, 256), 256, 0, st>>>(g.M, mom, acc);
  return hipGetLastError();
}

template <typename S>
hipError_t launch_moments(const GridP& g, const PartP<S>& p, const int64_t* offsets, double* mom,
                          hipStream_t st, const uint32_t* gather_perm) {
  const int waves = moment_waves(g);
  if (waves) {
    const GasP none{};
    return (waves == 4 ? moments_wide<S, 4> : moments_wide<S, 1>)(
        g, none, p, offsets, mom, 0.0, nullptr, nullptr, nullptr, st, gather_perm, 0);
  }
  const int64_t nb = cdiv(g.M * MOM_LANES, CELL_BLOCK);
  if (gather_perm)
    k_moments<S, true><<<nb, CELL_BLOCK, 0, st>>>(g, p, offsets, mom, gather_perm);
  else
    k_moments<S, false><<<nb, CELL_BLOCK, 0, st>>>(g, p, offsets, mom, nullptr);
  return hipGetLastError();
}

hipError_t launch_stencil(const GridP& g, const GasP& gas, double* cs, hipStream_t st) {
  if (g.dim != 0) k_stencil<<<cdiv(g.M, 256), 256, 0, st>>>(g, cs);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_cell_coef(g, gas, cs, st);
}

hipError_t launch_reconstruct(const GridP& g, const GasP& gas, const double* mom, double dt,
                              const double* dt_cell, double* cs, int64_t* counters, hipStream_t st) {
  if (g.M <= CELL_SMALL) {
    k_cell_state_small<<<1, 256, 0, st>>>(g, gas, mom, dt, dt_cell, cs, counters);
  } else {
    k_reconstruct<<<cdiv(g.M, 128), 128, 0, st>>>(g, gas, mom, dt, dt_cell, cs, counters);
    k_stencil<<<cdiv(g.M, 256), 256, 0, st>>>(g, cs);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the coefficient chain per cell, when the particle update takes it
  // from the cell
  return launch_cell_coef(g, gas, cs, st);
}

template <typename S>
hipError_t launch_cells(const GridP& g, const GasP& gas, const PartP<S>& p, const int64_t* offsets,
                        double* mom, double dt, const double* dt_cell, double* cs,
                        int64_t* counters, hipStream_t st, const uint32_t* gather_perm,
                        bool stencils) {
  const int waves = moment_waves(g);
  if (!waves) {
    const hipError_t e = launch_moments<S>(g, p, offsets, mom, st, gather_perm);
    return e != hipSuccess ? e : launch_reconstruct(g, gas, mom, dt, dt_cell, cs, counters, st);
  }
  const hipError_t e = (waves == 4 ? moments_wide<S, 4> : moments_wide<S, 1>)(
      g, gas, p, offsets, mom, dt, dt_cell, cs, counters, st, gather_perm, 1);
  if (e != hipSuccess) return e;
  return stencils ? launch_stencil(g, gas, cs, st) : launch_cell_coef(g, gas, cs, st);
}

template hipError_t launch_cells<float>(const GridP&, const GasP&, const PartP<float>&,
                                        const int64_t*, double*, double, const double*, double*,
                                        int64_t*, hipStream_t, const uint32_t*, bool);
template hipError_t launch_cells<double>(const GridP&, const GasP&, const PartP<double>&,
                                         const int64_t*, double*, double, const double*, double*,
                                         int64_t*, hipStream_t, const uint32_t*, bool);
template hipError_t launch_moments<float>(const GridP&, const PartP<float>&, const int64_t*,
                                          double*, hipStream_t, const uint32_t*);
template hipError_t launch_moments<double>(const GridP&, const PartP<double>&, const int64_t*,
                                           double*, hipStream_t, const uint32_t*);

}  // namespace usp
