// usp_moments.hip -- per-cell moments and the per-cell USP-FPM state.
#include "usp_cell.h"

namespace usp {

constexpr int CELL_BLOCK = 256;

// 16 lanes per cell, four cells per wave (every lane stays active for the
// row permutes; lanes of cells past M carry zeros).
template <typename S, bool G, bool AHEAD>
__global__ __launch_bounds__(CELL_BLOCK) void k_moments(GridP g, PartP<S> p, const int64_t* offsets,
                                                        double* mom, const uint32_t* perm) {
  const int64_t M = g.M;
  const int64_t c = ((int64_t)blockIdx.x * CELL_BLOCK + threadIdx.x) / MOM_LANES;
  const int sub = threadIdx.x & (MOM_LANES - 1);
  const bool valid = c < M;
  const int64_t o0 = valid ? offsets[c] : 0, o1 = valid ? offsets[c + 1] : 0;
  double v[NMOM];
  row_moments<S, G, AHEAD>(p.cx, p.cy, p.cz, p.erot, p.vib, o0, o1, sub, v, perm);
  if (valid) store_moments(mom, M, c, sub, v);
}

// On grids of few cells 16 lanes a cell leave the chip idle: a workgroup takes
// a cell (block_row_sums: the bits of k_moments), and with `state` one lane
// goes on to the cell state, which saves its launch where every cell has a CU
// to itself: the chain holds its workgroup's waves and LDS for some 10 us, and
// with several cells a CU the chains follow one another (a step of 256 cells
// of 200 particles: 55 us with its launch, 50 without; of 300 cells 57 and 63;
// of 4096 cells 131 and 160).  200 cells of 1000 particles: 22 + 10 us for
// the two kernels before, 14 together; 0.7M FP64 particles in 1800 cells: the
// moments 38 -> 18 us. (Each lane its own particles in all 20 sums took 12:
// other bits, which a FP32 state carries on.)
template <typename S, bool G, int BLOCK, int SC>
__global__ __launch_bounds__(BLOCK) void k_moments_wide(GridP g, GasP gas, PartP<S> p,
                                                        const int64_t* __restrict__ offsets,
                                                        double* mom,
                                                        const uint32_t* __restrict__ perm,
                                                        double dt, const double* dt_cell,
                                                        double* cs, int64_t* counters, int state) {
  __shared__ MomStage<SC> st;
  const int64_t M = g.M, c = blockIdx.x;
  const int64_t o0 = offsets[c], o1 = offsets[c + 1];
  double r0 = 0.0, r1 = 0.0, r2 = 0.0;
  if (o1 > o0) {
    int64_t j = o0;
    if constexpr (G) j = (int64_t)perm[o0];
    r0 = (double)p.cx[j]; r1 = (double)p.cy[j]; r2 = (double)p.cz[j];
  }
  block_row_sums<S, G, BLOCK, SC>(p.cx, p.cy, p.cz, p.erot, p.vib, o0, o1, r0, r1, r2, &st, perm);
  if (threadIdx.x >= 64) return;
  double s[20], v[NMOM];
#pragma unroll
  for (int k = 0; k < 20; ++k) s[k] = st.sums[k];
  moments_from_sums(s, o1 - o0, r0, r1, r2, v);
  const int lane = threadIdx.x;
  if (lane < MOM_LANES) store_moments(mom, M, c, lane, v);
  if (state && lane == 0) {
    double w[NCS];
    cell_state(g, gas, v, c, dt_cell ? dt_cell[c] : dt, w, counters);
    store_cell_state(cs, M, c, w);
  }
}

// 0: the 16-lane kernel; 1 and 2: a workgroup a cell, of 5 waves, or on the
// smallest grids of 8.  The 16 lanes' time is that of the fullest cell, the
// workgroups' grows with the cells, each of which costs its barriers.  Moments
// alone, 16 lanes against a workgroup, FP32: cells alike, 1024 x 800
// particles 9.7 / 10.8 us, 1800 x 220 7.7 / 8.5, 1800 x 800 10 / 18, 2592 x 220
// 7.8 / 11, 4096 x 200 7.2 / 17, 4096 x 800 12 / 39; with a shock layer of up to
// a dozen times the mean, 450 x 220 23 / 12, 1800 x 220 26 / 13, 2592 x 220 25 /
// 16, 4050 x 220 25 / 25 (FP64 34 / 25).  A step of cells alike: 300 x 200 62 /
// 58, 1024 x 200 73 / 72, 1800 x 200 96 / 100, 4096 x 200 119 / 131.  So up to
// 1024 cells, and up to 2048 in 2D, whose flows have dense layers (0D grids
// are batches of cells of any size and keep their two kernels).
static int moments_shape(const GridP& g) {
  if (g.dim == 0 || g.M > (g.dim == 2 ? 2048 : 1024)) return 0;
  return g.M <= 512 ? 2 : 1;
}

template <typename S, int BLOCK, int SC>
static hipError_t moments_wide(const GridP& g, const GasP& gas, const PartP<S>& p,
                               const int64_t* offsets, double* mom, double dt,
                               const double* dt_cell, double* cs, int64_t* counters,
                               hipStream_t st, const uint32_t* perm, int state) {
  const int nb = (int)g.M;
  if (perm)
    k_moments_wide<S, true, BLOCK, SC><<<nb, BLOCK, 0, st>>>(g, gas, p, offsets, mom, perm, dt,
                                                             dt_cell, cs, counters, state);
  else
    k_moments_wide<S, false, BLOCK, SC><<<nb, BLOCK, 0, st>>>(g, gas, p, offsets, mom, perm, dt,
                                                              dt_cell, cs, counters, state);
  return hipGetLastError();
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

// Grids of at most CELL_SMALL cells (usp_reconstruct, and the steps of 0D
// grids): the cell state and then the stencils in one block, the barrier between them standing in for
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
  const int shape = moments_shape(g);
  if (shape) {
    const GasP none{};
    return (shape == 2 ? moments_wide<S, 512, 512> : moments_wide<S, MOM_THREADS, 256>)(
        g, none, p, offsets, mom, 0.0, nullptr, nullptr, nullptr, st, gather_perm, 0);
  }
  const int64_t nb = cdiv(g.M * MOM_LANES, CELL_BLOCK);
  // Cells of fewer particles than lanes have none to load ahead.  600,000
  // cells, one by one / ahead, us: 5 FP32 particles 161 / 167, gathered 161 /
  // 172; 8 FP64 161 / 179, 193 / 214; 12 FP32 170 / 170, 197 / 179; 16 FP32 197
  // / 188, 239 / 227; 30 FP32 239 / 215, 280 / 240.
  const bool ahead = p.capacity > 10 * g.M;
#define USP_K(G, A) k_moments<S, G, A><<<nb, CELL_BLOCK, 0, st>>>(g, p, offsets, mom, gather_perm)
  if (gather_perm) {
    if (ahead) USP_K(true, true);
    else USP_K(true, false);
  } else {
    if (ahead) USP_K(false, true);
    else USP_K(false, false);
  }
#undef USP_K
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
                        int64_t* counters, hipStream_t st, const uint32_t* gather_perm) {
  if (g.dim == 0 || !update_solo(g)) {
    const hipError_t e = launch_moments<S>(g, p, offsets, mom, st, gather_perm);
    return e != hipSuccess ? e : launch_reconstruct(g, gas, mom, dt, dt_cell, cs, counters, st);
  }
  const hipError_t e = moments_wide<S, 512, 512>(g, gas, p, offsets, mom, dt, dt_cell, cs, counters,
                                                 st, gather_perm, 1);
  return e != hipSuccess ? e : launch_cell_coef(g, gas, cs, st);
}

template hipError_t launch_cells<float>(const GridP&, const GasP&, const PartP<float>&,
                                        const int64_t*, double*, double, const double*, double*,
                                        int64_t*, hipStream_t, const uint32_t*);
template hipError_t launch_cells<double>(const GridP&, const GasP&, const PartP<double>&,
                                         const int64_t*, double*, double, const double*, double*,
                                         int64_t*, hipStream_t, const uint32_t*);
template hipError_t launch_moments<float>(const GridP&, const PartP<float>&, const int64_t*,
                                          double*, hipStream_t, const uint32_t*);
template hipError_t launch_moments<double>(const GridP&, const PartP<double>&, const int64_t*,
                                           double*, hipStream_t, const uint32_t*);

}  // namespace usp
