// usp_batch.hip -- many independent 0D cells advanced several steps per
// launch (the persistent form of the step for dim 0).
//
// In 0D no particle changes cell and no cell reads a neighbour, so a
// workgroup that owns a tile of whole cells can run step after step without
// any grid-wide synchronisation: per step the moments of its cells (16 lanes
// or a wave each), their cell state (a thread each), the particle update
// (thread per particle) and the conservation (wave per cell), all on an LDS
// stage that holds the tile's velocities, rotational energies and levels
// from the first step to the last.
//
// Bound by the tiles of one or two large cells, in which the update is close
// to its instruction rate and the sums and the conservation leave waves idle.
// So the stage takes a cell of 4096 FP32 particles (a cell past the stage
// runs in place in global memory), 8 waves work on it, a wave shares a large
// cell's 20 sums out over its lanes, and a tile whose last cell does not fit
// beside the others runs that cell after them.  Cycles of a step for tiles of
// 4046 particles: cells 103 -> 68 thousand, update 245 -> 148, conservation
// 252 -> 47 (4 waves and half the stage before, such tiles in global memory).
// 4096 cells of 16 to 4096 FP32 particles, 20 steps: 5.15 -> 4.26 ms (4.08
// with the rows' loads ahead of their sums).
// Every phase calls the device functions of the step kernels in the same
// order, so the result is bit-identical to usp_step on the same state.
#include "usp_tile.h"

namespace usp {

template <typename S, bool STAGED, int CAP, int MODE>
__device__ __forceinline__ void batch_tile(const GridP& g, const GasP& gas, double dt,
                                           const double* dt_cell, double* mom, double* cs,
                                           const int64_t* __restrict__ offsets,
                                           const PartP<S>& p, int64_t c0, int64_t c1,
                                           int64_t i0, int64_t i1, const Stage<S>& st,
                                           uint16_t* esc_list, int* nesc,
                                           uint64_t seed, uint64_t step0, int nsteps,
                                           int64_t* counters,
                                           unsigned long long* wcnt) {
  // per-particle events of the update go to the workgroup's counts, which
  // are added to the global counters after every step
  const WgCounters wc{counters ? wcnt : nullptr};
  if (STAGED) {
    for (int64_t i = i0 + threadIdx.x; i < i1; i += UPD_BLOCK) st.store(i, load_state(p, i));
    __syncthreads();
  }
  for (int s = 0; s < nsteps; ++s) {
    const uint32_t step = (uint32_t)(step0 + (uint64_t)s);
    tile_cells<S>(g, gas, dt, dt_cell, mom, cs, offsets, c0, c1, st, counters);
    __syncthreads();
    if constexpr (MODE == MODE_CELL) {
      for (int64_t c = c0 + threadIdx.x; c < c1; c += UPD_BLOCK)
        cell_pcoefs(cs, g.M)[c] = cell_pcoef(gas, cs, g.M, c);
      __syncthreads();
    }
    tile_update<S, CAP, true, MODE>(g, gas, cs, p, i0, i1, st, st, esc_list, nesc, seed, step,
                                   wc);
    tile_conserve<S>(gas, cs, g.M, offsets, c0, c1, st, seed, step, counters);
    __syncthreads();
    wg_counters_flush(wcnt, counters);
  }
  if (STAGED) {
    for (int64_t i = i0 + threadIdx.x; i < i1; i += UPD_BLOCK) {
      const PartNew<S> v = st.load(i);
      p.cx[i] = v.cx; p.cy[i] = v.cy; p.cz[i] = v.cz; p.erot[i] = v.erot; p.vib[i] = (uint8_t)v.vib;
    }
  }
}

// Stage sizes (two workgroups' LDS on a CU), and the particles of one round of
// the update (the FP32 first pass lists its escalations for the second).
template <typename S> struct BatchCfg;
template <> struct BatchCfg<float> { static constexpr int STAGE = 4352, ROUND = 2048, ESC = 2048; };
template <> struct BatchCfg<double> { static constexpr int STAGE = 2304, ROUND = 2304, ESC = 1; };

template <typename S, int MODE>
__global__ __launch_bounds__(UPD_BLOCK, 4) void k_batch(GridP g, GasP gas, double dt,
                                                        const double* dt_cell, double* mom,
                                                        double* cs,
                                                        const int64_t* __restrict__ offsets,
                                                        const int32_t* __restrict__ first,
                                                        const int32_t* __restrict__ order,
                                                        PartP<S> p, uint64_t seed, uint64_t step0,
                                                        int nsteps, int64_t* counters) {
  constexpr int CAP = BatchCfg<S>::STAGE, ROUND = BatchCfg<S>::ROUND;
  __shared__ S scx[CAP], scy[CAP], scz[CAP], ser[CAP];
  __shared__ uint8_t svb[CAP];
  __shared__ uint16_t esc_list[BatchCfg<S>::ESC];
  __shared__ int nesc;
  __shared__ unsigned long long wcnt[USP_NCOUNTERS];
  const int64_t t = order[blockIdx.x];
  const int64_t c0 = first[t], c1 = first[t + 1];
  if (c0 >= c1) return;
  wg_counters_init(wcnt);  // ordered before use by the barriers ahead of the first update
  // the cells before the last one start and end within the window, which the
  // stage holds; the last cell alone may reach past it
  const int64_t span = offsets[c1] - offsets[c0];
  const int64_t cut = span <= CAP ? c1 : c1 - 1;
  for (int64_t a = c0; a < c1;) {
    const int64_t b = a < cut ? cut : c1;
    const int64_t i0 = offsets[a], i1 = offsets[b];
    if (i1 - i0 <= CAP) {
      Stage<S> st;
      st.cx = scx; st.cy = scy; st.cz = scz; st.erot = ser; st.vib = svb; st.base = i0;
      batch_tile<S, true, ROUND, MODE>(g, gas, dt, dt_cell, mom, cs, offsets, p, a, b, i0, i1, st,
                                       esc_list, &nesc, seed, step0, nsteps, counters, wcnt);
    } else {
      batch_tile<S, false, ROUND, MODE>(g, gas, dt, dt_cell, mom, cs, offsets, p, a, b, i0, i1,
                                        global_stage(p), esc_list, &nesc, seed, step0, nsteps,
                                        counters, wcnt);
    }
    __syncthreads();  // the stage and the counts are free again
    a = b;
  }
}

// Dispatch order of a batched launch: the tiles by descending particle
// count, so that the heaviest start first and the launch, in which every
// workgroup keeps its tile for all its steps, does not end on a heavy tile
// started late.  Counts are binned (ORDER_BINS bins up to the largest), the
// order inside a bin is left open (no result depends on it).  One block;
// a full sort of 3000 tiles took 55 us of a call.
constexpr int ORDER_BINS = 1024;

__global__ __launch_bounds__(1024) void k_tile_order(const int64_t* __restrict__ offsets,
                                                     const int32_t* __restrict__ first,
                                                     int64_t ntiles, int32_t* order) {
  __shared__ unsigned int hist[ORDER_BINS], wsum[16], most;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (threadIdx.x == 0) most = 0u;
  hist[threadIdx.x] = 0u;
  __syncthreads();
  auto count = [&](int64_t t) -> unsigned int {
    const int64_t w = offsets[first[t + 1]] - offsets[first[t]];
    return w > 0xFFFFFFFFLL ? 0xFFFFFFFFu : (unsigned int)w;
  };
  unsigned int m = 0u;
  for (int64_t t = threadIdx.x; t < ntiles; t += 1024) {
    const unsigned int w = count(t);
    m = w > m ? w : m;
  }
  atomicMax(&most, m);
  __syncthreads();
  const unsigned int width = most / ORDER_BINS + 1u;
  auto bin = [&](int64_t t) { return ORDER_BINS - 1 - (int)(count(t) / width); };
  for (int64_t t = threadIdx.x; t < ntiles; t += 1024) atomicAdd(&hist[bin(t)], 1u);
  __syncthreads();
  // exclusive scan of the bins, a thread each
  const unsigned int v = hist[threadIdx.x];
  unsigned int x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  unsigned int base = 0u;
  for (int w = 0; w < wid; ++w) base += wsum[w];
  hist[threadIdx.x] = base + x - v;
  __syncthreads();
  for (int64_t t = threadIdx.x; t < ntiles; t += 1024) order[atomicAdd(&hist[bin(t)], 1u)] = (int32_t)t;
}

template <typename S>
hipError_t launch_batch(const GridP& g, const GasP& gas, double dt, const double* dt_cell,
                        double* mom, double* cs, const int64_t* offsets, const PartP<S>& p,
                        int tile, int steps_per_launch, uint64_t seed, uint64_t step,
                        int nsteps, char* ws, const WsLayout& L, int64_t* counters,
                        hipStream_t st) {
  if (nsteps <= 0) return hipSuccess;
  int32_t* first = (int32_t*)(ws + L.tiles);
  const int spl = steps_per_launch > 0 ? steps_per_launch : nsteps;
  // The window (at most half the stage, so that the cells before a tile's
  // last one always fit it).  4096 cells of up to 4096 FP32 particles: 512
  // slots 4.81 ms, 1024 4.48, 1536 4.26, 2048 4.33, 4096 4.74 (short tiles
  // leave waves idle in the per-cell phases, long ones end in a cell run by
  // itself).
  const int64_t window = sizeof(S) == 4 ? (tile > 0 ? tile : 1536) : 512;
  const int64_t ntiles = cdiv(p.capacity, window);
  hipError_t e = launch_tiles(offsets, g.M, window, ntiles, first, st);
  // the order follows first[] in the workspace (sized for 128-slot windows)
  int32_t* order = first + ntiles + 1;
  if (e == hipSuccess) {
    k_tile_order<<<1, 1024, 0, st>>>(offsets, first, ntiles, order);
    e = hipGetLastError();
  }
  const int mode = update_mode(gas);
  for (int s = 0; s < nsteps && e == hipSuccess; s += spl) {
    const int k = nsteps - s < spl ? nsteps - s : spl;
#define USP_K_BATCH(MODE)                                                                       \
  k_batch<S, MODE><<<ntiles, UPD_BLOCK, 0, st>>>(g, gas, dt, dt_cell, mom, cs, offsets, first,    \
                                                 order, p, seed, step + (uint64_t)s, k, counters)
    if (mode == MODE_FPM) USP_K_BATCH(MODE_FPM);
    else if (mode == MODE_CELL) USP_K_BATCH(MODE_CELL);
    else USP_K_BATCH(MODE_USP);
#undef USP_K_BATCH
    e = hipGetLastError();
  }
  return e;
}

template hipError_t launch_batch<float>(const GridP&, const GasP&, double, const double*, double*,
                                        double*, const int64_t*, const PartP<float>&, int, int,
                                        uint64_t, uint64_t, int, char*, const WsLayout&, int64_t*,
                                        hipStream_t);
template hipError_t launch_batch<double>(const GridP&, const GasP&, double, const double*, double*,
                                         double*, const int64_t*, const PartP<double>&, int, int,
                                         uint64_t, uint64_t, int, char*, const WsLayout&,
                                         int64_t*, hipStream_t);

}  // namespace usp
