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
// With large cells, bound by the tiles of one or two of them, in which the
// update is close to its instruction rate and the sums and the conservation
// leave waves idle (thousands of small cells take another shape, see
// small_tiles).  So the stage takes a cell of 4096 FP32 particles (a cell past the stage
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

template <typename S, bool STAGED, int CAP, int MODE, int BLOCK>
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
    for (int64_t i = i0 + threadIdx.x; i < i1; i += BLOCK) st.store(i, load_state(p, i));
    __syncthreads();
  }
  for (int s = 0; s < nsteps; ++s) {
    const uint32_t step = (uint32_t)(step0 + (uint64_t)s);
    tile_cells<S, BLOCK>(g, gas, dt, dt_cell, mom, cs, offsets, c0, c1, st, counters);
    __syncthreads();
    if constexpr (MODE == MODE_CELL) {
      for (int64_t c = c0 + threadIdx.x; c < c1; c += BLOCK)
        cell_pcoefs(cs, g.M)[c] = cell_pcoef(gas, cs, g.M, c);
      __syncthreads();
    }
    tile_update<S, CAP, true, MODE, BLOCK>(g, gas, cs, p, i0, i1, st, st, esc_list, nesc, seed, step,
                                   wc);
    tile_conserve<S, BLOCK>(gas, cs, g.M, offsets, c0, c1, st, seed, step, counters);
    __syncthreads();
    wg_counters_flush(wcnt, counters);
  }
  if (STAGED) {
    for (int64_t i = i0 + threadIdx.x; i < i1; i += BLOCK) {
      const PartNew<S> v = st.load(i);
      p.cx[i] = v.cx; p.cy[i] = v.cy; p.cz[i] = v.cz; p.erot[i] = v.erot; p.vib[i] = (uint8_t)v.vib;
    }
  }
}

// Shapes of a tile's workgroup: threads, stage, the particles of one round of
// the update (the FP32 first pass lists its escalations for the second), and
// the smallest and largest window taken by itself.  V = 0: two workgroups of
// 8 waves on a CU; V = 1: four of 4 waves, with half the stage.
template <typename S, int V> struct BatchCfg;
template <> struct BatchCfg<float, 0> {
  static constexpr int BLOCK = 512, STAGE = 4352, ROUND = 2048, ESC = 2048, WMIN = 512, WMAX = 1536;
};
template <> struct BatchCfg<double, 0> {
  static constexpr int BLOCK = 512, STAGE = 2304, ROUND = 2304, ESC = 1, WMIN = 256, WMAX = 1024;
};
template <> struct BatchCfg<float, 1> {
  static constexpr int BLOCK = 256, STAGE = 2240, ROUND = 1024, ESC = 1024, WMIN = 512, WMAX = 1024;
};
template <> struct BatchCfg<double, 1> {
  static constexpr int BLOCK = 256, STAGE = 1200, ROUND = 1200, ESC = 1, WMIN = 256, WMAX = 512;
};

// Which shape.  Large cells leave waves idle in their sums and conservation,
// and want the stage and the waves of shape 0; thousands of small cells keep
// every wave busy, and four workgroups a CU hide each other's barriers better
// than two.  A step of M cells of up to n particles (16 to n, log-uniform),
// shape 0 / shape 1, each at its best window (and the 4-wave kernel with
// half the stage that shape 0 replaced), us:
//   FP32  1500 x 1500 61 / 70 (89)    2592 x 761 55 / 54 (63)    2592 x 1500 77 / 74 (95)
//         2592 x 4096 142 / 220 (204) 4096 x 256 56 / 51 (55)    4096 x 761 84 / 73 (71)
//         4096 x 1500 111 / 102 (109) 4096 x 4096 201 / 244 (248)
//   FP64  1500 x 4096 242 / 293 (312) 2592 x 761 83 / 78 (103)   2592 x 1500 126 / 144 (156)
//         2592 x 4096 290 / 327 (357) 4096 x 256 82 / 72 (83)    4096 x 761 128 / 115 (131)
//         4096 x 1500 182 / 159 (193) 4096 x 4096 419 / 363 (389)
// (a state of fewer than 3e5 FP32 particles does not fill shape 1's slots).
template <typename S>
static bool small_tiles(int64_t M, int64_t cap, int tile) {
  if (tile > BatchCfg<S, 1>::WMAX) return false;
  return sizeof(S) == 4 ? M >= 2500 && cap <= 400 * M && cap >= 300000 : M >= 3000;
}

// The window, of a launch that does not name one: at most half the stage, so
// that the cells before a tile's last one always fit it, and as many tiles as
// the chip runs at once while that leaves them WMIN slots (short tiles leave
// waves idle in the per-cell phases, long ones CUs; 2592 FP32 cells of up to 761,
// shape 0: 512 slots 71 us, 1024 55, 1536 64, 2048 67; 200 of up to 1500: 53, 55,
// 71, 72).  Shape 0 goes past 1024 FP32 slots only from 1.5M particles on (1500
// cells of up to 4096: 126, 128, 140, 144; 4096: 235, 221, 206, 201).
template <typename S, int V>
static int64_t batch_window(int64_t cap) {
  using C = BatchCfg<S, V>;
  static_assert(2 * C::WMAX <= C::STAGE && C::WMIN >= 2 * UPDATE_TILE_MIN, "windows and tile order");
  const int64_t most = sizeof(S) == 4 && cap < 1500000 ? 1024 : C::WMAX;
  const int64_t w = cdiv(cap, V == 0 ? 512 : 1024);
  return w < C::WMIN ? C::WMIN : w > most ? most : w;
}

template <typename S, int MODE, int V>
__global__ __launch_bounds__((BatchCfg<S, V>::BLOCK), 4) void k_batch(
    GridP g, GasP gas, double dt, const double* dt_cell, double* mom, double* cs,
    const int64_t* __restrict__ offsets, const int32_t* __restrict__ first,
    const int32_t* __restrict__ order, PartP<S> p, uint64_t seed, uint64_t step0, int nsteps,
    int64_t* counters) {
  using C = BatchCfg<S, V>;
  constexpr int CAP = C::STAGE;
  __shared__ S scx[CAP], scy[CAP], scz[CAP], ser[CAP];
  __shared__ uint8_t svb[CAP];
  __shared__ uint16_t esc_list[C::ESC];
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
      batch_tile<S, true, C::ROUND, MODE, C::BLOCK>(g, gas, dt, dt_cell, mom, cs, offsets, p, a, b,
                                                    i0, i1, st, esc_list, &nesc, seed, step0,
                                                    nsteps, counters, wcnt);
    } else {
      batch_tile<S, false, C::ROUND, MODE, C::BLOCK>(g, gas, dt, dt_cell, mom, cs, offsets, p, a, b,
                                                     i0, i1, global_stage(p), esc_list, &nesc, seed,
                                                     step0, nsteps, counters, wcnt);
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

template <typename S, int V>
static hipError_t batch_launches(const GridP& g, const GasP& gas, double dt, const double* dt_cell,
                                 double* mom, double* cs, const int64_t* offsets, const PartP<S>& p,
                                 int64_t window, int spl, uint64_t seed, uint64_t step, int nsteps,
                                 int32_t* first, int64_t* counters, hipStream_t st) {
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
#define USP_K_BATCH(MODE)                                                                        \
  k_batch<S, MODE, V><<<ntiles, (BatchCfg<S, V>::BLOCK), 0, st>>>(                                \
      g, gas, dt, dt_cell, mom, cs, offsets, first, order, p, seed, step + (uint64_t)s, k, counters)
    if (mode == MODE_FPM) USP_K_BATCH(MODE_FPM);
    else if (mode == MODE_CELL) USP_K_BATCH(MODE_CELL);
    else USP_K_BATCH(MODE_USP);
#undef USP_K_BATCH
    e = hipGetLastError();
  }
  return e;
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
  if (small_tiles<S>(g.M, p.capacity, tile))
    return batch_launches<S, 1>(g, gas, dt, dt_cell, mom, cs, offsets, p,
                                tile > 0 ? tile : batch_window<S, 1>(p.capacity), spl, seed, step,
                                nsteps, first, counters, st);
  return batch_launches<S, 0>(g, gas, dt, dt_cell, mom, cs, offsets, p,
                              tile > 0 ? tile : batch_window<S, 0>(p.capacity), spl, seed, step,
                              nsteps, first, counters, st);
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
