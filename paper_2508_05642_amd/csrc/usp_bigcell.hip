// usp_bigcell.hip -- the per-cell reductions of Sec. IV.D for cells far
// larger than a workgroup's share of the chip (a single 0D cell of 1e5
// particles): the moments of Sec. II.A and the conservation of Sec. IV.C
// with each cell's particles split into chunks of CHUNK slots and the
// chunks' partial sums combined in chunk order (the result does not depend
// on the launch).  A step of such a grid is latency-bound (1e5 particles are
// 1600 waves), so the element-wise passes carry the reductions' first level
// with them: the particle update sums its chunk's post-collision state, and
// in 0D the scalings of one step are applied by the pass that sums the next
// step's moments.  Four launches a 0D step, where separate passes took
// eight (1e5 particles, FP64: 0.165 -> 0.06 ms).  The sums are added in the
// separate passes' order; products are fused differently (the scalings in
// k_mom_chunks, the explicit fused products of mom_add), so a state differs from theirs
// by round-off (1e-15).
#include "usp_cell.h"
#include "usp_particle.h"

namespace usp {

constexpr int CHUNK = BIG_CHUNK;
constexpr int BIG_BLOCK = 256;
constexpr int BIG_WAVES = BIG_BLOCK / 64;
constexpr int CELL_BLOCK = 512;  // workgroup of one cell in the second levels
constexpr int NPART = BIG_PARTS;  // partial sums per chunk (moments 20; conservation 6 + lmax)
constexpr int NCONS = 7;

// The conservation's scalars of a cell, and the velocity its first particle
// has once they are applied (the shift of the next moments).
struct BigScalars {
  ConsScalars r;
  double c0[3];
};
static_assert(sizeof(BigScalars) <= CONS_SCALAR_BYTES, "conservation scalar record size");

// chunk_off[c] = first chunk of cell c (cdiv(N_c, CHUNK) chunks each);
// chunk_off[M] = total.  One block: each thread sums a contiguous run of
// cells, then the runs' totals are scanned in LDS.
__global__ __launch_bounds__(256) void k_chunk_offsets(const int64_t* __restrict__ offsets,
                                                       int64_t M, int64_t* chunk_off) {
  __shared__ int64_t run[256];
  const int64_t per = (M + 255) / 256;
  const int64_t c0 = threadIdx.x * per, c1 = c0 + per < M ? c0 + per : M;
  int64_t t = 0;
  for (int64_t c = c0; c < c1; ++c) t += (offsets[c + 1] - offsets[c] + CHUNK - 1) / CHUNK;
  run[threadIdx.x] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t a = 0;
    for (int k = 0; k < 256; ++k) {
      const int64_t v = run[k];
      run[k] = a;
      a += v;
    }
  }
  __syncthreads();
  int64_t a = run[threadIdx.x];
  for (int64_t c = c0; c < c1; ++c) {
    chunk_off[c] = a;
    a += (offsets[c + 1] - offsets[c] + CHUNK - 1) / CHUNK;
  }
  // the last thread's running sum is the total (threads past M have no cells)
  if (threadIdx.x == 255) chunk_off[M] = a;
}

// The cell of chunk k: the last c with chunk_off[c] <= k (binary search).
__device__ __forceinline__ int64_t chunk_cell(const int64_t* __restrict__ chunk_off, int64_t M,
                                              int64_t k) {
  int64_t lo = 0, hi = M;  // chunk_off[lo] <= k < chunk_off[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (chunk_off[mid] <= k) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Moments, first level: wave per chunk, the 20 sums of its slots shifted
// by the cell's first particle, reduced over the wave in a fixed order.
// With APPLY the previous step's scalings are applied on the way.
template <typename S, bool APPLY>
__global__ __launch_bounds__(BIG_BLOCK) void k_mom_chunks(PartP<S> p,
                                                          const int64_t* __restrict__ offsets,
                                                          const int64_t* __restrict__ chunk_off,
                                                          int64_t M, int64_t nmax,
                                                          const BigScalars* __restrict__ scal,
                                                          double* part) {
  const int lane = threadIdx.x & 63;
  const int64_t k = (int64_t)blockIdx.x * BIG_WAVES + (threadIdx.x >> 6);
  if (k >= nmax || k >= chunk_off[M]) return;
  const int64_t c = chunk_cell(chunk_off, M, k);
  const int64_t o0 = offsets[c], o1 = offsets[c + 1];
  const int64_t a = o0 + (k - chunk_off[c]) * CHUNK;
  const int64_t b = a + CHUNK < o1 ? a + CHUNK : o1;
  double r0, r1, r2;
  ConsScalars f;
  if constexpr (APPLY) {
    f = scal[c].r;
    r0 = scal[c].c0[0]; r1 = scal[c].c0[1]; r2 = scal[c].c0[2];
  } else {
    r0 = (double)p.cx[o0]; r1 = (double)p.cy[o0]; r2 = (double)p.cz[o0];
  }
  double s[NPART];
#pragma unroll
  for (int q = 0; q < NPART; ++q) s[q] = 0.0;
  // a lane's CHUNK / 64 particles: four loads in flight, summed in order
  for (int64_t i0 = a + lane; i0 < b; i0 += 4 * 64) {
    MomIn<S> v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + u * 64 < b ? i0 + u * 64 : i0;
      v[u] = mom_load<S>(p.cx, p.cy, p.cz, p.erot, p.vib, i);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + u * 64;
      if (i >= b) break;
      if constexpr (APPLY) {
        cons_apply<S, S>(f, 0, &v[u].c0, &v[u].c1, &v[u].c2, &v[u].e);
        p.cx[i] = v[u].c0; p.cy[i] = v[u].c1; p.cz[i] = v[u].c2; p.erot[i] = v[u].e;
      }
      mom_add(v[u], r0, r1, r2, s);
    }
  }
#pragma unroll
  for (int q = 0; q < NPART; ++q) s[q] = wave_sum(s[q]);
  if (lane < NPART) {
    double w = 0.0;
#pragma unroll
    for (int q = 0; q < NPART; ++q)
      if (q == lane) w = s[q];
    part[k * NPART + lane] = w;
  }
}

// The partial sums of a cell's chunks [k0, k1) in chunk order, Q of each
// chunk's NPART: staged in LDS by the workgroup, added up by one thread a
// quantity (out[q], LDS; MAXQ: that quantity is a maximum).  Every thread
// sees out on return.
constexpr int STAGE_CHUNKS = 192;
template <int Q, int MAXQ>
__device__ __forceinline__ void chunk_totals(const double* __restrict__ part, int64_t k0, int64_t k1,
                                             double* stage, double* out) {
  double t = 0.0;
  for (int64_t kb = k0; kb < k1; kb += STAGE_CHUNKS) {
    const int n = (int)(k1 - kb < STAGE_CHUNKS ? k1 - kb : STAGE_CHUNKS);
    for (int j = threadIdx.x; j < n * Q; j += CELL_BLOCK)
      stage[j] = part[(kb + j / Q) * NPART + j % Q];
    __syncthreads();
    if (threadIdx.x < Q) {
#pragma unroll 8
      for (int k = 0; k < n; ++k) {
        const double v = stage[k * Q + threadIdx.x];
        t = (int)threadIdx.x == MAXQ ? fmax(t, v) : t + v;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < Q) out[threadIdx.x] = t;
  __syncthreads();
}

// Moments, second level, and the cell state: workgroup per cell.
template <typename S>
__global__ __launch_bounds__(CELL_BLOCK) void k_mom_cells(GridP g, GasP gas, PartP<S> p,
                                                          const int64_t* __restrict__ offsets,
                                                          const int64_t* __restrict__ chunk_off,
                                                          const double* __restrict__ part,
                                                          double* mom, double dt,
                                                          const double* dt_cell, double* cs,
                                                          int64_t* counters) {
  __shared__ double stage[STAGE_CHUNKS * NPART], tot[NPART];
  const int64_t c = blockIdx.x, M = g.M;
  chunk_totals<NPART, -1>(part, chunk_off[c], chunk_off[c + 1], stage, tot);
  if (threadIdx.x != 0) return;
  const int64_t o0 = offsets[c], N = offsets[c + 1] - o0;
  double s[NPART];
#pragma unroll
  for (int q = 0; q < NPART; ++q) s[q] = tot[q];
  double r0 = 0.0, r1 = 0.0, r2 = 0.0;
  if (N > 0) { r0 = (double)p.cx[o0]; r1 = (double)p.cy[o0]; r2 = (double)p.cz[o0]; }
  double v[NMOM], w[NCS];
  moments_from_sums(s, N, r0, r1, r2, v);
#pragma unroll
  for (int q = 0; q < NMOM; ++q) mom[q * M + c] = v[q];
  cell_state(g, gas, v, c, dt_cell ? dt_cell[c] : dt, w, counters);
  store_cell_state(cs, M, c, w);
}

// The particle update, and the conservation's first level: workgroup per
// chunk of a cell, thread per particle; the first wave then sums the
// chunk's post-collision state about U^n (largest level too) in the order
// of a wave striding over the chunk.
template <typename S, int MODE>
__global__ __launch_bounds__(CHUNK) void k_collide_chunks(GridP g, GasP gas,
                                                          const double* __restrict__ cs, PartP<S> p,
                                                          const int64_t* __restrict__ offsets,
                                                          const int64_t* __restrict__ chunk_off,
                                                          uint64_t seed, uint32_t step, double* part,
                                                          int64_t* counters) {
  __shared__ S sx[CHUNK], sy[CHUNK], sz[CHUNK], se[CHUNK];
  __shared__ uint8_t sv[CHUNK];
  const int64_t M = g.M, k = blockIdx.x;
  if (k >= chunk_off[M]) return;
  const int64_t c = chunk_cell(chunk_off, M, k);
  if (cs[CS_COLLIDE * M + c] == 0.0) return;
  const int64_t o0 = offsets[c], o1 = offsets[c + 1];
  const int64_t a = o0 + (k - chunk_off[c]) * CHUNK;
  const int64_t b = a + CHUNK < o1 ? a + CHUNK : o1;
  const int64_t i = a + threadIdx.x;
  if (i < b) {
    uint32_t ev = 0;
    const PartNew<S> in = load_state(p, i);
    PartNew<S> o = collide_mode<MODE, S>(g, gas, cs, load_pos(p, i, g.dim), (int32_t)c, in, seed,
                                         step, &ev);
    if (o.changed) {
      p.cx[i] = o.cx; p.cy[i] = o.cy; p.cz[i] = o.cz; p.erot[i] = o.erot;
      p.vib[i] = (uint8_t)o.vib;
    } else {
      o = in;
    }
    sx[threadIdx.x] = o.cx; sy[threadIdx.x] = o.cy; sz[threadIdx.x] = o.cz;
    se[threadIdx.x] = o.erot; sv[threadIdx.x] = (uint8_t)o.vib;
    flush_events(counters, ev);
  }
  __syncthreads();
  const int lane = threadIdx.x;
  if (lane >= 64) return;
  const double Un[3] = {cs[CS_UX * M + c], cs[CS_UY * M + c], cs[CS_UZ * M + c]};
  double s[6] = {0, 0, 0, 0, 0, 0};
  int m = 0;
  cons_sums<S>(Un, a + lane, b, 64, sx, sy, sz, se, sv, a, nullptr, o0, false, s, &m);
#pragma unroll
  for (int q = 0; q < 6; ++q) s[q] = wave_sum(s[q]);
  // the wave's largest level: a fixed butterfly of integer maxima
  for (int off = 32; off >= 1; off >>= 1) {
    const int o = __shfl_xor(m, off, 64);
    m = o > m ? o : m;
  }
  if (lane < NCONS) {
    double w = (double)m;
#pragma unroll
    for (int q = 0; q < 6; ++q)
      if (q == lane) w = s[q];
    part[k * NPART + lane] = w;
  }
}

// wave_picks by a workgroup of CELL_BLOCK threads on the levels of a cell in
// global memory, CELL_BLOCK consecutive draws at a time (a large cell needs
// some hundred moves a step; 64 at a time each batch waits for the last
// one's atomics).  The outcome is that of the sequential draws, as there.
__device__ int block_picks(uint8_t* lv, int64_t N, int64_t Id, int64_t* SI_io, uint32_t c,
                           uint32_t step, uint64_t seed, bool low, int64_t* counters) {
  alignas(16) __shared__ uint32_t keys[CELL_BLOCK];
  __shared__ int wacc[CELL_BLOCK / 64], cut_s;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t maxatt = 64 * N;
  int64_t att = 0, SI = *SI_io;
  uint32_t jbase = 1;
  int moved = 0;
  const double Nd = (double)N;
  while (Id != 0) {
    if (att >= maxatt || (Id < 0 && SI == 0)) {
      if (tid == 0) count_event(counters, USP_CNT_PICK_FAIL);
      break;
    }
    const int64_t need = Id > 0 ? Id : -Id;
    const bool valid = att + tid < maxatt;
    const uint32_t j = jbase + (uint32_t)tid;
    const U4 w = philox(c, step, TAG_CONSERVE, j >> 2, seed);
    const uint32_t wj = (j & 3) == 0 ? w.w[0] : (j & 3) == 1 ? w.w[1] : (j & 3) == 2 ? w.w[2] : w.w[3];
    int64_t k = (int64_t)floor(u01d(wj) * Nd);
    if (k >= N) k = N - 1;
    bool acc = valid;
    if (!(Id > 0 && low)) {
      // earlier draws of the batch on the same particle, against its level
      // (read past the vector cache: earlier batches stepped it by atomics)
      const uintptr_t at = (uintptr_t)(lv + k);
      const uint32_t word = __hip_atomic_load((const uint32_t*)(at & ~(uintptr_t)3),
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int L = (int)((word >> (8 * (unsigned)(at & 3))) & 255u);
      keys[tid] = (uint32_t)k;
      __syncthreads();
      int dup = 0;
      for (int t = 0; t < (tid & ~63); t += 4) {
        const uint4 q = *(const uint4*)&keys[t];
        dup += (q.x == (uint32_t)k) + (q.y == (uint32_t)k) + (q.z == (uint32_t)k) +
               (q.w == (uint32_t)k);
      }
      for (int t = tid & ~63; t < tid; ++t) dup += keys[t] == (uint32_t)k;
      acc = valid && (Id > 0 ? (L + dup < VIB_MAX) : (dup < L));
    }
    const uint64_t accm = __ballot(acc);
    if (lane == 0) wacc[wid] = __popcll(accm);
    __syncthreads();
    int before = __popcll(accm & ((1ull << lane) - 1ull)), nacc = 0;
    for (int t = 0; t < CELL_BLOCK / 64; ++t) {
      before += t < wid ? wacc[t] : 0;
      nacc += wacc[t];
    }
    int64_t napp, consumed;
    bool apply = acc;
    if (nacc >= need) {
      // the need-th accepted draw is the last one made
      apply = acc && before < need;
      if (acc && before == need - 1) cut_s = tid;
      napp = need;
    } else {
      napp = nacc;
    }
    if (apply) level_step(lv + k, Id > 0 ? 1 : -1);
    __threadfence();
    __syncthreads();
    if (nacc >= need) consumed = cut_s + 1;
    else consumed = maxatt - att < CELL_BLOCK ? maxatt - att : CELL_BLOCK;
    if (napp) moved = 1;
    SI += Id > 0 ? napp : -napp;
    Id += Id > 0 ? -napp : napp;
    att += consumed;
    jbase += (uint32_t)consumed;
    __syncthreads();  // keys, wacc and cut_s are free again
  }
  *SI_io = SI;
  return moved;
}

// Conservation, second level: workgroup per colliding cell, the chunks'
// sums in chunk order, then the picks on the cell's levels (global) and the
// scalars of the scalings.
template <typename S>
__global__ __launch_bounds__(CELL_BLOCK) void k_cons_cells(GridP g, GasP gas,
                                                           const double* __restrict__ cs,
                                                           PartP<S> p,
                                                           const int64_t* __restrict__ offsets,
                                                           const int64_t* __restrict__ chunk_off,
                                                           const double* __restrict__ part,
                                                           BigScalars* scal, uint64_t seed,
                                                           uint32_t step, int64_t* counters) {
  __shared__ double stage[STAGE_CHUNKS * NCONS], tot[NCONS];
  const int64_t M = g.M, c = blockIdx.x;
  const int64_t o0 = offsets[c], N = offsets[c + 1] - o0;
  BigScalars out;
  out.r.frot = 0.0; out.r.sc = 0.0; out.r.moved = 0;
  const bool coll = N > 0 && cs[CS_COLLIDE * M + c] != 0.0;
  if (coll) {
    const ConsIn in = cons_in(cs, M, c, step, seed);
    chunk_totals<NCONS, NCONS - 1>(part, chunk_off[c], chunk_off[c + 1], stage, tot);
    double s[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) s[q] = tot[q];
    const int lmax = (int)tot[NCONS - 1];
    out.r = cons_scalars_of(gas, in, N, s, threadIdx.x == 0, counters, [&](int64_t Id, int64_t* SI) {
      return block_picks(p.vib + o0, N, Id, SI, (uint32_t)c, step, seed, moves_stay_low(lmax, Id),
                         counters);
    });
  }
  if (threadIdx.x != 0) return;
  S v[4] = {S(0), S(0), S(0), S(0)};
  if (N > 0) {
    v[0] = p.cx[o0]; v[1] = p.cy[o0]; v[2] = p.cz[o0];
    cons_apply<S, S>(out.r, 0, &v[0], &v[1], &v[2], &v[3]);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) out.c0[q] = (double)v[q];
  scal[c] = out;
}

// Conservation, the scalings: thread per particle of the binned state.
template <typename S>
__global__ void k_cons_apply(PartP<S> p, const BigScalars* __restrict__ scal) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.count[0]) return;
  const int32_t c = p.cell[i];
  if (c < 0) return;
  const ConsScalars r = scal[c].r;
  cons_apply<S, S>(r, i, p.cx, p.cy, p.cz, p.erot);
}

hipError_t launch_chunks(const GridP& g, const int64_t* offsets, char* ws, const WsLayout& L,
                         hipStream_t st) {
  k_chunk_offsets<<<1, 256, 0, st>>>(offsets, g.M, (int64_t*)(ws + L.chunk_off));
  return hipGetLastError();
}

template <typename S>
hipError_t launch_cells_split(const GridP& g, const GasP& gas, const PartP<S>& p,
                              const int64_t* offsets, double* mom, double dt, const double* dt_cell,
                              double* cs, bool apply, char* ws, const WsLayout& L,
                              int64_t* counters, hipStream_t st) {
  const int64_t* chunk_off = (const int64_t*)(ws + L.chunk_off);
  double* part = (double*)(ws + L.chunk_part);
  const BigScalars* scal = (const BigScalars*)(ws + L.cons_scal);
  const int64_t nmax = chunks_max(p.capacity, g.M);
  const int nb = (int)cdiv(nmax, BIG_WAVES);
  if (apply)
    k_mom_chunks<S, true><<<nb, BIG_BLOCK, 0, st>>>(p, offsets, chunk_off, g.M, nmax, scal, part);
  else
    k_mom_chunks<S, false><<<nb, BIG_BLOCK, 0, st>>>(p, offsets, chunk_off, g.M, nmax, scal, part);
  k_mom_cells<S><<<(int)g.M, CELL_BLOCK, 0, st>>>(g, gas, p, offsets, chunk_off, part, mom, dt,
                                                  dt_cell, cs, counters);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_stencil(g, gas, cs, st);
}

template <typename S>
hipError_t launch_collide_split(const GridP& g, const GasP& gas, const double* cs,
                                const int64_t* offsets, const PartP<S>& p, uint64_t seed,
                                uint64_t step, char* ws, const WsLayout& L, int64_t* counters,
                                hipStream_t st) {
  const int64_t* chunk_off = (const int64_t*)(ws + L.chunk_off);
  double* part = (double*)(ws + L.chunk_part);
  BigScalars* scal = (BigScalars*)(ws + L.cons_scal);
  const int nmax = (int)chunks_max(p.capacity, g.M);
  const uint32_t s32 = (uint32_t)step;
  const int mode = update_mode(gas);
#define USP_K(MODE)                                                                            \
  k_collide_chunks<S, MODE><<<nmax, CHUNK, 0, st>>>(g, gas, cs, p, offsets, chunk_off, seed, s32, \
                                                    part, counters)
  if (mode == MODE_FPM) USP_K(MODE_FPM);
  else if (mode == MODE_CELL) USP_K(MODE_CELL);
  else USP_K(MODE_USP);
#undef USP_K
  k_cons_cells<S><<<(int)g.M, CELL_BLOCK, 0, st>>>(g, gas, cs, p, offsets, chunk_off, part, scal,
                                                   seed, s32, counters);
  return hipGetLastError();
}

template <typename S>
hipError_t launch_cons_apply(const PartP<S>& p, char* ws, const WsLayout& L, hipStream_t st) {
  k_cons_apply<S><<<cdiv(p.capacity, 256), 256, 0, st>>>(p, (const BigScalars*)(ws + L.cons_scal));
  return hipGetLastError();
}

#define USP_INST(S)                                                                             \
  template hipError_t launch_cells_split<S>(const GridP&, const GasP&, const PartP<S>&,          \
                                            const int64_t*, double*, double, const double*,      \
                                            double*, bool, char*, const WsLayout&, int64_t*,     \
                                            hipStream_t);                                        \
  template hipError_t launch_collide_split<S>(const GridP&, const GasP&, const double*,          \
                                              const int64_t*, const PartP<S>&, uint64_t,         \
                                              uint64_t, char*, const WsLayout&, int64_t*,        \
                                              hipStream_t);                                      \
  template hipError_t launch_cons_apply<S>(const PartP<S>&, char*, const WsLayout&, hipStream_t)
USP_INST(float);
USP_INST(double);
#undef USP_INST

}  // namespace usp
