// usp_sort.hip -- binning as a stable counting sort of input chunks (the
// order of usp_bin: by cell, in input order inside a cell, removed particles
// dropped), for inputs whose order is not known and for small grids.
//
// A workgroup owns a chunk of consecutive input slots and counts the digits
// of its particles (k_sort_count: the cell, or with more than SORT_BUCKETS
// cells a bucket of 2^shift consecutive cells).  A particle's slot is then
// the digit's start, plus the digit's particles in earlier chunks, plus
// those in earlier waves of its chunk, plus its rank in its own wave (lanes
// of equal digit found by ballots): no atomics on memory, nothing to clear
// beforehand, and the result does not depend on the launch.  k_sort_place
// writes the final order, or (buckets) the list of (index, cell) pairs in
// bucket order, which k_sort_fine orders by cell, a workgroup per bucket
// (moving the particles, recording the order, or, for a large unordered
// input, recording it for k_sort_fetch).
#include "usp_binkey.h"

namespace usp {

constexpr int SORT_BLOCK = 512;
constexpr int SORT_WAVES = SORT_BLOCK / 64;
constexpr int SORT_U = 4;  // 64-particle groups whose keys are loaded together
constexpr int COUNT_U = 8;
constexpr int SUM_U = 10;  // rows of counts a thread has in flight

// Key of input slot i: the cell it holds on entry for the binned prefix
// (i < ns), else from its position; -1 for a removed particle.
template <typename S>
__device__ __forceinline__ int32_t sort_key(const GridP& g, const PartP<S>& in, int64_t i,
                                            int64_t ns, bool* solid) {
  *solid = false;
  if (i >= ns) return new_key<S>(g, in, i, solid);
  int32_t c = in.cell[i];
  if (c >= g.M) c = -1;
  if (c >= 0 && g.flags && (g.flags[c] & USP_FLAG_SOLID)) {
    c = -1;
    *solid = true;
  }
  return c;
}

// Slots of a chunk: n / SORT_CHUNKS in whole workgroups, of the n particles
// present and not of the buffer they lie in (20,000 particles of 1024 cells in
// 9.4M slots, with chunks of 9216 and of 2048: 66 -> 37 us a bin, unordered
// 90 -> 32).
__device__ __forceinline__ int64_t chunk_slots(int64_t n) {
  constexpr int64_t ALL = SORT_CHUNKS * SORT_BLOCK;
  const int64_t per = (int64_t)((uint64_t)(n + ALL - 1) / ALL) * SORT_BLOCK;
  // (the same for every lane, and kept on the scalar unit)
  return __builtin_amdgcn_readfirstlane((int)(per > SORT_CHUNK_MIN ? per : SORT_CHUNK_MIN));
}

// Chunks that n particles fill (n and the chunk fit 32 bits).
__device__ __forceinline__ int chunks_used(int64_t n, int64_t chunk) {
  return n > 0 ? (int)((uint32_t)(n - 1) / (uint32_t)chunk) + 1 : 0;
}

// Adds the wave's digits (d < 0: none) to an LDS histogram, one atomic per
// run of equal digits.
__device__ __forceinline__ void count_digits(uint32_t* hist, int32_t d) {
  int hl, len;
  wave_runs(d, &hl, &len);
  if (len > 0 && d >= 0) atomicAdd(&hist[d], (uint32_t)len);
}

// The lanes of the wave that hold the same digit as this lane (d < 0: an
// idle lane, result unused): up to three distinct values one by one, then,
// where more are present (an unordered input), one ballot per bit.
__device__ __forceinline__ uint64_t same_digit(int32_t d, int bits) {
  uint64_t rest = __ballot(d >= 0), same = 0ull;
  for (int t = 0; t < 3 && rest; ++t) {
    const int32_t v = __builtin_amdgcn_readlane(d, __ffsll((long long)rest) - 1);
    const uint64_t m = __ballot(d == v);
    if (d == v) same = m;
    rest &= ~m;
  }
  if (rest) {
    uint64_t m = rest;
    for (int b = 0; b < bits; ++b) {
      const bool bit = ((uint32_t)d >> b) & 1u;
      const uint64_t bm = __ballot(bit);
      m &= bit ? bm : ~bm;
    }
    if ((rest >> (threadIdx.x & 63)) & 1ull) same = m;
  }
  return same;
}

// Position of this lane's particle in digit order: next[d] counts up as the
// wave walks its slots in input order.
__device__ __forceinline__ uint32_t take_slot(uint32_t* next, int32_t d, int bits) {
  const uint64_t same = same_digit(d, bits);
  const int lane = threadIdx.x & 63;
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  uint32_t p = 0;
  if (d >= 0) {
    const uint32_t base = next[d];
    p = base + (uint32_t)__popcll(same & lt);
    // the last lane of the digit moves it on
    if ((same >> lane) == 1ull) next[d] = p + 1u;
  }
  // the next group of lanes reads what this one wrote
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  return p;
}

// Exclusive scan of v[0, n) (n <= SORT_BUCKETS, LDS) in place over the
// workgroup; returns the total.
__device__ __forceinline__ uint32_t scan_lds(uint32_t* v, int n) {
  __shared__ uint32_t wsum[SORT_WAVES];
  constexpr int PER = SORT_BUCKETS / SORT_BLOCK;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t a[PER], s = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int j = threadIdx.x * PER + k;
    a[k] = j < n ? v[j] : 0u;
    s += a[k];
  }
  uint32_t x = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wid] = x;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < SORT_WAVES; ++w) {
    if (w < wid) base += wsum[w];
    tot += wsum[w];
  }
  uint32_t run = base + x - s;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int j = threadIdx.x * PER + k;
    if (j < n) v[j] = run;
    run += a[k];
  }
  __syncthreads();
  return tot;
}

// Digit counts of chunk blockIdx.x, row blockIdx.x of T.  Keys of the slots
// past the binned prefix are kept in key[]; *ns_out receives the prefix
// length (the output offsets may overwrite old_off later).
template <typename S>
__global__ __launch_bounds__(SORT_BLOCK) void k_sort_count(GridP g, PartP<S> in,
                                                           const int64_t* old_off, int32_t* key,
                                                           uint32_t* T, SortPlan sp, int64_t* ns_out,
                                                           int64_t* counters) {
  __shared__ uint32_t hist[SORT_BUCKETS];
  for (int d = threadIdx.x; d < sp.ld; d += SORT_BLOCK) hist[d] = 0u;
  __syncthreads();
  const int64_t n = in.count[0];
  const int64_t ns = old_off ? sorted_len(old_off, g.M, in.count) : 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *ns_out = ns;
  const int64_t chunk = chunk_slots(n), i0 = (int64_t)blockIdx.x * chunk;
  if (i0 >= n) return;
  const int64_t i1 = i0 + chunk < n ? i0 + chunk : n;
  const int lane = threadIdx.x & 63;
  for (int64_t b = i0 + (threadIdx.x & ~63); b < i1; b += COUNT_U * SORT_BLOCK) {
    int32_t c[COUNT_U];
#pragma unroll
    for (int u = 0; u < COUNT_U; ++u) {
      const int64_t i = b + u * SORT_BLOCK + lane;
      bool solid = false;
      c[u] = -1;
      if (i < i1) {
        c[u] = sort_key<S>(g, in, i, ns, &solid);
        if (i >= ns) key[i] = c[u];
      }
      if (solid) count_event(counters, USP_CNT_SOLID_DROP);
    }
#pragma unroll
    for (int u = 0; u < COUNT_U; ++u) count_digits(hist, c[u] < 0 ? -1 : c[u] >> sp.shift);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < sp.ld; d += SORT_BLOCK) T[(int64_t)blockIdx.x * sp.ld + d] = hist[d];
}

// Column scan of T (rows = chunks in use): every entry becomes the digit's
// count in earlier chunks, tot[d] its total.  32 columns by 32 row groups a
// workgroup.
constexpr int SCAN_COLS = 32, SCAN_GROUPS = 32;
__global__ __launch_bounds__(SCAN_COLS* SCAN_GROUPS) void k_sort_scan(uint32_t* T, uint32_t* tot,
                                                                      SortPlan sp,
                                                                      const int64_t* in_count) {
  __shared__ uint32_t part[SCAN_GROUPS][SCAN_COLS + 1];
  const int nk = chunks_used(in_count[0], chunk_slots(in_count[0]));
  const int col = threadIdx.x & (SCAN_COLS - 1), rg = threadIdx.x / SCAN_COLS;
  const int d = blockIdx.x * SCAN_COLS + col;
  const int per = (nk + SCAN_GROUPS - 1) / SCAN_GROUPS;
  const int k0 = rg * per < nk ? rg * per : nk, k1 = k0 + per < nk ? k0 + per : nk;
  uint32_t s = 0;
  if (d < sp.nb) {
#pragma unroll 8
    for (int k = k0; k < k1; ++k) s += T[(int64_t)k * sp.ld + d];
  }
  part[rg][col] = s;
  __syncthreads();
  uint32_t run = 0;
  for (int q = 0; q < rg; ++q) run += part[q][col];
  if (d >= sp.nb) return;
  if (rg == SCAN_GROUPS - 1) tot[d] = run + s;
#pragma unroll 8
  for (int k = k0; k < k1; ++k) {
    const uint32_t v = T[(int64_t)k * sp.ld + d];
    T[(int64_t)k * sp.ld + d] = run;
    run += v;
  }
}

// Per-wave digit starts: start[d] (the workgroup's first slot of digit d) is
// handed to the waves in order, whist[w][d] = the wave's first slot.
__device__ __forceinline__ void wave_starts(const uint32_t* start, uint32_t (*whist)[SORT_BUCKETS],
                                            int nb) {
  for (int d = threadIdx.x; d < nb; d += SORT_BLOCK) {
    uint32_t run = start[d];
#pragma unroll
    for (int w = 0; w < SORT_WAVES; ++w) {
      const uint32_t t = whist[w][d];
      whist[w][d] = run;
      run += t;
    }
  }
}

// The chunk's particles to their slots: the final order (PAIRS = false: the
// digit is the cell), or (index, cell) pairs in bucket order.  With
// self-scan (few chunks times digits) every workgroup sums the columns of T
// itself; otherwise k_sort_scan has.
template <typename S, bool G, bool PAIRS>
__global__ __launch_bounds__(SORT_BLOCK) void k_sort_place(GridP g, PartP<S> in, PartP<S> out,
                                                           const int32_t* __restrict__ key,
                                                           const uint32_t* __restrict__ T,
                                                           const uint32_t* __restrict__ tot,
                                                           SortPlan sp, const int64_t* ns_in,
                                                           int64_t* offsets, uint32_t* gperm,
                                                           int32_t* pair_i, int32_t* pair_c,
                                                           uint32_t* bucket_off, TileIndex ti) {
  __shared__ uint32_t start[SORT_BUCKETS];
  alignas(16) __shared__ uint32_t whist[SORT_WAVES][SORT_BUCKETS];
  const int64_t n = in.count[0], ns = *ns_in;
  // the last workgroup has no chunk: it writes the offsets (and the tile
  // index), so that no placing one does both
  const bool index = blockIdx.x == gridDim.x - 1;
  const int64_t chunk = chunk_slots(n), i0 = (int64_t)blockIdx.x * chunk;
  if (i0 >= n && !index) return;
  const int64_t i1 = i0 + chunk < n ? i0 + chunk : n;
  const int nk = chunks_used(n, chunk);
  const int blk = (int)blockIdx.x;
  // column sums and the sums of the earlier chunks
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // each wave owns a run of consecutive slots of the chunk; the keys of its
  // first SORT_U groups (all of them in the smallest chunk) are requested
  // ahead of the column sums
  const int64_t sub = chunk / SORT_WAVES;
  const int64_t w0 = i0 + wid * sub, w1 = w0 + sub < i1 ? w0 + sub : i1;
  auto cells_at = [&](int64_t b, int32_t c[SORT_U]) {
#pragma unroll
    for (int u = 0; u < SORT_U; ++u) {
      const int64_t i = b + u * 64 + lane;
      c[u] = i >= w1 ? -1 : (i >= ns ? key[i] : in.cell[i]);
      if (c[u] >= g.M) c[u] = -1;
    }
    if (g.flags) {
#pragma unroll
      for (int u = 0; u < SORT_U; ++u)
        if (c[u] >= 0 && (g.flags[c[u]] & USP_FLAG_SOLID)) c[u] = -1;
    }
  };
  int32_t cf[SORT_U];
  cells_at(w0, cf);
  uint32_t* before = whist[0];  // free until the waves count
  if (sp.self_scan) {
    // four columns a load, the row groups' loads all in flight at once;
    // the groups' sums meet in LDS
    const int quads = sp.ld / 4, most = SORT_BLOCK / quads, groups = nk < most ? nk : most;
    const int rg = threadIdx.x / quads, q = threadIdx.x - rg * quads;
    uint4* part = (uint4*)&whist[0][0];  // [group][all, pre][quads]
    if (rg < groups) {
      uint4 all = {0, 0, 0, 0}, pre = {0, 0, 0, 0};
      const uint4* col = (const uint4*)T + q;
      for (int k = rg; k < nk; k += SUM_U * groups) {
        uint4 v[SUM_U];
#pragma unroll
        for (int u = 0; u < SUM_U; ++u) {
          const int r = k + u * groups;
          v[u] = col[(int64_t)(r < nk ? r : k) * quads];
        }
#pragma unroll
        for (int u = 0; u < SUM_U; ++u) {
          const int r = k + u * groups;
          const uint32_t m = r < nk ? ~0u : 0u, b = r < blk ? m : 0u;
          all.x += v[u].x & m; all.y += v[u].y & m; all.z += v[u].z & m; all.w += v[u].w & m;
          pre.x += v[u].x & b; pre.y += v[u].y & b; pre.z += v[u].z & b; pre.w += v[u].w & b;
        }
      }
      part[(rg * 2) * quads + q] = all;
      part[(rg * 2 + 1) * quads + q] = pre;
    }
    __syncthreads();
    uint32_t all[SORT_BUCKETS / SORT_BLOCK] = {0}, pre[SORT_BUCKETS / SORT_BLOCK] = {0};
    const uint32_t* flat = &whist[0][0];
#pragma unroll
    for (int u = 0; u < SORT_BUCKETS / SORT_BLOCK; ++u) {
      const int d = threadIdx.x + u * SORT_BLOCK;
      if (d < sp.nb)
        for (int k = 0; k < groups; ++k) {
          all[u] += flat[(k * 2) * sp.ld + d];
          pre[u] += flat[(k * 2 + 1) * sp.ld + d];
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < SORT_BUCKETS / SORT_BLOCK; ++u) {
      const int d = threadIdx.x + u * SORT_BLOCK;
      if (d < sp.nb) { start[d] = all[u]; before[d] = pre[u]; }
    }
  } else {
    for (int d = threadIdx.x; d < sp.nb; d += SORT_BLOCK) {
      start[d] = tot[d];
      before[d] = i0 < n ? T[(int64_t)blk * sp.ld + d] : 0u;
    }
  }
  __syncthreads();
  const uint32_t total = scan_lds(start, sp.nb);
  if (index) {
    if (PAIRS) {
      for (int d = threadIdx.x; d < sp.nb; d += SORT_BLOCK) bucket_off[d] = start[d];
      if (threadIdx.x == 0) bucket_off[sp.nb] = total;
    } else {
      for (int d = threadIdx.x; d < sp.nb; d += SORT_BLOCK) offsets[d] = (int64_t)start[d];
      if (threadIdx.x == 0) {
        offsets[sp.nb] = (int64_t)total;
        out.count[0] = (int64_t)total;
        out.count[1] = in.count[1];
      }
      if (ti.first) {
        const uint32_t W = (uint32_t)update_tile(ti.stage, total, g.M);
        for (int d = threadIdx.x; d < sp.nb; d += SORT_BLOCK)
          mark_tiles(ti, W, d, start[d], d + 1 < sp.nb ? start[d + 1] : total);
        mark_last_tiles(ti, W, g.M, total, threadIdx.x, SORT_BLOCK);
      }
    }
    return;
  }
  for (int d = threadIdx.x; d < sp.nb; d += SORT_BLOCK) start[d] += before[d];
  __syncthreads();
  for (int d = threadIdx.x; d < sp.nb; d += SORT_BLOCK)
#pragma unroll
    for (int w = 0; w < SORT_WAVES; ++w) whist[w][d] = 0u;
  __syncthreads();
  uint32_t* mine = whist[wid];
  for (int64_t b = w0; b < w1; b += SORT_U * 64) {
    int32_t c[SORT_U];
    if (b == w0) {
#pragma unroll
      for (int u = 0; u < SORT_U; ++u) c[u] = cf[u];
    } else {
      cells_at(b, c);
    }
#pragma unroll
    for (int u = 0; u < SORT_U; ++u) count_digits(mine, c[u] < 0 ? -1 : c[u] >> sp.shift);
  }
  __syncthreads();
  wave_starts(start, whist, sp.nb);
  __syncthreads();
  const bool hx = g.dim == 2, hy = g.dim >= 1;
  for (int64_t b = w0; b < w1; b += SORT_U * 64) {
    int32_t c[SORT_U];
    if (b == w0) {
#pragma unroll
      for (int u = 0; u < SORT_U; ++u) c[u] = cf[u];
    } else {
      cells_at(b, c);
    }
    uint32_t p[SORT_U], ii[SORT_U];
#pragma unroll
    for (int u = 0; u < SORT_U; ++u) {
      p[u] = take_slot(mine, c[u] < 0 ? -1 : c[u] >> sp.shift, sp.bits);
      ii[u] = (uint32_t)(b + u * 64 + lane);
    }
    if constexpr (PAIRS) {
#pragma unroll
      for (int u = 0; u < SORT_U; ++u)
        if (c[u] >= 0) {
          pair_i[p[u]] = (int32_t)ii[u];
          pair_c[p[u]] = c[u];
        }
    } else {
      place_many<G, SORT_U, S>(in, out, gperm, ii, p, c, hx, hy);
    }
  }
}

// One bucket of 2^shift consecutive cells: its pairs, already in input
// order, to the cells' slots.  Buckets of a flow are uneven (a dense layer
// holds a dozen times the mean), so a bucket gets a workgroup of 16 waves
// and each wave keeps FINE_U groups of loads in flight.
constexpr int FINE_BLOCK = 1024;
constexpr int FINE_WAVES = FINE_BLOCK / 64;
constexpr int FINE_U = 8;

template <typename S, bool G>
__global__ __launch_bounds__(FINE_BLOCK) void k_sort_fine(GridP g, PartP<S> in, PartP<S> out,
                                                          SortPlan sp, int64_t* offsets,
                                                          uint32_t* gperm,
                                                          const int32_t* __restrict__ pair_i,
                                                          const int32_t* __restrict__ pair_c,
                                                          const uint32_t* __restrict__ bucket_off,
                                                          TileIndex ti) {
  extern __shared__ uint32_t fine_lds[];  // start[F], then next[FINE_WAVES][F]
  const int F = 1 << sp.shift;
  uint32_t* start = fine_lds;
  const int64_t s0 = bucket_off[blockIdx.x], s1 = bucket_off[blockIdx.x + 1];
  const int32_t c0 = (int32_t)((int64_t)blockIdx.x << sp.shift);
  const int nf = (int)(g.M - c0 < F ? g.M - c0 : F);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  uint32_t* mine = fine_lds + F + wid * F;
  for (int d = lane; d < nf; d += 64) mine[d] = 0u;
  const int64_t sub = ((s1 - s0 + FINE_BLOCK - 1) / FINE_BLOCK) * 64;
  const int64_t w0 = s0 + wid * sub < s1 ? s0 + wid * sub : s1;
  const int64_t w1 = w0 + sub < s1 ? w0 + sub : s1;
  for (int64_t b = w0; b < w1; b += FINE_U * 64) {
    int32_t c[FINE_U];
#pragma unroll
    for (int u = 0; u < FINE_U; ++u) {
      const int64_t j = b + u * 64 + lane;
      c[u] = j < w1 ? pair_c[j] - c0 : -1;
    }
#pragma unroll
    for (int u = 0; u < FINE_U; ++u) count_digits(mine, c[u]);
  }
  __syncthreads();
  // the cells' totals, their scan by the first wave, the waves' first slots
  for (int d = threadIdx.x; d < nf; d += FINE_BLOCK) {
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < FINE_WAVES; ++w) t += fine_lds[F + w * F + d];
    start[d] = t;
  }
  __syncthreads();
  if (wid == 0) {
    uint32_t carry = (uint32_t)s0;
    for (int d0 = 0; d0 < nf; d0 += 64) {
      const int d = d0 + lane;
      const uint32_t v = d < nf ? start[d] : 0u;
      uint32_t x = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      if (d < nf) {
        start[d] = carry + x - v;
        offsets[c0 + d] = (int64_t)(carry + x - v);
      }
      carry += __shfl(x, 63, 64);
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    offsets[g.M] = s1;
    out.count[0] = s1;
    out.count[1] = in.count[1];
  }
  __syncthreads();
  if (ti.first) {
    const int64_t total = bucket_off[sp.nb];
    const uint32_t W = (uint32_t)update_tile(ti.stage, total, g.M);
    for (int d = threadIdx.x; d < nf; d += FINE_BLOCK)
      mark_tiles(ti, W, c0 + d, start[d], d + 1 < nf ? start[d + 1] : (uint32_t)s1);
    if (blockIdx.x == gridDim.x - 1) mark_last_tiles(ti, W, g.M, total, threadIdx.x, FINE_BLOCK);
  }
  for (int d = threadIdx.x; d < nf; d += FINE_BLOCK) {
    uint32_t run = start[d];
#pragma unroll
    for (int w = 0; w < FINE_WAVES; ++w) {
      const uint32_t t = fine_lds[F + w * F + d];
      fine_lds[F + w * F + d] = run;
      run += t;
    }
  }
  __syncthreads();
  const bool hx = g.dim == 2, hy = g.dim >= 1;
  constexpr int U = G ? FINE_U : SORT_U;
  for (int64_t b = w0; b < w1; b += U * 64) {
    int32_t c[U];
    uint32_t p[U], ii[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = b + u * 64 + lane;
      c[u] = j < w1 ? pair_c[j] - c0 : -1;
      ii[u] = j < w1 ? (uint32_t)pair_i[j] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) p[u] = take_slot(mine, c[u], sp.shift);
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = c[u] < 0 ? -1 : c0 + c[u];
    place_many<G, U, S>(in, out, gperm, ii, p, c, hx, hy);
  }
}

// An unordered input of many particles in two steps: the buckets only record
// the order (k_sort_fine<S, true>), then every slot fetches its particle.  A
// bucket of a shock layer holds seven times the mean, and a workgroup that
// also fetches its bucket's particles ends long after the others.  The fetch
// is bound by lines of memory: a word in an array of its own costs a line as
// much as 16 bytes side by side do, so the words are first laid in packs of
// the pairs' 16 bytes a particle (free by then), one pack after the other.
// 4.6M FP32 particles of a shocked cylinder in random order: 1030 us by
// buckets, 645 fetching one 16-byte pack and four words, 456 in two packs (FP64, four
// packs: 1157 -> 693).
constexpr int FETCH_BLOCK = 256;
constexpr int FETCH_U = 4;
// Workgroups at most (eight on each CU, four rounds); each goes on to the next
// slots while any are left.
constexpr int64_t FETCH_BLOCKS = 8192;

struct alignas(16) SortPack {
  uint32_t w[4];
};

// Pack K of a particle: FP32 (cx, cy, cz, erot), (x, y, pid, level); FP64
// (cx, cy), (cz, erot), (x, y), (pid, level).
template <typename S>
constexpr int SORT_PACKS = sizeof(S) == 4 ? 2 : 4;

template <typename S>
__device__ __forceinline__ void pack_words(SortPack* a, int at, S v) {
  __builtin_memcpy(&a->w[at * (int)(sizeof(S) / 4)], &v, sizeof(S));
}
template <typename S>
__device__ __forceinline__ S unpack_words(const SortPack& a, int at) {
  S v;
  __builtin_memcpy(&v, &a.w[at * (int)(sizeof(S) / 4)], sizeof(S));
  return v;
}

template <typename S, int K>
__global__ __launch_bounds__(FETCH_BLOCK) void k_sort_pack(PartP<S> in, SortPack* pack, bool has_x,
                                                           bool has_y) {
  constexpr bool WIDE = sizeof(S) == 8;
  const int64_t n = in.count[0];
  for (int64_t i = (int64_t)blockIdx.x * FETCH_BLOCK + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * FETCH_BLOCK) {
    SortPack a = {};
    if constexpr (K == 0) {
      pack_words<S>(&a, 0, in.cx[i]);
      pack_words<S>(&a, 1, in.cy[i]);
    }
    if constexpr (K == (WIDE ? 1 : 0)) {
      pack_words<S>(&a, WIDE ? 0 : 2, in.cz[i]);
      pack_words<S>(&a, WIDE ? 1 : 3, in.erot[i]);
    }
    if constexpr (K == (WIDE ? 2 : 1)) {
      if (has_x) pack_words<S>(&a, 0, in.x[i]);
      if (has_y) pack_words<S>(&a, 1, in.y[i]);
    }
    if constexpr (K == SORT_PACKS<S> - 1) {
      a.w[2] = in.pid[i];
      a.w[3] = in.vib[i];
    }
    pack[i] = a;
  }
}

template <typename S, int K>
__global__ __launch_bounds__(FETCH_BLOCK) void k_sort_fetch(PartP<S> out,
                                                            const SortPack* __restrict__ pack,
                                                            const uint32_t* __restrict__ perm,
                                                            bool has_x, bool has_y) {
  constexpr bool WIDE = sizeof(S) == 8;
  const int64_t n = out.count[0];
  for (int64_t p0 = (int64_t)blockIdx.x * (FETCH_BLOCK * FETCH_U) + threadIdx.x; p0 < n;
       p0 += (int64_t)gridDim.x * (FETCH_BLOCK * FETCH_U)) {
    uint32_t i[FETCH_U];
    SortPack a[FETCH_U];
#pragma unroll
    for (int u = 0; u < FETCH_U; ++u) {
      const int64_t p = p0 + u * FETCH_BLOCK;
      i[u] = perm[p < n ? p : p0];
    }
#pragma unroll
    for (int u = 0; u < FETCH_U; ++u) a[u] = pack[i[u]];
#pragma unroll
    for (int u = 0; u < FETCH_U; ++u) {
      const int64_t p = p0 + u * FETCH_BLOCK;
      if (p >= n) continue;
      if constexpr (K == 0) {
        out.cx[p] = unpack_words<S>(a[u], 0);
        out.cy[p] = unpack_words<S>(a[u], 1);
      }
      if constexpr (K == (WIDE ? 1 : 0)) {
        out.cz[p] = unpack_words<S>(a[u], WIDE ? 0 : 2);
        out.erot[p] = unpack_words<S>(a[u], WIDE ? 1 : 3);
      }
      if constexpr (K == (WIDE ? 2 : 1)) {
        if (has_x) out.x[p] = unpack_words<S>(a[u], 0);
        if (has_y) out.y[p] = unpack_words<S>(a[u], 1);
      }
      if constexpr (K == SORT_PACKS<S> - 1) {
        out.pid[p] = a[u].w[2];
        out.vib[p] = (uint8_t)a[u].w[3];
      }
    }
  }
}

template <typename S, int K = 0>
static void fetch_packs(const PartP<S>& in, const PartP<S>& out, SortPack* pack,
                        const uint32_t* perm, bool hx, bool hy, hipStream_t st) {
  if (!(sizeof(S) == 8 && K == 2 && !hy)) {  // a pack of positions alone
    auto blocks = [](int64_t n) { return (int)(n < FETCH_BLOCKS ? n : FETCH_BLOCKS); };
    k_sort_pack<S, K><<<blocks(cdiv(in.capacity, FETCH_BLOCK)), FETCH_BLOCK, 0, st>>>(in, pack, hx, hy);
    k_sort_fetch<S, K><<<blocks(cdiv(out.capacity, FETCH_BLOCK * FETCH_U)), FETCH_BLOCK, 0, st>>>(
        out, pack, perm, hx, hy);
  }
  if constexpr (K + 1 < SORT_PACKS<S>) fetch_packs<S, K + 1>(in, out, pack, perm, hx, hy, st);
}

SortPlan sort_plan(int64_t M, int64_t capacity) {
  SortPlan sp;
  sp.shift = 0;
  while (cdiv(M, (int64_t)1 << sp.shift) > SORT_BUCKETS) ++sp.shift;
  sp.nb = (int)cdiv(M, (int64_t)1 << sp.shift);
  sp.ld = (sp.nb + 3) / 4 * 4;
  sp.bits = 0;
  while ((1 << sp.bits) < sp.nb) ++sp.bits;
  // chunks that any count up to the capacity needs
  const int64_t most = cdiv(capacity, SORT_CHUNK_MIN);
  sp.nchunks = most < SORT_CHUNKS ? most : SORT_CHUNKS;
  sp.self_scan = sp.nchunks * sp.ld <= SORT_SELF_SCAN ? 1 : 0;
  return sp;
}

// Capacity from which an unordered input is fetched in packs (its 3 or 7 more
// launches cost 10 to 25 us).  Buckets against packs, capacity 1.6 times the
// particles: FP32 0.23M particles 50 / 58 us, 0.36M 67 / 71, 0.47M (shocked)
// 101 / 74, 0.73M 134 / 96; FP64 0.23M 56 / 80, 0.47M 111 / 108, 0.73M 147 /
// 145, 4.6M 1157 / 693.
template <typename S>
constexpr int64_t SORT_FETCH_CAP = sizeof(S) == 4 ? 5 << 17 : 1 << 20;

template <typename S, bool G>
hipError_t sort_launches(const GridP& g, const PartP<S>& in, const PartP<S>& out, int64_t* offsets,
                         const int64_t* in_offsets, char* ws, const WsLayout& L, uint32_t* perm,
                         int64_t* counters, hipStream_t st, const TileIndex& ti) {
  const SortPlan sp = sort_plan(g.M, in.capacity);
  int32_t* key = (int32_t*)(ws + L.key);
  uint32_t* T = (uint32_t*)(ws + L.sort_t);
  uint32_t* tot = (uint32_t*)(ws + L.sort_tot);
  uint32_t* bucket_off = tot + SORT_BUCKETS;
  int32_t* pair_i = (int32_t*)(ws + L.far);
  int32_t* pair_c = pair_i + in.capacity;
  int64_t* ns = (int64_t*)(ws + L.misc) + 6;
  const int nk = (int)sp.nchunks;
  k_sort_count<S><<<nk, SORT_BLOCK, 0, st>>>(g, in, in_offsets, key, T, sp, ns, counters);
  if (!sp.self_scan)
    k_sort_scan<<<(int)cdiv(sp.nb, SCAN_COLS), SCAN_COLS * SCAN_GROUPS, 0, st>>>(T, tot, sp, in.count);
  if (sp.shift == 0) {
    k_sort_place<S, G, false><<<nk + 1, SORT_BLOCK, 0, st>>>(g, in, out, key, T, tot, sp, ns, offsets,
                                                         perm, nullptr, nullptr, nullptr, ti);
  } else {
    k_sort_place<S, G, true><<<nk + 1, SORT_BLOCK, 0, st>>>(g, in, out, key, T, tot, sp, ns, offsets,
                                                        perm, pair_i, pair_c, bucket_off, ti);
    const size_t lds = sizeof(uint32_t) * (size_t)(FINE_WAVES + 1) << sp.shift;
    if constexpr (!G) {
      if (!in_offsets && in.capacity >= SORT_FETCH_CAP<S>) {
        perm = (uint32_t*)(ws + L.perm);
        k_sort_fine<S, true><<<sp.nb, FINE_BLOCK, lds, st>>>(g, in, out, sp, offsets, perm, pair_i,
                                                             pair_c, bucket_off, ti);
        // (the pairs have been read)
        fetch_packs<S>(in, out, (SortPack*)(ws + L.far), perm, g.dim == 2, g.dim >= 1, st);
        return hipGetLastError();
      }
    }
    k_sort_fine<S, G><<<sp.nb, FINE_BLOCK, lds, st>>>(g, in, out, sp, offsets, perm, pair_i, pair_c,
                                                    bucket_off, ti);
  }
  return hipGetLastError();
}

#define USP_INST(S, G)                                                                            \
  template hipError_t sort_launches<S, G>(const GridP&, const PartP<S>&, const PartP<S>&, int64_t*, \
                                          const int64_t*, char*, const WsLayout&, uint32_t*,        \
                                          int64_t*, hipStream_t, const TileIndex&)
USP_INST(float, true);
USP_INST(float, false);
USP_INST(double, true);
USP_INST(double, false);
#undef USP_INST

}  // namespace usp
