// usp_binkey.h -- device functions shared by the two routes of the bin
// (usp_bin.hip, usp_sort.hip): keys, runs of equal keys, the placing of a
// particle in its output slot.
#pragma once
#include "usp_device.h"

namespace usp {

// Runs of equal keys in consecutive lanes of a wave (particles arrive
// mostly sorted by cell, so a wave holds a few long runs).  Returns the
// lane of this lane's run head and, for heads, the run length.
__device__ __forceinline__ void wave_runs(int32_t key, int* head_lane, int* run_len) {
  const int lane = threadIdx.x & 63;
  const int32_t prev = __shfl_up(key, 1, 64);
  const bool head = lane == 0 || key != prev;
  const uint64_t heads = __ballot(head);
  const uint64_t upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  *head_lane = 63 - __clzll(heads & upto);
  const uint64_t above = heads & ~upto;
  const int next = above ? (__ffsll((long long)above) - 1) : 64;
  *run_len = head ? next - lane : 0;
}

template <typename S>
__device__ __forceinline__ int32_t new_key(const GridP& g, const PartP<S>& in, int64_t i,
                                           bool* solid) {
  int32_t c = in.cell[i];
  *solid = false;
  if (c >= 0) {
    if (g.dim == 0) {
      if (c >= g.M) c = -1;
    } else {
      c = cell_of<S>(g, g.dim == 2 ? in.x[i] : S(0), in.y[i]);
    }
  }
  if (c >= 0 && g.flags && (g.flags[c] & USP_FLAG_SOLID)) {
    c = -1;
    *solid = true;
  }
  return c;
}

__device__ __forceinline__ int64_t sorted_len(const int64_t* old_off, int64_t M, const int64_t* count) {
  const int64_t a = old_off[M], b = count[0];
  return a < b ? (a > 0 ? a : 0) : b;
}

template <typename S>
__device__ __forceinline__ void copy_particle(const PartP<S>& in, const PartP<S>& out, int64_t i,
                                              int64_t p, int32_t c, bool has_x, bool has_y) {
  if (has_x) out.x[p] = in.x[i];
  if (has_y) out.y[p] = in.y[i];
  out.cx[p] = in.cx[i];
  out.cy[p] = in.cy[i];
  out.cz[p] = in.cz[i];
  out.erot[p] = in.erot[i];
  out.vib[p] = in.vib[i];
  out.pid[p] = in.pid[i];
  out.cell[p] = c;
}

// Output slot p of input particle i: copied (G = false), or, for a binning
// that leaves the particles where they are (G = true), recorded as
// gperm[p] = i with the new cell in out.cell[p].
template <bool G, typename S>
__device__ __forceinline__ void place(const PartP<S>& in, const PartP<S>& out, uint32_t* gperm,
                                      int64_t i, int64_t p, int32_t c, bool has_x, bool has_y) {
  if constexpr (G) {
    gperm[p] = (uint32_t)i;
    out.cell[p] = c;
  } else {
    copy_particle<S>(in, out, i, p, c, has_x, has_y);
  }
}

// Tile index entries that cell c, with the output segment [o, o1), decides:
// the tiles whose window starts past the cell's first slot and not past
// its end begin at the next cell (window W); cell 0 also opens tile 0.
// (slots fit 32 bits, and a 32-bit division is a fifth of a 64-bit one)
__device__ __forceinline__ void mark_tiles(const TileIndex& ti, uint32_t W, int64_t c, uint32_t o,
                                           uint32_t o1) {
  if (c == 0) ti.first[0] = 0;
  int64_t hi = o1 / W;
  if (hi >= ti.ntiles) hi = ti.ntiles - 1;
  for (int64_t t = (int64_t)(o / W) + 1; t <= hi; ++t) ti.first[t] = (int32_t)(c + 1);
}

// The tiles past the last particle begin at cell M, and so does entry ntiles
// (by `stride` threads).
__device__ __forceinline__ void mark_last_tiles(const TileIndex& ti, int64_t W, int64_t M,
                                                int64_t total, int64_t thread, int64_t stride) {
  const int64_t past = total / W < ti.ntiles ? total / W + 1 : ti.ntiles;
  for (int64_t t = past + thread; t <= ti.ntiles; t += stride) ti.first[t] = (int32_t)M;
}

// U particles i[u] of a lane to the slots p[u] (c[u] < 0: none).  Copied
// array by array: all U loads of an array, and of the arrays around it, are
// in flight before the stores (an idle entry reads particle 0 of a non-empty
// input and stores nothing).
template <bool G, int U, typename S>
__device__ __forceinline__ void place_many(const PartP<S>& in, const PartP<S>& out, uint32_t* gperm,
                                           const uint32_t i[U], const uint32_t p[U],
                                           const int32_t c[U], bool has_x, bool has_y) {
  if constexpr (G) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c[u] >= 0) {
        gperm[p[u]] = i[u];
        out.cell[p[u]] = c[u];
      }
  } else {
    S x[U], y[U], v0[U], v1[U], v2[U], e[U];
    uint8_t lv[U];
    uint32_t id[U], j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) j[u] = c[u] >= 0 ? i[u] : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = has_x ? in.x[j[u]] : S(0);
#pragma unroll
    for (int u = 0; u < U; ++u) y[u] = has_y ? in.y[j[u]] : S(0);
#pragma unroll
    for (int u = 0; u < U; ++u) v0[u] = in.cx[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) v1[u] = in.cy[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) v2[u] = in.cz[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) e[u] = in.erot[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) lv[u] = in.vib[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) id[u] = in.pid[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c[u] < 0) continue;
      const int64_t q = p[u];
      if (has_x) out.x[q] = x[u];
      if (has_y) out.y[q] = y[u];
      out.cx[q] = v0[u];
      out.cy[q] = v1[u];
      out.cz[q] = v2[u];
      out.erot[q] = e[u];
      out.vib[q] = lv[u];
      out.pid[q] = id[u];
      out.cell[q] = c[u];
    }
  }
}

}  // namespace usp
