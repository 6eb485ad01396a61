// usp_internal.h -- shared declarations of libusp's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/usp.h"

namespace usp {

// moment planes, mom[k*M + c] (per unit mass, central about U)
enum Mom {
  M_N = 0, M_UX, M_UY, M_UZ, M_PXX, M_PYY, M_PZZ, M_PXY, M_PXZ, M_PYZ, M_EROT, M_IBAR,
  M_QTRX, M_QTRY, M_QTRZ, M_QROTX, M_QROTY, M_QROTZ, M_QIX, M_QIY, M_QIZ, NMOM
};
static_assert(NMOM == USP_NMOM, "moment plane count");

// cell-state planes, cs[k*M + c]
enum Cs {
  CS_NP = 0, CS_NDENS, CS_UX, CS_UY, CS_UZ, CS_TTR, CS_TROT, CS_TVIB,
  CS_PXX, CS_PYY, CS_PZZ, CS_PXY, CS_PXZ, CS_PYZ, CS_ETR, CS_EROT, CS_EVIB,
  CS_MU, CS_MUP, CS_TAUC, CS_ZROT, CS_ZVIB, CS_PR, CS_DT, CS_A, CS_B, CS_R2, CS_R3,
  CS_ALPHA, CS_OMA2, CS_NU, CS_EROT_NEW, CS_EVIB_NEW, CS_COLLIDE, CS_NBR_OK,
  // first-order FPM only: tau and the cell relaxation temperatures / level
  CS_FPM_TAU, CS_FPM_TTR_REL, CS_FPM_TROT_REL, CS_FPM_MREL, NCS
};
static_assert(NCS == USP_NCS, "cell-state plane count");

// Packed per-cell record for the particle update, stored after the FP64
// cell-state planes: the reconstructed fields and temperature floors in
// FP32, the quadrant stencils, and the cell coefficients.
struct alignas(16) CellRec {
  float U[3], T[3], P[6];  // interpolated fields (16-byte loads: 0..2)
  float fl[3];             // temperature floors, 5% of the cell values
  int32_t stencil;         // 4 quadrants x 5 bits: tx (2), ty (2), cross (1)
  float a, b, al, nu;
  double oma2, r2, A2, Pr, dt;
  int32_t collide, pad;
};
static_assert(sizeof(CellRec) == 128, "cell record size");

// Coefficients of the particle update taken from the cell (the per-cell
// reading of the coefficient chain): the chain of Secs. III.A.1-III.A.3
// at the cell's temperatures and Pi, in FP64.
struct alignas(16) CellPCoef {
  double L[6];             // Cholesky factor of Lambda
  double al, oma2, Trot_rel, mstar;
  int32_t flags, pad[3];   // PC_* bits
};
static_assert(sizeof(CellPCoef) == 96, "cell coefficient record size");
enum : int32_t { PC_SKIP = 1, PC_FALLBACK = 2, PC_NU_ZERO = 4, PC_CLAMP_ROT = 8, PC_CLAMP_M = 16 };

// bytes of the cell-state buffer: FP64 planes, then one CellRec per cell,
// then one CellPCoef per cell
__host__ __device__ inline size_t cellstate_bytes(int64_t M) {
  return (size_t)M * (NCS * sizeof(double) + sizeof(CellRec) + sizeof(CellPCoef));
}
__host__ __device__ inline CellRec* cell_records(double* cs, int64_t M) { return (CellRec*)(cs + (size_t)NCS * M); }
__host__ __device__ inline const CellRec* cell_records(const double* cs, int64_t M) {
  return (const CellRec*)(cs + (size_t)NCS * M);
}
__host__ __device__ inline CellPCoef* cell_pcoefs(double* cs, int64_t M) {
  return (CellPCoef*)(cell_records(cs, M) + M);
}
__host__ __device__ inline const CellPCoef* cell_pcoefs(const double* cs, int64_t M) {
  return (const CellPCoef*)(cell_records(cs, M) + M);
}

constexpr int VIB_MAX = 255;
constexpr int MAX_BOUNCE = 8;
constexpr int NB_KMAX = 512;
constexpr double KB = 1.380649e-23;
constexpr double PI = 3.14159265358979323846;

// stream tags of the counter-based generator
enum Tag : uint32_t { TAG_COLLIDE = 0, TAG_WALL = 1, TAG_CONSERVE = 2, TAG_INJECT = 3, TAG_FACE = 5 };

// Scalars the kernels need, passed by value (one copy per launch).
struct GasP {
  double R, theta, T_ref, mu_ref, omega, K;  // K = tau_c / (mu/p)
  int zrot_model; double Z_rot, Z_rot_inf, T_star;
  int zvib_model; double Z_vib, C1, C2, sigma_vib, d_ref;
  int pr_model; double Pr_const;
  int scheme;  // USP_SCHEME_USP or USP_SCHEME_FPM
  int gamma_cell, alpha_keep;  // USP_GAMMA_CELL, USP_ALPHA_SIGN_KEEP
};

// particle-update variants of the kernels: the USP-FPM chain per particle,
// the first-order FPM method, the USP-FPM chain taken from the cell
enum : int { MODE_USP = 0, MODE_FPM = 1, MODE_CELL = 2 };
inline int update_mode(const GasP& gas) {
  return gas.scheme == USP_SCHEME_FPM ? MODE_FPM : gas.gamma_cell ? MODE_CELL : MODE_USP;
}

struct GridP {
  int dim, nx, ny;
  int64_t M;
  double x0, y0, dx, dy, fnum;
  double idx, idy;  // 1/dx, 1/dy (first guess of a cell index; stencil weights)
  double inx;       // 1/nx (first guess of a cell's row)
  const double* volume;
  const uint8_t* flags;
};

struct BcP {
  int kind[4];
  double Tw[4];
  double fs_n, fs_T, fs_U[3], depth;
  int cyl;
  double cyl_xc, cyl_yc, cyl_r, cyl_Tw;
  double g[3];
  unsigned long long* surf;  // surface sums [element][USP_SURF_NQ] or null
  int surf_nbody;
};

template <typename S>
struct PartP {
  S *x, *y, *cx, *cy, *cz, *erot;
  uint8_t* vib;
  int32_t* cell;
  uint32_t* pid;
  int64_t* count;
  int64_t capacity;
};

// host-side argument checks of usp_update (without its workspace)
bool update_args_ok(const usp_grid* grid, const usp_gas* gas, const usp_bc* bc, double dt,
                    const double* cs, const int64_t* offsets, const usp_particles* p);

GasP make_gas(const usp_gas* g);
GridP make_grid(const usp_grid* g);
BcP make_bc(const usp_bc* b);
template <typename S> PartP<S> make_parts(const usp_particles* p);

// workspace layout (byte offsets into the caller's scratch buffer)
struct WsLayout {
  size_t key, perm, blocksums, t9, cell_i32, old_off, far_off, far, face_off, misc,
      tiles, chunk_off, chunk_part, cons_scal, sort_t, sort_tot, total;
};
// Cells split into chunks for the per-cell reductions (grids whose cells
// are far larger than a workgroup's share): slots per chunk, partial sums
// per chunk, bytes of a cell's conservation scalars, and the most chunks a
// binned state of `capacity` slots in M cells can have.
constexpr int BIG_CHUNK = 512;
constexpr int BIG_PARTS = 20;
constexpr size_t CONS_SCALAR_BYTES = 96;
inline int64_t chunks_max(int64_t capacity, int64_t M) {
  return (capacity + BIG_CHUNK - 1) / BIG_CHUNK + M;
}
// LDS stage of the fused particle phase, in particle slots (FP32 / FP64
// state), and the smallest tile window (the tile index array is sized for it)
constexpr int UPDATE_STAGE_F32 = 2048;
constexpr int UPDATE_STAGE_F64 = 1024;
constexpr int UPDATE_TILE_MIN = 128;
WsLayout ws_layout(int64_t M, int64_t capacity, int nfaces);

// The bin as a counting sort of input chunks (usp_sort.hip): nb digits (the
// cell, or a bucket of 2^shift cells), at most nchunks chunks.
constexpr int SORT_BUCKETS = 1024;
constexpr int64_t SORT_CHUNKS = 1024;
constexpr int64_t SORT_CHUNK_MIN = 2048;
constexpr int64_t SORT_SELF_SCAN = 32768;
struct SortPlan {
  int shift, nb, ld, bits, self_scan;  // ld: row stride of the digit counts
  int64_t nchunks;
};
SortPlan sort_plan(int64_t M, int64_t capacity);
// Which route the bin takes.  An input without segments is sorted (its
// order is unknown; 4.6M particles in random order: 0.46 ms against 2.2 ms
// through the appended-particle path).  A binned input is sorted on grids of
// at most SORT_BUCKETS cells (one pass, two launches: 19 against 73 us at
// 1e5 to 1e6 particles, and moves over any number of cells cost the same)
// and below a state size: the neighbour-group route moves fewer bytes per
// particle but takes twelve more launches.  On at most 1024 cells that holds
// for large states too: 1024 cells in a periodic box, 1M / 4M / 16M particles
// 49 / 123 / 490 us against 231 / 11,737 / 277,912 (particles that wrap round
// the box go to far cells, which the group route places cell by cell), and
// with no particle moved 31 / 85 / 332 against 82 / 271 / 1092.  Measured on
// cylinder grids, sort against group route: recording the order, 59 against 62 us at 1.7M
// particles, 111 against 94 at 4.6M, 133 against 92 at 6.6M; copying, 222
// against 325 at 4.6M and 289 against 250 at 6.6M.  The state size known
// on the host is the capacity (1.6 times the particles there).
constexpr int64_t SORT_GATHER_CAP = 5 << 20;
constexpr int64_t SORT_COPY_CAP = 8 << 20;
inline bool sort_route(int64_t M, int64_t capacity, bool binned, bool gather) {
  if (M > (int64_t)SORT_BUCKETS * SORT_BUCKETS) return false;
  return !binned || M <= SORT_BUCKETS || capacity <= (gather ? SORT_GATHER_CAP : SORT_COPY_CAP);
}
struct TileIndex;
template <typename S, bool G>
hipError_t sort_launches(const GridP& g, const PartP<S>& in, const PartP<S>& out, int64_t* offsets,
                         const int64_t* in_offsets, char* ws, const WsLayout& L, uint32_t* perm,
                         int64_t* counters, hipStream_t st, const TileIndex& ti);
int n_faces(const GridP& g);

// Tile index of the fused particle phase, made by the bin beside its
// offsets when first is not null: first[t] (t = 0..ntiles) as launch_tiles
// gives it.
struct TileIndex {
  int32_t* first;
  int64_t ntiles;
  int stage;
};

// launchers (return hipError_t of the last launch)
template <typename S>
hipError_t launch_bin(const GridP& g, const PartP<S>& in, const PartP<S>& out, int64_t* offsets,
                      const int64_t* in_offsets, char* ws, const WsLayout& L, int64_t* counters,
                      hipStream_t st, uint32_t* gather_perm = nullptr,
                      TileIndex ti = TileIndex{nullptr, 0, 0});
template <typename S>
hipError_t launch_moments(const GridP& g, const PartP<S>& p, const int64_t* offsets, double* mom,
                          hipStream_t st, const uint32_t* gather_perm = nullptr);
// the particle update's coefficients of every cell (MODE_CELL only; else
// nothing)
hipError_t launch_cell_coef(const GridP& g, const GasP& gas, double* cs, hipStream_t st);
hipError_t launch_reconstruct(const GridP& g, const GasP& gas, const double* mom, double dt,
                              const double* dt_cell, double* cs, int64_t* counters, hipStream_t st);
// launch_moments followed by launch_reconstruct; on 1D and 2D grids that
// update_solo takes in one launch, and without the stencil words, which the
// particle phase of a step makes there.
template <typename S>
hipError_t launch_cells(const GridP& g, const GasP& gas, const PartP<S>& p, const int64_t* offsets,
                        double* mom, double dt, const double* dt_cell, double* cs,
                        int64_t* counters, hipStream_t st, const uint32_t* gather_perm = nullptr);
hipError_t launch_sample_fields(const GridP& g, const double* mom, double* acc, hipStream_t st);
template <typename S>
hipError_t launch_collide(const GridP& g, const GasP& gas, const double* cs, const int64_t* offsets,
                          const PartP<S>& p, uint64_t seed, uint64_t step, int64_t* counters,
                          hipStream_t st);
// The stencils of the reconstruction (1D, 2D) and, under the per-cell
// reading, the cells' coefficients, after the cell state.
hipError_t launch_stencil(const GridP& g, const GasP& gas, double* cs, hipStream_t st);
// A step of a grid whose cells are split into chunks of BIG_CHUNK slots
// (partial sums combined in chunk order), on a binned state: the chunk
// index of the cells; the moments, cell state and stencils (apply: the
// scalings of the collision before are applied on the way); the particle
// update and the conservation's picks and scalars; the scalings alone.
hipError_t launch_chunks(const GridP& g, const int64_t* offsets, char* ws, const WsLayout& L,
                         hipStream_t st);
template <typename S>
hipError_t launch_cells_split(const GridP& g, const GasP& gas, const PartP<S>& p,
                              const int64_t* offsets, double* mom, double dt, const double* dt_cell,
                              double* cs, bool apply, char* ws, const WsLayout& L,
                              int64_t* counters, hipStream_t st);
template <typename S>
hipError_t launch_collide_split(const GridP& g, const GasP& gas, const double* cs,
                                const int64_t* offsets, const PartP<S>& p, uint64_t seed,
                                uint64_t step, char* ws, const WsLayout& L, int64_t* counters,
                                hipStream_t st);
template <typename S>
hipError_t launch_cons_apply(const PartP<S>& p, char* ws, const WsLayout& L, hipStream_t st);
template <typename S>
hipError_t launch_conserve(const GridP& g, const GasP& gas, const double* cs,
                           const int64_t* offsets, const PartP<S>& p, uint64_t seed, uint64_t step,
                           int64_t* counters, hipStream_t st);
template <typename S>
hipError_t launch_advect(const GridP& g, const GasP& gas, const BcP& bc, double dt,
                         const PartP<S>& p, uint64_t seed, uint64_t step, char* ws,
                         const WsLayout& L, int64_t* counters, hipStream_t st);

template <typename S>
hipError_t launch_inject(const GridP& g, const GasP& gas, const BcP& bc, double dt,
                         const PartP<S>& p, uint64_t seed, uint64_t step, char* ws,
                         const WsLayout& L, int64_t* counters, hipStream_t st);
// Where the particle phase of a taped step (FP64) keeps, per slot, the binned
// state, the velocity and rotational energy after the collision, the state
// after the conservation and the y velocity after the flight.
struct TapeOut {
  double *y, *cx, *cy, *cz, *erot;
  uint8_t* vib;
  int32_t* cell;
  uint32_t* pid;
  double *ccx, *ccy, *ccz, *cerot;
  double *kcx, *kcy, *kcz, *kerot;
  uint8_t* kvib;
  double* fcy;
};
// launch_update (in a step, gathering, USP-FPM per particle) that fills a
// tape.
hipError_t launch_update_taped(const GridP& g, const GasP& gas, const BcP& bc, double dt,
                               double* cs, const int64_t* offsets, const PartP<double>& p,
                               uint64_t seed, uint64_t step, char* ws, const WsLayout& L,
                               int64_t* counters, hipStream_t st, const PartP<double>& src,
                               const uint32_t* gather_perm, const TapeOut& tape);
// Grids whose particle phase takes one cell a workgroup (at most one on a
// CU).
inline bool update_solo(const GridP& g) { return g.M <= 256; }
// The fused particle phase on p (binned), or, with gather_perm, on the
// particles of `src` in the order gather_perm gives (slot j holds
// src[gather_perm[j]]), the results written to p (whose cells the
// gathering bin has set).  In a step, step_cs is cs: the tile index is made
// already, and on update_solo grids the stencil words are still to be.
template <typename S>
hipError_t launch_update(const GridP& g, const GasP& gas, const BcP& bc, double dt,
                         const double* cs, const int64_t* offsets, const PartP<S>& p,
                         uint64_t seed, uint64_t step, char* ws, const WsLayout& L,
                         int64_t* counters, hipStream_t st, const PartP<S>* src = nullptr,
                         const uint32_t* gather_perm = nullptr, hipEvent_t ev_begin = nullptr,
                         hipEvent_t ev_end = nullptr, double* step_cs = nullptr);
// Adds to *found the number of NaN or infinite values among the live
// particles' floating arrays and, when given, the moment and FP64
// cell-state planes of the occupied cells.
template <typename S>
hipError_t launch_check(const GridP& g, const PartP<S>& p, const double* mom, const double* cs,
                        int64_t* found, hipStream_t st);

// first[t] (t = 0..ntiles) = first cell of tile t: the cells whose first
// particle slot lies in [t T, (t+1) T).  With stage > 0 the window T is
// update_tile(stage, offsets[M], M), taken on the device from the binned
// count (the given T must be the window of a count at least as large, so
// that ntiles tiles cover it); with stage = 0 it is T as given.
hipError_t launch_tiles(const int64_t* offsets, int64_t M, int64_t T, int64_t ntiles,
                        int32_t* first, hipStream_t st, int stage = 0);
template <typename S>
hipError_t launch_batch(const GridP& g, const GasP& gas, double dt, const double* dt_cell,
                        double* mom, double* cs, const int64_t* offsets, const PartP<S>& p,
                        int tile, int steps_per_launch, uint64_t seed, uint64_t step,
                        int nsteps, char* ws, const WsLayout& L, int64_t* counters,
                        hipStream_t st);

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Tile window of the fused particle phase: a tile holds the cells whose
// first particle lies in one window, so it spans the window plus the part
// of its last cell past the window's end.  The window is the stage less
// 13/8 of the mean particles per cell (n / M), kept within [stage/8,
// 7 stage/8], so that most tiles fit the stage; a state too small to fill
// the chip with such windows is cut into UPDATE_TILES of them (two
// workgroups on each of 256 CUs, one round).  A step uncut and cut into 256,
// 512 and 1024: 4096 cells of 20 FP32 particles 129 / 94 / 94 / 102 us, of 50
// 106 / 91 / 88 / 96; 8000 of 50 116 / 112 / 107 / 112; 2048 of 400 145 / 145 /
// 145 / 138; FP64 1024 of 200 133 / 134 / 110 / 122, 2048 of 20 128 / 89 / 96 /
// 96.  (In a buffer of 47 times the particles the empty tiles come behind
// two full rounds of CUs instead of one: usp_update of 200,000 FP64 particles
// in 9.4M slots 70 uncut, 83 cut.)
constexpr int64_t UPDATE_TILES = 512;
__host__ __device__ inline int64_t stage_window(int stage, int64_t n, int64_t M) {
  const int64_t ppc = M > 0 ? (n + M - 1) / M : stage;
  int64_t t = stage - ppc - ppc / 2 - ppc / 8;
  const int64_t lo = stage / 8, hi = stage - stage / 8;
  if (t < lo) t = lo;
  if (t > hi) t = hi;
  return t < UPDATE_TILE_MIN ? UPDATE_TILE_MIN : t;
}
__host__ __device__ inline int64_t update_tile(int stage, int64_t n, int64_t M) {
  int64_t t = stage_window(stage, n, M);
  const int64_t even = (n + UPDATE_TILES - 1) / UPDATE_TILES;
  if (t > even) t = even;
  return t < UPDATE_TILE_MIN ? UPDATE_TILE_MIN : t;
}
// Tiles that any count up to `capacity` needs: the count over its window
// grows with the count, except that an evenly cut state needs UPDATE_TILES
// (and no window is below UPDATE_TILE_MIN).
inline int64_t update_ntiles(int stage, int64_t capacity, int64_t M) {
  const int64_t n = cdiv(capacity, update_tile(stage, capacity, M));
  const int64_t most = cdiv(capacity, UPDATE_TILE_MIN);
  const int64_t even = n > UPDATE_TILES ? n : UPDATE_TILES;
  return even < most ? even : most;
}

}  // namespace usp
