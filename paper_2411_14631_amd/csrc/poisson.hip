// Uniform-level Poisson solver on gfx950: the preconditioned conjugate-
// gradient iterates of PPCG (Ghysels & Vanroose 2014, Algorithm 4) with the
// seven-point preconditioner 13/12 (centre), 1/6 (face neighbours), in one of
// two forms chosen by the problem's size and shape (plan_sweeps):
//
// Pipelined form (small problems: each launch counts, the vectors sit in the
// caches; and thin grids).  One launch per iteration i: every workgroup sums the partials of
// gamma_i = r_i.u_i and delta_i = w_i.u_i that the launch before left, in
// one fixed order, and forms alpha_i and beta_i itself; then a z-marching
// stencil sweep forms m_i = M^-1 w_i and n_i = A m_i from w_i staged in LDS,
// updates the eight recurrence vectors (z, q, s, p, then x, r, u, w) and
// leaves the partials of gamma_{i+1}, delta_{i+1}.  128 bytes per cell.
//
// Two-sweep form (large problems: HBM bandwidth counts).  The same iterates
// with the fewest vectors streamed: u = M^-1 r, s = A p, q = M^-1 s, z = A q
// and w = A u hold by definition, so only x, r and p are kept and the others
// are applied on the fly, or formed when asked for:
//   direction  p_i = M^-1 r_i + beta_i p_{i-1} on the tile and its one-cell
//              halo, partials of p_i.(A p_i);
//   update     r_{i+1} = r_i - alpha_i A p_i on the tile and its one-cell
//              halo, x_{i+1}, partials of gamma_{i+1} = r_{i+1}.(M^-1 r_{i+1}).
// 64 bytes per cell (r, p read and p written; p, r, x read and r, x written).
// r and p are double-buffered: neighbouring workgroups read the old one.
// Measured per iteration: 256^3 243 us (pipelined, with its scalar step in a
// launch of its own: 420; a 1 GiB device copy runs at 5.07 TB/s, at which 64
// bytes per cell take 212 us), 160^3 60 us (117), 128^3 40 us (60).
//
// Kernel geometry of all sweeps: a workgroup owns a TX x TY column of cells
// and a chunk of z planes.  Every point of the plane with its two-cell halo
// has a thread of its own, so the neighbours along z are the thread's own
// registers, those in the plane are four LDS reads per stencil, and no lane
// branches: a lane outside the grid loads a clamped address and selects 0.
// The second stencil of a sweep runs one plane behind the first; with both
// planes double-buffered in LDS one barrier per plane orders everything.
// Loads run two planes ahead of their use.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/ry_poisson.h"
#include "staging.h"

namespace ryp {


// A TX x TY tile: the plane with its halo and its threads (two-sweep form).
// 32 x 16: of 32 x 10, 32 x 16, 32 x 24 and 60 x 12 the fastest (256^3: 301,
// 238, 279, 301 us per iteration): two 768-thread workgroups per CU, whole
// tiles on the usual sides.
template <int TX_, int TY_>
struct Tile {
  static constexpr int TX = TX_, TY = TY_, EX = TX + 4, EY = TY + 4;
  static constexpr int NT = (EX * EY + 63) / 64 * 64, NWV = NT / 64;
  static constexpr int PL = NT + 2 * EX;   // an LDS plane: every thread's four neighbours exist
};
using SmallTile = Tile<32, 8>;             // pipelined form
using LargeTile = Tile<32, 16>;            // two-sweep form
constexpr int NTH = 256;                   // threads of the whole-vector kernels
constexpr int BATCH = 16;                                // iterations per captured graph (even: see step[])
constexpr int NVEC = 9;                                  // pipelined: x r u w0 w1 z q s p; two-sweep: x r0 r1 p0 p1
// Cells from which the two-sweep form is the faster one: its second launch
// and reduction cost about 8 us an iteration more, its halved traffic gains
// more than that from here on (both forms, us per iteration: 96^3 22.3
// pipelined / 28.2 two-sweep, 101 x 99 x 103 29.0 / 32.7, 128^3 44.4 / 39.6,
// 160^3 105 / 60).
constexpr int64_t kTwoSweepCells = int64_t(5) << 18;
// They also have to be thick enough along z (a sweep loads four planes beside
// its chunk's own, and works on two of them) and to fill the larger tile (us
// per iteration, pipelined / two-sweep; n2 x n1 x n0): 1 x 2048^2 131 / 276, 3 x 1024^2 84 / 100,
// 4 x 1024^2 111 / 110, 6 x 1024^2 165 / 130; 30,000 x 8 x 8 (an eighth of the
// tile) 74 / 130, 10,000 x 12 x 12 (0.28) 53 / 60, 20,000 x 16 x 16 (a half) 147 / 107.
constexpr int kTwoSweepPlanes = 4;
constexpr double kTwoSweepFill = 1.0 / 3;
// Workgroups per sweep at most (z chunks are added up to it).  Large: two per
// CU, all resident, no second round.  Small: each workgroup pays the scalar
// step and four halo planes, so few, thicker chunks (64^3: 11.3 us per
// iteration with 512, 15.5 with 1024, 11.8 with 256) -- up to kLongChunk
// planes, past which the chain of planes counts: twice as many then, and as
// many as fit a CU (six) where hardly a lane has a cell (512 / 1024 / 1536
// workgroups: 30,000 x 8 x 8 83 / 74 / 91 us, 81,920 x 4 x 4 179 / 137 / 129,
// 1,310,720 x 1 x 1 2384 / 1736 / 1322).
constexpr int kTargetSmall = 512, kTargetLong = 1024, kTargetThin = 1536, kTargetLarge = 512;
constexpr int kLongChunk = 16;
constexpr double kThinFill = 1.0 / 8;
// Every workgroup of a sweep sums all partials itself, up to this many of
// them; past it a launch of 2.5 us leaves kSums of them for the sweeps to read
// (us per iteration without / with: 1000 x 1000 (2016 workgroups) 49 / 41,
// 16,384 x 128 (4096) 122 / 76, 1 x 4096^2 (32,768) 3106 / 480).
constexpr int kMaxPartials = 1024, kSums = 256;

struct Grid {
  int32_t n0, n1, n2, bc;
};

// Scalars carried between launches, device-resident.  A kernel's workgroups
// all read what one of them writes for the next launch, so nothing is read
// and written by the same kernel: the pipelined iteration i reads
// step[i & 1] and writes step[1 - (i & 1)] (the host knows i, so the slot is
// a launch argument); of the two-sweep form the direction kernel reads
// step[0] and writes dir, the update kernel the other way round.  Once the
// solve has stopped, the launches left in a graph only pass `done` on.
struct Scalars {
  double gamma0, eps_target;
  struct Step {
    double alpha_prev, gamma_prev;
    int32_t iter, done;   // index of the next iterate to test
  } step[2];
  struct Dir {
    double gamma;
    int32_t iter, done;
  } dir;
  int32_t max_iter;       // stop when the iterate's index reaches it
};

struct IterArgs {
  Grid g;
  double* w[2];
  double *x, *r, *u, *z, *q, *s, *p;
  Scalars* sc;
  double* hist;
  double* part;   // written: two sets (by parity) of [2][gridDim.x]
  double* sum;    // read: two sets of [2][nsum] (part itself, or its sums by reduce_kernel)
  int32_t nsum;
  int32_t cz;     // z planes per workgroup
  int32_t par;    // parity of the iteration index
};

struct CgArgs {
  Grid g;
  double *x, *r[2], *p[2];
  Scalars* sc;
  double* hist;
  double *part_g, *part_d;   // written: [gridDim.x] each
  double *sum_g, *sum_d;     // read: [nsum] each (as IterArgs::sum)
  int32_t nsum;
  int32_t cz;
};

__device__ __forceinline__ int wrap(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}

// Value of v at (X, Y, Z) under the boundary rule (zero Dirichlet: 0 off the grid).
__device__ __forceinline__ double grid_val(const double* __restrict__ v, const Grid& g, int X, int Y, int Z) {
  if (g.bc == RY_PBC_PERIODIC) {
    if (unsigned(X) >= unsigned(g.n0)) X = wrap(X, g.n0);
    if (unsigned(Y) >= unsigned(g.n1)) Y = wrap(Y, g.n1);
    if (unsigned(Z) >= unsigned(g.n2)) Z = wrap(Z, g.n2);
  } else if (X < 0 || X >= g.n0 || Y < 0 || Y >= g.n1 || Z < 0 || Z >= g.n2) {
    return 0.0;
  }
  return v[int64_t(X) + int64_t(g.n0) * (int64_t(Y) + int64_t(g.n1) * Z)];
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD a
// contiguous slab of columns so that halo rows stay in one L2.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
  const int x = bid & 7, j = bid >> 3;
  const int q = nblocks >> 3, r = nblocks & 7;
  return x * q + (x < r ? x : r) + j;
}

// Block-wide sum of NQ values per thread over the NWV wavefronts, to every
// thread, in a fixed order.
template <int NQ, int NWV>
__device__ __forceinline__ void block_sum(double (&v)[NQ], double (*red)[NWV]) {
  const int wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    v[k] = wave_sum(v[k]);
    if ((threadIdx.x & 63) == 0) red[k][wv] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    v[k] = 0.0;
#pragma unroll
    for (int j = 0; j < NWV; ++j) v[k] += red[k][j];
  }
}

// A thread's share of the sum of n partials over NTH threads: fixed order,
// loads in flight together.
__device__ __forceinline__ double strided_sum(const double* __restrict__ part, int n) {
  double a[4] = {};
  for (int k = threadIdx.x; k - int(threadIdx.x) < n; k += 4 * NTH) {
    double v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = part[min(k + j * NTH, n - 1)];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] += k + j * NTH < n ? v[j] : 0.0;
  }
  return (a[0] + a[1]) + (a[2] + a[3]);
}

// Sum of n partials by one wavefront, to each of its lanes: fixed order,
// loads in flight together.
__device__ __forceinline__ double wave_total(const double* __restrict__ part, int n) {
  const int lane = threadIdx.x & 63;
  double a[8] = {};
  for (int k = lane; k - lane < n; k += 8 * 64) {
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = part[min(k + j * 64, n - 1)];
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] += k + j * 64 < n ? v[j] : 0.0;
  }
  return wave_sum(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
}

// eps_i = sqrt(gamma_i / gamma_0) and whether the solve stops at iterate i.
__device__ __forceinline__ bool stop_at(const Scalars* sc, int i, double gamma, double& eps) {
  const double g0 = (i == 0) ? gamma : sc->gamma0;
  eps = (g0 > 0.0 && gamma > 0.0) ? sqrt(gamma / g0) : 0.0;
  return eps <= sc->eps_target || i >= sc->max_iter || i >= RY_POISSON_HIST - 1;
}

// The column of a workgroup: its first cell, its z planes, and the boundary
// rule.  DOWN: the chunk's planes are marched from the last to the first (the
// stencils are symmetric, so a sweep only sees other planes).
template <typename T, bool DOWN = false>
struct Chunk {
  int x0, y0, z0, z1, n2;
  bool periodic;
  int64_t plane;
  __device__ __forceinline__ Chunk(const Grid& g, int cz) {
    const int gx = (g.n0 + T::TX - 1) / T::TX, gy = (g.n1 + T::TY - 1) / T::TY;
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    x0 = (b % gx) * T::TX;
    y0 = ((b / gx) % gy) * T::TY;
    z0 = (b / (gx * gy)) * cz;
    z1 = min(z0 + cz, g.n2);
    n2 = g.n2;
    plane = int64_t(g.n0) * g.n1;
    periodic = g.bc == RY_PBC_PERIODIC;
  }
  __device__ __forceinline__ bool inside(const Grid& g, int X, int Y) const {
    return periodic || (X >= 0 && X < g.n0 && Y >= 0 && Y < g.n1);
  }
  // index in a grid plane of the point (X, Y) of the tile with its halo, or
  // of its periodic image; off a Dirichlet grid the nearest cell's
  __device__ __forceinline__ int index(const Grid& g, int X, int Y) const {
    if (periodic) {
      // past the halo of the last cell nothing is read: one period at most
      X = min(X, g.n0 + 1);
      Y = min(Y, g.n1 + 1);
      X = g.n0 == 1 ? 0 : (X < 0 ? X + g.n0 : (X >= g.n0 ? X - g.n0 : X));
      Y = g.n1 == 1 ? 0 : (Y < 0 ? Y + g.n1 : (Y >= g.n1 ? Y - g.n1 : Y));
    } else {
      X = min(max(X, 0), g.n0 - 1);
      Y = min(max(Y, 0), g.n1 - 1);
    }
    return X + g.n0 * Y;
  }
  // the grid's plane number of the march's plane z
  __device__ __forceinline__ int number(int z) const { return DOWN ? z0 + z1 - 1 - z : z; }
  // whether plane z is in the grid (or its continuation)
  __device__ __forceinline__ bool inz(int z) const { return periodic || unsigned(number(z)) < unsigned(n2); }
  // offset of the grid plane that plane z is (a neighbour of the grid: clamped)
  __device__ __forceinline__ int64_t at(int z) const {
    z = number(z);
    if (unsigned(z) >= unsigned(n2)) z = periodic ? wrap(z, n2) : (z < 0 ? 0 : n2 - 1);
    return plane * z;
  }
};

// A thread's point of its workgroup's column.  ix2: its index in a grid
// plane (any point with the two-cell halo); ix1, ix0: the index of the
// nearest point of the one-cell halo and of the tile's own cells, which a
// lane further out loads instead (no lines of its own).  in: inside the grid
// (or its periodic continuation); own: one of the tile's cells.
template <typename T, bool DOWN = false>
struct Point : Chunk<T, DOWN> {
  using C = Chunk<T, DOWN>;
  using C::z0, C::z1, C::plane, C::at, C::inz, C::number;
  int c, ix2, ix1, ix0;
  bool in, own;
  __device__ __forceinline__ Point(const Grid& g, int cz) : C(g, cz) {
    const int t = threadIdx.x, lx = t % T::EX - 2, ly = t / T::EX - 2;   // ly past the tile's halo: spare lanes
    c = t + T::EX;
    const int X = C::x0 + lx, Y = C::y0 + ly;
    own = lx >= 0 && lx < T::TX && ly >= 0 && ly < T::TY && X < g.n0 && Y < g.n1;
    in = C::inside(g, X, Y);
    auto into = [&](int h) {
      return C::index(g, C::x0 + min(max(lx, -h), T::TX - 1 + h), C::y0 + min(max(ly, -h), T::TY - 1 + h));
    };
    ix2 = into(2);
    ix1 = into(1);
    ix0 = min(C::x0 + min(max(lx, 0), T::TX - 1), g.n0 - 1) +
          g.n0 * min(C::y0 + min(max(ly, 0), T::TY - 1), g.n1 - 1);
  }
  // v at plane z (0 off the grid), loaded for every lane; planes past the
  // last one the chunk reads are that one again
  __device__ __forceinline__ double load2(const double* __restrict__ v, int z) const {
    z = min(z, z1 + 1);
    const double a = v[at(z) + ix2];
    return (in && inz(z)) ? a : 0.0;
  }
  // the chunk's planes and one either side, one-cell halo
  __device__ __forceinline__ double load1(const double* __restrict__ v, int z) const { return v[at(min(z, z1)) + ix1]; }
  // the chunk's own cells
  __device__ __forceinline__ int64_t cell(int z) const { return plane * number(max(z0, min(z, z1 - 1))) + ix0; }
};

// The four in-plane neighbours of point c in an LDS plane, then the ones
// below and above.
template <typename T>
__device__ __forceinline__ double six(const double* pl, int c, double below, double above) {
  double s = pl[c - 1];
  s += pl[c + 1];
  s += pl[c - T::EX];
  s += pl[c + T::EX];
  s += below;
  s += above;
  return s;
}

// ---------------------------------------------------------------------------
// The pipelined iteration.  Bound: at the sizes it serves, the chain of one
// launch; everything the first plane needs is requested together, before
// the partials' reduction, and the scalar step costs no launch of its own
// (48 x 40 x 36: 8.2 us per iteration, 12.7 with a one-workgroup launch for
// the scalars and loads issued plane by plane; 64^3 11.3, was 15.4; 96^3
// 22.3, was 34.7).  One thread per cell and two rounds over the halo points:
// a thread per halo point costs more wavefronts, whose prologue is what
// counts here (48 x 40 x 36 9.9 us).
//
// MANY: more workgroups than the chip holds at once (thin grids).  Their
// throughput counts instead: six to a CU instead of four, the recurrence
// vectors streamed past the caches, one sum per thread to read.
// ---------------------------------------------------------------------------
template <bool MANY>
__device__ __forceinline__ double stream_load(const double* p) {
  if constexpr (MANY) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool MANY>
__device__ __forceinline__ void stream_store(double v, double* p) {
  if constexpr (MANY) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <int PC, bool MANY>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(MANY ? 6 : 4))) void ppcg_iterate_kernel(IterArgs A) {
  constexpr int TX = SmallTile::TX, TY = SmallTile::TY;
  constexpr int WX = TX + 4, WPL = WX * (TY + 4), NW = (WPL + NTH - 1) / NTH;   // planes with a 2-cell halo
  constexpr int MX = TX + 2, MPL = MX * (TY + 2), NM = (MPL + NTH - 1) / NTH;   // and a 1-cell halo
  static_assert(TX * TY == NTH && kSums == NTH, "one thread per cell, and per sum");
  __shared__ double Wp[5][WPL], Mp[3][MPL];
  __shared__ double red[2][NTH / 64];
  Scalars* sc = A.sc;
  const Grid g = A.g;
  const Chunk<SmallTile> C(g, A.cz);
  const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
  const int nb = gridDim.x;
  const double* sum_in = A.sum + int64_t(A.par) * 2 * A.nsum;
  double* part_out = A.part + int64_t(A.par ^ 1) * 2 * nb;
  const double* __restrict__ win = A.w[A.par];
  double* __restrict__ wout = A.w[A.par ^ 1];
  const bool own = C.x0 + tx < g.n0 && C.y0 + ty < g.n1;
  const int64_t col = min(C.x0 + tx, g.n0 - 1) + int64_t(g.n0) * min(C.y0 + ty, g.n1 - 1);
  // the thread's points of a plane with the 2-cell halo: a grid index each
  // (off a Dirichlet grid: some index, and 0 selected)
  int ixw[NW];
  bool inw[NW], inm[NM];
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    const int k = min(tid + j * NTH, WPL - 1), X = C.x0 - 2 + k % WX, Y = C.y0 - 2 + k / WX;
    ixw[j] = C.index(g, X, Y);
    inw[j] = C.inside(g, X, Y);
  }
#pragma unroll
  for (int j = 0; j < NM; ++j) {
    const int k = tid + j * NTH;
    inm[j] = C.inside(g, C.x0 - 1 + k % MX, C.y0 - 1 + k / MX);
  }
  auto load_w = [&](int z, double (&v)[NW]) {
    const double* pl = win + C.at(z);
    const bool ok = C.inz(z);
#pragma unroll
    for (int j = 0; j < NW; ++j) v[j] = pl[ixw[j]];
#pragma unroll
    for (int j = 0; j < NW; ++j) v[j] = ok && inw[j] ? v[j] : 0.0;
  };
  struct Rec {
    double z, q, s, p, u, x, r;
  };
  auto load_rec = [&](int z) {
    const int64_t i = col + C.plane * z;
    return Rec{stream_load<MANY>(A.z + i), stream_load<MANY>(A.q + i), stream_load<MANY>(A.s + i),
               stream_load<MANY>(A.p + i), stream_load<MANY>(A.u + i), stream_load<MANY>(A.x + i),
               stream_load<MANY>(A.r + i)};
  };
  // the first plane's five w planes and recurrences, and the partials
  double wr[5][NW];
#pragma unroll
  for (int k = 0; k < 5; ++k) load_w(C.z0 - 2 + k, wr[k]);
  Rec rec{}, nxt{};
  if constexpr (!MANY) rec = load_rec(C.z0);
  double gd[2];
  if constexpr (MANY) {
    gd[0] = sum_in[tid];
    gd[1] = sum_in[kSums + tid];
  } else {
    gd[0] = strided_sum(sum_in, A.nsum);
    gd[1] = strided_sum(sum_in + A.nsum, A.nsum);
  }
  // looked at with the loads under way
  const Scalars::Step st = sc->step[A.par];
  if (st.done) {
    if (blockIdx.x == 0 && tid == 0) sc->step[A.par ^ 1] = st;
    return;
  }
  // plane slots: w at z in slot (z - z0 + 2) mod 5, m at z in (z - z0 + 1) mod 3
  auto wslot = [&](int z) { return (z - C.z0 + 2) % 5; };
  auto mslot = [&](int z) { return (z - C.z0 + 1) % 3; };
  auto store_w = [&](int slot, const double (&v)[NW]) {
#pragma unroll
    for (int j = 0; j < NW; ++j)
      if (tid + j * NTH < WPL) Wp[slot][tid + j * NTH] = v[j];
  };
#pragma unroll
  for (int k = 0; k < 5; ++k) store_w(k, wr[k]);
  block_sum(gd, red);   // its barrier also publishes the planes
  const double gamma = gd[0], delta = gd[1];
  double eps;
  const bool stop = stop_at(sc, st.iter, gamma, eps);
  double beta = 0.0, alpha = gamma / delta;
  if (st.iter > 0) {
    beta = gamma / st.gamma_prev;
    alpha = gamma / (delta - beta * gamma / st.alpha_prev);
  }
  if (blockIdx.x == 0 && tid == 0) {
    A.hist[st.iter] = eps;
    if (st.iter == 0) sc->gamma0 = gamma;
    if (stop) sc->step[A.par ^ 1] = {st.alpha_prev, st.gamma_prev, st.iter, 1};
    else sc->step[A.par ^ 1] = {alpha, gamma, st.iter + 1, 0};
  }
  if (stop) return;
  // the six neighbours of point c of plane b (row stride S), a below, d above
  auto six_lds = [](const double* a, const double* b, const double* d, int c, int S) {
    double s = b[c - 1];
    s += b[c + 1];
    s += b[c - S];
    s += b[c + S];
    s += a[c];
    s += d[c];
    return s;
  };
  // m = M^-1 w on the plane z (1-cell halo); 0 off the grid under Dirichlet
  auto comp_m = [&](int z) {
    const double *wm = Wp[wslot(z - 1)], *w0 = Wp[wslot(z)], *wp = Wp[wslot(z + 1)];
    double* dst = Mp[mslot(z)];
    const bool ok = C.inz(z);
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      const int k = tid + j * NTH;
      if (k >= MPL) continue;
      const int c = (k % MX + 1) + WX * (k / MX + 1);
      const double v = PC == RY_PC_STENCIL7 ? (13.0 / 12.0) * w0[c] + (1.0 / 6.0) * six_lds(wm, w0, wp, c, WX) : w0[c];
      dst[k] = ok && inm[j] ? v : 0.0;
    }
  };
  comp_m(C.z0 - 1);
  comp_m(C.z0);
  comp_m(C.z0 + 1);
  __syncthreads();
  double acc[2] = {0.0, 0.0};
  for (int z = C.z0; z < C.z1; ++z) {
    const bool more = z + 1 < C.z1;
    if (more) {
      load_w(z + 3, wr[0]);
      if constexpr (!MANY) nxt = load_rec(z + 1);
    }
    if constexpr (MANY) rec = load_rec(z);
    if (own) {
      const int64_t i = col + C.plane * z;
      const double* m0 = Mp[mslot(z)];
      const int c = (tx + 1) + MX * (ty + 1);
      const double mv = m0[c];
      const double nv = 6.0 * mv - six_lds(Mp[mslot(z - 1)], m0, Mp[mslot(z + 1)], c, MX);   // n_i = A m_i
      const double wv = Wp[wslot(z)][(tx + 2) + WX * (ty + 2)];
      const double zz = nv + beta * rec.z;
      const double qq = mv + beta * rec.q;
      const double ss = wv + beta * rec.s;
      const double pp = rec.u + beta * rec.p;
      const double rr = rec.r - alpha * ss;
      const double uu = rec.u - alpha * qq;
      const double ww = wv - alpha * zz;
      stream_store<MANY>(zz, A.z + i);
      stream_store<MANY>(qq, A.q + i);
      stream_store<MANY>(ss, A.s + i);
      stream_store<MANY>(pp, A.p + i);
      stream_store<MANY>(rec.x + alpha * pp, A.x + i);
      stream_store<MANY>(rr, A.r + i);
      stream_store<MANY>(uu, A.u + i);
      stream_store<MANY>(ww, wout + i);
      acc[0] += rr * uu;
      acc[1] += ww * uu;
    }
    if (more) {
      store_w(wslot(z + 3), wr[0]);
      __syncthreads();
      comp_m(z + 2);
      __syncthreads();
      if constexpr (!MANY) rec = nxt;
    }
  }
  block_sum(acc, red);   // the barrier after comp_m separates it from the first sum
  if (tid == 0) {
    part_out[blockIdx.x] = acc[0];
    part_out[nb + blockIdx.x] = acc[1];
  }
}

// ---------------------------------------------------------------------------
// The two sweeps of the large problems.  Bound: HBM (256^3: direction 105 us
// for 403 MB, update 137 us for 671 MB: 3.8 and 4.9 TB/s).  The direction
// sweep marches down, so that it starts on the planes the update sweep left
// in the caches (1.5% at 256^3).
// ---------------------------------------------------------------------------
// gamma_i, the stopping test and beta_i; p_i = M^-1 r_i + beta_i p_{i-1} on
// the tile and its one-cell halo; partials of p_i.(A p_i).
template <int PC>
__global__ __launch_bounds__(LargeTile::NT) void cg_direction_kernel(CgArgs A) {
  using T = LargeTile;
  Scalars* sc = A.sc;
  const Scalars::Step st = sc->step[0];
  if (st.done) return;
  __shared__ double Rp[2][T::PL], Pp[2][T::PL];
  __shared__ double red[1][T::NWV];
  const Point<T, true> P(A.g, A.cz);
  const double* __restrict__ r = A.r[st.iter & 1];
  const double* __restrict__ pold = A.p[st.iter & 1];
  double* __restrict__ pnew = A.p[(st.iter & 1) ^ 1];
  double rm = P.load2(r, P.z0 - 2), r0 = P.load2(r, P.z0 - 1), r1 = P.load2(r, P.z0);
  double rq[2] = {P.load2(r, P.z0 + 1), P.load2(r, P.z0 + 2)};
  double pq[2] = {P.load1(pold, P.z0 - 1), P.load1(pold, P.z0)};
  // the scalar step, by the first wavefront
  Rp[0][P.c] = r0;
  __shared__ double s_beta;
  __shared__ int s_stop;
  if (threadIdx.x < 64) {
    const double gamma = wave_total(A.sum_g, A.nsum);
    double eps;
    const bool stop = stop_at(sc, st.iter, gamma, eps);
    if (threadIdx.x == 0) {
      s_beta = st.iter > 0 ? gamma / st.gamma_prev : 0.0;
      s_stop = stop;
      if (blockIdx.x == 0) {
        A.hist[st.iter] = eps;
        if (st.iter == 0) sc->gamma0 = gamma;
        sc->dir = {gamma, st.iter, stop ? 1 : 0};
      }
    }
  }
  __syncthreads();
  if (s_stop) return;
  const double beta = s_beta;
  double pm = 0.0, p0 = 0.0;
  double acc[1] = {0.0};
  // p at plane z, then A p at plane z - 1; r holds z - 1 .. z + 1
  auto step = [&](int z, int b, double& rnext, double& pz) {
    if (z >= P.z0) {
      Rp[b][P.c] = r0;
      Pp[b ^ 1][P.c] = p0;
      __syncthreads();
    }
    const double u = PC == RY_PC_STENCIL7 ? (13.0 / 12.0) * r0 + (1.0 / 6.0) * six<T>(Rp[b], P.c, rm, r1) : r0;
    const double p1 = (P.in && P.inz(z)) ? u + beta * pz : 0.0;
    pz = P.load1(pold, z + 2);
    if (P.own && z >= P.z0 && z < P.z1) pnew[P.cell(z)] = p1;
    const double ap = 6.0 * p0 - six<T>(Pp[b ^ 1], P.c, pm, p1);
    acc[0] += (P.own && z > P.z0) ? p0 * ap : 0.0;
    rm = r0;
    r0 = r1;
    r1 = rnext;
    rnext = P.load2(r, z + 4);
    pm = p0;
    p0 = p1;
  };
  for (int z = P.z0 - 1; z <= P.z1; z += 2) {
    step(z, 0, rq[0], pq[0]);
    if (z + 1 <= P.z1) step(z + 1, 1, rq[1], pq[1]);
  }
  block_sum(acc, red);
  if (threadIdx.x == 0) A.part_d[blockIdx.x] = acc[0];
}

// alpha_i; r_{i+1} = r_i - alpha_i A p_i on the tile and its one-cell halo,
// x_{i+1} = x_i + alpha_i p_i; partials of gamma_{i+1}.
template <int PC>
__global__ __launch_bounds__(LargeTile::NT) void cg_update_kernel(CgArgs A) {
  using T = LargeTile;
  Scalars* sc = A.sc;
  const Scalars::Dir dir = sc->dir;
  if (dir.done) {
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->step[0].done = 1;
    return;
  }
  __shared__ double Pp[2][T::PL], Rp[2][T::PL];
  __shared__ double red[1][T::NWV];
  const Point<T> P(A.g, A.cz);
  const double* __restrict__ p = A.p[(dir.iter & 1) ^ 1];
  const double* __restrict__ rold = A.r[dir.iter & 1];
  double* __restrict__ rnew = A.r[(dir.iter & 1) ^ 1];
  double pm = P.load2(p, P.z0 - 2), p0 = P.load2(p, P.z0 - 1), p1 = P.load2(p, P.z0);
  double pq[2] = {P.load2(p, P.z0 + 1), P.load2(p, P.z0 + 2)};
  double rq[2] = {P.load1(rold, P.z0 - 1), P.load1(rold, P.z0)};
  auto load_x = [&](int z) { return A.x[P.cell(z)]; };
  double xq[2] = {0.0, 0.0};   // x is used one plane behind r: the first two planes only load it
  // the scalar step, by the first wavefront
  Pp[0][P.c] = p0;
  __shared__ double s_alpha;
  if (threadIdx.x < 64) {
    const double a = dir.gamma / wave_total(A.sum_d, A.nsum);
    if (threadIdx.x == 0) {
      s_alpha = a;
      if (blockIdx.x == 0) sc->step[0] = {a, dir.gamma, dir.iter + 1, 0};
    }
  }
  __syncthreads();
  const double alpha = s_alpha;
  double rm = 0.0, r0 = 0.0;
  double acc[1] = {0.0};
  // r at plane z, then everything else at plane z - 1; p holds z - 1 .. z + 1
  auto step = [&](int z, int b, double& pnext, double& rz, double& xz) {
    if (z >= P.z0) {
      Pp[b][P.c] = p0;
      Rp[b ^ 1][P.c] = r0;
      __syncthreads();
    }
    double r1 = rz - alpha * (6.0 * p0 - six<T>(Pp[b], P.c, pm, p1));
    r1 = (P.in && P.inz(z)) ? r1 : 0.0;
    rz = P.load1(rold, z + 2);
    const double u = PC == RY_PC_STENCIL7 ? (13.0 / 12.0) * r0 + (1.0 / 6.0) * six<T>(Rp[b ^ 1], P.c, rm, r1) : r0;
    if (P.own && z > P.z0) {
      const int64_t i = P.cell(z - 1);
      rnew[i] = r0;
      A.x[i] = xz + alpha * pm;
      acc[0] += r0 * u;
    }
    xz = load_x(z + 1);
    pm = p0;
    p0 = p1;
    p1 = pnext;
    pnext = P.load2(p, z + 4);
    rm = r0;
    r0 = r1;
  };
  for (int z = P.z0 - 1; z <= P.z1; z += 2) {
    step(z, 0, pq[0], rq[0], xq[0]);
    if (z + 1 <= P.z1) step(z + 1, 1, pq[1], rq[1], xq[1]);
  }
  block_sum(acc, red);
  if (threadIdx.x == 0) A.part_g[blockIdx.x] = acc[0];
}

// Sums of contiguous shares of n partials, one per workgroup (gridDim.y
// quantities), in a fixed order.  Also launched behind iterations that no
// longer run: the same partials then give the same sums again.
__global__ __launch_bounds__(NTH) void reduce_kernel(const double* __restrict__ part, int n,
                                                     double* __restrict__ sum) {
  __shared__ double red[1][NTH / 64];
  const int64_t b = blockIdx.x, m = gridDim.x;
  const int first = int(b * n / m), last = int((b + 1) * n / m);
  double a[1] = {strided_sum(part + int64_t(blockIdx.y) * n + first, last - first)};
  block_sum(a, red);
  if (threadIdx.x == 0) sum[blockIdx.y * m + b] = a[0];
}

// (Re)arm the stopping rule: absolute max_iter, or relative to the current
// iterate's index (held by step[slot]).
__global__ void ppcg_arm_kernel(Scalars* sc, double eps, int32_t max_iter, int32_t relative, int32_t slot) {
  sc->step[0].done = sc->step[1].done = sc->dir.done = 0;
  sc->eps_target = eps;
  sc->max_iter = relative ? sc->step[slot].iter + max_iter : max_iter;
}

__global__ void ppcg_reset_kernel(Scalars* sc) {
  *sc = Scalars{};
  sc->eps_target = -1.0;
  sc->step[0].done = sc->step[1].done = sc->dir.done = 1;
}

// ---------------------------------------------------------------------------
// Start-up sweeps (once per solve), and the operators applied to a whole
// vector (the two-sweep form's vectors on request).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double nb_sum(const double* v, const Grid& g, int X, int Y, int Z) {
  double s = grid_val(v, g, X - 1, Y, Z);
  s += grid_val(v, g, X + 1, Y, Z);
  s += grid_val(v, g, X, Y - 1, Z);
  s += grid_val(v, g, X, Y + 1, Z);
  s += grid_val(v, g, X, Y, Z - 1);
  s += grid_val(v, g, X, Y, Z + 1);
  return s;
}
__device__ __forceinline__ void cell_of(const Grid& g, int64_t i, int& X, int& Y, int& Z) {
  const uint32_t c = uint32_t(i), row = c / uint32_t(g.n0);   // fewer than 2^31 cells
  X = int(c - row * uint32_t(g.n0));
  Z = int(row / uint32_t(g.n1));
  Y = int(row) - Z * g.n1;
}

// r = b - A x (zero_x: from x = 0, which is stored), and zeros in the
// vectors of `clear`.  b may be one of them: each cell's b is read by the
// thread that clears it.
struct ClearList {
  double* v[4];
};
__global__ __launch_bounds__(256) void residual_kernel(Grid g, const double* b, double* __restrict__ x, int zero_x,
                                                       double* __restrict__ r, ClearList clear) {
  const int64_t N = int64_t(g.n0) * g.n1 * g.n2;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < N; i += int64_t(gridDim.x) * blockDim.x) {
    const double bv = b[i];
    double rv = bv;
    if (zero_x) {
      x[i] = 0.0;
    } else {
      int X, Y, Z;
      cell_of(g, i, X, Y, Z);
      rv = bv - (6.0 * x[i] - nb_sum(x, g, X, Y, Z));
    }
    r[i] = rv;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (clear.v[k]) clear.v[k][i] = 0.0;
  }
}

__device__ __forceinline__ double apply_m(const double* r, const Grid& g, int pc, int64_t i) {
  if (pc != RY_PC_STENCIL7) return r[i];
  int X, Y, Z;
  cell_of(g, i, X, Y, Z);
  return (13.0 / 12.0) * r[i] + (1.0 / 6.0) * nb_sum(r, g, X, Y, Z);
}
__device__ __forceinline__ double apply_a(const double* u, const Grid& g, int64_t i) {
  int X, Y, Z;
  cell_of(g, i, X, Y, Z);
  return 6.0 * u[i] - nb_sum(u, g, X, Y, Z);
}

__global__ __launch_bounds__(256) void minv_kernel(Grid g, int pc, const double* __restrict__ r,
                                                   double* __restrict__ u) {
  const int64_t N = int64_t(g.n0) * g.n1 * g.n2;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < N; i += int64_t(gridDim.x) * blockDim.x)
    u[i] = apply_m(r, g, pc, i);
}

__global__ __launch_bounds__(256) void apply_a_kernel(Grid g, const double* __restrict__ u, double* __restrict__ w) {
  const int64_t N = int64_t(g.n0) * g.n1 * g.n2;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < N; i += int64_t(gridDim.x) * blockDim.x)
    w[i] = apply_a(u, g, i);
}

// w = A u and the partials of r.u and w.u (pipelined form).
__global__ __launch_bounds__(NTH) void apply_a_dots_kernel(Grid g, const double* __restrict__ r,
                                                           const double* __restrict__ u, double* __restrict__ w,
                                                           double* part) {
  __shared__ double red[2][NTH / 64];
  const int64_t N = int64_t(g.n0) * g.n1 * g.n2;
  double ab[2] = {0.0, 0.0};
  for (int64_t i = blockIdx.x * int64_t(NTH) + threadIdx.x; i < N; i += int64_t(gridDim.x) * NTH) {
    const double wv = apply_a(u, g, i);
    w[i] = wv;
    ab[0] += r[i] * u[i];
    ab[1] += wv * u[i];
  }
  block_sum(ab, red);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = ab[0];
    part[gridDim.x + blockIdx.x] = ab[1];
  }
}

// Partials of r.(M^-1 r) (two-sweep form).
__global__ __launch_bounds__(NTH) void gamma_kernel(Grid g, int pc, const double* __restrict__ r, double* part) {
  __shared__ double red[1][NTH / 64];
  const int64_t N = int64_t(g.n0) * g.n1 * g.n2;
  double a[1] = {0.0};
  for (int64_t i = blockIdx.x * int64_t(NTH) + threadIdx.x; i < N; i += int64_t(gridDim.x) * NTH)
    a[0] += r[i] * apply_m(r, g, pc, i);
  block_sum(a, red);
  if (threadIdx.x == 0) part[blockIdx.x] = a[0];
}

}  // namespace ryp

// ===========================================================================
// Host side.
// ===========================================================================
using namespace ryp;

struct ry_poisson {
  ry_poisson_config cfg{};
  Grid g{};
  int64_t N = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::vector<void*> allocs;
  bool two_sweep = false;
  double* v[NVEC] = {};        // x r u w0 w1 z q s p; two-sweep: x r0 r1 p0 p1
  double* part = nullptr;      // pipelined: [2][2][nblk]; two-sweep: [2][nblk] (gamma, p.Ap)
  double* sum = nullptr;       // part, or as part with nsum for nblk
  double* hist = nullptr;
  Scalars* sc = nullptr;
  int32_t* h_done = nullptr;   // pinned
  int nblk = 0, nsum = 0, cz = 0;
  ry::Staging staging;         // pinned buffers of the downloads
  bool ready = false;          // set_rhs done
  int64_t iter = 0;            // the device's iteration index (once the stream's work is done)
  hipGraphExec_t graph[2] = {};   // by parity of the first iteration's index (two-sweep: [0])
  bool timing = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
  int64_t t_launches = 0;
  double t_ms = 0.0;
  std::string err;
};

namespace {

ry_status pfail(ry_poisson* p, ry_status s, const char* fmt, ...) {
  if (p) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    p->err = buf;
  }
  return s;
}

#define PCHK(p, call)                                                                        \
  do {                                                                                       \
    hipError_t e_ = (call);                                                                  \
    if (e_ != hipSuccess) return pfail((p), RY_EHIP, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)

void* palloc(ry_poisson* p, size_t bytes) {
  void* a = nullptr;
  if (p->cfg.dev_alloc) a = p->cfg.dev_alloc(bytes, p->cfg.alloc_user);
  else if (hipMalloc(&a, bytes) != hipSuccess) a = nullptr;
  if (a) p->allocs.push_back(a);
  else (void)hipGetLastError();   // a refused hipMalloc's, which the next launch's check would report
  return a;
}

void pfree_all(ry_poisson* p) {
  if (p->stream) hipStreamSynchronize(p->stream);
  for (void* a : p->allocs) {
    if (p->cfg.dev_free) p->cfg.dev_free(a, p->cfg.alloc_user);
    else if (!p->cfg.dev_alloc) hipFree(a);
  }
  p->allocs.clear();
  for (auto& gr : p->graph) {
    if (gr) hipGraphExecDestroy(gr);
    gr = nullptr;
  }
  for (auto& e : p->ev) {
    hipEventDestroy(e.first);
    hipEventDestroy(e.second);
  }
  p->ev.clear();
  p->staging.release();
  if (p->h_done) hipHostFree(p->h_done);
  p->h_done = nullptr;
}

IterArgs iter_args(ry_poisson* p, int par) {
  IterArgs a;
  a.g = p->g;
  a.x = p->v[0];
  a.r = p->v[1];
  a.u = p->v[2];
  a.w[0] = p->v[3];
  a.w[1] = p->v[4];
  a.z = p->v[5];
  a.q = p->v[6];
  a.s = p->v[7];
  a.p = p->v[8];
  a.sc = p->sc;
  a.hist = p->hist;
  a.part = p->part;
  a.sum = p->sum;
  a.nsum = p->nsum;
  a.cz = p->cz;
  a.par = par;
  return a;
}

CgArgs cg_args(ry_poisson* p) {
  CgArgs a;
  a.g = p->g;
  a.x = p->v[0];
  a.r[0] = p->v[1];
  a.r[1] = p->v[2];
  a.p[0] = p->v[3];
  a.p[1] = p->v[4];
  a.sc = p->sc;
  a.hist = p->hist;
  a.part_g = p->part;
  a.part_d = p->part + p->nblk;
  a.sum_g = p->sum;
  a.sum_d = p->sum + p->nsum;
  a.nsum = p->nsum;
  a.cz = p->cz;
  return a;
}

// The sums the sweeps read, from nq quantities' partials starting at set k
// (of nblk values each).
void launch_reduce(ry_poisson* p, int k, int nq) {
  if (p->nsum == p->nblk) return;
  hipLaunchKernelGGL(reduce_kernel, dim3(p->nsum, nq), dim3(NTH), 0, p->stream, p->part + int64_t(k) * p->nblk,
                     p->nblk, p->sum + int64_t(k) * p->nsum);
}

// The solver's form and its sweeps' workgroups (the constants at the top say
// where the lines lie).
void plan_sweeps(ry_poisson* p) {
  const Grid& g = p->g;
  int64_t cols = 0;
  double fill = 0.0;
  auto tiles = [&](int tx, int ty) {
    cols = int64_t((g.n0 + tx - 1) / tx) * ((g.n1 + ty - 1) / ty);
    fill = double(g.n0) * g.n1 / (double(cols) * tx * ty);
  };
  auto chunks = [&](int target) {
    const int64_t nch = std::max<int64_t>(1, std::min<int64_t>(target / cols, g.n2));
    p->cz = int32_t((g.n2 + nch - 1) / nch);
    p->nblk = int(cols * ((g.n2 + p->cz - 1) / p->cz));
  };
  tiles(LargeTile::TX, LargeTile::TY);
  chunks(kTargetLarge);
  p->two_sweep = p->N >= kTwoSweepCells && p->cz >= kTwoSweepPlanes && fill >= kTwoSweepFill;
  if (!p->two_sweep) {
    tiles(SmallTile::TX, SmallTile::TY);
    chunks(kTargetSmall);
    if (p->cz > kLongChunk) chunks(fill < kThinFill ? kTargetThin : kTargetLong);
  }
  p->nsum = p->nblk > kMaxPartials ? kSums : p->nblk;
}

// The slot of Scalars::step that the next iteration reads.
int step_slot(const ry_poisson* p) { return p->two_sweep ? 0 : int(p->iter & 1); }

// The iteration of parity `par` (which first tests the iterate it starts
// from and does nothing more when the solve stops there); `timed`: between
// two events.
ry_status launch_iteration(ry_poisson* p, int par, bool timed) {
  const dim3 grid(p->nblk), block(p->two_sweep ? LargeTile::NT : NTH);
  if (timed) {
    hipEvent_t a, b;
    // timing-only events: no system-scope fence (cache write-back) on recording
    PCHK(p, hipEventCreateWithFlags(&a, hipEventDisableSystemFence));
    PCHK(p, hipEventCreateWithFlags(&b, hipEventDisableSystemFence));
    PCHK(p, hipEventRecord(a, p->stream));
    p->ev.push_back({a, b});
  }
  const bool pc = p->cfg.precond == RY_PC_STENCIL7;
  if (p->two_sweep) {
    const CgArgs a = cg_args(p);
    if (pc) hipLaunchKernelGGL(cg_direction_kernel<RY_PC_STENCIL7>, grid, block, 0, p->stream, a);
    else hipLaunchKernelGGL(cg_direction_kernel<RY_PC_NONE>, grid, block, 0, p->stream, a);
    launch_reduce(p, 1, 1);
    if (pc) hipLaunchKernelGGL(cg_update_kernel<RY_PC_STENCIL7>, grid, block, 0, p->stream, a);
    else hipLaunchKernelGGL(cg_update_kernel<RY_PC_NONE>, grid, block, 0, p->stream, a);
    launch_reduce(p, 0, 1);
  } else {
    const IterArgs a = iter_args(p, par);
    const bool many = p->nsum != p->nblk;
    if (pc && many) hipLaunchKernelGGL((ppcg_iterate_kernel<RY_PC_STENCIL7, true>), grid, block, 0, p->stream, a);
    else if (pc) hipLaunchKernelGGL((ppcg_iterate_kernel<RY_PC_STENCIL7, false>), grid, block, 0, p->stream, a);
    else if (many) hipLaunchKernelGGL((ppcg_iterate_kernel<RY_PC_NONE, true>), grid, block, 0, p->stream, a);
    else hipLaunchKernelGGL((ppcg_iterate_kernel<RY_PC_NONE, false>), grid, block, 0, p->stream, a);
    launch_reduce(p, 2 * (par ^ 1), 2);
  }
  if (timed) PCHK(p, hipEventRecord(p->ev.back().second, p->stream));
  PCHK(p, hipGetLastError());
  return RY_OK;
}

// BATCH iterations as one graph, the first one's index of parity `par`.
ry_status ensure_graph(ry_poisson* p, int par) {
  hipGraphExec_t& ge = p->graph[par];
  if (ge) return RY_OK;
  PCHK(p, hipStreamBeginCapture(p->stream, hipStreamCaptureModeThreadLocal));
  ry_status s = RY_OK;
  for (int k = 0; k < BATCH && s == RY_OK; ++k) s = launch_iteration(p, (par + k) & 1, false);
  hipGraph_t gr = nullptr;
  const hipError_t e = hipStreamEndCapture(p->stream, &gr);
  if (s) {
    if (gr) hipGraphDestroy(gr);
    return s;
  }
  if (e != hipSuccess) return pfail(p, RY_EHIP, "graph capture: %s", hipGetErrorString(e));
  const hipError_t e2 = hipGraphInstantiate(&ge, gr, nullptr, nullptr, 0);
  hipGraphDestroy(gr);
  if (e2 != hipSuccess) {
    ge = nullptr;
    return pfail(p, RY_EHIP, "graph instantiate: %s", hipGetErrorString(e2));
  }
  return RY_OK;
}

void collect_times(ry_poisson* p) {
  for (auto& e : p->ev) {
    float ms = 0.f;
    hipEventSynchronize(e.second);
    hipEventElapsedTime(&ms, e.first, e.second);
    p->t_ms += ms;
    ++p->t_launches;
    hipEventDestroy(e.first);
    hipEventDestroy(e.second);
  }
  p->ev.clear();
}

}  // namespace

// No C++ exception crosses the C ABI: a failed host allocation inside an
// entry point becomes RY_ENOMEM, any other exception RY_EINVAL.
#define RY_ABI_TRY try {
#define RY_ABI_CATCH                    \
  }                                     \
  catch (const std::bad_alloc&) {       \
    return RY_ENOMEM;                   \
  }                                     \
  catch (...) {                         \
    return RY_EINVAL;                   \
  }

extern "C" {

ry_status ry_poisson_create(const ry_poisson_config* cfg, ry_poisson** out) {
  RY_ABI_TRY
  if (!cfg || !out) return RY_EINVAL;
  *out = nullptr;
  for (int a = 0; a < 3; ++a)
    if (cfg->n[a] < 1) return RY_EINVAL;
  const int64_t N = int64_t(cfg->n[0]) * cfg->n[1] * cfg->n[2];
  if (N >= (int64_t(1) << 31)) return RY_EINVAL;
  if (cfg->bc != RY_PBC_PERIODIC && cfg->bc != RY_PBC_DIRICHLET) return RY_EINVAL;
  if (cfg->precond != RY_PC_NONE && cfg->precond != RY_PC_STENCIL7) return RY_EINVAL;
  if ((cfg->dev_alloc == nullptr) != (cfg->dev_free == nullptr)) return RY_EINVAL;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return RY_EHIP;
  ry_poisson* p = new (std::nothrow) ry_poisson();
  if (!p) return RY_ENOMEM;
  p->cfg = *cfg;
  p->g = {cfg->n[0], cfg->n[1], cfg->n[2], cfg->bc};
  p->N = N;
  if (cfg->stream) {
    p->stream = (hipStream_t)cfg->stream;
  } else {
    if (hipStreamCreateWithFlags(&p->stream, hipStreamNonBlocking) != hipSuccess) {
      delete p;
      return RY_EHIP;
    }
    p->own_stream = true;
  }
  plan_sweeps(p);
  bool ok = true;
  for (int k = 0; k < (p->two_sweep ? 5 : NVEC) && ok; ++k) ok = (p->v[k] = static_cast<double*>(palloc(p, sizeof(double) * N))) != nullptr;
  ok = ok && (p->part = static_cast<double*>(palloc(p, sizeof(double) * 4 * p->nblk))) != nullptr;
  p->sum = p->part;
  if (ok && p->nsum != p->nblk) ok = (p->sum = static_cast<double*>(palloc(p, sizeof(double) * 4 * p->nsum))) != nullptr;
  ok = ok && (p->hist = static_cast<double*>(palloc(p, sizeof(double) * RY_POISSON_HIST))) != nullptr;
  ok = ok && (p->sc = static_cast<Scalars*>(palloc(p, sizeof(Scalars)))) != nullptr;
  if (ok && hipHostMalloc((void**)&p->h_done, sizeof(int32_t)) != hipSuccess) {
    p->h_done = nullptr;
    (void)hipGetLastError();
    ok = false;
  }
  if (!ok) {
    pfree_all(p);
    if (p->own_stream) hipStreamDestroy(p->stream);
    delete p;
    return RY_ENOMEM;
  }
  hipLaunchKernelGGL(ppcg_reset_kernel, dim3(1), dim3(1), 0, p->stream, p->sc);
  if (hipGetLastError() != hipSuccess) {
    pfree_all(p);
    if (p->own_stream) hipStreamDestroy(p->stream);
    delete p;
    return RY_EHIP;
  }
  *out = p;
  return RY_OK;
  RY_ABI_CATCH
}

void ry_poisson_destroy(ry_poisson* p) {
  if (!p) return;
  pfree_all(p);
  if (p->own_stream && p->stream) hipStreamDestroy(p->stream);
  delete p;
}

ry_status ry_poisson_set_rhs(ry_poisson* p, const double* b, const double* x0) {
  RY_ABI_TRY
  if (!p || !b) return RY_EINVAL;
  const size_t bytes = sizeof(double) * size_t(p->N);
  // b is staged in a vector that holds nothing yet: z (cleared once r has
  // been formed) or the second direction buffer (the first iteration writes it)
  double *x = p->v[0], *r = p->v[1], *stage = p->v[p->two_sweep ? 4 : 5];
  ClearList clear{};
  if (p->two_sweep) clear.v[0] = p->v[3];
  else
    for (int k = 0; k < 4; ++k) clear.v[k] = p->v[5 + k];
  PCHK(p, hipMemcpyAsync(stage, b, bytes, hipMemcpyHostToDevice, p->stream));
  if (x0) PCHK(p, hipMemcpyAsync(x, x0, bytes, hipMemcpyHostToDevice, p->stream));
  // b and x0 are the caller's again when this returns
  if (!ry::Staging::pageable(b) || (x0 && !ry::Staging::pageable(x0))) PCHK(p, hipStreamSynchronize(p->stream));
  const int blocks = int(std::min<int64_t>((p->N + 255) / 256, 8192));
  hipLaunchKernelGGL(residual_kernel, dim3(blocks), dim3(256), 0, p->stream, p->g, stage, x, x0 ? 0 : 1, r, clear);
  if (p->two_sweep) {
    hipLaunchKernelGGL(gamma_kernel, dim3(p->nblk), dim3(NTH), 0, p->stream, p->g, p->cfg.precond, r, p->part);
  } else {
    double *u = p->v[2], *w0 = p->v[3];
    hipLaunchKernelGGL(minv_kernel, dim3(blocks), dim3(256), 0, p->stream, p->g, p->cfg.precond, r, u);
    hipLaunchKernelGGL(apply_a_dots_kernel, dim3(p->nblk), dim3(NTH), 0, p->stream, p->g, r, u, w0, p->part);
  }
  launch_reduce(p, 0, p->two_sweep ? 1 : 2);
  hipLaunchKernelGGL(ppcg_reset_kernel, dim3(1), dim3(1), 0, p->stream, p->sc);
  PCHK(p, hipGetLastError());
  p->ready = true;
  p->iter = 0;
  return RY_OK;
  RY_ABI_CATCH
}

ry_status ry_poisson_solve(ry_poisson* p, double eps, int32_t max_iter, int32_t* n_iter) {
  RY_ABI_TRY
  if (!p) return RY_EINVAL;
  if (!p->ready) return pfail(p, RY_ESTATE, "ry_poisson_solve before ry_poisson_set_rhs");
  if (max_iter < 0 || max_iter > RY_POISSON_HIST - 1 || std::isnan(eps)) return RY_EINVAL;
  hipLaunchKernelGGL(ppcg_arm_kernel, dim3(1), dim3(1), 0, p->stream, p->sc, eps, max_iter, 0,
                     step_slot(p));
  PCHK(p, hipGetLastError());
  const int par = step_slot(p);
  if (!p->timing) {
    ry_status s = ensure_graph(p, par);
    if (s) return s;
  }
  // after a batch (an even number of iterations) the newest record is in the
  // slot it started from
  const int32_t* done = p->two_sweep ? &p->sc->dir.done : &p->sc->step[par].done;
  const int64_t batches = int64_t(max_iter) / BATCH + 2;
  for (int64_t k = 0; k < batches; ++k) {
    if (p->timing) {
      for (int j = 0; j < BATCH; ++j) {
        ry_status s = launch_iteration(p, (par + j) & 1, true);
        if (s) return s;
      }
    } else {
      PCHK(p, hipGraphLaunch(p->graph[par], p->stream));
    }
    PCHK(p, hipMemcpyAsync(p->h_done, done, sizeof(int32_t), hipMemcpyDeviceToHost, p->stream));
    PCHK(p, hipStreamSynchronize(p->stream));
    if (*p->h_done) break;
  }
  Scalars s{};
  PCHK(p, hipMemcpy(&s, p->sc, sizeof s, hipMemcpyDeviceToHost));
  if (!*p->h_done) return pfail(p, RY_ESTATE, "solver did not stop");
  p->iter = s.step[par].iter;
  if (n_iter) *n_iter = int32_t(p->iter);
  if (p->timing) collect_times(p);
  return RY_OK;
  RY_ABI_CATCH
}

ry_status ry_poisson_iterate(ry_poisson* p, int32_t n) {
  RY_ABI_TRY
  if (!p || n < 0) return RY_EINVAL;
  if (!p->ready) return pfail(p, RY_ESTATE, "ry_poisson_iterate before ry_poisson_set_rhs");
  if (p->iter + n > RY_POISSON_HIST - 1) return pfail(p, RY_EINVAL, "iteration history full");
  if (n == 0) return RY_OK;
  hipLaunchKernelGGL(ppcg_arm_kernel, dim3(1), dim3(1), 0, p->stream, p->sc, -1.0, n, 1,
                     step_slot(p));
  PCHK(p, hipGetLastError());
  const int par = step_slot(p);
  // n iterations plus one that only records eps of the last iterate
  if (p->timing) {
    for (int j = 0; j <= n; ++j) {
      ry_status s = launch_iteration(p, (par + j) & 1, j < n);
      if (s) return s;
    }
  } else {
    ry_status s = ensure_graph(p, par);
    if (s) return s;
    for (int j = 0; j <= n; j += BATCH) PCHK(p, hipGraphLaunch(p->graph[par], p->stream));
  }
  p->iter += n;
  return RY_OK;
  RY_ABI_CATCH
}

ry_status ry_poisson_eps_history(ry_poisson* p, double* eps, int32_t cap, int32_t* n) {
  RY_ABI_TRY
  if (!p || !eps || cap < 0) return RY_EINVAL;
  PCHK(p, hipStreamSynchronize(p->stream));
  const int32_t k = int32_t(std::min<int64_t>(p->iter + 1, cap));
  if (k > 0) PCHK(p, hipMemcpy(eps, p->hist, sizeof(double) * k, hipMemcpyDeviceToHost));
  if (n) *n = k;
  return RY_OK;
  RY_ABI_CATCH
}

ry_status ry_poisson_download(ry_poisson* p, int32_t which, double* host) {
  RY_ABI_TRY
  if (!p || !host || which < 0 || which >= RY_PV_COUNT) return RY_EINVAL;
  PCHK(p, hipStreamSynchronize(p->stream));
  int slot;
  if (p->two_sweep) {
    // x, r and p are kept; the others follow from them, formed in the two
    // buffers the next iteration overwrites
    const int cur = int(p->iter & 1), s1 = 1 + (cur ^ 1), s2 = 3 + (cur ^ 1);
    const int blocks = int(std::min<int64_t>((p->N + 255) / 256, 8192));
    auto minv = [&](int from, int to) {
      hipLaunchKernelGGL(minv_kernel, dim3(blocks), dim3(256), 0, p->stream, p->g, p->cfg.precond, p->v[from],
                         p->v[to]);
    };
    auto mul_a = [&](int from, int to) {
      hipLaunchKernelGGL(apply_a_kernel, dim3(blocks), dim3(256), 0, p->stream, p->g, p->v[from], p->v[to]);
    };
    slot = 0;
    if (which == RY_PV_R) {
      slot = 1 + cur;
    } else if (which == RY_PV_P) {
      slot = 3 + cur;
    } else if (which == RY_PV_U || which == RY_PV_W) {   // u = M^-1 r, w = A u
      minv(1 + cur, s1);
      if (which == RY_PV_W) mul_a(s1, s2);
      slot = which == RY_PV_W ? s2 : s1;
    } else if (which != RY_PV_X) {                       // s = A p, q = M^-1 s, z = A q
      mul_a(3 + cur, s1);
      if (which != RY_PV_S) minv(s1, s2);
      if (which == RY_PV_Z) mul_a(s2, s1);
      slot = which == RY_PV_Q ? s2 : s1;
    }
    PCHK(p, hipGetLastError());
  } else {
    // x r u w z q s p; w_i lives in buffer (i & 1)
    switch (which) {
      case RY_PV_X: slot = 0; break;
      case RY_PV_R: slot = 1; break;
      case RY_PV_U: slot = 2; break;
      case RY_PV_W: slot = 3 + int(p->iter & 1); break;
      default: slot = which + 1; break;   // z q s p -> 5..8
    }
  }
  const size_t bytes = sizeof(double) * size_t(p->N);
  PCHK(p, p->staging.download(host, p->v[slot], bytes, bytes, 1, p->stream));
  return RY_OK;
  RY_ABI_CATCH
}

ry_status ry_poisson_scalars(ry_poisson* p, double* alpha_prev, double* gamma_prev, int32_t* iter) {
  RY_ABI_TRY
  if (!p) return RY_EINVAL;
  Scalars s{};
  PCHK(p, hipStreamSynchronize(p->stream));
  PCHK(p, hipMemcpy(&s, p->sc, sizeof s, hipMemcpyDeviceToHost));
  const Scalars::Step& st = s.step[step_slot(p)];
  if (alpha_prev) *alpha_prev = st.alpha_prev;
  if (gamma_prev) *gamma_prev = st.gamma_prev;
  if (iter) *iter = st.iter;
  return RY_OK;
  RY_ABI_CATCH
}

ry_status ry_poisson_set_timing(ry_poisson* p, int32_t on) {
  RY_ABI_TRY
  if (!p) return RY_EINVAL;
  PCHK(p, hipStreamSynchronize(p->stream));
  collect_times(p);
  p->timing = on != 0;
  p->t_launches = 0;
  p->t_ms = 0.0;
  return RY_OK;
  RY_ABI_CATCH
}

ry_status ry_poisson_kernel_time(ry_poisson* p, int32_t* launches, double* total_ms) {
  RY_ABI_TRY
  if (!p) return RY_EINVAL;
  PCHK(p, hipStreamSynchronize(p->stream));
  collect_times(p);
  if (launches) *launches = int32_t(p->t_launches);
  if (total_ms) *total_ms = p->t_ms;
  return RY_OK;
  RY_ABI_CATCH
}

const char* ry_poisson_last_error(const ry_poisson* p) { return p ? p->err.c_str() : "null solver"; }

}  // extern "C"
