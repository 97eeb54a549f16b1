// ctmhd_device.h -- device-side structures and functions of libctmhd
// (gfx950), shared by the forward and the adjoint translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <type_traits>

#include "ctmhd.h"
#include "ctmhd_math.h"
#include "ctmhd_workgroup.h"

using namespace ctmhd;

namespace {

// ---------------------------------------------------------------------------
// Geometry of one ghosted box.
// ---------------------------------------------------------------------------
struct Geom {
  int n[3];    // interior cells
  int g;       // ghost layers
  int N[3];    // n + 2g
  int st[3];   // strides: 1, N0, N0*N1
  int elems;   // N0*N1*N2
  double dx[3];
  double idx[3];
};

Geom make_geom(const ctmhd_box& b) {
  Geom G;
  for (int d = 0; d < 3; ++d) {
    G.n[d] = b.n[d];
    G.N[d] = b.n[d] + 2 * b.ng;
    G.dx[d] = b.dx[d];
    G.idx[d] = 1.0 / b.dx[d];
  }
  G.g = b.ng;
  G.st[0] = 1;
  G.st[1] = G.N[0];
  G.st[2] = G.N[0] * G.N[1];
  G.elems = G.N[0] * G.N[1] * G.N[2];
  return G;
}

__device__ __forceinline__ int gidx() { return blockIdx.x * blockDim.x + threadIdx.x; }

// Storage stride of axis d.  The x stride is 1 by construction; returning it
// as a constant (d is known at compile time at every call site) lets the
// compiler fold x-neighbour offsets into the load instructions.
__device__ __forceinline__ int gstride(const Geom& G, int d) { return d == 0 ? 1 : G.st[d]; }

// Element s of a field array, addressed by a 32-bit byte offset (a box has
// less than 2^31 / 6 elements, so the offset of a double fits): the array's
// base stays in scalar registers and all arrays read at one position share one
// offset register, where a signed element index costs a 64-bit address per
// array (two registers and an add).
template <typename T>
__device__ __forceinline__ T& at(T* p, int s) {
  using B = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return *reinterpret_cast<T*>(reinterpret_cast<B*>(p) + (unsigned)s * (unsigned)sizeof(T));
}

// The element k positions along axis d from s (k a constant): x neighbours are
// immediate offsets of the load.
template <typename T>
__device__ __forceinline__ T& nbr(T* p, const Geom& G, int s, int d, int k) {
  return d == 0 ? at(p + k, s) : at(p, s + k * G.st[d]);
}

// Workgroups are dispatched to the 8 XCDs of the chip round-robin (workgroup
// i on XCD i mod 8), and each XCD has its own L2.  This permutation of the
// tiles of a launch gives each XCD a contiguous run of them, so that the
// neighbouring rows and planes a stencil reads were brought into the same
// L2.  It is a bijection on [0, gridDim.x): results do not depend on it.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_tile() {
  const int nb = (int)gridDim.x, b = (int)blockIdx.x;
  const int per = nb / kXcds;
  if (b >= per * kXcds) return b;
  return (b % kXcds) * per + b / kXcds;
}

// The banded alternative: XCD x takes tiles [j C + x m, j C + (x+1) m) of
// every chunk j of C = 8 m consecutive tiles, so that all XCDs sweep the box
// together, each on its own band of the same chunk.  With a chunk about one
// plane of a large box, the planes a z stencil re-reads are then shared by the
// whole chip in the Infinity Cache instead of being re-fetched from HBM by
// each XCD on its own.  A bijection on [0, gridDim.x) (the tail beyond the
// last complete chunk keeps its order); m = 0 gives xcd_tile().
__device__ __forceinline__ int xcd_band_tile(int m) {
  if (m <= 0) return xcd_tile();
  const int nb = (int)gridDim.x, b = (int)blockIdx.x;
  const int C = kXcds * m;
  if (b >= nb / C * C) return b;
  const int k = b / kXcds;
  return (k / m) * C + (b % kXcds) * m + k % m;
}

// the constant address space
#define CTMHD_CONST __attribute__((address_space(4)))

struct State {
  double* c[5];
  double* b[3];
};

constexpr int kMaxSlots = 64;  // spread of the CFL maximum over atomics

template <typename T>
struct Work {
  T* prim[8];       // rho, u0, u1, u2, p, bc0, bc1, bc2 (B25a / FS18 only)
  T* ecell[3];      // cell-centred ideal EMF (B25a)
  // Stored first steps of the two-step corner reconstructions (when
  // first_step_stored), the values on both sides (0 lower, 1 upper) of the
  // interface at each position.  B25a: ecell[c] with order 0 along a = c+1
  // first, order 1 along b = c+2 first.  FS18: velocity u_v along axis d.
  T* b25f[3][2][2];
  T* fsf[3][3][2];
  T* F[2][3][5];    // per stage, direction, component (global momentum order)
  T* ap[3];
  T* am[3];
  T* us[3];
  T* E[2][3];       // per stage, edge EMFs
  uint8_t* flag;    // interior cells, x0 fastest; a level of boxes: every storage position
  // CFL maxima (bits of non-negative doubles), kMaxSlots each: [0] fused into
  // the stage-2 update, [1] recomputed by a stage-2 fix-up
  unsigned long long* smax;
  double* dt;       // the step's dt
  int* stop;        // n + 1 once step n of the call found a non-finite dt
  int* nflag;       // flagged cells of stage 0 / 1; nflag[2]: stage-2 fix-up ran
};

inline int nblocks(long long n) { return (int)((n + kBlock - 1) / kBlock); }

// ---------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------
__device__ __forceinline__ int pwrap(int s, int g, int n) {
  int q = (s - g) % n;
  if (q < 0) q += n;
  return q + g;
}

// Copy-back at the end of a call, run by the last kernel of the call when it
// was stopped: step n (*stop = n + 1) leaves S^n in the buffer that it started
// from, which is the caller's when nsteps - n is even.
struct Restore {
  State user, other;
  int elems, nsteps;  // nsteps 0: not the last kernel
};
__device__ __forceinline__ void restore_state(const Restore& R, int stop) {
  if (R.nsteps == 0 || !((R.nsteps - (stop - 1)) & 1)) return;
  for (int t = gidx(); t < R.elems; t += gridDim.x * blockDim.x) {
#pragma unroll
    for (int m = 0; m < 5; ++m) R.user.c[m][t] = R.other.c[m][t];
#pragma unroll
    for (int a = 0; a < 3; ++a) R.user.b[a][t] = R.other.b[a][t];
  }
}

// ---------------------------------------------------------------------------
// Cell primitives from the conserved state (eq. state:primitive), FP64.
// ---------------------------------------------------------------------------
// The eleven loads behind the primitives of one cell: the conserved state
// and the two faces of the cell along each axis.  Split from the arithmetic
// so that a marching thread can issue the loads of its next cell before the
// stores of the current one (the compiler cannot move loads of the state
// across stores to the workspace, which it must assume may alias).
struct CellRaw {
  double c[5], bl[3], bh[3];
};

__device__ __forceinline__ void cell_load(const State& S, const Geom& G, int s, CellRaw& R) {
#pragma unroll
  for (int m = 0; m < 5; ++m) R.c[m] = S.c[m][s];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    R.bl[d] = S.b[d][s];
    R.bh[d] = S.b[d][s + G.st[d]];
  }
}

// The same loads by 32-bit offsets (at), in the loops of the face pass.
__device__ __forceinline__ void cell_load_at(const State& S, const Geom& G, int s, CellRaw& R) {
#pragma unroll
  for (int m = 0; m < 5; ++m) R.c[m] = at(S.c[m], s);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    R.bl[d] = at(S.b[d], s);
    R.bh[d] = nbr(S.b[d], G, s, d, 1);
  }
}

__device__ __forceinline__ void raw_prim(const CellRaw& R, double gamma, double& rho, double u[3],
                                         double& p, double bc[3]) {
  rho = R.c[0];
  double ir = trcp(rho);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    u[d] = R.c[1 + d] * ir;
    bc[d] = 0.5 * (R.bl[d] + R.bh[d]);
  }
  p = (gamma - 1.0) * (R.c[4] - 0.5 * rho * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) -
                       0.5 * (bc[0] * bc[0] + bc[1] * bc[1] + bc[2] * bc[2]));
}

__device__ __forceinline__ void cell_prim(const State& S, const Geom& G, int s, double gamma,
                                          double& rho, double u[3], double& p, double bc[3]) {
  CellRaw R;
  cell_load(S, G, s, R);
  raw_prim(R, gamma, rho, u, p, bc);
}

// CFL signal speed of one cell (eq. resistivity:cfl; the resistive term
// enters as the speed 2 eta / dx_min, i.e. 2 eta / dx_min^2 per unit length).
// NaN propagates.
__device__ __forceinline__ double cfl_signal(double rho, const double u[3], double p,
                                             const double bc[3], const Geom& G, double gamma,
                                             double sres) {
  double s = sres;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double cf = fast_speed<double>(rho, p, bc[d], bc[(d + 1) % 3], bc[(d + 2) % 3], gamma);
    double sd = (fabs(u[d]) + cf) * G.idx[d];
    s = (sd > s || sd != sd) ? sd : s;
  }
  return s;
}

// The maximum of a workgroup (block_max_bits) folded into one of kMaxSlots
// device slots by an atomic max.
__device__ __forceinline__ void block_max_to_slots(double s, unsigned long long* slots, int slot) {
  const unsigned long long m = block_max_bits(s);
  if (threadIdx.x == 0) atomicMax(&slots[slot], m);
}

// Start of a call, storage position t of a periodic box: the ghost image of
// the caller's state `src` into dst (the interior too when dst is another
// buffer) and the CFL signal of an interior cell (0 elsewhere, or without
// want_dt).  Reads only interior positions of src, so it may work in place.
__device__ __forceinline__ double start_at(const State& src, const State& dst, bool copy,
                                           const Geom& G, double gamma, double sres, bool want_dt,
                                           int t) {
  if (t >= G.elems) return 0.0;
  const int i = t % G.N[0];
  const int q = t / G.N[0];
  const int p3[3] = {i, q % G.N[1], q / G.N[1]};
  bool inter = true;
  int s = t, up[3];  // interior position behind t; steps to the upper neighbours
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int g = G.g, n = G.n[d], p = p3[d];
    const bool in = p >= g && p < g + n;
    inter = inter && in;
    if (!in) s += (pwrap(p, g, n) - p) * G.st[d];
    up[d] = p == g + n - 1 ? (1 - n) * G.st[d] : G.st[d];
  }
  const bool store = copy || !inter, sig = want_dt && inter;
  if (!store && !sig) return 0.0;
  CellRaw R;
#pragma unroll
  for (int m = 0; m < 5; ++m) R.c[m] = src.c[m][s];
#pragma unroll
  for (int d = 0; d < 3; ++d) R.bl[d] = src.b[d][s];
  double v = 0.0;
  if (sig) {
#pragma unroll
    for (int d = 0; d < 3; ++d) R.bh[d] = src.b[d][s + up[d]];
    double rho, u[3], p, bc[3];
    raw_prim(R, gamma, rho, u, p, bc);
    v = cfl_signal(rho, u, p, bc, G, gamma, sres);
  }
  if (store) {
#pragma unroll
    for (int m = 0; m < 5; ++m) dst.c[m][t] = R.c[m];
#pragma unroll
    for (int d = 0; d < 3; ++d) dst.b[d][t] = R.bl[d];
  }
  return v;
}

// One pass over the caller's state at the start of a call: ghost fill, the
// copy into the buffer that the first step starts from, and the CFL maximum,
// one partial value per workgroup (no counter needs clearing first); also
// clears the call's diagnostics and stop flag.  Bound
// by memory: at 512^3 in FP64 it reads and writes the 8 fields once (4.2 ms;
// separate ghost, CFL and copy passes took 5.5 ms; 128^3 65 against 109 us).
__global__ void __launch_bounds__(kBlock)
    k_start(State src, State dst, int copy, Geom G, double gamma, double sres, int want_dt,
            unsigned long long* part, long long* diag, int ndiag, int* stop) {
  if (blockIdx.x == 0) {
    for (int q = threadIdx.x; q < ndiag; q += kBlock) diag[q] = 0;
    if (threadIdx.x == 0) *stop = 0;
  }
  double s = 0.0;
  for (int t = gidx(); t < G.elems; t += gridDim.x * blockDim.x) {
    const double v = start_at(src, dst, copy != 0, G, gamma, sres, want_dt != 0, t);
    s = (v > s || v != v) ? v : s;
  }
  if (!want_dt) return;
  const unsigned long long m = block_max_bits(s);
  if (threadIdx.x == 0) part[blockIdx.x] = m;
}

// dt of step n of a call (one workgroup), and the reset of the slots and the
// flag counters.  First step: the CFL maximum is that of the npart partial
// values of k_start, and the stop flag is cleared.  Later steps:
// smax[0..kMaxSlots) holds it unless the previous step's second stage was
// fixed up (nflag[2]), whose recomputed maximum is in smax[kMaxSlots..).
struct DtStep {
  unsigned long long* smax;
  const unsigned long long* part;
  int npart, n;  // n < 0: none
  int* nflag;
  double cfl;
  const double* dt_fixed;
  double *dt, *dt_out;
  int* stop;
  long long* diag;  // this step's row, cleared by k_start
};
__device__ __forceinline__ void dt_step(const DtStep& D) {
  const int t = threadIdx.x;
  const bool first = D.n == 0;
  const unsigned long long* src = first ? D.part : (D.nflag[2] ? D.smax + kMaxSlots : D.smax);
  const int cnt = first ? D.npart : kMaxSlots;
  const int stopped = first ? 0 : *D.stop;
  unsigned long long m = 0;
  for (int q = t; q < cnt; q += kBlock) m = src[q] > m ? src[q] : m;
  m = block_max_bits(__longlong_as_double((long long)m));
  if (t < 2 * kMaxSlots) D.smax[t] = 0ull;
  if (t != 0) return;
  D.nflag[0] = D.nflag[1] = D.nflag[2] = 0;
  const double v =
      stopped ? 0.0 : (D.dt_fixed ? *D.dt_fixed : D.cfl / __longlong_as_double((long long)m));
  const int halt = stopped ? stopped : ((!(v > 0.0) || !__builtin_isfinite(v)) ? D.n + 1 : 0);
  if (D.diag) D.diag[3] = halt ? 1 : 0;
  *D.stop = halt;
  *D.dt = v;
  if (D.dt_out) *D.dt_out = v;
}
__global__ void __launch_bounds__(kBlock) k_dt_final(DtStep D) { dt_step(D); }

// ---------------------------------------------------------------------------
// Cell-centred fields for the two-step EMF schemes (B25a: ideal EMF; FS18:
// velocity), over cells whose upper faces are stored.
// ---------------------------------------------------------------------------
template <typename T, int EMF>
__device__ __forceinline__ void prim_at(const State& S, const Geom& G, const Work<T>& W,
                                        double gamma, int t) {
  if (t >= G.elems) return;
  int i = t % G.N[0];
  int q = t / G.N[0];
  int j = q % G.N[1];
  int k = q / G.N[1];
  if (i >= G.N[0] - 1 || j >= G.N[1] - 1 || k >= G.N[2] - 1) return;
  double rho, u[3], p, b[3];
  cell_prim(S, G, t, gamma, rho, u, p, b);
  if (EMF == kB25A) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      int a = (c + 1) % 3, bb = (c + 2) % 3;
      // eq. emf:b25a-emf-centre in the stencil type
      W.ecell[c][t] = -(T)u[a] * (T)b[bb] + (T)u[bb] * (T)b[a];
    }
  } else {
    W.prim[1][t] = (T)u[0];
    W.prim[2][t] = (T)u[1];
    W.prim[3][t] = (T)u[2];
  }
}

template <typename T, int EMF>
__global__ void __launch_bounds__(kBlock) k_prim(State S, Geom G, Work<T> W, double gamma,
                                                 const int* stop) {
  if (*stop) return;
  prim_at<T, EMF>(S, G, W, gamma, gidx());
}

// eta j_c at the edge stored at s (lower corner in a and b), eq.
// resistivity:current-stencil.
template <typename T>
__device__ __forceinline__ T eta_j(const State& S, const Geom& G, int s, int c, T eta) {
  int a = (c + 1) % 3, b = (c + 2) % 3;
  double j = (S.b[b][s] - S.b[b][s - gstride(G, a)]) * G.idx[a] -
             (S.b[a][s] - S.b[a][s - gstride(G, b)]) * G.idx[b];
  return eta * (T)j;
}

// Joule energy flux at the x_a face stored at s (Sec. 2.4): (eta j x b).n_a
// with eta j averaged over the face's bounding edges and b the mean of the two
// adjacent cells' cell-averaged field.
template <typename T>
__device__ __forceinline__ T joule(const State& S, const Geom& G, int s, int a, T eta) {
  int b = (a + 1) % 3, c = (a + 2) % 3;
  const int sb = gstride(G, b), sc = gstride(G, c);
  T eb = T(0.5) * (eta_j<T>(S, G, s, b, eta) + eta_j<T>(S, G, s + sc, b, eta));
  T ec = T(0.5) * (eta_j<T>(S, G, s, c, eta) + eta_j<T>(S, G, s + sb, c, eta));
  int l = s - gstride(G, a);
  T bbl = (T)(0.5 * (S.b[b][l] + S.b[b][l + sb]));
  T bbr = (T)(0.5 * (S.b[b][s] + S.b[b][s + sb]));
  T bcl = (T)(0.5 * (S.b[c][l] + S.b[c][l + sc]));
  T bcr = (T)(0.5 * (S.b[c][s] + S.b[c][s + sc]));
  return eb * (T(0.5) * (bcl + bcr)) - ec * (T(0.5) * (bbl + bbr));
}

// The same Joule flux at the x_a face between cells lo and hi from values the
// face pass already holds: each cell's transverse face fields
// t = {b_b lower, b_b upper, b_c lower, b_c upper} (b, c cyclic after a),
// the face's normal field bn = b_a, and its four in-plane neighbours
// nb = {b_a at -x_b, +x_b, -x_c, +x_c}.  Every edge current, cell-averaged
// field and product is formed as in joule().
template <typename T>
__device__ __forceinline__ T joule_pair(const Geom& G, int a, const double lo[4],
                                        const double hi[4], double bn, const double nb[4], T eta) {
  // no fused multiply-adds: the single-box and batched face kernels inline
  // this into different code, and must give the same bits
#pragma clang fp contract(off)
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  // eta j_b at the edges s and s + x_c, eta j_c at the edges s and s + x_b
  T eb = T(0.5) * (eta * (T)((bn - nb[2]) * G.idx[c] - (hi[2] - lo[2]) * G.idx[a]) +
                   eta * (T)((nb[3] - bn) * G.idx[c] - (hi[3] - lo[3]) * G.idx[a]));
  T ec = T(0.5) * (eta * (T)((hi[0] - lo[0]) * G.idx[a] - (bn - nb[0]) * G.idx[b]) +
                   eta * (T)((hi[1] - lo[1]) * G.idx[a] - (nb[1] - bn) * G.idx[b]));
  T bbl = (T)(0.5 * (lo[0] + lo[1]));
  T bbr = (T)(0.5 * (hi[0] + hi[1]));
  T bcl = (T)(0.5 * (lo[2] + lo[3]));
  T bcr = (T)(0.5 * (hi[2] + hi[3]));
  return eb * (T(0.5) * (bcl + bcr)) - ec * (T(0.5) * (bbl + bbr));
}

// ---------------------------------------------------------------------------
// Face pass (Sec. 2.2, eqs. emf:alpha-pm, emf:q26-facevel).
// ---------------------------------------------------------------------------
// Face ranges of one stage.  Faces of direction a are solved at s_a in
// [lo_a, lo_a + nf_a), transverse coordinates in [tlo, tlo + tlen).
// A box that is periodic on itself (per = 1) solves each face once, on its
// interior range, and stores the values at every position of the ghost shell
// that the edge and update passes read too: the transverse positions
// [plo, phi], and the upper boundary face along the normal.  Solving those
// copies instead costs (n+1)(n+2r+2)^2 / n^3 of the faces per direction (PPM,
// Q26: 1.03 at 512^3, 1.45 at 32^3, 3.4 at 8^3).  A box of a level (per = 0)
// solves the shell itself, from its neighbours' cells.  Measured per launch
// (with the x rows end to end, below): FP64 512^3 16.77 -> 16.46 ms, 128^3
// 277 -> 253 us; 2000 boxes of 8 to 64 cells per axis, FP32, 9.27 -> 7.37 ms.
struct FacePlan {
  int lo[3], nf[3];   // along the face normal
  int tlo, tlen[3];   // transverse range start (same on every axis) and length per axis
  int per, plo, phi[3];
  int ulo[3], ulen[3];  // faces read by the update (Joule flux only there)
  // x part: the rows, each extended by its halo to xw = nf + 2r + 1 cells, laid
  // end to end; an item is 64 consecutive cells of that line
  int xw, xlen, xwaves, xrows, xblocks;  // xwaves = items; xrows items per wavefront
  int xdx, xdy, xdz;  // step of one item (64 - 2r - 1 cells) in (cell, row y, row z)
  // y and z parts: lane blocks x chunks
  int chunk[3], lanes[3], blocks[3];
  // The box is cut into nby x nbz bricks of wy x wz whole rows (ranges in y and
  // z), each with all three parts of its faces, and cy / cz chunks of the y / z
  // marches: a large box's state then comes from HBM about once, not once per
  // direction.
  int nby, nbz, wy, wz, cy, cz;
  int brick_blocks, total_blocks;
};

// Face-local primitive of a cell for the face normal a (FP64 recovery, then T).
template <typename T>
__device__ __forceinline__ void face_local_raw(const CellRaw& R, int a, double gamma, T v[7]) {
  double rho, u[3], p, bc[3];
  raw_prim(R, gamma, rho, u, p, bc);
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  v[0] = (T)rho;
  v[1] = (T)u[a];
  v[2] = (T)u[b];
  v[3] = (T)u[c];
  v[4] = (T)p;
  v[5] = (T)bc[b];
  v[6] = (T)bc[c];
}

template <typename T>
__device__ __forceinline__ void face_local(const State& S, const Geom& G, int s, int a, double gamma,
                                           T v[7]) {
  CellRaw R;
  cell_load(S, G, s, R);
  face_local_raw<T>(R, a, gamma, v);
}

// What the face pass stores per face: the flux (global momentum order), the
// outer wave speeds and the face velocity.
template <typename T>
struct FaceOut {
  T F[5], ap, am, us;
};

template <typename T, int RIEMANN>
__device__ __forceinline__ int solve_face(int a, const T qL[7], const T qR[7], double bn_d,
                                          double gamma_d, T jflux, FaceOut<T>& o) {
  // the solver's arithmetic type: T, or float64 for kHLLD64 / kLLF64
  using RT = typename std::conditional<(RIEMANN >= kHLLD64), double, T>::type;
  FState<RT> L{(RT)qL[0], (RT)qL[1], (RT)qL[2], (RT)qL[3], (RT)qL[4], (RT)qL[5], (RT)qL[6]};
  FState<RT> R{(RT)qR[0], (RT)qR[1], (RT)qR[2], (RT)qR[3], (RT)qR[4], (RT)qR[5], (RT)qR[6]};
  const RT bn = (RT)bn_d;  // normal field of the face, S.b[a][s]
  RT Fr[5];
  T F[5], ap, am;
  int fb = 0;
  if (RIEMANN == kHLLD || RIEMANN == kHLLD64) {
    RT SL, SR;
    fb = hlld_flux(L, R, bn, (RT)gamma_d, Fr, SL, SR);
    ap = (T)tmax(RT(0), SR);
    am = (T)tmax(RT(0), -SL);
  } else {
    ap = am = (T)llf_flux(L, R, bn, (RT)gamma_d, Fr);
  }
#pragma unroll
  for (int m = 0; m < 5; ++m) F[m] = (T)Fr[m];
  F[4] += jflux;  // Joule energy flux (zero outside the faces the update reads, or eta = 0)
  o.F[0] = F[0];
  o.F[1 + a] = F[1];
  o.F[1 + (a + 1) % 3] = F[2];
  o.F[1 + (a + 2) % 3] = F[3];
  o.F[4] = F[4];
  o.ap = ap;
  o.am = am;
  o.us = (ap * (T)L.un + am * (T)R.un) * trcp(ap + am);
  return fb;
}

// Streaming stores: no later access of this kernel reads them, and keeping
// them out of the L2 leaves it to the state rows the marches re-read.
template <typename T>
__device__ __forceinline__ void store_flux(const Work<T>& W, int s, int a, int stage,
                                           const FaceOut<T>& o) {
#pragma unroll
  for (int m = 0; m < 5; ++m) __builtin_nontemporal_store(o.F[m], &at(W.F[stage][a][m], s));
}
template <typename T>
__device__ __forceinline__ void store_speeds(const Work<T>& W, int s, int a, const FaceOut<T>& o) {
  __builtin_nontemporal_store(o.ap, &at(W.ap[a], s));
  __builtin_nontemporal_store(o.am, &at(W.am[a], s));
  __builtin_nontemporal_store(o.us, &at(W.us[a], s));
}

// Periodic copies p + m n_d, m in [mlo, mhi], of coordinate p of a solved x_a
// face that the later passes read.
__device__ __forceinline__ void image_range(const FacePlan& FP, const Geom& G, int a, int d, int p,
                                            int& mlo, int& mhi) {
  const int n = G.n[d];
  mlo = 0;
  mhi = 0;
  if (d == a) {
    mhi = p == FP.lo[a] ? 1 : 0;  // the upper boundary face
  } else {
    mlo = -((p - FP.plo) / n);
    mhi = (FP.phi[d] - p) / n;
  }
}

// Whether a transverse coordinate p has periodic copies in the shell.
__device__ __forceinline__ bool has_image(const FacePlan& FP, const Geom& G, int d, int p) {
  return FP.per && (p - G.n[d] >= FP.plo || p + G.n[d] <= FP.phi[d]);
}

// The copies of a solved face (per = 1): the flux at the upper boundary face
// (the update reads it on interior rows only), alpha and u* at the positions
// the edges read, which lie outside the interior along one transverse axis at
// most.  Few faces get here: those within r + 1 of the box's sides.
template <typename T>
__device__ __forceinline__ void store_images(const Work<T>& W, const Geom& G, const FacePlan& FP,
                                             const int s3[3], int s, int a, int stage,
                                             const FaceOut<T>& o) {
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  int la, ha, lb, hb, lc, hc;
  image_range(FP, G, a, a, s3[a], la, ha);
  image_range(FP, G, a, b, s3[b], lb, hb);
  image_range(FP, G, a, c, s3[c], lc, hc);
  for (int ma = la; ma <= ha; ++ma) {
    const int sa = s + ma * G.n[a] * G.st[a];
    if (ma) store_flux(W, sa, a, stage, o);
    for (int mb = lb; mb <= hb; ++mb)
      if (mb || ma) store_speeds(W, sa + mb * G.n[b] * G.st[b], a, o);
    for (int mc = lc; mc <= hc; ++mc)
      if (mc) store_speeds(W, sa + mc * G.n[c] * G.st[c], a, o);
  }
}

// Positions a solved face stands for: the fallback counter counts every
// position of the shell as one solved face.
__device__ __forceinline__ int face_copies(const FacePlan& FP, const Geom& G, const int s3[3],
                                           int a) {
  int w = 1;
  if (FP.per) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      int lo, hi;
      image_range(FP, G, a, d, s3[d], lo, hi);
      w *= hi - lo + 1;
    }
  }
  return w;
}

// Solve the x_a face at s3 (storage index s) and store it; img: the face's
// transverse coordinates have periodic copies.
template <typename T, int RIEMANN>
__device__ __forceinline__ int face_item(const Work<T>& W, const Geom& G, const FacePlan& FP,
                                         const int s3[3], int s, int a, int stage, bool img,
                                         const T qL[7], const T qR[7], double bn, double gamma,
                                         T jflux) {
  FaceOut<T> o;
  const int fb = solve_face<T, RIEMANN>(a, qL, qR, bn, gamma, jflux, o);
  store_flux(W, s, a, stage, o);
  store_speeds(W, s, a, o);
  if (img || (FP.per && s3[a] == FP.lo[a])) store_images(W, G, FP, s3, s, a, stage, o);
  return fb ? face_copies(FP, G, s3, a) : 0;
}

// Whether the face pass's x_a face at s3 is one the update reads: [g, g+n]
// along the normal, [g, g+n) across (the Joule flux is needed only there).
__device__ __forceinline__ bool face_in_update(const FacePlan& FP, const int s3[3], int a) {
  bool in_upd = true;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    in_upd = in_upd && s3[d] >= FP.ulo[d] && s3[d] < FP.ulo[d] + FP.ulen[d] + (d == a ? 1 : 0);
  return in_upd;
}

// A cell's transverse face fields for the normal a, as joule_pair takes them.
__device__ __forceinline__ void cell_tfaces(const CellRaw& R, int a, double t[4]) {
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  t[0] = R.bl[b];
  t[1] = R.bh[b];
  t[2] = R.bl[c];
  t[3] = R.bh[c];
}

// The four in-plane neighbours of the normal field of the x_a face at s, as
// joule_pair takes them.
__device__ __forceinline__ void face_nb(const State& S, const Geom& G, int s, int a,
                                        double nb[4]) {
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  const double* ba = S.b[a];
  nb[0] = nbr(ba, G, s, b, -1);
  nb[1] = nbr(ba, G, s, b, 1);
  nb[2] = nbr(ba, G, s, c, -1);
  nb[3] = nbr(ba, G, s, c, 1);
}

// Value of the neighbouring lane (l - 1 for lane_prev, l + 1 for lane_next)
// by a DPP whole-wavefront shift, a VALU move; lane 0 (63) receives 0 by the
// bound control, so that no register has to be cleared for it first.
__device__ __forceinline__ int dpp_prev(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true);  // wave_shr:1
}
__device__ __forceinline__ int dpp_next(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true);  // wave_shl:1
}
__device__ __forceinline__ double lane_prev(double v) {
  return __hiloint2double(dpp_prev(__double2hiint(v)), dpp_prev(__double2loint(v)));
}
__device__ __forceinline__ double lane_next(double v) {
  return __hiloint2double(dpp_next(__double2hiint(v)), dpp_next(__double2loint(v)));
}
__device__ __forceinline__ float lane_prev(float v) {
  return __int_as_float(dpp_prev(__float_as_int(v)));
}
__device__ __forceinline__ float lane_next(float v) {
  return __int_as_float(dpp_next(__float_as_int(v)));
}

// x faces: one wavefront holds 64 consecutive cells of a row; lane l forms
// the primitives, the limited slope and the upper interface value of its own
// cell, neighbours come from whole-wavefront DPP shifts by one lane, and the
// face at lane l takes the upper value of lane l-1.  Faces at lanes [r+1, 63-r]
// are resolved; the next 64 cells start 2r + 1 before the end of these.
template <int RECON, typename T>
__device__ __forceinline__ void recon_lanes(T q, T& qm, T& qp) {
  if constexpr (RECON == kPC) {
    qm = q;
    qp = q;
  } else if constexpr (RECON == kPLM_MC || RECON == kPLM_MM) {
    T s = T(0.5) * plm_slope<RECON>(lane_prev(q), q, lane_next(q));
    qm = q - s;
    qp = q + s;
  } else {
    T qr = lane_next(q);
    T dm = ppm_slope(lane_prev(q), q, qr);
    T ihi = ppm_iface(q, qr, dm, lane_next(dm));
    T ilo = lane_prev(ihi);
    ppm_constrain(q, ilo, ihi);
    qm = ilo;
    qp = ihi;
  }
}

// The rows of the x part, each with its halo of r + 1 cells below and r above
// the faces, are laid end to end, and item i holds cells [i (63 - 2r), ... + 63]
// of that line, so that a wavefront wastes lanes on halos only: 89% of them
// resolve faces at n = 128 (67% with three whole segments per row), 57% at
// n = 8 (13%).
template <typename T, int RECON, int RIEMANN>
__device__ void faces_x(const State& S, const Geom& G, const Work<T>& W, const FacePlan& FP,
                        int y0, int z0, int wave, int stage, double gamma, double eta,
                        int& nfb) {
  constexpr int r = recon_halfwidth(RECON);
  const int lane = threadIdx.x & 63;
  // this wavefront takes items [it, end) and loads the cells of the next item
  // before it resolves the current one
  int it = wave * FP.xrows;
  const int end = it + FP.xrows < FP.xwaves ? it + FP.xrows : FP.xwaves;
  // lane's cell: position x of extended row (y, z), all counted from the
  // start (y0, z0) of the brick's ranges; lanes past them stay on the last row
  int x, y, z;
  {
    const int e = it * (63 - 2 * r) + lane;
    const int row = e / FP.xw;
    x = e - row * FP.xw;
    z = row / FP.wy;
    y = row - z * FP.wy;
  }
  const int ymax = FP.tlen[1] - 1 - y0, zmax = (FP.wz < FP.tlen[2] - z0 ? FP.wz : FP.tlen[2] - z0) - 1;
  auto locate = [&](int s3[3]) {
    s3[0] = FP.lo[0] - (r + 1) + x;
    s3[1] = FP.tlo + y0 + (y < ymax ? y : ymax);
    s3[2] = FP.tlo + z0 + (z < zmax ? z : zmax);
    return s3[0] + G.st[1] * s3[1] + G.st[2] * s3[2];
  };
  // whether this lane resolves a face: it holds a face position and its
  // stencil lies in the wavefront
  auto is_face = [&]() {
    return lane >= r + 1 && lane <= 63 - r && x >= r + 1 && x <= r + FP.nf[0] && y <= ymax &&
           z <= zmax;
  };
  // whether this lane's face of an item needs the Joule flux; if so its
  // normal-field neighbours are loaded with the item's cell
  auto joule_nb = [&](const int s3[3], int s, double nb[4]) {
    const bool j = eta > 0.0 && is_face() && face_in_update(FP, s3, 0);
    if (j) face_nb(S, G, s, 0, nb);
    return j;
  };
  int n3[3];
  int sn = locate(n3);
  CellRaw nxt;
  cell_load_at(S, G, sn, nxt);
  double nb_nxt[4] = {0.0, 0.0, 0.0, 0.0};
  bool j_nxt = joule_nb(n3, sn, nb_nxt);
  for (; it < end; ++it) {  // wavefront-uniform trip count (cross-lane shifts below)
    const CellRaw cur = nxt;
    const int s3[3] = {n3[0], n3[1], n3[2]};
    const int s = sn;
    double nb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) nb[k] = nb_nxt[k];
    const bool jf_need = j_nxt, face = is_face();
    if (it + 1 < end) {
      // the next item's cell: one item step, with carries into y and z
      x += FP.xdx;
      y += FP.xdy;
      z += FP.xdz;
      if (x >= FP.xw) {
        x -= FP.xw;
        ++y;
      }
      if (y >= FP.wy) {
        y -= FP.wy;
        ++z;
      }
      sn = locate(n3);
      cell_load_at(S, G, sn, nxt);
      j_nxt = joule_nb(n3, sn, nb_nxt);
    }
    T v[7];
    face_local_raw<T>(cur, 0, gamma, v);
    T qm[7], qp[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) recon_lanes<RECON>(v[k], qm[k], qp[k]);
    T qL[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) qL[k] = lane_prev(qp[k]);
    // transverse face fields of this lane's cell and of the cell below it
    double thi[4], tlo[4];
    cell_tfaces(cur, 0, thi);
#pragma unroll
    for (int k = 0; k < 4; ++k) tlo[k] = lane_prev(thi[k]);
    if (face) {
      const T jf = jf_need ? joule_pair<T>(G, 0, tlo, thi, cur.bl[0], nb, (T)eta) : T(0);
      const bool img = has_image(FP, G, 1, s3[1]) || has_image(FP, G, 2, s3[2]);
      nfb += face_item<T, RIEMANN>(W, G, FP, s3, s, 0, stage, img, qL, qm, cur.bl[0], gamma, jf);
    }
  }
}

// y / z faces: lanes over the transverse plane (x fastest), each thread
// marches along the face normal A through a chunk of faces, streaming the
// cells through a reconstruction pipeline (one slope and one interface value
// per cell); each cell is loaded and reconstructed once.
template <typename T, int RECON, int RIEMANN, int A>
__device__ void faces_march(const State& S, const Geom& G, const Work<T>& W, const FacePlan& FP,
                            int c0, int lblock, int chunk, int stage, double gamma, double eta,
                            int& nfb) {
  constexpr int r = recon_halfwidth(RECON);
  const int lane = lblock * kBlock + threadIdx.x;
  if (lane >= FP.lanes[A]) return;
  const int C = A == 1 ? 2 : 1;  // transverse axes: x (fastest) and C
  int s3[3];
  s3[0] = FP.tlo + lane % FP.tlen[0];
  s3[C] = FP.tlo + c0 + lane / FP.tlen[0];
  if (s3[C] >= FP.tlo + FP.tlen[C] || chunk * FP.chunk[A] >= FP.nf[A]) return;  // outside the box
  const int f0 = FP.lo[A] + chunk * FP.chunk[A];
  int f1 = f0 + FP.chunk[A];
  if (f1 > FP.lo[A] + FP.nf[A]) f1 = FP.lo[A] + FP.nf[A];
  const int sa = G.st[A];
  const int base = s3[0] + G.st[C] * s3[C];
  const bool img = has_image(FP, G, 0, s3[0]) || has_image(FP, G, C, s3[C]);
  ReconStream<RECON, T> rs[7];
  T qprev[7];
  // cells f0-1-r .. f1-1+r; the pushes before cell f0-1+r only warm up the
  // pipeline.  The loads of cell q+1 and the normal field of the face it
  // completes are issued before the stores of the face completed by cell q.
  int q = f0 - 1 - r;
  CellRaw nxt;
  cell_load_at(S, G, base + q * sa, nxt);
  double bn_next = 0.0;  // read only for the faces f0 .. f1-1
  // Joule flux of face q (between cells q-1 and q), formed when cell q
  // arrives and used r pushes later, when the face is solved: jd[k] holds the
  // flux of face q-k
  double tprev[4] = {0.0, 0.0, 0.0, 0.0};
  T jd[r + 1];
#pragma unroll
  for (int k = 0; k <= r; ++k) jd[k] = T(0);
  // the normal-field neighbours of face q+1 are loaded with cell q+1 when
  // that face needs the Joule flux
  double nb_next[4] = {0.0, 0.0, 0.0, 0.0};
  bool j_next = false;
  for (; q <= f1 - 1 + r; ++q) {
    const CellRaw cur = nxt;
    const double bn = bn_next;
    double nb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) nb[k] = nb_next[k];
    const bool jq = j_next;
    if (q < f1 - 1 + r) {
      cell_load_at(S, G, base + (q + 1) * sa, nxt);
      if (q + 1 - r >= f0) bn_next = at(S.b[A], base + (q + 1 - r) * sa);
      j_next = false;
      if (eta > 0.0 && q + 1 >= f0 && q + 1 < f1) {
        s3[A] = q + 1;
        j_next = face_in_update(FP, s3, A);
        if (j_next) face_nb(S, G, base + (q + 1) * sa, A, nb_next);
      }
    }
#pragma unroll
    for (int k = r; k > 0; --k) jd[k] = jd[k - 1];
    double tcur[4];
    cell_tfaces(cur, A, tcur);
    jd[0] = jq ? joule_pair<T>(G, A, tprev, tcur, cur.bl[A], nb, (T)eta) : T(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) tprev[k] = tcur[k];
    T v[7];
    face_local_raw<T>(cur, A, gamma, v);
    const int cell = q - r;  // completed by this push
    T qm[7], qp[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) rs[k].push(v[k], qm[k], qp[k]);
    if (cell >= f0) {
      s3[A] = cell;
      nfb += face_item<T, RIEMANN>(W, G, FP, s3, base + cell * sa, A, stage, img, qprev, qm, bn,
                                   gamma, jd[r]);
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) qprev[k] = qp[k];
  }
}

// One virtual block (256 threads) of the face pass.
template <typename T, int RECON, int RIEMANN>
__device__ __forceinline__ void faces_block(const State& S, const Geom& G, const Work<T>& W,
                                            const FacePlan& FP, int b, int stage, double gamma,
                                            double eta, int& nfb) {
  const int brick = b / FP.brick_blocks;
  b -= brick * FP.brick_blocks;
  const int iz = brick / FP.nby, iy = brick - iz * FP.nby;
  const int y0 = iy * FP.wy, z0 = iz * FP.wz;
  // long-running marching blocks first, the short x-face wavefronts fill in
  if (b < FP.blocks[2]) {
    faces_march<T, RECON, RIEMANN, 2>(S, G, W, FP, y0, b / FP.cz, iz * FP.cz + b % FP.cz, stage,
                                      gamma, eta, nfb);
  } else if ((b -= FP.blocks[2]) < FP.blocks[1]) {
    faces_march<T, RECON, RIEMANN, 1>(S, G, W, FP, z0, b / FP.cy, iy * FP.cy + b % FP.cy, stage,
                                      gamma, eta, nfb);
  } else {
    b -= FP.blocks[1];
    const int wave = b * (kBlock / 64) + (threadIdx.x >> 6);
    if (wave * FP.xrows < FP.xwaves)
      faces_x<T, RECON, RIEMANN>(S, G, W, FP, y0, z0, wave, stage, gamma, eta, nfb);
  }
}

template <typename T>
struct FaceArgs {
  State S;
  Geom G;
  Work<T> W;
  FacePlan FP;
  int stage;
  double gamma, eta;
  long long* diag;
  const int* stop;
  DtStep D;  // the step's dt, formed by an extra workgroup (first stage of a step)
};

// The arguments are read where they are used, through the kernel argument
// segment as constant memory: scalar loads inside the three parts.  As by-value
// arguments the compiler loads all of them (about 60 pointers) at the top of
// the kernel and spills what does not fit the scalar registers to vector lanes:
// 24 to 38 v_readlane per face in the marches, one in 25 VALU instructions.
template <typename T, int RECON, int RIEMANN>
__global__ void __launch_bounds__(kBlock) k_faces(FaceArgs<T> byval) {
  (void)byval;
  const FaceArgs<T>& A =
      *(const FaceArgs<T>*)(const CTMHD_CONST FaceArgs<T>*)__builtin_amdgcn_kernarg_segment_ptr();
  if ((int)blockIdx.x == A.FP.total_blocks) {
    // nothing before the update needs dt, so it has no launch of its own; the
    // faces of a step that this stops are solved in vain
    dt_step(A.D);
    return;
  }
  if (*A.stop) return;
  int nfb = 0;
  faces_block<T, RECON, RIEMANN>(A.S, A.G, A.W, A.FP, blockIdx.x, A.stage, A.gamma, A.eta, nfb);
  if (A.diag && nfb) atomicAdd((unsigned long long*)&A.diag[2], (unsigned long long)nfb);
}

// ---------------------------------------------------------------------------
// Edge pass (Sec. 2.3): face field reconstructed to the edge, four corner
// EMFs of the chosen compute scheme, LD04 averaging, plus eta j.
// ---------------------------------------------------------------------------
template <int RECON, typename T>
__device__ __forceinline__ void iface_along(const T* A, int s, int stride, T& lo, T& hi) {
  T q[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) q[m] = stencil_uses<RECON>(m) ? A[s + (m - 3) * stride] : T(0);
  recon_iface<RECON>(q, lo, hi);
}

template <int RECON, typename T>
__device__ __forceinline__ void iface_along_d(const double* A, int s, int stride, T& lo, T& hi) {
  T q[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) q[m] = stencil_uses<RECON>(m) ? (T)A[s + (m - 3) * stride] : T(0);
  recon_iface<RECON>(q, lo, hi);
}

// Two-step reconstruction of a cell-centred field to the four corners of the
// edge at s: first along d1 to the x_d1 face, then along d2 to the edge.
// out[s1 + 2*s2] with s = 0 lower side, 1 upper side along each direction.
template <int RECON, typename T>
__device__ __forceinline__ void two_step(const T* A, int s, int st1, int st2, T out[4]) {
  T seqlo[6], seqhi[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    if (!stencil_uses<RECON>(m)) {
      seqlo[m] = seqhi[m] = T(0);
    } else {
      iface_along<RECON>(A, s + (m - 3) * st2, st1, seqlo[m], seqhi[m]);
    }
  }
  T l0, l1, h0, h1;
  recon_iface<RECON>(seqlo, l0, l1);
  recon_iface<RECON>(seqhi, h0, h1);
  out[0] = l0;  // (lower along d1, lower along d2)
  out[1] = h0;  // (upper, lower)
  out[2] = l1;  // (lower, upper)
  out[3] = h1;  // (upper, upper)
}

// Whether the two-step corner reconstructions of B25a and FS18 store their
// first step once per stage (PPM) or the edge pass recomputes it for every
// edge that reads it (PC, PLM: there the stored arrays cost more traffic than
// the short stencils they save).
__host__ __device__ constexpr bool first_step_stored(int emf, int recon) {
  return emf != kQ26 && recon == kPPM;
}

// The first step of the two-step corner reconstructions at position t, for
// every field and axis the edges use; 0 where the stencil leaves the box.
template <typename T, int RECON, int EMF>
__device__ __forceinline__ void first_step_at(const Geom& G, const Work<T>& W, int t) {
  if (t >= G.elems) return;
  const int s3[3] = {t % G.N[0], (t / G.N[0]) % G.N[1], t / (G.N[0] * G.N[1])};
  constexpr int r = recon_halfwidth(RECON);
  constexpr int nf = EMF == kB25A ? 2 : 3;  // orders of ecell[c] / axes of u_v
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int o = 0; o < nf; ++o) {
      const int d1 = EMF == kB25A ? (o == 0 ? (c + 1) % 3 : (c + 2) % 3) : o;
      const T* A = EMF == kB25A ? W.ecell[c] : W.prim[1 + c];
      T lo = T(0), hi = T(0);
      if (s3[d1] - 1 - r >= 0 && s3[d1] + r < G.N[d1])
        iface_along<RECON>(A, t, gstride(G, d1), lo, hi);
      T* const* out = EMF == kB25A ? W.b25f[c][o] : W.fsf[c][o];
      __builtin_nontemporal_store(lo, &out[0][t]);  // read by the edge pass only
      __builtin_nontemporal_store(hi, &out[1][t]);
    }
}

template <typename T, int RECON, int EMF>
__global__ void __launch_bounds__(kBlock) k_first_step(Geom G, Work<T> W, const int* stop) {
  if (*stop) return;
  first_step_at<T, RECON, EMF>(G, W, gidx());
}

// Second step of a two-step reconstruction from the stored first-step
// values F[0] (lower side) and F[1] (upper side along d1), along d2 with
// stride st2: the same values as two_step.
template <int RECON, typename T>
__device__ __forceinline__ void second_step(T* const F[2], int s, int st2, T out[4]) {
  T seqlo[6], seqhi[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    seqlo[m] = stencil_uses<RECON>(m) ? F[0][s + (m - 3) * st2] : T(0);
    seqhi[m] = stencil_uses<RECON>(m) ? F[1][s + (m - 3) * st2] : T(0);
  }
  T l0, l1, h0, h1;
  recon_iface<RECON>(seqlo, l0, l1);
  recon_iface<RECON>(seqhi, h0, h1);
  out[0] = l0;
  out[1] = h0;
  out[2] = l1;
  out[3] = h1;
}

// Q26 corner EMFs (eq. emf:q26) from the edge-reconstructed face velocities
// u*_a (B/T along x_b), u*_b (L/R along x_a) and face fields, combined by LD04
// (eq. emf:ld04) with the edge wavespeeds (eq. emf:alpha-edge).
template <typename T>
__device__ __forceinline__ T q26_ld04(T uaB, T uaT, T ubL, T ubR, T baB, T baT, T bbL, T bbR,
                                      T apa, T ama, T apb, T amb) {
  const T e0 = -uaB * bbL + ubL * baB;
  const T e1 = -uaB * bbR + ubR * baB;
  const T e2 = -uaT * bbL + ubL * baT;
  const T e3 = -uaT * bbR + ubR * baT;
  return ld04(e0, e1, e2, e3, apa, ama, apb, amb, baB, baT, bbL, bbR);
}

// The Q26 EMF of the c edge at s from its edge-reconstructed face fields and
// face velocities: edge wave speeds (eq. emf:alpha-edge), Q26 corners with
// LD04, plus eta j.
template <typename T>
__device__ __forceinline__ T q26_edge(const State& S, const Geom& G, const Work<T>& W, int s, int c,
                                      T baB, T baT, T bbL, T bbR, T uaB, T uaT, T ubL, T ubR,
                                      double eta_d) {
  const int a = (c + 1) % 3, b = (c + 2) % 3;
  const int sa = gstride(G, a), sb = gstride(G, b);
  T apa = tmax(W.ap[a][s - sb], W.ap[a][s]);
  T ama = tmax(W.am[a][s - sb], W.am[a][s]);
  T apb = tmax(W.ap[b][s - sa], W.ap[b][s]);
  T amb = tmax(W.am[b][s - sa], W.am[b][s]);
  T eps = q26_ld04(uaB, uaT, ubL, ubR, baB, baT, bbL, bbR, apa, ama, apb, amb);
  if (eta_d > 0.0) eps += eta_j<T>(S, G, s, c, (T)eta_d);
  return eps;
}

template <typename T, int RECON, int EMF>
__device__ __forceinline__ T edge_emf(const State& S, const Geom& G, const Work<T>& W, int s, int c,
                                      double eta_d) {
  const int a = (c + 1) % 3, b = (c + 2) % 3;
  const int sa = gstride(G, a), sb = gstride(G, b);
  T baB, baT, bbL, bbR;
  iface_along_d<RECON>(S.b[a], s, sb, baB, baT);
  iface_along_d<RECON>(S.b[b], s, sa, bbL, bbR);
  if (EMF == kQ26) {
    T uaB, uaT, ubL, ubR;
    iface_along<RECON>(W.us[a], s, sb, uaB, uaT);
    iface_along<RECON>(W.us[b], s, sa, ubL, ubR);
    return q26_edge<T>(S, G, W, s, c, baB, baT, bbL, bbR, uaB, uaT, ubL, ubR, eta_d);
  }
  T apa = tmax(W.ap[a][s - sb], W.ap[a][s]);
  T ama = tmax(W.am[a][s - sb], W.am[a][s]);
  T apb = tmax(W.ap[b][s - sa], W.ap[b][s]);
  T amb = tmax(W.am[b][s - sa], W.am[b][s]);
  T e[4];  // LB, RB, LT, RT
  if (EMF == kB25A) {
    T ab[4], ba[4];  // [x_a x_b]: index sa_side + 2 sb_side; [x_b x_a]: sb_side + 2 sa_side
    if constexpr (first_step_stored(EMF, RECON)) {
      second_step<RECON>(W.b25f[c][0], s, sb, ab);
      second_step<RECON>(W.b25f[c][1], s, sa, ba);
    } else {
      two_step<RECON>(W.ecell[c], s, sa, sb, ab);
      two_step<RECON>(W.ecell[c], s, sb, sa, ba);
    }
    e[0] = T(0.5) * (ab[0] + ba[0]);
    e[1] = T(0.5) * (ab[1] + ba[2]);
    e[2] = T(0.5) * (ab[2] + ba[1]);
    e[3] = T(0.5) * (ab[3] + ba[3]);
  } else {
    T ua_ab[4], ua_ba[4], ub_ab[4], ub_ba[4];
    if constexpr (first_step_stored(EMF, RECON)) {
      second_step<RECON>(W.fsf[a][a], s, sb, ua_ab);
      second_step<RECON>(W.fsf[a][b], s, sa, ua_ba);
      second_step<RECON>(W.fsf[b][a], s, sb, ub_ab);
      second_step<RECON>(W.fsf[b][b], s, sa, ub_ba);
    } else {
      const T* ua = W.prim[1 + a];
      const T* ub = W.prim[1 + b];
      two_step<RECON>(ua, s, sa, sb, ua_ab);
      two_step<RECON>(ua, s, sb, sa, ua_ba);
      two_step<RECON>(ub, s, sa, sb, ub_ab);
      two_step<RECON>(ub, s, sb, sa, ub_ba);
    }
    const int perm[4] = {0, 2, 1, 3};  // corner q = sa_side + 2 sb_side -> [x_b x_a] index
    const T bbX[2] = {bbL, bbR}, baY[2] = {baB, baT};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      T u1 = T(0.5) * (ua_ab[q] + ua_ba[perm[q]]);
      T u2 = T(0.5) * (ub_ab[q] + ub_ba[perm[q]]);
      e[q] = -u1 * bbX[q & 1] + u2 * baY[q >> 1];
    }
  }
  T eps = ld04(e[0], e[1], e[2], e[3], apa, ama, apb, amb, baB, baT, bbL, bbR);
  if (eta_d > 0.0) eps += eta_j<T>(S, G, s, c, (T)eta_d);
  return eps;
}

// Edge directions [C0, C1) at the edge positions [g, g+n] on every axis (an
// edge of direction c exists for s_c < g + n_c).
template <typename T, int RECON, int EMF, int C0, int C1>
__device__ __forceinline__ void emf_at(const State& S, const Geom& G, const Work<T>& W, int stage,
                                       double eta_d, int t) {
  const int L0 = G.n[0] + 1, L1 = G.n[1] + 1, L2 = G.n[2] + 1;
  if (t >= L0 * L1 * L2) return;
  int s3[3] = {G.g + t % L0, G.g + (t / L0) % L1, G.g + t / (L0 * L1)};
  int s = s3[0] + G.st[1] * s3[1] + G.st[2] * s3[2];
#pragma unroll
  for (int c = C0; c < C1; ++c)
    if (s3[c] < G.g + G.n[c]) W.E[stage][c][s] = edge_emf<T, RECON, EMF>(S, G, W, s, c, eta_d);
}

// split > 0: one edge direction per thread, `split` workgroups per direction.
// A small box leaves the chip idle while each thread forms its three edges one
// after the other: 16^3 PPM Q26 12.0 -> 5.7 us per launch.
template <typename T, int RECON, int EMF>
__global__ void __launch_bounds__(kBlock)
    k_emf3(State S, Geom G, Work<T> W, int stage, double eta_d, int band, int split,
           const int* stop) {
  if (*stop) return;
  if (split > 0) {
    const int c = (int)blockIdx.x / split;
    const int t = ((int)blockIdx.x - c * split) * kBlock + (int)threadIdx.x;
    if (c == 0)
      emf_at<T, RECON, EMF, 0, 1>(S, G, W, stage, eta_d, t);
    else if (c == 1)
      emf_at<T, RECON, EMF, 1, 2>(S, G, W, stage, eta_d, t);
    else
      emf_at<T, RECON, EMF, 2, 3>(S, G, W, stage, eta_d, t);
    return;
  }
  emf_at<T, RECON, EMF, 0, 3>(S, G, W, stage, eta_d,
                              xcd_band_tile(band) * kBlock + (int)threadIdx.x);
}

// The same 1D interface values for a row of cells across a wavefront: q is the
// lane's cell, lo / hi the values on the lower and upper side of the interface
// below it (valid r + 1 lanes from the lower and r from the upper end).
template <int RECON, typename T>
__device__ __forceinline__ void iface_lanes(T q, T& lo, T& hi) {
  T qp;
  recon_lanes<RECON>(q, hi, qp);
  lo = lane_prev(qp);
}

// y interface values at s of an array whose own value is known (q0, cast to
// the stencil type); below: the element at s - sy.
template <int RECON, typename T, typename U>
__device__ __forceinline__ void iface_y(const U* A, int s, int sy, U q0, U& below, T& lo, T& hi) {
  T q[6];
  below = at(A, s - sy);
#pragma unroll
  for (int m = 0; m < 6; ++m)
    q[m] = !stencil_uses<RECON>(m) ? T(0)
           : m == 3 ? (T)q0 : m == 2 ? (T)below : (T)at(A, s + (m - 3) * sy);
  recon_iface<RECON>(q, lo, hi);
}

// Q26 EMFs of a row of edge columns per wavefront (64 consecutive x, y fixed),
// marching up z over [z0, z1).  Each of the twelve reconstructions of a
// position takes the cheapest form its axis allows, all of them the arithmetic
// of edge_emf on the same cells:
//   along z (B_y, u*_y at the x edges, B_x, u*_x at the y edges) streams that
//     take one cell and complete one per position, as in the face marches;
//   along x (B_y, u*_y at the z edges, B_z, u*_z at the y edges) one cell per
//     lane, neighbours by whole-wavefront shifts, as in the x faces: 59 of 64
//     lanes resolve positions with PPM;
//   along y (B_x, u*_x at the z edges, B_z, u*_z at the x edges) six loads each,
//     their own value from the stream or shared.
// Edge speeds and eta j take the x neighbours from the lane below and the z
// neighbours from the position before.  Against twelve six-point forms with the
// z ones streamed (1168 VALU instructions and 64 loads per position in the FP64
// PPM kernel, now 1040 and 38): 512^3 FP64 PPM 7.53 -> 6.40 ms per launch, 256^3
// FP64 PLM 767 -> 565 us, 256^3 FP32 604 -> 533, 128^3 FP64 146 -> 125.
template <typename T, int RECON>
__device__ __forceinline__ void emf_march_q26(const State& S, const Geom& G, const Work<T>& W,
                                              int stage, double eta_d, int item, int z0, int z1) {
  constexpr int r = recon_halfwidth(RECON);
  const int lane = threadIdx.x & 63;
  const int sy = G.st[1], sz = G.st[2];
  // this lane's column: cell xi of the extended row yi (rows of n0 + 1 edge
  // positions and their halo, laid end to end)
  const int xw = G.n[0] + 2 * r + 2;
  const int e = item * (63 - 2 * r) + lane;
  int yi = e / xw;
  const int xi = e - yi * xw;
  const bool mine = lane >= r + 1 && lane <= 63 - r && xi >= r + 1 && xi <= r + 1 + G.n[0] &&
                    yi <= G.n[1];
  if (yi > G.n[1]) yi = G.n[1];
  const int x = G.g - (r + 1) + xi, y = G.g + yi;
  const bool xe = mine && x < G.g + G.n[0], ye = mine && yi < G.n[1];  // x / y edges here
  const int base = x + sy * y;
  ReconStream<RECON, T> rs[4];  // B_y, u*_y (x edges), B_x, u*_x (y edges)
  T lo[4];                      // upper values of the cell below the next position
  // the position below: speeds of the x and y faces, b_x and b_y
  T apx0, amx0, apy0, amy0;
  double bx0, by0;
  {
    const int s = base + (z0 - 1) * sz;
    apx0 = at(W.ap[0], s);
    amx0 = at(W.am[0], s);
    apy0 = at(W.ap[1], s);
    amy0 = at(W.am[1], s);
    bx0 = at(S.b[0], s);
    by0 = at(S.b[1], s);
  }
  // cells z0-1-r .. z1-1+r; the pushes before cell z0-1+r only fill the
  // pipelines (their streams' cells lie in the ghost layers)
  for (int q = z0 - 1 - r; q <= z1 - 1 + r; ++q) {
    const int sq = base + q * sz;
    const T v[4] = {(T)at(S.b[1], sq), at(W.us[1], sq), (T)at(S.b[0], sq), at(W.us[0], sq)};
    T own[4];  // the values of the cell completed by this push
    T qm[4], qp[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      own[k] = RECON == kPPM ? rs[k].q2 : RECON == kPC ? v[k] : rs[k].q1;
      rs[k].push(v[k], qm[k], qp[k]);
    }
    const int z = q - r;
    if (z >= z0) {
      const int s = base + z * sz;
      const double bz = at(S.b[2], s);
      const T uz = at(W.us[2], s);
      // own face fields in double (the streams hold the stencil type)
      double bx, by;
      if constexpr (std::is_same<T, double>::value) {
        by = own[0];
        bx = own[2];
      } else {
        by = at(S.b[1], s);
        bx = at(S.b[0], s);
      }
      double bx_y, bz_y;  // b_x and b_z at s - sy
      T u_y;
      const T apx = at(W.ap[0], s), amx = at(W.am[0], s);
      const T apy = at(W.ap[1], s), amy = at(W.am[1], s);
      const T apz = at(W.ap[2], s), amz = at(W.am[2], s);
      // edge direction c with a = c+1, b = c+2
      T e0, e1, e2;
      {
        T zyL, zyR, uzyL, uzyR;
        iface_y<RECON>(S.b[2], s, sy, bz, bz_y, zyL, zyR);
        iface_y<RECON>(W.us[2], s, sy, uz, u_y, uzyL, uzyR);
        const T apz_y = at(W.ap[2], s - sy), amz_y = at(W.am[2], s - sy);
        e0 = q26_ld04(lo[1], qm[1], uzyL, uzyR, lo[0], qm[0], zyL, zyR, tmax(apy0, apy),
                      tmax(amy0, amy), tmax(apz_y, apz), tmax(amz_y, amz));
      }
      {
        T zxL, zxR, uzxL, uzxR;
        iface_lanes<RECON>((T)bz, zxL, zxR);
        iface_lanes<RECON>(uz, uzxL, uzxR);
        const T apz_x = lane_prev(apz), amz_x = lane_prev(amz);
        e1 = q26_ld04(uzxL, uzxR, lo[3], qm[3], zxL, zxR, lo[2], qm[2], tmax(apz_x, apz),
                      tmax(amz_x, amz), tmax(apx0, apx), tmax(amx0, amx));
      }
      {
        T xyL, xyR, uxyL, uxyR, yxL, yxR, uyxL, uyxR;
        iface_y<RECON>(S.b[0], s, sy, bx, bx_y, xyL, xyR);
        iface_y<RECON>(W.us[0], s, sy, own[3], u_y, uxyL, uxyR);
        iface_lanes<RECON>(own[0], yxL, yxR);
        iface_lanes<RECON>(own[1], uyxL, uyxR);
        const T apx_y = at(W.ap[0], s - sy), amx_y = at(W.am[0], s - sy);
        const T apy_x = lane_prev(apy), amy_x = lane_prev(amy);
        e2 = q26_ld04(uxyL, uxyR, uyxL, uyxR, xyL, xyR, yxL, yxR, tmax(apx_y, apx),
                      tmax(amx_y, amx), tmax(apy_x, apy), tmax(amy_x, amy));
      }
      if (eta_d > 0.0) {  // eta_j
        const T eta = (T)eta_d;
        const double by_x = lane_prev(by), bz_x = lane_prev(bz);
        const double j0 = (bz - bz_y) * G.idx[1] - (by - by0) * G.idx[2];
        const double j1 = (bx - bx0) * G.idx[2] - (bz - bz_x) * G.idx[0];
        const double j2 = (by - by_x) * G.idx[0] - (bx - bx_y) * G.idx[1];
        e0 += eta * (T)j0;
        e1 += eta * (T)j1;
        e2 += eta * (T)j2;
      }
      if (xe) at(W.E[stage][0], s) = e0;
      if (ye) at(W.E[stage][1], s) = e1;
      if (mine && z < G.g + G.n[2]) at(W.E[stage][2], s) = e2;
      apx0 = apx;
      amx0 = amx;
      apy0 = apy;
      amy0 = amy;
      bx0 = bx;
      by0 = by;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) lo[k] = qp[k];
  }
}

// Wavefront items of the z-marching Q26 edge pass.
__host__ __device__ inline int emf_march_items(const Geom& G, int r) {
  const int len = (G.n[0] + 2 * r + 2) * (G.n[1] + 1);
  return (len - 2 * r - 1 + 62 - 2 * r) / (63 - 2 * r);
}

// Q26 edge pass as z marches: workgroup tile = chunk * ctiles + tile of four
// items, z chunks of zc positions.  Through xcd_tile each XCD takes a contiguous
// run of tiles: a slab of z chunks over a band of rows, so the y neighbours a
// column reads share its XCD's L2.
// (Three wavefronts per SIMD: 166 registers.  At four the PPM kernel spills and
// takes twice as long.)
template <typename T, int RECON>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
    k_emf_march(State S, Geom G, Work<T> W, int stage, double eta_d, int ctiles, int zc,
                const int* stop) {
  if (*stop) return;
  const int tile = xcd_tile();
  const int item = (tile % ctiles) * (kBlock / 64) + (int)(threadIdx.x >> 6);
  if (item >= emf_march_items(G, recon_halfwidth(RECON))) return;  // whole wavefronts
  const int z0 = G.g + (tile / ctiles) * zc;
  const int zend = G.g + G.n[2] + 1;
  emf_march_q26<T, RECON>(S, G, W, stage, eta_d, item, z0, z0 + zc < zend ? z0 + zc : zend);
}

// ---------------------------------------------------------------------------
// Update (eqs. rk:increment-state, rk:increment-bfield, rk1:update,
// rk2:update).  stage 0: out = S^n + D^n.  stage 1: out = S^n + (D^n +
// D^{n+1/2})/2.  Increments are formed in FP64 from the stored fluxes and
// EMFs (which are single-valued per face and edge: conservation and div b
// hold to FP64 round-off in both precision forms), without contraction into
// fused multiply-adds.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ double dcons(const Geom& G, const Work<T>& W, int st, int s, int m,
                                        double dt) {
#pragma clang fp contract(off)
  double f = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const T* Fa = W.F[st][a][m];
    f += ((double)Fa[s] - (double)Fa[s + gstride(G, a)]) * G.idx[a];
  }
  return dt * f;
}

// increment of the face field b_a stored at s
template <typename T>
__device__ __forceinline__ double dface(const Geom& G, const Work<T>& W, int st, int s, int a,
                                        double dt) {
#pragma clang fp contract(off)
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  const T* Ec = W.E[st][c];
  const T* Eb = W.E[st][b];
  double circ = ((double)Ec[s] - (double)Ec[s + gstride(G, b)]) * G.idx[b] +
                ((double)Eb[s + gstride(G, c)] - (double)Eb[s]) * G.idx[c];
  return dt * circ;
}

// New face field.  stage 0: b^n + D^n.  stage 1, main pass: the SSP form
// (b^n + b^{n+1/2} + D^{n+1/2}) / 2, which equals b^n + (D^n + D^{n+1/2}) / 2
// up to round-off and does not re-read the first-stage EMFs; stage 1 after a
// first-order replacement: b^n + (D^n + D^{n+1/2}) / 2 with the replaced
// values of both stages.
template <typename T>
__device__ __forceinline__ double new_face(const State& base, const State& half, const Geom& G,
                                           const Work<T>& W, int stage, int fixup, int s, int a,
                                           double dt) {
#pragma clang fp contract(off)
  if (stage == 0) return base.b[a][s] + dface(G, W, 0, s, a, dt);
  if (!fixup) return 0.5 * (base.b[a][s] + half.b[a][s] + dface(G, W, 1, s, a, dt));
  return base.b[a][s] + 0.5 * (dface(G, W, 0, s, a, dt) + dface(G, W, 1, s, a, dt));
}

struct UpdateCfg {
  int fofc;          // flag the new state
  int crit;          // CTMHD_FLAG_*
  double gamma;
  double sres;       // resistive signal speed term of the CFL maximum
  const uint8_t* force;  // forced flags of this stage or null
  int flag_storage;  // 1: flags indexed by storage position (a level of boxes)
};

// The new conserved values c and lower face fields bl of the cell at s and,
// with need_state, its upper face fields bu (for the flags and the CFL signal).
// fix: the form after a first-order replacement.  bu takes the form of this
// cell, which is the one its owner stored but at the rim of a fix-up: between a
// rewritten cell and an unwritten one the two forms of the second stage differ
// by round-off, and so does the CFL signal there from that of the stored state.
// The stored fields have one owner each and are single-valued.
template <typename T, int stage, int fix>
__device__ __forceinline__ void cell_form(const State& base, const State& half, const Geom& G,
                                          const Work<T>& W, bool need_state, int s, double dt,
                                          double c[5], double bl[3], double bu[3]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    if (stage == 0)
      c[m] = base.c[m][s] + dcons(G, W, 0, s, m, dt);
    else if (!fix)
      c[m] = 0.5 * (base.c[m][s] + half.c[m][s] + dcons(G, W, 1, s, m, dt));
    else
      c[m] = base.c[m][s] + 0.5 * (dcons(G, W, 0, s, m, dt) + dcons(G, W, 1, s, m, dt));
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) bl[a] = new_face(base, half, G, W, stage, fix, s, a, dt);
  if (need_state) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
      bu[a] = new_face(base, half, G, W, stage, fix, s + gstride(G, a), a, dt);
  }
}

// The fix-up touches only the cells that the first-order values can reach: those
// with a flagged cell among their 27 neighbours (faces and edges are shared by
// no others).  The main update of a stage leaves, in the speed arrays that only
// the face and edge passes before it use, the list of its flagged cells and a
// word per item (256 strips cells): non-zero, in the second stage the item's
// CFL maximum.  The first-order pass works through the list and clears the
// words of the items it reaches; the fix-up skips the others.  On the 128^3
// Mach-5 box with some cells flagged (FP64 PPM Q26), first-order pass and fix-up
// of the first / second stage take 26 + 19 / 42 us; 57 + 144 / 262 us when both
// went over the whole box.  In a level, whose flags come from the neighbouring
// boxes too, both go over the whole boxes, for the same cells.
template <typename T>
__device__ __forceinline__ int* flag_list(const Work<T>& W) {
  return (int*)W.am[0];
}
template <typename T>
__device__ __forceinline__ unsigned* item_word(const Work<T>& W, int item) {
  return (unsigned*)W.ap[0] + 2 * (size_t)item;
}
// Whether the first-order pass works through the list (few flagged cells).
__device__ __forceinline__ bool few_flagged(const Geom& G, int nflag) {
  return 27LL * nflag < (long long)G.n[0] * G.n[1] * G.n[2];
}

__device__ __forceinline__ int interior_id(const Geom& G, int s0, int s1, int s2) {
  int i = (s0 - G.g) % G.n[0];
  if (i < 0) i += G.n[0];
  int j = (s1 - G.g) % G.n[1];
  if (j < 0) j += G.n[1];
  int k = (s2 - G.g) % G.n[2];
  if (k < 0) k += G.n[2];
  return i + G.n[0] * (j + G.n[1] * k);
}

// Flag of the cell at storage coordinates p3: periodic box (interior flags,
// wrapped) or a level of boxes (flags at every storage position, the ghost
// layers filled from the neighbouring boxes).
template <typename T>
__device__ __forceinline__ uint8_t flag_of(const Geom& G, const Work<T>& W, bool lvl,
                                           const int p3[3]) {
  if (lvl) return W.flag[p3[0] + G.st[1] * p3[1] + G.st[2] * p3[2]];
  return W.flag[interior_id(G, p3[0], p3[1], p3[2])];
}

// Whether a cell (storage coordinates) or one of its neighbours is flagged.
template <typename T>
__device__ __forceinline__ bool near_flagged(const Geom& G, const Work<T>& W, bool lvl,
                                             const int s3[3]) {
  int f = 0;
  for (int dz = -1; dz <= 1; ++dz)
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        const int p3[3] = {s3[0] + dx, s3[1] + dy, s3[2] + dz};
        f |= flag_of(G, W, lvl, p3);
      }
  return f != 0;
}

// fixup = 0: main update (flags, and for stage 1 the CFL maximum into slot 0)
// fixup = 1: after first-order replacement; runs only if this stage flagged
//            cells; stage 1 recomputes the CFL maximum into slot 1.
// stage and fixup as constants: each form of the update is straight-line
// code, so that every load of a cell can be issued before the first wait.
template <typename T, int stage, int fixup>
__device__ __forceinline__ void update_item(const State& base, const State& half,
                                              const State& out, const Geom& G, const Work<T>& W,
                                              const UpdateCfg& U, long long* diag, int vb,
                                              int strips, unsigned long long* slots, int slot) {
  // no fused multiply-adds: the update is memory-bound, and without them its
  // results cannot depend on how a calling kernel is specialised (the main
  // and fix-up calls, the single-box and batched kernels give the same bits)
#pragma clang fp contract(off)
  const int ninter = G.n[0] * G.n[1] * G.n[2];
  const double dt = *W.dt;
  double sigmax = 0.0;
  const bool words = U.fofc && !U.flag_storage;  // a level has none
  // held in vector registers: as scalars the address and the condition no
  // longer fit beside the other pointers, and the compiler then spills them and
  // drains the loads as it goes (stage 2 at 256^3 FP32: 1103 us, like this 924)
  unsigned* word = (words && threadIdx.x == 0) ? item_word(W, vb) : nullptr;
  asm volatile("" : "+v"(word));
  if (fixup && words) {
    const unsigned* w = item_word(W, vb);
    const unsigned long long m = w[0] | ((unsigned long long)w[1] << 32);
    if (m != 0) {  // no first-order value reaches this item
      if (stage == 1 && threadIdx.x == 0) {
        W.nflag[2] = 1;
        atomicMax(&slots[slot], m);
      }
      return;
    }
  }
  for (int strip = 0; strip < strips; ++strip) {
  const int t = (vb * strips + strip) * kBlock + (int)threadIdx.x;
  const bool live = t < ninter;
  int bad = 0;
  double sig = 0.0;
  if (live) {
    const int i0 = t % G.n[0];
    const int q = t / G.n[0];
    const int j0 = q % G.n[1];
    const int k0 = q / G.n[1];
    const int p3[3] = {i0, j0, k0};
    const int s = (i0 + G.g) + G.st[1] * (j0 + G.g) + G.st[2] * (k0 + G.g);
    const bool need_state = (U.fofc && !fixup) || stage == 1;
    double c[5], bl[3];
    // (formed before the stores below, which the compiler cannot move loads across)
    double bu[3] = {0.0, 0.0, 0.0};
    // fix-up: the other cells of an item keep their state; the second stage
    // forms their CFL signal again
    bool write = true;
    if constexpr (fixup) {
      const int g3[3] = {i0 + G.g, j0 + G.g, k0 + G.g};
      write = near_flagged(G, W, U.flag_storage != 0, g3);
    }
    if constexpr (!fixup) {
      cell_form<T, stage, 0>(base, half, G, W, need_state, s, dt, c, bl, bu);
    } else {
      if (write)
        cell_form<T, stage, 1>(base, half, G, W, need_state, s, dt, c, bl, bu);
      else if (stage == 1)
        cell_form<T, stage, 0>(base, half, G, W, need_state, s, dt, c, bl, bu);
    }
    // periodic images: every storage position congruent to this cell
    int mlo[3], mhi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int pos = p3[d] + G.g;
      mlo[d] = -(pos / G.n[d]);
      mhi[d] = (G.N[d] - 1 - pos) / G.n[d];
    }
    if (!write) mhi[2] = mlo[2] - 1;
    for (int mz = mlo[2]; mz <= mhi[2]; ++mz)
      for (int my = mlo[1]; my <= mhi[1]; ++my)
        for (int mx = mlo[0]; mx <= mhi[0]; ++mx) {
          const int sw = s + mx * G.n[0] + my * G.n[1] * G.st[1] + mz * G.n[2] * G.st[2];
#pragma unroll
          for (int m = 0; m < 5; ++m) out.c[m][sw] = c[m];
#pragma unroll
          for (int a = 0; a < 3; ++a) out.b[a][sw] = bl[a];
        }
    if (need_state) {
      const double rho = c[0];
      double u[3], bc[3];
      bool nonfin = false;
#pragma unroll
      for (int m = 0; m < 5; ++m) nonfin |= !__builtin_isfinite(c[m]);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        nonfin |= !__builtin_isfinite(bl[d]) || !__builtin_isfinite(bu[d]);
        bc[d] = 0.5 * (bl[d] + bu[d]);
        u[d] = c[1 + d] / rho;
      }
      const double p = (U.gamma - 1.0) * (c[4] - 0.5 * rho * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) -
                                          0.5 * (bc[0] * bc[0] + bc[1] * bc[1] + bc[2] * bc[2]));
      if (U.fofc && !fixup) {
        if ((U.crit & CTMHD_FLAG_RHO) && !(rho > 0.0)) bad = 1;
        if ((U.crit & CTMHD_FLAG_P) && !(p > 0.0)) bad = 1;
        if ((U.crit & CTMHD_FLAG_NONFINITE) && (nonfin || !__builtin_isfinite(p))) bad = 1;
        if (U.force && U.force[t]) bad = 1;
        W.flag[U.flag_storage ? s : t] = (uint8_t)bad;
      }
      if (stage == 1) sig = cfl_signal(rho, u, p, bc, G, U.gamma, U.sres);
    }
  }
  if (U.fofc && !fixup) {
    unsigned long long m = __ballot(bad);
    if (m) {
      const int lane = threadIdx.x & 63;
      int first = 0;
      if (lane == 0) {
        int cnt = __popcll(m);
        first = atomicAdd(&W.nflag[stage], cnt);
        if (diag) atomicAdd((unsigned long long*)&diag[stage], (unsigned long long)cnt);
      }
      first = __shfl(first, 0, 64);
      if (words && bad) flag_list(W)[first + __popcll(m & ((1ull << lane) - 1))] = t;
    }
  }
  sigmax = (sig > sigmax || sig != sig) ? sig : sigmax;
  }
  unsigned long long most = 1;
  if (stage == 1) {
    if (fixup && threadIdx.x == 0) W.nflag[2] = 1;
    most = block_max_bits(sigmax);
    if (threadIdx.x == 0) atomicMax(&slots[slot], most);
  }
  if (!fixup && word) {
    word[0] = (unsigned)most;
    word[1] = (unsigned)(most >> 32);
  }
}

// Three wavefronts per SIMD: bound by memory, the pass gains nothing from more,
// and loses locality (512^3 FP64, stage 1 / 2: 7.83 / 9.50 ms with three, 8.10 /
// 9.80 with the four and six that the registers allow, 8.08 / 9.16 with two,
// which cost 6% at 128^3).
template <typename T, int stage, int fixup>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 3)))
    k_update(State base, State half, State out, Geom G, Work<T> W, UpdateCfg U, long long* diag,
             int band, Restore R, const int* stop) {
  if (const int at_step = *stop) {
    // the face pass of the step that stopped may have counted fallbacks
    if (stage == 0 && !fixup && diag && gidx() == 0) diag[2] = 0;
    restore_state(R, at_step);
    return;
  }
  if (!fixup) {
    update_item<T, stage, 0>(base, half, out, G, W, U, diag, xcd_band_tile(band), 1, W.smax,
                             blockIdx.x % kMaxSlots);
    return;
  }
  // fix-up: a capped grid strides over the tiles (usually nothing is flagged
  // and every workgroup returns at once)
  if (W.nflag[stage] == 0) return;
  const int ntiles = (G.n[0] * G.n[1] * G.n[2] + kBlock - 1) / kBlock;
  for (int vb = blockIdx.x; vb < ntiles; vb += (int)gridDim.x)
    update_item<T, stage, fixup>(base, half, out, G, W, U, diag, vb, 1, W.smax + kMaxSlots,
                                 blockIdx.x % kMaxSlots);
}

// ---------------------------------------------------------------------------
// First-order flux correction (Sec. 2.5): faces touching a flagged cell take
// the PC + LLF flux of S^n, edges touching one the first-order EMF of S^n.
// ---------------------------------------------------------------------------
// First-order (PC + LLF) flux at the x_a face s; returns s_LLF and u*.
template <typename T>
__device__ __forceinline__ T fo_face(const State& S, const Geom& G, int s, int a, double gamma_d,
                                     T F[5], T& ustar) {
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  T vl[7], vr[7];
  face_local<T>(S, G, s - G.st[a], a, gamma_d, vl);
  face_local<T>(S, G, s, a, gamma_d, vr);
  FState<T> L{vl[0], vl[1], vl[2], vl[3], vl[4], vl[5], vl[6]};
  FState<T> R{vr[0], vr[1], vr[2], vr[3], vr[4], vr[5], vr[6]};
  T Fl[5];
  T sp = llf_flux(L, R, (T)S.b[a][s], (T)gamma_d, Fl);
  F[0] = Fl[0];
  F[1 + a] = Fl[1];
  F[1 + b] = Fl[2];
  F[1 + c] = Fl[3];
  F[4] = Fl[4];
  ustar = (sp * L.un + sp * R.un) / (sp + sp);
  return sp;
}

template <typename T, int EMF>
__device__ __forceinline__ T fo_corner_cell(const State& Sn, const Geom& G, int s, int a, int b,
                                            double gamma, T baY, T bbX) {
  // ideal EMF of a cell (PC): -u_a b_b + u_b b_a, from cell-centred values
  double rho, u[3], p, bc[3];
  cell_prim(Sn, G, s, gamma, rho, u, p, bc);
  if (EMF == kB25A) return -(T)u[a] * (T)bc[b] + (T)u[b] * (T)bc[a];
  return -(T)u[a] * bbX + (T)u[b] * baY;  // FS18 with PC: cell velocity, edge field
}

// One thread per cell position s: its three lower faces and the three edges
// at its lower corner.  Stage 1 writes both stored flux sets so that their RK
// average is the first-order value.
//   periodic box (lvl false): interior positions; the periodic images of the
//     upper boundary faces / edges are written as well (the update reads them);
//   a level of boxes (lvl true): positions 0..n along each axis, so that the
//     upper boundary faces / edges are computed from this box's ghost cells
//     and flags (bitwise the values the neighbour that owns them computes).
template <typename T, int EMF>
__device__ __forceinline__ void fo_at(const State& Sn, const Geom& G, const Work<T>& W, int stage,
                                      double gamma, double eta_d, int t, bool lvl) {
  const int e = lvl ? 1 : 0;
  const int m0 = G.n[0] + e, m1 = G.n[1] + e;
  if (t >= m0 * m1 * (G.n[2] + e)) return;
  const int s3[3] = {t % m0 + G.g, (t / m0) % m1 + G.g, t / (m0 * m1) + G.g};
  const int s = s3[0] + G.st[1] * s3[1] + G.st[2] * s3[2];
  bool up[3];  // on the upper boundary layer along each axis (level only)
#pragma unroll
  for (int d = 0; d < 3; ++d) up[d] = s3[d] == G.g + G.n[d];
  const bool f0 = flag_of(G, W, lvl, s3) != 0;
  for (int a = 0; a < 3; ++a) {
    if (up[(a + 1) % 3] || up[(a + 2) % 3]) continue;  // not a face of this box
    int l3[3] = {s3[0], s3[1], s3[2]};
    l3[a] -= 1;
    if (!f0 && !flag_of(G, W, lvl, l3)) continue;
    T F[5], us;
    fo_face<T>(Sn, G, s, a, gamma, F, us);
    if (eta_d > 0.0) F[4] += joule<T>(Sn, G, s, a, (T)eta_d);
    for (int rep = 0; rep < 2; ++rep) {
      if (rep && (lvl || s3[a] != G.g)) break;
      const int sw = s + (rep ? G.n[a] * G.st[a] : 0);
      for (int m = 0; m < 5; ++m) {
        W.F[stage][a][m][sw] = F[m];
        if (stage == 1) W.F[0][a][m][sw] = F[m];
      }
    }
  }
  for (int c = 0; c < 3; ++c) {
    const int a = (c + 1) % 3, b = (c + 2) % 3;
    if (up[c]) continue;  // not an edge of this box
    int fl = 0;
    for (int q = 0; q < 4; ++q) {
      int p3[3] = {s3[0], s3[1], s3[2]};
      p3[a] -= (q & 1);
      p3[b] -= (q >> 1);
      fl |= flag_of(G, W, lvl, p3);
    }
    if (!fl) continue;
    const int sa = G.st[a], sb = G.st[b];
    T F[5];
    T usaB, usaT, usbL, usbR;
    T apB = fo_face<T>(Sn, G, s - sb, a, gamma, F, usaB);
    T apT = fo_face<T>(Sn, G, s, a, gamma, F, usaT);
    T bpL = fo_face<T>(Sn, G, s - sa, b, gamma, F, usbL);
    T bpR = fo_face<T>(Sn, G, s, b, gamma, F, usbR);
    T baB = (T)Sn.b[a][s - sb], baT = (T)Sn.b[a][s];
    T bbL = (T)Sn.b[b][s - sa], bbR = (T)Sn.b[b][s];
    T e[4];
    if (EMF == kQ26) {
      e[0] = -usaB * bbL + usbL * baB;
      e[1] = -usaB * bbR + usbR * baB;
      e[2] = -usaT * bbL + usbL * baT;
      e[3] = -usaT * bbR + usbR * baT;
    } else {
      // corner XY is the cell on side X along a and side Y along b
      e[0] = fo_corner_cell<T, EMF>(Sn, G, s - sa - sb, a, b, gamma, baB, bbL);
      e[1] = fo_corner_cell<T, EMF>(Sn, G, s - sb, a, b, gamma, baB, bbR);
      e[2] = fo_corner_cell<T, EMF>(Sn, G, s - sa, a, b, gamma, baT, bbL);
      e[3] = fo_corner_cell<T, EMF>(Sn, G, s, a, b, gamma, baT, bbR);
    }
    T aa = tmax(apB, apT), ab = tmax(bpL, bpR);
    T eps = ld04(e[0], e[1], e[2], e[3], aa, aa, ab, ab, baB, baT, bbL, bbR);
    if (eta_d > 0.0) eps += eta_j<T>(Sn, G, s, c, (T)eta_d);
    for (int qa = 0; qa < 2; ++qa)
      for (int qb = 0; qb < 2; ++qb) {
        if ((qa || qb) && lvl) continue;
        if ((qa && s3[a] != G.g) || (qb && s3[b] != G.g)) continue;
        const int sw = s + (qa ? G.n[a] * sa : 0) + (qb ? G.n[b] * sb : 0);
        W.E[stage][c][sw] = eps;
        if (stage == 1) W.E[0][c][sw] = eps;
      }
  }
}

// Work unit q of the first-order pass of a periodic box (item: 256 strips
// cells), of fo_units: neighbour q % 27 of flagged cell q / 27, or cell q when
// many are flagged.  Two units may be the same cell; both write its values.
template <typename T>
__device__ __forceinline__ int fo_units(const Geom& G, const Work<T>& W, int stage) {
  const int nf = W.nflag[stage];
  return few_flagged(G, nf) ? 27 * nf : G.n[0] * G.n[1] * G.n[2];
}
template <typename T, int EMF>
__device__ __forceinline__ void fo_unit(const State& Sn, const Geom& G, const Work<T>& W, int stage,
                                        double gamma, double eta_d, int strips, int q) {
  int t = q;
  if (few_flagged(G, W.nflag[stage])) {
    const int f = flag_list(W)[q / 27], k = q % 27;
    t = interior_id(G, f % G.n[0] + k % 3 - 1 + G.g, f / G.n[0] % G.n[1] + k / 3 % 3 - 1 + G.g,
                    f / (G.n[0] * G.n[1]) + k / 9 - 1 + G.g);
  }
  unsigned* w = item_word(W, t / (kBlock * strips));
  w[0] = w[1] = 0;
  fo_at<T, EMF>(Sn, G, W, stage, gamma, eta_d, t, false);
}

template <typename T, int EMF>
__global__ void __launch_bounds__(kBlock)
    k_fo(State Sn, Geom G, Work<T> W, int stage, double gamma, double eta_d, const int* stop) {
  if (*stop) return;
  if (W.nflag[stage] == 0) return;
  // grid-stride: the launch is capped, so that the usual case (nothing
  // flagged) costs a few workgroups, not one per 256 cells
  const int n = fo_units(G, W, stage);
  for (int q = gidx(); q < n; q += (int)gridDim.x * kBlock)
    fo_unit<T, EMF>(Sn, G, W, stage, gamma, eta_d, 1, q);
}

// ---------------------------------------------------------------------------
// Batched boxes: one persistent launch per step drains a work queue of
// (phase, box, tile) items.  Items are ordered phase-major (largest boxes
// first inside a phase), so an item only ever waits for items that precede
// it in the queue (the previous phase of its own box): with workgroups that
// claim an item only after finishing the last one, the queue always drains.
// Each box is a periodic box of its own (ghosts wrapped per box), or the boxes
// tile one periodic domain (a level of an AMR hierarchy): then the ghost
// layers of every box are filled from the interiors of the boxes that own
// those cells (exchange phases after every update).
// ---------------------------------------------------------------------------
enum : int { PH_F = 0, PH_E, PH_U, PH_O, PH_X, PH_WRAP, PH_DT, PH_COPY, PH_P, PH_XCHG, PH_FIRST };
constexpr int kMaxPhases = 24;

// Exchange phase argument (PlanHeader::xarg): which state to fill, whether
// the invalid-cell flags travel too, and whether it runs only after a fix-up.
enum : int { XG_HALF = 0, XG_NEXT = 1, XG_CUR = 2, XG_TARGET = 3, XG_FLAGS = 4, XG_IF_FIXUP = 8 };

// One block of a box's ghost region whose cells are owned by one box (possibly
// itself, through the periodic wrap): dst and src are packed element indices
// of the block's first element, in the destination box's ghost region and the
// owner's interior.
struct XBlock {
  long long dst, src;
  int dsy, dsz, ssy, ssz;  // strides along axes 1 and 2 of both boxes
  int ex, ey;              // extents along axes 0 and 1 (axis 2: from the volume)
  int vol_lo;              // first ghost index of the block in its box's list
  int vol;                 // elements of the block
};

struct BoxDesc {
  Geom G;
  FacePlan FP;
  long long off;       // element offset of the box in the packed field arrays
  long long flag_off;  // offset of the box in the packed flag array
};

struct PlanHeader {
  int nbox, nphase, strips, magic;
  unsigned long long key;    // hash of the parameters and boxes the plan was built for
  int kind[kMaxPhases];      // PH_*
  int stage[kMaxPhases];     // RK stage of F/E/U/O/X phases
  int item_off[kMaxPhases];  // first queue index of each phase inside its launch
  int range[3][2];           // phase ranges [lo, hi) of the start, step and copy launches
  int range_items[3];        // items of each launch
  long long order_off, prefix_off, desc_off;  // byte offsets of the arrays below
  int xarg[kMaxPhases];      // XG_* of exchange phases
  int level;                 // 1: the boxes tile one periodic domain
  int nxblk;                 // exchange blocks
  long long xbox_off, xblk_off;
  // int order[nbox]; int prefix[nphase][nbox + 1]; BoxDesc desc[nbox];
  // level only: int xbox[nbox + 1] (first block of each box); XBlock xblk[nxblk]
};
constexpr int kPlanMagic = 0x43544d48;

template <typename T>
struct BatchArgs {
  State user, B, H;   // packed states (box offsets from the plan)
  Work<T> W;          // stencil arrays (regrouped by box, shift_work); per-box scalars below
  T* wbase;           // the first of them,
  long long wstride;  // the elements from one to the next
  int narr;           // and their number
  const char* plan;
  int* cursor;        // queue cursor of this launch
  int* done;          // [nphase][nbox] finished items
  int* nflag;         // [nbox][4]: flagged cells stage 0 / 1, stage-1 fix-up ran
  unsigned long long* slots;  // [nbox][2]: CFL maximum (main pass, fix-up)
  double* dt;         // [nbox] (per-box dt) or [1]
  int* stop;
  int* err;           // set when a dependency wait times out
  long long* diag;    // this step's counters or null
  int dt_per_box;
  const int* loc;     // where the current state lives: 0 `user`, 1 B (flipped by each step that
                      // ran; an odd number of steps starts from a copy in B)
  int launch;         // 0 start (wrap + CFL), 1 step, 2 copy-back
  unsigned long long key;  // must equal the plan's key
  unsigned long long tab;  // device address of BoxTab<T>[nbox]
  double gamma, eta;
  int fofc, crit;
  int level;          // the boxes tile one periodic domain
  int want_dt;        // the start of the call forms the CFL maxima
};

// Everything one box needs, with its pointers already shifted to the box:
// built once per batched call by k_btab in the workspace and read through the
// constant address space (uniform scalar loads that may be indexed at run
// time, as kernel arguments are in the single-box kernels).
template <typename T>
struct BoxTab {
  State su, sb, sh;  // the box in the caller's arrays, in B, in H
  Work<T> w;         // its stencil arrays and per-box scalars
  Geom G;
  FacePlan FP;
  double sres;  // resistive term of the CFL maximum
};

__device__ __forceinline__ State shift_state(const State& S, long long off) {
  State R;
#pragma unroll
  for (int m = 0; m < 5; ++m) R.c[m] = S.c[m] + off;
#pragma unroll
  for (int a = 0; a < 3; ++a) R.b[a] = S.b[a] + off;
  return R;
}

// The stencil arrays of one box.  All arrays of a box are stored next to each
// other (array k of the narr at element off narr + k elems, where the box's
// range [off, off + elems) of the packed extent is its own), so that the tens
// of arrays a workgroup touches lie in a few pages; array by array over all
// boxes, a step of 2000 boxes missed the address translation caches on every
// one of them.
template <typename T>
__device__ __forceinline__ Work<T> shift_work(const BatchArgs<T>& A, long long off, int elems) {
  const Work<T>& W0 = A.W;
  Work<T> W = W0;
  // k from the quotient in double, exact after rounding (p is k strides from the
  // base, k in the tens).  With a 64-bit integer division for each of the
  // sixty-odd pointers the table took 26 us for 64 boxes and 35 us for 2000, so 13
  // and 24.
  const double per = 1.0 / (double)A.wstride;
  auto box = [&](T* p) -> T* {
    if (!p) return nullptr;
    const long long k = (long long)(int)((double)(p - A.wbase) * per + 0.5);
    return A.wbase + off * A.narr + k * elems;
  };
#pragma unroll
  for (int v = 0; v < 8; ++v) W.prim[v] = box(W0.prim[v]);
#pragma unroll
  for (int c = 0; c < 3; ++c) W.ecell[c] = box(W0.ecell[c]);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int k = 0; k < 2; ++k) W.b25f[c][o][k] = box(W0.b25f[c][o][k]);
#pragma unroll
  for (int v = 0; v < 3; ++v)
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int k = 0; k < 2; ++k) W.fsf[v][d][k] = box(W0.fsf[v][d][k]);
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int m = 0; m < 5; ++m) W.F[st][a][m] = box(W0.F[st][a][m]);
      W.E[st][a] = box(W0.E[st][a]);
    }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    W.ap[a] = box(W0.ap[a]);
    W.am[a] = box(W0.am[a]);
    W.us[a] = box(W0.us[a]);
  }
  return W;
}

// Wait until *cnt >= need.  Thread 0 polls with relaxed loads (an acquire
// per poll would invalidate the XCD's L2 on every iteration and starve the
// working workgroups), then acquires once.  Bounded by wall-clock time
// (100 MHz counter, about 1 s): on a timeout the error flag is raised and
// every later wait returns at once.
__device__ __forceinline__ void wait_count(const int* cnt, int need, int* err) {
  if (threadIdx.x == 0) {
    const unsigned long long t0 = wall_clock64();
    while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
      if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
      __builtin_amdgcn_s_sleep(8);
      if (wall_clock64() - t0 > 100000000ull) {
        __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
    // the producer may sit on another XCD (another L2): one acquire for the
    // workgroup's CU and XCD caches
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

// Every wave releases its own stores at agent scope before thread 0 counts
// the item as done.
__device__ __forceinline__ void signal_count(int* cnt) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Ghost exchange of a level: element r of box b's ghost region in D takes the
// value of the cell (faces: the lower face of the cell) that owns it in S, for
// all 8 fields and, with `flags`, the invalid-cell flag.  Reads touch only
// interiors and writes only ghost positions, so one launch serves all boxes.
template <typename T>
__device__ __forceinline__ void xchg_at(const BatchArgs<T>& A, const State& S, const State& D,
                                        bool flags, int b, int r) {
  const PlanHeader* P = (const PlanHeader*)A.plan;
  const int* xbox = (const int*)(A.plan + P->xbox_off);
  const XBlock* xb = (const XBlock*)(A.plan + P->xblk_off);
  int k0 = xbox[b], k1 = xbox[b + 1];
  if (k0 >= k1) return;
  const XBlock& lastb = xb[k1 - 1];
  if (r >= lastb.vol_lo + lastb.vol) return;
  while (k1 - k0 > 1) {  // the block holding r: largest k with vol_lo <= r
    const int mid = (k0 + k1) >> 1;
    if (xb[mid].vol_lo <= r) k0 = mid; else k1 = mid;
  }
  const XBlock& B = xb[k0];
  const int l = r - B.vol_lo;
  const int x = l % B.ex, y = (l / B.ex) % B.ey, z = l / (B.ex * B.ey);
  const long long d = B.dst + x + (long long)B.dsy * y + (long long)B.dsz * z;
  const long long s = B.src + x + (long long)B.ssy * y + (long long)B.ssz * z;
#pragma unroll
  for (int m = 0; m < 5; ++m) D.c[m][d] = S.c[m][s];
#pragma unroll
  for (int a = 0; a < 3; ++a) D.b[a][d] = S.b[a][s];
  if (flags) A.W.flag[d] = A.W.flag[s];
}

// Start of a call on a box of a level, interior cell t (the ghost layers of
// dst are filled): its CFL signal (0 for t outside the box, or without
// want_dt) and, when dst is another buffer than src, its copy there.
__device__ __forceinline__ double level_start_at(const State& src, const State& dst, bool copy,
                                                 const Geom& G, double gamma, double sres,
                                                 bool want_dt, int t) {
  const int ninter = G.n[0] * G.n[1] * G.n[2];
  if (t >= ninter) return 0.0;
  const int p3[3] = {t % G.n[0], (t / G.n[0]) % G.n[1], t / (G.n[0] * G.n[1])};
  const int s = p3[0] + G.g + G.st[1] * (p3[1] + G.g) + G.st[2] * (p3[2] + G.g);
  CellRaw R;
#pragma unroll
  for (int m = 0; m < 5; ++m) R.c[m] = src.c[m][s];
#pragma unroll
  for (int d = 0; d < 3; ++d) R.bl[d] = src.b[d][s];
  double v = 0.0;
  if (want_dt) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
      R.bh[d] = (p3[d] == G.n[d] - 1 ? dst.b[d] : src.b[d])[s + G.st[d]];
    double rho, u[3], p, bc[3];
    raw_prim(R, gamma, rho, u, p, bc);
    v = cfl_signal(rho, u, p, bc, G, gamma, sres);
  }
  if (copy) {
#pragma unroll
    for (int m = 0; m < 5; ++m) dst.c[m][s] = R.c[m];
#pragma unroll
    for (int d = 0; d < 3; ++d) dst.b[d][s] = R.bl[d];
  }
  return v;
}

// One work item of a batched step: phase KIND of box b, tile `tile`.
template <typename T, int RECON, int RIEMANN, int EMF, int KIND>
__device__ __forceinline__ void batch_item(const BatchArgs<T>& A, int b, int stage, int tile,
                                           int strips, int cl, int xa) {
  const BoxTab<T>& tb = *(const BoxTab<T>*)((const CTMHD_CONST BoxTab<T>*)A.tab + b);
  const Geom& G = tb.G;
  const State& cur = cl == 0 ? tb.su : tb.sb;
  const Work<T>& W = tb.w;
  const State& Hs = tb.sh;
  const State& in = stage == 0 ? cur : Hs;
  if constexpr (KIND == PH_COPY) {  // the state of this box back into the caller's arrays
    for (int s = 0; s < strips; ++s) {
      const int t = (tile * strips + s) * kBlock + threadIdx.x;
      if (t < G.elems) {
#pragma unroll
        for (int m = 0; m < 5; ++m) tb.su.c[m][t] = tb.sb.c[m][t];
#pragma unroll
        for (int a = 0; a < 3; ++a) tb.su.b[a][t] = tb.sb.b[a][t];
      }
    }
  } else if constexpr (KIND == PH_P) {
    for (int s = 0; s < strips; ++s)
      prim_at<T, EMF>(in, G, W, A.gamma, (tile * strips + s) * kBlock + threadIdx.x);
  } else if constexpr (KIND == PH_FIRST) {
    for (int s = 0; s < strips; ++s)
      first_step_at<T, RECON, EMF>(G, W, (tile * strips + s) * kBlock + threadIdx.x);
  } else if constexpr (KIND == PH_F) {
    int nfb = 0;
    faces_block<T, RECON, RIEMANN>(in, G, W, tb.FP, tile, stage, A.gamma, A.eta, nfb);
    if (A.diag && nfb) atomicAdd((unsigned long long*)&A.diag[2], (unsigned long long)nfb);
  } else if constexpr (KIND == PH_E) {
    for (int s = 0; s < strips; ++s)
      emf_at<T, RECON, EMF, 0, 3>(in, G, W, stage, A.eta, (tile * strips + s) * kBlock + threadIdx.x);
  } else if constexpr (KIND == PH_U || KIND == PH_X) {
    const State& oth = cl == 0 ? tb.sb : tb.su;
    UpdateCfg U;
    U.fofc = A.fofc;
    U.crit = A.crit;
    U.gamma = A.gamma;
    U.sres = tb.sres;
    U.force = nullptr;
    U.flag_storage = A.level;
    constexpr int fix = KIND == PH_X ? 1 : 0;
    if (stage == 0)
      update_item<T, 0, fix>(cur, Hs, Hs, G, W, U, A.diag, tile, strips, W.smax, fix);
    else
      update_item<T, 1, fix>(cur, Hs, oth, G, W, U, A.diag, tile, strips, W.smax, fix);
  } else if constexpr (KIND == PH_O) {
    const int n = A.level ? 0 : fo_units(G, W, stage);
    for (int s = 0; s < strips; ++s) {
      const int q = (tile * strips + s) * kBlock + threadIdx.x;
      if (A.level)
        fo_at<T, EMF>(cur, G, W, stage, A.gamma, A.eta, q, true);
      else if (q < n)
        fo_unit<T, EMF>(cur, G, W, stage, A.gamma, A.eta, strips, q);
    }
  } else if constexpr (KIND == PH_WRAP) {
    double sig = 0.0;
    for (int s = 0; s < strips; ++s) {
      const double v = start_at(tb.su, cur, cl != 0, G, A.gamma, tb.sres, A.want_dt != 0,
                                (tile * strips + s) * kBlock + threadIdx.x);
      sig = (v > sig || v != v) ? v : sig;
    }
    if (A.want_dt) block_max_to_slots(sig, W.smax, 0);
  } else if constexpr (KIND == PH_XCHG) {
    const int tg = xa & XG_TARGET;
    // packed (unshifted) arrays: the owner of a ghost block is another box;
    // the caller's state goes to the buffer that the first step starts from
    const State& dst = tg == XG_HALF ? A.H : tg == XG_CUR ? (cl == 0 ? A.user : A.B)
                                                            : (cl == 0 ? A.B : A.user);
    const State& src = tg == XG_CUR ? A.user : dst;
    for (int s = 0; s < strips; ++s)
      xchg_at(A, src, dst, (xa & XG_FLAGS) != 0, b, (tile * strips + s) * kBlock + threadIdx.x);
  } else if constexpr (KIND == PH_DT) {
    double sig = 0.0;
    for (int s = 0; s < strips; ++s) {
      const double v = level_start_at(tb.su, cur, cl != 0, G, A.gamma, tb.sres, A.want_dt != 0,
                                      (tile * strips + s) * kBlock + threadIdx.x);
      sig = (v > sig || v != v) ? v : sig;
    }
    if (A.want_dt) block_max_to_slots(sig, W.smax, 0);
  }
}

// Per-box tables of a batched call (one thread per box).
template <typename T>
__global__ void __launch_bounds__(kBlock) k_btab(BatchArgs<T> A, int nbox) {
  const PlanHeader* P = (const PlanHeader*)A.plan;
  if (P->magic != kPlanMagic || P->key != A.key) return;  // refused by the step kernels
  const int b = blockIdx.x * kBlock + threadIdx.x;
  if (b >= nbox) return;
  const BoxDesc& d = ((const BoxDesc*)(A.plan + P->desc_off))[b];
  BoxTab<T>* tb = (BoxTab<T>*)A.tab + b;
  tb->su = shift_state(A.user, d.off);
  tb->sb = shift_state(A.B, d.off);
  tb->sh = shift_state(A.H, d.off);
  Work<T> W = shift_work(A, d.off, d.G.elems);
  W.flag = A.W.flag + d.flag_off;
  W.dt = A.dt + (A.dt_per_box ? b : 0);
  W.nflag = A.nflag + (A.level ? 0 : 4 * b);  // a level flags and fixes up as one domain
  W.smax = A.slots + 2 * b;
  W.stop = A.stop;
  tb->w = W;
  tb->G = d.G;
  tb->FP = d.FP;
  // from the call's eta: one plan serves calls of any eta
  const double dxmin = fmin(d.G.dx[0], fmin(d.G.dx[1], d.G.dx[2]));
  tb->sres = A.eta > 0.0 ? 2.0 * A.eta / (dxmin * dxmin) : 0.0;
}

// Flag counters of box b.
template <typename T>
__device__ __forceinline__ const int* tab_nflag(const BatchArgs<T>& A, int b) {
  return A.nflag + (A.level ? 0 : 4 * b);
}

// Plan lookup shared by both schedules: true if the plan was built for the
// call's parameters and boxes.
__device__ __forceinline__ bool plan_ok(const PlanHeader* P, unsigned long long key, int* err) {
  if (P->magic == kPlanMagic && P->key == key) return true;
  if (threadIdx.x == 0) atomicOr(err, 2);
  return false;
}

// Box (index into `order`, largest k with pre[k] <= r) of item r of a phase.
__device__ __forceinline__ int item_box(const int* pre, int nbox, int r) {
  int k0 = 0, k1 = nbox;
  while (k1 - k0 > 1) {
    int mid = (k0 + k1) >> 1;
    if (pre[mid] <= r) k0 = mid; else k1 = mid;
  }
  return k0;
}

// Persistent schedule: one launch per step (plus a start and a copy-back
// launch).  Workgroups claim queue items in phase-major order; an item waits
// only for all items of the previous phase of its own box.
template <typename T, int RECON, int RIEMANN, int EMF>
__global__ void __launch_bounds__(kBlock) k_batch(BatchArgs<T> A) {
  if (*A.stop && A.launch != 2) return;  // the copy-back runs even after a stop
  const PlanHeader* P = (const PlanHeader*)A.plan;
  if (!plan_ok(P, A.key, A.err)) return;
  const int* order = (const int*)(A.plan + P->order_off);
  const int* prefix = (const int*)(A.plan + P->prefix_off);
  const int nbox = P->nbox;
  const int lo = P->range[A.launch][0], hi = P->range[A.launch][1];
  const int total = P->range_items[A.launch];
  const int strips = P->strips;
  const int cl = *A.loc;  // fixed for the whole launch
  __shared__ int item_s;
  for (;;) {
    if (threadIdx.x == 0) item_s = atomicAdd(A.cursor, 1);
    __syncthreads();
    const int q = item_s;
    __syncthreads();
    if (q >= total) break;
    int p = lo;
    while (p + 1 < hi && P->item_off[p + 1] <= q) ++p;
    const int* pre = prefix + (long long)p * (nbox + 1);
    const int r = q - P->item_off[p];
    const int k0 = item_box(pre, nbox, r);
    const int b = order[k0];
    const int tile = r - pre[k0];
    if (p > lo) {
      const int* ppre = prefix + (long long)(p - 1) * (nbox + 1);
      wait_count(A.done + (long long)(p - 1) * nbox + b, ppre[k0 + 1] - ppre[k0], A.err);
    }
    const int kind = P->kind[p], stage = P->stage[p];
    switch (kind) {
      case PH_P: batch_item<T, RECON, RIEMANN, EMF, PH_P>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_FIRST: batch_item<T, RECON, RIEMANN, EMF, PH_FIRST>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_F: batch_item<T, RECON, RIEMANN, EMF, PH_F>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_E: batch_item<T, RECON, RIEMANN, EMF, PH_E>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_U: batch_item<T, RECON, RIEMANN, EMF, PH_U>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_X: if (tab_nflag(A, b)[stage]) batch_item<T, RECON, RIEMANN, EMF, PH_X>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_O: if (tab_nflag(A, b)[stage]) batch_item<T, RECON, RIEMANN, EMF, PH_O>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_WRAP: batch_item<T, RECON, RIEMANN, EMF, PH_WRAP>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_DT: batch_item<T, RECON, RIEMANN, EMF, PH_DT>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      case PH_XCHG: if (!(P->xarg[p] & XG_IF_FIXUP) || tab_nflag(A, b)[stage]) batch_item<T, RECON, RIEMANN, EMF, PH_XCHG>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
      default: batch_item<T, RECON, RIEMANN, EMF, PH_COPY>(A, b, stage, tile, strips, cl, P->xarg[p]); break;
    }
    signal_count(A.done + (long long)p * nbox + b);
  }
}

// Consecutive items per XCD (k_bphase).  Step with bands of 8 / 64 / 256 items
// and without: 2000 uneven boxes, FP32 31.2 / 30.1 / 29.8 / 31.5 ms, FP64 38.6 /
// 37.8 / 37.4 / 40.0; 300 boxes, FP64 5.48 / 5.37 / 5.39 / 5.50; a level of 64
// boxes of 32^3 1.91 / 1.89 / 1.90 / 1.94 ms.  Below about 60 boxes a few bands
// hold all items and share the XCDs out unevenly: 40 boxes, FP64, 0.78 / 0.84 /
// 0.78 / 0.79 ms.
constexpr int kBatchBand = 64;

// The lookup of an item's box reads the plan as constant memory (nothing writes
// it while a kernel runs): the binary search is a chain of scalar loads.
template <typename P>
__device__ __forceinline__ const P* as_const(const char* p) {
  return (const P*)(const CTMHD_CONST P*)(unsigned long long)(uintptr_t)p;
}

// Phased schedule: one launch per phase over all boxes, one workgroup per item
// of phase p, in bands of 64 consecutive items per XCD, so that the rows and
// planes that the tiles of a box share meet in one L2.  Launch boundaries
// order the phases.  2000 boxes, FP32, per launch: edge pass 2.90 -> 2.45 ms,
// update 4.56 -> 4.00 ms with the scalar lookup and the bands, 3.90 with the
// arrays of a box next to each other (shift_work); face pass 7.33 -> 7.14 ms.
template <typename T, int RECON, int RIEMANN, int EMF, int KIND>
__global__ void __launch_bounds__(kBlock) k_bphase(BatchArgs<T> A, int p) {
  if (*A.stop) return;
  const PlanHeader* P = as_const<PlanHeader>(A.plan);
  if (!plan_ok(P, A.key, A.err)) return;
  const int nbox = P->nbox;
  const int* pre = as_const<int>(A.plan + P->prefix_off) + (long long)p * (nbox + 1);
  const int r = xcd_band_tile(kBatchBand);
  if (r >= pre[nbox]) return;
  const int k0 = item_box(pre, nbox, r);
  const int b = as_const<int>(A.plan + P->order_off)[k0];
  batch_item<T, RECON, RIEMANN, EMF, KIND>(A, b, P->stage[p], r - pre[k0], P->strips, *A.loc,
                                           P->xarg[p]);
}

// A phase that most boxes have no work in (the first-order pass, the fix-up,
// a level's exchange after it and the copy-back of a stopped call): a grid of a few workgroups per CU
// looks for the boxes that have some, 256 at a time, and shares their tiles
// out.  With one workgroup per tile of every box, four such launches that
// found nothing took 1.7 ms of a step of 2000 boxes (2 x 430 + 2 x 370 us).
template <typename T, int EMF, int KIND>
__global__ void __launch_bounds__(kBlock) k_bsparse(BatchArgs<T> A, int p) {
  if (KIND == PH_COPY ? *A.loc == 0 : *A.stop != 0) return;  // a copy-back follows a stop
  const PlanHeader* P = (const PlanHeader*)A.plan;
  if (!plan_ok(P, A.key, A.err)) return;
  const int nbox = P->nbox, stage = P->stage[p];
  const int* pre = (const int*)(A.plan + P->prefix_off) + (long long)p * (nbox + 1);
  const int* order = (const int*)(A.plan + P->order_off);
  __shared__ unsigned long long found[kBlock / 64];
  int shift = 0;  // tiles of the boxes before, so that the next box starts on other workgroups
  for (int k0 = 0; k0 < nbox; k0 += kBlock) {
    const int k = k0 + (int)threadIdx.x;
    const bool has =
        k < nbox && (KIND == PH_COPY || tab_nflag(A, order[k])[stage] != 0);
    const unsigned long long bits = __ballot(has);
    if ((threadIdx.x & 63) == 0) found[threadIdx.x >> 6] = bits;
    __syncthreads();
    for (int w = 0; w < kBlock / 64; ++w) {
      unsigned long long f = found[w];
      while (f) {
        const int q = k0 + 64 * w + __ffsll((unsigned long long)f) - 1;
        f &= f - 1;
        const int cnt = pre[q + 1] - pre[q], grid = (int)gridDim.x;
        int tile = ((int)blockIdx.x - shift) % grid;
        if (tile < 0) tile += grid;
        for (; tile < cnt; tile += grid)
          batch_item<T, kPC, kHLLD, EMF, KIND>(A, order[q], stage, tile, P->strips, *A.loc,
                                               P->xarg[p]);
        shift = (shift + cnt) % grid;
      }
    }
    __syncthreads();
  }
}

// Reset before a launch of the queue (start / copy launches); init = 1 at the
// start of a call also clears the stop / error flags, the state location and
// the per-box CFL slots.
__global__ void k_breset(int nbox, int nphase, int* done, int* cursor, int init, int* stop,
                         int* err, int* loc, int loc0, unsigned long long* slots, int* nflag) {
  for (int i = threadIdx.x; i < nphase * nbox; i += kBlock) done[i] = 0;
  if (threadIdx.x < 4) cursor[threadIdx.x] = 0;
  if (!init) return;
  for (int b = threadIdx.x; b < nbox; b += kBlock) {
    slots[2 * b] = slots[2 * b + 1] = 0ull;
    nflag[4 * b] = nflag[4 * b + 1] = nflag[4 * b + 2] = nflag[4 * b + 3] = 0;
  }
  if (threadIdx.x == 0) {
    *stop = 0;
    *err = 0;
    *loc = loc0;
  }
}

// After a batched step: the new state is in the other buffer unless the step
// was stopped (non-finite dt), which leaves it where it was.
__global__ void k_bstep_end(int* loc, const int* stop, const int* err, long long* diag) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  if (diag) diag[3] |= *err << 1;
  if (!*stop) *loc ^= 1;
}

}  // namespace
