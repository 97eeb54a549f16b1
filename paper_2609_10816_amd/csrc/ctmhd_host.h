// ctmhd_host.h -- host-side helpers of libctmhd shared by its translation
// units: error reporting, argument checks, workspace carving, launches.
#pragma once

#include "ctmhd_device.h"

// one error message per host thread, shared by all entry points
extern thread_local char g_err[256];
// kernel timing hook (ctmhd_profile_events)
extern void* const* g_prof_events;
extern int g_prof_pairs;
extern int g_prof_used;

namespace {

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// Bytes of the stencil type of a precision form: float32 for both FP32 forms.
inline size_t stencil_bytes(const ctmhd_params* p) { return p->precision == CTMHD_FP64 ? 8 : 4; }

int fail(int code, const char* msg) {
  snprintf(g_err, sizeof(g_err), "%s", msg);
  return code;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Tuning knobs in ctmhd_params.tile: bits 0-7 minimum faces per marching
// chunk (0: automatic, up to 32), bits 8-15 256-element strips per batched
// work item (default 1), bit 16 batched schedule (0 per phase, 1 persistent),
// bits 19-20 XCD mapping, bits 21-22 Q26 edge kernel, bits 24-30 x-face items
// per wavefront (0: automatic, up to 4).
int tile_chunk(const ctmhd_params* p) {
  return p->tile & 0xff;
}
int tile_strips(const ctmhd_params* p) {
  int s = (p->tile >> 8) & 0xff;
  return s > 0 ? s : 1;
}
// bit 16: batched schedule, 0 one launch per phase, 1 persistent queue
int tile_sched(const ctmhd_params* p) { return (p->tile >> 16) & 1; }
// bits 19-20: XCD mapping of the edge and update passes of the single-box
// call: 0 automatic, 1 each XCD a contiguous range of tiles, 2 all XCDs on
// bands of the same plane
int tile_xcd_map(const ctmhd_params* p) { return (p->tile >> 19) & 3; }
// bits 21-22: Q26 edge kernel of the single-box call: 0 automatic, 1 one
// thread per edge position, 2 z marches (the same values)
int tile_emf(const ctmhd_params* p) { return (p->tile >> 21) & 3; }

// Tiles per XCD and chunk of the banded mapping (0: the contiguous mapping)
// for a pass whose tiles of kBlock positions run over planes of
// `plane_positions` positions.
int xcd_band(const ctmhd_params* p, long long plane_positions, long long total_positions) {
  int m = tile_xcd_map(p);
  // automatic: banded once a plane holds 2^15 positions (measured: +6-9% on
  // the step at 512^3, +2% at 256^3, neutral at 128^3)
  if (m == 0) m = plane_positions >= (1LL << 15) ? 2 : 1;
  if (m == 1) return 0;
  (void)total_positions;
  const long long tiles = (plane_positions + kBlock - 1) / kBlock;
  const long long band = (tiles + kXcds - 1) / kXcds;
  return band < 1 ? 1 : (int)band;
}

// bits 24-30: x-face items (runs of 64 cells) per wavefront (0: automatic)
int tile_xrows(const ctmhd_params* p) { return (p->tile >> 24) & 0x7f; }

int check_params(const ctmhd_params* p) {
  if (!p) return fail(CTMHD_EARG, "params is NULL");
  if (!(p->gamma > 1.0)) return fail(CTMHD_EARG, "gamma must be > 1");
  if (!(p->eta >= 0.0)) return fail(CTMHD_EARG, "eta must be >= 0");
  if (!(p->cfl > 0.0 && p->cfl < 1.0)) return fail(CTMHD_EARG, "cfl must be in (0, 1)");
  if (p->eta > 0.0 && !(p->cfl < 1.0 / 3.0))
    return fail(CTMHD_EARG, "cfl must be < 1/3 with eta > 0 (3D diffusive limit)");
  if (p->recon < 0 || p->recon > 3) return fail(CTMHD_EARG, "unknown reconstruction");
  if (p->riemann < 0 || p->riemann > 1) return fail(CTMHD_EARG, "unknown Riemann solver");
  if (p->emf_compute < 0 || p->emf_compute > 2) return fail(CTMHD_EARG, "unknown EMF scheme");
  if (p->emf_average != CTMHD_AVG_LD04) return fail(CTMHD_EUNSUPPORTED, "only LD04 averaging is built");
  if (p->precision != CTMHD_FP64 && p->precision != CTMHD_FP32 && p->precision != CTMHD_FP32_R64)
    return fail(CTMHD_EARG, "unknown precision");
  if (p->tile < 0 || (p->tile & ~0x7f79ffff) != 0 || ((p->tile >> 19) & 3) == 3 ||
      ((p->tile >> 21) & 3) == 3)
    return fail(CTMHD_EARG, "tile knob out of range");
  return CTMHD_OK;
}

int check_box(const ctmhd_params* p, const ctmhd_box* b) {
  if (!b) return fail(CTMHD_EARG, "box is NULL");
  for (int d = 0; d < 3; ++d) {
    if (b->n[d] < 1) return fail(CTMHD_EARG, "box dimensions must be >= 1");
    if (!(b->dx[d] > 0.0)) return fail(CTMHD_EARG, "dx must be > 0");
  }
  if (b->ng < recon_halfwidth(p->recon) + 2) return fail(CTMHD_EARG, "too few ghost layers");
  long long e = 1;
  for (int d = 0; d < 3; ++d) e *= (long long)(b->n[d] + 2 * b->ng);
  if (e * 6 >= (1LL << 31)) return fail(CTMHD_EARG, "box too large for 32-bit indexing");
  return CTMHD_OK;
}

// Workspace of one box for the stencil type of `tbytes` bytes.
size_t box_ws_bytes(const ctmhd_box& b, size_t tbytes, const ctmhd_params* p) {
  const int emf = p->emf_compute;
  size_t e = 1;
  for (int d = 0; d < 3; ++d) e *= (size_t)(b.n[d] + 2 * b.ng);
  size_t ninter = (size_t)b.n[0] * b.n[1] * b.n[2];
  size_t bytes = 0;
  bytes += 2 * 8 * align256(e * 8);           // two state buffers
  if (emf == CTMHD_EMF_B25A) bytes += 3 * align256(e * tbytes);  // cell EMF
  if (first_step_stored(emf, p->recon))     // stored first steps
    bytes += (emf == CTMHD_EMF_B25A ? 12 : 18) * align256(e * tbytes);
  if (emf == CTMHD_EMF_FS18) bytes += 3 * align256(e * tbytes);  // cell velocity
  bytes += 2 * 15 * align256(e * tbytes);     // fluxes, two stages
  bytes += 9 * align256(e * tbytes);          // alpha+, alpha-, u*
  bytes += 6 * align256(e * tbytes);          // EMFs, two stages
  bytes += align256(ninter);                  // flags
  bytes += align256(2 * kMaxSlots * 8) + 256; // CFL slots + scalars
  return bytes;
}

struct Carve {
  char* p;
  template <typename U>
  U* take(size_t n) {
    U* r = (U*)p;
    p += align256(n * sizeof(U));
    return r;
  }
};

template <typename T>
int build_work(const ctmhd_params* prm, void* ws, size_t ws_bytes, const ctmhd_box& b, Work<T>& W,
               State& A2, State& H) {
  size_t need = box_ws_bytes(b, sizeof(T), prm);
  if (!ws || ws_bytes < need) return fail(CTMHD_EARG, "workspace too small");
  if (((uintptr_t)ws & 255) != 0) return fail(CTMHD_EARG, "workspace must be 256-byte aligned");
  size_t e = 1;
  for (int d = 0; d < 3; ++d) e *= (size_t)(b.n[d] + 2 * b.ng);
  size_t ninter = (size_t)b.n[0] * b.n[1] * b.n[2];
  Carve cv{(char*)ws};
  for (int m = 0; m < 5; ++m) A2.c[m] = cv.take<double>(e);
  for (int a = 0; a < 3; ++a) A2.b[a] = cv.take<double>(e);
  for (int m = 0; m < 5; ++m) H.c[m] = cv.take<double>(e);
  for (int a = 0; a < 3; ++a) H.b[a] = cv.take<double>(e);
  for (int v = 0; v < 8; ++v) W.prim[v] = nullptr;
  for (int c = 0; c < 3; ++c) W.ecell[c] = nullptr;
  for (int c = 0; c < 3; ++c)
    for (int o = 0; o < 2; ++o) W.b25f[c][o][0] = W.b25f[c][o][1] = nullptr;
  for (int v = 0; v < 3; ++v)
    for (int d = 0; d < 3; ++d) W.fsf[v][d][0] = W.fsf[v][d][1] = nullptr;
  const bool first = first_step_stored(prm->emf_compute, prm->recon);
  if (prm->emf_compute == CTMHD_EMF_B25A) {
    for (int c = 0; c < 3; ++c) W.ecell[c] = cv.take<T>(e);
    if (first)
      for (int c = 0; c < 3; ++c)
        for (int o = 0; o < 2; ++o)
          for (int k = 0; k < 2; ++k) W.b25f[c][o][k] = cv.take<T>(e);
  }
  if (prm->emf_compute == CTMHD_EMF_FS18) {
    for (int v = 1; v < 4; ++v) W.prim[v] = cv.take<T>(e);
    if (first)
      for (int v = 0; v < 3; ++v)
        for (int d = 0; d < 3; ++d)
          for (int k = 0; k < 2; ++k) W.fsf[v][d][k] = cv.take<T>(e);
  }
  for (int st = 0; st < 2; ++st)
    for (int a = 0; a < 3; ++a)
      for (int m = 0; m < 5; ++m) W.F[st][a][m] = cv.take<T>(e);
  for (int a = 0; a < 3; ++a) W.ap[a] = cv.take<T>(e);
  for (int a = 0; a < 3; ++a) W.am[a] = cv.take<T>(e);
  for (int a = 0; a < 3; ++a) W.us[a] = cv.take<T>(e);
  for (int st = 0; st < 2; ++st)
    for (int c = 0; c < 3; ++c) W.E[st][c] = cv.take<T>(e);
  W.flag = cv.take<uint8_t>(ninter);
  W.smax = cv.take<unsigned long long>(2 * kMaxSlots);
  char* sc = cv.p;
  W.dt = (double*)sc;
  W.stop = (int*)(sc + 8);
  W.nflag = (int*)(sc + 16);
  return CTMHD_OK;
}


inline void prof_begin(hipStream_t st) {
  if (g_prof_events && g_prof_used < g_prof_pairs)
    (void)hipEventRecord((hipEvent_t)g_prof_events[2 * g_prof_used], st);
}
inline void prof_end(hipStream_t st) {
  if (g_prof_events && g_prof_used < g_prof_pairs) {
    (void)hipEventRecord((hipEvent_t)g_prof_events[2 * g_prof_used + 1], st);
    ++g_prof_used;
  }
}

#define LAUNCH(kern, blocks, ...)                                                  \
  do {                                                                             \
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBlock), 0, st, __VA_ARGS__);      \
    if (hipGetLastError() != hipSuccess) return fail(CTMHD_EHIP, "kernel launch failed: " #kern); \
  } while (0)

// Workgroups of the first-order, fix-up and copy-back launches, which stride
// over the box: enough to fill the chip when there is work, few enough that
// the usual launch that finds none costs microseconds.
inline int fix_blocks(int ninter) {
  const int nb = nblocks(ninter);
  return nb < 2048 ? nb : 2048;
}

// The update of one stage: main pass (fixup 0) or fix-up.  Each form is a
// kernel of its own, so that none carries the registers of the others.
template <typename T, int fixup>
int launch_update(hipStream_t st, int blocks, State base, State half, State out, const Geom& G,
                  const Work<T>& W, int stage, const UpdateCfg& U, long long* diag, int band,
                  const Restore& R = Restore{}) {
  if (stage == 0)
    LAUNCH((k_update<T, 0, fixup>), blocks, base, half, out, G, W, U, diag, band, R, W.stop);
  else
    LAUNCH((k_update<T, 1, fixup>), blocks, base, half, out, G, W, U, diag, band, R, W.stop);
  return CTMHD_OK;
}

// Partial CFL maxima of k_start: in the edge EMFs, which are not yet in use.
template <typename T>
unsigned long long* start_part(const Work<T>& W) {
  return (unsigned long long*)W.E[0][0];
}

// The start of a call on one box: the caller's state `user` with its ghost
// layers into A (copy: another buffer) and npart partial CFL maxima.
template <typename T>
int launch_start(hipStream_t st, const ctmhd_params* p, State user, State A, bool copy,
                 const Geom& G, const Work<T>& W, bool want_dt, double sres, long long* diag,
                 int ndiag, int& npart) {
  npart = fix_blocks(G.elems);
  LAUNCH(k_start, npart, user, A, copy ? 1 : 0, G, p->gamma, sres, want_dt ? 1 : 0, start_part(W),
         diag, ndiag, W.stop);
  return CTMHD_OK;
}

// The dt of step n of a call: given (dt_fixed) or from the CFL maximum.
template <typename T>
DtStep make_dt_step(const ctmhd_params* p, const Work<T>& W, int npart, int n,
                    const double* dt_fixed, double* dt_out, long long* diag) {
  return DtStep{W.smax, start_part(W), npart, n, W.nflag, p->cfl, dt_fixed, W.dt, dt_out, W.stop,
                diag};
}

// Launch shape of the face pass when the tile knob leaves it open, from the
// faces of the two marching directions of all boxes of a call: chunks of 32
// faces once they make kFaceWaves wavefronts, shorter ones on smaller calls,
// down to one face.  A call of many boxes, whose marches are of uneven length,
// takes at most 16.  A chunk is a serial chain of one Riemann solve (about 2 us)
// per face and 2r + 1 cheaper cells to fill its pipeline.  Measured per step,
// FP64 PPM: 16^3 94 us with chunks of 1, 112 with 4, 183 with 32; 64^3 267 / 220 /
// 216 / 241 / 329 us with 1 / 4 / 8 / 16 / 32; 128^3 1259 / 1194 / 1165 / 1155 us
// with 4 / 8 / 16 / 32; uneven boxes with 4 / 8 / 16 / 64: 2000 in FP32 29.6 / 29.7 /
// 30.1 / 31.2 ms, in FP64 39.1 / 38.1 / 37.6 / 37.5, 500 in FP32 7.18 / 7.30 / 7.40 /
// 7.88, in FP64 9.76 / 9.69 / 9.68 / 10.17 (the plan, which holds the chunk,
// serves every precision).
constexpr int kFaceWaves = 1024;
int auto_face_chunk(long long faces, int nbox) {
  const long long c = faces / (64LL * kFaceWaves);
  const long long most = nbox == 1 ? 32 : 16;
  return c < 1 ? 1 : (c > most ? (int)most : (int)c);
}
// Items per wavefront of the x part, one to four: 16^3 108 us with 4 against
// 94 with 1, 64^3 230 against 216; 128^3 1153 against 1172.
int auto_face_xrows(long long faces) {
  const long long x = faces / (4 * 64LL * kFaceWaves);
  return x < 1 ? 1 : (x > 4 ? 4 : (int)x);
}

// Faces of the two marching directions of one box.
long long march_faces(const ctmhd_box& b, int recon, int emf, bool periodic) {
  const int s = emf == CTMHD_EMF_Q26 ? recon_halfwidth(recon) : 0;
  const long long t = periodic ? 0 : 2 + 2 * s, e = periodic ? 0 : 1;
  return (b.n[0] + t) * ((b.n[1] + e) * (b.n[2] + t) + (b.n[2] + e) * (b.n[1] + t));
}

// Bricks of the face pass: boxes whose state is larger than kBrickFrom are cut
// into bricks of about kBrickBytes, so that the three parts of a brick read it
// from the 256 MB Infinity Cache after the first.  Measured per launch, without
// and with: FP32 PPM 160^3 (0.3 GB) 396 / 404 us, 200^3 814 / 742, 256^3 1601 /
// 1354, 384^3 5264 / 4670; FP64 PLM 256^3 1947 / 1755; FP64 PC 384^3 6143 /
// 5580; FP64 PPM LLF 200^3 989 / 826, 256^3 1925 / 1528; FP32 with the FP64
// Riemann solve, HLLD, PLM 200^3 774 / 718, 256^3 1551 / 1389, PPM 200^3 826 /
// 845, 256^3 1656 / 1619, 320^3 3217 / 3052 (the step: 2562 / 2601 at 184^3, 4063
// / 4066 at 216^3, 4922 / 4822 at 232^3).  FP64 PPM with HLLD is held up by its
// arithmetic instead (256^3 2088 / 2082, 512^3 16.40 / 16.50 ms), and keeps one
// brick, whose long marches all start first.
constexpr long long kBrickFrom = 384LL << 20, kBrickBytes = 64LL << 20;
// Face plan: ranges and launch shape of the fused face kernel.  What the tile
// knob leaves open is chosen from `faces`, march_faces summed over the nbox
// boxes of the call.
// (bricks: the box may be cut.  The plan of a batch serves every precision and
// solver, so it does not depend on them: its boxes stay whole.)
FacePlan make_face_plan(const Geom& G, const ctmhd_params* p, bool periodic, long long faces,
                        int nbox, bool bricks) {
  const int emf = p->emf_compute;
  int chunk_min = tile_chunk(p), xrows = tile_xrows(p);
  if (chunk_min <= 0) chunk_min = auto_face_chunk(faces, nbox);
  if (xrows <= 0) xrows = auto_face_xrows(faces);
  FacePlan P;
  const int r = recon_halfwidth(p->recon);
  const int g = G.g;
  // Q26 reconstructs u* along the transverse axes to the edges, which needs
  // faces r+1 beyond the edge range [g, g+n]; the other schemes only need
  // alpha on the faces next to the edges.
  const int shell = emf == CTMHD_EMF_Q26 ? r : 0;
  P.per = periodic ? 1 : 0;
  P.plo = g - 1 - shell;
  P.tlo = periodic ? g : P.plo;
  for (int d = 0; d < 3; ++d) {
    P.phi[d] = g + G.n[d] + shell;
    P.lo[d] = g;
    // faces g .. g+n are read by the update and the edges; face g+n of a
    // periodic box is a copy of face g
    P.nf[d] = G.n[d] + (periodic ? 0 : 1);
    P.tlen[d] = periodic ? G.n[d] : P.phi[d] - P.plo + 1;
    P.ulo[d] = g;
    P.ulen[d] = G.n[d];
  }
  // marches: enough chunks for ~8192 waves in flight
  int nchunk[3] = {0, 0, 0};
  for (int A = 1; A <= 2; ++A) {
    const int C = A == 1 ? 2 : 1;
    const int lblocks = (P.tlen[0] * P.tlen[C] + kBlock - 1) / kBlock;
    int want = (8192 * 64 / kBlock) / (lblocks > 0 ? lblocks : 1);
    int maxch = (P.nf[A] + chunk_min - 1) / chunk_min;  // chunk >= chunk_min faces (warm-up 2r+1)
    if (want > maxch) want = maxch;
    if (want < 1) want = 1;
    P.chunk[A] = (P.nf[A] + want - 1) / want;
    nchunk[A] = (P.nf[A] + P.chunk[A] - 1) / P.chunk[A];
  }
  P.chunk[0] = P.lanes[0] = P.blocks[0] = 0;
  // bricks
  P.nby = P.nbz = 1;
  const long long bytes = 64LL * G.elems;
  if (bytes > kBrickFrom && bricks) {
    P.nbz = nchunk[2];
    const long long slab = bytes / P.nbz;
    P.nby = (int)((slab + kBrickBytes - 1) / kBrickBytes);
    if (P.nby > nchunk[1]) P.nby = nchunk[1];
    if (P.nby < 1) P.nby = 1;
  }
  P.wy = (P.tlen[1] + P.nby - 1) / P.nby;
  P.wz = (P.tlen[2] + P.nbz - 1) / P.nbz;
  P.cy = (nchunk[1] + P.nby - 1) / P.nby;
  P.cz = (nchunk[2] + P.nbz - 1) / P.nbz;
  P.lanes[1] = P.tlen[0] * P.wz;
  P.lanes[2] = P.tlen[0] * P.wy;
  P.blocks[1] = (P.lanes[1] + kBlock - 1) / kBlock * P.cy;
  P.blocks[2] = (P.lanes[2] + kBlock - 1) / kBlock * P.cz;
  // x part of a brick
  const int xstep = 64 - 2 * r - 1;
  P.xw = P.nf[0] + 2 * r + 1;
  P.xlen = P.xw * P.wy * P.wz;
  P.xwaves = (P.xlen - 2 * r - 1 + xstep - 1) / xstep;
  P.xdx = xstep % P.xw;
  P.xdy = xstep / P.xw % P.wy;
  P.xdz = xstep / P.xw / P.wy;
  P.xrows = xrows;
  const int xwf = (P.xwaves + xrows - 1) / xrows;  // wavefronts of the x part
  P.xblocks = (xwf + kBlock / 64 - 1) / (kBlock / 64);
  P.brick_blocks = P.blocks[1] + P.blocks[2] + P.xblocks;
  P.total_blocks = P.brick_blocks * P.nby * P.nbz;
  return P;
}

// The face plan of a single periodic box.
FacePlan box_face_plan(const ctmhd_params* p, const ctmhd_box& b, const Geom& G) {
  const bool alu = p->precision == CTMHD_FP64 && p->recon == CTMHD_RECON_PPM &&
                   p->riemann == CTMHD_RIEMANN_HLLD;
  return make_face_plan(G, p, true, march_faces(b, p->recon, p->emf_compute, true), 1, !alu);
}

template <typename T, int RECON>
int launch_faces(hipStream_t st, const ctmhd_params* p, State S, const Geom& G, const Work<T>& W,
                 const FacePlan& FP, int stage, long long* diag, const DtStep* dt = nullptr) {
  const FaceArgs<T> A{S,    G,      W,    FP, stage, p->gamma, p->eta, diag,
                      W.stop, dt ? *dt : DtStep{}};
  const int blocks = FP.total_blocks + (dt ? 1 : 0);
  prof_begin(st);
  if constexpr (std::is_same<T, float>::value) {
    if (p->precision == CTMHD_FP32_R64) {
      if (p->riemann == CTMHD_RIEMANN_HLLD)
        LAUNCH((k_faces<T, RECON, kHLLD64>), blocks, A);
      else
        LAUNCH((k_faces<T, RECON, kLLF64>), blocks, A);
      prof_end(st);
      return CTMHD_OK;
    }
  }
  if (p->riemann == CTMHD_RIEMANN_HLLD)
    LAUNCH((k_faces<T, RECON, kHLLD>), blocks, A);
  else
    LAUNCH((k_faces<T, RECON, kLLF>), blocks, A);
  prof_end(st);
  return CTMHD_OK;
}

// Q26 edge pass as z marches: the most workgroups (so that the search below is
// short) and the shortest z chunk
constexpr int kEmfTiles = 32768;
constexpr int kEmfMinChunk = 5;
// Workgroups of the per-edge kernel up to which it is split by direction: two
// per CU, from where on three edges per thread fill the chip as well.  Step
// without / with the split, FP64, us: PPM Q26 16^3 76 / 64, 32^3 81 / 71, 48^3
// (460 workgroups) 121 / 116, 56^3 (724) 153 / 152, 80^3 (2076) 323 / 329; PPM FS18
// 32^3 118 / 104, 48^3 169 / 169, 56^3 213 / 218, 64^3 (1073) 294 / 282, 80^3 497 /
// 504; PLM Q26 32^3 66 / 65, 48^3 94 / 96, 56^3 123 / 126.
constexpr int kEmfSplitBlocks = 512;

// Workgroups of the z-marching edge kernel that the device holds at once (0 if
// the runtime cannot say).  Queried once per instantiation.
template <typename T, int RECON>
int emf_march_resident() {
  static const int n = [] {
    int dev = 0, ncu = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_emf_march<T, RECON>, kBlock, 0) !=
        hipSuccess)
      return 0;
    return ncu * per;
  }();
  return n;
}

template <typename T, int RECON>
int launch_emf(hipStream_t st, const ctmhd_params* p, State S, const Geom& G, const Work<T>& W,
               int stage) {
  const int cnt = (G.n[0] + 1) * (G.n[1] + 1) * (G.n[2] + 1);
  const int band = xcd_band(p, (long long)(G.n[0] + 1) * (G.n[1] + 1), cnt);
  // per-edge kernel: one edge direction per thread where the three together
  // leave CUs without a workgroup
  const int split = nblocks(cnt) <= kEmfSplitBlocks ? nblocks(cnt) : 0;
  const int blocks = split ? 3 * split : nblocks(cnt);
  if (p->emf_compute == CTMHD_EMF_Q26) {
    // z marches: the number of chunks with the smallest number of rounds of the
    // chip times the length of a march (its positions and the filling of its
    // pipelines, about a position and a half)
    const int ctiles = (emf_march_items(G, recon_halfwidth(RECON)) + kBlock / 64 - 1) / (kBlock / 64);
    const int L2 = G.n[2] + 1, res = emf_march_resident<T, RECON>();
    int nch = 1;
    double best = 0.0;
    for (int k = 1; k <= L2 / kEmfMinChunk && k <= kEmfTiles / ctiles + 1; ++k) {
      const int len = (L2 + k - 1) / k;
      const double rounds = res > 0 ? (double)((ctiles * ((L2 + len - 1) / len) + res - 1) / res) : 1.0;
      const double cost = rounds * (len + 1.5);
      if (k == 1 || cost < best) {
        best = cost;
        nch = k;
      }
    }
    const int zc = (L2 + nch - 1) / nch;
    nch = (L2 + zc - 1) / zc;
    // automatic: a small box gives the marches less than about one round of
    // the chip, where the per-edge kernel's many short workgroups fill it
    // better (the two give the same values)
    const int m = tile_emf(p);
    if (m == 2 || (m == 0 && 4LL * ctiles * nch >= 3LL * emf_march_resident<T, RECON>()))
      LAUNCH((k_emf_march<T, RECON>), ctiles * nch, S, G, W, stage, p->eta, ctiles, zc, W.stop);
    else
      LAUNCH((k_emf3<T, RECON, kQ26>), blocks, S, G, W, stage, p->eta, band, split, W.stop);
  } else if (p->emf_compute == CTMHD_EMF_B25A)
    LAUNCH((k_emf3<T, RECON, kB25A>), blocks, S, G, W, stage, p->eta, band, split, W.stop);
  else
    LAUNCH((k_emf3<T, RECON, kFS18>), blocks, S, G, W, stage, p->eta, band, split, W.stop);
  return CTMHD_OK;
}

}  // namespace
