// ctmhd.hip -- kernels and C ABI of libctmhd for gfx950 (MI355X).
//
// One RK2-SSP step with first-order flux correction (Sec. 2.5 of Kriel et al.)
// is a short sequence of stream-ordered kernels on a ghosted box:
//   k_start      once per call: ghost fill, CFL maximum and, for an odd number
//                of steps, the copy into the other buffer
//   per stage:
//   k_faces      reconstruction + Riemann solve at every face of all three
//                directions in one launch: x faces inside a wavefront (whole-
//                wavefront shifts), y and z faces by marching along the face
//                normal with a register window, so that every cell is loaded
//                and reconstructed once per direction; primitives are formed
//                on the fly (pressure recovery in FP64); in the first stage an
//                extra workgroup forms dt from the CFL maximum of the step's
//                starting state (or takes the caller's); a non-finite dt stops
//                the call
//   k_emf_march  Q26 edge EMFs of the three edge directions with LD04
//                averaging and eta j, a row of edge columns per wavefront
//                marching up z (z reconstructions streamed through registers,
//                x ones across the wavefront)
//   k_emf3       the same for small boxes and for B25a / FS18, one thread per
//                edge position (and direction, on the smallest)
//   k_update     flux divergence and CT curl, RK combination, periodic ghost
//                images, invalid-state flags and (second stage) the CFL
//                maximum of the new state for the next step
//   k_fo         first-order fluxes / EMFs from S^n around flagged cells
//   k_update     again (fix-up mode), only when something was flagged, for the
//                cells those values reach
// Face arrays hold the x_a face on the lower side of each cell, edge arrays
// the edge at the lower corner in the two transverse directions.
#include "ctmhd_host.h"

thread_local char g_err[256] = "";
void* const* g_prof_events = nullptr;
int g_prof_pairs = 0;
int g_prof_used = 0;

namespace {

template <typename T>
int launch_fo(hipStream_t st, const ctmhd_params* p, State Sn, const Geom& G, const Work<T>& W,
              int stage, int ninter) {
  const int nb = fix_blocks(ninter);
  if (p->emf_compute == CTMHD_EMF_Q26)
    LAUNCH((k_fo<T, kQ26>), nb, Sn, G, W, stage, p->gamma, p->eta, W.stop);
  else if (p->emf_compute == CTMHD_EMF_B25A)
    LAUNCH((k_fo<T, kB25A>), nb, Sn, G, W, stage, p->gamma, p->eta, W.stop);
  else
    LAUNCH((k_fo<T, kFS18>), nb, Sn, G, W, stage, p->gamma, p->eta, W.stop);
  return CTMHD_OK;
}

// One stage: fluxes and EMFs of `in`, update into `out` from `base` = S^n.
template <typename T, int RECON>
int run_stage(hipStream_t st, const ctmhd_params* p, const Geom& G, const Work<T>& W,
              const FacePlan& FP, State in, State base, State out, int stage, double sres,
              long long* diag, const Restore& R, const DtStep* dt) {
  int rc;
  if (p->emf_compute == CTMHD_EMF_B25A) {
    LAUNCH((k_prim<T, kB25A>), nblocks(G.elems), in, G, W, p->gamma, W.stop);
    if constexpr (first_step_stored(kB25A, RECON))
      LAUNCH((k_first_step<T, RECON, kB25A>), nblocks(G.elems), G, W, W.stop);
  } else if (p->emf_compute == CTMHD_EMF_FS18) {
    LAUNCH((k_prim<T, kFS18>), nblocks(G.elems), in, G, W, p->gamma, W.stop);
    if constexpr (first_step_stored(kFS18, RECON))
      LAUNCH((k_first_step<T, RECON, kFS18>), nblocks(G.elems), G, W, W.stop);
  }
  if ((rc = launch_faces<T, RECON>(st, p, in, G, W, FP, stage, diag, dt))) return rc;
  if ((rc = launch_emf<T, RECON>(st, p, in, G, W, stage))) return rc;
  const int ninter = G.n[0] * G.n[1] * G.n[2];
  UpdateCfg U;
  U.fofc = p->fofc;
  U.crit = p->flag_criteria;
  U.gamma = p->gamma;
  U.sres = sres;
  U.force = p->force_flags ? p->force_flags + (size_t)stage * ninter : nullptr;
  U.flag_storage = 0;
  const int band = xcd_band(p, (long long)G.n[0] * G.n[1], ninter);
  if ((rc = launch_update<T, 0>(st, nblocks(ninter), base, in, out, G, W, stage, U, diag, band,
                                p->fofc ? Restore{} : R)))
    return rc;
  if (!p->fofc) return CTMHD_OK;
  if ((rc = launch_fo<T>(st, p, base, G, W, stage, ninter))) return rc;
  return launch_update<T, 1>(st, fix_blocks(ninter), base, in, out, G, W, stage, U, diag, band, R);
}

template <typename T, int RECON>
int step_box(const ctmhd_params* p, const ctmhd_box* box, double* const cons[5],
             double* const bface[3], int nsteps, const double* dt_fixed, double* dt_out,
             int64_t* diag, void* ws, size_t ws_bytes, hipStream_t st) {
  Geom G = make_geom(*box);
  Work<T> W;
  State B, H;
  int rc = build_work<T>(p, ws, ws_bytes, *box, W, B, H);
  if (rc) return rc;
  State user;
  for (int m = 0; m < 5; ++m) user.c[m] = cons[m];
  for (int a = 0; a < 3; ++a) user.b[a] = bface[a];
  const FacePlan FP = box_face_plan(p, *box, G);
  double dxmin = fmin(G.dx[0], fmin(G.dx[1], G.dx[2]));
  double sres = p->eta > 0.0 ? 2.0 * p->eta / (dxmin * dxmin) : 0.0;
  // steps alternate between the caller's buffers and B; an odd number of them
  // starts from a copy in B, so that the last one ends in the caller's
  const bool odd = nsteps & 1;
  State A = odd ? B : user;
  if (odd) B = user;
  const State other = odd ? A : B;
  int npart = 0;
  if ((rc = launch_start(st, p, user, A, odd, G, W, dt_fixed == nullptr, sres,
                         (long long*)diag, diag ? 4 * nsteps : 0, npart)))
    return rc;
  for (int n = 0; n < nsteps; ++n) {
    long long* dg = diag ? (long long*)diag + 4 * n : nullptr;
    const DtStep D = make_dt_step(p, W, npart, n, dt_fixed ? dt_fixed + n : nullptr,
                                  dt_out ? dt_out + n : nullptr, dg);
    if ((rc = run_stage<T, RECON>(st, p, G, W, FP, A, A, H, 0, sres, dg, Restore{}, &D))) return rc;
    // the last kernel of the call brings a stopped call's state back
    const Restore R{user, other, G.elems, n == nsteps - 1 ? nsteps : 0};
    if ((rc = run_stage<T, RECON>(st, p, G, W, FP, H, A, B, 1, sres, dg, R, nullptr))) return rc;
    State tmp = A;
    A = B;
    B = tmp;
  }
  return CTMHD_OK;
}

template <typename T>
int step_box_t(const ctmhd_params* p, const ctmhd_box* box, double* const cons[5],
               double* const bface[3], int nsteps, const double* dt_fixed, double* dt_out,
               int64_t* diag, void* ws, size_t ws_bytes, hipStream_t st) {
  switch (p->recon) {
    case CTMHD_RECON_PC:
      return step_box<T, kPC>(p, box, cons, bface, nsteps, dt_fixed, dt_out, diag, ws, ws_bytes, st);
    case CTMHD_RECON_PLM_MC:
      return step_box<T, kPLM_MC>(p, box, cons, bface, nsteps, dt_fixed, dt_out, diag, ws, ws_bytes, st);
    case CTMHD_RECON_PLM_MINMOD:
      return step_box<T, kPLM_MM>(p, box, cons, bface, nsteps, dt_fixed, dt_out, diag, ws, ws_bytes, st);
    default:
      return step_box<T, kPPM>(p, box, cons, bface, nsteps, dt_fixed, dt_out, diag, ws, ws_bytes, st);
  }
}


}  // namespace

extern "C" {

int ctmhd_required_ghosts(const ctmhd_params* p) {
  int rc = check_params(p);
  if (rc) return rc;
  return recon_halfwidth(p->recon) + 2;
}

int64_t ctmhd_box_elems(const ctmhd_box* b) {
  if (!b) return 0;
  int64_t e = 1;
  for (int d = 0; d < 3; ++d) e *= (int64_t)(b->n[d] + 2 * b->ng);
  return e;
}

int ctmhd_step(const ctmhd_params* p, const ctmhd_box* box, double* const cons[5],
               double* const bface[3], int nsteps, const double* dt_fixed, double* dt_out,
               int64_t* diag, void* workspace, size_t ws_bytes, void* stream) {
  g_err[0] = 0;
  int rc = check_params(p);
  if (rc) return rc;
  if ((rc = check_box(p, box))) return rc;
  if (!cons || !bface) return fail(CTMHD_EARG, "state pointers are NULL");
  for (int m = 0; m < 5; ++m)
    if (!cons[m]) return fail(CTMHD_EARG, "a cons pointer is NULL");
  for (int a = 0; a < 3; ++a)
    if (!bface[a]) return fail(CTMHD_EARG, "a bface pointer is NULL");
  if (nsteps < 0) return fail(CTMHD_EARG, "nsteps must be >= 0");
  if (nsteps == 0) return CTMHD_OK;
  hipStream_t st = (hipStream_t)stream;
  if (p->precision != CTMHD_FP64)
    return step_box_t<float>(p, box, cons, bface, nsteps, dt_fixed, dt_out, diag, workspace,
                             ws_bytes, st);
  return step_box_t<double>(p, box, cons, bface, nsteps, dt_fixed, dt_out, diag, workspace,
                            ws_bytes, st);
}

int ctmhd_profile_events(void* const* events, int npairs) {
  if (npairs < 0) return fail(CTMHD_EARG, "npairs must be >= 0");
  g_prof_events = npairs > 0 ? events : nullptr;
  g_prof_pairs = events ? npairs : 0;
  g_prof_used = 0;
  return CTMHD_OK;
}

int ctmhd_profile_recorded(void) { return g_prof_used; }

const char* ctmhd_last_error(void) { return g_err; }

}  // extern "C"
