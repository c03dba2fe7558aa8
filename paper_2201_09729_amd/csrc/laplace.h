// Launchers of the Laplacian, Lanczos, projector and contraction kernels.
#pragma once
#include "../../include/dlma.h"
#include "kernels.h"

namespace dlma {

// qd (one vector per timeslice, nv = 1): also write the block partials of Re <qd, out>
// to part[t * lap_site_blocks(g) + block]
int lap_site_blocks(const Geo& g);
hipError_t launch_neg_lap(const double2* U64, const Geo& g, int t0, const double2* in, double2* out, long tsi, long tso,
                          int nt, hipStream_t s, int nv = 1, long vsi = 0, long vso = 0, const double2* qd = nullptr,
                          double* part = nullptr);
// ts*: timeslice strides of in, prev, out and qd
hipError_t launch_cheb_step(const double2* U64, const Geo& g, int t0, const double2* in, long tsi, const double2* prev, long tsp,
                            double2* out, long tso, int nt, double c1, double c2, hipStream_t s, const double2* qd = nullptr,
                            long tsqd = 0, double* part = nullptr);
hipError_t launch_rayleigh(const double2* y, const double2* ay, long n, int nvec, double* lam, double* res, hipStream_t s);
// <a, b> over n complex numbers; part: dot_parts(n) numbers
int dot_parts(long n);
hipError_t launch_dot(const double2* a, const double2* b, long n, double2* part, double2* out, hipStream_t s);
// Lanczos step with split reductions: alpha from the stencil's partials (nap per
// timeslice), Gram-Schmidt dots in GS_NCH element chunks, |w|^2 partials from the last
// subtraction (gs_sub_blocks(n) per timeslice) consumed by the normalisation.  prev =
// false: no beta_{j-1} q_{j-1} term (the first step after a thick restart, whose
// couplings to the kept Ritz vectors the Gram-Schmidt passes remove).
constexpr int GS_NCH = 8;
int gs_sub_blocks(long n);
hipError_t launch_lanczos_three_p(const double2* q, long tsq, long isq, double2* w, long tsw, long n, const double* apart, int nap,
                                  double* alpha, double* beta, int astride, int j, int nt, hipStream_t s, bool prev);
hipError_t launch_gs_dots(const double2* a, long tsa, long isa, const double2* b, long tsb, long n, double2* hp, int hstride, int ni,
                          int nt, hipStream_t s);
hipError_t launch_gs_sub(const double2* q, long tsq, long isq, const double2* hp, int hstride, int ni, double2* w, long tsw, long n,
                         int nt, double* npart, hipStream_t s);
hipError_t launch_scale_p(const double2* w, long tsw, double2* q, long tsq, long n, const double* npart, double* nrm, int ostride,
                          int j, int nt, hipStream_t s);
hipError_t launch_normalize_into(const double2* w, long tsw, double2* q, long tsq, long n, double* nrm, int ostride, int j, int nt,
                                 hipStream_t s);
hipError_t launch_ritz(const double2* q, long tsq, long isq, const double* S, int m, int nev, double2* y, long tsy, long n, int nt,
                       hipStream_t s);
// block eigensolver (vectors [t][k][n]; kb <= 64)
hipError_t launch_cheb_block(const double2* U64, const Geo& g, int t0, const double2* in, const double2* prev, double2* out,
                             int nt, int kb, double c1, double c2, hipStream_t s);
int block_gram_chunks(long n, int nt);
hipError_t launch_block_gram(const double2* A, const double2* B, long n, int kb, int nt, double2* part, double2* G,
                             hipStream_t s);
hipError_t launch_block_update(const double2* X, const double2* Z, long n, int kb, int kout, int nt, double2* Y, long ytstride,
                               hipStream_t s);
hipError_t launch_block_random(double2* V, long count, unsigned seed, hipStream_t s);
hipError_t launch_phase_fix(double2* y, long n, int nvec, hipStream_t s);
// contractions
// Column sets of 16 (label, spin) columns per source group: the groups of f0, or with
// noise the phi (f0) and phibar (f1) of each group in turn (sets 2 g, 2 g + 1).
struct ContractArgs {
    const double2 *Vall, *f0, *f1;
    long L3, fs;       // sites of a timeslice, complex numbers of a field
    const int* tlist;  // the nt timeslices, nullptr = t0 .. t0 + nt - 1
    int t0, tv0;       // tv0: timeslice of Vall's first entry
    int nt, nev, ng, ks;
    int nf;            // fields of f0 (4 ng, or fewer in the last group: its further columns repeat the last field)
    double2* taup;     // partials [ks][set][nt][nev][16] (unused with ks = 1)
    double2* gramp;    // [nt][ks][unit][noise ? 2 : 1][16][16]: (re, X) of (f0, f0), then (f1, f0)
    int nunit, k0, nkb;  // set by the launcher
    long chunk;
};
int contract_ks(const Geo& g, int nt, int units);
// tau[set][nt][nev][16], and with gram the Gram partials of nunit = noise ? ng : (ng + 1) / 2 units
hipError_t launch_contract(const ContractArgs& a, bool noise, bool gram, double2* tau, hipStream_t s);
// part[nt][proj_gram_parts()][16][16] of sum_g sum_k conj(tau[oa + st g]) tau[ob + st g]
int proj_gram_parts();
hipError_t launch_proj_gram(const double2* tau, int nt, int nev, int ng, int oa, int ob, int st, double2* part, hipStream_t s);
// box(t) of launch_project: coef and part hold coef_cap and part_cap complex numbers.  The
// coefficients of as many right-hand sides as coef holds are formed before the first of
// their outputs is written, in chunks that fit part.  The site chunks depend on the lattice
// and nev alone, so the result does not depend on the capacities.
constexpr long PROJ_PART_CAP = 524288;
int project_ks(const Geo& g, int nev);
hipError_t launch_project(const double2* Vt, const double2* in, double2* out, const Geo& g, int t, int nev, int nrhs, int mode,
                          double2* coef, long coef_cap, double2* part, long part_cap, hipStream_t s);
struct CorrPiecesArgs {
    const double2 *gd, *pd;         // dist: Gram partials [T][nud], projected partials
    const double2 *gn, *pn, *pq;    // noise: Gram partials [T][nun][2], projected (phi, phi) and (phibar, phi)
    const double2* W;               // [DLMA_NGAMMA][16][16] spin weights
    double2* C;                     // [DLMA_NGAMMA][DLMA_NPARTS][T]
    double inv_nvec;
    int T, t_src, nud, nun;
};
hipError_t launch_corr_pieces(const CorrPiecesArgs& a, hipStream_t s);
// tau' = WP tau for ngrp groups of N = noise ? 32 : 16 columns, WP [T][N][N]
hipError_t launch_tau_weights(const double2* tau, const double2* WP, const int* tlist, int nact, int nev, int ngrp, bool noise,
                              double2* o, hipStream_t s);
// backward of the correlator contractions (see contract.hip)
struct CorrGradArgs {
    const double2* Vall;                       // [T][nev][L3][3]
    const double2 *dist, *phi, *phibar;        // input fields, canonical, fs complex numbers each
    double2 *gdist, *gphi, *gphibar;           // gradient fields (written on every timeslice)
    const double2* W1n;                        // [T][32][32]: noise groups, (phi, phibar) x spin
    const double2* W1d;                        // [T][16][16]: distillation groups, phi_dist x spin
    const double2* taun;                       // [nnoise][nact][nev][32]: WP(t) V(t)^dag F, noise groups
    const double2* taud;                       // [ndist][nact][nev][16]
    const int* tact;                           // [T]: index among the weighted timeslices, or -1
    long L3, fs;
    int nev, ndist, nnoise, nact;
};
hipError_t launch_corr_grad(const CorrGradArgs& a, int T, hipStream_t s);

}  // namespace dlma
