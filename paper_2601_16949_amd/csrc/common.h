// Internal declarations of the RT-TDA gfx950 library (kernels + runtime).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <cstddef>
#include <cstdint>

#include "rttda.h"

namespace rttda {

// Device copy of rttda_pulse (identical layout, checked by static_assert in the runtime).
struct DevPulse {
  int32_t kind;
  int32_t reserved;
  double e0, omega, t0, fwhm, beta, phase;
  double dir[3];
};

// Device-resident propagation scalars.
struct DevState {
  long long step;      // absolute step index of the current state c
  long long pend;      // 1: the step's last epilogue has run and `step` is still the old one (the next
                       // field product adds it: the epilogue's own blocks read `step`)
  long long step0;     // step index at the start of the current propagate call
  long long bad_step;  // first step at which the norm guard tripped, -1 if none
  long long keep_ref;  // 1: the call resumes a run (the guard's reference norm and first bad step
                       // carry over from the previous call), 0: both restart with the call
  double *trace;       // trace row of step0 ([n_steps+1][nrhs]) or NULL; set per call, so a
  double *norms;       // captured step graph stays valid across calls with new output arrays
  double *corr;        // time-correlation output ([n_steps+1][nrhs][2]) or NULL, likewise
  double *pops;        // eigenstate populations output ([n_steps+1][nrhs][popk]) or NULL, likewise
  const double *popU;  // the popk unit vectors ([popk][o][v]) the states are projected on
  long long popk;
  double *energy;      // energy output <X|diag(0,A)|X> ([n_steps+1][nrhs]) or NULL, likewise
  const double *epart; // the epilogue's per-block energy partial sums [nrhs][nbe]
  long long nbe;
};
constexpr int POP_MAX = 64;  // eigenstates per populations output

constexpr double SQRT2 = 1.4142135623730951;
constexpr double FWHM_TO_SIGMA = 2.35482;

// Field of one pulse at time t (eqs. continuous wave, transform_limited, chirped_pulse).
// Delta pulses act as a kick at t = 0 and contribute no continuous field.
__device__ inline double pulse_field(const DevPulse &p, double t) {
  if (p.kind == RTTDA_PULSE_CW) return p.e0 * sin(p.omega * t + p.phase);
  if (p.kind == RTTDA_PULSE_GAUSS || p.kind == RTTDA_PULSE_CHIRP) {
    const double s = p.fwhm / FWHM_TO_SIGMA;
    const double tau = t - p.t0;
    const double env = exp(-tau * tau / (2.0 * s * s));
    const double arg = (p.kind == RTTDA_PULSE_GAUSS) ? p.omega * tau + p.phase
                                                      : (p.omega + 0.5 * p.beta * tau) * tau + p.phase;
    return p.e0 * env * sin(arg);
  }
  return 0.0;
}


// Per-RHS scalar slots (f64): g_re, g_im, E(t_stage), spare.
constexpr int SC_STRIDE = 4;
constexpr int SC_GRE = 0, SC_GIM = 1, SC_E = 2;
// Per-block partial sums of the field kernel (f64): g_re, g_im, <X|F>, |X|^2.
constexpr int PART_STRIDE = 4;

// Field-kernel tile (i x a) and its grid per RHS.
constexpr int FT_I = 16, FT_A = 16;
__host__ __device__ inline int field_blocks_a(int v) { return (v + FT_A - 1) / FT_A; }
__host__ __device__ inline int field_blocks_i(int o) { return (o + FT_I - 1) / FT_I; }
__host__ __device__ inline int field_blocks(int o, int v) { return 2 * field_blocks_a(v) * field_blocks_i(o); }

// k_scalar modes (bit mask).
enum : int {
  SM_TRACE = 1,     // write trace/norm samples at index step - step0, update the guard
  SM_C0 = 2,        // RK4 stage update of c0 with k0 = i E g
  SM_INC = 4,       // the step is done: `pend`
  SM_EFIELD = 8,    // E = pulse field at (step + node) dt (else E = 0 unless SM_KEEP_E)
  SM_SIGMA0 = 16,   // s0 = -E g with E preset by the host
  SM_OUT = 32,      // out[r] = <X|M|X>  (dipole_trace entry point)
  SM_KEEP_E = 64,   // keep the E slots written by the host
  SM_ENERGY = 128,  // energy sample at index step - step0 from the epilogue's partial sums
};

// Partial slabs of a stage's two-electron part: `n` of them to be added in FP64, the first `nc` as they are,
// each of the others the FP32 sum, in order, of `grp` neighbours in memory.
struct Slabs {
  int n, nc, grp;
};

// Epilogue modes.
enum : int { EP_RK4 = 0, EP_SIGMA = 1, EP_ENERGY = 2 };
// Field product of `blocks` / field_blocks(o, v) right-hand sides (see field.h), as a launch of its own or
// beside the blocks of another launch that reads the same X; blocks = 0: none.
struct FieldArgs {
  const double *X, *X0, *moo, *mov, *mvv;
  int o, v;
  double *F, *part;
  DevState *st;
  int blocks;
};

// Small problems (o v <= SMALL_OV_MAX, at most SMALL_R_MAX RHS): one launch for the Coulomb and
// exchange partial slabs of a stage and the field product, one for the stage update.
constexpr int SMALL_OV_MAX = 2048;
constexpr int SMALL_R_MAX = 64;
// the small path is the default up to this many exchange flops per stage at max_rhs: 16 steps of o10 v40
// N_Q120 with one RHS (1e7) take 0.91 ms, with the general kernels 1.46.  Above, the choice depends on the
// shape (o10 v40 N_Q120 with six RHS, 6e7: 1.56 against 1.69 ms; o13 v45 N_Q160 with two, 4.3e7: 1.36 and
// 1.36; o10 v40 N_Q120 with eight, 8e7: 1.70 against 1.43): a caller who knows can ask for it
constexpr double SMALL_DEFAULT_FLOPS = 2e7;
// (with the partial-sum kernel's LDS, a slice's X and W and one Q's B_vv and B_oo in FP32, the shapes that
// the path takes)
constexpr int SMALL_LDS_FLOATS = 12288;
inline bool small_shape_ok(int o, int v) {
  return (long long)o * v <= SMALL_OV_MAX && 2LL * o * v + (long long)v * v + (long long)o * o <= SMALL_LDS_FLOATS;
}
hipError_t prepare_small();  // one-time kernel attributes (dynamic LDS); call outside graph capture
hipError_t launch_small_2e(hipStream_t s, int b_dtype, const void *Bov, const void *Boo, const void *Bvv,
                           const float *X, int o, int v, int nq, int ns, int nsplit, int m, float cx, float *P,
                           const FieldArgs &f);
// Epilogue grid: blocks per RHS along ia (the energy partial sums come one per block)
constexpr int EP_BX_MAX = 2048;
int epilogue_blocks(long long ov);
// symplectic split-operator update modes (k_sso_update)
enum : int { SSO_KICK_FIRST = 0, SSO_KICK = 1, SSO_DRIFT = 2 };

// ---------------------------------------------------------------------------------------------
// Kernel launchers (all enqueue on `s`, return hipError_t of the launch)
// ---------------------------------------------------------------------------------------------
hipError_t launch_mu_blocks(hipStream_t s, const double *mu, const DevPulse *pulses, int o, int v, int R,
                            double *moo, double *mov, double *mvv);
hipError_t launch_gaps(hipStream_t s, const double *e_occ, const double *e_virt, int o, int v, double *D);
hipError_t launch_to_f32(hipStream_t s, const double *c, long long n, float *x32);
hipError_t launch_to_bf16x2(hipStream_t s, const double *c, long long n, float *x32, __hip_bfloat16 *hi,
                            __hip_bfloat16 *lo);
// Coulomb first product in `nes` ia chunks (partials dpart[nes][nq][ns], which the second product
// adds); gemv1_chunks picks nes (at most GEMV1_CHUNKS_MAX).
constexpr int GEMV1_CHUNKS_MAX = 16;
int gemv1_chunks(int nq, int ov);
hipError_t launch_gemv1(hipStream_t s, int b_dtype, const void *B, const float *X, int nq, int ov, int ns, int nes,
                        float *dpart, const FieldArgs &f);
hipError_t launch_gemv2(hipStream_t s, int b_dtype, const void *B, const float *dpart, int nes, int nq, int ov, int ns,
                        int nsplit, float *P);
// The same pair on the FP32 matrix cores for batches of many slices (the context's 2 max_rhs >= 32):
// d in nes ia chunks (coulomb_mfma_chunks, at most GEMV1_CHUNKS_MAX) summed into chunk slot 0 of
// dpart, then the partial slabs P[split][s][ia] of J.
int coulomb_mfma_chunks(int nq, int ov);
hipError_t launch_coulomb_mfma(hipStream_t s, int b_dtype, const void *B, const float *X, int nq, int ov, int ns,
                               int nes, int nsplit, float *dpart, float *P, const FieldArgs &f);
hipError_t launch_field(hipStream_t s, const FieldArgs &f);
hipError_t launch_scalar(hipStream_t s, int R, int nbf, int stage, int mode, double dt, const DevPulse *pulses,
                         DevState *st, const double *part, double *sc, double *c0, double *acc0, double *xs0,
                         double *out, double *normref, double *s0);
// The stage scalars an RK4 epilogue carries (mode: SM_TRACE, SM_C0, SM_INC, SM_EFIELD, SM_ENERGY; 0 for none)
struct StageScalars {
  int mode, nbf;
  const DevPulse *pulses;
  DevState *st;
  const double *part;
  double *c0, *acc0, *xs0, *normref;
};
// epart != NULL: also the per-block partial sums of <X, A X> per RHS ([R][epilogue_blocks(ov)])
hipError_t launch_epilogue(hipStream_t s, int prec, int R, int o, int v, Slabs slabs, int stage, int mode,
                           int use_field, double dt, const double *D, const float *P, const double *F, double *sc,
                           const double *Xin, double *c, double *acc, double *xs64, float *x32, __hip_bfloat16 *xhi,
                           __hip_bfloat16 *xlo, double *s_out, double *epart = nullptr,
                           const StageScalars *scalars = nullptr);
hipError_t launch_sso_update(hipStream_t s, int prec, int R, int o, int v, Slabs slabs, int mode, int use_field,
                             double dt, const double *D, const float *P, const double *F, const double *sc, double *c,
                             double *c0, double *W, double *W0, float *x32, __hip_bfloat16 *xhi,
                             __hip_bfloat16 *xlo);
hipError_t launch_plane_copy(hipStream_t s, int prec, int R, size_t ov, int plane, const double *c, float *x32,
                             __hip_bfloat16 *xhi, __hip_bfloat16 *xlo);
// Lanczos guard: a launch's block partial sums (at most LZ_BLOCKS_MAX) are added by the next launch, which
// leaves the coefficient in device memory; at most LZ_STEPS_MAX steps
constexpr int LZ_BLOCKS_MAX = 1024;
constexpr int LZ_STEPS_MAX = 500;
int lz_blocks(long long n);
hipError_t launch_lz_init(hipStream_t s, long long n, double *v, double *part);
// w = A v - beta vprev (beta: device, or null for 0), part = <w, v>
hipError_t launch_lz_apply(hipStream_t s, long long n, int nslab, const double *D, const float *P, const double *v,
                           const double *vprev, const double *beta, double *w, double *part);
// alpha = sum dots, w -= alpha v, part = <w, w>
hipError_t launch_lz_orth(hipStream_t s, long long n, const double *v, const double *dots, double *alpha, double *w,
                          double *part);
// beta = sqrt(sum dots), vprev = v (shift), v = w / beta and its stage copies
hipError_t launch_lz_next(hipStream_t s, int prec, long long n, const double *dots, double *beta, const double *w,
                          double *v, double *vprev, float *x32, __hip_bfloat16 *xhi, __hip_bfloat16 *xlo, int shift);
// Block Davidson (lowest eigenpairs of A) and populations: FP64 vectors of n = o*v stored one after
// another; per-block partial sums (at most DV_BLOCKS_MAX per vector) are added on the host.
constexpr int DV_BLOCKS_MAX = 1024;
constexpr int DV_SPACE_MAX = 64;  // largest search space (vectors)
int dv_blocks(long long n);
hipError_t launch_dv_apply(hipStream_t s, long long n, int nb, int nslab, const double *D, const float *P,
                           const double *V, double *W);
hipError_t launch_dv_dots(hipStream_t s, long long n, int m, const double *V, int nt, const double *T, double *out);
hipError_t launch_dv_combine(hipStream_t s, long long n, int m, const double *V, int nc, const double *C, int ldc,
                             int mode, double *out);
hipError_t launch_dv_resid(hipStream_t s, long long n, int nc, const double *X, const double *AX, const double *theta,
                           double *R, double *part);
hipError_t launch_dv_precond(hipStream_t s, long long n, int nc, const double *R, const double *theta,
                             const double *D, double *T);
hipError_t launch_dv_norm2(hipStream_t s, long long n, const double *T, double *part);
hipError_t launch_dv_scale(hipStream_t s, long long n, double scale, const double *T, double *out);
hipError_t launch_dv_unit(hipStream_t s, long long n, long long idx, double *V);
hipError_t launch_dv_diag(hipStream_t s, int b_dtype, int o, int v, int nq, const void *Bov, const void *Boo,
                          const void *Bvv, double cx, const double *D, double *diag);
hipError_t launch_kick(hipStream_t s, int R, int ov, const DevPulse *pulses, const double *F, const double *sc,
                       double *c, double *c0);
hipError_t launch_kick_term(hipStream_t s, int R, int ov, const DevPulse *pulses, const double *F, const double *sc,
                            double inv_j, double *T, double *T0, double *c, double *c0);
hipError_t launch_set_state(hipStream_t s, DevState *st, long long step0, double *trace, double *norms,
                            double *corr, double *pops, const double *popU, int popk, double *energy = nullptr,
                            const double *epart = nullptr, long long nbe = 0, int resume = 0);
// eigenstate populations |<U_I | X_r>|^2 at the current step (no-op unless st->pops is set)
hipError_t launch_pop(hipStream_t s, int R, size_t ov, const double *X, const DevState *st);
hipError_t launch_spectrum(hipStream_t s, int kind, const double *sig, int n_t, int nsig, double dt, double kappa,
                           int n_w, double w0, double dw, int average, double *out);
// time-correlation sample <Xref_r | X_r> (both planes and the ground amplitude) at the current step
hipError_t launch_corr(hipStream_t s, int R, size_t ov, const double *X, const double *X0, const double *xref,
                       const double *xref0, const DevState *st);

// Exchange: K partials P[split][slice][o][v] = scale * sum_{Q in split} B_oo^Q X_slice B_vv^Q.
// Large-o split-BF16 path (two batched GEMMs per chunk of Q through a W scratch buffer) for o >= XGEMM_O_MIN
// with v % 8 == 0; the scratch holds W hi/lo for up to XGEMM_SCRATCH_MAX bytes' worth of Q values.
constexpr int XGEMM_O_MIN = 65;
constexpr size_t XGEMM_SCRATCH_MAX = size_t(2048) << 20;
constexpr size_t XGEMM_SCRATCH_MID = size_t(256) << 20;  // below o = 128, where 256 MiB hold hundreds of Q
inline int xgemm_op(int o) { return (o + 7) / 8 * 8; }   // a slice's rows there: 16-byte groups
// bytes behind the W scratch for X (rows = slices x op) in the order the first GEMM stages it: columns in
// whole chunks of 32, rows in whole tiles of at most 256, hi and lo; and behind those B_oo of a chunk of
// Q, padded, where o is not a multiple of 8
inline size_t xgemm_x_bytes(int v, size_t rows) { return (size_t)((v + 31) / 32) * 32 * (rows + 255) * 4; }
inline size_t xgemm_o_bytes(int o, size_t qc) { return o % 8 ? qc * xgemm_op(o) * xgemm_op(o) * 2 : 0; }

// work of an X-resident exchange workgroup (see shape_xres)
struct ResShape {
  int tiles, qs;
  double q_cycles, start_cycles;
  bool ranges;  // whether a split may be cut into ranges
};

struct ExchangeVariant {
  int precision;  // RTTDA_PREC_*
  int o16;        // padded occupied count handled (o <= o16)
  int ks;         // slices per workgroup
  int nt;         // virtual columns per workgroup
  const char *name;
  hipError_t (*launch)(hipStream_t s, const void *Boo, const void *Bvv, const void *X, const void *Xlo, int o,
                       int v, int nq, int ns, int nsplit, float scale, float *P, void *scratch,
                       size_t scratch_bytes);
  size_t lds_bytes;
  hipError_t (*prepare)();  // one-time kernel attributes (dynamic LDS size); call outside graph capture
  int v_min = 1;            // applicability: v >= v_min, v % v_mod == 0, o % o_mod == 0, o >= o_min
  int v_mod = 1;
  int o_mod = 1;
  int o_min = 1;
  bool scratch = false;  // needs the W scratch region of the workspace
  int rank = 0;          // preference among variants of equal tile waste (higher first)
  int v_max = 1 << 30;
  void (*res)(int v, int ns, struct ResShape *) = nullptr;  // X resident in LDS (one workgroup fills a CU)
  // X-resident variants, of whose nsplit splits each is cut into m ranges of Q: a workgroup per split (whole), which
  // leaves their FP32 sum (FP32) or each (split BF16), or a workgroup per range, which leaves that.  A slab per
  // range left, every m of them to be added in FP32, in order, by the reader
  hipError_t (*launch_ranges)(hipStream_t s, const void *Boo, const void *Bvv, const void *X, const void *Xlo, int o,
                              int v, int nq, int ns, int nsplit, int m, bool whole, float scale, float *P) = nullptr;
  int rows = 0;  // scratch variants: stacked rows per tile of the first GEMM (nt: its columns)
  int cols = 0;  //                   columns per tile of the second
  bool applies(int o, int v) const {
    return o <= o16 && o >= o_min && v >= v_min && v <= v_max && v % v_mod == 0 && o % o_mod == 0;
  }
};

}  // namespace rttda
