// The library context (fq_ctx): host-side state of one problem, used by the
// C-ABI driver only. The kernels see the launch structures of internal.h.
#pragma once

#include "internal.h"

// The step propagator sum_l c_l T_l(Ht) as matrix products: T_1 .. T_s, then
// Clenshaw's recurrence in T_s over the blocks Q_0 .. Q_J-1 (g: s + 1
// coefficients of T_0 .. T_s per block, step phase included). FP64 plans hold the
// propagator without its multiple c0 of the identity and the T_l as S_l = T_l - sigma_l
// (see poly_plan_s).
struct PolyPlan {
  int s = 0, J = 0;
  std::vector<double> gr, gi;
  fq::PolyScalar c0;
};

// The same in split BF16 (see choose_mixed_poly): formats of T_l (index l), of the
// product that completes block j, and of the product with X; E = c0 + the plan's sum.
struct MixedPoly {
  PolyPlan plan;
  std::vector<int> t_fmt, b_fmt;
  int x_fmt = 0;
  std::complex<double> c0;
  double form = 0.0;  // cost of E, in units of a product's matrix instructions
  double err = 0.0;   // estimate of the error that the formats add to U_T
};

// ---- the context ---------------------------------------------------------------------------
struct fq_ctx {
  // system
  int64_t n = 0;
  int layout = 0;
  fq_system sys{};
  // params
  double T = 0, h = 0, tol = 0;
  int M = 0, L = 0, precision = 0, ckpt = 0;
  std::vector<double> f_nodes, a, b;  // host
  // scheme: 0 = Magnus-4 (H0 + a V + b K); 1 = the sixth-order scheme, whose
  // H_eff,k = H0 + a_k V + sum_j w6[k][j] B_j over nine fixed Hermitian nested
  // commutators B_j (device planes comm6, 2 planes each); a_k as above, b_k = 1
  // for the K slot, which then holds each step's sum over the B_j.
  int scheme = 0;
  // FQ_CF4 runs every step as spp = 2 half-steps: M, h and ckpt above count
  // those; M_user is the caller's step count (API indices are scaled by spp).
  int spp = 1, M_user = 0;
  // dense model given in H0's eigenbasis (sys.h0_diag = E_i): H0 planes hold
  // diag(E), and commutators with H0 are taken elementwise
  bool h0_eigen = false;
  // drive terms: S matrices Hmod_s; the drive block holds J planar matrices B_j
  // (re planes of all J, then im planes): one term -> [Hmod, K]; S >= 2 ->
  // [Hmod_s..., and for FQ_MAGNUS4 K_s = -i [H0, Hmod_s]..., K_st = -i [Hmod_s, Hmod_t]
  // (s < t)]; wS (M x J) are the per-(sub)step weights of the B_j when S >= 2.
  int S = 1, J = 2;
  bool pair_sums = false;             // floquet_grad: node-pair sums only (no K contraction)
  // the parameters the drive-dependent setup needs again on fq_set_drive
  double mixed_tol = 0.0;
  std::vector<int> term_formats;      // caller's term formats (empty: the library's schedule)
  bool interval_given = false;        // the caller fixed [e_min, e_max]
  double e_min_given = 0.0, e_max_given = 0.0;
  int L_given = 0;                    // the caller fixed L (> 0)
  bool drive_ok = true;               // false after a failed fq_set_drive
  // Ritz extremes of the fixed operators (H0, Hmod, ...), by operator pointer
  std::vector<std::pair<const void*, std::pair<double, double>>> ritz_cache;
  std::vector<double> wS;
  std::vector<double> w6;             // M x 9
  double* comm6 = nullptr;
  double e_min = 0, e_max = 0, beta = 0, dE = 0, R = 0;
  std::vector<double> weights;        // a_l = (2 - delta_l0) J_l(R), l = 0..L
  std::vector<double> coef;           // c_l = (2 - delta_l0) (-i)^l J_l(R), interleaved
  double phr = 1, phi = 0;            // exp(-i beta h), and what the doubles leave of it
  double phr_lo = 0, phi_lo = 0;
  // device
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  long np = 0;                        // padded dimension (dense)
  // dense planes
  double *h0r = nullptr, *h0i = nullptr, *vr = nullptr, *vi = nullptr, *kr = nullptr, *ki = nullptr;
  double *htr = nullptr, *hti = nullptr;
  double *xr = nullptr, *xi = nullptr, *yr = nullptr, *yi = nullptr;
  double *par = nullptr, *pai = nullptr, *pbr = nullptr, *pbi = nullptr;
  void* htx = nullptr;                // mixed builds: rescaled H in the product format
  double* pcr = nullptr;              // mixed builds: a third P buffer (format changes)
  std::vector<int> term_fmt;          // mixed builds: TermFmt of terms 1..L (index 0 unused)
  double mixed_err_est = 0.0;         // the schedule's estimate of the error it adds to U_T
  MixedPoly mpoly;                    // split-BF16 step polynomial (s = 0: none)
  double* tape = nullptr;             // checkpoints, each 2 planes
  int n_tape = 0;
  // gradient: per segment step X_{k-1}, P_{L-1}, P_L; two stacks; Lambda; d/da, d/db per step
  double* seg = nullptr;
  long seg_mats = 0;                  // ... of this many matrices (also for step polynomials)
  double* adj_pool = nullptr;         // tape and seg as adj_mats matrices (the sweep in segments)
  long adj_mats = 0;
  double* stack[2] = {nullptr, nullptr};
  double* lam = nullptr;
  double* d_grad = nullptr;
  float* drive32 = nullptr;           // FQ_FP32 gradient: the drive block in FP32 planes
  bool adj_f32 = false;               // reverse-sweep products on FP32 matrix cores
  double* save_pl = nullptr;          // when set, a step also stores P_L and P_{L-1} here
  double* save_plm1 = nullptr;
  // FP64 step operators: the matrices of H_eff (weights per step in d_w) and
  // scratch beyond the planes above. pool: pool_mats matrices for the segments
  // of a build run as one batch; extra: further matrices of a single step.
  std::vector<std::pair<const double*, const double*>> heff_ops;
  std::vector<int> heff_slot;
  double* d_w = nullptr;  // null: the weights go with the launches (PLAN_LEAN)
  int w_stride = 0;
  double* pool = nullptr;
  int pool_mats = 0;
  double* extra = nullptr;
  int n_extra = 0;
  bool from_identity = false;         // the running build starts at X = 1
  double* small = nullptr;            // 64 doubles of reduction scratch
  double* d_ab = nullptr;             // 2*M
  double* d_coef = nullptr;           // 2*(L+1)
  double* d_gauge = nullptr;          // tridiagonal: M x n complex gauge factors
  // tridiagonal gradient of resident columns: segments (their operators stay in
  // pool after a build), how many at a time, steps of the store, theta' rows
  int adj_seg = 0, adj_group = 0, adj_len = 0;
  double* adj_store = nullptr;
  double* d_theta = nullptr;
  double* d_tab = nullptr;            // tridiagonal: rows of every step (resident columns)
  double* d_fgrid = nullptr;          // tridiagonal: the period average's drive samples
  double* d_etab = nullptr;           // tridiagonal averages: operator rows in lane order
  double* d_stream = nullptr;         // tridiagonal n > resident size: two 8-plane states
  double* d_adj = nullptr;            // streamed reverse sweep: 10 complex n x n vectors
  double* d_vec = nullptr;            // 3 n doubles: period-average accumulators
  // state
  bool tape_valid = false;
  bool broken = false;
  fq_report last{};
  // profile mode: one event before every launch of a build (and one after the
  // last); launch i took the time between events i and i+1.
  bool profile = false;
  bool reortho = false;               // polar factor of U_T after the build
  bool small_chain = true;            // np = 64 FP64 steps in one launch (small_chain_kernel)
  bool c64 = false;                   // user state blocks (U, X, W, snapshots) in complex64
  void* snap = nullptr;               // propagate: snapshot buffer, every snap_every steps
  int snap_every = 0, snap_k0 = 0;
  long snap_ncols = 0;
  std::vector<hipEvent_t> events;
  std::vector<int> event_kind;
  size_t n_events = 0;
  // device time of a whole build (ms_build); off for the allocation-free
  // one-shot build, which creates no events
  bool timed = true;
  hipEvent_t build_ev[2] = {nullptr, nullptr};
  ~fq_ctx() {
    for (hipEvent_t e : events) (void)hipEventDestroy(e);
    for (hipEvent_t e : build_ev)
      if (e) (void)hipEventDestroy(e);
  }
};
