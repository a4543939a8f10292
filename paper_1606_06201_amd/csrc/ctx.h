// Library context: grid hierarchy, device buffers and the per-dimension kernel set.
#pragma once
#include "common.h"

namespace ipmg {

struct Ctx;

// Device memory of a context, given back when the context goes.  Buffers of less
// than 1 MB are cut from slabs of 4 MB instead of being allocations of their own:
// a small grid's kernels touch dozens of them, and each allocation is at least one
// page of its own to translate.
struct Arena {
  static constexpr size_t SLAB = (size_t)4 << 20, SMALL = (size_t)1 << 20, ALIGN = 256;
  std::vector<void*> blocks;
  char* slab = nullptr;
  size_t used = SLAB;
  void* raw(size_t bytes) {
    void* p = nullptr;
    blocks.reserve(blocks.size() + 1);
    if (hipMalloc(&p, bytes) != hipSuccess) {
      (void)hipGetLastError();                        // reported here, not by the next launch's check
      throw Error(IPMG_E_NOMEM, "device allocation failed");
    }
    blocks.push_back(p);
    return p;
  }
  void* alloc(size_t bytes) {
    bytes = (bytes + ALIGN - 1) / ALIGN * ALIGN;
    if (bytes == 0) bytes = ALIGN;
    if (bytes >= SMALL) return raw(bytes);
    if (used + bytes > SLAB) {
      slab = (char*)raw(SLAB);
      used = 0;
    }
    void* p = slab + used;
    used += bytes;
    return p;
  }
  // Memory for p unless it has some: what a call allocates on first use is asked for one
  // buffer at a time, so that a call after one that ran out of memory goes on with the
  // first buffer that is missing.
  template <typename P>
  void need(P*& p, size_t bytes) {
    if (!p) p = (P*)alloc(bytes);
  }
  void release() {
    for (void* p : blocks) (void)hipFree(p);
    blocks.clear();
    slab = nullptr;
    used = SLAB;
  }
};

// Level arrays (precision of the V-cycle, T = float or double).
struct Level {
  Dims d;
  void* r = nullptr;    // right-hand side of the level problem (n_slots + 1)
  void* z = nullptr;    // current iterate
  void* z2 = nullptr;   // Jacobi ping-pong partner
  void* t = nullptr;    // residual
  void* E = nullptr;    // coarse element matrices (NSYM * m), levels below the finest
  double* E64 = nullptr;// the same in FP64: the Galerkin chain is formed in FP64 (aliases E in FP64 mode)
  void* S = nullptr;    // node stencil (stencil.h), and the reciprocal diagonal per slot
  void* dinv = nullptr;
  void* bZ = nullptr;   // border vector of Z on this level (n_slots)
  double* bZ64 = nullptr;// the same in FP64 (aliases bZ in FP64 mode)
};

// Lambda entry of a level vector that its producer left as partials of b'v (see
// LamRef in kernels.h): the fields of the reference without its type.
struct LamPend {
  int kind = 0;
  const void* value = nullptr;
  const void* r = nullptr;
  const double* omg = nullptr;
  const double* part = nullptr;
  unsigned nb = 0;
};

// Passes of a level in node-stencil form (the kernels' StenMode).
enum StenPass { SP_JACOBI2 = 0, SP_JACOBI = 1, SP_RESID = 2, SP_BETA = 3 };
// Sizes of 2D levels where their passes change: from the first one on register-blocked
// tiles, below the second one fused passes that stage the element matrices in LDS.
// First one: 20 PCG steps on K with it at 2^16 / 2^17 / 2^18 nodes, ms: FP32 512x256 2.11 / 2.10 /
// 2.52, 704x352 2.38 / 2.37 / 2.79; FP64 3.04 / 3.03 / 3.61 and 3.43 / 3.37 / 4.05.  Tiles gain below
// it too, from 2^16 on: 400x200 1.52 / 1.91 / 1.90 in FP32, 2.07 / 2.30 / 2.30 in FP64, 384x176 (68145
// nodes) 1.91 / 2.24 / 2.25 in FP32.
constexpr int64_t TILED_MIN_NODES = (int64_t)1 << 17, STAGED_MAX_NODES = (int64_t)1 << 16;
// Largest order of the coarsest solve inside the one-workgroup V-cycle (its threads).
constexpr int TAIL_MAX_LD = 512;

// Kernel set of one dimension (implemented for 2 and 3 in ops2d.hip / ops3d.hip).
struct Ops {
  virtual ~Ops() {}
  virtual void element_stiffness(Ctx& c, double* dK0) = 0;           // into device buffer
  // Constants of the context's material: formed once from its element matrix, and
  // copied to the constant memory of the current device.
  virtual void form_constants(Ctx& c, const double* K0) = 0;
  virtual void load_constants() = 0;
  // One level pass (see LevelMode) on level lev with operator op.
  // omg: device pointer to the damping weight (Jacobi modes); sidx/sidx_in: scalar
  // slots of the mode's reductions.
  virtual void level(Ctx& c, int lev, int op, int mode, const void* v, const void* r, void* out,
                     const double* omg, int sidx, int sidx_in, const int* gate, const double* dot64 = nullptr) = 0;
  // p = -y + beta p_old; q = A p (FP64, finest level); alpha = rho / p'q on the device.
  // zs (only where dir_folds_solution): the previous step's solution update
  // zs += alpha p_old is done in the same pass when flags[F_ZPEND] is set, also
  // after the solve has stopped (gate set).
  virtual void dir_apply(Ctx& c, int op, const void* y, const double* pold, double* p, double* q, int first,
                         const int* gate, double* zs = nullptr) = 0;
  virtual bool dir_folds_solution(const Ctx& c) const = 0;
  // FP64 operator on the finest grid (PCG operator), y = A v.
  virtual void fine_apply64(Ctx& c, int op, const double* v, double* y, const int* gate) = 0;
  virtual void restrict_to(Ctx& c, int lev_f, const void* rf, void* rc, int aug, const int* gate) = 0;
  virtual void prolong_from(Ctx& c, int lev_f, void* z, const void* zc, int aug, const int* gate) = 0;
  // out = one Jacobi sweep from z2 + P zc on level lev (prolongation folded into the
  // sweep); false when that pass does not apply.
  virtual bool prolong_jacobi(Ctx& c, int lev, int op, const void* z2, const void* zc, const void* r, void* out,
                              const double* omg, const int* gate) = 0;
  // out = the first two damped-Jacobi sweeps from a zero iterate on level lev, in
  // one pass; false when that pass does not apply.
  virtual bool jacobi2(Ctx& c, int lev, int op, const void* r, void* out, const double* omg, const int* gate) = 0;
  // As jacobi2, and t = r - A out in the same pass; false when that pass does not apply.
  virtual bool jacobi2_resid(Ctx& c, int lev, int op, const void* r, void* out, void* t, const double* omg,
                             const int* gate) = 0;
  // out = z2 + P zc followed by two damped-Jacobi sweeps, in one pass (dot64: the
  // last sweep also accumulates the PCG ratio's partial sums, as M_JACOBI_BETA, and
  // its finalize follows); false when that pass does not apply.
  virtual bool prolong_jacobi2(Ctx& c, int lev, int op, const void* z2, const void* zc, const void* r, void* out,
                               const double* omg, const int* gate, const double* dot64) = 0;
  virtual void restrict64(Ctx& c, int lev_f, const double* rf, double* rc) = 0;    // border vectors
  virtual void galerkin(Ctx& c, int lev_f, int op) = 0;              // E64 of level lev_f-1
  virtual void dense_assemble(Ctx& c, int op, double* A, int n) = 0;
  virtual void power_start(Ctx& c, int lev, int aug, void* v) = 0;
  // Levels in node-stencil form (stencil.h).
  //   sten_level: the level's passes run on its stencil; tail_level: the highest
  //   level of the one-workgroup V-cycle (0: none); needs_elements: the level's
  //   passes read the element matrices in V-cycle precision.
  virtual bool sten_level(const Ctx& c, int lev, int op) const = 0;
  virtual bool pow_level(const Ctx& c, int lev, int op) const = 0;   // damping estimated on the stencil
  virtual int tail_level(const Ctx& c, int op) const = 0;
  virtual bool needs_elements(const Ctx& c, int lev, int op) const = 0;
  // Stencils and the damping of every level above.
  virtual void sten_setup(Ctx& c, int op) = 0;
  virtual void sten_damping(Ctx& c, int op, int steps, double product) = 0;
  // One pass (StenMode) over lev from v (lambda entry in) to out; returns how out's
  // lambda entry is found.  sten_jacobi0: the first sweep from zero alone.
  virtual LamPend sten_pass(Ctx& c, int lev, int op, int mode, void* v, const void* r, void* out, const LamPend& in,
                            const int* gate, const double* dot64) = 0;
  virtual void sten_jacobi0(Ctx& c, int lev, int op, const void* r, void* out, const int* gate) = 0;
  virtual bool sten_fuses_two(const Ctx& c, int lev, int op) const = 0;
  virtual void lam_store(Ctx& c, const LamPend& p, void* out, const int* gate) = 0;
  // V-cycle of levels 0..tail_level: lev.r -> lev.z of that level.
  virtual void tail(Ctx& c, int op, const int* gate, const double* beta64) = 0;
  // Fused passes of level lev (see fused2d.h): false when they do not apply.
  //   down: lev.r -> z2 (into z), coarse residual (into lev-1 .r)
  //   up:   z2 (in z), coarse correction zc -> out
  virtual bool fused_applies(const Ctx& c, int lev, int op) const = 0;
  // The fused down pass of lev forms its r as P' t from the finest residual t
  // (passed in Ctx::down_from_t) instead of reading a restricted one.
  virtual bool down_restricts(const Ctx& c, int lev, int op) const = 0;
  virtual void fused_down(Ctx& c, int lev, const int* gate) = 0;
  virtual void fused_up(Ctx& c, int lev, const void* zc, void* out, const int* gate) = 0;
  virtual void element_sens(Ctx& c, const double* w, const double* u, double scale, double* g) = 0;
  // 3D finest level: the diagonal of the hierarchy's operator per DOF slot (V-cycle
  // precision), formed once per set-up (no-op elsewhere)
  virtual void fine_diag(Ctx& c, int op) = 0;
  // SIMP model (Sec. 9): the density filter (mode 0: out = W in, 1: W' in, 2: W2 in
  // with (W2)_ji = W_ji^2; 3, 4: its scaled halves, see FilterMode, with x), and
  // x~^p / p x~^(p-1) E
  virtual void filter(Ctx& c, double rmin, const double* in, double* out, int mode, const double* x = nullptr,
                      const int* gate = nullptr) = 0;
  virtual void simp_pow(Ctx& c, const double* xt, double p, double* xp, double* q) = 0;
  // Interior-point method on the SIMP model (Sec. 9), see the kernels in ops_impl.h:
  //   elem: g_e = K0 u_e, E_e = u_e'g_e;  design: F3 from the filtered energy term t,
  //   G3, w = 1/D (ipG3, ipW) and the sums of ip_elements;  coef: border/rhs
  //   coefficients, the lumped rank-one factors h64/hT and their corner
  //   (scal[S_TMP7]);  nodes: F1, border bZ64, right-hand side;  gather: y_u +=
  //   sum coef_e g_e + b v_lambda;  recover: d_x, d_phi, d_psi, step length.
  virtual void simp_elem(Ctx& c, const double* u, double* g, double* E) = 0;
  virtual void simp_design(Ctx& c, const double* t, const double* x, const double* phi, const double* psi,
                           double lam, double s, double r, double xbar) = 0;
  virtual void simp_coef(Ctx& c, const double* cf, const double* Ww, const double* WGw, const double* W2w,
                         const double* g, double* bcoef, double* rcoef) = 0;
  virtual void simp_nodes(Ctx& c, const double* Ku, const double* f, const double* u, const double* g,
                          const double* bcoef, const double* rcoef, double* rhs) = 0;
  virtual void simp_dots(Ctx& c, const double* v, const double* g, const double* cf, double* a,
                         const int* gate) = 0;
  // returns the blocks whose partials of b'v_u and v_u'y_u it leaves
  virtual unsigned simp_gather(Ctx& c, const double* g, const double* coef, const double* v, double* y,
                               const int* gate) = 0;
  virtual void simp_recover(Ctx& c, const double* btdu, const double* du, const double* x, const double* phi,
                            const double* psi, double s, double r, double xbar, double frac, int all_blocks) = 0;
  // t_e = x_e (u_e'K0u_e)^q of the OC update (Sec. 4)
  virtual void oc_energy(Ctx& c, const double* u, const double* x, double q, double* t) = 0;
  // Interior point kernels (FP64).
  virtual void ip_elements(Ctx& c, const double* u, const double* x, const double* phi, const double* psi,
                           double lam, double s, double r, double xbar) = 0;
  virtual void ip_nodes(Ctx& c, const double* Ku, const double* f, const double* u, double* rhs) = 0;
  virtual void ip_recover(Ctx& c, const double* du, const double* x, const double* phi, const double* psi,
                          double s, double r, double xbar, double frac, int all_blocks) = 0;
  virtual void ip_update(Ctx& c, double* u, const double* du, double* x, double* phi, double* psi) = 0;
};

Ops* make_ops2d();
Ops* make_ops3d();

struct Ctx {
  Arena arena;
  ipmg_desc desc{};
  int device = 0;
  int dim = 2;
  bool fp32 = true;
  int L = 1;
  hipStream_t stream = nullptr;
  Ops* ops = nullptr;
  std::vector<Level> lev;      // lev[L-1] finest
  size_t tsz = 4;              // sizeof(T) of the V-cycle
  bool coarse_from_x = true;   // 2D K: first coarse level evaluated from the fine densities
  bool tiled2d = true;         // 2D level passes with register-blocked tiles
  int64_t tiled_min_nodes = TILED_MIN_NODES;   // ... on levels with at least this many nodes
  int nj32 = 4, nj64 = 2, nj_dir = 4;          // nodes per thread of the tiled passes
  bool fused2d = true;         // 2D K coarse levels: two fused launches per level
  bool fused_staged = true;    // ... with the element matrices staged in LDS (FP32 stored levels
  int64_t staged_max_nodes = STAGED_MAX_NODES;  // below this size)
  int cus = 256;               // compute units of the device
  bool mfma = true;            // first coarse level's fused passes on the matrix cores (FP32)
  bool lane_share = true;      // finest-level 2D passes of K on lane-shared tiles (neighbour columns by DPP)
  bool fuse_resid = true;      // ... and the residual formed in the pass of the two sweeps from zero
  bool fuse_post = true;       // ... and the prolongation and both post-sweeps in one pass
  bool fold_solution = true;         // PCG solution update folded into the next direction kernel
  bool fold_rn2_fin = true;          // PCG ||r||^2 finalize done by the V-cycle's first pass
  bool fold_restrict = true;         // finest residual restricted inside the first coarse down pass
  const void* down_from_t = nullptr; // ... the residual, pending for that pass
  bool tail_on = true;         // small levels' V-cycle in one workgroup
  bool sten2d = true;          // 2D levels on node stencils
  bool step_in_tail = false;   // the tail ends the PCG step (finest level in the tail) ...
  unsigned step_blocks = 0;    // ... whose direction kernel left this many blocks' partials
  int step_first = 0;
  LamPend lam_t, lam_z;        // lambda entries pending for the next restriction / prolongation
  int sten_par = 0;            // partial buffer of the next stencil pass
  double* pow_part = nullptr;  // partials of the batched damping estimate
  unsigned rn2_fin_blocks = 0;       // pending ||r||^2 finalize (partials of the update kernel) ...
  bool rn2_fin_zpend = false;        // ... and whether it marks z += alpha p pending
  bool fold_prolong = true;          // 2D tiled levels: prolongation folded into the first post-sweep, and
                                     // the finest level's first two pre-sweeps fused
  int power_steps = 12;        // power iterations of the damping estimate (K)
  int power_steps_z = 30;      // ... (augmented system Z)

  double K0[576] = {0};        // host copy of the element matrix
  int nd = 8;                  // DOFs per element

  // finest-level operator data
  double* x64 = nullptr;       // densities (m)
  void* xT = nullptr;          // V-cycle copy (aliases x64 in FP64 mode)
  double* h64 = nullptr;       // Z rank-one factors h_e (ND * m)
  void* hT = nullptr;
  void* hsbuf = nullptr;       // h_e'v_e per element (m values) for the 3D Z passes in gather form
  bool elem_hv = true;         // gather form of the 3D Z passes: form h_e'v_e per element first
  double* bZ64 = nullptr;      // border of Z on the finest grid (n_slots)
  double cZ = 0.0;             // corner of Z
  bool have_x = false;
  bool have_z = false;
  int hier_op = -1;            // operator the hierarchy currently holds (-1: none)

  // PCG work vectors (FP64, n_slots + 1)
  double *pr = nullptr, *pp = nullptr, *pq = nullptr, *pt = nullptr, *pb = nullptr, *pu = nullptr;
  double* pp2 = nullptr;       // second search-direction buffer (p is double-buffered)
  void* yT = nullptr;          // level buffer holding the last preconditioned residual

  // coarsest dense solve
  int ncoarse = 0;             // dense size incl. lambda (n_slots_coarse + 1)
  double *dA = nullptr, *dLi = nullptr, *dAi = nullptr;   // packed tiles: A (then L), L^-1, A^-1
  float* dAif = nullptr;       // A^-1 rounded to FP32 (FP32 V-cycle)
  double* dpart = nullptr;     // partial sums of the dense apply
  void* dfull = nullptr;       // A^-1 in full (V-cycle precision), for the one-workgroup V-cycle

  // per-level damping on the device: omega_dev[k] = weight, omega_dev[L + k] = rho estimate
  double* omega_dev = nullptr;

  // reductions / scalars
  Red red{};
  HostBox* box = nullptr;      // pinned host memory that kernels write ...
  double* hscal = nullptr;     // ... its scalars
  int* hflags = nullptr;       // ... and flags
  unsigned long long box_seq = 0;
  unsigned step_seq = 0;
  // Within a PCG iteration: the host slot that the iteration's last kernel (the
  // finalize of the fused PCG ratio) fills, and whether one did.
  FlagDst flag_dst;
  bool flag_written = false;
  FlagDst take_flag_dst() {
    const FlagDst p = flag_dst;
    if (p.p) flag_written = true;
    flag_dst = FlagDst{};
    return p;
  }

  // interior-point scratch (FP64, m or n_slots + 1)
  double *ipG3 = nullptr, *ipW = nullptr, *ipSW = nullptr, *ipDx = nullptr, *ipDphi = nullptr, *ipDpsi = nullptr;
  double *ipRhs = nullptr, *ipD = nullptr, *ipKu = nullptr;
  double ipV = 0.0;            // volume of the current interior-point problem

  std::string err;

  // 3D finest level: the set-up diagonal; for Z the displacements (0 on clamped
  // slots) whose K0 u_e, scaled by ipSW, is the rank-one factor h_e
  double* hu = nullptr;
  void* fine_dg = nullptr;
  bool elem_fine3 = true;

  // SIMP model: filtered densities and the penalised ones (m each)
  double* simp_xt = nullptr;
  double* simp_xp = nullptr;
  // SIMP interior point (Sec. 9): c = p x~^(p-1), g_e = K0 u_e (ND x m), E, work
  // vectors on the design variables, border/rhs coefficients
  double *simp_cf = nullptr, *simp_g = nullptr, *simp_E = nullptr, *simp_a = nullptr, *simp_t = nullptr;
  double *simp_b1 = nullptr, *simp_b2 = nullptr, *simp_b3 = nullptr, *simp_bcoef = nullptr, *simp_rcoef = nullptr;
  double simp_corner = 0.0;    // corner of the exact Newton matrix, sum w
  double simp_rmin = 0.0;      // > 0 during a solve with that matrix: PCG applies it in place of Z

  // OC update: t_e = x_e E_e^q (m) and the trial multipliers of a bisection pass
  double* oc_t = nullptr;
  double* oc_cand = nullptr;

  // this device's copy of the scratch array of the allocation-free PCG entry point
  unsigned char* noalloc_scratch = nullptr;

  // kernel timing (ipmg_profile_*): HIP event pairs around every launch of the
  // selected classes; prof_tag is the class of the next level pass
  unsigned prof_mask = 0;
  int prof_tag = -1;
  int prof_used = 0;
  std::vector<hipEvent_t> prof_ev;
  std::vector<int> prof_cls;

  const Dims& fine() const { return lev[L - 1].d; }
};

// Kernel classes timed by ipmg_profile_begin (bit k of the mask selects class k).
enum ProfClass {
  PC_FINE_JACOBI = 0,       // finest level, damped-Jacobi sweep from a nonzero iterate
  PC_DIR_APPLY = 1,         // FP64 finest-level apply of the PCG direction
  PC_FINE_RESID = 2,        // finest level, residual pass
  PC_PCG_UPDATE = 3,        // fused PCG vector update
  PC_SUB_JACOBI = 4,        // first coarse level, damped-Jacobi sweep from a nonzero iterate
  PC_FINE_JACOBI0 = 5,      // finest level, first sweep from a zero iterate
  PC_FINE_JACOBI_BETA = 6,  // finest level, last sweep with the fused PCG ratio
  PC_SUB_DOWN = 7,          // first coarse level, fused pre-smoothing + residual + restriction
  PC_SUB_UP = 8,            // first coarse level, fused prolongation + post-smoothing
  // 9 and 10: reserved (no kernel records them)
  PC_FINE_PJACOBI = 11,     // finest level, prolongation folded into the first post-smoothing sweep
  PC_FINE_JACOBI2 = 12,     // finest level, the first two pre-smoothing sweeps in one pass
  // 13 and 14: reserved (no kernel records them)
  PC_COUNT = 15
};

// Sets the class of the level passes enqueued in its scope.
struct ProfTag {
  Ctx& c;
  int old;
  ProfTag(Ctx& cc, int cls) : c(cc), old(cc.prof_tag) { c.prof_tag = cls; }
  ~ProfTag() { c.prof_tag = old; }
};

// Brackets the launch of one main kernel with a pair of events when its class is
// being timed (finalize kernels stay outside the bracket).
struct ProfScope {
  Ctx& c;
  bool on;
  int slot;
  ProfScope(Ctx& cc, int cls) : c(cc), on(false), slot(0) {
    if (cls >= 0 && ((c.prof_mask >> cls) & 1u) && 2 * (c.prof_used + 1) <= (int)c.prof_ev.size()) {
      on = true;
      slot = c.prof_used++;
      c.prof_cls[slot] = cls;
      (void)hipEventRecord(c.prof_ev[2 * slot], c.stream);
    }
  }
  ~ProfScope() {
    if (on) (void)hipEventRecord(c.prof_ev[2 * slot + 1], c.stream);
  }
};

// Timing of one launch by its own dispatch packet: the start and stop events of
// hipExtLaunchKernel (null when the class is not being timed).  The interval is
// the kernel's run alone, without the marker packets that a pair of hipEventRecord
// calls would place around the dispatch.
struct ProfLaunch {
  hipEvent_t t0 = nullptr, t1 = nullptr;
  ProfLaunch(Ctx& c, int cls) {
    if (cls >= 0 && ((c.prof_mask >> cls) & 1u) && 2 * (c.prof_used + 1) <= (int)c.prof_ev.size()) {
      const int slot = c.prof_used++;
      c.prof_cls[slot] = cls;
      t0 = c.prof_ev[2 * slot];
      t1 = c.prof_ev[2 * slot + 1];
    }
  }
};

// Host driver (solver.hip).
void ctx_init(Ctx& c, const ipmg_desc& d, hipStream_t st);
void ctx_free(Ctx& c);
void set_density(Ctx& c, const double* x);
void mg_setup(Ctx& c, int op, double* ms);
void* vcycle(Ctx& c, int op, const int* gate);    // lev[L-1].r -> returned level buffer
void vcycle64(Ctx& c, int op, const double* r, double* z);
int pcg(Ctx& c, int op, const double* b, double* u, double rtol, int maxit, ipmg_pcg_info* info);
// pcg with its work vectors and reduction scratch in the library's static device
// array (no allocation); needs the hierarchy of op set up.
int pcg_noalloc(Ctx& c, int op, const double* b, double* u, double rtol, int maxit, ipmg_pcg_info* info);
size_t pcg_noalloc_bytes(const Ctx& c);
void sync(Ctx& c);
// The context's material in the constant memory that its kernels read, for the life of
// the object: one array per process and device, shared by all contexts of a dimension.
// Calls of contexts with the same E and nu run side by side; a call with another
// material waits, in the order of arrival, until the calls before it have ended, and
// copies its own constants there.  A call leaves no kernel in flight when it ends.
struct MaterialUse {
  Ctx& c;
  int exceptions;
  explicit MaterialUse(Ctx& ctx);
  ~MaterialUse();
  MaterialUse(const MaterialUse&) = delete;
  MaterialUse& operator=(const MaterialUse&) = delete;
};
// Scalars and flags (and *extra) of the stream's work so far into hscal, hflags and
// box->extra; waits for them.
void read_scalars(Ctx& c, const double* extra = nullptr);
int ip_init(Ctx& c, const double* f, const ipmg_ip_params& p, ipmg_ip_state& st, ipmg_pcg_info* info);
void ip_prepare(Ctx& c, const double* f, const ipmg_ip_params& p, const ipmg_ip_state& st);
int ip_step(Ctx& c, const double* f, const ipmg_ip_params& p, ipmg_ip_state& st, ipmg_ip_info* info);
void oc_update(Ctx& c, const double* u, const double* x, double V, double xbar, double q, double lam_hi,
               double tau, const double* blend, double* x_new, ipmg_oc_info* info);
// Interior-point method on the SIMP model (Sec. 9): initial state (as ip_init with
// K^ in place of K) and one Newton step (as ip_step: the exact Newton matrix Z^
// applied matrix-free, PCG preconditioned by the V-cycle of the element-local
// approximation).
int simp_ip_init(Ctx& c, const double* f, const ipmg_ip_params& p, double rmin, double pexp, ipmg_ip_state& st,
                 ipmg_pcg_info* info);
int simp_ip_step(Ctx& c, const double* f, const ipmg_ip_params& p, double rmin, double pexp, ipmg_ip_state& st,
                 ipmg_ip_info* info);
int simp_compliance(Ctx& c, const double* x, const double* f, double rmin, double p, double rtol, int maxit,
                    double* u, double* grad, ipmg_pcg_info* info);

}  // namespace ipmg
