// Device-side structures and launch wrappers shared by the HIP translation
// units.  Every kernel works on a batch of instances (a single solve is a
// batch of one): per-instance pointers live in an InstPtrs array and the
// per-instance interior-point decisions in a Ctl block, both in device memory,
// so that a pass of the method needs no host decision and can be captured as a
// graph.  Each kernel file exposes plain host launch functions so no kernel
// symbol crosses a translation unit.
#ifndef NMPC_KERNELS_H
#define NMPC_KERNELS_H

#include <hip/hip_runtime.h>
#include <cstdint>

#include "../../include/nmpc.h"
#include "distill_layout.h"
#include "front_rules.h"
#include "plate_layout.h"
#include "reflux_layout.h"
#include "report.h"

namespace nmpc {

constexpr int kBlock = 256;          // threads per block of every vector kernel
constexpr int kFactorBlock = kSolveThreads;   // threads per supernode group of the solves
constexpr int kPanel = 8;            // columns per blocked step of a forward solve
constexpr int kMaxQ = 12;            // reduced quantities per phase
constexpr int kMaxSeed = 16;         // controls per stage the sensitivity seed can hold
constexpr int kFilterCapMax = 256;   // filter entries an instance can hold

struct DistillConst {
    double dt, alpha, F, rho;
};

// Stage-model family: constants its generated kernels read.  tag names the
// kernels meant for the instance; pc is null when the state rows hold the
// previous states with coefficient -1 each (implicit Euler), else the nx x nx
// coefficient matrix (row-major) of the previous states in the state rows.
struct StageConst {
    double dt;
    unsigned long long tag;
    const double* pc;
    double* scratch;   // H x (the model's per-stage scratch) doubles, or null
};

// Per-supernode read-only symbolic data of one instance.
// What the extend-add of one child reads:
// its update block (u_off), its rows' positions in the parent (rel_off), its
// update vector (uv_off) and its number of rows below its columns (nc).
struct ChildRec {
    int64_t u_off, rel_off, uv_off;
    int32_t nc, child;
};

struct SnView {
    const int64_t* rows_ptr;
    const int32_t* rows;
    const int32_t* child_ptr;
    const ChildRec* child_rec;    // the children of supernode s from child_ptr[s]
    const int64_t* uv_off;
    const int32_t* rel;
    const int32_t* k_fpos;
    // children of the large supernodes (factorization or solves): entries of row
    // and column j are [big_ptr[big_col[s] + j], big_ptr[big_col[s] + j + 1])
    const int32_t* big_col;
    const int32_t* big_ptr;
    const struct BigEntry* big_ent;
    const int32_t* chunk_pos;
};

// Phases of one Newton iteration of Algorithm 2 for one instance:
//   A  evaluate, optimality errors, convergence test, barrier update
//   B  condensed assembly (eqs. 14, 17), then the first factorization (eta = 0)
//   F  factorization retried with a larger eta (inertia correction)
//   S  solves (eqs. 22-25), remaining directions, fraction to the boundary (eq. 26)
//   T  one trial point of the backtracking line search
//   C  one second-order correction of the first trial point
//   U  accepted step: update, then as A for the next iteration
enum Phase : int { kPhA = 0, kPhB = 1, kPhF = 2, kPhS = 3, kPhT = 4, kPhC = 5, kPhU = 6, kPhDone = 7 };
// predicate values of the launch wrappers: a phase, or one of these
constexpr int kPredAll = -1;       // every instance, whatever its phase
constexpr int kPredFactor = 100;   // phases B and F
constexpr int kPredEval = 101;     // phases A and U: evaluation follows the update of the accepted instances

constexpr int kStatusRunning = -1;

// Interior-point state of one instance, read and written on the device.
struct Ctl {
    double mu, tau, alpha, eta, eta_last, f, E0, gamma;
    // filter line search: violation and barrier objective at the iterate, the
    // directional derivative of phi, the minimal step, the theta bounds and the
    // barrier value the filter belongs to
    double theta, phi0, dphi, amin, theta_max, theta_min, filter_mu;
    // second-order corrections: first trial step, last correction's step and violation
    double alpha0, soc_a, soc_theta;
    // l1-merit fallback: first step of the search, max |omega + d_omega| of the
    // direction, the penalty (kept over the solve)
    double amax0, om_max, nu;
    int ls_merit;        // the current search runs on the l1 merit
    int merit_trials;    // trial points of the merit search
    int filter_n;        // entries in the instance's filter
    int soc_p;           // corrections done in the current line search
    int use_soc;         // the accepted step is the correction's
    int status;          // kStatusRunning or a final nmpc status
    int phase;
    int it;              // accepted Newton steps
    int fail;            // set by the factorization: a pivot is not positive and finite
    int trials;          // trial points of the current line search
    int factorizations, ls_trials;
    // HyKKT (equalities kept exact, Newton system by the Cholesky factor of
    // K_gamma = K_c + hk_gamma J_c^T J_c and conjugate gradients on the Schur
    // complement): mode flag, and the running CG of the current step
    int hyk;
    int cg_it, cg_done, cg_total;
    double hk_gamma, cg_rr, cg_stop, cg_alpha, cg_beta;
    int exported, pad;   // the finished block is in pinned memory
};

// Where the device reports to the host without a copy or a wait for the stream:
// pinned words (report.h) that a kernel's last workgroup stores and the host
// polls, the reports numbered so that a stale one is told from the awaited one.
// cnt: device counters, zero before the first report.
constexpr int kRepCounters = 6;   // ticket, running, waiting, ended; reports of the passes, of the CG
struct Report {
    unsigned* cnt;
    unsigned long long* host;   // [0] passes, [1] conjugate gradients
    Ctl* ctl;                   // control blocks of finished instances, per instance
};

__host__ __device__ inline bool ctl_active(const Ctl* c, int pred) {
    if (pred == kPredAll) return true;
    const int ph = c->phase;
    if (pred == kPredFactor) return ph == kPhB || ph == kPhF;
    if (pred == kPredEval) return ph == kPhA || ph == kPhU;
    return ph == pred;
}

// Loads through a pointer in the global address space are global (not flat)
// instructions: they count only against the vector-memory counter, so waits
// for shared memory do not also wait for them.
typedef __attribute__((address_space(1))) double gdouble;
template <class T>
__device__ inline const __attribute__((address_space(1))) T* global(const T* p) {
    return (const __attribute__((address_space(1))) T*)p;
}
template <class T>
__device__ inline __attribute__((address_space(1))) T* global(T* p) {
    return (__attribute__((address_space(1))) T*)p;
}

// Everything a kernel needs to know about one instance.
struct InstPtrs {
    int family;
    int n, mc, md, ml, m, nx, nu, H;
    int64_t nnzk;
    DistillDims dd;
    DistillConst dc;
    PlateDims pd;
    PlateConst pc;
    RefluxDims rd;
    RefluxConst rc;
    StageConst gm;
    int ns, rps;        // variables and (dynamics block) equality rows per stage
    int nsp, ntr;       // setpoint and disturbance-trajectory lengths of the family
    // structure
    const int32_t *jptr, *jcol, *jt_ptr, *jt_slot, *jt_row;
    const double *lb, *ub;
    const int32_t* perm;
    SnView S;
    const int32_t *k_wslot, *k_diag, *kc_ptr, *kc_a, *kc_b, *kc_r;
    // parameters
    const double *x0, *zF, *uprev, *setp;
    // iterate and work vectors
    double *y, *s, *om, *be, *zl, *zu;
    double *c, *d, *jv, *wv, *grad, *fterm, *gtw, *sig, *rhs, *dy, *xp;
    double *Q, *r2, *r4, *qeff, *vcomb;
    double *ds, *dom, *dbe, *dzl, *dzu, *yt, *st;
    // second-order correction: r1 of the step, corrected residual and its
    // row combinations, right-hand side and directions
    double *r1v, *r4s, *vcomb_s, *rhs_s, *dy_s, *ds_s, *dom_s, *dbe_s, *dzl_s, *dzu_s;
    double *kv, *L, *U, *uvec;
    double *adj_rhs, *adj_w, *adj_out, *adj_b, *adj_d, *adj_lam, *adj_qr;
    double* adj_seed;   // seed of the sensitivities: u1 part (nu values), then the objective's
    const int32_t *wf_ptr, *wf_slot, *wf_col;   // Hessian rows, both triangles: (slot, column)
    const int32_t* kcol_ptr;   // KKT slots of each permuted column: [kcol_ptr[j], kcol_ptr[j + 1])
    double* dfac;     // factored diagonal blocks on their way into the panels: kBigDiag doubles per large front of a level
    double* bsum;     // large-supernode backward solves: rows-below products per column
    double* part;     // reduction partials: kMaxQ rows of this instance's blocks
    double* filter;   // (theta, phi) pairs, kFilterCapMax of them
    // HyKKT: CG iterate, residual, direction and S-product over the equality
    // rows (m_c each); J_c^T p and its solve with the factor (n each)
    double *hk_x, *hk_r, *hk_p, *hk_sp, *hk_t, *hk_w;
    Ctl* ctl;
};

// Layout check between the library and the code objects of generated stage
// models (both read InstPtrs): the library refuses a code object whose
// nmpc_stage_abi differs.
constexpr unsigned int kStageAbiVersion = 2;
constexpr unsigned int kStageAbi = kStageAbiVersion * 100000u + (unsigned int)sizeof(InstPtrs);

// Right-hand side and solution of the solves: 0 rhs -> dy (Newton step),
// 1 yt -> dzl (single-solve entry point), 2 adj_rhs -> adj_w (sensitivities),
// 3 adj_rhs -> adj_d (refinement corrections of the sensitivities),
// 4 rhs_s -> dy_s (second-order correction), 5 hk_t -> hk_w (HyKKT products
// with K_gamma^{-1}).
__host__ __device__ inline const double* solve_in(const InstPtrs& I, int which) {
    return which == 0 ? I.rhs : (which == 1 ? I.yt : (which == 4 ? I.rhs_s : (which == 5 ? I.hk_t : I.adj_rhs)));
}
__host__ __device__ inline double* solve_out(const InstPtrs& I, int which) {
    return which == 0 ? I.dy
                      : (which == 1 ? I.dzl
                                    : (which == 2 ? I.adj_w : (which == 3 ? I.adj_d : (which == 5 ? I.hk_w : I.dy_s))));
}

// Block -> instance map of one index space.  Instance i owns blocks
// [bfirst[i], bfirst[i + 1]); binst[b] is the instance of block b.
struct Space {
    const int32_t* binst;
    const int32_t* bfirst;
    int blocks;
};
enum SpaceKind : int { kSpN = 0, kSpNML = 1, kSpM = 2, kSpK = 3, kSpMN = 4, kSpMax = 5, kNumSpaces = 6 };
// size of an instance in each space
__host__ __device__ inline int64_t space_size(const InstPtrs& I, int kind) {
    switch (kind) {
        case kSpN: return I.n;
        case kSpNML: return (int64_t)I.n + I.ml;
        case kSpM: return I.m;
        case kSpK: return I.nnzk;
        case kSpMN: return (int64_t)I.m + I.n;
        default: return I.n > I.ml ? I.n : I.ml;
    }
}

// Instance of the calling block and the block's index within that instance.
__device__ inline int block_inst(const Space& sp, int& local_block) {
    const int i = sp.binst[blockIdx.x];
    local_block = (int)blockIdx.x - sp.bfirst[i];
    return i;
}

// Interior-point constants the device decisions use.
struct DevOpts {
    double tol, mu_min, kappa_eps, kappa_mu, theta_mu, tau_min, armijo, kappa_sigma;
    double eta_first, eta_min, eta_max, kp_first, kp, km;
    double g_theta, g_phi, s_theta, s_phi, delta, amin_frac, theta_max_fact, theta_min_fact, soc_kappa;
    int ls_max, max_iter, filter_cap, soc_max, merit_fallback, fixed_mu;
    double cg_tol;
    int cg_max;
};

// One supernode of a one-workgroup launch, its sizes and operands by absolute
// address, so that a workgroup reads its record and then its data.  A launch's
// array holds the first supernode of every workgroup, then the others, each
// pointed to by its predecessor (next, 0 at the end).
struct alignas(64) FactorTask {
    Ctl* ctl;
    double* L;             // its panel
    double* U;             // its update block
    double* xp;            // at its first column
    const int32_t* perm;   // at its first column
    const double* kv;      // its slots of the condensed matrix (nk) and their places
    const int32_t* fpos;
    const double* rhs;
    const double* Uall;    // the update blocks, update vectors and relative rows of all
    double* uvec;
    const int32_t* rel;
    const ChildRec* recs;  // its children (nchild)
    int64_t uv;            // its update vector; < 0: its forward solve is not fused
    int32_t w, m, nk, nchild, next, pad;
    ChildRec rec0, rec1;   // its first two children
};
// The solves run over other work vectors too (InstPtrs inst of the launch).
struct alignas(64) SolveTask {
    const Ctl* ctl;
    const double* L;
    const int32_t* rows;
    const int32_t* perm;   // at its first column
    int32_t f, w, m, inst, sn, next;
};

// ---- model evaluation (kernels_model.hip) -------------------------------------------
// Source of the point and multipliers: the iterate (y, om), the trial point
// (yt; values only), or a caller-given point staged in (yt, dom).
enum EvalSrc : int { kSrcIter = 0, kSrcTrial = 1, kSrcUser = 2 };
// full: c, d, Jacobian values, Lagrangian Hessian values, gradient and objective
// terms; otherwise c, d and objective terms.  Space kSpN, one lane per variable.
void launch_eval_distill(bool full, int src, int pred, const InstPtrs* I, const Space& sp, hipStream_t st);
void launch_eval_plate(bool full, int src, int pred, const InstPtrs* I, const Space& sp, hipStream_t st);
void launch_eval_reflux(bool full, int src, int pred, const InstPtrs* I, const Space& sp, hipStream_t st);

// ---- interior-point vector kernels and decisions (kernels_ipm.hip) ----------------
struct IpmSpaces {
    Space sp[kNumSpaces];
};
void launch_phaseA(const InstPtrs* I, const IpmSpaces& S, int ninst, int pred, const DevOpts& o, bool decide,
                   const Report& rep, hipStream_t st);
void launch_assemble(const InstPtrs* I, const IpmSpaces& S, int pred, hipStream_t st);
void launch_decideF(const InstPtrs* I, int ninst, const DevOpts& o, hipStream_t st);
void launch_phaseE(const InstPtrs* I, const IpmSpaces& S, int ninst, const DevOpts& o, hipStream_t st);
void launch_trial(const InstPtrs* I, const IpmSpaces& S, hipStream_t st);
void launch_phaseT(const InstPtrs* I, const IpmSpaces& S, int ninst, const DevOpts& o, hipStream_t st);
// second-order correction, before its solve (rows, right-hand side) and after
// it (directions and step bound, trial point), then its acceptance test
void launch_soc_prepare(const InstPtrs* I, const IpmSpaces& S, hipStream_t st);
void launch_soc_step(const InstPtrs* I, const IpmSpaces& S, int ninst, hipStream_t st);
void launch_soc_decide(const InstPtrs* I, const IpmSpaces& S, int ninst, const DevOpts& o, hipStream_t st);
// update of the accepted instances (the evaluation after it starts their next iteration)
void launch_update(const InstPtrs* I, const IpmSpaces& S, const DevOpts& o, hipStream_t st);
void launch_cold_start(const InstPtrs* I, const IpmSpaces& S, double bound_push, double slack_push, double mu0,
                       bool after_eval, hipStream_t st);
// HyKKT step (instances in phase S with the HyKKT flag): CG start after the
// solve of the right-hand side, one CG iteration as J_c^T p (pre), the solve
// hk_t -> hk_w that the caller enqueues, and the rest of the iteration (post);
// both write the number of instances whose CG still runs to *count.  finish:
// the right-hand side of the final solve.  from_lifted: convert the held
// Lifted-KKT iterate.
void launch_hk_cg_start(const InstPtrs* I, const IpmSpaces& S, int ninst, const DevOpts& o, const Report& rep,
                        hipStream_t st);
void launch_hk_cg_pre(const InstPtrs* I, const IpmSpaces& S, hipStream_t st);
void launch_hk_cg_post(const InstPtrs* I, const IpmSpaces& S, int ninst, const DevOpts& o, const Report& rep,
                       hipStream_t st);
void launch_hk_finish(const InstPtrs* I, const IpmSpaces& S, hipStream_t st);
void launch_hk_from_lifted(const InstPtrs* I, const IpmSpaces& S, hipStream_t st);
// shifted warm start: every stage-indexed quantity of the held iterate moves
// one stage earlier, the last stage keeps its own
void launch_shift(const InstPtrs* I, const IpmSpaces& S, hipStream_t st);
void launch_set_fail(const InstPtrs* I, int ninst, int value, hipStream_t st);
// sensitivities: rhs = seed_obj grad f + S_u^T seed_u, and the parameter contractions
void launch_adj_seed(const InstPtrs* I, const Space& spN, hipStream_t st);   // seed from adj_seed
void launch_cold_guess(const InstPtrs* I, const Space& spN, hipStream_t st);
// lam = omega+ - omega- and the inequality multipliers of instance 0 into caller buffers (NULL skips)
void launch_export_duals(const InstPtrs* I, double* lam, double* om_d, int rows, hipStream_t st);
// out = [x0 (nx) | setpoint (nsp) | trajectory (ntr) | u_prev (nu)] for instance 0
void launch_adj_gather(const InstPtrs* I, int family, int nx, hipStream_t st);
void launch_x0_map(const double* lam, int64_t stride, const double* pc, double* out, int nx, int K, hipStream_t st);
// Refinement of w = K^{-1} b against the uncondensed system [K0 J^T; J -Q^{-1}]
// (K0 = W + Sigma + eta I): start sets lam = Q J w; residual forms
// adj_rhs = b - K0 w - J^T lam + J^T qr with qr = lam - Q J w; update adds the
// correction adj_d: w += d, lam += Q J d - qr.
void launch_adj_refine(int step, const InstPtrs* I, const IpmSpaces& S, double eta, hipStream_t st);

// ---- numeric factorization and solves (kernels_linalg.hip) -------------------------
// Multifrontal Cholesky (eqs. 20-21) of a list of groups, one workgroup per
// group, for instances matching pred (kPredFactor during a solve) with eta
// from the control block, or every instance with eta_force (pred kPredAll).
// The fronts stay in shared memory (lds_bytes).
// variant: threads per workgroup, kFactorThreads (the same arithmetic).
constexpr int kFactorVariants = sizeof(kFactorThreads) / sizeof(kFactorThreads[0]);
constexpr int kFactorReplace = kFactorVariants;   // a pivot that is not positive and finite counts as 1, unreported
void launch_factor_groups(int variant, int pred, double eta_force, const FactorTask* t, int groups, size_t lds_bytes,
                          hipStream_t st);
void launch_fwd_groups(int pred, int which, const InstPtrs* I, const SolveTask* t, int groups, size_t lds_bytes,
                       hipStream_t st);
void launch_bwd_groups(int pred, int which, const InstPtrs* I, const SolveTask* t, int groups, size_t lds_bytes,
                       hipStream_t st);
// Raise the dynamic shared-memory limit of the front kernels (once per process).
hipError_t linalg_configure(size_t max_lds_bytes);

// ---- large supernodes (kernels_big.hip) ---------------------------------------------
constexpr int kBigPanel = 64;   // pivot columns per panel step of a large front
constexpr int kBigOuter = 512;  // columns per outer panel (one trailing update each)
constexpr int kBigChunk = 1024; // rows of a column one wave assembles
// One column of a child's update block among the columns a large front's column
// takes up, in child order: where the child's column starts in U, the child's
// row positions in rel (its update vector starts at the same offset of uvec),
// the column's index in the child, the child's rows, and the place in
// chunk_pos of the child's first row at or past every multiple of kBigChunk.
struct BigEntry {
    int64_t u_col, rel_off;
    int32_t jc, nc, chunk, pad;
};
constexpr int kBigDiag = kBigPanel * kBigPanel + kBigPanel;   // doubles of a factored diagonal block kept aside
// One workgroup's share of a step: the front's storage and sizes, then what the
// kind below names (a, b).  slot: the front's place in the instance's dfac.
struct BigTask {
    double *L, *U;        // panel (m x w), update block ((m - w) x (m - w))
    int64_t uv;           // update vector of the front, an offset into uvec
    int32_t inst, sn, a, b;
    int32_t f, w, m, fused;
    int32_t slot, pad;
};
static_assert(sizeof(BigTask) == 64, "one scalar load of 16 words");
enum BigKind : int {
    kBigAssemble = 1,   // a: first of kBigAsmCols columns, b: chunk of rows
    kBigPanelStep = 3,  // a: kb, b: row block
    kBigPanelReplace = 4,  // the same, a pivot that is not positive and finite counts as 1
    kBigUpdate = 5,     // a: kb, b: lower-triangle tile; b < 0: keep the diagonal block of columns a
    kBigFwdGather = 2,  // a: row block
    kBigFwdTri = 6,     // a: chunk
    kBigFwdGemv = 7,    // a: chunk, b: row block
    kBigBwdBelow = 8,   // a: column block
    kBigBwdTri = 9,     // a: chunk
    kBigUpdateInner = 10,  // a: ki, b: rectangular tile; b < 0: keep the diagonal block of columns a
    kBigBwdGemvT = 11   // a: chunk, b: column block
};
// One step for every task of a list (predicate and eta as for the groups;
// which selects the solve vectors).
void launch_big(int kind, int pred, double eta_force, int which, const InstPtrs* I, const BigTask* tasks, int count,
                hipStream_t st);
constexpr int kBigAsmCols = 4;   // columns per workgroup of the assembly, one per wave
int big_row_block();
int big_gather_rows();   // rows per workgroup of the forward gather
int big_tile();
int big_solve_rows();
int big_solve_cols();
int big_chunk();   // columns per chunk of a large supernode's solves

}  // namespace nmpc

#endif
