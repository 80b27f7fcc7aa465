// Numeric supernodal Cholesky and triangular solves (eqs. 20-25), multifrontal
// form: supernode s owns a dense front F_s of size m_s x m_s over its row list
// R_s (its w_s own columns first).  F_s starts from the KKT entries of its
// columns, receives the update blocks of its children by extend-add through
// precomputed relative positions, and is partially factored on its first w_s
// columns; the factored columns are the L panel (eq. 21 restricted to S_L) and
// the trailing block is the update passed to the parent.
//
// Scheduling: a launch covers a list of supernode groups; workgroup b factors
// the supernodes of group b one after another.  Wide levels of the supernodal
// tree are one group per supernode (one launch per level); the narrow top of
// the tree, where each level holds one or two supernodes, is a single group
// walked by one workgroup, so a chain of fronts costs one launch.  Every sum is
// taken in a fixed order, so results do not depend on scheduling.
#include <cmath>

#include "kernels.h"
#include "front_chol.h"

namespace nmpc {

namespace {

constexpr int kWave = 64;

__device__ inline double shfl(double v, int lane) { return __shfl(v, lane, kWave); }

constexpr int kBatch = 8;   // independent global loads in flight per thread

// Entry k of a read-only array, k the same in every lane of the launch's
// workgroup: a scalar load.  Sizes and offsets read this way stay in scalar
// registers, so that the loops and branches they bound are scalar too and
// their address arithmetic leaves the vector unit alone.
template <class T>
__device__ __attribute__((always_inline)) inline T uniform_at(const T* p, int k) {
    return ((const __attribute__((address_space(4))) T*)p)[k];
}

// Copy n values from global to shared memory, kBatch loads in flight per thread.
template <class T>
__device__ void g2s(T* dst, const T* __restrict__ src, int64_t n) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    for (int64_t base = 0; base < n; base += (int64_t)nthr * kBatch) {
        T v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t e = base + tid + (int64_t)u * nthr;
            v[u] = e < n ? src[e] : T(0);
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t e = base + tid + (int64_t)u * nthr;
            if (e < n) dst[e] = v[u];
        }
    }
}

// Loads of one round of a child's update block (nc x nc, lower triangle):
// row block rb (a row per lane), columns jb + Cols wave, ..., Cols per wave.
// A column is contiguous over the lanes; lane u < Cols also loads the front
// column of the wave's u-th, whose place leaves that lane through the scalar
// unit when the entries are added, so the round's loads stay in flight until
// then.  The first round of a row block also carries the block's entries of the
// child's update vector (fused forward solve), on wave 0.
template <int Cols>
struct ChildRound {
    double v[Cols];
    int cj;   // front column of the wave's column lane % Cols
    int ri;   // front row of the lane
    double uv;
};

// A record by scalar loads.
template <class T>
__device__ __attribute__((always_inline)) inline const __attribute__((address_space(4))) T* record_at(const T* p, int k) {
    return (const __attribute__((address_space(4))) T*)p + k;
}

// A child record by scalar loads (field by field: a structure copy does not
// cross address spaces).
__device__ __attribute__((always_inline)) inline ChildRec child_rec_at(const __attribute__((address_space(4))) ChildRec* g) {
    ChildRec r;
    r.u_off = g->u_off;
    r.rel_off = g->rel_off;
    r.uv_off = g->uv_off;
    r.nc = g->nc;
    r.child = g->child;
    return r;
}

// Whether an instance in phase ph takes part in a launch for pred.
__device__ __attribute__((always_inline)) inline bool in_phase(const Ctl* ctl, int pred) {
    if (pred == kPredAll) return true;
    const int ph = __builtin_amdgcn_readfirstlane(global(ctl)->phase);   // written by earlier kernels: a vector load
    return pred == kPredFactor ? (ph == kPhB || ph == kPhF) : ph == pred;
}

// One supernode: assemble the front, factor it, store the L panel and update.
// The front is a packed lower triangle in shared memory, of order m + 1: its last
// row holds the fused forward solve's right-hand side (zeros without it), which
// so takes every step as one more row, and its last entry is the spare slot.
template <int Cols, bool Replace>
__device__ __attribute__((always_inline)) void factor_one(const __attribute__((address_space(4))) FactorTask* T, double eta,
                           double* F, bool fwd) {
    const int w = T->w, m = T->m;
    const PackedIdx ix{m + 1};
    const int nb = m - w;
    const int spare = ((m + 1) * (m + 2)) / 2 - 1;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & (kWave - 1), wv = tid / kWave, nw = nthr / kWave;
    const bool fw = fwd && T->uv >= 0;
    // original entries of the condensed matrix in this supernode's columns, the
    // first kBatch per thread loaded before the children's rounds (so that
    // waiting for them does not wait for the rounds); a diagonal entry's
    // position is stored complemented and takes + eta
    const int nk = T->nk, nchild = T->nchild;
    const auto* fpos = global(T->fpos);
    const auto* kv = global(T->kv);
    const auto* perm = global(T->perm);
    const auto* rhs = global(T->rhs);
    const int32_t* rel = T->rel;
    int kp[kBatch];
    double kx[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
        const int t = tid + u * nthr;
        kp[u] = t < nk ? fpos[t] : 0;
        kx[u] = t < nk ? kv[t] : 0.0;
    }
    // The children's update blocks go in rounds, child after child, row block
    // after row block; the loads of two rounds are in flight ahead of the one
    // being added, the first two issued before the front is cleared.  The
    // records of the current and the next child are read ahead of their rounds.
    const int wvu = __builtin_amdgcn_readfirstlane(wv);
    struct RoundInfo {   // what the adds of an issued round need
        int child, nc, i0, j0;
        bool uv;
    };
    int pci = 0, prb = 0, pjb = 0;   // the next round to issue
    ChildRec prec = child_rec_at(&T->rec0), pnext = child_rec_at(&T->rec1);
    // the fused forward solve's right-hand side of the supernode's columns:
    // the permutation is read before the rounds, thread i's entry of the
    // right-hand side after them (loads complete in the order issued; the
    // right-hand side is waited for where the rounds are about to be added)
    const int pk0 = fw && tid < w ? perm[tid] : 0;
    auto issue = [&](ChildRound<Cols>& r, RoundInfo& info) -> bool {
        if (pci >= nchild) return false;
        const int nc = prec.nc;
        const int64_t uo = prec.u_off, ro = prec.rel_off;
        const int i0 = kWave * prb, j0 = pjb + Cols * wvu, i = min(i0 + lane, nc - 1);
        const auto* uc = global(T->Uall) + uo + i;
#pragma unroll
        for (int u = 0; u < Cols; ++u) r.v[u] = uc[min(j0 + u, nc - 1) * nc];
        r.cj = global(rel)[ro + min(j0 + lane % Cols, nc - 1)];
        r.ri = global(rel)[ro + i];
        const bool uv = fw && wvu == 0 && pjb == 0;
        r.uv = uv ? global(T->uvec)[prec.uv_off + i] : 0.0;
        info = RoundInfo{pci, nc, i0, j0, uv};
        pjb += Cols * nw;
        if (pjb >= min(nc, i0 + kWave)) {   // past the row block's last column
            pjb = 0;
            if (kWave * ++prb >= nc) {
                prb = 0;
                ++pci;
                prec = pnext;
                if (pci + 1 < nchild) pnext = child_rec_at(record_at(T->recs, pci + 1));
            }
        }
        return true;
    };
    ChildRound<Cols> ra, rb;
    RoundInfo ia{}, ib{};
    bool ha = issue(ra, ia);
    bool hb = issue(rb, ib);
    double rv = 0.0;
    if (fw && tid < w) rv = rhs[pk0];
    const int fsize = ((m + 1) * (m + 2)) / 2;
    for (int e = tid; e < fsize; e += nthr) F[e] = 0.0;
    __syncthreads();
    auto place = [&](int pos, double v) {
        if (pos < 0) {
            pos = ~pos;
            v += eta;
        }
        F[pos] = v;
    };
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
        if (tid + u * nthr < nk) place(kp[u], kx[u]);
    for (int t = tid + kBatch * nthr; t < nk; t += nthr) place(fpos[t], kv[t]);
    // fused forward solve of the Newton step: the last row starts from the
    // permuted right-hand side of the supernode's columns (before the barrier
    // that precedes the children's update vectors)
    if (fw)
        for (int i = tid; i < w; i += nthr) F[ix(m, i)] = i == tid ? rv : rhs[perm[i]];
    __syncthreads();
    // extend-add in fixed order; children are separated by barriers (two
    // children can add into the same entry, one child's entries are distinct)
    while (ha) {
        ChildRound<Cols> rc;
        RoundInfo ic{};
        const bool hc = issue(rc, ic);
        const int i = ia.i0 + lane;
        const int bj = ix.base(ra.cj);
        int at[Cols];
        double x[Cols];
#pragma unroll
        for (int u = 0; u < Cols; ++u) {   // entries outside the triangle go to the spare slot
            const int j = ia.j0 + u;
            at[u] = (i < ia.nc && j <= i) ? __builtin_amdgcn_readlane(bj, u) + ra.ri : spare;
            x[u] = F[at[u]];
        }
#pragma unroll
        for (int u = 0; u < Cols; ++u) F[at[u]] = x[u] + ra.v[u];
        if (ia.uv && i < ia.nc) F[ix(m, ra.ri)] += ra.uv;
        if (!hb || ib.child != ia.child) __syncthreads();
        ra = rb;
        ia = ib;
        ha = hb;
        rb = rc;
        ib = ic;
        hb = hc;
    }
    partial_cholesky<Replace>(F, ix, w, spare, &T->ctl->fail);
    // the update block (rows and columns w and on) takes its update before the
    // panel goes out: global stores in flight would hold the update's first
    // shared-memory loads until they complete (their data registers are reused)
    if (nb > 0) update_block(F, ix, w, spare);
    // kStore columns per wave at a time, so that their shared-memory reads are
    // in flight together
    constexpr int kStore = 4;
    auto* Ls = global(T->L);
    for (int jc = kStore * wvu; jc < w; jc += kStore * nw)
        for (int i = lane; i < m; i += kWave) {
            double x[kStore];
#pragma unroll
            for (int u = 0; u < kStore; ++u) {
                const int j = min(jc + u, w - 1);
                x[u] = F[ix(max(i, j), j)];
            }
#pragma unroll
            for (int u = 0; u < kStore; ++u)
                if (jc + u < w) Ls[i + (jc + u) * m] = i >= jc + u ? x[u] : 0.0;
        }
    if (fw) {   // the forward solve's part of the columns and the update vector
        for (int k = tid; k < w; k += nthr) global(T->xp)[k] = F[ix(m, k)];
        auto* us = global(T->uvec + T->uv);
        for (int i = w + tid; i < m; i += nthr) us[i - w] = F[ix(m, i)];
    }
    if (nb > 0) {
        auto* Us = global(T->U);
        for (int jj = kStore * wvu; jj < nb; jj += kStore * nw)
            for (int ii = (jj & ~(kWave - 1)) + lane; ii < nb; ii += kWave) {
                double x[kStore];
#pragma unroll
                for (int u = 0; u < kStore; ++u) {
                    const int j = min(jj + u, nb - 1);
                    x[u] = F[ix(w + max(ii, j), w + j)];
                }
#pragma unroll
                for (int u = 0; u < kStore; ++u)
                    if (jj + u <= ii) Us[ii + (jj + u) * nb] = x[u];
            }
    }
    __syncthreads();   // the front buffer is reused by the next supernode of the group
}

// Variants (threads per workgroup) the autotuner chooses from.
// (two waves per SIMD at least: at most 256 registers, so that the matrix cores'
// accumulators stay in the vector registers)
template <int Threads, bool Replace>
__global__ void __launch_bounds__(Threads, 2)
k_factor_groups(const FactorTask* __restrict__ tasks, int pred, double eta_force) {
    extern __shared__ double lds[];
    const auto* T = record_at(tasks, blockIdx.x);
    if (!in_phase(T->ctl, pred)) return;
    const double eta = pred == kPredAll ? eta_force : global(T->ctl)->eta;
    const bool fwd = pred == kPredFactor;   // in a pass: the Newton step's right-hand side is assembled
    while (true) {
        factor_one<8, Replace>(T, eta, lds, fwd);
        const int next = T->next;
        if (next == 0) break;
        T = record_at(tasks, next);
    }
}

// Forward solve with one supernode's panel P (m x w, column-major, lower w x w
// diagonal block first), staged in shared memory together with the
// reciprocals of its diagonal.  Columns go kPanel at a time: every thread
// solves the small diagonal block itself from broadcast reads, then updates
// the rows it owns; one barrier per block.  v[0:m) holds b; on return xs[0:w) =
// L_dd^{-1} b[0:w) and v[w:m) = b[w:m) - L_below xs.
__device__ __attribute__((always_inline)) void blocked_forward(const double* P, const double* rdiag, int m, int w, double* v, double* xs) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    for (int kb = 0; kb < w; kb += kPanel) {
        const int kw = min(kPanel, w - kb);
        double x[kPanel];
#pragma unroll
        for (int k = 0; k < kPanel; ++k) {
            double s = k < kw ? v[kb + k] : 0.0;
#pragma unroll
            for (int j = 0; j < k; ++j)
                if (k < kw) s = fma(-P[(kb + k) + (int64_t)(kb + j) * m], x[j], s);
            x[k] = k < kw ? s * rdiag[kb + k] : 0.0;
        }
        if (tid < kw) {
#pragma unroll
            for (int k = 0; k < kPanel; ++k)
                if (k == tid) xs[kb + k] = x[k];
        }
        for (int r = kb + kw + tid; r < m; r += nthr) {
            double acc = v[r];
#pragma unroll
            for (int j = 0; j < kPanel; ++j)
                if (j < kw) acc = fma(-P[r + (int64_t)(kb + j) * m], x[j], acc);
            v[r] = acc;
        }
        __syncthreads();
    }
}

// Stage one panel and the reciprocals of its diagonal in shared memory.
__device__ __attribute__((always_inline)) void stage_panel(const double* __restrict__ Ls, int m, int w, double* P, double* rdiag) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    g2s(P, Ls, (int64_t)m * w);
    for (int k = tid; k < w; k += nthr) rdiag[k] = 1.0 / Ls[k + (int64_t)k * m];
}

// Forward substitution L v = P b for one supernode: gather the permuted rhs of
// its columns, add the children's update vectors, solve with the diagonal
// block, then form the update vector of its rows below.
// Shared memory: panel (m w) + rdiag (w) + v (m) + xs (w).
__device__ __attribute__((always_inline)) void fwd_one(const __attribute__((address_space(4))) SolveTask* T, const SnView& S, double* __restrict__ uvec,
                        const double* __restrict__ rhs, double* __restrict__ xp, double* lds) {
    const int s = T->sn, f = T->f, w = T->w, m = T->m;
    const int32_t* perm = T->perm;
    const int tid = threadIdx.x, nthr = blockDim.x;
    double* P = lds;
    double* rdiag = P + (int64_t)m * w;
    double* v = rdiag + w;
    double* xs = v + m;
    stage_panel(T->L, m, w, P, rdiag);
    for (int i = tid; i < m; i += nthr) v[i] = i < w ? rhs[perm[i]] : 0.0;
    __syncthreads();
    for (int ci = uniform_at(S.child_ptr, s); ci < uniform_at(S.child_ptr, s + 1); ++ci) {
        const ChildRec rec = child_rec_at(record_at(S.child_rec, ci));
        const int nc = rec.nc;
        const double* uc = uvec + rec.uv_off;
        const int32_t* rc = S.rel + rec.rel_off;
        for (int i = tid; i < nc; i += nthr) v[rc[i]] += uc[i];
        __syncthreads();
    }
    blocked_forward(P, rdiag, m, w, v, xs);
    for (int k = tid; k < w; k += nthr) xp[f + k] = xs[k];
    double* us = uvec + uniform_at(S.uv_off, s);
    for (int i = w + tid; i < m; i += nthr) us[i - w] = v[i];
    __syncthreads();
}

__global__ void __launch_bounds__(kFactorBlock)
k_fwd_groups(const InstPtrs* __restrict__ Ia, const SolveTask* __restrict__ tasks, int pred, int which) {
    extern __shared__ double lds[];
    const auto* T = record_at(tasks, blockIdx.x);
    const InstPtrs& I = Ia[T->inst];
    if (!in_phase(T->ctl, pred)) return;
    while (true) {
        fwd_one(T, I.S, I.uvec, solve_in(I, which), I.xp, lds);
        const int next = T->next;
        if (next == 0) break;
        T = record_at(tasks, next);
    }
}

// Back substitution L^T x = v for one supernode, after all its ancestors:
// subtract the contribution of the rows below (already final), then solve
// with the transposed diagonal block; writes x unpermuted.  Every global load
// is issued before the first shared-memory store: the diagonal block (a column
// per wave at a time, the lanes over its rows; staged with leading dimension
// w | 1 and zeros on and above the diagonal), its diagonal, the supernode's
// entries of xp, the solution of the rows below (gathered through the row list)
// and the output permutation.  The rows below are read straight from the panel,
// 16 lanes per column and kBwdCols columns per lane group at once (a butterfly
// sums the lanes).  The diagonal block is solved by wave 0, 64 columns at a time
// from the last, and the earlier columns take the block's contribution before
// the next block.  A lone chain of dependent loads and lane reads bounds it (the
// matrix is small): 40 x 100 column, 5.2 us per launch, 7.7 with the solve's
// coefficients read in each step and sizes read through the schedule.
// Shared memory: diagonal block (w (w | 1)) + rdiag (w) + xb (m - w) + v (w) + xs (w).
constexpr int kBwdCols = 4;    // columns per 16-lane group in the rows-below product
constexpr int kBwdDepth = 8;   // rows per lane whose loads are in flight together
constexpr int kBwdSub = 16;    // lanes per column in the rows-below product

// Butterfly sums of kBwdCols values over each kBwdSub-lane group, one level for
// all columns at a time so that a level's lane exchanges are in flight together.
__device__ __attribute__((always_inline)) inline void group_sums(double (&acc)[kBwdCols]) {
#pragma unroll
    for (int off = kBwdSub / 2; off > 0; off >>= 1) {
        double x[kBwdCols];
#pragma unroll
        for (int u = 0; u < kBwdCols; ++u) x[u] = __shfl_xor(acc[u], off, kBwdSub);
#pragma unroll
        for (int u = 0; u < kBwdCols; ++u) acc[u] += x[u];
    }
}
__device__ __attribute__((always_inline)) void bwd_one(const __attribute__((address_space(4))) SolveTask* T, double* __restrict__ xp,
                        double* __restrict__ out, double* lds) {
    const int f = T->f, w = T->w, m = T->m;
    const int nb = m - w;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(tid / kWave), nw = nthr / kWave;
    const int ld = w | 1;
    double* D = lds;
    double* rdiag = D + w * ld;
    double* xb = rdiag + w;
    double* v = xb + nb;
    double* xs = v + w;
    const auto* Ls = global(T->L);
    const auto* rows = global(T->rows) + w;
    const int ri = rows[min(tid, max(nb, 1) - 1) - (nb == 0)];   // without rows below: the last column's own
    // a thread per column (one_workgroup_solve)
    const int tc = min(tid, w - 1);
    const int pk = global(T->perm)[tc];
    const double dg = Ls[tc + tc * m];
    // a round of the diagonal block: 64 rows from r0 of kDiag columns per wave from c0 + wv
    constexpr int kDiag = 16;
    double t[kDiag];
    auto load_diag = [&](int r0, int c0) {
        const auto* col = Ls + min(r0 + lane, w - 1);
#pragma unroll
        for (int u = 0; u < kDiag; ++u) t[u] = col[min(c0 + wv + u * nw, w - 1) * m];
    };
    auto store_diag = [&](int r0, int c0) {
        const int r = r0 + lane;
        if (r < w) {
#pragma unroll
            for (int u = 0; u < kDiag; ++u) {
                const int c = c0 + wv + u * nw;
                if (c < w) D[r + c * ld] = r > c ? t[u] : 0.0;
            }
        }
    };
    load_diag(0, 0);
    const double xv = global(xp)[f + tc];
    // rows-below product: 16 lanes per column, kBwdCols columns per lane group;
    // when it takes one pass (w <= kBwdCols * groups, nb <= kSub * kBwdDepth)
    // the panel's values are loaded here, with everything else
    constexpr int kSub = kBwdSub;
    const int sub = tid % kSub, grp = tid / kSub, ngrp = nthr / kSub;
    const bool one_pass = nb > 0 && w <= kBwdCols * ngrp && nb <= kSub * kBwdDepth;
    double lp[kBwdDepth][kBwdCols];
    if (one_pass && grp < w) {
#pragma unroll
        for (int u = 0; u < kBwdCols; ++u) {
            const int jc = grp + u * ngrp;
            const auto* col = Ls + (jc < w ? jc : 0) * m + w;
#pragma unroll
            for (int q = 0; q < kBwdDepth; ++q) lp[q][u] = col[min(sub + kSub * q, nb - 1)];
        }
    }
    const double xr = global(xp)[ri];
    store_diag(0, 0);
    const int span = kDiag * nw;   // columns per round
    for (int c0 = 0; c0 < w; c0 += span)
        for (int r0 = (c0 / kWave) * kWave; r0 < w; r0 += kWave) {
            if (r0 == 0 && c0 == 0) continue;
            load_diag(r0, c0);
            store_diag(r0, c0);
        }
    if (tid < nb) xb[tid] = xr;
    if (tid < w) {
        rdiag[tid] = 1.0 / dg;
        v[tid] = xv;
    }
    // a narrow supernode can have more rows below than threads
    for (int i = tid + nthr; i < nb; i += nthr) xb[i] = global(xp)[rows[i]];
    __syncthreads();
    if (one_pass) {
        if (grp < w) {   // uniform over each 16-lane group
            double acc[kBwdCols];
#pragma unroll
            for (int u = 0; u < kBwdCols; ++u) acc[u] = 0.0;
#pragma unroll
            for (int q = 0; q < kBwdDepth; ++q) {
                const int i = sub + kSub * q;
                const double x = i < nb ? xb[min(i, nb - 1)] : 0.0;
#pragma unroll
                for (int u = 0; u < kBwdCols; ++u) acc[u] = fma(lp[q][u], x, acc[u]);
            }
            group_sums(acc);
#pragma unroll
            for (int u = 0; u < kBwdCols; ++u) {
                const int jc = grp + u * ngrp;
                if (sub == 0 && jc < w) v[jc] -= acc[u];
            }
        }
    } else
    for (int jc0 = grp; jc0 < w; jc0 += kBwdCols * ngrp) {
        double acc[kBwdCols];
        const gdouble* col[kBwdCols];
#pragma unroll
        for (int u = 0; u < kBwdCols; ++u) {
            const int jc = jc0 + u * ngrp;
            acc[u] = 0.0;
            col[u] = Ls + (jc < w ? jc : 0) * m + w;
        }
        // kBwdDepth rows per lane at a time, all their loads issued together
        // (rows past nb load row nb - 1 and add zero; a column past w reads
        // column 0 and is not stored)
        for (int i0 = sub; i0 < nb; i0 += kSub * kBwdDepth) {
            double lv[kBwdDepth][kBwdCols], xv[kBwdDepth];
#pragma unroll
            for (int t = 0; t < kBwdDepth; ++t) {
                const int i = i0 + kSub * t, ic = min(i, nb - 1);
                xv[t] = i < nb ? xb[ic] : 0.0;
#pragma unroll
                for (int u = 0; u < kBwdCols; ++u) lv[t][u] = col[u][ic];
            }
#pragma unroll
            for (int t = 0; t < kBwdDepth; ++t)
#pragma unroll
                for (int u = 0; u < kBwdCols; ++u) acc[u] = fma(lv[t][u], xv[t], acc[u]);
        }
        group_sums(acc);
#pragma unroll
        for (int u = 0; u < kBwdCols; ++u) {
            const int jc = jc0 + u * ngrp;
            if (sub == 0 && jc < w) v[jc] -= acc[u];
        }
    }
    __syncthreads();
    for (int b0 = ((w - 1) / kWave) * kWave; b0 >= 0; b0 -= kWave) {
        const int bw = min(kWave, w - b0);
        if (wv == 0) {
            const int j = min(lane, bw - 1);
            const double r = rdiag[b0 + j];
            double vj = lane < bw ? v[b0 + j] : 0.0;
            const double* col = D + b0 + (b0 + j) * ld;
            for (int k0 = ((bw - 1) / kSolveSteps) * kSolveSteps; k0 >= 0; k0 -= kSolveSteps) {
                double c[kSolveSteps];
                if (k0 + kSolveSteps <= bw) {
#pragma unroll
                    for (int u = 0; u < kSolveSteps; ++u) c[u] = col[k0 + u];
                } else {   // steps past the block take nothing
#pragma unroll
                    for (int u = 0; u < kSolveSteps; ++u) {
                        const double x = col[min(k0 + u, bw - 1)];
                        c[u] = k0 + u < bw ? x : 0.0;
                    }
                }
                vj = solve_steps<true>(vj, r, c, k0);
            }
            vj *= r;
            if (lane < bw) {
                xs[b0 + lane] = vj;
                if (b0 == 0) {   // the other blocks' entries go out below
                    global(xp)[f + lane] = vj;
                    global(out)[pk] = vj;
                }
            }
        }
        if (b0 > 0) {   // columns before the block: v[c] -= L(block, c)^T x(block)
            __syncthreads();
            for (int c = tid; c < b0; c += nthr) {
                double acc = v[c];
                for (int q = 0; q < bw; ++q) acc = fma(-D[b0 + q + c * ld], xs[b0 + q], acc);
                v[c] = acc;
            }
            __syncthreads();
        }
    }
    if (tid >= kWave && tid < w) {
        global(xp)[f + tid] = xs[tid];
        global(out)[pk] = xs[tid];
    }
}

__global__ void __launch_bounds__(kFactorBlock)
k_bwd_groups(const InstPtrs* __restrict__ Ia, const SolveTask* __restrict__ tasks, int pred, int which) {
    extern __shared__ double lds[];
    const auto* T = record_at(tasks, blockIdx.x);
    const InstPtrs& I = Ia[T->inst];
    if (!in_phase(T->ctl, pred)) return;
    while (true) {
        bwd_one(T, I.xp, solve_out(I, which), lds);
        const int next = T->next;
        if (next == 0) break;
        __syncthreads();   // the next supernode reads this one's solution and reuses its shared memory
        T = record_at(tasks, next);
    }
}

}  // namespace

hipError_t linalg_configure(size_t max_lds_bytes) {
    const void* fns[] = {reinterpret_cast<const void*>(k_factor_groups<kFactorThreads[0], false>),
                         reinterpret_cast<const void*>(k_factor_groups<kFactorThreads[1], false>),
                         reinterpret_cast<const void*>(k_factor_groups<kFactorThreads[1], true>),
                         reinterpret_cast<const void*>(k_fwd_groups), reinterpret_cast<const void*>(k_bwd_groups)};
    for (const void* fn : fns) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds_bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

void launch_factor_groups(int variant, int pred, double eta_force, const FactorTask* t, int groups, size_t lds_bytes,
                          hipStream_t st) {
    if (groups <= 0) return;
    static_assert(kFactorVariants == 2, "a launch per variant");
    const auto kernel = variant == 0 ? k_factor_groups<kFactorThreads[0], false>
                        : variant == 1 ? k_factor_groups<kFactorThreads[1], false> : k_factor_groups<kFactorThreads[1], true>;
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(kFactorThreads[variant == 0 ? 0 : 1]), lds_bytes, st, t, pred, eta_force);
}

void launch_fwd_groups(int pred, int which, const InstPtrs* I, const SolveTask* t, int groups, size_t lds_bytes,
                       hipStream_t st) {
    if (groups <= 0) return;
    hipLaunchKernelGGL(k_fwd_groups, dim3(groups), dim3(kFactorBlock), lds_bytes, st, I, t, pred, which);
}

void launch_bwd_groups(int pred, int which, const InstPtrs* I, const SolveTask* t, int groups, size_t lds_bytes,
                       hipStream_t st) {
    if (groups <= 0) return;
    hipLaunchKernelGGL(k_bwd_groups, dim3(groups), dim3(kFactorBlock), lds_bytes, st, I, t, pred, which);
}

}  // namespace nmpc
