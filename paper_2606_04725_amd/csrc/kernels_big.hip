// Large supernodes: numeric factorization and solves (eqs. 20-25) spread over
// many workgroups.  A front that does not fit in shared memory is assembled
// and factored in place in its final storage: column j < w of the front is
// column j of the supernode's L panel (m x w, leading dimension m) and the
// trailing block is the update block handed to the parent ((m - w) x (m - w),
// leading dimension m - w).  Every launch covers one step for all large
// supernodes of one tree level (of every instance of a batch), described by a
// task list; every sum is taken in a fixed order, so results do not depend on
// how tasks are scheduled.
//
// Factorization of one level: assemble the fronts (KKT entries, + eta on the
// diagonal, and the children's update blocks); then per outer panel of kBigOuter
// columns, per inner panel of kBigPanel columns: factor the diagonal block and
// solve the rows below it (rows split over workgroups), and update the rest of
// the outer panel; then one rank-kBigOuter update of the trailing lower triangle.
// Updates run on the matrix cores (64 x 64 tiles over workgroups, one
// v_mfma_f64_16x16x4f64 per 4 columns); the outer panel keeps the update
// blocks' read-modify-write traffic to one pass per kBigOuter columns.
//
// Solves: forward, the right-hand side and the children's update vectors are
// gathered by rows over workgroups, then chunk by chunk one workgroup solves with
// the diagonal block and the rows after it are a GEMV split over workgroups;
// backward, the transposed GEMV with the rows below is split over column blocks,
// then chunk by chunk one workgroup solves with the transposed diagonal block.
#include <cmath>

#include "kernels.h"
#include "front_chol.h"
#include "front_rules.h"

namespace nmpc {

namespace {

constexpr int kWave = 64;
constexpr int kTile = 64;        // trailing-update tile
constexpr int kSolveRows = 64;   // GEMV rows per workgroup
constexpr int kSolveCols = 16;   // transposed-GEMV columns per workgroup
constexpr int kTri = kWave * (kWave + 1);   // a staged 64 x 64 triangle, leading dimension 65
constexpr int kStage = kWave * kWave / kBlock;   // entries of a 64 x 64 block staged per thread
constexpr int kUpdateDepth = 4;  // 4-column steps of an update tile whose loads are in flight while as many are multiplied

struct Front {
    double* L;     // panel, leading dimension m
    double* U;     // update block, leading dimension m - w
    int f, w, m;
};

// The front of a task: its storage and sizes come with the task record, so the
// first data loads wait for one dependent load, not for a chain through the
// instance and its supernode tables.
__device__ inline Front front_of(const BigTask& t) { return Front{t.L, t.U, t.f, t.w, t.m}; }

// address of front entry (i, j), i >= j
__device__ inline double* at(const Front& F, int i, int j) {
    return j < F.w ? F.L + i + (int64_t)j * F.m : F.U + (i - F.w) + (int64_t)(j - F.w) * (F.m - F.w);
}

// Fused forward substitution of the Newton step (eq. 23), run by the
// factorization of a supernode whose whole subtree runs it: the vector over
// the front's rows starts as the permuted right-hand side of its columns plus
// the children's update vectors; each panel's solution replaces its entries,
// and the rows below take the panel's product as their rows are solved.
// Entry i lives in xp (i < w) or in the supernode's update vector (i >= w),
// where the unfused solve leaves them too.
__device__ inline bool fwd_fused(const BigTask& t, int pred) { return pred == kPredFactor && t.fused; }
__device__ inline double* fwd_entry(const InstPtrs& I, const Front& F, const BigTask& t, int i) {
    return i < F.w ? I.xp + F.f + i : I.uvec + t.uv + (i - F.w);
}

// ---- factorization ---------------------------------------------------------------
// Assembly, task a = first column, b = chunk q of kBigChunk rows: wave v builds
// the chunk's part of column a + v in shared memory, the KKT slots of the column
// (a < w; eta added on the diagonal), then the children's columns that land
// there, in child order, through their relative row positions, and writes it
// once.  A front is so written once and its children's blocks are read once;
// zeroing it and adding each child in a launch of its own wrote it once more and
// read and wrote it again per child (32 x 32 x 50 plate: 1.07 ms per
// factorization for the two kernels).  One wave per column keeps 20 columns in
// flight per CU without a barrier; a wave's shared-memory operations complete in
// the order issued.
constexpr int kAsmDepth = 8;   // child rows per lane whose loads are in flight together
template <class T>
__device__ __attribute__((always_inline)) inline T uniform_at(const T* p, int64_t k) {   // read-only data, a scalar load
    return ((const __attribute__((address_space(4))) T*)p)[k];
}
__global__ void __launch_bounds__(kBigAsmCols * kWave)
k_big_assemble(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred, double eta_force) {
    __shared__ double cols[kBigAsmCols][kBigChunk];
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const double eta = pred == kPredAll ? eta_force : I.ctl->eta;
    const Front F = front_of(tk);
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int j = tk.a + wv;
    if (j >= F.m) return;
    const int base = tk.b * kBigChunk, r0 = max(base, j), r1 = min(F.m, base + kBigChunk);   // the chunk's rows
    if (r0 >= r1) return;
    double* col = cols[wv];   // row r at col[r - base]
    const int ce = uniform_at(I.S.big_col, tk.sn) + j;
    const int e0 = uniform_at(I.S.big_ptr, ce), e1 = uniform_at(I.S.big_ptr, ce + 1);
    const bool fw = fwd_fused(tk, pred) && j >= base;   // the chunk that holds the column's own row
    double fv = fw && j < F.w ? global(I.rhs)[uniform_at(I.perm, F.f + j)] : 0.0;
    for (int r = r0 + lane; r < r1; r += kWave) col[r - base] = 0.0;
    if (j < F.w) {
        const int t1 = uniform_at(I.kcol_ptr, F.f + j + 1);
        for (int t = uniform_at(I.kcol_ptr, F.f + j) + lane; t < t1; t += kWave) {
            const int r = global(I.S.k_fpos)[t];
            double v = global(I.kv)[t];
            if (r == j) v += eta;
            if (r >= r0 && r < r1) col[r - base] = v;
        }
    }
    for (int e = e0; e < e1; ++e) {
        const int64_t u_col = uniform_at(&I.S.big_ent->u_col, (int64_t)e * (sizeof(BigEntry) / sizeof(int64_t)));
        const int64_t rel_off = uniform_at(&I.S.big_ent->rel_off, (int64_t)e * (sizeof(BigEntry) / sizeof(int64_t)));
        const int jc = uniform_at(&I.S.big_ent->jc, (int64_t)e * (sizeof(BigEntry) / sizeof(int32_t)));
        const int nc = uniform_at(&I.S.big_ent->nc, (int64_t)e * (sizeof(BigEntry) / sizeof(int32_t)));
        const int ck = uniform_at(&I.S.big_ent->chunk, (int64_t)e * (sizeof(BigEntry) / sizeof(int32_t)));
        if (fw) fv += global(I.uvec)[rel_off + jc];
        const int i0 = max(jc, base > 0 ? uniform_at(I.S.chunk_pos, ck + tk.b) : 0);
        const int i1 = F.m > base + kBigChunk ? uniform_at(I.S.chunk_pos, ck + tk.b + 1) : nc;
        const auto* rg = global(I.S.rel) + rel_off;
        const auto* uc = global(I.U) + u_col;
        for (int ib = i0 + lane; ib < i1; ib += kAsmDepth * kWave) {
            int rr[kAsmDepth];
            double uv[kAsmDepth];
#pragma unroll
            for (int u = 0; u < kAsmDepth; ++u) {
                const int i = min(ib + u * kWave, i1 - 1);
                rr[u] = rg[i];
                uv[u] = uc[i];
            }
#pragma unroll
            for (int u = 0; u < kAsmDepth; ++u)
                if (ib + u * kWave < i1) col[rr[u] - base] += uv[u];
        }
    }
    gdouble* dst = global(at(F, j, j)) - j;   // entry (r, j) at dst[r]
    for (int r = r0 + lane; r < r1; r += kWave) dst[r] = col[r - base];
    if (fw && lane == 0) *fwd_entry(I, F, tk, j) = fv;
}

// One panel of a front: task a = kb, b = row block.  Every workgroup factors the
// 64 x 64 diagonal block D of columns [kb, kb + pw) itself, so that the rows
// below are solved in the same launch, as soon as a 16-column block of D is
// factored.  Wave 0 holds D's rows one per lane and takes 16 pivot columns at a
// time in registers (factor_rows: no shared memory, no barrier inside the 16
// columns); between blocks the next 16 columns take
// their update on the matrix cores.  Waves 1-4 solve 16 rows each, x D^T = a,
// block after block: the solved blocks' products on the matrix cores, then the
// 16 columns by broadcasts within the 16 lanes of a row group.  Wave 5 does the
// same for the fused forward solve, whose right-hand side is one more row.
// Columns past pw are padded with the identity.  The factored block of a front
// with several workgroups goes to dfac, from where the next update launch puts
// it into the panel: another workgroup may still have to read the original.
// A pivot that is not positive and finite sets the instance's failure flag
// (eq. 12) and the factor's values are not finite from there on, or, with
// Replace, it counts as 1 and nothing is reported.
// Wave 0's chain bounds it: of 40 thousand cycles 19 went to the four 16-column
// factorizations, 8 to the loads.  16.9 us per launch in the Cholesky of the 28 x
// 37 plate (20.3 with a test for every pivot and the next columns' tiles one
// after another; diagonal block and rows in launches of their own took 45).
constexpr int kPanelThreads = (kPanelRowWaves + 2) * kWave;
constexpr int kLdx = 17;   // leading dimension of a wave's 16 rows in shared memory
constexpr int kLdd = kBigPanel + 1;

// 16 pivot columns of D (shared memory, kLdd) from column c0, by one wave (a row
// from c0 on per lane); the reciprocals of the diagonal to rd.
template <bool Replace>
__device__ __attribute__((always_inline)) inline bool factor_16(double* D, double* rd, int c0) {
    const int lane = threadIdx.x & (kWave - 1), row = min(c0 + lane, kBigPanel - 1);
    double a[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) a[c] = D[row + (c0 + c) * kLdd];
    const bool bad = factor_rows<16, Replace>(a, 16);
    if (c0 + lane < kBigPanel) {
#pragma unroll
        for (int c = 0; c < 16; ++c) D[row + (c0 + c) * kLdd] = a[c];   // above the diagonal: never read again
    }
    __builtin_amdgcn_wave_barrier();   // the same wave reads them: program order suffices
    if (lane < 16) rd[c0 + lane] = 1.0 / D[(c0 + lane) * (kLdd + 1)];
    return bad;
}

// The 16 columns after the first 16 (P + 1) factored ones take their update, by
// one wave: the tiles below the diagonal at once, so that their products are
// independent and the operands are read ahead (tile by tile, 8.5 of the panel's
// 40 thousand cycles went here).
template <int P>
__device__ __attribute__((always_inline)) inline void update_next_16(double* D) {
    constexpr int n0 = 16 * (P + 1), nt = kBigPanel / 16 - 1 - P;
    const int lane = threadIdx.x & (kWave - 1), li = lane & 15, lk = lane >> 4;
    f64x4 u[nt];
#pragma unroll
    for (int t = 0; t < nt; ++t) u[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < n0; i += 4) {
        const double* col = D + n0 + li + (i + lk) * kLdd;
        const double bv = col[0];
#pragma unroll
        for (int t = 0; t < nt; ++t) u[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(col[16 * t], bv, u[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < nt; ++t) {
        double* d = D + n0 + 16 * t + lk + (n0 + li) * kLdd;   // entries above the diagonal are never used
#pragma unroll
        for (int r = 0; r < 4; ++r) d[4 * r] -= u[t][r];
    }
}

// Solve the 16 columns c0 of a 16-row tile in the matrix-core layout (lane (li,
// lk) holds rows lk, lk + 4, lk + 8, lk + 12 of column li) against D's diagonal
// block there.
__device__ __attribute__((always_inline)) inline void solve_16(f64x4& acc, const double* D, const double* rd, int c0) {
    const int li = threadIdx.x & 15;
    double T[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const double v = D[(c0 + li) + (c0 + k) * kLdd];
        T[k] = li > k ? v : 0.0;
    }
    const double r = rd[c0 + li];
    static_for<15>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = fma(-group_lane<k>(acc[q] * r), T[k], acc[q]);
        __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] *= r;
}

template <bool Replace>
__global__ void __launch_bounds__(kPanelThreads)
k_big_panel(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred) {
    static_assert(kBigPanel == kWave, "a lane per row of D");
    __shared__ double D[kTri];
    __shared__ double rd[kBigPanel];
    __shared__ double Xs[kPanelRowWaves + 1][kLdx * kBigPanel];
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const Front F = front_of(tk);
    const int kb = tk.a, pw = min(kBigPanel, F.w - kb), np = (pw + 15) / 16;
    const bool fw = fwd_fused(tk, pred);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave, li = lane & 15, lk = lane >> 4;
    const bool rhs_wave = wv == kPanelRowWaves + 1;
    const int rw = panel_first_row(kb, pw, tk.b, wv);   // first row of a row wave
    const bool row_wave = wv >= 1 && !rhs_wave && rw < F.m;
    const bool works = row_wave || (rhs_wave && fw);
    double* X = Xs[wv >= 1 ? wv - 1 : 0];
    gdouble* Lp = global(F.L) + (int64_t)kb * F.m;   // the panel's columns: 32-bit offsets from here
    {
        // every load of the thread (D and its wave's rows) before the first
        // store, from clamped addresses (no branch around a load)
        constexpr int kDiagStage = (kBigPanel * kBigPanel + kPanelThreads - 1) / kPanelThreads;
        double t[kDiagStage], x[16];
#pragma unroll
        for (int s = 0; s < kDiagStage; ++s) {
            const int e = tid + s * kPanelThreads, i = min(e % kBigPanel, pw - 1), j = min(e / kBigPanel, i);
            t[s] = Lp[kb + i + j * F.m];
        }
        const gdouble* src = rhs_wave ? global(I.xp) + F.f + kb : Lp + min(rw + li, F.m - 1);
        const int stride = rhs_wave ? 1 : F.m;
        const bool in = rhs_wave ? fw && li == 0 : rw + li < F.m;
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = src[min(4 * u + lk, pw - 1) * stride];
#pragma unroll
        for (int s = 0; s < kDiagStage; ++s) {
            const int e = tid + s * kPanelThreads, i = e % kBigPanel, j = e / kBigPanel;
            const double v = (i < pw && j <= i) ? t[s] : (i == j ? 1.0 : 0.0);
            if (e < kBigPanel * kBigPanel) D[i + j * kLdd] = v;
        }
        if (works) {
#pragma unroll
            for (int u = 0; u < 16; ++u) X[li + (4 * u + lk) * kLdx] = in && 4 * u + lk < pw ? x[u] : 0.0;
        }
    }
    __syncthreads();
    bool bad = false;
    for (int p = 0; p < np; ++p) {
        const int c0 = 16 * p;
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        if (wv == 0) {
            bad |= factor_16<Replace>(D, rd, c0);
        } else if (works) {   // the solved blocks' part, while wave 0 factors
            // (summed from zero: its roundings are the products' size, not the entries')
            for (int i = 0; i < c0; i += 4) {
                const double av = X[li + (i + lk) * kLdx];
                const double bv = D[(c0 + li) + (i + lk) * kLdd];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = X[(4 * r + lk) + (c0 + li) * kLdx] - acc[r];
        }
        __syncthreads();
        if (wv == 0) {
            if (p + 1 < np) {
                if (p == 0) update_next_16<0>(D);
                else if (p == 1) update_next_16<1>(D);
                else update_next_16<2>(D);
                __builtin_amdgcn_wave_barrier();   // the same wave reads them next: program order suffices
            }
        } else if (works) {
            solve_16(acc, D, rd, c0);
#pragma unroll
            for (int r = 0; r < 4; ++r) X[(4 * r + lk) + (c0 + li) * kLdx] = acc[r];
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (bad && tid == 0) I.ctl->fail = 1;
    if (fw) __syncthreads();   // the forward solve's row is read by the row waves
    if (row_wave) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int col = 4 * u + lk, r = rw + li;
            if (r < F.m && col < pw) Lp[r + col * F.m] = X[li + col * kLdx];
        }
        if (fw) {   // each row takes the panel's product with its solution: lane (li, lk) sums 16 columns
            const double* y = Xs[kPanelRowWaves];
            double dot = 0.0;
#pragma unroll
            for (int c = 0; c < 16; ++c)   // columns past 16 np are not solved: zero from the load
                dot = fma(X[li + (16 * lk + c) * kLdx], y[(16 * lk + c) * kLdx], dot);
            dot += __shfl_xor(dot, 16, kWave);
            dot += __shfl_xor(dot, 32, kWave);
            if (lk == 0 && rw + li < F.m) *fwd_entry(I, F, tk, rw + li) -= dot;
        }
    }
    if (tk.b == 0 && (wv == 0 || rhs_wave)) {
        const bool aside = F.m - kb - pw > kRowBlock;   // other workgroups share the block
        gdouble* scr = global(I.dfac) + (int64_t)tk.slot * kBigDiag;
        if (wv == 0) {
            for (int j = 0; j < pw; ++j)
                if (lane >= j && lane < pw) {
                    if (aside) scr[lane + j * kBigPanel] = D[lane + j * kLdd];
                    else Lp[kb + lane + j * F.m] = D[lane + j * kLdd];
                }
        } else if (fw && lane < pw) {
            const double v = X[lane * kLdx];
            if (aside) scr[kBigPanel * kBigPanel + lane] = v;
            else I.xp[F.f + kb + lane] = v;
        }
    }
}

// The factored diagonal block of columns kb (and the forward solve's entries)
// from dfac into the front's storage.
__device__ inline void keep_diagonal(const InstPtrs& I, const BigTask& tk, int pred) {
    const int kb = tk.a, pw = min(kBigPanel, tk.w - kb);
    const gdouble* scr = global(I.dfac) + (int64_t)tk.slot * kBigDiag;
    for (int e = threadIdx.x; e < kBigPanel * kBigPanel; e += blockDim.x) {
        const int i = e % kBigPanel, j = e / kBigPanel;
        if (i < pw && j <= i) global(tk.L)[(kb + i) + (int64_t)(kb + j) * tk.m] = scr[e];
    }
    if (fwd_fused(tk, pred) && (int)threadIdx.x < pw)
        I.xp[tk.f + kb + threadIdx.x] = scr[kBigPanel * kBigPanel + threadIdx.x];
}

// Tiles of one launch are handed out XCD by XCD: workgroups are dealt to the 8
// XCDs round-robin, so tile b % 8 * (n / 8) + b / 8 keeps neighbouring tiles
// (which share panel rows) on one XCD and its L2.
__device__ inline int xcd_tile(int b, int n) {
    const int full = (n / 8) * 8;
    return b < full ? (b % 8) * (n / 8) + b / 8 : b;
}

// C -= A B^T on one 64 x 64 tile, A and B the panel columns [k0, k0 + kw) of
// the tile's rows and columns.  Outer (Inner = false), task (inst, s, kb, tile):
// the lower triangle of the trailing block from kb + kw, kw = min(kBigOuter,
// w - kb).  Inner, task (inst, s, ki, tile): the rest of ki's outer panel,
// rows from ki + kw to m, columns [ki + kw, outer panel end), kw =
// min(kBigPanel, w - ki).  Wave v computes the 32 x 32 quarter (v / 2, v % 2).
// Two waves per SIMD at least, so that the accumulators stay in the vector
// registers: copied to the accumulation registers and back in every round, the
// round's loads behind branches and not ahead of the products, and the tile's
// own entries read last, the outer launches of a 32 x 32 x 50 plate took 72.9 us
// and the inner ones 14.2; now 57.8 and 11.2 (the outer ones at 0.3 of the rate
// of a large matrix product: tiles of neighbouring launches' ends leave compute
// units idle, and the panel's rows come from beyond the XCD's L2).
template <bool Inner>
__global__ void __launch_bounds__(kBlock, 2)
k_big_update(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred) {
    const BigTask tk = tasks[xcd_tile(blockIdx.x, gridDim.x)];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    if (tk.b < 0) {
        keep_diagonal(I, tk, pred);
        return;
    }
    const Front F = front_of(tk);
    const int k0 = tk.a;
    const int kw = min(Inner ? kBigPanel : kBigOuter, F.w - k0);
    const int t0 = k0 + kw;
    int ti, tj;
    if (Inner) {
        const int cend = min(F.w, k0 - k0 % kBigOuter + kBigOuter);
        const int tc = (cend - t0 + kTile - 1) / kTile;
        ti = tk.b / tc;
        tj = tk.b - ti * tc;
    } else {
        ti = (int)((sqrt(8.0 * tk.b + 1.0) - 1.0) * 0.5);
        while ((ti + 1) * (ti + 2) / 2 <= tk.b) ++ti;
        while (ti * (ti + 1) / 2 > tk.b) --ti;
        tj = tk.b - ti * (ti + 1) / 2;
    }
    const int cmax = Inner ? min(F.w, k0 - k0 % kBigOuter + kBigOuter) : F.m;
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int li = lane & 15, lk = lane >> 4;
    const int i0 = t0 + kTile * ti + 32 * (wv >> 1);
    const int j0 = t0 + kTile * tj + 32 * (wv & 1);
    if (j0 >= cmax || i0 >= F.m || j0 > i0 + 31) return;
    // Every load is from a clamped address: entries past the front or above the
    // diagonal compute something that is not stored (above the diagonal there is
    // no storage where a tile crosses from the panel into the update block, so
    // those read their column's diagonal entry).  The tile's own entries are
    // loaded before the products.
    const int m = F.m;
    gdouble* cp[2];
    int jb[2];
    f64x4 acc[2][2], c[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        jb[b] = min(j0 + 16 * b + li, cmax - 1);
        cp[b] = global(at(F, jb[b], jb[b])) - jb[b];   // entry (i, j), i >= j, at cp[i]
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int r = 0; r < 4; ++r) c[a][b][r] = cp[b][max(min(i0 + 16 * a + 4 * r + lk, m - 1), jb[b])];
        }
    // kUpdateDepth steps of 4 columns are in flight while the ones before them
    // are multiplied; a lane's place in a step is a 32-bit offset from the step's
    // first column, which is the same for the wave
    int ao[2], bo[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) ao[a] = lk * m + min(i0 + 16 * a + li, m - 1);
#pragma unroll
    for (int b = 0; b < 2; ++b) bo[b] = lk * m + min(j0 + 16 * b + li, cmax - 1);
    const gdouble* Lk = global(F.L) + (int64_t)k0 * m;
    struct Steps {
        double a[kUpdateDepth][2], b[kUpdateDepth][2];
    };
    auto load = [&](Steps& s, int k4) {   // k4 + 4 kUpdateDepth <= kw
        const gdouble* col = Lk + (int64_t)k4 * m;
#pragma unroll
        for (int u = 0; u < kUpdateDepth; ++u, col += 4 * m) {
#pragma unroll
            for (int a = 0; a < 2; ++a) s.a[u][a] = col[ao[a]];
#pragma unroll
            for (int b = 0; b < 2; ++b) s.b[u][b] = col[bo[b]];
        }
    };
    auto load_tail = [&](Steps& s, int k4) {   // columns past kw count as zero
#pragma unroll
        for (int u = 0; u < kUpdateDepth; ++u) {
            const int k = k4 + 4 * u + lk;
            const gdouble* col = Lk + (int64_t)min(k, kw - 1) * m;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const double x = col[ao[a] - lk * m];
                s.a[u][a] = k < kw ? x : 0.0;
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const double x = col[bo[b] - lk * m];
                s.b[u][b] = k < kw ? x : 0.0;
            }
        }
    };
    auto multiply = [&](const Steps& s) {
#pragma unroll
        for (int u = 0; u < kUpdateDepth; ++u)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.a[u][a], s.b[u][b], acc[a][b], 0, 0, 0);
    };
    constexpr int kStep = 4 * kUpdateDepth;
    const int full = kw / kStep, rest = kw % kStep;   // kw >= 1
    Steps s0, s1;
    if (full == 0) {
        load_tail(s0, 0);
        multiply(s0);
    } else {
        load(s0, 0);
        int q = 1;
        for (; q + 1 < full; q += 2) {
            load(s1, q * kStep);
            multiply(s0);
            load(s0, (q + 1) * kStep);
            multiply(s1);
        }
        if (q < full) {
            load(s1, q * kStep);
            multiply(s0);
            if (rest) load_tail(s0, full * kStep);
            multiply(s1);
            if (rest) multiply(s0);
        } else {
            if (rest) load_tail(s1, full * kStep);
            multiply(s0);
            if (rest) multiply(s1);
        }
    }
    if (i0 + 32 <= m && j0 + 32 <= cmax && j0 + 31 <= i0) {   // the whole tile is stored
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) cp[b][i0 + 16 * a + 4 * r + lk] = c[a][b][r] - acc[a][b][r];
    } else {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = i0 + 16 * a + 4 * r + lk, j = j0 + 16 * b + li;
                    if (i < m && j <= i && j < cmax) cp[b][i] = c[a][b][r] - acc[a][b][r];
                }
    }
}

// ---- solves ------------------------------------------------------------------------
// The columns of a large supernode are solved kChunk at a time.  Forward: the
// right-hand side over the supernode's columns goes into xp and the rows below
// into its update vector, each with the children's update vectors, a row per
// thread over many workgroups; then per chunk one workgroup solves its triangle
// and the rows after it (the rest of the diagonal part and the rows below) take
// the chunk's GEMV, split over workgroups.  Backward, from the last chunk: the
// rows below contribute L[w:m, k]^T x(rows below) to bsum (transposed GEMV),
// each chunk's triangle is solved by one workgroup, then the columns before the
// chunk take its transposed GEMV into bsum.  Sums run in a fixed order.
constexpr int kChunk = 256;

// Lower triangle of the diagonal block [b0, b0 + bw)^2 of L into registers (16
// entries per thread, loads only, from clamped addresses) ...
__device__ __attribute__((always_inline)) inline void load_triangle(const Front& F, int b0, int bw, double (&t)[kStage]) {
#pragma unroll
    for (int s = 0; s < kStage; ++s) {
        const int e = threadIdx.x + s * kBlock, i = min(e % kWave, bw - 1), j = min(e / kWave, i);
        t[s] = global(F.L)[(b0 + i) + (int64_t)(b0 + j) * F.m];
    }
}

// ... and from there to T (leading dimension kWave + 1), zero on and above the
// diagonal and past bw, with the reciprocals of the diagonal in rd (1 past bw):
// a wave holds every fourth column, so each lane finds its diagonal entry in one
// of the four waves and a wave divides once.  The caller synchronizes.
__device__ __attribute__((always_inline)) inline void store_triangle(const double (&t)[kStage], int bw, double* T, double* rd) {
    const int i = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    static_assert(kBlock == 4 * kWave, "four columns per step");
    double d = 1.0;
#pragma unroll
    for (int s = 0; s < kStage; ++s) {
        const int j = wv + 4 * s;
        T[i + j * (kWave + 1)] = j < i && i < bw ? t[s] : 0.0;
        d = j == i ? t[s] : d;
    }
    if ((i & 3) == wv) rd[i] = i < bw ? 1.0 / d : 1.0;
}

// Solve with the staged triangle (or, Back, its transpose) on one wave.
template <bool Back>
__device__ __attribute__((always_inline)) inline double solve_triangle(double vj, const double* T, const double* rd, int bw) {
    const int j = threadIdx.x & (kWave - 1);
    const double r = rd[j];
    for (int g = 0; g < kWave; g += kSolveSteps) {
        const int k0 = Back ? kWave - kSolveSteps - g : g;   // the group's first column
        if (k0 >= bw) continue;
        double c[kSolveSteps];
        const double* col = T + (Back ? k0 + j * (kWave + 1) : j + k0 * (kWave + 1));
#pragma unroll
        for (int u = 0; u < kSolveSteps; ++u) c[u] = col[Back ? u : u * (kWave + 1)];
        vj = solve_steps<Back>(vj, r, c, k0);
    }
    return vj * r;
}

// forward, task a = row block: a row i of the front per thread, its right-hand
// side (i < w) and the children's update vectors in child order, into xp (i < w)
// or the update vector.
__global__ void __launch_bounds__(kBlock)
k_bigfwd_gather(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred, int which) {
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const Front F = front_of(tk);
    const int i = tk.a * kBlock + threadIdx.x;
    if (i >= F.m) return;
    const int ce = uniform_at(I.S.big_col, tk.sn) + i;
    const int e0 = global(I.S.big_ptr)[ce], e1 = global(I.S.big_ptr)[ce + 1];
    double v = i < F.w ? global(solve_in(I, which))[global(I.perm)[F.f + i]] : 0.0;
    for (int e = e0; e < e1; ++e) {
        const auto* en = global(I.S.big_ent) + e;
        v += global(I.uvec)[en->rel_off + en->jc];
    }
    *fwd_entry(I, F, tk, i) = v;
}

// forward, task a = chunk: x[c0, c1) = L[c0:c1, c0:c1]^{-1} v[c0, c1) in xp, by
// blocks of 64 columns: the block's triangle staged in shared memory, wave 0
// solves it while the other waves load the entries of the chunk's later rows,
// one per thread, which then take the block's update.  The next block's triangle
// is loaded ahead (28 x 37 plate: 13.6 us per launch; 47.5 with the loads
// after the solve and a division per column).
__global__ void __launch_bounds__(kBlock)
k_bigfwd_tri(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred) {
    static_assert(kChunk == kBlock, "a row per thread past the first wave");
    __shared__ double T[kTri];
    __shared__ double rd[kWave];
    __shared__ double v[kChunk];
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const Front F = front_of(tk);
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    double* xs = I.xp + F.f;
    const int c0 = tk.a * kChunk, cw = min(kChunk, F.w - c0);
    double t[kStage];
    load_triangle(F, c0, min(kWave, cw), t);
    if (tid < cw) v[tid] = global(xs)[c0 + tid];
    for (int b0 = 0; b0 < cw; b0 += kWave) {
        const int bw = min(kWave, cw - b0), b1 = b0 + bw;
        store_triangle(t, bw, T, rd);
        __syncthreads();
        if (b1 < cw) load_triangle(F, c0 + b1, min(kWave, cw - b1), t);
        if (wv == 0) {
            const double x = solve_triangle<false>(tid < bw ? v[b0 + tid] : 0.0, T, rd, bw);
            if (tid < bw) v[b0 + tid] = x;
            __syncthreads();
        } else {
            const int i = b0 + tid;   // the thread's row; past cw there is none
            double l[kWave];
            if (b1 < cw) {   // then bw == kWave
                const gdouble* li = global(F.L) + (c0 + min(i, cw - 1)) + (int64_t)(c0 + b0) * F.m;
#pragma unroll
                for (int k = 0; k < kWave; ++k) l[k] = li[(int64_t)k * F.m];
            }
            __syncthreads();
            if (i < cw && b1 < cw) {
                double acc = v[i];
#pragma unroll
                for (int k = 0; k < kWave; ++k) acc = fma(-l[k], v[b0 + k], acc);
                v[i] = acc;
            }
        }
        __syncthreads();
    }
    if (tid < cw) xs[c0 + tid] = v[tid];
}

// forward, task a = chunk, b = row block: 64 rows i >= c1, v[i] -= L[i, c0:c1)
// x[c0, c1), in xp (i < w) or in the update vector (i >= w); a row per lane, a
// quarter of the chunk's columns per wave, the quarters added in order (a row
// per thread over the whole chunk left most of the chip idle: 10.5 us per launch,
// now 5.7).
__global__ void __launch_bounds__(kBlock)
k_bigfwd_gemv(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred) {
    static_assert(kSolveRows == kWave && kChunk % (kBlock / kWave) == 0, "a row per lane, equal shares of the columns");
    constexpr int kPart = kChunk / (kBlock / kWave);
    __shared__ double x[kChunk];
    __shared__ double sum[kBlock / kWave][kWave];
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const Front F = front_of(tk);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int c0 = tk.a * kChunk, cw = min(kChunk, F.w - c0), c1 = c0 + cw;
    const int i = c1 + tk.b * kSolveRows + lane;
    const gdouble* Li = global(F.L) + min(i, F.m - 1) + (int64_t)c0 * F.m;
    double* out = fwd_entry(I, F, tk, min(i, F.m - 1));
    const double xv = tid < cw ? global(I.xp)[F.f + c0 + tid] : 0.0;
    const double old = wv == 0 ? *global(out) : 0.0;
    double l[kPart];
#pragma unroll
    for (int k = 0; k < kPart; ++k) l[k] = Li[(int64_t)min(kPart * wv + k, cw - 1) * F.m];
    x[tid] = xv;
    __syncthreads();
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kPart; ++k) acc = fma(l[k], x[kPart * wv + k], acc);
    sum[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && i < F.m) *global(out) = old - (((sum[0][lane] + sum[1][lane]) + sum[2][lane]) + sum[3][lane]);
}

// backward, task a = column block: bsum[f + k] = L[w:m, k]^T x(rows below) for the
// block's kSolveCols columns: the rows' solution is gathered into shared memory
// once (kBelow rows at a time), then wave v takes columns k0 + v, k0 + v + 4,
// ..., all at once, lanes over the rows (a butterfly sums the lanes).  Gathered
// per column it took 18 us per launch (32 x 32 x 50 plate), now 9.
constexpr int kBelow = 2048;
__global__ void __launch_bounds__(kBlock)
k_bigbwd_below(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred) {
    constexpr int kPer = kSolveCols / (kBlock / kWave);   // columns per wave
    __shared__ double x[kBelow];
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const Front F = front_of(tk);
    const int32_t* rows = I.S.rows + uniform_at(I.S.rows_ptr, tk.sn);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave, nw = kBlock / kWave;
    const int k0 = tk.a * kSolveCols;
    const gdouble* col[kPer];
    double acc[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        col[q] = global(F.L) + (int64_t)min(k0 + wv + q * nw, F.w - 1) * F.m;
        acc[q] = 0.0;
    }
    for (int base = F.w; base < F.m; base += kBelow) {
        const int len = min(kBelow, F.m - base);
        if (base > F.w) __syncthreads();
        {
            int at[kBelow / kBlock];
            double g[kBelow / kBlock];
#pragma unroll
            for (int u = 0; u < kBelow / kBlock; ++u) at[u] = global(rows)[base + min(tid + u * kBlock, len - 1)];
#pragma unroll
            for (int u = 0; u < kBelow / kBlock; ++u) g[u] = global(I.xp)[at[u]];
#pragma unroll
            for (int u = 0; u < kBelow / kBlock; ++u) x[tid + u * kBlock] = g[u];
        }
        __syncthreads();
        constexpr int kDepth = 4;   // rows per lane whose loads are in flight together
        for (int i0 = lane; i0 < len; i0 += kDepth * kWave) {
            double l[kDepth][kPer];
#pragma unroll
            for (int u = 0; u < kDepth; ++u)
#pragma unroll
                for (int q = 0; q < kPer; ++q) l[u][q] = col[q][base + min(i0 + u * kWave, len - 1)];
#pragma unroll
            for (int u = 0; u < kDepth; ++u)
                if (i0 + u * kWave < len) {
                    const double xv = x[i0 + u * kWave];
#pragma unroll
                    for (int q = 0; q < kPer; ++q) acc[q] = fma(l[u][q], xv, acc[q]);
                }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int q = 0; q < kPer; ++q) acc[q] += __shfl_xor(acc[q], off, kWave);
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (lane == 0 && k0 + wv + q * nw < F.w) I.bsum[F.f + k0 + wv + q * nw] = acc[q];
}

// Whether bsum of a chunk's columns holds contributions: rows below the
// supernode, or a later chunk.
__device__ inline bool bsum_live(const Front& F, int c) { return F.m > F.w || (c + 1) * kChunk < F.w; }

// backward, task a = chunk: v = xp[c0, c1) - bsum; solve L[c0:c1, c0:c1]^T x = v
// by blocks of 64 from the last: wave 0 solves the block's staged triangle while
// the other waves bring its rows of the chunk's earlier columns into shared
// memory (coalesced), from where a thread per column takes the update.  With each
// thread reading its own column, 64 cache lines per load, a launch took 26 us
// (32 x 32 x 50 plate), now 13.  Writes xp and the unpermuted solution.
__global__ void __launch_bounds__(kBlock)
k_bigbwd_tri(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred, int which) {
    constexpr int kWaves = kBlock / kWave - 1;   // that load
    __shared__ double T[kTri];
    __shared__ double O[(kChunk - kWave) * (kWave + 1)];   // O[i + j (kWave + 1)] = L[b0 + i, j]
    __shared__ double rd[kWave];
    __shared__ double v[kChunk];
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const Front F = front_of(tk);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c0 = tk.a * kChunk, cw = min(kChunk, F.w - c0);
    const bool live = bsum_live(F, tk.a);
    const int nblk = (cw + kWave - 1) / kWave;
    double t[kStage];
    load_triangle(F, c0 + (nblk - 1) * kWave, cw - (nblk - 1) * kWave, t);
    const int pk = tid < cw ? global(I.perm)[F.f + c0 + tid] : 0;
    if (tid < cw) v[tid] = global(I.xp)[F.f + c0 + tid] - (live ? global(I.bsum)[F.f + c0 + tid] : 0.0);
    for (int bi = nblk - 1; bi >= 0; --bi) {
        const int b0 = bi * kWave, bw = min(kWave, cw - b0);
        store_triangle(t, bw, T, rd);
        __syncthreads();
        if (bi > 0) load_triangle(F, c0 + b0 - kWave, kWave, t);
        if (wv == 0) {
            const double x = solve_triangle<true>(tid < bw ? v[b0 + tid] : 0.0, T, rd, bw);
            v[b0 + tid] = tid < bw ? x : 0.0;
        } else if (bi > 0) {
            // columns wv - 1, wv - 1 + 3, ... < b0, 32 loads in flight
            const gdouble* li = global(F.L) + (c0 + b0 + min(lane, bw - 1)) + (int64_t)c0 * F.m;
            for (int j0 = wv - 1; j0 < b0; j0 += 32 * kWaves) {
                double l[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) l[u] = li[(int64_t)min(j0 + u * kWaves, b0 - 1) * F.m];
#pragma unroll
                for (int u = 0; u < 32; ++u) O[lane + min(j0 + u * kWaves, b0 - 1) * (kWave + 1)] = lane < bw ? l[u] : 0.0;
            }
        }
        __syncthreads();
        if (tid < b0) {
            double acc = v[tid];
            const double* o = O + tid * (kWave + 1);
#pragma unroll
            for (int i = 0; i < kWave; ++i) acc = fma(-o[i], v[b0 + i], acc);
            v[tid] = acc;
        }
        __syncthreads();
    }
    if (tid < cw) {
        global(I.xp)[F.f + c0 + tid] = v[tid];
        global(solve_out(I, which))[pk] = v[tid];
    }
}

// backward, task a = chunk, b = column block: for the block's columns
// k < c0, bsum[f + k] (+)= L[c0:c1, k]^T x[c0, c1) (the first contribution of a
// supernode without rows below sets it); wave per column, lanes over the rows.
__global__ void __launch_bounds__(kBlock)
k_bigbwd_gemvt(const InstPtrs* __restrict__ Ia, const BigTask* __restrict__ tasks, int pred) {
    __shared__ double x[kChunk];
    const BigTask tk = tasks[blockIdx.x];
    const InstPtrs& I = Ia[tk.inst];
    if (!ctl_active(I.ctl, pred)) return;
    const Front F = front_of(tk);
    const int c0 = tk.a * kChunk, cw = min(kChunk, F.w - c0);
    for (int k = threadIdx.x; k < cw; k += blockDim.x) x[k] = I.xp[F.f + c0 + k];
    __syncthreads();
    const bool live = bsum_live(F, tk.a);
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave, nw = blockDim.x / kWave;
    const int k0 = tk.b * kSolveCols;
    for (int k = k0 + wv; k < min(c0, k0 + kSolveCols); k += nw) {
        const gdouble* lk = global(F.L) + (int64_t)k * F.m + c0;
        double acc = 0.0;
        for (int i = lane; i < cw; i += kWave) acc = fma(lk[i], x[i], acc);
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
        if (lane == 0) I.bsum[F.f + k] = (live ? I.bsum[F.f + k] : 0.0) + acc;
    }
}

}  // namespace

int big_row_block() { return kRowBlock; }
int big_gather_rows() { return kBlock; }
int big_tile() { return kTile; }
int big_solve_rows() { return kSolveRows; }
int big_solve_cols() { return kSolveCols; }
int big_chunk() { return kChunk; }

void launch_big(int kind, int pred, double eta_force, int which, const InstPtrs* I, const BigTask* tasks, int count,
                hipStream_t st) {
    if (count <= 0) return;
    switch (kind) {
        case kBigAssemble:
            hipLaunchKernelGGL(k_big_assemble, dim3(count), dim3(kBigAsmCols * kWave), 0, st, I, tasks, pred, eta_force);
            break;
        case kBigPanelStep:
            hipLaunchKernelGGL(k_big_panel<false>, dim3(count), dim3(kPanelThreads), 0, st, I, tasks, pred);
            break;
        case kBigPanelReplace:
            hipLaunchKernelGGL(k_big_panel<true>, dim3(count), dim3(kPanelThreads), 0, st, I, tasks, pred);
            break;
        case kBigUpdate:
            hipLaunchKernelGGL(k_big_update<false>, dim3(count), dim3(kBlock), 0, st, I, tasks, pred);
            break;
        case kBigUpdateInner:
            hipLaunchKernelGGL(k_big_update<true>, dim3(count), dim3(kBlock), 0, st, I, tasks, pred);
            break;
        case kBigFwdGather:
            hipLaunchKernelGGL(k_bigfwd_gather, dim3(count), dim3(kBlock), 0, st, I, tasks, pred, which);
            break;
        case kBigFwdTri:
            hipLaunchKernelGGL(k_bigfwd_tri, dim3(count), dim3(kBlock), 0, st, I, tasks, pred);
            break;
        case kBigFwdGemv:
            hipLaunchKernelGGL(k_bigfwd_gemv, dim3(count), dim3(kBlock), 0, st, I, tasks, pred);
            break;
        case kBigBwdBelow:
            hipLaunchKernelGGL(k_bigbwd_below, dim3(count), dim3(kBlock), 0, st, I, tasks, pred);
            break;
        case kBigBwdTri:
            hipLaunchKernelGGL(k_bigbwd_tri, dim3(count), dim3(kBlock), 0, st, I, tasks, pred, which);
            break;
        case kBigBwdGemvT:
            hipLaunchKernelGGL(k_bigbwd_gemvt, dim3(count), dim3(kBlock), 0, st, I, tasks, pred);
            break;
        default:
            break;
    }
}

}  // namespace nmpc
