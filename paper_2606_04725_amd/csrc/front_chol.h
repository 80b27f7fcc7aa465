// Dense partial Cholesky of a front held in shared memory (the small-front
// kernels), and the lane broadcasts the large-front path shares with it.
#pragma once

#include <cmath>
#include <type_traits>

#include "front_rules.h"

namespace nmpc {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// A front's lower triangle packed by columns: column j holds rows j .. m-1, and
// base(j) + i is the position of entry (i, j), i >= j.  Front orders stay far
// below 2^12, so the products fit the full-rate 24-bit multiplier.
struct PackedIdx {
    int m;
    __device__ int base(int j) const { return __mul24(j, m) - (__mul24(j, j + 1) >> 1); }
    __device__ int operator()(int i, int j) const { return base(j) + i; }
};

// Tiles of a lower trapezoid of nt tile rows and nc <= nt tile columns, in
// row order: the triangle of the first nc rows, then nc tiles per row.
__device__ inline int tile_count(int nt, int nc) { return (__mul24(nc, nc + 1) >> 1) + __mul24(nt - nc, nc); }
__device__ inline void tile_of(int tt, int nc, int& ti, int& tj) {
    const int tri = __mul24(nc, nc + 1) >> 1;
    if (tt < tri) {   // tile row ti holds tiles ti (ti + 1) / 2 ...: single-precision root, integer correction
        ti = (int)((sqrtf(8.0f * (float)tt + 1.0f) - 1.0f) * 0.5f);
        while ((__mul24(ti + 1, ti + 2) >> 1) <= tt) ++ti;
        while ((__mul24(ti, ti + 1) >> 1) > tt) --ti;
        tj = tt - (__mul24(ti, ti + 1) >> 1);
    } else {
        const int r = tt - tri;
        ti = nc + r / nc;
        tj = r - __mul24(ti - nc, nc);
    }
}

// Value of v in lane K of the caller's 16-lane group, in every lane of the
// group (a row broadcast of the vector unit, no shared memory).
template <int K>
__device__ __attribute__((always_inline)) inline double group_lane(double v) {
    return __builtin_amdgcn_mov_dpp(v, 0x150 + K, 0xf, 0xf, true);   // row_newbcast:K
}

// f(0), ..., f(N - 1) with compile-time arguments.
template <int N, class F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f) {
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Value of v in lane K of the wave, in every lane (through the scalar unit).
template <int K>
__device__ __attribute__((always_inline)) inline double wave_lane(double v) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), K);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), K);
    return __hiloint2double(hi, lo);
}

// kSolveSteps columns, k0 .. k0 + kSolveSteps - 1, of a triangular solve on one
// wave: lane j holds v_j and the reciprocal r of its diagonal entry, c[u] is its
// entry of column k0 + u, zero where a step does not touch the lane.  The
// columns go upwards or, Back, downwards; x_k = v_k r_k leaves lane k through
// the scalar unit.  With the coefficients ready a step is a product, two lane
// reads and one multiply-add, about 30 cycles; read and selected in each step
// they made it 100.
constexpr int kSolveSteps = 16;
template <bool Back>
__device__ __attribute__((always_inline)) inline double solve_steps(double v, double r, const double (&c)[kSolveSteps], int k0) {
#pragma unroll
    for (int u = 0; u < kSolveSteps; ++u) {
        const int q = Back ? kSolveSteps - 1 - u : u;
        const double y = v * r;
        const int lo = __builtin_amdgcn_readlane(__double2loint(y), k0 + q);
        const int hi = __builtin_amdgcn_readlane(__double2hiint(y), k0 + q);
        v = fma(-c[q], __hiloint2double(hi, lo), v);
    }
    return v;
}

// 1 / sqrt(pivot), the hardware estimate y and one third-order step in 1 - pivot
// y^2; not finite for a pivot that is not positive and finite.  The product
// pivot y is the size of the root, so that it and its rounding, which the
// residual takes in, are normal numbers for every positive pivot: y^2 overflows
// for pivots below 5.6e-309, and is subnormal itself for those above 4.5e307.
__device__ __attribute__((always_inline)) inline double pivot_rsqrt(double piv) {
    const double y = __builtin_amdgcn_rsq(piv);
    const double p = piv * y, e = fma(-fma(piv, y, -p), y, fma(-p, y, 1.0));
    return fma(fma(e, 0.375, 0.5), y * e, y);
}

// kw <= P pivot columns of the rows one wave holds, a row per lane and the pivot
// rows in its first lanes: a[c] is the row's entry in column c, L(row, c) on
// return (c < kw; the columns after them hold no result).
// A pivot row's value L(j, k) reaches every lane through the scalar unit, so
// pivots, rows below and a right-hand side in a row of its own all go in the
// same instructions; a column's lane reads all come before its products (read
// and used in turn, each pair waits for the scalar unit: 5400 cycles for P = 16
// against 3000).  A lone wave issues about one instruction in 4 to 5 cycles,
// which bounds this.  The next pivot's reciprocal root is formed while the other
// columns take their updates.
// The second eight columns take the first eight's products as a sum formed from
// zero: subtracted from the entry one by one they round at the entry's size, and
// the error of a factorization and solve against 64 bits (300 matrices of plates
// of 8 to 48 points a side) was 0.8 % above that of panels of eight columns;
// with the sum it is 2.7 % below, in the same time (28 x 37 plate 1.000x, 40 x
// 100 column 0.997x).
// A pivot that is not positive and finite makes its reciprocal root, and through
// the updates every later one, not finite: only the last of the kw is tested
// (tested and replaced one by one they cost 7 instructions of a pivot's 27).
// Replace does that: such a pivot counts as 1, and what a matrix that is not
// positive definite leaves is a factor all the same; nothing is reported then.
template <int P, bool Replace>
__device__ __attribute__((always_inline)) inline bool factor_rows(double (&a)[16], int kw) {
    if constexpr (Replace) {
        const int lane = threadIdx.x & (kCholWave - 1);
        static_for<P>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            double piv = wave_lane<k>(a[k]);
            if (!(piv > 0.0) || !(piv < INFINITY)) piv = 1.0;
            a[k] = (lane == k ? piv : a[k]) * pivot_rsqrt(piv);
            static_for<P - 1 - k>([&](auto jc) {
                constexpr int j = k + 1 + decltype(jc)::value;
                a[j] = fma(-a[k], wave_lane<j>(a[k]), a[j]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        return false;
    }
    constexpr int H = 8;
    double inv = pivot_rsqrt(wave_lane<0>(a[0])), last = inv, sum[P > H ? P - H : 1] = {};
    static_for<P>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        a[k] *= inv;
        double b[P];
        static_for<P - 1 - k>([&](auto jc) {
            constexpr int j = k + 1 + decltype(jc)::value;
            b[j] = wave_lane<j>(a[k]);
        });
        static_for<P - 1 - k>([&](auto jc) {
            constexpr int j = k + 1 + decltype(jc)::value;
            if constexpr (k >= H || j < H) a[j] = fma(-a[k], b[j], a[j]);
            else if constexpr (k == 0) sum[j - H] = a[k] * b[j];
            else sum[j - H] = fma(a[k], b[j], sum[j - H]);
            if constexpr (k == H - 1 && j >= H) a[j] -= sum[j - H];
            if constexpr (j == k + 1) {
                inv = pivot_rsqrt(wave_lane<j>(a[j]));
                last = j < kw ? inv : last;
            }
        });
        __builtin_amdgcn_sched_barrier(0);   // one pivot at a time: the next ones' lane reads would fill the registers
    });
    return !(fabs(last) < INFINITY);
}

// Steps 1 and 2 of pivot columns [kb, kb + kw), kw <= 16: wave 0 holds rows kb
// .. kb + 63, wave v the 16 rows from kb (again, for their pivots) and 48 more.
// Rows below the block go back at once, the block after the next barrier
// (store_pivot_block, from a of wave 0): other waves may still read it.
template <bool Replace>
__device__ __attribute__((always_inline)) inline void panel_solve(double* F, PackedIdx ix, int kb, int kw, int* fail,
                                                                 double (&a)[16]) {
    const int lane = threadIdx.x & (kCholWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kCholWave);
    const int m = ix.m, own = panel_wave_begin(kb, wv);   // the row of lane 16
    if (wv != 0 && own >= m) return;
    const int r = lane < 16 ? kb + lane : own - 16 + lane;
    {
        // loads without a branch: rows clamped into the front, columns into the
        // panel; entries above the block's diagonal read some other entry of
        // the front (they only reach values that are never used)
        int at = ix.base(kb) + min(r, m - 1);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            a[c] = F[at];
            at += c + 1 < kw ? m - 1 - (kb + c) : 0;   // to the same row of the next column
        }
    }
    const bool bad = kw > 8 ? factor_rows<16, Replace>(a, kw) : factor_rows<8, Replace>(a, kw);
    if (bad && threadIdx.x == 0) *global(fail) = 1;
    if (lane >= (wv == 0 ? kw : 16) && r < m) {
        int at = ix.base(kb) + r;
        if (kw == 16) {
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                F[at] = a[c];
                at += m - 1 - (kb + c);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 15; ++c) {
                if (c < kw) F[at] = a[c];
                at += m - 1 - (kb + c);
            }
        }
    }
}

// The factored pivot block into the front by the first lanes of wave 0 (every
// wave that read it has passed the barrier before this call).  A lane's entries
// above the diagonal go to the spare slot: no branch per entry.
__device__ __attribute__((always_inline)) inline void store_pivot_block(double* F, PackedIdx ix, int kb, int kw, int spare,
                                                                       const double (&a)[16]) {
    const int li = threadIdx.x;
    if (li >= kw) return;
    int at = ix.base(kb) + kb + li;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        F[c <= li ? at : spare] = a[c];
        at += ix.m - 1 - (kb + c);
    }
}

// Step 3 on one 16 x 16 tile (ti, tj) of the lower trapezoid right of and
// below the 16 pivot columns from kb: rows [t0, m), columns [t0, w), t0 = kb +
// 16.  One v_mfma_f64_16x16x4f64 per 4 pivot columns.  Everything is loaded
// without a branch: operands from clamped rows, the tile's entries from their
// place or, outside the trapezoid, the spare slot, where they also go back.
__device__ __attribute__((always_inline)) inline void trapezoid_tile(double* F, PackedIdx ix, int w, int kb, int spare, int ti,
                                                                    int tj) {
    const int m = ix.m, lane = threadIdx.x & (kCholWave - 1), li = lane & 15, lk = lane >> 4;
    const int i0 = kb + 16 + 16 * ti, j0 = kb + 16 + 16 * tj;
    const int ra = min(i0 + li, m - 1), rb = min(j0 + li, m - 1);
    const int jc = j0 + li, cb = ix.base(min(jc, w - 1));
    int at[4];
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};   // from zero: its roundings are the products' size, not the entries'
    double own[4], av[4], bv[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
        const double* col = F + ix.base(kb + 4 * s4 + lk);
        av[s4] = col[ra];
        bv[s4] = col[rb];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int ir = i0 + 4 * r + lk;
        at[r] = (ir < m && jc <= ir && jc < w) ? cb + ir : spare;
        own[r] = F[at[r]];
    }
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s4], bv[s4], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) F[at[r]] = own[r] - acc[r];
}

// The update block of the front (rows and columns [w, m)) minus L21 L21^T,
// L21 = the panel's rows [w, m): pairs of 16 x 16 tiles of one tile row over
// the waves (a pair shares its row operand), two accumulators per tile so that
// four products are in flight (a dependent one waits 67 cycles, four
// independent ones take 80), each entry read and written once.
__device__ __attribute__((always_inline)) inline void update_block(double* F, PackedIdx ix, int w, int spare) {
    const int m = ix.m, tid = threadIdx.x;
    const int lane = tid & (kCholWave - 1), wv = __builtin_amdgcn_readfirstlane(tid / kCholWave), nw = blockDim.x / kCholWave;
    const int li = lane & 15, lk = lane >> 4;
    const int nt = (m - w + 15) / 16;
    int ti = 0, tp = wv;   // tile row ti holds pairs 0 .. ti / 2
    while (ti < nt && tp > ti / 2) {
        tp -= ti / 2 + 1;
        ++ti;
    }
    while (ti < nt) {
        const int i0 = w + 16 * ti, j0 = w + 32 * tp;
        const int ra = min(i0 + li, m - 1), rb0 = min(j0 + li, m - 1), rb1 = min(j0 + 16 + li, m - 1);
        int at[2][4];
        f64x4 own[2], acc[2][2];   // from zero, as in the tiles of the panels
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int jc = j0 + 16 * q + li, cb = ix.base(min(jc, m - 1));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ir = i0 + 4 * r + lk;
                at[q][r] = (ir < m && jc <= ir) ? cb + ir : spare;
                own[q][r] = F[at[q][r]];
                acc[q][0][r] = acc[q][1][r] = 0.0;
            }
        }
        // eight columns at a time: six operands, then the products; rows past
        // m repeat row m - 1 (their results go to the spare slot), columns
        // past w are zeroed
        for (int k8 = 0; k8 < w; k8 += 8) {
            double a[2], b0[2], b1[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int kk = k8 + 4 * u + lk;
                const double* col = F + ix.base(min(kk, w - 1));
                a[u] = col[ra];
                b0[u] = col[rb0];
                b1[u] = col[rb1];
                a[u] = kk < w ? a[u] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                acc[0][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b0[u], acc[0][u], 0, 0, 0);
                acc[1][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b1[u], acc[1][u], 0, 0, 0);
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) F[at[q][r]] = own[q][r] - (acc[q][0][r] + acc[q][1][r]);
        tp += nw;
        while (ti < nt && tp > ti / 2) {
            tp -= ti / 2 + 1;
            ++ti;
        }
    }
    __syncthreads();
}

// Right-looking partial Cholesky of the first w columns of a front (packed lower
// triangle of order m = ix.m), 16 pivot columns at a time:
//  1. every wave that owns rows below the block (and wave 0) factors the
//     diagonal block itself, in registers (identical arithmetic, no
//     communication), and
//  2. solves its rows of the panel against it in the same steps (panel_solve);
//  3. the panel's remaining columns take the rank-16 update on the matrix
//     cores in 16 x 16 tiles: first the tile column holding the next pivot
//     columns, then, after a barrier, the other tiles on the waves that have no
//     rows of the next panel, while the waves that do run steps 1 and 2 of the
//     next panel (the two touch different columns).
// The update block (rows and columns w and on) is left to update_block.  A row
// that holds a right-hand side is solved (and updated) like any other: the
// factored columns of that row are the forward substitution.
// A pivot that is not positive and finite sets *fail (eq. 12: the matrix is not
// numerically positive definite) and the values are not finite from there on,
// or, with Replace, it counts as 1 and nothing is reported.
// spare: a shared-memory slot (an index into F) that takes what lies outside.
template <bool Replace>
__device__ __attribute__((always_inline)) inline void partial_cholesky(double* F, PackedIdx ix, int w, int spare, int* fail) {
    constexpr int P = 16;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kCholWave), nw = blockDim.x / kCholWave;
    const int m = ix.m;
    double a[P];
    for (int kb = 0; kb < w; kb += P) {
        const int kw = min(P, w - kb), t0 = kb + kw;
        if (kb > 0) {   // the rest of the previous panel's update
            const int nt = (m - kb + 15) / 16, nc = (w - kb + 15) / 16;
            // waves with rows of this panel (wave 0 always takes part)
            const int busy = min(nw, 1 + max(0, (m - kb - kCholWave + kRowsPerWave - 1) / kRowsPerWave));
            const int rest = tile_count(nt - 1, nc - 1);
            const int first = busy < nw ? wv - busy : wv, stride = busy < nw ? nw - busy : nw;
            if (first >= 0)
                for (int tt = first; tt < rest; tt += stride) {
                    int ti, tj;
                    tile_of(tt, nc - 1, ti, tj);
                    trapezoid_tile(F, ix, w, kb - P, spare, ti + 1, tj + 1);
                }
        }
        panel_solve<Replace>(F, ix, kb, kw, fail, a);
        __syncthreads();
        if (wv == 0) store_pivot_block(F, ix, kb, kw, spare, a);
        if (t0 < w) {
            const int nt = (m - t0 + 15) / 16;
            for (int ti = nw - 1 - wv; ti < nt; ti += nw) trapezoid_tile(F, ix, w, kb, spare, ti, 0);
        }
        __syncthreads();
    }
}

}  // namespace nmpc
