// HIP kernels of the Dey--Mittra eigensolver (gfx950, wave64).
//
// A cell (i,j,k) owns its three low faces b_x[i,j,k], b_y[i,j,k], b_z[i,j,k].
// Transfers, K and the scalar kernels map one thread to one cell; the smoother
// and M take listed cut rows and, beside them, runs of vacuum rows or, over
// the whole grid, cells by class byte.  Blocks are remapped so that
// each of the 8 XCDs (which receive workgroups round-robin) works on one
// contiguous slab of the grid and keeps its stencil neighbours in its own L2.
// The stencil path is memory bound: no MFMA here.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>
#include <type_traits>

#include "dm_internal.h"

namespace dm {

namespace {

constexpr int kThreads = 256;
constexpr int kXcd = 8;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// grid of `n` work items in blocks of kThreads, padded to a multiple of 8 blocks
inline dim3 xcd_grid(int64_t n) {
    int64_t nb = ceil_div(n, kThreads);
    int64_t per = ceil_div(nb, kXcd);
    return dim3((unsigned)(per * kXcd));
}

// logical block of this workgroup: XCD x gets blocks [x*per, (x+1)*per)
__device__ inline int64_t xcd_item() {
    const int64_t per = gridDim.x / kXcd;
    const int64_t b = blockIdx.x;
    const int64_t logical = (b % kXcd) * per + b / kXcd;
    return logical * kThreads + threadIdx.x;
}

// Block kernels over nr vectors: a workgroup of 64 * nr threads takes 64
// consecutive items, wave q the vector q (coalesced loads per wave; the waves
// of a workgroup share the coefficient lines of their cells in the CU's
// cache).  Grid: ceil(items / 64) workgroups, padded to a multiple of 8.
inline dim3 xcd_grid_waves(int64_t items) {
    int64_t nb = ceil_div(items, 64);
    int64_t per = ceil_div(nb, kXcd);
    return dim3((unsigned)(per * kXcd));
}

__device__ inline int64_t wave_item(int &q) {
    const int64_t per = gridDim.x / kXcd;
    const int64_t b = blockIdx.x;
    const int64_t logical = (b % kXcd) * per + b / kXcd;
    q = threadIdx.x >> 6;
    return logical * 64 + (threadIdx.x & 63);
}

// item t (x fastest) -> cell; false past the grid.  A grid has fewer than 2^31
// padded elements (checked when the operator is built), so the divisions are
// 32-bit ones.
__device__ inline bool cell_of(const Grid &g, int64_t t, int &i, int &j, int &k) {
    if (t >= (int64_t)g.nx * g.ny * g.nz) return false;
    const uint32_t u = (uint32_t)t, nx = (uint32_t)g.nx, ny = (uint32_t)g.ny;
    const uint32_t r = u / nx, kk = r / ny;
    i = (int)(u - r * nx);
    j = (int)(r - kk * ny);
    k = (int)kk;
    return true;
}

// Item t of a launch over listed grid rows (k * ny + j, ascending) -> the
// cell item of the whole grid (past its end for t past the listed rows);
// without a list the item itself
__device__ inline int64_t listed_item(const Grid &g, const int32_t *rows, int64_t nrows, int64_t t) {
    if (!rows) return t;
    if (t >= nrows * g.nx) return (int64_t)g.nx * g.ny * g.nz;
    const uint32_t u = (uint32_t)t, nx = (uint32_t)g.nx, r = u / nx;
    return (int64_t)rows[r] * g.nx + (u - r * nx);
}

template <class T>
__device__ inline T inv_h2_of(const Grid &g) {
    return (T)(1.0 / (g.h * g.h));
}

// ---------------------------------------------------------------------------
// y = M x, y = K x, or r = f - M x
// ---------------------------------------------------------------------------
// The rows below are formed in several kernels (launched class updates, sweeps
// in LDS, apply and residual, one vector or a block), and a value may not
// depend on which of them formed it: where a product and a sum may or may not
// be contracted, the fused multiply-add is written out, with the row's largest
// term as the product that is not rounded.  (Left to the compiler, the sweeps
// in LDS rounded w_0 x_p of a cut row first: 4% more error in the FP32 V-cycle
// of the 16^3 sphere.)
__device__ inline float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }

// 7-point vacuum row of component array C at p (no 1/h^2)
template <class T, class TX = T>
__device__ inline T vac_row(const TX *C, int64_t p, int64_t dy, int64_t dz) {
    return fused(T(6), T(C[p]), -(T(C[p - 1]) + T(C[p + 1]))) - (T(C[p - dy]) + T(C[p + dy])) -
           (T(C[p - dz]) + T(C[p + dz]));
}

// the vacuum row of M at p, whose value is xp
template <class T, class TX = T>
__device__ inline T vac_row_m(const TX *C, int64_t p, int64_t dy, int64_t dz, T ih2, T sigma, T xp) {
    return fused(ih2, vac_row<T, TX>(C, p, dy, dz), -(sigma * xp));
}

// A table of cut rows as the kernels take it (kCutW x n, term-major; see
// cut_term): the weights in the vectors' type, the centre ones (w0, the term 0
// of a table of the same layout) in the type of the sums.
template <class T, class TA>
struct CutTab {
    const T *w;
    const TA *w0;
};

// the centre terms of a tabulated row: w_0 x_p - sigma a x_p
template <class T>
__device__ inline T centre_terms(T w0, T sigma, T a, T xp) {
    return fused(w0, xp, -(sigma * a * xp));
}

// y = K x: rows keep their curl-curl cross terms (no vacuum shortcut)
template <class T>
__device__ __forceinline__ void apply_k_body(const Grid &g, const Coefs<T> &c, const T *__restrict__ x,
                                             T *__restrict__ y, int64_t item) {
    int i, j, k;
    if (!cell_of(g, item, i, j, k)) return;
    const int64_t P = g.P, dy = g.sy, dz = g.sz;
    const int64_t p = pidx(g, i, j, k);
    const T *X = x, *Y = x + P, *Z = x + 2 * P;
    const T ih2 = inv_h2_of<T>(g);
    const uint8_t fl = c.flags[p];
    T yx = T(0), yy = T(0), yz = T(0);
    if (fl & (kFaceActive << 0)) yx = ih2 * row_x<T, false>(c, X, Y, Z, p, dy, dz);
    if (fl & (kFaceActive << 1)) yy = ih2 * row_y<T, false>(c, X, Y, Z, p, dy, dz);
    if (fl & (kFaceActive << 2)) yz = ih2 * row_z<T, false>(c, X, Y, Z, p, dy, dz);
    put_face<T>(g, y, 0, i, j, k, p, yx);
    put_face<T>(g, y + P, 1, i, j, k, p, yy);
    put_face<T>(g, y + 2 * P, 2, i, j, k, p, yz);
}

// put_face from a padded index: the cell's coordinates are only worked out
// where a PMC plane asks for ghost images
template <class T>
__device__ __forceinline__ void put_face_at(const Grid &g, T *arr, int comp, uint32_t p, T v) {
    if (!g.pmc) {
        arr[p] = v;
        return;
    }
    const uint32_t sy = (uint32_t)g.sy, sz = (uint32_t)g.sz;
    const uint32_t kk = p / sz, rr = p - kk * sz, jj = rr / sy;
    put_face<T>(g, arr, comp, (int)(rr - jj * sy) - 1, (int)jj - 1, (int)kk - 1, (int64_t)p, v);
}

// M x or f - M x at the cell of padded index p whose active rows are all
// vacuum rows (the other cells are listed and run the full body): the same
// values, written the same way, zeros on the inactive components included.
// act: bit c, the face of component c is active; image: the cell may have PMC
// ghost images.  (K alone has no vacuum shortcut: its rows keep the cross
// terms.)
template <class T, int KIND, class TX = T>
__device__ __forceinline__ void apply_vac_body(const Grid &g, T sigma, uint32_t act, bool image, uint32_t p,
                                               const T *__restrict__ f, const TX *__restrict__ x,
                                               T *__restrict__ y) {
    static_assert(KIND == AK_M || KIND == AK_RESID, "vacuum rows of M only");
    const int64_t P = g.P, dy = g.sy, dz = g.sz;
    const T ih2 = inv_h2_of<T>(g);
    T v[3] = {T(0), T(0), T(0)};
    if (act) {
        // one branch for the three rows, so that all their loads are in flight
        // together (every cell of the grid has its neighbours in the padding)
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            const TX *C = x + comp * P;
            v[comp] = vac_row_m<T, TX>(C, p, dy, dz, ih2, sigma, T(C[p]));
            if (KIND == AK_RESID) v[comp] = f[comp * P + p] - v[comp];
            if (!((act >> comp) & 1)) v[comp] = T(0);
        }
    }
    if (g.pmc && image) {
        put_face_at<T>(g, y, 0, p, v[0]);
        put_face_at<T>(g, y + P, 1, p, v[1]);
        put_face_at<T>(g, y + 2 * P, 2, p, v[2]);
    } else {
        y[p] = v[0];
        (y + P)[p] = v[1];
        (y + 2 * P)[p] = v[2];
    }
}

// the same at lane `lane` of a run, where the run visits the cell
template <class T, int KIND, class TX = T>
__device__ __forceinline__ void apply_run(const Grid &g, T sigma, const CellRun &run, uint32_t lane,
                                          const T *__restrict__ f, const TX *__restrict__ x, T *__restrict__ y) {
    if (!((run.visit >> lane) & 1)) return;
    const uint32_t act = ((run.act[0] >> lane) & 1) | ((run.act[1] >> lane) & 1) << 1 | ((run.act[2] >> lane) & 1) << 2;
    apply_vac_body<T, KIND, TX>(g, sigma, act, (run.pmc & 2) || (run.pmc && lane < 2), (uint32_t)run.p + lane, f, x, y);
}

template <class T>
__global__ void __launch_bounds__(kThreads)
k_apply_K(Grid g, Coefs<T> c, const T *__restrict__ x, T *__restrict__ y) {
    apply_k_body<T>(g, c, x, y, xcd_item());
}

// M x or f - M x at the face of component COMP of listed cell e (padded index
// p) from its tabulated row in W (3 x kCutW x ncut; see CutTab), summed in TA;
// an inactive face (a = 0) gets 0
template <class T, int KIND, int COMP, class TX, class TA>
__device__ __forceinline__ void apply_cut_row(const Grid &g, T sigma, const CutTab<T, TA> &W, int64_t ncut,
                                              int64_t e, uint32_t p, const T *__restrict__ f,
                                              const TX *__restrict__ x, T *__restrict__ y) {
    const int64_t P = g.P, dy = g.sy, dz = g.sz;
    const int64_t off = (int64_t)COMP * kCutW * ncut;
    const T *__restrict__ Wc = W.w + off;
    const T a = Wc[kCutTerms * ncut + e];
    T v = T(0);
    if (a != T(0)) {
        TA row = centre_terms((W.w0 + off)[e], TA(sigma), TA(a), TA(x[COMP * P + p]));
#pragma unroll
        for (int t = 1; t < kCutTerms; ++t) {
            const CutTerm ct = cut_term(COMP, t);
            row += TA(Wc[t * ncut + e]) * TA(x[ct.comp * P + p + ct.di + ct.dj * dy + ct.dk * dz]);
        }
        v = T(KIND == AK_RESID ? TA(f[COMP * P + p]) - row : row);
    }
    put_face_at<T>(g, y + COMP * P, COMP, p, v);
}

// entry i of the cut part: component i mod 3 of the 64 listed cells i / 3 of
// a wave, or (not split) the rows of the 64 listed cells i, one after the
// other (see kApplySplit)
template <class T, int KIND, class TX, class TA>
__device__ __forceinline__ void apply_cut_part(const Grid &g, T sigma, const CutTab<T, TA> &W,
                                               const int32_t *__restrict__ cut, int64_t ncut, bool split, uint32_t i,
                                               uint32_t lane, const T *__restrict__ f, const TX *__restrict__ x,
                                               T *__restrict__ y) {
    const uint32_t c = split ? i / 3 : i, comp = i - 3 * c, e = c * 64 + lane;
    if (e >= ncut) return;
    const uint32_t p = (uint32_t)cut[e];
    if (!split || comp == 0) apply_cut_row<T, KIND, 0, TX, TA>(g, sigma, W, ncut, e, p, f, x, y);
    if (!split || comp == 1) apply_cut_row<T, KIND, 1, TX, TA>(g, sigma, W, ncut, e, p, f, x, y);
    if (!split || comp == 2) apply_cut_row<T, KIND, 2, TX, TA>(g, sigma, W, ncut, e, p, f, x, y);
}

// the cut cells (their rows' table W), and the runs of the others or, without
// them, the cells' class bytes
template <class T>
struct ApplyArgs {
    const int32_t *cut;
    const T *W;
    const CellRun *cells;
    const uint8_t *flags;
    int64_t ncut;
    uint32_t ncb, nruns, split;
};

// Block forms of apply, restriction and prolongation: wave q of a workgroup
// applies the one-vector body to vector q of the workgroup's 64 cells (see
// wave_item), so every lane keeps the register budget of the one-vector
// body.  (Looping over the vectors inside a thread kept every vector's loads
// and addresses live at once: 170-240 VGPRs, two waves per SIMD; giving the
// vectors to neighbouring lanes split every load of a wave over NR arrays.)

// The block apply in two parts, as the smoother's class updates: the first
// ncb workgroups (a multiple of 8) take the cut-cell list, the
// rest the other cells, those of the listed runs or, without a list, every
// cell of the grid by its class byte; wave q of a workgroup takes vector q of
// 64 entries in either part.  (A run's record is 16 bytes for each lane of
// the load, a class byte one: over the whole grid runs of 16 lanes were 1.5 to
// 3% slower, FP64 at 104 x 88 x 80 and 128 x 128 x 96; runs pay where they
// leave rows out.)
template <class T, int KIND, int NR, class TX = T>
__global__ void __launch_bounds__(kThreads)
k_apply_split(Grid g, T sigma, ApplyArgs<T> A, VPtr<const T> f, VPtr<const TX> x, VPtr<T> y) {
    const uint32_t b = blockIdx.x;
    const int q = threadIdx.x >> 6;
    if (b < A.ncb) {
        const uint32_t L = (b % kXcd) * (A.ncb / kXcd) + b / kXcd;
        apply_cut_part<T, KIND, TX, T>(g, sigma, CutTab<T, T>{A.W, A.W}, A.cut, A.ncut, A.split, L, threadIdx.x & 63, f.p[q], x.p[q], y.p[q]);
        return;
    }
    const uint32_t bv = b - A.ncb, nvb = gridDim.x - A.ncb;
    const uint32_t t = ((bv % kXcd) * (nvb / kXcd) + bv / kXcd) * 64 + (threadIdx.x & 63);
    if (A.cells) {
        if (t >> kRunLog >= A.nruns) return;
        apply_run<T, KIND, TX>(g, sigma, A.cells[t >> kRunLog], t & (kRunLanes - 1), f.p[q], x.p[q], y.p[q]);
    } else {
        int i, j, k;
        if (!cell_of(g, t, i, j, k)) return;
        const uint32_t p = (uint32_t)pidx(g, i, j, k), fl = A.flags[p];
        if (!((fl & 7) & ~(fl >> 3))) apply_vac_body<T, KIND, TX>(g, sigma, fl & 7, true, p, f.p[q], x.p[q], y.p[q]);
    }
}

// y = A x
template <class T>
__global__ void __launch_bounds__(kThreads)
k_apply_A(Grid g, Coefs<T> c, const T *__restrict__ x, T *__restrict__ y) {
    int i, j, k;
    if (!cell_of(g, xcd_item(), i, j, k)) return;
    const int64_t P = g.P, p = pidx(g, i, j, k);
    put_face<T>(g, y, 0, i, j, k, p, c.ax[p] * x[p]);
    put_face<T>(g, y + P, 1, i, j, k, p, c.ay[p] * x[P + p]);
    put_face<T>(g, y + 2 * P, 2, i, j, k, p, c.az[p] * x[2 * P + p]);
}

// ---------------------------------------------------------------------------
// Red-black Gauss--Seidel: one (component, colour) class, colour = (i+j+k)&1.
// Threads cover half the cells of each row: i = 2*ih + ((j+k+colour)&1).
// A thread also refreshes the PMC ghost images of the value it updates; no
// row of the same class reads those images except its own.
// ---------------------------------------------------------------------------
// The two parts of a class update: smooth_vac_n updates the class's vacuum
// rows from their runs, smooth_cut_n entry e of the component's list of
// non-vacuum rows.  Rows of one class do not read each other, so the parts
// may run in any order; separating them keeps the waves of the vacuum part
// on the short path (a cut row in a wave made the whole wave take the long
// path as well).
//
// Below the finest level a class update is bound by its launch (1.85 us for
// an empty node of a graph) and the latency of its dependent loads, so both
// parts keep that chain at two: the run (or the listed index), then
// everything else at once.  Walking listed grid rows instead (row number,
// then the cell's class byte, then the values, with 64-bit divisions in
// between) took 2.98 us per launch on the 32^3 level of one vector's V-cycle
// and 516 us for the whole V-cycle at 128^3; the runs took 2.67 and 476 us (now
// 435, with narrower runs and the small levels in LDS).
template <class T, int COMP, int NR>
__device__ __forceinline__ void smooth_vac_n(const Grid &g, T sigma, const VPtr<const T> &f, const VPtr<T> &x,
                                             uint32_t t, const VacRun *__restrict__ runs, uint32_t nruns) {
    const uint32_t r = t >> kRunLog;
    if (r >= nruns) return;
    const VacRun run = runs[r];
    const uint32_t lane = t & (kRunLanes - 1);
    if (!((run.mask >> lane) & 1)) return;
    const int64_t P = g.P, dy = g.sy, dz = g.sz;
    const uint32_t p = (uint32_t)run.p + 2 * lane;
    const T ih2 = inv_h2_of<T>(g);
    const T d = fused(T(6), ih2, -sigma);
    T nv[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const T *xc = x.p[q] + COMP * P;
        const T xp = xc[p];
        const T row = vac_row_m<T>(xc, p, dy, dz, ih2, sigma, xp);
        nv[q] = xp + (f.p[q][COMP * P + p] - row) / d;
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) (x.p[q] + COMP * P)[p] = nv[q];
    if (run.image && (COMP != 0 || lane == 0)) {
        const int64_t off = COMP * P - 2 * (COMP == 0 ? 1 : COMP == 1 ? dy : dz);
#pragma unroll
        for (int q = 0; q < NR; ++q) (x.p[q] + off)[p] = nv[q];
    }
}

// entry e of the component's cut list (n entries, the colour in the sign bit)
// from its tabulated row (kCutW x n; see CutTab), for the update of colour
// `colour` paired as `pair` says (see ClassList): the row is
// -sigma a x_f + (own-component terms) + (cross-component terms), the latter
// summed first, inline or taken from S (n per vector, vector q0 + q).  The
// weights are loaded once for the NR vectors, those that every entry takes
// before the index they do not depend on; the sums are in TA, the cross sums
// rounded to T whether they are stored or not.  (The list keeps both colours
// in index order: sorted by colour, the first update of a pair walked the
// surface twice, 16.5 -> 21.5 us per launch at 128^3 for 3 vectors.)
template <class T, int COMP, int NR, class TA>
__device__ __forceinline__ void smooth_cut_n(const Grid &g, T sigma, const int32_t *__restrict__ cut, int64_t n,
                                             int colour, const CutTab<T, TA> &tab, int pair, T *__restrict__ S,
                                             int q0, const VPtr<const T> &f, const VPtr<T> &x, uint32_t e) {
    const int64_t P = g.P, dy = g.sy, dz = g.sz;
    const T *__restrict__ W = tab.w;
    T w[kCutTerms], cross[NR];
    const int32_t ce = cut[e];
    if (pair != kPairSecond) {
#pragma unroll
        for (int t = kCutOwn; t < kCutTerms; ++t) w[t] = W[t * n + e];
    }
    const uint32_t p = (uint32_t)ce & 0x7fffffffu;
    // the other colour's rows: nothing, or (first of a pair) their cross sums
    const bool mine = (ce < 0) == (colour != 0);
    if (!mine && pair != kPairFirst) return;
    if (pair == kPairSecond) {
#pragma unroll
        for (int q = 0; q < NR; ++q) cross[q] = S[(int64_t)(q0 + q) * n + e];
    } else {
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const T *X = x.p[q];
            TA c = TA(0);
#pragma unroll
            for (int t = kCutOwn; t < kCutTerms; ++t) {
                const CutTerm ct = cut_term(COMP, t);
                c += TA(w[t]) * TA((X + (ct.comp * P + ct.di + ct.dj * dy + ct.dk * dz))[p]);
            }
            cross[q] = T(c);
        }
        if (!mine) {
#pragma unroll
            for (int q = 0; q < NR; ++q) S[(int64_t)(q0 + q) * n + e] = cross[q];
            return;
        }
    }
    const TA w0 = tab.w0[e];
#pragma unroll
    for (int t = 1; t < kCutOwn; ++t) w[t] = W[t * n + e];
    const T a = W[kCutTerms * n + e];
    const T d = fused(-sigma, a, W[(kCutTerms + 1) * n + e]);
    T nv[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        const T *X = x.p[q];
        const T xs = (X + COMP * P)[p];
        TA row = centre_terms(w0, TA(sigma), TA(a), TA(xs));
#pragma unroll
        for (int t = 1; t < kCutOwn; ++t) {
            const CutTerm ct = cut_term(COMP, t);
            row += TA(w[t]) * TA((X + (ct.comp * P + ct.di + ct.dj * dy + ct.dk * dz))[p]);
        }
        row += TA(cross[q]);
        nv[q] = xs + T(TA((f.p[q] + COMP * P)[p]) - row) / d;
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) put_face_at<T>(g, x.p[q] + COMP * P, COMP, p, nv[q]);
}

// A class update from its two parts: the first ncb workgroups (a multiple of
// 8) take the cut rows, the rest the vacuum runs; each part maps its
// workgroups to the XCDs as xcd_item does.  With several vectors and a short list
// (wave_split) a cut workgroup takes 64 rows, wave q the vector q: the cut
// rows are latency-bound, and one thread per row and vector keeps more of
// them in flight (the waves share the rows' coefficient lines in cache); a
// long list fills the GPU with one thread per row looping over the vectors,
// which reuses the coefficients in registers.
template <class T>
struct SmoothArgs {
    const int32_t *cut;
    const T *W;
    T *S;
    const VacRun *runs;
    int64_t n;
    uint32_t nruns, ncb;
    int colour, pair, wave_split;
};

template <class T, int COMP, int NR>
__global__ void __launch_bounds__(kThreads)
k_smooth_split(Grid g, T sigma, SmoothArgs<T> A, VPtr<const T> f, VPtr<T> x) {
    const uint32_t b = blockIdx.x;
    if (b < A.ncb) {
        const uint32_t L = (b % kXcd) * (A.ncb / kXcd) + b / kXcd;
        const CutTab<T, T> W{A.W, A.W};
        if (!A.wave_split) {
            const uint32_t e = L * kThreads + threadIdx.x;
            if (e < A.n) smooth_cut_n<T, COMP, NR, T>(g, sigma, A.cut, A.n, A.colour, W, A.pair, A.S, 0, f, x, e);
        } else {
            const int q = threadIdx.x >> 6;
            const uint32_t e = L * 64 + (threadIdx.x & 63);
            if (q < NR && e < A.n)
                smooth_cut_n<T, COMP, 1, T>(g, sigma, A.cut, A.n, A.colour, W, A.pair, A.S, q, vptr1(f.p[q]),
                                         vptr1(x.p[q]), e);
        }
    } else {
        const uint32_t bv = b - A.ncb, nvb = gridDim.x - A.ncb;
        const uint32_t L = (bv % kXcd) * (nvb / kXcd) + bv / kXcd;
        smooth_vac_n<T, COMP, NR>(g, sigma, f, x, L * kThreads + threadIdx.x, A.runs, A.nruns);
    }
}

// Whole smoothing sweeps of one vector on a level whose iterate fits the LDS
// of one CU (lds_level): workgroup q runs the sweeps of vector q, one barrier
// per class.  Such a level's class update is a thousand rows, and as a launch
// of its own it is all launch and latency (2.75 us, 24 per level and V-cycle).
// Here it is bound by what one CU can fetch and issue: 17 weights per cut row
// from L2 (1.5 us per class in FP32, 2.3 us in FP64 on the 16^3 sphere); the
// rows are dealt to the threads as one list per class, cut rows first, so
// that waves of either kind run side by side, and only the next index is
// fetched ahead (fetching the next class's weights ahead as well gained
// nothing: the CU's load path is busy either way).  V-cycle of the 16^3 sphere,
// one vector: FP32 81 -> 60 us, FP64 87 -> 81 us.
constexpr int kLdsThreads = 1024;

// the tabulated row of a thread's entry of a class
template <class T, class TA>
struct LdsRow {
    TA w0;
    T w[kCutTerms], a, d;   // w[0] unused
};

// A workgroup barrier that orders LDS accesses only: loads from global memory
// stay in flight across it (__syncthreads waits for them)
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// the update of one row of component COMP in LDS (smooth_cut_n, smooth_vac_n)
template <class T, int COMP, bool PMC, class TA>
__device__ __forceinline__ void lds_update(const Grid &g, T sigma, T ih2, T dvac, T *xs, const LdsRow<T, TA> &r, bool cut,
                                           uint32_t p, T fv) {
    const int P = (int)g.P, dy = g.sy, dz = (int)g.sz;
    T *xc = xs + COMP * P;
    const T xp = xc[p];
    T nv;
    if (cut) {
        TA cross = TA(0), row = centre_terms(r.w0, TA(sigma), TA(r.a), TA(xp));
#pragma unroll
        for (int u = kCutOwn; u < kCutTerms; ++u) {
            const CutTerm ct = cut_term(COMP, u);
            cross += TA(r.w[u]) * TA(xs[(int)p + (ct.comp * P + ct.di + ct.dj * dy + ct.dk * dz)]);
        }
#pragma unroll
        for (int u = 1; u < kCutOwn; ++u) {
            const CutTerm ct = cut_term(COMP, u);
            row += TA(r.w[u]) * TA(xs[(int)p + (ct.comp * P + ct.di + ct.dj * dy + ct.dk * dz)]);
        }
        row += TA(T(cross));
        nv = xp + T(TA(fv) - row) / fused(-sigma, r.a, r.d);
    } else {
        nv = xp + (fv - vac_row_m<T>(xc, p, dy, dz, ih2, sigma, xp)) / dvac;
    }
    if (PMC) put_face_at<T>(g, xc, COMP, p, nv);
    else xc[p] = nv;
}

template <class T, bool PMC, class TA>
__device__ __forceinline__ void sweeps_lds_body(const Grid &g, T sigma, const LdsRows &R, const CutTab<T, TA> &W,
                                                int sweeps, int reverse, int zero, const T *__restrict__ f,
                                                T *__restrict__ x, T *xs) {
    const int P = (int)g.P, n3 = 3 * P;
    const T ih2 = inv_h2_of<T>(g), dvac = fused(T(6), ih2, -sigma);
    const int tid = threadIdx.x;
    for (int e = tid; e < n3; e += kLdsThreads) xs[e] = zero ? T(0) : x[e];
    auto load_p = [&](int q, int t) __attribute__((always_inline)) -> uint32_t {
        const int c0 = R.cut_off[q], nc = R.cut_off[q + 1] - c0, v0 = R.vac_off[q];
        if (t >= nc + R.vac_off[q + 1] - v0) return 0u;
        return (uint32_t)(t < nc ? R.cut[c0 + t] : R.vac[v0 + t - nc]) & 0x7fffffffu;
    };
    auto load_row = [&](LdsRow<T, TA> &r, int q, int t) __attribute__((always_inline)) {
        const int base = R.cut_off[q & ~1], n = R.cut_off[(q & ~1) + 2] - base;
        const int64_t off = (int64_t)kCutW * base + (R.cut_off[q] - base);
        const T *w = W.w + off;
        r.w0 = (W.w0 + off)[t];
#pragma unroll
        for (int u = 1; u < kCutTerms; ++u) r.w[u] = (w + u * n)[t];
        r.a = (w + kCutTerms * n)[t];
        r.d = (w + (kCutTerms + 1) * n)[t];
    };
    // One class: its thread's first row is in r, p and fv when it begins; the
    // index of the next class's first row is fetched meanwhile.  One loop
    // serves every class, its number in a scalar (a copy per class kept so
    // many addresses live that it spilled).
    int q = reverse ? 5 : 0;
    const int dq = reverse ? -1 : 1;
    uint32_t pn = load_p(q, tid);
#pragma unroll 1
    for (int it = 0; it < 6 * sweeps; ++it) {
        const int nc = R.cut_off[q + 1] - R.cut_off[q], n = nc + R.vac_off[q + 1] - R.vac_off[q], comp = q >> 1;
        LdsRow<T, TA> r;
        uint32_t p = pn;
        T fv = f[comp * P + p];
        if (tid < nc) load_row(r, q, tid);
        const int qn = q + dq < 0 ? 5 : q + dq > 5 ? 0 : q + dq;
        pn = load_p(qn, tid);
        lds_barrier();   // the class before is done everywhere
        int t = tid;
#pragma unroll 1
        while (t < n) {
            if (comp == 0) lds_update<T, 0, PMC>(g, sigma, ih2, dvac, xs, r, t < nc, p, fv);
            else if (comp == 1) lds_update<T, 1, PMC>(g, sigma, ih2, dvac, xs, r, t < nc, p, fv);
            else lds_update<T, 2, PMC>(g, sigma, ih2, dvac, xs, r, t < nc, p, fv);
            t += kLdsThreads;
            if (t >= n) break;
            p = load_p(q, t);
            fv = f[comp * P + p];
            if (t < nc) load_row(r, q, t);
        }
        q = qn;
    }
    __syncthreads();
    for (int e = tid; e < n3; e += kLdsThreads) x[e] = xs[e];
}

extern __shared__ __align__(16) unsigned char lds_raw[];

template <class T, bool PMC>
__global__ void __launch_bounds__(kLdsThreads)
k_sweeps_lds(Grid g, T sigma, LdsRows R, const T *__restrict__ W, int sweeps, int reverse, int zero, VPtr<const T> f,
             VPtr<T> x) {
    sweeps_lds_body<T, PMC, T>(g, sigma, R, CutTab<T, T>{W, W}, sweeps, reverse, zero, f.p[blockIdx.x], x.p[blockIdx.x],
                          reinterpret_cast<T *>(lds_raw));
}

// ---------------------------------------------------------------------------
// Staggered transfers.  P: linear along the normal, constant across; R = P^T/8.
// ---------------------------------------------------------------------------
template <class T>
// xz (optional): the coarse iterate, set to zero on the cell's faces (and
// their PMC ghost images) in the same pass, as the coarse V-cycle starts
// from zero
__device__ __forceinline__ void restrict_body(const Grid &gf, const Grid &gc, const Coefs<T> &cc,
                                              const T *__restrict__ r, T *__restrict__ fc, int64_t item,
                                              T *__restrict__ xz = nullptr) {
    int I, J, K;
    if (!cell_of(gc, item, I, J, K)) return;
    const int64_t Pf = gf.P, Pc = gc.P, fy = gf.sy, fz = gf.sz;
    const int64_t pc = pidx(gc, I, J, K);
    const T *RX = r, *RY = r + Pf, *RZ = r + 2 * Pf;
    const int64_t q = pidx(gf, 2 * I, 2 * J, 2 * K);
    // transpose of the area-weighted normal interpolation: the fine face
    // between coarse faces c and c' gives c the share a_c / (a_c + a_c')
    const T ax = cc.ax[pc], ay = cc.ay[pc], az = cc.az[pc];
    const T xm = ax > T(0) ? ax / (ax + cc.ax[pc - 1]) : T(0);
    const T xp = ax > T(0) ? ax / (ax + cc.ax[pc + 1]) : T(0);
    const T ym = ay > T(0) ? ay / (ay + cc.ay[pc - gc.sy]) : T(0);
    const T yp = ay > T(0) ? ay / (ay + cc.ay[pc + gc.sy]) : T(0);
    const T zm = az > T(0) ? az / (az + cc.az[pc - gc.sz]) : T(0);
    const T zp = az > T(0) ? az / (az + cc.az[pc + gc.sz]) : T(0);
    T sx = 0, sy = 0, sz = 0;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            // x: tangential offsets in y (a) and z (b)
            const int64_t qx = q + a * fy + b * fz;
            sx += RX[qx] + xm * RX[qx - 1] + xp * RX[qx + 1];
            const int64_t qy = q + a + b * fz;
            sy += RY[qy] + ym * RY[qy - fy] + yp * RY[qy + fy];
            const int64_t qz = q + a + b * fy;
            sz += RZ[qz] + zm * RZ[qz - fz] + zp * RZ[qz + fz];
        }
    const T e = T(0.125);
    put_face<T>(gc, fc, 0, I, J, K, pc, ax != T(0) ? e * sx : T(0));
    put_face<T>(gc, fc + Pc, 1, I, J, K, pc, ay != T(0) ? e * sy : T(0));
    put_face<T>(gc, fc + 2 * Pc, 2, I, J, K, pc, az != T(0) ? e * sz : T(0));
    if (xz) {
        put_face<T>(gc, xz, 0, I, J, K, pc, T(0));
        put_face<T>(gc, xz + Pc, 1, I, J, K, pc, T(0));
        put_face<T>(gc, xz + 2 * Pc, 2, I, J, K, pc, T(0));
    }
}

template <class T>
__global__ void __launch_bounds__(kThreads)
k_restrict(Grid gf, Grid gc, Coefs<T> cc, const T *__restrict__ r, T *__restrict__ fc) {
    restrict_body<T>(gf, gc, cc, r, fc, xcd_item());
}

template <class T, int NR>
__global__ void __launch_bounds__(kThreads)
k_restrict_b(Grid gf, Grid gc, Coefs<T> cc, const int32_t *__restrict__ rows, int64_t nrows, VPtr<const T> r,
             VPtr<T> fc, VPtr<T> xz) {
    int q;
    const int64_t t = wave_item(q);
    restrict_body<T>(gf, gc, cc, r.p[q], fc.p[q], listed_item(gc, rows, nrows, t), xz.p[q]);
}

// fine value between coarse faces c0, c1: (a0 x0 + a1 x1) / (a0 + a1)
template <class T>
__device__ __forceinline__ T wmean(T a0, T x0, T a1, T x1) {
    const T t = a0 + a1;
    return t > T(0) ? (a0 * x0 + a1 * x1) / t : T(0);
}

template <class T>
__device__ __forceinline__ void prolong_body(const Grid &gf, const Grid &gc, const Coefs<T> &cf, const Coefs<T> &cc,
                                             const T *__restrict__ xc, T *__restrict__ x, int64_t item) {
    int i, j, k;
    if (!cell_of(gf, item, i, j, k)) return;
    const int64_t Pf = gf.P, Pc = gc.P, cy = gc.sy, cz = gc.sz;
    const int64_t p = pidx(gf, i, j, k);
    const int64_t q = pidx(gc, i >> 1, j >> 1, k >> 1);
    const T *CX = xc, *CY = xc + Pc, *CZ = xc + 2 * Pc;
    if (cf.ax[p] != T(0))
        put_face<T>(gf, x, 0, i, j, k, p,
                    x[p] + ((i & 1) ? wmean(cc.ax[q], CX[q], cc.ax[q + 1], CX[q + 1]) : CX[q]));
    if (cf.ay[p] != T(0))
        put_face<T>(gf, x + Pf, 1, i, j, k, p,
                    x[Pf + p] + ((j & 1) ? wmean(cc.ay[q], CY[q], cc.ay[q + cy], CY[q + cy]) : CY[q]));
    if (cf.az[p] != T(0))
        put_face<T>(gf, x + 2 * Pf, 2, i, j, k, p,
                    x[2 * Pf + p] + ((k & 1) ? wmean(cc.az[q], CZ[q], cc.az[q + cz], CZ[q + cz]) : CZ[q]));
}

template <class T>
__global__ void __launch_bounds__(kThreads)
k_prolong_add(Grid gf, Grid gc, Coefs<T> cf, Coefs<T> cc, const T *__restrict__ xc,
              T *__restrict__ x) {
    prolong_body<T>(gf, gc, cf, cc, xc, x, xcd_item());
}

template <class T, int NR>
__global__ void __launch_bounds__(kThreads)
k_prolong_add_b(Grid gf, Grid gc, Coefs<T> cf, Coefs<T> cc, const int32_t *__restrict__ rows, int64_t nrows,
                VPtr<const T> xc, VPtr<T> x) {
    int q;
    const int64_t t = wave_item(q);
    prolong_body<T>(gf, gc, cf, cc, xc.p[q], x.p[q], listed_item(gf, rows, nrows, t));
}

// x = 0 (a kernel, not a memset: it may be recorded into a HIP graph)
template <class T>
__global__ void __launch_bounds__(kThreads) k_zero(int64_t n, T *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kThreads)
        x[e] = T(0);
}

template <class TI, class TO>
__global__ void k_cast(const TI *__restrict__ in, TO *__restrict__ out, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kThreads)
        out[e] = (TO)in[e];
}

// the cast over the listed units of a face vector (see Span)
template <class TI, class TO>
__global__ void k_cast_units(const TI *__restrict__ in, TO *__restrict__ out, int64_t n,
                             const int32_t *__restrict__ units, int64_t nunits) {
    const int64_t cnt = nunits * kSpanUnit;
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt;
         it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = (int64_t)units[it / kSpanUnit] * kSpanUnit + it % kSpanUnit;
        if (e < n) out[e] = (TO)in[e];
    }
}

// the casts of several vectors in one launch: grid row y takes vector y
template <class TI, class TO>
__global__ void __launch_bounds__(kThreads)
k_cast_b(VPtr<const TI> in, VPtr<TO> out, int64_t n, const int32_t *__restrict__ units, int64_t nunits) {
    const TI *__restrict__ a = in.p[blockIdx.y];
    TO *__restrict__ b = out.p[blockIdx.y];
    const int64_t cnt = units ? nunits * kSpanUnit : n;
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt; it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = units ? (int64_t)units[it / kSpanUnit] * kSpanUnit + it % kSpanUnit : it;
        if (e < n) b[e] = (TO)a[e];
    }
}

// copies of several vectors in one launch: grid row y takes vector y
__global__ void __launch_bounds__(kThreads) k_copy_many(CopyArgs A) {
    const float *__restrict__ a = A.in[blockIdx.y];
    float *__restrict__ b = A.out[blockIdx.y];
    const int64_t n = A.n[blockIdx.y];
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kThreads) b[e] = a[e];
}

// Coarsest level: x[idx[r]] = sum_c inv[r, c] f[idx[c]] (FP64 arithmetic);
// one row of the inverse serves every right-hand side
template <class T, int NR>
__device__ __forceinline__ void coarse_body_n(int n, const double *__restrict__ inv, const int64_t *__restrict__ idx,
                                              const VPtr<const T> &f, const VPtr<T> &x, int row) {
    double s[NR];
#pragma unroll
    for (int v = 0; v < NR; ++v) s[v] = 0.0;
    for (int col = threadIdx.x; col < n; col += kThreads) {
        const double w = inv[(int64_t)row * n + col];
        const int64_t e = idx[col];
#pragma unroll
        for (int v = 0; v < NR; ++v) s[v] += w * (double)f.p[v][e];
    }
    __shared__ double sh[NR][kThreads / 64];
#pragma unroll
    for (int v = 0; v < NR; ++v) {
        for (int off = 32; off > 0; off >>= 1) s[v] += __shfl_down(s[v], off, 64);
        if ((threadIdx.x & 63) == 0) sh[v][threadIdx.x >> 6] = s[v];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int v = 0; v < NR; ++v) {
            double t = 0.0;
            for (int w = 0; w < kThreads / 64; ++w) t += sh[v][w];
            x.p[v][idx[row]] = (T)t;
        }
    }
}

template <class T>
__device__ __forceinline__ void coarse_body(int n, const double *__restrict__ inv, const int64_t *__restrict__ idx,
                                            const T *__restrict__ f, T *__restrict__ x, int row) {
    coarse_body_n<T, 1>(n, inv, idx, vptr1(f), vptr1(x), row);
}

template <class T>
__global__ void __launch_bounds__(kThreads)
k_coarse_solve(int n, const double *__restrict__ inv, const int64_t *__restrict__ idx,
               const T *__restrict__ f, T *__restrict__ x) {
    coarse_body<T>(n, inv, idx, f, x, blockIdx.x);
}

template <class T, int NR>
__global__ void __launch_bounds__(kThreads)
k_coarse_solve_b(int n, const double *__restrict__ inv, const int64_t *__restrict__ idx, VPtr<const T> f,
                 VPtr<T> x) {
    coarse_body_n<T, NR>(n, inv, idx, f, x, blockIdx.x);
}

// PMC ghost layer of one plane (axis a) from the values next to it; planes
// are filled in the order x, y, z so corner ghosts get both mirrors.
template <class T>
__global__ void k_mirror_faces(Grid g, int a, T *__restrict__ x) {
    const int n[3] = {g.nx, g.ny, g.nz};
    const int b = a == 0 ? 1 : 0, d = a == 2 ? 1 : 2;
    const int nb = n[b] + 2, nd = n[d] + 2;
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= (int64_t)nb * nd) return;
    int idx[3];
    idx[b] = (int)(t % nb) - 1;
    idx[d] = (int)(t / nb) - 1;
    idx[a] = -1;
    const int64_t stride[3] = {1, g.sy, g.sz};
    const int64_t pg = pidx(g, idx[0], idx[1], idx[2]);
    for (int comp = 0; comp < 3; ++comp) {
        T *arr = x + comp * g.P;
        arr[pg] = comp == a ? arr[pg + 2 * stride[a]] : -arr[pg + stride[a]];
    }
}

template <class T>
__global__ void k_mirror_cells(Grid g, int a, T *__restrict__ x) {
    const int n[3] = {g.nx, g.ny, g.nz};
    const int b = a == 0 ? 1 : 0, d = a == 2 ? 1 : 2;
    const int nb = n[b] + 2, nd = n[d] + 2;
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= (int64_t)nb * nd) return;
    int idx[3];
    idx[b] = (int)(t % nb) - 1;
    idx[d] = (int)(t / nb) - 1;
    idx[a] = -1;
    const int64_t stride[3] = {1, g.sy, g.sz};
    const int64_t pg = pidx(g, idx[0], idx[1], idx[2]);
    x[pg] = -x[pg + stride[a]];
}

// ---------------------------------------------------------------------------
// Scalar problem: g = D A b, b -= D^T psi, S = D A D^T (weight w per level)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void div_DA_body(const Grid &g, const Coefs<double> &c, const double *__restrict__ b,
                                            double *__restrict__ out, int64_t item) {
    int i, j, k;
    if (!cell_of(g, item, i, j, k)) return;
    const int64_t P = g.P, dy = g.sy, dz = g.sz, p = pidx(g, i, j, k);
    const double *X = b, *Y = b + P, *Z = b + 2 * P;
    const double s = c.ax[p + 1] * X[p + 1] - c.ax[p] * X[p] + c.ay[p + dy] * Y[p + dy] -
                     c.ay[p] * Y[p] + c.az[p + dz] * Z[p + dz] - c.az[p] * Z[p];
    put_cell<double>(g, out, i, j, k, p, c.vinv[p] != 0.0 ? s / g.h : 0.0);
}

__device__ __forceinline__ void grad_sub_body(const Grid &g, const Coefs<double> &c, const double *__restrict__ psi,
                                              const double *bin, double *bout, double scale, int64_t item) {
    int i, j, k;
    if (!cell_of(g, item, i, j, k)) return;
    const int64_t P = g.P, dy = g.sy, dz = g.sz, p = pidx(g, i, j, k);
    const double s = scale / g.h;
    const double pp = psi[p];
    const double vx = c.ax[p] != 0.0 ? bin[p] - s * (psi[p - 1] - pp) : 0.0;
    const double vy = c.ay[p] != 0.0 ? bin[P + p] - s * (psi[p - dy] - pp) : 0.0;
    const double vz = c.az[p] != 0.0 ? bin[2 * P + p] - s * (psi[p - dz] - pp) : 0.0;
    put_face<double>(g, bout, 0, i, j, k, p, vx);
    put_face<double>(g, bout + P, 1, i, j, k, p, vy);
    put_face<double>(g, bout + 2 * P, 2, i, j, k, p, vz);
}

template <class T>
__device__ inline T s_row(const Coefs<T> &c, const T *x, int64_t p, int64_t dy, int64_t dz) {
    const T xp = x[p];
    return c.ax[p] * (xp - x[p - 1]) + c.ax[p + 1] * (xp - x[p + 1]) +
           c.ay[p] * (xp - x[p - dy]) + c.ay[p + dy] * (xp - x[p + dy]) +
           c.az[p] * (xp - x[p - dz]) + c.az[p + dz] * (xp - x[p + dz]);
}

template <class T>
__device__ __forceinline__ void s_apply_body(const Grid &g, const Coefs<T> &c, T w, int resid,
                                             const T *__restrict__ f, const T *__restrict__ x, T *__restrict__ y,
                                             int64_t item) {
    int i, j, k;
    if (!cell_of(g, item, i, j, k)) return;
    const int64_t p = pidx(g, i, j, k);
    T v = w * s_row<T>(c, x, p, g.sy, g.sz);
    if (resid) v = f[p] - v;
    put_cell<T>(g, y, i, j, k, p, c.vinv[p] != T(0) ? v : T(0));
}

// rows: optional list of the grid rows (k * ny + j) holding an active cell;
// the colour sweep then visits only those
template <class T>
__device__ __forceinline__ void s_smooth_body(const Grid &g, const Coefs<T> &c, T w, int colour,
                                              const T *__restrict__ f, T *__restrict__ x, int64_t t,
                                              const int32_t *__restrict__ rows = nullptr, int64_t nrows = 0) {
    const int nxh = (g.nx + 1) >> 1;
    if (t >= (rows ? nrows : (int64_t)g.ny * g.nz) * nxh) return;
    const uint32_t u = (uint32_t)t, ur = u / (uint32_t)nxh, r = rows ? (uint32_t)rows[ur] : ur;
    const int ih = (int)(u - ur * nxh);
    const uint32_t kk = r / (uint32_t)g.ny;
    const int j = (int)(r - kk * g.ny), k = (int)kk;
    const int i = 2 * ih + ((j + k + colour) & 1);
    if (i >= g.nx) return;
    const int64_t dy = g.sy, dz = g.sz, p = pidx(g, i, j, k);
    if (c.vinv[p] == T(0)) return;
    T d = c.ax[p] + c.ax[p + 1] + c.ay[p] + c.ay[p + dy] + c.az[p] + c.az[p + dz];
    // odd mirror across a PMC plane: the face in the plane counts twice
    if ((g.pmc & 1) && i == 0) d += c.ax[p];
    if ((g.pmc & 2) && j == 0) d += c.ay[p];
    if ((g.pmc & 4) && k == 0) d += c.az[p];
    d *= w;
    if (d == T(0)) return;
    put_cell<T>(g, x, i, j, k, p, x[p] + (f[p] - w * s_row<T>(c, x, p, dy, dz)) / d);
}

template <class T>
__device__ __forceinline__ void s_restrict_body(const Grid &gf, const Grid &gc, const Coefs<T> &cc,
                                                const T *__restrict__ r, T *__restrict__ fc, int64_t item,
                                                T *__restrict__ xz = nullptr) {
    int I, J, K;
    if (!cell_of(gc, item, I, J, K)) return;
    const int64_t pc = pidx(gc, I, J, K), q = pidx(gf, 2 * I, 2 * J, 2 * K);
    const int64_t fy = gf.sy, fz = gf.sz;
    T s = T(0);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) s += r[q + a * fy + b * fz] + r[q + 1 + a * fy + b * fz];
    put_cell<T>(gc, fc, I, J, K, pc, cc.vinv[pc] != T(0) ? T(0.125) * s : T(0));
    if (xz) put_cell<T>(gc, xz, I, J, K, pc, T(0));   // the coarse iterate starts at zero
}

template <class T>
__device__ __forceinline__ void s_prolong_body(const Grid &gf, const Grid &gc, const Coefs<T> &cf,
                                               const T *__restrict__ xc, T *__restrict__ x, int64_t item) {
    int i, j, k;
    if (!cell_of(gf, item, i, j, k)) return;
    const int64_t p = pidx(gf, i, j, k);
    if (cf.vinv[p] != T(0)) put_cell<T>(gf, x, i, j, k, p, x[p] + xc[pidx(gc, i >> 1, j >> 1, k >> 1)]);
}

__global__ void __launch_bounds__(kThreads)
k_div_DA(Grid g, Coefs<double> c, const double *__restrict__ b, double *__restrict__ out) {
    div_DA_body(g, c, b, out, xcd_item());
}

__global__ void __launch_bounds__(kThreads)
k_grad_sub(Grid g, Coefs<double> c, const double *__restrict__ psi, const double *bin, double *bout, double scale) {
    grad_sub_body(g, c, psi, bin, bout, scale, xcd_item());
}

__global__ void __launch_bounds__(kThreads)
k_s_apply(Grid g, Coefs<double> c, double w, int resid, const double *__restrict__ f,
          const double *__restrict__ x, double *__restrict__ y) {
    s_apply_body<double>(g, c, w, resid, f, x, y, xcd_item());
}

__global__ void __launch_bounds__(kThreads)
k_s_smooth(Grid g, Coefs<double> c, double w, int colour, const double *__restrict__ f,
           double *__restrict__ x) {
    s_smooth_body<double>(g, c, w, colour, f, x, xcd_item());
}

__global__ void __launch_bounds__(kThreads)
k_s_restrict(Grid gf, Grid gc, Coefs<double> cc, const double *__restrict__ r,
             double *__restrict__ fc) {
    s_restrict_body<double>(gf, gc, cc, r, fc, xcd_item());
}

__global__ void __launch_bounds__(kThreads)
k_s_prolong_add(Grid gf, Grid gc, Coefs<double> cf, const double *__restrict__ xc,
                double *__restrict__ x) {
    s_prolong_body<double>(gf, gc, cf, xc, x, xcd_item());
}

// block forms of the scalar kernels: NR lanes per cell, one vector each
template <int NR>
__global__ void __launch_bounds__(kThreads)
k_div_DA_b(Grid g, Coefs<double> c, VPtr<const double> b, VPtr<double> out) {
    int q;
    const int64_t t = wave_item(q);
    div_DA_body(g, c, b.p[q], out.p[q], t);
}

template <int NR>
__global__ void __launch_bounds__(kThreads)
k_grad_sub_b(Grid g, Coefs<double> c, VPtr<const double> psi, VPtr<const double> bin, VPtr<double> bout,
             double scale) {
    int q;
    const int64_t t = wave_item(q);
    grad_sub_body(g, c, psi.p[q], bin.p[q], bout.p[q], scale, t);
}

template <class T, int NR>
__global__ void __launch_bounds__(kThreads)
k_s_apply_b(Grid g, Coefs<T> c, T w, int resid, const int32_t *__restrict__ rows, int64_t nrows, VPtr<const T> f,
            VPtr<const T> x, VPtr<T> y) {
    int q;
    const int64_t t = wave_item(q);
    s_apply_body<T>(g, c, w, resid, f.p[q], x.p[q], y.p[q], listed_item(g, rows, nrows, t));
}

template <class T, int NR>
__global__ void __launch_bounds__(kThreads)
k_s_smooth_b(Grid g, Coefs<T> c, T w, int colour, const int32_t *__restrict__ rows, int64_t nrows, VPtr<const T> f,
             VPtr<T> x) {
    int q;
    const int64_t t = wave_item(q);
    s_smooth_body<T>(g, c, w, colour, f.p[q], x.p[q], t, rows, nrows);
}

template <class T, int NR>
__global__ void __launch_bounds__(kThreads)
k_s_restrict_b(Grid gf, Grid gc, Coefs<T> cc, const int32_t *__restrict__ rows, int64_t nrows, VPtr<const T> r,
               VPtr<T> fc, VPtr<T> xz) {
    int q;
    const int64_t t = wave_item(q);
    s_restrict_body<T>(gf, gc, cc, r.p[q], fc.p[q], listed_item(gc, rows, nrows, t), xz.p[q]);
}

template <class T, int NR>
__global__ void __launch_bounds__(kThreads)
k_s_prolong_add_b(Grid gf, Grid gc, Coefs<T> cf, const int32_t *__restrict__ rows, int64_t nrows,
                  VPtr<const T> xc, VPtr<T> x) {
    int q;
    const int64_t t = wave_item(q);
    s_prolong_body<T>(gf, gc, cf, xc.p[q], x.p[q], listed_item(gf, rows, nrows, t));
}

// ---------------------------------------------------------------------------
// FP64 vector helpers
// ---------------------------------------------------------------------------
__global__ void k_axpby(int64_t n, double a, const double *__restrict__ x, double b,
                        double *__restrict__ y) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kThreads)
        y[e] = a * x[e] + b * y[e];
}

__global__ void k_axpy(int64_t n, double a, const double *__restrict__ x, double *__restrict__ y) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kThreads)
        y[e] += a * x[e];
}

__global__ void k_scale(int64_t n, double a, double *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kThreads)
        x[e] *= a;
}

constexpr int kChunk = 8;  // vectors reduced per pass of k_mdot

// Reductions and multi-axpys stream long FP64 vectors: they read pairs of
// doubles (16-byte loads) when every pointer is 16-byte aligned and the
// length / stride are even (VEC = 2), else single doubles (VEC = 1).
template <int VEC>
struct Vec;
template <>
struct Vec<1> {
    using T = double;
    __device__ static T ld(const double *p, int64_t e) { return p[e]; }
    __device__ static void st(double *p, int64_t e, T v) { p[e] = v; }
    __device__ static double dot(T a, T b) { return a * b; }
    __device__ static T fma(double c, T a, T b) { return b + c * a; }
    __device__ static T mul(T a, T b) { return a * b; }
    __device__ static T scale(double c, T a) { return c * a; }
    __device__ static T zero() { return 0.0; }
};
template <>
struct Vec<2> {
    using T = double2;
    __device__ static T ld(const double *p, int64_t e) { return reinterpret_cast<const double2 *>(p)[e]; }
    __device__ static void st(double *p, int64_t e, T v) { reinterpret_cast<double2 *>(p)[e] = v; }
    __device__ static double dot(T a, T b) { return a.x * b.x + a.y * b.y; }
    __device__ static T fma(double c, T a, T b) { return make_double2(b.x + c * a.x, b.y + c * a.y); }
    __device__ static T mul(T a, T b) { return make_double2(a.x * b.x, a.y * b.y); }
    __device__ static T scale(double c, T a) { return make_double2(c * a.x, c * a.y); }
    __device__ static T zero() { return make_double2(0.0, 0.0); }
};

// Four doubles (two 16-byte loads): the width at which an FP32 basis column
// is read with 16-byte loads as well (VEC = 4 needs lengths and strides that
// are multiples of 4 and 16-byte aligned pointers)
struct D4 {
    double2 a, b;
};
template <>
struct Vec<4> {
    using T = D4;
    __device__ static T ld(const double *p, int64_t e) {
        const double2 *q = reinterpret_cast<const double2 *>(p) + 2 * e;
        return {q[0], q[1]};
    }
    __device__ static void st(double *p, int64_t e, T v) {
        double2 *q = reinterpret_cast<double2 *>(p) + 2 * e;
        q[0] = v.a;
        q[1] = v.b;
    }
    __device__ static double dot(T a, T b) { return Vec<2>::dot(a.a, b.a) + Vec<2>::dot(a.b, b.b); }
    __device__ static T fma(double c, T a, T b) { return {Vec<2>::fma(c, a.a, b.a), Vec<2>::fma(c, a.b, b.b)}; }
    __device__ static T mul(T a, T b) { return {Vec<2>::mul(a.a, b.a), Vec<2>::mul(a.b, b.b)}; }
    __device__ static T scale(double c, T a) { return {Vec<2>::scale(c, a.a), Vec<2>::scale(c, a.b)}; }
    __device__ static T zero() { return {Vec<2>::zero(), Vec<2>::zero()}; }
};

// VEC consecutive entries of a Krylov basis column in FP64: FP64 columns
// as they are, FP32 columns widened (the basis kept in FP32; every sum and
// update is still FP64)
template <int VEC, class TV>
struct BasisLd;
template <int VEC>
struct BasisLd<VEC, double> {
    __device__ static typename Vec<VEC>::T ld(const double *p, int64_t e) { return Vec<VEC>::ld(p, e); }
};
template <>
struct BasisLd<1, float> {
    __device__ static double ld(const float *p, int64_t e) { return (double)p[e]; }
};
template <>
struct BasisLd<2, float> {
    __device__ static double2 ld(const float *p, int64_t e) {
        const float2 v = reinterpret_cast<const float2 *>(p)[e];
        return make_double2((double)v.x, (double)v.y);
    }
};
template <>
struct BasisLd<4, float> {
    __device__ static D4 ld(const float *p, int64_t e) {
        const float4 v = reinterpret_cast<const float4 *>(p)[e];
        return {make_double2((double)v.x, (double)v.y), make_double2((double)v.z, (double)v.w)};
    }
};

// Index i of a grid-stride loop -> element (in VEC units) of the listed
// units; the whole vector without a list.  Elements past nvec (a partial
// last unit) are skipped by the caller.
template <int VEC>
__device__ __forceinline__ int64_t span_count(const Span &sp, int64_t nvec) {
    return sp.u ? sp.n * (kSpanUnit / VEC) : nvec;
}
template <int VEC>
__device__ __forceinline__ int64_t span_elem(const Span &sp, int64_t i) {
    constexpr int per = kSpanUnit / VEC;
    return sp.u ? (int64_t)sp.u[i / per] * per + (i % per) : i;
}

// part[i][block] = partial sums of V_i . (w * wt) over the block's elements;
// grid row y takes system y of A (`rows` partial rows each)
template <int VEC, class TV = double>
__global__ void __launch_bounds__(kThreads)
k_mdot(BasisArgs<TV> A, int64_t ld, const double *__restrict__ wt, int64_t n, double *__restrict__ part0, int rows,
       Span sp) {
    using O = Vec<VEC>;
    const int nv = A.s[blockIdx.y].nv;
    const TV *__restrict__ V = A.s[blockIdx.y].V;
    const double *__restrict__ w = A.s[blockIdx.y].w;
    double *__restrict__ part = part0 + (int64_t)blockIdx.y * rows * gridDim.x;
    const int64_t nvec = n / VEC, ldv = ld / VEC, cnt = span_count<VEC>(sp, nvec);
    for (int c0 = 0; c0 < nv; c0 += kChunk) {
        const int cn = min(kChunk, nv - c0);
        double acc[kChunk];
#pragma unroll
        for (int q = 0; q < kChunk; ++q) acc[q] = 0.0;
        for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt;
             it += (int64_t)gridDim.x * kThreads) {
            const int64_t e = span_elem<VEC>(sp, it);
            if (e >= nvec) continue;
            typename O::T wv = O::ld(w, e);
            if (wt) wv = O::mul(wv, O::ld(wt, e));
#pragma unroll
            for (int q = 0; q < kChunk; ++q)
                if (q < cn) acc[q] += O::dot(BasisLd<VEC, TV>::ld(V + (int64_t)(c0 + q) * ldv * VEC, e), wv);
        }
        if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
            const double wv = w[n - 1] * (wt ? wt[n - 1] : 1.0);
#pragma unroll
            for (int q = 0; q < kChunk; ++q)
                if (q < cn) acc[q] += V[(int64_t)(c0 + q) * ld + n - 1] * wv;
        }
        __shared__ double sh[kThreads / 64][kChunk];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int q = 0; q < kChunk; ++q) {
            double v = acc[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
            if (lane == 0) sh[wave][q] = v;
        }
        __syncthreads();
        if (threadIdx.x < cn) {
            double t = 0.0;
            for (int u = 0; u < kThreads / 64; ++u) t += sh[u][threadIdx.x];
            part[(int64_t)(c0 + threadIdx.x) * gridDim.x + blockIdx.x] = t;
        }
        __syncthreads();
    }
}

// part rows 0..nv-1: V_i . w; row nv: |w|^2  (chunks of kChunk vectors)
template <int VEC, class TV = double>
__global__ void __launch_bounds__(kThreads)
k_mdot_norm(int nv, const TV *__restrict__ V, int64_t ld, const double *__restrict__ w,
            int64_t n, double *__restrict__ part, Span sp) {
    using O = Vec<VEC>;
    const int64_t nvec = n / VEC, ldv = ld / VEC, cnt = span_count<VEC>(sp, nvec);
    __shared__ double sh[kThreads / 64][kChunk + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c0 = 0; c0 < nv; c0 += kChunk) {
        const int cn = min(kChunk, nv - c0);
        const bool last = c0 + kChunk >= nv;
        double acc[kChunk + 1];
#pragma unroll
        for (int q = 0; q <= kChunk; ++q) acc[q] = 0.0;
        for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt;
             it += (int64_t)gridDim.x * kThreads) {
            const int64_t e = span_elem<VEC>(sp, it);
            if (e >= nvec) continue;
            const typename O::T wv = O::ld(w, e);
#pragma unroll
            for (int q = 0; q < kChunk; ++q)
                if (q < cn) acc[q] += O::dot(BasisLd<VEC, TV>::ld(V + (int64_t)(c0 + q) * ldv * VEC, e), wv);
            if (last) acc[kChunk] += O::dot(wv, wv);
        }
        if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
            const double wv = w[n - 1];
#pragma unroll
            for (int q = 0; q < kChunk; ++q)
                if (q < cn) acc[q] += V[(int64_t)(c0 + q) * ld + n - 1] * wv;
            if (last) acc[kChunk] += wv * wv;
        }
#pragma unroll
        for (int q = 0; q <= kChunk; ++q) {
            double v = acc[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
            if (lane == 0) sh[wave][q] = v;
        }
        __syncthreads();
        if (threadIdx.x < cn || (last && threadIdx.x == cn)) {
            const int q = threadIdx.x < cn ? threadIdx.x : kChunk;
            double t = 0.0;
            for (int u = 0; u < kThreads / 64; ++u) t += sh[u][q];
            part[(int64_t)(c0 + threadIdx.x) * gridDim.x + blockIdx.x] = t;
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kThreads)
k_mdot_final(int nblk, const double *__restrict__ part, double *__restrict__ out) {
    const int v = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kThreads) s += part[(int64_t)v * nblk + b];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    __shared__ double sh[kThreads / 64];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int u = 0; u < kThreads / 64; ++u) t += sh[u];
        out[v] = t;
    }
}

// the final sums of k_mdot (extra = 0) and k_maxpy_mdot_norm (extra = 1):
// block (v, y) sums partial row v of system y
template <class TV>
__global__ void __launch_bounds__(kThreads)
k_basis_final(BasisArgs<TV> A, int nblk, const double *__restrict__ part, int rows, int extra) {
    const int v = blockIdx.x;
    if (v >= A.s[blockIdx.y].nv + extra) return;
    const double *row = part + ((int64_t)blockIdx.y * rows + v) * nblk;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kThreads) s += row[b];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    __shared__ double sh[kThreads / 64];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int u = 0; u < kThreads / 64; ++u) t += sh[u];
        A.s[blockIdx.y].dout[v] = t;
    }
}

// Dot products of up to kMaxRhs pairs in one pass:
//   part[q][block] = partial sum of X_q . (Y_q * wt) for the pairs with X_q set
// (wt, when given, is read once for all pairs), over the listed units of sp
template <int VEC>
__global__ void __launch_bounds__(kThreads)
k_dot_pairs(VPtr<const double> X, VPtr<const double> Y, const double *__restrict__ wt, int64_t n,
            double *__restrict__ part, Span sp) {
    using O = Vec<VEC>;
    const int64_t nvec = n / VEC, cnt = span_count<VEC>(sp, nvec);
    double acc[kMaxRhs];
#pragma unroll
    for (int q = 0; q < kMaxRhs; ++q) acc[q] = 0.0;
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt; it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = span_elem<VEC>(sp, it);
        if (e >= nvec) continue;
        const typename O::T w = wt ? O::ld(wt, e) : typename O::T{};
#pragma unroll
        for (int q = 0; q < kMaxRhs; ++q)
            if (X.p[q]) {
                const typename O::T x = O::ld(X.p[q], e);
                acc[q] += O::dot(wt ? O::mul(x, w) : x, O::ld(Y.p[q], e));
            }
    }
    if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        const double w = wt ? wt[n - 1] : 1.0;
#pragma unroll
        for (int q = 0; q < kMaxRhs; ++q)
            if (X.p[q]) acc[q] += X.p[q][n - 1] * w * Y.p[q][n - 1];
    }
    __shared__ double sh[kThreads / 64][kMaxRhs];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < kMaxRhs; ++q) {
        double v = acc[q];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) sh[wave][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < kMaxRhs) {
        double t = 0.0;
        for (int u = 0; u < kThreads / 64; ++u) t += sh[u][threadIdx.x];
        part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// out[v * stride] = sum of part row v (rows of nblk partial sums)
__global__ void __launch_bounds__(kThreads)
k_mdot_final_strided(int nblk, const double *__restrict__ part, double *__restrict__ out, int64_t stride) {
    const int v = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kThreads) s += part[(int64_t)v * nblk + b];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    __shared__ double sh[kThreads / 64];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int u = 0; u < kThreads / 64; ++u) t += sh[u];
        out[(int64_t)v * stride] = t;
    }
}

// block q: the sum of partial row q, turned into solve q's scalars (CgStep)
__global__ void __launch_bounds__(kThreads)
k_cg_final(CgStep step, int nblk, const double *__restrict__ part, CgState *st) {
    const int q = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kThreads) s += part[(int64_t)q * nblk + b];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    __shared__ double sh[kThreads / 64];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x != 0 || !st->act[q]) return;
    double t = 0.0;
    for (int u = 0; u < kThreads / 64; ++u) t += sh[u];
    if (step == kCgAlpha) {
        if (t > 0.0) {
            st->alpha[q] = st->rz[q] / t;
            ++st->its[q];
        } else {
            st->act[q] = 0;
        }
    } else if (step == kCgCheck) {
        if (sqrt(t) <= st->stop[q]) st->act[q] = 0;
    } else {
        st->beta[q] = st->its[q] == 0 ? 0.0 : t / st->rz[q];
        st->rz[q] = t;
    }
}

// One conjugate-gradient update of the active solves:
//   psi_q += a_q p_q,  r_q -= a_q q_q,  part[q][block] = partial of r_q . (r_q * wt)
// over the listed units of sp
__global__ void __launch_bounds__(kThreads)
k_cg_update(int nr, VPtr<const double> Pv, VPtr<const double> Qv, VPtr<double> Psi, VPtr<double> R,
            const double *__restrict__ wt, int64_t n, double *__restrict__ part, const CgState *__restrict__ st,
            Span sp) {
    double acc[kMaxRhs], a[kMaxRhs];
    bool on[kMaxRhs];
#pragma unroll
    for (int q = 0; q < kMaxRhs; ++q) {
        acc[q] = 0.0;
        on[q] = q < nr && st->act[q];
        a[q] = on[q] ? st->alpha[q] : 0.0;
    }
    const int64_t cnt = span_count<1>(sp, n);
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt; it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = span_elem<1>(sp, it);
        if (e >= n) continue;
        const double w = wt[e];
#pragma unroll
        for (int q = 0; q < kMaxRhs; ++q)
            if (on[q]) {
                Psi.p[q][e] += a[q] * Pv.p[q][e];
                const double r = R.p[q][e] - a[q] * Qv.p[q][e];
                R.p[q][e] = r;
                acc[q] += r * r * w;
            }
    }
    __shared__ double sh[kThreads / 64][kMaxRhs];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < kMaxRhs; ++q) {
        double v = acc[q];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) sh[wave][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < kMaxRhs) {
        double t = 0.0;
        for (int u = 0; u < kThreads / 64; ++u) t += sh[u][threadIdx.x];
        part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// Y_q = X_q + beta_q Y_q for the active solves, over the listed units of sp
__global__ void __launch_bounds__(kThreads)
k_cg_xpby(int nr, VPtr<const double> X, VPtr<double> Y, int64_t n, const CgState *__restrict__ st, Span sp) {
    double b[kMaxRhs];
    bool on[kMaxRhs];
#pragma unroll
    for (int q = 0; q < kMaxRhs; ++q) {
        on[q] = q < nr && st->act[q];
        b[q] = on[q] ? st->beta[q] : 0.0;
    }
    const int64_t cnt = span_count<1>(sp, n);
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt; it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = span_elem<1>(sp, it);
        if (e >= n) continue;
#pragma unroll
        for (int q = 0; q < kMaxRhs; ++q)
            if (on[q]) Y.p[q][e] = X.p[q][e] + b[q] * Y.p[q][e];
    }
}

// X_q -= scale * val[q * stride] where mask != 0, for the vectors with X_q set
__global__ void __launch_bounds__(kThreads)
k_sub_masked_b(int64_t n, const double *__restrict__ mask, const double *__restrict__ val, int64_t stride,
               double scale, VPtr<double> X) {
    double m[kMaxRhs];
#pragma unroll
    for (int q = 0; q < kMaxRhs; ++q) m[q] = X.p[q] ? val[q * stride] * scale : 0.0;
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kThreads)
        if (mask[e] != 0.0)
#pragma unroll
            for (int q = 0; q < kMaxRhs; ++q)
                if (X.p[q]) X.p[q][e] -= m[q];
}

// Block forms for the eigensolver's basis work (NW <= 8 vectors at once):
// part[(i*NW + q)][block] = partial sums of V_i . (W_q * wt) for i < nv; the
// basis is read once, W once per chunk of CH basis vectors (CH * NW ~ 16
// accumulators per thread)

template <int VEC, int NW, int CH>
__global__ void __launch_bounds__(kThreads)
k_mdot_multi(int nv, const double *__restrict__ V, int64_t ld, const double *__restrict__ W, int64_t ldw,
             const double *__restrict__ wt, int64_t n, double *__restrict__ part, Span sp) {
    using O = Vec<VEC>;
    const int64_t nvec = n / VEC, ldv = ld / VEC, ldwv = ldw / VEC, cnt = span_count<VEC>(sp, nvec);
    __shared__ double sh[kThreads / 64][CH * NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c0 = 0; c0 < nv; c0 += CH) {
        const int cn = min(CH, nv - c0);
        double acc[CH][NW];
#pragma unroll
        for (int a = 0; a < CH; ++a)
#pragma unroll
            for (int q = 0; q < NW; ++q) acc[a][q] = 0.0;
        for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt;
             it += (int64_t)gridDim.x * kThreads) {
            const int64_t e = span_elem<VEC>(sp, it);
            if (e >= nvec) continue;
            typename O::T wv[NW];
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                wv[q] = O::ld(W + (int64_t)q * ldwv * VEC, e);
                if (wt) wv[q] = O::mul(wv[q], O::ld(wt, e));
            }
#pragma unroll
            for (int a = 0; a < CH; ++a)
                if (a < cn) {
                    const typename O::T v = O::ld(V + (int64_t)(c0 + a) * ldv * VEC, e);
#pragma unroll
                    for (int q = 0; q < NW; ++q) acc[a][q] += O::dot(v, wv[q]);
                }
        }
        if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
            const double tv = wt ? wt[n - 1] : 1.0;
            for (int a = 0; a < cn; ++a)
                for (int q = 0; q < NW; ++q)
                    acc[a][q] += V[(int64_t)(c0 + a) * ld + n - 1] * W[(int64_t)q * ldw + n - 1] * tv;
        }
#pragma unroll
        for (int a = 0; a < CH; ++a)
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                double v = acc[a][q];
                for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
                if (lane == 0) sh[wave][a * NW + q] = v;
            }
        __syncthreads();
        for (int t = threadIdx.x; t < cn * NW; t += kThreads) {
            double v = 0.0;
            for (int u = 0; u < kThreads / 64; ++u) v += sh[u][t];
            part[(int64_t)(c0 * NW + t) * gridDim.x + blockIdx.x] = v;
        }
        __syncthreads();
    }
}

// Y_q = sum_i C[i][q] V_i (overwrite) or Y_q -= sum_i C[i][q] V_i for q < NW;
// C row-major (nv x NW, device); one read of the basis
template <int VEC, int NW>
__global__ void __launch_bounds__(kThreads)
k_maxpy_multi(int nv, const double *__restrict__ V, int64_t ld, const double *__restrict__ C,
              double *__restrict__ Y, int64_t ldy, int64_t n, int overwrite, Span sp) {
    using O = Vec<VEC>;
    __shared__ double cs[256 * NW];
    for (int t = threadIdx.x; t < nv * NW; t += kThreads) cs[t] = C[t];
    __syncthreads();
    const int64_t nvec = n / VEC, ldv = ld / VEC, ldyv = ldy / VEC, cnt = span_count<VEC>(sp, nvec);
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt;
         it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = span_elem<VEC>(sp, it);
        if (e >= nvec) continue;
        typename O::T acc[NW];
#pragma unroll
        for (int q = 0; q < NW; ++q) acc[q] = O::zero();
        for (int i = 0; i < nv; ++i) {
            const typename O::T v = O::ld(V + (int64_t)i * ldv * VEC, e);
#pragma unroll
            for (int q = 0; q < NW; ++q) acc[q] = O::fma(cs[i * NW + q], v, acc[q]);
        }
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            double *y = Y + (int64_t)q * ldyv * VEC;
            O::st(y, e, overwrite ? acc[q] : O::fma(-1.0, acc[q], O::ld(y, e)));
        }
    }
    if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        for (int q = 0; q < NW; ++q) {
            double sacc = 0.0;
            for (int i = 0; i < nv; ++i) sacc += cs[i * NW + q] * V[(int64_t)i * ld + n - 1];
            double *y = Y + (int64_t)q * ldy;
            y[n - 1] = overwrite ? sacc : y[n - 1] - sacc;
        }
    }
}

// y = sum_i c_i V_i (overwrite) or y -= sum_i c_i V_i; w: optional input
// (out = scale * (w - sum c_i V_i) when w != nullptr)
template <int VEC, class TV = double>
__global__ void __launch_bounds__(kThreads)
k_maxpy(int nv, const TV *__restrict__ V, int64_t ld, const double *__restrict__ c,
        const double *__restrict__ cscale, const double *w, double scale, double *y, int64_t n, int overwrite,
        Span sp) {
    using O = Vec<VEC>;
    __shared__ double cs[256];
    for (int q = threadIdx.x; q < nv; q += kThreads) cs[q] = cscale ? c[q] * cscale[q] : c[q];
    __syncthreads();
    const int64_t nvec = n / VEC, ldv = ld / VEC, cnt = span_count<VEC>(sp, nvec);
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt;
         it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = span_elem<VEC>(sp, it);
        if (e >= nvec) continue;
        typename O::T s = O::zero();
        for (int q = 0; q < nv; ++q) s = O::fma(cs[q], BasisLd<VEC, TV>::ld(V + (int64_t)q * ldv * VEC, e), s);
        typename O::T r;
        if (w) r = O::scale(scale, O::fma(-1.0, s, O::ld(w, e)));
        else if (overwrite) r = s;
        else r = O::fma(-1.0, s, O::ld(y, e));
        O::st(y, e, r);
    }
    if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        double s = 0.0;
        for (int q = 0; q < nv; ++q) s += cs[q] * V[(int64_t)q * ld + n - 1];
        y[n - 1] = w ? scale * (w[n - 1] - s) : (overwrite ? s : y[n - 1] - s);
    }
}

// y -= sum_i c_i V_i for FP32 columns V_i, in FP64 (each value widened
// before use: the same result as with the widened columns), over the
// listed units of the span
__global__ void __launch_bounds__(kThreads)
k_maxpy_f32(int nv, const float *__restrict__ V, int64_t ld, const double *__restrict__ c, double *y, int64_t n,
            Span sp) {
    __shared__ double cs[256];
    for (int q = threadIdx.x; q < nv; q += kThreads) cs[q] = c[q];
    __syncthreads();
    const int64_t nvec = n / 2, cnt = span_count<2>(sp, nvec);
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt; it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = span_elem<2>(sp, it);
        if (e >= nvec) continue;
        double2 acc = make_double2(0.0, 0.0);
        for (int q = 0; q < nv; ++q) {
            const float2 v = reinterpret_cast<const float2 *>(V + (int64_t)q * ld)[e];
            acc = Vec<2>::fma(cs[q], make_double2((double)v.x, (double)v.y), acc);
        }
        double2 *yy = reinterpret_cast<double2 *>(y);
        yy[e] = Vec<2>::fma(-1.0, acc, yy[e]);
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        double acc = 0.0;
        for (int q = 0; q < nv; ++q) acc += cs[q] * (double)V[(int64_t)q * ld + n - 1];
        y[n - 1] -= acc;
    }
}

// Fused Gram--Schmidt step for nv <= MAXV basis vectors:
//   w' = w - sum_i c_i V_i      (written back to w)
//   part rows 0..nv-1: V_i . w', row nv: |w'|^2
// One read of the basis (held in registers) serves the update and the dots.
// REREAD: the basis values are loaded a second time for the dot products
// instead of being held in registers (more vectors than registers allow; the
// second load is served by the L2 or the Infinity Cache).  Measured: for 32
// vectors holding them took 212 VGPRs (2 waves per SIMD) and rereading 149
// (3 waves), 3% faster on the 9-cell quarter; for 16 vectors holding them
// (144 VGPRs) stays faster than rereading (85).
template <int VEC, int MAXV, bool REREAD, class TV = double>
__global__ void __launch_bounds__(kThreads)
k_maxpy_mdot_norm(BasisArgs<TV> A, int64_t ld, int64_t n, double *__restrict__ part0, int rows, Span sp) {
    using O = Vec<VEC>;
    const int nv = A.s[blockIdx.y].nv;
    const TV *__restrict__ V = A.s[blockIdx.y].V;
    const double *__restrict__ c = A.s[blockIdx.y].c, *__restrict__ cscale = A.s[blockIdx.y].cscale;
    double *__restrict__ w = A.s[blockIdx.y].w;
    double *__restrict__ part = part0 + (int64_t)blockIdx.y * rows * gridDim.x;
    __shared__ double cs[MAXV];
    for (int q = threadIdx.x; q < nv; q += kThreads) cs[q] = cscale ? c[q] * cscale[q] : c[q];
    __syncthreads();
    double acc[MAXV + 1];
#pragma unroll
    for (int q = 0; q <= MAXV; ++q) acc[q] = 0.0;
    const int64_t nvec = n / VEC, ldv = ld / VEC, cnt = span_count<VEC>(sp, nvec);
    for (int64_t it = (int64_t)blockIdx.x * kThreads + threadIdx.x; it < cnt;
         it += (int64_t)gridDim.x * kThreads) {
        const int64_t e = span_elem<VEC>(sp, it);
        if (e >= nvec) continue;
        typename O::T s = O::ld(w, e);
        if (REREAD) {
#pragma unroll
            for (int q = 0; q < MAXV; ++q)
                if (q < nv) s = O::fma(-cs[q], BasisLd<VEC, TV>::ld(V + (int64_t)q * ldv * VEC, e), s);
            O::st(w, e, s);
            // keep the compiler from holding the first loads in registers
            // for the second use (that costs 200+ VGPRs, 2 waves per SIMD)
            asm volatile("" ::: "memory");
#pragma unroll
            for (int q = 0; q < MAXV; ++q)
                if (q < nv) acc[q] += O::dot(BasisLd<VEC, TV>::ld(V + (int64_t)q * ldv * VEC, e), s);
        } else {
            typename O::T vv[REREAD ? 1 : MAXV];
#pragma unroll
            for (int q = 0; q < MAXV; ++q)
                if (q < nv) {
                    vv[q] = BasisLd<VEC, TV>::ld(V + (int64_t)q * ldv * VEC, e);
                    s = O::fma(-cs[q], vv[q], s);
                }
            O::st(w, e, s);
#pragma unroll
            for (int q = 0; q < MAXV; ++q)
                if (q < nv) acc[q] += O::dot(vv[q], s);
        }
        acc[MAXV] += O::dot(s, s);
    }
    if (VEC == 2 && (n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        double t = w[n - 1];
#pragma unroll
        for (int q = 0; q < MAXV; ++q)
            if (q < nv) t -= cs[q] * V[(int64_t)q * ld + n - 1];
        w[n - 1] = t;
#pragma unroll
        for (int q = 0; q < MAXV; ++q)
            if (q < nv) acc[q] += V[(int64_t)q * ld + n - 1] * t;
        acc[MAXV] += t * t;
    }
    __shared__ double sh[kThreads / 64][MAXV + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q <= MAXV; ++q) {
        if (q < nv || q == MAXV) {
            double v = acc[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
            if (lane == 0) sh[wave][q] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x <= nv) {  // row nv carries |w'|^2
        const int q = threadIdx.x < nv ? threadIdx.x : MAXV;
        double t = 0.0;
        for (int u = 0; u < kThreads / 64; ++u) t += sh[u][q];
        part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

__global__ void k_sub_masked(int64_t n, const double *__restrict__ mask,
                             const double *__restrict__ val, double scale, double *__restrict__ x) {
    const double m = val[0] * scale;
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kThreads)
        if (mask[e] != 0.0) x[e] -= m;
}

__global__ void k_mask_mul(int64_t n, const double *__restrict__ mask, double *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kThreads)
        if (mask[e] == 0.0) x[e] = 0.0;
}

// SplitMix64 (Steele, Lea & Flood 2014) used as a counter-based hash:
// the value for counter c is the generator's output after c+1 steps from seed.
__device__ inline uint64_t splitmix64_at(uint64_t seed, uint64_t c) {
    uint64_t z = seed + (c + 1) * 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__global__ void k_randn(int64_t n, uint64_t seed, int64_t offset, const double *__restrict__ mask,
                        double *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kThreads) {
        if (mask[e] == 0.0) {
            x[e] = 0.0;
            continue;
        }
        const uint64_t c = 2 * (uint64_t)(e + offset);
        const double u1 = ((double)(splitmix64_at(seed, c) >> 11) + 1.0) * 0x1.0p-53;
        const double u2 = (double)(splitmix64_at(seed, c + 1) >> 11) * 0x1.0p-53;
        x[e] = sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
    }
}

// The transfers of the tilde form (eq. fullMat2): entry e of a face vector
// scaled by a^(1/2) (power > 0) or a^(-1/2) (power < 0) of its own face,
// a = coef[e] (the first three coefficient blocks are ax ay az in the face
// vector's layout); inactive entries become 0
template <class T>
__global__ void k_scale_a(int64_t n, const T *__restrict__ a, int power, T *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kThreads) {
        const T ae = a[e];
        x[e] = ae > T(0) ? (power > 0 ? x[e] * sqrt(ae) : x[e] / sqrt(ae)) : T(0);
    }
}

// x += a^(-1/2) r on the active entries
template <class T>
__global__ void k_add_scaled_a(int64_t n, const T *__restrict__ a, const T *__restrict__ r, T *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kThreads) {
        const T ae = a[e];
        if (ae > T(0)) x[e] += r[e] / sqrt(ae);
    }
}

// Electric field of an eigenvector at sample points: e = C^T b / k on the
// edges with l > 0 (zero on the others, e.g. the conducting walls), the
// circulation of b around each edge divided by h (the Yee scheme's Ampere
// law in the frequency domain), interpolated trilinearly from each
// component's own edge lattice (e_x at ((i + 1/2) h, j h, k h), ...).  One
// thread per point; a point whose stencil leaves the grid gets NaN.
__device__ inline double edge_e(const Grid &g, const Coefs<double> &c, const double *__restrict__ b, int comp, int i,
                                int j, int k, double inv_kh) {
    const int64_t P = g.P, dy = g.sy, dz = g.sz, p = pidx(g, i, j, k);
    const double *X = b, *Y = b + P, *Z = b + 2 * P;
    if (comp == 0) {
        if (!(c.lx[p] > 0.0)) return 0.0;
        return (Z[p] - Z[p - dy] - Y[p] + Y[p - dz]) * inv_kh;
    }
    if (comp == 1) {
        if (!(c.ly[p] > 0.0)) return 0.0;
        return (X[p] - X[p - dz] - Z[p] + Z[p - 1]) * inv_kh;
    }
    if (!(c.lz[p] > 0.0)) return 0.0;
    return (Y[p] - Y[p - 1] - X[p] + X[p - dy]) * inv_kh;
}

__global__ void k_sample_e(Grid g, Coefs<double> c, const double *__restrict__ b, double inv_kh, int npts,
                           const double *__restrict__ pts, double *__restrict__ out) {
    const int q = blockIdx.x * kThreads + threadIdx.x;
    if (q >= npts) return;
    const int n[3] = {g.nx, g.ny, g.nz};
    for (int comp = 0; comp < 3; ++comp) {
        int i0[3];
        double t[3];
        bool ok = true;
        for (int a = 0; a < 3; ++a) {
            const double u = pts[3 * q + a] / g.h - (a == comp ? 0.5 : 0.0);
            const double f = floor(u);
            i0[a] = (int)f;
            t[a] = u - f;
            // edge lattice along comp: 0 .. n-1; across: 0 .. n
            const int hi = a == comp ? n[a] - 1 : n[a];
            if (!(f >= 0.0) || i0[a] + 1 > hi) ok = false;
        }
        double v = 0.0;
        if (ok) {
            for (int corner = 0; corner < 8; ++corner) {
                const int dx = corner & 1, dy = (corner >> 1) & 1, dz = corner >> 2;
                const double w = (dx ? t[0] : 1.0 - t[0]) * (dy ? t[1] : 1.0 - t[1]) * (dz ? t[2] : 1.0 - t[2]);
                if (w != 0.0) v += w * edge_e(g, c, b, comp, i0[0] + dx, i0[1] + dy, i0[2] + dz, inv_kh);
            }
        } else {
            v = __builtin_nan("");
        }
        out[3 * q + comp] = v;
    }
}

// x = in where mask != 0, else 0
__global__ void k_copy_masked(int64_t n, const double *__restrict__ in, const double *__restrict__ mask,
                              double *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kThreads)
        x[e] = mask[e] != 0.0 ? in[e] : 0.0;
}

// ---------------------------------------------------------------------------
// Batched V-cycle steps (see BJob): the same bodies as the single-operator
// kernels.  The cut rows take the FP32 tables but for the centre weight, and
// are summed in FP64.  With a centre weight rounded to FP32 (6 / h^2 beside
// neighbours of 1 / h^2) and sums in FP32 the fused V-cycle of smooth fields
// was left with an error of 6.5e-8 (rms against FP64, eight cavities of 16^3 to
// 64^3), where rows formed from the fractions had 5.1e-8; these leave 4.6e-8
// at the same speed (885 and 893 us for 16 cavities of 32^3 to 96^3; FP64
// tables throughout left 4.4e-8 and took 973).  A block finds its job in a
// table (one scalar load; a search over the jobs' offsets took a dependent
// load per halving), and the XCDs, which blocks reach round-robin, each take
// one run of logical blocks.
// ---------------------------------------------------------------------------
template <int STEP, int COMP>
__global__ void __launch_bounds__(kThreads)
kb_step(const BJob *__restrict__ jobs, const int32_t *__restrict__ job_of) {
    const uint32_t L = blockIdx.x % kXcd * (gridDim.x / kXcd) + blockIdx.x / kXcd;
    const int q = job_of[L];
    if (q < 0) return;   // padding to a multiple of 8
    const BJob &J = jobs[q];
    const int64_t lb = (int64_t)L - J.block0;
    const int64_t item = lb * blockDim.x + threadIdx.x;
    using T = float;
    if (STEP == BS_ZERO) {
        if (item < J.items) J.out[item] = T(0);
    } else if (STEP == BS_SMOOTH) {
        if (lb < J.ncut) {
            if (item < J.n)
                smooth_cut_n<T, COMP, 1, double>(J.g, J.sigma, J.cut, J.n, J.colour, CutTab<T, double>{J.w, J.w0}, J.pair,
                                                 J.s, 0, vptr1(J.in), vptr1(J.out), (uint32_t)item);
        } else {
            smooth_vac_n<T, COMP, 1>(J.g, J.sigma, vptr1(J.in), vptr1(J.out), (uint32_t)(item - J.ncut * blockDim.x),
                                     J.runs, J.nruns);
        }
    } else if (STEP == BS_RESID) {
        if (lb < J.ncut) {
            apply_cut_part<T, AK_RESID, T, double>(J.g, J.sigma, CutTab<T, double>{J.w, J.w0}, J.cut, J.n, true,
                                                   (uint32_t)(item >> 6), (uint32_t)(item & 63), J.in, J.aux, J.out);
        } else {
            const uint32_t t = (uint32_t)(item - J.ncut * blockDim.x);
            if (t >> kRunLog >= J.nruns) return;
            const CellRun run = J.cells[t >> kRunLog];
            const uint32_t lane = t & (kRunLanes - 1);
            apply_run<T, AK_RESID, T>(J.g, J.sigma, run, lane, J.in, J.aux, J.out);
        }
    } else if (STEP == BS_RESTRICT) {
        restrict_body<T>(J.g, J.gc, coefs_of(J.cc, J.gc.P), J.in, J.out, listed_item(J.gc, J.rows, J.nrows, item), J.xz);
    } else if (STEP == BS_PROLONG) {
        prolong_body<T>(J.g, J.gc, coefs_of(J.c, J.g.P), coefs_of(J.cc, J.gc.P), J.in, J.out,
                        listed_item(J.g, J.rows, J.nrows, item));
    } else {
        coarse_body<T>(J.ncoarse, J.inv, J.idx, J.in, J.out, (int)lb);
    }
}

__global__ void __launch_bounds__(kLdsThreads)
kb_sweeps(const BJob *__restrict__ jobs) {
    const BJob &J = jobs[blockIdx.x];
    sweeps_lds_body<float, false, double>(J.g, J.sigma, J.lds, CutTab<float, double>{J.lds.w32, J.lds.w64}, J.sweeps,
                                          J.reverse, !J.reverse, J.in, J.out, reinterpret_cast<float *>(lds_raw));
}

}  // namespace

void launch_batched(int step, int comp, const BJob *jobs, const int32_t *job_of, int64_t nblocks, int tpb,
                    size_t lds, hipStream_t s) {
    const dim3 grid((unsigned)nblocks), block((unsigned)(step == BS_COARSE ? kThreads : tpb));
    switch (step) {
        case BS_ZERO: hipLaunchKernelGGL((kb_step<BS_ZERO, 0>), grid, block, 0, s, jobs, job_of); break;
        case BS_SMOOTH:
            if (comp == 0) hipLaunchKernelGGL((kb_step<BS_SMOOTH, 0>), grid, block, 0, s, jobs, job_of);
            else if (comp == 1) hipLaunchKernelGGL((kb_step<BS_SMOOTH, 1>), grid, block, 0, s, jobs, job_of);
            else hipLaunchKernelGGL((kb_step<BS_SMOOTH, 2>), grid, block, 0, s, jobs, job_of);
            break;
        case BS_RESID: hipLaunchKernelGGL((kb_step<BS_RESID, 0>), grid, block, 0, s, jobs, job_of); break;
        case BS_RESTRICT: hipLaunchKernelGGL((kb_step<BS_RESTRICT, 0>), grid, block, 0, s, jobs, job_of); break;
        case BS_PROLONG: hipLaunchKernelGGL((kb_step<BS_PROLONG, 0>), grid, block, 0, s, jobs, job_of); break;
        case BS_SWEEPS: hipLaunchKernelGGL(kb_sweeps, grid, dim3(kLdsThreads), lds, s, jobs); break;
        default: hipLaunchKernelGGL((kb_step<BS_COARSE, 0>), grid, block, 0, s, jobs, job_of); break;
    }
}

namespace {

inline dim3 flat_grid(int64_t n) {
    int64_t nb = ceil_div(n, kThreads);
    if (nb > 8192) nb = 8192;
    if (nb < 1) nb = 1;
    return dim3((unsigned)nb);
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <class T>
void launch_apply(const Grid &g, T sigma, int kind, const T *f, const T *x, T *y, hipStream_t s,
                  const ClassList &cut) {
    launch_apply_b<T>(g, sigma, kind, 1, vptr1(f), vptr1(x), vptr1(y), s, cut);
}

template <class T>
void launch_apply_K(const Grid &g, const T *coef, const T *x, T *y, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL((k_apply_K<T>), xcd_grid(n), dim3(kThreads), 0, s, g, coefs_of(coef, g.P), x, y);
}

template <class T>
void launch_apply_A_t(const Grid &g, const T *coef, const T *x, T *y, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL((k_apply_A<T>), xcd_grid(n), dim3(kThreads), 0, s, g, coefs_of(coef, g.P), x, y);
}

void launch_apply_A(const Grid &g, const double *coef, const double *x, double *y, hipStream_t s) {
    launch_apply_A_t<double>(g, coef, x, y, s);
}

template <class T>
void launch_smooth(const Grid &g, T sigma, int comp, const T *f, T *x, hipStream_t s, const ClassList &cl) {
    launch_smooth_b<T>(g, sigma, comp, 1, vptr1(f), vptr1(x), s, cl);
}

template <class T>
void launch_restrict(const Grid &gf, const Grid &gc, const T *coef_c, const T *r, T *fc,
                     hipStream_t s) {
    const int64_t n = (int64_t)gc.nx * gc.ny * gc.nz;
    hipLaunchKernelGGL((k_restrict<T>), xcd_grid(n), dim3(kThreads), 0, s, gf, gc,
                       coefs_of(coef_c, gc.P), r, fc);
}

template <class T>
void launch_prolong_add(const Grid &gf, const Grid &gc, const T *coef_f, const T *coef_c, const T *xc,
                        T *x, hipStream_t s) {
    const int64_t n = (int64_t)gf.nx * gf.ny * gf.nz;
    hipLaunchKernelGGL((k_prolong_add<T>), xcd_grid(n), dim3(kThreads), 0, s, gf, gc,
                       coefs_of(coef_f, gf.P), coefs_of(coef_c, gc.P), xc, x);
}

// ---- block forms: dispatch nr (1..kMaxRhs) to the template
#define DM_NR_SWITCH(nr, CALL)                      \
    switch (nr) {                                   \
        case 1: { constexpr int NR = 1; CALL; } break; \
        case 2: { constexpr int NR = 2; CALL; } break; \
        case 3: { constexpr int NR = 3; CALL; } break; \
        case 4: { constexpr int NR = 4; CALL; } break; \
        default: throw std::runtime_error("block of more than 4 vectors"); \
    }

namespace {
// A single vector's whole-grid product or residual gives each listed cell's
// rows to three threads below this many cut cells, and to one from there on:
// a short list is bound by its dependent loads, a long one by memory, and one
// thread's rows share their lines.  In us, split against not: residual FP32
// 2.56 and 3.24 for 5,606 cut cells (32^3), 4.59 and 4.66 for 22,688 (64^3),
// 5.61 and 5.48 for 28,730 (72^3), 9.07 and 8.60 for 41,906 (32 x 32 x 336
// quarter), 21.3 and 19.5 for 99,127 (48 x 48 x 512); FP64 9.28 and 9.32 for
// 28,730, 17.0 and 16.2 for 77,407 (16 x 128 x 256).  Several vectors share
// the tables' lines between their waves: split at every length (FP64, three
// vectors, 48 x 48 x 512: 86.6 and 89.8), as are the V-cycle's residuals,
// most of whose levels are short.
constexpr int64_t kApplySplit = 1 << 15;

template <class T>
ApplyArgs<T> apply_args(const Grid &g, const ClassList &cut, int nr, dim3 &grid) {
    if (cut.n > 0 && !cut_weights<T>(cut)) throw std::runtime_error("apply: cut-cell list without its row table");
    if (!cut.cells && !cut.flags) throw std::runtime_error("apply: neither runs nor class bytes");
    ApplyArgs<T> A;
    A.cut = cut.idx;
    A.W = cut_weights<T>(cut);
    A.cells = cut.cells;
    A.flags = cut.flags;
    A.ncut = cut.n;
    A.split = nr > 1 || cut.cells || cut.n < kApplySplit;
    A.ncb = (uint32_t)(ceil_div((A.split ? 3 : 1) * ceil_div(cut.n, 64), kXcd) * kXcd);
    A.nruns = (uint32_t)cut.nruns;
    const int64_t items = cut.cells ? cut.nruns << kRunLog : (int64_t)g.nx * g.ny * g.nz;
    grid = dim3((unsigned)(A.ncb + ceil_div(ceil_div(items, 64), kXcd) * kXcd));
    return A;
}
}  // namespace

template <class T>
void launch_apply_b(const Grid &g, T sigma, int kind, int nr, const VPtr<const T> &f,
                    const VPtr<const T> &x, const VPtr<T> &y, hipStream_t s, const ClassList &cut) {
    if (kind != AK_M && kind != AK_RESID) throw std::runtime_error("block apply: M or residual only");
    dim3 grid;
    const ApplyArgs<T> A = apply_args<T>(g, cut, nr, grid);
    if (grid.x == 0) return;   // no listed cell
    if (kind == AK_M)
        DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_apply_split<T, AK_M, NR>), grid, dim3(64 * NR), 0, s, g, sigma, A, f, x, y))
    else
        DM_NR_SWITCH(nr,
                     hipLaunchKernelGGL((k_apply_split<T, AK_RESID, NR>), grid, dim3(64 * NR), 0, s, g, sigma, A, f, x, y))
}

void launch_apply_m_f32in(const Grid &g, double sigma, int nr, const VPtr<const float> &x,
                         const VPtr<double> &y, hipStream_t s, const ClassList &cut) {
    dim3 grid;
    const ApplyArgs<double> A = apply_args<double>(g, cut, nr, grid);
    if (grid.x == 0) return;   // no listed cell
    const VPtr<const double> f{};
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_apply_split<double, AK_M, NR, float>), grid, dim3(64 * NR), 0, s, g, sigma, A,
                                        f, x, y))
}

template <class T>
void launch_smooth_b(const Grid &g, T sigma, int comp, int nr, const VPtr<const T> &f, const VPtr<T> &x,
                     hipStream_t s, const ClassList &cl) {
    if (cl.n > 0 && !cut_weights<T>(cl)) throw std::runtime_error("smoother: cut list without its row table");
    if (cl.pair != kPairNone && !cl.s) throw std::runtime_error("smoother: paired update without its sums");
    SmoothArgs<T> A;
    A.cut = cl.idx;
    A.W = cut_weights<T>(cl);
    A.S = static_cast<T *>(cl.s);
    A.runs = cl.runs;
    A.n = cl.n;
    A.colour = cl.colour;
    A.nruns = (uint32_t)cl.nruns;
    A.pair = cl.pair;
    A.wave_split = nr > 1 && cl.n < cl.wave_split_max;
    A.ncb = (uint32_t)(ceil_div(ceil_div(cl.n, A.wave_split ? 64 : kThreads), kXcd) * kXcd);
    const int64_t nvb = ceil_div(ceil_div(cl.nruns << kRunLog, kThreads), kXcd) * kXcd;
    const dim3 grid((unsigned)(A.ncb + nvb));
    if (grid.x == 0) return;   // no active face of the class on this level
    if (comp == 0)
        DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_smooth_split<T, 0, NR>), grid, dim3(kThreads), 0, s, g, sigma, A, f, x))
    else if (comp == 1)
        DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_smooth_split<T, 1, NR>), grid, dim3(kThreads), 0, s, g, sigma, A, f, x))
    else
        DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_smooth_split<T, 2, NR>), grid, dim3(kThreads), 0, s, g, sigma, A, f, x))
}

template <class T>
void launch_sweeps_lds(const Grid &g, T sigma, const LdsRows &R, int sweeps, int reverse, int zero, int nr,
                       const VPtr<const T> &f, const VPtr<T> &x, hipStream_t s) {
    if (3 * g.P * (int64_t)sizeof(T) > kLdsBytes) throw std::runtime_error("LDS sweeps: the level does not fit");
    const T *W = std::is_same<T, double>::value ? (const T *)R.w64 : (const T *)R.w32;
    if (R.cut_off[6] > 0 && !W) throw std::runtime_error("LDS sweeps: cut list without its row table");
    const size_t lds = (size_t)(3 * g.P) * sizeof(T);
    if (g.pmc)
        hipLaunchKernelGGL((k_sweeps_lds<T, true>), dim3((unsigned)nr), dim3(kLdsThreads), lds, s, g, sigma, R, W,
                           sweeps, reverse, zero, f, x);
    else
        hipLaunchKernelGGL((k_sweeps_lds<T, false>), dim3((unsigned)nr), dim3(kLdsThreads), lds, s, g, sigma, R, W,
                           sweeps, reverse, zero, f, x);
}

template <class T>
void launch_restrict_b(const Grid &gf, const Grid &gc, const T *coef_c, int nr, const VPtr<const T> &r,
                       const VPtr<T> &fc, hipStream_t s, const VPtr<T> &xz, const int32_t *rows, int64_t nrows) {
    const int64_t n = rows ? nrows * gc.nx : (int64_t)gc.nx * gc.ny * gc.nz;
    const Coefs<T> cc = coefs_of(coef_c, gc.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_restrict_b<T, NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, gf, gc, cc,
                                        rows, nrows, r, fc, xz))
}

template <class T>
void launch_prolong_add_b(const Grid &gf, const Grid &gc, const T *coef_f, const T *coef_c, int nr,
                          const VPtr<const T> &xc, const VPtr<T> &x, hipStream_t s, const int32_t *rows,
                          int64_t nrows) {
    const int64_t n = rows ? nrows * gf.nx : (int64_t)gf.nx * gf.ny * gf.nz;
    const Coefs<T> cf = coefs_of(coef_f, gf.P), cc = coefs_of(coef_c, gc.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_prolong_add_b<T, NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, gf, gc, cf,
                                        cc, rows, nrows, xc, x))
}

template <class T>
void launch_coarse_solve_b(int n, const double *inv, const int64_t *idx, int nr, const VPtr<const T> &f,
                           const VPtr<T> &x, hipStream_t s) {
    if (n <= 0) return;
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_coarse_solve_b<T, NR>), dim3(n), dim3(kThreads), 0, s, n, inv, idx, f, x))
}

void launch_div_DA_b(const Grid &g, const double *coef, int nr, const VPtr<const double> &b,
                     const VPtr<double> &out, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const Coefs<double> c = coefs_of(coef, g.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_div_DA_b<NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, g, c, b, out))
}

void launch_grad_sub_b(const Grid &g, const double *coef, int nr, const VPtr<const double> &psi,
                       const VPtr<const double> &b_in, const VPtr<double> &b_out, double scale, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    const Coefs<double> c = coefs_of(coef, g.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_grad_sub_b<NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, g, c, psi, b_in,
                                        b_out, scale))
}

template <class T>
void launch_s_apply_b(const Grid &g, const T *coef, double w, int resid, int nr, const VPtr<const T> &f,
                      const VPtr<const T> &x, const VPtr<T> &y, hipStream_t s, const int32_t *rows, int64_t nrows) {
    const int64_t n = rows ? nrows * g.nx : (int64_t)g.nx * g.ny * g.nz;
    const Coefs<T> c = coefs_of(coef, g.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_s_apply_b<T, NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, g, c, (T)w,
                                        resid, rows, nrows, f, x, y))
}

template <class T>
void launch_s_smooth_b(const Grid &g, const T *coef, double w, int colour, int nr, const VPtr<const T> &f,
                       const VPtr<T> &x, hipStream_t s, const int32_t *rows, int64_t nrows) {
    const int64_t n = (int64_t)((g.nx + 1) >> 1) * (rows ? nrows : (int64_t)g.ny * g.nz);
    const Coefs<T> c = coefs_of(coef, g.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_s_smooth_b<T, NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, g, c, (T)w,
                                        colour, rows, nrows, f, x))
}

template <class T>
void launch_s_restrict_b(const Grid &gf, const Grid &gc, const T *coef_c, int nr, const VPtr<const T> &r,
                         const VPtr<T> &fc, hipStream_t s, const VPtr<T> &xz, const int32_t *rows, int64_t nrows) {
    const int64_t n = rows ? nrows * gc.nx : (int64_t)gc.nx * gc.ny * gc.nz;
    const Coefs<T> cc = coefs_of(coef_c, gc.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_s_restrict_b<T, NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, gf, gc, cc,
                                        rows, nrows, r, fc, xz))
}

template <class T>
void launch_s_prolong_add_b(const Grid &gf, const Grid &gc, const T *coef_f, int nr, const VPtr<const T> &xc,
                            const VPtr<T> &x, hipStream_t s, const int32_t *rows, int64_t nrows) {
    const int64_t n = rows ? nrows * gf.nx : (int64_t)gf.nx * gf.ny * gf.nz;
    const Coefs<T> cf = coefs_of(coef_f, gf.P);
    DM_NR_SWITCH(nr, hipLaunchKernelGGL((k_s_prolong_add_b<T, NR>), xcd_grid_waves(n), dim3(64 * NR), 0, s, gf, gc,
                                        cf, rows, nrows, xc, x))
}

#define DM_SCALAR_BLOCK(T)                                                                                        \
    template void launch_s_apply_b<T>(const Grid &, const T *, double, int, int, const VPtr<const T> &,           \
                                      const VPtr<const T> &, const VPtr<T> &, hipStream_t, const int32_t *,       \
                                      int64_t);                                                                   \
    template void launch_s_smooth_b<T>(const Grid &, const T *, double, int, int, const VPtr<const T> &,          \
                                       const VPtr<T> &, hipStream_t, const int32_t *, int64_t);                   \
    template void launch_s_restrict_b<T>(const Grid &, const Grid &, const T *, int, const VPtr<const T> &,       \
                                         const VPtr<T> &, hipStream_t, const VPtr<T> &, const int32_t *,          \
                                         int64_t);                                                                \
    template void launch_s_prolong_add_b<T>(const Grid &, const Grid &, const T *, int, const VPtr<const T> &,    \
                                            const VPtr<T> &, hipStream_t, const int32_t *, int64_t);
DM_SCALAR_BLOCK(double)
DM_SCALAR_BLOCK(float)
#undef DM_SCALAR_BLOCK

#undef DM_NR_SWITCH

template <class TI, class TO>
void launch_cast(const TI *in, TO *out, int64_t n, hipStream_t s, Span sp) {
    if (sp.u)
        hipLaunchKernelGGL((k_cast_units<TI, TO>), flat_grid(sp.n * kSpanUnit), dim3(kThreads), 0, s, in, out, n,
                           sp.u, sp.n);
    else
        hipLaunchKernelGGL((k_cast<TI, TO>), flat_grid(n), dim3(kThreads), 0, s, in, out, n);
}

template <class T>
void launch_coarse_solve(int n, const double *inv, const int64_t *idx, const T *f, T *x,
                         hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL((k_coarse_solve<T>), dim3(n), dim3(kThreads), 0, s, n, inv, idx, f, x);
}

void launch_div_DA(const Grid &g, const double *coef, const double *b, double *gout,
                   hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_div_DA, xcd_grid(n), dim3(kThreads), 0, s, g, coefs_of(coef, g.P), b, gout);
}

void launch_grad_sub(const Grid &g, const double *coef, const double *psi, double *b_in,
                     double *b_out, double scale, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_grad_sub, xcd_grid(n), dim3(kThreads), 0, s, g, coefs_of(coef, g.P), psi,
                       (const double *)b_in, b_out, scale);
}

void launch_s_apply(const Grid &g, const double *coef, double w, int resid, const double *f,
                    const double *x, double *y, hipStream_t s) {
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_s_apply, xcd_grid(n), dim3(kThreads), 0, s, g, coefs_of(coef, g.P), w,
                       resid, f, x, y);
}

void launch_s_smooth(const Grid &g, const double *coef, double w, int colour, const double *f,
                     double *x, hipStream_t s) {
    const int64_t n = (int64_t)((g.nx + 1) >> 1) * g.ny * g.nz;
    hipLaunchKernelGGL(k_s_smooth, xcd_grid(n), dim3(kThreads), 0, s, g, coefs_of(coef, g.P), w,
                       colour, f, x);
}

void launch_s_restrict(const Grid &gf, const Grid &gc, const double *coef_c, const double *r,
                       double *fc, hipStream_t s) {
    const int64_t n = (int64_t)gc.nx * gc.ny * gc.nz;
    hipLaunchKernelGGL(k_s_restrict, xcd_grid(n), dim3(kThreads), 0, s, gf, gc,
                       coefs_of(coef_c, gc.P), r, fc);
}

void launch_s_prolong_add(const Grid &gf, const Grid &gc, const double *coef_f,
                          const double *xc, double *x, hipStream_t s) {
    const int64_t n = (int64_t)gf.nx * gf.ny * gf.nz;
    hipLaunchKernelGGL(k_s_prolong_add, xcd_grid(n), dim3(kThreads), 0, s, gf, gc,
                       coefs_of(coef_f, gf.P), xc, x);
}

template <class T>
void launch_mirror_faces(const Grid &g, T *x, hipStream_t s) {
    const int n[3] = {g.nx, g.ny, g.nz};
    for (int a = 0; a < 3; ++a) {
        if (!((g.pmc >> a) & 1)) continue;
        const int b = a == 0 ? 1 : 0, d = a == 2 ? 1 : 2;
        const int64_t cnt = (int64_t)(n[b] + 2) * (n[d] + 2);
        hipLaunchKernelGGL((k_mirror_faces<T>), dim3((unsigned)ceil_div(cnt, kThreads)), dim3(kThreads), 0, s, g, a, x);
    }
}

template <class T>
void launch_mirror_cells(const Grid &g, T *x, hipStream_t s) {
    const int n[3] = {g.nx, g.ny, g.nz};
    for (int a = 0; a < 3; ++a) {
        if (!((g.pmc >> a) & 1)) continue;
        const int b = a == 0 ? 1 : 0, d = a == 2 ? 1 : 2;
        const int64_t cnt = (int64_t)(n[b] + 2) * (n[d] + 2);
        hipLaunchKernelGGL(k_mirror_cells<T>, dim3((unsigned)ceil_div(cnt, kThreads)), dim3(kThreads), 0, s, g, a, x);
    }
}
template void launch_mirror_cells<double>(const Grid &, double *, hipStream_t);
template void launch_mirror_cells<float>(const Grid &, float *, hipStream_t);

template void launch_mirror_faces<double>(const Grid &, double *, hipStream_t);
template void launch_mirror_faces<float>(const Grid &, float *, hipStream_t);

void launch_axpy(int64_t n, double a, const double *x, double *y, hipStream_t s) {
    hipLaunchKernelGGL(k_axpy, flat_grid(n), dim3(kThreads), 0, s, n, a, x, y);
}
void launch_axpby(int64_t n, double a, const double *x, double b, double *y, hipStream_t s) {
    hipLaunchKernelGGL(k_axpby, flat_grid(n), dim3(kThreads), 0, s, n, a, x, b, y);
}
template <class T>
void launch_zero(int64_t n, T *x, hipStream_t s) {
    hipLaunchKernelGGL(k_zero<T>, flat_grid(n), dim3(kThreads), 0, s, n, x);
}
template void launch_zero<double>(int64_t, double *, hipStream_t);
template void launch_zero<float>(int64_t, float *, hipStream_t);

void launch_scale(int64_t n, double a, double *x, hipStream_t s) {
    hipLaunchKernelGGL(k_scale, flat_grid(n), dim3(kThreads), 0, s, n, a, x);
}
void launch_copy(int64_t n, const double *x, double *y, hipStream_t s) {
    (void)hipMemcpyAsync(y, x, n * sizeof(double), hipMemcpyDeviceToDevice, s);
}

namespace {
inline bool vec2_ok(int64_t n, int64_t ld, std::initializer_list<const void *> ptrs) {
    if ((n & 1) && ld != 0) return false;
    if (ld & 1) return false;
    for (const void *p : ptrs)
        if (p && ((uintptr_t)p & 15)) return false;
    return true;
}
// the same for a Krylov basis of element type TV with the FP64 vectors in
// `ptrs`: FP32 columns are read as pairs of floats (8-byte aligned)
template <class TV>
inline bool vec2_basis_ok(int64_t n, int64_t ld, const TV *V, std::initializer_list<const void *> ptrs) {
    if (sizeof(TV) == 8) return vec2_ok(n, ld, {V}) && vec2_ok(n, ld, ptrs);
    return ((uintptr_t)V & 7) == 0 && vec2_ok(n, ld, ptrs);
}
// an FP32 basis read four floats at a time: lengths and strides multiples
// of 4, every pointer 16-byte aligned
template <class TV>
inline bool vec4_basis_ok(int64_t n, int64_t ld, const TV *V, std::initializer_list<const void *> ptrs) {
    if (sizeof(TV) == 8 || (n & 3) || (ld & 3) || ((uintptr_t)V & 15)) return false;
    for (const void *p : ptrs)
        if (p && ((uintptr_t)p & 15)) return false;
    return true;
}
// f(width) with the widest load width (a std::integral_constant) that the
// basis type and the pointers allow: 4 (FP32 basis only), 2 or 1
template <class TV, class F>
inline void with_basis_width(int64_t n, int64_t ld, const TV *V, std::initializer_list<const void *> ptrs, F &&f) {
    if constexpr (sizeof(TV) == 4)
        if (vec4_basis_ok(n, ld, V, ptrs)) return f(std::integral_constant<int, 4>{});
    if (vec2_basis_ok(n, ld, V, ptrs)) return f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 1>{});
}

// workgroups of a reduction over `items` grid-stride items: a short vector
// takes no more than have an item (each further one would add a row of zeros
// to sum and its own shuffles: 8.0 us per launch for the 16^3 grid's 8,700
// pairs in 1,024 workgroups)
inline int reduce_grid(int64_t items, int most = kReduceBlocks) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(most, ceil_div(items, kThreads)));
}
inline int64_t span_items(const Span &sp, int64_t n) { return sp.u ? sp.n * kSpanUnit : n; }

template <class TV>
void basis_dots(int nsys, const BasisArgs<TV> &A, int64_t ld, const double *wt, int64_t n, double *part,
                hipStream_t s, Span sp) {
    int rows = 0;
    for (int q = 0; q < nsys; ++q) rows = std::max(rows, A.s[q].nv);
    if (rows <= 0) return;
    if (rows > 256 || (nsys > 1 && (rows + 1) * nsys > 256)) throw std::runtime_error("basis dots: too many vectors");
    // the widest load that every system's pointers allow
    int width = 4;
    for (int q = 0; q < nsys; ++q)
        with_basis_width(n, ld, A.s[q].V, {A.s[q].w, wt}, [&](auto w) { width = std::min(width, (int)decltype(w)::value); });
    const int nb = reduce_grid(span_items(sp, n) / width);
    const dim3 grid((unsigned)nb, (unsigned)nsys);
    if (sizeof(TV) == 4 && width == 4)
        hipLaunchKernelGGL((k_mdot<sizeof(TV) == 4 ? 4 : 2, TV>), grid, dim3(kThreads), 0, s, A, ld, wt, n, part, rows, sp);
    else if (width >= 2)
        hipLaunchKernelGGL((k_mdot<2, TV>), grid, dim3(kThreads), 0, s, A, ld, wt, n, part, rows, sp);
    else
        hipLaunchKernelGGL((k_mdot<1, TV>), grid, dim3(kThreads), 0, s, A, ld, wt, n, part, rows, sp);
    hipLaunchKernelGGL(k_basis_final<TV>, dim3((unsigned)rows, (unsigned)nsys), dim3(kThreads), 0, s, A, nb,
                       (const double *)part, rows, 0);
}

template <class TV>
void launch_mdot_t(int nv, const TV *V, int64_t ld, const double *w, const double *wt, int64_t n, double *part,
                   double *dout, hipStream_t s, Span sp) {
    if (nv > 256) throw std::runtime_error("launch_mdot: more than 256 vectors");
    BasisArgs<TV> A{};
    A.s[0] = {V, const_cast<double *>(w), nullptr, nullptr, dout, nv};
    basis_dots<TV>(1, A, ld, wt, n, part, s, sp);
}
}  // namespace

template <class TV>
void launch_basis_dots(int nsys, const BasisArgs<TV> &A, int64_t ld, int64_t n, double *part, hipStream_t s,
                       Span sp) {
    basis_dots<TV>(nsys, A, ld, nullptr, n, part, s, sp);
}
template void launch_basis_dots<double>(int, const BasisArgs<double> &, int64_t, int64_t, double *, hipStream_t, Span);
template void launch_basis_dots<float>(int, const BasisArgs<float> &, int64_t, int64_t, double *, hipStream_t, Span);

void launch_copy_many(int count, const CopyArgs &A, hipStream_t s) {
    if (count < 1 || count > kCopyMax) throw std::runtime_error("launch_copy_many: 1 to 64 vectors");
    int64_t most = 0;
    for (int q = 0; q < count; ++q) most = std::max(most, A.n[q]);
    hipLaunchKernelGGL(k_copy_many, dim3(flat_grid(ceil_div(most, 4)).x, (unsigned)count), dim3(kThreads), 0, s, A);
}

template <class TI, class TO>
void launch_cast_b(int nr, const VPtr<const TI> &in, const VPtr<TO> &out, int64_t n, hipStream_t s, Span sp) {
    const dim3 grid(flat_grid(span_items(sp, n)).x, (unsigned)nr);
    hipLaunchKernelGGL((k_cast_b<TI, TO>), grid, dim3(kThreads), 0, s, in, out, n, sp.u, sp.n);
}
template void launch_cast_b<double, double>(int, const VPtr<const double> &, const VPtr<double> &, int64_t, hipStream_t, Span);
template void launch_cast_b<double, float>(int, const VPtr<const double> &, const VPtr<float> &, int64_t, hipStream_t, Span);
template void launch_cast_b<float, double>(int, const VPtr<const float> &, const VPtr<double> &, int64_t, hipStream_t, Span);
template void launch_cast_b<float, float>(int, const VPtr<const float> &, const VPtr<float> &, int64_t, hipStream_t, Span);

void launch_mdot(int nv, const double *V, int64_t ld, const double *w, const double *wt,
                 int64_t n, double *part, double *dout, hipStream_t s, Span sp) {
    launch_mdot_t<double>(nv, V, ld, w, wt, n, part, dout, s, sp);
}
void launch_mdot(int nv, const float *V, int64_t ld, const double *w, const double *wt, int64_t n, double *part,
                 double *dout, hipStream_t s, Span sp) {
    launch_mdot_t<float>(nv, V, ld, w, wt, n, part, dout, s, sp);
}

#define DM_NW_SWITCH(nw, CALL)                                   \
    switch (nw) {                                                \
        case 1: { constexpr int NW = 1, CH = 16; CALL; } break;  \
        case 2: { constexpr int NW = 2, CH = 8; CALL; } break;   \
        case 3: { constexpr int NW = 3, CH = 5; CALL; } break;   \
        case 4: { constexpr int NW = 4, CH = 4; CALL; } break;   \
        case 5: { constexpr int NW = 5, CH = 2; CALL; } break;   \
        case 6: { constexpr int NW = 6, CH = 2; CALL; } break;   \
        case 7: { constexpr int NW = 7, CH = 2; CALL; } break;   \
        default: { constexpr int NW = 8, CH = 2; CALL; } break;  \
    }

void launch_mdot_multi(int nv, const double *V, int64_t ld, const double *W, int64_t ldw, int nw,
                       const double *wt, int64_t n, double *part, double *dout, hipStream_t s, Span sp) {
    if (nv <= 0 || nw <= 0) return;
    if (nw > kMultiMax || nv * nw > 256) throw std::runtime_error("launch_mdot_multi: too many products");
    const bool v2 = vec2_ok(n, ld, {V, W, wt}) && (ldw % 2 == 0);
    const int nb = reduce_grid(span_items(sp, n) / (v2 ? 2 : 1));
    const dim3 g((unsigned)nb), b(kThreads);
    if (v2) DM_NW_SWITCH(nw, hipLaunchKernelGGL((k_mdot_multi<2, NW, CH>), g, b, 0, s, nv, V, ld, W, ldw, wt, n, part,
                                                sp))
    else DM_NW_SWITCH(nw, hipLaunchKernelGGL((k_mdot_multi<1, NW, CH>), g, b, 0, s, nv, V, ld, W, ldw, wt, n, part, sp))
    hipLaunchKernelGGL(k_mdot_final, dim3(nv * nw), dim3(kThreads), 0, s, nb, (const double *)part, dout);
}

void launch_maxpy_multi(int nv, const double *V, int64_t ld, const double *C, int nw, double *Y, int64_t ldy,
                        int64_t n, int overwrite, hipStream_t s, Span sp) {
    if (nw <= 0 || (nv <= 0 && !overwrite)) return;
    if (nw > kMultiMax || nv > 256) throw std::runtime_error("launch_maxpy_multi: too many vectors");
    const int64_t cnt = sp.u ? sp.n * kSpanUnit : n;
    if (vec2_ok(n, ld, {V, Y}) && ldy % 2 == 0)
        DM_NW_SWITCH(nw, hipLaunchKernelGGL((k_maxpy_multi<2, NW>), flat_grid(cnt / 2), dim3(kThreads), 0, s, nv, V,
                                            ld, C, Y, ldy, n, overwrite, sp))
    else
        DM_NW_SWITCH(nw, hipLaunchKernelGGL((k_maxpy_multi<1, NW>), flat_grid(cnt), dim3(kThreads), 0, s, nv, V, ld,
                                            C, Y, ldy, n, overwrite, sp))
}

#undef DM_NW_SWITCH

namespace {
template <class TV>
void launch_maxpy_t(int nv, const TV *V, int64_t ld, const double *c, double *y, int64_t n, int overwrite,
                    hipStream_t s, const double *cscale, Span sp) {
    if (nv <= 0 && !overwrite) return;
    if (nv > 256) throw std::runtime_error("launch_maxpy: more than 256 vectors");
    const int64_t cnt = sp.u ? sp.n * kSpanUnit : n;
    with_basis_width(n, ld, V, {y}, [&](auto width) {
        constexpr int W = decltype(width)::value;
        hipLaunchKernelGGL((k_maxpy<W, TV>), flat_grid(cnt / W), dim3(kThreads), 0, s, nv, V, ld, c, cscale,
                           (const double *)nullptr, 1.0, y, n, overwrite, sp);
    });
}
}  // namespace

void launch_maxpy(int nv, const double *V, int64_t ld, const double *c, double *y, int64_t n,
                  int overwrite, hipStream_t s, const double *cscale, Span sp) {
    launch_maxpy_t<double>(nv, V, ld, c, y, n, overwrite, s, cscale, sp);
}
void launch_maxpy(int nv, const float *V, int64_t ld, const double *c, double *y, int64_t n, int overwrite,
                  hipStream_t s, const double *cscale, Span sp) {
    launch_maxpy_t<float>(nv, V, ld, c, y, n, overwrite, s, cscale, sp);
}

void launch_maxpy_f32(int nv, const float *V, int64_t ld, const double *c, double *y, int64_t n, hipStream_t s,
                      Span sp) {
    if (nv <= 0) return;
    if (nv > 256) throw std::runtime_error("launch_maxpy_f32: more than 256 vectors");
    if ((ld & 1) || ((uintptr_t)V & 7) || ((uintptr_t)y & 15))
        throw std::runtime_error("launch_maxpy_f32: columns must be 8-byte and y 16-byte aligned, ld even");
    const int64_t cnt = sp.u ? sp.n * kSpanUnit : n;
    hipLaunchKernelGGL(k_maxpy_f32, flat_grid(cnt / 2), dim3(kThreads), 0, s, nv, V, ld, c, y, n, sp);
}

// Workgroups of a grid-stride reduction kernel: as many as are resident at
// once (its occupancy times the CUs), at most kReduceBlocks.  Every
// workgroup carries the same share of the work, so a grid beyond what is
// resident leaves a partial second round (1024 workgroups of a kernel with
// three resident per CU ran as 768 + 256).  Computed once per kernel.
template <auto KERN>
int reduce_blocks() {
    static const int nb = [] {
        int dev = 0, cus = 0, per = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, KERN, kThreads, 0) != hipSuccess || cus <= 0 ||
            per <= 0)
            return kReduceBlocks;
        return std::min(kReduceBlocks, cus * per);
    }();
    return nb;
}

namespace {
// the fused update of nsys systems, nv <= 32: the basis held in registers, or
// read twice where they do not fit
template <class TV>
void basis_update(int nsys, const BasisArgs<TV> &A, int64_t ld, int64_t n, double *part, hipStream_t s, Span sp) {
    int nv = 0;
    for (int q = 0; q < nsys; ++q) nv = std::max(nv, A.s[q].nv);
    const int rows = nv + 1;
    if (nv < 1 || nv > kBasisMax) throw std::runtime_error("basis update: 1 to 32 vectors");
    int width = 4, nb = 0;
    for (int q = 0; q < nsys; ++q)
        with_basis_width(n, ld, A.s[q].V, {A.s[q].w}, [&](auto w) { width = std::min(width, (int)decltype(w)::value); });
    auto fused = [&](auto kern, int most) {
        nb = reduce_grid(span_items(sp, n) / width, most);
        hipLaunchKernelGGL(kern, dim3((unsigned)nb, (unsigned)nsys), dim3(kThreads), 0, s, A, ld, n, part, rows, sp);
    };
    auto by_size = [&](auto w) {
        constexpr int W = decltype(w)::value;
        if (nv <= 8) fused(k_maxpy_mdot_norm<W, 8, false, TV>, reduce_blocks<k_maxpy_mdot_norm<W, 8, false, TV>>());
        else if (nv <= 16) fused(k_maxpy_mdot_norm<W, 16, false, TV>, reduce_blocks<k_maxpy_mdot_norm<W, 16, false, TV>>());
        else fused(k_maxpy_mdot_norm<W, 32, true, TV>, reduce_blocks<k_maxpy_mdot_norm<W, 32, true, TV>>());
    };
    if constexpr (sizeof(TV) == 4) {
        if (width == 4) by_size(std::integral_constant<int, 4>{});
    }
    if (width < 4 || sizeof(TV) == 8) {
        if (width >= 2) by_size(std::integral_constant<int, 2>{});
        else by_size(std::integral_constant<int, 1>{});
    }
    hipLaunchKernelGGL(k_basis_final<TV>, dim3((unsigned)rows, (unsigned)nsys), dim3(kThreads), 0, s, A, nb,
                       (const double *)part, rows, 1);
}

template <class TV>
void launch_maxpy_mdot_norm_t(int nv, const TV *V, int64_t ld, const double *c, double *w, int64_t n,
                              double *part, double *dout, hipStream_t s, const double *cscale, Span sp) {
    if (nv < 1 || nv + 1 > 256) throw std::runtime_error("launch_maxpy_mdot_norm: nv out of range");
    if (nv <= kBasisMax) {
        BasisArgs<TV> A{};
        A.s[0] = {V, w, c, cscale, dout, nv};
        basis_update<TV>(1, A, ld, n, part, s, sp);
        return;
    }
    // too many vectors to hold in registers: update w, then a second pass for
    // the dots (the basis is read twice)
    const dim3 b(kThreads);
    with_basis_width(n, ld, V, {w}, [&](auto width) {
        constexpr int W = decltype(width)::value;
        launch_maxpy_t<TV>(nv, V, ld, c, w, n, 0, s, cscale, sp);
        hipLaunchKernelGGL((k_mdot_norm<W, TV>), dim3(kReduceBlocks), b, 0, s, nv, V, ld, (const double *)w, n, part, sp);
    });
    hipLaunchKernelGGL(k_mdot_final, dim3(nv + 1), dim3(kThreads), 0, s, (int)kReduceBlocks, (const double *)part, dout);
}
}  // namespace

template <class TV>
void launch_basis_update(int nsys, const BasisArgs<TV> &A, int64_t ld, int64_t n, double *part, hipStream_t s,
                         Span sp) {
    basis_update<TV>(nsys, A, ld, n, part, s, sp);
}
template void launch_basis_update<double>(int, const BasisArgs<double> &, int64_t, int64_t, double *, hipStream_t, Span);
template void launch_basis_update<float>(int, const BasisArgs<float> &, int64_t, int64_t, double *, hipStream_t, Span);

void launch_maxpy_mdot_norm(int nv, const double *V, int64_t ld, const double *c, double *w,
                            int64_t n, double *part, double *dout, hipStream_t s, const double *cscale,
                            Span sp) {
    launch_maxpy_mdot_norm_t<double>(nv, V, ld, c, w, n, part, dout, s, cscale, sp);
}
void launch_maxpy_mdot_norm(int nv, const float *V, int64_t ld, const double *c, double *w, int64_t n,
                            double *part, double *dout, hipStream_t s, const double *cscale, Span sp) {
    launch_maxpy_mdot_norm_t<float>(nv, V, ld, c, w, n, part, dout, s, cscale, sp);
}

void launch_maxpy_scale(int nv, const double *V, int64_t ld, const double *c, const double *w,
                        double scale, double *out, int64_t n, hipStream_t s) {
    if (nv < 0 || nv > 256) throw std::runtime_error("launch_maxpy_scale: nv out of range");
    if (vec2_ok(n, ld, {V, w, out}))
        hipLaunchKernelGGL(k_maxpy<2>, flat_grid(n / 2), dim3(kThreads), 0, s, nv, V, ld, c,
                           (const double *)nullptr, w, scale, out, n, 0, Span{});
    else
        hipLaunchKernelGGL(k_maxpy<1>, flat_grid(n), dim3(kThreads), 0, s, nv, V, ld, c,
                           (const double *)nullptr, w, scale, out, n, 0, Span{});
}

namespace {
// the partial sums of launch_dot_pairs and launch_cg_dot; returns the number
// of workgroups
int dot_pairs_part(int nr, const VPtr<const double> &X, const VPtr<const double> &Y, const double *wt, int64_t n,
                   double *part, hipStream_t s, Span sp) {
    if (nr < 1 || nr > kMaxRhs) throw std::runtime_error("dot pairs: 1 to 4 pairs");
    VPtr<const double> x{}, y{};
    for (int q = 0; q < nr; ++q) {
        x.p[q] = X.p[q];
        y.p[q] = X.p[q] ? Y.p[q] : nullptr;
    }
    bool v2 = vec2_ok(n, 0, {wt});
    for (int q = 0; q < nr; ++q) v2 = v2 && vec2_ok(n, 0, {x.p[q], y.p[q]});
    const int nb = reduce_grid(span_items(sp, n) / (v2 ? 2 : 1));
    if (v2) hipLaunchKernelGGL(k_dot_pairs<2>, dim3(nb), dim3(kThreads), 0, s, x, y, wt, n, part, sp);
    else hipLaunchKernelGGL(k_dot_pairs<1>, dim3(nb), dim3(kThreads), 0, s, x, y, wt, n, part, sp);
    return nb;
}
}  // namespace

void launch_dot_pairs(int nr, const VPtr<const double> &X, const VPtr<const double> &Y, const double *wt,
                      int64_t n, double *part, double *dout, int64_t dstride, hipStream_t s, Span sp) {
    const int nb = dot_pairs_part(nr, X, Y, wt, n, part, s, sp);
    hipLaunchKernelGGL(k_mdot_final_strided, dim3(nr), dim3(kThreads), 0, s, nb, (const double *)part, dout, dstride);
}

void launch_cg_dot(int nr, const VPtr<const double> &X, const VPtr<const double> &Y, const double *wt, int64_t n,
                   double *part, CgStep step, CgState *st, hipStream_t s, Span sp) {
    const int nb = dot_pairs_part(nr, X, Y, wt, n, part, s, sp);
    hipLaunchKernelGGL(k_cg_final, dim3(nr), dim3(kThreads), 0, s, step, nb, (const double *)part, st);
}

void launch_cg_update(int nr, const VPtr<const double> &Pv, const VPtr<const double> &Qv, const VPtr<double> &Psi,
                      const VPtr<double> &R, const double *wt, int64_t n, double *part, CgState *st, hipStream_t s,
                      Span sp) {
    if (nr < 1 || nr > kMaxRhs) throw std::runtime_error("launch_cg_update: 1 to 4 vectors");
    const int nb = reduce_grid(span_items(sp, n));
    hipLaunchKernelGGL(k_cg_update, dim3(nb), dim3(kThreads), 0, s, nr, Pv, Qv, Psi, R, wt, n, part,
                       (const CgState *)st, sp);
    hipLaunchKernelGGL(k_cg_final, dim3(nr), dim3(kThreads), 0, s, kCgCheck, nb, (const double *)part, st);
}

void launch_cg_xpby(int nr, const VPtr<const double> &X, const VPtr<double> &Y, int64_t n, const CgState *st,
                    hipStream_t s, Span sp) {
    hipLaunchKernelGGL(k_cg_xpby, flat_grid(span_items(sp, n)), dim3(kThreads), 0, s, nr, X, Y, n, st, sp);
}

void launch_sub_masked_b(int nr, int64_t n, const double *mask, const double *val, int64_t stride, double scale,
                         const VPtr<double> &X, hipStream_t s) {
    VPtr<double> x{};
    for (int q = 0; q < nr && q < kMaxRhs; ++q) x.p[q] = X.p[q];
    hipLaunchKernelGGL(k_sub_masked_b, flat_grid(n), dim3(kThreads), 0, s, n, mask, val, stride, scale, x);
}

void launch_sub_masked(int64_t n, const double *mask, const double *val, double scale, double *x,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_sub_masked, flat_grid(n), dim3(kThreads), 0, s, n, mask, val, scale, x);
}

void launch_mask_mul(int64_t n, const double *mask, double *x, hipStream_t s) {
    hipLaunchKernelGGL(k_mask_mul, flat_grid(n), dim3(kThreads), 0, s, n, mask, x);
}

void launch_randn(int64_t n, uint64_t seed, int64_t offset, const double *mask, double *x,
                  hipStream_t s) {
    hipLaunchKernelGGL(k_randn, flat_grid(n), dim3(kThreads), 0, s, n, seed, offset, mask, x);
}

void launch_sample_e(const Grid &g, const double *coef, const double *b, double k, int npts, const double *pts,
                     double *out, hipStream_t s) {
    if (npts <= 0) return;
    hipLaunchKernelGGL(k_sample_e, dim3((unsigned)ceil_div(npts, kThreads)), dim3(kThreads), 0, s, g,
                       coefs_of(coef, g.P), b, 1.0 / (k * g.h), npts, pts, out);
}

void launch_copy_masked(int64_t n, const double *in, const double *mask, double *x, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_masked, flat_grid(n), dim3(kThreads), 0, s, n, in, mask, x);
}

template <class T>
void launch_scale_a(int64_t n, const T *coef, int power, T *x, hipStream_t s) {
    hipLaunchKernelGGL((k_scale_a<T>), flat_grid(n), dim3(kThreads), 0, s, n, coef, power, x);
}
template <class T>
void launch_add_scaled_a(int64_t n, const T *coef, const T *r, T *x, hipStream_t s) {
    hipLaunchKernelGGL((k_add_scaled_a<T>), flat_grid(n), dim3(kThreads), 0, s, n, coef, r, x);
}
template void launch_scale_a<double>(int64_t, const double *, int, double *, hipStream_t);
template void launch_scale_a<float>(int64_t, const float *, int, float *, hipStream_t);
template void launch_add_scaled_a<double>(int64_t, const double *, const double *, double *, hipStream_t);
template void launch_add_scaled_a<float>(int64_t, const float *, const float *, float *, hipStream_t);

// explicit instantiations
#define DM_BLOCK_INST(T)                                                                                   \
    template void launch_apply_b<T>(const Grid &, T, int, int, const VPtr<const T> &,                            \
                                    const VPtr<const T> &, const VPtr<T> &, hipStream_t, const ClassList &);      \
    template void launch_smooth_b<T>(const Grid &, T, int, int, const VPtr<const T> &, const VPtr<T> &,          \
                                     hipStream_t, const ClassList &);                                             \
    template void launch_sweeps_lds<T>(const Grid &, T, const LdsRows &, int, int, int, int,                     \
                                       const VPtr<const T> &, const VPtr<T> &, hipStream_t);                      \
    template void launch_restrict_b<T>(const Grid &, const Grid &, const T *, int, const VPtr<const T> &,        \
                                       const VPtr<T> &, hipStream_t, const VPtr<T> &, const int32_t *, int64_t);                                             \
    template void launch_prolong_add_b<T>(const Grid &, const Grid &, const T *, const T *, int,                 \
                                          const VPtr<const T> &, const VPtr<T> &, hipStream_t, const int32_t *,   \
                                          int64_t);                   \
    template void launch_coarse_solve_b<T>(int, const double *, const int64_t *, int, const VPtr<const T> &,     \
                                           const VPtr<T> &, hipStream_t);
DM_BLOCK_INST(double)
DM_BLOCK_INST(float)
#undef DM_BLOCK_INST
template void launch_apply<double>(const Grid &, double, int, const double *, const double *, double *, hipStream_t,
                                   const ClassList &);
template void launch_apply<float>(const Grid &, float, int, const float *, const float *, float *, hipStream_t,
                                  const ClassList &);
template void launch_apply_K<double>(const Grid &, const double *, const double *, double *, hipStream_t);
template void launch_apply_K<float>(const Grid &, const float *, const float *, float *, hipStream_t);
template void launch_apply_A_t<float>(const Grid &, const float *, const float *, float *, hipStream_t);
template void launch_apply_A_t<double>(const Grid &, const double *, const double *, double *, hipStream_t);
template void launch_smooth<double>(const Grid &, double, int, const double *, double *, hipStream_t,
                                    const ClassList &);
template void launch_smooth<float>(const Grid &, float, int, const float *, float *, hipStream_t, const ClassList &);
template void launch_restrict<double>(const Grid &, const Grid &, const double *, const double *,
                                      double *, hipStream_t);
template void launch_restrict<float>(const Grid &, const Grid &, const float *, const float *,
                                     float *, hipStream_t);
template void launch_prolong_add<double>(const Grid &, const Grid &, const double *, const double *, const double *,
                                         double *, hipStream_t);
template void launch_prolong_add<float>(const Grid &, const Grid &, const float *, const float *, const float *,
                                        float *, hipStream_t);
template void launch_cast<double, float>(const double *, float *, int64_t, hipStream_t, Span);
template void launch_cast<float, double>(const float *, double *, int64_t, hipStream_t, Span);
template void launch_cast<float, float>(const float *, float *, int64_t, hipStream_t, Span);
template void launch_coarse_solve<double>(int, const double *, const int64_t *, const double *,
                                          double *, hipStream_t);
template void launch_coarse_solve<float>(int, const double *, const int64_t *, const float *,
                                         float *, hipStream_t);

}  // namespace dm
