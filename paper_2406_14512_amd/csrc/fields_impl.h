// Flux function and mask kernel, and the force-free node correction,
// templated on the working precision R.  Included (through fields_fused.h)
// by k_fields64.hip (compiled without FP contraction, so the FP64 path
// rounds every product and sum as written) and by k_fields32.hip.
//
// Field arrays are node-shaped, theta fastest (see include/ffpic.h).
#pragma once

#include <type_traits>

#include "device_common.h"
#include "math64.h"

namespace ffpic {

// ---------------------------------------------------------------------------
// eq. (psi): Psi(i, 0) = 0, Psi(i, j+1) = Psi(i, j) + B_r(i, j+1/2) A_r(i, j)
// with A_r = r_i^2 (cos theta_j - cos theta_{j+1}); FP64, sequential in j so
// that the rounding is fixed.  A workgroup takes ROWS radial rows and walks
// them in tiles of kPsiCols columns, in a pipeline over two tiles in LDS: one
// wave runs the serial sums of a tile, a row per lane, while four others write
// the tile before it back, coalesced, with the blending function f at its nodes
// (eq. transition, four thresholds) and the kill flag of each cell whose four
// corners have f = 1, and form the terms B_r A_r of the tile after it (each
// product rounded as in the serial form) from loads a step ahead.  A cell needs
// the row above it, so the blocks overlap by one row, which the next block
// writes.
//
// What bounds it: the serial sums, 3.5 us a tile, and beside them the
// write-back of the other rows, so a CU wants one workgroup with as many rows
// as the sums hide.  Mask phase of a step, us, against all waves summing,
// writing and loading in turn, in steps of fields alone: 300 x 517 FP32
// 14.2 -> 12.4, 1024^2 23.6 -> 19.8, 1500 x 3000 61 -> 46, 2048^2 50 -> 38 (FP64
// 53 -> 40), 4096^2 118 -> 84 (FP64 124 -> 119), 16 systems grouped 88 -> 63; a
// single tile, where nothing overlaps, as before (128^2 7.1).  After a push of
// 4e8 particles, which leaves none of B_r in the caches, 4096^2 takes 103 to
// 111 (FP64 120).
constexpr int kPsiCols = 256;
constexpr int kPsiThreads = kPsiCols + 64;   // one per column, and the summing wave
constexpr int kPsiRun = 32;     // terms a lane sums between LDS reads

// workgroup barrier that orders LDS accesses only: unlike __syncthreads it
// does not wait for the thread's global loads and stores, so the next
// tile's loads and the write-back stay in flight across it
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// the arguments of one system's flux function and mask
template <typename R>
struct PsiJob {
    int nr, nth, ld, ff;
    int blocks;                // workgroups of ROWS rows, ROWS - 1 apart
    const double *rn2, *dcn;   // r_i^2, cos theta_j - cos theta_{j+1}
    double t0, t1, t2, t3;
    const R *br;
    double *psi;
    R *f;
    uint8_t *kill;
};

constexpr int kPsiGroupRows = 16;   // 16 systems: 63 us, with 12 rows 77, with 8 91
// Rows of a block: the fewest that give each CU at most one block (a second on
// some of them costs more than longer blocks on all: 1024^2 25.2 us with 4 rows
// and 342 blocks, 19.1 with 6 and 205; 2048^2 FP64 50 with 8 and 293, 40 with
// 12 and 187; 1281 x 300 11.5 with 8, 13.6 with 12).  Larger grids have several
// blocks per CU in any case: in FP32 12 rows (4096^2 84 us, with 8 116, with 16
// 146), in FP64 8 (3000 x 1500 41 us, with 12 46 to 56, though 4096^2 119 and
// 100 to 120).
inline int psi_rows(int nr, bool fp64) {
    for (int rows : {4, 6, 8, 12})
        if (nr <= 256 * (rows - 1)) return rows;
    return fp64 ? 8 : 12;
}

template <int ROWS>
struct PsiSmem {
    double tile[2][ROWS][kPsiCols + 1];
    uint32_t one[kPsiCols + 1];   // per column, bit rr: f = 1 in row rr
};

// rows [bx * (ROWS - 1), ...) of one system; every thread of the workgroup
// calls it and returns from it together
template <typename R, int ROWS>
__device__ __forceinline__ void psi_block(const PsiJob<R> &P, int bx, PsiSmem<ROWS> &L) {
    constexpr int OWN = ROWS - 1;   // rows a block writes (the last: all of its own)
    const int t = threadIdx.x;
    const int i0 = bx * OWN;
    const int ld = P.ld, nr = P.nr, nth = P.nth;
    const int rows = min(ROWS, nr + 1 - i0);
    const int own = i0 + OWN < nr ? OWN : rows;   // rows written
    const int cells = min(own, nr - i0);          // rows of cells
    const int ntile = (nth + kPsiCols - 1) / kPsiCols;
    auto width = [&](int k) { return min(kPsiCols, nth - k * kPsiCols); };

    if (t >= kPsiCols) {
        // the summing wave, one row per lane: the sums of tile k while the
        // other waves write tile k - 1 back and form the terms of tile k + 1;
        // in blocks of kPsiRun terms (all reads, then the serial sums in
        // registers, then all writes), so that the chain of additions waits
        // for LDS once per block rather than every few terms
        const int lane = t - kPsiCols;
        double acc = 0.0;
        auto sum = [&](double *row, int k, int end) {
            if (lane >= rows) return;
            for (; k + kPsiRun <= end; k += kPsiRun) {
                double v[kPsiRun];
#pragma unroll
                for (int u = 0; u < kPsiRun; u++) v[u] = row[k + u];
#pragma unroll
                for (int u = 0; u < kPsiRun; u++) {
#pragma clang fp contract(off)
                    acc = acc + v[u];
                    v[u] = acc;
                }
#pragma unroll
                for (int u = 0; u < kPsiRun; u++) row[k + u] = v[u];
            }
            for (; k < end; k++) {
#pragma clang fp contract(off)
                acc = acc + row[k];
                row[k] = acc;
            }
        };
        lds_barrier();
        if (ntile == 1) {
            sum(L.tile[0][min(lane, ROWS - 1)], 0, width(0));
            lds_barrier();
            lds_barrier();
            return;
        }
        for (int k = 0; k <= ntile; k++) {
            const int w = k < ntile ? width(k) : 0, half = min(w, kPsiCols / 2);
            double *row = L.tile[k & 1][min(lane, ROWS - 1)];
            sum(row, 0, half);
            lds_barrier();
            sum(row, half, w);
            lds_barrier();
        }
        return;
    }

    const R *__restrict__ br = P.br;
    double *__restrict__ psi = P.psi;
    R *__restrict__ f = P.f;
    uint8_t *__restrict__ kill = P.kill;
    auto fval = [&](double v) { return P.ff ? blend(v, P.t0, P.t1, P.t2, P.t3) : 0.0; };
    // the column before the first tile: Psi = 0 on the axis
    const double f0 = fval(0.0);
    uint32_t last = f0 == 1.0 ? ~0u : 0u;
    double r2[ROWS];
#pragma unroll
    for (int rr = 0; rr < ROWS; rr++) r2[rr] = P.rn2[i0 + min(rr, rows - 1)];
    if (t < own) {
        psi[ix(ld, i0 + t, 0)] = 0.0;
        f[ix(ld, i0 + t, 0)] = (R)f0;
    }
    // B_r and column areas of a tile, in flight from one step of the loop to
    // the next.  Every lane loads every row: a lane past the last column or
    // row loads the last one's, whose terms nobody sums.
    R nxt[ROWS];
    double arn;
    auto load = [&](int k) {
        const int j = min(k * kPsiCols + t, nth - 1);
        arn = P.dcn[j];
#pragma unroll
        for (int rr = 0; rr < ROWS; rr++) nxt[rr] = br[ix(ld, i0 + min(rr, rows - 1), j)];
    };
    // the tile's terms B_r A_r, each product rounded as in the serial form
    auto terms = [&](int k) {
#pragma unroll
        for (int rr = 0; rr < ROWS; rr++) {
#pragma clang fp contract(off)
            L.tile[k & 1][rr][t] = (double)nxt[rr] * (r2[rr] * arn);
        }
    };
    // tile k back.  Every lane stores every row: a lane past the last column or
    // row stores the last one again (that entry's own value), so that with no
    // branch around the stores the compiler can count those still in flight,
    // and the wait for the next tile's loads does not also wait for this
    // write-back.
    auto write = [&](int k) {
        const auto &tile = L.tile[k & 1];
        const int j0 = k * kPsiCols, w = width(k), tc = min(t, w - 1);
        uint32_t one = 0;
        const double vl = tile[own - 1][tc];
        const R fl = (R)fval(vl);
#pragma unroll
        for (int rr = 0; rr < ROWS; rr++) {
            const double v = tile[rr][tc], fv = fval(v);
            one |= (fv == 1.0 ? 1u : 0u) << rr;
            const size_t at = ix(ld, i0 + min(rr, own - 1), j0 + 1 + tc);
            psi[at] = rr < own ? v : vl;
            f[at] = rr < own ? (R)fv : fl;
        }
        if (t == 0) L.one[0] = last;
        if (t < w) L.one[t + 1] = one;
    };
    // cells of its column: both columns' flags, and those of the row above
    auto flags = [&](int k) {
        const int j0 = k * kPsiCols, w = width(k), tc = min(t, w - 1);
        const uint32_t both = L.one[tc] & L.one[tc + 1], dead = both & (both >> 1);
        last = L.one[w];
#pragma unroll
        for (int rr = 0; rr < OWN; rr++) {
            const int rc = min(rr, cells - 1);
            kill[(size_t)(i0 + rc) * nth + j0 + tc] = (dead >> rc) & 1u;
        }
    };
    load(0);
    terms(0);
    if (ntile == 1) {   // nothing to overlap with
        lds_barrier();
        lds_barrier();
        write(0);
        lds_barrier();
        flags(0);
        return;
    }
    load(1);
    lds_barrier();
    lds_barrier();
    terms(1);
    load(2);
    lds_barrier();
    for (int k = 0; k < ntile; k++) {
        write(k);
        lds_barrier();
        if (k + 2 < ntile) terms(k + 2);
        load(k + 3);
        flags(k);
        lds_barrier();
    }
}

// (Two workgroups of five waves share a CU up to 128 registers.  FP32 with 12
// rows fits: 4096^2 84 us, 116 at 129 registers; FP64 would spill four: 2048^2
// 43 us against 40.)
template <typename R>
constexpr int kPsiWaves = std::is_same<R, float>::value ? 4 : 1;

template <typename R, int ROWS>
__global__ void __launch_bounds__(kPsiThreads, kPsiWaves<R>) k_psi(const PsiJob<R> P) {
    __shared__ PsiSmem<ROWS> L;
    psi_block<R, ROWS>(P, (int)blockIdx.x, L);
}

// The flux functions and masks of many systems in one launch of persistent
// workgroups taking row blocks from a counter (job k owns items
// [starts[k], starts[k + 1])).
template <typename R>
__global__ void __launch_bounds__(kPsiThreads) k_psi_group(const PsiJob<R> *__restrict__ jobs,
                                                        const int *__restrict__ starts,
                                                        int njobs, int *__restrict__ ctr) {
    __shared__ PsiSmem<kPsiGroupRows> L;
    __shared__ int next, job;
    __shared__ uint32_t stage[kJobWords];
    const int total = starts[njobs];
    if (threadIdx.x == 0) next = atomicAdd(&ctr[0], 1);
    __syncthreads();
    int item = __builtin_amdgcn_readfirstlane(next);
    while (item < total) {
        find_job(starts, njobs, item, &job);
        int nx = 0;                    // the next item, taken during this one
        if (threadIdx.x == 0) nx = atomicAdd(&ctr[0], 1);
        __syncthreads();
        const int lo = __builtin_amdgcn_readfirstlane(job);
        psi_block<R, kPsiGroupRows>(stage_uniform(jobs + lo, stage), item - starts[lo], L);
        if (threadIdx.x == 0) next = nx;
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(next);
    }
    group_done(ctr);
}

// force-free correction at a node: E.B projection then the |E| <= |B| cap
// (Sect. 3); B = 0 gives E = 0
__device__ __forceinline__ void ff_node(const double e[3], const double b[3], double o[3]) {
    const double b2 = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
    if (!(b2 > 0.0)) {
        o[0] = o[1] = o[2] = 0.0;
        return;
    }
    const double eb = e[0] * b[0] + e[1] * b[1] + e[2] * b[2];
    if (quot_ok(b2)) {
        const double y = rcp64(b2);
        for (int c = 0; c < 3; c++) o[c] = e[c] - quot(eb * b[c], b2, y);
    } else {
        for (int c = 0; c < 3; c++) o[c] = e[c] - eb * b[c] / b2;
    }
    const double e2 = o[0] * o[0] + o[1] * o[1] + o[2] * o[2];
    if (e2 >= b2 && e2 > 0.0) {
        const double s = sqrt(b2 / e2);
        for (int c = 0; c < 3; c++) o[c] = s * o[c];
    }
}

template <typename R>
PsiJob<R> psi_job(const ffpic_ctx *c, int rows) {
    PsiJob<R> P;
    P.nr = c->nr; P.nth = c->nth; P.ld = c->ld;
    P.ff = c->d.ff_enable ? 1 : 0;
    P.blocks = (c->nr + rows - 2) / (rows - 1);
    P.rn2 = c->dtab64[T_RN2];
    P.dcn = c->dtab64[T_DCN];
    P.br = (const R *)c->B[0];
    P.psi = c->psi;
    const double *t = c->d.psi_thr;
    P.t0 = t[0]; P.t1 = t[1]; P.t2 = t[2]; P.t3 = t[3];
    P.f = (R *)c->f;
    P.kill = c->kill;
    return P;
}

template <typename R>
static void run_psi_mask(ffpic_ctx *c) {
    const int rows = psi_rows(c->nr, std::is_same<R, double>::value);
    const PsiJob<R> P = psi_job<R>(c, rows);
    auto kern = rows == 4   ? k_psi<R, 4>
                : rows == 6 ? k_psi<R, 6>
                : rows == 8 ? k_psi<R, 8>
                            : k_psi<R, 12>;
    hipLaunchKernelGGL(kern, dim3(P.blocks), dim3(kPsiThreads), 0, c->stream, P);
    FFPIC_LAUNCH_CHECK();
}

}  // namespace ffpic
