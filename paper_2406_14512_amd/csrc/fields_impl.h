// Flux function and mask kernel, and the force-free node correction,
// templated on the working precision R.  Included (through fields_fused.h)
// by k_fields64.hip (compiled without FP contraction, so the FP64 path
// rounds every product and sum as written) and by k_fields32.hip.
//
// Field arrays are node-shaped, theta fastest (see include/ffpic.h).
#pragma once

#include "device_common.h"
#include "math64.h"

namespace ffpic {

// ---------------------------------------------------------------------------
// eq. (psi): Psi(i, 0) = 0, Psi(i, j+1) = Psi(i, j) + B_r(i, j+1/2) A_r(i, j)
// with A_r = r_i^2 (cos theta_j - cos theta_{j+1}); FP64, sequential in j so
// that the rounding is fixed.  A workgroup takes ROWS radial rows and
// walks them in tiles of kPsiCols columns: all 256 threads load a tile with
// coalesced reads along theta and form its terms B_r A_r in parallel (each
// product rounded as in the serial form) into LDS, then one lane per row
// runs the serial sum over the tile while the next tile's loads are in
// flight, and the tile of partial sums is written back coalesced, with the
// blending function f at its nodes (eq. transition, four thresholds) and the
// kill flag of each cell whose four corners have f = 1.  A cell needs the row
// above it, so the blocks overlap by one row, which the next block writes.
//
// Rows: few while the blocks do not fill the GPU, more where the overlap is
// traffic.  us with 4, 8 and 16 rows, and with 16 and the mask in a kernel of
// its own, which read Psi back:
//   128^2 FP64          5.4    6.5    9.1    11.7
//   300 x 517 FP32     12.8   15.7   23.5    18.9
//   1024^2 FP32        22.9   25.7           28.3
//   4096^2 FP32       153    116    128     130
//   16 systems        138    116     87      98    (one launch, 6e6 nodes)
constexpr int kPsiCols = 256;
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

constexpr int kPsiGroupRows = 16;
inline int psi_rows(int nr) { return nr < 2048 ? 4 : 8; }

template <int ROWS>
struct PsiSmem {
    double tile[ROWS][kPsiCols + 1];
    uint32_t one[kPsiCols + 1];   // per column, bit rr: f = 1 in row rr
};

// rows [bx * (ROWS - 1), ...) of one system; every thread of the workgroup
// calls it and returns from it together
template <typename R, int ROWS>
__device__ __forceinline__ void psi_block(const PsiJob<R> &P, int bx, PsiSmem<ROWS> &L) {
    constexpr int OWN = ROWS - 1;   // rows a block writes (the last: all of its own)
    auto &tile = L.tile;
    const int t = threadIdx.x;
    const int i0 = bx * OWN;
    const int ld = P.ld, nr = P.nr, nth = P.nth;
    const R *__restrict__ br = P.br;
    double *__restrict__ psi = P.psi;
    R *__restrict__ f = P.f;
    uint8_t *__restrict__ kill = P.kill;
    const int rows = min(ROWS, nr + 1 - i0);
    const int own = i0 + OWN < nr ? OWN : rows;   // rows written
    const int cells = min(own, nr - i0);                  // rows of cells
    auto fval = [&](double v) { return P.ff ? blend(v, P.t0, P.t1, P.t2, P.t3) : 0.0; };
    // the column before the tile: Psi = 0 on the axis
    const double f0 = fval(0.0);
    if (t == 0) L.one[0] = f0 == 1.0 ? ~0u : 0u;
    double r2[ROWS];
#pragma unroll
    for (int rr = 0; rr < ROWS; rr++) r2[rr] = rr < rows ? P.rn2[i0 + rr] : 0.0;
    double acc = 0.0;
    if (t < own) {
        psi[ix(ld, i0 + t, 0)] = 0.0;
        f[ix(ld, i0 + t, 0)] = (R)f0;
    }
    // The tile's B_r and column areas are loaded one tile ahead.
    R nxt[ROWS];
    double arn;
    auto load = [&](int jt) {
        arn = jt + t < nth ? P.dcn[jt + t] : 0.0;
#pragma unroll
        for (int rr = 0; rr < ROWS; rr++)
            nxt[rr] = (rr < rows && jt + t < nth) ? br[ix(ld, i0 + rr, jt + t)] : (R)0;
    };
    // the tile's terms B_r A_r, each product rounded as in the serial form
    auto terms = [&]() {
#pragma unroll
        for (int rr = 0; rr < ROWS; rr++) {
#pragma clang fp contract(off)
            tile[rr][t] = (double)nxt[rr] * (r2[rr] * arn);
        }
    };
    load(0);
    terms();
    for (int j0 = 0; j0 < nth; j0 += kPsiCols) {
        const int w = min(kPsiCols, nth - j0);
        lds_barrier();
        const int jn = j0 + kPsiCols;
        if (jn < nth) load(jn);
        if (t < rows) {
            // in blocks of kPsiRun terms: all reads, then the serial sums in
            // registers, then all writes, so that the chain of additions
            // waits for LDS once per block rather than every few terms
            double *__restrict__ row = tile[t];
            int k = 0;
            for (; k + kPsiRun <= w; k += kPsiRun) {
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
            for (; k < w; k++) {
#pragma clang fp contract(off)
                acc = acc + row[k];
                row[k] = acc;
            }
        }
        lds_barrier();
        // every lane stores every row: a lane past the last column or row
        // writes the last one instead (that entry's own value again), so
        // that with no branch around the stores the compiler can count those
        // still in flight, and the wait for the next tile's loads does not
        // also wait for this write-back
        const int tc = min(t, w - 1);
        uint32_t one = 0;
#pragma unroll
        for (int rr = 0; rr < ROWS; rr++) {
            const double v = tile[rr][tc], fv = fval(v);
            one |= (fv == 1.0 ? 1u : 0u) << rr;
            const size_t k = ix(ld, i0 + min(rr, own - 1), j0 + 1 + tc);
            const double vw = rr < own ? v : tile[own - 1][tc];
            psi[k] = vw;
            f[k] = (R)(rr < own ? fv : fval(vw));
        }
        if (t < w) L.one[t + 1] = one;
        lds_barrier();
        // cells of column j0 + t: both columns' flags, and those of the row above
        const uint32_t both = L.one[tc] & L.one[tc + 1], dead = both & (both >> 1);
        const uint32_t last = L.one[w];
#pragma unroll
        for (int rr = 0; rr < OWN; rr++)
            if (t < w && rr < cells) kill[(size_t)(i0 + rr) * nth + j0 + t] = (dead >> rr) & 1u;
        lds_barrier();
        if (t == 0) L.one[0] = last;
        if (jn < nth) terms();
    }
}

template <typename R, int ROWS>
__global__ void __launch_bounds__(kPsiCols) k_psi(const PsiJob<R> P) {
    __shared__ PsiSmem<ROWS> L;
    psi_block<R, ROWS>(P, (int)blockIdx.x, L);
}

// The flux functions and masks of many systems in one launch of persistent
// workgroups taking row blocks from a counter (job k owns items
// [starts[k], starts[k + 1])).
template <typename R>
__global__ void __launch_bounds__(kPsiCols) k_psi_group(const PsiJob<R> *__restrict__ jobs,
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
    const int rows = psi_rows(c->nr);
    const PsiJob<R> P = psi_job<R>(c, rows);
    auto kern = rows == 4 ? k_psi<R, 4> : k_psi<R, 8>;
    hipLaunchKernelGGL(kern, dim3(P.blocks), dim3(kPsiCols), 0, c->stream, P);
    FFPIC_LAUNCH_CHECK();
}

}  // namespace ffpic
