// The whole field step of Sect. 3 in one kernel: Faraday half step
// (eq. faraday, Stokes form on the primal faces), the force-free drift
// current at nodes (eq. JFFE: rho E x B / B^2 with rho = div E / 4 pi, from
// E^n and B^{n+1/2}), the blend of eq. (blending) at the staggered points
// (f averaged from the adjacent nodes) inside Ampere's law (eq. ampere, on
// the dual faces), the force-free E correction at nodes (E.B projected out,
// |E| capped at |B|, weighted by f) averaged back to the staggered points,
// the second Faraday half step, the absorbing layer of Sect. 4, and the
// totals the particle gather reads.  Corotation on the star: E_th and E_ph
// of row 0 are never updated; axis: E_ph = B_th = 0 on j = 0, nth.
//
// This file's kernel is the FP64 step, which evolves E and B.  The FP32
// step (fields_fused32.h, same stages and tiling) is a perturbation form.  In FP32 the
// static magnetosphere itself is the problem: the corotation E and the
// dipole B are discretely curl-free (or nearly so) in exact arithmetic, but
// once each component is rounded to FP32 their discrete curls are
// O(1e-7 |F| / cell) noise, which the Yee update would integrate into B_phi
// and E_phi every step.  So the FP32 state is dF = F - F0 about an FP64
// background F0 (the initial fields), whose discrete curls (the background
// rates) and charge density are evaluated once in FP64 on the host:
//   dB <- dB - h curl(dE) + h rateB0        (rateB0 = -curl E0)
//   dE <- dE + dt (curl(dB) + rateE0) - 4 pi dt J
//   rho = div(dE) / 4 pi + rho0
// Rounding then acts on the small perturbation, not on the background; the
// node quantities (J_FFE, the correction) use the totals F0 + dF, which the
// FP32 step also writes for the particle gather.
//
// Tiling.  A workgroup owns a strip of theta columns (plus kFzL halo columns
// before and kFzR after, one thread per column) and a slab of
// `rows` radial rows, and marches through the slab row by row, keeping the
// recent rows of each stage in registers (its own column) and in small
// LDS rings (the theta neighbours).  At iteration q it loads row q and
// computes
//   Faraday half step B^{n+1/2}    row q-1   (needs E^n rows q-1, q)
//   node J_FFE                     row q-1   (E^n rows q-2, q-1; B^{n+1/2} rows q-2, q-1)
//   Ampere E^{n+1}                 row q-2   (B^{n+1/2} rows q-3, q-2; J_FFE rows q-2, q-1)
//   node correction delta          row q-2   (E rows q-3, q-2; B^{n+1/2} rows q-3, q-2)
//   delta averaged back            row q-3   (delta rows q-3, q-2)
//   Faraday half step B^{n+1},     row q-4   (E rows q-4, q-3)
//   absorber, stores
// so each slab reads 2 rows above and 4 below its own, and every node is
// loaded and stored once.  Three workgroup barriers per row order the LDS
// exchanges.  Neighbouring slabs read each other's rows as halo, so the
// state is double-buffered (read one buffer, write the other), and so are
// the deposit accumulators: this step reads the push's and clears the
// other set for the next push.
//
// What bounds it.  A row is a serial chain of about 580 vector instructions
// per wave, and registers and LDS allow two workgroups per CU, so nothing
// else hides the latency of its loads: row q + 1 is therefore in flight while
// row q is worked on, the barriers wait for LDS alone, and the row's geometry
// comes through the scalar cache.  With the divisions by products of geometry
// factors taken as products of stored reciprocals, corrected to the rounded
// quotient, the FP64 step with the force-free stages went from 380 to 206 us
// at 2048^2, from 138 to 77 us at 1024^2; the reciprocals without the loads
// ahead gave 362 and 119 us.  With strips of 128 threads (fused_threads64)
// 194 and 72 us (152 B per node: 3.3 TB/s at 2048^2).
#pragma once

#include <algorithm>
#include <utility>

#include "fields_impl.h"

namespace ffpic {

constexpr int kFzT = 256;                 // threads = columns of a strip with its halo
constexpr int kFzL = 2, kFzR = 4;         // halo columns before and after
constexpr int kFzW = kFzT - kFzL - kFzR;  // owned columns per strip

// Geometry of one row as the stages read it, in one block of scalar loads: the
// factors and the reciprocals of those that are divided by (index 0 of the
// first differences and index nr of the half-cell ones are unused).
struct FusedRow {
    // primal: r_i, r_{i+1}, their difference, r_i^2 and (r_{i+1}^2 - r_i^2) / 2
    double rn, rn1, drn, rn2, y_rn2, dr2n, y_dr2n, pad;
    // dual: r_{i+1/2}, r_{i-1/2}, their difference, squares, and the dual
    // cell's area and volume factors
    double rh, rhm, drh, rh2, y_rh2, dr2h, y_dr2h, rh2m, dr3h, y_dr3h;
    double lamn, lamh;   // absorber factors at r_i and r_{i+1/2}
};

typedef const __attribute__((address_space(4))) FusedRow *RowPtr;

struct FusedArgs {
    using R = double;
    Geo<R> g;
    const FusedRow *row;       // [nr+1]
    R h;                       // half time step
    int rows;                  // owned rows per workgroup
    int absorb0;               // first row whose absorber factor is below 1
    const R *sE[3], *sB[3];    // state in: E, B
    R *oE[3], *oB[3];          // state out (the other buffer)
    const R *B0[3];            // initial B (the absorber relaxes B to it)
    const R *J[3];             // this step's deposit accumulators
    R *Jz[3];                  // the other accumulators, cleared here
    const R *f;                // blending function at nodes
};

// force-free correction at a node in FP32 (E.B projection, then
// |E| <= |B|), with the hardware reciprocal and square roots (about 1 ulp)
// in place of the divisions; B = 0 gives E = 0
__device__ __forceinline__ void ff_node_f(const float e[3], const float b[3], float o[3]) {
    const float b2 = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
    if (!(b2 > 0.f)) { o[0] = o[1] = o[2] = 0.f; return; }
    const float ib2 = __builtin_amdgcn_rcpf(b2);
    const float eb = (e[0] * b[0] + e[1] * b[1] + e[2] * b[2]) * ib2;
    for (int c = 0; c < 3; c++) o[c] = e[c] - eb * b[c];
    const float e2 = o[0] * o[0] + o[1] * o[1] + o[2] * o[2];
    if (e2 >= b2 && e2 > 0.f) {
        const float s = __builtin_amdgcn_sqrtf(b2) * __builtin_amdgcn_rsqf(e2);
        for (int c = 0; c < 3; c++) o[c] = s * o[c];
    }
}

template <bool FF, int T>
__global__ void __launch_bounds__(T) k_field_fused(const FusedArgs A) {
    constexpr int W = T - kFzL - kFzR;   // owned columns
    using R = double;
    const Geo<R> &g = A.g;
    const int nr = g.nr, nth = g.nth, ld = g.ld;
    const int t = threadIdx.x;
    const int j = (int)blockIdx.x * W + t - kFzL;
    const bool colok = j >= 0 && j <= nth;
    const int jc = min(max(j, 0), nth);
    const int tl = t > 0 ? t - 1 : t, tr = t < T - 1 ? t + 1 : t;
    const int i0 = (int)blockIdx.y * A.rows;
    const int iL = min(i0 + A.rows - 1, nr);
    const int qs = max(i0 - 2, 0);
    const R dt = g.dt, h = A.h, dth = g.dth;
    const R fourpi = (R)(4.0 * kPi);
    // column geometry (indices clamped; used only where the stage's
    // condition on j holds)
    // the row blocks are read through the constant address space: scalar
    // loads, which wait neither for the next row nor for the stores
    const RowPtr row = (RowPtr)A.row;
    const bool jlt = j < nth, jgt = j > 0, jin = j > 0 && j < nth;
    const R sn_j = g.sn[jc], sn_j1 = g.sn[min(jc + 1, nth)];
    const R sh_j = g.sh[min(jc, nth - 1)], sh_jm = g.sh[max(jc - 1, 0)];
    const R dcn_j = g.dcn[min(jc, nth - 1)], dcd_j = g.dcd[jc], dthd_j = g.dthd[jc];
    // reciprocals of the factors that the stages divide by
    const R y_sn = rcp64(sn_j), y_sh = rcp64(sh_j), y_dcn = rcp64(dcn_j), y_dcd = rcp64(dcd_j),
            y_dthd = rcp64(dthd_j), y_dth = rcp64(dth), y_dt = rcp64(dt);

    // LDS rings (theta neighbours); a ring slot holds one row of one quantity
    __shared__ R lE[2][3][T];          // E^n: r, phi, theta
    __shared__ R lB[4][2][T];          // B^{n+1/2}: r, phi
    __shared__ R lN[FF ? 2 : 1][T];    // J_FFE theta
    __shared__ R lF[FF ? 3 : 1][T];    // f
    __shared__ R lEa[FF ? 2 : 1][T];   // E after Ampere, theta
    __shared__ R lD[FF ? 2 : 1][T];    // delta theta
    __shared__ R lEf[2][2][T];         // final E: r, phi

    // own-column history (suffix = rows back from the newest loaded row q)
    R sE0[3] = {}, sE1[3] = {}, sE2[3] = {};        // E state rows q, q-1, q-2
    R sB0[3] = {}, sB1[3] = {};                     // B state rows q, q-1
    R f0 = 0, f1 = 0, f2 = 0;                       // f rows q, q-1, q-2
    R J0[3] = {}, J1[3] = {}, J2[3] = {};           // deposit rows q, q-1, q-2
    R Bh1[3] = {}, Bh2[3] = {}, Bh3[3] = {}, Bh4[3] = {};   // B^{n+1/2} rows q-1..q-4
    R n01 = 0, n02 = 0, n11 = 0, n12 = 0, n21 = 0, n22 = 0;   // J_FFE rows q-1, q-2
    R Ea2[3] = {}, Ea3[3] = {};                     // E after Ampere (state) rows q-2, q-3
    R Eat3r = 0;                                    // its E_r, row q-3
    R d02 = 0, d03 = 0, d13 = 0, d23 = 0;           // delta rows q-2, q-3
    R d12 = 0, d22 = 0;
    R Ef3[3] = {}, Ef4[3] = {};                     // final E (state) rows q-3, q-4

    // row q is loaded one iteration ahead.  Columns outside the grid load the
    // nearest one: no stage of an owned column uses their values.
    R nE[3], nB[3], nJ[3], nf = 0;
    auto load = [&](int row) {
        const size_t k0 = ix(ld, row, 0);
        const unsigned jk = jc;
#pragma unroll
        for (int c = 0; c < 3; c++) {
            nE[c] = (A.sE[c] + k0)[jk];
            nB[c] = (A.sB[c] + k0)[jk];
            nJ[c] = (A.J[c] + k0)[jk];
        }
        if constexpr (FF) nf = (A.f + k0)[jk];
    };
    load(qs);
    for (int q = qs; q <= iL + 4; q++) {
        // ---- row q; past the last row (which only drains the stages) the
        // last row again, so that the loads are the same in every iteration
        // and nothing but the next one waits for them
#pragma unroll
        for (int c = 0; c < 3; c++) {
            sE0[c] = nE[c];
            sB0[c] = nB[c];
            J0[c] = nJ[c];
        }
        f0 = nf;
        const int fr = q - 4;   // the row stored by this iteration
        const bool damp = fr >= A.absorb0 && fr >= i0 && fr <= iL;
        R b0[3];
        if (damp) {
#pragma unroll
            for (int c = 0; c < 3; c++) b0[c] = (A.B0[c] + ix(ld, fr, 0))[(unsigned)jc];
        }
        load(min(q + 1, nr));
        lE[q & 1][0][t] = sE0[0];
        lE[q & 1][1][t] = sE0[2];
        lE[q & 1][2][t] = sE0[1];
        if constexpr (FF) lF[q % 3][t] = f0;

        // ---- Faraday half step, row a = q - 1: B^{n+1/2}
        const int a = q - 1;
        if (a >= qs && a <= nr) {
            const auto &Ra = row[a];
            const R *nb = lE[a & 1][0];   // row a, E state r at j+1 is nb[tr]
            const R epn = lE[a & 1][1][tr];
            const R ern = nb[tr];
            R v[3];
            // B_r (j < nth)
            {
                R circ = Ra.rn * (sn_j1 * epn - sn_j * sE1[2]);
                v[0] = sB1[0] - quot(h * circ, Ra.rn2 * dcn_j, Ra.y_rn2 * y_dcn);
                if (!jlt) v[0] = sB1[0];
            }
            if (a < nr) {
                if (jin) {
                    R circ = sn_j * (Ra.rn1 * sE0[2] - Ra.rn * sE1[2]);
                    v[1] = sB1[1] + quot(h * circ, sn_j * Ra.dr2n, y_sn * Ra.y_dr2n);
                } else {
                    v[1] = (R)0;
                }
                if (jlt) {
                    R circ = dth * (Ra.rn1 * sE0[1] - Ra.rn * sE1[1]) - Ra.drn * (ern - sE1[0]);
                    v[2] = sB1[2] - quot(h * circ, dth * Ra.dr2n, y_dth * Ra.y_dr2n);
                } else {
                    v[2] = sB1[2];
                }
            } else {
                v[1] = sB1[1];
                v[2] = sB1[2];
            }
#pragma unroll
            for (int c = 0; c < 3; c++) Bh1[c] = v[c];
            lB[a & 3][0][t] = v[0];
            lB[a & 3][1][t] = v[2];
        }
        lds_barrier();

        // ---- node J_FFE, row b = q - 1 (needs B^{n+1/2} rows b-1, b)
        const int b = q - 1;
        if constexpr (FF) {
            if (b >= qs && b <= nr && (b == 0 || b - 1 >= qs)) {
                // rho = div E / 4 pi over the dual cell of node (max(b, 1), j)
                R rho = (R)0;
                if (b < nr) {
                    // rows ii and ii - 1 of the E state (own column), theta at j-1
                    const bool one = b == 0;
                    const int ii = one ? 1 : b;
                    const R er_i = one ? sE0[0] : sE1[0];
                    const R er_m = one ? sE1[0] : sE2[0];
                    const R et_i = one ? sE0[1] : sE1[1];
                    const R et_l = lE[ii & 1][2][tl];
                    const auto &Ri = row[ii];
                    R flux = Ri.rh2 * dcd_j * er_i - Ri.rh2m * dcd_j * er_m;
                    if (jlt) flux += sh_j * Ri.dr2h * et_i;
                    if (jgt) flux -= sh_jm * Ri.dr2h * et_l;
                    R dv = quot(flux, Ri.dr3h * dcd_j, Ri.y_dr3h * y_dcd);
                    rho = quot(dv, fourpi, 1.0 / fourpi);
                }
                // node E^n (totals) and B^{n+1/2} (totals)
                R e[3], bb[3];
                {
                    R tr_i = sE1[0];
                    R tr_m = sE2[0];
                    e[0] = b == 0 ? tr_i : b == nr ? tr_m : (R)0.5 * (tr_m + tr_i);
                    R tt_j = sE1[1];
                    R tt_l = lE[b & 1][2][tl];
                    e[1] = (j == 0 || j == nth) ? (R)0 : (R)0.5 * (tt_l + tt_j);
                    e[2] = sE1[2];
                }
                {
                    const R br_l = lB[b & 3][0][tl];
                    bb[0] = j == 0 ? Bh1[0] : j == nth ? br_l : (R)0.5 * (br_l + Bh1[0]);
                    bb[1] = b == 0 ? Bh1[1] : b == nr ? Bh2[1] : (R)0.5 * (Bh2[1] + Bh1[1]);
                    const R bp_l = lB[b & 3][1][tl];
                    if (j == 0 || j == nth) {
                        bb[2] = (R)0;
                    } else if (b == 0) {
                        bb[2] = (R)0.5 * (bp_l + Bh1[2]);
                    } else if (b == nr) {
                        bb[2] = (R)0.5 * (lB[(b - 1) & 3][1][tl] + Bh2[2]);
                    } else {
                        bb[2] = (R)0.25 * (lB[(b - 1) & 3][1][tl] + Bh2[2] + bp_l + Bh1[2]);
                    }
                }
                R b2 = bb[0] * bb[0] + bb[1] * bb[1] + bb[2] * bb[2];
                R x0 = e[1] * bb[2] - e[2] * bb[1];
                R x1 = e[2] * bb[0] - e[0] * bb[2];
                R x2 = e[0] * bb[1] - e[1] * bb[0];
                {
                    bool ok = b2 > (R)0;
                    const R y = rcp64(b2);
                    n01 = quot(rho * x0, b2, y);
                    n11 = quot(rho * x1, b2, y);
                    n21 = quot(rho * x2, b2, y);
                    if (!quot_ok(b2)) {
                        n01 = ok ? rho * x0 / b2 : (R)0;
                        n11 = ok ? rho * x1 / b2 : (R)0;
                        n21 = ok ? rho * x2 / b2 : (R)0;
                    }
                }
                lN[b & 1][t] = n11;
            }
        }

        // ---- Ampere, row c = q - 2: E after Ampere
        const int c = q - 2;
        if (c >= qs && c <= nr && (c == 0 || c - 1 >= qs)) {
            const auto &Rc = row[c];
            R v[3] = {sE2[0], sE2[1], sE2[2]};
            const R *bl = lB[c & 3][0];   // row c, B^{n+1/2} state r, j-1 at [tl]
            const R bp_l = lB[c & 3][1][tl];
            const R jrk = J2[0], jtk = J2[1], jpk = J2[2];
            if (c < nr) {
                const R Ar = Rc.rh2 * dcd_j, y = Rc.y_rh2 * y_dcd;
                R circ = (jlt ? Rc.rh * sh_j * Bh2[2] : (R)0) -
                         (jgt ? Rc.rh * sh_jm * bp_l : (R)0);
                R J;
                if constexpr (FF) {
                    R fs = (R)0.5 * (f2 + f1);
                    J = quot(((R)1 - fs) * jrk, dt * Ar, y_dt * y) + fs * (R)0.5 * (n02 + n01);
                } else {
                    J = quot(jrk, dt * Ar, y_dt * y);
                }
                v[0] = sE2[0] + (quot(dt * circ, Ar, y) - fourpi * dt * J);
            }
            if (c >= 1 && c < nr) {
                if (jlt) {
                    const R At = sh_j * Rc.dr2h, y = y_sh * Rc.y_dr2h;
                    R circ = -(Rc.rh * sh_j * Bh2[2] - Rc.rhm * sh_j * Bh3[2]);
                    R J;
                    if constexpr (FF) {
                        R fs = (R)0.5 * (f2 + lF[c % 3][tr]);
                        J = quot(((R)1 - fs) * jtk, dt * At, y_dt * y) +
                            fs * (R)0.5 * (n12 + lN[c & 1][tr]);
                    } else {
                        J = quot(jtk, dt * At, y_dt * y);
                    }
                    v[1] = sE2[1] + (quot(dt * circ, At, y) - fourpi * dt * J);
                }
                if (jin) {
                    const R Ap = dthd_j * Rc.dr2h, Vp = Rc.dr3h * dcd_j, yV = Rc.y_dr3h * y_dcd;
                    R circ = dth * (Rc.rh * Bh2[1] - Rc.rhm * Bh3[1]) -
                             Rc.drh * (Bh2[0] - bl[tl]);
                    R J;
                    if constexpr (FF) {
                        R fs = f2;
                        J = quot(((R)1 - fs) * jpk, Vp, yV) + fs * n22;
                    } else {
                        J = quot(jpk, Vp, yV);
                    }
                    v[2] = sE2[2] + (quot(dt * circ, Ap, y_dthd * Rc.y_dr2h) - fourpi * dt * J);
                }
            }
#pragma unroll
            for (int k = 0; k < 3; k++) Ea2[k] = v[k];
            if constexpr (FF) lEa[c & 1][t] = v[1];
        }
        lds_barrier();

        // ---- force-free correction at nodes, row d = q - 2
        const int d = q - 2;
        if constexpr (FF) {
            if (d >= qs && d <= nr && (qs == 0 || d >= qs + 2)) {
                R o[3] = {(R)0, (R)0, (R)0};
                if (f2 > (R)0) {
                    R e[3], bb[3], s[3];
                    const R tr_i = Ea2[0];
                    e[0] = d == 0 ? tr_i : d == nr ? Eat3r : (R)0.5 * (Eat3r + tr_i);
                    const R tt_j = Ea2[1];
                    e[1] = (j == 0 || j == nth) ? (R)0 : (R)0.5 * (lEa[d & 1][tl] + tt_j);
                    e[2] = Ea2[2];
                    const R br_l = lB[d & 3][0][tl];
                    bb[0] = j == 0 ? Bh2[0] : j == nth ? br_l : (R)0.5 * (br_l + Bh2[0]);
                    bb[1] = d == 0 ? Bh2[1] : d == nr ? Bh3[1] : (R)0.5 * (Bh3[1] + Bh2[1]);
                    const R bp_l = lB[d & 3][1][tl];
                    if (j == 0 || j == nth) {
                        bb[2] = (R)0;
                    } else if (d == 0) {
                        bb[2] = (R)0.5 * (bp_l + Bh2[2]);
                    } else if (d == nr) {
                        bb[2] = (R)0.5 * (lB[(d - 1) & 3][1][tl] + Bh3[2]);
                    } else {
                        bb[2] = (R)0.25 * (lB[(d - 1) & 3][1][tl] + Bh3[2] + bp_l + Bh2[2]);
                    }
                    ff_node(e, bb, s);
#pragma unroll
                    for (int k = 0; k < 3; k++) o[k] = f2 * (s[k] - e[k]);
                }
                d02 = o[0];
                d12 = o[1];
                d22 = o[2];
                lD[d & 1][t] = o[1];
            }
        }

        // ---- corrections averaged back, row e = q - 3: final E
        const int e = q - 3;
        if (e >= i0 && e <= nr) {
            R v[3] = {Ea3[0], Ea3[1], Ea3[2]};
            if constexpr (FF) {
                if (e < nr) v[0] = Ea3[0] + (R)0.5 * (d03 + d02);
                if (e >= 1 && e < nr) {
                    if (jlt) v[1] = Ea3[1] + (R)0.5 * (d13 + lD[e & 1][tr]);
                    if (jin) v[2] = Ea3[2] + d23;
                }
            }
#pragma unroll
            for (int k = 0; k < 3; k++) Ef3[k] = v[k];
            lEf[e & 1][0][t] = v[0];
            lEf[e & 1][1][t] = v[2];
        }

        // ---- Faraday half step, row f = q - 4: B^{n+1}, absorber, stores
        if (fr >= i0 && fr <= iL) {
            const R epn = lEf[fr & 1][1][tr];
            const R ern = lEf[fr & 1][0][tr];
            const auto &Rf = row[fr];
            R vb[3];
            {
                R circ = Rf.rn * (sn_j1 * epn - sn_j * Ef4[2]);
                vb[0] = Bh4[0] - quot(h * circ, Rf.rn2 * dcn_j, Rf.y_rn2 * y_dcn);
                if (!jlt) vb[0] = Bh4[0];
            }
            if (fr < nr) {
                if (jin) {
                    R circ = sn_j * (Rf.rn1 * Ef3[2] - Rf.rn * Ef4[2]);
                    vb[1] = Bh4[1] + quot(h * circ, sn_j * Rf.dr2n, y_sn * Rf.y_dr2n);
                } else {
                    vb[1] = (R)0;
                }
                if (jlt) {
                    R circ = dth * (Rf.rn1 * Ef3[1] - Rf.rn * Ef4[1]) - Rf.drn * (ern - Ef4[0]);
                    vb[2] = Bh4[2] - quot(h * circ, dth * Rf.dr2n, y_dth * Rf.y_dr2n);
                } else {
                    vb[2] = Bh4[2];
                }
            } else {
                vb[1] = Bh4[1];
                vb[2] = Bh4[2];
            }
            R ve[3] = {Ef4[0], Ef4[1], Ef4[2]};
            // absorbing layer: E damped, B relaxed to its initial value
            if (damp) {
                const R ln = Rf.lamn;
                const R lh = fr < nr ? Rf.lamh : (R)1;
                if (!(ln == (R)1 && lh == (R)1)) {
                    if (fr < nr) {
                        ve[0] *= lh;
                        const R b0t = b0[1];
                        vb[1] = b0t + lh * (vb[1] - b0t);
                        if (jlt) {
                            const R b0p = b0[2];
                            vb[2] = b0p + lh * (vb[2] - b0p);
                        }
                    }
                    ve[2] *= ln;
                    if (jlt) {
                        ve[1] *= ln;
                        const R b0r = b0[0];
                        vb[0] = b0r + ln * (vb[0] - b0r);
                    }
                }
            }
            if (t >= kFzL && t < kFzL + W && colok) {
                const size_t k0 = ix(ld, fr, 0);
                const unsigned jk = jc;
#pragma unroll
                for (int kk = 0; kk < 3; kk++) {
                    (A.oE[kk] + k0)[jk] = ve[kk];
                    (A.oB[kk] + k0)[jk] = vb[kk];
                    (A.Jz[kk] + k0)[jk] = (R)0;
                }
            }
        }
        lds_barrier();

        // ---- shift the own-column histories by one row
        Eat3r = Ea2[0];   // E_r after Ampere, row q-2
#pragma unroll
        for (int k = 0; k < 3; k++) {
            sE2[k] = sE1[k]; sE1[k] = sE0[k];
            sB1[k] = sB0[k];
            J2[k] = J1[k]; J1[k] = J0[k];
            Bh4[k] = Bh3[k]; Bh3[k] = Bh2[k]; Bh2[k] = Bh1[k];
            Ea3[k] = Ea2[k];
            Ef4[k] = Ef3[k];
        }
        if constexpr (FF) {
            f2 = f1; f1 = f0;
            n02 = n01; n12 = n11; n22 = n21;
            d03 = d02; d13 = d12; d23 = d22;
        }
    }
}

// Slab height: enough slabs that the grid fills the GPU once.  The rows of a
// slab are a serial chain (1.6 us a row in FP32, 2.8 in FP64 with the
// force-free stages), so a grid that cannot fill the GPU takes slabs as low as
// one row: the six halo rows of each then cost idle CUs, not time.  Step
// without particles, slabs of at least 32 rows against these: 128^2 FP64 151
// -> 34 us, 300 x 517 FP32 90 -> 39, 1024^2 FP32 120 -> 78, FP64 215 -> 138
// (FP64 before its rows were loaded ahead); from 2048^2 on 32 rows or more
// fill the GPU.  `shared`: the height for a
// launch that many systems share (0 = this system alone).
inline int fused_rows(const ffpic_ctx *c, int width, int shared = 0) {
    if (c->fused_rows > 0) return c->fused_rows;
    if (shared > 0) return shared;
    const int nbx = (c->nth + 1 + width - 1) / width;
    const int slots = c->fused_slots > 0 ? c->fused_slots : 768;
    const int slabs = std::max(1, slots / nbx);
    return (c->nr + 1 + slabs - 1) / slabs;
}

// the row blocks of the FP64 field step, as doubles
static std::vector<double> fused64_rows(const ffpic_ctx *c) {
    std::vector<FusedRow> row((size_t)c->nr + 1, FusedRow{});
    const std::vector<double> *T = c->tab;
    for (int i = 0; i <= c->nr; i++) {
        FusedRow &x = row[i];
        const bool half = i < c->nr;   // r_{i+1/2} is a row of the grid
        x.rn = T[T_RN][i];
        x.rn2 = T[T_RN2][i];
        x.lamn = T[T_LAMN][i];
        x.y_rn2 = 1.0 / x.rn2;
        if (half) {
            x.rn1 = T[T_RN][i + 1];
            x.drn = T[T_DRN][i];
            x.dr2n = T[T_DR2N][i];
            x.y_dr2n = 1.0 / x.dr2n;
            x.rh = T[T_RH][i];
            x.lamh = T[T_LAMH][i];
            x.rh2 = T[T_RH2][i];
            x.y_rh2 = 1.0 / x.rh2;
        }
        if (i >= 1) {
            x.rhm = T[T_RH][i - 1];
            x.rh2m = T[T_RH2][i - 1];
            x.drh = T[T_DRH][i];
        }
        x.dr2h = T[T_DR2H][i];
        x.y_dr2h = 1.0 / x.dr2h;
        x.dr3h = T[T_DR3H][i];
        x.y_dr3h = 1.0 / x.dr3h;
    }
    const double *p = (const double *)row.data();
    return {p, p + row.size() * (sizeof(FusedRow) / sizeof(double))};
}

// Threads of a workgroup of the FP64 field step: 128 where its strips cover
// the columns with fewer threads than those of 256 (a strip costs the same
// whatever part of it is on the grid), else 256, whose halo is a smaller part.
// Step without particles, us with 128 and 256: 128^2 17.5 and 19.8, 256^2 21.5
// and 25.5, 400 x 333 26.6 and 28.5, 1024^2 62 and 66, 2048^2 196 and 206,
// 3000 x 1500 217 and 232, 4096^2 (4352 threads a row either way) 673 and 655.
// The FP32 step, which waits for memory more, gains nothing from it (16 systems
// grouped 376 and 372 us, 4096^2 650 and 619).
inline int fused_threads64(int nth) {
    auto threads = [&](int t) { return (nth + t - kFzL - kFzR) / (t - kFzL - kFzR) * t; };
    return threads(128) < threads(256) ? 128 : 256;
}

// FP64 field step (E and B evolved directly)
static void run_field_fused64(ffpic_ctx *c) {
    using R = double;
    FusedArgs A{};
    A.row = (const FusedRow *)c->fz_row64;
    A.g = geo<R>(c);
    A.h = (R)(0.5 * c->dt);
    A.absorb0 = c->absorb_row0;
    for (int k = 0; k < 3; k++) {
        A.sE[k] = (const R *)c->E[k];  A.sB[k] = (const R *)c->B[k];
        A.oE[k] = (R *)c->stAlt[k];    A.oB[k] = (R *)c->stAlt[3 + k];
        A.B0[k] = (const R *)c->B0[k];
        A.J[k] = (const R *)c->J[k];
        A.Jz[k] = (R *)c->Jalt[k];
    }
    A.f = (const R *)c->f;
    const int T = fused_threads64(c->nth), width = T - kFzL - kFzR;
    auto kern = T == 128 ? (c->d.ff_enable ? k_field_fused<true, 128> : k_field_fused<false, 128>)
                         : (c->d.ff_enable ? k_field_fused<true, 256> : k_field_fused<false, 256>);
    if (c->fused_slots == 0) {   // workgroups resident at once, for the slab height
        int per_cu = 0, cus = 0, dev = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, T, 0) !=
                hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
            (void)hipGetLastError();
            per_cu = 3;
            cus = 256;
        }
        c->fused_slots = std::max(1, per_cu * cus);
    }
    A.rows = fused_rows(c, width);
    dim3 grd((c->nth + 1 + width - 1) / width, (c->nr + 1 + A.rows - 1) / A.rows);
    hipLaunchKernelGGL(kern, grd, dim3(T), 0, c->stream, A);
    FFPIC_LAUNCH_CHECK();
    // the new state and the cleared accumulators become current
    for (int k = 0; k < 3; k++) {
        std::swap(c->E[k], c->stAlt[k]);
        std::swap(c->B[k], c->stAlt[3 + k]);
        std::swap(c->J[k], c->Jalt[k]);
    }
}

}  // namespace ffpic
