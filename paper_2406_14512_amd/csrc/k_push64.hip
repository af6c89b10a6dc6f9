// FP64 particle push and charge-conserving deposit (plain FP64 GPU path).
//
// One thread per particle slot.  State per particle: r, theta, u_r,
// u_theta, u_phi (FP64 SoA); a dead slot has r = -1 until the next sort.
// The per-particle arithmetic follows the plain FP64 definition step by step.
// This file is compiled without FP contraction, so every operation up to the
// new state is rounded as written there (a particle's flux is the small
// difference of two in-cell offsets, so one unit in the last place of a
// radius shows in it); quotients, roots, the sine, cosine and logarithm below
// are rounded correctly but for rare ties, the new polar angle but for 2 % of
// the particles in a coarse grid's first columns and fewer beyond (the device
// library's arctangent: 25 % anywhere), at a fraction of the library's
// instructions.  The order in which currents are summed differs.
//
// Push (Sect. 3): eq. (motion) integrated with the Boris rotation; the
// Landau-Lifshitz force g with the effective field of eq. (bperp) is added
// explicitly with the time-centred velocity (its strength scaled by the
// ramp of Sect. 5); inside the shell around the star only the momentum
// along B is kept.  The particle is moved in the
// local Cartesian frame at azimuth 0 and rotated back to the meridional
// plane.  Deposit: zigzag (relay-point) split of the move in logical
// coordinates (log r / dlog, theta / dtheta), charge fluxes through the dual
// faces (exact discrete charge conservation), azimuthal current from v_phi
// at the mid-point.  Accumulation as in the FP32 path: an LDS patch per
// workgroup over the bounding box of its (cell-sorted) particles, in-cell
// moves summed across each 16-lane row first (DPP, one cell per row and
// pass), one global FP64 atomic per non-zero patch entry.
#include <algorithm>
#include <type_traits>

#include "gather.h"
#include "math64.h"

namespace ffpic {

constexpr int kWG64 = 256;
constexpr int kTile64 = 640;    // LDS current patch entries per component (FP64)
constexpr int kFld64 = 320;     // LDS field patch nodes (six components each)
constexpr int kSide64 = 112;     // rows and columns of a patch, at most
constexpr int kLone64 = 8;       // in-cell moves left in a wave that add by themselves
constexpr int kQueue64 = 64;    // queued cell-crossing moves per workgroup

struct P64 {
    int nr, nth, ld;
    double rmin, r_abs, dlog, dth, dt;
    double inv_dlog, inv_dth;   // reciprocals, for quot()
    float girm, gidl, gidt;     // cell guess: 1 / rmin, 1 / dlog, 1 / dth
    double dsub;                // spacing of the sine and cosine table
    float gids;                 // 1 / dsub, a little less
    const double *rn;
    double Q, wq, rr;
    double shell_r;        // r below this: only the momentum along B is kept
    int lds;               // the guesses are within a cell: the LDS patches may serve
};

struct Push64Args {
    P64 p;
    int nub;
    const int32_t *nslots;
    const uint8_t *kill;
    const double *E[3], *B[3];
    const double2 *lct;         // ln 2 and log(1 + k/16), in two parts each
    const double4 *sct;         // sines, cosines and their rounding errors
    double *R, *TH, *UR, *UT, *UP;
    double *J[3];
    unsigned long long *removed;
    uint32_t *err;
    // a push that places its species' sort: the place of each slot's particle
    // (-1: none) and the state of the new order
    const int32_t *dest;
    double *oR, *oTH, *oUR, *oUT, *oUP;
};

// the species of one launch (blockIdx.y)
struct Push64Jobs {
    Push64Args job[FFPIC_MAX_SPECIES];
};

// The arguments as the kernel finds them in constant memory.  The particle
// loop takes their address anew at each stage (opaque()), so that each value
// is a scalar load near its use: held across the loop they exceed the scalar
// registers and spill into lanes of vector registers.
typedef const __attribute__((address_space(4))) Push64Args *KArgs;

// element `idx` of an array (byte offset below 2^32) from a uniform base, so
// that no 64-bit address is formed per lane
template <typename T>
__device__ __forceinline__ T &at32(T *base, unsigned idx) {
    return *reinterpret_cast<T *>(
        reinterpret_cast<char *>(const_cast<typename std::remove_const<T>::type *>(base)) +
        (size_t)(idx * (unsigned)sizeof(T)));
}

// element `idx` of an array of any length
__device__ __forceinline__ double &at64(double *base, int idx) { return base[(size_t)idx]; }

template <typename P>
__device__ __forceinline__ P opaque(P t) {
    asm volatile("" : "+s"(t));
    return t;
}

// ---------------------------------------------------------------------------
// Square roots, rounded as the IEEE operation (quotients: math64.h): the
// hardware estimate (about 24 bits), Newton steps and the exact residual; a
// root with its reciprocal is 13 instructions, compiled ones 15 and 11.

// sqrt(x) and its reciprocal, x a positive normal number
__device__ __forceinline__ double root64(double x, double &inv) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    const double z = h + h;
    inv = __builtin_fma(__builtin_fma(-g, z, 1.0), z, z);
    return g;
}

// Coefficients of the series below, in constant memory and read like the
// arguments: as literals the compiler keeps all of them in registers across
// the loop (60 VGPRs).
typedef const __attribute__((address_space(4))) double *Poly64;
enum { KS = 0, KC = 4, KL = 8, KT = 14 };
__constant__ double kPoly64[21] = {
    // 1 / 9!, 7!, 5!, 3!
    1.0 / 362880.0, 1.0 / 5040.0, 1.0 / 120.0, 1.0 / 6.0,
    // 1 / 8!, 6!, 4!, 2!
    1.0 / 40320.0, 1.0 / 720.0, 1.0 / 24.0, 1.0 / 2.0,
    // 2 / 13, 11, ..., 3 (logarithm)
    2.0 / 13.0, 2.0 / 11.0, 2.0 / 9.0, 2.0 / 7.0, 2.0 / 5.0, 2.0 / 3.0,
    // 1 / 15, 13, ..., 3 (arctangent)
    1.0 / 15.0, 1.0 / 13.0, 1.0 / 11.0, 1.0 / 9.0, 1.0 / 7.0, 1.0 / 5.0, 1.0 / 3.0};

// sin and cos of th = t_j + d (d exact, 0 <= d <= 1/16), rounded correctly
// almost always, with their rounding errors (slo, clo): the sums
// S cos d + C sin d and C cos d - S sin d from the table angle's S = sin t_j
// and C = cos t_j (t: S, C and the errors of both), with the
// leading terms S, C, C d and S d carried in two parts and the Taylor
// remainders (below 1e-18 of the sums) in one
__device__ __forceinline__ void sincos_node(Poly64 K, const double4 t, double d, double &s,
                                            double &c, double &slo, double &clo) {
    const double z = d * d;
    double e = K[KS], q = K[KC];
#pragma unroll
    for (int k = 1; k < 4; k++) {
        e = __builtin_fma(-e, z, K[KS + k]);
        q = __builtin_fma(-q, z, K[KC + k]);
    }
    e *= -(d * z);                               // sin d - d
    q *= -z;                                     // cos d - 1
    {
        const double p = t.y * d, pl = __builtin_fma(t.y, d, -p);
        const double h = t.x + p, l = p - (h - t.x);     // |C d| <= |S| or S = 0
        const double r = l + (pl + (t.z + __builtin_fma(t.w, d, __builtin_fma(t.y, e, t.x * q))));
        s = h + r;
        slo = r - (s - h);
    }
    {
        const double p = -(t.x * d), pl = -__builtin_fma(t.x, d, p);
        const double h = t.y + p, v = h - t.y, l = (t.y - (h - v)) + (p - v);
        const double r = l + (pl + (t.w + __builtin_fma(-t.z, d, __builtin_fma(-t.x, e, t.y * q))));
        c = h + r;
        clo = r - (c - h);
    }
}

// log(q) of a positive normal q, rounded correctly almost always (coarse
// grids): q = 2^e m, m in [1, 2), log m = log c + 2 atanh((m - c) / (m + c))
// with c = 1 + k / 16 the nearest sixteenth; t: ln 2 and the log c, in two
// parts each (the first part of ln 2 has 32 bits, so e times it is exact)
__device__ __forceinline__ double log_wide(Poly64 K, const double2 *t, double q) {
    const int ex = __builtin_amdgcn_frexp_exp(q) - 1;
    const double m = 2.0 * __builtin_amdgcn_frexp_mant(q);
    const double kf = floor(__builtin_fma(m - 1.0, 16.0, 0.5)), c = 1.0 + kf * 0.0625;
    const double n = m - c, d = m + c, dv = d - m, dl = (m - (d - dv)) + (c - dv);
    const double y = rcp64(d), s = n * y, z = s * s;
    const double sl = (__builtin_fma(-s, d, n) - s * dl) * y;
    double R = K[KL];
#pragma unroll
    for (int k = 1; k < 6; k++) R = __builtin_fma(R, z, K[KL + k]);
    const double2 l2 = t[0], lc = t[1 + (int)kf];
    const double a = ex * l2.x;
    const double u = a + lc.x, uv = u - a, ul = (a - (u - uv)) + (lc.x - uv);
    const double s2 = s + s, w = u + s2, wv = w - u, wl = (u - (w - wv)) + (s2 - wv);
    return w + (wl + (ul + (__builtin_fma((double)ex, l2.y, lc.y) + __builtin_fma(s * z, R, sl + sl))));
}

// log(q) / dlog for q in [1, e^dlog): with SERIES (dlog <= 1/16)
// log(1 + f) = 2 atanh(s), s = f / (2 + f), written f - s (f - R) with the
// product carried in two parts, so that the sum is rounded correctly almost
// always, as the library's is (a particle's radial flux is the difference of
// two such logarithms, often a small one); the terms past s^13 are below
// 1e-19 of the sum
template <bool SERIES>
__device__ __forceinline__ double log_cells(KArgs A, Poly64 K, double q) {
    double l;
    if (SERIES) {
        const double f = q - 1.0, b = 2.0 + f, bl = f - (b - 2.0);
        const double y = rcp64(b), s = f * y, z = s * s;
        const double sl = (__builtin_fma(-s, b, f) - s * bl) * y;
        double R = K[KL];
#pragma unroll
        for (int k = 1; k < 6; k++) R = __builtin_fma(R, z, K[KL + k]);
        R *= z;
        const double t = f - R, tl = (f - t) - R;
        const double c = s * t;
        const double cl = __builtin_fma(s, t, -c) + (s * tl + sl * t);
        const double h = f - c;
        l = h + (((f - h) - c) - cl);
    } else {
        l = log_wide(K, A->lct, q);
    }
    return quot(l, A->p.dlog, A->p.inv_dlog);
}

// Starting cell of a position in single precision.  In theta it is off by the
// roundings of th, 1 / dth and their product, 3 * 2^-24 of up to 65535 cells or
// 1.2e-2 cells.  In r those of r / rmin and its logarithm, some 2^-22 together,
// count 1 / dlog cells each, the products up to 1.2e-2 more: a quarter of a cell
// at dlog = 2^-20, so there and above at most one cell off in each direction.
// In thinner shells, or with radii near the ends of the float range, the guess
// may be any cell, and the LDS patches, sized for one cell off, are not used
// (P64::lds).
__device__ __forceinline__ int guess_i(KArgs A, double r) {
    const float g = __logf((float)r * A->p.girm) * A->p.gidl;
    return g > 0.f ? (g < (float)(A->p.nr - 1) ? (int)g : A->p.nr - 1) : 0;
}
__device__ __forceinline__ int guess_j(KArgs A, double th) {
    const float g = (float)th * A->p.gidt;
    return g > 0.f ? (g < (float)(A->p.nth - 1) ? (int)g : A->p.nth - 1) : 0;
}

// Radii of the nodes: with the LDS patches, those of the chunk's rows and one
// cell around them, with their reciprocals, from LDS; others from the table.
struct Rows64 {
    const double2 *t;      // r_i and 1 / r_i of rows [i0, i0 + n)
    int i0, n;
};
template <bool LDS>
__device__ __forceinline__ double2 row64(KArgs A, const Rows64 &R, int i) {
    if (LDS && (unsigned)(i - R.i0) < (unsigned)R.n) return R.t[i - R.i0];
    const double x = at32(A->p.rn, i);
    return make_double2(x, rcp64(x));
}

// radial cell of r from the cell i (lo: radius and reciprocal of its inner
// node, rhi: radius of its outer one, in and out) and the offset in it; the
// comparisons settle the cell as locate64 does
template <bool LDS, bool SERIES>
__device__ __forceinline__ double settle_r(KArgs A, Poly64 K, const Rows64 &R, double r, int &i,
                                           double2 &lo, double &rhi) {
    while (i > 0 && r < lo.x) { i--; rhi = lo.x; lo = row64<LDS>(A, R, i); }
    while (i < A->p.nr - 1 && r >= rhi) {
        i++;
        lo = row64<LDS>(A, R, i);
        rhi = row64<LDS>(A, R, i + 1).x;
    }
    const double a = log_cells<SERIES>(A, K, quot(r, lo.x, lo.y));
    return fmin(fmax(a, 0.0), 1.0);
}
// polar cell of th from the cell j (theta_j = j dth, which the sort's table holds
// bit for bit, so that both settle the same cell)
__device__ __forceinline__ double settle_t(KArgs A, double th, int &j) {
    double tlo = j * A->p.dth, thi = (j + 1) * A->p.dth;
    while (j > 0 && th < tlo) { j--; thi = tlo; tlo = j * A->p.dth; }
    while (j < A->p.nth - 1 && th >= thi) { j++; tlo = thi; thi = (j + 1) * A->p.dth; }
    const double b = quot(th - tlo, A->p.dth, A->p.inv_dth);
    return fmin(fmax(b, 0.0), 1.0);
}

__device__ __forceinline__ double norm2(const double v[3]) {
    return v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
}

__device__ __forceinline__ void boris_rr(double u[3], const double E[3], const double B[3],
                                         double dt, double wq, double rr) {
    double h = 0.5 * dt * wq;
    double um[3], t[3], sv[3], up[3], uL[3];
    for (int k = 0; k < 3; k++) um[k] = u[k] + h * E[k];
    double igm;
    const double gm = root64(1.0 + norm2(um), igm);
    for (int k = 0; k < 3; k++) t[k] = quot(h * B[k], gm, igm);
    const double t2 = 1.0 + norm2(t);
    const double it2 = rcp64(t2);
    for (int k = 0; k < 3; k++) sv[k] = quot(2.0 * t[k], t2, it2);
    double c0 = um[1] * t[2] - um[2] * t[1];
    double c1 = um[2] * t[0] - um[0] * t[2];
    double c2 = um[0] * t[1] - um[1] * t[0];
    up[0] = um[0] + c0; up[1] = um[1] + c1; up[2] = um[2] + c2;
    c0 = up[1] * sv[2] - up[2] * sv[1];
    c1 = up[2] * sv[0] - up[0] * sv[2];
    c2 = up[0] * sv[1] - up[1] * sv[0];
    uL[0] = um[0] + c0 + h * E[0];
    uL[1] = um[1] + c1 + h * E[1];
    uL[2] = um[2] + c2 + h * E[2];
    if (rr != 0.0) {
        double ub[3], beta[3], Fv[3], igb;
        for (int k = 0; k < 3; k++) ub[k] = 0.5 * (u[k] + uL[k]);
        const double gb = root64(1.0 + norm2(ub), igb);
        for (int k = 0; k < 3; k++) beta[k] = quot(ub[k], gb, igb);
        Fv[0] = E[0] + (beta[1] * B[2] - beta[2] * B[1]);
        Fv[1] = E[1] + (beta[2] * B[0] - beta[0] * B[2]);
        Fv[2] = E[2] + (beta[0] * B[1] - beta[1] * B[0]);
        double be = beta[0] * E[0] + beta[1] * E[1] + beta[2] * E[2];
        double bp2 = (Fv[0] * Fv[0] + Fv[1] * Fv[1] + Fv[2] * Fv[2]) - be * be;
        if (bp2 < 0.0) bp2 = 0.0;
        double x0 = Fv[1] * B[2] - Fv[2] * B[1];
        double x1 = Fv[2] * B[0] - Fv[0] * B[2];
        double x2 = Fv[0] * B[1] - Fv[1] * B[0];
        uL[0] = uL[0] + dt * rr * (x0 + be * E[0] - gb * gb * bp2 * beta[0]);
        uL[1] = uL[1] + dt * rr * (x1 + be * E[1] - gb * gb * bp2 * beta[1]);
        uL[2] = uL[2] + dt * rr * (x2 + be * E[2] - gb * gb * bp2 * beta[2]);
    }
    u[0] = uL[0]; u[1] = uL[1]; u[2] = uL[2];
}

// a vector of the local (r, theta, phi) basis in the local Cartesian frame
// at azimuth 0 (x along the cylindrical radius, y along phi)
__device__ __forceinline__ void to_cart(double r, double t, double p, double st, double ct,
                                        double o[3]) {
    o[0] = r * st + t * ct;
    o[1] = p;
    o[2] = r * ct - t * st;
}

// a DPP lane permutation of a double (both 32-bit halves moved the same way)
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sums eight per-lane values over each 16-lane row, halving the number of
// values at every stage (exchange with lane^1, lane^2, a rotation by four
// lanes, a rotation by eight).  Lane l then holds the row sum of value
// 4*bit0(l) + 2*bit1(l) + bit2(l); keep[] are the four values a lane sums in
// the first stage (values 4..7 on lanes with bit 0 set, 0..3 otherwise),
// pass[] the four its neighbour sums.
__device__ __forceinline__ double row_sum8_64(const double keep[4], const double pass[4], bool b1,
                                              bool b2) {
    double y[4];
#pragma unroll
    for (int m = 0; m < 4; m++) y[m] = keep[m] + dpp64<0xB1>(pass[m]);
    const double z0 = (b1 ? y[2] : y[0]) + dpp64<0x4E>(b1 ? y[0] : y[2]);
    const double z1 = (b1 ? y[3] : y[1]) + dpp64<0x4E>(b1 ? y[1] : y[3]);
    const double w = (b2 ? z1 : z0) + dpp64<0x124>(b2 ? z0 : z1);
    return w + dpp64<0x128>(w);
}

// The eight adds of a move inside its cell, where the zigzag's two segments
// share the faces: J_r at (i, j) and (i, j+1), J_theta at (i, j) and (i+1, j),
// J_phi at the four nodes.  hx, hy: half the radial and polar charge flux, q4
// a quarter of the azimuthal one, X, Y twice the mid-point.
__device__ __forceinline__ void values8_64(double hx, double hy, double q4, double X, double Y,
                                           double s[8]) {
#pragma clang fp contract(fast)
    s[1] = hx * Y;
    s[0] = 2.0 * hx - s[1];
    s[3] = hy * X;
    s[2] = 2.0 * hy - s[3];
    const double u = q4 * X, z = 2.0 * q4 - u;
    s[7] = u * Y;
    s[5] = 2.0 * u - s[7];
    s[6] = z * Y;
    s[4] = 2.0 * z - s[6];
}

// where currents go: the LDS patch (tile) or the grid arrays
template <bool LDS>
struct Acc64 {
    double *tile;
    int ti0, tj0, TJ;
    double *g[3];
    int ld;
    __device__ __forceinline__ void add(int comp, int i, int j, double v) const {
        if (LDS) atomicAdd(&tile[comp * kTile64 + (i - ti0) * TJ + (j - tj0)], v);
        else gadd(&g[comp][ix(ld, i, j)], v);
    }
};

// general zigzag (relay-point) deposit of a move from (x1, y1) in cell (i, j)
// to (x2, y2) in the same frame, ending in cell (i + di, j + dj)
template <bool LDS>
__device__ __forceinline__ void zigzag64(KArgs A, const Acc64<LDS> &gacc, int i, int j, int di,
                                         int dj, double x1, double y1, double x2, double y2,
                                         double v1) {
    const int i2 = i + di, j2 = j + dj;
    double xr = fmin((di < 0 ? di : 0) + 1.0, fmax((double)(di > 0 ? di : 0), 0.5 * (x1 + x2)));
    double yr = fmin((dj < 0 ? dj : 0) + 1.0, fmax((double)(dj > 0 ? dj : 0), 0.5 * (y1 + y2)));
    double Q = A->p.Q;
    double fx1 = Q * (xr - x1), fy1 = Q * (yr - y1);
    double fx2 = Q * (x2 - xr), fy2 = Q * (y2 - yr);
    double wx1 = 0.5 * (x1 + xr), wy1 = 0.5 * (y1 + yr);
    double wx2 = 0.5 * (xr + x2) - di, wy2 = 0.5 * (yr + y2) - dj;
    gacc.add(0, i, j, fx1 * (1.0 - wy1));
    gacc.add(0, i, j + 1, fx1 * wy1);
    gacc.add(1, i, j, fy1 * (1.0 - wx1));
    gacc.add(1, i + 1, j, fy1 * wx1);
    gacc.add(0, i2, j2, fx2 * (1.0 - wy2));
    gacc.add(0, i2, j2 + 1, fx2 * wy2);
    gacc.add(1, i2, j2, fy2 * (1.0 - wx2));
    gacc.add(1, i2 + 1, j2, fy2 * wx2);
    double xm = 0.5 * (x1 + x2), ym = 0.5 * (y1 + y2);
    int im = (int)floor(xm), jm = (int)floor(ym);
    if (i + im > A->p.nr - 1) im = A->p.nr - 1 - i;
    if (j + jm > A->p.nth - 1) jm = A->p.nth - 1 - j;
    double wx = xm - im, wy = ym - jm;
    double qv = Q * v1;
    gacc.add(2, i + im, j + jm, qv * (1.0 - wx) * (1.0 - wy));
    gacc.add(2, i + im + 1, j + jm, qv * wx * (1.0 - wy));
    gacc.add(2, i + im, j + jm + 1, qv * (1.0 - wx) * wy);
    gacc.add(2, i + im + 1, j + jm + 1, qv * wx * wy);
}

// The field patch: six components of a node side by side, rows and columns
// from (fi0, fj0).  The polar half columns hold their axis ghosts (the edge
// column times the component's parity), so that a gather has no axis case.
struct Patch64 {
    const double *fld;
    int fi0, fj0, TJ;
    Rows64 rows;
    const double4 *cols;   // sine and cosine of the columns from fj0 + 1
};

// bilinear value of component COMP from the patch node at word offset o and
// its neighbours, with the weights of the four corners
template <int COMP>
__device__ __forceinline__ double bil64(const double *fld, int o, int rowW, double w00, double w10,
                                        double w01, double w11) {
    return w00 * fld[o + COMP] + w10 * fld[o + rowW + COMP] + w01 * fld[o + 6 + COMP] +
           w11 * fld[o + rowW + 6 + COMP];
}

struct Move64 {            // a queued cell-crossing move
    double x1, y1, x2, y2, v1;
    int c, d;
};

struct Counts64 {
    int kill, star, abs;
};

// the particles of one chunk (kWG64 * PPT slots from base), the patches in
// LDS (LDS) or the grid arrays read and added to directly
template <bool LDS, int PPT, bool SERIES, bool PLACE>
__device__ __forceinline__ void push_chunk64(KArgs A0, const Patch64 &F,
                                             const Acc64<LDS> &acc, double *kg, int n, int base,
                                             Move64 *queue, int *qn, Counts64 &cnt) {
    const int tid = threadIdx.x, lane = tid & 63;
    // the deposit value this lane adds after the row reduction: component,
    // radial and polar node offsets from the cell (values 0..7 below)
    const int rl = lane & 15;
    const bool b0 = rl & 1, b1 = rl & 2, b2 = rl & 4;
    const int kq = (b0 ? 4 : 0) + (b1 ? 2 : 0) + (b2 ? 1 : 0);
    const int kcomp = kq < 2 ? 0 : (kq < 4 ? 1 : 2);
    const int kdi = (kq == 3 || kq == 5 || kq == 7) ? 1 : 0;
    const int kdj = (kq == 1 || kq == 6 || kq == 7) ? 1 : 0;
    const int kofs = kcomp * kTile64 + (kdi - acc.ti0) * acc.TJ + kdj - acc.tj0;
    // the state of a slot (a slot past the last reads the last one and is
    // ignored)
    double r, th, ur, ut, up;
    int dn = -1;               // PLACE: the place of its particle
    auto load = [&](KArgs A, int q) {
        const unsigned qs = (unsigned)(min(q, n - 1) - base);
        r = at32(A->R + base, qs);
        th = at32(A->TH + base, qs);
        ur = at32(A->UR + base, qs);
        ut = at32(A->UT + base, qs);
        up = at32(A->UP + base, qs);
        if constexpr (PLACE) dn = at32(A->dest + base, qs);
    };
    load(opaque(A0), base + tid);
#pragma unroll 1
    for (int k = 0; k < PPT; k++) {
        const KArgs A = opaque(A0);
        const Poly64 K = opaque((Poly64)kPoly64);
        const int q = base + k * kWG64 + tid;
        const unsigned ql = (unsigned)(q - base);
        const int dq = dn;
        const bool live = q < n && r > 0.0 && (!PLACE || dq >= 0);
        bool simple = false, cross = false;
        double hx, hy, q4;                       // in-cell move: see values8_64
        int i = 0, j = 0, di = 0, dj = 0;
        double x1, y1, x2, y2, v1;
        if (live) {
            // ---- old cell and offsets
            i = guess_i(A, r);
            j = guess_j(A, th);
            double2 lo;
            double rhi;
            if constexpr (LDS) {               // the guesses lie in the box
                lo = F.rows.t[i - F.rows.i0];
                rhi = F.rows.t[i + 1 - F.rows.i0].x;
            } else {
                lo = row64<false>(A, F.rows, i);
                rhi = at32(A->p.rn, i + 1);
            }
            const double a = settle_r<LDS, SERIES>(A, K, F.rows, r, i, lo, rhi);
            const double b = settle_t(A, th, j);
            const bool killed = at32(A->kill, (unsigned)i * (unsigned)A->p.nth + (unsigned)j) != 0;
            // ---- staggered bilinear gather
            double Es[3], Bs[3];
            if (LDS) {
                const Lin rh = half_r(i, a, A->p.nr), thh = half_t(j, b);
                const double a1 = 1.0 - a, c1 = 1.0 - b, h1 = 1.0 - rh.w, g1 = 1.0 - thh.w;
                const int rowW = F.TJ * 6;
                const int on = (i - F.fi0) * rowW, oh = (rh.lo - F.fi0) * rowW;
                const int cn = (j - F.fj0) * 6, ch = (thh.lo - F.fj0) * 6;
                double w00 = h1 * c1, w10 = rh.w * c1, w01 = h1 * b, w11 = rh.w * b;
                Es[0] = bil64<0>(F.fld, oh + cn, rowW, w00, w10, w01, w11);
                Bs[1] = bil64<4>(F.fld, oh + cn, rowW, w00, w10, w01, w11);
                w00 = a1 * g1; w10 = a * g1; w01 = a1 * thh.w; w11 = a * thh.w;
                Es[1] = bil64<1>(F.fld, on + ch, rowW, w00, w10, w01, w11);
                Bs[0] = bil64<3>(F.fld, on + ch, rowW, w00, w10, w01, w11);
                w00 = a1 * c1; w10 = a * c1; w01 = a1 * b; w11 = a * b;
                Es[2] = bil64<2>(F.fld, on + cn, rowW, w00, w10, w01, w11);
                w00 = h1 * g1; w10 = rh.w * g1; w01 = h1 * thh.w; w11 = rh.w * thh.w;
                Bs[2] = bil64<5>(F.fld, oh + ch, rowW, w00, w10, w01, w11);
            } else {
                gather_eb(A->E[0], A->E[1], A->E[2], A->B[0], A->B[1], A->B[2], A->p.nr, A->p.nth, A->p.ld, i, j,
                          a, b, Es, Bs);
            }
            const KArgs A1 = opaque(A);
            double st, ct, stl, ctl;
            // (a coarse grid's table divides its cells, see ffpic_create)
            const int js = SERIES ? j : max((int)((float)th * A1->p.gids), 0);
            const double4 node = LDS && SERIES ? F.cols[j - F.fj0 - 1] : at32(A1->sct, js);
            sincos_node(K, node, th - js * (SERIES ? A1->p.dth : A1->p.dsub), st, ct, stl,
                        ctl);
            double E[3], B[3], u[3];
            to_cart(Es[0], Es[1], Es[2], st, ct, E);
            to_cart(Bs[0], Bs[1], Bs[2], st, ct, B);
            to_cart(ur, ut, up, st, ct, u);
            boris_rr(u, E, B, A1->p.dt, A1->p.wq, A1->p.rr);
            if (r < A1->p.shell_r) {
                // shell around the star (Sect. 5): drop the momentum across B
                const double bb = B[0] * B[0] + B[1] * B[1] + B[2] * B[2];
                if (bb > 0.0) {
                    const double ub = (u[0] * B[0] + u[1] * B[1] + u[2] * B[2]) / bb;
                    u[0] = ub * B[0]; u[1] = ub * B[1]; u[2] = ub * B[2];
                }
            }
            const KArgs A2 = opaque(A);
            double ig;
            const double g = root64(1.0 + norm2(u), ig);
            if (!isfinite(g) && !killed) atomicOr(A2->err, FFPIC_ERR_NONFINITE);
            const double v0 = quot(u[0], g, ig), vv2 = quot(u[2], g, ig);
            v1 = quot(u[1], g, ig);
            const double x = r * st + A2->p.dt * v0, y = A2->p.dt * v1, z = r * ct + A2->p.dt * vv2;
            const double ww = x * x + y * y;
            double iw;
            double w = root64(ww, iw);
            double cp = quot(x, w, iw), sp = quot(y, w, iw);
            if (!(ww > 0.0)) { w = 0.0; cp = 1.0; sp = 0.0; }
            const double ux = cp * u[0] + sp * u[1], uy = -sp * u[0] + cp * u[1], uz = u[2];
            double ir2;
            const double r2 = root64(w * w + z * z, ir2);
            // ---- new polar angle.  SERIES: th plus the small angle to (w, z),
            // whose sine is formed with the products' and st's and ct's rounding
            // errors, so that the sum is rounded as atan2(w, z) of the same
            // arguments almost always.  A move is at most dt <= rmin dth long,
            // so its tangent stays near dth <= 1/16, where the terms left out
            // are below 1e-18 of it.  That angle carries errors of its own last
            // place, which the sum drops unless it is itself as small: within
            // 1/12 of the axis (the first column at least) the angle is that of
            // (w, z) directly, with the quotient's rounding error.
            double th2;
            if (SERIES) {
                auto series = [&](double t2) {           // 1/3 - t2/5 + t2^2/7 - ...
                    double T = K[KT];
#pragma unroll
                    for (int m = 1; m < 7; m++) T = __builtin_fma(-T, t2, K[KT + m]);
                    return T;
                };
                if (w < z * (1.0 / 12.0)) {
                    const double y = rcp64(z), t = quot(w, z, y), t2 = t * t;
                    const double tl = __builtin_fma(-t, z, w) * y;
                    th2 = t + __builtin_fma(-(t * t2), series(t2), tl);
                } else {
                    const double zs = z * st;
                    double cr = __builtin_fma(w, ct, -zs) + __builtin_fma(-z, st, zs);
                    cr += w * ctl - z * stl;
                    const double dot = w * st + z * ct;
                    const double t = quot(cr, dot, rcp64(dot)), t2 = t * t;
                    th2 = fmin(fmax(th + __builtin_fma(-(t * t2), series(t2), t), 0.0), kPi);
                }
            } else {
                th2 = atan2(w, z);
            }
            const KArgs A3 = opaque(A);
            const bool star = !killed && !(r2 >= A3->p.rmin);
            const bool absb = !killed && !star && r2 >= A3->p.r_abs;
            const bool keep = !killed && !star && !absb;
            cnt.kill += killed;
            cnt.star += star;
            cnt.abs += absb;
            if (!keep) {
                if constexpr (PLACE) at64(A3->oR, dq) = -1.0;
                else at32(A3->R + base, ql) = -1.0;
            } else {
                const double st2 = quot(w, r2, ir2), ct2 = quot(z, r2, ir2);
                // ---- new cell: a move ends at most one cell away, so the
                // search starts from the old cell
                int i2 = i, j2 = j;
                const double a2 = settle_r<LDS, SERIES>(A3, K, F.rows, r2, i2, lo, rhi);
                const double bb2 = settle_t(A3, th2, j2);
                di = i2 - i;
                dj = j2 - j;
                const bool cfl = di > 1 || di < -1 || dj > 1 || dj < -1;
                if (cfl) atomicOr(A3->err, FFPIC_ERR_CFL);
                x1 = a; y1 = b; x2 = di + a2; y2 = dj + bb2;
                if constexpr (PLACE) {
                    at64(A3->oR, dq) = r2;
                    at64(A3->oTH, dq) = th2;
                    at64(A3->oUR, dq) = ux * st2 + uz * ct2;
                    at64(A3->oUT, dq) = ux * ct2 - uz * st2;
                    at64(A3->oUP, dq) = uy;
                } else {
                    at32(A3->R + base, ql) = r2;
                    at32(A3->TH + base, ql) = th2;
                    at32(A3->UR + base, ql) = ux * st2 + uz * ct2;
                    at32(A3->UT + base, ql) = ux * ct2 - uz * st2;
                    at32(A3->UP + base, ql) = uy;
                }
                // zigzag with both ends in the cell: the two segments share
                // the four faces of the cell, the relay point is the
                // mid-point (both ends lie in [0, 1]), and so is the cell of
                // J_phi unless the mid-point is the far corner itself
                const double xm = 0.5 * (x1 + x2), ym = 0.5 * (y1 + y2);
                simple = di == 0 && dj == 0 && xm < 1.0 && ym < 1.0;
                cross = !simple;
                const KArgs A4 = opaque(A);
                const double Q = A4->p.Q;
                hx = 0.5 * Q * (x2 - x1);
                hy = 0.5 * Q * (y2 - y1);
                q4 = 0.25 * Q * v1;
                if (LDS && cfl) {
                    // outside the patch: straight to the grid
                    const Acc64<false> gacc{nullptr, 0, 0, 0, {A4->J[0], A4->J[1], A4->J[2]},
                                            A4->p.ld};
                    zigzag64(A4, gacc, i, j, di, dj, x1, y1, x2, y2, v1);
                    cross = false;
                }
            }
        }
        // ---- the next particle's state is loaded here, past the part that needs
        // the registers, and travels during the deposit
        // ---- in-cell moves, one cell per 16-lane row and pass: the lanes of a
        // row whose cell is that of the row's first pending lane sum their eight
        // values over the row, and lanes 0..7 of the row add one sum each.  Every
        // pass retires at least the first pending lane of each row, so the loop
        // ends within 16 passes with every in-cell move deposited; when few
        // lanes of the wave are left, they add their values by themselves.
        if (PPT > 1) load(opaque(A0), q + kWG64);
        bool pend = simple;
        const int c = LDS ? i * acc.TJ + j : (i << 16) | j;
        const double X = x1 + x2, Y = y1 + y2;   // twice the mid-point
        unsigned long long m = __ballot(pend);
#pragma unroll 1
        while (m != 0ull) {
            const unsigned rowm = (unsigned)(m >> (lane & 48)) & 0xffffu;
            const int src = rowm ? (lane & 48) + __builtin_ctz(rowm) : lane;
            const int lc = __shfl(c, src, 64);
            const bool part = pend && c == lc;
            double s[8];
            values8_64(part ? hx : 0.0, part ? hy : 0.0, part ? q4 : 0.0, part ? X : 0.0,
                       part ? Y : 0.0, s);
            double pk[4], pp[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                pk[u] = b0 ? s[4 + u] : s[u];
                pp[u] = b0 ? s[u] : s[4 + u];
            }
            const double v = row_sum8_64(pk, pp, b1, b2);
            // a row with pending lanes has participants: its leader
            if ((lane & 8) == 0 && rowm != 0u) {
                if (LDS) {
                    atomicAdd(&acc.tile[lc + kofs], v);
                } else {
                    gadd(&kg[ix(A->p.ld, cell_row(lc) + kdi, (lc & 0xffff) + kdj)], v);
                }
            }
            pend = pend && !part;
            m = __ballot(pend);
            if (__popcll(m) <= kLone64) {
                if (pend) {
                    values8_64(hx, hy, q4, X, Y, s);
                    acc.add(0, i, j, s[0]);
                    acc.add(0, i, j + 1, s[1]);
                    acc.add(1, i, j, s[2]);
                    acc.add(1, i + 1, j, s[3]);
                    acc.add(2, i, j, s[4]);
                    acc.add(2, i + 1, j, s[5]);
                    acc.add(2, i, j + 1, s[6]);
                    acc.add(2, i + 1, j + 1, s[7]);
                }
                break;
            }
        }
        // ---- moves that leave their cell: queued and deposited after the
        // chunk, where one wave takes them all
        const unsigned long long cm = __ballot(cross);
        if (cm != 0ull) {
            int e0 = 0;
            if (lane == 0) e0 = atomicAdd(qn, __popcll(cm));
            e0 = __builtin_amdgcn_readfirstlane(e0);
            if (cross) {
                const int e = e0 + (int)__builtin_amdgcn_mbcnt_hi(
                                       (unsigned)(cm >> 32),
                                       __builtin_amdgcn_mbcnt_lo((unsigned)cm, 0u));
                if (e < kQueue64) {
                    queue[e] = Move64{x1, y1, x2, y2, v1, (i << 16) | j, (di & 0xffff) | (dj << 16)};
                } else {
                    zigzag64(A, acc, i, j, di, dj, x1, y1, x2, y2, v1);
                }
            }
        }
    }
    __syncthreads();
    const int nq = min(*qn, kQueue64);
    for (int e = tid; e < nq; e += kWG64) {
        const Move64 m = queue[e];
        zigzag64(A0, acc, cell_row(m.c), m.c & 0xffff, (int)(short)(m.d & 0xffff), m.d >> 16, m.x1, m.y1,
                 m.x2, m.y2, m.v1);
    }
}

// One workgroup takes PPT particles per thread.  The chunk's cell box is
// that of the single-precision cell guesses with a margin of one cell.
// Four waves per SIMD: 128 VGPRs and a quarter of a CU's LDS each.
//
// Bound by VALU issue (0.87 of the SIMDs' slots at the 2.0 GHz that FP64
// work runs at, 896 instructions a particle, two thirds of them FP64).  5e7
// particles of the 2048^2 sheet: 1.59 to 1.64 ms (2.5 TB/s of its 80 B a particle)
// against 2.60 ms for one particle per thread with the library's divisions,
// roots, sine, logarithm and arctangent and the gather from global memory
// (1751 instructions).  Of the last 0.10 ms, 0.06 came from loading the next
// state past the part that needs the registers, 0.03 from radii, sines and
// cosines in LDS, 0.01 from the deposit's values masked before they are
// formed.  The same sums on the FP64 matrix cores (4x4x4 products by ones in
// place of the DPP rows) took 0.09 ms more, with fewer instructions but a
// longer chain; three waves per SIMD without spills take the same time.
template <int PPT, bool SERIES, bool PLACE>
__global__ void __launch_bounds__(kWG64) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_push64(const Push64Jobs) {
    const KArgs KA = (KArgs)__builtin_amdgcn_kernarg_segment_ptr() + blockIdx.y;
    const auto &A = *KA;
    __shared__ double tile[3 * kTile64];
    __shared__ double fld[6 * kFld64];
    __shared__ double2 rows[kSide64];
    __shared__ double4 cols[kSide64];
    __shared__ Move64 queue[kQueue64];
    __shared__ int box[4];
    __shared__ int qn;
    const auto &p = A.p;
    const int tid = threadIdx.x, lane = tid & 63;
    // PLACE: the slots before the sort (the slot count holds the new order's)
    const int n = min(A.nub, A.nslots[PLACE ? 2 : 0]);
    const int base = (int)blockIdx.x * (kWG64 * PPT);
    if (base >= n) return;    // no slot in the chunk (uniform)
    double rb[PPT], tb[PPT];
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int qs = min(base + k * kWG64 + tid, n - 1);
        rb[k] = at32(A.R + base, (unsigned)(qs - base));
        tb[k] = at32(A.TH + base, (unsigned)(qs - base));
    }
    int imin = 1 << 30, imax = -1, jmin = 1 << 30, jmax = -1;
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        // (a slot past the last repeats the last one's box)
        if (rb[k] > 0.0) {
            const int i = guess_i(KA, rb[k]), j = guess_j(KA, tb[k]);
            imin = min(imin, i); imax = max(imax, i);
            jmin = min(jmin, j); jmax = max(jmax, j);
        }
    }
    if (tid == 0) {
        box[0] = 1 << 30; box[1] = -1; box[2] = 1 << 30; box[3] = -1;
        qn = 0;
    }
    __syncthreads();
    for (int o = 32; o >= 1; o >>= 1) {
        imin = min(imin, __shfl_xor(imin, o, 64));
        imax = max(imax, __shfl_xor(imax, o, 64));
        jmin = min(jmin, __shfl_xor(jmin, o, 64));
        jmax = max(jmax, __shfl_xor(jmax, o, 64));
    }
    if (lane == 0 && imax >= 0) {
        atomicMin(&box[0], imin); atomicMax(&box[1], imax);
        atomicMin(&box[2], jmin); atomicMax(&box[3], jmax);
    }
    __syncthreads();
    if (box[1] < 0) return;   // no live particle in the chunk (uniform)
    // cells of the chunk's particles: the guesses' box and one more
    const int i0 = max(box[0] - 1, 0), i1 = min(box[1] + 1, p.nr - 1);
    const int j0 = max(box[2] - 1, 0), j1 = min(box[3] + 1, p.nth - 1);
    // current patch: rows [i0-1, i1+2], columns [j0-1, j1+2]; field patch:
    // rows [i0-1, i1+1] and columns [j0-1, j1+1] (ghost columns included)
    const int TI = i1 - i0 + 4, TJ = j1 - j0 + 4;
    const int fi0 = max(i0 - 1, 0), fj0 = j0 - 1;
    const int TIf = i1 + 1 - fi0 + 1, TJf = j1 - j0 + 3;
    const bool use_lds = p.lds != 0 && TI * TJ <= kTile64 && TIf * TJf <= kFld64 &&
                         TI <= kSide64 && TJ <= kSide64;
    const int r0 = max(i0 - 1, 0), nrow = min(i1 + 2, p.nr) - r0 + 1;
    Counts64 cnt{0, 0, 0};
    if (use_lds) {
        const int m = TI * TJ;
        for (int e = tid; e < m; e += kWG64) {
            tile[e] = 0.0; tile[kTile64 + e] = 0.0; tile[2 * kTile64 + e] = 0.0;
        }
        const int mf = TIf * TJf;
        for (int e = tid; e < mf; e += kWG64) {
            const int ti = e / TJf, tj = e - ti * TJf;
            const int row = fi0 + ti, col = fj0 + tj;
            // node column, and the half column with its axis ghosts
            const size_t gn = ix(p.ld, row, min(max(col, 0), p.nth));
            const size_t gh = ix(p.ld, row, min(max(col, 0), p.nth - 1));
            const double par = col < 0 || col >= p.nth ? -1.0 : 1.0;
            fld[e * 6 + 0] = A.E[0][gn];
            fld[e * 6 + 1] = par * A.E[1][gh];
            fld[e * 6 + 2] = A.E[2][gn];
            fld[e * 6 + 3] = A.B[0][gh];
            fld[e * 6 + 4] = A.B[1][gn];
            fld[e * 6 + 5] = par * A.B[2][gh];
        }
        for (int e = tid; e < nrow; e += kWG64) {
            const double x = A.p.rn[r0 + e];
            rows[e] = make_double2(x, rcp64(x));
        }
        if (SERIES)
            for (int e = tid; e <= j1 - j0; e += kWG64) cols[e] = A.sct[j0 + e];
        __syncthreads();
        const Patch64 F{fld, fi0, fj0, TJf, Rows64{rows, r0, nrow}, cols};
        const Acc64<true> acc{tile, i0 - 1, j0 - 1, TJ, {A.J[0], A.J[1], A.J[2]}, p.ld};
        push_chunk64<true, PPT, SERIES, PLACE>(KA, F, acc, nullptr, n, base, queue, &qn, cnt);
        __syncthreads();
        for (int e = tid; e < m; e += kWG64) {
            const int ti = e / TJ, tj = e - ti * TJ;
            const int gi = i0 - 1 + ti, gj = j0 - 1 + tj;
            if (gi < 0 || gi > p.nr || gj < 0 || gj > p.nth) continue;
            const size_t gk = ix(p.ld, gi, gj);
            const double w0 = tile[e], w1 = tile[kTile64 + e], w2 = tile[2 * kTile64 + e];
            if (w0 != 0.0) gadd(&A.J[0][gk], w0);
            if (w1 != 0.0) gadd(&A.J[1][gk], w1);
            if (w2 != 0.0) gadd(&A.J[2][gk], w2);
        }
    } else {
        const Acc64<false> acc{nullptr, 0, 0, 0, {A.J[0], A.J[1], A.J[2]}, p.ld};
        // component of the row sum this lane adds (see push_chunk64)
        const int kc = (lane & 1) ? 2 : ((lane & 2) ? 1 : 0);
        double *kg = kc == 0 ? A.J[0] : (kc == 1 ? A.J[1] : A.J[2]);
        push_chunk64<false, PPT, SERIES, PLACE>(KA, Patch64{}, acc, kg, n, base, queue, &qn, cnt);
    }
    int tk = cnt.kill, ts = cnt.star, ta = cnt.abs;
    for (int o = 32; o >= 1; o >>= 1) {
        tk += __shfl_xor(tk, o, 64);
        ts += __shfl_xor(ts, o, 64);
        ta += __shfl_xor(ta, o, 64);
    }
    if (lane == 0) {
        if (tk) atomicAdd(&A.removed[1], (unsigned long long)tk);
        if (ts) atomicAdd(&A.removed[2], (unsigned long long)ts);
        if (ta) atomicAdd(&A.removed[3], (unsigned long long)ta);
    }
}

static Push64Args push64_job(ffpic_ctx *c, int s) {
    ffpic::Species &S = c->sp[s];
    Push64Args A{};
    P64 &p = A.p;
    p.nr = c->nr; p.nth = c->nth; p.ld = c->ld;
    p.rmin = c->d.rmin; p.r_abs = c->d.r_abs; p.dlog = c->dlog; p.dth = c->dth; p.dt = c->dt;
    p.inv_dlog = 1.0 / c->dlog;
    p.inv_dth = 1.0 / c->dth;
    p.girm = (float)(1.0 / c->d.rmin);
    p.gidl = (float)(1.0 / c->dlog);
    p.gidt = (float)(1.0 / c->dth);
    p.dsub = c->sct_dth;
    p.gids = (float)(1.0 / c->sct_dth) * 0.999999f;
    p.rn = c->dtab64[T_RN];
    double qm = S.qm;
    p.Q = (qm > 0 ? 1.0 : -1.0) * S.weight;
    p.wq = c->d.omega_b * qm;
    p.rr = c->d.rr_coef * rr_factor(c) * fabs(qm) * fabs(qm) * fabs(qm);
    p.shell_r = c->d.shell_r;
    p.lds = c->dlog >= 0x1p-20 && c->d.rmin >= 1e-30 && c->d.rmax <= 1e30;   // see guess_i
    A.nub = (int)S.nub;
    const bool place = c->sort_pending[s];
    A.nslots = place ? (const int32_t *)c->sort_tot[s] : c->nslots + s;
    A.kill = c->kill;
    for (int k = 0; k < 3; k++) {
        A.E[k] = (const double *)c->E[k];
        A.B[k] = (const double *)c->B[k];
        A.J[k] = (double *)c->J[k];
    }
    double **a = (double **)S.cur;
    A.R = a[0]; A.TH = a[1]; A.UR = a[2]; A.UT = a[3]; A.UP = a[4];
    if (place) {
        double **o = (double **)S.alt;
        A.dest = c->sort_dest[s];
        A.oR = o[0]; A.oTH = o[1]; A.oUR = o[2]; A.oUT = o[3]; A.oUP = o[4];
    }
    A.sct = (const double4 *)c->fz_colc;
    A.lct = (const double2 *)c->fz_log64;
    A.removed = c->removed + 4 * s;
    A.err = c->err;
    return A;
}

using Push64Kern = void (*)(const Push64Jobs);

template <bool PLACE>
static Push64Kern push64_kern(int ppt, bool series) {
    return !series ? k_push64<1, false, PLACE>
                   : (ppt == 1 ? k_push64<1, true, PLACE>
                               : (ppt == 2 ? k_push64<2, true, PLACE> : k_push64<8, true, PLACE>));
}

void push64(ffpic_ctx *c) {
    // (coarse grids, past the range of the series, take a logarithm of any
    // argument, log_wide, and the library's arctangent)
    const bool series = c->dlog <= 0.0625 && c->dth <= 0.0625;
    for (int place = 0; place < 2; place++) {
        // the species whose kernel is the same share a launch
        Push64Jobs P{};
        int m = 0;
        int64_t most = 0, per = 0;
        for (int s = 0; s < c->d.nspec; s++) {
            const int64_t w = (c->sp[s].nub + kWG64 - 1) / kWG64;
            if (w == 0 || (int)c->sort_pending[s] != place) continue;
            P.job[m++] = push64_job(c, s);
            most = std::max(most, w);
            per += w;
        }
        if (m == 0) continue;
        // eight particles per thread spread a chunk's box, patches and flush
        // over 2048 particles (5e7 particles, 2048^2 sheet: 1.74 ms against
        // 1.80 with four and 1.99 with one); species too small to fill the GPU
        // (1024 workgroups resident) several times that way take fewer per
        // thread (1e5 particles: 11.5 us with one, about 30 with eight)
        const int ppt = !series || per < 8 * 1024 ? 1 : (per < 16 * 1024 ? 2 : 8);
        const Push64Kern kern = place ? push64_kern<true>(ppt, series) : push64_kern<false>(ppt, series);
        hipLaunchKernelGGL(kern, dim3((unsigned)((most + ppt - 1) / ppt), m), dim3(kWG64), 0,
                           c->stream, P);
        FFPIC_LAUNCH_CHECK();
    }
    for (int s = 0; s < c->d.nspec; s++) after_push(c, s);
}

}  // namespace ffpic
