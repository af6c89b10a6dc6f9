// Species spectra over a region of the meridional plane (the observables of
// Sect. 5): the Lorentz-factor histogram, the leading power of the
// radiation-reaction force, P = K gamma^2 Bperp^2 (eq. bperp), and the
// synchrotron spectral energy distribution, each particle emitting the
// single-particle synchrotron spectrum normalised to its P:
//   nu dP/dnu = P x F(x) 9 sqrt(3) / (8 pi),  x = nu / nu_c,
//   nu_c = 3/(4 pi) gamma^2 omega_b |qm| Bperp,
// F(x) = x int_x^inf K_{5/3} the synchrotron function.
//
// A workgroup takes 768 slots at a time.  Each thread decodes one particle,
// bins gamma into an LDS histogram, gathers E and B at the particle (the
// interpolation of the FP64 push, in FP64 also for the FP32 fields) and
// lists its P and nu_c in LDS; then the threads share the (frequency, listed
// particle) pairs: a thread keeps one frequency and sums every S-th particle
// of the list for it, S = 768 / nnu.  The block adds its partial sums to the
// output with one global atomic per bin when it has no slots left.
//
// F comes from a table of ln F on a uniform grid in ln x over
// [1e-8, 100], built once by quadrature of
//   F(x) = x int_0^inf exp(-x cosh t) cosh(5t/3) / cosh t dt
// (the representation K_nu(s) = int_0^inf exp(-s cosh t) cosh(nu t) dt
// integrated over s), and interpolated linearly in (ln x, ln F); below the
// table F follows its x^(1/3) law, above it F < 1e-40 is taken as 0.
// The interpolation is evaluated as F_k exp(fr d_k), d_k = ln F_{k+1} -
// ln F_k in (-0.29, 0.001], with a polynomial for the exponential (its
// remainder is below 2e-14, and below 1e-16 for x < 40), ln x = ln nu -
// ln nu_c and x^(1/3) = nu^(1/3) nu_c^(-1/3) with the logarithms and cube
// roots taken once per frequency and particle.  Pairs (F_k, d_k) fill
// 128 KB of LDS, one workgroup per CU: the lanes of a wave read scattered
// entries, which a table in the cache serves a few lanes a clock.
//
// Bound by FP64 issue: about 36 instructions per pair (0.14 of the 0.34 ms),
// then by the latency of the decode, with 12 waves per CU.  2e6 particles of
// the 1024^2 sheet, 60 bins and 80 frequencies: 0.34 ms against 1.72 ms with
// a logarithm and an exponential per pair and one thread per frequency.
#include <algorithm>
#include <cmath>

#include "gather.h"

namespace ffpic {

namespace {

constexpr int kSpecWG = 768;             // threads, and slots per round
constexpr int kSyncN = 8192;
constexpr double kSyncX0 = 1e-8, kSyncX1 = 100.0;

struct SpecArgs {
    int nr, nth, ld, ngamma, nnu;
    double rmin, dlog, dth;
    const double *rn, *thn;
    double r0, r1, t0, t1;          // region
    double gmin, dlg;               // gamma bins
    const double *edge;             // ngamma + 1 edges
    const double *nu;               // nnu frequencies, their logarithms, F of the
                                    // x^(1/3) law at nu_c = 1
    double w, K, wb;                // weight, radiation-reaction coefficient, omega_b |qm|
    const double2 *tab;             // F_k, ln F_{k+1} - ln F_k
    double lx0, ihx;                // ln of the first abscissa, 1 / spacing
};

// exp(y) for -0.29 < y < 0.01: the Taylor polynomial through y^11
__device__ __forceinline__ double exp_small(double y) {
    double e = 1.0 / 39916800.0;
    e = __builtin_fma(e, y, 1.0 / 3628800.0);
    e = __builtin_fma(e, y, 1.0 / 362880.0);
    e = __builtin_fma(e, y, 1.0 / 40320.0);
    e = __builtin_fma(e, y, 1.0 / 5040.0);
    e = __builtin_fma(e, y, 1.0 / 720.0);
    e = __builtin_fma(e, y, 1.0 / 120.0);
    e = __builtin_fma(e, y, 1.0 / 24.0);
    e = __builtin_fma(e, y, 1.0 / 6.0);
    e = __builtin_fma(e, y, 0.5);
    e = __builtin_fma(e, y, 1.0);
    return __builtin_fma(e, y, 1.0);
}

// what the frequency sums need of a particle
struct Emitter {
    double P, inuc, lnuc, cnuc;     // power, 1 / nu_c, ln nu_c, nu_c^(-1/3)
};

template <bool FP64, typename T>
__global__ void __launch_bounds__(kSpecWG)
    k_spectra(SpecArgs A, int nub, const int32_t *__restrict__ nslots, const void *s0,
              const void *s1, const void *s2, const void *s3, const void *s4, const void *s5,
              const T *__restrict__ Er, const T *__restrict__ Et, const T *__restrict__ Ep,
              const T *__restrict__ Br, const T *__restrict__ Bt, const T *__restrict__ Bp,
              double *__restrict__ out) {
    __shared__ double2 tab[kSyncN];
    __shared__ Emitter list[kSpecWG];
    __shared__ double hist[FFPIC_SPEC_MAX], sed[FFPIC_SPEC_MAX];
    __shared__ int wcnt[kSpecWG / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = min(nub, nslots[0]);
    const int rounds = (n + kSpecWG - 1) / kSpecWG;
    if ((int)blockIdx.x >= rounds) return;
    for (int k = tid; k < kSyncN; k += kSpecWG) tab[k] = A.tab[k];
    for (int m = tid; m < FFPIC_SPEC_MAX; m += kSpecWG) hist[m] = sed[m] = 0.0;
    // this thread's frequency and its share of the list
    const int S = kSpecWG / A.nnu, f = tid % A.nnu, sl = tid / A.nnu;
    const double nu = A.nu[f], lnu = A.nu[A.nnu + f], fcb = A.nu[2 * A.nnu + f];
    double acc = 0.0, psum = 0.0;
    __syncthreads();
    for (int rd = blockIdx.x; rd < rounds; rd += gridDim.x) {
        const int q = rd * kSpecWG + tid;
        double P = 0.0, nuc = 0.0;
        bool in = false;
        int i = 0, j = 0;
        double a = 0.0, b = 0.0, r = 0.0, th = 0.0, u0 = 0.0, u1 = 0.0, u2 = 0.0;
        if (q < n) {
            if (FP64) {
                r = ((const double *)s0)[q];
                if (r > 0.0) {
                    th = ((const double *)s1)[q];
                    in = r >= A.r0 && r < A.r1 && th >= A.t0 && th < A.t1;
                    if (in) {
                        locate64(A.nr, A.nth, A.rmin, A.dlog, A.dth, A.rn, A.thn, r, th, i, j,
                                 a, b);
                        u0 = ((const double *)s2)[q];
                        u1 = ((const double *)s3)[q];
                        u2 = ((const double *)s4)[q];
                    }
                }
            } else {
                const int c = ((const int32_t *)s0)[q];
                if (cell_live(c)) {
                    i = cell_row(c);
                    j = c & 0xffff;
                    a = (double)((const float *)s1)[q];
                    b = (double)((const float *)s2)[q];
                    r = A.rn[i] * exp(a * A.dlog);
                    th = A.thn[j] + b * A.dth;
                    in = r >= A.r0 && r < A.r1 && th >= A.t0 && th < A.t1;
                    if (in) {
                        u0 = (double)((const float *)s3)[q];
                        u1 = (double)((const float *)s4)[q];
                        u2 = (double)((const float *)s5)[q];
                    }
                }
            }
        }
        if (in) {
            const double g = sqrt(1.0 + u0 * u0 + u1 * u1 + u2 * u2);
            // log bin, settled against the edge table
            int m = (int)floor(log(g / A.gmin) / A.dlg);
            if (m < 0) m = 0;
            if (m > A.ngamma - 1) m = A.ngamma - 1;
            while (m > 0 && g < A.edge[m]) m--;
            while (m < A.ngamma - 1 && g >= A.edge[m + 1]) m++;
            if (g >= A.edge[m] && g < A.edge[m + 1]) atomicAdd(&hist[m], A.w);
            double E[3], B[3];
            gather_eb(Er, Et, Ep, Br, Bt, Bp, A.nr, A.nth, A.ld, i, j, a, b, E, B);
            const double be0 = u0 / g, be1 = u1 / g, be2 = u2 / g;
            const double F0 = E[0] + (be1 * B[2] - be2 * B[1]);
            const double F1 = E[1] + (be2 * B[0] - be0 * B[2]);
            const double F2 = E[2] + (be0 * B[1] - be1 * B[0]);
            const double be = be0 * E[0] + be1 * E[1] + be2 * E[2];
            double bp2 = F0 * F0 + F1 * F1 + F2 * F2 - be * be;
            if (bp2 < 0.0) bp2 = 0.0;
            P = A.K * g * g * bp2;
            nuc = 3.0 / (4.0 * 3.14159265358979323846) * g * g * A.wb * sqrt(bp2);
            psum += A.w * P;
        }
        // the emitting particles, listed in slot order
        const bool emits = P > 0.0 && nuc > 0.0;
        const unsigned long long m = __ballot(emits);
        if (lane == 0) wcnt[wave] = __popcll(m);
        __syncthreads();
        int at = (int)__popcll(m & ((1ull << lane) - 1ull)), cnt = 0;
#pragma unroll
        for (int v = 0; v < kSpecWG / 64; v++) {
            if (v < wave) at += wcnt[v];
            cnt += wcnt[v];
        }
        if (emits) list[at] = Emitter{P, 1.0 / nuc, log(nuc), 1.0 / cbrt(nuc)};
        __syncthreads();
        if (sl < S) {
            for (int e = sl; e < cnt; e += S) {
                const Emitter p = list[e];
                const double x = nu * p.inuc, s = (lnu - p.lnuc - A.lx0) * A.ihx;
                const int k = min(max((int)s, 0), kSyncN - 1);
                const double2 t = tab[k];
                double F = t.x * exp_small((s - (double)k) * t.y);
                if (s < 0.0) F = fcb * p.cnuc;
                // past the table nothing is added (x may be infinite there)
                const double v = p.P * x * F;
                acc += s < (double)(kSyncN - 1) ? v : 0.0;
            }
        }
        __syncthreads();
    }
    if (sl < S && acc != 0.0) atomicAdd(&sed[f], acc);
    for (int o = 32; o >= 1; o >>= 1) psum += __shfl_xor(psum, o, 64);
    if (lane == 0 && psum != 0.0) gadd(&out[A.ngamma + A.nnu], psum);
    __syncthreads();
    for (int m = tid; m < A.ngamma; m += kSpecWG)
        if (hist[m] != 0.0) gadd(&out[m], hist[m]);
    for (int m = tid; m < A.nnu; m += kSpecWG)
        if (sed[m] != 0.0)
            gadd(&out[A.ngamma + m],
                 sed[m] * A.w * (9.0 * 1.7320508075688772 / (8.0 * 3.14159265358979323846)));
}

__global__ void k_spec_zero(double *p, int n) {
    for (int q = threadIdx.x; q < n; q += 256) p[q] = 0.0;
}

// The table: F(x) = x int_0^inf exp(-x cosh t) cosh(5t/3) / cosh t dt by the
// trapezoidal rule in t (geometric convergence for this even analytic
// integrand), one wave per abscissa, its lanes sharing the terms (up to
// about 1600).  Built by the GPU on a context's first request: 80 ms on the
// host.
__global__ void __launch_bounds__(256) k_sync_table(double l0, double l1, double2 *tab,
                                                    double *lnF) {
    const int k = (int)((blockIdx.x * 256 + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    const double h = 1.0 / 64.0, x = exp(l0 + (l1 - l0) * k / (kSyncN - 1));
    double sum = 0.0;
    for (int u = lane;; u += 64) {
        const double t = u * h, ch = cosh(t);
        if (x * ch > 745.0) break;
        sum += (u == 0 ? 0.5 : 1.0) * exp(-x * ch) * cosh(t * (5.0 / 3.0)) / ch;
    }
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) {
        const double F = x * h * sum;
        tab[k].x = F;
        lnF[k] = log(F);
    }
}
__global__ void __launch_bounds__(256) k_sync_slopes(const double *lnF, double2 *tab) {
    const int k = (int)(blockIdx.x * 256 + threadIdx.x);
    tab[k].y = k + 1 < kSyncN ? lnF[k + 1] - lnF[k] : 0.0;
}

void *dev_alloc(size_t bytes) {
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        throw std::bad_alloc();
    }
    return p;
}

}  // namespace

void spectra(ffpic_ctx *c, int s, const ffpic_spectra_req *rq, double *dev_out) {
#pragma clang fp contract(off)
    const int ng = rq->ngamma, nn = rq->nnu;
    if (c->spec_f0 == 0.0) {
        // (spec_edge also lends its place to ln F while the table is built)
        static_assert(kSyncN % 256 == 0 && kSyncN >= 4 * FFPIC_SPEC_MAX + 1, "whole blocks, room");
        if (!c->spec_edge) c->spec_edge = (double *)dev_alloc(kSyncN * sizeof(double));
        if (!c->spec_tab) c->spec_tab = (double *)dev_alloc(kSyncN * sizeof(double2));
        double *edge = c->spec_edge;
        double2 *tab = (double2 *)c->spec_tab;
        hipLaunchKernelGGL(k_sync_table, dim3(kSyncN / 4), dim3(256), 0, c->stream,
                           std::log(kSyncX0), std::log(kSyncX1), tab, edge);
        hipLaunchKernelGGL(k_sync_slopes, dim3(kSyncN / 256), dim3(256), 0, c->stream, edge, tab);
        FFPIC_LAUNCH_CHECK();
        if (hipMemcpyAsync(&c->spec_f0, tab, sizeof(double), hipMemcpyDeviceToHost, c->stream) !=
                hipSuccess ||
            hipStreamSynchronize(c->stream) != hipSuccess)
            throw std::runtime_error("reading back the synchrotron table failed");
    }
    // bin edges and frequencies in FP64 on the host
    // (kept in the context, so that they outlive the asynchronous copy: the
    // call ends with a synchronisation)
    std::vector<double> &h = c->spec_host;
    h.resize(ng + 1 + 3 * nn);
    const double dlg = std::log(rq->gmax / rq->gmin) / ng;
    for (int m = 0; m <= ng; m++) h[m] = rq->gmin * std::exp(m * dlg);
    for (int m = 0; m < nn; m++) {
        const double nu = nn > 1 ? rq->numin * std::exp(m * std::log(rq->numax / rq->numin) / (nn - 1))
                                 : rq->numin;
        h[ng + 1 + m] = nu;
        h[ng + 1 + nn + m] = std::log(nu);
        h[ng + 1 + 2 * nn + m] = c->spec_f0 * std::cbrt(nu / kSyncX0);
    }
    if (hipMemcpyAsync(c->spec_edge, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice,
                       c->stream) != hipSuccess)
        throw std::runtime_error("spectra set-up copy failed");
    hipLaunchKernelGGL(k_spec_zero, dim3(1), dim3(256), 0, c->stream, dev_out, ng + nn + 1);
    FFPIC_LAUNCH_CHECK();
    const ffpic::Species &S = c->sp[s];
    if (S.nub == 0) return;
    SpecArgs A{};
    A.nr = c->nr; A.nth = c->nth; A.ld = c->ld; A.ngamma = ng; A.nnu = nn;
    A.rmin = c->d.rmin; A.dlog = c->dlog; A.dth = c->dth;
    A.rn = c->dtab64[T_RN]; A.thn = c->dtab64[T_THN];
    A.r0 = rq->rmin; A.r1 = rq->rmax; A.t0 = rq->thmin; A.t1 = rq->thmax;
    A.gmin = rq->gmin; A.dlg = dlg; A.edge = c->spec_edge; A.nu = c->spec_edge + ng + 1;
    const double qm = S.qm;
    A.w = S.weight;
    A.K = c->d.rr_coef * rr_factor(c) * std::fabs(qm) * std::fabs(qm) * std::fabs(qm);
    A.wb = c->d.omega_b * std::fabs(qm);
    A.tab = (const double2 *)c->spec_tab;
    A.lx0 = std::log(kSyncX0);
    A.ihx = (kSyncN - 1) / (std::log(kSyncX1) - std::log(kSyncX0));
    // one workgroup per CU (its table takes 128 of the CU's 160 KB of LDS)
    const int nb = (int)std::min<int64_t>((S.nub + kSpecWG - 1) / kSpecWG, 256);
    void *const *a = S.cur;
    if (c->fp64) {
        double *const *E = (double *const *)c->E, *const *B = (double *const *)c->B;
        hipLaunchKernelGGL((k_spectra<true, double>), dim3(nb), dim3(kSpecWG), 0, c->stream, A,
                           (int)S.nub, c->nslots + s, a[0], a[1], a[2], a[3], a[4], a[4], E[0],
                           E[1], E[2], B[0], B[1], B[2], dev_out);
    } else {
        float *const *E = (float *const *)c->E, *const *B = (float *const *)c->B;
        hipLaunchKernelGGL((k_spectra<false, float>), dim3(nb), dim3(kSpecWG), 0, c->stream, A,
                           (int)S.nub, c->nslots + s, a[0], a[1], a[2], a[3], a[4], a[5], E[0],
                           E[1], E[2], B[0], B[1], B[2], dev_out);
    }
    FFPIC_LAUNCH_CHECK();
}

}  // namespace ffpic
