// FP32-mixed particle push and charge-conserving deposit.
//
// Particle state (SoA, 24 B): cell = (i << 16) | j (int32, negative from row
// 32768 on; -1 = dead slot),
// a = in-cell offset in log r / dlog, b = in-cell offset in theta / dtheta
// (FP32, in [0, 1)), u_r, u_theta, u_phi (FP32).  Splitting the position
// into an integer cell and a small FP32 offset keeps 2^-24 of a cell of
// resolution anywhere on the grid, where an absolute FP32 coordinate would
// lose several digits at r ~ 100.
//
// Physics as in the FP64 path (Sect. 3, eq. motion with the
// radiation-reaction force g and eq. bperp; Boris rotation; zigzag
// charge-conserving deposit), but the move is evaluated in the particle's
// local frame: the radial and polar displacements are formed from the
// small step itself (a log1p series for the radial one, an arctangent
// series for the polar one), so that no difference of two large FP32
// coordinates is ever taken.  Reciprocals and square roots use the
// hardware approximations (about 1 ulp).
//
// What bounds it.  From some 1e8 particles on, HBM: the 9.6 GB of state of 2e8
// particles on 4096^2 (11.3 GB of traffic) take 2.07 ms in the first steps of
// the sheet and 2.24 some fifty steps on, 5.0 to 5.4 TB/s, where a copy of the
// state takes 1.93 to 2.01 (4.8 to 5.0 TB/s from box to box); VALU issue is
// close behind (356 instructions a particle).  The earlier form (weights and
// node pairs for the gather, Cartesian move, 456 instructions) took 2.29 and
// 2.58.  So it is written for few and
// cheap instructions, and waits for nothing it need not: the loads of the
// next particle, which every lane makes, are waited for without the stores
// that follow them, index products use 24-bit multiplies, and the cross-lane
// sums are DPP row reductions.  Smaller species are bound by the
// chain of a workgroup's rounds and by the tail of the launch, hence shorter
// chunks (push_ppt).
//
// Gather: each workgroup takes a contiguous chunk of the (cell-sorted)
// particle array, finds the bounding box of its cells and builds in LDS, for
// every cell of the box with one of margin before it, the coefficients of each
// component's bilinear form on its own staggered cell (ghost rows and columns
// of the radial ends and the axes, with their signs, included).  A component
// is then one 16-byte LDS read and three fused multiply-adds, where weights,
// signs and two pairs of nodes were some twelve instructions.
//
// Deposit: the currents accumulate in a second LDS patch covering the box
// plus the one-cell reach of a step; the patch is then flushed to the FP32
// current arrays in HBM with one global atomic per non-zero entry.
// Particles that stay in their cell are summed across each 16-lane row
// first (DPP), one cell per row and pass, so a sorted wave issues one add
// instruction from 32 lanes (eight sums in each of four rows) per pass
// instead of eight from all 64; when few lanes are left they add their eight
// values each.  Moves that leave their cell (a few
// per cent of a step) are queued in LDS and deposited after the chunk, so the
// zigzag runs in one wave per chunk rather than in nearly every wave.
// A chunk whose box is too large for the patches is taken in parts with a box
// each; a part that is still too large (sparse regions) gathers
// from HBM through buffer resources and adds straight to HBM.
#include <algorithm>
#include <cstring>

#include "device_common.h"

namespace ffpic {

constexpr int kWG = 256;
constexpr int kMaxChunk = 32 * kWG;      // slots of a chunk, at most
static_assert(kStatePad >= kMaxChunk, "lanes past the last slot");
constexpr int kCells = 208;              // cells of the LDS field patch
constexpr int kTile = 448;               // LDS deposit patch entries per component
constexpr int kPart = 4;                 // rounds of a part of a chunk with a large box
constexpr int kLone = 8;                 // in-cell moves left in a wave that add by themselves
constexpr int kQueue = 64;               // queued cell-crossing moves per workgroup
constexpr int kRsrcWord3 = 0x00020000;   // raw dword buffer access (gfx9 family)

struct P32 {
    int nr, nth, ld;
    float dlog, dth, dt, inv_dlog, inv_dth;
    int iabs;                            // r_abs lies in radial cell iabs ...
    float aabs;                          // ... at offset aabs
    const float *rn, *sn, *cn;
    float Q, h, kk;                      // charge, dt omega_b qm / 2, dt K_s
    float weps;                          // 1e-9 of a step, see the move
    int ishell;                          // the shell of kept momentum along B ends in
    float ashell;                        // radial cell ishell at offset ashell
};

__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float frsq(float x) { return __builtin_amdgcn_rsqf(x); }
// index products: both factors are grid or patch indices below 2^24 and the
// products stay below 2^32, so the full-rate 24-bit multiply is exact
__device__ __forceinline__ unsigned mul24(int x, unsigned y) { return __umul24((unsigned)x, y); }

// 32-bit element offsets from a uniform base (element index < 2^30)
template <typename T>
__device__ __forceinline__ T ldo(const T *base, unsigned idx) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + (idx << 2));
}
template <typename T>
__device__ __forceinline__ void sto(T *base, unsigned idx, T v) {
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + (idx << 2)) = v;
}

// a b + c d + e
__device__ __forceinline__ float fma3(float a, float b, float c, float d, float e) {
    return __builtin_fmaf(a, b, __builtin_fmaf(c, d, e));
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Sums eight per-lane values over each 16-lane row, halving the number of
// values at every stage: a rotation by eight lanes (lanes 0..7 of the row keep
// values 0..3, the others 4..7), a mirror of each half row (quads 0 and 2 keep
// the first two, 1 and 3 the others), then an exchange with lane^1 (odd lanes
// keep the second) and with lane^2.  The bank masks write each half of a
// stage's sums where they are kept, with no select; the rows of a stage follow
// the last write of their operands by the two instructions that a DPP read
// has to.  Lane l then holds the row sum of value 4 bit3(l) + 2 bit2(l) +
// bit0(l); lanes l and l ^ 2 hold the same.  All lanes are active.
__device__ __forceinline__ float row_sum8(float s[8], bool b0) {
    float z0, z1;
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %4, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %5, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %4, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %5, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %4, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %5, %5, %5 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
        : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]), "=&v"(z0), "=&v"(z1)
        : "v"(s[4]), "v"(s[5]), "v"(s[6]), "v"(s[7]));
    const float w = b0 ? z1 : z0;
    return w + dpp<0x4E>(w);
}

// value (0..7) whose row sum a lane holds after row_sum8, and its component
// (0 = J_r, 1 = J_theta, 2 = J_phi): values 0, 1 are J_r, 2, 3 J_theta, 4..7 J_phi
__device__ __forceinline__ int lane_value(int lane) {
    return ((lane & 8) ? 4 : 0) + ((lane & 4) ? 2 : 0) + (lane & 1);
}
__device__ __forceinline__ int lane_comp(int lane) {
    const int kq = lane_value(lane);
    return kq < 2 ? 0 : (kq < 4 ? 1 : 2);
}

struct Fields {
    __amdgpu_buffer_rsrc_t er, et, ep, br, bt, bp;
};

// particle state arrays: 32-bit byte offsets (slot * 4) from uniform bases,
// so no 64-bit address is formed per access
struct State {
    int32_t *cell;
    float *a, *b, *ur, *ut, *up;
    __device__ __forceinline__ static float ld(const float *R, unsigned q) { return ldo(R, q); }
    __device__ __forceinline__ static void st(float *R, unsigned q, float v) { sto(R, q, v); }
    __device__ __forceinline__ int ldc(unsigned q) const { return ldo(cell, q); }
    __device__ __forceinline__ void stc(unsigned q, int v) const { sto(cell, q, v); }
};

template <bool LDS>
struct Acc {
    float *tile;     // LDS patch (LDS mode)
    int ti0, tj0, TJ;
    float *g[3];
    int ld;
    __device__ __forceinline__ void add(int comp, int i, int j, float v) const {
        if (LDS) atomicAdd(&tile[comp * kTile + mul24(i - ti0, TJ) + (j - tj0)], v);
        else gadd(reinterpret_cast<float *>(reinterpret_cast<char *>(g[comp]) +
                                            ((mul24(i, ld) + (unsigned)j) << 2)), v);
    }
};

struct PushJob;
// a job as the kernels find it in constant memory (the single launch's
// argument, the grouped launch's table): each phase takes its address anew
// (opaque), so that values of one phase are not held in scalar registers, or
// spilled to lanes of vector registers, across the particle loop
typedef const __attribute__((address_space(4))) PushJob *KJob;

template <typename P>
__device__ __forceinline__ P opaque(P t) {
    asm volatile("" : "+s"(t));
    return t;
}

// A cell of the LDS field patch: per component the bilinear form of its own
// staggered cell, c0 + c1 y + x (c2 + c3 y) in the fractions x, y of that
// cell, then the geometry of the grid cell and its kill flag.
struct PatchCell {
    float4 c[6];                         // E_r, E_th, E_ph, B_r, B_th, B_ph
    float4 geo;                          // r_i, sin theta_j, cos theta_j, kill flag
};
static_assert(sizeof(PatchCell) == 112, "byte offsets in the gather");
constexpr unsigned kCellB = sizeof(PatchCell);

// coefficients of the bilinear form through four values
__device__ __forceinline__ float4 form4(float v00, float v01, float v10, float v11) {
    return make_float4(v00, v01 - v00, v10 - v00, (v11 - v10) - (v01 - v00));
}
__device__ __forceinline__ float form(float4 c, float x, float y) {
    return __builtin_fmaf(x, __builtin_fmaf(c.w, y, c.z), __builtin_fmaf(c.y, y, c.x));
}
__device__ __forceinline__ float4 cell_form(const char *fld, unsigned o, int comp) {
    return reinterpret_cast<const float4 *>(fld + o)[comp];
}
// the same from HBM: rows at element offsets r0, r1, columns c0, c1 with signs
__device__ __forceinline__ float4 corners(__amdgpu_buffer_rsrc_t R, unsigned r0, unsigned r1,
                                          unsigned c0, unsigned c1, float o0, float o1) {
    auto at = [&](unsigned k) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(R, (int)(k << 2), 0, 0));
    };
    return form4(o0 * at(r0 + c0), o1 * at(r0 + c1), o0 * at(r1 + c0), o1 * at(r1 + c1));
}

struct Patch {
    const char *fld;                     // LDS field patch (LDS mode)
    unsigned rowB;                       // bytes per patch row
    int key0;                            // key (i * TJ + j) of its first cell
};

struct ChunkArgs {
    int n, base, iters;                  // slot count, first slot, rounds of kWG slots
    int cell0;                           // a cell of the box
    int tid, lane;
    float4 *queue;
    int *qn;
};

// Everything one push of one species reads from the host, by value: the
// single-system kernel takes it as its argument, the grouped kernel reads
// each system's from a table in device memory.
struct PushJob {
    P32 p;
    int nub;                             // slot bound known to the host
    int ppt;                             // particles per thread of a chunk
    const int32_t *nslots;               // slot count on the device
    const uint8_t *kill;
    const float *E[3], *B[3];
    int32_t *cell;
    float *a, *b, *ur, *ut, *up;
    float *J[3];
    unsigned long long *removed;         // this species' removal counters
    uint32_t *err;
    SortPlace SP;                        // placing push: where each slot goes
};

// zigzag (relay-point) deposit of a move from (x1, y1) in cell (i, j) to
// (x2, y2) in the same frame, ending in cell (i + di, j + dj): the radial and
// polar charge fluxes of the two straight segments, and J_phi at the midpoint
template <bool LDS>
__device__ __forceinline__ void zigzag(KJob A, const Acc<LDS> &acc, int i, int j, int di,
                                       int dj, float x1, float y1, float x2, float y2, float qv) {
    const int nr = A->p.nr, nth = A->p.nth;
    const int i2 = i + di, j2 = j + dj;
    const float xr = fminf((float)min(di, 0) + 1.f, fmaxf((float)max(di, 0), 0.5f * (x1 + x2)));
    const float yr = fminf((float)min(dj, 0) + 1.f, fmaxf((float)max(dj, 0), 0.5f * (y1 + y2)));
    const float Q = A->p.Q;
    const float fx1 = Q * (xr - x1), fy1 = Q * (yr - y1);
    const float fx2 = Q * (x2 - xr), fy2 = Q * (y2 - yr);
    const float wx1 = 0.5f * (x1 + xr), wy1 = 0.5f * (y1 + yr);
    const float wx2 = 0.5f * (xr + x2) - (float)di, wy2 = 0.5f * (yr + y2) - (float)dj;
    acc.add(0, i, j, fx1 * (1.f - wy1));
    acc.add(0, i, j + 1, fx1 * wy1);
    acc.add(1, i, j, fy1 * (1.f - wx1));
    acc.add(1, i + 1, j, fy1 * wx1);
    acc.add(0, i2, j2, fx2 * (1.f - wy2));
    acc.add(0, i2, j2 + 1, fx2 * wy2);
    acc.add(1, i2, j2, fy2 * (1.f - wx2));
    acc.add(1, i2 + 1, j2, fy2 * wx2);
    const float xm = 0.5f * (x1 + x2), ym = 0.5f * (y1 + y2);
    int im = (int)floorf(xm), jm = (int)floorf(ym);
    if (i + im > nr - 1) im = nr - 1 - i;
    if (j + jm > nth - 1) jm = nth - 1 - j;
    const float wx = xm - (float)im, wy = ym - (float)jm;
    const float qq = Q * qv;
    acc.add(2, i + im, j + jm, qq * (1.f - wx) * (1.f - wy));
    acc.add(2, i + im + 1, j + jm, qq * wx * (1.f - wy));
    acc.add(2, i + im, j + jm + 1, qq * (1.f - wx) * wy);
    acc.add(2, i + im + 1, j + jm + 1, qq * wx * wy);
}

// the eight adds of a move inside its cell: hx, hy half the radial and polar
// charge flux, q4 a quarter of the azimuthal one, X, Y twice the midpoint
__device__ __forceinline__ void values8(float hx, float hy, float q4, float X, float Y,
                                        float s[8]) {
    s[1] = hx * Y;
    s[0] = 2.f * hx - s[1];
    s[3] = hy * X;
    s[2] = 2.f * hy - s[3];
    const float u = q4 * X, z = 2.f * q4 - u;
    s[7] = u * Y;
    s[5] = 2.f * u - s[7];
    s[6] = z * Y;
    s[4] = 2.f * z - s[6];
}

template <bool LDS, bool SHELL, bool PLACE>
__device__ __forceinline__ void push_chunk(KJob A0, const Fields &F, const Patch &P,
                                           const Acc<LDS> &acc, const ChunkArgs &C, int &nkill,
                                           int &nstar, int &nabs, float *kg) {
    const KJob A = opaque(A0);
    const int n = C.n, base = C.base, tid = C.tid, lane = C.lane;
    // the chunk's slots: offsets from its first one, so that slots past a
    // capacity of 2^30 stay within 32-bit byte offsets
    const State S{A->cell + base, A->a + base, A->b + base, A->ur + base, A->ut + base,
                  A->up + base};
    const int32_t *dest = PLACE ? A->SP.dest + base : nullptr;
    // the constants of the particle loop
    const float dlog = A->p.dlog, dth = A->p.dth, dt = A->p.dt, h = A->p.h, kk = A->p.kk;
    const float weps = A->p.weps;
    const float inv_dlog = A->p.inv_dlog, inv_dth = A->p.inv_dth;
    const float Q2 = 0.5f * A->p.Q, Qp4 = 0.25f * A->p.Q / dt;
    const int nth = A->p.nth, iabs = A->p.iabs;
    // the deposit value this lane adds after the row reduction: component,
    // radial and polar node offsets from the cell (values 0..7 as below)
    const bool b0 = lane & 1;
    const int kq = lane_value(lane), kcomp = lane_comp(lane);
    const int kdi = (kq == 3 || kq == 5 || kq == 7) ? 1 : 0;
    const int kdj = (kq == 1 || kq == 6 || kq == 7) ? 1 : 0;
    const bool row_lead = (lane & 2) == 0;
    const float kscale = kcomp == 2 ? Qp4 : Q2;
    const int row0 = lane & 48;
    // LDS mode: a cell's key in the current patch is i * TJ + j (unique over
    // the patch's cells), and the entry this lane adds to after a row sum
    // lies kofs entries from it
    const int kofs = LDS ? kcomp * kTile + kdi * acc.TJ + kdj - acc.ti0 * acc.TJ - acc.tj0 : 0;
    // The next particle's state is loaded one iteration ahead.  Loads and
    // stores are made by every lane in every round (past the last slot into
    // the arrays' padding, see kStatePad), with no branch around them: the
    // compiler then knows how many stores follow a load, and the wait for the
    // load does not also wait for them.
    unsigned q = (unsigned)tid;
    int cn = S.ldc(q), dn = -1;
    if constexpr (PLACE) dn = ldo(dest, q);
    float an = State::ld(S.a, q), bn = State::ld(S.b, q);
    float urn = State::ld(S.ur, q), utn = State::ld(S.ut, q), upn = State::ld(S.up, q);
#pragma unroll 1
    for (int k = 0; k < C.iters; k++, q += kWG) {
        int c = cn;
        // PLACE: the slot's place in the new order (-1: no particle of it)
        const int dq = dn;
        const float a = an, b = bn, ur = urn, ut = utn, up = upn;
        {
            const unsigned qn = k + 1 < C.iters ? q + kWG : q;
            cn = S.ldc(qn);
            if constexpr (PLACE) dn = ldo(dest, qn);
            an = State::ld(S.a, qn);
            bn = State::ld(S.b, qn);
            urn = State::ld(S.ur, qn);
            utn = State::ld(S.ut, qn);
            upn = State::ld(S.up, qn);
        }
        if (base + (k + 1) * kWG > n) {        // the last slots (uniform)
            asm volatile("");                  // keeps it a branch
            if (base + (int)q >= n) c = -1;
        }
        const bool live = PLACE ? cell_live(c) && dq >= 0 : cell_live(c);
        // a lane without a particle computes in a cell of the box
        const int cc = live ? c : C.cell0;
        const int i = cell_row(cc), j = cc & 0xffff;
        const int ckey = LDS ? (int)mul24(i, (unsigned)acc.TJ) + j : cc;
        bool simple = false;       // stays in its cell: 8 adds at fixed offsets
        bool cross = false;        // leaves its cell: general zigzag
        int di, dj;
        float na, nb;              // the end point in the cell's frame
        float hx, hy, q4, qv;
        {
            // ---- staggered bilinear gather: x, y in the half-shifted cells
            const bool ah = a >= 0.5f, bh = b >= 0.5f;
            const float xh = a + (ah ? -0.5f : 0.5f), yh = b + (bh ? -0.5f : 0.5f);
            float esr, est, esp, bsr, bst, bsp, rn_i, sn_j, cn_j;
            bool killed;
            if constexpr (LDS) {
                const unsigned on = __umul24((unsigned)(ckey - P.key0), kCellB);
                const unsigned os = bh ? on : on - kCellB;           // shifted in theta
                const unsigned sr = ah ? 0u : P.rowB;                // shift in r
                const unsigned oh = on - sr, oq = os - sr;
                esr = form(cell_form(P.fld, oh, 0), xh, b);
                est = form(cell_form(P.fld, os, 1), a, yh);
                esp = form(cell_form(P.fld, on, 2), a, b);
                bsr = form(cell_form(P.fld, os, 3), a, yh);
                bst = form(cell_form(P.fld, oh, 4), xh, b);
                bsp = form(cell_form(P.fld, oq, 5), xh, yh);
                const float4 geo = cell_form(P.fld, on, 6);
                rn_i = geo.x; sn_j = geo.y; cn_j = geo.z;
                killed = geo.w != 0.f;
            } else {
                const KJob A1 = opaque(A);
                const int ld = A1->p.ld, nr = A1->p.nr;
                // the corners of the grid cell and of the half-shifted ones,
                // clamped and signed as fill_patch takes them
                const int hr = ah ? i : i - 1, ht = bh ? j : j - 1;
                const unsigned n0 = mul24(i, ld), n1 = mul24(i + 1, ld);
                const unsigned h0 = mul24(max(hr, 0), ld), h1 = mul24(min(hr + 1, nr - 1), ld);
                const unsigned c0 = j, c1 = j + 1, s0 = max(ht, 0), s1 = min(ht + 1, nth - 1);
                const float o0 = ht < 0 ? -1.f : 1.f, o1 = ht + 1 > nth - 1 ? -1.f : 1.f;
                esr = form(corners(F.er, h0, h1, c0, c1, 1.f, 1.f), xh, b);
                est = form(corners(F.et, n0, n1, s0, s1, o0, o1), a, yh);
                esp = form(corners(F.ep, n0, n1, c0, c1, 1.f, 1.f), a, b);
                bsr = form(corners(F.br, n0, n1, s0, s1, 1.f, 1.f), a, yh);
                bst = form(corners(F.bt, h0, h1, c0, c1, 1.f, 1.f), xh, b);
                bsp = form(corners(F.bp, h0, h1, s0, s1, o0, o1), xh, yh);
                rn_i = ldo(A1->p.rn, (unsigned)i);
                sn_j = ldo(A1->p.sn, (unsigned)j);
                cn_j = ldo(A1->p.cn, (unsigned)j);
                killed = A1->kill[mul24(i, nth) + (unsigned)j] != 0;
            }
            // ---- geometry: theta = theta_j + d (small-angle series), r = r_i exp(a dlog)
            const float d = b * dth, d2 = d * d;
            const float sd = d * (1.f + d2 * (d2 * (1.f / 120.f) - 1.f / 6.f));
            const float cd = 1.f + d2 * (d2 * (1.f / 24.f) - 0.5f);
            const float st = sn_j * cd + cn_j * sd;
            const float ct = cn_j * cd - sn_j * sd;
            const float xl = a * dlog;
            const float r =
                rn_i * (1.f + xl * (1.f + xl * (0.5f + xl * (1.f / 6.f + xl * (1.f / 24.f)))));
            // ---- Boris rotation and radiation reaction in the orthonormal
            // basis (r, theta, phi) at the particle: the vector algebra is the
            // same in any right-handed orthonormal basis
            const float mx = ur + h * esr, my = ut + h * est, mz = up + h * esp;
            const float ig = h * frsq(1.f + mx * mx + my * my + mz * mz);
            const float tx = bsr * ig, ty = bst * ig, tz = bsp * ig;
            const float sf = 2.f * frcp(1.f + tx * tx + ty * ty + tz * tz);
            const float px = fma3(my, tz, -mz, ty, mx), py = fma3(mz, tx, -mx, tz, my),
                        pz = fma3(mx, ty, -my, tx, mz);
            float nr = mx + sf * (py * tz - pz * ty) + h * esr;
            float nt = my + sf * (pz * tx - px * tz) + h * est;
            float np = mz + sf * (px * ty - py * tx) + h * esp;
            // ---- radiation reaction (explicit, time-centred velocity b = v / sqrt(4 + v^2)
            // with v the sum of the old and the new momentum, gamma^2 = (4 + v^2) / 4)
            if (kk != 0.f) {
                float bx = ur + nr, by = ut + nt, bz = up + np;
                const float g4 = 4.f + bx * bx + by * by + bz * bz;
                const float igb = frsq(g4);
                bx *= igb; by *= igb; bz *= igb;
                const float Fx = fma3(by, bsp, -bz, bst, esr), Fy = fma3(bz, bsr, -bx, bsp, est),
                            Fz = fma3(bx, bst, -by, bsr, esp);
                const float be = bx * esr + by * est + bz * esp;
                const float bp2 = fmaxf(Fx * Fx + Fy * Fy + Fz * Fz - be * be, 0.f);
                const float gg = 0.25f * g4 * bp2;
                nr += kk * ((Fy * bsp - Fz * bst) + be * esr - gg * bx);
                nt += kk * ((Fz * bsr - Fx * bsp) + be * est - gg * by);
                np += kk * ((Fx * bst - Fy * bsr) + be * esp - gg * bz);
            }
            if constexpr (SHELL) {
                const KJob A1 = opaque(A);
                if (i < A1->p.ishell || (i == A1->p.ishell && a < A1->p.ashell)) {
                    // shell around the star (Sect. 5): drop the momentum across B
                    const float b2 = bsr * bsr + bst * bst + bsp * bsp;
                    if (b2 > 0.f) {
                        const float ub = (nr * bsr + nt * bst + np * bsp) / b2;
                        nr = ub * bsr; nt = ub * bst; np = ub * bsp;
                    }
                }
            }
            // ---- move.  The displacement in the basis at the particle is
            // (dr, dt, dp); with W the new distance from the axis in the old
            // meridional plane, the new one is w2 = sqrt(W^2 + dp^2), and
            // turning into the new plane adds e = w2 - W along the cylindrical
            // radius (formed without cancellation on either side of the axis).
            // A particle that ends on the axis turns by no azimuth: W is 1e-9
            // of a step larger, far below the offsets' resolution, so that it
            // outweighs a dp of zero there; 1.2e-38 keeps the sum from zero.
            const float ivg = frsq(1.f + nr * nr + nt * nt + np * np);   // 1 / gamma
            const float vdt = dt * ivg;
            const float dr = nr * vdt, dtt0 = nt * vdt, dp = np * vdt;
            const float W = (r * st + (dr * st + dtt0 * ct)) + weps;
            const float dp2 = dp * dp + 1.2e-38f;
            const float w22 = W * W + dp2;
            const float iw2 = frsq(w22);
            const float w2 = w22 * iw2, aW = __builtin_fabsf(W);
            const float e = dp2 * frcp(w2 + aW) + (aW - W);
            const float drr = dr + e * st, dtt = dtt0 + e * ct;
            const float ir = frcp(r);
            const float yv = drr * ir, zv = dtt * ir;
            const float arg = yv * (2.f + yv) + zv * zv;       // (r'/r)^2 - 1
            const float sq = arg * frcp(2.f + arg);            // log1p(x) = 2 atanh(x / (2 + x))
            const float sq2 = sq * sq;
            const float dxi = sq * (1.f + sq2 * (1.f / 3.f + sq2 * (1.f / 5.f)));
            const float tq = dtt * frcp(r + drr);
            const float tq2 = tq * tq;
            const float dthe = tq * (1.f - tq2 * (1.f / 3.f - tq2 * (1.f / 5.f)));
            // the momentum in the basis at the new point: rotated by dthe in
            // the meridional plane and by the azimuth, whose cosine less one
            // and sine along the cylindrical radius make g
            const float dd2 = dthe * dthe;
            const float sdd = dthe * (1.f - dd2 * (1.f / 6.f));
            const float cdd = 1.f - 0.5f * dd2;
            const float st2 = st * cdd + ct * sdd, ct2 = ct * cdd - st * sdd;
            const float nx = nr * st + nt * ct;
            const float g = (dp * np - e * nx) * iw2;
            float ur2 = nr * cdd + nt * sdd + g * st2;
            float ut2 = nt * cdd - nr * sdd + g * ct2;
            float up2 = (W * np - dp * nx) * iw2;
            // ---- new cell and offsets (carry)
            na = a + dxi * inv_dlog;
            nb = b + dthe * inv_dth;
            const float fa = floorf(na), fb = floorf(nb);
            float oa = na - fa, ob = nb - fb;
            di = (int)fa;
            dj = (int)fb;
            int i2 = i + di, j2 = j + dj;
            // the common case: no NaN and no infinity (a sum keeps them), stays on
            // the grid below the absorbing radius, moves one cell at most, and
            // neither offset rounds up to one
            const float us = ur2 + ut2 + up2;
            bool keep = live && !killed && __builtin_isfinite(us) &&
                        __builtin_fabsf(na - 0.5f) < 1.5f && __builtin_fabsf(nb - 0.5f) < 1.5f &&
                        (unsigned)i2 < (unsigned)iabs && (unsigned)j2 < (unsigned)nth &&
                        fmaxf(oa, ob) < 1.f;
            int c2 = (i2 << 16) | j2;
            bool cfl = false;
            if (__ballot(!keep) != 0ull) {
                const KJob A2 = opaque(A);
                const bool finite = __builtin_isfinite(us + na + nb);
                if (oa >= 1.f) { oa -= 1.f; di++; }
                if (ob >= 1.f) { ob -= 1.f; dj++; }
                i2 = i + di;
                j2 = j + dj;
                if (j2 < 0) { j2 = 0; ob = 0.f; dj = -j; }
                if (j2 > nth - 1) { j2 = nth - 1; ob = 0.99999994f; dj = j2 - j; }
                cfl = di > 1 || di < -1 || dj > 1 || dj < -1;
                // a particle in a force-free cell is removed before it moves
                const bool moves = live && !killed && finite;
                const bool star = moves && i2 < 0;
                const bool absb = moves && !star && (i2 > iabs || (i2 == iabs && oa >= A2->p.aabs));
                keep = moves && !star && !absb;
                nkill += live && killed ? 1 : 0;
                nstar += star ? 1 : 0;
                nabs += absb ? 1 : 0;
                if (cfl && live && !killed) atomicOr(A2->err, FFPIC_ERR_CFL);
                // non-finite state is flagged in the error word and never deposited
                if (!finite && live && !killed) atomicOr(A2->err, FFPIC_ERR_NONFINITE);
                // the end point as stored
                na = (float)di + oa;
                nb = (float)dj + ob;
                c2 = keep ? (i2 << 16) | j2 : -1;
                // a slot without a particle keeps what it holds
                if (!PLACE && !keep) {
                    oa = a; ob = b;
                    ur2 = State::ld(S.ur, q);
                    ut2 = State::ld(S.ut, q);
                    up2 = State::ld(S.up, q);
                }
            }
            if constexpr (PLACE) {
                if (live) {
                    const KJob A3 = opaque(A);
                    const unsigned d = (unsigned)dq;
                    sto(A3->SP.cell, d, c2);
                    sto(A3->SP.a, d, oa);
                    sto(A3->SP.b, d, ob);
                    sto(A3->SP.ur, d, ur2);
                    sto(A3->SP.ut, d, ut2);
                    sto(A3->SP.up, d, up2);
                }
            } else {
                S.stc(q, c2);
                State::st(S.a, q, oa);
                State::st(S.b, q, ob);
                State::st(S.ur, q, ur2);
                State::st(S.ut, q, ut2);
                State::st(S.up, q, up2);
            }
            const bool incell = (di | dj) == 0;
            simple = keep && !cfl && incell;
            cross = keep && !cfl && !incell;
            hx = na - a;
            hy = nb - b;
            q4 = dp;                               // v_phi before rotation, times dt
            qv = np * ivg;
            if (cross) {                           // in-cell: na = oa, nb = ob
                na = (float)di + oa;
                nb = (float)dj + ob;
            }
        }
        // ---- in-cell moves, one cell per 16-lane row and pass: the lanes of
        // a row whose cell is that of the row's first pending lane sum their
        // eight values over the row, and lanes 0..7 of the row add one sum
        // each.  Every pass retires at least the first pending lane of each
        // row, so the loop ends within 16 passes with every in-cell move
        // deposited.  (Sorted particles drift into neighbouring cells between
        // sorts, so a wave holds several cells; the passes with few lanes
        // still cost less than per-lane adds, until kLone are left.)
        bool pend = simple;
        const float X = a + na, Y = b + nb;        // twice the midpoint
        unsigned long long m = __ballot(pend);
#pragma unroll 1
        while (m != 0ull) {
            // the row's pending lanes and the key of the first (of any lane,
            // where there is none)
            const unsigned rowm =
                __builtin_amdgcn_ubfe(lane < 32 ? (unsigned)m : (unsigned)(m >> 32), row0 & 16, 16);
            const int lc = __builtin_amdgcn_ds_bpermute((row0 + __builtin_ctz(rowm | 0x10000u)) << 2, ckey);
            const bool part = pend && ckey == lc;
            // the eight values of the lanes that take part: J_r at (i, j) and
            // (i, j+1), J_theta at (i, j) and (i+1, j), J_phi at the four
            // nodes, each without its factor
            float s[8];
            values8(part ? hx : 0.f, part ? hy : 0.f, part ? q4 : 0.f, part ? X : 0.f,
                    part ? Y : 0.f, s);
            const float v = row_sum8(s, b0) * kscale;
            // a row with pending lanes has participants: its leader
            if (row_lead && rowm != 0u) {
                if (LDS) {
                    atomicAdd(&acc.tile[lc + kofs], v);
                } else {
                    const int li = cell_row(lc) + kdi, lj = (lc & 0xffff) + kdj;
                    gadd(reinterpret_cast<float *>(reinterpret_cast<char *>(kg) +
                                                   ((mul24(li, acc.ld) + (unsigned)lj) << 2)), v);
                }
            }
            pend = pend && !part;
            m = __ballot(pend);
            if (__popcll(m) <= kLone) {
                if (pend) {
                    values8(Q2 * hx, Q2 * hy, Qp4 * q4, X, Y, s);
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
        // moves that leave their cell go to the workgroup's queue and are
        // deposited after the chunk, where one wave takes them all instead of
        // every wave that holds one running the zigzag with a few lanes
        const unsigned long long cm = __ballot(cross);
        if (cm != 0ull) {
            int e0 = 0;
            if (lane == 0) e0 = atomicAdd(C.qn, __popcll(cm));
            e0 = __builtin_amdgcn_readfirstlane(e0);
            if (cross) {
                const int e = e0 + (int)__builtin_amdgcn_mbcnt_hi(
                                       (unsigned)(cm >> 32),
                                       __builtin_amdgcn_mbcnt_lo((unsigned)cm, 0u));
                if (e < kQueue) {
                    C.queue[2 * e] = make_float4(__int_as_float(c),
                                                 __int_as_float((di + 1) | ((dj + 1) << 2)), a, b);
                    C.queue[2 * e + 1] = make_float4(na, nb, qv, 0.f);
                } else {
                    zigzag(opaque(A), acc, i, j, di, dj, a, b, na, nb, qv);
                }
            }
        }
    }
    __syncthreads();
    const int nq = min(*C.qn, kQueue);
    if (tid < nq) {
        const float4 r0 = C.queue[2 * tid], r1 = C.queue[2 * tid + 1];
        const int c = __float_as_int(r0.x), dd = __float_as_int(r0.y);
        zigzag(opaque(A), acc, cell_row(c), c & 0xffff, (dd & 3) - 1, ((dd >> 2) & 3) - 1, r0.z, r0.w,
               r1.x, r1.y, r1.z);
    }
}

// the species of one launch (blockIdx.y)
struct PushJobs {
    PushJob job[FFPIC_MAX_SPECIES];
};

struct PushSmem {
    float *tile;
    PatchCell *fld;
    float4 *queue;
    int *box, *qn;
};

// Bounding box of the cells of slots [base, base + iters * kWG) into box
// (first and last row, first and last column; last row -1: no particle).
// Every thread of the workgroup calls it.
__device__ __forceinline__ void cell_box(const int32_t *cell, int n, int base, int iters, int tid,
                                         int *box) {
    int imin = 1 << 30, imax = -1, jmin = 1 << 30, jmax = -1;
    // four cells at a time (a slot past the last reads the last slot's cell
    // and ignores it; behind a branch each, the loads would wait one after
    // the other)
    for (int k = 0; k < iters; k += 4) {
        int cb[4];
#pragma unroll
        for (int u = 0; u < 4; u++)
            cb[u] = ldo(cell, (unsigned)min(base + (k + u) * kWG + tid, n - 1));
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int ck = base + (k + u) * kWG + tid < n && k + u < iters ? cb[u] : -1;
            if (cell_live(ck)) {
                const int i = cell_row(ck), j = ck & 0xffff;
                imin = min(imin, i); imax = max(imax, i);
                jmin = min(jmin, j); jmax = max(jmax, j);
            }
        }
    }
    if (tid == 0) {
        box[0] = 1 << 30; box[1] = -1; box[2] = 1 << 30; box[3] = -1;
    }
    __syncthreads();
    for (int o = 32; o >= 1; o >>= 1) {
        imin = min(imin, __shfl_xor(imin, o, 64));
        imax = max(imax, __shfl_xor(imax, o, 64));
        jmin = min(jmin, __shfl_xor(jmin, o, 64));
        jmax = max(jmax, __shfl_xor(jmax, o, 64));
    }
    if ((tid & 63) == 0 && imax >= 0) {
        atomicMin(&box[0], imin); atomicMax(&box[1], imax);
        atomicMin(&box[2], jmin); atomicMax(&box[3], jmax);
    }
    __syncthreads();
}

// the cells of the field patch and the entries of the deposit patch of a box
__device__ __forceinline__ bool box_fits(const int *box) {
    const int ni = box[1] - box[0], nj = box[3] - box[2];
    return (ni + 2) * (nj + 4) <= kCells && (ni + 4) * (nj + 4) <= kTile;
}

// The field patch of rows [i0, i0 + ni) and columns [j0, j0 + nj) of cells
// (i0 and j0 are -1 at the least, for the half-shifted cells before the
// first).  Rows are clamped to those a component has (its value is constant
// past the last); a half column past an axis is the edge column, with the
// sign flipped for the odd components E_theta and B_phi.
__device__ __forceinline__ void fill_patch(KJob A0, PatchCell *fld, int i0, int j0, int ni, int nj,
                                           int stride, int tid) {
    const KJob A = opaque(A0);
    const int nr = A->p.nr, nth = A->p.nth, ld = A->p.ld;
    for (int e = tid; e < ni * nj; e += kWG) {
        const int ti = e / nj, tj = e - ti * nj, i = i0 + ti, j = j0 + tj;
        const int ic = max(i, 0), jc = max(j, 0);
        // node rows and columns, half rows and columns of the four corners
        const unsigned n0 = (unsigned)(ic * ld), n1 = (unsigned)(min(i + 1, nr) * ld);
        const unsigned h0 = n0, h1 = (unsigned)(min(i + 1, nr - 1) * ld);
        const unsigned c0 = jc, c1 = min(j + 1, nth), s0 = jc, s1 = min(j + 1, nth - 1);
        const float o0 = j < 0 ? -1.f : 1.f, o1 = j + 1 > nth - 1 ? -1.f : 1.f;
        PatchCell P;
        const float *E0 = A->E[0], *E1 = A->E[1], *E2 = A->E[2];
        const float *B0 = A->B[0], *B1 = A->B[1], *B2 = A->B[2];
        P.c[0] = form4(ldo(E0, h0 + c0), ldo(E0, h0 + c1), ldo(E0, h1 + c0), ldo(E0, h1 + c1));
        P.c[1] = form4(o0 * ldo(E1, n0 + s0), o1 * ldo(E1, n0 + s1), o0 * ldo(E1, n1 + s0),
                       o1 * ldo(E1, n1 + s1));
        P.c[2] = form4(ldo(E2, n0 + c0), ldo(E2, n0 + c1), ldo(E2, n1 + c0), ldo(E2, n1 + c1));
        P.c[3] = form4(ldo(B0, n0 + s0), ldo(B0, n0 + s1), ldo(B0, n1 + s0), ldo(B0, n1 + s1));
        P.c[4] = form4(ldo(B1, h0 + c0), ldo(B1, h0 + c1), ldo(B1, h1 + c0), ldo(B1, h1 + c1));
        P.c[5] = form4(o0 * ldo(B2, h0 + s0), o1 * ldo(B2, h0 + s1), o0 * ldo(B2, h1 + s0),
                       o1 * ldo(B2, h1 + s1));
        P.geo = make_float4(ldo(A->p.rn, (unsigned)ic), ldo(A->p.sn, (unsigned)jc),
                            ldo(A->p.cn, (unsigned)jc),
                            A->kill[mul24(min(ic, nr - 1), nth) + (unsigned)min(jc, nth - 1)] ? 1.f : 0.f);
        fld[ti * stride + tj] = P;
    }
}

// One chunk of kWG * ppt slots.  Every thread of the workgroup calls it
// and returns from it together.
template <bool SHELL, bool PLACE>
__device__ __forceinline__ void push_block(KJob A0, int chunk, const PushSmem &sm) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    float *tile = sm.tile;
    int *box = sm.box;
    // PLACE: the slots before the sort (the slot count already holds the
    // new order's)
    const int n = min(A0->nub, A0->nslots[PLACE ? 2 : 0]);
    const int ppt = A0->ppt;
    const int first = chunk * (kWG * ppt);
    if (first >= n) return;    // no slot in the chunk (uniform)
    cell_box(A0->cell, n, first, ppt, tid, box);
    if (box[1] < 0) return;    // no live particle in the chunk (uniform)
    // a box too large for the patches: the chunk in parts of kPart rounds
    const bool whole = box_fits(box);
    const int rounds = whole ? ppt : min(ppt, kPart);
    int nkill = 0, nstar = 0, nabs = 0;
    for (int k0 = 0; k0 < ppt; k0 += rounds) {
        const int base = first + k0 * kWG;
        if (base >= n) break;
        if (!whole) {
            __syncthreads();   // the box and the patches of the part before are read
            cell_box(A0->cell, n, base, rounds, tid, box);
            if (box[1] < 0) continue;
        }
        const int bi = box[0], bj = box[2], ni = box[1] - bi + 1, nj = box[3] - bj + 1;
        if (tid == 0) *sm.qn = 0;
        const ChunkArgs C{n, base, rounds, (bi << 16) | bj, tid, lane, sm.queue, sm.qn};
        if (box_fits(box)) {
            // the deposit patch covers rows [imin-1, imax+2] and columns
            // [jmin-1, jmax+2]: every add of a particle that moves at most one
            // cell lands inside
            const int ti0 = bi - 1, tj0 = bj - 1, TJ = nj + 3, m = (ni + 3) * TJ;
            for (int e = tid; e < m; e += kWG) {
                tile[e] = 0.f; tile[kTile + e] = 0.f; tile[2 * kTile + e] = 0.f;
            }
            // the field patch: cells of rows [imin-1, imax], columns [jmin-1, jmax]
            // (rows as long as the deposit patch's, so that one key serves both)
            fill_patch(A0, sm.fld, bi - 1, bj - 1, ni + 1, nj + 1, TJ, tid);
            __syncthreads();
            const Patch P{reinterpret_cast<const char *>(sm.fld), (unsigned)TJ * kCellB,
                          ti0 * TJ + tj0};
            Acc<true> acc{tile, ti0, tj0, TJ, {nullptr, nullptr, nullptr}, 0};
            push_chunk<true, SHELL, PLACE>(A0, Fields{}, P, acc, C, nkill, nstar, nabs, nullptr);
            __syncthreads();
            const KJob A = opaque(A0);
            float *Jr = A->J[0], *Jt = A->J[1], *Jp = A->J[2];
            const int nr = A->p.nr, nth = A->p.nth, ld = A->p.ld;
            for (int e = tid; e < m; e += kWG) {
                const int ti = e / TJ, tj = e - ti * TJ;
                const int gi = ti0 + ti, gj = tj0 + tj;
                if (gi < 0 || gi > nr || gj < 0 || gj > nth) continue;
                const unsigned g = ((unsigned)(gi * ld + gj)) << 2;
                const float v0 = tile[e], v1 = tile[kTile + e], v2 = tile[2 * kTile + e];
                if (v0 != 0.f) gadd(reinterpret_cast<float *>(reinterpret_cast<char *>(Jr) + g), v0);
                if (v1 != 0.f) gadd(reinterpret_cast<float *>(reinterpret_cast<char *>(Jt) + g), v1);
                if (v2 != 0.f) gadd(reinterpret_cast<float *>(reinterpret_cast<char *>(Jp) + g), v2);
            }
        } else {
            __syncthreads();   // the queue is empty
            // the gather reads the fields through buffer resources in this mode
            // (nr + 1) * ld stays near the 2^29-node grid limit, so the byte count
            // fits 32 unsigned bits
            const KJob A = opaque(A0);
            const int nbytes = (int)((unsigned)(A->p.nr + 1) * (unsigned)A->p.ld * 4u);
            Fields F;
            F.er = __builtin_amdgcn_make_buffer_rsrc((void *)A->E[0], 0, nbytes, kRsrcWord3);
            F.et = __builtin_amdgcn_make_buffer_rsrc((void *)A->E[1], 0, nbytes, kRsrcWord3);
            F.ep = __builtin_amdgcn_make_buffer_rsrc((void *)A->E[2], 0, nbytes, kRsrcWord3);
            F.br = __builtin_amdgcn_make_buffer_rsrc((void *)A->B[0], 0, nbytes, kRsrcWord3);
            F.bt = __builtin_amdgcn_make_buffer_rsrc((void *)A->B[1], 0, nbytes, kRsrcWord3);
            F.bp = __builtin_amdgcn_make_buffer_rsrc((void *)A->B[2], 0, nbytes, kRsrcWord3);
            float *Jr = A->J[0], *Jt = A->J[1], *Jp = A->J[2];
            Acc<false> acc{nullptr, 0, 0, 0, {Jr, Jt, Jp}, A->p.ld};
            const int kc = lane_comp(lane);
            float *kg = kc == 0 ? Jr : (kc == 1 ? Jt : Jp);
            push_chunk<false, SHELL, PLACE>(A0, F, Patch{nullptr, 0u, 0u}, acc, C, nkill, nstar,
                                            nabs, kg);
        }
    }
    if (__ballot((nkill | nstar | nabs) != 0) == 0ull) return;
    int tk = nkill, ts = nstar, ta = nabs;
    for (int o = 32; o >= 1; o >>= 1) {
        tk += __shfl_xor(tk, o, 64);
        ts += __shfl_xor(ts, o, 64);
        ta += __shfl_xor(ta, o, 64);
    }
    if (lane == 0) {
        unsigned long long *removed = opaque(A0)->removed;
        if (tk) atomicAdd(&removed[1], (unsigned long long)tk);
        if (ts) atomicAdd(&removed[2], (unsigned long long)ts);
        if (ta) atomicAdd(&removed[3], (unsigned long long)ta);
    }
}

// Five workgroups per CU: LDS and registers (96, some values between the phases
// spilled) both end there.  2e8 particles in the sheet's first steps: 2.16 ms
// with four and larger patches, 2.07 with five; six (80 registers) spill in the particle loop.
template <bool SHELL, bool PLACE>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(5, 8)))
k_push32(const PushJobs) {
    __shared__ float tile[3 * kTile];
    __shared__ PatchCell fld[kCells];
    __shared__ float4 queue[2 * kQueue];
    __shared__ int box[4];
    __shared__ int qn;
    push_block<SHELL, PLACE>((KJob)__builtin_amdgcn_kernarg_segment_ptr() + blockIdx.y, (int)blockIdx.x,
                             PushSmem{tile, fld, queue, box, &qn});
}

// The pushes of many systems in one launch of persistent workgroups: each
// workgroup takes chunks (items) from a counter in device memory until none
// is left.  Job k owns items [starts[k], starts[k + 1]).  The workgroup that
// finishes last returns both counters to zero for the next launch.
template <bool SHELL, bool PLACE>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(5, 8)))
k_push32_group(const PushJob *__restrict__ jobs, const int *__restrict__ starts, int njobs,
               int *__restrict__ ctr) {
    __shared__ float tile[3 * kTile];
    __shared__ PatchCell fld[kCells];
    __shared__ float4 queue[2 * kQueue];
    __shared__ int box[4];
    __shared__ int qn;
    __shared__ int next, job;
    const PushSmem sm{tile, fld, queue, box, &qn};
    const int total = starts[njobs];
    if (threadIdx.x == 0) next = atomicAdd(&ctr[0], 1);
    __syncthreads();
    int item = __builtin_amdgcn_readfirstlane(next);
    while (item < total) {
        find_job(starts, njobs, item, &job);
        // the next item is taken now, so that the counter's round trip
        // overlaps this item's work
        int nx = 0;
        if (threadIdx.x == 0) nx = atomicAdd(&ctr[0], 1);
        __syncthreads();
        const int lo = __builtin_amdgcn_readfirstlane(job);
        push_block<SHELL, PLACE>((KJob)(jobs + lo), item - starts[lo], sm);
        if (threadIdx.x == 0) next = nx;
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(next);
    }
    group_done(ctr);
}

// the kernel instance of a species' push: shell, placing
struct PushKey {
    bool shell, place;
};

PushKey push_key(const ffpic_ctx *c, int s) {
    return {c->d.shell_r > c->d.rmin, c->sort_pending[s]};
}

int push_key_index(const PushKey &k) { return (k.shell ? 1 : 0) + (k.place ? 2 : 0); }

// Particles per thread of a chunk where the caller sets none: the tuned number
// (8, 16 or 32; 16 untuned), but fewer where the launch's slots would not give every CU its five workgroups, or give them
// in few rounds with a nearly empty last one.  A chunk costs about two rounds
// of its particles besides (its box and patches), so one per thread pays only
// while most CUs are idle.  us per launch by particles per thread:
//   slots       1      2      4      8     16
//   1.0e5     8.4    9.6   12.6   19.2   35.2
//   3.0e5    12.3   12.8   15.8   23.8   45.8
//   6.5e5    19.5   15.2   19.4   29.5   47.8
//   1.3e6    36.1   29.4   26.3   36.2   57.4
//   4.0e6   109     82.1   73.6   77.3   90.0
//   1.0e7   257    180    151    146    157
//   2.0e7   509    349    283    268    270
//   2.8e7  1332    737    508    480    508   (16 systems of a batch)
//   5.0e7  1199    812    664    616    593
int push_chunk(int ppt, int64_t slots) {
    const int64_t rounds = slots / kWG;
    const int most = rounds < 1536 ? 1 : rounds < 4096 ? 2 : rounds < 24576 ? 4 : rounds < 131072 ? 8 : 32;
    return std::min(ppt, most);
}
int push_ppt(const ffpic_ctx *c, int64_t slots) {
    return c->push_fixed ? c->push_ppt : push_chunk(c->push_ppt, slots);
}

// the job of one species' push from the context's state, and the host
// bookkeeping that follows the launch (a placing push leaves the new order
// in the second buffer)
PushJob make_push_job(ffpic_ctx *c, int s, int ppt) {
    ffpic::Species &S = c->sp[s];
    PushJob J{};
    P32 &p = J.p;
    p.nr = c->nr; p.nth = c->nth; p.ld = c->ld;
    p.dlog = (float)c->dlog; p.dth = (float)c->dth; p.dt = (float)c->dt;
    p.inv_dlog = (float)(1.0 / c->dlog);
    p.inv_dth = (float)(1.0 / c->dth);
    double xa = log(c->d.r_abs / c->d.rmin) / c->dlog;
    p.iabs = (int)floor(xa);
    p.aabs = (float)(xa - floor(xa));
    p.rn = (const float *)c->dtab[T_RN];
    p.sn = (const float *)c->dtab[T_SN];
    p.cn = (const float *)c->dtab[T_CN];
    double qm = S.qm;
    p.Q = (float)((qm > 0 ? 1.0 : -1.0) * S.weight);
    p.h = (float)(0.5 * c->dt * c->d.omega_b * qm);
    p.kk = (float)(c->dt * c->d.rr_coef * rr_factor(c) * fabs(qm) * fabs(qm) * fabs(qm));
    p.weps = (float)(1e-9 * c->dt);
    // the shell radius in cell units, split like r_abs
    const bool shell = c->d.shell_r > c->d.rmin;
    const double xs = shell ? log(c->d.shell_r / c->d.rmin) / c->dlog : 0.0;
    p.ishell = (int)floor(xs);
    p.ashell = (float)(xs - floor(xs));
    J.nub = (int)S.nub;
    J.ppt = ppt;
    const bool place = c->sort_pending[s];
    // the placing push runs over the slots before the sort: the third
    // entry of the sort's totals
    J.nslots = place ? (const int32_t *)c->sort_tot[s] : c->nslots + s;
    J.kill = c->kill;
    for (int k = 0; k < 3; k++) {
        J.E[k] = (const float *)c->E[k];
        J.B[k] = (const float *)c->B[k];
        J.J[k] = (float *)c->J[k];
    }
    J.cell = (int32_t *)S.cur[0];
    J.a = (float *)S.cur[1];
    J.b = (float *)S.cur[2];
    J.ur = (float *)S.cur[3];
    J.ut = (float *)S.cur[4];
    J.up = (float *)S.cur[5];
    J.removed = c->removed + 4 * s;
    J.err = c->err;
    if (place) J.SP = c->place[s];
    return J;
}

using PushKern = void (*)(const PushJobs);
using PushGroupKern = void (*)(const PushJob *, const int *, int, int *);

void push32(ffpic_ctx *c) {
    // the species whose kernel is the same share a launch: side by side they
    // fill the GPU, and its last round, better (two of 6.5e5: 2 x 15 -> 24 us)
    bool done[FFPIC_MAX_SPECIES] = {};
    for (int s0 = 0; s0 < c->d.nspec; s0++) {
        if (done[s0] || c->sp[s0].nub == 0) continue;
        const PushKey k = push_key(c, s0);
        int64_t slots = 0;
        for (int s = s0; s < c->d.nspec; s++)
            if (!done[s] && c->sort_pending[s] == k.place) slots += c->sp[s].nub;
        const int ppt = push_ppt(c, slots), chunk = kWG * ppt;
        PushJobs P{};
        int m = 0, nb = 0;
        for (int s = s0; s < c->d.nspec; s++) {
            ffpic::Species &S = c->sp[s];
            if (done[s] || S.nub == 0 || c->sort_pending[s] != k.place) continue;
            done[s] = true;
            P.job[m++] = make_push_job(c, s, ppt);
            nb = std::max(nb, (int)((S.nub + chunk - 1) / chunk));
            after_push(c, s);
        }
        const PushKern kern = k.shell ? (k.place ? k_push32<true, true> : k_push32<true, false>)
                                      : (k.place ? k_push32<false, true> : k_push32<false, false>);
        hipLaunchKernelGGL(kern, dim3(nb, m), dim3(kWG), 0, c->stream, P);
        FFPIC_LAUNCH_CHECK();
    }
}

// ---- grouped pushes of several contexts (batches)

size_t push_job_bytes() { return sizeof(PushJob); }

int push_group_key(const ffpic_ctx *c, int s) { return push_key_index(push_key(c, s)); }

int push_job(ffpic_ctx *c, int s, void *out, int ppt, int64_t slots) {
    ffpic::Species &S = c->sp[s];
    if (ppt == 0) ppt = push_ppt(c, slots);
    const PushJob J = make_push_job(c, s, ppt);
    std::memcpy(out, &J, sizeof(J));
    after_push(c, s);
    const int chunk = kWG * ppt;
    return (int)((S.nub + chunk - 1) / chunk);
}

static PushGroupKern group_kern_of(int key) {
    const bool shell = key & 1, place = key & 2;
    return shell ? (place ? k_push32_group<true, true> : k_push32_group<true, false>)
                 : (place ? k_push32_group<false, true> : k_push32_group<false, false>);
}
static_assert(kPushKeys == 4, "shell or not, placing or not");

int push_group_slots(int key) {
    int per_cu = 0, cus = 0, dev = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)group_kern_of(key), kWG,
                                                     0) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 1024;
    }
    return std::max(1, per_cu) * std::max(1, cus);
}

void push_group_launch(hipStream_t st, int key, const void *jobs, const int *starts, int njobs,
                       int grid, int *ctr) {
    hipLaunchKernelGGL(group_kern_of(key), dim3(grid), dim3(kWG), 0, st,
                       (const PushJob *)jobs, starts, njobs, ctr);
    FFPIC_LAUNCH_CHECK();
}

}  // namespace ffpic
