// Device code and host helpers shared by the two forms of the incremental
// sort: movers sorted by radix passes (k_sort.hip) or by buckets
// (k_sort_bucket.hip).
#pragma once

#include "device_common.h"
#include "sort_view.h"

namespace ffpic {

constexpr int kTile = 1 << kTileShift;      // slots per classify tile (8 per thread)
constexpr int kTileWords = kTile / 64;      // 64-slot words per tile
constexpr int kGroup = 1 << kGroupShift;    // tiles per group of the tile scan
constexpr int kKeyShift = 10;               // keys per block of the per-key passes: 1024
constexpr int kKeyBlocks = 2048;            // such blocks, in the bucket form at most

// ---------------------------------------------------------------------------
// small device helpers

__device__ __forceinline__ uint64_t lanes_below() {
    return (1ull << (threadIdx.x & 63)) - 1ull;
}

// exclusive scan of one value per thread over a block of T threads; the
// block total in *total.  Contains barriers: every thread of the block must
// call it.
template <int T>
__device__ __forceinline__ uint64_t block_scan(uint64_t v, uint64_t *total) {
    __shared__ uint64_t wt[T / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wt[w] = x;
    __syncthreads();
    uint64_t pre = 0, all = 0;
#pragma unroll
    for (int u = 0; u < T / 64; u++) {
        if (u < w) pre += wt[u];
        all += wt[u];
    }
    *total = all;
    __syncthreads();
    return pre + x - v;
}
__device__ __forceinline__ uint64_t block_scan256(uint64_t v, uint64_t *total) {
    return block_scan<256>(v, total);
}

// lanes of the wave whose (valid) digit equals this lane's
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool valid) {
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; b++) {
        const bool bit = (d >> b) & 1u;
        const uint64_t x = __ballot(bit);
        m &= bit ? x : ~x;
    }
    return m;
}

// the state arrays of a species in the old and the new order
template <typename T, int NA>
struct PtrSet {
    const T *src[NA];
    T *dst[NA];
};

template <typename T, int NA>
PtrSet<T, NA> state_ptrs(ffpic::Species &S) {
    PtrSet<T, NA> P;
    for (int a = 0; a < NA; a++) {
        P.src[a] = (const T *)S.cur[a];
        P.dst[a] = (T *)S.alt[a];
    }
    return P;
}

// first index in [lo, hi) whose value is >= x
__device__ __forceinline__ int lower_bound_u32(const uint32_t *a, int lo, int hi, uint32_t x) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

struct ClassArgs {
    int nub, nth, nr;
    uint32_t dead;
    const int32_t *nslots, *nsorted;
    const uint8_t *kill;
    const int32_t *offold;                      // cell offsets of the last sort
    unsigned long long *removed;
    // FP32 state: the cell; FP64 state: r, theta and the geometry
    int32_t *cell;
    double *R;
    const double *TH, *rn, *thn;
    double rmin, dlog, dth;
    uint32_t *keys;                             // FP64: key of every slot (out)
    uint64_t *smask, *mmask;
    uint32_t *wsm;
    uint2 *tc;                                  // stayers, movers of each tile
    uint32_t *tot;                              // [2]: the slot count before the sort
    uint32_t *tkey, *tval;                      // movers of each tile, compacted in it
    // buckets: movers of each key, of each block of 2^kKeyShift keys, and each
    // mover's arrival rank in its key's bucket
    int nkeys;
    unsigned long long *kcnt;
    uint32_t *kpart, *rank;
};

// The key a slot had at the last sort is the one whose range of that
// sort's cell offsets holds the slot: a particle keeps its key since then
// exactly when its slot lies in [OFF[key], OFF[key+1]).  Two reads of the
// per-key offsets instead of a stored key per slot (sorted particles of a
// wave mostly share a key, so the reads share cache lines).  lo, hi: the
// key's OFF[key], OFF[key+1]; nold: the slots the last sort ordered.
__device__ __forceinline__ bool in_old_range(int q, int nold, int lo, int hi) {
    return q < nold && lo <= q && q < hi;
}

// key of every slot, the removal of killed particles, the class bits and
// counts, and the movers of the tile compacted in slot order
// (BUCKETS: instead of the compacted movers, each mover's arrival rank in the
// bucket of its key; see k_sort_bucket.hip)
// by a workgroup of T threads
template <bool FP64, bool BUCKETS, int T = 256>
__device__ __forceinline__ void classify_tile(const ClassArgs &A, int tile) {
    constexpr int K = kTile / T, W = T / 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int base = tile * kTile;
    const int ns = A.nslots[0], no = A.nsorted[0];
    if (tile == 0 && tid == 0) A.tot[2] = (uint32_t)ns;   // for a push that places
    uint32_t key[K];
    int cl[K], lo[K];
    if (!FP64) {
        // the cells of all K slots, then for every slot its cell's kill flag
        // and its key's old offset range, loaded whether needed or not (a
        // slot without a particle reads those of key 0): with no branch
        // around them, all 3K loads are in flight together instead of one
        // round trip after another
        int cell[K];
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int q = base + k * T + tid;
            cell[k] = q < ns ? A.cell[q] : -1;
        }
        uint8_t kf[K];
        int hi[K];
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int c = cell[k];
            const uint32_t kk = cell_live(c) ? cell_key(c, A.nth) : 0u;
            key[k] = kk;
            kf[k] = A.kill[kk];
            lo[k] = A.offold[kk];
            hi[k] = A.offold[kk + 1];
        }
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int q = base + k * T + tid;
            const bool live = cell_live(cell[k]);
            const bool killed = live && kf[k] != 0;
            if (killed) A.cell[q] = -1;
            if (!live || killed) key[k] = A.dead;
            cl[k] = key[k] >= A.dead ? 0 : (in_old_range(q, no, lo[k], hi[k]) ? 1 : 2);
            count_wave(&A.removed[1], killed);
        }
    } else {
        // the positions of all K slots, their cells, then (as in the FP32
        // branch) the kill flags and old offset ranges, loaded unconditionally
        double r[K], th[K];
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int q = base + k * T + tid;
            r[k] = q < ns ? A.R[q] : -1.0;
            th[k] = q < ns ? A.TH[q] : 0.0;
        }
        int cix[K];                                 // i * nth + j, -1: no particle
#pragma unroll
        for (int k = 0; k < K; k++) {
            cix[k] = -1;
            if (r[k] > 0.0) {
                int i, j;
                double a, b;
                locate64(A.nr, A.nth, A.rmin, A.dlog, A.dth, A.rn, A.thn, r[k], th[k], i, j, a, b);
                cix[k] = i * A.nth + j;
            }
        }
        uint8_t kf[K];
        int hi[K];
#pragma unroll
        for (int k = 0; k < K; k++) {
            const uint32_t kk = cix[k] >= 0 ? (uint32_t)cix[k] : 0u;
            kf[k] = A.kill[kk];
            lo[k] = A.offold[kk];
            hi[k] = A.offold[kk + 1];
        }
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int q = base + k * T + tid;
            const bool live = cix[k] >= 0;
            const bool killed = live && kf[k] != 0;
            if (killed) A.R[q] = -1.0;
            key[k] = live && !killed ? (uint32_t)cix[k] : A.dead;
            if (q < A.nub) A.keys[q] = key[k];
            cl[k] = key[k] >= A.dead ? 0 : (in_old_range(q, no, lo[k], hi[k]) ? 1 : 2);
            count_wave(&A.removed[1], killed);
        }
    }
    // the tile's words are staged in LDS and written by 16 lanes at once
    __shared__ uint64_t wmask[2][kTileWords];
    __shared__ uint32_t wpre[2][kTileWords];
    uint64_t mm[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        const uint64_t sm = __ballot(cl[k] == 1);
        mm[k] = __ballot(cl[k] == 2);
        if (lane == 0) {
            wmask[0][k * W + w] = sm;
            wmask[1][k * W + w] = mm[k];
        }
    }
    __syncthreads();
    const int nwu = (A.nub + 63) >> 6;
    if (tid < kTileWords) {
        uint32_t ps = 0, pm = 0;
        for (int u = 0; u < tid; u++) {
            ps += (uint32_t)__popcll(wmask[0][u]);
            pm += (uint32_t)__popcll(wmask[1][u]);
        }
        wpre[0][tid] = ps;
        wpre[1][tid] = pm;
        const int gw = (base >> 6) + tid;
        if (gw < nwu) {
            A.smask[gw] = wmask[0][tid];
            A.mmask[gw] = wmask[1][tid];
            A.wsm[gw] = ps | (pm << 16);
        }
        if (tid == kTileWords - 1)
            A.tc[tile] = make_uint2(ps + (uint32_t)__popcll(wmask[0][tid]),
                                          pm + (uint32_t)__popcll(wmask[1][tid]));
    }
    if constexpr (BUCKETS) {
        // One add per key in the wave (most movers of a wave go to a few
        // cells) and one per block of keys in the tile: with an add per mover
        // and one per block of keys in the wave, the adds to the same few
        // addresses took 36 of the 47 us of 1.3e6 slots on 300 x 517
        __shared__ uint32_t kb[kKeyBlocks];
        for (int b = tid; b <= A.nkeys >> kKeyShift; b += T) kb[b] = 0u;
        __syncthreads();
        uint64_t peers[K];
        uint32_t rank[K];
        const uint64_t below = lanes_below();
#pragma unroll
        for (int k = 0; k < K; k++) {
            peers[k] = 0;
            uint64_t m = mm[k];
            while (m) {
                const uint32_t k0 = __builtin_amdgcn_readlane(key[k], __ffsll((long long)m) - 1);
                const uint64_t in = __ballot(key[k] == k0) & mm[k];
                if (key[k] == k0) peers[k] = in;
                if (lane == 0) atomicAdd(&kb[k0 >> kKeyShift], (uint32_t)__popcll(in));
                m &= ~in;
            }
        }
#pragma unroll
        for (int k = 0; k < K; k++) {
            // count of the key, and above it the count from slots before the
            // key's old range
            const uint64_t early = __ballot(base + k * T + tid < lo[k]);
            rank[k] = 0u;
            if (cl[k] == 2 && (peers[k] & below) == 0)
                rank[k] = (uint32_t)atomicAdd(
                    &A.kcnt[key[k]], (unsigned long long)__popcll(peers[k]) |
                                         (unsigned long long)__popcll(peers[k] & early) << 32);
        }
        __syncthreads();
        for (int b = tid; b <= A.nkeys >> kKeyShift; b += T)
            if (kb[b]) atomicAdd(&A.kpart[b], kb[b]);
#pragma unroll
        for (int k = 0; k < K; k++) {
            const uint32_t r0 = __shfl(rank[k], cl[k] == 2 ? __ffsll((long long)peers[k]) - 1 : lane, 64);
            if (cl[k] == 2) A.rank[base + k * T + tid] = r0 + (uint32_t)__popcll(peers[k] & below);
        }
    } else {
        __syncthreads();
        const uint64_t below = lanes_below();
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (cl[k] == 2) {
                const int r = (int)wpre[1][k * W + w] + (int)__popcll(mm[k] & below);
                A.tkey[base + r] = key[k];
                A.tval[base + r] = (uint32_t)(base + k * T + tid);
            }
        }
    }
}

// first key past every live one (see k_sort.hip)
uint32_t dead_key(const ffpic_ctx *c);
// where a sort of species s records its permutation (null: nowhere)
int32_t *perm_out(ffpic_ctx *c, int s);
// the next push of species s writes its particles in the sorted order
void place_by_push(ffpic_ctx *c, int s);
// the bucket form: scratch, whether a species' next sort takes it, the sort
void bucket_alloc(ffpic_ctx *c, int s, void *(*dmalloc)(size_t));
bool bucket_sort_ok(const ffpic_ctx *c, int s);
void sort_bucketed(const SortItem *items, int n, hipStream_t st, bool defer);

}  // namespace ffpic
