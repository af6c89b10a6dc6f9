// The incremental sort of species that do not fill the GPU, by buckets (see
// k_sort.hip for the order it produces and for stayers and movers).
//
// Its time there is launches: a radix sort of the movers takes three kernels
// per digit, and with the scans around it a sort is some 17 dependent kernels
// of 4 to 12 us each, per species.  Here the movers are sorted by counting
// them per key, in four kernels that all sorting species share (blockIdx.y):
//   1. classify: as in the radix form, but a mover adds itself to its key's
//      count, which returns its arrival rank in the key's bucket, and to the
//      count of its block of 1024 keys;
//   2. keys: the movers before each key (a scan inside the block of keys, on
//      the sum of the blocks before it), with that the key's new offset and
//      the movers before its stayers (the movers of the key from slots before
//      its old range were counted apart), and the tiles' stayers before them;
//   3. fill: every mover's slot to its bucket, in order of arrival;
//   4. place (or, for a push that places, the places alone): a stayer as in
//      the radix form; a mover's rank is the movers before its key plus those
//      of its bucket from lower slots, counted by reading the bucket.
// A bucket of more than kBucketScan movers is sorted by slot in step 3, by the
// workgroup that completes it, and step 4 bisects it.
//
// Both species of a step, kernel time of the radix form -> this one: 1e5
// particles each on 128^2 in FP64, sorted every step, 208 -> 29 us; 6.5e5 on
// 300 x 517 in FP32, every eighth, 240 -> 53; 1e6 on 512^2 in FP64 303 -> 96.
#include <algorithm>
#include <vector>

#include "sort_impl.h"

namespace ffpic {

constexpr int kBucketTiles = 1024;                       // tiles the key pass scans in LDS
constexpr int64_t kBucketSlots = (int64_t)kBucketTiles * kTile;   // 2,097,152
constexpr int64_t kBucketKeys = (int64_t)kKeyBlocks << kKeyShift; // 2,097,152 cells, one less at most
// movers of a bucket that are counted one by one: with buckets sorted from 257
// on, 2.1e6 slots on 512^2 took 77 + 58 us for fill and places, from 1025 on
// 11 + 66; 6.5e5 on 380^2 70 + 28 and 6 + 37
constexpr int kBucketScan = 1024;
constexpr int kBucketJobs = 8;                           // species per launch

struct BucketJob {
    ClassArgs A;
    int ntile;
    uint2 *ts, *gs;
    int32_t *off;              // movers before each key [nkeys + 1]
    uint32_t *mq, *mq2;        // mover slots by bucket; scratch of the same size
    int32_t *mst, *offnew, *nalive, *nslots, *nsorted;
    int32_t *dest, *perm;
    void *src[6], *dst[6];
};

struct BucketArgs {
    BucketJob job[kBucketJobs];
};
static_assert(sizeof(BucketArgs) <= 4096, "kernel arguments");

__device__ __forceinline__ ClassView bucket_view(const BucketJob &J) {
    return ClassView{J.A.nub, J.A.smask, J.A.mmask, J.A.wsm, J.ts, J.gs, J.A.tot};
}

// Workgroups of 1024 threads, two slots each: so few tiles leave most CUs idle,
// and more waves per tile shorten its chain of loads and adds.
constexpr int kBucketThreads = 1024;

template <bool FP64>
__global__ void __launch_bounds__(kBucketThreads) k_bucket_classify(const BucketArgs P) {
    const BucketJob &J = P.job[blockIdx.y];
    if ((int)blockIdx.x >= J.ntile) return;
    classify_tile<FP64, true, kBucketThreads>(J.A, (int)blockIdx.x);
}

__global__ void __launch_bounds__(256) k_bucket_keys(const BucketArgs P) {
    const BucketJob &J = P.job[blockIdx.y];
    const int n = J.A.nkeys + 1, tid = threadIdx.x;
    if ((int)blockIdx.x << kKeyShift >= n) return;
    __shared__ uint32_t pre[kBucketTiles];   // stayers before each tile
    // this block's loads first; a key past the last reads the last key's
    const int base = ((int)blockIdx.x << kKeyShift) + tid * 4;
    unsigned long long cu[4];
    int x[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
        cu[u] = base + u < n ? J.A.kcnt[base + u] : 0ull;
        x[u] = J.A.offold[min(base + u, n - 1)];
    }
    constexpr int kT = kBucketTiles / 256;
    uint2 tc[kT];
#pragma unroll
    for (int u = 0; u < kT; u++)
        tc[u] = kT * tid + u < J.ntile ? J.A.tc[kT * tid + u] : make_uint2(0u, 0u);
    uint32_t before = 0;
    for (int b = tid; b < (int)blockIdx.x; b += 256) before += J.A.kpart[b];
    // stayers before an old offset, inside its tile (an offset at or past the
    // slot bound reads slot nub - 1's and takes the stayer total instead)
    uint32_t sb[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const int xs = min(x[u], J.A.nub - 1), wd = xs >> 6;
        sb[u] = (J.A.wsm[wd] & 0xffffu) +
                (uint32_t)__popcll(J.A.smask[wd] & ((1ull << (xs & 63)) - 1ull));
    }
    // tiles: stayers in the low half, movers in the high one
    uint64_t t = 0, tot, all, kbase;
#pragma unroll
    for (int u = 0; u < kT; u++) t += (uint64_t)tc[u].x | ((uint64_t)tc[u].y << 32);
    uint64_t ex = block_scan256(t, &tot);
#pragma unroll
    for (int u = 0; u < kT; u++) {
        pre[kT * tid + u] = (uint32_t)ex;
        if (blockIdx.x == 0 && kT * tid + u < J.ntile)   // for the placing kernels
            J.ts[kT * tid + u] = make_uint2((uint32_t)ex, (uint32_t)(ex >> 32));
        ex += (uint64_t)tc[u].x | ((uint64_t)tc[u].y << 32);
    }
    if (blockIdx.x == 0) {
        if (tid == 0) {
            J.gs[0] = make_uint2(0u, 0u);
            J.A.tot[0] = (uint32_t)tot;
            J.A.tot[1] = (uint32_t)(tot >> 32);
        }
    }
    (void)block_scan256(before, &kbase);     // its barriers also publish pre[]
    uint64_t sum = 0;
#pragma unroll
    for (int u = 0; u < 4; u++) sum += (uint32_t)cu[u];
    uint32_t lo = (uint32_t)(block_scan256(sum, &all) + kbase);
#pragma unroll
    for (int u = 0; u < 4; u++) {
        const int k = base + u;
        if (k >= n) break;
        const uint32_t stay = x[u] >= J.A.nub ? (uint32_t)tot : sb[u] + pre[x[u] >> kTileShift];
        const int v = (int)(stay + lo);
        J.offnew[k] = v;
        J.off[k] = (int32_t)lo;
        if (k == J.A.nkeys) {
            J.nalive[0] = v;
            J.nslots[0] = v;
            J.nsorted[0] = v;
        } else {
            J.mst[k] = (int32_t)(lo + (uint32_t)(cu[u] >> 32));
            if (cu[u]) J.A.kcnt[k] = 0ull;
        }
        lo += (uint32_t)cu[u];
    }
}

// n slots of a bucket in ascending order, by one workgroup: stable passes of
// 8 bits between a and b (as k_rs_scatter, one tile after the other); every
// thread of the workgroup calls it.  run: 256 words; wc: 256 per wave.
template <int T>
__device__ void sort_bucket(uint32_t *a, uint32_t *b, int n, int bits, uint32_t *run,
                            uint32_t (*wc)[256]) {
    const int tid = threadIdx.x, w = tid >> 6;
    const uint64_t below = lanes_below();
    uint32_t *src = a, *dst = b;
    for (int shift = 0; shift < bits; shift += 8) {
        if (tid < 256) run[tid] = 0;
        for (int u = tid; u < T / 64 * 256; u += T) wc[u >> 8][u & 255] = 0;
        __syncthreads();
        for (int i = tid; i < n; i += T) atomicAdd(&run[(src[i] >> shift) & 255u], 1u);
        __syncthreads();
        uint64_t tot;
        const uint32_t at = (uint32_t)block_scan<T>(tid < 256 ? run[tid] : 0u, &tot);
        if (tid < 256) run[tid] = at;
        __syncthreads();
        for (int i0 = 0; i0 < n; i0 += T) {
            const bool valid = i0 + tid < n;
            const uint32_t v = valid ? src[i0 + tid] : 0u;
            const uint32_t d = (v >> shift) & 255u;
            const uint64_t peers = digit_peers(d, valid);
            if (valid && (peers & below) == 0) wc[w][d] = (uint32_t)__popcll(peers);
            __syncthreads();
            if (valid) {
                uint32_t o = run[d] + (uint32_t)__popcll(peers & below);
                for (int u = 0; u < w; u++) o += wc[u][d];
                dst[o] = v;
            }
            __syncthreads();
            if (tid < 256) {
                uint32_t add = 0;
#pragma unroll
                for (int u = 0; u < T / 64; u++) {
                    add += wc[u][tid];
                    wc[u][tid] = 0;
                }
                run[tid] += add;
            }
            __syncthreads();
        }
        uint32_t *t = src;
        src = dst;
        dst = t;
    }
    if (src != a) {
        for (int i = tid; i < n; i += T) a[i] = src[i];
        __syncthreads();
    }
}

template <bool FP64>
__global__ void __launch_bounds__(kBucketThreads) k_bucket_fill(const BucketArgs P) {
    const BucketJob &J = P.job[blockIdx.y];
    if ((int)blockIdx.x >= J.ntile) return;
    constexpr int T = kBucketThreads, K = kTile / T;
    const int tid = threadIdx.x, lane = tid & 63;
    const int base = (int)blockIdx.x * kTile;
    __shared__ uint32_t done[kTile], run[256], wc[T / 64][256];
    __shared__ int ndone;
    if (tid == 0) ndone = 0;
    // the counts of the blocks of keys, zero again for the next sort
    if (blockIdx.x == 0)
        for (int b = tid; b << kKeyShift <= J.A.nkeys; b += T) J.A.kpart[b] = 0u;
    __syncthreads();
    const int wbase = __builtin_amdgcn_readfirstlane(base + (tid & ~63));
    uint32_t key[K], rank[K];
    bool mov[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int q0 = wbase + k * T, q = q0 + lane;
        mov[k] = q0 < J.A.nub && ((J.A.mmask[q0 >> 6] >> lane) & 1ull);
        key[k] = 0u;
        rank[k] = 0u;
        if (mov[k]) {
            if constexpr (FP64) {
                key[k] = J.A.keys[q];
            } else {
                key[k] = cell_key(J.A.cell[q], J.A.nth);
            }
            rank[k] = J.A.rank[q];
        }
    }
    int lo[K], hi[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        lo[k] = J.off[key[k]];
        hi[k] = J.off[key[k] + 1];
    }
#pragma unroll
    for (int k = 0; k < K; k++) {
        if (!mov[k]) continue;
        J.mq[(uint32_t)lo[k] + rank[k]] = (uint32_t)(wbase + k * T + lane);
        if (hi[k] - lo[k] > kBucketScan) {
            // the mover that completes a large bucket has it sorted here
            __threadfence();
            if ((int)atomicAdd(&J.A.kcnt[key[k]], 1ull) + 1 == hi[k] - lo[k]) {
                J.A.kcnt[key[k]] = 0ull;
                done[atomicAdd(&ndone, 1)] = key[k];
            }
        }
    }
    __syncthreads();
    const int nd = ndone;
    if (nd == 0) return;
    __threadfence();
    const int bits = 32 - __clz(J.A.nub);
    for (int i = 0; i < nd; i++) {
        const int l = J.off[done[i]], n = J.off[done[i] + 1] - l;
        sort_bucket<T>(J.mq + l, J.mq2 + l, n, bits, run, wc);
    }
}

// new place of the mover in slot q
__device__ __forceinline__ uint32_t mover_place(const BucketJob &J, const ClassView &V,
                                                uint32_t key, int q) {
    const int lo = J.off[key], hi = J.off[key + 1];
    const int o0 = J.A.offold[key], o1 = J.A.offold[key + 1];
    int rank = 0;
    if (hi - lo <= kBucketScan) {
        int i = lo;
        for (; i + 4 <= hi; i += 4) {
            const uint32_t a = J.mq[i], b = J.mq[i + 1], c = J.mq[i + 2], d = J.mq[i + 3];
            rank += (a < (uint32_t)q) + (b < (uint32_t)q) + (c < (uint32_t)q) + (d < (uint32_t)q);
        }
        for (; i < hi; i++) rank += J.mq[i] < (uint32_t)q;
    } else {
        rank = lower_bound_u32(J.mq, lo, hi, (uint32_t)q) - lo;
    }
    const int cq = q < o0 ? o0 : (q > o1 ? o1 : q);
    return (uint32_t)(lo + rank) + stayers_before(V, cq);
}

// stayers and movers to their places, one slot per thread in two rounds (so
// that the loads of both are in flight together)
template <typename T, int NA, bool FP64>
__global__ void __launch_bounds__(256) k_bucket_place(const BucketArgs P) {
    const BucketJob &J = P.job[blockIdx.y];
    const int q0 = (int)blockIdx.x * 512 + threadIdx.x;
    if (q0 - (int)threadIdx.x >= J.A.nub) return;
    const ClassView V = bucket_view(J);
    T v[2][NA];
#pragma unroll
    for (int k = 0; k < 2; k++)
#pragma unroll
        for (int a = 0; a < NA; a++)
            v[k][a] = q0 + k * 256 < V.nub ? ((const T *)J.src[a])[q0 + k * 256] : T(0);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int q = q0 + k * 256;
        if (q >= V.nub) continue;
        const uint64_t bit = 1ull << (q & 63);
        const bool stay = V.smask[q >> 6] & bit, move = V.mmask[q >> 6] & bit;
        if (!stay && !move) continue;         // holds no particle of the new order
        uint32_t key;
        if constexpr (FP64) {
            key = J.A.keys[q];
        } else {
            key = cell_key((int)v[k][0], J.A.nth);
        }
        const uint32_t d = stay ? stayers_before(V, q) + (uint32_t)J.mst[key]
                                : mover_place(J, V, key, q);
#pragma unroll
        for (int a = 0; a < NA; a++) ((T *)J.dst[a])[d] = v[k][a];
        if (J.perm) J.perm[d] = q;
    }
}

// For a push that places the sort: the place of the particle in every slot, -1
// for a slot that holds no particle of the new order
template <bool FP64>
__global__ void __launch_bounds__(256) k_bucket_dest(const BucketArgs P) {
    const BucketJob &J = P.job[blockIdx.y];
    const int q0 = (int)blockIdx.x * 512 + threadIdx.x;
    if (q0 - (int)threadIdx.x >= J.A.nub) return;
    const ClassView V = bucket_view(J);
    int c[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int q = q0 + k * 256;
        c[k] = q < V.nub ? (FP64 ? (int)J.A.keys[q] : J.A.cell[q]) : -1;
    }
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int q = q0 + k * 256;
        if (q >= V.nub) continue;
        const uint64_t bit = 1ull << (q & 63);
        const bool stay = V.smask[q >> 6] & bit, move = V.mmask[q >> 6] & bit;
        int32_t d = -1;
        if (stay || move) {
            const uint32_t key = FP64 ? (uint32_t)c[k] : cell_key(c[k], J.A.nth);
            d = (int32_t)(stay ? stayers_before(V, q) + (uint32_t)J.mst[key]
                               : mover_place(J, V, key, q));
            if (J.perm) J.perm[d] = q;
        }
        J.dest[q] = d;
    }
}

// ---------------------------------------------------------------------------

// Species of up to 2^21 slots on fewer than 2^21 cells: the key pass scans all
// tiles and sums the blocks of keys before its own, and a bucket that has most
// of a species in it is sorted by one workgroup.  Kernel time of a sort of both
// species, radix form against this one (sheets of width 0.05): 2.1e6 slots on
// 1024^2 308 / 104 us in FP32, 379 / 157 in FP64; on 512^2, with up to 1000
// movers to a cell, 285 / 112.  Above the line the radix passes are no longer
// all launch: 4.2e6 on 512^2 338 / 303, and 1e7 on 1024^2 lose.
static bool bucket_keys_ok(const ffpic_ctx *c) {
    return (int64_t)c->nr * c->nth < kBucketKeys;
}
bool bucket_sort_ok(const ffpic_ctx *c, int s) {
    return c->sort_valid[s] && c->incremental_sort && bucket_keys_ok(c) && c->sp[s].nub > 0 &&
           c->sp[s].nub <= kBucketSlots;
}

// one allocation per species: counts, block counts (both zero between sorts),
// offsets, buckets, their scratch, and the FP64 keys and ranks
static int64_t bucket_layout(const ffpic_ctx *c, int s, int64_t at[7]) {
    const int64_t nk1 = (int64_t)c->nr * c->nth + 1, cap = std::min(c->sp[s].cap, kBucketSlots);
    const int64_t len[7] = {2 * nk1, (nk1 >> kKeyShift) + 1, nk1, cap, cap, c->fp64 ? cap : 0,
                            c->fp64 ? cap : 0};
    int64_t n = 0;
    for (int k = 0; k < 7; k++) {
        at[k] = n;
        n += len[k];
    }
    return n;
}

void bucket_alloc(ffpic_ctx *c, int s, void *(*dmalloc)(size_t)) {
    if (!bucket_keys_ok(c) || c->sp[s].cap < 1) return;
    int64_t at[7];
    const size_t n = (size_t)bucket_layout(c, s, at) * 4;
    c->sort_bucket[s] = (uint32_t *)dmalloc(n);
    if (hipMemset(c->sort_bucket[s], 0, (size_t)at[2] * 4) != hipSuccess)
        throw std::runtime_error("hipMemset failed");
}

static BucketJob bucket_job(ffpic_ctx *c, int s, bool defer) {
    ffpic::Species &S = c->sp[s];
    const int t = c->sort_cur[s];
    int64_t at[7];
    (void)bucket_layout(c, s, at);
    uint32_t *mem = c->sort_bucket[s];
    BucketJob J{};
    ClassArgs &A = J.A;
    A.nub = (int)S.nub;
    A.nth = c->nth;
    A.nr = c->nr;
    A.dead = dead_key(c);
    A.nslots = c->nslots + s;
    A.nsorted = c->nsorted + s;
    A.kill = c->kill;
    A.offold = c->soff[s][t];
    A.removed = c->removed + 4 * s;
    A.smask = c->sort_smask[s];
    A.mmask = c->sort_mmask[s];
    A.wsm = c->sort_wsm[s];
    A.tc = c->sort_tc[s];
    A.tot = c->sort_tot[s];
    A.kcnt = (unsigned long long *)(mem + at[0]);
    A.kpart = mem + at[1];
    if (c->fp64) {
        A.R = (double *)S.cur[0];
        A.TH = (const double *)S.cur[1];
        A.rn = c->dtab64[T_RN];
        A.thn = c->dtab64[T_THN];
        A.rmin = c->d.rmin;
        A.dlog = c->dlog;
        A.dth = c->dth;
        A.keys = mem + at[5];
        A.rank = mem + at[6];
    } else {
        A.cell = (int32_t *)S.cur[0];
        A.rank = (uint32_t *)c->sort_dest[s];   // until the places are written
    }
    J.ntile = (A.nub + kTile - 1) / kTile;
    A.nkeys = c->nr * c->nth;
    J.ts = c->sort_ts[s];
    J.gs = c->sort_gs[s];
    J.off = (int32_t *)(mem + at[2]);
    J.mq = mem + at[3];
    J.mq2 = mem + at[4];
    J.mst = c->sort_mst[s];
    J.offnew = c->soff[s][1 - t];
    J.nalive = c->nalive + s;
    J.nslots = c->nslots + s;
    J.nsorted = c->nsorted + s;
    J.dest = defer ? c->sort_dest[s] : nullptr;
    J.perm = perm_out(c, s);
    for (int a = 0; a < S.narr; a++) {
        J.src[a] = S.cur[a];
        J.dst[a] = S.alt[a];
    }
    return J;
}

// sorts n species (each with bucket_sort_ok, all FP64 or all FP32) on stream
// st; with defer their next pushes place the particles
void sort_bucketed(const SortItem *items, int n, hipStream_t st, bool defer) {
    for (int i0 = 0; i0 < n; i0 += kBucketJobs) {
        const int m = std::min(n - i0, kBucketJobs);
        BucketArgs P{};
        int ntile = 1, nbk = 1, nub = 1;
        const bool fp64 = items[i0].c->fp64;
        for (int k = 0; k < m; k++) {
            BucketJob &J = P.job[k];
            J = bucket_job(items[i0 + k].c, items[i0 + k].s, defer);
            ntile = std::max(ntile, J.ntile);
            nbk = std::max(nbk, (J.A.nkeys >> kKeyShift) + 1);
            nub = std::max(nub, J.A.nub);
        }
        const dim3 tiles(ntile, m), wide(kBucketThreads), blk(256), place((nub + 511) / 512, m);
        if (fp64) {
            hipLaunchKernelGGL(k_bucket_classify<true>, tiles, wide, 0, st, P);
            hipLaunchKernelGGL(k_bucket_keys, dim3(nbk, m), blk, 0, st, P);
            hipLaunchKernelGGL(k_bucket_fill<true>, tiles, wide, 0, st, P);
            if (defer) hipLaunchKernelGGL(k_bucket_dest<true>, place, blk, 0, st, P);
            else hipLaunchKernelGGL((k_bucket_place<uint64_t, 5, true>), place, blk, 0, st, P);
        } else {
            hipLaunchKernelGGL(k_bucket_classify<false>, tiles, wide, 0, st, P);
            hipLaunchKernelGGL(k_bucket_keys, dim3(nbk, m), blk, 0, st, P);
            hipLaunchKernelGGL(k_bucket_fill<false>, tiles, wide, 0, st, P);
            if (defer) hipLaunchKernelGGL(k_bucket_dest<false>, place, blk, 0, st, P);
            else hipLaunchKernelGGL((k_bucket_place<uint32_t, 6, false>), place, blk, 0, st, P);
        }
        FFPIC_LAUNCH_CHECK();
        for (int k = 0; k < m; k++) {
            ffpic_ctx *c = items[i0 + k].c;
            const int s = items[i0 + k].s;
            ffpic::Species &S = c->sp[s];
            c->sort_cur[s] = 1 - c->sort_cur[s];
            if (defer) {
                place_by_push(c, s);
            } else {
                for (int a = 0; a < S.narr; a++) std::swap(S.cur[a], S.alt[a]);
            }
        }
    }
}

}  // namespace ffpic
