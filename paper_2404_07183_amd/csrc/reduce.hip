// reduce.hip -- reductions of groups of PCFs (paper, Section 2.1
// "Combinations and reductions"; Section 4, reduction trees and Algorithm
// ReducePair): sum, max and min by the induced reduction, mean = sum / n and
// the sample standard deviation sqrt(sum_i (f_i - mean)^2 / (n - 1)); and
// the combinations h_*(x_i, y_i) of two sets (also a - b, ab, (a - b)^2) as
// reductions of the interleaved set in groups of two.
//
// Tree. A group of M PCFs is reduced by a binary tree: at level l the items
// 2j and 2j+1 (each covering 2^l consecutive PCFs) are merged into item j of
// level l+1, and an unpaired last item moves up unchanged. Every group takes
// the same ceil(log2 M_max) levels, up to four of them in one pass for all
// groups (red_fuse), or, where the groups are many and short (kFuseFew,
// kFuseRows) and for trees of one level, a launch a level (red_level).
//
// Merge without compaction. A level keeps every position of the merged
// breakpoint lists (ties: the first list first), so item j of level l+1
// holds exactly the rows of its 2^(l+1) PCFs, in the same place: position q
// of a pair is row offsets[first PCF] + q of the output buffer. Every row
// with time x carries h(f(x), g(x)): a list's value at x is its next row's
// when that row also lies at x (all rows at one time carry the same value,
// by induction from the strictly increasing inputs), else its last row's.
// Positions are independent given the merge state, so one launch covers all
// rows of all pairs (red_level: a lane walks kMergeK consecutive rows after a
// merge-path search, moving on to the next pair in place when it crosses
// one). ReducePair's row rule (keep t = 0 and value changes) is applied once,
// to the root, where runs of rows at one time collapse to their first: the
// same function and the same minimal rows as pruning at every level, since
// the values at each breakpoint do not depend on which rows the
// intermediate PCFs kept. The root pass is cut into chunks of rows; red_scan
// turns the chunk counts into output offsets.
//
// Standard deviation. For every breakpoint x of the group's root,
// (f_i(x) - mean(x))^2 is summed over i in the tree's order (a binary
// counter over i reproduces the level-by-level pairing), then the root rule
// and x -> sqrt(x / (n - 1)) are applied.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "launch.hpp"
#include "reduce.hpp"

namespace pcf {

namespace {

// merged positions per lane (4 measured fastest against 2, 8 and 16)
constexpr int kMergeK = 4;
// waves a workgroup of the level kernel
constexpr int kLevelWaves = 8;  // (3 % faster than 4, 11 % faster than 1)
constexpr int kChunkRows = 1024;  // rows per wave in the root pass
constexpr int64_t kStdSmall = 64;  // groups of at most this many PCFs: red_std_small

template <typename T, int OP>
__device__ __forceinline__ T red_op(T a, T b)
{
    if constexpr (OP == RO_MAX)
        return a >= b ? a : b;
    else if constexpr (OP == RO_MIN)
        return a <= b ? a : b;
    else if constexpr (OP == RO_SUB)
        return a - b;
    else if constexpr (OP == RO_MUL)
        return a * b;
    else if constexpr (OP == RO_SQDIFF)
        return (a - b) * (a - b);
    else
        return a + b;
}

// Last index k in [0, n) with x[k] <= r (x[0] <= r).
__device__ __forceinline__ int64_t last_le(const int64_t *x, int64_t n, int64_t r)
{
    int64_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (x[mid] <= r)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The pair of a level that holds a row: its lists' row ranges and the row
// where the pair's output begins.
struct PairAt {
    int64_t b;         // group
    int64_t iA, iE;    // first PCF of the pair, one past its last PCF
    int64_t sA, nA, sB, nB;
};

__device__ __forceinline__ void pair_from(const RedLevelArgs &a, int64_t b, int64_t iA,
                                          int64_t span, PairAt &p)
{
    const int64_t ge = a.groups[b + 1];
    const int64_t iB = iA + span < ge ? iA + span : ge;
    const int64_t iE = iA + 2 * span < ge ? iA + 2 * span : ge;
    p.b = b;
    p.iA = iA;
    p.iE = iE;
    p.sA = a.offsets[iA];
    p.sB = a.offsets[iB];
    p.nA = p.sB - p.sA;
    p.nB = a.offsets[iE] - p.sB;
}

}  // namespace

// Wave-private ordering of LDS accesses (the staging buffers are per wave).
__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave takes 64 * kMergeK consecutive rows; lane l walks rows
// l * kMergeK .. of them. The results go through a wave-private LDS buffer
// so that the stores to memory are coalesced.
template <typename T, int OP>
__global__ __launch_bounds__(64 * kLevelWaves) void red_level(RedLevelArgs a)
{
    const T *__restrict__ tin = reinterpret_cast<const T *>(a.tin);
    const T *__restrict__ vin = reinterpret_cast<const T *>(a.vin);
    T *__restrict__ tout = reinterpret_cast<T *>(a.tout);
    T *__restrict__ vout = reinterpret_cast<T *>(a.vout);
    constexpr int64_t kPerWave = 64 * kMergeK;
    __shared__ T st_t[kLevelWaves][kPerWave], st_v[kLevelWaves][kPerWave];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t span = (int64_t)1 << a.level;
    const int64_t r0g = a.offsets[a.groups[0]], r1g = a.offsets[a.groups[a.B]];
    for (int64_t wb = r0g + ((int64_t)blockIdx.x * kLevelWaves + wv) * kPerWave; wb < r1g;
         wb += (int64_t)gridDim.x * kLevelWaves * kPerWave) {
        const int64_t r0 = wb + (int64_t)lane * kMergeK;
        if (r0 < r1g) {
            const int64_t r1 = r0 + kMergeK < r1g ? r0 + kMergeK : r1g;
            // the pair holding row r0, and the merge state at its position
            const int64_t pcf = a.row_pcf[r0];
            const int64_t b = last_le(a.groups, (int64_t)a.B + 1, pcf);
            PairAt p;
            pair_from(a, b, a.groups[b] + ((pcf - a.groups[b]) / (2 * span)) * (2 * span), span,
                      p);
            int64_t q = r0 - p.sA;
            int64_t i, j;
            {
                int64_t lo = q - p.nB > 0 ? q - p.nB : 0, hi = q < p.nA ? q : p.nA;
                const T *tA = tin + p.sA, *tB = tin + p.sB;
                while (lo < hi) {  // A's share of the first q merged positions
                    const int64_t mid = (lo + hi) >> 1;
                    if (tA[mid] <= tB[q - 1 - mid])
                        lo = mid + 1;
                    else
                        hi = mid;
                }
                i = lo;
                j = q - lo;
            }
            for (int64_t r = r0; r < r1; ++r) {
                if (q == p.nA + p.nB) {  // crossed into the next pair (or group)
                    int64_t nb = p.b, ni = p.iE;
                    if (ni == a.groups[nb + 1])
                        ++nb;
                    pair_from(a, nb, ni, span, p);
                    q = i = j = 0;
                }
                const T *tA = tin + p.sA, *vA = vin + p.sA, *tB = tin + p.sB, *vB = vin + p.sB;
                T x, val;
                if (p.nB == 0) {  // unpaired: moves up unchanged
                    x = tA[q];
                    val = vA[q];
                } else {
                    T fx, gx;
                    if (i < p.nA && (j >= p.nB || tA[i] <= tB[j])) {
                        x = tA[i];
                        fx = vA[i];
                        ++i;
                        gx = (j < p.nB && tB[j] == x) ? vB[j] : vB[j > 0 ? j - 1 : 0];
                    } else {
                        x = tB[j];
                        gx = vB[j];
                        ++j;
                        fx = (i < p.nA && tA[i] == x) ? vA[i] : vA[i > 0 ? i - 1 : 0];
                    }
                    val = red_op<T, OP>(fx, gx);
                }
                st_t[wv][r - wb] = x;
                st_v[wv][r - wb] = val;
                ++q;
            }
        }
        wave_sync_lds();
        const int64_t cnt = r1g - wb < kPerWave ? r1g - wb : kPerWave;
        for (int64_t k = lane; k < cnt; k += 64) {
            tout[wb + k] = st_t[wv][k];
            vout[wb + k] = st_v[wv][k];
        }
        wave_sync_lds();
    }
}


// ---------------------------------------------------------------------------
// Several levels of the tree in one pass.
//
// A level run alone reads and writes every row and is bound by the chain of
// dependent loads in front of each window (its pair, the offsets, a search of
// up to 21 steps): 76 us for 5.5 million FP64 rows at any level. Here a bundle
// of up to 16 items is merged a tile at a time, four levels in LDS, so a row
// crosses memory once for four levels: 91 us, and 44 us for the tiles' starts.
//
// Tiles. Rows of a bundle are ordered by (time, item, index), the order of
// the levels' outputs. Every item is sampled each kFuseSpacing rows; a tile
// starts at every kFuseRanks-th sample of the bundle in that order. Between two
// neighbouring starts an item has fewer than kFuseSpacing rows beyond those of
// its samples there, so a tile holds at most kFuseTile rows (24 * 48 on
// average), whatever the data. That is 31 KiB of LDS in FP64, five workgroups a
// CU; 16 x 64 (four workgroups) takes 111 us, 32 x 64 119 us, 8 x 64 127 us.
// red_split finds the samples' ranks, one lane for every (sample, item): a
// search of the item's samples, summed over the sample's 16 lanes; a sample
// that starts a tile goes on to its exact row in each item.
//
// Values. A row at time x carries h of both sides' values at x (file comment);
// a side's value at x may come from the row before its part of the tile, or,
// on equal times, from the row after it. Both are loaded with the tile and
// merged like the rows: the value before, and the time and value after.

// Entries t[0], t[stride], .. (n of them, in order) below x, or, with `before`,
// at x too.
template <typename T>
__device__ __forceinline__ int64_t fuse_count(const T *t, int64_t n, int64_t stride, T x,
                                              bool before)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        const T y = t[mid * stride];
        if (y < x || (before && y == x))
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

constexpr int kSplitBatch = 2;  // samples of sixteen lanes at once (independent searches)

template <typename T>
__global__ __launch_bounds__(256) void red_split(RedFuseArgs a)
{
    constexpr int N = kSplitBatch;
    const T *__restrict__ tin = reinterpret_cast<const T *>(a.tin);
    const int l = threadIdx.x & (kFuseLists - 1);
    const int shift = (threadIdx.x & 63) & ~(kFuseLists - 1);
    const int64_t per = (int64_t)blockDim.x / kFuseLists * N;
    const int64_t span = (int64_t)1 << a.level;
    // (whole groups of lanes: the lanes past the end repeat the last sample)
    for (int64_t s0 = blockIdx.x * per; s0 < a.nsamples; s0 += gridDim.x * per) {
        int64_t bun[N], tile0[N], r[N], n[N], m[N], ui[N], c[N];
        int own[N];
        bool live[N];
        T x[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int64_t sk = s0 + (int64_t)(threadIdx.x / kFuseLists) * N + k;
            live[k] = sk < a.nsamples;
            const int64_t s = live[k] ? sk : a.nsamples - 1;
            // the bundle of sample s, sixteen candidates a round (the second
            // sample's is the first's or lies after it)
            int64_t lo = k == 0 ? 0 : bun[0];
            int64_t width = k == 0 ? a.nbundles : 1;
            if (k > 0 && lo + 1 < a.nbundles && a.bundles[lo + 1].sample0 <= s)
                width = a.nbundles - lo;
            while (width > 1) {
                const int64_t step = (width + kFuseLists - 1) / kFuseLists;
                const bool le = l * step < width && a.bundles[lo + l * step].sample0 <= s;
                const int got = __popcll((__ballot(le) >> shift) & 0xffffu);  // at least 1
                lo += (got > 0 ? got - 1 : 0) * step;
                width -= (got > 0 ? got - 1 : 0) * step;
                width = width < step ? width : step;
            }
            const RedBundle b = a.bundles[lo];
            bun[k] = lo;
            tile0[k] = b.tile0;
            // lane l: item l's rows and samples
            const int64_t p = b.p0 + l * span < b.pend ? b.p0 + l * span : b.pend;
            const int64_t pe = p + span < b.pend ? p + span : b.pend;
            r[k] = a.offsets[p];
            n[k] = a.offsets[pe] - r[k];
            m[k] = (n[k] + kFuseSpacing - 1) / kFuseSpacing;
            int64_t inc = m[k];
#pragma unroll
            for (int h = 1; h < kFuseLists; h <<= 1) {
                const int64_t o = __shfl_up(inc, h, kFuseLists);
                if (l >= h)
                    inc += o;
            }
            // the sample's item (its samples hold number s - sample0), and
            // its number there
            const int64_t u = s - b.sample0;
            const bool mine = u >= inc - m[k] && u < inc;
            const uint64_t vote = __ballot(mine) >> shift;
            own[k] = __builtin_ctz((unsigned)(vote & 0xffffu) | 0x8000u);
            ui[k] = u - __shfl(inc - m[k], own[k], kFuseLists);
            x[k] = tin[__shfl(r[k], own[k], kFuseLists) + ui[k] * kFuseSpacing];
        }
        // samples of every item below x: the searches in step
        int64_t lo[N], hi[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            lo[k] = l == own[k] ? ui[k] : 0;
            hi[k] = l == own[k] ? ui[k] : m[k];
        }
        for (;;) {
            bool more = false;
            T y[N];
#pragma unroll
            for (int k = 0; k < N; ++k)
                if (lo[k] < hi[k])
                    y[k] = tin[r[k] + ((lo[k] + hi[k]) >> 1) * kFuseSpacing];
#pragma unroll
            for (int k = 0; k < N; ++k)
                if (lo[k] < hi[k]) {
                    const int64_t mid = (lo[k] + hi[k]) >> 1;
                    if (y[k] < x[k] || (l < own[k] && y[k] == x[k]))
                        lo[k] = mid + 1;
                    else
                        hi[k] = mid;
                    more = more || lo[k] < hi[k];
                }
            if (!more)
                break;
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            c[k] = lo[k];
            int64_t rank = c[k];
#pragma unroll
            for (int h = 1; h < kFuseLists; h <<= 1)
                rank += __shfl_xor(rank, h, kFuseLists);
            if (live[k] && rank % kFuseRanks == 0) {
                // exact: between the last sample below x and the next one
                int64_t at = 0;
                if (l == own[k]) {
                    at = ui[k] * kFuseSpacing;
                } else if (c[k] > 0) {
                    const int64_t base = (c[k] - 1) * kFuseSpacing + 1;
                    const int64_t end = c[k] * kFuseSpacing < n[k] ? c[k] * kFuseSpacing : n[k];
                    at = base + fuse_count<T>(tin + r[k] + base, end > base ? end - base : 0, 1,
                                              x[k], l < own[k]);
                }
                int64_t *to = a.split + (tile0[k] + rank / kFuseRanks) * kFuseSplit;
                to[l] = at;
                if (l == own[k])
                    to[kFuseLists] = bun[k];
            }
        }
    }
}

// (with 512 threads the searches double and the pass takes 146 us; with 128,
// 149 us: too few waves)
constexpr int kFuseThreads = 256;
constexpr int kFuseRun = (kFuseTile + kFuseThreads - 1) / kFuseThreads;  // most rows a thread
static_assert(kFuseRun * kFuseThreads >= kFuseTile, "a thread's run of a full tile");

template <typename T> struct FuseNode {
    T before, after_v, after_t;  // value before the tile's rows; the row after them
};

template <typename T, int OP>
__global__ __launch_bounds__(kFuseThreads, sizeof(T) == 8 ? 5 : 7) void red_fuse(RedFuseArgs a)
{
    const T *__restrict__ tin = reinterpret_cast<const T *>(a.tin);
    const T *__restrict__ vin = reinterpret_cast<const T *>(a.vin);
    T *__restrict__ tout = reinterpret_cast<T *>(a.tout);
    T *__restrict__ vout = reinterpret_cast<T *>(a.vout);
    __shared__ T lt[kFuseTile], lv[kFuseTile];
    __shared__ FuseNode<T> node[2][kFuseLists];
    __shared__ int32_t seg[2][kFuseLists + 1];
    __shared__ int64_t src[kFuseLists];  // first row of each item's part
    __shared__ int64_t first_out;
    const int tid = threadIdx.x;
    const int64_t span = (int64_t)1 << a.level;
    const T inf = __builtin_inf();
    for (int64_t tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
        // (in bounds also for times that break the order)
        int64_t lo = a.split[tile * kFuseSplit + kFuseLists];
        lo = lo < 0 ? 0 : (lo < a.nbundles ? lo : a.nbundles - 1);
        const RedBundle b = a.bundles[lo];
        const int64_t tend = lo + 1 < a.nbundles ? a.bundles[lo + 1].tile0 : a.ntiles;
        const int items = (int)((b.pend - b.p0 + span - 1) / span);
        if (tid < kFuseLists) {
            const int64_t p = b.p0 + tid * span < b.pend ? b.p0 + tid * span : b.pend;
            const int64_t pe = p + span < b.pend ? p + span : b.pend;
            const int64_t r = a.offsets[p], n = a.offsets[pe] - r;
            int64_t s = a.split[tile * kFuseSplit + tid];
            int64_t e = tile + 1 < tend ? a.split[(tile + 1) * kFuseSplit + tid] : n;
            s = s < 0 ? 0 : (s < n ? s : n);
            e = e < s ? s : (e < n ? e : n);
            int64_t skip = s;  // rows of the bundle before the tile
            int32_t inc = e - s < kFuseTile ? (int32_t)(e - s) : kFuseTile;
            const int32_t len = inc;
#pragma unroll
            for (int h = 1; h < kFuseLists; h <<= 1) {
                const int32_t o = __shfl_up(inc, h, kFuseLists);
                if (tid >= h)
                    inc += o;
                skip += __shfl_xor(skip, h, kFuseLists);
            }
            const int32_t end = inc < kFuseTile ? inc : kFuseTile;
            const int32_t beg = inc - len < kFuseTile ? inc - len : kFuseTile;
            e = s + (end - beg);
            seg[0][tid + 1] = end;
            if (tid == 0) {
                seg[0][0] = 0;
                first_out = a.offsets[b.p0] + skip;
            }
            src[tid] = r + s;
            FuseNode<T> d;
            d.before = n > 0 ? vin[r + (s > 0 ? s - 1 : 0)] : T(0);
            d.after_t = e < n ? tin[r + e] : inf;
            d.after_v = e < n ? vin[r + e] : T(0);
            node[0][tid] = d;
        }
        __syncthreads();
        const int32_t total = seg[0][kFuseLists];
        for (int32_t q = tid; q < total; q += kFuseThreads) {
            int l = 0;  // the item whose part holds row q
#pragma unroll
            for (int h = kFuseLists / 2; h > 0; h >>= 1)
                l += seg[0][l + h] <= q ? h : 0;
            const int64_t r = src[l] + (q - seg[0][l]);
            lt[q] = tin[r];
            lv[q] = vin[r];
        }
        __syncthreads();
        const int32_t run = (total + kFuseThreads - 1) / kFuseThreads;
        const int32_t q0 = tid * run;
        const int32_t q1 = q0 + run < total ? q0 + run : total;
        int cnt = items;
        for (int lev = 0; lev < a.depth; ++lev) {
            const int32_t *sg = seg[lev & 1];
            const FuseNode<T> *nd = node[lev & 1];
            const int pairs = (cnt + 1) / 2;
            T xt[kFuseRun], xv[kFuseRun];
            if (q0 < q1) {
                int k = 0;  // the pair that holds row q0
#pragma unroll
                for (int h = kFuseLists / 4; h > 0; h >>= 1)
                    k += k + h < pairs && sg[2 * (k + h)] <= q0 ? h : 0;
                int32_t sA = sg[2 * k], sB = sg[2 * k + 1];
                int32_t nA = sB - sA, nB = 2 * k + 1 < cnt ? sg[2 * k + 2] - sB : 0;
                int32_t q = q0 - sA, i, j;
                {
                    int32_t l = q - nB > 0 ? q - nB : 0, h = q < nA ? q : nA;
                    while (l < h) {  // A's share of the first q merged rows
                        const int32_t mid = (l + h) >> 1;
                        if (lt[sA + mid] <= lt[sB + (q - 1 - mid)])
                            l = mid + 1;
                        else
                            h = mid;
                    }
                    i = l;
                    j = q - l;
                }
// both sides' next rows (or the ones after their parts) and the
                // values before those
                T tA, vA, pA, tB, vB, pB;
                auto heads = [&]() {
                    const FuseNode<T> &na = nd[2 * k];
                    tA = i < nA ? lt[sA + i] : na.after_t;
                    vA = i < nA ? lv[sA + i] : na.after_v;
                    pA = i > 0 ? lv[sA + i - 1] : na.before;
                    tB = vB = pB = T(0);
                    if (2 * k + 1 < cnt) {
                        const FuseNode<T> &nb = nd[2 * k + 1];
                        tB = j < nB ? lt[sB + j] : nb.after_t;
                        vB = j < nB ? lv[sB + j] : nb.after_v;
                        pB = j > 0 ? lv[sB + j - 1] : nb.before;
                    }
                };
                heads();
#pragma unroll
                for (int u = 0; u < kFuseRun; ++u) {
                    if (q0 + u < q1) {
                        if (q == nA + nB) {
                            do {  // the next pair with rows
                                ++k;
                                sA = sg[2 * k];
                                sB = sg[2 * k + 1];
                                nA = sB - sA;
                                nB = 2 * k + 1 < cnt ? sg[2 * k + 2] - sB : 0;
                            } while (nA + nB == 0);
                            q = i = j = 0;
                            heads();
                        }
                        const bool fromA = i < nA && (j >= nB || tA <= tB);
                        const T x = fromA ? tA : tB, y = fromA ? vA : vB;
                        const T ot = fromA ? tB : tA;
                        const T z = ot == x ? (fromA ? vB : vA) : (fromA ? pB : pA);
                        xt[u] = x;
                        // (an unpaired item moves up unchanged)
                        xv[u] = 2 * k + 1 >= cnt ? y
                                : fromA          ? red_op<T, OP>(y, z)
                                                 : red_op<T, OP>(z, y);
                        ++q;
                        if (fromA) {
                            ++i;
                            pA = y;
                            tA = i < nA ? lt[sA + i] : nd[2 * k].after_t;
                            vA = i < nA ? lv[sA + i] : nd[2 * k].after_v;
                        } else {
                            ++j;
                            pB = y;
                            tB = j < nB ? lt[sB + j] : nd[2 * k + 1].after_t;
                            vB = j < nB ? lv[sB + j] : nd[2 * k + 1].after_v;
                        }
                    }
                }
            }
            // the pairs' parts and the values around them
            if (tid < pairs) {
                FuseNode<T> d = nd[2 * tid];
                int32_t end = sg[2 * tid + 1];
                if (2 * tid + 1 < cnt) {
                    const FuseNode<T> A = d, Bn = nd[2 * tid + 1];
                    const int32_t sA = sg[2 * tid], sB = end;
                    end = sg[2 * tid + 2];
                    d.before = red_op<T, OP>(A.before, Bn.before);
                    d.after_t = A.after_t <= Bn.after_t ? A.after_t : Bn.after_t;
                    const T va = A.after_t == d.after_t ? A.after_v
                                                        : (sB > sA ? lv[sB - 1] : A.before);
                    const T vb = Bn.after_t == d.after_t ? Bn.after_v
                                                         : (end > sB ? lv[end - 1] : Bn.before);
                    d.after_v = red_op<T, OP>(va, vb);
                }
                node[(lev + 1) & 1][tid] = d;
                seg[(lev + 1) & 1][tid + 1] = end;
                if (tid == 0)
                    seg[(lev + 1) & 1][0] = 0;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kFuseRun; ++u)
                if (q0 + u < q1) {
                    lt[q0 + u] = xt[u];
                    lv[q0 + u] = xv[u];
                }
            __syncthreads();
            cnt = pairs;
        }
        for (int32_t q = tid; q < total; q += kFuseThreads) {
            tout[first_out + q] = lt[q];
            vout[first_out + q] = lv[q];
        }
        __syncthreads();  // (the tile's tables are rewritten next)
    }
}

// row_pcf[r] = the PCF holding row r: one wave per PCF.
__global__ void red_rowmap(const int64_t *__restrict__ offsets, int64_t n,
                           int32_t *__restrict__ row_pcf)
{
    const int lane = threadIdx.x & 63;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; i < n;
         i += nwaves)
        for (int64_t r = offsets[i] + lane; r < offsets[i + 1]; r += 64)
            row_pcf[r] = (int32_t)i;
}

// Sum over i of (f_i(x) - mean(x))^2 at every root breakpoint x, in the
// tree's order, for the rows of groups of more than kStdSmall PCFs: a binary
// search of every PCF of the group per root row.
template <typename T>
__global__ void red_std_terms(RedStdArgs a)
{
#pragma clang fp contract(off)
    const T *__restrict__ t = reinterpret_cast<const T *>(a.t);
    const T *__restrict__ v = reinterpret_cast<const T *>(a.v);
    const T *__restrict__ rt = reinterpret_cast<const T *>(a.rt);
    const T *__restrict__ rv = reinterpret_cast<const T *>(a.rv);
    T *__restrict__ q = reinterpret_cast<T *>(a.q);
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < a.rows;
         r += (int64_t)gridDim.x * blockDim.x) {
        // the group whose root holds row r: last b with offsets[groups[b]] <= r
        int32_t lo = 0, hi = a.B - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (a.offsets[a.groups[mid]] <= r)
                lo = mid;
            else
                hi = mid - 1;
        }
        const int64_t gb = a.groups[lo], ge = a.groups[lo + 1];
        if (ge - gb <= kStdSmall)
            continue;  // red_std_small's rows
        const T x = rt[r];
        const T mean = rv[r] / (T)(ge - gb);
        // binary counter over the group's PCFs: after k terms, st[h] holds
        // the sum of a complete subtree of 2^h terms for every set bit h of
        // k (the level-by-level pairing), in two levels of 15 heights
        // (blocks of 2^15 terms, then blocks; groups below 2^30 PCFs) so
        // that the loops unroll to constant indices into small arrays.
        constexpr int kIn = 15;
        T st[kIn], st2[kIn];
        int64_t k = 0;
        for (int64_t i = gb; i < ge; ++i, ++k) {
            const int64_t o = a.offsets[i], ni = a.offsets[i + 1] - o;
            int64_t l = 0, h = ni;  // rows with t <= x
            while (l < h) {
                const int64_t m = (l + h) >> 1;
                if (t[o + m] <= x)
                    l = m + 1;
                else
                    h = m;
            }
            const T d = v[o + (l > 0 ? l - 1 : 0)] - mean;
            T s = d * d;
            bool placed = false;
#pragma unroll
            for (int hh = 0; hh < kIn; ++hh) {
                if ((k >> hh) & 1) {
                    s = st[hh] + s;
                } else {
                    st[hh] = s;
                    placed = true;
                    break;
                }
            }
            if (!placed) {  // a complete block of 2^15 terms
                const int64_t kb = k >> kIn;
#pragma unroll
                for (int hh = 0; hh < kIn; ++hh) {
                    if ((kb >> hh) & 1) {
                        s = st2[hh] + s;
                    } else {
                        st2[hh] = s;
                        break;
                    }
                }
            }
        }
        // fold the partial sums from the smallest subtree up
        const int64_t M = ge - gb;
        T acc = T(0);
        bool have = false;
#pragma unroll
        for (int hh = 0; hh < kIn; ++hh) {
            if ((M >> hh) & 1) {
                acc = have ? st[hh] + acc : st[hh];
                have = true;
            }
        }
#pragma unroll
        for (int hh = 0; hh < kIn; ++hh) {
            if (((M >> kIn) >> hh) & 1) {
                acc = have ? st2[hh] + acc : st2[hh];
                have = true;
            }
        }
        q[r] = acc;
    }
}

// The same sums for groups of at most kStdSmall PCFs: one block per chunk of
// root rows (the root pass's chunks).
//
// The root of a group holds every row of its PCFs once (the levels keep all
// merged positions). For chunk [c0, c1) with first time xf, and x1 the first
// time of the group's next chunk, the rows of PCF i that the chunk's times
// can select lie between its row at or before xf and its row at or before x1
// (its last row for the group's last chunk): together at most
// (c1 - c0) + 2m - 1 rows over the group (one per root row c0 + 1 .. c1,
// m - 1 more that tie with x1 past it, and the m rows at or before xf).
// red_std_bounds bisects every PCF once per chunk for the rows at or before
// xf; red_std_small stages the window of (t, v) records in LDS.
//
// A record of the window that lies past xf is one root row of the chunk: it
// is found there by one bisection of the chunk's times, and its PCF noted as
// the row's owner (any order within a run of equal times will do, since every
// row of the run selects by the run's last). The record that PCF i gives a row
// is then a count: its records before the row's block of 64, and, by a ballot
// over the block's owners, those up to the row. One bisection a record in place
// of one for every PCF and two rows: 1,000 groups of 20 PCFs, 5.5 million FP64
// rows, 111 us against 166 (bound by the chain of dependent reads of a chunk:
// at 64 VGPRs, and so four blocks a CU, 111 us, at 78 VGPRs and three 133). A
// block whose last row ties with the next one bisects every PCF for each of its
// rows instead. Each lane takes one row and adds
// (f_i(x) - mean(x))^2 to a binary counter, which sums the m terms in the
// reduction tree's order (pairs (2j, 2j + 1), then pairs of pairs, an unpaired
// last block moving up), as red_std_terms.
constexpr int kStdThreads = 512;
constexpr int kStdBlocks = kChunkRows / 64;
constexpr int kStdRows = kChunkRows / kStdThreads;
constexpr int kStdWindow = kChunkRows + 2 * (int)kStdSmall;
constexpr int kStdLoads = (kStdWindow + kStdThreads - 1) / kStdThreads;
constexpr int kStdBatch = 4;  // PCFs whose values are read together
constexpr int kStdHeights = 5;  // subtrees of kStdBatch 2^h terms
static_assert(kChunkRows % kStdThreads == 0 && kStdSmall == 64 &&
                  (kStdBatch << kStdHeights) > kStdSmall,
              "red_std_small's layout");

// chunk_first[64c + i] = the last row of PCF i (i < m) with t at or before
// the first root time of chunk c, for the chunks of groups of at most
// kStdSmall PCFs.
template <typename T>
__global__ void red_std_bounds(RedStdArgs a)
{
    const T *__restrict__ t = reinterpret_cast<const T *>(a.t);
    const T *__restrict__ rt = reinterpret_cast<const T *>(a.rt);
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < a.nchunks * kStdSmall;
         u += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = u / kStdSmall, i = u % kStdSmall;
        const int64_t b = a.chunk_grp[c];
        const int64_t gb = a.groups[b], m = a.groups[b + 1] - gb;
        if (m > kStdSmall || i >= m)
            continue;
        const T x = rt[a.chunk_row[c]];
        const int64_t o = a.offsets[gb + i], n = a.offsets[gb + i + 1] - o;
        int64_t lo = 0, hi = n - 1;  // t[o] = 0 <= x
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (t[o + mid] <= x)
                lo = mid;
            else
                hi = mid - 1;
        }
        a.chunk_first[u] = lo;
    }
}

template <typename T>
struct StdRecord {
    T t, v;
};

// Subtree number j (from 0) of kStdBatch terms in the binary counter: after
// j + 1 of them st[h] holds a complete subtree of kStdBatch 2^h terms for every
// set bit h of j + 1; s joins the subtrees below the lowest clear bit of j,
// smallest first, each on the left. (Fixed indices: a loop over h becomes one
// store at a variable index, and that a copy of all of st for every subtree.)
template <int h, typename T>
__device__ __forceinline__ void std_join(T (&st)[kStdHeights], T s, int j)
{
#pragma clang fp contract(off)
    if constexpr (h == kStdHeights - 1) {
        st[h] = s;
    } else {
        if ((j >> h) & 1)  // (j is the same on every lane)
            std_join<h + 1>(st, st[h] + s, j);
        else
            st[h] = s;
    }
}

template <typename T>
__global__ __launch_bounds__(kStdThreads, 8) void red_std_small(RedStdArgs a)
{
#pragma clang fp contract(off)
    const T *__restrict__ t = reinterpret_cast<const T *>(a.t);
    const T *__restrict__ v = reinterpret_cast<const T *>(a.v);
    const T *__restrict__ rt = reinterpret_cast<const T *>(a.rt);
    const T *__restrict__ rv = reinterpret_cast<const T *>(a.rv);
    T *__restrict__ q = reinterpret_cast<T *>(a.q);
    __shared__ StdRecord<T> rec[kStdWindow];
    __shared__ T times[kChunkRows + 1];  // inf past the group's rows
    __shared__ int32_t owner[kChunkRows];  // the row's PCF, -1: none
    __shared__ int32_t first[kStdBlocks][kStdSmall];  // counts, then the first record
    __shared__ int64_t row0[kStdSmall];
    __shared__ int32_t wbase[kStdSmall + 1];
    __shared__ int32_t bad;
    const int tid = threadIdx.x, lane = tid & 63;
    const T inf = __builtin_inf();
    for (int64_t c = blockIdx.x; c < a.nchunks; c += gridDim.x) {
        const int64_t b = a.chunk_grp[c];
        const int64_t gb = a.groups[b];
        const int m = (int)(a.groups[b + 1] - gb);
        if (m > kStdSmall)
            continue;  // red_std_terms' rows (block-uniform)
        const int64_t c0 = a.chunk_row[c], g1 = a.offsets[gb + m];
        const int64_t c1 = c0 + kChunkRows < g1 ? c0 + kChunkRows : g1;
        const int rows = (int)(c1 - c0);
        // window offsets: an inclusive scan of the record counts in wave 0
        if (tid < 64) {
            int64_t len = 0;
            if (tid < m) {
                const int64_t o = a.offsets[gb + tid], n = a.offsets[gb + tid + 1] - o;
                const int64_t k0 = a.chunk_first[kStdSmall * c + tid];
                const int64_t k1 =
                    c1 < g1 ? a.chunk_first[kStdSmall * (c + 1) + tid] : n - 1;
                row0[tid] = o + k0;
                len = k1 - k0 + 1;
            }
            int32_t s = len < 1 || len > kStdWindow ? kStdWindow + 1 : (int32_t)len;
            for (int h = 1; h < 64; h <<= 1) {
                const int32_t o = __shfl_up(s, h, 64);
                if (tid >= h)
                    s += o;
            }
            wbase[tid + 1] = s;
            // a window over the bound only comes from times that do not
            // increase (PCF rules broken): the chunk's sums become NaN
            const uint64_t over = __ballot(tid < m && s > kStdWindow);
            if (tid == 0) {
                wbase[0] = 0;
                bad = over != 0;
            }
        }
        T mean[kStdRows];  // of the thread's rows tid + u kStdThreads
#pragma unroll
        for (int u = 0; u < kStdRows; ++u) {
            const int r = tid + u * kStdThreads;
            times[r] = r < rows ? rt[c0 + r] : inf;
            mean[u] = r < rows ? rv[c0 + r] : T(0);
            owner[r] = -1;
        }
        if (tid == 0)
            times[kChunkRows] = c1 < g1 ? rt[c1] : inf;
        for (int r = tid; r < kStdBlocks * (int)kStdSmall; r += kStdThreads)
            (&first[0][0])[r] = 0;
        __syncthreads();
        const int32_t L = wbase[m];
        const bool ok = bad == 0;
        int32_t pcf[kStdLoads];
        if (ok) {
#pragma unroll
            for (int u = 0; u < kStdLoads; ++u) {
                const int32_t e = tid + u * kStdThreads;
                int32_t lo = 0;  // the PCF whose window holds record e
#pragma unroll
                for (int32_t h = (int32_t)kStdSmall / 2; h > 0; h >>= 1)
                    lo += lo + h < m && wbase[lo + h] <= e ? h : 0;
                pcf[u] = lo;
                if (e < L) {
                    const int64_t r = row0[lo] + (e - wbase[lo]);
                    rec[e].t = t[r];
                    rec[e].v = v[r];
                }
            }
            // the records' rows (the first of a PCF's window lies at or
            // before the chunk's first time, some of the last past its end)
            const auto place = [&](auto from, auto to) {
                int32_t at[kStdLoads];  // rows with times below x
                T x[kStdLoads];
#pragma unroll
                for (int u = from; u < to; ++u) {
                    const int32_t e = tid + u * kStdThreads;
                    x[u] = rec[e < kStdWindow ? e : 0].t;
                    at[u] = 0;
                }
#pragma unroll
                for (int32_t h = kChunkRows / 2; h > 0; h >>= 1)
#pragma unroll
                    for (int u = from; u < to; ++u)
                        at[u] += times[at[u] + h - 1] < x[u] ? h : 0;
#pragma unroll
                for (int u = from; u < to; ++u) {
                    const int32_t e = tid + u * kStdThreads;
                    if (e < L && e > wbase[pcf[u]]) {
                        // (PCF i looks at the run's row i first: its own where all
                        // PCFs share the time. All from the first row on, 200
                        // groups of 64 PCFs on one grid of 275 times, whole
                        // calls: 707 us, so 438, 434 where no times are shared)
                        int32_t k = at[u] + pcf[u];
                        if (k >= rows || times[k] != x[u] || atomicCAS(&owner[k], -1, pcf[u]) != -1)
                            for (k = at[u]; k < rows && times[k] == x[u]; ++k)
                                if (atomicCAS(&owner[k], -1, pcf[u]) == -1)
                                    break;
                        if (k < rows && times[k] == x[u])
                            atomicAdd(&first[k >> 6][pcf[u]], 1);
                    }
                }
            };
            using std::integral_constant;
            place(integral_constant<int, 0>(), integral_constant<int, kStdRows>());
            if (kStdRows * kStdThreads + __builtin_amdgcn_readfirstlane(tid) < L)
                place(integral_constant<int, kStdRows>(), integral_constant<int, kStdLoads>());
        }
        __syncthreads();
        if (tid < m) {
            int32_t at = wbase[tid];
#pragma unroll
            for (int k = 0; k < kStdBlocks; ++k) {
                const int32_t n = first[k][tid];
                first[k][tid] = at;
                at += n;
            }
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kStdRows; ++w) {
            const int blk = __builtin_amdgcn_readfirstlane(tid >> 6) + w * (kStdThreads / 64);
            if (blk * 64 >= rows)
                break;
            const int r = blk * 64 + lane;
            const bool live = r < rows;
            const T x = times[r];
            const T mu = mean[w] / (T)m;
            const int32_t own = owner[r];
            const uint64_t same = __ballot(live && times[r + 1] == x);
            const int last = rows - blk * 64 < 64 ? rows - blk * 64 - 1 : 63;
            const bool tied = (same >> last) & 1;
            // rows up to the end of this row's run of equal times
            const int end = lane + __builtin_ctzll(~(same >> lane));
            const uint64_t upto = end >= 63 ? ~0ull : (2ull << end) - 1;
            const uint32_t ulo = (uint32_t)upto, uhi = (uint32_t)(upto >> 32);
            T st[kStdHeights], acc = T(0);
#pragma unroll
            for (int h = 0; h < kStdHeights; ++h)
                st[h] = T(0);
            bool have = false;  // acc holds the group's last m % kStdBatch terms
            for (int i0 = 0; ok && i0 < m; i0 += kStdBatch) {
                T d[kStdBatch];
                if (tied) {
#pragma unroll 1
                    for (int u = 0; u < kStdBatch; ++u) {
                        const int i = i0 + u < m ? i0 + u : m - 1;
                        int32_t lo = wbase[i], hi = wbase[i + 1] - 1;
                        while (lo < hi) {  // rec[lo].t <= x
                            const int32_t mid = (lo + hi + 1) >> 1;
                            if (rec[mid].t <= x)
                                lo = mid;
                            else
                                hi = mid - 1;
                        }
                        const T f = rec[lo].v;
#pragma unroll
                        for (int j = 0; j < kStdBatch; ++j)
                            d[j] = j == u ? f : d[j];
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < kStdBatch; ++u) {
                        // (past the group: the last PCF again, not used)
                        const int i = i0 + u < m ? i0 + u : m - 1;
                        const uint64_t mine = __builtin_amdgcn_ballot_w64(own == i);
                        d[u] = rec[first[blk][i] + __popc((uint32_t)mine & ulo) +
                                   __popc((uint32_t)(mine >> 32) & uhi)].v;
                    }
                }
#pragma unroll
                for (int u = 0; u < kStdBatch; ++u) {
                    d[u] -= mu;
                    d[u] *= d[u];
                }
                const T pair = d[0] + d[1];
                const int left = m - i0;
                if (left >= kStdBatch) {
                    std_join<0>(st, pair + (d[2] + d[3]), i0 / kStdBatch);
                } else {
                    have = true;
                    acc = left == 1 ? d[0] : left == 2 ? pair : pair + d[2];
                }
            }
            // fold the subtrees from the smallest up and store
#pragma unroll
            for (int h = 0; h < kStdHeights; ++h) {
                if ((m / kStdBatch >> h) & 1) {
                    acc = have ? st[h] + acc : st[h];
                    have = true;
                }
            }
            if (live)
                q[c0 + r] = ok ? acc : __builtin_nan("");
        }
        __syncthreads();  // the records and tables are rewritten next
    }
}

// Root rows kept by ReducePair's rule (all rows of a one-PCF group), and
// their values after the group's transformation. One wave per chunk of at
// most kChunkRows rows of one group.
template <typename T>
__device__ __forceinline__ T red_finish(int op, T x, int64_t m)
{
    if (op == RO_MEAN)
        return x / (T)m;
    if (op == RO_STD)
        return sqrt(x / (T)(m - 1));
    return x;
}

template <typename T>
__global__ void red_emit(RedEmitArgs a)
{
    const T *__restrict__ rt = reinterpret_cast<const T *>(a.rt);
    const T *__restrict__ rv = reinterpret_cast<const T *>(a.rv);
    T *__restrict__ t_out = reinterpret_cast<T *>(a.t_out);
    T *__restrict__ v_out = reinterpret_cast<T *>(a.v_out);
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t c = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; c < a.nchunks;
         c += nwaves) {
        const int64_t b = a.chunk_grp[c];
        const int64_t gb = a.groups[b], m = a.groups[b + 1] - gb;
        const int64_t g0 = a.offsets[gb], g1 = a.offsets[gb + m];
        const int64_t c0 = a.chunk_row[c];
        const int64_t c1 = c0 + kChunkRows < g1 ? c0 + kChunkRows : g1;
        int64_t w = a.fill ? a.chunk_off[c] : 0;
        const int64_t end = a.fill ? *a.out_end : 0;
        for (int64_t base = c0; base < c1; base += 64) {
            const int64_t k = base + lane;
            const bool keep = k < c1 && (m == 1 || k == g0 ||
                                         (rt[k] != rt[k - 1] && rv[k] != rv[k - 1]));
            const uint64_t mask = __ballot(keep);
            const int64_t pos = w + __popcll(mask & below);
            if (a.fill && keep && pos < end) {
                t_out[pos] = rt[k];
                v_out[pos] = red_finish<T>(a.op, rv[k], m);
            }
            w += __popcll(mask);
        }
        if (!a.fill && lane == 0)
            a.chunk_cnt[c] = w;
    }
}

// Chunk counts to the chunks' output rows and the groups' offsets (one
// workgroup; the counts stay on the device, so the host reads the offsets
// alone and writes nothing back).
__global__ __launch_bounds__(1024) void red_scan(RedScanArgs a)
{
    __shared__ int64_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t before = 0;
    if (tid == 0)
        a.offsets_out[0] = 0;
    for (int64_t c0 = 0; c0 < a.nchunks; c0 += 1024) {
        const int64_t c = c0 + tid;
        const int64_t n = c < a.nchunks ? a.chunk_cnt[c] : 0;
        int64_t inc = n;
#pragma unroll
        for (int h = 1; h < 64; h <<= 1) {
            const int64_t o = __shfl_up(inc, h, 64);
            if (lane >= h)
                inc += o;
        }
        if (lane == 63)
            wsum[wave] = inc;
        __syncthreads();
        int64_t base = before, all = before;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            base += w < wave ? wsum[w] : 0;
            all += wsum[w];
        }
        if (c < a.nchunks) {
            a.chunk_off[c] = base + inc - n;
            // a group's last chunk ends its rows
            if (c + 1 == a.nchunks || a.chunk_grp[c + 1] != a.chunk_grp[c])
                a.offsets_out[a.chunk_grp[c] + 1] = base + inc;
        }
        before = all;
        __syncthreads();  // (wsum is rewritten next)
    }
}

hipError_t launch_red_scan(const RedScanArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(red_scan, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
}

static int64_t grid_for(int64_t units, int64_t per_block, int64_t cap)
{
    int64_t g = (units + per_block - 1) / per_block;
    return g < 1 ? 1 : (g > cap ? cap : g);
}

hipError_t launch_red_rowmap(const int64_t *offsets, int64_t n, int32_t *row_pcf, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(red_rowmap, dim3((unsigned)grid_for(n, 4, 8192)), dim3(256), 0, s,
                       offsets, n, row_pcf);
    return hipGetLastError();
}

template <typename T>
static void launch_red_level_t(int op, const RedLevelArgs &a, dim3 g, dim3 blk, hipStream_t s)
{
    switch (op) {
    case RO_MAX: hipLaunchKernelGGL((red_level<T, RO_MAX>), g, blk, 0, s, a); break;
    case RO_MIN: hipLaunchKernelGGL((red_level<T, RO_MIN>), g, blk, 0, s, a); break;
    case RO_SUB: hipLaunchKernelGGL((red_level<T, RO_SUB>), g, blk, 0, s, a); break;
    case RO_MUL: hipLaunchKernelGGL((red_level<T, RO_MUL>), g, blk, 0, s, a); break;
    case RO_SQDIFF: hipLaunchKernelGGL((red_level<T, RO_SQDIFF>), g, blk, 0, s, a); break;
    default: hipLaunchKernelGGL((red_level<T, RO_SUM>), g, blk, 0, s, a); break;  // sum, mean, std
    }
}

hipError_t launch_red_level(bool f64, int op, const RedLevelArgs &a, int64_t rows,
                            hipStream_t s)
{
    if (rows <= 0)
        return hipSuccess;
    const dim3 g((unsigned)grid_for((rows + kMergeK - 1) / kMergeK, 64 * kLevelWaves,
                                    16384 * 4 / kLevelWaves)),
        blk(64 * kLevelWaves);
    static_assert(kMergeK >= 1 && kMergeK <= 32, "positions per lane");
    if (f64)
        launch_red_level_t<double>(op, a, g, blk, s);
    else
        launch_red_level_t<float>(op, a, g, blk, s);
    return hipGetLastError();
}

template <typename T>
static void launch_red_fuse_t(int op, const RedFuseArgs &a, dim3 gs, dim3 gf, hipStream_t s)
{
    hipLaunchKernelGGL(red_split<T>, gs, dim3(256), 0, s, a);
    const dim3 blk(kFuseThreads);
    switch (op) {
    case RO_MAX: hipLaunchKernelGGL((red_fuse<T, RO_MAX>), gf, blk, 0, s, a); break;
    case RO_MIN: hipLaunchKernelGGL((red_fuse<T, RO_MIN>), gf, blk, 0, s, a); break;
    default: hipLaunchKernelGGL((red_fuse<T, RO_SUM>), gf, blk, 0, s, a); break;  // sum, mean, std
    }
}

hipError_t launch_red_fuse(bool f64, int op, const RedFuseArgs &a, hipStream_t s)
{
    if (a.ntiles <= 0)
        return hipSuccess;
    const dim3 gs((unsigned)grid_for(a.nsamples, 256 / kFuseLists * kSplitBatch, 65536)),
        gf((unsigned)grid_for(a.ntiles, 1, 65536));
    if (f64)
        launch_red_fuse_t<double>(op, a, gs, gf, s);
    else
        launch_red_fuse_t<float>(op, a, gs, gf, s);
    return hipGetLastError();
}

// The rows of X's PCF i and then Y's PCF i at Z's PCFs 2i and 2i+1: one
// wave per i.
template <typename T>
__global__ void red_interleave(int64_t n, const int64_t *__restrict__ xo,
                               const T *__restrict__ xt, const T *__restrict__ xv,
                               const int64_t *__restrict__ yo, const T *__restrict__ yt,
                               const T *__restrict__ yv, const int64_t *__restrict__ zo,
                               T *__restrict__ zt, T *__restrict__ zv)
{
    const int lane = threadIdx.x & 63;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; i < n;
         i += nwaves) {
        const int64_t x0 = xo[i], nx = xo[i + 1] - x0, y0 = yo[i], ny = yo[i + 1] - y0;
        const int64_t z0 = zo[2 * i], z1 = zo[2 * i + 1];
        for (int64_t k = lane; k < nx; k += 64) {
            zt[z0 + k] = xt[x0 + k];
            zv[z0 + k] = xv[x0 + k];
        }
        for (int64_t k = lane; k < ny; k += 64) {
            zt[z1 + k] = yt[y0 + k];
            zv[z1 + k] = yv[y0 + k];
        }
    }
}

hipError_t launch_red_interleave(bool f64, int64_t n, const int64_t *xo, const void *xt,
                                 const void *xv, const int64_t *yo, const void *yt,
                                 const void *yv, const int64_t *zo, void *zt, void *zv,
                                 hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    const dim3 g((unsigned)grid_for(n, 4, 8192)), blk(256);
    if (f64)
        hipLaunchKernelGGL(red_interleave<double>, g, blk, 0, s, n, xo, (const double *)xt,
                           (const double *)xv, yo, (const double *)yt, (const double *)yv, zo,
                           (double *)zt, (double *)zv);
    else
        hipLaunchKernelGGL(red_interleave<float>, g, blk, 0, s, n, xo, (const float *)xt,
                           (const float *)xv, yo, (const float *)yt, (const float *)yv, zo,
                           (float *)zt, (float *)zv);
    return hipGetLastError();
}

hipError_t launch_red_std(bool f64, const RedStdArgs &a, hipStream_t s)
{
    if (a.rows <= 0)
        return hipSuccess;
    const dim3 g((unsigned)grid_for(a.rows, 256, 8192)), blk(256);
    if (f64)
        hipLaunchKernelGGL(red_std_terms<double>, g, blk, 0, s, a);
    else
        hipLaunchKernelGGL(red_std_terms<float>, g, blk, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_red_std_small(bool f64, const RedStdArgs &a, hipStream_t s)
{
    if (a.nchunks <= 0)
        return hipSuccess;
    const dim3 gb((unsigned)grid_for(a.nchunks * kStdSmall, 256, 16384)), bb(256);
    const dim3 g((unsigned)grid_for(a.nchunks, 1, 16384)), blk(kStdThreads);
    if (f64) {
        hipLaunchKernelGGL(red_std_bounds<double>, gb, bb, 0, s, a);
        hipLaunchKernelGGL(red_std_small<double>, g, blk, 0, s, a);
    } else {
        hipLaunchKernelGGL(red_std_bounds<float>, gb, bb, 0, s, a);
        hipLaunchKernelGGL(red_std_small<float>, g, blk, 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_red_emit(bool f64, const RedEmitArgs &a, hipStream_t s)
{
    if (a.nchunks <= 0)
        return hipSuccess;
    const dim3 g((unsigned)grid_for(a.nchunks, 4, 8192)), blk(256);
    if (f64)
        hipLaunchKernelGGL(red_emit<double>, g, blk, 0, s, a);
    else
        hipLaunchKernelGGL(red_emit<float>, g, blk, 0, s, a);
    return hipGetLastError();
}

}  // namespace pcf
