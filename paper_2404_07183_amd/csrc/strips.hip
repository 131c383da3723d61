// strips.hip -- the forward kernel for sets whose PCFs fit LDS several at a
// time: row blocks held in LDS, columns streamed through it, no workgroup
// barrier between the two.
//
// Method. The merge, its records and its step are those of kernels.hip. A job
// is a row block (R consecutive PCFs, their records staged once) against a
// run of columns; its columns are cut into groups of one or a few consecutive
// PCFs. Every wave takes groups from the job's counter on its own: it copies
// the group's records into its part of a ring in LDS, splits the R x M pairs'
// total step count over its 64 lanes (merge-path starts, contiguous runs),
// merges, adds each pair's partial sums in lane order and stores the results.
//
// Why. With the whole workgroup on one tile (kernels.hip) all waves of a SIMD
// sit in the same phase and meet at four barriers a tile: the work around the
// merge (prefix sums, merge-path searches, staging, sums of partial results)
// is short, dependent and full of latency, 41 % of an FP64 tile. Here a
// SIMD's waves drift apart and one wave's latency is covered by the others'
// merges. What bounds it (20,000 PCFs of 50 to 500 rows, L1 FP64, counters):
// LDS 87 % of the time, 59 % of that in bank conflicts of the records' random
// 16-byte reads (16 lanes on 16 slots collide three deep on average), VALU
// 78 % (tile kernel 70 %). Kernel times, tile kernel / this one: that matrix
// 63.4 / 57.3 ms; FP64 PCFs of 400 rows on average, 5,120 of them,
// 9.09 / 6.40 ms; of 25 rows, 20,480, 12.4 / 6.4 ms (a tile's 32 x 32 PCFs
// leave most of LDS empty there); FP32, 100 to 1000 rows, a window of 1,500 x
// 12,000, 5.33 / 4.78 ms. Sixteen waves a workgroup against twelve: 5 to 20 %
// faster although the ring takes more of LDS.
//
// A row block fills what the ring leaves of LDS (12 rows of that matrix); a
// job's row records and a wave's next group are loaded into registers while
// the previous work merges (4 to 8 % for launches of a millisecond or less).
//
// The ring. Group g's place is fixed by the plan: its records occupy virtual
// positions [virt(g), virt(g) + len) of an endless record stream (positions
// skipped so that no group crosses the ring's end), at virt(g) modulo the
// ring size. A wave may write its group once every unfinished earlier group
// starts at or after virt(g) + len - ring (busy[], one entry a wave, always
// at or below the start of the wave's current group). The wave holding the
// earliest group never waits (a group is at most the ring), so some wave
// always advances and every wait ends.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <utility>

#include "common.hpp"
#include "launch.hpp"
#include "tile.hpp"

namespace pcf {

namespace {

// A decoded job (LDS).
struct StripJobDesc {
    int64_t r_lo, rrec0;             // first row PCF, its first record
    int64_t obase, ldo, row0, col0;  // output mapping of the segment
    int32_t R, rrecs;                // rows, their records
    int32_t g0, g1;                  // column groups
    int32_t sym, mirror, swap;       // see Segment
    int32_t rmag;                    // floor(2^16 / R) + 1 (see div_rows)
    int32_t valid;
};

struct StripShared {
    StripJobDesc job[2];
    int32_t rn[kStripMaxRows];  // rows of each row PCF
    int32_t rb[kStripMaxRows];      // its first record in the row area
    uint32_t busy[kStripMaxWaves];
    int32_t next;                   // next group of the job
};
static_assert(sizeof(StripShared) <= kStripSharedBytes, "strip_lds");

// k / R for 0 <= k < kStripMaxPairs and 1 <= R <= 64 by a multiply: with
// m = floor(2^16 / R) + 1 the product exceeds k / R by less than k / 2^16 <
// 1/64 <= 1/R, which cannot carry it past the next integer.
static_assert(kStripMaxRows <= 64 && kStripMaxPairs <= 1024, "div_rows range");
__device__ __forceinline__ int32_t div_rows(int32_t k, int32_t rmag)
{
    return (int32_t)(((uint32_t)k * (uint32_t)rmag) >> 16);
}

// Orders this wave's LDS accesses for the compiler (the hardware runs one
// wave's LDS operations in order).
__device__ __forceinline__ void wave_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-wide inclusive scans by DPP row shifts and row broadcasts (lanes
// without a source take 0, the identity of both for non-negative values).
template <bool Max> __device__ __forceinline__ int32_t wave_scan(int32_t v)
{
    int32_t u;
#define PCF_SCAN_STEP(ctrl, rows)                                        \
    u = __builtin_amdgcn_update_dpp(0, v, ctrl, rows, 0xf, false);       \
    v = Max ? (u > v ? u : v) : v + u;
    PCF_SCAN_STEP(0x111, 0xf)  // row_shr:1
    PCF_SCAN_STEP(0x112, 0xf)  // row_shr:2
    PCF_SCAN_STEP(0x114, 0xf)  // row_shr:4
    PCF_SCAN_STEP(0x118, 0xf)  // row_shr:8
    PCF_SCAN_STEP(0x142, 0xa)  // row_bcast:15
    PCF_SCAN_STEP(0x143, 0xc)  // row_bcast:31
#undef PCF_SCAN_STEP
    return v;
}

__device__ __forceinline__ int32_t padded_steps(int32_t na, int32_t nb)
{
    return (na + nb - 2 + kStepBlock - 1) & ~(kStepBlock - 1);
}

// The workgroup's next job (one lane; next, end: its current run of jobs,
// ticket: the run after that, or -1 when it is still to be taken).
__device__ __forceinline__ void next_job(StripJobDesc &d, int32_t &next, int32_t &end,
                                         int32_t ticket, const unsigned char *ws)
{
    const WsHeader &h = hdr_of(ws);
    if (next == end) {
        // (the first run of a workgroup is its own; the queue starts after them)
        if (ticket < 0)
            ticket = (int32_t)(gridDim.x +
                               atomicAdd(const_cast<uint32_t *>(&h.counter[0]), 1u));
        if (ticket >= h.ntiles) {
            d.valid = 0;
            return;
        }
        const int32_t *runs = reinterpret_cast<const int32_t *>(ws + h.off_runs);
        next = runs[ticket];
        end = runs[ticket + 1];
    }
    const StripJob j = reinterpret_cast<const StripJob *>(ws + h.off_jobs)[next++];
    const Segment &s = reinterpret_cast<const Segment *>(ws + h.off_segs)[j.seg];
    const StripBlock b = reinterpret_cast<const StripBlock *>(ws + h.off_sblocks)[j.block];
    d.r_lo = b.lo;
    d.R = b.rows;
    d.rmag = (1 << 16) / b.rows + 1;
    d.rrec0 = b.rec0;
    d.rrecs = b.recs;
    d.g0 = j.g0;
    d.g1 = j.g1;
    d.obase = s.obase;
    d.ldo = s.ldo;
    d.row0 = s.row0;
    d.col0 = s.col0;
    d.sym = s.type == kSegTriangle ? 1 : 0;
    d.mirror = s.mirror;
    d.swap = s.swap;
    asm volatile("" ::: "memory");  // (valid last: see load_job's caller)
    d.valid = 1;
}

// Copies n records to LDS with `stride` threads, four loads in flight each.
template <typename T>
__device__ __forceinline__ void copy_records(Rec<T> *dst, const Rec<T> *src, int32_t n,
                                             int32_t at, int32_t stride)
{
    typedef typename RecVec<T>::type V;
    const V *s = reinterpret_cast<const V *>(src);
    V *d = reinterpret_cast<V *>(dst);
    for (int32_t q = at; q < n; q += 4 * stride) {
        V r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t k = q + u * stride;
            r[u] = s[k < n ? k : q];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t k = q + u * stride;
            if (k < n)
                d[k] = r[u];
        }
    }
}

// A wave's records of a group: the first 64 A loaded ahead into
// registers (while it merges the group before), the rest directly.
template <typename T, int A>
__device__ __forceinline__ void load_ahead(typename RecVec<T>::type *r, const Rec<T> *src,
                                           int32_t n, int32_t lane)
{
    typedef typename RecVec<T>::type V;
    const V *s = reinterpret_cast<const V *>(src);
#pragma unroll
    for (int u = 0; u < A; ++u) {
        const int32_t k = lane + u * 64;
        r[u] = s[k < n ? k : 0];
    }
}

template <typename T, int A>
__device__ __forceinline__ void store_ahead(Rec<T> *dst, const typename RecVec<T>::type *r,
                                            int32_t n, int32_t lane)
{
    typedef typename RecVec<T>::type V;
    V *d = reinterpret_cast<V *>(dst);
#pragma unroll
    for (int u = 0; u < A; ++u) {
        const int32_t k = lane + u * 64;
        if (k < n)
            d[k] = r[u];
    }
}

// A pair's entry in the wave's table: the LDS address of the row PCF's first
// record, that plus the column's (LdsWalk's q and S), and the pair's steps.
struct alignas(16) StripPair {
    uint32_t q, S;
    int32_t steps;
    int32_t excl;  // steps of the item's pairs before it
};

// A lane's merge state (kernels.hip, Chain): P the piece loaded last, Q the
// other one.
template <typename T> struct StripChain {
    typedef typename RecVec<T>::type V;
    typedef const __attribute__((address_space(3))) V *ptr;
    V P;
    T tQ, vQ;
    LdsWalk<T> w;
    T x;
    double acc;
    int32_t left;  // steps left in the pair

    // both pieces from the walk's addresses
    __device__ __forceinline__ void load()
    {
        P = *(ptr)(size_t)w.q;
        const V Q = *(ptr)(size_t)(w.S - w.q);
        tQ = Q.x;
        vQ = Q.y;
    }
};

template <int K, typename T, int HK, int E>
__device__ __forceinline__ void strip_step(StripChain<T> &ch, T &part, T p)
{
    const T tP = ch.P.x, tQ = ch.tQ;
    const T y = min_raw(tP, tQ);
    part = fma(hval<T, HK, E>(ch.P.y, ch.vQ, p), y - ch.x, part);
    ch.x = y;
    const bool c = tP <= tQ;
    ch.vQ = c ? ch.vQ : ch.P.y;
    ch.tQ = max_raw(tP, tQ);
    ch.P = ch.w.template advance<K>(c);
}

template <typename T, int HK, int... Ks>
__device__ __forceinline__ void strip_block(StripChain<T> &ch, T &part, T p,
                                            std::integer_sequence<int, Ks...>)
{
    with_exponent<HK>(p, [&](auto e) { (strip_step<Ks, T, HK, e()>(ch, part, p), ...); });
    ch.w.end_block();
}

// Merge-path start of a pair at step d: the walk and the start x of the cell
// (merge_path and pair_start of tile.hpp on LDS addresses; na, nb rows).
template <typename T>
__device__ __forceinline__ void strip_start(LdsWalk<T> &w, T &x, const StripPair &e, int32_t na,
                                            int32_t nb, int32_t d)
{
    typedef const __attribute__((address_space(3))) T *time_ptr;
    constexpr uint32_t kRec = sizeof(Rec<T>);
    const uint32_t qa = e.q, qb = e.S - e.q;
    w.q = qa;
    w.S = e.S;
    x = T(0);
    if (d > 0) {
        int32_t lo = d - (nb - 1);
        lo = lo < 0 ? 0 : lo;
        int32_t hi = d < (na - 1) ? d : (na - 1);
        const uint32_t qd = qb + (uint32_t)(d - 1) * kRec;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            const T ta = *(time_ptr)(size_t)(qa + (uint32_t)mid * kRec);
            const T tb = *(time_ptr)(size_t)(qd - (uint32_t)mid * kRec);
            if (ta <= tb)
                lo = mid + 1;
            else
                hi = mid;
        }
        const int32_t j = d - lo;
        w.q = qa + (uint32_t)lo * kRec;
        const uint32_t wb = qb + (uint32_t)j * kRec;
        w.S = w.q + wb;
        const T xa = lo > 0 ? *(time_ptr)(size_t)(w.q - kRec) : T(0);
        const T xb = j > 0 ? *(time_ptr)(size_t)(wb - kRec) : T(0);
        x = xa > xb ? xa : xb;
    }
}

}  // namespace

template <typename T, int HK, int RT>
__global__ __launch_bounds__(kThreads) void pairwise_strips(FwdArgs args)
{
    extern __shared__ __align__(16) unsigned char smem[];
    StripShared &sh = *reinterpret_cast<StripShared *>(smem);
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = nthr >> 6;
    const unsigned char *ws = args.ws;
    const WsHeader &h = hdr_of(ws);
    const int32_t pair_cap = h.strip_pairs, col_cap = h.strip_cols;
    const int32_t row_recs = h.strip_row_recs, ring = h.strip_ring_recs;
    // this wave's partial-sum slots (pair + lane) and column metadata
    unsigned char *mine = smem + kStripSharedBytes + wave * strip_wave_bytes(pair_cap, col_cap);
    double *part = reinterpret_cast<double *>(mine);
    int32_t *head = reinterpret_cast<int32_t *>(mine);  // before the merge
    StripPair *pairs = reinterpret_cast<StripPair *>(mine + (pair_cap + 64 + 1) / 2 * 16);
    int32_t *cn = reinterpret_cast<int32_t *>(pairs + pair_cap);
    int32_t *cb = cn + col_cap;
    // one array of records: the row area, then the ring
    Rec<T> *lrec = reinterpret_cast<Rec<T> *>(
        smem + kStripSharedBytes + waves * strip_wave_bytes(pair_cap, col_cap));
    const Rec<T> *grec = reinterpret_cast<const Rec<T> *>(ws + h.off_rec);
    const StripGroup *groups = reinterpret_cast<const StripGroup *>(ws + h.off_groups);
    const int64_t *offsets = args.offsets;
    int32_t run_next = 0, run_end = 0;  // (the lane that takes the jobs)
    const T p = (T)args.p;
    T *out = reinterpret_cast<T *>(args.out);
    // (volatile LDS accesses; a generic pointer would make them flat ones)
    typedef volatile __attribute__((address_space(3))) uint32_t *lds_u32;
    const lds_u32 busy = (lds_u32)(size_t)lds_address(sh.busy);

    typedef typename RecVec<T>::type V;
    // What a wave loads ahead of a job: its threads' share of the row records,
    // and its first group (wave w starts with group g0 + w) with its records.
    // (the general powers' kernels have no registers to spare for it)
    constexpr int kRA = HK <= kProd ? kStripRowAhead : 0, kGA = HK <= kProd ? kStripAhead : 0;
    V rows[kRA > 0 ? kRA : 1], ahead[kGA > 0 ? kGA : 1];
    StripGroup gr;
    auto load_job = [&](const StripJobDesc &d) {
        const V *s = reinterpret_cast<const V *>(grec) + d.rrec0;
        const int32_t n = d.rrecs;
#pragma unroll
        for (int u = 0; u < kRA; ++u) {
            const int32_t k = tid + u * nthr;
            rows[u] = s[k < n ? k : 0];
        }
        const int32_t g = d.g0 + wave;
        gr = groups[g < d.g1 ? g : d.g1];
        load_ahead<T, kGA>(ahead, grec + gr.rec0, gr.size & ((1 << kStripColShift) - 1), lane);
    };
    typedef volatile __attribute__((address_space(3))) int32_t *lds_i32;
    if (tid == nthr - 64)
        next_job(sh.job[0], run_next, run_end, (int32_t)blockIdx.x, ws);
    sync_lds();
    if (sh.job[0].valid)
        load_job(sh.job[0]);
    for (int cur = 0; sh.job[cur].valid; cur ^= 1) {
        const StripJobDesc &J = sh.job[cur];
        const int32_t R = J.R, g1 = J.g1;
        {
            V *d = reinterpret_cast<V *>(lrec);
            const int32_t n = J.rrecs;
#pragma unroll
            for (int u = 0; u < kRA; ++u) {
                const int32_t k = tid + u * nthr;
                if (k < n)
                    d[k] = rows[u];
            }
            if (n > kRA * nthr)
                copy_records<T>(lrec, grec + J.rrec0, n, tid + kRA * nthr, nthr);
        }
        if (tid < R) {
            const int64_t o = offsets[J.r_lo + tid], e = offsets[J.r_lo + tid + 1];
            sh.rn[tid] = (int32_t)(e - o);
            sh.rb[tid] = (int32_t)(o + (J.r_lo + tid) * kPad - J.rrec0);
        }
        if (tid < kStripMaxWaves)
            busy[tid] = groups[J.g0].virt;
        if (tid == 0)
            sh.next = J.g0 + waves;
        if (tid == nthr - 64)
            *(lds_i32)(size_t)lds_address(&sh.job[cur ^ 1].valid) = -1;  // not known yet
        sync_lds();
        if (tid == nthr - 64)  // the next job, while the others start on this one
            next_job(sh.job[cur ^ 1], run_next, run_end, -1, ws);

        // this lane's pair of an item's first 64 (pair k: row k % R of column
        // k / R), as far as the job fixes it
        const int32_t j0 = div_rows(lane, J.rmag), r0 = lane - j0 * R;
        const int32_t rn0 = sh.rn[r0];
        const uint32_t qa0 = lds_address(lrec + sh.rb[r0]);
        const int64_t row_at = J.obase + (J.r_lo + r0 - J.row0) * J.ldo - J.col0;
        const int64_t col_at = J.obase + (J.r_lo + r0) - J.col0;
        const int32_t gram = args.gram;

        // the wave's next group (its table entry loaded an item ahead)
        auto take = [&]() {
            int32_t g = 0;
            if (lane == 0)
                g = atomicAdd(&sh.next, 1);
            return __builtin_amdgcn_readfirstlane(g);
        };
        int32_t g = J.g0 + wave;
        while (g < g1) {
            const int64_t c0 = gr.start;
            const int32_t M = __builtin_amdgcn_readfirstlane(gr.size >> kStripColShift);
            const int32_t len = gr.size & ((1 << kStripColShift) - 1);
            const int32_t at = row_recs + (int32_t)(gr.virt % (uint32_t)ring);
            int64_t oc = 0;
            if (M > 1)  // (a single column's rows follow from its records)
                oc = offsets[c0 + (lane < M ? lane : M)];
            if (lane == 0)
                busy[wave] = gr.virt;
            const uint32_t lowest = gr.virt + (uint32_t)len - (uint32_t)ring;
            for (;;) {
                const uint32_t b = busy[lane < waves ? lane : 0];
                if (__builtin_amdgcn_ballot_w64((int32_t)(b - lowest) < 0) == 0)
                    break;
                __builtin_amdgcn_s_sleep(2);
            }
            wave_lds();
            store_ahead<T, kGA>(lrec + at, ahead, len, lane);
            if (len > 64 * kGA)
                copy_records<T>(lrec + at, grec + gr.rec0, len, lane + 64 * kGA, 64);
            if (M > 1) {
                const int32_t rel =
                    (int32_t)(oc - __shfl(oc, 0, 64)) + (lane < M ? lane : M) * kPad;
                const int32_t nxt = __shfl_down(rel, 1, 64);
                if (lane < M) {
                    cn[lane] = nxt - rel - kPad;
                    cb[lane] = at + rel;
                }
            }
            head[lane] = 0;
            const int32_t gnext = take();
            const StripGroup grn = groups[gnext < g1 ? gnext : g1];
            wave_lds();
            load_ahead<T, kGA>(ahead, grec + grn.rec0, grn.size & ((1 << kStripColShift) - 1), lane);

            // pair (r, j) is live when r < diag + j (below the diagonal of a
            // block of a symmetric part), or r == diag + j for `gram`
            const int32_t diag =
                J.sym && c0 < J.r_lo + R ? (int32_t)(c0 - J.r_lo) : (int32_t)1 << 20;
            const int32_t P = R * M;
            const uint32_t qat = lds_address(lrec + at);
            // pair k's row, column, their rows and the column's address (the
            // usual item is one column: no division, no table)
            auto pair_of = [&](int32_t k, int32_t &r, int32_t &j, int32_t &n, int32_t &m,
                               uint32_t &qa, uint32_t &qb) {
                if (M == 1) {
                    j = 0;
                    r = k;
                    m = len - kPad;
                    qb = qat;
                } else {
                    j = k < 64 ? j0 : div_rows(k, J.rmag);
                    r = k < 64 ? r0 : k - j * R;
                    m = cn[j];
                    qb = lds_address(lrec + cb[j]);
                }
                n = k < 64 ? rn0 : sh.rn[r];
                qa = k < 64 ? qa0 : lds_address(lrec + sh.rb[r]);
            };
            // the pairs' table and the prefix of their steps; per: steps of
            // a lane's run
            int32_t total = 0;
            for (int32_t u = 0; u < P; u += 64) {
                const int32_t k = u + lane;
                StripPair e = {0, 0, 0, 0};
                if (k < P) {
                    int32_t r, j, n, m;
                    uint32_t qb;
                    pair_of(k, r, j, n, m, e.q, qb);
                    e.S = e.q + qb;
                    e.steps = r < diag + j + gram ? padded_steps(n, m) : 0;
                }
                const int32_t inc = wave_scan<false>(e.steps);
                e.excl = total + inc - e.steps;
                total += __builtin_amdgcn_readlane(inc, 63);
                if (k < P)
                    pairs[k] = e;
            }
            total = __builtin_amdgcn_readfirstlane(total);
            int32_t per = ((total + 63) / 64 + kStepBlock - 1) & ~(kStepBlock - 1);
            per = per < kStepBlock ? kStepBlock : per;
            const float inv_per = __builtin_amdgcn_rcpf((float)per);
            // x / per (quot_small with the reciprocal at hand)
            auto by_per = [&](int32_t x) {
                int32_t q = (int32_t)((float)x * inv_per);
                const int32_t rem = x - q * per;
                return q + (rem >= per ? 1 : 0) - (rem < 0 ? 1 : 0);
            };
            wave_lds();
            // for each lane the pair holding its first step: the last pair
            // with steps that starts at or before it
            for (int32_t u = 0; u < P; u += 64) {
                const int32_t k = u + lane;
                if (k < P) {
                    const int32_t f = by_per(pairs[k].excl + per - 1);
                    if (f < 64 && pairs[k].steps > 0)
                        atomicMax(&head[f], k);
                }
            }
            wave_lds();
            const int32_t k0 = wave_scan<true>(head[lane]);
            wave_lds();

            const int32_t s0 = lane * per;
            if (s0 < total) {
                StripChain<T> ch;
                double *slot = part + (k0 + lane);
                const StripPair *next = pairs + k0;
                int32_t todo = s0 + per < total ? per : total - s0;
                {
                    const StripPair e = *next;
                    const int32_t j = M == 1 ? 0 : div_rows(k0, J.rmag);
                    const int32_t na = sh.rn[k0 - j * R], nb = M == 1 ? len - kPad : cn[j];
                    const int32_t d = s0 - e.excl;
                    strip_start<T>(ch.w, ch.x, e, na, nb, d);
                    ch.left = e.steps - d;
                }
                ch.load();
                ch.acc = 0.0;
                // left: steps to the end of the pair or of the run; todo: the
                // run's steps after that
                ch.left = ch.left < todo ? ch.left : todo;
                todo -= ch.left;
                for (;;) {
                    T sum = T(0);
                    strip_block<T, HK>(ch, sum, p,
                                       std::make_integer_sequence<int, kStepBlock>());
                    ch.acc += (double)sum;
                    ch.left -= kStepBlock;
                    if (ch.left == 0) {
                        *slot = ch.acc;
                        if (todo == 0)
                            break;
                        // the next pair with steps (row by row of a column,
                        // then the next column)
                        StripPair e;
                        do {
                            ++slot;
                            e = *++next;
                        } while (e.steps == 0);
                        ch.w.q = e.q;
                        ch.w.S = e.S;
                        ch.left = e.steps < todo ? e.steps : todo;
                        todo -= ch.left;
                        ch.load();
                        ch.x = T(0);
                        ch.acc = 0.0;
                    }
                }
            }
            wave_lds();

            // finish: a pair's partial sums in lane order, the unbounded-tail
            // rule, the root, and the entry's two places
#pragma unroll 1
            for (int32_t k = lane; k < P; k += 64) {
                int32_t r, j, n, m;
                uint32_t qa, qb;
                pair_of(k, r, j, n, m, qa, qb);
                if (r > diag + j)
                    continue;  // the mirrored half of a diagonal block
                const int32_t s = pairs[k].steps, b = pairs[k].excl;
                double val = 0.0;
                if (s > 0) {
                    const double *q = part + (k + by_per(b));
                    const double *const q1 = part + (k + by_per(b + s - 1));
                    for (; q + 3 <= q1; q += 4) {
                        const double v0 = q[0], v1 = q[1], v2 = q[2], v3 = q[3];
                        val = (((val + v0) + v1) + v2) + v3;
                    }
                    for (; q <= q1; ++q)
                        val += *q;
                }
                typedef const __attribute__((address_space(3))) Rec<T> *rec_ptr;
                const T lr = ((rec_ptr)(size_t)qa)[n - 1].v;
                const T lc = ((rec_ptr)(size_t)qb)[m - 1].v;
                const T ht = hval<T, HK>(lr, lc, p);
                if (ht != T(0))
                    val = ht > T(0) ? INFINITY : -INFINITY;
                if constexpr (RT == kRootSqrt)
                    val = sqrt(val);
                else if constexpr (RT == kRootPow)
                    val = pow(val, args.inv_p);
                if (args.accumulate != 0)  // a term of a sum (no root: checked on the host)
                    val *= args.coef;
                const T res = (T)val;
                const int64_t c = M == 1 ? c0 : c0 + j;
                const int64_t dr = k < 64 ? 0 : r - r0;  // (from the first 64 pairs' row)
                const int64_t at_row = row_at + dr * J.ldo + c;
                const int64_t at_col = col_at + dr + (c - J.row0) * J.ldo;
                const bool first = !J.swap;
                const bool second = J.swap || (J.mirror && r != diag + j);
                if (args.accumulate == 1) {
                    // each entry has one writer per launch; the terms'
                    // launches are ordered on the stream
                    if (first)
                        out[at_row] += res;
                    if (second)
                        out[at_col] += res;
                } else {
                    if (first)
                        out[at_row] = res;
                    if (second)
                        out[at_col] = res;
                }
            }
            wave_lds();
            g = gnext;
            gr = grn;
        }
        // nothing of this job is waited for any more
        if (lane == 0)
            busy[wave] = groups[g1].virt + 0x20000000u;
        // load for the next job while the other waves finish (once it is
        // known: its fields are written before valid)
        const int32_t known = *(lds_i32)(size_t)lds_address(&sh.job[cur ^ 1].valid);
        if (known > 0) {
            asm volatile("" ::: "memory");  // (the fields after valid)
            load_job(sh.job[cur ^ 1]);
        }
        sync_lds();
        if (known < 0 && sh.job[cur ^ 1].valid)
            load_job(sh.job[cur ^ 1]);
    }
}

template <typename T, int HK, int RT>
static hipError_t launch_strips_t(const FwdArgs &a, const StripLaunch &l, hipStream_t s)
{
    const hipError_t e = ensure_dynamic_lds(
        reinterpret_cast<const void *>(&pairwise_strips<T, HK, RT>), kStripLdsBytes);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((pairwise_strips<T, HK, RT>), dim3(l.grid), dim3(64 * l.waves),
                       (size_t)l.lds_bytes, s, a);
    return hipGetLastError();
}

// The (h, root) combinations of launch_forward.
template <typename T>
static hipError_t launch_strips_dtype(int hk, const FwdArgs &a, const StripLaunch &l,
                                      hipStream_t s)
{
    switch (hk) {
    case kAbs: return launch_strips_t<T, kAbs, kRootNone>(a, l, s);
    case kProd: return launch_strips_t<T, kProd, kRootNone>(a, l, s);
    case kSqr:
        return a.root == kRootSqrt ? launch_strips_t<T, kSqr, kRootSqrt>(a, l, s)
                                   : launch_strips_t<T, kSqr, kRootNone>(a, l, s);
    case kPowHalf:
        return a.root == kRootPow ? launch_strips_t<T, kPowHalf, kRootPow>(a, l, s)
                                  : launch_strips_t<T, kPowHalf, kRootNone>(a, l, s);
    case kPowInt:
        return a.root == kRootPow ? launch_strips_t<T, kPowInt, kRootPow>(a, l, s)
                                  : launch_strips_t<T, kPowInt, kRootNone>(a, l, s);
    default:
        return a.root == kRootPow ? launch_strips_t<T, kPow, kRootPow>(a, l, s)
                                  : launch_strips_t<T, kPow, kRootNone>(a, l, s);
    }
}

hipError_t launch_strips(bool f64, int hk, const FwdArgs &a, const StripLaunch &l,
                         hipStream_t s)
{
    return f64 ? launch_strips_dtype<double>(hk, a, l, s)
               : launch_strips_dtype<float>(hk, a, l, s);
}

}  // namespace pcf
