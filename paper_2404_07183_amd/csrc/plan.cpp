// plan.cpp -- host-side tile planner (see plan.hpp).
#include "plan.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace pcf {

int64_t lds_record_capacity(int rec_bytes, bool backward)
{
    // the adjoint keeps two 64-bit gradient accumulators per record slot,
    // at a fixed distance from the records
    if (backward)
        return adj_lds_records(rec_bytes);
    return kLdsRecordBytes / rec_bytes;
}

int64_t block_budget(int rec_bytes, bool backward, const TileShape &shape)
{
    const int32_t d = shape.budget_div >= 2 ? shape.budget_div : 2;
    return lds_record_capacity(rec_bytes, backward) / d;
}

void build_blocks(const int64_t *offsets, int64_t lo, int64_t hi,
                  std::vector<int64_t> cuts, int64_t budget, int32_t max_block,
                  std::vector<int32_t> &blocks)
{
    std::sort(cuts.begin(), cuts.end());
    size_t ci = 0;
    for (int64_t i = lo; i < hi;) {
        blocks.push_back((int32_t)i);
        while (ci < cuts.size() && cuts[ci] <= i)
            ++ci;
        int64_t most = std::min(hi, i + std::max(max_block, 1));
        if (ci < cuts.size())
            most = std::min(most, cuts[ci]);
        // the most PCFs within the budget (at least one)
        const int64_t limit = offsets[i] + i * kPad + budget;
        int64_t e = i + 1;
        if (offsets[most] + most * kPad <= limit)
            e = most;
        while (e < most) {
            const int64_t mid = (e + most + 1) / 2;
            if (offsets[mid] + mid * kPad <= limit)
                e = mid;
            else
                most = mid - 1;
        }
        i = e;
    }
}

namespace {

// Index of the block starting at PCF i (i is a block boundary).
int32_t block_at(const std::vector<int32_t> &blocks, int64_t i)
{
    auto it = std::lower_bound(blocks.begin(), blocks.end(), (int32_t)i);
    return (int32_t)(it - blocks.begin());
}

bool check_offsets(int64_t n, const int64_t *offsets, std::string &err)
{
    if (n < 0) {
        err = "n < 0";
        return false;
    }
    if (n > 0 && offsets == nullptr) {
        err = "offsets is NULL";
        return false;
    }
    if (n > 0 && offsets[0] != 0) {
        err = "offsets[0] != 0";
        return false;
    }
    if (n >= ((int64_t)1 << 31)) {
        err = "more than 2^31 - 1 PCFs";
        return false;
    }
    for (int64_t i = 0; i < n; ++i) {
        if (offsets[i + 1] <= offsets[i]) {
            err = "PCF " + std::to_string(i) +
                  " has no rows (every PCF needs at least one row)";
            return false;
        }
        if (offsets[i + 1] - offsets[i] >= kMaxRows) {
            err = "PCF " + std::to_string(i) + " has 2^30 rows or more";
            return false;
        }
    }
    return true;
}

// A rectangle or triangle of the matrix with one output mapping: PCF rows
// [ra, rb) against columns [ca, cb) (triangle: of [ra, rb) with itself).
struct Region {
    int64_t ra, rb, ca, cb;
    Segment map;  // type, mirror and the output mapping
};

double region_pairs(const Region &g)
{
    const double m = (double)(g.rb - g.ra);
    return g.map.type == kSegTriangle ? 0.5 * m * (m + 1) : m * (double)(g.cb - g.ca);
}

// Strip plans (strips.hip): waves a workgroup (16 beat 12 by 3 to 20 % and 8
// by 25 % and more: fewer hide less of each other's latency); ring records
// over the records in flight (less makes waves wait for the oldest group,
// more takes rows from the row blocks; FP32 records leave room for more); the
// share of the work left that goes into the next run of every CU (the XCDs
// differ by up to 15 % in speed, so the first runs must leave enough to even
// that out); the fewest items a wave in a run; an item's and a job's cost
// beside the merge, in steps of a wave.
constexpr int kStripWaves = 16;
constexpr double kRunShare = 0.55, kRunLeast = 2.0, kItemSteps = 16.0, kJobSteps = 40.0;
constexpr double strip_ring(int rec_bytes, int64_t mean)
{
    return rec_bytes == 16 || mean > 400 ? 1.25 : 1.45;
}

// Whether a strip plan is the faster one, for PCFs of `mean` rows and K steps
// for every lane of the chip. Measured on MI355X (L1, tile kernel / strip
// kernel, us; row counts uniform around the mean):
//   FP64 rows  25: K 300 122 / 100   K 3000 1014 / 576   K 40000 12420 / 6435
//   FP64 rows 200: K 1000 180 / 195  K 3000  480 / 474   K 40000  5929 / 5125
//   FP64 rows 400: K 1000 253 / 232  K 3000  731 / 579   K 40000  9093 / 6400
//   FP32 rows  50: K 300  78 /  73   K 3000  656 / 374   K 40000  8331 / 3661
//   FP32 rows  85: K 1500 207 / 195  K 3000  402 / 330   K 12000  1483 / 1066
//   FP32 rows 120: K 1500 181 / 187  K 3000  333 / 313   K 12000  1307 / 1022
//   FP32 rows 150: K 1500 169 / 188  K 3000  315 / 327   K  6000   612 /  553
//   FP32 rows 200: K 1500 161 / 189  K 6000  552 / 555   K 12000  1076 / 1000
//   FP32 rows 800: K 1000 153 / 188  K 3000  430 / 414   K 40000  5031 / 4527
// Tiles of short PCFs are bounded by their PCF count and fill LDS badly;
// elsewhere a strip's jobs must outweigh their starts and ends.
// `spread` is the mean square of the row counts over their squared mean, and
// so spread times mean the length of the PCF that a step belongs to: columns
// of very different lengths make waves wait for the oldest one's place in the
// ring. That decides where the columns of all waves are long against LDS (7,000
// PCFs: 1 % of 2,500 rows among 20, FP64 2896 / 4270; 0.5 % of 2,000 among 40, FP64
// 2013 / 2079, FP32 1972 / 2229; 3 % of 600 among 30, FP64 2469 / 2063) or the gain
// is small (10 % of 400 among 100, 2,500 PCFs 485 / 535; 1 % of 3,000 among 700, 600
// PCFs 325 / 368; 128 problems of geometric row counts, spread 2, 2350 / 2500).
// A strip plan also takes the host longer to make and to copy, by about 25 us
// and 5 us more for every thousand PCFs. Where that outweighs the gain of a
// short launch it decides for sets used once (L1 FP64, us, calls in a stream
// and alone): rows 46, 1,600 PCFs 126 / 125 and 133 / 157; 2,200 229 / 182 and
// 237 / 221; 600 x 4,400 195 / 188 and 209 / 244. Rows 100, 600 x 6,600 470 / 478
// and 507 / 541; 2,850 PCFs 501 / 470 and 522 / 515. Rows 200, 100 x 20,000 520 /
// 500 and 599 / 630; rows 275, 301 x 5,003 527 / 488 and 605 / 604; rows 400, 50 x
// 5,500 234 / 248 and 276 / 313; 820 PCFs 270 / 250 and 295 / 286. FP32, rows 100,
// 300 x 13,107 362 / 349 and 422 / 463; 2,804 PCFs 360 / 332 and 392 / 376; rows 150,
// 300 x 17,476 611 / 588 and 680 / 712.
bool strips_pay(double mean, double spread, double longest, double K, double lane_pairs,
                int64_t pcfs, int rec_bytes)
{
    const double n = (double)pcfs;
    const bool f64 = rec_bytes == 16;
    if (mean < 100.0 && spread * mean > (f64 ? 400.0 : 550.0))
        return false;
    if (mean <= 64.0)
        return K >= 200.0 && lane_pairs >= 3.0 + n / 600.0;
    // (the line rises no further from 10,000 PCFs on, for sets used again: 519
    // problems of 100 PCFs of 200 rows, FP64, reused 831 / 717, new and alone 1087 /
    // 1210)
    const double plan = std::min(n, 1e4);
    if (spread > (mean < 100.0 || mean >= 300.0 ? 1.6 : (f64 ? 1.3 : 1.4)) ||
        (mean >= 100.0 && longest > 4.0 * mean))
        return false;
    if (!f64) {
        if (mean >= 200.0)
            return K >= (mean >= 600.0 ? 3000.0 : 16000.0);
        return K >= (mean >= 150.0 ? 5700.0 : (mean >= 100.0 ? 2700.0 : 2500.0)) +
                        plan / 12.5;
    }
    if (mean >= 300.0)
        return K >= (mean >= 600.0 ? 300.0 : 800.0) + plan / 25.0;
    return K >= (mean >= 150.0 ? 2700.0 : 2850.0) + plan / 12.5;
}

// The most rows of a block, so that no column takes the wave that merges it
// with the block longer than a share of the whole launch: the steps of a lane
// against those the launch has for each (a pair counts 64 steps more, what else
// it costs). 64 rows where that is within 0.3 of them, else rows for 0.2. (The
// first rows of a triangle are no columns of another block.) Tile kernel, 64
// rows, rows so bounded, us: 2,000 PCFs, 1 % of 600 rows among 30, FP64 203 / 242 /
// 169, FP32 171 / 192 / 125; 5 % of 400 among 20 228 / 321 / 195 and 185 / 238 / 126;
// 3,000 PCFs, 3 % of 800 among 20, FP32 441 / 495 / 377; 2,003 of geometric counts
// and four of 900, FP64 185 / 201 / 142. Tiles are faster below 12 rows (3,000 PCFs,
// four of 3,000 rows among 40, FP32, 11 rows 324 / 400 / 386) and where one column
// fills a sixth of LDS, so that fewer rows leave no room for more columns at a
// time (the same, FP64, 27 rows 406 / 410 / 446).
constexpr int64_t kStripTailRows = 12;
int64_t strip_tail_rows(const int64_t *offsets, const std::vector<Region> &regions, double mean,
                        double lane_pairs, int64_t longest_bytes)
{
    if (mean >= 100.0)  // (no column much longer than the others: strips_pay)
        return kStripMaxRows;
    int64_t column = 1;
    for (const Region &g : regions) {
        const bool tri = g.map.type == kSegTriangle;
        const bool tall = g.rb - g.ra > g.cb - g.ca;  // (its rows stream)
        const int64_t a = tri ? g.ra + kStripMaxRows : (tall ? g.ra : g.ca);
        const int64_t b = tri || tall ? g.rb : g.cb;
        for (int64_t i = a; i < b; ++i)
            column = std::max(column, offsets[i + 1] - offsets[i]);
    }
    const double rows = lane_pairs * (2.0 * mean + 64.0) * 64.0 / (double)column;
    if (0.3 * rows >= (double)kStripMaxRows)
        return kStripMaxRows;
    return 6 * longest_bytes > kStripLdsBytes ? 0 : (int64_t)(0.2 * rows);
}

// Strip plan of the regions over PCFs [lo, hi); false where the tile plan is
// the better one or a PCF is too long for LDS beside the others.
bool build_strips(const int64_t *offsets, int64_t lo, int64_t hi,
                  const std::vector<int64_t> &cuts, std::vector<Region> regions,
                  int rec_bytes, const TileShape &shape, int cus, Plan &plan)
{
    int64_t longest = 0;
    double squares = 0.0;
    for (int64_t i = lo; i < hi; ++i) {
        const int64_t r = offsets[i + 1] - offsets[i];
        longest = std::max(longest, r + kPad);
        squares += (double)r * (double)r;
    }
    const int64_t recs = offsets[hi] - offsets[lo] + (hi - lo) * kPad;
    const int64_t mean = (recs + (hi - lo) - 1) / (hi - lo);
    double pairs = 0.0;
    for (const Region &g : regions)
        pairs += region_pairs(g);
    // Steps of a lane's run in an item, s. An item costs about kItemSteps
    // steps of a wave's time beside its merge, and at a job's end a wave waits
    // for half an item on average: with K steps for every lane of the chip the
    // time goes with (s + kItemSteps) (K / s + 1/2), smallest at
    // s = sqrt(2 K kItemSteps).
    const double mean_steps = 2.0 * (double)(mean - kPad);
    const double rows = (double)(offsets[hi] - offsets[lo]) / (double)(hi - lo);
    const double lane_pairs = pairs / (64.0 * cus * kStripWaves);
    if (!strips_pay(rows, squares / (double)(hi - lo) / (rows * rows), (double)(longest - kPad),
                    lane_pairs * mean_steps, lane_pairs, hi - lo, rec_bytes))
        return false;
    const int64_t tail_rows =
        strip_tail_rows(offsets, regions, rows, lane_pairs, longest * rec_bytes);
    if (tail_rows < kStripTailRows)
        return false;
    int waves = kStripWaves;
    int64_t R = 0, M = 1, ring = 0, area = 0;
    for (; waves >= 4; waves -= 4) {  // (fewer waves for long PCFs)
        const double K = pairs * mean_steps / (64.0 * cus * waves);
        const double run = std::min({K, std::sqrt(2.0 * K * kItemSteps), 400.0});
        const double item = std::max(1.0, run * 64.0 / mean_steps);  // pairs
        int64_t most = shape.max_block >= kMaxBlock ? kStripMaxRows : shape.max_block;
        most = std::max<int64_t>(1, std::min({most, (int64_t)item, tail_rows}));
        auto fit = [&](int64_t cols) {
            M = cols;
            R = most;
            for (int it = 0; it < 3; ++it) {  // (the rows a block gets depend on the
                                              // waves' areas, and they on the rows)
                const int64_t bytes =
                    kStripLdsBytes - kStripSharedBytes -
                    (int64_t)waves * strip_wave_bytes((int)(R * M), (int)M);
                ring = std::max((int64_t)(strip_ring(rec_bytes, mean) * (double)(waves * M * mean)),
                                longest + 2 * M * mean);
                area = bytes / rec_bytes - ring;
                // (short PCFs among the rows let a block hold more than the
                // mean)
                R = std::max<int64_t>(1, std::min(most, area * 13 / 10 / mean));
            }
            return area >= longest && area >= 4 * mean;
        };
        bool fits = fit(1);
        // (another column only where a full row block is too little work, and
        // the longest PCF still fits beside it)
        while (fits && R >= tail_rows && (double)(R * (M + 1)) <= item + 1.0 &&
               R * (M + 1) <= kStripMaxPairs && M < kStripMaxCols) {
            if (!fit(M + 1)) {
                fit(M - 1);
                break;
            }
        }
        if (fits)
            break;
    }
    if (waves < 4)
        return false;
    area = std::min(area, R * longest);
    if (shape.budget_div > 2)
        area = std::max(longest, area * 2 / shape.budget_div);

    plan.blocks.clear();
    build_blocks(offsets, lo, hi, cuts, area, (int32_t)R, plan.blocks);
    plan.blocks.push_back((int32_t)hi);
    const int64_t nblk = (int64_t)plan.blocks.size() - 1;
    // column groups: at most M PCFs, within one block, at their ring places
    const int64_t most_recs = std::max(longest, M * mean * 5 / 4);
    std::vector<int32_t> gfirst((size_t)nblk + 1);
    const size_t most_groups = (size_t)(M == 1 ? hi - lo : (hi - lo) * 2 / M + nblk) + 1;
    plan.groups.clear();
    plan.groups.reserve(most_groups);
    plan.sblocks.reserve((size_t)nblk);
    std::vector<int32_t> longs;  // groups far longer than the others
    uint32_t virt = 0;
    int64_t at = 0;  // virt modulo the ring
    auto place = [&](int64_t start, int64_t cols, int64_t len) {
        if (len > 3 * M * mean)
            longs.push_back((int32_t)plan.groups.size());
        if (at + len > ring) {  // no group crosses the ring's end
            virt += (uint32_t)(ring - at);
            at = 0;
        }
        plan.groups.push_back({(int32_t)start, (int32_t)(offsets[start] + start * kPad),
                               (int32_t)(len + (cols << kStripColShift)), virt});
        virt += (uint32_t)len;
        at += len;
    };
    for (int64_t b = 0; b < nblk; ++b) {
        gfirst[(size_t)b] = (int32_t)plan.groups.size();
        int64_t i = plan.blocks[(size_t)b];
        const int64_t e = plan.blocks[(size_t)b + 1];
        plan.sblocks.push_back({(int32_t)i, (int32_t)(e - i), (int32_t)(offsets[i] + i * kPad),
                                (int32_t)(offsets[e] - offsets[i] + (e - i) * kPad)});
        while (i < e) {
            int64_t j = i, len = 0;
            do {
                len += offsets[j + 1] - offsets[j] + kPad;
                ++j;
            } while (j < e && j - i < M &&
                     len + offsets[j + 1] - offsets[j] + kPad <= most_recs);
            place(i, j - i, len);
            i = j;
        }
    }
    gfirst[(size_t)nblk] = (int32_t)plan.groups.size();
    plan.groups.push_back({(int32_t)hi, 0, 0, virt});

    plan.strips = true;
    plan.strip_waves = waves;
    plan.strip_row_recs = (int32_t)area;
    plan.strip_ring_recs = (int32_t)ring;
    plan.strip_pairs = (int32_t)(R * M);
    plan.strip_cols = (int32_t)M;
    // Runs of equal cost: the (row block, group) items of all regions in
    // order, cut into runs (a workgroup's work between two tickets). One run a
    // CU unless the launch is long (then the queue evens out what the cost
    // misses); a run that crosses row blocks holds several jobs.
    // (a block's cost over groups [g0, g1) by the offsets of their first PCFs)
    auto range_cost = [&](int64_t rows, int64_t rowrows, int64_t g0, int64_t g1) {
        const int64_t c0 = plan.groups[(size_t)g0].start, c1 = plan.groups[(size_t)g1].start;
        return (double)(g1 - g0) * kItemSteps +
               (double)(rows * (offsets[c1] - offsets[c0]) + (c1 - c0) * rowrows) / 64.0;
    };
    double total = 0.0, items = 0.0;
    for (Region &g : regions) {
        if (g.map.type == kSegRect && g.rb - g.ra > g.cb - g.ca) {
            // the longer side streams
            std::swap(g.ra, g.ca);
            std::swap(g.rb, g.cb);
            g.map.swap = 1;
        }
        Segment s = g.map;
        s.b0 = block_at(plan.blocks, g.ra);
        s.b1 = block_at(plan.blocks, g.rb);
        s.c0 = block_at(plan.blocks, g.ca);
        s.c1 = block_at(plan.blocks, g.cb);
        plan.segs.push_back(s);
        for (int32_t b = s.b0; b < s.b1; ++b) {
            const int64_t lo_ = plan.blocks[(size_t)b], hi_ = plan.blocks[(size_t)b + 1];
            const int64_t g0 = gfirst[(size_t)(s.type == kSegTriangle ? b : s.c0)];
            total += kJobSteps * waves +
                     range_cost(hi_ - lo_, offsets[hi_] - offsets[lo_], g0,
                                gfirst[(size_t)s.c1]);
            items += (double)(gfirst[(size_t)s.c1] - g0);
        }
    }
    // a run for every CU from a share of what is left, then again: few long
    // runs first, short ones last
    const double least = std::min(total / items * kRunLeast * waves, total / cus);
    double left = total, target = 0.0;
    int batch = 0;
    auto next_target = [&]() {
        if (batch == 0) {
            target = std::max(least, left * kRunShare / cus);
            batch = cus;
        }
        --batch;
    };
    next_target();
    double used = 0.0;  // cost of the current run so far
    plan.runs.push_back(0);
    for (size_t q = 0; q < plan.segs.size(); ++q) {
        const Segment &s = plan.segs[q];
        const int64_t gend = gfirst[(size_t)s.c1];
        for (int32_t b = s.b0; b < s.b1; ++b) {
            const int64_t rows = plan.blocks[(size_t)b + 1] - plan.blocks[(size_t)b];
            const int64_t rowrows = offsets[plan.blocks[(size_t)b + 1]] -
                                    offsets[plan.blocks[(size_t)b]];
            int64_t g0 = gfirst[(size_t)(s.type == kSegTriangle ? b : s.c0)];
            while (g0 < gend) {
                // the groups that fit the run (records of a job's columns stay
                // below 2^28, see busy in strips.hip)
                const double room = target - used - kJobSteps * waves;
                auto fits = [&](int64_t g) {
                    return range_cost(rows, rowrows, g0, g) <= room &&
                           plan.groups[(size_t)g].virt - plan.groups[(size_t)g0].virt <
                               (1u << 28);
                };
                // most groups within the room (at least one): from where the
                // row block's mean cost a group puts it, by growing steps
                const double guess =
                    room * (double)(gend - g0) / range_cost(rows, rowrows, g0, gend);
                int64_t lo_ = g0 + 1, hi_ = gend;
                if (guess < (double)(gend - g0)) {
                    const int64_t g = std::max(lo_, g0 + (int64_t)guess);
                    if (g == lo_ || fits(g)) {
                        lo_ = g;
                        for (int64_t d = 1; lo_ + d <= gend; d *= 2) {
                            if (!fits(lo_ + d)) {
                                hi_ = lo_ + d - 1;
                                break;
                            }
                            lo_ += d;
                        }
                    } else {
                        hi_ = g - 1;
                        for (int64_t d = 1; hi_ - d > lo_; d *= 2) {
                            if (fits(hi_ - d)) {
                                lo_ = hi_ - d;
                                break;
                            }
                            hi_ -= d;
                        }
                    }
                }
                while (lo_ < hi_) {
                    const int64_t mid = (lo_ + hi_ + 1) / 2;
                    if (fits(mid))
                        lo_ = mid;
                    else
                        hi_ = mid - 1;
                }
                // (a few items left of the row block stay with it)
                if (gend - lo_ < waves &&
                    plan.groups[(size_t)gend].virt - plan.groups[(size_t)g0].virt < (1u << 28))
                    lo_ = gend;
                plan.jobs.push_back({(int32_t)q, b, (int32_t)g0, (int32_t)lo_});
                // (a job lasts at least as long as its longest item, which one
                // wave merges while the others wait)
                const double work = range_cost(rows, rowrows, g0, lo_);
                double cost = work;
                for (auto l = std::lower_bound(longs.begin(), longs.end(), (int32_t)g0);
                     l != longs.end() && *l < lo_; ++l)
                    cost = std::max(cost, waves * range_cost(rows, rowrows, *l, *l + 1));
                used += kJobSteps * waves + cost;
                left -= kJobSteps * waves + work;
                g0 = lo_;
                if (used >= 0.9 * target) {
                    plan.runs.push_back((int32_t)plan.jobs.size());
                    used = 0.0;
                    next_target();
                }
            }
        }
    }
    if (plan.runs.back() != (int32_t)plan.jobs.size())
        plan.runs.push_back((int32_t)plan.jobs.size());
    plan.ntiles = (int64_t)plan.runs.size() - 1;
    return true;
}

// The most PCFs a block of a tile plan should hold on `cus` CUs. Where the
// largest blocks give far fewer tiles than CUs, smaller ones spread the steps:
// a tile then takes its lanes' runs of steps, against a start of workgroups
// that grows with their number (about 100 steps for one on every CU; beyond
// two thirds of the CUs nothing is gained). Kernel with its launch, 200 PCFs
// of 10 to 100 rows, L1 FP64, by PCFs a block: 32 (28 tiles) 31.3 us, 20 25.4,
// 16 (91 tiles) 23.6, 10 (210 tiles) 23.6, 8 33.2. Not for the adjoint, whose
// FP32 gradients round once for every tile that adds to them.
int32_t tile_block_cap(const int64_t *offsets, int64_t lo, int64_t hi,
                       const std::vector<Region> &regions, int64_t budget, int cus)
{
    constexpr double kStartSteps = 100.0, kMostCus = 0.66;
    const double n = (double)(hi - lo), recs = (double)(offsets[hi] - offsets[lo]) + n * kPad;
    const double mean = recs / n, steps = 2.0 * (mean - kPad) + kStepBlock / 2;
    int32_t best = kMaxBlock;
    double best_time = 0.0;
    for (int32_t m = kMaxBlock; m >= 4; --m) {
        const double b = std::min((double)m, std::max(1.0, (double)budget / mean));
        double tiles = 0.0;
        for (const Region &g : regions) {
            const double nr = std::ceil((double)(g.rb - g.ra) / b);
            tiles += g.map.type == kSegTriangle
                         ? 0.5 * nr * (nr + 1.0)
                         : nr * std::ceil((double)(g.cb - g.ca) / b);
        }
        if (tiles > kMostCus * cus)
            break;
        const double time = b * b * steps / kThreads + kStartSteps * tiles / cus;
        if (m == kMaxBlock || time < best_time) {
            best = m;
            best_time = time;
        }
    }
    return best;
}

void add_segment(Plan &plan, Segment s, int64_t tiles)
{
    if (tiles <= 0)
        return;
    s.tile_begin = plan.ntiles;
    plan.segs.push_back(s);
    plan.ntiles += tiles;
}

}  // namespace

bool plan_matrix(int64_t n, const int64_t *offsets, int rec_bytes,
                 bool backward, bool windowed, int64_t r0, int64_t r1,
                 int64_t c0, int64_t c1, bool upper_only, int64_t ldo,
                 const TileShape &shape, Plan &plan, std::string &err,
                 int cus)
{
    plan = Plan();
    if (!check_offsets(n, offsets, err))
        return false;
    if (!windowed) {
        r0 = c0 = 0;
        r1 = c1 = n;
    }
    if (r0 < 0 || r1 < r0 || r1 > n || c0 < 0 || c1 < c0 || c1 > n) {
        err = "window out of range";
        return false;
    }
    if (ldo < (c1 - c0) || ldo < 1) {
        if (!(r1 == r0 || c1 == c0)) {
            err = "ldo smaller than the window width";
            return false;
        }
    }
    plan.npcf = n;
    plan.rec_count = (n > 0 ? offsets[n] : 0) + n * kPad;
    plan.lds_records = lds_record_capacity(rec_bytes, backward);
    plan.backward = backward;
    if (r1 == r0 || c1 == c0)
        return true;

    const int64_t d0 = std::max(r0, c0), d1 = std::min(r1, c1);
    const bool has_d = d0 < d1;
    const int64_t lo = std::min(r0, c0), hi = std::max(r1, c1);
    std::vector<int64_t> cuts = {r0, r1, c0, c1};
    if (has_d) {
        cuts.push_back(d0);
        cuts.push_back(d1);
    }
    // the window's parts: the triangle of its symmetric part; rows outside
    // the overlap against every column; overlap rows against columns outside
    // it (the transposes of these entries lie outside the window, so nothing
    // is mirrored)
    std::vector<Region> regions;
    Segment base{};
    base.obase = 0;
    base.ldo = ldo;
    base.row0 = r0;
    base.col0 = c0;
    auto rect = [&](int64_t ra, int64_t rb, int64_t ca, int64_t cb) {
        if (ra >= rb || ca >= cb)
            return;
        Segment s = base;
        s.type = kSegRect;
        regions.push_back({ra, rb, ca, cb, s});
    };
    if (has_d) {
        Segment s = base;
        s.type = kSegTriangle;
        s.mirror = upper_only ? 0 : 1;
        regions.push_back({d0, d1, d0, d1, s});
        rect(r0, std::min(r1, d0), c0, c1);
        rect(std::max(r0, d1), r1, c0, c1);
        rect(d0, d1, c0, std::min(c1, d0));
        rect(d0, d1, std::max(c0, d1), c1);
    } else {
        rect(r0, r1, c0, c1);
    }
    if (cus > 0 && !backward &&
        build_strips(offsets, lo, hi, cuts, regions, rec_bytes, shape, cus, plan))
        return true;

    const int64_t budget = block_budget(rec_bytes, backward, shape);
    build_blocks(offsets, lo, hi, cuts, budget,
                 cus > 0 && !backward && shape.preset
                     ? tile_block_cap(offsets, lo, hi, regions, budget, cus)
                     : shape.max_block,
                 plan.blocks);
    plan.blocks.push_back((int32_t)hi);
    for (const Region &g : regions) {
        Segment s = g.map;
        s.b0 = block_at(plan.blocks, g.ra);
        s.b1 = block_at(plan.blocks, g.rb);
        s.c0 = block_at(plan.blocks, g.ca);
        s.c1 = block_at(plan.blocks, g.cb);
        const int64_t nb = s.b1 - s.b0;
        add_segment(plan, s,
                    s.type == kSegTriangle ? nb * (nb + 1) / 2 : nb * (s.c1 - s.c0));
    }
    return true;
}

bool plan_batched(int32_t B, const int64_t *set_offsets,
                  const int64_t *out_offsets, const int64_t *offsets,
                  int64_t n, int rec_bytes, bool upper_only,
                  const TileShape &shape, Plan &plan, std::string &err,
                  int cus)
{
    plan = Plan();
    if (B < 0 || (B > 0 && (!set_offsets || !out_offsets))) {
        err = "bad batch description";
        return false;
    }
    if (!check_offsets(n, offsets, err))
        return false;
    for (int32_t b = 0; b < B; ++b) {
        if (set_offsets[b] < 0 || set_offsets[b + 1] < set_offsets[b] ||
            set_offsets[b + 1] > n) {
            err = "set_offsets out of range at problem " + std::to_string(b);
            return false;
        }
        if (out_offsets[b] < 0) {
            err = "negative out_offsets at problem " + std::to_string(b);
            return false;
        }
    }
    plan.npcf = n;
    plan.rec_count = (n > 0 ? offsets[n] : 0) + n * kPad;
    plan.lds_records = lds_record_capacity(rec_bytes, false);
    if (B == 0)
        return true;
    const int64_t lo = set_offsets[0], hi = set_offsets[B];
    std::vector<int64_t> cuts(set_offsets, set_offsets + B + 1);
    struct Item {
        double cost;
        Region g;
    };
    std::vector<Item> items;
    for (int32_t b = 0; b < B; ++b) {
        const int64_t a = set_offsets[b], e = set_offsets[b + 1];
        if (a == e)
            continue;
        Segment s{};
        s.type = kSegTriangle;
        s.mirror = upper_only ? 0 : 1;
        s.obase = out_offsets[b];
        s.ldo = e - a;
        s.row0 = s.col0 = a;
        // merge steps of a set of s PCFs with R rows in total: about
        // s * R (every PCF meets every other once)
        const double cost =
            (double)(e - a) * (double)(offsets[e] - offsets[a]);
        items.push_back({cost, {a, e, a, e, s}});
    }
    std::stable_sort(items.begin(), items.end(),
                     [](const Item &x, const Item &y) { return x.cost > y.cost; });
    if (items.empty())
        return true;
    int32_t cap = shape.max_block;
    const int64_t budget = block_budget(rec_bytes, false, shape);
    if (cus > 0) {
        std::vector<Region> regions;
        for (auto &it : items)
            regions.push_back(it.g);
        if (build_strips(offsets, lo, hi, cuts, regions, rec_bytes, shape, cus, plan))
            return true;
        if (shape.preset)
            cap = tile_block_cap(offsets, lo, hi, regions, budget, cus);
    }
    build_blocks(offsets, lo, hi, cuts, budget, cap, plan.blocks);
    plan.blocks.push_back((int32_t)hi);
    for (auto &it : items) {
        Segment s = it.g.map;
        s.b0 = s.c0 = block_at(plan.blocks, it.g.ra);
        s.b1 = s.c1 = block_at(plan.blocks, it.g.rb);
        const int64_t nb = s.b1 - s.b0;
        add_segment(plan, s, nb * (nb + 1) / 2);
    }
    return true;
}

// FP32 adjoint plans: two 64-bit sums a row for PCF_DETERMINISTIC (FP64
// plans keep them in the gradient arrays themselves).
int64_t adj_acc_bytes(const Plan &plan, int rec_bytes)
{
    if (!plan.backward || rec_bytes == 16)
        return 0;
    const int64_t rows = plan.rec_count - plan.npcf * kPad;
    return align_up(rows * 16, 256);
}

int64_t plan_workspace_bytes(const Plan &plan, int rec_bytes)
{
    int64_t off = kHeaderBytes;
    off += align_up((int64_t)plan.blocks.size() * 4, 256);
    off += align_up((int64_t)plan.segs.size() * (int64_t)sizeof(Segment), 256);
    off += align_up((int64_t)plan.groups.size() * (int64_t)sizeof(StripGroup), 256);
    off += align_up((int64_t)plan.jobs.size() * (int64_t)sizeof(StripJob), 256);
    off += align_up((int64_t)plan.runs.size() * 4, 256);
    off += align_up((int64_t)plan.sblocks.size() * (int64_t)sizeof(StripBlock), 256);
    off += align_up(plan.rec_count * rec_bytes, 256);
    off += adj_acc_bytes(plan, rec_bytes);
    return off;
}

int64_t plan_workspace_bound(const Plan &plan, int rec_bytes)
{
    int64_t off = kHeaderBytes;
    off += align_up((plan.npcf + 1) * 4, 256);
    off += align_up((int64_t)plan.segs.size() * (int64_t)sizeof(Segment), 256);
    off += align_up(plan.rec_count * rec_bytes, 256);
    off += adj_acc_bytes(plan, rec_bytes);
    if (!plan.backward) {
        // a strip plan's groups and jobs (at most one job a row block of each
        // of a window's parts beside the division by size)
        off += align_up((plan.npcf + 2) * (int64_t)sizeof(StripGroup), 256);
        off += align_up((plan.npcf + 2) * (int64_t)sizeof(StripBlock), 256);
        off += align_up((3 * plan.npcf + 16384) * (int64_t)sizeof(StripJob), 256);
        off += align_up(16384 * 4, 256);
    }
    return off;
}

void plan_serialise(const Plan &plan, int rec_bytes,
                    std::vector<unsigned char> &buf, WsHeader &hdr)
{
    std::memset(&hdr, 0, sizeof(hdr));
    hdr.ntiles = plan.ntiles;
    hdr.nseg = (int64_t)plan.segs.size();
    hdr.nblocks = plan.blocks.empty() ? 0 : (int64_t)plan.blocks.size() - 1;
    hdr.npcf = plan.npcf;
    hdr.off_blocks = kHeaderBytes;
    hdr.off_segs = hdr.off_blocks + align_up((int64_t)plan.blocks.size() * 4, 256);
    hdr.off_groups = hdr.off_segs +
                     align_up((int64_t)plan.segs.size() * (int64_t)sizeof(Segment), 256);
    hdr.off_jobs = hdr.off_groups +
                   align_up((int64_t)plan.groups.size() * (int64_t)sizeof(StripGroup), 256);
    hdr.off_runs = hdr.off_jobs +
                   align_up((int64_t)plan.jobs.size() * (int64_t)sizeof(StripJob), 256);
    hdr.off_sblocks = hdr.off_runs + align_up((int64_t)plan.runs.size() * 4, 256);
    hdr.off_rec = hdr.off_sblocks +
                  align_up((int64_t)plan.sblocks.size() * (int64_t)sizeof(StripBlock), 256);
    hdr.strip_row_recs = plan.strip_row_recs;
    hdr.strip_ring_recs = plan.strip_ring_recs;
    hdr.strip_pairs = plan.strip_pairs;
    hdr.strip_cols = plan.strip_cols;
    hdr.rec_count = plan.rec_count;
    hdr.rec_bytes = rec_bytes;
    hdr.first_bad = -1;
    hdr.lds_records = plan.lds_records;
    hdr.off_acc = adj_acc_bytes(plan, rec_bytes) > 0
                      ? hdr.off_rec + align_up(plan.rec_count * rec_bytes, 256)
                      : 0;
    buf.assign((size_t)hdr.off_rec, 0);
    std::memcpy(buf.data(), &hdr, sizeof(hdr));
    if (!plan.blocks.empty())
        std::memcpy(buf.data() + hdr.off_blocks, plan.blocks.data(),
                    plan.blocks.size() * 4);
    if (!plan.segs.empty())
        std::memcpy(buf.data() + hdr.off_segs, plan.segs.data(),
                    plan.segs.size() * sizeof(Segment));
    if (!plan.groups.empty())
        std::memcpy(buf.data() + hdr.off_groups, plan.groups.data(),
                    plan.groups.size() * sizeof(StripGroup));
    if (!plan.jobs.empty())
        std::memcpy(buf.data() + hdr.off_jobs, plan.jobs.data(),
                    plan.jobs.size() * sizeof(StripJob));
    if (!plan.runs.empty())
        std::memcpy(buf.data() + hdr.off_runs, plan.runs.data(), plan.runs.size() * 4);
    if (!plan.sblocks.empty())
        std::memcpy(buf.data() + hdr.off_sblocks, plan.sblocks.data(),
                    plan.sblocks.size() * sizeof(StripBlock));
}

}  // namespace pcf
