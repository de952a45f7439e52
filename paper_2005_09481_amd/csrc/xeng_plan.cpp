// Stream-K style decomposition of the upper-triangle tiles into pieces.
#include "xeng_plan.h"
#include "xeng_plan_single.h"

#include <algorithm>
#include <cstdint>
#include <numeric>
#include <unordered_map>

namespace xeng {

std::vector<std::pair<int, int>> plan_units(int n, TileShape shape)
{
    std::vector<std::pair<int, int>> u;
    const int nt = n_tiles_side(n);
    if (shape == TileShape::Narrow) {
        u.emplace_back(0, 0);
    } else if (shape == TileShape::Region) {
        const int nr = (n + REGION - 1) / REGION;
        for (int ri = 0; ri < nr; ++ri)
            for (int rj = ri; rj < nr; ++rj) u.emplace_back(ri, rj);
    } else if (shape != TileShape::Wide) {
        for (int ti = 0; ti < nt; ++ti)
            for (int tj = ti; tj < nt; ++tj) u.emplace_back(ti, tj);
    } else {
        const int nj2 = (nt + 1) / 2;
        for (int ti = 0; ti < nt; ++ti)
            for (int j2 = ti / 2; j2 < nj2; ++j2) u.emplace_back(ti, j2);
    }
    return u;
}

// Cost of a piece beyond its stages, in stage units: its prologue (the
// first stages' loads are not yet overlapped) and its flush of the tile's
// accumulators to memory.  Measured on the DMA kernel's 128 x 256 tiles at
// about 16 stage times; a 128 x 128 tile of the general kernel flushes half
// as much.  The tile kernel's stages take half as long (24 measured best of
// 8 to 40), the region kernel's a fifth (40 best of 24 to 64).
int64_t piece_overhead(TileShape shape)
{
    switch (shape) {
    case TileShape::Wide: return 16;
    case TileShape::Tile: return 24;
    case TileShape::Region: return 40;
    default: return 8;
    }
}

int64_t piece_cap(TileShape shape) { return shape == TileShape::Square ? MAX_PIECE_STAGES : MAX_PIECE_STAGES_WIDE; }

namespace {

struct UnitRef {
    int job, ti, tj;
    int64_t ns;   // stages
    int64_t t;    // samples
    int64_t wc;   // cost of one stage (unit_stage_cost)
};

// The smallest budget from `lo` upward that fits, where every larger one then
// fits too: steps of `step`, twice as long each time, then bisection.
template <typename Fits> int64_t smallest_budget(int64_t lo, int64_t step, Fits fits)
{
    int64_t hi = lo;
    while (!fits(hi)) {
        lo = hi + 1;
        hi += step;
        step *= 2;
    }
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (fits(mid))
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// Greedy fill: workgroups in order, each taking pieces of the linear (job,
// unit, stage) order until its cost (stage costs + overhead per piece)
// would exceed `budget`.  Returns the number of workgroups used (or grid + 1 if
// the work does not fit), emitting pieces when `out` is given.
template <typename Emit>
int64_t fill(const std::vector<UnitRef> &units, int64_t budget, int64_t overhead, int64_t cap, int64_t grid,
             Emit emit)
{
    int64_t w = 0, left = budget;
    for (size_t u = 0; u < units.size(); ++u) {
        int64_t done = 0;
        const int64_t wc = units[u].wc;
        while (done < units[u].ns) {
            if (left - overhead < wc) {
                if (++w >= grid) return grid + 1;
                left = budget;
            }
            // (a whole rest that fits needs no division)
            const int64_t rest = units[u].ns - done;
            const int64_t take = rest <= cap && rest * wc <= left - overhead
                                     ? rest
                                     : std::min({rest, (left - overhead) / wc, cap});
            emit(w, u, done, done + take);
            done += take;
            left -= take * wc + overhead;
        }
    }
    return w + 1;
}

}  // namespace

Plan make_plan(const PlanJob *jobs, int n_jobs, int max_wgs, int min_stages, TileShape shape, int64_t cap_override)
{
    Plan plan;
    if (min_stages < 1) min_stages = 1;
    if (max_wgs < 1) max_wgs = 1;
    const int64_t cap = cap_override > 0 ? cap_override : piece_cap(shape);
    const int64_t ovh = piece_overhead(shape) * STAGE_COST;

    std::vector<UnitRef> units;
    int64_t total = 0, total_cost = 0;
    for (int j = 0; j < n_jobs; ++j) {
        if (jobs[j].t <= 0 || jobs[j].n <= 0) continue;
        const int64_t ns = (jobs[j].t + STAGE - 1) / STAGE;
        const int64_t nt = n_tiles_side(jobs[j].n);
        for (const auto &unit : plan_units(jobs[j].n, shape)) {
            const int64_t wc = unit_stage_cost(shape == TileShape::Wide, unit.first, unit.second, nt);
            units.push_back(UnitRef{j, unit.first, unit.second, ns, jobs[j].t, wc});
            total += ns;
            total_cost += ns * wc;
        }
    }
    if (total == 0) {
        plan.grid = 0;
        plan.wg_off.assign(1, 0);
        return plan;
    }
    const int64_t grid = std::max<int64_t>(
        1, std::min<int64_t>({(int64_t)max_wgs,
                              std::max<int64_t>((total + min_stages - 1) / min_stages, (int64_t)units.size()),
                              (int64_t)units.size() * MAX_UNIT_SPLIT}));

    // Smallest per-workgroup budget with which the greedy fill fits in
    // `grid` workgroups (the fill is monotone in the budget), from the mean
    // cost upward: every unit pays the overhead at least once.
    auto none = [](int64_t, size_t, int64_t, int64_t) {};
    const int64_t mean = (total_cost + ovh * (int64_t)units.size() + grid - 1) / grid;
    const int64_t lo = smallest_budget(std::max(ovh + STAGE_COST, mean), ovh, [&](int64_t budget) {
        return fill(units, budget, ovh, cap, grid, none) <= grid;
    });

    struct Raw { Piece p; int32_t wg; size_t unit; };
    std::vector<Raw> raw;
    std::vector<int32_t> pieces_of_unit(units.size(), 0);
    const int64_t used = fill(units, lo, ovh, cap, grid, [&](int64_t w, size_t u, int64_t a, int64_t b) {
        Raw r;
        r.p.job = units[u].job;
        r.p.tile = units[u].ti | (units[u].tj << 16);
        r.p.t0 = (int32_t)(a * STAGE);
        r.p.t1_atomic = (int32_t)std::min<int64_t>(b * STAGE, units[u].t);
        r.wg = (int32_t)w;
        r.unit = u;
        raw.push_back(r);
        pieces_of_unit[u]++;
    });
    plan.grid = (int32_t)used;
    plan.wg_off.assign((size_t)used + 1, 0);
    // a tile cut into several pieces is flushed with atomics
    for (Raw &r : raw)
        if (pieces_of_unit[r.unit] > 1) r.p.t1_atomic |= (int32_t)0x80000000u;
    // pieces come out ordered by workgroup already
    plan.pieces.reserve(raw.size());
    plan.piece_wg.reserve(raw.size());
    for (const Raw &r : raw) {
        plan.pieces.push_back(r.p);
        plan.piece_wg.push_back(r.wg);
        plan.wg_off[(size_t)r.wg + 1]++;
    }
    for (size_t w = 0; w < (size_t)used; ++w) plan.wg_off[w + 1] += plan.wg_off[w];
    return plan;
}

namespace {

// Interleaved bits of (a, b): units close in both coordinates come close
// together in this order, so a run of consecutive units covers a compact
// block of the triangle (few distinct row and column blocks).
uint32_t spread(uint32_t x)   // bit k of the low 16 to bit 2 k
{
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    return (x | (x << 1)) & 0x55555555u;
}
uint32_t morton(uint32_t a, uint32_t b) { return spread(a) << 1 | spread(b); }

// One candidate of make_plan_xcd: segments of length L (in stages of a full
// unit).  A unit whose stages cost less takes longer segments of the same
// cost, so units of one stage cost are cut alike.
struct XSeg {
    int64_t u, s0, s1;
};

struct XcdCut {
    struct Class {
        int64_t wc, units;   // stage cost, units of that cost
        int64_t len, full, tail;   // segment length, full segments of a unit, stages left over
    } cls[2];
    int64_t main = 0;         // full segments of all units
    int64_t tails = 0;        // units with a tail
    int64_t tail_cost = 0;    // of their stages
    int64_t worst = 0;        // largest cost of a full segment with its overhead
};

void cut(XcdCut &x, int64_t ns, int64_t L, int64_t ovh, int64_t cap)
{
    x.main = x.tails = x.tail_cost = x.worst = 0;
    for (XcdCut::Class &c : x.cls) {
        if (c.units == 0) continue;
        c.len = std::min({ns, cap, std::max<int64_t>(1, L * STAGE_COST / c.wc)});
        c.full = ns / c.len;
        c.tail = ns - c.full * c.len;
        x.main += c.units * c.full;
        if (c.tail > 0) {
            x.tails += c.units;
            x.tail_cost += c.units * c.tail * c.wc;
        }
        x.worst = std::max(x.worst, c.len * c.wc + ovh);
    }
}

// The tails of units of classes cls[..] by the stream-K fill, over workgroups
// `first` .. G - 1 of `budget` each: emit(workgroup, unit, first stage, end
// stage).  False if they do not fit.
template <typename Emit>
bool fill_tails(const XcdCut &x, const std::vector<uint8_t> &cls, int64_t first, int64_t G, int64_t budget, int64_t ovh,
                int64_t cap, Emit emit)
{
    int64_t k = first, left = budget;
    for (size_t u = 0; u < cls.size(); ++u) {
        const XcdCut::Class &c = x.cls[cls[u]];
        int64_t done = 0;
        while (done < c.tail) {
            if (left - ovh < c.wc) {
                if (++k >= G) return false;
                left = budget;
            }
            const int64_t rest = c.tail - done;
            const int64_t take = rest <= cap && rest * c.wc <= left - ovh
                                     ? rest
                                     : std::min({rest, (left - ovh) / c.wc, cap});
            emit(k, u, c.full * c.len + done, c.full * c.len + done + take);
            done += take;
            left -= take * c.wc + ovh;
        }
    }
    return true;
}

}  // namespace

bool make_plan_xcd(const PlanJob &job, int max_wgs, TileShape shape, Plan *out, int64_t cap_override)
{
    const int64_t G = max_wgs;
    if (G < XCDS || G % XCDS != 0 || job.n <= 0 || job.t <= 0 || shape == TileShape::Narrow) return false;
    const int64_t nt = n_tiles_side(job.n);
    const int64_t ns = (job.t + STAGE - 1) / STAGE;
    const int64_t ovh = piece_overhead(shape) * STAGE_COST;
    const int64_t cap = cap_override > 0 ? cap_override : piece_cap(shape);
    const std::vector<std::pair<int, int>> rows = plan_units(job.n, shape);
    const size_t U = rows.size();
    XcdCut x;
    x.cls[0] = {STAGE_COST, 0, 0, 0, 0};
    x.cls[1] = {HALF_WINDOW_COST, 0, 0, 0, 0};
    for (const auto &u : rows)
        x.cls[unit_stage_cost(shape == TileShape::Wide, u.first, u.second, nt) == STAGE_COST ? 0 : 1].units++;
    const int64_t total_cost = ns * (x.cls[0].units * x.cls[0].wc + x.cls[1].units * x.cls[1].wc);
    // segment lengths around the balanced share (longer ones leave less
    // for the tail workgroups): the candidate with the smallest largest
    // workgroup cost wins
    const int64_t L0 = (total_cost + STAGE_COST * G - 1) / (STAGE_COST * G);
    if (L0 < XCD_MIN_SEGMENT || L0 >= ns) return false;

    // the units in Morton order
    std::vector<std::pair<uint32_t, uint32_t>> order(U);   // (key, index into rows)
    const int col_scale = shape == TileShape::Wide ? 2 : 1;
    for (size_t u = 0; u < U; ++u)
        order[u] = {morton((uint32_t)rows[u].first, (uint32_t)(col_scale * rows[u].second)), (uint32_t)u};
    std::sort(order.begin(), order.end());
    std::vector<std::pair<int, int>> units(U);
    std::vector<uint8_t> cls(U);
    for (size_t u = 0; u < U; ++u) {
        units[u] = rows[order[u].second];
        cls[u] = unit_stage_cost(shape == TileShape::Wide, units[u].first, units[u].second, nt) == STAGE_COST ? 0 : 1;
    }

    // A candidate is cut in constant time.  The fill of its tails, a pass over
    // the units, runs where their mean leaves it a chance, and the search for
    // its smallest budget only if it fits the best cost so far (of equal
    // candidates the one of the longest segments wins).  Taken in scattered
    // order, few candidates are better than all before them.  N = 512, T =
    // 30000 (36 regions): 20 us, 1400 with every candidate's budget searched.
    auto none = [](int64_t, size_t, int64_t, int64_t) {};
    auto tails_mean = [&] { return (x.tail_cost + ovh * x.tails + G - x.main - 1) / (G - x.main); };
    auto fits = [&](int64_t b) { return fill_tails(x, cls, x.main, G, b, ovh, cap, none); };
    const int64_t L_min = std::max<int64_t>(XCD_MIN_SEGMENT, L0 - piece_overhead(shape));
    const int64_t L_count = std::min({L0 + 4 * piece_overhead(shape), cap, ns - 1}) - L_min + 1;
    int64_t best_L = -1, best_cost = INT64_MAX, step = std::max<int64_t>(1, L_count * 5 / 8);
    while (std::gcd(step, L_count) > 1) ++step;
    for (int64_t k = 0; k < L_count; ++k) {
        const int64_t L = L_min + k * step % L_count;
        cut(x, ns, L, ovh, cap);
        if (x.main > G || (x.tails > 0 && x.main == G)) continue;
        const int64_t limit = L > best_L ? best_cost : best_cost - 1;   // what this one may cost
        int64_t cost = x.worst;
        if (x.tails > 0) cost = std::max(cost, tails_mean());
        if (cost > limit) continue;
        if (x.tails > 0 && !fits(cost)) {
            if (limit < INT64_MAX - 1 && !fits(limit)) continue;
            cost = smallest_budget(cost + 1, ovh, fits);
        }
        best_cost = cost;
        best_L = L;
    }
    if (best_L < 0) return false;
    // The linear order where this one costs more than a piece's overhead
    // beyond its mean, a bound that order keeps.  It does where a few
    // workgroups are left for the tails of many units: N = 3840, T = 4096,
    // 240 windows, 16 workgroups.
    const int64_t linear = (total_cost + ovh * (int64_t)U + G - 1) / G + 2 * ovh;
    if (best_cost > linear) return false;
    cut(x, ns, best_L, ovh, cap);
    std::vector<std::vector<XSeg>> logical((size_t)G);
    size_t next = 0;
    for (int64_t p = 0; p < std::max(x.cls[0].full, x.cls[1].full); ++p)
        for (size_t u = 0; u < U; ++u) {
            const XcdCut::Class &c = x.cls[cls[u]];
            if (p < c.full) logical[next++].push_back(XSeg{(int64_t)u, p * c.len, (p + 1) * c.len});
        }
    if (x.tails > 0)
        fill_tails(x, cls, x.main, G, smallest_budget(std::max(ovh + STAGE_COST, tails_mean()), ovh, fits), ovh, cap,
                   [&](int64_t k, size_t u, int64_t s0, int64_t s1) {
                       logical[(size_t)k].push_back(XSeg{(int64_t)u, s0, s1});
                   });
    // a unit cut into several pieces is shared: flushed with atomics
    std::vector<int> pieces_of(U, 0);
    for (const auto &v : logical)
        for (const XSeg &sg : v) pieces_of[(size_t)sg.u]++;
    // logical workgroup k runs on XCD k / (G / XCDS): physical id
    // (k % (G / XCDS)) * XCDS + k / (G / XCDS), workgroups being dealt to the
    // XCDs in turn
    const int64_t per_xcd = G / XCDS;
    std::vector<const std::vector<XSeg> *> by_wg((size_t)G);
    for (int64_t k = 0; k < G; ++k) by_wg[(size_t)((k % per_xcd) * XCDS + k / per_xcd)] = &logical[(size_t)k];
    Plan plan;
    plan.wg_off.assign((size_t)G + 1, 0);
    for (int64_t w = 0; w < G; ++w) {
        for (const XSeg &sg : *by_wg[(size_t)w]) {
            Piece pc;
            pc.job = 0;
            pc.tile = units[(size_t)sg.u].first | (units[(size_t)sg.u].second << 16);
            pc.t0 = (int32_t)(sg.s0 * STAGE);
            pc.t1_atomic = (int32_t)std::min<int64_t>(sg.s1 * STAGE, job.t);
            if (pieces_of[(size_t)sg.u] > 1) pc.t1_atomic |= (int32_t)0x80000000u;
            plan.pieces.push_back(pc);
            plan.piece_wg.push_back((int32_t)w);
        }
        plan.wg_off[(size_t)w + 1] = (int32_t)plan.pieces.size();
    }
    // every physical id up to G - 1 is launched (workgroups without pieces
    // return at once), so that the XCD placement holds
    plan.grid = (int32_t)G;
    *out = std::move(plan);
    return true;
}

namespace {

// Time model of a shape's kernel (microseconds).  Up to one unit per
// workgroup: per stage, and more per stage past `long_from` of them on a
// workgroup; prologue and flush of a piece that owns its unit; prologue of a
// shared one; and the share of one shared piece in the atomic flushes, which
// all workgroups' together move at about 2 TB/s.
struct ShapeCost {
    TileShape shape;
    double stage, owned, prologue, shared;
    double long_from, long_more;
    double batch_long_from, batch_long_more;   // the same for the jobs of a batch
    // One job of more units than compute units, whose flushes move tens to
    // hundreds of MB: whole units in rounds (launch, a stage of every round, a
    // round, the flushes per unit and compute unit), or the work in equal
    // shares (launch with the shared pieces' atomics, stage, flushes, and more
    // per stage past share_long_from).
    double rounds_launch, round_stage, round, round_flush;
    double shares_launch, share_stage, share_flush, share_long_from, share_long;
};
constexpr double LAUNCH_US = 4.0;
constexpr ShapeCost SHAPE_COSTS[] = {
    {TileShape::Wide, 1.1, 13.0, 5.0, 0.13, 1e9, 0.0, 1e9, 0.0, 1.0, 1.1, 3.9, 18.0, 41.0, 0.84, 16.5, 60, 0.45},
    {TileShape::Tile, 0.62, 8.0, 3.0, 0.065, 100, 0.04, 100, 0.04, 2.0, 0.59, 8.0, 5.4, 23.0, 0.5, 11.3, 100, 0.2},
    {TileShape::Region, 0.20, 4.3, 3.0, 0.016, 160, 0.02, 60, 0.20, 2.0, 0.24, 5.7, 0.0, 12.5, 0.2, 4.6, 100, 0.2}};

// Units of one job (the length of plan_units).
int64_t shape_units(int32_t n, TileShape shape)
{
    const int64_t nt = n_tiles_side(n);
    if (shape == TileShape::Region) return tri64((n + REGION - 1) / REGION);
    if (shape == TileShape::Tile) return tri64(nt);
    int64_t units = 0;
    for (int64_t i = 0; i < nt; ++i) units += (nt + 1) / 2 - i / 2;
    return units;
}

// The stages of one workgroup.  They take longer where the work is long: the
// clock settles under the load, and where the workgroups walk time apart
// from each other their operands no longer meet in the L2s.
double stages_us(const ShapeCost &c, double stages, bool batch = false)
{
    const double from = batch ? c.batch_long_from : c.long_from, more = batch ? c.batch_long_more : c.long_more;
    return stages * c.stage + std::max(0.0, stages - from) * more;
}

// Whether the planner's costs (in stages) lead it to give every unit to one
// workgroup, `rounds` of them each, rather than to equal shares.
bool whole_units(const ShapeCost &c, int64_t units, int64_t longest, int64_t stages, int cus)
{
    const int64_t rounds = (units + cus - 1) / cus, ovh = piece_overhead(c.shape);
    return rounds * (longest + ovh) * cus <= stages + ovh * (units + cus);
}

}  // namespace

DmaChoice choose_dma(int32_t n, int64_t t, int cus, int min_stages, TileShape only)
{
    const int64_t ns = std::max<int64_t>(1, (t + STAGE - 1) / STAGE);
    DmaChoice best{TileShape::Wide, 0};
    double best_us = -1.0;
    auto consider = [&](TileShape shape, int64_t wgs, double us) {
        if (best_us < 0.0 || us < best_us) {
            best_us = us;
            best = DmaChoice{shape, (int)wgs};
        }
    };
    for (const ShapeCost &c : SHAPE_COSTS) {
        if (only != TileShape::Square && c.shape != only) continue;
        const int64_t units = shape_units(n, c.shape);
        const double s = (double)units * (double)ns / cus, per_cu = (double)units / cus;
        if (units > cus) {
            const double rounds = (double)((units + cus - 1) / cus);
            consider(c.shape, 0,
                     whole_units(c, units, ns, units * ns, cus)
                         ? c.rounds_launch + rounds * ((double)ns * c.round_stage + c.round) + c.round_flush * per_cu
                         : c.shares_launch + s * c.share_stage + c.share_flush * per_cu +
                               std::max(0.0, s - c.share_long_from) * c.share_long);
            continue;
        }
        // every unit whole, or in k equal pieces, whose workgroups walk the
        // same time together (the region kernel's stages then stay at their
        // price however many there are: N = 1408, 253 whole regions, T = 4096
        // 21 us, 8192 33, 16384 58)
        for (int64_t k = 1; k * units <= cus && k <= MAX_UNIT_SPLIT && (k == 1 || k * min_stages <= ns); ++k) {
            const double st = (double)((ns + k - 1) / k);
            const double run = c.shape == TileShape::Region ? st * c.stage : stages_us(c, st);
            consider(c.shape, k * units,
                     LAUNCH_US + run + (k == 1 ? c.owned : c.prologue + (double)(k * units) * c.shared));
        }
        // the work in equal shares of every workgroup; a job of fewer units
        // than compute units has been seen above unless it is long enough
        if (units * MAX_UNIT_SPLIT >= cus && units * ns >= (int64_t)cus * min_stages)
            consider(c.shape, 0, LAUNCH_US + stages_us(c, s) + c.owned * per_cu + cus * c.shared);
    }
    return best;
}

TileShape choose_dma_batch(const PlanJob *jobs, int n_jobs, int cus)
{
    TileShape best = TileShape::Wide;
    double best_us = -1.0;
    for (const ShapeCost &c : SHAPE_COSTS) {
        int64_t units = 0, stages = 0, longest = 0;
        for (int k = 0; k < n_jobs; ++k) {
            const int64_t ns = (jobs[k].t + STAGE - 1) / STAGE, u = shape_units(jobs[k].n, c.shape);
            units += u;
            stages += u * ns;
            longest = std::max(longest, ns);
        }
        // (Wide comes first: its count decides for the others)
        if (c.shape == TileShape::Wide && units > cus) return TileShape::Wide;
        if (c.shape == TileShape::Region && 4 * units > 5 * (int64_t)cus) continue;
        double us;
        if (whole_units(c, units, longest, stages, cus)) {
            const double k = (double)((units + cus - 1) / cus);
            // a second region's flush also waits for the first one's stores
            const double owned = c.shape == TileShape::Region && k > 1 ? 1.5 * c.owned : c.owned;
            us = stages_us(c, k * (double)longest, true) + k * owned;
        } else {
            us = stages_us(c, (double)stages / cus, true) + c.prologue + c.owned * (double)units / cus + cus * c.shared;
        }
        // the wide kernel unless another is clearly ahead
        if (c.shape != TileShape::Wide) us *= 1.05;
        if (best_us < 0.0 || us < best_us) {
            best_us = us;
            best = c.shape;
        }
    }
    return best;
}

SinglePlanArgs single_plan(int32_t n, int64_t t, TileShape shape, int max_wgs, int min_stages, int64_t *n_pieces,
                          int64_t *used)
{
    SinglePlanArgs a;
    a.n = n;
    a.t = t;
    a.wide = shape == TileShape::Wide ? 1 : 0;
    a.overhead = piece_overhead(shape) * STAGE_COST;
    a.cap = shape == TileShape::Wide ? MAX_PIECE_STAGES_WIDE : MAX_PIECE_STAGES;
    if (min_stages < 1) min_stages = 1;
    if (max_wgs < 1) max_wgs = 1;
    const int64_t units = single_units(a);
    const int64_t total = units * single_stages(a);
    a.grid = std::max<int64_t>(
        1, std::min<int64_t>({(int64_t)max_wgs, std::max<int64_t>((total + min_stages - 1) / min_stages, units),
                              units * MAX_UNIT_SPLIT}));
    auto none = [](int64_t, int32_t, int32_t, int64_t, int64_t, int64_t) {};
    // the budget search of make_plan, over the same unit order (total
    // stages at full cost bound the total cost from above)
    int64_t lo = a.overhead + STAGE_COST, hi = a.overhead + total * STAGE_COST + 1;
    hi = std::max(hi, (total * STAGE_COST + a.grid - 1) / a.grid + a.overhead * (units + 1) + 1);
    a.budget = hi;
    while (single_fill(a, none) > a.grid) a.budget = (hi *= 2);
    while (lo < hi) {
        a.budget = lo + (hi - lo) / 2;
        if (single_fill(a, none) <= a.grid)
            hi = a.budget;
        else
            lo = a.budget + 1;
    }
    a.budget = lo;
    int64_t np = 0;
    *used = single_fill(a, [&np](int64_t, int32_t, int32_t, int64_t, int64_t, int64_t) { ++np; });
    *n_pieces = np;
    return a;
}

}  // namespace xeng
