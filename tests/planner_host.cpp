// C entry points over the planner (csrc/xeng_plan.cpp) for tests on the CPU.
#include <chrono>

#include "xeng_plan.h"

using namespace xeng;

namespace {
std::vector<PlanJob> make_jobs(const int32_t *n, const int64_t *t, int32_t count)
{
    std::vector<PlanJob> jobs((size_t)count);
    for (int32_t k = 0; k < count; ++k) jobs[(size_t)k] = PlanJob{n[k], t[k]};
    return jobs;
}
}  // namespace

extern "C" {

// The pieces of a plan as rows (job, i, j, t0, t1, atomic, workgroup); xcd:
// the XCD-aware plan of one job.  Returns the number of pieces (at most `cap`
// are written), or -1 where that plan does not apply.
int64_t host_plan(const int32_t *n, const int64_t *t, int32_t count, int32_t wgs, int32_t min_stages, int32_t shape,
                  int32_t xcd, int64_t piece_cap, int64_t *out, int64_t cap)
{
    const std::vector<PlanJob> jobs = make_jobs(n, t, count);
    Plan p;
    if (xcd) {
        if (!make_plan_xcd(jobs[0], wgs, (TileShape)shape, &p, piece_cap)) return -1;
    } else {
        p = make_plan(jobs.data(), count, wgs, min_stages, (TileShape)shape, piece_cap);
    }
    for (size_t k = 0; k < p.pieces.size() && (int64_t)k < cap; ++k) {
        const Piece &q = p.pieces[k];
        const int64_t row[7] = {q.job, q.tile & 0xFFFF, (q.tile >> 16) & 0xFFFF, q.t0, q.t1_atomic & 0x7FFFFFFF,
                                q.t1_atomic < 0, p.piece_wg[k]};
        std::copy(row, row + 7, out + 7 * k);
    }
    return (int64_t)p.pieces.size();
}

// The shape and workgroups (0: one per compute unit) a single job takes, and
// the shape a batch takes.
int32_t host_choose(int32_t n, int64_t t, int32_t cus, int32_t min_stages, int32_t *wgs)
{
    const DmaChoice c = choose_dma(n, t, cus, min_stages);
    *wgs = c.wgs;
    return (int32_t)c.shape;
}
int32_t host_choose_batch(const int32_t *n, const int64_t *t, int32_t count, int32_t cus)
{
    return (int32_t)choose_dma_batch(make_jobs(n, t, count).data(), count, cus);
}

// Microseconds to plan one job, the best of `reps`.
double host_plan_us(int32_t n, int64_t t, int32_t wgs, int32_t shape, int32_t reps)
{
    const PlanJob job{n, t};
    double best = 1e30;
    for (int32_t k = 0; k < reps; ++k) {
        const auto a = std::chrono::steady_clock::now();
        Plan p;
        if (!make_plan_xcd(job, wgs, (TileShape)shape, &p)) p = make_plan(&job, 1, wgs, 4, (TileShape)shape);
        best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - a).count());
    }
    return best;
}
}
