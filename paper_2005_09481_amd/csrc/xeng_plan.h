// Work decomposition of a (batched) correlation into per-workgroup pieces.
// Host only; no HIP dependency, so it is unit-testable without a GPU.
#pragma once

#include <stdint.h>
#include <utility>
#include <vector>

#include "xeng_internal.h"
#include "xeng_plan_single.h"

namespace xeng {

struct PlanJob {
    int32_t n;      // inputs
    int64_t t;      // samples
};

struct Plan {
    std::vector<Piece> pieces;      // grouped by workgroup
    std::vector<int32_t> wg_off;    // size grid + 1
    std::vector<int32_t> piece_wg;  // workgroup of each piece (for inspection)
    int32_t grid = 0;               // workgroups to launch
};

// Split the upper-triangle tiles of every job, each over its samples in
// STAGE-sample stages, into `max_wgs` (or fewer) nearly equal contiguous
// ranges of a linear (job, tile, stage) order: the stream-K decomposition.
// A tile cut into several pieces is marked atomic.  Every (i <= j, t) of
// every job is covered by exactly one piece.
//
// Square and Tile: units are the tiles (ti <= tj) of 128 x 128.  Region: the
// 64 x 64 regions.  Wide: units are
// workgroup tiles (I, J2) of 128 rows x 256 columns, i.e. accumulator tiles
// (I, 2 J2) and (I, 2 J2 + 1), for every I <= 2 J2 + 1 (for I = 2 J2 + 1
// the left tile lies below the diagonal: the DMA kernel leaves it out).
// `cap` (stages), when positive, replaces the shape's longest piece.
// `min_stages` limits how far units are cut, never their number: a unit of
// fewer stages is still a workgroup's own where there are workgroups left
// (N = 2048, T = 64: 72 windows of one stage on 72 workgroups 14.5 us, on the
// 18 that pieces of four stages would make 44).
Plan make_plan(const PlanJob *jobs, int n_jobs, int max_wgs, int min_stages,
               TileShape shape = TileShape::Square, int64_t cap = 0);

// Units of one job in the plan's order: pairs (row index, column index)
// in the shape's own units.
std::vector<std::pair<int, int>> plan_units(int n, TileShape shape);

// XCD-aware, time-aligned decomposition of ONE job.  MI355X deals the
// workgroups of a launch to its 8 XCDs in turn (workgroup w on XCD w % 8),
// and each XCD has its own L2.  The job's units, in Morton order of their
// (row, column) tile coordinates, are cut into full time segments of L
// stages (L about the balanced share, total / grid) plus a tail each;
// logical workgroup k takes the k-th full segment in (time window, unit)
// order, and the tails are spread over the remaining workgroups by the
// stream-K fill.  Logical workgroups 32 x .. 32 x + 31 are placed on XCD x,
// so each XCD's workgroups work on one time window over a compact block of
// units and share those input rows and columns in its L2.  Every workgroup
// has one piece, or a few for the tails, as in the linear plan.  Returns
// false (nothing written) for a grid that is not a multiple of 8 or a job
// too short for one segment of XCD_MIN_SEGMENT stages per workgroup.  `cap`
// as in make_plan.  False as well where the linear order is clearly better.
constexpr int XCDS = 8;
constexpr int64_t XCD_MIN_SEGMENT = 32;
bool make_plan_xcd(const PlanJob &job, int max_wgs, TileShape shape, Plan *out, int64_t cap = 0);

// Stage-equivalents charged per piece (prologue and flush) by the planners.
int64_t piece_overhead(TileShape shape);
// Longest piece of a shape's kernel, in stages: its int32 register sums
// stay exact (the general kernel's B operands carry 16x the samples, the
// DMA and narrow kernels' A and B operands both do).
int64_t piece_cap(TileShape shape);

// The shape of one job that the DMA kernels read (N > NARROW_MAX_N), and the
// workgroups to plan it for (0: one per compute unit): the smallest of the
// modelled times of the wide, tile and region kernels, each with its units
// whole, in equal pieces, or in equal shares of every workgroup, and with more
// units than compute units in rounds of whole units or in shares, as the
// planner splits them.  The model's constants come from sweeps of N from 80 to
// 8192 and T from 1 to 131072 with every kernel; over those 400 sizes the
// choice takes 0.5 % longer than the fastest of them in the mean.
// Where it draws the lines, with both sides measured (correlation alone, us):
//   N = 1024, T = 16384 region 38, tile 46, wide 60; T = 32768 74, 68, 81
//   N = 1408, T = 8192 whole regions 33, tile 44; T = 32768 tile 106, region 110
//   N = 1536, T = 256 whole tiles 12, region 17; T = 2048 26, 22
//   N = 2048, T = 512 whole tiles 16, wide 21, region 26; T = 2048 28, 40, 33;
//     T = 3000 tile 42, region 39; T = 4096 44, 50; T = 16384 tile 107, wide 120
//   N = 3072, T = 512 whole windows 25, tile 44; T = 20000 wide 259, tile 268
//   N = 4096, T = 64 whole windows 30, tile 35, region 54; T = 4096 tile 118,
//     wide 128; T = 12000 288, 281
//   N = 5008, T = 512 whole windows 53, tile 76; N = 6000, T = 2048 wide 138,
//     tile 155
// What decides between whole units and shares is the flush: shares of a tile
// meet on the same words, and all atomic flushes together ran at some 2 TB/s
// whatever their order and placement (N = 2048, T = 2048: 28 us in 136 whole
// tiles, 36 in 256 shares).
struct DmaChoice {
    TileShape shape;
    int wgs;
};
// `only`, unless Square: the best split of that shape alone.
DmaChoice choose_dma(int32_t n, int64_t t, int cus, int min_stages, TileShape only = TileShape::Square);

// The same choice for the jobs of a batch that one DMA launch takes, planned
// over every compute unit: the modelled time of the planner's two regimes,
// every unit whole or all work in equal shares.  From more wide windows than
// compute units on, the wide kernel flushes them whole and reads least; the
// region kernel reads most, and is left out past a quarter more regions than
// compute units.  Correlations of T samples with the launch and the exports,
// wide / tile / region, us: 4 jobs of N = 512, T to 4096 51 / 45 / 33; 16 of
// N = 512, T to 1024 60 / 46 / 51; 8 of N = 1024, T to 4096 87 / 70 / 127; 8 of
// N = 2048, T to 4096 (576 windows) 198 / 222 / 433.  Long batches leave the
// region kernel, whose workgroups then read different times of different jobs:
// 16 of N = 256, T = 6000 60 / 53 / 49, T = 12000 70 / 62 / 73, T = 32768 103 /
// 94 / 150; 2 of N = 640, T = 12000 63 / 55 / 44, T = 32768 84 / 80 / 123.
TileShape choose_dma_batch(const PlanJob *jobs, int n_jobs, int cus);

// Plan parameters of one job as make_plan would choose them (grid and
// budget), for the container-free planner of xeng_plan_single.h; also the
// number of pieces and of workgroups used.  Host only, allocates nothing.
SinglePlanArgs single_plan(int32_t n, int64_t t, TileShape shape, int max_wgs, int min_stages, int64_t *n_pieces,
                          int64_t *used);

}  // namespace xeng
