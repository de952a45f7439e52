// gfx950 correlation kernel that splits time over a workgroup's waves:
// 64 x 64 regions of the upper triangle, for jobs too small to fill the
// chip with the wide kernel's 128 x 256 tiles.
//
// The product, operand forms, samples in LDS and slot layout are the wide
// kernel's (see xeng_kernel_dma.hip); the split of the work is the narrow
// kernel's.  The wide kernel gives a tile's 256 KiB of sums to one
// workgroup, so a job of few tiles is cut into short pieces that each flush
// all of them: at N = 512, T = 8192 some hundred workgroups added 25 MB with
// atomics on 1.3 MB of addresses, which took longer than their products.
// Here a workgroup takes one 64 x 64 region, its eight waves every eighth
// half stage (32 samples) of the piece, and their sums meet in LDS before
// they leave the CU: 32 KiB per piece to flush, and no barrier in the main
// loop.  The price is operand traffic (128 bytes per 64 x 64 products and
// sample, 2.7 times the wide kernel's), so the wide kernel stays ahead where
// a job has work enough for its tiles.  Correlation alone, before (wide
// kernel) and after: N = 512, T = 8192 23.8 -> 13.6 us, N = 1024, T = 2048
// 30.5 -> 12.3, N = 512, T = 65536 72 -> 36, N = 1536, T = 4096 53 -> 31.
// What bounds it: at small T the launch, the first loads' latency, the
// reduction and the flush (13.6 us without, 9.7 us with the flush left out
// at N = 512, T = 8192); at large T the operand path (N = 1024, T = 16384
// 40 us, 31 us with the loop's loads left out, 34 us with its MFMAs left out).
//
//   * global -> LDS by DMA into a ring of four half stages private to the
//     wave, four issued ahead of their use (128 KiB in flight per CU);
//     regions on the diagonal load their 64 inputs once;
//   * LDS -> registers by transposed reads, unpacked one k-step ahead of the
//     MFMAs, as in the wide kernel, ordered by the wave's own waits alone;
//   * end of a piece: LDS atomic adds into one 32 KiB array, then every wave
//     flushes its share of the region's rows.
#include <hip/hip_runtime.h>

#include "xeng_dma_ops.h"

namespace xeng {
namespace region {

using namespace dma;

constexpr int WAVES = 8;
constexpr int WIDTH = 64;                   // inputs of a region's side
constexpr int HALF = 32;                    // samples per half stage
constexpr int SIDE = HALF * WIDTH;          // 2 KiB: one side's samples of a half stage
constexpr int SLOT = 2 * SIDE;
constexpr int NSLOT = 4;
constexpr int RING = NSLOT * SLOT;          // 16 KiB per wave
constexpr int SUM_OFFSET = WAVES * RING;
constexpr int SUM_I32 = 4 * 2 * 16 * 64;    // [block][re, im][register][lane]
constexpr int LDS_BYTES = SUM_OFFSET + SUM_I32 * 4;   // 160 KiB
static_assert(LDS_BYTES <= 160 * 1024, "the CU's LDS");

// Instruction mix of a k-step (see xeng_dma_ops.h)
struct L {
    static constexpr int PITCH_A = WIDTH, PITCH_B = WIDTH;
    static constexpr int BW = 2;
    static constexpr int MFMA_PER_K = 8;
    static constexpr int READS_PER_K = 4;
    static constexpr int VALU_PER_MFMA = 4;
};

// Loads of half stage `h` of this wave into its ring.  A DMA instruction
// fills 1 KiB, 16 rows of one side (the job's last 16 inputs for a chunk at
// or past n: what they add reaches only pairs with i or j >= n, which are
// never exported).  Rows at or past t1 read the zero-sample
// buffer, so every half stage is whole and the count of loads in flight
// constant.
template <int K>
__device__ __forceinline__ void issue_half(uint32_t ring, const uint8_t *samples, const uint8_t *zeros, int64_t stride,
                                           const uint32_t (&off)[K], int ts, int t1, int slot, int lane)
{
    uint32_t lds[K];
#pragma unroll
    for (int k = 0; k < K; ++k) lds[k] = ring + slot * SLOT + 1024 * k;
    if (ts + HALF <= t1) {
        dma16_s_stage<K>(samples + (int64_t)ts * stride, off, lds);
    } else {
        const int r = dma_row<WIDTH>(lane);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool ok = ts + 16 * (k & 1) + r < t1;
            dma16_v(ok ? samples + (int64_t)ts * stride + off[k] : zeros, lds[k]);
        }
    }
}

// This wave's half stages of a piece: wave + 8 h, h = 0, 1, ...  Entering
// iteration h, the unpacked operands of (h, k-step 0) and the raw data of
// (h, 1) are in registers, so the slot of h is free for half stage h + 4.
template <bool RE_LOW, bool DIAG>
__device__ __forceinline__ void run_piece(Acc<L, false> &acc, uint32_t ring, const JobDesc &jd, const uint8_t *zeros,
                                          int row0, int col0, int t0, int t1, int wave, int lane)
{
    constexpr int K = DIAG ? 2 : 4;   // DMA instructions per half stage
    const int nh = (t1 - t0 + HALF - 1) / HALF;
    const int m = wave < nh ? (nh - wave + WAVES - 1) / WAVES : 0;
    if (m == 0) return;
    uint32_t off[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int row = 16 * (k & 1) + dma_row<WIDTH>(lane);
        const int in = (k < 2 ? row0 : col0) + 16 * dma_chunk<WIDTH>(0, lane);
        off[k] = (uint32_t)((int64_t)row * jd.stride) + (uint32_t)min(in, jd.n - 16);
    }
    auto issue = [&](int h, int slot) {
        issue_half<K>(ring, jd.samples, zeros, jd.stride, off, t0 + HALF * (wave + WAVES * h), t1, slot, lane);
    };
    ReadLane<L> rl;
    read_lane_setup<L>(rl, 0, 0, DIAG ? 0 : SIDE, lane);

    // nothing else in flight: the vmcnt waits then count DMA only
    __builtin_amdgcn_s_waitcnt(XENG_VMCNT(0));
#pragma unroll
    for (int h = 0; h < NSLOT; ++h) issue(h, h);
    __builtin_amdgcn_s_waitcnt(XENG_VMCNT((NSLOT - 1) * K));
    asm volatile("" ::: "memory");
    Raw<L> r0, r1;
    Ops<L> u0, u1;
    read_k<L>(r0, ring, rl, 0);
    read_k<L>(r1, ring, rl, 1);
    unpack_k<L, RE_LOW, false, false>(u0, r0);
    int cur = 0;
    for (int h = 0; h < m; ++h) {
        const int nxt = (cur + 1) & (NSLOT - 1);
        // the reads of half stage h are done: its slot takes h + 4
        __builtin_amdgcn_s_waitcnt(XENG_LGKMCNT0);
        asm volatile("" ::: "memory");
        issue(h + NSLOT, cur);
        // half stage h + 1 has landed (three newer ones in flight)
        __builtin_amdgcn_s_waitcnt(XENG_VMCNT((NSLOT - 1) * K));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        read_k<L>(r0, ring + nxt * SLOT, rl, 0);
        unpack_k<L, RE_LOW, false, false>(u1, r1);
        mfma_k<L, DIAG>(acc, u0);
        kstep_schedule<L, DIAG>();
        __builtin_amdgcn_sched_barrier(0);
        read_k<L>(r1, ring + nxt * SLOT, rl, 1);
        unpack_k<L, RE_LOW, false, false>(u0, r0);
        mfma_k<L, DIAG>(acc, u1);
        kstep_schedule<L, DIAG>();
        __builtin_amdgcn_sched_barrier(0);
        cur = nxt;
    }
    // the next piece's loads reuse the slots
    __builtin_amdgcn_s_waitcnt(XENG_VMCNT(0));
    __builtin_amdgcn_s_waitcnt(XENG_LGKMCNT0);
    asm volatile("" ::: "memory");
}

// Row `q` of the region's sums in the order they are flushed: register
// q % 16 of block q / 16 of the blocks (0,0), (0,1), (1,1) and, off the
// diagonal, (1,0).
__device__ __forceinline__ constexpr int blk_a(int b) { return b >> 1; }
__device__ __forceinline__ constexpr int blk_b(int b) { return b == 1 || b == 2 ? 1 : 0; }

// A wave's partial sums into the workgroup's by LDS atomic adds.
template <bool DIAG> __device__ __forceinline__ void add_to_sum(int32_t *sum, const Acc<L, false> &acc, int lane)
{
#pragma unroll
    for (int b = 0; b < (DIAG ? 3 : 4); ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            atomicAdd(&sum[((2 * b) * 16 + r) * 64 + lane], acc.re[blk_a(b)][blk_b(b)][r]);
            atomicAdd(&sum[((2 * b + 1) * 16 + r) * 64 + lane], acc.im[blk_a(b)][blk_b(b)][r]);
        }
}

// This wave's share of the region's rows to the slot; the old values of a
// read-modify-write are all loaded before any is stored back.
template <bool DIAG>
__device__ __forceinline__ void flush_rows(const JobDesc &jd, const int32_t *sum, int ri, int rj, bool atomic,
                                           int wave, int lane)
{
    constexpr int ROWS = (DIAG ? 3 : 4) * 16 / WAVES;
    const int ti = ri >> 1, tj = rj >> 1;
    const int64_t tile = (int64_t)ti * jd.nt - (int64_t)ti * (ti - 1) / 2 + (tj - ti);
    gw64 *tb = (gw64 *)jd.acc + tile * TILE_W + lane;
    gw64 *w[ROWS];
    uint64_t v[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const int q = wave * ROWS + i, b = q / 16, r = q % 16;
        w[i] = tb + ((2 * (ri & 1) + blk_a(b)) * BLKS + 2 * (rj & 1) + blk_b(b)) * BLOCK_W + r * 64;
        v[i] = pack_pair(sum[((2 * b) * 16 + r) * 64 + lane] >> 8, sum[((2 * b + 1) * 16 + r) * 64 + lane] >> 8);
    }
    // the diagonal's imaginary sums are the slot's biases: waves 0 and 1
    // take blocks (0, 0) and (1, 1), one lane per input
    if (DIAG && wave < 2 && jd.bias != nullptr) {
        const int b = 2 * wave, r = diag_reg(lane), j = WIDTH * ri + BLK * wave + (lane & 31);
        if (r >= 0 && j < jd.n)
            __hip_atomic_fetch_add(jd.bias + j, sum[((2 * b + 1) * 16 + r) * 64 + lane] >> 8, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
    if (atomic) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
            __hip_atomic_fetch_add(w[i], v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    uint64_t old[ROWS];
    const bool fresh = (jd.flags & JOB_FRESH) != 0;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) old[i] = fresh ? 0 : *w[i];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) *w[i] = old[i] + v[i];
}

// Persistent kernel: workgroup w runs pieces [wg_off[w], wg_off[w+1]); a
// piece's tile field holds the region (I, J): inputs 64 I.. against 64 J..
__global__ __launch_bounds__(64 * WAVES, 1) void xcorr_region(KernelArgs args)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    // a prepared batch's device guard refused this launch
    if (args.skip != nullptr && *args.skip != 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t ring = (uint32_t)__builtin_amdgcn_readfirstlane(
                              (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds) +
                          wave * RING;
    int32_t *sum = reinterpret_cast<int32_t *>(lds + SUM_OFFSET);
    const uint8_t *zeros = uniform(args.zeros);
    // clock probe (measurement only): workgroup 0's start and end
    const bool stamp = args.clock != nullptr && blockIdx.x == 0 && threadIdx.x == 0;
    if (stamp) {
        args.clock[0] = (int64_t)__builtin_amdgcn_s_memtime();
        args.clock[1] = (int64_t)__builtin_amdgcn_s_memrealtime();
    }
    const int p_begin = args.wg_off[blockIdx.x], p_end = args.wg_off[blockIdx.x + 1];
    for (int pi = p_begin; pi < p_end; ++pi) {
        const Piece pce = args.pieces[pi];
        JobDesc jd = args.jobs ? args.jobs[__builtin_amdgcn_readfirstlane(pce.job)] : args.job0;
        jd.samples = uniform(jd.samples);
        jd.acc = uniform(jd.acc);
        jd.bias = uniform(jd.bias);
        jd.stride = uniform(jd.stride);
        jd.n = __builtin_amdgcn_readfirstlane(jd.n);
        jd.nt = __builtin_amdgcn_readfirstlane(jd.nt);
        jd.flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)jd.flags);
        const int tile = __builtin_amdgcn_readfirstlane(pce.tile);
        const int ri = tile & 0xFFFF, rj = (tile >> 16) & 0xFFFF;
        const int t1a = __builtin_amdgcn_readfirstlane(pce.t1_atomic);
        const bool atomic = t1a < 0;
        const int t0 = __builtin_amdgcn_readfirstlane(pce.t0), t1 = t1a & 0x7FFFFFFF;
        // the workgroup's sums start at zero (the barrier at the end of the
        // previous piece: its flush has read them)
        for (int i = threadIdx.x; i < SUM_I32 / 4; i += 64 * WAVES)
            reinterpret_cast<v4i *>(sum)[i] = v4i{0, 0, 0, 0};
        Acc<L, false> acc;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc.re[a][b][r] = 0;
                    acc.im[a][b][r] = 0;
                }
        const bool re_low = (jd.flags & JOB_RE_LOW) != 0, diag = ri == rj;
        const int row0 = WIDTH * ri, col0 = WIDTH * rj;
        if (diag && re_low)
            run_piece<true, true>(acc, ring, jd, zeros, row0, col0, t0, t1, wave, lane);
        else if (diag)
            run_piece<false, true>(acc, ring, jd, zeros, row0, col0, t0, t1, wave, lane);
        else if (re_low)
            run_piece<true, false>(acc, ring, jd, zeros, row0, col0, t0, t1, wave, lane);
        else
            run_piece<false, false>(acc, ring, jd, zeros, row0, col0, t0, t1, wave, lane);
        __syncthreads();   // the sums are zeroed
        if (diag) add_to_sum<true>(sum, acc, lane);
        else add_to_sum<false>(sum, acc, lane);
        __syncthreads();   // every wave's partial sums are in
        if (diag) flush_rows<true>(jd, sum, ri, rj, atomic, wave, lane);
        else flush_rows<false>(jd, sum, ri, rj, atomic, wave, lane);
        __syncthreads();   // the flush has read the sums
    }
    if (stamp) {
        args.clock[2] = (int64_t)__builtin_amdgcn_s_memtime();
        args.clock[3] = (int64_t)__builtin_amdgcn_s_memrealtime();
    }
}

}  // namespace region

// Once per device, before any launch: the kernel's LDS exceeds the default
// dynamic-LDS limit.
hipError_t init_region_kernel()
{
    return hipFuncSetAttribute((const void *)region::xcorr_region, hipFuncAttributeMaxDynamicSharedMemorySize,
                               region::LDS_BYTES);
}

hipError_t launch_correlate_region(const KernelArgs &a, int grid, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(region::xcorr_region, dim3(grid), dim3(64 * region::WAVES), region::LDS_BYTES, stream, a);
    return hipGetLastError();
}

}  // namespace xeng
