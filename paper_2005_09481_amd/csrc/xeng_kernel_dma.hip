// gfx950 correlation kernel for 16-byte-aligned sample arrays (base and row
// stride) of N a multiple of 16.
//
// Same product as the general kernel -- for a tile of the upper triangle,
//   V_ij = sum_t x_i(t) conj(x_j(t))                      (Sec. 2.2, eta)
// on v_mfma_i32_32x32x32_i8 -- but the packed samples never leave their
// 4-bit form in shared memory:
//   * global -> LDS by DMA (global_load_lds_dwordx4): 16 bytes per lane, no
//     registers and no instructions beyond the load itself, into a ring of
//     NSLOT 64-sample stages, AHEAD of them issued before they are needed;
//   * LDS -> registers by transposed reads (ds_read_b64_tr_b8): a 16-lane
//     group reads 8 time rows x 16 inputs and each lane receives the 8
//     samples of one input -- exactly one lane's share of an MFMA operand;
//   * the nibble unpack to int8 happens in registers, one k-step ahead of
//     the MFMAs that use it.
//
// Operands.  With R, I the 4-bit parts of a sample (two's complement values
// in [-8, 7]) and ~R = -R - 1:
//   B (columns j)      = [16 R_j | 16 I_j]
//   A, real part       = [16 R_i | 16 I_i]   -> 256 (R_i R_j + I_i I_j)
//   A, imaginary part  = [16 I_i | 16 ~R_i]  -> 256 (I_i R_j - R_i I_j - I_j)
// Every byte is a 4-bit value in the high half of a byte, made from the
// packed sample by one XOR and one AND (no sign extension), and ~R never
// overflows int8 where -R would (R = -8).  The imaginary accumulator thus
// holds Im V_ij - S_j with S_j = sum_t I_j(t); since Im V_jj = 0 its diagonal
// holds -S_j, which the waves on the diagonal also add to the slot's biases
// for the export to subtract.  The general kernel stores the same form.
//
// Workgroup tile: 128 rows (A) x 256 columns (B), NW waves in two rows of
// NW / 2; wave (wa, wb) computes rows 64wa..64wa+63 against 256 / (NW / 2)
// columns, i.e. 2 x BW MFMA blocks for both Re and Im.  Four waves (one per
// SIMD, 256 accumulator registers each) read the fewest operand bytes per
// MFMA; eight (two per SIMD, 128 each; the default) let one wave's MFMAs run
// while the other waits on LDS, a barrier or its DMA issue -- with eight,
// waves 0..3 (one per SIMD) issue all of a stage's DMA, since a burst of DMA
// instructions holds the issuing wave for tens of cycles per instruction.
// Regions and blocks wholly below the diagonal are not computed.
//
// The tile kernel (xcorr_tile) is the same code on 128 x 128 tiles: the wave
// of a 64 x 64 quarter is a pair, each taking every other 64 samples, whose
// sums meet in LDS at the end of a piece.  A workgroup then flushes half as
// much as the wide kernel's, no window has idle quarters left of the
// diagonal, and jobs of few tiles cut into fewer pieces; its operands cost a
// third more LDS DMA per product.  Correlation alone, wide kernel / tile
// kernel: N = 2048, T = 1024 42 / 20 us, T = 8192 79 / 67, T = 16384 121 /
// 112, T = 32768 202 / 204; N = 1008, T = 32768 79 / 69.  Bound at these
// sizes by its shared pieces' atomic flushes (N = 1024, T = 16384 46 us, 26
// with the flush left out), past T = 32768 by power, like the wide kernel.
//
// LDS stage layout: the A side, then the B side, each row-major by time row
// with the 16-byte chunks of a row permuted (swizzle, xeng_dma_ops.h).  Every
// DMA instruction then reads whole rows of its side, 128 or 256 contiguous
// bytes each, where the chunk-major layout used before (8 rows x 16 bytes
// contiguous in LDS) made neighbouring lanes read 16 bytes of different rows:
// a quarter as many cache accesses for the same bytes, and no bank conflict
// in either.  N = 2048, T = 32768: 213.5 -> 209.3 us a correlate + export
// step in alternating runs, N = 2048, T = 2048: 60.2 -> 57.1 us.
#include <hip/hip_runtime.h>

#include "xeng_dma_ops.h"

namespace xeng {
namespace dma {

constexpr int WA_ROWS = 128;            // A rows per workgroup tile
constexpr int A_STAGE = STAGE * WA_ROWS;    // 8 KB of packed samples
constexpr int DMA_A = A_STAGE / 1024;       // 1 KB DMA instructions per stage: 8

// The kernels' shapes: NWAVES waves in TIMES time groups over 128 x COLS
// inputs, a ring of SLOTS slots of a 64-sample stage per time group, DMA
// waves per time group issuing its loads.
template <int NWAVES, int TIMES, int COLS, int SLOTS, int DMA> struct Shape {
    static constexpr int NW = NWAVES;
    static constexpr int TG = TIMES;
    static constexpr int PITCH_A = WA_ROWS, PITCH_B = COLS;   // bytes per time row of a side in LDS
    static constexpr int WB_COLS = COLS;                     // B columns per workgroup tile
    static constexpr int TILES = COLS / TILE;                // accumulator tiles side by side
    static constexpr int B_STAGE = STAGE * COLS;
    static constexpr int GROUP = A_STAGE + B_STAGE;          // one time group's stage
    static constexpr int SLOT = TG * GROUP;
    static constexpr int ROWS = TG * STAGE;                  // samples per slot
    static constexpr int NSLOT = SLOTS;
    static constexpr int AHEAD = SLOTS - 1;                  // stages issued ahead
    static constexpr int LDS_BYTES = SLOTS * SLOT;
    static constexpr int DMA_B = B_STAGE / 1024;
    static constexpr int WB_WAVES = NWAVES / TG / 2;         // waves across the columns
    static constexpr int BW = COLS / BLK / WB_WAVES;         // B blocks per wave
    static constexpr int DMA_WAVES = DMA;
    static constexpr int DMA_PER_WAVE = (DMA_A + DMA_B) / DMA;
    static constexpr int MFMA_PER_K = 4 * BW;                // MFMAs per k-step
    static constexpr int READS_PER_K = 2 + BW;               // transposed reads per k-step
    static constexpr int VALU_PER_MFMA = BW == 4 ? 3 : 4;    // unpack share between MFMAs
};

// The wide kernel: 128 x 256, six 24 KB stages.  With eight waves, the DMA
// is left to one wave per SIMD (the other wave's MFMAs then run while the
// issuing wave waits to issue).
template <int NW> using Layout = Shape<NW, 1, 256, 6, 4>;
// The tile kernel: 128 x 128, four waves for each half of a 128-sample slot,
// five 32 KB slots (four measured the same).
using TileLayout = Shape<8, 2, 128, 5, 4>;

struct Tile {
    const uint8_t *samples;
    const uint8_t *zeros;   // 16 bytes of zero samples (0x88)
    int64_t stride;
    int n;                  // inputs (a multiple of 16)
    int row0, col0;         // first A input, first B input
    int t0, t1;             // samples, t0 that of the wave's time group
    int ns;                 // ring slots of the piece
};

// Geometry of DMA instruction `inst` (0..23, or 0..15 of the tile kernel) of
// a stage for this lane: its LDS offset in the slot (wave-uniform), the time
// row in the stage and the first of the 16 inputs the lane fetches.
// Instructions 0..7 fill 8 rows of the A side each, the others 4 rows (8 in
// the tile kernel) of the B side.
// A chunk at or past input n (the edge tiles of an N that is not a multiple
// of the tile) is fetched from inputs n - 16.. instead: every load stays in
// its row, and what lands in those rows or columns of the tile only reaches
// accumulator entries (i, j) with i or j >= n, which are never exported.
template <typename L>
__device__ __forceinline__ void dma_geom(int inst, int lane, int n, int row0, int col0, int &lds_off, int &t,
                                         int &in)
{
    lds_off = inst * 1024;   // the B side follows the A side
    if (inst < DMA_A) {
        const int first = inst * (1024 / L::PITCH_A);
        t = first + dma_row<L::PITCH_A>(lane);
        in = row0 + 16 * dma_chunk<L::PITCH_A>(first, lane);
    } else {
        const int first = (inst - DMA_A) * (1024 / L::PITCH_B);
        t = first + dma_row<L::PITCH_B>(lane);
        in = col0 + 16 * dma_chunk<L::PITCH_B>(first, lane);
    }
    in = min(in, n - 16);
}

// Index of this wave among the DMA-issuing waves, or -1.  Waves 0..3 sit on
// SIMDs 0..3 (waves of a workgroup are placed on the SIMDs in turn).
template <typename L> __device__ __forceinline__ int dma_wave(int wave)
{
    if (L::TG > 1) return wave % (L::NW / L::TG);
    if (L::DMA_WAVES == L::NW) return wave;
    return wave < 4 ? wave : -1;
}

// Per-lane byte offsets (row * stride + input) of this wave's DMA
// instructions from a stage's first row, fixed for a piece.
template <typename L> struct DmaLane {
    uint32_t off[L::DMA_PER_WAVE];
};

template <typename L>
__device__ __forceinline__ void dma_lane_setup(DmaLane<L> &dl, const Tile &tl, int wave, int lane)
{
#pragma unroll
    for (int k = 0; k < L::DMA_PER_WAVE; ++k) {
        int lds_off, t, in;
        dma_geom<L>(dma_wave<L>(wave) + L::DMA_WAVES * k, lane, tl.n, tl.row0, tl.col0, lds_off, t, in);
        dl.off[k] = (uint32_t)((int64_t)t * tl.stride) + (uint32_t)in;
    }
}

// This wave's share of one stage's DMA: instructions dw, dw + DMA_WAVES, ...
// of the 24, dw being the wave's index among the issuing waves (the others
// issue none).  Rows at or past t1 (the last, partial stage of a piece, and stages
// past its end, issued so that the count of loads in flight stays
// constant) are read from the zero-sample buffer, so that every stage the
// compute loop sees is whole.
template <typename L>
__device__ __forceinline__ void issue_stage(uint32_t slot_addr, const Tile &tl, const DmaLane<L> &dl, int stage,
                                            int wave, int lane)
{
    const int dw = dma_wave<L>(wave);
    if (dw < 0) return;
    const int ts = tl.t0 + stage * L::ROWS;
    if (ts + STAGE <= tl.t1) {
        const uint8_t *row = tl.samples + (int64_t)ts * tl.stride;
        uint32_t lds[L::DMA_PER_WAVE];
#pragma unroll
        for (int k = 0; k < L::DMA_PER_WAVE; ++k) {
            int lds_off, t, in;
            dma_geom<L>(dw + L::DMA_WAVES * k, lane, tl.n, tl.row0, tl.col0, lds_off, t, in);
            lds[k] = slot_addr + (uint32_t)lds_off;
        }
        dma16_s_stage<L::DMA_PER_WAVE>(row, dl.off, lds);
    } else {
#pragma unroll
        for (int k = 0; k < L::DMA_PER_WAVE; ++k) {
            int lds_off, t, in;
            dma_geom<L>(dw + L::DMA_WAVES * k, lane, tl.n, tl.row0, tl.col0, lds_off, t, in);
            const uint8_t *src =
                ts + t < tl.t1 ? tl.samples + (int64_t)(ts + t) * tl.stride + in : tl.zeros;
            dma16_v(src, slot_addr + (uint32_t)lds_off);
        }
    }
}

template <typename L>
__device__ __forceinline__ void wait_stage_and_sync()
{
    // this wave's loads of the next stage have landed (L::AHEAD - 1 newer
    // stages in flight) and its LDS reads are done; the barrier extends both
    // to the workgroup
    __builtin_amdgcn_s_waitcnt(XENG_VMCNT((L::AHEAD - 1) * L::DMA_PER_WAVE));
    __builtin_amdgcn_s_waitcnt(XENG_LGKMCNT0);
    __syncthreads();
}

// One piece, software-pipelined over its stages.  Entering iteration s, the
// unpacked operands of (s, k-step 0) and the raw data of (s, 1) are in
// registers; the iteration reads (s, 2), (s, 3), (s+1, 0), (s+1, 1) and
// unpacks one k-step ahead of its MFMAs.  The DMA of stage s + L::AHEAD goes
// into the slot stage s - 1 used, which every wave finished reading before
// the barrier of iteration s - 1; that barrier sits before the first read of
// stage s.  The last iteration's reads of "stage ns" touch a slot whose
// contents are never used.
//
// In the unsigned form the waves on the diagonal (DIAG) also add up the
// nibbles of their A rows into `ps`, at the k-steps they multiply (the
// reads of "stage ns" never count).
template <typename L, bool RE_LOW, bool DIAG, bool U, bool F>
__device__ __forceinline__ void run_piece(Acc<L, F> &acc, PreSum &ps, uint32_t ring, const Tile &tl, int wave,
                                          int lane, const ReadLane<L> &rl)
{
    constexpr bool SUMS = U && DIAG;
    const int ns = L::TG == 1 ? (tl.t1 - tl.t0 + STAGE - 1) / STAGE : tl.ns;
    DmaLane<L> dl;
    dma_lane_setup<L>(dl, tl, wave, lane);
    // nothing else in flight: the ring's vmcnt waits then count DMA only
    __builtin_amdgcn_s_waitcnt(XENG_VMCNT(0));
#pragma unroll
    for (int d = 0; d < L::AHEAD; ++d) issue_stage<L>(ring + d * L::SLOT, tl, dl, d, wave, lane);
    wait_stage_and_sync<L>();

    Raw<L> r0, r1;
    Ops<L> u0, u1;
    if constexpr (F) {
        // FP8: a k-step pair at a time.  Entering each half stage, the raw
        // data of its two k-steps is in r0, r1; both are unpacked, the next
        // pair's reads are issued, then the pair's products.
        {
            read_k<L>(r0, ring, rl, 0);
            read_k<L>(r1, ring, rl, 1);
        }
        int cur = 0;
        for (int s = 0; s < ns; ++s) {
            const int nxt = cur == L::NSLOT - 1 ? 0 : cur + 1;
            const int iss = cur == 0 ? L::NSLOT - 1 : cur - 1;
            issue_stage<L>(ring + iss * L::SLOT, tl, dl, s + L::AHEAD, wave, lane);
            __builtin_amdgcn_sched_barrier(0);
            // k-steps 0, 1
            unpack_k<L, RE_LOW, U, F>(u0, r0);
            unpack_k<L, RE_LOW, U, F>(u1, r1);
            read_k<L>(r0, ring + cur * L::SLOT, rl, 2);
            read_k<L>(r1, ring + cur * L::SLOT, rl, 3);
            mfma_pair<L, DIAG>(acc, u0, u1);
            if constexpr (SUMS) {
                presum_k<L>(ps, u0);
                presum_k<L>(ps, u1);
            }
            __builtin_amdgcn_sched_barrier(0);
            // k-steps 2, 3; stage s + 1 must be in LDS before its first read
            unpack_k<L, RE_LOW, U, F>(u0, r0);
            unpack_k<L, RE_LOW, U, F>(u1, r1);
            wait_stage_and_sync<L>();
            read_k<L>(r0, ring + nxt * L::SLOT, rl, 0);
            read_k<L>(r1, ring + nxt * L::SLOT, rl, 1);
            mfma_pair<L, DIAG>(acc, u0, u1);
            if constexpr (SUMS) {
                presum_k<L>(ps, u0);
                presum_k<L>(ps, u1);
            }
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
        }
        __builtin_amdgcn_s_waitcnt(XENG_VMCNT(0));
        __syncthreads();       // the next piece's DMA reuses the slots
    } else {
        {
            read_k<L>(r0, ring, rl, 0);
            read_k<L>(r1, ring, rl, 1);
            unpack_k<L, RE_LOW, U, F>(u0, r0);
        }
        int cur = 0;    // slot of stage s
        for (int s = 0; s < ns; ++s) {
            const int nxt = cur == L::NSLOT - 1 ? 0 : cur + 1;
            const int iss = cur == 0 ? L::NSLOT - 1 : cur - 1;   // slot of stage s - 1 = s + L::AHEAD
            issue_stage<L>(ring + iss * L::SLOT, tl, dl, s + L::AHEAD, wave, lane);
            __builtin_amdgcn_sched_barrier(0);
            // k-step 0
            read_k<L>(r0, ring + cur * L::SLOT, rl, 2);
            unpack_k<L, RE_LOW, U, F>(u1, r1);
            mfma_k<L, DIAG>(acc, u0);
            if constexpr (SUMS) presum_k<L>(ps, u0);
            kstep_schedule<L, DIAG>();
            __builtin_amdgcn_sched_barrier(0);
            // k-step 1
            read_k<L>(r1, ring + cur * L::SLOT, rl, 3);
            unpack_k<L, RE_LOW, U, F>(u0, r0);
            mfma_k<L, DIAG>(acc, u1);
            if constexpr (SUMS) presum_k<L>(ps, u1);
            kstep_schedule<L, DIAG>();
            __builtin_amdgcn_sched_barrier(0);
            // k-step 2: stage s + 1 must be in LDS before its first read
            wait_stage_and_sync<L>();
            read_k<L>(r0, ring + nxt * L::SLOT, rl, 0);
            unpack_k<L, RE_LOW, U, F>(u1, r1);
            mfma_k<L, DIAG>(acc, u0);
            if constexpr (SUMS) presum_k<L>(ps, u0);
            kstep_schedule<L, DIAG>();
            __builtin_amdgcn_sched_barrier(0);
            // k-step 3
            read_k<L>(r1, ring + nxt * L::SLOT, rl, 1);
            unpack_k<L, RE_LOW, U, F>(u0, r0);
            mfma_k<L, DIAG>(acc, u1);
            if constexpr (SUMS) presum_k<L>(ps, u1);
            kstep_schedule<L, DIAG>();
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
        }
        __builtin_amdgcn_s_waitcnt(XENG_VMCNT(0));
        __syncthreads();       // the next piece's DMA reuses the slots
    }
}

// A wave whose accumulator region lies wholly below the diagonal: its
// products would never be stored, so it computes nothing (which also spares
// the power that work would draw), but it keeps its share of the
// workgroup's DMA and passes the same barriers as run_piece.
template <typename L>
__device__ __forceinline__ void idle_piece(uint32_t ring, const Tile &tl, int wave, int lane)
{
    const int ns = L::TG == 1 ? (tl.t1 - tl.t0 + STAGE - 1) / STAGE : tl.ns;
    DmaLane<L> dl;
    dma_lane_setup<L>(dl, tl, wave, lane);
    __builtin_amdgcn_s_waitcnt(XENG_VMCNT(0));
#pragma unroll
    for (int d = 0; d < L::AHEAD; ++d) issue_stage<L>(ring + d * L::SLOT, tl, dl, d, wave, lane);
    wait_stage_and_sync<L>();
    int cur = 0;
    for (int s = 0; s < ns; ++s) {
        const int iss = cur == 0 ? L::NSLOT - 1 : cur - 1;
        issue_stage<L>(ring + iss * L::SLOT, tl, dl, s + L::AHEAD, wave, lane);
        wait_stage_and_sync<L>();
        cur = cur == L::NSLOT - 1 ? 0 : cur + 1;
    }
    __builtin_amdgcn_s_waitcnt(XENG_VMCNT(0));
    __syncthreads();
}

// Accumulators hold 256x the stored values (both operands carry 16x the
// sample parts), so a flush adds acc >> 8; every value is a multiple of
// 256, so this is exact.  Pairs go to the slot as packed 64-bit words (see
// the layout note): a tile shared with other pieces takes one 64-bit atomic
// add per pair.
//
// FP8 accumulators hold the integer sums x 2^-18 (each operand carries
// 2^-9), below 2^24 in magnitude: scaling by 2^18 recovers them exactly.
template <int SHIFT> __device__ __forceinline__ int32_t acc_val(int32_t v) { return v >> SHIFT; }
template <int SHIFT> __device__ __forceinline__ int32_t acc_val(float v) { return (int32_t)(v * 262144.0f); }

template <int SHIFT, typename V>
__device__ __forceinline__ void flush_atomic(gw64 *blk, const V &re, const V &im)
{
#pragma unroll
    for (int r = 0; r < 16; ++r)
        __hip_atomic_fetch_add(blk + r * 64, pack_pair(acc_val<SHIFT>(re[r]), acc_val<SHIFT>(im[r])),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The diagonal's stored imaginary parts (-S_j, see the top) of one wave's
// blocks on the diagonal of tile (ti, ti) into the slot's biases: one lane
// per input, whichever register holds its pair (j, j).
template <typename L, int SHIFT>
__device__ __forceinline__ void add_bias(int32_t *bias, const Acc<L, false> &acc, int n, int ti, int wa, int cb0,
                                         int lane, int a0, int a1)
{
    const int dr = diag_reg(lane);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (L::TG == 2 && (a < a0 || a >= a1)) continue;
        int32_t v = 0;
        if constexpr (L::BW == 2) {
            // a 64 x 64 region: its diagonal blocks are (0, 0) and (1, 1)
#pragma unroll
            for (int r = 0; r < 16; ++r) v = dr == r ? acc.im[a][a][r] : v;
        } else {
#pragma unroll
            for (int b = 0; b < L::BW; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) v = (cb0 + b == 2 * wa + a && dr == r) ? acc.im[a][b][r] : v;
        }
        const int j = WA_ROWS * ti + 64 * wa + 32 * a + (lane & 31);
        if (dr >= 0 && j < n)
            __hip_atomic_fetch_add(bias + j, acc_val<SHIFT>(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// A slot word, through the caches or past them (NT).
template <bool NT> __device__ __forceinline__ uint64_t load_word(const gw64 *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT> __device__ __forceinline__ void store_word(gw64 *p, uint64_t v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Whole-tile flush of one wave's 2 x BW blocks (column blocks cb0..): stores
// if the slot holds zeros, else read-modify-write with the loads of a row of
// blocks issued together (one memory latency per row, not one per value).
// NT: past the caches (JOB_STREAM; the four-wave kernel has no registers for
// a second form).  `b0`: the four-wave kernel's column blocks before it lie
// below the diagonal.
template <typename L, int SHIFT, bool F, bool NT>
__device__ __forceinline__ void flush_owned(gw64 *tb, const Acc<L, F> &acc, int wa, int cb0, bool fresh, int a0, int a1,
                                            int b0)
{
    constexpr int BW = L::BW;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (L::TG == 2 && (a < a0 || a >= a1)) continue;
        gw64 *blk[BW];
#pragma unroll
        for (int b = 0; b < BW; ++b) blk[b] = tb + ((2 * wa + a) * BLKS + cb0 + b) * BLOCK_W;
        uint64_t old[BW][16];
#pragma unroll
        for (int b = 0; b < BW; ++b) {
            if (BW == 4 && b < b0) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) old[b][r] = fresh ? 0 : load_word<NT>(blk[b] + r * 64);
        }
#pragma unroll
        for (int b = 0; b < BW; ++b) {
            if (BW == 4 && b < b0) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                store_word<NT>(blk[b] + r * 64, old[b][r] + pack_pair(acc_val<SHIFT>(acc.re[a][b][r]),
                                                                      acc_val<SHIFT>(acc.im[a][b][r])));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Two time groups: the two waves of a region exchange half of their sums
// through LDS (`mine`, `other`: 16 KiB each of the ring, which the end of a
// piece has left free), wave KEEP of the pair ending with the sums of both
// over row block KEEP of the region.
template <typename L, int KEEP>
__device__ __forceinline__ void give_half(uint8_t *mine, const Acc<L, false> &acc, int lane)
{
#pragma unroll
    for (int b = 0; b < L::BW; ++b)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const auto &v = q < 4 ? acc.re[1 - KEEP][b] : acc.im[1 - KEEP][b];
            const int r = 4 * (q & 3);
            *reinterpret_cast<v4i *>(mine + ((b * 8 + q) * 64 + lane) * 16) =
                v4i{v[r], v[r + 1], v[r + 2], v[r + 3]};
        }
}
template <typename L, int KEEP>
__device__ __forceinline__ void take_half(const uint8_t *other, Acc<L, false> &acc, int lane)
{
#pragma unroll
    for (int b = 0; b < L::BW; ++b)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const v4i w = *reinterpret_cast<const v4i *>(other + ((b * 8 + q) * 64 + lane) * 16);
            auto &v = q < 4 ? acc.re[KEEP][b] : acc.im[KEEP][b];
            const int r = 4 * (q & 3);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[r + k] += w[k];
        }
}

// Persistent kernels: workgroup w runs pieces [wg_off[w], wg_off[w+1]).  A
// piece's tile field holds (I, J): A rows 128 I.., B columns from 128 L::TILES J,
// i.e. accumulator tiles (I, L::TILES J ..) where they are in the upper
// triangle.  U: the unsigned form; F (with U): its FP8 products.
template <typename L, bool U, bool F>
__device__ __forceinline__ void run_workgroup(const KernelArgs &args)
{
    static_assert(U || !F, "the FP8 form multiplies the unsigned nibbles");
    static_assert(L::TG == 1 || !U, "two time groups: the signed form only");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    // a prepared batch's device guard refused this launch
    if (args.skip != nullptr && *args.skip != 0) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // wave-uniform, so that everything derived from it stays scalar
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the wave's time group, and its place among the group's waves
    constexpr int GW = L::NW / L::TG;
    const int tg = L::TG == 1 ? 0 : wave / GW, gw = L::TG == 1 ? wave : wave % GW;
    // LDS byte address of the time group's part of the ring, wave-uniform
    // (scalar register)
    const uint32_t ring = (uint32_t)__builtin_amdgcn_readfirstlane(
                              (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds) +
                          tg * L::GROUP;
    // clock probe (measurement only): workgroup 0's start and end
    const bool stamp = args.clock != nullptr && blockIdx.x == 0 && tid == 0;
    if (stamp) {
        args.clock[0] = (int64_t)__builtin_amdgcn_s_memtime();
        args.clock[1] = (int64_t)__builtin_amdgcn_s_memrealtime();
    }
    const int p_begin = args.wg_off[blockIdx.x], p_end = args.wg_off[blockIdx.x + 1];
    for (int pi = p_begin; pi < p_end; ++pi) {
        const Piece pce = args.pieces[pi];
        JobDesc jd = args.jobs ? args.jobs[pce.job] : args.job0;
        // every field is wave-uniform: keep them in scalar registers
        jd.acc = uniform(jd.acc);
        jd.bias = uniform(jd.bias);
        jd.presum = uniform(jd.presum);
        jd.n = __builtin_amdgcn_readfirstlane(jd.n);
        jd.nt = __builtin_amdgcn_readfirstlane(jd.nt);
        jd.flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)jd.flags);
        const int tile = __builtin_amdgcn_readfirstlane(pce.tile);
        const int ti = tile & 0xFFFF, tj0 = L::TILES * ((tile >> 16) & 0xFFFF);
        const bool atomic = __builtin_amdgcn_readfirstlane(pce.t1_atomic) < 0;
        Tile tl;
        tl.samples = uniform(jd.samples);
        tl.zeros = uniform(args.zeros);
        tl.stride = uniform(jd.stride);
        tl.n = jd.n;
        tl.row0 = __builtin_amdgcn_readfirstlane(ti * WA_ROWS);
        tl.col0 = __builtin_amdgcn_readfirstlane(tj0 * TILE);
        const int t0 = __builtin_amdgcn_readfirstlane(pce.t0);
        tl.t0 = t0 + STAGE * tg;
        tl.t1 = __builtin_amdgcn_readfirstlane(pce.t1_atomic & 0x7FFFFFFF);
        tl.ns = (tl.t1 - t0 + L::ROWS - 1) / L::ROWS;
        // this wave's region: rows 64 wa.. of the A block against column
        // blocks of the B block.  The waves of a workgroup run on SIMD
        // wave % 4.  Where one tile of the window is not in the triangle
        // (below the diagonal: the window of an odd tile row that starts one
        // tile left of it; or past the last tile column), four of the eight
        // regions have no work; the region map then puts the other four on
        // four different SIMDs instead of two waves each on two of them,
        // halving the matrix time of such a window's stages.
        int wa = gw / L::WB_WAVES, wb = gw % L::WB_WAVES;
        if constexpr (L::NW == 8 && L::TILES == 2) {
            const bool vl = tj0 >= ti && tj0 < jd.nt, vr = tj0 + 1 >= ti && tj0 + 1 < jd.nt;
            if (vr && !vl && wa == 0) wb ^= 2;
            if (vl && !vr && wa == 1) wb ^= 2;
        }
        ReadLane<L> rl;
        read_lane_setup<L>(rl, 4 * wa, 2 * L::BW * wb, A_STAGE, lane);
        // this wave's accumulator tile; a region wholly below the diagonal
        // is neither computed nor stored (the wave stays in step for the
        // workgroup's DMA and barriers)
        constexpr int PER_TILE = L::WB_WAVES / L::TILES;   // waves across a tile
        const int tj = tj0 + wb / PER_TILE;
        const int cb0 = (wb % PER_TILE) * L::BW;   // first column block in the tile
        const bool valid = tj >= ti && tj < jd.nt;
        // rows 64 wa.. of tile ti against columns 32 cb0 .. 32 (cb0 + BW) - 1
        // of tile tj: wholly below the diagonal?
        const bool below = WA_ROWS * (tj - ti) + BLK * (cb0 + L::BW) <= 64 * wa;
        // or wholly past the last input (rows or columns >= N: never
        // exported; small N and the edge tiles of N not a multiple of 256)
        const bool outside = WA_ROWS * ti + 64 * wa >= jd.n || WA_ROWS * tj + BLK * cb0 >= jd.n;

        Acc<L, F> acc;
        PreSum ps = {{0u, 0u}, {0u, 0u}};
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < L::BW; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc.re[a][b][r] = 0;
                    acc.im[a][b][r] = 0;
                }
        // a 64 x 64 region on the diagonal skips its block below it
        const bool diag = L::BW == 2 && tj == ti && cb0 == 2 * wa;
        // a wave whose tile lies past the last tile column (odd tile count)
        // has nothing to compute either
        if (below || outside || tj >= jd.nt)
            idle_piece<L>(ring, tl, wave, lane);
        else if (jd.flags & JOB_RE_LOW) {
            if (diag)
                run_piece<L, true, true, U, F>(acc, ps, ring, tl, wave, lane, rl);
            else
                run_piece<L, true, false, U, F>(acc, ps, ring, tl, wave, lane, rl);
        } else {
            if (diag)
                run_piece<L, false, true, U, F>(acc, ps, ring, tl, wave, lane, rl);
            else
                run_piece<L, false, false, U, F>(acc, ps, ring, tl, wave, lane, rl);
        }

        // unsigned form: the diagonal waves of a job's tiles see every A
        // row of the job over every sample exactly once (each window's
        // pieces split its samples; a diagonal wave is never idle while its
        // rows hold inputs), so their nibble sums are the job's pre-sums;
        // lanes l and l + 32 hold the same row
        if constexpr (U) {
            int32_t *const presum = args.presum != nullptr ? args.presum : jd.presum;
            if (diag && presum != nullptr && !outside) {
                const int n4 = (jd.n + 3) & ~3;
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const uint32_t r = ps.r[a] + (uint32_t)__shfl_xor((int)ps.r[a], 32);
                    const uint32_t i = ps.i[a] + (uint32_t)__shfl_xor((int)ps.i[a], 32);
                    const int row = WA_ROWS * ti + 64 * wa + 32 * a + lane;
                    if (lane < 32 && row < jd.n) {
                        __hip_atomic_fetch_add(presum + row, (int32_t)r, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                        __hip_atomic_fetch_add(presum + n4 + row, (int32_t)i, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        }

        const bool work = valid && !below && !outside;
        int a0 = 0, a1 = 2;   // row blocks of the region this wave flushes
        if constexpr (L::TG == 2) {
            uint8_t *mine = lds + wave * 16384;
            const uint8_t *other = lds + ((wave + GW) % L::NW) * 16384;
            if (work) {
                if (tg == 0) give_half<L, 0>(mine, acc, lane);
                else give_half<L, 1>(mine, acc, lane);
            }
            __syncthreads();
            if (work) {
                if (tg == 0) take_half<L, 0>(other, acc, lane);
                else take_half<L, 1>(other, acc, lane);
            }
            __syncthreads();   // the next piece's DMA reuses the ring
            a0 = tg;
            a1 = tg + 1;
        }
        if (work) {
            // the sums carry 256x the values (both operands 16x), or 8x in
            // the unsigned form (the FP8 form's scale is undone in acc_val)
            constexpr int SHIFT = U ? 3 : 8;
            // the unsigned form carries no bias
            if constexpr (!U)
                if (tj == ti && (L::BW == 4 || diag) && jd.bias != nullptr)
                    add_bias<L, SHIFT>(jd.bias, acc, jd.n, ti, wa, cb0, lane, a0, a1);
            const int64_t tile_idx = (int64_t)ti * jd.nt - (int64_t)ti * (ti - 1) / 2 + (tj - ti);
            gw64 *tb = (gw64 *)(jd.acc + tile_idx * TILE_I32) + lane;
            // blocks below the diagonal of a wave that has both are not
            // stored (their words hold the slot's bias bases, see BASE_I32)
            const int b0 = L::BW == 4 && tj == ti ? 2 * wa : 0;
            if (atomic) {
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < L::BW; ++b) {
                        if (L::TG == 2 && (a < a0 || a >= a1)) continue;
                        if (diag && a == 1 && b == 0) continue;   // below the diagonal, never computed
                        if (L::BW == 4 && b < b0) continue;
                        flush_atomic<SHIFT>(tb + ((2 * wa + a) * BLKS + cb0 + b) * BLOCK_W, acc.re[a][b],
                                            acc.im[a][b]);
                        // one block at a time: keeps the register file for the main loop
                        __builtin_amdgcn_sched_barrier(0);
                    }
            } else if (L::NW == 8 && (jd.flags & JOB_STREAM)) {
                if (jd.flags & JOB_FRESH) flush_owned<L, SHIFT, F, true>(tb, acc, wa, cb0, true, a0, a1, b0);
                else flush_owned<L, SHIFT, F, true>(tb, acc, wa, cb0, false, a0, a1, b0);
            } else if (jd.flags & JOB_FRESH) {
                flush_owned<L, SHIFT, F, false>(tb, acc, wa, cb0, true, a0, a1, b0);
            } else {
                flush_owned<L, SHIFT, F, false>(tb, acc, wa, cb0, false, a0, a1, b0);
            }
        }
    }
    if (stamp) {
        args.clock[2] = (int64_t)__builtin_amdgcn_s_memtime();
        args.clock[3] = (int64_t)__builtin_amdgcn_s_memrealtime();
    }
}

template <int NW, bool U = false, bool F = false>
__global__ __launch_bounds__(64 * NW, 1) void xcorr_dma(KernelArgs args)
{
    run_workgroup<Layout<NW>, U, F>(args);
}

// The tile kernel: 128 x 128 tiles, each quarter's time split over two waves.
__global__ __launch_bounds__(64 * TileLayout::NW, 1) void xcorr_tile(KernelArgs args)
{
    run_workgroup<TileLayout, false, false>(args);
}

}  // namespace dma

constexpr int DMA_LDS_BYTES = dma::Layout<8>::LDS_BYTES;

// Both instances are built: eight waves (two per SIMD, so one wave's
// unpack overlaps the other's matrix work) and four (one per SIMD, four
// column blocks each, fewer transposed reads per multiply).  The launch
// configuration picks one per call.
//
// Once per device, before any launch (and outside any stream capture): the
// kernel's LDS ring exceeds the default dynamic-LDS limit.
hipError_t init_dma_kernel()
{
    hipError_t e = hipFuncSetAttribute((const void *)dma::xcorr_dma<8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       DMA_LDS_BYTES);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)dma::xcorr_dma<4>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                DMA_LDS_BYTES);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)dma::xcorr_dma<8, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                DMA_LDS_BYTES);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)dma::xcorr_dma<8, true, true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, DMA_LDS_BYTES);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)dma::xcorr_tile, hipFuncAttributeMaxDynamicSharedMemorySize,
                                dma::TileLayout::LDS_BYTES);
    return e;
}

hipError_t launch_correlate_tile(const KernelArgs &a, int grid, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(dma::xcorr_tile, dim3(grid), dim3(64 * dma::TileLayout::NW), dma::TileLayout::LDS_BYTES, stream, a);
    return hipGetLastError();
}

// The unsigned form (pre-sum path): eight waves, int8 or (fp8) FP8
// products; `a.zeros` must then point at zero bytes (nibbles u = 0), the
// zero sample of that form.  FP8 pieces must stay within
// MAX_PIECE_STAGES_FP8_UNSIGNED stages.
hipError_t launch_correlate_dma_unsigned(const KernelArgs &a, int grid, bool fp8, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    if (fp8)
        hipLaunchKernelGGL((dma::xcorr_dma<8, true, true>), dim3(grid), dim3(64 * 8), DMA_LDS_BYTES, stream, a);
    else
        hipLaunchKernelGGL((dma::xcorr_dma<8, true>), dim3(grid), dim3(64 * 8), DMA_LDS_BYTES, stream, a);
    return hipGetLastError();
}

hipError_t launch_correlate_dma(const KernelArgs &a, int grid, int waves, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    if (waves == 4)
        hipLaunchKernelGGL(dma::xcorr_dma<4>, dim3(grid), dim3(64 * 4), DMA_LDS_BYTES, stream, a);
    else
        hipLaunchKernelGGL(dma::xcorr_dma<8>, dim3(grid), dim3(64 * 8), DMA_LDS_BYTES, stream, a);
    return hipGetLastError();
}

}  // namespace xeng
