// Device code shared by the kernels that stage packed samples by LDS DMA
// (the wide, tile and region kernels): LDS DMA, transposed LDS reads, the
// nibble unpack and the MFMAs of a k-step.  `L` is the kernel's shape: it
// gives PITCH_A, PITCH_B (bytes per time row of its A and B sides in LDS),
// BW (B blocks per wave) and the instruction mix of a k-step.
#pragma once

#include <hip/hip_runtime.h>

#include "xeng_internal.h"

namespace xeng {
namespace dma {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) v2i lds_v2i;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(1))) uint64_t gw64;

// s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, expcnt 6:4 and
// lgkmcnt 11:8 at their maxima (no wait on those); and lgkmcnt(0) alone.
#define XENG_VMCNT(n) (((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
#define XENG_LGKMCNT0 (0xF | (0x3 << 14) | (0x7 << 4))

// A wave-uniform 64-bit value moved to scalar registers.
template <typename T> __device__ __forceinline__ T uniform(T v)
{
    static_assert(sizeof(T) == 8, "64-bit values only");
    uint64_t u;
    __builtin_memcpy(&u, &v, 8);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)u);
    u = ((uint64_t)hi << 32) | lo;
    __builtin_memcpy(&v, &u, 8);
    return v;
}

// 16-byte-per-lane DMAs into LDS at byte address `lds_addr` + 16 * lane,
// written as inline assembly so that the compiler, which cannot tell that
// reads of other ring slots never alias the slot being filled, does not
// drain every load in flight before each LDS read; the ring's own vmcnt
// waits order the accesses.  The instructions have no register result; M0
// (their LDS base) is saved and restored around them.  Wait states: one
// between an SALU write of M0 and the DMA; five between a VALU write of an
// SGPR (readfirstlane) and a memory instruction that reads it as its base.
// (readfirstlane is a no-op on values already in scalar registers; it
// returns a signed int, so each half of a pointer is widened as unsigned.)
//
// Vector-address form: a 64-bit address per lane.
__device__ __forceinline__ void dma16_v(const uint8_t *addr, uint32_t lds_addr)
{
    const uint32_t sl = (uint32_t)__builtin_amdgcn_readfirstlane(lds_addr);
    uint32_t saved;
    asm volatile("s_mov_b32 %0, m0\n\t"
                 "s_mov_b32 m0, %2\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, off\n\t"
                 "s_mov_b32 m0, %0"
                 : "=&s"(saved)
                 : "v"(addr), "s"(sl)
                 : "memory");
}

// Scalar-base form, wave-uniform 64-bit base + per-lane 32-bit offsets: a
// whole stage's share of DMAs (K of them) in one statement:
// M0 saved once, one s_nop 4 ahead of the first instruction (covering a
// VALU write of any SGPR operand, which the statement's own instructions
// never make), and between instructions only the one wait state an SALU
// write of M0 needs before an LDS DMA.
template <int K>
__device__ __forceinline__ void dma16_s_stage(const uint8_t *base, const uint32_t (&lane_off)[K],
                                              const uint32_t (&lds_addr)[K])
{
    static_assert(K == 6 || K == 4 || K == 2, "6, 4 or 2 instructions per wave");
    const uint64_t b = (uint64_t)(uintptr_t)base;
    const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint64_t sb = ((uint64_t)b_hi << 32) | (uint64_t)b_lo;
    uint32_t sl[K];
#pragma unroll
    for (int k = 0; k < K; ++k) sl[k] = (uint32_t)__builtin_amdgcn_readfirstlane(lds_addr[k]);
    uint32_t saved;
    if constexpr (K == 6) {
        asm volatile("s_mov_b32 %0, m0\n\t"
                     "s_mov_b32 m0, %8\n\t"
                     "s_nop 4\n\t"
                     "global_load_lds_dwordx4 %1, %7\n\t"
                     "s_mov_b32 m0, %9\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %7\n\t"
                     "s_mov_b32 m0, %10\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %3, %7\n\t"
                     "s_mov_b32 m0, %11\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %4, %7\n\t"
                     "s_mov_b32 m0, %12\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %5, %7\n\t"
                     "s_mov_b32 m0, %13\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %6, %7\n\t"
                     "s_mov_b32 m0, %0"
                     : "=&s"(saved)
                     : "v"(lane_off[0]), "v"(lane_off[1]), "v"(lane_off[2]), "v"(lane_off[3]),
                       "v"(lane_off[4]), "v"(lane_off[5]), "s"(sb), "s"(sl[0]), "s"(sl[1]), "s"(sl[2]),
                       "s"(sl[3]), "s"(sl[4]), "s"(sl[5])
                     : "memory");
    } else if constexpr (K == 2) {
        asm volatile("s_mov_b32 %0, m0\n\t"
                     "s_mov_b32 m0, %4\n\t"
                     "s_nop 4\n\t"
                     "global_load_lds_dwordx4 %1, %3\n\t"
                     "s_mov_b32 m0, %5\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %3\n\t"
                     "s_mov_b32 m0, %0"
                     : "=&s"(saved)
                     : "v"(lane_off[0]), "v"(lane_off[1]), "s"(sb), "s"(sl[0]), "s"(sl[1])
                     : "memory");
    } else {
        asm volatile("s_mov_b32 %0, m0\n\t"
                     "s_mov_b32 m0, %6\n\t"
                     "s_nop 4\n\t"
                     "global_load_lds_dwordx4 %1, %5\n\t"
                     "s_mov_b32 m0, %7\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %5\n\t"
                     "s_mov_b32 m0, %8\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %3, %5\n\t"
                     "s_mov_b32 m0, %9\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %4, %5\n\t"
                     "s_mov_b32 m0, %0"
                     : "=&s"(saved)
                     : "v"(lane_off[0]), "v"(lane_off[1]), "v"(lane_off[2]), "v"(lane_off[3]), "s"(sb), "s"(sl[0]),
                       "s"(sl[1]), "s"(sl[2]), "s"(sl[3])
                     : "memory");
    }
}

// Packed operand data of one k-step (2 A blocks, BW B blocks) and its
// unpacked form.
template <typename L> struct Raw {
    v2i a[2];
    v2i b[L::BW];
};
template <typename L> struct Ops {
    v8i a[2];   // {16R, 16R, 16I, 16I, 16~R, 16~R, -, -}: real A = s0123, imaginary A = s2345
    v4i b[L::BW];   // {16R, 16R, 16I, 16I}
};
template <typename L, bool F> struct Acc {
    v16i re[2][L::BW];
    v16i im[2][L::BW];
};
template <typename L> struct Acc<L, true> {
    v16f re[2][L::BW];
    v16f im[2][L::BW];
};

// LDS layout of a side (A or B region) of a stage: row-major, `PITCH` bytes
// (one per input) per time row, the 16-byte chunk c of row r at chunk
// position c ^ swizzle(r).  Consecutive lanes of a DMA instruction then fill
// consecutive chunks of a row, so that they read whole cache lines from
// memory; and the 8 rows x 2 chunks that 32 lanes of a transposed read touch
// sit in 16 different 16-byte bank groups.
template <int PITCH> __device__ __forceinline__ constexpr int swizzle(int row)
{
    return 2 * ((row & 7) / (256 / PITCH));
}

// A 1 KB DMA instruction covers 1024 / PITCH rows: this lane's row among
// them, and the chunk it fetches when the first of them is row `first`.
template <int PITCH> __device__ __forceinline__ int dma_row(int lane) { return lane / (PITCH / 16); }
template <int PITCH> __device__ __forceinline__ int dma_chunk(int first, int lane)
{
    return (lane % (PITCH / 16)) ^ swizzle<PITCH>(first + dma_row<PITCH>(lane));
}

// This lane's byte offset in a side for the transposed reads of the 32
// inputs that start at chunk `chunk` (even): its 16-lane group reads 8 time
// rows (the first or second 8 of a k-step's 16) of 16 inputs, lane l % 16
// of the group supplying bytes 8 (l % 2) .. of row (l % 16) / 2.
template <int PITCH> __device__ __forceinline__ uint32_t read_offset(int chunk, int lane)
{
    const int grp = lane >> 4, jl = lane & 15, r = jl >> 1;
    return (uint32_t)(PITCH * (8 * (grp >> 1) + r) + 16 * ((chunk + (grp & 1)) ^ swizzle<PITCH>(r)) + 8 * (jl & 1));
}

// A wave's read offsets in a stage slot: its A blocks start at chunk `ca`, its
// B blocks at chunk `cb` of the side that starts at byte `b_side`.
// (With four B blocks only the first's offset is kept: chunks cb, cb + 2, ..
// of an aligned group of eight differ in two bits, which the swizzle's XOR
// carries over to the offset.)
template <typename L> struct ReadLane {
    uint32_t a[2], b[L::BW == 2 ? 2 : 1];
};
template <typename L>
__device__ __forceinline__ void read_lane_setup(ReadLane<L> &rl, int ca, int cb, int b_side, int lane)
{
#pragma unroll
    for (int k = 0; k < 2; ++k) rl.a[k] = read_offset<L::PITCH_A>(ca + 2 * k, lane);
#pragma unroll
    for (int k = 0; k < (L::BW == 2 ? 2 : 1); ++k) rl.b[k] = b_side + read_offset<L::PITCH_B>(cb + 2 * k, lane);
}

// Transposed reads of k-step q of the stage in `slot` (LDS byte address).
template <typename L>
__device__ __forceinline__ void read_k(Raw<L> &r, uint32_t slot, const ReadLane<L> &rl, int q)
{
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const lds_u8 *p = (const lds_u8 *)(uintptr_t)(slot + rl.a[a]);
        r.a[a] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(p + 16 * L::PITCH_A * q));
    }
#pragma unroll
    for (int b = 0; b < L::BW; ++b) {
        const uint32_t off = L::BW == 2 ? rl.b[b] : rl.b[0] ^ (32u * b);
        const lds_u8 *p = (const lds_u8 *)(uintptr_t)(slot + off);
        r.b[b] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i *)(p + 16 * L::PITCH_B * q));
    }
}

// 16 x (4-bit value) in the high half of each byte: from the high nibbles,
// (p ^ 0x88) & 0xF0 per byte; from the low nibbles, the same on p << 4.
// XOR with 0x77 instead of 0x88 gives 16 x the bitwise complement.
//
// Unsigned form (U): the stored nibbles u in 0..15 themselves, no offset
// removed -- A real [uR | uI], A imaginary [uI | -uR] (per byte
// (0x80 - u) ^ 0x80: no borrows), B [8 uR | 8 uI] (at most 120) -- so the
// sums are 8 x the exact products of the stored values, with no bias.
//
// FP8 form (F, unsigned): a byte holding u in 0..15 is the OCP E4M3 code of
// u x 2^-9 (codes 0..7 are the subnormals m x 2^-9, codes 8..15 the first
// binade (8 + m) x 2^-9), and setting its top bit negates it exactly.  So A
// real [uR | uI], A imaginary [uI | -uR] and B [uR | uI] are the masked
// nibbles themselves (and the sign bit), and the fp32 sums hold the exact
// integer sums x 2^-18.
template <typename L, bool RE_LOW, bool U, bool F>
__device__ __forceinline__ void unpack_k(Ops<L> &o, const Raw<L> &r)
{
    if constexpr (F) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const uint32_t x0 = (uint32_t)r.a[a].x, x1 = (uint32_t)r.a[a].y;
            const uint32_t h0 = (x0 >> 4) & 0x0F0F0F0Fu, h1 = (x1 >> 4) & 0x0F0F0F0Fu;
            const uint32_t l0 = x0 & 0x0F0F0F0Fu, l1 = x1 & 0x0F0F0F0Fu;
            const uint32_t re0 = RE_LOW ? l0 : h0, re1 = RE_LOW ? l1 : h1;
            const uint32_t im0 = RE_LOW ? h0 : l0, im1 = RE_LOW ? h1 : l1;
            o.a[a] = v8i{(int)re0, (int)re1, (int)im0, (int)im1, (int)(re0 | 0x80808080u), (int)(re1 | 0x80808080u),
                         0, 0};
        }
#pragma unroll
        for (int b = 0; b < L::BW; ++b) {
            const uint32_t x0 = (uint32_t)r.b[b].x, x1 = (uint32_t)r.b[b].y;
            const uint32_t h0 = (x0 >> 4) & 0x0F0F0F0Fu, h1 = (x1 >> 4) & 0x0F0F0F0Fu;
            const uint32_t l0 = x0 & 0x0F0F0F0Fu, l1 = x1 & 0x0F0F0F0Fu;
            o.b[b] = RE_LOW ? v4i{(int)l0, (int)l1, (int)h0, (int)h1} : v4i{(int)h0, (int)h1, (int)l0, (int)l1};
        }
        return;
    }
    if constexpr (U) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const uint32_t x0 = (uint32_t)r.a[a].x, x1 = (uint32_t)r.a[a].y;
            const uint32_t h0 = (x0 >> 4) & 0x0F0F0F0Fu, h1 = (x1 >> 4) & 0x0F0F0F0Fu;
            const uint32_t l0 = x0 & 0x0F0F0F0Fu, l1 = x1 & 0x0F0F0F0Fu;
            const uint32_t re0 = RE_LOW ? l0 : h0, re1 = RE_LOW ? l1 : h1;
            const uint32_t im0 = RE_LOW ? h0 : l0, im1 = RE_LOW ? h1 : l1;
            const uint32_t n0 = (0x80808080u - re0) ^ 0x80808080u, n1 = (0x80808080u - re1) ^ 0x80808080u;
            o.a[a] = v8i{(int)re0, (int)re1, (int)im0, (int)im1, (int)n0, (int)n1, 0, 0};
        }
#pragma unroll
        for (int b = 0; b < L::BW; ++b) {
            const uint32_t x0 = (uint32_t)r.b[b].x, x1 = (uint32_t)r.b[b].y;
            const uint32_t h0 = (x0 >> 1) & 0x78787878u, h1 = (x1 >> 1) & 0x78787878u;   // 8 x high nibble
            const uint32_t l0 = (x0 << 3) & 0x78787878u, l1 = (x1 << 3) & 0x78787878u;   // 8 x low nibble
            o.b[b] = RE_LOW ? v4i{(int)l0, (int)l1, (int)h0, (int)h1} : v4i{(int)h0, (int)h1, (int)l0, (int)l1};
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const uint32_t x0 = (uint32_t)r.a[a].x, x1 = (uint32_t)r.a[a].y;
        const uint32_t s0 = x0 << 4, s1 = x1 << 4;
        const uint32_t h0 = (x0 ^ 0x88888888u) & 0xF0F0F0F0u, h1 = (x1 ^ 0x88888888u) & 0xF0F0F0F0u;
        const uint32_t l0 = (s0 ^ 0x80808080u) & 0xF0F0F0F0u, l1 = (s1 ^ 0x80808080u) & 0xF0F0F0F0u;
        if (RE_LOW) {
            const uint32_t n0 = (s0 ^ 0x70707070u) & 0xF0F0F0F0u, n1 = (s1 ^ 0x70707070u) & 0xF0F0F0F0u;
            o.a[a] = v8i{(int)l0, (int)l1, (int)h0, (int)h1, (int)n0, (int)n1, 0, 0};
        } else {
            const uint32_t n0 = (x0 ^ 0x77777777u) & 0xF0F0F0F0u, n1 = (x1 ^ 0x77777777u) & 0xF0F0F0F0u;
            o.a[a] = v8i{(int)h0, (int)h1, (int)l0, (int)l1, (int)n0, (int)n1, 0, 0};
        }
    }
#pragma unroll
    for (int b = 0; b < L::BW; ++b) {
        const uint32_t x0 = (uint32_t)r.b[b].x, x1 = (uint32_t)r.b[b].y;
        const uint32_t h0 = (x0 ^ 0x88888888u) & 0xF0F0F0F0u, h1 = (x1 ^ 0x88888888u) & 0xF0F0F0F0u;
        const uint32_t l0 = ((x0 << 4) ^ 0x80808080u) & 0xF0F0F0F0u;
        const uint32_t l1 = ((x1 << 4) ^ 0x80808080u) & 0xF0F0F0F0u;
        o.b[b] = RE_LOW ? v4i{(int)l0, (int)l1, (int)h0, (int)h1} : v4i{(int)h0, (int)h1, (int)l0, (int)l1};
    }
}

// Pre-sums of the unsigned form from the operands a wave multiplies: per A
// block, this lane's row (lane % 32) over the k-step's samples it holds,
// real nibbles (words 0, 1) and imaginary ones (words 2, 3), each a byte
// sum by v_dot4_u32_u8 against ones.
struct PreSum {
    uint32_t r[2], i[2];
};
template <typename L> __device__ __forceinline__ void presum_k(PreSum &ps, const Ops<L> &o)
{
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        ps.r[a] = __builtin_amdgcn_udot4((uint32_t)o.a[a][0], 0x01010101u, ps.r[a], false);
        ps.r[a] = __builtin_amdgcn_udot4((uint32_t)o.a[a][1], 0x01010101u, ps.r[a], false);
        ps.i[a] = __builtin_amdgcn_udot4((uint32_t)o.a[a][2], 0x01010101u, ps.i[a], false);
        ps.i[a] = __builtin_amdgcn_udot4((uint32_t)o.a[a][3], 0x01010101u, ps.i[a], false);
    }
}

// DIAG: the wave's 2 x 2 blocks sit on the diagonal (eight waves, rows
// 64 wa.. against columns 64 wa.. of a diagonal tile); block (1, 0) lies
// strictly below it and is skipped.
template <typename L, bool DIAG> __device__ __forceinline__ constexpr bool skip_block(int a, int b)
{
    return DIAG && a == 1 && b == 0;
}

// The real products of a k-step first, then the imaginary ones: measured a
// little faster than alternating them (the chip runs at its power limit, and
// this order drew less).
//
// FP8 form: the products of two k-steps at once on
// v_mfma_f32_32x32x64_f8f6f4 (E4M3 on both sides, no block scale), whose
// 32-byte operands are the two k-steps' unpacked words side by side: real
// [R | I | R' | I'] . [R | I | R' | I'], imaginary [I | -R | I' | -R'] .
// [R | I | R' | I'].  All real products of the pair first, then the
// imaginary ones, so that no product waits for the one before it.
template <typename L, bool DIAG>
__device__ __forceinline__ void mfma_pair(Acc<L, true> &acc, const Ops<L> &o0, const Ops<L> &o1)
{
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int b = 0; b < L::BW; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (skip_block<L, DIAG>(a, b)) continue;
                const int w = 2 * p;   // real: words 0..3, imaginary: words 2..5
                const v8i av = {o0.a[a][w], o0.a[a][w + 1], o0.a[a][w + 2], o0.a[a][w + 3],
                                o1.a[a][w], o1.a[a][w + 1], o1.a[a][w + 2], o1.a[a][w + 3]};
                const v8i bv = {o0.b[b][0], o0.b[b][1], o0.b[b][2], o0.b[b][3],
                                o1.b[b][0], o1.b[b][1], o1.b[b][2], o1.b[b][3]};
                v16f &c = p == 0 ? acc.re[a][b] : acc.im[a][b];
                c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 0, 0, 0, 0, 0, 0);
            }
}

template <typename L, bool DIAG>
__device__ __forceinline__ void mfma_k(Acc<L, false> &acc, const Ops<L> &o)
{
#pragma unroll
    for (int b = 0; b < L::BW; ++b)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if (skip_block<L, DIAG>(a, b)) continue;
            const v4i re_a = __builtin_shufflevector(o.a[a], o.a[a], 0, 1, 2, 3);
            acc.re[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(re_a, o.b[b], acc.re[a][b], 0, 0, 0);
        }
#pragma unroll
    for (int b = 0; b < L::BW; ++b)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if (skip_block<L, DIAG>(a, b)) continue;
            const v4i im_a = __builtin_shufflevector(o.a[a], o.a[a], 2, 3, 4, 5);
            acc.im[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(im_a, o.b[b], acc.im[a][b], 0, 0, 0);
        }
}

// Instruction order of a k-step: the MFMAs, each followed by a share of the
// unpack of the next k-step (which the matrix core's 32-cycle MFMAs hide)
// and, after the first few, one of the LDS reads of a later k-step -- spread
// out rather than issued as a burst that would stall the wave at issue.
template <typename L, bool DIAG>
__device__ __forceinline__ void kstep_schedule()
{
    constexpr int MFMAS = L::MFMA_PER_K - (DIAG ? 2 : 0);
    constexpr int VALU = DIAG ? (L::VALU_PER_MFMA * L::MFMA_PER_K + MFMAS - 1) / MFMAS : L::VALU_PER_MFMA;
#pragma unroll
    for (int m = 0; m < MFMAS; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        if (m < L::READS_PER_K) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read
        __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);   // VALU
    }
}

}  // namespace dma
}  // namespace xeng
